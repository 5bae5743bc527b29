// Word map of the host blob of an index, shared by the export and import entry points and their kernels.
#pragma once

#include "lc_internal.h"

struct LcBlobMap {
    int32_t hdr[16];            // the blob's header
    unsigned long long nodes;   // first word of the node records (behind the sequence records and boundaries)
    unsigned long long total;   // words of the blob
};

// The kernels find a word's place with a table of one row per sequence: {first word of the sequence's
// record, first word of its nodes, T, M, N_1, ..., N_{L-1}}.
__host__ __device__ inline int lc_blob_row(int L) { return 3 + L; }

// Move words [w0, w0 + n) of the blob between the index and a pinned host window.
int lc_launch_blob_export(const LcDev& ix, const LcBlobMap& m, const long long* table, unsigned long long w0, unsigned n,
                          uint32_t* window, hipStream_t stream);
int lc_launch_blob_import(const LcDev& ix, const LcBlobMap& m, const long long* table, unsigned long long w0, unsigned n,
                          const uint32_t* window, hipStream_t stream);
