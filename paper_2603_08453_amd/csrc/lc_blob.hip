// The flat host blob of an index (lychee.h: lc_index_export / lc_index_import), written and read by one
// kernel per window instead of one blocking copy per array.
//
// A blob is a few MB cut into thousands of small arrays (five per level, head and sequence): as single
// copies it costs a round trip to the device each (32K tokens, 8 heads, 3 levels: 242 copies, 3.6 ms for
// 2 MB out and in).  Here the kernel maps every 32-bit word of the blob to its place in the index by
// arithmetic and moves it from or to a pinned host window; the host copies windows while the next one
// is in flight.  What bounds it then is the host's own copy between the blob and the window.
#include "lc_blob.h"

#include "lc_device.h"

namespace {

constexpr int LC_BLOB_THREADS = 256;
constexpr int LC_BLOB_WORDS = 8;              // words per thread: all in flight together (a read of host memory takes microseconds)
constexpr int LC_BLOB_LDS_ROWS = 4096;        // sequence table entries kept in LDS

// Where word w of the blob lives in the index.
struct Place {
    uint32_t* word;          // 32-bit place, or null
    uint32_t* also;          // second place of the word on import (the radius at build time), or null
    uint16_t* half;          // bfloat16 place, or null
    uint32_t value;          // neither: a constant of the header or of a sequence's record
};

// U: unsigned, or a 64-bit integer for blobs of 2^32 words and more.
template <typename U>
__device__ __forceinline__ Place place_of(const LcDev& ix, const LcBlobMap& m, const long long* tab, U w) {
    Place p{nullptr, nullptr, nullptr, 0u};
    const int L = ix.L, R = lc_blob_row(L);
    if (w < 16u) { p.value = (uint32_t)m.hdr[w]; return p; }
    const int field = w >= (U)m.nodes ? 1 : 0;                 // which of the two start columns to search
    int lo = 0, hi = ix.B;                                     // last sequence that starts at or before w
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((U)tab[mid * R + field] <= w) lo = mid; else hi = mid;
    }
    const long long* row = tab + lo * R;
    U r = w - (U)row[field];
    const int b = lo;
    if (field == 0) {                                          // T, M, N_1 ..., then the boundaries
        if (r < (U)(L + 1)) p.value = (uint32_t)row[2 + (int)r];
        else p.word = reinterpret_cast<uint32_t*>(ix.bounds + (size_t)b * (ix.cap[0] + 1) + (r - (U)(L + 1)));
        return p;
    }
    U head = 0;                                                // words of one head's levels
    for (int l = 0; l < L; ++l) head += (U)row[3 + l] * (LC_D + 4);
    const U h = r / head;
    r -= h * head;
    int l = 0;
    while (l + 1 < L && r >= (U)row[3 + l] * (LC_D + 4)) { r -= (U)row[3 + l] * (LC_D + 4); ++l; }
    const U n = (U)row[3 + l];
    const size_t base = ((size_t)b * ix.H + (size_t)h) * ix.cap[l];
    if (r < n * LC_D) {
        if (l == 0 && ix.c0_bf16) p.half = reinterpret_cast<uint16_t*>(ix.center[0]) + base * LC_D + r;
        else p.word = reinterpret_cast<uint32_t*>(ix.center[l] + base * LC_D + r);
        return p;
    }
    r -= n * LC_D;
    const int which = (r >= n ? 1 : 0) + (r >= 2 * n ? 1 : 0) + (r >= 3 * n ? 1 : 0);
    r -= (U)which * n;
    if (which == 0) {
        p.word = reinterpret_cast<uint32_t*>(ix.radius[l] + base + r);
        if (l >= 1) p.also = reinterpret_cast<uint32_t*>(ix.rbuild[l] + base + r);
    } else {
        int* const a = which == 1 ? ix.parent[l] : (which == 2 ? ix.ntok[l] : ix.nchunk[l]);
        p.word = reinterpret_cast<uint32_t*>(a + base + r);
    }
    return p;
}

// The sequence table in LDS if it fits, else where it is (pinned host memory).
__device__ __forceinline__ const long long* stage_table(const long long* tab, int n, long long* lds) {
    if (n > LC_BLOB_LDS_ROWS) return tab;
    for (int i = threadIdx.x; i < n; i += LC_BLOB_THREADS) lds[i] = tab[i];
    __syncthreads();
    return lds;
}

// Words [w0, w0 + n) of the blob: index -> pinned host window.
template <typename U>
__global__ void __launch_bounds__(LC_BLOB_THREADS)
lc_blob_export_kernel(LcDev ix, LcBlobMap m, const long long* table, U w0, unsigned n, uint32_t* window) {
    __shared__ long long lds[LC_BLOB_LDS_ROWS];
    const long long* tab = stage_table(table, ix.B * lc_blob_row(ix.L), lds);
    const unsigned i0 = blockIdx.x * (LC_BLOB_THREADS * LC_BLOB_WORDS) + threadIdx.x;
    uint32_t v[LC_BLOB_WORDS];
#pragma unroll
    for (int k = 0; k < LC_BLOB_WORDS; ++k) {
        const Place p = place_of<U>(ix, m, tab, w0 + min(i0 + k * LC_BLOB_THREADS, n - 1u));
        v[k] = p.value;
        if (p.word) v[k] = *p.word;
        if (p.half) v[k] = (uint32_t)*p.half << 16;
    }
#pragma unroll
    for (int k = 0; k < LC_BLOB_WORDS; ++k)
        if (i0 + k * LC_BLOB_THREADS < n) window[i0 + k * LC_BLOB_THREADS] = v[k];
}

// Words [w0, w0 + n) of the blob: pinned host window -> index.  (Header, records and boundaries have
// been read by the host; a bfloat16 center is rounded to nearest even if the word is none already.)
template <typename U>
__global__ void __launch_bounds__(LC_BLOB_THREADS)
lc_blob_import_kernel(LcDev ix, LcBlobMap m, const long long* table, U w0, unsigned n, const uint32_t* window) {
    __shared__ long long lds[LC_BLOB_LDS_ROWS];
    const unsigned i0 = blockIdx.x * (LC_BLOB_THREADS * LC_BLOB_WORDS) + threadIdx.x;
    uint32_t v[LC_BLOB_WORDS];
#pragma unroll
    for (int k = 0; k < LC_BLOB_WORDS; ++k) v[k] = window[min(i0 + k * LC_BLOB_THREADS, n - 1u)];
    const long long* tab = stage_table(table, ix.B * lc_blob_row(ix.L), lds);
#pragma unroll
    for (int k = 0; k < LC_BLOB_WORDS; ++k) {
        const unsigned i = i0 + k * LC_BLOB_THREADS;
        if (i >= n || w0 + i < (U)m.nodes) continue;
        const Place p = place_of<U>(ix, m, tab, w0 + i);
        if (p.word) *p.word = v[k];
        if (p.also) *p.also = v[k];
        if (p.half) *p.half = (uint16_t)((v[k] + 0x7fffu + ((v[k] >> 16) & 1u)) >> 16);
    }
}

unsigned blocks_for(unsigned n) { return (n + LC_BLOB_THREADS * LC_BLOB_WORDS - 1) / (LC_BLOB_THREADS * LC_BLOB_WORDS); }

}  // namespace

int lc_launch_blob_export(const LcDev& ix, const LcBlobMap& m, const long long* table, unsigned long long w0, unsigned n,
                          uint32_t* window, hipStream_t stream) {
    if (m.total < (1ull << 32))
        hipLaunchKernelGGL(lc_blob_export_kernel<unsigned>, dim3(blocks_for(n)), dim3(LC_BLOB_THREADS), 0, stream, ix, m,
                           table, (unsigned)w0, n, window);
    else
        hipLaunchKernelGGL(lc_blob_export_kernel<unsigned long long>, dim3(blocks_for(n)), dim3(LC_BLOB_THREADS), 0, stream,
                           ix, m, table, w0, n, window);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}

int lc_launch_blob_import(const LcDev& ix, const LcBlobMap& m, const long long* table, unsigned long long w0, unsigned n,
                          const uint32_t* window, hipStream_t stream) {
    if (m.total < (1ull << 32))
        hipLaunchKernelGGL(lc_blob_import_kernel<unsigned>, dim3(blocks_for(n)), dim3(LC_BLOB_THREADS), 0, stream, ix, m,
                           table, (unsigned)w0, n, window);
    else
        hipLaunchKernelGGL(lc_blob_import_kernel<unsigned long long>, dim3(blocks_for(n)), dim3(LC_BLOB_THREADS), 0, stream,
                           ix, m, table, w0, n, window);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}
