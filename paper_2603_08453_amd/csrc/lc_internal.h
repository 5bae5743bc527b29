// Host-side structures shared by the translation units of liblychee.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include <atomic>
#include <vector>

#include "lychee.h"

// Most chunks per (sequence, head) that the workgroups of a decode step share out, and with that the keys they post.
#define LC_STEP_SHARE_MAX_CHUNKS 2560
constexpr int lc_posted_slots(int cap0) { return cap0 < LC_STEP_SHARE_MAX_CHUNKS ? cap0 : LC_STEP_SHARE_MAX_CHUNKS; }

// Device-side view of an index, passed to kernels by value.
// Per-level arrays are indexed [(b * H + h) * cap[l] + n]; centers carry d floats per node, except that
// center[0] points at rows of d bfloat16 values when c0_bf16 is set (read it through lc_c0_*).
struct LcDev {
    int B, H, d, L, F;
    int c0_bf16;
    int cap[LC_MAX_LEVELS];
    int* state;      // [B][H][4]: {T, M, 0, 0}: tokens written, closed chunks (one copy per head)
    int* nlev;       // [B][LC_MAX_LEVELS]: nodes per level (entry 0 unused: level 0 has M nodes)
    int* bounds;     // [B][cap[0] + 1]: chunk boundaries (shared by the heads of a sequence)
    int* sync;       // [B][H][4]: arrival counters of the fused kernels (0, 1), zero between calls; 3: number of the next decode step whose
                     // workgroups share the scoring (never 0)
    unsigned long long* posted;   // [B][H][lc_posted_slots(cap[0])]: score keys that those workgroups post for each other: key, number of the step << 32
    float* center[LC_MAX_LEVELS];
    float* radius[LC_MAX_LEVELS];
    int* parent[LC_MAX_LEVELS];
    int* ntok[LC_MAX_LEVELS];
    int* nchunk[LC_MAX_LEVELS];
    float* rbuild[LC_MAX_LEVELS];   // levels >= 1: the radius as the last (re)build left it (baseline of lc_index_drift)
};

struct lc_index {
    lc_config cfg;
    int B, H_kv, d;
    int device;
    void* buf;
    size_t bytes;
    LcDev dev;
    std::vector<int> T;      // host mirror, per sequence
    std::vector<int> M;      // host mirror, per sequence
    std::vector<int> N;      // [B][LC_MAX_LEVELS] nodes per level (N[b][0] mirrors M)
    std::vector<int> tail;   // host mirror, per sequence: tokens behind the last closed chunk
};

// Layout of the index buffer: fills dev pointers from base; returns total bytes.
size_t lc_layout_index(const lc_config* cfg, int B, int H, int d, void* base, LcDev* dev);

// Workspace carve-up (all offsets 256-byte aligned).
#define LC_KM_FLAGS 64       // k-means iterations whose progress flags the workspace holds
struct LcWs {
    // retrieval
    uint32_t* keys;      // [B][H][cap0] order-preserving score keys of the chunks (0 = not a candidate)
    uint8_t* want;       // [B][H][cap0] 1 = this chunk's score is needed
    int* scratch;        // [B][H][4 * cap0] chunk-level staging when it does not fit in LDS; chunk entries of the fused step
    int32_t* ids_tmp;    // [B][H][cap0] chunk list of a decode step that has to run as two kernels
    int32_t* counts_tmp; // [B][H]
    // decode
    float* part_acc;     // [B][H][S][G][d]
    float* part_ml;      // [B][H][S][G][2]
    // build
    float* dirs;         // [B][H][cap0][d] unit directions of the chunks (and of every second level above)
    uint16_t* dirs16;    // the same rounded to bfloat16
    float* next_pts;     // [B][H][cap1][d] unit directions of the other levels
    uint16_t* next_pts16;
    float* cent[2];      // [B][H][cap1][d] centroids of the level being clustered, start of the next level's
    uint16_t* cent16[2];
    int* kflags;         // [level][B][H][LC_KM_FLAGS] "iteration t of the k-means moved a point" (tiled kernels only)
    float* rounds;       // what the workgroups of a clustering post for each other (lc_kmeans_rounds_kernel), behind `total`
    size_t rounds_bytes; // of it in this workspace; a smaller one does without
    int first_parts;     // > 0: the workgroups of a clustering in one kernel come in two launches (lc_bench_recluster_in_two)
    size_t total;
};
// Clusterings in one kernel: most (sequence, head)s, iterations and points; most clusters.
#define LC_RK_MAX_PAIRS 128
#define LC_RK_MAX_SHARE 64
#define LC_RK_MAX_ITERS 16
#define LC_RK_MAX_POINTS 8192
#define LC_RK_MAX_CLUSTERS 256
size_t lc_rounds_bytes(const lc_config* cfg, int B, int H);
// with_build = false leaves out the build scratch (directions, centroids): what a decode step needs.
size_t lc_layout_ws(const lc_config* cfg, int B, int H_q, int H, int d, int splits, void* base, LcWs* ws,
                    bool with_build = true);
// Up to this many chunks per (sequence, head) the workgroups of a decode step may score all of them themselves.
#define LC_STEP_SINGLE_MAX_CHUNKS 128
#define LC_COMPUTE_UNITS 256                // of an MI355X
#define LC_DEC_MIN_TOKENS_PER_SPLIT 64      // tokens of a split of the attention kernel, at least
int lc_auto_splits(const lc_config* cfg, int B, int H);

void lc_set_hip_error(hipError_t e);
#define LC_HIP_CHECK(expr)                       \
    do {                                         \
        hipError_t _e = (expr);                  \
        if (_e != hipSuccess) {                  \
            lc_set_hip_error(_e);                \
            return LC_ERR_HIP;                   \
        }                                        \
    } while (0)

// Runs a call that has to succeed once per device (setting a kernel's attribute) and remembers that it did.
struct LcOnce {
    std::atomic<unsigned long long> done{0};     // one bit per device; devices beyond 63 run it every time
    template <typename F>
    hipError_t run(F f) {
        int dev = 0;
        const hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const unsigned long long bit = dev >= 0 && dev < 64 ? 1ull << dev : 0ull;
        if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
        const hipError_t r = f();
        if (r == hipSuccess) done.fetch_or(bit, std::memory_order_release);
        return r;
    }
};

// lc_decode_step with a switch for the measurement aid that launches its last kernel alone
// (C linkage: defined among the entry points), and whether that one kernel is all of it.
extern "C" int lc_decode_step_impl(const lc_index* idx, const void* q, const void* K, const void* V,
                                   const int64_t kv_strides[3], int H_q, int budget, float* out, float* lse,
                                   int32_t* chunk_ids, int32_t* counts, int cap, void* ws, size_t ws_bytes,
                                   void* stream, bool last_kernel_only);
extern "C" int lc_decode_step_is_one_kernel(const lc_index* idx, int H_q, int budget);
// lc_recluster with LcWs::first_parts.
extern "C" int lc_recluster_impl(lc_index* idx, void* ws, size_t ws_bytes, void* stream, int first_parts);

// Limits of the two level walks (pure host functions).
int lc_walk_max_internal_nodes();   // exact walk: internal nodes of one (sequence, head), all levels together
int lc_beam_max_level_nodes();      // top-k per level: nodes of one internal level of one (sequence, head)

// Launchers (each enqueues on `stream` and returns LC_OK or LC_ERR_HIP).
int lc_launch_build(const lc_index* idx, const LcWs& ws, const void* K, const int64_t ks[3],
                    int max_M, hipStream_t stream);
int lc_launch_retrieve(const lc_index* idx, const LcWs& ws, const void* q, int G, int budget,
                       int32_t* ids, int32_t* counts, float* scores, int cap,
                       int max_M, int max_upper, int score_only, hipStream_t stream);
int lc_launch_decode(const lc_index* idx, const LcWs& ws, const void* q, const void* K, const void* V,
                     const int64_t ks[3], const int32_t* ids, const int32_t* counts, int cap, int G,
                     int splits, float* out, float* lse, hipStream_t stream);
// Who scores the chunks of a fused step: a kernel before it (chunk entries in ws.scratch, lc_launch_retrieve with score_only), every
// workgroup all of them (up to LC_STEP_SINGLE_MAX_CHUNKS), or the workgroups of a (sequence, head) a share each (up to LC_STEP_SHARE_CHUNKS of
// LC_STEP_SHARE_MAX_CHUNKS in all).
enum { LC_SCORED_BEFORE = 0, LC_SCORED_HERE = 1, LC_SCORED_SHARED = 2 };
#define LC_STEP_SHARE_CHUNKS 128
// One kernel or two (without a level walk): every workgroup scoring all chunks costs 0.5 us per 64 chunks at group
// size 4, twice that at 7 or 8, times the workgroups that share a compute unit; the scoring kernel costs about 2 us.
// Measured from 16 to 256 chunks, 8 to 128 (sequence, head) pairs and group sizes 1, 4 and 7: up to 64 chunks
// one kernel is always faster (by 0.3 to 2.8 us), up to 128 unless a large group meets several workgroups per unit
// (16 sequences x 4 heads of group size 7: 1 us slower), at 192 hardly ever.
inline bool lc_step_is_single(int max_M, int G, long long workgroups) {
    return max_M <= 64 || (max_M <= LC_STEP_SINGLE_MAX_CHUNKS && (G <= 4 || workgroups <= 256));
}
// Fused step: selection + attention; `single`: the scoring too.  lc_decode_fused_fits tells whether a selecting workgroup holds max_M chunks.
bool lc_decode_fused_fits(int G, int max_M);
int lc_launch_decode_fused(const lc_index* idx, const LcWs& ws, const void* q, const void* K, const void* V,
                           const int64_t ks[3], int G, int splits, int budget, int32_t* ids_out,
                           int32_t* counts_out, int cap, int max_M, bool single, float* out, float* lse, hipStream_t stream);
// out (device): [B][H][4] floats: sum of radii at build, sum now, largest growth, nodes counted
int lc_launch_drift(const lc_index* idx, int level, float* out, hipStream_t stream);
// Puts a staged [state | nlev | offsets | chunk boundaries of all sequences] block (pinned host memory) in place
// and zeroes the arrival counters; the second one nlev alone.
int lc_launch_place_state(const lc_index* idx, const int32_t* staged, int max_M, hipStream_t stream);
int lc_launch_place_counts(const lc_index* idx, const int32_t* staged, hipStream_t stream);
int lc_launch_append(const lc_index* idx, void* K, void* V, const int64_t ks[3],
                     const void* k_new, const void* v_new, const uint8_t* close_dev_flags_or_null,
                     uint32_t close_mask_lo, hipStream_t stream);
