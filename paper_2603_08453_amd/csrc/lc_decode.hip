// Sparse attention for one decode step: split-K flash-decode over the selected
// chunks (plus the open tail), merged by the last split to finish.
//
// Grid (split, KV head, sequence), 256 threads = 16 groups of 16 lanes.  A group
// owns a contiguous run of the split's tokens and handles them U at a time.
//   Q.K^T runs on the matrix cores: the 4 groups of a wavefront together hold 16
//   tokens, whose K rows form the 16 x 128 A operand of four 16x16x32 bf16 MFMAs;
//   the B operand is the query block (head n in column n).  The result leaves lane
//   (group, n) with the logits of the group's own tokens for head n, so each lane
//   keeps the online softmax (base 2) of one head.
//   P.V runs there too, without a value crossing lanes: a lane's four probabilities are
//   its share of the A operand (row n: head n), and the eight columns [8n, 8n + 8) it
//   loaded of its group's four V rows are, column by column, its share of eight B operands
//   (operand c: columns c, c + 8, ...).  V is bfloat16 as stored; a probability goes in
//   as three bfloat16 terms that add up to its float32 value (lc_split3), so that
//   products and sums are those of float32.
//   With P.V on the vector ALU a batch of 16 tokens took a wavefront 150 instructions at
//   group size 4 and 250 at 7 (with half the lanes' K loads empty there, for want of
//   registers), now about 100 and 64 cycles of the matrix pipe, and the groups' sums need
//   no combining.  A step: 18.1 -> 16.9 us (4 x 32K tokens), 20.2 -> 19.2 (128K), 29.9 ->
//   27.6 (16 ragged sequences, group size 7).  Relative error against float64 over steps
//   of the sizes in use: 3.88e-7, on the vector ALU 3.91e-7 (both with logits rounded before
//   the reference was subtracted; random steps of 300 to 20000 tokens at group size 4: 2.40e-7
//   then, 2.35e-7 with one rounding, the log-sum-exp 4.0e-7 and 2.6e-7).
#include <type_traits>

#include "lc_device.h"
#include "lc_internal.h"
#include "lc_select.h"

#ifndef LC_DEC_THREADS
#define LC_DEC_THREADS 256
#endif
#define LC_INLINE __attribute__((always_inline))       // (lambdas that hold registers by reference)
#define LC_DEC_GROUPS (LC_DEC_THREADS / 16)
#define LC_DEC_MAX_SPLITS 256
#define LC_DEC_TILE 1024          // tokens of a split whose cache rows are resolved into LDS at a time
#define LC_DEC_LAG 8              // powers of two that a logit may lie above the softmax's reference
#define LC_DEC_FAINT -101.f       // logits that lie further below the reference have probabilities that lc_split3 does not hold (below 2^-109)
#define LC_DEC_LOOKS 128          // times a wavefront looks for keys before it scores them itself (27 to 43 us for all of them on a quiet device, 0.6 us each while others score)
#define LC_DEC_E 2                // selected ids per thread and pass of the row resolution
#define LC_LOG2E 1.4426950408889634f
#define LC_LN2 0.6931471805599453f

typedef __bf16 lc_bf16x8 __attribute__((ext_vector_type(8)));
typedef float lc_f32x4 __attribute__((ext_vector_type(4)));


struct LcDecodeArgs {
    LcDev ix;
    const uint16_t* q;
    const uint16_t* K;
    const uint16_t* V;
    long long ks_seq, ks_head, ks_tok;
    const int32_t* ids;
    const int32_t* counts;
    int cap;
    float* part_acc;      // [B][H][S][G][d]
    float* part_ml;       // [B][H][S][G][2]
    float* out;           // [B][H*G][d]
    float* lse;           // [B][H*G] or null
    // fused step only (the kernel selects the chunks itself from their score keys):
    const int* entries;   // [B][H][cap0] chunk entries (LcChunkEntry) of the scoring kernel (unused where this kernel scores)
    int32_t* ids_out;     // [B][H][cap] selected ids, ascending, or null
    int32_t* counts_out;  // [B][H] or null
    int budget, sink;     // token budget, tokens of the pinned prefix
    int ew;               // fused step: rows of 64 chunks per wavefront that hold the longest sequence (host side: picks EC)
    int max_tokens;       // rows of one (sequence, head) slab of K and V
    int share;            // chunks that a workgroup scores (LC_SCORED_SHARED), a multiple of four
};

// N probabilities as three bfloat16 terms each, packed in pairs: t[s] holds the terms number s.  The three add up to
// the float32 value exactly: each takes the upper eight of the bits that are left, and where those are all of them, one unit less, so
// that something is left (a term of zero would turn an infinite V into a not-a-number).  Below 2^-109 one in 65536
// has a term of zero, below 2^-110 the lowest bits have no place in bfloat16's range: where such a probability meets a value of 2^64 or more, infinities among them, the split is done
// again on the vector ALU (attend_plain) by the workgroup that merges; smaller values are off by less than 2^-69.
template <int N>
__device__ __forceinline__ void lc_split3(const float (&p)[N], int (&t)[3][N / 2]) {
    float r[N];
#pragma unroll
    for (int u = 0; u < N; ++u) r[u] = p[u];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        uint32_t w[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            w[u] = __float_as_uint(r[u]);
            if (s < 2) {
                w[u] = __builtin_elementwise_sub_sat(w[u], 1u);     // (0 stays 0)
                r[u] -= __uint_as_float(w[u] & 0xffff0000u);
            }
        }
#pragma unroll
        for (int k = 0; k < N / 2; ++k) t[s][k] = (int)__builtin_amdgcn_perm(w[2 * k + 1], w[2 * k], 0x07060302u);   // the upper halves
    }
}
// a in the lower half of the wavefront and b in the upper half, each summed over the two halves
__device__ __forceinline__ float lc_add_halves(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// a in the even 16-lane rows and b in the odd ones, each summed over a row and its neighbour
__device__ __forceinline__ float lc_add_rows(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// maximum over the four 16-lane groups, in every lane
__device__ __forceinline__ float lc_max_groups(float v) {
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// 2^(x - LC_DEC_LAG) of a logit that lies x above its reference, -inf included: at most 1 where x is at most LC_DEC_LAG, so that P.V
// overflows no sooner than the values' own sum.  (The exponent is lowered behind the exponential and not in x, which would lose its lowest
// bits, by the factor that keeps small results out of the instruction's reach of zero: no instruction more than without.)
__device__ __forceinline__ float lc_probability(float x) {
    const bool small = x < -64.f;
    return __builtin_amdgcn_exp2f(x + (small ? 64.f : 0.f)) * (small ? __builtin_ldexpf(1.f, -64 - LC_DEC_LAG) : __builtin_ldexpf(1.f, -LC_DEC_LAG));
}

// Sums whose references lie `by` powers of two apart are added by fma with 2^by.  Where that is below float32's range, an infinite sum has
// become something that is no number; only then the sums are added once more, each with its infinities (multiplied by 2^-149
// twice: once would leave 2^-22 of the largest finite ones).
__device__ __forceinline__ bool lc_no_number(const float4& x) { return __ballot(!((x.x + x.y) + (x.z + x.w) == (x.x + x.y) + (x.z + x.w))) != 0ull; }
__device__ __forceinline__ void lc_add_scaled(float4& sum, const float4& x, float by) {
    const float f = by == 0.f ? __builtin_ldexpf(1.f, -149) : 1.f, g = by == 0.f ? f : by;
    sum.x = fmaf(x.x * f, g, sum.x); sum.y = fmaf(x.y * f, g, sum.y);
    sum.z = fmaf(x.z * f, g, sum.z); sum.w = fmaf(x.w * f, g, sum.w);
}

// FUSED = false: the chunk list comes from a.ids / a.counts.  FUSED = true: every workgroup first
// repeats the budget selection of its (sequence, head) from the chunk score keys -- the same
// deterministic routine on the same keys, so all splits agree -- and never reads a chunk list.
//
// SCORE = LC_SCORED_HERE (with FUSED): it scores the chunks as well, so that the step is one kernel.  That costs every split
// the scoring of all chunks -- four per group of lanes, 0.5 us and more for every 64 of them -- and saves a launch
// and a pass through memory (113 chunks, 8 heads: 12.9 -> 11.3 us; where the line lies: lc_step_is_single).
//
// SCORE = LC_SCORED_SHARED (with FUSED): each of the workgroups of a (sequence, head) scores a share of the chunks and posts their keys in the
// index, all read all of them.  A key is posted together with the number of the step (`sync`), in one 8-byte access at agent scope, so a reader sees from the
// word itself whether it is this step's: no counter, no wait for stores.  No workgroup depends on another one to get ahead: a wavefront that has
// looked LC_DEC_LOOKS times for keys that are not there (a workgroup that has no place yet, behind another stream's kernel) scores
// its chunks itself, posts what the others would have posted, and looks once more.
//
// Either way the selected chunks sit in a list, in id order; the wavefronts write the cache row of
// every token of the split's tile into LDS, 64 lanes per overlapping chunk.
template <int G, bool FUSED, int EC, int SCORE>
// (two wavefronts per SIMD asked for: without that the compiler puts the accumulators into the other half of the register
// file and copies them back and forth)
__global__ void __launch_bounds__(LC_DEC_THREADS, 2)
lc_decode_kernel(const LcDecodeArgs a) {
    lc_fetch_args<sizeof(LcDecodeArgs)>();
    // FUSED: the selection's chunk lists (written 8 bytes at a time: from a base that is not a multiple of 8 that took 0.7 us more)
    extern __shared__ __attribute__((aligned(16))) int lds_dyn[];
    using SelStore = typename std::conditional<FUSED, LcLeafSelSh, int>::type;
    using FusedStore = typename std::conditional<FUSED, LcFusedSh<LC_DEC_THREADS>, int>::type;
    // What is used one after the other shares its place, so that the two workgroups per compute unit that the registers allow fit its LDS with
    // the longest chunk lists as well (group size 8: 26 KB and 49 KB of lists; side by side the parts would be 42 KB and more).
    union Phases {
        SelStore sel;                            // selection, crowded cutoff bin
        struct {                                 // the wavefronts' sums
            float4 acc[LC_DEC_THREADS / 64][G][LC_D / 4];
            float ml[LC_DEC_THREADS / 64][G][2];
        } comb;
        float scale[LC_DEC_THREADS / 32][LC_DEC_MAX_SPLITS + 128];      // merge
    };
    union Rows {
        int row[LC_DEC_TILE];                    // cache rows of the tile's tokens
        float4 red[LC_DEC_THREADS];              // merge
    };
    __shared__ __attribute__((aligned(16))) Phases ph;
    __shared__ __attribute__((aligned(16))) Rows rw;
    __shared__ __attribute__((aligned(16))) FusedStore fused_store;
    __shared__ lc_v4i entry_sh[SCORE == LC_SCORED_HERE ? LC_STEP_SINGLE_MAX_CHUNKS : 1];
    __shared__ int scan_sh[8];
    __shared__ int last_sh;
    static_assert(sizeof(rw.red) <= sizeof(rw.row), "");

    constexpr int U = 4;                         // tokens per group and batch of loads; a step takes two batches
    constexpr int E = LC_DEC_E;
    const LcDev& ix = a.ix;
    const int s = blockIdx.x, S = gridDim.x, h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = tid & 15, grp = tid >> 4, q4 = lane >> 4;

    const int* bnd = ix.bounds + (size_t)b * (ix.cap[0] + 1);
    // the query block in MFMA B layout (lane (q4, n): head n, columns 8 q4 + 32 j + [0, 8), loaded once)
    uint4 qb[4];
    {
        const uint16_t* qh = a.q + ((size_t)b * ix.H * G + (size_t)h * G + min(sub, G - 1)) * LC_D + 8 * q4;
#pragma unroll
        for (int j = 0; j < 4; ++j) qb[j] = *reinterpret_cast<const uint4*>(qh + 32 * j);
    }

    // ---- the attended tokens are the selected chunks in ascending id order, then the open tail.
    // Entry i of that list is (first cache row, length).  Both variants end up with: n_runs entries,
    // n_tok tokens, and a way to find the cache row of every token of a tile.
    int n_runs = 0, n_tok, T;
    // FUSED = false: thread t of a pass owns entries [E t, E t + E); the first pass stays in registers
    const int32_t* ids = nullptr;
    int n_ids = 0, M = 0;
    int idv[E], st0[E], ln0[E];
    int ex0 = 0, tot0 = 0;
    // FUSED = true: this lane's chunks and the totals of the selection
    LcChunkSel<EC> cs;

    auto entries = [&](int base, bool preloaded, int (&st)[E], int (&ln)[E]) -> int {
        int sum = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = base + tid * E + e;
            st[e] = 0;
            ln[e] = 0;
            if (i < n_ids) {
                const int id = max(0, min(preloaded ? idv[e] : ids[i], M - 1));
                st[e] = bnd[id];
                ln[e] = max(0, bnd[id + 1] - st[e]);
            } else if (i == n_ids) {
                st[e] = bnd[M];
                ln[e] = max(0, T - st[e]);
            }
            sum += ln[e];
        }
        return sum;
    };

    // Scoring of chunks in this kernel, N to a group of lanes at a time (1, 2 or 4).
    struct Pass {
        LcNodeFrag f[4];
        float R;
        int s0, s1;
    };
    uint32_t qp[SCORE != LC_SCORED_BEFORE ? G : 1][4];
    float qn[SCORE != LC_SCORED_BEFORE ? G : 1];
    // chunks j .. j + N - 1 (of this lane's group): their centers; radius and boundaries of number (sub & (N - 1)) of them.  From `end` on
    // nothing is fetched (the offsets are past the arrays' ends).
    auto load = [&](auto count, Pass& w, int j, int end) LC_INLINE {
        constexpr int N = decltype(count)::value;
        const int rows = lc_posted_slots(ix.cap[0]);
        j = j < end ? j : rows;
        const size_t cb = (size_t)bh * ix.cap[0];
        const bool c0b = ix.c0_bf16 != 0;
        const int cen_row = c0b ? LC_D * 2 : LC_D * 4;
        const __amdgpu_buffer_rsrc_t cen_r = lc_buffer(reinterpret_cast<const char*>(ix.center[0]) + cb * cen_row, rows * cen_row);
        const __amdgpu_buffer_rsrc_t rad_r = lc_buffer(ix.radius[0] + cb, rows * 4);
        const __amdgpu_buffer_rsrc_t bnd_r = lc_buffer(bnd, (rows + 1) * 4);
        if (c0b) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const lc_v2i x = __builtin_amdgcn_raw_buffer_load_b64(cen_r, (j + k) * cen_row + 8 * sub, 0, 0);
                const lc_v2i y = __builtin_amdgcn_raw_buffer_load_b64(cen_r, (j + k) * cen_row + 8 * sub + 128, 0, 0);
                w.f[k].a = make_float4(__int_as_float(x.x), __int_as_float(x.y), 0.f, 0.f);
                w.f[k].b = make_float4(__int_as_float(y.x), __int_as_float(y.y), 0.f, 0.f);
            }
        } else {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                w.f[k].a = lc_buf_load_f32x4(cen_r, (j + k) * cen_row + 16 * sub);
                w.f[k].b = lc_buf_load_f32x4(cen_r, (j + k) * cen_row + 16 * sub + 256);
            }
        }
        const int own = j + (sub & (N - 1));
        w.R = lc_buf_load_f32(rad_r, own);
        w.s0 = lc_buf_load_i32(bnd_r, own);
        w.s1 = lc_buf_load_i32(bnd_r, own + 1);
    };
    // key of chunk j + (sub & (N - 1)), in the lanes with (sub & 4) set
    auto score = [&](auto count, Pass& w) LC_INLINE -> uint32_t {
        constexpr int N = decltype(count)::value;
        if (ix.c0_bf16) {
#pragma unroll
            for (int k = 0; k < N; ++k) w.f[k] = lc_widen_chunk_frag(w.f[k]);
        }
        const float sc = lc_score_packed<SCORE != LC_SCORED_BEFORE ? G : 1, N>(w.f, w.R, sub, qp, qn);
        return a.budget > 0 && w.s0 >= a.sink ? lc_score_key(sc) : 0u;
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    using Four = std::integral_constant<int, 4>;
    // LC_SCORED_HERE: entries of the chunks, 64 at a time: group `grp` has chunks 64 p + 4 grp + (0..3) of pass p < 2
    static_assert(LC_STEP_SINGLE_MAX_CHUNKS <= 128 && LC_STEP_SHARE_CHUNKS <= 128, "two passes");
    auto score_chunks = [&]() LC_INLINE {
        // (both loads go out before the chunk count is known)
        Pass first, second;
        load(Four(), first, 4 * grp, LC_STEP_SINGLE_MAX_CHUNKS);
        if (ix.cap[0] > 64) load(Four(), second, 64 + 4 * grp, LC_STEP_SINGLE_MAX_CHUNKS);
        lc_load_query_packed<SCORE != LC_SCORED_BEFORE ? G : 1>(a.q + (size_t)b * ix.H * G * LC_D, h, sub, qp, qn);
        auto enter = [&](Pass& w, int p) LC_INLINE {
            lc_v4i e;
            e.x = (int)score(Four(), w);
            e.y = w.s0;
            e.z = max(0, w.s1 - w.s0);
            e.w = 0;
            if ((sub >> 2) == 1) entry_sh[64 * p + 4 * grp + (sub & 3)] = e;
        };
        enter(first, 0);
        if (ix.state[bh * 4 + 1] > 64) enter(second, 1);
        lc_barrier_lds();
    };
    // LC_SCORED_SHARED: this workgroup's share of the chunks is scored and posted, then this lane's chunks j0 + 64 e are read
    auto share_scores = [&](int j0, uint32_t (&key)[EC], int (&begin)[EC], int (&end)[EC]) LC_INLINE {
        const int rows = lc_posted_slots(ix.cap[0]);
        const __amdgpu_buffer_rsrc_t bnd_r = lc_buffer(bnd, (rows + 1) * 4);
        const __amdgpu_buffer_rsrc_t posted_r = lc_buffer(ix.posted + (size_t)bh * rows, rows * 8);
        const int lo = s * a.share, hi = min(lo + a.share, rows);
        const int M = min(ix.state[bh * 4 + 1], rows), number = ix.sync[bh * 4 + 3];
        __builtin_amdgcn_sched_barrier(0);                          // (on their way before the first wait)
        Pass first, second;
        // (64 chunks first, or 32; a few more a chunk to a group)
        const bool small = a.share <= 32, few_more = a.share <= 80;
        if (small) load(Two(), first, lo + 2 * grp, hi);
        else load(Four(), first, lo + 4 * grp, hi);
        if (a.share > 64) {
            if (few_more) load(One(), second, lo + 64 + grp, hi);
            else load(Four(), second, lo + 64 + 4 * grp, hi);
        }
        lc_load_query_packed<SCORE != LC_SCORED_BEFORE ? G : 1>(a.q + (size_t)b * ix.H * G * LC_D, h, sub, qp, qn);
        // (a chunk of its own per lane that stores; past the buffer's end nothing is stored)
        auto post = [&](auto count, Pass& w, int j, int end) LC_INLINE {
            constexpr int N = decltype(count)::value;
            const lc_v2i x = {(int)score(count, w), number};
            const int own = j + (sub & 3);
            if ((sub >> 2) == 1 && (sub & 3) < N && own < end) __builtin_amdgcn_raw_buffer_store_b64(x, posted_r, own * 8, 0, 16);
        };
        const int mine = min(hi, M);                                // (whole wavefronts without a chunk have nothing to do)
        if (small) {
            if (lo + 8 * wave < mine) post(Two(), first, lo + 2 * grp, hi);
        } else {
            if (lo + 16 * wave < mine) post(Four(), first, lo + 4 * grp, hi);
            if (few_more) {
                if (lo + 64 + 4 * wave < mine) post(One(), second, lo + 64 + grp, hi);
            } else {
                if (lo + 64 + 16 * wave < mine) post(Four(), second, lo + 64 + 4 * grp, hi);
            }
        }
#pragma unroll
        for (int e = 0; e < EC; ++e) {
            begin[e] = __builtin_amdgcn_raw_buffer_load_b32(bnd_r, j0 * 4, e * 256, 0);
            end[e] = __builtin_amdgcn_raw_buffer_load_b32(bnd_r, j0 * 4 + 4, e * 256, 0);
        }
        // The keys of the others are on their way for as long as a store takes to reach the memory side (about 0.6 us): a look before
        // that fails, holds the next one back by 0.6 us and takes bandwidth from those that still score.  20 * 64 cycles of waiting, against none:
        // 4 sequences of 32K 16.5 -> 15.8 us, eight layers of 128K 153.1 -> 146.7, 16 ragged sequences 23.9 -> 23.5; 18 to 26 are the same within 0.5 %,
        // 6 gives half of it and 44 a quarter to half.
        __builtin_amdgcn_s_sleep(20);
        // Before the first look the chunks behind all shares, if there are any (an index that has grown since this launch was captured), 16 for each workgroup
        // in turn; left to the wavefronts that look for them, a replay took 38 to 55 us where a step captured anew takes 12.  After LC_DEC_LOOKS of them all
        // chunks of this wavefront, then one look more: the loop ends whatever is in memory.  (One copy of the scoring for both, a chunk to a group: what is
        // fetched of a kernel's code is in every step's time.  Eight layers of 128K with two copies 150.1 us, four chunks to a group 147.9, so 147.3, without any 146.8.)
        const int behind = S * a.share;
        for (int looks = 0;; ++looks) {
            if (__builtin_expect(looks == 0 ? behind < M : looks == LC_DEC_LOOKS, 0)) {
                const int step = looks == 0 ? 16 * S : 4, end = looks == 0 ? M : min((wave + 1) * (EC * 64), M);
                for (int j = looks == 0 ? behind + 16 * s + 4 * wave : wave * (EC * 64); j < end; j += step) {
                    load(One(), first, j + q4, end);
                    post(One(), first, j + q4, end);
                }
                __builtin_amdgcn_s_waitcnt(0);                      // (at the next look they are there)
            }
            // (a load through a resource is an ordinary one to the compiler: every look is to be one of its own.  Marked volatile, each of the EC loads
            // would be waited for before the next)
            __atomic_signal_fence(__ATOMIC_ACQ_REL);
            lc_v2i x[EC];
#pragma unroll
            for (int e = 0; e < EC; ++e) x[e] = __builtin_amdgcn_raw_buffer_load_b64(posted_r, j0 * 8, e * 512, 16);
            bool there = true;
#pragma unroll
            for (int e = 0; e < EC; ++e) {
                key[e] = (uint32_t)x[e].x;
                there = there && (x[e].y == number || j0 + 64 * e >= M);
            }
            if (__ballot(there) == ~0ull || looks == LC_DEC_LOOKS) break;
        }
    };

    if constexpr (!FUSED) {
        ids = a.ids + (size_t)bh * a.cap;
        // independent loads first: the ids a thread will need are fetched before the count is known
#pragma unroll
        for (int e = 0; e < E; ++e) idv[e] = (tid * E + e < a.cap) ? ids[tid * E + e] : 0;
        T = ix.state[bh * 4 + 0];
        M = ix.state[bh * 4 + 1];
        n_ids = a.counts[bh];
        n_ids = (M > 0) ? max(0, min(n_ids, a.cap)) : 0;
        n_runs = n_ids + 1;
        ex0 = lc_block_scan<LC_DEC_THREADS>(entries(0, true, st0, ln0), scan_sh, &tot0);
        n_tok = tot0;
        for (int base = LC_DEC_THREADS * E; base < n_runs; base += LC_DEC_THREADS * E) {
            int st[E], ln[E], tot;
            lc_block_scan<LC_DEC_THREADS>(entries(base, false, st, ln), scan_sh, &tot);
            n_tok += tot;
        }
    } else {
        const __amdgpu_buffer_rsrc_t ent_r = lc_buffer(a.entries + (size_t)bh * 4 * ix.cap[0], ix.cap[0] * 16);
        const int first = wave * (EC * 64) + lane;
        uint32_t key[EC];
        int begin[EC], end[EC];
        if constexpr (SCORE == LC_SCORED_HERE) score_chunks();
        if constexpr (SCORE == LC_SCORED_SHARED) share_scores(first, key, begin, end);
        auto entry = [&](int e) -> lc_v4i {
            if constexpr (SCORE == LC_SCORED_HERE) return entry_sh[min(first + 64 * e, LC_STEP_SINGLE_MAX_CHUNKS - 1)];
            else if constexpr (SCORE == LC_SCORED_SHARED) return lc_v4i{(int)key[e], begin[e], max(0, end[e] - begin[e]), 0};
            else return __builtin_amdgcn_raw_buffer_load_b128(ent_r, first * 16, e * 1024, 0);
        };
        lc_select_chunks<LC_DEC_THREADS, EC>(ix, b, bh, entry, a.budget, a.sink, s == 0 ? a.ids_out : nullptr,
                                             a.counts_out, a.cap, ph.sel, fused_store, lds_dyn, cs);
        T = cs.T;
        M = cs.M;
        n_tok = cs.n_tok;
    }
    int S_eff = (n_tok + LC_DEC_MIN_TOKENS_PER_SPLIT - 1) / LC_DEC_MIN_TOKENS_PER_SPLIT;
    S_eff = max(1, min(S, S_eff));

    const float scale = 0.08838834764831845f * LC_LOG2E;     // log2(e) / sqrt(128)
    // Softmax state of head `sub` (lanes sub >= G repeat head G - 1): the reference that is subtracted from the
    // logits, one for the wavefront's tokens, and the sum over this group's tokens.  acc[c][r]: columns
    // 8 sub + c of head 4 q4 + r over the wavefront's tokens.
    float m_ref = LC_NEG_INF, l_run = 0.f;
    lc_f32x4 acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = lc_f32x4{0.f, 0.f, 0.f, 0.f};
    // K and V of this (sequence, head) as buffer resources: one 32-bit byte offset per row
    // (the host has checked that the slab spans less than 2 GiB)
    // (the resources end with the last row the index may ever hold, so a wrong row cannot fault)
    const int row_bytes = (int)a.ks_tok * 2;
    const int slab_bytes = (a.max_tokens - 1) * row_bytes + LC_D * 2;
    const __amdgpu_buffer_rsrc_t Kr = lc_buffer(a.K + (size_t)b * a.ks_seq + (size_t)h * a.ks_head, slab_bytes);
    const __amdgpu_buffer_rsrc_t Vr = lc_buffer(a.V + (size_t)b * a.ks_seq + (size_t)h * a.ks_head, slab_bytes);

    // A lane loads K for token (sub & 3) of group (sub >> 2) of its wavefront -- row `sub` of the
    // MFMA A operand -- and V for the tokens of its own group.
    const int gk = (wave << 2) + (sub >> 2), uk = sub & 3;
    int tv = 0, tv_end = 0, tk = 0, tk_end = 0;
    // Two batches' loads, branch-free: a branch around a load would put each row lookup (an LDS read) and its load in a
    // basic block of its own, waited for one after the other.  All row lookups go out together (slot 0 stands in where
    // there is no token; the empty statement keeps the compiler from guarding them) and a load without a token gets
    // an offset past the resource's end, which the range check answers with zeros.
    auto k_offsets = [&](int it, int (&o)[2]) LC_INLINE {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int tok = tk + (it + i) * U + uk;
            int row = rw.row[tok < tk_end ? tok : 0];
            asm volatile("" : "+v"(row));
            o[i] = tok < tk_end ? row * row_bytes + 16 * q4 : slab_bytes;
        }
    };
    auto v_offsets = [&](int it, int (&o)[2 * U]) LC_INLINE {
        int row[2 * U];
#pragma unroll
        for (int u = 0; u < 2 * U; ++u) {
            const int tok = tv + it * U + u;
            row[u] = rw.row[tok < tv_end ? tok : 0];
        }
#pragma unroll
        for (int u = 0; u < 2 * U; ++u) {
            asm volatile("" : "+v"(row[u]));
            o[u] = tv + it * U + u < tv_end ? row[u] * row_bytes + 16 * sub : slab_bytes;
        }
    };
    auto load_k = [&](const int (&o)[2], lc_v4i (&kA)[4], lc_v4i (&kB)[4]) LC_INLINE {
#pragma unroll
        for (int j = 0; j < 4; ++j) kA[j] = __builtin_amdgcn_raw_buffer_load_b128(Kr, o[0] + 64 * j, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) kB[j] = __builtin_amdgcn_raw_buffer_load_b128(Kr, o[1] + 64 * j, 0, 0);
    };
    auto load_v = [&](const int (&o)[2 * U], lc_v4i (&vA)[U], lc_v4i (&vB)[U]) LC_INLINE {
#pragma unroll
        for (int u = 0; u < U; ++u) vA[u] = __builtin_amdgcn_raw_buffer_load_b128(Vr, o[u], 0, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) vB[u] = __builtin_amdgcn_raw_buffer_load_b128(Vr, o[U + u], 0, 0);
    };
    // logits of 16 tokens of the wavefront for all heads: d[i] is token 4 q4 + i = token i of this lane's group, head `sub`
    auto logits = [&](const lc_v4i (&kv)[4]) LC_INLINE -> lc_f32x4 {
        lc_f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lc_bf16x8, kv[j]),
                                                        __builtin_bit_cast(lc_bf16x8, qb[j]), d, 0, 0, 0);
        return d;
    };
    // one online-softmax update of this lane's head with the logits of batches it and it + 1 (N = 8) or it alone (N = 4);
    // whether any of the probabilities is too small for attend1 and attend2 (uniform).  `plain`: for attend_plain, which takes probabilities
    // over the whole of float32's range: the reference does not lag, nothing is lowered, -0 for a logit of -inf.
    auto softmax = [&](auto count, auto plain, int it, lc_f32x4 dA, lc_f32x4 dB, auto& p) LC_INLINE -> bool {
        constexpr int N = decltype(count)::value;
        constexpr bool PLAIN = decltype(plain)::value;
        constexpr float LAG = PLAIN ? 0.f : (float)LC_DEC_LAG;
        float x[N];                                             // logits, not yet scaled
        float mx = LC_NEG_INF;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            x[u] = (tv + it * U + u < tv_end) ? (u < U ? dA[u % U] : dB[u % U]) : LC_NEG_INF;
            mx = fmaxf(mx, x[u]);
        }
        mx = lc_max_groups(mx) * scale;
        // The reference follows the maximum only when it falls behind by more than LC_DEC_LAG: the accumulators are scaled once or
        // not at all per split instead of once per step.  It is a whole number, so that scaling rounds nothing (and leaves an infinite sum one).
        if (__ballot(mx > m_ref + LAG) != 0ull) {
            const float m_new = mx > m_ref + LAG ? ceilf(mx) : m_ref;
            const int by = (int)fmaxf(m_ref - m_new, -1024.f);    // (of sums that are not zero: their reference is not -inf)
            const bool started = __ballot(m_ref > LC_NEG_INF) != 0ull;
            m_ref = m_new;
            if (started) {                                      // (before that the accumulators are zero)
                l_run = __builtin_ldexpf(l_run, by);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int by_r = __shfl(by, 4 * q4 + r);
#pragma unroll
                    for (int c = 0; c < 8; ++c) acc[c][r] = __builtin_ldexpf(acc[c][r], by_r);
                }
            }
        }
        const float ref = (m_ref == LC_NEG_INF) ? 0.f : m_ref;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const float y = fmaf(x[u], scale, -ref);
            if constexpr (PLAIN) p[u] = x[u] == LC_NEG_INF ? -0.f : exp2f(y);
            else p[u] = lc_probability(y);
        }
        float l = (p[0] + p[1]) + (p[2] + p[3]);
        if constexpr (N == 8) l += (p[4] + p[5]) + (p[6] + p[7]);
        l_run += l;
        float mn = fminf(fminf(dA[0], dA[1]), fminf(dA[2], dA[3]));            // (0 where there is no token)
        if constexpr (N == 8) mn = fminf(mn, fminf(fminf(dB[0], dB[1]), fminf(dB[2], dB[3])));
        return __ballot(fmaf(mn, scale, -ref) < LC_DEC_FAINT) != 0ull;
    };
    auto pv = [&](const lc_v4i& t, const lc_v4i& b, lc_f32x4& a) LC_INLINE {
        a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lc_bf16x8, t), __builtin_bit_cast(lc_bf16x8, b), a, 0, 0, 0);
    };
    // column c of rows v[2k], v[2k + 1], packed
    auto column = [&](const lc_v4i (&v)[U], int c, int k) LC_INLINE -> int {
        return (int)__builtin_amdgcn_perm((uint32_t)v[2 * k + 1][c / 2], (uint32_t)v[2 * k][c / 2], (c & 1) ? 0x07060302u : 0x05040100u);
    };
    // P.V: of two batches, one instruction per term of P and column; of one, the first two terms share one.  The smallest
    // terms go first: fewer roundings at full size.  (All instructions have one shape: with a 16x16x16 one adding to
    // the result of a 16x16x32 one the compiler left too few wait states between the two.)
    auto attend2 = [&](const float (&p)[2 * U], const lc_v4i (&vA)[U], const lc_v4i (&vB)[U]) LC_INLINE {
        int t[3][U];
        lc_split3<2 * U>(p, t);
#pragma unroll
        for (int c0 = 0; c0 < 8; c0 += 4) {
            lc_v4i bc[4];                                       // column c0 + c's eight tokens
#pragma unroll
            for (int c = 0; c < 4; ++c)
                bc[c] = lc_v4i{column(vA, c0 + c, 0), column(vA, c0 + c, 1), column(vB, c0 + c, 0), column(vB, c0 + c, 1)};
#pragma unroll
            for (int s = 2; s >= 0; --s)
#pragma unroll
                for (int c = 0; c < 4; ++c) pv(lc_v4i{t[s][0], t[s][1], t[s][2], t[s][3]}, bc[c], acc[c0 + c]);
        }
    };
    auto attend1 = [&](const float (&p)[U], const lc_v4i (&v)[U]) LC_INLINE {
        int t[3][U / 2];
        lc_split3<U>(p, t);
#pragma unroll
        for (int c0 = 0; c0 < 8; c0 += 4) {
            int b0[4], b1[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) { b0[c] = column(v, c0 + c, 0); b1[c] = column(v, c0 + c, 1); }
#pragma unroll
            for (int c = 0; c < 4; ++c) pv(lc_v4i{t[2][0], t[2][1], 0, 0}, lc_v4i{b0[c], b1[c], 0, 0}, acc[c0 + c]);
#pragma unroll
            for (int c = 0; c < 4; ++c) pv(lc_v4i{t[1][0], t[1][1], t[0][0], t[0][1]}, lc_v4i{b0[c], b1[c], b0[c], b1[c]}, acc[c0 + c]);
        }
    };

    // Whether any of a step's values is 2^64 or more, infinite or not a number (uniform).
    auto large = [&](const lc_v4i (&vA)[U], const lc_v4i (&vB)[U]) LC_INLINE -> bool {
        typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
        u16x2 m = {0, 0};
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, vA[u][w] & 0x7fff7fff));
                m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, vB[u][w] & 0x7fff7fff));
            }
        return __ballot(m.x >= 0x5f80 || m.y >= 0x5f80) != 0ull;
    };
    // P.V of two batches in float32 on the vector ALU: this lane's columns of its group's tokens, a head at a time, then summed over the
    // groups.  An infinite value reaches its column however little its token weighs (unless its logit is -inf).
    auto attend_plain = [&](const float (&p)[2 * U], const lc_v4i (&vA)[U], const lc_v4i (&vB)[U]) LC_INLINE {
#pragma unroll 1
        for (int g = 0; g < G; ++g) {
            float y[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) y[c] = 0.f;
#pragma unroll
            for (int u = 0; u < 2 * U; ++u) {
                float pu = __shfl(p[u], 16 * q4 + g), f = 1.f;
                if (__float_as_uint(pu) == 0u) pu = f = __builtin_ldexpf(1.f, -149);      // below float32's range: 0 but for infinite values
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const uint32_t w = (uint32_t)(u < U ? vA[u % U][c / 2] : vB[u % U][c / 2]);
                    y[c] = fmaf(pu, ((c & 1) ? lc_bf16_hi(w) : lc_bf16_lo(w)) * f, y[c]);
                }
            }
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                y[c] = lc_add_halves(y[c], y[c]);
                y[c] = lc_add_rows(y[c], y[c]);
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[c][r] += 4 * q4 + r == g ? y[c] : 0.f;
            }
        }
    };

    // The split's tokens are handled in tiles; for each tile the workgroup first writes the cache
    // row of every token into LDS, then every group streams a contiguous slice of the tile.
    auto over_tiles = [&](int split, auto stream) LC_INLINE {
        // tokens [n_tok split / S_eff, n_tok (split + 1) / S_eff), in 32 bits: with n_tok = each S_eff + more, more < S_eff <= 256
        const uint32_t each = (uint32_t)n_tok / (uint32_t)S_eff, more = (uint32_t)n_tok % (uint32_t)S_eff;
        const int lo = (int)(each * (uint32_t)split + more * (uint32_t)split / (uint32_t)S_eff);
        const int hi = (int)(each * (uint32_t)(split + 1) + more * (uint32_t)(split + 1) / (uint32_t)S_eff);
        for (int tile0 = lo; tile0 < hi; tile0 += LC_DEC_TILE) {
            const int tl = min(LC_DEC_TILE, hi - tile0);
            const int row_max = max(T - 1, 0);
            // 64 lanes per selected chunk that overlaps the tile (its lane's values are read by number)
            auto fill = [&](int o, int st, int ln) {
                const int k0 = max(o, tile0), k1 = min(o + ln, tile0 + tl);
                for (int k = k0 + lane; k < k1; k += 64) rw.row[k - tile0] = max(0, min(st + (k - o), row_max));
            };
            auto fill_round = [&](int off, int st, int ln) {
                unsigned long long mask = __ballot(ln > 0 && off < tile0 + tl && tile0 < off + ln);
                while (mask != 0ull) {
                    const int l = __ffsll((long long)mask) - 1;
                    mask &= mask - 1ull;
                    fill(lc_readlane(off, l), lc_readlane(st, l), lc_readlane(ln, l));
                }
            };
            if (tile0 != lo) lc_barrier_lds();                      // the previous tile's rows have been used
            if constexpr (FUSED) {
                fill_round(cs.base_tok + cs.off0, cs.st0, cs.ln0);
                int carry = cs.base_tok + lc_readlane(cs.off0 + cs.ln0, 63);
                for (int r = 64; r < cs.n_list; r += 64) {
                    int st, ln;
                    lc_sel_entry<LC_DEC_THREADS, EC>(cs, fused_store, r + lane, &st, &ln);
                    const int inc = lc_wave_scan_incl(ln);
                    fill_round(carry + inc - ln, st, ln);
                    carry += lc_readlane(inc, 63);
                }
                if (wave == 0 && cs.tail_ln > 0 && cs.n_sel_tok < tile0 + tl && tile0 < cs.n_sel_tok + cs.tail_ln)
                    fill(cs.n_sel_tok, cs.tail_st, cs.tail_ln);
            } else {
                auto visit = [&](int off, const int (&st)[E], const int (&ln)[E]) {
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        fill_round(off, st[e], ln[e]);
                        off += ln[e];
                    }
                };
                visit(ex0, st0, ln0);
                int carry = tot0;
                for (int base = LC_DEC_THREADS * E; base < n_runs; base += LC_DEC_THREADS * E) {
                    int st[E], ln[E], tot;
                    const int ex = lc_block_scan<LC_DEC_THREADS>(entries(base, false, st, ln), scan_sh, &tot);
                    visit(carry + ex, st, ln);
                    carry += tot;
                }
            }
            lc_barrier_lds();
            const int per = (tl + LC_DEC_GROUPS - 1) / LC_DEC_GROUPS;
            const int n_it = (per + U - 1) / U;            // the same for every wavefront: the MFMA needs all lanes
            tv = min(tl, grp * per);
            tv_end = min(tl, tv + per);
            tk = min(tl, gk * per);
            tk_end = min(tl, tk + per);
            stream(n_it);
        }
    };
    // ---- the accumulators hold the sums over the wavefront's tokens; the wavefronts meet in LDS
    // (`again`: the splits' merge is to do this split again, which it sees by a reference that is not a number: no other reference is one,
    // and with the mark in a word that is read anyway a step costs what it did; a vote of its own in LDS took 0.2 us)
    auto meet = [&](bool again) LC_INLINE {
        float l = lc_add_halves(l_run, l_run);
        l = lc_add_rows(l, l);
        if (lane < G) { ph.comb.ml[wave][lane][0] = again ? __builtin_nanf("") : m_ref; ph.comb.ml[wave][lane][1] = l; }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int g = 4 * q4 + r;
            if (g < G) {
                float4* const o = &ph.comb.acc[wave][g][2 * sub];
                o[0] = make_float4(acc[0][r], acc[1][r], acc[2][r], acc[3][r]);
                o[1] = make_float4(acc[4][r], acc[5][r], acc[6][r], acc[7][r]);
            }
        }
    };
    // one float4 slot of the split's partial per thread, stored at agent scope
    auto store_partial = [&](int split) LC_INLINE {
        float* pml = a.part_ml + ((size_t)bh * S + split) * G * 2;
        const __amdgpu_buffer_rsrc_t pacc_w = lc_buffer(a.part_acc + ((size_t)bh * S + split) * G * LC_D);
        for (int v = tid; v < G * (LC_D / 4); v += LC_DEC_THREADS) {
            const int g = v / (LC_D / 4), c4 = v % (LC_D / 4);
            float mx = LC_NEG_INF;
#pragma unroll
            for (int w = 0; w < LC_DEC_THREADS / 64; ++w) mx = __builtin_elementwise_maximum(mx, ph.comb.ml[w][g][0]);      // (hands on what is not a number)
            float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
            float den = 0.f;
            const float ref = mx == LC_NEG_INF ? 0.f : mx;
#pragma unroll
            for (int w = 0; w < LC_DEC_THREADS / 64; ++w) {
                const float sc = exp2f(ph.comb.ml[w][g][0] - ref);
                const float4 x = ph.comb.acc[w][g][c4];
                num.x = fmaf(x.x, sc, num.x); num.y = fmaf(x.y, sc, num.y);
                num.z = fmaf(x.z, sc, num.z); num.w = fmaf(x.w, sc, num.w);
                den = fmaf(ph.comb.ml[w][g][1], sc, den);
            }
            if (__builtin_expect(lc_no_number(num), 0)) {
                num = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
                for (int w = 0; w < LC_DEC_THREADS / 64; ++w) lc_add_scaled(num, ph.comb.acc[w][g][c4], exp2f(ph.comb.ml[w][g][0] - ref));
            }
            lc_store_agent4(pacc_w, v * 16, num);
            if (c4 == 0) { lc_store_agent(&pml[2 * g], mx); lc_store_agent(&pml[2 * g + 1], den); }
        }
    };

    if (s < S_eff) {
        bool again = false;                                             // (the same for the wavefront)
        over_tiles(s, [&](int n_it) LC_INLINE {
            // steps of two batches, a last one of one; a step's K rows are fetched while the step before is at its softmax and
            // P.V, its V rows behind that (batches past the last one load nothing)
            lc_v4i kA[4], vA[U], kB[4], vB[U];
            int ko[2], vo[2 * U];
            k_offsets(0, ko);
            load_k(ko, kA, kB);
            v_offsets(0, vo);
            load_v(vo, vA, vB);
            int it = 0;
            for (; it + 1 < n_it; it += 2) {
                const bool more = it + 2 < n_it;
                const lc_f32x4 dA = logits(kA), dB = logits(kB);
                if (more) { k_offsets(it + 2, ko); load_k(ko, kA, kB); }
                float p[2 * U];
                const bool faint = softmax(std::integral_constant<int, 2 * U>(), std::false_type(), it, dA, dB, p);
                if (__builtin_expect(faint, 0)) again = again || large(vA, vB);
                attend2(p, vA, vB);
                if (more) { v_offsets(it + 2, vo); load_v(vo, vA, vB); }
            }
            if (it < n_it) {
                const lc_f32x4 dA = logits(kA);
                float p[U];
                const bool faint = softmax(std::integral_constant<int, U>(), std::false_type(), it, dA, dA, p);
                if (__builtin_expect(faint, 0)) again = again || large(vA, vA);
                attend1(p, vA);
            }
        });
        meet(again);
        __syncthreads();
        store_partial(s);
    }

    // ---- the last split to arrive merges (log-sum-exp merge of the partial results)
    if (!lc_arrive_last(&ix.sync[bh * 4 + 1], S, &last_sh)) return;

    // The accumulator partials do not depend on the scales, so their loads go out first and fly while the
    // (m, l) pairs are fetched.  Every 32 lanes take one head (slot v of the output below) and turn its
    // splits' pairs into scales by themselves: no barrier until the sums meet.
    const int n_part = (n_tok > 0) ? S_eff : 0;
    // (the resource ends with the last split's partial: slots past it read 0)
    const __amdgpu_buffer_rsrc_t pacc_r = lc_buffer(a.part_acc + (size_t)bh * S * G * LC_D, n_part * G * LC_D * 4);
    const float* pml = a.part_ml + (size_t)bh * S * G * 2;
    constexpr int NV = G * (LC_D / 4);                       // float4 slots of the output
    constexpr int WAYS = (LC_DEC_THREADS / NV) > 0 ? (LC_DEC_THREADS / NV) : 1;
    constexpr int MR = (G <= 4) ? 16 : 8;                    // partials per round and thread
    const int v = tid % NV, wy = tid / NV;
    const int g = v / (LC_D / 4), c4 = v % (LC_D / 4);
    float4 x[MR];
    auto load_round = [&](int sp0) {
#pragma unroll
        for (int k = 0; k < MR; ++k)
            x[k] = lc_load_agent4(pacc_r, (((sp0 + k * WAYS) * G + g) * LC_D + 4 * c4) * 4);
    };
    const int half = tid >> 5, hl = tid & 31;
    float m_all = LC_NEG_INF, den = 0.f;
    float m0 = LC_NEG_INF, l0 = 0.f;                         // the first 32 splits (all of them unless more were asked for)
    auto fetch = [&]() LC_INLINE -> bool {                   // whether a split is to be done again (the same for the workgroup)
        load_round(wy);                                      // (by all threads: values kept from a load before would be in the way of doing splits again)
        if (hl < n_part) {
            m0 = lc_load_agent(pml + 2 * (hl * G + g));
            l0 = lc_load_agent(pml + 2 * (hl * G + g) + 1);
        }
        m_all = m0;
        bool again = m0 != m0;
        for (int sp = hl + 32; sp < n_part; sp += 32) {
            const float m = lc_load_agent(pml + 2 * (sp * G + g));
            again = again || m != m;
            m_all = fmaxf(m_all, m);
        }
        return __ballot(again) != 0ull;
    };
    if (__builtin_expect(fetch(), 0)) {
        // Splits with tokens too light for lc_split3 and large values: done here once more, one after the other, without it.
        for (int sp = 0; sp < n_part; ++sp) {
            const float mark = lc_load_agent(pml + 2 * sp * G);
            if (__ballot(mark != mark) == 0ull) continue;
            m_ref = LC_NEG_INF;
            l_run = 0.f;
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] = lc_f32x4{0.f, 0.f, 0.f, 0.f};
            __syncthreads();                                 // (everyone has the mark, and is done with the rows and sums before)
            over_tiles(sp, [&](int n_it) LC_INLINE {
#pragma unroll 1
                for (int it = 0; it < n_it; it += 2) {
                    lc_v4i kA[4], vA[U], kB[4], vB[U];
                    int ko[2], vo[2 * U];
                    k_offsets(it, ko);
                    load_k(ko, kA, kB);
                    v_offsets(it, vo);
                    load_v(vo, vA, vB);
                    float p[2 * U];
                    softmax(std::integral_constant<int, 2 * U>(), std::true_type(), it, logits(kA), logits(kB), p);
                    attend_plain(p, vA, vB);
                }
            });
            // (what lc_probability does to the others' probabilities)
            l_run *= __builtin_ldexpf(1.f, -LC_DEC_LAG);
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] *= __builtin_ldexpf(1.f, -LC_DEC_LAG);
            meet(false);
            __syncthreads();
            store_partial(sp);
            __builtin_amdgcn_s_waitcnt(0);
        }
        __syncthreads();
        fetch();
    }
    {
        m_all = fmaxf(m_all, lc_dpp<0xB1>(m_all));
        m_all = fmaxf(m_all, lc_dpp<0x4E>(m_all));
        m_all = fmaxf(m_all, lc_dpp<0x141>(m_all));
        m_all = fmaxf(m_all, lc_dpp<0x140>(m_all));
        {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(m_all), __float_as_uint(m_all), false, false);
            m_all = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
        }
        // (up to the end of the last round, where sums are zero)
        const float ref = m_all == LC_NEG_INF ? 0.f : m_all;
        const int n_slots = (n_part + MR * WAYS - 1) / (MR * WAYS) * (MR * WAYS);
        for (int sp = hl; sp < n_slots; sp += 32) {
            float ms = m0, ls = l0;
            if (sp >= 32) {
                ms = sp < n_part ? lc_load_agent(pml + 2 * (sp * G + g)) : LC_NEG_INF;
                ls = sp < n_part ? lc_load_agent(pml + 2 * (sp * G + g) + 1) : 0.f;
            }
            const float sc = exp2f(ms - ref);
            ph.scale[half][sp] = sc;
            den = fmaf(ls, sc, den);
        }
        den = lc_sum16(den);
        den = lc_add_rows(den, den);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    float4 acc4 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (wy < WAYS) {
        for (int sp0 = wy; sp0 < n_part; sp0 += MR * WAYS) {
            if (sp0 != wy) load_round(sp0);
#pragma unroll
            for (int k = 0; k < MR; ++k) {
                const int sp = sp0 + k * WAYS;
                const float sc = ph.scale[half][sp];
                acc4.x = fmaf(x[k].x, sc, acc4.x);
                acc4.y = fmaf(x[k].y, sc, acc4.y);
                acc4.z = fmaf(x[k].z, sc, acc4.z);
                acc4.w = fmaf(x[k].w, sc, acc4.w);
            }
        }
        if (__builtin_expect(lc_no_number(acc4), 0)) {
            acc4 = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
            for (int sp = wy; sp < n_part; sp += WAYS)
                lc_add_scaled(acc4, lc_load_agent4(pacc_r, ((sp * G + g) * LC_D + 4 * c4) * 4), ph.scale[half][sp]);
        }
        if (WAYS > 1 && wy > 0) rw.red[(wy - 1) * NV + v] = acc4;
    }
    __syncthreads();
    if (wy == 0) {
#pragma unroll
        for (int k = 1; k < WAYS; ++k) {
            const float4 o4 = rw.red[(k - 1) * NV + v];
            acc4.x += o4.x; acc4.y += o4.y; acc4.z += o4.z; acc4.w += o4.w;
        }
        const float inv = den > 0.f ? 1.0f / den : 0.f;
        const size_t o = ((size_t)b * ix.H * G + (size_t)h * G + g);
        *reinterpret_cast<float4*>(a.out + o * LC_D + 4 * c4) =
            make_float4(acc4.x * inv, acc4.y * inv, acc4.z * inv, acc4.w * inv);
        if (a.lse && c4 == 0) {
            int e;                                              // (whole powers of two aside, the logarithm is of a number near 1)
            const float part = frexpf(den, &e);
            a.lse[o] = den > 0.f ? fmaf(m_all + (float)(e + LC_DEC_LAG), LC_LN2, logf(part)) : LC_NEG_INF;
        }
    }
    if (tid == 0) ix.sync[bh * 4 + 1] = 0;
    if (SCORE == LC_SCORED_SHARED && tid == 0) {                 // (every workgroup has read the number: it arrives behind that)
        const int number = ix.sync[bh * 4 + 3];
        ix.sync[bh * 4 + 3] = number == -1 ? 1 : (int)((uint32_t)number + 1u);
    }
}

template <int G>
static int launch_decode_g(const LcDecodeArgs& a, int splits, hipStream_t stream) {
    hipLaunchKernelGGL((lc_decode_kernel<G, false, 1, LC_SCORED_BEFORE>), dim3(splits, a.ix.H, a.ix.B), dim3(LC_DEC_THREADS), 0, stream, a);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}

static void fill_common(LcDecodeArgs& a, const lc_index* idx, const LcWs& ws, const void* q, const void* K,
                        const void* V, const int64_t ks[3], float* out, float* lse) {
    a.ix = idx->dev;
    a.q = static_cast<const uint16_t*>(q);
    a.K = static_cast<const uint16_t*>(K);
    a.V = static_cast<const uint16_t*>(V);
    a.ks_seq = ks[0];
    a.ks_head = ks[1];
    a.ks_tok = ks[2];
    a.ids = nullptr;
    a.counts = nullptr;
    a.cap = 0;
    a.part_acc = ws.part_acc;
    a.part_ml = ws.part_ml;
    a.out = out;
    a.lse = lse;
    a.entries = nullptr;
    a.ids_out = nullptr;
    a.counts_out = nullptr;
    a.budget = 0;
    a.sink = 0;
    a.ew = 0;
    a.share = 0;
    a.max_tokens = idx->cfg.max_tokens;
}

int lc_launch_decode(const lc_index* idx, const LcWs& ws, const void* q, const void* K, const void* V,
                     const int64_t ks[3], const int32_t* ids, const int32_t* counts, int cap, int G,
                     int splits, float* out, float* lse, hipStream_t stream) {
    LcDecodeArgs a;
    fill_common(a, idx, ws, q, K, V, ks, out, lse);
    a.ids = ids;
    a.counts = counts;
    a.cap = cap;
    switch (G) {
        case 1: return launch_decode_g<1>(a, splits, stream);
        case 2: return launch_decode_g<2>(a, splits, stream);
        case 3: return launch_decode_g<3>(a, splits, stream);
        case 4: return launch_decode_g<4>(a, splits, stream);
        case 5: return launch_decode_g<5>(a, splits, stream);
        case 6: return launch_decode_g<6>(a, splits, stream);
        case 7: return launch_decode_g<7>(a, splits, stream);
        case 8: return launch_decode_g<8>(a, splits, stream);
    }
    return LC_ERR_BAD_SHAPE;
}

// ---- fused step
// Rows of 64 chunks per wavefront that the kernel instances hold in registers: a (sequence, head)
// with up to 256 * EC chunks runs in the smallest instance that holds it.
#define LC_DEC_EC_MAX 16

bool lc_decode_fused_fits(int G, int max_M) {
    return G >= 1 && G <= LC_MAX_GROUP && max_M <= LC_DEC_THREADS * LC_DEC_EC_MAX;
}

template <int G, int EC, int SCORE>
static int launch_fused_ge(const LcDecodeArgs& a, int splits, hipStream_t stream) {
    const size_t lds = lc_select_lds<LC_DEC_THREADS, EC>();   // the selection's chunk lists
    if (lds > 16 * 1024) {      // static + dynamic may pass the default per-workgroup allowance: raised once per device
        static LcOnce raised;
        LC_HIP_CHECK(raised.run([&] {
            return hipFuncSetAttribute(reinterpret_cast<const void*>(&lc_decode_kernel<G, true, EC, SCORE>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        }));
    }
    hipLaunchKernelGGL((lc_decode_kernel<G, true, EC, SCORE>), dim3(splits, a.ix.H, a.ix.B), dim3(LC_DEC_THREADS), lds, stream, a);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}
template <int G>
static int launch_fused_g(const LcDecodeArgs& a, int scoring, int splits, hipStream_t stream) {
    if (scoring == LC_SCORED_HERE) return launch_fused_ge<G, 1, LC_SCORED_HERE>(a, splits, stream);
    if (scoring == LC_SCORED_SHARED) {
        static_assert(LC_STEP_SHARE_MAX_CHUNKS <= 10 * LC_DEC_THREADS, "");
        if (a.ew <= 2) return launch_fused_ge<G, 2, LC_SCORED_SHARED>(a, splits, stream);
        if (a.ew <= 4) return launch_fused_ge<G, 4, LC_SCORED_SHARED>(a, splits, stream);
        if (a.ew <= 6) return launch_fused_ge<G, 6, LC_SCORED_SHARED>(a, splits, stream);
        return launch_fused_ge<G, 10, LC_SCORED_SHARED>(a, splits, stream);
    }
    if (a.ew <= 2) return launch_fused_ge<G, 2, LC_SCORED_BEFORE>(a, splits, stream);
    if (a.ew <= 4) return launch_fused_ge<G, 4, LC_SCORED_BEFORE>(a, splits, stream);
    if (a.ew <= 6) return launch_fused_ge<G, 6, LC_SCORED_BEFORE>(a, splits, stream);
    if (a.ew <= 10) return launch_fused_ge<G, 10, LC_SCORED_BEFORE>(a, splits, stream);
    return launch_fused_ge<G, LC_DEC_EC_MAX, LC_SCORED_BEFORE>(a, splits, stream);
}

int lc_launch_decode_fused(const lc_index* idx, const LcWs& ws, const void* q, const void* K, const void* V,
                           const int64_t ks[3], int G, int splits, int budget, int32_t* ids_out,
                           int32_t* counts_out, int cap, int max_M, bool single, float* out, float* lse,
                           hipStream_t stream) {
    LcDecodeArgs a;
    fill_common(a, idx, ws, q, K, V, ks, out, lse);
    a.entries = ws.scratch;
    const int scoring = !single ? LC_SCORED_BEFORE
                                : (lc_step_is_single(max_M, G, (long long)idx->B * idx->H_kv * splits) ? LC_SCORED_HERE : LC_SCORED_SHARED);
    if (scoring == LC_SCORED_HERE && max_M > LC_STEP_SINGLE_MAX_CHUNKS) return LC_ERR_CAPACITY;
    a.share = ((max_M + splits - 1) / splits + 3) / 4 * 4;
    if (scoring == LC_SCORED_SHARED && (a.share > LC_STEP_SHARE_CHUNKS || max_M > LC_STEP_SHARE_MAX_CHUNKS)) return LC_ERR_CAPACITY;
    a.ids_out = ids_out;
    a.counts_out = counts_out;
    a.cap = cap;
    a.budget = budget;
    a.sink = idx->cfg.sink_tokens;
    a.ew = ((max_M > 0 ? max_M : 1) + LC_DEC_THREADS - 1) / LC_DEC_THREADS;
    if (a.ew > LC_DEC_EC_MAX) return LC_ERR_CAPACITY;
    switch (G) {
        case 1: return launch_fused_g<1>(a, scoring, splits, stream);
        case 2: return launch_fused_g<2>(a, scoring, splits, stream);
        case 3: return launch_fused_g<3>(a, scoring, splits, stream);
        case 4: return launch_fused_g<4>(a, scoring, splits, stream);
        case 5: return launch_fused_g<5>(a, scoring, splits, stream);
        case 6: return launch_fused_g<6>(a, scoring, splits, stream);
        case 7: return launch_fused_g<7>(a, scoring, splits, stream);
        case 8: return launch_fused_g<8>(a, scoring, splits, stream);
    }
    return LC_ERR_BAD_SHAPE;
}
