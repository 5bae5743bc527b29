// Index construction (prefill side) and the lazy update for streamed tokens.
//
// Build, per (sequence, KV head):
//   lc_pool_kernel    chunk representative = mean-pooled keys; covering radius; unit direction
//   lc_kmeans_*       spherical k-means on unit directions: strided start, then
//                     `iters` x (assign by largest inner product, normalised-sum update)
//   lc_kmeans_rounds_kernel  all iterations of a level, and its nodes, in one kernel of several workgroups per (sequence, head)
//   lc_center_*       node center (mean of all descendant chunks), counts, direction (small levels: in lc_kmeans_small_kernel)
//   lc_radius_kernel  radii of every level over all descendant chunks' balls, after the last level
// Append: lc_append_kernel writes the token's k, v; on a chunk close it pools the
// open tail, finds the level-1 node of nearest direction and updates the path to the top.
//
// Every reduction runs in a fixed order, so results are reproducible run to run.
#include "lc_device.h"
#include "lc_internal.h"
#include "lc_rounds_planes.h"
#include "lc_select.h"

#include <algorithm>
#include <type_traits>

#define LC_INLINE __attribute__((always_inline))       // (lambdas that hold registers by reference)

#define LC_BT 256                 // threads per block
#define LC_BG (LC_BT / 16)        // 16-lane groups per block
#define LC_RADIUS_PAD 4e-6f       // stored radii are inflated by this relative amount so that
                                  // float32 rounding in the distance never leaves a member outside

__device__ __forceinline__ float lc_pad_radius(float r) { return r > 0.f ? r * (1.0f + LC_RADIUS_PAD) : r; }

// ---------------------------------------------------------------------------------
// pooling of rows [lo, hi) of one (sequence, head) key cache; block-wide.
// On return every lane holds, for its 8 columns [8 sub, 8 sub + 8), the stored center
// `mu` (rounded to bfloat16 first if the chunk level is stored that way, so that the radius
// covers the tokens around the value that is stored), and all threads hold the stored radius.
// sh: LC_BG * 128 + LC_BG floats.
// ---------------------------------------------------------------------------------
#define LC_POOL_KEEP 8            // rows per 16-lane group that stay in registers between the two passes (chunks up to 128 tokens are read once)
__device__ __forceinline__ void lc_pool_rows(const uint16_t* __restrict__ Kbh, long long ks_tok, int lo, int hi,
                                             int geometry, bool round_bf16, float* sh, float (&mu)[8], float* radius) {
    const int tid = threadIdx.x, sub = tid & 15, grp = tid >> 4;
    float sum[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) sum[i] = 0.f;
    uint4 keep[LC_POOL_KEEP];
#pragma unroll
    for (int k = 0; k < LC_POOL_KEEP; ++k) {
        const int r = lo + grp + k * LC_BG;
        keep[k] = make_uint4(0u, 0u, 0u, 0u);
        if (r < hi) keep[k] = *reinterpret_cast<const uint4*>(Kbh + (long long)r * ks_tok + 8 * sub);
    }
#pragma unroll
    for (int k = 0; k < LC_POOL_KEEP; ++k) {          // (rows past the chunk hold zeros: they add nothing)
        float f[8];
        lc_unpack8(keep[k], f);
#pragma unroll
        for (int i = 0; i < 8; ++i) sum[i] += f[i];
    }
    for (int r = lo + grp + LC_POOL_KEEP * LC_BG; r < hi; r += LC_BG) {
        const uint4 v = *reinterpret_cast<const uint4*>(Kbh + (long long)r * ks_tok + 8 * sub);
        float f[8];
        lc_unpack8(v, f);
#pragma unroll
        for (int i = 0; i < 8; ++i) sum[i] += f[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) sh[grp * LC_D + 8 * sub + i] = sum[i];
    __syncthreads();
    const float inv_n = 1.0f / (float)(hi - lo);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float s = 0.f;
        for (int g = 0; g < LC_BG; ++g) s += sh[g * LC_D + 8 * sub + i];
        mu[i] = s * inv_n;
    }
    if (geometry == LC_GEOMETRY_PAPER_UNIT) {
        float n2 = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) n2 = fmaf(mu[i], mu[i], n2);
        n2 = lc_sum16(n2);
        if (n2 > 0.f) {
            const float inv = 1.0f / sqrtf(n2);
#pragma unroll
            for (int i = 0; i < 8; ++i) mu[i] *= inv;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) mu[i] = (sub == 0 && i == 0) ? 1.f : 0.f;
        }
        if (round_bf16) {
#pragma unroll
            for (int i = 0; i < 8; ++i) mu[i] = lc_round_bf16(mu[i]);
        }
        *radius = 0.f;
        __syncthreads();
        return;
    }
    if (round_bf16) {
#pragma unroll
        for (int i = 0; i < 8; ++i) mu[i] = lc_round_bf16(mu[i]);
    }
    float far2 = 0.f;
    auto reach = [&](const uint4& v) {
        float f[8];
        lc_unpack8(v, f);
        float d2 = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) { const float t = f[i] - mu[i]; d2 = fmaf(t, t, d2); }
        d2 = lc_sum16(d2);
        far2 = fmaxf(far2, d2);
    };
#pragma unroll
    for (int k = 0; k < LC_POOL_KEEP; ++k)
        if (lo + grp + k * LC_BG < hi) reach(keep[k]);
    for (int r = lo + grp + LC_POOL_KEEP * LC_BG; r < hi; r += LC_BG)
        reach(*reinterpret_cast<const uint4*>(Kbh + (long long)r * ks_tok + 8 * sub));
    __syncthreads();
    if (sub == 0) sh[grp] = far2;
    __syncthreads();
    float mx = 0.f;
    for (int g = 0; g < LC_BG; ++g) mx = fmaxf(mx, sh[g]);
    *radius = lc_pad_radius(sqrtf(mx));
    __syncthreads();
}

// unit direction of the 8-column fragments (zero vector -> e_0)
__device__ __forceinline__ void lc_unit_frag(const float (&v)[8], int sub, float (&u)[8]) {
    float n2 = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) n2 = fmaf(v[i], v[i], n2);
    n2 = lc_sum16(n2);
    if (n2 > 0.f) {
        const float inv = 1.0f / sqrtf(n2);
#pragma unroll
        for (int i = 0; i < 8; ++i) u[i] = v[i] * inv;
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) u[i] = (sub == 0 && i == 0) ? 1.f : 0.f;
    }
}

__device__ __forceinline__ void lc_store8(float* p, const float (&v)[8]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
// the same 8 columns of a direction rounded to bfloat16 (16 bytes per lane); its not-a-numbers are the hardware's own
// (lc_unit_frag), which rounding keeps
__device__ __forceinline__ void lc_store8_bf16(uint16_t* p, const float (&v)[8]) {
    uint32_t h[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = lc_f32_to_bf16_bits(v[i]);
    *reinterpret_cast<uint4*>(p) = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
}
template <typename Acc>
__device__ __forceinline__ void lc_store_acc8(Acc* p, const Acc (&v)[8]) {
#pragma unroll
    for (int t = 0; t < 8; ++t) p[t] = v[t];
}
__device__ __forceinline__ void lc_load8(const float* p, float (&v)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// Chunk-level center of node n, columns [8 sub, 8 sub + 8), in the index's storage format.
// (`v` already holds bfloat16-representable values when the level is stored as bfloat16.)
__device__ __forceinline__ void lc_c0_store8(const LcDev& ix, size_t n, int sub, const float (&v)[8]) {
    if (ix.c0_bf16) {
        uint4 w;
        w.x = (__float_as_uint(v[0]) >> 16) | (__float_as_uint(v[1]) & 0xffff0000u);
        w.y = (__float_as_uint(v[2]) >> 16) | (__float_as_uint(v[3]) & 0xffff0000u);
        w.z = (__float_as_uint(v[4]) >> 16) | (__float_as_uint(v[5]) & 0xffff0000u);
        w.w = (__float_as_uint(v[6]) >> 16) | (__float_as_uint(v[7]) & 0xffff0000u);
        *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(ix.center[0]) + n * LC_D + 8 * sub) = w;
    } else {
        lc_store8(ix.center[0] + n * LC_D + 8 * sub, v);
    }
}
__device__ __forceinline__ void lc_c0_load8(const LcDev& ix, size_t n, int sub, float (&v)[8]) {
    if (ix.c0_bf16) {
        const uint4 w = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(ix.center[0]) + n * LC_D + 8 * sub);
        lc_unpack8(w, v);
    } else {
        lc_load8(ix.center[0] + n * LC_D + 8 * sub, v);
    }
}

// ---------------------------------------------------------------------------------
// level 0: one wavefront per chunk
// ---------------------------------------------------------------------------------
// The four 16-lane groups of a wavefront take the chunk's rows in turn (lane `sub` of a group holds
// columns [8 sub, 8 sub + 8) of a row), LC_POOLW_KEEP rows per group to a batch.  The bound is reading K once; the radius pass needs every
// row again.  The first two batches are loaded together and stay in registers for it, the third waits in LDS (8 KB a wavefront, as
// many as leave the resident count to the registers): chunks of up to 96 tokens read K once, longer ones find the rest in the
// caches.  Instructions were the other half of the time -- 1261 per chunk of 57 rows --: the sums are the matrix cores' work, range-checked
// loads zero the rows past the chunk, eight rows' distances are reduced over the lanes together.  One wavefront per workgroup, so
// that a long chunk holds up no neighbour's place.  268 MB of K in 128K tokens x 8 heads, 57 to a chunk: 72 us with sums by
// addition, one batch in registers and seven rows per group in LDS; 69 us with two and none; 62 us now (292 MB with what is
// written: 4.7 TB/s).  16 sequences of ragged length: 157 us, now 143 (734 MB: 5.1 TB/s).  Chunks of 8 to 16 tokens: 130 and 118 us.
#define LC_POOLW_KEEP 8
typedef __bf16 lc_bf16x8_p __attribute__((ext_vector_type(8)));
typedef float lc_f32x4_p __attribute__((ext_vector_type(4)));
// Progress flags of the k-means of every level, [level][sequence, head][LC_KM_FLAGS]: cleared by the first kernel of a build.
__device__ __forceinline__ int* lc_level_flags(const LcDev& ix, int* flags, int l, int bh) {
    return flags + ((size_t)l * ix.B * ix.H + bh) * LC_KM_FLAGS;
}
// Centroid c of a clustering of N points into k starts at point floor(c * N / k).  The kernels that write a
// level's points also write the rows of those that start a centroid (c <= k <= N, so a point starts at most
// one): the cluster that point i of N starts, or -1.
__device__ __forceinline__ int lc_seed_of(int i, int N, int k) {
    if ((long long)N * k < (1ll << 31)) {                           // (64-bit divisions are long routines)
        const unsigned c = ((unsigned)i * (unsigned)k + (unsigned)N - 1u) / (unsigned)N;
        return c < (unsigned)k && c * (unsigned)N / (unsigned)k == (unsigned)i ? (int)c : -1;
    }
    const long long c = ((long long)i * k + N - 1) / N;
    return c < k && (c * N) / k == i ? (int)c : -1;
}
// unit direction of point i (8 columns per lane): float32 and bfloat16 rows, and the centroid it starts
struct LcPointRows {
    float* pts;              // [B][H][cap][d]
    uint16_t* pts16;
    int cap;
    float* cent;             // [B][H][cent_cap][d]; null if the level is not clustered
    uint16_t* cent16;
    int cent_cap;
};
__device__ __forceinline__ void lc_store_point(const LcPointRows& w, int bh, int i, int N, int k, int sub, const float (&u)[8]) {
    const size_t o = ((size_t)bh * w.cap + i) * LC_D + 8 * sub;
    lc_store8(w.pts + o, u);
    lc_store8_bf16(w.pts16 + o, u);
    const int c = w.cent ? lc_seed_of(i, N, k) : -1;
    if (c >= 0) {
        const size_t q = ((size_t)bh * w.cent_cap + c) * LC_D + 8 * sub;
        lc_store8(w.cent + q, u);
        lc_store8_bf16(w.cent16 + q, u);
    }
}
__device__ __forceinline__ void lc_clear_flags(const LcDev& ix, int bh, int* flags) {
    if (blockIdx.x == 0 && threadIdx.x < LC_KM_FLAGS)
        for (int l = 0; l + 1 < ix.L; ++l) lc_level_flags(ix, flags, l, bh)[threadIdx.x] = 0;
}
// What the workgroups of lc_kmeans_rounds_kernel post for each other: in a first kernel's hands only the part that it marks as not posted yet.
struct LcUnposted {
    lc_v4i* at;              // 16-byte pieces
    int n;
};
#define LC_UNPOSTED (-1)     // the bits of no label and of no number that an update makes (its not-a-numbers are the hardware's own)
template <int NT>
__device__ __forceinline__ void lc_clear_posts(const LcUnposted& u) {
    if (u.n == 0) return;
    const int blocks = gridDim.x * gridDim.y * gridDim.z;
    const int per = (u.n + blocks - 1) / blocks;                    // a run of pieces for each workgroup
    const int first = (int)(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)) * per;
    const int end = min(first + per, u.n);
    for (int i = first + (int)threadIdx.x; i < end; i += NT) u.at[i] = lc_v4i{LC_UNPOSTED, LC_UNPOSTED, LC_UNPOSTED, LC_UNPOSTED};
}
__device__ __forceinline__ float lc_sum_groups4(float v) { v += __shfl_xor(v, 16); v += __shfl_xor(v, 32); return v; }
// A batch of rows, row base + 4 k + (lane / 16) of it in buf[k]; rows past the chunk read as zeros, all loads in flight together.  NEAR:
// a batch lies within a range-checked buffer (rows of 256 bytes or more that do not overlap, 31 bits of offset), whose
// checks replace the zeroing and whose addresses are one addition each.
template <bool NEAR>
__device__ __forceinline__ void lc_pool_batch(const uint16_t* Kbh, long long ks_tok, int base, int hi, lc_v4i (&buf)[LC_POOLW_KEEP]) {
    const int lane = threadIdx.x & 63, sub = lane & 15, g4 = lane >> 4;
    if constexpr (NEAR) {
        const int row = (int)ks_tok * 2, rows = min(hi - base, 4 * LC_POOLW_KEEP);
        const __amdgpu_buffer_rsrc_t r = lc_buffer(Kbh + (long long)base * ks_tok, rows > 0 ? (rows - 1) * row + 2 * LC_D : 0);
        const int at = g4 * row + 16 * sub;
#pragma unroll
        for (int k = 0; k < LC_POOLW_KEEP; ++k) buf[k] = __builtin_amdgcn_raw_buffer_load_b128(r, at + 4 * k * row, 0, 0);
    } else {
#pragma unroll
        for (int k = 0; k < LC_POOLW_KEEP; ++k) {
            const int r = base + g4 + 4 * k;
            const lc_v4i v = *reinterpret_cast<const lc_v4i*>(Kbh + (long long)max(min(r, hi - 1), 0) * ks_tok + 8 * sub);
            buf[k] = r < hi ? v : lc_v4i{0, 0, 0, 0};
        }
    }
}
template <bool NEAR>
__global__ void __launch_bounds__(64)
lc_pool_kernel(LcDev ix, const uint16_t* K, long long ks_seq, long long ks_head, long long ks_tok,
               int geometry, LcPointRows out, int* flags, LcUnposted unposted) {
    lc_fetch_args<sizeof(LcDev) + 40 + sizeof(LcPointRows)>();
    const int h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    lc_clear_flags(ix, bh, flags);
    lc_clear_posts<64>(unposted);
    const int lane = threadIdx.x & 63, sub = lane & 15, g4 = lane >> 4;
    const int j = blockIdx.x;
    const int M = ix.state[bh * 4 + 1];
    if (j >= M) return;                                            // (whole wavefronts leave: nothing below waits across them)
    const int* bnd = ix.bounds + (size_t)b * (ix.cap[0] + 1);
    const int lo = bnd[j], hi = bnd[j + 1];
    const uint16_t* Kbh = K + b * ks_seq + h * ks_head;
    const bool round_bf16 = ix.c0_bf16 != 0;
    constexpr int ROWS = 4 * LC_POOLW_KEEP;
    __shared__ lc_v4i parked[LC_POOLW_KEEP][64];                    // (a lane reads its own entries only)
    lc_v4i keep[LC_POOLW_KEEP], second[LC_POOLW_KEEP];
    lc_pool_batch<NEAR>(Kbh, ks_tok, lo, hi, keep);
    const bool two = hi - lo > ROWS;                                // (uniform)
    if (two) lc_pool_batch<NEAR>(Kbh, ks_tok, lo + ROWS, hi, second);
    // ---- sums over the rows, on the matrix cores: a lane's registers as they are loaded are column `sub` of a B operand whose 32
    // rows are (row of K of this group of lanes, column 8 sub + t); the A operand picks t = i mod 8.  Row 4 g4 + r of the result
    // is the sum of column 8 sub + (4 g4 + r) mod 8: products by one and zero are exact, sums are float32.
    const int t = sub & 7, one = (t & 1) ? 0x3f800000 : 0x00003f80;
    const lc_v4i pick = lc_v4i{t >> 1 == 0 ? one : 0, t >> 1 == 1 ? one : 0, t >> 1 == 2 ? one : 0, t >> 1 == 3 ? one : 0};
    lc_f32x4_p acc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = lc_f32x4_p{0.f, 0.f, 0.f, 0.f};
    auto add_batch = [&](const lc_v4i (&buf)[LC_POOLW_KEEP]) LC_INLINE {
#pragma unroll
        for (int k = 0; k < LC_POOLW_KEEP; ++k)                     // (zero rows add nothing)
            acc[k & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lc_bf16x8_p, pick),
                                                                 __builtin_bit_cast(lc_bf16x8_p, buf[k]), acc[k & 3], 0, 0, 0);
    };
    add_batch(keep);
    if (two) {
        add_batch(second);
        for (int base = lo + 2 * ROWS; base < hi; base += ROWS) {
            lc_v4i more[LC_POOLW_KEEP];
            lc_pool_batch<NEAR>(Kbh, ks_tok, base, hi, more);
            add_batch(more);
            if (base == lo + 2 * ROWS) {
#pragma unroll
                for (int k = 0; k < LC_POOLW_KEEP; ++k) parked[k][lane] = more[k];
            }
        }
    }
    float mu[8];
    const float inv_n = 1.0f / (float)(hi - lo);
    {
        float z = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float s = (acc[0][r] + acc[1][r]) + (acc[2][r] + acc[3][r]), o = __shfl_xor(s, 16);
            mu[r] = (g4 & 1) ? o : s;
            mu[4 + r] = (g4 & 1) ? s : o;
            z += s - s;
        }
        if (__ballot(!(z == 0.f)) != 0ull) {
            // infinities and what is no number (times zero, they have reached their neighbours' sums): column by column
            float sum[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) sum[i] = 0.f;
            for (int r = lo + g4; r < hi; r += 4) {
                float f[8];
                lc_unpack8(*reinterpret_cast<const uint4*>(Kbh + (long long)r * ks_tok + 8 * sub), f);
#pragma unroll
                for (int i = 0; i < 8; ++i) sum[i] += f[i];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) mu[i] = lc_sum_groups4(sum[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) mu[i] *= inv_n;
    float radius = 0.f;
    if (geometry == LC_GEOMETRY_PAPER_UNIT) {
        float un[8];
        lc_unit_frag(mu, sub, un);
#pragma unroll
        for (int i = 0; i < 8; ++i) mu[i] = round_bf16 ? lc_round_bf16(un[i]) : un[i];
    } else {
        if (round_bf16) {
#pragma unroll
            for (int i = 0; i < 8; ++i) mu[i] = lc_round_bf16(mu[i]);
        }
        float far2 = 0.f;
        // Squared distances of a batch's rows.  Eight rows' parts are reduced over the 16 lanes together: at each of three steps a
        // lane passes on the half of them that its partner goes on with, and ends with one row's, number 4 (sub bit 1) + 2 (bit 2) + (bit 3).
        const bool b3 = (sub & 8) != 0, b2 = (sub & 4) != 0, b1 = (sub & 2) != 0;
        const int mine = g4 + 4 * ((b1 ? 4 : 0) + (b2 ? 2 : 0) + (b3 ? 1 : 0));
        auto reach = [&](const lc_v4i (&buf)[LC_POOLW_KEEP], int n) LC_INLINE {
            float d[LC_POOLW_KEEP];
#pragma unroll
            for (int k = 0; k < LC_POOLW_KEEP; ++k) {
                d[k] = 0.f;
                if (4 * k < n) {                                    // (uniform)
                    float f[8];
                    lc_unpack8(__builtin_bit_cast(uint4, buf[k]), f);
#pragma unroll
                    for (int i = 0; i < 8; ++i) { const float x = f[i] - mu[i]; d[k] = fmaf(x, x, d[k]); }
                }
            }
            static_assert(LC_POOLW_KEEP == 8, "three halvings");
#pragma unroll
            for (int k = 0; k < 4; ++k) { const float give = b3 ? d[2 * k] : d[2 * k + 1]; d[k] = (b3 ? d[2 * k + 1] : d[2 * k]) + lc_dpp<0x140>(give); }
#pragma unroll
            for (int k = 0; k < 2; ++k) { const float give = b2 ? d[2 * k] : d[2 * k + 1]; d[k] = (b2 ? d[2 * k + 1] : d[2 * k]) + lc_dpp<0x141>(give); }
            const float give = b1 ? d[0] : d[1];
            float v = (b1 ? d[1] : d[0]) + lc_dpp<0x4E>(give);
            v += lc_dpp<0xB1>(v);
            far2 = mine < n ? fmaxf(far2, v) : far2;
        };
        reach(keep, hi - lo);
        if (two) {
            reach(second, hi - lo - ROWS);
            for (int base = lo + 2 * ROWS; base < hi; base += ROWS) {
                lc_v4i more[LC_POOLW_KEEP];
                if (base == lo + 2 * ROWS) {
#pragma unroll
                    for (int k = 0; k < LC_POOLW_KEEP; ++k) more[k] = parked[k][lane];
                } else {
                    lc_pool_batch<NEAR>(Kbh, ks_tok, base, hi, more);
                }
                reach(more, hi - base);
            }
        }
        far2 = fmaxf(far2, lc_dpp<0x4E>(far2));
        far2 = fmaxf(far2, lc_dpp<0x141>(far2));
        far2 = fmaxf(far2, lc_dpp<0x140>(far2));
        far2 = fmaxf(far2, __shfl_xor(far2, 16));
        far2 = fmaxf(far2, __shfl_xor(far2, 32));
        radius = lc_pad_radius(sqrtf(far2));
    }
    const size_t n = (size_t)bh * ix.cap[0] + j;
    if (g4 == 0) {
        lc_c0_store8(ix, n, sub, mu);
        float u[8];
        lc_unit_frag(mu, sub, u);
        lc_store_point(out, bh, j, M, ix.L > 1 ? ix.nlev[b * LC_MAX_LEVELS + 1] : 0, sub, u);
        if (sub == 0) {
            ix.radius[0][n] = radius;
            ix.parent[0][n] = -1;
            ix.ntok[0][n] = hi - lo;
            ix.nchunk[0][n] = 1;
        }
    }
}

// Re-clustering starts from the chunk nodes already in the index: unit directions of their centers.
__global__ void __launch_bounds__(LC_BT)
lc_dirs_kernel(LcDev ix, LcPointRows out, int* flags, LcUnposted unposted) {
    lc_fetch_args<sizeof(LcDev) + sizeof(LcPointRows)>();
    const int h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    lc_clear_flags(ix, bh, flags);
    lc_clear_posts<LC_BT>(unposted);
    const int M = ix.state[bh * 4 + 1];
    const int sub = threadIdx.x & 15;
    const int j = blockIdx.x * LC_BG + (threadIdx.x >> 4);
    if (j >= M) return;
    const size_t n = (size_t)bh * ix.cap[0] + j;
    float mu[8], u[8];
    lc_c0_load8(ix, n, sub, mu);
    lc_unit_frag(mu, sub, u);
    lc_store_point(out, bh, j, M, ix.L > 1 ? ix.nlev[b * LC_MAX_LEVELS + 1] : 0, sub, u);
    if (sub == 0) ix.parent[0][n] = -1;
}

// ---------------------------------------------------------------------------------
// spherical k-means
// ---------------------------------------------------------------------------------
// Number of points / clusters of sequence b when clustering level `l` into level l+1.
__device__ __forceinline__ int lc_level_count(const LcDev& ix, int b, int bh, int l) {
    return l == 0 ? ix.state[bh * 4 + 1] : ix.nlev[b * LC_MAX_LEVELS + l];
}

// label(i) = argmax_c <x_i, m_c>, ties to the lower c: the one dense contraction of the build
// (N x k x 128 per iteration), on the matrix cores.  The similarities that decide are float32
// (v_mfma_f32_16x16x4_f32); which of them are needed at all is found with bfloat16 ones at a sixteenth of
// the cost (lc_kmeans_assign_kernel).
// Float32 blocks: a wavefront takes 16 points (the A operand) and 16 centroids (the B operand).  Both
// operands walk the 128 dimensions in the same permuted order -- step (t, u) pairs dimension
// 16 t + 4 kk + u of a point with the same dimension of a centroid, kk = lane / 16 being the
// instruction's K index -- so that each lane fetches its share of a row as eight 16-byte pieces.  The
// result tile leaves lane (q, j) with the similarities of points 4 q + r (r < 4) to centroid j of the
// block; every lane keeps the best of its column per point, and the 16 lanes of a row merge (value, then
// lower id) at the end.
#define LC_AS_ROW (LC_D + 4)      // floats per staged centroid row (the pad spreads the 16 rows of a block over the banks)
typedef float lc_f32x4_b __attribute__((ext_vector_type(4)));
// One 16 x 16 block of similarities: the wavefront's 16 points (xa, the A operand) against the 16
// centroid rows of which `brow` is this lane's (already offset by 4 * kk); lane j's centroid has id c.
__device__ __forceinline__ void lc_assign_block(const float4 (&xa)[8], const float* brow, int c, int k,
                                                float (&best)[4], int (&arg)[4]) {
    lc_f32x4_b d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float4 mb = *reinterpret_cast<const float4*>(brow + 16 * t);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].x, mb.x, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].y, mb.y, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].z, mb.z, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].w, mb.w, d, 0, 0, 0);
    }
    if (c < k) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (d[r] > best[r]) { best[r] = d[r]; arg[r] = c; }
    }
}
// Two blocks at once: the two accumulators are independent chains, so the matrix pipe is not left
// waiting for one instruction's result before the next can start (a wavefront is alone on its
// SIMD here).  Each block's own sum runs in the same order as in lc_assign_block: same bits.
__device__ __forceinline__ void lc_assign_block2(const float4 (&xa)[8], const float* brow0, const float* brow1,
                                                 int c0, int c1, int k, float (&best)[4], int (&arg)[4]) {
    lc_f32x4_b d0 = {0.f, 0.f, 0.f, 0.f}, d1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float4 m0 = *reinterpret_cast<const float4*>(brow0 + 16 * t);
        const float4 m1 = *reinterpret_cast<const float4*>(brow1 + 16 * t);
        d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].x, m0.x, d0, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].x, m1.x, d1, 0, 0, 0);
        d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].y, m0.y, d0, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].y, m1.y, d1, 0, 0, 0);
        d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].z, m0.z, d0, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].z, m1.z, d1, 0, 0, 0);
        d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].w, m0.w, d0, 0, 0, 0);
        d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[t].w, m1.w, d1, 0, 0, 0);
    }
    if (c0 < k) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (d0[r] > best[r]) { best[r] = d0[r]; arg[r] = c0; }
    }
    if (c1 < k) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (d1[r] > best[r]) { best[r] = d1[r]; arg[r] = c1; }
    }
}
// merge the 16 columns of a row: larger similarity wins, equal ones go to the lower centroid id (the maximum first, then the lowest of
// the ids that have it: ten instructions, where carrying both through every step took forty)
__device__ __forceinline__ void lc_assign_merge(float& bv, int& ba) {
    float v = bv;
    v = fmaxf(v, lc_dpp<0xB1>(v));
    v = fmaxf(v, lc_dpp<0x4E>(v));
    v = fmaxf(v, lc_dpp<0x141>(v));
    v = fmaxf(v, lc_dpp<0x140>(v));
    int id = bv == v ? ba : 0x7fffffff;
    id = min(id, __builtin_amdgcn_update_dpp(0, id, 0xB1, 0xF, 0xF, true));
    id = min(id, __builtin_amdgcn_update_dpp(0, id, 0x4E, 0xF, 0xF, true));
    id = min(id, __builtin_amdgcn_update_dpp(0, id, 0x141, 0xF, 0xF, true));
    id = min(id, __builtin_amdgcn_update_dpp(0, id, 0x140, 0xF, 0xF, true));
    bv = v;
    ba = id;
}
// Orders a wavefront's own LDS accesses (no other wavefront is involved).
__device__ __forceinline__ void lc_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// `flags` (may be null): flags[level][bh][t] = iteration t moved a point.  An iteration that moves none is a
// fixed point -- the update would rebuild the same centroids from the same members and every later
// iteration would repeat it -- so from then on the kernels of this (sequence, head) return at once:
// iteration `it` assigns only if it <= 1 or iteration it - 1 moved a point, and leaves its own flag
// at zero otherwise, which passes the verdict on.
//
// Which centroids can be a point's nearest: similarities of the bfloat16-rounded directions
// (v_mfma_f32_16x16x32_bf16, 16 times the float32 rate) are off by at most LC_AS_EPS, because points and
// centroids are unit vectors and rounding moves each by at most 2^-9 of its length.  So the nearest
// centroid is among those whose bfloat16 similarity reaches a float32 similarity the point is known to
// have minus LC_AS_EPS, or the largest bfloat16 similarity minus twice that.  Nearly always that is one
// centroid and it is the label; the few points with more candidates get them compared in float32, in
// the arithmetic of lc_assign_block (16 (point, candidate) pairs to a block, the diagonal of the result);
// a point with more than LC_AS_CAND candidates is compared with every centroid that way.  The labels are
// those of the float32 argmax over all centroids, ties included.
#define LC_AS_TILE 64             // centroids per LDS tile
#define LC_AS_RES 256             // most centroids kept in LDS
#define LC_AS_PITCH 272           // bytes per staged bfloat16 row (the pad spreads the 16 rows of a block over the banks)
#define LC_AS_CAND 16             // candidates a point can hold (with 8, one point in 40 K had more: a tail of several times the kernel)
#define LC_AS_REFRESH 256         // first iteration: centroids between two looks at what is known of the points (a power of two)
#define LC_AS_SAMPLE 1024         // first iteration: centroids up to which the first sweep takes all of them (see lc_kmeans_assign_kernel)
#define LC_AS_PAIRS 128           // pairs a wavefront compares at a time (and no fewer than its points)
#define LC_AS_EPS 0.0040f         // 2^-8 (both operands' rounding, Cauchy-Schwarz) and room for the float32 sums
typedef __bf16 lc_bf16x8_b __attribute__((ext_vector_type(8)));

// LDS of the candidates of a workgroup's points: NW wavefronts, WP points each.
template <int WP, int NW>
struct LcAssignSh {
    int cand_n[NW][WP];
    int cand[NW][WP][LC_AS_CAND];
    uint8_t rest_p[NW * WP];
    int n_rest;
};
template <int NW>
struct LcAssignPairs {
    float pair_v[NW][LC_AS_PAIRS];
    int pair_c[NW][LC_AS_PAIRS];
    uint8_t pair_p[NW][LC_AS_PAIRS];
};
__device__ __forceinline__ void lc_assign_take(int* n, int* list, int c) {
    const int at = atomicAdd(n, 1);
    if (at < LC_AS_CAND) list[at] = c;
}

// From the candidates of this workgroup's points (the first is w0, wavefront's first p0) to their labels; all
// threads call.  P, C: float32 rows of the points and centroids; lab: the labels, old_label this lane's.  Returns the label of
// this lane's point, -1 without one; every wavefront is past its last use of the centroid rows then.
template <int WP, int NW>
__device__ __forceinline__ int lc_assign_finish(LcAssignSh<WP, NW>& sh, LcAssignPairs<NW>& pairs, const float* P, const float* C, int N, int k, int w0,
                                                 int p0, int* lab, int old_label, int* flag) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, kk = lane >> 4;
    // ---- points with one candidate are done; the others' candidates become pairs, 16 to a block, as many
    // points at a time as the pair list takes
    const int my_p = lane < WP ? lane : WP - 1;
    const int n_c = sh.cand_n[wave][my_p];
    const bool mine = lane < WP && p0 + lane < N;
    bool open = mine && n_c >= 2 && n_c <= LC_AS_CAND;
    int ba = n_c == 1 ? sh.cand[wave][my_p][0] : 0;
    while (__ballot(open) != 0ull) {
        const int want = open ? n_c : 0;
        const int incl = lc_wave_scan_incl(want);
        const int first = incl - want;
        const bool now = open && incl <= LC_AS_PAIRS;               // (the first open point always fits)
        const int n_pairs = (int)lc_wave_max_u((uint32_t)(now ? incl : 0));
        if (now)
            for (int e = 0; e < n_c; ++e) {
                pairs.pair_c[wave][first + e] = sh.cand[wave][my_p][e];
                pairs.pair_p[wave][first + e] = (uint8_t)my_p;
            }
        lc_wave_sync();
        for (int q0 = 0; q0 < n_pairs; q0 += 16) {
            const int q = min(q0 + j, n_pairs - 1);
            const float* xr = P + (size_t)(p0 + (int)pairs.pair_p[wave][q]) * LC_D + 4 * kk;
            const float* mr = C + (size_t)pairs.pair_c[wave][q] * LC_D + 4 * kk;
            float4 x[8], m[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                x[t] = *reinterpret_cast<const float4*>(xr + 16 * t);
                m[t] = *reinterpret_cast<const float4*>(mr + 16 * t);
            }
            lc_f32x4_b d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t].x, m[t].x, d, 0, 0, 0);
                d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t].y, m[t].y, d, 0, 0, 0);
                d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t].z, m[t].z, d, 0, 0, 0);
                d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t].w, m[t].w, d, 0, 0, 0);
            }
            const float diag = (j & 2) ? ((j & 1) ? d[3] : d[2]) : ((j & 1) ? d[1] : d[0]);    // row 4 kk + (j & 3) = column j
            if (kk == (j >> 2) && q0 + j < n_pairs) pairs.pair_v[wave][q0 + j] = diag;
        }
        lc_wave_sync();
        if (now) {
            float bv = LC_NEG_INF;
            int bc = 0x7fffffff;
            for (int e = 0; e < n_c; ++e) {
                const float v = pairs.pair_v[wave][first + e];
                const int c = pairs.pair_c[wave][first + e];
                if (v > bv || (v == bv && c < bc)) { bv = v; bc = c; }
            }
            ba = bc < k ? bc : 0;
            open = false;
        }
        lc_wave_sync();
    }
    // ---- too many candidates (or none, or marked as such: not-a-number): every centroid in float32, 16 such points of the
    // workgroup at a time, an equal share of the centroids per wavefront
    if (mine && (n_c == 0 || n_c > LC_AS_CAND)) sh.rest_p[atomicAdd(&sh.n_rest, 1)] = (uint8_t)(wave * WP + lane);
    __syncthreads();
    const int rest = sh.n_rest;
    for (int q0 = 0; q0 < rest; q0 += 16) {
        const float* xr = P + (size_t)(w0 + sh.rest_p[min(q0 + j, rest - 1)]) * LC_D + 4 * kk;
        float4 x[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t] = *reinterpret_cast<const float4*>(xr + 16 * t);
        float best[4];
        int arg[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) { best[r] = LC_NEG_INF; arg[r] = 0x7fffffff; }
        for (int c = 32 * wave; c < k; c += 32 * NW)
            lc_assign_block2(x, C + (size_t)min(c + j, k - 1) * LC_D + 4 * kk, C + (size_t)min(c + 16 + j, k - 1) * LC_D + 4 * kk,
                             c + j, c + 16 + j, k, best, arg);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            lc_assign_merge(best[r], arg[r]);
            if (j == 0) { pairs.pair_v[wave][4 * kk + r] = best[r]; pairs.pair_c[wave][4 * kk + r] = arg[r]; }
        }
        __syncthreads();
        for (int e = 0; e < 16 && q0 + e < rest; ++e) {             // the owner takes the best of the shares
            if (mine && sh.rest_p[q0 + e] == wave * WP + lane) {
                float bv = LC_NEG_INF;
                int bc = 0x7fffffff;
                for (int w = 0; w < NW; ++w)
                    if (pairs.pair_v[w][e] > bv || (pairs.pair_v[w][e] == bv && pairs.pair_c[w][e] < bc)) {
                        bv = pairs.pair_v[w][e];
                        bc = pairs.pair_c[w][e];
                    }
                ba = bc < k ? bc : 0;
            }
        }
        __syncthreads();
    }
    if (mine) {
        if (flag && old_label != ba) *flag = 1;                     // (every writer stores the same value)
        lab[p0 + lane] = ba;
    }
    return mine ? ba : -1;
}

// Which points belong to a cluster, as bits: word [block][cluster] of a (sequence, head) has bit i set if point 64 * block + i
// carries that label.  The assignment of up to LC_AS_RES centroids leaves them, so that the update of a cluster reads a word per 64
// points instead of every label, and knows from the words of the iteration before whether it has anything to do.
struct LcMemberBits {
    unsigned long long* w[2];        // by parity of the iteration; null: not kept
    long long stride[2];             // words of a (sequence, head)
    int pitch;                       // words of a block
};

// Up to 16 NBLK centroids: all of them in LDS, a wavefront's similarities all in registers.  NW
// wavefronts of 16 points each share the staged rows.  A chain of four memory round trips (counts, rows,
// pairs, labels) with little between them; the blocks carry no branches so that their LDS reads and
// products overlap (with one around each block a block took 500 clocks).
// Measured, 8 heads of 2275 points x 143 centroids: 16.7 -> 8.8 us an iteration.
template <int NBLK, int NW>
__global__ void __launch_bounds__(64 * NW, NBLK == 16 ? 2 : NW / 2)
lc_kmeans_assign_res_kernel(LcDev ix, int l, const float* pts, const uint16_t* pts16, int pts_cap, const float* cent,
                            const uint16_t* cent16, int cent_cap, int it, int* flags_all, LcMemberBits bits) {
    lc_fetch_args<sizeof(LcDev) + 40>();
    constexpr int PIECES = NBLK * 256 / (64 * NW);                  // 16-byte pieces of the rows per thread
    __shared__ __attribute__((aligned(16))) unsigned char rows[16 * NBLK * LC_AS_PITCH];
    // (16 blocks under eight wavefronts: the pairs come where the rows were, behind the bits, so that two workgroups fit a compute unit)
    constexpr bool SHARE = NBLK == 16 && NW == 8;
    constexpr int BITS_END = NW / 4 * 16 * NBLK * 8;
    using Pairs = LcAssignPairs<NW>;
    __shared__ LcAssignSh<16, NW> sh;
    __shared__ __attribute__((aligned(16))) unsigned char own_pairs[SHARE ? 16 : sizeof(Pairs)];
    static_assert(!SHARE || BITS_END + sizeof(Pairs) <= sizeof(rows), "");
    Pairs& pairs = *reinterpret_cast<Pairs*>(SHARE ? rows + BITS_END : own_pairs);
    const int h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    int* const flags = flags_all ? lc_level_flags(ix, flags_all, l, bh) : nullptr;
    const int N = lc_level_count(ix, b, bh, l);
    const int k = ix.nlev[b * LC_MAX_LEVELS + l + 1];
    if (flags && it >= 2 && flags[it - 1] == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 15, kk = lane >> 4;
    const int w0 = blockIdx.x * (16 * NW), p0 = w0 + wave * 16;     // first point of the workgroup, of this wavefront
    if (w0 >= N) return;
    const uint16_t* const C16 = cent16 + (size_t)bh * cent_cap * LC_D;
    int* const lab = ix.parent[l] + (size_t)bh * ix.cap[l];

    // every load goes out at once: A operand (point p0 + j, dimensions 32 s + 8 kk + (0..7)), the centroid
    // rows this thread stages (rows past the last centroid repeat it), the label
    lc_v4i xa[4], st[PIECES];
    {
        const uint16_t* row = pts16 + ((size_t)bh * pts_cap + min(p0 + j, N - 1)) * LC_D + 8 * kk;
#pragma unroll
        for (int s = 0; s < 4; ++s) xa[s] = *reinterpret_cast<const lc_v4i*>(row + 32 * s);
    }
#pragma unroll
    for (int e = 0; e < PIECES; ++e)
        st[e] = *reinterpret_cast<const lc_v4i*>(C16 + (size_t)min(4 * NW * e + (tid >> 4), k - 1) * LC_D + 8 * (tid & 15));
    const int old_label = lab[min(p0 + lane, N - 1)];
    if (lane < 16) sh.cand_n[wave][lane] = 0;
    if (tid == 0) sh.n_rest = 0;
#pragma unroll
    for (int e = 0; e < PIECES; ++e)
        *reinterpret_cast<lc_v4i*>(rows + (4 * NW * e + (tid >> 4)) * LC_AS_PITCH + 16 * (tid & 15)) = st[e];
    __syncthreads();

    lc_f32x4_b d[NBLK];
#pragma unroll
    for (int e = 0; e < NBLK; ++e) {
        const unsigned char* row = rows + (16 * e + j) * LC_AS_PITCH + 16 * kk;
        d[e] = lc_f32x4_b{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s)
            d[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lc_bf16x8_b, xa[s]),
                                                           __builtin_bit_cast(lc_bf16x8_b, *reinterpret_cast<const lc_v4i*>(row + 64 * s)),
                                                           d[e], 0, 0, 0);
    }
    float top[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {                                   // largest of every row, less the margin
        top[r] = d[0][r];
#pragma unroll
        for (int e = 1; e < NBLK; ++e) top[r] = fmaxf(top[r], d[e][r]);
        top[r] = fmaxf(top[r], lc_dpp<0xB1>(top[r]));
        top[r] = fmaxf(top[r], lc_dpp<0x4E>(top[r]));
        top[r] = fmaxf(top[r], lc_dpp<0x141>(top[r]));
        top[r] = fmaxf(top[r], lc_dpp<0x140>(top[r])) - 2.0f * LC_AS_EPS;
    }
    // this lane's candidates as a bit mask: bit 4 (e mod 8) + r of word e / 8
#pragma unroll
    for (int w = 0; w < (NBLK + 7) / 8; ++w) {
        unsigned hit = 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (8 * w + e < NBLK) {
#pragma unroll
                for (int r = 0; r < 4; ++r) hit |= d[8 * w + e < NBLK ? 8 * w + e : 0][r] >= top[r] ? 1u << (4 * e + r) : 0u;
            }
        while (hit != 0u) {
            const int v = __ffs((int)hit) - 1;
            hit &= hit - 1u;
            const int c = 16 * (8 * w + (v >> 2)) + j, p = 4 * kk + (v & 3);
            if (c < k) lc_assign_take(&sh.cand_n[wave][p], sh.cand[wave][p], c);
        }
    }
    if (SHARE) __syncthreads();                                     // the rows have been read
    else lc_wave_sync();
    const int label = lc_assign_finish<16, NW>(sh, pairs, pts + (size_t)bh * pts_cap * LC_D, cent + (size_t)bh * cent_cap * LC_D, N, k,
                                               w0, p0, lab, old_label, flags ? flags + it : nullptr);
    // the members' bits of this workgroup's blocks of 64 points, collected where the centroid rows were
    unsigned long long* const mb = bits.w[it & 1];
    if (mb == nullptr) return;
    constexpr int BLOCKS = NW / 4;
    unsigned* const half = reinterpret_cast<unsigned*>(rows);
    static_assert(BLOCKS * 16 * NBLK * 8 <= (int)sizeof(rows), "bits in the place of the rows");
    for (int i = tid; i < BLOCKS * k * 2; i += 64 * NW) half[i] = 0u;
    lc_barrier_lds();
    const int at = 16 * wave + lane;                                // this lane's point, from the workgroup's first
    if (label >= 0) atomicOr(&half[2 * ((at >> 6) * k + label) + ((at >> 5) & 1)], 1u << (at & 31));
    lc_barrier_lds();
    unsigned long long* const o = mb + bh * bits.stride[it & 1] + (size_t)(w0 >> 6) * bits.pitch;
    for (int i = tid; i < BLOCKS * k; i += 64 * NW) {
        const int blk = BLOCKS == 1 ? 0 : i / k, c = i - blk * k;
        if (w0 + 64 * blk < N) o[(size_t)blk * bits.pitch + c] = reinterpret_cast<const unsigned long long*>(rows)[i];
    }
}

// More centroids: tiles of LC_AS_TILE of them pass through LDS (the next tile's rows are fetched while the
// current one is multiplied) under the 16 MA points per wavefront held in registers.  The threshold enters
// as the matrix instruction's starting accumulator, so a candidate is a result >= 0, and a step of 32
// centroids costs a maximum over its results and a branch that is rarely taken.  Later iterations start from the
// similarity to the point's previous centroid (a float32 dot product).  The first one has no such centroid.  Up to LC_AS_SAMPLE
// centroids, a sweep over all of them finds the largest similarity; of more, a sweep over a quarter -- 16 of every 64, so that
// every neighbourhood is in it -- gives one that about three others exceed, and each candidate found raises it, with effect from the next
// LC_AS_REFRESH centroids on.  (The more candidates cost a fixed time per point, the shorter sweep saves one by the centroid.  Clusterings
// of 8 heads with the quarter and with all: 5.8 K points x 361 centroids 480 and 452 us, 10.9 K x 682 741 and 707,
// x 1365 492 and 488 -- of 2 heads 322 and 325 --, x 2730 513 and 514 -- 299 and 308 --, x 5461 516 and 574.)  Hits are read off
// the results' sign bits, and a result that is not a number may have either: so a point of which no similarity compares is marked beforehand as one
// with too many candidates (float32 decides: cluster 0), and what a centroid of that kind adds to the other points'
// candidates falls away in the float32 comparison, where their nearest one always is a candidate too.
// Measured, 8 heads of 10.9 K points x 5461 centroids (122 GFLOP a sweep): first iteration 218 us, the second
// 149 us; the three iterations of such a clustering took 2.7 ms in float32 and take 0.5 ms.
template <int MA>
__global__ void __launch_bounds__(LC_BT, 2)
lc_kmeans_assign_kernel(LcDev ix, int l, const float* pts, const uint16_t* pts16, int pts_cap, const float* cent,
                        const uint16_t* cent16, int cent_cap, int it, int* flags_all) {
    lc_fetch_args<sizeof(LcDev) + 40>();
    constexpr int WP = 16 * MA;                                     // points per wavefront
    __shared__ __attribute__((aligned(16))) unsigned char tiles[2][LC_AS_TILE * LC_AS_PITCH];
    using Sh = LcAssignSh<WP, 4>;
    __shared__ Sh sh;
    __shared__ __attribute__((aligned(16))) LcAssignPairs<4> pairs;      // (pair_v is read 16 bytes at a time)
    const int h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    int* const flags = flags_all ? lc_level_flags(ix, flags_all, l, bh) : nullptr;
    const int N = lc_level_count(ix, b, bh, l);
    const int k = ix.nlev[b * LC_MAX_LEVELS + l + 1];
    if (flags && it >= 2 && flags[it - 1] == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 15, kk = lane >> 4;
    const int w0 = blockIdx.x * (4 * WP), p0 = w0 + wave * WP;      // first point of the workgroup, of this wavefront
    if (w0 >= N) return;
    const float* const P = pts + (size_t)bh * pts_cap * LC_D;
    const float* const C = cent + (size_t)bh * cent_cap * LC_D;
    const uint16_t* const C16 = cent16 + (size_t)bh * cent_cap * LC_D;
    int* const lab = ix.parent[l] + (size_t)bh * ix.cap[l];
    const int old_label = lab[min(p0 + lane, N - 1)];

    // A operand: point p0 + 16 a + j, dimensions 32 s + 8 kk + (0..7)
    lc_v4i xa[MA][4];
#pragma unroll
    for (int a = 0; a < MA; ++a) {
        const uint16_t* row = pts16 + ((size_t)bh * pts_cap + min(p0 + 16 * a + j, N - 1)) * LC_D + 8 * kk;
#pragma unroll
        for (int s = 0; s < 4; ++s) xa[a][s] = *reinterpret_cast<const lc_v4i*>(row + 32 * s);
    }
    if (lane < WP) sh.cand_n[wave][lane] = 0;
    if (tid == 0) sh.n_rest = 0;

    lc_f32x4_b start[MA];                                           // starting accumulators of this lane's rows (4 kk + r)
    auto load_block = [&](const unsigned char* row, lc_v4i (&m)[4]) LC_INLINE {
#pragma unroll
        for (int s = 0; s < 4; ++s) m[s] = *reinterpret_cast<const lc_v4i*>(row + 64 * s);
    };
    auto multiply = [&](const lc_v4i (&m)[4], lc_f32x4_b (&d)[MA]) LC_INLINE {
#pragma unroll
        for (int a = 0; a < MA; ++a) d[a] = start[a];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int a = 0; a < MA; ++a)
                d[a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lc_bf16x8_b, xa[a][s]),
                                                               __builtin_bit_cast(lc_bf16x8_b, m[s]), d[a], 0, 0, 0);
    };
    // n staged rows, a multiple of 32: two blocks per step, the next step's rows read before this one's
    // products (the last step reads its own again)
    auto sweep = [&](const unsigned char* rows, int n, auto use) LC_INLINE {
        const unsigned char* row = rows + j * LC_AS_PITCH + 16 * kk;
        lc_v4i m0[4], m1[4];
        load_block(row, m0);
        for (int c = 0; c < n; c += 32) {
            lc_f32x4_b d0[MA], d1[MA];
            load_block(row + (c + 16) * LC_AS_PITCH, m1);
            multiply(m0, d0);
            load_block(row + min(c + 32, n - 32) * LC_AS_PITCH, m0);
            multiply(m1, d1);
            use(c, d0, d1);
        }
    };
    constexpr int PF = LC_AS_TILE * 16 / LC_BT;                     // 16-byte pieces per thread and tile
    lc_v4i pf[PF];
    // (rows past the last centroid repeat it; of a sample, 16-row block j is block j mod 4 of the centroids' tile number j)
    auto fetch = [&](bool sample, int c0) LC_INLINE {
#pragma unroll
        for (int e = 0; e < PF; ++e) {
            const int blk = (c0 >> 4) + e;
            const int row = sample ? LC_AS_TILE * blk + 16 * (blk & 3) : 16 * blk;
            pf[e] = *reinterpret_cast<const lc_v4i*>(C16 + (size_t)min(row + (tid >> 4), k - 1) * LC_D + 8 * (tid & 15));
        }
    };
    auto over_tiles = [&](bool sample, int rows, auto use) LC_INLINE {       // two tile buffers: one barrier per tile
        int at = 0;
        for (int c0 = 0; c0 < rows; c0 += LC_AS_TILE) {
            unsigned char* const buf = tiles[at];
#pragma unroll
            for (int e = 0; e < PF; ++e)
                *reinterpret_cast<lc_v4i*>(buf + (16 * e + (tid >> 4)) * LC_AS_PITCH + 16 * (tid & 15)) = pf[e];
            if (c0 + LC_AS_TILE < rows) fetch(sample, c0 + LC_AS_TILE);
            lc_barrier_lds();
            use(buf, c0, min(LC_AS_TILE, (rows - c0 + 31) & ~31));
            at ^= 1;
        }
    };
    // The largest similarity a point is known to have, as an integer that orders like it (similarities lie above -2).
    int* const known = reinterpret_cast<int*>(pairs.pair_v[wave]);
    auto threshold = [&]() LC_INLINE {
#pragma unroll
        for (int a = 0; a < MA; ++a) {
            const int4 v = *reinterpret_cast<const int4*>(known + 16 * a + 4 * kk);
            start[a] = lc_f32x4_b{2.0f * LC_AS_EPS + 2.0f - __int_as_float(v.x), 2.0f * LC_AS_EPS + 2.0f - __int_as_float(v.y),
                                  2.0f * LC_AS_EPS + 2.0f - __int_as_float(v.z), 2.0f * LC_AS_EPS + 2.0f - __int_as_float(v.w)};
        }
    };
    const bool sample = it == 0 && k > LC_AS_SAMPLE;
    fetch(sample, 0);
    // similarity to the previous centroid -- before the first iteration to the one that this point or a neighbour of it starts --,
    // one 16-lane group per point (group kk takes points 4 MA kk + e; the accumulators want points 16 a + 4 kk + r)
    if (it == 0 && !sample) {
        if (lane < WP) pairs.pair_v[wave][lane] = LC_NEG_INF;
    } else {
#pragma unroll 2
        for (int e = 0; e < 4 * MA; ++e) {
            const int i = min(p0 + 4 * MA * kk + e, N - 1);
            const int c = it == 0 ? min((int)(((long long)i * k + N - 1) / N), k - 1) : max(0, min(lab[i], k - 1));
            float x[8], m[8];
            lc_load8(P + (size_t)i * LC_D + 8 * j, x);
            lc_load8(C + (size_t)c * LC_D + 8 * j, m);
            float s = 0.f;
#pragma unroll
            for (int t = 0; t < 8; ++t) s = fmaf(x[t], m[t], s);
            s = lc_sum16(s);
            if (j == 0) pairs.pair_v[wave][4 * MA * kk + e] = it == 0 ? s - 2e-5f + 2.0f : s;      // (as `known`; less its own rounding)
        }
    }
    lc_wave_sync();
    if (it == 0) {
        float top[MA][4];
#pragma unroll
        for (int a = 0; a < MA; ++a) {
            start[a] = lc_f32x4_b{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 4; ++r) top[a][r] = LC_NEG_INF;
        }
        over_tiles(sample, sample ? (k + LC_AS_TILE - 1) / LC_AS_TILE * 16 : k, [&](const unsigned char* buf, int, int n) LC_INLINE {
            sweep(buf, n, [&](int, const lc_f32x4_b (&d0)[MA], const lc_f32x4_b (&d1)[MA]) LC_INLINE {
#pragma unroll
                for (int a = 0; a < MA; ++a)
#pragma unroll
                    for (int r = 0; r < 4; ++r) top[a][r] = fmaxf(top[a][r], fmaxf(d0[a][r], d1[a][r]));
            });
        });
        fetch(false, 0);
#pragma unroll
        for (int a = 0; a < MA; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {                           // largest of the 16 columns of every row
                float v = top[a][r];
                v = fmaxf(v, lc_dpp<0xB1>(v));
                v = fmaxf(v, lc_dpp<0x4E>(v));
                v = fmaxf(v, lc_dpp<0x141>(v));
                v = fmaxf(v, lc_dpp<0x140>(v));
                if (j == 0) atomicMax(&known[16 * a + 4 * kk + r], __float_as_int(v + 2.0f));
            }
        lc_barrier_lds();                                           // the last tile has been used
        threshold();
    } else {
#pragma unroll
        for (int a = 0; a < MA; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) start[a][r] = (LC_AS_EPS + 2e-5f) - pairs.pair_v[wave][16 * a + 4 * kk + r];
    }
    if (lane < WP && !(pairs.pair_v[wave][lane] > LC_NEG_INF)) sh.cand_n[wave][lane] = LC_AS_CAND + 1;     // (see above)
    lc_wave_sync();
    over_tiles(false, k, [&](const unsigned char* buf, int c0, int n) LC_INLINE {
        if (it == 0 && c0 != 0 && (c0 & (LC_AS_REFRESH - 1)) == 0) threshold();
        sweep(buf, n, [&](int c, const lc_f32x4_b (&d0)[MA], const lc_f32x4_b (&d1)[MA]) LC_INLINE {
            float any = LC_NEG_INF;
#pragma unroll
            for (int a = 0; a < MA; ++a)
#pragma unroll
                for (int r = 0; r < 4; ++r) any = fmaxf(any, fmaxf(d0[a][r], d1[a][r]));
            if (any >= 0.f) {
                if (it == 0) {
#pragma unroll
                    for (int a = 0; a < MA; ++a)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float m = fmaxf(d0[a][r], d1[a][r]);
                            if (m >= 0.f) atomicMax(&known[16 * a + 4 * kk + r], __float_as_int(m - start[a][r] + 2.0f));
                        }
                }
                unsigned neg = 0u;                                  // sign bits, the last result in bit 0
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int a = 0; a < MA; ++a)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(q ? d1[a][r] : d0[a][r]), 31);
                unsigned hit = ~neg & (8 * MA >= 32 ? 0xffffffffu : (1u << (8 * MA & 31)) - 1u);
                while (hit != 0u) {
                    const int v = 8 * MA - 1 - (__ffs((int)hit) - 1);       // (q * MA + a) * 4 + r
                    hit &= hit - 1u;
                    const int q = v / (4 * MA), p = 16 * ((v >> 2) - q * MA) + 4 * kk + (v & 3);
                    const int id = c0 + c + 16 * q + j;
                    if (id < k) lc_assign_take(&sh.cand_n[wave][p], sh.cand[wave][p], id);
                }
            }
        });
    });
    __syncthreads();
    lc_assign_finish<WP, 4>(sh, pairs, P, C, N, k, w0, p0, lab, old_label, flags ? flags + it : nullptr);
}

// Ascending list, in LDS, of the i in [base, base + LC_MEM_WIN) below n with label c; returns its length in
// every thread.  Every label is loaded once, coalesced, all loads in flight together (lc_load_labels, which
// a caller of several windows issues one window ahead); positions come from wavefront ballots and one scan
// of the 64 (row, wavefront) counts, so the order is fixed.  cnt: 2 * 64 + 1 ints of LDS; mem: LC_MEM_WIN
// ints.  All NT threads must call.
#define LC_MEM_WIN 4096
template <int NT, typename LabF>
__device__ __forceinline__ void lc_load_labels(LabF lab, int n, int base, int (&lv)[LC_MEM_WIN / NT]) {
#pragma unroll
    for (int e = 0; e < LC_MEM_WIN / NT; ++e) {
        lv[e] = -1;
        if (base + e * NT < n) {                                    // (uniform: whole rows past the end are skipped)
            const int i = base + e * NT + (int)threadIdx.x;
            const int v = lab(min(i, n - 1));
            lv[e] = i < n ? v : -1;
        }
    }
}
template <int NT>
__device__ __forceinline__ int lc_list_members(const int (&lv)[LC_MEM_WIN / NT], int base, int c, int* mem, int* cnt) {
    constexpr int E = LC_MEM_WIN / NT;
    constexpr int W = NT / 64;
    static_assert(E * W == 64, "one wavefront scans the (row, wavefront) counts");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const unsigned long long m = __ballot(lv[e] == c);
        if (lane == 0) cnt[e * W + wave] = __popcll(m);
    }
    lc_barrier_lds();
    if (wave == 0) {
        const int v = cnt[lane];
        const int inc = lc_wave_scan_incl(v);
        cnt[64 + lane] = inc - v;
        if (lane == 63) cnt[128] = inc;
    }
    lc_barrier_lds();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const unsigned long long m = __ballot(lv[e] == c);
        if (lv[e] == c) mem[cnt[64 + e * W + wave] + lc_mbcnt(m)] = base + e * NT + tid;
    }
    lc_barrier_lds();
    return cnt[128];
}
template <int NT, typename LabF>
__device__ __forceinline__ int lc_collect_members(LabF lab, int n, int base, int c, int* mem, int* cnt) {
    int lv[LC_MEM_WIN / NT];
    lc_load_labels<NT>(lab, n, base, lv);
    return lc_list_members<NT>(lv, base, c, mem, cnt);
}

// Member lists of up to LC_UB_MAX consecutive clusters at once, for levels of many small clusters: the
// workgroup reads the labels once, drops every match into an unordered list, sorts that by cluster and,
// inside a cluster, into the order in which the sums are taken.
// That order: a cluster's members, ascending, are dealt to 16 partial sums in turn (starting over every
// LC_MEM_WIN points), and the partial sums are added up in turn.  A 16-lane group that takes the members
// as listed, adding up its running sum whenever the partial changes, forms exactly those sums.
// list[off[c] .. off[c + 1]): members of cluster c0 + c, part[]: the partial sum each belongs to.
#define LC_UB_MAX 64              // clusters of a workgroup
#define LC_UB_LIST 2048           // members they may have together; beyond that the clusters are listed one by one
#define LC_UB_BIG 64              // a cluster of more members is summed by the whole workgroup
struct LcBuckets {
    int n[LC_UB_MAX], off[LC_UB_MAX + 1];
    int total;
    int raw[2 * LC_UB_LIST];      // matches as found: point; cluster and position among its matches
    int list[LC_UB_LIST];
    uint8_t part[LC_UB_LIST];
};
// Returns false (in every thread) if the clusters have more members than the list holds.  All LC_BT threads must call.
template <typename LabF>
__device__ __forceinline__ bool lc_fill_buckets(LabF lab, int N, int c0, int n_c, LcBuckets& s) {
    const int tid = threadIdx.x;
    int* const raw_i = s.raw;
    int* const raw_cs = s.raw + LC_UB_LIST;
    if (tid < LC_UB_MAX) s.n[tid] = 0;
    if (tid == 0) s.total = 0;
    __syncthreads();
    constexpr int E = 8;
    for (int base = 0; base < N; base += E * LC_BT) {
        int lv[E];
#pragma unroll
        for (int e = 0; e < E; ++e) lv[e] = lab(min(base + e * LC_BT + tid, N - 1));
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = base + e * LC_BT + tid;
            const int c = lv[e] - c0;
            if (i < N && c >= 0 && c < n_c) {
                const int q = atomicAdd(&s.total, 1);
                const int at = atomicAdd(&s.n[c], 1);
                if (q < LC_UB_LIST) { raw_i[q] = i; raw_cs[q] = (c << 16) | at; }
            }
        }
    }
    __syncthreads();
    const int total = s.total;
    if (total > LC_UB_LIST) return false;
    if (tid < 64) {
        const int v = tid < LC_UB_MAX ? s.n[tid] : 0;
        const int inc = lc_wave_scan_incl(v);
        s.off[tid] = inc - v;
        if (tid == 63) s.off[LC_UB_MAX] = inc;
    }
    __syncthreads();
    for (int q = tid; q < total; q += LC_BT) s.list[s.off[raw_cs[q] >> 16] + (raw_cs[q] & 0xffff)] = raw_i[q];
    __syncthreads();
    // partial sum of every member (its rank among the cluster's members of its window, mod 16), then its place
    constexpr int PER = LC_UB_LIST / LC_BT;
    int mi[PER], mg[PER], mc[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int q = tid + e * LC_BT;
        mi[e] = -1;
        if (q < total) {
            const int c = raw_cs[q] >> 16, i = raw_i[q];
            const int w0 = i & ~(LC_MEM_WIN - 1);
            int r = 0;
            for (int t = s.off[c]; t < s.off[c + 1]; ++t) r += (s.list[t] >= w0 && s.list[t] < i) ? 1 : 0;
            mi[e] = i;
            mg[e] = r & 15;
            mc[e] = c;
            s.part[s.off[c] + (raw_cs[q] & 0xffff)] = (uint8_t)mg[e];
        }
    }
    __syncthreads();
    int mp[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        if (mi[e] >= 0) {
            int at = s.off[mc[e]];
            for (int t = s.off[mc[e]]; t < s.off[mc[e] + 1]; ++t) {
                const int g = s.part[t];
                at += (g < mg[e] || (g == mg[e] && s.list[t] < mi[e])) ? 1 : 0;
            }
            mp[e] = at;
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e)
        if (mi[e] >= 0) { s.list[mp[e]] = mi[e]; s.part[mp[e]] = (uint8_t)mg[e]; }
    __syncthreads();
    return true;
}

// One row more in a sum: plain float32 rows, or rows of weight w (0: left out, whatever the row holds) in float64.
template <int N>
__device__ __forceinline__ void lc_add_row(float (&acc)[N], const float (&x)[N], int) {
#pragma unroll
    for (int t = 0; t < N; ++t) acc[t] += x[t];
}
template <int N>
__device__ __forceinline__ void lc_add_row(double (&acc)[N], const float (&x)[N], int w) {
#pragma unroll
    for (int t = 0; t < N; ++t) acc[t] = fma((double)(w > 0 ? x[t] : 0.f), (double)w, acc[t]);
}

// Sum of the rows of list[t0, t1) as described above, by one 16-lane group (8 columns per lane); with
// `flush` false only the running sum of one partial is wanted (all members of one partial).
// row(i, x): columns [8 sub, 8 sub + 8) of member i's row; returns its weight.
template <typename Acc, typename RowF>
__device__ __forceinline__ void lc_sum_listed(const LcBuckets& s, int t0, int t1, RowF row, Acc (&sum)[8]) {
    constexpr int BATCH = 8;                                        // rows in flight per group
    Acc run[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) { sum[u] = 0; run[u] = 0; }
    int g = t0 < t1 ? s.part[t0] : 0;
    for (int t = t0; t < t1; t += BATCH) {
        float x[BATCH][8];
        int w[BATCH];
#pragma unroll
        for (int e = 0; e < BATCH; ++e) w[e] = row(s.list[min(t + e, t1 - 1)], x[e]);
#pragma unroll
        for (int e = 0; e < BATCH; ++e) {
            if (t + e < t1) {
                const int ge = s.part[t + e];
                if (ge != g) {
                    g = ge;
#pragma unroll
                    for (int u = 0; u < 8; ++u) { sum[u] += run[u]; run[u] = 0; }
                }
                lc_add_row(run, x[e], w[e]);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) sum[u] += run[u];
}

// The sums of the rows of clusters [c0, c0 + n_c), each handed to done(c, n, sum) in one whole 16-lane group
// (c: cluster, n: members, sum: 8 columns per lane).  Small clusters one per group, clusters of more than
// LC_UB_BIG members by the workgroup, 16 groups for the 16 partial sums.  sh: 16 * LC_D values.
// Acc: the type the rows are summed in.
template <typename Acc, typename LabF, typename RowF, typename DoneF>
__device__ __forceinline__ void lc_cluster_sums(LabF lab, int N, int c0, int n_c, LcBuckets& s, Acc* sh, RowF row,
                                                DoneF done) {
    const int sub = threadIdx.x & 15, grp = threadIdx.x >> 4;
    if (N > 0 && !lc_fill_buckets(lab, N, c0, n_c, s)) {
        // ---- more members than the list holds: cluster by cluster
        int* const mem = s.raw;
        int* const cnt = s.list;
        static_assert(sizeof(s.raw) >= LC_MEM_WIN * sizeof(int), "window of the one-by-one listing");
        for (int c = 0; c < n_c; ++c) {
            Acc sum[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) sum[u] = 0;
            int n = 0;
            for (int base = 0; base < N; base += LC_MEM_WIN) {
                const int nm = lc_collect_members<LC_BT>(lab, N, base, c0 + c, mem, cnt);
#pragma unroll 4
                for (int t = grp; t < nm; t += LC_BG) {
                    float x[8];
                    const int w = row(mem[t], x);
                    lc_add_row(sum, x, w);
                }
                n += nm;
                __syncthreads();                                    // the list is rewritten by the next window
            }
            lc_store_acc8(sh + grp * LC_D + 8 * sub, sum);
            __syncthreads();
            if (grp == 0) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    Acc a = 0;
                    for (int g = 0; g < LC_BG; ++g) a += sh[g * LC_D + 8 * sub + u];
                    sum[u] = a;
                }
                done(c0 + c, n, sum);
            }
            __syncthreads();
        }
        return;
    }
    if (N == 0) {
        for (int c = grp; c < n_c; c += LC_BG) {
            Acc sum[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) sum[u] = 0;
            done(c0 + c, 0, sum);
        }
        return;
    }
    for (int c = grp; c < n_c; c += LC_BG) {
        if (s.n[c] > LC_UB_BIG) continue;
        Acc sum[8];
        lc_sum_listed(s, s.off[c], s.off[c + 1], row, sum);
        done(c0 + c, s.n[c], sum);
    }
    for (int c = 0; c < n_c; ++c) {                                 // (uniform)
        if (s.n[c] <= LC_UB_BIG) continue;
        int lo = s.off[c], hi = s.off[c + 1];                       // this group's partial: a run of the list
        {
            int a = lo, z = hi;
            while (a < z) { const int m = (a + z) >> 1; if (s.part[m] < grp) a = m + 1; else z = m; }
            lo = a;
            z = hi;
            while (a < z) { const int m = (a + z) >> 1; if (s.part[m] <= grp) a = m + 1; else z = m; }
            hi = a;
        }
        Acc sum[8];
        lc_sum_listed(s, lo, hi, row, sum);
        __syncthreads();
        lc_store_acc8(sh + grp * LC_D + 8 * sub, sum);
        __syncthreads();
        if (grp == 0) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                Acc a = 0;
                for (int g = 0; g < LC_BG; ++g) a += sh[g * LC_D + 8 * sub + u];
                sum[u] = a;
            }
            done(c0 + c, s.n[c], sum);
        }
    }
}

// Sum of the rows of the members of ONE cluster u by a whole workgroup: the members are listed window by
// window, 16-lane group g takes them in turn for partial sum g mod 16, and the partial sums are added up
// in turn (the order of lc_cluster_sums).  With 1024 threads the groups split the columns of a partial four
// ways, for four times the loads in flight.  visit(mem, nm) sees every window's list.
// On return sh[128] .. hold nothing of use and threads < 16 have the sum (8 columns each); returns the number
// of members in every thread.  All NT threads must call.
template <int NT, typename Acc>
struct LcSumSh {
    Acc part[LC_BG][LC_D];
    int mem[LC_MEM_WIN];
    int cnt[2 * 64 + 1];
};
// The partial sums `acc` (number `part`, columns from `col` on) added up in turn, a column per thread; threads < 16 get eight columns each.
template <int NT, typename Acc, int COLS>
__device__ __forceinline__ void lc_sum_partials(LcSumSh<NT, Acc>& s, int col, int part, const Acc (&acc)[COLS], Acc (&sum)[8]) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int q = 0; q < COLS; ++q) s.part[part][col + q] = acc[q];
    __syncthreads();
    if (tid < LC_D) {
        Acc a = 0;
#pragma unroll
        for (int g = 0; g < LC_BG; ++g) a += s.part[g][tid];
        s.part[0][tid] = a;                                         // (this thread's column alone)
    }
    __syncthreads();
    if (tid < 16) {
#pragma unroll
        for (int t = 0; t < 8; ++t) sum[t] = s.part[0][8 * tid + t];
    }
}
template <int NT, typename Acc, typename LabF, typename RowF, typename VisitF>
__device__ __forceinline__ int lc_member_sum(LabF lab, int N, int u, LcSumSh<NT, Acc>& s, RowF row, VisitF visit, Acc (&sum)[8]) {
    constexpr int COLS = 8 * 256 / NT;                              // columns per lane
    constexpr int BATCH = NT == 256 ? 4 : 16;                       // rows in flight per group
    const int tid = threadIdx.x, sub = tid & 15, part = (tid >> 4) & 15;
    const int col = (tid >> 8) * (COLS * 16) + COLS * sub;
    Acc acc[COLS];
#pragma unroll
    for (int t = 0; t < COLS; ++t) acc[t] = 0;
    int n = 0;
    int lv[LC_MEM_WIN / NT];
    if (N > 0) lc_load_labels<NT>(lab, N, 0, lv);
    for (int base = 0; base < N; base += LC_MEM_WIN) {
        const int nm = lc_list_members<NT>(lv, base, u, s.mem, s.cnt);
        if (base + LC_MEM_WIN < N) lc_load_labels<NT>(lab, N, base + LC_MEM_WIN, lv);
        for (int t = part; t < nm; t += BATCH * 16) {
            float x[BATCH][COLS];
            int w[BATCH];
#pragma unroll
            for (int e = 0; e < BATCH; ++e) {
                w[e] = 0;
                if (t + 16 * e < nm) w[e] = row(s.mem[t + 16 * e], col, x[e]);
                else {
#pragma unroll
                    for (int q = 0; q < COLS; ++q) x[e][q] = 0.f;
                }
            }
#pragma unroll
            for (int e = 0; e < BATCH; ++e)
                if (t + 16 * e < nm) lc_add_row(acc, x[e], w[e]);
        }
        visit(s.mem, nm);
        n += nm;
        if (base + LC_MEM_WIN < N) lc_barrier_lds();                // the list is rewritten by the next window
    }
    lc_sum_partials(s, col, part, acc, sum);
    return n;
}

// m_c = normalise(sum of members); a cluster without members (or with a zero sum) keeps m_c.
__device__ __forceinline__ void lc_write_centroid(float* cent, uint16_t* cent16, size_t o, float (&s)[8]) {
    float n2 = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) n2 = fmaf(s[t], s[t], n2);
    n2 = lc_sum16(n2);
    if (n2 > 0.f) {
        const float inv = 1.0f / sqrtf(n2);
#pragma unroll
        for (int t = 0; t < 8; ++t) s[t] *= inv;
        lc_store8(cent + o, s);
        lc_store8_bf16(cent16 + o, s);
    }
}
// One workgroup per cluster: for clusters of more than LC_UPD_FEW points on average (their rows are then
// the larger part of what a workgroup reads, and 16 groups fetch them at once).
#define LC_UPD_FEW 8
#define LC_UPD_FEW_MANY 20        // (with thousands of clusters)
__global__ void __launch_bounds__(LC_BT)
lc_kmeans_update_kernel(LcDev ix, int l, const float* pts, int pts_cap, float* cent, uint16_t* cent16, int cent_cap, int it,
                        int* flags_all) {
    lc_fetch_args<sizeof(LcDev) + 40>();
    __shared__ __attribute__((aligned(16))) LcSumSh<LC_BT, float> sh;
    const int c = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    const int* const flags = flags_all ? lc_level_flags(ix, flags_all, l, bh) : nullptr;
    if (flags && it >= 1 && flags[it] == 0) return;                 // no point moved: the centroids stand
    const int N = lc_level_count(ix, b, bh, l);
    if (c >= ix.nlev[b * LC_MAX_LEVELS + l + 1]) return;
    const int* labels = ix.parent[l] + (size_t)bh * ix.cap[l];
    const float* P = pts + (size_t)bh * pts_cap * LC_D;
    float sum[8];
    lc_member_sum<LC_BT, float>([&](int i) { return labels[i]; }, N, c, sh,
                                [&](int i, int col, float (&x)[8]) { lc_load8(P + (size_t)i * LC_D + col, x); return 1; },
                                [](const int*, int) {}, sum);
    if (threadIdx.x < 16)
        lc_write_centroid(cent, cent16, ((size_t)bh * cent_cap + c) * LC_D + 8 * threadIdx.x, sum);
}
// The same from the members' bits (LcMemberBits): a window's list is a scan over 64 words, and a cluster whose words are those of
// the iteration before keeps its centroid (the sum would be the same one).  Same members in the same order: same bits as above.
// What bounds it is three round trips, counts, words and rows.  8 heads, 2275 points in 143 clusters: 7.7 us from the labels, now
// 4.5; 5461 points in 249: 23.3 and 9.2.
__global__ void __launch_bounds__(LC_BT)
lc_kmeans_update_bits_kernel(LcDev ix, int l, const float* pts, int pts_cap, float* cent, uint16_t* cent16, int cent_cap, int it,
                             int* flags_all, LcMemberBits bits) {
    lc_fetch_args<sizeof(LcDev) + 40 + sizeof(LcMemberBits)>();
    __shared__ __attribute__((aligned(16))) LcSumSh<LC_BT, float> sh;
    const int c = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    const int* const flags = flags_all ? lc_level_flags(ix, flags_all, l, bh) : nullptr;
    const int N = lc_level_count(ix, b, bh, l), k = ix.nlev[b * LC_MAX_LEVELS + l + 1];
    if (flags && it >= 1 && flags[it] == 0) return;                 // no point moved: the centroids stand
    if (c >= k) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = threadIdx.x & 15, part = threadIdx.x >> 4;
    const int blocks = (N + 63) >> 6;
    const unsigned long long* const now = bits.w[it & 1] + bh * bits.stride[it & 1] + c;
    const unsigned long long* const old = bits.w[~it & 1] + bh * bits.stride[~it & 1] + c;
    auto word = [&](const unsigned long long* w, int blk) { return blk < blocks ? w[(size_t)blk * bits.pitch] : 0ull; };
    unsigned long long m = word(now, lane);                         // (every wavefront reads them: none waits for another's verdict)
    if (it >= 1) {
        bool moved = m != word(old, lane);
        for (int w0 = 64; w0 < blocks; w0 += 64) moved = moved || word(now, w0 + lane) != word(old, w0 + lane);
        if (__ballot(moved) == 0ull) return;
    }
    const float* P = pts + (size_t)bh * pts_cap * LC_D;
    constexpr int BATCH = 4;
    float acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = 0.f;
    for (int w0 = 0; w0 < blocks; w0 += 64) {                       // windows of 64 blocks: LC_MEM_WIN points
        static_assert(LC_MEM_WIN == 64 * 64, "a word per lane");
        const int n = __popcll(m), inc = lc_wave_scan_incl(n);
        const int nm = lc_readlane(inc, 63);
        if (wave == 0)
            for (int at = inc - n; m != 0ull; m &= m - 1ull) sh.mem[at++] = 64 * (w0 + lane) + __ffsll((long long)m) - 1;
        if (w0 + 64 < blocks) m = word(now, w0 + 64 + lane);
        lc_barrier_lds();
        for (int t = part; t < nm; t += BATCH * LC_BG) {
            float x[BATCH][8];
#pragma unroll
            for (int e = 0; e < BATCH; ++e) {
                const int at = min(t + e * LC_BG, nm - 1);
                lc_load8(P + (size_t)sh.mem[at] * LC_D + 8 * sub, x[e]);
            }
#pragma unroll
            for (int e = 0; e < BATCH; ++e)
                if (t + e * LC_BG < nm) lc_add_row(acc, x[e], 1);
        }
        if (w0 + 64 < blocks) lc_barrier_lds();                     // the list is rewritten by the next window
    }
    float sum[8];
    lc_sum_partials(sh, 8 * sub, part, acc, sum);
    if (threadIdx.x < 16)
        lc_write_centroid(cent, cent16, ((size_t)bh * cent_cap + c) * LC_D + 8 * threadIdx.x, sum);
}
// Several clusters per workgroup: for many small clusters.  One workgroup each would read all the labels k
// times (5461 clusters of 10.9 K points, 8 heads: 1.9 GB of L2 reads per iteration).
__global__ void __launch_bounds__(LC_BT)
lc_kmeans_update_few_kernel(LcDev ix, int l, const float* pts, int pts_cap, float* cent, uint16_t* cent16, int cent_cap,
                            int it, int per, int* flags_all) {
    lc_fetch_args<sizeof(LcDev) + 40>();
    __shared__ LcBuckets bk;
    __shared__ __attribute__((aligned(16))) float sh[LC_BG * LC_D];
    const int h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    const int* const flags = flags_all ? lc_level_flags(ix, flags_all, l, bh) : nullptr;
    if (flags && it >= 1 && flags[it] == 0) return;                 // no point moved: the centroids stand
    const int sub = threadIdx.x & 15;
    const int N = lc_level_count(ix, b, bh, l);
    const int k = ix.nlev[b * LC_MAX_LEVELS + l + 1];
    const int c0 = blockIdx.x * per;
    if (c0 >= k) return;
    const int* labels = ix.parent[l] + (size_t)bh * ix.cap[l];
    const float* P = pts + (size_t)bh * pts_cap * LC_D;
    lc_cluster_sums<float>(
        [&](int i) { return labels[i]; }, N, c0, min(per, k - c0), bk, sh,
        [&](int i, float (&x)[8]) { lc_load8(P + (size_t)i * LC_D + 8 * sub, x); return 1; },
        [&](int c, int, float (&s)[8]) { lc_write_centroid(cent, cent16, ((size_t)bh * cent_cap + c) * LC_D + 8 * sub, s); });
}

// What is stored of node u of level l + 1 except its radius: center (mean of the descendant chunks'
// centers; the centroid for the unit geometry and for a node without chunks), counts, unit direction (the
// next level's point); the radius starts at -inf.  Called by one 16-lane group; centroid(mu): this lane's columns of the centroid.
struct LcNodeArgs {
    const float* cent;       // this level's centroids
    int cent_cap;
    int geometry;
    LcPointRows next;        // the next level's points and starting centroids
    __device__ __forceinline__ const float* centroid(int bh, int u) const { return cent + ((size_t)bh * cent_cap + u) * LC_D; }
};
template <typename Acc, typename CentroidF>
__device__ __forceinline__ void lc_write_node(const LcDev& ix, int b, int bh, int l, int u, int n_chunks, int n_tok,
                                              const Acc (&sum)[8], const LcNodeArgs& w, CentroidF centroid) {
    const int sub = threadIdx.x & 15;
    float mu[8];
    if (n_chunks > 0 && w.geometry == LC_GEOMETRY_TOKEN_BALL) {
        const Acc inv = (Acc)1 / (Acc)n_chunks;
#pragma unroll
        for (int t = 0; t < 8; ++t) mu[t] = (float)(sum[t] * inv);
    } else if (lc_level_count(ix, b, bh, l) > 0) {
        centroid(mu);
    } else {                                                        // (a sequence without chunks: no centroid was started)
#pragma unroll
        for (int t = 0; t < 8; ++t) mu[t] = (sub == 0 && t == 0) ? 1.f : 0.f;
    }
    const size_t n = (size_t)bh * ix.cap[l + 1] + u;
    lc_store8(ix.center[l + 1] + n * LC_D + 8 * sub, mu);
    float d[8];
    lc_unit_frag(mu, sub, d);
    if (w.next.pts)
        lc_store_point(w.next, bh, u, ix.nlev[b * LC_MAX_LEVELS + l + 1], ix.nlev[b * LC_MAX_LEVELS + l + 2], sub, d);
    if (sub == 0) {
        ix.radius[l + 1][n] = LC_NEG_INF;
        ix.rbuild[l + 1][n] = LC_NEG_INF;
        ix.parent[l + 1][n] = -1;
        ix.ntok[l + 1][n] = n_tok;
        ix.nchunk[l + 1][n] = n_chunks;
    }
}

// What a node of level l + 1 is made of: the chunks under it, or above the first level its child nodes, each weighted by
// the chunks it holds: a child's center is their mean, so the weighted sum is the sum over all descendant chunks.  It is taken in
// float64, so that its error is no larger than that of the float32 sum of the chunks (relative to the center, level 2 and
// 3 of 2275 chunks: 8.8e-8 and 2.2e-7 as the chunks' sum, 7.0e-8 and 1.3e-7 now).  Children instead of chunks: 143 nodes into 9
// and 9 into 1, 8 heads, 27 and 10 us, then 6.8 and 5.5; 5461 nodes into 249: 62 us, now 34.
template <bool NODES>
struct LcMembers {
    const float* center;             // rows of the members: float32, or bfloat16 at the chunk level if `half`
    const int* label;
    const int* ntok;
    const int* nchunk;               // NODES
    bool half;
    int n;
    __device__ __forceinline__ LcMembers(const LcDev& ix, int b, int bh, int l) {
        const size_t at = (size_t)bh * ix.cap[NODES ? l : 0];
        half = !NODES && ix.c0_bf16 != 0;
        center = half ? reinterpret_cast<const float*>(reinterpret_cast<const uint16_t*>(ix.center[0]) + at * LC_D)
                      : ix.center[NODES ? l : 0] + at * LC_D;
        label = ix.parent[NODES ? l : 0] + at;
        ntok = ix.ntok[NODES ? l : 0] + at;
        nchunk = NODES ? ix.nchunk[l] + at : nullptr;
        n = NODES ? ix.nlev[b * LC_MAX_LEVELS + l] : ix.state[bh * 4 + 1];
    }
    // columns [col, col + COLS) of member j's row; returns its weight
    template <int COLS>
    __device__ __forceinline__ int row(int j, int col, float (&x)[COLS]) const {
        const size_t o = (size_t)j * LC_D + col;
        const uint16_t* const c16 = reinterpret_cast<const uint16_t*>(center);
        if constexpr (COLS == 8) {
            if (half) lc_unpack8(*reinterpret_cast<const uint4*>(c16 + o), x);
            else lc_load8(center + o, x);
        } else if (half) {
            const uint32_t v = *reinterpret_cast<const uint32_t*>(c16 + o);
            x[0] = lc_bf16_lo(v);
            x[1] = lc_bf16_hi(v);
        } else {
            const float2 v = *reinterpret_cast<const float2*>(center + o);
            x[0] = v.x;
            x[1] = v.y;
        }
        return chunks(j);
    }
    __device__ __forceinline__ int chunks(int j) const { return NODES ? nchunk[j] : 1; }
};

// The whole clustering of a small level (up to LC_KS_MAX_N points into up to LC_KS_MAX_K clusters)
// in one kernel, one workgroup per (sequence, head): points, centroids and labels live in LDS (a wavefront's 16 points in its
// registers as well), the iterations are separated by workgroup barriers instead of kernel boundaries.  Same steps as the
// three kernels above: strided start, assign (ties to the lower id), normalised member sums (members
// added in ascending order; a cluster without members or with a zero sum keeps its centroid).
// What bounds an iteration is a chain: 32 dependent matrix instructions for each tile of a SIMD (2.2 us for the three of 143 points), two barriers, and
// the longest cluster's members one after the other, 16 rows in flight.  Up to 16 clusters (WIDE) a wavefront lists its cluster's members itself; beyond
// that all wavefronts make one list, between two more barriers.  With it for 143 points into 9 clusters too, and the one cluster of the 9 looked up
// for each of them, prefill of 128K tokens on one machine took 226.8 us, now 222.8 (the look-up alone 2.2 of it).  Without WIDE, sequences of up
// to 16 clusters beside a larger one still have a wavefront to a cluster: 4 of 224 to 100 points in 18 to 8 clusters 60.9 us without, now 59.7.
// The nodes themselves follow in the same kernel: the members' lists are in LDS, and a launch and its first round trips are worth more than
// the compute units that a workgroup per node would have.  143 nodes into 9 and 9 into 1: 27.6 and 6.5 us and
// 5.7 for each's nodes in a kernel of their own, 31.8 and 8.9 together (and two launches less); prefill of 128K tokens 288 us, now 285.
#define LC_KS_THREADS 1024        // a wavefront per 16 points, a 16-lane group per cluster
#define LC_KS_MAX_N 224
#define LC_KS_MAX_K 64
static_assert(LC_KS_MAX_N <= 16 * (LC_KS_THREADS / 64) && LC_KS_MAX_K <= LC_KS_THREADS / 16, "one tile per wavefront, one cluster per group");
static inline size_t lc_kmeans_small_lds(int N, int k) {
    return (size_t)((N > 0 ? N : 1) + ((k + 15) & ~15)) * LC_AS_ROW * sizeof(float);
}
template <bool NODES, bool WIDE>
__global__ void __launch_bounds__(LC_KS_THREADS)
lc_kmeans_small_kernel(LcDev ix, int l, const float* pts, int pts_cap, LcNodeArgs w, int iters, int x_rows) {
    lc_fetch_args<sizeof(LcDev) + 32 + sizeof(LcNodeArgs)>();
    extern __shared__ __attribute__((aligned(16))) float ks_dyn[];   // x_rows point rows, then the centroid rows
    __shared__ int lab[LC_KS_MAX_N];
    __shared__ int count[LC_KS_MAX_K];
    __shared__ __attribute__((aligned(16))) unsigned short mem[LC_KS_MAX_N + 8 * LC_KS_MAX_K];     // a cluster's list begins at a multiple of 8
    __shared__ __attribute__((aligned(16))) float sums[LC_KS_THREADS / 64][LC_D];
    __shared__ int changed[2];                    // labels changed in this iteration (one flag per parity of `it`)
    const int h = blockIdx.x, b = blockIdx.y;
    const int bh = b * ix.H + h;
    const int tid = threadIdx.x, sub = tid & 15, grp = tid >> 4, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, kk = lane >> 4;
    const int N = min(min(lc_level_count(ix, b, bh, l), LC_KS_MAX_N), x_rows);
    const int k = min(ix.nlev[b * LC_MAX_LEVELS + l + 1], WIDE ? LC_KS_THREADS / 64 : LC_KS_MAX_K);
    const int k16 = (k + 15) & ~15;
    const int rounds = (N + 63) >> 6;
    const float* P = pts + (size_t)bh * pts_cap * LC_D;
    float* X = ks_dyn;
    float* cs = ks_dyn + (size_t)x_rows * LC_AS_ROW;
    for (int v = tid; v < N * (LC_D / 4); v += LC_KS_THREADS) {
        const int i = v / (LC_D / 4), q = v % (LC_D / 4);
        *reinterpret_cast<float4*>(X + i * LC_AS_ROW + 4 * q) = *reinterpret_cast<const float4*>(P + (size_t)i * LC_D + 4 * q);
    }
    for (int i = tid; i < N; i += LC_KS_THREADS) { lab[i] = 0; mem[i] = (unsigned short)i; }
    if (tid < 2) changed[tid] = 0;
    __syncthreads();
    for (int v = tid; v < k16 * LC_D; v += LC_KS_THREADS) {
        const int c = v / LC_D, t = v % LC_D;
        float m = 0.f;
        if (c < k) m = N > 0 ? X[(int)(((long long)c * N) / k) * LC_AS_ROW + t] : (t == 0 ? 1.f : 0.f);
        cs[c * LC_AS_ROW + t] = m;
    }
    const int i0 = 16 * wave;                                       // this wavefront's points
    float4 xa[8];
    if (i0 < N) {
        const float* row = X + min(i0 + j, N - 1) * LC_AS_ROW + 4 * kk;
#pragma unroll
        for (int t = 0; t < 8; ++t) xa[t] = *reinterpret_cast<const float4*>(row + 16 * t);
    }
    __syncthreads();
    int n_c = lane == 0 ? N : 0, first = 0;                         // lane c: members of cluster c, where its list begins
    // WIDE: a wavefront to a cluster, which lists the members itself where its sums go afterwards.
    unsigned short* const own = reinterpret_cast<unsigned short*>(sums[wave]);
    static_assert(LC_KS_MAX_N * 2 + 32 <= sizeof(sums[0]), "read 16 members at a time");
    int n_own = 0;
    auto list_own = [&]() LC_INLINE {
        constexpr int R = (LC_KS_MAX_N + 63) / 64;
        int c[R];
#pragma unroll
        for (int r = 0; r < R; ++r) c[r] = lab[min(64 * r + lane, LC_KS_MAX_N - 1)];
        n_own = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool in = 64 * r + lane < N && c[r] == wave;
            const unsigned long long m = __ballot(in);
            if (in) own[n_own + lc_mbcnt(m)] = (unsigned short)(64 * r + lane);
            n_own += __popcll(m);
        }
        lc_wave_sync();
    };
    for (int it = 0; it < iters; ++it) {
        if (i0 < N && k > 1) {                                      // (one cluster: the labels stand as they are)
            float best[4];
            int arg[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) { best[r] = LC_NEG_INF; arg[r] = 0x7fffffff; }
            int cj = 0;
            for (; cj + 16 < k; cj += 32)
                lc_assign_block2(xa, cs + (cj + j) * LC_AS_ROW + 4 * kk, cs + (cj + 16 + j) * LC_AS_ROW + 4 * kk,
                                 cj + j, cj + 16 + j, k, best, arg);
            if (cj < k) lc_assign_block(xa, cs + (cj + j) * LC_AS_ROW + 4 * kk, cj + j, k, best, arg);
#pragma unroll
            for (int r = 0; r < 4; ++r) lc_assign_merge(best[r], arg[r]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ba = arg[r] < k ? arg[r] : 0, i = i0 + 4 * kk + r;     // (no similarity that compares: not-a-number)
                if (j == 0 && i < N) {
                    if (lab[i] != ba) changed[it & 1] = 1;
                    lab[i] = ba;
                }
            }
        }
        if (tid == 0) changed[(it + 1) & 1] = 0;                    // (last read before the previous barrier)
        __syncthreads();
        // An iteration that moves no point is a fixed point: the update would rebuild the same
        // centroids from the same members and every later iteration would repeat it, so the
        // remaining iterations are skipped (the first iteration always runs its update).
        if (it > 0 && changed[it & 1] == 0) break;
        if constexpr (WIDE) {
            if (wave < k) {
                list_own();
                float2 s = make_float2(0.f, 0.f);
                auto add = [&](auto rows, int q) LC_INLINE {        // (past the end: the batch's first row again)
                    constexpr int E = decltype(rows)::value;
                    unsigned id[E / 2];
                    float2 x[E];
#pragma unroll
                    for (int e = 0; e < E / 8; ++e) {
                        const uint4 v = *reinterpret_cast<const uint4*>(own + q + 8 * e);
                        id[4 * e] = v.x; id[4 * e + 1] = v.y; id[4 * e + 2] = v.z; id[4 * e + 3] = v.w;
                    }
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const int i = q + e < n_own ? (int)((id[e / 2] >> (16 * (e & 1))) & 0xffffu) : (int)(id[0] & 0xffffu);
                        x[e] = *reinterpret_cast<const float2*>(X + i * LC_AS_ROW + 2 * lane);
                    }
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        if (q + e < n_own) { s.x += x[e].x; s.y += x[e].y; }
                };
                int q = 0;
                for (; n_own - q > 8; q += 16) add(std::integral_constant<int, 16>(), q);
                if (q < n_own) add(std::integral_constant<int, 8>(), q);
                lc_wave_sync();                                     // (the list has been read)
                *reinterpret_cast<float2*>(sums[wave] + 2 * lane) = s;
                lc_wave_sync();
                float sum[8];
                lc_load8(sums[wave] + 8 * sub, sum);                // (every group the same)
                float n2 = 0.f;
#pragma unroll
                for (int t = 0; t < 8; ++t) n2 = fmaf(sum[t], sum[t], n2);
                n2 = lc_sum16(n2);
                if (n2 > 0.f) {
                    const float inv = 1.0f / sqrtf(n2);
#pragma unroll
                    for (int t = 0; t < 8; ++t) sum[t] *= inv;
                    if (lane < 16) lc_store8(cs + wave * LC_AS_ROW + 8 * sub, sum);
                }
                lc_wave_sync();                                     // (the next list comes where the sums were)
            }
            __syncthreads();
            continue;
        }
        // members of every cluster, ascending, as one list ordered by cluster: counts, then every wavefront works out the places
        for (int c = wave; c < k; c += LC_KS_THREADS / 64) {
            int n = 0;
            for (int r = 0; r < rounds; ++r) {
                const int i = lane + 64 * r;
                n += __popcll(__ballot(i < N && lab[i] == c));
            }
            if (lane == 0) count[c] = n;
        }
        __syncthreads();
        n_c = lane < k ? count[lane] : 0;
        const int room = (n_c + 7) & ~7;
        first = lc_wave_scan_incl(room) - room;
        for (int c = wave; c < k; c += LC_KS_THREADS / 64) {
            int at = lc_readlane(first, c);
            for (int r = 0; r < rounds; ++r) {
                const int i = lane + 64 * r;
                const bool in = i < N && lab[i] == c;
                const unsigned long long m = __ballot(in);
                if (in) mem[at + lc_mbcnt(m)] = (unsigned short)i;
                at += __popcll(m);
            }
        }
        __syncthreads();
        {
            // up to 16 clusters: a wavefront each, two columns per lane; beyond that a 16-lane group each, eight columns per lane
            const bool wide = k <= LC_KS_THREADS / 64;
            const int c = wide ? wave : grp;                        // (clusters past the last have no members)
            const int n = __shfl(n_c, min(c, 63)), at = __shfl(first, min(c, 63));
            float sum[8];
            auto add_rows = [&](auto cols, int col) LC_INLINE {
                constexpr int C = decltype(cols)::value;
#pragma unroll
                for (int t = 0; t < 8; ++t) sum[t] = 0.f;
                for (int q = 0; q < n; q += 8) {
                    const uint4 id = *reinterpret_cast<const uint4*>(mem + at + q);
                    const uint32_t w[4] = {id.x, id.y, id.z, id.w};
                    float x[8][C];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {                   // (past the end: the batch's first row again)
                        const int i = q + e < n ? (int)((w[e / 2] >> (16 * (e & 1))) & 0xffffu) : (int)(w[0] & 0xffffu);
                        if constexpr (C == 8) {
                            lc_load8(X + i * LC_AS_ROW + col, x[e]);
                        } else {
                            const float2 v = *reinterpret_cast<const float2*>(X + i * LC_AS_ROW + col);
                            x[e][0] = v.x;
                            x[e][1] = v.y;
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (q + e < n) {
#pragma unroll
                            for (int t = 0; t < C; ++t) sum[t] += x[e][t];
                        }
                }
            };
            if (wide) {
                add_rows(std::integral_constant<int, 2>(), 2 * lane);
                *reinterpret_cast<float2*>(sums[wave] + 2 * lane) = make_float2(sum[0], sum[1]);
                lc_wave_sync();
                lc_load8(sums[wave] + 8 * sub, sum);                // (every group the same)
            } else {
                add_rows(std::integral_constant<int, 8>(), 8 * sub);
            }
            float n2 = 0.f;
#pragma unroll
            for (int t = 0; t < 8; ++t) n2 = fmaf(sum[t], sum[t], n2);
            n2 = lc_sum16(n2);
            if (n > 0 && n2 > 0.f) {
                const float inv = 1.0f / sqrtf(n2);
#pragma unroll
                for (int t = 0; t < 8; ++t) sum[t] *= inv;
                if (!wide || lane < 16) lc_store8(cs + c * LC_AS_ROW + 8 * sub, sum);
            }
        }
        __syncthreads();
    }
    for (int i = tid; i < N; i += LC_KS_THREADS) ix.parent[l][(size_t)bh * ix.cap[l] + i] = lab[i];
    // ---- the nodes: the lists are those of the labels as they stand.  A wavefront per node, its groups taking the members in turn, or
    // beyond 16 nodes a group each; four rows per group in flight.
    const bool wide = WIDE || k <= LC_KS_THREADS / 64;
    if (WIDE && wave < k) list_own();
    const int c = wide ? wave : grp;
    const int n = WIDE ? n_own : __shfl(n_c, min(c, 63)), at = WIDE ? 0 : __shfl(first, min(c, 63));     // (while every lane is there)
    const unsigned short* const list = WIDE ? own : mem;
    if (c >= k) return;
    const LcMembers<NODES> m(ix, b, bh, l);
    const int step = wide ? 4 : 1;
    double sum[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) sum[t] = 0.0;
    for (int q = wide ? kk : 0; q < n; q += 4 * step) {
        float x[4][8];
        int weight[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) weight[e] = m.row((int)list[at + min(q + step * e, n - 1)], 8 * sub, x[e]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (q + step * e < n) lc_add_row(sum, x[e], weight[e]);
    }
    int tok = 0, chunks = 0;
    for (int q = wide ? lane : sub; q < n; q += 16 * step) {
        const int i = list[at + q];
        tok += m.ntok[i];
        chunks += m.chunks(i);
    }
    tok = lc_sum16_i(tok);
    chunks = lc_sum16_i(chunks);
    if (wide) {
        tok += __shfl_xor(tok, 16);
        chunks += __shfl_xor(chunks, 16);
        tok += __shfl_xor(tok, 32);
        chunks += __shfl_xor(chunks, 32);
#pragma unroll
        for (int t = 0; t < 8; ++t) sum[t] += __shfl_xor(sum[t], 16);
#pragma unroll
        for (int t = 0; t < 8; ++t) sum[t] += __shfl_xor(sum[t], 32);
    }
    if (!wide || lane < 16) lc_write_node(ix, b, bh, l, c, chunks, tok, sum, w, [&](float (&mu)[8]) { lc_load8(cs + c * LC_AS_ROW + 8 * sub, mu); });
}

// ---------------------------------------------------------------------------------
// A whole clustering into up to LC_AS_RES clusters, and its nodes, in one kernel of several workgroups per (sequence, head)
// ---------------------------------------------------------------------------------
// An iteration is two steps, labels and centroids, each of which needs all of the other's results.  As launches of
// lc_kmeans_assign_res_kernel and lc_kmeans_update_*_kernel each step costs its launch, three dependent round trips and the
// wait for the slowest of all (sequence, head)s.  Here the workgroups of a (sequence, head) stay, one to a compute unit, and post for each
// other: labels, then the centroids of the clusters that a label came to or left; all read all labels and those centroids.
// Every iteration posts into memory of its own that an earlier kernel has filled with LC_UNPOSTED, so each 32-bit word shows by
// itself whether it has been posted: there is no counter, no order between stores and nothing that a late workgroup could overwrite.
// Nobody depends on another workgroup: a wavefront that has looked for a word LC_RK_LOOKS times works out what is missing itself --
// everything follows from the points and the words before -- and posts it (same bits), so every wait ends whatever else occupies the device.
// What a wavefront works out for others it takes from the missing words by its workgroup's number, so that those that wait share
// it.  Re-clustering with half of each head's workgroups in a second launch, us when all took the first missing word after twice as many
// looks, and now: 8 heads of 1000 points 507 and 265, of 2275 830 and 445, of 5461 2200 and 880 (all in one launch: 83, 119 and 262).
// On a device that is shared (8 heads of 2275 points, an index of two levels, us a build with two kernels an iteration and now):
// alone 177 and 134; with another build at the same time 228 and 222 for both, with two 300 and 576 for the three (948 when all took the first
// missing word); beside eight decode steps 203 and 232, beside 4096^3 matrix products 963 and 508, beside copies of a gigabyte 331 and 490.
// A cluster that has lost its members keeps its centroid: the one of an earlier iteration's plane, all of which the workgroup has seen (LcPlanes).
// Labels, centroids and nodes are the bits of the kernels it stands for: members are added in the same order.
// What bounds an iteration of about 10 us is single wavefronts' instructions: 3 us a cluster (its members listed, their rows' round trip, the sum and
// its direction), 2 us 16 points against 160 centroids, and twice a store's way and a look.  512 threads: with 1024 the registers of a sum do not fit.
// Where the numbers of points allow it the workgroups of a (sequence, head) share an XCD, whose L2 then holds the points' rows (lay_out_shares).
// Measured, us a build with two kernels an iteration and now: 8 heads of 2275 points, 143 clusters and two small levels 234 and 203; 64 pairs of up
// to 1820 in 57 334 and 307; 8 of 820 in 52 121 and 88; 8 of 10.9 K in 5461, then of those in 249 850 and 792.
#define LC_RK_THREADS 512
#define LC_RK_WAVES (LC_RK_THREADS / 64)
#define LC_RK_MAX_N LC_RK_MAX_POINTS
#define LC_RK_LIST 768                       // members that a wavefront lists before it adds their rows
#define LC_RK_LOOKS 64                       // times a wavefront looks (1.6 us each) before it works out what is missing
#define LC_RK_LOOKS_AGAIN 1                  // and once it has (twice as many after each wait that ended by itself)
#define LC_RK_LOOK_MEMBERS 16                // members that are added in the time of a look, at least: it waits so much longer for a centroid
#define LC_RK_LOOKS_MOST 1024                // more than a wavefront has words to wait for: the wait ends whatever is in memory
#define LC_RK_WAIT_ROWS 20                   // 64 clocks each: a wavefront without clusters of its own waits before it looks for centroids,
#define LC_RK_WAIT_LABELS 20                 // one without points before it looks for labels
struct LcRounds {
    float* rows;             // [iters + 1][B][H][k][d] centroids: those that iteration i starts with in plane i, as far as they are new there
    int* labels;             // [iters][B][H][words] two labels a word
    int k, words;            // most clusters; words of a (sequence, head), 8 for 16 points
    int row_bytes, label_bytes;
    LcUnposted unposted;     // planes 1 and up, and the labels
};
// Which part of which (sequence, head) a workgroup is: pair, part << 8, parts of the pair << 16; LC_RK_NO_PART without work.
#define LC_RK_NO_PART 0xffffffffu
struct LcShares {
    uint32_t of[LC_COMPUTE_UNITS];
};
struct LcRkWave {
    union {
        struct {
            unsigned long long best[16];             // of a point: similarity (as an integer that orders like it), ~centroid
            int pair[LC_AS_PAIRS];                   // centroid << 4 | point
        };
        unsigned short list[LC_RK_LIST + 8];     // (a place for what is not listed)
    };
};
// similarities of 16 points and 16 centroids, 32 columns a lane (see lc_assign_block)
__device__ __forceinline__ lc_f32x4_b lc_assign_products(const float4 (&x)[8], const float4 (&m)[8]) {
    lc_f32x4_b d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t].x, m[t].x, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t].y, m[t].y, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t].z, m[t].z, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t].w, m[t].w, d, 0, 0, 0);
    }
    return d;
}
// Labels of 16 points, `n` of them real, by one wavefront; the label of point `lane` in lanes < 16.  Candidates are found as in
// lc_kmeans_assign_res_kernel: a point with one has its label, the others' candidates are compared in float32, 16 (point,
// candidate) pairs to a block of products of all 16 points with 16 candidates; beyond LC_AS_PAIRS of them with all centroids.
// rows: the centroids in bfloat16 (LDS, the last one repeated); centroid(c, q): piece q of four columns of centroid c's float32 row;
// meanwhile(): called once the bfloat16 similarities have been looked through.
struct LcTile {
    lc_v4i half[4];          // A operand in bfloat16
    float4 full[8];          // and in float32
};
template <int NBLK, typename CentroidF, typename MeanwhileF>
__device__ __forceinline__ int lc_rounds_label(LcRkWave& sh, const unsigned char* rows, const LcTile& p, int n, int k, CentroidF centroid,
                                               MeanwhileF meanwhile) {
    const int lane = threadIdx.x & 63, j = lane & 15, kk = lane >> 4;
    // one or two blocks at a time, the next one's rows read before their products (each with its own reads in front of it took 350 clocks)
    lc_f32x4_b d[NBLK];
    constexpr int AT = NBLK <= 4 ? 2 : 1;                           // (registers)
    lc_v4i m[2][AT][4];
    auto read = [&](int e) LC_INLINE {
#pragma unroll
        for (int q = 0; q < AT; ++q)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                m[(e / AT) & 1][q][s] = *reinterpret_cast<const lc_v4i*>(rows + (16 * (e + q) + j) * LC_AS_PITCH + 16 * kk + 64 * s);
    };
    read(0);
#pragma unroll
    for (int e = 0; e < NBLK; e += AT) {
        if (e + AT < NBLK) read(e + AT);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < AT; ++q) d[e + q] = lc_f32x4_b{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int q = 0; q < AT; ++q)
                d[e + q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(lc_bf16x8_b, p.half[s]),
                                                                   __builtin_bit_cast(lc_bf16x8_b, m[(e / AT) & 1][q][s]), d[e + q], 0, 0, 0);
    }
    if (lane < 16) sh.best[lane] = 0ull;
    constexpr int WORDS = (NBLK + 7) / 8;
    unsigned hit[WORDS][4];                                         // [w][r]: candidates 16 (8 w + e) + j of point 4 kk + r in bit 7 - e
    int only[4];                                                    // candidates of point 4 kk + r << 16, and the sum of their numbers
    float top[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        top[r] = d[0][r];
#pragma unroll
        for (int e = 1; e < NBLK; ++e) top[r] = fmaxf(top[r], d[e][r]);
    }
    // largest of every row (the four rows' steps together: none waits for the one before), less the margin
#pragma unroll
    for (int r = 0; r < 4; ++r) top[r] = fmaxf(top[r], lc_dpp<0xB1>(top[r]));
#pragma unroll
    for (int r = 0; r < 4; ++r) top[r] = fmaxf(top[r], lc_dpp<0x4E>(top[r]));
#pragma unroll
    for (int r = 0; r < 4; ++r) top[r] = fmaxf(top[r], lc_dpp<0x141>(top[r]));
#pragma unroll
    for (int r = 0; r < 4; ++r) top[r] = fmaxf(top[r], lc_dpp<0x140>(top[r])) - 2.0f * LC_AS_EPS;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        only[r] = 0;
#pragma unroll
        for (int w = 0; w < WORDS; ++w) {
            unsigned below = 0u;                                    // sign bits, the last block's in bit 0
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (8 * w + e < NBLK) below = __builtin_amdgcn_alignbit(below, __float_as_uint(d[8 * w + e < NBLK ? 8 * w + e : 0][r] - top[r]), 31);
                else below = below << 1 | 1u;
            const int real = min(max((k - 128 * w - j + 15) >> 4, 0), 8);       // blocks with a centroid in this column
            const unsigned h = ~below & (0xff00u >> real) & 0xffu;
            hit[w][r] = h;
            const int own = (__popc(h) << 16) + 16 * (8 * w + 8 - __ffs((int)h)) + j;
            only[r] += h != 0u ? own : 0;                           // (one of several: the number is not used then)
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) only[r] += __builtin_amdgcn_update_dpp(0, only[r], 0xB1, 0xF, 0xF, true);
#pragma unroll
    for (int r = 0; r < 4; ++r) only[r] += __builtin_amdgcn_update_dpp(0, only[r], 0x4E, 0xF, 0xF, true);
#pragma unroll
    for (int r = 0; r < 4; ++r) only[r] += __builtin_amdgcn_update_dpp(0, only[r], 0x141, 0xF, 0xF, true);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        only[r] += __builtin_amdgcn_update_dpp(0, only[r], 0x140, 0xF, 0xF, true);
        only[r] = 4 * kk + r < n ? only[r] : 1 << 16;
    }
    meanwhile();
    lc_wave_sync();
    int n_pairs = 0;
    bool all = false;                                               // no similarity that compares
    const bool two = max(max(only[0], only[1]), max(only[2], only[3])) >= 2 << 16, none = min(min(only[0], only[1]), min(only[2], only[3])) < 1 << 16;
    if (__ballot(two || none) != 0ull) {
        all = __ballot(none) != 0ull;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int w = 0; w < WORDS; ++w) {
                unsigned h = only[r] >= 2 << 16 ? hit[w][r] : 0u;
                for (unsigned long long m; (m = __ballot(h != 0u)) != 0ull;) {
                    const int at = n_pairs + lc_mbcnt(m), e = 8 - __ffs((int)h);
                    if (h != 0u && at < LC_AS_PAIRS) sh.pair[at] = (16 * (8 * w + e) + j) << 4 | (4 * kk + r);
                    h &= h - 1u;
                    n_pairs += __popcll(m);
                }
            }
        all = all || n_pairs > LC_AS_PAIRS;
        lc_wave_sync();
    }
    const auto take = [&](float v, int c, int i) LC_INLINE {        // (not a number: compares with nothing)
        const unsigned u = __float_as_uint(v + 0.0f), key = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
        if (v == v) atomicMax(&sh.best[i], (unsigned long long)key << 32 | (unsigned)~c);
    };
    for (int q0 = 0; q0 < (all ? 0 : n_pairs); q0 += 16) {
        const int pair = sh.pair[min(q0 + j, n_pairs - 1)], c = pair >> 4, i = pair & 15;
        float4 m[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) m[t] = centroid(c, 4 * t + kk);
        const lc_f32x4_b s = lc_assign_products(p.full, m);         // row i, column j
        const float v = (i & 2) ? ((i & 1) ? s[3] : s[2]) : ((i & 1) ? s[1] : s[0]);
        if (kk == (i >> 2)) take(v, c, i);
    }
    if (all) {
        for (int c0 = 0; c0 < k; c0 += 16) {
            const int c = min(c0 + j, k - 1);
            float4 m[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) m[t] = centroid(c, 4 * t + kk);
            const lc_f32x4_b s = lc_assign_products(p.full, m);
#pragma unroll
            for (int r = 0; r < 4; ++r) take(s[r], c, 4 * kk + r);
        }
    }
    lc_wave_sync();
    const int r = lane & 3, from = (lane & 12) << 2;                // point `lane`: row r of lanes 16 (lane / 4) + (0..15)
    const int o0 = __shfl(only[0], from), o1 = __shfl(only[1], from), o2 = __shfl(only[2], from), o3 = __shfl(only[3], from);
    const int o = (r & 2) ? ((r & 1) ? o3 : o2) : ((r & 1) ? o1 : o0);
    const unsigned long long b = sh.best[lane & 15];
    lc_wave_sync();
    if (!all && o >> 16 == 1) return o & 0xffff;
    const int c = b != 0ull ? (int)~(unsigned)b : 0;
    return c < k ? c : 0;
}
// Exchanges between the rows of 16 lanes: afterwards `a` holds the even rows' a and b, `b` the odd rows' (rows 0, 1 and 2, 3), and the
// same for the wavefront's halves.
__device__ __forceinline__ void lc_swap16(float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void lc_swap32(float& a, float& b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void lc_swap16(double& a, double& b) {
    const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    a = __longlong_as_double((long long)((unsigned long long)hi[0] << 32 | lo[0]));
    b = __longlong_as_double((long long)((unsigned long long)hi[1] << 32 | lo[1]));
}
__device__ __forceinline__ void lc_swap32(double& a, double& b) {
    const unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
    a = __longlong_as_double((long long)((unsigned long long)hi[0] << 32 | lo[0]));
    b = __longlong_as_double((long long)((unsigned long long)hi[1] << 32 | lo[1]));
}
// Sum of the rows of a cluster's members, by one wavefront, in the order of lc_cluster_sums: the members, ascending, are dealt to 16
// partial sums in turn (starting over every LC_MEM_WIN points), and the partial sums are added up in turn.  Group g of 16 lanes keeps the
// partials 4 e + g.  members(b): this lane's word of the 64 blocks of 64 points from block b on, a bit per member; row(i, x): columns
// [8 sub, 8 sub + 8) of point i's row, returns its weight, zeros for i < 0; visit(i) once per member.  Every group gets the sums.
template <typename Acc, typename MembersF, typename RowF, typename VisitF>
__device__ __forceinline__ void lc_rounds_sum(int N, unsigned short* list, MembersF members, RowF row, VisitF visit, Acc (&sum)[8]) {
    constexpr int U = sizeof(Acc) == 4 ? 2 : 1;                     // rows of a partial in flight
    static_assert(LC_MEM_WIN == 64 * 64 && LC_RK_LIST % 16 == 0, "a word per lane; a partial is a place in the list modulo 16");
    const int lane = threadIdx.x & 63, g4 = lane >> 4;
    Acc acc[4][8];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[e][t] = 0;
    for (int base = 0; base < N; base += LC_MEM_WIN) {
        const unsigned long long word = members(base >> 6);
        const int n = __popcll(word), inc = lc_wave_scan_incl(n), total = lc_readlane(inc, 63);
        for (int r0 = 0; r0 < total; r0 += LC_RK_LIST) {
            lc_wave_sync();                                         // (the list's place had another use)
            unsigned lo = (unsigned)word, hi = (unsigned)(word >> 32);
            for (int a = inc - n - r0, z = a + __popc(lo); (lo | hi) != 0u; lo &= lo - 1u, hi &= hi - 1u, ++a, ++z) {
                list[lo != 0u && (unsigned)a < LC_RK_LIST ? a : LC_RK_LIST] = (unsigned short)(base + 64 * lane + __ffs((int)lo) - 1);
                list[hi != 0u && (unsigned)z < LC_RK_LIST ? z : LC_RK_LIST] = (unsigned short)(base + 64 * lane + __ffs((int)hi) + 31);
            }
            const int m = min(total - r0, LC_RK_LIST);
            lc_wave_sync();
            for (int t0 = 0; t0 < m; t0 += 16 * U) {
                float x[4 * U][8];
                int w[4 * U];
#pragma unroll
                for (int e = 0; e < 4 * U; ++e) {
                    const int t = t0 + 4 * e + g4;
                    const int i = list[min(t, m - 1)];
                    w[e] = row(t < m ? i : -1, x[e]);
                }
#pragma unroll
                for (int e = 0; e < 4 * U; ++e) lc_add_row(acc[e & 3], x[e], w[e]);
            }
            for (int t = lane; t < m; t += 64) visit((int)list[t]);
        }
    }
    // two columns a lane of all 16 partials, added up in turn, then eight columns again
    Acc s2[2] = {0, 0};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int t = 0; t < 4; ++t) lc_swap32(acc[e][t], acc[e][t + 4]);     // [t]: groups 0, 1; [t + 4]: groups 2, 3; columns t + 4 (g4 / 2)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            lc_swap16(acc[e][t], acc[e][t + 2]);                             // groups 0 and 1; columns t + 2 g4
            lc_swap16(acc[e][t + 4], acc[e][t + 6]);                         // groups 2 and 3
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            s2[t] += acc[e][t];
            s2[t] += acc[e][t + 2];
            s2[t] += acc[e][t + 4];
            s2[t] += acc[e][t + 6];
        }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) { sum[t] = s2[t]; sum[t + 2] = s2[t]; lc_swap16(sum[t], sum[t + 2]); }
#pragma unroll
    for (int t = 0; t < 4; ++t) { sum[t + 4] = sum[t]; lc_swap32(sum[t], sum[t + 4]); }
}
// The number of the n-th bit that is set (from 0; there are more than n).
__device__ __forceinline__ int lc_nth_bit(unsigned long long m, int n) {
    for (; n > 0; --n) m &= m - 1ull;
    return __ffsll((long long)m) - 1;
}
template <int NBLK, bool NODES>
__global__ void __launch_bounds__(LC_RK_THREADS)
lc_kmeans_rounds_kernel(LcDev ix, int l, const float* pts, const uint16_t* pts16, int pts_cap, LcNodeArgs w, int iters, LcRounds rd, LcShares shares) {
    lc_fetch_args<sizeof(LcDev) + 32 + sizeof(LcNodeArgs) + sizeof(LcRounds)>();
    const unsigned share = shares.of[blockIdx.x];
    if (share == LC_RK_NO_PART) return;
    __shared__ __attribute__((aligned(16))) unsigned char rows[16 * NBLK * LC_AS_PITCH];
    constexpr bool FULL = NBLK <= 10;             // the float32 rows find room as well, piece q of row c at q ^ (c mod 32)
    __shared__ lc_v4i full[FULL ? 16 * NBLK * 32 : 1];
    __shared__ lc_v4i lab[LC_RK_MAX_N / 8];
    __shared__ __attribute__((aligned(16))) LcRkWave own_sh[LC_RK_WAVES];
    __shared__ int fresh[LC_AS_RES];              // iteration that starts with a new centroid of this cluster
    __shared__ LcPlanes<LC_AS_RES> planes;        // plane of the centroid that is in `rows`
    __shared__ int moved;                         // last iteration that moved a point
    constexpr int BITS = NBLK <= 10 && NBLK > 8 ? 512 : 2048;
    __shared__ unsigned long long bits[BITS];     // [mine][blocks] members of this workgroup's clusters, a bit per point
    __shared__ signed char mine_of[LC_AS_RES];    // which of this workgroup's clusters this is, or -1
    const int bh = share & 0xff, BH = ix.B * ix.H;
    const int b = bh / ix.H;
    const int part = (share >> 8) & 0xff, parts = (share >> 16) & 0xff;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, kk = lane >> 4, sub = j;
    const int first = part + parts * wave, step = parts * LC_RK_WAVES;     // this wavefront's tiles of 16 points, and its clusters
    const int N = min(min(lc_level_count(ix, b, bh, l), LC_RK_MAX_N), 2 * rd.words);
    const int k = min(min(ix.nlev[b * LC_MAX_LEVELS + l + 1], 16 * NBLK), rd.k);
    const int tiles = (N + 15) >> 4, pieces = 2 * tiles, blocks = (N + 63) >> 6;
    const int n_mine = (part < k ? k - 1 - part : -1) / parts + 1;
    const bool keep_bits = n_mine <= 127 && n_mine * blocks <= BITS;
    LcRkWave& sh = own_sh[wave];
    const float* const P = pts + (size_t)bh * pts_cap * LC_D;
    const __amdgpu_buffer_rsrc_t points_r = lc_buffer(P, N * LC_D * 4);
    const __amdgpu_buffer_rsrc_t rows_r = lc_buffer(rd.rows, rd.row_bytes), labels_r = lc_buffer(rd.labels, rd.label_bytes);
    auto row_at = [&](int p, int c) LC_INLINE { return ((p * BH + bh) * rd.k + c) * (LC_D * 4); };
    auto label_at = [&](int it, int word) LC_INLINE { return ((it * BH + bh) * rd.words + word) * 4; };
    auto load_half = [&](lc_v4i (&half)[4], int t) LC_INLINE {
        const uint16_t* const row = pts16 + ((size_t)bh * pts_cap + min(16 * t + j, N - 1)) * LC_D + 8 * kk;
#pragma unroll
        for (int s = 0; s < 4; ++s) half[s] = *reinterpret_cast<const lc_v4i*>(row + 32 * s);
    };
    // this lane's word of the blocks from b0 on (see lc_rounds_sum): kept as labels change for my own clusters, from the labels for others
    auto members = [&](int own, int c, int b0) LC_INLINE {
        if (own >= 0) return b0 + lane < blocks ? bits[own * blocks + min(b0 + lane, blocks - 1)] : 0ull;
        unsigned long long word = 0ull;
        for (int i = 0; i < min(blocks - b0, 64); ++i) {
            const unsigned long long m = __ballot(reinterpret_cast<const unsigned short*>(lab)[64 * (b0 + i) + lane] == c);
            word = lane == i ? m : word;
        }
        return word;
    };
    auto centroid = [&](int it, int c, int q) LC_INLINE {
        if constexpr (FULL) return __builtin_bit_cast(float4, full[32 * c + (q ^ (c & 31))]);
        else return lc_load_agent4(rows_r, row_at(planes.now(it, c), c) + 16 * q);
    };
    constexpr int PIECES = LC_RK_MAX_N / 8 / LC_RK_THREADS;         // pieces of labels of a thread
#pragma unroll
    for (int e = 0; e < PIECES; ++e) lab[tid + e * LC_RK_THREADS] = lc_v4i{-1, -1, -1, -1};
    if (tid < LC_AS_RES) { fresh[tid] = 0; planes.start(tid); }
    if (tid == 0) moved = -1;
    if (keep_bits)
        for (int i = tid; i < n_mine * blocks; i += LC_RK_THREADS) bits[i] = 0ull;
    if (tid < LC_AS_RES) mine_of[tid] = (signed char)(keep_bits && tid < k && tid % parts == part ? tid / parts : -1);
    lc_barrier_lds();
    int patience = LC_RK_LOOKS;
    for (int it = 0; N > 0; ++it) {
        // ---- the centroids of my clusters that the last iteration changed; then everybody's, into LDS
        constexpr int R = 8 * NBLK / LC_RK_WAVES;                   // rows of a lane: half a wavefront to a row
        unsigned open = 0u;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int c = 2 * (wave + LC_RK_WAVES * i) + (lane >> 5);
            open |= it < iters && c < k && fresh[min(c, LC_AS_RES - 1)] == it ? 1u << i : 0u;
        }
        if (tid < LC_AS_RES) planes.enter(it, tid, fresh[tid] == it);     // (by the wavefronts that look for the rows: 3.5 us of prefill's 228)
        int looks = 0;
        lc_v4i next[4];                                             // the next tile's rows in bfloat16
        if (it > 0 && first >= k) __builtin_amdgcn_s_sleep(LC_RK_WAIT_ROWS);
        for (int own = it == 0 ? k : first, at = wave;;) {
            int c, mine = -1;
            if (own < k) {
                c = own;
                mine = keep_bits ? at : -1;
                own += step;
                at += LC_RK_WAVES;
                if (__builtin_amdgcn_readfirstlane(fresh[c]) != it) continue;
            } else {
                if (looks == 0) load_half(next, min(first, tiles - 1));
                lc_v4i v[R];
                asm volatile("" ::: "memory");                      // every look is a load of its own
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const int row = 2 * (wave + LC_RK_WAVES * i) + (lane >> 5);
                    v[i] = __builtin_amdgcn_raw_buffer_load_b128(rows_r, (open >> i) & 1u ? row_at(it, row) + 16 * (lane & 31) : 0x7ffffff0, 0, 16);
                }
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const int row = 2 * (wave + LC_RK_WAVES * i) + (lane >> 5);
                    const bool there = it == 0 || (v[i].x != LC_UNPOSTED && v[i].y != LC_UNPOSTED && v[i].z != LC_UNPOSTED && v[i].w != LC_UNPOSTED);
                    if (((open >> i) & 1u) && there) {
                        const int x = v[i].x, y = v[i].y, z = v[i].z, u = v[i].w;
                        *reinterpret_cast<uint2*>(rows + row * LC_AS_PITCH + 8 * (lane & 31)) =
                            make_uint2(lc_f32_to_bf16_bits(__int_as_float(x)) | (lc_f32_to_bf16_bits(__int_as_float(y)) << 16),
                                       lc_f32_to_bf16_bits(__int_as_float(z)) | (lc_f32_to_bf16_bits(__int_as_float(u)) << 16));
                        if (row == k - 1)                           // (absent centroids repeat the last)
                            for (int a = k; a < 16 * NBLK; ++a)
                                *reinterpret_cast<uint2*>(rows + a * LC_AS_PITCH + 8 * (lane & 31)) = *reinterpret_cast<const uint2*>(rows + row * LC_AS_PITCH + 8 * (lane & 31));
                        if constexpr (FULL) full[32 * row + ((lane & 31) ^ (row & 31))] = v[i];
                        open &= ~(1u << i);
                    }
                }
                if (__ballot(open != 0u) == 0ull || looks == LC_RK_LOOKS_MOST) break;
                if (++looks <= patience) { __builtin_amdgcn_s_sleep(1); continue; }
                unsigned missing = 0u;                              // rows of this wavefront; another one to each workgroup that helps
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    const unsigned long long m = __ballot((open >> i) & 1u);
                    missing |= (unsigned)((unsigned)m != 0u) << (2 * i) | (unsigned)((unsigned)(m >> 32) != 0u) << (2 * i + 1);
                }
                const int row = lc_nth_bit(missing, part % __popc(missing));
                c = 2 * (wave + LC_RK_WAVES * (row >> 1)) + (row & 1);
                int n = 0;                                          // (a large cluster takes whoever has begun with it as long)
                for (int b0 = 0; b0 < blocks; b0 += 64) n += lc_wave_sum_i(__popcll(members(-1, c, b0)));
                if (looks <= patience + n / LC_RK_LOOK_MEMBERS) { __builtin_amdgcn_s_sleep(1); continue; }
                patience = LC_RK_LOOKS_AGAIN;
            }
            float sum[8];
            lc_rounds_sum<float>(N, sh.list, [&](int b0) LC_INLINE { return members(mine, c, b0); },
                                 [&](int i, float (&x)[8]) LC_INLINE {        // (no member: past the end, which reads as zeros)
                                     const int o = i >= 0 ? i * (LC_D * 4) + 32 * sub : 0x7fffffe0;
                                     const float4 a = lc_buf_load_f32x4(points_r, o), z = lc_buf_load_f32x4(points_r, o + 16);
                                     x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
                                     x[4] = z.x; x[5] = z.y; x[6] = z.z; x[7] = z.w;
                                     return 1;
                                 }, [](int) {}, sum);
            float n2 = 0.f;
#pragma unroll
            for (int t = 0; t < 8; ++t) n2 = fmaf(sum[t], sum[t], n2);
            n2 = lc_sum16(n2);
            const float inv = 1.0f / sqrtf(n2);
#pragma unroll
            for (int t = 0; t < 8; ++t) sum[t] *= inv;
            float4 half = kk == 0 ? make_float4(sum[0], sum[1], sum[2], sum[3]) : make_float4(sum[4], sum[5], sum[6], sum[7]);
            const int o = 32 * sub + 16 * (kk & 1);
            // no members, or none in sum: the centroid stands, and this iteration's plane may still be in the making
            if (!(n2 > 0.f)) half = lc_load_agent4(rows_r, row_at(planes.before(it, c), c) + o);
            auto posted = [](float f) LC_INLINE { return __float_as_int(f) == LC_UNPOSTED ? __int_as_float(0x7fc00000) : f; };
            half = make_float4(posted(half.x), posted(half.y), posted(half.z), posted(half.w));
            if (kk < 2) lc_store_agent4(rows_r, row_at(it, c) + o, half);
            if (own >= k) __builtin_amdgcn_s_waitcnt(0);            // (my own posts are there when I look)
        }
        if (it == iters) break;
        if (looks <= patience) patience = min(2 * patience, LC_RK_LOOKS);
        lc_barrier_lds();
        // ---- the labels of my points, then everybody's
        lc_v4i v[PIECES];
        bool wait[PIECES];
#pragma unroll
        for (int e = 0; e < PIECES; ++e) { v[e] = lc_v4i{0, 0, 0, 0}; wait[e] = tid + e * LC_RK_THREADS < pieces; }
        looks = 0;
        if (first >= tiles) __builtin_amdgcn_s_sleep(LC_RK_WAIT_LABELS);
        for (int own = first;;) {
            int t;
            if (own < tiles) {
                t = own;
                own += step;
            } else {
                asm volatile("" ::: "memory");
#pragma unroll
                for (int e = 0; e < PIECES; ++e)
                    if (wait[e]) v[e] = __builtin_amdgcn_raw_buffer_load_b128(labels_r, label_at(it, 4 * (tid + e * LC_RK_THREADS)), 0, 16);
                unsigned long long missing[PIECES];
                int n_missing = 0;
#pragma unroll
                for (int e = 0; e < PIECES; ++e) {
                    wait[e] = wait[e] && (v[e].x == LC_UNPOSTED || v[e].y == LC_UNPOSTED || v[e].z == LC_UNPOSTED || v[e].w == LC_UNPOSTED);
                    missing[e] = __ballot(wait[e]);
                    n_missing += __popcll(missing[e]);
                }
                if (n_missing == 0 || looks == LC_RK_LOOKS_MOST) break;
                if (++looks <= patience) { __builtin_amdgcn_s_sleep(1); continue; }
                patience = LC_RK_LOOKS_AGAIN;
                int n = 2 * part % n_missing, piece = -1;           // (two pieces to a tile; another tile to each workgroup that helps)
#pragma unroll
                for (int e = 0; e < PIECES; ++e) {
                    const int here = __popcll(missing[e]);
                    if (piece < 0 && n < here) piece = 64 * wave + e * LC_RK_THREADS + lc_nth_bit(missing[e], n);
                    n -= here;
                }
                t = piece >> 1;
            }
            const bool help = looks > 0;
            if (help) load_half(next, t);
            LcTile tile;                                            // (its float32 rows come while the bfloat16 ones are multiplied)
            const float* const row = P + (size_t)min(16 * t + j, N - 1) * LC_D + 4 * kk;
#pragma unroll
            for (int s = 0; s < 8; ++s) tile.full[s] = *reinterpret_cast<const float4*>(row + 16 * s);
#pragma unroll
            for (int s = 0; s < 4; ++s) tile.half[s] = next[s];
            const int label = lc_rounds_label<NBLK>(sh, rows, tile, min(N - 16 * t, 16), k, [&](int c, int q) LC_INLINE { return centroid(it, c, q); },
                                                    [&]() LC_INLINE { load_half(next, min(own, tiles - 1)); });
            const int mine = 16 * t + j < N ? label : 0xfffe;       // (no label behind the last point)
            const int two = __shfl(mine, 2 * (lane & 7)) | (__shfl(mine, 2 * (lane & 7) + 1) << 16);
            if (lane < 8) __builtin_amdgcn_raw_buffer_store_b32(two, labels_r, label_at(it, 8 * t + lane), 0, 16);

            if (help) __builtin_amdgcn_s_waitcnt(0);
        }
        if (looks <= patience) patience = min(2 * patience, LC_RK_LOOKS);
        bool any = false;
#pragma unroll
        for (int e = 0; e < PIECES; ++e) {
            const int piece = tid + e * LC_RK_THREADS;
            if (piece >= pieces) continue;
            const lc_v4i old = lab[piece];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (v[e][q] != old[q]) {
                    any = true;
#pragma unroll
                    for (int s = 0; s < 32; s += 16) {
                        const int a = ((unsigned)v[e][q] >> s) & 0xffff, z = ((unsigned)old[q] >> s) & 0xffff;
                        if (a == z) continue;
                        const int at = 8 * piece + 2 * q + s / 16;
                        if (a < LC_AS_RES) {
                            fresh[a] = it + 1;
                            if (mine_of[a] >= 0) atomicOr(reinterpret_cast<unsigned*>(bits + mine_of[a] * blocks) + (at >> 5), 1u << (at & 31));
                        }
                        if (z < LC_AS_RES) {
                            fresh[z] = it + 1;
                            if (mine_of[z] >= 0) atomicAnd(reinterpret_cast<unsigned*>(bits + mine_of[z] * blocks) + (at >> 5), ~(1u << (at & 31)));
                        }
                    }
                }
            lab[piece] = v[e];
        }
        if (any) moved = it;
        lc_barrier_lds();
        // An iteration that moves no point is a fixed point: every later one would repeat it.
        if (__builtin_amdgcn_readfirstlane(moved) != it) break;
    }
    // ---- the labels of my points for good, and my nodes
    for (int t = first; t < tiles; t += step)
        if (lane < 16 && 16 * t + lane < N)
            ix.parent[l][(size_t)bh * ix.cap[l] + 16 * t + lane] = reinterpret_cast<const unsigned short*>(lab)[16 * t + lane];
    using Acc = typename std::conditional<NODES, double, float>::type;
    const LcMembers<NODES> m(ix, b, bh, l);
    for (int c = first, own = wave; c < k; c += step, own += LC_RK_WAVES) {
        Acc sum[8];
        int tok = 0, chunks = 0;
        lc_rounds_sum<Acc>(N, sh.list, [&](int b0) LC_INLINE { return members(keep_bits ? own : -1, c, b0); },
                           [&](int i, float (&x)[8]) LC_INLINE {
                               const int n = m.row(max(i, 0), 8 * sub, x);
#pragma unroll
                               for (int t = 0; t < 8; ++t) x[t] = i >= 0 ? x[t] : 0.f;
                               return i >= 0 ? n : 0;
                           },
                           [&](int i) LC_INLINE { tok += m.ntok[i]; chunks += m.chunks(i); }, sum);
        tok = lc_wave_sum_i(tok);
        chunks = lc_wave_sum_i(chunks);
        const int at = row_at(fresh[c], c) + 32 * sub;
        if (lane < 16)
            lc_write_node(ix, b, bh, l, c, chunks, tok, sum, w, [&](float (&mu)[8]) LC_INLINE {
                const float4 a = lc_load_agent4(rows_r, at), z = lc_load_agent4(rows_r, at + 16);
                mu[0] = a.x; mu[1] = a.y; mu[2] = a.z; mu[3] = a.w;
                mu[4] = z.x; mu[5] = z.y; mu[6] = z.z; mu[7] = z.w;
            });
    }
}

// Centers of a level of many small nodes (LC_UPD_FEW members or fewer on average): a workgroup lists the
// members of `per` nodes and gives each node to a 16-lane group.
template <bool NODES>
__global__ void __launch_bounds__(LC_BT)
lc_center_few_kernel(LcDev ix, int l, LcNodeArgs w, int per) {
    lc_fetch_args<sizeof(LcDev) + sizeof(LcNodeArgs)>();
    using Acc = typename std::conditional<NODES, double, float>::type;
    __shared__ LcBuckets bk;
    __shared__ __attribute__((aligned(16))) Acc sh[LC_BG * LC_D];
    const int h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    const int sub = threadIdx.x & 15;
    const int k = ix.nlev[b * LC_MAX_LEVELS + l + 1];
    const int u0 = blockIdx.x * per;
    if (u0 >= k) return;
    const LcMembers<NODES> m(ix, b, bh, l);
    lc_cluster_sums<Acc>(
        [&](int j) { return m.label[j]; }, m.n, u0, min(per, k - u0), bk, sh,
        [&](int j, float (&x)[8]) { return m.row(j, 8 * sub, x); },
        [&](int u, int n, Acc (&sum)[8]) {
            int tok = 0, chunks = 0;
            auto count = [&](int j) { tok += m.ntok[j]; chunks += m.chunks(j); };
            if (m.n > 0 && bk.total <= LC_UB_LIST) {                // the list is still there
                for (int t = bk.off[u - u0] + sub; t < bk.off[u - u0] + n; t += 16) count(bk.list[t]);
            } else {                                                // nodes listed one by one
                for (int j = sub; j < m.n; j += 16)
                    if (m.label[j] == u) count(j);
            }
            lc_write_node(ix, b, bh, l, u, lc_sum16_i(chunks), lc_sum16_i(tok), sum, w, [&](float (&mu)[8]) { lc_load8(w.centroid(bh, u) + 8 * sub, mu); });
        });
}

// Centers of a level of larger nodes: a workgroup per node, of 1024 threads where nodes hold more than
// LC_CENTER_WIDE members on average (there a single compute unit's rate of reading rows is the bound).
#define LC_CENTER_WIDE 128
template <int NT, bool NODES>
__global__ void __launch_bounds__(NT)
lc_center_kernel(LcDev ix, int l, LcNodeArgs w) {
    lc_fetch_args<sizeof(LcDev) + sizeof(LcNodeArgs)>();
    using Acc = typename std::conditional<NODES, double, float>::type;
    __shared__ __attribute__((aligned(16))) LcSumSh<NT, Acc> sh;
    __shared__ int tok_sh[NT / 64], chunk_sh[NT / 64];
    const int u = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    if (u >= ix.nlev[b * LC_MAX_LEVELS + l + 1]) return;
    const int tid = threadIdx.x;
    constexpr int COLS = 8 * 256 / NT;
    const LcMembers<NODES> m(ix, b, bh, l);
    int tok = 0, chunks = 0;
    Acc sum[8];
    lc_member_sum<NT, Acc>(
        [&](int j) { return m.label[j]; }, m.n, u, sh, [&](int j, int col, float (&x)[COLS]) { return m.row(j, col, x); },
        [&](const int* mem, int nm) {
            for (int t = tid; t < nm; t += NT) { tok += m.ntok[mem[t]]; chunks += m.chunks(mem[t]); }
        }, sum);
    tok = lc_wave_scan_incl(tok);
    chunks = lc_wave_scan_incl(chunks);
    if ((tid & 63) == 63) { tok_sh[tid >> 6] = tok; chunk_sh[tid >> 6] = chunks; }
    __syncthreads();
    if (tid < 16) {
        int n_tok = 0, n_chunks = 0;
        for (int v = 0; v < NT / 64; ++v) { n_tok += tok_sh[v]; n_chunks += chunk_sh[v]; }
        lc_write_node(ix, b, bh, l, u, n_chunks, n_tok, sum, w, [&](float (&mu)[8]) { lc_load8(w.centroid(bh, u) + 8 * tid, mu); });
    }
}

// Radii of all levels above the chunks, once every center stands: for each chunk and each of its
// ancestors the reach |center - ancestor's center| + chunk radius, maximum per node.  One pass over the
// chunk rows instead of one per level.  Levels of few nodes collect their maxima in LDS first -- all levels if together they have
// no more than LC_RD_LDS nodes, else those above level 1 --, so that a node is not one address that every chunk under it queues
// for: the atomics are the larger part of the time where they go to memory, two per chunk and level (radius and its copy for the drift).
// Radii are >= 0 (what is not a number is left out, as fmaxf would), so their bits order like integers, and a maximum does not
// depend on the order.
// PER chunks per 16-lane group: 4 while that gives each compute unit no more than one workgroup, 8 beyond (more rows in flight).  us with level 1 in
// memory and 4 per group; in LDS with 4; with 8: 820 chunks x 8 heads under 52 nodes 7.5, 5.8, 7.7; 2299 x 8 under 143 13.0, 11.6, 11.2; 64 pairs
// of up to 1820 under 57 18.4, 10.8, 11.0; 10.9 K x 8 under 5461 (level 1 in memory all the same) 29, 30, 23.3.
#define LC_RD_LDS 512             // nodes whose maxima are collected in LDS
template <int PER>
__global__ void __launch_bounds__(LC_BT)
lc_radius_kernel(LcDev ix) {
    constexpr int CHUNKS = PER * LC_BG;                             // of a workgroup
    lc_fetch_args<sizeof(LcDev)>();
    __shared__ int best[LC_RD_LDS];
    const int h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    const int tid = threadIdx.x, sub = tid & 15, grp = tid >> 4;
    const int M = ix.state[bh * 4 + 1];
    if ((int)blockIdx.x * CHUNKS >= M) return;
    const size_t cb = (size_t)bh * ix.cap[0];
    int n_up = 0, lowest = 1;                                       // nodes of level `lowest` and above, in level order
    for (int l = 1; l < ix.L; ++l) n_up += ix.nlev[b * LC_MAX_LEVELS + l];
    if (n_up > LC_RD_LDS) {
        n_up -= ix.nlev[b * LC_MAX_LEVELS + 1];
        lowest = 2;
    }
    const bool in_lds = n_up <= LC_RD_LDS;
    if (in_lds) {
        for (int i = tid; i < n_up; i += LC_BT) best[i] = -1;
        __syncthreads();
    }
    auto raise = [&](int l, int a, int bits) {
        atomicMax(reinterpret_cast<int*>(ix.radius[l]) + (size_t)bh * ix.cap[l] + a, bits);
        atomicMax(reinterpret_cast<int*>(ix.rbuild[l]) + (size_t)bh * ix.cap[l] + a, bits);
    };
    float c[PER][8], r0[PER];
    int anc[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int j = min((int)blockIdx.x * CHUNKS + e * LC_BG + grp, M - 1);
        anc[e] = ix.parent[0][cb + j];
        lc_c0_load8(ix, cb + j, sub, c[e]);
        r0[e] = ix.radius[0][cb + j];
    }
    int up = 0;
    for (int l = 1; l < ix.L; ++l) {
        float mu[PER][8];
        int next[PER];
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const size_t n = (size_t)bh * ix.cap[l] + max(anc[e], 0);
            lc_load8(ix.center[l] + n * LC_D + 8 * sub, mu[e]);
            next[e] = l + 1 < ix.L ? ix.parent[l][n] : -1;
        }
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            float d2 = 0.f;
#pragma unroll
            for (int t = 0; t < 8; ++t) { const float x = c[e][t] - mu[e][t]; d2 = fmaf(x, x, d2); }
            d2 = lc_sum16(d2);
            const float reach = lc_pad_radius(lc_pad_radius(sqrtf(d2)) + r0[e]);
            if (sub == 0 && anc[e] >= 0 && reach >= 0.f) {          // (not a number: reaches nothing)
                if (l >= lowest && in_lds) atomicMax(&best[up + anc[e]], __float_as_int(reach));
                else raise(l, anc[e], __float_as_int(reach));
            }
            anc[e] = anc[e] >= 0 ? next[e] : -1;
        }
        if (l >= lowest) up += ix.nlev[b * LC_MAX_LEVELS + l];
    }
    if (in_lds) {
        __syncthreads();
        int l = lowest, o = 0;
        for (int i = tid; i < n_up; i += LC_BT) {
            while (i - o >= ix.nlev[b * LC_MAX_LEVELS + l]) { o += ix.nlev[b * LC_MAX_LEVELS + l]; ++l; }
            if (best[i] >= 0) raise(l, i - o, best[i]);
        }
    }
}

namespace {

// most nodes that a sequence of the batch has at level l (host mirror)
int most_nodes(const lc_index* idx, int l) {
    int n = 0;
    for (int b = 0; b < idx->B; ++b) n = idx->N[b * LC_MAX_LEVELS + l] > n ? idx->N[b * LC_MAX_LEVELS + l] : n;
    return n;
}
bool small_level(int n, int k) { return n <= LC_KS_MAX_N && k <= LC_KS_MAX_K; }

// Workgroups of lc_kmeans_rounds_kernel for a (sequence, head) if all get as many: they run at the same time, one to a compute unit.  Beyond 64 they
// gain nothing (2 heads x 8000 points under 250 nodes, whole builds, us by workgroups a head: 16 360, 32 259, 64 224, 128 216; x 2000 under 250:
// 67.5, 64.6, 64.1, 64.4).
int rounds_share(long long BH) { return (int)(BH * 64 <= LC_COMPUTE_UNITS ? 64 : LC_COMPUTE_UNITS / BH); }

// The parts of lc_kmeans_rounds_kernel: returns the workgroups to launch.  A (sequence, head) gets parts in proportion to its points, as the
// kernel lasts as long as the one with the most points to a part.  Workgroups are dealt to the XCDs in turn, so the parts of a
// (sequence, head) are 8 apart where they are to share one; they are, unless that means over an eighth more points to a part.
// Prefill of 16 sequences of 16K to 64K tokens x 4 heads (455 to 1820 points): 349.6 us with equal parts, 338.7 in proportion; of one
// sequence x 8 heads the same.
int lay_out_shares(const lc_index* idx, int l, LcShares* s) {
    constexpr int XCDS = 8, EACH = LC_COMPUTE_UNITS / XCDS;
    const int H = idx->H_kv, BH = idx->B * H;
    int n[LC_RK_MAX_PAIRS], order[LC_RK_MAX_PAIRS], near[LC_RK_MAX_PAIRS], far[LC_RK_MAX_PAIRS], xcd[LC_RK_MAX_PAIRS];
    for (int p = 0; p < BH; ++p) {
        n[p] = idx->N[p / H * LC_MAX_LEVELS + l] + 1;
        order[p] = p;
    }
    std::stable_sort(order, order + BH, [&](int x, int y) { return n[x] > n[y]; });
    // as few points to a part of the pairs of one XCD (or of all: x < 0) as give no more than `slots` parts
    auto deal = [&](int (&parts)[LC_RK_MAX_PAIRS], int x, int slots) {
        int lo = 1, hi = n[order[0]];                               // (hi: a part each)
        auto count = [&](int points) {
            int sum = 0;
            for (int p = 0; p < BH; ++p)
                if (x < 0 || xcd[p] == x) sum += parts[p] = std::min((n[p] + points - 1) / points, LC_RK_MAX_SHARE);
            return sum;
        };
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (count(mid) <= slots) hi = mid;
            else lo = mid + 1;
        }
        count(hi);
    };
    auto worst = [&](const int (&parts)[LC_RK_MAX_PAIRS]) {
        int w = 0;
        for (int p = 0; p < BH; ++p) w = std::max(w, (n[p] + parts[p] - 1) / parts[p]);
        return w;
    };
    deal(far, -1, LC_COMPUTE_UNITS);
    bool share_xcd = BH >= XCDS;
    if (share_xcd) {
        long long load[XCDS] = {};
        int pairs[XCDS] = {};
        for (int i = 0; i < BH; ++i) {
            int to = -1;
            for (int x = 0; x < XCDS; ++x)
                if (pairs[x] < EACH && (to < 0 || load[x] < load[to])) to = x;
            xcd[order[i]] = to;
            load[to] += n[order[i]];
            ++pairs[to];
        }
        for (int x = 0; x < XCDS; ++x) deal(near, x, EACH);
        share_xcd = worst(near) * 8 <= worst(far) * 9;
    }
    for (int i = 0; i < LC_COMPUTE_UNITS; ++i) s->of[i] = LC_RK_NO_PART;
    int next[XCDS] = {}, at = 0, groups = 0;
    for (int z = 0; z < LC_RK_MAX_SHARE; ++z)
        for (int i = 0; i < BH; ++i) {
            const int p = order[i], parts = share_xcd ? near[p] : far[p];
            if (z >= parts) continue;
            const int slot = share_xcd ? xcd[p] + XCDS * next[xcd[p]]++ : at++;
            s->of[slot] = (uint32_t)p | (uint32_t)z << 8 | (uint32_t)parts << 16;
            groups = std::max(groups, slot + 1);
        }
    return groups;
}

// Whether a level of n points and k clusters is clustered by lc_kmeans_rounds_kernel, and what that posts, in the workspace's place for it.
// Measured as whole builds of two levels with random keys, 1 to 128 pairs, 300 to 8192 points, 2 to 4000 members a cluster (2200 shapes), the time with
// it in parts of that with two kernels an iteration, which have no members' bits for over 4096 points: up to 4096 points 0.43 to 1.04, median 0.87;
// beyond 0.56 to 1.01, median 0.82.  Not so, and left to the two kernels:
// - a cluster is one wavefront's work, 16 groups' or a whole workgroup's with the two.  Fewer than 24 pairs with more than 64 members a cluster 0.95 to
//   1.06 (at 64 0.87 to 1.02); 24 and more with more than 128 members 0.90 to 1.49 (at 128 0.90 to 1.00); over 4096 points, more than
//   256 members 0.89 to 1.94 (at 256 0.86 to 1.01);
// - up to 4 pairs of 3400 to 4096 points, where the two kernels have workgroups enough as well: 0.93 to 1.10;
// - pairs that leave a fifth of the compute units without a workgroup and have more than 256 points to each: 96 of 1000 to 4000 points 0.92 to
//   1.18 (of 500 0.75 to 1.02); that leave an eighth, of over 2048 points in more than 160: 72 and 104 pairs 0.91 to 1.06;
// - more than 100 clusters to a workgroup: 128 pairs of 1000 points in 250 1.04.
bool lay_out_rounds(const LcWs& ws, long long BH, int n, int k, int iters, LcRounds* r) {
    if (iters < 1 || iters > LC_RK_MAX_ITERS || n > LC_RK_MAX_N || BH > LC_RK_MAX_PAIRS) return false;
    const int share = rounds_share(BH), groups = (int)BH * share;
    if (n > (n > 4096 ? 256 : BH < 24 ? 64 : 128) * k) return false;
    if (n <= 4096 && ((BH <= 4 && n > 3400) || k > 100 * share ||
                      (BH > 4 && groups * 5 < LC_COMPUTE_UNITS * 4 && n > 256 * share) ||
                      (BH > 4 && groups * 8 < LC_COMPUTE_UNITS * 7 && n > 2048 && k > 160))) return false;
    r->k = k;
    r->words = (n + 15) / 16 * 8;
    const long long plane = BH * k * LC_D * 4, row_bytes = (iters + 1) * plane, label_bytes = iters * BH * r->words * 4;
    if (row_bytes + label_bytes > (long long)ws.rounds_bytes || row_bytes >= (1ll << 31) - 16) return false;
    r->rows = ws.rounds;
    r->labels = reinterpret_cast<int*>(reinterpret_cast<char*>(ws.rounds) + row_bytes);
    r->row_bytes = (int)row_bytes;
    r->label_bytes = (int)label_bytes;
    r->unposted.at = reinterpret_cast<lc_v4i*>(reinterpret_cast<char*>(ws.rounds) + plane);
    r->unposted.n = (int)((row_bytes + label_bytes - plane) / 16);
    return true;
}

}  // namespace

// K == nullptr: keep the chunk nodes (level 0) as they are and rebuild only the levels above them.
int lc_launch_build(const lc_index* idx, const LcWs& ws, const void* Kp, const int64_t ks[3],
                    int max_M, hipStream_t stream) {
    const LcDev& ix = idx->dev;
    const uint16_t* K = static_cast<const uint16_t*>(Kp);
    const int geometry = idx->cfg.geometry;
    const int B = ix.B, H = ix.H, L = ix.L;
    const long long BH = (long long)B * H;
    const int iters = idx->cfg.kmeans_iters;
    int* const kflags = iters < LC_KM_FLAGS ? ws.kflags : nullptr;   // (more iterations: no early exit)
    // points and centroids of the level being clustered, and of the next one (whose rows are written while
    // this one's centroids are still read)
    LcPointRows cur{ws.dirs, ws.dirs16, ix.cap[0], L > 1 ? ws.cent[0] : nullptr, ws.cent16[0], ix.cap[1]};
    // The level that lc_kmeans_rounds_kernel clusters, if there is one: the first that is neither small nor of too many clusters or points.
    int rounds_level = -1;
    LcRounds rounds{nullptr, nullptr, 0, 0, 0, 0, {nullptr, 0}};
    for (int l = 0; l + 1 < L && rounds_level < 0; ++l) {
        const int n = most_nodes(idx, l), k = most_nodes(idx, l + 1);
        if (n > 0 && k <= LC_AS_RES && !small_level(n, k)) {
            if (lay_out_rounds(ws, BH, n, k, iters, &rounds)) rounds_level = l;
            break;
        }
    }
    if (rounds_level == 0) { cur.cent = rounds.rows; cur.cent_cap = rounds.k; }
    if (max_M > 0 && K != nullptr) {
        const bool near = ks[2] >= LC_D && ks[2] * 2 * (4 * LC_POOLW_KEEP) < (1ll << 31);     // (see lc_pool_batch)
        hipLaunchKernelGGL(near ? lc_pool_kernel<true> : lc_pool_kernel<false>, dim3(max_M, H, B), dim3(64), 0, stream, ix, K,
                           (long long)ks[0], (long long)ks[1], (long long)ks[2], geometry, cur, ws.kflags, rounds.unposted);
        LC_HIP_CHECK(hipGetLastError());
    } else if (max_M > 0) {
        hipLaunchKernelGGL(lc_dirs_kernel, dim3((max_M + LC_BG - 1) / LC_BG, H, B), dim3(LC_BT), 0, stream, ix, cur, ws.kflags, rounds.unposted);
        LC_HIP_CHECK(hipGetLastError());
    }
    for (int l = 0; l + 1 < L; ++l) {
        LcPointRows next{nullptr, nullptr, 0, nullptr, nullptr, 0};
        if (l + 2 < L) {
            const bool even = (l & 1) == 0;                          // level 0's points give way to level 2's
            next = LcPointRows{even ? ws.next_pts : ws.dirs, even ? ws.next_pts16 : ws.dirs16, even ? ix.cap[1] : ix.cap[0],
                               ws.cent[even ? 1 : 0], ws.cent16[even ? 1 : 0], ix.cap[1]};
            if (rounds_level == l + 1) { next.cent = rounds.rows; next.cent_cap = rounds.k; }
        }
        const int maxN = most_nodes(idx, l), maxK = most_nodes(idx, l + 1);
        // Several clusters per workgroup where they are small, or where one each would be thousands of workgroups that all read every
        // label.  Clusterings with one and with several, us by members a cluster (clusters in all): 8 heads x 3000 points 206 and 201 at 9 (2672),
        // 252 and 260 at 11 (2184); x 6000 483 and 419 at 15 (3200), 478 and 480 at 17 (2824), 504 and 519 at 19 (2528); x 10.9K 1022 and 766 at 19 (4592), 916
        // and 761 at 28 (3120), 793 and 852 at 33 (2648); 16 pairs x 5000 627 and 593 at 19 (4224), 500 and 560 at 28 (2864); 32 x 4000 466 and 453 at 19 (6752);
        // 2 heads x 40K 2405 and 1246 at 21 (3810); one x 60K 2281 and 1369 at 28 (2143).  So where every cluster reads few labels (below 8192 points) it
        // takes more clusters; with many points the line could be at more members than it is.
        const bool few = maxN <= (long long)maxK * LC_UPD_FEW || (maxN <= (long long)maxK * LC_UPD_FEW_MANY && maxK * BH > (maxN < 8192 ? 2600 : 2048));
        // clusters per workgroup of the kernels that list several: one per 16-lane group, more of them where
        // that would be over a thousand workgroups that each read all the labels
        const int per = (maxK + LC_BG - 1) / LC_BG * BH > 1024 ? LC_UB_MAX : LC_BG;
        const dim3 per_grid((maxK + per - 1) / per, H, B);
        const LcNodeArgs w{cur.cent, cur.cent_cap, geometry, next};
        if (l == rounds_level) {                                       // a clustering in one kernel of several workgroups
            LcShares shares;
            const int groups = lay_out_shares(idx, l, &shares);
            auto launch = [&](auto kernel, const LcShares& of) {
                hipLaunchKernelGGL(kernel, dim3(groups), dim3(LC_RK_THREADS), 0, stream, ix, l, (const float*)cur.pts,
                                   (const uint16_t*)cur.pts16, cur.cap, w, iters, rounds, of);
            };
            auto run = [&](auto kernel) {
                if (ws.first_parts <= 0) return launch(kernel, shares);
                LcShares first = shares, rest = shares;
                for (int i = 0; i < LC_COMPUTE_UNITS; ++i)
                    ((int)(shares.of[i] >> 8 & 0xff) < ws.first_parts ? rest : first).of[i] = LC_RK_NO_PART;
                launch(kernel, first);
                launch(kernel, rest);
            };
            // Absent centroids of an instance's blocks are multiplied too, which is what a point's wavefront takes longest for.  Re-clustering with
            // two kernels an iteration, blocks for 160 clusters, and these, us: 2400 points in 67 136, 156 and 127; 2 heads of 2800 in 70
            // 140, 170 and 137; 4 of 3200 in 67 150, 176 and 143; 8 of 3200 in 80 167, 181 and 148.
            auto run_blocks = [&](auto blocks) {
                if (l == 0) run(&lc_kmeans_rounds_kernel<decltype(blocks)::value, false>);
                else run(&lc_kmeans_rounds_kernel<decltype(blocks)::value, true>);
            };
            if (maxK <= 64) run_blocks(std::integral_constant<int, 4>());
            else if (maxK <= 96) run_blocks(std::integral_constant<int, 6>());
            else if (maxK <= 128) run_blocks(std::integral_constant<int, 8>());
            else if (maxK <= 160) run_blocks(std::integral_constant<int, 10>());
            else if (maxK <= 208) run_blocks(std::integral_constant<int, 13>());
            else run_blocks(std::integral_constant<int, 16>());
            LC_HIP_CHECK(hipGetLastError());
            cur = next;
            continue;
        }
        if (maxN > 0 && small_level(maxN, maxK)) {                     // the whole level in one workgroup per (sequence, head)
            const size_t lds = lc_kmeans_small_lds(maxN, maxK);
            const auto kernel = maxK <= LC_KS_THREADS / 64 ? (l == 0 ? &lc_kmeans_small_kernel<false, true> : &lc_kmeans_small_kernel<true, true>)
                                                           : (l == 0 ? &lc_kmeans_small_kernel<false, false> : &lc_kmeans_small_kernel<true, false>);
            LC_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
            hipLaunchKernelGGL(kernel, dim3(H, B), dim3(LC_KS_THREADS), lds, stream, ix, l, (const float*)cur.pts, cur.cap, w, iters, maxN);
            LC_HIP_CHECK(hipGetLastError());
            cur = next;
            continue;
        }
        if (maxN > 0) {
            // Many centroids: 64 MA points per workgroup.  The fuller a wavefront's A operand, the fewer LDS reads per
            // product (LDS bandwidth for two blocks of products with MA = 1); MA is the one with the least work on the
            // busiest compute unit, the larger one if equal.
            int ma = 1;
            long long least = 0;
            for (int m = 1; m <= 4; ++m) {
                const long long load = ((maxN + 64 * m - 1) / (64 * m) * BH + 255) / 256 * (m > 2 ? m : 2);
                if (m == 1 || load <= least) { least = load; ma = m; }
            }
            // Few centroids: as many blocks as hold them (work for absent centroids costs: 40000 points x 4 heads, us by blocks,
            // 64 points per workgroup: 2: 20.6, 4: 22.3, 6: 26, 8: 31, 10: 33, 12: 43, 16: 48; 2275 x 8: 8.0, 9.0, 9.6, 9.7, 10.3, 11.1,
            // 12.6), and 64 points per workgroup.  128 points stage half as many rows, at the price of registers: with more
            // than two workgroups per compute unit that pays at 12 blocks (33 instead of 43 us; 4200 x 16: 20.9 instead of 24),
            // hardly at 8 and 10 (29.6 instead of 31.2, 31.3 instead of 33.5; 4200 x 16: 18.4 instead of 17.4) and not at 2, 4
            // or 6 (24.1, 25.9, 27.5 us).  At 16 blocks it does since two of them fit a compute unit: 5461 x 8 points under 249 centroids
            // 14.8 instead of 17.4 us, whole clusterings of 10.9 K x 8 points 722 instead of 760, of 4166 x 64 under 208 1081 instead of 1219.
            const bool wide = (maxN + 63) / 64 * BH > 512;
            auto assign = [&](auto kernel, int points, int threads, int it, auto... more) {
                hipLaunchKernelGGL(kernel, dim3((maxN + points - 1) / points, H, B), dim3(threads), 0, stream, ix, l,
                                   (const float*)cur.pts, (const uint16_t*)cur.pts16, cur.cap, (const float*)cur.cent,
                                   (const uint16_t*)cur.cent16, cur.cent_cap, it, kflags, more...);
            };
            // Members' bits, for clusters that are updated one by one from up to LC_AS_RES centroids: they take the place of the next
            // level's points and centroids, which nothing has written yet, where both hold them (up to 4096 points always).
            LcMemberBits bits{{nullptr, nullptr}, {0, 0}, maxK};
            {
                const bool even = (l & 1) == 0;
                const long long need = ((long long)maxN + 63) / 64 * maxK * 8;
                const long long room[2] = {(long long)(even ? ix.cap[1] : ix.cap[0]) * LC_D * 4, (long long)ix.cap[1] * LC_D * 4};
                if (maxK <= LC_AS_RES && maxN > (long long)maxK * LC_UPD_FEW && need <= room[0] && need <= room[1])
                    for (int i = 0; i < 2; ++i) {
                        bits.w[i] = reinterpret_cast<unsigned long long*>(i == 1 ? ws.cent[even ? 1 : 0] : (even ? ws.next_pts : ws.dirs));
                        bits.stride[i] = room[i] / 8;
                    }
            }
            for (int it = 0; it < iters; ++it) {
                if (maxK <= 32) assign(&lc_kmeans_assign_res_kernel<2, 4>, 64, 256, it, bits);
                else if (maxK <= 64) assign(&lc_kmeans_assign_res_kernel<4, 4>, 64, 256, it, bits);
                else if (maxK <= 96) assign(&lc_kmeans_assign_res_kernel<6, 4>, 64, 256, it, bits);
                else if (maxK <= 128 && wide) assign(&lc_kmeans_assign_res_kernel<8, 8>, 128, 512, it, bits);
                else if (maxK <= 128) assign(&lc_kmeans_assign_res_kernel<8, 4>, 64, 256, it, bits);
                else if (maxK <= 160 && wide) assign(&lc_kmeans_assign_res_kernel<10, 8>, 128, 512, it, bits);
                else if (maxK <= 160) assign(&lc_kmeans_assign_res_kernel<10, 4>, 64, 256, it, bits);
                else if (maxK <= 192 && wide) assign(&lc_kmeans_assign_res_kernel<12, 8>, 128, 512, it, bits);
                else if (maxK <= 192) assign(&lc_kmeans_assign_res_kernel<12, 4>, 64, 256, it, bits);
                else if (maxK <= LC_AS_RES && wide) assign(&lc_kmeans_assign_res_kernel<16, 8>, 128, 512, it, bits);
                else if (maxK <= LC_AS_RES) assign(&lc_kmeans_assign_res_kernel<16, 4>, 64, 256, it, bits);
                else if (ma == 4) assign(&lc_kmeans_assign_kernel<4>, 256, LC_BT, it);
                else if (ma == 3) assign(&lc_kmeans_assign_kernel<3>, 192, LC_BT, it);
                else if (ma == 2) assign(&lc_kmeans_assign_kernel<2>, 128, LC_BT, it);
                else assign(&lc_kmeans_assign_kernel<1>, 64, LC_BT, it);
                if (few && bits.w[0] == nullptr)
                    hipLaunchKernelGGL(lc_kmeans_update_few_kernel, per_grid, dim3(LC_BT), 0, stream, ix, l,
                                       (const float*)cur.pts, cur.cap, cur.cent, cur.cent16, cur.cent_cap, it, per, kflags);
                else if (bits.w[0])
                    hipLaunchKernelGGL(lc_kmeans_update_bits_kernel, dim3(maxK, H, B), dim3(LC_BT), 0, stream, ix, l,
                                       (const float*)cur.pts, cur.cap, cur.cent, cur.cent16, cur.cent_cap, it, kflags, bits);
                else
                    hipLaunchKernelGGL(lc_kmeans_update_kernel, dim3(maxK, H, B), dim3(LC_BT), 0, stream, ix, l,
                                       (const float*)cur.pts, cur.cap, cur.cent, cur.cent16, cur.cent_cap, it, kflags);
            }
            LC_HIP_CHECK(hipGetLastError());
        }
        auto center = [&](auto nodes) {
            constexpr bool NODES = decltype(nodes)::value;
            if (few)
                hipLaunchKernelGGL(lc_center_few_kernel<NODES>, per_grid, dim3(LC_BT), 0, stream, ix, l, w, per);
            else if (maxN <= (long long)maxK * LC_CENTER_WIDE)
                hipLaunchKernelGGL((lc_center_kernel<256, NODES>), dim3(maxK, H, B), dim3(256), 0, stream, ix, l, w);
            else
                hipLaunchKernelGGL((lc_center_kernel<1024, NODES>), dim3(maxK, H, B), dim3(1024), 0, stream, ix, l, w);
        };
        if (l == 0) center(std::false_type());
        else center(std::true_type());
        LC_HIP_CHECK(hipGetLastError());
        cur = next;
    }
    if (L > 1 && max_M > 0) {
        const int per = (max_M + 4 * LC_BG - 1) / (4 * LC_BG) * BH <= LC_COMPUTE_UNITS ? 4 : 8;
        hipLaunchKernelGGL(per == 4 ? lc_radius_kernel<4> : lc_radius_kernel<8>, dim3((max_M + per * LC_BG - 1) / (per * LC_BG), H, B),
                           dim3(LC_BT), 0, stream, ix);
        LC_HIP_CHECK(hipGetLastError());
    }
    return LC_OK;
}

// ---------------------------------------------------------------------------------
// drift of one level's radii since the last (re)build
// ---------------------------------------------------------------------------------
// One workgroup per (sequence, head): over the nodes with a finite radius at build time, the sum of
// those radii, the sum of the radii now, the largest growth and the count (fixed reduction order).
// What bounds it is round trips, a head's nodes being one workgroup's: LC_DR_NODES of a thread are on their way at once (8 heads of 5461 nodes, one
// at a time 14.5 us, now 4.4).
#define LC_DR_NODES 16
__global__ void __launch_bounds__(LC_BT)
lc_drift_kernel(LcDev ix, int level, float* out) {
    __shared__ float sh[4][LC_BT / 64];
    const int h = blockIdx.x, b = blockIdx.y;
    const int bh = b * ix.H + h;
    const int n_l = min(ix.nlev[b * LC_MAX_LEVELS + level], ix.cap[level]);
    const size_t base = (size_t)bh * ix.cap[level];
    float s_then = 0.f, s_now = 0.f, grow = 0.f, cnt = 0.f;
    for (int n0 = threadIdx.x; n0 < n_l; n0 += LC_DR_NODES * LC_BT) {
        float r0[LC_DR_NODES], r1[LC_DR_NODES];
#pragma unroll
        for (int e = 0; e < LC_DR_NODES; ++e) {
            const size_t n = base + min(n0 + e * LC_BT, n_l - 1);
            r0[e] = ix.rbuild[level][n];
            r1[e] = ix.radius[level][n];
        }
#pragma unroll
        for (int e = 0; e < LC_DR_NODES; ++e)
            if (n0 + e * LC_BT < n_l && r0[e] > LC_NEG_INF) {
                s_then += r0[e];
                s_now += r1[e];
                grow = fmaxf(grow, r1[e] - r0[e]);
                cnt += 1.f;
            }
    }
    s_then = lc_sum64(s_then);
    s_now = lc_sum64(s_now);
    grow = lc_max64(grow);
    cnt = lc_sum64(cnt);
    if ((threadIdx.x & 63) == 0) {
        const int w = threadIdx.x >> 6;
        sh[0][w] = s_then; sh[1][w] = s_now; sh[2][w] = grow; sh[3][w] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float a = 0.f, c = 0.f, g = 0.f, k = 0.f;
        for (int w = 0; w < LC_BT / 64; ++w) { a += sh[0][w]; c += sh[1][w]; g = fmaxf(g, sh[2][w]); k += sh[3][w]; }
        out[bh * 4 + 0] = a; out[bh * 4 + 1] = c; out[bh * 4 + 2] = g; out[bh * 4 + 3] = k;
    }
}

// staged (pinned host memory) = [state: B*H*4 | nlev: B*LC_MAX_LEVELS | where each sequence's boundaries begin: B |
// boundaries: M_0 + 1, M_1 + 1, ...]; row b < B of the grid moves sequence b's boundaries and clears its posted keys, row B moves the counts (and
// clears the arrival counters).  What bounds it is the way over the bus: two round trips, four words per thread in flight.  The keys are
// cleared meanwhile, eight a thread: by a grid sized from the boundaries alone, over as many keys as the index has chunks of capacity, a build of 8 heads of 100 chunks took 97 us
// instead of 31 with 131072 chunks of capacity, and 16 sequences of them 49 instead of 46 with 4100.
#define LC_PS_WORDS (4 * LC_BT)
#define LC_PS_KEYS (8 * LC_BT)
__global__ void __launch_bounds__(LC_BT)
lc_place_state_kernel(LcDev ix, const int32_t* staged, int B) {
    const int b = blockIdx.y, tid = threadIdx.x;
    const int n_state = B * ix.H * 4, n_nlev = B * LC_MAX_LEVELS;
    if (b == B) {
        for (int i0 = blockIdx.x * LC_PS_WORDS; i0 < n_state + n_nlev; i0 += gridDim.x * LC_PS_WORDS) {
            int v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = staged[min(i0 + k * LC_BT + tid, n_state + n_nlev - 1)];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = i0 + k * LC_BT + tid;
                if (i < n_state) { ix.state[i] = v[k]; ix.sync[i] = (i & 3) == 3 ? 1 : 0; }
                else if (i < n_state + n_nlev) ix.nlev[i - n_state] = v[k];
            }
        }
        return;
    }
    const int off = staged[n_state + n_nlev + b], n = staged[b * ix.H * 4 + 1] + 1;
    const int n_keys = ix.H * lc_posted_slots(ix.cap[0]);
    unsigned long long* const keys = ix.posted + (size_t)b * n_keys;
    for (int i = blockIdx.x * LC_BT + tid; i < n_keys; i += gridDim.x * LC_BT) keys[i] = 0ull;
    int* dst = ix.bounds + (size_t)b * (ix.cap[0] + 1);
    const int i0 = blockIdx.x * LC_PS_WORDS;
    if (i0 >= n) return;
    int v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = staged[off + min(i0 + k * LC_BT + tid, n - 1)];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = i0 + k * LC_BT + tid;
        if (i < n) dst[i] = v[k];
    }
}
__global__ void __launch_bounds__(LC_BT)
lc_place_counts_kernel(int* dst, const int32_t* staged, int n) {
    for (int i = blockIdx.x * LC_BT + threadIdx.x; i < n; i += gridDim.x * LC_BT) dst[i] = staged[i];
}

int lc_launch_place_state(const lc_index* idx, const int32_t* staged, int max_M, hipStream_t stream) {
    const int for_bounds = max_M / LC_PS_WORDS + 1, for_keys = (idx->H_kv * lc_posted_slots(idx->cfg.max_chunks) + LC_PS_KEYS - 1) / LC_PS_KEYS;
    hipLaunchKernelGGL(lc_place_state_kernel, dim3(for_bounds > for_keys ? for_bounds : for_keys, idx->B + 1), dim3(LC_BT), 0, stream, idx->dev, staged, idx->B);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}
int lc_launch_place_counts(const lc_index* idx, const int32_t* staged, hipStream_t stream) {
    hipLaunchKernelGGL(lc_place_counts_kernel, dim3(1), dim3(LC_BT), 0, stream, idx->dev.nlev, staged, idx->B * LC_MAX_LEVELS);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}

int lc_launch_drift(const lc_index* idx, int level, float* out, hipStream_t stream) {
    hipLaunchKernelGGL(lc_drift_kernel, dim3(idx->dev.H, idx->dev.B), dim3(LC_BT), 0, stream, idx->dev, level, out);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}

// ---------------------------------------------------------------------------------
// lazy update
// ---------------------------------------------------------------------------------
struct LcCloseBits { uint32_t w[32]; };       // one bit per sequence (B <= 1024)

__global__ void __launch_bounds__(LC_BT)
lc_append_kernel(LcDev ix, uint16_t* K, uint16_t* V, long long ks_seq, long long ks_head, long long ks_tok,
                 const uint16_t* k_new, const uint16_t* v_new, LcCloseBits close, int geometry, int max_tokens) {
    lc_fetch_args<sizeof(LcDev) + 64 + sizeof(LcCloseBits)>();
    __shared__ float sh[LC_BG * LC_D + LC_BG];
    __shared__ float best_sim[LC_BG];
    __shared__ int best_arg[LC_BG];
    const int h = blockIdx.x, b = blockIdx.y;
    const int bh = b * ix.H + h;
    const int tid = threadIdx.x, sub = tid & 15, grp = tid >> 4;
    // The new rows do not depend on the counts: they are on their way before the counts arrive.  (What bounds a token
    // that closes no chunk is two round trips to memory, these loads and the stores; with the loads behind the
    // counts it was three.)
    uint4 row = make_uint4(0u, 0u, 0u, 0u);
    if (tid < 32)
        row = *reinterpret_cast<const uint4*>((tid < 16 ? k_new : v_new) + (size_t)bh * LC_D + 8 * sub);
    const int T = ix.state[bh * 4 + 0];
    const int M = ix.state[bh * 4 + 1];
    // The host checks the capacities against its own counts before it launches; these guards are for
    // a caller who replays the launch from a captured graph, where the host is not asked again.
    if (T >= max_tokens) return;
    uint16_t* Kbh = K + b * ks_seq + h * ks_head;
    uint16_t* Vbh = V + b * ks_seq + h * ks_head;
    if (tid < 32)
        *reinterpret_cast<uint4*>((tid < 16 ? Kbh : Vbh) + (long long)T * ks_tok + 8 * sub) = row;
    const bool do_close = ((close.w[b >> 5] >> (b & 31)) & 1u) && M < ix.cap[0];
    if (!do_close) {
        if (tid == 0) ix.state[bh * 4 + 0] = T + 1;
        return;
    }
    __threadfence_block();
    __syncthreads();

    int* bnd = ix.bounds + (size_t)b * (ix.cap[0] + 1);
    const int lo = bnd[M], hi = T + 1;
    float mu_x[8], r_x;
    lc_pool_rows(Kbh, ks_tok, lo, hi, geometry, ix.c0_bf16 != 0, sh, mu_x, &r_x);
    const int n_x = hi - lo;
    int p = -1;
    if (ix.L > 1) {
        float xh[8];
        lc_unit_frag(mu_x, sub, xh);
        const float xh0 = __shfl(xh[0], (tid & 48), 64);        // first component, from the group's lane 0
        const int n1 = ix.nlev[b * LC_MAX_LEVELS + 1];
        const size_t b1 = (size_t)bh * ix.cap[1];
        float bs = LC_NEG_INF;
        int ba = 0x7fffffff;
        for (int c = grp; c < n1; c += LC_BG) {
            float m[8];
            lc_load8(ix.center[1] + (b1 + c) * LC_D + 8 * sub, m);
            float dot = 0.f, n2 = 0.f;
#pragma unroll
            for (int t = 0; t < 8; ++t) { dot = fmaf(xh[t], m[t], dot); n2 = fmaf(m[t], m[t], n2); }
            dot = lc_sum16(dot);
            n2 = lc_sum16(n2);
            const float sim = n2 > 0.f ? dot / sqrtf(n2) : xh0;
            if (sim > bs) { bs = sim; ba = c; }
        }
        if (sub == 0) { best_sim[grp] = bs; best_arg[grp] = ba; }
        __syncthreads();
        float s = LC_NEG_INF;
        p = 0x7fffffff;
        for (int g = 0; g < LC_BG; ++g) {
            const float sg = best_sim[g];
            const int ag = best_arg[g];
            if (sg > s || (sg == s && ag < p)) { s = sg; p = ag; }
        }
        if (p >= n1) p = 0;                                 // (no similarity that compares: an infinite key)
        // path to the top: moving-average centers, monotone radii
        if (tid < 16) {
            int a = p;
            for (int l = 1; l < ix.L; ++l) {
                const size_t n = (size_t)bh * ix.cap[l] + a;
                const int n_a = ix.nchunk[l][n];
                float mu_a[8], nw[8];
                lc_load8(ix.center[l] + n * LC_D + 8 * sub, mu_a);
                const float inv = 1.0f / (float)(n_a + 1);
#pragma unroll
                for (int t = 0; t < 8; ++t) nw[t] = fmaf((float)n_a, mu_a[t], mu_x[t]) * inv;
                if (geometry == LC_GEOMETRY_PAPER_UNIT) {
                    float un[8];
                    lc_unit_frag(nw, sub, un);
#pragma unroll
                    for (int t = 0; t < 8; ++t) nw[t] = un[t];
                }
                float sh2 = 0.f, re2 = 0.f;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const float e = nw[t] - mu_a[t];
                    const float f = mu_x[t] - nw[t];
                    sh2 = fmaf(e, e, sh2);
                    re2 = fmaf(f, f, re2);
                }
                sh2 = lc_sum16(sh2);
                re2 = lc_sum16(re2);
                const float R_old = ix.radius[l][n];
                const float grown = R_old + lc_pad_radius(sqrtf(sh2));
                const float reach = lc_pad_radius(sqrtf(re2)) + r_x;
                const int next = ix.parent[l][n];
                lc_store8(ix.center[l] + n * LC_D + 8 * sub, nw);
                if (sub == 0) {
                    ix.radius[l][n] = lc_pad_radius(fmaxf(grown, reach));
                    ix.ntok[l][n] += n_x;
                    ix.nchunk[l][n] = n_a + 1;
                }
                a = next;
            }
        }
    }
    const size_t n0 = (size_t)bh * ix.cap[0] + M;
    if (tid < 16) {
        lc_c0_store8(ix, n0, sub, mu_x);
        if (sub == 0) {
            ix.radius[0][n0] = r_x;
            ix.parent[0][n0] = p;
            ix.ntok[0][n0] = n_x;
            ix.nchunk[0][n0] = 1;
            if (h == 0) bnd[M + 1] = hi;
            ix.state[bh * 4 + 0] = T + 1;
            ix.state[bh * 4 + 1] = M + 1;
        }
    }
}

int lc_launch_append(const lc_index* idx, void* K, void* V, const int64_t ks[3],
                     const void* k_new, const void* v_new, const uint8_t* close_host,
                     uint32_t, hipStream_t stream) {
    const LcDev& ix = idx->dev;
    LcCloseBits bits;
    for (int i = 0; i < 32; ++i) bits.w[i] = 0u;
    if (close_host)
        for (int b = 0; b < ix.B; ++b)
            if (close_host[b]) bits.w[b >> 5] |= 1u << (b & 31);
    hipLaunchKernelGGL(lc_append_kernel, dim3(ix.H, ix.B), dim3(LC_BT), 0, stream, ix,
                       static_cast<uint16_t*>(K), static_cast<uint16_t*>(V),
                       (long long)ks[0], (long long)ks[1], (long long)ks[2],
                       static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new), bits,
                       idx->cfg.geometry, idx->cfg.max_tokens);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}
