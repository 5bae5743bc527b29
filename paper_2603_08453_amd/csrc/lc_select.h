// Budget selection of one (sequence, head) from the chunk entries the scoring kernel left, by one workgroup.
// Used by every workgroup of the select+attend kernel of a decode step.  (lc_select_kernel does the same for the two separate calls.)
#pragma once

#include "lc_device.h"
#include "lc_internal.h"

#define LC_SEL_CAND 16            // chunks of the cutoff bin per wavefront that are ranked directly
#define LC_SEL_FEW 8              // of them in one step, a lane per pair
#define LC_SEL_BINS_MAX 1024      // most bins of the selection histogram

// Workgroup barrier that orders LDS accesses only: global loads issued before it stay in flight
// (a plain __syncthreads() also waits for every outstanding global load of the wavefront).
__device__ __forceinline__ void lc_barrier_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ int lc_readlane(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ int lc_wave_sum_i(int v) {                       // all 64 lanes active
    return lc_readlane(lc_wave_scan_incl(v), 63);
}

// What the scoring kernel leaves per chunk (16 bytes, one load): order-preserving score key (0 = not a
// candidate), first cache row, length.
struct LcChunkEntry {
    uint32_t key;
    int start, len, unused;
};

// LDS of the fused step's selection (the general select routine, used when the cutoff bin
// overflows its short list, has its own block)
template <int NT>
struct LcFusedSh {
    int hw[LC_SEL_BINS_MAX + 64];    // chunk lengths per bin; the slots after the last bin take, lane by lane, what is in none
    int4 cand[NT / 64][LC_SEL_CAND]; // chunks of the cutoff bin, by wavefront: key, length, id
    int n_cand[NT / 64];
    uint32_t kmin[NT / 64], kmax[NT / 64];
    int wtok[NT / 64], wcnt[NT / 64];
};
// min / max over a wavefront, uniform result: DPP within the four 16-lane rows, then the rows' values by lane reads
__device__ __forceinline__ uint32_t lc_wave_min_uniform(uint32_t v) {
    v = min(v, lc_dpp_u<0xB1>(v)); v = min(v, lc_dpp_u<0x4E>(v));
    v = min(v, lc_dpp_u<0x141>(v)); v = min(v, lc_dpp_u<0x140>(v));
    const uint32_t r0 = (uint32_t)lc_readlane((int)v, 0), r1 = (uint32_t)lc_readlane((int)v, 16);
    const uint32_t r2 = (uint32_t)lc_readlane((int)v, 32), r3 = (uint32_t)lc_readlane((int)v, 48);
    return min(min(r0, r1), min(r2, r3));
}
__device__ __forceinline__ uint32_t lc_wave_max_uniform(uint32_t v) {
    v = max(v, lc_dpp_u<0xB1>(v)); v = max(v, lc_dpp_u<0x4E>(v));
    v = max(v, lc_dpp_u<0x141>(v)); v = max(v, lc_dpp_u<0x140>(v));
    const uint32_t r0 = (uint32_t)lc_readlane((int)v, 0), r1 = (uint32_t)lc_readlane((int)v, 16);
    const uint32_t r2 = (uint32_t)lc_readlane((int)v, 32), r3 = (uint32_t)lc_readlane((int)v, 48);
    return max(max(r0, r1), max(r2, r3));
}
// number of set bits of `mask` below this lane
__device__ __forceinline__ int lc_mbcnt(unsigned long long mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Selected chunks of one workgroup, in id order: wavefront w's chunks are list entries
// [w * 64 EC, w * 64 EC + n_list), 64 of them per round; the first round stays in registers.
template <int EC>
struct LcChunkSel {
    int2* l_row;         // LDS: first row; length, or -1 - c for chunk c of the cutoff bin
    int* l_id;           // LDS: id (where the ids are wanted)
    int seg, n_list;     // this wavefront's entries (those of the cutoff bin among them, selected or not)
    unsigned long long in_cut;     // chunks of the cutoff bin that are selected: this wavefront's chunk c at bit (cut_first + c) << cut_shift
    int cut_first, cut_shift;
    int st0, ln0, off0;  // this lane's entry of the first round: row, length (0 = not selected), offset among the wavefront's tokens
    int base_tok;        // selected tokens of the wavefronts before this one
    int n_sel_tok;       // selected tokens of the (sequence, head), without the open tail
    int tail_st, tail_ln;
    int n_tok;           // n_sel_tok + tail_ln
    int T, M;
};
// Row and length of a list entry (length 0 past the end or if the budget cut it off).
template <int NT, int EC>
__device__ __forceinline__ void lc_sel_entry(const LcChunkSel<EC>& o, const LcFusedSh<NT>& fs, int r, int* st, int* ln) {
    const int p = o.seg + min(r, max(o.n_list - 1, 0));
    const int2 x = o.l_row[p];
    int l = r < o.n_list ? x.y : 0;
    *st = x.x;
    if (l < 0) {                                                    // (rare: one or two chunks of a wavefront)
        const int c = -1 - l;
        l = ((o.in_cut >> ((o.cut_first + c) << o.cut_shift)) & 1ull) ? fs.cand[threadIdx.x >> 6][c].y : 0;
    }
    *ln = l;
}

// Wavefront w owns the chunks [64 EC w, 64 EC (w + 1)), lane l of it the chunks (EC w + e) * 64 + l
// for e < EC, so every load is coalesced and the id order is (wavefront, e, lane).  The loops over e carry
// no branches, so that the EC copies of each step overlap in the pipeline (one wavefront per SIMD has nothing
// else to hide a dependent instruction's latency behind), and there are few of them: what bounds the
// selection is instructions per chunk, so only the key range, the histogram and one compaction look at
// every chunk; ranking and prefix sums run on the list of the selected ones, a few per cent.
//   1. range of the candidate keys (one exchange), histogram of chunk lengths over it (LDS
//      atomics), every wavefront scans all bins from the top: cutoff bin, budget left for it;
//   2. chunks in that bin and above go to the wavefront's list, those in it also to a short list, which
//      every wavefront ranks (key descending, id ascending) -- or, if it overflows (a crowded or tied
//      bin), the general select routine runs on them;
//   3. token offsets by a wavefront scan of the list, one exchange of the wavefronts' totals.
// (The compaction is six vector instructions per chunk and lane, without a branch; with branches around its writes
// and the short list's in the same loop it was fifty, and a step at 2275 chunks per head took 21.5 us instead of 20.2.)
// `entry(e)`: entry e of this lane (LcChunkEntry; past the array's end anything); chunks whose first token lies below `sink` are pinned: always selected, not
// charged to the budget.  With `ids_out` (per (sequence, head) `cap` entries) the selected ids are also
// written in ascending order and their number to counts_out[bh].  `lds_dyn`: lc_select_lds<NT, EC>() bytes.
// All NT threads must call; NT / 64 wavefronts; holds up to EC * NT chunks.
template <int NT, int EC>
constexpr size_t lc_select_lds() { return (size_t)(EC * NT) * 12 + 64 * 8; }
template <int NT, int EC, typename Entry>
__device__ __forceinline__ void lc_select_chunks(const LcDev& ix, int b, int bh, Entry entry, int budget,
                                                 int sink, int32_t* ids_out, int32_t* counts_out, int cap,
                                                 LcLeafSelSh& sel_sh, LcFusedSh<NT>& fs, int* lds_dyn,
                                                 LcChunkSel<EC>& o) {
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int* bnd = ix.bounds + (size_t)b * (ix.cap[0] + 1);
    // bins of the histogram: about one per four chunks, so that the cutoff bin holds a handful
    constexpr int BITS = EC * NT <= 1024 ? 8 : (EC * NT <= 2560 ? 9 : 10);
    constexpr int BINS = 1 << BITS;
    // ---- every load of the selection goes out at once, before the chunk count is known (what lies past the
    // count is masked below)
    const int j0 = wave * (EC * 64) + lane;                      // this lane's chunk e is j0 + 64 e
    lc_v4i ent[EC];
#pragma unroll
    for (int e = 0; e < EC; ++e) ent[e] = entry(e);
    o.T = ix.state[bh * 4 + 0];
    const int M_all = ix.state[bh * 4 + 1];
    o.l_row = reinterpret_cast<int2*>(lds_dyn);
    o.l_id = lds_dyn + 2 * (EC * NT + 64);
    o.seg = wave * (EC * 64);
    // meanwhile: empty histogram and list (their first use is behind the barrier of the key range)
    for (int i = tid; i < BINS; i += NT) fs.hw[i] = 0;
    o.M = min(M_all, EC * NT);
    o.tail_st = bnd[M_all];
    const int W = budget > 0 ? budget : 0;
    // ---- what is past the count is no candidate (key 0)
    uint32_t ck[EC];
    uint32_t kmin1 = 0xffffffffu, kmax = 0u;                    // (lowest candidate key) - 1, highest
#pragma unroll
    for (int e = 0; e < EC; ++e) {
        const uint32_t k_e = (uint32_t)ent[e].x;
        ck[e] = j0 + 64 * e < o.M ? k_e : 0u;
        kmin1 = min(kmin1, ck[e] - 1u);                         // key 0 wraps to the largest value: ignored
        kmax = max(kmax, ck[e]);
        if (EC > 10 && (e & 3) == 3) __builtin_amdgcn_sched_barrier(0);       // (the conditions of sixteen at a time do not fit the scalar registers)
    }
    {
        const uint32_t wmin = lc_wave_min_uniform(kmin1), wmax = lc_wave_max_uniform(kmax);
        if (lane == 0) { fs.kmin[wave] = wmin; fs.kmax[wave] = wmax; }
    }
    lc_barrier_lds();
    kmin1 = fs.kmin[0];
    kmax = fs.kmax[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) { kmin1 = min(kmin1, fs.kmin[w]); kmax = max(kmax, fs.kmax[w]); }
    const uint32_t kmin = kmin1 + 1u;
    // ---- Histogram of chunk lengths over the upper half of the scores' range (as lc_select_kernel has it, and by its rule): the budget nearly always
    // ends there, and LDS atomics of all chunks, most of them in the same few bins, are most of the step's time otherwise.  Over all of the range if the
    // upper half fits the budget whole, and at once if the budget is a third of the tokens or more.  Bins are even steps of the key, or of the score
    // where the keys' range is over 32 binary orders: keys of scores of both signs crowd around zero, with the chunks that
    // matter in two or three bins (unit-norm centers, 4 x 32K tokens in chunks of 16 to 128: 17.6 us a step, now 14.2; one sequence of 49K in
    // chunks of 8 to 16: 23.5 and 16.6).
    constexpr int PER = BINS / 64;
    int cbin[EC];                                               // -1: no candidate, or below the range
    int fb = -1, remW = W;                                      // cutoff bin (-1: every candidate fits), budget left for it
    const bool signs = kmax - kmin > (32u << 23);
    for (bool half = W < o.T / 3;; half = false) {
        uint32_t lo = half ? kmax - (kmax - kmin) / 2u : kmin;
        bool by_key = true;                                     // (uniform)
        if (__builtin_expect(signs, 0)) {
            const float s_hi = lc_key_score(kmax), s_all = s_hi - lc_key_score(kmin);
            by_key = !(s_all > 1e-30f && s_all < 1e30f);        // (infinities)
            if (!by_key) {
                const float s_lo = half ? s_hi - 0.5f * s_all : lc_key_score(kmin);
                const float per_bin = (float)BINS * __builtin_amdgcn_rcpf(half ? 0.5f * s_all : s_all);
#pragma unroll
                for (int e = 0; e < EC; ++e) {
                    const float s = lc_key_score(ck[e]) - s_lo;
                    cbin[e] = ck[e] != 0u && s >= 0.f ? min((int)(s * per_bin), BINS - 1) : -1;
                    atomicAdd(&fs.hw[cbin[e] >= 0 ? cbin[e] : BINS + lane], ent[e].z);
                }
            }
        }
        if (__builtin_expect(by_key, 1)) {
            lo = max(lo, 1u);                                   // (key 0 is no candidate)
            const uint32_t span = kmax - lo;
            const int bits = (kmax != 0u && span) ? 32 - __clz(span) : 0;
            const int shift = bits > BITS ? bits - BITS : 0;    // (span >> shift) < BINS
#pragma unroll
            for (int e = 0; e < EC; ++e) {
                cbin[e] = ck[e] >= lo ? (int)((ck[e] - lo) >> shift) : -1;
                atomicAdd(&fs.hw[ck[e] >= lo ? cbin[e] : BINS + lane], ent[e].z);
            }
        }
        lc_barrier_lds();
        // every wavefront scans all bins from the top: lane l holds bins BINS - 1 - PER l - i, i < PER
        int pw[PER];                                            // inclusive prefix sums within the lane, bins descending
        const int4* hw4 = reinterpret_cast<const int4*>(fs.hw + BINS - PER * (lane + 1));
#pragma unroll
        for (int v = 0; v < PER / 4; ++v) {
            const int4 x = hw4[PER / 4 - 1 - v];
            pw[4 * v + 0] = x.w; pw[4 * v + 1] = x.z; pw[4 * v + 2] = x.y; pw[4 * v + 3] = x.x;
        }
#pragma unroll
        for (int i = 1; i < PER; ++i) pw[i] += pw[i - 1];
        const int cw = lc_wave_scan_incl(pw[PER - 1]) - pw[PER - 1];      // length of all higher lanes' bins
        // bins of this lane that still fit (prefix sums grow, so they are the first `fit` ones) and their total
        int fit = 0, fitw = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const bool ok = cw + pw[i] <= W;
            fit += ok ? 1 : 0;
            fitw = ok ? pw[i] : fitw;
        }
        const unsigned long long bal = __ballot(fit < PER);     // the prefix ends in the first bin that no longer fits
        if (bal != 0ull) {
            const int fl = __ffsll((long long)bal) - 1;         // lowest lane = highest bins
            fb = BINS - 1 - (PER * fl + lc_readlane(fit, fl));
            remW = W - (lc_readlane(cw, fl) + lc_readlane(fitw, fl));
            break;
        }
        if (!half) break;
        lc_barrier_lds();                                       // the bins have been read
        for (int i = tid; i < BINS; i += NT) fs.hw[i] = 0;
        lc_barrier_lds();
    }
    // ---- chunks of that bin and above, and the pinned ones, to this wavefront's list; those in it to the short list
    if (sink > 0) {                                             // (pinned chunks: as if in a bin above all)
#pragma unroll
        for (int e = 0; e < EC; ++e) cbin[e] = j0 + 64 * e < o.M && ent[e].y < sink ? BINS : cbin[e];
    }
    const bool want_ids = ids_out != nullptr;                   // (uniform)
    const int lowest = max(fb, 0), cutoff = fb >= 0 ? fb : -2;
    int n_cut = 0;
    o.n_list = 0;
    unsigned long long mi[EC], mc[EC];
    // (no branch: a lane without a chunk for the list writes to a slot of its own behind it)
#pragma unroll
    for (int e = 0; e < EC; ++e) {
        mi[e] = __ballot(cbin[e] >= lowest);
        mc[e] = __ballot(cbin[e] == cutoff);
        const int at = o.seg + o.n_list + lc_mbcnt(mi[e]);
        o.l_row[cbin[e] >= lowest ? at : EC * NT + lane] = make_int2(ent[e].y, ent[e].z);
        o.n_list += __popcll(mi[e]);
    }
    if (want_ids) {
        int first = o.seg;
#pragma unroll
        for (int e = 0; e < EC; ++e) {
            if (cbin[e] >= lowest) o.l_id[first + lc_mbcnt(mi[e])] = j0 + 64 * e;
            first += __popcll(mi[e]);
        }
    }
    int first = o.seg;
#pragma unroll
    for (int e = 0; e < EC; ++e) {
        if (mc[e] != 0ull) {                                    // (uniform; few of the rows)
            const int c = n_cut + lc_mbcnt(mc[e]);
            if (cbin[e] == cutoff) {
                o.l_row[first + lc_mbcnt(mi[e])].y = -1 - c;
                if (c < LC_SEL_CAND) fs.cand[wave][c] = make_int4((int)ck[e], ent[e].z, j0 + 64 * e, 0);
            }
            n_cut += __popcll(mc[e]);
        }
        first += __popcll(mi[e]);
    }
    if (lane == 0) fs.n_cand[wave] = n_cut;
    lc_barrier_lds();
    bool crowded = false;
    int nc = 0, after[NW];                                      // chunks of the short list: all, up to each wavefront's last
    o.cut_first = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int n = lc_readlane(fs.n_cand[w], 0);
        crowded = crowded || n > LC_SEL_CAND;
        if (w == wave) o.cut_first = nc;
        nc += n;
        after[w] = nc;
    }
    o.in_cut = 0ull;
    o.cut_shift = 0;
    if (!crowded) {
        // ---- the short list ranked by (key descending, id ascending): a chunk is selected if it fits with those before it.
        // A few, as nearly always, by a lane for each pair of them; more by a lane for each.  (One after the other through scalar registers, every
        // chunk of the list cost 0.06 us: 0.6 us at the median, 1.1 in one step of twenty, now 0.25.)
        static_assert(NW * LC_SEL_CAND <= 64, "one lane per slot of the short list, one bit of the result for each");
        auto listed = [&](int i) -> int4 {
            int w = 0, c = i;
#pragma unroll
            for (int x = 0; x + 1 < NW; ++x)
                if (i >= after[x]) { w = x + 1; c = i - after[x]; }
            return fs.cand[w][min(c, LC_SEL_CAND - 1)];
        };
        auto precedes = [](const int4& x, const int4& y) { return (uint32_t)x.x > (uint32_t)y.x || (x.x == y.x && x.z < y.z); };
        if (nc <= LC_SEL_FEW) {
            const int i = lane / LC_SEL_FEW, j = lane % LC_SEL_FEW;
            const int4 me = listed(i), other = listed(j);
            int before = j < nc && precedes(other, me) ? other.y : 0;
            before += __builtin_amdgcn_update_dpp(0, before, 0xB1, 0xF, 0xF, true);      // over eight lanes
            before += __builtin_amdgcn_update_dpp(0, before, 0x4E, 0xF, 0xF, true);
            before += __builtin_amdgcn_update_dpp(0, before, 0x141, 0xF, 0xF, true);
            o.in_cut = __ballot(i < nc && before + me.y <= remW);
            o.cut_shift = 3;
        } else {
            const int4 me = listed(lane);
            int before = 0;
            for (int c = 0; c < nc; ++c) {                      // (uniform)
                const int4 other = make_int4(lc_readlane(me.x, c), lc_readlane(me.y, c), lc_readlane(me.z, c), 0);
                before += precedes(other, me) ? other.y : 0;
            }
            o.in_cut = __ballot(lane < nc && before + me.y <= remW);
        }
    } else {
        // ---- a crowded or tied cutoff bin: the general select routine on its chunks alone, then the lists anew
        uint32_t* skey = reinterpret_cast<uint32_t*>(lds_dyn);
        int* slen = lds_dyn + EC * NT;
        lc_leaf_select_prepare<NT>(sel_sh);
        lc_barrier_lds();
        uint32_t bmin = 0xffffffffu, bmax = 0u;
#pragma unroll
        for (int e = 0; e < EC; ++e) {
            const int j = j0 + 64 * e;
            const bool cnd = fb >= 0 && cbin[e] == fb;
            const uint32_t k = cnd ? (ck[e] == 0xffffffffu ? 0xfffffffeu : ck[e]) : 0u;     // the mark is reserved
            skey[j] = k;
            slen[j] = ent[e].z;
            if (cnd) { bmin = min(bmin, k); bmax = max(bmax, k); }
        }
        lc_leaf_select_range(bmin, bmax, sel_sh);
        lc_barrier_lds();
        const uint32_t thr = lc_leaf_select<NT>(o.M, skey, slen, (long long)remW, 0x7fffffffLL, sel_sh);
        __syncthreads();
        bool keep[EC];
#pragma unroll
        for (int e = 0; e < EC; ++e) keep[e] = fb >= 0 && cbin[e] == fb && skey[j0 + 64 * e] > thr;
        __syncthreads();
        o.n_list = 0;
#pragma unroll
        for (int e = 0; e < EC; ++e) {
            const int j = j0 + 64 * e;
            const bool in = keep[e] || cbin[e] > fb;
            const unsigned long long m = __ballot(in);
            const int p = o.seg + o.n_list + lc_mbcnt(m);
            if (in) { o.l_row[p] = make_int2(ent[e].y, ent[e].z); if (want_ids) o.l_id[p] = j; }
            o.n_list += __popcll(m);
        }
        lc_barrier_lds();
    }
    // ---- token offsets in id order: a scan of the list (one round of 64 nearly always), then the wavefronts' totals
    {
        lc_sel_entry<NT, EC>(o, fs, lane, &o.st0, &o.ln0);
        const int inc = lc_wave_scan_incl(o.ln0);
        o.off0 = inc - o.ln0;
        int tok = lc_readlane(inc, 63), cnt = __popcll(__ballot(o.ln0 > 0));
        for (int r = 64; r < o.n_list; r += 64) {
            int st, ln;
            lc_sel_entry<NT, EC>(o, fs, r + lane, &st, &ln);
            tok += lc_wave_sum_i(ln);
            cnt += __popcll(__ballot(ln > 0));
        }
        if (lane == 0) { fs.wtok[wave] = tok; fs.wcnt[wave] = cnt; }
    }
    lc_barrier_lds();
    o.base_tok = 0;
    o.n_sel_tok = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int wt = fs.wtok[w];
        if (w < wave) o.base_tok += wt;
        o.n_sel_tok += wt;
    }
    o.tail_ln = max(0, o.T - o.tail_st);
    o.n_tok = o.n_sel_tok + o.tail_ln;
    if (ids_out != nullptr) {                                   // (uniform) the chunk list, for callers that want it
        int at = 0, n_sel = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int wc = fs.wcnt[w];
            if (w < wave) at += wc;
            n_sel += wc;
        }
        int32_t* io = ids_out + (size_t)bh * cap;
        for (int r = 0; r < o.n_list; r += 64) {
            int st, ln;
            lc_sel_entry<NT, EC>(o, fs, r + lane, &st, &ln);
            const unsigned long long m = __ballot(ln > 0);
            const int p = at + lc_mbcnt(m);
            if (ln > 0 && p < cap) io[p] = o.l_id[o.seg + r + lane];
            at += __popcll(m);
        }
        if (tid == 0 && counts_out != nullptr) counts_out[bh] = min(n_sel, cap);
    }
}
