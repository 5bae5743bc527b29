// Retrieval kernels: Eq. 2 node scoring, level-by-level pruning, budget selection.
//
// lc_upper_kernel (EXACT policy with the level walk on): one workgroup per (sequence, KV head).
// It stages the internal nodes' small arrays (parents, subtree token counts) in LDS with a few
// batched loads, scores every internal node (levels >= 1), and walks the levels top-down with
// the frontier held in LDS: a probe pass gives a lower bound tau0 of the selection cutoff, the
// verify pass keeps every node whose bound reaches tau0.  It leaves one byte per level-1 node:
// score the chunks below it or not.
//
// lc_beam_kernel (BEAM policy, Algorithm 1): one workgroup per (sequence, KV head) does the whole
// retrieval -- per level score the candidates, keep the beam[l] best, gather their children; at
// the chunk level cut by the token budget and write the ids.
//
// lc_score_kernel: one 16-byte entry (key, first token, length) per chunk, many workgroups per (sequence, KV head).  First kernel of
// a decode step, whose attention workgroups select from the entries, and of lc_retrieve, whose
// second kernel does:
//
// lc_select_kernel: one workgroup per (sequence, KV head) selects from the entries and writes the ids (lc_retrieve, and the
// decode step beyond what its selecting workgroups hold).
//
// lc_leaf_kernel (the same beyond what lc_select_kernel's registers hold, and in one band below: launch_retrieve_g): many workgroups per
// (sequence, KV head) score the wanted chunks; the last workgroup to finish for a (sequence, head) pulls the keys into LDS, runs the weighted histogram select (weights =
// chunk lengths) and emits the ids in ascending order.
//
// The kernels are latency-bound at batch 1, so global loads are issued in batches
// and nothing reads global memory element by element inside a dependent loop.
#include "lc_device.h"
#include "lc_internal.h"
#include "lc_select.h"
#include "lc_walk_layout.h"

#include <type_traits>

#define LC_INLINE __attribute__((always_inline))       // (lambdas that hold registers by reference)
#define LC_TAU_SLACK 1e-3f
#define LC_COUNT_SELECT_MAX 1024         // up to this many candidates the O(n^2 / threads) rank is used


struct LcRetrieveArgs {
    LcDev ix;
    const uint16_t* q;       // [B][H_q][d]
    uint32_t* keys;          // [B][H][cap0]
    uint8_t* want;           // [B][H][cap0], first N_1 entries used: 1 = this level-1 node was kept, i.e. the
                             // chunks below it are to be scored (the chunk kernel looks its chunks' parents up)
    float* scores;           // [B][H][cap0] or null
    int32_t* ids;            // [B][H][cap]
    int32_t* counts;         // [B][H]
    int* scratch;            // [B][H][4 * cap0] ints: chunk-level staging when it does not fit in LDS; the
                             // chunk entries of lc_score_kernel
    int cap;
    int budget;
    int policy;
    int sink;
    int beam[LC_MAX_LEVELS];
    int upper_cap;           // LDS entries for internal nodes
    int walk;                // 1 = the internal levels were walked and `want` is valid
    int chunk_cap;           // upper kernel: LDS entries of the probe list; leaf kernel: LDS entries for
                             // the select's staging, 0 = stage in `scratch` (global memory)
    int score_only;          // 1 = only the score keys are wanted (lc_score_kernel; the fused decode step selects)
};

// Selection among n <= LC_COUNT_SELECT_MAX candidates whose keys / weights sit in 16-byte aligned,
// zero-padded LDS arrays: keeps the shortest prefix whose weight reaches W (everything if it never does).
// Writes flags[i] for i < n.  With REDUCE it also returns, in every thread, the smallest kept key
// (0 if nothing kept) and whether the kept weight reached W; that costs three barriers.
template <int NT, bool REDUCE>
__device__ __forceinline__ void lc_small_select(int n, long long W, const uint32_t* keys,
                                                const int* wgts, uint8_t* flags, int* sh, uint32_t* min_kept,
                                                int* reached) {
    uint32_t mk = 0xffffffffu;
    int hit = 0;
    const int part = threadIdx.x & 15;
    for (int base = 0; base < n; base += NT / 16) {           // NT/16 items per round, 16 lanes each
        const int i = base + (threadIdx.x >> 4);
        const uint32_t ki = i < n ? keys[i] : 0u;
        int cb, wb;
        lc_rank_before16(ki != 0u ? n : 0, keys, wgts, i, ki, part, &cb, &wb);
        int keep = 0;
        if (ki != 0u) {
            const int wi = wgts[i];
            keep = ((long long)wb < W) ? 1 : 0;
            if (keep && (long long)wb + wi >= W) hit = 1;
        }
        if (part == 0 && i < n) flags[i] = (uint8_t)keep;
        if (keep) mk = min(mk, ki);
    }
    if (!REDUCE) {                   // flags only: the caller synchronises before it reads them
        *min_kept = 0u;
        *reached = 0;
        return;
    }
    mk = lc_wave_min_u(mk);
    hit = (int)lc_wave_max_u((uint32_t)(hit != 0));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) { sh[threadIdx.x >> 6] = (int)mk; sh[32 + (threadIdx.x >> 6)] = hit; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) { mk = min(mk, (uint32_t)sh[w]); hit |= sh[32 + w]; }
    __syncthreads();
    *min_kept = (mk == 0xffffffffu) ? 0u : mk;
    *reached = hit;
}

// ---------------------------------------------------------------------------------
// lc_upper_kernel: internal levels (EXACT walk)
// ---------------------------------------------------------------------------------
// (LDS layout: lc_walk_layout.h: 13 bytes per internal-node slot, 16 per select-scratch slot, 12 per probe-list slot)

// One workgroup of 1024 threads (64 groups of 16 lanes) per (sequence, head).  All
// global loads of a phase are issued before any of them is used: at batch 1 the
// kernel's duration is a chain of memory round trips, not bandwidth.
#define LC_UP_THREADS 1024
#define LC_UP_GROUPS (LC_UP_THREADS / 16)
#define LC_UP_PER_THREAD 4

template <int G>
__global__ void __launch_bounds__(LC_UP_THREADS)
lc_upper_kernel(const LcRetrieveArgs a) {
    extern __shared__ int lds_dyn[];
    __shared__ int sel_sh[LC_SEL_SH];
    __shared__ int off_sh[LC_MAX_LEVELS + 1];
    constexpr int NB = (G <= 4) ? 4 : 2;          // nodes in flight per group

    const LcDev& ix = a.ix;
    const int h = blockIdx.x, b = blockIdx.y;
    const int bh = b * ix.H + h;
    const int tid = threadIdx.x;
    const int sub = tid & 15, grp = tid >> 4;
    const int L = ix.L;
    const int M = ix.state[bh * 4 + 1];

    if (tid == 0) {
        int o = 0;
        for (int l = 1; l < L; ++l) { off_sh[l] = o; o += ix.nlev[b * LC_MAX_LEVELS + l]; }
        off_sh[L] = o;
        off_sh[0] = 0;
    }
    // LDS carve-up: internal nodes (UC entries each), select scratch, probe list (PC entries each)
    const int UC = a.upper_cap, PC = a.chunk_cap;
    const LcUpperLayout ly = lc_upper_layout(UC, PC);
    char* const lds_b = reinterpret_cast<char*>(lds_dyn);
    uint32_t* ukey = reinterpret_cast<uint32_t*>(lds_b + ly.ukey);
    int* untok = reinterpret_cast<int*>(lds_b + ly.untok);
    int* upar = reinterpret_cast<int*>(lds_b + ly.upar);
    uint8_t* kp = reinterpret_cast<uint8_t*>(lds_b + ly.kp);
    // two (key, weight) staging buffers for the per-level selects, used alternately
    uint32_t* ekA = reinterpret_cast<uint32_t*>(lds_b + ly.ekA);
    int* ewA = reinterpret_cast<int*>(lds_b + ly.ewA);
    uint32_t* ekB = reinterpret_cast<uint32_t*>(lds_b + ly.ekB);
    int* ewB = reinterpret_cast<int*>(lds_b + ly.ewB);
    int* plist = reinterpret_cast<int*>(lds_b + ly.plist);
    int* plen = reinterpret_cast<int*>(lds_b + ly.plen);
    uint32_t* pkey = reinterpret_cast<uint32_t*>(lds_b + ly.pkey);

    // Query fragments: widened once for small groups; for large ones kept as packed bfloat16 words
    // and widened per node, which keeps this 1024-thread kernel within its 128 registers per lane.
    constexpr bool QP = G > 4;
    float qf[QP ? 1 : G][8], qn[G];
    uint32_t qp[QP ? G : 1][4];
    if constexpr (QP) lc_load_query_packed<G>(a.q + (size_t)b * ix.H * G * LC_D, h, sub, qp, qn);
    else lc_load_query_frags<G>(a.q + (size_t)b * ix.H * G * LC_D, h, sub, qf, qn);
    auto score_node = [&](const LcNodeFrag& f, float R) -> float {
        if constexpr (QP) return lc_score_frag_packed<G>(f, R, qp, qn);
        else return lc_score_frag<G>(f, R, qf, qn);
    };
    // prefetch what the chunk pass will need much later (parents and boundaries of this thread's
    // first LC_UP_PER_THREAD chunks): the arrays are cap[0] long, so no count is needed to load them
    int pf_p[LC_UP_PER_THREAD], pf_s[LC_UP_PER_THREAD + 1];
    {
        const int* bnd_e = ix.bounds + (size_t)b * (ix.cap[0] + 1);
        const int* par_e = ix.parent[0] + (size_t)bh * ix.cap[0];
        const int j0 = tid * LC_UP_PER_THREAD;
#pragma unroll
        for (int k = 0; k < LC_UP_PER_THREAD; ++k) pf_p[k] = par_e[min(j0 + k, ix.cap[0] - 1)];
#pragma unroll
        for (int k = 0; k <= LC_UP_PER_THREAD; ++k) pf_s[k] = bnd_e[min(j0 + k, ix.cap[0])];
    }
    __syncthreads();
    const int NU = off_sh[L];

    // ---- internal nodes, all levels as one list: parents, token counts, scores
    auto level_of = [&](int u) -> int {
        int l = 1;
        while (l + 1 < L && u >= off_sh[l + 1]) ++l;
        return l;
    };
    for (int u = tid; u < NU; u += LC_UP_THREADS) {
        const int l = level_of(u);
        const size_t n = (size_t)bh * ix.cap[l] + (u - off_sh[l]);
        untok[u] = ix.ntok[l][n];
        upar[u] = ix.parent[l][n];
    }
    for (int u0 = grp; u0 < NU; u0 += NB * LC_UP_GROUPS) {
        LcNodeFrag f[NB];
        float R[NB];
        int nc[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int u = min(u0 + k * LC_UP_GROUPS, NU - 1);
            const int l = level_of(u);
            const size_t n = (size_t)bh * ix.cap[l] + (u - off_sh[l]);
            f[k] = lc_load_node(ix.center[l] + n * LC_D, sub);
            R[k] = ix.radius[l][n];
            nc[k] = ix.nchunk[l][n];
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int u = u0 + k * LC_UP_GROUPS;
            float s = score_node(f[k], R[k]);
            if (nc[k] <= 0) s = LC_NEG_INF;
            if (sub == 0 && u < NU) ukey[u] = lc_score_key(s);
        }
    }
    __syncthreads();

    uint8_t* want = a.want + (size_t)bh * ix.cap[0];
    const int* bnd = ix.bounds + (size_t)b * (ix.cap[0] + 1);
    const int* par0 = ix.parent[0] + (size_t)bh * ix.cap[0];
    const int o1 = off_sh[1];
    const int n_1 = (L > 2 ? off_sh[2] : off_sh[L]) - o1;
    if (a.budget <= 0) {
        for (int i = tid; i < n_1; i += LC_UP_THREADS) want[i] = 0;
        return;
    }

    // the outcome of the walk: which level-1 nodes were kept (the chunk kernel maps chunks to them)
    auto write_want = [&]() {
        for (int i = tid; i < n_1; i += LC_UP_THREADS) want[i] = kp[o1 + i];
    };
    // Per-level selection.  The candidates of a level (frontier nodes: key, weight; others: 0) sit in
    // one staging buffer; the select writes kept flags; the children of the kept nodes are staged into
    // the other buffer for the next level.  Two barriers per level.
    uint32_t* ek = ekA;
    int* ew = ewA;
    uint32_t* ek_next = ekB;
    int* ew_next = ewB;
    {
        const int o = off_sh[L - 1], n_l = off_sh[L] - o;
        for (int i = tid; i < ((n_l + 3) & ~3); i += LC_UP_THREADS) {
            ek[i] = i < n_l ? ukey[o + i] : 0u;
            ew[i] = i < n_l ? untok[o + i] : 0;
        }
        __syncthreads();
    }
    for (int l = L - 1; l >= 1; --l) {
        const int o = off_sh[l], n_l = off_sh[l + 1] - o;
        uint32_t mk;
        int reached;
        {
            // EXACT, probe pass: keep the best frontier nodes until their subtree token counts reach the budget
            if (n_l <= LC_COUNT_SELECT_MAX) {
                lc_small_select<LC_UP_THREADS, false>(n_l, (long long)a.budget, ek, ew, kp + o, sel_sh, &mk, &reached);
            } else {
                auto keyf = [&](int i) -> uint32_t { return ek[i]; };
                auto wf = [&](int i) -> int { return ew[i]; };
                const LcSel r = lc_block_select<LC_UP_THREADS>(n_l, (long long)a.budget - 1, 0x7fffffffLL, keyf, wf, sel_sh);
                for (int i = tid; i < n_l; i += LC_UP_THREADS)
                    kp[o + i] = (ek[i] != 0u && (r.all || ek[i] >= r.kstar)) ? 1 : 0;      // whole tie group
            }
        }
        __syncthreads();
        if (l >= 2) {                 // stage the children of the kept nodes as the next level's candidates
            const int ob = off_sh[l - 1], n_b = off_sh[l] - ob;
            for (int n = tid; n < ((n_b + 3) & ~3); n += LC_UP_THREADS) {
                const bool in = n < n_b && kp[o + upar[ob + n]];
                ek_next[n] = in ? ukey[ob + n] : 0u;
                ew_next[n] = in ? untok[ob + n] : 0;
            }
            __syncthreads();
            uint32_t* tk = ek; ek = ek_next; ek_next = tk;
            int* tw = ew; ew = ew_next; ew_next = tw;
        }
    }
    // ---- compact the probe's chunks (children of the kept level-1 nodes, not pinned) into LDS.
    // The list holds at most PC chunks; dropping the rest only weakens tau0, never the result.
    int n_probe = 0;
    for (int base = 0; base < M; base += LC_UP_THREADS * LC_UP_PER_THREAD) {
        const int j0 = base + tid * LC_UP_PER_THREAD;
        int p[LC_UP_PER_THREAD], s0[LC_UP_PER_THREAD + 1];
        if (base == 0) {
#pragma unroll
            for (int k = 0; k < LC_UP_PER_THREAD; ++k) p[k] = pf_p[k];
#pragma unroll
            for (int k = 0; k <= LC_UP_PER_THREAD; ++k) s0[k] = pf_s[k];
        } else {
#pragma unroll
            for (int k = 0; k < LC_UP_PER_THREAD; ++k) p[k] = par0[max(0, min(j0 + k, M - 1))];
#pragma unroll
            for (int k = 0; k <= LC_UP_PER_THREAD; ++k) s0[k] = bnd[min(j0 + k, M)];
        }
        int f[LC_UP_PER_THREAD], cnt = 0;
#pragma unroll
        for (int k = 0; k < LC_UP_PER_THREAD; ++k) {
            f[k] = (j0 + k < M && s0[k] >= a.sink && kp[o1 + p[k]]) ? 1 : 0;
            cnt += f[k];
        }
        int tot;
        int pos = n_probe + lc_block_scan<LC_UP_THREADS>(cnt, sel_sh, &tot);
#pragma unroll
        for (int k = 0; k < LC_UP_PER_THREAD; ++k) {
            if (f[k]) {
                if (pos < PC) { plist[pos] = j0 + k; plen[pos] = s0[k + 1] - s0[k]; }
                ++pos;
            }
        }
        n_probe += tot;
    }
    n_probe = min(n_probe, PC);
    __syncthreads();
    // ---- score them
    {
        const size_t cb = (size_t)bh * ix.cap[0];
        const bool c0b = ix.c0_bf16 != 0;
        for (int i0 = grp; i0 < n_probe; i0 += NB * LC_UP_GROUPS) {
            LcNodeFrag f[NB];
            float R[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const int j = plist[min(i0 + k * LC_UP_GROUPS, n_probe - 1)];
                f[k] = lc_load_chunk_node(ix.center[0], c0b, cb + j, sub);
                R[k] = ix.radius[0][cb + j];
            }
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const int i = i0 + k * LC_UP_GROUPS;
                const float s = score_node(c0b ? lc_widen_chunk_frag(f[k]) : f[k], R[k]);
                if (sub == 0 && i < n_probe) pkey[i] = lc_score_key(s);
            }
        }
        // zero padding for the vector reads of the select
        if (tid < 4 && n_probe + tid < ((n_probe + 3) & ~3)) { pkey[n_probe + tid] = 0u; plen[n_probe + tid] = 0; }
    }
    __syncthreads();
    // ---- tau0: the score at which the probe chunks' cumulative length reaches the budget
    uint32_t tau_key = 1u;                  // keep everything unless the probe proves a cutoff
    {
        uint32_t cut = 0u;
        int reached = 0;
        if (n_probe <= LC_COUNT_SELECT_MAX) {
            lc_small_select<LC_UP_THREADS, true>(n_probe, (long long)a.budget, pkey, plen,
                                                 reinterpret_cast<uint8_t*>(ekA), sel_sh, &cut, &reached);
        } else {
            auto keyf = [&](int i) -> uint32_t { return pkey[i]; };
            auto wf = [&](int i) -> int { return plen[i]; };
            const LcSel r = lc_block_select<LC_UP_THREADS>(n_probe, (long long)a.budget - 1, 0x7fffffffLL, keyf, wf, sel_sh);
            reached = r.all ? 0 : 1;
            cut = r.kstar;
        }
        if (reached && cut != 0u) {
            const float tau = lc_key_score(cut);
            tau_key = lc_score_key(tau - LC_TAU_SLACK * fmaxf(1.0f, fabsf(tau)));
            if (tau_key == 0u) tau_key = 1u;
        }
    }
    // ---- verify pass: keep every node whose bound reaches tau0 and whose parent was kept
    {
        const int o = off_sh[L - 1], n_l = off_sh[L] - o;
        for (int i = tid; i < n_l; i += LC_UP_THREADS) kp[o + i] = (ukey[o + i] >= tau_key) ? 1 : 0;
        __syncthreads();
    }
    for (int l = L - 2; l >= 1; --l) {
        const int o = off_sh[l], n_l = off_sh[l + 1] - o, oa = off_sh[l + 1];
        for (int i = tid; i < n_l; i += LC_UP_THREADS)
            kp[o + i] = (ukey[o + i] >= tau_key && kp[oa + upar[o + i]]) ? 1 : 0;
        __syncthreads();
    }
    write_want();
}


// ---------------------------------------------------------------------------------
// top-k per level (Algorithm 1): the whole retrieval in one workgroup per (sequence, KV head)
// ---------------------------------------------------------------------------------
// Only the children of the kept nodes are ever scored, so the work follows the beam sizes, not the
// size of the index: per level, score the candidate list (ascending node order, so that equal
// scores fall to the lower id), keep the best, mark them in a bitmap, gather their children.
// The chunks under the kept level-1 nodes are scored the same way, cut by the token budget (and the
// chunk-count limit beam[0]) and written out in ascending order behind the pinned chunks.
//
// One compute unit works on a (sequence, head), one stage after the other: what bounds it is the chain of
// memory round trips, and the unit's instruction rate -- an instruction that all sixteen wavefronts execute takes
// 16 cycles.  So
//   - the query and the top level's first rows, whose addresses depend on no result, are on their way before the first
//     wait; when they have come, the parent pointers of all levels go straight into LDS (those that fit: the
//     upper levels first);
//   - a group of 16 lanes scores four nodes at a time (lc_score_packed), the best are found by one wavefront from a
//     histogram of 64 bins (lc_wave_cut), a list is written from the lanes' marks by one scan and one
//     exchange of counts (gather below);
//   - all levels run through one loop, so that the later ones find its code in the instruction cache;
//   - the lists are in LDS, and code that reads them knows that they are (an address that may be either
//     LDS or memory costs a wait for both); a list longer than `list_slots` goes to the workspace.
// 10.9 K chunks under 5461 and 249 nodes, 43 and 8 of them kept, 8 heads: 34.7 us with a copy of the code per level,
// every node scored by itself and ranks by counting, 25.2 us now; 2275 chunks under four levels: 26 and 24.4 us.  A step over the first, with
// three passes over LDS per cut (2.0 us of 183 candidates) and the parent pointers ahead of the rows 31.8 us, now 29.2 (a cut 1.3 us;
// of 500 chunks by their lengths 3.1 and 1.7); with 512 threads 34.1, with 256 43.6.
// A flat scan of up to this many chunks is the same with one level: one kernel (8 heads of 48 chunks: 7.6 us as scoring and
// selection, 6.7 here; of 63 7.3 and 6.7); beyond, one compute unit's scoring and cut cost more (240: 6.7 and 10.1 us).
#define LC_FLAT_MAX_CHUNKS 64
#define LC_BM_THREADS 1024
#define LC_BM_WAVES (LC_BM_THREADS / 64)
#define LC_BM_GROUPS (LC_BM_THREADS / 16)
#define LC_BM_MAX_LEVEL_NODES 65536       // marks of kept nodes: one byte each in LDS
#define LC_BM_RANK_MAX 24                // lists up to this length are ranked by one wavefront,
#define LC_BM_CUT_MAX 1024               // up to this length cut by one wavefront with a histogram, longer ones by the workgroup
#define LC_BM_STATIC_LDS (8 * 1024)      // what the kernel's own arrays take, rounded up
#define LC_BM_SPAN 8                     // blocks of 4096 items that one pass of the gather looks at

// The kernel's arguments by level, from the top (0) to the chunks (L - 1): what a level needs is together, and the
// top level's part has a fixed address in the argument block (an entry that is looked up by a number known
// only at run time waits for its own read of that block).
struct LcBeamLevel {
    const float* center;
    const float* radius;
    const int* nchunk;
    const int* parent;
    int cap, beam;
    int par_words;           // LDS words its parent pointers take
};
struct LcBeamArgs {
    LcBeamLevel lev[LC_MAX_LEVELS];
    const uint16_t* q;
    const int* bounds;
    const int* state;
    const int* nlev;
    float* scores;
    int32_t* ids;
    int32_t* counts;
    int* scratch;
    int H, L, cap0, cap, budget, sink, c0_bf16;
    int list_slots;          // LDS entries of each candidate list
    int kept_words;          // LDS words for the marks of kept nodes
    int par_slots;           // LDS words for parent pointers
};

// Bins of a key range [a, b], 64 of them: even steps of the score (keys of scores of both signs crowd around zero)
// or of the key.  Higher keys are in the same bin or a higher one.
struct LcKeyBins {
    uint32_t a, b;
    float s_lo, step;
    int shift;
    bool by_score;
    __device__ __forceinline__ void over(uint32_t lo, uint32_t hi, bool score) {
        a = lo;
        b = hi;
        const uint32_t span = b - a;
        shift = span >= 64u ? 26 - __clz((int)span) : 0;             // (span >> shift) < 64
        s_lo = lc_key_score(a);
        step = 64.0f * __builtin_amdgcn_rcpf(lc_key_score(b) - s_lo);
        by_score = score && step > 0.f && step < 1e30f;             // (not for one key, nor for infinities)
    }
    __device__ __forceinline__ int of(uint32_t k) const {            // -1: not in the range, or no candidate
        const int by_s = min(max((int)((lc_key_score(k) - s_lo) * step), 0), 63);
        return k >= a && k <= b && k != 0u ? (by_score ? by_s : (int)((k - a) >> shift)) : -1;
    }
};
// The first round of lc_wave_cut where a lane holds all its R candidates (positions lane + 64 r, n <= 64 R) in registers: one pass over the LDS instead of
// three, no loops.  False (and nothing changed) where bins over the score make no sense or the bin of the cut has more than 64
// candidates.
template <int R>
__device__ __forceinline__ bool lc_wave_cut_held(int n, uint32_t* key, const int* wgt, bool weighted, int W, int C, int* hist, uint32_t* cut) {
    const int lane = threadIdx.x & 63;
    const bool counted = C < 0x7fffffff;
    uint32_t k[R];
    int w[R], bin[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = min(64 * r + lane, n - 1);
        k[r] = key[i];
        w[r] = wgt[i];
    }
    hist[lane] = 0;
    hist[64 + lane] = 0;
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        k[r] = 64 * r + lane < n ? k[r] : 0u;
        lo = min(lo, k[r] - 1u);                                    // (key 0 wraps to the largest value: ignored)
        hi = max(hi, k[r]);
    }
    lo = lc_wave_min_uniform(lo) + 1u;
    hi = lc_wave_max_uniform(hi);
    const float s_lo = lc_key_score(lo), step = 64.0f * __builtin_amdgcn_rcpf(lc_key_score(hi) - s_lo);
    if (!(hi != 0u && step > 0.f && step < 1e30f)) return false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        // (no branch around the additions: what is no candidate adds to a slot that nobody reads)
        const int slot = 63 - min((int)((lc_key_score(k[r]) - s_lo) * step), 63);
        bin[r] = k[r] != 0u ? slot : -1;
        if (weighted) atomicAdd(&hist[k[r] != 0u ? slot : 128 + lane], w[r]);
        if (counted) atomicAdd(&hist[k[r] != 0u ? 64 + slot : 128 + lane], 1);
    }
    __builtin_amdgcn_wave_barrier();
    const int hw = hist[lane], hc = hist[64 + lane];                // lane l: the l-th bin from the top
    const int sw = weighted ? lc_wave_scan_incl(hw) : 0, sc = counted ? lc_wave_scan_incl(hc) : 0;
    const unsigned long long over = __ballot(sw > W || sc > C);
    if (over == 0ull) {
        *cut = lo - 1u;                                             // everything fits
        return true;
    }
    const int l = __ffsll((long long)over) - 1;                     // the prefix ends in this bin
    W -= lc_readlane(sw - hw, l);
    C -= counted ? lc_readlane(sc - hc, l) : 0;
    int in = 0;
    uint32_t top = 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const unsigned long long m = __ballot(bin[r] == l);
        if (m != 0ull) {                                            // (uniform)
            const int at = in + lc_mbcnt(m);
            if (bin[r] == l && at < 64) { hist[at] = 64 * r + lane; hist[64 + at] = (int)k[r]; hist[128 + at] = w[r]; }
            top = max(top, bin[r] == l ? k[r] : 0u);
            in += __popcll(m);
        }
    }
    if (in > 64) return false;
    __builtin_amdgcn_wave_barrier();
    *cut = lc_wave_max_uniform(top);                                // (at least one of the bin is not kept)
    // those of the bin ranked against each other: up to eight by a lane for each pair, more by a lane for each
    const int i = in <= 8 ? lane >> 3 : lane, at = min(i, in - 1);
    const int me = hist[at], mw = weighted ? hist[128 + at] : 0;
    const uint32_t mk = (uint32_t)hist[64 + at];
    int c_before = 0, w_before = 0;
    if (in <= 8) {
        const int o = min(lane & 7, in - 1);
        const uint32_t ok = (uint32_t)hist[64 + o];
        const bool before = (lane & 7) < in && (ok > mk || (ok == mk && o < at));
        c_before = before ? 1 : 0;
        w_before = before && weighted ? hist[128 + o] : 0;
        c_before += __builtin_amdgcn_update_dpp(0, c_before, 0xB1, 0xF, 0xF, true);
        w_before += __builtin_amdgcn_update_dpp(0, w_before, 0xB1, 0xF, 0xF, true);
        c_before += __builtin_amdgcn_update_dpp(0, c_before, 0x4E, 0xF, 0xF, true);
        w_before += __builtin_amdgcn_update_dpp(0, w_before, 0x4E, 0xF, 0xF, true);
        c_before += __builtin_amdgcn_update_dpp(0, c_before, 0x141, 0xF, 0xF, true);
        w_before += __builtin_amdgcn_update_dpp(0, w_before, 0x141, 0xF, 0xF, true);
    } else {
        for (int c = 0; c < in; ++c) {
            const uint32_t ok = (uint32_t)lc_readlane((int)mk, c);
            const bool before = ok > mk || (ok == mk && c < lane);
            c_before += before ? 1 : 0;
            w_before += before ? lc_readlane(mw, c) : 0;
        }
    }
    if (i < in) key[me] = c_before < C && w_before + mw <= W ? 0xffffffffu : 0u;      // (of a pair's eight lanes all write the same)
    return true;
}
// The longest prefix (key descending, position ascending) of at most C candidates, and if `weighted` of total weight
// <= W, of a list in LDS: candidate i is in it iff key[i] > the returned value; keys at the cut have been replaced by
// the highest value (in) or 0 (not).  64 bins over the range of the keys, a scan from the top for the bin in which
// the prefix ends, and that bin's candidates ranked against each other; a bin of more than 64 is split again.
// One wavefront's work: an instruction that all sixteen wavefronts of a workgroup execute costs their compute
// unit 16 cycles, so what one of them can do alone is not shared out (249 candidates ranked against each other by
// all wavefronts: 6 us; halving the key range: 3 us; here: 2 us).  `hist`: 192 ints of LDS.
__device__ __forceinline__ uint32_t lc_wave_cut(int n, uint32_t* key, const int* wgt, bool weighted, int W, int C, int* hist) {
    const int lane = threadIdx.x & 63;
    const bool counted = C < 0x7fffffff;
    auto four = [&](int i0, uint32_t (&k)[4]) LC_INLINE {           // candidates i0 + lane + 64 r; past the end: key 0
        const int last = n - 1;
        uint32_t x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = key[min(i0 + 64 * r + lane, last)];
#pragma unroll
        for (int r = 0; r < 4; ++r) k[r] = i0 + 64 * r + lane < n ? x[r] : 0u;
    };
    // candidates of a list position each, ranked against each other: kept ones get the highest key, the others 0
    auto rank = [&](int in, int me, uint32_t mine) LC_INLINE {
        const int w = weighted ? wgt[me] : 0;
        int c_before = 0, w_before = 0;
        for (int c = 0; c < in; ++c) {
            const uint32_t k = (uint32_t)lc_readlane((int)mine, c);
            const bool before = k > mine || (k == mine && c < lane);
            c_before += before ? 1 : 0;
            w_before += before ? lc_readlane(w, c) : 0;
        }
        if (lane < in) key[me] = mine != 0u && c_before < C && w_before + w <= W ? 0xffffffffu : 0u;
    };
    if (n <= C && !weighted) return 0u;
    if (n <= LC_BM_RANK_MAX) {                                      // (too few for the histogram to pay)
        const int me = min(lane, max(n - 1, 0));
        rank(n, me, key[me]);
        return 0u;
    }
    uint32_t cut;
    if (n <= 256 ? lc_wave_cut_held<4>(n, key, wgt, weighted, W, C, hist, &cut)
                 : n <= 512 && lc_wave_cut_held<8>(n, key, wgt, weighted, W, C, hist, &cut)) return cut;
    uint32_t lo = 0xffffffffu, hi = 0u;
    for (int i0 = 0; i0 < n; i0 += 256) {
        uint32_t k[4];
        four(i0, k);
#pragma unroll
        for (int r = 0; r < 4; ++r) { lo = min(lo, k[r] - 1u); hi = max(hi, k[r]); }      // (key 0 wraps to the largest value: ignored)
    }
    uint32_t a = lc_wave_min_uniform(lo) + 1u, b = lc_wave_max_uniform(hi);               // range that is still open
    LcKeyBins bins;
    bins.over(a, b, true);
    for (;;) {
        hist[lane] = 0;
        hist[64 + lane] = 0;
        for (int i0 = 0; i0 < n; i0 += 256) {
            uint32_t k[4];
            four(i0, k);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // (no branch around the additions: what is no candidate adds to a slot that nobody reads)
                const int bin = bins.of(k[r]), slot = bin >= 0 ? 63 - bin : 128 + lane;
                if (weighted) atomicAdd(&hist[slot], wgt[min(i0 + 64 * r + lane, n - 1)]);
                if (counted) atomicAdd(&hist[bin >= 0 ? slot + 64 : slot], 1);
            }
        }
        __builtin_amdgcn_wave_barrier();
        const int hw = hist[lane], hc = hist[64 + lane];            // lane l: bin 63 - l
        const int sw = weighted ? lc_wave_scan_incl(hw) : 0, sc = counted ? lc_wave_scan_incl(hc) : 0;
        const unsigned long long over = __ballot(sw > W || sc > C);
        if (over == 0ull) return a - 1u;                            // everything (that is open) fits
        const int l = __ffsll((long long)over) - 1;                 // the prefix ends in this lane's bin
        W -= lc_readlane(sw - hw, l);
        C -= counted ? lc_readlane(sc - hc, l) : 0;
        lo = 0xffffffffu;
        hi = 0u;
        int in = 0;
        for (int i0 = 0; i0 < n; i0 += 256) {
            uint32_t k[4];
            four(i0, k);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool here = bins.of(k[r]) == 63 - l;
                const unsigned long long m = __ballot(here);
                const int at = in + lc_mbcnt(m);
                if (here && at < 64) hist[at] = i0 + 64 * r + lane;
                in += __popcll(m);
                lo = min(lo, here ? k[r] : 0xffffffffu);
                hi = max(hi, here ? k[r] : 0u);
            }
        }
        if (in <= 64) {
            // few enough to rank: lane c has the c-th of them (in order of position)
            const int me = hist[min(lane, in - 1)];
            b = lc_wave_max_uniform(hi);                            // (at least one of them is not kept)
            rank(in, me, key[me]);
            return b;
        }
        a = lc_wave_min_uniform(lo);
        b = lc_wave_max_uniform(hi);
        if (a == b) {                                               // equal keys are cut in order
            for (int i0 = 0; i0 < n; i0 += 64) {
                const int i = i0 + lane;
                const bool tie = i < n && key[min(i, n - 1)] == b;
                const unsigned long long e = __ballot(tie);
                if (e == 0ull) continue;
                const int inc = lc_wave_scan_incl(tie && weighted ? wgt[i] : 0);
                const unsigned long long sel = __ballot(tie && inc <= W && lc_mbcnt(e) < C);
                if (tie) key[i] = ((sel >> lane) & 1ull) ? 0xffffffffu : 0u;
                W = sel == e ? W - lc_readlane(inc, 63) : -1;
                C -= __popcll(sel);
            }
            return b;
        }
        bins.over(a, b, false);
    }
}

// The same by a workgroup, for long lists (in LDS or in the workspace).  `sh`: 256 + 6 NT / 64 ints.  Begins behind a
// barrier and ends with one.
template <int NT>
__device__ __forceinline__ uint32_t lc_block_cut(int n, uint32_t* key, const int* wgt, bool weighted, int W, int C, int* sh) {
    constexpr int NW = NT / 64;
    static_assert(NW == 16, "a row of 16 lanes goes over the wavefronts' parts");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool counted = C < 0x7fffffff;
    int* const slots = sh + 256;
    uint32_t lo = 0xffffffffu, hi = 0u;
    int in = 0, turn = 0;
    for (int i = threadIdx.x; i < n; i += NT) { const uint32_t k = key[i]; lo = min(lo, k - 1u); hi = max(hi, k); }
    LcKeyBins bins;
    // lowest and highest key and number over the workgroup; the next histogram is emptied meanwhile
    auto exchange = [&]() LC_INLINE {
        lo = lc_wave_min_uniform(lo);
        hi = lc_wave_max_uniform(hi);
        in = lc_wave_sum_i(in);
        int* const s = slots + turn * 3 * NW;
        if (lane == 0) { s[wave] = (int)lo; s[NW + wave] = (int)hi; s[2 * NW + wave] = in; }
        if (threadIdx.x < 128) sh[turn * 128 + threadIdx.x] = 0;
        __syncthreads();
        lo = lc_wave_min_uniform((uint32_t)s[lane & 15]);
        hi = lc_wave_max_uniform((uint32_t)s[NW + (lane & 15)]);
        in = lc_readlane(lc_sum16_i(s[2 * NW + (lane & 15)]), 0);
    };
    exchange();
    uint32_t a = lo + 1u, b = hi;
    bins.over(a, b, true);
    for (;;) {
        int* const hist = sh + turn * 128;
        for (int i = threadIdx.x; i < n; i += NT) {
            const int bin = bins.of(key[i]);
            if (bin >= 0) {
                if (weighted) atomicAdd(&hist[63 - bin], wgt[i]);
                if (counted) atomicAdd(&hist[127 - bin], 1);
            }
        }
        __syncthreads();
        const int hw = hist[lane], hc = hist[64 + lane];
        const int sw = weighted ? lc_wave_scan_incl(hw) : 0, sc = counted ? lc_wave_scan_incl(hc) : 0;
        const unsigned long long over = __ballot(sw > W || sc > C);
        if (over == 0ull) {
            b = a - 1u;
            break;
        }
        const int l = __ffsll((long long)over) - 1;
        W -= lc_readlane(sw - hw, l);
        C -= counted ? lc_readlane(sc - hc, l) : 0;
        lo = 0xffffffffu;
        hi = 0u;
        in = 0;
        for (int i = threadIdx.x; i < n; i += NT) {
            const uint32_t k = key[i];
            if (bins.of(k) == 63 - l) { lo = min(lo, k); hi = max(hi, k); ++in; }
        }
        turn ^= 1;
        exchange();
        a = lo;
        b = hi;
        if (in == 1) break;
        if (a == b) {
            if (wave == 0) {
                for (int i0 = 0; i0 < n; i0 += 64) {
                    const int i = i0 + lane;
                    const bool tie = i < n && key[min(i, n - 1)] == b;
                    const unsigned long long e = __ballot(tie);
                    if (e == 0ull) continue;
                    const int inc = lc_wave_scan_incl(tie && weighted ? wgt[i] : 0);
                    const unsigned long long sel = __ballot(tie && inc <= W && lc_mbcnt(e) < C);
                    if (tie) key[i] = ((sel >> lane) & 1ull) ? 0xffffffffu : 0u;
                    W = sel == e ? W - lc_readlane(inc, 63) : -1;
                    C -= __popcll(sel);
                }
            }
            break;
        }
        bins.over(a, b, false);
    }
    __syncthreads();
    return b;
}

template <int G>
__global__ void __launch_bounds__(LC_BM_THREADS)
lc_beam_kernel(const LcBeamArgs a) {
    lc_fetch_args<sizeof(LcBeamArgs)>();
    extern __shared__ int lds_dyn[];
    __shared__ int cnt_sh[LC_BM_SPAN * LC_BM_WAVES];
    __shared__ int hist_sh[256 + 6 * LC_BM_WAVES];       // (of either cut)
    __shared__ uint32_t cut_sh;
    constexpr int STEP = 4 * LC_BM_GROUPS;               // four nodes per group of 16 lanes at a time

    const int h = blockIdx.x, b = blockIdx.y;
    const int bh = b * a.H + h;
    int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = tid & 15, grp = tid >> 4;
    const int L = a.L, bottom = L - 1;                   // levels are counted from the top here: 0 .. L - 1 (the chunks)
    const int cap0 = a.cap0;
    const size_t cb = (size_t)bh * cap0;
    const bool c0b = a.c0_bf16 != 0;
    const int* const n_lev = a.nlev + b * LC_MAX_LEVELS + (L - 1);      // nodes of level v: n_lev[-v]
    const int* const bnd = a.bounds + (size_t)b * (cap0 + 1);
    const int W = a.budget > 0 ? a.budget : 0;

    // candidate lists: ids of the current level, ids of the next, keys, weights; in LDS up to CL entries, in the
    // workspace beyond
    const int CL = a.list_slots;
    const LcBeamLayout ly = lc_beam_layout(CL);
    int* l_cid = lds_dyn + ly.cid / 4;
    int* l_nxt = lds_dyn + ly.nxt / 4;
    uint32_t* const l_key = reinterpret_cast<uint32_t*>(lds_dyn + ly.key / 4);
    int* const l_wgt = lds_dyn + ly.wgt / 4;
    // behind them: a mark for each node of a level that is kept, and parent pointers
    uint8_t* const kept = reinterpret_cast<uint8_t*>(lds_dyn + ly.total / 4);
    const int KW = a.kept_words;                         // (a multiple of four: what follows is read 16 bytes at a time)
    uint32_t* const kept_w = reinterpret_cast<uint32_t*>(kept);
    int* const l_par = lds_dyn + ly.total / 4 + KW;
    int* const gs = a.scratch + 4 * cb;
    int* g_cid = gs;
    int* g_nxt = gs + cap0;
    uint32_t* const g_key = reinterpret_cast<uint32_t*>(gs + 2 * cap0);
    int* const g_wgt = gs + 3 * cap0;

    // ---- Candidates base + 4 grp .. + 3 of a list: their centers; radius and two integers, whose difference is a node's
    // chunk count or a chunk's length, of number (sub & 3) of them (range-checked buffers: an address is one
    // register, rows past the end read 0).
    LcNodeFrag f[4];
    float R;
    int x0, x1, own;
    auto load = [&](const LcBeamLevel& v, bool chunks, int valid, const int (&id)[4]) LC_INLINE {
        const size_t at = (size_t)bh * v.cap;
        const bool half = chunks && c0b;
        const char* const base = reinterpret_cast<const char*>(v.center);
        const __amdgpu_buffer_rsrc_t cen_r = lc_buffer(base + at * (half ? 2 * LC_D : 4 * LC_D), v.cap * (half ? 2 * LC_D : 4 * LC_D));
        const __amdgpu_buffer_rsrc_t rad_r = lc_buffer(v.radius + at, v.cap * 4);
        const __amdgpu_buffer_rsrc_t end_r = chunks ? lc_buffer(bnd + 1, cap0 * 4) : lc_buffer(v.nchunk + at, v.cap * 4);
        const __amdgpu_buffer_rsrc_t beg_r = lc_buffer(bnd, chunks ? cap0 * 4 : 0);
        if (16 * wave >= valid) return;                  // (whole wavefronts: rows nobody needs would take the cache's time)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (half) {
                const lc_v2i x = __builtin_amdgcn_raw_buffer_load_b64(cen_r, id[k] * (LC_D * 2) + 8 * sub, 0, 0);
                const lc_v2i y = __builtin_amdgcn_raw_buffer_load_b64(cen_r, id[k] * (LC_D * 2) + 8 * sub + 128, 0, 0);
                f[k].a.x = __int_as_float(x.x); f[k].a.y = __int_as_float(x.y);
                f[k].b.x = __int_as_float(y.x); f[k].b.y = __int_as_float(y.y);
            } else {
                f[k].a = lc_buf_load_f32x4(cen_r, id[k] * (LC_D * 4) + 16 * sub);
                f[k].b = lc_buf_load_f32x4(cen_r, id[k] * (LC_D * 4) + 16 * sub + 256);
            }
        }
        R = lc_buf_load_f32(rad_r, own);
        x0 = lc_buf_load_i32(beg_r, own);
        x1 = lc_buf_load_i32(end_r, own);
    };
    own = 4 * grp + (sub & 3);
    {
        const int id[4] = {4 * grp, 4 * grp + 1, 4 * grp + 2, 4 * grp + 3};
        load(a.lev[0], L == 1, a.lev[0].cap, id);        // top level: every node is a candidate
    }
    // ---- parent pointers, those of level v at l_par + o: the levels from the top down as long as there is room
    auto parents_of = [&](const LcBeamLevel& v) LC_INLINE {
        return lc_buffer(v.parent ? v.parent + (size_t)bh * v.cap : nullptr, v.parent ? v.cap * 4 : 0);     // (none: reads return 0)
    };
    // (They go out when the query has come, and with it the top level's rows, in wavefronts that do not cut: together with the rows, on one compute unit's
    // way to memory, they kept the last wavefront's rows waiting 1.2 us.  From within the loop over the levels it was 1 to 3 % slower, most with long
    // lists: 8 heads of group size 7 with 9.6 K candidates 180 us, here 174.)
    auto fetch_parents = [&]() LC_INLINE {
        constexpr int FIRST = LC_BM_WAVES / 4;
        if (wave < FIRST) return;
        int at = 0;                                      // LDS words taken
        for (int v = 1; v < L; ++v) {
            const int words = a.lev[v].par_words;
            if (at + words <= a.par_slots) {
                const __amdgpu_buffer_rsrc_t r = parents_of(a.lev[v]);
                for (int w = 256 * (wave - FIRST); w < words; w += 256 * (LC_BM_WAVES - FIRST))
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(l_par + at + w), 16, 16 * lane, 4 * w, 0, 0);
                at += words;
            }
        }
    };
    int next_par = 0;                                    // LDS words of the levels before
    // (scalar reads that would otherwise wait for their own round trip further down)
    const int M = min(a.state[bh * 4 + 1], cap0);
    int n_c = L > 1 ? n_lev[0] : (W > 0 ? M : 0), n_dn = L > 1 ? n_lev[-1] : 0;
    asm volatile("" :: "s"(M), "s"(n_c), "s"(n_dn));
    uint32_t qp[G][4];
    float qn[G];
    lc_load_query_packed<G>(a.q + (size_t)b * a.H * G * LC_D, h, sub, qp, qn);
    fetch_parents();

    for (int i = tid; i < KW; i += LC_BM_THREADS) kept_w[i] = 0u;
    // optional score output: everything that is never scored reads -inf
    float* const scores = a.scores ? a.scores + cb : nullptr;
    if (scores) {
        for (int j = tid; j < M; j += LC_BM_THREADS) scores[j] = LC_NEG_INF;
        __syncthreads();
    }
    // pinned chunks (first token below `sink`) are the leading ones: their number, counted by every wavefront
    int n_pin = 0;
    if (a.sink > 0)
        for (;;) {
            const int j = n_pin + lane;
            const int c = __popcll(__ballot(j < M && bnd[min(j, cap0)] < a.sink));
            n_pin += c;
            if (c < 64) break;
        }

    // ---- Items i < n that `in(i)` accepts (bits of four of them from i on), in ascending order, through put(i, position):
    // a wavefront takes 256 consecutive items of every 4096, a lane four of them; a scan of the lanes' counts
    // and one exchange of the wavefronts' give the places.
    auto gather = [&](int n, auto in, auto put) LC_INLINE -> int {
        int total = 0;
        for (int s0 = 0; s0 < n; s0 += LC_BM_SPAN * 4 * LC_BM_THREADS) {     // (once, nearly always)
            unsigned mask = 0u;
            const int blocks = min(LC_BM_SPAN, (n - s0 + 4 * LC_BM_THREADS - 1) / (4 * LC_BM_THREADS));
            for (int e = 0; e < blocks; ++e) {
                const int first = s0 + (e * LC_BM_WAVES + wave) * 256;
                int c = 0;
                if (first < n) {                                    // (whole wavefronts)
                    const int i = first + 4 * lane;
                    const unsigned q = in(i) & ((1u << min(max(n - i, 0), 4)) - 1u);
                    mask |= q << (4 * e);
                    c = lc_wave_sum_i(__popc(q));
                }
                if (lane == 0) cnt_sh[e * LC_BM_WAVES + wave] = c;
            }
            lc_barrier_lds();
            for (int e = 0; e < blocks; ++e) {
                const int c = cnt_sh[e * LC_BM_WAVES + (lane & 15)];
                const int inc = lc_wave_scan_incl((lane < 16) ? c : 0);
                static_assert(LC_BM_WAVES == 16, "one count per lane of a row");
                unsigned q = (mask >> (4 * e)) & 15u;
                if (__ballot(q != 0u) != 0ull) {
                    const int mine = __popc(q);
                    int at = total + lc_readlane(inc - c, wave) + lc_wave_scan_incl(mine) - mine;
                    const int i = s0 + (e * LC_BM_WAVES + wave) * 256 + 4 * lane;
                    while (q != 0u) {                               // (one or two of four, mostly)
                        put(i + __ffs((int)q) - 1, at++);
                        q &= q - 1u;
                    }
                }
                total += lc_readlane(inc, 15);
            }
            if (s0 + LC_BM_SPAN * 4 * LC_BM_THREADS < n) lc_barrier_lds();      // the counts are written anew
        }
        return total;
    };

    // ---- All levels run through this one loop, NB x 64 candidates at a time: the code of a level is fetched
    // once and found in the instruction cache by the levels after it.
    int v = 0, base = 0, n_sel = 0, n_own = n_c;                      // (uniform: what depends on them stays in scalar registers)
    bool in_lds = n_c <= CL;
    if (n_c > STEP || L == 1) {                          // (the first STEP are on their way)
        for (int i = tid; i < n_c; i += LC_BM_THREADS) {
            if (i < CL) l_cid[i] = i;
            if (!in_lds) g_cid[i] = i;
        }
        if (in_lds) lc_barrier_lds();                    // other wavefronts read what this one wrote from the second STEP on
        else __syncthreads();
    }
    int32_t* const ids = a.ids + (size_t)bh * a.cap;
    int C = a.lev[0].beam, par_words = a.lev[1].par_words, n_next = L > 2 ? n_lev[-2] : 0;
    for (;;) {
        const bool last = v == bottom;
        // (what is derived from the thread's number is worked out anew where it is needed: hoisted out of this
        // loop, as the compiler would, it fills the registers)
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63, sub = tid & 15, grp = tid >> 4;
        if (base + 16 * wave < n_c) {                               // (whole wavefronts)
            if (last && c0b) {
#pragma unroll
                for (int k = 0; k < 4; ++k) f[k] = lc_widen_chunk_frag(f[k]);
            }
            const float sc = lc_score_packed<G, 4>(f, R, sub, qp, qn);
            const int i = base + 4 * grp + (sub & 3);
            const int w = max(x1 - x0, 0);
            uint32_t key = lc_score_key(sc);
            if (key == 0xffffffffu) key = 0xfffffffeu;             // (the highest value marks chosen equal keys)
            if (last ? own < n_pin : w == 0) key = 0u;              // pinned chunks and empty nodes are no candidates
            if ((sub >> 2) == 1 && i < n_c) {
                if (in_lds) { l_key[i] = key; l_wgt[i] = w; }
                else { g_key[i] = key; g_wgt[i] = w; }
                if (last && scores && key != 0u) scores[own] = sc;
            }
        }
        base += STEP;
        if (base >= n_c) {
            // ---- the level is scored: keep the beam's best (at the chunks: what the budget holds as well)
            if (in_lds) lc_barrier_lds();
            else __syncthreads();
            C = C > 0 ? C : 0x7fffffff;
            const int n_up = n_own;
            if (v + 1 == bottom) n_dn = W > 0 ? M : 0;
            auto mark = [&](int node) LC_INLINE { kept[node] = 1; };
            if (n_c <= LC_BM_CUT_MAX) {
                if (wave == 0) {
                    const uint32_t b = lc_wave_cut(n_c, l_key, l_wgt, last, W, C, hist_sh);
                    if (tid == 0) cut_sh = b;
                }
                lc_barrier_lds();
                const uint32_t b = cut_sh;
                if (!last) {
                    if (tid < n_c && l_key[tid] > b) mark(v == 0 ? tid : l_cid[tid]);
                } else if (64 * wave < n_c || wave == 0) {
                    int at = n_pin;
                    n_sel = 0;
                    for (int i0 = 0; i0 < n_c; i0 += 64) {          // (the wavefronts before this one: their number alone)
                        const bool keep = i0 + lane < n_c && l_key[i0 + lane] > b;
                        const unsigned long long m = __ballot(keep);
                        if (i0 == 64 * wave) {
                            at += n_sel + lc_mbcnt(m);
                            if (keep && at < a.cap) ids[at] = l_cid[i0 + lane];
                        }
                        n_sel += __popcll(m);
                    }
                }
            } else {
                // a longer list (generic pointers: LDS or workspace)
                uint32_t* const key = in_lds ? l_key : g_key;
                const int* const wgt = in_lds ? l_wgt : g_wgt;
                const int* const cid = in_lds ? l_cid : g_cid;
                const uint32_t b = lc_block_cut<LC_BM_THREADS>(n_c, key, wgt, last, W, C, hist_sh);
                if (!last) {
                    for (int i = tid; i < n_c; i += LC_BM_THREADS)
                        if (key[i] > b) mark(v == 0 ? i : cid[i]);
                } else {
                    n_sel = gather(n_c, [&](int i) LC_INLINE -> unsigned {
                        unsigned q = 0u;
#pragma unroll
                        for (int k = 0; k < 4; ++k) q |= key[min(i + k, n_c - 1)] > b ? 1u << k : 0u;
                        return q;
                    }, [&](int i, int at) LC_INLINE { if (n_pin + at < a.cap) ids[n_pin + at] = cid[i]; });
                }
            }
            if (last) break;
            if (v == 0) __builtin_amdgcn_s_waitcnt(0);              // (this wavefront's share of the parent pointers)
            lc_barrier_lds();
            // ---- the kept nodes' children are the next level's candidates: a list in LDS as far as it fits, in
            // the workspace too if there may be more of them
            ++v;
            const LcBeamLevel& lev = a.lev[v];
            const bool both = n_dn > CL;
            auto kept_of = [&](int p) LC_INLINE -> unsigned { return kept[min((unsigned)p, (unsigned)n_up)]; };     // (no node n_up: 0)
            auto put = [&](int i, int at) LC_INLINE {
                if (at < CL) l_nxt[at] = i;
                if (both) g_nxt[at] = i;
            };
            const int o = next_par;
            const bool here = o + par_words <= a.par_slots;
            if (here) next_par += par_words;
            if (here && n_dn <= par_words) {
                n_c = gather(n_dn, [&](int i) LC_INLINE -> unsigned {
                    const int4 p = *reinterpret_cast<const int4*>(l_par + o + i);      // (past n: other words of the LDS)
                    return kept_of(p.x) | kept_of(p.y) << 1 | kept_of(p.z) << 2 | kept_of(p.w) << 3;
                }, put);
            } else {
                const __amdgpu_buffer_rsrc_t r = parents_of(lev);
                n_c = gather(n_dn, [&](int i) LC_INLINE -> unsigned {
                    int p[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) p[k] = lc_buf_load_i32(r, i + k);
                    return kept_of(p[0]) | kept_of(p[1]) << 1 | kept_of(p[2]) << 2 | kept_of(p[3]) << 3;
                }, put);
            }
            int* const tl = l_cid; l_cid = l_nxt; l_nxt = tl;
            int* const tg = g_cid; g_cid = g_nxt; g_nxt = tg;
            in_lds = n_c <= CL;
            if (in_lds) lc_barrier_lds();
            else __syncthreads();
            for (int i = tid; i < KW; i += LC_BM_THREADS) kept_w[i] = 0u;
            base = 0;
            n_own = n_dn;
            n_dn = n_next;
            // (what the end of the next level needs)
            C = a.lev[v].beam;
            par_words = a.lev[min(v + 1, LC_MAX_LEVELS - 1)].par_words;
            n_next = v + 2 < L ? n_lev[-v - 2] : 0;
        }
        // (entries past the list's end hold anything: their rows' scores are dropped)
        int id[4];
        if (in_lds) {
            const int4 x = *reinterpret_cast<const int4*>(l_cid + base + 4 * grp);
            id[0] = x.x; id[1] = x.y; id[2] = x.z; id[3] = x.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) id[k] = g_cid[min(base + 4 * grp + k, n_c - 1)];
        }
        own = (sub & 2) ? ((sub & 1) ? id[3] : id[2]) : ((sub & 1) ? id[1] : id[0]);
        load(a.lev[v], v == bottom, n_c - base, id);
    }
    for (int j = tid; j < min(n_pin, a.cap); j += LC_BM_THREADS) ids[j] = j;
    if (tid == 0) a.counts[bh] = min(n_pin + n_sel, a.cap);
}

template <int G>
static int launch_beam_g(const LcRetrieveArgs& r, int max_M, int max_nodes, hipStream_t stream) {
    const LcDev& ix = r.ix;
    LcBeamArgs a = {};
    const int L = ix.L;
    int want = 0;
    for (int l = 0; l < L; ++l) {
        LcBeamLevel& v = a.lev[L - 1 - l];
        v.center = ix.center[l];
        v.radius = ix.radius[l];
        v.nchunk = l > 0 ? ix.nchunk[l] : nullptr;
        v.parent = l + 1 < L ? ix.parent[l] : nullptr;
        v.cap = ix.cap[l];
        v.beam = r.beam[l];
        v.par_words = l + 1 < L ? ((l == 0 ? max_M : ix.cap[l]) + 255) / 256 * 256 : 0;
        want += v.par_words;
    }
    a.q = r.q;
    a.bounds = ix.bounds;
    a.state = ix.state;
    a.nlev = ix.nlev;
    a.scores = r.scores;
    a.ids = r.ids;
    a.counts = r.counts;
    a.scratch = r.scratch;
    a.H = ix.H;
    a.L = L;
    a.cap0 = ix.cap[0];
    a.cap = r.cap;
    a.budget = r.budget;
    a.sink = r.sink;
    a.c0_bf16 = ix.c0_bf16;
    // LDS: lists for up to LC_BEAM_LIST_MAX candidates per level (more go to the workspace), marks of the kept
    // nodes, and as many parent pointers as fit beside them
    a.list_slots = lc_beam_list_slots(max_nodes);
    const int most = L > 1 ? (ix.cap[1] < LC_BM_MAX_LEVEL_NODES ? ix.cap[1] : LC_BM_MAX_LEVEL_NODES) : 0;
    a.kept_words = (most + 16) / 16 * 4;                             // (one more than there are nodes)
    const int lists = lc_beam_layout(a.list_slots).total + 4 * a.kept_words;
    const int room = (LC_WALK_LDS_LIMIT - LC_BM_STATIC_LDS - lists) / 4;
    a.par_slots = want < room ? want : (room > 0 ? room : 0);
    const size_t lds = (size_t)lists + 4 * (size_t)a.par_slots;
    if (lds + LC_BM_STATIC_LDS > 48 * 1024)
        LC_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&lc_beam_kernel<G>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(lc_beam_kernel<G>, dim3(ix.H, ix.B), dim3(LC_BM_THREADS), lds, stream, a);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}

// lc_leaf_kernel runs 1024 threads = 64 groups: one chunk per group while scoring; the last workgroup
// has enough threads to hold a few keys each during the select.
#define LC_LF_THREADS 1024
#define LC_LF_GROUPS (LC_LF_THREADS / 16)

// ---------------------------------------------------------------------------------
// lc_leaf_kernel: chunk scoring + budget selection by the last workgroup
// ---------------------------------------------------------------------------------
// BF16: how the chunk-level centers are stored (a compile-time copy of the index's flag).
template <int G, int R, bool BF16>
__global__ void __launch_bounds__(LC_LF_THREADS)
lc_leaf_kernel(const LcRetrieveArgs a) {
    lc_fetch_args<sizeof(LcRetrieveArgs)>();
    extern __shared__ int lds_dyn[];
    __shared__ LcLeafSelSh sel_sh;
    __shared__ int last_sh;

    const LcDev& ix = a.ix;
    const int h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    const int tid = threadIdx.x;
    const int sub = tid & 15, grp = tid >> 4;
    const size_t cb = (size_t)bh * ix.cap[0];
    constexpr bool c0b = BF16;
    const int cap0 = ix.cap[0];
    const int* bnd = ix.bounds + (size_t)b * (cap0 + 1);
    uint32_t* keys = a.keys + cb;
    float* scores = a.scores ? a.scores + cb : nullptr;
    // the per-chunk arrays of the scoring part through range-checked buffer resources (an index
    // derived from stored values -- a parent pointer -- cannot reach memory outside its array)
    const __amdgpu_buffer_rsrc_t bnd_r = lc_buffer(bnd, (cap0 + 1) * 4);
    const __amdgpu_buffer_rsrc_t want_r = lc_buffer(a.want + cb, cap0);
    const __amdgpu_buffer_rsrc_t par_r = lc_buffer(ix.parent[0] + cb, cap0 * 4);
    const __amdgpu_buffer_rsrc_t rad_r = lc_buffer(ix.radius[0] + cb, cap0 * 4);
    const bool have_want = a.walk != 0;

    // loads that do not depend on M are issued together with it (the arrays are cap0 long)
    const int j_lo = blockIdx.x * (R * LC_LF_GROUPS);
    int jj[R];
    int wv[R];
    float rv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = min(j_lo + r * LC_LF_GROUPS + grp, cap0 - 1);
        jj[r] = j;
        // (rows past the chunk count hold whatever the buffer held: the result is unused)
        wv[r] = (lc_buf_load_i32(bnd_r, j) >= a.sink ? 1 : 0) & (have_want ? lc_buf_load_u8(want_r, lc_buf_load_i32(par_r, j)) : 1);
        rv[r] = lc_buf_load_f32(rad_r, j);
    }
    // Without a level walk every chunk below M is scored, so its center can be fetched right away
    // instead of one memory round trip later (with a walk the centers of pruned chunks are the
    // traffic the walk exists to save, so there the load waits for the verdict).
    constexpr bool kSpec = R <= 2 || (R == 4 && G <= 7);      // as far as the registers of a 1024-thread workgroup go
    LcNodeFrag pre[kSpec ? R : 1];
    if (kSpec && !have_want) {
#pragma unroll
        for (int r = 0; r < (kSpec ? R : 1); ++r) pre[r] = lc_load_chunk_node(ix.center[0], c0b, cb + jj[r], sub);
    }
    // (group size 7 with four speculative centers per group: the query stays packed, see lc_upper_kernel)
    constexpr bool QP = kSpec && R == 4 && G >= 7;
    float qf[QP ? 1 : G][8], qn[G];
    uint32_t qp[QP ? G : 1][4];
    if constexpr (QP) lc_load_query_packed<G>(a.q + (size_t)b * ix.H * G * LC_D, h, sub, qp, qn);
    else lc_load_query_frags<G>(a.q + (size_t)b * ix.H * G * LC_D, h, sub, qf, qn);
    auto score_chunk = [&](const LcNodeFrag& raw, float Rv) -> float {
        if constexpr (QP) return lc_score_frag_packed<G>(c0b ? lc_widen_chunk_frag(raw) : raw, Rv, qp, qn);
        else return lc_score_chunk_frag<G>(raw, c0b, Rv, qf, qn);
    };
    const int M = ix.state[bh * 4 + 1];

    if (j_lo < M) {
        if (a.budget > 0) {
            float sv[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int j = j_lo + r * LC_LF_GROUPS + grp;
                sv[r] = LC_NEG_INF;
                if (j < M && wv[r]) {
                    if (kSpec && !have_want) sv[r] = score_chunk(pre[kSpec ? r : 0], rv[r]);
                    else sv[r] = score_chunk(lc_load_chunk_node(ix.center[0], c0b, cb + jj[r], sub), rv[r]);
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int j = j_lo + r * LC_LF_GROUPS + grp;
                if (j < M && sub == 0) {
                    lc_store_agent(&keys[j], lc_score_key(sv[r]));
                    if (scores) scores[j] = sv[r];
                }
            }
        } else {
            for (int j = j_lo + tid; j < min(M, j_lo + (R * LC_LF_GROUPS)); j += LC_LF_THREADS) {
                lc_store_agent(&keys[j], 0u);
                if (scores) scores[j] = LC_NEG_INF;
            }
        }
    }

    // ---- last workgroup of this (sequence, head) selects
    // (every workgroup empties its select histogram on the way: whichever turns out to be the last
    // finds it ready behind the barriers of the arrival)
    lc_leaf_select_prepare<LC_LF_THREADS>(sel_sh);
    if (!lc_arrive_last(&ix.sync[bh * 4 + 0], (int)gridDim.x, &last_sh)) return;

    // stage keys and lengths (pinned chunks get length -1) in LDS, or fall back to global scratch
    uint32_t* skey;
    int* slen;
    if (a.chunk_cap > 0) {
        skey = reinterpret_cast<uint32_t*>(lds_dyn);
        slen = lds_dyn + a.chunk_cap;
    } else {
        int* g = a.scratch + (size_t)bh * 4 * ix.cap[0];
        skey = reinterpret_cast<uint32_t*>(g);
        slen = g + ix.cap[0];
    }
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    // (batches of eight chunks per thread, all their loads in flight together: a memory round trip
    // per batch instead of one per chunk)
    constexpr int SB = 8;
    for (int j0 = tid; j0 < M; j0 += SB * LC_LF_THREADS) {
        int s0[SB], s1[SB];
        uint32_t kv[SB];
#pragma unroll
        for (int e = 0; e < SB; ++e) {
            const int j = min(j0 + e * LC_LF_THREADS, M - 1);
            s0[e] = bnd[j];
            s1[e] = bnd[j + 1];
            kv[e] = lc_load_agent(&keys[j]);
        }
#pragma unroll
        for (int e = 0; e < SB; ++e) {
            const int j = j0 + e * LC_LF_THREADS;
            if (j < M) {
                skey[j] = kv[e];
                slen[j] = (s0[e] < a.sink) ? -1 : (s1[e] - s0[e]);
                if (kv[e] != 0u) { kmin = min(kmin, kv[e]); kmax = max(kmax, kv[e]); }
            }
        }
    }
    lc_leaf_select_range(kmin, kmax, sel_sh);
    __syncthreads();

    const long long C = (a.policy == LC_POLICY_BEAM && a.beam[0] > 0) ? a.beam[0] : 0x7fffffffLL;
    const uint32_t thr = lc_leaf_select<LC_LF_THREADS>(M, skey, slen, a.budget > 0 ? (long long)a.budget : 0LL, C,
                                                       sel_sh);

    // each thread owns a contiguous run of chunks, so the ids come out ascending: count, scan, write
    int E = (M + LC_LF_THREADS - 1) / LC_LF_THREADS;
    E |= 1;                                             // odd stride: no LDS bank conflicts
    const int lo = min(M, tid * E), hi = min(M, lo + E);
    // (the verdicts of up to 64 chunks stay in a register mask; longer runs read LDS again)
    unsigned long long mask = 0ull;
    int my_sel = 0;
    for (int i = lo; i < hi; ++i) {
        const bool sel = slen[i] < 0 || skey[i] > thr;
        if (sel && i - lo < 64) mask |= 1ull << (i - lo);
        my_sel += sel ? 1 : 0;
    }
    int tot_s;
    int pos = lc_block_scan<LC_LF_THREADS>(my_sel, sel_sh.scan, &tot_s);
    int32_t* ids = a.ids + (size_t)bh * a.cap;
    while (mask) {
        const int k = __ffsll((long long)mask) - 1;
        mask &= mask - 1ull;
        if (pos < a.cap) ids[pos] = lo + k;
        ++pos;
    }
    for (int i = lo + 64; i < hi; ++i) {
        if (slen[i] < 0 || skey[i] > thr) {
            if (pos < a.cap) ids[pos] = i;
            ++pos;
        }
    }
    if (tid == 0) {
        a.counts[bh] = min(tot_s, a.cap);
        ix.sync[bh * 4 + 0] = 0;                 // ready for the next call
    }
}

// ---------------------------------------------------------------------------------
// launcher
// ---------------------------------------------------------------------------------
// ---------------------------------------------------------------------------------
// lc_score_kernel: chunk scoring only (the second kernel selects by itself)
// ---------------------------------------------------------------------------------
// The same scoring as lc_leaf_kernel without the selection behind it, so without its LDS and its
// 1024-thread workgroups: NT threads = NT/16 groups, R chunks per group.
#define LC_SC_THREADS 256
#define LC_SCORE_MAX_WGS 1024          // measured flat between 512 and 2048 workgroups
// Two chunks per group longer where the centers are float32: four of them are twice the registers of bfloat16 ones, one wavefront
// less per SIMD (lc_retrieve on 8 heads of 10.9 K chunks at 2731 workgroups 17.1 us, at 1366 18.3; on 64 pairs of 910 at 1856 workgroups
// 14.4 and 14.9, with bfloat16 centers 13.9 and 13.1; of 3276 at 6592 34.5 and 32.8).
#define LC_SCORE_MAX_WGS_F32 4096
// A group's R chunks are scored together, each head's query words widened once for them and the sums over lanes shared (lc_score_packed); they were
// scored one after the other, with the query's norms worked out by every group when the centers had come.  What bounds it is the centers' way from
// memory where they are float32, and arithmetic at group size 7.  us of lc_retrieve and lc_sparse_decode, before and now: 8 heads of 1820 chunks at group
// size 4 17.0 and 16.7, 16 pairs of 1820 at size 1 and of 7 queries 19.4 and 19.1, 22.5 and 21.8, 8 heads of 10.9 K float32 25.4 and 25.4, bfloat16 25.3 and 24.9;
// a step over 2 x 4 x 4.2 K at group size 7 21.3 and 20.8.  With the query's loads behind the centers' it was slower than before (25.8 for 25.5).
// BF16: how the chunk-level centers are stored (a compile-time copy of the index's flag).
template <int G, int R, bool BF16>
__global__ void __launch_bounds__(LC_SC_THREADS)
lc_score_kernel(const LcRetrieveArgs a) {
    lc_fetch_args<sizeof(LcRetrieveArgs)>();
    constexpr int PER = R * (LC_SC_THREADS / 16);
    constexpr int ROW = BF16 ? LC_D * 2 : LC_D * 4;
    const LcDev& ix = a.ix;
    const int h = blockIdx.y, b = blockIdx.z;
    const int bh = b * ix.H + h;
    const int tid = threadIdx.x;
    const int sub = tid & 15, grp = tid >> 4;
    const size_t cb = (size_t)bh * ix.cap[0];
    const int cap0 = ix.cap[0];
    const int j_lo = blockIdx.x * PER;
    // the per-chunk arrays through range-checked buffer resources (an index derived from stored
    // values -- a parent pointer -- cannot reach memory outside its array)
    const __amdgpu_buffer_rsrc_t bnd_r = lc_buffer(ix.bounds + (size_t)b * (cap0 + 1), (cap0 + 1) * 4);
    const __amdgpu_buffer_rsrc_t ent_r = lc_buffer(a.scratch + 4 * cb, cap0 * 16);
    const __amdgpu_buffer_rsrc_t want_r = lc_buffer(a.want + cb, cap0);
    const __amdgpu_buffer_rsrc_t par_r = lc_buffer(ix.parent[0] + cb, cap0 * 4);
    const __amdgpu_buffer_rsrc_t rad_r = lc_buffer(ix.radius[0] + cb, cap0 * 4);
    const int rows = max(0, min(cap0 - j_lo, PER));                 // (of this workgroup)
    const __amdgpu_buffer_rsrc_t cen_r = lc_buffer(reinterpret_cast<const char*>(ix.center[0]) + (cb + min(j_lo, cap0)) * ROW, rows * ROW);
    const bool have_want = a.walk != 0;
    // group `grp` has chunks j_lo + R grp + (0 .. R - 1), lane `sub` of it boundaries and radius of number sub mod R
    // (rows past the chunk count hold whatever the buffer held, past the array's end zero: the result is unused)
    const int own = j_lo + R * grp + (sub & (R - 1));
    int st = 0, en = 0;
    float rv = 0.f;
    unsigned wanted = (1u << R) - 1u;
    LcNodeFrag f[4];
    uint32_t qp[G][4];
    float qn[G];
    lc_load_query_packed<G>(a.q + (size_t)b * ix.H * G * LC_D, h, sub, qp, qn, [&]() LC_INLINE {
        __builtin_amdgcn_sched_barrier(0);
        st = lc_buf_load_i32(bnd_r, own);
        en = lc_buf_load_i32(bnd_r, own + 1);
        rv = lc_buf_load_f32(rad_r, own);
        if (have_want) {
            const bool w = lc_buf_load_u8(want_r, lc_buf_load_i32(par_r, own)) != 0;
            wanted = (unsigned)(__ballot(w) >> (tid & 48)) & 0xffffu;
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int at = ((wanted >> k) & 1u) ? R * grp + k : rows;   // (nothing is fetched from `rows` on)
            if (BF16) {
                const lc_v2i x = __builtin_amdgcn_raw_buffer_load_b64(cen_r, at * ROW + 8 * sub, 0, 0);
                const lc_v2i y = __builtin_amdgcn_raw_buffer_load_b64(cen_r, at * ROW + 8 * sub + 128, 0, 0);
                f[k].a = make_float4(__int_as_float(x.x), __int_as_float(x.y), 0.f, 0.f);
                f[k].b = make_float4(__int_as_float(y.x), __int_as_float(y.y), 0.f, 0.f);
            } else {
                f[k].a = lc_buf_load_f32x4(cen_r, at * ROW + 16 * sub);
                f[k].b = lc_buf_load_f32x4(cen_r, at * ROW + 16 * sub + 256);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    });
    const int M = ix.state[bh * 4 + 1];
    if (j_lo >= M) return;
    if (BF16) {
#pragma unroll
        for (int k = 0; k < R; ++k) f[k] = lc_widen_chunk_frag(f[k]);
    }
    const float sc = lc_score_packed<G, R>(f, rv, sub, qp, qn);
    if ((sub >> 2) == 1 && (sub & 3) < R && own < M) {              // one 16-byte entry per chunk (LcChunkEntry)
        const float sv = a.budget > 0 && st >= a.sink && ((wanted >> (sub & 3)) & 1u) ? sc : LC_NEG_INF;
        if (a.scores) a.scores[cb + own] = sv;
        lc_v4i w;
        w.x = (int)lc_score_key(sv);
        w.y = st;
        w.z = max(0, en - st);
        w.w = 0;
        __builtin_amdgcn_raw_buffer_store_b128(w, ent_r, own * 16, 0, 0);
    }
}


// ---------------------------------------------------------------------------------
// lc_select_kernel: the chunk list from the entries, one workgroup per (sequence, head)
// ---------------------------------------------------------------------------------
// The selection of lc_select_chunks for a caller that wants the ids: wavefront w owns chunks [64 EC w, 64 EC (w + 1)), lane l of it
// (EC w + e) 64 + l, everything stays in registers -- a bit per chunk says whether it is selected -- and the ids go out by
// one exchange of the wavefronts' counts.  What bounds it is one compute unit's instruction rate, some 20 instructions per chunk and lane,
// and one cold round trip.  As a kernel of its own behind lc_score_kernel it costs a launch, and saves the arrival of all scoring
// workgroups at one counter, keys staged in LDS and two passes over them: lc_retrieve on 8 heads of 10.9 K chunks 21.2 us as one
// kernel (lc_leaf_kernel), 17.4 as two; of 2299 11.5 and 9.3; of 500 9.2 and 7.4.
// Where the budget ends among the bulk of the chunks, the cutoff bin holds tens or hundreds of them.  The wavefronts share their ranking and take
// up to LC_SL_CAND of them: with 64, ranked by every wavefront (four of them on each SIMD) and all beyond left to the general routine, half of
// the tokens as the budget cost 12.1 us at 8 heads of 1000 chunks, now 8.0; at 11 K 30.9, now 19.7; at 64 x 500 11.7, now 9.5 (one kernel: 8.8); and a
// twelfth at 11 K 19.1, now 17.5.
#define LC_SL_THREADS 1024
#define LC_SL_CAND 256            // chunks of the cutoff bin that are ranked directly
#define LC_SL_FEW 4               // by every wavefront for itself
#define LC_SL_EC_MAX 12
struct LcSelectArgs {
    const int* entries;      // [B][H][cap0] LcChunkEntry
    const int* state;
    int32_t* ids;
    int32_t* counts;
    int cap0, cap, budget, sink;
};
template <int EC>
__global__ void __launch_bounds__(LC_SL_THREADS)
lc_select_kernel(const LcSelectArgs a) {
    constexpr int NT = LC_SL_THREADS, NW = NT / 64;
    constexpr int BITS = EC == 1 ? 8 : (EC == 2 ? 9 : 10);
    constexpr int BINS = 1 << BITS;
    extern __shared__ __attribute__((aligned(16))) int lds_dyn[];   // crowded cutoff bin: keys and lengths
    __shared__ __attribute__((aligned(16))) int hist[BINS];
    __shared__ int4 cand[LC_SL_CAND];
    __shared__ int ahead[LC_SL_CAND];                               // length of the chunks of the list that come before this one
    __shared__ uint32_t range[2 * NW];
    __shared__ int number[NW], n_cand;
    __shared__ LcLeafSelSh sel_sh;
    const int bh = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const __amdgpu_buffer_rsrc_t ent_r = lc_buffer(a.entries + (size_t)bh * 4 * a.cap0, a.cap0 * 16);
    const int j0 = wave * (EC * 64) + lane;                         // this lane's chunk e is j0 + 64 e
    uint32_t ck[EC];
    int len[EC], bin[EC];
    int T;
    {
        lc_v4i ent[EC];
#pragma unroll
        for (int e = 0; e < EC; ++e) ent[e] = __builtin_amdgcn_raw_buffer_load_b128(ent_r, j0 * 16, e * 1024, 0);
        for (int i = tid; i < BINS; i += NT) hist[i] = 0;
        if (tid < LC_SL_CAND) ahead[tid] = 0;
        if (tid == 0) n_cand = 0;
        T = a.state[bh * 4 + 0];
        const int M = a.state[bh * 4 + 1];
#pragma unroll
        for (int e = 0; e < EC; ++e) {
            const bool in = j0 + 64 * e < M;
            ck[e] = in ? (uint32_t)ent[e].x : 0u;
            len[e] = ent[e].z;
            bin[e] = in && ent[e].y < a.sink ? BINS : -1;           // pinned chunks: as if in a bin above all
        }
    }
    const int W = a.budget > 0 ? a.budget : 0;
    uint32_t kmin1 = 0xffffffffu, kmax = 0u;                        // (lowest candidate key) - 1, highest
#pragma unroll
    for (int e = 0; e < EC; ++e) { kmin1 = min(kmin1, ck[e] - 1u); kmax = max(kmax, ck[e]); }       // (key 0 wraps: ignored)
    kmin1 = lc_wave_min_uniform(kmin1);
    kmax = lc_wave_max_uniform(kmax);
    if (lane == 0) { range[wave] = kmin1; range[NW + wave] = kmax; }
    lc_barrier_lds();
    static_assert(NW == 16, "a row of 16 lanes goes over the wavefronts' parts");
    const uint32_t kmin = lc_wave_min_uniform(range[lane & 15]) + 1u;
    kmax = lc_wave_max_uniform(range[NW + (lane & 15)]);
    // ---- Histogram of chunk lengths over the upper half of the scores' range: the budget nearly always ends there, few chunks are in it (LDS
    // atomics of all of them, most in the same few bins, are the longest step otherwise), and its bins are finer.  Over all of the
    // range if the upper half fits the budget whole, and at once if the budget is a third of the tokens or more (then the upper half rarely
    // goes beyond it: whole range first against half first, 0.90 to 0.97 of the time at two thirds, a half and a third of the tokens, 1.00 to
    // 1.03 at a quarter and less, over 8 to 256 pairs of 200 to 11 K chunks).  Bins are even steps of the key, which cost less, or of the score where the keys'
    // range is over 32 binary orders (keys of scores of both signs crowd around zero: of 1.6 K such chunks the top 40 were in three
    // bins, and the crowded bin's way took 13.5 us, now 5.1).
    int fb = -1, remW = W;                                          // cutoff bin (-1: every candidate fits), budget left for it
    const float s_hi = lc_key_score(kmax), s_all = s_hi - lc_key_score(kmin);
    const bool by_score = kmax - kmin > (32u << 23) && s_all > 1e-30f && s_all < 1e30f;      // (not for infinities)
    for (bool half = W < T / 3;; half = false) {
        if (by_score) {
            const float s_lo = half ? s_hi - 0.5f * s_all : lc_key_score(kmin);
            const float per_bin = (float)BINS * __builtin_amdgcn_rcpf(half ? 0.5f * s_all : s_all);
#pragma unroll
            for (int e = 0; e < EC; ++e) {
                const float s = lc_key_score(ck[e]) - s_lo;
                const bool in = ck[e] != 0u && s >= 0.f;
                bin[e] = in ? min((int)(s * per_bin), BINS - 1) : (bin[e] == BINS ? BINS : -1);
                if (in) atomicAdd(&hist[bin[e]], len[e]);
                if (EC > 8 && (e & 3) == 3) __builtin_amdgcn_sched_barrier(0);      // (twelve at a time do not fit the registers)
            }
        } else {
            const uint32_t lo = half ? kmax - (kmax - kmin) / 2u : kmin, span = kmax - lo;
            const int bits = (kmax != 0u && span) ? 32 - __clz(span) : 0;
            const int shift = bits > BITS ? bits - BITS : 0;        // (span >> shift) < BINS
#pragma unroll
            for (int e = 0; e < EC; ++e) {
                const bool in = ck[e] >= lo && ck[e] != 0u;
                const int b = (int)((ck[e] - lo) >> shift);
                bin[e] = in ? b : (bin[e] == BINS ? BINS : -1);
                if (in) atomicAdd(&hist[b], len[e]);
            }
        }
        lc_barrier_lds();
        // every wavefront scans all bins from the top: lane l holds bins BINS - 1 - PER l - i, i < PER
        constexpr int PER = BINS / 64;
        int pw[PER];
        const int4* hw4 = reinterpret_cast<const int4*>(hist + BINS - PER * (lane + 1));
#pragma unroll
        for (int v = 0; v < PER / 4; ++v) {
            const int4 x = hw4[PER / 4 - 1 - v];
            pw[4 * v + 0] = x.w; pw[4 * v + 1] = x.z; pw[4 * v + 2] = x.y; pw[4 * v + 3] = x.x;
        }
#pragma unroll
        for (int i = 1; i < PER; ++i) pw[i] += pw[i - 1];
        const int cw = lc_wave_scan_incl(pw[PER - 1]) - pw[PER - 1];
        int fit = 0, fitw = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const bool ok = cw + pw[i] <= W;
            fit += ok ? 1 : 0;
            fitw = ok ? pw[i] : fitw;
        }
        const unsigned long long bal = __ballot(fit < PER);         // the prefix ends in the first bin that no longer fits
        if (bal != 0ull) {
            const int fl = __ffsll((long long)bal) - 1;
            fb = BINS - 1 - (PER * fl + lc_readlane(fit, fl));
            remW = W - (lc_readlane(cw, fl) + lc_readlane(fitw, fl));
            break;
        }
        if (!half) break;
        lc_barrier_lds();                                           // the bins have been read
        for (int i = tid; i < BINS; i += NT) hist[i] = 0;
        lc_barrier_lds();
    }
    // ---- chunks above that bin are selected, those in it go to a list
    unsigned sel = 0u;                                              // bit e: this lane's chunk e is selected
    const int cutoff = fb >= 0 ? fb : -2;
#pragma unroll
    for (int e = 0; e < EC; ++e) {
        sel |= bin[e] > fb ? 1u << e : 0u;
        if (__ballot(bin[e] == cutoff) != 0ull) {                   // (uniform; few of the rows)
            if (bin[e] == cutoff) {
                const int at = atomicAdd(&n_cand, 1);
                if (at < LC_SL_CAND) cand[at] = make_int4((int)ck[e], len[e], j0 + 64 * e, 0);
            }
        }
    }
    lc_barrier_lds();
    const int nc = n_cand;
    if (nc <= LC_SL_CAND) {
        // ---- the list in order (key descending, id ascending): lane c adds up the lengths before chunk c, then a wavefront takes its own of
        // those that fit.  A few are ranked by every wavefront; of more, a wavefront adds up every 16th and the sums meet in LDS (a barrier, 0.2 us).
        auto precedes = [](const int4& o, const int4& me) LC_INLINE { return (uint32_t)o.x > (uint32_t)me.x || (o.x == me.x && o.z < me.z); };
        auto take = [&](int c0, const int4& me, int before) LC_INLINE {
            const int e_me = (me.z >> 6) - wave * EC;
            for (unsigned long long won = __ballot(c0 + lane < nc && e_me >= 0 && e_me < EC && before + me.y <= remW); won != 0ull; won &= won - 1ull) {
                const int id = lc_readlane(me.z, __ffsll((long long)won) - 1);
                sel |= lane == (id & 63) ? 1u << ((id >> 6) - wave * EC) : 0u;       // (uniform but for the lane)
            }
        };
        if (nc <= LC_SL_FEW) {
            const int4 me = cand[min(lane, max(nc - 1, 0))];
            int sum = 0;
            for (int c = 0; c < nc; ++c) {                          // (uniform)
                const int4 o = make_int4(lc_readlane(me.x, c), lc_readlane(me.y, c), lc_readlane(me.z, c), 0);
                sum += precedes(o, me) ? o.y : 0;
            }
            take(0, me, sum);
        } else {
            for (int c0 = 0; c0 < nc; c0 += 64) {
                const int4 me = cand[min(c0 + lane, nc - 1)];
                int sum = 0;
                for (int c = wave; c < nc; c += NW) sum += precedes(cand[c], me) ? cand[c].y : 0;
                if (sum != 0 && c0 + lane < nc) atomicAdd(&ahead[c0 + lane], sum);
            }
            lc_barrier_lds();
            for (int c0 = 0; c0 < nc; c0 += 64) {
                const int c = min(c0 + lane, nc - 1);
                take(c0, cand[c], ahead[c]);
            }
        }
    } else {
        // ---- a crowded or tied cutoff bin: the general select routine on its chunks alone
        uint32_t* const skey = reinterpret_cast<uint32_t*>(lds_dyn);
        int* const slen = lds_dyn + EC * NT;
        lc_leaf_select_prepare<NT>(sel_sh);
        lc_barrier_lds();
        uint32_t bmin = 0xffffffffu, bmax = 0u;
#pragma unroll
        for (int e = 0; e < EC; ++e) {
            const uint32_t k = bin[e] == cutoff ? (ck[e] == 0xffffffffu ? 0xfffffffeu : ck[e]) : 0u;      // the mark is reserved
            skey[j0 + 64 * e] = k;
            slen[j0 + 64 * e] = len[e];
            if (k != 0u) { bmin = min(bmin, k); bmax = max(bmax, k); }
        }
        lc_leaf_select_range(bmin, bmax, sel_sh);
        lc_barrier_lds();
        const uint32_t thr = lc_leaf_select<NT>(EC * NT, skey, slen, (long long)remW, 0x7fffffffLL, sel_sh);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < EC; ++e) sel |= bin[e] == cutoff && skey[j0 + 64 * e] > thr ? 1u << e : 0u;
    }
    // ---- the ids, ascending
    unsigned long long row[EC];
    int total = 0;
#pragma unroll
    for (int e = 0; e < EC; ++e) {
        row[e] = __ballot((sel >> e) & 1u);
        total += __popcll(row[e]);
    }
    if (lane == 0) number[wave] = total;
    lc_barrier_lds();
    const int n = lane < NW ? number[lane] : 0, before = lc_wave_scan_incl(n) - n;
    int at = lc_readlane(before, wave);
    int32_t* const ids = a.ids + (size_t)bh * a.cap;
#pragma unroll
    for (int e = 0; e < EC; ++e) {
        const int p = at + lc_mbcnt(row[e]);
        if (((sel >> e) & 1u) && p < a.cap) ids[p] = j0 + 64 * e;
        at += __popcll(row[e]);
    }
    if (tid == 0) a.counts[bh] = min(lc_readlane(before + n, NW - 1), a.cap);
}
template <int EC>
static int launch_select_e(const LcSelectArgs& a, int pairs, hipStream_t stream) {
    constexpr size_t lds = (size_t)EC * LC_SL_THREADS * 8;
    if (lds > 16 * 1024) {                                          // static + dynamic beyond the default allowance: raised once per device
        static LcOnce raised;
        LC_HIP_CHECK(raised.run([&] {
            return hipFuncSetAttribute(reinterpret_cast<const void*>(&lc_select_kernel<EC>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        }));
    }
    hipLaunchKernelGGL(lc_select_kernel<EC>, dim3(pairs), dim3(LC_SL_THREADS), lds, stream, a);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}
static int launch_select(const LcRetrieveArgs& r, int max_M, hipStream_t stream) {
    const LcSelectArgs a{r.scratch, r.ix.state, r.ids, r.counts, r.ix.cap[0], r.cap, r.budget, r.sink};
    const int pairs = r.ix.B * r.ix.H, rows = (max_M + LC_SL_THREADS - 1) / LC_SL_THREADS;
    if (rows <= 1) return launch_select_e<1>(a, pairs, stream);
    if (rows <= 2) return launch_select_e<2>(a, pairs, stream);
    if (rows <= 4) return launch_select_e<4>(a, pairs, stream);
    if (rows <= 8) return launch_select_e<8>(a, pairs, stream);
    return launch_select_e<LC_SL_EC_MAX>(a, pairs, stream);
}

template <int G, int R>
static int launch_score(const LcRetrieveArgs& a, int max_M, hipStream_t stream) {
    const int per = R * (LC_SC_THREADS / 16);
    const int nblk = max_M > 0 ? (max_M + per - 1) / per : 1;
    if (a.ix.c0_bf16)
        hipLaunchKernelGGL((lc_score_kernel<G, R, true>), dim3(nblk, a.ix.H, a.ix.B), dim3(LC_SC_THREADS), 0, stream, a);
    else
        hipLaunchKernelGGL((lc_score_kernel<G, R, false>), dim3(nblk, a.ix.H, a.ix.B), dim3(LC_SC_THREADS), 0, stream, a);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}

template <int G, int R, bool BF16>
static int launch_leaf_t(const LcRetrieveArgs& a, int max_M, size_t lds, hipStream_t stream) {
    if (lds + sizeof(LcLeafSelSh) + 1024 > 48 * 1024)             // static + dynamic beyond the default allowance
        LC_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&lc_leaf_kernel<G, R, BF16>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const int per = R * LC_LF_GROUPS;
    const int nblk = max_M > 0 ? (max_M + per - 1) / per : 1;
    hipLaunchKernelGGL((lc_leaf_kernel<G, R, BF16>), dim3(nblk, a.ix.H, a.ix.B), dim3(LC_LF_THREADS), lds, stream, a);
    LC_HIP_CHECK(hipGetLastError());
    return LC_OK;
}
template <int G, int R>
static int launch_leaf(const LcRetrieveArgs& a, int max_M, size_t lds, hipStream_t stream) {
    return a.ix.c0_bf16 ? launch_leaf_t<G, R, true>(a, max_M, lds, stream) : launch_leaf_t<G, R, false>(a, max_M, lds, stream);
}

template <int G>
static int launch_retrieve_g(LcRetrieveArgs& a, int max_M, hipStream_t stream) {
    const LcDev& ix = a.ix;
    const int mc = ((max_M + 63) / 64) * 64;
    const size_t lds_limit = LC_WALK_LDS_LIMIT;
    if (a.policy == LC_POLICY_BEAM) return launch_beam_g<G>(a, max_M, a.upper_cap > max_M ? a.upper_cap : max_M, stream);
    if (a.walk) {
        // as long a probe list as LDS holds next to the internal-node slots (the host has checked that one fits)
        int uc, pc;
        if (!lc_upper_launch_shape(a.upper_cap, max_M, &uc, &pc)) return LC_ERR_CAPACITY;
        a.upper_cap = uc;
        a.chunk_cap = pc;
        const size_t lds = lc_upper_lds_bytes(uc, pc);
        if (lds > 48 * 1024)
            LC_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&lc_upper_kernel<G>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        hipLaunchKernelGGL(lc_upper_kernel<G>, dim3(ix.H, ix.B), dim3(LC_UP_THREADS), lds, stream, a);
        LC_HIP_CHECK(hipGetLastError());
    }
    // lc_retrieve: two kernels as far as the selecting one holds a (sequence, head)'s chunks in registers (measured there).  Not with seven
    // or eight queries per KV head on float32 centers where the one kernel's workgroups, of up to 512 chunks, are on the device at once and nearly
    // fill it: scoring is arithmetic then, and a group of lanes has eight chunks for a query it unpacks once.  us with one and two kernels at
    // group size 7, a quarter of the tokens: 256 (sequence, head) pairs of 250 chunks 15.2 and 14.0, of 300 14.4 and 15.8, of 450 17.6 and 19.7; 208 of 440
    // 16.5 and 17.0; 192 of 450 16.4 and 16.9, of 510 17.1 and 17.5; 176 of 510 17.1 and 16.8; 128 of 850 18.9 and 19.0, of 900 19.1 and 19.7, of 1020 20.2 and
    // 20.8; 64 of 1500 18.8 and 17.5, of 1750 19.3 and 19.5, of 1850 19.8 and 20.2, of 2400 (in turns) 30.4 and 24.1.  bfloat16 centers: 2 to 30 % slower as one.
    // (The scoring kernel has become 0.3 to 0.7 us faster there since: 256 pairs of 300 and 450 chunks still 1.8 us slower as two, 208 of 440 0.5, fewer pairs
    // between 0.4 us slower and 0.7 faster, either way within 1 % of a retrieval with its attention.)
    const int pairs = ix.H * ix.B;
    const bool full = pairs >= 64 && (long long)((max_M + 511) / 512) * pairs <= LC_COMPUTE_UNITS &&
                      ((long long)pairs * max_M >= 116000 || (pairs >= 200 && max_M > 256));
    const bool one = G >= 7 && !ix.c0_bf16 && !a.walk && full;
    const bool two = !a.score_only && !one && max_M > LC_FLAT_MAX_CHUNKS && max_M <= LC_SL_THREADS * LC_SL_EC_MAX;
    if (a.score_only || two) {
        // chunks per group: enough work per workgroup without leaving compute units idle
        int rs = 1;
        while (rs < 4) {
            const long long wgs = (long long)((max_M + 16 * rs - 1) / (16 * rs)) * ix.H * ix.B;
            if (wgs <= (rs == 2 && !ix.c0_bf16 ? LC_SCORE_MAX_WGS_F32 : LC_SCORE_MAX_WGS)) break;
            rs *= 2;
        }
        const int rc = rs == 1 ? launch_score<G, 1>(a, max_M, stream)
                               : (rs == 2 ? launch_score<G, 2>(a, max_M, stream) : launch_score<G, 4>(a, max_M, stream));
        return rc != LC_OK || !two ? rc : launch_select(a, max_M, stream);
    }
    if (!a.walk && max_M <= LC_FLAT_MAX_CHUNKS) {        // one level, every chunk a candidate
        LcRetrieveArgs f = a;
        f.ix.L = 1;
        f.beam[0] = 0;
        return launch_beam_g<G>(f, max_M, max_M, stream);
    }
    a.chunk_cap = ((size_t)mc * 8 + sizeof(LcLeafSelSh) + 1024 <= lds_limit) ? mc : 0;
    const size_t lds2 = (size_t)a.chunk_cap * 8;
    // chunks per group: the fewest for which there is at most one workgroup per compute unit
    // (measured: beyond that the kernel gets slower, not faster)
    int r = 1;
#ifdef LC_LEAF_FORCE_R
    r = LC_LEAF_FORCE_R;
#else
    while (r < 8 && (long long)((max_M + 64 * r - 1) / (64 * r)) * ix.H * ix.B > 256) r *= 2;
#endif
    if (r == 1) return launch_leaf<G, 1>(a, max_M, lds2, stream);
    if (r == 2) return launch_leaf<G, 2>(a, max_M, lds2, stream);
    if (r == 4) return launch_leaf<G, 4>(a, max_M, lds2, stream);
    return launch_leaf<G, 8>(a, max_M, lds2, stream);
}

// Most internal nodes of one (sequence, head) that the exact level walk holds in LDS (with the shortest probe list).
int lc_walk_max_internal_nodes() { return lc_upper_max_internal_nodes(); }
int lc_beam_max_level_nodes() { return LC_BM_MAX_LEVEL_NODES; }

int lc_launch_retrieve(const lc_index* idx, const LcWs& ws, const void* q, int G, int budget,
                       int32_t* ids, int32_t* counts, float* scores, int cap,
                       int max_M, int max_upper, int score_only, hipStream_t stream) {
    LcRetrieveArgs a;
    a.score_only = score_only;
    a.ix = idx->dev;
    a.q = static_cast<const uint16_t*>(q);
    a.keys = ws.keys;
    a.want = ws.want;
    a.scores = scores;
    a.ids = ids;
    a.counts = counts;
    a.scratch = ws.scratch;
    a.cap = cap;
    a.budget = budget;
    a.policy = idx->cfg.policy;
    a.sink = idx->cfg.sink_tokens;
    for (int l = 0; l < LC_MAX_LEVELS; ++l) a.beam[l] = idx->cfg.beam[l];
    a.walk = (max_upper >= 0 && idx->cfg.levels > 1) ? 1 : 0;
    if (max_upper < 0) max_upper = 0;
    a.upper_cap = ((max_upper + 63) / 64) * 64;
    if (a.upper_cap < 64) a.upper_cap = 64;
    a.chunk_cap = 0;
    switch (G) {
        case 1: return launch_retrieve_g<1>(a, max_M, stream);
        case 2: return launch_retrieve_g<2>(a, max_M, stream);
        case 3: return launch_retrieve_g<3>(a, max_M, stream);
        case 4: return launch_retrieve_g<4>(a, max_M, stream);
        case 5: return launch_retrieve_g<5>(a, max_M, stream);
        case 6: return launch_retrieve_g<6>(a, max_M, stream);
        case 7: return launch_retrieve_g<7>(a, max_M, stream);
        case 8: return launch_retrieve_g<8>(a, max_M, stream);
    }
    return LC_ERR_BAD_SHAPE;
}
