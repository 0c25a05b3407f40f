// The large sets of a small batch, shared by several blocks in one launch.
//
// k_small takes a set per block, and the host knows only the batch's total, so
// a set may be too large for its block: k_small leaves those (more than
// SM_TRY points, or more survivors than its LDS holds) to this kernel.  Each
// is cut into parts of BIG_PART points, which fit a block's LDS at every step,
// and the steps of the general path follow one another in phases: a block
// claims the next part (or set) of the phase, and no block begins a phase
// before the one before it is finished.  A claimed part is in the hands of a
// running block, so every wait ends however many blocks run at a time, and
// with no such set the kernel moves the hulls to their places and ends.
//
// What bounds it is the phases' latency, 8 to 30 us each.  240000 points and
// sixty sets of 30: 177 (square), 194 (annulus), 593 us (circle) with k_small,
// against 201, 212 and 684 with the launches of the general path and 412, 890
// and 10100 with one block per set; 16000 on a circle and ten more 358, 495
// and 799.  Parts of 8192 points took 1.2 to 1.5 times as long.
#include "hg_device.h"

namespace hg {

constexpr int BIG_THREADS = 1024, BIG_WAVES = BIG_THREADS / WAVE;
constexpr int BIG_PART = 4096;               // points of a part
constexpr int BIG_CAP = 8192;                // keys of a list in LDS
constexpr int BIG_MERGE = 2048;              // a set's chains that one block sorts together
constexpr int64_t BIG_POINTS = 1 << 18;      // of the batch
constexpr int BIG_SETS = BIG_POINTS / SM_CAP;                // at most: each has more than SM_CAP points
constexpr int BIG_PARTS = BIG_POINTS / BIG_PART + BIG_SETS;
constexpr int BIG_BLOCKS = 128;
constexpr int BIG_SEGS = BIG_WAVES / 2;      // waves per chain
static_assert(BIG_PARTS <= BIG_BLOCKS, "a part per block");

constexpr int VMCNT_0 = 0x0F70;              // s_waitcnt: vector memory done, the other counters as they are

enum BigPhase {
    B_EXTREMES = 0, B_DISCARD, B_ROUND, B_CHAINS = B_ROUND + REF_ROUNDS, B_MERGE, B_RANK, B_SLICE,
    B_JOIN, B_LOOKUP, B_NPHASES
};

// State of a call in global memory: zeroed claims, and what parts and sets
// leave for later phases.
struct BigState {
    uint32_t claim[B_NPHASES], done[B_NPHASES];
    int surv[BIG_PARTS], cand[BIG_PARTS];    // a part's survivors and candidates
    int len[2][BIG_PARTS];                   // its lower and upper chain
    uint32_t slice[2][BIG_PARTS];            // chains of the slices of the merged lists
    uint32_t chain[2][BIG_SETS];             // a set's chains
    int hard[BIG_SETS];                      // its parts' chains together do not fit LDS
    double pval[BIG_PARTS * MAX_SLOTS];      // the parts' extremes
    uint32_t pidx[BIG_PARTS * MAX_SLOTS];
};

// Workspace: entries of a set, and of its parts, at its own points' positions.
struct BigWs {
    BigState *st;
    const int32_t *defer;                    // [S] from k_small: not done
    Poly *polys;
    unsigned long long *far;                 // [S][RE_CAP]: round r's from (2^r - 1) MAX_SLOTS on
    uint32_t *idx, *cidx;
    uint64_t *key, *ckey, *lo[2], *up[2];
    uint16_t *edge;
    uint32_t *hull, *hcnt;
    int32_t *scnt;
};
static_assert(((1 << REF_ROUNDS) - 1) * MAX_SLOTS <= RE_CAP, "the rounds' farthest keys fit a set's entries");

struct BigLds {
    // a lower and an upper list; a part's keys and indices; or samples of the chains
    uint64_t key[BIG_CAP];
    uint64_t up[BIG_CAP];
    unsigned long long far[RE_CAP];
    REdge tab[2][RE_CAP];
    Poly P;
    PolyScratch G;
    uint32_t sl[MAX_SLOTS];
    SlotBest best[BIG_WAVES][MAX_SLOTS];
    int seg[2][BIG_SEGS], total[2];
    int64_t sh[3 + 2 * CHAIN_G];
    // the sets: index, first point, size, first part
    int nset, set[BIG_SETS], n[BIG_SETS], part0[BIG_SETS + 1];
    int64_t a[BIG_SETS];
    int plen[2][BIG_PARTS];
    int wcnt[BIG_WAVES], count, task;
};

// Step 1 of points [a, e), at most BIG_PART: values and indices of the
// evaluated slots, twelve at a time (more would not fit 128 registers).
template <int PRESET>
__device__ __forceinline__ void big_extremes(BigLds &L, const float *__restrict__ x, const float *__restrict__ y,
                                             int64_t a, int64_t e, const Dirs &dirs, double *pval, uint32_t *pidx) {
    constexpr int NF = 4 * Proj<PRESET>::NG, TURNS = (NF + 11) / 12, NT = NF / TURNS;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
#pragma unroll
    for (int turn = 0; turn < TURNS; turn++) {
        double lb[NT];
        uint32_t li[NT];
#pragma unroll
        for (int k = 0; k < NT; k++) {
            lb[k] = slot_is_min(turn * NT + k, NF) ? INFINITY : -INFINITY;
            li[k] = NONE;
        }
        for (int64_t i = a + tid; i < e; i += BIG_THREADS) {
            double key[NF];
            slot_keys<PRESET, 0>(dirs, nullptr, nullptr, (double)x[i], (double)y[i], key);
#pragma unroll
            for (int k = 0; k < NT; k++) {
                const double v = key[turn * NT + k];
                const bool b = slot_is_min(turn * NT + k, NF) ? v < lb[k] : v > lb[k];
                lb[k] = b ? v : lb[k];
                li[k] = b ? (uint32_t)i : li[k];
            }
        }
        // the best value, then the lowest index that has it; empty records hold NONE
#pragma unroll
        for (int k = 0; k < NT; k++) {
            const double m = slot_is_min(turn * NT + k, NF) ? wave_extreme<true>(lb[k]) : wave_extreme<false>(lb[k]);
            const uint32_t i = wave_min_u32(lb[k] == m ? li[k] : NONE);
            if (lane == 0) L.best[w][turn * NT + k] = SlotBest{m, i};
        }
    }
    __syncthreads();
    if (tid < NF) {
        SlotBest b = L.best[0][tid];
        for (int ww = 1; ww < BIG_WAVES; ww++) {
            const SlotBest o = L.best[ww][tid];
            const bool t = (slot_is_min(tid, NF) ? o.v < b.v : o.v > b.v) || (o.v == b.v && o.i < b.i);
            b.v = t ? o.v : b.v;
            b.i = t ? o.i : b.i;
        }
        pval[tid] = b.v;
        pidx[tid] = b.i;
    }
}

// The chains of the sorted lists key[0..nl0) and up[0..nu0): half the waves
// take a part of the lower list each, half of the upper one, then one wave per
// list joins the parts.  The lengths go to L.total.
__device__ __forceinline__ void big_chains(BigLds &L, int nl0, int nu0) {
    const int lane = lane_id(), w = threadIdx.x >> 6;
    const int kind = w >= BIG_SEGS, q = w % BIG_SEGS, M = kind ? nu0 : nl0;
    const int per = ((M + BIG_SEGS - 1) / BIG_SEGS + WAVE - 1) / WAVE * WAVE;
    uint64_t *list = kind ? L.up : L.key;
    const int b0 = min(M, q * per), c = min(M, b0 + per) - b0;
    const int r = kind ? list_chain<true, 1, 16>(list + b0, c) : list_chain<false, 1, 16>(list + b0, c);
    if (lane == 0) L.seg[kind][q] = r;
    __syncthreads();
    if (q == 0) {
        const int mine = lane < BIG_SEGS ? L.seg[kind][lane] : 0;
        const int t = kind ? join_pieces<true>(list, per, BIG_SEGS, mine) : join_pieces<false>(list, per, BIG_SEGS, mine);
        if (lane == 0) L.total[kind] = t;
    }
    __syncthreads();
}

// Sort n keys (n <= BIG_PART) by the block.
__device__ __forceinline__ void big_sort(uint64_t *b, int n) {
    const int P = sort_width(n);
    for (int i = n + (int)threadIdx.x; i < P; i += BIG_THREADS) b[i] = ~0ull;
    __syncthreads();
    block_sort<BIG_PART>(b, P);
}

// The place of each key of a part's sorted list in the merged lists of its
// set's np parts: its own index plus what is before it in the others (equal
// keys: the earlier part's first).  The others come through LDS one by one
// (searched in global memory, 760 us for the 240000 of a circle; now 134).
__device__ __forceinline__ void big_rank(uint64_t *buf, const uint64_t *__restrict__ lists,
                                         const int *__restrict__ len, int np, int p, uint64_t *__restrict__ out) {
    constexpr int U = BIG_PART / BIG_THREADS;
    const int tid = threadIdx.x, n = len[p];
    uint64_t k[U], v[U];
    int rank[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int i = tid + u * BIG_THREADS;
        k[u] = i < n ? lists[(int64_t)p * BIG_PART + i] : 0;
        rank[u] = i;
    }
    auto load = [&](int q) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int i = tid + u * BIG_THREADS;
            v[u] = i < len[q] ? lists[(int64_t)q * BIG_PART + i] : ~0ull;
        }
    };
    const int q0 = p ? 0 : 1;
    if (q0 < np) load(q0);
    for (int q = q0; q < np;) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; u++) buf[tid + u * BIG_THREADS] = v[u];       // ~0 behind the list
        __syncthreads();
        const int next = q + 1 == p ? q + 2 : q + 1;
        if (next < np) load(next);                                           // in flight under the search
        int pos[U];
#pragma unroll
        for (int u = 0; u < U; u++) pos[u] = 0;
        for (int step = BIG_PART / 2; step > 0; step >>= 1)
#pragma unroll
            for (int u = 0; u < U; u++) pos[u] += buf[pos[u] + step - 1] < search_key(k[u], q < p) ? step : 0;
#pragma unroll
        for (int u = 0; u < U; u++) rank[u] += pos[u] + (int)(buf[pos[u]] < search_key(k[u], q < p));
        q = next;
    }
#pragma unroll
    for (int u = 0; u < U; u++)
        if (tid + u * BIG_THREADS < n) out[rank[u]] = k[u];
    __syncthreads();
}

// The number of keys below k in list[0..n), of which samp holds every
// stride-th: a search in LDS, then one of the stride between two samples.
__device__ __forceinline__ int big_below(const uint64_t *list, int n, const uint64_t *samp, int stride, uint64_t k) {
    int a = 0, b = (n + stride - 1) / stride;
    while (a < b) {
        const int m = (a + b) >> 1;
        if (samp[m] < k) a = m + 1; else b = m;
    }
    b = min(n, a * stride);              // a samples are below k: list[(a - 1) stride] < k <= list[a stride]
    a = a ? (a - 1) * stride + 1 : 0;
    while (a < b) {
        const int m = (a + b) >> 1;
        if (list[m] < k) a = m + 1; else b = m;
    }
    return a;
}

__global__ __launch_bounds__(BIG_THREADS) void k_big(const float *__restrict__ x, const float *__restrict__ y,
                                                     int64_t n_total, int phase, const int64_t *__restrict__ off,
                                                     int64_t S, int preset, Dirs dirs, BigWs ws,
                                                     int64_t *__restrict__ hoff, uint32_t *__restrict__ hull,
                                                     int64_t *__restrict__ counts) {
    __shared__ BigLds L;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const uint64_t lt = lanemask_lt();
    BigState &St = *ws.st;

    bool mine = false;
    for (int64_t s = tid; s < S; s += BIG_THREADS) mine |= ws.defer[s] != 0;
    if (!__syncthreads_or(mine)) {
        small_out<BIG_THREADS>(off, S, ws.hcnt, ws.scnt, ws.hull, hoff, hull, counts, reinterpret_cast<int64_t *>(L.key), L.sh);
        return;
    }

    // the sets left to this kernel, in order, the same in every block
    if (tid == 0) L.nset = 0;
    for (int64_t s0 = 0; s0 < S; s0 += BIG_THREADS) {
        const bool d = s0 + tid < S && ws.defer[s0 + tid];
        const uint64_t b = __ballot(d);
        __syncthreads();
        if (lane == 0) L.wcnt[w] = __popcll(b);
        __syncthreads();
        int at = L.nset, all = 0;
        for (int ww = 0; ww < BIG_WAVES; ww++) {
            at += ww < w ? L.wcnt[ww] : 0;
            all += L.wcnt[ww];
        }
        at += __popcll(b & lt);
        if (d && at < BIG_SETS) {
            const int64_t a = off[s0 + tid];
            L.set[at] = (int)(s0 + tid);
            L.a[at] = a;
            L.n[at] = (int)(min(off[s0 + tid + 1], n_total) - a);
        }
        __syncthreads();
        if (tid == 0) L.nset = min(L.nset + all, BIG_SETS);
    }
    __syncthreads();
    if (tid == 0) {
        int p = 0, i = 0;
        for (; i < L.nset; i++) {
            L.part0[i] = p;
            const int np = (L.n[i] + BIG_PART - 1) / BIG_PART;
            if (p + np > BIG_PARTS) break;       // only with offsets that overlap
            p += np;
        }
        L.part0[i] = p;
        L.nset = i;
    }
    __syncthreads();
    const int NS = L.nset, NP = L.part0[NS];

    // f(task) for the phase's tasks that this block claims, then the wait for
    // those of the others
    auto run = [&](int ph, int tasks, auto &&f) {
        for (;;) {
            __syncthreads();
            if (tid == 0) L.task = (int)atomicAdd(&St.claim[ph], 1u);
            __syncthreads();
            const int t = L.task;
            if (t >= tasks) break;
            f(t);
            // every wave's stores are in the L2 before thread 0 releases them
            // to the other XCDs (with a release by each of the sixteen waves
            // the phases took twice as long)
            __builtin_amdgcn_s_waitcnt(VMCNT_0);
            __syncthreads();
            if (tid == 0) {
                __threadfence();
                atomicAdd(&St.done[ph], 1u);
            }
        }
        if (tid == 0) {
            while (__hip_atomic_load(&St.done[ph], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (uint32_t)tasks)
                __builtin_amdgcn_s_sleep(2);
            __threadfence();
        }
        __syncthreads();
    };
    // part t: its set i, first point a and size n
    auto part = [&](int t, int &i, int64_t &a, int &n) {
        i = 0;
        while (i + 1 < NS && L.part0[i + 1] <= t) i++;
        const int at = (t - L.part0[i]) * BIG_PART;
        a = L.a[i] + at;
        n = min(BIG_PART, L.n[i] - at);
    };
    // the lengths of set i's part chains into L.plen, and their sums
    auto lens = [&](int i, int *n) {
        const int p0 = L.part0[i], np = L.part0[i + 1] - p0, k = tid >> 9, p = tid & 511;
        if (p < np) L.plen[k][p] = St.len[k][p0 + p];
        __syncthreads();
        n[0] = n[1] = 0;
        for (int q = 0; q < np; q++) {
            n[0] += L.plen[0][q];
            n[1] += L.plen[1][q];
        }
    };
    auto load_poly = [&](int s) {
        const uint32_t *src = reinterpret_cast<const uint32_t *>(ws.polys + s);
        for (int j = tid; j < (int)(sizeof(Poly) / 4); j += BIG_THREADS) reinterpret_cast<uint32_t *>(&L.P)[j] = src[j];
    };
    auto flush_far = [&](int s, int r) {     // L.far into round r's keys of set s
        for (int k = tid; k < MAX_SLOTS << r; k += BIG_THREADS)
            if (L.far[k]) atomicMax(&ws.far[(int64_t)s * RE_CAP + ((1 << r) - 1) * MAX_SLOTS + k], L.far[k]);
    };

    run(B_EXTREMES, NP, [&](int t) {
        int i, n;
        int64_t a;
        part(t, i, a, n);
        double *pv = St.pval + t * MAX_SLOTS;
        uint32_t *pi = St.pidx + t * MAX_SLOTS;
        switch (preset) {
        case 0: big_extremes<0>(L, x, y, a, a + n, dirs, pv, pi); break;
        case 1: big_extremes<1>(L, x, y, a, a + n, dirs, pv, pi); break;
        case 2: big_extremes<2>(L, x, y, a, a + n, dirs, pv, pi); break;
        case 3: big_extremes<3>(L, x, y, a, a + n, dirs, pv, pi); break;
        case 4: big_extremes<4>(L, x, y, a, a + n, dirs, pv, pi); break;
        case 5: big_extremes<5>(L, x, y, a, a + n, dirs, pv, pi); break;
        case 6: big_extremes<6>(L, x, y, a, a + n, dirs, pv, pi); break;
        default: big_extremes<7>(L, x, y, a, a + n, dirs, pv, pi); break;
        }
    });
    run(B_DISCARD, NP, [&](int t) {
        int i, n;
        int64_t a;
        part(t, i, a, n);
        // the set's polygon from its parts' extremes, by each part
        const int s = L.set[i], nf = 4 * preset_eval_groups(preset);
        const int p0 = L.part0[i], np = L.part0[i + 1] - p0;
        SlotBest *parts = reinterpret_cast<SlotBest *>(L.key);
        for (int j = tid; j < np * MAX_SLOTS; j += BIG_THREADS)
            parts[j] = SlotBest{St.pval[p0 * MAX_SLOTS + j], St.pidx[p0 * MAX_SLOTS + j]};
        __syncthreads();
        if (tid < MAX_SLOTS) {
            SlotBest b{0.0, NONE};
            for (int p = 0; tid < nf && p < np; p++) {
                const SlotBest o = parts[p * MAX_SLOTS + tid];
                const bool t = (int)(o.i != NONE) & ((int)(b.i == NONE) | (int)(tid & 1 ? o.v > b.v : o.v < b.v));
                b.v = t ? o.v : b.v;         // parts in index order: the first of equal ones stays
                b.i = t ? o.i : b.i;
            }
            L.sl[tid] = b.i;
            L.far[tid] = 0;
        }
        if (tid == 0) L.count = 0;
        __syncthreads();
        if (preset == 1 && tid == 0) {    // the 120-degree group repeats the 30-degree one
            L.sl[12] = L.sl[7];
            L.sl[13] = L.sl[6];
            L.sl[14] = L.sl[4];
            L.sl[15] = L.sl[5];
        }
        __syncthreads();
        build_polygon(L.G, L.sl, x, y, (L.a[i] + L.n[i] - tile_base(L.a[i], phase) + TILE - 1) / TILE, L.P);
        if (t == L.part0[i])
            for (int j = tid; j < (int)(sizeof(Poly) / 4); j += BIG_THREADS)
                reinterpret_cast<uint32_t *>(ws.polys + s)[j] = reinterpret_cast<const uint32_t *>(&L.P)[j];
        const int m = L.P.m;
        for (int j0 = 0; j0 < n; j0 += BIG_THREADS) {
            const int j = j0 + tid;
            const double px = j < n ? (double)(int32_t)(x[a + j] * GRIDF) : 0, py = j < n ? (double)(int32_t)(y[a + j] * GRIDF) : 0;
            bool in = m >= 3;
            for (int k = 0; k < m; k++) in = (int)in & (int)(edge_eval(L.P.ex[k], L.P.ey[k], L.P.c[k], px, py) > 0);
            const bool out = j < n && !in;
            const uint64_t b = __ballot(out);
            if (!b) continue;
            int at = 0;
            if (lane == 0) at = atomicAdd(&L.count, __popcll(b));
            at = __builtin_amdgcn_readfirstlane(at) + __popcll(b & lt);
            if (!out) continue;
            L.key[at] = ((uint64_t)((uint32_t)(int32_t)px & 0xFFFFFFu) << 24) | ((uint32_t)(int32_t)py & 0xFFFFFFu);
            reinterpret_cast<uint32_t *>(L.up)[at] = (uint32_t)(a + j);
        }
        __syncthreads();
        for (int j = tid; j < L.count; j += BIG_THREADS) {
            const uint64_t key = L.key[j];
            const uint32_t id = reinterpret_cast<const uint32_t *>(L.up)[j];
            double dist;
            uint16_t eo;
            small_edges<1>(L.P, &key, &eo, &dist);
            const unsigned long long fk = far_key(dist, id);
            if (eo != RE_NONE && L.far[eo] < fk) atomicMax(&L.far[eo], fk);
            ws.key[a + j] = key;
            ws.idx[a + j] = id;
            ws.edge[a + j] = eo;
        }
        __syncthreads();
        flush_far(s, 0);
        if (tid == 0) {
            St.surv[t] = L.count;
            atomicAdd(&ws.scnt[s * SM_COUNTS], L.count);
        }
    });
    for (int r = 0; r < REF_ROUNDS; r++)
        run(B_ROUND + r, NP, [&](int t) {
            int i, n;
            int64_t a;
            part(t, i, a, n);
            const int s = L.set[i], K = St.surv[t];
            load_poly(s);
            if (tid == 0) L.count = 0;
            __syncthreads();
            // the children of rounds 0 .. r from the polygon's edges
            const int m = L.P.m >= 2 ? L.P.m : 0;
            for (int k = tid; k < MAX_SLOTS; k += BIG_THREADS) {
                const int b = k + 1 < m ? k + 1 : 0;
                L.tab[0][k] = k < m ? REdge{L.P.vx[k], L.P.vy[k], L.P.vx[b], L.P.vy[b]} : redge_empty();
            }
            for (int q = 0; q <= r; q++) {
                __syncthreads();
                const unsigned long long *far = ws.far + (int64_t)s * RE_CAP + ((1 << q) - 1) * MAX_SLOTS;
                for (int k = tid; k < MAX_SLOTS << q; k += BIG_THREADS) {
                    REdge c0, c1;
                    split_pair(x, y, L.tab[q & 1][k], far[k], &c0, &c1);
                    L.tab[(q + 1) & 1][2 * k] = c0;
                    L.tab[(q + 1) & 1][2 * k + 1] = c1;
                }
            }
            for (int k = tid; k < RE_CAP; k += BIG_THREADS) L.far[k] = 0;
            __syncthreads();
            int alive = 0;
            for (int j = tid; j < K; j += BIG_THREADS) {
                const uint16_t st = ws.edge[a + j];
                uint16_t out = st;
                if (st < RE_DROP) {
                    double dist;
                    out = small_step(L.tab[(r + 1) & 1], st, ws.key[a + j], &dist);
                    ws.edge[a + j] = out;
                    if (out < RE_DROP) atomicMax(&L.far[out], (unsigned long long)far_key(dist, ws.idx[a + j]));
                }
                alive += out != RE_DROP;
            }
            alive = (int)wave_sum_i64(alive);
            if (lane == 0 && alive) atomicAdd(&L.count, alive);
            __syncthreads();
            if (r + 1 < REF_ROUNDS) flush_far(s, r + 1);
            if (tid == 0) atomicAdd(&ws.scnt[s * SM_COUNTS + r + 1], L.count);
        });
    run(B_CHAINS, NP, [&](int t) {
        int i, n;
        int64_t a;
        part(t, i, a, n);
        const int K = St.surv[t];
        if (tid == 0) L.count = 0;
        __syncthreads();
        for (int j0 = 0; j0 < K; j0 += BIG_THREADS) {
            const int j = j0 + tid;
            const bool keep = j < K && ws.edge[a + j] != RE_DROP;
            const uint64_t b = __ballot(keep);
            if (!b) continue;
            int at = 0;
            if (lane == 0) at = atomicAdd(&L.count, __popcll(b));
            at = __builtin_amdgcn_readfirstlane(at) + __popcll(b & lt);
            if (!keep) continue;
            const uint64_t key = ws.key[a + j];
            L.key[at] = key;
            ws.ckey[a + at] = key;
            ws.cidx[a + at] = ws.idx[a + j];
        }
        __syncthreads();
        const int M = L.count;
        big_sort(L.key, M);
        for (int j = tid; j < M; j += BIG_THREADS) L.up[j] = L.key[j];
        __syncthreads();
        big_chains(L, M, M);
        for (int j = tid; j < L.total[0]; j += BIG_THREADS) ws.lo[0][a + j] = L.key[j];
        for (int j = tid; j < L.total[1]; j += BIG_THREADS) ws.up[0][a + j] = L.up[j];
        if (tid == 0) {
            St.cand[t] = M;
            St.len[0][t] = L.total[0];
            St.len[1][t] = L.total[1];
        }
    });
    run(B_MERGE, NS, [&](int i) {
        int n[2];
        lens(i, n);
        const bool hard = n[0] > BIG_MERGE || n[1] > BIG_MERGE;
        if (tid == 0) St.hard[i] = hard;
        if (hard) return;
        for (int k = 0; k < 2; k++) {
            const uint64_t *lists = (k ? ws.up : ws.lo)[0] + L.a[i];
            for (int j = tid; j < n[k]; j += BIG_THREADS) {
                int p = 0, at = j;               // key j of all: its part, and its place there
                while (at >= L.plen[k][p]) at -= L.plen[k][p++];
                (k ? L.up : L.key)[j] = lists[(int64_t)p * BIG_PART + at];
            }
        }
        __syncthreads();
        big_sort(L.key, n[0]);
        big_sort(L.up, n[1]);
        big_chains(L, n[0], n[1]);
        for (int j = tid; j < L.total[0]; j += BIG_THREADS) ws.lo[1][L.a[i] + j] = L.key[j];
        for (int j = tid; j < L.total[1]; j += BIG_THREADS) ws.up[1][L.a[i] + j] = L.up[j];
        for (int j = tid; j < (int)hull_size(L.total[0], L.total[1]); j += BIG_THREADS) ws.hull[L.a[i] + j] = NONE;
        if (tid < 2) St.chain[tid][i] = (uint32_t)L.total[tid];
    });
    bool any = false;
    for (int i = 0; i < NS; i++) any |= St.hard[i] != 0;
    if (any) {
        // chains that LDS does not hold: merged by ranks, cut into slices
        // along x, and the slices' chains joined
        run(B_RANK, 2 * NP, [&](int t) {
            const int kind = t & 1;
            int i, n, all[2];
            int64_t a;
            part(t >> 1, i, a, n);
            if (!St.hard[i]) return;
            lens(i, all);
            const int p0 = L.part0[i], np = L.part0[i + 1] - p0;
            big_rank(L.key, (kind ? ws.up : ws.lo)[0] + L.a[i], L.plen[kind], np, (t >> 1) - p0,
                     (kind ? ws.up : ws.lo)[1] + L.a[i]);
        });
        run(B_SLICE, NP, [&](int t) {
            int i, n, m[2];
            int64_t a;
            part(t, i, a, n);
            if (!St.hard[i]) return;
            for (int j = tid; j < n; j += BIG_THREADS) ws.hull[a + j] = NONE;
            // slice of BIG_CAP keys of either list
            lens(i, m);
            const int at = (t - L.part0[i]) * BIG_CAP;
            const int64_t o = L.a[i] + at;
            for (int k = 0; k < 2; k++) {
                m[k] = max(0, min(BIG_CAP, m[k] - at));
                for (int j = tid; j < m[k]; j += BIG_THREADS) (k ? L.up : L.key)[j] = (k ? ws.up : ws.lo)[1][o + j];
            }
            __syncthreads();
            big_chains(L, m[0], m[1]);
            for (int j = tid; j < L.total[0]; j += BIG_THREADS) ws.lo[0][o + j] = L.key[j];
            for (int j = tid; j < L.total[1]; j += BIG_THREADS) ws.up[0][o + j] = L.up[j];
            if (tid < 2) St.slice[tid][t] = (uint32_t)L.total[tid];
        });
        run(B_JOIN, 2 * NS, [&](int t) {
            const int i = t >> 1;
            if (!St.hard[i]) return;
            const int p0 = L.part0[i], np = min(CHAIN_G, L.part0[i + 1] - p0);
            static_assert(BIG_POINTS / BIG_CAP <= CHAIN_G, "a set's slices are one group");
            if (t & 1)
                merge_group_block<true>(ws.up[0] + L.a[i], St.slice[1] + p0, np, BIG_CAP, 0, ws.up[1] + L.a[i],
                                        &St.chain[1][i], L.sh);
            else
                merge_group_block<false>(ws.lo[0] + L.a[i], St.slice[0] + p0, np, BIG_CAP, 0, ws.lo[1] + L.a[i],
                                         &St.chain[0][i], L.sh);
        });
    }
    run(B_LOOKUP, NP, [&](int t) {
        int i, n;
        int64_t a;
        part(t, i, a, n);
        const int nl = (int)St.chain[0][i], nu = (int)St.chain[1][i], h = (int)hull_size(nl, nu), M = St.cand[t];
        if (tid == 0 && t == L.part0[i]) ws.hcnt[L.set[i]] = (uint32_t)h;
        const uint64_t *lo = ws.lo[1] + L.a[i], *up = ws.up[1] + L.a[i];
        const int sl = (nl + BIG_CAP - 1) / BIG_CAP, su = (nu + BIG_CAP - 1) / BIG_CAP;
        for (int j = tid; j * sl < nl; j += BIG_THREADS) L.key[j] = lo[(int64_t)j * sl];
        for (int j = tid; j * su < nu; j += BIG_THREADS) L.up[j] = up[(int64_t)j * su];
        __syncthreads();
        for (int j = tid; j < M; j += BIG_THREADS) {
            const uint64_t k = ws.ckey[a + j];
            // the upper chain's ends are the lower one's
            int q = big_below(lo, nl, L.key, sl, k), p = -1;
            if (q < nl && lo[q] == k) {
                p = q;
            } else {
                q = big_below(up, nu, L.up, su, k);
                if (q > 0 && q < nu - 1 && up[q] == k) p = nl + (nu - 2 - q);
            }
            if (p >= 0 && p < h) atomicMin(&ws.hull[L.a[i] + p], ws.cidx[a + j]);
        }
    });
    __syncthreads();
    small_out<BIG_THREADS>(off, S, ws.hcnt, ws.scnt, ws.hull, hoff, hull, counts, reinterpret_cast<int64_t *>(L.key), L.sh);
}

}  // namespace hg
