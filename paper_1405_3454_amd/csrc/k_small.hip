// The whole method for small inputs, one block per set: extremes, polygon,
// discard, refinement rounds, sort, chains and index lookup in one launch,
// with the survivors, the edge tables and the chains in LDS.
//
// What bounds small inputs is the number of launches (24 for one set, 41 for
// several, 2 to 12 us each) and the latency of each kernel's few loads, not
// bandwidth, so the steps of the general path run here one after another on
// one CU with a barrier between them: 1000 points 97 -> 20 us, 64 sets of 500
// to 8000 points 232 -> 52 us.  What is left is the latency of each step's
// chain of LDS reads, and instructions fetched for the first time: code that
// runs once is kept in loops rather than unrolled.  The results, and the
// candidate counts of every stage, are the general path's: the same predicates
// on the same slots, edges and farthest keys.
//
// A set has at most SM_CAP survivors here, and so candidates, which fit the
// block's LDS; in batches that may hold larger sets, those with more survivors
// (or more than SM_TRY points) are left to k_big.
#include "hg_device.h"

namespace hg {

constexpr int SM_CAP = 8192;          // survivors of a set
constexpr int SM_TRY = 2 * SM_CAP;    // points of a set that may have no more (16000 of an annulus: 92 us)
constexpr int SM_LIGHT = 2048;        // up to here both fit side by side
constexpr int SM_THREADS = 512;       // per block: 256 took 84 us on 8000 annulus points, 512 53 us; 1000 points 20 us both
constexpr int SM_COUNTS = 1 + REF_ROUNDS;
constexpr int SM_UP = SM_CAP * 8 + 64;   // room for two keys more before it: lower + upper have two shared ends
constexpr int SM_RAW = SM_UP + SM_CAP * 8;

struct SmallLds {
    // survivors: keys [0, 64 KB), indices [64 KB, 96 KB), edges [96 KB, 112 KB);
    // chains: with at most SM_LIGHT survivors lower at 16 KB, upper at 32 KB and
    // hull at 48 KB; else lower from 0, upper and then hull from SM_UP
    char raw[SM_RAW];
    unsigned long long far[2][RE_CAP];
    REdge tab[2][RE_CAP];
    uint64_t fpt[RE_CAP];             // farthest point (key) of the edges about to split
    Poly P;
    int nsurv, ncand, alive[SM_COUNTS];
    int seg[2][8];
    PolyScratch G;
    uint32_t sl[MAX_SLOTS];
    SlotBest wbest[16][MAX_SLOTS];
};

// Workspace of a call: list entries of a set at its own points' positions.
struct SmallWs {
    uint32_t *cidx;                   // candidates
    uint64_t *ckey;
    uint32_t *hull;                   // several sets: each set's hull
    uint32_t *hcnt;
    int32_t *scnt;                    // [S][SM_COUNTS]
    // batches with room for sets of more points (else null): sets left to
    // k_big; its claims and the sets' farthest keys, cleared for it
    int32_t *defer;
    unsigned long long *far;          // [S][RE_CAP]
    uint32_t *claims;
    int nclaim;
};

// Step 1 of points [a, e): the slots into sl.
template <int PRESET, int BS>
__device__ __forceinline__ void small_extremes(const float *__restrict__ x, const float *__restrict__ y,
                                               int64_t a, int64_t e, const Dirs &dirs,
                                               SlotBest (*wbest)[MAX_SLOTS], uint32_t *sl, char *raw) {
    constexpr int NF = 4 * Proj<PRESET>::NG;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    double lb[NF];
    uint32_t li[NF];
#pragma unroll
    for (int k = 0; k < NF; k++) {
        lb[k] = slot_is_min(k, NF) ? INFINITY : -INFINITY;
        li[k] = NONE;
    }
    constexpr int U = 4;              // loads in flight
    for (int64_t i0 = a + tid; i0 < e; i0 += U * BS) {
        float xv[U], yv[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t i = min(i0 + u * BS, e - 1);
            xv[u] = x[i];
            yv[u] = y[i];
        }
#pragma unroll 1
        for (int u = 0; u < U; u++) {         // one copy of the code: it runs from a cold cache
            if (i0 + u * BS >= e) break;
            double key[NF];
            slot_keys<PRESET, 0>(dirs, nullptr, nullptr, (double)(u < 2 ? u == 0 ? xv[0] : xv[1] : u == 2 ? xv[2] : xv[3]),
                                 (double)(u < 2 ? u == 0 ? yv[0] : yv[1] : u == 2 ? yv[2] : yv[3]), key);
#pragma unroll
            for (int k = 0; k < NF; k++) {
                const bool b = slot_is_min(k, NF) ? key[k] < lb[k] : key[k] > lb[k];
                lb[k] = b ? key[k] : lb[k];
                li[k] = b ? (uint32_t)(i0 + u * BS) : li[k];
            }
        }
    }
    // reduced through LDS: thread t takes slot t % R of every (BS / R)-th
    // thread's records, then lanes of a wave and the waves combine.  Rows are
    // padded by four records: the 16 or 32 slots a wave reads at once then lie
    // in different banks.  24 slots of 512 threads take two turns.
    constexpr int ROW = BS + 4, TURNS = NF * ROW * 12 > SM_RAW ? 2 : 1, NT = NF / TURNS;
    constexpr int R = NT <= 4 ? 4 : NT <= 8 ? 8 : NT <= 16 ? 16 : 32;
    double *lv = reinterpret_cast<double *>(raw);
    uint32_t *lx = reinterpret_cast<uint32_t *>(raw + sizeof(double) * NT * ROW);
    SlotBest b;
    bool mn;
    // empty records hold the identity value and NONE, so the plain comparison
    // does (bitwise: branches would put each load's latency after the last)
    auto take = [&](double v, uint32_t i) {
        const int less = mn ? v < b.v : v > b.v;
        const bool t = less | ((int)(v == b.v) & (int)(i < b.i));
        b.v = t ? v : b.v;
        b.i = t ? i : b.i;
    };
#pragma unroll
    for (int turn = 0; turn < TURNS; turn++) {
        if (turn) __syncthreads();
#pragma unroll
        for (int k = 0; k < NT; k++) {
            lv[k * ROW + tid] = lb[turn * NT + k];
            lx[k * ROW + tid] = li[turn * NT + k];
        }
        __syncthreads();
        const int k = tid & (R - 1);
        mn = slot_is_min(turn * NT + k, NF);
        b = SlotBest{mn ? INFINITY : -INFINITY, NONE};
        if (k < NT)
#pragma unroll 8
            for (int t = tid / R; t < BS; t += BS / R) take(lv[k * ROW + t], lx[k * ROW + t]);
#pragma unroll 1
        for (int o = R; o < WAVE; o <<= 1) take(__shfl_xor(b.v, o), (uint32_t)__shfl_xor((int)b.i, o));
        if (lane < NT) wbest[w][turn * NT + lane] = b;
    }
    __syncthreads();
    if (tid < MAX_SLOTS) {
        mn = slot_is_min(tid, NF);
        b = SlotBest{mn ? INFINITY : -INFINITY, NONE};
        if (tid < NF)
#pragma unroll
            for (int ww = 0; ww < BS / WAVE; ww++) take(wbest[ww][tid].v, wbest[ww][tid].i);
        sl[tid] = b.i;
    }
    __syncthreads();
    if (PRESET == 1 && tid == 0) {    // the 120-degree group repeats the 30-degree one
        sl[12] = sl[7];
        sl[13] = sl[6];
        sl[14] = sl[4];
        sl[15] = sl[5];
    }
    __syncthreads();
}

// The polygon edge that the discard pass assigns to each of N survivors:
// the first edge meeting its row that it is strictly outside of, or the first
// of all edges outside the rows and in rows that more than four edges meet.
template <int N>
__device__ __forceinline__ void small_edges(const Poly &P, const uint64_t *key, uint16_t *edge, double *dist) {
    double px[N], py[N], dany[N], dmet[N];
    int64_t y0[N], y1[N];
    bool rows[N];
    uint16_t any[N], met[N];
    int nmet[N];
    const int m = P.m < 2 ? 0 : P.m;
#pragma unroll
    for (int j = 0; j < N; j++) {
        const int32_t ky = (int32_t)(key[j] & 0xFFFFFF);
        px[j] = (double)(uint32_t)((key[j] >> 24) & 0xFFFFFF);
        py[j] = (double)ky;
        const uint32_t dy = (uint32_t)(ky - P.ky_lo);
        rows[j] = P.yspan >= 0 && dy <= (uint32_t)P.yspan;
        y0[j] = (int64_t)P.ky_lo + ((int64_t)(dy >> P.shift) << P.shift);
        y1[j] = min(y0[j] + (int64_t(1) << P.shift) - 1, (int64_t)P.ky_lo + P.yspan);
        any[j] = met[j] = RE_NONE;
        dany[j] = dmet[j] = 0.0;
        nmet[j] = 0;
    }
    for (int e = 0; e < m; e++) {
        const double ex = P.ex[e], ey = P.ey[e], ec = P.c[e];
        const int32_t ya = P.vy[e], yb = P.vy[e + 1 < m ? e + 1 : 0];
        const int32_t ylo = min(ya, yb), yhi = max(ya, yb);
#pragma unroll
        for (int j = 0; j < N; j++) {
            const double E = edge_eval(ex, ey, ec, px[j], py[j]);
            const int meets = (int)(ylo <= y1[j]) & (int)(yhi >= y0[j]);
            nmet[j] += meets;
            const bool a = (int)(E < 0) & (int)(any[j] == RE_NONE);
            const bool b = (int)(E < 0) & meets & (int)(met[j] == RE_NONE);
            any[j] = a ? (uint16_t)e : any[j];
            dany[j] = a ? -E : dany[j];
            met[j] = b ? (uint16_t)e : met[j];
            dmet[j] = b ? -E : dmet[j];
        }
    }
#pragma unroll
    for (int j = 0; j < N; j++) {
        const bool use = rows[j] && nmet[j] <= 4;
        edge[j] = use ? met[j] : any[j];
        dist[j] = use ? dmet[j] : dany[j];
    }
}

// A survivor of edge st (below RE_DROP) against the edge's two children: its
// next state, and its distance beyond the child it moves to.
__device__ __forceinline__ uint16_t small_step(const REdge *tab, uint16_t st, uint64_t k, double *dist) {
    const int e0 = 2 * (int)st;
    const double px = (double)(uint32_t)((k >> 24) & 0xFFFFFF), py = (double)(uint32_t)(k & 0xFFFFFF);
    const double E1 = edge_eval(edge_f(tab[e0]), px, py), E2 = edge_eval(edge_f(tab[e0 + 1]), px, py);
    uint16_t out = (E1 > 0 && E2 > 0) ? RE_DROP : RE_NONE;
    *dist = 0.0;
    if (E2 < 0) { out = (uint16_t)(e0 + 1); *dist = -E2; }
    if (E1 < 0) { out = (uint16_t)e0; *dist = -E1; }
    return out;
}

// Position of key k in the hull whose lower chain is lo[0, nl) and upper
// chain up[0, nu), or -1.
__device__ __forceinline__ int small_find(const uint64_t *lo, int nl, const uint64_t *up, int nu, uint64_t k) {
    int a = 0, b = nl;
    while (a < b) {
        const int m = (a + b) >> 1;
        if (lo[m] < k) a = m + 1; else b = m;
    }
    if (a < nl && lo[a] == k) return a;
    a = 1;
    b = nu - 1;
    while (a < b) {
        const int m = (a + b) >> 1;
        if (up[m] < k) a = m + 1; else b = m;
    }
    if (a < nu - 1 && up[a] == k) return nl + (nu - 2 - a);
    return -1;
}

template <int BS>
__global__ __launch_bounds__(BS) void k_small(const float *__restrict__ x, const float *__restrict__ y,
                                              int64_t n_total, int phase, const int64_t *__restrict__ off,
                                              int64_t n1, int preset, Dirs dirs, int nofilter, int refine,
                                              SmallWs ws, uint32_t *__restrict__ hull1,
                                              int64_t *__restrict__ h1, int64_t *__restrict__ counts) {
    constexpr int NW = BS / WAVE;
    __shared__ SmallLds L;
    const int64_t s = blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const uint64_t lt = lanemask_lt();
    const int64_t a = set_begin(off, s), e = max(a, min(set_end(off, n1, s), n_total));
    const int n = (int)(e - a);
    uint64_t *lkey = reinterpret_cast<uint64_t *>(L.raw);
    uint32_t *lidx = reinterpret_cast<uint32_t *>(L.raw + SM_CAP * 8);
    uint16_t *ledge = reinterpret_cast<uint16_t *>(L.raw + SM_CAP * 12);
    if (tid == 0) { L.nsurv = 0; L.ncand = 0; }
    if (tid < SM_COUNTS) L.alive[tid] = 0;
    auto leave = [&]() {
        if (tid == 0) {
            ws.defer[s] = 1;
            ws.hcnt[s] = 0;
        }
        if (tid < SM_COUNTS) ws.scnt[s * SM_COUNTS + tid] = 0;
        for (int k = tid; k < RE_CAP; k += BS) ws.far[s * RE_CAP + k] = 0;
    };
    if (ws.defer) {
        if (s == 0 && tid < ws.nclaim) ws.claims[tid] = 0;
        if (n > SM_TRY) return leave();
        if (tid == 0) ws.defer[s] = 0;
    }

    // Steps 1 and 2
    if (!nofilter) {
        uint32_t *sl = L.sl;
        SlotBest (*wbest)[MAX_SLOTS] = L.wbest;
        switch (preset) {
        case 0: small_extremes<0, BS>(x, y, a, e, dirs, wbest, sl, L.raw); break;
        case 1: small_extremes<1, BS>(x, y, a, e, dirs, wbest, sl, L.raw); break;
        case 2: small_extremes<2, BS>(x, y, a, e, dirs, wbest, sl, L.raw); break;
        case 3: small_extremes<3, BS>(x, y, a, e, dirs, wbest, sl, L.raw); break;
        case 4: small_extremes<4, BS>(x, y, a, e, dirs, wbest, sl, L.raw); break;
        case 5: small_extremes<5, BS>(x, y, a, e, dirs, wbest, sl, L.raw); break;
        case 6: small_extremes<6, BS>(x, y, a, e, dirs, wbest, sl, L.raw); break;
        default: small_extremes<7, BS>(x, y, a, e, dirs, wbest, sl, L.raw); break;
        }
        const int64_t ts = n ? (e - tile_base(a, phase) + TILE - 1) / TILE : 0;
        build_polygon(L.G, sl, x, y, ts, L.P);
        const int m = L.P.m >= 2 ? L.P.m : 0;
        for (int k = tid; k < MAX_SLOTS; k += BS) {
            const int b = k + 1 < m ? k + 1 : 0;
            L.tab[0][k] = k < m ? REdge{L.P.vx[k], L.P.vy[k], L.P.vx[b], L.P.vy[b]} : redge_empty();
            L.far[0][k] = 0;
        }
    }
    __syncthreads();

    // Step 3: the survivors, in any order
    const int m = nofilter ? 0 : L.P.m;
    constexpr int U = 4;              // points per thread and step
    for (int i0 = tid; i0 - tid < n; i0 += U * BS) {
        float fx[U], fy[U];
        double px[U], py[U];
        bool in[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int i = min(i0 + u * BS, n - 1);
            fx[u] = x[a + i];
            fy[u] = y[a + i];
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            px[u] = (double)(int32_t)(fx[u] * GRIDF);
            py[u] = (double)(int32_t)(fy[u] * GRIDF);
            in[u] = m >= 3;
        }
        for (int k = 0; k < m; k++) {
            const double ex = L.P.ex[k], ey = L.P.ey[k], ec = L.P.c[k];
#pragma unroll
            for (int u = 0; u < U; u++) in[u] = (int)in[u] & (int)(edge_eval(ex, ey, ec, px[u], py[u]) > 0);
        }
        uint64_t b[U];
        int total = 0;
#pragma unroll
        for (int u = 0; u < U; u++) {
            b[u] = __ballot(i0 + u * BS < n && !in[u]);
            total += __popcll(b[u]);
        }
        if (!total) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&L.nsurv, total);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int u = 0; u < U; u++) {
            if ((b[u] >> lane) & 1) {
                const int o = at + __popcll(b[u] & lt);
                const uint64_t key = ((uint64_t)((uint32_t)(int32_t)px[u] & 0xFFFFFFu) << 24) |
                                     ((uint32_t)(int32_t)py[u] & 0xFFFFFFu);
                const uint32_t id = (uint32_t)(a + i0 + u * BS);
                if (o < SM_CAP) {
                    lkey[o] = key;
                    lidx[o] = id;
                }
            }
            at += __popcll(b[u]);
        }
    }
    __syncthreads();
    const int K = L.nsurv;
    if (K > SM_CAP) return leave();

    // refinement rounds: the survivors' edges, then per round the children of
    // each edge at its farthest point (k_ref_pass on one block)
    auto rounds = [&]() {
        if (!refine) {
            for (int i = tid; i < K; i += BS) ledge[i] = RE_NONE;
            __syncthreads();
            return;
        }
        for (int i = tid; i < K; i += BS) {
            const uint64_t k = lkey[i];
            double dist;
            uint16_t eo;
            small_edges<1>(L.P, &k, &eo, &dist);
            ledge[i] = eo;
            if (eo != RE_NONE) {
                const unsigned long long fk = far_key(dist, lidx[i]);
                if (L.far[0][eo] < fk) atomicMax(&L.far[0][eo], fk);
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int r = 0; r < REF_ROUNDS; r++) {
            const int p = r & 1, q = 1 - p, er = MAX_SLOTS << r;
            for (int k = tid; k < er; k += BS) {
                REdge c0, c1;
                split_pair(x, y, L.tab[p][k], L.far[p][k], &c0, &c1);
                L.tab[q][2 * k] = c0;
                L.tab[q][2 * k + 1] = c1;
                L.far[q][2 * k] = 0;
                L.far[q][2 * k + 1] = 0;
            }
            __syncthreads();
            int alive = 0;
            for (int i = tid; i < K; i += BS) {
                const uint16_t st = ledge[i];
                if (st == RE_DROP) continue;
                uint16_t out = st;
                if (st < RE_DROP) {
                    double dist;
                    out = small_step(L.tab[q], st, lkey[i], &dist);
                    ledge[i] = out;
                    if (out < RE_DROP) atomicMax(&L.far[q][out], (unsigned long long)far_key(dist, lidx[i]));
                }
                alive += out != RE_DROP;
            }
            alive = (int)wave_sum_i64(alive);
            if (lane == 0 && alive) atomicAdd(&L.alive[r + 1], alive);
            __syncthreads();
        }
    };
    // the same with a thread's survivors in registers; the one that holds an
    // edge's farthest key leaves its point for the split (instead of a read
    // from the inputs each round)
    auto rounds_reg = [&](auto rs) {
        constexpr int RS = decltype(rs)::value;
        uint64_t key[RS], fk[RS];
        uint32_t idx[RS];
        uint16_t st[RS];
        double dist[RS];
#pragma unroll
        for (int j = 0; j < RS; j++) {
            const int i = tid + j * BS;
            key[j] = i < K ? lkey[i] : 0;
            idx[j] = i < K ? lidx[i] : 0;
        }
        small_edges<RS>(L.P, key, st, dist);
#pragma unroll
        for (int j = 0; j < RS; j++) {
            if (tid + j * BS >= K) st[j] = RE_DROP;
            fk[j] = 0;
            if (st[j] < RE_DROP) {
                fk[j] = far_key(dist[j], idx[j]);
                if (L.far[0][st[j]] < fk[j]) atomicMax(&L.far[0][st[j]], (unsigned long long)fk[j]);
            }
        }
#pragma unroll 1
        for (int r = 0; r < REF_ROUNDS; r++) {
            const int p = r & 1, q = 1 - p, er = MAX_SLOTS << r;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < RS; j++)
                if (fk[j] && L.far[p][st[j]] == fk[j]) L.fpt[st[j]] = key[j];
            __syncthreads();
            for (int k = tid; k < er; k += BS) {
                const REdge cur = L.tab[p][k];
                REdge c0 = redge_empty(), c1 = redge_empty();
                if (cur.ax != INT32_MIN) {
                    c0 = cur;
                    if (L.far[p][k]) {
                        const int32_t fx = (int32_t)((L.fpt[k] >> 24) & 0xFFFFFF), fy = (int32_t)(L.fpt[k] & 0xFFFFFF);
                        c0 = REdge{cur.ax, cur.ay, fx, fy};
                        c1 = REdge{fx, fy, cur.bx, cur.by};
                    }
                }
                L.tab[q][2 * k] = c0;
                L.tab[q][2 * k + 1] = c1;
                L.far[q][2 * k] = 0;
                L.far[q][2 * k + 1] = 0;
            }
            __syncthreads();
            int alive = 0;
#pragma unroll
            for (int j = 0; j < RS; j++) {
                fk[j] = 0;
                if (st[j] < RE_DROP) {
                    double d;
                    st[j] = small_step(L.tab[q], st[j], key[j], &d);
                    if (st[j] < RE_DROP) {
                        fk[j] = far_key(d, idx[j]);
                        atomicMax(&L.far[q][st[j]], (unsigned long long)fk[j]);
                    }
                }
                alive += __popcll(__ballot(st[j] != RE_DROP));
            }
            if (lane == 0 && alive) atomicAdd(&L.alive[r + 1], alive);
        }
#pragma unroll
        for (int j = 0; j < RS; j++)
            if (tid + j * BS < K) ledge[tid + j * BS] = st[j];
        __syncthreads();
    };
    if (refine && K <= BS) rounds_reg(std::integral_constant<int, 1>());
    else if (refine && K <= 4 * BS) rounds_reg(std::integral_constant<int, 4>());
    else rounds();

    // candidates: in LDS side by side with a light survivor list, else in the
    // workspace (index and key), the keys back to LDS from there
    const bool light = K <= SM_LIGHT;
    uint64_t *lo = reinterpret_cast<uint64_t *>(light ? L.raw + SM_LIGHT * 8 : L.raw);
    uint64_t *up = reinterpret_cast<uint64_t *>(light ? L.raw + SM_LIGHT * 16 : L.raw + SM_UP);
    for (int i0 = 0; i0 < K; i0 += BS) {
        const int i = i0 + tid;
        const bool keep = i < K && ledge[i] != RE_DROP;
        const uint64_t b = __ballot(keep);
        if (!b) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&L.ncand, __popcll(b));
        at = __builtin_amdgcn_readfirstlane(at) + __popcll(b & lt);
        if (!keep) continue;
        if (light) {
            lo[at] = lkey[i];
        } else {
            ws.ckey[a + at] = lkey[i];
            ws.cidx[a + at] = lidx[i];
        }
    }
    __syncthreads();
    const int M = L.ncand;

    const uint64_t *clo = lo, *cup = up;
    uint32_t *hull_out = off ? ws.hull + a : hull1;
    int pw = 1;
    while (pw < M) pw <<= 1;
    if (light && M <= BS) {       // a rank per thread
        const uint64_t mine = tid < M ? lo[tid] : 0;
        int rank = 0;
#pragma unroll 16
        for (int j = 0; j < M; j++) {
            const uint64_t o = lo[j];
            rank += (int)(o < mine) | ((int)(o == mine) & (int)(j < tid));
        }
        __syncthreads();
        if (tid < M) lo[rank] = mine;
        pw = 0;
    } else if (light) {
        for (int i = M + tid; i < pw; i += BS) lo[i] = ~0ull;
    } else {
        for (int i = tid; i < pw; i += BS) lo[i] = i < M ? ws.ckey[a + i] : ~0ull;
    }
    __syncthreads();
    for (int k = 2; k <= pw; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = tid; t < (pw >> 1); t += BS) {
                const int i = 2 * j * (t / j) + (t % j), l = i + j;
                const bool asc = (i & k) == 0;
                const uint64_t u = lo[i], v = lo[l];
                if ((u > v) == asc) {
                    lo[i] = v;
                    lo[l] = u;
                }
            }
            __syncthreads();
        }
    for (int i = tid; i < M; i += BS) up[i] = lo[i];
    __syncthreads();
    // chains: half the waves take a part of the lower list each, the
    // others of the upper one; then one wave per list the joined parts
    const int nseg = M > 256 ? NW / 2 : 1;
    const int kind = w >= NW / 2, q = w % (NW / 2);
    const int per = ((M + nseg - 1) / nseg + WAVE - 1) / WAVE * WAVE;
    uint64_t *list = kind ? up : lo;
    auto chain = [&](uint64_t *l, int c) { return kind ? list_chain<true, 1, 16>(l, c) : list_chain<false, 1, 16>(l, c); };
    if (q < nseg) {
        const int b0 = min(M, q * per), c = min(M, b0 + per) - b0;
        const int r = chain(list + b0, c);
        if (lane == 0) L.seg[kind][q] = r;
    }
    __syncthreads();
    if (q == 0) {
        const int mine = lane < nseg ? L.seg[kind][lane] : 0;
        int c = (int)wave_sum_i64(mine);
        if (c > 4 * WAVE) {       // long parts; short ones are taken as one list again (2 us less)
            c = kind ? join_pieces<true>(list, per, nseg, mine) : join_pieces<false>(list, per, nseg, mine);
        } else if (nseg > 1) {
            int at = __shfl(mine, 0);
            for (int t = 1; t < nseg; t++) {
                const int b0 = min(M, t * per), ct = __shfl(mine, t);
                for (int i0 = 0; i0 < ct; i0 += WAVE) {   // moved down: at + i <= b0 + i
                    const uint64_t v = i0 + lane < ct ? list[b0 + i0 + lane] : 0;
                    wave_sync();
                    if (i0 + lane < ct) list[at + i0 + lane] = v;
                    wave_sync();
                }
                at += ct;
            }
            c = chain(list, c);
        }
        if (lane == 0) L.seg[kind][0] = c;
    }
    __syncthreads();
    const int nl = L.seg[0][0], nu = L.seg[1][0];
    const int h = (int)hull_size(nl, nu);
    if (!light) {                 // the upper chain behind the lower one makes room for the hull
        for (int i = tid; i < nu; i += BS) lo[nl + i] = up[i];
        cup = lo + nl;
        __syncthreads();
    }
    uint32_t *hull = reinterpret_cast<uint32_t *>(light ? L.raw + SM_LIGHT * 24 : L.raw + SM_UP);
    for (int i = tid; i < h; i += BS) hull[i] = NONE;
    __syncthreads();
    if (light) {
        for (int i = tid; i < K; i += BS) {
            if (ledge[i] == RE_DROP) continue;
            const int p = small_find(clo, nl, cup, nu, lkey[i]);
            if (p >= 0 && p < h) atomicMin(&hull[p], lidx[i]);
        }
    } else {
        for (int i = tid; i < M; i += BS) {
            const int p = small_find(clo, nl, cup, nu, ws.ckey[a + i]);
            if (p >= 0 && p < h) atomicMin(&hull[p], ws.cidx[a + i]);
        }
    }
    __syncthreads();
    for (int i = tid; i < h; i += BS) hull_out[i] = hull[i];
    if (tid == 0) {
        if (off) ws.hcnt[s] = (uint32_t)h;
        else *h1 = h;
    }
    if (tid < SM_COUNTS) {
        const int c = tid == 0 ? K : refine ? L.alive[tid] : -1;
        if (off) ws.scnt[s * SM_COUNTS + tid] = c;
        else counts[tid] = c;
    }
}

// Several sets after k_small: the hull offsets (S + 1), the sets' hulls moved
// to their places, and the summed counts.  Every block (BS threads) scans the
// sizes for the sets it moves (S is at most SM_SETS).  pre: SM_SETS + 1
// entries of LDS, sh: BS / 64.
constexpr int SM_SETS = 2048;

template <int BS>
__device__ __forceinline__ void small_out(const int64_t *__restrict__ off, int64_t S,
                                          const uint32_t *__restrict__ hcnt, const int32_t *__restrict__ scnt,
                                          const uint32_t *__restrict__ tmp, int64_t *__restrict__ hoff,
                                          uint32_t *__restrict__ hull, int64_t *__restrict__ counts, int64_t *pre,
                                          int64_t *sh) {
    constexpr int NW = BS / WAVE;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    int64_t carry = 0;
    for (int64_t b = 0; b < S; b += BS) {
        const int64_t s = b + tid;
        const int64_t c = s < S ? hcnt[s] : 0, inc = wave_incl_scan_i64(c);
        if (lane == WAVE - 1) sh[w] = inc;
        __syncthreads();
        int64_t before = carry;
#pragma unroll
        for (int ww = 0; ww < NW; ww++) {
            before += ww < w ? sh[ww] : 0;
            carry += sh[ww];
        }
        if (s < S) pre[s] = before + inc - c;
        __syncthreads();
    }
    if (tid == 0) pre[S] = carry;
    __syncthreads();
    if (blockIdx.x == 0) {
        for (int64_t s = tid; s <= S; s += BS) hoff[s] = pre[s];
        for (int r = w; r < SM_COUNTS; r += NW) {
            int64_t c = 0, none = 0;
            for (int64_t s = lane; s < S; s += WAVE) {
                const int32_t v = scnt[s * SM_COUNTS + r];
                c += v;
                none |= v < 0;
            }
            c = wave_sum_i64(c);
            if (lane == 0) counts[r] = c;
            if (__ballot(none) && lane == 0) counts[r] = -1;
        }
    }
    for (int64_t s = (int64_t)blockIdx.x * NW + (tid >> 6); s < S; s += (int64_t)gridDim.x * NW) {
        const int64_t a = off[s], o = pre[s], h = pre[s + 1] - o;
        for (int64_t i = lane; i < h; i += WAVE) hull[o + i] = tmp[a + i];
    }
}

__global__ __launch_bounds__(256) void k_small_out(const int64_t *__restrict__ off, int64_t S,
                                                   const uint32_t *__restrict__ hcnt,
                                                   const int32_t *__restrict__ scnt,
                                                   const uint32_t *__restrict__ tmp,
                                                   int64_t *__restrict__ hoff, uint32_t *__restrict__ hull,
                                                   int64_t *__restrict__ counts) {
    __shared__ int64_t sh[5];
    __shared__ int64_t pre[SM_SETS + 1];
    small_out<256>(off, S, hcnt, scnt, tmp, hoff, hull, counts, pre, sh);
}

}  // namespace hg
