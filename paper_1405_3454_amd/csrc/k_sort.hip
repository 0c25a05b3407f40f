// Key-only LSD radix sort of uint64 point keys (8-bit digits, stable per
// pass).  The key count is read from device memory so the whole sort can run
// behind earlier kernels without a host round trip.
//
// One kernel counts the digits of every pass over all keys (the digits'
// starts in each pass's output).  Then one kernel per pass, which reads each
// key once: a block claims the next tile of keys (a counter, so tiles are
// taken in order), holds it in registers, ranks its digits with wave ballots
// and per-wave counters in LDS, publishes the tile's digit counts, sums those
// of the tiles before it by decoupled look-back (a tile's entry holds its own
// counts or, once known, the counts of all tiles up to it), and writes the
// keys out digit by digit through LDS.  Tiles are 6144 keys (of 2^23 keys a
// pass takes 64 us; 4096-key tiles 77, 8192-key tiles 69), 2048 for up to
// 2^20 keys (which would otherwise occupy few CUs).  A pass is bound by its
// scattered writes and the look-back: a copy of the keys takes 26 us; with
// two reads of 2048-key tiles behind eight barriers each it took 102.
//
// The hull stage needs its keys (set, x, y) in order of (set, x) only: among
// points of one x the chains use the lowest and the highest.  So its sort
// skips the three passes over y, and k_sort_ties then orders each run of
// equal (set, x): short runs in place, a long one by its lowest key, copies
// of it, and its highest key (the keys between them are never vertices, and
// the index lookup reads the candidates, not the sorted keys).
#include "hg_device.h"

namespace hg {

constexpr int SORT_THREADS = 512;
constexpr int SORT_WAVES = SORT_THREADS / WAVE;
constexpr int SORT_KPT = 12, SORT_KPT_FEW = 4;          // keys per thread
constexpr int SORT_TILE = SORT_THREADS * SORT_KPT;
constexpr int64_t SORT_FEW = 1 << 20;                   // up to this many keys: small tiles
constexpr int SORT_BLOCKS = 768;
constexpr int RADIX = 256;
constexpr int SORT_SMALL = 4096;      // up to this many keys one block sorts them (k_sort_small)
constexpr int SMALL_THREADS = 1024;
constexpr int SMALL_CLEAR_BLOCKS = 32;  // k_sort_small's blocks after the first: clear the passes' state
constexpr int Y_DIGITS = 3;             // the low digits, which the hull stage's sort skips

// Several sets of more than 1024 candidates in all are sorted set by set: 256
// sets of about 16 candidates in 9 us, where one block took 47 for all 4000.
__device__ __forceinline__ int64_t sort_small(const int *seg_fallback) {
    return seg_fallback ? SMALL_THREADS : SORT_SMALL;
}
__host__ __device__ __forceinline__ int64_t sort_tile(int64_t count) {
    return count <= SORT_FEW ? SORT_THREADS * SORT_KPT_FEW : SORT_TILE;
}
__host__ __device__ __forceinline__ int64_t sort_tiles(int64_t count) {
    return (count + sort_tile(count) - 1) / sort_tile(count);
}
// Most tiles of any count up to n.
__host__ __device__ __forceinline__ int64_t sort_tiles_max(int64_t n) {
    const int64_t few = n < SORT_FEW ? n : SORT_FEW;
    const int64_t a = sort_tiles(few), b = sort_tiles(n);
    return (a > b ? a : b) + 1;
}

// Tile look-back entries: pass tag (pass + 1) << 56 | state << 54 | value,
// 0 = not yet written this call.
constexpr uint64_t LB_AGG = 1ull << 54, LB_INC = 2ull << 54;
constexpr uint64_t LB_VAL = (1ull << 54) - 1, LB_TAG = ~((1ull << 56) - 1);
constexpr int SORT_MAX_PASSES = 8;

// The passes' shared state: digit totals, tile counters, and the long runs.
struct SortState {
    uint32_t total[SORT_MAX_PASSES][RADIX];
    uint32_t claim[SORT_MAX_PASSES];
    uint32_t nlong[2];                   // long runs: a wave's, a block's
    unsigned long long huge;             // and everyone's: runs << 32 | parts of them
    uint32_t part, done;                 // parts claimed, and finished
};

// P keys in LDS (a power of two, at least 256) sorted by the 1024 threads of a
// block.  Every wave ranks its 64 keys; then, up to 1024 keys, each key is
// searched for in all the other runs of 64, four at a time, and goes to its
// place at once; above, runs are merged in pairs, each key searched for in the
// other run of its pair and moved to its own index plus what is below it there
// (ties: the first run's first).  A bitonic network's barriers, log2(P)
// (log2(P) + 1) / 2 of them, bound it before: 4096 sets of 600 keys took 103 us,
// now 65 (73 with merges from 16 keys on, whose searches wait for one another); one
// list of 4000 keys 50, now 23.
__host__ __device__ __forceinline__ int sort_width(int n) {
    int P = 4 * WAVE;
    while (P < n) P <<= 1;
    return P;
}
// The place of mine (key tid & 63 of the run at w0) in its run of 64 keys.
__device__ __forceinline__ int run_rank(const uint64_t *b, int w0, uint64_t mine, int me) {
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < WAVE; j++) {
        const uint64_t o = b[w0 + j];
        rank += (int)(o < mine) | ((int)(o == mine) & (int)(j < me));
    }
    return rank;
}
// Keys of a later run come after equal ones of an earlier one: they are
// searched for as key + 1.  Not padding (no key has its set field, 65535),
// which may then land on padding: the places it leaves, beyond every key,
// hold padding.
__device__ __forceinline__ uint64_t search_key(uint64_t k, bool later) {
    return k + (uint64_t)(later && k != ~0ull);
}
__device__ __forceinline__ void sort_1024(uint64_t *b, int P) {
    const int tid = threadIdx.x, w0 = tid & ~(WAVE - 1);
    const bool on = tid < P;
    const uint64_t mine = on ? b[tid] : 0;
    int rank = 0;
    if (on) {
        rank = run_rank(b, w0, mine, tid - w0);
        wave_sync();
        b[w0 + rank] = mine;
    }
    __syncthreads();
    if (on)
        for (int r0 = 0; r0 < P; r0 += 4 * WAVE) {
            int pos[4] = {0, 0, 0, 0};
#pragma unroll
            for (int step = WAVE / 2; step > 0; step >>= 1)
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int r = r0 + u * WAVE;
                    pos[u] += b[r + pos[u] + step - 1] < search_key(mine, r < w0) ? step : 0;
                }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int r = r0 + u * WAVE;
                pos[u] += b[r + pos[u]] < search_key(mine, r < w0) ? 1 : 0;
                rank += r == w0 ? 0 : pos[u];
            }
        }
    __syncthreads();
    if (on) b[rank] = mine;
    __syncthreads();
}
template <int K>
__device__ __forceinline__ void merge_1024(uint64_t *b) {     // P = K * 1024
    const int tid = threadIdx.x;
    uint64_t k[K], lim[K];
    int pos[K];
#pragma unroll
    for (int i = 0; i < K; i++) {
        const int w0 = (tid & ~(WAVE - 1)) + i * SMALL_THREADS, me = tid & (WAVE - 1);
        k[i] = b[w0 + me];
        pos[i] = run_rank(b, w0, k[i], me);
        wave_sync();
        b[w0 + pos[i]] = k[i];
    }
    for (int run = WAVE; run < K * SMALL_THREADS; run <<= 1) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < K; i++) {
            const int at = tid + i * SMALL_THREADS;
            k[i] = b[at];
            lim[i] = search_key(k[i], (at & run) != 0);
            pos[i] = 0;
        }
        for (int step = run >> 1; step > 0; step >>= 1)
#pragma unroll
            for (int i = 0; i < K; i++) {
                const int sib = ((tid + i * SMALL_THREADS) & ~(run - 1)) ^ run;
                pos[i] += b[sib + pos[i] + step - 1] < lim[i] ? step : 0;
            }
#pragma unroll
        for (int i = 0; i < K; i++) {
            const int sib = ((tid + i * SMALL_THREADS) & ~(run - 1)) ^ run;
            pos[i] += b[sib + pos[i]] < lim[i] ? 1 : 0;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < K; i++) {
            const int at = tid + i * SMALL_THREADS;
            b[(at & ~(2 * run - 1)) + (at & (run - 1)) + pos[i]] = k[i];
        }
    }
    __syncthreads();
}
template <int PMAX>
__device__ __forceinline__ void block_sort(uint64_t *b, int P) {
    if (P <= SMALL_THREADS) sort_1024(b, P);
    else if (P == 2 * SMALL_THREADS) merge_1024<2>(b);
    else if (P == 4 * SMALL_THREADS || PMAX == 4 * SMALL_THREADS) merge_1024<4>(b);
    else if constexpr (PMAX > 4 * SMALL_THREADS) merge_1024<8>(b);
}

// At most SORT_SMALL keys: block 0 sorts them in LDS, padded with the largest
// key, and writes them where the radix passes would have left them; the
// passes then return at once.  Above SORT_SMALL the other blocks clear the
// passes' state and the look-back entries of the tiles.  The sort is by key
// only, so equal keys are interchangeable.
__global__ __launch_bounds__(SMALL_THREADS) void k_sort_small(const uint64_t *__restrict__ keys,
                                                              const int64_t *__restrict__ cnt_ptr,
                                                              uint64_t *__restrict__ out,
                                                              unsigned long long *__restrict__ status,
                                                              SortState *__restrict__ state,
                                                              int *__restrict__ seg_fallback) {
    __shared__ uint64_t b[SORT_SMALL];
    const int64_t count = *cnt_ptr;
    const int tid = threadIdx.x;
    if (seg_fallback && blockIdx.x == 0 && tid == 0) *seg_fallback = 0;
    if (count > sort_small(seg_fallback)) {
        if (blockIdx.x == 0) return;
        const int64_t nst = sort_tiles(count) * RADIX;
        const int64_t nt = (int64_t)(gridDim.x - 1) * SMALL_THREADS;
        for (int64_t i = (int64_t)(blockIdx.x - 1) * SMALL_THREADS + tid; i < nst; i += nt) status[i] = 0;
        if (blockIdx.x == 1)
            for (int i = tid; i < (int)(sizeof(SortState) / 4); i += SMALL_THREADS)
                reinterpret_cast<uint32_t *>(state)[i] = 0;
        return;
    }
    if (blockIdx.x != 0 || count <= 0) return;
    const int n = (int)count;
    const int P = sort_width(n);
    for (int i = tid; i < P; i += SMALL_THREADS) b[i] = i < n ? keys[i] : ~0ull;
    __syncthreads();
    block_sort<SORT_SMALL>(b, P);
    for (int i = tid; i < n; i += SMALL_THREADS) out[i] = b[i];
}

// Several sets.  The candidates of the hull stage arrive grouped by set in
// ascending set order (the filter's regions follow the tiles, and the tiles
// follow the sets), so each set can be sorted alone: start[s] = the first
// candidate of set s for s = 0..S (start[S] = n), from the keys' set field;
// a key whose set is below its predecessor's raises SEG_UNORDERED in
// *fallback, and the radix passes then sort everything.  Without it the
// starts are also the sets' ranges in the sorted keys (the sort keeps each
// set's range), which the chain stage reads.
constexpr int SEG_TOO_BIG = 1, SEG_UNORDERED = 2;

__global__ __launch_bounds__(256) void k_set_starts(const uint64_t *__restrict__ keys,
                                                    const int64_t *__restrict__ cnt_ptr, int64_t S,
                                                    int64_t *__restrict__ start, int *__restrict__ fallback) {
    const int64_t n = *cnt_ptr;
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i <= n;
         i += int64_t(gridDim.x) * blockDim.x) {
        const int64_t prev = i == 0 ? -1 : (int64_t)(keys[i - 1] >> 48);
        const int64_t cur = i == n ? S : (int64_t)(keys[i] >> 48);
        if (cur < prev) atomicOr(fallback, SEG_UNORDERED);
        for (int64_t t = prev + 1; t <= cur && t <= S; t++) start[t] = i;
    }
}

constexpr int SEG_THREADS = 1024, SEG_WAVES = SEG_THREADS / WAVE;
constexpr int SEG_MAX = 8192;         // keys of one set a block sorts in LDS (64 KB)

// Each set's range [start[s], start[s + 1]) sorted in LDS into out, where the
// radix passes would have left it: up to 64 keys by one wave (a block's
// barriers and its 256 places bound thousands of such sets: 3000 sets of some
// 50 candidates 33 us, now 6), more by one block; block b takes the sets b, b +
// gridDim.x, ...  A set of more than SEG_MAX keys, or a key in a range that is
// not its set's, raises *fallback.
__global__ __launch_bounds__(SEG_THREADS, 8) void k_sort_sets(const uint64_t *__restrict__ keys,
                                                           const int64_t *__restrict__ cnt_ptr, int64_t S,
                                                           const int64_t *__restrict__ start,
                                                           uint64_t *__restrict__ out,
                                                           int *__restrict__ fallback) {
    __shared__ uint64_t b[SEG_MAX];
    __shared__ int bad;
    const int64_t n = *cnt_ptr;
    if (n <= sort_small(fallback)) return;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    for (int64_t s = (int64_t)blockIdx.x * SEG_WAVES + w; s < S; s += (int64_t)gridDim.x * SEG_WAVES) {
        const int64_t a = start[s], m = start[s + 1] - a;
        if (m <= 0 || m > WAVE) continue;
        const uint64_t k = lane < m ? keys[a + lane] : ~0ull;
        if (__ballot(lane < m && (int64_t)(k >> 48) != s)) {
            if (lane == 0) atomicOr(fallback, SEG_UNORDERED);
            continue;
        }
        b[w * WAVE + lane] = k;
        wave_sync();
        const int rank = run_rank(b, w * WAVE, k, lane);
        if (lane < m) out[a + rank] = k;
        wave_sync();
    }
    __syncthreads();
    for (int64_t s = blockIdx.x; s < S; s += gridDim.x) {
        const int64_t a = start[s], e = start[s + 1];
        if (e - a <= WAVE) continue;
        if (e - a > SEG_MAX) {
            if (tid == 0) atomicOr(fallback, SEG_TOO_BIG);
            continue;
        }
        const int m = (int)(e - a);
        const int P = sort_width(m);
        if (tid == 0) bad = 0;
        __syncthreads();
        for (int i = tid; i < P; i += SEG_THREADS) {
            const uint64_t k = i < m ? keys[a + i] : ~0ull;
            if (i < m && (int64_t)(k >> 48) != s) bad = 1;
            b[i] = k;
        }
        __syncthreads();
        if (bad) {
            if (tid == 0) atomicOr(fallback, SEG_UNORDERED);
            __syncthreads();
            continue;
        }
        block_sort<SEG_MAX>(b, P);
        for (int i = tid; i < m; i += SEG_THREADS) out[a + i] = b[i];
        __syncthreads();      // b is refilled for the next set
    }
}

// Digit totals of the passes (digits first .. first + passes - 1) over all
// keys, into state->total (cleared by k_sort_small): each block counts in LDS
// and adds its counts at the end.
__global__ __launch_bounds__(SORT_THREADS) void k_sort_prep(const uint64_t *__restrict__ keys,
                                                            const int64_t *__restrict__ cnt_ptr, int first,
                                                            int passes, SortState *__restrict__ state,
                                                            const int *__restrict__ seg_fallback) {
    __shared__ uint32_t h[SORT_MAX_PASSES][RADIX];
    const int tid = threadIdx.x;
    const int64_t count = *cnt_ptr;
    if (count <= sort_small(seg_fallback)) return;
    if (seg_fallback && *seg_fallback == 0) return;    // k_sort_sets has sorted every set
    constexpr int U = 8, STEP = SORT_THREADS * U;
    if ((int64_t)blockIdx.x * STEP >= count) return;
    for (int i = tid; i < passes * RADIX; i += SORT_THREADS) h[i / RADIX][i % RADIX] = 0;
    __syncthreads();
    for (int64_t base = (int64_t)blockIdx.x * STEP; base < count; base += (int64_t)gridDim.x * STEP) {
        uint64_t k[U];
#pragma unroll
        for (int r = 0; r < U; r++) {
            const int64_t i = base + r * SORT_THREADS + tid;
            k[r] = i < count ? keys[i] : 0;
        }
#pragma unroll
        for (int r = 0; r < U; r++) {
            if (base + r * SORT_THREADS + tid >= count) continue;
            for (int ps = 0; ps < passes; ps++)
                atomicAdd(&h[ps][(uint32_t)(k[r] >> (8 * (first + ps))) & (RADIX - 1)], 1u);
        }
    }
    __syncthreads();
    for (int i = tid; i < passes * RADIX; i += SORT_THREADS)
        if (h[i / RADIX][i % RADIX]) atomicAdd(&state->total[i / RADIX][i % RADIX], h[i / RADIX][i % RADIX]);
}

// Sum of the digit-d counts of the tiles before tile r (thread d), from their
// look-back entries: an entry with the tile's own counts (LB_AGG) is added
// and the walk goes on, one with the counts up to and including that tile
// (LB_INC) ends it; an entry not yet written this pass is read again.  Tiles
// are claimed in order by running blocks, and each publishes its own counts
// before it looks back, so every wait ends.
__device__ __forceinline__ int64_t look_back(const unsigned long long *__restrict__ status, int64_t r,
                                             int d, uint64_t tag) {
    constexpr int LB = 16;
    int64_t excl = 0;
    int64_t k = r - 1;
    while (k >= 0) {
        uint64_t v[LB];
#pragma unroll
        for (int i = 0; i < LB; i++)
            v[i] = k - i >= 0 ? __hip_atomic_load(&status[(k - i) * RADIX + d], __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT)
                              : 0;
        int used = 0;
        bool done = false;
#pragma unroll
        for (int i = 0; i < LB; i++) {
            if (done || used < i || k - i < 0) continue;
            if ((v[i] & LB_TAG) != tag) continue;     // not written yet: read it again
            excl += (int64_t)(v[i] & LB_VAL);
            used = i + 1;
            if (v[i] & LB_INC) done = true;
        }
        if (done) break;
        k -= used;
        if (used == 0) __builtin_amdgcn_s_sleep(1);
    }
    return excl;
}

struct SortLds {
    uint64_t buf[SORT_TILE];
    uint32_t wcnt[SORT_WAVES][RADIX];    // a wave's digit counts, then its starts in the tile
    uint32_t dstart[RADIX];              // the tile's digits' starts
    int64_t run[RADIX];                  // digit d's output position less its start in the tile
    uint32_t wsum[SORT_WAVES];
    int64_t tile;
};

// One tile of at most SORT_THREADS * KPT keys.  A wave's keys are its
// consecutive KPT * 64, row by row, so ranks in (wave, row, lane) order keep
// the input order of equal digits.
template <int KPT>
__device__ __forceinline__ void sort_one_tile(SortLds &L, const uint64_t *__restrict__ in, int64_t base, int n,
                                              int64_t t, int shift, uint64_t tag, int64_t start,
                                              unsigned long long *__restrict__ status,
                                              uint64_t *__restrict__ out) {
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const uint64_t lt = lanemask_lt();
    const int o0 = w * KPT * WAVE + lane;
    uint64_t k[KPT];
    uint32_t rank[KPT];
#pragma unroll
    for (int r = 0; r < KPT; r++) {
        const int i = o0 + r * WAVE;
        k[r] = i < n ? in[base + i] : 0;
    }
    for (int i = tid; i < SORT_WAVES * RADIX; i += SORT_THREADS) L.wcnt[i / RADIX][i % RADIX] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < KPT; r++) {
        const bool has = o0 + r * WAVE < n;
        const uint32_t d = (uint32_t)(k[r] >> shift) & (RADIX - 1);
        uint64_t peers = __ballot(has);
#pragma unroll
        for (int b = 0; b < 8; b++) {
            const bool bit = (d >> b) & 1;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        // every lane of a digit reads the wave's count, its first lane raises it
        const uint32_t old = L.wcnt[w][d];
        rank[r] = old + (uint32_t)__popcll(peers & lt);
        wave_sync();
        if (has && (peers & lt) == 0) L.wcnt[w][d] = old + (uint32_t)__popcll(peers);
        wave_sync();
    }
    __syncthreads();
    uint32_t mine = 0;                   // digit tid's keys in the tile
    if (tid < RADIX) {
#pragma unroll
        for (int ww = 0; ww < SORT_WAVES; ww++) mine += L.wcnt[ww][tid];
        __hip_atomic_store(&status[t * RADIX + tid], tag | (t ? LB_AGG : LB_INC) | mine, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    uint32_t inc = mine;                 // the digits' starts in the tile
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const uint32_t v = __shfl_up(inc, o);
        if (lane >= o) inc += v;
    }
    if (lane == WAVE - 1) L.wsum[w] = inc;
    __syncthreads();
    if (tid < RADIX) {
        uint32_t at = inc - mine;
        for (int ww = 0; ww < w; ww++) at += L.wsum[ww];
        L.dstart[tid] = at;
#pragma unroll
        for (int ww = 0; ww < SORT_WAVES; ww++) {
            const uint32_t c = L.wcnt[ww][tid];
            L.wcnt[ww][tid] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < KPT; r++)
        if (o0 + r * WAVE < n) L.buf[L.wcnt[w][(uint32_t)(k[r] >> shift) & (RADIX - 1)] + rank[r]] = k[r];
    if (tid < RADIX) {
        int64_t excl = 0;
        if (t) {
            excl = look_back(status, t, tid, tag);
            __hip_atomic_store(&status[t * RADIX + tid], tag | LB_INC | (uint64_t)(excl + mine), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
        L.run[tid] = start + excl - (int64_t)L.dstart[tid];
    }
    __syncthreads();
#pragma unroll 4
    for (int i = tid; i < n; i += SORT_THREADS) {
        const uint64_t kk = L.buf[i];
        out[L.run[(uint32_t)(kk >> shift) & (RADIX - 1)] + i] = kk;
    }
}

// Pass `pass` by digit `digit`.
__global__ __launch_bounds__(SORT_THREADS) void k_sort_pass(const uint64_t *__restrict__ in,
                                                            const int64_t *__restrict__ cnt_ptr, int pass,
                                                            int digit, SortState *__restrict__ state,
                                                            unsigned long long *__restrict__ status,
                                                            uint64_t *__restrict__ out,
                                                            const int *__restrict__ seg_fallback) {
    __shared__ SortLds L;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const int64_t count = *cnt_ptr;
    if (count <= sort_small(seg_fallback)) return;     // k_sort_small has sorted them
    if (seg_fallback && *seg_fallback == 0) return;    // k_sort_sets has sorted every set
    const int64_t tiles = sort_tiles(count), tile = sort_tile(count);
    if ((int64_t)blockIdx.x >= tiles) return;
    // digit tid's start in the output
    int64_t start = 0;
    {
        const int64_t c = tid < RADIX ? (int64_t)state->total[pass][tid] : 0;
        const int64_t inc = wave_incl_scan_i64(c);
        if (lane == WAVE - 1) L.run[w] = inc;
        __syncthreads();
        start = inc - c;
        for (int ww = 0; ww < w; ww++) start += L.run[ww];
    }
    const uint64_t tag = (uint64_t)(pass + 1) << 56;
    for (;;) {
        __syncthreads();                 // the previous tile is done with L
        if (tid == 0) L.tile = (int64_t)atomicAdd(&state->claim[pass], 1u);
        __syncthreads();
        const int64_t t = L.tile;
        if (t >= tiles) return;
        const int64_t base = t * tile;
        const int n = (int)min(tile, count - base);
        if (tile == SORT_TILE) sort_one_tile<SORT_KPT>(L, in, base, n, t, 8 * digit, tag, start, status, out);
        else sort_one_tile<SORT_KPT_FEW>(L, in, base, n, t, 8 * digit, tag, start, status, out);
    }
}

// Runs of equal (set, x) in keys sorted by (set, x).  The chains need of a run
// its lowest and its highest key, so it becomes its lowest key, copies of it,
// and its highest: in LDS a run of up to TIE_THREAD keys by the thread at its
// head and one of up to TIE_SHORT by a wave (a thread walks 250 keys in 60
// us), a longer one by k_sort_long, which finds it in a list.  A list entry
// is an atomic on one counter, about 9 ns each, so few runs may need one: with
// 2^27 clamped normal points (about 30 keys a run) and runs of up to 16 sorted
// by their threads and longer ones listed this took 38.1 ms, now 1.2; with
// 2^27 points of a square (8 a run) 5.7 ms, now 0.9.
constexpr int TIE_THREAD = 32, TIE_SHORT = 256;
constexpr int TIE_STEP = 4;              // keys read together along a run
constexpr int64_t TIE_WAVE = 1 << 12, TIE_BLOCK = 1 << 18;
constexpr int64_t TIE_PART = 1 << 15;    // keys of a run above TIE_BLOCK that a block takes at once
struct LongRun {
    int64_t a, e;                        // keys [a, e)
    unsigned long long lo, hi;
    int64_t first;                       // everyone's: the number of its first part
};
// The lists' parts: everyone's runs (over TIE_BLOCK keys), a block's, a wave's.
__device__ __forceinline__ LongRun *tie_list(LongRun *runs, int64_t n, int kind) {
    const int64_t all = n / TIE_BLOCK + 1, block = n / TIE_WAVE + 1;
    return runs + (kind == 2 ? 0 : kind == 1 ? all : all + block);
}

// A block takes TIE_TILE keys through LDS (with the key before and those
// after them); the runs that start in the tile are its own, and it writes
// back what it changed.  Blocks compare only the (set, x) of keys that are not
// theirs, which every order of a run keeps.
constexpr int TIE_TILE = 2048;

__global__ __launch_bounds__(256) void k_sort_ties(uint64_t *__restrict__ keys,
                                                   const int64_t *__restrict__ cnt_ptr,
                                                   SortState *__restrict__ state, LongRun *__restrict__ runs,
                                                   const int *__restrict__ seg_fallback) {
    constexpr int TW = TIE_TILE + TIE_SHORT + TIE_STEP + 1;
    constexpr uint32_t Y = (1u << (8 * Y_DIGITS)) - 1;
    __shared__ uint64_t k[TW];                   // k[j]: key base - 1 + j
    __shared__ uint16_t heads[TIE_TILE / TIE_THREAD];   // where runs of more than TIE_THREAD keys start
    __shared__ int nheads;
    const int64_t n = *cnt_ptr;
    if (n <= sort_small(seg_fallback)) return;
    if (seg_fallback && *seg_fallback == 0) return;
    const int tid = threadIdx.x, lane = lane_id();
    for (int64_t base = (int64_t)blockIdx.x * TIE_TILE; base < n; base += (int64_t)gridDim.x * TIE_TILE) {
        __syncthreads();
        constexpr int U = (TW + 255) / 256;
        uint64_t v[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t i = base - 1 + tid + u * 256;
            v[u] = i >= 0 && i < n && tid + u * 256 < TW ? keys[i] : ~0ull;       // no key's (set, x)
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (tid + u * 256 < TW) k[tid + u * 256] = v[u];
        if (tid == 0) nheads = 0;
        __syncthreads();
        for (int t = tid; t < TIE_TILE && base + t < n; t += 256) {
            const int j = t + 1;
            const uint64_t g = k[j] >> (8 * Y_DIGITS);
            if ((k[j + 1] >> (8 * Y_DIGITS)) != g || (k[j - 1] >> (8 * Y_DIGITS)) == g) continue;
            uint32_t ylo = (uint32_t)k[j] & Y, yhi = ylo;
            int len = 1;
            for (bool more = true; more;) {
                uint64_t c[TIE_STEP];
#pragma unroll
                for (int u = 0; u < TIE_STEP; u++) c[u] = k[j + len + u];
#pragma unroll
                for (int u = 0; u < TIE_STEP; u++) {
                    more = more & ((c[u] >> (8 * Y_DIGITS)) == g);
                    const uint32_t y = (uint32_t)c[u] & Y;
                    ylo = more ? min(ylo, y) : ylo;
                    yhi = more ? max(yhi, y) : yhi;
                    len += more;
                }
                more = more & (len <= TIE_THREAD);
            }
            if (len > TIE_THREAD) {
                heads[atomicAdd(&nheads, 1)] = (uint16_t)t;
                continue;
            }
            const uint64_t low = g << (8 * Y_DIGITS) | ylo;
            for (int q = 0; q < len - 1; q++) k[j + q] = low;
            k[j + len - 1] = g << (8 * Y_DIGITS) | yhi;
        }
        __syncthreads();
        for (int h = tid >> 6; h < nheads; h += 256 / WAVE) {
            const int t = heads[h], j = t + 1;
            const uint64_t g = k[j] >> (8 * Y_DIGITS);
            uint32_t ylo = Y, yhi = 0;
            int len = 0;
            for (bool more = true; more && len <= TIE_SHORT;) {
                const int i = j + len + lane;
                const uint64_t c = i < TW ? k[i] : ~0ull;
                const uint64_t in = __ballot((c >> (8 * Y_DIGITS)) == g);
                const int m = ~in ? __builtin_ctzll(~in) : WAVE;
                if (lane < m) {
                    ylo = min(ylo, (uint32_t)c & Y);
                    yhi = max(yhi, (uint32_t)c & Y);
                }
                len += m;
                more = m == WAVE;
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                ylo = min(ylo, (uint32_t)__shfl_xor((int)ylo, o));
                yhi = max(yhi, (uint32_t)__shfl_xor((int)yhi, o));
            }
            if (len <= TIE_SHORT) {
                for (int q = lane; q < len; q += WAVE) k[j + q] = g << (8 * Y_DIGITS) | (q == len - 1 ? yhi : ylo);
            } else if (lane == 0) {
                const int64_t i = base + t;
                int64_t lo = i + TIE_SHORT, hi = n;  // the first key past the run
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if ((keys[mid] >> (8 * Y_DIGITS)) == g) lo = mid + 1; else hi = mid;
                }
                const int64_t m = lo - i;
                if (m > TIE_BLOCK) {
                    const uint64_t at = atomicAdd(&state->huge, 1ull << 32 | (uint64_t)((m + TIE_PART - 1) / TIE_PART));
                    tie_list(runs, n, 2)[at >> 32] = LongRun{i, lo, ~0ull, 0ull, (int64_t)(uint32_t)at};
                } else {
                    const int kind = m > TIE_WAVE ? 1 : 0;
                    tie_list(runs, n, kind)[atomicAdd(&state->nlong[kind], 1u)] = LongRun{i, lo, ~0ull, 0ull, 0};
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int t = tid + u * 256;
            if (t < TW && k[t] != v[u]) keys[base - 1 + t] = k[t];
        }
    }
}

// The long runs: lowest key, copies of it, highest key.  Up to TIE_WAVE keys
// a wave takes a run, up to TIE_BLOCK a block.  All blocks share the parts of
// the longer ones: parts are claimed in order for their extremes, and once all
// are finished the blocks write them.  (A claimed part is in the hands of a
// running block, so the wait for it ends however many blocks run.  With the
// last block to finish writing every such run alone, 2^26 points of one x took
// 10.1 ms, now 3.3.)
constexpr int TIE_THREADS = 512;

__global__ __launch_bounds__(TIE_THREADS) void k_sort_long(uint64_t *__restrict__ keys,
                                                           const int64_t *__restrict__ cnt_ptr,
                                                           SortState *__restrict__ state,
                                                           LongRun *__restrict__ runs,
                                                           const int *__restrict__ seg_fallback) {
    __shared__ unsigned long long lo, hi;
    __shared__ uint32_t claimed;
    const int64_t n = *cnt_ptr;
    if (n <= sort_small(seg_fallback)) return;
    if (seg_fallback && *seg_fallback == 0) return;
    const int tid = threadIdx.x, lane = lane_id();
    // lowest and highest of keys a + t, a + t + step, ... below e, over a wave
    auto wave_extremes = [&](int64_t a, int64_t e, int t, int step, unsigned long long *l, unsigned long long *h) {
        unsigned long long l1 = ~0ull, h1 = 0ull;
        for (int64_t i = a + t; i < e; i += step) {
            const unsigned long long k = keys[i];
            l1 = k < l1 ? k : l1;
            h1 = k > h1 ? k : h1;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const unsigned long long l2 = __shfl_xor(l1, o), h2 = __shfl_xor(h1, o);
            l1 = l2 < l1 ? l2 : l1;
            h1 = h2 > h1 ? h2 : h1;
        }
        *l = l1;
        *h = h1;
    };
    auto fill = [&](int64_t a, int64_t e, int t, int step, uint64_t l, uint64_t h) {
        for (int64_t i = a + t; i < e; i += step) keys[i] = i == e - 1 ? h : l;
    };
    auto block_extremes = [&](int64_t a, int64_t e) {
        __syncthreads();
        if (tid == 0) { lo = ~0ull; hi = 0ull; }
        __syncthreads();
        unsigned long long l, h;
        wave_extremes(a, e, tid, TIE_THREADS, &l, &h);
        if (lane == 0) {
            atomicMin(&lo, l);
            atomicMax(&hi, h);
        }
        __syncthreads();
    };
    const uint32_t nw = state->nlong[0], nb = state->nlong[1], np = (uint32_t)state->huge;
    const LongRun *R = tie_list(runs, n, 0);
    constexpr int WPB = TIE_THREADS / WAVE;
    for (uint32_t r = blockIdx.x * WPB + (tid >> 6); r < nw; r += gridDim.x * WPB) {
        const int64_t a = R[r].a, e = R[r].e;
        unsigned long long l, h;
        wave_extremes(a, e, lane, WAVE, &l, &h);
        fill(a, e, lane, WAVE, l, h);
    }
    R = tie_list(runs, n, 1);
    for (uint32_t r = blockIdx.x; r < nb; r += gridDim.x) {
        const int64_t a = R[r].a, e = R[r].e;
        block_extremes(a, e);
        fill(a, e, tid, TIE_THREADS, lo, hi);
    }
    if (np == 0) return;
    LongRun *H = tie_list(runs, n, 2);
    const int64_t na = (int64_t)(state->huge >> 32);
    // the run that part t belongs to, and the part's keys
    auto part_of = [&](uint32_t t, int64_t *pa, int64_t *pe) {
        int64_t r = 0, h = na - 1;
        while (r < h) {
            const int64_t mid = (r + h + 1) >> 1;
            if (H[mid].first <= (int64_t)t) r = mid; else h = mid - 1;
        }
        *pa = H[r].a + (t - H[r].first) * TIE_PART;
        *pe = min(H[r].e, *pa + TIE_PART);
        return r;
    };
    for (;;) {
        __syncthreads();
        if (tid == 0) claimed = atomicAdd(&state->part, 1u);
        __syncthreads();
        const uint32_t t = claimed;
        if (t >= np) break;
        int64_t pa, pe;
        const int64_t r = part_of(t, &pa, &pe);
        block_extremes(pa, pe);
        if (tid == 0) {
            atomicMin(&H[r].lo, lo);
            atomicMax(&H[r].hi, hi);
            __threadfence();
            atomicAdd(&state->done, 1u);
        }
    }
    if (tid == 0)
        while (__hip_atomic_load(&state->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < np)
            __builtin_amdgcn_s_sleep(8);
    __syncthreads();
    __threadfence();
    for (uint32_t t = blockIdx.x; t < np; t += gridDim.x) {
        int64_t pa, pe;
        const int64_t r = part_of(t, &pa, &pe);
        const uint64_t l = __hip_atomic_load(&H[r].lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t h = __hip_atomic_load(&H[r].hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int64_t i = pa + tid; i < pe; i += TIE_THREADS) keys[i] = i == H[r].e - 1 ? h : l;
    }
}

}  // namespace hg
