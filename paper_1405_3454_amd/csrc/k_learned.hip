// Learned direction proposal (this project's extension, not the paper's):
// a 32 x 32 occupancy histogram of each set feeds a small MLP that scores 64
// candidate directions; the eight best are added to the fixed extremes.
// Extra extremes can only enlarge the filter polygon inside the hull, so the
// hull never depends on the network.
#include "hg_device.h"

namespace hg {

constexpr int NCAND = 64;

// Candidate directions phi_d = 2 pi d / 64 as correctly rounded binary64
// (cos, sin); multiples of 90 degrees are exact.
static const double kCandCos[NCAND] = {
    0x1.0000000000000p+0, 0x1.fd88da3d12526p-1, 0x1.f6297cff75cb0p-1, 0x1.e9f4156c62ddap-1,
    0x1.d906bcf328d46p-1, 0x1.c38b2f180bdb1p-1, 0x1.a9b66290ea1a3p-1, 0x1.8bc806b151741p-1,
    0x1.6a09e667f3bcdp-1, 0x1.44cf325091dd6p-1, 0x1.1c73b39ae68c8p-1, 0x1.e2b5d3806f63bp-2,
    0x1.87de2a6aea963p-2, 0x1.294062ed59f06p-2, 0x1.8f8b83c69a60bp-3, 0x1.917a6bc29b42cp-4,
    0.0, -0x1.917a6bc29b42cp-4, -0x1.8f8b83c69a60bp-3, -0x1.294062ed59f06p-2,
    -0x1.87de2a6aea963p-2, -0x1.e2b5d3806f63bp-2, -0x1.1c73b39ae68c8p-1, -0x1.44cf325091dd6p-1,
    -0x1.6a09e667f3bcdp-1, -0x1.8bc806b151741p-1, -0x1.a9b66290ea1a3p-1, -0x1.c38b2f180bdb1p-1,
    -0x1.d906bcf328d46p-1, -0x1.e9f4156c62ddap-1, -0x1.f6297cff75cb0p-1, -0x1.fd88da3d12526p-1,
    -0x1.0000000000000p+0, -0x1.fd88da3d12526p-1, -0x1.f6297cff75cb0p-1, -0x1.e9f4156c62ddap-1,
    -0x1.d906bcf328d46p-1, -0x1.c38b2f180bdb1p-1, -0x1.a9b66290ea1a3p-1, -0x1.8bc806b151741p-1,
    -0x1.6a09e667f3bcdp-1, -0x1.44cf325091dd6p-1, -0x1.1c73b39ae68c8p-1, -0x1.e2b5d3806f63bp-2,
    -0x1.87de2a6aea963p-2, -0x1.294062ed59f06p-2, -0x1.8f8b83c69a60bp-3, -0x1.917a6bc29b42cp-4,
    0.0, 0x1.917a6bc29b42cp-4, 0x1.8f8b83c69a60bp-3, 0x1.294062ed59f06p-2,
    0x1.87de2a6aea963p-2, 0x1.e2b5d3806f63bp-2, 0x1.1c73b39ae68c8p-1, 0x1.44cf325091dd6p-1,
    0x1.6a09e667f3bcdp-1, 0x1.8bc806b151741p-1, 0x1.a9b66290ea1a3p-1, 0x1.c38b2f180bdb1p-1,
    0x1.d906bcf328d46p-1, 0x1.e9f4156c62ddap-1, 0x1.f6297cff75cb0p-1, 0x1.fd88da3d12526p-1,
};
static const double kCandSin[NCAND] = {
    0.0, 0x1.917a6bc29b42cp-4, 0x1.8f8b83c69a60bp-3, 0x1.294062ed59f06p-2,
    0x1.87de2a6aea963p-2, 0x1.e2b5d3806f63bp-2, 0x1.1c73b39ae68c8p-1, 0x1.44cf325091dd6p-1,
    0x1.6a09e667f3bcdp-1, 0x1.8bc806b151741p-1, 0x1.a9b66290ea1a3p-1, 0x1.c38b2f180bdb1p-1,
    0x1.d906bcf328d46p-1, 0x1.e9f4156c62ddap-1, 0x1.f6297cff75cb0p-1, 0x1.fd88da3d12526p-1,
    0x1.0000000000000p+0, 0x1.fd88da3d12526p-1, 0x1.f6297cff75cb0p-1, 0x1.e9f4156c62ddap-1,
    0x1.d906bcf328d46p-1, 0x1.c38b2f180bdb1p-1, 0x1.a9b66290ea1a3p-1, 0x1.8bc806b151741p-1,
    0x1.6a09e667f3bcdp-1, 0x1.44cf325091dd6p-1, 0x1.1c73b39ae68c8p-1, 0x1.e2b5d3806f63bp-2,
    0x1.87de2a6aea963p-2, 0x1.294062ed59f06p-2, 0x1.8f8b83c69a60bp-3, 0x1.917a6bc29b42cp-4,
    0.0, -0x1.917a6bc29b42cp-4, -0x1.8f8b83c69a60bp-3, -0x1.294062ed59f06p-2,
    -0x1.87de2a6aea963p-2, -0x1.e2b5d3806f63bp-2, -0x1.1c73b39ae68c8p-1, -0x1.44cf325091dd6p-1,
    -0x1.6a09e667f3bcdp-1, -0x1.8bc806b151741p-1, -0x1.a9b66290ea1a3p-1, -0x1.c38b2f180bdb1p-1,
    -0x1.d906bcf328d46p-1, -0x1.e9f4156c62ddap-1, -0x1.f6297cff75cb0p-1, -0x1.fd88da3d12526p-1,
    -0x1.0000000000000p+0, -0x1.fd88da3d12526p-1, -0x1.f6297cff75cb0p-1, -0x1.e9f4156c62ddap-1,
    -0x1.d906bcf328d46p-1, -0x1.c38b2f180bdb1p-1, -0x1.a9b66290ea1a3p-1, -0x1.8bc806b151741p-1,
    -0x1.6a09e667f3bcdp-1, -0x1.44cf325091dd6p-1, -0x1.1c73b39ae68c8p-1, -0x1.e2b5d3806f63bp-2,
    -0x1.87de2a6aea963p-2, -0x1.294062ed59f06p-2, -0x1.8f8b83c69a60bp-3, -0x1.917a6bc29b42cp-4,
};

__constant__ double dCandCos[NCAND];
__constant__ double dCandSin[NCAND];

constexpr int HBINS = 1024;                   // 32 x 32 histogram
constexpr int HSAMPLE = 16384;                // at most this many sampled points
constexpr int HRUNS = HSAMPLE / WAVE;          // in runs of WAVE consecutive points
constexpr int L1 = 512, L2 = 512, NOUT = NCAND;
// parameter layout (float32): W1[512][1024] b1[512] W2[512][512] b2[512] W3[64][512] b3[64]
constexpr int64_t P_W1 = 0, P_B1 = P_W1 + (int64_t)L1 * HBINS, P_W2 = P_B1 + L1,
                  P_B2 = P_W2 + (int64_t)L2 * L1, P_W3 = P_B2 + L2, P_B3 = P_W3 + (int64_t)NOUT * L2,
                  P_TOTAL = P_B3 + NOUT;
// bf16 copies of the weight matrices: W1b | W2b | W3b, and the transposes of
// the last two, which the backward products read along their rows
constexpr int64_t Q_W1 = 0, Q_W2 = Q_W1 + (int64_t)L1 * HBINS, Q_W3 = Q_W2 + (int64_t)L2 * L1,
                  Q_W2T = Q_W3 + (int64_t)NOUT * L2, Q_W3T = Q_W2T + (int64_t)L1 * L2,
                  Q_TOTAL = Q_W3T + (int64_t)L2 * NOUT;

typedef uint16_t bf16_t;   // storage of bfloat16 values
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bfloat16, round to nearest even (inputs here are finite)
__device__ __forceinline__ bf16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float((uint32_t)h << 16); }

// ---------------------------------------------------------------------------
// 32 x 32 occupancy histogram of each set (one block per set).  Sample: every
// point of a set of up to 16384, else 256 runs of 64 consecutive points spread
// evenly over the set.  Bins cover a square window of side w = max(width,
// height) of the sample's bounding box (grid units), centred on the box, so
// that the set's aspect ratio and the angles of its features are kept: origin
// (x0 - (w - wx) / 2, y0 - (w - wy) / 2), bin = (k - origin) * 32 / w in
// integer arithmetic; value = count * 1024 / ns (binary64 product and
// quotient, then float, then bf16).
constexpr int HIST_THREADS = 1024;
constexpr int HPER = HSAMPLE / HIST_THREADS;    // samples per thread, held in registers
static_assert(HSAMPLE % HIST_THREADS == 0, "the samples split evenly over the threads");

__global__ __launch_bounds__(HIST_THREADS) void k_hist32(const float *__restrict__ x,
                                                         const float *__restrict__ y,
                                                         const int64_t *__restrict__ off, int64_t n1,
                                                         int64_t S, bf16_t *__restrict__ hist,
                                                         float *__restrict__ hist_f) {
    constexpr int NW = HIST_THREADS / WAVE;
    __shared__ uint32_t cnt[HBINS];
    __shared__ int32_t bb[NW][4];
    const int64_t s = blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const int64_t a = set_begin(off, s), n = set_end(off, n1, s) - a;
    for (int b = tid; b < HBINS; b += blockDim.x) cnt[b] = 0;
    if (n <= 0) {
        __syncthreads();
        for (int b = tid; b < HBINS; b += blockDim.x) {
            hist[s * HBINS + b] = 0;
            if (hist_f) hist_f[s * HBINS + b] = 0.0f;
        }
        return;
    }
    // the sample: every point when n <= HSAMPLE, else HRUNS runs of WAVE
    // consecutive points, run r from floor(r (n - WAVE) / (HRUNS - 1)); each
    // sample loaded once, all of a thread's loads issued together (a wave
    // reads one run: whole cache lines)
    const int64_t ns = n <= HSAMPLE ? n : HSAMPLE;
    int32_t kx[HPER], ky[HPER];
#pragma unroll
    for (int i = 0; i < HPER; i++) {
        const int64_t j = tid + (int64_t)i * HIST_THREADS;
        const int64_t p = n <= HSAMPLE ? j : (j / WAVE) * (n - WAVE) / (HRUNS - 1) + j % WAVE;
        kx[i] = j < ns ? (int32_t)(x[a + p] * GRIDF) : 0;
        ky[i] = j < ns ? (int32_t)(y[a + p] * GRIDF) : 0;
    }
    int32_t x0 = 0x7fffffff, x1 = -1, y0 = 0x7fffffff, y1 = -1;
#pragma unroll
    for (int i = 0; i < HPER; i++) {
        if (tid + (int64_t)i * HIST_THREADS < ns) {
            x0 = min(x0, kx[i]); x1 = max(x1, kx[i]); y0 = min(y0, ky[i]); y1 = max(y1, ky[i]);
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        x0 = min(x0, __shfl_xor(x0, o)); x1 = max(x1, __shfl_xor(x1, o));
        y0 = min(y0, __shfl_xor(y0, o)); y1 = max(y1, __shfl_xor(y1, o));
    }
    if (lane == 0) { bb[w][0] = x0; bb[w][1] = x1; bb[w][2] = y0; bb[w][3] = y1; }
    __syncthreads();
    x0 = bb[0][0]; x1 = bb[0][1]; y0 = bb[0][2]; y1 = bb[0][3];
    for (int ww = 1; ww < NW; ww++) {
        x0 = min(x0, bb[ww][0]); x1 = max(x1, bb[ww][1]);
        y0 = min(y0, bb[ww][2]); y1 = max(y1, bb[ww][3]);
    }
    const int64_t wx = (int64_t)x1 - x0 + 1, wy = (int64_t)y1 - y0 + 1, wd = max(wx, wy);
    const int64_t cx0 = x0 - (wd - wx) / 2, cy0 = y0 - (wd - wy) / 2;
    // bin = floor((k - c0) * 32 / wd): 0 <= k - c0 < wd <= 2^24, so the
    // product stays below 2^29 and a 32-bit division is exact
    const uint32_t uwd = (uint32_t)wd;
#pragma unroll
    for (int i = 0; i < HPER; i++) {
        if (tid + (int64_t)i * HIST_THREADS < ns) {
            const uint32_t bx = (uint32_t)((int64_t)kx[i] - cx0) * 32u / uwd;
            const uint32_t by = (uint32_t)((int64_t)ky[i] - cy0) * 32u / uwd;
            atomicAdd(&cnt[by * 32 + bx], 1u);
        }
    }
    __syncthreads();
    for (int b = tid; b < HBINS; b += blockDim.x) {
        float v = (float)((double)cnt[b] * 1024.0 / (double)ns);
        hist[s * HBINS + b] = f2bf(v);
        if (hist_f) hist_f[s * HBINS + b] = v;
    }
}

// ---------------------------------------------------------------------------
// The network's products: C[M x N] = A[M x K] * B[N x K]^T in bf16 on MFMA
// (16x16x32), fp32 accumulation; A and B with K along their rows (row strides
// lda, ldb), M and N multiples of 64, K of 32.  A block makes a 32 R x 32 R
// tile, each of its four waves a 16 R x 16 R one over the whole of K, step by
// step into one accumulator each (the results are rounded to bf16 for the next layer, so the
// order of the sums is kept), with the operands loaded straight into the
// lanes that feed them to MFMA, eight steps ahead.  The products here are
// small (512 x 512 x 1024 at a batch of 512), so what bounds them is the
// latency of the loads along K and the launches, not the matrix cores: small
// tiles put a 512 x 512 product on all 256 CUs, loads far ahead hide the
// latency, and independent products share a launch.  (64 x 64 tiles with K
// staged through LDS 32 at a time, one product a launch, took 17 us for the
// first layer; forward, then forward and backward, with their helpers at a
// batch of 512: 320 us, now 88 us.)  With R = 2 or 4 each operand is read half
// or a quarter as often, which is what bounds products of many tiles: the
// forward pass of 20000 sets took 453 us with R = 1 (234 with those tiles),
// 255 with R = 2, now 186.
enum GemmMode { G_RELU_BF16 = 0, G_BIAS_F32 = 1, G_MASK_BF16 = 2, G_F32 = 3 };
constexpr int GT = 32;                       // tile side
constexpr int GKS = 32;                      // K per MFMA step
constexpr int GAHEAD = 8;                    // steps loaded together (4: 86 us, 16: 97 us for the same)

struct GemmJob {
    const bf16_t *A, *B;
    int lda, ldb, K;
    int tm, tn;              // tiles along M and N
    int mode;
    int arows;               // rows of A in memory; the others count as zeros
    int crows;               // rows of C to write (G_BIAS_F32, G_F32)
    const float *bias;       // G_RELU_BF16, G_BIAS_F32: [N]
    const bf16_t *mask;      // G_MASK_BF16: C is 0 where mask [M][N] is not positive
    bf16_t *Cb, *CT;         // bf16 results [M][N] and transposed [N][M] (either may be null)
    float *Cf;               // fp32 results [M][N]
    float *asum;             // sums over K of A's rows (bias gradients), or null
};
struct GemmJobs {
    GemmJob j[2];
    int n;
};

template <int R>
__global__ __launch_bounds__(256) void k_gemm(GemmJobs jobs) {
    constexpr int TS = GT * R, TP = TS + 4, AHEAD = GAHEAD / R;
    __shared__ __attribute__((aligned(8))) uint16_t tile16[TS * TP];
    int tile = blockIdx.x;
    const int first = jobs.j[0].tm / R * (jobs.j[0].tn / R);
    const bool second = tile >= first;
    if (second) tile -= first;
    const GemmJob &J = jobs.j[second ? 1 : 0];
    const int tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = tile / (J.tn / R) * TS, n0 = tile % (J.tn / R) * TS;
    const int wm = (w >> 1) * 16 * R, wn = (w & 1) * 16 * R;
    const int steps = J.K / GKS;
    const int r = lane & 15, k8 = (lane >> 4) * 8;
    const bool sums = J.asum && n0 + wn == 0;
    float as[R];
    bool live[R];
    const bf16_t *pa[R], *pb[R];
    f32x4 acc[R][R];
#pragma unroll
    for (int i = 0; i < R; i++) {
        const int row = m0 + wm + 16 * i + r;
        as[i] = 0.f;
        live[i] = row < J.arows;
        pa[i] = J.A + (int64_t)(live[i] ? row : 0) * J.lda + k8;
        pb[i] = J.B + (int64_t)(n0 + wn + 16 * i + r) * J.ldb + k8;
#pragma unroll
        for (int j = 0; j < R; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    bf16x8 a[2][AHEAD][R], b[2][AHEAD][R];
    auto load = [&](int s0, bf16x8 (*va)[R], bf16x8 (*vb)[R]) {
#pragma unroll
        for (int d = 0; d < AHEAD; d++) {
            const int k = min(s0 + d, steps - 1) * GKS;      // past the end: the last step again
#pragma unroll
            for (int i = 0; i < R; i++) {
                va[d][i] = *reinterpret_cast<const bf16x8 *>(pa[i] + k);
                vb[d][i] = *reinterpret_cast<const bf16x8 *>(pb[i] + k);
            }
        }
    };
    auto multiply = [&](int s0, bf16x8 (*va)[R], bf16x8 (*vb)[R]) {
#pragma unroll
        for (int d = 0; d < AHEAD; d++) {
            if (s0 + d >= steps) break;
#pragma unroll
            for (int i = 0; i < R; i++) {
                const bf16x8 av = live[i] ? va[d][i] : bf16x8{};
#pragma unroll
                for (int j = 0; j < R; j++)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, vb[d][j], acc[i][j], 0, 0, 0);
                if (sums)
#pragma unroll
                    for (int t = 0; t < 8; t++) as[i] += (float)av[t];
            }
        }
    };
    load(0, a[0], b[0]);
    for (int s0 = 0; s0 < steps; s0 += 2 * AHEAD) {
        if (s0 + AHEAD < steps) load(s0 + AHEAD, a[1], b[1]);
        multiply(s0, a[0], b[0]);
        if (s0 + AHEAD >= steps) break;
        if (s0 + 2 * AHEAD < steps) load(s0 + 2 * AHEAD, a[0], b[0]);
        multiply(s0 + AHEAD, a[1], b[1]);
    }
    if (sums)
#pragma unroll
        for (int i = 0; i < R; i++) {
            as[i] += __shfl_xor(as[i], 16);
            as[i] += __shfl_xor(as[i], 32);
            if (lane < 16) J.asum[m0 + wm + 16 * i + lane] = as[i];
        }
    const int ldc = J.tn * GT;
#pragma unroll
    for (int i = 0; i < R; i++)
#pragma unroll
        for (int j = 0; j < R; j++) {
            // lane: column n0 + n, rows m0 + m .. m0 + m + 3
            const int n = wn + 16 * j + r, m = wm + 16 * i + (lane >> 4) * 4;
            const int64_t o = (int64_t)(m0 + m) * ldc + n0 + n;
            float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
            if (J.mode == G_RELU_BF16 || J.mode == G_BIAS_F32) {
                const float bias = J.bias[n0 + n];
#pragma unroll
                for (int q = 0; q < 4; q++) v[q] += bias;
            }
            if (J.mode == G_BIAS_F32 || J.mode == G_F32) {
#pragma unroll
                for (int q = 0; q < 4; q++)
                    if (m0 + m + q < J.crows) J.Cf[o + (int64_t)q * ldc] = v[q];
                continue;
            }
            uint16_t c[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                if (J.mode == G_RELU_BF16) c[q] = f2bf(fmaxf(v[q], 0.0f));
                else c[q] = bf2f(J.mask[o + (int64_t)q * ldc]) > 0.0f ? f2bf(v[q]) : (uint16_t)0;
            }
            if (J.CT)
                *reinterpret_cast<ushort4 *>(J.CT + (int64_t)(n0 + n) * (J.tm * GT) + m0 + m) =
                    make_ushort4(c[0], c[1], c[2], c[3]);
            if (J.Cb)
#pragma unroll
                for (int q = 0; q < 4; q++) tile16[(m + q) * TP + n] = c[q];
        }
    if (J.mode == G_BIAS_F32 || J.mode == G_F32 || !J.Cb) return;
    __syncthreads();
#pragma unroll
    for (int e = tid * 4; e < TS * TS; e += 256 * 4) {       // four neighbours of one row per thread
        const int tr = e / TS, tc = e % TS;
        *reinterpret_cast<ushort4 *>(J.Cb + (int64_t)(m0 + tr) * ldc + n0 + tc) =
            *reinterpret_cast<const ushort4 *>(&tile16[tr * TP + tc]);
    }
}

// float32 -> bf16 copy (weights after an update, or inputs); with cols > 0
// also the transpose of the [n / cols][cols] matrix
__global__ void k_to_bf16(const float *__restrict__ src, int64_t n, bf16_t *__restrict__ dst, int cols,
                          bf16_t *__restrict__ dstT) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x) {
        const bf16_t v = f2bf(src[i]);
        dst[i] = v;
        if (cols) dstT[(i % cols) * (n / cols) + i / cols] = v;
    }
}

// Histogram rows into the network's input matrix, for arrays that are not
// 16-byte aligned.
__global__ void k_copy_rows(const bf16_t *__restrict__ src, int64_t n, bf16_t *__restrict__ dst) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x)
        dst[i] = src[i];
}

// What the backward products read along the batch: the histograms'
// transpose XT [1024][Bp] and, from float32 output gradients (if given), dS
// [Bp][64] in bf16 and its transpose.  Rows past the batch are zeros.  A
// block turns a 64 x 64 tile through LDS; the last column of blocks does dS.
__global__ __launch_bounds__(256) void k_backward_prep(const bf16_t *__restrict__ X, int64_t B, int Bp,
                                                       bf16_t *__restrict__ XT, const float *__restrict__ d,
                                                       bf16_t *__restrict__ dS, bf16_t *__restrict__ dST) {
    __shared__ bf16_t t[64][66];
    const int b0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
    const bool grad = blockIdx.x == HBINS / 64;
    const int c = threadIdx.x & 63, r0 = threadIdx.x >> 6;
    for (int r = r0; r < 64; r += 4) {
        const int64_t b = b0 + r;
        bf16_t v = 0;
        if (b < B) v = grad ? f2bf(d[b * NOUT + c]) : X[b * HBINS + c0 + c];
        if (grad) dS[b * NOUT + c] = v;
        t[r][c] = v;
    }
    __syncthreads();
    for (int r = r0; r < 64; r += 4) {
        if (grad) dST[(int64_t)r * Bp + b0 + c] = t[c][r];
        else XT[(int64_t)(c0 + r) * Bp + b0 + c] = t[c][r];
    }
}

// Loss: targets t = gain / max(gain) per set (0 when no direction gains),
// L = mean over sets and directions of (score - t)^2.  dS = dL/dscore (bf16
// for the backward products); per-set partial losses for a fixed-order sum.
__global__ void k_loss(const float *__restrict__ scores, const float *__restrict__ gain, int64_t B,
                       int64_t Bp, bf16_t *__restrict__ dS, bf16_t *__restrict__ dST,
                       float *__restrict__ part) {
    const int64_t b = blockIdx.x;
    const int d = threadIdx.x;   // 64 threads
    float s = 0.0f, t = 0.0f;
    if (b < B) {
        float g = gain[b * NOUT + d];
        float mx = g;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        t = mx > 0.0f ? g / mx : 0.0f;
        s = scores[b * NOUT + d];
    }
    float diff = b < B ? s - t : 0.0f;
    const bf16_t g16 = f2bf(2.0f * diff / (float)(B * NOUT));
    dS[b * NOUT + d] = g16;
    dST[(int64_t)d * Bp + b] = g16;
    float sq = diff * diff;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sq += __shfl_xor(sq, o);
    if (d == 0) part[b] = sq;
}

__global__ void k_loss_sum(const float *__restrict__ part, int64_t B, float *__restrict__ loss) {
    if (threadIdx.x == 0) {
        double acc = 0.0;
        for (int64_t b = 0; b < B; b++) acc += part[b];
        *loss = (float)(acc / (double)(B * NOUT));
    }
}

// Adam on the float32 master parameters; refreshes the bf16 weight copies.
__global__ void k_adam(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int64_t n, float lr, float b1, float b2, float eps,
                       float c1, float c2, bf16_t *__restrict__ wb) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x) {
        float gi = g[i];
        float mi = b1 * m[i] + (1.0f - b1) * gi;
        float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        w[i] = wi;
        int64_t q = -1;   // position of weight-matrix entries in the bf16 copy
        if (i < P_B1) q = Q_W1 + (i - P_W1);
        else if (i >= P_W2 && i < P_B2) q = Q_W2 + (i - P_W2);
        else if (i >= P_W3 && i < P_B3) q = Q_W3 + (i - P_W3);
        if (q >= 0) wb[q] = f2bf(wi);
        int64_t qt = -1;  // and in the transposes
        if (i >= P_W2 && i < P_B2) qt = Q_W2T + ((i - P_W2) % L1) * L2 + (i - P_W2) / L1;
        else if (i >= P_W3 && i < P_B3) qt = Q_W3T + ((i - P_W3) % L2) * NOUT + (i - P_W3) / L2;
        if (qt >= 0) wb[qt] = f2bf(wi);
    }
}

// Top eight of the 64 scores of each set (higher first, lower index on
// ties; NaN counts as -inf); their (cos, sin) go to set_dirs.  One wave per
// set, lane d holds direction d.  Scores are compared through an
// order-preserving integer image; a direction already taken ranks below all.
__device__ __forceinline__ int32_t score_rank(float v) {
    if (!(v == v)) v = -INFINITY;
    v = v + 0.0f;   // -0 ranks with +0
    uint32_t u = __float_as_uint(v);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
    return (int32_t)(u - 0x80000000u);
}

// Eight directions per set (one wave per set): repeatedly the highest score
// (lowest index on ties, NaN as -inf) among the directions still available;
// each pick removes itself and, for gap > 0, the directions within gap steps
// of it on the circle of 64, so that picks are at least gap + 1 steps apart.
// gap <= 3 always leaves eight picks.
__global__ void k_top8(const float *__restrict__ scores, int64_t S, int gap,
                       int32_t *__restrict__ dirs, double *__restrict__ set_dirs) {
    const int64_t s = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
    const int d = lane_id();
    if (s >= S) return;
    int32_t key = score_rank(scores[s * NOUT + d]);
    for (int r = 0; r < MAX_DIRS; r++) {
        int32_t bk = key;
        int bi = d;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            int32_t k2 = __shfl_xor(bk, o);
            int i2 = __shfl_xor(bi, o);
            if (k2 > bk || (k2 == bk && i2 < bi)) { bk = k2; bi = i2; }
        }
        if (d == 0) {
            if (dirs) dirs[s * MAX_DIRS + r] = bi;
            set_dirs[(s * MAX_DIRS + r) * 2 + 0] = dCandCos[bi];
            set_dirs[(s * MAX_DIRS + r) * 2 + 1] = dCandSin[bi];
        }
        const int dist = min((d - bi) & (NOUT - 1), (bi - d) & (NOUT - 1));
        if (dist <= gap) key = INT32_MIN;
    }
}

// ---------------------------------------------------------------------------
// Training labels, from the fixed filter's survivors of each set.
//
// A survivor is not strictly inside some edges of the base polygon: its
// "out" mask, usually one bit.  The mask says which of the 64 directions the
// survivor matters for, so both passes below sort their survivors by it (a
// chunk at a time, in LDS) and a wave then walks the few directions of its
// batch's class with the edge and direction constants uniform over the wave.
// They are bound by vector instructions: about 16 edge tests per survivor and
// 6-8 directions instead of 64.  (The former passes walked every point eight
// times with one block per set, and 64 polygons of up to 17 edges per
// survivor: 1391 and 6689 us for 256 mixtures of 2^16 points, now 143 and 46;
// without the heights below 568 and 46.)
constexpr int LAB_THREADS = 512;
constexpr int LAB_WAVES = LAB_THREADS / WAVE;
constexpr int LAB_PER = 4;
constexpr int LAB_CHUNK = LAB_THREADS * LAB_PER;
constexpr int LAB_CLASSES = FIXED_SLOTS + 1;          // one edge each; the rest
constexpr int LAB_SPLIT = 16;                         // most blocks per set
constexpr int LAB_NOTES = 1024;
constexpr int LAB_BINS = LAB_THREADS / FIXED_SLOTS;   // height bins along a base edge
// Blocks per set: eight per CU in all, since sets differ in survivors by a
// factor of ten and with fewer most CUs wait for a few (256 sets, both passes:
// 274, 250, 208 and 253 us with three, four, eight and sixteen per CU); more
// sets than that have one each.
// More blocks than CUs have at least LAB_POINTS points of a set of mean size
// each, since each sets up the directions (300 sets of 1000 points: labels 171
// us with seven blocks each, 134 with one).
constexpr int LAB_BLOCKS_PER_CU = 8;
constexpr int64_t LAB_POINTS = 2048;
static unsigned lab_split(int64_t S, int64_t n_total, int cus) {
    const int64_t k = (LAB_BLOCKS_PER_CU * (int64_t)cus + S - 1) / S,
                  most = std::max<int64_t>(n_total / (S * LAB_POINTS), cus / S);
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(std::min(k, most), LAB_SPLIT));
}

// Partial extreme of one direction over a block's share of a set.
struct CandPart {
    double v;
    uint32_t i;
    uint32_t pad;
};

struct LabShared {
    float x[LAB_CHUNK], y[LAB_CHUNK];
    uint32_t id[LAB_CHUNK];
    uint16_t out[LAB_CHUNK];
    uint32_t cnt[LAB_CLASSES];                        // survivors of each class in the chunk
    uint32_t start[LAB_CLASSES + 1];                  // the classes' first entries
    uint32_t batch[LAB_CLASSES + 1];                  // and first batches of 64
};

// Heights below which a survivor outside one edge only cannot matter: for edge
// e and a survivor whose foot lies in bin b of the edge, -E < h[e][b].
struct LabHeights {
    double h[FIXED_SLOTS][LAB_BINS];
    double u0[FIXED_SLOTS], scale[FIXED_SLOTS];       // bin = (ex px + ey py - u0) scale
};

// The base polygon's edges (E > 0: strictly inside).  A polygon of two
// vertices counts as two edges, there and back, that nothing is inside of;
// with fewer vertices all points are one, and there are no edges.
struct LabEdges {
    double ex[FIXED_SLOTS], ey[FIXED_SLOTS], c[FIXED_SLOTS];
    __device__ __forceinline__ int load(const Poly &P) {      // every thread; sync before use
        const int k = threadIdx.x, m = P.m;
        if (m >= 3) {
            if (k < m) { ex[k] = P.ex[k]; ey[k] = P.ey[k]; c[k] = P.c[k]; }
            return m;
        }
        if (m == 2 && k < 2) {
            const double ax = P.vx[k], ay = P.vy[k];
            const double ddx = P.vx[1 - k] - ax, ddy = P.vy[1 - k] - ay;
            ex[k] = ddx;
            ey[k] = ddy;
            c[k] = fma(ddy, ax, -(ddx * ay));
        }
        return m == 2 ? 2 : 0;
    }
};

// Load survivors [c0, c1) (at most LAB_CHUNK) into L, grouped by class, less
// those that H (if given) leaves out.  Every thread of the block calls it;
// L.cnt holds the class counts after.
__device__ __forceinline__ void lab_chunk(LabShared &L, const float *__restrict__ x,
                                          const float *__restrict__ y, const uint32_t *__restrict__ surv,
                                          int64_t c0, int64_t c1, const LabEdges &E, int m,
                                          const LabHeights *H) {
    const int tid = threadIdx.x;
    __syncthreads();                                  // the previous chunk is done with L
    if (tid < LAB_CLASSES) L.cnt[tid] = 0;
    float px[LAB_PER], py[LAB_PER];
    uint32_t id[LAB_PER], out[LAB_PER], rank[LAB_PER];
    int cls[LAB_PER];
#pragma unroll
    for (int q = 0; q < LAB_PER; q++) {
        const int64_t j = c0 + tid + q * LAB_THREADS;
        id[q] = j < c1 ? surv[j] : NONE;
    }
#pragma unroll
    for (int q = 0; q < LAB_PER; q++) {
        px[q] = id[q] != NONE ? x[id[q]] : 0.0f;
        py[q] = id[q] != NONE ? y[id[q]] : 0.0f;
        out[q] = 0;
    }
    for (int e = 0; e < m; e++) {
        const double ex = E.ex[e], ey = E.ey[e], ec = E.c[e];
#pragma unroll
        for (int q = 0; q < LAB_PER; q++)
            if (!(edge_eval(ex, ey, ec, (double)px[q] * GRIDD, (double)py[q] * GRIDD) > 0)) out[q] |= 1u << e;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < LAB_PER; q++) {
        cls[q] = __popc(out[q]) == 1 ? __ffs((int)out[q]) - 1 : FIXED_SLOTS;
        if (H && cls[q] < FIXED_SLOTS) {
            const int e = cls[q];
            const double gx = (double)px[q] * GRIDD, gy = (double)py[q] * GRIDD;
            const double b = (fma(E.ex[e], gx, E.ey[e] * gy) - H->u0[e]) * H->scale[e];
            if (b >= 0 && b < LAB_BINS && -edge_eval(E.ex[e], E.ey[e], E.c[e], gx, gy) < H->h[e][(int)b])
                id[q] = NONE;
        }
        const bool has = id[q] != NONE;
        // lanes of the same class: one LDS addition per class and wave
        uint64_t same = __ballot(has);
#pragma unroll
        for (int b = 0; b < 5; b++) {
            const uint64_t bit = __ballot((cls[q] >> b) & 1);
            same &= ((cls[q] >> b) & 1) ? bit : ~bit;
        }
        uint32_t base = 0;
        const int lead = has ? __ffsll((unsigned long long)same) - 1 : 0;
        if (has && lead == lane_id()) base = atomicAdd(&L.cnt[cls[q]], (uint32_t)__popcll(same));
        rank[q] = __shfl(base, lead) + (uint32_t)__popcll(same & lanemask_lt());
    }
    __syncthreads();
    if (tid <= LAB_CLASSES) {
        uint32_t at = 0, b = 0;
        for (int c = 0; c < LAB_CLASSES; c++) {
            const uint32_t n = L.cnt[c];
            at += c < tid ? n : 0;
            b += c < tid ? (n + WAVE - 1) / WAVE : 0;
        }
        L.start[tid] = at;
        L.batch[tid] = b;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < LAB_PER; q++) {
        if (id[q] == NONE) continue;
        const uint32_t at = L.start[cls[q]] + rank[q];
        L.x[at] = px[q];
        L.y[at] = py[q];
        L.id[at] = id[q];
        L.out[at] = (uint16_t)out[q];
    }
    __syncthreads();
}

// Batch b of a chunk: up to 64 survivors of one class.  Returns false past
// the last batch.
__device__ __forceinline__ bool lab_batch(const LabShared &L, int b, int *cls, int *at, int *len) {
    const int lane = lane_id();
    const int c = __popcll(__ballot(lane < LAB_CLASSES && b >= (int)L.batch[min(lane, LAB_CLASSES - 1) + 1]));
    if (c >= LAB_CLASSES) return false;
    const int rel = (b - (int)L.batch[c]) * WAVE;
    *cls = c;
    *at = (int)L.start[c] + rel;
    *len = min(WAVE, (int)L.cnt[c] - rel);
    return true;
}

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}
__device__ __forceinline__ uint64_t wave_or_u64(uint64_t v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v |= (uint64_t)__shfl_xor((unsigned long long)v, o);
    return uniform_u64(v);
}

// (1) Extreme point of every set along each of the 64 candidate directions
//     (argmax of c*x + s*y, lowest index on ties), one partial per block.
//     Only survivors can be one: a point strictly inside the base polygon lies
//     at least 2^-49 inside each of its edges, more than the roundings of two
//     values (2^-51), so it neither beats nor ties the best vertex.  The same
//     bound holds edge by edge: a survivor strictly inside both edges at the
//     base vertex that is extreme along d is not extreme along d.  So edge j's
//     class visits the directions whose extreme base vertex (or one within
//     2^-40 of it) is an end of edge j.
//     The block shares one best value per direction, raised by an LDS maximum
//     and started at the best base vertex; a survivor that reaches the best
//     when it is seen is noted in a list, from which the lowest index of each
//     final best is taken (a vertex has the lowest of its copies; of a wave's
//     ties only the lowest index is noted).  Should the list run over, the
//     survivors are walked once more for it.  A best per wave, found with
//     cross-lane reductions, took as long.
//     A thin set's long edges end at vertices that are extreme along most of
//     the directions, so their class (most of the survivors) visits them all.
//     There a height per bin of the edge leaves out the survivors that stay
//     2^-45 below every direction's best so far (unit coordinates; the
//     arithmetic errs by less than 2^-50): of the class, few remain.  The
//     heights are taken at the start, after the first 512 survivors of a
//     block and whenever the chunks done are four times as many.
//     Of points on the segment of a two-vertex polygon only the ends can be
//     extreme, but for the directions that the segment is nearly perpendicular
//     to: with the ends' values 2^-25 apart, two grid points of the segment (at
//     most 2^24 steps) are 2^-49 apart, more than the roundings.  Points that
//     are all one point need no walk.  (Visited as others, 256 sets of 65536
//     such points took 2.0 ms on a line and 8.5 ms in one place; 1.6 and 1.7
//     with the former walk of every point; now 0.5 and 0.35.)
__global__ __launch_bounds__(LAB_THREADS) void k_cand_extremes(
    const float *__restrict__ x, const float *__restrict__ y, const Poly *__restrict__ polys,
    const uint32_t *__restrict__ surv, const int64_t *__restrict__ surv_off, CandPart *__restrict__ part) {
    __shared__ LabShared L;
    __shared__ uint64_t dirs[LAB_CLASSES];
    __shared__ double bv[NCAND];                      // best value, and its lowest index
    __shared__ uint32_t bi[NCAND];
    __shared__ double vv[NCAND];                      // the best vertex's value and index
    __shared__ uint32_t vi[NCAND];
    __shared__ uint64_t flat;                         // two vertices: directions across the segment
    __shared__ double cc[NCAND], ss[NCAND];
    __shared__ double nv[LAB_NOTES];                  // noted survivors: value, index, direction
    __shared__ uint32_t ni[LAB_NOTES];
    __shared__ uint8_t nd[LAB_NOTES];
    __shared__ uint32_t notes;
    __shared__ LabHeights H;
    __shared__ LabEdges E;
    const int64_t s = blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const Poly &P = polys[s];
    CandPart *mine = part + (s * gridDim.y + blockIdx.y) * NCAND;
    if (P.m < 2) {
        if (tid < NCAND) mine[tid] = CandPart{0.0, P.m == 1 && blockIdx.y == 0 ? P.verts[0] : NONE, 0};
        return;
    }
    const int m = E.load(P);
    if (w == 0) {
        const int d = lane;
        double first = -INFINITY;
        cc[d] = dCandCos[d];
        ss[d] = dCandSin[d];
        uint32_t id = NONE;
        double v0 = 0, v1 = 0;
        for (int k = 0; k < m; k++) {
            const double v = proj_dir(cc[d], ss[d], P.vx[k] * (1.0 / GRIDD), P.vy[k] * (1.0 / GRIDD));
            const uint32_t q = P.verts[k];
            if (k == 0) v0 = v;
            if (k == 1) v1 = v;
            const bool t = (int)(v > first) | ((int)(v == first) & (int)(q < id));
            first = t ? v : first;
            id = t ? q : id;
        }
        uint32_t edges = 0;
        for (int k = 0; k < m; k++) {
            const double v = proj_dir(cc[d], ss[d], P.vx[k] * (1.0 / GRIDD), P.vy[k] * (1.0 / GRIDD));
            if (v >= first - 0x1p-40) edges |= (1u << k) | (1u << (k ? k - 1 : m - 1));
        }
        bv[d] = vv[d] = first;
        bi[d] = vi[d] = id;
        const uint64_t f = __ballot(fabs(v0 - v1) <= 0x1p-25);
        if (d == 0) {
            flat = f;
            notes = 0;
        }
        for (int c = 0; c < LAB_CLASSES; c++) {
            const uint64_t b = __ballot((edges >> c) & 1);
            if (lane == 0) dirs[c] = b;
        }
    }
    const int64_t sa = surv_off[s], sb = surv_off[s + 1];
    const int64_t share = (sb - sa + gridDim.y - 1) / gridDim.y;
    const int64_t ba = min(sb, sa + share * blockIdx.y), bb = min(sb, ba + share);
    if (tid < m) {
        const double ex = E.ex[tid], ey = E.ey[tid];
        H.u0[tid] = fma(ex, (double)P.vx[tid], ey * (double)P.vy[tid]);
        H.scale[tid] = LAB_BINS / fma(ex, ex, ey * ey);
    }
    auto heights = [&]() {
        __syncthreads();                              // bv raised by every wave
        const int e = tid / LAB_BINS, b = tid % LAB_BINS;
        if (e < m) {
            const double ex = E.ex[e], ey = E.ey[e], l2 = fma(ex, ex, ey * ey);
            const double wx = P.vx[e] * (1.0 / GRIDD), wy = P.vy[e] * (1.0 / GRIDD);
            double h = INFINITY;
            for (uint64_t dm = dirs[e]; dm; dm &= dm - 1) {
                const int d = __builtin_ctzll(dm);
                const double de = (cc[d] * ex + ss[d] * ey) * (1.0 / GRIDD);       // along the edge
                const double dn = (cc[d] * ey - ss[d] * ex) * (1.0 / GRIDD);       // outward
                const double t = de > 0 ? (b + 1.0) / LAB_BINS : (double)b / LAB_BINS;
                const double g = bv[d] - 0x1p-45 - proj_dir(cc[d], ss[d], wx, wy) - t * de;
                if (!(g > 0)) h = 0;
                else if (dn > 0) h = fmin(h, g * __builtin_amdgcn_rcp(dn));
            }
            H.h[e][b] = h * l2 * (1.0 - 0x1p-16);     // the reciprocals err by less
        }
    };
    // walk(f): f(direction, value, index, lane in use) for the survivors of
    // the block's share that can matter and the directions of their class
    const bool tall = bb - ba > LAB_THREADS;          // few survivors are walked sooner than heights are made
    auto walk = [&](bool refresh, auto &&f) {
        int64_t done = 0, next = 0;
        for (int64_t c0 = ba, c1; c0 < bb; c0 = c1, done++) {
            c1 = min(bb, c0 + (c0 == ba ? LAB_THREADS : LAB_CHUNK));
            if (refresh && tall && done == next) {
                heights();
                next = next ? next * 4 : 1;
            }
            lab_chunk(L, x, y, surv, c0, c1, E, m, tall ? &H : nullptr);
            int cls, at, len;
            for (int b = w; lab_batch(L, b, &cls, &at, &len); b += LAB_WAVES) {
                const bool has = lane < len;
                const int i = at + min(lane, len - 1);
                const double xd = L.x[i], yd = L.y[i];
                const uint32_t id = L.id[i];
                uint64_t dm;
                if (cls < FIXED_SLOTS) dm = uniform_u64(dirs[cls]);
                else if (m == 2) dm = uniform_u64(flat);
                else {
                    dm = 0;
                    for (uint32_t o = L.out[i]; o; o &= o - 1) dm |= dirs[__ffs((int)o) - 1];
                    dm = wave_or_u64(dm);
                }
                while (dm) {
                    const int d = __builtin_ctzll(dm);
                    dm &= dm - 1;
                    f(d, proj_dir(cc[d], ss[d], xd, yd), id, has);
                }
            }
        }
    };
    walk(true, [&](int d, double v, uint32_t id, bool has) {
        bool hit = has && v >= bv[d];
        if (!__ballot(hit)) return;
        hit = hit && !(v == vv[d] && id >= vi[d]);    // the vertex, its copies, and ties behind it
        const uint64_t any = __ballot(hit);
        if (!any) return;
        if (any & (any - 1)) {                        // of several the best, of ties the lowest
            const double most = wave_extreme<false>(hit ? v : -INFINITY);
            hit = hit && v == most;
            const uint32_t low = wave_min_u32(hit ? id : NONE);
            hit = hit && id == low;
        }
        if (hit) atomicMax(&bv[d], v);
        wave_sync();
        hit = hit && v >= bv[d];
        const uint64_t who = __ballot(hit);
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&notes, (uint32_t)__popcll(who));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(who & lanemask_lt());
        if (hit && at < LAB_NOTES) {
            nv[at] = v;
            ni[at] = id;
            nd[at] = (uint8_t)d;
        }
    });
    __syncthreads();
    if (tid < NCAND && bv[tid] > vv[tid]) bi[tid] = NONE;        // a survivor beyond every vertex
    __syncthreads();
    if (notes <= LAB_NOTES) {
        for (uint32_t i = tid; i < notes; i += LAB_THREADS)
            if (nv[i] == bv[nd[i]]) atomicMin(&bi[nd[i]], ni[i]);
    } else {
        if (tall) heights();
        walk(false, [&](int d, double v, uint32_t id, bool has) {
            if (has && v == bv[d]) atomicMin(&bi[d], id);
        });
    }
    __syncthreads();
    if (tid < NCAND) mine[tid] = CandPart{bv[tid], bi[tid], 0};
}

// The extreme of each direction from a set's partials (NONE for an empty
// set), and cleared counters for k_labels.  One wave per set.
__global__ void k_cand_pick(const CandPart *__restrict__ part, int split, uint32_t *__restrict__ cand,
                            uint32_t *__restrict__ cnt) {
    const int64_t s = blockIdx.x;
    const int d = threadIdx.x;
    double v = -INFINITY;
    uint32_t i = NONE;
    for (int b = 0; b < split; b++) {
        const CandPart q = part[(s * split + b) * NCAND + d];
        if (q.i == NONE) continue;
        if (q.v > v || (q.v == v && q.i < i)) { v = q.v; i = q.i; }
    }
    cand[s * NCAND + d] = i;
    cnt[s * NCAND + d] = 0;
}

// (2) cnt[s][d] += #{survivors of the block's share strictly inside
//     hull(base polygon + e_d)}.  That polygon keeps the base edges that e_d
//     is strictly inside of and replaces the others (a run of neighbours) by
//     two edges through e_d; an e_d outside no edge adds nothing.  So a
//     survivor is inside it iff e_d replaces every edge in its out mask and
//     it is strictly inside the two new edges.
__global__ __launch_bounds__(LAB_THREADS) void k_labels(
    const float *__restrict__ x, const float *__restrict__ y, const Poly *__restrict__ polys,
    const uint32_t *__restrict__ cand, const uint32_t *__restrict__ surv,
    const int64_t *__restrict__ surv_off, uint32_t *__restrict__ cnt) {
    __shared__ LabShared L;
    __shared__ uint64_t dirs[LAB_CLASSES];            // directions whose e_d replaces edge c
    __shared__ double ne[2][3][NCAND];                // the new edges' ex, ey, c
    __shared__ LabEdges E;
    __shared__ uint32_t wcnt[LAB_WAVES][NCAND];
    const int64_t s = blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const Poly &P = polys[s];
    const int m = E.load(P);
    __syncthreads();
    if (w == 0) {
        const int d = lane;
        const uint32_t e = cand[s * NCAND + d];
        uint32_t gone = 0, neg = 0;
        int first = 0, last = 0;                      // e_d joins the ends of the run it replaces
        double gx = 0, gy = 0;
        if (e != NONE) {
            gx = (double)x[e] * GRIDD;
            gy = (double)y[e] * GRIDD;
            for (int k = 0; k < m; k++) {
                const double v = edge_eval(E.ex[k], E.ey[k], E.c[k], gx, gy);
                if (v < 0) neg |= 1u << k;
                if (!(v > 0)) gone |= 1u << k;
            }
            for (int k = 0; k < m; k++) {
                const int prev = k ? k - 1 : m - 1, next = k + 1 < m ? k + 1 : 0;
                if (!((gone >> k) & 1)) continue;
                if (!((gone >> prev) & 1)) first = k;
                if (!((gone >> next) & 1)) last = next;
            }
        }
        if (!neg) gone = 0;
        const double ux = m ? P.vx[first] : 0, uy = m ? P.vy[first] : 0;
        const double vx = m ? P.vx[last] : 0, vy = m ? P.vy[last] : 0;
        ne[0][0][d] = gx - ux;
        ne[0][1][d] = gy - uy;
        ne[0][2][d] = fma(gy - uy, ux, -((gx - ux) * uy));
        ne[1][0][d] = vx - gx;
        ne[1][1][d] = vy - gy;
        ne[1][2][d] = fma(vy - gy, gx, -((vx - gx) * gy));
        for (int c = 0; c < LAB_CLASSES; c++) {
            const uint64_t b = __ballot((gone >> c) & 1);
            if (lane == 0) dirs[c] = b;
        }
    }
    const int64_t sa = surv_off[s], sb = m ? surv_off[s + 1] : sa;
    uint32_t mine = 0;                                // lane d: the wave's count for direction d
    for (int64_t c0 = sa + (int64_t)blockIdx.y * LAB_CHUNK; c0 < sb; c0 += (int64_t)gridDim.y * LAB_CHUNK) {
        lab_chunk(L, x, y, surv, c0, min(sb, c0 + LAB_CHUNK), E, m, nullptr);
        int cls, at, len;
        for (int b = w; lab_batch(L, b, &cls, &at, &len); b += LAB_WAVES) {
            const bool has = lane < len;
            const int i = at + min(lane, len - 1);
            const double px = (double)L.x[i] * GRIDD, py = (double)L.y[i] * GRIDD;
            uint64_t lm = ~uint64_t(0);               // the lane's directions
            if (cls < FIXED_SLOTS) lm = dirs[cls];
            else
                for (uint32_t o = L.out[i]; o; o &= o - 1) lm &= dirs[__ffs((int)o) - 1];
            if (!has) lm = 0;
            uint64_t dm = cls < FIXED_SLOTS ? uniform_u64(lm) : wave_or_u64(lm);
            while (dm) {
                const int d = __builtin_ctzll(dm);
                dm &= dm - 1;
                bool in = (lm >> d) & 1;
                in = in && edge_eval(ne[0][0][d], ne[0][1][d], ne[0][2][d], px, py) > 0 &&
                     edge_eval(ne[1][0][d], ne[1][1][d], ne[1][2][d], px, py) > 0;
                const uint32_t c = (uint32_t)__popcll(__ballot(in));
                mine += lane == d ? c : 0;
            }
        }
    }
    wcnt[w][lane] = mine;
    __syncthreads();
    if (tid < NCAND) {
        uint32_t c = 0;
        for (int ww = 0; ww < LAB_WAVES; ww++) c += wcnt[ww][tid];
        if (c) atomicAdd(&cnt[s * NCAND + tid], c);
    }
}

// gain[s][d] = cnt[s][d] / n_s (0 for an empty set).
__global__ void k_label_gain(const int64_t *__restrict__ off, int64_t n1, int64_t S,
                             const uint32_t *__restrict__ cnt, float *__restrict__ gain) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x, s = i / NCAND;
    if (s >= S) return;
    const int64_t n = set_end(off, n1, s) - set_begin(off, s);
    gain[i] = n > 0 ? (float)((double)cnt[i] / (double)n) : 0.0f;
}

// Greedy joint training targets (this project's extension).  One block per
// set.  V starts as the fixed filter's polygon vertices; each of R rounds
// adds the candidate extreme whose polygon hull(V + {e_d}) newly contains,
// strictly inside, the most of the fixed filter's survivors (ties: lowest
// d); a round whose best gain is zero ends the sequence.  Targets: the
// direction chosen in round r gets 1 - r / (2R); every other direction gets
// 0.5 g_d / g_max with g_d its round-0 gain (0 if g_max = 0).
constexpr int LT_MAXR = MAX_DIRS;
constexpr int LT_V = FIXED_SLOTS + LT_MAXR + 1;       // vertices of hull(V + {e_d})

// Edges of the convex hull of k points sorted by (x, y) without repeats
// (Andrew's monotone chain, collinear points dropped); returns the vertex
// count, or 0 when fewer than 3 vertices remain.
__device__ int hull_edges_sorted(const double *px, const double *py, int k, double *ex, double *ey,
                                 double *ec) {
    int st[2 * LT_V + 2];
    int h = 0;
    if (k >= 3) {
        for (int j = 0; j < k; j++) {
            while (h >= 2 && orient(px[st[h - 2]], py[st[h - 2]], px[st[h - 1]], py[st[h - 1]],
                                    px[j], py[j]) <= 0)
                h--;
            st[h++] = j;
        }
        const int lo = h + 1;
        for (int j = k - 2; j >= 0; j--) {
            while (h >= lo && orient(px[st[h - 2]], py[st[h - 2]], px[st[h - 1]], py[st[h - 1]],
                                     px[j], py[j]) <= 0)
                h--;
            st[h++] = j;
        }
        h--;
    }
    if (h < 3) return 0;
    for (int i = 0; i < h; i++) {
        const int p0 = st[i], p1 = st[(i + 1) % h];
        const double ddx = px[p1] - px[p0], ddy = py[p1] - py[p0];
        ex[i] = ddx;
        ey[i] = ddy;
        ec[i] = fma(ddy, px[p0], -(ddx * py[p0]));
    }
    return h;
}

// Insert (gx, gy) into the (x, y)-sorted list of k points unless it is
// already there; writes k' points to (ox, oy) and returns k'.
__device__ int merge_point(const double *vx, const double *vy, int k, double gx, double gy,
                           double *ox, double *oy) {
    int o = 0;
    bool ins = true;
    for (int i = 0; i < k; i++) {
        if (ins && (gx < vx[i] || (gx == vx[i] && gy <= vy[i]))) {
            if (!(gx == vx[i] && gy == vy[i])) { ox[o] = gx; oy[o] = gy; o++; }
            ins = false;
        }
        ox[o] = vx[i]; oy[o] = vy[i]; o++;
    }
    if (ins) { ox[o] = gx; oy[o] = gy; o++; }
    return o;
}

__global__ __launch_bounds__(256) void k_label_targets(
    const float *__restrict__ x, const float *__restrict__ y, const int64_t *__restrict__ off,
    int64_t n1, int64_t S, const Poly *__restrict__ polys, const uint32_t *__restrict__ cand,
    const uint32_t *__restrict__ surv, const int64_t *__restrict__ surv_off, int R,
    float *__restrict__ target, int32_t *__restrict__ order) {
    __shared__ double vx[LT_V], vy[LT_V];                  // current vertex set, sorted
    __shared__ int nv;
    __shared__ double ex[NCAND][LT_V], ey[NCAND][LT_V], ec[NCAND][LT_V];
    __shared__ int ne[NCAND];
    __shared__ double cex[LT_V], cey[LT_V], cec[LT_V];     // hull(V)
    __shared__ int cm;
    __shared__ uint32_t pcnt[4][NCAND];
    __shared__ uint32_t g0[NCAND];
    __shared__ int chosen[LT_MAXR];
    __shared__ int stop;
    const int64_t s = blockIdx.x;
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const int64_t a = set_begin(off, s), n = set_end(off, n1, s) - a;
    const Poly &P = polys[s];
    if (tid == 0) {
        int k = 0;
        for (int i = 0; i < P.m; i++) {       // insertion sort by (x, y)
            const uint32_t id = P.verts[i];
            const double gx = (double)x[id] * GRIDD, gy = (double)y[id] * GRIDD;
            int p = k++;
            while (p > 0 && (vx[p - 1] > gx || (vx[p - 1] == gx && vy[p - 1] > gy))) {
                vx[p] = vx[p - 1]; vy[p] = vy[p - 1];
                p--;
            }
            vx[p] = gx; vy[p] = gy;
        }
        nv = k;
        stop = n <= 0;
    }
    if (tid < LT_MAXR) chosen[tid] = -1;
    __syncthreads();
    const int64_t sa = surv_off[s], sb = surv_off[s + 1];
    for (int r = 0; r < R && !stop; r++) {
        if (tid < NCAND) {
            const uint32_t e = cand[s * NCAND + tid];
            double px[LT_V], py[LT_V];
            int k = nv;
            if (e != NONE) {
                k = merge_point(vx, vy, nv, (double)x[e] * GRIDD, (double)y[e] * GRIDD, px, py);
            } else {
                for (int i = 0; i < nv; i++) { px[i] = vx[i]; py[i] = vy[i]; }
            }
            ne[tid] = hull_edges_sorted(px, py, k, ex[tid], ey[tid], ec[tid]);
        } else if (tid == NCAND) {
            cm = hull_edges_sorted(vx, vy, nv, cex, cey, cec);
        }
        __syncthreads();
        uint32_t cnt[NCAND];
#pragma unroll
        for (int d = 0; d < NCAND; d++) cnt[d] = 0;
        for (int64_t j = sa + tid; j < sb; j += blockDim.x) {
            const uint32_t id = surv[j];
            const double qx = (double)x[id] * GRIDD, qy = (double)y[id] * GRIDD;
            bool in = cm >= 3;
            for (int i = 0; i < cm && in; i++) in = edge_eval(cex[i], cey[i], cec[i], qx, qy) > 0;
            if (in) continue;                 // already inside hull(V): no candidate gains it
#pragma unroll
            for (int d = 0; d < NCAND; d++) {
                const int m = ne[d];
                bool ind = m >= 3;
                for (int i = 0; i < m && ind; i++) ind = edge_eval(ex[d][i], ey[d][i], ec[d][i], qx, qy) > 0;
                cnt[d] += ind;
            }
        }
#pragma unroll
        for (int d = 0; d < NCAND; d++) {
            uint32_t c = cnt[d];
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o);
            if (lane == 0) pcnt[w][d] = c;
        }
        __syncthreads();
        if (tid == 0) {
            int best = -1;
            uint32_t bc = 0;
            for (int d = 0; d < NCAND; d++) {
                uint32_t c = 0;
                for (int ww = 0; ww < (int)(blockDim.x >> 6); ww++) c += pcnt[ww][d];
                if (r == 0) g0[d] = c;
                if (c > bc) { bc = c; best = d; }
            }
            if (best < 0) {
                stop = 1;
            } else {
                chosen[r] = best;
                const uint32_t e = cand[s * NCAND + best];
                double tx[LT_V], ty[LT_V];
                const int k = merge_point(vx, vy, nv, (double)x[e] * GRIDD, (double)y[e] * GRIDD, tx, ty);
                for (int i = 0; i < k; i++) { vx[i] = tx[i]; vy[i] = ty[i]; }
                nv = k;
            }
        }
        __syncthreads();
    }
    if (tid < NCAND) {
        uint32_t gmax = 0;
        bool g0_set = !(n <= 0);
        for (int d = 0; d < NCAND && g0_set; d++) gmax = max(gmax, g0[d]);
        float t = (g0_set && gmax > 0) ? (float)(0.5 * ((double)g0[tid] / (double)gmax)) : 0.0f;
        for (int r = 0; r < R; r++)
            if (chosen[r] == tid) t = (float)(1.0 - (double)r / (2.0 * R));
        target[s * NCAND + tid] = t;
    }
    if (tid < R) order[s * R + tid] = chosen[tid];
}

struct LearnedState {
    bool loaded = false;
    int64_t bcap = 0;          // rows the activation buffers hold
    int64_t step = 0;          // Adam step counter
    float *params = nullptr, *grads = nullptr, *m1 = nullptr, *m2 = nullptr;
    bf16_t *wb = nullptr;      // bf16 weight matrices
    bf16_t *X = nullptr, *H1 = nullptr, *H2 = nullptr, *dS = nullptr, *dZ2 = nullptr;
    // transposes, [columns][rows]
    bf16_t *XT = nullptr, *H1T = nullptr, *H2T = nullptr, *dST = nullptr, *dZ2T = nullptr, *dZ1T = nullptr;
    float *scores = nullptr, *part = nullptr;
};

static size_t learned_ws_bytes(int64_t S) {
    return (size_t)S * HBINS * sizeof(bf16_t) + (size_t)S * NCAND * sizeof(float) + 256;
}

static void learned_free(LearnedState &L) {
    void *ps[] = {L.params, L.grads, L.m1, L.m2, L.wb, L.X, L.H1, L.H2, L.dS, L.dZ2, L.XT, L.H1T, L.H2T,
                  L.dST, L.dZ2T, L.dZ1T, L.scores, L.part};
    for (void *p : ps)
        if (p) (void)hipFree(p);
    L = LearnedState();
}

}  // namespace hg
