// Learned preconditioner: per-event grid-count features, a 12 -> 64 -> 64 -> 1
// tanh network (forward, back-propagation, Adam) and the running-average mass
// update that consumes either its prediction or the exact Hessian diagonal.
//
// The network predicts, from cheap features of free event m, log H_m: the log
// of Eq. 5's Hessian diagonal, which the paper uses as the HMC mass.  The mass
// formed from it is theta_m^2 exp(prediction) + P_mm (the prior's precision
// added when the mass is formed).  The exact column pass remains the training
// target, the periodic fallback and the judge, so the sampler stays exact: any
// positive mass leaves the target distribution invariant.
//
// hawkes_mlp_train_step_noalloc is the training step for callers that cannot
// allocate: its workspace and gradient live in a fixed device array of this
// file (one copy per GPU, held until the process ends).
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <mutex>

#include "hawkes_internal.h"

#define MLP_IN 12
#define MLP_H 64
#define MLP_OFF_W1 0
#define MLP_OFF_B1 (MLP_OFF_W1 + MLP_H * MLP_IN)
#define MLP_OFF_W2 (MLP_OFF_B1 + MLP_H)
#define MLP_OFF_B2 (MLP_OFF_W2 + MLP_H * MLP_H)
#define MLP_OFF_W3 (MLP_OFF_B2 + MLP_H)
#define MLP_OFF_B3 (MLP_OFF_W3 + MLP_H)
#define MLP_NP (MLP_OFF_B3 + 1)

static_assert(MLP_NP == 5057, "parameter count");

namespace {

inline unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

// ---- network -----------------------------------------------------------------------------
// A batch row index outside [0, n_rows) is not read: the sample is dropped
// (zero input, zero target weight) and bit 1 of *err is set.
__device__ __forceinline__ int64_t checked_row(const int *rows, int64_t s, int64_t n_rows, int *err, bool &ok) {
    const int64_t row = rows ? (int64_t)rows[s] : s;
    ok = row >= 0 && row < n_rows;
    if (!ok && err) atomicOr(err, 1);
    return ok ? row : 0;
}

// The network's batch kernel: forward (GRAD = false: y only) or forward,
// back-propagation and the weight gradient's partial sums in one pass.
//
// What bounds it: a batch is 1e8 operations, below a microsecond of the chip, so
// the cost is the chain of dependent steps.  A block of eight wavefronts takes 32
// samples at a time: wavefront (sg, ng) has 16 samples and 16 of the 64 neurons,
// so each layer is one short chain of FP32 matrix instructions (16x16x4) per
// wavefront, with the weights held in registers for the whole kernel and the
// activations passed through LDS (rows padded to 68 floats: 16-byte aligned and
// four banks apart).  The contraction index is permuted the same way on both
// sides (lane group q holds k = 16 q + t at step t), so that a lane reads its
// operands as contiguous runs.
//
// The weight gradient is a contraction over the batch in FP64 (exact products of
// FP32 factors): FP64 matrix instructions (16x16x4) over the 32 samples in LDS,
// accumulated in registers over the block's groups, one slice of MLP_NP sums per
// block at the end; k_mlp_apply adds the slices in a fixed order.  A batch of
// 4,096 rows takes 128 blocks.  Batch 4,096: one thread per sample and one
// wavefront per parameter took 190 us a step in five kernels; this form takes 17.5
// in two (13.4 here, 4.1 in k_mlp_apply).
constexpr int MLP_BS = 32;        // samples per block and group
constexpr int MLP_LDH = MLP_H + 4;
constexpr int MLP_THREADS = 512;
constexpr int64_t MLP_MAX_BLOCKS = 256;  // slices of partial sums (40 KB each)

typedef float mlp_f4 __attribute__((ext_vector_type(4)));
typedef double mlp_d4 __attribute__((ext_vector_type(4)));

inline int mlp_blocks(int64_t B) { return (int)std::min<int64_t>(MLP_MAX_BLOCKS, (B + MLP_BS - 1) / MLP_BS); }

// sum over the 16 lanes that share lane / 16 (fixed order; every lane gets it)
__device__ __forceinline__ double sum16(double v) {
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) v += __shfl_xor(v, off);
    return v;
}

template <bool GRAD>
__global__ __launch_bounds__(MLP_THREADS) void k_mlp_batch(const float *__restrict__ params, const float *__restrict__ X,
                                                           int64_t n_rows, const int *__restrict__ rows,
                                                           const float *__restrict__ target, int64_t B,
                                                           float *__restrict__ y_out, double *__restrict__ part,
                                                           double *__restrict__ loss_part, int *__restrict__ err) {
    struct Lds {
        float h1[MLP_BS][MLP_LDH];
        double ysum[MLP_BS / 16][4][16];
        float d1[GRAD ? MLP_BS : 1][MLP_LDH];
        float d2[GRAD ? MLP_BS : 1][MLP_LDH];
        float x[GRAD ? MLP_BS : 1][16];  // columns 12..15 stay zero
        double bsum[GRAD ? 3 : 1][MLP_H];
        double ssum[2];
        double w1[GRAD ? 4 : 1][4][HK_WAVE];
    };
    __shared__ Lds L;
    const int tid = threadIdx.x, lane = tid & (HK_WAVE - 1), w = __builtin_amdgcn_readfirstlane(tid / HK_WAVE);
    const int ng = w & 3, sg = w >> 2, q = lane >> 4, c = lane & 15;
    // a lane's weights: rows of its 16 neurons as left operands (and, for the
    // backward pass, columns), its four output neurons 4 q + r of each layer
    float w1[3], w2[16], w2t[16], b1[4], b2[4], w3[4];
#pragma unroll
    for (int t = 0; t < 3; ++t) w1[t] = params[MLP_OFF_W1 + (ng * 16 + c) * MLP_IN + q * 3 + t];
    __builtin_memcpy(w2, params + MLP_OFF_W2 + (ng * 16 + c) * MLP_H + q * 16, sizeof(w2));
#pragma unroll
    for (int t = 0; t < 16; ++t) w2t[t] = GRAD ? params[MLP_OFF_W2 + (q * 16 + t) * MLP_H + ng * 16 + c] : 0.0f;
    const int k0 = ng * 16 + 4 * q;
    __builtin_memcpy(b1, params + MLP_OFF_B1 + k0, sizeof(b1));
    __builtin_memcpy(b2, params + MLP_OFF_B2 + k0, sizeof(b2));
    __builtin_memcpy(w3, params + MLP_OFF_W3 + k0, sizeof(w3));
    const float b3 = params[MLP_OFF_B3];

    double g_b1[4] = {}, g_b2[4] = {}, g_w3[4] = {}, g_b3 = 0.0, r2 = 0.0;
    mlp_d4 gA = {}, gB = {}, gX = {};
    const int kt = w >> 1, jt = (w & 1) * 2;  // the wavefront's tiles of the W2 gradient: (kt, jt), (kt, jt + 1)
    if (GRAD) L.x[tid / 16][tid & 15] = 0.0f;

    for (int64_t g0 = (int64_t)blockIdx.x * MLP_BS; g0 < B; g0 += (int64_t)gridDim.x * MLP_BS) {
        const int si = sg * 16 + c;
        const int64_t s = g0 + si;
        const bool live = s < B;
        bool ok = false;
        int64_t row = 0;
        if (live) row = checked_row(rows, s, n_rows, err, ok);
        float x[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) x[t] = ok ? X[row * MLP_IN + q * 3 + t] : 0.0f;
        float tgt = 0.0f;
        if (GRAD && ok) tgt = target[row];
        // layer 1
        mlp_f4 a = {b1[0], b1[1], b1[2], b1[3]};
#pragma unroll
        for (int t = 0; t < 3; ++t) a = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[t], x[t], a, 0, 0, 0);
        mlp_f4 h1;
#pragma unroll
        for (int r = 0; r < 4; ++r) h1[r] = live ? tanhf(a[r]) : 0.0f;
        if (GRAD) __syncthreads();  // the previous group's weight gradient has read the arrays
        *(mlp_f4 *)&L.h1[si][k0] = h1;
        if (GRAD && ng == 0) {
#pragma unroll
            for (int t = 0; t < 3; ++t) L.x[si][q * 3 + t] = x[t];
        }
        __syncthreads();
        // layer 2
        float bop[16];
#pragma unroll
        for (int t = 0; t < 4; ++t) *(mlp_f4 *)&bop[4 * t] = *(const mlp_f4 *)&L.h1[si][q * 16 + 4 * t];
        a = mlp_f4{b2[0], b2[1], b2[2], b2[3]};
#pragma unroll
        for (int t = 0; t < 16; ++t) a = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[t], bop[t], a, 0, 0, 0);
        // the output is summed in FP64: an FP32 sum's error is most of what separates
        // the gradient (a sum of residuals that nearly cancel) from its FP64 value
        mlp_f4 h2;
        double yp = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            h2[r] = tanhf(a[r]);
            yp = fma((double)w3[r], (double)h2[r], yp);
        }
        // output: the lane groups' and wavefronts' partial sums
        yp += __shfl_xor(yp, 16);
        yp += __shfl_xor(yp, 32);
        if (q == 0) L.ysum[sg][ng][c] = yp;
        __syncthreads();
        const double y = ((L.ysum[sg][0][c] + L.ysum[sg][1][c]) + L.ysum[sg][2][c]) + L.ysum[sg][3][c] + (double)b3;
        if (!GRAD) {
            if (live && ng == 0 && q == 0) y_out[s] = (float)y;
            continue;  // the next group's writes of h1 follow this group's ysum barrier
        }
        // back-propagation: dy = 2 (y - t) / B, d2 = dy w3 (1 - h2^2), d1 = (W2^T d2) (1 - h1^2)
        const float r = ok ? (float)(y - (double)tgt) : 0.0f;
        const float dy = 2.0f * r / (float)B;
        if (ng == 0 && q == 0) {
            r2 += (double)r * (double)r;
            g_b3 += (double)dy;
        }
        mlp_f4 d2;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            d2[k] = live ? dy * w3[k] * (1.0f - h2[k] * h2[k]) : 0.0f;
            g_b2[k] += (double)d2[k];
            g_w3[k] += live ? (double)dy * (double)h2[k] : 0.0;
        }
        *(mlp_f4 *)&L.d2[si][k0] = d2;
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 4; ++t) *(mlp_f4 *)&bop[4 * t] = *(const mlp_f4 *)&L.d2[si][q * 16 + 4 * t];
        a = mlp_f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int t = 0; t < 16; ++t) a = __builtin_amdgcn_mfma_f32_16x16x4f32(w2t[t], bop[t], a, 0, 0, 0);
        mlp_f4 d1;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            d1[k] = live ? a[k] * (1.0f - h1[k] * h1[k]) : 0.0f;
            g_b1[k] += (double)d1[k];
        }
        *(mlp_f4 *)&L.d1[si][k0] = d1;
        __syncthreads();
        // weight gradients over the 32 samples: four per matrix instruction; the
        // two wavefronts of a row kt share its W1 tile, half of the samples each
#pragma unroll
        for (int u = 0; u < MLP_BS / 4; ++u) {
            const int e = 4 * u + q;
            const double da = (double)L.d2[e][kt * 16 + c];
            gA = __builtin_amdgcn_mfma_f64_16x16x4f64(da, (double)L.h1[e][jt * 16 + c], gA, 0, 0, 0);
            gB = __builtin_amdgcn_mfma_f64_16x16x4f64(da, (double)L.h1[e][jt * 16 + 16 + c], gB, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < MLP_BS / 8; ++u) {
            const int e = 4 * ((w & 1) * (MLP_BS / 8) + u) + q;
            gX = __builtin_amdgcn_mfma_f64_16x16x4f64((double)L.d1[e][kt * 16 + c], (double)L.x[e][c], gX, 0, 0, 0);
        }
    }
    if (!GRAD) return;
    // the block's slice of partial sums; the FP64 matrix result holds row 4 r + q, column c
    double *out = part + (int64_t)blockIdx.x * MLP_NP;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        double *o = out + MLP_OFF_W2 + (kt * 16 + 4 * r + q) * MLP_H + jt * 16 + c;
        o[0] = gA[r];
        o[16] = gB[r];
        if (w & 1) L.w1[kt][r][lane] = gX[r];
        g_b1[r] = sum16(g_b1[r]);
        g_b2[r] = sum16(g_b2[r]);
        g_w3[r] = sum16(g_w3[r]);
    }
    r2 = sum16(r2);
    g_b3 = sum16(g_b3);
    if (sg == 1 && c == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            L.bsum[0][k0 + r] = g_b1[r];
            L.bsum[1][k0 + r] = g_b2[r];
            L.bsum[2][k0 + r] = g_w3[r];
        }
        if (ng == 0 && q == 0) {
            L.ssum[0] = g_b3;
            L.ssum[1] = r2;
        }
    }
    __syncthreads();
    if (!(w & 1) && c < MLP_IN) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            out[MLP_OFF_W1 + (kt * 16 + 4 * r + q) * MLP_IN + c] = gX[r] + L.w1[kt][r][lane];
    }
    if (sg == 0 && c == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            out[MLP_OFF_B1 + k0 + r] = g_b1[r] + L.bsum[0][k0 + r];
            out[MLP_OFF_B2 + k0 + r] = g_b2[r] + L.bsum[1][k0 + r];
            out[MLP_OFF_W3 + k0 + r] = g_w3[r] + L.bsum[2][k0 + r];
        }
        if (ng == 0 && q == 0) {
            out[MLP_OFF_B3] = g_b3 + L.ssum[0];
            loss_part[blockIdx.x] = r2 + L.ssum[1];
        }
    }
}

// The gradient from the blocks' slices (64 parameters per block, the slices
// split over eight wavefronts and combined in a fixed order), the loss in one
// block more, and, with ADAM, the update (Kingma & Ba 2015, bias-corrected, step
// t >= 1) of the parameters in place.  Reads 40 KB per slice (5 MB at batch 4,096).
struct AdamArgs {
    float *params, *m, *v;
    int t;
    float lr, b1, b2, eps;
};

constexpr int MLP_APPLY_WAVES = 8;
template <bool ADAM>
__global__ __launch_bounds__(MLP_APPLY_WAVES * HK_WAVE) void k_mlp_apply(const double *__restrict__ part,
                                                                       const double *__restrict__ loss_part,
                                                                       int slices, int64_t B, double *__restrict__ grad,
                                                                       double *__restrict__ loss, const AdamArgs ad) {
    __shared__ double sh[MLP_APPLY_WAVES][HK_WAVE];
    const int lane = threadIdx.x & (HK_WAVE - 1), w = threadIdx.x / HK_WAVE;
    const bool is_loss = blockIdx.x == (MLP_NP + HK_WAVE - 1) / HK_WAVE;
    const int p = blockIdx.x * HK_WAVE + lane;
    double acc = 0.0;
    if (is_loss) {
        for (int k = w * HK_WAVE + lane; k < slices; k += MLP_APPLY_WAVES * HK_WAVE) acc += loss_part[k];
    } else if (p < MLP_NP) {
#pragma unroll 8
        for (int k = w; k < slices; k += MLP_APPLY_WAVES) acc += part[(int64_t)k * MLP_NP + p];
    }
    sh[w][lane] = acc;
    __syncthreads();
    if (w != 0) return;
#pragma unroll
    for (int k = 1; k < MLP_APPLY_WAVES; ++k) acc += sh[k][lane];
    if (is_loss) {
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
        if (lane == 0 && loss) loss[0] = acc / (double)B;
        return;
    }
    if (p >= MLP_NP) return;
    grad[p] = acc;
    if (ADAM) {
        const float g = (float)acc;
        const float mq = ad.b1 * ad.m[p] + (1.0f - ad.b1) * g;
        const float vq = ad.b2 * ad.v[p] + (1.0f - ad.b2) * g * g;
        ad.m[p] = mq;
        ad.v[p] = vq;
        const float mh = mq / (1.0f - powf(ad.b1, (float)ad.t));
        const float vh = vq / (1.0f - powf(ad.b2, (float)ad.t));
        ad.params[p] -= ad.lr * mh / (sqrtf(vh) + ad.eps);
    }
}

// ---- features -------------------------------------------------------------------------------
// Disc and time-window counts around each free event, exact by their
// definition: a counting sort of all events by grid cell gives each free event
// the candidates near it, and what decides a count is the FP64 distance and
// time of each candidate.  Distances are dx * dx + dy * dy and radii r * r, each
// rounded once in FP64 (no contraction), so every count is the same integer as
// the definition's.
//
// The sort takes the events in time order in `nb` runs of `per` events, and
// keeps every cell's events in the order of the runs: off[b (cells + 1) + c] is
// the first of cell c's events from runs >= b.  A free event's time windows
// (-1/omega .. 6/omega: a few of hundreds of 1/omega) then meet only the cell's
// events of two or three runs, and the two counts over all times need a
// distance alone.  Cells are h wide where at most kFeatCells of them cover the
// events (else 2 h or 3 h, else 3 h and one run): a cell inside the 3h disc is
// counted whole, so only the cells that a circle crosses are tested.
//
// N = 100,000, 6,874 free events: cells of 3h whose every event was tested for
// all nine sums, in two passes, took 257 us (bound by L2: 3 GB of candidates)
// after 123 us of counting sort by global atomics (contended in the clusters);
// this form 49 us after 23 (sums of 440 and 75 us per prediction with the network).
struct FeatGrid {
    double gx0, gy0, s;  // origin and cell size
    int nx, ny;
    int nb, per;         // runs of the time-ordered events, events per run
};

// The discs and windows, formed once on the host (FP64 divisions cost a wavefront
// some 20 instructions each).
struct FeatConst {
    double r0, r1;          // squared radii h^2, (3h)^2
    double w1, w3, w6;      // 1, 3 and 6 over omega
    double inv_h2, inv_s;   // 1 / h^2, 1 / cell
    double R0, R1;          // the radii in cells
    double omega;
};

constexpr int kFeatCells = 8192;  // cells of a run's histogram in LDS (32 KB)
constexpr int kFeatRuns = 64;     // one lane per run in k_features
constexpr int kFeatGroup = HK_WAVE;  // cells per block of the offsets kernel, a lane each
constexpr int kFeatOffWaves = 4;     // its wavefronts, a quarter of the runs each
constexpr int kFeatThreads = 1024;
constexpr int kFeatWindows = 2;   // columns whose windows' candidates a lane loads together
constexpr int kFeatTests = 8;     // candidates a lane of k_features loads together
// candidates of one cell's windows above which the whole wavefront takes them: where a
// few crowded cells hold most of a free event's windows, the other lane groups waited
// for the one that had them (N = 100,000, 400 free events, h = 4, omega = 0.001 / 0.5
// with 6,874 of h = 1, us: lane groups alone 4,993 / 171, 512 999 / 171, 128 1,000 / 170,
// 32 992 / 162; 6,874 of h = 0.3, omega = 0.01, lists of some 40: 118, 115, 116, 121)
constexpr int kFeatLong = 32;
constexpr int kFeatBatch = 4;     // events a thread of the sort loads together

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return min(max(v, lo), hi); }

__device__ __forceinline__ int cell_x(double x, const FeatGrid &G) {
    return clampi((int)floor((x - G.gx0) / G.s), 0, G.nx - 1);
}
__device__ __forceinline__ int cell_y(double y, const FeatGrid &G) {
    return clampi((int)floor((y - G.gy0) / G.s), 0, G.ny - 1);
}
__device__ __forceinline__ int64_t cell_of(const double *__restrict__ xy, int64_t e, const FeatGrid &G) {
    return (int64_t)cell_y(xy[2 * e + 1], G) * G.nx + cell_x(xy[2 * e], G);
}

// Per run (one block): its events per cell, and their sums over kFeatGroup cells.
__global__ __launch_bounds__(kFeatThreads) void k_cell_hist(const double *__restrict__ xy, const int *__restrict__ perm,
                                                           int64_t n, const FeatGrid G, int *__restrict__ off,
                                                           int *__restrict__ gsum) {
    __shared__ __attribute__((aligned(16))) int cnt[kFeatCells];
    const int cells = G.nx * G.ny, b = blockIdx.x;
    for (int c = threadIdx.x; c < kFeatCells; c += kFeatThreads) cnt[c] = 0;
    const int64_t i1 = min(n, (int64_t)(b + 1) * G.per);
    for (int64_t i0 = (int64_t)b * G.per; i0 < i1; i0 += kFeatBatch * kFeatThreads) {
        int cell[kFeatBatch];
#pragma unroll
        for (int k = 0; k < kFeatBatch; ++k) {
            const int64_t i = i0 + k * kFeatThreads + threadIdx.x;
            cell[k] = i < i1 ? (int)cell_of(xy, perm[i], G) : -1;
        }
        if (i0 == (int64_t)b * G.per) __syncthreads();
#pragma unroll
        for (int k = 0; k < kFeatBatch; ++k)
            if (cell[k] >= 0) atomicAdd(&cnt[cell[k]], 1);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < cells; c += kFeatThreads) off[(int64_t)b * (cells + 1) + c] = cnt[c];
    // a thread's cells, then the threads of a group
    constexpr int own = kFeatCells / kFeatThreads, thr = kFeatGroup / own;
    int v = 0;
#pragma unroll
    for (int k = 0; k < own; ++k) v += cnt[threadIdx.x * own + k];
    for (int o = 1; o < thr; o <<= 1) v += __shfl_xor(v, o);
    if (threadIdx.x % thr == 0) gsum[(threadIdx.x * own + b * kFeatCells) / kFeatGroup] = v;
}

// Counts to offsets in place: a block has kFeatGroup cells; the events of the
// groups before it come from the runs' sums.  Bound by the latency of its loads:
// N = 100,000 (6,806 cells, 64 runs) 5.4 us, with 256 cells per block and
// every run of a cell in one thread 9.8.
__global__ __launch_bounds__(kFeatOffWaves * HK_WAVE) void k_cell_off(const int *__restrict__ gsum, int64_t n,
                                                                      const FeatGrid G, int *__restrict__ off) {
    constexpr int groups = kFeatCells / kFeatGroup, threads = kFeatOffWaves * HK_WAVE;
    constexpr int per = kFeatRuns / kFeatOffWaves;
    __shared__ int before[kFeatOffWaves], tot[kFeatOffWaves][HK_WAVE];
    const int lane = threadIdx.x % HK_WAVE, w = threadIdx.x / HK_WAVE;
    const int cells = G.nx * G.ny, c = blockIdx.x * kFeatGroup + lane;
    // the cell's counts of the wavefront's runs, loaded together
    int cnt[per], sum = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const int b = w * per + k;
        cnt[k] = b < G.nb && c < cells ? off[(int64_t)b * (cells + 1) + c] : 0;
    }
    int v = 0;
#pragma unroll 8
    for (int k = threadIdx.x; k < G.nb * groups; k += threads) v += k % groups < (int)blockIdx.x ? gsum[k] : 0;
    for (int o = HK_WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (lane == 0) before[w] = v;
#pragma unroll
    for (int k = 0; k < per; ++k) sum += cnt[k];
    tot[w][lane] = sum;
    __syncthreads();
    int all = 0, run = 0;
#pragma unroll
    for (int q = 0; q < kFeatOffWaves; ++q) {
        run += before[q] + (q < w ? tot[q][lane] : 0);
        all += tot[q][lane];
    }
    run -= all;
    for (int o = 1; o < HK_WAVE; o <<= 1) {  // the cells before it in the group
        const int u = __shfl_up(all, o);
        if (lane >= o) all += u;
    }
    run += all;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        const int b = w * per + k;
        if (b < G.nb && c < cells) off[(int64_t)b * (cells + 1) + c] = run;
        run += cnt[k];
    }
    if (c == 0 && w == 0) off[cells] = (int)n;  // end of the last cell
}

// Per run: its events to their places (the order inside a cell and run does not
// matter: counts are integers and feature 8 is summed in fixed point).
__global__ __launch_bounds__(kFeatThreads) void k_cell_place(const double *__restrict__ t, const double *__restrict__ xy,
                                                            const int *__restrict__ perm, int64_t n, const FeatGrid G,
                                                            const int *__restrict__ off, double *__restrict__ ct,
                                                            double2 *__restrict__ cxy) {
    __shared__ int next[kFeatCells];
    const int cells = G.nx * G.ny, b = blockIdx.x;
    constexpr int own = kFeatCells / kFeatThreads;
    int first[own];  // loaded together
#pragma unroll
    for (int k = 0; k < own; ++k) {
        const int c = threadIdx.x + k * kFeatThreads;
        first[k] = c < cells ? off[(int64_t)b * (cells + 1) + c] : 0;
    }
#pragma unroll
    for (int k = 0; k < own; ++k) next[threadIdx.x + k * kFeatThreads] = first[k];
    const int64_t i1 = min(n, (int64_t)(b + 1) * G.per);
    for (int64_t i0 = (int64_t)b * G.per; i0 < i1; i0 += kFeatBatch * kFeatThreads) {
        double x[kFeatBatch], y[kFeatBatch], tt[kFeatBatch];
#pragma unroll
        for (int k = 0; k < kFeatBatch; ++k) {
            const int64_t i = i0 + k * kFeatThreads + threadIdx.x;
            const int64_t e = i < i1 ? perm[i] : 0;
            x[k] = xy[2 * e];
            y[k] = xy[2 * e + 1];
            tt[k] = t[e];
        }
        if (i0 == (int64_t)b * G.per) __syncthreads();
#pragma unroll
        for (int k = 0; k < kFeatBatch; ++k) {
            if (i0 + k * kFeatThreads + threadIdx.x >= i1) break;
            const int q = atomicAdd(&next[cell_y(y[k], G) * G.nx + cell_x(x[k], G)], 1);
            ct[q] = tt[k];
            cxy[q] = make_double2(x[k], y[k]);
        }
    }
}

// The same sort with one run for grids too large for LDS (a wide domain over
// small cells: few events share one), by global atomics.
__global__ void k_fill_zero(int *__restrict__ a, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = 0;
}

__global__ void k_cell_count(const double *__restrict__ xy, int64_t n, const FeatGrid G, int *__restrict__ cnt) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= n) return;
    atomicAdd(&cnt[cell_of(xy, e, G)], 1);
}

// Exclusive scan of the cell counts by one block: each thread scans a
// contiguous segment, the segment totals are scanned in LDS, then each thread
// writes its segment's offsets.  start[cells] = n.  fill is cleared for the
// scatter.
constexpr int kScanThreads = 1024;
__global__ __launch_bounds__(kScanThreads) void k_cell_scan(const int *__restrict__ cnt, int64_t cells,
                                                           int *__restrict__ start, int *__restrict__ fill) {
    __shared__ int tot[kScanThreads];
    const int64_t seg = (cells + kScanThreads - 1) / kScanThreads;
    const int64_t lo = min(cells, threadIdx.x * seg), hi = min(cells, lo + seg);
    int sum = 0;
    for (int64_t c = lo; c < hi; ++c) sum += cnt[c];
    tot[threadIdx.x] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int k = 0; k < kScanThreads; ++k) {
            const int v = tot[k];
            tot[k] = run;
            run += v;
        }
        start[cells] = run;
    }
    __syncthreads();
    int run = tot[threadIdx.x];
    for (int64_t c = lo; c < hi; ++c) {
        start[c] = run;
        run += cnt[c];
        fill[c] = 0;
    }
}

__global__ void k_cell_scatter(const double *__restrict__ t, const double *__restrict__ xy, int64_t n,
                               const FeatGrid G, const int *__restrict__ start, int *__restrict__ fill,
                               double *__restrict__ ct, double2 *__restrict__ cxy) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int64_t c = cell_of(xy, e, G);
    const int64_t q = start[c] + atomicAdd(&fill[c], 1);
    ct[q] = t[e];
    cxy[q] = make_double2(xy[2 * e], xy[2 * e + 1]);
}

// One wavefront per free event; its lanes take the grid rows of the 3h disc
// side by side (8 or 16 lanes a row) to find the rows' ranges and for the time
// windows, and the whole wavefront goes through one range of candidates after the
// other for the counts over all times.  The counts are summed across the wavefront
// (integers: exact in any order).
//
// Bound by its instructions, mostly the tests, and by how the wavefronts fill the
// chip (N = 100,000, 6,874 free events, 6.7 wavefronts per SIMD): candidates side
// by side, a row per lane group, left most lanes idle behind the longest row (a
// wavefront 3,580 vector instructions, 79 us); ranges one by one 2,600 and 62 us;
// constants formed on the host, blocks of one wavefront and seven of them per
// SIMD, so that all are in flight at once, 49 us (six: 52; eight spill).
//
// A cell counts as inside the 3h disc, or as out of reach of a disc, with a
// margin of 1e-6 cells, far above the rounding of its edges (positions relative
// to the grid's origin are within 2^26 2^-53 cells); whatever is nearer is
// tested.  The runs a time window meets are found with a margin in the same way.
//
// Feature 8 is the forward sum of the squared excitation kernel,
//   S_m = sum over e with r2_e < (3h)^2, 0 < dt_e <= 6/omega of
//         exp(a_e),  a_e = -2 omega dt_e - r2_e / h^2,
// which is Eq. 5's H_m without the weights c_e / lambda_e: as
// max(log2 S_m, HK_KSUM_LOG2_FLOOR) / 8.  The candidates' order in the cells
// depends on the grid's scatter, so the sum is formed in a way that does not
// depend on it: the largest exponent a_max (a maximum is exact) and then
// sum_e rint(2^36 exp(a_e - a_max)) in 64-bit integers (exact up to 2^27
// terms), each exponential by the FP32 exp2 (a feature needs no more).
__global__ __launch_bounds__(HK_WAVE, 7) void k_features(const double *__restrict__ t, const double *__restrict__ xy,
                                                  const int64_t *__restrict__ cidx, const int *__restrict__ pos,
                                                  const int *__restrict__ slot, const int *__restrict__ g,
                                                  const double *__restrict__ ts, const double *__restrict__ z,
                                                  int64_t m, int64_t n, double t0, double t1, const FeatConst F,
                                                  const FeatGrid G, const int *__restrict__ off,
                                                  const double *__restrict__ ct, const double2 *__restrict__ cxy,
                                                  float *__restrict__ feat) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x, r = blockIdx.x, k = slot[r];
    const int64_t e = cidx[k];
    const double xm = xy[2 * e], ym = xy[2 * e + 1], tm = t[e];
    const double r0 = F.r0, r1 = F.r1, w1 = F.w1, w3 = F.w3, w6 = F.w6;
    // the runs that hold events of the time windows: the last one that starts
    // before the earliest window, up to the last that starts inside the latest
    int b_lo = 0, b_hi = 0;
    if (G.nb > 1) {
        const double slack = 1e-9 * w6 + 1e-15 * fabs(tm);
        const bool in = lane < G.nb && (int64_t)lane * G.per < n;
        const double tb = in ? ts[(int64_t)lane * G.per] : INFINITY;
        b_lo = max(0, (int)__popcll(__ballot(tb < tm - w1 - slack)) - 1);
        b_hi = max(b_lo, (int)__popcll(__ballot(tb <= tm + w6 + slack)) - 1);
    }
    const int64_t stride = (int64_t)G.nx * G.ny + 1;
    const int *__restrict__ w_lo = off + b_lo * stride;
    // (past the last run a cell ends where the next begins)
    const int *__restrict__ w_hi = b_hi + 1 < G.nb ? off + (b_hi + 1) * stride : off + 1;
    // positions in cells relative to the grid's origin
    const double um = (xm - G.gx0) * F.inv_s, vm = (ym - G.gy0) * F.inv_s;
    const double R0 = F.R0, R1 = F.R1, tol = 1e-6;
    const int y_lo = clampi((int)floor(vm - R1 - tol), 0, G.ny - 1), y_hi = clampi((int)floor(vm + R1 + tol), 0, G.ny - 1);
    // at most 8 rows and columns (6 h over cells of at least h)
    const int lpr = y_hi - y_lo < 4 ? 16 : 8;
    const int lr = lane % lpr, yy = y_lo + lane / lpr;
    const int64_t row = (int64_t)yy * G.nx;
    const bool live = yy <= y_hi;

    int c[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int xa = 0, xb = -1;  // the columns the 3h disc reaches in the lane's row
    // the row's candidates: [la, lb) and [ra, rb) for the 3h disc, [ha, hb) for the h disc
    int la = 0, lb = 0, ra = 0, rb = 0, ha = 0, hb = 0;
    int wq = 0, wn = 0;   // first event and number of events in the time windows' runs, of column xa + lr
    if (live) {
        // least and largest distance in y to the row's cells
        const double below = (double)yy - vm, above = (double)(yy + 1) - vm;
        const double dn = fmax(0.0, fmax(below, -above)), df = fmax(fabs(below), fabs(above));
        // the 3h disc: cells it reaches, cells inside it
        const double wo = sqrt(fmax(0.0, R1 * R1 - dn * dn)) + tol;
        xa = clampi((int)floor(um - wo), 0, G.nx - 1);
        xb = clampi((int)floor(um + wo), 0, G.nx - 1);
        if (lr <= xb - xa) {
            wq = w_lo[row + xa + lr];
            wn = w_hi[row + xa + lr] - wq;
        }
        const double wi = sqrt(fmax(0.0, R1 * R1 - df * df)) - tol;
        const int xi = max(xa, (int)floor(um - wi) + 1), xj = min(xb, (int)floor(um + wi) - 1);
        const int qa = off[row + xa], qb = off[row + xb + 1];
        int qi = qb, qj = qb;  // [qa, qi) and [qj, qb) are tested, [qi, qj) counted whole
        if (wi > 0.0 && xi <= xj) {
            qi = off[row + xi];
            qj = off[row + xj + 1];
            if (lr == 0) c[1] += qj - qi;
        }
        la = qa;
        lb = qi;
        ra = qj;
        rb = qb;
        // the h disc over all times
        if (dn <= R0 + tol) {
            const double wh = sqrt(fmax(0.0, R0 * R0 - dn * dn)) + tol;
            const int x0 = clampi((int)floor(um - wh), 0, G.nx - 1), x1 = clampi((int)floor(um + wh), 0, G.nx - 1);
            ha = off[row + x0];
            hb = off[row + x1 + 1];
        }
    }
    // the candidates of a row, by the whole wavefront: a range's start is uniform, so
    // that a test is a load, a distance and a bit of a ballot
    int n0 = 0, n1 = 0;
    const auto within = [&](int qa, int qb, double lim) {
        int cnt = 0;
        for (int q = qa; q < qb; q += kFeatTests * HK_WAVE) {
            const double2 *__restrict__ p0 = cxy + q;
            double2 p[kFeatTests];
#pragma unroll
            for (int u = 0; u < kFeatTests; ++u)
                if (u == 0 || q + u * HK_WAVE < qb) p[u] = p0[min(u * HK_WAVE + lane, qb - q - 1)];
#pragma unroll
            for (int u = 0; u < kFeatTests; ++u) {
                if (u != 0 && q + u * HK_WAVE >= qb) break;
                const double dx = p[u].x - xm, dy = p[u].y - ym;
                cnt += (int)__popcll(__ballot(dx * dx + dy * dy < lim && u * HK_WAVE + lane < qb - q));
            }
        }
        return cnt;
    };
    for (int y = 0; y <= y_hi - y_lo; ++y) {
        const int l = y * lpr;
        n1 += within(__builtin_amdgcn_readlane(la, l), __builtin_amdgcn_readlane(lb, l), r1);
        n1 += within(__builtin_amdgcn_readlane(ra, l), __builtin_amdgcn_readlane(rb, l), r1);
        n0 += within(__builtin_amdgcn_readlane(ha, l), __builtin_amdgcn_readlane(hb, l), r0);
    }
    // the time windows: one candidate, and its exponent in feature 8 (-inf: no term)
    const auto window_at = [&](const double2 p, double tq) {
        const double dx = p.x - xm, dy = p.y - ym;
        const double d2 = dx * dx + dy * dy;
        const double dt = tq - tm;
        const bool prev = dt >= -w1 && dt < 0.0, next = dt > 0.0 && dt <= w1, next3 = dt > 0.0 && dt <= w3;
        if (!(d2 < r1)) return -(double)INFINITY;
        c[6] += prev;
        c[7] += next;
        if (d2 < r0) {
            c[3] += prev;
            c[4] += next;
            c[5] += next3;
        }
        if (!(dt > 0.0 && dt <= w6)) return -(double)INFINITY;
        c[2] += 1;
        return -2.0 * F.omega * dt - d2 * F.inv_h2;
    };
    const auto window = [&](int q) { return window_at(cxy[q], ct[q]); };
    // each column's first lpr candidates are loaded together, one per lane (nearly
    // always all of them); their exponents are kept
    double ae[8], amax = -INFINITY;  // largest exponent of feature 8's terms
    int cq[8], cn[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        cq[i] = __shfl(wq, lane - lr + i);
        cn[i] = __shfl(wn, lane - lr + i);
    }
#pragma unroll
    for (int i = 0; i < 8; i += kFeatWindows) {
        double2 p[kFeatWindows];
        double tq[kFeatWindows];
#pragma unroll
        for (int u = 0; u < kFeatWindows; ++u) {
            const int q = lr < cn[i + u] ? cq[i + u] + lr : 0;
            p[u] = cxy[q];
            tq[u] = ct[q];
        }
#pragma unroll
        for (int u = 0; u < kFeatWindows; ++u) {
            ae[i + u] = lr < cn[i + u] ? window_at(p[u], tq[u]) : -INFINITY;
            amax = fmax(amax, ae[i + u]);
        }
    }
    // the others: a short list by the lane group, a long one (windows of many runs over
    // a crowded cell) by the whole wavefront
    const uint64_t longs = __ballot(wn > kFeatLong);
    const auto others = [&](const auto &take) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (cn[i] <= kFeatLong)
                for (int s = lr + lpr; s < cn[i]; s += lpr) take(cq[i] + s);
        for (uint64_t mk = longs; mk != 0; mk &= mk - 1) {
            const int l = __ffsll((unsigned long long)mk) - 1;
            const int q0 = __builtin_amdgcn_readlane(wq, l), n = __builtin_amdgcn_readlane(wn, l);
#pragma unroll 4
            for (int s = lpr + lane; s < n; s += HK_WAVE) take(q0 + s);
        }
    };
    others([&](int q) { amax = fmax(amax, window(q)); });
#pragma unroll
    for (int a = 1; a < 8; ++a) {
#pragma unroll
        for (int o = 1; o < HK_WAVE; o <<= 1) c[a] += __shfl_xor(c[a], o);
    }
#pragma unroll
    for (int o = 1; o < HK_WAVE; o <<= 1) amax = fmax(amax, __shfl_xor(amax, o));
    // feature 8's terms relative to the largest, in fixed point (2^36 units)
    long long ksum = 0;
    if (amax > -INFINITY) {
        const auto term = [&](double a) {  // a <= amax
            return llrint((double)exp2f((float)((a - amax) * 1.4426950408889634)) * 68719476736.0);
        };
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (ae[i] > -INFINITY) ksum += term(ae[i]);
        others([&](int q) {
            const double2 p = cxy[q];
            const double dx = p.x - xm, dy = p.y - ym;
            const double d2 = dx * dx + dy * dy;
            const double dt = ct[q] - tm;
            if (d2 < r1 && dt > 0.0 && dt <= w6) ksum += term(-2.0 * F.omega * dt - d2 * F.inv_h2);
        });
#pragma unroll
        for (int o = 1; o < HK_WAVE; o <<= 1) ksum += __shfl_xor(ksum, o);
    }
    // lane a forms feature a (the event itself is inside every disc)
    if (lane >= MLP_IN) return;
    int cnt = lane < 2 ? n0 - 1 : c[2];
    if (lane == 1) cnt = c[1] + n1 - 1;
#pragma unroll
    for (int a = 3; a < 8; ++a)
        if (lane == a) cnt = c[a];
    float f = (float)log1p((double)cnt);
    if (lane == 8) {
        // log2 S_m = log2(ksum) - 36 + a_max / ln 2 (S_m = 0: the floor)
        const double l2s = ksum > 0 ? log2((double)ksum) - 36.0 + amax * 1.4426950408889634 : -INFINITY;
        f = (float)(fmax(l2s, HK_KSUM_LOG2_FLOOR) * 0.125);
    }
    if (lane == 9) f = (float)z[k];
    if (lane == 10) f = (float)((double)g[pos[r]] / (double)n);
    if (lane == 11) {
        const double span = t1 - t0;
        f = (float)(span > 0.0 ? (t1 - tm) / span : 0.0);
    }
    feat[(int64_t)k * MLP_IN + lane] = f;
}

// ---- mass update ------------------------------------------------------------------------
// mass <- (count mass + e_k) / (count + 1) with the learned estimate
// e_k = theta^2 exp(pred_k) + P_kk (pred: the network's log H_k; the exact one is
// formed by the column finalisation).
__global__ void k_mass_update(int64_t m, const float *__restrict__ pred, const double *__restrict__ theta,
                              const int64_t *__restrict__ cidx, const double *__restrict__ pdiag, double inv_s2,
                              double count, double *__restrict__ mass) {
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= m) return;
    const double th = theta[cidx[k]];
    const double est = th * th * exp((double)pred[k]) + hk_prior_prec(pdiag, (int)k, inv_s2);
    mass[k] = (count * mass[k] + est) / (count + 1.0);
}

}  // namespace

extern "C" int64_t hawkes_mlp_num_params(void) { return MLP_NP; }

extern "C" int64_t hawkes_mlp_workspace_floats(int64_t B) {
    // one slice of FP64 gradient sums and one loss sum per block, 8-byte aligned
    return 2 * ((int64_t)MLP_NP + 1) * mlp_blocks(B) + 64;
}

extern "C" hawkes_status hawkes_mlp_forward(const float *d_params, const float *d_x, int64_t B, float *d_y,
                                            hipStream_t stream) {
    if (!d_params || !d_x || !d_y || B < 1) return HAWKES_E_INVALID;
    // a block's weights stay in registers over its groups: at most eight blocks per CU
    const unsigned nb = (unsigned)std::min<int64_t>(2048, (B + MLP_BS - 1) / MLP_BS);
    hipLaunchKernelGGL(k_mlp_batch<false>, dim3(nb), dim3(MLP_THREADS), 0, stream, d_params, d_x, B,
                       (const int *)nullptr, (const float *)nullptr, B, d_y, (double *)nullptr, (double *)nullptr,
                       (int *)nullptr);
    HK_CHECK(hipGetLastError());
    return HAWKES_OK;
}

// Gradient and loss, and with `adam` the update of the parameters.
static void mlp_grad_launch(const float *d_params, const float *d_x, int64_t n_rows, const int *d_rows,
                            const float *d_target, int64_t B, float *d_work, double *d_grad, double *d_loss,
                            int *d_err, const AdamArgs *adam, hipStream_t stream) {
    double *part = (double *)(((uintptr_t)d_work + 7) & ~(uintptr_t)7);
    const int nb = mlp_blocks(B);
    double *lpart = part + (int64_t)nb * MLP_NP;
    hipLaunchKernelGGL(k_mlp_batch<true>, dim3(nb), dim3(MLP_THREADS), 0, stream, d_params, d_x, n_rows, d_rows,
                       d_target, B, (float *)nullptr, part, lpart, d_err);
    const dim3 grid((MLP_NP + HK_WAVE - 1) / HK_WAVE + (d_loss ? 1 : 0)), block(MLP_APPLY_WAVES * HK_WAVE);
    if (adam)
        hipLaunchKernelGGL(k_mlp_apply<true>, grid, block, 0, stream, part, lpart, nb, B, d_grad, d_loss, *adam);
    else
        hipLaunchKernelGGL(k_mlp_apply<false>, grid, block, 0, stream, part, lpart, nb, B, d_grad, d_loss, AdamArgs{});
}

extern "C" hawkes_status hawkes_mlp_grad(const float *d_params, const float *d_x, int64_t n_rows,
                                         const int *d_rows, const float *d_target, int64_t B, float *d_work,
                                         double *d_grad, double *d_loss, int *d_err, hipStream_t stream) {
    if (!d_params || !d_x || !d_target || !d_work || !d_grad || B < 1 || n_rows < 1) return HAWKES_E_INVALID;
    if (!d_rows && B > n_rows) return HAWKES_E_INVALID;
    mlp_grad_launch(d_params, d_x, n_rows, d_rows, d_target, B, d_work, d_grad, d_loss, d_err, nullptr, stream);
    HK_CHECK(hipGetLastError());
    return HAWKES_OK;
}

// ---- allocation-free training step ---------------------------------------------------------
// The workspace of mlp_grad_launch for a batch of at most HK_NOALLOC_MLP_MAX_B
// samples (the blocks' slices of FP64 sums), then, 256-byte aligned, the FP64
// gradient.  Every kernel of the step writes the parts it reads before reading
// them, so nothing needs clearing between calls.
constexpr int64_t kNoallocBlocks = HK_NOALLOC_MLP_MAX_B / MLP_BS;
static_assert(HK_NOALLOC_MLP_MAX_B % MLP_BS == 0 && kNoallocBlocks <= MLP_MAX_BLOCKS, "slices of the largest batch");
constexpr int64_t kNoallocWorkFloats = (2 * ((int64_t)MLP_NP + 1) * kNoallocBlocks + 63) / 64 * 64;
constexpr int64_t kNoallocFloats = kNoallocWorkFloats + 2 * (int64_t)MLP_NP;
static __device__ __align__(256) float scratch[kNoallocFloats];

// Device address of `scratch` on the current device, looked up once per device
// (each GPU holds its own copy of the array at its own address).  In host code
// the array's name is only a host-side stand-in, never a device address.
static constexpr int kNoallocMaxDevices = 64;

static hawkes_status noalloc_scratch(float **out) {
    static std::mutex mu;
    static float *ptr[kNoallocMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kNoallocMaxDevices) return HAWKES_E_DEVICE;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return HAWKES_E_DEVICE;
        ptr[dev] = (float *)p;
    }
    *out = ptr[dev];
    return HAWKES_OK;
}

extern "C" int64_t hawkes_mlp_noalloc_max_batch(void) { return HK_NOALLOC_MLP_MAX_B; }

extern "C" hawkes_status hawkes_mlp_train_step_noalloc(float *d_params, float *d_adam_m, float *d_adam_v, int step,
                                                       float lr, const float *d_x, int64_t n_rows,
                                                       const int *d_rows, const float *d_target, int64_t B,
                                                       double *d_loss, int *d_err, hipStream_t stream) {
    if (!d_params || !d_adam_m || !d_adam_v || step < 1 || !d_x || !d_target || B < 1 || n_rows < 1)
        return HAWKES_E_INVALID;
    if (!d_rows && B > n_rows) return HAWKES_E_INVALID;
    if (B > HK_NOALLOC_MLP_MAX_B) return HAWKES_E_CAPACITY;
    float *work = nullptr;
    const hawkes_status st = noalloc_scratch(&work);
    if (st != HAWKES_OK) return st;
    double *grad = (double *)(work + kNoallocWorkFloats);
    const AdamArgs ad{d_params, d_adam_m, d_adam_v, step, lr, 0.9f, 0.999f, 1e-8f};
    mlp_grad_launch(d_params, d_x, n_rows, d_rows, d_target, B, work, grad, d_loss, d_err, &ad, stream);
    HK_CHECK(hipGetLastError());
    return HAWKES_OK;
}

extern "C" hawkes_status hawkes_mlp_train_step(float *d_params, float *d_adam_m, float *d_adam_v, int step,
                                               float lr, const float *d_x, int64_t n_rows, const int *d_rows,
                                               const float *d_target, int64_t B, float *d_work, double *d_grad,
                                               double *d_loss, int *d_err, hipStream_t stream) {
    if (!d_params || !d_adam_m || !d_adam_v || step < 1 || !d_x || !d_target || !d_work || !d_grad || B < 1 ||
        n_rows < 1)
        return HAWKES_E_INVALID;
    if (!d_rows && B > n_rows) return HAWKES_E_INVALID;
    const AdamArgs ad{d_params, d_adam_m, d_adam_v, step, lr, 0.9f, 0.999f, 1e-8f};
    mlp_grad_launch(d_params, d_x, n_rows, d_rows, d_target, B, d_work, d_grad, d_loss, d_err, &ad, stream);
    HK_CHECK(hipGetLastError());
    return HAWKES_OK;
}

extern "C" hawkes_status hawkes_features(hawkes_plan p, const hawkes_hyper *hy, const double *d_t,
                                         const double *d_xy, const double *d_z, double gx0, double gy0,
                                         float *d_feat, hipStream_t stream) {
    if (!p || !hk_hyper_ok(hy) || !d_t || !d_xy || !d_z || !d_feat) return HAWKES_E_INVALID;
    if (!p->sub) return HAWKES_E_UNSUPPORTED;
    if (!(gx0 <= p->xmin) || !(gy0 <= p->ymin)) return HAWKES_E_INVALID;
    FeatGrid G;
    G.gx0 = gx0;
    G.gy0 = gy0;
    const auto fits = [&](double size, double most) {
        G.s = size;
        const double nx = floor((p->xmax - gx0) / G.s) + 1.0, ny = floor((p->ymax - gy0) / G.s) + 1.0;
        if (!(nx * ny <= most)) return false;
        G.nx = (int)nx;
        G.ny = (int)ny;
        return true;
    };
    if (!fits(3.0 * hy->h, (double)((1 << 26) - 1))) return HAWKES_E_UNSUPPORTED;
    const bool lds = fits(hy->h, kFeatCells) || fits(2.0 * hy->h, kFeatCells) || fits(3.0 * hy->h, kFeatCells);
    const int64_t n = p->n, cells = (int64_t)G.nx * G.ny;
    // runs of at least 256 events
    const int64_t runs = std::min<int64_t>(kFeatRuns, (n + 255) / 256);
    G.nb = lds ? (int)runs : 1;
    G.per = (int)((n + G.nb - 1) / G.nb);
    // int workspace: offsets [nb][cells + 1], then the runs' group sums, or one
    // run's counts and fill marks; then (16-byte aligned) the events' coordinates
    // and times in cell order [3 n]
    const int64_t offs = G.nb * (cells + 1);
    const int64_t ints = (offs + (lds ? (int64_t)G.nb * (kFeatCells / kFeatGroup) : 2 * cells) + 3) / 4 * 4;
    // the number of cells jumps where the cell width goes from one multiple of h to
    // another, so there is always room for the LDS sort's largest grid: the workspace
    // then grows only as h falls (a larger one may follow under capture)
    const int64_t room = (runs * (kFeatCells + 1 + kFeatCells / kFeatGroup) + 3) / 4 * 4;
    hawkes_status st = hk_subset_grid(p, std::max(ints, room) + 6 * n, stream);
    if (st != HAWKES_OK) return st;
    int *off = hk_subset_grid_ptr(p), *rest = off + offs;
    double2 *cxy = (double2 *)(off + ints);
    double *ct = (double *)(cxy + n);
    if (lds) {
        hipLaunchKernelGGL(k_cell_hist, dim3(G.nb), dim3(kFeatThreads), 0, stream, d_xy, p->perm, n, G, off, rest);
        hipLaunchKernelGGL(k_cell_off, dim3(nblk(cells, kFeatGroup)), dim3(kFeatOffWaves * HK_WAVE), 0, stream, rest, n, G, off);
        hipLaunchKernelGGL(k_cell_place, dim3(G.nb), dim3(kFeatThreads), 0, stream, d_t, d_xy, p->perm, n, G, off, ct,
                           cxy);
    } else {
        int *cnt = rest, *fill = rest + cells;
        hipLaunchKernelGGL(k_fill_zero, dim3(std::min<int64_t>(nblk(cells, 256), 4096)), dim3(256), 0, stream, cnt,
                           cells);
        hipLaunchKernelGGL(k_cell_count, dim3(nblk(n, 256)), dim3(256), 0, stream, d_xy, n, G, cnt);
        hipLaunchKernelGGL(k_cell_scan, dim3(1), dim3(kScanThreads), 0, stream, cnt, cells, off, fill);
        hipLaunchKernelGGL(k_cell_scatter, dim3(nblk(n, 256)), dim3(256), 0, stream, d_t, d_xy, n, G, off, fill, ct,
                           cxy);
    }
    int64_t m;
    const int64_t *cidx;
    const int *pos, *slot;
    hk_subset_view(p, &m, &cidx, &pos, &slot);
    const double h3 = 3.0 * hy->h, inv_s = 1.0 / G.s;
    const FeatConst F{hy->h * hy->h,  h3 * h3, 1.0 / hy->omega, 3.0 / hy->omega, 6.0 / hy->omega, 1.0 / (hy->h * hy->h),
                      inv_s, hy->h * inv_s, h3 * inv_s, hy->omega};
    hipLaunchKernelGGL(k_features, dim3((unsigned)m), dim3(HK_WAVE), 0, stream, d_t, d_xy, cidx, pos, slot,
                       p->g, p->ts, d_z, m, n, p->t0, p->t1, F, G, off, ct, cxy, d_feat);
    HK_CHECK(hipGetLastError());
    return HAWKES_OK;
}

// The prior's precision diagonal for prior = 0 (iid: NULL, 1/sigma^2) or 1 (the
// plan's tree); false when the prior is unknown or its tree is not set.
static bool prior_diag(hawkes_plan p, int prior, int64_t m, const double **pdiag) {
    *pdiag = nullptr;
    if (prior == 0) return true;
    if (prior != 1 || hk_tree_tips(p) != m) return false;
    *pdiag = hk_tree_precision_diag(p);
    return *pdiag != nullptr;
}

extern "C" hawkes_status hawkes_mass_update(hawkes_plan p, const hawkes_hyper *hy, const double *d_theta,
                                            const float *d_pred, double sigma_z, int prior, int64_t count,
                                            double *d_mass, hipStream_t stream) {
    if (!p || !hk_hyper_ok(hy) || !d_theta || !d_mass || !(sigma_z > 0.0) || count < 0) return HAWKES_E_INVALID;
    if (!p->sub) return HAWKES_E_UNSUPPORTED;
    int64_t m;
    const int64_t *cidx;
    const int *pos, *slot;
    hk_subset_view(p, &m, &cidx, &pos, &slot);
    const double *pdiag;
    if (!prior_diag(p, prior, m, &pdiag)) return prior == 1 ? HAWKES_E_UNSUPPORTED : HAWKES_E_INVALID;
    const double inv_s2 = 1.0 / (sigma_z * sigma_z);
    if (!d_pred) {
        SubOut out{};
        out.theta = d_theta;
        out.pdiag = pdiag;
        out.inv_s2 = inv_s2;
        out.mass = d_mass;
        out.count = (double)count;
        return hk_subset_exact(p, hy, d_theta, stream, out);
    }
    hipLaunchKernelGGL(k_mass_update, dim3(nblk(m, 256)), dim3(256), 0, stream, m, d_pred, d_theta, cidx, pdiag, inv_s2,
                       (double)count, d_mass);
    HK_CHECK(hipGetLastError());
    return HAWKES_OK;
}

extern "C" hawkes_status hawkes_subset_curvature(hawkes_plan p, const hawkes_hyper *hy, const double *d_theta,
                                                 double sigma_z, int prior, double *d_curv, float *d_log_h,
                                                 hipStream_t stream) {
    if (!p || !hk_hyper_ok(hy) || !d_theta || !(sigma_z > 0.0) || (!d_curv && !d_log_h)) return HAWKES_E_INVALID;
    if (!p->sub) return HAWKES_E_UNSUPPORTED;
    int64_t m;
    const int64_t *cidx;
    const int *pos, *slot;
    hk_subset_view(p, &m, &cidx, &pos, &slot);
    const double *pdiag;
    if (!prior_diag(p, prior, m, &pdiag)) return prior == 1 ? HAWKES_E_UNSUPPORTED : HAWKES_E_INVALID;
    SubOut out{};
    out.theta = d_theta;
    out.pdiag = pdiag;
    out.inv_s2 = 1.0 / (sigma_z * sigma_z);
    out.curv = d_curv;
    out.log_h = d_log_h;
    return hk_subset_exact(p, hy, d_theta, stream, out);
}
