// The phylogenetic prior in two short phases, shared by its own launches and by
// the subset passes, which give each phase some extra blocks (not installed).
#pragma once
#include "hawkes_internal.h"

// V^{-1} z and z^T V^{-1} z (hawkes_tree.hip states the recursions).  Walking the
// tree level by level is a chain of some 30 dependent levels up and down (25 us
// for 1,610 tips in one block, the prior's whole cost).  Instead the tree is cut
// into its R maximal subtrees of at most HK_TREE_SUB tips, and the recursions are
// carried out once, in closed form, on unit vectors, which leaves two dense and
// parallel steps per evaluation:
//
//   low   per subtree s (one wavefront): y = M_s z_s, the subtree's part of
//         V^{-1} z, its root's mean m_s = w_s . z_s and its part of the quadratic
//         form;
//   top   adj = Q m with Q the inverse covariance of the subtree roots' means,
//         then V^{-1} z = y + w adj(subtree).
//
// M_s and Q come from the recursions, so their entries carry no cancellation;
// M_s has zero row sums and Q row sums e_r, so both products are taken over
// differences, and the quadratic form over their squares (off-diagonals are <= 0:
// every term is >= 0).  Needing z alone, the two steps ride as extra blocks on
// the row pass and on the column pass: N = 23,422, 1,610 tips, HMC iteration
// under this prior 1,117 us with the level walk, 638 us with these (619 us under
// the independent prior).
#define HK_TREE_SUB 64           // tips per subtree: one wavefront
#define HK_TREE_MAX_ROOTS 1024   // more subtrees (a random tree of over some 33,000 tips) take the level walk

struct TreeDense {
    int R;                // subtrees (0: none)
    const int *tip0;      // [R + 1] first tip of each subtree, in subtree order
    const int *tip;       // [m] subset slot of each tip
    const int *sub;       // [m] its subtree
    const int64_t *mat0;  // [R] first entry of each M_s
    const double *mat;    // M_s [n][n] one after the other (symmetric)
    const double *w;      // [m] weight of the tip in its root's mean
    const double *Q;      // [R][R] (symmetric)
    const double *qrow;   // [R] row sums of Q
    double *y;            // [m] low step's part of V^{-1} z
    double *mean;         // [R] root means
    double *qlow;         // [R] quadratic form below each root
    double *quad;         // [R] parts of z^T V^{-1} z (their sum is the form)
};

constexpr int HK_TREE_TOP_THREADS = 64, HK_TREE_TOP_ROOTS = 4;  // per block of the top step
constexpr int hk_tree_top_blocks(int R) { return (R + HK_TREE_TOP_ROOTS - 1) / HK_TREE_TOP_ROOTS; }

// Low step of subtree r, by one wavefront.
__device__ __forceinline__ void hk_tree_low(const TreeDense &t, const double *__restrict__ z, int r) {
    const int lane = threadIdx.x & (HK_WAVE - 1);
    const int k0 = t.tip0[r], n = t.tip0[r + 1] - k0;
    const bool in = lane < n;
    const double zi = in ? z[t.tip[k0 + lane]] : 0.0, wi = in ? t.w[k0 + lane] : 0.0;
    const double *__restrict__ M = t.mat + t.mat0[r] + (in ? lane : 0);
    double y = 0.0, q = 0.0, mean = wi * zi;
#pragma unroll 8
    for (int j = 0; j < n; ++j) {
        const double mj = M[(int64_t)j * n];
        const double zj = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(zi), j),
                                           __builtin_amdgcn_readlane(__double2loint(zi), j));
        const double d = zj - zi, md = mj * d;
        y += md;
        q = fma(-0.5 * md, d, q);
    }
    if (!in) q = 0.0;
    for (int o = 32; o > 0; o >>= 1) {
        mean += __shfl_xor(mean, o);
        q += __shfl_xor(q, o);
    }
    if (in) t.y[k0 + lane] = y;
    if (lane == 0) {
        t.mean[r] = mean;
        t.qlow[r] = q;
    }
}

// Top step of HK_TREE_TOP_ROOTS subtrees, by a block of HK_TREE_TOP_THREADS.
__device__ __forceinline__ void hk_tree_top(const TreeDense &t, int block, double *__restrict__ vz) {
    __shared__ double adj[HK_TREE_TOP_ROOTS];
    const int l = threadIdx.x / 16, c = threadIdx.x % 16, r0 = block * HK_TREE_TOP_ROOTS, r = min(r0 + l, t.R - 1);
    const double mr = t.mean[r], qr = t.qrow[r];
    const double *__restrict__ Qr = t.Q + (int64_t)r * t.R;
    double s = 0.0, q = 0.0;
#pragma unroll 8
    for (int k = c; k < t.R; k += 16) {
        const double d = t.mean[k] - mr, qd = Qr[k] * d;
        s += qd;
        q = fma(-0.5 * qd, d, q);
    }
    for (int o = 1; o < 16; o <<= 1) {
        s += __shfl_xor(s, o);
        q += __shfl_xor(q, o);
    }
    if (c == 0) adj[l] = fma(qr, mr, s);
    if (c == 0 && r0 + l < t.R) t.quad[r] = fma(qr * mr, mr, q) + t.qlow[r];
    __syncthreads();
    const int k1 = t.tip0[min(t.R, r0 + HK_TREE_TOP_ROOTS)];
    for (int k = t.tip0[r0] + threadIdx.x; k < k1; k += HK_TREE_TOP_THREADS)
        vz[t.tip[k]] = fma(t.w[k], adj[t.sub[k] - r0], t.y[k]);
}

// The plan's cut tree, NULL where it has none or takes the level walk.
const TreeDense *hk_tree_dense(hawkes_plan p);
