// Phylogenetic Brownian prior on the free log-rates (Sec. 2.2, Eq. 2).
//
// The log-rates z of the M tips of a bifurcating tree follow a Brownian
// diffusion: the root value is N(0, tau0 sigma^2), each child is its parent
// plus N(0, w sigma^2) for its branch length w, so z ~ N(0, sigma^2 V) with
// V_nm = tau0 + (length of the path from the root to the common ancestor of
// tips n and m).  Eq. 2 needs V^{-1}, O(M^3) dense; the tree structure gives
// log p(z) and its gradient in O(M) by message passing (the paper uses the
// dynamic programming of Pybus et al. 2012):
//
//  * post-order: a tip carries (m, v) = (z_k, 0).  An internal node a with
//    children b, c carries v_a = 1 / (1/(v_b + w_b) + 1/(v_c + w_c)) and
//    m_a = alpha_b m_b + alpha_c m_c, alpha_x = v_a / (v_x + w_x); the pair
//    contributes (m_b - m_c)^2 / s_a, s_a = v_b + w_b + v_c + w_c, to the
//    quadratic form, the root m_root^2 / (v_root + tau0);
//  * z^T V^{-1} z is the sum of those contributions and
//    log |V| = sum_a log s_a + log(v_root + tau0);
//  * V^{-1} z is the gradient of half the quadratic form: a pre-order pass
//    pushes the adjoint of each node to its children,
//    mbar_b = alpha_b mbar_a + d_a, mbar_c = alpha_c mbar_a - d_a,
//    d_a = (m_b - m_c) / s_a, starting from mbar_root = m_root / (v_root + tau0);
//  * the diagonal of V^{-1} (the prior's precision, used by the diagonal mass
//    matrix) is 1 / Var(z_k | every other tip): a pre-order pass carries the
//    variance u_a of what the rest of the tree says about node a, u_root =
//    tau0, u_b = (u_a (v_c + w_c)) / (u_a + v_c + w_c) + w_b for child b with
//    sibling c, and (V^{-1})_kk = 1 / u_k at tip k.
//
// The v, alpha, s depend on the tree only and are formed once on the host in
// FP64.  On the device the prior is two dense steps over the tree cut into
// subtrees (hawkes_tree.h); for a tree that needs too many of them, and alone for a
// shallow one, one block walks the levels of the tree (nodes grouped by height, so
// that all children of a level are done before it), one thread per node of a level,
// with a barrier between levels.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <utility>
#include <vector>

#include "hawkes_internal.h"
#include "hawkes_tree.h"

struct hk_tree {
    int64_t m;           // tips (= subset size)
    int levels;          // height levels of internal nodes
    double logdet;       // log |V|
    // device arrays, all in `store`
    int *order;          // [n_int] internal nodes, grouped by level (increasing height)
    int *level0;         // [levels + 1] first entry of each level in order[]
    int *child;          // [2 (2m - 1)] children of each node (internal only)
    double *coef;        // [3 (2m - 1)] alpha_b, alpha_c, 1 / s_a per internal node
    double *mv;          // [2m - 1] node means (post-order), then adjoints
    double *dd;          // [2m - 1] d_a per internal node
    int root;
    double root_inv;     // 1 / (v_root + tau0)
    double *pdiag;       // [m] diagonal of V^{-1}, tip (slot) order (device)
    TreeDense dense;     // the cut tree (R = 0: none)
    void *store;
};

namespace {

constexpr int TREE_THREADS = 1024;
// hawkes_tree_prior alone takes the level walk for a tree of at most this many levels
// (two more where a level is one node per thread): one launch of some 10 dependent
// levels against the dense steps' two (a balanced tree of 400 / 1,600 / 3,000 / 6,000
// tips, 9 / 11 / 12 / 13 levels, walk 12.1 / 14.9 / 17.4 / 23.2 us, dense 15.6 / 16.2 /
// 16.4 / 17.6; a random one of 64 / 128 / 800, 13 / 15 / 23 levels, walk 12.4 / 14.8 /
// 21.3, dense 13.4 / 14.0 / 15.4).  In hmc_step the dense steps cost no launch.
constexpr int TREE_WALK_LEVELS = 11;

__global__ __launch_bounds__(TREE_THREADS) void k_tree_prior(const double *__restrict__ z, int64_t m,
                                                             const int *__restrict__ order,
                                                             const int *__restrict__ level0, int levels,
                                                             const int *__restrict__ child,
                                                             const double *__restrict__ coef, int root,
                                                             double root_inv, double *__restrict__ mv,
                                                             double *__restrict__ dd, double *__restrict__ vz,
                                                             double *__restrict__ quad) {
    __shared__ double red[TREE_THREADS];
    const int tid = threadIdx.x;
    double q = 0.0;
    for (int64_t k = tid; k < m; k += TREE_THREADS) mv[k] = z[k];
    __syncthreads();
    // post-order: level by level of increasing height
    for (int l = 0; l < levels; ++l) {
        for (int e = level0[l] + tid; e < level0[l + 1]; e += TREE_THREADS) {
            const int a = order[e];
            const int b = child[2 * a], c = child[2 * a + 1];
            const double mb = mv[b], mc = mv[c];
            const double ab = coef[3 * a], ac = coef[3 * a + 1], is = coef[3 * a + 2];
            mv[a] = ab * mb + ac * mc;
            const double d = mb - mc;
            q += d * d * is;
            dd[a] = d * is;
        }
        __syncthreads();
    }
    const double mroot = mv[root];
    if (tid == 0) q += mroot * mroot * root_inv;
    __syncthreads();
    // pre-order: adjoints of half the quadratic form, root level first (the
    // node means are no longer needed, so mv now holds adjoints)
    if (tid == 0) mv[root] = mroot * root_inv;
    __syncthreads();
    for (int l = levels - 1; l >= 0; --l) {
        for (int e = level0[l] + tid; e < level0[l + 1]; e += TREE_THREADS) {
            const int a = order[e];
            const int b = child[2 * a], c = child[2 * a + 1];
            const double ma = mv[a], d = dd[a];
            mv[b] = coef[3 * a] * ma + d;
            mv[c] = coef[3 * a + 1] * ma - d;
        }
        __syncthreads();
    }
    if (vz)
        for (int64_t k = tid; k < m; k += TREE_THREADS) vz[k] = mv[k];
    // fixed-order reduction of the quadratic form
    red[tid] = q;
    __syncthreads();
    for (int h = TREE_THREADS / 2; h > 0; h >>= 1) {
        if (tid < h) red[tid] += red[tid + h];
        __syncthreads();
    }
    if (tid == 0 && quad) quad[0] = red[0];
}

__global__ __launch_bounds__(HK_WAVE) void k_tree_low(const TreeDense t, const double *__restrict__ z) {
    hk_tree_low(t, z, blockIdx.x);
}

__global__ __launch_bounds__(HK_TREE_TOP_THREADS) void k_tree_top(const TreeDense t, double *__restrict__ vz) {
    hk_tree_top(t, blockIdx.x, vz);
}

// One inner node of a piece of the cut (a subtree, or the top with the subtrees'
// roots for leaves): what the entries of the leaves that meet in it need.
struct TreeStep {
    double x, alpha_b, alpha_c;
    int b0, b1, c0, c1;  // the leaves below its children b and c, within the piece
};

// M_s of each subtree and Q (the last block), the recursions on unit vectors in
// closed form.  Let a node a have children b and c, and kappa_a be the adjoint of a for
// a unit mean of a and zero ones beside it: 0 at a subtree's root, 1 / (v_root + tau0)
// at the tree's.  Then kappa_b = alpha_b^2 kappa_a + 1/s_a, and the adjoint of b for a
// unit mean of c is x_a = alpha_b alpha_c kappa_a - 1/s_a, so that the entry of two leaves
// that meet in a is w x_a w', with w a leaf's weight in the mean of its child of a: the
// product of the alphas between.  (The steps read differences: the diagonals are left
// 0.)  A block takes its piece node by node, children first.
//
// Once per tree.  Formed on the host, column by column of the recursions, this was
// most of hawkes_plan_set_tree: a balanced tree of 20,000 tips 5.2 ms, a single lineage
// of 1,087 tips (1,023 steps at the top) 12.6 ms; now 1.1 and 0.96.
constexpr int TREE_CUT_THREADS = 256;
__global__ __launch_bounds__(TREE_CUT_THREADS) void k_tree_cut(const TreeStep *__restrict__ steps,
                                                               const int *__restrict__ step0, int R,
                                                               const int *__restrict__ tip0,
                                                               const int64_t *__restrict__ mat0, double root_inv,
                                                               double *__restrict__ mat, double *__restrict__ wgt,
                                                               double *__restrict__ Q, double *__restrict__ qrow) {
    __shared__ double w[HK_TREE_MAX_ROOTS];  // (more than HK_TREE_SUB)
    const int s = blockIdx.x, tid = threadIdx.x;
    const bool top = s == R;
    const int n = top ? R : tip0[s + 1] - tip0[s];
    double *__restrict__ out = top ? Q : mat + mat0[s];
    for (int k = tid; k < n; k += TREE_CUT_THREADS) {
        w[k] = 1.0;
        out[(int64_t)k * n + k] = 0.0;
    }
    __syncthreads();
    for (int e = step0[s]; e < step0[s + 1]; ++e) {
        const TreeStep a = steps[e];
        const int nb = a.b1 - a.b0, nc = a.c1 - a.c0;
        for (int k = tid; k < nb * nc; k += TREE_CUT_THREADS) {
            const int i = a.b0 + k / nc, j = a.c0 + k % nc;
            out[(int64_t)i * n + j] = out[(int64_t)j * n + i] = w[i] * a.x * w[j];
        }
        __syncthreads();
        for (int k = tid; k < nb; k += TREE_CUT_THREADS) w[a.b0 + k] *= a.alpha_b;
        for (int k = tid; k < nc; k += TREE_CUT_THREADS) w[a.c0 + k] *= a.alpha_c;
        __syncthreads();
    }
    for (int k = tid; k < n; k += TREE_CUT_THREADS) {
        if (top) qrow[k] = w[k] * root_inv;
        else wgt[tip0[s] + k] = w[k];
    }
}

// z^T V^{-1} z from the subtrees' parts (by one wavefront in a fixed order; without
// parts it is in `quad`), log p(z) = -(m log(2 pi sigma^2) + log|V| + z^T V^{-1} z /
// sigma^2) / 2 and its gradient -V^{-1} z / sigma^2
__global__ void k_tree_logp(const double *__restrict__ parts, int np, double *__restrict__ quad,
                            const double *__restrict__ vz, int64_t m, double sigma2, double logdet,
                            double *__restrict__ logp, double *__restrict__ grad) {
    const int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k < HK_WAVE) {
        double q = 0.0;
        for (int r = (int)k; r < np; r += HK_WAVE) q += parts[r];
        for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o);
        if (k == 0) {
            if (parts) quad[0] = q;
            else q = quad[0];
            if (logp) logp[0] = -0.5 * ((double)m * log(2.0 * 3.141592653589793 * sigma2) + logdet + q / sigma2);
        }
    }
    if (k < m && grad) grad[k] = -vz[k] / sigma2;
}

}  // namespace

void hk_tree_free(hawkes_plan p) {
    hk_tree *t = p->tree;
    if (!t) return;
    if (t->store) (void)hipFree(t->store);
    delete t;
    p->tree = nullptr;
}

int64_t hk_tree_tips(hawkes_plan p) { return p->tree ? p->tree->m : 0; }

const double *hk_tree_precision_diag(hawkes_plan p) { return p->tree ? p->tree->pdiag : nullptr; }

const TreeDense *hk_tree_dense(hawkes_plan p) { return p->tree && p->tree->dense.R > 0 ? &p->tree->dense : nullptr; }

hawkes_status hk_tree_walk(hawkes_plan p, const double *d_z, double *d_vz, double *d_quad, hipStream_t stream) {
    hk_tree *t = p->tree;
    if (!t) return HAWKES_E_UNSUPPORTED;
    hipLaunchKernelGGL(k_tree_prior, dim3(1), dim3(TREE_THREADS), 0, stream, d_z, t->m, t->order, t->level0, t->levels,
                       t->child, t->coef, t->root, t->root_inv, t->mv, t->dd, d_vz, d_quad);
    HK_CHECK(hipGetLastError());
    return HAWKES_OK;
}

static hawkes_status set_tree(hawkes_plan p, int64_t n_nodes, const int64_t *parent, const double *length,
                              double tau0) {
    if (!p || !parent || !length || n_nodes < 1 || n_nodes % 2 == 0 || !(tau0 > 0.0) || !isfinite(tau0))
        return HAWKES_E_INVALID;
    const int64_t m = (n_nodes + 1) / 2;
    if (m > (int64_t)1 << 30) return HAWKES_E_INVALID;
    // structure: nodes 0..m-1 are tips, exactly one root, every internal node
    // has two children, lengths finite and >= 0
    std::vector<int> nchild(n_nodes, 0), child(2 * n_nodes, -1);
    int64_t root = -1;
    for (int64_t v = 0; v < n_nodes; ++v) {
        const int64_t pa = parent[v];
        if (pa < 0) {
            if (root >= 0) return HAWKES_E_INVALID;
            root = v;
            continue;
        }
        if (pa >= n_nodes || pa < m || pa == v) return HAWKES_E_INVALID;
        if (!(length[v] >= 0.0) || !isfinite(length[v])) return HAWKES_E_INVALID;
        if (nchild[pa] >= 2) return HAWKES_E_INVALID;
        child[2 * pa + nchild[pa]++] = (int)v;
    }
    if (root < 0) return HAWKES_E_INVALID;
    if (m == 1 && root != 0) return HAWKES_E_INVALID;
    for (int64_t v = m; v < n_nodes; ++v)
        if (nchild[v] != 2) return HAWKES_E_INVALID;
    // heights by an explicit post-order from the root (also proves the graph is
    // one tree: every node must be reached exactly once)
    std::vector<int> height(n_nodes, -1), stack;
    std::vector<char> seen(n_nodes, 0);
    std::vector<int> post;
    post.reserve(n_nodes);
    stack.push_back((int)root);
    while (!stack.empty()) {
        const int v = stack.back();
        if (!seen[v]) {
            seen[v] = 1;
            if (v >= m) {
                for (int k = 0; k < 2; ++k) {
                    const int c = child[2 * v + k];
                    if (seen[c]) return HAWKES_E_INVALID;
                    stack.push_back(c);
                }
            }
        } else {
            stack.pop_back();
            post.push_back(v);
        }
    }
    if ((int64_t)post.size() != n_nodes) return HAWKES_E_INVALID;
    std::vector<double> var(n_nodes, 0.0), coef(3 * n_nodes, 0.0);
    double logdet = 0.0;
    for (int v : post) {
        if (v < m) {
            height[v] = 0;
            continue;
        }
        const int b = child[2 * v], c = child[2 * v + 1];
        height[v] = 1 + std::max(height[b], height[c]);
        const double vb = var[b] + length[b], vc = var[c] + length[c];
        const double s = vb + vc;
        if (!(s > 0.0)) return HAWKES_E_INVALID;  // two zero-variance children: V is singular
        const double va = vb * vc / s;
        var[v] = va;
        coef[3 * v] = vc / s;      // alpha_b = v_a / vb
        coef[3 * v + 1] = vb / s;  // alpha_c = v_a / vc
        coef[3 * v + 2] = 1.0 / s;
        logdet += log(s);
    }
    const double rv = var[root] + tau0;
    logdet += log(rv);
    // diagonal of V^{-1}: pre-order pass of the outside variances (reverse post-order)
    std::vector<double> outside(n_nodes, 0.0), pdiag(m, 0.0);
    outside[root] = tau0;
    for (auto it = post.rbegin(); it != post.rend(); ++it) {
        const int v = *it;
        if (v < m) {
            if (!(outside[v] > 0.0)) return HAWKES_E_INVALID;  // tip fixed by the others: V is singular
            pdiag[v] = 1.0 / outside[v];
            continue;
        }
        for (int k = 0; k < 2; ++k) {
            const int b = child[2 * v + k], c = child[2 * v + 1 - k];
            const double u = outside[v], vs = var[c] + length[c];
            const double x = u + vs > 0.0 ? u * vs / (u + vs) : 0.0;
            outside[b] = x + length[b];
        }
    }
    const int H = m > 1 ? height[root] : 0;
    const size_t M = (size_t)m;
    std::vector<int> level0(H + 1, 0), order;
    for (int64_t v = m; v < n_nodes; ++v) level0[height[v]]++;  // heights 1..H
    // level l holds height l + 1
    std::vector<int> cnt(H + 1, 0);
    for (int l = 0; l < H; ++l) cnt[l] = level0[l + 1];
    std::vector<int> start(H + 1, 0);
    for (int l = 0; l < H; ++l) start[l + 1] = start[l] + cnt[l];
    order.assign(std::max<int64_t>(n_nodes - m, 1), 0);
    std::vector<int> fill(start.begin(), start.end());
    for (int64_t v = m; v < n_nodes; ++v) order[fill[height[v] - 1]++] = (int)v;

    // the cut: maximal subtrees of at most HK_TREE_SUB tips, in post-order, so that
    // they and the leaves of each node are contiguous in it
    const size_t N = (size_t)n_nodes;
    std::vector<int> tips(N, 0), tip0(1, 0), tipv;
    std::vector<int64_t> mat0;
    std::vector<char> is_sub(N, 0);
    size_t n_mat = 0;
    for (int v : post) {
        tips[v] = v < m ? 1 : tips[child[2 * v]] + tips[child[2 * v + 1]];
        if (v < m) tipv.push_back(v);
    }
    for (int v : post) {
        if (tips[v] > HK_TREE_SUB || (parent[v] >= 0 && tips[parent[v]] <= HK_TREE_SUB)) continue;
        is_sub[v] = 1;
        mat0.push_back((int64_t)n_mat);
        tip0.push_back(tip0.back() + tips[v]);
        n_mat += (size_t)tips[v] * tips[v];
    }
    const int R = mat0.size() <= HK_TREE_MAX_ROOTS ? (int)mat0.size() : 0;
    // its steps for k_tree_cut: the subtrees' inner nodes, then the top's, children first
    std::vector<int> step0(1, 0), sub(m);
    std::vector<TreeStep> steps;
    if (R > 0) {
        std::vector<double> kappa(N, 0.0), x(N, 0.0);
        kappa[root] = 1.0 / rv;
        for (auto it = post.rbegin(); it != post.rend(); ++it) {
            const int v = *it;
            if (is_sub[v]) kappa[v] = 0.0;
            if (v < m) continue;
            const double ab = coef[3 * (size_t)v], ac = coef[3 * (size_t)v + 1], is = coef[3 * (size_t)v + 2];
            x[v] = ab * ac * kappa[v] - is;
            kappa[child[2 * v]] = ab * ab * kappa[v] + is;
            kappa[child[2 * v + 1]] = ac * ac * kappa[v] + is;
        }
        std::vector<int> first(N), last(N);  // leaves of each node within its piece
        steps.reserve(N - M);
        const auto step = [&](int v) {
            const int b = child[2 * v], c = child[2 * v + 1];
            steps.push_back({x[v], coef[3 * (size_t)v], coef[3 * (size_t)v + 1], first[b], last[b], first[c], last[c]});
            first[v] = std::min(first[b], first[c]);
            last[v] = std::max(last[b], last[c]);
        };
        int leaf = 0, r = 0;
        for (int v : post) {
            if (tips[v] > HK_TREE_SUB) continue;
            if (v < m) {
                sub[tip0[r] + leaf] = r;
                first[v] = leaf++;
                last[v] = leaf;
            } else {
                step(v);
            }
            if (is_sub[v]) {
                step0.push_back((int)steps.size());
                first[v] = r++;
                last[v] = r;
                leaf = 0;
            }
        }
        for (int v : post)
            if (tips[v] > HK_TREE_SUB) step(v);
        step0.push_back((int)steps.size());
    } else {
        mat0.clear();
        tip0.clear();
        tipv.clear();
        sub.clear();
        n_mat = 0;
    }

    // one allocation, filled by one copy: 8-byte arrays, then integers; then what the
    // device writes
    std::vector<char> host;
    host.reserve(8 * (4 * N + M + R) + sizeof(TreeStep) * steps.size() + 4 * (6 * N + 2 * M + R) + 256);
    const auto put = [&](const auto &v) {
        const size_t at = (host.size() + 7) / 8 * 8, bytes = sizeof(v[0]) * v.size();
        host.resize(at + bytes);
        if (bytes) memcpy(host.data() + at, v.data(), bytes);
        return at;
    };
    const size_t o_coef = put(coef), o_pdiag = put(pdiag), o_steps = put(steps), o_mat0 = put(mat0), o_order = put(order),
                 o_level0 = put(start), o_child = put(child), o_step0 = put(step0), o_tip0 = put(tip0), o_tip = put(tipv),
                 o_sub = put(sub);
    const size_t RR = (size_t)R, host_bytes = (host.size() + 7) / 8 * 8;
    const size_t n_dev = 2 * N + (R > 0 ? n_mat + 2 * M + RR * RR + 4 * RR : 0);

    hk_tree *t = new hk_tree();
    hk_tree_free(p);
    p->tree = t;
    t->dense = TreeDense{};
    t->m = m;
    t->levels = H;
    t->logdet = logdet;
    t->root = (int)root;
    t->root_inv = 1.0 / rv;
    t->store = nullptr;
    hipError_t e = hipMalloc(&t->store, host_bytes + 8 * n_dev);
    if (e == hipSuccess) e = hipMemcpy(t->store, host.data(), host.size(), hipMemcpyHostToDevice);
    char *const base = (char *)t->store;
    double *dev = (double *)(base + host_bytes);
    const auto take = [&](size_t n) { return std::exchange(dev, dev + n); };
    t->coef = (double *)(base + o_coef);
    t->pdiag = (double *)(base + o_pdiag);
    t->order = (int *)(base + o_order);
    t->level0 = (int *)(base + o_level0);
    t->child = (int *)(base + o_child);
    t->mv = take(N);
    t->dd = take(N);
    if (R > 0 && e == hipSuccess) {
        double *mat = take(n_mat), *w = take(M), *Q = take(RR * RR), *qrow = take(RR);
        TreeDense &td = t->dense;
        td.R = R;
        td.tip0 = (int *)(base + o_tip0);
        td.tip = (int *)(base + o_tip);
        td.sub = (int *)(base + o_sub);
        td.mat0 = (int64_t *)(base + o_mat0);
        td.mat = mat;
        td.w = w;
        td.Q = Q;
        td.qrow = qrow;
        td.y = take(M);
        td.mean = take(RR);
        td.qlow = take(RR);
        td.quad = take(RR);
        hipLaunchKernelGGL(k_tree_cut, dim3(R + 1), dim3(TREE_CUT_THREADS), 0, 0, (const TreeStep *)(base + o_steps),
                           (const int *)(base + o_step0), R, td.tip0, td.mat0, t->root_inv, mat, w, Q, qrow);
        e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(0);
    }
    if (e != hipSuccess) {
        hk_tree_free(p);
        return e == hipErrorOutOfMemory ? HAWKES_E_NOMEM : HAWKES_E_DEVICE;
    }
    return HAWKES_OK;
}

extern "C" hawkes_status hawkes_plan_set_tree(hawkes_plan p, int64_t n_nodes, const int64_t *parent,
                                              const double *length, double tau0) {
    try {
        return set_tree(p, n_nodes, parent, length, tau0);
    } catch (const std::bad_alloc &) {  // (the plan's former tree, if any, is still set)
        return HAWKES_E_NOMEM;
    }
}

extern "C" hawkes_status hawkes_tree_prior(hawkes_plan p, const double *d_z, double sigma, double *d_logp,
                                           double *d_grad, double *d_quad, hipStream_t stream) {
    if (!p || !d_z || !(sigma > 0.0) || !isfinite(sigma) || !d_quad) return HAWKES_E_INVALID;
    hk_tree *t = p->tree;
    if (!t) return HAWKES_E_UNSUPPORTED;
    p->last_stream = stream;
    // the walk leaves the adjoints of the tips in mv[0..m), the dense steps V^{-1} z there
    const bool walk = t->levels <= TREE_WALK_LEVELS + (t->m <= TREE_THREADS ? 2 : 0);
    const TreeDense *td = walk ? nullptr : hk_tree_dense(p);
    if (td) {
        hipLaunchKernelGGL(k_tree_low, dim3(td->R), dim3(HK_WAVE), 0, stream, *td, d_z);
        hipLaunchKernelGGL(k_tree_top, dim3(hk_tree_top_blocks(td->R)), dim3(HK_TREE_TOP_THREADS), 0, stream, *td,
                           t->mv);
    } else {
        const hawkes_status st = hk_tree_walk(p, d_z, nullptr, d_quad, stream);
        if (st != HAWKES_OK) return st;
    }
    if (td || d_logp || d_grad)
        hipLaunchKernelGGL(k_tree_logp, dim3(d_grad ? (unsigned)((t->m + 255) / 256) : 1), dim3(256), 0, stream,
                           td ? td->quad : (const double *)nullptr, td ? td->R : 0, d_quad, t->mv, t->m, sigma * sigma,
                           t->logdet, d_logp, d_grad);
    HK_CHECK(hipGetLastError());
    return HAWKES_OK;
}
