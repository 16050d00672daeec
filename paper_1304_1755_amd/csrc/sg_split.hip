// Kernels of the block-triangular preconditioner with the 2 x 2 split of
// Sec. 4.2, B_T = [[A_hat, 0], [W, D]]: A_hat (the modes of degree <= p-1)
// is inverted by one multigrid cycle for the coupled system, with point
// Gauss-Seidel on the assembled A_hat_l in its natural order (mode by mode,
// inside a mode node by node, x fastest).
//
// Modes of one total degree do not couple (G_k(alpha, beta) != 0 only for
// beta = alpha +- e_k), and the mode order is graded, so a Gauss-Seidel sweep
// in that order updates all modes of degree d together: each from the new
// values of degree d-1 and the old ones of degree d+1 (backward sweep: the
// reverse), by one lexicographic sweep of its diagonal block K_0 against the
// right-hand side f_alpha - sum_k sum_beta G_k(alpha, beta) K_k u_beta.  This
// file holds that coupling (also the residual of A_hat_l when the K_0 term is
// included) and the direct solve on the coarsest level; the lexicographic
// sweep and the transfers are those of the K_0 hierarchy.

#include "sg_internal.h"

namespace sg {

namespace {

// out[node, t] = f[node, lo+t] - self (K_0 u_{lo+t})(node)
//                - sum over the partners beta of alpha = lo+t of G_k(alpha, beta) (K_k u_beta)(node).
// Four adjacent lanes per (node, output mode), modes fastest: lane g takes the partners g, g + 4, ... (the
// K_0 term is lane 3's last), so that a lane's few stencils have all their loads in flight at once; the
// lanes' sums meet by shuffles.  (With one lane an output the partners' dependent loads run one after
// another: 13.8 -> 5.9 us a launch over the couplings of the 65 x 65 problem's cycles, 1 to 84 modes on 7^2 to
// 63^2 nodes.)  The stencils of K_k on this level
// are block k of sten ((m+1) x N x 9); the partners of a mode are packed first in its row of pidx
// (beta | k << 16), -1 after the last.
constexpr int kCoupleLanes = 4;
constexpr int kCoupleTerms = 4;  // terms of a lane
static_assert(kCoupleLanes * kCoupleTerms >= 2 * kMaxM, "a mode has up to 2 m partners: a term would be dropped");
__global__ void __launch_bounds__(256) k_split_couple(const double* __restrict__ sten, int N,
                                                      const int* __restrict__ pidx,
                                                      const double* __restrict__ pcoef, int npart,
                                                      const double* __restrict__ u, int ldu,
                                                      const double* __restrict__ f, int ldf,
                                                      double* __restrict__ out, int ldo, int nx, int lo, int width,
                                                      int self) {
    const long idx = ((long)blockIdx.x * blockDim.x + threadIdx.x) / kCoupleLanes;
    const int g = threadIdx.x % kCoupleLanes;
    if (idx >= (long)N * width) return;  // whole groups of lanes
    const int node = (int)(idx / width), t = (int)(idx - (long)node * width), a = lo + t;
    const int y = node / nx, x = node - y * nx;
    // the nine nodes around this one, clamped into the grid, and which of them it has
    int nb[9];
    bool in[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) {
        const int xx = x + e % 3 - 1, yy = y + e / 3 - 1;
        in[e] = xx >= 0 && xx < nx && yy >= 0 && yy < nx;
        nb[e] = in[e] ? yy * nx + xx : node;
    }
    int p[kCoupleTerms];
    double c[kCoupleTerms];
#pragma unroll
    for (int i = 0; i < kCoupleTerms; ++i) {
        const int q = g + i * kCoupleLanes;
        p[i] = q < npart ? pidx[a * npart + q] : -1;
        c[i] = q < npart ? pcoef[a * npart + q] : 0.0;
    }
    // (K_k u_b)(node)
    auto stencil = [&](int k, int b) -> double {
        const double* s9 = sten + ((size_t)k * N + node) * 9;
        double s[9], w[9], v = 0.0;
#pragma unroll
        for (int e = 0; e < 9; ++e) {
            s[e] = s9[e];
            w[e] = u[(size_t)nb[e] * ldu + b];
        }
#pragma unroll
        for (int e = 0; e < 9; ++e) v = fma(s[e], in[e] ? w[e] : 0.0, v);
        return v;
    };
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < kCoupleTerms; ++i)
        if (p[i] >= 0) acc = fma(c[i], stencil(p[i] >> 16, p[i] & 0xFFFF), acc);
    if (self && g == kCoupleLanes - 1) acc += stencil(0, a);
#pragma unroll
    for (int o = 1; o < kCoupleLanes; o <<= 1) acc += __shfl_xor(acc, o);
    if (g == 0) out[(size_t)node * ldo + t] = f[(size_t)node * ldf + a] - acc;
}

// u = A_hat_c^{-1} f on the coarsest level: one wavefront per row of the
// inverse (rows and columns indexed node * Pa + alpha), lanes over columns.
__global__ void __launch_bounds__(256) k_split_coarse(const double* __restrict__ cinv, int nA, int Pa,
                                                      const double* __restrict__ f, int ldf,
                                                      double* __restrict__ u, int ldu) {
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= nA) return;  // uniform per wavefront
    double acc = 0.0;
    for (int j = lane; j < nA; j += 64) {
        const int nd = j / Pa, b = j - nd * Pa;
        acc = fma(cinv[(size_t)row * nA + j], f[(size_t)nd * ldf + b], acc);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane == 0) {
        const int nd = row / Pa, a = row - nd * Pa;
        u[(size_t)nd * ldu + a] = acc;
    }
}

}  // namespace

int launch_split_couple(sg_ctx* c, int l, const double* u, int ldu, const double* f, int ldf, double* out, int ldo,
                        int lo, int width, int self) {
    const SplitDev& sp = c->split;
    const Level& lv = c->levels[l];
    const long total = (long)lv.N * width * kCoupleLanes;
    if (total == 0) return SG_OK;
    hipLaunchKernelGGL(k_split_couple, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, c->stream, sp.sten[l],
                       lv.N, sp.pidx, sp.pcoef, sp.npart, u, ldu, f, ldf, out, ldo, lv.nx, lo, width, self);
    return hipGetLastError() == hipSuccess ? SG_OK : SG_EHIP;
}

int launch_split_coarse(sg_ctx* c, const double* f, int ldf, double* u, int ldu) {
    const SplitDev& sp = c->split;
    const int nA = c->levels.back().N * sp.Pa;
    hipLaunchKernelGGL(k_split_coarse, dim3((nA + 3) / 4), dim3(256), 0, c->stream, sp.cinv, nA, sp.Pa, f, ldf, u,
                       ldu);
    return hipGetLastError() == hipSuccess ? SG_OK : SG_EHIP;
}

}  // namespace sg
