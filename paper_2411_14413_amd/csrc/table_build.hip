// table_build.hip -- FP64 scattering-angle and cross-section tables on the GPU.
//
// The paper names a screened-Coulomb interaction with Moliere screening for the
// collisions of sputtered atoms with the gas (closing calculation paragraph of
// Methods).  In reduced units x = r/a, beta = b/a, eps = a E_r/(Z1 Z2 e^2) the
// classical centre-of-mass deflection is
//     theta = pi - 2 (beta/x0) Int_0^1 du / sqrt(h(u)),
//     h(u) = 1 - u Phi(x0/u)/(x0 eps) - beta^2 u^2/x0^2,
// with x0 the distance of closest approach (h(1) = 0).  Substituting u = cos(psi)
// turns the integral into Int_0^{pi/2} sqrt(sin^2 psi / h(cos psi)) d psi, whose
// integrand is smooth with vanishing odd derivatives at both ends for a screened
// potential, so the midpoint rule in psi converges faster than any power of 1/N.
// The table depends only on (eps, b/b_max): one table serves every species pair.
#include <hip/hip_runtime.h>
#include <math.h>

#include "spx_host.hpp"

namespace spx {

__device__ __forceinline__ double moliere(double x)
{
    return 0.35 * exp(-0.3 * x) + 0.55 * exp(-1.2 * x) + 0.10 * exp(-6.0 * x);
}

// h(1) as a function of x: 1 - Phi(x)/(x eps) - beta^2/x^2 (increasing in x).
__device__ __forceinline__ double f_root(double x, double eps, double beta)
{
    return 1.0 - moliere(x) / (x * eps) - beta * beta / (x * x);
}

constexpr int NQ = 512;                 // quadrature nodes

// The nodes' sines and cosines, the same for every angle of the table: once per block in LDS
// instead of once per node and angle (a double sincos is a third of a node's work).
__device__ __forceinline__ void quadrature_nodes(double* sn, double* cn)
{
    const double dpsi = 0.5 * M_PI / NQ;
    for (int k = threadIdx.x; k < NQ; k += blockDim.x) {
        double sp, cp;
        sincos((k + 0.5) * dpsi, &sp, &cp);
        sn[k] = sp;
        cn[k] = cp;
    }
    __syncthreads();
}

// Bisection by a group of G = 2^L lanes, bit for bit the one-lane loop
//     mid = (lo + hi) / 2; stop if mid <= lo or mid >= hi; lo or hi = mid
// L halvings a round: lane n of the group evaluates the n-th node (1 .. G - 1) of the binary tree of
// the next L midpoints, each midpoint formed by halving along its path as the loop would.
__device__ __forceinline__ double tree_mid(double lo, double hi, int n)
{
    double mid = 0.5 * (lo + hi);
    for (int d = 30 - __clz(n > 0 ? n : 1); d >= 0; --d) {
        if ((n >> d) & 1) lo = mid; else hi = mid;
        mid = 0.5 * (lo + hi);
    }
    return mid;
}
// Follow the tree by the nodes' answers (bit n of `high`: hi becomes the midpoint of node n).
// Returns whether the bisection ended.
template <int L> __device__ __forceinline__ bool tree_follow(double& lo, double& hi, uint64_t high, int& left)
{
    int n = 1;
    for (int l = 0; l < L; ++l) {
        const double mid = 0.5 * (lo + hi);
        if (left <= 0 || mid <= lo || mid >= hi) return true;
        --left;
        const bool up = (high >> n) & 1u;
        if (up) hi = mid; else lo = mid;
        n = 2 * n + (up ? 0 : 1);
    }
    return false;
}

// Closest approach by a group of G = 2^L lanes of one (eps, beta); g: lane of the group, base: its
// first lane.  The upper end is doubled until it lies beyond the root (G doublings a round), then
// the root is bisected.
template <int G, int L> __device__ double closest_approach(double eps, double beta, int g, int base)
{
    constexpr uint64_t MASK = G == 64 ? ~0ull : (1ull << (G & 63)) - 1;
    double lo = beta, hi = beta > 1.0 ? beta : 1.0;
    for (int k = 0; k < 2100; k += G) {
        const uint64_t beyond = (__ballot(!(f_root(ldexp(hi, g), eps, beta) <= 0.0)) >> base) & MASK;
        if (beyond) {
            hi = ldexp(hi, __ffsll((unsigned long long)beyond) - 1);
            break;
        }
        hi = ldexp(hi, G);
    }
    int left = 200;
    bool done = false;
    while (!done) {
        const uint64_t high = (__ballot(f_root(tree_mid(lo, hi, g), eps, beta) > 0.0) >> base) & MASK;
        done = tree_follow<L>(lo, hi, high, left);
    }
    return 0.5 * (lo + hi);
}

// Integrand of the deflection at one node.
__device__ __forceinline__ double theta_term(double eps, double x0, double ib, double sp, double cp)
{
    const double u = cp;
    double h = 1.0 - u * moliere(x0 / u) / (x0 * eps) - ib * ib * u * u;
    h = h > 1e-300 ? h : 1e-300;
    return sqrt(sp * sp / h);
}
__device__ __forceinline__ double theta_of(double ib, double sum)
{
    const double dpsi = 0.5 * M_PI / NQ;
    return M_PI - 2.0 * ib * sum * dpsi;
}

// theta_cm of one (eps, beta) by a wave: eight nodes a lane, their terms through LDS and added in
// node order by every lane alike (the sum of a one-lane loop, bit for bit).
__device__ double theta_wave(double eps, double beta, const double* sn, const double* cn, double* term, int lane)
{
    if (beta <= 0.0) return M_PI;
    const double x0 = closest_approach<64, 6>(eps, beta, lane, 0);
    const double ib = beta / x0;
    for (int k = lane; k < NQ; k += 64) term[k] = theta_term(eps, x0, ib, sn[k], cn[k]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    double sum = 0.0;
#pragma unroll 16
    for (int k = 0; k < NQ; ++k) sum += term[k];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return theta_of(ib, sum);
}

// beta_max of one eps node per block: eight doublings of the upper end a round, then three
// halvings a round (the seven midpoints of their tree, one wave each), every decision that of the
// one-thread search.  Bound by the chain of rounds (about 20, each a root search, eight nodes a
// lane and an ordered sum): one thread per eps node, 57 dependent quadratures each, took 15.1 ms
// for 256 nodes.
constexpr int BM_WAVES = 8;
__global__ void __launch_bounds__(64 * BM_WAVES) k_betamax(int ne, double lo, double hi, double theta_min,
                                                           double* __restrict__ betamax, float* __restrict__ betamax32)
{
    __shared__ double sn[NQ], cn[NQ], term[BM_WAVES][NQ], th[2][BM_WAVES];
    const int i = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    quadrature_nodes(sn, cn);
    const double eps = pow(10.0, lo + (hi - lo) * (double)i / (double)(ne - 1));
    double blo = 0.0, bhi = 1.0;
    int par = 0;                            // results of successive rounds alternate: one barrier a round
    for (int k = 0; k < 64; k += BM_WAVES) {
        const double t = theta_wave(eps, ldexp(bhi, wv), sn, cn, term[wv], lane);
        if (lane == 0) th[par][wv] = t;
        __syncthreads();
        int n = 0;
        while (n < BM_WAVES && th[par][n] > theta_min) ++n;
        par ^= 1;
        if (n > 0) {
            blo = ldexp(bhi, n - 1);
            bhi = ldexp(bhi, n);
        }
        if (n < BM_WAVES) break;
    }
    int left = 200;
    bool done = false;
    while (!done) {
        const double t = wv == 0 ? 0.0 : theta_wave(eps, tree_mid(blo, bhi, wv), sn, cn, term[wv], lane);
        if (lane == 0) th[par][wv] = t;
        __syncthreads();
        uint64_t high = 0;
        for (int n = 1; n < BM_WAVES; ++n) high |= (uint64_t)(th[par][n] > theta_min ? 0 : 1) << n;
        par ^= 1;
        done = tree_follow<3>(blo, bhi, high, left);
    }
    if (threadIdx.x == 0) {
        const double b = 0.5 * (blo + bhi);
        betamax[i] = b;
        betamax32[i] = (float)b;
    }
}

template <int I> __device__ __forceinline__ double quad_lane(double v)
{
    constexpr int CTRL = I * 0x55;          // quad_perm [I, I, I, I]
    const int l = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int h = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(h, l);
}

// theta(eps, b / b_max), four lanes an angle: each evaluates every fourth node, and all four add the
// terms in node order.  Bound by FP64 issue (about 160 instructions a node); four waves per SIMD at
// the default table hide the chains that one lane an angle left open, and the column b = 0 (pi) is
// written without a lane of its own, so that 256 x 256 angles fill the SIMDs evenly: 474 us before.
__global__ void __launch_bounds__(256) k_theta(int ne, int ns, double lo, double hi, const double* __restrict__ betamax,
                                               double* __restrict__ theta, float* __restrict__ theta32)
{
    __shared__ double sn[NQ], cn[NQ];
    quadrature_nodes(sn, cn);
    const int lane = threadIdx.x & 63, g = lane & 3, base = lane & ~3;
    const int64_t id = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 2, n = (int64_t)ne * (ns - 1);
    const int64_t a = id < n ? id : n - 1;          // lanes past the end repeat the last angle
    const int i = (int)(a / (ns - 1)), j = (int)(a - (int64_t)i * (ns - 1)) + 1;
    const double eps = pow(10.0, lo + (hi - lo) * (double)i / (double)(ne - 1));
    const double s = (double)j / (double)(ns - 1);
    const double beta = s * betamax[i];
    double t = M_PI;
    if (beta > 0.0) {
        const double x0 = closest_approach<4, 2>(eps, beta, g, base);
        const double ib = beta / x0;
        double sum = 0.0;
        for (int k = 0; k < NQ; k += 4) {
            const double v = theta_term(eps, x0, ib, sn[k + g], cn[k + g]);
            sum += quad_lane<0>(v);
            sum += quad_lane<1>(v);
            sum += quad_lane<2>(v);
            sum += quad_lane<3>(v);
        }
        t = theta_of(ib, sum);
    }
    if (id < n && g == 0) {
        const int64_t idx = (int64_t)i * ns + j;
        theta[idx] = t;
        theta32[idx] = (float)t;
        if (j == 1) {
            theta[idx - 1] = M_PI;
            theta32[idx - 1] = (float)M_PI;
        }
    }
}

int build_tables(Plan* P)
{
    const int ne = P->params.table_ne, ns = P->params.table_ns;
    const double lo = P->params.log_eps_lo, hi = P->params.log_eps_hi;
    hipStream_t st = P->work_stream;
    hipLaunchKernelGGL(k_betamax, dim3(ne), dim3(64 * BM_WAVES), 0, st, ne, lo, hi, P->params.theta_min, P->d_betamax64,
                       P->d_betamax32);
    SPX_HIP(hipGetLastError());
    const int64_t lanes = 4 * (int64_t)ne * (ns - 1);
    hipLaunchKernelGGL(k_theta, dim3((unsigned)((lanes + 255) / 256)), dim3(256), 0, st, ne, ns, lo, hi, P->d_betamax64,
                       P->d_theta64, P->d_theta32);
    SPX_HIP(hipGetLastError());
    P->h_betamax.resize(ne);
    SPX_HIP(hipMemcpyAsync(P->h_betamax.data(), P->d_betamax64, sizeof(double) * ne, hipMemcpyDeviceToHost, st));
    SPX_HIP(hipStreamSynchronize(st));
    return SPX_OK;
}

}  // namespace spx
