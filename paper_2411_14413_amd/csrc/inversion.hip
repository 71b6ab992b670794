// inversion.hip -- recovering a geometry parameter from a sweep of simulated libraries.
//
// The cathode-tilt study of the Results repeats the simulation over a range of tilts and
// compares every simulated library with the measured one, by the compositional area it covers
// (Figure 8: for a ternary library, the area of the convex hull of its compositions in the
// ternary diagram) and by d_e.  After the transport of the whole sweep in one launch and the
// area gather, three kernels finish the inversion on the device:
//   k_sweep_composition  at.% of each sweep point's library, normalised by its own calibration
//                        value (the mean of its area values), in double;
//   k_hull_area          covered area of each ternary library: the points are sorted in LDS
//                        (bitonic), then two waves walk the chains of Andrew's algorithm;
//   k_sweep_fit          the sweep value that minimises a misfit, or at which a curve reaches a
//                        target.
// Decisions (the hull's turns, the bracket of a fit) are taken in double with contraction off,
// so that they are the plain IEEE operations a reader would write down.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "spx_host.hpp"

namespace spx {

constexpr int SWEEP_KMAX = 16;
constexpr int SWEEP_WAVE_AREAS = 1536;
constexpr int HULL_JMAX = 2048;
constexpr int FIT_TMAX = 256;
constexpr double SQRT3 = 1.7320508075688772;   // sqrt(3) rounded to double

// ---- compositions of a sweep -----------------------------------------------------------
// One workgroup per sweep point t.  fref[k] = (sum_j f[t,k,j]) / J in the order of 256 strided partial sums and a
// tree over them, so results are repeatable: a wave per element (lane l holds partials l, l + 64, l + 128
// and l + 192) and one barrier, or LONG the whole workgroup for one element after the other, a partial a
// thread, the same bits.  Bound by the workgroup's chain of loads.  A wave / the workgroup [us]: 8 points of 342
// areas and 3 elements 11.6 / 10.8, of 16 14.6 / 21.3; 1500 areas 12.7 / 12.0, 38 / 43; 2048 14.9 / 12.7, 50 / 45;
// 40000 224 / 163, 1434 / 960.
template <int THREADS, bool LONG>
__global__ __launch_bounds__(THREADS) void k_sweep_composition(const double* __restrict__ f,
                                                               const double* __restrict__ a,
                                                               const double* __restrict__ bb,
                                                               const double* __restrict__ P,
                                                               const double* __restrict__ M,
                                                               const double* __restrict__ rho,
                                                               float* __restrict__ c, int J, int K)
{
    __shared__ double w[SWEEP_KMAX];
    __shared__ double part[LONG ? 2 : 1][LONG ? THREADS : 1];   // of successive elements in turn
    const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const double* ft = f + (size_t)t * K * J;
    for (int k = LONG ? 0 : tid >> 6; k < K; k += LONG ? 1 : THREADS / 64) {
        double v;
        if constexpr (LONG) {
            static_assert(THREADS == 256, "a partial sum a thread");
            double s = 0.0;
#pragma unroll 8
            for (int j = tid; j < J; j += 256) s += ft[(size_t)k * J + j];
            part[k & 1][tid] = s;
            __syncthreads();
            if (tid >= 64) continue;
            const double* p = part[k & 1] + lane;
            v = (p[0] + p[128]) + (p[64] + p[192]);
        } else {
            double s[4] = {0.0, 0.0, 0.0, 0.0};
            for (int j0 = 0; j0 < J; j0 += 256) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int j = j0 + 64 * q + lane;
                    if (j < J) s[q] += ft[(size_t)k * J + j];
                }
            }
            s[0] += s[2];
            s[1] += s[3];
            v = s[0] + s[1];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
        if (lane == 0) {
            const double fref = v / (double)J;
            w[k] = (a[k] * P[k] + bb[k]) * rho[k] / (M[k] * fref);
        }
    }
    __syncthreads();
    for (int j = tid; j < J; j += THREADS) {
        double y[SWEEP_KMAX];
        double S = 0.0;
#pragma unroll
        for (int k = 0; k < SWEEP_KMAX; ++k)
            if (k < K) {
                y[k] = w[k] * ft[(size_t)k * J + j];
                S += y[k];
            }
        float* out = c + ((size_t)t * J + j) * K;
#pragma unroll
        for (int k = 0; k < SWEEP_KMAX; ++k)
            if (k < K) out[k] = (float)(100.0 * y[k] / S);
    }
}

// ---- covered area of a ternary library ---------------------------------------------------
#pragma clang fp contract(off)
__device__ __forceinline__ double turn(double ox, double oy, double ax, double ay, double bx, double by)
{
    return (ax - ox) * (by - oy) - (ay - oy) * (bx - ox);
}

__device__ __forceinline__ bool key_less(double x0, double y0, double x1, double y1)
{
    return x0 < x1 || (x0 == x1 && y0 < y1);
}

// One chain of Andrew's algorithm over the sorted points, by a whole wave doing the same on every lane
// (so that every branch is uniform): points i0, i0 + di, ... are pushed onto the stack, which is kept in
// place in the chain's own copy of the points, its two top points in registers.  Returns its length.
__device__ __forceinline__ int hull_chain(double* x, double* y, int J, bool down, int lane)
{
    // slot s of the stack lies where the s-th point of the walk lay: it is read before it is written
    const int i0 = down ? J - 1 : 0, di = down ? -1 : 1;
    int n = 0;
    double ox = 0.0, oy = 0.0, ax = 0.0, ay = 0.0;      // below the top, top
    double bx = x[i0], by = y[i0];
    for (int s = 0; s < J; ++s) {
        const int in = i0 + di * (s + 1 < J ? s + 1 : s);
        const double nx = x[in], ny = y[in];            // the next point, on its way
        while (n >= 2 && __ballot(turn(ox, oy, ax, ay, bx, by) <= 0.0) != 0) {
            --n;
            ax = ox;
            ay = oy;
            if (n >= 2) {
                ox = x[i0 + di * (n - 2)];
                oy = y[i0 + di * (n - 2)];
            }
        }
        if (lane == 0) {
            x[i0 + di * n] = bx;
            y[i0 + di * n] = by;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        ox = ax;
        oy = ay;
        ax = bx;
        ay = by;
        ++n;
        bx = nx;
        by = ny;
    }
    return n;
}

// One workgroup per library.  Points go to LDS in ternary-diagram coordinates.  Of many points those
// that lie inside the polygon of the extreme points in 16 directions, by a margin above the rounding of the
// FP32 test (0.1 at.%^2 of every edge's cross product; where no coordinate exceeds 128 the factors are at most 256,
// each within 3e-5, and the error is below 0.04: beyond that no point is left out), cannot be on the hull
// and are left out: a point to the left of every edge of a closed polygon lies in the hull of its vertices,
// whatever the vertices are, and a degenerate set has no such point.  The others, padded to a power
// of two with +inf, are sorted by (x, y) with a bitonic network (a barrier only where pairs cross the
// 128 points of a wave); wave 0 then builds the lower chain and wave 1 the upper one, and the shoelace
// over the hull is summed in the order lower chain, then upper chain.  Bound by the chains' latency,
// about two turns a point one after the other, 0.23 us a point: with one lane walking both over index
// stacks, a library of 342 areas took 203 us, with the two waves over all points 96 us.
constexpr int HULL_DIRS = 16, HULL_FILTER_MIN = 64;
constexpr float HULL_FILTER_REACH = 128.f;
__constant__ const float HULL_COS[HULL_DIRS] = {1.f, 0.9238795f, 0.70710678f, 0.38268343f, 0.f, -0.38268343f, -0.70710678f,
                                                -0.9238795f, -1.f, -0.9238795f, -0.70710678f, -0.38268343f, 0.f,
                                                0.38268343f, 0.70710678f, 0.9238795f};
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_hull_area(const float* __restrict__ c, int J, float* __restrict__ area)
{
    extern __shared__ double pts[];                     // x, y sorted; x, y for the upper chain
    __shared__ int len[2];
    __shared__ float vx[HULL_DIRS], vy[HULL_DIRS];      // the extreme points
    __shared__ int vi[HULL_DIRS], kept, far;            // far: an extreme point lies beyond the filter's reach
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    if (J < 3) {
        if (tid == 0) area[b] = 0.f;
        return;
    }
    int n = 1;
    while (n < J) n <<= 1;
    double *px = pts, *py = pts + n, *qx = pts + 2 * n, *qy = pts + 2 * n + J;
    const float* cb = c + (size_t)b * J * 3;
    const bool filter = J >= HULL_FILTER_MIN;
    for (int j = tid; j < J; j += THREADS) {
        const double c1 = (double)cb[3 * j + 1], c2 = (double)cb[3 * j + 2];
        qx[j] = c1 + 0.5 * c2;
        qy[j] = c2 * (SQRT3 / 2.0);
    }
    if (tid == 0) {
        kept = 0;
        far = 0;
    }
    __syncthreads();
    if (filter) {
        // four directions a wave: the lanes' extremes of their points, then those of the lanes
        constexpr int D = HULL_DIRS / (THREADS / 64);
        const int d0 = (tid >> 6) * D;
        float best[D];
        int at[D];
        for (int d = 0; d < D; ++d) {
            best[d] = -INFINITY;
            at[d] = 0;
        }
        for (int j = lane; j < J; j += 64) {
            const float x = (float)qx[j], y = (float)qy[j];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                // sin t = cos(t - 90 deg)
                const float v = HULL_COS[d0 + d] * x + HULL_COS[(d0 + d + 12) & 15] * y;
                at[d] = v > best[d] ? j : at[d];
                best[d] = v > best[d] ? v : best[d];
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const float v = __shfl_xor(best[d], o);
                const int i = __shfl_xor(at[d], o);
                at[d] = v > best[d] ? i : at[d];
                best[d] = v > best[d] ? v : best[d];
            }
        if (lane == 0)
            for (int d = 0; d < D; ++d) {
                vi[d0 + d] = at[d];
                vx[d0 + d] = (float)qx[at[d]];
                vy[d0 + d] = (float)qy[at[d]];
                if (!(fabsf(vx[d0 + d]) <= HULL_FILTER_REACH && fabsf(vy[d0 + d]) <= HULL_FILTER_REACH)) far = 1;
            }
        __syncthreads();
        const bool near = far == 0;
        for (int j0 = 0; j0 < J; j0 += THREADS) {
            const int j = j0 + tid;
            bool keep = j < J;
            double x = 0.0, y = 0.0;
            if (keep) {
                x = qx[j];
                y = qy[j];
                const float fx = (float)x, fy = (float)y;
                bool inside = true;
                int edges = 0;
                for (int d = 0; d < HULL_DIRS; ++d) {
                    const int p = (d + HULL_DIRS - 1) & (HULL_DIRS - 1);
                    const float cr = (vx[d] - vx[p]) * (fy - vy[p]) - (vy[d] - vy[p]) * (fx - vx[p]);
                    const bool edge = vi[d] != vi[p];
                    inside = inside && (!edge || cr > 0.1f);
                    edges += edge ? 1 : 0;
                }
                keep = !(inside && near && edges >= 3);
            }
            const uint64_t m = __ballot(keep);
            int base = 0;
            if (lane == 0) base = atomicAdd(&kept, (int)__popcll(m));
            base = __shfl(base, 0) + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (keep) {
                px[base] = x;
                py[base] = y;
            }
        }
        __syncthreads();
        J = kept;                                       // at least the polygon's vertices
        n = 1;
        while (n < J) n <<= 1;
        for (int j = J + tid; j < n; j += THREADS) {
            px[j] = INFINITY;
            py[j] = INFINITY;
        }
    } else {
        for (int j = tid; j < n; j += THREADS) {
            px[j] = j < J ? qx[j] : INFINITY;
            py[j] = j < J ? qy[j] : INFINITY;
        }
    }
    __syncthreads();
    for (int size = 2; size <= n; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < n / 2; i += THREADS) {
                const int lo_i = 2 * i - (i & (stride - 1));          // first of the pair
                const int hi_i = lo_i + stride;
                const bool up_dir = (lo_i & size) == 0;
                const double x0 = px[lo_i], y0 = py[lo_i], x1 = px[hi_i], y1 = py[hi_i];
                const bool swap = up_dir ? key_less(x1, y1, x0, y0) : key_less(x0, y0, x1, y1);
                if (swap) {
                    px[lo_i] = x1;
                    py[lo_i] = y1;
                    px[hi_i] = x0;
                    py[hi_i] = y0;
                }
            }
            // pairs up to 64 apart stay within the 128 points of a wave
            const int next = stride > 1 ? stride >> 1 : size;
            if (stride > 64 || next > 64) {
                __syncthreads();
            } else {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
    __syncthreads();
    for (int j = tid; j < J; j += THREADS) {
        qx[j] = px[j];
        qy[j] = py[j];
    }
    __syncthreads();
    const int wv = tid >> 6;
    if (wv < 2) {
        const int m = hull_chain(wv ? qx : px, wv ? qy : py, J, wv == 1, lane);
        if (lane == 0) len[wv] = m;
    }
    __syncthreads();
    if (tid != 0) return;
    const int nl = len[0], nu = len[1];
    // hull = lower chain without its last point, then upper chain (walked downwards from the end of its
    // copy) without its last point
    const int nh = (nl - 1) + (nu - 1);
    double s = 0.0, x0 = px[0], y0 = py[0];
    const double fx = x0, fy = y0;
    for (int h = 0; h < nh; ++h) {
        const int h1 = h + 1;
        const bool first = h1 == nh, lower = h1 < nl - 1;
        const int u = J - 1 - (h1 - (nl - 1));
        const double x1 = first ? fx : lower ? px[h1] : qx[u], y1 = first ? fy : lower ? py[h1] : qy[u];
        s += x0 * y1 - x1 * y0;
        x0 = x1;
        y0 = y1;
    }
    area[b] = (float)(0.5 * s / (SQRT3 / 4.0 * 100.0 * 100.0));
}

// ---- fit over a sweep ----------------------------------------------------------------------
struct SweepX {
    double x[FIT_TMAX];
};

// Sweep values as u = (x - mean) / half-range in [-1, 1]; curves are centred on their mean, so a
// flat curve fits exactly zero.  Sums run over t in ascending order.
__device__ void sweep_coords(const SweepX& X, int T, double& xm, double& h)
{
    double sx = 0.0;
    for (int t = 0; t < T; ++t) sx += X.x[t];
    xm = sx / (double)T;
    h = 0.5 * (X.x[T - 1] - X.x[0]);
}

__device__ double mean_of(const float* y, int T)
{
    double s = 0.0;
    for (int t = 0; t < T; ++t) s += (double)y[t];
    return s / (double)T;
}

// Least-squares parabola y - mean(y) ~ p0 + p1 u + p2 u^2 (normal equations, Cramer's rule);
// its vertex if it opens upwards, kept inside the sweep, else the smallest sample.
__device__ double fit_min(const SweepX& X, const float* y, int T)
{
    int i = 0;
    for (int t = 1; t < T; ++t)
        if ((double)y[t] < (double)y[i]) i = t;
    if (T < 3) return X.x[i];
    double xm, h;
    sweep_coords(X, T, xm, h);
    const double ym = mean_of(y, T);
    double S[5] = {0, 0, 0, 0, 0}, Y[3] = {0, 0, 0};
    for (int t = 0; t < T; ++t) {
        const double u = (X.x[t] - xm) / h, yc = (double)y[t] - ym;
        double uk = 1.0;
        for (int k = 0; k < 5; ++k) {
            S[k] += uk;
            if (k < 3) Y[k] += yc * uk;
            uk *= u;
        }
    }
    // | S0 S1 S2 |       | Y0 |
    // | S1 S2 S3 | p  =  | Y1 |
    // | S2 S3 S4 |       | Y2 |
    const double c00 = S[2] * S[4] - S[3] * S[3], c01 = S[1] * S[4] - S[3] * S[2], c02 = S[1] * S[3] - S[2] * S[2];
    const double det = S[0] * c00 - S[1] * c01 + S[2] * c02;
    const double d1 = S[0] * (Y[1] * S[4] - S[3] * Y[2]) - Y[0] * c01 + S[2] * (S[1] * Y[2] - Y[1] * S[2]);
    const double d2 = S[0] * (S[2] * Y[2] - Y[1] * S[3]) - S[1] * (S[1] * Y[2] - Y[1] * S[2]) + Y[0] * c02;
    const double p1 = d1 / det, p2 = d2 / det;
    if (!(p2 > 0.0)) return X.x[i];
    const double v = xm - h * p1 / (2.0 * p2);
    return fmin(fmax(v, X.x[0]), X.x[T - 1]);
}

// Least-squares line through the samples; where it reaches the target, NaN outside the sweep
// or for a flat line.
__device__ double fit_match(const SweepX& X, const float* y, int T, double target)
{
    if (T < 2) return NAN;
    double xm, h;
    sweep_coords(X, T, xm, h);
    const double ym = mean_of(y, T);
    double su = 0.0;
    for (int t = 0; t < T; ++t) su += (X.x[t] - xm) / h;
    const double um = su / (double)T;
    double sxy = 0.0, sxx = 0.0;
    for (int t = 0; t < T; ++t) {
        const double uc = (X.x[t] - xm) / h - um;
        sxy += uc * ((double)y[t] - ym);
        sxx += uc * uc;
    }
    const double q1 = sxy / sxx;
    if (q1 == 0.0) return NAN;
    const double v = xm + h * (um + (target - ym) / q1);
    return (v >= X.x[0] && v <= X.x[T - 1]) ? v : NAN;
}

__global__ __launch_bounds__(64) void k_sweep_fit(SweepX X, const float* __restrict__ y, int B, int T, int mode,
                                                  const float* __restrict__ target, double* __restrict__ out)
{
    for (int b = threadIdx.x; b < B; b += 64)
        out[b] = mode == SPX_FIT_MIN ? fit_min(X, y + (size_t)b * T, T)
                                     : fit_match(X, y + (size_t)b * T, T, (double)target[b]);
}
#pragma clang fp contract(on)

}  // namespace spx

using namespace spx;

extern "C" int spx_sweep_composition(const double* d_f, const double* d_a, const double* d_b, const double* d_P,
                                     const double* d_M, const double* d_rho, float* d_c, int32_t T, int32_t J,
                                     int32_t K, void* stream)
{
    if (T <= 0 || J <= 0 || K <= 0 || K > SWEEP_KMAX) {
        set_error("spx_sweep_composition: need T, J > 0 and 0 < K <= 16");
        return SPX_EINVAL;
    }
    if (!d_f || !d_a || !d_b || !d_P || !d_M || !d_rho || !d_c) {
        set_error("spx_sweep_composition: null pointer");
        return SPX_EINVAL;
    }
    for (int64_t t0 = 0; t0 < T; t0 += GRID_MAX) {
        const auto kern = J > SWEEP_WAVE_AREAS ? k_sweep_composition<256, true> : k_sweep_composition<256, false>;
        hipLaunchKernelGGL(kern, dim3((unsigned)std::min<int64_t>(T - t0, GRID_MAX)), dim3(256), 0, (hipStream_t)stream,
                           d_f + t0 * K * J, d_a, d_b, d_P, d_M, d_rho, d_c + t0 * J * K, J, K);
        SPX_HIP(hipGetLastError());
    }
    return SPX_OK;
}

extern "C" int spx_hull_area(const float* d_c, int32_t B, int32_t J, float* d_area, void* stream)
{
    if (B <= 0 || J <= 0 || J > HULL_JMAX || !d_c || !d_area) {
        set_error("spx_hull_area: need B > 0, 0 < J <= 2048 and non-null pointers");
        return SPX_EINVAL;
    }
    int n = 1;
    while (n < J) n <<= 1;
    const size_t smem = sizeof(double) * 2 * (size_t)(n + J);       // at most 64 KB, besides 0.2 KB of the kernel's own
    for (int64_t b0 = 0; b0 < B; b0 += GRID_MAX) {
        hipLaunchKernelGGL(k_hull_area<256>, dim3((unsigned)std::min<int64_t>(B - b0, GRID_MAX)), dim3(256), smem,
                           (hipStream_t)stream, d_c + 3 * b0 * J, J, d_area + b0);
        SPX_HIP(hipGetLastError());
    }
    return SPX_OK;
}

extern "C" int spx_sweep_fit(const double* h_x, const float* d_y, int32_t B, int32_t T, int32_t mode,
                             const float* d_target, double* d_xfit, void* stream)
{
    if (B <= 0 || T <= 0 || T > FIT_TMAX || !h_x || !d_y || !d_xfit) {
        set_error("spx_sweep_fit: need B > 0, 0 < T <= 256 and non-null pointers");
        return SPX_EINVAL;
    }
    if (mode != SPX_FIT_MIN && mode != SPX_FIT_MATCH) {
        set_error("spx_sweep_fit: unknown mode");
        return SPX_EINVAL;
    }
    if (mode == SPX_FIT_MATCH && !d_target) {
        set_error("spx_sweep_fit: SPX_FIT_MATCH needs targets");
        return SPX_EINVAL;
    }
    SweepX X{};
    for (int t = 0; t < T; ++t) {
        if (!std::isfinite(h_x[t]) || (t > 0 && !(h_x[t] > h_x[t - 1]))) {
            set_error("spx_sweep_fit: sweep values must be finite and strictly increasing");
            return SPX_EINVAL;
        }
        X.x[t] = h_x[t];
    }
    hipLaunchKernelGGL(k_sweep_fit, dim3(1), dim3(64), 0, (hipStream_t)stream, X, d_y, B, T, mode, d_target, d_xfit);
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}
