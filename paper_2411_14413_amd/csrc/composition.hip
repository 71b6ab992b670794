// composition.hip -- from deposition profiles to at.% and back.
//
// The paper converts the simulated arrival fraction of each element into a
// composition by weighting it with the element's sputter rate, which is linear in
// the cathode power, and then with its nominal bulk density over atomic mass
// (Introduction, and the calculation paragraph closing Methods).  The accuracy
// measure is the Euclidean distance d_e of compositions (Results).  With
//   w[b,k] = (a_k P[b,k] + bb_k) rho_k / (M_k fref_k),  y = w[b,k] f[k,j],
//   c[b,j,k] = 100 y[b,j,k] / S[b,j],  S = sum_k y[b,j,k],
// the backward pass is
//   gy[b,j,m] = (100 gc[b,j,m] - sum_k gc[b,j,k] c[b,j,k]) / S[b,j]
//   gw[b,m]   = sum_j gy[b,j,m] f[m,j]          gf[m,j] = sum_b gy[b,j,m] w[b,m]
//   gP = gw a rho/(M fref); ga = sum_b gw P rho/(M fref); gb = sum_b gw rho/(M fref);
//   grho = sum_b gw w/rho; gM = -sum_b gw w/M; gfref = -sum_b gw w/fref.
// Every reduction is a fixed-order tree in LDS: results are deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "spx_host.hpp"

namespace spx {

constexpr int KMAX = 16;
// Rows of the squared distance from which each is a wave's: the device holds 8192 waves, and fewer rows leave
// it empty towards the end of long ones.  A wave / a block per row, loss and loss with gradient [us]: 4096
// rows of 1368 10.1 + 12.1 / 8.2 + 10.2, of 160000 1188 + 1802 / 729 + 1165; 6144 rows of 1368 11.0 + 13.4 /
// 11.5 + 13.8, of 160000 1294 + 2024 / 1089 + 1742; 8192 rows of 1368 10.9 + 16.3 / 14.9 + 17.2, of 160000
// 1401 + 2311 / 1448 + 2315.
constexpr int SQDIST_WAVE_ROWS = 8192;

__device__ __forceinline__ float weight(const float* a, const float* bb, const float* P, const float* M,
                                        const float* rho, const float* fref, int b, int k, int K)
{
    return (a[k] * P[(size_t)b * K + k] + bb[k]) * rho[k] / (M[k] * fref[k]);
}

// Forward: a block takes `rows` consecutive power vectors, whose weights it makes once (in LDS), and its
// threads run over `span` (a multiple of 256) of the rows' (b, j), which are contiguous in c.  Bound by HBM (4 K B written per (b, j)):
// with the weights made anew for every (b, j), two divisions each, and K stores of 4 B, 32768 x 342 x 4
// took 68.9 us.  VEC: K == 4 and c aligned to 16 B, one store per (b, j); otherwise the compositions of
// 256 (b, j) go through LDS, so that stores are contiguous (32768 x 342 x 3: 55 us with K stores K apart).
constexpr int FWD_ROWS = 64;        // rows a block at most
// Blocks that rows of many areas are split into, the device's 2048 resident ones twice.  One block a row / 512 / 2048 / 4096
// blocks [us]: 1 x 1e6 x 4 1586, 8.9, 8.9, 8.7; 300 x 40000 x 4 76, 43, 34, 32; 2000 x 40000 x 3 391, 387, 239, 250;
// 64 x 40000 x 9 472, 67, 38, 36.
constexpr int64_t FWD_BLOCKS = 4096;
// ... of four times 256 (b, j) at least: for fewer the weights cost more (1024 x 342 x 4 5.2 us unsplit, 5.9 in thirds).
constexpr int64_t FWD_TILES = 4;
template <int KT, bool VEC>
__global__ void __launch_bounds__(256) k_comp_forward(const float* __restrict__ f, const float* __restrict__ a,
                                                      const float* __restrict__ bb, const float* __restrict__ P,
                                                      const float* __restrict__ M, const float* __restrict__ rho,
                                                      const float* __restrict__ fref, float* __restrict__ c, int B,
                                                      int J, int Kr, int rows, int64_t span)
{
    constexpr int KM = KT > 0 ? KT : KMAX;      // KT: elements known when compiled (0: any number)
    const int K = KT > 0 ? KT : Kr;
    __shared__ float w[FWD_ROWS * KMAX];
    __shared__ __align__(16) float tile[VEC ? 4 : KT > 0 ? 512 * KT : 256 * KMAX];
    const int b0 = blockIdx.x * rows, n_rows = B - b0 < rows ? B - b0 : rows;
    for (int i = threadIdx.x; i < n_rows * K; i += 256) w[i] = weight(a, bb, P, M, rho, fref, b0 + i / K, i % K, K);
    __syncthreads();
    float* cb = c + (size_t)b0 * J * K;
    const uint32_t dr = 256 / J, dj = 256 - dr * J;     // (unsigned: j + dj may pass 2^31)
    const int64_t first = blockIdx.y * span, total = (int64_t)n_rows * J, end = first + span < total ? first + span : total;
    int r = first == 0 ? (int)threadIdx.x / J : (int)((first + threadIdx.x) / J);
    uint32_t j = (uint32_t)(first + threadIdx.x - (int64_t)r * J);
    for (int64_t i0 = first; i0 < end; i0 += 256) {
        if (VEC) {
            if (r < n_rows) {
                const float* wr = w + r * 4;
                float y[4], S = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    y[k] = wr[k] * f[(size_t)k * J + j];
                    S += y[k];
                }
                const float inv = 100.f / S;
                ((float4*)cb)[i0 + threadIdx.x] = make_float4(y[0] * inv, y[1] * inv, y[2] * inv, y[3] * inv);
            }
        } else {
            // two tiles in turn: one barrier each
            float* tl = tile + (KT > 0 && ((i0 >> 8) & 1) ? 256 * KT : 0);
            if (r < n_rows) {
                const float* wr = w + r * K;
                float y[KM], S = 0.f;
#pragma unroll
                for (int k = 0; k < KM; ++k) {
                    if (k < K) {
                        y[k] = wr[k] * f[(size_t)k * J + j];
                        S += y[k];
                    }
                }
                const float inv = 100.f / S;
#pragma unroll
                for (int k = 0; k < KM; ++k)
                    if (k < K) tl[threadIdx.x * K + k] = y[k] * inv;
            }
            __syncthreads();
            const int64_t left = end - i0;
            const int n = (int)(left < 256 ? left : 256) * K;
            float* out = cb + i0 * K;
            if (((uintptr_t)out & 15) == 0) {
                for (int i = threadIdx.x; i < n / 4; i += 256) ((float4*)out)[i] = ((const float4*)tl)[i];
                for (int i = (n & ~3) + threadIdx.x; i < n; i += 256) out[i] = tl[i];
            } else {
                for (int i = threadIdx.x; i < n; i += 256) out[i] = tl[i];
            }
            if (KT == 0) __syncthreads();
        }
        r += dr;
        j += dj;
        if (j >= (uint32_t)J) {
            j -= J;
            ++r;
        }
    }
}

// gy for one (b, j): returns S and fills gy[k]
__device__ __forceinline__ void comp_gy(const float* f, const float* a, const float* bb, const float* P,
                                        const float* M, const float* rho, const float* fref, const float* gc, int b,
                                        int j, int J, int K, float* w, float* gy)
{
    float y[KMAX];
    float S = 0.f;
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        if (k < K) {
            w[k] = weight(a, bb, P, M, rho, fref, b, k, K);
            y[k] = w[k] * f[(size_t)k * J + j];
            S += y[k];
        }
    }
    const float* g = gc + ((size_t)b * J + j) * K;
    float dotgc = 0.f;
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        if (k < K) dotgc += g[k] * (100.f * y[k] / S);
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        if (k < K) gy[k] = (100.f * g[k] - dotgc) / S;
}

template <int NT> __device__ __forceinline__ float block_sum(float v, float* sh)
{
    sh[threadIdx.x] = v;
    __syncthreads();
#pragma unroll
    for (int s = NT / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    const float r = sh[0];
    __syncthreads();
    return r;
}

// One block per batch row b: gw[b, m] = sum_j gy[b,j,m] f[m,j], written to gP (scratch).
template <int NT>
__global__ void __launch_bounds__(NT) k_comp_bw_w(const float* f, const float* a, const float* bb, const float* P,
                                                  const float* M, const float* rho, const float* fref,
                                                  const float* gc, float* gw_out, int B, int J, int K)
{
    __shared__ float sh[NT];
    const int b = blockIdx.x;
    float part[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) part[k] = 0.f;
    for (int j = threadIdx.x; j < J; j += NT) {
        float w[KMAX], gy[KMAX];
        comp_gy(f, a, bb, P, M, rho, fref, gc, b, j, J, K, w, gy);
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
            if (k < K) part[k] += gy[k] * f[(size_t)k * J + j];
    }
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        if (k < K) {   // uniform across the block
            const float s = block_sum<NT>(part[k], sh);
            if (threadIdx.x == 0) gw_out[(size_t)b * K + k] = s;
        }
    }
}

// One block per area j: gf[m, j] = sum_b gy[b,j,m] w[b,m].
template <int NT>
__global__ void __launch_bounds__(NT) k_comp_bw_f(const float* f, const float* a, const float* bb, const float* P,
                                                  const float* M, const float* rho, const float* fref,
                                                  const float* gc, float* gf, int B, int J, int K)
{
    __shared__ float sh[NT];
    const int j = blockIdx.x;
    float part[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) part[k] = 0.f;
    for (int b = threadIdx.x; b < B; b += NT) {
        float w[KMAX], gy[KMAX];
        comp_gy(f, a, bb, P, M, rho, fref, gc, b, j, J, K, w, gy);
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
            if (k < K) part[k] += gy[k] * w[k];
    }
#pragma unroll
    for (int k = 0; k < KMAX; ++k) {
        if (k < K) {   // uniform across the block
            const float s = block_sum<NT>(part[k], sh);
            if (threadIdx.x == 0) gf[(size_t)k * J + j] = s;
        }
    }
}

// One block per element m: reductions over b of gw (held in gP), then gP in place.
template <int NT>
__global__ void __launch_bounds__(NT) k_comp_bw_params(const float* a, const float* bb, const float* P,
                                                       const float* M, const float* rho, const float* fref,
                                                       float* gP, float* ga, float* gb, float* gM, float* grho,
                                                       float* gfref, int B, int K)
{
    __shared__ float sh[NT];
    const int m = blockIdx.x;
    const float q = rho[m] / (M[m] * fref[m]);
    float sa = 0.f, sb = 0.f, sw = 0.f;
    for (int b = threadIdx.x; b < B; b += NT) {
        const float gw = gP[(size_t)b * K + m];
        const float Pm = P[(size_t)b * K + m];
        const float w = (a[m] * Pm + bb[m]) * q;
        sa += gw * Pm;
        sb += gw;
        sw += gw * w;
    }
    const float Sa = block_sum<NT>(sa, sh);
    const float Sb = block_sum<NT>(sb, sh);
    const float Sw = block_sum<NT>(sw, sh);
    if (threadIdx.x == 0) {
        ga[m] = Sa * q;
        gb[m] = Sb * q;
        grho[m] = Sw / rho[m];
        gM[m] = -Sw / M[m];
        gfref[m] = -Sw / fref[m];
    }
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += NT) gP[(size_t)b * K + m] *= a[m] * q;
}

// A wave (WPR = 1) or a block (WPR = 4) per row.  The sum is that of 256 strided partial sums added in a
// tree: a wave holds partials l, l + 64, l + 128 and l + 192 in lane l and needs neither LDS nor
// barrier; a block shares them once.  Bound by HBM (32768 rows of 1368: 39 us for the loss, 75 with
// the gradient; a block per row with nine barriers took 52 and 74), in small batches by latency.
template <int WPR>
__global__ void __launch_bounds__(256) k_sqdist(const float* __restrict__ c, const float* __restrict__ ct, int Bt,
                                                const float* __restrict__ gloss, float* __restrict__ loss,
                                                float* __restrict__ gc, int B, int J, int K)
{
    constexpr int Q = 4 / WPR;              // partials of a lane
    __shared__ float sh[WPR == 4 ? 256 : 1];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int b = WPR == 1 ? blockIdx.x * 4 + wv : blockIdx.x;
    if (b >= B) return;
    const size_t n = (size_t)J * K;
    const float* cb = c + (size_t)b * n;
    const float* tb = ct + (Bt == 1 ? 0 : (size_t)b * n);
    float* gb = gc ? gc + (size_t)b * n : nullptr;
    const float gl = gloss ? gloss[b] : 1.f;
    const size_t first = WPR == 1 ? lane : threadIdx.x;
    float s[Q] = {};
    size_t i0 = 0;
#pragma unroll 2
    for (; i0 + 256 <= n; i0 += 256) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const size_t i = i0 + 64 * q + first;
            const float d = cb[i] - tb[i];
            s[q] += d * d;
            if (gb) gb[i] = 2.f * d * gl;
        }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const size_t i = i0 + 64 * q + first;
        if (i < n) {
            const float d = cb[i] - tb[i];
            s[q] += d * d;
            if (gb) gb[i] = 2.f * d * gl;
        }
    }
    if (!loss) return;
    float v;
    if (WPR == 1) {
        v = (s[0] + s[2 % Q]) + (s[1 % Q] + s[3 % Q]);
    } else {
        sh[threadIdx.x] = s[0];
        __syncthreads();
        if (wv != 0) return;
        v = (sh[lane] + sh[lane + 128]) + (sh[lane + 64] + sh[lane + 192]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if (lane == 0) loss[b] = v;
}

// Backward in one pass over gc, for callers that give scratch: a wave (WPR = 1, J <= 384) or a block
// (WPR = 4, J <= 1536) per row b, its lanes over the areas.  gw[b, k] is summed over the lanes, gP written
// and the parameter sums added at once; gf is kept per lane over the rows the wave takes and its
// partials, one set per block, are added by k_comp_bw_sum in a fixed order (deterministic).  Bound by
// HBM (4 K B read per (b, j)).  The three kernels without scratch read gc twice, one of them 16 B at a
// time and J K 4 B apart: 496 + 300 + 66 us for 32768 x 342 x 4.
constexpr int BW_JM = 6, BW_KMAX = 8;       // areas and elements a lane holds at most
constexpr int BW_BLOCKS = 1024;             // 32768 x 342 x 4: 58 us, 76 at 512, 63 at 2048
template <int K, int WPR>
__global__ void __launch_bounds__(256) k_comp_bw(const float* __restrict__ f, const float* __restrict__ a,
                                                 const float* __restrict__ bb, const float* __restrict__ P,
                                                 const float* __restrict__ M, const float* __restrict__ rho,
                                                 const float* __restrict__ fref, const float* __restrict__ gc,
                                                 float* __restrict__ gP, float* __restrict__ part, int B, int J, int vec)
{
    constexpr int JS = 64 * WPR, RPB = 4 / WPR;     // lanes of a row, rows of a block at a time
    __shared__ float sh[BW_JM * JS * K];
    __shared__ float sw4[2][4][K];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int jt = WPR == 1 ? lane : threadIdx.x;
    float fr[BW_JM][K], acc[BW_JM][K];
#pragma unroll
    for (int m = 0; m < BW_JM; ++m) {
        const int j = jt + m * JS;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            fr[m][k] = j < J ? f[(size_t)k * J + j] : 1.f;
            acc[m][k] = 0.f;
        }
    }
    // lane k < K owns element k of the row sums
    const int ko = lane < K ? lane : 0;
    const float q = rho[ko] / (M[ko] * fref[ko]);
    float sa = 0.f, sb = 0.f, sw = 0.f;
    int par = 0;
    for (int b = blockIdx.x * RPB + (WPR == 1 ? wv : 0); b < B; b += gridDim.x * RPB) {
        const float wl = weight(a, bb, P, M, rho, fref, b, ko, K);
        float w[K], part_w[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            w[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wl), k));
            part_w[k] = 0.f;
        }
        const float* gb = gc + (size_t)b * J * K;
#pragma unroll
        for (int m = 0; m < BW_JM; ++m) {
            if (m * JS >= J) break;
            const int j = jt + m * JS;
            if (j < J) {
                float g[K];
                if (K == 4 && vec) {
                    const float4 v = ((const float4*)gb)[j];
                    const float t[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int k = 0; k < K; ++k) g[k] = t[k & 3];
                } else {
#pragma unroll
                    for (int k = 0; k < K; ++k) g[k] = gb[(size_t)j * K + k];
                }
                float y[K], S = 0.f, dotgc = 0.f;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    y[k] = w[k] * fr[m][k];
                    S += y[k];
                }
                const float inv = 1.f / S;          // g times a fraction: no product beyond the range of its factors
#pragma unroll
                for (int k = 0; k < K; ++k) dotgc += g[k] * (y[k] * inv);
                dotgc *= 100.f;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const float gyk = (100.f * g[k] - dotgc) / S;
                    part_w[k] += gyk * fr[m][k];
                    acc[m][k] += gyk * w[k];
                }
            }
        }
        float gw = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float v = part_w[k];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
            if (lane == k) gw = v;
        }
        if (WPR == 4) {
            // alternating buffers: one barrier a row
            if (lane < K) sw4[par][wv][lane] = gw;
            __syncthreads();
            gw = (sw4[par][0][ko] + sw4[par][1][ko]) + (sw4[par][2][ko] + sw4[par][3][ko]);
            par ^= 1;
        }
        if (lane < K && (WPR == 1 || wv == 0)) {
            const float Pm = P[(size_t)b * K + lane];
            gP[(size_t)b * K + lane] = gw * (a[lane] * q);
            sa += gw * Pm;
            sb += gw;
            sw += gw * wl;
        }
    }
    // the block's partials: the waves' gf sets added one after the other (WPR = 1), then the row sums
    float* out = part + (size_t)blockIdx.x * (K * J + 3 * K);
    for (int turn = 0; turn < RPB; ++turn) {
        __syncthreads();
        if (WPR == 4 || wv == turn) {
#pragma unroll
            for (int m = 0; m < BW_JM; ++m)
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    float* d = &sh[(k * BW_JM + m) * JS + jt];
                    *d = turn == 0 ? acc[m][k] : *d + acc[m][k];
                }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < K * J; i += 256) {
        const int k = i / J, j = i - k * J;
        out[i] = sh[k * BW_JM * JS + j];
    }
    __syncthreads();
    if (lane < K) {
        sh[(0 * 4 + wv) * K + lane] = sa;
        sh[(1 * 4 + wv) * K + lane] = sb;
        sh[(2 * 4 + wv) * K + lane] = sw;
    }
    __syncthreads();
    if (threadIdx.x < 3 * K) {
        const int t = threadIdx.x / K, k = threadIdx.x - t * K;
        float v = 0.f;
        for (int u = 0; u < (WPR == 1 ? 4 : 1); ++u) v += sh[(t * 4 + u) * K + k];
        out[K * J + threadIdx.x] = v;
    }
}

// Sums of the blocks' partials: 64 outputs a block, its 16 waves each a strided sixteenth of the sets.
__global__ void __launch_bounds__(1024) k_comp_bw_sum(const float* __restrict__ part, int n_part,
                                                      const float* __restrict__ M, const float* __restrict__ rho,
                                                      const float* __restrict__ fref, float* __restrict__ gf,
                                                      float* __restrict__ ga, float* __restrict__ gb,
                                                      float* __restrict__ gM, float* __restrict__ grho,
                                                      float* __restrict__ gfref, int J, int K)
{
    __shared__ float sh[16][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, n = K * J + 3 * K, o = blockIdx.x * 64 + lane;
    float v = 0.f;
    if (o < n) {
#pragma unroll 8
        for (int p = wv; p < n_part; p += 16) v += part[(size_t)p * n + o];
    }
    sh[wv][lane] = v;
    __syncthreads();
    for (int h = 8; h > 0; h >>= 1) {
        if (wv < h) sh[wv][lane] += sh[wv + h][lane];
        __syncthreads();
    }
    if (wv != 0 || o >= n) return;
    v = sh[0][lane];
    if (o < K * J) {
        gf[o] = v;
        return;
    }
    const int t = (o - K * J) / K, k = (o - K * J) - t * K;
    const float q = rho[k] / (M[k] * fref[k]);
    if (t == 0) ga[k] = v * q;
    if (t == 1) gb[k] = v * q;
    if (t == 2) {
        grho[k] = v / rho[k];
        gM[k] = -v / M[k];
        gfref[k] = -v / fref[k];
    }
}

// Blocks of the one-pass backward: a row a wave (J > 384: a block), then more of them each above BW_BLOCKS blocks.
static int bw_blocks(int B, int J)
{
    const int rpb = J <= 64 * BW_JM ? 4 : 1;
    const int64_t all = ((int64_t)B + rpb - 1) / rpb;
    return (int)(all < BW_BLOCKS ? all : BW_BLOCKS);
}
static bool bw_fits(int J, int K) { return K <= BW_KMAX && J <= 4 * 64 * BW_JM; }

// Area average: G lanes per square (profile, area) over the bins it meets, row by row, the lanes' sums added in a
// tree.  Few squares of many bins are bound by the latency of one square's bins, many small ones by the
// instructions spent per square, which G lanes all spend: G is 1, 8 or 64 by the bins of a square (area_lanes).
template <int G>
__global__ void __launch_bounds__(256) k_area_gather(const double* __restrict__ prof, int64_t n, int nu, int nv,
                                                     double half_u, double half_v, const double* __restrict__ cen,
                                                     int n_areas, double hw, double* __restrict__ out)
{
    const uint32_t g = threadIdx.x & (G - 1);
    const double du = 2.0 * half_u / nu, dv = 2.0 * half_v / nv;
    for (int64_t idx = (int64_t)blockIdx.x * (256 / G) + threadIdx.x / G; idx < n; idx += (int64_t)gridDim.x * (256 / G)) {
        const int64_t p = idx / n_areas;
        const int ai = (int)(idx - p * n_areas);
        const double cu = cen[2 * ai], cv = cen[2 * ai + 1];
        int iu0 = (int)floor((cu - hw + half_u) / du), iu1 = (int)floor((cu + hw + half_u) / du);
        int iv0 = (int)floor((cv - hw + half_v) / dv), iv1 = (int)floor((cv + hw + half_v) / dv);
        iu0 = iu0 < 0 ? 0 : iu0;
        iv0 = iv0 < 0 ? 0 : iv0;
        iu1 = iu1 > nu - 1 ? nu - 1 : iu1;
        iv1 = iv1 > nv - 1 ? nv - 1 : iv1;
        const double* pr = prof + (size_t)p * nu * nv;
        double sw = 0.0, s = 0.0;
        // (a square beyond the grid, however far, has its first row past the last; unsigned: no sum below wraps)
        if (iu0 <= iu1 && iv0 <= iv1) {
            const uint32_t w = (uint32_t)(iu1 - iu0) + 1, dr = G / w, dc = G - dr * w;
            uint32_t iv = (uint32_t)iv0 + g / w, iu = (uint32_t)iu0 + g % w;
            while (iv <= (uint32_t)iv1) {
                const double v0 = -half_v + iv * dv, u0 = -half_u + iu * du;
                const double ov = fmin(v0 + dv, cv + hw) - fmax(v0, cv - hw);
                const double ou = fmin(u0 + du, cu + hw) - fmax(u0, cu - hw);
                if (ov > 0.0 && ou > 0.0) {
                    const double wt = ou * ov;
                    sw += wt;
                    s += wt * pr[(size_t)iv * nu + iu];
                }
                iv += dr;
                iu += dc;
                if (iu > (uint32_t)iu1) {
                    iu -= w;
                    ++iv;
                }
            }
        }
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) {
            sw += __shfl_xor(sw, o);
            s += __shfl_xor(s, o);
        }
        if (g == 0) out[idx] = sw > 0.0 ? s / sw : 0.0;
    }
}

}  // namespace spx

using namespace spx;

extern "C" int spx_comp_forward(const float* d_f, const float* d_a, const float* d_b, const float* d_P,
                                const float* d_M, const float* d_rho, const float* d_fref, float* d_c, int32_t B,
                                int32_t J, int32_t K, void* stream)
{
    if (B <= 0 || J <= 0 || K <= 0 || K > KMAX) {
        set_error("spx_comp_forward: need B, J > 0 and 0 < K <= 16");
        return SPX_EINVAL;
    }
    if (!d_f || !d_a || !d_b || !d_P || !d_M || !d_rho || !d_fref || !d_c) {
        set_error("spx_comp_forward: null pointer");
        return SPX_EINVAL;
    }
    // up to eight rows a block while every CU keeps two blocks; with few areas enough rows for its threads
    int rows = B >= 8 * 512 ? 8 : B >= 1024 ? B / 512 : 1;
    if ((int64_t)rows * J < 256) rows = std::min(FWD_ROWS, 255 / J + 1);
    const bool vec = K == 4 && ((uintptr_t)d_c & 15) == 0;
    using Kernel = void (*)(const float*, const float*, const float*, const float*, const float*, const float*,
                            const float*, float*, int, int, int, int, int64_t);
    static const Kernel by_k[] = {k_comp_forward<0, false>, k_comp_forward<1, false>, k_comp_forward<2, false>,
                                  k_comp_forward<3, false>, k_comp_forward<4, false>, k_comp_forward<5, false>,
                                  k_comp_forward<6, false>, k_comp_forward<7, false>, k_comp_forward<8, false>};
    const Kernel kern = vec ? k_comp_forward<4, true> : by_k[K <= 8 ? K : 0];
    for (int64_t b0 = 0; b0 < B; b0 += GRID_MAX * rows) {
        const int n = (int)std::min<int64_t>(B - b0, GRID_MAX * rows);
        const int64_t groups = (n + rows - 1) / rows, tiles = ((int64_t)rows * J + 255) / 256;
        const int64_t parts = std::min((tiles + FWD_TILES - 1) / FWD_TILES, (FWD_BLOCKS + groups - 1) / groups);
        const int64_t span = (tiles + parts - 1) / parts * 256;
        hipLaunchKernelGGL(kern, dim3((unsigned)groups, (unsigned)parts), dim3(256), 0, (hipStream_t)stream, d_f, d_a,
                           d_b, d_P + b0 * K, d_M, d_rho, d_fref, d_c + b0 * J * K, n, J, K, rows, span);
        SPX_HIP(hipGetLastError());
    }
    return SPX_OK;
}

static int check_backward(const float* const* ptrs, int n, int32_t B, int32_t J, int32_t K)
{
    if (B <= 0 || J <= 0 || K <= 0 || K > KMAX) {
        set_error("spx_comp_backward: need B, J > 0 and 0 < K <= 16");
        return SPX_EINVAL;
    }
    for (int i = 0; i < n; ++i)
        if (!ptrs[i]) {
            set_error("spx_comp_backward: null pointer");
            return SPX_EINVAL;
        }
    return SPX_OK;
}

extern "C" uint64_t spx_comp_backward_scratch(int32_t B, int32_t J, int32_t K)
{
    if (B <= 0 || J <= 0 || K <= 0 || !bw_fits(J, K)) return 0;
    return (uint64_t)bw_blocks(B, J) * (uint64_t)(K * J + 3 * K);
}

extern "C" int spx_comp_backward_with(const float* d_f, const float* d_a, const float* d_b, const float* d_P,
                                      const float* d_M, const float* d_rho, const float* d_fref, const float* d_gc,
                                      float* d_gf, float* d_ga, float* d_gb, float* d_gP, float* d_gM, float* d_grho,
                                      float* d_gfref, float* d_scratch, uint64_t n_scratch, int32_t B, int32_t J,
                                      int32_t K, void* stream)
{
    const float* ptrs[] = {d_f,  d_a,  d_b,  d_P,  d_M,    d_rho,   d_fref,   d_gc,
                           d_gf, d_ga, d_gb, d_gP, d_gM,   d_grho,  d_gfref,  d_scratch};
    SPX_TRY(check_backward(ptrs, 16, B, J, K));
    const uint64_t need = spx_comp_backward_scratch(B, J, K);
    if (need == 0 || n_scratch < need) {
        set_error("spx_comp_backward_with: scratch smaller than spx_comp_backward_scratch asks for");
        return SPX_EINVAL;
    }
    hipStream_t st = (hipStream_t)stream;
    const int blocks = bw_blocks(B, J), vec = K == 4 && ((uintptr_t)d_gc & 15) == 0 ? 1 : 0;
    using Kernel = void (*)(const float*, const float*, const float*, const float*, const float*, const float*,
                            const float*, const float*, float*, float*, int, int, int);
    static const Kernel wave[] = {k_comp_bw<1, 1>, k_comp_bw<2, 1>, k_comp_bw<3, 1>, k_comp_bw<4, 1>,
                                  k_comp_bw<5, 1>, k_comp_bw<6, 1>, k_comp_bw<7, 1>, k_comp_bw<8, 1>};
    static const Kernel block[] = {k_comp_bw<1, 4>, k_comp_bw<2, 4>, k_comp_bw<3, 4>, k_comp_bw<4, 4>,
                                   k_comp_bw<5, 4>, k_comp_bw<6, 4>, k_comp_bw<7, 4>, k_comp_bw<8, 4>};
    const Kernel kern = J <= 64 * BW_JM ? wave[K - 1] : block[K - 1];
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, st, d_f, d_a, d_b, d_P, d_M, d_rho, d_fref, d_gc, d_gP,
                       d_scratch, B, J, vec);
    SPX_HIP(hipGetLastError());
    const int n = K * J + 3 * K;
    hipLaunchKernelGGL(k_comp_bw_sum, dim3((n + 63) / 64), dim3(1024), 0, st, d_scratch, blocks, d_M, d_rho, d_fref, d_gf,
                       d_ga, d_gb, d_gM, d_grho, d_gfref, J, K);
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

extern "C" int spx_comp_backward(const float* d_f, const float* d_a, const float* d_b, const float* d_P,
                                 const float* d_M, const float* d_rho, const float* d_fref, const float* d_gc,
                                 float* d_gf, float* d_ga, float* d_gb, float* d_gP, float* d_gM, float* d_grho,
                                 float* d_gfref, int32_t B, int32_t J, int32_t K, void* stream)
{
    const float* ptrs[] = {d_f,  d_a,  d_b,  d_P,  d_M,   d_rho,  d_fref, d_gc,
                           d_gf, d_ga, d_gb, d_gP, d_gM,  d_grho, d_gfref};
    SPX_TRY(check_backward(ptrs, 15, B, J, K));
    hipStream_t st = (hipStream_t)stream;
    for (int64_t b0 = 0; b0 < B; b0 += GRID_MAX) {
        const int n = (int)std::min<int64_t>(B - b0, GRID_MAX);
        hipLaunchKernelGGL(k_comp_bw_w<256>, dim3((unsigned)n), dim3(256), 0, st, d_f, d_a, d_b, d_P + b0 * K, d_M, d_rho,
                           d_fref, d_gc + b0 * J * K, d_gP + b0 * K, n, J, K);
    }
    hipLaunchKernelGGL(k_comp_bw_f<256>, dim3(J), dim3(256), 0, st, d_f, d_a, d_b, d_P, d_M, d_rho, d_fref, d_gc,
                       d_gf, B, J, K);
    hipLaunchKernelGGL(k_comp_bw_params<256>, dim3(K), dim3(256), 0, st, d_a, d_b, d_P, d_M, d_rho, d_fref, d_gP,
                       d_ga, d_gb, d_gM, d_grho, d_gfref, B, K);
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

extern "C" int spx_comp_sqdist(const float* d_c, const float* d_ct, int32_t B_t, const float* d_gloss, float* d_loss,
                               float* d_gc, int32_t B, int32_t J, int32_t K, void* stream)
{
    if (B <= 0 || J <= 0 || K <= 0 || (B_t != 1 && B_t != B) || !d_c || !d_ct || (!d_loss && !d_gc)) {
        set_error("spx_comp_sqdist: invalid arguments");
        return SPX_EINVAL;
    }
    if (B < SQDIST_WAVE_ROWS)
        hipLaunchKernelGGL(k_sqdist<4>, dim3((unsigned)B), dim3(256), 0, (hipStream_t)stream, d_c, d_ct, B_t, d_gloss,
                           d_loss, d_gc, B, J, K);
    else
        for (int64_t b0 = 0; b0 < B; b0 += 4 * GRID_MAX) {
            const int n = (int)std::min<int64_t>(B - b0, 4 * GRID_MAX);
            const int64_t o = b0 * J * K;
            hipLaunchKernelGGL(k_sqdist<1>, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, (hipStream_t)stream, d_c + o,
                               B_t == 1 ? d_ct : d_ct + o, B_t, d_gloss ? d_gloss + b0 : nullptr,
                               d_loss ? d_loss + b0 : nullptr, d_gc ? d_gc + o : nullptr, n, J, K);
        }
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}

// Lanes of a square, by the bins it meets at most.  At 1, 8, 64 lanes [us]: 4e6 squares of 2 bins 50, 218, 1840;
// 6.8e5 of 11 37, 49, 319; 8208 of 30 11.2, 8.8, 8.5; 6.8e5 of 100 908, 174, 376; 8208 of 100 26.2, 8.7, 8.8; 6.8e5
// of 360 (bound 400) -, 443, 528, 8208 of them -, 21, 11; 8208 of 14641 4298, 733, 160.
static int area_lanes(int nu, int nv, double half_u, double half_v, double half_width)
{
    const double bins = std::min<double>(nu, half_width / half_u * nu + 2.0) *
                        std::min<double>(nv, half_width / half_v * nv + 2.0);
    return bins <= 20.0 ? 1 : bins <= 256.0 ? 8 : 64;
}

extern "C" int spx_area_gather(const double* d_profiles, int32_t n_prof, int32_t nu, int32_t nv, double half_u,
                               double half_v, const double* d_centres, int32_t n_areas, double half_width,
                               double* d_out, void* stream)
{
    if (!d_profiles || !d_centres || !d_out || n_prof <= 0 || nu <= 0 || nv <= 0 || n_areas <= 0 ||
        !(half_u > 0) || !(half_v > 0) || !(half_width > 0)) {
        set_error("spx_area_gather: invalid arguments");
        return SPX_EINVAL;
    }
    const int64_t n = (int64_t)n_prof * n_areas;
    const int G = area_lanes(nu, nv, half_u, half_v, half_width);
    const auto kern = G == 1 ? k_area_gather<1> : G == 8 ? k_area_gather<8> : k_area_gather<64>;
    const int64_t blocks = std::min<int64_t>((n + 256 / G - 1) / (256 / G), GRID_MAX);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, d_profiles, n, nu, nv, half_u,
                       half_v, d_centres, n_areas, half_width, d_out);
    SPX_HIP(hipGetLastError());
    return SPX_OK;
}
