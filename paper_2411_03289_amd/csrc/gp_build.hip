// Once-per-GP-update build of the residual GPs in FP64 on the GPU
// (Rasmussen & Williams Alg. 2.1 with the explicit inverse factor), both outputs
// side by side in every launch:
//   A = K(Z, Z) + sn^2 I         SE-ARD covariance (Sec. III-A, Sec. V-A)
//   L = chol(A), W = L^-1        right-looking over block columns of 32, one launch each
//   alpha = W^T (W y) = A^-1 y
// and the packing of W, alpha and the scaled inputs into the FP32 / BF16
// layouts the rollout streams.  Padding rows/columns (M <= i < Mpad) carry
// the identity in A and are zeroed when packing.
//
// Every element is one chain of fused multiply-adds in ascending order of the
// summed index (the FP64 matrix cores add a product's four terms in that order, each
// rounded), followed by the division by the pivot.
#include <cmath>

#include "device_common.hpp"
#include "kernels.hpp"

namespace gpmppi {

constexpr int NB = 32;   // tile edge
constexpr int kBlk = NB * NB;
typedef double v4d __attribute__((ext_vector_type(4)));

// The factorization's array: 32x32 blocks, block (b, a) at (b nb + a) 1024.
//   b >= a  A's block of rows b and columns a, element [column][row]
//   b < a   block (a, b) of what is left of L W = I, element [row][column]
// so that one product with the row index from a's vectors and the column index from
// b's updates either kind.
__global__ void kmat_kernel(const double *Zs, int M, int Mpad, GpKernelParams kp, double *As) {
    const int o = blockIdx.z;
    const int j = blockIdx.x * 16 + threadIdx.y;
    const int i = blockIdx.y * 16 + threadIdx.x;
    if (i >= Mpad || j >= Mpad || (i / NB) < (j / NB)) return;
    const double *Z = Zs + (size_t)o * 4 * M;
    const double i0 = kp.i[o][0], i1 = kp.i[o][1], i2 = kp.i[o][2], i3 = kp.i[o][3];
    double v;
    if (i < M && j < M) {
        const double d0 = Z[4 * i] - Z[4 * j], d1 = Z[4 * i + 1] - Z[4 * j + 1];
        const double d2 = Z[4 * i + 2] - Z[4 * j + 2], d3 = Z[4 * i + 3] - Z[4 * j + 3];
        const double r2 = d0 * d0 * i0 + d1 * d1 * i1 + d2 * d2 * i2 + d3 * d3 * i3;
        v = kp.sf2[o] * exp(-0.5 * r2) + (i == j ? kp.sn2[o] : 0.0);
    } else {
        v = (i == j) ? 1.0 : 0.0;
    }
    double *A = As + (size_t)o * Mpad * Mpad;
    A[((size_t)(i / NB) * (Mpad / NB) + j / NB) * kBlk + (j % NB) * NB + i % NB] = v;
}

__device__ __forceinline__ double readlane64(double x, int lane) {
    uint64_t u;
    __builtin_memcpy(&u, &x, 8);
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    u = lo | (hi << 32);
    __builtin_memcpy(&x, &u, 8);
    return x;
}

// Square root s of a normal d (rounded to nearest) and r close to 1 / s: Newton's step for
// 1 / sqrt(d) coupled with the root (Goldschmidt) from the hardware's estimate, then the root
// corrected by its remainder (Markstein), twice.  The estimate of the reciprocal is a
// by-product, so a pivot costs one chain instead of a square root and a division.
__device__ __forceinline__ void sqrt_rcp(double d, double &s, double &r) {
    const double y = __builtin_amdgcn_rsq(d);
    double g = d * y, h = 0.5 * y;
    double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    e = fma(-h, g, 0.5);
    h = fma(h, e, h);
    g = fma(fma(-g, g, d), h, g);
    s = fma(fma(-g, g, d), h, g);
    r = 2.0 * h;
    r = fma(fma(-s, r, 1.0), r, r);
}

// Solves L x = v for one vector per lane of the upper half wave, L the Cholesky factor of
// the diagonal block whose rows are the vectors of the lower half: both halves take the
// same steps, x_c = v_c / L_cc and v_j -= x_c L_jc for j > c (lower half: x is L's row).
// The quotient is v times the reciprocal, twice corrected by its remainder: the rounded
// quotient.  Returns whether a pivot was not positive.
__device__ __forceinline__ bool panel_solve(double (&v)[NB]) {
    bool bad = false;
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        double d = readlane64(v[c], c);
        if (!(d > 0.0)) {
            bad = true;
            d = 1.0;
        }
        double s, r;
        sqrt_rcp(d, s, r);
        double x = v[c] * r;
        x = fma(fma(-x, s, v[c]), r, x);
        x = fma(fma(-x, s, v[c]), r, x);
        v[c] = x;
#pragma unroll
        for (int j = c + 1; j < NB; ++j) v[j] = fma(-x, readlane64(x, j), v[j]);
    }
    return bad;
}

// Step k of the factorization and of the inverse factor.  The vectors of block m are the
// rows of L_mk (m > k) or the columns of W_km (m <= k): the solutions of panel_solve for
// the block (m, k) (the identity for m = k).  A job of four waves solves two blocks a > k
// and two blocks b, and subtracts the four products from the blocks (b, a); b >= a: the
// trailing part of A, b <= k: what is left of L W = I.  Jobs n_upd ..: four blocks m of
// W's row k, written to W (row-major) and, m < k, to block (k, m) as [column][row], where
// L_km is no longer needed.
//
// Bound by the panel's serial chain (32 pivots of a root, a quotient and a rank-one update),
// so every job repeats the pivot block's factorization instead of waiting for another launch to
// do it: 9 to 18 us a step.  A whole update of both GPs (host calls, packing) went from
// 9.9 ms to 0.77 ms at M = 1024; before, each output's block columns took two launches that
// streamed the columns to the left (58 + 21 us) and one workgroup per column inverted L
// (1.9 ms), alpha took 0.2 ms per product (one uncoalesced lane per row), now 28 us.
__global__ __launch_bounds__(256) void factor_step_kernel(double *As, double *Ws, int nb, int k, int n_row, int n_upd,
                                                          uint32_t *flag) {
    __shared__ double X[4][kBlk];
    const int o = blockIdx.y, lane = threadIdx.x & 63, col = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int Mpad = nb * NB;
    double *A = As + (size_t)o * Mpad * Mpad;
    const int job = blockIdx.x;
    const bool upd = job < n_upd;
    int m, last, a0 = 0, b0 = 0;
    if (upd) {
        int I, J = job;   // column pairs J of every row pair I: the trailing pairs up to I, then those of W
        const int n_col = k / 2 + 1, tri = n_row * (n_row + 1) / 2;
        if (job < tri) {
            I = 0;
            while (J > I) J -= ++I;
            a0 = k + 1 + 2 * J;
            b0 = k + 1 + 2 * I;
        } else {
            I = (job - tri) / n_col;
            a0 = k + 1 + 2 * I;
            b0 = 2 * ((job - tri) % n_col);
        }
        m = w < 2 ? a0 + w : b0 + w - 2;
        last = w < 2 || b0 > k ? nb - 1 : k;
    } else {
        m = 4 * (job - n_upd) + w;
        last = k;
    }
    const bool have = m <= last;
    // this wave's products: blocks (b, a)
    const int a = a0 + (w & 1), b = b0 + (w >> 1);
    const bool prod = upd && a < nb && b <= (b0 > k ? nb - 1 : k) && (b0 <= k || b >= a);
    double *T = A + ((size_t)b * nb + a) * kBlk;
    v4d acc[2][2];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[s][t][r] = prod && b != k ? T[(16 * s + 4 * r + (lane >> 4)) * NB + 16 * t + (lane & 15)] : 0.0;
    if (have) {
        double v[NB];
        const double *src = A + ((size_t)(lane < 32 ? k : m) * nb + k) * kBlk + col;
#pragma unroll
        for (int p = 0; p < NB; ++p) v[p] = src[p * NB];
        if (m == k && lane >= 32) {
#pragma unroll
            for (int p = 0; p < NB; ++p) v[p] = p == col ? 1.0 : 0.0;
        }
        const bool bad = panel_solve(v);
        if (bad && job == 0 && lane == 0) atomicOr(flag, 1u << o);
        if (lane >= 32) {
            if (upd) {
#pragma unroll
                for (int p = 0; p < NB; ++p) X[w][p * NB + col] = v[p];
            } else {
                double *W = Ws + (size_t)o * Mpad * Mpad + (size_t)k * NB * Mpad + m * NB + col;
#pragma unroll
                for (int p = 0; p < NB; ++p) W[(size_t)p * Mpad] = v[p];
                if (m < k) {
                    double2 *C = reinterpret_cast<double2 *>(A + ((size_t)k * nb + m) * kBlk + col * NB);
#pragma unroll
                    for (int p = 0; p < NB / 2; ++p) C[p] = make_double2(v[2 * p], v[2 * p + 1]);
                }
            }
        }
    }
    if (!upd) return;
    __syncthreads();
    if (!prod) return;
    const double *xa = X[w & 1] + (lane >> 4) * NB + (lane & 15), *xb = X[2 + (w >> 1)] + (lane >> 4) * NB + (lane & 15);
#pragma unroll
    for (int p = 0; p < NB; p += 4) {
        const double va[2] = {-xa[p * NB], -xa[p * NB + 16]}, vb[2] = {xb[p * NB], xb[p * NB + 16]};
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                acc[s][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(va[s], vb[t], acc[s][t], 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) T[(16 * s + 4 * r + (lane >> 4)) * NB + 16 * t + (lane & 15)] = acc[s][t][r];
}

// u = W y (a wave per block row, a lane per row; the blocks below the diagonal as
// factor_step_kernel left them in As) and alpha = W^T u (a lane per column).  One chain of
// multiply-adds per entry, the next block's 32 elements loaded beside it.
template <bool TRANS>
__global__ __launch_bounds__(64) void matvec_kernel(const double *As, const double *Ws, int nb, const double *xs,
                                                    size_t x_stride, double *ys, size_t y_stride) {
    __shared__ double xl[32 * NB];
    const int o = blockIdx.y, blk = blockIdx.x, lane = threadIdx.x, r = lane & 31;
    const int Mpad = nb * NB;
    const double *A = As + (size_t)o * Mpad * Mpad, *W = Ws + (size_t)o * Mpad * Mpad;
    const double *x = xs + (size_t)o * x_stride;
    for (int i = lane; i < Mpad; i += 64) xl[i] = x[i];
    const int first = TRANS ? blk : 0, end = TRANS ? nb : blk + 1;
    double cur[NB], nxt[NB];
    auto load = [&](double (&v)[NB], int q) {
        if (TRANS) {
            const double *p = W + (size_t)q * NB * Mpad + blk * NB + r;
#pragma unroll
            for (int c = 0; c < NB; ++c) v[c] = p[(size_t)c * Mpad];
        } else if (q < blk) {
            const double *p = A + ((size_t)blk * nb + q) * kBlk + r;
#pragma unroll
            for (int c = 0; c < NB; ++c) v[c] = p[c * NB];
        } else {
            const double *p = W + (size_t)(blk * NB + r) * Mpad + blk * NB;
#pragma unroll
            for (int c = 0; c < NB; ++c) v[c] = p[c];
        }
    };
    load(cur, first);
    __syncthreads();
    double acc = 0.0;
    for (int q = first; q < end; ++q) {
        if (q + 1 < end) load(nxt, q + 1);
#pragma unroll
        for (int c = 0; c < NB; ++c) acc = fma(cur[c], xl[q * NB + c], acc);
#pragma unroll
        for (int c = 0; c < NB; ++c) cur[c] = nxt[c];
    }
    if (lane < NB) ys[(size_t)o * y_stride + blk * NB + r] = acc;
}

// alpha [n_out outputs] for targets y: u is scratch.
static void launch_alpha(const GpBuildBuffers &b, int Mpad, int n_out, const double *A, const double *W,
                         const double *y, double *alpha, hipStream_t st) {
    const int nb = Mpad / NB;
    hipLaunchKernelGGL(matvec_kernel<false>, dim3(nb, n_out), dim3(64), 0, st, A, W, nb, y, (size_t)Mpad, b.u,
                       (size_t)Mpad);
    hipLaunchKernelGGL(matvec_kernel<true>, dim3(nb, n_out), dim3(64), 0, st, A, W, nb, b.u, (size_t)Mpad, alpha,
                       (size_t)Mpad);
}

hipError_t factor_gps(const GpBuildBuffers &b, int M, int Mpad, const GpKernelParams &kp, hipStream_t st) {
    const int nb = Mpad / NB;
    hipLaunchKernelGGL(kmat_kernel, dim3(Mpad / 16, Mpad / 16, 2), dim3(16, 16), 0, st, b.Z, M, Mpad, kp, b.A);
    for (int k = 0; k < nb; ++k) {
        const int n_row = (nb - k) / 2;   // pairs of trailing blocks
        const int n_upd = n_row * (n_row + 1) / 2 + n_row * (k / 2 + 1);
        hipLaunchKernelGGL(factor_step_kernel, dim3(n_upd + k / 4 + 1, 2), dim3(256), 0, st, b.A, b.W, nb, k, n_row,
                           n_upd, b.flag);
    }
    launch_alpha(b, Mpad, 2, b.A, b.W, b.y, b.alpha, st);
    return hipGetLastError();
}

// alpha = W^T (W y) for another target vector y of output o on the same W (b.u is scratch).
hipError_t alpha_for_targets(const GpBuildBuffers &b, int Mpad, int o, const double *y_d, double *alpha_d,
                             hipStream_t st) {
    const size_t at = (size_t)o * Mpad * Mpad;
    launch_alpha(b, Mpad, 1, b.A + at, b.W + at, y_d, alpha_d, st);
    return hipGetLastError();
}

__global__ void combine_alpha_kernel(const double *alpha_terr, int n_terr, int Mpad, TerrainWeights w,
                                     double sf2, float *alpha32, float *alphas) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= Mpad) return;
    double a = 0.0;
    for (int i = 0; i < n_terr; ++i) a += w.w[i] * alpha_terr[(size_t)i * Mpad + j];
    alpha32[j] = (float)a;
    alphas[j] = (float)(a * sf2 * 0x1p-15);
}

hipError_t combine_alpha(const double *alpha_terr, int n_terr, int Mpad, TerrainWeights w, double sf2,
                         float *alpha32, float *alphas, hipStream_t st) {
    hipLaunchKernelGGL(combine_alpha_kernel, dim3((Mpad + 255) / 256), dim3(256), 0, st, alpha_terr, n_terr, Mpad, w,
                       sf2, alpha32, alphas);
    return hipGetLastError();
}

// Q = W^T W = A^-1 in FP64 for the adjoint's r = Q k, rounded into the matrix-core
// operand order of the FP32 W blocks: block b = t NT + it, float4 [b][q][lane], component
// c holds Q[32t + l%32][32 it + 2(4q+c) + l/32].  Rows/columns beyond M are zero.  A
// workgroup per block on or below the diagonal, a wave per 16x16 quarter; the block is
// stored with its mirror image.
__global__ __launch_bounds__(256) void qmat_kernel(const double *W, int M, int Mpad, float *q32) {
    const int NT = Mpad / NB;
    int t = 0, it = blockIdx.x;
    while (it > t) it -= ++t;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i0 = NB * t + 16 * (w & 1), j0 = NB * it + 16 * (w >> 1);
    const double *p = W + (size_t)(NB * t + (lane >> 4)) * Mpad + (lane & 15);
    v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
    for (int k = NB * t; k < Mpad; k += NB) {
        double va[NB / 4], vb[NB / 4];
#pragma unroll
        for (int i = 0; i < NB / 4; ++i, p += (size_t)4 * Mpad) {
            va[i] = p[i0];
            vb[i] = p[j0];
        }
#pragma unroll
        for (int i = 0; i < NB / 4; ++i) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(va[i], vb[i], acc, 0, 0, 0);
    }
    auto put = [&](int i, int j, float v) {
        const int c = j & 31;
        q32[((size_t)((i >> 5) * NT + (j >> 5)) * 256 + (c >> 3) * 64 + (i & 31) + 32 * (c & 1)) * 4 + ((c >> 1) & 3)] = v;
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = i0 + 4 * r + (lane >> 4), j = j0 + (lane & 15);
        const float v = i < M && j < M ? (float)acc[r] : 0.0f;
        put(i, j, v);
        if (t != it) put(j, i, v);
    }
}

hipError_t pack_q(const GpBuildBuffers &b, int M, int Mpad, int o, float4 *q32, hipStream_t st) {
    const int NT = Mpad / NB;
    hipLaunchKernelGGL(qmat_kernel, dim3(NT * (NT + 1) / 2), dim3(256), 0, st, b.W + (size_t)o * Mpad * Mpad, M, Mpad,
                       reinterpret_cast<float *>(q32));
    return hipGetLastError();
}

// Terrain means at n queries: out[q][i][o] = k_o(q)^T alpha_{o,i}; one
// workgroup per query, threads over training points, FP64 accumulation of the
// FP32 kernel values.  alpha_terr is [2][n_terr][Mpad] FP64.
__global__ __launch_bounds__(256) void terrain_means_kernel(const float *q, int n, const float *zs, const double *alpha_terr,
                                                            int n_terr, int Mpad, float s00, float s01, float s02,
                                                            float s03, float s10, float s11, float s12, float s13,
                                                            float c20, float c21, float *out) {
    __shared__ double red[8][4];
    const int qi = blockIdx.x, tid = threadIdx.x;
    const float4 qq = reinterpret_cast<const float4 *>(q)[qi];
    for (int o = 0; o < 2; ++o) {
        const float sc[4] = {o ? s10 : s00, o ? s11 : s01, o ? s12 : s02, o ? s13 : s03};
        const float qs[4] = {qq.x * sc[0], qq.y * sc[1], qq.z * sc[2], qq.w * sc[3]};
        const float c2 = o ? c21 : c20;
        double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int j = tid; j < Mpad; j += 256) {
            const float4 z = reinterpret_cast<const float4 *>(zs)[(size_t)o * Mpad + j];
            const float d0 = qs[0] - z.x, d1 = qs[1] - z.y, d2 = qs[2] - z.z, d3 = qs[3] - z.w;
            const double kv = (double)exp2f(c2 - (d0 * d0 + d1 * d1 + d2 * d2 + d3 * d3));
            for (int i = 0; i < n_terr; ++i) acc[i] += kv * alpha_terr[((size_t)o * n_terr + i) * Mpad + j];
        }
        for (int i = 0; i < n_terr; ++i) {
            double v = acc[i];
            for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
            if ((tid & 63) == 0) red[i][tid >> 6] = v;
        }
        __syncthreads();
        if (tid < n_terr) {
            const double v = red[tid][0] + red[tid][1] + red[tid][2] + red[tid][3];
            out[((size_t)qi * n_terr + tid) * 2 + o] = (float)v;
        }
        __syncthreads();
    }
}

hipError_t launch_terrain_means(const float *q, int n, const GpDev &g, const double *alpha_terr, int n_terr,
                                float *out, hipStream_t st) {
    hipLaunchKernelGGL(terrain_means_kernel, dim3(n), dim3(256), 0, st, q, n, g.zs, alpha_terr, n_terr, g.Mpad,
                       g.scale[0][0], g.scale[0][1], g.scale[0][2], g.scale[0][3], g.scale[1][0], g.scale[1][1],
                       g.scale[1][2], g.scale[1][3], g.c2[0], g.c2[1], out);
    return hipGetLastError();
}

// Scale of each row of W for the FP16 splits: with max_j |sf W_ij| in [2^(e-1), 2^e) the
// row is packed as sf W 2^(14 - e), and wrs = 2^(e - 29) turns its product with the
// kernel values scaled by 2^15 / sf^2 back into (W k)_i / sf.  One wave per row.
__global__ void row_scale_kernel(const double *W, int M, int Mpad, double sf, float *wrs) {
    const int i = blockIdx.x;
    double m = 0.0;
    if (i < M)
        for (int j = threadIdx.x; j <= i; j += 64) m = fmax(m, fabs(W[(size_t)i * Mpad + j]));
    for (int d = 32; d >= 1; d >>= 1) m = fmax(m, __shfl_xor(m, d, 64));
    int e = 0;
    if (m > 0.0) (void)frexp(sf * m, &e);
    if (threadIdx.x == 0) wrs[i] = ldexpf(1.0f, e - 29);
}

// Packs the W blocks in the rollout's pair-major order: block index
// b = 2 (u (u + 1) + it) + side holds rows of tile t = 2u + side and columns of
// block column it (it <= 2u + 1); entries above the diagonal or beyond M are 0.
__global__ void pack_w_kernel(const double *W, int M, int Mpad, double sf, const float *wrs, float4 *w32, uint4 *wbh,
                              uint4 *wbl, uint4 *wfh, uint4 *wfl) {
    const int blk = blockIdx.x, lane = threadIdx.x;
    const int side = blk & 1, half_idx = blk >> 1;   // half_idx = u (u + 1) + it
    int u = 0;
    while ((u + 1) * (u + 2) <= half_idx) ++u;
    const int it = half_idx - u * (u + 1);
    const int t = 2 * u + side;
    const int i = 32 * t + (lane & 31);
    const int half = lane >> 5;
    auto wval = [&](int j) -> float {
        return (i < M && j < M && j <= i) ? (float)W[(size_t)i * Mpad + j] : 0.0f;
    };
    for (int q = 0; q < 4; ++q) {
        float4 v;
        v.x = wval(32 * it + 2 * (4 * q + 0) + half);
        v.y = wval(32 * it + 2 * (4 * q + 1) + half);
        v.z = wval(32 * it + 2 * (4 * q + 2) + half);
        v.w = wval(32 * it + 2 * (4 * q + 3) + half);
        w32[(size_t)blk * 256 + q * 64 + lane] = v;
    }
    for (int h = 0; h < 2; ++h) {
        uint16_t hi[8], lo[8];
        for (int e = 0; e < 8; ++e) {
            const float x = wval(32 * it + 16 * h + 8 * half + e);
            hi[e] = bf16_rne(x);
            lo[e] = bf16_rne(x - bf16_to_f32(hi[e]));
        }
        uint4 H, Lo;
        H.x = hi[0] | ((uint32_t)hi[1] << 16);
        H.y = hi[2] | ((uint32_t)hi[3] << 16);
        H.z = hi[4] | ((uint32_t)hi[5] << 16);
        H.w = hi[6] | ((uint32_t)hi[7] << 16);
        Lo.x = lo[0] | ((uint32_t)lo[1] << 16);
        Lo.y = lo[2] | ((uint32_t)lo[3] << 16);
        Lo.z = lo[4] | ((uint32_t)lo[5] << 16);
        Lo.w = lo[6] | ((uint32_t)lo[7] << 16);
        wbh[(size_t)blk * 128 + h * 64 + lane] = H;
        wbl[(size_t)blk * 128 + h * 64 + lane] = Lo;
    }
    // FP16 hi / lo terms of the scaled row (the row's scale is 2^-15 / wrs)
    const double scale = sf * 0x1p-15 / (double)wrs[i];
    for (int h = 0; h < 2; ++h) {
        uint16_t hi[8], lo[8];
        for (int e = 0; e < 8; ++e) {
            const int j = 32 * it + 16 * h + 8 * half + e;
            const double x = (i < M && j < M && j <= i) ? W[(size_t)i * Mpad + j] * scale : 0.0;
            const _Float16 xh = (_Float16)(float)x;
            const _Float16 xl = (_Float16)(float)(x - (double)xh);
            __builtin_memcpy(&hi[e], &xh, 2);
            __builtin_memcpy(&lo[e], &xl, 2);
        }
        wfh[(size_t)blk * 128 + h * 64 + lane] =
            make_uint4(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16),
                       hi[4] | ((uint32_t)hi[5] << 16), hi[6] | ((uint32_t)hi[7] << 16));
        wfl[(size_t)blk * 128 + h * 64 + lane] =
            make_uint4(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16),
                       lo[4] | ((uint32_t)lo[5] << 16), lo[6] | ((uint32_t)lo[7] << 16));
    }
}

__global__ void pack_vec_kernel(const double *Z, const double *alpha, int M, int Mpad, double s0, double s1,
                                double s2, double s3, double c2, double sf2, float *zs, float *al, float *als,
                                float *zs2, float *cz) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= Mpad) return;
    double z[4] = {0.0, 0.0, 0.0, 0.0}, a = 0.0;
    if (j < M) {
        z[0] = Z[4 * j] * s0;
        z[1] = Z[4 * j + 1] * s1;
        z[2] = Z[4 * j + 2] * s2;
        z[3] = Z[4 * j + 3] * s3;
        a = alpha[j];
    }
    const float zf[4] = {(float)z[0], (float)z[1], (float)z[2], (float)z[3]};
    double zz = 0.0;
    for (int d = 0; d < 4; ++d) {
        zs[4 * j + d] = zf[d];
        zs2[4 * j + d] = 2.0f * zf[d];
        zz += (double)zf[d] * (double)zf[d];
    }
    al[j] = (float)a;
    als[j] = (float)(a * sf2 * 0x1p-15);
    cz[j] = (float)(c2 - zz);
}

// Three BF16 terms whose sum is the FP32 value x (round to nearest even at
// each stage; each remainder is exact in FP32).
__device__ __forceinline__ void split3_bf16(float x, uint16_t &h, uint16_t &m, uint16_t &l) {
    const __bf16 bh = (__bf16)x;
    const float r1 = x - (float)bh;
    const __bf16 bm = (__bf16)r1;
    const float r2 = r1 - (float)bm;
    const __bf16 bl = (__bf16)r2;
    __builtin_memcpy(&h, &bh, 2);
    __builtin_memcpy(&m, &bm, 2);
    __builtin_memcpy(&l, &bl, 2);
}

// A operands of the exponent products of the BF16 form.  For column tile jt
// the kernel-vector exponent of point j and sample s,
//   e_js = (c2 - |zs_j|^2) - |qs_s|^2 + sum_d (2 zs_jd) qs_sd,
// is the 32 x 32 product of two 32 x 32 x 16 matrix-core steps with the FP32
// factors split into three BF16 terms (h + m + l); the kept partial products
// hh, hm, mh, hl, mm, lh carry every bit down to 2^-24 of each factor:
//   step 0 slots:  0-3 zh   4-7 zh   8-11 zm   12-15 zh        (B: qh qm qh ql)
//   step 1 slots:  0-3 zm   4-7 zl   8-10 (c2 - |zs|^2) h m l, 11-13 one, 14-15 zero
//                                                              (B: qm qh 1 1 1 -qq h m l 0 0)
// Row rho of a tile holds point 32 jt + P(rho), P(8a + 4b + c) = 16 (a / 2) + 8 b + 4 (a % 2) + c,
// so that lane l of the product's accumulator (rows 8(r/4) + 4(l/32) + r%4) ends
// up with points 8 (l / 32) + r (r < 8) and 16 + 8 (l / 32) + r - 8: the k operand
// of the variance products in its lane order without any exchange.
// zop[(jt * 2 + step) * 64 + lane] = 8 BF16 slots 8 (lane / 32) .. + 7 of row lane % 32.
// zop16: the same 32 slots as one 16 x 16 x 32 product per 16 points: product p's row 4a + c
// holds point 8a + 4p + c, so that the accumulators of the two products give lane l the
// points 8 (l / 16) + r; zop16[(jt * 2 + p) * 64 + lane] = slots 8 (lane / 16) .. + 7 of
// row lane % 16.
__global__ void pack_zop_kernel(const float *zs2, const float *cz, int Mpad, uint4 *zop, uint4 *zop16) {
    const int NT = Mpad / 32;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NT * 128) return;
    const int lane = i & 63, step = (i >> 6) & 1, jt = i >> 7;
    // slots 0 .. 31 of point j: zh zh zm zh | zm zl (c2 - |zs|^2) h m l, 1 1 1, 0 0
    auto slots = [&](int j, uint16_t (&slot)[32]) {
        uint16_t zh[4], zm[4], zl[4], ch, cm, cl;
        for (int d = 0; d < 4; ++d) split3_bf16(zs2[4 * j + d], zh[d], zm[d], zl[d]);
        split3_bf16(cz[j], ch, cm, cl);
        const uint16_t one = 0x3f80;
        for (int d = 0; d < 4; ++d) {
            slot[d] = slot[4 + d] = slot[12 + d] = zh[d];
            slot[8 + d] = slot[16 + d] = zm[d];
            slot[20 + d] = zl[d];
        }
        slot[24] = ch;
        slot[25] = cm;
        slot[26] = cl;
        slot[27] = slot[28] = slot[29] = one;
        slot[30] = slot[31] = 0;
    };
    auto pack = [](const uint16_t *sv) {
        return make_uint4(sv[0] | ((uint32_t)sv[1] << 16), sv[2] | ((uint32_t)sv[3] << 16),
                          sv[4] | ((uint32_t)sv[5] << 16), sv[6] | ((uint32_t)sv[7] << 16));
    };
    uint16_t slot[32];
    const int rho = lane & 31, a = rho >> 3, bb = (rho >> 2) & 1, c = rho & 3;
    slots(32 * jt + 16 * (a >> 1) + 8 * bb + 4 * (a & 1) + c, slot);
    zop[i] = pack(slot + 16 * step + 8 * (lane >> 5));
    const int r16 = lane & 15;
    slots(32 * jt + 8 * (r16 >> 2) + 4 * step + (r16 & 3), slot);
    zop16[i] = pack(slot + 8 * (lane >> 4));
}

hipError_t pack_gp_output(const GpBuildBuffers &b, int M, int Mpad, int o, const double scale[4], double sf2,
                          const GpPacked &p, hipStream_t st) {
    const int NP = (Mpad / 32 + 1) / 2;
    const double *W = b.W + (size_t)o * Mpad * Mpad;
    hipLaunchKernelGGL(row_scale_kernel, dim3(Mpad), dim3(64), 0, st, W, M, Mpad, std::sqrt(sf2), p.wrs);
    hipLaunchKernelGGL(pack_w_kernel, dim3(2 * NP * (NP + 1)), dim3(64), 0, st, W, M, Mpad, std::sqrt(sf2), p.wrs,
                       p.w32, p.wbh, p.wbl, p.wfh, p.wfl);
    hipLaunchKernelGGL(pack_vec_kernel, dim3((Mpad + 255) / 256), dim3(256), 0, st, b.Z + (size_t)o * 4 * M,
                       b.alpha + (size_t)o * Mpad, M, Mpad, scale[0], scale[1], scale[2], scale[3], std::log2(sf2),
                       sf2, p.zs, p.alpha, p.alphas, p.zs2, p.cz);
    hipLaunchKernelGGL(pack_zop_kernel, dim3((Mpad / 32 * 128 + 255) / 256), dim3(256), 0, st, p.zs2, p.cz, Mpad, p.zop,
                       p.zop16);
    return hipGetLastError();
}

}  // namespace gpmppi
