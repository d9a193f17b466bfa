// Gradient of the smoothed expected cost
//   J(U, log ell, log sf) = (1/K) sum_s S~^s
// on gfx950, where S~ is the rollout cost of Alg. 1 Step 1 (Eqs. 1-3, 10-16, one
// combined stage cost) with the lane-exit and collision indicators replaced by
// sigmoid((d_lane - r_bar)/tau) and sigmoid(-min_j d_bar_j / tau).  The noise
// is fixed by the seed; u = clip(U + eps) has derivative 1 strictly inside the
// box.  The derivative in the GP hyperparameters is total (through k, alpha and
// A^-1, A = K(Z, Z) + sn^2 I).
//
// The only recursions are those of the forward states and of their adjoints; everything
// else is the same work for every (step, sample) and runs over all of them at once:
//   rollout            the FP32 rollout (rollout_core.hpp, no track, no obstacles) with its
//                      trace: states, controls, GP variances
//   grad_cov_kernel    Sigma_{k+1} = A Sigma A^T + dt^2 diag(s2), a thread per sample
//   grad_stage_kernel  smoothed stage cost and its adjoint, a thread per (k, s)
//   grad_gp_kernel     r = Q k, Q = A^-1 = W^T W, and the sums over points from which the GP's
//                      share of the adjoint follows by the adjoints s2b, mb of its outputs.
//                      With kappa_j = k_j (2 s2b r_j - mb alpha_j), d = qs - zs_j:
//                        dq_d        = 2 ln2 s_d sum_j kappa_j d_d
//                        d log ell_d = -2 ln2 sum_j kappa_j d_d^2     (through k)
//                      so sum k r d, sum k alpha d, sum k r d^2, sum k alpha d^2, |r|^2 and
//                      r^T alpha are kept per (output, step, sample), and the variance in FP32
//                      operands, which d log sf is sensitive to (see below)
//   grad_back_kernel   the adjoint recursion, a thread per sample
//   grad_syrk_kernel, grad_bterm_kernel, grad_final_kernel
//                      the length-scales' dependence through A:
//                      sum_ij (P_ij - b_i alpha_j) dA_ij/dlog ell_d with b = sum mb r and
//                      P = sum s2b r r^T over all (k, s), contracted on the fly
// The signal variance scales k and K(Z, Z) alike (dA/dlog sf = 2 (A - sn^2 I)),
// so with A r = k and A alpha = y its total derivative folds into per-sample
// terms in which the large parts through k and through A^-1 cancel exactly:
//   d log sf    = 2 s2b (s2 - sn^2 - sn^2 |r|^2) + 2 sn^2 mb r^T alpha
// (s2 - sn^2 = sf^2 - |W k|^2, the latent variance).  What is systematic in it is left over
// after the cancellation: the rollout's variance, whose 16-bit matrix cores round their sums towards
// zero, makes 1e-5 of d log sf where FP32 makes 2e-6 (400 points), so grad_gp_kernel
// computes it again.
//
// The samples are taken in chunks where the workspace (8 Mpad + 280 bytes per (k, s)) is
// limited; a (k, s)'s results do not depend on its chunk.
//
// Measured, K = 4096, T = 50, M = 512: 7.6 ms -> 5.4 ms; K = 256, T = 20, M = 200: 0.94 ms ->
// 0.25 ms.  Before, one kernel ran everything inside the recursion (its r = Q k once
// per reversed step, its variance twice per step: forward and again from checkpoints).
#include "adjoint_step.hpp"
#include "gp_tiles.hpp"

namespace gpmppi {

namespace {

constexpr float kLn2 = 0.69314718055994531f;
constexpr int kGpRows = 32;    // (k, s) entries per workgroup of grad_gp_kernel
constexpr int kGpWaves = 8;

// Sample s0 + threadIdx of chunk c and its place.
struct ChunkPos {
    int s0, sl, s;
    bool valid;
};
__device__ __forceinline__ ChunkPos chunk_pos(const GradArgs &a, int c, int sl) {
    ChunkPos p;
    p.s0 = c * a.Kc;
    p.sl = sl;
    p.s = p.s0 + sl;
    p.valid = sl < a.Kc && p.s < a.K;
    return p;
}

}  // namespace

// Latency of one sample's chain: 1.0 us a step (sine, cosine and 60 multiply-adds).
__global__ __launch_bounds__(64) void grad_cov_kernel(GradArgs a, int chunk) {
    const ChunkPos c = chunk_pos(a, chunk, blockIdx.x * 64 + threadIdx.x);
    if (!c.valid) return;
    const size_t K = a.K, Kc = a.Kc;
    const float dt = a.dyn.dt;
    float p[15] = {};
    const float *x = a.x + c.s, *s2 = a.s2 + c.s;
    float *out = a.cov + c.sl;
    for (int k = 0; k < a.T; ++k) {
        const float th = x[(5 * (size_t)k + 2) * K], v = x[(5 * (size_t)k + 3) * K];
        const float e0 = s2[2 * (size_t)k * K], e1 = s2[(2 * (size_t)k + 1) * K];
        float sth, cth;
        sincosf(th, &sth, &cth);
        const Jac J{-dt * v * sth, dt * cth, dt * v * cth, dt * sth};
        float P[15];
        cov_forward(p, J, dt, a.dyn.a33, a.dyn.a44, dt * dt * e0, dt * dt * e1, P);
#pragma unroll
        for (int i = 0; i < 15; ++i) {
            p[i] = P[i];
            out[(15 * (size_t)k + i) * Kc] = P[i];
        }
    }
}

// Argmin over the polyline segments and obstacles, the smoothed stage cost at (x_{k+1},
// Sigma_{k+1}, s2_k) and its adjoint.  Every lane goes through the whole world at the
// same index, so the geometry comes through the scalar cache; bound by its vector
// instructions (about a dozen per segment).
__global__ __launch_bounds__(256) void grad_stage_kernel(GradArgs a, int chunk) {
    const int k = blockIdx.y;
    const ChunkPos c = chunk_pos(a, chunk, blockIdx.x * 256 + threadIdx.x);
    if (!c.valid) return;
    const size_t K = a.K, Kc = a.Kc;
    const Geometry &geo = a.geo;
    float x1[5], p1[15];
#pragma unroll
    for (int i = 0; i < 5; ++i) x1[i] = a.x[(5 * (size_t)(k + 1) + i) * K + c.s];
    p1[0] = a.cov[(15 * (size_t)k + 0) * Kc + c.sl];
    p1[1] = a.cov[(15 * (size_t)k + 1) * Kc + c.sl];
    p1[5] = a.cov[(15 * (size_t)k + 5) * Kc + c.sl];
    const float s2[2] = {a.s2[2 * (size_t)k * K + c.s], a.s2[(2 * (size_t)k + 1) * K + c.s]};
    const float X = x1[0], Y = x1[1], sa = p1[0], sb = p1[1], sc = p1[5];
    float da, db, dc;
    const float lmax = lmax_grad(sa, sb, sc, da, db, dc);
    float best = INFINITY, om = INFINITY;
    int iseg = -1, iobs = -1;
    if (geo.path_kind != 0) {
        const const_v4p segs = (const_v4p)geo.seg;
        const const_fp sinv = (const_fp)geo.seg_inv;
#pragma unroll 4
        for (int i = 0; i < geo.P; ++i) {
            const v4f sgm = segs[i];
            const float rx = X - sgm.x, ry = Y - sgm.y;
            float t = (rx * sgm.z + ry * sgm.w) * sinv[i];
            t = fminf(fmaxf(t, 0.0f), 1.0f);
            const float ex = rx - t * sgm.z, ey = ry - t * sgm.w;
            const float d2 = ex * ex + ey * ey;
            if (d2 < best) {
                best = d2;
                iseg = i;
            }
        }
    }
    const const_v4p obs = (const_v4p)geo.obs;
#pragma unroll 2
    for (int j = 0; j < geo.n_obs; ++j) {
        const v4f ob = obs[j];
        const float dx = X - ob.x, dyy = Y - ob.y;
        const float rho2 = dx * dx + dyy * dyy;
        const float rho = sqrtf(rho2);
        const float vn = rho > 0.0f ? (sa * dx * dx + 2.0f * sb * dx * dyy + sc * dyy * dyy) / rho2 : lmax;
        const float m = (rho - ob.z) - geo.z_p * sqrtf(fmaxf(vn, 0.0f));
        if (m < om) {
            om = m;
            iobs = j;
        }
    }
    float disc = 1.0f;
    for (int i = 0; i < k; ++i) disc *= a.cw.discount;
    const StageAdj t = stage_adjoint(geo, a.cw, a.inv_tau, a.inv_K, disc, x1, p1, iseg, iobs);
    float *out = a.stage + 6 * (size_t)k * Kc + c.sl;
    out[0 * Kc] = smoothed_stage(geo, a.cw, a.inv_tau, disc, x1, p1, s2, iseg, iobs);
    out[1 * Kc] = t.X;
    out[2 * Kc] = t.Y;
    out[3 * Kc] = t.sa;
    out[4 * Kc] = t.sb;
    out[5 * Kc] = t.sc;
}

namespace {

// LDS of grad_gp_kernel: the k operand ([chunk of 8 points][64] float4), then points and alpha of the output; the waves' partial sums reuse the k operand's place.
__host__ __device__ constexpr int grad_gp_points_off(int Mpad) {
    return Mpad * 128 > kGpWaves * kGradSums * kGpRows * 4 ? Mpad * 128 : kGpWaves * kGradSums * kGpRows * 4;
}
__host__ __device__ constexpr int grad_gp_lds(int Mpad) { return grad_gp_points_off(Mpad) + Mpad * 20; }

}  // namespace

// r = Q k, |W k|^2 and the sums over points of 32 (k, s) entries of one output.  The product stays on the
// FP32 matrix cores: A^-1 magnifies what is systematic in r's error, and the 16-bit ones round
// their sums towards zero (r by FP16 terms of Q and k, exact operands: its error is two thirds of
// FP32's, but d log ell's is three times FP32's, 2.3e-5 against 0.7e-5 at 512 points).
//
// A wave takes row tiles w, w + 8, ... over all columns, the next block in flight; a lane ends up
// with 16 rows of one entry, and adds them up on the vector unit.  Two workgroups to a compute
// unit: one multiplies while the other generates kernel vectors or adds up.
__global__ __launch_bounds__(64 * kGpWaves, 4) void grad_gp_kernel(GradArgs a, int chunk) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, sl = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int o = blockIdx.y, NT = a.gp.NT, Mpad = a.gp.Mpad;
    const GpDev &g = a.gp;
    const int s0 = chunk * a.Kc, kc = a.K - s0 < a.Kc ? a.K - s0 : a.Kc;   // this chunk's samples
    const long long N = (long long)a.T * kc;
    const long long n0 = (long long)blockIdx.x * kGpRows;
    v4f *zs = reinterpret_cast<v4f *>(lds + grad_gp_points_off(Mpad));
    float *al = reinterpret_cast<float *>(zs + Mpad);
    for (int i = tid; i < Mpad; i += 64 * kGpWaves) {
        zs[i] = reinterpret_cast<const v4f *>(g.zs)[(size_t)o * Mpad + i];
        al[i] = g.alpha[(size_t)o * Mpad + i];
    }
    float qs[4];
    {
        const long long nc = n0 + sl < N ? n0 + sl : N - 1;
        const size_t k = (size_t)(nc / kc), s = (size_t)(s0 + nc % kc), K = a.K;
        const float q[4] = {a.x[(5 * k + 3) * K + s], a.x[(5 * k + 4) * K + s], a.u[2 * k * K + s],
                            a.u[(2 * k + 1) * K + s]};
#pragma unroll
        for (int d = 0; d < 4; ++d) qs[d] = q[d] * g.scale[o][d];
    }
    __syncthreads();
    for (int c = 2 * w + half; c < NT * 4; c += 2 * kGpWaves) {   // a lane per entry, 8 points a turn
        float kv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const v4f z = zs[8 * c + e];
            float x = g.c2[o];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const float df = qs[d] - z[d];
                x = fmaf(-df, df, x);
            }
            kv[e] = __builtin_amdgcn_exp2f(x);
        }
        float4 *Kp = reinterpret_cast<float4 *>(lds) + c * 64;
        Kp[sl] = make_float4(kv[0], kv[2], kv[4], kv[6]);
        Kp[32 + sl] = make_float4(kv[1], kv[3], kv[5], kv[7]);
    }
    __syncthreads();
    // k r d (4), k alpha d (4), k r d^2 (4), k alpha d^2 (4), r r, r alpha, (W k)^2
    float sum[kGradSums] = {};
    auto load = [&](float4 (&f)[4], const float4 *p) {
#pragma unroll
        for (int q = 0; q < 4; ++q) f[q] = p[64 * q];
    };
    auto block = [&](v16f &acc, const float4 (&f)[4], int c) {
        float4 kq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) kq[q] = reinterpret_cast<const float4 *>(lds)[(4 * c + q) * 64 + lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 k = kq[q];
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f[q].x, k.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f[q].y, k.y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f[q].z, k.z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f[q].w, k.w, acc, 0, 0, 0);
        }
    };
    // columns 0 .. n - 1 of a row tile whose block c is at p + c stride
    auto walk = [&](v16f &acc, const float4 *p, int n, int stride) {
        float4 f0[4], f1[4];
        load(f0, p);
        for (int c = 0; c < n; c += 2) {   // the barriers keep the loads ahead of the products
            load(f1, p + (size_t)(c + 1 < n ? c + 1 : c) * stride);
            __builtin_amdgcn_sched_barrier(0);
            block(acc, f0, c);
            if (c + 1 >= n) break;
            load(f0, p + (size_t)(c + 2 < n ? c + 2 : c) * stride);
            __builtin_amdgcn_sched_barrier(0);
            block(acc, f1, c + 1);
        }
    };
    for (int i = 0; i * kGpWaves < NT; ++i) {   // W's row tiles, the long ones with the short ones
        const int t = kGpWaves * i + ((i & 1) ? kGpWaves - 1 - w : w);
        if (t >= NT) continue;
        v16f acc = v16f{};
        const int u = t >> 1;
        walk(acc, g.w32 + o * g.w32_stride + (size_t)(2 * u * (u + 1) + (t & 1)) * 256 + lane, t + 1, 512);
#pragma unroll
        for (int e = 0; e < 16; ++e) sum[18] = fmaf(acc[e], acc[e], sum[18]);
    }
    const float4 *Qo = a.q32 + (size_t)o * a.q_stride + lane;
    // this workgroup's rows of R; stores beyond the chunk's last entry are dropped
    const __amdgpu_buffer_rsrc_t Rr = uniform_rsrc(a.R + ((size_t)o * a.T * a.Kc + n0) * Mpad,
                                                   (N - n0 < kGpRows ? N - n0 : kGpRows) * Mpad * 4);
    for (int t = w; t < NT; t += kGpWaves) {
        v16f acc = v16f{};
        walk(acc, Qo + (size_t)t * NT * 256, NT, 256);
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            const int row = 32 * t + 8 * e4 + 4 * half;
            const v4f av = *reinterpret_cast<const v4f *>(al + row);
            // kernel values of rows row .. + 3 (even and odd points are apart in the operand)
            const float4 *Kp = reinterpret_cast<const float4 *>(lds) + (t * 4 + e4) * 64 + sl;
            const float2 ke = reinterpret_cast<const float2 *>(Kp)[half];
            const float2 ko = reinterpret_cast<const float2 *>(Kp + 32)[half];
            const float kv[4] = {ke.x, ko.x, ke.y, ko.y};
            uint32_t __attribute__((ext_vector_type(4))) ru;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const v4f z = zs[row + e];
                const float r = acc[4 * e4 + e];
                ru[e] = __float_as_uint(r);
                const float kr = kv[e] * r, ka = kv[e] * av[e];
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const float df = qs[d] - z[d];
                    const float x = kr * df, y = ka * df;
                    sum[d] += x;
                    sum[4 + d] += y;
                    sum[8 + d] = fmaf(x, df, sum[8 + d]);
                    sum[12 + d] = fmaf(y, df, sum[12 + d]);
                }
                sum[16] = fmaf(r, r, sum[16]);
                sum[17] = fmaf(r, av[e], sum[17]);
            }
            __builtin_amdgcn_raw_buffer_store_b128(ru, Rr, (sl * Mpad + row) * 4, 0, 0);
        }
    }
    __syncthreads();   // the k operand's last readers are done
    float *red = reinterpret_cast<float *>(lds);   // [wave][sum][32]
#pragma unroll
    for (int j = 0; j < kGradSums; ++j) {
        const float x = sum[j] + shfl_xor(sum[j], 32);
        if (half == 0) red[(w * kGradSums + j) * kGpRows + sl] = x;
    }
    __syncthreads();
    for (int i = tid; i < kGradSums * kGpRows; i += 64 * kGpWaves) {
        const int j = i / kGpRows, l = i % kGpRows;
        float x = 0.0f;
#pragma unroll
        for (int v = 0; v < kGpWaves; ++v) x += red[(v * kGradSums + j) * kGpRows + l];
        if (j == 18) x = g.vscale[o] * (g.sn2[o] + fmaxf(0.0f, g.sf2[o] - x));
        if (n0 + l < N) a.sums[((size_t)o * kGradSums + j) * a.T * a.Kc + n0 + l] = x;
    }
}

// The adjoint recursion, last step first, a thread per sample; the next step's records are
// loaded beside a step's arithmetic.
__global__ __launch_bounds__(64) void grad_back_kernel(GradArgs a, int chunk) {
    __shared__ double hred[10][64];
    const int lane = threadIdx.x;
    const ChunkPos c = chunk_pos(a, chunk, blockIdx.x * 64 + lane);
    const size_t K = a.K, Kc = a.Kc;
    const int kc = a.K - c.s0 < a.Kc ? a.K - c.s0 : a.Kc;
    const size_t NS = (size_t)a.T * a.Kc;   // stride of the chunk arrays
    const int s = c.valid ? c.s : a.K - 1, sl = c.valid ? c.sl : kc - 1;
    const int slot = chunk * gridDim.x + blockIdx.x;
    const GpDev &g = a.gp;
    const float cbar = c.valid ? a.inv_K : 0.0f;
    const NoiseParams np = a.noise;
    {   // Eq. 5's sum, Kahan-compensated, in step order
        float S = 0.0f, Sc = 0.0f;
        const float *st = a.stage + sl;
#pragma unroll 8
        for (int k = 0; k < a.T; ++k) {
            const float yk = st[6 * (size_t)k * Kc] - Sc;
            const float tk = S + yk;
            Sc = (tk - S) - yk;
            S = tk;
        }
        if (c.valid) a.costs[s] = S;
    }
    struct Rec {
        float th, v, v1, p[15];
        StageAdj t;
        float sum[2][kGradSums];
    };
    auto load = [&](Rec &r, int k) {
        const size_t kk = k;
        r.th = a.x[(5 * kk + 2) * K + s];
        r.v = a.x[(5 * kk + 3) * K + s];
        r.v1 = a.x[(5 * (kk + 1) + 3) * K + s];
#pragma unroll
        for (int i = 0; i < 15; ++i) r.p[i] = k > 0 ? a.cov[(15 * (kk - 1) + i) * Kc + sl] : 0.0f;
        const float *st = a.stage + 6 * kk * Kc + sl;
        r.t = StageAdj{st[Kc], st[2 * Kc], st[3 * Kc], st[4 * Kc], st[5 * Kc]};
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int j = 0; j < kGradSums; ++j) r.sum[o][j] = a.sums[(o * kGradSums + j) * NS + kk * kc + sl];
    };
    double hyp[2][5] = {};
    float xb[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    float pb[15] = {};
    Rec r, nx;
    load(r, a.T - 1);
    for (int k = a.T - 1; k >= 0; --k) {
        if (k > 0) load(nx, k - 1);
        StepAdj sa;
        chain_adjoint(a.cw, a.dyn, cbar, r.th, r.v, r.p, r.v1, r.t, xb, pb, sa);
        float qb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const float *t = r.sum[o];
            const float sbo = t[18] > g.sn2[o] ? sa.s2b[o] : 0.0f, mb = sa.mb[o];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                qb[d] += 2.0f * kLn2 * g.scale[o][d] * (2.0f * sbo * t[d] - mb * t[4 + d]);
                hyp[o][d] += (double)(-2.0f * kLn2 * (2.0f * sbo * t[8 + d] - mb * t[12 + d]));
            }
            {   // log sf: the folded per-sample terms (k and A^-1 parts cancelled)
                const double sn2 = (double)g.sn2[o];
                hyp[o][4] += 2.0 * (double)sbo * (((double)t[18] - sn2) - sn2 * (double)t[16]) +
                             2.0 * sn2 * (double)mb * (double)t[17];
            }
            if (c.valid) {
                float *wg = a.wgt + (size_t)o * 2 * NS + (size_t)k * kc + sl;
                wg[0] = sbo;
                wg[NS] = mb;
            }
        }
        xb[3] += qb[0];
        xb[4] += qb[1];
        // the nominal control's adjoint through the clip (1 strictly inside the box)
        const float2 raw = sampled_raw(np, k, s, a.U[2 * k], a.U[2 * k + 1]);
        float ub[2] = {sa.ub[0] + qb[2], sa.ub[1] + qb[3]};
        if (!(c.valid && raw.x > np.umin0 && raw.x < np.umax0)) ub[0] = 0.0f;
        if (!(c.valid && raw.y > np.umin1 && raw.y < np.umax1)) ub[1] = 0.0f;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) ub[i] += shfl_xor(ub[i], m);
            if (lane == 0) a.upart[((size_t)slot * a.T + k) * 2 + i] = ub[i];
        }
        r = nx;
    }
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int i = 0; i < 5; ++i) hred[o * 5 + i][lane] = c.valid ? hyp[o][i] : 0.0;
    __syncthreads();
    if (lane < 10) {
        double sum = 0.0;
        for (int i = 0; i < 64; ++i) sum += hred[lane][i];
        a.hpart[(size_t)slot * 10 + lane] = sum;
    }
}

__global__ __launch_bounds__(kThreads) void exchange_clear_kernel(unsigned long long *rec, size_t n_rec, uint32_t *xep,
                                                                  uint32_t *repair, int n_blk) {
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n_rec) rec[i] = 0ull;
    if (i < 2) xep[i] = 0u;
    if (i < (size_t)n_blk) repair[i] = 0u;
}

hipError_t launch_exchange_clear(unsigned long long *rec, size_t n_rec, uint32_t *xep, uint32_t *repair, int n_blk,
                                 hipStream_t st) {
    const size_t n = n_rec > (size_t)n_blk ? n_rec : (size_t)n_blk;
    hipLaunchKernelGGL(exchange_clear_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                       rec, n_rec, xep, repair, n_blk);
    return hipGetLastError();
}

// dA_ij / dlog ell_d contracted with a weight c_ij: K_ij = exp2(c2 - |zs_i - zs_j|^2),
// dA/dlog ell_d = K 2 ln2 (zs_id - zs_jd)^2 (the sn^2 I part does not depend on it).
__device__ __forceinline__ void dA_contract(float cval, const float4 &zi, const float4 &zj, float c2, double acc[4]) {
    const float d0 = zi.x - zj.x, d1 = zi.y - zj.y, d2 = zi.z - zj.z, d3 = zi.w - zj.w;
    const float e0 = d0 * d0, e1 = d1 * d1, e2 = d2 * d2, e3 = d3 * d3;
    const float Kij = __builtin_amdgcn_exp2f(c2 - (e0 + e1 + e2 + e3));
    const float ck = cval * Kij;
    const float c2l = 2.0f * kLn2 * ck;
    acc[0] += (double)(c2l * e0);
    acc[1] += (double)(c2l * e1);
    acc[2] += (double)(c2l * e2);
    acc[3] += (double)(c2l * e3);
}

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
    return x;
}

// P = sum_n g_n r_n r_n^T over rows n in [n0, n1) of one output, for one
// 128 x 128 block (bi <= bj) of the Mpad x Mpad result, contracted with dA/dlog ell:
// ppart[((o * nslot + slot) * npairs + pair) * 4 + d], slot = chunk nsplit + split.  Wave w
// owns the 32 x 32 tiles (2 (w >> 1) + {0, 1}, 2 (w & 1) + {0, 1}) of the block.  The blocks on
// the diagonal also sum their rows' share of b = sum_n mb_n r_n into bpart[slot][o].
__global__ __launch_bounds__(kThreads) void grad_syrk_kernel(GradArgs a, int chunk) {
    __shared__ double red[kWaves][4];
    // consecutive workgroups go to the eight XCDs in turn: every block pair of the same rows on one
    // XCD, whose L2 then holds the rows
    const int npairs = a.npairs, nsplit = a.nsplit, Mpad = a.gp.Mpad;
    const int group = ((int)blockIdx.x / (8 * npairs)) * 8 + (int)(blockIdx.x & 7), pair = ((int)blockIdx.x >> 3) % npairs;
    if (group >= 2 * nsplit) return;
    const int split = group >> 1, o = group & 1;
    const int slot = chunk * nsplit + split, nslot = a.nchunk * nsplit;
    const int s0 = chunk * a.Kc, kc = a.K - s0 < a.Kc ? a.K - s0 : a.Kc;
    const long long TK = (long long)a.T * kc;
    const int nb = (Mpad + 127) / 128;
    int bi = 0, rem = pair;
    while (rem >= nb - bi) {
        rem -= nb - bi;
        ++bi;
    }
    const int bj = bi + rem;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ti0 = 4 * bi + 2 * (w >> 1), tj0 = 4 * bj + 2 * (w & 1);
    const int NT = Mpad >> 5;
    const bool vi[2] = {ti0 < NT, ti0 + 1 < NT}, vj[2] = {tj0 < NT, tj0 + 1 < NT};
    const long long rows = (TK + nsplit - 1) / nsplit;
    const long long n0 = (long long)split * rows;
    const long long n1 = n0 + rows < TK ? n0 + rows : TK;
    const size_t NS = (size_t)a.T * a.Kc;
    const float *Ro = a.R + o * NS * Mpad;
    const float *Go = a.wgt + o * 2 * NS;
    const bool bsum = bi == bj && (w & 1) == 0;
    double bacc[2] = {0.0, 0.0};
    v16f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = v16f{};
    const int col = lane & 31, rsel = lane >> 5;
    // rows in chunks of kD row pairs, the next chunk's loads in flight beside a chunk's products;
    // rows past the end count with weight 0
    constexpr int kD = 4;
    struct Rows {
        float g[kD], m[kD], ra[kD][2], rb[kD][2];
    };
    auto load = [&](Rows &r, long long n) {
#pragma unroll
        for (int q = 0; q < kD; ++q) {
            const long long at = n + 2 * q + rsel;
            const bool ok = at < n1;
            const long long row = ok ? at : n0;
            const float *rp = Ro + (size_t)row * Mpad + col;
            r.g[q] = ok ? Go[row] : 0.0f;
            r.m[q] = ok && bsum ? Go[NS + row] : 0.0f;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                r.ra[q][i] = vi[i] ? rp[32 * (ti0 + i)] : 0.0f;
                r.rb[q][i] = vj[i] ? rp[32 * (tj0 + i)] : 0.0f;
            }
        }
    };
    auto multiply = [&](const Rows &r) {
#pragma unroll
        for (int q = 0; q < kD; ++q) {
            const float av[2] = {r.g[q] * r.ra[q][0], r.g[q] * r.ra[q][1]};
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i], r.rb[q][j], acc[i][j], 0, 0, 0);
            if (bsum) {
                bacc[0] += (double)(r.m[q] * r.ra[q][0]);
                bacc[1] += (double)(r.m[q] * r.ra[q][1]);
            }
        }
    };
    if (n0 < n1) {
        Rows r0, r1;
        load(r0, n0);
        for (long long n = n0; n < n1; n += 4 * kD) {
            load(r1, n + 2 * kD);
            __builtin_amdgcn_sched_barrier(0);   // the loads stay ahead of the products
            multiply(r0);
            load(r0, n + 4 * kD);
            __builtin_amdgcn_sched_barrier(0);
            multiply(r1);
        }
    }
    if (bsum) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const double v = bacc[i] + __shfl_xor(bacc[i], 32, 64);
            if (rsel == 0 && vi[i]) a.bpart[((size_t)slot * 2 + o) * Mpad + 32 * (ti0 + i) + col] = v;
        }
    }
    // epilogue: sum_ij P_ij dA_ij/dtheta over the wave's tiles (both triangles of a
    // diagonal block; off-diagonal blocks stand for their mirror image too)
    const float c2 = a.gp.c2[o];
    const float4 *z = reinterpret_cast<const float4 *>(a.gp.zs) + (size_t)o * Mpad;
    const float weight = bi == bj ? 1.0f : 2.0f;
    double cacc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (!vi[i] || !vj[j]) continue;
            const float4 zj = z[32 * (tj0 + j) + col];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = 32 * (ti0 + i) + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                dA_contract(weight * acc[i][j][e], z[row], zj, c2, cacc);
            }
        }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const double v = wave_sum(cacc[t]);
        if (lane == 0) red[w][t] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const double v = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
        a.ppart[(((size_t)o * nslot + slot) * npairs + pair) * 4 + threadIdx.x] = v;
    }
}

// b = sum of the partial b, then sum_ij b_i alpha_j dA_ij/dlog ell_d: a workgroup per 32 rows
// i, eight threads a row that take every eighth j; bterm[(o * gridDim.x + block) * 4 + d].
__global__ __launch_bounds__(kThreads) void grad_bterm_kernel(GradArgs a) {
    __shared__ double red[kWaves][4];
    const int o = blockIdx.y, Mpad = a.gp.Mpad, nslot = a.nchunk * a.nsplit;
    const int i = blockIdx.x * 32 + (threadIdx.x >> 3), part = threadIdx.x & 7;
    const float c2 = a.gp.c2[o];
    const float4 *z = reinterpret_cast<const float4 *>(a.gp.zs) + (size_t)o * Mpad;
    const float *al = a.gp.alpha + (size_t)o * Mpad;
    double b = 0.0;
    for (int s = part; s < nslot; s += 8) b += a.bpart[((size_t)s * 2 + o) * Mpad + i];
#pragma unroll
    for (int m = 1; m < 8; m <<= 1) b += __shfl_xor(b, m, 64);
    const float4 zi = z[i];
    const float bf = (float)b;
    double cacc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int j = part; j < Mpad; j += 8) dA_contract(bf * al[j], zi, z[j], c2, cacc);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const double v = wave_sum(cacc[t]);
        if (lane == 0) red[w][t] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const double v = red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
        a.bterm[((size_t)o * gridDim.x + blockIdx.x) * 4 + threadIdx.x] = v;
    }
}

// Fixed-order final sums, a workgroup each: J = mean smoothed cost and the hyperparameter
// gradient (block 0), dU[k][c] (the others).  log ell_d = direct (through k) +
// (P - b alpha^T) : dA/dlog ell_d; log sf = its folded per-sample terms.
__global__ __launch_bounds__(kThreads) void grad_final_kernel(GradArgs a, int nslot_back) {
    __shared__ double red[kThreads];
    const int tid = threadIdx.x;
    // sum over i < n of p[i stride], in a fixed order
    auto total = [&](auto p, size_t n, size_t stride) {
        double v = 0.0;
        for (size_t i = tid; i < n; i += kThreads) v += (double)p[i * stride];
        __syncthreads();
        red[tid] = v;
        __syncthreads();
        for (int h = kThreads / 2; h > 0; h >>= 1) {
            if (tid < h) red[tid] += red[tid + h];
            __syncthreads();
        }
        return red[0];
    };
    const int b = blockIdx.x;
    if (b < 2 * a.T) {
        const double v = total(a.upart + b, nslot_back, (size_t)2 * a.T);
        if (tid == 0) a.dU[b] = (float)v;
        return;
    }
    const int i = b - 2 * a.T;
    if (i == 10) {
        const double v = total(a.costs, a.K, 1);
        if (tid == 0) a.J[0] = (float)(v / (double)a.K);
        return;
    }
    const int o = i / 5, t = i % 5;
    const double direct = total(a.hpart + i, nslot_back, 10);
    if (t == 4) {
        if (tid == 0) a.dlog_sf[o] = (float)direct;
        return;
    }
    const size_t np = (size_t)a.nchunk * a.nsplit * a.npairs;
    const double mat = total(a.ppart + (size_t)o * np * 4 + t, np, 4);
    const double bt = total(a.bterm + (size_t)o * a.nbterm * 4 + t, a.nbterm, 4);
    if (tid == 0) a.dlog_ell[o * 4 + t] = (float)(direct + mat - bt);
}

hipError_t launch_grad(const GradArgs &a, hipStream_t st) {
    const int nblk = (a.Kc + 63) / 64;
    const int lds = grad_gp_lds(a.gp.Mpad);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(grad_gp_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    for (int c = 0; c < a.nchunk; ++c) {
        const int kc = a.K - c * a.Kc < a.Kc ? a.K - c * a.Kc : a.Kc;
        const long long N = (long long)a.T * kc;
        hipLaunchKernelGGL(grad_cov_kernel, dim3(nblk), dim3(64), 0, st, a, c);
        hipLaunchKernelGGL(grad_stage_kernel, dim3((kc + 255) / 256, a.T), dim3(256), 0, st, a, c);
        hipLaunchKernelGGL(grad_gp_kernel, dim3((unsigned)((N + kGpRows - 1) / kGpRows), 2), dim3(64 * kGpWaves), lds, st, a, c);
        hipLaunchKernelGGL(grad_back_kernel, dim3(nblk), dim3(64), 0, st, a, c);
        hipLaunchKernelGGL(grad_syrk_kernel, dim3((2 * a.nsplit + 7) / 8 * 8 * a.npairs), dim3(kThreads), 0, st, a,
                           c);
    }
    hipLaunchKernelGGL(grad_bterm_kernel, dim3(a.nbterm, 2), dim3(kThreads), 0, st, a);
    hipLaunchKernelGGL(grad_final_kernel, dim3(2 * a.T + 11), dim3(kThreads), 0, st, a, a.nchunk * nblk);
    return hipGetLastError();
}

}  // namespace gpmppi
