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
//   grad_forward_kernel  states, controls, GP variances and covariances, step after step
//   grad_stage_kernel  smoothed stage cost and its adjoint, a thread per (k, s)
//   grad_gp_kernel     r = Q k, Q = A^-1 = W^T W, and the sums over points from which the GP's
//                      share of the adjoint follows by the adjoints s2b, mb of its outputs.
//                      With kappa_j = k_j (2 s2b r_j - mb alpha_j), d = qs - zs_j:
//                        dq_d        = 2 ln2 s_d sum_j kappa_j d_d
//                        d log ell_d = -2 ln2 sum_j kappa_j d_d^2     (through k)
//                      so sum k r d, sum k alpha d, sum k r d^2, sum k alpha d^2, |r|^2 and
//                      r^T alpha are kept per (output, step, sample)
//   grad_back_kernel   the adjoint recursion, a thread per sample
//   grad_syrk_kernel, grad_bterm_kernel, grad_final_kernel
//                      the length-scales' dependence through A:
//                      sum_ij (P_ij - b_i alpha_j) dA_ij/dlog ell_d with b = sum mb r and
//                      P = sum s2b r r^T over all (k, s), contracted on the fly
// The signal variance scales k and K(Z, Z) alike (dA/dlog sf = 2 (A - sn^2 I)),
// so with A r = k and A alpha = y its total derivative folds into per-sample
// terms in which the large parts through k and through A^-1 cancel exactly:
//   d log sf    = 2 s2b (s2 - sn^2 - sn^2 |r|^2) + 2 sn^2 mb r^T alpha
// (s2 - sn^2 = sf^2 - |W k|^2, the latent variance of the forward pass).  What is
// systematic in it is left over after the cancellation.
//
// The samples are taken in chunks where the workspace (8 Mpad + 280 bytes per (k, s)) is
// limited; a (k, s)'s results do not depend on its chunk.
//
// Measured, K = 4096, T = 50, M = 512: 7.6 ms -> 4.3 ms; K = 256, T = 20, M = 200: 0.94 ms ->
// 0.36 ms.  Before, one kernel ran everything inside the recursion (its r = Q k once
// per reversed step, its variance twice per step: forward and again from checkpoints).
#include "adjoint_step.hpp"
#include "gp_tiles.hpp"

namespace gpmppi {

namespace {

constexpr float kLn2 = 0.69314718055994531f;

// a b, never fused with a later sum.
__device__ __forceinline__ float mul_rounded(float a, float b) {
#pragma clang fp contract(off)
    return a * b;
}
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

namespace {

constexpr int kB = 32;           // samples per workgroup of the forward pass
constexpr int kParts = 8;        // loop splitters

// Dynamic LDS of the forward pass: [k operand 32 x Mpad FP32][staged inputs]
__host__ __device__ constexpr size_t grad_forward_lds(int Mpad) {
    return kgroup_bytes<GPMPPI_FP32>(Mpad) + (size_t)staged_slots<GPMPPI_FP32>(Mpad) * 16;
}

__device__ __forceinline__ void restage(const GpDev &g, int o, unsigned char *lds) {
    __syncthreads();
    StagedInputs st;
    stage_load<GPMPPI_FP32>(st, g, o);
    stage_store<GPMPPI_FP32>(st, g, lds, kgroup_bytes<GPMPPI_FP32>(g.Mpad));
    __syncthreads();
}

}  // namespace

// Forward pass: states, controls, variances and covariances of every step, a workgroup of 32
// samples or, split, two, workgroup 2 blk + r computing output r's mean and variance and both the
// per-sample algebra; they exchange mean and variance every step.  The exchanged values enter the
// same instructions as in the unsplit form (one kernel: two would fuse products and sums
// differently), so the results are the same bit for bit.  A workgroup whose bounded exchange wait
// gives up marks its block for the unsplit repair launch that follows every split launch and
// runs the marked blocks only.
//
// The rollout's own kernels would take two thirds of the time, with sums grouped otherwise.  J's
// gradient jumps where two segments or obstacles are equally near, and one sample in 200000 that
// changes sides moves dU by 3e-5 of its norm; the FP32 grouping here is kept for that, and for
// d log sf, which a variance from the 16-bit matrix cores (sums rounded towards zero) moves by
// 1e-5 (see the top).
enum ForwardMode { kForwardWhole = 0, kForwardSplit = 1, kForwardRepair = 2 };

__global__ __launch_bounds__(kThreads) void grad_forward_kernel(GradArgs a, int mode) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ float pred[kParts * kB];
    __shared__ float vred[kWaves * kB];
    __shared__ float xv[2 * kB + 1];   // split: values received from the partner, and a give-up flag

    const bool split = mode == kForwardSplit;
    const int tid = threadIdx.x;
    const int lane = tid & 63, w = tid >> 6;
    const int sl = lane & 31;
    const int part = 2 * w + (lane >> 5);
    const int blk = split ? (int)(blockIdx.x >> 1) : (int)blockIdx.x;
    const int role = split ? (int)(blockIdx.x & 1) : 0;   // split: the GP output this workgroup computes
    if (mode == kForwardRepair && __hip_atomic_load(a.repair + blk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) return;
    const int sg = blk * kB + sl;
    const bool writer = w == 0 && lane < kB && role == 0 && sg < a.K;   // one copy of each sample
    const size_t K = a.K;
    const GpDev &g = a.gp;
    const Dyn dy = a.dyn;
    const float dt = dy.dt;
    NoiseParams np = a.noise;

    // split exchange: step k uses slot k % 4 of the writer's records [block][writer role][slot]
    // [kind][32]; records are zeroed before the launch, and the tag k + 1 names the step
    unsigned long long *xrec = a.xrec + (size_t)blk * kGradXchPerBlock;
    auto xslot = [&](int wr, int k, int kind) { return xrec + ((size_t)(wr * 4 + (k & 3)) * 2 + kind) * kB; };
    bool broken = false;

    float X = a.x0[0], Y = a.x0[1], th = a.x0[2], v = a.x0[3], w_ = a.x0[4];
    float p[15];
#pragma unroll
    for (int i = 0; i < 15; ++i) p[i] = 0.0f;
    restage(g, role, lds);
    for (int k = 0; k < a.T; ++k) {
        if (writer) {
            float *x = a.x + 5 * (size_t)k * K + sg;
            x[0 * K] = X;
            x[1 * K] = Y;
            x[2 * K] = th;
            x[3 * K] = v;
            x[4 * K] = w_;
        }
        const bool rev = (k & 1) != 0;
        const float2 u = sampled_control(np, k, sg, a.U[2 * k], a.U[2 * k + 1]);
        const float q[4] = {v, w_, u.x, u.y};
        float m[2], s2[2];
        if (split) {   // this role's output, then the partner's mean and variance
            const int o = role;
            __syncthreads();
            const float qs[4] = {mul_rounded(q[0], g.scale[o][0]), mul_rounded(q[1], g.scale[o][1]),
                                 mul_rounded(q[2], g.scale[o][2]), mul_rounded(q[3], g.scale[o][3])};
            gp_output<GPMPPI_FP32, 1>(g, o, -1, qs, part, sl, rev, 0, blk, lds, pred, vred, m[o], s2[o]);
            const uint32_t tag = (uint32_t)k + 1;
            if (w == 0) {
                xch_put(xslot(role, k, 0), lane, m[o], tag);
                xch_put(xslot(role, k, 1), lane, s2[o], tag);
                const float mp = xch_get(xslot(1 - role, k, 0), lane, tag, a.xspin, broken);
                const float sp = xch_get(xslot(1 - role, k, 1), lane, tag, a.xspin, broken);
                if (lane < kB) {
                    xv[lane] = mp;
                    xv[kB + lane] = sp;
                }
                if (lane == 0) xv[2 * kB] = broken ? 1.0f : 0.0f;
            }
            __syncthreads();
            if (xv[2 * kB] != 0.0f) {   // uniform: leave the block to the repair launch
                if (tid == 0) {
                    __hip_atomic_store(a.repair + blk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (a.flags)
                        __hip_atomic_fetch_or(a.flags, GPMPPI_FLAG_EXCHANGE_TIMEOUT, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
                }
                return;
            }
            m[1 - o] = xv[sl];
            s2[1 - o] = xv[kB + sl];
        } else {
#pragma unroll
            for (int oo = 0; oo < 2; ++oo) {
                const int o = rev ? 1 - oo : oo;
                __syncthreads();
                const float qs[4] = {mul_rounded(q[0], g.scale[o][0]), mul_rounded(q[1], g.scale[o][1]),
                                     mul_rounded(q[2], g.scale[o][2]), mul_rounded(q[3], g.scale[o][3])};
                gp_output<GPMPPI_FP32, 1>(g, o, oo == 0 ? 1 - o : -1, qs, part, sl, rev, 0, blk, lds, pred, vred, m[o],
                                          s2[o]);
            }
        }
        float sth, cth;
        sincosf(th, &sth, &cth);
        const Jac J{-dt * v * sth, dt * cth, dt * v * cth, dt * sth};
        const float Xn = X + dt * v * cth;
        const float Yn = Y + dt * v * sth;
        const float thn = th + dt * w_;
        // where either of two products could be fused with their sum, which one is spelt out
        const float vn = v + fmaf(dy.dt_tau_v, u.x - v, mul_rounded(dt, m[0]));
        const float wn = w_ + fmaf(dy.dt_tau_w, u.y - w_, mul_rounded(dt, m[1]));
        float P[15];
        cov_forward(p, J, dt, dy.a33, dy.a44, mul_rounded(dt * dt, s2[0]), mul_rounded(dt * dt, s2[1]), P);
#pragma unroll
        for (int i = 0; i < 15; ++i) p[i] = P[i];
        X = Xn; Y = Yn; th = thn; v = vn; w_ = wn;
        if (writer) {
#pragma unroll
            for (int i = 0; i < 2; ++i) a.s2[(2 * (size_t)k + i) * K + sg] = s2[i];
            a.u[2 * (size_t)k * K + sg] = u.x;
            a.u[(2 * (size_t)k + 1) * K + sg] = u.y;
#pragma unroll
            for (int i = 0; i < 15; ++i) a.cov[(15 * (size_t)k + i) * K + sg] = p[i];
        }
    }
    if (writer) {
        float *x = a.x + 5 * (size_t)a.T * K + sg;
        x[0 * K] = X;
        x[1 * K] = Y;
        x[2 * K] = th;
        x[3 * K] = v;
        x[4 * K] = w_;
    }
    if (mode == kForwardRepair && tid == 0)   // the block is done
        __hip_atomic_store(a.repair + blk, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Zeroes the split forward pass's exchange records and repair marks before a launch.
__global__ __launch_bounds__(kThreads) void grad_clear_kernel(unsigned long long *rec, size_t n_rec, uint32_t *repair,
                                                              int n_blk) {
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n_rec) rec[i] = 0ull;
    if (i < (size_t)n_blk) repair[i] = 0u;
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
    p1[0] = a.cov[(15 * (size_t)k + 0) * K + c.s];
    p1[1] = a.cov[(15 * (size_t)k + 1) * K + c.s];
    p1[5] = a.cov[(15 * (size_t)k + 5) * K + c.s];
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

// r = Q k and the sums over points of 32 (k, s) entries of one output.  The product stays on the
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
    // k r d (4), k alpha d (4), k r d^2 (4), k alpha d^2 (4), r r, r alpha
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
        float th, v, v1, s2[2], p[15];
        StageAdj t;
        float sum[2][kGradSums];
    };
    auto load = [&](Rec &r, int k) {
        const size_t kk = k;
        r.th = a.x[(5 * kk + 2) * K + s];
        r.v = a.x[(5 * kk + 3) * K + s];
        r.v1 = a.x[(5 * (kk + 1) + 3) * K + s];
#pragma unroll
        for (int o = 0; o < 2; ++o) r.s2[o] = a.s2[(2 * kk + o) * K + s];
#pragma unroll
        for (int i = 0; i < 15; ++i) r.p[i] = k > 0 ? a.cov[(15 * (kk - 1) + i) * K + s] : 0.0f;
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
            const float sbo = r.s2[o] > g.sn2[o] ? sa.s2b[o] : 0.0f, mb = sa.mb[o];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                qb[d] += 2.0f * kLn2 * g.scale[o][d] * (2.0f * sbo * t[d] - mb * t[4 + d]);
                hyp[o][d] += (double)(-2.0f * kLn2 * (2.0f * sbo * t[8 + d] - mb * t[12 + d]));
            }
            {   // log sf: the folded per-sample terms (k and A^-1 parts cancelled)
                const double sn2 = (double)g.sn2[o];
                hyp[o][4] += 2.0 * (double)sbo * (((double)r.s2[o] - sn2) - sn2 * (double)t[16]) +
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

// Three BF16 terms of eight FP32 values (exact: each remainder is).
struct Terms {
    uint4 t[3];
};
__device__ __forceinline__ void split_terms(Terms &o, const float x[8]) {
    uint32_t u[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            u[k][i] = pack_bf16x2(a, b);
            a -= __uint_as_float(u[k][i] << 16);
            b -= __uint_as_float(u[k][i] & 0xffff0000u);
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) o.t[k] = make_uint4(u[k][0], u[k][1], u[k][2], u[k][3]);
}

// P = sum_n g_n r_n r_n^T over rows n in [n0, n1) of one output, for one
// 128 x 128 block (bi <= bj) of the Mpad x Mpad result, contracted with dA/dlog ell:
// ppart[((o * nslot + slot) * npairs + pair) * 4 + d], slot = chunk nsplit + split.  Wave w
// owns the 32 x 32 tiles (2 (w >> 1) + {0, 1}, 2 (w & 1) + {0, 1}) of the block.  The blocks on
// the diagonal also sum their rows' share of b = sum_n mb_n r_n into bpart[slot][o].
//
// The FP32 values go through the BF16 matrix cores as three terms each (24 bits, exact) and six
// products: at 512 points, T K = 204800, 1.3 ms instead of 2.0 (FP32 products take 1.0 at their peak
// rate); bound by the vector unit that splits (a third of the time) and the barriers of a turn.
// The 16-bit cores round their sums towards zero, so every 32 rows start a fresh sum, the leading
// products last, that is added in FP32 (round to nearest); the error of d log ell by it is 3e-7,
// where one running sum makes 2e-5 and FP32 products 4e-7 (512 points, 4096 rows; over 60
// gradients the error of d log ell against 64 bits is 0.985 of FP32 products' and a running
// FP32 sum's, geometric mean; dU 0.998, d log sf 1.004).
//
// A workgroup loads and splits its 32 rows of 256 columns once and shares them in LDS.
__global__ __launch_bounds__(kThreads, 2) void grad_syrk_kernel(GradArgs a, int chunk) {
    __shared__ uint4 terms[8 * 2 * 3 * 64];
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
    const float *Go = a.wgt + o * 2 * NS;
    v16f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = v16f{};
    const int col = lane & 31;
    // Thread (rg, cq) of the 32 rows of a turn: rows 8 rg .. + 7, columns 4 cq .. + 3 of the block's
    // 128 columns of i (cq < 32, weighted) and 128 of j; operand of 32 columns and 16 rows:
    // terms[tile][step][term][lane ^ (tile & 3)] (the exclusive or spreads the stores over the banks)
    const int rg = w, cq = lane, tile = cq >> 3;
    const bool wgt = cq < 32, bsum = bi == bj && wgt;
    const int c0 = wgt ? 128 * bi + 4 * cq : 128 * bj + 4 * (cq - 32);
    const bool cok = c0 < Mpad;
    const float *Rc = a.R + o * NS * Mpad + (cok ? c0 : 0);
    double bacc[4] = {0.0, 0.0, 0.0, 0.0};
    struct Rows {
        v4f r[8];
        float g[8];
    };
    auto load = [&](Rows &x, long long n) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const long long at = n + 8 * rg + e;
            const bool ok = at < n1;
            const long long row = ok ? at : n0;
            x.r[e] = *reinterpret_cast<const v4f *>(Rc + (size_t)row * Mpad);
            x.g[e] = ok && cok ? Go[row] : 0.0f;
        }
    };
    auto store = [&](const Rows &x, long long n) {
        if (bsum) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const long long at = n + 8 * rg + e;
                const float m = at < n1 && cok ? Go[NS + at] : 0.0f;
#pragma unroll
                for (int c = 0; c < 4; ++c) bacc[c] += (double)(m * x.r[e][c]);
            }
        }
        uint4 *out = terms + (size_t)(tile * 2 + (rg >> 1)) * 3 * 64;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = wgt ? mul_rounded(x.g[e], x.r[e][c]) : cok ? x.r[e][c] : 0.0f;
            Terms t;
            split_terms(t, v);
            const int p = (4 * (cq & 7) + c + 32 * (rg & 1)) ^ (tile & 3);
#pragma unroll
            for (int k = 0; k < 3; ++k) out[k * 64 + p] = t.t[k];
        }
    };
    auto operand = [&](int tl, int step, int term) {
        return terms[(size_t)((tl * 2 + step) * 3 + term) * 64 + (lane ^ (tl & 3))];
    };
    if (n0 < n1) {
        Rows x;
        load(x, n0);
        for (long long n = n0; n < n1; n += 32) {
            __syncthreads();   // the last turn's readers are done
            store(x, n);
            __syncthreads();
            if (n + 32 < n1) load(x, n + 32);
            __builtin_amdgcn_sched_barrier(0);   // the loads stay ahead of the products
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                v16f t[2] = {v16f{}, v16f{}};
                auto mma = [&](const uint4 (&x)[2], const uint4 &y) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        t[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf(x[i]), as_bf(y), t[i], 0, 0, 0);
                };
                const int tj = 4 + 2 * (w & 1) + j;
#pragma unroll
                for (int step = 0; step < 2; ++step) {
                    uint4 h[2], m[2], l[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        h[i] = operand(2 * (w >> 1) + i, step, 0);
                        m[i] = operand(2 * (w >> 1) + i, step, 1);
                        l[i] = operand(2 * (w >> 1) + i, step, 2);
                    }
                    const uint4 bh = operand(tj, step, 0), bm = operand(tj, step, 1);
                    mma(h, operand(tj, step, 2));
                    mma(l, bh);
                    mma(m, bm);
                    mma(h, bm);
                    mma(m, bh);
                    __builtin_amdgcn_sched_barrier(0);   // one step's operands at a time
                }
#pragma unroll
                for (int step = 0; step < 2; ++step) {
                    const uint4 h[2] = {operand(2 * (w >> 1), step, 0), operand(2 * (w >> 1) + 1, step, 0)};
                    mma(h, operand(tj, step, 0));
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][j][e] += t[i][e];
            }
        }
    }
    if (bi == bj) {   // the four row groups' sums of m r, in order
        double *bs = reinterpret_cast<double *>(terms);   // [row group][128]
        __syncthreads();
        if (wgt) {
#pragma unroll
            for (int c = 0; c < 4; ++c) bs[rg * 128 + 4 * cq + c] = bacc[c];
        }
        __syncthreads();
        const int i = threadIdx.x;
        if (i < 128 && 128 * bi + i < Mpad)
            a.bpart[((size_t)slot * 2 + o) * Mpad + 128 * bi + i] = (bs[i] + bs[128 + i]) + (bs[256 + i] + bs[384 + i]);
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

// Fixed-order final sums, a workgroup each: dU[k][c] (blocks 0 to 2T - 1), the ten hyperparameter
// derivatives, J = mean smoothed cost (the last).  log ell_d = direct (through k) +
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

int grad_split_capacity(int Mpad) {
    const size_t lds = grad_forward_lds(Mpad);
    int dev = 0, ncu = 0, per_cu = 0;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(grad_forward_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(grad_forward_kernel),
                                                     kThreads, lds) != hipSuccess)
        return 0;
    return per_cu * ncu;
}

static hipError_t launch_forward(const GradArgs &a, ForwardMode mode, hipStream_t st) {
    const size_t lds = grad_forward_lds(a.gp.Mpad);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(grad_forward_kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int nwg = (a.K + kB - 1) / kB;
    hipLaunchKernelGGL(grad_forward_kernel, dim3(mode == kForwardSplit ? 2 * nwg : nwg), dim3(kThreads), lds, st, a,
                       (int)mode);
    return hipGetLastError();
}

hipError_t launch_grad(const GradArgs &a, hipStream_t st) {
    hipError_t e;
    if (a.split) {
        const int nwg = (a.K + kB - 1) / kB;
        if (!a.xrec || !a.repair || 2 * nwg > grad_split_capacity(a.gp.Mpad)) return hipErrorInvalidValue;
        const size_t n_rec = (size_t)nwg * kGradXchPerBlock;   // > nwg
        hipLaunchKernelGGL(grad_clear_kernel, dim3((unsigned)((n_rec + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                           a.xrec, n_rec, a.repair, nwg);
        if ((e = launch_forward(a, kForwardSplit, st)) != hipSuccess) return e;
        if ((e = launch_forward(a, kForwardRepair, st)) != hipSuccess) return e;   // the repair launch
    } else if ((e = launch_forward(a, kForwardWhole, st)) != hipSuccess) {
        return e;
    }
    const int nblk = (a.Kc + 63) / 64;
    const int lds = grad_gp_lds(a.gp.Mpad);
    if ((e = hipFuncSetAttribute(reinterpret_cast<const void *>(grad_gp_kernel),
                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds)) != hipSuccess)
        return e;
    for (int c = 0; c < a.nchunk; ++c) {
        const int kc = a.K - c * a.Kc < a.Kc ? a.K - c * a.Kc : a.Kc;
        const long long N = (long long)a.T * kc;
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
