// K-sample x T-step rollout of the GP-augmented chance-constrained MPPI
// controller on gfx950 (Alg. 1 Step 1 with Eqs. 1-3, 10, 11-16): the kernels around
// rollout_core (one workgroup per sample block; FP32 and BF16x3 forms), their output
// split and persistent batch, and the GP prediction.
#include "rollout_core.hpp"

namespace gpmppi {

using namespace core;

// ---- output split
// The two GP outputs of one sample block can run on two workgroups of a doubled
// grid, workgroup 2 blk + r computing output r: where the sample count alone
// would leave compute units idle, this halves each workgroup's kernel-vector
// and variance work.  Role 0 carries the full sample state, the covariance, the
// obstacle loop and the cost; role 1 the pose and velocities that its queries
// and the polyline loop need.  Both loops are dealt over all of a role's waves.
// The roles exchange, per step, the two GP means, the second output's variance
// and the squared distance to the polyline as 64-bit records (value, tag)
// stored and loaded at agent scope, one
// record per sample: a record is valid once its tag names this launch's epoch
// and the step, so no flag and no store-completion wait is needed.  Slots cycle
// over four steps (a writer runs at most two steps ahead of a slot's reader).
// The values reach the same arithmetic as in rollout_core, so the results are
// bitwise those of the unsplit kernel.  The launcher admits the shape only
// where the whole doubled grid fits the device at once, but other work on the
// device can still keep one role waiting: every wait is bounded
// (RolloutArgs::xspin polls), and a workgroup whose wait gives up abandons the
// exchange, marks its block in RolloutArgs::repair and sets the exchange
// time-out bit of the context's status word (its partner, waiting in turn,
// does the same).  The launcher follows every split launch with a repair
// launch of the unsplit kernel that recomputes exactly the marked blocks (the
// same results bit for bit) and exits at once elsewhere.

constexpr int kXvFail = 3 * 32;   // xv slot of wave 0's "an exchange wait gave up" flag

__device__ __forceinline__ uint32_t xch_tag(uint32_t epoch, int k) {
    return ((epoch & 0x7FFFFu) << 13) | (uint32_t)(k + 1);   // k + 1 <= 4096 < 2^13
}

// LDS of the split kernel: one output's k, its row factors and partial sums.
struct SplitPlan {
    int rs, mp, vp, ored, bytes;
};
template <int PREC, int NW>
__host__ __device__ constexpr SplitPlan split_plan(int NT) {
    SplitPlan p{};
    p.rs = NT * 2 * kTerms * 1024;
    p.mp = p.rs + (PREC == GPMPPI_FP32 ? NT * 32 * 4 : 0);
    p.vp = p.mp + kClasses * 32 * 4;
    p.ored = p.vp + NT * 32 * 4;
    p.bytes = p.ored + 2 * NW * 32 * 4;
    return p;
}

// Role `role` of sample block blk (32 samples); see above.
template <int PREC, int NW>
__device__ __forceinline__ void rollout_block_split(const RolloutArgs &a, int blk, int role, unsigned char *lds,
                                                    float *xv) {
    constexpr int G = 2, B = 32;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sl = lane % B, sg = blk * B + sl;
    const int K = a.K, NT = a.gp.NT;
    const GpCore gp{a.gp, a.terms};
    const bool writer = role == 0 && sg < K && w == 0 && lane < B;
    const SplitPlan pl = split_plan<PREC, NW>(NT);
    float *rs = reinterpret_cast<float *>(lds + pl.rs) - role * NT * 32;   // rows of this role's output
    float *mp = reinterpret_cast<float *>(lds + pl.mp);
    float *vp = reinterpret_cast<float *>(lds + pl.vp);
    float *ored = reinterpret_cast<float *>(lds + pl.ored);

    NoiseParams np = a.noise;
    {
        uint64_t seed = a.seed;
        if (a.step_counter) seed += (uint64_t)(*a.step_counter);
        np.key0 = (uint32_t)seed;
        np.key1 = (uint32_t)(seed >> 32);
    }
    const Dyn dy = a.dyn;
    const CostWeights cw = a.cw;
    const Geometry &geo = a.geo;
    const float dt = dy.dt;
    const uint32_t epoch =
        __builtin_amdgcn_readfirstlane(__hip_atomic_load(a.xep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    unsigned long long *rec = a.xrec + (size_t)blk * kXchRecPerBlock;
    // kind: m0, m1, s2 of output 1, squared polyline distance at x_{k+1}
    auto slot = [&](int k, int kind) { return rec + ((k & 3) * 4 + kind) * 32; };
    bool broken = false;
    bool alone = false;   // set (uniformly) when an exchange wait gave up: the block is left to the repair
    const int spin = a.xspin;

    float X = a.x0[0], Y = a.x0[1], th = a.x0[2], v = a.x0[3], w_ = a.x0[4];
    Cov P{};
    float S_ = 0.0f, Sc = 0.0f, disc = 1.0f;
    float dgoal_min = INFINITY;
    if (writer && a.trace.x_d) {
        a.trace.x_d[0 * K + sg] = X;
        a.trace.x_d[1 * K + sg] = Y;
        a.trace.x_d[2 * K + sg] = th;
        a.trace.x_d[3 * K + sg] = v;
        a.trace.x_d[4 * K + sg] = w_;
    }
    if (writer && a.trace.sxy_d) {
        a.trace.sxy_d[0 * K + sg] = 0.0f;
        a.trace.sxy_d[1 * K + sg] = 0.0f;
        a.trace.sxy_d[2 * K + sg] = 0.0f;
    }
    if constexpr (PREC == GPMPPI_FP32)
        for (int i = tid; i < NT * 32; i += 64 * NW) rs[role * NT * 32 + i] = gp.t.wrs[role * NT * 32 + i];
    const WTerms<PREC> wt = wterms<PREC>(gp, lane);
    const UnitList ul = unit_list<NW>(w, NT, 1, role, a.rotate ? blk : 0);
    // this role's output at query q: mean (complete after the barrier), then the variance
    auto mean_of = [&](const float q[4]) {
        GenIn<PREC> in;
        if (w < NT) gen_load<PREC>(in, gp, role, w, lane);
        gen_output<PREC, G, NW>(gp, role, q, w, lane, lds, mp, in,
                                [&](GenIn<PREC> &t, int jt) { gen_load<PREC>(t, gp, role, jt, lane); });
        __syncthreads();
        return gp_mean_of(mp, B, sl);
    };
    WFrag<PREC> none[1];   // every block of W streams from L2 each step
    UnitCursor<true> first;
    resident_load<PREC, 0>(none, wt, first, ul);
    auto contract = [&]() {
        walk_units<PREC, G, 0, true>(wt, none, first, lane, ul, lds, role, NT, rs, vp - role * NT * B);
    };

    StageIn prev{};        // role 0: the previous step's cost inputs, completed by that step's s2 of output 1
    float s20_prev = 0.0f;
    for (int k = 0; k < a.T; ++k) {
        const uint32_t tag = xch_tag(epoch, k);
        const float2 u = sampled_control(np, k, sg, a.U[2 * k], a.U[2 * k + 1]);
        const float q[4] = {v, w_, u.x, u.y};
        float sth, cth;
        sincosf(th, &sth, &cth);
        if (role == 1) {
            advance_pose(dy, v, w_, sth, cth, X, Y, th);
            __syncthreads();   // the previous step's k-operand and loop-result readers are done
            const float m1 = mean_of(q);
            if (w == 0) xch_put(slot(k, 1), lane, m1, tag);
            contract();
            world_share<NW, B>(geo, w, lane, X, Y, 0.0f, 0.0f, 0.0f, 0.0f, ored, true, false);
            if (w == 0) {
                const float m0 = xch_get(slot(k, 0), lane, tag, spin, broken);
                if (lane < 32) xv[lane] = m0;
                if (lane == 0) xv[kXvFail] = broken ? 1.0f : 0.0f;
            }
            __syncthreads();
            if (xv[kXvFail] != 0.0f) {   // the partner did not answer: leave the block to the repair
                alone = true;
                break;
            }
            if (w == 0) {
                xch_put(slot(k, 2), lane, gp_variance<PREC>(gp, 1, row_classes(vp, NT, B, sl)), tag);
                if (geo.path_kind != 0) {
                    float best = INFINITY;
#pragma unroll
                    for (int p = 0; p < NW; ++p) best = fminf(best, ored[p * B + sl]);
                    xch_put(slot(k, 3), lane, best, tag);
                }
            }
            step_velocities(dy, u, xv[sl], m1, v, w_);
            continue;
        }

        // ---- role 0: position and heading (Eqs. 1, 10)
        const StepJac jac = step_jacobian(dy, v, sth, cth);
        advance_pose(dy, v, w_, sth, cth, X, Y, th);
        __syncthreads();
        const float m0 = mean_of(q);
        if (w == 0) xch_put(slot(k, 0), lane, m0, tag);

        // ---- chance-constraint geometry at (x_{k+1}, Sigma_{k+1}) (Eqs. 13-16): the position
        // block of A Sigma A^T does not involve the second output's variance of step k - 1,
        // which arrives during this step's contraction
        float sa, sb, sc;
        propagate_pos_block(P, jac, sa, sb, sc);
        if (a.tight_sxy) {
            sa = a.tight_sxy[3 * (k + 1)];
            sb = a.tight_sxy[3 * (k + 1) + 1];
            sc = a.tight_sxy[3 * (k + 1) + 2];
        }
        const float lmax = lambda_max(sa, sb, sc);
        contract();
        world_share<NW, B>(geo, w, lane, X, Y, sa, sb, sc, lmax, ored, false, true);
        if (w == 0) {
            const float m1 = xch_get(slot(k, 1), lane, tag, spin, broken);
            const uint32_t tp = xch_tag(epoch, k - 1);
            const float s21p = k > 0 ? xch_get(slot(k - 1, 2), lane, tp, spin, broken) : 0.0f;
            const float bestp = k > 0 && geo.path_kind != 0 ? xch_get(slot(k - 1, 3), lane, tp, spin, broken) : 0.0f;
            if (lane < 32) {
                xv[lane] = m1;
                xv[32 + lane] = s21p;
                xv[64 + lane] = bestp;
            }
            if (lane == 0) xv[kXvFail] = broken ? 1.0f : 0.0f;
        }
        __syncthreads();
        if (xv[kXvFail] != 0.0f) {   // the partner did not answer: leave the block to the repair
            alone = true;
            break;
        }
        const float s20 = gp_variance<PREC>(gp, 0, row_classes(vp, NT, B, sl));
        const float m1 = xv[sl];
        if (k > 0) {   // step k - 1 completed: its second variance into Sigma_ww, its lane distance, its cost
            const float s21p = xv[32 + sl];
            add_gp_variance(P.p44, dt, s21p);
            if (geo.path_kind != 0) prev.dl = sqrtf(xv[64 + sl]);
            core_stage_cost(cw, geo, prev, s20_prev, s21p, disc, S_, Sc);
            if (writer) {
                write_variances(a.trace, K, sg, k - 1, s20_prev, s21p);
                write_margins(a.trace, K, sg, k - 1, prev);
            }
        }
        propagate_cov(P, jac);
        step_velocities(dy, u, m0, m1, v, w_);
        add_gp_variance(P.p33, dt, s20);
        prev = stage_geometry(geo, cw, X, Y, v, lmax, dgoal_min);
#pragma unroll
        for (int p = 0; p < NW; ++p) prev.om = fminf(prev.om, ored[(NW + p) * B + sl]);
        s20_prev = s20;
        if (writer) write_step(a.trace, K, sg, k, X, Y, th, v, w_, P, m0, m1, u);
    }
    if (role == 0 && !alone) {
        const uint32_t tl = xch_tag(epoch, a.T - 1);
        const float s21p = xch_get(slot(a.T - 1, 2), lane, tl, spin, broken);
        if (geo.path_kind != 0) prev.dl = sqrtf(xch_get(slot(a.T - 1, 3), lane, tl, spin, broken));
        alone = __syncthreads_or(broken) != 0;
        if (!alone) {
            core_stage_cost(cw, geo, prev, s20_prev, s21p, disc, S_, Sc);
            if (writer) {
                write_variances(a.trace, K, sg, a.T - 1, s20_prev, s21p);
                write_margins(a.trace, K, sg, a.T - 1, prev);
            }
            if (cw.w_term != 0.0f && !(dgoal_min <= cw.goal_tol)) {
                const float yk = cw.w_term - Sc;
                S_ = S_ + yk;
            }
            if (writer) a.costs[sg] = S_;
        }
    }
    if (alone && tid == 0) {   // hand the block to the repair launch that follows
        __hip_atomic_store(a.repair + blk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (a.flags)
            __hip_atomic_fetch_or(a.flags, GPMPPI_FLAG_EXCHANGE_TIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the last workgroup to finish advances the epoch for the next launch
    __syncthreads();
    if (tid == 0) {
        const uint32_t n = __hip_atomic_fetch_add(a.xep + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (n == gridDim.x - 1) {
            __hip_atomic_store(a.xep + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a.xep, epoch + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <int PREC, int NW>
__global__ __launch_bounds__(64 * NW) void rollout_split_kernel(RolloutArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ float xv[kXvFail + 1];
    const int role = __builtin_amdgcn_readfirstlane((int)(blockIdx.x & 1));
    rollout_block_split<PREC, NW>(a, blockIdx.x >> 1, role, lds, xv);
}

// a.repair == NULL: every block.  Otherwise the repair launch after an output
// split (32-sample blocks): only the blocks the split launch marked, whose marks it clears.
template <int PREC, int G, int LAYOUT>
__global__ __launch_bounds__(64 * kCoreWaves) void rollout_kernel(RolloutArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];
    if (G == 2 && a.repair &&
        __hip_atomic_load(a.repair + blockIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u)
        return;
    rollout_core<PREC, G, LAYOUT>(a, blockIdx.x, lds);
    if (G == 2 && a.repair && threadIdx.x == 0)
        __hip_atomic_store(a.repair + blockIdx.x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The problems of a batch, read-only for the whole launch: through the constant
// address space their fields come in by scalar loads the compiler may repeat
// where they are used, as a kernel argument's do, instead of vector loads kept
// live in registers across the item.
typedef const RolloutArgs __attribute__((address_space(4))) ConstRolloutArgs;

// Persistent rollout of many independent problems: every workgroup takes
// (problem, sample block) items from a shared counter until the list (sorted
// longest first) is exhausted.  Results do not depend on which workgroup
// runs an item.  *counter must be 0 at launch.  Problems whose whole layout fits run
// 32-sample blocks of it; GS > 0: the others run blocks of 16 GS samples of the serial or sweep
// layout.
template <int PREC, int GS>
__global__ __launch_bounds__(64 * kCoreWaves) void rollout_batch_kernel(ConstRolloutArgs *probs, const int2 *items,
                                                                         int n_items, uint32_t *counter) {
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int next_item;
    for (;;) {
        __syncthreads();   // every thread has read the previous item
        if (threadIdx.x == 0) next_item = (int)atomicAdd(counter, 1u);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(next_item);
        if (it >= n_items) break;
        const int2 pb = items[it];
        const int p = __builtin_amdgcn_readfirstlane(pb.x);
        const int b = __builtin_amdgcn_readfirstlane(pb.y);
        const RolloutArgs &a = *(const RolloutArgs *)&probs[p];
        if (a.gp.NT <= kResidentTiles) {
            rollout_core<PREC, 2, kWholeResident>(a, b, lds);
        } else {
            if constexpr (GS == 2) rollout_core<PREC, 2, kSerial>(a, b, lds);
            if constexpr (GS == 4) {
                if (a.gp.NT <= serial_tiles<PREC>()) rollout_core<PREC, 4, kSerial>(a, b, lds);
                else rollout_core<PREC, 4, kSweep>(a, b, lds);
            }
        }
    }
}

template <int PREC, int G>
__global__ __launch_bounds__(kThreads) void gp_predict_kernel(GpDev g, const float *q, int n, float *mean,
                                                              float *var) {
    using S = Shapes<PREC, G>;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ float pred[S::rparts * S::B];
    __shared__ float vred[kWaves * S::B];
    const int tid = threadIdx.x;
    const int lane = tid & 63, w = tid >> 6;
    const int sl = lane % S::B;
    const int part = (G == 2) ? w : 2 * w + (lane >> 5);
    const int sg = blockIdx.x * S::B + sl;
    const int sc = sg < n ? sg : n - 1;
    const float4 qq = reinterpret_cast<const float4 *>(q)[sc];
    const float qv[4] = {qq.x, qq.y, qq.z, qq.w};
    const size_t zs_off = G * kgroup_bytes<PREC>(g.Mpad);
    if constexpr (mfma_gen<PREC>()) {
        stage_alpha<kWaves>(g, lds, zs_off);
    } else if constexpr (!scalar_inputs<G>()) {
        StagedInputs st;
        stage_load<PREC>(st, g, 0);
        stage_store<PREC>(st, g, lds, zs_off);
    }
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        __syncthreads();
        const float qs[4] = {qv[0] * g.scale[o][0], qv[1] * g.scale[o][1], qv[2] * g.scale[o][2],
                             qv[3] * g.scale[o][3]};
        float m, s2;
        gp_output<PREC, G>(g, o, o == 0 ? 1 : -1, qs, part, sl, false, 0, blockIdx.x, lds, pred, vred, m, s2);
        if (sg < n && w == 0 && lane < S::B) {
            mean[(size_t)o * n + sg] = m;
            var[(size_t)o * n + sg] = s2;
        }
    }
}

size_t rollout_lds_bytes(int precision, int G, int Mpad) {
    switch (precision) {
        case GPMPPI_FP32: return G == 2 ? dyn_lds_bytes<GPMPPI_FP32, 2>(Mpad) : dyn_lds_bytes<GPMPPI_FP32, 1>(Mpad);
        case GPMPPI_BF16: return G == 2 ? dyn_lds_bytes<GPMPPI_BF16, 2>(Mpad) : dyn_lds_bytes<GPMPPI_BF16, 1>(Mpad);
        default: return G == 2 ? dyn_lds_bytes<GPMPPI_BF16X3, 2>(Mpad) : dyn_lds_bytes<GPMPPI_BF16X3, 1>(Mpad);
    }
}

// Sample groups of 32 the launch shape allows: two when two groups' k operand of one
// output (and the staged inputs of the prediction kernel) fit the 160 KB LDS of a CDNA4
// compute unit, else one.
static int groups_for(int precision, int Mpad) {
    return rollout_lds_bytes(precision, 2, Mpad) <= 160 * 1024 - 8 * 1024 ? 2 : 1;
}

int rollout_groups(int precision, int Mpad) { return groups_for(precision, Mpad); }

template <typename F>
static hipError_t set_lds(F *fn, size_t bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// The block of more row tiles than the whole layouts hold.  64 samples, 8193 of them, T = 10, serial
// against sweep where the serial layout's k fits LDS: FP32 M = 300 189 us against 264, 448 263 against
// 317; BF16x3 300 182 against 239, 512 278 against 313.
template <int PREC>
static CoreShape long_shape(int NT, bool big) {
    if (!big) return CoreShape{2, kSerial};
    return CoreShape{4, NT <= serial_tiles<PREC>() ? kSerial : kSweep};
}

// The block of one problem: the smallest that still gives every compute unit at most one
// workgroup, as the horizon is a serial chain and a block's step gets longer with its
// samples; 64 samples where the blocks outnumber the compute units anyway.  big: 64-sample
// blocks are allowed.  A rollout on 256 compute units, FP32 (BF16x3 within 13 % and on the same
// side unless said):
//   16 samples against 32, T = 20: resident M = 64 K = 4096 67 us, 94; K = 4097 123, 94;
//     M = 256 106, 149 and 198, 150; streamed against serial M = 300 167, 256 and 309, 255;
//     M = 448 248, 343 and 448, 343 (BF16x3 M = 576 345, 413 and 640, 414)
//   32 samples against 64, T = 10: M = 448 K = 8192 191, 263; K = 8193 352, 263; M = 700 331, 548
//     and 556, 543; M = 1024 603, 932 and 1059, 931; K = 16384 1141, 1023.  M = 700 is level up to
//     K = 16384 (613, 614; BF16x3 560, 580).
template <int PREC>
static CoreShape core_shape_t(int NT, int K, bool big, int cus) {
    const int whole = NT <= kResidentTiles ? kWholeResident : kWholeStream;
    const bool w1 = core_plan<PREC, 1, kWholeStream>(NT).bytes <= kCoreLdsMax;
    const long long n16 = (K + 15) / 16;
    if (w1 && n16 <= cus) return CoreShape{1, whole};
    if (whole == kWholeResident) return CoreShape{2, whole};
    return long_shape<PREC>(NT, big && n16 > 2LL * cus);
}

CoreShape core_shape(int precision, int Mpad, int K, int groups, int cus) {
    const bool big = groups == groups_for(precision, Mpad);   // the largest group count: 64-sample blocks allowed
    return precision == GPMPPI_FP32 ? core_shape_t<GPMPPI_FP32>(Mpad / 32, K, big, cus)
                                    : core_shape_t<GPMPPI_BF16X3>(Mpad / 32, K, big, cus);
}

// A batched problem's block (see rollout_batch_kernel); big: the batch's blocks of more than
// kResidentTiles row tiles hold 64 samples.
CoreShape batch_shape(int precision, int Mpad, bool big) {
    if (Mpad / 32 <= kResidentTiles) return CoreShape{2, kWholeResident};
    return precision == GPMPPI_FP32 ? long_shape<GPMPPI_FP32>(Mpad / 32, big) : long_shape<GPMPPI_BF16X3>(Mpad / 32, big);
}

template <int PREC>
static int core_lds_t(int NT, CoreShape s) {
    if (s.layout == kSweep) return core_plan<PREC, 4, kSweep>(NT).bytes;
    if (s.layout == kSerial)
        return s.G == 4 ? core_plan<PREC, 4, kSerial>(NT).bytes : core_plan<PREC, 2, kSerial>(NT).bytes;
    return s.G == 1 ? core_plan<PREC, 1, kWholeStream>(NT).bytes : core_plan<PREC, 2, kWholeResident>(NT).bytes;
}

int core_lds(int precision, int Mpad, CoreShape s) {
    return precision == GPMPPI_FP32 ? core_lds_t<GPMPPI_FP32>(Mpad / 32, s) : core_lds_t<GPMPPI_BF16X3>(Mpad / 32, s);
}

template <int PREC, int G, int LAYOUT>
static hipError_t launch_core(const RolloutArgs &args, hipStream_t st) {
    RolloutArgs a = args;
    int lds = core_lds_t<PREC>(a.gp.NT, CoreShape{G, LAYOUT});
    const long long world = 20LL * a.geo.P + 16LL * a.geo.n_obs;
    a.world_lds = G == 1 && lds + world <= kCoreLdsMax;
    if (a.world_lds) lds += (int)world;
    if (lds > kCoreLdsMax) return hipErrorInvalidValue;
    hipError_t e = set_lds(rollout_kernel<PREC, G, LAYOUT>, lds);
    if (e != hipSuccess) return e;
    const dim3 grid((a.K + 16 * G - 1) / (16 * G));
    hipLaunchKernelGGL((rollout_kernel<PREC, G, LAYOUT>), grid, dim3(64 * kCoreWaves), lds, st, a);
    return hipGetLastError();
}

template <int PREC>
static hipError_t launch_core_p(const RolloutArgs &a, CoreShape s, hipStream_t st) {
    if (s.layout == kSweep) return launch_core<PREC, 4, kSweep>(a, st);
    if (s.layout == kSerial)
        return s.G == 4 ? launch_core<PREC, 4, kSerial>(a, st) : launch_core<PREC, 2, kSerial>(a, st);
    if (s.layout == kWholeStream) return launch_core<PREC, 1, kWholeStream>(a, st);
    return s.G == 1 ? launch_core<PREC, 1, kWholeResident>(a, st) : launch_core<PREC, 2, kWholeResident>(a, st);
}

static int device_cus() {
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
        return 1;
    return ncu;
}

// Largest sample count whose split launch at this shape can be resident at once.
template <int PREC, int NW>
static int split_capacity_t(int Mpad) {
    const int lds = split_plan<PREC, NW>(Mpad / 32).bytes;
    int per_cu = 0;
    if (lds > kCoreLdsMax - 1024 || set_lds(rollout_split_kernel<PREC, NW>, lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu,
                                                     reinterpret_cast<const void *>(rollout_split_kernel<PREC, NW>),
                                                     64 * NW, lds) != hipSuccess)
        return 0;
    return 32 * (per_cu * device_cus() / 2);
}

template <int PREC, int NW>
static hipError_t launch_rollout_split_t(const RolloutArgs &a, hipStream_t st) {
    if (!a.xrec || !a.xep || !a.repair) return hipErrorInvalidValue;
    if (a.K > split_capacity_t<PREC, NW>(a.gp.Mpad))
        return hipErrorCooperativeLaunchTooLarge;   // both roles of every block resident together
    const int nblk = (a.K + 31) / 32;
    const SplitPlan plan = split_plan<PREC, NW>(a.gp.NT);
    hipLaunchKernelGGL((rollout_split_kernel<PREC, NW>), dim3(2 * nblk), dim3(64 * NW), plan.bytes, st, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // the repair launch: the unsplit kernel recomputes the blocks whose exchange gave up
    return launch_core_p<PREC>(a, CoreShape{2, a.gp.NT <= kResidentTiles ? kWholeResident : kSerial}, st);
}

template <int PREC>
static hipError_t launch_rollout_p(const RolloutArgs &a, int groups, int NW, int split, hipStream_t st) {
    if (split) return NW == 8 ? launch_rollout_split_t<PREC, 8>(a, st) : launch_rollout_split_t<PREC, kWaves>(a, st);
    RolloutArgs b = a;
    b.repair = nullptr;   // an unsplit launch computes every block
    return launch_core_p<PREC>(b, core_shape(PREC, a.gp.Mpad, a.K, groups, device_cus()), st);
}

template <int PREC, int GS>
static hipError_t launch_rollout_batch_t(const RolloutArgs *probs, const int2 *items, int n_items, uint32_t *counter,
                                         int lds, int grid, hipStream_t st) {
    hipError_t e = set_lds(rollout_batch_kernel<PREC, GS>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((rollout_batch_kernel<PREC, GS>), dim3(grid), dim3(64 * kCoreWaves), lds, st,
                       (ConstRolloutArgs *)probs, items, n_items, counter);
    return hipGetLastError();
}

template <int PREC>
static hipError_t launch_rollout_batch_p(const RolloutArgs *probs, const int2 *items, int n_items, uint32_t *counter,
                                         int GS, int lds, int grid, hipStream_t st) {
    if (GS == 4) return launch_rollout_batch_t<PREC, 4>(probs, items, n_items, counter, lds, grid, st);
    if (GS == 2) return launch_rollout_batch_t<PREC, 2>(probs, items, n_items, counter, lds, grid, st);
    return launch_rollout_batch_t<PREC, 0>(probs, items, n_items, counter, lds, grid, st);
}

hipError_t launch_rollout_batch(const RolloutArgs *probs_d, const int2 *items_d, int n_items, uint32_t *counter,
                                int precision, int GS, int lds, int grid, hipStream_t st) {
    if ((GS != 0 && GS != 2 && GS != 4) || grid < 1 || lds > kBatchLdsMax) return hipErrorInvalidValue;
    if (precision == GPMPPI_FP32)
        return launch_rollout_batch_p<GPMPPI_FP32>(probs_d, items_d, n_items, counter, GS, lds, grid, st);
    return launch_rollout_batch_p<GPMPPI_BF16X3>(probs_d, items_d, n_items, counter, GS, lds, grid, st);
}

hipError_t launch_rollout(const RolloutArgs &args, int precision, int G, int NW, int split, hipStream_t st) {
    if (NW == kPipeWaves) {
        if (split) return hipErrorInvalidValue;
        RolloutArgs a = args;
        a.repair = nullptr;
        return launch_rollout_pipe(a, precision, G, st);
    }
    if (G < 1 || G > groups_for(precision, args.gp.Mpad) || (NW != kWaves && NW != 8) || (split != 0 && split != 1) ||
        (split && G != 1))
        return hipErrorInvalidValue;
    switch (precision) {
        case GPMPPI_FP32: return launch_rollout_p<GPMPPI_FP32>(args, G, NW, split, st);
        case GPMPPI_BF16: return launch_rollout_bf16(args, G, NW, split, st);
        default: return launch_rollout_p<GPMPPI_BF16X3>(args, G, NW, split, st);
    }
}

int rollout_split_capacity(int precision, int Mpad, int NW) {
    if (NW != kWaves && NW != 8) return 0;
    switch (precision) {
        case GPMPPI_FP32: return NW == 8 ? split_capacity_t<GPMPPI_FP32, 8>(Mpad) : split_capacity_t<GPMPPI_FP32, kWaves>(Mpad);
        case GPMPPI_BF16: return rollout_split_capacity_bf16(Mpad, NW);
        default: return NW == 8 ? split_capacity_t<GPMPPI_BF16X3, 8>(Mpad) : split_capacity_t<GPMPPI_BF16X3, kWaves>(Mpad);
    }
}

template <int PREC, int G>
static hipError_t launch_predict_t(const GpDev &g, const float *q, int n, float *mean, float *var,
                                   hipStream_t st) {
    const size_t lds = dyn_lds_bytes<PREC, G>(g.Mpad);
    hipError_t e = set_lds(gp_predict_kernel<PREC, G>, lds);
    if (e != hipSuccess) return e;
    const dim3 grid((n + 32 * G - 1) / (32 * G));
    hipLaunchKernelGGL((gp_predict_kernel<PREC, G>), grid, dim3(kThreads), lds, st, g, q, n, mean, var);
    return hipGetLastError();
}

hipError_t launch_gp_predict(const GpDev &g, int precision, const float *q, int n, float *mean, float *var,
                             hipStream_t st) {
    const int G = groups_for(precision, g.Mpad);
    switch (precision) {
        case GPMPPI_FP32: return G == 2 ? launch_predict_t<GPMPPI_FP32, 2>(g, q, n, mean, var, st)
                                        : launch_predict_t<GPMPPI_FP32, 1>(g, q, n, mean, var, st);
        case GPMPPI_BF16: return G == 2 ? launch_predict_t<GPMPPI_BF16, 2>(g, q, n, mean, var, st)
                                        : launch_predict_t<GPMPPI_BF16, 1>(g, q, n, mean, var, st);
        default: return G == 2 ? launch_predict_t<GPMPPI_BF16X3, 2>(g, q, n, mean, var, st)
                               : launch_predict_t<GPMPPI_BF16X3, 1>(g, q, n, mean, var, st);
    }
}

}  // namespace gpmppi
