// The rollout of one sample block on gfx950 (Alg. 1 Step 1 with Eqs. 1-3, 10-16):
// GP kernel vectors, means and variances, dynamics, covariance, chance
// constraints and costs, software-pipelined over the horizon.
//
// A workgroup of eight wave64s owns B = 16 G samples (G column groups of the 16x16x32
// matrix-core product).  The horizon is a sequence of phases, one workgroup
// barrier each.  In a phase the waves
//   * contract the variance v = W k of the current chunk of kernel-vector column
//     tiles (W = L^-1 streamed from L2, k from LDS),
//   * generate the next chunk of k into the other LDS buffer,
//   * take their share of the polyline and obstacle loops of the last position,
// and two of them, instead of the loops, integrate pose and covariance and add up the
// cost.  The next query needs only the GP means, which are complete before the
// last chunk's contraction starts, so generation (VALU) and contraction (matrix
// cores) of neighbouring chunks run side by side, half of the waves in the opposite
// order (not in the serial layout).  Everything that does not feed the next query is delayed:
// step k's variances enter the covariance in step k + 1, its constraint loops run
// in step k + 1 and its cost is added in step k + 2.
//
// Layouts of a step:
//   whole  one phase per step: both outputs' k in LDS at once, double-buffered; the
//          row tiles of W of both outputs are dealt to the waves longest first.  Up to
//          256 points all of W stays in registers over the horizon (nine 32x32 blocks a
//          wave), so a step reads nothing from memory; up to 448 points (BF16x3 form 576)
//          five blocks do and the rest come through a four-deep ring
//   serial two phases per step, one per output: all of its k into LDS, a barrier, its row
//          tiles dealt to the waves, W through the four-deep ring.  Nothing of the vector
//          work is hidden, but W streams without a pause: 41K cycles for one output of 1024 points,
//          where 64 bytes a clock, a compute unit's L1, would take 34K.  32 samples up
//          to 1024 points, 64 where their k fits LDS (448 points, BF16x3 form 512).  Odd steps
//          take the outputs in the opposite order: one output's W stays in the XCD's 4 MB of
//          L2 from step to step, both (4.3 MB at 1024 points) would not
//   sweep  chunks of eight column tiles of one output; every wave keeps the
//          accumulators of all its row tiles over the chunks, so LDS holds two chunks
//          only and a block may own 64 samples at M_pad = 1024 (W is streamed once
//          per 64 samples instead of once per 32)
// A step of the serial layout against one of 32-sample blocks in chunks of the sweep's kind (two
// blocks of W in flight per wave and a barrier every sixteen): K = 512, M = 1024 47 us against 68
// (BF16x3; 48 against 71 FP32), K = 2048, M = 700 25 against 38.  64 samples, K = 9000, M = 500:
// 30 against 35 (BF16x3).
//
// Sums are grouped the same way in every layout, block size and wave count, so
// results do not depend on them (bit for bit):
//   mean      eight classes of column tiles (tile % 8) x four octets of points, each
//             one chain of fused multiply-adds; octets, then classes, added pairwise
//   variance  per row tile: quads of rows, then pairwise; row tiles in eight classes
//             (8i + c and 8i + 7 - c for odd i) in ascending order; classes pairwise
//   v = W k   column tiles in ascending order, per tile the products hi*hi, hi*lo, lo*hi
//
// Operands of the contraction:
//   FP32    W and k as two FP16 terms each (hi + lo, 22 significant bits), three
//           products.  k is scaled to (0, 2^15] (k / sf^2 2^15) and every row of W by a
//           power of two into FP16's normal range, so neither term loses bits to the
//           exponent range; the row factors are undone on the FP32 sums.  The FP32
//           matrix cores run at a sixteenth of this rate.  A sum is rounded (towards zero)
//           once per 32 columns and product instead of once per two columns: over rollouts
//           the rms error of s2 against 64 bits is 0.91 (M = 16), 0.84 (64), 0.72 (256),
//           0.70 (512), 0.68 (1024) of that with FP32 products (sn = 0.1 sf; 1.11 at
//           M = 16 and sn = 0.01 sf).  Truncation leaves s2 too large on average by
//           7e-8 sf^2 at M = 1024, a sixth of the rms; gp_predict, FP32 products in one chain,
//           9e-8.
//   BF16x3  two BF16 terms each, three products
// (The BF16 form has its own kernels, rollout_bf16.hip and rollout_pipe.hip.)
//
// Measured (one whole control step, against four-wave workgroups of 32 samples that took
// generation, contraction, constraint loops and state update one after another, with FP32
// operands in the FP32 form):
//   K     T    M     form     before    now      bound now
//   256   20   50    FP32     219 us    62 us    the pose and covariance chain, 3 us a step
//   2500  40   300   FP32     2089 us   317 us   W streamed per 16 samples, vector work of k
//   2048  30   256   FP32 (*) 1954 us   306 us   the chain, twice (nominal sequence first)
//   4096  50   256   BF16x3   953 us    272 us   vector work of k beside the products, 5 us a step
//   16384 100  1024  BF16x3   9.9 ms    9.5 ms   issue of the products, vector work of k between them
//   16384 100  1024  FP32     26.5 ms   10.3 ms  the same
// Counters, matrix cores and vector unit busy of the cycles of the compute units in use: 2 % and 36 %
// (first row), 15 and 42 (second), 15 and 56 (fourth), 51 and 38 at 2.2 GHz (fifth), 47 and 38 (sixth);
// the sweep reads W at 22 bytes a clock, and two waves of a SIMD issue a 16x16x32 product every 22
// cycles or so, of which it keeps the matrix core for 16.
// (*) three terrains, tightening along the nominal sequence.  Geometric ratio of the errors
// against 64 bits of U, costs and weights, now over before, FP32: 1.00, 1.00, 1.00 of the first (60 seeds), 0.97,
// 0.94, 0.89 of the third (60), 0.92, 0.87, 0.73 of the second (12).  Single draws scatter by
// a factor of two either way.
#pragma once
#include "core_step.hpp"
#include "device_common.hpp"
#include "gp_tiles.hpp"
#include "kernels.hpp"

namespace gpmppi {
namespace core {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));

constexpr int kTerms = 2;             // hi and lo terms of W and of k
constexpr float kKScale = 32768.0f;   // scale of the FP32 form's k operand (2^15)
constexpr int kSweepTiles = 8;        // column tiles per chunk of the sweep layout
constexpr int kClasses = 8;           // partial-sum classes of column and row tiles
constexpr int kCoreWaves = 8;         // wave64s per rollout workgroup

template <int PREC>
__device__ __forceinline__ v4f mma16(const uint4 &x, const uint4 &y, v4f acc) {
    if constexpr (PREC == GPMPPI_FP32) {
        v8h p, q;
        __builtin_memcpy(&p, &x, 16);
        __builtin_memcpy(&q, &y, 16);
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(p, q, acc, 0, 0, 0);
    } else {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(x), as_bf(y), acc, 0, 0, 0);
    }
}

// One 32x32 block of W as two 16-row A operands (lane l: row 16 s + l % 16, columns
// 8 (l / 16) .. + 7), read from the [h][lane] words of the packed block.
template <int PREC>
struct WFrag {
    uint4 h[2];
    uint4 l[2];
    __device__ __forceinline__ void pin() {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            pin_word(h[s]);
            pin_word(l[s]);
        }
    }
    static __device__ __forceinline__ void pin_word(uint4 &x) {
        typedef unsigned int v4u __attribute__((ext_vector_type(4)));
        v4u t;
        __builtin_memcpy(&t, &x, 16);
        __asm__ __volatile__("" : "+v"(t));
        __builtin_memcpy(&x, &t, 16);
    }
};

__device__ __forceinline__ int wfrag_voff(int lane) {
    const int q = lane >> 4;
    return (q >> 1) * 1024 + ((lane & 15) + 32 * (q & 1)) * 16;
}

// The packed W terms of both outputs.
template <int PREC>
struct WTerms {
    __amdgpu_buffer_rsrc_t h, l;
    int out;    // bytes per output
    int voff;   // the lane's offset in a block
};

template <int PREC>
__device__ __forceinline__ WTerms<PREC> wterms(const GpCore &g, int lane) {
    const long long bytes = g.d.wb_stride * 32;
    WTerms<PREC> t;
    t.h = uniform_rsrc(PREC == GPMPPI_FP32 ? g.t.wfh : g.d.wbh, bytes);
    t.l = uniform_rsrc(PREC == GPMPPI_FP32 ? g.t.wfl : g.d.wbl, bytes);
    t.out = __builtin_amdgcn_readfirstlane((int)(g.d.wb_stride * 16));
    t.voff = wfrag_voff(lane);
    return t;
}

// Block blk of output o; the block index is wave-uniform.
// have: whether there is one; otherwise the address is that behind the last block, where the resource's
// bounds check returns zeros without a memory access.
template <int PREC>
__device__ __forceinline__ void wfrag_load(WFrag<PREC> &f, const WTerms<PREC> &t, int o, int blk, bool have = true) {
    const int at = __builtin_amdgcn_readfirstlane(have ? (o ? t.out : 0) + blk * 2048 : 2 * t.out);
    f.h[0] = buf_load16(t.h, t.voff, at);
    f.h[1] = buf_load16(t.h, t.voff + 256, at);
    f.l[0] = buf_load16(t.l, t.voff, at);
    f.l[1] = buf_load16(t.l, t.voff + 256, at);
}

// One group's k operand of one column tile, from LDS ([term][lane] of 16 bytes).
template <int PREC>
struct KTerm {
    uint4 h;
    uint4 l;
};
template <int PREC>
__device__ __forceinline__ void kterm_load(KTerm<PREC> &k, const unsigned char *kt, int lane) {
    const uint4 *K = reinterpret_cast<const uint4 *>(kt) + lane;
    k.h = K[0];
    k.l = K[64];
}

// acc[s][g0 ..] += W block . k tile of N groups.  A product's sum waits for the one before it: term by
// term, the two halves of every group lie between two products of one sum.
template <int PREC, int N, int G>
__device__ __forceinline__ void groups_mma(v4f (&acc)[2][G], int g0, const WFrag<PREC> &f, const KTerm<PREC> *k) {
#pragma unroll
    for (int term = 0; term < 3; ++term)
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                acc[s][g0 + i] = mma16<PREC>(term == 2 ? f.l[s] : f.h[s], term == 1 ? k[i].l : k[i].h, acc[s][g0 + i]);
}

// Sum of a wave's four quarters, halves first (every quarter gets it), by exchanges between
// registers: through LDS each of the two steps would wait some hundred cycles.
__device__ __forceinline__ float quarter_sum(float x) {
    const uint32_t a = __float_as_uint(x);
    const auto h = __builtin_amdgcn_permlane32_swap(a, a, false, false);
    const uint32_t b = __float_as_uint(__uint_as_float(h[0]) + __uint_as_float(h[1]));
    const auto q = __builtin_amdgcn_permlane16_swap(b, b, false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// Sum of squares over a finished row tile's 32 rows, per sample (every quarter-wave
// gets the total); FP32 form: rs holds the row factors of this tile.
template <int PREC>
__device__ __forceinline__ float tile_sq(const v4f &a0, const v4f &a1, const v4f &r0, const v4f &r1) {
    float q[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        v4f a = s ? a1 : a0;
        if constexpr (PREC == GPMPPI_FP32) {
            const v4f r = s ? r1 : r0;
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] *= r[e];
        }
        q[s] = fmaf(a[3], a[3], fmaf(a[2], a[2], fmaf(a[1], a[1], a[0] * a[0])));
    }
    return quarter_sum(q[0] + q[1]);
}

// The eight class sums, added pairwise.
__device__ __forceinline__ float class_sum(const float s[kClasses]) {
    return ((s[0] + s[4]) + (s[2] + s[6])) + ((s[1] + s[5]) + (s[3] + s[7]));
}

// Predictive variance of output o from the sum of squares (FP32 form: of W k / sf).
template <int PREC>
__device__ __forceinline__ float gp_variance(const GpCore &g, int o, float sq) {
    const float sf2 = g.d.sf2[o];
    const float lat = PREC == GPMPPI_FP32 ? fmaf(-sf2, sq, sf2) : sf2 - sq;
    return g.d.vscale[o] * (g.d.sn2[o] + fmaxf(0.0f, lat));
}

// ---------------------------------------------------------------- kernel vectors
// Tile jt of 32 points: the lane's octet of kernel values kv[8] (points 8 (l / 16) + r)
// of one 16-sample group goes to LDS as the contraction's B operand.
template <int PREC>
__device__ __forceinline__ void store_octet(unsigned char *kt, int slot, const float kv[8]) {
    uint4 *K = reinterpret_cast<uint4 *>(kt) + slot;
    if constexpr (PREC == GPMPPI_FP32) {
        typedef _Float16 v2h __attribute__((ext_vector_type(2)));
        typedef float v2f __attribute__((ext_vector_type(2)));
        uint32_t h[4], l[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const v2f x = {kv[2 * i], kv[2 * i + 1]};
            const v2h hi = __builtin_convertvector(x, v2h);   // round to nearest even
            const v2f r = {x[0] - (float)hi[0], x[1] - (float)hi[1]};   // exact
            const v2h lo = __builtin_convertvector(r, v2h);
            __builtin_memcpy(&h[i], &hi, 4);
            __builtin_memcpy(&l[i], &lo, 4);
        }
        K[0] = make_uint4(h[0], h[1], h[2], h[3]);
        K[64] = make_uint4(l[0], l[1], l[2], l[3]);
    } else {
        uint32_t h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) h[i] = pack_bf16x2(kv[2 * i], kv[2 * i + 1]);
        K[0] = make_uint4(h[0], h[1], h[2], h[3]);
        uint32_t l[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            l[i] = pack_bf16x2(kv[2 * i] - bf16_to_f32((uint16_t)h[i]),
                               kv[2 * i + 1] - bf16_to_f32((uint16_t)(h[i] >> 16)));
        K[64] = make_uint4(l[0], l[1], l[2], l[3]);
    }
}

// exp2(-|q - z|^2) 2^15 by exact differences.
__device__ __forceinline__ float kval32(const float qs[4], v4f z) {
    const float d0 = qs[0] - z.x, d1 = qs[1] - z.y, d2 = qs[2] - z.z, d3 = qs[3] - z.w;
    float e = -d0 * d0;
    e = fmaf(-d1, d1, e);
    e = fmaf(-d2, d2, e);
    e = fmaf(-d3, d3, e);
    return __builtin_amdgcn_exp2f(e) * kKScale;
}

// Point inputs of a lane's octet of one tile: FP32 form the scaled points, BF16x3 form the
// A operands of the exponent products; alpha (FP32 form: alpha sf^2 / 2^15, for the
// scaled kernel values).
template <int PREC>
struct GenIn {
    v4f z[PREC == GPMPPI_FP32 ? 8 : 1];
    uint4 a[PREC == GPMPPI_FP32 ? 1 : 2];
    v4f al[2];
};

// FP32 form: points z and alpha al of the tile, in global memory or LDS.
__device__ __forceinline__ void gen_load_points(GenIn<GPMPPI_FP32> &t, const v4f *z, const float *al, int lane) {
    const int q = lane >> 4;
#pragma unroll
    for (int r = 0; r < 8; ++r) t.z[r] = z[8 * q + r];
    const v4f *ap = reinterpret_cast<const v4f *>(al) + 2 * q;
    t.al[0] = ap[0];
    t.al[1] = ap[1];
}

template <int PREC>
__device__ __forceinline__ void gen_load(GenIn<PREC> &t, const GpCore &g, int o, int jt, int lane) {
    const size_t p0 = (size_t)o * g.d.Mpad + 32 * jt;
    if constexpr (PREC == GPMPPI_FP32) {
        gen_load_points(t, reinterpret_cast<const v4f *>(g.d.zs) + p0, g.t.alphas + p0, lane);
    } else {
        const uint4 *a = g.t.zop16 + o * g.d.zop_stride + (size_t)jt * 128 + lane;
        t.a[0] = a[0];
        t.a[1] = a[64];
        const v4f *al = reinterpret_cast<const v4f *>(g.d.alpha + p0) + 2 * (lane >> 4);
        t.al[0] = al[0];
        t.al[1] = al[1];
    }
}

// The query of one 16-sample group as the lanes need it: FP32 form the scaled query of
// sample l % 16, BF16x3 form its slots 8 (l / 16) .. + 7 of the exponent product.
template <int PREC>
struct GenQ {
    float qs[PREC == GPMPPI_FP32 ? 4 : 1];
    uint4 b;
};

template <int PREC>
__device__ __forceinline__ void gen_query(GenQ<PREC> &t, const float qs[4], int lane) {
    if constexpr (PREC == GPMPPI_FP32) {
#pragma unroll
        for (int d = 0; d < 4; ++d) t.qs[d] = qs[d];
    } else {
        const float qq = fmaf(qs[3], qs[3], fmaf(qs[2], qs[2], fmaf(qs[1], qs[1], qs[0] * qs[0])));
        uint32_t h[4], m[4], l[4], n[3];
#pragma unroll
        for (int d = 0; d < 4; ++d) split3_bits(qs[d], h[d], m[d], l[d]);
        split3_bits(-qq, n[0], n[1], n[2]);
        const uint32_t one = 0x3f80u;
        const uint2 H = make_uint2(h[0] | h[1] << 16, h[2] | h[3] << 16);
        const uint2 Mm = make_uint2(m[0] | m[1] << 16, m[2] | m[3] << 16);
        const uint2 L = make_uint2(l[0] | l[1] << 16, l[2] | l[3] << 16);
        // slots 0-7: qh qm, 8-15: qh ql, 16-23: qm qh, 24-31: 1 1 1 -qq(h m l) 0 0
        const int q = lane >> 4;
        uint2 a = q == 2 ? Mm : H, b = q == 0 ? Mm : (q == 1 ? L : H);
        if (q == 3) {
            a = make_uint2(one | one << 16, one | n[0] << 16);
            b = make_uint2(n[1] | n[2] << 16, 0u);
        }
        t.b = make_uint4(a.x, a.y, b.x, b.y);
    }
}

// The lane's octet of one tile for one 16-sample group: k into LDS and the mean chain.
template <int PREC>
__device__ __forceinline__ void gen_octet(const GenIn<PREC> &t, const GenQ<PREC> &q, unsigned char *kt, int lane,
                                          float &ms) {
    float kv[8];
    if constexpr (PREC == GPMPPI_FP32) {
#pragma unroll
        for (int r = 0; r < 8; ++r) kv[r] = kval32(q.qs, t.z[r]);
    } else {
        const v4f e0 = mma16<PREC>(t.a[0], q.b, v4f{0.0f, 0.0f, 0.0f, 0.0f});
        const v4f e1 = mma16<PREC>(t.a[1], q.b, v4f{0.0f, 0.0f, 0.0f, 0.0f});
#pragma unroll
        for (int r = 0; r < 8; ++r) kv[r] = __builtin_amdgcn_exp2f(r < 4 ? e0[r & 3] : e1[r & 3]);
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) ms = fmaf(kv[r], t.al[r >> 2][r & 3], ms);
    store_octet<PREC>(kt, lane, kv);
}

// The query scaled by the lengthscales.  Contraction is off: fused into the differences
// of kval32, the product would not be rounded, depending on the code in between.
__device__ __forceinline__ void scaled_query(const GpCore &g, int o, const float q[4], float qs[4]) {
#pragma clang fp contract(off)
#pragma unroll
    for (int d = 0; d < 4; ++d) qs[d] = q[d] * g.d.scale[o][d];
}

// The queries of the G groups: group i's from the lanes of its samples (lane l holds sample
// l % (16 G), scaled query qs).
template <int PREC, int G>
__device__ __forceinline__ void gen_queries(GenQ<PREC> (&gq)[G], const float qs[4], int lane) {
    float qg[G][4];   // gathered together: one LDS round trip
#pragma unroll
    for (int i = 0; i < G; ++i)
#pragma unroll
        for (int d = 0; d < 4; ++d) qg[i][d] = G == 1 ? qs[d] : __shfl(qs[d], 16 * i + (lane & 15), 64);
#pragma unroll
    for (int i = 0; i < G; ++i) gen_query<PREC>(gq[i], qg[i], lane);
}

// One tile for the G groups.  inputs(in) gives the tile's inputs, for each group anew: where they
// come from LDS, reading them again is cheaper than keeping forty registers for them.
template <int PREC, int G, class Inputs>
__device__ __forceinline__ void gen_tile16(const Inputs &inputs, const GenQ<PREC> (&gq)[G], unsigned char *kt, int lane,
                                           float (&ms)[G]) {
#pragma unroll
    for (int i = 0; i < G; ++i) {
        GenIn<PREC> in;
        inputs(in);
        gen_octet<PREC>(in, gq[i], kt + i * kTerms * 1024, lane, ms[i]);
    }
}

// Wave wv's column tiles (classes wv, wv + NW, ...) of output o: k into kb (tile jt at
// jt tile_bytes) and the classes' means into mr[class][B].  in: the inputs of tile wv;
// load(in, jt) fetches a later tile's.
template <int PREC, int G, int NW, class Load>
__device__ __forceinline__ void gen_output(const GpCore &g, int o, const float q[4], int wv, int lane, unsigned char *kb,
                                           float *mr, GenIn<PREC> &in, const Load &load) {
    constexpr int B = 16 * G, S = kTerms;
    constexpr bool kAhead = PREC != GPMPPI_FP32;   // the next tile's inputs (sixteen registers) load beside this one
    float qs[4];
    scaled_query(g, o, q, qs);
    GenQ<PREC> gq[G];
    gen_queries<PREC, G>(gq, qs, lane);
    GenIn<PREC> next = in;
    for (int cl = wv; cl < kClasses; cl += NW) {
        float ms[G];
#pragma unroll
        for (int i = 0; i < G; ++i) ms[i] = 0.0f;
        for (int jt = cl; jt < g.d.NT; jt += kClasses) {
            if constexpr (kAhead) {
                in = next;
                const int jn = jt + kClasses < g.d.NT ? jt + kClasses : cl + NW;
                if (jn < g.d.NT) load(next, jn);
            } else if (jt != wv) {
                load(in, jt);
            }
            gen_tile16<PREC, G>([&](GenIn<PREC> &t) { t = in; }, gq, kb + jt * (G * S * 1024), lane, ms);
        }
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const float t = quarter_sum(ms[i]);
            if (lane < 16) mr[cl * B + 16 * i + lane] = t;
        }
    }
}

// A sample's GP mean from its class means.
__device__ __forceinline__ float gp_mean_of(const float *mr, int B, int s) {
    float c[kClasses];
#pragma unroll
    for (int i = 0; i < kClasses; ++i) c[i] = mr[i * B + s];
    return class_sum(c);
}

// ---------------------------------------------------------------- constraint loops
// Share wv of NS of both loops at (X, Y) with position covariance (sa, sb, sc): lane l
// holds sample l % B; the 64 / B lane groups take different segments and obstacles.
// The least squared segment distance goes to out[wv][B], the least tightened
// obstacle distance to out[NS + wv][B] (minima: the split does not change them).
// seg, inv, obs: the geometry in global memory or LDS.
template <int NS, int B, class Seg, class Inv, class Obs>
__device__ __forceinline__ void world_share(const Geometry &geo, Seg seg, Inv inv, Obs obs, int wv, int lane, float X,
                                            float Y, float sa, float sb, float sc, float lmax, float *out, bool poly,
                                            bool obst) {
    constexpr int LG = 64 / B;
    const int first = LG == 1 ? wv : wv * LG + lane / B;
    if (poly && geo.path_kind != 0) {
        float best = INFINITY;
#pragma unroll 4
        for (int i = first; i < geo.P; i += NS * LG) best = fminf(best, segment_dist2(seg[i], inv[i], X, Y));
#pragma unroll
        for (int m = B; m < 64; m *= 2) best = fminf(best, shfl_xor(best, m));
        if (lane < B) out[wv * B + lane] = best;
    }
    if (obst) {
        float om = INFINITY;
#pragma unroll 2
        for (int j = first; j < geo.n_obs; j += NS * LG) {
            const v4f o = obs[j];
            om = fminf(om, obstacle_distance(X - o.x, Y - o.y, o.z, sa, sb, sc, lmax, geo.z_p));
        }
#pragma unroll
        for (int m = B; m < 64; m *= 2) om = fminf(om, shfl_xor(om, m));
        if (lane < B) out[(NS + wv) * B + lane] = om;
    }
}

// The geometry in global memory: through the scalar cache where a wave's index is uniform.
template <int NS, int B>
__device__ __forceinline__ void world_share(const Geometry &geo, int wv, int lane, float X, float Y, float sa, float sb,
                                            float sc, float lmax, float *out, bool poly, bool obst) {
    if constexpr (B == 64)
        world_share<NS, B>(geo, (const_v4p)geo.seg, (const_fp)geo.seg_inv, (const_v4p)geo.obs, wv, lane, X, Y, sa, sb,
                           sc, lmax, out, poly, obst);
    else
        world_share<NS, B>(geo, reinterpret_cast<const v4f *>(geo.seg), geo.seg_inv,
                           reinterpret_cast<const v4f *>(geo.obs), wv, lane, X, Y, sa, sb, sc, lmax, out, poly, obst);
}

// ---------------------------------------------------------------- LDS plan
struct CorePlan {
    int rs, z, mp, vp, un, geo, ps, cs, ored, bytes;   // byte offsets; the two k buffers come first
    int kbuf;                                  // bytes per k buffer
    int ns;                                    // steps per half of the noise table
};

enum CoreLayout { kWholeResident = 0, kWholeStream = 1, kSweep = 2, kSerial = 3 };

// The whole layouts keep two copies of each small array by step parity; in the others the phases of
// a step separate writers and readers.
constexpr int core_parities(int layout) { return layout == kSweep || layout == kSerial ? 1 : 2; }

template <int PREC, int G, int LAYOUT>
__host__ __device__ constexpr CorePlan core_plan(int NT) {
    constexpr bool SWEEP = LAYOUT == kSweep, SERIAL = LAYOUT == kSerial;
    constexpr int B = 16 * G, NW = kCoreWaves, PP = core_parities(LAYOUT);
    CorePlan p{};
    p.ns = G == 1 ? 16 : G == 2 ? 8 : 2;
    p.kbuf = (SWEEP ? kSweepTiles : SERIAL ? NT : 2 * NT) * G * kTerms * 1024;
    int off = (SERIAL ? 1 : 2) * p.kbuf;
    auto take = [&](int bytes) {
        const int at = off;
        off += (bytes + 15) / 16 * 16;
        return at;
    };
    p.rs = take(PREC == GPMPPI_FP32 && !SWEEP ? 2 * NT * 32 * 4 : 0);
    // FP32 form: points and alpha, of both outputs (whole) or of two chunks (sweep); serial: from memory
    p.z = take(PREC == GPMPPI_FP32 && !SERIAL ? 2 * (SWEEP ? kSweepTiles : NT) * 32 * 20 : 0);
    p.mp = take(PP * 2 * kClasses * B * 4);
    p.vp = take((SERIAL ? 3 : PP * 2) * (SWEEP ? kClasses : NT) * B * 4);
    p.un = take(2 * p.ns * B * 8);
    p.geo = take(PP * 6 * B * 4);
    p.ps = take(16 * B * 4);
    p.cs = take(10 * B * 4);
    p.ored = take(PP * 2 * (NW - 2) * B * 4);
    p.bytes = off;
    return p;
}

constexpr int kCoreLdsMax = 160 * 1024;
constexpr int kBatchLdsMax = kCoreLdsMax - 64;   // the batch kernel keeps its item in LDS too
static_assert(core_plan<GPMPPI_FP32, 4, kSweep>(32).bytes <= kBatchLdsMax, "64-sample blocks fit at M_pad = 1024");
// Row tiles up to which the serial layout of 64-sample blocks fits LDS (FP32 form 14, BF16x3 form 16).
template <int PREC>
__host__ __device__ constexpr int serial_tiles() {
    int nt = 32;
    while (core_plan<PREC, 4, kSerial>(nt).bytes > kBatchLdsMax) --nt;
    return nt;
}
static_assert(core_plan<GPMPPI_FP32, 2, kSerial>(32).bytes <= kBatchLdsMax, "32-sample blocks fit at M_pad = 1024");

// ---------------------------------------------------------------- contraction
// Whole layout.  Units (output o, row tile t) of both outputs, t descending, are dealt
// to the waves in snake order (a tile's work is t + 1 blocks, so the waves' totals
// are within a block or two of each other); 8 bits per unit: t | o << 7.  At most eight units
// a wave (32 row tiles of one output over four waves, or of both over eight): one word, as a
// choice of words would lie in scratch memory, whose read waits for every W block in flight.
struct UnitList {
    uint64_t units;
    int n, blocks;
    __device__ __forceinline__ int at(int i) const { return (int)(units >> (8 * i)) & 0xFF; }
};

// NO outputs (2, or 1: output o1 only) over NW waves.
template <int NW>
__device__ __forceinline__ UnitList unit_list(int w, int NT, int NO, int o1, int rot) {
    UnitList l{0, 0, 0};
    const int total = NO * NT;
    for (int r = 0; r * NW < total; ++r) {
        const int i = r * NW + ((r & 1) ? NW - 1 - w : w);
        if (i >= total) continue;
        const int t = NT - 1 - (NO == 2 ? i >> 1 : i), o = NO == 2 ? i & 1 : o1;
        l.units |= (uint64_t)(t | (o << 7)) << (8 * l.n);
        ++l.n;
        l.blocks += t + 1;
    }
    if (rot && l.n > 1) {   // start at a block-dependent unit
        const int s = rot % l.n;
        uint64_t u = 0;
        for (int i = 0; i < l.n; ++i) u |= (uint64_t)l.at((i + s) % l.n) << (8 * i);
        l.units = u;
    }
    // scalar registers for the cursors
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)l.units) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(l.units >> 32)) << 32;
    return UnitList{u, __builtin_amdgcn_readfirstlane(l.n), __builtin_amdgcn_readfirstlane(l.blocks)};
}

// SCALAR: in scalar registers, whose branches cost less where the loop over the blocks is long;
// the unrolled steps of the resident layout are 2 % faster without them.
template <bool SCALAR>
struct UnitCursor {
    int n, c, t, o, base;
    __device__ __forceinline__ void unit(const UnitList &l) {
        int e = n < l.n ? l.at(n) : 0;   // past the end: row tile 0 (a valid block)
        if constexpr (!SCALAR) __asm__ __volatile__("" : "+v"(e));
        t = e & 0x7F;
        o = e >> 7;
        const int u = t >> 1;
        base = 2 * u * (u + 1) + (t & 1);
        c = 0;
    }
    __device__ __forceinline__ void start(const UnitList &l) {
        n = 0;
        unit(l);
    }
    __device__ __forceinline__ bool next(const UnitList &l) {   // true: the block just left closed its unit
        if (__builtin_expect(++c <= t, 1)) return false;
        ++n;
        unit(l);
        return true;
    }
    __device__ __forceinline__ int block() const { return base + 2 * c; }
};

// A finished unit's sums of squares to vp[(o NT + t) B]; the accumulators start over.
template <int PREC, int G>
__device__ __forceinline__ void unit_finish(v4f (&acc)[2][G], int o, int t, int NT, int lane, const float *rs,
                                            float *vp) {
    v4f r0{}, r1{};
    if constexpr (PREC == GPMPPI_FP32) {
        const v4f *rp = reinterpret_cast<const v4f *>(rs + (o * NT + t) * 32) + (lane >> 4);
        r0 = rp[0];
        r1 = rp[4];
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float q = tile_sq<PREC>(acc[0][g], acc[1][g], r0, r1);
        if (lane < 16) vp[(o * NT + t) * 16 * G + 16 * g + lane] = q;
        acc[0][g] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        acc[1][g] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    }
}

// The wave's units over all their column tiles.  The first RB blocks stay in registers for
// the whole horizon (res, loaded by resident_load); STREAM: the others run through a
// register ring four blocks deep every step.  kb: tile (o, c) at ((o - o0) NT + c)
// tile_bytes; sums of squares to vp[(o NT + t) B].
template <int PREC, int RB, bool SCALAR>
__device__ __forceinline__ void resident_load(WFrag<PREC> (&res)[RB ? RB : 1], const WTerms<PREC> &wt,
                                              UnitCursor<SCALAR> &c, const UnitList &ul) {
    c.start(ul);
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        wfrag_load<PREC>(res[i], wt, c.o, c.block());
        c.next(ul);
    }
    // arrived here: or every step's first use would wait, and for the loads behind it
#pragma unroll
    for (int i = 0; i < RB; ++i) res[i].pin();
}

template <int PREC, int G, int RB, bool STREAM>
__device__ __forceinline__ void walk_units(const WTerms<PREC> &wt, const WFrag<PREC> (&res)[RB ? RB : 1],
                                           const UnitCursor<STREAM> &first, int lane, const UnitList &ul,
                                           const unsigned char *kb, int o0, int NT, const float *rs, float *vp) {
    constexpr int TB = G * kTerms * 1024;
    const int nb = ul.blocks;
    if (nb == 0) return;
    WFrag<PREC> ring[STREAM ? 4 : 1];
    UnitCursor<STREAM> pc = first, mc;
    auto fetch = [&](int r) {
        wfrag_load<PREC>(ring[r], wt, pc.o, pc.block());
        pc.next(ul);
    };
    if constexpr (STREAM) {   // not only where blocks are left: on a way without these loads the waits below would
#pragma unroll                // be for whatever the registers were loaded with last
        for (int r = 0; r < 4; ++r) fetch(r);
    }
    v4f acc[2][G];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int g = 0; g < G; ++g) acc[s][g] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    mc.start(ul);
    KTerm<PREC> kc[G], kn[G];
    // k of the cursor's block (past the end the cursor stands on a valid tile)
    auto kload = [&](KTerm<PREC> (&k)[G], const UnitCursor<STREAM> &c) {
        const unsigned char *kt = kb + ((c.n < ul.n ? c.o - o0 : 0) * NT + c.c) * TB;
#pragma unroll
        for (int g = 0; g < G; ++g) kterm_load<PREC>(k[g], kt + g * kTerms * 1024, lane);
    };
    auto block = [&](const WFrag<PREC> &f) {   // one block, the next one's k a block ahead
        const int t = mc.t, o = mc.o;
        const bool end = mc.next(ul);
        kload(kn, mc);
        if constexpr (STREAM) __builtin_amdgcn_sched_barrier(0);   // not sunk behind the products, to its use
        groups_mma<PREC, G>(acc, 0, f, kc);
        if (end) unit_finish<PREC, G>(acc, o, t, NT, lane, rs, vp);
#pragma unroll
        for (int g = 0; g < G; ++g) kc[g] = kn[g];
    };
    kload(kc, mc);
#pragma unroll
    for (int i = 0; i < RB; ++i)
        if (i < nb) block(res[i]);
    if constexpr (STREAM) {
        int base = RB;
        for (; base + 4 <= nb; base += 4) {   // no way out inside a turn: it would come back to the loop's
#pragma unroll                                // head with other loads last, and the wait there be for all of them
            for (int r = 0; r < 4; ++r) {
                block(ring[r]);
                fetch(r);
                __builtin_amdgcn_sched_barrier(0);   // two blocks' products together would wait for both
            }
        }
#pragma unroll
        for (int r = 0; r < 3; ++r)
            if (base + r < nb) block(ring[r]);
    }
}

// Class c's row tiles of the whole layout, in ascending order.
__device__ __forceinline__ float row_classes(const float *vp, int NT, int B, int s) {
    float cs[kClasses];
#pragma unroll
    for (int c = 0; c < kClasses; ++c) cs[c] = 0.0f;
    for (int i = 0; 8 * i < NT; ++i) {
#pragma unroll
        for (int c = 0; c < kClasses; ++c) {
            const int t = 8 * i + ((i & 1) ? 7 - c : c);
            if (t < NT) cs[c] += vp[t * B + s];
        }
    }
    return class_sum(cs);
}

// Sweep layout.  Wave w owns the row tiles 8i + wc and 8i + 7 - wc (odd i), wc = w or
// 11 - w so that the two waves of a SIMD hold complementary rows; it keeps their
// accumulators over the chunks of an output.  A chunk goes row by row, the row on the
// diagonal last, two blocks per turn of a register ring two blocks deep.  Every turn
// issues the same loads, so the waits count them exactly; a fetch that is not needed (past
// the diagonal or the last row) lies beyond the resource and costs no memory access.
template <int PREC, int G, int NW>
struct Sweep {
    static constexpr int RPW = 4, TB = G * kTerms * 1024;
    static_assert(NW == 8 && kSweepTiles == 8, "row tiles are dealt to eight waves, one per chunk column");
    static constexpr int RD = 2;   // ring depth; four blocks at 64 samples leave no registers for the rest
    WFrag<PREC> ring[RD];
    v4f acc[RPW][2][G];
    int wc, NT, nrows;   // row class, row tiles, the wave's rows

    __device__ __forceinline__ int row(int i) const { return (i & 1) ? 8 * i + 7 - wc : 8 * i + wc; }

    // The block of row i in column c of output o into ring slot q.
    __device__ __forceinline__ void fetch(int q, int i, int o, int c, bool have, const WTerms<PREC> &wt) {
        const int t = row(i), u = t >> 1;
        wfrag_load<PREC>(ring[q], wt, o, 2 * u * (u + 1) + (t & 1) + 2 * c, have && c <= t);
    }
    // The first RD blocks of chunk ci.
    __device__ __forceinline__ void prefetch(int o, int ci, const WTerms<PREC> &wt) {
#pragma unroll
        for (int q = 0; q < RD; ++q) fetch(q, nrows - 1, o, kSweepTiles * ci + q, ci < nrows, wt);
    }
    // The accumulators in registers here (a reload that is still under way would be waited
    // for inside the loops, and the W blocks in flight with it).
    __device__ __forceinline__ void pin() {
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int g = 0; g < G; ++g) __asm__ __volatile__("" : "+v"(acc[i][s][g]));
    }
    // The ring's values are not needed any more (nor live across the code before this point).
    __device__ __forceinline__ void forget() {
        typedef unsigned int v4u __attribute__((ext_vector_type(4)));
        auto drop = [](uint4 &x) {
            v4u t;
            __asm__ __volatile__("" : "=v"(t));
            __builtin_memcpy(&x, &t, 16);
        };
#pragma unroll
        for (int i = 0; i < RD; ++i)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                drop(ring[i].h[s]);
                drop(ring[i].l[s]);
            }
    }
    __device__ __forceinline__ void init(int w, int nt) {
        wc = w < 4 ? w : 11 - w;
        NT = nt;
        nrows = 0;
        for (int i = 0; i < RPW; ++i) nrows += row(i) < nt;
        clear();
    }
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int g = 0; g < G; ++g) acc[i][s][g] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    }
    // Chunk ci of output o from the buffer kb, after prefetch(o, ci).
    __device__ __forceinline__ void chunk(int o, int ci, const unsigned char *kb, int lane, const WTerms<PREC> &wt) {
        constexpr int KB = kTerms * 1024;
        const int ca = kSweepTiles * ci, nc = min(kSweepTiles, NT - ca);
        KTerm<PREC> k[G];   // each group's next column follows its last use
#pragma unroll
        for (int g = 0; g < G; ++g) kterm_load<PREC>(k[g], kb + g * KB, lane);
#pragma unroll
        for (int i = RPW - 1; i >= 0; --i) {
            if (i < ci || i >= nrows) continue;
            const int ncol = min(nc, row(i) - ca + 1);
#pragma unroll 1
            for (int c0 = 0; c0 < ncol; c0 += RD) {
#pragma unroll
                for (int q = 0; q < RD; ++q) {
                    const int c = c0 + q;
                    if (c < ncol) {
#pragma unroll
                        for (int g = 0; g < G; g += 2) {
                            groups_mma<PREC, 2>(acc[i], g, ring[q], k + g);
#pragma unroll
                            for (int e = g; e < g + 2; ++e)
                                kterm_load<PREC>(k[e], kb + (c + 1 < ncol ? (c + 1) * TB : 0) + e * KB, lane);
                            __builtin_amdgcn_sched_barrier(0);   // not sunk to its use
                        }
                    }
                    const bool same = c0 + RD < ncol;   // a turn ahead: this row or the next
                    if (i > 0) fetch(q, same ? i : i - 1, o, ca + q + (same ? c0 + RD : 0), same || i > ci, wt);
                    else fetch(q, i, o, ca + q + c0 + RD, same, wt);
                }
            }
        }
    }
    // The output is complete: its class sum per sample to vp[class][B].
    __device__ __forceinline__ void finish(const GpCore &g, int o, int lane, float *vp) {
        constexpr int B = 16 * G;
        float cls[G];
#pragma unroll
        for (int gg = 0; gg < G; ++gg) cls[gg] = 0.0f;
#pragma unroll
        for (int i = 0; i < RPW; ++i) {
            const int t = row(i);
            if (t >= NT) break;
            v4f r0{}, r1{};
            if constexpr (PREC == GPMPPI_FP32) {
                const v4f *rp = reinterpret_cast<const v4f *>(g.t.wrs + (o * NT + t) * 32) + (lane >> 4);
                r0 = rp[0];
                r1 = rp[4];
            }
#pragma unroll
            for (int gg = 0; gg < G; ++gg) cls[gg] += tile_sq<PREC>(acc[i][0][gg], acc[i][1][gg], r0, r1);
        }
        clear();
#pragma unroll
        for (int gg = 0; gg < G; ++gg)
            if (lane < 16) vp[wc * B + 16 * gg + lane] = cls[gg];
    }
};

// ---------------------------------------------------------------- the rollout of one sample block
// Registers of the whole layout: RB resident blocks of W, and whether more are streamed.
// Eight waves hold every block at up to eight row tiles per output (72 blocks, nine each).
constexpr int kResidentTiles = 8;
template <bool STREAM>
__host__ __device__ constexpr int resident_blocks() { return STREAM ? 5 : 9; }

// Called by all threads of a workgroup of eight waves with core_plan's LDS.
template <int PREC, int G, int LAYOUT>
__device__ __forceinline__ void rollout_core(const RolloutArgs &a, int blk, unsigned char *lds) {
    constexpr bool SWEEP = LAYOUT == kSweep, SERIAL = LAYOUT == kSerial, STREAM = LAYOUT == kWholeStream;
    constexpr bool WHOLE = !SWEEP && !SERIAL;
    constexpr int B = 16 * G, S = kTerms, TB = G * S * 1024, NW = kCoreWaves;
    constexpr int PM = core_parities(LAYOUT) - 1;   // step parity mask of the small arrays
    constexpr int RB = WHOLE ? resident_blocks<STREAM>() : 0;
    constexpr bool kPoints = PREC == GPMPPI_FP32;
    constexpr int NS = NW - 2;   // waves that share the constraint loops
    int tid = threadIdx.x, lane = tid & 63, sl = lane % B, sg = blk * B + sl;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = a.K, T = a.T, NT = a.gp.NT;
    const GpCore gp{a.gp, a.terms};
    const Geometry &geo = a.geo;
    const Dyn dy = a.dyn;
    const CorePlan pl = core_plan<PREC, G, LAYOUT>(NT);
    // The thread index, opaque from here on: called in every phase, so that the many addresses
    // made from it are recomputed there instead of staying live across the whole horizon
    // (they cost some 60 registers).
    auto refresh_lane = [&]() {
        __asm__ __volatile__("" : "+v"(tid));
        lane = tid & 63;
        sl = lane % B;
        sg = blk * B + sl;
    };
    float *rs = reinterpret_cast<float *>(lds + pl.rs);
    float *mp = reinterpret_cast<float *>(lds + pl.mp);     // [parity][output][class][B]
    float *vp = reinterpret_cast<float *>(lds + pl.vp);     // [parity][output][row tile or class][B]; serial: [3][row tile][B]
    float2 *un = reinterpret_cast<float2 *>(lds + pl.un);   // [half][ns][B] sampled controls
    float *gx = reinterpret_cast<float *>(lds + pl.geo);    // [parity][6][B] position, covariance, lambda_max
    float *ored = reinterpret_cast<float *>(lds + pl.ored); // [parity][2 NS][B]
    const int VR = SWEEP ? kClasses : NT;                   // rows of vp per output
    const int ns = pl.ns;
    // two waves (3 and 7, of one SIMD) carry what is not shared out: pose and covariance, and the cost
    const bool pose = w == NW / 2 - 1, cost = w == NW - 1;

    NoiseParams np = a.noise;
    {
        uint64_t seed = a.seed;
        if (a.step_counter) seed += (uint64_t)(*a.step_counter);
        np.key0 = (uint32_t)seed;
        np.key1 = (uint32_t)(seed >> 32);
    }
    // sampled controls of steps s0 .. s0 + ns - 1 into their half of the table
    auto noise_fill = [&](int s0) {
        if (tid >= ns * B) return;
        const int st = s0 + tid / B, s = tid % B;
        if (st < T) un[(s0 / ns & 1) * ns * B + tid] = sampled_control(np, st, blk * B + s, a.U[2 * st], a.U[2 * st + 1]);
    };
    auto writer = [&]() { return lane < B && sg < K; };   // one copy of each sample
    const gpmppi_trace &tr = a.trace;
    const bool traced = tr.x_d || tr.sxy_d || tr.gp_mean_d || tr.gp_var_d || tr.d_lane_d || tr.lane_margin_d ||
                        tr.obs_margin_d || tr.u_d;
    auto control = [&](int st) { return un[((st / ns & 1) * ns + st % ns) * B + sl]; };

    const WTerms<PREC> wt = wterms<PREC>(gp, lane);
    const int nch = SWEEP ? (NT + kSweepTiles - 1) / kSweepTiles : 1;   // chunks per output
    const int nph = WHOLE ? 1 : 2 * nch;                                // phases per step

    // points of the FP32 form.  Whole: both outputs for the whole horizon, z [2][Mpad] then
    // alpha [2][Mpad].  Sweep: two chunks, each z [256] then alpha [256], refilled two phases
    // ahead through one register quadruple per thread.
    v4f *zl = reinterpret_cast<v4f *>(lds + pl.z);
    constexpr int kChunkPts = 32 * kSweepTiles;
    v4f znext{};
    auto points_load = [&](int j) {
        const int o = j >= nch, p = (j - o * nch) * kChunkPts + (tid < kChunkPts ? tid : 4 * (tid - kChunkPts));
        if (tid >= kChunkPts + kChunkPts / 4 || p >= 32 * NT) return;
        znext = tid < kChunkPts ? reinterpret_cast<const v4f *>(gp.d.zs)[o * 32 * NT + p]
                                : *reinterpret_cast<const v4f *>(gp.t.alphas + o * 32 * NT + p);
    };
    auto points_store = [&](int j) {
        if (tid < kChunkPts + kChunkPts / 4) zl[(j & 1) * (kChunkPts + kChunkPts / 4) + tid] = znext;
    };

    noise_fill(0);
    if constexpr (kPoints && SERIAL) {
        for (int i = tid; i < 2 * NT * 32; i += 64 * NW) rs[i] = gp.t.wrs[i];
    }
    if constexpr (kPoints && WHOLE) {
        for (int i = tid; i < 2 * NT * 32; i += 64 * NW) {
            rs[i] = gp.t.wrs[i];
            zl[i] = reinterpret_cast<const v4f *>(gp.d.zs)[i];
            reinterpret_cast<float *>(zl + 2 * NT * 32)[i] = gp.t.alphas[i];
        }
    }
    if constexpr (kPoints && SWEEP) {
        points_load(0);
        points_store(0);
        points_load(1);
        points_store(1);
    }
    __syncthreads();

    // velocities (every wave, all samples) and the query's control
    float v = a.x0[3], w_ = a.x0[4];
    float2 u = control(0);
    // pose wave: heading and covariance, in LDS between its turns (with the position in gx)
    float *pstate = reinterpret_cast<float *>(lds + pl.ps);
    if (pose && lane < B) {
        gx[sl] = a.x0[0];
        gx[B + sl] = a.x0[1];
        pstate[sl] = a.x0[2];
#pragma unroll
        for (int i = 1; i < 16; ++i) pstate[i * B + sl] = 0.0f;
    }
    // cost wave: the sum and the last step's terms and variances, in LDS between its turns
    float *cstate = reinterpret_cast<float *>(lds + pl.cs);
    if (cost && lane < B) {
        cstate[sl] = cstate[B + sl] = 0.0f;
        cstate[2 * B + sl] = 1.0f;
        cstate[3 * B + sl] = INFINITY;
    }
    if (pose && writer() && a.trace.x_d) {
#pragma unroll
        for (int i = 0; i < 5; ++i) a.trace.x_d[i * K + sg] = a.x0[i];
    }
    if (pose && writer() && a.trace.sxy_d) {
        a.trace.sxy_d[0 * K + sg] = 0.0f;
        a.trace.sxy_d[1 * K + sg] = 0.0f;
        a.trace.sxy_d[2 * K + sg] = 0.0f;
    }

    UnitList ul{};   // serial: output 0's
    UnitCursor<STREAM> ufirst{};
    WFrag<PREC> res[RB ? RB : 1];
    Sweep<PREC, G, NW> sw;
    if constexpr (SWEEP) {
        sw.init(w, NT);
        if (w >= NW / 2) sw.prefetch(0, 0, wt);
    } else if constexpr (SERIAL) {
        ul = unit_list<NW>(w, NT, 1, 0, 0);
    } else {
        ul = unit_list<NW>(w, NT, 2, 0, 0);
        resident_load<PREC, RB>(res, wt, ufirst, ul);
    }
    float msw[G];   // sweep: mean chains of the output being generated
    auto sweep_tile = [&](int j) { return (j - (j >= nch) * nch) * kSweepTiles + (j >= nch ? NW - 1 - w : w); };

    // Kernel vectors of chunk j of step ks (query (v, w_, u)) into kb, and their means.
    auto generate = [&](int ks, int j, unsigned char *kb) {
        float *mrow = mp + (ks & PM) * 2 * kClasses * B;
        const float q[4] = {v, w_, u.x, u.y};
        if constexpr (SERIAL) {
            const int o = j ^ (ks & 1), wv = j ? NW - 1 - w : w;
            GenIn<PREC> in;
            if (wv < NT) gen_load<PREC>(in, gp, o, wv, lane);
            gen_output<PREC, G, NW>(gp, o, q, wv, lane, kb, mrow + o * kClasses * B, in,
                                    [&](GenIn<PREC> &t, int jt) { gen_load<PREC>(t, gp, o, jt, lane); });
        } else if constexpr (SWEEP) {
            const int o = j >= nch, ca = (j - o * nch) * kSweepTiles, jt = sweep_tile(j), cl = jt - ca;
            if (ca == 0) {
#pragma unroll
                for (int g = 0; g < G; ++g) msw[g] = 0.0f;
            }
            if (jt < NT) {
                unsigned char *kt = kb + cl * TB;
                float qs[4];
                scaled_query(gp, o, q, qs);
                GenQ<PREC> gq[G];
                gen_queries<PREC, G>(gq, qs, lane);
                if constexpr (kPoints) {
                    const v4f *zc = zl + (j & 1) * (kChunkPts + kChunkPts / 4);
                    gen_tile16<PREC, G>(
                        [&](GenIn<PREC> &t) {
                            gen_load_points(t, zc + 32 * cl, reinterpret_cast<const float *>(zc + kChunkPts) + 32 * cl,
                                            lane);
                        },
                        gq, kt, lane, msw);
                } else {
                    GenIn<PREC> in;
                    gen_load<PREC>(in, gp, o, jt, lane);
                    gen_tile16<PREC, G>([&](GenIn<PREC> &t) { t = in; }, gq, kt, lane, msw);
                }
            }
            if (ca + kSweepTiles >= NT) {
                float *mr = mrow + (o * kClasses + cl) * B;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float t = quarter_sum(msw[g]);
                    if (lane < 16) mr[16 * g + lane] = t;
                }
            }
        } else {
            auto load = [&](int o, GenIn<PREC> &t, int jt) {
                if constexpr (kPoints) {
                    const int p = o * 32 * NT + 32 * jt;
                    gen_load_points(t, zl + p, reinterpret_cast<const float *>(zl + 2 * 32 * NT) + p, lane);
                } else {
                    gen_load<PREC>(t, gp, o, jt, lane);
                }
            };
            GenIn<PREC> in[2];
            if constexpr (!STREAM) {   // at most one tile per output and wave
                const int t0 = w, t1 = NW - 1 - w;
                float m0[G], m1[G];
#pragma unroll
                for (int g = 0; g < G; ++g) m0[g] = m1[g] = 0.0f;
                auto tile = [&](int o, int jt, float (&ms)[G]) {
                    float qs[4];
                    scaled_query(gp, o, q, qs);
                    GenQ<PREC> gq[G];
                    gen_queries<PREC, G>(gq, qs, lane);
                    gen_tile16<PREC, G>([&](GenIn<PREC> &t) { t = in[o]; }, gq, kb + (o * NT + jt) * TB, lane, ms);
                };
                if (t0 < NT) load(0, in[0], t0);
                if (!kPoints && t1 < NT) load(1, in[1], t1);
                if (t0 < NT) tile(0, t0, m0);
                if (kPoints && t1 < NT) load(1, in[1], t1);
                if (t1 < NT) tile(1, t1, m1);
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float a0 = quarter_sum(m0[g]), a1 = quarter_sum(m1[g]);
                    if (lane < 16) {
                        mrow[t0 * B + 16 * g + lane] = a0;
                        mrow[(kClasses + t1) * B + 16 * g + lane] = a1;
                    }
                }
                return;
            }
            if constexpr (!kPoints) {   // from memory: both outputs' first tiles together
                if (w < NT) load(0, in[0], w);
                if (NW - 1 - w < NT) load(1, in[1], NW - 1 - w);
            }
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const int wv = o ? NW - 1 - w : w;
                if constexpr (kPoints) {
                    if (wv < NT) load(o, in[o], wv);
                }
                gen_output<PREC, G, NW>(gp, o, q, wv, lane, kb + o * NT * TB, mrow + o * kClasses * B, in[o],
                                        [&](GenIn<PREC> &t, int jt) { load(o, t, jt); });
            }
        }
    };
    // Serial: the rows of vp of output o in step ks.  The outputs' turns take three places in rotation: a step's
    // are read beside the next step's first turn.
    auto serial_rows = [&](int ks, int o) { return vp + (2 * ks + (o ^ (ks & 1))) % 3 * NT * B; };
    // Variance contraction of chunk j of step ks.
    auto contract = [&](int ks, int j, const unsigned char *kb) {
        float *vrow = vp + (ks & PM) * 2 * VR * B;
        if constexpr (SWEEP) {
            const int o = j >= nch, ca = (j - o * nch) * kSweepTiles;
            sw.pin();
            if (w < NW / 2) sw.prefetch(o, ca / kSweepTiles, wt);   // the others fetched before the barrier
            sw.chunk(o, ca / kSweepTiles, kb, lane, wt);
            if (ca + kSweepTiles >= NT) sw.finish(gp, o, lane, vrow + o * VR * B);
        } else if constexpr (SERIAL) {
            const int o = j ^ (ks & 1);
            const UnitList l{ul.units | (o ? 0x8080808080808080u : 0u), ul.n, ul.blocks};
            UnitCursor<true> first;
            first.start(l);
            walk_units<PREC, G, 0, true>(wt, res, first, lane, l, kb, o, NT, rs, serial_rows(ks, o) - o * NT * B);
        } else {
            walk_units<PREC, G, RB, STREAM>(wt, res, ufirst, lane, ul, kb, 0, NT, rs, vrow);
        }
    };
    // Both outputs' variances of step ks.
    auto variances = [&](int ks, float &sa, float &sb) {
        const float *r = vp + (ks & PM) * 2 * VR * B, *r0 = SERIAL ? serial_rows(ks, 0) : r;
        const float *r1 = SERIAL ? serial_rows(ks, 1) : r + VR * B;
        sa = gp_variance<PREC>(gp, 0, row_classes(r0, VR, B, sl));
        sb = gp_variance<PREC>(gp, 1, row_classes(r1, VR, B, sl));
    };
    // Step ks's constraint loops at its final position, by the six waves that carry neither
    // pose nor cost; 16-sample blocks read the geometry from LDS where it fits.
    v4f *wseg = reinterpret_cast<v4f *>(lds + pl.bytes), *wobs = wseg + geo.P;
    float *winv = reinterpret_cast<float *>(wobs + geo.n_obs);
    auto world = [&](int ks) {
        if (pose || cost) return;
        const float *r = gx + ((ks + 1) & PM) * 6 * B + sl;
        float *out = ored + ((ks + 1) & PM) * 2 * NS * B;
        const int wv = w < NW / 2 ? w : w - 1;
        if (G == 1 && WHOLE && a.world_lds)
            world_share<NS, B>(geo, wseg, winv, wobs, wv, lane, r[0], r[B], r[2 * B], r[3 * B], r[4 * B], r[5 * B], out,
                               true, true);
        else
            world_share<NS, B>(geo, wv, lane, r[0], r[B], r[2 * B], r[3 * B], r[4 * B], r[5 * B], out, true, true);
    };
    if (G == 1 && WHOLE && a.world_lds) {
        for (int i = tid; i < geo.P; i += 64 * NW) {
            wseg[i] = reinterpret_cast<const v4f *>(geo.seg)[i];
            winv[i] = geo.seg_inv[i];
        }
        for (int i = tid; i < geo.n_obs; i += 64 * NW) wobs[i] = reinterpret_cast<const v4f *>(geo.obs)[i];
    }
    // Cost wave: the terms of step ks that need no loop, at its final position and speed vn,
    // and its variances.
    auto stage = [&](int ks, float vn, float sa, float sb) {
        const float *r = gx + ((ks + 1) & PM) * 6 * B + sl;
        float *c = cstate + sl, dmin = c[3 * B];
        const StageIn st = stage_geometry(geo, a.cw, r[0], r[B], vn, r[5 * B], dmin);
        if (lane < B) {
            c[3 * B] = dmin;
            c[4 * B] = st.dl;
            c[5 * B] = st.rbar;
            c[6 * B] = st.dv;
            c[7 * B] = st.dg;
            c[8 * B] = sa;
            c[9 * B] = sb;
        }
    };
    // Cost wave: step ks's cost, its loops' results being complete; returns the sum.
    auto settle = [&](int ks) {
        const float *r = ored + ((ks + 1) & PM) * 2 * NS * B + sl;
        float *c = cstate + sl;
        StageIn st{c[4 * B], c[5 * B], INFINITY, c[6 * B], c[7 * B]};
        float best = INFINITY;
#pragma unroll
        for (int p = 0; p < NS; ++p) {
            if (geo.path_kind != 0) best = fminf(best, r[p * B]);
            st.om = fminf(st.om, r[(NS + p) * B]);
        }
        if (geo.path_kind != 0) st.dl = sqrtf(best);
        float S_ = c[0], Sc = c[B], disc = c[2 * B];
        core_stage_cost(a.cw, geo, st, c[8 * B], c[9 * B], disc, S_, Sc);
        if (lane < B) {
            c[0] = S_;
            c[B] = Sc;
            c[2 * B] = disc;
        }
        if (traced && writer()) write_margins(a.trace, K, sg, ks, st);
    };

    if constexpr (!SERIAL) {
        generate(0, 0, lds);
        __syncthreads();
    }
    int buf = 0;
    for (int k = 0; k < T; ++k) {
        for (int j = 0; j < nph; ++j) {
            const bool last = j == nph - 1;
            refresh_lane();
            float m0 = 0.0f, m1 = 0.0f;
            const float vk = v, wk = w_;
            const float2 uk = u;
            if constexpr (SERIAL) {
                generate(k, j, lds);
                __syncthreads();
                refresh_lane();
            }
            if constexpr (kPoints && SWEEP) points_load(j + 2 < nph ? j + 2 : j + 2 - nph);
            if (last) {   // step k's means are complete: the next query
                const float *r = mp + (k & PM) * 2 * kClasses * B;
                m0 = gp_mean_of(r, B, sl);
                m1 = gp_mean_of(r + kClasses * B, B, sl);
                step_velocities(dy, u, m0, m1, v, w_);
                if (k + 1 < T) u = control(k + 1);
                if (k % ns == 0) noise_fill(k + ns);
            }
            const unsigned char *kc = lds + buf * pl.kbuf;
            unsigned char *kn = lds + (1 - buf) * pl.kbuf;
            buf ^= 1;
            // half of the waves contract first, so both pipes of a SIMD have work
            const bool gen_first = w < NW / 2;
            if constexpr (SERIAL) contract(k, j, lds);
#pragma unroll 1
            for (int pass = 0; pass < (SERIAL ? 0 : 2); ++pass) {
                refresh_lane();
                if ((pass == 0) == gen_first) {
                    if (!(last && k + 1 == T)) generate(last ? k + 1 : k, last ? 0 : j + 1, kn);
                    if constexpr (SWEEP) sw.forget();
                } else {
                    contract(k, j, kc);
                }
            }
            refresh_lane();
            if (j == 0 && k >= 1) {   // step k - 1: constraint loops, variances
                world(k - 1);
                if (pose || cost) {
                    float sa, sb;
                    variances(k - 1, sa, sb);
                    if (pose && lane < B) {   // Sigma_k is complete
                        float *ps = pstate + sl;
                        add_gp_variance(ps[13 * B], dy.dt, sa);
                        add_gp_variance(ps[15 * B], dy.dt, sb);
                    }
                    if (cost) {
                        if (WHOLE && k >= 2) settle(k - 2);
                        stage(k - 1, vk, sa, sb);
                        if (traced && writer()) write_variances(a.trace, K, sg, k - 1, sa, sb);
                    }
                }
            }
            if (last && !WHOLE && cost && k >= 1) settle(k - 1);
            if (last && pose) {
                const float *g0 = gx + (k & PM) * 6 * B + sl;
                float *ps = pstate + sl;
                float X = g0[0], Y = g0[B], th = ps[0];
                Cov P{ps[B], ps[2 * B], ps[3 * B], ps[4 * B], ps[5 * B], ps[6 * B], ps[7 * B], ps[8 * B],
                      ps[9 * B], ps[10 * B], ps[11 * B], ps[12 * B], ps[13 * B], ps[14 * B], ps[15 * B]};
                // position, heading and A Sigma A^T (Eqs. 1, 10); the geometry at (x_{k+1}, Sigma_{k+1}),
                // with Step 2 tightening the nominal sequence's covariance (Eqs. 13-16)
                float sth, cth;
                sincosf(th, &sth, &cth);
                const StepJac jac = step_jacobian(dy, vk, sth, cth);
                advance_pose(dy, vk, wk, sth, cth, X, Y, th);
                propagate_cov(P, jac);
                float ca = P.p00, cb = P.p01, cc = P.p11;
                if (a.tight_sxy) {
                    ca = a.tight_sxy[3 * (k + 1)];
                    cb = a.tight_sxy[3 * (k + 1) + 1];
                    cc = a.tight_sxy[3 * (k + 1) + 2];
                }
                if (lane < B) {
                    float *r = gx + ((k + 1) & PM) * 6 * B + sl;
                    r[0] = X;
                    r[B] = Y;
                    r[2 * B] = ca;
                    r[3 * B] = cb;
                    r[4 * B] = cc;
                    r[5 * B] = lambda_max(ca, cb, cc);
                    ps[0] = th;
                    const float c[15] = {P.p00, P.p01, P.p02, P.p03, P.p04, P.p11, P.p12, P.p13,
                                         P.p14, P.p22, P.p23, P.p24, P.p33, P.p34, P.p44};
#pragma unroll
                    for (int i = 0; i < 15; ++i) ps[(i + 1) * B] = c[i];
                }
                if (traced && writer()) write_step(a.trace, K, sg, k, X, Y, th, v, w_, P, m0, m1, uk);
            }
            if constexpr (SWEEP) {
                if (w >= NW / 2) {   // contracts first: the next chunk's first blocks
                    const int jn = j + 1 < nph ? j + 1 : 0;
                    sw.prefetch(jn >= nch, jn - (jn >= nch) * nch, wt);
                }
            }
            if constexpr (kPoints && SWEEP) points_store(j);
            __syncthreads();
        }
    }
    // the last steps' costs
    world(T - 1);
    if (cost) {
        float sa, sb;
        variances(T - 1, sa, sb);
        if (traced && writer()) write_variances(a.trace, K, sg, T - 1, sa, sb);
        if (WHOLE && T >= 2) settle(T - 2);
        stage(T - 1, v, sa, sb);
    }
    __syncthreads();
    if (cost) {
        settle(T - 1);
        float S_ = cstate[sl];
        if (a.cw.w_term != 0.0f && !(cstate[3 * B + sl] <= a.cw.goal_tol)) S_ = S_ + (a.cw.w_term - cstate[B + sl]);
        if (writer()) a.costs[sg] = S_;
    }
}

}  // namespace core
}  // namespace gpmppi
