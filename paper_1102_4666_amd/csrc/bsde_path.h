// bsde_path.h -- the Monte Carlo path kernel of one Picard iteration of
// Algorithm "algodetail" (Labart & Lelong, arXiv:1102.4666, Section 4.1),
// templated on the dimension d, the basis degree eta and the path precision.
// Instantiated per dimension in bsde_inst_d*.hip.
//
//   a_m for every (point i, path m): Philox4x32-10 normals in registers,
//   Box-Muller, Euler scheme of the log-price (eq. 4) with coefficients
//   frozen at the last node (eq. eqs3), the interpolated state at the random
//   time tau = t_i + (T - t_i) U (eq. psiN), the Chebyshev basis row at
//   (tau, X_tau) contracted with the derivative channels of u^k, the
//   penalised driver (eq. bsde-penal-2) and the frozen generator; per-lane
//   FP64 sums reduced through wavefront shuffles and LDS in a fixed order.
#pragma once

#include "bsde_common.h"
#include "bsde_f64_math.h"

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

namespace bsde {

// The FP64 kernels' tables of logarithms, sines, cosines and powers of two
// (bsde_f64_math.h), one copy per workgroup, filled when it starts
// (fill_path_tables).
static __shared__ f64::Tables f64_tables;

// ---------------------------------------------------------------------------
// Precision-specific arithmetic.  FP32: hardware transcendentals (v_log_f32
// is log2, v_sin/v_cos take revolutions); FP64: bsde_f64_math.h in the
// step loop, the device math library outside it.
// ---------------------------------------------------------------------------
template <typename Real>
struct Arith;

template <>
struct Arith<float> {
    static __device__ __forceinline__ float u01(uint32_t w)
    {
        return fmaf((float)w, 0x1p-32f, 0x1p-33f); // (w + 1/2) 2^-32
    }
    // Box-Muller pair scaled by sqrt(v): R = sqrt(-2 v ln ua), computed as
    // sqrt((-2 ln2 v) log2 ua); angle 2 pi ub (v_sin/v_cos take revolutions)
    static __device__ __forceinline__ float bm_scale(float v)
    {
        return -1.38629436111989061883f * v;
    }
    // c32, c33: 2^-32 and 2^-33 of u01, passed in so that the caller can
    // hold them in vector registers
    static __device__ __forceinline__ void box_muller(uint32_t wa, uint32_t wb,
                                                      float scale, float &n0,
                                                      float &n1, float c32 = 0x1p-32f,
                                                      float c33 = 0x1p-33f)
    {
        const float ua = fmaf((float)wa, c32, c33);
        float R = __builtin_amdgcn_sqrtf(scale * __builtin_amdgcn_logf(ua));
        // angle: 1 + (top 23 bits of wb) 2^-23 in [1, 2) revolutions, built
        // by one funnel shift that puts the exponent of 1.0 above them
        // (sine and cosine have period one revolution)
        const float ub = __builtin_bit_cast(float, __builtin_amdgcn_alignbit(0x7Fu, wb, 9u));
        n0 = R * __builtin_amdgcn_cosf(ub);
        n1 = R * __builtin_amdgcn_sinf(ub);
    }
    static __device__ __forceinline__ float exp(float x) { return __expf(x); }
    static __device__ __forceinline__ float exp_nonpos(float x) { return __expf(x); }
    static __device__ __forceinline__ float sqrt(float x)
    {
        return __builtin_amdgcn_sqrtf(x); // v_sqrt_f32, no refinement
    }
    static __device__ __forceinline__ float frac33(uint64_t num)
    {
        // (num mod 2^33) 2^-33 from the top 32 of the low 33 bits
        return (float)(uint32_t)((num & 0x1FFFFFFFFull) >> 1) * 0x1p-32f;
    }
};

template <>
struct Arith<double> {
    static __device__ __forceinline__ double u01(uint32_t w)
    {
        return ((double)w + 0.5) * 0x1p-32;
    }
    // v is kept above 2^-800 (it is zero for points at T, whose paths do not
    // move: a normal of 2^-400 adds nothing to the state either), so that the
    // radius' square root needs no case for zero
    static __device__ __forceinline__ double bm_scale(double v)
    {
        return -2.0 * fmax(v, 0x1p-800);
    }
    // Box-Muller pair scaled by sqrt(v), scale = -2 v: R = sqrt(-2 v ln ua);
    // ln ua and the sine and cosine of the angle 2 pi ub from the words
    // themselves (bsde_f64_math.h)
    static __device__ __forceinline__ void box_muller(uint32_t wa, uint32_t wb,
                                                      double scale, double &n0,
                                                      double &n1, double = 0.0,
                                                      double = 0.0)
    {
        double R = f64::sqrt_pos(scale * f64::log_word_tab(wa, f64_tables));
        double s, c;
        f64::sincos_turn_tab(wb, f64_tables, s, c);
        n0 = R * c;
        n1 = R * s;
    }
    static __device__ __forceinline__ double exp(double x) { return ::exp(x); }
    // e^x for x <= 0 (the volatilities' Gaussian factors)
    static __device__ __forceinline__ double exp_nonpos(double x)
    {
        return f64::exp_nonpos_tab(x, f64_tables);
    }
    static __device__ __forceinline__ double sqrt(double x) { return ::sqrt(x); }
    static __device__ __forceinline__ double frac33(uint64_t num)
    {
        return (double)(num & 0x1FFFFFFFFull) * 0x1p-33;
    }
};

// Time factors of the Dupire-type volatility of eq. vol_locale, uniform
// across the paths of a point at one Euler step: with S = e^x,
// sigma(t, S) = A(t) - B(t) e^{-0.001 (S e^{r t} - s)^2}, A = 0.72 e^{-0.05
// sqrt t}, B = 0.6 e^{-0.1 t} e^{-0.05 sqrt t}, rt = r t.
template <typename Real>
struct VolTime {
    Real A, B, rt;
};
template <int VOL, typename Real>
__device__ __forceinline__ VolTime<Real> vol_time(Real t, Real r)
{
    VolTime<Real> v{Real(0), Real(0), Real(0)};
    if constexpr (VOL == kVolDupire) {
        const Real damp = Arith<Real>::exp(Real(-0.05) * Arith<Real>::sqrt(t));
        v.A = Real(0.72) * damp;
        v.B = Real(0.6) * damp * Arith<Real>::exp(Real(-0.1) * t);
        v.rt = r * t;
    }
    return v;
}

// sigma_j of log-price x: constant; bump level (1 + a e^{-(x - log c)^2})
// = level + (level a) e^{...}; or the Dupire-type form above
template <int VOL, typename Real>
__device__ __forceinline__ Real local_vol(Real level, Real level_a, Real lc,
                                          Real spot, const VolTime<Real> &vt,
                                          Real x)
{
    if constexpr (VOL == kVolBump) {
        Real dx = x - lc;
        return fma(level_a, Arith<Real>::exp_nonpos(-dx * dx), level);
    } else if constexpr (VOL == kVolDupire) {
        const Real dev = Arith<Real>::exp(x + vt.rt) - spot;
        return fma(-vt.B, Arith<Real>::exp_nonpos(Real(-0.001) * dev * dev), vt.A);
    }
    return level;
}

// Coordinates of the Euler state.  With the bump volatility the paths carry
// y = kappa (x - log c) -- kappa^2 = log2 e in FP32, 256 log2 e in FP64 --
// so that the volatility costs a square, one exponential and one fused
// multiply-add per asset and step: level + (level a) 2^{-y^2} (FP32), level +
// (level a) 2^{-y^2/256} (FP64: the table exponential needs no reduction by
// ln 2, and takes the square unrounded).  Every increment of x is scaled by
// kappa as well.  The other volatility kinds keep y = x.
template <int VOL, typename Real>
struct EulerState {
    static constexpr bool kShift = VOL == kVolBump;
    static constexpr Real kappa = !kShift ? Real(1)
                                  : sizeof(Real) == 4 ? Real(1.2011224087864498)
                                                      : Real(19.217958540583197);
    static __device__ __forceinline__ Real to(Real x, Real lc)
    {
        if constexpr (kShift) return (x - lc) * kappa;
        else return x;
    }
    static __device__ __forceinline__ Real from(Real y, Real lc)
    {
        if constexpr (kShift) return fma(y, Real(1) / kappa, lc);
        else return y;
    }
    static __device__ __forceinline__ Real vol(Real level, Real level_a, Real spot,
                                               const VolTime<Real> &vt, Real y)
    {
        if constexpr (kShift) {
            if constexpr (sizeof(Real) == 4)
                return fmaf(level_a, __builtin_amdgcn_exp2f(-y * y), level);
            else
                return fma(level_a, f64::exp2_neg_sq_tab(y, f64_tables), level);
        } else {
            return local_vol<VOL>(level, level_a, Real(0), spot, vt, y);
        }
    }
};

template <int D, typename Real>
__device__ __forceinline__ Real payoff(int kind, Real K, const Real *x)
{
    Real s = 0;
    if (kind == kPutArith || kind == kCallArith || kind == kFwdArith) {
#pragma unroll
        for (int j = 0; j < D; ++j) s += Arith<Real>::exp(x[j]);
        s *= Real(1.0 / D);
    } else {
#pragma unroll
        for (int j = 0; j < D; ++j) s += x[j];
        if (kind == kQuad) return s * s;
        s = Arith<Real>::exp(s * Real(1.0 / D));
    }
    switch (kind) {
    case kPutArith:
    case kPutGeom: return fmax(K - s, Real(0));
    case kCallArith:
    case kCallGeom: return fmax(s - K, Real(0));
    default: return s - K; // kFwdArith
    }
}

// Chebyshev values T_0..T_ETA of z
template <int ETA, typename Real>
__device__ __forceinline__ void cheb(Real z, Real *Tz)
{
    Tz[0] = Real(1);
    if (ETA >= 1) Tz[1] = z;
#pragma unroll
    for (int a = 1; a < ETA; ++a) Tz[a + 1] = Real(2) * z * Tz[a] - Tz[a - 1];
}

// Position of row l (time degree zero) among the rows with time degree zero
template <typename BS>
constexpr int terminal_index(int l)
{
    int n = 0;
    for (int q = 0; q < l; ++q) n += BS::tab.nu[q][0] == 0;
    return n;
}

// One Philox4x32-10 round in the path kernel (the function of philox_round).
// Bit 0 / bit 1 of X3 select, for the new word 0 / word 2, the three-way
// XOR (high half ^ counter word ^ key) as one v_bitop3_b32 with truth table
// 0x96 (a ^ b ^ c) instead of two v_xor_b32.  That pays only where the
// counter word varies across the wave: with a uniform counter word the two
// uniform operands combine on the scalar unit and leave one vector XOR,
// while v_bitop3_b32 (one scalar operand at most) would need a move too.
template <int X3>
__device__ __forceinline__ void philox_round_dev(u32x4 &c, uint32_t &k0, uint32_t &k1)
{
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
    const uint32_t h1 = (uint32_t)(p1 >> 32), h0 = (uint32_t)(p0 >> 32);
    const uint32_t n0 = (X3 & 1) ? __builtin_amdgcn_bitop3_b32(h1, c.y, k0, 0x96)
                                 : h1 ^ c.y ^ k0;
    const uint32_t n2 = (X3 & 2) ? __builtin_amdgcn_bitop3_b32(h0, c.w, k1, 0x96)
                                 : h0 ^ c.w ^ k1;
    c = {n0, (uint32_t)p1, n2, (uint32_t)p0};
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
}

// One Philox4x32-10 block in the path kernel (the same function as
// philox10) on the counter (m, i, k, word 3): m varies across the wave, the
// other three words are uniform.  Rounds 1 and 2 keep their hoistable work
// on the uniform words; after round 2 only word 3 is still uniform, and from
// round 4 on every word varies, so with kXor3 round 3 takes the three-input
// XOR for word 0 and rounds 4-10 for both.  All kernels but the FP64 d = 1
// ones take it (10 fewer of the ~53 vector instructions of a block; the
// d = 10 launches 3-5% faster); the FP64 d = 1 kernels keep the two-XOR
// form, under which they fit 128 registers (four waves per SIMD).
// After the second round the key passes through an empty asm statement, so
// that the keys of rounds 3-10, k + r (W0, W1), are formed on the scalar
// unit per block instead of being hoisted out of the path loops, where
// sixteen of them would stay live in scalar registers (at d >= 5 the
// compiler parks the excess in vector-register lanes and reads it back with
// one vector instruction per use).
// Keys of rounds 3-10, k + r (W0, W1) for r = 2..9, held in vector
// registers: v_bitop3_b32 with all three operands in vector registers
// issues in about three cycles instead of four.
struct PhiloxKeys {
    uint32_t a[8], b[8];
};

__device__ __forceinline__ PhiloxKeys philox_vector_keys(uint32_t k0, uint32_t k1)
{
    PhiloxKeys kv;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        kv.a[r] = k0 + (uint32_t)(r + 2) * 0x9E3779B9u;
        kv.b[r] = k1 + (uint32_t)(r + 2) * 0xBB67AE85u;
        asm volatile("" : "+v"(kv.a[r]), "+v"(kv.b[r]));
    }
    return kv;
}

template <bool kXor3>
__device__ __forceinline__ u32x4 philox_block(uint32_t c0, uint32_t c1, uint32_t c2,
                                              uint32_t c3, uint32_t k0, uint32_t k1)
{
    u32x4 c{c0, c1, c2, c3};
    philox_round_dev<0>(c, k0, k1);
    philox_round_dev<0>(c, k0, k1);
    asm volatile("" : "+s"(k0), "+s"(k1));
    philox_round_dev<kXor3 ? 1 : 0>(c, k0, k1);
#pragma unroll
    for (int r = 3; r < 10; ++r) philox_round_dev<kXor3 ? 3 : 0>(c, k0, k1);
    return c;
}

// The same block with the keys of rounds 3-10 taken from vector registers
// (every XOR of those rounds one v_bitop3_b32; in round 3 the uniform word
// 3 is its one scalar operand).
__device__ __forceinline__ u32x4 philox_block(uint32_t c0, uint32_t c1, uint32_t c2,
                                              uint32_t c3, uint32_t k0, uint32_t k1,
                                              const PhiloxKeys &kv)
{
    u32x4 c{c0, c1, c2, c3};
    philox_round_dev<0>(c, k0, k1);
    philox_round_dev<0>(c, k0, k1);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        uint32_t ka = kv.a[r], kb = kv.b[r];
        philox_round_dev<3>(c, ka, kb);
    }
    return c;
}

// The per-asset constants of a launch as a constant-address-space object
// at the uniform address cbase of its PathParams (the kernel-argument
// segment, or the batch's descriptor table), through an address the
// compiler cannot see through, so that their scalar loads are issued where
// they are used instead of being hoisted out of the loop.
template <typename Real>
using ConstAssets = const __attribute__((address_space(4))) AssetConsts<Real>;

template <typename Real>
__device__ __forceinline__ ConstAssets<Real> &reload_consts(uint64_t cbase)
{
    uint64_t a = cbase + (sizeof(Real) == 8 ? offsetof(PathParams, cd)
                                            : offsetof(PathParams, cf));
    asm volatile("" : "+s"(a));
    return *(ConstAssets<Real> *)a;
}

// The FP64 kernels' tables, copied once per workgroup before its first tile
template <typename Real>
__device__ __forceinline__ void fill_path_tables()
{
    if constexpr (sizeof(Real) == 8) {
        f64::fill_tables(f64_tables, (int)threadIdx.x, kBlock);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// u, d_t u, grad u and grad^2 u by the cubic form (bsde_common.h) at the
// mapped coordinates z, folded into u and the frozen generator gen = d_t u +
// b grad u + tr(a grad^2 u), a_jk = sg_j sg_k C_jk / 2, with bst and sg in
// units of z, tz = dz_0/dt and rho the correlation; and u(T, x) at the spatial
// coordinates zT.  table: the problem's table (uniform address).
//
// FP32: every row is one row of a 4 x 4 x 1 matrix product of 16 blocks
// (v_mfma_f32_4x4x1_16b_f32), in which each lane's column is its own path and
// the four rows of the product land in the lane's own registers.  The rows'
// coefficients come 64 at a time in one register (one coalesced load), and
// each product broadcasts one of its 16 groups of four to every block.  A
// product issues in 4 cycles and does 4 fused multiply-adds a lane on the
// matrix cores beside the other waves' vector work; with the coefficient as
// scalar operand each costs the vector unit 4 cycles.  All 64 lanes have to
// be active (the loads serve the other lanes' products).
// FP64: rows as fused multiply-adds with scalar operands.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int D, typename Real>
struct CubicFold {
    static constexpr int DP = D + 1;
    const Real *z, *sg, *bst;
    const Real tz, rho;
    Real q[DP], u, gen, off;
    __device__ __forceinline__ CubicFold(const Real *z_, const Real *sg_, const Real *bst_,
                                         Real tz_, Real rho_)
        : z(z_), sg(sg_), bst(bst_), tz(tz_), rho(rho_), u(0), gen(0), off(0)
    {
#pragma unroll
        for (int v = 0; v < DP; ++v) q[v] = Real(0);
    }
    // adds d_v u = g to gen and z_v g / f to u
    template <int V>
    __device__ __forceinline__ void gradient(Real g, Real f)
    {
        u = fma(z[V], f * g, u);
        gen = fma(V == 0 ? tz : bst[V == 0 ? 0 : V - 1], g, gen);
    }
    // row R of the table's rows at tau
    template <int R>
    __device__ __forceinline__ void row(Real h)
    {
        constexpr int pairs = DP * (DP + 1) / 2;
        if constexpr (R < pairs) {
            constexpr int v = hess_j(DP, R), w = hess_k(DP, R);
            q[v] = fma(h, z[w], q[v]);
            if constexpr (v != w) q[w] = fma(h, z[v], q[w]);
            if constexpr (v > 0) {
                // tr(a H) = sum_j sg_j (sg_j H_jj / 2 + rho sum_{k > j} sg_k H_jk)
                if constexpr (v == w) {
                    gen = fma(Real(0.5) * sg[v - 1] * sg[v - 1], h, gen);
                    off = Real(0);
                } else {
                    off = fma(sg[w - 1], h, off);
                    if constexpr (w == D) gen = fma(rho * sg[v - 1], off, gen);
                }
            }
        } else if constexpr (R < pairs + DP) {
            gradient<R - pairs>(h, Real(2.0 / 3.0));
        } else if constexpr (R == pairs + DP) {
            u += h;
        }
    }
    // the single-variate terms c4 z^4 + c5 z^5 of variate V (w = c4 + c5 z):
    // their derivatives are z^3 (4 w + c5 z) and 4 z^2 (3 w + 2 c5 z)
    template <int V>
    __device__ __forceinline__ void quintic(Real c4, Real c5)
    {
        const Real x = z[V], x2 = x * x, t = c5 * x, w = t + c4;
        u = fma(x2 * x2, w, u);
        gen = fma(V == 0 ? tz : bst[V == 0 ? 0 : V - 1], x2 * x * fma(Real(4), w, t), gen);
        if constexpr (V > 0)
            gen = fma(Real(2) * sg[V - 1] * sg[V - 1], x2 * fma(Real(3), w, t + t), gen);
    }
    // the parts of the gradient and of u that come with q
    __device__ __forceinline__ void finish()
    {
        static_for<DP>([&](auto vc) {
            constexpr int v = decltype(vc)::value;
            gradient<v>(Real(0.5) * q[v], Real(1.0 / 3.0));
        });
    }
};

// the terms of degree 4 and 5 at T (table: c4, c5 of each variate; z_0 = 1
// there, in the constant)
template <int D, typename Table, typename Real>
__device__ __forceinline__ void quintic_terms_t(Table table, const Real *zT, Real &uT)
{
    static_for<D>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const Real x2 = zT[j] * zT[j];
        uT = fma(x2 * x2, fma(Real(table[2 * j + 3]), zT[j], Real(table[2 * j + 2])), uT);
    });
}
// and at tau
template <int D, typename Table, typename Real>
__device__ __forceinline__ void quintic_terms(Table table, CubicFold<D, Real> &f)
{
    static_for<D + 1>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        f.template quintic<v>(table[2 * v], table[2 * v + 1]);
    });
}

template <int D, int KIND>
__device__ __forceinline__ void cubic_eval(uint64_t table, const float *z, const float *zT,
                                           const float *sg, const float *bst, float rho,
                                           float tz, float &u, float &gen, float &uT)
{
    constexpr CubicLayout lay(D, true, KIND);
    constexpr int kChunks = lay.off_q / 64;
    constexpr int GB = 2; // groups of rows at a time
    const auto tab = (const __attribute__((address_space(1))) float *)table + (threadIdx.x & 63);
    float ch[kChunks];
    // a few groups of rows at a time: their products do not wait for each
    // other.  A batch's chunks are loaded during the batch before it; its
    // rows are folded before the next batch (pin: the sums pass through an
    // empty asm statement) and nothing moves across, so that two batches'
    // chunks and one batch's rows are what is live
    auto rows = [&](auto off, auto nrows, auto nk, const float *v, auto &&fold, auto &&pin) {
        constexpr int OFF = decltype(off)::value / 4, NR = decltype(nrows)::value,
                      NK = decltype(nk)::value, NG = CubicLayout::groups(NR);
        auto load = [&](auto bc) { // the chunks first needed by batch bc
            constexpr int b = decltype(bc)::value;
            constexpr int p0 = OFF + GB * b * NK,
                          p1 = OFF + (GB * b + GB < NG ? GB * b + GB : NG) * NK;
            constexpr int c0 = b == 0 ? p0 / 16 : (p0 + 15) / 16, c1 = (p1 + 15) / 16;
            static_for<c1 - c0>([&](auto cc) {
                constexpr int c = c0 + decltype(cc)::value;
                ch[c] = tab[64 * c];
            });
        };
        load(std::integral_constant<int, 0>{});
        static_for<(NG + GB - 1) / GB>([&](auto bc) {
            constexpr int g0 = decltype(bc)::value * GB, ng = NG - g0 < GB ? NG - g0 : GB;
            if constexpr (g0 + GB < NG) load(std::integral_constant<int, g0 / GB + 1>{});
            f32x4 acc[GB];
#pragma unroll
            for (int g = 0; g < GB; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
            static_for<NK>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                const float b = k == 0 ? 1.0f : v[k == 0 ? 0 : k - 1];
                static_for<ng>([&](auto gc) {
                    constexpr int g = decltype(gc)::value;
                    constexpr int pos = OFF + (g0 + g) * NK + k;
                    acc[g] = __builtin_amdgcn_mfma_f32_4x4x1f32(ch[pos / 16], b, acc[g], 4,
                                                                pos % 16, 0);
                });
            });
            static_for<4 * ng>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                if constexpr (4 * g0 + r < NR)
                    fold(std::integral_constant<int, 4 * g0 + r>{}, acc[r / 4][r % 4]);
            });
            pin();
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using std::integral_constant;
    float t = 0.f;
    uT = 0.f;
    rows(integral_constant<int, lay.off_t>{}, integral_constant<int, lay.rows_t>{},
         integral_constant<int, lay.kt>{}, zT, [&](auto rc, float h) {
             constexpr int r = decltype(rc)::value;
             if constexpr (r < lay.pairs_t) {
                 constexpr int j = hess_j(D, r), k = hess_k(D, r);
                 t = k == j ? h * zT[k] : fmaf(h, zT[k], t);
                 if constexpr (k == D - 1) uT = fmaf(zT[j], t, uT);
             } else {
                 uT += h;
             }
         },
         [&]() { asm volatile("" : "+v"(t), "+v"(uT)); });
    const auto terms = (const __attribute__((address_space(4))) float *)table + lay.off_q;
    if constexpr (KIND == 2) {
        quintic_terms_t<D>(terms, zT, uT);
        asm volatile("" : "+v"(uT));
        __builtin_amdgcn_sched_barrier(0);
    }
    CubicFold<D, float> f(z, sg, bst, tz, rho);
    rows(integral_constant<int, 0>{}, integral_constant<int, lay.rows>{},
         integral_constant<int, lay.ka>{}, z, [&](auto rc, float h) {
             f.template row<decltype(rc)::value>(h);
         },
         [&]() {
             asm volatile("" : "+v"(f.u), "+v"(f.gen), "+v"(f.off));
#pragma unroll
             for (int v = 0; v <= D; ++v) asm volatile("" : "+v"(f.q[v]));
         });
    if constexpr (KIND == 2) quintic_terms<D>(terms, f);
    f.finish();
    u = f.u;
    gen = f.gen;
}

template <int D, int KIND>
__device__ __forceinline__ void cubic_eval(uint64_t table, const double *z, const double *zT,
                                           const double *sg, const double *bst, double rho,
                                           double tz, double &u, double &gen, double &uT)
{
    constexpr CubicLayout lay(D, false, KIND);
    const auto tab = (const __attribute__((address_space(4))) double *)table;
    // u(T, x), nested
    {
        int e = lay.off_t;
        uT = tab[e++];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            double a = tab[e++];
#pragma unroll
            for (int k = j; k < D; ++k) {
                double b = tab[e++];
#pragma unroll
                for (int l = k; l < D; ++l) b = fma(zT[l], tab[e++], b);
                a = fma(zT[k], b, a);
            }
            uT = fma(zT[j], a, uT);
        }
    }
    CubicFold<D, double> f(z, sg, bst, tz, rho);
    static_for<lay.rows>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        double h = tab[r * lay.ka];
#pragma unroll
        for (int v = 0; v <= D; ++v) h = fma(z[v], tab[r * lay.ka + 1 + v], h);
        f.template row<r>(h);
    });
    if constexpr (KIND == 2) {
        quintic_terms_t<D>(tab + lay.off_q, zT, uT);
        quintic_terms<D>(tab + lay.off_q, f);
    }
    f.finish();
    u = f.u;
    gen = f.gen;
}

// ---------------------------------------------------------------------------
// The Monte Carlo path kernel.
// Grid: n * groups workgroups of kBlock lanes; workgroup (i, g) runs the
// paths m = (g * ppl + r) * kBlock + lane, r < ppl, m < M, of point i and
// writes the mean and the sum of squared deviations of its FP64 path terms
// to partial[2 (i groups + g)].
// ---------------------------------------------------------------------------
// Gamma is read-only, uniform across the workgroup and read once per basis
// function and channel per path: its loads must stay scalar (SGPR) loads,
// so GammaPtr is a global restrict pointer or a constant-address-space one.
template <int D, int ETA, typename Real, int VOL, int Q, typename GammaPtr,
          int OP = kOpBasis, bool RELOAD = false>
__device__ __forceinline__ void run_tile(const PathParams &prm, uint64_t cbase,
                                         const double *__restrict__ pts,
                                         GammaPtr gamma, const int i,
                                         const int g, double *__restrict__ out)
{
    constexpr int DP = D + 1;
    [[maybe_unused]] constexpr int C = num_channels(D);
    using BS = Basis<DP, ETA, Q>;
    constexpr int NP = BS::P;
    // steps per group so that a group uses whole Philox blocks
    constexpr int SG = (D % 4 == 0) ? 1 : ((D % 2 == 0) ? 2 : 4);
    constexpr int NB = SG * D / 4;
    constexpr int NBB = (D + 3) / 4; // bridge blocks
    constexpr int kCubicKind = OP == kOpBasis ? cubic_kind_of<DP, ETA, Q>() : 0;
    constexpr bool kCubic = kCubicKind > 0;
    // Normals of a group of several blocks are made at the first step that
    // needs them: later steps' normals do not wait in registers (the FP64
    // d = 5 kernel keeps its Euler loop free of spills), and a path's last
    // group makes no block beyond its last step.  Not at d = 10, two steps a
    // group: at the FP64 kernels' two waves per SIMD the blocks made together
    // hide each other's latencies (8192 points, M = 500, N = 50: 4.49 ms
    // against 4.95; degree 2, constant volatility, 3072 points, M = 1000, N = 50:
    // 2.05 against 2.20), and the FP32 kernels would spill more.
    constexpr bool kLateNormals = NB > 1 && D < 10;
    constexpr bool kXor3 = sizeof(Real) == 4 || D >= 2; // Philox XOR form
    // FP64 at d = 10: the constant volatilities pass through an empty asm
    // statement on each path, so that what follows from them alone (55 entries of
    // the covariance) is formed there and not kept across the path loop, in
    // scratch memory for the most part (degree 2, 3072 points, M = 1000: N = 5
    // 0.626 -> 0.457 ms, N = 50 2.19 -> 2.05)
    constexpr bool kOpaqueVol = VOL == kVolConst && sizeof(Real) == 8 && D >= 10;
    // FP32 round keys in vector registers (16 of them): at d = 1, and at
    // d = 2 from eta = 5 on, where the kernel's own registers already hold
    // it to four waves per SIMD and the keys still fit (below, they would
    // cost waves).  Not in the kernel operator, whose pair loop, not the
    // Euler loop, sets the time and which would lose waves.  At d = 10 in the
    // cubic form, which leaves the registers for it at three waves (with the
    // constants of kVecConst: 8192 points, M = 500, N = 50 1.57 -> 1.50 ms).
    constexpr bool kVKeys = sizeof(Real) == 4 && OP == kOpBasis &&
                            (D == 1 || (D == 2 && ETA >= 5) || (D >= 10 && kCubic));

    const uint32_t k0 = (uint32_t)prm.seed, k1 = (uint32_t)(prm.seed >> 32);
    PhiloxKeys kv{};
    if constexpr (kVKeys) kv = philox_vector_keys(k0, k1);
    auto block = [&](uint32_t m, uint32_t w3) -> u32x4 {
        if constexpr (kVKeys) return philox_block((uint32_t)m, (uint32_t)i, prm.k, w3, k0, k1, kv);
        else return philox_block<kXor3>((uint32_t)m, (uint32_t)i, prm.k, w3, k0, k1);
    };

    const double *row = pts + (size_t)i * DP;
    const Real T = (Real)prm.T;
    const Real t0 = (Real)row[0];
    const Real h = (T - t0) / (Real)prm.N;
    // A point at T: its paths have no time to move in, every one ends where
    // it starts with the same path term.  One path a lane without Euler steps
    // gives the mean and the spread (zero) of all of them.  Every tensor or
    // random grid has its last time node there: with 10 nodes, d = 5, 40 960
    // points, M = 1000, N = 50 the launch takes 14.6 ms instead of 16.1 in
    // FP64 and 5.57 instead of 6.2 in FP32.
    const bool still = t0 == T;
    const int passes = still ? 1 : prm.paths_per_lane;
    const int ngroups = still ? 0 : (prm.N + SG - 1) / SG;
    // Euler state coordinates y = kappa (x - off); step normals come out of
    // Box-Muller already scaled by kappa sqrt(h)
    using ES = EulerState<VOL, Real>;
    const Real step_scale = Arith<Real>::bm_scale(h * (ES::kappa * ES::kappa));
    const Real r = (Real)prm.r, omega = (Real)prm.omega, K = (Real)prm.K;
    const Real lc = (Real)prm.log_bump_c;
    const Real rho = (Real)prm.rho;
    // per-asset constants, read as uniform scalars where they are used.
    // The Cholesky factor of the uniform correlation rho 11' + (1 - rho) I
    // has columns constant below the diagonal (Lcol[k] = L[j][k], j > k),
    // so (L G)_j = S_j + L_jj G_j with S_{j+1} = S_j + Lcol[j] G_j -- the
    // terms of sum_k L_jk G_k in the same order, O(d) instead of O(d^2)
    const AssetConsts<Real> &ac = asset_consts<Real>(prm);
    // FP64 one-problem kernels read the per-asset constants of the Euler
    // step again for every group of steps (RELOAD; cbase is then the
    // address of prm in constant memory)
    constexpr bool kReloadConsts = RELOAD && sizeof(Real) == 8;
    const Real tscale = Real(2) / T;
    Real neg_half_hk = Real(-0.5) * ES::kappa * h;
    // (FP64 d = 3: opaque, so that its scalar operands are not kept beside
    // it, which would overflow the scalar registers)
    if constexpr (sizeof(Real) == 8 && D == 3) asm volatile("" : "+v"(neg_half_hk));
    const Real hk = ES::kappa * h;
    // The volatility levels as vector operands: the volatility's fused
    // multiply-add has another scalar operand (level a) already, and a
    // second one costs a register move per asset and step.  At d = 10
    // outside the FP32 cubic form the vector registers are the scarcer ones
    // (the moves are cheaper than the spills that ten more live registers
    // cause).
    constexpr bool kVecLevel = D <= 5 || (sizeof(Real) == 4 && kCubic);
    Real lev[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
        lev[j] = ac.level[j];
        if constexpr (kVecLevel) asm volatile("" : "+v"(lev[j]));
    }
    // gfx950 issues a 32-bit vector instruction whose operands are all
    // vector registers in two cycles, one with a scalar or literal operand
    // in four.  The FP32 kernels up to d = 5 and in the cubic form therefore
    // also hold the other loop-invariant operands of the Euler step (level a,
    // (r - delta) h kappa) and the constants of the uniform map in vector
    // registers.
    constexpr bool kVecConst = sizeof(Real) == 4 && kVecLevel;
    Real lva[D], dhk[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
        lva[j] = ac.level_a[j];
        dhk[j] = ac.drift[j] * hk;
        if constexpr (kVecConst) asm volatile("" : "+v"(lva[j]), "+v"(dhk[j]));
    }
    Real c32 = Real(0x1p-32), c33 = Real(0x1p-33);
    if constexpr (kVecConst) asm volatile("" : "+v"(c32), "+v"(c33));
    // X and the normals G at the step j* of each path: written to LDS by
    // the one step that matches, a store under the lane mask, where a
    // select in every step would take two vector-ALU slots per asset
    struct alignas(2 * sizeof(Real)) Rec {
        Real y, g;
    };
    __shared__ Rec rec[D][kBlock];

    // this lane's paths: count, mean and sum of squared deviations, updated
    // path by path (Welford), so the sum of squares never dwarfs the spread
    int cnt = 0;
    double mean = 0.0, m2 = 0.0;
    // FP32 paths on the cubic form use the matrix cores, whose products need
    // every lane of the wave: its lanes beyond M run a path that is not counted
    constexpr bool kWholeWave = kCubic && sizeof(Real) == 4;
    for (int rr = 0; rr < passes; ++rr) {
        int m = (g * prm.paths_per_lane + rr) * kBlock + (int)threadIdx.x;
        if constexpr (kWholeWave) {
            if (__builtin_amdgcn_readfirstlane(m & ~63) >= prm.M) break;
        } else {
            if (m >= prm.M) break;
        }

        // U, j* = floor(U N) and theta = U N - j* in integer arithmetic
        const u32x4 wu = block((uint32_t)m, 1u << 24);
        const uint64_t num = (2ull * wu.x + 1ull) * (uint64_t)prm.N;
        const int jstar = (int)(num >> 33);
        const Real theta = Arith<Real>::frac33(num);
        const Real U = Arith<Real>::u01(wu.x);
        const Real tau = t0 + (T - t0) * U;

        Real X[D];
#pragma unroll
        for (int j = 0; j < D; ++j) X[j] = ES::to((Real)row[1 + j], lc);
        if (still) {
#pragma unroll
            for (int j = 0; j < D; ++j) rec[j][threadIdx.x] = Rec{X[j], Real(0)};
        }
        for (int grp = 0; grp < ngroups; ++grp) {
            // FP64: the per-asset constants of the step are read again for
            // every group of steps through an address the compiler cannot
            // see through (scalar loads from the constant cache); held
            // across the loop they overflow the scalar registers and come
            // back from vector-register lanes with one vector instruction
            // per use
            Real G[4 * NB];
            auto normals = [&](auto bc) {
                constexpr int b = decltype(bc)::value;
                const u32x4 w = block((uint32_t)m, (uint32_t)(grp * NB + b));
                Arith<Real>::box_muller(w.x, w.y, step_scale, G[4 * b],
                                        G[4 * b + 1], c32, c33);
                Arith<Real>::box_muller(w.z, w.w, step_scale, G[4 * b + 2],
                                        G[4 * b + 3], c32, c33);
            };
            if constexpr (!kLateNormals) static_for<NB>(normals);
            auto steps = [&](auto &acs) {
            static_for<SG>([&](auto sc) {
                constexpr int ss = decltype(sc)::value;
                const int s = grp * SG + ss;
                if (s < prm.N) {
                    // the blocks first needed by this step
                    constexpr int b0 = (ss * D + 3) / 4, b1 = (ss * D + D + 3) / 4;
                    if constexpr (kLateNormals)
                        static_for<b1 - b0>([&](auto bc) {
                            normals(std::integral_constant<int, b0 + decltype(bc)::value>{});
                        });
                    if (s == jstar) {
#pragma unroll
                        for (int j = 0; j < D; ++j)
                            rec[j][threadIdx.x] = Rec{X[j], G[ss * D + j]};
                    }
                    const VolTime<Real> vt = vol_time<VOL>(t0 + Real(s) * h, r);
                    Real S = Real(0);
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        // kappa sqrt(h) (L G)_j; the first row of the Cholesky
                        // factor of a correlation matrix is (1, 0, ..., 0)
                        Real lg = G[ss * D];
                        if (j > 0) lg = fma(acs.Ldiag[j], G[ss * D + j], S);
                        if (j + 1 < D) S = j == 0 ? acs.Lcol[0] * G[ss * D]
                                                  : fma(acs.Lcol[j], G[ss * D + j], S);
                        const Real sig = ES::vol(lev[j],
                                                 kReloadConsts ? acs.level_a[j] : lva[j],
                                                 acs.spot[j], vt, X[j]);
                        // X += (r - delta - sigma^2/2) h + sigma sqrt(h) (L G)
                        //    = X + (r - delta) h + sigma (sqrt(h) (L G) - h sigma / 2),
                        // every term times kappa
                        const Real inner = fma(sig, fma(neg_half_hk, sig, lg), X[j]);
                        if constexpr (kVecConst) X[j] = inner + dhk[j];
                        else X[j] = fma(acs.drift[j], hk, inner);
                    }
                }
            });
            };
            if constexpr (kReloadConsts) steps(reload_consts<Real>(cbase));
            else steps(ac);
        }

        // frozen coefficients at the last node t_{j*} and X at tau: the
        // bridge normals are scaled by sqrt(theta (1 - theta) h)
        const Real bridge_scale =
            Arith<Real>::bm_scale(theta * (Real(1) - theta) * h);
        Real Gb[4 * NBB];
#pragma unroll
        for (int b = 0; b < NBB; ++b) {
            const u32x4 w = block((uint32_t)m, (1u << 24) | (uint32_t)(1 + b));
            Arith<Real>::box_muller(w.x, w.y, bridge_scale, Gb[4 * b],
                                    Gb[4 * b + 1]);
            Arith<Real>::box_muller(w.z, w.w, bridge_scale, Gb[4 * b + 2],
                                    Gb[4 * b + 3]);
        }
        // back to x: the state at T and at t_{j*} with sqrt(h) (L G) of the
        // step j* (every j* < N is a step of the path, so each lane has
        // written its own record)
        Real Xs[D], LGs[D];
        {
            Real Sr = Real(0);
#pragma unroll
            for (int j = 0; j < D; ++j) {
                const Rec rj = rec[j][threadIdx.x];
                Xs[j] = ES::from(rj.y, lc);
                Real lg = rj.g;
                if (j > 0) lg = fma(ac.Ldiag[j], rj.g, Sr);
                if (j + 1 < D) Sr = j == 0 ? ac.Lcol[0] * rj.g : fma(ac.Lcol[j], rj.g, Sr);
                LGs[j] = lg * (Real(1) / ES::kappa);
                X[j] = ES::from(X[j], lc);
            }
        }
        Real sgs[D], bst[D], Xt[D];
        Real Sb = Real(0);
        const VolTime<Real> vts = vol_time<VOL>(t0 + Real(jstar) * h, r);
#pragma unroll
        for (int j = 0; j < D; ++j) {
            Real lgb = Gb[0];
            if (j > 0) lgb = fma(ac.Ldiag[j], Gb[j], Sb);
            if (j + 1 < D) Sb = j == 0 ? ac.Lcol[0] * Gb[0] : fma(ac.Lcol[j], Gb[j], Sb);
            sgs[j] = local_vol<VOL>(ac.level[j], ac.level_a[j], lc, ac.spot[j], vts,
                                    Xs[j]);
            if constexpr (kOpaqueVol) asm volatile("" : "+v"(sgs[j]));
            bst[j] = fma(Real(-0.5) * sgs[j], sgs[j], ac.drift[j]);
            Xt[j] = Xs[j] + bst[j] * theta * h +
                    sgs[j] * fma(theta, LGs[j], lgb);
        }

        // payoff at tau (for the penalty) and the terminal term
        // Phi(X_T) - u^k(T, X_T)
        Real phi_tau = payoff<D>(prm.payoff, K, Xt);
        Real u = Real(0), gen = Real(0), uT = Real(0), terminal;
        if constexpr (OP != kOpBasis) {
            // u^k = h[y] of the kernel operator (Section 3.2) in its
            // normalised form h = S1 / S0, S0 = sum_i w_i, S1 = sum_i y_i w_i,
            // w_i = exp(-min(|z - z_i|^2 / (2 b^2), clamp)) in the mapped
            // coordinates z; a clamped weight is constant (no derivative).
            // With L the frozen generator (d_t + b*.grad + sum_jk a_jk d_jk,
            // a_jk = sigma*_j sigma*_k C_jk / 2), in z units,
            //   L h = [L S1 - h L S0 - 2 sum_jk a_jk d_j h d_k S0] / S0,
            //   d_j h = (d_j S1 - h d_j S0) / S0,
            // and L w_i / w_i = l(dz), the polynomial below.  The table rows
            // {z_0, .., z_d, y} are uniform across the workgroup (scalar loads).
            const Real b2 = Real(prm.kbw * prm.kbw);
            const Real invb2 = Real(1) / b2;
            // FP32: the exponent in base 2 (log2 e folded into the scale and
            // the clamp), so that a weight is one v_exp_f32
            constexpr bool kF32 = sizeof(Real) == 4;
            const Real kq = Real(0.5 / (prm.kbw * prm.kbw) * (kF32 ? 1.4426950408889634 : 1.0));
            const Real clamp = Real(kKernelClamp * (kF32 ? 1.4426950408889634 : 1.0));
            auto weight = [&](Real e) {
                if constexpr (kF32) return __builtin_amdgcn_exp2f(-fminf(e, clamp));
                else return ::exp(-fmin(e, clamp));
            };
            Real zt[DP], zT[DP];
            zt[0] = tau * tscale - Real(1);
            zT[0] = Real(1);
#pragma unroll
            for (int j = 0; j < D; ++j) {
                zt[1 + j] = (Xt[j] - ac.mid[j]) * ac.scale[j];
                zT[1 + j] = (X[j] - ac.mid[j]) * ac.scale[j];
            }
            // l(dz) = c0 + ct dz_0 + sum_j cj dz_j + sum_{j<=k} cjk dz_j dz_k
            Real ajk[D][D];
#pragma unroll
            for (int j = 0; j < D; ++j)
#pragma unroll
                for (int k = 0; k < D; ++k)
                    ajk[j][k] = Real(0.5) * sgs[j] * sgs[k] * (j == k ? Real(1) : rho) *
                                ac.scale[j] * ac.scale[k];
            const Real ct = -tscale * invb2;
            Real cj[D], cjk[D][D], c0 = Real(0);
#pragma unroll
            for (int j = 0; j < D; ++j) {
                cj[j] = -bst[j] * ac.scale[j] * invb2;
                c0 -= ajk[j][j] * invb2;
#pragma unroll
                for (int k = j; k < D; ++k)
                    cjk[j][k] = (j == k ? ajk[j][j] : Real(2) * ajk[j][k]) * invb2 * invb2;
            }
            Real S0 = 0, S1 = 0, L0 = 0, L1 = 0, S0T = 0, S1T = 0;
            Real G0[D], G1[D]; // sum w dz_j and sum y w dz_j (unclamped weights)
#pragma unroll
            for (int j = 0; j < D; ++j) G0[j] = G1[j] = Real(0);
            if constexpr (OP == kOpProduct) {
                // Product points: e^{-e} of a pair is the product of its
                // time node's and its spatial point's factors, so a pair
                // costs a product, a maximum (the clamp: max(e^{-e}, e^{-clamp})
                // = e^{-min(e, clamp)}) and its share of the sums instead of
                // two exponentials and the squared distances (FP32, d = 1:
                // 512 points, M = 1000: 189 -> 109 us).  The path's time
                // factors wait in LDS; the sums over a spatial point's times
                // of the unclamped weights and their first moments in dz_0
                // give the moments in dz_j.
                __shared__ Real kop_w[kKopTimes][kBlock];
                const int nt = prm.kop_nt, ns = prm.n / nt, stride = kop_row(D, nt);
                auto factor = [&](Real e) {
                    if constexpr (kF32) return __builtin_amdgcn_exp2f(-e);
                    else return ::exp(-e);
                };
                const Real wc = factor(clamp);
                for (int a = 0; a < nt; ++a) {
                    const Real d0 = zt[0] - gamma[2 * a];
                    kop_w[a][threadIdx.x] = factor(d0 * d0 * kq);
                }
                for (int sp = 0; sp < ns; ++sp) {
                    const auto row = gamma + (2 * kKopTimes + (size_t)sp * stride);
                    Real dz[D], e = Real(0), eT = Real(0);
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        dz[j] = zt[1 + j] - row[j];
                        e = fma(dz[j], dz[j], e);
                        const Real dT = zT[1 + j] - row[j];
                        eT = fma(dT, dT, eT);
                    }
                    const Real wx = factor(e * kq), wxT = factor(eT * kq);
                    // sums over the times: unclamped weights, with y, and both
                    // with dz_0
                    Real A0 = 0, B0 = 0, A1 = 0, B1 = 0;
#pragma unroll 4
                    for (int a = 0; a < nt; ++a) {
                        const Real y = row[D + a], d0 = zt[0] - gamma[2 * a];
                        const Real w = kop_w[a][threadIdx.x] * wx;
                        const Real wm = fmax(w, wc);
                        S0 += wm;
                        S1 = fma(wm, y, S1);
                        const Real wd = w >= wc ? w : Real(0), wyd = wd * y;
                        A0 += wd;
                        B0 += wyd;
                        A1 = fma(wd, d0, A1);
                        B1 = fma(wyd, d0, B1);
                        const Real wT = fmax(gamma[2 * a + 1] * wxT, wc);
                        S0T += wT;
                        S1T = fma(wT, y, S1T);
                    }
                    Real l = c0;
#pragma unroll
                    for (int j = 0; j < D; ++j) {
                        l = fma(cj[j], dz[j], l);
#pragma unroll
                        for (int k = j; k < D; ++k) l = fma(cjk[j][k], dz[j] * dz[k], l);
                        G0[j] = fma(A0, dz[j], G0[j]);
                        G1[j] = fma(B0, dz[j], G1[j]);
                    }
                    L0 = fma(l, A0, fma(ct, A1, L0));
                    L1 = fma(l, B0, fma(ct, B1, L1));
                }
            } else {
#pragma unroll 4
            for (int q = 0; q < prm.n; ++q) {
                const auto row = gamma + (size_t)q * kKernelRow;
                Real dz[DP], qq = Real(0), qT = Real(0);
#pragma unroll
                for (int v = 0; v < DP; ++v) {
                    dz[v] = zt[v] - row[v];
                    qq = fma(dz[v], dz[v], qq);
                    const Real dT = zT[v] - row[v];
                    qT = fma(dT, dT, qT);
                }
                const Real y = row[1 + D];
                const Real e = qq * kq;
                const bool flat = e > clamp;
                const Real w = weight(e);
                const Real wy = w * y;
                S0 += w;
                S1 += wy;
                const Real wd = flat ? Real(0) : w, wyd = flat ? Real(0) : wy;
                Real l = fma(ct, dz[0], c0);
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    l = fma(cj[j], dz[1 + j], l);
#pragma unroll
                    for (int k = j; k < D; ++k) l = fma(cjk[j][k], dz[1 + j] * dz[1 + k], l);
                    G0[j] = fma(wd, dz[1 + j], G0[j]);
                    G1[j] = fma(wyd, dz[1 + j], G1[j]);
                }
                L0 = fma(wd, l, L0);
                L1 = fma(wyd, l, L1);
                const Real wT = weight(qT * kq);
                S0T += wT;
                S1T = fma(wT, y, S1T);
            }
            }
            u = S1 / S0;
            // d_j S = -G_j / b^2 (z units), d_j h = (d_j S1 - h d_j S0) / S0
            Real hj[D];
#pragma unroll
            for (int j = 0; j < D; ++j) hj[j] = -(G1[j] - u * G0[j]) * invb2 / S0;
            Real acc = L1 - u * L0;
#pragma unroll
            for (int j = 0; j < D; ++j)
#pragma unroll
                for (int k = 0; k < D; ++k)
                    acc -= Real(2) * ajk[j][k] * hj[j] * (-G0[k] * invb2);
            gen = acc / S0;
            uT = S1T / S0T;
            terminal = payoff<D>(prm.payoff, K, X) - uT;
        } else if constexpr (kCubic) {
            if constexpr (D >= 5) asm volatile("" : "+v"(phi_tau));
            terminal = payoff<D>(prm.payoff, K, X);
            Real z[DP], zT[D], sz[D], bz[D];
            z[0] = fma(tau, tscale, Real(-1));
#pragma unroll
            for (int j = 0; j < D; ++j) {
                z[1 + j] = (Xt[j] - ac.mid[j]) * ac.scale[j];
                zT[j] = (X[j] - ac.mid[j]) * ac.scale[j];
                sz[j] = sgs[j] * ac.scale[j];
                bz[j] = bst[j] * ac.scale[j];
            }
            // (the table's address is made opaque once per path, so that its
            // loads stay in the path's iteration instead of being hoisted out
            // of the path loop into registers)
            uint64_t pa = (uint64_t)(uintptr_t)&gamma[0];
            asm volatile("" : "+s"(pa));
            cubic_eval<D, kCubicKind>(pa, z, zT, sz, bz, rho, tscale, u, gen, uT);
            terminal -= uT;
        } else {
            if constexpr (D >= 5) asm volatile("" : "+v"(phi_tau));
            // basis row at (tau, X_tau) contracted with the channel table,
            // and the value u^k(T, X_T) (z_0 = 1 there, so every T_a(z_0) = 1)
            Real Tz[DP][ETA + 1], TzT[DP][ETA + 1];
            cheb<ETA>(tau * tscale - Real(1), Tz[0]);
#pragma unroll
            for (int a = 0; a <= ETA; ++a) TzT[0][a] = Real(1);
#pragma unroll
            for (int j = 0; j < D; ++j) {
                cheb<ETA>((Xt[j] - ac.mid[j]) * ac.scale[j], Tz[1 + j]);
                cheb<ETA>((X[j] - ac.mid[j]) * ac.scale[j], TzT[1 + j]);
            }
            // basis function l as the product of its non-zero Chebyshev
            // factors (at most eta of them), so that no earlier basis value
            // has to stay live in registers
            auto basis = [&](auto lc, const Real(&Tv)[DP][ETA + 1]) {
                constexpr int l = decltype(lc)::value;
                Real v = Real(1);
                static_for<DP>([&](auto vc) {
                    constexpr int w = decltype(vc)::value;
                    constexpr int e = BS::tab.nu[l][w];
                    if constexpr (e > 0) v *= Tv[w][e];
                });
                return v;
            };
            // fold of channel c of V (this lane's path) into u and the
            // frozen generator
            auto fold = [&](auto cc, Real vc) {
                constexpr int c = decltype(cc)::value;
                if constexpr (c == 0) {
                    u = vc;
                } else if constexpr (c == 1) {
                    gen += vc;
                } else if constexpr (c < 2 + D) {
                    gen += bst[c - 2] * vc;
                } else {
                    constexpr int j = hess_j(D, c - 2 - D);
                    constexpr int k = hess_k(D, c - 2 - D);
                    const Real cov = (j == k) ? Real(0.5) * sgs[j] * sgs[j]
                                              : rho * sgs[j] * sgs[k];
                    gen += cov * vc;
                }
            };
            {
                // V = B Gamma over the live rows of the channel table only
                // (channel_row_live): the derivative channels of a
                // polynomial over a downward-closed set have lower degree,
                // so the 67 channels of d = 10, eta = 3 need 1,882 of the
                // 364 x 67 products and the 22 of d = 5, eta = 3 need 357 of
                // 84 x 22.  The packed table is uniform across the wave:
                // each fused multiply-add takes its entry as a scalar
                // operand and the basis value as the vector one.  The
                // table's address is made opaque once per path, so that its
                // loads stay in the path's iteration instead of being
                // hoisted out of the path loop into registers.
                using CR = ChannelRows<DP, ETA, Q>;
                uint64_t pa = (uint64_t)(uintptr_t)&gamma[0];
                asm volatile("" : "+s"(pa));
                const auto pk = (const __attribute__((address_space(4))) Real *)pa;
                // u^k(T, X_T): z_0 = 1, so the functions of each spatial
                // multi-index share one coefficient, their sum (after the
                // channels in the table, in the order of the rows with time
                // degree zero)
                static_for<NP>([&](auto lc) {
                    constexpr int l = decltype(lc)::value;
                    if constexpr (BS::tab.nu[l][0] == 0) {
                        constexpr int e = CR::tab.goff[NP] + terminal_index<BS>(l);
                        uT = fma(basis(lc, TzT), pk[e], uT);
                    }
                });
                terminal = payoff<D>(prm.payoff, K, X) - uT;
                // second derivatives first, one channel at a time, each
                // folded as soon as it is complete: their live rows are
                // those of degree at most eta - 2 (at total degree 3 the
                // constant and the linear ones, whose basis values are the
                // coordinates themselves), so no accumulator of theirs
                // stays live through the rest of the rows
                static_for<CR::tab.NH>([&](auto hc) {
                    constexpr int h = decltype(hc)::value;
                    Real vc = Real(0);
                    static_for<NP>([&](auto lc) {
                        constexpr int e = CR::tab.hpos[h][decltype(lc)::value];
                        if constexpr (e >= 0) vc = fma(basis(lc, Tz), pk[e], vc);
                    });
                    fold(std::integral_constant<int, 2 + D + h>{}, vc);
                });
                // then u, d_t u and the gradient over every row in order
                Real V[2 + D];
#pragma unroll
                for (int c = 0; c < 2 + D; ++c) V[c] = Real(0);
                static_for<NP>([&](auto lc) {
                    constexpr int l = decltype(lc)::value;
                    constexpr int e0 = CR::tab.goff[l];
                    const Real b = basis(lc, Tz);
                    V[0] = fma(b, pk[l], V[0]);
                    static_for<CR::tab.goff[l + 1] - e0>([&](auto ec) {
                        constexpr int e = e0 + decltype(ec)::value;
                        constexpr int c = CR::tab.gch[e - CR::tab.goff[0]];
                        V[c] = fma(b, pk[e], V[c]);
                    });
                });
                static_for<2 + D>([&](auto cc) { fold(cc, V[decltype(cc)::value]); });
            }
        }

        // penalised driver f = -r u + omega (Phi - u)_+ and the path term
        const Real f = -r * u + omega * fmax(phi_tau - u, Real(0));
        const Real a = (T - t0) * (f + gen) + terminal;
        const double ad = (double)a;
        if constexpr (kWholeWave)
            if (m >= prm.M) continue;
        cnt += 1;
        const double dev = ad - mean;
        mean = rr == 0 ? ad : mean + dev / (double)cnt;
        m2 = fma(dev, ad - mean, m2);
    }

    // fixed-order reduction of the lanes' moments (combine_moments):
    // butterfly within the wavefront, then waves in order through LDS
    double n = (double)cnt;
    if (__all(cnt == __builtin_amdgcn_readfirstlane(cnt))) {
        // lanes with as many paths each (every wave but the one that M ends
        // in): the same combination with its quotients n_b / n = 1/2
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double d = __shfl_xor(mean, off) - mean, m2b = __shfl_xor(m2, off);
            mean = fma(d, 0.5, mean);
            m2 = fma(d * d, 0.5 * n, m2 + m2b);
            n += n;
        }
    } else {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double nb = __shfl_xor(n, off), mb = __shfl_xor(mean, off),
                         m2b = __shfl_xor(m2, off);
            combine_moments(n, mean, m2, nb, mb, m2b);
        }
    }
    __shared__ double red[3][kBlock / 64];
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wave] = n;
        red[1][wave] = mean;
        red[2][wave] = m2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double nw = 0.0, mw = 0.0, m2w = 0.0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w)
            combine_moments(nw, mw, m2w, red[0][w], red[1][w], red[2][w]);
        out[0] = mw;
        out[1] = m2w;
    }
    __syncthreads(); // red[] may be reused by the next tile
}

// Waves per SIMD the register allocation must allow.  The d = 5 FP64 and the
// d = 10 FP32 kernels are held to three waves (168 registers a lane): left to
// themselves those of the channel form took 180-240 and ran at two, and at three
// they ran 10-17% faster, with what does not fit (76 to 148 bytes a lane at d = 5
// in FP64, up to 20 at d = 10) stored and reloaded once per path, outside the
// Euler loop.  (FP32 takes 74 to 101 registers at d = 5, five waves, and 76 to 168
// at d = 10.)  At four waves (128 registers) the FP64 d = 5 kernel spills inside
// the Euler loop and takes 60% longer, and the FP32 d = 10 one gained 2%.  d = 10 in
// FP64 runs at two waves, with up to 132 bytes a lane at degree 2 and 20 at degree
// 3.  d = 2 in FP64 takes 105 to 142 registers, within the bound of two waves, and
// runs at four or three.
template <int D, typename Real>
constexpr int min_waves()
{
    if (D >= 10) return sizeof(Real) == 4 ? 3 : 2;
    if (D == 5) return 3;
    if (D == 2) return sizeof(Real) == 4 ? 1 : 2;
    return 1;
}

// One problem: workgroup b runs a tile (i, g) of point i = b / groups and
// writes its moments to partial[2 (i groups + g)].
template <int D, int ETA, typename Real, int VOL, int Q, int OP = kOpBasis>
__global__ __launch_bounds__(kBlock, (min_waves<D, Real>())) void path_kernel(
    const PathParams prm, const double *__restrict__ pts,
    const Real *__restrict__ gamma, double *__restrict__ partial)
{
    const int i = blockIdx.x / prm.groups;
    // Consecutive workgroups go to the 8 XCDs in turn and, within one, to its
    // 4 shader engines: 32 of them, so that 16 points of two groups or more
    // meet every engine.  The groups move on by one every 16 points; else the
    // last group, whose paths end at M, would fall to the same engines at
    // every point (n = 3000, M = 3000, eight groups of two blocks: 4.2 ms,
    // 3.2 with the turn).
    const int g = (blockIdx.x - i * prm.groups + (i >> 4)) % prm.groups;
    fill_path_tables<Real>();
    // prm is the first kernel argument: its copy at the start of the
    // kernel-argument segment is the one the scalar loads read
    run_tile<D, ETA, Real, VOL, Q, const Real *__restrict__, OP, true>(
        prm, (uint64_t)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr(), pts,
        gamma, i, g, partial + 2 * ((size_t)i * prm.groups + g));
}

// Many problems of one kernel signature in one persistent launch.  Tiles
// of problem q are tile_begin[q] .. tile_begin[q+1]-1 (problems ordered by
// decreasing tile cost); every workgroup takes the next tile from an
// atomic counter until none is left -- dynamic per-tile dispatch.  A tile
// computes exactly what the one-problem kernel computes for the same
// (i, g), so a problem's result does not depend on the batch.
template <int D, int ETA, typename Real, int VOL, int Q>
__global__ __launch_bounds__(kBlock, (min_waves<D, Real>())) void batch_path_kernel(
    const BatchTileDesc *__restrict__ probs, int nprob,
    const long long *__restrict__ tile_begin, unsigned int *counter)
{
    __shared__ long long next;
    const long long total = tile_begin[nprob];
    fill_path_tables<Real>();
    for (;;) {
        if (threadIdx.x == 0) next = (long long)atomicAdd(counter, 1u);
        __syncthreads();
        // the tile index is the same in every lane: keep it (and the
        // problem lookup and parameter loads that follow) scalar
        const long long tl = next;
        const long long t =
            (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(
                             (int)(tl >> 32))
                         << 32) |
                        (unsigned)__builtin_amdgcn_readfirstlane((int)tl));
        __syncthreads();
        if (t >= total) break;
        int lo = 0, hi = nprob - 1; // last q with tile_begin[q] <= t
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tile_begin[mid] <= t) lo = mid;
            else hi = mid - 1;
        }
        const BatchTileDesc &q = probs[lo];
        const long long local = t - tile_begin[lo];
        const int i = (int)(local / q.prm.groups);
        const int g = (int)(local - (long long)i * q.prm.groups);
        using ConstReal = const __attribute__((address_space(4))) Real *;
        run_tile<D, ETA, Real, VOL, Q>(q.prm, 0, q.pts, (ConstReal)q.gamma, i, g,
                                    q.partial + 2 * local);
    }
}

// ---------------------------------------------------------------------------
// Instantiation and dispatch.  For one (d, eta) the kernels exist for FP32
// paths and, when FP64 is set, FP64 paths; for the constant and bump
// volatilities and, when DUP is set, the Dupire-type one.
// ---------------------------------------------------------------------------
template <typename T>
struct TypeTag {
    using type = T;
};

// Path precisions a set is instantiated for (a bit set)
enum PrecisionSet { kPrecF32 = 1, kPrecF64 = 2, kPrecBoth = 3 };

// calls f(TypeTag<Real>, integral_constant<VOL>) for the variant at hand;
// hipErrorInvalidValue when it is not instantiated
template <int D, int E, int PREC, bool DUP, typename F>
hipError_t dispatch_variant(bool fp32, int vol, F &&f)
{
    auto by_vol = [&](auto rt) -> hipError_t {
        if (vol == kVolConst) return f(rt, std::integral_constant<int, kVolConst>{});
        if (vol == kVolBump) return f(rt, std::integral_constant<int, kVolBump>{});
        if constexpr (DUP) {
            if (vol == kVolDupire) return f(rt, std::integral_constant<int, kVolDupire>{});
        }
        return hipErrorInvalidValue;
    };
    if (fp32) {
        if constexpr ((PREC & kPrecF32) != 0) return by_vol(TypeTag<float>{});
    } else {
        if constexpr ((PREC & kPrecF64) != 0) return by_vol(TypeTag<double>{});
    }
    return hipErrorInvalidValue;
}

template <int D, int E, int Q>
int copy_index_table(int8_t *nu, int cap)
{
    constexpr int DP = D + 1;
    constexpr auto &t = Basis<DP, E, Q>::tab;
    constexpr int P = Basis<DP, E, Q>::P;
    if (nu && cap >= P)
        for (int l = 0; l < P; ++l)
            for (int v = 0; v < DP; ++v) nu[l * DP + v] = t.nu[l][v];
    return P;
}

} // namespace bsde

// Defines launch_path_dD, index_table_dD, launch_batch_dD,
// batch_occupancy_dD and has_variant_dD for the (eta, q-norm, precisions,
// Dupire) sets listed by SETS(X) as X(E, Q, PREC, DUP), with q = Q / 10 and
// PREC a PrecisionSet.
// Path kernels of the kernel operator (Section 3.2) for d = D: FP32 and
// FP64 paths, constant and bump volatility; table = rows {z, y} or, when the
// problem has one, the product table.  A kernel for each: the product form's
// factors in LDS and its registers would cost the plain rows waves they have no
// use for (FP64 d = 1 four a SIMD to two, FP32 eight to six;
// 3000 uniform points, M = 300, N = 20, bump: 7.91 ms in one kernel for both,
// 7.21 apart in FP64 at d = 2, 6.59 and 6.27 at d = 1, 2.22 and 2.13 in FP32)
#define BSDE_DEFINE_KERNEL_OP(D)                                               \
    hipError_t launch_kernel_path_d##D(bool fp32, int blocks, hipStream_t s,   \
                                       const PathParams &prm,                  \
                                       const double *pts, const void *table,   \
                                       double *partial, hipEvent_t ev0,        \
                                       hipEvent_t ev1)                         \
    {                                                                          \
        return dispatch_variant<D, 1, kPrecBoth, false>(                            \
            fp32, prm.vol_kind, [&](auto rt, auto vt) -> hipError_t {          \
                using R = typename decltype(rt)::type;                         \
                constexpr int V = decltype(vt)::value;                         \
                if (prm.kop_nt > 0)                                            \
                    hipExtLaunchKernelGGL((path_kernel<D, 1, R, V, 10, kOpProduct>), \
                                          dim3(blocks), dim3(kBlock), 0, s, ev0, ev1, \
                                          0u, prm, pts, (const R *)table, partial); \
                else                                                           \
                    hipExtLaunchKernelGGL((path_kernel<D, 1, R, V, 10, kOpKernel>), \
                                          dim3(blocks), dim3(kBlock), 0, s, ev0, ev1, \
                                          0u, prm, pts, (const R *)table, partial); \
                return hipGetLastError();                                      \
            });                                                                \
    }

#define BSDE_DEFINE_DIMENSION(D, SETS) BSDE_DEFINE_DIMENSION_NAMED(D, D, SETS)
// the same for a second group of sets of dimension D in a translation unit
// of its own: the functions are named with NAME (launch_path_dNAME, ...)
#define BSDE_DEFINE_DIMENSION_NAMED(D, NAME, SETS)                             \
    hipError_t launch_path_d##NAME(int eta, int q10, bool fp32, int blocks,    \
                                hipStream_t s,                                 \
                                const PathParams &prm, const double *pts,      \
                                const void *gamma, double *partial,            \
                                hipEvent_t ev0, hipEvent_t ev1)                \
    {                                                                          \
        constexpr int D_ = D;                                                  \
        SETS(BSDE_PATH_SET)                                                    \
        return hipErrorInvalidValue;                                           \
    }                                                                          \
    int index_table_d##NAME(int eta, int q10, int8_t *nu, int cap)                \
    {                                                                          \
        constexpr int D_ = D;                                                  \
        SETS(BSDE_TABLE_SET)                                                   \
        return 0;                                                              \
    }                                                                          \
    hipError_t launch_batch_d##NAME(int eta, int q10, bool fp32, int vol,         \
                                 int blocks,                                   \
                                 hipStream_t s, const BatchTileDesc *probs,    \
                                 int nprob, const long long *tile_begin,       \
                                 unsigned int *counter)                        \
    {                                                                          \
        constexpr int D_ = D;                                                  \
        SETS(BSDE_BATCH_SET)                                                   \
        return hipErrorInvalidValue;                                           \
    }                                                                          \
    int batch_occupancy_d##NAME(int eta, int q10, bool fp32, int vol)             \
    {                                                                          \
        constexpr int D_ = D;                                                  \
        int nb = 0;                                                            \
        SETS(BSDE_OCC_SET)                                                     \
        return nb;                                                             \
    }                                                                          \
    bool has_variant_d##NAME(int eta, int q10, bool fp32, int vol)                \
    {                                                                          \
        constexpr int D_ = D;                                                  \
        SETS(BSDE_HAS_SET)                                                     \
        return false;                                                          \
    }

#define BSDE_PATH_SET(E, Q, PREC, DUP)                                          \
    if (eta == E && q10 == Q)                                                  \
        return dispatch_variant<D_, E, PREC, DUP>(                              \
            fp32, prm.vol_kind, [&](auto rt, auto vt) -> hipError_t {          \
                using R = typename decltype(rt)::type;                         \
                /* ev0/ev1 (may be null) take the start and end times   \
                   of the dispatch itself: no marker packets around it */  \
                hipExtLaunchKernelGGL(                                         \
                    (path_kernel<D_, E, R, decltype(vt)::value, Q>),           \
                    dim3(blocks), dim3(kBlock), 0, s, ev0, ev1, 0u, prm, pts,  \
                    (const R *)gamma, partial);                                \
                return hipGetLastError();                                      \
            });
#define BSDE_TABLE_SET(E, Q, PREC, DUP)                                         \
    if (eta == E && q10 == Q) return copy_index_table<D_, E, Q>(nu, cap);
#define BSDE_BATCH_SET(E, Q, PREC, DUP)                                         \
    if (eta == E && q10 == Q)                                                  \
        return dispatch_variant<D_, E, PREC, DUP>(                              \
            fp32, vol, [&](auto rt, auto vt) -> hipError_t {                   \
                using R = typename decltype(rt)::type;                         \
                hipLaunchKernelGGL(                                            \
                    (batch_path_kernel<D_, E, R, decltype(vt)::value, Q>),     \
                    dim3(blocks), dim3(kBlock), 0, s, probs, nprob,            \
                    tile_begin, counter);                                      \
                return hipGetLastError();                                      \
            });
#define BSDE_OCC_SET(E, Q, PREC, DUP)                                           \
    if (eta == E && q10 == Q)                                                  \
        (void)dispatch_variant<D_, E, PREC, DUP>(                               \
            fp32, vol, [&](auto rt, auto vt) -> hipError_t {                   \
                using R = typename decltype(rt)::type;                         \
                return hipOccupancyMaxActiveBlocksPerMultiprocessor(           \
                    &nb, batch_path_kernel<D_, E, R, decltype(vt)::value, Q>,  \
                    kBlock, 0);                                                \
            });
#define BSDE_HAS_SET(E, Q, PREC, DUP)                                           \
    if (eta == E && q10 == Q)                                                  \
        return dispatch_variant<D_, E, PREC, DUP>(                              \
                   fp32, vol, [](auto, auto) { return hipSuccess; }) ==        \
               hipSuccess;
