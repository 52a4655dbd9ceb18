// gfx950 kernels of libtotalconv: reduced Wigner elements by the l-recursion
// and the total-convolution sum with its adjoint (Prezeau & Reinecke,
// arXiv:1002.1050, Secs. 3.2 and 4).
//
// Mapping.  A workgroup owns one (mb, msky) column and NT*R ring slots of it;
// each lane walks R chains (one per ring slot) up in l, in lock-step, so the
// per-l recursion coefficients and weights are uniform across the workgroup.
// A lane takes R consecutive slots and a wave 64 R (slots run from the pole to
// the equator), so that the chains of a wave share their regime: all still below
// the skip threshold, or not, over the same stretch of l.
// They are built per block of NT values of l in LDS by the whole workgroup and read
// back as broadcasts.  A ring slot is either a mirror pair (beta, pi - beta) -- one
// recursion serves both rings through d^l_{-mb,msky}(pi-beta) =
// (-1)^(l-msky) d^l_{mb,msky}(beta) (appendix eq. pithetasym) -- or a single ring.
//
// Numbers.  Everything is FP64.  The seed at l0 = max(|mb|,|msky|) is formed
// as a logarithm in double-double (Sec. 3.2 eq. logstart) and split into a
// significand and a power of two.  While a chain's value is below 2^-900 it is
// carried as d * 2^E with E < 0 a multiple of 900; every RS_STEPS steps a scaled chain
// that has grown past 1 is multiplied by exactly 2^-900 (E += 900), and at E = 0 it is a
// plain double, as Sec. 3.2 prescribes (its S = 2^90 with a larger step).  The checks are wave-uniform branches, so the inner
// loop has no per-step branches.

#include <hip/hip_runtime.h>

#include "tc_internal.h"

namespace tc {
namespace {

// Tile parameters (template arguments): R chains per lane, NT lanes per workgroup, TB
// row times per block of the adjoint's emitted sums (the forward ignores it); TR is kept in the
// tile triple (value 4) and shapes no kernel: the adjoint's row sums move every step.
constexpr int TS = 8;         // steps per unrolled group
constexpr int FOLD_EXP = -900;  // fold scaled values into plain doubles at 2^-900
// A step of the normalised walk (below) multiplies max(|e^l|, |e^{l-1}|) by at most
// alpha F0 |x - F1| + 1 <= 2 (l+1) 2 + 1 < 2^17 for l <= 16384 (F0 <= l+1, |x - F1| <= 2,
// alpha <= 2).
constexpr int GROWTH_BITS_PER_STEP = 17;
// Chains are looked at every RS_STEPS steps.  A chain left scaled (E < 0) then is below 1 in its
// own units, so its significand stays below 2^(17 RS_STEPS) = 2^544, and below 2^-900 in truth, so
// it stays below 2^-356: it is not rescaled and not tested for the skip until the next look.
// Plain chains are tested with the staged bound of the next RS_STEPS steps' growth (grow_bits).
constexpr int RS_STEPS = 32;
constexpr int SKIP_EXP_MAX = -(FOLD_EXP + GROWTH_BITS_PER_STEP * RS_STEPS);  // 356
static_assert(RS_STEPS % TS == 0 && GROWTH_BITS_PER_STEP * RS_STEPS < 1023 && SKIP_EXP_MAX >= 100,
              "look period: no overflow of a scaled significand, no missed hot chain at skip 2^-100");

__device__ __forceinline__ bool wave_any(bool p) { return __ballot(p) != 0ull; }

// Loads and stores through a pointer taken from a struct in memory (the batched
// kernels read their arguments from a device array) are marked as global memory, so that
// they compile to global rather than flat instructions, with a scalar base where the
// address is uniform.
template <class T>
__device__ __forceinline__ T ldg(const T* p) { return *(const __attribute__((address_space(1))) T*)p; }
template <class T>
__device__ __forceinline__ void stg(T* p, T v) { *(__attribute__((address_space(1))) T*)p = v; }
// double2 is a class (its copy takes a generic reference): move it as a native vector
typedef double native_double2 __attribute__((ext_vector_type(2)));
template <>
__device__ __forceinline__ double2 ldg(const double2* p)
{
    const native_double2 v = *(const __attribute__((address_space(1))) native_double2*)p;
    return make_double2(v.x, v.y);
}
template <>
__device__ __forceinline__ void stg(double2* p, double2 v)
{
    native_double2 w;
    w.x = v.x;
    w.y = v.y;
    *(__attribute__((address_space(1))) native_double2*)p = w;
}

// Minimum resident waves per SIMD asked of the compiler for R chains per lane
// (bounds the VGPR budget: 512 / waves).
template <int R>
constexpr int min_waves() { return R >= 8 ? 2 : (R >= 4 ? 3 : 4); }

// Polarised forward: NC > 1 outputs carry 4 NC sums per chain, so their budget is one
// step lower than the scalar kernel's; the summed output (NC = 1) keeps the scalar one.
template <int R, int NC, int NP>
constexpr int fwd_min_waves() { return NC == 1 ? min_waves<R>() : (R >= 4 ? 2 : 3); }

// The forward's even / odd form holds 2 complex sums per chain in the same registers but
// needs fewer temporaries: R = 4 fits 4 waves per SIMD (its few spills sit outside the
// step loop), which hides more of each step's broadcast LDS reads.
template <int R>
constexpr int rows_min_waves() { return R >= 8 ? 2 : 4; }

// The adjoint's LDS (46 KB per workgroup with TB = 32, 80 KB with TB = 64; mostly the emitted
// row sums of two blocks) caps residency at 3 or 2 workgroups (waves per SIMD) per CU.
template <int R, int TB>
constexpr int adj_min_waves() { return min_waves<R>() < (TB >= 64 ? 2 : 3) ? min_waves<R>() : (TB >= 64 ? 2 : 3); }

// ------------------------------------------------------------- double-double
__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e)
{
    s = a + b;
    const double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

__device__ __forceinline__ void fast_two_sum(double a, double b, double& s, double& e)
{
    s = a + b;
    e = b - (s - a);
}

// (sh, sl) += n * (ah + al), n an integer held exactly in a double
__device__ __forceinline__ void dd_add_times(double& sh, double& sl, double n, double ah, double al)
{
    const double ph = n * ah;
    const double pl = fma(n, ah, -ph) + n * al;
    double s, e;
    two_sum(sh, ph, s, e);
    e += sl + pl;
    fast_two_sum(s, e, sh, sl);
}

__device__ __forceinline__ void dd_mul(double ah, double al, double bh, double bl, double& yh, double& yl)
{
    const double p = ah * bh;
    const double e = fma(ah, bh, -p) + (ah * bl + al * bh);
    fast_two_sum(p, e, yh, yl);
}

// --------------------------------------------------------------------- seeds
// Seed d^{l0}_{mb,ms} = A c^p (+-s)^q at l0 = max(|mb|,|ms|), c = cos(beta/2),
// s = sin(beta/2) (Sec. 3.2 eqs. ini1..ini2; the printed row labels are read as
// d_{l,m}, d_{-l,m}, d_{m,l}, d_{m,-l}).
struct SeedShape {
    int p, q;
    bool neg;
};

__device__ __forceinline__ SeedShape seed_shape(int mb, int ms)
{
    const int amb = abs(mb), ams = abs(ms);
    const int l0 = max(amb, ams);
    SeedShape s;
    if (ams >= amb) {
        if (ms >= 0) { s.p = l0 + mb; s.q = l0 - mb; s.neg = false; }   // d_{m,l}
        else         { s.p = l0 - mb; s.q = l0 + mb; s.neg = (s.q & 1); }  // d_{m,-l}
    } else {
        if (mb > 0)  { s.p = l0 + ms; s.q = l0 - ms; s.neg = (s.q & 1); }  // d_{l,m}
        else         { s.p = l0 - ms; s.q = l0 + ms; s.neg = false; }   // d_{-l,m}
    }
    return s;
}

// ln|d| = lnA + p ln c + q ln s in double-double, then d = 2^f * 2^k.
// Returns the value in (d, E) form, d * 2^E: E = 0 and d plain when |d| >= 2^-900, otherwise E a
// negative multiple of 900 and |d| in [2^-899, 2).  A zero base with a positive power gives the
// zero chain (Sec. 3.2, the -infinity case).
__device__ __forceinline__ void seed_value(double lnAh, double lnAl, SeedShape sh,
                                           double lch, double lcl, double lsh, double lsl,
                                           double& d, int& E)
{
    if ((sh.p > 0 && __builtin_isinf(lch)) || (sh.q > 0 && __builtin_isinf(lsh))) {
        d = 0.0;
        E = 0;
        return;
    }
    double h = lnAh, lo = lnAl;
    if (sh.p > 0) dd_add_times(h, lo, (double)sh.p, lch, lcl);
    if (sh.q > 0) dd_add_times(h, lo, (double)sh.q, lsh, lsl);
    double yh, yl;
    dd_mul(h, lo, 0x1.71547652b82fep+0, 0x1.777d0ffda0d24p-56, yh, yl);   // ln -> log2
    const double k = floor(yh);
    const double f = (yh - k) + yl;
    const double m = exp2(f);
    const int ik = (int)k;
    E = ik >= FOLD_EXP ? 0 : ik / -FOLD_EXP * -FOLD_EXP;   // a multiple of 900, ik - E in (-900, 0]
    d = ldexp(m, ik - E);
    if (sh.neg) d = -d;
}

// ------------------------------------------------------------ normalised walk
// The walks carry e^l = c_l d^l with c_{l0} = c_{l0+1} = 1 and c_{l+1} = c_{l-1} / F2_l.
// The step then reads e^{l+1} = alpha_l F0 (x - F1) e^l - e^{l-1} with alpha_l = c_{l+1} / c_l:
// two FP64 instructions, u = fma(x, A', nB') and e' = fma(u, e, -e_prev) with A' = alpha F0 and
// nB' = -alpha F0 F1, where the plain step takes three.  A value d^l is e^l / c_l: the forward
// folds 1/c_l into its weights, the adjoint into its per-l sums, the Wigner walk into its stores.
// Each factor (l+1)^2 - a^2 of F2's denominator exceeds l^2 - a^2 by at least 2l + 1, so
// F2_l <= (l+1)/l (l/(l+1))^2 = l/(l+1) < 1: c_l >= 1 grows along each parity of l, |d| <= |e|,
// and every skip test taken on e is conservative.  alpha is largest at its start,
// q(l0+2)/q(l0+1) <= 2 with q(l)^2 = (l^2 - mb^2)(l^2 - msky^2) / l^2 (the bound the growth
// constant above assumes; the host tests check it over the extreme columns up to l = 16384).
struct NormCoef {
    double A, nB;   // alpha_l F0_l, -alpha_l F0_l F1_l (0 from l = lmax on: the step is off)
    double ic;      // 1 / c_l
};

// Coefficients of one block of NT values of l, staged by the whole workgroup: lane tid takes l =
// lb + tid, so every wave stages 64 of them.  (With one wave staging a block of 64 while the others
// wait at the barrier, the staging wave's SIMD is late in every block.)  c_l is a product over
// segments of NORM_SEG values of l, each taking the last two c of the one before in order, so it
// rounds the same way for every NT.
//
// With S(l) = sqrt((l^2 - mb^2)(l^2 - msky^2)) the closed forms are F0_l = (l+1)(2l+1) / S(l+1) and
// F2_l = (l+1) S(l) / (l S(l+1)), so c_l / c_{l-2} = (l-1) S(l) / (l S(l-1)).  A lane takes the root at
// l + 1 and its reciprocal by a joint iteration and gets those at l from its neighbour; the
// quotients come from these reciprocals with one correction, to within rounding of the correctly
// rounded ones.  (Products with the reciprocals alone, uncorrected, were 0.5% faster at lmax 4096
// and doubled the error of C and of the gradients.)  About 150 VALU operations per wave and 64
// values of l, where four roots and four divisions at each of l and l - 1 took about 350.
constexpr int NORM_SEG = 32;

template <int NT>
struct NormShared {
    double edge[NT / 64 + 1][3];   // S(l+1), 1/S(l+1), c_{l+1} / c_{l-1} of a wave's last l; [0]: of the block before
    double tot[NT / NORM_SEG][2];  // product of c_l / c_{l-2} over a segment, per parity
    double carry[2];               // c of the last two l of the block before
};

// Bits by which one step with coefficients A', nB' may grow max(|e^l|, |e^{l-1}|) (|x| <= 1).
__device__ __forceinline__ int grow_bits(double A, double nB)
{
    return (__double2hiint(fabs(A) + fabs(nB) + 1.0) >> 20) - 1022;
}

// 1 / a for normal a: the hardware's estimate (relative error 2^-24) and two Newton steps.
__device__ __forceinline__ double rcp_newton(double a)
{
    double y = __builtin_amdgcn_rcp(a);
    y = fma(y, fma(-a, y, 1.0), y);
    return fma(y, fma(-a, y, 1.0), y);
}

// sqrt(p) and 1 / sqrt(p) for normal p > 0: the hardware's estimate of the reciprocal root, two
// joint Newton (Goldschmidt) steps, one correction of each.
__device__ __forceinline__ void sqrt_and_rsqrt(double p, double& root, double& recip)
{
    const double y = __builtin_amdgcn_rsq(p);
    double g = p * y, h = 0.5 * y;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double r = fma(-h, g, 0.5);
        g = fma(g, r, g);
        h = fma(h, r, h);
    }
    g = fma(fma(-g, g, p), h, g);
    h = fma(h, fma(-h, g, 0.5), h);
    root = g;
    recip = 2.0 * h;
}

// a / b given y = 1 / b to a few ulp.
__device__ __forceinline__ double div_corrected(double a, double b, double y)
{
    const double q = a * y;
    return fma(fma(-b, q, a), y, q);
}

// The value of v in lane addr / 4.
__device__ __forceinline__ double lane_value(int addr, double v)
{
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(addr, __double2hiint(v)),
                            __builtin_amdgcn_ds_bpermute(addr, __double2loint(v)));
}

// The value N lanes below in the row of 16, 1 where there is none.
template <int N>
__device__ __forceinline__ double row_below_or_one(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x110 + N, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0x3ff00000, __double2hiint(v), 0x110 + N, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

struct NormLane {                  // what a lane keeps from one block to the next
    double S, rS, m, c;            // S(l + 1), its reciprocal, c_{l+1} / c_{l-1}, c_l
};

// grow[k] receives the largest grow_bits of the block's k-th RS_STEPS steps.
// Two barriers inside; the caller's barrier after it has stored the coefficients ends the stage.
// The first one also ends every wave's use of the block before.
template <int NT>
__device__ __forceinline__ NormCoef norm_coefs_group(int lb, int l0, int mb, int ms, int lmax, bool first,
                                                     NormLane& st, NormShared<NT>& sh, int* grow)
{
    static_assert(NT % 64 == 0 && NORM_SEG == 32, "whole waves, segments of two rows");
    static_assert(NORM_SEG == RS_STEPS, "one growth bound per segment");
    const int tid = threadIdx.x, i = tid & 63, wave = tid >> 6;
    const int l = lb + tid;
    if (tid >= NT - 2) sh.carry[tid - (NT - 2)] = first ? 1.0 : st.c;   // first block: c = 1
    if (tid == NT - 1) {           // not used by a first block
        sh.edge[0][0] = st.S; sh.edge[0][1] = st.rS; sh.edge[0][2] = st.m;
    }
    const double ll = (double)l, l1 = ll + 1.0;
    const double b2 = (double)mb * (double)mb, s2 = (double)ms * (double)ms, ll1 = l1 * l1;
    const double rl1 = rcp_newton(l1);
    double S, rS;
    sqrt_and_rsqrt((ll1 - b2) * (ll1 - s2), S, rS);
    const int below = ((i - 1) & 63) * 4;
    const double S0 = lane_value(below, S), rS0 = lane_value(below, rS);   // at l
    double rl = lane_value(below, rl1);
    double m_next = div_corrected(ll * S, l1 * S0, rl1 * rS0);   // c_{l+1} / c_{l-1}
    if (i == 63) { sh.edge[wave + 1][0] = S; sh.edge[wave + 1][1] = rS; sh.edge[wave + 1][2] = m_next; }
    __syncthreads();
    if (i == 0) {
        rl = rcp_newton(ll);
        m_next = div_corrected(ll * S, l1 * sh.edge[wave][0], rl1 * sh.edge[wave][1]);
    }
    double m = lane_value(below, m_next);                        // c_l / c_{l-2}
    if (i == 0) m = sh.edge[wave][2];
    double c = (l >= l0 + 2 && l <= lmax) ? m : 1.0;
    double A = 0.0, nB = 0.0;
    if (l < lmax) {
        A = div_corrected(l1 * (2.0 * ll + 1.0), S, rS);
        if (l > 0) nB = -(A * div_corrected((double)mb * (double)ms, ll * l1, rl * rl1));
    }
    // products over the lanes of one parity within the segment: within rows of 16, then across
    c *= row_below_or_one<2>(c);
    c *= row_below_or_one<4>(c);
    c *= row_below_or_one<8>(c);
    const int j = i & (NORM_SEG - 1);
    const double row_end = lane_value(((i & 32) + 14 + (i & 1)) * 4, c);   // the segment's first row
    if (j >= 16) c *= row_end;
    const int seg = tid / NORM_SEG;
    if (j >= NORM_SEG - 2) sh.tot[seg][tid & 1] = c;
    __syncthreads();
    double cr = sh.carry[tid & 1];
    for (int g = 0; g < 2 * wave; ++g) cr *= sh.tot[g][tid & 1];
    const double t0 = sh.tot[2 * wave][tid & 1];
    c *= (i < NORM_SEG) ? cr : cr * t0;
    const double c_below = lane_value(below, c);
    double c_next = lane_value(((i + 1) & 63) * 4, c);        // c_{l+1}
    if (i == 63) c_next = (l < lmax) ? m_next * c_below : c_below;   // as the next wave's first lane
    const double ic = rcp_newton(c), alpha = div_corrected(c_next, c, ic);
    st.S = S; st.rS = rS; st.m = m_next; st.c = c;
    int g = grow_bits(alpha * A, alpha * nB);
#pragma unroll
    for (int off = NORM_SEG / 2; off > 0; off /= 2) g = max(g, __shfl_xor(g, off, 64));
    if (j == 0) grow[seg] = g;
    return NormCoef{alpha * A, alpha * nB, ic};
}

// The skip test of a wave's plain chains (E = 0): whether any may reach 2^-skip_exp within the next
// RS_STEPS steps, each of which grows max(|d|, |d_prev|) by at most 2^bits.  Only high words are
// compared (the threshold is a power of two): three integer operations a chain, where the maxima
// of doubles take four and more with the operands' canonicalisation.  Testing every 8 steps with
// 17 bits a step cost as many instructions as the skipped steps themselves (forward, lmax 4096:
// 4.17 VALU operations per chain step, 3.6 of them multiply-adds).
template <int R>
__device__ __forceinline__ bool wave_may_be_hot(const double (&d)[R], const double (&dp)[R], const int (&E)[R],
                                                bool scaled, int skip_exp, int bits)
{
    unsigned m = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        unsigned h = max((unsigned)__double2hiint(d[r]) & 0x7fffffffu, (unsigned)__double2hiint(dp[r]) & 0x7fffffffu);
        if (scaled) h = E[r] == 0 ? h : 0u;
        m = max(m, h);
    }
    return wave_any(m >= (unsigned)(1023 - skip_exp - bits * RS_STEPS) << 20);
}

// Rescale of a scaled chain (every RS_STEPS steps of the convolution walks): once max(|d|, |d_prev|)
// has reached 1 both are multiplied by exactly 2^-900 and E rises by 900, to a plain double at 0.
// A chain still scaled afterwards is below 1, so below 2^-900 in truth, which is what RS_STEPS is
// derived from.  Returns the factor (1 or 2^-900) for sums held in the chain's units.  About ten VALU
// operations a chain where taking both exponents with frexp and renormalising took about 25.
__device__ __forceinline__ double rescale_chain(double& d, double& dp, int& E)
{
    const unsigned h = max((unsigned)__double2hiint(d) & 0x7fffffffu, (unsigned)__double2hiint(dp) & 0x7fffffffu);
    const bool up = (E < 0) & (h >= 0x3ff00000u);
    const double f = up ? 0x1p-900 : 1.0;
    E = up ? E - FOLD_EXP : E;
    d *= f;
    dp *= f;
    return f;
}

__device__ __forceinline__ size_t packed_index(int lmax, int l, int m)
{
    return (size_t)m * (size_t)(2 * lmax + 1 - m) / 2 + (size_t)l;
}

// ================================================================ wigner_d_rings
// One lane walks one ring of one (mb, msky) pair and stores d^l for every l: NT consecutive rings
// of a row leave as 512-byte pieces per wave.  A call has few chains (9 pairs on 2001 rings: 288
// waves on 1024 SIMDs) and up to lmax + 1 steps each, so it is bound by the latency of a step and,
// with many pairs, by the stores; one chain per lane spreads the walks over the most SIMDs, and NT
// lanes stage NT values of l at a time.  9 pairs on 2001 rings at lmax 1500: 63 us, 3.4 TB/s of stores
// (315 us with four chains per lane, coefficients staged by one wave per 32 values of l and a scale
// check every 8 steps); 100 pairs on 2048 rings at lmax 2048: 595 us, 5.6 TB/s (635 us).  NT 256 took
// 65 and 620 us, NT 64 64 and 600 us.
template <int NT>
struct WignerShared {
    double2 ab[NT];          // {A', nB'} of the block
    double ic[NT];           // 1 / c_l
    NormShared<NT> norm;
    int grow[NT / RS_STEPS];
};

template <int NT>
__global__ void __launch_bounds__(NT) k_wigner(const WignerArgs a)
{
    __shared__ WignerShared<NT> sh_;
    const int tid = threadIdx.x;
    const int pair = blockIdx.x / a.ntile;
    const int tile = blockIdx.x - pair * a.ntile;
    const int mb = a.col.mb[pair], ms = a.col.ms[pair];
    const int L = a.lmax;
    const int l0 = max(abs(mb), abs(ms));
    const int j = tile * NT + tid;
    const bool live = j < a.nring;
    double x = 0.0, d = 0.0, dp = 0.0;
    int E = 0;
    double* out = a.d + (size_t)pair * (size_t)(L + 1) * (size_t)a.nring + (live ? j : 0);
    const size_t row = (size_t)a.nring;
    if (live) {
        x = a.ring.x[j];
        seed_value(a.col.lnA[2 * pair], a.col.lnA[2 * pair + 1], seed_shape(mb, ms), a.ring.lch[j], a.ring.lcl[j],
                   a.ring.lsh[j], a.ring.lsl[j], d, E);
#pragma unroll 8
        for (int l = 0; l < l0; ++l) stg(out + (size_t)l * row, 0.0);
    }
    out += (size_t)l0 * row;
    bool scaled = wave_any(E < 0);
    NormLane st;
    auto stage = [&](int lb, bool first) {
        const NormCoef k = norm_coefs_group<NT>(lb, l0, mb, ms, L, first, st, sh_.norm, sh_.grow);
        sh_.ab[tid] = make_double2(k.A, k.nB);
        sh_.ic[tid] = k.ic;
        __syncthreads();
    };
    auto step = [&](const double2 k) {
        const double u = fma(x, k.x, k.y);
        const double dn = fma(u, d, -dp);
        dp = d;
        d = dn;
    };
    stage(l0, true);
    const int n = L - l0 + 1;
    for (int b0 = 0; b0 < n; b0 += NT) {
        const int send = min(NT, n - b0);
        for (int s1 = 0; s1 < send; s1 += RS_STEPS) {
            if (scaled) {
                (void)rescale_chain(d, dp, E);
                scaled = wave_any(E < 0);
            }
            const int s2 = min(s1 + RS_STEPS, send);
            int s = s1;
            // a group's coefficients are read together and its values stored together: a read and a
            // branch per step would wait for LDS at every step
            for (; s + TS <= s2; s += TS) {
                double2 k[TS];
                double v[TS];
#pragma unroll
                for (int t = 0; t < TS; ++t) { k[t] = sh_.ab[s + t]; v[t] = sh_.ic[s + t]; }
                if (scaled) {
#pragma unroll
                    for (int t = 0; t < TS; ++t) {
                        v[t] *= ldexp(d, E);
                        step(k[t]);
                    }
                } else {
#pragma unroll
                    for (int t = 0; t < TS; ++t) {
                        v[t] *= d;
                        step(k[t]);
                    }
                }
                if (live) {
#pragma unroll
                    for (int t = 0; t < TS; ++t) stg(out + (size_t)t * row, v[t]);
                }
                out += TS * row;
            }
            for (; s < s2; ++s) {
                if (live) stg(out, ldexp(d, E) * sh_.ic[s]);
                step(sh_.ab[s]);
                out += row;
            }
        }
        if (b0 + NT < n) stage(l0 + b0 + NT, false);
    }
}

// ================================================================== forward
// Weights of step l for the (sky, beam) pair p: w1 = conj(b^p_{l,mb}) s^p_{l,msky} for
// the direct ring and w2 = (-1)^(l-msky) conj(b^p_{l,-mb}) s^p_{l,msky} for the mirror
// ring.  Scalar convolution: one pair.  Polarised convolution (footnote of Sec. 4.1):
// the temperature, gradient and curl pairs share the recursion, each with its own
// weights (NC = NP outputs) or with their weights summed (one output, NC = 1).  Detectors
// that share lmax and rings share it the same way, one output each (batched plans).
// Pair p's beam and output rows run over mb = -pmbmax[p] .. pmbmax[p].
struct RawW {
    double br, bi, b2r, b2i, sr, si;
};

__device__ __forceinline__ RawW load_weights_raw(const FwdArgs& a, int p, int l, int mb, int ms)
{
    RawW w{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (l <= a.lmax) {
        const double2* blm = reinterpret_cast<const double2*>(a.blm[p]);
        const double2* alm = reinterpret_cast<const double2*>(a.alm[p]);
        const double2 b1 = ldg(blm + (size_t)(mb + a.pmbmax[p]) * (a.lmax + 1) + l);
        const double2 b2 = ldg(blm + (size_t)(-mb + a.pmbmax[p]) * (a.lmax + 1) + l);
        const double2 s = ldg(alm + packed_index(a.sky_lmax, l, ms));
        w = RawW{b1.x, b1.y, b2.x, b2.y, s.x, s.y};
    }
    return w;
}

__device__ __forceinline__ double4 pair_weights(const RawW& w, int l, int ms)
{
    // conj(b) * s
    const double w1r = w.br * w.sr + w.bi * w.si;
    const double w1i = w.br * w.si - w.bi * w.sr;
    const double sg = ((l - ms) & 1) ? -1.0 : 1.0;
    const double w2r = sg * (w.b2r * w.sr + w.b2i * w.si);
    const double w2i = sg * (w.b2r * w.si - w.b2i * w.sr);
    return make_double4(w1r, w1i, w2r, w2i);
}

// Output c's weights from the raw loads of the NP pairs: pair c itself, or (NC = 1)
// the sum over all pairs in pair order.
template <int NC, int NP>
__device__ __forceinline__ double4 output_weights(const RawW (&raw)[NP], int c, int l, int ms)
{
    if (NC == NP) return pair_weights(raw[c], l, ms);
    double4 w = pair_weights(raw[0], l, ms);
#pragma unroll
    for (int p = 1; p < NP; ++p) {
        const double4 v = pair_weights(raw[p], l, ms);
        w.x += v.x; w.y += v.y; w.z += v.z; w.w += v.w;
    }
    return w;
}

// LDS slots (16 bytes) of one l: {A, nB}, then per output {w1r, w1i} and, in the general form,
// {w2r, w2i}.
template <int NC, bool ROWS>
constexpr int coef_slots() { return ROWS ? 1 + NC : 1 + 2 * NC; }

// The weights take the factor 1/c_l of the normalised walk.
template <int NC, int NP>
__device__ __forceinline__ void stage_block(const NormCoef& k, const RawW (&raw)[NP], int l, int ms, double2* slot)
{
    slot[0] = make_double2(k.A, k.nB);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const double4 w = output_weights<NC, NP>(raw, c, l, ms);
        slot[1 + 2 * c] = make_double2(w.x * k.ic, w.y * k.ic);
        slot[2 + 2 * c] = make_double2(w.z * k.ic, w.w * k.ic);
    }
}

// The even / odd form needs w1 only: b^c_{l,mb} of each output and its sky.  The outputs of a batched
// walk share one sky (NSKY 1), polarised pairs have one each (NSKY NC).
template <int NC, int NSKY>
struct RawRows {
    double br[NC], bi[NC];
    double sr[NSKY], si[NSKY];
};

template <int NC, int NSKY, int P0>
__device__ __forceinline__ RawRows<NC, NSKY> load_rows_raw(const FwdArgs& a, int l, int mb, int ms)
{
    static_assert(NSKY == 1 || NSKY == NC, "one sky, or one per output");
    RawRows<NC, NSKY> w;
#pragma unroll
    for (int c = 0; c < NSKY; ++c) { w.sr[c] = 0.0; w.si[c] = 0.0; }
#pragma unroll
    for (int c = 0; c < NC; ++c) { w.br[c] = 0.0; w.bi[c] = 0.0; }
    if (l <= a.lmax) {
        const size_t k = packed_index(a.sky_lmax, l, ms);
#pragma unroll
        for (int c = 0; c < NSKY; ++c) {
            const double2 s = ldg(reinterpret_cast<const double2*>(a.alm[P0 + c]) + k);
            w.sr[c] = s.x; w.si[c] = s.y;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double2* blm = reinterpret_cast<const double2*>(a.blm[P0 + c]);
            const double2 b = ldg(blm + (size_t)(mb + a.pmbmax[P0 + c]) * (a.lmax + 1) + l);
            w.br[c] = b.x; w.bi[c] = b.y;
        }
    }
    return w;
}

template <int NC, int NSKY>
__device__ __forceinline__ void stage_block_rows(const NormCoef& k, const RawRows<NC, NSKY>& w, double2* slot)
{
    slot[0] = make_double2(k.A, k.nB);
#pragma unroll
    for (int c = 0; c < NC; ++c) {   // conj(b) * s, as in pair_weights, times 1/c_l
        const double sr = w.sr[NSKY == 1 ? 0 : c], si = w.si[NSKY == 1 ? 0 : c];
        slot[1 + c] = make_double2((w.br[c] * sr + w.bi[c] * si) * k.ic, (w.br[c] * si - w.bi[c] * sr) * k.ic);
    }
}

template <int R, int NC, bool ACC, int NS>
__device__ __forceinline__ void fwd_steps(const double2 (*cf)[NS], int s0,
                                          const double (&x)[R], double (&d)[R], double (&dp)[R],
                                          double (&c1r)[NC][R], double (&c1i)[NC][R],
                                          double (&c2r)[NC][R], double (&c2i)[NC][R])
{
#pragma unroll
    for (int t = 0; t < TS; ++t) {
        const double2 k = cf[s0 + t][0];
        double2 w1[NC], w2[NC];
        if constexpr (ACC) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                w1[c] = cf[s0 + t][1 + 2 * c];
                w2[c] = cf[s0 + t][2 + 2 * c];
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (ACC) {
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    c1r[c][r] = fma(w1[c].x, d[r], c1r[c][r]);
                    c1i[c][r] = fma(w1[c].y, d[r], c1i[c][r]);
                    c2r[c][r] = fma(w2[c].x, d[r], c2r[c][r]);
                    c2i[c][r] = fma(w2[c].y, d[r], c2i[c][r]);
                }
            }
            const double u = fma(x[r], k.x, k.y);
            const double dn = fma(u, d[r], -dp[r]);
            dp[r] = d[r];
            d[r] = dn;
        }
    }
}

// Beam rows mb and -mb related by a sign s (b_{l,-mb} = s b_{l,mb}, as for a beam with
// real coefficients): then w2 = s (-1)^(l-msky) w1, and the direct and mirror sums both
// follow from the sums of w1 d over the even and over the odd steps of the walk, so a
// step adds w1 d into one of two sums (2 instead of 4 fused multiply-adds per chain and
// output).  The step parity is that of t (blocks and groups have even lengths): P0 += at
// even t, P1 at odd t, in the c1 and c2 registers of the general form.
template <int R, int NC, int NS>
__device__ __forceinline__ void fwd_steps_rows(const double2 (*cf)[NS], int s0,
                                               const double (&x)[R], double (&d)[R], double (&dp)[R],
                                               double (&p0r)[NC][R], double (&p0i)[NC][R],
                                               double (&p1r)[NC][R], double (&p1i)[NC][R])
{
    // With one output, each step's coefficients and weights are read during the step before (more
    // outputs leave no registers for it: their walks read them at the step).
    constexpr bool AHEAD = NC == 1;
    double2 kn = cf[s0][0], vn[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) vn[c] = cf[s0][1 + c];
#pragma unroll
    for (int t = 0; t < TS; ++t) {
        if (!AHEAD && t > 0) {
            kn = cf[s0 + t][0];
#pragma unroll
            for (int c = 0; c < NC; ++c) vn[c] = cf[s0 + t][1 + c];
        }
        const double2 k = kn;
        double2 w[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) w[c] = vn[c];
        if (AHEAD && t + 1 < TS) {
            kn = cf[s0 + t + 1][0];
#pragma unroll
            for (int c = 0; c < NC; ++c) vn[c] = cf[s0 + t + 1][1 + c];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if ((t & 1) == 0) {
                    p0r[c][r] = fma(w[c].x, d[r], p0r[c][r]);
                    p0i[c][r] = fma(w[c].y, d[r], p0i[c][r]);
                } else {
                    p1r[c][r] = fma(w[c].x, d[r], p1r[c][r]);
                    p1i[c][r] = fma(w[c].y, d[r], p1i[c][r]);
                }
            }
            const double u = fma(x[r], k.x, k.y);
            const double dn = fma(u, d[r], -dp[r]);
            dp[r] = d[r];
            d[r] = dn;
        }
    }
}

// One block of NT values of l: the workgroup stages it together, walks it, and stages the next
// one over it (the stage's first barrier waits for the last reader).
template <int NT, int NS>
struct FwdShared {
    double2 cf[NT][NS];      // coefficient slots of the block
    NormShared<NT> norm;
    int grow[NT / RS_STEPS]; // growth bounds of the block's steps
};

// One (column, ring tile) work item of the forward over pairs P0 .. P0 + NP - 1 into outputs
// P0 .. P0 + NC - 1.  ROWS: the even / odd form, output c with beam row sign rows_sign[c], of NSKY skies.
template <int R, int NT, int NC, int NP, bool ROWS, int P0, int NS, int NSKY = 1>
__device__ __forceinline__ void fwd_column_walk(const FwdArgs& a, int ci, int tile, const int* rows_sign,
                                                FwdShared<NT, NS>& sh_)
{
    static_assert(NC == 1 || NC == NP, "one output per pair, or one summed output");
    static_assert(!ROWS || NC == NP, "the even / odd form: one output per pair");
    static_assert(NS >= coef_slots<NC, ROWS>() && P0 + NP <= kMaxPairs, "coefficient slots, pairs");
    static_assert(NT % RS_STEPS == 0 && RS_STEPS % TS == 0, "whole rescale periods per block");
    const int tid = threadIdx.x;
    const int mb = ldg(a.col.mb + ci), ms = ldg(a.col.ms + ci);
    const int L = a.lmax;
    const int l0 = max(abs(mb), ms);
    const SeedShape sh = seed_shape(mb, ms);
    const double lnAh = ldg(a.col.lnA + 2 * ci), lnAl = ldg(a.col.lnA + 2 * ci + 1);

    // the ring indices of the slots are read again for the stores (not held through the walk)
    const int s_base = tile * (NT * R) + tid * R;   // a wave: 64 R consecutive ring pairs
    double x[R], d[R], dp[R], c1r[NC][R], c1i[NC][R], c2r[NC][R], c2i[NC][R];
    int E[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int s = s_base + r;
        x[r] = 0.0; d[r] = 0.0; dp[r] = 0.0; E[r] = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            c1r[c][r] = 0.0; c1i[c][r] = 0.0; c2r[c][r] = 0.0; c2i[c][r] = 0.0;
        }
        if (s < a.nslot) {
            const int j = ldg(a.slots + 2 * s);
            x[r] = ldg(a.ring.x + j);
            seed_value(lnAh, lnAl, sh, ldg(a.ring.lch + j), ldg(a.ring.lcl + j), ldg(a.ring.lsh + j),
                       ldg(a.ring.lsl + j), d[r], E[r]);
        }
    }
    bool scaled = false;
#pragma unroll
    for (int r = 0; r < R; ++r) scaled |= (E[r] < 0);
    scaled = wave_any(scaled);
    bool acc_on = (a.skip_exp <= 0);

    RawW raw[NP];         // general form: the loads of the next block, in flight during a block
    RawRows<NC, NSKY> rraw;   // even / odd form
    auto load_raw = [&](int l) {
        if constexpr (ROWS) {
            rraw = load_rows_raw<NC, NSKY, P0>(a, l, mb, ms);
        } else {
#pragma unroll
            for (int p = 0; p < NP; ++p) raw[p] = load_weights_raw(a, P0 + p, l, mb, ms);
        }
    };
    NormLane st;
    auto stage_raw = [&](int lb, bool first) {
        const NormCoef k = norm_coefs_group<NT>(lb, l0, mb, ms, L, first, st, sh_.norm, sh_.grow);
        if constexpr (ROWS)
            stage_block_rows<NC, NSKY>(k, rraw, sh_.cf[tid]);
        else
            stage_block<NC, NP>(k, raw, lb + tid, ms, sh_.cf[tid]);
        __syncthreads();
    };
    load_raw(l0 + tid);
    stage_raw(l0, true);
    const int n = L - l0 + 1;              // l values of a chain
    // a wave beyond the last ring slot only stages
    const bool idle = tile * (NT * R) + __builtin_amdgcn_readfirstlane(tid >> 6) * (64 * R) >= a.nslot;
    for (int b0 = 0; b0 < n; b0 += NT) {
        const bool more = b0 + NT < n;
        if (more) load_raw(l0 + b0 + NT + tid);     // in flight during the block
        const int send = idle ? 0 : min(NT, n - b0);
        for (int s1 = 0; s1 < send; s1 += RS_STEPS) {
            if (scaled) {
                bool any = false;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const double f = rescale_chain(d[r], dp[r], E[r]);
                    if (acc_on) {   // sums in the chain's scaled units follow it
#pragma unroll
                        for (int c = 0; c < NC; ++c) { c1r[c][r] *= f; c1i[c][r] *= f; c2r[c][r] *= f; c2i[c][r] *= f; }
                    }
                    any |= (E[r] < 0);
                }
                scaled = wave_any(any);
            }
            if (!acc_on) acc_on = wave_may_be_hot<R>(d, dp, E, scaled, a.skip_exp, sh_.grow[s1 / RS_STEPS]);
            const int s2 = min(s1 + RS_STEPS, send);
            // kept rolled: unrolled, the 4-wave forward spills twice as many registers
#pragma unroll 1
            for (int s0 = s1; s0 < s2; s0 += TS) {
                if (!acc_on)
                    fwd_steps<R, NC, false>(sh_.cf, s0, x, d, dp, c1r, c1i, c2r, c2i);
                else if constexpr (ROWS)
                    fwd_steps_rows<R, NC>(sh_.cf, s0, x, d, dp, c1r, c1i, c2r, c2i);
                else
                    fwd_steps<R, NC, true>(sh_.cf, s0, x, d, dp, c1r, c1i, c2r, c2i);
            }
        }
        if (more) stage_raw(l0 + b0 + NT, false);
    }

    if constexpr (ROWS) {
        // direct sum P0 + P1; mirror sum s (-1)^(msky + l0) (P0 - P1)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double sg = ((ms + l0) & 1) ? -(double)rows_sign[c] : (double)rows_sign[c];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double er = c1r[c][r] + c2r[c][r], ei = c1i[c][r] + c2i[c][r];
                const double mr = sg * (c1r[c][r] - c2r[c][r]), mi = sg * (c1i[c][r] - c2i[c][r]);
                c1r[c][r] = er; c1i[c][r] = ei; c2r[c][r] = mr; c2i[c][r] = mi;
            }
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int M = a.pmbmax[P0 + c];
        const size_t row_d = ((size_t)(mb + M) * (L + 1) + ms) * (size_t)a.nring;
        const size_t row_m = ((size_t)(-mb + M) * (L + 1) + ms) * (size_t)a.nring;
        double2* C = reinterpret_cast<double2*>(a.C[P0 + c]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int s = s_base + r;
            if (s < a.nslot) {
                const int jd = ldg(a.slots + 2 * s), jm = ldg(a.slots + 2 * s + 1);
                stg(C + row_d + jd, make_double2(ldexp(c1r[c][r], E[r]), ldexp(c1i[c][r], E[r])));
                if (jm >= 0)
                    stg(C + row_m + jm, make_double2(ldexp(c2r[c][r], E[r]), ldexp(c2i[c][r], E[r])));
            }
        }
    }
}

// The sign by which the walks take beam rows mb and -mb as related, from the signs sym of the rows
// -mbmax .. mbmax (0: not related).  Row 0 equals itself, so its column could always take the shorter
// form; where no other rows are related it is left with the others: alone in the launch of the short
// form its lmax + 1 workgroups last as long as the longest chain (forward of a complex beam at lmax
// 260: 30 of 100 us).
__device__ __forceinline__ int related_sign(const int* sym, int mbmax, int mb)
{
    const int s = ldg(sym + mb + mbmax);
    if (mb != 0 || mbmax == 0) return s;
    int any = 0;
    for (int m = 1; m <= mbmax; ++m) any |= ldg(sym + m + mbmax);
    return any ? s : 0;
}

// The same for pair p of the forward.
__device__ __forceinline__ int row_sign(const FwdArgs& a, int p, int mb)
{
    return related_sign(a.beam_sym[p], a.pmbmax[p], mb);
}

// The signs of the NC polarised pairs for row mb, from the words that k_prep packs (pair p's
// sign + 1 in byte p); whether the column takes the even / odd form: all rows related, and not row 0
// alone (as related_sign).
template <int NC>
__device__ __forceinline__ bool pol_row_signs(const FwdArgs& a, int mb, int (&s)[NC])
{
    const int* sym = a.beam_sym[0] + a.pmbmax[0];
    auto all = [&](int m) {
        const int w = ldg(sym + m);
        bool r = true;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            s[c] = ((w >> (8 * c)) & 255) - 1;
            r = r && s[c] != 0;
        }
        return r;
    };
    if (mb == 0 && a.pmbmax[0] > 0) {
        bool any = false;
        for (int m = 1; m <= a.pmbmax[0]; ++m) any = any || all(m);
        if (!any) return false;
    }
    return all(mb);
}

// The scalar forward with 256 lanes runs as two launches over every (column, tile): k_fwd_rows takes
// the columns whose beam rows are equal up to a sign, k_fwd the others; a workgroup whose column belongs
// to the other launch returns at once.  Polarised pairs with separate outputs are split the same way
// between k_fwd_pol_rows and k_fwd; summed pairs take k_fwd alone.
template <int R, int NT, int NC, int NP>
__global__ void __launch_bounds__(NT, (fwd_min_waves<R, NC, NP>())) k_fwd(const FwdArgs a)
{
    __shared__ FwdShared<NT, coef_slots<NC, false>()> sh;
    const int ci = blockIdx.x / a.ntile;
    if constexpr (NC == 1 && NP == 1) {
        if (row_sign(a, 0, ldg(a.col.mb + ci)) != 0) return;
    }
    int s[NC] = {};
    if constexpr (NC > 1) {   // k_fwd_pol_rows's columns
        if (a.beam_sym[0] && pol_row_signs<NC>(a, ldg(a.col.mb + ci), s)) return;
    }
    fwd_column_walk<R, NT, NC, NP, false, 0>(a, ci, blockIdx.x - ci * a.ntile, s, sh);
}

// Polarised pairs with an output each, on the columns where every pair's beam rows mb and -mb are related
// by a sign (a detector on its axes: temperature and gradient rows real and even in mb, curl rows
// imaginary and odd): one recursion and one even / odd sum per pair, 2 + 2 NC multiply-adds per chain
// step instead of 2 + 4 NC.  Three pairs at lmax 1024, mbmax 9, 2048 rings: 4.55 -> 3.00 ms, at lmax 1500 13.96 -> 9.13 ms.
template <int R, int NT, int NC>
__global__ void __launch_bounds__(NT, 2) k_fwd_pol_rows(const FwdArgs a)
{
    __shared__ FwdShared<NT, coef_slots<NC, true>()> sh;
    const int ci = blockIdx.x / a.ntile;
    int s[NC];
    if (!pol_row_signs<NC>(a, ldg(a.col.mb + ci), s)) return;
    fwd_column_walk<R, NT, NC, NC, true, 0, coef_slots<NC, true>(), NC>(a, ci, blockIdx.x - ci * a.ntile, s, sh);
}

template <int R, int NT>
__global__ void __launch_bounds__(NT, (rows_min_waves<R>())) k_fwd_rows(const FwdArgs a)
{
    __shared__ FwdShared<NT, coef_slots<1, true>()> sh;
    const int ci = blockIdx.x / a.ntile;
    const int s[1] = {row_sign(a, 0, ldg(a.col.mb + ci))};
    if (s[0] == 0) return;
    fwd_column_walk<R, NT, 1, 1, true, 0>(a, ci, blockIdx.x - ci * a.ntile, s, sh);
}

// Both forms in one launch, for the workgroups of small ring sets (NT < 256), whose calls last not much
// longer than a launch (lmax 64: 48 -> 43 us a call, lmax 500: 248 -> 243 us).  At NT 256, R 8 the two
// forms in one kernel cost the even / odd one 2%, so there each has its launch.
template <int R, int NT>
__global__ void __launch_bounds__(NT, (rows_min_waves<R>() < fwd_min_waves<R, 1, 1>() ? rows_min_waves<R>() : fwd_min_waves<R, 1, 1>()))
k_fwd_either(const FwdArgs a)
{
    __shared__ FwdShared<NT, coef_slots<1, false>()> sh;
    const int ci = blockIdx.x / a.ntile, tile = blockIdx.x - ci * a.ntile;
    const int s[1] = {row_sign(a, 0, ldg(a.col.mb + ci))};
    if (s[0] != 0)
        fwd_column_walk<R, NT, 1, 1, true, 0>(a, ci, tile, s, sh);
    else
        fwd_column_walk<R, NT, 1, 1, false, 0>(a, ci, tile, s, sh);
}

// Batched form: one workgroup per (walk, column, ring tile) item, the items in order of cost,
// longest first (workgroups start in index order).  A walk serves the npair <= walk_pairs<R>()
// detectors that share its lmax and rings, ordered by mbmax, largest first: the first k of them
// have the column's beam row mb.  When all k have that row pair equal up to a sign, one even /
// odd walk feeds the k outputs; otherwise each detector takes a walk of its own, in the form a
// plain call would take, so every output is the one a plain call with this tile writes.
//
// Detectors per walk: the even / odd sums take 8 VGPRs per chain and output, so R = 8 chains
// per lane hold two outputs within the 2-wave budget and R <= 4 hold four.
template <int R>
constexpr int walk_pairs() { return R >= 8 ? 2 : 4; }

template <int R>
constexpr int items_min_waves() { return R >= 4 ? 2 : 3; }

template <int R, int NT, int NS, int P>
__device__ __forceinline__ void fwd_item_alone(const FwdArgs& a, int ci, int tile, int k, const int (&s)[kMaxPairs],
                                               FwdShared<NT, NS>& cf)
{
    if (P < k) {
        if (s[P] != 0)
            fwd_column_walk<R, NT, 1, 1, true, P>(a, ci, tile, s + P, cf);
        else
            fwd_column_walk<R, NT, 1, 1, false, P>(a, ci, tile, s + P, cf);
    }
}

template <int R, int NT>
__global__ void __launch_bounds__(NT, (items_min_waves<R>())) k_fwd_items(const FwdArgs* __restrict__ walks,
                                                                          const int* __restrict__ items)
{
    constexpr int K = walk_pairs<R>();
    static_assert(K == 2 || K == 4, "walk sizes");
    constexpr int NS = coef_slots<K, true>() > coef_slots<1, false>() ? coef_slots<K, true>() : coef_slots<1, false>();
    __shared__ FwdShared<NT, NS> cf;
    const int* item = items + 3 * (size_t)blockIdx.x;
    const FwdArgs a = walks[item[0]];
    const int ci = item[1], tile = item[2];
    const int mb = ldg(a.col.mb + ci);
    int k = 0, s[kMaxPairs];
    bool rows = true;
#pragma unroll
    for (int p = 0; p < kMaxPairs; ++p) {
        s[p] = 0;
        if (p < K && p < a.npair && a.pmbmax[p] >= abs(mb)) {
            k = p + 1;
            s[p] = row_sign(a, p, mb);
            rows = rows && s[p] != 0;
        }
    }
    if (rows) {
        if (k == 1) { fwd_column_walk<R, NT, 1, 1, true, 0>(a, ci, tile, s, cf); return; }
        if (k == 2) { fwd_column_walk<R, NT, 2, 2, true, 0>(a, ci, tile, s, cf); return; }
        if constexpr (K == 4) {
            if (k == 3) { fwd_column_walk<R, NT, 3, 3, true, 0>(a, ci, tile, s, cf); return; }
            fwd_column_walk<R, NT, 4, 4, true, 0>(a, ci, tile, s, cf);
            return;
        }
    }
    fwd_item_alone<R, NT, NS, 0>(a, ci, tile, k, s, cf);
    fwd_item_alone<R, NT, NS, 1>(a, ci, tile, k, s, cf);
    if constexpr (K == 4) {
        fwd_item_alone<R, NT, NS, 2>(a, ci, tile, k, s, cf);
        fwd_item_alone<R, NT, NS, 3>(a, ci, tile, k, s, cf);
    }
}

// ================================================================== adjoint
// Per column and l: u_l = sum_j d^l(beta_j) Cbar_j over the direct rings (U)
// and sum_j d^l(beta_j) Cbar_{-mb,msky}(pi - beta_j) over the mirror rings (V).
//
// Systolic row sums.  The 16 lanes of a row walk skewed: lane k (k = lane mod 16) is k
// steps behind lane 0 of its row, so at the row's time t it is at l = l0 + t - k.  Each
// lane carries four running sums (U re/im, V re/im).  Every step the sums move one lane
// up the row (DPP row_shr:1; lane 0 of the row starts a fresh sum at 0) and the lane adds
// d * Cbar of its R chains for its own l: a sum visits the 16 lanes of the row at the
// same l and leaves lane 15 complete, 15 steps after it began, where it is written to
// LDS.  After the TB block's barrier the four rows' and the waves' sums of each l are
// added in a fixed order and written out.  No LDS round trip sits in the step loop and
// nothing is reduced across lanes but the one shift per sum and step; the order of
// every sum is fixed, so the result is deterministic.

constexpr int ROW = 16;             // lanes per systolic row
constexpr int SKEW = ROW - 1;       // steps lane 15 trails lane 0 of its row

// The value of the lane one below in the same row of 16; lane 0 of a row gets 0.
__device__ __forceinline__ double row_shift_up(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x111, 0xF, 0xF, true);   // row_shr:1
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x111, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// The sky gradient alone (SKY).  Column mb adds b_{l,mb} U_l + (-1)^(l-msky) b_{l,-mb} V_l to sky_bar_l;
// where the beam's rows are related by a sign, b_{l,-mb} = s b_{l,mb}, that is b_{l,mb} times the one sum
// sum_j d^l (Cbar_j + s (-1)^(l-msky) Cbar_{-mb,msky}(pi - beta_j)).  A lane holds the two
// combinations of its chains' cotangents, one for its even and one for its odd row times, and a step
// takes 2 + 2 instead of 2 + 4 multiply-adds per chain and shifts one complex sum instead of two.
// Sky gradient of 1001 slots at lmax 1023: 2.20 -> 1.66 ms, of 2048 at lmax 2048 22.7 -> 17.6 ms.

// Emitted row sums: slot (t - 16) mod 2 TB for the sum that leaves lane 15 at time t
// (l offset t - 15), then (wave, row, component); slots are out_stride doubles apart: two more
// than the NW 4 NS they hold, an even count, so that every slot is 16-byte aligned and a step
// group's emissions are 128-bit stores at constant offsets from one address (the reads of the
// block sum, one slot per lane, then meet at most two to a bank).  NS components: 4 per cotangent of
// the walk, 2 for the sky gradient alone.
template <int NT, int NS>
constexpr int out_stride() { return (NT / 64) * 4 * NS + 2; }

// The coefficient ring holds the last two staged blocks of NT l offsets plus a copy of its first
// TS slots behind its end, so that the TS consecutive offsets of a step group never wrap.
// NSMAX: the most components a walk in this workgroup sums.
template <int NT, int TB, int NSMAX>
struct AdjShared {
    double2 cfa[2 * NT + TS];                     // {A', nB'} per l offset, slot = offset mod 2 NT
    double cic[2 * NT];                           // 1 / c_l per l offset
    double out[2 * TB * out_stride<NT, NSMAX>()]; // emitted row sums
    NormShared<NT> norm;
    int grow[2 * NT / RS_STEPS];                  // growth bounds, slot = offset / RS_STEPS mod 2 NT / RS_STEPS
};

template <int NT, int TB, int NSMAX>
constexpr size_t adj_lds_bytes() { return sizeof(AdjShared<NT, TB, NSMAX>); }

// One ring tile of column ci for the cotangents 0 .. NC - 1 of the walk (a.Cbar[c], sums into
// a.U[c], a.V[c], rows of cotangent c offset by a.pmbmax[c]).  SKY: the sky gradient alone of one
// cotangent on a column whose beam rows are related by the sign sky_sign, its one sum into a.U[0].
template <int R, int NT, int TB, int NC, bool SKY, int NSMAX>
__device__ __forceinline__ void adj_column(const AdjArgs& a, int ci, int tile, int sky_sign,
                                           AdjShared<NT, TB, NSMAX>& sh_)
{
    static_assert(TB % RS_STEPS == 0 && NT % TB == 0 && TS % 2 == 0 && TB >= ROW, "step groups: pairs of steps, TS per check");
    static_assert(NC <= kMaxPairs && (!SKY || NC == 1), "cotangents per walk");
    constexpr int NW = NT / 64;
    constexpr int NS = SKY ? 2 : 4 * NC;    // running sums per lane: (U re, U im, V re, V im) per cotangent
    static_assert(NS <= NSMAX, "emitted components");
    constexpr int CF_N = 2 * NT;            // coefficient ring: the staged block of NT offsets and the one before
    constexpr int CF_MASK = CF_N - 1;
    constexpr int OUT_MASK = 2 * TB - 1;    // emitted sums: windows kb (written) and kb-1 (summed)
    constexpr int OS = out_stride<NT, NS>();
    static_assert((CF_N & CF_MASK) == 0 && (2 * TB & OUT_MASK) == 0 && (SKEW + 1) % TS == 0, "ring sizes");
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int kr = lane & (ROW - 1), row = lane >> 4;
    const int mb = ldg(a.col.mb + ci), ms = ldg(a.col.ms + ci);
    const int L = a.lmax;
    const int l0 = max(abs(mb), ms);
    const int n = L - l0 + 1;              // l values of a chain
    const SeedShape sh = seed_shape(mb, ms);
    const double lnAh = ldg(a.col.lnA + 2 * ci), lnAl = ldg(a.col.lnA + 2 * ci + 1);
    const int s_base = tile * (NT * R) + tid * R;   // a wave: 64 R consecutive ring slots

    double x[R], d[R], dp[R], g1r[NC][R], g1i[NC][R], g2r[NC][R], g2i[NC][R];
    int E[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int s = s_base + r;
        x[r] = 0.0; d[r] = 0.0; dp[r] = 0.0; E[r] = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c) { g1r[c][r] = 0.0; g1i[c][r] = 0.0; g2r[c][r] = 0.0; g2i[c][r] = 0.0; }
        if (s < a.nslot) {
            const int j = ldg(a.slots + 2 * s);
            x[r] = ldg(a.ring.x + j);
            seed_value(lnAh, lnAl, sh, ldg(a.ring.lch + j), ldg(a.ring.lcl + j), ldg(a.ring.lsh + j),
                       ldg(a.ring.lsl + j), d[r], E[r]);
        }
    }
    // A scaled chain (E < 0, |d| < 2^-900) contributes nothing; its cotangents are
    // loaded when it folds into plain doubles.
    auto load_g = [&](int r) {
        const int s = s_base + r;
        if (s < a.nslot && E[r] == 0) {
            const int jd = ldg(a.slots + 2 * s), jm = ldg(a.slots + 2 * s + 1);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const double2* Cbar = reinterpret_cast<const double2*>(a.Cbar[c]);
                const int M = a.pmbmax[c];
                const size_t row_d = ((size_t)(mb + M) * (L + 1) + ms) * (size_t)a.nring;
                const size_t row_m = ((size_t)(-mb + M) * (L + 1) + ms) * (size_t)a.nring;
                const double2 v1 = ldg(Cbar + row_d + jd);
                g1r[c][r] = v1.x; g1i[c][r] = v1.y;
                if (jm >= 0) {
                    const double2 v2 = ldg(Cbar + row_m + jm);
                    g2r[c][r] = v2.x; g2i[c][r] = v2.y;
                }
                if constexpr (SKY) {   // g1, g2: the combinations at even and at odd row times
                    const double sg = ((l0 - ms + kr) & 1) ? -(double)sky_sign : (double)sky_sign;
                    const double mr = sg * g2r[c][r], mi = sg * g2i[c][r];
                    g2r[c][r] = g1r[c][r] - mr; g2i[c][r] = g1i[c][r] - mi;
                    g1r[c][r] += mr; g1i[c][r] += mi;
                }
            }
        }
    };
#pragma unroll
    for (int r = 0; r < R; ++r) load_g(r);
    bool scaled = false;
#pragma unroll
    for (int r = 0; r < R; ++r) scaled |= (E[r] < 0);
    scaled = wave_any(scaled);
    bool acc_on = (a.skip_exp <= 0);    // wave-uniform

    // one U and one V row per column and cotangent: ring tile 0 writes them, each later tile
    // (walked after it by the same workgroup) adds to them
    const size_t urow = packed_index(L, 0, ms);   // + l

    NormLane st;
    auto stage = [&](int off, bool first) {   // offsets off .. off + NT - 1, off a multiple of NT
        const int slot = (off + tid) & CF_MASK;
        const NormCoef k = norm_coefs_group<NT>(l0 + off, l0, mb, ms, L, first, st, sh_.norm,
                                                sh_.grow + (off & CF_MASK) / RS_STEPS);
        sh_.cfa[slot] = make_double2(k.A, k.nB);
        sh_.cic[slot] = k.ic;
        if (slot < TS) sh_.cfa[CF_N + slot] = make_double2(k.A, k.nB);   // the copy behind the ring's end
    };
    // Lane 15 of each row stores the sums that leave it.  The sums alternate between two
    // register sets step by step, so that the two sums a pair of steps completes are both
    // still held after it and one store (a branch: only these lanes take it) serves two steps.
    const bool exit_lane = kr == SKEW;
    double* const outw = sh_.out + (wave * 4 + row) * NS;
    double sa[NS], sb[NS];   // set a: the sums after an odd step; set b: after an even step
#pragma unroll
    for (int q = 0; q < NS; ++q) { sa[q] = 0.0; sb[q] = 0.0; }
    auto emit2 = [&](int t) {   // step t completed set b, step t + 1 set a; slots t - 16, t - 15
        if (exit_lane) {
            double* o = outw + ((t - SKEW - 1) & OUT_MASK) * OS;
#pragma unroll
            for (int q = 0; q < NS; ++q) o[q] = sb[q];
            o = outw + ((t - SKEW) & OUT_MASK) * OS;
#pragma unroll
            for (int q = 0; q < NS; ++q) o[q] = sa[q];
        }
    };
    // The same for step t0 + h of a step group that starts at t0, a multiple of TS: the group's
    // slots t0 - 16 .. t0 - 16 + TS - 1 do not wrap the ring (t0 - 16 is a multiple of TS too), so
    // they are og (the group's first slot, one address per group) plus constant offsets.
    static_assert((SKEW + 1) % TS == 0 && (2 * TB) % TS == 0, "a step group's slots do not wrap");
    auto emit2_in = [&](double* og, int h) {
        if (exit_lane) {
            double* o = og + h * OS;
#pragma unroll
            for (int q = 0; q < NS; ++q) o[q] = sb[q];
            o = og + (h + 1) * OS;
#pragma unroll
            for (int q = 0; q < NS; ++q) o[q] = sa[q];
        }
    };
    auto shift_a_to_b = [&]() {
#pragma unroll
        for (int q = 0; q < NS; ++q) sb[q] = row_shift_up(sa[q]);
    };
    auto shift_b_to_a = [&]() {
#pragma unroll
        for (int q = 0; q < NS; ++q) sa[q] = row_shift_up(sb[q]);
    };
    // the sums s take e * Cbar of chain r; odd: an odd row time (SKY)
    auto add = [&](double dd, int r, double (&s)[NS], bool odd) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if constexpr (SKY) {
                s[0] = fma(dd, odd ? g2r[c][r] : g1r[c][r], s[0]);
                s[1] = fma(dd, odd ? g2i[c][r] : g1i[c][r], s[1]);
            } else {
                s[4 * c + 0] = fma(dd, g1r[c][r], s[4 * c + 0]);
                s[4 * c + 1] = fma(dd, g1i[c][r], s[4 * c + 1]);
                s[4 * c + 2] = fma(dd, g2r[c][r], s[4 * c + 2]);
                s[4 * c + 3] = fma(dd, g2i[c][r], s[4 * c + 3]);
            }
        }
    };
    // one step of the R chains of this lane: coefficients k
    auto step = [&](const double2 k, double (&s)[NS], bool odd) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            add(d[r], r, s, odd);
            const double u = fma(x[r], k.x, k.y);
            const double dn = fma(u, d[r], -dp[r]);
            dp[r] = d[r];
            d[r] = dn;
        }
    };

    stage(0, true);
    __syncthreads();
    // lane 15 of a row finishes l = L at time n - 1 + SKEW; the last block runs whole step groups
    const int T = n + SKEW;
    // waves beyond the last ring slot only stage and sum
    const int nact = min(NW, (a.nslot - tile * (NT * R) + 64 * R - 1) / (64 * R));
    const bool idle = __builtin_amdgcn_readfirstlane(wave) >= nact;
    for (int buf_t = 0; buf_t < T; buf_t += TB) {
        const int send = idle ? 0 : min(TB, T - buf_t);
        for (int s1 = 0; s1 < send; s1 += RS_STEPS) {
            if (scaled) {
                bool any = false;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const bool was = E[r] < 0;
                    (void)rescale_chain(d[r], dp[r], E[r]);
                    if (was && E[r] == 0) load_g(r);
                    any |= (E[r] < 0);
                }
                scaled = wave_any(any);
            }
            // a lane that has not started yet holds its seed, so the test covers it; lanes trail
            // by up to 15 steps, so the bound of the offsets before counts as well
            if (!acc_on) {
                constexpr int GROW_N = CF_N / RS_STEPS;
                const int gs = (buf_t + s1) / RS_STEPS;
                int bits = sh_.grow[gs % GROW_N];
                if (gs > 0) bits = max(bits, sh_.grow[(gs - 1) % GROW_N]);
                acc_on = wave_may_be_hot<R>(d, dp, E, scaled, a.skip_exp, bits);
            }
            const int s2 = min(s1 + RS_STEPS, send);
            for (int s0 = s1; s0 < s2; s0 += TS) {
                const int t0 = buf_t + s0;   // row time of the group's first step
                if (t0 < SKEW) {
                    // start of the walk: lane k holds its chain (seed, 0) until time k and adds nothing
#pragma unroll
                    for (int t = 0; t < TS; ++t) {
                        const int tt = t0 + t;
                        const bool live = tt >= kr;
                        const int off = live ? tt - kr : 0;
                        const double2 k = sh_.cfa[off & CF_MASK];
                        if (t & 1) shift_b_to_a(); else shift_a_to_b();
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const double dd = (live && acc_on) ? d[r] : 0.0;
                            if (t & 1) add(dd, r, sa, true);
                            else add(dd, r, sb, false);
                            const double u = fma(x[r], k.x, k.y);
                            const double dn = fma(u, d[r], -dp[r]);
                            dp[r] = live ? d[r] : dp[r];
                            d[r] = live ? dn : d[r];
                        }
                        if (t & 1) emit2(tt - 1);
                    }
                } else if (acc_on) {
                    // pairs of steps; each pair's coefficients are read during the pair before
                    const int cb = (t0 - kr) & CF_MASK;
                    double* const og = outw + ((t0 - SKEW - 1) & OUT_MASK) * OS;
                    double2 kn0 = sh_.cfa[cb], kn1 = sh_.cfa[cb + 1];
#pragma unroll
                    for (int h = 0; h < TS; h += 2) {
                        const double2 k0 = kn0, k1 = kn1;
                        if (h + 2 < TS) {
                            kn0 = sh_.cfa[cb + h + 2]; kn1 = sh_.cfa[cb + h + 3];
                        }
                        shift_a_to_b();
                        step(k0, sb, false);
                        shift_b_to_a();
                        step(k1, sa, true);
                        emit2_in(og, h);
                    }
                } else {
                    const int cb = (t0 - kr) & CF_MASK;
#pragma unroll
                    for (int t = 0; t < TS; ++t) {
                        const double2 k = sh_.cfa[cb + t];
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const double u = fma(x[r], k.x, k.y);
                            const double dn = fma(u, d[r], -dp[r]);
                            dp[r] = d[r];
                            d[r] = dn;
                        }
                    }
                    // nothing is added yet: every sum of these steps is zero
#pragma unroll
                    for (int q = 0; q < NS; ++q) { sa[q] = 0.0; sb[q] = 0.0; }
                    double* const og = outw + ((t0 - SKEW - 1) & OUT_MASK) * OS;
#pragma unroll
                    for (int t = 0; t < TS; t += 2) emit2_in(og, t);
                }
            }
        }
        const int next = buf_t + TB;
        if ((next & (NT - 1)) == 0 && next < T) stage(next, false);
        __syncthreads();
        // the sums of l offsets buf_t - 15 .. buf_t + TB - 16, all emitted in this block; the waves
        // and rows in a fixed order (the next block writes the other window)
        for (int q = tid; q < TB * NS; q += NT) {
            const int o = buf_t - SKEW + q / NS, comp = q % NS;
            if (o >= 0 && o < n) {
                const double* src = sh_.out + ((o - 1) & OUT_MASK) * OS + comp;
                double v = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    if (w < nact) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) v += src[NS * (4 * w + k)];
                    }
                }
                v *= sh_.cic[o & CF_MASK];   // e^l back to d^l
                const int c = SKY ? 0 : comp >> 2, part = comp & 3;
                // the cotangent's rows by selection: a runtime index into the argument
                // record would move the record to scratch memory
                double* uv = part < 2 ? a.U[0] : a.V[0];
                int M = a.pmbmax[0];
#pragma unroll
                for (int cc = 1; cc < NC; ++cc)
                    if (c == cc) { uv = part < 2 ? a.U[cc] : a.V[cc]; M = a.pmbmax[cc]; }
                double* dst = uv + 2 * ((size_t)(mb + M) * (size_t)a.P + urow + l0 + o) + (part & 1);
                stg(dst, (tile == 0) ? v : ldg(dst) + v);
            }
        }
    }
}

// All ring tiles of column ci, one after the other in one workgroup: tile 0 writes the
// column's U and V rows, each later tile adds to them (the same thread writes an element in
// every tile), so no launch has to wait for another.  The column's values the compiler keeps
// across tiles spill outside the step loops only.
template <int R, int NT, int TB, int NC, bool SKY, int NSMAX>
__device__ __forceinline__ void adj_tiles(const AdjArgs& a, int ci, int sky_sign, AdjShared<NT, TB, NSMAX>& sh)
{
    for (int tile = 0; tile < a.ntile; ++tile) {
        if (tile > 0) __syncthreads();   // the tile before still reads the LDS ring in its last block sums
        adj_column<R, NT, TB, NC, SKY, NSMAX>(a, ci, tile, sky_sign, sh);
    }
}

template <int R, int NT, int TB>
__global__ void __launch_bounds__(NT, (adj_min_waves<R, TB>())) k_adj(const AdjArgs a)
{
    static_assert(adj_lds_bytes<NT, TB, 4>() * adj_min_waves<R, TB>() * 256 / NT <= 160 * 1024, "LDS per CU");
    __shared__ AdjShared<NT, TB, 4> sh;
    if (a.beam_sym && related_sign(a.beam_sym, a.pmbmax[0], ldg(a.col.mb + blockIdx.x)) != 0) return;   // k_adj_one_sum's
    adj_tiles<R, NT, TB, 1, false, 4>(a, blockIdx.x, 0, sh);
}

// The columns whose beam rows are related by a sign, for the sky gradient alone.
template <int R, int NT, int TB>
__global__ void __launch_bounds__(NT, (adj_min_waves<R, TB>())) k_adj_one_sum(const AdjArgs a)
{
    __shared__ AdjShared<NT, TB, 2> sh;
    const int s = related_sign(a.beam_sym, a.pmbmax[0], ldg(a.col.mb + blockIdx.x));
    if (s != 0) adj_tiles<R, NT, TB, 1, true, 2>(a, blockIdx.x, s, sh);
}

// Both in one launch, for the workgroups of small ring sets (NT < 256).
template <int R, int NT, int TB>
__global__ void __launch_bounds__(NT, (adj_min_waves<R, TB>())) k_adj_either(const AdjArgs a)
{
    __shared__ AdjShared<NT, TB, 4> sh;
    const int s = related_sign(a.beam_sym, a.pmbmax[0], ldg(a.col.mb + blockIdx.x));
    if (s != 0) adj_tiles<R, NT, TB, 1, true, 4>(a, blockIdx.x, s, sh);
    else adj_tiles<R, NT, TB, 1, false, 4>(a, blockIdx.x, 0, sh);
}

// Batched form: one workgroup per (walk, column) item, the items longest first.  A walk serves
// the npair <= adj_walk_pairs<TB>() detectors that share its lmax and rings, ordered by mbmax,
// largest first: the first k of them have the column's beam row mb, and one walk adds into
// the sums of all k (2 + 4 k instructions and 4 k / R row shifts per chain step, where k walks
// of their own take 6 k and 4 k / R).  Two cotangents double the emitted-sum buffer, which
// with TB 64 would leave one workgroup per CU, and hold 8 cotangent doubles per chain, which
// at R 8 exceed the 256 registers of two waves per SIMD: paired walks are built with TB 32 and
// R <= 4 only (two workgroups per CU).
template <int R, int TB>
constexpr int adj_walk_pairs() { return (R <= 4 && TB <= 32) ? 2 : 1; }

// Paired walks hold two workgroups per CU (their LDS), which is the register budget they get.
template <int R, int TB>
constexpr int adj_items_min_waves() { return adj_walk_pairs<R, TB>() == 2 ? 2 : adj_min_waves<R, TB>(); }

template <int R, int NT, int TB>
__global__ void __launch_bounds__(NT, (adj_items_min_waves<R, TB>())) k_adj_items(const AdjArgs* __restrict__ dets,
                                                                            const int* __restrict__ items)
{
    constexpr int K = adj_walk_pairs<R, TB>();
    static_assert(adj_lds_bytes<NT, TB, 4 * K>() * (NT == 64 ? 7 : 512 / NT) <= 160 * 1024, "about two waves per SIMD");
    __shared__ AdjShared<NT, TB, 4 * K> sh;
    const int* item = items + 2 * (size_t)blockIdx.x;
    const int ci = item[1];
    if constexpr (K == 2) {
        // read in place: a copy of the record would sit in scratch memory in this form
        const AdjArgs& a = dets[item[0]];
        if (a.npair > 1 && a.pmbmax[1] >= abs(ldg(a.col.mb + ci)))
            adj_tiles<R, NT, TB, 2, false, 4 * K>(a, ci, 0, sh);
        else
            adj_tiles<R, NT, TB, 1, false, 4 * K>(a, ci, 0, sh);
    } else {
        const AdjArgs a = dets[item[0]];
        adj_tiles<R, NT, TB, 1, false, 4 * K>(a, ci, 0, sh);
    }
}

// Adds sum_mb b_{l,mb} u(mb, ms, l) of one detector to (ar, ai), mb ascending, where
// u(mb, ms, l) = U[mb] + (-1)^(l-ms) V[-mb], defined for l >= max(|mb|, ms).  The rows are
// read SKY_ROWS at a time before any is used, so that a thread keeps that many row loads in
// flight instead of one.
constexpr int SKY_ROWS = 8;
__device__ __forceinline__ void sky_grad_terms(const EpiArgs& e, int ms, int l, double& ar, double& ai)
{
    const size_t k = packed_index(e.lmax, l, ms);
    const double2* U = reinterpret_cast<const double2*>(e.U) + k;
    const double2* V = reinterpret_cast<const double2*>(e.V) + k;
    const double2* blm = reinterpret_cast<const double2*>(e.blm) + l;
    const int M = e.mbmax, lo = max(-M, -l), hi = min(M, l);   // rows with l >= |mb|
    const double sg = ((l - ms) & 1) ? -1.0 : 1.0;
    const int* one_sum = e.beam_sym;
    for (int mb0 = lo; mb0 <= hi; mb0 += SKY_ROWS) {
        double2 ua[SKY_ROWS], va[SKY_ROWS], ba[SKY_ROWS];
#pragma unroll
        for (int q = 0; q < SKY_ROWS; ++q) {
            const int mb = min(mb0 + q, hi);   // past the last row: a repeat of it, not added
            ua[q] = ldg(U + (size_t)(mb + M) * e.P);
            if (!one_sum || related_sign(one_sum, M, mb) == 0) va[q] = ldg(V + (size_t)(-mb + M) * e.P);
            else va[q] = make_double2(0.0, 0.0);
            ba[q] = ldg(blm + (size_t)(mb + M) * (e.lmax + 1));
        }
#pragma unroll
        for (int q = 0; q < SKY_ROWS; ++q) {
            if (mb0 + q <= hi) {
                const double2 u = make_double2(ua[q].x + sg * va[q].x, ua[q].y + sg * va[q].y);
                const double2 b = ba[q];
                ar += b.x * u.x - b.y * u.y;
                ai += b.x * u.y + b.y * u.x;
            }
        }
    }
}

// alm_bar_{l,ms} = sum_mb b_{l,mb} u(mb, ms, l)
__device__ __forceinline__ void sky_grad(const EpiArgs& e, int ms, int l)
{
    if (l > e.sky_lmax) return;
    double ar = 0.0, ai = 0.0;
    if (l <= e.lmax) sky_grad_terms(e, ms, l, ar, ai);
    stg(reinterpret_cast<double2*>(e.alm_bar) + packed_index(e.sky_lmax, l, ms), make_double2(ar, ai));
}

__global__ void __launch_bounds__(256) k_adj_sky(const EpiArgs e)
{
    sky_grad(e, blockIdx.y, (int)(blockIdx.y + blockIdx.x * blockDim.x + threadIdx.x));
}

// Batched form: the sky gradient of ndet detectors, summed in their order; with accumulate the
// sum is added to what alm_bar holds (the detectors of earlier launches), else it replaces it.
__global__ void __launch_bounds__(256) k_adj_sky_multi(const EpiArgs* __restrict__ eps, int ndet, int sky_lmax,
                                                       int accumulate, double* __restrict__ alm_bar)
{
    const int ms = blockIdx.y;
    const int l = ms + blockIdx.x * blockDim.x + threadIdx.x;
    if (l > sky_lmax) return;
    double2* out = reinterpret_cast<double2*>(alm_bar) + packed_index(sky_lmax, l, ms);
    double ar = 0.0, ai = 0.0;
    if (accumulate) {
        const double2 o = ldg(out);
        ar = o.x;
        ai = o.y;
    }
    for (int dt = 0; dt < ndet; ++dt) {
        const EpiArgs& e = eps[dt];
        if (l <= e.lmax) sky_grad_terms(e, ms, l, ar, ai);
    }
    stg(out, make_double2(ar, ai));
}

// blm_bar_{l,mb} = sum_{ms <= l} s_{l,ms} conj(u(mb, ms, l)).  A workgroup takes one mb and 64 values of l;
// wave w sums ms = w, w + BEAM_W, ..., and the waves' sums are added in their order.  Bound by reading U and V
// once and the sky from the caches.  One thread per (l, mb), all ms in turn, left one wave per SIMD and a chain
// of 512 round trips to memory at lmax 2048 (mbmax 14: 0.76 ms, now 0.40, 7.2 TB/s of U, V and sky values; lmax
// 64, mbmax 4: 12 us, now 4; four waves instead of eight 0.41 ms and 5 us).  Workgroups of one l tile follow
// each other (they share its sky values), the long sums of the largest l first.
constexpr int BEAM_W = 8;       // waves per workgroup
constexpr int BEAM_U = 4;       // values of ms a wave has in flight
__device__ __forceinline__ void beam_grad(const EpiArgs& e, int ntile, int block, double2 (&part)[BEAM_W][64])
{
    const int nmb = 2 * e.mbmax + 1;
    const int mb = block % nmb - e.mbmax;
    const int l0 = (ntile - 1 - block / nmb) * 64;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int l = l0 + lane, lc = min(l, e.lmax), lmax_tile = min(l0 + 63, e.lmax);
    const double2* U = reinterpret_cast<const double2*>(e.U) + (size_t)(mb + e.mbmax) * e.P + lc;
    const double2* V = reinterpret_cast<const double2*>(e.V) + (size_t)(-mb + e.mbmax) * e.P + lc;
    const double2* alm = reinterpret_cast<const double2*>(e.alm) + lc;
    double br = 0.0, bi = 0.0;
    auto add = [&](int ms, double2 u, double2 v, double2 s) {
        const double sg = ((l - ms) & 1) ? -1.0 : 1.0;
        const double x = u.x + sg * v.x, y = u.y + sg * v.y;
        br += s.x * x + s.y * y;
        bi += s.y * x - s.x * y;
    };
    for (int ms0 = wave; ms0 <= lmax_tile; ms0 += BEAM_U * BEAM_W) {
        double2 u[BEAM_U], v[BEAM_U], s[BEAM_U];
#pragma unroll
        for (int q = 0; q < BEAM_U; ++q) {   // rows above a lane's l: an entry of an earlier row, not added
            const int ms = min(ms0 + q * BEAM_W, lmax_tile);
            const size_t k = packed_index(e.lmax, 0, ms);
            u[q] = ldg(U + k);
            v[q] = ldg(V + k);
            s[q] = ldg(alm + packed_index(e.sky_lmax, 0, ms));
        }
#pragma unroll
        for (int q = 0; q < BEAM_U; ++q)
            if (ms0 + q * BEAM_W <= lc) add(ms0 + q * BEAM_W, u[q], v[q], s[q]);
    }
    part[wave][lane] = make_double2(br, bi);
    __syncthreads();
    if (wave == 0 && l <= e.lmax) {
#pragma unroll
        for (int w = 1; w < BEAM_W; ++w) {
            br += part[w][lane].x;
            bi += part[w][lane].y;
        }
        const bool in = l >= abs(mb);
        stg(reinterpret_cast<double2*>(e.blm_bar) + (size_t)(mb + e.mbmax) * (e.lmax + 1) + l,
            make_double2(in ? br : 0.0, in ? bi : 0.0));
    }
}

__global__ void __launch_bounds__(64 * BEAM_W) k_adj_beam(const EpiArgs e, int ntile)
{
    __shared__ double2 part[BEAM_W][64];
    beam_grad(e, ntile, blockIdx.x, part);
}

// Both gradients in one launch: the beam's workgroups first, then the sky's rows in pieces of 64 BEAM_W.  The
// two take 0.77 ms either way at lmax 2048, mbmax 14; at lmax 64, mbmax 4 one launch less takes 3.7 of the
// call's 33 us.
__global__ void __launch_bounds__(64 * BEAM_W) k_adj_grads(const EpiArgs e, int ntile, int nbeam, int npiece)
{
    __shared__ double2 part[BEAM_W][64];
    if ((int)blockIdx.x < nbeam) {
        beam_grad(e, ntile, blockIdx.x, part);
        return;
    }
    const int b = (int)blockIdx.x - nbeam;
    const int ms = b / npiece;
    sky_grad(e, ms, ms + (b % npiece) * (64 * BEAM_W) + (int)threadIdx.x);
}

template <typename Args>
int launch_grid(void (*kern)(Args), const Args& a, int blocks, int nt, void* stream)
{
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(nt), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

// Whether row mb of a beam equals row -mb up to a sign for every l >= mb: +1 (also when both signs hold, as
// for zero rows and mb = 0), -1, or 0.  All threads of the workgroup take part.
__device__ __forceinline__ int beam_row_sign(const double2* blm, int lmax, int mbmax, int mb)
{
    const double2* bp = blm + (size_t)(mbmax + mb) * (lmax + 1);
    const double2* bm = blm + (size_t)(mbmax - mb) * (lmax + 1);
    bool plus = true, minus = true;
    for (int l = mb + (int)threadIdx.x; l <= lmax; l += 256) {
        const double2 p = ldg(bp + l), m = ldg(bm + l);
        plus = plus && (m.x == p.x) && (m.y == p.y);
        minus = minus && (m.x == -p.x) && (m.y == -p.y);
    }
    plus = __syncthreads_and(plus);
    minus = __syncthreads_and(minus);
    return plus ? 1 : (minus ? -1 : 0);
}

// Row signs of one beam: sym[M + mb] = sym[M - mb], one workgroup per mb = 0 .. mbmax.
__global__ void __launch_bounds__(256) k_beam_symmetry(const double2* __restrict__ blm, int lmax, int mbmax,
                                                       int* __restrict__ sym)
{
    const int mb = blockIdx.x;
    const int s = beam_row_sign(blm, lmax, mbmax, mb);
    if (threadIdx.x == 0) {
        sym[mbmax + mb] = s;
        sym[mbmax - mb] = s;
    }
}

// What a call needs before its walks, in one launch: its tables, read by the copy workgroups from the
// pinned host image (mapped memory) into the workspace, and the row signs of its beams by mbmax + 1 more
// (for two or three polarised pairs, pair p's sign + 1 in byte p of a word).  A copy by the DMA engine and
// the kernel that waits for it cost 20 to 27 us of a small call; this launch takes 4 to 5.
constexpr int PREP_LOADS = 4;   // 16-byte loads in flight per lane
__global__ void __launch_bounds__(256) k_prep(const PrepArgs a, int ncopy)
{
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < ncopy) {
        typedef unsigned v4 __attribute__((ext_vector_type(4)));
        const v4* src = static_cast<const v4*>(a.src);
        v4* dst = static_cast<v4*>(a.dst);
        const size_t n = a.bytes / 16, i0 = (size_t)blockIdx.x * (256 * PREP_LOADS) + tid;
        v4 v[PREP_LOADS];
#pragma unroll
        for (int k = 0; k < PREP_LOADS; ++k)
            if (i0 + 256 * k < n) v[k] = src[i0 + 256 * k];
#pragma unroll
        for (int k = 0; k < PREP_LOADS; ++k)
            if (i0 + 256 * k < n) dst[i0 + 256 * k] = v[k];
        return;
    }
    const int mb = blockIdx.x - ncopy;
    int word = 0;
#pragma unroll
    for (int p = 0; p < 3; ++p)
        if (p < a.npair) {
            const int s = beam_row_sign(reinterpret_cast<const double2*>(a.blm[p]), a.lmax, a.mbmax, mb);
            word |= a.npair == 1 ? s : (s + 1) << (8 * p);
        }
    if (tid == 0) {
        a.sym[a.mbmax + mb] = word;
        a.sym[a.mbmax - mb] = word;
    }
}

}  // namespace

// Built tile variants (NT lanes per workgroup).  Forward: R in {2, 4, 8} (polarised: {2, 4}) with
// NT in {64, 128, 256}; TB shapes no forward kernel (a block is NT values of l).  Adjoint: R in
// {2, 4, 8}, TB 32 with each NT, TB 64 with NT 256.  Wigner: NT 128 with one chain per lane (R in {1, 4} is
// accepted and shapes nothing).
bool tile_supported(int op, Tile t)
{
    const bool nt_ok = t.NT == 64 || t.NT == 128 || t.NT == 256;
    const bool tb_ok = t.TB == 32 || t.TB == 64;
    const bool r_ok = t.R == 2 || t.R == 4 || t.R == 8;
    if (op == 0) return (t.R == 1 || t.R == 4) && t.TB == 32;
    if (op == 1) return r_ok && tb_ok && nt_ok;
    if (op == 2) return r_ok && tb_ok && t.TR == 4 && (t.NT == 256 || (nt_ok && t.TB == 32));
    if (op == 3) return (t.R == 2 || t.R == 4) && tb_ok && nt_ok;
    return false;
}

int launch_wigner(const WignerArgs& a, Tile t, void* stream)
{
    if (t.R != 1 || t.NT != 128) return (int)hipErrorInvalidValue;   // a.ntile counts tiles of 128 rings
    return launch_grid(k_wigner<128>, a, a.npair * a.ntile, 128, stream);
}

// Maps a runtime (R, NT[, TB]) onto the template instantiation F<R, NT[, TB]>.
#define TC_NT(X, r) X(r, 64) X(r, 128) X(r, 256)
#define TC_FWD_VARIANTS(X) TC_NT(X, 2) TC_NT(X, 4) TC_NT(X, 8)
#define TC_NT_POL(X, r, c, p) X(r, 64, c, p) X(r, 128, c, p) X(r, 256, c, p)
#define TC_FWDPOL_VARIANTS(X)                                                                  \
    TC_NT_POL(X, 2, 1, 2) TC_NT_POL(X, 4, 1, 2) TC_NT_POL(X, 2, 1, 3) TC_NT_POL(X, 4, 1, 3)    \
    TC_NT_POL(X, 2, 2, 2) TC_NT_POL(X, 4, 2, 2) TC_NT_POL(X, 2, 3, 3) TC_NT_POL(X, 4, 3, 3)
#define TC_POL_ROWS_NT(Y, r, c) Y(r, 64, c) Y(r, 128, c) Y(r, 256, c)
#define TC_POL_ROWS_VARIANTS(Y) TC_POL_ROWS_NT(Y, 2, 2) TC_POL_ROWS_NT(Y, 4, 2) TC_POL_ROWS_NT(Y, 2, 3) TC_POL_ROWS_NT(Y, 4, 3)
#define TC_ADJ_NT(X, r) X(r, 64, 32) X(r, 128, 32) X(r, 256, 32) X(r, 256, 64)
#define TC_ADJ_VARIANTS(X) TC_ADJ_NT(X, 2) TC_ADJ_NT(X, 4) TC_ADJ_NT(X, 8)

int launch_beam_symmetry(const double* blm, int lmax, int mbmax, int* sym, void* stream)
{
    hipLaunchKernelGGL(k_beam_symmetry, dim3(mbmax + 1), dim3(256), 0, (hipStream_t)stream,
                       reinterpret_cast<const double2*>(blm), lmax, mbmax, sym);
    return (int)hipGetLastError();
}

int launch_prep(const PrepArgs& a, void* stream)
{
    const int ncopy = (int)((a.bytes / 16 + 256 * PREP_LOADS - 1) / (256 * PREP_LOADS));
    const int blocks = ncopy + (a.npair > 0 ? a.mbmax + 1 : 0);
    if (blocks == 0) return 0;
    hipLaunchKernelGGL(k_prep, dim3(blocks), dim3(256), 0, (hipStream_t)stream, a, ncopy);
    return (int)hipGetLastError();
}

// The scalar forward of one column set: for NT < 256 one launch of both forms, else one of each.
template <int R, int NT>
static int launch_fwd_scalar(const FwdArgs& a, void* stream)
{
    const int blocks = a.ncol * a.ntile;
    if constexpr (NT < 256) {
        return launch_grid(k_fwd_either<R, NT>, a, blocks, NT, stream);
    } else {
        const int rc = launch_grid(k_fwd_rows<R, NT>, a, blocks, NT, stream);
        return rc ? rc : launch_grid(k_fwd<R, NT, 1, 1>, a, blocks, NT, stream);
    }
}

// The adjoint's columns; with row signs (the sky gradient alone) the same split.
template <int R, int NT, int TB>
static int launch_adj_columns(const AdjArgs& a, void* stream)
{
    if (a.beam_sym) {
        if constexpr (NT < 256) {
            return launch_grid(k_adj_either<R, NT, TB>, a, a.ncol, NT, stream);
        } else {
            const int rc = launch_grid(k_adj_one_sum<R, NT, TB>, a, a.ncol, NT, stream);
            if (rc) return rc;
        }
    }
    return launch_grid(k_adj<R, NT, TB>, a, a.ncol, NT, stream);   // every ring tile of a column in one workgroup
}

int launch_fwd(const FwdArgs& a, Tile t, void* stream)
{
    const int blocks = a.ncol * a.ntile;
    if (a.npair == 1) {
        if (!a.beam_sym[0]) return (int)hipErrorInvalidValue;   // a call of one pair always has its row signs
#define X(r, nt) if (t.R == r && t.NT == nt) return launch_fwd_scalar<r, nt>(a, stream);
        TC_FWD_VARIANTS(X)
#undef X
        return (int)hipErrorInvalidValue;
    }
    const int nc = a.sum ? 1 : a.npair;
    if (nc > 1 && a.beam_sym[0]) {   // the columns where every pair's rows are related
        int rc = 0;
#define Y(r, nt, c) if (!rc && t.R == r && t.NT == nt && nc == c) rc = launch_grid(k_fwd_pol_rows<r, nt, c>, a, blocks, nt, stream);
        TC_POL_ROWS_VARIANTS(Y)
#undef Y
        if (rc) return rc;
    }
#define X(r, nt, c, p)                                         \
    if (t.R == r && t.NT == nt && nc == c && a.npair == p)     \
        return launch_grid(k_fwd<r, nt, c, p>, a, blocks, nt, stream);
    TC_FWDPOL_VARIANTS(X)
#undef X
    return (int)hipErrorInvalidValue;
}

int launch_adj(const AdjArgs& a, Tile t, void* stream)
{
#define X(r, nt, tb) if (t.R == r && t.NT == nt && t.TB == tb) return launch_adj_columns<r, nt, tb>(a, stream);
    TC_ADJ_VARIANTS(X)
#undef X
    return (int)hipErrorInvalidValue;
}

int launch_adj_epilogue(const EpiArgs& e, void* stream)
{
    const int nt = 256;
    if (e.alm_bar && e.blm_bar) {
        const int ntile = (e.lmax + 64) / 64, nbeam = ntile * (2 * e.mbmax + 1);
        const int npiece = (e.sky_lmax + 64 * BEAM_W) / (64 * BEAM_W);
        hipLaunchKernelGGL(k_adj_grads, dim3(nbeam + npiece * (e.sky_lmax + 1)), dim3(64 * BEAM_W), 0,
                           (hipStream_t)stream, e, ntile, nbeam, npiece);
        return (int)hipGetLastError();
    }
    if (e.alm_bar) {
        dim3 grid((e.sky_lmax + 1 + nt - 1) / nt, e.sky_lmax + 1);
        hipLaunchKernelGGL(k_adj_sky, grid, dim3(nt), 0, (hipStream_t)stream, e);
        const int rc = (int)hipGetLastError();
        if (rc) return rc;
    }
    if (e.blm_bar) return launch_adj_beam(e, stream);
    return 0;
}

int launch_adj_beam(const EpiArgs& e, void* stream)
{
    const int ntile = (e.lmax + 64) / 64;
    hipLaunchKernelGGL(k_adj_beam, dim3(ntile * (2 * e.mbmax + 1)), dim3(64 * BEAM_W), 0, (hipStream_t)stream, e, ntile);
    return (int)hipGetLastError();
}

int launch_fwd_items(const FwdArgs* walks, const int* items, int nitems, Tile t, void* stream)
{
    if (nitems <= 0) return 0;
    hipStream_t s = (hipStream_t)stream;
#define X(r, nt)                                                                                         \
    if (t.R == r && t.NT == nt) {                                                                        \
        hipLaunchKernelGGL((k_fwd_items<r, nt>), dim3(nitems), dim3(nt), 0, s, walks, items);            \
        return (int)hipGetLastError();                                                                   \
    }
    TC_FWD_VARIANTS(X)
#undef X
    return (int)hipErrorInvalidValue;
}

int fwd_walk_pairs(Tile t) { return t.R >= 8 ? walk_pairs<8>() : walk_pairs<4>(); }

int adj_walk_pairs_of(Tile t)
{
    if (t.TB > 32) return adj_walk_pairs<4, 64>();
    return t.R >= 8 ? adj_walk_pairs<8, 32>() : adj_walk_pairs<4, 32>();
}

int launch_adj_items(const AdjArgs* dets, const int* items, int nitems, Tile t, void* stream)
{
    if (nitems <= 0) return 0;
    hipStream_t s = (hipStream_t)stream;
#define X(r, nt, tb)                                                                                    \
    if (t.R == r && t.NT == nt && t.TB == tb) {                                                         \
        hipLaunchKernelGGL((k_adj_items<r, nt, tb>), dim3(nitems), dim3(nt), 0, s, dets, items);        \
        return (int)hipGetLastError();                                                                  \
    }
    TC_ADJ_VARIANTS(X)
#undef X
    return (int)hipErrorInvalidValue;
}

int launch_adj_sky_multi(const EpiArgs* eps, int ndet, int sky_lmax, bool accumulate, double* alm_bar, void* stream)
{
    const int nt = 256;
    dim3 grid((sky_lmax + 1 + nt - 1) / nt, sky_lmax + 1);
    hipLaunchKernelGGL(k_adj_sky_multi, grid, dim3(nt), 0, (hipStream_t)stream, eps, ndet, sky_lmax,
                       accumulate ? 1 : 0, alm_bar);
    return (int)hipGetLastError();
}

}  // namespace tc
