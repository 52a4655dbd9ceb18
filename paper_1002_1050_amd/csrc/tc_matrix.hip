// gfx950 kernel of the full reduced Wigner matrix at one l (Sec. 3.1): every
// d^l_{m m'}(beta_j), -l <= m, m' <= l, for a set of rings.
//
// Sec. 3.1 walks a row of fixed l and m in m' with the three-term relation of
// Sec. 2 (eq. mrec), as ratios anchored at d^l_{00}.  Here the same relation runs
// on the values, downwards from the closed-form end point d^l_{m,l} = A c^{l+m}
// s^{l-m} (the seed of Sec. 3.2, as a logarithm, with exact power-of-two scaling
// while the values are tiny), on the triangle 0 <= m <= m' <= l only, where the
// wanted solution grows or oscillates in the direction of the walk:
//
//   d_{m,m'-1} = [2 (m' cot(beta) - m csc(beta)) d_{m,m'} - b_{m'} d_{m,m'+1}] / a_{m'},
//   a_{m'} = sqrt((l+m')(l-m'+1)),  b_{m'} = sqrt((l-m')(l+m'+1)).
//
// The rest of the matrix follows from the symmetries of the appendix:
//   d_{m',m} = (-1)^(m-m') d_{m,m'},  d_{-m,-m'} = (-1)^(m-m') d_{m,m'},
//   d_{m,-m'}(beta) = (-1)^(l+m) d_{m,m'}(pi - beta),
// so a workgroup walks the triangle at beta (side 0) or at pi - beta (side 1, rows
// m >= 1, whose images are the quadrants with m m' < 0) and writes each value to
// its images.  One lane walks one row m of one ring; per-step coefficients depend on
// the ring and m' only and are staged in LDS.

#include <hip/hip_runtime.h>

#include "tc_internal.h"

namespace tc {
namespace {

constexpr int MS_TS = 8;          // steps between scale checks
constexpr int MS_FOLD = -900;     // scaled values fold into plain doubles at 2^-900

__device__ __forceinline__ bool wave_any_m(bool p) { return __ballot(p) != 0ull; }

__device__ __forceinline__ void two_sum_m(double a, double b, double& s, double& e)
{
    s = a + b;
    const double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// (sh, sl) += n * (ah + al), n an integer held exactly in a double
__device__ __forceinline__ void dd_add_times_m(double& sh, double& sl, double n, double ah, double al)
{
    const double ph = n * ah;
    const double pl = fma(n, ah, -ph) + n * al;
    double s, e;
    two_sum_m(sh, ph, s, e);
    e += sl + pl;
    sh = s + e;
    sl = e - (sh - s);
}

// d^l_{m,l} = A c^p s^q (p = l+m, q = l-m, c, s > 0 here) as a significand in
// [1, 2) times 2^E (E < 0), or a plain double (E = 0) once >= 2^-900.
__device__ __forceinline__ void row_seed(double lnAh, double lnAl, int p, int q, double lch, double lcl,
                                         double lsh, double lsl, double& d, int& E)
{
    double h = lnAh, lo = lnAl;
    if (p > 0) dd_add_times_m(h, lo, (double)p, lch, lcl);
    if (q > 0) dd_add_times_m(h, lo, (double)q, lsh, lsl);
    // ln -> log2 in double-double
    const double L2h = 0x1.71547652b82fep+0, L2l = 0x1.777d0ffda0d24p-56;
    const double ph = h * L2h;
    const double pe = fma(h, L2h, -ph) + (h * L2l + lo * L2h);
    const double yh = ph + pe, yl = pe - (yh - ph);
    const double k = floor(yh);
    const double m = exp2((yh - k) + yl);
    const int ik = (int)k;
    if (ik >= MS_FOLD) { d = ldexp(m, ik); E = 0; }
    else { d = m; E = ik; }
}

// The four images of the walked element (m, mp) (mp >= m >= 0).  Side 0: v =
// d_{m,mp}(beta) goes to (m, mp), (mp, m), (-m, -mp), (-mp, -m) with signs 1, s, s, 1
// (s = (-1)^(m-mp)).  Side 1: u = (-1)^(l+m) v with v = d_{m,mp}(pi - beta) is
// d_{m,-mp}(beta) and goes to (m, -mp), (-mp, m), (-m, mp), (mp, -m), signs 1, s, s, 1.
// Images 1 and 3 run along an output row as m runs, images 0 and 2 as mp runs.
//
// What bounds it: 8 bytes of stores per element, and how they reach memory.  Lines written in two parts
// are what costs most: with every 1 KB piece of a row starting where its tile does, 5% of the write
// requests were parts of a line and the rate was 3.1 TB/s; with all pieces on line boundaries (rows padded,
// to time it) 4.3.  Rows are 2l + 1 doubles, so the boundaries differ from row to row:
//  - images 1 and 3 (pieces along m): a workgroup walks ROWS = 128 rows and owns the lines whose
//    lowest m is one of its first OWN = 112, so the last 16 rows are walked twice;
//  - images 0 and 2 (pieces along m'): rows keep up to 15 steps back until their line is complete, in a
//    ring of RING = FL + 16 steps.
// Two of the eight waves walk 128 steps into LDS, then all eight store the four images 16 bytes per
// lane; the walk of the next 128 steps runs while those stores drain.  l = 4096 on 16 rings (8.6 GB):
// 2.87 ms with two waves that walked, stored images 1 and 3 step by step and the others every 128 steps;
// 2.78 ms with eight waves storing whole pieces wherever their lines lay; now 1.87 ms, 4.6 TB/s.
constexpr int M_NT = kMatrixLanes, ROWS = 128, OWN = 112, FL = 128, RING = FL + 16;
constexpr int LINE = 16;   // doubles per line

// A pair of neighbouring elements of an output row, on an 8-byte boundary.
typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ void st(double* p, double v) { *(__attribute__((address_space(1))) double*)p = v; }
__device__ __forceinline__ void st2(double* p, double a, double b)
{
    pair_t v;
    v.x = a;
    v.y = b;
    *(__attribute__((address_space(1))) pair_t*)p = v;
}

__global__ void __launch_bounds__(M_NT) k_wigner_row(const MatrixArgs a)
{
    static_assert(FL == 128 && ROWS == 128 && FL % MS_TS == 0 && RING % MS_TS == 0, "pairs of 64 lanes cover a piece");
    static_assert(OWN % LINE == 0 && FL % LINE == 0 && ROWS >= OWN + LINE - 1, "whole lines");
    __shared__ double4 cf[2][FL];             // per step: {A, nB, F2, -}: d_next = (m A + nB) d - F2 d_prev
    __shared__ double held[RING][ROWS + 1];   // values u of the last RING steps, per row
    const int tid = threadIdx.x;
    const int per_tile = 2 * a.nring;
    const int tile = blockIdx.x / per_tile;
    const int rem = blockIdx.x - tile * per_tile;
    const int j = rem >> 1, side = rem & 1;
    const int l = a.l;
    const int W = 2 * l + 1;
    double* __restrict__ out = a.d + (size_t)j * (size_t)W * (size_t)W;
    const double x = a.ring.x[j];
    const int m_base = tile * OWN;
    const int m_lo = max(m_base, side);       // lowest row of the workgroup
    if (m_lo > l) return;
    const bool walker = tid < ROWS;           // waves 0 and 1
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), ln = tid & 63;

    const bool pole = (x == 1.0 || x == -1.0);
    const bool ident = (side == 0) == (x == 1.0);   // at a pole: the walked triangle is at beta = 0
    double cot = 0.0, csc = 0.0;
    double xm = 0.0, d = 0.0, dp = 0.0, rs = 1.0;
    int E = 0, mrow = 0;
    bool scaled = false;
    if (!pole) {
        cot = side ? -a.trig[2 * j] : a.trig[2 * j];
        csc = a.trig[2 * j + 1];
    }
    if (walker) {
        mrow = min(max(m_base + tid, side), l);   // lanes without a row repeat one, and are not stored
        xm = (double)mrow;
        if (!pole) {
            // c' = cos((pi - beta)/2) = sin(beta/2) on side 1
            const double lch = side ? a.ring.lsh[j] : a.ring.lch[j], lcl = side ? a.ring.lsl[j] : a.ring.lcl[j];
            const double lsh = side ? a.ring.lch[j] : a.ring.lsh[j], lsl = side ? a.ring.lcl[j] : a.ring.lsl[j];
            row_seed(a.lnA[2 * mrow], a.lnA[2 * mrow + 1], l + mrow, l - mrow, lch, lcl, lsh, lsl, d, E);
        }
        rs = (side == 1 && ((l + mrow) & 1)) ? -1.0 : 1.0;   // side 1 carries (-1)^(l+m)
        scaled = wave_any_m(E < 0);
    }

    // step s: from m' = l - s to m' - 1; steps needed: l - m_lo
    const int nsteps = l - m_lo;
    auto coefs = [&](int s) {
        const int mp = l - s;
        double4 c = make_double4(0.0, 0.0, 0.0, 0.0);
        if (!pole && s < nsteps) {
            const double av = sqrt((double)(l + mp) * (double)(l - mp + 1));
            const double bv = sqrt((double)(l - mp) * (double)(l + mp + 1));
            c = make_double4(-2.0 * csc / av, 2.0 * (double)mp * cot / av, bv / av, 0.0);
        }
        return c;
    };
    if (tid < FL) cf[0][tid] = coefs(tid);
    auto at = [&](int row, int col) { return out + (size_t)(row + l) * (size_t)W + (size_t)(col + l); };
    // place of column 0 of an output row within its line
    const unsigned out_pos = (unsigned)((reinterpret_cast<uintptr_t>(out) >> 3) & (LINE - 1));
    auto pos0 = [&](int row) { return (int)((out_pos + (unsigned)(row + l) * (unsigned)W + (unsigned)l) & (LINE - 1)); };
    // the lowest m' >= mp at which a line of the output row ends (images along m' = col or -col)
    auto line_end = [&](int row, bool minus, int mp) {
        const int p = pos0(row);
        return mp + (minus ? (p + 1 - mp) & (LINE - 1) : -(p + mp) & (LINE - 1));
    };
    auto ring = [&](int s) { return s < RING ? s : s - RING; };
    int hb = 0;   // s0 mod RING
    for (int s0 = 0, kb = 0; s0 <= nsteps; s0 += FL, ++kb, hb = ring(hb + FL)) {
        const int buf = kb & 1;
        const int n = min(FL, nsteps + 1 - s0);   // steps of this block
        const int mp_a = l - s0 + 1;              // lowest m' of the block before
        const int mp_b = l - (s0 + n - 1);        // lowest m' now
        __syncthreads();                          // coefficients there, the block before stored
        if (walker) {
            int h = hb;
            for (int t0 = 0; t0 < n; t0 += MS_TS, h = ring(h + MS_TS)) {   // a group does not wrap the ring
                if (scaled) {
                    // exact power-of-two rescale; fold into plain doubles at 2^-900
                    int e1, e2;
                    frexp(d, &e1);
                    frexp(dp, &e2);
                    const bool nz = (d != 0.0) | (dp != 0.0);
                    const int e = max(d != 0.0 ? e1 : -(1 << 20), dp != 0.0 ? e2 : -(1 << 20));
                    const bool sc = nz & (E < 0);
                    const bool fold = (E + e) >= MS_FOLD;
                    const int k = sc ? (fold ? E : -e) : 0;
                    E = sc ? (fold ? 0 : E + e) : E;
                    d = ldexp(d, k);
                    dp = ldexp(dp, k);
                    scaled = wave_any_m(E < 0);
                }
                double4 kk[MS_TS];   // zero beyond the last step
#pragma unroll
                for (int t = 0; t < MS_TS; ++t) kk[t] = cf[buf][t0 + t];
#pragma unroll
                for (int t = 0; t < MS_TS; ++t) {
                    double v = scaled ? ldexp(d, E) : d;
                    if (pole) {
                        const int mp = l - (s0 + t0 + t);
                        v = ident ? (mp == mrow ? 1.0 : 0.0)
                                  : ((mrow == 0 && mp == 0) ? ((l & 1) ? -1.0 : 1.0) : 0.0);
                    }
                    held[h + t][tid] = rs * v;
                    const double w = fma(xm, kk[t].x, kk[t].y);
                    const double dn = fma(-kk[t].z, dp, w * d);
                    dp = d;
                    d = dn;
                }
            }
        } else if (tid >= M_NT - FL && s0 + FL <= nsteps) {
            cf[buf ^ 1][tid - (M_NT - FL)] = coefs(s0 + FL + tid - (M_NT - FL));
        }
        __syncthreads();
        constexpr int NW = M_NT / 64, U = 4;
        auto at_step = [&](int s) {   // ring slot of step s in (s0 - LINE, s0 + FL)
            const int h = hb + (s - s0);
            return h < 0 ? h + RING : ring(h);
        };

        // Images 0 and 2: a wave per row m, its line-complete stretch of m'.  Each image has its own line
        // boundaries; past the last block that still has m' > m the rest of the row goes out.
        if (s0 > 0 && n == FL && mp_b > m_base + OWN - 1) {
            for (int k0 = 0; k0 < OWN / NW; k0 += 2) {
                double u0[2][2], u1[2][2];
                int top[2][2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int q = wave + NW * (k0 + k), m = m_base + q;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {   // image 2 i
                        top[k][i] = line_end(i ? -m : m, (side == 1) != (i == 1), mp_a) - 1;
                        const int s = l - top[k][i] + 2 * ln;
                        u0[k][i] = held[at_step(s)][q];
                        u1[k][i] = held[at_step(s + 1)][q];
                    }
                }
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int m = m_base + wave + NW * (k0 + k);
                    if (m < side) continue;   // row 0 belongs to side 0
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int mp = top[k][i] - 2 * ln;   // and mp - 1
                        double f0 = u0[k][i], f1 = u1[k][i];
                        if (i) { if ((m - mp) & 1) f0 = -f0; else f1 = -f1; }
                        if ((side == 1) != (i == 1)) st2(at(i ? -m : m, -mp), f0, f1);
                        else st2(at(i ? -m : m, mp - 1), f1, f0);
                    }
                }
            }
        } else {
            for (int q = wave; q < OWN; q += NW) {
                const int m = m_base + q;
                if (m < side || m > l || (s0 > 0 && mp_a <= m)) continue;
                for (int i = 0; i < 2; ++i) {
                    const bool minus = (side == 1) != (i == 1);
                    const int row = i ? -m : m;
                    const int hi = s0 > 0 ? line_end(row, minus, mp_a) - 1 : l;
                    const int lo = mp_b <= m ? m : line_end(row, minus, mp_b);
                    for (int mp = hi - ln; mp >= lo; mp -= 64) {
                        const double u = held[at_step(l - mp)][q];
                        st(at(row, minus ? -mp : mp), (i && ((m - mp) & 1)) ? -u : u);
                    }
                }
            }
        }

        // Images 1 and 3: a wave per step m', the lines whose lowest m is an owned row (and, in the first
        // tile, the part of a line before the first).
        const bool full = mp_b >= m_base + ROWS - 1;   // every owned line lies within m <= m'
        for (int t0 = wave; t0 < n; t0 += NW * U) {
            double u0[U][2], u1[U][2];
            int ms[U][2];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int t = min(t0 + NW * k, n - 1), mp = l - s0 - t;
                const int r1 = side ? -mp : mp, p1 = pos0(r1), p3 = pos0(-r1);
                ms[k][0] = m_base + (-(m_base + p1) & (LINE - 1));
                ms[k][1] = m_base + ((p3 + 1 - m_base) & (LINE - 1));
                const int h = ring(hb + t);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int c = ms[k][i] - m_base + 2 * min(ln, OWN / 2 - 1);
                    u0[k][i] = held[h][c];
                    u1[k][i] = held[h][c + 1];
                }
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int t = t0 + NW * k, mp = l - s0 - t;
                if (t >= n) continue;
                const int r1 = side ? -mp : mp;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int m = ms[k][i] + 2 * ln;   // and m + 1
                    double f0 = u0[k][i], f1 = u1[k][i];
                    if (!i) { if ((m - mp) & 1) f0 = -f0; else f1 = -f1; }
                    double* const p = i ? at(-r1, -m - 1) : at(r1, m);
                    const bool in0 = ln < OWN / 2 && m >= side && m <= mp;
                    const bool in1 = ln < OWN / 2 && m + 1 >= side && m + 1 <= mp;
                    if (full ? (ln < OWN / 2 && m >= side) : (in0 && in1)) {
                        if (i) st2(p, f1, f0); else st2(p, f0, f1);
                    } else {
                        if (in0) st(i ? p + 1 : p, f0);
                        if (in1) st(i ? p : p + 1, f1);
                    }
                    if (tile == 0 && ln < ms[k][i] && ln >= side && ln <= mp) {   // m = ln before the first whole line
                        const double u = held[ring(hb + t)][ln];
                        st(i ? at(-r1, -ln) : at(r1, ln), (!i && ((ln - mp) & 1)) ? -u : u);
                    }
                }
            }
        }
    }
}

}  // namespace

// Rows m one workgroup owns.  One kernel serves every tile id (0 to 2, tc_set_tile).
int matrix_rows_per_group(int v) { return v >= 0 && v <= 2 ? OWN : 0; }

int launch_matrix(const MatrixArgs& a, int v, void* stream)
{
    if (matrix_rows_per_group(v) == 0) return (int)hipErrorInvalidValue;
    hipLaunchKernelGGL(k_wigner_row, dim3(a.ntile * 2 * a.nring), dim3(M_NT), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

}  // namespace tc
