// gfx950 kernels of the data-cube stage (Sec. 4.1, eq. conviqt):
//
//   c(alpha_a, beta_j, gamma_g) = sum_{mb=-M}^{M} sum_{msky=-L}^{L}
//                                 e^{-i mb alpha_a} e^{-i msky gamma_g} C_{mb,msky}(beta_j)
//
// on alpha_a = 2 pi a / nalpha, gamma_g = 2 pi g / ngamma, with the columns msky < 0
// taken from C_{-mb,-msky} = conj(C_{mb,msky}) (real sky and beam, Sec. 4.2.3), so
// that c is real.
//
// Two passes over each chunk of rings, both bound by HBM bandwidth.  At lmax 2048, mbmax 14, 2000 rings,
// 29 x 4096 angles (1.9 GB of C in, 1.9 GB of P out and in, 1.9 GB of cube out) they take 0.93 and 0.85 ms,
// 4.1 and 4.5 TB/s of reads and writes together; the call 1.77 ms (2.42 ms with unpadded rows of P, the passes
// side by side in smaller chunks, gamma workgroups of 256 lanes for every row and a sum over mb term by term):
//  1. k_cube_alpha: P[j][a][k] = sum_mb e^{-i mb alpha_a} C[mb][k][j] for k = msky >= 0 -- the
//     short sum over mb, done directly over pairs (mb, -mb) and (alpha, -alpha) with the host's
//     table of phases, and the transpose from ring-fastest C to rows (ring, alpha) with msky
//     fastest.
//  2. k_cube_gamma: one workgroup per row turns P_0..P_L into the real row
//     c[g] = Re P_0 + 2 Re sum_{k>=1} P_k e^{-2 pi i k g / N}: the Hermitian
//     spectrum is folded into its half X_0..X_{N/2}, packed into one complex
//     sequence of length H = N/2 (even outputs in the real part, odd outputs in the
//     imaginary part) and transformed by a Stockham FFT in LDS (radix-16 passes and
//     one smaller one), twiddles from the host's table W^m = e^{-2 pi i m / N}.

#include <hip/hip_runtime.h>

#include "tc_internal.h"

namespace tc {
namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x));
}

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }

// Streaming store of a cube element (written once, read by no later pass here).
typedef double nt_d2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_stream(double2* p, double2 v)
{
    nt_d2 w;
    w.x = v.x; w.y = v.y;
    __builtin_nontemporal_store(w, reinterpret_cast<nt_d2*>(p));
}

// ------------------------------------------------------------ alpha sums
// A workgroup's tile: CA_J rings (256-byte reads of C) by CA_K values of msky (256-byte stores of P, whole
// lines: the rows of P are padded to lines).  Tiles of 16 x 32 or 32 x 16 with 512 lanes took 3 to 6% longer
// (two workgroups' barriers per compute unit instead of four).
constexpr int CA_J = 16, CA_K = 16, CA_NT = CA_J * CA_K;
constexpr int CA_S = 4;     // slots (8 values of alpha) per transposed store
constexpr int CA_U = 4;     // values of |mb| whose C are in flight together

// Each lane owns one (msky, ring) element.  With c, s = cos, sin of 2 pi m q / nalpha,
//   e^{-i theta} C_m + e^{i theta} C_{-m} = c S + s T,  S = C_m + C_{-m},  T = -i (C_m - C_{-m}),
// and alpha nalpha - q takes the same with -s: so slot q keeps A = sum_m c S and B = sum_m s T, four FMAs per
// |mb| for two values of alpha, and P_q = A + B, P_{nalpha-q} = A - B: one FMA where the sum term by term took
// four.  At mbmax 14 and 29 alphas that hides the arithmetic behind the loads (0.98 -> 0.93 ms at 2000 rings
// of lmax 2048, the call of 4000 rings at lmax 4096 8.00 -> 7.25 ms); at mbmax 25 and 66 alphas, where it was
// the bound, the call takes 0.75 ms instead of 1.90 (1000 rings, lmax 512).  The second launch bound holds the
// accumulators of 16 slots and 8 loads to two waves per SIMD; without it the compiler takes registers that
// leave one, 1.01 ms.  Slot 0 holds alpha 0 and, for even nalpha, alpha nalpha / 2, whose phases are 1 and (-1)^m:
// its A sums S over even m, its B over odd m.  The table [|mb|][slot] of (c, s) is read with uniform 64-byte
// loads, four slots at a time, so the phases arrive in scalar registers.
struct alignas(64) Phase4 {
    double2 v[4];
};

template <int QS>
__global__ void __launch_bounds__(CA_NT, 2) k_cube_alpha(const CubeArgs c, const double2* __restrict__ C,
                                                    const Phase4* __restrict__ E4, double2* __restrict__ P)
{
    static_assert(QS % 4 == 0 && QS % CA_S == 0, "phases come in fours");
    __shared__ double2 tile[2 * CA_S][CA_K][CA_J + 1];
    const int M = c.mbmax;
    const int ns = (c.nalpha + 1) / 2;      // slots
    const int ns4 = (ns + 3) / 4;           // Phase4 entries per row
    const int tid = threadIdx.x;
    const int jj = tid % CA_J, kk = tid / CA_J;
    const int j0 = blockIdx.x * CA_J, k0 = blockIdx.y * CA_K;
    const int j = j0 + jj, k = k0 + kk;
    const int L1 = c.lmax + 1;
    const bool in = (j < c.nring_chunk) && (k <= c.lmax);
    const size_t mb_stride = (size_t)L1 * c.nring;
    for (int s0 = 0; s0 < ns; s0 += QS) {
        double ax[QS], ay[QS], bx[QS], by[QS];
#pragma unroll
        for (int q = 0; q < QS; ++q) { ax[q] = 0.0; ay[q] = 0.0; bx[q] = 0.0; by[q] = 0.0; }
        if (in) {
            const double2* src = C + (size_t)M * mb_stride + (size_t)k * c.nring + (c.ring0 + j);
            for (int m0 = 0; m0 <= M; m0 += CA_U) {
                double2 vp[CA_U], vm[CA_U];
#pragma unroll
                for (int u = 0; u < CA_U; ++u) {
                    const int m = m0 + u;
                    vp[u] = m <= M ? src[(size_t)m * mb_stride] : make_double2(0.0, 0.0);
                    vm[u] = m > 0 && m <= M ? *(src - (size_t)m * mb_stride) : make_double2(0.0, 0.0);
                }
#pragma unroll
                for (int u = 0; u < CA_U; ++u) {
                    const int m = m0 + u;
                    if (m <= M) {
                        const double2 S = cadd(vp[u], vm[u]);
                        const double2 T = m > 0 ? make_double2(vp[u].y - vm[u].y, vm[u].x - vp[u].x)
                                                : make_double2(0.0, 0.0);
                        const double2 T0 = s0 == 0 ? S : T;
                        const Phase4* row = E4 + (size_t)m * ns4 + s0 / 4;
#pragma unroll
                        for (int q4 = 0; q4 < QS / 4; ++q4) {
                            if (s0 + 4 * q4 < ns) {
                                const Phase4 e = row[q4];
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    const int q = 4 * q4 + i;
                                    ax[q] = fma(e.v[i].x, S.x, ax[q]);
                                    ay[q] = fma(e.v[i].x, S.y, ay[q]);
                                    bx[q] = fma(e.v[i].y, q ? T.x : T0.x, bx[q]);
                                    by[q] = fma(e.v[i].y, q ? T.y : T0.y, by[q]);
                                }
                            }
                        }
                    }
                }
            }
        }
        // transposed stores, CA_S slots at a time: lanes with consecutive msky
#pragma unroll
        for (int q0 = 0; q0 < QS; q0 += CA_S) {
            if (s0 + q0 >= ns) break;
#pragma unroll
            for (int q = 0; q < CA_S; ++q) {
                tile[2 * q][kk][jj] = make_double2(ax[q0 + q] + bx[q0 + q], ay[q0 + q] + by[q0 + q]);
                tile[2 * q + 1][kk][jj] = make_double2(ax[q0 + q] - bx[q0 + q], ay[q0 + q] - by[q0 + q]);
            }
            __syncthreads();
            const int jw = tid / CA_K, kw = tid % CA_K;
            if (j0 + jw < c.nring_chunk && k0 + kw <= c.lmax) {
                double2* row = P + (size_t)(j0 + jw) * c.nalpha * c.prow + (k0 + kw);
                for (int q = 0; q < CA_S && s0 + q0 + q < ns; ++q) {
                    const int a = s0 + q0 + q, other = a ? c.nalpha - a : c.nalpha % 2 ? 0 : c.nalpha / 2;
                    row[(size_t)a * c.prow] = tile[2 * q][kw][jw];
                    if (other) row[(size_t)other * c.prow] = tile[2 * q + 1][kw][jw];
                }
            }
            __syncthreads();
        }
    }
}

// ------------------------------------------------------------ gamma FFT
// Forward DFT of size R (sign -) in registers: bit-reversed reorder, then radix-2
// stages with the 16th roots of unity as constants.
__device__ __forceinline__ double2 root16(int m, double2 z)
{
    // z * e^{-2 pi i m / 16}, m in [0, 8)
    constexpr double C1 = 0.9238795325112867;   // cos(pi/8)
    constexpr double S1 = 0.3826834323650898;   // sin(pi/8)
    constexpr double H2 = 0.7071067811865476;   // cos(pi/4)
    switch (m) {
    case 0: return z;
    case 4: return make_double2(z.y, -z.x);
    case 1: return cmul(z, make_double2(C1, -S1));
    case 2: return cmul(z, make_double2(H2, -H2));
    case 3: return cmul(z, make_double2(S1, -C1));
    case 5: return cmul(z, make_double2(-S1, -C1));
    case 6: return cmul(z, make_double2(-H2, -H2));
    default: return cmul(z, make_double2(-C1, -S1));
    }
}

template <int R>
__device__ __forceinline__ void dft_regs(double2 (&v)[R])
{
    constexpr int LOG = R == 2 ? 1 : R == 4 ? 2 : R == 8 ? 3 : 4;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        int r = 0;
#pragma unroll
        for (int b = 0; b < LOG; ++b) r |= ((i >> b) & 1) << (LOG - 1 - b);
        if (i < r) {
            const double2 t = v[i];
            v[i] = v[r];
            v[r] = t;
        }
    }
#pragma unroll
    for (int half = 1; half < R; half <<= 1) {
#pragma unroll
        for (int b = 0; b < R; b += 2 * half) {
#pragma unroll
            for (int q = 0; q < half; ++q) {
                const double2 t = root16(q * (8 / half), v[b + q + half]);
                v[b + q + half] = csub(v[b + q], t);
                v[b + q] = cadd(v[b + q], t);
            }
        }
    }
}

// LDS slot of element i: one pad slot per 16 elements, so that the first pass's
// stride-16 stores (and every other pass's accesses) spread over the banks.
__device__ __forceinline__ int pad(int i) { return i + (i >> 4); }

// Twiddles w_r = W^{r m1} for r < R from W^{m1}, W^{2 m1}, W^{4 m1}, W^{8 m1} of the
// host table: every w_r is a table entry or a product of at most three of them.
template <int R>
__device__ __forceinline__ void twiddle_base(const double2* __restrict__ tw, int m1, double2 (&b)[4])
{
    b[0] = tw[m1];
    if (R > 2) b[1] = tw[2 * m1];
    if (R > 4) b[2] = tw[4 * m1];
    if (R > 8) b[3] = tw[8 * m1];
}

template <int R>
__device__ __forceinline__ void apply_twiddles(double2 (&v)[R], const double2 (&b)[4])
{
    double2 w[R];
    w[1] = b[0];
    if (R > 2) { w[2] = b[1]; w[3] = cmul(b[0], b[1]); }
    if (R > 4) {
        w[4] = b[2];
#pragma unroll
        for (int r = 5; r < 8; ++r) w[r] = cmul(b[2], w[r - 4]);
    }
    if (R > 8) {
        w[8] = b[3];
#pragma unroll
        for (int r = 9; r < 16; ++r) w[r] = cmul(b[3], w[r - 8]);
    }
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(v[r], w[r]);
}

// Entry b in [0, H] of the half spectrum: X_b = Z_b + Z_{b-N} with Z_0 = Re P_0,
// Z_k = P_k and Z_{-k} = conj(P_k) for 1 <= k <= L (zero beyond L).
__device__ __forceinline__ double2 half_spec(const double2* __restrict__ P, int b, int N, int L)
{
    double2 z = make_double2(0.0, 0.0);
    if (b == 0) z = make_double2(P[0].x, 0.0);
    else if (b <= L) z = P[b];
    if (b > 0 && N - b <= L) z = cadd(z, cconj(P[N - b]));
    return z;
}

// Packed input of the half-length transform: F_k = (X_k + conj X_{H-k}) + i W^k (X_k - conj X_{H-k}).
__device__ __forceinline__ double2 packed(double2 a, double2 b, double2 w)
{
    const double2 s = cadd(a, cconj(b)), d = cmul(w, csub(a, cconj(b)));
    return make_double2(s.x - d.y, s.y + d.x);
}

// First Stockham pass (stride Ns = 1, unit twiddles), fed straight from HBM: lane g
// forms F_{g + r H/R} for r < R from the row of P and transforms them in registers.
// All of a lane's loads are issued before the first is used.  The result goes to LDS,
// or, when this is the only pass, to the output row.
template <int R, int HMAX, int NT>
__device__ __forceinline__ void first_pass(const double2* __restrict__ P, const double2* __restrict__ tw,
                                           int H, int N, int L, double2* X, double2* out, bool last)
{
    constexpr int GM = HMAX / (R * NT) > 0 ? HMAX / (R * NT) : 1;
    const int tid = threadIdx.x;
    const int ng = H / R;
    double2 v[GM][R];
#pragma unroll
    for (int i = 0; i < GM; ++i) {
        const int g = tid + NT * i;
        if (g < ng) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int k = g + r * ng;
                v[i][r] = packed(half_spec(P, k, N, L), half_spec(P, H - k, N, L), tw[k]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < GM; ++i) {
        const int g = tid + NT * i;
        if (g < ng) {
            dft_regs<R>(v[i]);
            if (last) {
#pragma unroll
                for (int r = 0; r < R; ++r) store_stream(out + g * R + r, v[i][r]);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) X[pad(g * R + r)] = v[i][r];
            }
        }
    }
    if (!last) __syncthreads();
}

// One later Stockham pass of radix R over X[0..H) in place (all reads, barrier, all
// writes, barrier); HMAX bounds H, hence the groups a lane handles.  The last pass
// (Ns = H / R, so each lane's outputs g + r Ns are contiguous across lanes) writes
// the output row instead.
template <int R, int HMAX, int NT, bool LAST>
__device__ __forceinline__ void stockham_pass(double2* X, int H, int Ns, int N, const double2* __restrict__ tw,
                                              double2* __restrict__ out)
{
    constexpr int GM = HMAX / (R * NT) > 0 ? HMAX / (R * NT) : 1;
    const int tid = threadIdx.x;
    const int ng = H / R;
    const int step = N / (Ns * R);
    double2 v[GM][R], b[GM][4];
    // twiddle loads first (their latency overlaps the LDS reads and the barrier)
#pragma unroll
    for (int i = 0; i < GM; ++i) {
        const int g = tid + NT * i;
        if (g < ng) twiddle_base<R>(tw, (g & (Ns - 1)) * step, b[i]);
    }
#pragma unroll
    for (int i = 0; i < GM; ++i) {
        const int g = tid + NT * i;
        if (g < ng) {
#pragma unroll
            for (int r = 0; r < R; ++r) v[i][r] = X[pad(g + r * ng)];
        }
    }
    if (!LAST) __syncthreads();
#pragma unroll
    for (int i = 0; i < GM; ++i) {
        const int g = tid + NT * i;
        if (g < ng) {
            const int k = g & (Ns - 1);
            apply_twiddles<R>(v[i], b[i]);
            dft_regs<R>(v[i]);
            const int base = (g - k) * R + k;
            if (LAST) {
#pragma unroll
                for (int r = 0; r < R; ++r) store_stream(out + base + r * Ns, v[i][r]);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) X[pad(base + r * Ns)] = v[i][r];
            }
        }
    }
    if (!LAST) __syncthreads();
}

template <int HMAX, int NT>
__global__ void __launch_bounds__(NT) k_cube_gamma(const CubeArgs c)
{
    extern __shared__ double2 X[];   // pad(H) + 1 entries
    const int row = blockIdx.x;      // (ring within the chunk) * nalpha + alpha
    const int N = c.ngamma, H = N / 2, L = c.lmax;
    const double2* P = reinterpret_cast<const double2*>(c.P) + (size_t)row * c.prow;
    const double2* tw = reinterpret_cast<const double2*>(c.tw);
    // f_n = c[2n] + i c[2n+1] is the length-H transform of F
    double2* out = reinterpret_cast<double2*>(c.cube) + ((size_t)c.ring0 * c.nalpha + row) * (size_t)H;
    switch (H) {
    case 1:
        if (threadIdx.x == 0) out[0] = packed(half_spec(P, 0, N, L), half_spec(P, 1, N, L), tw[0]);
        return;
    case 2: first_pass<2, HMAX, NT>(P, tw, H, N, L, X, out, true); return;
    case 4: first_pass<4, HMAX, NT>(P, tw, H, N, L, X, out, true); return;
    case 8: first_pass<8, HMAX, NT>(P, tw, H, N, L, X, out, true); return;
    default: break;
    }
    first_pass<16, HMAX, NT>(P, tw, H, N, L, X, out, H == 16);
    int Ns = 16, rem = H / 16;
    while (rem > 16) { stockham_pass<16, HMAX, NT, false>(X, H, Ns, N, tw, out); Ns *= 16; rem /= 16; }
    if (rem == 16) stockham_pass<16, HMAX, NT, true>(X, H, Ns, N, tw, out);
    else if (rem == 8) stockham_pass<8, HMAX, NT, true>(X, H, Ns, N, tw, out);
    else if (rem == 4) stockham_pass<4, HMAX, NT, true>(X, H, Ns, N, tw, out);
    else if (rem == 2) stockham_pass<2, HMAX, NT, true>(X, H, Ns, N, tw, out);
}

}  // namespace

// The gamma pass's builds: (half length up to, lanes), one radix-16 group of the first pass per lane at the
// largest half length, two at 8192.  With 256 lanes for every length half of them or more had no group at
// 2048 and below, and still held registers: 1.06 ms instead of 0.84 at half length 2048 (2000 x 29 rows),
// and 0.64 instead of 0.56 the call at half length 1024 (2000 x 19 rows, lmax 1000) with twice the lanes.
#define TC_CUBE_GAMMA(G) G(1024, 64) G(2048, 128) G(4096, 256) G(8192, 256)

int launch_cube_alpha(const CubeArgs& c, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    dim3 g1((c.nring_chunk + CA_J - 1) / CA_J, (c.lmax + 1 + CA_K - 1) / CA_K);
    const double2* C = reinterpret_cast<const double2*>(c.C);
    const Phase4* E = reinterpret_cast<const Phase4*>(c.phase);
    double2* P = reinterpret_cast<double2*>(c.P);
    if (c.nalpha <= 8)
        hipLaunchKernelGGL(k_cube_alpha<4>, g1, dim3(CA_NT), 0, s, c, C, E, P);
    else if (c.nalpha <= 16)
        hipLaunchKernelGGL(k_cube_alpha<8>, g1, dim3(CA_NT), 0, s, c, C, E, P);
    else
        hipLaunchKernelGGL(k_cube_alpha<16>, g1, dim3(CA_NT), 0, s, c, C, E, P);
    return (int)hipGetLastError();
}

int launch_cube_gamma(const CubeArgs& c, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    const int H = c.ngamma / 2;
    const size_t sh2 = sizeof(double2) * ((size_t)H + (H >> 4) + 1);
    const int rows = c.nring_chunk * c.nalpha;
#define G(hmax, nt)                                                                                       \
    if (H <= hmax) {                                                                                      \
        hipLaunchKernelGGL((k_cube_gamma<hmax, nt>), dim3(rows), dim3(nt), sh2, s, c);                    \
        return (int)hipGetLastError();                                                                    \
    }
    TC_CUBE_GAMMA(G)
#undef G
    return (int)hipErrorInvalidValue;
}

int cube_set_lds_limits()
{
    // the gamma pass needs up to (8192 + 512 + 1) * 16 bytes of LDS
    int rc = 0;
#define G(hmax, nt)                                                                                          \
    if (!rc)                                                                                                 \
        rc = (int)hipFuncSetAttribute((const void*)k_cube_gamma<hmax, nt>, hipFuncAttributeMaxDynamicSharedMemorySize, \
                                      (hmax + hmax / 16 + 1) * (int)sizeof(double2));
    TC_CUBE_GAMMA(G)
#undef G
    return rc;
}

}  // namespace tc
