// Host side of libtotalconv: argument checks, the small per-call tables
// (built in x87 long double and stored as double or double-double), the
// workspace layout and the extern "C" entry points declared in totalconv.h.
//
// Tables (Sec. 4.2.2 of Prezeau & Reinecke, "compute just once"):
//   rings      : from colatitudes beta_j, x_j = cos(beta_j) in long double rounded once, with
//                rings j and nring-1-j made exact mirrors when beta_j + beta_{nring-1-j} is pi
//                to within 2^-48 (see tc_rings_from_beta)
//   per ring  j: x_j, ln cos(beta_j/2), ln sin(beta_j/2)
//   per column : ln A = ln sqrt((2 l0)! / ((l0+m)! (l0-m)!)), the seed normalisation
//                of Sec. 3.2 eq. logstart, with ln n! from lgammal
//   ring slots : mirror pairs (j, nring-1-j) with x exactly negated, then the rest
//   column list: every (mb, msky) column, longest chains (smallest l0) first
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <list>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/totalconv.h"
#include "tc_internal.h"

namespace {

thread_local std::string g_error;

int fail(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_error = buf;
    return code;
}

int hip_fail(int rc, const char* what)
{
    return fail(TC_EHIP, "%s: %s", what, hipGetErrorString((hipError_t)rc));
}

constexpr size_t kAlign = 256;

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Whether two arrays of `bytes` share memory.
bool overlap(const void* p, const void* q, size_t bytes)
{
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = reinterpret_cast<uintptr_t>(q);
    return a < b ? b - a < bytes : a - b < bytes;
}

typedef long double ld;

void split_dd(ld v, double& hi, double& lo)
{
    hi = (double)v;
    lo = std::isinf(hi) ? 0.0 : (double)(v - (ld)hi);
}

constexpr long double kPiL = 3.14159265358979323846264338327950288L;
// Rings j and nring-1-j whose colatitudes add up to pi within this bound are taken as an
// exact mirror pair (a grid symmetric about the equator, rounded to doubles).
constexpr long double kMirrorTol = 0x1p-48L;

// cos(b) for b in [0, pi] as a double-double, from cos and sin at the nearest k / 32 (long double, as
// double pairs) and the Taylor series of the exact remainder |r| <= 1/64, to within 2^-63; x is the high
// word.  Returns whether x is certain to be what the long double cosine, itself within 2^-63, rounds
// to: the low word then stays 2^-61 clear of the half ulp where the rounding changes.  (2.5% of the
// colatitudes of a grid are not certain; 20 ns where cosl takes 100 to 130.)
__attribute__((target("fma"))) bool cos_certain(double b, double& x)
{
    struct Table {
        double ch[104], cl[104], sh[104], sl[104];
        Table()
        {
            for (int k = 0; k < 104; ++k) {
                const ld c = cosl((ld)k / 32), s = sinl((ld)k / 32);
                ch[k] = (double)c; cl[k] = (double)(c - (ld)ch[k]);
                sh[k] = (double)s; sl[k] = (double)(s - (ld)sh[k]);
            }
        }
    };
    static const Table t;
    const int k = (int)(b * 32.0 + 0.5);
    const double r = b - k * (1.0 / 32);                      // exact
    const double C = t.ch[k], S = t.sh[k];
    const double p = r * r, e = __builtin_fma(r, r, -p);      // r^2
    const double q = p * p * (1.0 / 24 + p * (-1.0 / 720 + p * (1.0 / 40320 + p * (-1.0 / 3628800))));   // cos r - 1 + r^2 / 2
    const double s = r * p * (-1.0 / 6 + p * (1.0 / 120 + p * (-1.0 / 5040 + p * (1.0 / 362880))));      // sin r - r
    const double B = -S * r, Bl = -__builtin_fma(S, r, B);
    const double hp = -0.5 * p, D = C * hp, Dl = __builtin_fma(C, hp, -D);
    const double h1 = C + B, b1 = h1 - C, e1 = (C - (h1 - b1)) + (B - b1);
    const double h2 = h1 + D, b2 = h2 - h1, e2 = (h1 - (h2 - b2)) + (D - b2);
    const double lo = e1 + e2 + (Bl + Dl) + (t.cl[k] - t.sl[k] * r + t.cl[k] * hp) + (C * (q - 0.5 * e) - S * s);
    const double h = h2 + lo, l = lo - (h - h2);
    x = h;
    uint64_t bits;
    std::memcpy(&bits, &h, sizeof bits);
    const uint64_t expo = bits & 0x7ff0000000000000ull;
    if ((bits & 0x000fffffffffffffull) == 0 || expo <= (uint64_t)54 << 52) return false;   // a power of two, or tiny
    const uint64_t half_bits = expo - ((uint64_t)53 << 52);
    double half;                                              // half an ulp of h
    std::memcpy(&half, &half_bits, sizeof half);
    return half - std::fabs(l) > 0x1p-61;
}

// The cosine in long double, rounded once to double.
double ring_cosine(double b)
{
    static const bool has_fma = __builtin_cpu_supports("fma");
    double x;
    return has_fma && cos_certain(b, x) ? x : (double)cosl((ld)b);
}

// x_j = cos(beta_j) in long double rounded once to double; then for each j < k = nring-1-j
// with |beta_j + beta_k - pi| <= 2^-48 the ring with the larger colatitude is set to the
// exact negative of the other's x (the pi - beta symmetry of Sec. 4.2.3 then holds exactly).
int rings_from_beta(int nring, const double* beta, std::vector<double>& x)
{
    if (nring < 1) return fail(TC_EINVAL, "nring must be >= 1 (got %d)", nring);
    if (!beta) return fail(TC_EINVAL, "beta is NULL");
    const double pi_d = (double)kPiL;   // the largest double not above pi
    for (int j = 0; j < nring; ++j)
        if (!(beta[j] >= 0.0 && beta[j] <= pi_d))
            return fail(TC_EINVAL, "beta[%d] = %.17g is not a colatitude in [0, pi]", j, beta[j]);
    x.resize(nring);
    for (int j = 0; j < (nring + 1) / 2; ++j) {
        const int k = nring - 1 - j;
        if (j < k && fabsl((long double)beta[j] + (long double)beta[k] - kPiL) <= kMirrorTol) {
            if (beta[j] <= beta[k]) { x[j] = ring_cosine(beta[j]); x[k] = -x[j]; }
            else { x[k] = ring_cosine(beta[k]); x[j] = -x[k]; }
        } else {
            x[j] = ring_cosine(beta[j]);
            if (k != j) x[k] = ring_cosine(beta[k]);
        }
    }
    return TC_OK;
}

// ---------------------------------------------------------------- tile choice

constexpr int kNumOps = 6;   // TC_OP_WIGNER, TC_OP_FWD, TC_OP_ADJ, TC_OP_FWD_POL, TC_OP_CUBE, TC_OP_MATRIX
tc::Tile g_tile_override[kNumOps] = {{0, 256, 0, 0}, {0, 256, 0, 0}, {0, 256, 0, 0}, {0, 256, 0, 0}, {0, 256, 0, 0}, {0, 256, 0, 0}};   // 0 = built-in

int g_matrix_R = 0;   // rows per lane of wigner_d_matrix (tc_set_tile); 0 = built-in

tc::Tile default_tile(int op, int lmax)
{
    // R of plans, TB of every call, and what tc_get_tile reports (plain calls take R by walk_cost).
    tc::Tile t{4, 256, 32, 4};
    if (op == TC_OP_FWD) t = lmax >= 256 ? tc::Tile{4, 256, 64, 4} : tc::Tile{2, 256, 32, 4};
    if (op == TC_OP_ADJ) t = lmax >= 256 ? tc::Tile{8, 256, 64, 4} : tc::Tile{2, 256, 32, 4};
    if (op == TC_OP_FWD_POL) t = lmax >= 256 ? tc::Tile{4, 256, 64, 4} : tc::Tile{2, 256, 32, 4};
    if (op >= 0 && op < kNumOps) {
        const tc::Tile& o = g_tile_override[op];
        if (o.R > 0) t.R = o.R;
        if (o.TB > 0) t.TB = o.TB;
        if (o.TR > 0) t.TR = o.TR;
    }
    return t;
}

int count_slots(int nring, const double* x)
{
    if (!x) return nring;   // size queries: at most nring slots
    int n = 0;
    for (int j = 0; j < nring; ++j) {
        const int jp = nring - 1 - j;
        if (j < jp && x[jp] == -x[j]) ++n;          // pair (j, jp)
        else if (j > jp && x[j] == -x[jp]) continue;  // partner of an earlier pair
        else ++n;                                   // single ring
    }
    return n;
}

// Cost of a walk over nslot ring slots with R chains per lane and NT lanes, in slots of a walk
// without overheads.  The terms, each fitted to timings over 65 to 4096 slots on MI355X:
//  - the slots of whole ring tiles (idle chains walk too);
//  - a lane's cost per chain and step: the forward reads a step's coefficients from LDS once for R
//    chains (R 2 is bound by it), the adjoint moves its sums once for R chains (6 + 8 / R operations);
//  - the wave is the unit of the skip test: 64 R slots leave the skipped range together, so wide
//    waves on few slots skip less;
//  - staging and the block sums, per block of NT steps, over the NT R chains that share them.
double walk_cost(int op, int R, int NT, int nslot)
{
    const bool adj = op == TC_OP_ADJ;
    const double step = adj ? 6.0 + 8.0 / R : 5.0;
    const double lane = adj ? step / 7.0 : (R >= 8 ? 1.0 : R >= 4 ? 1.01 : 1.15);
    const double skip = 1.0 + (adj ? 0.12 : 0.25) * 64.0 * R / nslot;
    const double stage = 1.0 + (adj ? 440.0 : 200.0) / (NT * R * step);
    const int ntile = (nslot + NT * R - 1) / (NT * R);
    return (double)ntile * NT * R * lane * skip * stage;
}

// The tile of a call over nslot ring slots: R as set or, at 0, the cheapest built one, with the
// cheapest number of lanes per workgroup for it.  The adjoint's smaller workgroups are built with TB 32: a TB 64
// that was set keeps 256 lanes.
tc::Tile fit_tile(int op, tc::Tile t, int nslot)
{
    const int R0 = t.R;
    double best = 0.0;
    for (int R : {8, 4, 2}) {
        if ((R0 > 0 && R != R0) || (op == TC_OP_FWD_POL && R > 4)) continue;
        for (int NT : {256, 128, 64}) {
            if (op == TC_OP_ADJ && NT < 256 && g_tile_override[op].TB > 32) continue;
            const double c = walk_cost(op, R, NT, nslot);
            if (best == 0.0 || c < best) { best = c; t.R = R; t.NT = NT; }
        }
    }
    if (op == TC_OP_ADJ && t.NT < 256) t.TB = 32;
    return t;
}

// The tile of a plain convolution call: the built-in choice goes by the call's ring slots.
tc::Tile call_tile(int op, int lmax, int nslot)
{
    tc::Tile t = default_tile(op, lmax);
    t.R = g_tile_override[op].R;
    return fit_tile(op, t, nslot);
}

// ------------------------------------------------------------ kernel timing

// Event pairs recorded around the recursion kernel of each call (tc_timing_*).
struct KernelTiming {
    int cap = 0;
    std::vector<hipEvent_t> start[kNumOps], stop[kNumOps];
    long long recorded[kNumOps] = {0, 0, 0, 0, 0, 0};
};
KernelTiming g_timing;

void timing_release()
{
    for (int op = 0; op < kNumOps; ++op) {
        for (hipEvent_t e : g_timing.start[op]) if (e) (void)hipEventDestroy(e);
        for (hipEvent_t e : g_timing.stop[op]) if (e) (void)hipEventDestroy(e);
        g_timing.start[op].clear();
        g_timing.stop[op].clear();
        g_timing.recorded[op] = 0;
    }
    g_timing.cap = 0;
}

// Launch `launch` between the op's next event pair (plain launch when timing is off).
template <class F>
int timed_launch(int op, void* stream, F launch)
{
    if (!g_timing.cap) return launch();
    const int i = (int)(g_timing.recorded[op] % g_timing.cap);
    int rc = (int)hipEventRecord(g_timing.start[op][i], (hipStream_t)stream);
    if (rc) return rc;
    if ((rc = launch())) return rc;
    if ((rc = (int)hipEventRecord(g_timing.stop[op][i], (hipStream_t)stream))) return rc;
    ++g_timing.recorded[op];
    return 0;
}

// ------------------------------------------------------------- table layout

struct Layout {
    size_t ring = 0, slots = 0, colmb = 0, colms = 0, lna = 0, tables_end = 0;
    size_t U = 0, V = 0, sym = 0, total = 0;
    int nslot = 0, ncol = 0, ntile = 0;
    long long P = 0;
};

Layout make_layout(int op, int lmax, int mbmax_or_npair, int nring, const double* x, tc::Tile t)
{
    Layout L;
    const bool conv = op != TC_OP_WIGNER;
    L.nslot = conv ? count_slots(nring, x) : nring;
    L.ncol = conv ? (2 * mbmax_or_npair + 1) * (lmax + 1) : mbmax_or_npair;
    L.ntile = (L.nslot + t.NT * t.R - 1) / (t.NT * t.R);
    size_t off = 0;
    L.ring = off;  off = align_up(off + sizeof(double) * 5 * (size_t)nring);
    L.slots = off; off = align_up(off + sizeof(int) * 2 * (size_t)L.nslot);
    L.colmb = off; off = align_up(off + sizeof(int) * (size_t)L.ncol);
    L.colms = off; off = align_up(off + sizeof(int) * (size_t)L.ncol);
    L.lna = off;   off = align_up(off + sizeof(double) * 2 * (size_t)L.ncol);
    L.tables_end = off;
    if (op == TC_OP_FWD || op == TC_OP_FWD_POL) {   // beam row signs, computed on the device
        L.sym = off; off = align_up(off + sizeof(int) * (size_t)(2 * mbmax_or_npair + 1));
    }
    if (op == TC_OP_ADJ) {   // one U and one V row per column, whatever the number of ring tiles
        L.P = (long long)(lmax + 1) * (lmax + 2) / 2;
        const size_t ubytes = (size_t)16 * (size_t)(2 * mbmax_or_npair + 1) * (size_t)L.P;
        L.U = off; off = align_up(off + ubytes);
        L.V = off; off = align_up(off + ubytes);
    }
    L.total = off;
    return L;
}

// Seed normalisation index m of column (mb, ms) at l0 = max(|mb|, |ms|).
int seed_m(int mb, int ms) { return std::abs(ms) >= std::abs(mb) ? mb : ms; }

ld ln_A(int mb, int ms)
{
    const int l0 = std::max(std::abs(mb), std::abs(ms));
    const int m = seed_m(mb, ms);
    return 0.5L * (lgammal((ld)(2 * l0 + 1)) - lgammal((ld)(l0 + m + 1)) - lgammal((ld)(l0 - m + 1)));
}

// Fill the table part of the workspace image.
void build_rings(int nring, const double* x, std::vector<char>& img, const Layout& L)
{
    double* r = reinterpret_cast<double*>(img.data() + L.ring);
    double *rx = r, *lch = r + nring, *lcl = r + 2 * nring, *lsh = r + 3 * nring, *lsl = r + 4 * nring;
    for (int j = 0; j < nring; ++j) {
        const ld X = (ld)x[j];
        const ld c2 = (1.0L + X) / 2.0L;   // cos^2(beta/2)
        const ld s2 = (1.0L - X) / 2.0L;   // sin^2(beta/2)
        ld lc, ls;
        if (c2 == 0.0L) lc = -INFINITY;
        else lc = 0.5L * (X > 0 ? log1pl(-s2) : logl(c2));
        if (s2 == 0.0L) ls = -INFINITY;
        else ls = 0.5L * (X < 0 ? log1pl(-c2) : logl(s2));
        rx[j] = x[j];
        split_dd(lc, lch[j], lcl[j]);
        split_dd(ls, lsh[j], lsl[j]);
    }
}

void build_slots(int nring, const double* x, std::vector<char>& img, const Layout& L)
{
    int* s = reinterpret_cast<int*>(img.data() + L.slots);
    int n = 0;
    std::vector<int> single;
    for (int j = 0; j < nring; ++j) {
        const int jp = nring - 1 - j;
        if (j < jp && x[jp] == -x[j]) { s[2 * n] = j; s[2 * n + 1] = jp; ++n; }
        else if (j > jp && x[j] == -x[jp]) continue;
        else single.push_back(j);
    }
    for (int j : single) { s[2 * n] = j; s[2 * n + 1] = -1; ++n; }
}

void build_columns(int lmax, int mbmax, std::vector<char>& img, const Layout& L)
{
    struct Col { int mb, ms, l0; };
    std::vector<Col> cols;
    cols.reserve(L.ncol);
    for (int mb = -mbmax; mb <= mbmax; ++mb)
        for (int ms = 0; ms <= lmax; ++ms)
            cols.push_back({mb, ms, std::max(std::abs(mb), ms)});
    std::stable_sort(cols.begin(), cols.end(), [](const Col& a, const Col& b) { return a.l0 < b.l0; });
    int* cmb = reinterpret_cast<int*>(img.data() + L.colmb);
    int* cms = reinterpret_cast<int*>(img.data() + L.colms);
    double* lna = reinterpret_cast<double*>(img.data() + L.lna);
    for (int i = 0; i < L.ncol; ++i) {
        cmb[i] = cols[i].mb;
        cms[i] = cols[i].ms;
        split_dd(ln_A(cols[i].mb, cols[i].ms), lna[2 * i], lna[2 * i + 1]);
    }
}

void build_pairs(int npair, const int* mb, const int* ms, std::vector<char>& img, const Layout& L)
{
    int* cmb = reinterpret_cast<int*>(img.data() + L.colmb);
    int* cms = reinterpret_cast<int*>(img.data() + L.colms);
    double* lna = reinterpret_cast<double*>(img.data() + L.lna);
    for (int i = 0; i < npair; ++i) {
        cmb[i] = mb[i];
        cms[i] = ms[i];
        split_dd(ln_A(mb[i], ms[i]), lna[2 * i], lna[2 * i + 1]);
    }
}

int check_rings(int nring, const double* x)
{
    if (nring < 1) return fail(TC_EINVAL, "nring must be >= 1 (got %d)", nring);
    if (!x) return fail(TC_EINVAL, "cosbeta is NULL");
    for (int j = 0; j < nring; ++j)
        if (!(x[j] >= -1.0 && x[j] <= 1.0))
            return fail(TC_EINVAL, "cosbeta[%d] = %g is not a ring cosine in [-1, 1]", j, x[j]);
    return TC_OK;
}

int check_sizes(int lmax, int mbmax)
{
    if (lmax < 0 || lmax > TC_LMAX_LIMIT)
        return fail(TC_EINVAL, "lmax = %d outside [0, %d]", lmax, TC_LMAX_LIMIT);
    if (mbmax < 0 || mbmax > lmax)
        return fail(TC_EINVAL, "mbmax = %d outside [0, lmax = %d]", mbmax, lmax);
    return TC_OK;
}

int check_ws(const Layout& L, void* ws, size_t ws_bytes)
{
    if (ws_bytes < L.total)
        return fail(TC_ENOMEM, "workspace of %zu bytes is smaller than the %zu bytes needed", ws_bytes, L.total);
    if (!ws) return fail(TC_EINVAL, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(ws) % kAlign)
        return fail(TC_EINVAL, "workspace must be %zu-byte aligned", kAlign);
    return TC_OK;
}

// Host images of the per-call tables, kept in pinned memory for repeated calls with the same
// (kind, sizes, tile, ring set, pair list) on the same device: a repeated call skips the long
// double prep and the column sort, and its upload is a kernel that reads the mapped image (launch_prep).
// Least recently used entries are dropped beyond kCacheEntries or kCacheBytes; the memory of an image is
// given back once nothing can read it: no graph that a call was captured into holds it, and the
// device has been waited for (any stream may have its upload queued).  The images never change once built.
struct HostImage {
    int dev = 0;
    void* pinned = nullptr;
    void* mapped = nullptr;         // `pinned` as the device sees it
    size_t bytes = 0;
};
typedef std::shared_ptr<HostImage> ImageRef;

struct TableImage {
    std::vector<int> head;          // kind, device, lmax, mbmax / npair, nring, R, NT, bytes
    std::vector<double> x;          // ring cosines
    std::vector<int> pairs;         // (mb, msky) pairs of wigner_d_rings
    ImageRef image;
};

constexpr size_t kCacheEntries = 64;
constexpr size_t kCacheBytes = (size_t)1 << 30;
std::recursive_mutex g_cache_mu;   // upload_tables calls upload
std::list<TableImage> g_cache;      // front: most recently used
std::vector<ImageRef> g_dropped;    // images out of the cache whose memory has not been given back yet

// What a graph holds of a captured call: a user object of the graph and of the executable graphs made from
// it, released with the last of them.  The release may come from any thread, inside any runtime call, and
// must call nothing of the runtime: it hands the hold to the next upload (reap_graph_holds).
struct GraphHold {
    ImageRef image;
    std::vector<char> bytes;        // pageable tables (upload)
    GraphHold* next = nullptr;
};
std::atomic<GraphHold*> g_released{nullptr};

void release_graph_hold(void* p)
{
    GraphHold* h = static_cast<GraphHold*>(p);
    h->next = g_released.load();
    while (!g_released.compare_exchange_weak(h->next, h)) {}
}

// The graph that `stream` is being captured into, or null.
hipGraph_t capturing_graph(void* stream)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    hipGraph_t g = nullptr;
    const hipGraphNode_t* deps = nullptr;
    size_t ndep = 0;
    if (hipStreamGetCaptureInfo_v2((hipStream_t)stream, &st, &id, &g, &deps, &ndep) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    return st == hipStreamCaptureStatusActive ? g : nullptr;
}

// The graph, and every executable graph made from it, keeps what `hold` owns (hipError_t value).
int hold_for_graph(hipGraph_t graph, std::unique_ptr<GraphHold> hold)
{
    hipUserObject_t u = nullptr;
    int rc = (int)hipUserObjectCreate(&u, hold.get(), release_graph_hold, 1, hipUserObjectNoDestructorSync);
    if (rc) return rc;
    (void)hold.release();           // the user object's from here on
    rc = (int)hipGraphRetainUserObject(graph, u, 1, hipGraphUserObjectMove);
    if (rc) (void)hipUserObjectRelease(u, 1);
    return rc;
}

// Drop a reference to an image; the last one leaves it to free_dropped.  Under g_cache_mu.
void drop_image(ImageRef& r)
{
    if (r && r.use_count() == 1) g_dropped.push_back(std::move(r));
    r.reset();
}

// Under g_cache_mu.
void reap_graph_holds()
{
    if (!g_released.load(std::memory_order_relaxed)) return;
    for (GraphHold* h = g_released.exchange(nullptr); h;) {
        GraphHold* next = h->next;
        drop_image(h->image);
        delete h;
        h = next;
    }
}

// Copy tables from pageable memory.  The copy has read them when hipMemcpyAsync returns, a captured one
// reads them on every replay.
int upload(void* ws, std::vector<char> img, void* stream)
{
    const hipGraph_t graph = capturing_graph(stream);
    int rc = (int)hipMemcpyAsync(ws, img.data(), img.size(), hipMemcpyHostToDevice, (hipStream_t)stream);
    if (!rc && graph) {
        std::lock_guard<std::recursive_mutex> lock(g_cache_mu);
        reap_graph_holds();
        std::unique_ptr<GraphHold> hold(new GraphHold);
        hold->bytes = std::move(img);
        rc = hold_for_graph(graph, std::move(hold));
    }
    return rc ? hip_fail(rc, "table upload (hipMemcpyAsync)") : TC_OK;
}

// Give the dropped images' memory back, each once its device has finished all that was enqueued; one whose
// device cannot be waited for stays for a later call.  Under g_cache_mu, not during a capture.
void free_dropped()
{
    if (g_dropped.empty()) return;
    int cur = 0, synced = -1;
    if (hipGetDevice(&cur) != hipSuccess) return;
    std::vector<ImageRef> keep;
    for (ImageRef& r : g_dropped) {
        if (synced != r->dev) {
            const bool ok = (r->dev == cur || hipSetDevice(r->dev) == hipSuccess) && hipDeviceSynchronize() == hipSuccess;
            if (r->dev != cur) (void)hipSetDevice(cur);
            if (!ok) { (void)hipGetLastError(); keep.push_back(std::move(r)); continue; }
            synced = r->dev;
        }
        (void)hipHostFree(r->pinned);
    }
    g_dropped.swap(keep);
}

bool same_key(const TableImage& e, const std::vector<int>& head, int nring, const double* x, int npair,
              const int* mb, const int* ms)
{
    if (e.head != head || (int)e.x.size() != nring || (int)e.pairs.size() != 2 * npair) return false;
    if (nring && std::memcmp(e.x.data(), x, sizeof(double) * nring)) return false;
    for (int i = 0; i < npair; ++i)
        if (e.pairs[2 * i] != mb[i] || e.pairs[2 * i + 1] != ms[i]) return false;
    return true;
}

// The row signs of a call's beams (npair 0: none wanted).
int launch_signs(tc::PrepArgs signs, void* stream)
{
    if (signs.npair == 0) return TC_OK;
    signs.bytes = 0;
    const int rc = tc::launch_prep ? tc::launch_prep(signs, stream) : (int)hipErrorInvalidDeviceFunction;
    return rc ? hip_fail(rc, "beam symmetry launch") : TC_OK;
}

// Upload the table image for this call into the workspace, building it on a miss with
// build(img), and find the row signs of its beams.  kind: TC_OP_* of the layout.  For wigner_d_rings
// pass the pairs (else npair 0).
template <class Build>
int upload_tables(int kind, int lmax, int mbmax_or_npair, int nring, const double* x, int npair, const int* mb,
                  const int* ms, const Layout& L, tc::Tile t, void* ws, void* stream, Build build,
                  tc::PrepArgs signs = tc::PrepArgs{})
{
    int dev = 0;
    int rc = (int)hipGetDevice(&dev);
    if (rc) return hip_fail(rc, "table upload: hipGetDevice");
    const std::vector<int> head = {kind, dev, lmax, mbmax_or_npair, nring, t.R, t.NT, (int)L.tables_end};
    const hipGraph_t graph = capturing_graph(stream);
    std::lock_guard<std::recursive_mutex> lock(g_cache_mu);
    reap_graph_holds();
    auto it = g_cache.begin();
    for (; it != g_cache.end(); ++it)
        if (same_key(*it, head, nring, x, npair, mb, ms)) break;
    if (it == g_cache.end()) {
        std::vector<char> img(L.tables_end, 0);
        build(img);
        TableImage e;
        e.head = head;
        e.x.assign(x, x + nring);
        for (int i = 0; i < npair; ++i) { e.pairs.push_back(mb[i]); e.pairs.push_back(ms[i]); }
        e.image = std::make_shared<HostImage>();
        e.image->dev = dev;
        e.image->bytes = img.size();
        if (hipHostMalloc(&e.image->pinned, e.image->bytes, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();   // no pinned memory: upload from the pageable image, uncached
            rc = upload(ws, std::move(img), stream);
            return rc ? rc : launch_signs(signs, stream);
        }
        if (hipHostGetDevicePointer(&e.image->mapped, e.image->pinned, 0) != hipSuccess) {
            (void)hipGetLastError();
            e.image->mapped = nullptr;
        }
        std::memcpy(e.image->pinned, img.data(), img.size());
        g_cache.push_front(std::move(e));
        it = g_cache.begin();
        if (!graph) {   // during a capture nothing can be waited for: a later call drops entries
            size_t total = 0;
            for (const TableImage& c : g_cache) total += c.image->bytes;
            while (g_cache.size() > kCacheEntries || (g_cache.size() > 1 && total > kCacheBytes)) {
                total -= g_cache.back().image->bytes;
                drop_image(g_cache.back().image);
                g_cache.pop_back();
            }
            free_dropped();
        }
    } else if (it != g_cache.begin()) {
        g_cache.splice(g_cache.begin(), g_cache, it);
        it = g_cache.begin();
    }
    const HostImage& im = *it->image;
    if (tc::launch_prep && im.mapped) {
        signs.src = im.mapped; signs.dst = ws; signs.bytes = im.bytes;
        rc = tc::launch_prep(signs, stream);
        signs.npair = 0;
    } else {
        rc = (int)hipMemcpyAsync(ws, im.pinned, im.bytes, hipMemcpyHostToDevice, (hipStream_t)stream);
    }
    if (!rc && graph) {
        std::unique_ptr<GraphHold> hold(new GraphHold);
        hold->image = it->image;
        rc = hold_for_graph(graph, std::move(hold));
    }
    return rc ? hip_fail(rc, "table upload") : launch_signs(signs, stream);
}

tc::RingTables ring_ptrs(void* ws, const Layout& L, int nring)
{
    const double* r = reinterpret_cast<const double*>(static_cast<char*>(ws) + L.ring);
    return tc::RingTables{r, r + nring, r + 2 * nring, r + 3 * nring, r + 4 * nring};
}

tc::ColumnTables col_ptrs(void* ws, const Layout& L)
{
    char* b = static_cast<char*>(ws);
    return tc::ColumnTables{reinterpret_cast<const int*>(b + L.colmb), reinterpret_cast<const int*>(b + L.colms),
                            reinterpret_cast<const double*>(b + L.lna)};
}

int check_grid(const Layout& L)
{
    if ((long long)L.ncol * L.ntile > 0x7fffffffLL)
        return fail(TC_EUNSUPPORTED, "launch of %lld workgroups exceeds the grid limit", (long long)L.ncol * L.ntile);
    return TC_OK;
}

// Work items of one launch.  A launch packet counts them in 32 bits; the runtime refuses 2^32 and lets a larger
// product wrap (2^32 + 512 work items: no error, one workgroup of 512 runs), so larger calls take several launches.
constexpr long long kGridItems = 0xffffffffLL;

// The units (columns, pairs, rings, ...) one launch takes, each of `groups` workgroups of `lanes` lanes.
int per_launch(long long groups, int lanes)
{
    return (int)std::max(1LL, std::min(0x7fffffffLL, kGridItems / lanes / groups));
}

// Forward for npair (sky, beam) pairs: one output per pair, or (sum) one output.
int fwd_impl(int op, int lmax, int mbmax, int nring, const double* cosbeta, int npair, const double* const* alm,
             const double* const* blm, int sum, double* const* C, void* workspace, size_t ws_bytes, void* stream,
             bool cached = true)
{
    int rc = check_sizes(lmax, mbmax);
    if (rc || (rc = check_rings(nring, cosbeta))) return rc;
    const int nout = sum ? 1 : npair;
    for (int p = 0; p < npair; ++p) {
        if (!alm[p] || !blm[p]) return fail(TC_EINVAL, "alm or blm of pair %d is NULL", p);
        if (!aligned16(alm[p]) || !aligned16(blm[p])) return fail(TC_EINVAL, "complex arrays must be 16-byte aligned");
    }
    for (int c = 0; c < nout; ++c) {
        if (!C[c]) return fail(TC_EINVAL, "C of output %d is NULL", c);
        if (!aligned16(C[c])) return fail(TC_EINVAL, "complex arrays must be 16-byte aligned");
    }
    const tc::Tile t = call_tile(op, lmax, count_slots(nring, cosbeta));
    const Layout L = make_layout(op, lmax, mbmax, nring, cosbeta, t);
    if ((rc = check_ws(L, workspace, ws_bytes)) || (rc = check_grid(L))) return rc;
    auto build = [&](std::vector<char>& img) {
        build_rings(nring, cosbeta, img, L);
        build_slots(nring, cosbeta, img, L);
        build_columns(lmax, mbmax, img, L);
    };
    // columns whose beam rows are related by a sign take the even / odd sums (summed pairs have no use for it)
    tc::PrepArgs signs{};
    if (npair == 1 || !sum) {
        signs.npair = npair; signs.lmax = lmax; signs.mbmax = mbmax;
        for (int p = 0; p < npair; ++p) signs.blm[p] = blm[p];
        signs.sym = reinterpret_cast<int*>(static_cast<char*>(workspace) + L.sym);
    }
    if (cached) {
        rc = upload_tables(TC_OP_FWD, lmax, mbmax, nring, cosbeta, 0, nullptr, nullptr, L, t, workspace, stream, build,
                           signs);
    } else {   // no pinned image: built here and copied from pageable host memory
        std::vector<char> img(L.tables_end, 0);
        build(img);
        if (!(rc = upload(workspace, std::move(img), stream))) rc = launch_signs(signs, stream);
    }
    if (rc) return rc;
    tc::FwdArgs a{};
    a.lmax = lmax; a.mbmax = mbmax; a.nring = nring; a.nslot = L.nslot; a.ncol = L.ncol; a.ntile = L.ntile;
    a.sky_lmax = lmax;
    a.skip_exp = 100;
    a.ring = ring_ptrs(workspace, L, nring);
    a.slots = reinterpret_cast<const int*>(static_cast<char*>(workspace) + L.slots);
    a.col = col_ptrs(workspace, L);
    a.npair = npair;
    a.sum = sum;
    for (int p = 0; p < npair; ++p) { a.alm[p] = alm[p]; a.blm[p] = blm[p]; a.pmbmax[p] = mbmax; }
    for (int c = 0; c < nout; ++c) a.C[c] = C[c];
    a.beam_sym[0] = signs.sym;
    const tc::ColumnTables col = a.col;
    const int step = per_launch(L.ntile, t.NT);
    rc = timed_launch(op, stream, [&] {
        int r = 0;
        for (long long c0 = 0; c0 < L.ncol && !r; c0 += step) {
            a.ncol = (int)std::min<long long>(step, L.ncol - c0);
            a.col = tc::ColumnTables{col.mb + c0, col.ms + c0, col.lnA + 2 * c0};
            r = tc::launch_fwd(a, t, stream);
        }
        return r;
    });
    return rc ? hip_fail(rc, "totalconv_fwd launch") : TC_OK;
}

// Adjoint for npair pairs.  Summed outputs share one cotangent, hence one u per
// column and l; separate outputs have one cotangent each, reduced one after the other.
int adj_impl(int lmax, int mbmax, int nring, const double* cosbeta, int npair, const double* const* alm,
             const double* const* blm, int sum, const double* const* Cbar, double* const* alm_bar,
             double* const* blm_bar, void* workspace, size_t ws_bytes, void* stream)
{
    int rc = check_sizes(lmax, mbmax);
    if (rc || (rc = check_rings(nring, cosbeta))) return rc;
    const int ncot = sum ? 1 : npair;
    bool any = false;
    for (int p = 0; p < npair; ++p) {
        double* ab = alm_bar ? alm_bar[p] : nullptr;
        double* bb = blm_bar ? blm_bar[p] : nullptr;
        if (!alm[p] || !blm[p]) return fail(TC_EINVAL, "alm or blm of pair %d is NULL", p);
        if (!aligned16(alm[p]) || !aligned16(blm[p]) || (ab && !aligned16(ab)) || (bb && !aligned16(bb)))
            return fail(TC_EINVAL, "complex arrays must be 16-byte aligned");
        any |= (ab != nullptr) || (bb != nullptr);
    }
    for (int k = 0; k < ncot; ++k) {
        if (!Cbar[k]) return fail(TC_EINVAL, "Cbar of output %d is NULL", k);
        if (!aligned16(Cbar[k])) return fail(TC_EINVAL, "complex arrays must be 16-byte aligned");
    }
    if (!any) return TC_OK;   // nothing requested
    const tc::Tile t = call_tile(TC_OP_ADJ, lmax, count_slots(nring, cosbeta));
    const Layout L = make_layout(TC_OP_ADJ, lmax, mbmax, nring, cosbeta, t);
    if ((rc = check_ws(L, workspace, ws_bytes)) || (rc = check_grid(L))) return rc;
    // The sky gradient of one pair alone: with the row signs of its beam, a column whose rows are
    // related by one forms one sum instead of two.  The signs (2 mbmax + 1 ints) lie in front of V:
    // the first mbmax complex values of its row mb = -mbmax are those of l < mbmax at msky = 0, which
    // no column writes and no epilogue reads.
    int* const sym = reinterpret_cast<int*>(static_cast<char*>(workspace) + L.V);
    auto sky_alone = [&](int p0, int p1) {
        return p1 - p0 == 1 && mbmax >= 1 && alm_bar && alm_bar[p0] && !(blm_bar && blm_bar[p0]);
    };
    tc::PrepArgs signs{};
    if (sky_alone(0, npair)) {
        signs.npair = 1; signs.lmax = lmax; signs.mbmax = mbmax; signs.blm[0] = blm[0]; signs.sym = sym;
    }
    rc = upload_tables(TC_OP_FWD, lmax, mbmax, nring, cosbeta, 0, nullptr, nullptr, L, t, workspace, stream,
                       [&](std::vector<char>& img) {
                           build_rings(nring, cosbeta, img, L);
                           build_slots(nring, cosbeta, img, L);
                           build_columns(lmax, mbmax, img, L);
                       }, signs);
    if (rc) return rc;
    tc::AdjArgs a{};
    a.lmax = lmax; a.mbmax = mbmax; a.nring = nring; a.nslot = L.nslot; a.ncol = L.ncol; a.ntile = L.ntile;
    a.skip_exp = 100;
    a.ring = ring_ptrs(workspace, L, nring);
    a.slots = reinterpret_cast<const int*>(static_cast<char*>(workspace) + L.slots);
    a.col = col_ptrs(workspace, L);
    a.npair = 1;
    a.pmbmax[0] = mbmax;
    a.U[0] = reinterpret_cast<double*>(static_cast<char*>(workspace) + L.U);
    a.V[0] = reinterpret_cast<double*>(static_cast<char*>(workspace) + L.V);
    a.P = L.P;
    for (int k = 0; k < ncot; ++k) {
        const int p0 = sum ? 0 : k, p1 = sum ? npair : k + 1;   // pairs served by cotangent k
        bool need = false;
        for (int p = p0; p < p1; ++p)
            need |= (alm_bar && alm_bar[p]) || (blm_bar && blm_bar[p]);
        if (!need) continue;
        a.Cbar[0] = Cbar[k];
        a.beam_sym = nullptr;
        if (sky_alone(p0, p1)) {
            if (npair > 1 && (rc = tc::launch_beam_symmetry(blm[p0], lmax, mbmax, sym, stream)))   // V is reused
                return hip_fail(rc, "beam symmetry launch");
            a.beam_sym = sym;
        }
        // one workgroup per column walks its ring tiles in order: tile 0 writes U and V, later tiles add
        rc = timed_launch(TC_OP_ADJ, stream, [&] { return tc::launch_adj(a, t, stream); });
        if (rc) return hip_fail(rc, "totalconv_adj launch");
        // summed outputs: the pairs share this U, V, which one launch reads once for every
        // pair's sky gradient; the beam gradients take one launch per pair
        bool sky_shared = false;
        if (p1 - p0 > 1 && alm_bar) {
            tc::EpiPairsArgs e{};
            e.lmax = lmax; e.mbmax = mbmax; e.P = L.P; e.sky_lmax = lmax; e.npair = p1 - p0;
            e.U = a.U[0]; e.V = a.V[0];
            for (int p = p0; p < p1; ++p) {
                e.blm[p - p0] = blm[p];
                e.alm_bar[p - p0] = alm_bar[p];
                sky_shared |= alm_bar[p] != nullptr;
            }
            if (sky_shared && (rc = tc::launch_adj_sky_pairs(e, stream)))
                return hip_fail(rc, "totalconv_adj epilogue launch");
        }
        for (int p = p0; p < p1; ++p) {
            tc::EpiArgs e{};
            e.lmax = lmax; e.mbmax = mbmax; e.P = L.P; e.sky_lmax = lmax;
            e.U = a.U[0]; e.V = a.V[0]; e.alm = alm[p]; e.blm = blm[p];
            e.alm_bar = (alm_bar && !sky_shared) ? alm_bar[p] : nullptr;
            e.blm_bar = blm_bar ? blm_bar[p] : nullptr;
            e.beam_sym = a.beam_sym;
            // One launch forms both gradients side by side.  A gradient written over its input (blm_bar over
            // blm, which the sky gradient reads; alm_bar over alm, which the beam gradient reads) takes the
            // two one after the other, the sky gradient first.
            const size_t beam_bytes = (size_t)16 * (2 * mbmax + 1) * (lmax + 1), sky_bytes = (size_t)16 * L.P;
            if (e.alm_bar && e.blm_bar &&
                (overlap(e.blm_bar, e.blm, beam_bytes) || overlap(e.alm_bar, e.alm, sky_bytes))) {
                tc::EpiArgs sky = e;
                sky.blm_bar = nullptr;
                if ((rc = tc::launch_adj_epilogue(sky, stream))) return hip_fail(rc, "totalconv_adj epilogue launch");
                e.alm_bar = nullptr;
            }
            if ((rc = tc::launch_adj_epilogue(e, stream))) return hip_fail(rc, "totalconv_adj epilogue launch");
        }
    }
    return TC_OK;
}

// ------------------------------------------------------------- full matrix

struct MatrixLayout {
    size_t ring = 0, trig = 0, lna = 0, total = 0;
};

MatrixLayout make_matrix_layout(int l, int nring)
{
    MatrixLayout M;
    size_t off = 0;
    M.ring = off; off = align_up(off + sizeof(double) * 5 * (size_t)nring);
    M.trig = off; off = align_up(off + sizeof(double) * 2 * (size_t)nring);
    M.lna = off;  off = align_up(off + sizeof(double) * 2 * (size_t)(l + 1));
    M.total = off;
    return M;
}

// ---------------------------------------------------------------- data cube

// Alpha sums held at a time.  The alpha pass of a chunk of rings and its FFTs run one after the other on the
// call's stream: side by side (the FFTs of a chunk on a second stream, next to the alpha pass of the next) both
// passes, bound by memory alone, took no less together, and two buffers left chunks of half the size.  Larger
// chunks spend less on the ramps and tails of their launches: 2000 rings at lmax 2048 (1.9 GB of sums) take
// 1.99 ms by 500 rings, 1.89 ms at once; 4000 at lmax 4096 7.21 ms by 500 and 6.99 ms at once.  (Chunks that
// stay in the 256 MB last-level cache lose more to the ramps than the cache saves: 2.55 ms by 64 rings.)
constexpr size_t kCubeSumBytes = (size_t)2 << 30;
constexpr size_t kCubeOldSumBytes = (size_t)768 << 20;

struct CubeLayout {
    size_t phase = 0, tw = 0, P = 0, total = 0;
    int chunk = 0;        // rings per chunk
    int prow = 0;         // row stride of P (complex)
};

int g_cube_chunk = 0;   // rings per chunk of the data cube (tc_set_tile); 0 = built-in

// P in bytes of at most `bytes`, its rows of `prow` entries, `buffers` chunks of it.
CubeLayout cube_layout(int mbmax, int nring, int nalpha, int ngamma, int prow, size_t bytes, int buffers)
{
    CubeLayout C;
    C.prow = prow;
    const size_t per_ring = (size_t)16 * (size_t)nalpha * (size_t)prow;
    size_t chunk = std::max<size_t>(1, bytes / per_ring);
    if (chunk >= 16) chunk = chunk / 16 * 16;   // whole 16-ring tiles of the alpha pass
    if (g_cube_chunk > 0) chunk = (size_t)g_cube_chunk;
    else if (buffers == 1 && chunk >= 16 && (size_t)nring > chunk) {   // chunks of equal size
        const size_t n = ((size_t)nring + chunk - 1) / chunk;
        chunk = (((size_t)nring + n - 1) / n + 15) / 16 * 16;
    }
    C.chunk = (int)std::min<size_t>((size_t)nring, chunk);
    size_t off = 0;
    C.phase = off; off = align_up(off + (size_t)16 * ((nalpha + 3) / 4 * 4) * (2 * mbmax + 1));   // half is used
    C.tw = off;    off = align_up(off + (size_t)16 * ngamma);
    C.P = off;     off += (size_t)buffers * align_up(per_ring * (size_t)C.chunk);
    C.total = off;
    return C;
}

// Rows of P padded to whole 128-byte lines: a store that ends inside a line is written as two partial ones.
CubeLayout make_cube_layout(int lmax, int mbmax, int nring, int nalpha, int ngamma)
{
    return cube_layout(mbmax, nring, nalpha, ngamma, (lmax + 8) / 8 * 8, kCubeSumBytes, 1);
}

// The layout of a workspace of ws bytes.  One too small for make_cube_layout's, but of the size that was asked
// for when two chunks of 768 MB were held, unpadded, takes such chunks.
CubeLayout fit_cube_layout(int lmax, int mbmax, int nring, int nalpha, int ngamma, size_t ws)
{
    const CubeLayout C = make_cube_layout(lmax, mbmax, nring, nalpha, ngamma);
    const CubeLayout old = cube_layout(mbmax, nring, nalpha, ngamma, lmax + 1, kCubeOldSumBytes, 2);
    return ws < C.total && ws >= old.total ? old : C;
}

int check_cube(int lmax, int mbmax, int nring, int nalpha, int ngamma)
{
    if (lmax < 0 || lmax > 8192) return fail(TC_EINVAL, "data cube: lmax = %d outside [0, 8192]", lmax);
    if (mbmax < 0 || mbmax > lmax) return fail(TC_EINVAL, "data cube: mbmax = %d outside [0, lmax]", mbmax);
    if (nring < 1) return fail(TC_EINVAL, "data cube: nring must be >= 1");
    if (nalpha < 1 || (long long)nalpha * (2 * mbmax + 1) > 4096)
        return fail(TC_EINVAL, "data cube: nalpha = %d must be >= 1 with nalpha*(2*mbmax+1) <= 4096", nalpha);
    if (ngamma < 2 || ngamma > 16384 || (ngamma & (ngamma - 1)) || ngamma < 2 * lmax)
        return fail(TC_EINVAL, "data cube: ngamma = %d must be a power of two in [max(2, 2*lmax), 16384]", ngamma);
    return TC_OK;
}

}  // namespace

extern "C" {

size_t wigner_d_matrix_workspace_bytes(int l, int nring)
{
    if (l < 0 || l > TC_LMAX_LIMIT || nring < 1) return 0;
    return make_matrix_layout(l, nring).total;
}

int wigner_d_matrix_x(int l, int nring, const double* cosbeta, double* d, void* workspace, size_t ws_bytes,
                    void* stream)
{
    g_error.clear();
    if (l < 0 || l > TC_LMAX_LIMIT) return fail(TC_EINVAL, "l = %d outside [0, %d]", l, TC_LMAX_LIMIT);
    int rc = check_rings(nring, cosbeta);
    if (rc) return rc;
    if (!d) return fail(TC_EINVAL, "d is NULL");
    if (reinterpret_cast<uintptr_t>(d) % 8) return fail(TC_EINVAL, "d must be 8-byte aligned");
    const MatrixLayout M = make_matrix_layout(l, nring);
    if (ws_bytes < M.total)
        return fail(TC_ENOMEM, "workspace of %zu bytes is smaller than the %zu bytes needed", ws_bytes, M.total);
    if (!workspace) return fail(TC_EINVAL, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign)
        return fail(TC_EINVAL, "workspace must be %zu-byte aligned", kAlign);
    const int R = g_matrix_R;   // 0: the built-in variant
    const int rows = tc::matrix_rows_per_group(R);
    const int ntile = (l + 1 + rows - 1) / rows;
    if ((long long)ntile * 2 * nring > 0x7fffffffLL)
        return fail(TC_EUNSUPPORTED, "launch of %lld workgroups exceeds the grid limit", (long long)ntile * 2 * nring);
    std::vector<char> img(M.total, 0);
    Layout RL;
    RL.ring = M.ring;
    build_rings(nring, cosbeta, img, RL);
    double* trig = reinterpret_cast<double*>(img.data() + M.trig);
    for (int j = 0; j < nring; ++j) {   // cot and csc of beta from x in long double
        const ld X = (ld)cosbeta[j];
        const ld sn = sqrtl((1.0L - X) * (1.0L + X));
        trig[2 * j] = sn > 0 ? (double)(X / sn) : 0.0;
        trig[2 * j + 1] = sn > 0 ? (double)(1.0L / sn) : 0.0;
    }
    double* lna = reinterpret_cast<double*>(img.data() + M.lna);
    for (int m = 0; m <= l; ++m) {      // ln sqrt((2l)! / ((l+m)! (l-m)!))
        const ld v = 0.5L * (lgammal((ld)(2 * l + 1)) - lgammal((ld)(l + m + 1)) - lgammal((ld)(l - m + 1)));
        split_dd(v, lna[2 * m], lna[2 * m + 1]);
    }
    if ((rc = upload(workspace, std::move(img), stream))) return rc;
    tc::MatrixArgs a{};
    a.l = l; a.nring = nring; a.ntile = ntile;
    a.ring = ring_ptrs(workspace, RL, nring);
    a.trig = reinterpret_cast<const double*>(static_cast<char*>(workspace) + M.trig);
    a.lnA = reinterpret_cast<const double*>(static_cast<char*>(workspace) + M.lna);
    a.d = d;
    const tc::MatrixArgs all = a;
    const int step = per_launch(2LL * ntile, tc::kMatrixLanes);
    rc = timed_launch(TC_OP_MATRIX, stream, [&] {
        int r = 0;
        for (long long j0 = 0; j0 < nring && !r; j0 += step) {
            a.nring = (int)std::min<long long>(step, nring - j0);
            a.ring = tc::RingTables{all.ring.x + j0, all.ring.lch + j0, all.ring.lcl + j0, all.ring.lsh + j0, all.ring.lsl + j0};
            a.trig = all.trig + 2 * j0;
            a.d = all.d + j0 * (2LL * l + 1) * (2LL * l + 1);
            r = tc::launch_matrix(a, R, stream);
        }
        return r;
    });
    return rc ? hip_fail(rc, "wigner_d_matrix launch") : TC_OK;
}

size_t totalconv_datacube_workspace_bytes(int lmax, int mbmax, int nring, int nalpha, int ngamma)
{
    const std::string saved = g_error;
    const int rc = check_cube(lmax, mbmax, nring, nalpha, ngamma);
    g_error = saved;
    return rc ? 0 : make_cube_layout(lmax, mbmax, nring, nalpha, ngamma).total;
}

int totalconv_datacube_ring_chunk(int lmax, int mbmax, int nring, int nalpha, int ngamma)
{
    const std::string saved = g_error;
    const int rc = check_cube(lmax, mbmax, nring, nalpha, ngamma);
    g_error = saved;
    return rc ? 0 : make_cube_layout(lmax, mbmax, nring, nalpha, ngamma).chunk;
}

int totalconv_datacube(int lmax, int mbmax, int nring, const double* C, int nalpha, int ngamma, double* cube,
                       void* workspace, size_t ws_bytes, void* stream)
{
    g_error.clear();
    int rc = check_cube(lmax, mbmax, nring, nalpha, ngamma);
    if (rc) return rc;
    if (!C || !cube) return fail(TC_EINVAL, "C or cube is NULL");
    if (!aligned16(C) || !aligned16(cube)) return fail(TC_EINVAL, "C and cube must be 16-byte aligned");
    const CubeLayout CL = fit_cube_layout(lmax, mbmax, nring, nalpha, ngamma, ws_bytes);
    if (ws_bytes < CL.total)
        return fail(TC_ENOMEM, "workspace of %zu bytes is smaller than the %zu bytes needed", ws_bytes, CL.total);
    if (!workspace) return fail(TC_EINVAL, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign)
        return fail(TC_EINVAL, "workspace must be %zu-byte aligned", kAlign);
    int dev = 0, lds_max = 0;
    if ((rc = (int)hipGetDevice(&dev)) ||
        (rc = (int)hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev)))
        return hip_fail(rc, "data cube: device query");
    (void)tc::cube_set_lds_limits();   // opt-in beyond 64 KB where the runtime asks for it
    // LDS per workgroup: the FFT row (padded); the alpha pass uses a fixed 34 KB tile
    const size_t need = (size_t)16 * (ngamma / 2 + ngamma / 32 + 1);
    if (need > (size_t)lds_max)
        return fail(TC_EUNSUPPORTED, "data cube needs %zu bytes of LDS per workgroup, the device allows %d", need,
                    lds_max);
    // tables: (cos, sin)(2 pi m q / nalpha) ([m][slot q], rows padded with zeros to whole groups of 4; slot 0,
    // alphas 0 and nalpha / 2: 1 for the sum that m belongs to) and e^{-2 pi i m / ngamma}, in long double,
    // rounded once
    std::vector<char> img(CL.P, 0);
    double* ph = reinterpret_cast<double*>(img.data() + CL.phase);
    const int nslot = (nalpha + 1) / 2;
    for (int m = 0; m <= mbmax; ++m) {
        double* row = ph + 2 * (size_t)m * ((nslot + 3) / 4 * 4);
        row[m & 1] = 1.0;
        for (int q = 1; q < nslot; ++q) {
            const ld ang = 2.0L * kPiL * (ld)((long long)m * q % nalpha) / (ld)nalpha;
            row[2 * q] = (double)cosl(ang);
            row[2 * q + 1] = (double)sinl(ang);
        }
    }
    double* tw = reinterpret_cast<double*>(img.data() + CL.tw);
    for (int m = 0; m < ngamma; ++m) {
        const ld ang = 2.0L * kPiL * (ld)m / (ld)ngamma;
        tw[2 * m] = (double)cosl(ang);
        tw[2 * m + 1] = (double)-sinl(ang);
    }
    if ((rc = upload(workspace, std::move(img), stream))) return rc;
    tc::CubeArgs c{};
    c.lmax = lmax; c.mbmax = mbmax; c.nring = nring; c.nalpha = nalpha; c.ngamma = ngamma;
    c.C = C;
    c.phase = reinterpret_cast<const double*>(static_cast<char*>(workspace) + CL.phase);
    c.tw = reinterpret_cast<const double*>(static_cast<char*>(workspace) + CL.tw);
    c.cube = cube;
    c.prow = CL.prow;
    if ((long long)CL.chunk * nalpha > 0x7fffffffLL) return fail(TC_EUNSUPPORTED, "data cube: too many rows in one launch");
    c.P = reinterpret_cast<double*>(static_cast<char*>(workspace) + CL.P);
    const int step = std::min(CL.chunk, per_launch(nalpha, 256));   // a gamma workgroup per row, of up to 256 lanes
    rc = timed_launch(TC_OP_CUBE, stream, [&] {
        int r = 0;
        for (long long j0 = 0; j0 < nring && !r; j0 += step) {
            c.ring0 = (int)j0;
            c.nring_chunk = (int)std::min<long long>(step, nring - j0);
            r = tc::launch_cube_alpha(c, stream);
            if (!r) r = tc::launch_cube_gamma(c, stream);
        }
        return r;
    });
    return rc ? hip_fail(rc, "totalconv_datacube launch") : TC_OK;
}

}  // extern "C"

extern "C" {

const char* tc_last_error(void) { return g_error.c_str(); }

int tc_set_tile_ex(int op, int R, int TB, int TR)
{
    if (op < 0 || op >= kNumOps) return fail(TC_EINVAL, "tc_set_tile: unknown op %d", op);
    if (R < 0 || TB < 0 || TR < 0) return fail(TC_EINVAL, "tc_set_tile: negative tile parameter");
    if (op == TC_OP_MATRIX) {
        if (R > 2 || (TB && TB != 32) || (TR && TR != 4))
            return fail(TC_EINVAL, "tc_set_tile: (R %d, TB %d, TR %d) is not built for op %d", R, TB, TR, op);
        g_matrix_R = R;
        return TC_OK;
    }
    if (op == TC_OP_CUBE) {   // R: largest ring chunk of the data cube
        if (TB || TR) return fail(TC_EINVAL, "tc_set_tile: the data cube takes a ring chunk only");
        g_cube_chunk = R;
        return TC_OK;
    }
    const tc::Tile o = g_tile_override[op];
    g_tile_override[op] = tc::Tile{R, 256, TB, TR};
    if (!tc::tile_supported(op, default_tile(op, 1 << 20))) {
        g_tile_override[op] = o;
        return fail(TC_EINVAL, "tc_set_tile: (R %d, TB %d, TR %d) is not built for op %d", R, TB, TR, op);
    }
    return TC_OK;
}

int tc_set_tile(int op, int R)
{
    if (op < 0 || op >= kNumOps) return fail(TC_EINVAL, "tc_set_tile: unknown op %d", op);
    const tc::Tile o = g_tile_override[op];
    return tc_set_tile_ex(op, R, o.TB, o.TR);
}

int tc_get_tile(int op, int lmax)
{
    if (op < 0 || op >= kNumOps) return 0;
    if (op == TC_OP_CUBE) return g_cube_chunk;
    if (op == TC_OP_MATRIX) return g_matrix_R > 0 ? g_matrix_R : 1;
    return default_tile(op, lmax).R;
}

int tc_get_tile_ex(int op, int lmax, int* R, int* TB, int* TR)
{
    if (op < 0 || op >= kNumOps || !R || !TB || !TR) return fail(TC_EINVAL, "tc_get_tile_ex: bad arguments");
    const tc::Tile t = default_tile(op, lmax);
    *R = op == TC_OP_MATRIX ? (g_matrix_R > 0 ? g_matrix_R : 1) : t.R;
    *TB = op == TC_OP_MATRIX ? 32 : t.TB;
    *TR = t.TR;
    return TC_OK;
}

int tc_abi_version(void) { return 2; }

int tc_timing_enable(int n)
{
    if (n < 0 || n > 65536) return fail(TC_EINVAL, "tc_timing_enable: n = %d outside [0, 65536]", n);
    timing_release();
    if (n == 0) return TC_OK;
    for (int op = 0; op < kNumOps; ++op) {
        g_timing.start[op].assign(n, nullptr);
        g_timing.stop[op].assign(n, nullptr);
        for (int i = 0; i < n; ++i) {
            int rc = (int)hipEventCreate(&g_timing.start[op][i]);
            if (!rc) rc = (int)hipEventCreate(&g_timing.stop[op][i]);
            if (rc) {
                timing_release();
                return hip_fail(rc, "tc_timing_enable: hipEventCreate");
            }
        }
    }
    g_timing.cap = n;
    return TC_OK;
}

int tc_timing_read(int op, float* ms, int n)
{
    if (op < 0 || op >= kNumOps) return fail(TC_EINVAL, "tc_timing_read: unknown op %d", op);
    if (n < 0 || (n > 0 && !ms)) return fail(TC_EINVAL, "tc_timing_read: bad output buffer");
    if (!g_timing.cap) return 0;
    const long long rec = g_timing.recorded[op];
    const int k = (int)std::min<long long>(std::min<long long>(n, rec), g_timing.cap);
    for (int t = 0; t < k; ++t) {
        const int i = (int)((rec - k + t) % g_timing.cap);
        int rc = (int)hipEventSynchronize(g_timing.stop[op][i]);
        if (!rc) rc = (int)hipEventElapsedTime(&ms[t], g_timing.start[op][i], g_timing.stop[op][i]);
        if (rc) return hip_fail(rc, "tc_timing_read");
    }
    return k;
}

size_t totalconv_workspace_bytes(int op, int lmax, int mbmax, int nring)
{
    if (nring < 1 || lmax < 0 || lmax > TC_LMAX_LIMIT) return 0;
    if (op == TC_OP_WIGNER) {
        if (mbmax < 1) return 0;
    } else if (op == TC_OP_FWD || op == TC_OP_ADJ || op == TC_OP_FWD_POL) {
        if (mbmax < 0 || mbmax > lmax) return 0;
    } else {
        return 0;
    }
    return make_layout(op, lmax, mbmax, nring, nullptr, default_tile(op, lmax)).total;
}

size_t totalconv_workspace_bytes_rings_x(int op, int lmax, int mbmax, int nring, const double* cosbeta)
{
    if (!cosbeta || totalconv_workspace_bytes(op, lmax, mbmax, nring) == 0) return 0;
    for (int j = 0; j < nring; ++j)
        if (!(cosbeta[j] >= -1.0 && cosbeta[j] <= 1.0)) return 0;
    return make_layout(op, lmax, mbmax, nring, cosbeta, default_tile(op, lmax)).total;
}

int wigner_d_rings_x(int lmax, int npair, const int* mb, const int* msky, int nring, const double* cosbeta,
                   double* d, void* workspace, size_t ws_bytes, void* stream)
{
    g_error.clear();
    if (lmax < 0 || lmax > TC_LMAX_LIMIT) return fail(TC_EINVAL, "lmax = %d outside [0, %d]", lmax, TC_LMAX_LIMIT);
    if (npair < 1) return fail(TC_EINVAL, "npair must be >= 1 (got %d)", npair);
    if (!mb || !msky) return fail(TC_EINVAL, "mb / msky is NULL");
    for (int i = 0; i < npair; ++i)
        if (std::abs(mb[i]) > lmax || std::abs(msky[i]) > lmax)
            return fail(TC_EINVAL, "pair %d: |mb| = %d or |msky| = %d exceeds lmax = %d", i, std::abs(mb[i]),
                        std::abs(msky[i]), lmax);
    int rc = check_rings(nring, cosbeta);
    if (rc) return rc;
    if (!d) return fail(TC_EINVAL, "d is NULL");
    tc::Tile t = default_tile(TC_OP_WIGNER, lmax);
    t.R = 1; t.NT = 128;   // the one built shape: a ring per lane
    const Layout L = make_layout(TC_OP_WIGNER, lmax, npair, nring, cosbeta, t);
    if ((rc = check_ws(L, workspace, ws_bytes)) || (rc = check_grid(L))) return rc;
    rc = upload_tables(TC_OP_WIGNER, lmax, npair, nring, cosbeta, npair, mb, msky, L, t, workspace, stream,
                       [&](std::vector<char>& img) {
                           build_rings(nring, cosbeta, img, L);
                           build_pairs(npair, mb, msky, img, L);
                       });
    if (rc) return rc;
    tc::WignerArgs a{};
    a.lmax = lmax; a.npair = npair; a.nring = nring; a.ntile = L.ntile;
    a.ring = ring_ptrs(workspace, L, nring);
    a.col = col_ptrs(workspace, L);
    a.d = d;
    const tc::WignerArgs all = a;
    const int step = per_launch(L.ntile, t.NT);
    rc = timed_launch(TC_OP_WIGNER, stream, [&] {
        int r = 0;
        for (long long i0 = 0; i0 < npair && !r; i0 += step) {
            a.npair = (int)std::min<long long>(step, npair - i0);
            a.col = tc::ColumnTables{all.col.mb + i0, all.col.ms + i0, all.col.lnA + 2 * i0};
            a.d = all.d + i0 * (lmax + 1) * nring;
            r = tc::launch_wigner(a, t, stream);
        }
        return r;
    });
    return rc ? hip_fail(rc, "wigner_d_rings launch") : TC_OK;
}

int totalconv_fwd_x(int lmax, int mbmax, int nring, const double* cosbeta, const double* alm, const double* blm,
                  double* C, void* workspace, size_t ws_bytes, void* stream)
{
    g_error.clear();
    return fwd_impl(TC_OP_FWD, lmax, mbmax, nring, cosbeta, 1, &alm, &blm, 0, &C, workspace, ws_bytes, stream);
}

int totalconv_fwd_pol_x(int lmax, int mbmax, int nring, const double* cosbeta, int npair, const double* const* alm,
                      const double* const* blm, int mode, double* const* C, void* workspace, size_t ws_bytes,
                      void* stream)
{
    g_error.clear();
    if (npair < 1 || npair > 3) return fail(TC_EINVAL, "npair = %d outside [1, 3]", npair);
    if (mode != TC_POL_SEPARATE && mode != TC_POL_SUM) return fail(TC_EINVAL, "unknown mode %d", mode);
    if (!alm || !blm || !C) return fail(TC_EINVAL, "alm, blm or C pointer array is NULL");
    return fwd_impl(TC_OP_FWD_POL, lmax, mbmax, nring, cosbeta, npair, alm, blm, mode == TC_POL_SUM ? 1 : 0, C,
                    workspace, ws_bytes, stream);
}

int totalconv_adj_x(int lmax, int mbmax, int nring, const double* cosbeta, const double* alm, const double* blm,
                  const double* Cbar, double* alm_bar, double* blm_bar, void* workspace, size_t ws_bytes,
                  void* stream)
{
    g_error.clear();
    return adj_impl(lmax, mbmax, nring, cosbeta, 1, &alm, &blm, 0, &Cbar, &alm_bar, &blm_bar, workspace, ws_bytes,
                    stream);
}

int totalconv_adj_pol_x(int lmax, int mbmax, int nring, const double* cosbeta, int npair, const double* const* alm,
                      const double* const* blm, int mode, const double* const* Cbar, double* const* alm_bar,
                      double* const* blm_bar, void* workspace, size_t ws_bytes, void* stream)
{
    g_error.clear();
    if (npair < 1 || npair > 3) return fail(TC_EINVAL, "npair = %d outside [1, 3]", npair);
    if (mode != TC_POL_SEPARATE && mode != TC_POL_SUM) return fail(TC_EINVAL, "unknown mode %d", mode);
    if (!alm || !blm || !Cbar) return fail(TC_EINVAL, "alm, blm or Cbar pointer array is NULL");
    return adj_impl(lmax, mbmax, nring, cosbeta, npair, alm, blm, mode == TC_POL_SUM ? 1 : 0, Cbar, alm_bar,
                    blm_bar, workspace, ws_bytes, stream);
}

// ----------------------------------------------------- entry points on colatitudes
// Each forms the rings once (tc_rings_from_beta) and runs its *_x twin on them.

int tc_rings_from_beta(int nring, const double* beta, double* cosbeta)
{
    g_error.clear();
    if (!cosbeta) return fail(TC_EINVAL, "cosbeta (output) is NULL");
    std::vector<double> x;
    const int rc = rings_from_beta(nring, beta, x);
    if (rc) return rc;
    std::memcpy(cosbeta, x.data(), sizeof(double) * (size_t)nring);
    return TC_OK;
}

size_t totalconv_workspace_bytes_rings(int op, int lmax, int mbmax, int nring, const double* beta)
{
    const std::string saved = g_error;
    std::vector<double> x;
    const int rc = rings_from_beta(nring, beta, x);
    g_error = saved;
    return rc ? 0 : totalconv_workspace_bytes_rings_x(op, lmax, mbmax, nring, x.data());
}

int wigner_d_rings(int lmax, int npair, const int* mb, const int* msky, int nring, const double* beta, double* d,
                   void* workspace, size_t ws_bytes, void* stream)
{
    g_error.clear();
    std::vector<double> x;
    const int rc = rings_from_beta(nring, beta, x);
    return rc ? rc : wigner_d_rings_x(lmax, npair, mb, msky, nring, x.data(), d, workspace, ws_bytes, stream);
}

int wigner_d_matrix(int l, int nring, const double* beta, double* d, void* workspace, size_t ws_bytes, void* stream)
{
    g_error.clear();
    std::vector<double> x;
    const int rc = rings_from_beta(nring, beta, x);
    return rc ? rc : wigner_d_matrix_x(l, nring, x.data(), d, workspace, ws_bytes, stream);
}

int totalconv_fwd(int lmax, int mbmax, int nring, const double* beta, const double* alm, const double* blm, double* C,
                  void* workspace, size_t ws_bytes, void* stream)
{
    g_error.clear();
    std::vector<double> x;
    const int rc = rings_from_beta(nring, beta, x);
    return rc ? rc : totalconv_fwd_x(lmax, mbmax, nring, x.data(), alm, blm, C, workspace, ws_bytes, stream);
}

int totalconv_fwd_pol(int lmax, int mbmax, int nring, const double* beta, int npair, const double* const* alm,
                      const double* const* blm, int mode, double* const* C, void* workspace, size_t ws_bytes,
                      void* stream)
{
    g_error.clear();
    std::vector<double> x;
    const int rc = rings_from_beta(nring, beta, x);
    return rc ? rc
              : totalconv_fwd_pol_x(lmax, mbmax, nring, x.data(), npair, alm, blm, mode, C, workspace, ws_bytes,
                                    stream);
}

int totalconv_adj(int lmax, int mbmax, int nring, const double* beta, const double* alm, const double* blm,
                  const double* Cbar, double* alm_bar, double* blm_bar, void* workspace, size_t ws_bytes,
                  void* stream)
{
    g_error.clear();
    std::vector<double> x;
    const int rc = rings_from_beta(nring, beta, x);
    return rc ? rc
              : totalconv_adj_x(lmax, mbmax, nring, x.data(), alm, blm, Cbar, alm_bar, blm_bar, workspace, ws_bytes,
                                stream);
}

int totalconv_adj_pol(int lmax, int mbmax, int nring, const double* beta, int npair, const double* const* alm,
                      const double* const* blm, int mode, const double* const* Cbar, double* const* alm_bar,
                      double* const* blm_bar, void* workspace, size_t ws_bytes, void* stream)
{
    g_error.clear();
    std::vector<double> x;
    const int rc = rings_from_beta(nring, beta, x);
    return rc ? rc
              : totalconv_adj_pol_x(lmax, mbmax, nring, x.data(), npair, alm, blm, mode, Cbar, alm_bar, blm_bar,
                                    workspace, ws_bytes, stream);
}

}  // extern "C"

// ============================================================ no-allocation forward
namespace tc {

int fail_hip(int rc, const char* what) { return hip_fail(rc, what); }

int fwd_noalloc(int lmax, int mbmax, int nring, const double* beta, const double* alm, const double* blm, double* C,
                void* scratch, size_t scratch_bytes, void* stream)
{
    g_error.clear();
    std::vector<double> x;
    int rc = rings_from_beta(nring, beta, x);
    if (rc) return rc;
    if ((rc = check_sizes(lmax, mbmax))) return rc;
    const Layout L = make_layout(TC_OP_FWD, lmax, mbmax, nring, x.data(), default_tile(TC_OP_FWD, lmax));
    if (L.total > scratch_bytes)
        return fail(TC_ENOMEM, "totalconv_fwd_noalloc: the tables need %zu bytes, more than the %zu bytes of "
                               "its static device array", L.total, scratch_bytes);
    return fwd_impl(TC_OP_FWD, lmax, mbmax, nring, x.data(), 1, &alm, &blm, 0, &C, scratch, scratch_bytes, stream,
                    false);
}

}  // namespace tc

// ===================================================================== plans
//
// A plan holds, in one device allocation, the tables of every walk, the kernel-argument
// records, the work items sorted by cost (longest first) and, for the adjoint, the partial
// sums.  A walk serves several detectors that share lmax and rings: in the forward up to
// fwd_walk_pairs of its tile (one recursion feeds each member's output), in the adjoint
// adj_walk_pairs_of.  Forward graph: beam row signs, then one launch per (R, NT) of the walks, side by
// side.  Adjoint graph: one launch per (R, NT, lmax), one after the other, each followed on a second
// stream by its detectors' sky gradients (one launch) and beam gradients (one each).

struct tc_plan_s {
    int op = 0;
    int ndet = 0;
    int nwalk = 0;
    int sky_lmax = 0;
    tc::Tile tile{8, 256, 32, 4};
    void* dmem = nullptr;
    size_t dbytes = 0;
    int nitems = 0;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipEvent_t done = nullptr;
};

namespace {

void destroy_plan(tc_plan_s* p)
{
    if (!p) return;
    // Teardown is best effort: errors here cannot be acted on by the caller.
    if (p->done) (void)hipEventSynchronize(p->done);
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    if (p->done) (void)hipEventDestroy(p->done);
    if (p->dmem) (void)hipFree(p->dmem);
    delete p;
}

// The rings of detector d: from its colatitudes (beta) or, when beta is NULL, its cosines.
int detector_rings(int i, const tc_detector& d, std::vector<double>& x)
{
    int rc = TC_OK;
    if (d.beta) {
        rc = rings_from_beta(d.nring, d.beta, x);
    } else {
        rc = check_rings(d.nring, d.cosbeta);
        if (!rc) x.assign(d.cosbeta, d.cosbeta + d.nring);
    }
    if (rc) g_error = "detector " + std::to_string(i) + ": " + g_error;
    return rc;
}

int check_detector(int i, const tc_detector& d, int op, int lmax_sky)
{
    if (d.lmax < 0 || d.lmax > lmax_sky)
        return fail(TC_EINVAL, "detector %d: lmax = %d outside [0, lmax_sky = %d]", i, d.lmax, lmax_sky);
    if (d.mbmax < 0 || d.mbmax > d.lmax)
        return fail(TC_EINVAL, "detector %d: mbmax = %d outside [0, lmax = %d]", i, d.mbmax, d.lmax);
    if (!d.blm || !aligned16(d.blm)) return fail(TC_EINVAL, "detector %d: blm NULL or not 16-byte aligned", i);
    if (op == TC_OP_FWD && (!d.C || !aligned16(d.C)))
        return fail(TC_EINVAL, "detector %d: C NULL or not 16-byte aligned", i);
    if (op == TC_OP_ADJ) {
        if (!d.Cbar || !aligned16(d.Cbar)) return fail(TC_EINVAL, "detector %d: Cbar NULL or misaligned", i);
        if (d.blm_bar && !aligned16(d.blm_bar)) return fail(TC_EINVAL, "detector %d: blm_bar misaligned", i);
    }
    return TC_OK;
}

// R of a walk over nslot ring slots: the plan's R, halved while half of it still covers every
// slot in one ring tile of 256 lanes (fit_tile then takes the lanes).
int walk_R(const tc::Tile& t, int nslot)
{
    int R = t.R;
    while (R > 2 && 256 * (R / 2) >= nslot) R /= 2;
    return R;
}

struct Walk {
    std::vector<int> mem;   // detectors, largest mbmax first
    tc::Tile tile;          // the plan's tile with the walk's R
};

// Walks of a plan: detectors with the same lmax and the same ring cosines (bit for bit) form
// one class, whose walks take the class's R; each class, ordered by mbmax (largest first, then
// by index), is cut into walks of as many detectors as a walk at that tile serves.  Walks come
// in the order of their first detector.
std::vector<Walk> group_detectors(int op, int ndet, const tc_detector* dets,
                                  const std::vector<std::vector<double>>& xr, const tc::Tile& t)
{
    std::vector<std::vector<int>> cls;
    for (int i = 0; i < ndet; ++i) {
        bool placed = false;
        for (auto& c : cls) {
            const int j = c.front();
            if (dets[j].lmax == dets[i].lmax && xr[j] == xr[i]) {
                c.push_back(i);
                placed = true;
                break;
            }
        }
        if (!placed) cls.push_back({i});
    }
    std::vector<Walk> walks;
    for (auto& c : cls) {
        std::stable_sort(c.begin(), c.end(), [&](int a, int b) { return dets[a].mbmax > dets[b].mbmax; });
        tc::Tile wt = t;
        const int nslot = count_slots(dets[c[0]].nring, xr[c[0]].data());
        wt.R = walk_R(t, nslot);
        wt = fit_tile(op, wt, nslot);
        const size_t per_walk = (size_t)(op == TC_OP_FWD ? tc::fwd_walk_pairs(wt) : tc::adj_walk_pairs_of(wt));
        for (size_t k = 0; k < c.size(); k += per_walk)
            walks.push_back({std::vector<int>(c.begin() + k, c.begin() + std::min(c.size(), k + per_walk)), wt});
    }
    return walks;
}

}  // namespace

extern "C" {

int tc_plan_create(void** plan, int op, int ndet, const tc_detector* dets, int lmax_sky, const double* alm,
                   double* alm_bar, void* stream)
{
    g_error.clear();
    if (!plan) return fail(TC_EINVAL, "plan is NULL");
    *plan = nullptr;
    if (op != TC_OP_FWD && op != TC_OP_ADJ) return fail(TC_EINVAL, "plans support TC_OP_FWD and TC_OP_ADJ only");
    if (ndet < 1 || !dets) return fail(TC_EINVAL, "ndet must be >= 1 with a detector array");
    if (lmax_sky < 0 || lmax_sky > TC_LMAX_LIMIT) return fail(TC_EINVAL, "lmax_sky = %d out of range", lmax_sky);
    if (!alm || !aligned16(alm)) return fail(TC_EINVAL, "alm NULL or not 16-byte aligned");
    if (alm_bar && !aligned16(alm_bar)) return fail(TC_EINVAL, "alm_bar not 16-byte aligned");
    std::vector<std::vector<double>> xr(ndet);   // every detector's ring cosines
    for (int i = 0; i < ndet; ++i) {
        if (int rc = check_detector(i, dets[i], op, lmax_sky)) return rc;
        if (int rc = detector_rings(i, dets[i], xr[i])) return rc;
    }
    const tc::Tile tile = default_tile(op, 1 << 20);   // the largest R of the plan's walks
    const std::vector<Walk> walks = group_detectors(op, ndet, dets, xr, tile);
    const int nwalk = (int)walks.size();

    tc_plan_s* p = new tc_plan_s;
    p->op = op;
    p->ndet = ndet;
    p->nwalk = nwalk;
    p->sky_lmax = lmax_sky;
    p->tile = tile;

    // ---- layout of the plan's device memory: per walk the tables of its first detector (the
    // largest mbmax: its columns cover every member's), per detector its beam row signs
    std::vector<Layout> lay(nwalk);
    std::vector<size_t> base(nwalk), sym_off(ndet);
    size_t off = 0;
    long long nitems = 0;
    for (int w = 0; w < nwalk; ++w) {
        const tc_detector& d = dets[walks[w].mem[0]];
        lay[w] = make_layout(op, d.lmax, d.mbmax, d.nring, xr[walks[w].mem[0]].data(), walks[w].tile);
        base[w] = off;
        off = align_up(off + lay[w].total);
        nitems += (long long)lay[w].ncol * lay[w].ntile;
    }
    for (int i = 0; i < ndet; ++i) {
        sym_off[i] = off;
        off = align_up(off + sizeof(int) * (size_t)(2 * dets[i].mbmax + 1));
    }
    // adjoint: the U and V rows of a walk's later members (the first uses its walk's layout)
    std::vector<size_t> uv_off(ndet, 0);
    for (int w = 0; w < nwalk && op == TC_OP_ADJ; ++w)
        for (size_t q = 1; q < walks[w].mem.size(); ++q) {
            const int i = walks[w].mem[q];
            uv_off[i] = off;
            off = align_up(off + 2 * align_up((size_t)16 * (size_t)(2 * dets[i].mbmax + 1) * (size_t)lay[w].P));
        }
    if (nitems > 0x7fffffffLL / 3) { destroy_plan(p); return fail(TC_EUNSUPPORTED, "too many work items"); }
    const size_t args_off = off;
    const size_t args_bytes = op == TC_OP_FWD ? sizeof(tc::FwdArgs) * nwalk : sizeof(tc::AdjArgs) * nwalk;
    off = align_up(off + args_bytes);
    const size_t epi_off = off;
    off = align_up(off + sizeof(tc::EpiArgs) * ndet);
    const size_t items_off = off;
    off = align_up(off + sizeof(int) * 3 * (size_t)nitems);
    p->dbytes = off;
    int rc = (int)hipMalloc(&p->dmem, p->dbytes);
    if (rc) {
        (void)hipGetLastError();   // the failed allocation must not be reported by the next launch check
        destroy_plan(p);
        return fail(TC_ENOMEM, "plan: hipMalloc of %zu bytes failed", off);
    }
    char* dm = static_cast<char*>(p->dmem);

    // ---- tables, argument records, items
    std::vector<tc::FwdArgs> fa(op == TC_OP_FWD ? nwalk : 0);
    std::vector<tc::AdjArgs> aa(op == TC_OP_ADJ ? nwalk : 0);
    std::vector<tc::EpiArgs> ea(ndet);
    // Launch groups: the walks of one R and NT (forward), and of one lmax too (adjoint: each group's
    // epilogues run beside the next group's walks).
    struct Group { int R, NT, lmax; tc::Tile tile; long long cost; std::vector<int> walks; };
    std::vector<Group> groups;
    struct Item { int grp, walk, col, tile; long long cost; };
    std::vector<Item> items;
    items.reserve((size_t)nitems);
    for (int w = 0; w < nwalk; ++w) {
        const std::vector<int>& mem = walks[w].mem;
        const tc::Tile& wt = walks[w].tile;
        const tc_detector& d = dets[mem[0]];
        const Layout& L = lay[w];
        const int glmax = op == TC_OP_ADJ ? d.lmax : -1;
        int grp = 0;
        while (grp < (int)groups.size() &&
               !(groups[grp].R == wt.R && groups[grp].NT == wt.NT && groups[grp].lmax == glmax))
            ++grp;
        if (grp == (int)groups.size()) groups.push_back({wt.R, wt.NT, glmax, wt, 0, {}});
        groups[grp].walks.push_back(w);
        std::vector<char> img(L.tables_end, 0);
        build_rings(d.nring, xr[mem[0]].data(), img, L);
        build_slots(d.nring, xr[mem[0]].data(), img, L);
        build_columns(d.lmax, d.mbmax, img, L);
        rc = (int)hipMemcpy(dm + base[w], img.data(), img.size(), hipMemcpyHostToDevice);
        if (rc) { destroy_plan(p); return hip_fail(rc, "plan: table upload"); }
        void* ws = dm + base[w];
        const int* cms = reinterpret_cast<const int*>(img.data() + L.colms);
        const int* cmb = reinterpret_cast<const int*>(img.data() + L.colmb);
        for (int c = 0; c < L.ncol; ++c) {
            const int len = d.lmax - std::max(std::abs(cmb[c]), cms[c]) + 1;
            int k = 0;   // members with this column's beam row
            for (int i : mem) k += dets[i].mbmax >= std::abs(cmb[c]);
            if (op == TC_OP_ADJ) {   // one item walks every ring tile of the column
                // a step costs about 2 + 5k operations per chain (the recursion, k cotangents' sums)
                items.push_back({grp, w, c, 0, (long long)len * L.nslot * (2 + 5 * k)});
                continue;
            }
            for (int t = 0; t < L.ntile; ++t) {
                const int slots = std::min(wt.NT * wt.R, L.nslot - t * wt.NT * wt.R);
                // a step costs about 2 + 2k operations per chain (the recursion, k outputs' sums)
                items.push_back({grp, w, c, t, (long long)len * slots * (2 + 2 * k)});
            }
        }
        if (op == TC_OP_FWD) {
            tc::FwdArgs& a = fa[w];
            a = tc::FwdArgs{};
            a.lmax = d.lmax; a.mbmax = d.mbmax; a.nring = d.nring; a.nslot = L.nslot; a.ncol = L.ncol;
            a.ntile = L.ntile; a.sky_lmax = lmax_sky; a.skip_exp = 100;
            a.ring = ring_ptrs(ws, L, d.nring);
            a.slots = reinterpret_cast<const int*>(static_cast<char*>(ws) + L.slots);
            a.col = col_ptrs(ws, L);
            a.npair = (int)mem.size(); a.sum = 0;
            for (size_t q = 0; q < mem.size(); ++q) {
                const tc_detector& m = dets[mem[q]];
                a.pmbmax[q] = m.mbmax; a.alm[q] = alm; a.blm[q] = m.blm; a.C[q] = m.C;
                a.beam_sym[q] = reinterpret_cast<const int*>(dm + sym_off[mem[q]]);
            }
        } else {
            tc::AdjArgs& a = aa[w];
            a = tc::AdjArgs{};
            a.lmax = d.lmax; a.mbmax = d.mbmax; a.nring = d.nring; a.nslot = L.nslot; a.ncol = L.ncol;
            a.ntile = L.ntile; a.skip_exp = 100;
            a.ring = ring_ptrs(ws, L, d.nring);
            a.slots = reinterpret_cast<const int*>(static_cast<char*>(ws) + L.slots);
            a.col = col_ptrs(ws, L);
            a.P = L.P;
            a.npair = (int)mem.size();
            for (size_t q = 0; q < mem.size(); ++q) {
                const tc_detector& m = dets[mem[q]];
                char* uv = q == 0 ? static_cast<char*>(ws) + L.U : dm + uv_off[mem[q]];
                const size_t ubytes = (size_t)16 * (size_t)(2 * m.mbmax + 1) * (size_t)L.P;
                a.pmbmax[q] = m.mbmax;
                a.Cbar[q] = m.Cbar;
                a.U[q] = reinterpret_cast<double*>(uv);
                a.V[q] = reinterpret_cast<double*>(q == 0 ? static_cast<char*>(ws) + L.V : uv + align_up(ubytes));
                tc::EpiArgs& e = ea[mem[q]];
                e = tc::EpiArgs{};
                e.lmax = m.lmax; e.mbmax = m.mbmax; e.P = L.P; e.sky_lmax = lmax_sky;
                e.U = a.U[q]; e.V = a.V[q]; e.alm = alm; e.blm = m.blm; e.alm_bar = nullptr; e.blm_bar = m.blm_bar;
            }
        }
    }
    // one launch per group, the costliest group first, each over its items longest first
    for (const Item& it : items) groups[it.grp].cost += it.cost;
    std::vector<int> rank(groups.size());
    {
        std::vector<int> order(groups.size());
        for (size_t g = 0; g < groups.size(); ++g) order[g] = (int)g;
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return groups[a].cost > groups[b].cost; });
        for (size_t r = 0; r < order.size(); ++r) rank[order[r]] = (int)r;
    }
    p->nitems = (int)items.size();
    std::stable_sort(items.begin(), items.end(), [&](const Item& a, const Item& b) {
        return rank[a.grp] != rank[b.grp] ? rank[a.grp] < rank[b.grp] : a.cost > b.cost;
    });
    struct Launch { int grp, first, n; };
    std::vector<Launch> launches;
    for (size_t k = 0; k < items.size(); ++k) {
        if (launches.empty() || launches.back().grp != items[k].grp) launches.push_back({items[k].grp, (int)k, 0});
        launches.back().n += 1;
    }
    const int per_item = op == TC_OP_FWD ? 3 : 2;
    std::vector<int> it3((size_t)per_item * items.size());
    for (size_t k = 0; k < items.size(); ++k) {
        it3[per_item * k] = items[k].walk;
        it3[per_item * k + 1] = items[k].col;
        if (per_item == 3) it3[per_item * k + 2] = items[k].tile;
    }
    // adjoint: the epilogue records of each launch's detectors, launch by launch
    std::vector<tc::EpiArgs> eg;
    std::vector<int> eg_first(launches.size() + 1, 0);
    for (size_t k = 0; k < launches.size() && op == TC_OP_ADJ; ++k) {
        eg_first[k] = (int)eg.size();
        for (int w : groups[launches[k].grp].walks)
            for (int i : walks[w].mem) eg.push_back(ea[i]);
    }
    eg_first[launches.size()] = (int)eg.size();
    rc = (int)hipMemcpy(dm + args_off, op == TC_OP_FWD ? (const void*)fa.data() : (const void*)aa.data(), args_bytes,
                        hipMemcpyHostToDevice);
    if (!rc && op == TC_OP_ADJ)
        rc = (int)hipMemcpy(dm + epi_off, eg.data(), sizeof(tc::EpiArgs) * eg.size(), hipMemcpyHostToDevice);
    if (!rc) rc = (int)hipMemcpy(dm + items_off, it3.data(), sizeof(int) * it3.size(), hipMemcpyHostToDevice);
    if (rc) { destroy_plan(p); return hip_fail(rc, "plan: argument upload"); }

    // ---- capture the graph on a private stream (the caller's stream may be the legacy one).
    // Forward: the launches run side by side, the costliest on the capture stream, each other on
    // a stream of its own forked from it and joined back.  Adjoint: the launches run one after the
    // other on the capture stream; after each, a second stream runs the epilogues of its
    // detectors (memory-bound) beside the next launch's walks (ALU-bound): the sky gradient, summed
    // launch by launch in a fixed order (the first launch writes it, the others add to it), and
    // each detector's beam gradient.
    const int nside = op == TC_OP_FWD ? std::max(0, (int)launches.size() - 1) : 1;
    const int nev = op == TC_OP_FWD ? nside : (int)launches.size() + 1;
    std::vector<hipStream_t> side(nside, nullptr);
    std::vector<hipEvent_t> evs(nev, nullptr);
    hipEvent_t fork = nullptr;
    hipStream_t cs = nullptr;
    auto release_capture = [&] {
        for (hipStream_t q : side) if (q) (void)hipStreamDestroy(q);
        for (hipEvent_t e : evs) if (e) (void)hipEventDestroy(e);
        if (fork) (void)hipEventDestroy(fork);
        if (cs) (void)hipStreamDestroy(cs);
    };
    rc = (int)hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
    if (!rc) rc = (int)hipEventCreateWithFlags(&fork, hipEventDisableTiming);
    for (int k = 0; k < nside && !rc; ++k) rc = (int)hipStreamCreateWithFlags(&side[k], hipStreamNonBlocking);
    for (int k = 0; k < nev && !rc; ++k) rc = (int)hipEventCreateWithFlags(&evs[k], hipEventDisableTiming);
    if (rc) { release_capture(); destroy_plan(p); return hip_fail(rc, "plan: capture streams"); }
    rc = (int)hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    const int* d_items = reinterpret_cast<const int*>(dm + items_off);
    if (op == TC_OP_FWD) {
        for (int i = 0; i < ndet && !rc; ++i)   // beam row signs, on every execution
            rc = tc::launch_beam_symmetry(dets[i].blm, dets[i].lmax, dets[i].mbmax,
                                          reinterpret_cast<int*>(dm + sym_off[i]), cs);
        if (!rc && nside > 0) rc = (int)hipEventRecord(fork, cs);
        for (size_t k = 0; k < launches.size() && !rc; ++k) {
            hipStream_t q = k == 0 ? cs : side[k - 1];
            if (k > 0) rc = (int)hipStreamWaitEvent(q, fork, 0);
            const Launch& l = launches[k];
            const tc::Tile& wt = groups[l.grp].tile;
            for (long long i = 0, step = per_launch(1, wt.NT); i < l.n && !rc; i += step)
                rc = tc::launch_fwd_items(reinterpret_cast<const tc::FwdArgs*>(dm + args_off),
                                          d_items + 3 * (size_t)(l.first + i), (int)std::min(step, l.n - i), wt, q);
            if (!rc && k > 0) rc = (int)hipEventRecord(evs[k - 1], q);
        }
        for (int k = 0; k < nside && !rc; ++k) rc = (int)hipStreamWaitEvent(cs, evs[k], 0);
    } else {
        hipStream_t es = side[0];
        const tc::EpiArgs* d_eg = reinterpret_cast<const tc::EpiArgs*>(dm + epi_off);
        for (size_t k = 0; k < launches.size() && !rc; ++k) {
            const Launch& l = launches[k];
            const tc::Tile& wt = groups[l.grp].tile;
            for (long long i = 0, step = per_launch(1, wt.NT); i < l.n && !rc; i += step)
                rc = tc::launch_adj_items(reinterpret_cast<const tc::AdjArgs*>(dm + args_off),
                                          d_items + 2 * (size_t)(l.first + i), (int)std::min(step, l.n - i), wt, cs);
            if (!rc) rc = (int)hipEventRecord(evs[k], cs);
            if (!rc) rc = (int)hipStreamWaitEvent(es, evs[k], 0);
            if (!rc && alm_bar)
                rc = tc::launch_adj_sky_multi(d_eg + eg_first[k], eg_first[k + 1] - eg_first[k], lmax_sky, k > 0,
                                              alm_bar, es);
            for (int e = eg_first[k]; e < eg_first[k + 1] && !rc; ++e)
                if (eg[e].blm_bar) rc = tc::launch_adj_beam(eg[e], es);
        }
        if (!rc) rc = (int)hipEventRecord(evs[launches.size()], es);
        if (!rc) rc = (int)hipStreamWaitEvent(cs, evs[launches.size()], 0);
    }
    hipGraph_t g = nullptr;
    const int rc_end = (int)hipStreamEndCapture(cs, &g);
    release_capture();
    p->graph = g;
    if (rc || rc_end) { destroy_plan(p); return hip_fail(rc ? rc : rc_end, "plan: graph capture"); }
    rc = (int)hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0);
    if (!rc) rc = (int)hipEventCreateWithFlags(&p->done, hipEventDisableTiming);
    if (rc) { destroy_plan(p); return hip_fail(rc, "plan: graph instantiation"); }
    (void)stream;
    *plan = p;
    return TC_OK;
}

int tc_plan_execute(void* plan, void* stream)
{
    g_error.clear();
    tc_plan_s* p = static_cast<tc_plan_s*>(plan);
    if (!p || !p->exec) return fail(TC_EINVAL, "invalid plan");
    int rc = (int)hipGraphLaunch(p->exec, (hipStream_t)stream);
    if (!rc) rc = (int)hipEventRecord(p->done, (hipStream_t)stream);
    return rc ? hip_fail(rc, "tc_plan_execute") : TC_OK;
}

size_t tc_plan_device_bytes(void* plan)
{
    return plan ? static_cast<tc_plan_s*>(plan)->dbytes : 0;
}

int tc_plan_tile(void* plan)
{
    return plan ? static_cast<tc_plan_s*>(plan)->tile.R : 0;
}

int tc_plan_destroy(void* plan)
{
    destroy_plan(static_cast<tc_plan_s*>(plan));
    return TC_OK;
}

}  // extern "C"
