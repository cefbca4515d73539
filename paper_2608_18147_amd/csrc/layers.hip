// dp_APX (Sec. 5, eq. apx_base / apx_rec) for one multiplier, layer by layer
// with bounds: every F_i[j] is the minimum over all predecessors k bit for
// bit, but a predecessor is evaluated only where a lower bound of its
// candidate does not already exceed an upper bound of the column's minimum.
//
// One launch per layer, one workgroup per block of columns (a unit: 16 columns,
// or 64).  F_{i-1} is whole when the launch starts, so no workgroup waits for
// another.  A workgroup
//   1. evaluates its first and its last column against the last predecessor of
//      every far unit and takes the best unit of each;
//   2. evaluates all its columns against a few predecessors around those units
//      and before its own columns, which bounds every minimum from above: u_j;
//   3. tests the predecessors around those units one by one, evaluates those
//      left and so tightens u_j;
//   4. tests every other unit of predecessors as a whole against its columns
//      (first 8 units at once where there are many), the units left against
//      each group of 16 columns, and the predecessors of those left one by one,
//      and evaluates what is left.
//
// Bounds, for predecessors a and columns b > a, with tu(a, b) = sum over x in
// (a, b] of (x - a), td(a, b) = sum of (b - x), n the entries in (a, b], U = tu /
// (b - a), D = td / (b - a) and d the distance moved:
//   - in b, dC/db = tu, which grows; in a, dC/da = -td, and C is convex: from the
//     unit's last value and the first column, C rises by at least d tu towards the
//     last column, d td towards the unit's first value, and d d' n for both;
//   - between entries dD/db = tu / (b - a)^2 and dU/da = -td / (b - a)^2, D is
//     continuous in b and U in a, and U + D = n.  Bounding the rates by their ends
//     and n by a band around its line makes each of U and D run between two
//     planes over the rectangle unit x columns;
//   - h is concave, so h of a plane is at least the interpolation of its corners;
//   - F_{i-1} over a unit lies above a line kept from the layer before, and the
//     u_j lie under a line over the columns.
// So candidate - u_j is at least the interpolation of four corner values: where
// all are positive, no predecessor of the unit holds any column's minimum.  A
// single predecessor leaves two corners.
//
// Rounding.  The bounds are statements about exact sums; a candidate and its
// bound are both computed from prefix sums rounded to 53 bits.  With vm =
// max(|a|, |b|), N and S2 the inclusive prefixes at the last column (which bound
// those before it; |S| <= sqrt(N S2)), each term of C is at most vm^2 N + S2 up
// to a small factor and carries a few roundings: its error is below 2^-48 of
// that.  The tests give 2^-44 (vm^2 N + S2 + |u|) + 2^-40 lambda' away, widen U
// and D by 2^-20 and their rates by 2^-18 of themselves (the approximate
// reciprocal is good to 2^-24) plus the error 2^-44 (vm N + sqrt(N S2)) of tu and
// td over the width, and lower the 32-bit h by 2^-18 of itself and 2^-20 y
// (v_log_f32 is good to about an ulp).  Where sums cancel that error may exceed 1:
// computed frequencies then pass 1, h is negative there, and so are the bounds.
//
// What bounds it: the latency of a workgroup's stages, about 30 us a layer at 16384
// values (1024 workgroups, of which 768 fit the chip at once: three wavefronts a SIMD at 137
// and 168 registers), and with many values the work left: 160 us a layer at 2^18 at
// lambda = 0, 235 above, where VALU issue is 46% used and wavefronts wait 40% of their time
// for data or at barriers.  2^18 weight-like values, 32 layers: 5.6 ms at lambda = 0, 12.2
// at 0.01, 8.6 at 0.1 to 2, where the sweep over all pairs takes 95 and 132 ms; of the
// p^2 / 2 pairs of a layer 0.03% to 0.2% are evaluated and 0.05% to 1% tested one by one.
// Bounds that are constant over a unit (no lines) left 1% to 3% and took twice to three
// times as long.
#include "device.hpp"
#include "launch.hpp"

namespace ecasq {

namespace {

constexpr int kSB = 64;       // predecessors per block
constexpr int kGC = 16;       // columns of a wavefront (4 predecessors side by side)
constexpr int64_t kWideP = 49152;
constexpr int kList = 1024;   // blocks tested per round (those left are listed in LDS)

// What is left of the far predecessors after the tests of units, in steps of a wavefront: one
// for four predecessors evaluated, four for 64 tested one by one.  Few for ordinary inputs; most
// of the predecessors where prefix sums cancel so far that no bound holds (values over 60
// decades, an outlier of 1e18), and then the sweep, which forms each cost once for all
// layers, is up to ten times faster (2^18 such values, 32 layers: 1390 ms against 132).  So the
// steps are counted: a workgroup reports its own at its end if a wavefront has p / 32 of them
// (fewer for many layers; most never do), and adds them to a word only where needed, since
// additions to one word wait for each other, 6 ns each.  When the longest chains of the
// layers and a kCrowd-th of all steps pass the layer's limit, the solve gives up (the
// failure word is kSweepGaveUp) and the host takes the sweep: 203 ms in that example, 3.4
// against 2.9 for 16384 values.  Counting costs ordinary inputs 0 to 1.5% (a report between
// rounds too, which can stop a layer half way, 1 to 2.5%; the example then takes 169 ms).
struct LayWork {
    unsigned long long all;
    uint32_t chain;       // sum over the layers of the most steps of a wavefront
    uint32_t longest[2];  // that of the layer (parity)
    uint32_t gone[2];     // the layer or one before it has given up (parity)
    uint32_t pad;
    int32_t* fail;        // the failure word
    uint32_t limit[256];  // of each layer
};
constexpr uint32_t kCrowd = 2048;
constexpr size_t kWorkBytes = 2048;
static_assert(sizeof(LayWork) <= kWorkBytes, "the work words fit before the units");
constexpr uint32_t kSample = 16;  // one workgroup of so many adds to `all`

template <class T>
__device__ __forceinline__ T fresh(const T* at) {
    return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct LayArgs {
    Hist H;
    double* F;    // [I+1][ld], rows 2..I
    double2* SB;  // kUnit per unit: (v, N), (S, S2) of its last value, the same of its
                  // first, and how far N_last - N_k lies from its line
    double2* LN;  // two rows of nun: F_i[k] >= x + y (v_k - v_first) in the unit (layer parity)
    double* FE;   // two rows of nun: F_i at the unit's last value
    int32_t* K;   // K[nblk]: the failure word of eq. apx_final's kernel
    int64_t ld, nblk, nun;
    int32_t I;
    double lamp;
    const double* lampp;
    const int32_t* runp;
};
constexpr int kUnit = 5;
// units left of a round above which they are tested against single columns
constexpr int kMany = 128;

__device__ __forceinline__ bool live(LayArgs& a) {
    if (a.runp && *a.runp == 0) return false;
    if (a.lampp) a.lamp = *a.lampp;
    return true;
}

// The steps up to layer i at whose rate the layers after it would take as long as the whole
// solve by the sweep, and some on top for layers that need more than the rest: a twentieth of
// the sweep's time, and what a column far from all others (the last of a heavy tail) takes
// by itself.  In microseconds: the sweep's time (a chain of blocks for few values, cells at a
// rate for many: 5000 values and 16 layers 0.58 ms, 16384 and 32 2.6, 128 5.6, 65536 and 32
// 13.2, 2^18 and 32 132 and 95 at lambda = 0), a layer with few steps, and 0.18 for a step
// (0.166 to 0.184 from inputs with 1000 to 5000 steps of a wavefront in a layer; half at
// lambda = 0).
__device__ __forceinline__ uint32_t work_limit(int64_t p, int32_t I, int32_t i, bool zero) {
    const double n = (double)p, left = (double)(I - i), step = zero ? 0.09 : 0.18;
    if (left < 1.0) return 0xFFFFFFFFu;
    const double sweep =
        n * __builtin_fmax(0.08 + 0.002 * I + 7e-7 * n, (zero ? 4.4e-8 : 6.2e-8) * n * I);
    const double layer = 18.0 + n / 1500.0;
    const double alone = n / (p < kWideP ? 16.0 : 8.0);
    const double rest = (double)(i - 2) * __builtin_fmax(0.0, sweep / left - layer);
    return (uint32_t)__builtin_fmin(__builtin_fmax(0.05 * sweep / step, alone) + rest / step, 4e9);
}

__device__ __forceinline__ LayWork* work_of(const LayArgs& a) {
    return reinterpret_cast<LayWork*>(reinterpret_cast<char*>(a.SB) - kWorkBytes);
}

// A line under F_i over each unit of UN columns and F_i at its end, as the next
// layer reads them; f, v = F_i and the value of the thread's column j, +inf past
// p - 1.  The line is lowered by 2^-48 of the unit's largest F.
template <int UN>
__device__ __forceinline__ void put_summary(const LayArgs& a, int32_t i, int64_t j, double f,
                                            double v) {
    const int l0 = (threadIdx.x % 64) / UN * UN;
    const double inf = __builtin_huge_val();
    const double f0 = __shfl(f, l0), f1 = __shfl(f, l0 + UN - 1);
    const double v0 = __shfl(v, l0), v1 = __shfl(v, l0 + UN - 1);
    const bool fin = f < inf;
    const double y = f0 < inf && f1 < inf && v1 > v0 ? (f1 - f0) / (v1 - v0) : 0.0;
    double x = fin ? f - y * (v - v0) : inf;
    double m = fin ? __builtin_fabs(f) : 0.0;
#pragma unroll
    for (int off = UN / 2; off > 0; off >>= 1) {
        x = __builtin_fmin(x, __shfl_xor(x, off));
        m = __builtin_fmax(m, __shfl_xor(m, off));
    }
    const int64_t q = j / UN;
    if (q >= a.nun) return;
    if (j % UN == 0) a.LN[(i & 1) * a.nun + q] = make_double2(x - 0x1p-48 * m, y);
    if (j % UN == UN - 1) a.FE[(i & 1) * a.nun + q] = f;
}

// Layer 2 (eq. apx_base) and the units' end values.
template <int UN>
__global__ __launch_bounds__(256) void k_layer_base(LayArgs a) {
    __shared__ double2 tab[kLog2Size];
    if (!live(a)) return;
    load_log2_table(tab);
    __syncthreads();
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t p = a.H.p, jj = min(j, p - 1);
    const double2 vn = make_double2(a.H.v[jj], a.H.N[jj]);
    const double2 ss = make_double2(a.H.S[jj], a.H.S2[jj]);
    double f = __builtin_huge_val();
    if (j < p) {
        if (j >= 1) {
            double C, P;
            cell_at(a.H, 0, j, tab, C, P);
            f = __builtin_fma(-a.lamp, P, 0.0 + C);
        }
        a.F[2 * a.ld + j] = f;
    }
    const int l1 = (threadIdx.x % 64) / UN * UN + UN - 1;
    const double v1 = __shfl(vn.x, l1), N1 = __shfl(vn.y, l1);
    const double v0 = __shfl(vn.x, l1 + 1 - UN), N0 = __shfl(vn.y, l1 + 1 - UN);
    // N_last - N_k against the line through the unit's ends
    const double nu = v1 > v0 ? (N1 - N0) / (v1 - v0) : 0.0;
    double lo = (N1 - vn.y) - nu * (v1 - vn.x), hi = lo;
#pragma unroll
    for (int off = UN / 2; off > 0; off >>= 1) {
        lo = __builtin_fmin(lo, __shfl_xor(lo, off));
        hi = __builtin_fmax(hi, __shfl_xor(hi, off));
    }
    lo = __builtin_fmin(lo, 0.0) - 0x1p-40 * (N1 - N0);
    hi = __builtin_fmax(hi, 0.0) + 0x1p-40 * (N1 - N0);
    const int64_t q = j / UN;
    if (q < a.nun) {
        double2* o = a.SB + kUnit * q;
        if (j % UN == 0) {
            o[2] = vn;
            o[3] = ss;
            o[4] = make_double2(lo, hi);
        }
        if (j % UN == UN - 1) {
            o[0] = vn;
            o[1] = ss;
        }
    }
    put_summary<UN>(a, 2, j, f, vn.x);
    if (blockIdx.x == 0) {  // (256 threads, and at most 255 layers)
        LayWork* W = work_of(a);
        if (threadIdx.x == 0) {
            a.K[a.nblk] = 0;
            W->all = 0;
            W->chain = 0;
            W->longest[0] = W->longest[1] = W->gone[0] = W->gone[1] = 0;
            W->fail = a.K + a.nblk;
        }
        W->limit[threadIdx.x] = work_limit(p, a.I, (int32_t)threadIdx.x, a.lamp == 0.0);
    }
}

// What the tests know of a set of columns.
struct Cols {
    double2 vn0, ss0;    // first column
    double2 vn1, ss1;    // last column
    double sN;           // sqrt(N S2) at the last column
    double nu, n0, n1;   // N_j - N_first lies in nu (v_j - v_first) + [n0, n1], in entries / d
    double alpha, beta;  // u_j <= alpha + beta (v_j - v_first); alpha = -inf: no column has a chain
    double aa;           // the larger |alpha + beta (v_j - v_first)| of the ends, 0 for -inf
    double db;           // v_last - v_first
};

// A lower bound of h(y) for a computed frequency y, clamped at 0 as the cell clamps it.
// h is negative above 1: exact frequencies stay below it, but the computed ones pass it
// where the prefix sums cancel (an entry of 1e16 times the others' spread takes their sums
// with it, and a grid's steps may lie far below an ulp of its values).
__device__ __forceinline__ float h_floor1(float y) {
    const float l = -__builtin_amdgcn_logf(y);
    return y > 1e-30f
               ? y * (__builtin_fmaf(-0x1p-18f, __builtin_fabsf(l), l) - 0x1p-20f)
               : 0.0f;
}
// The least h over [lo, hi]: h is concave, so it lies at an end.
__device__ __forceinline__ float h_floor(float lo, float hi) {
    return __builtin_fminf(h_floor1(lo), h_floor1(hi));
}
// A computed frequency passes an exact one (at most 1) by at most e.
__device__ __forceinline__ float freq_cap(double e) { return (float)(1.0 + 0x1p-20 + e); }

// The same over [lo, hi] whose ends move on straight lines from (lo0, hi0) to
// (lo1, hi1): h of each end is concave along the way, so the least h lies above
// the line between the two bounds added to f0 and f1.  That needs the ends above 0;
// there, and where an end passes 1 (the cap is the better bound), the least h over
// all of the range below the cap is added instead.
__device__ __forceinline__ void h_floor_line(double lo0, double hi0, double lo1, double hi1,
                                             float cap, float& f0, float& f1) {
    const float l0 = (float)lo0, l1 = (float)lo1, h0 = (float)hi0, h1 = (float)hi1;
    const float hm = __builtin_fmaxf(h0, h1), hc = __builtin_fminf(hm, cap);
    const bool ok = __builtin_fminf(l0, l1) > 1e-30f && hm <= 1.0f;
    f0 += h_floor(ok ? l0 : 0.0f, ok ? h0 : hc);
    f1 += h_floor(ok ? l1 : 0.0f, ok ? h1 : hc);
}

// False if predecessor (vn, ss) with F_{i-1} = f cannot hold the minimum of any
// of the columns.
__device__ __forceinline__ bool may_hold(double f, double2 vn, double2 ss, const Cols& c,
                                         double lamp, double rd) {
    const double n0 = c.vn0.y - vn.y, sa = c.ss0.x - ss.x;
    const double tu0 = __builtin_fma(-vn.x, n0, sa);
    const double C0 = __builtin_fma(c.vn0.x, tu0, __builtin_fma(vn.x, sa, -(c.ss0.y - ss.y)));
    const double vm = __builtin_fmax(__builtin_fabs(vn.x), __builtin_fabs(c.vn1.x));
    const double mg = 0x1p-44 * (__builtin_fma(vm * vm, c.vn1.y, c.ss1.y) + c.aa);
    const double eS = 0x1p-44 * __builtin_fma(vm, c.vn1.y, c.sN);
    const double tul = __builtin_fmax(tu0 - eS, 0.0);
    double base0 = f + (C0 - mg);
    double base1 = __builtin_fma(c.db, tul, base0);
    if (lamp != 0.0) {  // uniform
        const double r0 = __builtin_amdgcn_rcp(c.vn0.x - vn.x);
        const double r1 = __builtin_amdgcn_rcp(c.vn1.x - vn.x);
        const double rr = r0 * rd, e = eS * rr;
        const double U = tu0 * rr, D = __builtin_fma(c.vn0.x, n0, -sa) * rr;
        const double uA = __builtin_fma(U, 1.0 - 0x1p-20, -e);
        const double uB = __builtin_fma(U, 1.0 + 0x1p-20, e);
        const double dA = __builtin_fma(D, 1.0 - 0x1p-20, -e);
        const double dB = __builtin_fma(D, 1.0 + 0x1p-20, e);
        // dD/db = tu / (b - a)^2 between rA and rB, dU/db that of N less it
        const double tu1 = __builtin_fma(-vn.x, c.vn1.y - vn.y, c.ss1.x - ss.x);
        const double rA = tul * r1 * r1 * (rd * (1.0 - 0x1p-18));
        const double rB = (tu1 + eS) * r0 * r0 * (rd * (1.0 + 0x1p-18));
        const float cap = freq_cap(e);
        float phi0 = 0.0f, phi1 = 0.0f;
        h_floor_line(uA + c.n0, uB + c.n1, __builtin_fma(c.db, c.nu - rB, uA + c.n0),
                     __builtin_fma(c.db, c.nu - rA, uB + c.n1), cap, phi0, phi1);
        h_floor_line(dA, dB, __builtin_fma(c.db, rA, dA), __builtin_fma(c.db, rB, dB), cap, phi0,
                     phi1);
        base0 = __builtin_fma(lamp, (double)phi0 - 0x1p-40, base0);
        base1 = __builtin_fma(lamp, (double)phi1 - 0x1p-40, base1);
    }
    return base0 <= c.alpha || base1 <= __builtin_fma(c.beta, c.db, c.alpha);
}

// Four corners of a line's rectangle: as h_floor_line over both directions.
__device__ __forceinline__ void h_floor_rect(double lo, double hi, double lt, double ht, double lb,
                                             double hb, float cap, float (&f)[4]) {
    const float l[4] = {(float)lo, (float)(lo + lt), (float)(lo + lb), (float)(lo + lt + lb)};
    const float h[4] = {(float)hi, (float)(hi + ht), (float)(hi + hb), (float)(hi + ht + hb)};
    const float lm = __builtin_fminf(__builtin_fminf(l[0], l[1]), __builtin_fminf(l[2], l[3]));
    const float hm = __builtin_fmaxf(__builtin_fmaxf(h[0], h[1]), __builtin_fmaxf(h[2], h[3]));
    const float hc = __builtin_fminf(hm, cap);
    const bool ok = lm > 1e-30f && hm <= 1.0f;
#pragma unroll
    for (int x = 0; x < 4; x++) f[x] += h_floor(ok ? l[x] : 0.0f, ok ? h[x] : hc);
}

// False if no predecessor of a unit (its end values at o, F_{i-1} above the
// line ln) can hold the minimum of any of the columns.
__device__ __forceinline__ bool unit_may_hold(const double2* __restrict__ o, double2 ln,
                                              const Cols& c, double lamp, double rd) {
    const double2 vn1 = o[0], ss1 = o[1], vn0 = o[2];
    const double n0 = c.vn0.y - vn1.y, sa = c.ss0.x - ss1.x;
    const double tu0 = __builtin_fma(-vn1.x, n0, sa);
    const double td0 = __builtin_fma(c.vn0.x, n0, -sa);
    const double C0 = __builtin_fma(c.vn0.x, tu0,
                                    __builtin_fma(vn1.x, sa, -(c.ss0.y - ss1.y)));
    const double vm = __builtin_fmax(__builtin_fabs(vn0.x), __builtin_fabs(c.vn1.x));
    const double mg = 0x1p-44 * (__builtin_fma(vm * vm, c.vn1.y, c.ss1.y) + c.aa);
    const double eS = 0x1p-44 * __builtin_fma(vm, c.vn1.y, c.sN);
    const double tul = __builtin_fmax(tu0 - eS, 0.0), tdl = __builtin_fmax(td0 - eS, 0.0);
    const double da = vn1.x - vn0.x;
    // b[0]: last value and first column; +1: first value; +2: last column
    double b[4];
    b[0] = __builtin_fma(ln.y, da, ln.x) + (C0 - mg);
    b[1] = ln.x + (__builtin_fma(da, tdl, C0) - mg);
    b[2] = __builtin_fma(c.db, tul, b[0]);
    b[3] = __builtin_fma(c.db, __builtin_fma(da, n0, tul), b[1]);
    if (lamp != 0.0) {  // uniform
        const double2 ss0 = o[3], u01 = o[4];
        const double nu = vn1.y - vn0.y;  // entries passed from the last value to the first
        const double rS = __builtin_amdgcn_rcp(c.vn0.x - vn1.x);
        const double rL = __builtin_amdgcn_rcp(c.vn0.x - vn0.x);
        const double r1 = __builtin_amdgcn_rcp(c.vn1.x - vn0.x);
        const double rr = rS * rd, e = eS * rr;
        const double U = tu0 * rr, D = td0 * rr;
        const double lo = rd * (1.0 - 0x1p-18), hi = rd * (1.0 + 0x1p-18);
        // towards the first value: U rises by td / (b - a)^2, D by that of N less it
        const double td1 = __builtin_fma(c.vn0.x, c.vn0.y - vn0.y, -(c.ss0.x - ss0.x)) + eS;
        const double qA = da * (tdl * rL * rL * lo), qB = da * (td1 * rS * rS * hi);
        // towards the last column: D rises by tu / (b - a)^2, U by that of N less it
        const double tu1 = __builtin_fma(-vn0.x, c.vn1.y - vn0.y, c.ss1.x - ss0.x) + eS;
        const double rA = c.db * (tul * r1 * r1 * lo), rB = c.db * (tu1 * rS * rS * hi);
        const float cap = freq_cap(e);
        float phi[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        const double mc = c.db * c.nu, mu = nu * rd;
        h_floor_rect(__builtin_fma(U, 1.0 - 0x1p-20, c.n0 - e),
                     __builtin_fma(U, 1.0 + 0x1p-20, c.n1 + e), qA, qB, mc - rB, mc - rA, cap,
                     phi);
        h_floor_rect(__builtin_fma(D, 1.0 - 0x1p-20, __builtin_fma(u01.x, rd, -e)),
                     __builtin_fma(D, 1.0 + 0x1p-20, __builtin_fma(u01.y, rd, e)), mu - qB,
                     mu - qA, rA, rB, cap, phi);
#pragma unroll
        for (int x = 0; x < 4; x++) b[x] = __builtin_fma(lamp, (double)phi[x] - 0x1p-40, b[x]);
    }
    return __builtin_fmin(b[0], b[1]) <= c.alpha ||
           __builtin_fmin(b[2], b[3]) <= __builtin_fma(c.beta, c.db, c.alpha);
}

// The same for predecessors between the end values (vn1, ss1) and (vn0, ss0)
// with F_{i-1} >= f, from the ends of the ranges of U and D.
__device__ __forceinline__ bool span_may_hold(double f, double2 vn1, double2 ss1, double2 vn0,
                                              double2 ss0, const Cols& c, double lamp, double rd) {
    const double n0 = c.vn0.y - vn1.y, sa = c.ss0.x - ss1.x;
    const double tu0 = __builtin_fma(-vn1.x, n0, sa);
    const double C0 = __builtin_fma(c.vn0.x, tu0,
                                    __builtin_fma(vn1.x, sa, -(c.ss0.y - ss1.y)));
    const double vm = __builtin_fmax(__builtin_fabs(vn0.x), __builtin_fabs(c.vn1.x));
    const double mg = 0x1p-44 * (__builtin_fma(vm * vm, c.vn1.y, c.ss1.y) + c.aa);
    const double eS = 0x1p-44 * __builtin_fma(vm, c.vn1.y, c.sN);
    double base = f + (C0 - mg);
    if (lamp != 0.0) {  // uniform
        const double rS = __builtin_amdgcn_rcp(c.vn0.x - vn1.x) * rd;
        const double r1 = __builtin_amdgcn_rcp(c.vn1.x - vn0.x) * rd;
        const double e = eS * rS;
        const double n1 = c.vn1.y - vn0.y, s1 = c.ss1.x - ss0.x;
        const float cap = freq_cap(e);
        auto range = [&](double tl, double th) {  // between tl r1 and th rS
            return h_floor((float)__builtin_fma(tl * r1, 1.0 - 0x1p-20, -e),
                           __builtin_fminf((float)__builtin_fma(th * rS, 1.0 + 0x1p-20, e), cap));
        };
        const float phi = range(tu0, __builtin_fma(-vn0.x, n1, s1)) +
                          range(__builtin_fma(c.vn0.x, n0, -sa), __builtin_fma(c.vn1.x, n1, -s1));
        base = __builtin_fma(lamp, (double)phi - 0x1p-40, base);
    }
    const double rise = c.db * __builtin_fmax(tu0 - eS, 0.0);
    return base <= c.alpha || base + rise <= __builtin_fma(c.beta, c.db, c.alpha);
}

// F + Q of one predecessor and column, the cost as the other schedules form it.
__device__ __forceinline__ double candidate(double f, double2 vn, double2 ss, double cv, double cN,
                                            double cS, double cS2, double dd, double lamp,
                                            const double2* __restrict__ tab) {
    if (lamp == 0.0) return f + cell_c(vn.x, vn.y, ss.x, ss.y, cv, cN, cS, cS2);  // uniform
    double C, P;
    cell_terms(vn.x, vn.y, ss.x, ss.y, cv, cN, cS, cS2, dd, false, 0.0, tab, C, P);
    return f + __builtin_fma(-lamp, P, C);
}

__device__ __forceinline__ double uniform(double x) {
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)),
                            __builtin_amdgcn_readfirstlane(__double2loint(x)));
}
__device__ __forceinline__ double2 uniform(double2 x) {
    return make_double2(uniform(x.x), uniform(x.y));
}

// The line and the other facts of columns f0..l0 (uniform), lane x of each
// `lanes` holding column f0 + x: its u, v, N; in: it exists and has a chain;
// at0: the first lane that has one.
__device__ __forceinline__ Cols make_cols(const Hist& H, int64_t f0, int64_t l0, double u,
                                          double v, double N, bool in, int lanes, int at0,
                                          double rd) {
    Cols r;
    r.vn0 = uniform(make_double2(H.v[f0], H.N[f0]));
    r.ss0 = uniform(make_double2(H.S[f0], H.S2[f0]));
    r.vn1 = uniform(make_double2(H.v[l0], H.N[l0]));
    r.ss1 = uniform(make_double2(H.S[l0], H.S2[l0]));
    r.sN = __builtin_sqrt(r.vn1.y * r.ss1.y);
    r.db = r.vn1.x - r.vn0.x;
    const int at1 = (int)(l0 - f0);
    at0 = min(at0, at1);
    const double u0 = __shfl(u, at0), u1 = __shfl(u, at1);
    const double dv = __shfl(v, at1) - __shfl(v, at0);
    r.beta = uniform(at1 > at0 && u1 > u0 ? (u1 - u0) / dv : 0.0);
    double al = in ? u - r.beta * (v - r.vn0.x) : -__builtin_huge_val();
    r.nu = r.db > 0.0 ? (r.vn1.y - r.vn0.y) / r.db : 0.0;
    const double off_line = in ? (N - r.vn0.y) - r.nu * (v - r.vn0.x) : 0.0;
    double n0 = __builtin_fmin(off_line, 0.0), n1 = __builtin_fmax(off_line, 0.0);
    for (int off = lanes / 2; off > 0; off >>= 1) {
        al = __builtin_fmax(al, __shfl_xor(al, off));
        n0 = __builtin_fmin(n0, __shfl_xor(n0, off));
        n1 = __builtin_fmax(n1, __shfl_xor(n1, off));
    }
    r.alpha = uniform(al);
    r.aa = r.alpha > -__builtin_huge_val()
               ? __builtin_fmax(__builtin_fabs(r.alpha),
                                __builtin_fabs(__builtin_fma(r.beta, r.db, r.alpha)))
               : 0.0;
    r.nu = uniform(r.nu * rd);
    // (rounding of the line: 2^-40 of the largest step)
    r.n0 = uniform((n0 - 0x1p-40 * (r.vn1.y - r.vn0.y)) * rd);
    r.n1 = uniform((n1 + 0x1p-40 * (r.vn1.y - r.vn0.y)) * rd);
    return r;
}

// One layer: CW groups of 16 columns per workgroup, the predecessors of each
// shared between KS wavefronts.  Lane: column c = lane % 16 of the wavefront's
// group, predecessor slot kq = lane / 16.  SUP: 8 units are tested together
// before each by itself.  A unit is as many predecessors as a workgroup has
// columns.
template <int CW, int KS, bool SUP>
__global__ __launch_bounds__(64 * CW * KS) void k_layer(LayArgs a, int32_t i) {
    constexpr int W = CW * KS, T = 64 * W, NC = kGC * CW;
    constexpr int UN = NC, UW = kSB / UN;  // units in a wavefront's 64 predecessors
    __shared__ double2 tab[kLog2Size];
    __shared__ double2 bA[W][kSB], bB[W][kSB];  // (v, N), (S, S2) of the predecessors left
    __shared__ double bF[W][kSB];
    __shared__ double red[KS][NC];
    __shared__ double rv[2][W];
    __shared__ int32_t rq[2][W];
    __shared__ uint16_t slist[SUP ? kList : 1];
    __shared__ uint16_t list[kList], glist[CW > 1 ? CW : 1][kList], clist[CW][kList];
    __shared__ int32_t nslist, nlist, nglist[CW], nclist[CW];
    __shared__ uint32_t steps[W];
    {
        // three loads in flight together (gone: written by earlier launches only)
        const int32_t run = a.runp ? *a.runp : 1;
        LayWork* work = work_of(a);
        const uint32_t gone = work->gone[(i - 1) & 1];
        if (a.lampp) a.lamp = *a.lampp;
        if (run == 0 || gone != 0) {  // uniform
            if (gone != 0 && blockIdx.x == 0 && threadIdx.x == 0) work->gone[i & 1] = 1;
            return;
        }
    }
    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int cg = wave % CW, sl = wave / CW;
    const int c = lane % kGC, kq = lane / kGC;
    const int64_t p = a.H.p;
    const double lamp = a.lamp, dd = a.H.dd, rd = 1.0 / dd;
    // the last column blocks have the most predecessors: they start first
    const int64_t J = (int64_t)gridDim.x - 1 - blockIdx.x;
    const int64_t j0 = J * NC;
    const int64_t j1 = min(j0 + NC, p) - 1;
    const int64_t jg = j0 + kGC * cg;  // the group's first column
    const int64_t j = jg + c;
    const int64_t jj = min(j, p - 1);
    const bool in = j < p && j >= i - 1;  // the column exists and has a chain
    const double cv = a.H.v[jj], cN = a.H.N[jj], cS = a.H.S[jj], cS2 = a.H.S2[jj];
    const double* Fp = a.F + (int64_t)(i - 1) * a.ld;
    const double* FEp = a.FE + ((i - 1) & 1) * a.nun;
    const double2* LNp = a.LN + ((i - 1) & 1) * a.nun;
    // predecessors from kd = 64 [j0 / 64] on and the 64 before them are near, the
    // qn units before those are far
    const int64_t kd = j0 / kSB * kSB;
    const int64_t kn = kd >= kSB ? kd - kSB : 0, qn = kn / UN;
    if (lamp != 0.0) load_log2_table(tab);
    double best = __builtin_huge_val();
    auto eval = [&](double f, double2 vn, double2 ss) {
        best = __builtin_fmin(best, candidate(f, vn, ss, cv, cN, cS, cS2, dd, lamp, tab));
    };
    auto eval_at = [&](int64_t k) {
        eval(Fp[k], make_double2(a.H.v[k], a.H.N[k]), make_double2(a.H.S[k], a.H.S2[k]));
    };
    // the least over the wavefronts of a column, in every lane of the column
    auto merge = [&](bool again) {
        best = __builtin_fmin(best, __shfl_xor(best, 16));
        best = __builtin_fmin(best, __shfl_xor(best, 32));
        if (again) __syncthreads();
        if (kq == 0) red[sl][kGC * cg + c] = best;
        __syncthreads();
#pragma unroll
        for (int s = 0; s < KS; s++) best = __builtin_fmin(best, red[s][kGC * cg + c]);
    };
    if (tid == 0) {
#pragma unroll
        for (int w = 0; w < W; w++) steps[w] = 0;
        if (blockIdx.x == 0) work_of(a)->longest[(i + 1) & 1] = 0;
    }
    __syncthreads();  // the table
    // the far units that are best for columns j0 and j1, judged by their last
    // predecessors; the end of each is the middle of 128 predecessors, from kA and
    // from kB >= kA on
    int64_t kA = 0, kB = 0;
    if (qn > 0) {
        const double bv[2] = {a.H.v[j0], a.H.v[j1]}, bN[2] = {a.H.N[j0], a.H.N[j1]};
        const double bS[2] = {a.H.S[j0], a.H.S[j1]}, bS2[2] = {a.H.S2[j0], a.H.S2[j1]};
        constexpr int ST = SUP ? 8 : UW;
        double bb[2] = {__builtin_huge_val(), __builtin_huge_val()};
        int32_t bq[2] = {0, 0};
        auto look = [&](int64_t q) {
            const double f = FEp[q];
            const double2 qa = a.SB[kUnit * q], qb = a.SB[kUnit * q + 1];
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const double v = candidate(f, qa, qb, bv[e], bN[e], bS[e], bS2[e], dd, lamp, tab);
                if (v < bb[e]) {
                    bb[e] = v;
                    bq[e] = (int32_t)q;
                }
            }
        };
        auto fold = [&]() {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
                for (int e = 0; e < 2; e++) {
                    const double ov = __shfl_xor(bb[e], off);
                    const int32_t oq = __shfl_xor(bq[e], off);
                    if (ov < bb[e]) {
                        bb[e] = ov;
                        bq[e] = oq;
                    }
                }
            }
        };
        for (int64_t q = (int64_t)tid * ST + ST - 1; q < qn; q += (int64_t)T * ST) look(q);
        fold();
        if (lane < 2) {
            rv[lane][wave] = lane ? bb[1] : bb[0];
            rq[lane][wave] = lane ? bq[1] : bq[0];
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 2; e++) {
            bb[e] = rv[e][0];
            bq[e] = rq[e][0];
            for (int w = 1; w < W; w++)
                if (rv[e][w] < bb[e]) {
                    bb[e] = rv[e][w];
                    bq[e] = rq[e][w];
                }
        }
        if (SUP) {  // the units around them, in every wavefront
            const int64_t q = (lane < 32 ? bq[0] : bq[1]) - 15 + (lane & 31);
            if (q >= 0 && q < qn) look(q);
            fold();
        }
        const int qa = __builtin_amdgcn_readfirstlane(min(bq[0], bq[1]));
        const int qb = __builtin_amdgcn_readfirstlane(max(bq[0], bq[1]));
        kA = max<int64_t>((int64_t)(qa + 1) * UN - kSB, 0);
        kB = max<int64_t>((int64_t)(qb + 1) * UN - kSB, 0);
    }
    // first bounds: the group's own columns (k < j), and predecessors spread
    // over the 128 from kA and from kB on, those between (columns far apart, as the
    // last of a heavy tail) and the 64 before kd
    for (int y = sl; y < kGC / 4; y += KS) {
        const int64_t k = jg + 4 * y + kq;
        if (k < j && j < p) eval_at(k);
    }
    if (sl == 0 && qn > 0) {
        const int64_t k = kA + 32 * kq + 31;
        if (k < kn) eval_at(k);
    }
    if (kB > kA) {  // uniform
        if (sl == KS - 1 && kB + 32 * kq + 31 < kn) eval_at(kB + 32 * kq + 31);
        if (kB > kA + 2 * kSB)
            for (int y = 4 * sl + kq; y < 32; y += 4 * KS) eval_at(kA + (kB - kA) * (y + 1) / 33);
    }
    if (sl == KS - 1 && kd > 0) eval_at(kd - 1 - 16 * kq);
    merge(false);
    Cols g = make_cols(a.H, min(jg, p - 1), min(jg + kGC - 1, p - 1), best, cv, cN, in, kGC,
                       (int)max<int64_t>(0, i - 1 - jg), rd);
    // The predecessors of a block (one per lane) that may hold a minimum of the
    // group, packed, then evaluated four side by side.
    double2 vn, ss;
    double f;
    auto fetch = [&](int64_t kk) {
        const int64_t k = min(kk, p - 1);
        vn = make_double2(a.H.v[k], a.H.N[k]);
        ss = make_double2(a.H.S[k], a.H.S2[k]);
        f = Fp[k];
    };
    double2* wA = bA[wave];
    double2* wB = bB[wave];
    double* wF = bF[wave];
    auto pick = [&](bool keep) {
        const uint64_t mask = __ballot(keep);
        if (mask) {
            const int at = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (keep) {
                wA[at] = vn;
                wB[at] = ss;
                wF[at] = f;
            }
        }
        return __builtin_popcountll(mask);
    };
    // Thread 0: the workgroup's steps so far (see LayWork).
    LayWork* work = work_of(a);
    auto report = [&]() {
        uint32_t most = 0, sum = 0;
#pragma unroll
        for (int w = 0; w < W; w++) {
            most = max(most, steps[w]);
            sum += steps[w];
        }
        if ((int64_t)most < p >> (a.I < 64 ? 5 : a.I < 128 ? 6 : 7)) return;
        uint32_t had = fresh(&work->longest[i & 1]);
        if (most > had) {
            had = atomicMax(&work->longest[i & 1], most);
            if (most > had) atomicAdd(&work->chain, most - had);
        }
        if (blockIdx.x % kSample == 0) {
            atomicAdd(&work->all, (unsigned long long)kSample * sum);
        }
        if (fresh(&work->chain) + fresh(&work->all) / kCrowd > work->limit[i]) {
            *work->fail = kSweepGaveUp;
            __hip_atomic_store(&work->gone[i & 1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    auto run = [&](int ns) {
        if (ns == 0) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll 2
        for (int y = 0; y < ns; y += 4) {
            const int z = min(y + kq, ns - 1);
            eval(wF[z], wA[z], wB[z]);
        }
        __builtin_amdgcn_wave_barrier();
    };
    // the 128 predecessors from kA on, those from kB on, the 64 before kd, and from
    // kd to the group
    const int64_t kB0 = max(kB, kA + 2 * kSB), kB1 = min(kB + 2 * kSB, kn);
    for (int y = sl; y < 6; y += KS) {
        const int64_t k0 = y <= 1 ? kA + kSB * y : y == 2 ? kd - kSB : y == 3 ? kd
                                                 : kB0 + kSB * (y - 4);
        const int64_t ke = y <= 1 ? min(kA + 2 * kSB, kn) : y == 2 ? kd : y == 3 ? jg : kB1;
        if (k0 < 0 || k0 >= ke || jg >= p) continue;  // uniform
        fetch(k0 + lane);
        run(pick(k0 + lane < ke && may_hold(f, vn, ss, g, lamp, rd)));
    }
    merge(true);
    if (qn > 0) {
        g = make_cols(a.H, min(jg, p - 1), min(jg + kGC - 1, p - 1), best, cv, cN, in, kGC,
                      (int)max<int64_t>(0, i - 1 - jg), rd);
        Cols b = g;
        if constexpr (CW > 1) {
            const int64_t jl = j0 + lane, jc = min(jl, p - 1);
            double ul = __builtin_huge_val();
            if (lane < NC) {
                ul = red[0][lane];
#pragma unroll
                for (int s = 1; s < KS; s++) ul = __builtin_fmin(ul, red[s][lane]);
            }
            b = make_cols(a.H, j0, j1, ul, a.H.v[jc], a.H.N[jc],
                          lane < NC && jl < p && jl >= i - 1, 64,
                          (int)max<int64_t>(0, i - 1 - j0), rd);
        }
        // the wavefronts of a group test every unit that is left against it when
        // few are; against each of its columns first when many are (columns far
        // apart, as the last of a heavy tail)
        Cols one;
        one.vn0 = one.vn1 = make_double2(cv, cN);
        one.ss0 = one.ss1 = make_double2(cS, cS2);
        one.sN = __builtin_sqrt(cN * cS2);
        one.nu = one.n0 = one.n1 = one.beta = one.db = 0.0;
        one.alpha = in ? best : -__builtin_huge_val();
        one.aa = in ? __builtin_fabs(best) : 0.0;
        // one round: at most kList units, unit(x) for x < nx
        auto round = [&](int nx, auto unit) {
            __syncthreads();  // the lists are free
            if (tid == 0) nlist = 0;
            if (tid < CW) nglist[tid] = nclist[tid] = 0;
            __syncthreads();
            uint32_t done = 0;
            for (int x = tid; x < nx; x += T) {
                const int64_t q = unit(x), dA = q * UN - kA, dB = q * UN - kB;
                if (q < qn && (dA < 0 || dA >= 2 * kSB) && (dB < 0 || dB >= 2 * kSB) &&
                    unit_may_hold(a.SB + kUnit * q, LNp[q], b, lamp, rd))
                    list[atomicAdd(&nlist, 1)] = (uint16_t)x;
            }
            __syncthreads();
            const int nl = nlist;
            const uint16_t* todo = list;
            int n = nl;
            if constexpr (CW > 1) {
                if (nl > 0) {  // uniform in the workgroup
                    for (int x = sl * 64 + lane; x < nl; x += 64 * KS) {
                        const int o = list[x];
                        const int64_t q = unit(o);
                        if (unit_may_hold(a.SB + kUnit * q, LNp[q], g, lamp, rd))
                            glist[cg][atomicAdd(&nglist[cg], 1)] = (uint16_t)o;
                    }
                    __syncthreads();
                    todo = glist[cg];
                    n = nglist[cg];
                }
            }
            if (nl > kMany) {  // uniform in the workgroup
                // many are left: each unit against each column, 4 units at a time
                for (int x = 4 * sl; x < n; x += 4 * KS) {
                    done += 4;
                    bool any = false;
                    int o = 0;
                    if (x + kq < n) {
                        o = todo[x + kq];
                        const int64_t q = unit(o);
                        any = unit_may_hold(a.SB + kUnit * q, LNp[q], one, lamp, rd);
                    }
                    const uint64_t mask = __ballot(any);
                    if (c == 0 && ((mask >> (kGC * kq)) & 0xffffu))
                        clist[cg][atomicAdd(&nclist[cg], 1)] = (uint16_t)o;
                }
                __syncthreads();
                todo = clist[cg];
                n = nclist[cg];
            }
            // UW units at a time, one predecessor per lane
            auto next = [&](int x) {
                const int y = x * UW + lane / UN;
                const int64_t q = unit(todo[min(y, n - 1)]);
                fetch(q * UN + lane % UN);
            };
            const int nw = (n + UW - 1) / UW;
            if (sl < nw) next(sl);
            for (int x = sl; x < nw; x += KS) {
                const int ns = pick(x * UW + lane / UN < n && may_hold(f, vn, ss, g, lamp, rd));
                // the next loads are in flight while these are evaluated
                if (x + KS < nw) next(x + KS);
                run(ns);
                done += 4 + (uint32_t)(ns + 3) / 4;
            }
            if (lane == 0) steps[wave] += done;
        };
        if constexpr (SUP) {
            const int64_t nsup = (qn + 7) / 8;
            for (int64_t sc = 0; sc < nsup; sc += kList) {
                __syncthreads();
                if (tid == 0) nslist = 0;
                __syncthreads();
                const int64_t se = min(sc + kList, nsup);
                for (int64_t s8 = sc + tid; s8 < se; s8 += T) {
                    const int64_t q0 = 8 * s8, q1 = min(q0 + 7, qn - 1);
                    double m = __builtin_huge_val();
#pragma unroll
                    for (int z = 0; z < 8; z++) {
                        const int64_t q = min(q0 + z, q1);
                        const double2 ln = LNp[q];
                        const double da = a.SB[kUnit * q].x - a.SB[kUnit * q + 2].x;
                        m = __builtin_fmin(m, __builtin_fmin(ln.x, __builtin_fma(ln.y, da, ln.x)));
                    }
                    if (span_may_hold(m, a.SB[kUnit * q1], a.SB[kUnit * q1 + 1],
                                      a.SB[kUnit * q0 + 2], a.SB[kUnit * q0 + 3], b, lamp, rd))
                        slist[atomicAdd(&nslist, 1)] = (uint16_t)(s8 - sc);
                }
                __syncthreads();
                const int ns = nslist;
                for (int s0 = 0; s0 < ns; s0 += kList / 8)
                    round(8 * min(kList / 8, ns - s0), [&](int x) {
                        return 8 * (sc + slist[s0 + x / 8]) + x % 8;
                    });
            }
        } else {
            for (int64_t qc = 0; qc < qn; qc += kList)
                round((int)min<int64_t>(kList, qn - qc), [&](int x) { return qc + x; });
        }
        merge(true);
    }
    if (tid < 64) {
        const int64_t jo = j0 + tid;
        double fo = __builtin_huge_val();
        if (tid < NC && jo < p) {
#pragma unroll
            for (int s = 0; s < KS; s++) fo = __builtin_fmin(fo, red[s][tid]);
            a.F[(int64_t)i * a.ld + jo] = fo;
        }
        if (tid < NC) put_summary<UN>(a, i, jo, fo, a.H.v[min(jo, p - 1)]);
        if (tid == 0 && qn > 0) report();
    }
}

template <int CW, int KS, bool SUP>
hipError_t launch_all(LayArgs a, hipStream_t st) {
    constexpr int NC = kGC * CW;
    a.nun = (a.H.p + NC - 1) / NC;
    k_layer_base<kGC * CW><<<(unsigned)((a.H.p + 255) / 256), 256, 0, st>>>(a);
    for (int32_t i = 3; i <= a.I; i++)
        k_layer<CW, KS, SUP><<<(unsigned)((a.H.p + NC - 1) / NC), 64 * CW * KS, 0, st>>>(a, i);
    return hipGetLastError();
}

}  // namespace

namespace {

// The work words, the units' end values, then the two rows of lines and of unit-end values (a
// unit is at least 16 values): 8 bytes a value and a little, where rows 0 and 1 of F have 16.
size_t scratch_bytes(int64_t p) {
    const size_t nun = (size_t)(p + kGC - 1) / kGC;
    return kWorkBytes + align256(16 * kUnit * nun) + align256(2 * 16 * nun) +
           align256(2 * 8 * nun);
}

}  // namespace

hipError_t launch_layers(const SweepSolve& S, hipStream_t st) {
    LayArgs a;
    a.H = S.H;
    a.F = S.F;
    a.nblk = (S.H.p + kSB - 1) / kSB;
    a.nun = (S.H.p + kGC - 1) / kGC;
    if (scratch_bytes(S.H.p) > 2 * sizeof(double) * (size_t)S.ld) return hipErrorInvalidValue;
    char* o = reinterpret_cast<char*>(S.F) + kWorkBytes;
    a.SB = reinterpret_cast<double2*>(o);
    o += align256(16 * kUnit * (size_t)a.nun);
    a.LN = reinterpret_cast<double2*>(o);
    o += align256(2 * 16 * (size_t)a.nun);
    a.FE = reinterpret_cast<double*>(o);
    a.K = S.K;
    a.ld = S.ld;
    a.I = S.I;
    a.lamp = S.lamp;
    a.lampp = S.lampp;
    a.runp = S.runp;
    // Below about 48 000 values the blocks of 64 columns are too few to share the
    // work evenly: blocks of 16 (32 763 values, 32 layers: 2.4 ms against 4.2; at
    // 65 500 and 64 layers 12.2 against 8.3).
    return S.H.p < kWideP ? launch_all<1, 4, false>(a, st) : launch_all<4, 1, true>(a, st);
}

}  // namespace ecasq
