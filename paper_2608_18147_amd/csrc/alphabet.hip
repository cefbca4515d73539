// Permissible alphabets P != X (App. D): the DP's candidate values are a grid
// over [min X, max X] instead of the distinct input values, and the interval
// quantities come from the input's prefix count, sum and sum of squares at the
// grid points (the entries <= p).  With min X and max X as the first and last
// grid points, every later step (DP, search, refinement, metrics, rounding)
// runs unchanged on the grid.
//
//   uniform  p_k = min X + k * ((max X - min X) / (m - 1)) for 0 < k < m-1,
//            each operation rounded to nearest, p_0 = min X, p_{m-1} = max X;
//   quantile p_k = the input value at rank floor(k (d - 1) / (m - 1)).
// A point equal to its predecessor (or, for the uniform grid, an inner point
// not below max X) is dropped.  One workgroup walks the grid in tiles of 4096 points,
// a tile-wide scan of the kept flags placing the survivors.
#include "device.hpp"
#include "launch.hpp"

namespace ecasq {

namespace {

constexpr int kAT = 1024;
// Points of a thread, and the one before them.  Their binary searches go level by
// level together: a search is a chain of about 20 loads, and one after another (and each
// point's predecessor again) they took 97 us for 4096 points of 2^20 values.
constexpr int kAP = 4;
constexpr int kAN = kAP + 1;

// For each q: the last index i with v[i] <= q (v ascending, v[0] <= q).
__device__ __forceinline__ void last_le(const double* v, int64_t n, const double (&q)[kAN],
                                        int64_t (&lo)[kAN]) {
    int64_t hi[kAN];
#pragma unroll
    for (int u = 0; u < kAN; u++) {
        lo[u] = 0;
        hi[u] = n - 1;
    }
    for (int64_t w = n - 1; w > 0; w >>= 1) {
        double x[kAN];
#pragma unroll
        for (int u = 0; u < kAN; u++) x[u] = v[lo[u] + (hi[u] - lo[u] + 1) / 2];
#pragma unroll
        for (int u = 0; u < kAN; u++) {
            const int64_t mid = lo[u] + (hi[u] - lo[u] + 1) / 2;
            if (lo[u] < hi[u]) {
                if (x[u] <= q[u]) lo[u] = mid;
                else hi[u] = mid - 1;
            }
        }
    }
}

// For each r: the first index i with N[i] > r (N ascending integer counts, N[n-1] > r).
__device__ __forceinline__ void first_gt(const double* N, int64_t n, const double (&r)[kAN],
                                         int64_t (&lo)[kAN]) {
    int64_t hi[kAN];
#pragma unroll
    for (int u = 0; u < kAN; u++) {
        lo[u] = 0;
        hi[u] = n - 1;
    }
    for (int64_t w = n - 1; w > 0; w >>= 1) {
        double x[kAN];
#pragma unroll
        for (int u = 0; u < kAN; u++) x[u] = N[lo[u] + (hi[u] - lo[u]) / 2];
#pragma unroll
        for (int u = 0; u < kAN; u++) {
            const int64_t mid = lo[u] + (hi[u] - lo[u]) / 2;
            if (lo[u] < hi[u]) {
                if (x[u] > r[u]) hi[u] = mid;
                else lo[u] = mid + 1;
            }
        }
    }
}

struct AlphaArgs {
    const double *v, *N, *S, *S2;  // distinct input values and their prefix sums
    int64_t px;                    // number of distinct input values (>= 2)
    int64_t d;
    int64_t m;                     // requested grid size (2 <= m <= d)
    int32_t kind;                  // 1 uniform, 2 quantile
    double *gv, *gN, *gS, *gS2;    // the grid and the prefix sums at its points
    int64_t* count;                // number of grid points kept
};

// Grid points k0, k0 + 1, ..: their values and the indices of the last input values
// <= them (k clamped to the grid).
__device__ __forceinline__ void points(const AlphaArgs& a, int64_t k0, double (&q)[kAN],
                                       int64_t (&idx)[kAN]) {
    if (a.kind == 1) {
        const double lo = a.v[0], hi = a.v[a.px - 1];
        const double step = (hi - lo) / (double)(a.m - 1);
#pragma unroll
        for (int u = 0; u < kAN; u++) {
            const int64_t k = min(max<int64_t>(k0 + u, 0), a.m - 1);
            q[u] = k == 0 ? lo : k == a.m - 1 ? hi : lo + (double)k * step;
        }
        last_le(a.v, a.px, q, idx);
    } else {
        double r[kAN];
#pragma unroll
        for (int u = 0; u < kAN; u++) {
            const int64_t k = min(max<int64_t>(k0 + u, 0), a.m - 1);
            r[u] = (double)((k * (a.d - 1)) / (a.m - 1));
        }
        first_gt(a.N, a.px, r, idx);
#pragma unroll
        for (int u = 0; u < kAN; u++) q[u] = a.v[idx[u]];
    }
}

__global__ __launch_bounds__(kAT) void k_alphabet(AlphaArgs a) {
    constexpr int W = kAT / 64;
    __shared__ int32_t part[2][W];
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    int64_t base = 0;
    int odd = 0;
    const double hi = a.v[a.px - 1];
    for (int64_t t0 = 0; t0 < a.m; t0 += kAT * kAP, odd ^= 1) {
        const int64_t k0 = t0 + (int64_t)kAP * tid;
        double q[kAN];
        int64_t idx[kAN];
        points(a, k0 - 1, q, idx);
        bool keep[kAP];
        int32_t own = 0;
#pragma unroll
        for (int u = 0; u < kAP; u++) {
            const int64_t k = k0 + u;
            // the points rise with k, so the predecessor is the largest
            // point kept so far or a repeat of it
            keep[u] = k < a.m && (k == 0 || (a.kind == 1 && k == a.m - 1) ||
                                  (a.kind == 1 ? q[u + 1] > q[u] && q[u + 1] < hi
                                               : idx[u + 1] > idx[u]));
            own += keep[u];
        }
        int32_t at = own;  // inclusive scan over the wavefront, then the wavefronts
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t y = __shfl_up(at, off);
            if (lane >= off) at += y;
        }
        if (lane == 63) part[odd][wave] = at;
        __syncthreads();
        int32_t total = 0;
#pragma unroll
        for (int w = 0; w < W; w++) {
            const int32_t y = part[odd][w];
            at += w < wave ? y : 0;
            total += y;
        }
        int64_t o = base + at - own;
#pragma unroll
        for (int u = 0; u < kAP; u++) {
            if (keep[u]) {
                a.gv[o] = q[u + 1];
                a.gN[o] = a.N[idx[u + 1]];
                a.gS[o] = a.S[idx[u + 1]];
                a.gS2[o] = a.S2[idx[u + 1]];
                o++;
            }
        }
        base += total;
    }
    if (tid == 0) *a.count = base;
}

}  // namespace

hipError_t launch_alphabet(int32_t kind, int64_t m, int64_t d, const double* v, const double* N,
                           const double* S, const double* S2, int64_t px, double* gv, double* gN,
                           double* gS, double* gS2, int64_t* count, hipStream_t st) {
    if ((kind != 1 && kind != 2) || m < 2 || m > d || px < 2) return hipErrorInvalidValue;
    AlphaArgs a{v, N, S, S2, px, d, m, kind, gv, gN, gS, gS2, count};
    k_alphabet<<<1, kAT, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace ecasq
