// dp_APX (Sec. 5, eq. apx_base / apx_rec) for one multiplier and few values (p <=
// 4096): every pair's cost Q = C - lambda' Phi is formed once and stays in
// registers, and a layer is an addition and a minimum for each of them.
//
// p^2 / 2 costs of 8 bytes are 67 MB at p = 4096, half of the chip's registers.
// One launch, workgroups of 1024 threads; a workgroup owns W columns, a thread R
// predecessors (k = thread + 1024 r) against each of them.  Layer by layer it
// takes F_{i-1} of its predecessors, reduces the candidates of each column over
// the workgroup and writes F_i of its columns.  The values themselves are the
// signal: every entry of rows 3..I holds a NaN that no layer produces until its
// value is stored, and a thread polls the entries that it needs (64-bit atomics
// at device scope, so there is nothing to fence).
//
// A workgroup takes its columns by ticket, in the order in which workgroups start, and
// F_{i-1}[k] is needed for k below the columns alone: it only ever waits for
// workgroups that have started, whatever else runs on the device.  Workgroups
// of low columns need few others, run ahead and leave their place to those of
// high columns.  A wait that finds nothing for about a second sets the failure
// word, and every later wait then ends at once.
//
// Columns per workgroup: 8 while that gives at most 256 workgroups (p <= 2048);
// up to 3072, 32 of the first 1024, 16 of the next 1024 and 8 beyond (32 costs in a
// thread of each).  Above, that would be up to 352 workgroups for 256 CUs, the last of
// them after the first have ended: there workgroups of 512 threads hold up to 96
// costs in a thread (half as many threads keep half as much beside them), 64 to 8
// columns, 254 workgroups at 4096.
//
// What bounds it: the way of a value from one workgroup to another and the
// reduction, 1.6 us a layer at 1024 values, 2.6 at 3071 and about 4 at 4096.  A
// solve of 4096 values and 64 layers takes about 240 us (275 with the workgroups of
// 1024 threads, in two rounds) where the column-block sweep takes 810, one of 1024
// and 16 layers 25 where it takes 86.
#include "device.hpp"
#include "launch.hpp"

namespace ecasq {

namespace {

constexpr int kHT = 1024;
constexpr int kHTBig = 512;
constexpr uint64_t kUnset = ~0ull;
// polls before a wait gives up (about a second)
constexpr uint32_t kHeldSpin = 1u << 20;
constexpr int64_t kNarrowP = 2048;
constexpr int64_t kBigP = 3072;

struct HeldArgs {
    Hist H;
    double* F;    // [I+1][ld]
    int32_t* K;   // K[nblk]: the failure word; K[nblk + 1]: the next ticket
    int64_t ld, nblk;
    int32_t I;
    double lamp;
    const double* lampp;
    const int32_t* runp;
};

__device__ __forceinline__ bool live(HeldArgs& a) {
    if (a.runp && *a.runp == 0) return false;
    if (a.lampp) a.lamp = *a.lampp;
    return true;
}

// Layer 2 (eq. apx_base) in row 2, kUnset in the rows of the other layers.
__global__ __launch_bounds__(256) void k_held_base(HeldArgs a) {
    __shared__ double2 tab[kLog2Size];
    if (!live(a)) return;
    const int32_t i = 2 + (int32_t)blockIdx.y;
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i == 2) {  // uniform
        load_log2_table(tab);
        __syncthreads();
        if (j == 0) a.K[a.nblk] = a.K[a.nblk + 1] = 0;
    }
    if (j >= a.H.p) return;
    double* at = a.F + (int64_t)i * a.ld + j;
    if (i > 2) {
        *reinterpret_cast<uint64_t*>(at) = kUnset;
        return;
    }
    double f = __builtin_huge_val();
    if (j >= 1) {
        double C, P;
        cell_at(a.H, 0, j, tab, C, P);
        f = __builtin_fma(-a.lamp, P, 0.0 + C);
    }
    *at = f;
}

struct HeldSmem {
    double2 tab[kLog2Size];
    // each row of 16 lanes' minima of W columns (layer parity)
    double part[2][2048];
    int32_t ticket;
};

template <int CTRL>
__device__ __forceinline__ double lane_move(double x) {
    return __hiloint2double(
        __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true),
        __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor8 = 0x128;  // quad permutations, row rotation by 8

// F_{i-1} of the thread's predecessors, +inf for those at or past kend.
template <int T, int R>
__device__ __forceinline__ void await(const HeldArgs& a, const double* Fp, int64_t kend,
                                      double (&f)[R]) {
    uint64_t b[R];
    for (uint32_t spin = 0;; spin++) {
        bool miss = false;
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int64_t k = (int64_t)threadIdx.x + T * r;
            b[r] = 0x7FF0000000000000ull;
            if (k < kend)
                b[r] = __hip_atomic_load(reinterpret_cast<const uint64_t*>(Fp + k),
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int r = 0; r < R; r++) miss |= b[r] == kUnset;
        if (!miss) break;
        if (spin % 64 == 63) {
            const bool failed = __hip_atomic_load(a.K + a.nblk, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT) != 0;
            if (failed || spin >= kHeldSpin) {
                __hip_atomic_store(a.K + a.nblk, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int r = 0; r < R; r++)
                    if (b[r] == kUnset) b[r] = 0x7FF0000000000000ull;
                break;
            }
        }
        __builtin_amdgcn_s_sleep(1);
    }
#pragma unroll
    for (int r = 0; r < R; r++) f[r] = __longlong_as_double((long long)b[r]);
}

// Layers 3..I of columns c0 .. c0 + W - 1 (c0 + W - 1 <= T R).
template <int T, int W, int R>
__device__ __forceinline__ void held(const HeldArgs& a, int64_t c0, HeldSmem& sm) {
    constexpr int ROWS = T / 16;  // rows of 16 lanes
    static_assert(ROWS * W <= 2048 && W / 8 <= T / 64, "a workgroup's minima and their waves");
    const int tid = threadIdx.x, lane = tid % 64;
    const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int64_t p = a.H.p;
    const double inf = __builtin_huge_val();
    double q[R][W];
    {
        double v[R], N[R], S[R], S2[R];
#pragma unroll
        for (int r = 0; r < R; r++) {
            const int64_t k = min((int64_t)tid + T * r, p - 1);
            v[r] = a.H.v[k];
            N[r] = a.H.N[k];
            S[r] = a.H.S[k];
            S2[r] = a.H.S2[k];
        }
#pragma unroll
        for (int c = 0; c < W; c++) {
            const int64_t j = c0 + c, jj = min(j, p - 1);
            const double jv = a.H.v[jj], jN = a.H.N[jj], jS = a.H.S[jj], jS2 = a.H.S2[jj];
#pragma unroll
            for (int r = 0; r < R; r++) {
                double e;
                if (a.lamp == 0.0) {  // uniform
                    e = cell_c(v[r], N[r], S[r], S2[r], jv, jN, jS, jS2);
                } else {
                    double C, P;
                    cell_terms(v[r], N[r], S[r], S2[r], jv, jN, jS, jS2, a.H.dd, false, 0.0,
                               sm.tab, C, P);
                    e = __builtin_fma(-a.lamp, P, C);
                }
                q[r][c] = (int64_t)tid + T * r < j && j < p ? e : inf;
            }
        }
    }
    const int64_t kend = min(c0 + W - 1, p);
    for (int32_t i = 3; i <= a.I; i++) {
        double* part = sm.part[i & 1];
        double f[R];
        await<T, R>(a, a.F + (int64_t)(i - 1) * a.ld, kend, f);
#pragma unroll
        for (int g = 0; g < W / 8; g++) {
            double m[8];
#pragma unroll
            for (int c = 0; c < 8; c++) {
                m[c] = f[0] + q[0][8 * g + c];
#pragma unroll
                for (int r = 1; r < R; r++) m[c] = __builtin_fmin(m[c], f[r] + q[r][8 * g + c]);
            }
            // halves go to the lanes that keep them: 8 columns, 4, 2, 1 a lane
            const bool h0 = lane & 1, h1 = lane & 2, h3 = lane & 8;
            double x[4], y[2];
#pragma unroll
            for (int c = 0; c < 4; c++)
                x[c] = __builtin_fmin(h0 ? m[4 + c] : m[c],
                                      lane_move<kXor1>(h0 ? m[c] : m[4 + c]));
#pragma unroll
            for (int c = 0; c < 2; c++)
                y[c] = __builtin_fmin(h1 ? x[2 + c] : x[c],
                                      lane_move<kXor2>(h1 ? x[c] : x[2 + c]));
            double z = __builtin_fmin(h3 ? y[1] : y[0], lane_move<kXor8>(h3 ? y[0] : y[1]));
            z = __builtin_fmin(z, __shfl_xor(z, 4));
            const int col = 8 * g + (h0 ? 4 : 0) + (h1 ? 2 : 0) + (h3 ? 1 : 0);
            if (!(lane & 4)) part[(4 * wave + lane / 16) * W + col] = z;
        }
        __syncthreads();
        // (the next layer writes the other half of part, the one after it follows
        // that layer's barrier)
        if (wave < W / 8) {
            const int col = 8 * wave + lane % 8;
            double z = part[(lane / 8) * W + col];
#pragma unroll
            for (int u = 1; u < ROWS / 8; u++) z = __builtin_fmin(z, part[(8 * u + lane / 8) * W + col]);
            z = __builtin_fmin(z, lane_move<kXor8>(z));
            z = __builtin_fmin(z, __shfl_xor(z, 16));
            z = __builtin_fmin(z, __shfl_xor(z, 32));
            const int64_t j = c0 + col;
            if (lane < 8 && j < p)
                __hip_atomic_store(
                    reinterpret_cast<uint64_t*>(a.F + (int64_t)i * a.ld + j),
                    (uint64_t)__double_as_longlong(z), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// The workgroup's place in the order of starting; also loads the log2 table.
__device__ __forceinline__ int64_t take_ticket(const HeldArgs& a, HeldSmem& sm) {
    if (threadIdx.x == 0)
        sm.ticket = __hip_atomic_fetch_add(a.K + a.nblk + 1, 1, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
    if (a.lamp != 0.0) load_log2_table(sm.tab);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(sm.ticket);
}

__global__ __launch_bounds__(kHT) void k_held(HeldArgs a) {
    __shared__ HeldSmem sm;
    if (!live(a)) return;  // uniform
    const int64_t g = take_ticket(a, sm);
    if (a.H.p <= kNarrowP) {
        if (8 * g + 8 <= kHT)
            held<kHT, 8, 1>(a, 8 * g, sm);
        else
            held<kHT, 8, 2>(a, 8 * g, sm);
    } else if (g < 32) {
        held<kHT, 32, 1>(a, 32 * g, sm);
    } else if (g < 96) {
        held<kHT, 16, 2>(a, kHT + 16 * (g - 32), sm);
    } else {
        held<kHT, 8, 3>(a, 2 * kHT + 8 * (g - 96), sm);
    }
}

// p > kBigP: 8 workgroups of 64 columns, 10 of 48 (512 to 991), 44 of 24 (to 2047), 64 of 16
// (to 3071), then 8 columns each.
__global__ __launch_bounds__(kHTBig) void k_held_big(HeldArgs a) {
    __shared__ HeldSmem sm;
    if (!live(a)) return;  // uniform
    const int64_t g = take_ticket(a, sm);
    if (g < 8)
        held<kHTBig, 64, 1>(a, 64 * g, sm);
    else if (g < 18)
        held<kHTBig, 48, 2>(a, 512 + 48 * (g - 8), sm);
    else if (g < 62)
        held<kHTBig, 24, 4>(a, 992 + 24 * (g - 18), sm);
    else if (g < 126)
        held<kHTBig, 16, 6>(a, 2048 + 16 * (g - 62), sm);
    else
        held<kHTBig, 8, 8>(a, 3072 + 8 * (g - 126), sm);
}

}  // namespace

hipError_t launch_held(const SweepSolve& S, hipStream_t st) {
    HeldArgs a;
    a.H = S.H;
    a.F = S.F;
    a.K = S.K;
    a.ld = S.ld;
    a.nblk = (S.H.p + 63) / 64;
    a.I = S.I;
    a.lamp = S.lamp;
    a.lampp = S.lampp;
    a.runp = S.runp;
    const int64_t p = S.H.p;
    if (p < 2 || p > kHeldMaxP || a.I < 2) return hipErrorInvalidValue;
    k_held_base<<<dim3((unsigned)((p + 255) / 256), (unsigned)(a.I - 1)), 256, 0, st>>>(a);
    if (a.I > 2 && p > kBigP)
        k_held_big<<<(unsigned)(126 + (p - kBigP + 7) / 8), kHTBig, 0, st>>>(a);
    else if (a.I > 2 && p > kNarrowP)
        k_held<<<(unsigned)(96 + (p - kNarrowP + 7) / 8), kHT, 0, st>>>(a);
    else if (a.I > 2)
        k_held<<<(unsigned)((p + 7) / 8), kHT, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace ecasq
