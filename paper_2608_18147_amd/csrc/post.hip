// Steps after the DP: three-colour refinement (Sec. 6), solution metrics,
// codebook gather, and the final unbiased stochastic rounding (Sec. 2) with
// a plug-in entropy of the symbol histogram.
#include <hip/hip_fp16.h>

#include <mutex>

#include "chain.hpp"
#include "device.hpp"
#include "launch.hpp"

namespace ecasq {

namespace {

constexpr int kMaxT = 256;

// The whole refinement in one block: rounds of colour substeps 0, 1, 2.  All
// movers of a colour are independent (their objectives share no frequency)
// and are searched in parallel; a substep whose result
// violates the budget (budget mode) is undone; refinement stops after a round
// without a committed move.  stats: rounds run, moves committed.
//
// One evaluation of the objective is a chain of loads, divisions and logarithms of
// about half a microsecond, and a mover's binary search takes two of them for each of its log2(p) steps.
// 16 lanes search for a mover together: they evaluate both sides of all 7
// comparisons that the next three steps may ask for, so that three steps cost one evaluation.  The
// comparisons and their outcomes are those of the one-by-one search.  The
// entropy of the budget check is formed one value per thread and summed in order by
// one.
constexpr int kRefT = 1024;
constexpr int kRefG = 16;  // lanes of a mover

__global__ __launch_bounds__(kRefT) void k_refine(Hist H, int32_t t, int32_t* __restrict__ ug,
                                                  double lamp, double b, int32_t budget,
                                                  int32_t rounds, int32_t exhaustive,
                                                  int32_t* __restrict__ stats) {
    __shared__ double2 tab[kLog2Size];
    __shared__ int32_t u[kMaxT], nu[kMaxT];
    __shared__ int32_t moved_s, commit_s;
    __shared__ double redv[kRefT];
    __shared__ int64_t redi[kRefT];
    double* sU = redv;  // (the reduction arrays are free when these are used)
    double* sD = redv + kMaxT;
    double* sh = redv + 2 * kMaxT;
    const int tid = threadIdx.x;
    load_log2_table(tab);
    for (int r = tid; r < t; r += blockDim.x) u[r] = ug[r];
    __syncthreads();
    int32_t nrun = 0, nmoves = 0;
    for (int32_t rd = 0; rd < rounds; rd++) {
        int any = 0;
        for (int32_t c = 0; c < 3; c++) {
            for (int r = tid; r < t; r += blockDim.x) nu[r] = u[r];
            if (tid == 0) moved_s = 0;
            __syncthreads();
            if (!exhaustive) {
                const int sub = tid % kRefG;
                // the first mover of the colour is c, or 3 for colour 0
                for (int32_t r = (c ? c : 3) + 3 * (tid / kRefG); r <= t - 2;
                     r += 3 * (kRefT / kRefG)) {
                    const int64_t L = u[r - 1], R = u[r + 1];
                    if (R - L < 3) continue;
                    int64_t lo = L + 1, hi = R - 1;
                    while (lo < hi) {
                        // lane 2 x + s evaluates side s of comparison x of the tree: x = 0
                        // the next one, 2 x + 1 and 2 x + 2 those that follow its outcomes
                        int64_t a = lo, e = hi;
                        const int x1 = sub / 2 + 1;  // 1 b1 b2: the outcomes on the way
                        for (int bit = 30 - __builtin_clz((unsigned)x1); bit >= 0; bit--) {
                            const int64_t mid = a + (e - a) / 2;
                            if (a >= e) break;
                            if ((x1 >> bit) & 1) a = mid + 1;
                            else e = mid;
                        }
                        const bool on = a < e && sub < 14;
                        const int64_t m = on ? a + (e - a) / 2 + (sub & 1) : lo;
                        const double val = refine_local(H, t, u, r, m, lamp, tab);
                        const double other = __shfl_xor(val, 1);
                        const uint32_t less =
                            (uint32_t)(__ballot((sub & 1) == 0 && other < val) >>
                                       (tid % 64 / kRefG * kRefG)) & 0xFFFFu;
                        int x = 0;
                        for (int step = 0; step < 3 && lo < hi; step++) {
                            const int64_t mid = lo + (hi - lo) / 2;
                            const bool up = (less >> (2 * x)) & 1u;
                            if (up) lo = mid + 1;
                            else hi = mid;
                            x = 2 * x + (up ? 2 : 1);
                        }
                    }
                    if (lo != u[r]) {
                        const double val =
                            refine_local(H, t, u, r, sub & 1 ? (int64_t)u[r] : lo, lamp, tab);
                        const double was = __shfl_xor(val, 1);
                        if (sub == 0 && val < was) {
                            nu[r] = (int32_t)lo;
                            atomicAdd(&moved_s, 1);
                        }
                    }
                }
            } else {
                for (int32_t r = 1; r <= t - 2; r++) {
                    if (r % 3 != c) continue;
                    const int64_t L = u[r - 1], R = u[r + 1];
                    if (R - L < 3) continue;
                    double bv = __builtin_huge_val();
                    int64_t bm = -1;
                    for (int64_t m = L + 1 + tid; m < R; m += blockDim.x) {
                        const double val = refine_local(H, t, u, r, m, lamp, tab);
                        if (val < bv) {
                            bv = val;
                            bm = m;
                        }
                    }
                    redv[tid] = bv;
                    redi[tid] = bm;
                    __syncthreads();
                    for (int off = blockDim.x / 2; off > 0; off >>= 1) {
                        if (tid < off) {
                            const double ov = redv[tid + off];
                            const int64_t oi = redi[tid + off];
                            if (oi >= 0 && (redi[tid] < 0 || ov < redv[tid] ||
                                            (ov == redv[tid] && oi < redi[tid]))) {
                                redv[tid] = ov;
                                redi[tid] = oi;
                            }
                        }
                        __syncthreads();
                    }
                    if (tid == 0) {
                        const int64_t m = redi[0];
                        if (m != u[r] &&
                            redv[0] < refine_local(H, t, u, r, u[r], lamp, tab)) {
                            nu[r] = (int32_t)m;
                            moved_s += 1;
                        }
                    }
                    __syncthreads();
                }
            }
            __syncthreads();
            if (budget && moved_s) {  // uniform
                // expected frequencies and their terms as chain_hout forms them
                for (int32_t r = tid; r + 1 < t; r += blockDim.x)
                    ud_at(H, nu[r], nu[r + 1], sU[r], sD[r]);
                __syncthreads();
                for (int32_t r = tid; r < t; r += blockDim.x)
                    sh[r] = hf(H, r == 0 ? H.c0 + sD[0] : r == t - 1 ? sU[r - 1] : sU[r - 1] + sD[r],
                               tab);
                __syncthreads();
            }
            if (tid == 0) {
                int32_t moved = moved_s;
                if (moved && budget) {
                    double ho = 0.0;
                    for (int32_t r = 0; r < t; r++) ho = ho + sh[r];
                    if (ho > b) moved = 0;
                }
                commit_s = moved;
            }
            __syncthreads();
            const int32_t moved = commit_s;
            if (moved) {
                for (int r = tid; r < t; r += blockDim.x) u[r] = nu[r];
                any = 1;
                nmoves += moved;
            }
            __syncthreads();
        }
        nrun++;
        if (!any) break;
    }
    for (int r = tid; r < t; r += blockDim.x) ug[r] = u[r];
    if (tid == 0) {
        stats[0] = nrun;
        stats[1] = nmoves;
    }
}

// out: MSE, vNMSE, H(Xhat), H(I,B), vNMSE + lambda H(Xhat), H(Xhat) + 32t/d.
// The interval terms and the values' entropy terms are formed one per
// thread; one thread then sums them in index order (the sums of the chain
// walk in chain_hout and of the path accumulators, bit for bit).
__global__ void k_metrics(Hist H, int32_t t, const int32_t* __restrict__ u, double lam,
                          double s2tot, double* __restrict__ out) {
    __shared__ double2 tab[kLog2Size];
    __shared__ double sC[kMaxT], sP[kMaxT], sU[kMaxT], sD[kMaxT], sh[kMaxT];
    load_log2_table(tab);
    __syncthreads();
    for (int32_t r = threadIdx.x; r + 1 < t; r += blockDim.x) {
        double C, P, U, D;
        cell_at(H, u[r], u[r + 1], tab, C, P);
        ud_at(H, u[r], u[r + 1], U, D);
        sC[r] = C;
        sP[r] = P;
        sU[r] = U;
        sD[r] = D;
    }
    __syncthreads();
    // expected frequency of value q (as chain_hout forms it), then h(f / d)
    for (int32_t q = threadIdx.x; q < t; q += blockDim.x) {
        double f;
        if (t == 1) f = H.dd;
        else if (q == 0) f = H.c0 + sD[0];
        else if (q == t - 1) f = sU[t - 2];
        else f = sU[q - 1] + sD[q];
        sh[q] = hf(H, f, tab);
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double mse = 0.0, hs = 0.0;
    for (int32_t r = 0; r + 1 < t; r++) {
        mse = mse + sC[r];
        hs = hs - sP[r];
    }
    double ho = sh[0];
    if (t > 1) {
        ho = 0.0;
        for (int32_t q = 0; q < t; q++) ho = ho + sh[q];
    }
    const double vn = s2tot > 0.0 ? mse / s2tot : 0.0;
    const double lr = __builtin_isfinite(lam) ? lam : 0.0;
    out[0] = mse;
    out[1] = vn;
    out[2] = ho;
    out[3] = hs;
    out[4] = __builtin_fma(lr, ho, vn);
    out[5] = ho + (32.0 * (double)t) / H.dd;
}

__global__ void k_gather(const double* __restrict__ v, const int32_t* __restrict__ u, int32_t t,
                         double* __restrict__ codebook, int32_t* __restrict__ rank) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= t) return;
    codebook[r] = v[u[r]];
    if (rank) rank[r] = u[r];
}

// Philox4x32-10 (Salmon et al., SC'11) at counter (c0, 0, c2, 0): ten rounds of
// two 32x32->64 products mixed with the other words and the round key; the key
// advances by the two Weyl increments between rounds.  (With an inlined call the
// products of the words that are zero or the same in every thread fold away:
// 18 of 20 remain for c2 = 0.)
__device__ __forceinline__ void philox4x32_10(uint32_t (&c)[4], uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int rnd = 0; rnd < 10; rnd++) {
        if (rnd) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        // each 32 x 32 -> 64 product in one instruction (hi and lo halves)
        const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        // (truth table of a three-way exclusive or, one instruction each)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32(hi1, c[1], k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32(hi0, c[3], k1, 0x96);
        c[0] = n0;
        c[1] = lo1;
        c[2] = n2;
        c[3] = lo0;
    }
}

// Entry i of x as a float (each type's values are floats).
template <int DT>
__device__ __forceinline__ float load_x(const void* x, int64_t i) {
    if (DT == 0) return reinterpret_cast<const float*>(x)[i];
    if (DT == 1) return __half2float(reinterpret_cast<const __half*>(x)[i]);
    return __uint_as_float(((uint32_t)reinterpret_cast<const uint16_t*>(x)[i]) << 16);
}

// Entries i .. i + 3 by one load, at any alignment.
template <int DT>
__device__ __forceinline__ void load_x4(const void* x, int64_t i, float (&v)[4]) {
    if (DT == 0) {
        __builtin_memcpy(v, reinterpret_cast<const float*>(x) + i, 16);
    } else {
        uint32_t w[2];
        __builtin_memcpy(w, reinterpret_cast<const uint16_t*>(x) + i, 8);
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint32_t h = k % 2 ? w[k / 2] >> 16 : w[k / 2] & 0xFFFFu;
            v[k] = DT == 1 ? __half2float(__ushort_as_half((uint16_t)h))
                           : __uint_as_float(h << 16);
        }
    }
}

// The rounding's codebook in LDS: the values q_0 .. q_{t-1} and each interval's
// width D_r = q_{r+1} - q_r in 64 bits; s, the search's copy in 32 bits: the
// largest floats not above q_0 .. q_{t-2} (for a float x, q < x exactly if that
// float is below x: a float above it is above q), followed by +inf (so the search needs no bound: no x is below
// +inf, and a bracket never starts at q_{t-1}); R_r, about 1 / D_r, for D_r in
// [2^-100, 2^100] (NaN otherwise, which sends every entry of that interval to
// the exact quotient).
struct RoundBook {
    double q[kMaxT], D[kMaxT];
    float s[2 * kMaxT], R[kMaxT];
};

__device__ __forceinline__ float float_below(double q) {
    const float f = (float)q;  // nearest: at most one step above q
    if (!((double)f > q)) return f;
    const uint32_t b = __float_as_uint(f);
    // the float before f (f > q, so f is not -inf)
    return __uint_as_float((b & 0x7FFFFFFFu) == 0u ? 0x80000001u : (b >> 31) ? b + 1u : b - 1u);
}

__device__ __forceinline__ void load_book(RoundBook& B, const double* __restrict__ cb, int32_t t) {
    for (int r = threadIdx.x; r < kMaxT; r += blockDim.x) B.q[r] = r < t ? cb[r] : 0.0;
    for (int r = threadIdx.x; r < 2 * kMaxT; r += blockDim.x)
        B.s[r] = r <= t - 2 ? float_below(cb[r]) : __builtin_huge_valf();
    __syncthreads();
    for (int r = threadIdx.x; r + 1 < t; r += blockDim.x) {
        const double D = B.q[r + 1] - B.q[r];
        B.D[r] = D;
        B.R[r] = (D >= 0x1p-100 && D <= 0x1p+100) ? 1.0f / (float)D : __builtin_nanf("");
    }
}

__device__ __forceinline__ int32_t search_step(int32_t t) {
    return t >= 3 ? (int32_t)(1u << (31 - __builtin_clz((uint32_t)(t - 2)))) : 0;
}

__device__ __forceinline__ double uniform53(uint32_t lo, uint32_t hi) {
    const uint64_t bits = ((((uint64_t)hi) << 32) | lo) >> 11;
    return (double)bits * 0x1p-53;
}

// Symbol of x under the codebook (t >= 2) and the 53-bit uniform u of words
// (lo, hi): the bracket r (the largest r <= t-2 with q_r < x, else 0, by a search
// over powers of two from the largest power h <= t-2: indices up to 2h - 1 <
// 2 kMaxT; that of NE entries side by side, to have their LDS reads in flight
// together), then up iff u < RN((x - q_r) / D_r).  The quotient and u are first
// taken in 32 bits: N = x - q_r (64 bits) to a float, times R_r, is within 2^-21
// of the quotient for quotients up to 2 and above 1 beyond that (N or the product may
// round to an infinity or a zero: of the quotient's sign, and 2^-21 away at most), and the
// high word's float within 2^-24 of u: where they differ by more than 2^-20
// the comparison is decided.  Only a u this close (one entry in 2^19), or NaN,
// takes the 64-bit division.
__device__ __forceinline__ uint32_t round_at(const RoundBook& B, int32_t r, float x, uint32_t lo,
                                             uint32_t hi) {
    const double N = (double)x - B.q[r];
    const float e = (float)hi * 0x1p-32f - (float)N * B.R[r];
    bool up = e < 0.0f;
    if (!(__builtin_fabsf(e) > 0x1p-20f)) up = uniform53(lo, hi) < N / B.D[r];
    return (uint32_t)r + (up ? 1u : 0u);
}

template <int NE>
__device__ __forceinline__ void brackets(const RoundBook& B, int32_t h, const float (&x)[NE],
                                         int32_t (&r)[NE]) {
#pragma unroll
    for (int e = 0; e < NE; e++) r[e] = 0;
    for (int32_t step = h; step > 0; step >>= 1) {
        float m[NE];
#pragma unroll
        for (int e = 0; e < NE; e++) m[e] = B.s[r[e] + step];
#pragma unroll
        for (int e = 0; e < NE; e++) r[e] += m[e] < x[e] ? step : 0;
    }
}

// Final stochastic rounding (Sec. 2): entries 2j and 2j+1 take words (0, 1) and
// (2, 3) of Philox4x32-10 at counter (j, 0, 0, 0) (j < 2^27) with key (k0, k1); a
// thread takes two j by one load and one store.  Symbol counts gather in LDS, in
// eight copies (lanes with the same symbol wait for each other), and each
// workgroup adds its sums to hist: workgroups are large and few, because the
// additions of all of them to one count wait for each other too (4096 workgroups of
// 256 threads took 104 us for 3 million bf16 entries and 256 values, 90 us of
// it these additions).
constexpr int kQT = 1024;
constexpr int kQCopies = 8;
constexpr int kQPad = kMaxT + 1;

template <int DT>
__device__ __forceinline__ void quantize_part(const RoundBook& B, unsigned int* __restrict__ lh,
                                              const void* __restrict__ x, int64_t d, int32_t t,
                                              uint32_t k0, uint32_t k1,
                                              uint8_t* __restrict__ symbols) {
    const int32_t h = search_step(t);
    unsigned int* mine = lh + (threadIdx.x % kQCopies) * kQPad;
    const int64_t nquad = (d + 3) / 4;
    for (int64_t j = (int64_t)blockIdx.x * kQT + threadIdx.x; j < nquad;
         j += (int64_t)gridDim.x * kQT) {
        const int64_t i0 = 4 * j;
        const int n = (int)min((int64_t)4, d - i0);
        float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (n == 4) {
            load_x4<DT>(x, i0, v);
        } else {
#pragma unroll
            for (int k = 0; k < 3; k++)
                if (k < n) v[k] = load_x<DT>(x, i0 + k);
        }
        uint32_t s[4] = {0u, 0u, 0u, 0u};
        if (t > 1) {
            int32_t r[4];
            brackets<4>(B, h, v, r);
#pragma unroll
            for (int e = 0; e < 2; e++) {
                uint32_t c[4] = {(uint32_t)(2 * j + e), 0u, 0u, 0u};
                philox4x32_10(c, k0, k1);
                s[2 * e] = round_at(B, r[2 * e], v[2 * e], c[0], c[1]);
                s[2 * e + 1] = round_at(B, r[2 * e + 1], v[2 * e + 1], c[2], c[3]);
            }
        }
        if (n == 4) {
            const uint32_t w = s[0] | (s[1] << 8) | (s[2] << 16) | (s[3] << 24);
            __builtin_memcpy(symbols + i0, &w, 4);
#pragma unroll
            for (int k = 0; k < 4; k++) atomicAdd(&mine[s[k]], 1u);
        } else {
#pragma unroll
            for (int k = 0; k < 3; k++)
                if (k < n) {
                    symbols[i0 + k] = (uint8_t)s[k];
                    atomicAdd(&mine[s[k]], 1u);
                }
        }
    }
}

__device__ __forceinline__ unsigned int fold_copies(const unsigned int* __restrict__ lh, int r) {
    unsigned int n = 0;
#pragma unroll
    for (int c = 0; c < kQCopies; c++) n += lh[c * kQPad + r];
    return n;
}

// PARTS: each workgroup's counts in a row of its own, 256 words (nothing to
// clear before); otherwise added to hist.
template <int DT, bool PARTS>
__global__ __launch_bounds__(kQT) void k_quantize(const void* __restrict__ x, int64_t d,
                                                  const double* __restrict__ cb, int32_t t,
                                                  uint32_t k0, uint32_t k1,
                                                  uint8_t* __restrict__ symbols,
                                                  unsigned long long* __restrict__ hist,
                                                  uint32_t* __restrict__ parts) {
    __shared__ RoundBook B;
    __shared__ unsigned int lh[kQCopies * kQPad];
    for (int r = threadIdx.x; r < kQCopies * kQPad; r += kQT) lh[r] = 0u;
    load_book(B, cb, t);
    __syncthreads();
    quantize_part<DT>(B, lh, x, d, t, k0, k1, symbols);
    __syncthreads();
    if ((int)threadIdx.x < t) {
        const unsigned int n = fold_copies(lh, threadIdx.x);
        if constexpr (PARTS)
            parts[(int64_t)blockIdx.x * kMaxT + threadIdx.x] = n;
        else if (n)
            atomicAdd(&hist[threadIdx.x], (unsigned long long)n);
    }
}

// Time-shared rounding (Sec. 7): entry i takes the second codebook iff its
// partition uniform, from Philox counter (j_lo, j_hi, 1, 0) with j = i / 2
// (words (0, 1) for even i, (2, 3) for odd), is below alpha, and is then
// rounded with its codebook exactly as k_quantize rounds it (counter (j_lo,
// j_hi, 0, 0)).  hist: the first codebook's t0 counts, then the second's t1;
// part[i] = 1 for the second.
template <int DT>
__global__ __launch_bounds__(256) void k_quantize_ts(
    const void* __restrict__ x, int64_t d, const double* __restrict__ cb0, int32_t t0,
    const double* __restrict__ cb1, int32_t t1, double alpha, uint32_t k0, uint32_t k1,
    uint8_t* __restrict__ symbols, uint8_t* __restrict__ part,
    unsigned long long* __restrict__ hist) {
    __shared__ RoundBook B[2];
    __shared__ unsigned int lh[2][kMaxT];
    for (int r = threadIdx.x; r < kMaxT; r += blockDim.x) {
        lh[0][r] = 0u;
        lh[1][r] = 0u;
    }
    load_book(B[0], cb0, t0);
    load_book(B[1], cb1, t1);
    __syncthreads();
    const int32_t h0 = search_step(t0), h1 = search_step(t1);
    const int64_t npair = (d + 1) / 2;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < npair;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i0 = 2 * j;
        const bool two = i0 + 1 < d;
        uint32_t w[4] = {(uint32_t)j, 0u, 1u, 0u};  // j < 2^27
        philox4x32_10(w, k0, k1);
        uint32_t c[4] = {(uint32_t)j, 0u, 0u, 0u};
        philox4x32_10(c, k0, k1);
#pragma unroll
        for (int e = 0; e < 2; e++) {
            const int64_t i = i0 + e;
            if (e == 1 && !two) break;
            const int pw = uniform53(w[2 * e], w[2 * e + 1]) < alpha ? 1 : 0;
            const int32_t t = pw ? t1 : t0;
            uint32_t sym = 0;
            if (t > 1) {
                const float v[1] = {load_x<DT>(x, i)};
                int32_t r[1];
                brackets<1>(B[pw], pw ? h1 : h0, v, r);
                sym = round_at(B[pw], r[0], v[0], c[2 * e], c[2 * e + 1]);
            }
            symbols[i] = (uint8_t)sym;
            if (part) part[i] = (uint8_t)pw;
            atomicAdd(&lh[pw][sym], 1u);
        }
    }
    __syncthreads();
    for (int r = threadIdx.x; r < t0; r += blockDim.x)
        if (lh[0][r]) atomicAdd(&hist[r], (unsigned long long)lh[0][r]);
    for (int r = threadIdx.x; r < t1; r += blockDim.x)
        if (lh[1][r]) atomicAdd(&hist[t0 + r], (unsigned long long)lh[1][r]);
}

// Sum over the first 256 threads of a workgroup (a butterfly per wavefront, then
// the four wavefront sums in order); every thread gets the total.
__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();  // red is free
    if (threadIdx.x % 64 == 0 && threadIdx.x < 256) red[threadIdx.x / 64] = v;
    __syncthreads();
    return ((red[0] + red[1]) + red[2]) + red[3];
}

// Plug-in entropy of one symbol histogram (t <= 256 counts, one per thread):
// H = sum of h(n_r / n) over the nonzero counts, n = the counts' total
// (d for the plain rounding, the part's size for a time-shared part).
__device__ __forceinline__ double plugin_entropy(const unsigned long long* __restrict__ hist,
                                                 int32_t t, double n, int64_t* hist_out,
                                                 const double2* __restrict__ tab, double* red) {
    const int r = threadIdx.x;
    double h = 0.0;
    if (r < t) {
        const unsigned long long c = hist[r];
        if (hist_out) hist_out[r] = (int64_t)c;
        if (c) h = hfun((double)c / n, tab);
    }
    return block_sum(h, red);
}

// Entropy of a time-shared rounding: each part's plug-in entropy over its own
// entries, weighted by its size: (n_0 H_0 + n_1 H_1) / d.
__global__ __launch_bounds__(256) void k_entropy_ts(const unsigned long long* __restrict__ hist,
                                                    int32_t t0, int32_t t1, int64_t d,
                                                    double* __restrict__ ent,
                                                    int64_t* __restrict__ hist_out) {
    __shared__ double2 tab[kLog2Size];
    __shared__ double red[4];
    load_log2_table(tab);
    __syncthreads();
    double total = 0.0;
    int32_t base = 0;
    for (int w = 0; w < 2; w++) {
        const int32_t t = w ? t1 : t0;
        const int r = threadIdx.x;
        const double nr = r < t ? (double)hist[base + r] : 0.0;  // counts < 2^53: exact
        const double n = block_sum(nr, red);
        if (n > 0.0) {
            const double H = plugin_entropy(hist + base, t, n, hist_out ? hist_out + base : nullptr,
                                            tab, red);
            total = total + n * H;
        } else if (hist_out && r < t) {
            hist_out[base + r] = 0;
        }
        base += t;
    }
    if (threadIdx.x == 0) *ent = total / (double)d;
}

__global__ __launch_bounds__(256) void k_entropy(const unsigned long long* __restrict__ hist,
                                                 int32_t t, int64_t d, double* __restrict__ ent,
                                                 int64_t* __restrict__ hist_out) {
    __shared__ double2 tab[kLog2Size];
    __shared__ double red[4];
    load_log2_table(tab);
    __syncthreads();
    const double H = plugin_entropy(hist, t, (double)d, hist_out, tab, red);
    if (threadIdx.x == 0) *ent = H;
}

// The same from the rows of n workgroups (d < 2^32 entries in all).
__global__ __launch_bounds__(kQT) void k_entropy_parts(const uint32_t* __restrict__ parts,
                                                       int32_t n, int32_t t, int64_t d,
                                                       double* __restrict__ ent,
                                                       int64_t* __restrict__ hist_out) {
    constexpr int G = kQT / kMaxT;
    __shared__ double2 tab[kLog2Size];
    __shared__ double red[4];
    __shared__ uint32_t sum[G][kMaxT];
    __shared__ unsigned long long hist[kMaxT];
    load_log2_table(tab);
    const int r = threadIdx.x % kMaxT, g = threadIdx.x / kMaxT;
    uint32_t c = 0;
    if (r < t) {
#pragma unroll 8
        for (int32_t b = g; b < n; b += G) c += parts[(int64_t)b * kMaxT + r];
    }
    sum[g][r] = c;
    __syncthreads();
    if (g == 0) {
        uint32_t a = 0;
#pragma unroll
        for (int k = 0; k < G; k++) a += sum[k][r];
        hist[r] = a;
    }
    __syncthreads();
    const double H = plugin_entropy(hist, t, (double)d, hist_out, tab, red);
    if (threadIdx.x == 0) *ent = H;
}

// Rounding and entropy of a small input in one launch of one workgroup: no
// counts in memory, nothing to clear, no second kernel.
template <int DT>
__global__ __launch_bounds__(kQT) void k_quantize_small(const void* __restrict__ x, int64_t d,
                                                        const double* __restrict__ cb, int32_t t,
                                                        uint32_t k0, uint32_t k1,
                                                        uint8_t* __restrict__ symbols,
                                                        double* __restrict__ ent,
                                                        int64_t* __restrict__ hist_out) {
    __shared__ RoundBook B;
    __shared__ double2 tab[kLog2Size];
    __shared__ double red[4];
    __shared__ unsigned int lh[kQCopies * kQPad];
    __shared__ unsigned long long hist[kMaxT];
    for (int r = threadIdx.x; r < kQCopies * kQPad; r += kQT) lh[r] = 0u;
    load_log2_table(tab);
    load_book(B, cb, t);
    __syncthreads();
    quantize_part<DT>(B, lh, x, d, t, k0, k1, symbols);
    __syncthreads();
    if ((int)threadIdx.x < t) hist[threadIdx.x] = fold_copies(lh, threadIdx.x);
    __syncthreads();
    const double H = plugin_entropy(hist, t, (double)d, hist_out, tab, red);
    if (threadIdx.x == 0) *ent = H;
}

// Symbol counts of the allocation-free rounding entry point: one array per
// device, alive until the process ends, shared by every such call on that
// device (calls that overlap on one device race on it).
static __device__ __align__(256) unsigned long long scratch[kMaxT];

__global__ void k_zero_counts(unsigned long long* __restrict__ h, int32_t n) {
    for (int32_t r = threadIdx.x; r < n; r += blockDim.x) h[r] = 0ull;
}

}  // namespace

// Device address of `scratch` on the current device, looked up once per
// device (the host-side name is not a device address).
hipError_t quantize_scratch(unsigned long long** out) {
    constexpr int kMaxDev = 64;
    static std::mutex mu;
    static unsigned long long* ptr[kMaxDev] = {};
    static hipError_t err[kMaxDev] = {};
    static bool done[kMaxDev] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDev) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!done[dev]) {
        void* p = nullptr;
        err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        ptr[dev] = static_cast<unsigned long long*>(p);
        done[dev] = true;
    }
    if (err[dev] != hipSuccess) return err[dev];
    *out = ptr[dev];
    return hipSuccess;
}

hipError_t launch_zero_counts(unsigned long long* h, int32_t n, hipStream_t st) {
    k_zero_counts<<<1, 256, 0, st>>>(h, n);
    return hipGetLastError();
}

hipError_t launch_refine(const Hist& H, int32_t t, int32_t* u, double lamp, double b,
                         int32_t budget, int32_t rounds, int32_t exhaustive, int32_t* stats,
                         hipStream_t st) {
    k_refine<<<1, kRefT, 0, st>>>(H, t, u, lamp, b, budget, rounds, exhaustive, stats);
    return hipGetLastError();
}

hipError_t launch_metrics(const Hist& H, int32_t t, const int32_t* u, double lam, double s2tot,
                          double* out, hipStream_t st) {
    if (t < 1 || t > kMaxT) return hipErrorInvalidValue;
    k_metrics<<<1, 256, 0, st>>>(H, t, u, lam, s2tot, out);
    return hipGetLastError();
}

hipError_t launch_gather(const double* v, const int32_t* u, int32_t t, double* codebook,
                         int32_t* rank, hipStream_t st) {
    k_gather<<<(t + 63) / 64, 64, 0, st>>>(v, u, t, codebook, rank);
    return hipGetLastError();
}

// One workgroup up to here: a call of 4096 entries takes 14 us, of 20000 14 to 18 and of 32768 14
// to 25 (2 to 256 values), one through the counts' allocation, a second launch and the
// release 30 to 43.  Without an allocation the three launches take 15 us up to 200000 entries;
// one workgroup takes 9 + (1.2 to 2.6 us, with the steps of the bracket's search) for each 4096
// entries above 8192: 15 us at 32768 entries and 2 values, 24576 and 32, 16384 and 256.
constexpr int64_t kQSmall = 32 * kQT;

bool quantize_is_small(int64_t d, int32_t t, bool noalloc) {
    const int64_t steps = 32 - __builtin_clz((unsigned)t);  // 2 to 9 from 2 to 256 values
    return d <= kQSmall && (!noalloc || d * (4 + steps) <= 13 * 16 * kQT);
}

hipError_t launch_quantize_small(const void* x, int dt, int64_t d, const double* codebook,
                                 int32_t t, uint64_t seed, uint8_t* symbols, double* ent,
                                 int64_t* hist_out, hipStream_t st) {
    if (d > kQSmall) return hipErrorInvalidValue;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    if (dt == 0)
        k_quantize_small<0><<<1, kQT, 0, st>>>(x, d, codebook, t, k0, k1, symbols, ent, hist_out);
    else if (dt == 1)
        k_quantize_small<1><<<1, kQT, 0, st>>>(x, d, codebook, t, k0, k1, symbols, ent, hist_out);
    else
        k_quantize_small<2><<<1, kQT, 0, st>>>(x, d, codebook, t, k0, k1, symbols, ent, hist_out);
    return hipGetLastError();
}

// Rows of counts up to here (one launch less to clear a count array, and up to 256
// rows are summed in about 5 us); above, the workgroups are twice as many
// and their time is what counts.
constexpr int64_t kQParts = (int64_t)1 << 22;

size_t quantize_scratch_bytes(int64_t d) {
    return d <= kQParts ? sizeof(uint32_t) * kMaxT * 256 : sizeof(unsigned long long) * kMaxT;
}

namespace {

template <bool PARTS>
void quantize_groups(const void* x, int dt, int64_t d, const double* codebook, int32_t t,
                     uint64_t seed, uint8_t* symbols, unsigned long long* hist, uint32_t* parts,
                     unsigned g, hipStream_t st) {
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    if (dt == 0)
        k_quantize<0, PARTS><<<g, kQT, 0, st>>>(x, d, codebook, t, k0, k1, symbols, hist, parts);
    else if (dt == 1)
        k_quantize<1, PARTS><<<g, kQT, 0, st>>>(x, d, codebook, t, k0, k1, symbols, hist, parts);
    else
        k_quantize<2, PARTS><<<g, kQT, 0, st>>>(x, d, codebook, t, k0, k1, symbols, hist, parts);
}

}  // namespace

hipError_t launch_quantize(const void* x, int dt, int64_t d, const double* codebook, int32_t t,
                           uint64_t seed, uint8_t* symbols, unsigned long long* hist,
                           hipStream_t st) {
    // 8 entries per thread at least, two workgroups (all wavefronts) per CU at most
    int64_t g = (d + 8 * kQT - 1) / (8 * kQT);
    if (g > 512) g = 512;
    quantize_groups<false>(x, dt, d, codebook, t, seed, symbols, hist, nullptr, (unsigned)g, st);
    return hipGetLastError();
}

hipError_t launch_quantize_scratch(const void* x, int dt, int64_t d, const double* codebook,
                                   int32_t t, uint64_t seed, uint8_t* symbols, double* ent,
                                   int64_t* hist_out, void* scratch, hipStream_t st) {
    if (d > kQParts) {
        auto* hist = static_cast<unsigned long long*>(scratch);
        hipError_t e = hipMemsetAsync(hist, 0, sizeof(unsigned long long) * kMaxT, st);
        if (e == hipSuccess)
            e = launch_quantize(x, dt, d, codebook, t, seed, symbols, hist, st);
        return e == hipSuccess ? launch_entropy(hist, t, d, ent, hist_out, st) : e;
    }
    auto* parts = static_cast<uint32_t*>(scratch);
    int64_t g = (d + 8 * kQT - 1) / (8 * kQT);
    if (g > 256) g = 256;
    quantize_groups<true>(x, dt, d, codebook, t, seed, symbols, nullptr, parts, (unsigned)g, st);
    k_entropy_parts<<<1, kQT, 0, st>>>(parts, (int32_t)g, t, d, ent, hist_out);
    return hipGetLastError();
}

hipError_t launch_entropy(const unsigned long long* hist, int32_t t, int64_t d, double* ent,
                          int64_t* hist_out, hipStream_t st) {
    k_entropy<<<1, 256, 0, st>>>(hist, t, d, ent, hist_out);
    return hipGetLastError();
}

hipError_t launch_quantize_ts(const void* x, int dt, int64_t d, const double* cb0, int32_t t0,
                              const double* cb1, int32_t t1, double alpha, uint64_t seed,
                              uint8_t* symbols, uint8_t* part, unsigned long long* hist,
                              double* ent, int64_t* hist_out, hipStream_t st) {
    int64_t g = ((d + 1) / 2 + 255) / 256;  // a thread per pair of entries
    if (g > 4096) g = 4096;
    if (g < 1) g = 1;
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    if (dt == 0)
        k_quantize_ts<0><<<(unsigned)g, 256, 0, st>>>(x, d, cb0, t0, cb1, t1, alpha, k0, k1,
                                                      symbols, part, hist);
    else if (dt == 1)
        k_quantize_ts<1><<<(unsigned)g, 256, 0, st>>>(x, d, cb0, t0, cb1, t1, alpha, k0, k1,
                                                      symbols, part, hist);
    else
        k_quantize_ts<2><<<(unsigned)g, 256, 0, st>>>(x, d, cb0, t0, cb1, t1, alpha, k0, k1,
                                                      symbols, part, hist);
    k_entropy_ts<<<1, 256, 0, st>>>(hist, t0, t1, d, ent, hist_out);
    return hipGetLastError();
}

}  // namespace ecasq
