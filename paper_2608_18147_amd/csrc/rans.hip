// Entropy coding of the final symbols with rANS (Duda, arXiv:1311.2540), so
// that the rate the paper charges (App. F.1: the payload at about H(Xhat)
// bits per entry plus a 16-bit descriptor per codebook value) is realised as
// bytes.
//
//   frequencies  f_q = max(1, floor(n_q M / d)), M = 2^16; a surplus goes to
//                the largest f (lowest q among ties), a deficit is taken one
//                unit at a time from the largest f > 1; c_q = f_0 + .. + f_{q-1}
//   state        x in [L, 256 L), L = 2^23, bytes out
//   encode       a segment's symbols in reverse: while x >= 2^15 f_q emit
//                x's low byte, x >>= 8; x = floor(x/f_q) 2^16 + x mod f_q + c_q;
//                finally emit x's four bytes, low first; the segment's stream
//                is the emitted bytes in reverse order
//   decode       x = 4 bytes big-endian; slot = x mod 2^16, q: c_q <= slot <
//                c_q + f_q, x = f_q (x >> 16) + slot - c_q, refill bytes while
//                x < L; every segment ends at x = L
//   stream       t u16 (f_q - 1, little-endian), one u32 per segment of 4096
//                symbols (its end, counted from the payload start), payload
//
// Segments are coded independently, one lane each: encoding writes a
// segment's bytes backwards into a private slot of the scratch buffer, a scan
// of the lengths places them, and a copy packs them.
//
// What bounds both directions is one segment's chain of 4096 states, each
// formed from the last: the time hardly grows until every SIMD holds a whole
// wavefront of segments.  Segments are therefore dealt to as many wavefronts
// as there are SIMDs before a wavefront takes a second one (lanes_of), so that
// the few segments of a small call do not wait for each other's branches, and
// all that does not depend on the state is taken out of the chain: table
// entries, symbols and stream bytes are read ahead, the division is a product.
// While a wavefront has one segment (d <= 2^22) it keeps the whole of it in LDS,
// symbols and stream, so that no step waits for memory: a load's wait also waits
// for the stores before it, which cost the direct kernels about a microsecond every
// 16 symbols.
#include "device.hpp"
#include "launch.hpp"

namespace ecasq {

namespace {

constexpr int kRSeg = 4096;
constexpr uint32_t kRL = 1u << 23;
constexpr uint32_t kRM = 1u << 16;
constexpr int64_t kRSegCap = 2 * kRSeg + 16;  // 2 bytes per symbol at most, plus the state

constexpr int kRWaves = 4;        // wavefronts of a coding workgroup, one per SIMD
constexpr int kRT = 64 * kRWaves;
constexpr int kRFill = 1024;      // wavefronts that fill the chip's SIMDs once

// Segments per wavefront (<= 64 for d <= 2^28).
int32_t lanes_of(int64_t nseg) { return (int32_t)((nseg + kRFill - 1) / kRFill); }

// Segments of nseg <= kRFill are staged in LDS.
bool staged(int64_t nseg) { return nseg <= kRFill; }

// Counts of a rounding's symbols: 16 symbols per load, and eight private
// counts per value, so that the few values most symbols have do not make the
// LDS additions of a wavefront wait for each other.
constexpr int kHCopies = 8;
constexpr int kHPad = 257;

__global__ __launch_bounds__(256) void k_sym_hist(const uint8_t* __restrict__ sym, int64_t d,
                                                  int32_t t, unsigned long long* __restrict__ hist,
                                                  unsigned int* __restrict__ bad) {
    __shared__ unsigned int lh[kHCopies * kHPad];
    for (int x = threadIdx.x; x < kHCopies * kHPad; x += 256) lh[x] = 0u;
    __syncthreads();
    unsigned int* h = lh + (threadIdx.x % kHCopies) * kHPad;
    const int64_t nv = d / 16;
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int64_t i = id; i < nv; i += (int64_t)gridDim.x * 256) {
        uint32_t w[4];
        __builtin_memcpy(w, sym + 16 * i, 16);
#pragma unroll
        for (int k = 0; k < 16; k++) atomicAdd(&h[(w[k / 4] >> (8 * (k % 4))) & 255u], 1u);
    }
    if (id < d - 16 * nv) atomicAdd(&h[sym[16 * nv + id]], 1u);
    __syncthreads();
    unsigned int n = 0;
#pragma unroll
    for (int c = 0; c < kHCopies; c++) n += lh[c * kHPad + threadIdx.x];
    if (n) {
        atomicAdd(&hist[threadIdx.x], (unsigned long long)n);
        if ((int32_t)threadIdx.x >= t) atomicAdd(bad, n);
    }
}

// What encoding needs of a symbol with frequency f and cumulated frequency c,
// for a state x < 2^15 f: floor(x / f) = (x m) >> (32 + s), and the next state
// floor(x/f) 2^16 + x mod f + c = x + c + floor(x/f) (2^16 - f).  With l =
// ceil(log2 f), s = l - 1 and m = floor(2^(31 + l) / f) + 1 the quotient is
// exact for x < 2^31 (Granlund and Montgomery, PLDI'94: m f - 2^(31 + l) lies
// in [1, 2^l]).  f = 1 would need m = 2^32 + 1: there m = 2^32 - 1 and s = 0
// give x - 1 (x >= 1), and the bias makes up for it.
struct EncSym {
    uint32_t xtop;  // 2^15 f - 1: x above gives off a byte first
    uint32_t m;
    uint32_t bias;
    uint32_t cs;    // 2^16 - f, s in the top byte
};

// Bits that state x gives off before the symbol: a byte if x > xtop, two if x / 2^8
// is (x < 2^31: at most two), from the differences' signs.
__device__ __forceinline__ uint32_t bits_off(uint32_t x, uint32_t xtop) {
    return (((xtop - x) >> 31) + ((xtop - (x >> 8)) >> 31)) << 3;
}

__device__ __forceinline__ EncSym enc_sym(uint32_t f, uint32_t c) {
    EncSym e;
    e.xtop = (f << 15) - 1u;
    if (f == 1u) {
        e.m = 0xFFFFFFFFu;
        e.bias = c + kRM - 1u;
        e.cs = kRM - 1u;
        return e;
    }
    const int l = 32 - __builtin_clz(f - 1u);  // 1..16
    e.m = (uint32_t)(((uint64_t)1 << (31 + l)) / f) + 1u;
    e.bias = c;
    e.cs = (kRM - f) | ((uint32_t)(l - 1) << 24);
    return e;
}

// Frequencies of the t symbols, the encoding table of all 256 (those from t on
// are reported by the histogram: they get f = 1, c = 0 here) and the stream's
// frequency header.  One wavefront, symbols 4 lane .. 4 lane + 3 in a lane.
__global__ __launch_bounds__(64) void k_rans_freqs(const unsigned long long* __restrict__ hist,
                                                   int32_t t, int64_t d,
                                                   EncSym* __restrict__ tab,
                                                   uint8_t* __restrict__ head) {
    const int lane = threadIdx.x;
    uint32_t f[4];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int q = 4 * lane + k;
        f[k] = 0u;
        if (q < t) {
            const uint64_t v = (hist[q] * (uint64_t)kRM) / (uint64_t)d;
            f[k] = v > 0 ? (uint32_t)v : 1u;
        }
        s += f[k];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    // the largest f, lowest q among ties, as f 2^8 + 255 - q
    auto top = [&]() {
        uint32_t b = 0;
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (4 * lane + k < t) b = max(b, (f[k] << 8) | (255u - (uint32_t)(4 * lane + k)));
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) b = max(b, (uint32_t)__shfl_xor(b, off));
        return (int)(255u - (b & 255u));
    };
    int32_t diff = (int32_t)kRM - (int32_t)s;  // uniform
    if (diff > 0) {
        const int j = top();
#pragma unroll
        for (int k = 0; k < 4; k++) f[k] += j == 4 * lane + k ? (uint32_t)diff : 0u;
    }
    for (; diff < 0; diff++) {  // the largest is above 1: the sum is above 2^16 >= t
        const int j = top();
#pragma unroll
        for (int k = 0; k < 4; k++) f[k] -= j == 4 * lane + k ? 1u : 0u;
    }
    uint32_t c = f[0] + f[1] + f[2] + f[3];
    const uint32_t own = c;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(c, off);
        if (lane >= off) c += y;
    }
    c -= own;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int q = 4 * lane + k;
        tab[q] = q < t ? enc_sym(f[k], c) : enc_sym(1u, 0u);
        c += f[k];
        if (q < t) {
            head[2 * q] = (uint8_t)((f[k] - 1u) & 0xFFu);
            head[2 * q + 1] = (uint8_t)((f[k] - 1u) >> 8);
        }
    }
}

// A lane per segment (some repeated).  The state's chain is two compares, two selects, a
// shift, the product's high half, a shift and a multiply-add; the bytes given
// off gather in 64 bits and leave four at a time.
__global__ __launch_bounds__(kRT) void k_rans_encode(const uint8_t* __restrict__ sym, int64_t d,
                                                     const EncSym* __restrict__ tab,
                                                     int32_t lanes, uint8_t* __restrict__ scratch,
                                                     uint32_t* __restrict__ lens, int64_t nseg) {
    __shared__ EncSym st[256];
    st[threadIdx.x] = tab[threadIdx.x];
    __syncthreads();
    const int lane = threadIdx.x % 64;
    const int64_t seg0 = ((int64_t)blockIdx.x * kRWaves + threadIdx.x / 64) * lanes;
    if (seg0 >= nseg) return;
    const int64_t seg = min(seg0 + lane % lanes, nseg - 1);
    const bool own = lane < lanes;  // the others' stores would only repeat these
    const uint8_t* in = sym + seg * kRSeg;
    const int n = (int)min((int64_t)kRSeg, d - seg * kRSeg);
    uint8_t* reg = scratch + seg * kRSegCap;
    int w = (int)kRSegCap;
    uint32_t x = kRL;
    uint64_t acc = 0;  // its low cnt bits: bytes not yet stored, the oldest on top
    uint32_t cnt = 0;
    auto flush = [&]() {
        if (cnt >= 32u) {
            cnt -= 32u;
            w -= 4;
            if (own) *reinterpret_cast<uint32_t*>(reg + w) = (uint32_t)(acc >> cnt);
        }
    };
    auto put = [&](uint32_t q) {
        const EncSym e = st[q];
        const uint32_t sh = bits_off(x, e.xtop);
        const uint32_t two = __builtin_amdgcn_perm(0u, x, 0x0c0c0001u);  // low two bytes, swapped
        acc = (acc << sh) | (two >> (16u - sh));
        cnt += sh;
        flush();
        x >>= sh;
        const uint32_t k = __umulhi(e.m, x) >> (e.cs >> 24);
        x = x + e.bias + __umul24(k, e.cs & 0xFFFFu);
    };
    const int nb = n / 16;
    uint32_t v[4] = {0u, 0u, 0u, 0u};
    if (nb > 0) __builtin_memcpy(v, in + 16 * (nb - 1), 16);
    for (int i = n - 1; i >= 16 * nb; i--) put(in[i]);
    for (int b = nb - 1; b >= 0; b--) {
        uint32_t u[4];
        __builtin_memcpy(u, in + 16 * max(b - 1, 0), 16);
#pragma unroll
        for (int k = 15; k >= 0; k--) put((v[k / 4] >> (8 * (k % 4))) & 255u);
#pragma unroll
        for (int k = 0; k < 4; k++) v[k] = u[k];
    }
    // the four bytes of the last state, low first
    acc = (acc << 32) | __builtin_bswap32(x);
    cnt += 32u;
    flush();
    while (cnt > 0u) {
        cnt -= 8u;
        reg[--w] = (uint8_t)(acc >> cnt);
    }
    lens[seg] = (uint32_t)(kRSegCap - w);
}

// One segment per wavefront, in LDS, coded by every lane alike.  A step stores two bytes
// below w and moves w by those that count (later bytes overwrite the others), so
// there is no branch in it; the table entries of the next 8 symbols are read
// while 8 are coded.
__global__ __launch_bounds__(kRT) void k_rans_encode_staged(const uint8_t* __restrict__ sym,
                                                            int64_t d,
                                                            const EncSym* __restrict__ tab,
                                                            uint8_t* __restrict__ scratch,
                                                            uint32_t* __restrict__ lens,
                                                            int64_t nseg) {
    __shared__ EncSym st[256];
    __shared__ __align__(16) uint8_t sy[kRWaves][kRSeg];
    __shared__ __align__(16) uint8_t so[kRWaves][kRSegCap];
    st[threadIdx.x] = tab[threadIdx.x];
    __syncthreads();
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int64_t seg = (int64_t)blockIdx.x * kRWaves + wave;
    if (seg >= nseg) return;
    const uint8_t* in = sym + seg * kRSeg;
    const int n = (int)min((int64_t)kRSeg, d - seg * kRSeg);
    const int nb = n / 8;
    for (int i = 16 * lane; i < n; i += 16 * 64) {
        uint32_t v[4] = {0u, 0u, 0u, 0u};
        if (i + 16 <= n)
            __builtin_memcpy(v, in + i, 16);
        else
            for (int k = 0; i + k < n; k++) v[k / 4] |= (uint32_t)in[i + k] << (8 * (k % 4));
        *reinterpret_cast<uint4*>(&sy[wave][i]) = make_uint4(v[0], v[1], v[2], v[3]);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    int w = (int)kRSegCap;
    {
        uint8_t* out = so[wave];
        const uint8_t* si = sy[wave];
        uint32_t x = kRL;
        auto put = [&](const EncSym& e) {
            const uint32_t sh = bits_off(x, e.xtop);
            out[w - 1] = (uint8_t)x;
            out[w - 2] = (uint8_t)(x >> 8);
            w -= (int)(sh >> 3);
            x >>= sh;
            const uint32_t k = __umulhi(e.m, x) >> (e.cs >> 24);
            x = x + e.bias + __umul24(k, e.cs & 0xFFFFu);
        };
        EncSym e[8], g[8];
        auto fetch = [&](int b, EncSym (&t)[8]) {
            const uint2 v = *reinterpret_cast<const uint2*>(si + 8 * max(b, 0));
#pragma unroll
            for (int k = 0; k < 8; k++) t[k] = st[((k < 4 ? v.x : v.y) >> (8 * (k % 4))) & 255u];
        };
        if (nb > 0) fetch(nb - 1, e);
        for (int i = n - 1; i >= 8 * nb; i--) put(st[si[i]]);
        for (int b = nb - 1; b >= 0; b--) {
            fetch(b - 1, g);
#pragma unroll
            for (int k = 7; k >= 0; k--) put(e[k]);
#pragma unroll
            for (int k = 0; k < 8; k++) e[k] = g[k];
        }
        for (int k = 0; k < 4; k++) out[--w] = (uint8_t)(x >> (8 * k));
    }
    w = __builtin_amdgcn_readfirstlane(w);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // whole 16-byte pieces of the slot (the bytes before w are not read)
    uint8_t* reg = scratch + seg * kRSegCap;
    for (int i = (w & ~15) + 16 * lane; i < (int)kRSegCap; i += 16 * 64)
        *reinterpret_cast<uint4*>(reg + i) = *reinterpret_cast<const uint4*>(&so[wave][i]);
    if (lane == 0) lens[seg] = (uint32_t)(kRSegCap - w);
}

// Inclusive scan of the segment lengths into the stream's end table
// (little-endian u32, byte by byte: the table need not be aligned); *total =
// the payload size.  One workgroup.
constexpr int kRScan = 1024;

__global__ __launch_bounds__(kRScan) void k_rans_offsets(const uint32_t* __restrict__ lens,
                                                         int64_t nseg, uint8_t* __restrict__ ends,
                                                         uint32_t* __restrict__ starts,
                                                         unsigned long long* __restrict__ total) {
    __shared__ uint32_t part[2][kRScan / 64];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    uint32_t carry = 0u;
    int odd = 0;
    for (int64_t b0 = 0; b0 < nseg; b0 += kRScan, odd ^= 1) {
        const int64_t k = b0 + threadIdx.x;
        const uint32_t v = k < nseg ? lens[k] : 0u;
        uint32_t e = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(e, off);
            if (lane >= off) e += y;
        }
        if (lane == 63) part[odd][wave] = e;
        __syncthreads();
        uint32_t sum = 0;
#pragma unroll
        for (int w = 0; w < kRScan / 64; w++) {
            const uint32_t y = part[odd][w];
            e += w < wave ? y : 0u;
            sum += y;
        }
        e += carry;
        carry += sum;
        if (k < nseg) {
            starts[k] = e - v;
            for (int q = 0; q < 4; q++) ends[4 * k + q] = (uint8_t)((e >> (8 * q)) & 0xFFu);
        }
    }
    if (threadIdx.x == 0) *total = carry;
}

// 16 bytes per thread at any alignment.
__global__ __launch_bounds__(256) void k_rans_pack(const uint8_t* __restrict__ scratch,
                                                   const uint32_t* __restrict__ lens,
                                                   const uint32_t* __restrict__ starts,
                                                   uint8_t* __restrict__ payload) {
    const int64_t seg = blockIdx.x;
    const uint32_t n = lens[seg];
    const uint8_t* src = scratch + seg * kRSegCap + (kRSegCap - n);
    uint8_t* dst = payload + starts[seg];
    const uint32_t nv = n / 16;
    for (uint32_t i = threadIdx.x; i < nv; i += 256) {
        uint32_t v[4];
        __builtin_memcpy(v, src + 16 * i, 16);
        __builtin_memcpy(dst + 16 * i, v, 16);
    }
    if (threadIdx.x < n - 16 * nv) dst[16 * nv + threadIdx.x] = src[16 * nv + threadIdx.x];
}

// Decoding table: an entry for every SL slots holds the symbol of the first of
// them, its c and its f - 1, and whether all have it: one LDS read takes a slot to
// its symbol except in the (at most t) entries that are shared, which go on
// through c.
constexpr uint32_t kDShared = 256u;
// Up to kDFew symbols an entry serves kDFewSlots slots: filling a table of 8 slots an entry takes
// about 10 us with 256 values (decoding 8 symbols: 75 us a call, 60 with the small table).
constexpr int kDFew = 32, kDFewSlots = 1024;

template <int SL>
struct DecBook {
    uint2 tab[kRM / SL];  // c | (f - 1) << 16; q | kDShared
    uint32_t sc[257];
    uint32_t part[kRWaves];
};

// False (in all threads) if the frequencies do not sum to 2^16.
template <int SL>
__device__ __forceinline__ bool load_dec_book(DecBook<SL>& B, const uint8_t* __restrict__ in,
                                              int32_t t) {
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    const uint32_t f0 =
        tid < t ? ((uint32_t)in[2 * tid] | ((uint32_t)in[2 * tid + 1] << 8)) + 1u : 0u;
    uint32_t cum = f0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(cum, off);
        if (lane >= off) cum += y;
    }
    if (lane == 63) B.part[wave] = cum;
    __syncthreads();
    uint32_t sum = 0;
#pragma unroll
    for (int w = 0; w < kRWaves; w++) {
        const uint32_t y = B.part[w];
        cum += w < wave ? y : 0u;
        sum += y;
    }
    if (sum != kRM) return false;
    B.sc[tid + 1] = cum;
    if (tid == 0) B.sc[0] = 0u;
    __syncthreads();
    uint32_t q = 0, c = 0, e = B.sc[1];
    if constexpr (SL == kDFewSlots) {  // one entry a thread: its symbol by a search (sc rises
                                       // up to sc[t] = 2^16)
#pragma unroll
        for (uint32_t step = 128; step > 0; step >>= 1)
            q += B.sc[q + step] <= (uint32_t)(SL * tid) ? step : 0u;
        c = B.sc[q];
        e = B.sc[q + 1];
    }
    for (int b = tid; b < (int)kRM / SL; b += kRT) {
        const uint32_t slot = (uint32_t)(SL * b);
        while (e <= slot) {  // sc[t] = 2^16 ends it
            q++;
            c = e;
            e = B.sc[q + 1];
        }
        B.tab[b] = make_uint2(c | ((e - c - 1u) << 16), q | (e < slot + SL ? kDShared : 0u));
    }
    __syncthreads();
    return true;
}

// Symbol of state x and the state without it (before its bytes).
template <int SL>
__device__ __forceinline__ uint32_t take_symbol(const DecBook<SL>& B, uint32_t x, uint32_t& q) {
    const uint32_t slot = x & (kRM - 1u);
    const uint2 e = B.tab[slot / SL];
    uint32_t c = e.x & 0xFFFFu, f1 = e.x >> 16;
    q = e.y;
    if (q & kDShared) {
        q &= 255u;
        uint32_t top = c + f1 + 1u;
        while (top <= slot) {
            q++;
            c = top;
            top = B.sc[q + 1];
        }
        f1 = top - c - 1u;
    }
    const uint32_t xh = x >> 16;
    return __umul24(f1, xh) + (xh + (slot - c));
}

// Where segment seg's bytes lie: false if they are too few or past the end.
__device__ __forceinline__ bool segment_bytes(const uint8_t* __restrict__ in, int64_t nin,
                                              int32_t t, int64_t nseg, int64_t seg, int64_t& lo,
                                              int64_t& hi) {
    const uint8_t* ends = in + 2 * t;
    auto end_at = [&](int64_t k) {
        return (int64_t)((uint32_t)ends[4 * k] | ((uint32_t)ends[4 * k + 1] << 8) |
                         ((uint32_t)ends[4 * k + 2] << 16) | ((uint32_t)ends[4 * k + 3] << 24));
    };
    const int64_t pay = 2 * (int64_t)t + 4 * nseg;
    lo = pay + (seg == 0 ? 0 : end_at(seg - 1));
    hi = pay + end_at(seg);
    return !(lo + 4 > hi || hi > nin);
}

// The first state, at pos; pos moves on.  No stream of the encoder starts below
// L: there the first symbol may need any number of bytes and is decoded here, q >= 0
// (afterwards x >= L, and a symbol takes two bytes at most).  False: out of bytes.
template <int SL>
__device__ __forceinline__ bool first_state(const DecBook<SL>& B, const uint8_t* __restrict__ in,
                                            int64_t hi, int64_t& pos, uint32_t& x, int& q) {
    x = ((uint32_t)in[pos] << 24) | ((uint32_t)in[pos + 1] << 16) | ((uint32_t)in[pos + 2] << 8) |
        (uint32_t)in[pos + 3];
    pos += 4;
    q = -1;
    if (x >= kRL) return true;
    uint32_t q0;
    x = take_symbol(B, x, q0);
    while (x < kRL) {
        if (pos >= hi) return false;
        x = (x << 8) | in[pos++];
    }
    q = (int)q0;
    return true;
}

// x after symbol q's bytes b0, b1 (y >= 2^7); n: how many it took, one below L =
// 2^23 and two below 2^15, from the leading zeros: a select waits longer for its compare than
// these shifts take.
__device__ __forceinline__ uint32_t with_bytes(uint32_t y, uint32_t b0, uint32_t b1, uint32_t& n) {
    const uint32_t z = (uint32_t)__builtin_clz(y);
    const uint32_t sh = __builtin_elementwise_sub_sat(z, 1u) & 24u;
    n = sh >> 3;
    const uint64_t w = ((uint64_t)y << 32) | (b0 << 24) | (b1 << 16);
    return (uint32_t)((w << sh) >> 32);
}

// Many segments: one lane each, straight from and to memory.  An entry for every 4
// slots (128 KB: one workgroup to a CU), so that the shared ones are rarely met by any of a
// wavefront's lanes; each lane keeps its next 64 stream bytes in LDS, and a copy
// of the first after the last (a byte and the one after it are always neighbours).
// bad: set when the frequencies do not sum to 2^16 or a segment runs past its
// bytes or does not end in the initial state.
constexpr int kDRing = 17;  // 32-bit words

__global__ __launch_bounds__(kRT) void k_rans_decode(const uint8_t* __restrict__ in, int64_t nin,
                                                     int64_t d, int32_t t, int32_t lanes,
                                                     int64_t nseg, uint8_t* __restrict__ sym,
                                                     unsigned int* __restrict__ bad) {
    __shared__ DecBook<4> B;
    __shared__ uint32_t ring[kRT][kDRing];
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    if (!load_dec_book(B, in, t)) {  // uniform
        if (tid == 0) atomicAdd(bad, 1u);
        return;
    }
    const int64_t seg0 = ((int64_t)blockIdx.x * kRWaves + wave) * lanes;
    if (seg0 >= nseg) return;
    const int64_t seg = min(seg0 + lane % lanes, nseg - 1);
    int64_t pos, hi;
    uint32_t x;
    int q0;
    if (!segment_bytes(in, nin, t, nseg, seg, pos, hi) || !first_state(B, in, hi, pos, x, q0)) {
        atomicAdd(bad, 1u);
        return;
    }
    uint8_t* out = sym + seg * kRSeg;
    const int n = (int)min((int64_t)kRSeg, d - seg * kRSeg);
    int i = 0;
    if (q0 >= 0) out[i++] = (uint8_t)q0;
    uint32_t* rg = ring[tid];
    const uint8_t* rb = reinterpret_cast<const uint8_t*>(rg);
    auto load16 = [&](int64_t at, uint32_t* v) {
        if (at + 16 <= nin) {
            __builtin_memcpy(v, in + at, 16);
        } else {
#pragma unroll
            for (int w = 0; w < 4; w++) {
                v[w] = 0u;
                for (int k = 0; k < 4; k++)
                    if (at + 4 * w + k < nin) v[w] |= (uint32_t)in[at + 4 * w + k] << (8 * k);
            }
        }
    };
    // bytes wr.. of the segment are not in the ring yet; the next 32 wait in R
    uint32_t R[8];
    uint32_t rd = 0, wr = 64;
#pragma unroll
    for (int h = 0; h < 2; h++) {
        load16(pos + 32 * h, R);
        load16(pos + 32 * h + 16, R + 4);
#pragma unroll
        for (int k = 0; k < 8; k++) rg[8 * h + k] = R[k];
        if (h == 0) rg[16] = R[0];
    }
    load16(pos + wr, R);
    load16(pos + wr + 16, R + 4);
    // 16 symbols take at most 32 bytes
    auto refill = [&]() {
        if (wr - rd <= 32u) {
            const uint32_t at = wr & 63u;
#pragma unroll
            for (int k = 0; k < 8; k++) rg[at / 4 + k] = R[k];
            if (at == 0u) rg[16] = R[0];
            wr += 32u;
            load16(pos + wr, R);
            load16(pos + wr + 16, R + 4);
        }
    };
    auto step = [&]() {
        const uint32_t at = rd & 63u;
        const uint32_t b0 = rb[at], b1 = rb[at + 1];
        uint32_t q, nt;
        const uint32_t y = take_symbol(B, x, q);
        x = with_bytes(y, b0, b1, nt);
        rd += nt;
        return q;
    };
    for (; i + 16 <= n; i += 16) {
        refill();
        uint32_t o[4];
#pragma unroll
        for (int k = 0; k < 16; k++) {
            const uint32_t q = step();
            o[k / 4] = k % 4 == 0 ? q : o[k / 4] | (q << (8 * (k % 4)));
        }
        if (lane < lanes) __builtin_memcpy(out + i, o, 16);
    }
    refill();
    for (; i < n; i++) out[i] = (uint8_t)step();
    if (x != kRL || pos + (int64_t)rd != hi) atomicAdd(bad, 1u);
}

// One segment per wavefront, in LDS (entries of 8 slots leave room for it), decoded
// by every lane alike.  From its first state on a segment takes at most two bytes a symbol.
constexpr int kDSegCap = 2 * kRSeg;

template <int SL>
__global__ __launch_bounds__(kRT) void k_rans_decode_staged(const uint8_t* __restrict__ in,
                                                            int64_t nin, int64_t d, int32_t t,
                                                            int64_t nseg,
                                                            uint8_t* __restrict__ sym,
                                                            unsigned int* __restrict__ bad) {
    __shared__ DecBook<SL> B;
    __shared__ __align__(16) uint8_t si[kRWaves][kDSegCap + 16];
    __shared__ __align__(16) uint8_t so[kRWaves][kRSeg];
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
    if (!load_dec_book(B, in, t)) {  // uniform
        if (tid == 0) atomicAdd(bad, 1u);
        return;
    }
    const int64_t seg = (int64_t)blockIdx.x * kRWaves + wave;
    if (seg >= nseg) return;
    int64_t pos, hi;
    uint32_t x;
    int q0;
    // (all lanes alike)
    if (!segment_bytes(in, nin, t, nseg, seg, pos, hi) || !first_state(B, in, hi, pos, x, q0) ||
        hi - pos > kDSegCap) {
        if (lane == 0) atomicAdd(bad, 1u);
        return;
    }
    const int len = (int)(hi - pos);
    for (int i = 16 * lane; i < len; i += 16 * 64) {
        uint32_t v[4] = {0u, 0u, 0u, 0u};
        if (i + 16 <= len)
            __builtin_memcpy(v, in + pos + i, 16);
        else
            for (int k = 0; i + k < len; k++) v[k / 4] |= (uint32_t)in[pos + i + k] << (8 * (k % 4));
        *reinterpret_cast<uint4*>(&si[wave][i]) = make_uint4(v[0], v[1], v[2], v[3]);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int n = (int)min((int64_t)kRSeg, d - seg * kRSeg);
    {
        const uint8_t* src = si[wave];
        uint32_t* dst = reinterpret_cast<uint32_t*>(so[wave]);
        uint32_t rd = 0;
        auto step = [&]() {
            // (past its bytes a segment reads the last ones again: rd != len reports it)
            const uint32_t at = min(rd, (uint32_t)kDSegCap);
            const uint32_t b0 = src[at], b1 = src[at + 1];
            uint32_t q, nt;
            const uint32_t y = take_symbol(B, x, q);
            x = with_bytes(y, b0, b1, nt);
            rd += nt;
            return q;
        };
        int i = 0;
        uint32_t o = 0;
        if (q0 >= 0) {
            // the word that the first symbol opens
            o = (uint32_t)q0;
            for (i = 1; i < 4 && i < n; i++) o |= step() << (8 * i);
            dst[0] = o;
        }
        for (; i + 4 <= n; i += 4) {
            o = step();
#pragma unroll
            for (int k = 1; k < 4; k++) o |= step() << (8 * k);
            dst[i / 4] = o;
        }
        if (i < n) {
            o = 0;
            for (int k = 0; i + k < n; k++) o |= step() << (8 * k);
            dst[i / 4] = o;
        }
        if (lane == 0 && (x != kRL || rd != (uint32_t)len)) atomicAdd(bad, 1u);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    uint8_t* out = sym + seg * kRSeg;
    for (int i = 16 * lane; i < n; i += 16 * 64) {
        if (i + 16 <= n)
            __builtin_memcpy(out + i, &so[wave][i], 16);
        else
            for (int k = 0; i + k < n; k++) out[i + k] = so[wave][i + k];
    }
}

}  // namespace

int64_t rans_segments(int64_t d) { return (d + kRSeg - 1) / kRSeg; }

size_t rans_bound(int64_t d, int32_t t) {
    const int64_t nseg = rans_segments(d);
    return (size_t)(2 * (int64_t)t + 8 * nseg + 2 * d);
}

// the counts, the encoding table, what the host reads back (RansResult), the
// segments' lengths and starts, then their slots
size_t rans_scratch_bytes(int64_t d) {
    const int64_t nseg = rans_segments(d);
    return align256(sizeof(unsigned long long) * 256 + sizeof(RansResult)) +
           align256(sizeof(EncSym) * 256) + 2 * align256(sizeof(uint32_t) * (size_t)nseg) +
           (size_t)nseg * kRSegCap;
}

hipError_t launch_rans_encode(const uint8_t* sym, int64_t d, int32_t t, uint8_t* out,
                              char* scratch, const RansResult** result, hipStream_t st) {
    const int64_t nseg = rans_segments(d);
    char* p = scratch;
    auto take = [&](size_t b) {
        char* r = p;
        p += align256(b);
        return r;
    };
    constexpr size_t kHist = sizeof(unsigned long long) * 256;
    auto* hist = reinterpret_cast<unsigned long long*>(take(kHist + sizeof(RansResult)));
    auto* res = reinterpret_cast<RansResult*>(reinterpret_cast<char*>(hist) + kHist);
    auto* tab = reinterpret_cast<EncSym*>(take(sizeof(EncSym) * 256));
    auto* lens = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t) * (size_t)nseg));
    auto* starts = reinterpret_cast<uint32_t*>(take(sizeof(uint32_t) * (size_t)nseg));
    auto* regions = reinterpret_cast<uint8_t*>(p);
    *result = res;
    hipError_t e = hipMemsetAsync(hist, 0, kHist + sizeof(RansResult), st);
    if (e != hipSuccess) return e;
    int64_t g = (d + 4095) / 4096;
    if (g > 1024) g = 1024;
    k_sym_hist<<<(unsigned)g, 256, 0, st>>>(sym, d, t, hist, &res->bad);
    k_rans_freqs<<<1, 64, 0, st>>>(hist, t, d, tab, out);
    const int32_t lanes = lanes_of(nseg);
    const int64_t per = (int64_t)lanes * kRWaves;
    const unsigned wg = (unsigned)((nseg + per - 1) / per);
    if (staged(nseg))
        k_rans_encode_staged<<<wg, kRT, 0, st>>>(sym, d, tab, regions, lens, nseg);
    else
        k_rans_encode<<<wg, kRT, 0, st>>>(sym, d, tab, lanes, regions, lens, nseg);
    k_rans_offsets<<<1, kRScan, 0, st>>>(lens, nseg, out + 2 * t, starts, &res->total);
    k_rans_pack<<<(unsigned)nseg, 256, 0, st>>>(regions, lens, starts,
                                                out + 2 * (int64_t)t + 4 * nseg);
    return hipGetLastError();
}

hipError_t launch_rans_decode(const uint8_t* in, int64_t nin, int64_t d, int32_t t, uint8_t* sym,
                              unsigned int* bad, hipStream_t st) {
    const int64_t nseg = rans_segments(d);
    const int32_t lanes = lanes_of(nseg);
    const int64_t per = (int64_t)lanes * kRWaves;
    const unsigned wg = (unsigned)((nseg + per - 1) / per);
    if (d <= kDFew)
        k_rans_decode_staged<kDFewSlots><<<wg, kRT, 0, st>>>(in, nin, d, t, nseg, sym, bad);
    else if (staged(nseg))
        k_rans_decode_staged<8><<<wg, kRT, 0, st>>>(in, nin, d, t, nseg, sym, bad);
    else
        k_rans_decode<<<wg, kRT, 0, st>>>(in, nin, d, t, lanes, nseg, sym, bad);
    return hipGetLastError();
}

}  // namespace ecasq
