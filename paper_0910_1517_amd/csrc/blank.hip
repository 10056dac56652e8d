// Time-domain MAD voltage blanker (section 5, Eq. 3 and 4) and its noise
// table.
//
// The blanker runs on the int8 voltage rows the F-engine reads, before the
// FFT.  Each block of B consecutive samples of one signal gets its median x~
// and MAD = median |x - x~|.  A sample with |x - x~| > M MAD / 0.6745 is
// replaced by rint(x~ + sigma z) clamped to int8, where sigma = MAD / 0.6745
// (the robust estimate of the voltage RMS for normal noise) and z comes from a
// precomputed Gaussian noise table with one row per signal, so the
// replacements of different antennas are independent.  A block with MAD = 0
// has no scale estimate and passes unchanged.
//
// A block (up to 64 KiB) is loaded once into registers, 32 G samples a lane,
// by one wave up to 8192 samples (out of place 4096) and by two, four or eight
// above, and never re-read.  Its statistics are exact order statistics taken bit by bit: each
// group of 32 samples of a lane is transposed into 8 words, one per bit (word
// p holds bit p of the 32 samples), after which one instruction handles 32
// samples.  The k-th smallest value is found from its top bit down: of the
// candidates, count those with the bit clear; if k of them or more, keep
// these, else keep the others and take k less.  |x - x~| is a subtraction in
// the same form (the median is uniform, so its bits are constants), the
// comparison of Eq. 4 another.  What it costs: about 50 instructions of
// transposing and 90 of selection per 32 samples, and one sum over the wave
// per bit.  A histogram, the other way to the same numbers, needs one LDS atomic
// per sample: 64 x 8388613 four-bit samples in blocks of 4096 took 424 us that
// way, now 200 us (0.54 GB read; 91 us at the card's read rate; the vector ALUs
// are busy 92% of it), 64 x 2^24 eight-bit samples in blocks of 4096 582 us, now
// 297, in blocks of 16384 297 and 285.
// The threshold test |x - x~| > M MAD / 0.6745 is one FP64 expression per
// block, turned into the integer range [lo, hi] of values kept.  The blanked
// positions of a block are queued in LDS, and all lanes then compute their
// replacements from the table in FP64 and store them as single bytes.  Out of
// place, the block is copied (where the registers hold it that long, just before
// the replacements) and they patch the copy; in place, only the blanked bytes are
// written.
//
// Noise table: entry j of signal s is the Irwin-Hall sum of twelve 16-bit
// uniforms (U + 1/2) / 65536, minus 6.  The uniforms are the 16-bit halves
// (low, then high) of words 0..3 of Philox4x32-10 at counter (j, j >> 32, s,
// 0) and of words 0..1 at counter (j, j >> 32, s, 1), keyed by the 64-bit
// seed (Salmon, Moraes, Dror and Shaw, SC'11).  Every entry is a multiple of
// 2^-16 below 6 in magnitude, so it is exact in float.

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>

#include "corr_internal.h"

namespace {

constexpr int kBlankQueue = 2048;                 // 16-bit positions a wave's LDS queue holds
constexpr int kBlankMaxSignals = 65535;           // grid y
constexpr int kBlankMaxBlock = 65536;             // eight waves of 8192 samples
constexpr int64_t kBlankMaxTable = 1ll << 31;

// ---------------------------------------------------------------- Philox
// One Philox4x32-10 block: ten rounds of two 32x32->64 products whose halves
// are mixed with the other two words and the round key; the key advances by
// the Weyl constants between rounds.
__device__ inline uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(0xD2511F53u, c.x), lo0 = 0xD2511F53u * c.x;
        const uint32_t hi1 = __umulhi(0xCD9E8D57u, c.z), lo1 = 0xCD9E8D57u * c.z;
        c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

__device__ inline uint32_t halves(uint32_t w) { return (w & 0xFFFFu) + (w >> 16); }

__global__ __launch_bounds__(256) void noise_table_kernel(uint32_t k0, uint32_t k1, int64_t total, int lg_L,
                                                          float *table) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        const uint64_t j = (uint64_t)e & ((1ull << lg_L) - 1);
        const uint32_t s = (uint32_t)((uint64_t)e >> lg_L);
        const uint4 a = philox4x32_10(make_uint4((uint32_t)j, (uint32_t)(j >> 32), s, 0u), k0, k1);
        const uint4 b = philox4x32_10(make_uint4((uint32_t)j, (uint32_t)(j >> 32), s, 1u), k0, k1);
        const int32_t sum = (int32_t)(halves(a.x) + halves(a.y) + halves(a.z) + halves(a.w) + halves(b.x) +
                                      halves(b.y));
        // sum of (U + 1/2) / 65536 over 12, minus 6; |numerator| < 2^19: exact
        table[e] = (float)(sum + 6 - 6 * 65536) * (1.0f / 65536.0f);
    }
}

// ---------------------------------------------------------------- blanker
// Inclusive prefix sum of v over the wave's lanes: row shifts, then the totals
// of the rows before.
__device__ inline uint32_t wave_prefix(uint32_t v) {
    int x = (int)v;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, true);  // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, true);  // row_bcast:31 into rows 2 and 3
    return (uint32_t)x;
}

// v / 0.6745, correctly rounded: a first quotient from the rounded reciprocal,
// corrected once by its exact remainder (Markstein).  v is 0 or at least 2^-151.
__device__ inline double over_6745(double v) {
    constexpr double c = 0.6745, y = 1.0 / c;
    const double q = v * y;
    return fma(fma(-q, c, v), y, q);
}

// Replacement value of a blanked sample: rint(x~ + sigma z), clamped, all in
// FP64 with every product and sum rounded on its own.
__device__ inline uint32_t replacement(double half_med2, double sigma, float z) {
#pragma clang fp contract(off)
    double r = rint(half_med2 + sigma * (double)z);
    r = fmin(fmax(r, -128.0), 127.0);
    return (uint32_t)(int32_t)r & 0xFFu;
}

// Bits of 32 samples, one word per sample bit: word p, bit 8 b + r = bit p of
// byte b of w[r] (an 8 x 8 bit transpose in each byte lane).
__device__ inline void bit_planes(uint32_t (&w)[8]) {
    auto swap = [&](int i, int j, int sh, uint32_t m) {  // exchange the sh-bit fields of rows i < j
        const uint32_t a = w[i], b = w[j];
        w[i] = (a & m) | ((b << sh) & ~m);
        w[j] = ((a >> sh) & m) | (b & ~m);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) swap(i, i + 4, 4, 0x0F0F0F0Fu);
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (!(i & 2)) swap(i, i + 2, 2, 0x33333333u);
#pragma unroll
    for (int i = 0; i < 8; i += 2) swap(i, i + 1, 1, 0x55555555u);
}

// NW waves hold one block, G groups of 32 samples a lane (a workgroup of four
// waves has four blocks when NW = 1): group g, chunk h of lane l is chunk
// l + 64 NW (2 g + h) of the block.  A lane's words past the block's end, whole
// or in part, are left out by the groups' valid masks.  COPY: how the block gets
// to the output of a call out of place -- early, as it is loaded, or late, just
// before the replacements patch it, which finds the lines still in L2 (64 x 2^24
// samples in blocks of 4096: 522 us early, 395 late; in place 297) where the
// registers hold the samples meanwhile.
constexpr int kInPlace = 0, kCopyEarly = 1, kCopyLate = 2;
template <int G, int NW, int COPY>
__global__ __launch_bounds__(NW == 1 ? 256 : 64 * NW) void blank_kernel(
    const int8_t *__restrict__ x, int8_t *out, int64_t row_stride, int64_t n, int B, double M,
    const float *__restrict__ table, int64_t L, int64_t sample0, int32_t *counts, int32_t *stats) {
    constexpr int TB = 64 * NW;               // threads of a block
    constexpr int WPG = NW == 1 ? 4 : NW;     // waves of the workgroup
    __shared__ uint16_t queue_lds[WPG * kBlankQueue];
    __shared__ uint32_t red[2][NW];
    const int t = NW == 1 ? threadIdx.x & 63 : threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t nblk = (n + B - 1) / B, blk = NW == 1 ? (int64_t)blockIdx.x * 4 + wave : blockIdx.x;
    if (blk >= nblk) return;  // a whole wave; NW = 1 has no barrier
    const int s = blockIdx.y;
    const int64_t i0 = blk * B;
    const int len = (int)min((int64_t)B, n - i0);
    const int8_t *xr = x + (int64_t)s * row_stride + i0;
    int8_t *orow = out + (int64_t)s * row_stride + i0;

    uint32_t u[G][8], valid[G];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = t + TB * (2 * g + h);
            const uint4 v = c * 16 < len ? *reinterpret_cast<const uint4 *>(xr + c * 16) : make_uint4(0, 0, 0, 0);
            u[g][4 * h] = v.x;
            u[g][4 * h + 1] = v.y;
            u[g][4 * h + 2] = v.z;
            u[g][4 * h + 3] = v.w;
        }
    auto copy = [&](const uint32_t (&v)[G][8]) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c = t + TB * (2 * g + h), nv = len - c * 16;
                const uint32_t *w = &v[g][4 * h];
                if (nv >= 16) {
                    *reinterpret_cast<uint4 *>(orow + c * 16) = make_uint4(w[0], w[1], w[2], w[3]);
                } else if (nv > 0) {
#pragma unroll
                    for (int k = 0; k < 16; ++k)
                        if (k < nv) orow[c * 16 + k] = (int8_t)(w[k >> 2] >> (8 * (k & 3)));
                }
            }
    };
    if constexpr (COPY == kCopyEarly) copy(u);
    uint32_t raw[COPY == kCopyLate ? G : 1][8];
    if constexpr (COPY == kCopyLate) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int q = 0; q < 8; ++q) raw[g][q] = u[g][q];
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        bit_planes(u[g]);
        u[g][7] = ~u[g][7];  // two's complement -> x + 128
        uint32_t m = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int nv = len - (t + TB * (2 * g + h)) * 16;  // samples of the chunk
            if (nv >= 16) {
                m |= 0x0F0F0F0Fu << (4 * h);
            } else if (nv > 0) {  // sample 4 d + b of the chunk: bit 8 b + 4 h + d
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    if (k < nv) m |= 1u << (8 * (k & 3) + 4 * h + (k >> 2));
            }
        }
        valid[g] = m;
    }

    int parity = 0;
    auto block_total = [&](uint32_t v) -> uint32_t {  // of the waves' totals v
        if constexpr (NW > 1) {
            if (t % 64 == 0) red[parity][wave] = v;
            __syncthreads();  // the other half of red may still be read by a wave behind
            v = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) v += red[parity][w];
            v = __builtin_amdgcn_readfirstlane(v);
            parity ^= 1;
        }
        return v;
    };
    auto wave_total = [&](uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)wave_prefix(v), 63); };
    // k-th smallest (k >= 1) of the valid values in planes p, and the (k + 1)-th if
    // there is one
    auto select = [&](const uint32_t (&p)[G][8], uint32_t k, uint32_t &rest) -> int {
        uint32_t cand[G], ceq = (uint32_t)len;
        int value = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) cand[g] = valid[g];
#pragma unroll
        for (int b = 7; b >= 0; --b) {
            uint32_t c = 0;
#pragma unroll
            for (int g = 0; g < G; ++g) c += __builtin_popcount(cand[g] & ~p[g][b]);
            c = block_total(wave_total(c));
            const bool low = k <= c;
            const uint32_t flip = low ? ~0u : 0u;
            value |= low ? 0 : 1 << b;
            k -= low ? 0 : c;
            ceq = low ? c : ceq - c;
#pragma unroll
            for (int g = 0; g < G; ++g) cand[g] &= p[g][b] ^ flip;
        }
        rest = ceq - k;  // values equal to it that rank after it
        return value;
    };
    auto select2 = [&](const uint32_t (&p)[G][8], uint32_t k1, uint32_t k2) -> int {  // sum of the two
        uint32_t rest, unused;
        const int v1 = select(p, k1, rest);
        return v1 + (k2 == k1 || rest > 0 ? v1 : select(p, k2, unused));
    };

    // median (Eq. 3): half the sum of the k1-th and k2-th smallest (equal for odd
    // len); med2 = 2 x~, medu = 2 (x~ + 128)
    const uint32_t k1 = (uint32_t)(len + 1) >> 1, k2 = (uint32_t)(len >> 1) + 1;
    const int medu = select2(u, k1, k2), med2 = medu - 256;

    // MAD (Eq. 3): with m = ceil(medu / 2) and D = u - m, |2 x - med2| is 2 |D| for
    // an even medu; for an odd one it is 2 D + 1 where D >= 0 and 2 (-D - 1) + 1
    // where D < 0.  e = |D|, or D with its bits inverted where negative: D xor its
    // sign, plus the sign when medu is even.
    const int m = (medu + 1) >> 1;
    const uint32_t even = (medu & 1) ? 0u : ~0u;
    // (e takes u's place: Eq. 4 is tested on it)
#pragma unroll
    for (int g = 0; g < G; ++g) {
        uint32_t borrow = 0;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint32_t mb = ((m >> b) & 1) ? ~0u : 0u, a = u[g][b], d = a ^ mb;
            u[g][b] = d ^ borrow;
            borrow = (~a & mb) | (~d & borrow);
        }
        uint32_t carry = borrow & even;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint32_t d = u[g][b] ^ borrow;
            u[g][b] = d ^ carry;
            carry &= d;
        }
    }
    const int mad4 = 2 * select2(u, k1, k2) + (even ? 0 : 2);

    // Eq. 4, |2x - med2| > 2 M MAD / 0.6745, as e > most: e of 2 e or 2 e + 1
    int most = 255;
    if (mad4 > 0) {
        const double mad = (double)mad4 * 0.25;
        const double thr2 = 2.0 * over_6745(M * mad);
        const int dmax = thr2 >= 511.0 ? 511 : (int)floor(thr2);
        most = even ? dmax >> 1 : (dmax - 1) >> 1;
    }
    uint32_t mine = 0, bad[G];
#pragma unroll
    for (int g = 0; g < G; ++g) bad[g] = 0;
    if (most < 255) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            uint32_t gt = 0;
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const uint32_t hb = ((most >> b) & 1) ? ~0u : 0u, a = u[g][b];
                gt = (a & ~hb) | (~(a ^ hb) & gt);
            }
            bad[g] = (most < 0 ? ~0u : gt) & valid[g];
            mine += (uint32_t)__builtin_popcount(bad[g]);
        }
    }
    const uint32_t pre = wave_prefix(mine);
    const int total = __builtin_amdgcn_readlane((int)pre, 63);  // of this wave
    const int n_out = (int)block_total((uint32_t)total);
    if (t == 0) {
        const int64_t o = (int64_t)s * nblk + blk;
        if (counts) counts[o] = n_out;
        if (stats) {
            stats[2 * o] = med2;
            stats[2 * o + 1] = mad4;
        }
    }
    if constexpr (COPY == kCopyLate) copy(raw);
    if (n_out == 0) return;  // nothing to blank (uniform over the block)

    const float *trow = table + (int64_t)s * L;
    const int64_t Lmask = L - 1, p_blk = sample0 + i0;
    const double half_med2 = 0.5 * (double)med2;
    const double sigma = over_6745((double)mad4 * 0.25);
    // bit q of group g of lane l of this wave: chunk, word and byte of the block
    const int l0 = NW == 1 ? 0 : wave * 64;
    auto place = [&](int e) {
        const int l = e >> 8, g = (e >> 5) & 7, q = e & 31;
        return (l0 + l + TB * (2 * g + ((q >> 2) & 1))) * 16 + 4 * (q & 3) + (q >> 3);
    };
    auto value = [&](int pos) { return trow[(p_blk + pos) & Lmask]; };
    auto put = [&](int pos, float z) { orow[pos] = (int8_t)replacement(half_med2, sigma, z); };
    if constexpr (NW > 1) __syncthreads();  // out of place: every wave's copy is on its way
    const int lane = threadIdx.x & 63;
    // Each wave queues its blanked samples (lane, group, bit), then replaces them with
    // all its lanes: all groups at once, or, where there are more than the queue holds
    // (strong interference, a small M), a group at a time, whose samples always fit.
    // 64 x 2^22 samples out of place, two thirds of them blanked: 293 us in blocks of 4096,
    // 349 of 16384; with each lane replacing its own in that case 827 and 729.
    static_assert(G <= 8, "14 bits an entry");
    static_assert(64 * 32 <= kBlankQueue, "a group fits");
    uint16_t *queue = queue_lds + wave * kBlankQueue;
    auto push = [&](uint16_t *next, int g) {
        for (uint32_t w = bad[g]; w; w &= w - 1) *next++ = (uint16_t)(lane << 8 | g << 5 | __builtin_ctz(w));
        return next;
    };
    auto wave_order = [] {  // the wave's own LDS order suffices
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto replace = [&](int n) {
        wave_order();
        int i = lane;
        // many: four table values of a lane in flight (one at a time each waits out the
        // memory latency, which the few waves of the larger blocks do not hide: 64 x 2^22
        // samples in blocks of 16384, bursts on 30%: 281 us so, 219 now)
        constexpr int F = 4;
        for (; n - (i - lane) >= 64 * F; i += 64 * F) {
            int pos[F];
            float z[F];
#pragma unroll
            for (int f = 0; f < F; ++f) pos[f] = place(queue[i + 64 * f]);
#pragma unroll
            for (int f = 0; f < F; ++f) z[f] = value(pos[f]);
#pragma unroll
            for (int f = 0; f < F; ++f) put(pos[f], z[f]);
        }
        for (; i < n; i += 64) {
            const int pos = place(queue[i]);
            put(pos, value(pos));
        }
    };
    if (total <= kBlankQueue) {
        uint16_t *next = queue + (pre - mine);
#pragma unroll
        for (int g = 0; g < G; ++g) next = push(next, g);
        replace(total);
        return;
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint32_t own = (uint32_t)__builtin_popcount(bad[g]), upto = wave_prefix(own);
        push(queue + (upto - own), g);
        replace(__builtin_amdgcn_readlane((int)upto, 63));
        wave_order();
    }
}

template <int G, int NW, int COPY>
hipError_t launch_blank(const int8_t *x, int8_t *out, int64_t row_stride, int S, int64_t n, int B, double M,
                        const float *table, int64_t L, int64_t sample0, int32_t *counts, int32_t *stats,
                        hipStream_t st) {
    const int64_t nblk = (n + B - 1) / B;
    const dim3 grid((unsigned)(NW == 1 ? (nblk + 3) / 4 : nblk), (unsigned)S);
    hipLaunchKernelGGL((blank_kernel<G, NW, COPY>), grid, dim3(NW == 1 ? 256 : 64 * NW), 0, st, x, out, row_stride, n,
                       B, M, table, L, sample0, counts, stats);
    return hipGetLastError();
}

thread_local char g_blank_err[512];

corr_status blank_fail(corr_status st, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(g_blank_err, sizeof(g_blank_err), fmt, ap);
    va_end(ap);
    return st;
}

bool is_aligned(const void *p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

}  // namespace

extern "C" {

corr_status corr_blank_noise_table(uint64_t seed, int32_t S, int64_t L, float *d_table, void *stream) {
    g_blank_err[0] = 0;
    if (!d_table) return blank_fail(CORR_ERR_NULL, "d_table is required");
    if (!is_aligned(d_table, 4)) return blank_fail(CORR_ERR_ALIGN, "d_table must be 4-byte aligned");
    if (S < 1 || S > kBlankMaxSignals) return blank_fail(CORR_ERR_INVALID, "S=%d outside [1, %d]", S, kBlankMaxSignals);
    if (L < 1 || L > kBlankMaxTable || (L & (L - 1)))
        return blank_fail(CORR_ERR_INVALID, "L=%lld must be a power of two in [1, 2^31]", (long long)L);
    int lg = 0;
    while ((1ll << lg) < L) ++lg;
    const int64_t total = (int64_t)S * L;
    const int64_t want = (total + 255) / 256;
    const unsigned grid = (unsigned)(want < 65536 ? want : 65536);
    hipLaunchKernelGGL(noise_table_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, (uint32_t)seed,
                       (uint32_t)(seed >> 32), total, lg, d_table);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? CORR_OK
                           : blank_fail(CORR_ERR_DEVICE, "noise table launch: %s", hipGetErrorString(e));
}

corr_status corr_blank_voltages(const int8_t *d_x, int64_t row_stride, int32_t S, int64_t n, int32_t block, float M,
                                const float *d_table, int64_t table_len, int64_t sample0, int8_t *d_out,
                                int32_t *d_counts, int32_t *d_stats, void *stream) {
    g_blank_err[0] = 0;
    if (!d_x || !d_table || !d_out) return blank_fail(CORR_ERR_NULL, "d_x, d_table and d_out are required");
    if (!is_aligned(d_x, 16) || !is_aligned(d_out, 16) || !is_aligned(d_table, 4) ||
        (d_counts && !is_aligned(d_counts, 4)) || (d_stats && !is_aligned(d_stats, 4)))
        return blank_fail(CORR_ERR_ALIGN, "d_x and d_out need 16-byte, d_table, d_counts and d_stats 4-byte alignment");
    if (S < 1 || S > kBlankMaxSignals) return blank_fail(CORR_ERR_INVALID, "S=%d outside [1, %d]", S, kBlankMaxSignals);
    if (n < 0) return blank_fail(CORR_ERR_INVALID, "n=%lld is negative", (long long)n);
    if (row_stride % 16 || row_stride < n)
        return blank_fail(CORR_ERR_INVALID, "row_stride=%lld must be a multiple of 16 and >= n", (long long)row_stride);
    if (block < 16 || block > kBlankMaxBlock || block % 16)
        return blank_fail(CORR_ERR_INVALID, "block=%d must be a multiple of 16 in [16, %d]", block, kBlankMaxBlock);
    if (!(M > 0.f) || !std::isfinite(M)) return blank_fail(CORR_ERR_INVALID, "threshold M must be finite and > 0");
    if (table_len < 1 || table_len > kBlankMaxTable || (table_len & (table_len - 1)))
        return blank_fail(CORR_ERR_INVALID, "table_len=%lld must be a power of two in [1, 2^31]", (long long)table_len);
    if (sample0 < 0 || sample0 > INT64_MAX - n)
        return blank_fail(CORR_ERR_INVALID, "sample0 must be >= 0 with sample0 + n <= 2^63 - 1");
    const int64_t nblk = (n + block - 1) / block;
    if (nblk > 0x7FFFFFFF) return blank_fail(CORR_ERR_INVALID, "more than 2^31 - 1 blocks per row");
    if (n == 0) return CORR_OK;
    hipStream_t st = (hipStream_t)stream;
    auto go = [&](auto launch) {
        return launch(d_x, d_out, row_stride, S, n, block, (double)M, d_table, table_len, sample0, d_counts, d_stats, st);
    };
    // 32 G samples a lane and 64 NW lanes: one wave as far as four waves of it fit the
    // registers of a SIMD, above that groups of waves, whose sums meet in LDS.  us in
    // place at 64 x 2^24 samples, blocks of 16384: <8, 1> 444, <4, 2> 272; of 12288: <6, 1>
    // 295, <4, 2> 420; of 20000: <6, 2> 324, <4, 4> 432; out of place of 65536 early 538,
    // late 913.  Out of place of 8192, whose copy fills the registers of <4, 1>: at 64 x 2^22
    // samples <2, 2> 111 and <4, 1> 118, with bursts on 45% of them 200 and 268.
    const bool in_place = d_out == d_x;
    hipError_t e;
    if (block <= 2048) e = in_place ? go(launch_blank<1, 1, kInPlace>) : go(launch_blank<1, 1, kCopyLate>);
    else if (block <= 4096) e = in_place ? go(launch_blank<2, 1, kInPlace>) : go(launch_blank<2, 1, kCopyLate>);
    else if (block <= 8192) e = in_place ? go(launch_blank<4, 1, kInPlace>) : go(launch_blank<2, 2, kCopyLate>);
    else if (block <= 12288 && in_place) e = go(launch_blank<6, 1, kInPlace>);
    else if (block <= 16384) e = in_place ? go(launch_blank<4, 2, kInPlace>) : go(launch_blank<4, 2, kCopyLate>);
    else if (block <= 24576 && in_place) e = go(launch_blank<6, 2, kInPlace>);
    else if (block <= 32768) e = in_place ? go(launch_blank<4, 4, kInPlace>) : go(launch_blank<4, 4, kCopyLate>);
    else e = in_place ? go(launch_blank<4, 8, kInPlace>) : go(launch_blank<4, 8, kCopyEarly>);
    return e == hipSuccess ? CORR_OK : blank_fail(CORR_ERR_DEVICE, "blanker launch: %s", hipGetErrorString(e));
}

const char *corr_blank_last_error(void) { return g_blank_err; }

}  // extern "C"
