// xengine.hip -- X-engine of the FX correlator on gfx950 matrix cores.
//
// For every channel k the visibility matrix is the Hermitian rank-T update
//   V_k = sum_m y_m y_m^H      (y_m = the S signals' spectra at (m, k))
// over all signal pairs, autocorrelations and cross polarisations included
// (section 2.1: RR*, RL*, LR*, LL* of every baseline; the MAC of sections
// 2.3.2 / 3.4).  With y = r + i q:
//   Re V = r r^T + q q^T        Im V = M - M^T,  M = q r^T
// so each channel needs three real products over the spectra: r r^T and q q^T
// on the upper triangle of 32x32 signal tiles and M on all tiles.  They map
// directly onto 32x32 MFMA tiles whose K dimension is the time axis:
//   INT8   v_mfma_i32_32x32x32_i8   (exact int32 sums)
//   FP8    v_mfma_f32_32x32x16_fp8_fp8 (OCP e4m3, FP32 sums)
//   FP32   v_mfma_f32_32x32x16_bf16 on the three BF16 parts of each value
//          (v_mfma_f32_32x32x2_f32 for data that are not finite; below)
// A and B operands are loaded straight from the X layout into registers: lane
// l holds signal 32a + (l mod 32) and the chunks of spectra picked by l / 32;
// since A and B lanes hold the same spectra in the same byte order, the
// product is exact regardless of how the hardware orders K inside a lane.
// X layout: 16-byte chunks indexed [g][k/8][s][k mod 8] (g = chunk of spectra),
// so the chunks of 8 consecutive channels of one signal form one 128-byte
// line.  A workgroup of 8 waves owns 8 consecutive channels and one split of
// the spectra; wave w handles channel 8 kb + w.  The workgroup stages each
// K-step's lines through LDS (below).  Each wave keeps its accumulator tiles in
// registers and at the
// end forms Im = M - M^T through LDS and adds its result into
// acc[split][k][p] (sole owner, so no atomics and a fixed order).
#include <type_traits>

#include "corr_internal.h"

namespace corr {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int ntri(int nt) { return nt * (nt + 1) / 2; }
constexpr int kXcds = 8;  // MI355X: workgroups are dealt to its 8 XCDs in turn

// index of tile pair (a <= b) in the upper triangle
__device__ __forceinline__ constexpr int tri_idx(int a, int b) { return b * (b + 1) / 2 + a; }

// Row of accumulator register r held by lane group lg (32x32 MFMA D layout).
__device__ __forceinline__ int acc_row(int r, int lg) { return 8 * (r >> 2) + 4 * lg + (r & 3); }

// Epilogue shared by all precisions: accR / accM hold sums in ACC type.
template <int NT, typename ACC, typename V16>
__device__ __forceinline__ void x_epilogue(const V16 (&accR)[ntri(NT)], const V16 (&accM)[NT * NT],
                                           ACC *acc_out, int S, int64_t P, ACC (*mlds)[32][33]) {
    const int lane = threadIdx.x & 63, col = lane & 31, lg = lane >> 5;
#pragma unroll
    for (int t = 0; t < NT * NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) mlds[t][acc_row(r, lg)][col] = accM[t][r];
    __syncthreads();
    // A tile's 16 old sums of a lane are all read before any is written back
    // (distinct pairs): a read, add and write per pair waits out the memory
    // latency 16 times over, which a launch of few K-steps cannot hide (two
    // pulsar gates at 64 x 2048 x 8192 int8: 966 -> 918 us with their
    // integration; FP32 at 64 x 512 x 16384, 16 splits: the step 3240 -> 3191 us).
    struct alignas(2 * sizeof(ACC)) Pair {
        ACC re, im;
    };
#pragma unroll
    for (int b = 0; b < NT; ++b)
#pragma unroll
        for (int a = 0; a <= b; ++a) {
            const int J = 32 * b + col;
            Pair *out = reinterpret_cast<Pair *>(acc_out) + (int64_t)J * (J + 1) / 2 + 32 * a;
            Pair sum[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = acc_row(r, lg);
                sum[r] = J < S && 32 * a + i <= J ? out[i] : Pair{};
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = acc_row(r, lg);
                sum[r].re += accR[tri_idx(a, b)][r];
                sum[r].im += mlds[a * NT + b][i][col] - mlds[b * NT + a][col][i];
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = acc_row(r, lg);
                if (J < S && 32 * a + i <= J) out[i] = sum[r];
            }
        }
}

// K-step st covers chunks g0..g0+3, g0 = 4 (split offset + st): lanes 0-31
// take chunks g0 and g0+2, lanes 32-63 chunks g0+1 and g0+3 (the two lane
// groups form the K halves).  INT8/FP8 chunk: 8 real bytes then 8 imaginary
// bytes (8 spectra); FP32 chunk: 2 complex64.
//
// Staging: the workgroup's 8 channels x S signals of one chunk form one
// contiguous block of S x 128 bytes; the 512 threads copy the 4 blocks of the
// next K-step with one 16-byte load each per block (fully coalesced) while the
// MFMAs of the current step run, then store them into LDS with a 144-byte row
// pitch per signal so that the per-channel 16-byte operand reads of a wave
// (stride 144 B across lanes) are free of bank conflicts.  Double-buffered;
// the accumulator exchange of the epilogue reuses the same LDS.
constexpr int kXWaves = 8;                  // channels (waves) per workgroup
constexpr int kRowPitch = 144;              // LDS bytes per signal row (8 x 16 + 16)
constexpr int kBlk = kMaxSignals * kRowPitch;  // LDS bytes per staged chunk block

template <int NT>
constexpr int x_lds_bytes() {
    return (2 * 4 * kBlk > kXWaves * NT * NT * 32 * 33 * 4) ? 2 * 4 * kBlk : kXWaves * NT * NT * 32 * 33 * 4;
}

// 0xFF in every byte of w that equals b (exact zero-byte test of w ^ b).
__device__ inline uint32_t eq_bytes(uint32_t w, uint32_t b4) {
    const uint32_t x = w ^ b4;
    const uint32_t z = ~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu);  // 0x80 in zero bytes
    return (z << 1) - (z >> 7);                                                   // 0x80 -> 0xFF
}

// 4 bits -> 4 bytes of 0x00 / 0xFF
__device__ inline uint32_t keep_bytes(uint32_t b) { return ((b * 0x00204081u) & 0x01010101u) * 0xFFu; }

// Zero the flagged cells of a staged 16-byte chunk: kb8 holds the chunk's keep
// bits (bit i = spectrum i of the chunk kept; 8 spectra for INT8 / FP8, whose
// chunk is 8 real bytes then 8 imaginary bytes, 2 for FP32's two complex64).
template <int PREC>
__device__ __forceinline__ uint4 keep_chunk(uint4 v, uint32_t kb8) {
    if constexpr (PREC == CORR_FP32) {
        if (!(kb8 & 1u)) v.x = v.y = 0u;
        if (!(kb8 & 2u)) v.z = v.w = 0u;
    } else {
        const uint32_t lo = keep_bytes(kb8 & 15u), hi = keep_bytes((kb8 >> 4) & 15u);
        v.x &= lo;
        v.y &= hi;
        v.z &= lo;
        v.w &= hi;
    }
    return v;
}

// One (channel block kb, split sp) of one correlation: PREC is CORR_FP32,
// CORR_INT8 or CORR_FP8_E4M3; ACC float or int32_t; lds holds at least
// x_lds_bytes<NT>() bytes.  GATED: only the spectra m with gate[m] == bin
// are summed (the B operand of every product is masked per spectrum).
// MASKED: the flagged cells (keep bits clear; keep words [C/8][T/32][S][8],
// bit i of word w = spectrum 32 w + i) are zeroed as the chunks are staged,
// which is the product of zeroed spectra without writing them.
// NB = 2 (8-bit codes, GATED): the workgroup takes half of the block's channels,
// 4 (channel half + ...), for two bins: wave w channel w mod 4, bin + w / 4 (left
// out at or past n_bins).  The spectra are staged once for both bins; acc_elems
// elements apart are the bins' accumulators.
template <int NT, int PREC, typename ACC, bool GATED = false, bool MASKED = false, int NB = 1>
__device__ __forceinline__ void xengine_block(const uint8_t *__restrict__ spec, ACC *acc, int S, int C, int T,
                                              int splits, int kb, int sp, uint8_t *lds,
                                              const uint8_t *__restrict__ gate = nullptr, int bin = 0,
                                              const uint32_t *__restrict__ keep = nullptr, int half = 0,
                                              int n_bins = 0, int64_t acc_elems = 0) {
    static_assert(NB == 1 || (NB == 2 && GATED && !MASKED && PREC != CORR_FP32), "bins per workgroup");
    using V16 = typename std::conditional<PREC == CORR_INT8, v16i, v16f>::type;
    constexpr int NCH = kXWaves / NB;                                  // channels of the workgroup
    constexpr int kRowPitch = NB == 1 ? corr::kRowPitch : 80;          // bytes per signal row: NCH x 16 and a pad of 16
    constexpr int kBlk = kMaxSignals * kRowPitch;
    const int wv = threadIdx.x >> 6, ch = wv % NCH, c = kXWaves * kb + half * NCH + ch;
    if constexpr (NB > 1) bin += wv / NCH;
    const int lane = threadIdx.x & 63, row = lane & 31, lg = lane >> 5;
    const int G = (PREC == CORR_FP32) ? kChunk32 : kChunk8;
    const int steps = T / G / 4 / splits;
    const int64_t P = (int64_t)S * (S + 1) / 2;
    if (steps < 1) return;  // no K-step (the plan's splits always leave one): nothing to add

    // staging copy: thread i moves bytes [16 i, 16 i + 16) of each block
    // (NB = 2: unit i mod 256 of the workgroup's 4 channels, threads 0..255 in the
    // blocks 0 and 2 of a K-step, the others in 1 and 3)
    const int i = threadIdx.x, u = NB == 1 ? i : i & 255;
    const bool cp = u < S * NCH;
    const int lds_dst = (u / NCH) * kRowPitch + (u % NCH) * 16 + (NB == 1 ? 0 : (i >> 8) * kBlk);
    // threads beyond the block load its last 16 bytes and discard them, so
    // every thread issues the same loads (the compiler can then count the
    // loads in flight across steps and wait only for the older set)
    const int unit = cp ? u : S * NCH - 1;
    const uint4 *gsrc = reinterpret_cast<const uint4 *>(spec) + (int64_t)kb * S * 8 + (unit / NCH) * 8 + half * NCH +
                        unit % NCH + (NB == 1 ? 0 : (i >> 8) * (int64_t)C * S);
    const int64_t gstride = (int64_t)C * S;  // 16-byte units between chunks g and g+1
    // keep words of this thread's (channel, signal): a K-step's 4 chunks are 32
    // spectra (one word) for INT8 / FP8 and 8 spectra (one byte) for FP32; the
    // words of the block's S x 8 chunks for one span of 32 spectra are
    // contiguous, in the staging threads' order
    const uint32_t *kw0 = nullptr;
    const int64_t kwstride = (int64_t)S * 8;
    if constexpr (MASKED) kw0 = keep + (int64_t)kb * (T / 32) * kwstride + (cp ? i : S * 8 - 1);
    // two register sets (a, b) alternate between the next two K-steps'
    // chunks, so each load has two steps of MFMA work to land before its LDS
    // store
    uint4 pa0 = make_uint4(0, 0, 0, 0), pa1 = pa0, pa2 = pa0, pa3 = pa0, pb0 = pa0, pb1 = pa0, pb2 = pa0, pb3 = pa0;
    uint32_t pak = 0xFFFFFFFFu, pbk = 0xFFFFFFFFu;  // keep bits of the step each set holds (MASKED)
#define X_GLOAD(st, R)                                                \
    {                                                                 \
        const int64_t s_ = (int64_t)sp * steps + (st);                \
        const uint4 *g_ = gsrc + 4 * s_ * gstride;                    \
        R##0 = g_[0];                                                 \
        R##2 = g_[2 * gstride];                                       \
        if constexpr (NB == 1) {                                      \
            R##1 = g_[gstride];                                       \
            R##3 = g_[3 * gstride];                                   \
        }                                                             \
        if constexpr (MASKED) {                                       \
            if constexpr (PREC == CORR_FP32)                          \
                R##k = kw0[(s_ >> 2) * kwstride] >> (8 * (s_ & 3));   \
            else                                                      \
                R##k = kw0[s_ * kwstride];                            \
        }                                                             \
    }
#define X_LSTORE(buf, R)                                              \
    if (cp) {                                                         \
        uint8_t *l_ = lds + (buf) * 4 * kBlk + lds_dst;               \
        constexpr int SH_ = PREC == CORR_FP32 ? 2 : 8;                \
        if constexpr (MASKED) {                                       \
            R##0 = keep_chunk<PREC>(R##0, R##k);                      \
            R##1 = keep_chunk<PREC>(R##1, R##k >> SH_);               \
            R##2 = keep_chunk<PREC>(R##2, R##k >> (2 * SH_));         \
            R##3 = keep_chunk<PREC>(R##3, R##k >> (3 * SH_));         \
        }                                                             \
        *reinterpret_cast<uint4 *>(l_) = R##0;                        \
        *reinterpret_cast<uint4 *>(l_ + 2 * kBlk) = R##2;             \
        if constexpr (NB == 1) {                                      \
            *reinterpret_cast<uint4 *>(l_ + kBlk) = R##1;             \
            *reinterpret_cast<uint4 *>(l_ + 3 * kBlk) = R##3;         \
        }                                                             \
    }

    V16 accR[ntri(NT)], accM[NT * NT];
#pragma unroll
    for (int t = 0; t < ntri(NT); ++t) accR[t] = V16{0};
#pragma unroll
    for (int t = 0; t < NT * NT; ++t) accM[t] = V16{0};
    bool valid[NT];
#pragma unroll
    for (int a = 0; a < NT; ++a) valid[a] = (32 * a + row) < S;

    // gates of a K-step's 4 G spectra (GATED)
    struct GateStep {
        uint32_t w[PREC == CORR_FP32 ? 2 : 8];
    };
    auto gate_step = [&](int st) __attribute__((always_inline)) {
        GateStep g = {};
        if constexpr (GATED) {
            const uint32_t *w = reinterpret_cast<const uint32_t *>(gate) + ((int64_t)sp * steps + st) * G;
#pragma unroll
            for (int q = 0; q < (int)(sizeof(g.w) / 4); ++q) g.w[q] = w[q];
        }
        return g;
    };
    GateStep gates = gate_step(0);

    X_GLOAD(0, pa)
    X_LSTORE(0, pa)
    X_GLOAD(steps > 1 ? 1 : 0, pa)
    __syncthreads();
    // K-step st (B = st is odd): set a (even st) or b (odd st) holds step
    // st + 1's chunks, stored to the other LDS buffer at the end; the other
    // set receives step st + 2's
    auto kstep = [&](int st, auto odd) __attribute__((always_inline)) {
        constexpr bool B = decltype(odd)::value;
        const int buf = st & 1;
        // step st + 2's chunks (the last step's again near the end: unused)
        const int nx = st + 2 < steps ? st + 2 : steps - 1;
        if constexpr (B) {
            X_GLOAD(nx, pa)
        } else {
            X_GLOAD(nx, pb)
        }
        v4i c0[NT], c1[NT];
#pragma unroll
        for (int a = 0; a < NT; ++a) {
            const uint8_t *b = lds + (buf * 4 + lg) * kBlk + (32 * a + row) * kRowPitch + ch * 16;
            c0[a] = valid[a] ? *reinterpret_cast<const v4i *>(b) : v4i{0};
            c1[a] = valid[a] ? *reinterpret_cast<const v4i *>(b + 2 * kBlk) : v4i{0};
        }
        // B operands: masked to the gate's spectra when GATED
        v4i b0[NT], b1[NT];
        if constexpr (GATED) {
            // the K-step's gates, the same in every lane: scalar loads a step ahead and
            // byte masks on the scalar unit (as vector loads their wait, in order
            // behind them, drained the spectra's prefetch at every step); then this lane's
            // chunks are g0 + lg and g0 + 2 + lg
            const uint32_t b4 = (uint32_t)bin * 0x01010101u;
            const GateStep gs = gates;
            gates = gate_step(st + 1 < steps ? st + 1 : st);
            if constexpr (PREC == CORR_FP32) {  // 2 spectra per chunk: one mask word per spectrum
                const uint32_t e0 = eq_bytes(gs.w[0], b4), e1 = eq_bytes(gs.w[1], b4);
                const uint32_t q0 = lg ? e0 >> 16 : e0, q1 = lg ? e1 >> 16 : e1;
                const int m00 = -(int)(q0 & 1u), m01 = -(int)((q0 >> 8) & 1u);
                const int m10 = -(int)(q1 & 1u), m11 = -(int)((q1 >> 8) & 1u);
#pragma unroll
                for (int a = 0; a < NT; ++a) {
                    b0[a] = v4i{c0[a].x & m00, c0[a].y & m00, c0[a].z & m01, c0[a].w & m01};
                    b1[a] = v4i{c1[a].x & m10, c1[a].y & m10, c1[a].z & m11, c1[a].w & m11};
                }
            } else {  // 8 spectra per chunk: real bytes 0-7, imaginary bytes 8-15
                uint32_t e[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) e[q] = eq_bytes(gs.w[q], b4);
                const int m0l = (int)(lg ? e[2] : e[0]), m0h = (int)(lg ? e[3] : e[1]);
                const int m1l = (int)(lg ? e[6] : e[4]), m1h = (int)(lg ? e[7] : e[5]);
#pragma unroll
                for (int a = 0; a < NT; ++a) {
                    b0[a] = v4i{c0[a].x & m0l, c0[a].y & m0h, c0[a].z & m0l, c0[a].w & m0h};
                    b1[a] = v4i{c1[a].x & m1l, c1[a].y & m1h, c1[a].z & m1l, c1[a].w & m1h};
                }
            }
        } else {
#pragma unroll
            for (int a = 0; a < NT; ++a) {
                b0[a] = c0[a];
                b1[a] = c1[a];
            }
        }
        if constexpr (PREC == CORR_INT8) {
            v4i im[NT], re[NT];  // imaginary bytes (A side) / real bytes (B side) of both chunks
#pragma unroll
            for (int a = 0; a < NT; ++a) {
                im[a] = v4i{c0[a].z, c0[a].w, c1[a].z, c1[a].w};
                re[a] = v4i{b0[a].x, b0[a].y, b1[a].x, b1[a].y};
            }
#pragma unroll
            for (int b = 0; b < NT; ++b) {
#pragma unroll
                for (int a = 0; a <= b; ++a) {
                    V16 &d = accR[tri_idx(a, b)];
                    d = __builtin_amdgcn_mfma_i32_32x32x32_i8(c0[a], b0[b], d, 0, 0, 0);
                    d = __builtin_amdgcn_mfma_i32_32x32x32_i8(c1[a], b1[b], d, 0, 0, 0);
                }
#pragma unroll
                for (int a = 0; a < NT; ++a)
                    accM[a * NT + b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(im[a], re[b], accM[a * NT + b], 0, 0, 0);
            }
        } else if constexpr (PREC == CORR_FP8_E4M3) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                long re[NT], im[NT], reB[NT], imB[NT];  // A side, and the (masked) B side
#pragma unroll
                for (int a = 0; a < NT; ++a) {
                    const v4i v = h ? c1[a] : c0[a];
                    const v4i w = h ? b1[a] : b0[a];
                    re[a] = (long)(((unsigned long)(unsigned)v.y << 32) | (unsigned)v.x);
                    im[a] = (long)(((unsigned long)(unsigned)v.w << 32) | (unsigned)v.z);
                    reB[a] = (long)(((unsigned long)(unsigned)w.y << 32) | (unsigned)w.x);
                    imB[a] = (long)(((unsigned long)(unsigned)w.w << 32) | (unsigned)w.z);
                }
#pragma unroll
                for (int b = 0; b < NT; ++b) {
#pragma unroll
                    for (int a = 0; a <= b; ++a) {
                        V16 &d = accR[tri_idx(a, b)];
                        d = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(re[a], reB[b], d, 0, 0, 0);
                        d = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(im[a], imB[b], d, 0, 0, 0);
                    }
#pragma unroll
                    for (int a = 0; a < NT; ++a)
                        accM[a * NT + b] = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(im[a], reB[b], accM[a * NT + b], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {  // spectra (chunk 0: 0, 1; chunk 1: 2, 3)
                float rr[NT], qq[NT], rrB[NT], qqB[NT];  // A side, and the (masked) B side
#pragma unroll
                for (int a = 0; a < NT; ++a) {
                    const v4i v = (q < 2) ? c0[a] : c1[a];
                    const v4i w = (q < 2) ? b0[a] : b1[a];
                    rr[a] = __int_as_float((q & 1) ? v.z : v.x);
                    qq[a] = __int_as_float((q & 1) ? v.w : v.y);
                    rrB[a] = __int_as_float((q & 1) ? w.z : w.x);
                    qqB[a] = __int_as_float((q & 1) ? w.w : w.y);
                }
#pragma unroll
                for (int b = 0; b < NT; ++b) {
#pragma unroll
                    for (int a = 0; a <= b; ++a) {
                        V16 &d = accR[tri_idx(a, b)];
                        d = __builtin_amdgcn_mfma_f32_32x32x2f32(rr[a], rrB[b], d, 0, 0, 0);
                        d = __builtin_amdgcn_mfma_f32_32x32x2f32(qq[a], qqB[b], d, 0, 0, 0);
                    }
#pragma unroll
                    for (int a = 0; a < NT; ++a)
                        accM[a * NT + b] = __builtin_amdgcn_mfma_f32_32x32x2f32(qq[a], rrB[b], accM[a * NT + b], 0, 0, 0);
                }
            }
        }
        if (st + 1 < steps) {
            if constexpr (B) {
                X_LSTORE(buf ^ 1, pb)
            } else {
                X_LSTORE(buf ^ 1, pa)
            }
        }
        __syncthreads();
    };
    int st = 0;
    for (; st + 1 < steps; st += 2) {  // whole pairs, so every loop entry sees the same loads in flight
        kstep(st, std::false_type{});
        kstep(st + 1, std::true_type{});
    }
    if (st < steps) kstep(st, std::false_type{});
#undef X_GLOAD
#undef X_LSTORE
    // the staging buffers are free now: the epilogue's M-tile exchange reuses them
    auto *mlds = reinterpret_cast<ACC(*)[32][33]>(lds + wv * NT * NT * 32 * 33 * 4);
    if constexpr (NB > 1) acc += bin * acc_elems;
    x_epilogue<NT, ACC>(accR, accM, acc + ((int64_t)sp * C + c) * P * 2, NB == 1 || bin < n_bins ? S : 0, P, mlds);
    __syncthreads();  // the LDS may be reused by the next block of a persistent loop
}

// ------------------------------------------------ FP32 on the BF16 matrix cores
//
// The FP32 X-engine was bound by the FP32 matrix cores (0.16 PFLOP/s, 1/16 of
// the BF16 rate).  An FP32 number is the exact sum of three BF16 numbers (each
// the nearest BF16 of what the ones before leave: 8 significant bits apiece, 24
// in all), so a product of two is nine BF16 products, each exact in FP32.  The
// three smallest, below 2^-25 of the whole, are left out; the other six go through
// v_mfma_f32_32x32x16_bf16, which takes 16 spectra where the FP32 instruction
// takes 2: 6/16 of the matrix time.  The sums are rounded a sixteenth as often,
// so they are more exact: 2.3e-7 of the visibilities at 64 x 512 x 16384 before
// (against 64 bits, the F-engine's part included), 0.8e-7 now.  The kernel took
// 1.70 ms there, now 1.06 ms (4.1 TB/s; its loads alone 0.83 ms, its arithmetic
// alone 0.88 ms at the 1.7 GHz this load leaves the clock).
//
// Values of 2^-110 and more in magnitude (and zeros) split exactly: the matrix
// cores take subnormal BF16 numbers, down to 2^-133, and keep subnormal products
// (amplitudes of 2^-62 to 2^58 have the same errors).  A value that is infinite or
// NaN, or within half a BF16 step of the largest FP32 number, leaves a NaN in every
// sum it takes part in; a block with a sum that is not finite is done on the FP32
// instructions instead, all its 8 channels (so a bad cell moves the last bits of the
// other seven): the bad pairs come out as those instructions give them.  A dead
// antenna, NaN throughout, shows before the first
// step and costs what it cost when every block ran on the FP32 instructions (64 x
// 512 x 16384: 1450 us, 1480 then; two gates 2910 and 3540; with flags that leave it in
// and 33 to 48 signals 15% more).  Found only at the end of a block it had cost 3600 us,
// also because that left the registers of the products and of the fallback's loads to
// share: 49 to 62 a lane went through scratch memory.  A bad cell elsewhere costs its
// own block what both passes take, at most.
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t bf16_pair(float x, float y) {  // nearest BF16 of x (low half) and y
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){x, y}, v2bf));
}

// p[i] = the i-th BF16 parts of x (low half) and y (high half)
__device__ __forceinline__ void split_pair(float x, float y, uint32_t (&p)[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        p[i] = bf16_pair(x, y);
        if (i < 2) {
            x -= __uint_as_float(p[i] << 16);
            y -= __uint_as_float(p[i] & 0xFFFF0000u);
        }
    }
}

constexpr int kSplitChunks = 8;  // chunks of 2 spectra per K-step

// A value that is the same in every lane, into scalar registers (the result of a
// division comes in a vector register).
template <typename T>
__device__ __forceinline__ T uniform(T v) {
    union {
        T v;
        int w[sizeof(T) / 4];
    } u;
    u.v = v;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) u.w[i] = __builtin_amdgcn_readfirstlane(u.w[i]);
    return u.v;
}

// The block of xengine_block, for FP32 spectra.  A K-step is 16 spectra: lanes
// 0-31 take its first four chunks of their signal, lanes 32-63 the other four
// (8 spectra each, the K slots of a lane).  The chunks go from global memory
// straight into LDS (the sums, the six parts of both operands and a tile in
// progress leave no registers to hold them), double-buffered, 64 KB per
// compute unit in flight during a step.  Rows of 128 bytes, and the chunk of
// channel k of signal s in place k xor (s mod 8) of its row: the lanes of a
// DMA load choose which channel they fetch, and 8 rows of an operand read
// cover the banks once.  A wave splits the operands of its channel after
// reading them, once for all products, since the same registers serve as A and
// B.  Flagged cells are zeroed before the split.
template <int NT, bool GATED, bool MASKED>
__device__ __forceinline__ void xengine_block_split(const uint8_t *__restrict__ spec, float *out, int S, int C, int T,
                                                    int splits, int kb, int sp, uint8_t *lds,
                                                    const uint8_t *__restrict__ gate, int bin,
                                                    const uint32_t *__restrict__ keep) {
    constexpr int blk = 32 * NT * 128;  // LDS bytes of a staged chunk block
    static_assert(2 * kSplitChunks * blk <= x_lds_bytes<NT>(), "both buffers fit");
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = kXWaves * kb + wv;
    const int lane = threadIdx.x & 63, row = lane & 31, lg = lane >> 5;
    const int steps = uniform(T / (2 * kSplitChunks) / splits);
    const int64_t P = (int64_t)S * (S + 1) / 2;
    if (steps < 1) return;

    // staging: thread i fills the 16 bytes i of each chunk block
    const int i = threadIdx.x, si = i >> 3;
    const bool cp = si < S;
    const uint32_t src = si * 128 + 16 * ((i & 7) ^ (si & 7));
    const int64_t gstride = (int64_t)C * S * 16;  // bytes between chunks
    const uint8_t *gbase = spec + (int64_t)kb * S * 128 + (int64_t)sp * steps * kSplitChunks * gstride;
    auto stage = [&](int st, int buf) __attribute__((always_inline)) {
        const uint8_t *g = gbase + (int64_t)st * kSplitChunks * gstride + src;
        uint8_t *l = lds + buf * kSplitChunks * blk + wv * 1024;
        if (cp) {
#pragma unroll
            for (int j = 0; j < kSplitChunks; ++j)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(g + j * gstride),
                                                 (__attribute__((address_space(3))) void *)(l + j * blk), 16, 0, 0);
        }
    };
    // keep bits of this lane's 8 spectra of a step, per row tile (shifted at once,
    // which waits for the chunks in flight: 1260 us at 64 x 512 x 16384, 1295 with the
    // shift a phase later)
    uint32_t kb8[NT];
    const uint32_t *kw = nullptr;
    uint32_t koff[NT];
    if constexpr (MASKED) {
        kw = keep + (int64_t)kb * (T / 32) * S * 8;
#pragma unroll
        for (int a = 0; a < NT; ++a) koff[a] = min(32 * a + row, S - 1) * 8 + wv;
    }
    auto load_keep = [&](int st) __attribute__((always_inline)) {
        if constexpr (MASKED) {
            const int64_t s_ = (int64_t)sp * steps + st;
#pragma unroll
            for (int a = 0; a < NT; ++a) kb8[a] = (kw + (s_ >> 1) * S * 8)[koff[a]] >> (16 * (s_ & 1) + 8 * lg);
        }
    };

    constexpr int NTILE = ntri(NT) + NT * NT;  // the R tiles (upper triangle), then the M tiles
    v16f acc[NTILE];
#pragma unroll
    for (int t = 0; t < NTILE; ++t) acc[t] = v16f{0};

    // rows past S stay zero, so that every operand read is unconditional
    for (int e = i; e < 2 * kSplitChunks * (32 * NT - S) * 8; e += 64 * kXWaves) {
        const int ch = e / ((32 * NT - S) * 8), r = e % ((32 * NT - S) * 8);
        *reinterpret_cast<uint4 *>(lds + ch * blk + S * 128 + r * 16) = make_uint4(0, 0, 0, 0);
    }
    v4u re[NT][3], im[NT][3];  // operand parts; word j: spectra 2 j, 2 j + 1 of this lane's eight
    v4u m;                     // the gate's spectra (B operands)
    uint32_t k8[NT];
    // operand parts of row tile a in step st; k: its keep bits
    auto split = [&](int a, int st, uint32_t k) __attribute__((always_inline)) {
        const uint8_t *lb = lds + ((st & 1) * kSplitChunks + 4 * lg) * blk + row * 128 + 16 * (wv ^ (row & 7));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v4u x = *reinterpret_cast<const v4u *>(lb + j * blk + 32 * a * 128);
            if constexpr (MASKED) {
                const uint32_t m0 = 0u - ((k >> (2 * j)) & 1u), m1 = 0u - ((k >> (2 * j + 1)) & 1u);
                x &= v4u{m0, m0, m1, m1};
            }
            uint32_t p[3], q[3];
            split_pair(__uint_as_float(x[0]), __uint_as_float(x[2]), p);
            split_pair(__uint_as_float(x[1]), __uint_as_float(x[3]), q);
#pragma unroll
            for (int h = 0; h < 3; ++h) {
                re[a][h][j] = p[h];
                im[a][h][j] = q[h];
            }
        }
    };
    // the gates of a step are the same in every lane: scalar loads (a vector load's
    // wait would drain the chunks in flight)
    auto load_gate = [&](int st) __attribute__((always_inline)) {
        if constexpr (GATED) {
            const uint32_t *w = reinterpret_cast<const uint32_t *>(gate) + 4 * ((int64_t)sp * steps + st);
            const uint32_t b4 = (uint32_t)bin * 0x01010101u;
            const uint32_t e0 = eq_bytes(w[0], b4), e1 = eq_bytes(w[1], b4), e2 = eq_bytes(w[2], b4),
                           e3 = eq_bytes(w[3], b4);
            const uint32_t lo = lg ? e2 : e0, hi = lg ? e3 : e1;
            m = v4u{__builtin_amdgcn_perm(0u, lo, 0x01010000u), __builtin_amdgcn_perm(0u, lo, 0x03030202u),
                    __builtin_amdgcn_perm(0u, hi, 0x01010000u), __builtin_amdgcn_perm(0u, hi, 0x03030202u)};
        }
    };
    auto mac = [&](const v4u &x, const v4u &y, v16f &d) __attribute__((always_inline)) {
        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, x),
                                                    __builtin_bit_cast(v8bf, GATED ? (v4u)(y & m) : y), d, 0, 0, 0);
    };
    // Tiles of the step: the products of each, the smaller ones first, go into a
    // sum of their own, which then joins the running one (an addition into the
    // large running sum rounds at its size, and the matrix cores round it less
    // exactly than the vector ALUs: with one chain into it the error was 3.5
    // times larger).  The tiles' chains alternate.
    constexpr int NR = ntri(NT);
    auto product = [&](auto tag, int h, bool second, v16f &d) __attribute__((always_inline)) {
        constexpr int t = decltype(tag)::value;
        constexpr int pi[6] = {0, 1, 2, 0, 1, 0}, pj[6] = {2, 1, 0, 1, 0, 0};
        if constexpr (t < NR) {
            constexpr int b = t == 0 ? 0 : 1, a = t == 2 ? 1 : 0;
            if (second) mac(im[a][pi[h]], im[b][pj[h]], d);
            else mac(re[a][pi[h]], re[b][pj[h]], d);
        } else if (!second) {
            constexpr int a = (t - NR) / NT, b = (t - NR) % NT;
            mac(im[a][pi[h]], re[b][pj[h]], d);
        }
    };
    auto tiles = [&](auto... tags) __attribute__((always_inline)) {
        v16f d[sizeof...(tags)];
#pragma unroll
        for (int q = 0; q < (int)sizeof...(tags); ++q) d[q] = v16f{0};
#pragma unroll
        for (int h = 0; h < 6; ++h) {
            int q = 0;
            (product(tags, h, false, d[q++]), ...);
            q = 0;
            (product(tags, h, true, d[q++]), ...);
        }
        int q = 0;
        ((acc[decltype(tags)::value] += d[q++]), ...);
    };
    // interleave n products with v vector instructions after each
#define X_MIX(n, v)                                        \
    _Pragma("unroll") for (int q_ = 0; q_ < (n); ++q_) {   \
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); \
        __builtin_amdgcn_sched_group_barrier(0x002, v, 0); \
    }
    auto arrived = [&]() __attribute__((always_inline)) {  // this wave's loads are in LDS, then every wave's
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };
    // Data that are not finite are done on the FP32 instructions (below); most such data,
    // an antenna that is NaN throughout, show in the first chunk, which each thread
    // looks at where it has put it, before a step is lost on them.
    __shared__ __attribute__((aligned(16))) uint32_t spoilt[2][kXWaves], in_gate[GATED ? kXWaves : 1];
    auto not_finite = [](float x) __attribute__((always_inline)) { return __builtin_amdgcn_classf(x, 0x207); };
    stage(0, 0);
    load_keep(0);
    load_gate(0);
    if constexpr (GATED) {
        // The split's spectra of this gate.  A sum of four and fewer is more exact on the
        // FP32 instructions, with two roundings a spectrum (one spectrum: 3.3e-8 rms of the
        // pair's power and 1.2e-7 at most, here 3.8e-8 and 2.1e-7; four 3.2e-8 and 3.3e-8;
        // 16 4.8e-8 and 3.3e-8).  Counting costs calls of four K-steps 4%, longer ones nothing.
        const uint32_t *w = reinterpret_cast<const uint32_t *>(gate) + 4 * (int64_t)sp * steps;
        uint32_t n = 0;
        for (int e = i; e < 4 * steps; e += 64 * kXWaves)
            n += (uint32_t)__builtin_popcount(eq_bytes(w[e], (uint32_t)bin * 0x01010101u)) / 8;
        n = min(n, 7u);  // a wave's sum of these is enough
        in_gate[wv] = __popcll(__ballot(n & 1)) + 2 * __popcll(__ballot(n & 2)) + 4 * __popcll(__ballot(n & 4));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    bool bad = false;
    if (cp) {
        v4u x = *reinterpret_cast<const v4u *>(lds + i * 16);
        if constexpr (MASKED) {
            const int64_t s_ = (int64_t)sp * steps;
            const uint32_t k = (kw + (s_ >> 1) * S * 8)[si * 8 + ((i & 7) ^ (si & 7))] >> (16 * (s_ & 1));
            const uint32_t m0 = 0u - (k & 1u), m1 = 0u - (k >> 1 & 1u);
            x &= v4u{m0, m0, m1, m1};
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) bad |= not_finite(__uint_as_float(x[q]));
    }
    spoilt[0][wv] = __any(bad);
    __syncthreads();
    auto told = [&](int turn) __attribute__((always_inline)) {  // by any wave
        const v4u *w = reinterpret_cast<const v4u *>(spoilt[turn]), c = w[0] | w[1];
        return __builtin_amdgcn_readfirstlane(c[0] | c[1] | c[2] | c[3]) != 0;
    };
    bool redo = told(0);
    if constexpr (GATED) {
        uint32_t n = 0;
#pragma unroll
        for (int q = 0; q < kXWaves; ++q) n += in_gate[q];
        n = __builtin_amdgcn_readfirstlane(n);
        redo |= n >= 1 && n <= 4;
    }
    if constexpr (NT == 2) {
        // The parts of row tile 0 are made a phase ahead of their use, and those of
        // tile 1 during the products of tile 0, so that vector and matrix
        // instructions share a wave's time (they took turns before, 33% and 43% of
        // it).  A buffer is filled again as soon as every wave has read tile 1 from
        // it, with the next step's loads still in flight: these alone are waited
        // for, by count.  Past the end the last step is loaded again, unused.
        using std::integral_constant;
        auto clamped = [&](int st) { return st < steps ? st : steps - 1; };
        k8[0] = MASKED ? kb8[0] : 0u;
        k8[1] = MASKED ? kb8[1] : 0u;
        stage(clamped(1), 1);
        load_keep(clamped(1));
        split(0, 0, k8[0]);
        // What is not finite later shows in the sums: after every kSpan steps each wave
        // looks at one register of the tiles on the diagonal (a bad signal spoils its
        // whole column there) and tells the others, who read it a span later and all
        // leave.  (Two sets of words in turn: none is written where a wave may still read.)
        constexpr int kSpan = 16;
        for (int st = 0, end, turn = 0; st < steps && !redo; turn ^= 1) {
            end = min(steps, st + kSpan);
#pragma unroll 1
            for (; st < end; ++st) {
                __builtin_amdgcn_sched_barrier(0);
                split(1, st, k8[1]);
                tiles(integral_constant<int, 0>{}, integral_constant<int, 3>{});
                X_MIX(18, 6)
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (MASKED) {
                    k8[0] = kb8[0];
                    k8[1] = kb8[1];
                }
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                stage(clamped(st + 2), st & 1);
                load_keep(clamped(st + 2));
                __builtin_amdgcn_sched_barrier(0);
                tiles(integral_constant<int, 4>{}, integral_constant<int, 1>{}, integral_constant<int, 5>{});
                X_MIX(24, 2)
                __builtin_amdgcn_sched_barrier(0);
                // step st + 1's chunks: all but the loads issued since (8, and the keep words;
                // a wave without a signal of its own waits for nothing)
                if constexpr (MASKED) asm volatile("s_waitcnt vmcnt(10)\n\ts_barrier" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                split(0, st + 1, k8[0]);
                tiles(integral_constant<int, 2>{}, integral_constant<int, 6>{});
                X_MIX(18, 6)
                __builtin_amdgcn_sched_barrier(0);
                load_gate(clamped(st + 1));
            }
            redo = told(turn);
            spoilt[turn ^ 1][wv] = __any(not_finite(acc[0][0]) || not_finite(acc[2][0]));
        }
        arrived();
    } else {
#pragma unroll 1
        for (int st = 0; st < steps && !redo; ++st) {
            k8[0] = MASKED ? kb8[0] : 0u;
            if (st + 1 < steps) {  // into the buffer that was last read a step ago
                stage(st + 1, (st + 1) & 1);
                load_keep(st + 1);
            }
            split(0, st, k8[0]);
            tiles(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
            load_gate(st + 1 < steps ? st + 1 : st);
            arrived();
        }
    }
#undef X_MIX
    float z = 0.f;  // NaN if a sum is not finite
#pragma unroll
    for (int t = 0; t < NTILE; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) z = fmaf(acc[t][r], 0.f, z);
    if (redo || __syncthreads_or(z != z)) {
        xengine_block<NT, CORR_FP32, float, GATED, MASKED>(spec, out, S, C, T, splits, kb, sp, lds, gate, bin, keep);
        return;
    }
    v16f accR[ntri(NT)], accM[NT * NT];
#pragma unroll
    for (int t = 0; t < ntri(NT); ++t) accR[t] = acc[t];
#pragma unroll
    for (int t = 0; t < NT * NT; ++t) accM[t] = acc[ntri(NT) + t];
    auto *mlds = reinterpret_cast<float(*)[32][33]>(lds + wv * NT * NT * 32 * 33 * 4);
    x_epilogue<NT, float>(accR, accM, out + ((int64_t)sp * C + c) * P * 2, S, P, mlds);
    __syncthreads();
}

template <int NT, int PREC, typename ACC, bool MASKED>
__global__ void __launch_bounds__(64 * kXWaves)
xengine_kernel(const uint8_t *__restrict__ spec, const uint32_t *__restrict__ keep, ACC *acc, int S, int C, int T,
               int splits) {
    if constexpr (PREC == CORR_FP32) {
        __shared__ __attribute__((aligned(16))) uint8_t lds[x_lds_bytes<NT>()];
        xengine_block_split<NT, false, MASKED>(spec, acc, S, C, T, splits, blockIdx.x, blockIdx.y, lds, nullptr, 0,
                                               keep);
    } else {
        __shared__ __attribute__((aligned(16))) uint8_t lds[x_lds_bytes<NT>()];
        xengine_block<NT, PREC, ACC, false, MASKED>(spec, acc, S, C, T, splits, blockIdx.x, blockIdx.y, lds, nullptr,
                                                   0, keep);
    }
}

// Gated correlation: task = (channel block kb, split sp); it sums the spectra of
// gate bin `bin` into accumulator set `bin` (acc_elems elements apart).  A task
// has `per` workgroups: one per bin (NB = 1), or, for 8-bit codes, one per channel
// half and pair of bins (NB = 2), so that the spectra are staged once for two
// bins instead of once for each: two bins at 64 x 2048 x 8192 int8 take 545 us,
// 660 us with NB = 1 (and 860 us before the gates came by scalar loads; the
// spectra's 2.1 GB take 365 us at the card's read rate).  The workgroups of a task read the
// same lines, so they are given ids 8 apart: workgroups go to the 8 XCDs in turn,
// so those land on the same XCD, run side by side and share its L2 (the later
// reads hit).  w -> xcd = w mod 8, j = w / 8, part = j mod per,
// task = 8 (j / per) + xcd.
template <int NT, int PREC, typename ACC, int NB>
__global__ void __launch_bounds__(64 * kXWaves)
xengine_gated_kernel(const uint8_t *__restrict__ spec, const uint8_t *__restrict__ gate, ACC *acc, int64_t acc_elems,
                     int S, int C, int T, int splits, int n_bins) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[x_lds_bytes<NT>()];
    const int per = NB * ((n_bins + NB - 1) / NB);
    const int w = blockIdx.x, xcd = w & (kXcds - 1), j = w / kXcds;
    const int part = j % per, task = kXcds * (j / per) + xcd;
    const int nkb = C / kXWaves;
    if (task >= nkb * splits) return;  // padding of the last group of 8 tasks
    if constexpr (PREC == CORR_FP32)
        xengine_block_split<NT, true, false>(spec, acc + uniform(part) * acc_elems, S, C, T, splits, uniform(task % nkb),
                                             uniform(task / nkb), lds, gate, uniform(part), nullptr);
    else if constexpr (NB == 1)
        xengine_block<NT, PREC, ACC, true>(spec, acc + part * acc_elems, S, C, T, splits, task % nkb, task / nkb, lds,
                                           gate, part);
    else
        xengine_block<NT, PREC, ACC, true, false, 2>(spec, acc, S, C, T, splits, task % nkb, task / nkb, lds, gate,
                                                     part / 2 * 2, nullptr, part % 2, n_bins, acc_elems);
}

// One launch over the tasks of a batch of correlations of different shapes
// (one per sub-array).  The batch table travels by value as the kernel
// argument, so every field is a uniform scalar; workgroup b runs task b: the
// correlation whose task range holds b, then its (channel block, split).  Each
// task runs the body of its sub-array's size, as corr_xengine would: two
// 32-signal tiles above 32 signals, one tile otherwise (the two-tile body on
// a small sub-array issues 7 matrix products per step where 3 suffice).  The
// branch is uniform per workgroup.
__global__ void __launch_bounds__(64 * kXWaves) xengine_batch_kernel(XBatchArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[x_lds_bytes<2>()];
    const int b = blockIdx.x;
    int i = 0;
    while (i + 1 < a.n && b >= a.first[i + 1]) ++i;
    const XBatchEntry &e = a.cor[i];
    const int local = b - a.first[i];
    const int nkb = e.C / kXWaves;
    if (e.S > 32)
        xengine_block<2, CORR_INT8, int32_t>((const uint8_t *)e.spec, (int32_t *)e.acc, e.S, e.C, e.T, e.splits,
                                             local % nkb, local / nkb, lds);
    else
        xengine_block<1, CORR_INT8, int32_t>((const uint8_t *)e.spec, (int32_t *)e.acc, e.S, e.C, e.T, e.splits,
                                             local % nkb, local / nkb, lds);
}

// --------------------------------------------------------------- xpack ----
// Corner turn [S][T][C][2] -> X layout, bound by HBM (every byte read and
// written once).  The channel count is a power of two and signals are a grid
// index, so no thread divides.
//
// 8-bit codes: a thread takes 8 channels of 8 spectra of one signal -- eight
// 16-byte loads, consecutive lanes consecutive channels -- transposes them in
// registers and writes the 8 chunks, one whole 128-byte line; the waves of a
// workgroup take 4 adjacent signals, whose lines are adjacent.  With a thread per
// chunk that loaded and stored single bytes (the lanes across signals, T C
// apart) 30 x 1024 x 4096 took 804 us, now 123 us (0.5 GB,
// 4.1 TB/s).
//
// Bytes 0..3 of four words, gathered by place: out[j] = byte j of w[0..3].
__device__ __forceinline__ void transpose4(const uint32_t (&w)[4], uint32_t (&out)[4]) {
    const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), b = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
    const uint32_t c = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u), d = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    out[0] = __builtin_amdgcn_perm(c, a, 0x05040100u);
    out[1] = __builtin_amdgcn_perm(c, a, 0x07060302u);
    out[2] = __builtin_amdgcn_perm(d, b, 0x05040100u);
    out[3] = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

__global__ void __launch_bounds__(256) xpack8_kernel(const uint8_t *__restrict__ in, uint4 *__restrict__ out, int S,
                                                     int64_t T, int lgC) {
    const int64_t idx = (int64_t)blockIdx.x * 64 + threadIdx.x;  // over [T/8][C/8]
    const int s = blockIdx.y * 4 + threadIdx.y;
    if (s >= S) return;
    const int64_t g = idx >> (lgC - 3), kb = idx & ((1 << (lgC - 3)) - 1);
    const uint4 *src = reinterpret_cast<const uint4 *>(in + ((((int64_t)s * T + 8 * g) << lgC) + 8 * kb) * 2);
    uint4 v[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) v[m] = src[(int64_t)m << (lgC - 3)];
    uint4 *dst = out + (((g << (lgC - 3)) + kb) * S + s) * 8;
#pragma unroll
    for (int d = 0; d < 4; ++d) {  // word d of a row: re, im of channel 2 d, re, im of channel 2 d + 1
        uint32_t lo[4], hi[4], tl[4], th[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            lo[m] = d == 0 ? v[m].x : d == 1 ? v[m].y : d == 2 ? v[m].z : v[m].w;
            hi[m] = d == 0 ? v[m + 4].x : d == 1 ? v[m + 4].y : d == 2 ? v[m + 4].z : v[m + 4].w;
        }
        transpose4(lo, tl);
        transpose4(hi, th);
        dst[2 * d] = make_uint4(tl[0], th[0], tl[1], th[1]);
        dst[2 * d + 1] = make_uint4(tl[2], th[2], tl[3], th[3]);
    }
}

// FP32: a thread takes one channel of 2 spectra, one chunk; 8 lanes fill a line.
__global__ void __launch_bounds__(256) xpack32_kernel(const float2 *__restrict__ in, float4 *__restrict__ out, int S,
                                                      int64_t T, int lgC) {
    const int64_t idx = (int64_t)blockIdx.x * 64 + threadIdx.x;  // over [T/2][C]
    const int s = blockIdx.y * 4 + threadIdx.y;
    if (s >= S) return;
    const int64_t g = idx >> lgC, k = idx & ((1 << lgC) - 1);
    const float2 *src = in + (((int64_t)s * T + 2 * g) << lgC) + k;
    const float2 a = src[0], b = src[(int64_t)1 << lgC];
    out[((((g << lgC) + k) >> 3) * S + s) * 8 + (k & 7)] = make_float4(a.x, a.y, b.x, b.y);
}

// Requantisation of FP32 spectra [S][T][C][2] to codes [S][T][C][2] with
// the F-engines' encoders: q = enc(v * (1 / scale[s][k])) per component.  Bound
// by HBM (8 bytes in, 2 out a cell).  A thread takes V adjacent channels of 8
// spectra (all loads first, the reciprocals once for the 8 rows); V = 4 where the
// buffers are 16-byte (codes 8-byte) aligned, else 1.  One complex value per
// thread with its own division and 64-bit index division took 358 us at
// 30 x 1024 x 4096, now 244 us (1.26 GB, 5.2 TB/s).
template <int PREC, int V>
__global__ void __launch_bounds__(256) requantize_kernel(const float2 *__restrict__ in, const float *__restrict__ scale,
                                                         int64_t T, int lgC, uint16_t *__restrict__ out) {
    constexpr int R = 8, LGV = V == 4 ? 2 : 0;
    static_assert(V == 1 || V == 4, "channels per thread");
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;  // over [T/R][C/V]
    const int s = blockIdx.y;
    const int64_t g = idx >> (lgC - LGV), k = (idx & ((1 << (lgC - LGV)) - 1)) * V;
    const int64_t o = (((int64_t)s * T + R * g) << lgC) + k;
    struct alignas(8 * V) In {
        float2 c[V];
    };
    struct alignas(2 * V) Out {
        uint16_t c[V];
    };
    In v[R];
#pragma unroll
    for (int m = 0; m < R; ++m) v[m] = *reinterpret_cast<const In *>(in + o + ((int64_t)m << lgC));
    float inv[V];
#pragma unroll
    for (int j = 0; j < V; ++j) inv[j] = 1.0f / scale[((int64_t)s << lgC) + k + j];
#pragma unroll
    for (int m = 0; m < R; ++m) {
        Out q;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const float x = v[m].c[j].x * inv[j], y = v[m].c[j].y * inv[j];
            if constexpr (PREC == CORR_INT8)
                q.c[j] = (uint16_t)((quant_i8(x) & 0xFFu) | ((quant_i8(y) & 0xFFu) << 8));
            else
                q.c[j] = (uint16_t)(e4m3_pair(x, y) & 0xFFFFu);
        }
        *reinterpret_cast<Out *>(out + o + ((int64_t)m << lgC)) = q;
    }
}

int log2_of(int v) {
    int r = 0;
    while ((1 << r) < v) ++r;
    return r;
}

}  // namespace

hipError_t launch_requantize(int precision, const float *in, const float *scale, int S, int64_t T, int C,
                             uint8_t *out, hipStream_t st) {
    const bool wide = !(reinterpret_cast<uintptr_t>(in) & 31) && !(reinterpret_cast<uintptr_t>(out) & 7);
    const float2 *src = reinterpret_cast<const float2 *>(in);
    uint16_t *dst = reinterpret_cast<uint16_t *>(out);
    auto go = [&](auto kernel, int V) {  // T is a multiple of 32, C a power of two >= 256: whole workgroups
        hipLaunchKernelGGL(kernel, dim3((unsigned)(T / 8 * (C / V) / 256), S), dim3(256), 0, st, src, scale, T,
                           log2_of(C), dst);
        return hipGetLastError();
    };
    if (precision == CORR_INT8)
        return wide ? go(requantize_kernel<CORR_INT8, 4>, 4) : go(requantize_kernel<CORR_INT8, 1>, 1);
    if (precision == CORR_FP8_E4M3)
        return wide ? go(requantize_kernel<CORR_FP8_E4M3, 4>, 4) : go(requantize_kernel<CORR_FP8_E4M3, 1>, 1);
    return hipErrorInvalidValue;
}

hipError_t launch_xengine(int precision, const void *spec, const uint32_t *keep, void *acc, int S, int C, int T,
                          int splits, hipStream_t st) {
    const dim3 grid(C / kXWaves, splits), block(64 * kXWaves);
    const uint8_t *sp8 = (const uint8_t *)spec;
    auto go = [&](auto kernel, auto *a) { hipLaunchKernelGGL(kernel, grid, block, 0, st, sp8, keep, a, S, C, T, splits); };
    const bool two = S > 32, m = keep != nullptr;
    int32_t *ai = (int32_t *)acc;
    float *af = (float *)acc;
    switch (precision) {
    case CORR_INT8:
        if (two) m ? go(xengine_kernel<2, CORR_INT8, int32_t, true>, ai) : go(xengine_kernel<2, CORR_INT8, int32_t, false>, ai);
        else m ? go(xengine_kernel<1, CORR_INT8, int32_t, true>, ai) : go(xengine_kernel<1, CORR_INT8, int32_t, false>, ai);
        break;
    case CORR_FP8_E4M3:
        if (two) m ? go(xengine_kernel<2, CORR_FP8_E4M3, float, true>, af) : go(xengine_kernel<2, CORR_FP8_E4M3, float, false>, af);
        else m ? go(xengine_kernel<1, CORR_FP8_E4M3, float, true>, af) : go(xengine_kernel<1, CORR_FP8_E4M3, float, false>, af);
        break;
    case CORR_FP32:
        if (two) m ? go(xengine_kernel<2, CORR_FP32, float, true>, af) : go(xengine_kernel<2, CORR_FP32, float, false>, af);
        else m ? go(xengine_kernel<1, CORR_FP32, float, true>, af) : go(xengine_kernel<1, CORR_FP32, float, false>, af);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_xengine_gated(int precision, const void *spec, const uint8_t *gate, int n_bins, void *acc,
                                int64_t acc_elems, int S, int C, int T, int splits, hipStream_t st) {
    const int tasks = (C / kXWaves) * splits;
    // Pairs of bins where the staging they share is what bounds a launch: from two K-steps
    // a split on (four signals, eight bins of 512 channels x 64 spectra: 28.6 us in pairs, 26.4
    // single; of 2048 x 512, eight steps: 62 and 71).  The empty half of an odd number's last
    // pair costs a workgroup: five bins of 4 x 2048 x 64 22.4 and 17.8 us, of 64 x 8192 x 256
    // 571 and 564, three of 64 x 2048 x 8192 1090 and 990.  With one signal tile it still pays
    // off for more than 20 signals (five bins of 32 x 2048 x 512: 14% faster in pairs; of 24
    // signals 4%; of 20, 2% slower) or from nine bins of eight steps on (4 x 2048 x 512: 4%;
    // of four steps 5% slower).
    const bool two = S > 32;
    const int steps = T / 32 / splits;  // of 8-bit codes
    const bool odd = !two && n_bins > 3 && (S > 20 || (n_bins >= 9 && steps >= 8));
    const bool pair = precision != CORR_FP32 && steps > 1 && (n_bins % 2 == 0 || odd) &&
                      // (the rounding up included, a launch has fewer than 2^32 threads in x)
                      (int64_t)(tasks + kXcds) * (n_bins + 1) * 64 * kXWaves < (int64_t)1 << 32;
    const int per = pair ? 2 * ((n_bins + 1) / 2) : n_bins;
    const dim3 grid((unsigned)((tasks + kXcds - 1) / kXcds * kXcds * per)), block(64 * kXWaves);
    const uint8_t *sp8 = (const uint8_t *)spec;
    auto go = [&](auto kernel, auto *a) {
        hipLaunchKernelGGL(kernel, grid, block, 0, st, sp8, gate, a, acc_elems, S, C, T, splits, n_bins);
    };
    int32_t *ai = (int32_t *)acc;
    float *af = (float *)acc;
    switch (precision) {
    case CORR_INT8:
        if (two) pair ? go(xengine_gated_kernel<2, CORR_INT8, int32_t, 2>, ai) : go(xengine_gated_kernel<2, CORR_INT8, int32_t, 1>, ai);
        else pair ? go(xengine_gated_kernel<1, CORR_INT8, int32_t, 2>, ai) : go(xengine_gated_kernel<1, CORR_INT8, int32_t, 1>, ai);
        break;
    case CORR_FP8_E4M3:
        if (two) pair ? go(xengine_gated_kernel<2, CORR_FP8_E4M3, float, 2>, af) : go(xengine_gated_kernel<2, CORR_FP8_E4M3, float, 1>, af);
        else pair ? go(xengine_gated_kernel<1, CORR_FP8_E4M3, float, 2>, af) : go(xengine_gated_kernel<1, CORR_FP8_E4M3, float, 1>, af);
        break;
    case CORR_FP32:
        if (two) go(xengine_gated_kernel<2, CORR_FP32, float, 1>, af);
        else go(xengine_gated_kernel<1, CORR_FP32, float, 1>, af);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_xengine_batch(const XBatchArgs &a, hipStream_t st) {
    if (a.n < 1 || a.n > kMaxBatch) return hipErrorInvalidValue;
    hipLaunchKernelGGL(xengine_batch_kernel, dim3(a.first[a.n]), dim3(64 * kXWaves), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_xpack(int precision, const void *in, void *spec, int S, int C, int T, hipStream_t st) {
    // T is a multiple of 32 and C a power of two >= 256, so the waves are whole.  The
    // signals are the y extent of grid and workgroup: a launch has fewer than 2^32
    // threads in x, here T C / 2 at most, whatever S is (FP32 spectra of 64 GiB a signal).
    const unsigned ny = (unsigned)((S + 3) / 4);
    const dim3 block(64, (unsigned)(S < 4 ? S : 4));
    if (precision == CORR_FP32)
        hipLaunchKernelGGL(xpack32_kernel, dim3((unsigned)((int64_t)(T / 2) * C / 64), ny), block, 0, st,
                           (const float2 *)in, (float4 *)spec, S, (int64_t)T, log2_of(C));
    else
        hipLaunchKernelGGL(xpack8_kernel, dim3((unsigned)((int64_t)(T / 8) * (C / 8) / 64), ny), block, 0, st,
                           (const uint8_t *)in, (uint4 *)spec, S, (int64_t)T, log2_of(C));
    return hipGetLastError();
}

}  // namespace corr
