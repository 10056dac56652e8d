// cnn.hip -- the learned RFI flagger.
//
// The paper removes interference with the MAD statistic (section 5, Eq. 3 and
// Eq. 4) and notes that better filtering leaves room for improvement; this
// flagger learns from those MAD labels.  Network, per 64 x 256 (spectra x
// channels) tile of one signal's power P, each tile its own zero-padded image:
//   x  = log(1 + P / m),  m = median over the tile's channels of the channel's
//        mean power over the tile's spectra (1 when that median is not > 0)
//   z1 = conv3x3(x; 1 -> 16),   a1 = ReLU(z1)
//   z2 = conv3x3(a1; 16 -> 16), a2 = ReLU(z2)
//   z3 = conv3x3(a2; 16 -> 1)   (logit; flag when sigmoid(z3) > threshold)
// with conv3x3 the "same"-size cross-correlation
//   y[o][r][c] = b[o] + sum_i sum_{u,v} w[o][i][u][v] a[i][r + u - 1][c + v - 1].
// Training minimises the mean binary cross-entropy against MAD labels with
// Adam (Kingma & Ba 2015).
//
// Two implementations:
//   * training path (FP32; the 16-channel layers on the FP32 matrix cores):
//     layer by layer on a batch of tiles with every activation kept for the backward pass, the
//     weight gradients reduced per block and then over blocks in FP64;
//   * inference (FP16 operands, FP32 accumulation, MFMA): one workgroup per
//     tile runs all three layers with the activations in LDS ring buffers and
//     writes only the flags (and optionally the logits).
#include <algorithm>
#include <type_traits>

#include "corr_internal.h"

namespace corr {
namespace {

constexpr int H = kFlagTileSpectra;   // 64 spectra per tile
constexpr int W = kFlagTileChannels;  // 256 channels per tile
constexpr int HW = kCnnPixels;
// parameter offsets in the flat vector
constexpr int kW1 = 0, kB1 = 144, kW2 = 160, kB2 = 2464, kW3 = 2480, kB3 = 2624;

// Training blocks: 8 rows x 64 columns of one tile, staged with a one-pixel halo.
constexpr int BR = 8, BC = 64;
constexpr int LR = BR + 2, LC = BC + 2;
static_assert((H / BR) * (W / BC) == kCnnBlocksPerTile, "block count");

__device__ inline void tile_coords(int tile, int64_t T, int C, int &s, int64_t &m0, int &k0) {
    const int ntk = C / W;
    const int64_t ntm = T / H;
    k0 = (tile % ntk) * W;
    const int64_t rest = tile / ntk;
    m0 = (rest % ntm) * H;
    s = (int)(rest / ntm);
}

// ------------------------------------------------------------------ training

// Reference level m of each batch tile (median of its 256 channel means), then
// x = log(1 + P / m) and the labels as 0/1 floats.  A tile id outside the data
// is recorded in err and gives x = y = 0.
// A batch is a few tiles, far fewer than compute units, so latency bounds this:
// kGatherSplit workgroups share a tile; each takes the level itself (1024
// threads, 16 rows of a column each, every load issued before the first sum;
// one wave takes the median in registers) and writes its own rows.  16 tiles:
// 49 us with one 256-thread workgroup per tile walking its rows twice, 20 us
// with one of 1024 threads (the logarithms on 16 compute units), 8 us now.
constexpr int kGatherThreads = 1024, kGatherRows = H * W / kGatherThreads, kGatherSplit = 8;
__global__ void __launch_bounds__(kGatherThreads) cnn_gather_kernel(const float *__restrict__ power,
                                                                    const uint8_t *__restrict__ labels, int S,
                                                                    int64_t T, int C,
                                                                    const int32_t *__restrict__ tiles, float *x,
                                                                    float *y, uint32_t *err) {
    constexpr int NG = kGatherThreads / W;           // row groups
    constexpr int OUT = H / kGatherSplit, NO = OUT / NG;  // rows this workgroup writes, per thread
    __shared__ float v[NG][W];
    __shared__ float level;
    const int b = blockIdx.x / kGatherSplit, r0 = (blockIdx.x % kGatherSplit) * OUT;
    const int t = threadIdx.x, c = t % W, g = t / W;
    const int tile = tiles[b];
    const int64_t n_tiles = (int64_t)S * (T / H) * (C / W);
    float *xb = x + (int64_t)b * HW, *yb = y + (int64_t)b * HW;
    if (tile < 0 || tile >= n_tiles) {
        if (t == 0) atomicOr(err, 1u);
        for (int p = r0 * W + t; p < (r0 + OUT) * W; p += kGatherThreads) xb[p] = yb[p] = 0.f;
        return;
    }
    int s, k0;
    int64_t m0;
    tile_coords(tile, T, C, s, m0, k0);
    const int64_t base = ((int64_t)s * T + m0) * C + k0 + c;
    float p[kGatherRows], own[NO];
    uint8_t lab[NO];
#pragma unroll
    for (int i = 0; i < kGatherRows; ++i) p[i] = power[base + (int64_t)(NG * i + g) * C];
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        const int64_t o = base + (int64_t)(r0 + NG * i + g) * C;
        own[i] = power[o];
        lab[i] = labels ? labels[o] : 0;
    }
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < kGatherRows; ++i) acc += p[i];
    v[g][c] = acc;
    __syncthreads();
    if (t < 64) {
        float m[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float sum = 0.f;
#pragma unroll
            for (int h = 0; h < NG; ++h) sum += v[h][4 * t + q];
            m[q] = sum * (1.0f / H);
        }
        const float med = wave_median256(m, t);
        if (t == 0) level = med > 0.f ? med : 1.f;
    }
    __syncthreads();
    const float lv = level;
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        const int o = (r0 + NG * i + g) * W + c;
        xb[o] = log1pf(own[i] / lv);
        yb[o] = lab[i] ? 1.f : 0.f;
    }
}

// Direct 3x3 convolution of one channel, [B][H][W] -> [B][16][H][W], one 8 x 64
// block per workgroup, two pixels (rows t/64 and t/64 + 4) per thread.
//   MODE 0  forward (layer 1)
//   MODE 2  data gradient of layer 2's output: input is dz3, the weights are
//           layer 3's, flipped (da2[o] = w3[o] * dz3 shifted), and the output
//           is gated by z2 > 0.
template <int MODE>
__global__ void __launch_bounds__(256) cnn_conv1_kernel(const float *__restrict__ in, const float *__restrict__ w,
                                                        const float *__restrict__ bias,
                                                        const float *__restrict__ gate, float *__restrict__ out) {
    constexpr int CO = 16;
    __shared__ float sx[LR][LC];
    const int blk = blockIdx.x % kCnnBlocksPerTile;
    const int64_t b = blockIdx.x / kCnnBlocksPerTile;
    const int r0 = (blk / (W / BC)) * BR, c0 = (blk % (W / BC)) * BC;
    const int t = threadIdx.x;
    const float *src = in + b * HW;
    for (int e = t; e < LR * LC; e += 256) {
        const int rr = e / LC, cc = e % LC;
        const int r = r0 + rr - 1, c = c0 + cc - 1;
        sx[rr][cc] = (r >= 0 && r < H && c >= 0 && c < W) ? src[r * W + c] : 0.f;
    }
    __syncthreads();
    const int c = t % BC, ra = t / BC;
    float acc0[CO], acc1[CO];
#pragma unroll
    for (int o = 0; o < CO; ++o) acc0[o] = acc1[o] = MODE == 2 ? 0.f : bias[o];
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            const float x0 = sx[ra + u][c + v], x1 = sx[ra + 4 + u][c + v];
#pragma unroll
            for (int o = 0; o < CO; ++o) {
                const float wv = MODE == 2 ? w[(o * 3 + 2 - u) * 3 + 2 - v] : w[(o * 3 + u) * 3 + v];
                acc0[o] = fmaf(wv, x0, acc0[o]);
                acc1[o] = fmaf(wv, x1, acc1[o]);
            }
        }
    const int p0 = (r0 + ra) * W + c0 + c, p1 = p0 + 4 * W;
#pragma unroll
    for (int o = 0; o < CO; ++o) {
        const int64_t ob = (b * CO + o) * HW;
        float v0 = acc0[o], v1 = acc1[o];
        if (MODE == 2) {
            v0 = gate[ob + p0] > 0.f ? v0 : 0.f;
            v1 = gate[ob + p1] > 0.f ? v1 : 0.f;
        }
        out[ob + p0] = v0;
        out[ob + p1] = v1;
    }
}

// The 16-channel layers of the training path run on the FP32 matrix cores
// (v_mfma_f32_16x16x4f32: D[m][n] += sum of A[m][k] B[k][n] over four k; lane l
// gives A at (l mod 16, l / 16), B at (l / 16, l mod 16) and holds D at rows
// 4 (l / 16) + r, column l mod 16).  They are bound by their multiply-adds
// (2304 a pixel), which the vector ALUs issued at a third of their rate behind
// 16 scalar weight loads a tap; every operand keeps FP32.
typedef float trn4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ trn4 mfma4(float a, float b, trn4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// An 8 x 64 block of CH channels with its halo into LDS planes [LR][LC] at a
// pitch of PITCH floats: a wave takes the 64 middle columns of a row.  Rows
// outside the tile load a row inside it and store zero, so that every load is
// issued and none waits for a branch.
template <int CH, int PITCH, bool RELU>
__device__ __forceinline__ void stage_halo(const float *__restrict__ src, int r0, int c0, float *s) {
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    constexpr int ROWS = CH * LR, NR = ROWS / 4, NE = (2 * ROWS + 255) / 256;
    static_assert(BC == 64 && ROWS % 4 == 0, "whole rows of a wave");
    float v[NR], e[NE];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int k = wv + 4 * i, r = r0 + k % LR - 1;
        v[i] = src[(int64_t)(k / LR) * HW + min(max(r, 0), H - 1) * W + c0 + lane];
    }
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int k = min((t + 256 * i) >> 1, ROWS - 1), r = r0 + k % LR - 1, c = (t & 1) ? c0 + BC : c0 - 1;
        e[i] = src[(int64_t)(k / LR) * HW + min(max(r, 0), H - 1) * W + min(max(c, 0), W - 1)];
    }
    auto put = [&](int k, int cc, float x, bool in) {
        s[(k / LR) * PITCH + (k % LR) * LC + cc] = !in ? 0.f : RELU ? fmaxf(x, 0.f) : x;
    };
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int k = wv + 4 * i, r = r0 + k % LR - 1;
        put(k, 1 + lane, v[i], r >= 0 && r < H);
    }
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int k = (t + 256 * i) >> 1, r = r0 + k % LR - 1, c = (t & 1) ? c0 + BC : c0 - 1;
        if (k < ROWS) put(k, (t & 1) ? LC - 1 : 0, e[i], r >= 0 && r < H && c >= 0 && c < W);
    }
}

// 3x3 convolution of 16 channels to 16, [B][16][H][W] -> [B][16][H][W].
//   MODE 1  forward: input is z of the previous layer (ReLU applied on load)
//   MODE 2  data gradient: input is dz of the layer, the weights flipped and
//           transposed (da[i] = sum_o w[o][i] * dz[o] shifted), the output
//           gated by z of the previous layer > 0.
// One 8 x 64 block per workgroup; wave w takes the 16 columns 16 w .. of all
// eight rows (rows of D = output channels, columns = pixels).  Backward, K is
// four channels of one tap: a staged value then serves the three output rows
// it touches, 120 LDS reads for 288 products (planes 16 modulo the 64 banks
// apart).  Forward, K is four of the 144 (channel, tap) pairs in the weights'
// order, so that the sum of every pixel runs in that order too: the sign of z2
// decides what the gradient passes through.  16 tiles: 40.5 us each as direct
// convolutions on the vector ALUs, 27 us forward and 21 us backward now.
constexpr int kConvPitch = 720;
template <int MODE>
__global__ void __launch_bounds__(256) cnn_conv16_kernel(const float *__restrict__ in, const float *__restrict__ w,
                                                         const float *__restrict__ bias,
                                                         const float *__restrict__ gate, float *__restrict__ out) {
    __shared__ float sx[16 * kConvPitch];
    const int blk = blockIdx.x % kCnnBlocksPerTile;
    const int64_t b = blockIdx.x / kCnnBlocksPerTile;
    const int r0 = (blk / (W / BC)) * BR, c0 = (blk % (W / BC)) * BC;
    const int t = threadIdx.x, lane = t & 63, col = lane & 15, quad = lane >> 4, cw = 16 * (t >> 6);
    float A[4][9];  // [group of four channels][tap, or K quad of the group's 36 pairs]
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int k = 0; k < 9; ++k)
            A[g][k] = MODE == 2 ? w[((4 * g + quad) * 16 + col) * 9 + 8 - k] : w[col * 144 + 36 * g + 4 * k + quad];
    stage_halo<16, kConvPitch, MODE == 1>(in + b * 16 * HW, r0, c0, sx);
    trn4 acc[BR];
#pragma unroll
    for (int i = 0; i < BR; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][r] = MODE == 2 ? 0.f : bias[4 * quad + r];
    __syncthreads();
    if constexpr (MODE == 1) {
        const float *sb[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const int q = 4 * k + quad, tap = q % 9;
            sb[k] = sx + (q / 9) * kConvPitch + (tap / 3) * LC + tap % 3 + cw + col;
        }
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int k = 0; k < 9; ++k)
#pragma unroll
                for (int i = 0; i < BR; ++i) acc[i] = mfma4(A[g][k], sb[k][4 * g * kConvPitch + i * LC], acc[i]);
    } else {
        const float *sb = sx + quad * kConvPitch + cw + col;
#pragma unroll
        for (int rr = 0; rr < LR; ++rr)
#pragma unroll
            for (int v = 0; v < 3; ++v)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float x = sb[4 * g * kConvPitch + rr * LC + v];
#pragma unroll
                    for (int u = 0; u < 3; ++u)
                        if (rr - u >= 0 && rr - u < BR) acc[rr - u] = mfma4(A[g][3 * u + v], x, acc[rr - u]);
                }
    }
#pragma unroll
    for (int i = 0; i < BR; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t o = (b * 16 + 4 * quad + r) * HW + (r0 + i) * W + c0 + cw + col;
            float v = acc[i][r];
            if (MODE == 2) v = gate[o] > 0.f ? v : 0.f;
            out[o] = v;
        }
}

// Layer 3, 16 channels to 1: the 9 tap products of every pixel,
// U[tap][q] = sum_i w3[i][tap] ReLU(z2[i][q]), on the matrix cores (rows of D =
// taps) straight from global memory, then z3[p] = b3 + the sum of U over p's
// nine shifted neighbours from LDS.  An 8 x 64 block with its halo as 10 rows
// of five 16-pixel groups.  16 tiles: 21 us as a direct convolution, 10.5 us now.
__global__ void __launch_bounds__(256) cnn_conv_out_kernel(const float *__restrict__ in, const float *__restrict__ w,
                                                           const float *__restrict__ bias, float *__restrict__ out) {
    constexpr int NG = 5, UC = 16 * NG + 1;  // column groups; padded row of U
    __shared__ float us[9][LR][UC];
    const int blk = blockIdx.x % kCnnBlocksPerTile;
    const int64_t b = blockIdx.x / kCnnBlocksPerTile;
    const int r0 = (blk / (W / BC)) * BR, c0 = (blk % (W / BC)) * BC;
    const int t = threadIdx.x, lane = t & 63, col = lane & 15, quad = lane >> 4;
    float A[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) A[g] = col < 9 ? w[(4 * g + quad) * 9 + col] : 0.f;
    const float *src = in + b * 16 * HW;
    constexpr int NK = (LR * NG + 3) / 4;  // groups a wave takes; the last may repeat one, with the same values
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    float x[NK][4];
#pragma unroll
    for (int i = 0; i < NK; ++i) {
        const int k = min(wv + 4 * i, LR * NG - 1);
        const int r = min(max(r0 + k / NG - 1, 0), H - 1), c = min(max(c0 + 16 * (k % NG) + col - 1, 0), W - 1);
#pragma unroll
        for (int g = 0; g < 4; ++g) x[i][g] = src[(int64_t)(4 * g + quad) * HW + r * W + c];
    }
#pragma unroll
    for (int i = 0; i < NK; ++i) {
        const int k = min(wv + 4 * i, LR * NG - 1);
        const int rr = k / NG, cc = 16 * (k % NG) + col;  // columns from c0 - 1
        const int r = r0 + rr - 1, c = c0 + cc - 1;
        const bool ok = r >= 0 && r < H && c >= 0 && c < W;
        trn4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < 4; ++g) d = mfma4(A[g], ok ? fmaxf(x[i][g], 0.f) : 0.f, d);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (4 * quad + q < 9) us[4 * quad + q][rr][cc] = d[q];
    }
    __syncthreads();
    const float b3 = bias[0];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int c = t % BC, ra = t / BC + 4 * h;
        float z = b3;
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int v = 0; v < 3; ++v) z += us[3 * u + v][ra + u][c + v];
        out[b * HW + (r0 + ra) * W + c0 + c] = z;
    }
}

// Weight and bias gradients of layer 2 over one 8 x 64 block:
//   part[blk][(o 16 + i) 9 + 3u + v] = sum_p dz[o][p] a[i][p + (u - 1, v - 1)]
//   part[blk][2304 + o]             = sum_p dz[o][p],  a = ReLU(z1)
// Rows of D = o, columns = i, K = four pixels of a row; wave w takes 4 of the
// 16 column groups, and an input row it reads serves the three dz rows it
// meets.  The plane pitches are 4 modulo the 64 banks (16 channels x 4 pixels
// a read).  The four waves' sums meet in LDS.  16 tiles: 48 us with a sliding
// window per channel pair on the vector ALUs, 21 us now.
constexpr int kGradPitchA = 708, kGradPitchD = BR * BC + 4;
__global__ void __launch_bounds__(256) cnn_wgrad16_kernel(const float *__restrict__ ain, const float *__restrict__ dz,
                                                          float *__restrict__ part) {
    constexpr int E = kCnnGradEntries;
    __shared__ float sa[16 * kGradPitchA], sd[16 * kGradPitchD];
    static_assert(4 * 9 * 256 <= 16 * kGradPitchA && 4 * 16 <= 16 * kGradPitchD, "the waves' sums reuse the planes");
    const int blk = blockIdx.x % kCnnBlocksPerTile;
    const int64_t b = blockIdx.x / kCnnBlocksPerTile;
    const int r0 = (blk / (W / BC)) * BR, c0 = (blk % (W / BC)) * BC;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, ch = lane & 15, quad = lane >> 4;
    stage_halo<16, kGradPitchA, true>(ain + b * 16 * HW, r0, c0, sa);
#pragma unroll
    for (int i = 0; i < 16 * BR / 4; ++i) {
        const int k = wv + 4 * i;
        sd[(k / BR) * kGradPitchD + (k % BR) * BC + lane] = dz[(b * 16 + k / BR) * HW + (r0 + k % BR) * W + c0 + lane];
    }
    __syncthreads();
    trn4 acc[3][3];
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int v = 0; v < 3; ++v) acc[u][v] = trn4{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
#pragma unroll 1
    for (int g = wv; g < BC / 4; g += 4) {
        const float *pa = sa + ch * kGradPitchA + 4 * g + quad, *pd = sd + ch * kGradPitchD + 4 * g + quad;
        float d[BR];
#pragma unroll
        for (int r = 0; r < BR; ++r) {
            d[r] = pd[r * BC];
            bsum += d[r];
        }
#pragma unroll
        for (int rr = 0; rr < LR; ++rr)
#pragma unroll
            for (int v = 0; v < 3; ++v) {
                const float x = pa[rr * LC + v];
#pragma unroll
                for (int u = 0; u < 3; ++u)
                    if (rr - u >= 0 && rr - u < BR) acc[u][v] = mfma4(d[rr - u], x, acc[u][v]);
            }
    }
    bsum += __shfl_xor(bsum, 16);
    bsum += __shfl_xor(bsum, 32);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int r = 0; r < 4; ++r) sa[wv * 2304 + ((4 * quad + r) * 16 + ch) * 9 + 3 * u + v] = acc[u][v][r];
    if (lane < 16) sd[wv * 16 + lane] = bsum;
    __syncthreads();
    float *pb = part + (int64_t)blockIdx.x * E;
    for (int e = t; e < E; e += 256)
        pb[e] = e < 2304 ? (sa[e] + sa[2304 + e]) + (sa[4608 + e] + sa[6912 + e])
                         : (sd[e - 2304] + sd[e - 2288]) + (sd[e - 2272] + sd[e - 2256]);
}

// Weight and bias gradients of the layers with one channel on one side, over
// one 8 x 64 block, t one channel and y sixteen:
//   layer 1 (SIGN = +1, t = x, y = dz1):
//     part[o 9 + 3u + v] = sum_p dz1[o][p] x[p + (u - 1, v - 1)]
//     part[144 + o]      = sum_p dz1[o][p]
//   layer 3 (SIGN = -1, t = dz3, y = ReLU(z2)):
//     part[i 9 + 3u + v] = sum_p dz3[p] a2[i][p + (u - 1, v - 1)]
//                        = sum_q a2[i][q] dz3[q - (u - 1, v - 1)]
//     part[144]          = sum_p dz3[p]
// Rows of D = the nine taps (and a row of ones for layer 1's bias), columns =
// channels, K = pixels: only the single channel needs a halo, and y goes from
// global memory into the products, 16 bytes a lane (the four pixels of a lane
// are one K slot each of four products).  A pixel of layer 3 outside the tile
// has a2 = 0, and q runs over the tile's own pixels, so the sums over blocks
// are the same.  16 tiles: 16 (layer 1) and 22 us (layer 3) as sliding windows
// on the vector ALUs, 7 us now.
template <int SIGN>
__global__ void __launch_bounds__(256) cnn_wgrad9_kernel(const float *__restrict__ tin, const float *__restrict__ yin,
                                                         float *__restrict__ part) {
    constexpr int E = 16 * 9 + (SIGN > 0 ? 16 : 1);
    __shared__ float st[LR][LC];
    __shared__ float red[4][16][16];
    __shared__ float bred[4];
    const int blk = blockIdx.x % kCnnBlocksPerTile;
    const int64_t b = blockIdx.x / kCnnBlocksPerTile;
    const int r0 = (blk / (W / BC)) * BR, c0 = (blk % (W / BC)) * BC;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6, n = lane & 15, quad = lane >> 4;
    // this wave's y: rows wv and wv + 4, four groups of 16 pixels each
    float4 y[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            y[h][g] = *reinterpret_cast<const float4 *>(yin + (b * 16 + n) * HW + (r0 + wv + 4 * h) * W + c0 + 16 * g +
                                                        4 * quad);
    for (int e = t; e < LR * LC; e += 256) {
        const int r = r0 + e / LC - 1, c = c0 + e % LC - 1;
        st[e / LC][e % LC] = (r >= 0 && r < H && c >= 0 && c < W) ? tin[b * HW + r * W + c] : 0.f;
    }
    __syncthreads();
    const int tap = n < 9 ? n : 0, du = SIGN * (tap / 3 - 1), dv = SIGN * (tap % 3 - 1);
    trn4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float *row = &st[wv + 4 * h + 1 + du][16 * g + 4 * quad + 1 + dv];
            const float yy[4] = {y[h][g].x, y[h][g].y, y[h][g].z, y[h][g].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float a = n < 9 ? row[j] : n == 9 ? 1.f : 0.f;
                acc = mfma4(a, SIGN > 0 ? yy[j] : fmaxf(yy[j], 0.f), acc);
            }
        }
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wv][4 * quad + r][n] = acc[r];
    if (SIGN < 0) {  // the bias of layer 3: the sum of the block's dz3
        float s = st[wv + 1][lane + 1] + st[wv + 5][lane + 1];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m);
        if (lane == 0) bred[wv] = s;
    }
    __syncthreads();
    float *pb = part + (int64_t)blockIdx.x * E;
    if (t < 160) {
        const int k = t < 144 ? t % 9 : 9, c = t < 144 ? t / 9 : t - 144;
        const float s = (red[0][k][c] + red[1][k][c]) + (red[2][k][c] + red[3][k][c]);
        if (t < 144 || SIGN > 0) pb[t] = s;
        if (SIGN < 0 && t == 144) pb[t] = (bred[0] + bred[1]) + (bred[2] + bred[3]);
    }
}

// grad[e] = sum over blocks of part[blk][e], in FP64 and in a fixed order: a
// workgroup takes 16 entries, thread (l, q) the blocks q, q + 64, ... of entry
// l, and the 64 partial sums meet in LDS.  The sum is a chain of loads, so its
// length is what bounds it: one thread per entry walked all n blocks (119 us
// for the 512 blocks of 16 tiles), now n / 64 of them (5 us).
constexpr int kRedEntries = 16, kRedSlices = 64;
__global__ void __launch_bounds__(kRedEntries *kRedSlices) cnn_reduce_kernel(const float *__restrict__ part,
                                                                             int nparts, int E, float *grad) {
    __shared__ double red[kRedSlices][kRedEntries];
    const int l = threadIdx.x % kRedEntries, q = threadIdx.x / kRedEntries;
    const int e = blockIdx.x * kRedEntries + l;
    double s = 0.0;
    if (e < E) {
#pragma unroll 8
        for (int k = q; k < nparts; k += kRedSlices) s += part[(int64_t)k * E + e];
    }
    red[q][l] = s;
    __syncthreads();
#pragma unroll
    for (int h = kRedSlices / 2; h > 0; h >>= 1) {
        if (q < h) red[q][l] += red[q + h][l];
        __syncthreads();
    }
    if (q == 0 && e < E) grad[e] = (float)red[0][l];
}

// Binary cross-entropy with logits: loss terms max(z, 0) - z y + log(1 + e^-|z|)
// summed per block (FP64), dz = (sigmoid(z) - y) / n.
__global__ void __launch_bounds__(256) cnn_bce_kernel(const float *__restrict__ z, const float *__restrict__ y,
                                                      int64_t n, float *dz, double *lpart) {
    __shared__ double red[256];
    const float inv_n = (float)(1.0 / (double)n);
    double acc = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (int64_t)gridDim.x * 256) {
        const float zz = z[p], yy = y[p];
        acc += (double)(fmaxf(zz, 0.f) - zz * yy + log1pf(expf(-fabsf(zz))));
        dz[p] = (1.f / (1.f + expf(-zz)) - yy) * inv_n;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) lpart[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(256) cnn_loss_final_kernel(const double *__restrict__ lpart, int nb, int64_t n,
                                                             float *loss) {
    __shared__ double red[256];
    double s = 0.0;
    for (int k = threadIdx.x; k < nb; k += 256) s += lpart[k];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = (float)(red[0] / (double)n);
}

// Adam: m = b1 m + (1 - b1) g, v = b2 v + (1 - b2) g^2,
// p -= lr (m c1) / (sqrt(v c2) + eps), c1 = 1 / (1 - b1^t), c2 = 1 / (1 - b2^t).
__global__ void cnn_adam_kernel(float *p, float *m, float *v, const float *__restrict__ g, int n, float lr,
                                float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// ----------------------------------------------------------------- inference

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef short short2v __attribute__((ext_vector_type(2)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int XCOLS = W + 4;  // input columns: zero column on the left, three on the right
constexpr int PC = W + 2;     // activation row pitch: one zero column at each edge
constexpr int RX = 8;         // rows kept of the input, of the layer-1 output and of the tap sums
constexpr int XPITCH = 10;    // halves per input column: RX rows + 2 pad (odd dword stride)
constexpr int IWG = 1024;     // 16 waves, two for each 32-column strip

// Accumulator layout of a 32 x 32 MFMA: register j of lane l holds row
// 8 (j / 4) + 4 (l / 32) + j mod 4, column l mod 32.
__device__ inline int acc_row(int j, int half) { return 8 * (j / 4) + 4 * half + (j & 3); }

// Two floats -> two FP16 (round to nearest even) with negatives set to +0:
// ReLU commutes with the monotone conversion, and on FP16 bit patterns the
// signed 16-bit max against 0 clears exactly the negative values.
__device__ inline uint32_t relu_h2(float a, float b) {
    const half2v h = __builtin_convertvector((float2v){a, b}, half2v);
    const short2v m = __builtin_elementwise_max(__builtin_bit_cast(short2v, h), (short2v){0, 0});
    return __builtin_bit_cast(uint32_t, m);
}

// Byte offset of the 16-byte half `h` (channels 8h .. 8h + 7) of pixel column
// pcol in a layer-1 output row: the halves swap places by bit 2 xor bit 3 of
// the column, so the 16-byte reads of 8 (or 16) consecutive lanes cover all 32
// (or 64) LDS banks once.
__device__ inline int a1_off(int pcol, int h) { return 32 * pcol + 16 * (h ^ (((pcol >> 2) ^ (pcol >> 3)) & 1)); }

// One workgroup per compute unit, looping over tiles.  Two waves own columns
// 32 w .. 32 w + 31 and walk the tile two rows at a time in a software pipeline
// with one barrier per step j.  The row wave takes
//   x rows 2j + 5, 2j + 6 = log(1 + P / m) (FP16) into the input ring,
//   layer 1 for rows 2j + 2, 2j + 3,
//   the logits of rows 2j - 6, 2j - 5,
// mostly vector instructions and LDS accesses, the other
//   layer 2 and the layer-3 tap sums for rows 2j - 2, 2j - 1,
// mostly matrix products, which so run beside the first, each stage reading only
// what earlier steps wrote, from rings of 8 rows.  A wave that took all the stages in
// turn had every unit waiting for another (matrix cores, vector ALUs and LDS each
// busy 42%; 64 x 4096 x 4096 FP16 cells with 8 such waves 8030 us, now 7280).  The
// layer-2 waves have the higher priority (4% slower without): their step is the
// longer one.
// Layer 2 of a row pair reads layer-1 rows 2j - 3 .. 2j; the first two were
// read by the previous step and stay in registers.  Layer-1 rows -1 and 64
// are zero rows in the ring.  Steps run four at a time (the ring period), so
// every ring slot is a constant.  While a tile is processed, the column sums
// of the next tile and the input rows its first step needs are fetched.
// MFMA roles (32 x 32 x 16, FP16 in, FP32 out):
//   layer 1: rows = (row slot, out channel) for two rows; K = 4 input rows x 4
//            column offsets, lane half h taking input rows 2h and 2h + 1,
//            slot j = (row 2h + j mod 2, offset j / 2): with the input stored
//            column-major each slot pair is one aligned dword (offset 3 has
//            zero weight; the bias rides on slot 7 of half 0, set to 1);
//   layer 2: rows = (row slot, out channel); one product per (input row,
//            column offset), K = 16 channels, the weights of the taps a row
//            slot does not use set to zero;
//   layer 3: U[tap][q] = sum_i w3[i][tap] a2[i][q] with rows = the 9 taps, fed
//            directly from the layer-2 accumulator (its 8 channels per lane
//            are exactly one lane's K slots), then z3[p] = b3 + sum of U over
//            the 9 shifted neighbours of p.
template <typename PT, bool LOGITS>
__global__ void __launch_bounds__(IWG) cnn_infer_kernel(const float *__restrict__ params,
                                                        const PT *__restrict__ power, int64_t T, int C,
                                                        int n_tiles, float thr_logit, float guard_m,
                                                        uint8_t *__restrict__ flags,
                                                        float *__restrict__ logits) {
    __shared__ __align__(16) _Float16 xs[XCOLS][XPITCH];  // column-major input ring (slot = (row + 1) mod 8)
    __shared__ __align__(16) _Float16 a1s[RX][PC][16];   // layer-1 ring (slot = row mod 8)
    __shared__ float us[RX][PC][9];                      // tap-sum ring (slot = row mod 8)
    __shared__ float colv[2][W];                         // column sums of even / odd rows
    __shared__ __align__(16) float srt[W];               // sorted channel means (guard)
    __shared__ uint8_t guard[W / 4];
    __shared__ float level;                              // the tile's median

    const int t = threadIdx.x, lane = t & 63, wv = (t >> 6) & 7;
    const int half = lane >> 5, col = lane & 31;

    // ---- zero border columns, written once (never overwritten below)
    for (int e = t; e < 4 * XPITCH; e += IWG) xs[(e / XPITCH) == 0 ? 0 : W + (e / XPITCH)][e % XPITCH] = (_Float16)0.f;
    for (int e = t; e < RX * 2 * 16; e += IWG) {
        const int rr = e / 32, side = (e / 16) & 1, ch = e & 15;
        a1s[rr][side ? PC - 1 : 0][ch] = (_Float16)0.f;
    }
    for (int e = t; e < RX * 2 * 9; e += IWG) {
        const int rr = e / 18, side = (e / 9) & 1, k = e % 9;
        us[rr][side ? PC - 1 : 0][k] = 0.f;
    }

    const int arow = lane & 31, aslot = arow >> 4, ao = arow & 15;  // A operands: lane: row = lane mod 32, K slots 8 half + j
    const float16v zero16 = {};
    const int c0 = wv * 32;
    const int pc = c0 + col + 1;  // padded column of this lane's pixel
    const uint32_t *xl = reinterpret_cast<const uint32_t *>(&xs[c0 + col][0]);
    const uint32_t bias_and = half ? 0xFFFFFFFFu : 0x0000FFFFu;  // half 0: slot 7 := 1.0
    const uint32_t bias_or = half ? 0u : 0x3C000000u;
    char *a1base = reinterpret_cast<char *>(&a1s[0][0][0]);
    const int a1w0 = a1_off(pc, 0) + 8 * half, a1w1 = a1_off(pc, 1) + 8 * half;
    int a1rd[3];
#pragma unroll
    for (int dv = 0; dv < 3; ++dv) a1rd[dv] = a1_off(pc - 1 + dv, half);
    float *uw = &us[0][pc][4 * half];
    const float *ur = &us[0][pc - 1][0];
    constexpr int AROW = PC * 16 * 2, UROW = PC * 9;  // bytes, floats

    // the two halves of the workgroup pass the same barriers: three at the top of a
    // tile and one after each of its steps
    if (__builtin_amdgcn_readfirstlane(t) >= IWG / 2) {
        __builtin_amdgcn_s_setprio(2);
        half8 A3, A2[4][3];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int ch = 8 * (j / 4) + 4 * half + (j & 3);
            A3[j] = (_Float16)(arow < 9 ? params[kW3 + ch * 9 + arow] : 0.f);
        }
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int dv = 0; dv < 3; ++dv)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int cin = 8 * half + j, u = p - aslot;
                    A2[p][dv][j] = (_Float16)((u >= 0 && u <= 2) ? params[kW2 + ((ao * 16 + cin) * 3 + u) * 3 + dv] : 0.f);
                }
        float bias2[8];  // of accumulator registers j and j + 8
#pragma unroll
        for (int j = 0; j < 8; ++j) bias2[j] = params[kB2 + acc_row(j, half)];
        for (int tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
            __syncthreads();
            __syncthreads();
            __syncthreads();
            half8 Fa[3], Fb[3];  // layer-1 operands of rows 2j - 3, 2j - 2, read by the previous step
            // Layer 2 and the tap sums (mostly the matrix cores), rows r2, r2 + 1,
            // r2 = 2j - 2 (layer-1 rows r2 - 1 .. r2 + 2):
            auto stage_layer2 = [&](const int j, auto body_tag) __attribute__((always_inline)) {
                constexpr bool BODY = decltype(body_tag)::value;
                if (!BODY && (j < 0 || j > H / 2)) return;
                half8 Fc[3], Fd[3];  // layer-1 rows 2j - 1, 2j
                const char *fc = a1base + ((2 * j - 1) & (RX - 1)) * AROW;
                const char *fd = a1base + ((2 * j) & (RX - 1)) * AROW;
#pragma unroll
                for (int dv = 0; dv < 3; ++dv) {
                    Fc[dv] = *reinterpret_cast<const half8 *>(fc + a1rd[dv]);
                    Fd[dv] = *reinterpret_cast<const half8 *>(fd + a1rd[dv]);
                }
                if (BODY || j >= 1) {
                    const int r2 = 2 * j - 2;
                    float16v D;
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        asm("" : "+v"(bias2[q]));  // otherwise the compiler keeps the copies, in 16 registers
                        D[q] = D[q + 8] = bias2[q];
                    }
#pragma unroll
                    for (int dv = 0; dv < 3; ++dv) D = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[0][dv], Fa[dv], D, 0, 0, 0);
#pragma unroll
                    for (int dv = 0; dv < 3; ++dv) D = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[1][dv], Fb[dv], D, 0, 0, 0);
#pragma unroll
                    for (int dv = 0; dv < 3; ++dv) D = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[2][dv], Fc[dv], D, 0, 0, 0);
#pragma unroll
                    for (int dv = 0; dv < 3; ++dv) D = __builtin_amdgcn_mfma_f32_32x32x16_f16(A2[3][dv], Fd[dv], D, 0, 0, 0);
#pragma unroll
                    for (int sl = 0; sl < 2; ++sl) {
                        u32x4 bu;
#pragma unroll
                        for (int q = 0; q < 4; ++q) bu[q] = relu_h2(D[8 * sl + 2 * q], D[8 * sl + 2 * q + 1]);
                        const float16v U =
                            __builtin_amdgcn_mfma_f32_32x32x16_f16(A3, __builtin_bit_cast(half8, bu), zero16, 0, 0, 0);
                        float *dst = uw + ((r2 + sl) & (RX - 1)) * UROW;
#pragma unroll
                        for (int q = 0; q < 4; ++q) dst[q] = U[q];
                        if (half == 0) dst[8] = U[4];
                    }
                }
#pragma unroll
                for (int dv = 0; dv < 3; ++dv) {
                    Fa[dv] = Fc[dv];
                    Fb[dv] = Fd[dv];
                }
            };
            auto steps = [&](const int jb, auto body_tag) __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    stage_layer2(jb + q, body_tag);
                    __syncthreads();
                }
            };
            steps(-1, std::false_type{});
#pragma unroll 1
            for (int i = 1; i < H / 8; ++i) steps(4 * i - 1, std::true_type{});
            steps(H / 2 - 1, std::false_type{});
        }
        return;
    }

    half8 A1;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int rho = 2 * half + (j & 1), dv = j >> 1, u = rho - aslot;
        float w = (dv < 3 && u >= 0 && u <= 2) ? params[kW1 + ao * 9 + u * 3 + dv] : 0.f;
        if (half == 0 && j == 7) w = params[kB1 + ao];  // constant-1 slot: the bias
        A1[j] = (_Float16)w;
    }
    const float b3 = params[kB3];
    const int xc = t & (W - 1), xh = (t >> 8) & 1;  // input staging: column xc, rows of parity xh
    auto tile_base = [&](int tl) {
        int s, k0;
        int64_t m0;
        tile_coords(tl, T, C, s, m0, k0);
        return ((int64_t)s * T + m0) * C + k0;
    };
    // First tile: column sums of rows xh, xh + 2, ... and the input rows -1 + xh,
    // 1 + xh, 3 + xh of its first steps.  Later tiles get these during the previous one.
    // Offsets inside a tile (row r < 2^6, column c, C up to 2^22: operands of 24 bits,
    // r C + c < 2^29) are 32-bit; tile bases are uniform 64-bit pointers.
    auto roff = [&](int r, int c) { return __umul24((uint32_t)r, (uint32_t)C) + (uint32_t)c; };
    int tile = blockIdx.x;
    // p0, p1: input rows -1 + xh, 1 + xh of a tile; p2 .. p5: rows 3 + xh ..
    // 9 + xh, the first four slots of the input ring
    float csum = 0.f, p0 = 0.f, p1 = 0.f, p2 = 0.f, p3 = 0.f, p4 = 0.f, p5 = 0.f;
    if (tile < n_tiles) {
        const PT *tb = power + tile_base(tile);
#pragma unroll 8
        for (int q = 0; q < 32; ++q) csum += tb[roff(2 * q + xh, xc)];
        p0 = xh ? tb[xc] : 0.f;
        p1 = tb[roff(1 + xh, xc)];
        p2 = tb[roff(3 + xh, xc)];
        p3 = tb[roff(5 + xh, xc)];
        p4 = tb[roff(7 + xh, xc)];
        p5 = tb[roff(9 + xh, xc)];
    }
    for (; tile < n_tiles; tile += gridDim.x) {
        const int64_t base = tile_base(tile);
        const PT *tb = power + base;
        const bool has_next = tile + (int)gridDim.x < n_tiles;
        const PT *tn = has_next ? power + tile_base(tile + gridDim.x) : tb;
        uint8_t *fb = flags + base;
        float *lb = logits + (LOGITS ? base : 0);

        // ---- reference level: median over the 256 channels of each channel's mean power
        colv[xh][xc] = csum;
        for (int e = t; e < PC * 2; e += IWG / 2)  // layer-1 row -1 (slot 7): zero
            reinterpret_cast<uint4 *>(a1base + (RX - 1) * AROW)[e] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        // One wave takes the statistics: eight, alike, shared the SIMDs' issue slots (16 x
        // 4096 x 4096 FP16 cells 2010 us, now 1934).
        if (__builtin_amdgcn_readfirstlane(t) < 64) {
            float cv[4], cm[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) cm[q] = cv[q] = (colv[0][4 * lane + q] + colv[1][4 * lane + q]) * (1.0f / H);
            const float m = wave_median256(cv, lane);  // sorts cv
            // column guard: the channel means are the MAD column statistic (section 5, Eq. 3
            // and 4); a column whose mean is an outlier is flagged whole.  guard[l]: the
            // guard bits of columns 4 l .. 4 l + 3.
            uint32_t bits = 0u;
            if (guard_m > 0.f) {
                const float mad = wave_mad256_sorted(cv, m, lane, srt);
                const float thr = guard_m * mad / 0.6745f;
#pragma unroll
                for (int q = 0; q < 4; ++q) bits |= (fabsf(cm[q] - m) > thr ? 1u : 0u) << q;
            }
            guard[lane] = (uint8_t)bits;
            if (lane == 0) level = m;
        }
        __syncthreads();
        const float med = level;
        const float inv = 1.0f / (med > 0.f ? med : 1.f);
        const uint32_t gcol = (guard[(c0 + col) >> 2] >> (col & 3)) & 1u;  // of this lane's output column
        // x of tile row r -> input ring slot (r + 1) mod 8, zero outside the tile
        auto x_put = [&](int r, float pv) {
            const float v = (r >= 0 && r < H) ? __logf(1.0f + pv * inv) : 0.f;
            xs[xc + 1][(r + 1) & (RX - 1)] = (_Float16)v;
        };
        x_put(-1 + xh, p0);
        x_put(1 + xh, p1);
        // input ring: step j puts row 2j + 5 + xh from slot (j + 1) mod 4 and
        // loads row 2j + 13 + xh, which step j + 4 puts, into the same slot
        float xr0 = p2, xr1 = p3, xr2 = p4, xr3 = p5, cnext = 0.f;
        csum = 0.f;
        __syncthreads();

        // The stages of a step.  BODY: steps 3 .. 30, where every stage has its rows.
        // Rows of the input, layer 1 and the logits (mostly the vector ALUs and the LDS):
        auto stage_rows = [&](const int j, auto slot_tag, auto body_tag) __attribute__((always_inline)) {
            constexpr int SL = decltype(slot_tag)::value;  // (j + 1) mod 4
            constexpr bool BODY = decltype(body_tag)::value;
            float &xs_slot = SL == 0 ? xr0 : SL == 1 ? xr1 : SL == 2 ? xr2 : xr3;
            // layer 1 for rows R, R + 1, R = 2j + 2 (input rows R - 1 .. R + 2); row 64 is zero
            const int R = 2 * j + 2;
            const int r3 = 2 * j - 6;  // logits of rows r3 (lanes 0-31) and r3 + 1 (lanes 32-63)
            const int r = r3 + half;
            u32x4 bx;
            float uv[3][3];
            if (BODY || R < H) {
                const uint32_t *xr = xl + (((R + 2 * half) & (RX - 1)) >> 1);
#pragma unroll
                for (int dv = 0; dv < 4; ++dv) bx[dv] = xr[dv * (XPITCH / 2)];
            }
            if (BODY || (r3 >= 0 && r3 < H)) {
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    const float *row = ur + ((r + u - 1) & (RX - 1)) * UROW;
#pragma unroll
                    for (int v = 0; v < 3; ++v) uv[u][v] = row[9 * v + 3 * u + v];
                }
            }
            float16v D1;
            if (BODY || R < H) {
                bx[3] = (bx[3] & bias_and) | bias_or;
                D1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(A1, __builtin_bit_cast(half8, bx), zero16, 0, 0, 0);
            }
            if (BODY || (r3 >= 0 && r3 < H)) {
                float z = b3;
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    const int rr = r + u - 1;
                    float zu = 0.f;
#pragma unroll
                    for (int v = 0; v < 3; ++v) zu += uv[u][v];
                    z += ((BODY && u > 0) || (rr >= 0 && (BODY || rr < H))) ? zu : 0.f;  // BODY: rr -1 .. 56
                }
                const uint32_t gp = roff(r, c0 + col);
                fb[gp] = (uint8_t)((z > thr_logit ? 1u : 0u) | gcol);
                if constexpr (LOGITS) lb[gp] = z;
            }
            // input row 2j + 5 + xh; row 2j + 13 + xh is fetched for step j + 4, and row
            // 2j + 2 + xh of the next tile for its column sums (added one step later).
            // Both loads are issued at every step (rows clamped into the tile, values
            // past its end unused), so the loads in flight are the same on every path.
            {
                const int rx = 2 * j + 5 + xh;
                x_put(rx, xs_slot);
                xs_slot = tb[roff(rx + 8 < H ? rx + 8 : H - 1, xc)];
                if (BODY || (j >= 0 && j <= H / 2 - 1)) csum += cnext;
                const int rc = 2 * j + 2 + xh;
                const float cn = tn[roff(rc < H ? (rc > 0 ? rc : 0) : H - 1, xc)];
                cnext = ((BODY || j <= H / 2 - 2) && has_next) ? cn : 0.f;
                if (!BODY && j == H / 2 && has_next) {
                    p0 = xh ? tn[xc] : 0.f;
                    p1 = tn[roff(1 + xh, xc)];
                    p2 = tn[roff(3 + xh, xc)];
                    p3 = tn[roff(5 + xh, xc)];
                    p4 = tn[roff(7 + xh, xc)];
                    p5 = tn[roff(9 + xh, xc)];
                }
            }
            if (BODY || R < H) {
#pragma unroll
                for (int sl = 0; sl < 2; ++sl) {
                    char *row = a1base + ((R + sl) & (RX - 1)) * AROW;
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
                        const int j0 = 8 * sl + 4 * g;
                        uint2 v;
                        v.x = relu_h2(D1[j0 + 0], D1[j0 + 1]);
                        v.y = relu_h2(D1[j0 + 2], D1[j0 + 3]);
                        *reinterpret_cast<uint2 *>(row + (g ? a1w1 : a1w0)) = v;
                    }
                }
            } else if (R == H) {
                char *row = a1base + (R & (RX - 1)) * AROW;
                *reinterpret_cast<uint2 *>(row + a1w0) = make_uint2(0u, 0u);
                *reinterpret_cast<uint2 *>(row + a1w1) = make_uint2(0u, 0u);
            }
        };
        // steps -1 .. 34, four at a time: 2j mod 8 is fixed within each group
        auto steps = [&](const int jb, auto body_tag) __attribute__((always_inline)) {
            stage_rows(jb, std::integral_constant<int, 0>{}, body_tag);
            __syncthreads();
            stage_rows(jb + 1, std::integral_constant<int, 1>{}, body_tag);
            __syncthreads();
            stage_rows(jb + 2, std::integral_constant<int, 2>{}, body_tag);
            __syncthreads();
            stage_rows(jb + 3, std::integral_constant<int, 3>{}, body_tag);
            __syncthreads();
        };
        steps(-1, std::false_type{});
#pragma unroll 1
        for (int i = 1; i < H / 8; ++i) steps(4 * i - 1, std::true_type{});
        steps(H / 2 - 1, std::false_type{});
    }
}

}  // namespace

hipError_t launch_cnn_gather(const float *power, const uint8_t *labels, int S, int64_t T, int C,
                             const int32_t *tiles, int n, const CnnTrainBufs &b, hipStream_t st) {
    hipLaunchKernelGGL(cnn_gather_kernel, dim3(n * kGatherSplit), dim3(kGatherThreads), 0, st, power, labels, S, T, C,
                       tiles, b.x, b.y, b.err);
    return hipGetLastError();
}

hipError_t launch_cnn_forward(const float *params, int n, const CnnTrainBufs &b, hipStream_t st) {
    const dim3 grid(n * kCnnBlocksPerTile), blk(256);
    hipLaunchKernelGGL(cnn_conv1_kernel<0>, grid, blk, 0, st, b.x, params + kW1, params + kB1, nullptr, b.z1);
    hipLaunchKernelGGL(cnn_conv16_kernel<1>, grid, blk, 0, st, b.z1, params + kW2, params + kB2, nullptr, b.z2);
    hipLaunchKernelGGL(cnn_conv_out_kernel, grid, blk, 0, st, b.z2, params + kW3, params + kB3, b.z3);
    return hipGetLastError();
}

hipError_t launch_cnn_backward(const float *params, int n, const CnnTrainBufs &b, float *grad, float *loss,
                               hipStream_t st) {
    const int64_t npx = (int64_t)n * HW;
    const int nb = (int)std::min<int64_t>(kCnnLossBlocks, (npx + 255) / 256);
    hipLaunchKernelGGL(cnn_bce_kernel, dim3(nb), dim3(256), 0, st, b.z3, b.y, npx, b.d3, b.lpart);
    hipLaunchKernelGGL(cnn_loss_final_kernel, dim3(1), dim3(256), 0, st, b.lpart, nb, npx, loss);
    const dim3 grid(n * kCnnBlocksPerTile), blk(256);
    const int nparts = n * kCnnBlocksPerTile;
    auto reduce = [&](int E, float *out) {
        hipLaunchKernelGGL(cnn_reduce_kernel, dim3((E + kRedEntries - 1) / kRedEntries),
                           dim3(kRedEntries * kRedSlices), 0, st, b.part, nparts, E, out);
    };
    // layer 3: weights from a2 = ReLU(z2) and dz3; dz2 = (W3^T * dz3) gated by z2 > 0
    hipLaunchKernelGGL(cnn_wgrad9_kernel<-1>, grid, blk, 0, st, b.d3, b.z2, b.part);
    reduce(16 * 9 + 1, grad + kW3);
    hipLaunchKernelGGL(cnn_conv1_kernel<2>, grid, blk, 0, st, b.d3, params + kW3, nullptr, b.z2, b.d2);
    // layer 2
    hipLaunchKernelGGL(cnn_wgrad16_kernel, grid, blk, 0, st, b.z1, b.d2, b.part);
    reduce(kCnnGradEntries, grad + kW2);
    hipLaunchKernelGGL(cnn_conv16_kernel<2>, grid, blk, 0, st, b.d2, params + kW2, nullptr, b.z1, b.d1);
    // layer 1
    hipLaunchKernelGGL(cnn_wgrad9_kernel<1>, grid, blk, 0, st, b.x, b.d1, b.part);
    reduce(16 * 9 + 16, grad + kW1);
    return hipGetLastError();
}

hipError_t launch_cnn_adam(float *params, float *m, float *v, const float *grad, float lr, float beta1,
                           float beta2, float eps, float c1, float c2, hipStream_t st) {
    hipLaunchKernelGGL(cnn_adam_kernel, dim3((kCnnParams + 255) / 256), dim3(256), 0, st, params, m, v, grad,
                       kCnnParams, lr, beta1, beta2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_cnn_infer(const float *params, const void *power, bool f16, int S, int64_t T, int C,
                            float thr_logit, float guard_m, uint8_t *flags, float *logits, hipStream_t st) {
    const int n_tiles = (int)((int64_t)S * (T / H) * (C / W));
    // persistent: one workgroup per compute unit (the LDS use allows one), each
    // fetching its next tile's power while it computes the current one
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    const int grid = std::max(1, std::min(n_tiles, cus));
    auto launch = [&](auto kernel, auto *p) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(IWG), 0, st, params, p, T, C, n_tiles, thr_logit, guard_m, flags,
                           logits);
    };
    const _Float16 *p16 = static_cast<const _Float16 *>(power);
    const float *p32 = static_cast<const float *>(power);
    if (f16 && logits) launch(cnn_infer_kernel<_Float16, true>, p16);
    else if (f16) launch(cnn_infer_kernel<_Float16, false>, p16);
    else if (logits) launch(cnn_infer_kernel<float, true>, p32);
    else launch(cnn_infer_kernel<float, false>, p32);
    return hipGetLastError();
}

}  // namespace corr
