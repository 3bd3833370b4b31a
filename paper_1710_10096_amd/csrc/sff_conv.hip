// Learned feature extractor: 3x3 convolutions on BF16 NHWC tensors with FP32
// accumulation on the matrix cores (v_mfma_f32_16x16x32_bf16), used in place
// of the WHT features of the matching cost (Section 3.1).  Zero padding,
// dilation d; weights [Cout][3][3][Cin] (tap (ky, kx) reads offset
// ((ky - 1) d, (kx - 1) d)), bias FP32.
//
//   forward:  y = act(b + sum_tap W_tap x_shift)            implicit GEMM, K = 9 Cin
//   dgrad:    dx = conv(dz, W') with W'[i][ky][kx][o] = W[o][2-ky][2-kx][i],
//             dz = dy * (relu_out > 0) when the layer had a ReLU
//   wgrad:    dW_tap = sum_p dz[p] x[p + tap]^T,  db = sum_p dz[p]
//
// MFMA lane layout (16 x 16 x 32): lane l supplies row (A) / column (B) l % 16
// and eight K values for lane group l / 16; it receives C[4 (l / 16) + e][l % 16].
#include <hip/hip_bfloat16.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "sff_internal.hpp"

namespace sff {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint16_t bf16_t;  // raw bfloat16 bits in memory

__device__ __forceinline__ float bf2f(bf16_t v) { return __uint_as_float((uint32_t)v << 16); }

// Two values rounded to nearest even by the conversion instruction of gfx950
// (v_cvt_pk_bf16_f32; infinities kept, NaNs quiet), packed (lo, hi).
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){lo, hi}, v2bf));
}

constexpr int kTilePx = 64;  // output pixels per block (one row segment)
constexpr int kMaxDil = 16;  // largest dilation

// ---------------------------------------------------------------- forward --
// Block: 64 consecutive pixels of one row, 4 waves of 16 pixels, all COUT
// channels.  LDS: weights [COUT][KP] and the im2col tile [64][KP] (KP = 9 CIN
// rounded up to 32, zero padded).  `mask` (optional) multiplies each input
// value by (mask > 0), which folds a ReLU derivative into the gradient path.
template <int CIN, int COUT>
__global__ void __launch_bounds__(256) conv_fwd_kernel(const bf16_t* __restrict__ x,
                                                       const bf16_t* __restrict__ mask,
                                                       const bf16_t* __restrict__ w,
                                                       const float* __restrict__ bias,
                                                       bf16_t* __restrict__ y, int H, int W, int dil,
                                                       int relu) {
    constexpr int K = 9 * CIN, KP = (K + 31) / 32 * 32;
    __shared__ __align__(16) bf16_t wl[COUT * KP];
    __shared__ __align__(16) bf16_t col[kTilePx * KP];
    const int x0 = blockIdx.x * kTilePx, row = blockIdx.y, n = blockIdx.z;
    const size_t img = (size_t)n * H * W;
    for (int e = threadIdx.x; e < COUT * KP; e += 256) {
        const int o = e / KP, k = e - o * KP;
        wl[e] = k < K ? w[(size_t)o * K + k] : (bf16_t)0;
    }
    for (int e = threadIdx.x; e < kTilePx * KP; e += 256) {
        const int p = e / KP, k = e - p * KP;
        bf16_t v = 0;
        if (k < K) {
            const int tap = k / CIN, i = k - tap * CIN;
            const int yy = row + (tap / 3 - 1) * dil, xx = x0 + p + (tap % 3 - 1) * dil;
            if (yy >= 0 && yy < H && xx >= 0 && xx < W && x0 + p < W) {
                const size_t o = (img + (size_t)yy * W + xx) * CIN + i;
                v = x[o];
                if (mask && !(bf2f(mask[o]) > 0.f)) v = 0;
            }
        }
        col[e] = v;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ln = lane & 15, g = lane >> 4;
    v4f acc[COUT / 16];
#pragma unroll
    for (int t = 0; t < COUT / 16; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
    const bf16_t* bcol = col + (wv * 16 + ln) * KP + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KP / 32; ++ks) {
        const v8bf bv = *reinterpret_cast<const v8bf*>(bcol + ks * 32);
#pragma unroll
        for (int t = 0; t < COUT / 16; ++t) {
            const v8bf av = *reinterpret_cast<const v8bf*>(wl + (t * 16 + ln) * KP + ks * 32 + 8 * g);
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc[t], 0, 0, 0);
        }
    }
    const int px = x0 + wv * 16 + ln;
    if (px >= W) return;
    bf16_t* out = y + (img + (size_t)row * W + px) * COUT;
#pragma unroll
    for (int t = 0; t < COUT / 16; ++t) {
        uint32_t packed[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float v0 = acc[t][2 * h] + (bias ? bias[t * 16 + 4 * g + 2 * h] : 0.f);
            float v1 = acc[t][2 * h + 1] + (bias ? bias[t * 16 + 4 * g + 2 * h + 1] : 0.f);
            if (relu) {
                v0 = fmaxf(v0, 0.f);
                v1 = fmaxf(v1, 0.f);
            }
            packed[h] = f2bf2(v0, v1);
        }
        *reinterpret_cast<uint2*>(out + t * 16 + 4 * g) = make_uint2(packed[0], packed[1]);
    }
}

constexpr int kTile32 = 256;
constexpr int kStageW = kTile32 + 2 * kMaxDil;
constexpr int kRows32 = 4;  // output rows per block of the first layer (the weight fragments are loaded once)

// Raw buffer descriptor of one tensor row (wave-uniform base): a load at an
// offset at or past `bytes` returns zeros without a memory access, which is
// the zero padding.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const bf16_t* p, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), (short)0,
                                             (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}
constexpr int kOutside = 0x7FFFFFF0;  // offset past every row

typedef short v2s __attribute__((ext_vector_type(2)));
typedef uint32_t v4u8a __attribute__((ext_vector_type(4), aligned(8)));

// v with every bf16 whose mask value is not > 0 (zero, negative, NaN) cleared.
__device__ __forceinline__ uint4 relu_masked(uint4 v, uint4 m) {
    const uint32_t mw[4] = {m.x, m.y, m.z, m.w};
    uint32_t vw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        // the sign of -b & ~b & ~(inf - b) is set for b > 0 that is no NaN
        const v2s b = __builtin_bit_cast(v2s, mw[h]);
        const uint32_t neg = __builtin_bit_cast(uint32_t, (v2s)(-b));
        const uint32_t nan = __builtin_bit_cast(uint32_t, (v2s)((v2s){0x7F80, 0x7F80} - b));
        vw[h] &= __builtin_bit_cast(uint32_t, (v2s)(__builtin_bit_cast(v2s, neg & ~(mw[h] | nan)) >> 15));
    }
    return make_uint4(vw[0], vw[1], vw[2], vw[3]);
}

// A lane's 8 output channels (two tiles of 4): bias, ReLU, rounded to BF16.
__device__ __forceinline__ v4u8a pack8(const v4f (&acc)[2], const float (&bz)[2][4], int relu) {
    v4u8a o;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float v0 = acc[t][2 * h] + bz[t][2 * h];
            float v1 = acc[t][2 * h + 1] + bz[t][2 * h + 1];
            if (relu) {
                v0 = fmaxf(v0, 0.f);
                v1 = fmaxf(v1, 0.f);
            }
            o[2 * t + h] = f2bf2(v0, v1);
        }
    return o;
}

// A lane's 8 channels (8 g .. 8 g + 7 of pixel ln, BF16) as int16 descriptor values
// rint(scale f / |f|), with the operations of quantise_kernel in its order: the
// sum of squares runs through the pixel's four lanes, channel by channel.  Must be
// called by all lanes of the wave.
__device__ __forceinline__ v4u8a quantise8(const v4u8a& o, int ln, int g, float scale) {
    float v[8];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        v[2 * h] = __uint_as_float(o[h] << 16);
        v[2 * h + 1] = __uint_as_float(o[h] & 0xFFFF0000u);
    }
    float ss = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        float t = s == 0 ? 0.f : __shfl(ss, ln + 16 * (s - 1));
#pragma unroll
        for (int c = 0; c < 8; ++c) t = fmaf(v[c], v[c], t);
        ss = g == s ? t : ss;
    }
    const float inv = scale / fmaxf(sqrtf(__shfl(ss, ln + 48)), 1e-12f);
    v4u8a q;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int a = (int)rintf(v[2 * h] * inv), b = (int)rintf(v[2 * h + 1] * inv);
        q[h] = (uint32_t)(uint16_t)(int16_t)a | ((uint32_t)(uint16_t)(int16_t)b << 16);
    }
    return q;
}

// The same convolution for Cin = Cout = 32, with neither an im2col tile nor
// LDS: with K ordered (tap, channel), the 32 K values of one MFMA step are the
// 32 channels of one input pixel, so lane (pixel l % 16, group l / 16) needs 16
// contiguous bytes of it and a wave's operand for one tap is 1 KB of
// consecutive memory.  A wave takes a column of 16 pixels and walks down R
// rows: a row's three operands (kx = 0..2) stay in registers for the three
// output rows that read them, so each output row costs three loads, two rows
// ahead of their use.  With dilation d the rows of one residue mod d are such a
// column of their own (row k of phase f is image row f + d k).  The weight rows
// are dealt to the two output tiles so that a lane ends up with 8 consecutive
// channels: one 16-byte store per pixel and lane, 1 KB per wave.  Every output is
// the MFMAs of conv_fwd_kernel<32, 32> in the same order on the same values, so
// the results are identical.  x, w (and mask) must be 16-byte aligned.
// Bound: HBM (128 B per pixel, 192 with the mask): on four 1242 x 375 images
// 49 us (4.9 TB/s, the rate of a large copy) and 88 us with the mask (357 MB,
// past the 256 MB of the Infinity Cache), where rows staged in LDS for each of
// the three output rows that read them took 167 and 190 us.
// RECORDS: the network's last layer written as descriptor records in place of
// BF16 features (on four 1024 x 436 images 58 us in place of 50 and 48 us with a
// pass of its own over the stored features).
template <bool MASK, bool RECORDS>
__global__ void __launch_bounds__(256, 2) conv32_column_kernel(const bf16_t* __restrict__ x,
                                                            const bf16_t* __restrict__ mask,
                                                            const bf16_t* __restrict__ w,
                                                            const float* __restrict__ bias,
                                                            bf16_t* __restrict__ y, int H, int W, int dil,
                                                            int relu, int R, float scale) {
    constexpr int kAhead = 2, NR = 3 + kAhead;  // rows in flight past the window; rows in registers
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ln = lane & 15, g = lane >> 4;
    const int c0 = __builtin_amdgcn_readfirstlane(blockIdx.x * 64 + wv * 16);
    if (c0 >= W) return;
    const int p = c0 + ln;
    const int phase = blockIdx.y % dil, k0 = blockIdx.y / dil * R;
    const int nk = min(R, (H - phase + dil - 1) / dil - k0);
    if (nk <= 0) return;
    const size_t img = (size_t)blockIdx.z * H * W;
    int off[3];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
        const int xx = p + (kx - 1) * dil;
        off[kx] = xx >= 0 && xx < W ? xx * 64 + 16 * g : kOutside;
    }
    // tile t, row r holds output channel 8 (r / 4) + 4 t + r % 4
    v8bf a[2][9];
    float bz[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int o = 8 * (ln >> 2) + 4 * t + (ln & 3);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
            a[t][tap] = *reinterpret_cast<const v8bf*>(w + ((size_t)o * 9 + tap) * 32 + 8 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) bz[t][e] = bias ? bias[8 * g + 4 * t + e] : 0.f;
    }
    uint4 f[NR][3], fm[NR][3];  // row k0 - 1 + i in slot i % NR
    auto load_row = [&](int i, uint4 (&v)[3], uint4 (&m)[3]) {
        const int yy = phase + dil * (k0 - 1 + i);
        const bool in = yy >= 0 && yy < H && i <= nk + 1;
        const size_t row = (img + (size_t)(in ? yy : 0) * W) * 32;
        const __amdgpu_buffer_rsrc_t rx = row_rsrc(x + row, in ? (uint32_t)W * 64u : 0u);
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
            v[kx] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rx, off[kx], 0, 0));
        if constexpr (MASK) {
            const __amdgpu_buffer_rsrc_t rm = row_rsrc(mask + row, in ? (uint32_t)W * 64u : 0u);
#pragma unroll
            for (int kx = 0; kx < 3; ++kx)
                m[kx] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rm, off[kx], 0, 0));
        }
    };
    auto ready = [&](uint4 (&v)[3], const uint4 (&m)[3]) {
        if constexpr (MASK) {
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) v[kx] = relu_masked(v[kx], m[kx]);
        }
    };
#pragma unroll
    for (int i = 0; i < NR - 1; ++i) load_row(i, f[i], fm[i]);
    ready(f[0], fm[0]);
    ready(f[1], fm[1]);
    for (int j0 = 0; j0 < nk; j0 += NR) {
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int j = j0 + u;
            if (j >= nk) return;
            load_row(j + NR - 1, f[(u + NR - 1) % NR], fm[(u + NR - 1) % NR]);
            ready(f[(u + 2) % NR], fm[(u + 2) % NR]);
            v4f acc[2] = {v4f{0.f, 0.f, 0.f, 0.f}, v4f{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                const v8bf bv = __builtin_bit_cast(v8bf, f[(u + tap / 3) % NR][tap % 3]);
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][tap], bv, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1][tap], bv, acc[1], 0, 0, 0);
            }
            const int yy = phase + dil * (k0 + j);
            v4u8a o = pack8(acc, bz, relu);
            if constexpr (RECORDS) o = quantise8(o, ln, g, scale);
            if (p < W) *reinterpret_cast<v4u8a*>(y + (img + (size_t)yy * W + p) * 32 + 8 * g) = o;
        }
    }
}

// The first layer (Cin = 3: K = 27, one MFMA step) without an im2col tile:
// the input rows that the 4 output rows of a 256-pixel tile read are staged in
// LDS together (6 with dilation 1, else 12), so their loads are in flight at
// once and the block waits at one barrier, and each lane reads its 8 (tap,
// channel) K values straight from them; the two weight fragments stay in
// registers, their rows dealt as in conv32_column_kernel so that a lane stores 16
// bytes.  Same operands as conv_fwd_kernel<3, 32>, so the same results.
// Bound: the stores (64 B per pixel; 24 us on four 1242 x 375 images at the
// rate of a large copy): 35 us there, against 58 us with three rows staged per
// output row between two barriers.
__global__ void __launch_bounds__(256) conv3_fwd_kernel(const bf16_t* __restrict__ x,
                                                        const bf16_t* __restrict__ w,
                                                        const float* __restrict__ bias,
                                                        bf16_t* __restrict__ y, int H, int W, int dil,
                                                        int relu) {
    __shared__ bf16_t rows[3 * kRows32][kStageW * 3];
    const int x0 = blockIdx.x * kTile32, r0 = blockIdx.y * kRows32, n = blockIdx.z;
    const size_t img = (size_t)n * H * W;
    const int nx3 = (kTile32 + 2 * dil) * 3;  // staged values per row
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ln = lane & 15, g = lane >> 4;
    // slot of output row rr's input row ky: rr + ky with dilation 1 (shared), else 3 rr + ky
    const int per = dil == 1 ? 1 : 3, ns = dil == 1 ? kRows32 + 2 : 3 * kRows32;
    for (int s = 0; s < ns; ++s) {
        const int yy = dil == 1 ? r0 + s - 1 : r0 + s / 3 + (s % 3 - 1) * dil;
        const bool in = yy >= 0 && yy < H;
        const __amdgpu_buffer_rsrc_t rs = row_rsrc(x + (img + (size_t)(in ? yy : 0) * W) * 3, in ? (uint32_t)W * 6u : 0u);
        for (int e = threadIdx.x; e < nx3; e += 256) {
            const int j = (x0 - dil) * 3 + e;  // value of the row
            rows[s][e] = (bf16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, j >= 0 ? 2 * j : kOutside, 0, 0);
        }
    }
    v8bf a[2];
    float bz[2][4];
    int koff[8];  // LDS offset of K value 8 g + e relative to the lane's pixel (-1: zero padding)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) bz[t][e] = bias ? bias[8 * g + 4 * t + e] : 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int k = 8 * g + e;
#pragma unroll
        for (int t = 0; t < 2; ++t)
            a[t][e] = __builtin_bit_cast(
                __bf16, k < 27 ? w[(size_t)(8 * (ln >> 2) + 4 * t + (ln & 3)) * 27 + k] : (bf16_t)0);
        const int tap = k / 3, ci = k - 3 * tap, ky = tap / 3, kx = tap - 3 * ky;
        koff[e] = k < 27 ? ky * kStageW * 3 + kx * dil * 3 + ci : -1;
    }
    __syncthreads();
    for (int rr = 0; rr < kRows32; ++rr) {
        const int row = r0 + rr;
        if (row >= H) break;
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
            const int p = wv * 64 + grp * 16 + ln;
            const bf16_t* src = &rows[per * rr][p * 3];
            v8bf bv;
#pragma unroll
            for (int e = 0; e < 8; ++e) bv[e] = __builtin_bit_cast(__bf16, koff[e] >= 0 ? src[koff[e]] : (bf16_t)0);
            v4f acc[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], bv, v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            const int px = x0 + p;
            if (px < W) *reinterpret_cast<v4u8a*>(y + (img + (size_t)row * W + px) * 32 + 8 * g) = pack8(acc, bz, relu);
        }
    }
}

// W'[i][ky][kx][o] = W[o][2 - ky][2 - kx][i]
__global__ void flip_weights_kernel(const bf16_t* __restrict__ w, bf16_t* __restrict__ wt, int cin,
                                    int cout) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= cin * 9 * cout) return;
    const int i = e / (9 * cout), r = e - i * 9 * cout;
    const int tap = r / cout, o = r - tap * cout;
    wt[e] = w[((size_t)o * 9 + (8 - tap)) * cin + i];
}

// ------------------------------------------------------------ weight grad --
// dW[o][tap][i] = sum over pixels: the K dimension of the MFMAs is 32
// consecutive pixels of one row, so both operands are needed transposed
// (channel-major), while memory holds the channels of a pixel together.  A wave
// takes a column of 32 pixels and walks down R rows (with dilation d: rows of
// one residue mod d).  Per row it puts the 32 + 2 d input pixels and the 32
// pixels of dz = dy (masked by the ReLU) into its own LDS slice as they come
// (16-byte writes) and reads them back through the transposing LDS load
// (ds_read_b64_tr_b16: 16 lanes read 4 pixels x 16 channels and lane i gets
// channel i of the 4 pixels).  The operand of an input row serves the three
// kernel rows at once: dz of the three output rows around it is kept in
// registers, so a row is staged and read once (16 transposing reads for 36
// MFMAs), and the whole 32 x 288 gradient is accumulated in the wave's
// registers.  The waves of a block are added in order at the end, the blocks by
// wgrad_reduce_kernel.  For Cin = 3 the staged row holds the 9 (kx, channel)
// values of each pixel, padded to 16.  The bias gradient is dz times a matrix of
// ones.  Global loads run one row ahead.
// Bound: HBM (192 B per pixel with the mask: 357 MB on four 1242 x 375 images,
// 73 us at the rate of a large copy).  There, with dy and its mask one tensor
// (238 MB): 56 us for Cin = 32 and 37 us for Cin = 3, against 328 and 270 us for
// blocks that scattered every row transposed into LDS in 2-byte writes, three
// times over.
constexpr int kWgPx = 32, kWgWaves = 8;
constexpr int kWgXPx = kWgPx + 2 * kMaxDil;                  // staged input pixels, at most
constexpr int kWgSlice = kWgXPx * 32 + kWgPx * 32;           // bf16 of one wave: input row, dz row
constexpr int kWgRedTiles = 6;                               // accumulator tiles summed at a time
template <int CIN>
constexpr int kWgTiles = CIN == 32 ? 36 : 6;  // (ot, it, tap) or (ot, ky) tiles of 16 x 16

typedef short v4s __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16_t* lds_bf16;

// 8 K values (pixels px .. px + 7 of the lane's group) of channel c0 + l % 16
// from a staged row of `stride` bf16 per pixel.
__device__ __forceinline__ v8bf read_transposed(lds_bf16 row, int px, int c0, int stride) {
    const int i = threadIdx.x & 15;
    lds_bf16 p = row + (px + (i >> 2)) * stride + c0 + 4 * (i & 3);
    struct {
        v4s lo, hi;
    } r;
    r.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)p);
    r.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)(p + 4 * stride));
    return __builtin_bit_cast(v8bf, r);
}

// 8 bf16 at byte offset off of a row: one 16-byte load, or eight 2-byte ones
// where the tensor is not 16-byte aligned.
template <bool VEC>
__device__ __forceinline__ uint4 load_piece(__amdgpu_buffer_rsrc_t rs, int off) {
    if constexpr (VEC) {
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
    } else {
        uint32_t w[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b16(rs, off + 4 * h, 0, 0);
            const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b16(rs, off + 4 * h + 2, 0, 0);
            w[h] = (lo & 0xFFFFu) | (hi << 16);
        }
        return make_uint4(w[0], w[1], w[2], w[3]);
    }
}

template <int CIN, bool VEC>
__global__ void __launch_bounds__(64 * kWgWaves) wgrad_column_kernel(const bf16_t* __restrict__ x,
                                                                     const bf16_t* __restrict__ dy,
                                                                     const bf16_t* __restrict__ mask,
                                                                     float* __restrict__ part, int H, int W, int dil,
                                                                     int R, int strips, int chunks, int units) {
    constexpr int NT = kWgTiles<CIN>;
    constexpr int kRed = kWgWaves * kWgRedTiles * 256;  // floats
    constexpr int kStage = kWgWaves * kWgSlice / 2;     // floats
    __shared__ __align__(16) float lds[kRed > kStage ? kRed : kStage];
    const int lane = threadIdx.x & 63, wv = wave_id();
    const int g = lane >> 4;
    v4f acc[NT], accb[2];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = v4f{0.f, 0.f, 0.f, 0.f};
    accb[0] = accb[1] = v4f{0.f, 0.f, 0.f, 0.f};
    for (int unit = blockIdx.x * kWgWaves + wv; unit < units; unit += gridDim.x * kWgWaves) {
        const int strip = unit % strips, c = unit / strips, n = c / chunks, cy = c % chunks;
        const int phase = cy % dil, k0 = cy / dil * R, x0 = strip * kWgPx;
        const int nk = min(R, (H - phase + dil - 1) / dil - k0);
        const size_t img = (size_t)n * H * W;
        lds_bf16 xs = (lds_bf16)(lds) + wv * kWgSlice, zs = xs + kWgXPx * 32;
        constexpr int XP = CIN == 32 ? 4 : 1;  // 16-byte pieces of the input row per lane
        // byte offsets of this lane's pieces in a row of x and of dy
        int xo[CIN == 32 ? XP : 8], zo[2];
        if constexpr (CIN == 32) {
#pragma unroll
            for (int k = 0; k < XP; ++k) {
                const int e = 64 * k + lane, px = e >> 2, xx = x0 - dil + px;
                xo[k] = px < kWgPx + 2 * dil && xx >= 0 && xx < W ? xx * 64 + 16 * (e & 3) : kOutside;
            }
        } else {  // pixel lane / 2, (kx, channel) values 8 (lane & 1) .. + 7
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int e = 8 * (lane & 1) + k, kx = e / 3, xx = x0 + (lane >> 1) + (kx - 1) * dil;
                xo[k] = e < 9 && xx >= 0 && xx < W ? (xx * 3 + e - 3 * kx) * 2 : kOutside;
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int e = 64 * k + lane, xx = x0 + (e >> 2);
            zo[k] = xx < W ? xx * 64 + 16 * (e & 3) : kOutside;
        }
        uint32_t keep[4];  // the K values (pixels 8 g + e) inside the image
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int px = x0 + 8 * g + 2 * h;
            keep[h] = (px < W ? 0xFFFFu : 0u) | (px + 1 < W ? 0xFFFF0000u : 0u);
        }
        uint4 xv[XP], zv[2], mv[2];
        auto load_x = [&](int i) {  // input row i (the window's row of output row i)
            const int yy = phase + dil * (k0 + i);
            const bool in = yy >= 0 && yy < H && i <= nk;
            const __amdgpu_buffer_rsrc_t rs =
                row_rsrc(x + (img + (size_t)(in ? yy : 0) * W) * CIN, in ? (uint32_t)W * 2u * CIN : 0u);
            if constexpr (CIN == 32) {
#pragma unroll
                for (int k = 0; k < XP; ++k)
                    if (k < 3 || dil > 8) xv[k] = load_piece<VEC>(rs, xo[k]);
            } else {
                uint32_t w[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) w[k] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, xo[k], 0, 0) & 0xFFFFu;
                xv[0] = make_uint4(w[0] | w[1] << 16, w[2] | w[3] << 16, w[4] | w[5] << 16, w[6] | w[7] << 16);
            }
        };
        auto load_z = [&](int i) {  // dz row i, zero outside the chunk
            const bool in = i >= 0 && i < nk;
            const size_t row = (img + (size_t)(in ? phase + dil * (k0 + i) : 0) * W) * 32;
            const __amdgpu_buffer_rsrc_t rs = row_rsrc(dy + row, in ? (uint32_t)W * 64u : 0u);
#pragma unroll
            for (int k = 0; k < 2; ++k) zv[k] = load_piece<VEC>(rs, zo[k]);
            if (mask) {
                const __amdgpu_buffer_rsrc_t rm = row_rsrc(mask + row, in ? (uint32_t)W * 64u : 0u);
#pragma unroll
                for (int k = 0; k < 2; ++k) mv[k] = load_piece<VEC>(rm, zo[k]);
            }
        };
        v8bf ones;
#pragma unroll
        for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
        v8bf dz[3][2];  // dz rows i - 1, i, i + 1 at step i
#pragma unroll
        for (int r = 0; r < 3; ++r) dz[r][0] = dz[r][1] = (v8bf)(__bf16)0.0f;
        load_x(-1);
        load_z(0);
        for (int i = -1; i <= nk; ++i) {
            // the wave's slice is its own; its LDS operations run in order
            auto put = [&](lds_bf16 p, uint4 v) { *reinterpret_cast<__attribute__((address_space(3))) v4u*>(p) = __builtin_bit_cast(v4u, v); };
            if constexpr (CIN == 32) {
#pragma unroll
                for (int k = 0; k < XP; ++k)
                    if (k < 3 || dil > 8) put(xs + (64 * k + lane) * 8, xv[k]);
            } else {
                put(xs + lane * 8, xv[0]);
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) put(zs + (64 * k + lane) * 8, mask ? relu_masked(zv[k], mv[k]) : zv[k]);
            load_x(i + 1);
            load_z(i + 2);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                dz[0][t] = dz[1][t];
                dz[1][t] = dz[2][t];
                dz[2][t] = read_transposed(zs, 8 * g, 16 * t, 32);
                accb[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dz[2][t], ones, accb[t], 0, 0, 0);
            }
            // input row i meets output row i + 1 - ky at kernel row ky.  Past the ends of
            // the chunk and the image's columns there is no output: the zeros in its place
            // must not meet an infinite x (NaN), so x is cleared there too.  Always, with
            // masks: 56 us where 50 without; a branch around them takes 60 and spills
            auto operand = [&](const v8bf& b, int ky) {
                const uint32_t row = i + 1 - ky >= 0 && i + 1 - ky < nk ? ~0u : 0u;
                v4u v = __builtin_bit_cast(v4u, b);
#pragma unroll
                for (int h = 0; h < 4; ++h) v[h] &= keep[h] & row;
                return __builtin_bit_cast(v8bf, v);
            };
            if constexpr (CIN == 32) {
#pragma unroll
                for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                    for (int it = 0; it < 2; ++it) {
                        const v8bf b = read_transposed(xs, 8 * g + kx * dil, 16 * it, 32);
#pragma unroll
                        for (int ky = 0; ky < 3; ++ky) {
                            const v8bf bk = operand(b, ky);
#pragma unroll
                            for (int ot = 0; ot < 2; ++ot) {
                                v4f& q = acc[(ot * 2 + it) * 9 + 3 * ky + kx];
                                q = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dz[2 - ky][ot], bk, q, 0, 0, 0);
                            }
                        }
                    }
            } else {
                const v8bf b = read_transposed(xs, 8 * g, 0, 16);
#pragma unroll
                for (int ky = 0; ky < 3; ++ky) {
                    const v8bf bk = operand(b, ky);
#pragma unroll
                    for (int ot = 0; ot < 2; ++ot)
                        acc[ot * 3 + ky] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dz[2 - ky][ot], bk, acc[ot * 3 + ky], 0, 0, 0);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    // sums of the block's waves, in wave order: kWgRedTiles tiles at a time;
    // partial layout [block][NT + 2 tiles][element][lane] (the last two: dz times ones)
    float* out = part + (size_t)blockIdx.x * (NT + 2) * 256;
#pragma unroll
    for (int t0 = 0; t0 < NT + 2; t0 += kWgRedTiles) {
        constexpr int N = kWgRedTiles;
        __syncthreads();
#pragma unroll
        for (int t = 0; t < N; ++t)
            if (t0 + t < NT + 2) {
                const v4f v = t0 + t < NT ? acc[t0 + t < NT ? t0 + t : 0] : accb[t0 + t < NT ? 0 : t0 + t - NT];
#pragma unroll
                for (int e = 0; e < 4; ++e) lds[(wv * N + t) * 256 + e * 64 + lane] = v[e];
            }
        __syncthreads();
        const int cnt = min(N, NT + 2 - t0) * 256;
        for (int e = threadIdx.x; e < cnt; e += 64 * kWgWaves) {
            float sum = lds[e];
#pragma unroll
            for (int k = 1; k < kWgWaves; ++k) sum += lds[k * N * 256 + e];
            out[t0 * 256 + e] = sum;
        }
    }
}

// Sum of the per-block partials, in a fixed order: 32 accumulator elements per
// block, 8 threads per element; thread s sums blocks s, s + 8, s + 16, ... with
// four independent accumulators (their loads in flight together), and the 8
// segment sums are added in order through LDS.
constexpr int kRedOut = 32, kRedSeg = 8;

__global__ void __launch_bounds__(256) wgrad_reduce_kernel(const float* __restrict__ part, float* __restrict__ dw,
                                                           float* __restrict__ db, int nblk, int cin) {
    __shared__ float seg[kRedSeg][kRedOut];
    const int lo = threadIdx.x % kRedOut, sg = threadIdx.x / kRedOut;
    const int e = blockIdx.x * kRedOut + lo;  // tile, element, lane
    const int nt = cin == 32 ? kWgTiles<32> : kWgTiles<3>;
    const size_t stride = (size_t)(nt + 2) * 256;
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
    const float* src = part + e;
    int b = sg;
    for (; b + 3 * kRedSeg < nblk; b += 4 * kRedSeg) {
        a0 += src[(size_t)b * stride];
        a1 += src[(size_t)(b + kRedSeg) * stride];
        a2 += src[(size_t)(b + 2 * kRedSeg) * stride];
        a3 += src[(size_t)(b + 3 * kRedSeg) * stride];
    }
    for (; b < nblk; b += kRedSeg) a0 += src[(size_t)b * stride];
    seg[sg][lo] = (a0 + a1) + (a2 + a3);
    __syncthreads();
    if (sg != 0) return;
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < kRedSeg; ++k) t += seg[k][lo];
    const int tile = e >> 8, r = 4 * ((e & 63) >> 4) + ((e >> 6) & 3), col = e & 15;
    if (tile >= nt) {
        if (col == 0) db[16 * (tile - nt) + r] = t;
    } else if (cin == 32) {  // tile (ot 2 + it) 9 + tap
        const int oi = tile / 9, tap = tile - 9 * oi;
        dw[((size_t)((oi >> 1) * 16 + r) * 9 + tap) * 32 + (oi & 1) * 16 + col] = t;
    } else if (col < 9) {  // tile ot 3 + ky, column kx 3 + channel
        const int ot = tile / 3, ky = tile - 3 * ot;
        dw[(size_t)(ot * 16 + r) * 27 + ky * 9 + col] = t;
    }
}

// Rows per wave of the weight gradient: at most 2048 waves, the most that are
// resident at once (one block of 8 per CU), so no wave starts late; at least 8
// rows, so that the two halo rows stay a small share of small calls.  Where
// columns alone are more than 2048, a wave takes several, one after another.
struct WgradSplit {
    int strips, R, chunks, units, blocks;
};
WgradSplit wgrad_split(int n, int H, int W, int dil) {
    WgradSplit s;
    s.strips = (W + kWgPx - 1) / kWgPx;
    const size_t rows = (size_t)s.strips * n * H;
    const int hp = (H + dil - 1) / dil;
    s.R = (int)std::min<size_t>(std::max<size_t>((rows + 2047) / 2048, 8), (size_t)hp);
    do {
        s.chunks = dil * ((hp + s.R - 1) / s.R);
        s.units = n * s.strips * s.chunks;
    } while (s.units > 2048 && s.R++ < hp);
    s.blocks = std::min((s.units + kWgWaves - 1) / kWgWaves, 256);
    return s;
}

bool conv_shape_ok(int n, int H, int W, int cin, int cout, int dil) {
    if (n < 1 || H < 1 || W < 1 || H > 16384 || W > 16384 || n > 65535) return false;
    if (dil < 1 || dil > kMaxDil) return false;
    return (cin == 3 || cin == 32) && cout == 32;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// conv32_column_kernel and the 32-channel weight gradient read x, w (and mask, dy)
// in 16-byte pieces; unaligned tensors and SFF_CONV_IM2COL=1 (testing and
// timing) take the element-wise kernels (the im2col forward, element-wise
// staging of the gradient tiles), which give the same results.
bool staged_conv_enabled() {
    const char* e = std::getenv("SFF_CONV_IM2COL");
    return !(e && std::strcmp(e, "1") == 0);
}

// ------------------------------------------------------- fused 4 layers --
// The whole network (3 -> 32 -> 32 -> 32 -> 32, ReLU after the first three,
// dilation 1) for one kFusedY x kFusedX output tile per block, the layers'
// activations kept in LDS: layer l is computed on the tile grown by 3 - l
// pixels on every side (its inputs' halo), from the LDS region the layer
// before it left there; only the three-channel input is read from and the
// 32-channel output written to HBM.  Positions outside the image are stored
// as zeros (the zero padding the next layer reads), every layer's output is
// rounded to BF16 as the per-layer kernels store it, and each output element
// is the same MFMAs in the same order on the same values as conv3_fwd_kernel
// and conv32_column_kernel, so the results are identical (tested).
// Tiles are 26 wide so that every layer's region is at most two 16-pixel
// groups wide (32, 30, 28 and 26 pixels: 15 % of the computed groups fall
// outside a region, against 22 % for 64-wide tiles) and 24 tall, the most that
// fits 150 KB of LDS with that width (four KITTI-size images: 0.35 ms with
// 64 x 8 tiles, 0.31 with 58 x 10, 0.28 with 42 x 15, 0.27 with 26 x 24).
constexpr int kFusedX = 26, kFusedY = 24;
constexpr int kFIn[2] = {kFusedY + 8, kFusedX + 8};   // input region (3 channels, packed)
constexpr int kF1[2] = {kFusedY + 6, kFusedX + 6};    // layer-1 output (and layer 3's, in place later)
constexpr int kF2[2] = {kFusedY + 4, kFusedX + 4};    // layer-2 output
constexpr int kFPx = 40;                              // bf16 per staged pixel (32 used): 80-byte stride

// This lane's biases: output channels 16 t + 4 (l / 16) + e (zero without bias).
__device__ __forceinline__ void fused_bias(const float* __restrict__ bias, float (&bz)[2][4]) {
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) bz[t][e] = bias ? bias[t * 16 + 4 * g + e] : 0.f;
}

// Round acc + bias, ReLU, to BF16 pairs for output channels 16 t + 4 g .. + 3.
__device__ __forceinline__ uint2 fused_pack(const v4f& acc, const float (&bz)[4], bool relu) {
    uint32_t packed[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float v0 = acc[2 * h] + bz[2 * h];
        float v1 = acc[2 * h + 1] + bz[2 * h + 1];
        if (relu) {
            v0 = fmaxf(v0, 0.f);
            v1 = fmaxf(v1, 0.f);
        }
        packed[h] = f2bf2(v0, v1);
    }
    return make_uint2(packed[0], packed[1]);
}

// The 18 weight fragments of a 32 -> 32 layer for this lane: output channel
// 16 t + l % 16, tap, input channels 8 (l / 16) .. + 7.
__device__ __forceinline__ void fused_weights(const bf16_t* __restrict__ w, v8bf (&a)[2][9]) {
    const int lane = threadIdx.x & 63, ln = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
            a[t][tap] = *reinterpret_cast<const v8bf*>(w + ((size_t)(t * 16 + ln) * 9 + tap) * 32 + 8 * g);
}

// One 32 -> 32 layer from LDS region `in` (OH + 2) x (OW + 2) to region `out`
// OH x OW (or, for the last layer, to y), the region's pixel (0, 0) at image
// (oy, ox).  Work items are (row, 16-pixel group), dealt to the 8 waves, two
// at a time per wave (four independent accumulator chains in flight).
template <int OH, int OW, bool LAST>
__device__ __forceinline__ void fused_layer32(const bf16_t* in, bf16_t* out, const v8bf (&a)[2][9],
                                              const float (&bz)[2][4], bool relu, int oy, int ox,
                                              int H, int W, bf16_t* __restrict__ y, size_t img) {
    constexpr int IW = OW + 2, NG = (OW + 15) / 16, NI = OH * NG;
    typedef const v8bf __attribute__((address_space(3)))* lds_v8;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ln = lane & 15, g = lane >> 4;
    for (int i0 = wv; i0 < NI; i0 += 16) {
        int r[2], p[2];
        lds_v8 src[2];
        v4f acc[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int item = min(i0 + 8 * h, NI - 1);  // a missing second item repeats the last
            r[h] = item / NG;
            p[h] = (item - r[h] * NG) * 16 + ln;
            const int pr = min(p[h], OW - 1);  // lanes past the row read a valid pixel
            // 32-bit LDS addresses; the taps are constant offsets from the lane's first one
            src[h] = (lds_v8)((const __attribute__((address_space(3))) bf16_t*)in + (r[h] * IW + pr) * kFPx + 8 * g);
            acc[h][0] = v4f{0.f, 0.f, 0.f, 0.f};
            acc[h][1] = v4f{0.f, 0.f, 0.f, 0.f};
        }
        // the B operands of tap t + kAhead are read from LDS while tap t's
        // products run (a ring of kAhead + 1 taps), so the LDS latency is not
        // waited on at every tap
        constexpr int kAhead = 3;
        v8bf bv[kAhead + 1][2];
        auto read_tap = [&](int tap, v8bf (&b)[2]) {
            const int ky = tap / 3, kx = tap - 3 * ky;
#pragma unroll
            for (int h = 0; h < 2; ++h) b[h] = src[h][(ky * IW + kx) * kFPx / 8];
        };
#pragma unroll
        for (int tap = 0; tap < kAhead; ++tap) read_tap(tap, bv[tap]);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            if (tap + kAhead < 9) read_tap(tap + kAhead, bv[(tap + kAhead) % (kAhead + 1)]);
            __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of the products
            const v8bf (&b)[2] = bv[tap % (kAhead + 1)];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                acc[h][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][tap], b[h], acc[h][0], 0, 0, 0);
                acc[h][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1][tap], b[h], acc[h][1], 0, 0, 0);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (p[h] >= OW || (h == 1 && i0 + 8 >= NI)) continue;
            const int iy = oy + r[h], ix = ox + p[h];
            const bool inside = iy >= 0 && iy < H && ix >= 0 && ix < W;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint2 v = inside ? fused_pack(acc[h][t], bz[t], relu) : make_uint2(0u, 0u);
                if constexpr (LAST) {
                    if (inside) *reinterpret_cast<uint2*>(y + (img + (size_t)iy * W + ix) * 32 + t * 16 + 4 * g) = v;
                } else {
                    *reinterpret_cast<uint2*>(out + (r[h] * OW + p[h]) * kFPx + t * 16 + 4 * g) = v;
                }
            }
        }
    }
}

__global__ void __launch_bounds__(512) featnet_fwd_kernel(const bf16_t* __restrict__ x,
                                                          const bf16_t* __restrict__ w0, const float* __restrict__ b0,
                                                          const bf16_t* __restrict__ w1, const float* __restrict__ b1,
                                                          const bf16_t* __restrict__ w2, const float* __restrict__ b2,
                                                          const bf16_t* __restrict__ w3, const float* __restrict__ b3,
                                                          bf16_t* __restrict__ y, int H, int W) {
    __shared__ __align__(16) bf16_t xin[kFIn[0] * kFIn[1] * 3];
    __shared__ __align__(16) bf16_t bufA[kF1[0] * kF1[1] * kFPx];
    __shared__ __align__(16) bf16_t bufB[kF2[0] * kF2[1] * kFPx];
    const int x0 = blockIdx.x * kFusedX, y0 = blockIdx.y * kFusedY, n = blockIdx.z;
    const size_t img = (size_t)n * H * W;
    v8bf wa[2][9];
    float bz0[2][4], bz[2][4];
    fused_weights(w1, wa);  // layer 2's, in flight during the staging and layer 1
    fused_bias(b0, bz0);
    fused_bias(b1, bz);
    // input region: image rows y0 - 4 .., columns x0 - 4 .., zero outside
    for (int e = threadIdx.x; e < kFIn[0] * kFIn[1] * 3; e += 512) {
        const int px = e / 3, ci = e - 3 * px, r = px / kFIn[1], c = px - r * kFIn[1];
        const int iy = y0 - 4 + r, ix = x0 - 4 + c;
        xin[e] = (iy >= 0 && iy < H && ix >= 0 && ix < W) ? x[(img + (size_t)iy * W + ix) * 3 + ci] : (bf16_t)0;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int ln = lane & 15, g = lane >> 4;
    // layer 1 (3 -> 32, K = 27 in one MFMA step) into bufA: kF1 region at image (y0 - 3, x0 - 3)
    {
        v8bf a[2];
        int koff[8];  // offset of K value 8 g + e from the lane's pixel in xin (-1: zero padding)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = 8 * g + e;
#pragma unroll
            for (int t = 0; t < 2; ++t)
                a[t][e] = __builtin_bit_cast(__bf16, k < 27 ? w0[(size_t)(t * 16 + ln) * 27 + k] : (bf16_t)0);
            const int tap = k / 3, ci = k - 3 * tap, ky = tap / 3, kx = tap - 3 * ky;
            koff[e] = k < 27 ? (ky * kFIn[1] + kx) * 3 + ci : -1;
        }
        constexpr int NG = (kF1[1] + 15) / 16;
        for (int item = wv; item < kF1[0] * NG; item += 8) {
            const int r = item / NG, p = (item - r * NG) * 16 + ln;
            const int pr = min(p, kF1[1] - 1);
            const bf16_t* src = xin + (r * kFIn[1] + pr) * 3;
            v8bf bv;
#pragma unroll
            for (int e = 0; e < 8; ++e) bv[e] = __builtin_bit_cast(__bf16, koff[e] >= 0 ? src[koff[e]] : (bf16_t)0);
            v4f acc[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], bv, v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            if (p >= kF1[1]) continue;
            const int iy = y0 - 3 + r, ix = x0 - 3 + p;
            const bool inside = iy >= 0 && iy < H && ix >= 0 && ix < W;
#pragma unroll
            for (int t = 0; t < 2; ++t)
                *reinterpret_cast<uint2*>(bufA + (r * kF1[1] + p) * kFPx + t * 16 + 4 * g) =
                    inside ? fused_pack(acc[t], bz0[t], true) : make_uint2(0u, 0u);
        }
    }
    __syncthreads();
    // the next layer's weight fragments are loaded while this one computes
    v8bf wb[2][9];
    float bz2[2][4];
    fused_weights(w2, wb);
    fused_bias(b2, bz2);
    fused_layer32<kF2[0], kF2[1], false>(bufA, bufB, wa, bz, true, y0 - 2, x0 - 2, H, W, nullptr, img);
    __syncthreads();
    fused_weights(w3, wa);
    fused_bias(b3, bz);
    fused_layer32<kFusedY + 2, kFusedX + 2, false>(bufB, bufA, wb, bz2, true, y0 - 1, x0 - 1, H, W, nullptr, img);
    __syncthreads();
    fused_layer32<kFusedY, kFusedX, true>(bufA, nullptr, wa, bz, false, y0, x0, H, W, y, img);
}

bool use_conv32(const void* x, const void* mask, const void* w = nullptr) {
    const uintptr_t at = reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(mask) | reinterpret_cast<uintptr_t>(w);
    return (at & 15) == 0 && staged_conv_enabled();
}

// scale > 0: y receives descriptor records (without mask).
void launch_conv32(const bf16_t* x, const bf16_t* mask, const bf16_t* w, const float* bias, bf16_t* y, int n, int H,
                   int W, int dil, int relu, hipStream_t st, float scale = 0.f) {
    // Rows per wave: about 4608 waves (one and a half rounds of three waves per
    // SIMD), so the two halo rows a wave reads on top stay a small share; more,
    // shorter waves reread more, fewer leave the chip idle at the end (four
    // 1242 x 375 images: 49 us with 4608 waves, 56 with 3072, 53 with 6144, 60
    // with 12288).  At least 4 rows where the call is too small to fill the chip.
    const size_t rows = (size_t)((W + 15) / 16) * n * H;  // 16-pixel rows
    const int R = (int)std::min<size_t>(std::max<size_t>(rows / 4608, 4), 64);
    const int hp = (H + dil - 1) / dil;
    const dim3 grid((W + 63) / 64, dil * ((hp + R - 1) / R), n);
    if (mask)
        hipLaunchKernelGGL((conv32_column_kernel<true, false>), grid, dim3(256), 0, st, x, mask, w, bias, y, H, W, dil, relu,
                           R, 0.f);
    else if (scale > 0.f)
        hipLaunchKernelGGL((conv32_column_kernel<false, true>), grid, dim3(256), 0, st, x, mask, w, bias, y, H, W, dil, relu,
                           R, scale);
    else
        hipLaunchKernelGGL((conv32_column_kernel<false, false>), grid, dim3(256), 0, st, x, mask, w, bias, y, H, W, dil,
                           relu, R, 0.f);
}

// Partials of the weight gradient, for whichever dilation takes most.
size_t wgrad_part_bytes(int n, int H, int W, int cin) {
    size_t blocks = 0;
    for (int d = 1; d <= kMaxDil; ++d) blocks = std::max(blocks, (size_t)wgrad_split(n, H, W, d).blocks);
    return align256(blocks * ((cin == 32 ? kWgTiles<32> : kWgTiles<3>) + 2) * 256 * sizeof(float));
}

}  // namespace
}  // namespace sff

using namespace sff;

extern "C" sff_status sff_conv3x3_bf16_fwd(int32_t n, int32_t H, int32_t W, int32_t cin,
                                           int32_t cout, int32_t dil, int32_t relu,
                                           const uint16_t* x, const uint16_t* w, const float* bias,
                                           uint16_t* y, void* stream) {
    if (!conv_shape_ok(n, H, W, cin, cout, dil) || !x || !w || !y) return SFF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(y) & 7) != 0) return SFF_ERR_INVALID_ARG;
    const dim3 grid((W + kTilePx - 1) / kTilePx, H, n);
    hipStream_t st = as_stream(stream);
    if (cin == 3 && staged_conv_enabled())
        hipLaunchKernelGGL(conv3_fwd_kernel, dim3((W + kTile32 - 1) / kTile32, (H + kRows32 - 1) / kRows32, n),
                           dim3(256), 0, st, x, w, bias, y, H, W, dil, relu);
    else if (cin == 3)
        hipLaunchKernelGGL((conv_fwd_kernel<3, 32>), grid, dim3(256), 0, st, x, nullptr, w, bias, y,
                           H, W, dil, relu);
    else if (use_conv32(x, nullptr, w))
        launch_conv32(x, nullptr, w, bias, y, n, H, W, dil, relu, st);
    else
        hipLaunchKernelGGL((conv_fwd_kernel<32, 32>), grid, dim3(256), 0, st, x, nullptr, w, bias,
                           y, H, W, dil, relu);
    return launch_status();
}

extern "C" sff_status sff_conv3x3_bf16_records(int32_t n, int32_t H, int32_t W, int32_t dil, const uint16_t* x,
                                               const uint16_t* w, const float* bias, float scale,
                                               int16_t* desc, void* stream) {
    if (!conv_shape_ok(n, H, W, 32, 32, dil) || !x || !w || !desc || !(scale > 0.f) || scale > 8192.f)
        return SFF_ERR_INVALID_ARG;
    if (((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(desc)) & 15) != 0)
        return SFF_ERR_INVALID_ARG;
    launch_conv32(x, nullptr, w, bias, reinterpret_cast<uint16_t*>(desc), n, H, W, dil, 0, as_stream(stream), scale);
    return launch_status();
}

extern "C" size_t sff_conv3x3_bf16_bwd_workspace_bytes(int32_t n, int32_t H, int32_t W,
                                                       int32_t cin, int32_t cout) {
    if (!conv_shape_ok(n, H, W, cin, cout, 1)) return 0;
    return align256((size_t)cin * 9 * cout * sizeof(uint16_t)) +
           wgrad_part_bytes(n, H, W, cin);
}

extern "C" sff_status sff_conv3x3_bf16_dgrad(int32_t n, int32_t H, int32_t W, int32_t cin,
                                             int32_t cout, int32_t dil, const uint16_t* dy,
                                             const uint16_t* relu_out, const uint16_t* w,
                                             uint16_t* dx, void* workspace,
                                             size_t workspace_bytes, void* stream) {
    if (!conv_shape_ok(n, H, W, cin, cout, dil) || cin != 32 || !dy || !w || !dx)
        return SFF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(dx) & 7) != 0) return SFF_ERR_INVALID_ARG;
    const size_t need = align256((size_t)cin * 9 * cout * sizeof(uint16_t));
    if (!workspace || workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return SFF_ERR_WORKSPACE;
    hipStream_t st = as_stream(stream);
    uint16_t* wt = static_cast<uint16_t*>(workspace);
    hipLaunchKernelGGL(flip_weights_kernel, dim3((cin * 9 * cout + 255) / 256), dim3(256), 0, st, w,
                       wt, cin, cout);
    if (use_conv32(dy, relu_out))
        launch_conv32(dy, relu_out, wt, nullptr, dx, n, H, W, dil, 0, st);
    else
        hipLaunchKernelGGL((conv_fwd_kernel<32, 32>), dim3((W + kTilePx - 1) / kTilePx, H, n), dim3(256),
                           0, st, dy, relu_out, wt, nullptr, dx, H, W, dil, 0);
    return launch_status();
}

extern "C" sff_status sff_conv3x3_bf16_wgrad(int32_t n, int32_t H, int32_t W, int32_t cin,
                                             int32_t cout, int32_t dil, const uint16_t* x,
                                             const uint16_t* dy, const uint16_t* relu_out,
                                             float* dw, float* db, void* workspace,
                                             size_t workspace_bytes, void* stream) {
    if (!conv_shape_ok(n, H, W, cin, cout, dil) || !x || !dy || !dw || !db)
        return SFF_ERR_INVALID_ARG;
    const size_t off = align256((size_t)cin * 9 * cout * sizeof(uint16_t));
    const size_t need = off + wgrad_part_bytes(n, H, W, cin);
    if (!workspace || workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return SFF_ERR_WORKSPACE;
    hipStream_t st = as_stream(stream);
    float* part = reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + off);
    const WgradSplit sp = wgrad_split(n, H, W, dil);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(sp.blocks), dim3(64 * kWgWaves), 0, st, x, dy, relu_out, part, H, W, dil, sp.R,
                           sp.strips, sp.chunks, sp.units);
    };
    const bool vec = use_conv32(dy, relu_out);
    if (cin == 3)
        vec ? launch(wgrad_column_kernel<3, true>) : launch(wgrad_column_kernel<3, false>);
    else
        vec && use_conv32(x, nullptr) ? launch(wgrad_column_kernel<32, true>) : launch(wgrad_column_kernel<32, false>);
    const int nt = cin == 32 ? kWgTiles<32> : kWgTiles<3>;
    hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((nt + 2) * 256 / kRedOut), dim3(256), 0, st, part, dw, db, sp.blocks,
                       cin);
    return launch_status();
}

extern "C" sff_status sff_featnet_fwd_bf16(int32_t n, int32_t H, int32_t W, int32_t dil,
                                           const uint16_t* x, const uint16_t* w0, const float* b0,
                                           const uint16_t* w1, const float* b1, const uint16_t* w2,
                                           const float* b2, const uint16_t* w3, const float* b3,
                                           uint16_t* y, void* stream) {
    if (!conv_shape_ok(n, H, W, 3, 32, dil) || !x || !w0 || !w1 || !w2 || !w3 || !y)
        return SFF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(y) & 7) != 0 || (reinterpret_cast<uintptr_t>(w1) & 15) != 0 ||
        (reinterpret_cast<uintptr_t>(w2) & 15) != 0 || (reinterpret_cast<uintptr_t>(w3) & 15) != 0)
        return SFF_ERR_INVALID_ARG;
    if (dil != 1) return SFF_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(featnet_fwd_kernel, dim3((W + kFusedX - 1) / kFusedX, (H + kFusedY - 1) / kFusedY, n),
                       dim3(512), 0, as_stream(stream), x, w0, b0, w1, b1, w2, b2, w3, b3, y, H, W);
    return launch_status();
}
