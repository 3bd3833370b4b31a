// The paper's own matching cost (SceneFlowFields, Section 3.1, "Matching
// Cost", eq. (1)): per pixel, the Euclidean distances between the first three
// principal components of dense SIFT features, summed over a 7 x 7 window and
// the temporal, stereo and cross correspondences; principal axes from the SIFT
// features of all four images of the pair; boundary pixels replicated.
//
// Dense SIFT as in SIFT flow (Liu et al., TPAMI 2011) after Lowe (IJCV 2004):
// central-difference gradients, 8 orientation bins of 45 degrees with linear
// interpolation between bin centres, 4 x 4 cells of 3 x 3 pixels around the
// pixel (rows and columns -6 .. +5, flat window, clamped), unit length, clamp
// at 0.2, unit length again.  The gradients are taken on the channel sum
// (integers, exact in FP32): a constant factor changes neither orientations
// nor the normalised descriptor.
//
// Pipeline of sff_sift_pca: cell-sum planes -> Gram
// matrix and sum of all descriptors of the pair (exact digit products, FP64 for
// descriptors with very small entries; a partial per block, reduced in a fixed
// order) -> covariance -> the three leading eigenvectors (subspace iteration on a
// power of the covariance in one block, or a direct solution) -> projected features.
// Descriptors are recomputed from the cell-sum planes in the Gram and the
// projection pass instead of being stored (512 B per pixel).
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "sff_internal.hpp"

namespace sff {
namespace {

constexpr int kBins = 8;
constexpr int kCell = 3;
constexpr int kHalf = 6;                    // descriptor window -6 .. +5
constexpr int kExt = 2 * kHalf - kCell;     // 9 extra rows / columns of the cell-sum planes
constexpr int kDesc = 128;
constexpr float kClampV = 0.2f;
constexpr int kGramPx = 64;                 // descriptors per Gram step (4 threads each)
constexpr int kMaxGramBlocks = 256;  // one block per CU
constexpr size_t kGramMaxPx = 16384;  // descriptors per Gram block (exact int32 sums)
constexpr int kPart = 36 * 256 + kDesc;  // doubles per Gram partial: upper 16 x 16 tiles, sums
constexpr int kSub = 8;                     // subspace dimension of the eigen iteration
constexpr int kCheck = 4;                   // iterations between Rayleigh-Ritz checks
constexpr int kMaxIter = 16;                // then the direct solution
constexpr int kWinR = 3;                    // cost window -3 .. +3
constexpr int kCT = 16;                     // cost tile side

struct SiftGeom {
    int H, W, He, We;
    size_t npx, plane_c;  // pixels, cells of an image
};

inline SiftGeom sift_geom(const sff_params& p) {
    SiftGeom g;
    g.H = p.H;
    g.W = p.W;
    g.He = p.H + kExt;
    g.We = p.W + kExt;
    g.npx = (size_t)p.H * p.W;
    g.plane_c = (size_t)g.He * g.We;
    return g;
}

// At most one block per CU, each with at least six steps of 128 descriptors if there
// are that many (the same for every batch, so that a pair's sums do not depend on it),
// and never more than kGramMaxPx.  A block costs a partial of 75 KB: a 96 x 160 pair
// needs 8.8 MB of workspace, 34.6 with two steps a block and whole matrices; its
// features take as long (597 and 599 us; 617 with eight steps).
inline int gram_blocks(const SiftGeom& g) {
    const size_t per = 4 * g.npx;
    const size_t nb = (per + 12 * kGramPx - 1) / (12 * kGramPx);
    return (int)std::max(std::max<size_t>(1, std::min<size_t>(kMaxGramBlocks, nb)), (per + kGramMaxPx - 1) / kGramMaxPx);
}

// Descriptors that a wave of the Gram pass may hand to the FP64 one.
constexpr int kGramWaves = 8, kGramStep = 2 * kGramPx;  // waves of a block, descriptors per step
inline int gram_list(const SiftGeom& g) {
    const int steps = (int)((4 * g.npx + kGramStep - 1) / kGramStep), nb = gram_blocks(g);
    return (steps + nb - 1) / nb * (kGramStep / kGramWaves);
}

struct SiftWs {
    size_t Cs, part, list, count, gsum, sq, ax32, total;
};

inline SiftWs sift_ws(const SiftGeom& g, int nimg) {
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const int pairs = (nimg + 3) / 4;
    SiftWs L;
    L.Cs = 0;
    L.part = L.Cs + al((size_t)nimg * kBins * g.plane_c * sizeof(float));
    const size_t waves = (size_t)pairs * gram_blocks(g) * kGramWaves;
    L.list = L.part + al((size_t)pairs * gram_blocks(g) * kPart * sizeof(double));
    L.count = L.list + al(waves * gram_list(g) * sizeof(int));
    L.gsum = L.count + al(waves * sizeof(int));
    L.sq = L.gsum + al((size_t)pairs * kPart * sizeof(double));
    L.ax32 = L.sq + al((size_t)pairs * 2 * kDesc * kDesc * sizeof(double));
    L.total = L.ax32 + al((size_t)pairs * 4 * kDesc * sizeof(float));
    return L;
}

// ------------------------------------------------------------------ SIFT --

// Cs[m][Y + 6][X + 6][b] = sum over the 3 x 3 cell whose top-left pixel is
// (Y, X), coordinates clamped, of the orientation energy in bin b: a pixel's
// gradient magnitude split between the two bins whose centres enclose its
// orientation.  Y in -6 .. H + 2, X in -6 .. W + 2.  The 8 bins of a cell are
// contiguous (32 bytes, two 16-byte loads).  A block forms the energies of the
// (kCellY + 2) x (kCellX + 2) pixels its cells cover in LDS (a bin per plane),
// then sums them.  Bound: HBM (32 B written per cell).  A KITTI-size pair's four
// images: 43 us, against 86 us with the energies written to planes in memory
// (another 32 B per pixel each way) by a kernel of their own.
constexpr int kCellX = 64, kCellY = 8;
constexpr int kEnX = kCellX + kCell - 1, kEnY = kCellY + kCell - 1;

__global__ void __launch_bounds__(256) cellsum_kernel(const uint8_t* __restrict__ img, float* __restrict__ Cs,
                                                      int H, int W, int C) {
    __shared__ float en[kBins][kEnY][kEnX];
    const int He = H + kExt, We = W + kExt;
    const int m = blockIdx.z;
    const int X0 = blockIdx.x * kCellX, Y0 = blockIdx.y * kCellY;  // first cell, plane coordinates
    const uint8_t* im = img + (size_t)m * H * W * C;
    for (int e = threadIdx.x; e < kEnY * kEnX; e += 256) {
        const int r = e / kEnX, c = e - r * kEnX;
        const int y = clampi(Y0 + r - kHalf, 0, H - 1), x = clampi(X0 + c - kHalf, 0, W - 1);
        auto sum = [&](int yy, int xx) {
            const uint8_t* q = im + ((size_t)yy * W + xx) * C;
            int t = 0;
            for (int ch = 0; ch < C; ++ch) t += q[ch];
            return t;
        };
        const float gx = (float)(sum(y, min(x + 1, W - 1)) - sum(y, max(x - 1, 0)));
        const float gy = (float)(sum(min(y + 1, H - 1), x) - sum(max(y - 1, 0), x));
        const float mag = sqrtf(gx * gx + gy * gy);  // exact integers below 2^24 under the root
        float pos = atan2f(gy, gx) * (float)(4.0 / M_PI);
        if (pos < 0.f) pos += 8.f;
        const float lo = floorf(pos);
        const float frac = pos - lo;
        const int b0 = (int)lo & 7, b1 = (b0 + 1) & 7;
#pragma unroll
        for (int b = 0; b < kBins; ++b) en[b][r][c] = b == b0 ? mag * (1.f - frac) : (b == b1 ? mag * frac : 0.f);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kCellY * kCellX; e += 256) {
        const int r = e / kCellX, c = e - r * kCellX;
        if (Y0 + r >= He || X0 + c >= We) continue;
        float sum[kBins];
#pragma unroll
        for (int b = 0; b < kBins; ++b) {
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < kCell; ++i)
#pragma unroll
                for (int j = 0; j < kCell; ++j) s += en[b][r + i][c + j];
            sum[b] = s;
        }
        float4* cs = reinterpret_cast<float4*>(Cs + (((size_t)m * He + Y0 + r) * We + X0 + c) * kBins);
        cs[0] = make_float4(sum[0], sum[1], sum[2], sum[3]);
        cs[1] = make_float4(sum[4], sum[5], sum[6], sum[7]);
    }
}

// Sum over the 4 lanes of a quad (DPP quad permutations).
__device__ __forceinline__ float quad_sum(float v) {
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));
    return v;
}

// v / n for r = 1 / n correctly rounded: the product's remainder is exact in an
// fma, and adding it back rounds the quotient correctly (Markstein, IBM J. Res.
// Dev. 34, 1990), so the result is that of the division, in 3 operations instead
// of about 10.  n is a norm (finite, > 0) and v at most n, zero or far above the
// subnormal range.
__device__ __forceinline__ float div_by(float v, float n, float r) {
    const float q = v * r;
    return fmaf(fmaf(-q, n, v), r, q);
}

// Image and pixel of descriptor g of a pair (g < 4 npx < 2^31).
__device__ __forceinline__ void desc_pixel(int g, int npx, int W, int& m, int& y, int& x) {
    m = (int)(g >= npx) + (int)(g >= 2 * npx) + (int)(g >= 3 * npx);
    const int p = g - m * npx;
    y = p / W;
    x = p - y * W;
}

// Quarter q (cell row q: 4 cells x 8 bins, descriptor entries 32 q .. 32 q + 31)
// of the normalised descriptor of pixel (y, x); the 4 quarters of a pixel sit in
// one quad of lanes, which must all be active.
__device__ __forceinline__ void desc_cells(const float* __restrict__ cs, int We, int y, int x, int q,
                                           float4 (&c)[8]) {
    const float4* row = reinterpret_cast<const float4*>(cs + ((size_t)(y + kCell * q) * We + x) * kBins);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        c[2 * j] = row[2 * kCell * j];
        c[2 * j + 1] = row[2 * kCell * j + 1];
    }
}

// The entries are multiplied by `scale`, a power of two or zero (exact).
__device__ __forceinline__ void desc_normalise(const float4 (&c)[8], float (&v)[32], float scale = 1.f) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[4 * j + 0] = c[j].x;
        v[4 * j + 1] = c[j].y;
        v[4 * j + 2] = c[j].z;
        v[4 * j + 3] = c[j].w;
    }
    // the order of the sums' roundings is written out, so that every kernel forms
    // the same descriptor to the bit
    auto square_sum = [&]() {
        float s = fmaf(v[0], v[0], v[1] * v[1]);
#pragma unroll
        for (int k = 2; k < 32; ++k) s = fmaf(v[k], v[k], s);
        return quad_sum(s);
    };
    const float ss = square_sum();
    if (ss > 0.f) {
        const float n = sqrtf(ss), rn = 1.f / n;
#pragma unroll
        for (int k = 0; k < 32; ++k) v[k] = fminf(div_by(v[k], n, rn), kClampV);
        const float s2 = square_sum();
        const float n2 = sqrtf(s2), rn2 = 1.f / n2;
#pragma unroll
        for (int k = 0; k < 32; ++k) v[k] = div_by(v[k], n2, rn2) * scale;
    }
}

__device__ __forceinline__ void desc_quarter(const float* __restrict__ cs, int We, int y, int x, int q,
                                             float (&v)[32]) {
    float4 c[8];
    desc_cells(cs, We, y, x, q, c);
    desc_normalise(c, v);
}

// Dense SIFT written out: [nimg][H][W][128], 64 pixels per block.
__global__ void __launch_bounds__(256) sift_out_kernel(const float* __restrict__ Cs, float* __restrict__ out,
                                                       int H, int W, int nimg) {
    const int He = H + kExt, We = W + kExt;
    const int t = threadIdx.x, q = t & 3;
    const long total = (long)nimg * H * W;
    const long g = (long)blockIdx.x * kGramPx + (t >> 2);
    const long ge = g < total ? g : total - 1;  // whole quads stay active
    const int m = (int)(ge / ((long)H * W));
    const int p = (int)(ge - (long)m * H * W);
    const int y = p / W, x = p - y * W;
    float v[32];
    desc_quarter(Cs + (size_t)m * kBins * He * We, We, y, x, q, v);
    if (g >= total) return;
    float4* o = reinterpret_cast<float4*>(out + (size_t)ge * kDesc + 32 * q);
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = make_float4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
}

// ------------------------------------------------------------------- PCA --

// Gram matrix and sum of the descriptors of one pair (4 H W of them), summed
// exactly in integers on the int8 matrix cores.  An entry f (0 <= f <= 1, FP32)
// is the fixed-point number F 2^-38 with F = sum_i d_i 256^i, five digits d_i in
// [-128, 127]: exact for f = 0 and f >= 2^-15 (24 significant bits).  A descriptor
// with an entry between (one in twenty to a hundred of textured images, most on
// images with faint texture) is left out here and listed for gram_rest_kernel, which
// sums its products in FP64.
// With digit planes D_i, G = sum_ij 2^(8 (i + j) - 76) D_i D_j^T; the 22
// products with i + j >= 2 are formed (v_mfma_i32_16x16x64_i8, K = 64 pixels),
// those of one i + j in one accumulator, exact below 2^31 (5 products of 2^14 per
// pixel, at most kGramMaxPx pixels per block).  The dropped ones are at most
// 2^-53 per pixel, with mixed signs (a lowest digit is zero for f >= 2^-7): against
// exact sums of the same descriptors the result is 4e-18 of the matrix's norm off and
// less, where FP64 sums are 1e-17 to 7e-17 off.  (Without i + j = 2: 1e-14.)
// Each block takes every nblk-th group of 128 descriptors: a thread forms a
// quarter descriptor and writes its entries' upper four digits (a word) and
// lowest digit (a byte) entry-major to LDS; wave w turns entries 16 w .. + 15
// into digit operands (16 pixels of one entry and digit per lane: byte
// permutations of 4 x 4 words), left in LDS for all waves.  An entry's pixels are
// turned and exchanged in runs of 4 (slot and digit addresses below) so that
// neither the writes nor the reads meet in a bank.  Waves 2 p and 2 p + 1 share
// the tile rows p and 7 - p of the upper triangle (9 of the 36 16 x 16 tiles).
// Partials (FP64, upper tiles only) go to part[pair][block].
// Bound: the vector ALU (forming and splitting descriptors) and the matrix units
// beside it. The int8 products take less than half
// of the FP64 products' time at the units' rates; KITTI-size pair: 421 us and 38 for
// the listed descriptors (5 %), against 742 us with v_mfma_f64_16x16x4f64 for all.
// Measured with i + j >= 3 alone, 369 us: 408 us with all waves of a block in the same
// phase, 470 us with two blocks of 4 waves per CU (their accumulators spill).
struct GramArgs {
    const float* Cs;
    double* part;
    int *list, *count;  // [pair][block][wave][cap] descriptors for gram_rest_kernel, [pair][block][wave]
    int H, W, nblk, cap;
};

typedef int i32x4 __attribute__((ext_vector_type(4)));
constexpr int kDigits = 5, kSum0 = 2, kSums = 7;  // digits of an entry; values of i + j, from kSum0
constexpr float kFix = 0x1p30f;        // scale of the upper four digits
constexpr float kFixMin = 0x1p15f;     // smallest entry that five digits hold exactly, scaled

// Place of entry (r, c) of tile (I, J), I <= J, in a partial.
__host__ __device__ constexpr int gram_at(int I, int J, int r, int c) {
    return ((I * (17 - I)) / 2 + J - I) * 256 + r * 16 + c;
}
constexpr int kSumAt = 36 * 256;  // and of the sums
static_assert(gram_at(7, 7, 15, 15) + 1 == kSumAt, "36 tiles");

// Tile n (of 9) of wave (pair) p: rows p (8 - p tiles), then 7 - p.
__device__ __forceinline__ void gram_tile(int p, int n, int& I, int& J) {
    const bool first = n < 8 - p;
    I = first ? p : 7 - p;
    J = first ? p + n : n - 1;  // 7 - p + n - (8 - p)
}

// Digit planes of 4 words (digit i of word n in byte i) transposed: byte n of
// word i of the result is digit i of word n.
__device__ __forceinline__ void digits_4x4(const uint32_t (&w)[4], uint32_t (&d)[4]) {
    const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), b = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
    const uint32_t c = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u), e = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    d[0] = __builtin_amdgcn_perm(b, a, 0x05040100u);
    d[1] = __builtin_amdgcn_perm(b, a, 0x07060302u);
    d[2] = __builtin_amdgcn_perm(e, c, 0x05040100u);
    d[3] = __builtin_amdgcn_perm(e, c, 0x07060302u);
}

constexpr int kGramTiles = 5;  // tiles of a wave, at most

__global__ void __launch_bounds__(64 * kGramWaves) gram_kernel(GramArgs a) {
    __shared__ __align__(16) uint32_t hi[2][kDesc * kGramPx];  // entry-major: upper digits,
    __shared__ __align__(16) int8_t low[2][kDesc * kGramPx];   // lowest digit
    __shared__ i32x4 ops[2][8 * kDigits * 64];                 // operands [tile][digit][lane]
    const int t = threadIdx.x, q = t & 3, px = (t >> 2) & 63, lane = t & 63, w = wave_id();
    const int H = a.H, W = a.W, He = H + kExt, We = W + kExt;
    const int npx = H * W, total = 4 * npx;
    const int pair = blockIdx.y;
    const float* Cs = a.Cs + (size_t)pair * 4 * kBins * He * We;
    i32x4 acc[kGramTiles][kSums];
    int64_t dsum = 0;  // this lane's sum of F of entry 16 w + l % 16
    const int slot_w = (pair * a.nblk + blockIdx.x) * kGramWaves + w;
    int listed = 0;  // of this wave
#pragma unroll
    for (int n = 0; n < kGramTiles; ++n)
#pragma unroll
        for (int k = 0; k < kSums; ++k) acc[n][k] = i32x4{0, 0, 0, 0};
    const int wp = w >> 1, n0 = (w & 1) * kGramTiles, nt = w & 1 ? 9 - kGramTiles : kGramTiles;
    float4 rows[8];  // the cells of the step after next
    auto load = [&](int base) {
        int m, y, x;
        desc_pixel(min(base + (t >> 2), total - 1), npx, W, m, y, x);
        desc_cells(Cs + (size_t)m * kBins * He * We, We, y, x, q, rows);
    };
    // digits of the descriptors in `rows`, to LDS
    auto digits = [&](int base) {
        float v[32];
        desc_normalise(rows, v, base + (t >> 2) < total ? kFix : 0.f);
        uint32_t least = ~0u;  // smallest entry above zero (its bits, less one)
#pragma unroll
        for (int k = 0; k < 32; ++k) least = min(least, __float_as_uint(v[k]) - 1u);
        if (const uint64_t small = __ballot(least < __float_as_uint(kFixMin) - 1u)) {
            const uint64_t quads = (small | small >> 1 | small >> 2 | small >> 3) & 0x1111111111111111ull;
            if ((quads >> (lane & ~3)) & 1) {
#pragma unroll
                for (int k = 0; k < 32; ++k) v[k] = 0.f;
                if (q == 0)
                    a.list[(size_t)slot_w * a.cap + listed + __popcll(quads & ((1ull << lane) - 1ull))] = base + (t >> 2);
            }
            listed += __popcll(quads);
        }
        // pixel slot turned by the quarter, so that a wave's writes meet all banks
        int slot = (px + 16 * q) & 63;
        asm("" : "+v"(slot));  // addresses formed here, not kept in registers between steps
        uint32_t* hs = hi[w >> 2];
        int8_t* ls = low[w >> 2];
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            // lowest digit, rounded, + 128: its bit 8 carries into the upper ones
            const uint32_t l = (uint32_t)fmaf(__builtin_amdgcn_fractf(v[k]), 256.f, 128.5f);
            const int e = 32 * q + k;  // e & 15 = k & 15, (e >> 2) & 3 = (k >> 2) & 3
            hs[e * kGramPx + (slot ^ (4 * (k & 15)))] = ((uint32_t)v[k] + (l >> 8) + 0x00808080u) ^ 0x00808080u;
            ls[e * kGramPx + (slot ^ (16 * ((k >> 2) & 3)))] = (int8_t)(l ^ 0x80u);
        }
    };
    // digit operands of entry tile w: lane = entry l % 16, pixels 16 (l / 16) .. + 15
    // (the entries are quarter w / 2's)
    auto operands = [&]() {
#pragma unroll 1
        for (int s = 0; s < 2; ++s) {
            int ln = lane;
            asm("" : "+v"(ln));  // as for the digits' addresses: 252 registers, no spills
            const int li = ln & 15, lg = ((ln >> 4) + wp) & 3, e = 16 * w + li;
            uint32_t d[kDigits][4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint4 v4 = *reinterpret_cast<const uint4*>(hi[s] + e * kGramPx + 4 * ((4 * lg + c) ^ li));
                const uint32_t ww[4] = {v4.x, v4.y, v4.z, v4.w};
                uint32_t dd[4];
                digits_4x4(ww, dd);
#pragma unroll
                for (int i = 0; i < 4; ++i) d[i + 1][c] = dd[i];
            }
            const uint4 l4 = *reinterpret_cast<const uint4*>(low[s] + e * kGramPx + 16 * (lg ^ ((li >> 2) & 3)));
            d[0][0] = l4.x;
            d[0][1] = l4.y;
            d[0][2] = l4.z;
            d[0][3] = l4.w;
#pragma unroll
            for (int i = 0; i < kDigits; ++i) {
                ops[s][(w * kDigits + i) * 64 + lane] = i32x4{(int)d[i][0], (int)d[i][1], (int)d[i][2], (int)d[i][3]};
                int sum = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) sum = __builtin_amdgcn_sdot4((int)d[i][c], 0x01010101, sum, false);
                dsum += (int64_t)sum << (8 * i);
            }
        }
    };
    auto products = [&]() {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            i32x4 opa[kDigits];
#pragma unroll
            for (int n = 0; n < kGramTiles; ++n) {
                if (n >= nt) break;  // wave-uniform
                int I, J;
                gram_tile(wp, n0 + n, I, J);
                if (n == 0 || n0 + n == 8 - wp)
#pragma unroll
                    for (int i = 0; i < kDigits; ++i) opa[i] = ops[s][(I * kDigits + i) * 64 + lane];
                i32x4 opb[kDigits];
#pragma unroll
                for (int j = 0; j < kDigits; ++j) opb[j] = ops[s][(J * kDigits + j) * 64 + lane];
#pragma unroll
                for (int i = 0; i < kDigits; ++i)
#pragma unroll
                    for (int j = max(0, kSum0 - i); j < kDigits; ++j)
                        acc[n][i + j - kSum0] =
                            __builtin_amdgcn_mfma_i32_16x16x64_i8(opa[i], opb[j], acc[n][i + j - kSum0], 0, 0, 0);
            }
        }
    };
    const int first = blockIdx.x * kGramStep, step = a.nblk * kGramStep;
    load(first);
    digits(first);
    load(first + step);
    for (int base = first; base < total; base += step) {
        __syncthreads();
        operands();
        __syncthreads();
        // this step's products and the next step's digits use different LDS; the
        // two waves of a SIMD take them in opposite order, so that the matrix
        // unit and the vector ALU are both busy
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
            if (h == (w >> 2)) {
                products();
            } else {
                digits(base + step);
                load(base + 2 * step);
            }
        }
    }
    double* part = a.part + ((size_t)pair * a.nblk + blockIdx.x) * kPart;
    // accumulator element v of lane l: row 4 (l / 16) + v, column l % 16 of the tile
#pragma unroll
    for (int n = 0; n < kGramTiles; ++n) {
        if (n >= nt) break;
        int I, J;
        gram_tile(wp, n0 + n, I, J);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double gs = 0.0;
#pragma unroll
            for (int k = 0; k < kSums; ++k) gs = fma((double)acc[n][k][v], (double)(1ull << (8 * k)), gs);
            part[gram_at(I, J, 4 * (lane >> 4) + v, lane & 15)] = gs * 0x1p-60;
        }
    }
    // over the four pixel groups (below 2^53)
    double sum = (double)dsum;
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    if (lane < 16) part[kSumAt + 16 * w + lane] = sum * 0x1p-38;
    if (lane == 0) a.count[slot_w] = listed;
}

// The listed descriptors' products and sums in FP64, added to the block's partials
// (v_mfma_f64_16x16x4f64: A = 16 entries of 4 descriptors, B = 16 entries of the same
// ones).  The descriptors are staged in LDS, 64 at a time; wave w owns the tile rows w
// and 7 - w, and the operand of tile column J is also the A operand of tile row J.
// Bound: the FP64 matrix cores where most descriptors are listed; on textured images
// reading and writing the partials.
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int W>
__device__ __forceinline__ void rest_tiles(const float (*D)[kDesc + 4], int n, int lane, f64x4 (&acc)[9]) {
    const int li = lane & 15, lk = lane >> 4;
    for (int k0 = 0; k0 < n; k0 += 4) {
        double b[8];
#pragma unroll
        for (int J = W; J < 8; ++J) b[J] = (double)D[k0 + lk][16 * J + li];
#pragma unroll
        for (int m = 0; m < 9; ++m) {
            constexpr int I1 = 7 - W;
            const int I = m < 8 - W ? W : I1, J = m < 8 - W ? W + m : I1 + m - (8 - W);
            acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(b[I], b[J], acc[m], 0, 0, 0);
        }
    }
}

__global__ void __launch_bounds__(256) gram_rest_kernel(GramArgs a) {
    __shared__ float D[kGramPx][kDesc + 4];
    const int t = threadIdx.x, q = t & 3, px = t >> 2, lane = t & 63, w = wave_id();
    const int pair = blockIdx.y, block = pair * a.nblk + blockIdx.x;
    int first[kGramWaves + 1];  // of a wave's list in the block's
    first[0] = 0;
#pragma unroll
    for (int i = 0; i < kGramWaves; ++i) first[i + 1] = first[i] + a.count[block * kGramWaves + i];
    const int n = first[kGramWaves];
    if (n == 0) return;
    const int He = a.H + kExt, We = a.W + kExt, npx = a.H * a.W;
    f64x4 acc[9];
#pragma unroll
    for (int m = 0; m < 9; ++m) acc[m] = f64x4{0.0, 0.0, 0.0, 0.0};
    double sum = 0.0;
    for (int base = 0; base < n; base += kGramPx) {
        const int e = min(base + px, n - 1);
        int wave = 0;
#pragma unroll
        for (int i = 1; i < kGramWaves; ++i) wave += e >= first[i];
        int at = e;  // in the wave's list
#pragma unroll
        for (int i = 1; i < kGramWaves; ++i) at = wave == i ? e - first[i] : at;
        int m, y, x;
        desc_pixel(a.list[(size_t)(block * kGramWaves + wave) * a.cap + at], npx, a.W, m, y, x);
        float v[32];
        desc_quarter(a.Cs + ((size_t)pair * 4 + m) * kBins * He * We, We, y, x, q, v);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 32; ++k) D[px][32 * q + k] = base + px < n ? v[k] : 0.f;
        __syncthreads();
        const int here = min(n - base, kGramPx);
        switch (w) {  // wave-uniform
            case 0: rest_tiles<0>(D, here, lane, acc); break;
            case 1: rest_tiles<1>(D, here, lane, acc); break;
            case 2: rest_tiles<2>(D, here, lane, acc); break;
            default: rest_tiles<3>(D, here, lane, acc); break;
        }
        if (t < kDesc)
            for (int k = 0; k < here; ++k) sum += (double)D[k][t];
    }
    double* part = a.part + (size_t)block * kPart;
    // accumulator element v of lane l: row l / 16 + 4 v, column l % 16 of the tile
#pragma unroll
    for (int m = 0; m < 9; ++m) {
        int I, J;
        gram_tile(w, m, I, J);
#pragma unroll
        for (int v = 0; v < 4; ++v) part[gram_at(I, J, (lane >> 4) + 4 * v, lane & 15)] += acc[m][v];
    }
    if (t < kDesc) part[kSumAt + t] += sum;
}

// Partials summed per entry with 8 interleaved accumulators combined in a fixed
// order: deterministic.
__global__ void __launch_bounds__(256) gram_sum_kernel(const double* __restrict__ part, int nblk,
                                                       double* __restrict__ gsum) {
    const int e = blockIdx.x * 256 + threadIdx.x, pair = blockIdx.y;
    if (e >= kPart) return;
    const double* P = part + (size_t)pair * nblk * kPart + e;
    double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int b = 0;
    for (; b + 8 <= nblk; b += 8)
#pragma unroll
        for (int u = 0; u < 8; ++u) s[u] += P[(size_t)(b + u) * kPart];
    for (; b < nblk; ++b) s[0] += P[(size_t)b * kPart];
    gsum[(size_t)pair * kPart + e] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// mean = S / N, cov = G / N - mean mean^T (G from its upper tiles).
__global__ void __launch_bounds__(kDesc) gram_cov_kernel(const double* __restrict__ gsum, double inv_n,
                                                        double* __restrict__ mean, double* __restrict__ cov) {
    const int r = blockIdx.x, pair = blockIdx.y, c = threadIdx.x;
    const double* g = gsum + (size_t)pair * kPart;
    const int lo = min(r, c), hi = max(r, c);
    const bool up = (r >> 4) != (c >> 4);  // a diagonal tile is stored whole
    const int a = up ? lo : r, b = up ? hi : c;
    const double grc = g[gram_at(a >> 4, b >> 4, a & 15, b & 15)];
    const double mr = g[kSumAt + r] * inv_n, mc = g[kSumAt + c] * inv_n;
    cov[((size_t)pair * kDesc + r) * kDesc + c] = grc * inv_n - mr * mc;
    if (r == 0) mean[(size_t)pair * kDesc + c] = mc;
}

// Small dense linear algebra of one thread, every loop fully unrolled so
// that the arrays stay in registers.

// Rinv = R^-1 for G = R^T R (Cholesky, R upper).  A column that is
// (numerically) in the span of the previous ones keeps a unit diagonal and no
// coupling instead of being scaled up, so a rank-deficient covariance cannot
// make the iteration overflow.
__device__ __forceinline__ void chol_inverse(const double (*Gs)[kSub], double (*Rinv_out)[kSub]) {
    double R[kSub][kSub], Ri[kSub][kSub];
    double gmax = 0.0;
#pragma unroll
    for (int i = 0; i < kSub; ++i) gmax = fmax(gmax, Gs[i][i]);
#pragma unroll
    for (int j = 0; j < kSub; ++j) {
#pragma unroll
        for (int i = 0; i < kSub; ++i) R[i][j] = 0.0;
#pragma unroll
        for (int i = 0; i < j; ++i) {
            double s = Gs[i][j];
#pragma unroll
            for (int k = 0; k < i; ++k) s -= R[k][i] * R[k][j];
            R[i][j] = s * Ri[i][i];
        }
        double s = Gs[j][j];
#pragma unroll
        for (int k = 0; k < j; ++k) s -= R[k][j] * R[k][j];
        if (s > 1e-24 * gmax && gmax > 0.0) {
            R[j][j] = sqrt(s);
        } else {
#pragma unroll
            for (int i = 0; i < j; ++i) R[i][j] = 0.0;
            R[j][j] = 1.0;
        }
        Ri[j][j] = 1.0 / R[j][j];
    }
#pragma unroll
    for (int j = 0; j < kSub; ++j) {
#pragma unroll
        for (int i = j + 1; i < kSub; ++i) Ri[i][j] = 0.0;
#pragma unroll
        for (int i = j - 1; i >= 0; --i) {
            double s = 0.0;
#pragma unroll
            for (int k = i + 1; k <= j; ++k) s += R[i][k] * Ri[k][j];
            Ri[i][j] = -s * Ri[i][i];
        }
    }
#pragma unroll
    for (int i = 0; i < kSub; ++i)
#pragma unroll
        for (int j = 0; j < kSub; ++j) Rinv_out[i][j] = Ri[i][j];
}

// Eigenpairs of the symmetric part of Ts by Jacobi rotations, sorted by
// eigenvalue, largest first: values to th_out, vectors to the columns of S_out.
// Called by one wave: lane l holds element (l / 8, l % 8) of the matrix and of the
// vectors, and a sweep is seven rounds of four disjoint rotations (the pairs of a
// round-robin of eight), so the divisions and roots of four angles run side by
// side.  Bound: that serial chain; the 28 rotations of a sweep one after the other
// in one lane took 12 us more.
__device__ __forceinline__ void ritz_small(const double (*Ts)[kSub], double* th_out, double (*S_out)[kSub]) {
    static_assert(kSub == 8, "a lane per element");
    const int lane = threadIdx.x & 63, i = lane >> 3, j = lane & 7;
    double a = 0.5 * (Ts[i][j] + Ts[j][i]), v = i == j ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 40; ++sweep) {
        double tot = a * a, off = i == j ? 0.0 : tot;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            tot += __shfl_xor(tot, m);
            off += __shfl_xor(off, m);
        }
        if (off <= 1e-32 * tot) break;
#pragma unroll 1
        for (int r = 0; r < 7; ++r) {
            // players x and y of round r meet: x + y = 2 r (mod 7), r meets 7
            auto partner = [&](int x) { return x == 7 ? r : x == r ? 7 : (2 * r + 7 - x) % 7; };
            const int pi = partner(i), pj = partner(j), p = min(j, pj), q = max(j, pj);
            const double app = __shfl(a, 9 * p), aqq = __shfl(a, 9 * q), apq = __shfl(a, 8 * p + q);
            double c = 1.0, sn = 0.0;
            if (apq != 0.0) {
                const double th = (aqq - app) / (2.0 * apq);
                const double tt = (th >= 0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
                c = 1.0 / sqrt(tt * tt + 1.0);
                sn = j == p ? -(tt * c) : tt * c;
            }
            const double ci = __shfl(c, i), si = __shfl(sn, i);  // of the row's pair
            const double t = c * a + sn * __shfl(a, 8 * i + pj);
            a = ci * t + si * __shfl(t, 8 * pi + j);
            if (j == pi) a = 0.0;
            v = c * v + sn * __shfl(v, 8 * i + pj);
        }
    }
    const double d = __shfl(a, 9 * j);
    int rank = 0;
#pragma unroll
    for (int k = 0; k < kSub; ++k) {
        const double dk = __shfl(a, 9 * k);
        rank += dk > d || (dk == d && k < j);
    }
    if (i == 0) th_out[rank] = d;
    S_out[i][rank] = v;
}

// Sum over the block (N threads) of one double per thread.
template <int N>
__device__ double block_sum(double v, double* red) {
    const int t = threadIdx.x;
    red[t] = v;
    __syncthreads();
    for (int s = N / 2; s > 0; s >>= 1) {
        if (t < s) red[t] += red[t + s];
        __syncthreads();
    }
    const double r = red[0];
    __syncthreads();
    return r;
}

// The three leading eigenvectors of one pair's covariance A.  A SIFT covariance
// often has a flat spectrum (neighbouring eigenvalues within a few percent), so
// plain subspace iteration converges slowly; the iteration runs
// on M = A^(2^kSquare) instead (same eigenvectors, ratios raised to that
// power), formed beforehand by square_kernel (squarings normalised by the
// trace).  Subspace iteration with
// kSub vectors: Z = M Q, Q = orth(Z) (Cholesky QR, twice).  Every kCheck-th
// step multiplies by A itself and does a Rayleigh-Ritz step in span(Q): Ritz
// pairs of A and their residuals ||A y - theta y|| (A y = Z s); it stops when
// the three leading ones are unit vectors with residuals below 1e-12 theta_1.
// Where the spectrum falls steeply (images that are flat in part, stripes), M has
// lost the second or third vector in its rounding ((theta_3 / theta_1)^64 below
// 1e-6 for a ratio below 0.8); such a pair, and one that has not
// converged after kMaxIter steps, is solved directly (direct_eigen).
// The matrices are read from global memory (symmetric: row r of M Q is read
// down column r, coalesced).  Each axis is signed so that its component of
// largest magnitude is positive.  Also writes the FP32 axes and mean used by
// the projection.
constexpr int kSquare = 6;  // A^64: KITTI-size pair 1.68 ms of features vs 1.78 with A^32 (A^128: no gain)

// One 16 x 16 tile of C = B B / trace(B)^2 per block, for a symmetric positive
// semidefinite B (trace(C) is in [1 / 128, 1]): every block sums the diagonal in
// the same order, so all tiles share one scale, and C[r][c] = sum_k B[k][r] B[k][c]
// with the two factors of a term commuting in fma, so C is exactly symmetric again.
// Bound: latency (a load, a block sum and a chain of 128 fma): 5.9 us; 9.9 with
// trace(B B), which every block took from all of B.
__global__ void __launch_bounds__(256) square_kernel(const double* __restrict__ B_all, size_t b_stride,
                                                     double* __restrict__ C_all, size_t c_stride) {
    __shared__ double colr[kDesc][16], colc[kDesc][16];
    __shared__ double red[256];
    const int t = threadIdx.x, ti = blockIdx.x >> 3, tj = blockIdx.x & 7;
    const double* B = B_all + (size_t)blockIdx.y * b_stride;
    double* C = C_all + (size_t)blockIdx.y * c_stride;
    const double tr = block_sum<256>(t < kDesc ? B[(size_t)t * (kDesc + 1)] : 0.0, red);
#pragma unroll
    for (int e = t; e < kDesc * 16; e += 256) {
        const int k = e >> 4, c = e & 15;
        colr[k][c] = B[(size_t)k * kDesc + 16 * ti + c];
        colc[k][c] = B[(size_t)k * kDesc + 16 * tj + c];
    }
    __syncthreads();
    const int r = t >> 4, c = t & 15;
    double acc = 0.0;
    for (int k = 0; k < kDesc; ++k) acc = fma(colr[k][r], colc[k][c], acc);
    const double sc = tr > 0.0 ? 1.0 / tr : 1.0;
    C[(size_t)(16 * ti + r) * kDesc + 16 * tj + c] = acc * sc * sc;
}

constexpr int kEigParts = 4, kEigThreads = kEigParts * kDesc;

template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}
__device__ __forceinline__ double lane_double(double v, int lane) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}
// Sum over the wave, the same in every lane.  All lanes must be active.
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_double<0xB1>(v);   // quad_perm 1,0,3,2
    v += dpp_double<0x4E>(v);   // quad_perm 2,3,0,1
    v += dpp_double<0x141>(v);  // row_half_mirror
    v += dpp_double<0x140>(v);  // row_mirror
    return (lane_double(v, 0) + lane_double(v, 16)) + (lane_double(v, 32) + lane_double(v, 48));
}

// 1 / v by two Newton steps on the hardware's estimate: within a few ulp.
__device__ __forceinline__ double rcp_double(double v) {
    double r = __builtin_amdgcn_rcp(v);
    r = fma(fma(-v, r, 1.0), r, r);
    return fma(fma(-v, r, 1.0), r, r);
}

// Working set of direct_eigen.  The factors of the tridiagonal systems take the
// place of the reduction's partial sums.
struct DirectLds {
    double v[kDesc][kDesc];
    union {
        double part[kEigThreads / 64][kDesc];
        struct {
            double u0[3][kDesc], u1[3][kDesc], u2[3][kDesc], mult[3][kDesc];
        };
    };
    double d[kDesc], e[kDesc], beta[kDesc], head[kDesc], x[3][kDesc];
    double red[kEigThreads / 64];
    int count[6], swapped[3][kDesc];
};

// The three largest eigenvalues of the symmetric A and orthonormal eigenvectors
// (to th[0..2] and Y), whatever the spectrum: Householder reduction to a
// tridiagonal matrix (the matrix in registers), the eigenvalues by bisection on Sturm counts (128
// shifts a round for each), the vectors by inverse iteration, orthogonalised in
// order (equal eigenvalues), and transformed back (Golub and Van Loan, "Matrix
// Computations", sections 8.3 to 8.5).  Errors are a few ulp of the norm.
// Bound: latency: 126 reduction steps of two barriers (half of the time), then
// serial recurrences; 370 us, 510 with the matrix in LDS.  A pair that does not need
// it costs an empty launch (less than keeping both methods' code and LDS in one
// kernel: 590 against 602 us for a KITTI-size pair's features).
__device__ __forceinline__ void direct_eigen(const double* __restrict__ A, DirectLds& L, double* th, double (*Y)[kDesc]) {
    constexpr int kWaves = kEigThreads / 64, kRows = kDesc / kWaves;
    const int t = threadIdx.x, lane = t & 63, wv = wave_id(), c1 = lane + 64;
    const int h = wv >> 1, r = t & (kDesc - 1);
    // rows wv + 8 i of the matrix, columns l and l + 64, scaled by a power of two to
    // entries below 2
    double a0[kRows], a1[kRows], amax = 0.0;
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        a0[i] = A[(size_t)(wv + kWaves * i) * kDesc + lane];
        a1[i] = A[(size_t)(wv + kWaves * i) * kDesc + c1];
        amax = fmax(amax, fmax(fabs(a0[i]), fabs(a1[i])));
    }
    for (int m = 1; m < 64; m <<= 1) amax = fmax(amax, __shfl_xor(amax, m));
    if (lane == 0) L.red[wv] = amax;
    __syncthreads();
    for (int k = 0; k < kWaves; ++k) amax = fmax(amax, L.red[k]);
    if (!(amax > 1e-290)) {  // nothing to tell apart (a flat image)
        if (t < kDesc)
            for (int k = 0; k < 3; ++k) Y[k][t] = t == k ? 1.0 : 0.0;
        if (t < 3) th[t] = 0.0;
        __syncthreads();
        return;
    }
    const int ex = ilogb(amax);
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        a0[i] = ldexp(a0[i], -ex);
        a1[i] = ldexp(a1[i], -ex);
    }
    if (wv == 0) {
        L.v[0][lane] = a0[0];
        L.v[0][c1] = a1[0];
    }
    __syncthreads();
    // step k: row k, left in L.v by its wave, is made alpha e_(k+1) by the reflection
    // 1 - beta v v^T; v stays there but for its first element, `head`.  Every wave
    // forms v and w itself, elements l and l + 64 in lane l, and broadcasts those of its
    // rows by readlane.
#pragma unroll 1
    for (int k = 0; k < kDesc - 2; ++k) {
        double v0 = lane > k ? L.v[k][lane] : 0.0, v1 = c1 > k ? L.v[k][c1] : 0.0;
        const double diag = L.v[k][k], first = lane_double(k + 1 < 64 ? v0 : v1, (k + 1) & 63);
        const double n2 = wave_sum(v0 * v0 + v1 * v1);
        double alpha = 0.0, beta = 0.0, head = 0.0;
        if (n2 > 1e-60) {  // below: nothing left in the row
            alpha = first > 0.0 ? -sqrt(n2) : sqrt(n2);
            head = first - alpha;
            beta = rcp_double(n2 - alpha * first);
        }
        v0 = lane == k + 1 ? head : v0;
        v1 = c1 == k + 1 ? head : v1;
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int i = 0; i < kRows; ++i)
            if (wv + kWaves * i > k) {  // wave-uniform
                const double v = lane_double(i < kRows / 2 ? v0 : v1, (wv + kWaves * i) & 63);
                s0 = fma(a0[i], v, s0);
                s1 = fma(a1[i], v, s1);
            }
        L.part[wv][lane] = s0;
        L.part[wv][c1] = s1;
        __syncthreads();
        double w0 = 0.0, w1 = 0.0;
#pragma unroll
        for (int i = 0; i < kWaves; ++i) {
            w0 += L.part[i][lane];
            w1 += L.part[i][c1];
        }
        w0 = lane > k ? beta * w0 : 0.0;
        w1 = c1 > k ? beta * w1 : 0.0;
        const double f = 0.5 * beta * wave_sum(v0 * w0 + v1 * w1);
        w0 -= f * v0;
        w1 -= f * v1;
#pragma unroll
        for (int i = 0; i < kRows; ++i)
            if (wv + kWaves * i > k) {
                const int c = (wv + kWaves * i) & 63;
                const double v = lane_double(i < kRows / 2 ? v0 : v1, c), w = lane_double(i < kRows / 2 ? w0 : w1, c);
                a0[i] -= fma(v, w0, w * v0);
                a1[i] -= fma(v, w1, w * v1);
                if (wv + kWaves * i <= k + 2) {  // the next row; the last ones are read below
                    L.v[wv + kWaves * i][lane] = a0[i];
                    L.v[wv + kWaves * i][c1] = a1[i];
                }
            }
        __syncthreads();
        if (t == 0) {
            L.d[k] = diag;
            L.e[k] = alpha;
            L.beta[k] = beta;
            L.head[k] = head;
        }
    }
    if (t == 0) {
        L.d[kDesc - 2] = L.v[kDesc - 2][kDesc - 2];
        L.d[kDesc - 1] = L.v[kDesc - 1][kDesc - 1];
        L.e[kDesc - 2] = L.v[kDesc - 2][kDesc - 1];
        L.e[kDesc - 1] = 0.0;
    }
    __syncthreads();
    // eigenvalue k: #{eigenvalues >= lo} > k >= #{eigenvalues >= hi}; the norm is at most 2 kDesc
    const int k3 = min(h, 2);
    double lo = -2.0 * kDesc - 4.0, hi = -lo;
#pragma unroll 1
    for (int round = 0; round < 9; ++round) {
        const double w = hi - lo, sigma = lo + w * ((r + 1) * (1.0 / (kDesc + 1)));
        double q = L.d[0] - sigma;
        int below = q < 0.0;
#pragma unroll 4
        for (int i = 1; i < kDesc; ++i) {
            const double e = L.e[i - 1];
            if (fabs(q) < 1e-200) q = -1e-200;
            q = fma(-e * e, rcp_double(q), L.d[i] - sigma);
            below += q < 0.0;
        }
        const uint64_t yes = __ballot(kDesc - below > k3);
        if (lane == 0 && h < 3) L.count[wv] = __popcll(yes);
        __syncthreads();
        const int n = L.count[2 * k3] + L.count[2 * k3 + 1];
        if (n < kDesc) hi = lo + w * ((n + 1) * (1.0 / (kDesc + 1)));
        if (n > 0) lo = lo + w * (n * (1.0 / (kDesc + 1)));
        __syncthreads();
    }
    const double lam = 0.5 * (lo + hi);
    // T - lam = L U with row exchanges, by one lane per eigenvalue; pivots no smaller than 1e-15
    auto pivot = [](double v) { return fabs(v) >= 1e-15 ? v : (v < 0.0 ? -1e-15 : 1e-15); };
    const bool solver = r == 0 && h < 3;
    if (solver) {
        double a = L.d[0] - lam, b = L.e[0];
#pragma unroll 4
        for (int i = 0; i + 1 < kDesc; ++i) {
            const double sub = L.e[i], dg = L.d[i + 1] - lam, sup = L.e[i + 1];
            const bool swap = fabs(a) < fabs(sub);
            const double u = rcp_double(pivot(swap ? sub : a)), m = (swap ? a : sub) * u;
            L.u0[h][i] = u;
            L.u1[h][i] = swap ? dg : b;
            L.u2[h][i] = swap ? sup : 0.0;
            L.mult[h][i] = m;
            L.swapped[h][i] = swap;
            a = swap ? b - m * dg : dg - m * b;
            b = swap ? -m * sup : sup;
        }
        L.u0[h][kDesc - 1] = 1.0 / pivot(a);
        L.u1[h][kDesc - 1] = L.u2[h][kDesc - 1] = 0.0;
        th[h] = ldexp(lam, ex);
    }
    for (int i = t; i < 3 * kDesc; i += kEigThreads) {
        uint32_t z = (uint32_t)(i + 1) * 2654435761u;
        z ^= z >> 15;
        z *= 2246822519u;
        z ^= z >> 13;
        L.x[i / kDesc][i % kDesc] = (double)(z & 0xFFFF) / 32768.0 - 1.0;
    }
    __syncthreads();
#pragma unroll 1
    for (int it = 0; it < 3; ++it) {
        if (solver) {
            double* x = L.x[h];
            double cur = x[0];
#pragma unroll 4
            for (int i = 0; i + 1 < kDesc; ++i) {
                const double nxt = x[i + 1], m = L.mult[h][i];
                const bool swap = L.swapped[h][i] != 0;
                x[i] = swap ? nxt : cur;
                cur = swap ? cur - m * nxt : nxt - m * cur;
            }
            double y1 = 0.0, y2 = 0.0;  // elements i + 1 and i + 2
#pragma unroll 4
            for (int i = kDesc - 1; i >= 0; --i) {
                const double b = i == kDesc - 1 ? cur : x[i];
                const double y = (b - L.u1[h][i] * y1 - L.u2[h][i] * y2) * L.u0[h][i];
                x[i] = y;
                y2 = y1;
                y1 = y;
            }
        }
        __syncthreads();
        if (wv == 0) {  // unit vectors, each orthogonal to those before it
            double a[3], b[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                a[k] = L.x[k][lane];
                b[k] = L.x[k][lane + 64];
                auto unit = [&]() {
                    const double f = 1.0 / sqrt(wave_sum(a[k] * a[k] + b[k] * b[k]));
                    a[k] *= f;
                    b[k] *= f;
                };
                unit();
#pragma unroll
                for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
                    for (int j = 0; j < k; ++j) {
                        const double f = wave_sum(a[j] * a[k] + b[j] * b[k]);
                        a[k] -= f * a[j];
                        b[k] -= f * b[j];
                    }
                    if (k > 0) unit();
                }
                L.x[k][lane] = a[k];
                L.x[k][lane + 64] = b[k];
            }
        }
        __syncthreads();
    }
    if (wv < 3) {
        const int c1 = lane + 64;
        double y0 = L.x[wv][lane], y1 = L.x[wv][c1];
#pragma unroll 1
        for (int k = kDesc - 3; k >= 0; --k) {
            const double head = L.head[k];
            const double v0 = lane == k + 1 ? head : lane > k ? L.v[k][lane] : 0.0;
            const double v1 = c1 == k + 1 ? head : c1 > k ? L.v[k][c1] : 0.0;
            const double f = L.beta[k] * wave_sum(v0 * y0 + v1 * y1);
            y0 -= f * v0;
            y1 -= f * v1;
        }
        Y[wv][lane] = y0;
        Y[wv][c1] = y1;
    }
    __syncthreads();
}


// Eigenvalues and signed axes of a pair, in FP64 and (with the mean) FP32.
__device__ __forceinline__ void write_axes(int pair, const double (*Y)[kDesc], const double* th,
                                           const double* __restrict__ mean_all, double* __restrict__ eigval,
                                           double* __restrict__ axes, float* __restrict__ ax32) {
    const int t = threadIdx.x, lane = t & 63, k = wave_id();
    if (k < 3) {  // the first component of largest magnitude decides the sign
        double y0 = Y[k][lane], y1 = Y[k][lane + 64], m = fmax(fabs(y0), fabs(y1));
        for (int d = 1; d < 64; d <<= 1) m = fmax(m, __shfl_xor(m, d));
        const uint64_t b0 = __ballot(fabs(y0) == m), b1 = __ballot(fabs(y1) == m);
        const double top = b0 ? lane_double(y0, __builtin_ctzll(b0)) : b1 ? lane_double(y1, __builtin_ctzll(b1)) : 0.0;
        const double sg = top < 0.0 ? -1.0 : 1.0;
        y0 *= sg;
        y1 *= sg;
        const size_t o = ((size_t)pair * 3 + k) * kDesc + lane, o32 = ((size_t)pair * 4 + k) * kDesc + lane;
        axes[o] = y0;
        axes[o + 64] = y1;
        ax32[o32] = (float)y0;
        ax32[o32 + 64] = (float)y1;
        if (lane == 0) eigval[(size_t)pair * 3 + k] = th[k];
    }
    if (t < kDesc) ax32[((size_t)pair * 4 + 3) * kDesc + t] = (float)mean_all[(size_t)pair * kDesc + t];
}

// Bound: latency: four products (each 128 KB from beyond the L2s by one CU), seven
// small factorisations in one thread, one small eigenproblem.  KITTI-size pair: 62 us;
// 118 with 256 threads that each summed a row with 16 loads in flight (16 us a
// product).
constexpr int kEigRow = kDesc + 4;  // the rows' bank offsets differ
__global__ void __launch_bounds__(kEigThreads) eig_kernel(const double* __restrict__ cov_all,
                                                  const double* __restrict__ mean_all,
                                                  double* __restrict__ sq_all, double* __restrict__ eigval,
                                                  double* __restrict__ axes, float* __restrict__ ax32) {
    __shared__ double Q[kSub][kEigRow], Z[kSub][kEigRow], part[kEigParts][kSub][kDesc];
    __shared__ double G[kSub][kSub], Rinv[kSub][kSub], S[kSub][kSub], th[kSub];
    __shared__ double Y[3][kDesc], red[2][3][2];
    __shared__ int done;  // 1 converged, 2 to be solved directly
    const int t = threadIdx.x, pair = blockIdx.x;
    const double* A = cov_all + (size_t)pair * kDesc * kDesc;
    double* sq = sq_all + (size_t)pair * 2 * kDesc * kDesc;
    const int r = t & (kDesc - 1), h = t >> 7;  // row; part of a product's sum, pair of vectors

    // M = A^(2^kSquare), trace-normalised at each squaring (square_kernel)
    const double* M = sq + (size_t)((kSquare - 1) & 1) * kDesc * kDesc;

    // deterministic pseudo-random start
    for (int i = t; i < kSub * kDesc; i += kEigThreads) {
        uint32_t z = (uint32_t)(i + 1) * 2654435761u;
        z ^= z >> 15;
        z *= 2246822519u;
        z ^= z >> 13;
        Z[i / kDesc][i % kDesc] = (double)(z & 0xFFFF) / 32768.0 - 1.0;
    }
    __syncthreads();

    // G[i][j] = X_i . Y_j, four lanes to an entry
    auto inner = [&](const double (*X)[kEigRow], const double (*Y)[kEigRow]) {
        if (t >= 4 * kSub * kSub) return;
        const int i = t / (4 * kSub), j = t / 4 % kSub, q = t & 3;
        double s = 0.0;
#pragma unroll 8
        for (int k = q; k < kDesc; k += 4) s = fma(X[i][k], Y[j][k], s);
        s += __shfl_xor(s, 1);
        s += __shfl_xor(s, 2);
        if (q == 0) G[i][j] = s;
    };
    // Q = orth(Z) by Cholesky QR, twice
    auto orth = [&]() {
        for (int pass = 0; pass < 2; ++pass) {
            inner(Z, Z);
            __syncthreads();
            if (t == 0) chol_inverse(G, Rinv);
            __syncthreads();
            double z[kSub];
#pragma unroll
            for (int u = 0; u < kSub; ++u) z[u] = Z[u][r];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kSub / kEigParts; ++u) {
                const int vv = kSub / kEigParts * h + u;
                double s = 0.0;
#pragma unroll
                for (int w = 0; w < kSub; ++w)
                    if (w <= vv) s = fma(z[w], Rinv[w][vv], s);
                Z[vv][r] = s;
            }
            __syncthreads();
        }
#pragma unroll
        for (int u = 0; u < kSub / kEigParts; ++u) {
            const int vv = kSub / kEigParts * h + u;
            Q[vv][r] = Z[vv][r];
        }
        __syncthreads();
    };
    orth();

    for (int it = 1; it <= kMaxIter; ++it) {
        const bool check = it % kCheck == 0 || it == kMaxIter;
        const double* Mi = check ? A : M;
        {
            // thread (r, h): rows 32 h .. 32 h + 31 of the sum for all vectors, so the
            // loads of a product are in flight together
            constexpr int kn = kDesc / kEigParts;
            double m[kn], s[kSub] = {};
#pragma unroll
            for (int i = 0; i < kn; ++i) m[i] = Mi[(size_t)(kn * h + i) * kDesc + r];
#pragma unroll
            for (int i = 0; i < kn; ++i)
#pragma unroll
                for (int u = 0; u < kSub; ++u) s[u] = fma(m[i], Q[u][kn * h + i], s[u]);
#pragma unroll
            for (int u = 0; u < kSub; ++u) part[h][u][r] = s[u];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kSub / kEigParts; ++u) {
                const int vv = kSub / kEigParts * h + u;
                double z = part[0][vv][r];
#pragma unroll
                for (int i = 1; i < kEigParts; ++i) z += part[i][vv][r];
                Z[vv][r] = z;
            }
        }
        __syncthreads();
        if (check) {
            // Rayleigh-Ritz on A: T = Q^T (A Q)
            inner(Q, Z);
            __syncthreads();
            if (t < 64) ritz_small(G, th, S);
            __syncthreads();
            if (t < kDesc) {  // residuals and norms, squared, of two waves
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    double az = 0.0, y = 0.0;
#pragma unroll
                    for (int i = 0; i < kSub; ++i) {
                        az = fma(Z[i][t], S[i][k], az);
                        y = fma(Q[i][t], S[i][k], y);
                    }
                    const double e = az - th[k] * y;
                    const double e2 = wave_sum(e * e), y2 = wave_sum(y * y);
                    if ((t & 63) == 0) {
                        red[t >> 6][k][0] = e2;
                        red[t >> 6][k][1] = y2;
                    }
                }
            }
            __syncthreads();
            if (t == 0) {
                const double tol = 1e-12 * fabs(th[0]);
                bool unit = true, close = true;
                for (int k = 0; k < 3; ++k) {
                    close = close && sqrt(red[0][k][0] + red[1][k][0]) <= tol;
                    unit = unit && fabs(red[0][k][1] + red[1][k][1] - 1.0) < 1e-10;
                }
                // (a covariance that is all rounding is not positive: descriptors are unit vectors)
                done = unit && close && th[0] > 1e-13 ? 1 : !unit || !(th[2] > 0.8 * th[0]) || it == kMaxIter ? 2 : 0;
            }
            __syncthreads();
            if (done) break;
        }
        orth();
    }

    // the first squarings are used up: their place tells eig_direct_kernel whether it
    // is needed
    if (t == 0) sq[0] = done == 2 ? 1.0 : 0.0;
    if (done == 2) return;  // block-uniform
    // Ritz vectors y_k = Q s_k, signed, written out
    if (t < kDesc)
        for (int k = 0; k < 3; ++k) {
            double y = 0.0;
#pragma unroll
            for (int i = 0; i < kSub; ++i) y = fma(Q[i][t], S[i][k], y);
            Y[k][t] = y;
        }
    __syncthreads();
    write_axes(pair, Y, th, mean_all, eigval, axes, ax32);
}

// The pairs that eig_kernel leaves.
__global__ void __launch_bounds__(kEigThreads) eig_direct_kernel(const double* __restrict__ cov_all,
                                                                 const double* __restrict__ mean_all,
                                                                 const double* __restrict__ sq_all,
                                                                 double* __restrict__ eigval, double* __restrict__ axes,
                                                                 float* __restrict__ ax32) {
    __shared__ DirectLds lds;
    __shared__ double Y[3][kDesc], th[3];
    const int pair = blockIdx.x;
    if (sq_all[(size_t)pair * 2 * kDesc * kDesc] == 0.0) return;
    direct_eigen(cov_all + (size_t)pair * kDesc * kDesc, lds, th, Y);
    write_axes(pair, Y, th, mean_all, eigval, axes, ax32);
}

// phi = axes (f - mean) per pixel of the pair's four images, float4 (phi, 0).
// A lane keeps its quarter of the three axes and the mean in registers (128
// values) for all the pixels it projects; loaded for every pixel they were four
// fifths of the kernel's reads (442 us on a KITTI-size pair).  Two waves per SIMD.
constexpr int kProjBlocks = 512;  // per pair at most: two blocks per CU
__global__ void __launch_bounds__(256, 2) project_kernel(const float* __restrict__ Cs,
                                                         const float* __restrict__ ax32,
                                                         float4* __restrict__ phi, int H, int W) {
    const int He = H + kExt, We = W + kExt;
    const int t = threadIdx.x, q = t & 3;
    const int npx = H * W, total = 4 * npx;
    const int pair = blockIdx.y;
    const float* ax = ax32 + (size_t)pair * 4 * kDesc + 32 * q;
    float A[4][32];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int k = 0; k < 32; ++k) A[c][k] = ax[c * kDesc + k];
#pragma unroll 1
    for (int base = blockIdx.x * kGramPx; base < total; base += gridDim.x * kGramPx) {
        const int g = base + (t >> 2), ge = min(g, total - 1);
        int m, y, x;
        desc_pixel(ge, npx, W, m, y, x);
        float v[32];
        desc_quarter(Cs + ((size_t)pair * 4 + m) * kBins * He * We, We, y, x, q, v);
        float f[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            const float d = v[k] - A[3][k];
#pragma unroll
            for (int c = 0; c < 3; ++c) f[c] = fmaf(A[c][k], d, f[c]);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) f[c] = quad_sum(f[c]);
        if (g < total && q == 0) phi[(size_t)pair * total + ge] = make_float4(f[0], f[1], f[2], 0.f);
    }
}

// ------------------------------------------------------------------ cost --

// Euclidean distance of the first three components, every operation rounded
// as written (no contraction), so that sums agree bit for bit with the FP32
// definition: ((e0^2 + e1^2) + e2^2), correctly rounded square root.  sqrtf
// is correctly rounded in this toolchain's default FP32 mode (a committed test
// checks it against the host); __fsqrt_rn is not (15% of 2^20 inputs differ by
// an ulp).  HIP contracts multiply-adds by default (the __f*_rn helpers
// included): switched off here, with plain operators under the pragma.
__device__ __forceinline__ float fdist3(float4 a, float4 b) {
#pragma clang fp contract(off)
    const float e0 = a.x - b.x, e1 = a.y - b.y, e2 = a.z - b.z;
    float q = e0 * e0;
    q = q + e1 * e1;
    q = q + e2 * e2;
    return sqrtf(q);
}

// Views of one field: (R, T, S, X) = (l0, l1, r0, r1) for s = +1 and
// (r1, r0, l1, l0) for s = -1.
struct SiftViews {
    const float4 *R, *T, *S, *X;
    int H, W, s;
};

__device__ __forceinline__ SiftViews sift_views(const float4* phi_pair, int H, int W, int s) {
    const size_t npx = (size_t)H * W;
    SiftViews V;
    V.R = phi_pair + (size_t)(s > 0 ? 0 : 3) * npx;
    V.T = phi_pair + (size_t)(s > 0 ? 1 : 2) * npx;
    V.S = phi_pair + (size_t)(s > 0 ? 2 : 1) * npx;
    V.X = phi_pair + (size_t)(s > 0 ? 3 : 0) * npx;
    V.H = H;
    V.W = W;
    V.s = s;
    return V;
}

// Eq. (1) of (u, v, d0, d1) at (x, y): window rows wy = -3..3, columns wx, and
// for each window pixel the temporal, stereo and cross distances, added in
// that order.  The terms are non-negative, so the partial sum only grows: once
// it reaches `bound` after a window row the remaining rows are skipped and a
// value >= bound is returned; below `bound` the exact sum is returned.
__device__ __forceinline__ float sift_cost_below(const SiftViews& V, int x, int y, int u, int v, int d0,
                                                 int d1, float bound) {
    const int H = V.H, W = V.W, s = V.s;
    float sum = 0.f;
    for (int wy = -kWinR; wy <= kWinR; ++wy) {
        const int py = y + wy;
        const size_t rr = (size_t)clampi(py, 0, H - 1) * W, rv = (size_t)clampi(py + v, 0, H - 1) * W;
#pragma unroll
        for (int wx = -kWinR; wx <= kWinR; ++wx) {
            const int px = x + wx;
            const float4 r = V.R[rr + clampi(px, 0, W - 1)];
            const float4 t = V.T[rv + clampi(px + u, 0, W - 1)];
            const float4 sv = V.S[rr + clampi(px - s * d0, 0, W - 1)];
            const float4 xv = V.X[rv + clampi(px + u - s * d1, 0, W - 1)];
            sum = sum + fdist3(r, t);
            sum = sum + fdist3(r, sv);
            sum = sum + fdist3(r, xv);
        }
        if (sum >= bound) return sum;
    }
    return sum;
}

// Eq. (1) at fixed vectors: one thread per pixel of a 16 x 16 tile.
__global__ void __launch_bounds__(256) cost_sift_kernel(const float4* __restrict__ phi,
                                                        const int16_t* __restrict__ hyp,
                                                        float* __restrict__ cost, int H, int W, int dir) {
    const int b = blockIdx.z;
    const size_t npx = (size_t)H * W;
    const SiftViews V = sift_views(phi + (size_t)b * 4 * npx, H, W, dir);
    const int y = blockIdx.y * kCT + threadIdx.x / kCT, x = blockIdx.x * kCT + threadIdx.x % kCT;
    if (y >= H || x >= W) return;
    const short4 h = reinterpret_cast<const short4*>(hyp)[(size_t)b * npx + (size_t)y * W + x];
    cost[(size_t)b * npx + (size_t)y * W + x] = sift_cost_below(V, x, y, h.x, h.y, h.z, h.w, INFINITY);
}

// Full-resolution matching with eq. (1) (Section 3.1, "Multi-Scale
// Propagation" at the finest scale): one red-black half-step of both fields.
// Per-lane form (SFF_SIFT_EVAL=lane; the wave-shared form follows further
// down): block = 4 image rows x 64 pixels of the half-step's colour; each lane
// scores its own candidates (left, up, right, down, then the random-search
// samples, one at a time, strict improvement).  Random stream: Philox4x32-10
// with the counter's level field 16 and radii R0 >> t.
struct SiftMatchArgs {
    const float4* phi;       // [batch][4][H][W]
    const uint64_t* seeds;   // [batch]
    int16_t* hyp;            // [ndir][batch][H][W][4]
    float* cost;             // [ndir][batch][H][W]
    int H, W, rs_r0, rs_samples, fmax, dmax, batch, ndir, dir0;
};

constexpr uint32_t kSiftLevelTag = 16;

__global__ void __launch_bounds__(256) sift_cost_init_kernel(SiftMatchArgs a) {
    const int z = blockIdx.y, di = z / a.batch, b = z - di * a.batch;
    const int s = a.ndir == 2 ? (di == 0 ? 1 : -1) : a.dir0;
    const size_t npx = (size_t)a.H * a.W;
    const int p = blockIdx.x * 256 + threadIdx.x;
    if ((size_t)p >= npx) return;
    const SiftViews V = sift_views(a.phi + (size_t)b * 4 * npx, a.H, a.W, s);
    const short4 h = reinterpret_cast<const short4*>(a.hyp)[(size_t)z * npx + p];
    a.cost[(size_t)z * npx + p] = sift_cost_below(V, p % a.W, p / a.W, h.x, h.y, h.z, h.w, INFINITY);
}

__global__ void __launch_bounds__(256) sift_half_step_kernel(SiftMatchArgs a, int it, int colour, int tiles_x,
                                                             int tiles_y) {
    const int per_field = tiles_x * tiles_y;
    const int z = blockIdx.x / per_field;
    const int tr = blockIdx.x - z * per_field;
    const int ty = tr / tiles_x, tx = tr - ty * tiles_x;
    const int lane = threadIdx.x & 63;
    const int i = ty * 4 + wave_id();
    if (i >= a.H) return;  // whole wave
    const int j = 2 * (tx * 64 + lane) + ((i + colour) & 1);
    const bool act = j < a.W;
    const int jj = min(j, a.W - 1);
    const int di = z / a.batch, b = z - di * a.batch;
    const int s = a.ndir == 2 ? (di == 0 ? 1 : -1) : a.dir0;
    const size_t npx = (size_t)a.H * a.W;
    const SiftViews V = sift_views(a.phi + (size_t)b * 4 * npx, a.H, a.W, s);
    short4* field = reinterpret_cast<short4*>(a.hyp) + (size_t)z * npx;
    float* cost = a.cost + (size_t)z * npx;
    const size_t o = (size_t)i * a.W + jj;
    short4 best = field[o];
    float bestc = cost[o];
    const short4 own = best;
    const int ni[4] = {i, i - 1, i, i + 1};
    const int nj[4] = {jj - 1, jj, jj + 1, jj};
    short4 nh[4];
    bool in[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        in[q] = act && ni[q] >= 0 && ni[q] < a.H && nj[q] >= 0 && nj[q] < a.W;
        nh[q] = in[q] ? field[(size_t)ni[q] * a.W + nj[q]] : own;
    }
    auto eq = [](short4 p, short4 q) { return p.x == q.x && p.y == q.y && p.z == q.z && p.w == q.w; };
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        // a vector equal to one already scored has the same cost: no strict improvement
        bool dup = eq(nh[q], own);
#pragma unroll
        for (int p = 0; p < q; ++p) dup = dup || (in[p] && eq(nh[q], nh[p]));
        const bool want = in[q] && !dup;
        if (!__any(want)) continue;
        if (want) {
            const float c = sift_cost_below(V, jj, i, nh[q].x, nh[q].y, nh[q].z, nh[q].w, bestc);
            if (c < bestc) {
                bestc = c;
                best = nh[q];
            }
        }
    }
    const short4 centre = best;
    const uint64_t seed = a.seeds[b];
    for (int t = 0; t < a.rs_samples; ++t) {
        const int r = max(1, a.rs_r0 >> t);
        U4 ctr;
        ctr.x = (uint32_t)(i * a.W + jj);
        ctr.y = (uint32_t)it;
        ctr.z = (kSiftLevelTag << 16) | ((uint32_t)t << 8) | (s < 0 ? 1u : 0u);
        ctr.w = 0u;
        const U4 rnd = philox4x32_10(ctr, (uint32_t)seed, (uint32_t)(seed >> 32));
        short4 c;
        c.x = (short)clampi(centre.x + uniform_offset(rnd.x, r), -a.fmax, a.fmax);
        c.y = (short)clampi(centre.y + uniform_offset(rnd.y, r), -a.fmax, a.fmax);
        c.z = (short)clampi(centre.z + uniform_offset(rnd.z, r), 0, a.dmax);
        c.w = (short)clampi(centre.w + uniform_offset(rnd.w, r), 0, a.dmax);
        const bool want = act && !eq(c, centre);
        if (!__any(want)) continue;
        if (want) {
            const float cc = sift_cost_below(V, jj, i, c.x, c.y, c.z, c.w, bestc);
            if (cc < bestc) {
                bestc = cc;
                best = c;
            }
        }
    }
    if (act) {
        field[o] = best;
        cost[o] = bestc;
    }
}

// Window gathers shared by the wave (64 pixels of one image row).  Per window
// row, slot f = 64 k + lane (k < 7) serves owner f / 7 at window column
// f % 7 - 3: it loads that column's R, T, S and X elements (the 7 columns of one
// owner are consecutive lanes, so a load instruction reads a few contiguous runs
// instead of 64 scattered elements) and writes the three distances to LDS; the
// owner then adds its 21 distances in the per-lane kernel's order (column, then
// temporal, stereo, cross), so every sum is the same FP32 value, and stops
// after the first row whose partial sum reaches the bound.  Tiles are
// numbered column-major and dealt to the XCDs in vertical strips, which keeps
// the window gathers of neighbouring tiles in one L2 (KITTI-size pair: one
// matching iteration 1.72 vs 2.45 ms with tiles dealt in launch order).
constexpr int kSiftSlots = 2 * kWinR + 1;           // slot loads per window row
constexpr int kDistStride = 3 * kSiftSlots + 3;     // 24 floats per owner in LDS

__device__ __forceinline__ void sift_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct SiftCoop {
    SiftViews V;
    float* dist;              // this wave's LDS [64][kDistStride]
    int lane, y;
    int so[kSiftSlots];       // owner of slot k
    int sx[kSiftSlots];       // x of the slot's window column (owner's x + offset)
    int sd[kSiftSlots];       // LDS word of the slot's first distance

    // Eq. (1) of each owner's (u, v, d0, d1) at its pixel (x_o, y), the same
    // value as sift_cost_below (>= bound once a row's partial sum reaches it).
    // want = false: no candidate, result meaningless.  Called by all lanes.
    __device__ __forceinline__ float cost_below(bool want, short4 h, float bound) const {
        const int H = V.H, W = V.W, s = V.s;
        const uint32_t uv = (uint32_t)(uint16_t)h.x | ((uint32_t)(uint16_t)h.y << 16);
        const uint32_t dd = (uint32_t)(uint16_t)h.z | ((uint32_t)(uint16_t)h.w << 16);
        int su[kSiftSlots], svv[kSiftSlots], sd0[kSiftSlots], sd1[kSiftSlots];
#pragma unroll
        for (int k = 0; k < kSiftSlots; ++k) {
            const uint32_t a = (uint32_t)__shfl((int)uv, so[k]), b = (uint32_t)__shfl((int)dd, so[k]);
            su[k] = (int)(int16_t)(a & 0xFFFFu);
            svv[k] = (int)(int16_t)(a >> 16);
            sd0[k] = (int)(int16_t)(b & 0xFFFFu);
            sd1[k] = (int)(int16_t)(b >> 16);
        }
        float sum = 0.f;
        bool alive = want;
        for (int wy = -kWinR; wy <= kWinR; ++wy) {
            if (!__any(alive)) break;
            const int py = clampi(y + wy, 0, H - 1);
#pragma unroll
            for (int k = 0; k < kSiftSlots; ++k) {
                if (__shfl((int)alive, so[k])) {
                    const int pyv = clampi(y + wy + svv[k], 0, H - 1);
                    const int px = sx[k];
                    const float4 r = V.R[py * W + clampi(px, 0, W - 1)];
                    const float4 t = V.T[pyv * W + clampi(px + su[k], 0, W - 1)];
                    const float4 sv = V.S[py * W + clampi(px - s * sd0[k], 0, W - 1)];
                    const float4 xv = V.X[pyv * W + clampi(px + su[k] - s * sd1[k], 0, W - 1)];
                    dist[sd[k] + 0] = fdist3(r, t);
                    dist[sd[k] + 1] = fdist3(r, sv);
                    dist[sd[k] + 2] = fdist3(r, xv);
                }
            }
            sift_wave_sync();
            if (alive) {
                const float* d = dist + lane * kDistStride;
#pragma unroll
                for (int e = 0; e < 3 * kSiftSlots; ++e) sum = sum + d[e];
                alive = sum < bound;
            }
            sift_wave_sync();
        }
        return sum;
    }
};

// The half-step with the window gathers shared by the wave as above, and the
// costs compared by estimates.  A candidate is taken only if its exact FP32 sum
// (the per-lane kernel's, every operation rounded in its order) is below the
// current vector's; the estimate forms the same 147 distances with fused
// multiply-adds and the hardware root (a quarter of the operations of the exact
// one) and adds them in whatever order is cheapest (a slot keeps its own sum
// over the window rows, an owner adds 7 of them).  It is within 32 u of the true
// sum, the exact one within 150 u of it (u = 2^-24), so the exact sum lies within
// 2^-15 of the estimate, and disjoint intervals decide a comparison.  Where they
// overlap (ties, mostly) both sums are formed exactly, and so is, once at the
// end, the cost of a vector that was taken; 9 owners at a time (63 lanes, one per
// owner and window column).  Estimates that are infinite, or so small that a
// subnormal square could matter, decide nothing; a NaN estimate means a NaN sum,
// which is never taken.  Partial sums are lower bounds, looked at after the last
// four window rows (6.2 of the 7 rows are needed on average on a KITTI-size pair,
// so earlier looks cost more than they save).
// A block is 4 waves on 4 consecutive rows; the reference elements their windows
// read (10 x 134) are staged in LDS once, clamped, for all candidates, so a slot
// gathers three elements of 12 bytes per window row.
// Bound: the texture data path (three gathers of 64 x 12 bytes, ~20 cache
// accesses each, per slot and window row: 83 % busy), the vector ALU at 55 %.
// KITTI-size pair, both fields: 574 us per half-step, where exact sums of all
// candidates with four gathers took 753 us (one matching iteration with them 1.43
// -> 1.12 ms); three and four waves per SIMD (168 and 128 VGPRs) spill: 9.2 and
// 11.0 ms per 6 iterations against 8.0 ms, measured with an earlier form.
constexpr int kHsRows = 4;                                  // image rows (waves) per block
constexpr int kHsCols = 2 * 63 + 1 + 1 + 2 * kWinR;         // reference columns of a tile
constexpr int kExactOwners = 64 / kSiftSlots;               // 9
constexpr int kExactRows = 4;                               // window rows summed per pass over LDS
constexpr int kExactStride = kExactRows * 3 * kSiftSlots;   // floats per owner
constexpr int kHsSlice = kSiftSlots * 64;                   // floats of a wave's slice (estimate sums)
static_assert(kExactOwners * kExactStride + 16 <= 2 * kHsSlice, "wave slice");
constexpr int kNoElement = 0x7FFFFFF0;                      // offset past every image's map
constexpr float kEstimateErr = 0x1p-15f;

typedef float v3f __attribute__((ext_vector_type(3)));

// Raw buffer descriptor of one image's features (wave-uniform): loads at or past
// its size return zeros without a memory access.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t phi_rsrc(const float4* p, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), (short)0,
                                             (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

__device__ __forceinline__ v3f load3(__amdgpu_buffer_rsrc_t rs, int off, int soff) {
    return __builtin_bit_cast(v3f, __builtin_amdgcn_raw_buffer_load_b96(rs, off, soff, 0));
}

// Distance for the estimate: fused, hardware root (1 ulp).
__device__ __forceinline__ float fdist3_fast(v3f a, v3f b) {
    const float e0 = a.x - b.x, e1 = a.y - b.y, e2 = a.z - b.z;
    return __builtin_amdgcn_sqrtf(fmaf(e2, e2, fmaf(e1, e1, e0 * e0)));
}

struct SiftHalf {
    __amdgpu_buffer_rsrc_t rT, rS, rX;
    const float4* ref;  // the block's reference tile in LDS, at the wave's first window row
    float* slice;       // this wave's LDS [2 kHsSlice]
    int H, W, s, y, lane, x0, par;

    // Window column (slot f of the 64 owners): owner, x, and the vector handed over.
    struct Column {
        int xt, xs, xx, yv, lc;
    };
    __device__ __forceinline__ Column column(int o, int c, uint32_t uv, uint32_t dd, bool use) const {
        const int u = (int)(int16_t)(uv & 0xFFFFu), v = (int)(int16_t)(uv >> 16);
        const int d0 = (int)(int16_t)(dd & 0xFFFFu), d1 = (int)(int16_t)(dd >> 16);
        Column q;
        q.lc = 2 * o + par + c;
        const int px = x0 - kWinR + q.lc;
        q.xt = use ? clampi(px + u, 0, W - 1) * 16 : kNoElement;
        q.xs = use ? clampi(px - s * d0, 0, W - 1) * 16 : kNoElement;
        q.xx = use ? clampi(px + u - s * d1, 0, W - 1) * 16 : kNoElement;
        q.yv = y + v;
        return q;
    }
    __device__ __forceinline__ void load_row(const Column& q, int wy, v3f& r, v3f& t, v3f& sv, v3f& xv) const {
        const uint32_t row = (uint32_t)clampi(q.yv + wy, 0, H - 1), W16 = (uint32_t)W * 16u;
        const float4 rr = ref[(wy + kWinR) * kHsCols + q.lc];
        r = v3f{rr.x, rr.y, rr.z};
        t = load3(rT, (int)(__umul24(row, W16) + (uint32_t)q.xt), 0);
        sv = load3(rS, q.xs, clampi(y + wy, 0, H - 1) * W * 16);
        xv = load3(rX, (int)(__umul24(row, W16) + (uint32_t)q.xx), 0);
    }

    // Estimate of the cost of each owner's candidate h, [lo, hi] around the
    // exact sum.  A lane ends early (lo >= bound) once a partial sum says so;
    // lo = infinity without a candidate.  Called by all lanes.
    __device__ __forceinline__ void estimate(bool want, short4 h, float bound, float& lo, float& hi) const {
        const uint32_t uv = (uint32_t)(uint16_t)h.x | ((uint32_t)(uint16_t)h.y << 16);
        const uint32_t dd = (uint32_t)(uint16_t)h.z | ((uint32_t)(uint16_t)h.w << 16);
        uint64_t open = __ballot(want);
        Column q[kSiftSlots];
        float acc[kSiftSlots];
#pragma unroll
        for (int k = 0; k < kSiftSlots; ++k) {
            const int f = 64 * k + lane, o = f / kSiftSlots;
            q[k] = column(o, f - kSiftSlots * o, (uint32_t)__shfl((int)uv, o), (uint32_t)__shfl((int)dd, o),
                          (open >> o) & 1);
            acc[k] = 0.f;
        }
        lo = hi = INFINITY;
        // rows -3 .. 0, then one at a time: few sums reach the bound earlier
#pragma unroll 1
        for (int wy = -kWinR; wy <= kWinR; ++wy) {
            v3f r[kSiftSlots], t[kSiftSlots], sv[kSiftSlots], xv[kSiftSlots];
#pragma unroll
            for (int k = 0; k < kSiftSlots; ++k) load_row(q[k], wy, r[k], t[k], sv[k], xv[k]);
#pragma unroll
            for (int k = 0; k < kSiftSlots; ++k) {
                acc[k] += fdist3_fast(r[k], t[k]);
                acc[k] += fdist3_fast(r[k], sv[k]);
                acc[k] += fdist3_fast(r[k], xv[k]);
            }
            if (wy < 0) continue;
#pragma unroll
            for (int k = 0; k < kSiftSlots; ++k) slice[64 * k + lane] = acc[k];
            sift_wave_sync();
            float sum = 0.f;
#pragma unroll
            for (int c = 0; c < kSiftSlots; ++c) sum += slice[kSiftSlots * lane + c];
            sift_wave_sync();
            if (want && ((open >> lane) & 1)) {
                const bool sure = sum > 1e-10f && sum < INFINITY;
                lo = sure ? sum * (1.f - kEstimateErr) : sum != sum ? INFINITY : 0.f;  // NaN: never taken
                hi = sure ? sum * (1.f + kEstimateErr) : INFINITY;
            }
            open = __ballot(lo < bound);
            if (open == 0) return;
#pragma unroll
            for (int k = 0; k < kSiftSlots; ++k)  // owners turned down gather nothing more
                if (!((open >> ((64 * k + lane) / kSiftSlots)) & 1)) q[k].xt = q[k].xs = q[k].xx = kNoElement;
        }
    }

    // The exact sums of the owners in `open` (eq. (1), sift_cost_below's value
    // without its early end); meaningless in the other lanes.
    __device__ __forceinline__ float exact(bool open, short4 h) const {
        const uint32_t uv = (uint32_t)(uint16_t)h.x | ((uint32_t)(uint16_t)h.y << 16);
        const uint32_t dd = (uint32_t)(uint16_t)h.z | ((uint32_t)(uint16_t)h.w << 16);
        uint32_t* list = reinterpret_cast<uint32_t*>(slice + kExactOwners * kExactStride);
        const int j = lane / kSiftSlots, c = lane - kSiftSlots * j;
        float sum = 0.f;
        uint64_t left = __ballot(open);
        while (left) {
            const int rank = __popcll(left & ((1ull << lane) - 1ull));
            const bool mine = ((left >> lane) & 1) && rank < kExactOwners;
            if (mine) list[rank] = (uint32_t)lane;
            sift_wave_sync();
            const bool serve = j < min(kExactOwners, __popcll(left));
            const int o = serve ? (int)list[j] : 0;
            const Column q = column(o, c, (uint32_t)__shfl((int)uv, o), (uint32_t)__shfl((int)dd, o), serve);
#pragma unroll
            for (int w0 = -kWinR; w0 <= kWinR; w0 += kExactRows) {
                v3f r[kExactRows], t[kExactRows], sv[kExactRows], xv[kExactRows];
#pragma unroll
                for (int e = 0; e < kExactRows; ++e)
                    if (w0 + e <= kWinR) load_row(q, w0 + e, r[e], t[e], sv[e], xv[e]);
#pragma unroll
                for (int e = 0; e < kExactRows; ++e)
                    if (w0 + e <= kWinR && serve) {
                        float* d = slice + j * kExactStride + e * 3 * kSiftSlots + 3 * c;
                        const float4 a = make_float4(r[e].x, r[e].y, r[e].z, 0.f);
                        d[0] = fdist3(a, make_float4(t[e].x, t[e].y, t[e].z, 0.f));
                        d[1] = fdist3(a, make_float4(sv[e].x, sv[e].y, sv[e].z, 0.f));
                        d[2] = fdist3(a, make_float4(xv[e].x, xv[e].y, xv[e].z, 0.f));
                    }
                sift_wave_sync();
                if (mine) {
                    const float* d = slice + rank * kExactStride;
#pragma unroll
                    for (int e = 0; e < 3 * kSiftSlots * kExactRows; ++e)
                        if (w0 + e / (3 * kSiftSlots) <= kWinR) sum = sum + d[e];
                }
                sift_wave_sync();
            }
            left &= ~__ballot(mine);
        }
        return sum;
    }
};

__global__ void __launch_bounds__(64 * kHsRows) sift_half_step_wave_kernel(SiftMatchArgs a, int it, int colour,
                                                                           int tiles_x, int tiles_y) {
    __shared__ float4 ref_lds[(kHsRows + 2 * kWinR) * kHsCols];
    __shared__ float slices[kHsRows][2 * kHsSlice];
    const int per_field = tiles_x * tiles_y;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);  // column-major tiles, a strip per XCD
    const int z = tile / per_field;
    const int tr = tile - z * per_field;
    const int tx = tr / tiles_y, i0 = (tr - tx * tiles_y) * kHsRows;
    const int di = z / a.batch, b = z - di * a.batch;
    const int s = a.ndir == 2 ? (di == 0 ? 1 : -1) : a.dir0;
    const size_t npx = (size_t)a.H * a.W;
    const SiftViews V = sift_views(a.phi + (size_t)b * 4 * npx, a.H, a.W, s);
    for (int e = threadIdx.x; e < (kHsRows + 2 * kWinR) * kHsCols; e += 64 * kHsRows) {
        const int r = e / kHsCols, c = e - r * kHsCols;
        ref_lds[e] = V.R[(size_t)clampi(i0 - kWinR + r, 0, a.H - 1) * a.W + clampi(2 * tx * 64 - kWinR + c, 0, a.W - 1)];
    }
    __syncthreads();
    const int w = wave_id(), i = i0 + w;
    if (i >= a.H) return;  // whole wave, after the block's only barrier
    const int lane = threadIdx.x & 63;
    const int par = (i + colour) & 1;
    const int j = 2 * (tx * 64 + lane) + par;
    const bool act = j < a.W;
    const int jj = min(j, a.W - 1);
    SiftHalf E;
    const uint32_t bytes = (uint32_t)(npx * 16);
    E.rT = phi_rsrc(V.T, bytes);
    E.rS = phi_rsrc(V.S, bytes);
    E.rX = phi_rsrc(V.X, bytes);
    E.ref = ref_lds + w * kHsCols;
    E.slice = slices[w];
    E.H = a.H;
    E.W = a.W;
    E.s = s;
    E.y = i;
    E.lane = lane;
    E.x0 = 2 * tx * 64;
    E.par = par;
    short4* field = reinterpret_cast<short4*>(a.hyp) + (size_t)z * npx;
    float* cost = a.cost + (size_t)z * npx;
    const size_t o = (size_t)i * a.W + jj;
    short4 best = field[o];
    const float bestc = cost[o];
    const short4 own = best;
    const int ni[4] = {i, i - 1, i, i + 1};
    const int nj[4] = {jj - 1, jj, jj + 1, jj};
    short4 nh[4];
    bool in[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        in[q] = act && ni[q] >= 0 && ni[q] < a.H && nj[q] >= 0 && nj[q] < a.W;
        nh[q] = in[q] ? field[(size_t)ni[q] * a.W + nj[q]] : own;
    }
    auto eq = [](short4 p, short4 q) { return p.x == q.x && p.y == q.y && p.z == q.z && p.w == q.w; };
    // the current vector's cost lies in [blo, bhi] (both its exact cost at first)
    float blo = bestc, bhi = bestc;
    auto score = [&](bool want, short4 h) {
        want = want && bhi > 0.f;  // a cost of zero (or NaN) cannot be improved on
        if (!__any(want)) return;
        float lo, hi;
        E.estimate(want, h, bhi, lo, hi);
        bool take = want && hi < blo;
        const bool close = want && !take && lo < bhi;  // the estimates do not decide
        if (__any(close)) {
            const bool redo = close && blo < bhi;
            const float eb = E.exact(redo, best);
            if (redo) blo = bhi = eb;
            const float eh = E.exact(close, h);
            if (close && eh < bhi) {
                take = true;
                lo = hi = eh;
            }
        }
        if (take) {
            blo = lo;
            bhi = hi;
            best = h;
        }
    };
    const short4 n0 = nh[0], n1 = nh[1], n2 = nh[2], n3 = nh[3];
    // a vector equal to one already scored has the same cost: no strict improvement
    const bool w0 = in[0] && !eq(n0, own);
    const bool w1 = in[1] && !eq(n1, own) && !(in[0] && eq(n1, n0));
    const bool w2 = in[2] && !eq(n2, own) && !(in[0] && eq(n2, n0)) && !(in[1] && eq(n2, n1));
    const bool w3 = in[3] && !eq(n3, own) && !(in[0] && eq(n3, n0)) && !(in[1] && eq(n3, n1)) && !(in[2] && eq(n3, n2));
    short4 centre = best;
    const uint64_t seed = a.seeds[b];
#pragma unroll 1
    for (int t = -4; t < a.rs_samples; ++t) {  // left, up, right, down, then the samples
        short4 c;
        bool want;
        if (t < 0) {
            c = t == -4 ? n0 : t == -3 ? n1 : t == -2 ? n2 : n3;
            want = t == -4 ? w0 : t == -3 ? w1 : t == -2 ? w2 : w3;
        } else {
            if (t == 0) centre = best;
            const int r = max(1, a.rs_r0 >> t);
            U4 ctr;
            ctr.x = (uint32_t)(i * a.W + jj);
            ctr.y = (uint32_t)it;
            ctr.z = (kSiftLevelTag << 16) | ((uint32_t)t << 8) | (s < 0 ? 1u : 0u);
            ctr.w = 0u;
            const U4 rnd = philox4x32_10(ctr, (uint32_t)seed, (uint32_t)(seed >> 32));
            c.x = (short)clampi(centre.x + uniform_offset(rnd.x, r), -a.fmax, a.fmax);
            c.y = (short)clampi(centre.y + uniform_offset(rnd.y, r), -a.fmax, a.fmax);
            c.z = (short)clampi(centre.z + uniform_offset(rnd.z, r), 0, a.dmax);
            c.w = (short)clampi(centre.w + uniform_offset(rnd.w, r), 0, a.dmax);
            want = act && !eq(c, centre);
        }
        score(want, c);
    }
    const bool redo = act && blo < bhi;
    const float eb = E.exact(redo, best);
    if (act) {
        field[o] = best;
        cost[o] = redo ? eb : blo;
    }
}

// Eq. (1) at fixed vectors with the wave-shared gathers: 64 consecutive
// pixels of one row per wave (block), every field z of hyp/cost ([ndir][batch]
// or [batch]) in one launch; the same values as sift_cost_below.
__global__ void __launch_bounds__(64) sift_cost_coop_kernel(SiftMatchArgs a, int tiles_x) {
    __shared__ float dist_lds[64 * kDistStride];
    const int per_field = tiles_x * a.H;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);  // column-major tiles, a strip per XCD
    const int z = tile / per_field;
    const int tr = tile - z * per_field;
    const int tx = tr / a.H, i = tr - tx * a.H;
    const int lane = threadIdx.x;
    const int j = tx * 64 + lane;
    const bool act = j < a.W;
    const int jj = min(j, a.W - 1);
    const int di = z / a.batch, b = z - di * a.batch;
    const int s = a.ndir == 2 ? (di == 0 ? 1 : -1) : a.dir0;
    const size_t npx = (size_t)a.H * a.W;
    SiftCoop E;
    E.V = sift_views(a.phi + (size_t)b * 4 * npx, a.H, a.W, s);
    E.dist = dist_lds;
    E.lane = lane;
    E.y = i;
#pragma unroll
    for (int k = 0; k < kSiftSlots; ++k) {
        const int f = 64 * k + lane, o = f / kSiftSlots, c = f - kSiftSlots * o;
        E.so[k] = o;
        E.sx[k] = min(tx * 64 + o, a.W - 1) + c - kWinR;
        E.sd[k] = o * kDistStride + 3 * c;
    }
    const size_t o = (size_t)z * npx + (size_t)i * a.W + jj;
    const short4 h = reinterpret_cast<const short4*>(a.hyp)[o];
    const float c = E.cost_below(act, h, INFINITY);
    if (act) a.cost[o] = c;
}

// The cost's square root (sqrtf) over an array, to check its rounding.
__global__ void __launch_bounds__(256) sift_sqrt_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                        int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) out[i] = sqrtf(in[i]);
}

bool sift_shape_ok(const sff_params* p, int64_t nimg) {
    if (!params_ok(p) || nimg < 1) return false;
    // flattened indices stay below 2^31 in every kernel
    return nimg * (int64_t)(p->H + kExt) * (p->W + kExt) * kBins < (int64_t(1) << 31);
}

void launch_cells(const SiftGeom& g, int nimg, int C, const uint8_t* img, float* Cs, hipStream_t st) {
    hipLaunchKernelGGL(cellsum_kernel, dim3((g.We + kCellX - 1) / kCellX, (g.He + kCellY - 1) / kCellY, nimg),
                       dim3(256), 0, st, img, Cs, g.H, g.W, C);
}

}  // namespace
}  // namespace sff

using namespace sff;

extern "C" size_t sff_sift_workspace_bytes(const sff_params* p, int32_t nimg) {
    if (!sift_shape_ok(p, nimg)) return 0;
    return sift_ws(sift_geom(*p), nimg).total;
}

extern "C" sff_status sff_dense_sift(const sff_params* p, int32_t nimg, const uint8_t* img, float* sift,
                                     void* workspace, size_t workspace_bytes, void* stream) {
    if (!sift_shape_ok(p, nimg) || !img || !sift || (reinterpret_cast<uintptr_t>(sift) & 15) != 0)
        return SFF_ERR_INVALID_ARG;
    const SiftGeom g = sift_geom(*p);
    const SiftWs L = sift_ws(g, nimg);
    if (!workspace || workspace_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return SFF_ERR_WORKSPACE;
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    float* Cs = reinterpret_cast<float*>(ws + L.Cs);
    hipStream_t st = as_stream(stream);
    launch_cells(g, nimg, p->C, img, Cs, st);
    const long total = (long)nimg * g.npx;
    hipLaunchKernelGGL(sift_out_kernel, dim3((unsigned)((total + kGramPx - 1) / kGramPx)), dim3(256), 0, st,
                       Cs, sift, g.H, g.W, nimg);
    return launch_status();
}

extern "C" sff_status sff_sift_pca(const sff_params* p, int32_t batch, const uint8_t* imgs, double* mean,
                                   double* cov, double* eigval, double* axes, float* phi, void* workspace,
                                   size_t workspace_bytes, void* stream) {
    if (batch < 1 || batch > 65535 || !sift_shape_ok(p, 4 * (int64_t)batch) || !imgs || !mean || !cov ||
        !eigval || !axes || !phi)
        return SFF_ERR_INVALID_ARG;
    if (((reinterpret_cast<uintptr_t>(mean) | reinterpret_cast<uintptr_t>(cov) |
          reinterpret_cast<uintptr_t>(eigval) | reinterpret_cast<uintptr_t>(axes)) & 7) != 0 ||
        (reinterpret_cast<uintptr_t>(phi) & 15) != 0)
        return SFF_ERR_INVALID_ARG;
    const SiftGeom g = sift_geom(*p);
    const int nimg = 4 * batch;
    const SiftWs L = sift_ws(g, nimg);
    if (!workspace || workspace_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return SFF_ERR_WORKSPACE;
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    float* Cs = reinterpret_cast<float*>(ws + L.Cs);
    double* part = reinterpret_cast<double*>(ws + L.part);
    float* ax32 = reinterpret_cast<float*>(ws + L.ax32);
    hipStream_t st = as_stream(stream);
    launch_cells(g, nimg, p->C, imgs, Cs, st);
    const int nblk = gram_blocks(g);
    GramArgs ga{Cs, part, reinterpret_cast<int*>(ws + L.list), reinterpret_cast<int*>(ws + L.count), g.H, g.W, nblk,
                gram_list(g)};
    hipLaunchKernelGGL(gram_kernel, dim3(nblk, batch), dim3(64 * kGramWaves), 0, st, ga);
    hipLaunchKernelGGL(gram_rest_kernel, dim3(nblk, batch), dim3(256), 0, st, ga);
    double* gsum = reinterpret_cast<double*>(ws + L.gsum);
    hipLaunchKernelGGL(gram_sum_kernel, dim3((kPart + 255) / 256, batch), dim3(256), 0, st, part, nblk,
                       gsum);
    hipLaunchKernelGGL(gram_cov_kernel, dim3(kDesc, batch), dim3(kDesc), 0, st, gsum,
                       1.0 / (4.0 * (double)g.npx), mean, cov);
    double* sqm = reinterpret_cast<double*>(ws + L.sq);  // [batch][2][kDesc][kDesc]
    for (int i = 0; i < kSquare; ++i) {
        const double* src = i == 0 ? cov : sqm + (size_t)((i - 1) & 1) * kDesc * kDesc;
        const size_t src_stride = i == 0 ? (size_t)kDesc * kDesc : (size_t)2 * kDesc * kDesc;
        hipLaunchKernelGGL(square_kernel, dim3(64, batch), dim3(256), 0, st, src, src_stride,
                           sqm + (size_t)(i & 1) * kDesc * kDesc, (size_t)2 * kDesc * kDesc);
    }
    hipLaunchKernelGGL(eig_kernel, dim3(batch), dim3(kEigThreads), 0, st, cov, mean, sqm, eigval, axes, ax32);
    hipLaunchKernelGGL(eig_direct_kernel, dim3(batch), dim3(kEigThreads), 0, st, cov, mean, sqm, eigval, axes, ax32);
    const long total = 4L * (long)g.npx;
    const long groups = (total + kGramPx - 1) / kGramPx;
    hipLaunchKernelGGL(project_kernel, dim3((unsigned)std::min<long>(groups, kProjBlocks), batch), dim3(256), 0,
                       st, Cs, ax32, reinterpret_cast<float4*>(phi), g.H, g.W);
    return launch_status();
}

extern "C" sff_status sff_cost_sift(const sff_params* p, int32_t batch, int32_t dir, const float* phi,
                                    const int16_t* hyp, float* cost, void* stream) {
    if (!params_ok(p) || batch < 1 || batch > 65535 || (dir != SFF_DIR_FORWARD && dir != SFF_DIR_INVERSE) ||
        !phi || !hyp || !cost || (int64_t)batch * 4 * p->H * p->W >= (int64_t(1) << 31))
        return SFF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(phi) & 15) != 0 || (reinterpret_cast<uintptr_t>(hyp) & 7) != 0 ||
        (reinterpret_cast<uintptr_t>(cost) & 3) != 0)
        return SFF_ERR_INVALID_ARG;
    const char* e = std::getenv("SFF_SIFT_EVAL");
    if (e && std::strcmp(e, "lane") == 0) {
        hipLaunchKernelGGL(cost_sift_kernel, dim3((p->W + kCT - 1) / kCT, (p->H + kCT - 1) / kCT, batch),
                           dim3(256), 0, as_stream(stream), reinterpret_cast<const float4*>(phi), hyp, cost,
                           p->H, p->W, dir == SFF_DIR_FORWARD ? 1 : -1);
        return launch_status();
    }
    SiftMatchArgs a{};
    a.phi = reinterpret_cast<const float4*>(phi);
    a.hyp = const_cast<int16_t*>(hyp);  // read only by this kernel
    a.cost = cost;
    a.H = p->H;
    a.W = p->W;
    a.batch = batch;
    a.ndir = 1;
    a.dir0 = dir == SFF_DIR_FORWARD ? 1 : -1;
    const int tiles_x = (p->W + 63) / 64;
    hipLaunchKernelGGL(sift_cost_coop_kernel, dim3(tiles_x * p->H * batch), dim3(64), 0, as_stream(stream), a,
                       tiles_x);
    return launch_status();
}

extern "C" sff_status sff_match_sift(const sff_params* p, int32_t batch, int32_t dir, const float* phi,
                                     const uint64_t* seeds, int32_t iters, int16_t* hyp, float* cost,
                                     void* stream) {
    if (!params_ok(p) || batch < 1 || batch > 32767 || (dir != SFF_DIR_FORWARD && dir != SFF_DIR_INVERSE &&
                                                         dir != SFF_DIR_BOTH) ||
        !phi || !seeds || !hyp || !cost || iters < 0 || iters > 64 ||
        (int64_t)batch * 4 * p->H * p->W >= (int64_t(1) << 31))
        return SFF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(phi) & 15) != 0 || (reinterpret_cast<uintptr_t>(hyp) & 7) != 0 ||
        (reinterpret_cast<uintptr_t>(cost) & 3) != 0 || (reinterpret_cast<uintptr_t>(seeds) & 7) != 0)
        return SFF_ERR_INVALID_ARG;
    SiftMatchArgs a;
    a.phi = reinterpret_cast<const float4*>(phi);
    a.seeds = seeds;
    a.hyp = hyp;
    a.cost = cost;
    a.H = p->H;
    a.W = p->W;
    a.rs_r0 = p->rs_r0;
    a.rs_samples = p->rs_samples;
    a.fmax = p->fmax;
    a.dmax = p->dmax;
    a.batch = batch;
    a.ndir = dir == SFF_DIR_BOTH ? 2 : 1;
    a.dir0 = dir == SFF_DIR_BOTH ? 1 : dir;
    const int nz = a.ndir * batch;
    hipStream_t st = as_stream(stream);
    const size_t npx = (size_t)p->H * p->W;
    // SFF_SIFT_EVAL=lane forces the per-lane kernels (same results; testing and timing)
    const char* e = std::getenv("SFF_SIFT_EVAL");
    const bool lane = e && std::strcmp(e, "lane") == 0;
    if (lane)
        hipLaunchKernelGGL(sift_cost_init_kernel, dim3((unsigned)((npx + 255) / 256), nz), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL(sift_cost_coop_kernel, dim3(((p->W + 63) / 64) * p->H * nz), dim3(64), 0, st, a,
                           (p->W + 63) / 64);
    // the wave-shared half-step's 32-bit offsets reach maps below 2 GiB per image
    const bool lane_step = lane || npx * sizeof(float4) >= (size_t)kNoElement;
    const int tiles_x = ((p->W + 1) / 2 + 63) / 64, tiles_y = (p->H + 3) / 4;
    for (int it = 0; it < iters; ++it)
        for (int colour = 0; colour < 2; ++colour) {
            if (lane_step)
                hipLaunchKernelGGL(sift_half_step_kernel, dim3(tiles_x * tiles_y * nz), dim3(256), 0, st, a,
                                   it, colour, tiles_x, tiles_y);
            else
                hipLaunchKernelGGL(sift_half_step_wave_kernel, dim3(tiles_x * tiles_y * nz), dim3(64 * kHsRows), 0, st,
                                   a, it, colour, tiles_x, tiles_y);
        }
    return launch_status();
}

extern "C" sff_status sff_sift_sqrt(const float* in, float* out, int64_t n, void* stream) {
    if (!in || !out || n < 0 || n > (int64_t(1) << 31)) return SFF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(in) & 3) != 0 || (reinterpret_cast<uintptr_t>(out) & 3) != 0)
        return SFF_ERR_INVALID_ARG;
    if (n == 0) return SFF_OK;
    hipLaunchKernelGGL(sift_sqrt_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, as_stream(stream), in,
                       out, n);
    return launch_status();
}
