// Disparity fill (SceneFlowFields, Section 3.1, last paragraph of "Consistency
// Check"): a second disparity map by semi-global matching (Hirschmueller,
// TPAMI 2008) and the check of the disparity matches alone against it.
//
// Cost: Hamming distance of 5 x 5 census words of the channel-mean images,
// right pixel x - d clamped to the image.  Aggregation along 8 paths,
//   L(p, d) = C(p, d) + min(L(q, d), L(q, d +- 1) + P1, min_k L(q, k) + P2)
//             - min_k L(q, k),   q = p - r,
// summed over the paths; the disparity minimises the sum (smallest d on ties).
// 8, 16 or 32 lanes walk a path line sequentially, eight disparities per lane in
// packed 16-bit halves, neighbouring disparities exchanged by DPP lane moves and
// the minimum over d by a DPP reduction; each direction's costs (at most 24 + P2 <= 255) are written as
// uint8 and summed per pixel at the end.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "sff_internal.hpp"

namespace sff {
namespace {

constexpr int kMaxD = 256;
constexpr int kPad = kMaxD;  // left pad of the right census rows

__global__ void __launch_bounds__(256) grey_kernel(const uint8_t* __restrict__ img, uint8_t* __restrict__ g,
                                                   int npx, int C, size_t pair_stride) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= npx) return;
    const uint8_t* src = img + (size_t)blockIdx.y * pair_stride + (size_t)p * C;
    int s = 0;
    for (int c = 0; c < C; ++c) s += src[c];
    g[(size_t)blockIdx.y * npx + p] = (uint8_t)((s + C / 2) / C);
}

// bit k set when neighbour k (row-major over the 5 x 5 window without the
// centre) is darker than the centre; replicated border
// Census words of one image, rows of kPad + W words when pad = kPad (the pad
// words repeat column 0, so x - d reads the clamped pixel without a clamp).
__global__ void __launch_bounds__(256) census_kernel(const uint8_t* __restrict__ g,
                                                     uint32_t* __restrict__ cw, int H, int W, int pad) {
    const int Wo = W + pad;
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= H * Wo) return;
    const uint8_t* gi = g + (size_t)blockIdx.y * H * W;
    const int y = p / Wo, x = max(p - y * Wo - pad, 0);
    const int c = gi[y * W + x];
    uint32_t w = 0;
    int k = 0;
#pragma unroll
    for (int dy = -2; dy <= 2; ++dy)
#pragma unroll
        for (int dx = -2; dx <= 2; ++dx) {
            if (dx == 0 && dy == 0) continue;
            const int v = gi[clampi(y + dy, 0, H - 1) * W + clampi(x + dx, 0, W - 1)];
            w |= (uint32_t)(v < c) << k;
            ++k;
        }
    cw[(size_t)blockIdx.y * H * Wo + p] = w;
}

struct PathArgs {
    const uint32_t *cl, *cr;  // census words; cr rows have kPad words of pad
    uint8_t* L;               // [8][batch][H][W][Dp] path costs per direction
    int H, W, D, Dp, P1, P2, batch;  // Dp = D rounded up to 8
};

__constant__ int kDirs[8][2] = {{1, 0}, {-1, 0}, {0, 1}, {0, -1}, {1, 1}, {-1, -1}, {1, -1}, {-1, 1}};

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 as2(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
__device__ __forceinline__ uint32_t as1(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }

// The value of lane l - 1 (lane l + 1) of a group of LPL lanes, `edge` in the
// group's first (last) lane, and the minimum over the group, by DPP (and
// exchanges of 16- and 32-lane rows): the per-step chain never goes through the
// LDS crossbar.
template <int LPL>
__device__ __forceinline__ uint32_t from_lane_below(uint32_t v, bool first, uint32_t edge) {
    if constexpr (LPL == 16) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x111, 0xF, 0xF, false);  // row_shr:1
    } else {
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x138, 0xF, 0xF, false);
        return LPL < 64 && first ? edge : o;
    }
}
template <int LPL>
__device__ __forceinline__ uint32_t from_lane_above(uint32_t v, bool last, uint32_t edge) {
    if constexpr (LPL == 16) {
        return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x101, 0xF, 0xF, false);  // row_shl:1
    } else {
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)v, 0x130, 0xF, 0xF, false);
        return LPL < 64 && last ? edge : o;
    }
}
template <int LPL>
__device__ __forceinline__ uint32_t group_min(uint32_t m) {
    m = min(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, false));   // quad_perm 1,0,3,2
    m = min(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, false));   // quad_perm 2,3,0,1
    m = min(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x141, 0xF, 0xF, false));  // row_half_mirror
    if constexpr (LPL >= 16)
        m = min(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x140, 0xF, 0xF, false));  // row_mirror
    if constexpr (LPL >= 32) {
        // both rows of a pair: one result has each pair's even row twice, the other its odd row
        const auto r = __builtin_amdgcn_permlane16_swap(m, m, false, false);
        m = min((uint32_t)r[0], (uint32_t)r[1]);
    }
    if constexpr (LPL == 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(m, m, false, false);
        m = min((uint32_t)r[0], (uint32_t)r[1]);
    }
    return m;
}

__device__ __forceinline__ int wave_min_uniform(int m) {
    m = (int)group_min<16>((uint32_t)m);
    return min(min(__builtin_amdgcn_readlane(m, 0), __builtin_amdgcn_readlane(m, 16)),
               min(__builtin_amdgcn_readlane(m, 32), __builtin_amdgcn_readlane(m, 48)));
}

// The smallest of three per half.  The halves are whole numbers below 0x7C00,
// which order as the fp16 numbers of the same bits do.
__device__ __forceinline__ u16x2 min3(u16x2 a, u16x2 b, u16x2 c) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    auto h = [](u16x2 v) { return __builtin_bit_cast(h2, v); };
    return __builtin_bit_cast(u16x2, __builtin_elementwise_minimum(__builtin_elementwise_minimum(h(a), h(b)), h(c)));
}

// One wave walks 64 / LPL path lines of direction r; lane l of a line holds
// disparities 2 NP l .. 2 NP l + 2 NP - 1 as NP packed pairs, their census words
// NP / 2 16-byte loads kAhead - 1 steps ahead in a register ring.  The line's left
// words are loaded LPL steps at a time, one step per lane, and broadcast through
// the LDS crossbar a step ahead.  The walk starts from zero costs, which makes
// the first step L = C (P1, P2 >= 0).
// A disparity past the range has 255 added to its cost: its L is at least 255
// and the line's minimum at most 24 (some disparity takes the previous minimum),
// so it is no minimum, and as a neighbour it offers 255 + P1, no less than the
// minimum plus P2 <= 24 + 231 that every disparity may take.
template <int LPL, int NP>
__device__ __forceinline__ void walk_lines(const PathArgs& a, int r, int dx, int dy, int line0, int lines) {
    const int lane = threadIdx.x & 63, ll = lane % LPL;
    const int H = a.H, W = a.W, d0 = 2 * NP * ll;
    const int ncol = dx != 0 ? H : 0;
    const bool live = line0 + lane / LPL < lines;
    const int line = min(line0 + lane / LPL, lines - 1);
    int x0, y0;
    if (line < ncol) {
        x0 = dx > 0 ? 0 : W - 1;
        y0 = line;
    } else {
        const int k = line - ncol;
        x0 = dx != 0 ? (dx > 0 ? 1 + k : W - 2 - k) : k;
        y0 = dy > 0 ? 0 : H - 1;
    }
    const int nx = dx > 0 ? W - x0 : (dx < 0 ? x0 + 1 : INT_MAX);
    const int ny = dy > 0 ? H - y0 : (dy < 0 ? y0 + 1 : INT_MAX);
    const int len = min(nx, ny);
    const int maxlen = __builtin_amdgcn_readfirstlane((int)__reduce_max_sync(~0ull, (unsigned)len));
    const int minlen = __builtin_amdgcn_readfirstlane((int)__reduce_min_sync(~0ull, (unsigned)len));
    const size_t vol = (size_t)H * W * a.Dp;
    bool put[(NP + 3) / 4];  // Dp is a multiple of 8
#pragma unroll
    for (int j = 0; j < (NP + 3) / 4; ++j) put[j] = live && d0 + 8 * j < a.Dp;
    const long stride = (long)(dy * W + dx) * a.Dp;
    uint8_t* dst = a.L + ((size_t)r * a.batch + blockIdx.y) * vol + ((size_t)y0 * W + x0) * a.Dp + d0;
    const int Wr = W + kPad;
    // words x - d0 - 2 NP + 1 .. x - d0 of the right row: at least x - 255, inside the pad
    const uint32_t* src = a.cr + ((size_t)blockIdx.y * H + y0) * Wr + kPad + x0 - d0 - (2 * NP - 1);
    const long rstride = (long)dy * Wr + dx;
    const uint32_t* lsrc = a.cl + ((size_t)blockIdx.y * H + y0) * W + x0;
    const long lstride = (long)dy * W + dx;
    constexpr int kAhead = NP == 2 ? 8 : 6;
    constexpr uint32_t kEdge = 0x3FFF3FFFu;  // above every cost, and so with P1 or P2 added
    const u16x2 P1 = as2((uint32_t)a.P1 * 0x10001u), P2 = as2((uint32_t)a.P2 * 0x10001u);
    const bool firstl = ll == 0, lastl = ll == LPL - 1;
    uint32_t past[2 * NP];
#pragma unroll
    for (int k = 0; k < 2 * NP; ++k) past[k] = d0 + k < a.D ? 0u : 255u;
    struct Words {
        uint32_t w[2 * NP];
    };
    auto left = [&](int t) { return lsrc[(long)min(t + ll, len - 1) * lstride]; };
    uint32_t lw = left(0), lnext = left(LPL);
    const int lane0 = (lane - ll) * 4;
    auto left_word = [&](int t) {
        return (uint32_t)__builtin_amdgcn_ds_bpermute(lane0 + 4 * (t % LPL), (int)lw);
    };
    u16x2 L[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) L[j] = as2(0u);
    u16x2 pm = as2(0u);  // previous minimum, in both halves
    uint32_t wl = left_word(0);
    // ring slot i holds step t + i at the top of each group of kAhead steps;
    // GUARD: a line of the wave may end here (steps past its end reload its last pixel)
    Words ring[kAhead];
    int loaded = 0;  // step the next load is for
    auto load = [&](Words& c, auto guard) {
        __builtin_memcpy(&c, src, sizeof(Words));  // 16-byte loads, 4-byte aligned
        if constexpr (decltype(guard)::value) {
            src += loaded + 1 < len ? rstride : 0;
        } else {
            src += rstride;
        }
        ++loaded;
    };
    auto step = [&](int t, const Words& cw, auto guard) {
        u16x2 c[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const uint32_t lo = __popc(wl ^ cw.w[2 * NP - 1 - 2 * j]) + past[2 * j];
            const uint32_t hi = __popc(wl ^ cw.w[2 * NP - 2 - 2 * j]) + past[2 * j + 1];
            c[j] = as2(hi << 16 | lo);
        }
        if ((t + 1) % LPL == 0) {  // uniform
            lw = lnext;
            lnext = left(t + 1 + LPL);
        }
        wl = left_word(t + 1);
        const uint32_t below = from_lane_below<LPL>(as1(L[NP - 1]), firstl, kEdge);
        const uint32_t above = from_lane_above<LPL>(as1(L[0]), lastl, kEdge);
        // q[j] = disparities (2j - 1, 2j): the lower neighbours of pair j, the upper ones of pair j - 1
        u16x2 q[NP + 1];
        q[0] = as2(__builtin_amdgcn_alignbit(as1(L[0]), below, 16));
#pragma unroll
        for (int j = 1; j < NP; ++j) q[j] = as2(__builtin_amdgcn_alignbit(as1(L[j]), as1(L[j - 1]), 16));
        q[NP] = as2(__builtin_amdgcn_alignbit(above, as1(L[NP - 1]), 16));
        const u16x2 jump = pm + P2;
#pragma unroll
        for (int j = 0; j < NP; ++j)
            L[j] = min3(__builtin_elementwise_min(q[j], q[j + 1]) + P1, L[j], jump) - pm + c[j];
        if (!decltype(guard)::value || t < len) {
#pragma unroll
            for (int i = 0; i < NP; i += 4) {
                uint32_t o[NP < 4 ? 1 : 2];
#pragma unroll
                for (int j = 0; j < std::min(NP, 4); j += 2)
                    o[j / 2] = __builtin_amdgcn_perm(as1(L[i + j + 1]), as1(L[i + j]), 0x06040200u);
                if (put[i / 4]) {  // non-temporal: wta_kernel reads them only after the last line (177 -> 132 us)
                    if constexpr (NP == 2)
                        __builtin_nontemporal_store(o[0], reinterpret_cast<uint32_t*>(dst));
                    else
                        __builtin_nontemporal_store((uint64_t)o[1] << 32 | o[0], reinterpret_cast<uint64_t*>(dst + 2 * i));
                }
            }
        }
        dst += stride;
        u16x2 m2 = __builtin_elementwise_min(L[0], L[1]);
#pragma unroll
        for (int j = 2; j < NP; j += 2) m2 = min3(m2, L[j], L[j + 1]);
        pm = as2(group_min<LPL>(min(as1(m2) & 0xFFFFu, as1(m2) >> 16)) * 0x10001u);
    };
    using Open = std::integral_constant<bool, false>;
    using Guard = std::integral_constant<bool, true>;
#pragma unroll
    for (int j = 0; j < kAhead - 1; ++j) load(ring[j], Guard{});
    int t = 0;
    // every load's successor, step t + 2 kAhead - 1, is inside every line
    for (; t + 2 * kAhead <= minlen; t += kAhead) {
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            load(ring[(j + kAhead - 1) % kAhead], Open{});
            step(t + j, ring[j], Open{});
        }
    }
    for (; t + kAhead <= maxlen; t += kAhead) {
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            load(ring[(j + kAhead - 1) % kAhead], Guard{});
            step(t + j, ring[j], Guard{});
        }
    }
#pragma unroll
    for (int j = 0; j < kAhead - 1; ++j)
        if (t + j < maxlen) step(t + j, ring[j], Guard{});
}

// Blocks per direction: horizontal, vertical, diagonal.
struct PathBlocks {
    int h, v, d;
};

// 4 waves per block, blockIdx.y = batch element; LPL lanes per line with 2 NP
// disparities each, HL lanes with four disparities each for a horizontal line.
// The horizontal lines are the longest chains (W serial steps): they take the
// fewest operations per step, the first blocks (which lie on different CUs; alone
// 178 us against 248 us with other blocks between them) and the issue slots first.
// Bound: the vector ALU (about 275 us of issue for the case below); with the
// stores left out it takes 318 us.
// 375 x 1242, D = 193: 334 us.  Measured against it: four disparities per lane in
// 32 bits with one wave per line and four 4-byte loads of right words per step,
// 471 us (vector ALU and texture data path 80 % busy); all lines with eight
// disparities per lane, 382 us; costs formed once and read as bytes, 550 us;
// sixteen disparities per lane, 335 us.
template <int LPL, int NP, int HL>
__global__ void __launch_bounds__(256, 4) sgm_path_kernel(PathArgs a, PathBlocks n) {
    const int b = blockIdx.x;
    if (b < 2 * n.h) {
        const int r = b >= n.h, line0 = ((b - r * n.h) * 4 + wave_id()) * (64 / HL);
        if (line0 >= a.H) return;  // whole wave
        __builtin_amdgcn_s_setprio(2);
        walk_lines<HL, 2>(a, r, kDirs[r][0], 0, line0, a.H);
        return;
    }
    const int vd = b - 2 * n.h - 2 * n.v;  // first block of the diagonals: 0
    const int r = vd < 0 ? 2 + (vd + n.v >= 0) : 4 + vd / n.d;
    const int i = vd < 0 ? vd + (r == 2 ? 2 : 1) * n.v : vd % n.d;
    const int dx = kDirs[r][0], dy = kDirs[r][1];
    const int lines = dx != 0 ? a.H + a.W - 1 : a.W, line0 = (i * 4 + wave_id()) * (64 / LPL);
    if (line0 >= lines) return;
    walk_lines<LPL, NP>(a, r, dx, dy, line0, lines);
}

template <int LPL, int NP, int HL>
void launch_paths(const PathArgs& a, hipStream_t st) {
    constexpr int per = 4 * (64 / LPL), hper = 4 * (64 / HL);  // lines per block
    const PathBlocks n{(a.H + hper - 1) / hper, (a.W + per - 1) / per, (a.H + a.W - 1 + per - 1) / per};
    hipLaunchKernelGGL(HIP_KERNEL_NAME(sgm_path_kernel<LPL, NP, HL>), dim3(2 * n.h + 2 * n.v + 4 * n.d, a.batch),
                       dim3(256), 0, st, a, n);
}

// Winner-take-all over the summed path costs: one wave per pixel, lane l
// holds disparities 4l .. 4l + 3 (one dword of each direction's plane), the
// 8 planes are summed two bytes at a time in 16-bit fields (at most 8 * 255),
// and the minimum of (sum, d) over the wave gives the smallest d on ties.
// Each wave takes kWtaPix consecutive pixels with all their loads in flight.
constexpr int kWtaPix = 4;
__global__ void __launch_bounds__(256) wta_kernel(const uint32_t* __restrict__ L4,
                                                  int16_t* __restrict__ disp, int npx, int D, int nd,
                                                  int batch) {
    const int lane = threadIdx.x & 63;
    const int p0 = (blockIdx.x * 4 + wave_id()) * kWtaPix;
    if (p0 >= npx) return;  // whole wave
    const size_t plane = (size_t)batch * npx * nd;
    const uint32_t* s = L4 + ((size_t)blockIdx.y * npx + p0) * nd + lane;
    const int np = min(kWtaPix, npx - p0);
    const bool on = lane < nd;
    uint32_t w[kWtaPix][8];
#pragma unroll
    for (int j = 0; j < kWtaPix; ++j)
#pragma unroll
        for (int r = 0; r < 8; ++r) w[j][r] = on && j < np ? s[r * plane + (size_t)j * nd] : 0u;
#pragma unroll
    for (int j = 0; j < kWtaPix; ++j) {
        uint32_t lo = 0, hi = 0;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            lo += w[j][r] & 0x00FF00FFu;
            hi += (w[j][r] >> 8) & 0x00FF00FFu;
        }
        const uint32_t sum[4] = {lo & 0xFFFFu, hi & 0xFFFFu, lo >> 16, hi >> 16};
        int best = 0x7FFFFFFF;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int d = 4 * lane + k;
            if (d < D) best = min(best, (int)(sum[k] << 8) | d);
        }
        best = wave_min_uniform(best);
        if (lane == 0 && j < np) disp[(size_t)blockIdx.y * npx + p0 + j] = (int16_t)(best & 0xFF);
    }
}

__global__ void __launch_bounds__(256) fill_kernel(const int16_t* __restrict__ hyp,
                                                   const uint8_t* __restrict__ valid,
                                                   const int16_t* __restrict__ disp,
                                                   uint8_t* __restrict__ fill, int H, int W, int tau) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= H * W) return;
    const size_t o = (size_t)blockIdx.y * H * W + p;
    const int x = p % W;
    const int d0 = hyp[o * 4 + 2];
    const int e = d0 - disp[o];
    fill[o] = (valid[o] || (x - d0 >= 0 && e <= tau && e >= -tau)) ? 1 : 0;
}

// Disparities of a pixel in the path costs: D rounded up to 8.
inline int sgm_dp(int D) { return (D + 7) & ~7; }

struct SgmWs {
    size_t grey, census, census_r, S, total;
};

SgmWs sgm_ws(const sff_params& p, int batch) {
    const size_t npx = (size_t)p.H * p.W, n = (size_t)batch;
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    SgmWs L;
    L.grey = 0;
    L.census = al(2 * n * npx);
    L.census_r = L.census + al(n * npx * sizeof(uint32_t));
    L.S = L.census_r + al(n * p.H * (p.W + (size_t)kPad) * sizeof(uint32_t));
    L.total = L.S + al(8 * n * npx * (size_t)sgm_dp(p.dmax + 1));
    return L;
}

}  // namespace
}  // namespace sff

using namespace sff;

extern "C" size_t sff_sgm_workspace_bytes(const sff_params* p, int32_t batch) {
    if (!params_ok(p) || batch < 1 || batch > 32767) return 0;
    return sgm_ws(*p, batch).total;
}

extern "C" sff_status sff_sgm_disparity(const sff_params* p, int32_t batch, const uint8_t* left,
                                        const uint8_t* right, size_t pair_stride, int32_t P1,
                                        int32_t P2, int16_t* disp, void* workspace,
                                        size_t workspace_bytes, void* stream) {
    if (!params_ok(p) || batch < 1 || batch > 32767 || !left || !right || !disp || P1 < 0 ||
        P2 < P1 || P2 > 231 || (reinterpret_cast<uintptr_t>(disp) & 1) != 0)
        return SFF_ERR_INVALID_ARG;
    const size_t img_bytes = (size_t)p->H * p->W * p->C;
    if (batch > 1 && pair_stride < img_bytes) return SFF_ERR_INVALID_ARG;
    const int D = p->dmax + 1;
    if (D > kMaxD) return SFF_ERR_UNSUPPORTED;
    const SgmWs L = sgm_ws(*p, batch);
    if (!workspace || workspace_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return SFF_ERR_WORKSPACE;
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    const int H = p->H, W = p->W, npx = H * W;
    uint8_t* gl = ws + L.grey;
    uint8_t* gr = gl + (size_t)batch * npx;
    uint32_t* cl = reinterpret_cast<uint32_t*>(ws + L.census);
    uint32_t* cr = reinterpret_cast<uint32_t*>(ws + L.census_r);
    uint8_t* L8 = ws + L.S;
    hipStream_t st = as_stream(stream);
    const dim3 pgrid((npx + 255) / 256, batch);
    hipLaunchKernelGGL(grey_kernel, pgrid, dim3(256), 0, st, left, gl, npx, p->C, pair_stride);
    hipLaunchKernelGGL(grey_kernel, pgrid, dim3(256), 0, st, right, gr, npx, p->C, pair_stride);
    hipLaunchKernelGGL(census_kernel, pgrid, dim3(256), 0, st, gl, cl, H, W, 0);
    hipLaunchKernelGGL(census_kernel, dim3((H * (W + kPad) + 255) / 256, batch), dim3(256), 0, st, gr, cr,
                       H, W, kPad);
    const int Dp = sgm_dp(D);
    PathArgs a{cl, cr, L8, H, W, D, Dp, P1, P2, batch};
    // the fewest lanes per line that hold all disparities: the most lines per wave
    if (Dp <= 64)
        launch_paths<8, 4, 16>(a, st);
    else if (Dp <= 128)
        launch_paths<16, 4, 32>(a, st);
    else
        launch_paths<32, 4, 64>(a, st);
    hipLaunchKernelGGL(wta_kernel, dim3((npx + 4 * kWtaPix - 1) / (4 * kWtaPix), batch), dim3(256), 0, st,
                       reinterpret_cast<const uint32_t*>(L8), disp, npx, D, Dp / 4, batch);
    return launch_status();
}

extern "C" sff_status sff_disparity_fill(const sff_params* p, int32_t batch, const int16_t* hyp_fwd,
                                         const uint8_t* valid, const int16_t* disp, uint8_t* fill,
                                         void* stream) {
    if (!params_ok(p) || batch < 1 || batch > 32767 || !hyp_fwd || !valid || !disp || !fill ||
        (reinterpret_cast<uintptr_t>(hyp_fwd) & 7) != 0 || (reinterpret_cast<uintptr_t>(disp) & 1) != 0)
        return SFF_ERR_INVALID_ARG;
    hipLaunchKernelGGL(fill_kernel, dim3((p->H * p->W + 255) / 256, batch), dim3(256), 0,
                       as_stream(stream), hyp_fwd, valid, disp, fill, p->H, p->W, p->tau);
    return launch_status();
}
