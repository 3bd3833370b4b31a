// Multi-scale propagation and random search at one level (SceneFlowFields,
// Section 3.1, "Multi-Scale Propagation"), with the eq. (1) matching cost.
//
// Schedule: per iteration a red half-step (pixels with (i + j) even) then a
// black one.  Pixels of one colour only read the other colour's vectors, so a
// half-step is a race-free Jacobi sweep and its result does not depend on the
// order in which threads run.  Each pixel: cheapest of [own, left, up, right,
// down] under strict improvement, then rs_samples random-search samples around
// that vector (Philox4x32-10), kept on strict improvement.
//
// The hand-off from the coarser level is fused into iteration 0: a pixel whose
// level-k vector has not been written yet reads its parent's vector from the
// coarse field and computes its cost at this level.
//
// Two kinds of feature maps feed the same kernel: descriptor records (one
// record of C x 16 int16 per pixel: the WHT descriptors, or any descriptors
// such as learned ones; sff_match_level), and the WHT descriptors' bin-sum
// planes (sff_match_level_bins).  The descriptor of a pixel is the 4x4
// lowest-sequency block of the WHT of its 8x8 patch, i.e. the 4-point Hadamard
// transform along both axes of the patch's 4 x 4 grid of 2 x 2-bin sums; that
// transform is orthogonal up to a factor of 4 per axis, so the squared
// distance of two descriptors is exactly 16 times the squared distance of
// their bin grids (all integers).  The bin grids of neighbouring pixels
// overlap, so one level's planes (BinGeom: 24 bytes per position at C = 3,
// each bin stored for four rows) are a fifth of the descriptor records' size
// and the gathers mostly hit the L2 instead of streaming records.
#include <algorithm>
#include <cstdlib>
#include <cstring>

#include <type_traits>

#include "sff_device.hpp"

namespace sff {
namespace {

struct MatchArgs {
    const uint8_t* maps;        // [batch][4] images of descriptor records or bin planes
    size_t img_bytes;           // bytes of one image's map
    const uint64_t* seeds;      // [batch]
    const int16_t* hyp_coarse;  // [ndir][batch][Hc][Wc][4] or null
    int16_t* hyp;               // [ndir][batch][Hk][Wk][4]
    uint32_t* cost;             // [ndir][batch][Hk][Wk]
    int H, W, n, level, Hk, Wk, Hc, Wc;
    int sh, Hq, Wq;             // bin planes (BinGeom)
    int rs_r0, rs_samples, fmax, dmax;
    int batch, dir0, ndir;
};

struct Hyp {
    int u, v, d0, d1;
};

__device__ __forceinline__ Hyp unpack(uint2 h) {
    Hyp r;
    r.u = (int)(int16_t)(h.x & 0xFFFFu);
    r.v = (int)(int16_t)(h.x >> 16);
    r.d0 = (int)(int16_t)(h.y & 0xFFFFu);
    r.d1 = (int)(int16_t)(h.y >> 16);
    return r;
}

__device__ __forceinline__ uint2 pack(const Hyp& h) {
    uint2 r;
    r.x = (uint32_t)(uint16_t)(int16_t)h.u | ((uint32_t)(uint16_t)(int16_t)h.v << 16);
    r.y = (uint32_t)(uint16_t)(int16_t)h.d0 | ((uint32_t)(uint16_t)(int16_t)h.d1 << 16);
    return r;
}

__device__ __forceinline__ bool same(const Hyp& a, const Hyp& b) {
    return a.u == b.u && a.v == b.v && a.d0 == b.d0 && a.d1 == b.d1;
}

// Wave-level ordering of LDS accesses made by different lanes of one wave.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Raw buffer descriptor of one image's map (wave-uniform base), with the
// image's size as its range: a load at an offset at or past `bytes` returns
// zeros without a memory access.  Offsets are 32-bit, so a map is smaller than
// 2 GiB.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t map_rsrc(const void* M, uint32_t bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(M);
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)p) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(p >> 32)) << 32);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), (short)0,
                                             (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// Offset of no patch: past the range of every image (images are smaller).
constexpr int kNoTarget = 0x7FFFFFF0;

// Map of view v (0..3 in the canonical order) for direction s: the forward
// field has reference I_l^0 and targets I_l^1 (temporal), I_r^0 (stereo),
// I_r^1 (cross); the inverse field has reference I_r^1 and targets I_r^0,
// I_l^1, I_l^0.
struct Views {
    const uint8_t *R, *T, *S, *X;
    __device__ __forceinline__ Views(const MatchArgs& a, int b, int s) {
        const uint8_t* base = a.maps + (size_t)b * 4 * a.img_bytes;
        R = base + (size_t)(s > 0 ? 0 : 3) * a.img_bytes;
        T = base + (size_t)(s > 0 ? 1 : 2) * a.img_bytes;
        S = base + (size_t)(s > 0 ? 2 : 1) * a.img_bytes;
        X = base + (size_t)(s > 0 ? 3 : 0) * a.img_bytes;
    }
};

// s * v for a direction s = +1 or -1.
__device__ __forceinline__ int dirmul(int s, int v) { return s > 0 ? v : -v; }

// eq. (1): temporal (x+u, y+v), stereo (x - s d0, y), cross (x+u - s d1, y+v),
// each target clamped to the image.  The three squared distances are
// non-negative, so once a partial sum reaches `bound` the candidate cannot be
// strictly cheaper than `bound`: the remaining gathers are skipped and a value
// >= bound is returned.  Below `bound` the exact cost is returned.  Lanes with
// want = false have no candidate; their result is meaningless.  The views are
// taken cross, temporal, stereo: the cross target moves with three of the four
// components (u, v, d1), the stereo one with d0 only, so this order rejects a
// poor candidate soonest (measured 1.8% faster at level 0 than temporal,
// stereo, cross).
//
// Evaluators with the same results: per lane (LaneEval for record maps of 2 GiB
// and more, and with BinLane the reference that the tests compare with) and
// cooperative (PatchCoop: fewest cache-line lookups), which must be called by all
// lanes of the wave.
template <int C>
struct LaneEval {
    static constexpr int kOwners = 64;
    static constexpr int kLdsWords = 1;
    static constexpr int kPG = 1, kRG = 1;
    static constexpr bool kGroups = false;
    const uint4 *T, *S, *X, *R;
    int H, W, s;
    Desc<C> ref;

    __device__ __forceinline__ void setup(const MatchArgs& a, int b, int sd) {
        const Views v(a, b, sd);
        R = reinterpret_cast<const uint4*>(v.R);
        T = reinterpret_cast<const uint4*>(v.T);
        S = reinterpret_cast<const uint4*>(v.S);
        X = reinterpret_cast<const uint4*>(v.X);
        H = a.H;
        W = a.W;
        s = sd;
    }

    template <class F>
    __device__ __forceinline__ void init(int x, int y, int, uint32_t*, F) {
        ref = load_desc<C>(reinterpret_cast<const int16_t*>(R), (size_t)y * W + x);
    }

    __device__ __forceinline__ uint32_t map_ssd(const uint4* M, int pix) const {
        return desc_ssd<C>(ref, load_desc<C>(reinterpret_cast<const int16_t*>(M), (size_t)pix));
    }

    __device__ __forceinline__ uint32_t cost_below(bool want, int x, int y, const Hyp& h,
                                                   uint32_t bound) {
        if (!want) return 0xFFFFFFFFu;
        const int ty = clampi(y + h.v, 0, H - 1);
        uint32_t c = map_ssd(X, ty * W + clampi(x + h.u - dirmul(s, h.d1), 0, W - 1));
        if (c >= bound) return c;
        c += map_ssd(T, ty * W + clampi(x + h.u, 0, W - 1));
        if (c >= bound) return c;
        return c + map_ssd(S, y * W + clampi(x - dirmul(s, h.d0), 0, W - 1));
    }

    template <int N>
    __device__ __forceinline__ void cost_belowN(const bool (&)[N], const Hyp (&)[N], int, int,
                                                uint32_t, uint32_t (&)[N]) {}
};

// Bin planes: eq. (1) as 16 x the bin-grid squared distance of the reference
// patch and the three target patches, with the same early-out and view order as
// the descriptor records.  A patch is P = bin_pieces(C) pieces of 16 bytes,
// contiguous (4 entries of 4 plane rows; 4 pieces of packed bins for C = 3).
// BinLane: each lane gathers its own patches (reference for the tests).
template <int C>
struct BinLane {
    static constexpr int P = bin_pieces(C);
    static constexpr int kOwners = 64;
    static constexpr int kLdsWords = 1;
    static constexpr int kPG = 1, kRG = 1;
    static constexpr bool kGroups = false;
    __amdgpu_buffer_rsrc_t rR, rT, rS, rX;
    BinAddr<C> addr;
    int H, W, s;
    BinRef<C> ref[P];

    __device__ __forceinline__ void setup(const MatchArgs& a, int b, int sd) {
        const Views v(a, b, sd);
        const uint32_t bytes = (uint32_t)a.img_bytes;
        rR = map_rsrc(v.R, bytes);
        rT = map_rsrc(v.T, bytes);
        rS = map_rsrc(v.S, bytes);
        rX = map_rsrc(v.X, bytes);
        H = a.H;
        W = a.W;
        s = sd;
        addr.sh = a.sh;
        addr.Hq = a.Hq;
        addr.RS = a.Wq * bin_entry_bytes(C);
    }

    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int off, uint4* v) const {
#pragma unroll
        for (int k = 0; k < P; ++k)
            v[k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16 * k, 0, 0));
    }

    template <class F>
    __device__ __forceinline__ void init(int x, int y, int, uint32_t*, F) {
        uint4 v[P];
        load(rR, addr(x, y), v);
#pragma unroll
        for (int k = 0; k < P; ++k) ref[k] = bin_ref<C>(v[k]);
    }

    __device__ __forceinline__ uint32_t view_cost(__amdgpu_buffer_rsrc_t rs, int X, int Y) const {
        uint4 v[P];
        load(rs, addr(X, Y), v);
        int acc = 0;
#pragma unroll
        for (int k = 0; k < P; ++k) acc = bin_piece_ssd<C>(ref[k], v[k], acc);
        return 16u * (uint32_t)acc;
    }

    __device__ __forceinline__ uint32_t cost_below(bool want, int x, int y, const Hyp& h,
                                                   uint32_t bound) {
        if (!want) return 0xFFFFFFFFu;
        const int ty = clampi(y + h.v, 0, H - 1);
        uint32_t c = view_cost(rX, clampi(x + h.u - dirmul(s, h.d1), 0, W - 1), ty);
        if (c >= bound) return c;
        c += view_cost(rT, clampi(x + h.u, 0, W - 1), ty);
        if (c >= bound) return c;
        return c + view_cost(rS, clampi(x - dirmul(s, h.d0), 0, W - 1), y);
    }

    template <int N>
    __device__ __forceinline__ void cost_belowN(const bool (&)[N], const Hyp (&)[N], int, int,
                                                uint32_t, uint32_t (&)[N]) {}
};

// What a cooperative gather reads: P contiguous pieces of 16 bytes per patch at
// the byte offset of a target, a piece's squared distance to the reference
// piece, and the factor from those sums to the cost.  Bin patches:
template <int C>
struct BinMap {
    static constexpr int P = bin_pieces(C);
    static constexpr uint32_t kScale = 16u;
    using Ref = BinRef<C>;
    BinAddr<C> addr;
    __device__ __forceinline__ void setup(const MatchArgs& a) {
        addr.sh = a.sh;
        addr.Hq = a.Hq;
        addr.RS = a.Wq * bin_entry_bytes(C);
    }
    __device__ __forceinline__ int operator()(int X, int Y) const { return addr(X, Y); }
    static __device__ __forceinline__ Ref ref(uint4 v) { return bin_ref<C>(v); }
    static __device__ __forceinline__ int ssd(const Ref& r, uint4 v, int acc) { return bin_piece_ssd<C>(r, v, acc); }
};

// Descriptor records (2 C pieces, aligned to their padded size: one cache line):
template <int C>
struct RecMap {
    static constexpr int P = 2 * C;
    static constexpr uint32_t kScale = 1u;
    using Ref = uint4;
    int W;
    __device__ __forceinline__ void setup(const MatchArgs& a) { W = a.W; }
    __device__ __forceinline__ int operator()(int X, int Y) const { return (Y * W + X) * (32 * kRecC<C>); }
    static __device__ __forceinline__ Ref ref(uint4 v) { return v; }
    static __device__ __forceinline__ int ssd(const Ref& r, uint4 v, int acc) { return piece_ssd(r, v, acc); }
};

// The patches of a wave's O owners (lane l owns one pixel: its reference patch
// and hypothesis) gathered cooperatively: gathering one patch per owner takes
// K = O P / 64 wave-wide loads; in load k lane l fetches piece f mod P of owner
// f / P, f = 64 k + l, so one load reads the whole patches of a few owners
// instead of one piece each of 64 unrelated ones: the texture path handles about
// one 64-byte sector per clock per CU, and with the maps resident in the L2 that,
// not the L2, bounds a full chip.  Each lane keeps the reference pieces of its
// slots in registers, forms the pieces' partial squared distances, and the P
// partials of an owner are summed through the wave's LDS slice.  Owners without
// a target get an offset past the map's range (the load returns zeros without a
// memory access).  With O < 64 lanes O..63 only help (more waves for a level too
// small to fill the chip).  PG neighbour candidates and RG random-search samples
// are scored together, their gathers in flight at once; XTS: all three views in
// one round.
template <class M, int PG, int RG, int O = 64, bool XTS = false>
struct PatchCoop {
    static_assert(O == 64 || O == 32 || O == 16, "owners per wave");
    static_assert(O * M::P % 64 == 0, "whole loads per gather");
    static constexpr int P = M::P;
    static constexpr int K = O * P / 64;  // wave-wide loads per patch gather
    static constexpr int kOwners = O;
    static constexpr int kPG = PG, kRG = RG;
    static constexpr int kGroup = PG > RG ? PG : RG;
    static constexpr int kLdsWords = kGroup * 64 * K;
    static constexpr bool kGroups = true;
    __amdgpu_buffer_rsrc_t rR, rT, rS, rX;
    M addr;
    int H, W, s;
    typename M::Ref refp[K];  // reference piece of slot k
    uint32_t* part;  // this wave's LDS slice
    int lane;

    __device__ __forceinline__ void setup(const MatchArgs& a, int b, int sd) {
        const Views v(a, b, sd);
        const uint32_t bytes = (uint32_t)a.img_bytes;
        rR = map_rsrc(v.R, bytes);
        rT = map_rsrc(v.T, bytes);
        rS = map_rsrc(v.S, bytes);
        rX = map_rsrc(v.X, bytes);
        H = a.H;
        W = a.W;
        s = sd;
        addr.setup(a);
    }

    __device__ __forceinline__ static int owner(int k, int l) { return (64 * k + l) / P; }
    __device__ __forceinline__ static int piece(int k, int l) { return (64 * k + l) % P; }

    // Offset of slot (k, lane): piece of its owner's patch at ob; an owner
    // without a target has ob = kNoTarget, and its slots, kNoTarget plus at
    // most 16 (P - 1) as unsigned 32-bit offsets, lie past every map's range
    // (maps are at most kNoTarget bytes), so their loads return zeros.
    __device__ __forceinline__ int slot_off(int ob, int k) const {
        return (int)((uint32_t)__shfl(ob, owner(k, lane)) + (uint32_t)(piece(k, lane) * 16));
    }

    template <class F>
    __device__ __forceinline__ void init(int x, int y, int l, uint32_t* lds, F) {
        lane = l;
        part = lds;
        const int ob = addr(x, y);
#pragma unroll
        for (int k = 0; k < K; ++k)
            refp[k] = M::ref(
                __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rR, slot_off(ob, k), 0, 0)));
    }

    // Squared distances (scaled) of N patches per owner, all gathers in flight
    // together; ob[m] = kNoTarget marks no target (result 0).  Must be called by all
    // lanes of the wave.
    // Patch m is read through rs_of(m) (views may differ between patches).
    template <int N, class RS>
    __device__ __forceinline__ void ssdN(RS rs_of, const int (&ob)[N], uint32_t (&c)[N]) {
        uint4 v[N][K];
        int so[N][K];
#pragma unroll
        for (int m = 0; m < N; ++m)
#pragma unroll
            for (int k = 0; k < K; ++k) so[m][k] = slot_off(ob[m], k);
#pragma unroll
        for (int m = 0; m < N; ++m)
#pragma unroll
            for (int k = 0; k < K; ++k)
                v[m][k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_of(m), so[m][k], 0, 0));
#pragma unroll
        for (int m = 0; m < N; ++m)
#pragma unroll
            for (int k = 0; k < K; ++k)
                part[64 * (m * K + k) + lane] = (uint32_t)M::ssd(refp[k], v[m][k], 0);
        wave_sync();
        const int ol = lane & (O - 1);  // lanes past the owners read a valid slot
#pragma unroll
        for (int m = 0; m < N; ++m) {
            uint32_t t = 0;
#pragma unroll
            for (int w = 0; w < P; ++w) t += part[64 * K * m + ol * P + w];
            c[m] = ob[m] != kNoTarget ? M::kScale * t : 0u;
        }
        wave_sync();
    }

    // The cross, temporal and stereo distances summed, of N candidates
    // per owner: the 3 N patches of ob (cross ones first, then temporal, then
    // stereo; a candidate without a target has kNoTarget in all three, result
    // 0) gathered together, and a slot's three pieces summed before the
    // partials go through LDS.  Must be called by all lanes of the wave.
    template <int N>
    __device__ __forceinline__ void ssd_views(const int (&ob)[3 * N], uint32_t (&c)[3 * N]) {
        uint4 v[3 * N][K];
        int so[3 * N][K];
#pragma unroll
        for (int m = 0; m < 3 * N; ++m)
#pragma unroll
            for (int k = 0; k < K; ++k) so[m][k] = slot_off(ob[m], k);
#pragma unroll
        for (int m = 0; m < 3 * N; ++m) {
            const __amdgpu_buffer_rsrc_t rs = m < N ? rX : m < 2 * N ? rT : rS;
#pragma unroll
            for (int k = 0; k < K; ++k)
                v[m][k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, so[m][k], 0, 0));
        }
#pragma unroll
        for (int m = 0; m < N; ++m)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                int acc = M::ssd(refp[k], v[m][k], 0);
                acc = M::ssd(refp[k], v[N + m][k], acc);
                part[64 * (m * K + k) + lane] = (uint32_t)M::ssd(refp[k], v[2 * N + m][k], acc);
            }
        wave_sync();
        const int ol = lane & (O - 1);  // lanes past the owners read a valid slot
#pragma unroll
        for (int m = 0; m < N; ++m) {
            uint32_t t = 0;
#pragma unroll
            for (int w = 0; w < P; ++w) t += part[64 * K * m + ol * P + w];
            c[m] = ob[m] != kNoTarget ? M::kScale * t : 0u;
        }
        wave_sync();
    }

    __device__ __forceinline__ uint32_t cost_below(bool want, int x, int y, const Hyp& h,
                                                   uint32_t bound) {
        bool w[1] = {want};
        Hyp hh[1] = {h};
        uint32_t c[1];
        cost_belowN<1>(w, hh, x, y, bound, c);
        return c[0];
    }

    // cost_below for N candidates of each lane, their gathers issued together
    // view by view with the early-out between views, or (XTS) all three views
    // in one round; same results as N calls with the same bound: a candidate
    // stopped at a view has a partial cost at or above the bound, one that
    // passes (or is scored in full) its exact cost.
    template <int N>
    __device__ __forceinline__ void cost_belowN(const bool (&w)[N], const Hyp (&h)[N], int x, int y,
                                                uint32_t bound, uint32_t (&c)[N]) {
        int ty[N], ob[N];
        bool al[N];
        bool any = false;
#pragma unroll
        for (int m = 0; m < N; ++m) {
            ty[m] = clampi(y + h[m].v, 0, H - 1);
            ob[m] = w[m] ? addr(clampi(x + h[m].u - dirmul(s, h[m].d1), 0, W - 1), ty[m]) : kNoTarget;
        }
        if constexpr (XTS) {
            int o3[3 * N];
            uint32_t c3[3 * N];
#pragma unroll
            for (int m = 0; m < N; ++m) {
                o3[m] = ob[m];
                o3[N + m] = w[m] ? addr(clampi(x + h[m].u, 0, W - 1), ty[m]) : kNoTarget;
                o3[2 * N + m] = w[m] ? addr(clampi(x - dirmul(s, h[m].d0), 0, W - 1), y) : kNoTarget;
            }
            ssd_views<N>(o3, c3);
#pragma unroll
            for (int m = 0; m < N; ++m) c[m] = c3[m];
            return;
        }
        ssdN<N>([&](int) { return rX; }, ob, c);
#pragma unroll
        for (int m = 0; m < N; ++m) {
            al[m] = w[m] && c[m] < bound;
            any = any || al[m];
            ob[m] = al[m] ? addr(clampi(x + h[m].u, 0, W - 1), ty[m]) : kNoTarget;
        }
        if (!__any(any)) return;
        uint32_t d[N];
        ssdN<N>([&](int) { return rT; }, ob, d);
        any = false;
#pragma unroll
        for (int m = 0; m < N; ++m) {
            c[m] += d[m];
            al[m] = al[m] && c[m] < bound;
            any = any || al[m];
            ob[m] = al[m] ? addr(clampi(x - dirmul(s, h[m].d0), 0, W - 1), y) : kNoTarget;
        }
        if (!__any(any)) return;
        ssdN<N>([&](int) { return rS; }, ob, d);
#pragma unroll
        for (int m = 0; m < N; ++m) c[m] += d[m];
    }
};

// mode: 0 = regular half-step; 1 = iteration-0 red half after a hand-off (own
// and neighbours from the coarse field); 2 = iteration-0 black half after a
// hand-off (own from the coarse field, neighbours already at this level);
// 3 = hand-off only (no propagation or search), used when iters == 0.
//
// Block = one wave: E::kOwners (64, 32, or 16 for the smallest launches) pixels of
// the half-step's colour in one grid row (all pixels for mode 3).  Lanes past
// the row's end or past the owners stay in the wave (for the cooperative
// gathers) without a pixel of their own.  One-wave blocks let a
// finished wave's slot be refilled at once; the early-out makes wave times
// uneven (level 0 of the KITTI-size pair: 1.459 vs 1.482 ms per step with
// four-row blocks, level 2: 0.262 vs 0.286 ms).
template <int C, class E>
__global__ void __launch_bounds__(64) half_step_kernel(MatchArgs a, int it, int colour, int mode,
                                                       int tiles_x, int tiles_y) {
    __shared__ uint32_t part_lds[E::kLdsWords];
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int per_field = tiles_x * tiles_y;
    const int z = tile / per_field;
    const int tr = tile - z * per_field;
    const int tx = tr / tiles_y, ty = tr - tx * tiles_y;
    const int lane = threadIdx.x;
    const int i = ty;
    const int par = mode == 3 ? 0 : ((i + colour) & 1);
    const int step = mode == 3 ? 1 : 2;
    constexpr int O = E::kOwners;
    const int j = step * (tx * O + lane) + par;
    const bool act = lane < O && j < a.Wk;
    const int di = z / a.batch, b = z - di * a.batch;
    const int s = (a.ndir == 2) ? (di == 0 ? 1 : -1) : a.dir0;
    E V;
    V.setup(a, b, s);
    const int n = a.n;
    const int x = n * min(j, a.Wk - 1), y = n * i;
    {
        const int j0 = step * tx * O + par, W = a.W, Wk1 = a.Wk - 1;
        V.init(x, y, lane, part_lds, [=](int o) { return y * W + n * min(j0 + step * o, Wk1); });
    }

    const size_t field_off = (size_t)z * a.Hk * a.Wk;
    const uint2* field = reinterpret_cast<const uint2*>(a.hyp) + field_off;
    const uint2* coarse = mode == 0 ? nullptr
                                    : reinterpret_cast<const uint2*>(a.hyp_coarse) +
                                          (size_t)z * a.Hc * a.Wc;
    const int jj = min(j, a.Wk - 1);
    const size_t o = (size_t)i * a.Wk + jj;

    Hyp best;
    uint32_t bestc;
    if (mode == 0) {
        best = unpack(field[o]);
        bestc = a.cost[field_off + o];
    } else {
        best = unpack(coarse[(size_t)(i >> 1) * a.Wc + (jj >> 1)]);
        bestc = V.cost_below(act, x, y, best, 0xFFFFFFFFu);
    }
    if (mode != 3) {
        // propagation: left, up, right, down.  A vector equal to one already
        // scored has the same cost and cannot be a strict improvement.
        const int ni[4] = {i, i - 1, i, i + 1};
        const int nj[4] = {jj - 1, jj, jj + 1, jj};
        uint2 nh[4];
        bool in[4];
        const uint2 own = pack(best);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            in[q] = act && ni[q] >= 0 && ni[q] < a.Hk && nj[q] >= 0 && nj[q] < a.Wk;
            nh[q] = own;
            if (in[q])
                nh[q] = mode == 1 ? coarse[(size_t)(ni[q] >> 1) * a.Wc + (nj[q] >> 1)]
                                  : field[(size_t)ni[q] * a.Wk + nj[q]];
        }
        bool want[4];
        Hyp hq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            bool dup = nh[q].x == own.x && nh[q].y == own.y;
#pragma unroll
            for (int p = 0; p < q; ++p) dup = dup || (in[p] && nh[q].x == nh[p].x && nh[q].y == nh[p].y);
            want[q] = in[q] && !dup;
            hq[q] = unpack(nh[q]);
        }
        // Candidates are accepted one after the other in their order.  The
        // cooperative evaluator scores a group at a time against the bound
        // from before the group: a later candidate rejected against that bound
        // is at least as costly as the updated best, and one scored below it
        // has its exact cost, so the results are those of one at a time, and
        // the group's gathers are in flight together instead of in sequence.
        auto take = [&](bool w, const Hyp& h, uint32_t c) {
            if (w && c < bestc) {
                bestc = c;
                best = h;
            }
        };
        constexpr int kPropGroup = E::kPG;
        if constexpr (E::kGroups) {
#pragma unroll
            for (int q0 = 0; q0 < 4; q0 += kPropGroup) {
                bool wg[kPropGroup];
                Hyp hg[kPropGroup];
                bool any = false;
#pragma unroll
                for (int m = 0; m < kPropGroup; ++m) {
                    wg[m] = want[q0 + m];
                    hg[m] = hq[q0 + m];
                    any = any || wg[m];
                }
                if (!__any(any)) continue;
                uint32_t c[kPropGroup];
                V.template cost_belowN<kPropGroup>(wg, hg, x, y, bestc, c);
#pragma unroll
                for (int m = 0; m < kPropGroup; ++m) take(wg[m], hg[m], c[m]);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (!__any(want[q])) continue;
                take(want[q], hq[q], V.cost_below(want[q], x, y, hq[q], bestc));
            }
        }
        // random search around the propagated vector
        const Hyp centre = best;
        const uint64_t seed = a.seeds[b];
        const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
        auto draw = [&](int t, int col) {  // the Philox draws of sample t at grid column col
            U4 ctr;
            ctr.x = (uint32_t)(i * a.Wk + col);
            ctr.y = (uint32_t)it;
            ctr.z = ((uint32_t)a.level << 16) | ((uint32_t)t << 8) | (s < 0 ? 1u : 0u);
            ctr.w = 0u;
            return philox4x32_10(ctr, k0, k1);
        };
        auto offset = [&](int t, const U4& rnd) {
            const int r = max(1, a.rs_r0 >> t) * n;
            Hyp c;
            c.u = clampi(centre.u + uniform_offset(rnd.x, r), -a.fmax, a.fmax);
            c.v = clampi(centre.v + uniform_offset(rnd.y, r), -a.fmax, a.fmax);
            c.d0 = clampi(centre.d0 + uniform_offset(rnd.z, r), 0, a.dmax);
            c.d1 = clampi(centre.d1 + uniform_offset(rnd.w, r), 0, a.dmax);
            return c;
        };
        auto sample = [&](int t) { return offset(t, draw(t, jj)); };
        // samples t .. t + G - 1 as one group
        auto group = [&](auto size, int t) {
            constexpr int G = decltype(size)::value;
            Hyp cg[G];
            bool wg[G];
            bool any = false;
            if constexpr (O < 64) {
                // the lanes past the owners draw too: lane group g = lane / O
                // draws sample t + LG p + g of owner lane mod O in pass p, and
                // each owner collects its draws by shuffles (the same numbers,
                // fewer Philox evaluations per lane)
                constexpr int LG = 64 / O, NP = (G + LG - 1) / LG;
                const int og = lane % O, grp = lane / O;
                const int col = min(step * (tx * O + og) + par, a.Wk - 1);
                U4 rr[NP];
#pragma unroll
                for (int p = 0; p < NP; ++p) rr[p] = draw(t + LG * p + grp, col);
#pragma unroll
                for (int m = 0; m < G; ++m) {
                    const int src = (m % LG) * O + og;
                    U4 d;
                    d.x = (uint32_t)__shfl((int)rr[m / LG].x, src);
                    d.y = (uint32_t)__shfl((int)rr[m / LG].y, src);
                    d.z = (uint32_t)__shfl((int)rr[m / LG].z, src);
                    d.w = (uint32_t)__shfl((int)rr[m / LG].w, src);
                    cg[m] = offset(t + m, d);
                }
            } else {
#pragma unroll
                for (int m = 0; m < G; ++m) cg[m] = sample(t + m);
            }
#pragma unroll
            for (int m = 0; m < G; ++m) {
                wg[m] = act && !same(cg[m], centre);
                any = any || wg[m];
            }
            if (!__any(any)) return;
            uint32_t cc[G];
            if constexpr (E::kGroups) V.template cost_belowN<G>(wg, cg, x, y, bestc, cc);
#pragma unroll
            for (int m = 0; m < G; ++m) take(wg[m], cg[m], cc[m]);
        };
        // Whole groups; what is left of a group of 6 as one of 5 or 3; then one by one.
        // us for 3 to 5 samples, three iterations, records 375 x 1242: 410, 437, 454 (all
        // one by one 433, 482, 535; in a group of 6 with places to spare 439, 448, 461);
        // bins 97 x 161: 60, 66, 70 (63, 68, 74; 71, 71, 72).  Two samples in a group of 3:
        // 122 us, one by one 116 (bins 240 x 400).
        constexpr int kRS = E::kRG;
        for (int t = 0; t < a.rs_samples;) {
            const int left = a.rs_samples - t;
            if (kRS > 1 && left >= kRS) {
                group(std::integral_constant<int, kRS>{}, t);
                t += kRS;
            } else if (kRS == 6 && left == 5) {
                group(std::integral_constant<int, kRS == 6 ? 5 : 1>{}, t);
                t += 5;
            } else if (kRS == 6 && left >= 3) {
                group(std::integral_constant<int, kRS == 6 ? 3 : 1>{}, t);
                t += 3;
            } else {
                const Hyp c0 = sample(t);
                const bool w0 = act && !same(c0, centre);
                if (__any(w0)) take(w0, c0, V.cost_below(w0, x, y, c0, bestc));
                ++t;
            }
        }
    }
    if (act) {
        reinterpret_cast<uint2*>(a.hyp)[field_off + o] = pack(best);
        a.cost[field_off + o] = bestc;
    }
}

template <int C, class E>
sff_status launch_level(const MatchArgs& a, int iters, hipStream_t st) {
    const int nz = a.ndir * a.batch;
    const int tiles_y = a.Hk;
    const dim3 block(64);
    if (a.hyp_coarse && iters == 0) {
        const int tiles_x = (a.Wk + E::kOwners - 1) / E::kOwners;
        hipLaunchKernelGGL((half_step_kernel<C, E>), dim3(tiles_x * tiles_y * nz), block, 0, st, a,
                           0, 0, 3, tiles_x, tiles_y);
        return launch_status();
    }
    const int tiles_x = ((a.Wk + 1) / 2 + E::kOwners - 1) / E::kOwners;
    for (int it = 0; it < iters; ++it)
        for (int colour = 0; colour < 2; ++colour) {
            int mode = 0;
            if (a.hyp_coarse && it == 0) mode = colour == 0 ? 1 : 2;
            hipLaunchKernelGGL((half_step_kernel<C, E>), dim3(tiles_x * tiles_y * nz), block, 0, st,
                               a, it, colour, mode, tiles_x, tiles_y);
        }
    return launch_status();
}

// Below this many pixel updates per launch (about a wave per SIMD) the chain of
// dependent round trips sets the time: all three views in one round and 16 owners
// per wave (32 where a patch has fewer than four pieces).
constexpr long kHalfOwnersMaxUpdates = 50000, kBinC1MaxUpdates = 80000;

// From this many updates per half-step a wave of the bin matcher has 64 owners
// (below: 32, groups of 4 neighbours and 3 samples, view by view); the second at
// level 0 for C >= 3.
constexpr long kBinFullMinUpdates = 200000, kBinFullMinUpdates0 = 262144;

// Bin-plane evaluators by launch size (updates per half-step), measured on the
// KITTI-size pair (C = 3, packed bins, fields on two streams from 100,000
// updates) with every shape giving identical fields; ms per level:
//  - level 2 (29,328 updates, under one wave per SIMD): all 4 neighbours and
//    all 6 samples in one group each, every view in one round, 16 owners per
//    wave: 0.16 (32 owners with the view-by-view early-out: 0.18; groups of
//    2 and 3 with 64 owners: 0.24) -- a lone wave's chain of dependent round
//    trips is what these launches wait on, so the fewest rounds and the most
//    waves win;
//  - level 1 (116,936 updates): groups of 4 neighbours and 3 samples, view by
//    view, 32 owners: 0.29 (one candidate with three views a round, 64
//    owners: 0.31);
//  - level 0 (465,750 updates): groups of 2 and 2, view by view, 64 owners: 0.70
//    (one candidate with its three views a round 0.70, groups of 2 and 3 0.71, of
//    4 and 3 0.72; 32 owners: 0.90).
// With the chip full the early-out between the views saves gathers, which set the
// time (texture data path 92 % busy), the more the coarser the level, whose patches
// lie further apart: ms per level of 16 KITTI-size pairs with one candidate and three
// views a round and now: level 2 (469,248 updates) 1.85 -> 1.29, level 1
// (1,870,976) 4.64 -> 3.66, both with groups of 4 and 3; level 0 (7,452,000) 12.4 ->
// 11.5 with 2 and 2 (4 and 3: 11.9).  C = 1 and 2 prefer 4 and 3 at level 0 too
// (3,726,000 updates, C = 1: 3.86 -> 3.20, 2 and 2 3.37; 1,863,000, C = 2: 2.61 ->
// 2.24, 2.31), C = 4 2 and 2 (1,863,000: 4.27 -> 3.77; 4 and 3 4.20).
// 64 against 32 owners, groups of 4 and 3: 233,872 updates (level 1, C = 3) 0.44 against
// 0.49, 117,312 (level 2) 0.37 against 0.32, 116,936 (level 1) 0.29 against 0.30; 2 and 2
// against them, 251,424 updates (sixteen 97 x 161 pairs, level 0) 0.57 against 0.55.
// The shortest chain wins down to the smallest calls, where each lane gathering
// its own patches (fewest instructions) had been taken below 20,000 updates; us
// per matching stage: 96 x 160, C = 1 (15,360 updates; 32 owners, three views a
// round) 170 -> 145, 16 x 16 108 -> 81, 97 x 161, C = 3, two levels 364 -> 256,
// C = 4 252 -> 214, 30 x 40, C = 3 188 -> 126.  C = 1 keeps it to 80,000
// updates (240 x 320, two levels, 76,800: 250 against 277 with 43-32; six 96 x 160
// pairs, 92,160: 309 against 305).
// Other tile orders were slower (row-major 1.10 ms at level 0, no XCD
// grouping 1.37 ms, with unpacked patches).
enum class BinShape { kLane, kSmall, k43x32, k22, k43 };

template <int C>
sff_status launch_bin_shape(BinShape shape, const MatchArgs& a, int iters, hipStream_t st) {
    switch (shape) {
        case BinShape::kLane: return launch_level<C, BinLane<C>>(a, iters, st);
        case BinShape::k43x32: return launch_level<C, PatchCoop<BinMap<C>, 4, 3, 32>>(a, iters, st);
        case BinShape::k22:
            if constexpr (C >= 3) return launch_level<C, PatchCoop<BinMap<C>, 2, 2>>(a, iters, st);
            [[fallthrough]];
        case BinShape::k43: return launch_level<C, PatchCoop<BinMap<C>, 4, 3>>(a, iters, st);
        case BinShape::kSmall: break;
    }
    return launch_level<C, PatchCoop<BinMap<C>, 4, 6, 16 * bin_pieces(C) % 64 == 0 ? 16 : 32, true>>(a, iters, st);
}

// The value of an environment variable among `names`, else -1.
int env_choice(const char* var, std::initializer_list<const char*> names) {
    const char* e = std::getenv(var);
    int i = 0;
    for (const char* n : names) {
        if (e && std::strcmp(e, n) == 0) return i;
        ++i;
    }
    return -1;
}

// The forward and inverse fields of a level are independent (each reads only
// its own field and the read-only planes), so for large launches they run as
// two launch sequences on two streams: the caller's and a helper stream of
// the library, joined to the caller's by events before and after.  A launch
// that drains (its last waves finishing while most compute units idle) then
// overlaps the other field's launch instead of the next half-step waiting for
// it: level 0 of the KITTI-size pair 0.96 -> 0.82 ms, level 1 0.345 -> 0.334
// (measured with 18-operation unpacking); below ~100,000 updates (level 2:
// 0.167 vs 0.176 ms) one launch per half-step for both fields is faster.
// Identical fields either way.
constexpr long kSplitMinUpdates = 100000;

template <class F>
sff_status run_split(const MatchArgs& a, hipStream_t st, F launch) {
    // field 0 (forward) on the caller's stream, field 1 (inverse) on the helper
    MatchArgs f0 = a, f1 = a;
    f0.ndir = f1.ndir = 1;
    f0.dir0 = 1;
    f1.dir0 = -1;
    const size_t fine = (size_t)a.batch * a.Hk * a.Wk, coarse = (size_t)a.batch * a.Hc * a.Wc;
    f1.hyp = a.hyp + 4 * fine;
    f1.cost = a.cost + fine;
    if (a.hyp_coarse) f1.hyp_coarse = a.hyp_coarse + 4 * coarse;
    HelperUse helper(st);
    if (!helper.stream()) return launch(a, st);
    const sff_status r0 = launch(f0, st);
    const sff_status r1 = launch(f1, helper.stream());
    // join even after a launch error, so the caller's stream never runs ahead
    if (!helper.join()) return SFF_ERR_HIP;
    return r0 != SFF_OK ? r0 : r1;
}

// SFF_MATCH_EVAL = "lane" (each lane gathers its own patches), "coop-46-16-xts" (the
// smallest calls' shape), "coop-43-32", "coop-22", "coop-43" (64 owners) and
// SFF_MATCH_SPLIT = "0" (one launch sequence for both fields) or "1" (two streams)
// force one (identical results; to test and time each), names of shapes that are no
// longer built the nearest one; anything else: by launch size.
template <int C>
sff_status run_bin_level(const MatchArgs& a, int iters, hipStream_t st) {
    const long updates = (long)a.ndir * a.batch * a.Hk * ((a.Wk + 1) / 2);
    // C = 3 unpacks its bins and C = 4 has as many pieces again: at level 0, where patches
    // overlap most, these are bound by the vector ALU as much as by the gathers
    const bool wide = C >= 3 && a.level == 0;
    BinShape shape = updates < (C == 1 ? kBinC1MaxUpdates : kHalfOwnersMaxUpdates) ? BinShape::kSmall
                     : updates < (wide ? kBinFullMinUpdates0 : kBinFullMinUpdates) ? BinShape::k43x32
                     : wide                                                        ? BinShape::k22
                                                                                   : BinShape::k43;
    const int eval = env_choice("SFF_MATCH_EVAL", {"lane", "coop-46-16-xts", "coop-43-32", "coop-22", "coop-43",  // as listed
                                                   "coop-xts", "coop-32", "coop-46-32", "coop"});
    constexpr BinShape kNearest[] = {BinShape::kSmall, BinShape::k43x32, BinShape::k43x32, BinShape::k43};
    if (eval >= 0) shape = eval < 5 ? (BinShape)eval : kNearest[eval - 5];
    const int forced = env_choice("SFF_MATCH_SPLIT", {"0", "1"});
    const bool split = a.ndir == 2 && (forced >= 0 ? forced == 1 : updates >= kSplitMinUpdates);
    if (!split) return launch_bin_shape<C>(shape, a, iters, st);
    return run_split(a, st, [&](const MatchArgs& f, hipStream_t fs) { return launch_bin_shape<C>(shape, f, iters, fs); });
}

// Largest descriptor map (bytes) the cooperative evaluators address (32-bit offsets).
constexpr size_t kMaxCoopMapBytes = (size_t)kNoTarget;

enum class RecShape { kLane, kSmall, k46x32 };

template <int C>
sff_status launch_rec_shape(RecShape shape, const MatchArgs& a, int iters, hipStream_t st) {
    switch (shape) {
        case RecShape::kLane: return launch_level<C, LaneEval<C>>(a, iters, st);
        case RecShape::k46x32: return launch_level<C, PatchCoop<RecMap<C>, 4, 6, 32>>(a, iters, st);
        case RecShape::kSmall: break;
    }
    if constexpr (C % 2 == 0)  // 16-owner waves need 4 or 8 pieces a record
        return launch_level<C, PatchCoop<RecMap<C>, 4, 6, 16, true>>(a, iters, st);
    else
        return launch_level<C, PatchCoop<RecMap<C>, 4, 3, 32, true>>(a, iters, st);
}

// Record evaluators by launch size (updates per half-step).  One level's records
// (64 bytes a pixel at C = 2) are beyond the L2s, and a half-step of the
// 436 x 1024 learned matcher's level 0 (446,464 updates) gathers 0.9 GB: these
// launches wait on the caches beyond them, so what pays is more gathers in flight
// (all 4 neighbours, then all 6 samples, in one group) on more waves (32 owners),
// still view by view with the early-out, and from 100,000 updates the two fields
// on two streams.  ms per 12 half-steps, before (2/3 or 4/3 groups, one launch
// sequence) and now:
//     C = 2 learned  446,464 updates 1.29 -> 1.11, 111,616 0.44 -> 0.38
//     C = 2          465,750 1.09 -> 0.91, 116,936 0.40 -> 0.36, 29,328 0.18 -> 0.17
//     C = 1          465,750 0.72 -> 0.60, 116,936 0.32 -> 0.27, 29,328 0.16 -> 0.15
//     C = 3          465,750 1.34 -> 1.26, 116,936 0.45 -> 0.41, 29,328 0.20 -> 0.20
//     C = 4          465,750 1.39 -> 1.30, 116,936 0.47 -> 0.42, 29,328 0.21 -> 0.20
// From a million updates a launch's tail no longer counts and two streams only
// share the caches (1,863,000 updates: C = 2 3.76 in one sequence and 3.78 in
// two, C = 3 4.94 and 5.03; before 3.86 and 5.07).  Below 50,000 updates the chain
// of round trips sets the time: all three views in one round, and 16 owners per
// wave where the records' pieces allow it (learned 97 x 161, 15,714 updates:
// 0.148 ms with a gather per lane, 0.113 in groups of 4/6 view by view, 0.101).
// One candidate at a time with its views in one round (the bins' choice for large
// launches): 1.63 at 446,464 updates.
// SFF_MATCH_EVAL = "lane" (each lane gathers its own records), "coop-xts" (the
// smallest calls' shape) or "coop-46-32" (also by the names of cooperative shapes that
// are no longer built) forces an evaluator, SFF_MATCH_SPLIT the split (identical
// results; to test and time each); anything else: by launch size.
constexpr long kRecSplitMaxUpdates = 1000000;
template <int C>
sff_status run_level(const MatchArgs& a, int iters, hipStream_t st) {
    const long updates = (long)a.ndir * a.batch * a.Hk * ((a.Wk + 1) / 2);
    RecShape shape = updates < kHalfOwnersMaxUpdates ? RecShape::kSmall : RecShape::k46x32;
    const int eval = env_choice("SFF_MATCH_EVAL", {"lane", "coop-xts", "coop-46-32",  // as listed
                                                   "coop", "coop-narrow", "coop-wide", "coop-narrow-32", "coop-wide-32"});
    if (eval >= 0) shape = (RecShape)std::min(eval, (int)RecShape::k46x32);
    if (a.img_bytes > kMaxCoopMapBytes) shape = RecShape::kLane;
    const int forced = env_choice("SFF_MATCH_SPLIT", {"0", "1"});
    const bool split =
        a.ndir == 2 && (forced >= 0 ? forced == 1 : updates >= kSplitMinUpdates && updates < kRecSplitMaxUpdates);
    if (!split) return launch_rec_shape<C>(shape, a, iters, st);
    return run_split(a, st, [&](const MatchArgs& f, hipStream_t fs) { return launch_rec_shape<C>(shape, f, iters, fs); });
}

}  // namespace
}  // namespace sff

using namespace sff;

extern "C" sff_status sff_match_level(const sff_params* p, int32_t batch, int32_t dir,
                                      int32_t level, const int16_t* desc, const uint64_t* seeds,
                                      const int16_t* hyp_coarse, int16_t* hyp, uint32_t* cost,
                                      void* stream) {
    if (!params_ok(p) || batch < 1 || batch > 32767 || (dir != 1 && dir != -1 && dir != 0) ||
        level < 0 || level >= p->levels || !desc || !seeds || !hyp || !cost)
        return SFF_ERR_INVALID_ARG;
    if (hyp_coarse && level >= p->levels - 1) return SFF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(desc) & 15) != 0 || (reinterpret_cast<uintptr_t>(hyp) & 7) != 0 ||
        (reinterpret_cast<uintptr_t>(cost) & 3) != 0 ||
        (reinterpret_cast<uintptr_t>(hyp_coarse) & 7) != 0)
        return SFF_ERR_INVALID_ARG;
    const LevelGeom g = level_geom(*p, level);
    const int ndir = dir == 0 ? 2 : 1;
    const size_t fine_bytes = (size_t)ndir * batch * g.Hk * g.Wk * 8;
    if (hyp_coarse) {
        const LevelGeom gc = level_geom(*p, level + 1);
        const size_t coarse_bytes = (size_t)ndir * batch * gc.Hk * gc.Wk * 8;
        const uintptr_t f0 = reinterpret_cast<uintptr_t>(hyp), f1 = f0 + fine_bytes;
        const uintptr_t c0 = reinterpret_cast<uintptr_t>(hyp_coarse), c1 = c0 + coarse_bytes;
        if (f0 < c1 && c0 < f1) return SFF_ERR_INVALID_ARG;
    }
    MatchArgs a;
    a.maps = reinterpret_cast<const uint8_t*>(desc);
    a.img_bytes = (size_t)p->H * p->W * rec_channels(p->C) * 32;
    a.sh = a.Hq = a.Wq = 0;
    a.seeds = seeds;
    a.hyp_coarse = hyp_coarse;
    a.hyp = hyp;
    a.cost = cost;
    a.H = p->H;
    a.W = p->W;
    a.n = g.n;
    a.level = level;
    a.Hk = g.Hk;
    a.Wk = g.Wk;
    if (hyp_coarse) {
        const LevelGeom gc = level_geom(*p, level + 1);
        a.Hc = gc.Hk;
        a.Wc = gc.Wk;
    } else {
        a.Hc = a.Wc = 0;
    }
    a.rs_r0 = p->rs_r0;
    a.rs_samples = p->rs_samples;
    a.fmax = p->fmax;
    a.dmax = p->dmax;
    a.batch = batch;
    a.ndir = ndir;
    a.dir0 = dir == 0 ? 1 : dir;
    hipStream_t st = as_stream(stream);
    switch (p->C) {
        case 1: return run_level<1>(a, p->iters, st);
        case 2: return run_level<2>(a, p->iters, st);
        case 3: return run_level<3>(a, p->iters, st);
        default: return run_level<4>(a, p->iters, st);
    }
}

extern "C" sff_status sff_match_level_bins(const sff_params* p, int32_t batch, int32_t dir,
                                           int32_t level, const uint16_t* bins, const uint64_t* seeds,
                                           const int16_t* hyp_coarse, int16_t* hyp, uint32_t* cost,
                                           void* stream) {
    if (!params_ok(p) || batch < 1 || batch > 32767 || (dir != 1 && dir != -1 && dir != 0) ||
        level < 0 || level >= p->levels || !bins || !seeds || !hyp || !cost)
        return SFF_ERR_INVALID_ARG;
    if (hyp_coarse && level >= p->levels - 1) return SFF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(bins) & 15) != 0 || (reinterpret_cast<uintptr_t>(hyp) & 7) != 0 ||
        (reinterpret_cast<uintptr_t>(cost) & 3) != 0 ||
        (reinterpret_cast<uintptr_t>(hyp_coarse) & 7) != 0)
        return SFF_ERR_INVALID_ARG;
    const size_t img_bytes = bin_image_bytes(*p, level);
    if (img_bytes > (size_t)kNoTarget) return SFF_ERR_UNSUPPORTED;  // 32-bit gather offsets
    const LevelGeom g = level_geom(*p, level);
    const BinGeom bg = bin_geom(*p, level);
    const int ndir = dir == 0 ? 2 : 1;
    const size_t fine_bytes = (size_t)ndir * batch * g.Hk * g.Wk * 8;
    MatchArgs a;
    if (hyp_coarse) {
        const LevelGeom gc = level_geom(*p, level + 1);
        const size_t coarse_bytes = (size_t)ndir * batch * gc.Hk * gc.Wk * 8;
        const uintptr_t f0 = reinterpret_cast<uintptr_t>(hyp), f1 = f0 + fine_bytes;
        const uintptr_t c0 = reinterpret_cast<uintptr_t>(hyp_coarse), c1 = c0 + coarse_bytes;
        if (f0 < c1 && c0 < f1) return SFF_ERR_INVALID_ARG;
        a.Hc = gc.Hk;
        a.Wc = gc.Wk;
    } else {
        a.Hc = a.Wc = 0;
    }
    a.maps = reinterpret_cast<const uint8_t*>(bins);
    a.img_bytes = img_bytes;
    a.seeds = seeds;
    a.hyp_coarse = hyp_coarse;
    a.hyp = hyp;
    a.cost = cost;
    a.H = p->H;
    a.W = p->W;
    a.n = g.n;
    a.level = level;
    a.Hk = g.Hk;
    a.Wk = g.Wk;
    a.sh = bg.sh;
    a.Hq = bg.Hq;
    a.Wq = bg.Wq;
    a.rs_r0 = p->rs_r0;
    a.rs_samples = p->rs_samples;
    a.fmax = p->fmax;
    a.dmax = p->dmax;
    a.batch = batch;
    a.ndir = ndir;
    a.dir0 = dir == 0 ? 1 : dir;
    hipStream_t st = as_stream(stream);
    switch (p->C) {
        case 1: return run_bin_level<1>(a, p->iters, st);
        case 2: return run_bin_level<2>(a, p->iters, st);
        case 3: return run_bin_level<3>(a, p->iters, st);
        default: return run_bin_level<4>(a, p->iters, st);
    }
}
