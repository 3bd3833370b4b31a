// Window form of the matching cost on real-valued feature maps and its
// gradient (SceneFlowFields, Section 3.1, eq. (1): feature distances summed
// over a window around the pixel for the temporal, stereo and cross
// correspondences; replicated borders).
//
//   cost(p) = sum_corr sum_{w in {-3..4}^2} sum_c
//             (F_R(clamp(p + w), c) - F_corr(clamp(t_corr(p) + w), c))^2,
//   t_corr(p) = clamp(p + o_corr(h_p)),  o_T = (u, v), o_S = (-s d0, 0),
//   o_X = (u - s d1, v).
//
// Backward for L = sum_p g_p cost(p): each term with difference delta adds
// 2 g_p delta to the reference entry and subtracts it from the target entry.
//   * reference map: a gather over the preimage {(p, w) : clamp(p + w) = q};
//   * target maps: pixels are grouped by their (clamped) target centre with a
//     stable radix sort (hand-written, 8-bit digits), then every target entry
//     gathers over the centres whose window covers it.
// Both are deterministic (no floating-point atomics).
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <optional>
#include <type_traits>

#include "sff_internal.hpp"

namespace sff {
namespace {

constexpr int kWin0 = -3, kWin1 = 4;  // window offsets, the descriptors' 8x8 patch

struct CostArgs {
    const float* feat;      // [batch][4][H][W][CF]
    const int16_t* hyp;     // [batch][H][W][4]
    const float* gcost;     // [batch][H][W] (backward)
    float* out;             // cost [batch][H][W] or gradient [batch][4][H][W][CF]
    int H, W, s, batch;
};

template <int CF>
__device__ __forceinline__ void load_vec(const float* __restrict__ f, float* v) {
    const float4* p = reinterpret_cast<const float4*>(f);
#pragma unroll
    for (int k = 0; k < CF / 4; ++k) {
        const float4 x = p[k];
        v[4 * k] = x.x;
        v[4 * k + 1] = x.y;
        v[4 * k + 2] = x.z;
        v[4 * k + 3] = x.w;
    }
}

__device__ __forceinline__ int view(int s, int role) {  // canonical map of R, T, S, X
    return s > 0 ? role : 3 - role;
}

struct Targets {
    int y[3], x[3];
};

__device__ __forceinline__ Targets targets(const int16_t* hyp, size_t pix, int y, int x, int s,
                                           int H, int W) {
    const uint2 h = reinterpret_cast<const uint2*>(hyp)[pix];
    const int u = (int16_t)(h.x & 0xFFFFu), v = (int16_t)(h.x >> 16);
    const int d0 = (int16_t)(h.y & 0xFFFFu), d1 = (int16_t)(h.y >> 16);
    Targets t;
    t.y[0] = clampi(y + v, 0, H - 1);
    t.x[0] = clampi(x + u, 0, W - 1);
    t.y[1] = y;
    t.x[1] = clampi(x - s * d0, 0, W - 1);
    t.y[2] = t.y[0];
    t.x[2] = clampi(x + u - s * d1, 0, W - 1);
    return t;
}

// One thread per pixel; block = 64 pixels of 4 rows.  Partial sums per window
// position, then per window row, keep the FP32 rounding error near 10^-5.
template <int CF>
__global__ void __launch_bounds__(256) cost_fwd_kernel(CostArgs a) {
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int b = blockIdx.z;
    if (x >= a.W || y >= a.H) return;
    const int H = a.H, W = a.W;
    const size_t HW = (size_t)H * W;
    const float* base = a.feat + (size_t)b * 4 * HW * CF;
    const float* R = base + (size_t)view(a.s, 0) * HW * CF;
    const float* M[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) M[k] = base + (size_t)view(a.s, k + 1) * HW * CF;
    const Targets t = targets(a.hyp, (size_t)b * HW + (size_t)y * W + x, y, x, a.s, H, W);
    float total = 0.f;
    for (int dy = kWin0; dy <= kWin1; ++dy) {
        const int ry = clampi(y + dy, 0, H - 1);
        int ty[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) ty[k] = clampi(t.y[k] + dy, 0, H - 1);
        float rsum = 0.f;
        for (int dx = kWin0; dx <= kWin1; ++dx) {
            float ref[CF];
            load_vec<CF>(R + ((size_t)ry * W + clampi(x + dx, 0, W - 1)) * CF, ref);
            float psum = 0.f;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                float tg[CF];
                load_vec<CF>(M[k] + ((size_t)ty[k] * W + clampi(t.x[k] + dx, 0, W - 1)) * CF, tg);
#pragma unroll
                for (int c = 0; c < CF; ++c) {
                    const float d = ref[c] - tg[c];
                    psum = fmaf(d, d, psum);
                }
            }
            rsum += psum;
        }
        total += rsum;
    }
    a.out[(size_t)b * HW + (size_t)y * W + x] = total;
}

// The same cost with CF / 4 lanes per pixel, four channels each: a gathered
// vector is CF / 4 neighbouring 16-byte loads.  Each lane sums its channels
// in the nested order above; the CF / 4 lane sums are combined by an xor
// butterfly (every lane ends with the same value), so the result is
// deterministic; it rounds differently from cost_fwd_kernel (within the same
// error bound).
template <int CF>
__global__ void __launch_bounds__(256) cost_fwd_coop_kernel(CostArgs a) {
    constexpr int L = CF / 4, QPB = 256 / L;
    const int sub = threadIdx.x % L;
    const int H = a.H, W = a.W, b = blockIdx.y;
    const size_t HW = (size_t)H * W;
    const size_t q = (size_t)xcd_tile(blockIdx.x, gridDim.x) * QPB + threadIdx.x / L;  // a band of rows per XCD
    if (q >= HW) return;  // all L lanes of the pixel together
    const int y = (int)(q / W), x = (int)(q - (size_t)y * W);
    const float* base = a.feat + (size_t)b * 4 * HW * CF;
    const float4* R = reinterpret_cast<const float4*>(base + (size_t)view(a.s, 0) * HW * CF) + sub;
    const float4* M[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) M[k] = reinterpret_cast<const float4*>(base + (size_t)view(a.s, k + 1) * HW * CF) + sub;
    const Targets t = targets(a.hyp, (size_t)b * HW + q, y, x, a.s, H, W);
    float total = 0.f;
    for (int dy = kWin0; dy <= kWin1; ++dy) {
        const int ry = clampi(y + dy, 0, H - 1);
        int ty[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) ty[k] = clampi(t.y[k] + dy, 0, H - 1);
        float rsum = 0.f;
        for (int dx = kWin0; dx <= kWin1; ++dx) {
            const float4 r = R[((size_t)ry * W + clampi(x + dx, 0, W - 1)) * L];
            float psum = 0.f;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float4 tg = M[k][((size_t)ty[k] * W + clampi(t.x[k] + dx, 0, W - 1)) * L];
                const float d0 = r.x - tg.x, d1 = r.y - tg.y, d2 = r.z - tg.z, d3 = r.w - tg.w;
                psum = fmaf(d0, d0, psum);
                psum = fmaf(d1, d1, psum);
                psum = fmaf(d2, d2, psum);
                psum = fmaf(d3, d3, psum);
            }
            rsum += psum;
        }
        total += rsum;
    }
#pragma unroll
    for (int off = L / 2; off >= 1; off >>= 1) total += __shfl_xor(total, off, L);
    if (sub == 0) a.out[(size_t)b * HW + q] = total;
}

// Preimage of the clamped coordinate: {p in [0, n) : clamp(p + w, 0, n - 1) = q}.
__device__ __forceinline__ void preimage(int q, int w, int n, int& lo, int& hi) {
    if (n == 1) {
        lo = hi = 0;
        return;
    }
    if (q == 0) {
        lo = 0;
        hi = min(-w, n - 1);
    } else if (q == n - 1) {
        lo = max(n - 1 - w, 0);
        hi = n - 1;
    } else {
        lo = hi = q - w;
        if (lo < 0 || lo > n - 1) hi = lo - 1;  // empty
    }
}

// The gradient entries gather their terms in row_split(CF) parts of
// consecutive window rows, summed alone and then added in pairs: eight
// single rows up to 32 channels, four pairs of rows at 64 (the CF / 4 lanes of
// every part of an entry share one wave).
constexpr int row_split(int cf) { return cf <= 32 ? 8 : 4; }
constexpr int kWinN = kWin1 - kWin0 + 1;  // 8 window rows and columns

// The parts of an entry added in pairs, pairs of pairs, ...: into part 0.
template <int S, int CF>
__device__ __forceinline__ void pair_sums(float (&acc)[S][CF]) {
#pragma unroll
    for (int d = 1; d < S; d *= 2)
#pragma unroll
        for (int t = 0; t < S; t += 2 * d)
#pragma unroll
            for (int c = 0; c < CF; ++c) acc[t][c] += acc[t + d][c];
}

// Reference-map gradient, one thread per entry q of R (testing and timing).
// The terms of q are the (p, w) with clamp(p + w) = q, taken by window row wy,
// preimage row py, window column wx, preimage column px and correspondence;
// each part of the window rows is summed alone, then the parts in pairs.
template <int CF>
__global__ void __launch_bounds__(256) grad_ref_kernel(CostArgs a) {
    const int qx = blockIdx.x * 64 + (threadIdx.x & 63);
    const int qy = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int b = blockIdx.z;
    if (qx >= a.W || qy >= a.H) return;
    const int H = a.H, W = a.W;
    const size_t HW = (size_t)H * W;
    const float* base = a.feat + (size_t)b * 4 * HW * CF;
    const int mR = view(a.s, 0);
    const float* M[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) M[k] = base + (size_t)view(a.s, k + 1) * HW * CF;
    constexpr int kSplit = row_split(CF), kPartRows = kWinN / kSplit;
    float fq[CF], part_acc[kSplit][CF];
    load_vec<CF>(base + ((size_t)mR * HW + (size_t)qy * W + qx) * CF, fq);
#pragma unroll
    for (int part = 0; part < kSplit; ++part) {
        float(&acc)[CF] = part_acc[part];
#pragma unroll
        for (int c = 0; c < CF; ++c) acc[c] = 0.f;
        for (int wy = kWin0 + part * kPartRows; wy < kWin0 + (part + 1) * kPartRows; ++wy) {
            int ylo, yhi;
            preimage(qy, wy, H, ylo, yhi);
            for (int py = ylo; py <= yhi; ++py)
                for (int wx = kWin0; wx <= kWin1; ++wx) {
                    int xlo, xhi;
                    preimage(qx, wx, W, xlo, xhi);
                    for (int px = xlo; px <= xhi; ++px) {
                        const size_t pix = (size_t)b * HW + (size_t)py * W + px;
                        const float g2 = 2.f * a.gcost[pix];
                        const Targets t = targets(a.hyp, pix, py, px, a.s, H, W);
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            float tg[CF];
                            load_vec<CF>(M[k] + ((size_t)clampi(t.y[k] + wy, 0, H - 1) * W +
                                                 clampi(t.x[k] + wx, 0, W - 1)) * CF, tg);
#pragma unroll
                            for (int c = 0; c < CF; ++c) acc[c] = fmaf(g2, fq[c] - tg[c], acc[c]);
                        }
                    }
                }
        }
    }
    pair_sums<kSplit, CF>(part_acc);
    const float(&sum)[CF] = part_acc[0];
    float4* o = reinterpret_cast<float4*>(a.out + ((size_t)b * 4 * HW + (size_t)mR * HW +
                                                   (size_t)qy * W + qx) * CF);
#pragma unroll
    for (int k = 0; k < CF / 4; ++k) o[k] = make_float4(sum[4 * k], sum[4 * k + 1], sum[4 * k + 2], sum[4 * k + 3]);
}

__device__ __forceinline__ void grad_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Grouping of the pixels by target centre, all three correspondences in one
// list: element k * n + i (pixel i of the batch, n pixels) has the key
// k * n + (centre cell of correspondence k) and the value i.  After a stable
// sort by key, the pixels of each centre cell are in ascending pixel order.
// A thread takes a pixel and writes its three elements (375 x 1242: 6 us; a thread
// per element with 64-bit divisions 38).
__global__ void __launch_bounds__(256) target_keys_kernel(const int16_t* __restrict__ hyp, uint32_t* __restrict__ keys,
                                                          uint32_t* __restrict__ vals, int H, int W, int s, uint32_t n) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= n) return;
    const uint32_t HW = (uint32_t)H * W, b = i / HW, pix = i - b * HW;
    const int y = (int)(pix / W), x = (int)(pix - (uint32_t)y * W);
    const Targets t = targets(hyp, i, y, x, s, H, W);
#pragma unroll
    for (uint32_t k = 0; k < 3; ++k) {
        const size_t e = (size_t)k * n + i;
        keys[e] = k * n + b * HW + (uint32_t)t.y[k] * W + t.x[k];
        vals[e] = i;
    }
}

// Least-significant-digit radix sort of (key, value) pairs, 8-bit digits, one
// pass = histogram per block, exclusive scan over (digit, block), stable
// scatter.  A block of 4 waves takes kSortTile consecutive elements.
constexpr int kSortTile = 2048;

__global__ void __launch_bounds__(256) sort_hist_kernel(const uint32_t* __restrict__ keys, size_t N,
                                                        int sh, uint32_t* __restrict__ hist,
                                                        uint32_t nblk) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const size_t base = (size_t)blockIdx.x * kSortTile;
    for (int j = 0; j < kSortTile / 256; ++j) {
        const size_t i = base + (size_t)j * 256 + threadIdx.x;
        if (i < N) atomicAdd(&h[(keys[i] >> sh) & 255u], 1u);
    }
    __syncthreads();
    hist[(size_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// Exclusive prefix sum of v over the 1024 threads of the block; *total gets
// the sum.
__device__ uint32_t block_scan_1024(uint32_t v, uint32_t* total) {
    __shared__ uint32_t wsum[16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(x, off);
        if (lane >= off) x += t;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    if (w == 0) {
        uint32_t y = lane < 16 ? wsum[lane] : 0u;
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const uint32_t t = __shfl_up(y, off);
            if (lane >= off) y += t;
        }
        if (lane < 16) wsum[lane] = y;  // inclusive
    }
    __syncthreads();
    const uint32_t before = w ? wsum[w - 1] : 0u;
    *total = wsum[15];
    __syncthreads();  // wsum is reused by the next call
    return before + x - v;
}

// Exclusive scan of h[0 .. total) in two steps: each block of 1024 threads
// scans its chunk of 1024 entries in place and writes the chunk's sum; one
// block then scans the chunk sums (sort_scan_sums_kernel).  A scanned entry
// is h[i] + sums[i / 1024].
__global__ void __launch_bounds__(1024) sort_scan_chunks_kernel(uint32_t* __restrict__ h, size_t total,
                                                                uint32_t* __restrict__ sums) {
    const size_t i = (size_t)blockIdx.x * 1024 + threadIdx.x;
    const uint32_t v = i < total ? h[i] : 0u;
    uint32_t sum;
    const uint32_t ex = block_scan_1024(v, &sum);
    if (i < total) h[i] = ex;
    if (threadIdx.x == 0) sums[blockIdx.x] = sum;
}

__global__ void __launch_bounds__(1024) sort_scan_sums_kernel(uint32_t* __restrict__ sums, size_t nchunks) {
    uint32_t run = 0;
    for (size_t c = 0; c < nchunks; c += 1024) {
        const size_t i = c + threadIdx.x;
        const uint32_t v = i < nchunks ? sums[i] : 0u;
        uint32_t sum;
        const uint32_t ex = block_scan_1024(v, &sum);
        if (i < nchunks) sums[i] = run + ex;
        run += sum;
    }
}

// Stable scatter of one pass.  A wave takes a run of kSortTile / 4 consecutive
// elements, 64 at a time and all loaded at the start: it counts its digits, and
// after one barrier knows where each of its digits begins; the rank among 64
// comes from the lanes with the same digit.  Bound: the scattered stores and a
// chain of ballots per 64 elements.  375 x 1242 (1.4 M elements), beside the
// reference gradient: 31 us a pass; 49 with
// 256 elements of the block a round between three barriers and their loads.
__global__ void __launch_bounds__(256) sort_scatter_kernel(const uint32_t* __restrict__ kin,
                                                           const uint32_t* __restrict__ vin,
                                                           uint32_t* __restrict__ kout,
                                                           uint32_t* __restrict__ vout, size_t N,
                                                           int sh, const uint32_t* __restrict__ scan,
                                                           const uint32_t* __restrict__ sums,
                                                           uint32_t nblk) {
    constexpr int kRounds = kSortTile / 256;
    __shared__ uint32_t wc[4][256];  // counts, then positions, of a wave's digits
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const size_t hi = (size_t)t * nblk + blockIdx.x;
    const uint32_t start = scan[hi] + sums[hi / 1024];
    const size_t base = (size_t)blockIdx.x * kSortTile + (size_t)w * (kSortTile / 4) + lane;
    uint32_t key[kRounds], val[kRounds];
#pragma unroll
    for (int j = 0; j < kRounds; ++j) {
        const size_t i = base + 64 * j;
        key[j] = i < N ? kin[i] : 0u;
        val[j] = i < N ? vin[i] : 0u;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) wc[q][t] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kRounds; ++j)
        if (base + 64 * j < N) atomicAdd(&wc[w][(key[j] >> sh) & 255u], 1u);
    __syncthreads();
    {
        uint32_t p = start;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t c = wc[q][t];
            wc[q][t] = p;
            p += c;
        }
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int j = 0; j < kRounds; ++j) {
        const bool ok = base + 64 * j < N;
        const uint32_t d = (key[j] >> sh) & 255u;
        uint64_t m = __ballot(ok);
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const bool on = (d >> bit) & 1u;
            const uint64_t bb = __ballot(on);
            m &= on ? bb : ~bb;
        }
        const uint32_t rank = (uint32_t)__popcll(m & below), cnt = (uint32_t)__popcll(m);
        const uint32_t at = wc[w][d];
        grad_wave_sync();
        if (ok) {
            kout[at + rank] = key[j];
            vout[at + rank] = val[j];
            if (rank == cnt - 1) wc[w][d] = at + cnt;  // the group's last lane
        }
        grad_wave_sync();
    }
}

// start[c] = first position of a sorted key >= c, for every cell c in [0, N].  A
// block of 256 cells first finds the positions of its first cell and of the cell
// past its last (64 probes a step), then each cell searches between them.
// 375 x 1242: 37 us; 51 with a binary search over all keys per cell.
__global__ void __launch_bounds__(256) cell_starts_kernel(const uint32_t* __restrict__ keys, uint32_t* __restrict__ start,
                                                          size_t N) {
    __shared__ size_t ends[2];
    const size_t c0 = (size_t)blockIdx.x * 256, c = c0 + threadIdx.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (w < 2) {
        const size_t want = c0 + 256 * (size_t)w;
        size_t lo = 0, hi = N;  // the answer is in [lo, hi]
        while (lo < hi) {
            // probe l is the last of the first (l + 1) / 64 of the range
            const size_t len = hi - lo, p = lo + (len * (size_t)(lane + 1) + 63) / 64 - 1;
            const uint64_t less = __ballot((size_t)keys[p] < want);  // a prefix of the lanes
            const int k = __popcll(less);
            const size_t l0 = lo;
            if (k > 0) lo = l0 + (len * (size_t)k + 63) / 64;
            if (k < 64) hi = l0 + (len * (size_t)(k + 1) + 63) / 64 - 1;
        }
        if (lane == 0) ends[w] = lo;
    }
    __syncthreads();
    if (c > N) return;
    size_t lo = ends[0], hi = ends[1];
    while (lo < hi) {
        const size_t mid = lo + (hi - lo) / 2;
        if ((size_t)keys[mid] < c) lo = mid + 1;
        else hi = mid;
    }
    start[c] = (uint32_t)lo;
}

// Gradient of target map k, one thread per entry q of that map (testing and
// timing).  The terms of q are the (pixel, w) with clamp(centre + w) = q, in
// the canonical order: window row wy ascending, cell row ty of its preimage
// ascending, window column wx descending (cells by ascending x), cell column
// tx of its preimage ascending, the pixels grouped at the cell in sorted
// order.  Term i goes to accumulator i mod row_split(CF); the accumulators are
// added in pairs.  (Dealing the terms round-robin keeps the
// tiled kernel's lanes busy however unevenly the pixels crowd the cells.)
template <int CF>
__global__ void __launch_bounds__(256) grad_target_kernel(CostArgs a, int k, size_t n,
                                                          const uint32_t* __restrict__ start,
                                                          const uint32_t* __restrict__ order) {
    const int qx = blockIdx.x * 64 + (threadIdx.x & 63);
    const int qy = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int b = blockIdx.z;
    if (qx >= a.W || qy >= a.H) return;
    const int H = a.H, W = a.W;
    const size_t HW = (size_t)H * W;
    const float* base = a.feat + (size_t)b * 4 * HW * CF;
    const float* R = base + (size_t)view(a.s, 0) * HW * CF;
    const int mk = view(a.s, k + 1);
    constexpr int S = row_split(CF);
    float fq[CF], acc[S][CF];
    load_vec<CF>(base + ((size_t)mk * HW + (size_t)qy * W + qx) * CF, fq);
#pragma unroll
    for (int t = 0; t < S; ++t)
#pragma unroll
        for (int c = 0; c < CF; ++c) acc[t][c] = 0.f;
    uint32_t i = 0;
    for (int wy = kWin0; wy <= kWin1; ++wy) {
        int ylo, yhi;
        preimage(qy, wy, H, ylo, yhi);
        for (int ty = ylo; ty <= yhi; ++ty)
            for (int wx = kWin1; wx >= kWin0; --wx) {
                int xlo, xhi;
                preimage(qx, wx, W, xlo, xhi);
                for (int tx = xlo; tx <= xhi; ++tx) {
                    const size_t cell = (size_t)k * n + (size_t)b * HW + (size_t)ty * W + tx;
                    const uint32_t e0 = start[cell], e1 = start[cell + 1];
                    for (uint32_t e = e0; e < e1; ++e, ++i) {
                        const uint32_t pix = order[e];
                        const int pl = (int)(pix - (size_t)b * HW);
                        const int py = pl / W, px = pl - py * W;
                        const float g2 = 2.f * a.gcost[pix];
                        float r[CF];
                        load_vec<CF>(R + ((size_t)clampi(py + wy, 0, H - 1) * W +
                                          clampi(px + wx, 0, W - 1)) * CF, r);
                        float* ac = acc[i % S];
#pragma unroll
                        for (int c = 0; c < CF; ++c) ac[c] = fmaf(-g2, r[c] - fq[c], ac[c]);
                    }
                }
            }
    }
    float4* o = reinterpret_cast<float4*>(a.out + ((size_t)b * 4 * HW + (size_t)mk * HW +
                                                   (size_t)qy * W + qx) * CF);
    pair_sums<S, CF>(acc);
#pragma unroll
    for (int kk = 0; kk < CF / 4; ++kk)
        o[kk] = make_float4(acc[0][4 * kk], acc[0][4 * kk + 1], acc[0][4 * kk + 2], acc[0][4 * kk + 3]);
}

// Tiled gradient kernels: a block takes kTileQ consecutive entries of one row
// of one map and first stages in LDS what all of them read besides the
// gathered feature vectors; then CF / 4 lanes (four channels each) per part
// of the window rows and row_split(CF) parts per entry gather the vectors and
// add the same terms in the same order as the one-thread kernels (each part
// alone, then the parts in pairs by exchanges), so the results are identical.
// Tiles are numbered ((map * batch + b) * H + row) * tiles_x + column tile and
// given out by XCD, so an XCD's L2 holds a band of rows.
constexpr int kTileQ = 32;
constexpr int kTileC = kTileQ + kWinN - 1;  // staged columns: the tile's and the window's
constexpr int kStageCap = 2048;             // staged pixels per target-gradient tile
constexpr int kMaxRuns = 15 * 15;           // (window row, cell row) by (window column, cell column) at a corner

// Add the four-channel part of the terms of one pixel: fma(g, x - y, acc).
__device__ __forceinline__ void fma4(float g, const float4& x, const float4& y, float4& acc) {
    acc.x = fmaf(g, x.x - y.x, acc.x);
    acc.y = fmaf(g, x.y - y.y, acc.y);
    acc.z = fmaf(g, x.z - y.z, acc.z);
    acc.w = fmaf(g, x.w - y.w, acc.w);
}

// One image's feature map read 16 bytes per lane, at the vector with the given
// unit: its byte offset (BUF: a raw buffer with 32-bit offsets, maps below 2
// GiB; kSkipOff reads nothing) or its index in 16-byte pieces.
constexpr int kSkipOff = 0x7FFFFFF0;
template <bool BUF>
struct Vec4Map {
    const float4* p;
    __amdgpu_buffer_rsrc_t rs;
    __device__ __forceinline__ void init(const float* base, size_t bytes) {
        p = reinterpret_cast<const float4*>(base);
        if constexpr (BUF) {
            const uint64_t a = reinterpret_cast<uint64_t>(base);
            const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a) |
                               ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) << 32);
            rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), (short)0,
                                                   (int)__builtin_amdgcn_readfirstlane((uint32_t)bytes),
                                                   0x00020000);
        }
    }
    // Unit of the vector of pixel i, L pieces of 16 bytes per vector.
    template <int L>
    __device__ __forceinline__ static uint32_t unit(int i) {
        return (uint32_t)i * (BUF ? 16u * L : (uint32_t)L);
    }
    // Piece `sub` of the vector at unit u.
    __device__ __forceinline__ float4 ld(uint32_t u, int sub) const {
        if constexpr (BUF) {
            const uint4 v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(u + 16u * sub), 0, 0));
            return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z),
                               __uint_as_float(v.w));
        } else {
            return p[u + sub];
        }
    }
};

// Sum of the entry's parts (groups of L lanes), in pairs, in all its lanes.
template <int kSplit, int L>
__device__ __forceinline__ float4 sum_parts(float4 v) {
#pragma unroll
    for (int d = 1; d < kSplit; d *= 2) {
        v.x += __shfl_xor(v.x, d * L);
        v.y += __shfl_xor(v.y, d * L);
        v.z += __shfl_xor(v.z, d * L);
        v.w += __shfl_xor(v.w, d * L);
    }
    return v;
}

// Reference-map gradient: the tile stages 2 g and the three target centres of
// the pixels its entries' windows reach (8 rows by kTileC columns).
template <int CF, bool BUF>
__global__ void __launch_bounds__(256) grad_ref_tile_kernel(CostArgs a, int tiles_x) {
    constexpr int kSplit = row_split(CF), kPartRows = kWinN / kSplit;
    constexpr int L = CF / 4, G = kSplit * L, EPB = 256 / G;
    static_assert(G <= 64 && 64 % G == 0, "the parts of an entry share one wave");
    using Map = Vec4Map<BUF>;
    __shared__ float s_g[kWinN][kTileC];
    __shared__ uint32_t s_t[3][kWinN][kTileC];  // (ty << 16) | tx
    __shared__ uint4 s_d[kWinN][kTileC];        // unit of each centre less the pixel's, and 2 g
    __shared__ float4 s_fq[kTileQ * L];         // the entries' own vectors
    const int H = a.H, W = a.W;
    const size_t HW = (size_t)H * W;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int tq = tile % tiles_x, rest = tile / tiles_x;
    const int qy = rest % H, b = rest / H;
    const int qx0 = tq * kTileQ;
    const int py0 = qy - kWin1, px0 = qx0 - kWin1;  // staged pixel (0, 0)
    bool clamps = false;  // a window of this thread's pixels leaves the image
    for (int idx = threadIdx.x; idx < kWinN * kTileC; idx += 256) {
        const int r = idx / kTileC, c = idx - r * kTileC;
        const int py = py0 + r, px = px0 + c;
        if (py < 0 || py >= H || px < 0 || px >= W) continue;
        const size_t pix = (size_t)b * HW + (size_t)py * W + px;
        s_g[r][c] = 2.f * a.gcost[pix];
        const Targets t = targets(a.hyp, pix, py, px, a.s, H, W);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            s_t[k][r][c] = ((uint32_t)t.y[k] << 16) | (uint32_t)t.x[k];
            clamps = clamps || t.y[k] + kWin0 < 0 || t.y[k] + kWin1 >= H || t.x[k] + kWin0 < 0 || t.x[k] + kWin1 >= W;
        }
        const uint32_t self = Map::template unit<L>(py * W + px);
        s_d[r][c] = make_uint4(Map::template unit<L>(t.y[0] * W + t.x[0]) - self,
                               Map::template unit<L>(t.y[1] * W + t.x[1]) - self,
                               Map::template unit<L>(t.y[2] * W + t.x[2]) - self, __float_as_uint(s_g[r][c]));
    }
    const float* base = a.feat + (size_t)b * 4 * HW * CF;
    const int mR = view(a.s, 0);
    for (int idx = threadIdx.x; idx < kTileQ * L; idx += 256) {
        const int qx = qx0 + idx / L;
        if (qx < W)
            s_fq[idx] = reinterpret_cast<const float4*>(base + ((size_t)mR * HW + (size_t)qy * W + qx) * CF)[idx % L];
    }
    clamps = __syncthreads_or(clamps);
    Map M[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) M[k].init(base + (size_t)view(a.s, k + 1) * HW * CF, HW * CF * 4);
    const int sub = threadIdx.x % L, part = (threadIdx.x / L) % kSplit;
    const int wy0 = kWin0 + part * kPartRows;
    for (int e0 = 0; e0 < kTileQ; e0 += EPB) {
        const int qx = qx0 + e0 + (int)threadIdx.x / G;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        const bool live = qx < W && qx < qx0 + kTileQ;
        const size_t q = (size_t)qy * W + qx;
        float4 fq = make_float4(0.f, 0.f, 0.f, 0.f);
        if (live) fq = s_fq[(qx - qx0) * L + sub];
        if (live && qy >= kWin1 && qy <= H - 1 + kWin0 && qx >= kWin1 && qx <= W - 1 + kWin0) {
            // interior: the preimage of q under w is the one pixel q - w; half a
            // window row, 12 gathers, at a time: fewer registers, more waves
            constexpr int JH = kWinN / 2;
            const uint32_t uq = Map::template unit<L>((int)q);
            for (int wy = wy0; wy < wy0 + kPartRows; ++wy) {
                const int r = qy - wy - py0;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float4 tg[JH][3];
                    float g2[JH];
                    if (!clamps) {
                        // no window of the tile's pixels leaves the image: the target of
                        // q is q moved as the pixel's centre, one add per gather
#pragma unroll
                        for (int jj = 0; jj < JH; ++jj) {  // wx = kWin0 + j
                            const uint4 d = s_d[r][qx - (kWin0 + h * JH + jj) - px0];
                            tg[jj][0] = M[0].ld(uq + d.x, sub);
                            tg[jj][1] = M[1].ld(uq + d.y, sub);
                            tg[jj][2] = M[2].ld(uq + d.z, sub);
                            g2[jj] = __uint_as_float(d.w);
                        }
                    } else {
#pragma unroll
                        for (int jj = 0; jj < JH; ++jj) {
                            const int wx = kWin0 + h * JH + jj, c = qx - wx - px0;
                            g2[jj] = s_g[r][c];
#pragma unroll
                            for (int k = 0; k < 3; ++k) {
                                const uint32_t t = s_t[k][r][c];
                                tg[jj][k] = M[k].ld(Map::template unit<L>(clampi((int)(t >> 16) + wy, 0, H - 1) * W +
                                                                          clampi((int)(t & 0xFFFFu) + wx, 0, W - 1)), sub);
                            }
                        }
                    }
#pragma unroll
                    for (int jj = 0; jj < JH; ++jj)
#pragma unroll
                        for (int k = 0; k < 3; ++k) fma4(g2[jj], fq, tg[jj][k], acc);
                }
            }
        } else if (live) {
            for (int wy = wy0; wy < wy0 + kPartRows; ++wy) {
                int ylo, yhi;
                preimage(qy, wy, H, ylo, yhi);
                for (int py = ylo; py <= yhi; ++py)
                    for (int wx = kWin0; wx <= kWin1; ++wx) {
                        int xlo, xhi;
                        preimage(qx, wx, W, xlo, xhi);
                        for (int px = xlo; px <= xhi; ++px) {
                            const int r = py - py0, c = px - px0;
                            const float g2 = s_g[r][c];
#pragma unroll
                            for (int k = 0; k < 3; ++k) {
                                const uint32_t t = s_t[k][r][c];
                                const int ty = (int)(t >> 16), tx = (int)(t & 0xFFFFu);
                                const float4 tg = M[k].ld(Map::template unit<L>(clampi(ty + wy, 0, H - 1) * W + clampi(tx + wx, 0, W - 1)), sub);
                                fma4(g2, fq, tg, acc);
                            }
                        }
                    }
            }
        }
        const float4 sum = sum_parts<kSplit, L>(acc);
        if (live && part == 0)
            reinterpret_cast<float4*>(a.out + ((size_t)b * 4 * HW + (size_t)mR * HW + q) * CF)[sub] = sum;
    }
}

// Target-map gradients (all three maps in one launch): the tile stages the
// pixels grouped at the centre cells its entries' windows reach (8 rows of
// kTileC cells; position, 2 g and cell column of each, and the run bounds of
// every cell).  A tile whose cells hold more than kStageCap pixels reads them
// from the sorted lists in global memory instead, in the same order.  The
// row_split(CF) groups of CF / 4 lanes of an entry are its accumulators (terms
// dealt round-robin, as in grad_target_kernel).
template <int CF, bool BUF>
__global__ void __launch_bounds__(256) grad_target_tile_kernel(CostArgs a, int tiles_x, size_t n,
                                                               const uint32_t* __restrict__ start,
                                                               const uint32_t* __restrict__ skeys,
                                                               const uint32_t* __restrict__ svals) {
    constexpr int kSplit = row_split(CF);
    constexpr int L = CF / 4, G = kSplit * L, EPB = 256 / G;
    static_assert(G <= 64 && 64 % G == 0, "the parts of an entry share one wave");
    __shared__ uint32_t s_st[kWinN][kTileC + 1];  // staged run start of each cell, and the row's end
    __shared__ uint32_t s_row[kWinN + 1];         // staged offset of each row's run
    __shared__ uint32_t s_gb[kWinN];              // sorted position of each row's run
    __shared__ uint32_t s_pos[kStageCap];         // (py << 16) | px
    __shared__ float s_g[kStageCap];
    __shared__ uint8_t s_cx[kStageCap];           // cell column - tx_lo
    __shared__ float4 s_fq[kTileQ * L];           // the entries' own vectors
    __shared__ uint2 s_term[4][64];               // terms of a wave's block: unit of the gathered vector, -2 g
    // runs of a border entry: first term, staged (or sorted) position, window offset
    __shared__ uint32_t s_rt[4][kMaxRuns], s_re[4][kMaxRuns];
    __shared__ uint16_t s_rw[4][kMaxRuns];
    const int H = a.H, W = a.W;
    const size_t HW = (size_t)H * W;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int tq = tile % tiles_x, rest = tile / tiles_x;
    const int qy = rest % H, kb = rest / H;
    const int b = kb % a.batch, k = kb / a.batch;
    const int qx0 = tq * kTileQ;
    const int ty0 = qy - kWin1;                                    // staged row 0
    const int tx_lo = max(qx0 - kWin1, 0), tx_hi = min(qx0 + kTileQ - 1 - kWin0, W - 1);
    const int ncol = tx_hi - tx_lo + 1;
    const size_t cbase = (size_t)k * n + (size_t)b * HW;          // cell (0, 0) of map k, image b
    if (threadIdx.x < kWinN) {
        const int r = threadIdx.x, ty = ty0 + r;
        uint32_t g0 = 0, len = 0;
        if (ty >= 0 && ty < H) {
            const size_t c0 = cbase + (size_t)ty * W + tx_lo;
            g0 = start[c0];
            len = start[c0 + ncol] - g0;
        }
        s_gb[r] = g0;
        s_row[r + 1] = len;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        s_row[0] = 0;
        for (int r = 0; r < kWinN; ++r) s_row[r + 1] += s_row[r];
    }
    __syncthreads();
    const uint32_t total = s_row[kWinN];
    const bool staged = total <= (uint32_t)kStageCap;
    if (staged) {
        for (int idx = threadIdx.x; idx < kWinN * (kTileC + 1); idx += 256) {
            const int r = idx / (kTileC + 1), j = idx - r * (kTileC + 1), ty = ty0 + r;
            if (j > ncol) continue;
            uint32_t v = s_row[r];
            if (ty >= 0 && ty < H) v += start[cbase + (size_t)ty * W + tx_lo + j] - s_gb[r];
            s_st[r][j] = v;
        }
        for (uint32_t e = threadIdx.x; e < total; e += 256) {
            int r = 0;
#pragma unroll
            for (int rr = 1; rr < kWinN; ++rr) r += e >= s_row[rr] ? 1 : 0;
            const uint32_t ge = s_gb[r] + (e - s_row[r]);
            const uint32_t pix = svals[ge];
            const int cc = (int)((size_t)skeys[ge] - cbase - (size_t)(ty0 + r) * W);
            const int pl = (int)(pix - (size_t)b * HW);
            const int py = pl / W, px = pl - py * W;
            s_pos[e] = ((uint32_t)py << 16) | (uint32_t)px;
            s_g[e] = 2.f * a.gcost[pix];
            s_cx[e] = (uint8_t)(cc - tx_lo);
        }
    }
    const float* base = a.feat + (size_t)b * 4 * HW * CF;
    for (int idx = threadIdx.x; idx < kTileQ * L; idx += 256) {
        const int qx = qx0 + idx / L;
        if (qx < W)
            s_fq[idx] = reinterpret_cast<const float4*>(
                base + ((size_t)view(a.s, k + 1) * HW + (size_t)qy * W + qx) * CF)[idx % L];
    }
    __syncthreads();
    using Map = Vec4Map<BUF>;
    Map R;
    R.init(base + (size_t)view(a.s, 0) * HW * CF, HW * CF * 4);
    const int mk = view(a.s, k + 1);
    const int sub = threadIdx.x % L, part = (threadIdx.x / L) % kSplit;  // part = accumulator
    const int lane = threadIdx.x & 63, wv = wave_id();
    uint2* term = s_term[wv];
    // term at staged (or sorted) position e, gathered at window offset (wy, wx) of its pixel
    auto term_at = [&](uint32_t e, int wy, int wx) {
        int py, px;
        float g2;
        if (staged) {
            const uint32_t pos = s_pos[e];
            py = (int)(pos >> 16);
            px = (int)(pos & 0xFFFFu);
            g2 = s_g[e];
        } else {
            const uint32_t pix = svals[e];
            const int pl = (int)(pix - (size_t)b * HW);
            py = pl / W;
            px = pl - py * W;
            g2 = 2.f * a.gcost[pix];
        }
        return make_uint2(Map::template unit<L>(clampi(py + wy, 0, H - 1) * W + clampi(px + wx, 0, W - 1)),
                          __float_as_uint(-g2));
    };
    // N terms of this lane's accumulator from the table at `tab`, which holds the terms
    // from i0 on: part, part + kSplit, ..., all loads in flight together.  The entry has m
    // terms in all; table places past them are left out.
    auto add_terms = [&](auto count, const uint2* tab, uint32_t i0, uint32_t m, const float4& fq, float4& acc) {
        constexpr int N = decltype(count)::value;
        uint2 tt[N];
        float4 rv[N];
#pragma unroll
        for (int u = 0; u < N; ++u) tt[u] = tab[u * kSplit + part];
#pragma unroll
        for (int u = 0; u < N; ++u) rv[u] = R.ld(tt[u].x, sub);
        if (__all(i0 + (uint32_t)(N * kSplit) <= m)) {
#pragma unroll
            for (int u = 0; u < N; ++u) fma4(__uint_as_float(tt[u].y), rv[u], fq, acc);
        } else {
#pragma unroll
            for (int u = 0; u < N; ++u)
                if (i0 + (uint32_t)(u * kSplit + part) < m) fma4(__uint_as_float(tt[u].y), rv[u], fq, acc);
        }
    };
    // A block of B terms: as many rounds as the longest of the wave's entries needs.
    auto add_block = [&](auto block, const uint2* tab, uint32_t i0, uint32_t m, uint32_t mmax, const float4& fq,
                         float4& acc) {
        constexpr int U = decltype(block)::value / kSplit;
        const uint32_t left = mmax - i0;
        if (U >= 4 && left <= (uint32_t)(U / 4 * kSplit))
            add_terms(std::integral_constant<int, (U >= 4 ? U / 4 : 1)>{}, tab, i0, m, fq, acc);
        else if (U >= 2 && left <= (uint32_t)(U / 2 * kSplit))
            add_terms(std::integral_constant<int, (U >= 2 ? U / 2 : 1)>{}, tab, i0, m, fq, acc);
        else
            add_terms(std::integral_constant<int, U>{}, tab, i0, m, fq, acc);
    };
    for (int e0 = 0; e0 < kTileQ; e0 += EPB) {
        const int qx = qx0 + e0 + (int)threadIdx.x / G;
        const bool live = qx < W;
        const size_t q = (size_t)qy * W + qx;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 fq = make_float4(0.f, 0.f, 0.f, 0.f);
        if (live) fq = s_fq[(qx - qx0) * L + sub];
        const bool interior = qy >= kWin1 && qy <= H - 1 + kWin0 && qx >= kWin1 && qx <= W - 1 + kWin0;
        const int lg = (int)threadIdx.x % G, gbase = lane - lg;
        bool any = true;  // (wave-uniform) some entry of the wave has terms
        // the whole wave takes the interior path or none of it does; a tile too crowded to
        // stage reads the same terms from the sorted lists in global memory
        if (__all(!live || interior)) {
            // the terms are the runs of the window rows wy = -3 .. 4 (cells (qy - wy, qx - 4 ..
            // qx + 3)), one after the other, in blocks of G: lane lg of the entry's G lanes
            // finds term i0 + lg (row, staged pixel, gathered vector, 2 g) once and leaves it
            // in LDS, where the lanes of accumulator `part` take terms part, part + kSplit, ...
            const int j0 = qx - kWin1 - tx_lo;
            uint32_t rb[kWinN], rend[kWinN];
            uint32_t m = 0;
#pragma unroll
            for (int t = 0; t < kWinN; ++t) {
                const int r = qy - (kWin0 + t) - ty0;
                uint32_t b0 = 0, b1 = 0;
                if (live && staged) {
                    b0 = s_st[r][j0];
                    b1 = s_st[r][j0 + kWinN];
                } else if (live) {
                    const size_t c0 = cbase + (size_t)(ty0 + r) * W + (qx - kWin1);
                    b0 = start[c0];
                    b1 = start[c0 + kWinN];
                }
                rb[t] = b0 - m;  // staged (or sorted) index of term i of this row: rb[t] + i
                m += b1 - b0;
                rend[t] = m;
            }
            const uint32_t mmax = G == 64 ? (uint32_t)__builtin_amdgcn_readfirstlane(m) : (uint32_t)__reduce_max_sync(~0ull, m);
            any = mmax > 0;
            for (uint32_t i0 = 0; i0 < mmax; i0 += G) {
                const uint32_t it = i0 + (uint32_t)lg;
                uint2 tm = make_uint2(0u, 0u);
                if (it < m) {
                    int t = 0;
                    uint32_t e = rb[0];
#pragma unroll
                    for (int tt = 0; tt < kWinN - 1; ++tt) {
                        const bool past = it >= rend[tt];
                        t += past ? 1 : 0;
                        e = past ? rb[tt + 1] : e;
                    }
                    e += it;
                    const int wy = kWin0 + t;
                    const int wx = staged ? qx - tx_lo - (int)s_cx[e]
                                          : qx - (int)((size_t)skeys[e] - cbase - (size_t)(qy - wy) * W);
                    tm = term_at(e, wy, wx);
                }
                term[lane] = tm;
                grad_wave_sync();
                add_block(std::integral_constant<int, G>{}, term + gbase, i0, m, mmax, fq, acc);
                grad_wave_sync();
            }
        } else {
            // entries at the border have more cells in their preimage: the wave lists the
            // runs of its entries one entry after the other (window row, cell row, window
            // column descending, cell column) and deals their terms the same way
#pragma unroll 1
            for (int en = 0; en < 64 / G; ++en) {
                const int ex = __shfl(qx, en * G);
                if (ex >= W) break;  // wave-uniform
                int nr = 0, nc = 0;
                for (int w = kWin0; w <= kWin1; ++w) {
                    int lo, hi;
                    preimage(qy, w, H, lo, hi);
                    nr += max(hi - lo + 1, 0);
                    preimage(ex, w, W, lo, hi);
                    nc += max(hi - lo + 1, 0);
                }
                const int nrun = nr * nc;
                uint32_t m = 0;
                for (int s0 = 0; s0 < nrun; s0 += 64) {
                    const int sg = s0 + lane;
                    uint32_t len = 0, pos = 0;
                    int wy = kWin0, wx = kWin1, ty = 0, tx = 0;
                    if (sg < nrun) {
                        int ri = sg / nc, ci = sg - ri * nc;
                        for (; wy <= kWin1; ++wy) {
                            int lo, hi;
                            preimage(qy, wy, H, lo, hi);
                            const int cnt = max(hi - lo + 1, 0);
                            if (ri < cnt) {
                                ty = lo + ri;
                                break;
                            }
                            ri -= cnt;
                        }
                        for (; wx >= kWin0; --wx) {
                            int lo, hi;
                            preimage(ex, wx, W, lo, hi);
                            const int cnt = max(hi - lo + 1, 0);
                            if (ci < cnt) {
                                tx = lo + ci;
                                break;
                            }
                            ci -= cnt;
                        }
                        uint32_t p1;
                        if (staged) {
                            pos = s_st[ty - ty0][tx - tx_lo];
                            p1 = s_st[ty - ty0][tx - tx_lo + 1];
                        } else {
                            const size_t cell = cbase + (size_t)ty * W + tx;
                            pos = start[cell];
                            p1 = start[cell + 1];
                        }
                        len = p1 - pos;
                    }
                    uint32_t incl = len;  // inclusive sum over the lanes
#pragma unroll
                    for (int d = 1; d < 64; d *= 2) {
                        const uint32_t o = (uint32_t)__shfl_up((int)incl, d);
                        if (lane >= d) incl += o;
                    }
                    if (sg < nrun) {
                        s_rt[wv][sg] = m + incl - len;
                        s_re[wv][sg] = pos;
                        s_rw[wv][sg] = (uint16_t)((wy - kWin0) * kWinN + (wx - kWin0));
                    }
                    m += (uint32_t)__shfl((int)incl, 63);
                }
                grad_wave_sync();
                const bool mine = (int)threadIdx.x / G % (64 / G) == en;
                for (uint32_t i0 = 0; i0 < m; i0 += 64) {
                    const uint32_t it = i0 + (uint32_t)lane;
                    uint2 tm = make_uint2(0u, 0u);
                    if (it < m) {
                        int lo = 0, hi = nrun;  // the last run that starts at or before the term
                        while (hi - lo > 1) {
                            const int mid = (lo + hi) >> 1;
                            if (s_rt[wv][mid] <= it) lo = mid;
                            else hi = mid;
                        }
                        const int wo = s_rw[wv][lo];
                        tm = term_at(s_re[wv][lo] + (it - s_rt[wv][lo]), kWin0 + wo / kWinN, kWin0 + wo % kWinN);
                    }
                    term[lane] = tm;
                    grad_wave_sync();
                    if (mine) add_block(std::integral_constant<int, 64>{}, term, i0, m, m, fq, acc);
                    grad_wave_sync();
                }
            }
        }
        const float4 sum = any ? sum_parts<kSplit, L>(acc) : acc;
        if (live && part == 0)
            reinterpret_cast<float4*>(a.out + ((size_t)b * 4 * HW + (size_t)mk * HW + q) * CF)[sub] = sum;
    }
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Workspace of the backward: the key/value lists (two buffers each for the
// sort passes), the cell starts and the per-block digit counts.
struct BwdWs {
    size_t N, nblk, keys_a, vals_a, keys_b, vals_b, start, hist, sums, total;
};

BwdWs bwd_ws(size_t n) {
    BwdWs L;
    L.N = 3 * n;
    L.nblk = (L.N + kSortTile - 1) / kSortTile;
    L.keys_a = 0;
    L.vals_a = L.keys_a + align256(L.N * 4);
    L.keys_b = L.vals_a + align256(L.N * 4);
    L.vals_b = L.keys_b + align256(L.N * 4);
    L.start = L.vals_b + align256(L.N * 4);
    L.hist = L.start + align256((L.N + 1) * 4);
    L.sums = L.hist + align256(256 * L.nblk * 4);
    L.total = L.sums + align256((256 * L.nblk + 1023) / 1024 * 4);
    return L;
}

// Largest batch * H * W the backward takes: its lists hold 3 entries per pixel
// with 32-bit positions.
constexpr size_t kBwdMaxPixels = (size_t)1 << 30;

bool shape_ok(int batch, int H, int W, int cf, int dir) {
    if (batch < 1 || H < 1 || W < 1 || H > 16384 || W > 16384) return false;
    if ((size_t)batch * H * W >= (1ull << 31)) return false;
    if (cf != 4 && cf != 8 && cf != 16 && cf != 32 && cf != 64) return false;
    return dir == 1 || dir == -1;
}

template <template <int> class K, typename... Args>
void launch_cf(int cf, dim3 g, hipStream_t st, Args... args) {
    switch (cf) {
        case 4: hipLaunchKernelGGL(K<4>::fn, g, dim3(256), 0, st, args...); break;
        case 8: hipLaunchKernelGGL(K<8>::fn, g, dim3(256), 0, st, args...); break;
        case 16: hipLaunchKernelGGL(K<16>::fn, g, dim3(256), 0, st, args...); break;
        case 32: hipLaunchKernelGGL(K<32>::fn, g, dim3(256), 0, st, args...); break;
        default: hipLaunchKernelGGL(K<64>::fn, g, dim3(256), 0, st, args...); break;
    }
}

template <int CF>
struct FwdK {
    static constexpr auto fn = cost_fwd_kernel<CF>;
};

template <int CF>
struct FwdCoopK {
    static constexpr auto fn = cost_fwd_coop_kernel<CF>;
};
template <int CF>
struct RefK {
    static constexpr auto fn = grad_ref_kernel<CF>;
};
template <int CF>
struct TgtK {
    static constexpr auto fn = grad_target_kernel<CF>;
};

template <int CF>
struct RefTileK {
    static constexpr auto fn = grad_ref_tile_kernel<CF, true>;
};

template <int CF>
struct TgtTileK {
    static constexpr auto fn = grad_target_tile_kernel<CF, true>;
};

template <int CF>
struct RefTileWideK {
    static constexpr auto fn = grad_ref_tile_kernel<CF, false>;
};

template <int CF>
struct TgtTileWideK {
    static constexpr auto fn = grad_target_tile_kernel<CF, false>;
};

}  // namespace
}  // namespace sff

using namespace sff;

extern "C" sff_status sff_cost_f32_fwd(int32_t batch, int32_t H, int32_t W, int32_t cf, int32_t dir,
                                       const float* feat, const int16_t* hyp, float* cost_px,
                                       void* stream) {
    if (!shape_ok(batch, H, W, cf, dir) || !feat || !hyp || !cost_px) return SFF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(feat) & 15) != 0 || (reinterpret_cast<uintptr_t>(hyp) & 7) != 0 ||
        (reinterpret_cast<uintptr_t>(cost_px) & 3) != 0)
        return SFF_ERR_INVALID_ARG;
    CostArgs a{feat, hyp, nullptr, cost_px, H, W, dir, batch};
    // SFF_COST_F32_EVAL=lane: one lane per pixel (testing and timing)
    const char* ev = std::getenv("SFF_COST_F32_EVAL");
    if (ev && std::strcmp(ev, "lane") == 0)
        launch_cf<FwdK>(cf, dim3((W + 63) / 64, (H + 3) / 4, batch), as_stream(stream), a);
    else
        launch_cf<FwdCoopK>(cf, dim3((unsigned)(((size_t)H * W * (cf / 4) + 255) / 256), batch), as_stream(stream),
                            a);
    return launch_status();
}

extern "C" size_t sff_cost_f32_bwd_workspace_bytes(int32_t batch, int32_t H, int32_t W) {
    if (batch < 1 || H < 1 || W < 1 || (size_t)batch * H * W > kBwdMaxPixels) return 0;
    return bwd_ws((size_t)batch * H * W).total;
}

extern "C" sff_status sff_cost_f32_bwd(int32_t batch, int32_t H, int32_t W, int32_t cf,
                                       int32_t dir, const float* feat, const int16_t* hyp,
                                       const float* grad_cost, float* grad_feat, void* workspace,
                                       size_t workspace_bytes, void* stream) {
    if (!shape_ok(batch, H, W, cf, dir) || !feat || !hyp || !grad_cost || !grad_feat)
        return SFF_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(feat) & 15) != 0 || (reinterpret_cast<uintptr_t>(hyp) & 7) != 0 ||
        (reinterpret_cast<uintptr_t>(grad_cost) & 3) != 0 ||
        (reinterpret_cast<uintptr_t>(grad_feat) & 15) != 0)
        return SFF_ERR_INVALID_ARG;
    const size_t n = (size_t)batch * H * W;
    if (n > kBwdMaxPixels) return SFF_ERR_UNSUPPORTED;
    const BwdWs L = bwd_ws(n);
    if (!workspace || workspace_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0)
        return SFF_ERR_WORKSPACE;
    hipStream_t st = as_stream(stream);
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    uint32_t* ka = reinterpret_cast<uint32_t*>(ws + L.keys_a);
    uint32_t* va = reinterpret_cast<uint32_t*>(ws + L.vals_a);
    uint32_t* kb = reinterpret_cast<uint32_t*>(ws + L.keys_b);
    uint32_t* vb = reinterpret_cast<uint32_t*>(ws + L.vals_b);
    uint32_t* start = reinterpret_cast<uint32_t*>(ws + L.start);
    uint32_t* hist = reinterpret_cast<uint32_t*>(ws + L.hist);
    uint32_t* sums = reinterpret_cast<uint32_t*>(ws + L.sums);
    const size_t nhist = 256 * L.nblk, nchunks = (nhist + 1023) / 1024;
    CostArgs a{feat, hyp, grad_cost, grad_feat, H, W, dir, batch};
    // SFF_COST_F32_EVAL=lane: one lane per gradient entry (same results; testing and timing)
    const char* ev = std::getenv("SFF_COST_F32_EVAL");
    const bool lane_grad = ev && std::strcmp(ev, "lane") == 0;
    const int tiles_x = (W + kTileQ - 1) / kTileQ;
    const dim3 grid((W + 63) / 64, (H + 3) / 4, batch);
    // maps below 2 GiB are read through 32-bit buffer offsets
    const bool buf = (size_t)H * W * cf * 4 <= (size_t)kSkipOff;
    // The reference-map gradient and the target-map gradients (with the
    // grouping they need) read the same inputs and write different maps, so
    // the reference gradient runs on a helper stream of the library beside them
    // (SFF_COST_F32_SPLIT=0: one stream; identical results either way).
    const char* sp = std::getenv("SFF_COST_F32_SPLIT");
    std::optional<HelperUse> helper;
    if (!(sp && std::strcmp(sp, "0") == 0)) helper.emplace(st);
    const bool split = helper && helper->stream();
    hipStream_t sr = split ? helper->stream() : st;
    if (lane_grad)
        launch_cf<RefK>(cf, grid, sr, a);
    else if (buf)
        launch_cf<RefTileK>(cf, dim3((unsigned)((size_t)batch * H * tiles_x)), sr, a, tiles_x);
    else
        launch_cf<RefTileWideK>(cf, dim3((unsigned)((size_t)batch * H * tiles_x)), sr, a, tiles_x);
    // group the pixels by target centre: keys, then a stable radix sort
    const size_t N = L.N;
    hipLaunchKernelGGL(target_keys_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, hyp,
                       ka, va, H, W, dir, (uint32_t)n);
    int bits = 1;
    while (bits < 32 && (1ull << bits) < N) ++bits;
    uint32_t *kin = ka, *vin = va, *kout = kb, *vout = vb;
    for (int sh = 0; sh < bits; sh += 8) {
        hipLaunchKernelGGL(sort_hist_kernel, dim3((unsigned)L.nblk), dim3(256), 0, st,
                           (const uint32_t*)kin, N, sh, hist, (uint32_t)L.nblk);
        hipLaunchKernelGGL(sort_scan_chunks_kernel, dim3((unsigned)nchunks), dim3(1024), 0, st, hist,
                           nhist, sums);
        hipLaunchKernelGGL(sort_scan_sums_kernel, dim3(1), dim3(1024), 0, st, sums, nchunks);
        hipLaunchKernelGGL(sort_scatter_kernel, dim3((unsigned)L.nblk), dim3(256), 0, st,
                           (const uint32_t*)kin, (const uint32_t*)vin, kout, vout, N, sh,
                           (const uint32_t*)hist, (const uint32_t*)sums, (uint32_t)L.nblk);
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
    hipLaunchKernelGGL(cell_starts_kernel, dim3((unsigned)((N + 1 + 255) / 256)), dim3(256), 0, st,
                       (const uint32_t*)kin, start, N);
    if (lane_grad) {
        for (int k = 0; k < 3; ++k)
            launch_cf<TgtK>(cf, grid, st, a, k, n, (const uint32_t*)start, (const uint32_t*)vin);
    } else if (buf) {
        launch_cf<TgtTileK>(cf, dim3((unsigned)((size_t)3 * batch * H * tiles_x)), st, a, tiles_x, n,
                            (const uint32_t*)start, (const uint32_t*)kin, (const uint32_t*)vin);
    } else {
        launch_cf<TgtTileWideK>(cf, dim3((unsigned)((size_t)3 * batch * H * tiles_x)), st, a, tiles_x, n,
                                (const uint32_t*)start, (const uint32_t*)kin, (const uint32_t*)vin);
    }
    const sff_status r = launch_status();
    if (split && !helper->join()) return SFF_ERR_HIP;
    return r;
}
