// HIP kernels of the TLSPH damage step for gfx950 (MI355X).
//
// Data layout (all per-particle arrays in Hilbert order of their cells,
// stride np, a multiple of 64): field component c of particle i at
// [c * np + i].  The neighbour list is "sliced": the 64 particles of slice
// s = i / 64 keep their k-th neighbour at col[slice_ptr[s] + 64 k + (i % 64)],
// so the 64 lanes of a wavefront read 64 consecutive indices per neighbour
// step.  One lane owns one particle and sums its neighbours in a fixed order:
// no floating-point atomics anywhere, results independent of the launch
// shape.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "tlsph_internal.h"
#include "tlsph_math.h"
#include "tlsph_passes.h"

namespace tlsph {

// ===========================================================================
// neighbour-list build (Sec. 2: S_i fixed in the reference configuration)
// ===========================================================================

// Position of cell (x, y, z) along a three-dimensional Hilbert curve over
// 2^kCellBits cells per axis: the coordinates are turned into the curve's
// index in transposed form (Skilling's method: undo the excess rotations and
// reflections from the top bit down, then Gray-decode), whose bits are then
// interleaved, highest level first.  Consecutive keys are face-adjacent
// cells, so a run of keys (a tile) is a compact region; a run of Morton keys
// may jump across the domain, which puts more of a tile's neighbours outside
// it.
__device__ __forceinline__ uint64_t cell_key(uint32_t x, uint32_t y, uint32_t z) {
    uint32_t X[3] = {x, y, z};
    for (uint32_t Q = 1u << (kCellBits - 1); Q > 1; Q >>= 1) {
        const uint32_t P = Q - 1;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (X[i] & Q) {
                X[0] ^= P;
            } else {
                const uint32_t t = (X[0] ^ X[i]) & P;
                X[0] ^= t;
                X[i] ^= t;
            }
        }
    }
    X[1] ^= X[0];
    X[2] ^= X[1];
    uint32_t t = 0;
    for (uint32_t Q = 1u << (kCellBits - 1); Q > 1; Q >>= 1)
        if (X[2] & Q) t ^= Q - 1;
    uint64_t key = 0;
    for (int b = kCellBits - 1; b >= 0; --b)
#pragma unroll
        for (int i = 0; i < 3; ++i) key = (key << 1) | (((X[i] ^ t) >> b) & 1u);
    return key;
}

// Per-specimen record of 8 doubles (caller order, particles contiguous per
// specimen): bounding box lo[3], hi[3], then 1 / cell edge.  The edge is the
// specimen's h, or with graded spacing the largest support h_per_spacing
// (max V0)^(1/3), each a hair larger so that pairs closer than the support
// never sit two cells apart after rounding.
// Found by all compute units: each specimen's chunks (those of the diagnostics,
// at most kBBoxParts workgroups of them) reduce in LDS and meet in atomics on the
// extrema as ordered integers, kept in the record itself.  One workgroup per
// specimen took 281 us for 200k particles, this 11; with a grid row per specimen
// and columns for the chunks of them all, nearly all empty, 70000 specimens of
// eight took 33 ms to build, so 1.1.
constexpr int kBBox = 8;
constexpr int kBBoxParts = 256;
__device__ __forceinline__ unsigned long long ordered_bits(double x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    return b ^ ((b >> 63) ? ~0ull : 1ull << 63);
}
__device__ __forceinline__ double from_ordered_bits(unsigned long long b) {
    return __longlong_as_double((long long)(b ^ ((b >> 63) ? 1ull << 63 : ~0ull)));
}
__global__ void k_bbox_clear(unsigned long long* __restrict__ bits, int n_spec) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = t % kBBox;
    if (t < n_spec * kBBox) bits[t] = ordered_bits(c < 3 ? 1e300 : c < 6 ? -1e300 : 0.0);
}
__global__ void __launch_bounds__(256) k_bbox(const double* __restrict__ X,
                                              const double* __restrict__ V0, int64_t n,
                                              const int64_t* __restrict__ off,
                                              const int64_t* __restrict__ seg, int n_spec,
                                              unsigned long long* __restrict__ bits) {
    __shared__ double red[7][256];
    // the specimen of chunk b: every one has a chunk, so it lies within the
    // chunks beyond one each below b
    const int64_t b = blockIdx.x, more = seg[n_spec] - n_spec;
    int64_t s = b > more ? b - more : 0, top = b < n_spec ? b : n_spec - 1;
    while (s < top) {
        const int64_t mid = (s + top + 1) >> 1;
        if (seg[mid] <= b) s = mid; else top = mid - 1;
    }
    const int64_t all = seg[s + 1] - seg[s], parts = all < kBBoxParts ? all : kBBoxParts;
    if (b - seg[s] >= parts) return;
    const int64_t last = off[s + 1], beg = off[s] + (b - seg[s]) * 256;
    const int64_t m = last - beg;   // (lanes past the specimen's end hold nothing)
    double lo[3] = {1e300, 1e300, 1e300}, hi[3] = {-1e300, -1e300, -1e300}, vmax = 0.0;
    for (int64_t i = beg + threadIdx.x; i < last; i += parts * 256) {
        for (int c = 0; c < 3; ++c) {
            const double x = X[c * n + i];
            lo[c] = x < lo[c] ? x : lo[c];
            hi[c] = x > hi[c] ? x : hi[c];
        }
        vmax = V0[i] > vmax ? V0[i] : vmax;
    }
    for (int c = 0; c < 3; ++c) {
        red[c][threadIdx.x] = lo[c];
        red[3 + c][threadIdx.x] = hi[c];
    }
    red[6][threadIdx.x] = vmax;
    __syncthreads();
    int w = 128;
    while (w >= m && w > 0) w >>= 1;
    for (; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            for (int c = 0; c < 3; ++c) {
                red[c][threadIdx.x] = fmin(red[c][threadIdx.x], red[c][threadIdx.x + w]);
                red[3 + c][threadIdx.x] = fmax(red[3 + c][threadIdx.x], red[3 + c][threadIdx.x + w]);
            }
            red[6][threadIdx.x] = fmax(red[6][threadIdx.x], red[6][threadIdx.x + w]);
        }
        __syncthreads();
    }
    const int t = threadIdx.x;
    if (t < 3) atomicMin(&bits[kBBox * s + t], ordered_bits(red[t][0]));
    else if (t < 7) atomicMax(&bits[kBBox * s + t], ordered_bits(red[t][0]));
}
__global__ void k_bbox_final(double* __restrict__ bbox, int n_spec,
                             const DevSpec* __restrict__ specs) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_spec) return;
    double* b = bbox + kBBox * s;
    double v[7];
    for (int c = 0; c < 7; ++c)
        v[c] = from_ordered_bits((unsigned long long)__double_as_longlong(b[c]));
    for (int c = 0; c < 6; ++c) b[c] = v[c];
    const DevSpec& P = specs[s];
    b[6] = P.h_per_spacing > 0.0 ? 1.0 / (P.h_per_spacing * cbrt(v[6]) * (1.0 + 1e-9))
                                 : P.inv_cell;
    b[7] = 0.0;
}

__device__ __forceinline__ int spec_of(const int64_t* off, int n_spec, int64_t i) {
    int lo = 0, hi = n_spec;  // largest s with off[s] <= i
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ void cell_of(const double* bb, double x, double y, double z,
                                        int32_t c[3]) {
    const double xs[3] = {x, y, z};
    for (int a = 0; a < 3; ++a) {
        const double q = floor((xs[a] - bb[a]) * bb[6]);
        c[a] = q < 0.0 ? 0 : (int32_t)q;
    }
}

__global__ void k_keys(const double* __restrict__ X, int64_t n, int64_t n_pow2,
                       const int64_t* __restrict__ off, int n_spec,
                       const double* __restrict__ bbox, uint64_t* __restrict__ keys,
                       int32_t* __restrict__ vals, int32_t* __restrict__ err) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_pow2) return;
    if (i >= n) {
        keys[i] = ~0ull;
        vals[i] = 0x7fffffff;
        return;
    }
    const int s = spec_of(off, n_spec, i);
    int32_t c[3];
    cell_of(bbox + kBBox * s, X[i], X[n + i], X[2 * n + i], c);
    if (c[0] >= (1 << kCellBits) || c[1] >= (1 << kCellBits) || c[2] >= (1 << kCellBits))
        atomicOr(&err[3], 1);
    keys[i] = ((uint64_t)s << kSpecShift) | cell_key(c[0], c[1], c[2]);
    vals[i] = (int32_t)i;
}

// Compare-exchange of (key, val) pairs of a bitonic sort, in registers.
__device__ __forceinline__ void sort_pair(uint64_t& ka, int32_t& va, uint64_t& kb, int32_t& vb,
                                          bool asc) {
    const bool a_gt_b = (ka > kb) || (ka == kb && va > vb);
    if (a_gt_b == asc) {
        const uint64_t k = ka; ka = kb; kb = k;
        const int32_t v = va; va = vb; vb = v;
    }
}
// One stage (kTwo: the stages j and j / 2, which four elements share, in one
// pass over memory) of the sort: a thread per group of 2 (4) elements.
template <bool kTwo>
__global__ void k_bitonic(uint64_t* __restrict__ keys, int32_t* __restrict__ vals, int64_t N,
                          int64_t j, int64_t k) {
    constexpr int M = kTwo ? 4 : 2;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= N / M) return;
    const int64_t d = kTwo ? j >> 1 : j;   // distance of the group's elements
    const int64_t i = M * (t & ~(d - 1)) + (t & (d - 1));
    uint64_t ke[M];
    int32_t ve[M];
#pragma unroll
    for (int e = 0; e < M; ++e) {
        ke[e] = keys[i + e * d];
        ve[e] = vals[i + e * d];
    }
    const bool asc = (i & k) == 0;
    if constexpr (kTwo) {
        sort_pair(ke[0], ve[0], ke[2], ve[2], asc);
        sort_pair(ke[1], ve[1], ke[3], ve[3], asc);
        sort_pair(ke[0], ve[0], ke[1], ve[1], asc);
        sort_pair(ke[2], ve[2], ke[3], ve[3], asc);
    } else {
        sort_pair(ke[0], ve[0], ke[1], ve[1], asc);
    }
#pragma unroll
    for (int e = 0; e < M; ++e) {
        keys[i + e * d] = ke[e];
        vals[i + e * d] = ve[e];
    }
}

// The stages of the same sort whose partners lie within one block of kSortB
// elements (j < kSortB), run in LDS: with k <= kSortB every stage of the
// network from k = 2 (the block's own sort), else the stages j < kSortB of
// the merge of size k.  Blocks of kSortB / 2 threads, one pair per stage each;
// N (a power of two) below kSortB makes one block of N elements.
constexpr int kSortB = 2048;
__global__ void __launch_bounds__(kSortB / 2) k_bitonic_lds(uint64_t* __restrict__ keys,
                                                            int32_t* __restrict__ vals, int64_t N,
                                                            int64_t k_merge) {
    __shared__ uint64_t sk[kSortB];
    __shared__ int32_t sv[kSortB];
    const int B = (int)(N < kSortB ? N : kSortB);
    const int64_t base = (int64_t)blockIdx.x * B;
    for (int e = threadIdx.x; e < B; e += blockDim.x) {
        sk[e] = keys[base + e];
        sv[e] = vals[base + e];
    }
    __syncthreads();
    const int64_t k_lo = k_merge > 0 ? k_merge : 2;
    const int64_t k_hi = k_merge > 0 ? k_merge : B;
    for (int64_t k = k_lo; k <= k_hi; k <<= 1) {
        for (int64_t j = (k >> 1 < B ? k >> 1 : B >> 1); j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < B / 2; t += blockDim.x) {
                // the t-th pair (e, e + j) of the stage
                const int e = (int)(((t / j) * 2 * j) + (t % j));
                const int l = e + (int)j;
                const uint64_t ka = sk[e], kb = sk[l];
                const int32_t va = sv[e], vb = sv[l];
                const bool a_gt_b = (ka > kb) || (ka == kb && va > vb);
                const bool asc = ((base + e) & k) == 0;
                if (a_gt_b == asc) {
                    sk[e] = kb; sk[l] = ka;
                    sv[e] = vb; sv[l] = va;
                }
            }
            __syncthreads();
        }
    }
    for (int e = threadIdx.x; e < B; e += blockDim.x) {
        keys[base + e] = sk[e];
        vals[base + e] = sv[e];
    }
}

// Sort N (a power of two, >= 2) (key, val) pairs ascending by key, then val:
// the bitonic network, its stages with partners closer than kSortB run in
// LDS, the others two to a launch.
hipError_t launch_bitonic_sort(uint64_t* keys, int32_t* vals, int64_t N, hipStream_t st) {
    constexpr int T = 256;
    const int B = (int)(N < kSortB ? N : kSortB);
    const unsigned blocks = (unsigned)(N / B);
    k_bitonic_lds<<<blocks, B / 2, 0, st>>>(keys, vals, N, 0);
    for (int64_t k = 2 * (int64_t)B; k <= N; k <<= 1) {
        int64_t j = k >> 1;
        for (; j >= 2 * (int64_t)B; j >>= 2)
            k_bitonic<true><<<(unsigned)((N / 4 + T - 1) / T), T, 0, st>>>(keys, vals, N, j, k);
        if (j >= B)
            k_bitonic<false><<<(unsigned)((N / 2 + T - 1) / T), T, 0, st>>>(keys, vals, N, j, k);
        k_bitonic_lds<<<blocks, B / 2, 0, st>>>(keys, vals, N, k);
    }
    return hipGetLastError();
}

__global__ void k_apply_perm(DevState s, const double* __restrict__ X_in,
                             const double* __restrict__ V0_in, const int32_t* __restrict__ bc_in,
                             const uint64_t* __restrict__ keys, const int32_t* __restrict__ vals,
                             D4* __restrict__ XV, int32_t* __restrict__ specs_out,
                             int32_t* __restrict__ bcs, int32_t* __restrict__ perm,
                             int32_t* __restrict__ iperm) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= s.np) return;
    const int64_t n = s.n;
    if (p < n) {
        const int32_t o = vals[p];
        perm[p] = o;
        iperm[o] = (int32_t)p;
        XV[p] = D4{X_in[o], X_in[n + o], X_in[2 * n + o], V0_in[o]};
        int32_t g = bc_in[o];
        if (g < -1 || g >= s.n_bc) {  // reported as an argument error by the host
            atomicOr(&s.err[3], 2);
            g = -1;
        }
        bcs[p] = g;
        const int32_t sp = (int32_t)(keys[p] >> kSpecShift);
        specs_out[p] = sp;
        const DevSpec& P = s.specs[sp];
        s.hs[p] = P.h_per_spacing > 0.0 ? P.h_per_spacing * cbrt(V0_in[o]) : P.h;
        s.arad[p] = 0.5 * cbrt(V0_in[o]);
    } else {
        perm[p] = -1;
        s.hs[p] = 0.0;
        s.arad[p] = 0.0;
        XV[p] = D4{0.0, 0.0, 0.0, 0.0};
        bcs[p] = -1;
        specs_out[p] = 0;
    }
}

// sorted particle range of every specimen
__global__ void k_spec_ranges(DevSpec* specs, int n_spec, const uint64_t* __restrict__ keys,
                              int64_t n) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_spec) return;
    auto lower = [&](uint64_t key) {
        int64_t lo = 0, hi = n;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (keys[mid] < key) lo = mid + 1; else hi = mid;
        }
        return lo;
    };
    specs[s].first = lower((uint64_t)s << kSpecShift);
    specs[s].last = lower((uint64_t)(s + 1) << kSpecShift);
}

// The occupied cells as a hash table of their first sorted particle (open
// addressing; H, a power of two, at least twice the particles, so that a
// search always meets a free slot).
constexpr uint64_t kNoCell = ~0ull;
__global__ void k_cells_clear(CSlot* __restrict__ cell, int64_t H) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < H) cell[t].key = kNoCell;
}
__global__ void k_cells_insert(DevState s, const uint64_t* __restrict__ keys,
                               const double* __restrict__ bbox, CSlot* __restrict__ cell,
                               int64_t H, int shift) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= s.n || (p > 0 && keys[p - 1] == keys[p])) return;   // the first of its cell
    int64_t end = p + 1;
    while (end < s.n && keys[end] == keys[p]) ++end;
    const int sp = s.spec[p];
    const D4 x = s.XV[p];
    int32_t c[3];
    cell_of(bbox + kBBox * sp, x.x, x.y, x.z, c);
    const uint64_t key = grid_key(sp, c[0], c[1], c[2]);
    for (int64_t h = cell_home(key, shift);; h = (h + 1) & (H - 1))
        if (atomicCAS(reinterpret_cast<unsigned long long*>(&cell[h].key), kNoCell, key) == kNoCell) {
            cell[h].start = (int32_t)p;
            cell[h].cnt = (int32_t)(end - p);
            return;
        }
}

// Visit the neighbours of sorted particle p over the 27 cells around it, in
// a fixed order.  The distance test is evaluated exactly as written (no
// fused multiply-add) so membership is decided identically to a plain
// evaluation of |X_j - X_i|^2 < h^2.  What bounds the search is its chain of
// loads, so a layer's nine table slots are loaded together, and the particles
// of a cell four at a time.
template <typename F>
__device__ __forceinline__ int for_neighbours(const DevState& s, const double* bbox,
                                              const CSlot* cell, int64_t H, int shift, int64_t p,
                                              F&& visit) {
#pragma clang fp contract(off)
    const int sp = s.spec[p];
    const DevSpec& P = s.specs[sp];
    const D4 xp = s.XV[p];
    const double xi = xp.x, yi = xp.y, zi = xp.z;
    int32_t c[3];
    cell_of(bbox + kBBox * sp, xi, yi, zi, c);
    const double hp = s.hs[p];
    const double lim0 = P.h2;
    constexpr int kLayer = 9, kU = 4;
    constexpr uint32_t kCells = 1u << kCellBits;
    int count = 0;
    for (int dz = -1; dz <= 1; ++dz) {
        uint64_t key[kLayer];
        int64_t h[kLayer];
        CSlot slot[kLayer];
        bool in[kLayer];
#pragma unroll
        for (int e = 0; e < kLayer; ++e) {
            const int32_t cx = c[0] + e % 3 - 1, cy = c[1] + e / 3 - 1, cz = c[2] + dz;
            in[e] = (uint32_t)cx < kCells && (uint32_t)cy < kCells && (uint32_t)cz < kCells;
            key[e] = in[e] ? grid_key(sp, cx, cy, cz) : grid_key(sp, c[0], c[1], c[2]);
            h[e] = cell_home(key[e], shift);
            slot[e] = cell[h[e]];
        }
#pragma unroll
        for (int e = 0; e < kLayer; ++e) {
            while (slot[e].key != key[e] && slot[e].key != kNoCell) {
                h[e] = (h[e] + 1) & (H - 1);
                slot[e] = cell[h[e]];
            }
            const int m = in[e] && slot[e].key == key[e] ? slot[e].cnt : 0;
            for (int q0 = 0; q0 < m; q0 += kU) {
                D4 xq[kU];
                double hq[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int64_t q = slot[e].start + (q0 + u < m ? q0 + u : 0);
                    xq[u] = s.XV[q];
                    hq[u] = s.var_h ? s.hs[q] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int64_t q = slot[e].start + q0 + u;
                    const double d0 = xq[u].x - xi;
                    const double d1 = xq[u].y - yi;
                    const double d2 = xq[u].z - zi;
                    const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
                    double lim = lim0;
                    if (s.var_h) {   // graded spacing: the pair's support (h_p + h_q) / 2
                        const double hpq = 0.5 * (hp + hq[u]);
                        lim = hpq * hpq;
                    }
                    if (q0 + u < m && q != p && r2 < lim) visit(count++, (int32_t)q);
                }
            }
        }
    }
    return count;
}

// One search per particle: its neighbours go to `found` (neighbour k of particle
// p at k n + p, as many as k_cap), its slice's width (64 times the most
// neighbours of one of its particles: a slice is a wave) to slice_ptr[slice + 1],
// for the scan.  Cells are found through the table; a binary search of the
// sorted keys for each, once to count and once more to fill, took 277 + 290 us
// for 200k particles, this and k_fill 160 + 10.
static_assert(kSlice == 64, "a slice is a wave");
__global__ void __launch_bounds__(256) k_count(DevState s, const double* __restrict__ bbox,
                                               const CSlot* __restrict__ cell, int64_t H, int shift, int k_cap,
                                               int32_t* __restrict__ nnb,
                                               int64_t* __restrict__ slice_ptr,
                                               int32_t* __restrict__ found) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= s.np) return;   // (whole waves: np is a multiple of the slice)
    int cnt = 0;
    if (p < s.n)
        cnt = for_neighbours(s, bbox, cell, H, shift, p, [&](int k, int32_t q) {
            if (k < k_cap) found[(int64_t)k * s.n + p] = q;
        });
    nnb[p] = cnt;
    const uint64_t grouped = __ballot(p < s.n && s.bc[p] >= 0);
    int most = cnt, sum = cnt;
    for (int w = 32; w > 0; w >>= 1) {
        most = max(most, __shfl_xor(most, w));
        sum += __shfl_xor(sum, w);
    }
    if (p % kSlice == 0) {
        slice_ptr[p / kSlice + 1] = (int64_t)most * kSlice;
        if (p == 0) slice_ptr[0] = 0;
        atomicMax(&s.err[1], most);
        if (grouped) atomicAdd(&s.err[5], (int)__popcll(grouped));
        atomicAdd(reinterpret_cast<unsigned long long*>(&s.err[6]), (unsigned long long)sum);
    }
}

// In-place inclusive scan of a[0..m) with no memory but a itself, so that calls
// on several streams share nothing: chunks of kScanB kScanPer values, then
// their last values (the chunks' sums) by one workgroup, then each chunk from
// the last value of the one before it, which its own workgroup leaves alone.
constexpr int kScanB = 256, kScanPer = 8;
constexpr int64_t kScanChunk = kScanB * kScanPer;
// Inclusive scan of v over the workgroup; total: its sum.
__device__ __forceinline__ int64_t block_scan(int64_t v, int64_t* red, int64_t* total) {
    const int t = threadIdx.x;
    red[t] = v;
    __syncthreads();
    for (int w = 1; w < kScanB; w <<= 1) {
        const int64_t u = t >= w ? red[t - w] : 0;
        __syncthreads();
        red[t] += u;
        __syncthreads();
    }
    v = red[t];
    *total = red[kScanB - 1];
    __syncthreads();
    return v;
}
__global__ void __launch_bounds__(kScanB) k_scan_chunks(int64_t* __restrict__ a, int64_t m) {
    __shared__ int64_t red[kScanB];
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanPer;
    int64_t v[kScanPer], sum = 0, total;
#pragma unroll
    for (int u = 0; u < kScanPer; ++u) {
        if (base + u < m) sum += a[base + u];
        v[u] = sum;
    }
    const int64_t before = block_scan(sum, red, &total) - sum;
#pragma unroll
    for (int u = 0; u < kScanPer; ++u)
        if (base + u < m) a[base + u] = before + v[u];
}
__global__ void __launch_bounds__(kScanB) k_scan_ends(int64_t* __restrict__ a, int64_t m,
                                                      int64_t chunks) {
    __shared__ int64_t red[kScanB];
    int64_t before = 0;
    for (int64_t c0 = 0; c0 < chunks; c0 += kScanB) {
        const int64_t c = c0 + threadIdx.x;
        const int64_t end = (c + 1) * kScanChunk < m ? (c + 1) * kScanChunk : m;
        int64_t total;
        const int64_t v = block_scan(c < chunks ? a[end - 1] : 0, red, &total);
        if (c < chunks) a[end - 1] = before + v;
        before += total;
    }
}
__global__ void __launch_bounds__(kScanB) k_scan_add(int64_t* __restrict__ a, int64_t m) {
    const int64_t beg = ((int64_t)blockIdx.x + 1) * kScanChunk;   // (the first chunk is done)
    const int64_t end = beg + kScanChunk < m ? beg + kScanChunk : m;
    const int64_t before = a[beg - 1];
    for (int64_t q = beg + threadIdx.x; q < end - 1; q += kScanB) a[q] += before;
}
static hipError_t launch_scan(int64_t* a, int64_t m, hipStream_t st) {
    const int64_t chunks = (m + kScanChunk - 1) / kScanChunk;
    if (chunks == 0) return hipSuccess;
    k_scan_chunks<<<(unsigned)chunks, kScanB, 0, st>>>(a, m);
    if (chunks > 1) {
        k_scan_ends<<<1, kScanB, 0, st>>>(a, m, chunks);
        k_scan_add<<<(unsigned)(chunks - 1), kScanB, 0, st>>>(a, m);
    }
    return hipGetLastError();
}

__global__ void k_fill(DevState s, const int32_t* __restrict__ found, int32_t* __restrict__ col) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= s.np) return;
    const int64_t sl = p / kSlice;
    const int w = (int)((s.slice_ptr[sl + 1] - s.slice_ptr[sl]) / kSlice);
    int32_t* base = col + s.slice_ptr[sl] + (p % kSlice);
    const int cnt = p < s.n ? s.nnb[p] : 0;
    // the rest of the slice's width points at the particle itself (a valid
    // address for loops that run to the slice width and mask the excess)
    const int32_t self = p < s.n ? (int32_t)p : 0;
    for (int k = 0; k < w; ++k)
        base[(int64_t)k * kSlice] = k < cnt ? found[(int64_t)k * s.n + p] : self;
}

// Correction matrix L_i = sum_j V_j (X_j - X_i) (x) gradW_ij (eq.
// correction_matrix) and its inverse, in double.
__global__ void k_shape(DevState s, double* __restrict__ Linv, float* __restrict__ Linv32) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= s.np) return;
    const int64_t np = s.np;
    if (p >= s.n) {
        for (int k = 0; k < 9; ++k) {
            Linv[k * np + p] = 0.0;
            if (Linv32) Linv32[k * np + p] = 0.0f;
        }
        return;
    }
    const DevSpec& P = s.specs[s.spec[p]];
    const D4 xp = s.XV[p];
    double L[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int cnt = s.nnb[p];
    const int32_t* cp = s.col + s.slice_ptr[p / kSlice] + (p % kSlice);
    for (int k = 0; k < cnt; ++k) {
        const int32_t j = cp[(int64_t)k * kSlice];
        const D4 xj = s.XV[j];
        const double d[3] = {xj.x - xp.x, xj.y - xp.y, xj.z - xp.z};
        const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        double W, dW;
        if (s.var_h) {   // the pair's support
            const double h = 0.5 * (s.hs[p] + s.hs[j]);
            spline(r, 1.0 / h, 8.0 / (M_PI * h * h * h), W, dW);
        } else {
            spline(r, P.inv_h, P.wnorm, W, dW);
        }
        const double g = xj.w * dW / r;
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) L[3 * a + b] += d[a] * g * d[b];
    }
    double nrm = 0.0;
    for (int k = 0; k < 9; ++k) nrm += L[k] * L[k];
    nrm = sqrt(nrm);
    const double det = det33(L);
    double Li[9];
    if (!(fabs(det) > 1e-12 * nrm * nrm * nrm)) {
        atomicMin(&s.err[0], (int32_t)p);
        for (int k = 0; k < 9; ++k) Li[k] = 0.0;
    } else {
        inv33(L, Li);
    }
    for (int k = 0; k < 9; ++k) {
        Linv[k * np + p] = Li[k];
        if (Linv32) Linv32[k * np + p] = (float)Li[k];
    }
}

// initial state: u = 0, v = 0, F = I, stresses and accumulators 0, f = f0,
// D = q1 f*(f0) under GTN, Q = 0, t = 0
__global__ void k_init(DevState s) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < s.n_spec) s.t[p] = 0.0;
    if (p >= s.np) return;
    const int64_t np = s.np;
    const DevSpec& P = s.specs[s.spec[p]];
    const double D0 = (P.damage == 3) ? gtn_D(P, P.f0) : 0.0;
    s.U[0][p] = D4{0.0, 0.0, 0.0, 0.0};
    s.U[1][p] = D4{0.0, 0.0, 0.0, 0.0};
    s.VW[p] = D4{0.0, 0.0, 0.0, s.XV[p].w * (1.0 - D0)};
    for (int c = 0; c < 3; ++c) {
        s.force[c * np + p] = 0.0;
        s.fvisc[c * np + p] = 0.0;
    }
    s.ccnt[p] = 0;
    if (s.GQ) {
        GQRec<double> g;
        GHRec<double> h;
        for (int k = 0; k < 9; ++k) { g.q[k] = 0.0; h.h[k] = 0.0; }
        g.omd = 1.0 - D0;
        h.vw = s.XV[p].w * g.omd;
        s.GQ[p] = g;
        s.GH[p] = h;
    } else {
        GQRec<float> g;
        GHRec<float> h;
        for (int k = 0; k < 9; ++k) { g.q[k] = 0.0f; h.h[k] = 0.0f; }
        g.omd = (float)(1.0 - D0);
        h.vw = float(s.XV[p].w) * g.omd;
        s.GQ32[p] = g;
        s.GH32[p] = h;
    }
    for (int k = 0; k < 6; ++k) {
        if (s.sig) s.sig[k * np + p] = 0.0;
        if (s.sig32) s.sig32[k * np + p] = 0.0f;
    }
    s.eps_p[p] = 0.0;
    s.eps_rate[p] = 0.0;
    s.d_init[p] = 0.0;
    s.w_p[p] = 0.0;
    s.e[p] = 0.0;
    s.f_void[p] = P.f0;
    s.D[p] = D0;
}

hipError_t launch_build_count(DevState& s, const BuildBuffers& b, hipStream_t st) {
    const int T = 256;
    unsigned long long* bits = reinterpret_cast<unsigned long long*>(b.bbox);
    k_bbox_clear<<<(s.n_spec * kBBox + T - 1) / T, T, 0, st>>>(bits, s.n_spec);
    k_bbox<<<(unsigned)b.chunks, 256, 0, st>>>(b.X_in, b.V0_in, s.n, b.spec_off, b.seg, s.n_spec,
                                               bits);
    k_bbox_final<<<(s.n_spec + T - 1) / T, T, 0, st>>>(b.bbox, s.n_spec, s.specs);
    k_keys<<<(unsigned)((b.n_pow2 + T - 1) / T), T, 0, st>>>(b.X_in, s.n, b.n_pow2, b.spec_off,
                                                             s.n_spec, b.bbox, b.keys, b.vals,
                                                             s.err);
    hipError_t e = launch_bitonic_sort(b.keys, b.vals, b.n_pow2, st);
    if (e != hipSuccess) return e;
    const unsigned gp = (unsigned)((s.np + T - 1) / T);
    k_apply_perm<<<gp, T, 0, st>>>(s, b.X_in, b.V0_in, b.bc_in, b.keys, b.vals,
                                   const_cast<D4*>(s.XV), const_cast<int32_t*>(s.spec),
                                   const_cast<int32_t*>(s.bc), const_cast<int32_t*>(s.perm),
                                   const_cast<int32_t*>(s.iperm));
    k_spec_ranges<<<(s.n_spec + 63) / 64, 64, 0, st>>>(const_cast<DevSpec*>(s.specs), s.n_spec,
                                                      b.keys, s.n);
    const unsigned gh = (unsigned)((b.H + T - 1) / T);
    k_cells_clear<<<gh, T, 0, st>>>(b.cell, b.H);
    const int shift = table_shift(b.H);
    k_cells_insert<<<(unsigned)((s.n + T - 1) / T), T, 0, st>>>(s, b.keys, b.bbox, b.cell, b.H,
                                                                shift);
    k_count<<<gp, T, 0, st>>>(s, b.bbox, b.cell, b.H, shift, b.k_cap,
                              const_cast<int32_t*>(s.nnb), const_cast<int64_t*>(s.slice_ptr),
                              b.found);
    return launch_scan(const_cast<int64_t*>(s.slice_ptr) + 1, s.np / kSlice, st);
}

// One workgroup per tile of T particles: collect the indices of the tile's
// neighbours outside the tile, each once (a hash set in LDS, whose E slots
// hold every entry even if all differ), sort them (bitonic, in LDS: the halo,
// ascending), then give every neighbour entry its local slot: j - start
// inside the tile, T + position in the halo outside.  Sorting the distinct
// indices alone (about two per particle) instead of all T k_cap entries is
// what this form is for: 200k particles, tiles of 196, 82 us against
// 688.
__global__ void __launch_bounds__(256) k_halo(DevState s, int E, int32_t* __restrict__ halo,
                                              int32_t* __restrict__ halo_cnt,
                                              uint16_t* __restrict__ lcol,
                                              uint32_t* __restrict__ pslot) {
    extern __shared__ int32_t sh[];
    int32_t* set = sh;            // [E]
    int32_t* hl = sh + E;         // [E]
    int32_t* count = sh + 2 * E;  // [1]
    constexpr int32_t kNone = 0x7fffffff;
    const int tid = threadIdx.x;
    const int T = s.tile;                  // particles per tile (<= 256 threads)
    const int64_t t = blockIdx.x;
    const int64_t start = t * T;
    const int64_t end = start + T < s.n ? start + T : s.n;
    for (int e = tid; e < E; e += 256) set[e] = kNone;
    if (tid == 0) *count = 0;
    __syncthreads();
    const int64_t p = start + tid;
    const bool mine = tid < T;             // thread tid holds particle start + tid
    int cnt = 0;
    const int32_t* cp = nullptr;
    if (mine && p < s.n) {
        cnt = s.nnb[p];
        cp = s.col + s.slice_ptr[p / kSlice] + (p % kSlice);
        for (int k = 0; k < cnt; ++k) {
            const int32_t j = cp[(int64_t)k * kSlice];
            if (j >= start && j < end) continue;
            // (a free slot always comes up: at most T k_cap <= E entries go in)
            for (uint32_t h = (uint32_t)j * 2654435761u >> 7;; ++h) {
                const int32_t was = atomicCAS(&set[h & (E - 1)], kNone, j);
                if (was == kNone) hl[atomicAdd(count, 1)] = j;
                if (was == kNone || was == j) break;
            }
        }
    }
    __syncthreads();
    const int H = *count;
    int N = 64;
    while (N < H) N <<= 1;        // (N <= E, a power of two that holds H)
    for (int e = H + tid; e < N; e += 256) hl[e] = kNone;
    __syncthreads();
    for (int k = 2; k <= N; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int q = tid; q < N / 2; q += 256) {
                const int e = 2 * q - (q & (j - 1)), l = e + j;
                const int32_t a = hl[e], b = hl[l];
                if ((a > b) == ((e & k) == 0)) {
                    hl[e] = b;
                    hl[l] = a;
                }
            }
            __syncthreads();
        }
    for (int h = tid; h < H; h += 256) halo[t * s.halo_cap + h] = hl[h];
    // past the count, n (no particle) for as far as a staging round reads
    const int pad_end = H + kHaloPad < s.halo_cap ? H + kHaloPad : s.halo_cap;
    for (int h = H + tid; h < pad_end; h += 256) halo[t * s.halo_cap + h] = (int32_t)s.n;
    if (tid == 0) {
        halo_cnt[t] = H;
        atomicMax(&s.err[4], H);
    }
    if (mine && p < s.np) {
        const int64_t sl = p / kSlice;
        const int w = (int)((s.slice_ptr[sl + 1] - s.slice_ptr[sl]) / kSlice);
        uint16_t* lp = lcol + s.slice_ptr[sl] + (p % kSlice);
        for (int k = cnt; k < w; ++k) lp[(int64_t)k * kSlice] = (uint16_t)tid;
    }
    if (mine && p < s.n) {
        uint16_t* lp = lcol + s.slice_ptr[p / kSlice] + (p % kSlice);
        for (int k = 0; k < cnt; ++k) {
            const int32_t j = cp[(int64_t)k * kSlice];
            int loc;
            if (j >= start && j < end) {
                loc = (int)(j - start);
            } else {
                int lo = 0, hi = H;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (hl[mid] < j) lo = mid + 1; else hi = mid;
                }
                loc = T + lo;
            }
            lp[(int64_t)k * kSlice] = (uint16_t)loc;
        }
        if (!pslot) return;
        // the first kPackGroups groups of kSub neighbours as they are read (see
        // Slots), the first neighbour (or the particle) past the last
        uint32_t o[kPackWords];
#pragma unroll
        for (int w = 0; w < kPackWords; ++w) {
            o[w] = 0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int e = 2 * w + q, k = (e % kPackGroups) * kSub + e / kPackGroups;
                const uint32_t m = cnt > 0 ? lp[(int64_t)(k < cnt ? k : 0) * kSlice] : (uint32_t)tid;
                o[w] |= m << (16 * q);
            }
        }
        uint4* out = reinterpret_cast<uint4*>(pslot + p * kPackWords);
#pragma unroll
        for (int w = 0; w < kPackWords / 4; ++w)
            out[w] = uint4{o[4 * w], o[4 * w + 1], o[4 * w + 2], o[4 * w + 3]};
    }
}

hipError_t launch_halo(const DevState& s, int k_cap, int T, int32_t* halo, int32_t* halo_cnt,
                       uint16_t* lcol, uint32_t* pslot, hipStream_t st) {
    if (T < 1 || T > kTile) return hipErrorInvalidValue;
    int E = 256;
    while (E < T * k_cap) E <<= 1;
    const size_t lds = (2 * (size_t)E + 257) * sizeof(int32_t);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_halo),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    DevState t = s;   // the kernel reads the tile size and list stride from it
    t.tile = T;
    t.halo_cap = T * k_cap;
    const unsigned tiles = (unsigned)((s.n + T - 1) / T);
    k_halo<<<tiles, 256, lds, st>>>(t, E, halo, halo_cnt, lcol, pslot);
    return hipGetLastError();
}

// Only after the host has checked that the sliced list fits col.
hipError_t launch_build_fill(DevState& s, const BuildBuffers& b, hipStream_t st) {
    const int T = 256;
    const unsigned gp = (unsigned)((s.np + T - 1) / T);
    k_fill<<<gp, T, 0, st>>>(s, b.found, const_cast<int32_t*>(s.col));
    return hipGetLastError();
}

hipError_t launch_shape_and_init(const DevState& s, bool mixed, hipStream_t st) {
    const int T = 256;
    const unsigned gp = (unsigned)((s.np + T - 1) / T);
    k_shape<<<gp, T, 0, st>>>(s, const_cast<double*>(s.Linv),
                              mixed ? const_cast<float*>(s.Linv32) : nullptr);
    const int64_t m = s.np > s.n_spec ? s.np : s.n_spec;
    k_init<<<(unsigned)((m + T - 1) / T), T, 0, st>>>(s);
    return hipGetLastError();
}

// ===========================================================================
// the step
// ===========================================================================

// Two sweeps with two lanes per particle.
__global__ void __launch_bounds__(staged_block_max(2))
__attribute__((amdgpu_waves_per_eu(staged_waves_min<2>(), 8))) k_pass_b_wide(DevState s, int par) {
    pass_b_sweeps<2, false>(s, par);
}

template <int S>
static hipError_t launch_b(const DevState& s, int parity, int block, bool mixed, hipStream_t st,
                           size_t lds_bytes) {
    if (s.staged) {
        const unsigned grid = (unsigned)s.grid_b;
        const int threads = s.tile * S;
        if (s.form_b == kFormOne) {
            if (s.var_h) {   // graded spacing: per-pair supports
                if (mixed)
                    k_pass_b_one<float, S, true><<<grid, threads, lds_bytes, st>>>(s, parity);
                else
                    k_pass_b_one<double, S, true><<<grid, threads, lds_bytes, st>>>(s, parity);
            } else if (mixed) {
                k_pass_b_one<float, S><<<grid, threads, lds_bytes, st>>>(s, parity);
            } else {
                k_pass_b_one<double, S><<<grid, threads, lds_bytes, st>>>(s, parity);
            }
        } else if (s.form_b == kFormPipe) {
            if (S != 2 || s.var_h) return hipErrorInvalidValue;
            if (!mixed) return launch_pipe_fp64(s, parity, st, lds_bytes);
            k_pass_b_staged<float, 2><<<grid, threads, lds_bytes, st>>>(s, parity);
        } else {
            if (mixed) return hipErrorInvalidValue;
            if (s.var_h)
                k_pass_b_staged<double, S, true><<<grid, threads, lds_bytes, st>>>(s, parity);
            else if constexpr (S == 2)
                k_pass_b_wide<<<grid, threads, lds_bytes, st>>>(s, parity);
            else
                k_pass_b_staged<double, S><<<grid, threads, lds_bytes, st>>>(s, parity);
        }
        return hipGetLastError();
    }
    const unsigned grid = (unsigned)((s.n * S + block - 1) / block);
    if (s.var_h) {   // graded spacing: per-pair supports
        if (mixed)
            k_pass_b<float, S, true><<<grid, block, 0, st>>>(s, parity);
        else
            k_pass_b<double, S, true><<<grid, block, 0, st>>>(s, parity);
        return hipGetLastError();
    }
    if (mixed)
        k_pass_b<float, S><<<grid, block, 0, st>>>(s, parity);
    else
        k_pass_b<double, S><<<grid, block, 0, st>>>(s, parity);
    return hipGetLastError();
}

hipError_t launch_pass_b(const DevState& s, int parity, int block, int sub, bool mixed,
                         hipStream_t st, size_t lds_bytes) {
    if (!s.staged && (block <= 0 || block > 256 || block % sub != 0)) return hipErrorInvalidValue;
    switch (sub) {
        case 1: return launch_b<1>(s, parity, block, mixed, st, lds_bytes);
        case 2: return launch_b<2>(s, parity, block, mixed, st, lds_bytes);
        case 4: return launch_b<4>(s, parity, block, mixed, st, lds_bytes);
        default: return hipErrorInvalidValue;
    }
}

const char* pass_b_name(const DevState& s, int sub) {
    if (!s.staged) return "k_pass_b";
    if (s.form_b == kFormOne) return "k_pass_b_one";
    return s.form_b == kFormSweeps && sub == 2 && !s.var_h ? "k_pass_b_wide" : "k_pass_b_staged";
}

const char* pass_a_name(const DevState& s, int block, bool mixed) {
    if (block != 0) return "k_pass_a";
    return mixed && !s.flow_general && !s.var_h && update_packed(s) ? "k_pass_a_packed"
                                                                    : "k_pass_a_staged";
}

int staged_tile_max(int sub) { return staged_block_max(sub) / sub; }

size_t staged_one_bytes(bool mixed, bool var_h) {
    return (size_t)(mixed ? LdsOne<float>::kUnits : LdsOne<double>::kUnits) * 16 + (var_h ? 8 : 0);
}

size_t staged_sweep_bytes(bool var_h) { return LdsB<double>::kBytes + (var_h ? 8 : 0); }

size_t staged_pipe_bytes(bool mixed) {
    return (size_t)(mixed ? LdsP<float>::kBytes : LdsP<double>::kBytes);
}

int staged_pipe_neighbours() { return kSub * kPipeGroups; }

// Workgroups of the pipelined force pass (threads and LDS bytes each) that
// share a CU.
hipError_t staged_blocks_per_cu(bool mixed, int threads, size_t lds_bytes, int* out) {
    const void* f = mixed ? reinterpret_cast<const void*>(&k_pass_b_staged<float, 2>) : pipe_fp64();
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(out, f, threads, lds_bytes);
}

size_t staged_a_record_bytes(bool var_h) { return kLdsABytes + (var_h ? 8 : 0); }

// Dynamic LDS above the default limit must be allowed per kernel.
hipError_t prepare_staged(size_t lds_bytes_b) {
    const void* const fns[] = {
        reinterpret_cast<const void*>(&k_pass_b_wide),
        reinterpret_cast<const void*>(&k_pass_b_staged<double, 1>),
        pipe_fp64(),
        reinterpret_cast<const void*>(&k_pass_b_staged<float, 2>),
        reinterpret_cast<const void*>(&k_pass_b_staged<double, 4>),
        reinterpret_cast<const void*>(&k_pass_b_staged<double, 1, true>),
        reinterpret_cast<const void*>(&k_pass_b_staged<double, 2, true>),
        reinterpret_cast<const void*>(&k_pass_b_staged<double, 4, true>),
        reinterpret_cast<const void*>(&k_pass_b_one<double, 1>),
        reinterpret_cast<const void*>(&k_pass_b_one<float, 1>),
        reinterpret_cast<const void*>(&k_pass_b_one<double, 2>),
        reinterpret_cast<const void*>(&k_pass_b_one<float, 2>),
        reinterpret_cast<const void*>(&k_pass_b_one<double, 4>),
        reinterpret_cast<const void*>(&k_pass_b_one<float, 4>),
        reinterpret_cast<const void*>(&k_pass_b_one<double, 1, true>),
        reinterpret_cast<const void*>(&k_pass_b_one<float, 1, true>),
        reinterpret_cast<const void*>(&k_pass_b_one<double, 2, true>),
        reinterpret_cast<const void*>(&k_pass_b_one<float, 2, true>),
        reinterpret_cast<const void*>(&k_pass_b_one<double, 4, true>),
        reinterpret_cast<const void*>(&k_pass_b_one<float, 4, true>)};
    for (const void* f : fns) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds_bytes_b);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int DM, bool kFlow, bool kVarH = false>
static void launch_a(const DevState& s, int parity, int block, bool mixed, hipStream_t st) {
    if (mixed) {
        if constexpr (registers_full<float, DM, kFlow>())
            launch_update_full(s, parity, block, DM, true, st);
        else
            launch_update<float, DM, kFlow, kVarH>(s, parity, block, st);
    } else {
        if constexpr (registers_full<double, DM, kFlow>())
            launch_update_full(s, parity, block, DM, false, st);
        else
            launch_update<double, DM, kFlow, kVarH>(s, parity, block, st);
    }
}

hipError_t launch_pass_a(const DevState& s, int parity, int block, bool mixed, hipStream_t st) {
    if (block == 0 && (!s.staged_lds_a || s.a_group < 1 || s.a_group > 2 ||
                       s.tile_a * s.a_group > 256))
        return hipErrorInvalidValue;
    if (s.var_h) {   // graded spacing: the general variant with per-pair supports
        launch_a<-1, true, true>(s, parity, block, mixed, st);
        return hipGetLastError();
    }
    if (s.flow_general) {
        switch (s.model) {
            case 0: launch_a<0, true>(s, parity, block, mixed, st); break;
            case 1: launch_a<1, true>(s, parity, block, mixed, st); break;
            case 2: launch_a<2, true>(s, parity, block, mixed, st); break;
            case 3: launch_a<3, true>(s, parity, block, mixed, st); break;
            default: launch_a<-1, true>(s, parity, block, mixed, st); break;
        }
    } else {
        switch (s.model) {
            case 0: launch_a<0, false>(s, parity, block, mixed, st); break;
            case 1: launch_a<1, false>(s, parity, block, mixed, st); break;
            case 2: launch_a<2, false>(s, parity, block, mixed, st); break;
            case 3: launch_a<3, false>(s, parity, block, mixed, st); break;
            default: launch_a<-1, false>(s, parity, block, mixed, st); break;
        }
    }
    return hipGetLastError();
}

// ===========================================================================
// field access in caller order
// ===========================================================================

enum Field {
    F_X = 0, F_U, F_V, F_DEFGRAD, F_SIGMA, F_EPS_P, F_EPS_P_RATE, F_D_INIT, F_W_P, F_VOID,
    F_D, F_E_INT, F_FORCE, F_Q, F_TIME, F_LINV, F_VISC, F_H
};

struct FieldRef {
    const double* d;   // double storage, or
    const float* f;    // float storage
    int comps;
    int kind;          // 0 plain, 1 deformation gradient stored as F - I, 2 damage
    int64_t cs, ps;    // element (particle p, component c) at [c * cs + p * ps]
};

__device__ __forceinline__ FieldRef field_ref(const DevState& s, int field, int par) {
    const int64_t np = s.np;
    constexpr int64_t kRec32 = sizeof(GQRec<float>) / 4;
    switch (field) {
        case F_X: return {reinterpret_cast<const double*>(s.XV), nullptr, 3, 0, 1, 4};
        case F_U: return {reinterpret_cast<const double*>(s.U[par]), nullptr, 3, 0, 1, 4};
        case F_V: return {reinterpret_cast<const double*>(s.VW), nullptr, 3, 0, 1, 4};
        case F_DEFGRAD:
            return s.GH ? FieldRef{reinterpret_cast<const double*>(s.GH), nullptr, 9, 1, 1, 10}
                        : FieldRef{nullptr, reinterpret_cast<const float*>(s.GH32), 9, 1, 1, kRec32};
        case F_H:   // F - I as stored, without the round trip through F
            return s.GH ? FieldRef{reinterpret_cast<const double*>(s.GH), nullptr, 9, 0, 1, 10}
                        : FieldRef{nullptr, reinterpret_cast<const float*>(s.GH32), 9, 0, 1, kRec32};
        case F_Q:
            return s.GQ ? FieldRef{reinterpret_cast<const double*>(s.GQ), nullptr, 9, 0, 1, 10}
                        : FieldRef{nullptr, reinterpret_cast<const float*>(s.GQ32), 9, 0, 1, kRec32};
        case F_SIGMA:
            return s.sig ? FieldRef{s.sig, nullptr, 6, 0, np, 1} : FieldRef{nullptr, s.sig32, 6, 0, np, 1};
        case F_EPS_P: return {s.eps_p, nullptr, 1, 0, np, 1};
        case F_EPS_P_RATE: return {s.eps_rate, nullptr, 1, 0, np, 1};
        case F_D_INIT: return {s.d_init, nullptr, 1, 0, np, 1};
        case F_W_P: return {s.w_p, nullptr, 1, 0, np, 1};
        case F_VOID: return {s.f_void, nullptr, 1, 0, np, 1};
        case F_D: return {s.D, nullptr, 1, 2, np, 1};
        case F_E_INT: return {s.e, nullptr, 1, 0, np, 1};
        case F_FORCE: return {s.force, nullptr, 3, 0, np, 1};
        case F_LINV: return {s.Linv, nullptr, 9, 0, np, 1};
        case F_VISC: return {s.fvisc, nullptr, 3, 0, np, 1};
        default: return {nullptr, nullptr, 0, 0, 0, 0};
    }
}

__global__ void k_get(DevState s, int field, int par, double* __restrict__ dst) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= s.n) return;
    const FieldRef r = field_ref(s, field, par);
    const int64_t p = s.iperm[i];
    for (int c = 0; c < r.comps; ++c) {
        const int64_t at = c * r.cs + p * r.ps;
        double x = r.d ? r.d[at] : (double)r.f[at];
        if (r.kind == 1 && (c % 4 == 0)) x += 1.0;
        dst[c * s.n + i] = x;
    }
}

// Writes keep the gathered copies consistent: damage also sets 1 - D and V0 (1
// - D) in the force-pass records and V0 (1 - D) in the velocity record.
__global__ void k_set(DevState s, int field, int par, const double* __restrict__ src) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= s.n) return;
    const FieldRef r = field_ref(s, field, par);
    const int64_t p = s.iperm[i];
    for (int c = 0; c < r.comps; ++c) {
        double x = src[c * s.n + i];
        if (r.kind == 1 && (c % 4 == 0)) x -= 1.0;
        const int64_t at = c * r.cs + p * r.ps;
        if (r.d)
            const_cast<double*>(r.d)[at] = x;
        else
            const_cast<float*>(r.f)[at] = (float)x;
    }
    if (r.kind == 2) {
        const double D = src[i];
        if (s.GQ) {
            s.GQ[p].omd = 1.0 - D;
            s.GH[p].vw = s.XV[p].w * s.GQ[p].omd;
        } else {
            s.GQ32[p].omd = (float)(1.0 - D);
            s.GH32[p].vw = float(s.XV[p].w) * s.GQ32[p].omd;
        }
        s.VW[p].w = s.XV[p].w * (1.0 - D);
    }
}

hipError_t launch_get_field(const DevState& s, int field, int parity, bool, double* dst,
                            hipStream_t st) {
    const int T = 256;
    k_get<<<(unsigned)((s.n + T - 1) / T), T, 0, st>>>(s, field, parity, dst);
    return hipGetLastError();
}

hipError_t launch_set_field(const DevState& s, int field, int parity, bool, const double* src,
                            hipStream_t st) {
    const int T = 256;
    k_set<<<(unsigned)((s.n + T - 1) / T), T, 0, st>>>(s, field, parity, src);
    return hipGetLastError();
}

// ===========================================================================
// neighbour export (caller order, ascending rows)
// ===========================================================================

__global__ void k_export_count(DevState s, int64_t* __restrict__ row_ptr) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) row_ptr[0] = 0;
    if (i >= s.n) return;
    row_ptr[i + 1] = s.nnb[s.iperm[i]];
}

__global__ void k_export_fill(DevState s, const int64_t* __restrict__ row_ptr,
                              int32_t* __restrict__ col_out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= s.n) return;
    const int64_t p = s.iperm[i];
    const int cnt = s.nnb[p];
    const int32_t* cp = s.col + s.slice_ptr[p / kSlice] + (p % kSlice);
    int32_t* out = col_out + row_ptr[i];
    for (int k = 0; k < cnt; ++k) {
        const int32_t v = s.perm[cp[(int64_t)k * kSlice]];
        int q = k;
        while (q > 0 && out[q - 1] > v) {
            out[q] = out[q - 1];
            --q;
        }
        out[q] = v;
    }
}

hipError_t launch_export_neighbors(const DevState& s, int64_t* row_ptr, int32_t* col,
                                   hipStream_t st) {
    const int T = 256;
    const unsigned g = (unsigned)((s.n + T - 1) / T);
    k_export_count<<<g, T, 0, st>>>(s, row_ptr);
    hipError_t e = launch_scan(row_ptr + 1, s.n, st);
    if (e != hipSuccess) return e;
    k_export_fill<<<g, T, 0, st>>>(s, row_ptr, col);
    return hipGetLastError();
}

// ===========================================================================
// diagnostics
// ===========================================================================

// Members of each prescribed-velocity group, ordered by (group, sorted index):
// the m particles with a group, in any order (their number, counted with the
// neighbours, counts down to 0), and padding to N, to be sorted.
__global__ void k_bc_keys(DevState s, uint64_t* __restrict__ keys, int32_t* __restrict__ vals,
                          int64_t m, int64_t N) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int g = (p < s.n) ? s.bc[p] : -1;
    if (g >= 0) {
        const int64_t at = (int64_t)atomicSub(&s.err[5], 1) - 1;
        keys[at] = ((uint64_t)g << 32) | (uint64_t)p;
        vals[at] = (int32_t)p;
    }
    if (p >= m && p < N) {
        keys[p] = ~0ull;
        vals[p] = 0x7fffffff;
    }
}

__global__ void k_bc_ptr(DevState s, const uint64_t* __restrict__ keys, int64_t n,
                         const int32_t* __restrict__ vals, int32_t* __restrict__ bc_list,
                         int64_t* __restrict__ bc_ptr) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t <= s.n_bc) {
        const uint64_t key = (uint64_t)t << 32;
        int64_t lo = 0, hi = n;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (keys[mid] < key) lo = mid + 1; else hi = mid;
        }
        bc_ptr[t] = lo;
    }
    if (t < n) bc_list[t] = vals[t];
}

// ===========================================================================
// penalty contact: candidate lists from the current configuration
// ===========================================================================

// Bounding box of the current positions and the largest contact radius over
// every particle, in two stages: kCBoxParts workgroups each reduce a
// contiguous share of the particles to 7 partial extrema (lo[3], hi[3],
// max a) after the header, then one workgroup reduces those to the header:
// cbox = lo[3], hi[3], 1 / cell edge, cell edge (the edge 2 max a + skin, a
// hair larger), then the grid's extent in cells along x, y, z and whether
// the grid is dense (its cells fit the slot table, see CHash).  Minima and
// maxima do not depend on the order of reduction.
constexpr int kCBoxThreads = 256;

__device__ __forceinline__ void cbox_reduce(double (*red)[kCBoxThreads], double v[7]) {
    for (int a = 0; a < 7; ++a) red[a][threadIdx.x] = v[a];
    __syncthreads();
    for (int w = kCBoxThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int a = 0; a < 7; ++a) {
                const double o = red[a][threadIdx.x + w];
                red[a][threadIdx.x] = a < 3 ? fmin(red[a][threadIdx.x], o)
                                            : fmax(red[a][threadIdx.x], o);
            }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kCBoxThreads) k_cbox_part(DevState s, int par,
                                                             double* __restrict__ cbox) {
    __shared__ double red[7][kCBoxThreads];
    const D4* __restrict__ Uc = s.U[par];
    double v[7] = {1e300, 1e300, 1e300, -1e300, -1e300, -1e300, 0.0};
    const int64_t share = (s.n + kCBoxParts - 1) / kCBoxParts;
    const int64_t p0 = (int64_t)blockIdx.x * share;
    const int64_t p1 = p0 + share < s.n ? p0 + share : s.n;
    for (int64_t p = p0 + threadIdx.x; p < p1; p += kCBoxThreads) {
        const D4 x = s.XV[p], u = Uc[p];
        const double c[3] = {x.x + u.x, x.y + u.y, x.z + u.z};
        for (int a = 0; a < 3; ++a) {
            v[a] = fmin(v[a], c[a]);
            v[3 + a] = fmax(v[3 + a], c[a]);
        }
        v[6] = fmax(v[6], s.arad[p]);
    }
    cbox_reduce(red, v);
    if (threadIdx.x < 7) cbox[kCBoxHead + (int64_t)blockIdx.x * 7 + threadIdx.x] = red[threadIdx.x][0];
}

__global__ void __launch_bounds__(kCBoxThreads) k_cbox_final(DevState s, double* __restrict__ cbox,
                                                              int64_t n_slots) {
    __shared__ double red[7][kCBoxThreads];
    double v[7] = {1e300, 1e300, 1e300, -1e300, -1e300, -1e300, 0.0};
    for (int b = threadIdx.x; b < kCBoxParts; b += kCBoxThreads)
        for (int a = 0; a < 7; ++a) {
            const double o = cbox[kCBoxHead + (int64_t)b * 7 + a];
            v[a] = a < 3 ? fmin(v[a], o) : fmax(v[a], o);
        }
    cbox_reduce(red, v);
    if (threadIdx.x < 6) cbox[threadIdx.x] = red[threadIdx.x][0];
    if (threadIdx.x == 0) {
        const double edge = (2.0 * red[6][0] + s.contact_skin) * (1.0 + 1e-9);
        const double inv = 1.0 / edge;
        cbox[6] = inv;
        cbox[7] = edge;
        // the cell of the largest coordinate, computed as every particle's
        // own (so no particle lies beyond it), bounds the extent
        double cells = 1.0;
        for (int a = 0; a < 3; ++a) {
            // (no finite position at all: an empty box, one cell)
            const double q = floor((red[3 + a][0] - red[a][0]) * inv);
            const double e = !(q >= 0.0) ? 1.0
                             : q >= (double)((1 << kCellBits) - 1) ? (double)(1 << kCellBits)
                                                                     : q + 1.0;
            cbox[9 + a] = e;
            cells *= e;
        }
        cbox[8] = cells <= (double)n_slots ? 1.0 : 0.0;
    }
}

__device__ __forceinline__ bool contact_cell(const double* cb, double x, double y, double z,
                                             int32_t c[3]) {
    constexpr double kLast = (double)((1 << kCellBits) - 1);
    const double xs[3] = {x, y, z};
    bool ok = true;
    for (int a = 0; a < 3; ++a) {
        const double q = floor((xs[a] - cb[a]) * cb[6]);
        // (a position that is not a number lands in cell 0 and is flagged)
        c[a] = !(q >= 0.0) ? 0 : (q >= kLast ? (1 << kCellBits) - 1 : (int32_t)q);
        if (!(q < kLast)) ok = false;
    }
    return ok;
}

// Packed key of a contact cell (coordinates below 2^kCellBits each).
__device__ __forceinline__ uint64_t ccell_key(const int32_t c[3]) {
    return (uint64_t)c[0] | ((uint64_t)c[1] << kCellBits) |
           ((uint64_t)c[2] << (2 * kCellBits));
}

// The grid as the rebuild's kernels read it from the bounding box: dense
// (slot = linear cell index, x fastest) or hashed, and its extent.
struct CGrid {
    bool dense;
    int32_t ext[3];
};
__device__ __forceinline__ CGrid cgrid(const double* cbox) {
    return CGrid{cbox[8] != 0.0, {(int32_t)cbox[9], (int32_t)cbox[10], (int32_t)cbox[11]}};
}
__device__ __forceinline__ int64_t cgrid_slot(const CGrid& g, int32_t x, int32_t y, int32_t z) {
    return ((int64_t)z * g.ext[1] + y) * g.ext[0] + x;
}

// First slot probed for a key (Fibonacci hashing), then linear probing.

__global__ void k_chash_clear(CHash h) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= h.H) return;
    h.slot[t] = CSlot{~0ull, 0, 0};
}

// Each particle claims (or finds) its cell's slot and takes a place in the
// cell's group: rank[p] = slot << 32 | place (the place depends on the order
// of the atomics; the groups are put in index order afterwards).  Keys only
// ever go from empty to set, so particles of one cell, probing the same
// sequence, all stop at the same slot.
__global__ void k_chash_insert(DevState s, int par, const double* __restrict__ cbox, CHash h,
                               uint64_t* __restrict__ rank) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= s.n) return;
    const D4 x = s.XV[p], u = s.U[par][p];
    int32_t c[3];
    if (!contact_cell(cbox, x.x + u.x, x.y + u.y, x.z + u.z, c)) atomicOr(&s.err[2], kErrContact);
    const CGrid G = cgrid(cbox);
    int64_t t;
    if (G.dense) {
        // every cell lies inside the extent (the extent is the cell of the
        // largest coordinate, computed the same way); the clamp only keeps
        // the slot inside the table whatever the input
        for (int a = 0; a < 3; ++a) c[a] = c[a] < G.ext[a] ? c[a] : G.ext[a] - 1;
        t = cgrid_slot(G, c[0], c[1], c[2]);
    } else {
        const uint64_t key = ccell_key(c);
        t = cell_home(key, h.shift);
        for (;;) {
            const unsigned long long old =
                atomicCAS((unsigned long long*)&h.slot[t].key, ~0ull, (unsigned long long)key);
            if (old == ~0ull || old == key) break;
            t = (t + 1) & (h.H - 1);
        }
    }
    const int32_t place = atomicAdd(&h.slot[t].cnt, 1);
    rank[p] = ((uint64_t)t << 32) | (uint32_t)place;
}

// Exclusive prefix sum of the slot counts, first within blocks of
// kCHashScanB slots (256 threads, 16 consecutive slots each) into the slots'
// start, each block's total into boff; then over the blocks
// (k_chash_scan_top).
__global__ void __launch_bounds__(256) k_chash_scan(CHash h) {
    constexpr int kPer = kCHashScanB / 256;
    __shared__ int32_t tot[256];
    const int64_t i0 = (int64_t)blockIdx.x * kCHashScanB + (int64_t)threadIdx.x * kPer;
    int32_t v[kPer];
    int32_t run = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int32_t c = (i0 + k < h.H) ? h.slot[i0 + k].cnt : 0;
        v[k] = run;
        run += c;
    }
    tot[threadIdx.x] = run;
    __syncthreads();
    // inclusive scan of the thread totals (Hillis-Steele)
    for (int d = 1; d < 256; d <<= 1) {
        const int32_t o = (int)threadIdx.x >= d ? tot[threadIdx.x - d] : 0;
        __syncthreads();
        tot[threadIdx.x] += o;
        __syncthreads();
    }
    const int32_t base = tot[threadIdx.x] - run;
#pragma unroll
    for (int k = 0; k < kPer; ++k)
        if (i0 + k < h.H) h.slot[i0 + k].start = base + v[k];
    if (threadIdx.x == 255) h.boff[blockIdx.x] = tot[255];
}

__global__ void __launch_bounds__(1024) k_chash_scan_top(CHash h, int32_t n_blocks) {
    __shared__ int32_t tot[1024];
    int32_t carry = 0;
    for (int32_t b0 = 0; b0 < n_blocks; b0 += 1024) {
        const int32_t b = b0 + (int32_t)threadIdx.x;
        const int32_t mine = b < n_blocks ? h.boff[b] : 0;
        tot[threadIdx.x] = mine;
        __syncthreads();
        for (int d = 1; d < 1024; d <<= 1) {
            const int32_t o = (int)threadIdx.x >= d ? tot[threadIdx.x - d] : 0;
            __syncthreads();
            tot[threadIdx.x] += o;
            __syncthreads();
        }
        if (b < n_blocks) h.boff[b] = carry + tot[threadIdx.x] - mine;
        carry += tot[1023];
        __syncthreads();
    }
}

__global__ void k_chash_scatter(DevState s, CHash h, const uint64_t* __restrict__ rank,
                                int32_t* __restrict__ members) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= s.n) return;
    const uint64_t r = rank[p];
    const int64_t t = (int64_t)(r >> 32);
    members[(int64_t)h.slot[t].start + h.boff[t / kCHashScanB] + (uint32_t)r] = (int32_t)p;
}

// Every slot's offset made global (so that in a dense grid the cells of a
// row along x are one contiguous range) and each group put in ascending
// particle index (insertion sort; a group holds a few particles).
__global__ void k_chash_order(CHash h, int32_t* __restrict__ members) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= h.H) return;
    const int32_t m = h.slot[t].cnt;
    const int32_t g0 = h.slot[t].start + h.boff[t / kCHashScanB];
    h.slot[t].start = g0;
    if (m < 2) return;
    int32_t* g = members + g0;
    for (int32_t i = 1; i < m; ++i) {
        const int32_t v = g[i];
        int32_t j = i - 1;
        while (j >= 0 && g[j] > v) {
            g[j + 1] = g[j];
            --j;
        }
        g[j + 1] = v;
    }
}

// Current position and contact radius, reference position and support
// radius of every particle, in grouped order.
__global__ void k_chash_gather(DevState s, int par, CHash h,
                               const int32_t* __restrict__ members) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= s.n) return;
    const int32_t q = members[j];
    const D4 x = s.XV[q], u = s.U[par][q];
    h.gpos[j] = D4{x.x + u.x, x.y + u.y, x.z + u.z, s.arad[q]};
    h.gref[j] = D4{x.x, x.y, x.z, s.hs[q]};
}

// Candidates of particle p: particles q != p within a_p + a_q + skin, over
// the 27 cells around p (in z, y, x order, particles by index within a
// cell); bit 31 marks a reference neighbour of the same specimen, i.e. one
// inside the support in the reference configuration (the neighbour search's
// own test, with the same arithmetic, so the mark agrees with the complete
// reference lists).  More than kContactCap candidates: flagged, the rest
// dropped.
struct CFill {
    int64_t p, np;
    double px, py, pz, ap, skin;
    D4 xp;
    int64_t first, last;
    double h2, hp;
    bool var_h;
    int cnt;
};

// Test one particle q (current position and radius g, reference position
// and support radius at gref[src]) and append it when it is a candidate.
__device__ __forceinline__ void cfill_try(const DevState& s, const CHash& h, CFill& f,
                                          int32_t q, const D4& g, int64_t src) {
    if (q == f.p) return;
    const double d0 = g.x - f.px, d1 = g.y - f.py, d2 = g.z - f.pz;
    const double rr = f.ap + g.w + f.skin;
    if (!(d0 * d0 + d1 * d1 + d2 * d2 < rr * rr)) return;
    bool ref = false;
    if (q >= f.first && q < f.last) {
        const D4 xq = h.gref[src];
        const double e0 = xq.x - f.xp.x, e1 = xq.y - f.xp.y, e2 = xq.z - f.xp.z;
        const double r2 = e0 * e0 + e1 * e1 + e2 * e2;
        double lim = f.h2;
        if (f.var_h) {
            const double hpq = 0.5 * (f.hp + xq.w);
            lim = hpq * hpq;
        }
        ref = r2 < lim;
    }
    if (f.cnt < kContactCap)
        s.ccol[(int64_t)f.cnt * f.np + f.p] = (int32_t)((uint32_t)q | (ref ? 0x80000000u : 0u));
    ++f.cnt;
}

// The 27 cells of a hashed grid: the three cells of a row along x are
// looked up together.
__device__ void cfill_hashed(const DevState& s, const CHash& h, const int32_t* members,
                             const int32_t c[3], CFill& f) {
    constexpr int32_t kAxis = 1 << kCellBits;
    for (int row = 0; row < 9; ++row) {
        const int32_t cy = c[1] + row % 3 - 1, cz = c[2] + row / 3 - 1;
        if (cy < 0 || cz < 0 || cy >= kAxis || cz >= kAxis) continue;
        uint64_t key[3];
        int64_t t[3];
        CSlot r[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int32_t cc[3] = {c[0] + k - 1, cy, cz};
            key[k] = (cc[0] >= 0 && cc[0] < kAxis) ? ccell_key(cc) : ~0ull;
            t[k] = cell_home(key[k], h.shift);
            r[k] = h.slot[t[k]];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (key[k] == ~0ull) continue;
            while (r[k].key != key[k] && r[k].key != ~0ull) {
                t[k] = (t[k] + 1) & (h.H - 1);
                r[k] = h.slot[t[k]];
            }
            if (r[k].key != key[k]) continue;
            for (int32_t i = r[k].start, e = r[k].start + r[k].cnt; i < e; ++i)
                cfill_try(s, h, f, members[i], h.gpos[i], i);
        }
    }
}

// One thread per particle.  In a dense grid the three cells of each of the
// nine rows along x are one contiguous range of the grouped list; otherwise
// the cells are looked up in the hash table.
__global__ void k_cfill(DevState s, int par, const double* __restrict__ cbox, CHash h,
                        const int32_t* __restrict__ members) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t np = s.np;
    if (p >= np) return;
    if (p >= s.n) {
        s.ccnt[p] = 0;
        return;
    }
    CFill f;
    const D4 xp = s.XV[p], up = s.U[par][p];
    f.p = p;
    f.np = np;
    f.px = xp.x + up.x;
    f.py = xp.y + up.y;
    f.pz = xp.z + up.z;
    s.ubuild[p] = up.x;
    s.ubuild[np + p] = up.y;
    s.ubuild[2 * np + p] = up.z;
    f.ap = s.arad[p];
    f.skin = s.contact_skin;
    f.xp = xp;
    const DevSpec& P = s.specs[s.spec[p]];
    f.first = P.first;
    f.last = P.last;
    f.h2 = P.h2;
    f.hp = s.hs[p];
    f.var_h = s.var_h;
    f.cnt = 0;
    int32_t c[3];
    contact_cell(cbox, f.px, f.py, f.pz, c);
    const CGrid G = cgrid(cbox);
    if (G.dense) {
        for (int a = 0; a < 3; ++a) c[a] = c[a] < G.ext[a] ? c[a] : G.ext[a] - 1;
        // the nine rows' ranges first, then each row's particles four at a
        // time (their loads issued together)
        const int32_t x0 = c[0] > 0 ? c[0] - 1 : 0;
        const int32_t x1 = c[0] + 1 < G.ext[0] ? c[0] + 1 : G.ext[0] - 1;
        int32_t j0[9], j1[9];
#pragma unroll
        for (int row = 0; row < 9; ++row) {
            const int32_t cy = c[1] + row % 3 - 1, cz = c[2] + row / 3 - 1;
            j0[row] = j1[row] = 0;
            if (cy < 0 || cz < 0 || cy >= G.ext[1] || cz >= G.ext[2]) continue;
            j0[row] = h.slot[cgrid_slot(G, x0, cy, cz)].start;
            const CSlot r1 = h.slot[cgrid_slot(G, x1, cy, cz)];
            j1[row] = r1.start + r1.cnt;
        }
        for (int row = 0; row < 9; ++row)
            for (int32_t j = j0[row]; j < j1[row]; j += 4) {
                int32_t q[4];
                D4 g[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int32_t i = j + k < j1[row] ? j + k : j;
                    q[k] = members[i];
                    g[k] = h.gpos[i];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (j + k < j1[row]) cfill_try(s, h, f, q[k], g[k], j + k);
            }
    } else {
        cfill_hashed(s, h, members, c, f);
    }
    if (f.cnt > kContactCap) {
        atomicOr(&s.err[2], kErrContact);
        f.cnt = kContactCap;
    }
    s.ccnt[p] = f.cnt;
}

// The rebuild: bounding box and cell edge, the occupied cells' hash table
// with a counting sort of the particles by cell (ranks in keys, the grouped
// list in vals, grouped positions in gpos and gref), then the lists.
hipError_t launch_contact_build(const DevState& s, int parity, uint64_t* keys, int32_t* vals,
                                const CHash& h, double* cbox, hipStream_t st) {
    k_cbox_part<<<kCBoxParts, kCBoxThreads, 0, st>>>(s, parity, cbox);
    k_cbox_final<<<1, kCBoxThreads, 0, st>>>(s, cbox, h.H);
    constexpr int T = 256;
    const unsigned gh = (unsigned)((h.H + T - 1) / T), gn = (unsigned)((s.n + T - 1) / T);
    const int32_t n_blocks = (int32_t)((h.H + kCHashScanB - 1) / kCHashScanB);
    k_chash_clear<<<gh, T, 0, st>>>(h);
    k_chash_insert<<<gn, T, 0, st>>>(s, parity, cbox, h, keys);
    k_chash_scan<<<(unsigned)n_blocks, 256, 0, st>>>(h);
    k_chash_scan_top<<<1, 1024, 0, st>>>(h, n_blocks);
    k_chash_scatter<<<gn, T, 0, st>>>(s, h, keys, vals);
    k_chash_order<<<gh, T, 0, st>>>(h, vals);
    k_chash_gather<<<gn, T, 0, st>>>(s, parity, h, vals);
    k_cfill<<<(unsigned)((s.np + T - 1) / T), T, 0, st>>>(s, parity, cbox, h, vals);
    return hipGetLastError();
}

hipError_t launch_bc_lists(const DevState& s, uint64_t* keys, int32_t* vals, int64_t m,
                           int32_t* bc_list, int64_t* bc_ptr, hipStream_t st) {
    const int T = 256;
    int64_t N = 2;
    while (N < m) N <<= 1;
    const int64_t w = N > s.n ? N : s.n;
    k_bc_keys<<<(unsigned)((w + T - 1) / T), T, 0, st>>>(s, keys, vals, m, N);
    hipError_t e = launch_bitonic_sort(keys, vals, N, st);
    if (e != hipSuccess) return e;
    const int64_t u = (m > s.n_bc + 1) ? m : s.n_bc + 1;
    k_bc_ptr<<<(unsigned)((u + T - 1) / T), T, 0, st>>>(s, keys, m, vals, bc_list, bc_ptr);
    return hipGetLastError();
}

// ===========================================================================
// run control: specimens of a batch that stop on their own
// ===========================================================================

// One block per specimen, after a step that read U[par] and wrote U[par ^ 1]:
// count the step, sum the watched group's force component in a fixed order
// (each thread a strided share of the group's list, then a tree), update the
// running peak, and stop the specimen once failed or at its cap.  A specimen
// that stops gets its new displacement copied into the other buffer too, so
// that it stays put whichever buffer later steps read.
__global__ void __launch_bounds__(256) k_run_control(DevState s, int par, RunSpec* __restrict__ run,
                                                     const int32_t* __restrict__ bc_list,
                                                     const int64_t* __restrict__ bc_ptr) {
    __shared__ double red[256];
    __shared__ int32_t why_s;
    const int sp = blockIdx.x;
    if (s.done[sp] != kRunning) return;
    RunSpec& C = run[sp];
    const int g = C.group;
    double acc = 0.0;
    if (g >= 0) {
        const double* __restrict__ f = s.force + (int64_t)C.axis * s.np;
        for (int64_t k = bc_ptr[g] + threadIdx.x; k < bc_ptr[g + 1]; k += blockDim.x)
            acc += f[bc_list[k]];
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const int64_t steps = C.steps + 1;
        C.steps = steps;
        int32_t why = kRunning;
        if (g >= 0) {
            const double r = C.sign * red[0];
            C.last = r;
            if (r > C.peak) C.peak = r;
            if (C.peak > 0.0 && C.peak >= C.min_peak && r < C.drop * C.peak) why = kStopFailed;
        }
        if (why == kRunning && C.cap > 0 && steps >= C.cap) why = kStopCap;
        why_s = why;
        if (why != kRunning) {
            s.done[sp] = why;
            atomicOr(&s.run_count[1], 1);
        }
    }
    __syncthreads();
    if (why_s == kRunning) return;
    const DevSpec& P = s.specs[sp];
    D4* __restrict__ dst = s.U[par];
    const D4* __restrict__ src = s.U[par ^ 1];
    for (int64_t i = P.first + threadIdx.x; i < P.last; i += blockDim.x) dst[i] = src[i];
}

// Append, in ascending order, the tiles of T particles (sorted order) that
// hold a running specimen's particle to `list`; returns their count (every
// thread).  Specimens are contiguous in sorted order, so a tile holds those
// from its first particle's to its last's.  One block of up to 1024 threads.
__device__ int64_t list_running_tiles(const DevState& s, int64_t n_tiles, int T,
                                      int32_t* __restrict__ list, int32_t* wave_cnt) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t base = 0;
    for (int64_t t0 = 0; t0 < n_tiles; t0 += blockDim.x) {
        const int64_t t = t0 + threadIdx.x;
        bool act = false;
        if (t < n_tiles) {
            const int64_t a = t * T;
            const int64_t b = (a + T < s.n ? a + T : s.n) - 1;
            for (int sp = s.spec[a]; sp <= s.spec[b] && !act; ++sp) act = s.done[sp] == kRunning;
        }
        const uint64_t m = __ballot(act);
        if (lane == 0) wave_cnt[wave] = __popcll(m);
        __syncthreads();
        int64_t off = base, tot = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
            off += w < wave ? wave_cnt[w] : 0;
            tot += wave_cnt[w];
        }
        if (act) list[off + __popcll(m & ((1ull << lane) - 1))] = (int32_t)t;
        base += tot;
        __syncthreads();
    }
    return base;
}

// The run-control tile lists of both passes (one when they share their
// tiles) and the number of running specimens.  One block; unless `force`, it
// returns at once when no specimen stopped since the last lists.
__global__ void __launch_bounds__(1024) k_tile_list(DevState s, int force) {
    __shared__ int32_t wave_cnt[16];
    __shared__ int32_t running;
    int32_t* __restrict__ cnt = s.run_count;
    if (!force && cnt[1] == 0) return;
    if (threadIdx.x == 0) running = 0;
    __syncthreads();
    const int64_t nb = list_running_tiles(s, (s.n + s.tile - 1) / s.tile, s.tile, s.tile_list,
                                          wave_cnt);
    int64_t na = nb;
    if (s.tile_list_a != s.tile_list)
        na = list_running_tiles(s, (s.n + s.tile_a - 1) / s.tile_a, s.tile_a, s.tile_list_a,
                                wave_cnt);
    int32_t mine = 0;
    for (int sp = threadIdx.x; sp < s.n_spec; sp += blockDim.x) mine += s.done[sp] == kRunning;
    if (mine) atomicAdd(&running, mine);
    __syncthreads();
    if (threadIdx.x == 0) {
        cnt[0] = (int32_t)nb;
        cnt[1] = 0;
        cnt[2] = running;
        cnt[3] = (int32_t)na;
    }
}

hipError_t launch_run_control(const DevState& s, int parity, RunSpec* run, const int32_t* bc_list,
                              const int64_t* bc_ptr, hipStream_t st) {
    k_run_control<<<(unsigned)s.n_spec, 256, 0, st>>>(s, parity, run, bc_list, bc_ptr);
    return hipGetLastError();
}

hipError_t launch_tile_list(const DevState& s, int force, hipStream_t st) {
    k_tile_list<<<1, 1024, 0, st>>>(s, force);
    return hipGetLastError();
}

template <int NV>
__device__ __forceinline__ void block_reduce(double (*red)[256], double v[NV], const bool is_max[NV]) {
    for (int q = 0; q < NV; ++q) red[q][threadIdx.x] = v[q];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int q = 0; q < NV; ++q)
                red[q][threadIdx.x] = is_max[q] ? fmax(red[q][threadIdx.x], red[q][threadIdx.x + w])
                                                : red[q][threadIdx.x] + red[q][threadIdx.x + w];
        __syncthreads();
    }
}

__device__ __forceinline__ int find_segment(const int64_t* seg, int n_seg, int64_t b) {
    int lo = 0, hi = n_seg;   // seg[lo] <= b < seg[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (seg[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

// One block per chunk of kDiagChunk particles of one segment.  Specimen
// partials: kinetic energy, internal energy, failed count, max D; group
// partials: force sum, displacement sum, count.
__global__ void __launch_bounds__(256) k_diag_part(DevState s, int par, const int32_t* __restrict__ list,
                                                   const int64_t* __restrict__ bc_ptr,
                                                   const int64_t* __restrict__ seg, int n_seg,
                                                   double* __restrict__ part) {
    __shared__ double red[7][256];
    const int64_t b = blockIdx.x;
    const int q = find_segment(seg, n_seg, b);
    const int64_t c = b - seg[q];
    const int64_t np = s.np;
    double* o = part + kNDiag * b;
    if (q < s.n_spec) {
        const DevSpec& P = s.specs[q];
        const int64_t beg = P.first + c * kDiagChunk;
        const int64_t end = beg + kDiagChunk < P.last ? beg + kDiagChunk : P.last;
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        for (int64_t p = beg + threadIdx.x; p < end; p += 256) {
            const double m = P.rho0 * s.XV[p].w;
            const D4 vv = s.VW[p];
            v[0] += 0.5 * m * (vv.x * vv.x + vv.y * vv.y + vv.z * vv.z);
            v[1] += m * s.e[p];
            const double D = s.D[p];
            v[2] += D >= 1.0 ? 1.0 : 0.0;
            v[3] = fmax(v[3], D);
        }
        const bool mx[4] = {false, false, false, true};
        block_reduce<4>(red, v, mx);
        if (threadIdx.x < kNDiag) o[threadIdx.x] = threadIdx.x < 4 ? red[threadIdx.x][0] : 0.0;
    } else {
        const int g = q - s.n_spec;
        const int64_t beg = bc_ptr[g] + c * kDiagChunk;
        const int64_t end = beg + kDiagChunk < bc_ptr[g + 1] ? beg + kDiagChunk : bc_ptr[g + 1];
        const D4* uc = s.U[par];
        double v[7] = {0, 0, 0, 0, 0, 0, 0};
        for (int64_t k = beg + threadIdx.x; k < end; k += 256) {
            const int64_t p = list[k];
            for (int cc = 0; cc < 3; ++cc) v[cc] += s.force[cc * np + p];
            const D4 up = uc[p];
            v[3] += up.x; v[4] += up.y; v[5] += up.z;
            v[6] += 1.0;
        }
        const bool mx[7] = {false, false, false, false, false, false, false};
        block_reduce<7>(red, v, mx);
        if (threadIdx.x < kNDiag) o[threadIdx.x] = threadIdx.x < 7 ? red[threadIdx.x][0] : 0.0;
    }
}

// One block per segment: the chunk partials in a fixed order.
__global__ void __launch_bounds__(256) k_diag_final(DevState s, const int64_t* __restrict__ seg,
                                                    const double* __restrict__ part,
                                                    double* __restrict__ spec_out,
                                                    double* __restrict__ bc_out) {
    __shared__ double red[7][256];
    const int q = blockIdx.x;
    const bool spec = q < s.n_spec;
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int64_t b = seg[q] + threadIdx.x; b < seg[q + 1]; b += 256) {
        const double* pp = part + kNDiag * b;
        for (int k = 0; k < 7; ++k) v[k] = (spec && k == 3) ? fmax(v[k], pp[k]) : v[k] + pp[k];
    }
    const bool mx_spec[7] = {false, false, false, true, false, false, false};
    const bool mx_bc[7] = {false, false, false, false, false, false, false};
    block_reduce<7>(red, v, spec ? mx_spec : mx_bc);
    if (threadIdx.x != 0) return;
    if (spec) {
        double* o = spec_out + kNDiag * q;
        o[0] = red[0][0]; o[1] = red[1][0]; o[2] = red[2][0]; o[3] = red[3][0];
        o[4] = s.t[q]; o[5] = 0.0; o[6] = 0.0; o[7] = 0.0;
    } else {
        double* o = bc_out + kNDiag * (q - s.n_spec);
        const double cnt = red[6][0];
        for (int c = 0; c < 3; ++c) {
            o[c] = red[c][0];
            o[3 + c] = cnt > 0 ? red[3 + c][0] / cnt : 0.0;
        }
        o[6] = cnt;
        o[7] = 0.0;
    }
}

// ===========================================================================
// scratch of the allocation-free diagnostics entry point
// ===========================================================================

// Chunk partials of tlsph_get_diagnostics_static: one array per device, held
// until the process ends.  Host code must not pass `scratch` itself to a
// kernel (on the host it names a stand-in, not device memory): scratch_ptr
// looks up each device's address once, with that device current.
static __device__ __align__(256) double scratch[kScratchDoubles];

hipError_t scratch_ptr(double** out) {
    constexpr int kMaxDev = 64;
    static std::mutex mu;
    static double* addr[kMaxDev] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDev) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = static_cast<double*>(p);
    }
    *out = addr[dev];
    return hipSuccess;
}

hipError_t launch_diagnostics(const DevState& s, int parity, const int32_t* bc_list,
                              const int64_t* bc_ptr, const int64_t* seg, int32_t n_seg,
                              int64_t n_chunks, double* part, double* spec_diag, double* bc_diag,
                              hipStream_t st) {
    if (n_chunks <= 0 || n_seg <= 0) return hipErrorInvalidValue;
    k_diag_part<<<(unsigned)n_chunks, 256, 0, st>>>(s, parity, bc_list, bc_ptr, seg, n_seg, part);
    k_diag_final<<<(unsigned)n_seg, 256, 0, st>>>(s, seg, part, spec_diag, bc_diag);
    return hipGetLastError();
}

}  // namespace tlsph
