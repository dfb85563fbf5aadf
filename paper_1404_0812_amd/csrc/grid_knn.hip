// Stencil gather (Sec. 4: each node and its n-1 nearest neighbours by
// Euclidean distance in R^3).  The paper builds a k-d tree (Sec. 4.1); here a
// uniform grid hash does the job on the GPU:
//   1. bounding box (two-pass reduction),
//   2. cell size ~ the expected stencil radius, cells keyed by the Morton code
//      of their integer coordinates,
//   3. counting sort of nodes by cell key (stable within a cell by node index),
//      which also yields the spatial order used by the sparse operator,
//   4. one wavefront per query: the candidates of the 27 cells around it in
//      registers, cut to few more than n - 1 by a threshold and sorted by
//      (squared distance, index); then shells of cells until the n-1-th best
//      distance is inside the searched box.
// Squared distances are ((dx*dx + dy*dy) + dz*dz) in FP64 with contraction
// disabled, so the order (and ties, broken by node index) is exact.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <vector>

#pragma clang fp contract(off)

namespace {

#ifndef KNN_CELL_SCALE
#define KNN_CELL_SCALE 1.0  // cell edge relative to the expected stencil radius
#endif
// Candidate list per query in LDS (entries; a power of two for the bitonic
// sort), for shells past the first block and blocks with more candidates than
// the registers take.  At least need + 64 = 191 for n <= 128, so that a chunk
// fits after a cut.  512 leaves room for 24 queries per CU; their registers
// allow 28.
constexpr int KNN_CAP = 512;
static_assert(KNN_CAP >= 127 + 64 && (KNN_CAP & (KNN_CAP - 1)) == 0, "candidate buffer");
constexpr int MAX_BITS = 9;    // Morton bits per axis (2^27 cells at most)

__device__ __forceinline__ uint32_t spread3(uint32_t v) {
    v &= 0x3ffu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__device__ __forceinline__ uint32_t morton3(uint32_t x, uint32_t y, uint32_t z) {
    return spread3(x) | (spread3(y) << 1) | (spread3(z) << 2);
}

struct Grid {
    double lo[3];
    double h;      // cell size
    double inv_h;
    int g[3];      // cells per axis
};

__device__ __forceinline__ int cell_coord(double x, double lo, double inv_h, int g) {
    int c = (int)floor((x - lo) * inv_h);
    return c < 0 ? 0 : (c >= g ? g - 1 : c);
}

__global__ void k_bbox_partial(int64_t N, const double* __restrict__ xyz, double* __restrict__ part) {
    __shared__ double s[6][256];
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < N;
         i += (int64_t)gridDim.x * blockDim.x) {
        for (int d = 0; d < 3; ++d) {
            double v = xyz[3 * i + d];
            mn[d] = fmin(mn[d], v);
            mx[d] = fmax(mx[d], v);
        }
    }
    for (int d = 0; d < 3; ++d) {
        s[d][threadIdx.x] = mn[d];
        s[3 + d][threadIdx.x] = mx[d];
    }
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) {
            for (int d = 0; d < 3; ++d) {
                s[d][threadIdx.x] = fmin(s[d][threadIdx.x], s[d][threadIdx.x + st]);
                s[3 + d][threadIdx.x] = fmax(s[3 + d][threadIdx.x], s[3 + d][threadIdx.x + st]);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < 6) part[blockIdx.x * 6 + threadIdx.x] = s[threadIdx.x][0];
}

// One wavefront per bound (a serial pass over 256 partials took 36 us).
__global__ __launch_bounds__(384) void k_bbox_final(int nblk, const double* __restrict__ part,
                                                    double* __restrict__ out) {
    const int d = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double v = d < 3 ? INFINITY : -INFINITY;
    for (int b = lane; b < nblk; b += 64) {
        const double p = part[b * 6 + d];
        v = d < 3 ? fmin(v, p) : fmax(v, p);
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double p = __shfl_xor(v, o, 64);
        v = d < 3 ? fmin(v, p) : fmax(v, p);
    }
    if (lane == 0) out[d] = v;
}

__global__ void k_cell_keys(int64_t N, const double* __restrict__ xyz, Grid G, uint32_t* __restrict__ key,
                            int32_t* __restrict__ count) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= N) return;
    int cx = cell_coord(xyz[3 * i + 0], G.lo[0], G.inv_h, G.g[0]);
    int cy = cell_coord(xyz[3 * i + 1], G.lo[1], G.inv_h, G.g[1]);
    int cz = cell_coord(xyz[3 * i + 2], G.lo[2], G.inv_h, G.g[2]);
    uint32_t k = morton3(cx, cy, cz);
    key[i] = k;
    atomicAdd(&count[k], 1);
}

// ---- exclusive scan of int32 counts (in place into `start`, K+1 entries) ----
constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;

// sh: SCAN_BLOCK / 64 words
__device__ int block_exclusive_scan(int v, int* sh, int* total) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) sh[wv] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < SCAN_BLOCK / 64; ++w) {
        before += w < wv ? sh[w] : 0;
        all += sh[w];
    }
    *total = all;
    __syncthreads();
    return before + incl - v;
}

__global__ void k_scan_tiles(int64_t K, const int32_t* __restrict__ in, int32_t* __restrict__ out,
                             int32_t* __restrict__ tile_sums) {
    __shared__ int sh[SCAN_BLOCK / 64];
    static_assert(SCAN_ITEMS == 8, "two vectors");
    const int64_t base = blockIdx.x * (int64_t)SCAN_TILE + threadIdx.x * SCAN_ITEMS;
    const bool whole = base + SCAN_ITEMS <= K;
    int v[SCAN_ITEMS];
    if (whole) {
        *reinterpret_cast<int4*>(v) = *reinterpret_cast<const int4*>(in + base);
        *reinterpret_cast<int4*>(v + 4) = *reinterpret_cast<const int4*>(in + base + 4);
    } else {
#pragma unroll
        for (int t = 0; t < SCAN_ITEMS; ++t) v[t] = base + t < K ? in[base + t] : 0;
    }
    int s = 0;
#pragma unroll
    for (int t = 0; t < SCAN_ITEMS; ++t) s += v[t];
    int tot;
    int ex = block_exclusive_scan(s, sh, &tot);
#pragma unroll
    for (int t = 0; t < SCAN_ITEMS; ++t) {
        const int c = v[t];
        v[t] = ex;
        ex += c;
    }
    if (whole) {
        *reinterpret_cast<int4*>(out + base) = *reinterpret_cast<const int4*>(v);
        *reinterpret_cast<int4*>(out + base + 4) = *reinterpret_cast<const int4*>(v + 4);
    } else {
#pragma unroll
        for (int t = 0; t < SCAN_ITEMS; ++t)
            if (base + t < K) out[base + t] = v[t];
    }
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

// single block: exclusive scan of the tile sums (sequential chunks of SCAN_TILE)
__global__ void k_scan_sums(int ntiles, int32_t* __restrict__ sums, int32_t* __restrict__ grand) {
    __shared__ int sh[SCAN_BLOCK / 64];
    int carry = 0;
    for (int b = 0; b < ntiles; b += SCAN_TILE) {
        const int i0 = b + (int)threadIdx.x * SCAN_ITEMS;
        int v[SCAN_ITEMS], sum = 0;
#pragma unroll
        for (int t = 0; t < SCAN_ITEMS; ++t) {
            v[t] = i0 + t < ntiles ? sums[i0 + t] : 0;
            sum += v[t];
        }
        int tot;
        int ex = block_exclusive_scan(sum, sh, &tot) + carry;
#pragma unroll
        for (int t = 0; t < SCAN_ITEMS; ++t) {
            if (i0 + t < ntiles) sums[i0 + t] = ex;
            ex += v[t];
        }
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) *grand = carry;
}

__global__ void k_scan_add(int64_t K, int32_t* __restrict__ out, const int32_t* __restrict__ sums) {
    const int64_t base = blockIdx.x * (int64_t)SCAN_TILE + threadIdx.x * SCAN_ITEMS;
    const int32_t s = sums[blockIdx.x];
    if (base + SCAN_ITEMS <= K) {
        int4* o = reinterpret_cast<int4*>(out + base);
        const int4 a = o[0], b = o[1];
        o[0] = make_int4(a.x + s, a.y + s, a.z + s, a.w + s);
        o[1] = make_int4(b.x + s, b.y + s, b.z + s, b.w + s);
    } else {
        for (int64_t i = base; i < K; ++i) out[i] += s;
    }
}

// Each node into some place of its cell; uses up the counts.
__global__ void k_scatter(int64_t N, const uint32_t* __restrict__ key, const int32_t* __restrict__ start,
                          int32_t* __restrict__ cnt, int32_t* __restrict__ placed) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= N) return;
    uint32_t k = key[i];
    placed[start[k] + atomicSub(&cnt[k], 1) - 1] = (int32_t)i;
}

// The nodes of a cell in index order: a node's place is the number of smaller
// indices in its cell (cells hold a few dozen nodes; one thread per cell
// sorting by insertion took 19 us at N = 1e5 and 45 at 1e6, and the
// coordinates another kernel).
__global__ void k_place(int64_t N, const uint32_t* __restrict__ key, const int32_t* __restrict__ start,
                        const int32_t* __restrict__ placed, const double* __restrict__ xyz,
                        int32_t* __restrict__ order, double* __restrict__ xs, double* __restrict__ ys,
                        double* __restrict__ zs) {
    int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int i = placed[p];
    const uint32_t k = key[i];
    const double x = xyz[3 * (int64_t)i], y = xyz[3 * (int64_t)i + 1], z = xyz[3 * (int64_t)i + 2];
    const int s = start[k], e = start[k + 1];
    int at = s;
#pragma unroll 4
    for (int q = s; q < e; ++q) at += placed[q] < i;
    order[at] = i;
    xs[at] = x;
    ys[at] = y;
    zs[at] = z;
}

__device__ __forceinline__ bool key_less(double da, int ia, double db, int ib) {
    return da < db || (da == db && ia < ib);
}

// v of lane ^ M in registers (DPP within 16 lanes, the row swaps above), where
// a shuffle is a trip through the LDS pipe.
template <int M>
__device__ __forceinline__ int lane_xor(int v) {
    if constexpr (M == 1) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);   // quad 1 0 3 2
    else if constexpr (M == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);  // quad 2 3 0 1
    else if constexpr (M == 4)  // mirror of 8, then of 4: 7 - (3 - ..)
        return __builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true), 0x1B, 0xf, 0xf,
                                           true);
    else if constexpr (M == 8) return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, true);  // row rotated by 8
    else if constexpr (M == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return threadIdx.x & 16 ? r[0] : r[1];
    } else {
        static_assert(M == 32, "one bit");
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return threadIdx.x & 32 ? r[0] : r[1];
    }
}
template <int M>
__device__ __forceinline__ double lane_xor(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)lane_xor<M>((int)(uint32_t)u), hi = (uint32_t)lane_xor<M>((int)(u >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// One step (pairs J apart, ascending where position & K is 0) of the sort below
// on the entry at position lane + OFF.
template <int J, int K, int OFF>
__device__ __forceinline__ void lane_exchange(double& v, int& x) {
    const double ov = lane_xor<J>(v);
    const int ox = lane_xor<J>(x);
    const int pos = threadIdx.x + OFF;
    const bool keep_max = ((pos & J) == 0) != ((pos & K) == 0);
    // equal entries (padding) may be taken either way
    const bool take = ((ov < v) | ((ov == v) & (ox < x))) != keep_max;
    v = take ? ov : v;
    x = take ? ox : x;
}
template <int J, int K>
__device__ __forceinline__ void merge64(double& v, int& x) {
    lane_exchange<J, K, 0>(v, x);
    if constexpr (J > 1) merge64<J / 2, K>(v, x);
}
// (distance, index) of the 64 lanes in ascending order
template <int K = 2>
__device__ __forceinline__ void sort64(double& v, int& x) {
    merge64<K / 2, K>(v, x);
    if constexpr (K < 64) sort64<2 * K>(v, x);
}
template <int J, int K>
__device__ __forceinline__ void merge128(double& v0, int& x0, double& v1, int& x1) {
    if constexpr (J == 64) {  // the pair (lane, lane + 64) is in one lane
        if (key_less(v1, x1, v0, x0)) {
            const double tv = v0;
            const int tx = x0;
            v0 = v1; x0 = x1;
            v1 = tv; x1 = tx;
        }
    } else {
        lane_exchange<J, K, 0>(v0, x0);
        lane_exchange<J, K, 64>(v1, x1);
    }
    if constexpr (J > 1) merge128<J / 2, K>(v0, x0, v1, x1);
}
// 128 entries, lane and lane + 64
template <int K = 2>
__device__ __forceinline__ void sort128(double& v0, int& x0, double& v1, int& x1) {
    merge128<K / 2, K>(v0, x0, v1, x1);
    if constexpr (K < 128) sort128<2 * K>(v0, x0, v1, x1);
}

template <int J, int K>
__device__ __forceinline__ void merge64(uint32_t& v) {
    const uint32_t o = (uint32_t)lane_xor<J>((int)v);
    const bool keep_max = ((threadIdx.x & J) == 0) != ((threadIdx.x & K) == 0);
    v = keep_max ? max(v, o) : min(v, o);
    if constexpr (J > 1) merge64<J / 2, K>(v);
}
template <int K = 2>
__device__ __forceinline__ void sort64(uint32_t& v) {
    merge64<K / 2, K>(v);
    if constexpr (K < 64) sort64<2 * K>(v);
}
// The first `count` (<= 64) entries sorted, distances at most `top`.  Sorts
// 26-bit steps of the distance with the lane below them, a quarter of the
// instructions of the exact sort, and puts the entries in that order; only if
// two entries share a step (or top is not a positive finite number) the exact
// sort decides.
__device__ __forceinline__ void sort_entries(double& v, int& x, int count, double top) {
    const int lane = threadIdx.x;
    const double scale = (double)((1 << 26) - 4) / top;
    uint32_t k = lane < count ? (uint32_t)(v * scale) << 6 | (uint32_t)lane : 0xffffffffu;
    sort64(k);
    const uint32_t below = (uint32_t)__shfl_up((int)k, 1, 64);
    const bool tie = lane > 0 && lane < count && (k >> 6) == (below >> 6);
    if (__ballot(tie) != 0 || !(top > 0.0 && top < 1e300 && scale < 1e300)) {
        sort64(v, x);
        return;
    }
    const double sv = __shfl(v, (int)(k & 63), 64);
    const int sx = __shfl(x, (int)(k & 63), 64);
    v = lane < count ? sv : INFINITY;
    x = lane < count ? sx : 0x7fffffff;
}

// Bitonic sort of the first S (power of two) entries of the wave's buffer, up
// to 128 of them in registers.  Entries S.. of the network are padding (+inf,
// INT_MAX) that sorts last, and only the first S are written back.
__device__ void wave_bitonic(double* d2, int* id, int S) {
    const int lane = threadIdx.x;
    if (S <= 128) {
        double v0 = lane < S ? d2[lane] : INFINITY, v1 = lane + 64 < S ? d2[lane + 64] : INFINITY;
        int x0 = lane < S ? id[lane] : 0x7fffffff, x1 = lane + 64 < S ? id[lane + 64] : 0x7fffffff;
        if (S <= 64) sort64(v0, x0);
        else sort128(v0, x0, v1, x1);
        __syncthreads();  // every lane has read its entries
        if (lane < S) {
            d2[lane] = v0;
            id[lane] = x0;
        }
        if (lane + 64 < S) {
            d2[lane + 64] = v1;
            id[lane + 64] = x1;
        }
        __syncthreads();
        return;
    }
    for (int k = 2; k <= S; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = lane; t < S; t += 64) {
                int u = t ^ j;
                if (u > t) {
                    double a = d2[t], b = d2[u];
                    int ia = id[t], ib = id[u];
                    bool up = (t & k) == 0;
                    bool sw = up ? key_less(b, ib, a, ia) : key_less(a, ia, b, ib);
                    if (sw) {
                        d2[t] = b;
                        d2[u] = a;
                        id[t] = ib;
                        id[u] = ia;
                    }
                }
            }
            __syncthreads();
        }
    }
}

__device__ __forceinline__ int next_pow2(int v) {
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

// Drop candidates that cannot be among the `need` nearest before the sort.
// Entry t belongs to group (t / 64) % NG of lane t % 64; each of the 64 NG
// groups' minimum is a distance attained by a distinct candidate, so the
// need-th smallest of those minima (need <= 64 NG) bounds the need-th smallest
// distance from above.  Entries with a larger distance are discarded (ties
// with the bound are kept) and the rest compacted to the front.  Returns the
// new count.
template <int NG>
__device__ int prefilter(double* cd, int* cid, int cnt, int need) {
    const int lane = threadIdx.x;
    double lm[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) lm[g] = INFINITY;
    for (int b = 0; b < cnt; b += 64 * NG) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int t = b + 64 * g + lane;
            if (t < cnt) lm[g] = fmin(lm[g], cd[t]);
        }
    }
    double bound = INFINITY;
    if constexpr (NG == 1) {
        // the need-th smallest of the 64 minima: bitonic sort across the lanes
        double v = lm[0];
#pragma unroll
        for (int k = 2; k <= 64; k <<= 1) {
#pragma unroll
            for (int j = k >> 1; j > 0; j >>= 1) {
                const double o = __shfl_xor(v, j, 64);
                const bool keep_min = ((lane & j) == 0) == ((lane & k) == 0);
                v = keep_min ? fmin(v, o) : fmax(v, o);
            }
        }
        bound = __shfl(v, need - 1, 64);
    } else {
        static_assert(NG == 2, "64 or 128 groups");
        // 128 minima, lm[0] and lm[1] of every lane: the same sort, two per lane
        double v0 = lm[0], v1 = lm[1];
#pragma unroll
        for (int k = 2; k <= 128; k <<= 1) {
#pragma unroll
            for (int j = k >> 1; j > 0; j >>= 1) {
                if (j == 64) {  // the pair (lane, lane + 64) is in one lane
                    const bool asc = (lane & k) == 0;
                    const double lo = fmin(v0, v1), hi = fmax(v0, v1);
                    v0 = asc ? lo : hi;
                    v1 = asc ? hi : lo;
                } else {
                    const double o0 = __shfl_xor(v0, j, 64), o1 = __shfl_xor(v1, j, 64);
                    const bool m0 = ((lane & j) == 0) == ((lane & k) == 0);
                    const bool m1 = (((lane + 64) & j) == 0) == (((lane + 64) & k) == 0);
                    v0 = m0 ? fmin(v0, o0) : fmax(v0, o0);
                    v1 = m1 ? fmin(v1, o1) : fmax(v1, o1);
                }
            }
        }
        bound = need - 1 < 64 ? __shfl(v0, need - 1, 64) : __shfl(v1, need - 1 - 64, 64);
    }
    int kept = 0;
    for (int b = 0; b < cnt; b += 64) {
        const int t = b + lane;
        double d = INFINITY;
        int id = 0;
        bool keep = false;
        if (t < cnt) {
            d = cd[t];
            id = cid[t];
            keep = d <= bound;
        }
        const uint64_t m = __ballot(keep);
        __syncthreads();  // every lane has read its entry of this block
        if (keep) {
            const int pos = kept + __popcll(m & ((1ull << lane) - 1ull));  // pos <= t: earlier blocks are done
            cd[pos] = d;
            cid[pos] = id;
        }
        kept += __popcll(m);
        __syncthreads();
    }
    return kept;
}

// d rounded up to float, as bits (d >= 0: they compare like the numbers)
__device__ __forceinline__ uint32_t round_up_bits(double d) {
    const float f = (float)d;
    return __float_as_uint(f) + ((double)f < d ? 1u : 0u);
}

// A threshold T with `need` <= count(key <= T) for keys that hold positive
// floats, and count <= limit unless equal keys forbid it.  On a surface the
// count grows about in proportion to the squared distance, so guesses follow
// the last count (two or three as a rule); after eight, bisection of the bits.
template <int NC>
__device__ __forceinline__ uint32_t select_bits(const uint32_t (&key)[NC], float guess, int need, int limit, int cnt,
                                                int& kept) {
    uint32_t lo = 0, hi = 0x7f800000u;  // the answer is in (lo, hi]
    kept = cnt;
    float t = guess;
    for (int it = 0; hi - lo > 1 && kept > limit; ++it) {
        uint32_t b = __builtin_amdgcn_readfirstlane(__float_as_uint(t));
        if (it >= 8 || b <= lo || b >= hi) b = lo + ((hi - lo) >> 1);
        int c = 0;
#pragma unroll
        for (int q = 0; q < NC; ++q) c += __popcll(__ballot(key[q] <= b));
        if (c < need) {
            lo = b;
        } else {
            hi = b;
            kept = c;
        }
        t = __uint_as_float(b) * ((0.5f * (float)(need + limit)) / (float)(c > 0 ? c : 1));
    }
    return hi;
}

template <int CTRL>
__device__ __forceinline__ int dpp_or_zero(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}

// One wavefront per query position p (spatial order; each XCD takes one
// contiguous range).  Bound by vector instructions: 950 per query at N = 1e6, n =
// 50 keep the units busy for 86 % of 1.8 ms.  The candidates of the 27 cells around the query are
// taken at once when they are at most 64 NC: keys of all of them in registers,
// a threshold that leaves few more than are needed, and only those are sorted.
// More candidates, and shells further out, go through a list in LDS.
template <int NC>
__global__ __launch_bounds__(64) void k_knn(int64_t N, int n, Grid G, const double* __restrict__ xs,
                                             const double* __restrict__ ys, const double* __restrict__ zs,
                                             const int32_t* __restrict__ order, const int32_t* __restrict__ start,
                                             int32_t* __restrict__ idx_out) {
    __shared__ double cd[KNN_CAP];
    __shared__ int cid[KNN_CAP];
    __shared__ int cstart[27], cexcl[27], delta[27];
    __shared__ uint64_t mark[NC];
    const int lane = threadIdx.x;
    const int64_t nb = gridDim.x, bx = blockIdx.x & 7, rem = nb & 7;
    const int64_t p = bx * (nb >> 3) + (bx < rem ? bx : rem) + (blockIdx.x >> 3);
    if (p >= N) return;
    const double qx = xs[p], qy = ys[p], qz = zs[p];
    const int q = order[p];
    const int cx = cell_coord(qx, G.lo[0], G.inv_h, G.g[0]);
    const int cy = cell_coord(qy, G.lo[1], G.inv_h, G.g[1]);
    const int cz = cell_coord(qz, G.lo[2], G.inv_h, G.g[2]);
    const int need = n - 1;  // neighbours besides the centre
    int cnt = 0;
    double bound = INFINITY;  // current need-th best squared distance once known
    bool done = need == 0 || qx != qx || qy != qy || qz != qz;  // a NaN is near nothing
    // One chunk of up to 64 candidates (point index j in cell order, valid
    // when in range): squared distances, those within the bound appended to
    // the LDS list; on overflow the list is cut to its best `need` first.
    auto consider = [&](int j, bool valid) {
        double d2 = INFINITY;
        int oj = -1;
        bool ok = false;
        if (valid) {
            double ddx = xs[j] - qx, ddy = ys[j] - qy, ddz = zs[j] - qz;
            d2 = (ddx * ddx + ddy * ddy) + ddz * ddz;
            oj = order[j];
            ok = (oj != q) && (d2 <= bound);
        }
        uint64_t m = __ballot(ok);
        int add = __popcll(m);
        if (add == 0) return;
        if (cnt + add > KNN_CAP) {
            // keep only the best `need` candidates
            int S = next_pow2(cnt);
            for (int t = cnt + lane; t < S; t += 64) {
                cd[t] = INFINITY;
                cid[t] = 0x7fffffff;
            }
            __syncthreads();
            wave_bitonic(cd, cid, S);
            cnt = need;
            bound = cd[need - 1];
            ok = ok && (d2 <= bound);
            m = __ballot(ok);
            add = __popcll(m);
        }
        if (ok) {
            int pos = cnt + __popcll(m & ((1ull << lane) - 1ull));
            cd[pos] = d2;
            cid[pos] = oj;
        }
        cnt += add;
        __syncthreads();
    };
    auto covers = [&](int R) {
        return (cx - R <= 0) && (cy - R <= 0) && (cz - R <= 0) && (cx + R >= G.g[0] - 1) && (cy + R >= G.g[1] - 1) &&
               (cz + R >= G.g[2] - 1);
    };
    // With the need-th best distance known: stop once the box of the shells up
    // to R provably holds the `need` nearest (or covers the whole grid).
    auto finish = [&](int R) {
        double r_safe = INFINITY;
        const double q3[3] = {qx, qy, qz};
        const int c3[3] = {cx, cy, cz};
        for (int d = 0; d < 3; ++d) {
            if (c3[d] - R > 0) r_safe = fmin(r_safe, q3[d] - (G.lo[d] + (c3[d] - R) * G.h));
            if (c3[d] + R < G.g[d] - 1) r_safe = fmin(r_safe, (G.lo[d] + (c3[d] + R + 1) * G.h) - q3[d]);
        }
        if (covers(R) || (r_safe > 0 && bound < r_safe * r_safe * (1.0 - 1e-12))) done = true;
    };
    // After the shells up to R: sort and bound.
    auto settle = [&](int R) {
        if (cnt >= need) {
            if (need <= 64 && cnt > 128) cnt = prefilter<1>(cd, cid, cnt, need);
            else if (need <= 128 && cnt > 256) cnt = prefilter<2>(cd, cid, cnt, need);
            // a second pass over the survivors (groups of one or two) usually
            // leaves at most 64 (128) to sort
            if (need <= 64 && cnt > 64) cnt = prefilter<1>(cd, cid, cnt, need);
            else if (need <= 128 && cnt > 128) cnt = prefilter<2>(cd, cid, cnt, need);
            if (cnt <= 64) {
                __syncthreads();
                double v = lane < cnt ? cd[lane] : INFINITY;
                int x = lane < cnt ? cid[lane] : 0x7fffffff;
                sort_entries(v, x, cnt, bound);  // none is above a finite bound
                __syncthreads();
                if (lane < need) {
                    cd[lane] = v;
                    cid[lane] = x;
                }
                __syncthreads();
            } else {
                int S = next_pow2(cnt);
                for (int t = cnt + lane; t < S; t += 64) {
                    cd[t] = INFINITY;
                    cid[t] = 0x7fffffff;
                }
                __syncthreads();
                wave_bitonic(cd, cid, S);
            }
            cnt = need;
            bound = cd[need - 1];
            finish(R);
        } else if (covers(R)) {
            done = true;  // only where NaN coordinates leave fewer than n nodes
        }
    };
    if (!done) {
        // R = 0 and 1 at once: the 27 cells of the 3 x 3 x 3 block, their point
        // ranges read by 27 lanes together and swept as one list (in place of
        // 27 sequential cell visits, each waiting on its range)
        int s0 = 0, c0 = 0;
        if (lane < 27) {
            const int ix = cx + lane % 3 - 1, iy = cy + (lane / 3) % 3 - 1, iz = cz + lane / 9 - 1;
            if (ix >= 0 && ix < G.g[0] && iy >= 0 && iy < G.g[1] && iz >= 0 && iz < G.g[2]) {
                const uint32_t k = morton3(ix, iy, iz);
                s0 = start[k];
                c0 = start[k + 1] - s0;
            }
        }
        // inclusive prefix sum of the counts (lanes 27.. hold none)
        int incl = c0;
        incl += dpp_or_zero<0x111>(incl);  // from 1, 2, 4 and 8 lanes below in the row of 16
        incl += dpp_or_zero<0x112>(incl);
        incl += dpp_or_zero<0x114>(incl);
        incl += dpp_or_zero<0x118>(incl);
        const int row0 = __builtin_amdgcn_readlane(incl, 15);
        if (lane & 16) incl += row0;
        const int total = __builtin_amdgcn_readlane(incl, 31), excl = incl - c0;
        // position t of the list is point t + delta[r] of the r-th cell that is
        // not empty; r follows from the bits set where the cells begin
        const uint64_t used = __ballot(c0 > 0);
        if (lane < NC) mark[lane] = 0;
        __syncthreads();
        if (c0 > 0) {
            delta[__builtin_amdgcn_mbcnt_hi((uint32_t)(used >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)used, 0))] =
                s0 - excl;
            if (excl < 64 * NC) atomicOr((unsigned long long*)&mark[excl >> 6], 1ull << (excl & 63));
        }
        __syncthreads();
        bool taken = false;
        if (total <= 64 * NC && total > need) {
            const int chunks = (total + 63) >> 6, found = total - 1, limit = need <= 64 ? 64 : 128;
            uint32_t key[NC];
            int at[NC], before = -1;
            double x[NC], y[NC], z[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (c < chunks) {
                    const uint64_t m = mark[c];
                    const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)m);
                    const uint32_t m1 = __builtin_amdgcn_readfirstlane((uint32_t)(m >> 32));
                    const uint64_t w = (uint64_t)m1 << 32 | m0, v = w >> 1;
                    // cells that begin at or before the lane's position
                    const int r = before + (int)(w & 1) +
                                  (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(v >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)v, 0));
                    before += __popcll(w);
                    const int t = 64 * c + lane;
                    at[c] = (t < total ? t : total - 1) + delta[r];
                    x[c] = xs[at[c]];
                    y[c] = ys[at[c]];
                    z[c] = zs[at[c]];
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                key[c] = 0xffffffffu;
                if (c < chunks) {
                    const double ddx = x[c] - qx, ddy = y[c] - qy, ddz = z[c] - qz;
                    const uint32_t u = round_up_bits((ddx * ddx + ddy * ddy) + ddz * ddz);
                    if (64 * c + lane < total && at[c] != (int)p) key[c] = u;
                }
            }
            int most;
            // about the area of the block over its candidates, times the number wanted
            const float guess = (float)(G.h * G.h) * (9.0f / 3.1416f) * 0.5f * (float)(need + limit) / (float)found;
            const uint32_t T = select_bits<NC>(key, guess, need, limit, found, most);
            // what is written below is what may be read: candidates at no
            // distance (a NaN coordinate) have keys above every T, so with
            // all `found` <= limit taken there can be fewer than `most`
            int kept = 0;
            if (most <= limit) {
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    if (c < chunks) {
                        const bool keep = key[c] <= T;
                        const uint64_t m = __ballot(keep);
                        if (keep)
                            cid[kept + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0))] = at[c];
                        kept += __popcll(m);
                    }
                }
                __syncthreads();
            }
            if (kept >= need) {
                taken = true;
                double v[2] = {INFINITY, INFINITY};
                int id[2] = {0x7fffffff, 0x7fffffff};
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (64 * h + lane < kept) {
                        const int j = cid[64 * h + lane];
                        const double ddx = xs[j] - qx, ddy = ys[j] - qy, ddz = zs[j] - qz;
                        v[h] = (ddx * ddx + ddy * ddy) + ddz * ddz;
                        id[h] = order[j];
                    }
                }
                if (kept <= 64) sort_entries(v[0], id[0], kept, (double)__uint_as_float(T));
                else sort128(v[0], id[0], v[1], id[1]);
                __syncthreads();
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (64 * h + lane < need) {
                        cd[64 * h + lane] = v[h];
                        cid[64 * h + lane] = id[h];
                    }
                }
                cnt = need;
                __syncthreads();
                bound = cd[need - 1];
                finish(1);
            }
        }
        if (!taken) {
            if (lane < 27) {
                cstart[lane] = s0;
                cexcl[lane] = excl;
            }
            __syncthreads();
            for (int b = 0; b < total; b += 64) {
                const int t = b + lane;
                int j = 0;
                if (t < total) {
                    int lo = 0, hi = 26;  // the cell whose exclusive prefix is the last <= t
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (cexcl[mid] <= t) lo = mid;
                        else hi = mid - 1;
                    }
                    j = cstart[lo] + (t - cexcl[lo]);
                }
                consider(j, t < total);
            }
            settle(1);
        }
    }
    for (int R = 2; !done; ++R) {
        // the shell of cells at Chebyshev distance R from the query's cell, one
        // per lane: the faces z = -R and R, then the rings between them.  Cells
        // further away than the bound are left out (distances relative to the
        // grid's origin, as the cells were assigned; slack for their rounding).
        const int side = 2 * R + 1, face = side * side, shell = 2 * face + (side - 2) * 8 * R;
        for (int b = 0; b < shell; b += 64) {
            int t = b + lane, dx, dy, dz;
            const bool in_shell = t < shell;
            if (t < 2 * face) {
                dz = t < face ? -R : R;
                t -= t < face ? 0 : face;
                dx = t % side - R;
                dy = t / side - R;
            } else {
                t -= 2 * face;
                dz = t / (8 * R) - (R - 1);
                t %= 8 * R;
                const int edge = t / (2 * R), v = t % (2 * R);
                dx = edge == 0 ? v - R : (edge == 2 ? R - v : (edge == 1 ? R : -R));
                dy = edge == 1 ? v - R : (edge == 3 ? R - v : (edge == 2 ? R : -R));
            }
            const int ix = cx + dx, iy = cy + dy, iz = cz + dz;
            int s0 = 0, c0 = 0;
            if (in_shell && ix >= 0 && ix < G.g[0] && iy >= 0 && iy < G.g[1] && iz >= 0 && iz < G.g[2]) {
                auto gap = [&](double q, double lo, int c, int g) {
                    const double u = q - lo;
                    const double d = fmax(c * G.h - u, c < g - 1 ? u - (c + 1) * G.h : 0.0) - 1e-9 * G.h;
                    return fmax(d, 0.0);
                };
                const double gx = gap(qx, G.lo[0], ix, G.g[0]), gy = gap(qy, G.lo[1], iy, G.g[1]),
                             gz = gap(qz, G.lo[2], iz, G.g[2]);
                if ((gx * gx + gy * gy + gz * gz) * (1.0 - 1e-12) <= bound) {
                    const uint32_t k = morton3(ix, iy, iz);
                    s0 = start[k];
                    c0 = start[k + 1] - s0;
                }
            }
            for (uint64_t left = __ballot(c0 > 0); left; left &= left - 1) {
                const int from = __builtin_ctzll(left);
                const int s = __builtin_amdgcn_readlane(s0, from), e = s + __builtin_amdgcn_readlane(c0, from);
                for (int a = s; a < e; a += 64) consider(a + lane, a + lane < e);
            }
        }
        settle(R);
    }
    int32_t* row = idx_out + (int64_t)q * n;
    if (lane == 0) row[0] = q;
    // short of neighbours (a node or too many others with a NaN coordinate): no index
    for (int t = lane; t < need; t += 64) row[1 + t] = t < cnt ? cid[t] : -1;
}

}  // namespace

int knn_internal(rbffd_ctx ctx, int64_t N, const double* xyz, int32_t n, int32_t* idx, int32_t* perm) {
    hipStream_t st = ctx->stream;
    const int nblk_bbox = 256;
    // bbox first (small scratch)
    int rc = ensure_scratch(ctx, nblk_bbox * 6 * sizeof(double) + 64);
    if (rc) return rc;
    double* part = (double*)ctx->scratch;
    double* bb = part + nblk_bbox * 6;
    hipLaunchKernelGGL(k_bbox_partial, dim3(nblk_bbox), dim3(256), 0, st, N, xyz, part);
    hipLaunchKernelGGL(k_bbox_final, dim3(1), dim3(384), 0, st, nblk_bbox, part, bb);
    double hb[6];
    HIP_TRY(ctx, hipMemcpyAsync(hb, bb, sizeof(hb), hipMemcpyDeviceToHost, st));
    HIP_TRY(ctx, hipStreamSynchronize(st));
    for (int d = 0; d < 6; ++d)
        if (!std::isfinite(hb[d])) return set_error(ctx, RBFFD_E_ARG, "non-finite node coordinates");
    double ext[3] = {hb[3] - hb[0], hb[4] - hb[1], hb[5] - hb[2]};
    double emax = std::max(ext[0], std::max(ext[1], ext[2]));
    if (emax <= 0) emax = 1.0;
    // surface-area proxy: half the bounding-box surface; cell ~ expected stencil radius
    double area = ext[0] * ext[1] + ext[1] * ext[2] + ext[0] * ext[2];
    if (area <= 0) area = emax * emax;
    double h = KNN_CELL_SCALE * std::sqrt(std::max(n, 8) * area / (M_PI * (double)N));
    if (!(h > 0)) h = emax;
    h = std::max(h, emax / (double)(1 << MAX_BITS));
    Grid G;
    for (int d = 0; d < 3; ++d) {
        G.lo[d] = hb[d];
        G.g[d] = std::max(1, std::min(1 << MAX_BITS, (int)std::ceil(ext[d] / h)));
    }
    // the last cell must contain the maximum coordinate
    for (int d = 0; d < 3; ++d)
        while (G.g[d] < (1 << MAX_BITS) && G.lo[d] + G.g[d] * h <= hb[3 + d]) G.g[d]++;
    G.h = h;
    G.inv_h = 1.0 / h;
    int bits = 0;
    int gmax = std::max(G.g[0], std::max(G.g[1], G.g[2]));
    while ((1 << bits) < gmax) ++bits;
    const int64_t K = (int64_t)1 << (3 * bits);
    const int64_t ntiles = (K + 1 + SCAN_TILE - 1) / SCAN_TILE;
    // scratch layout
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    size_t o_key = take(N * sizeof(uint32_t));
    size_t o_cnt = take((K + 1) * sizeof(int32_t));
    size_t o_start = take((K + 1) * sizeof(int32_t));
    size_t o_placed = take(N * sizeof(int32_t));
    size_t o_sums = take((ntiles + 1) * sizeof(int32_t));
    size_t o_order = take(N * sizeof(int32_t));
    size_t o_xs = take(N * sizeof(double));
    size_t o_ys = take(N * sizeof(double));
    size_t o_zs = take(N * sizeof(double));
    rc = ensure_scratch(ctx, off);
    if (rc) return rc;
    char* base = (char*)ctx->scratch;
    uint32_t* key = (uint32_t*)(base + o_key);
    int32_t* cnt = (int32_t*)(base + o_cnt);
    int32_t* start = (int32_t*)(base + o_start);
    int32_t* placed = (int32_t*)(base + o_placed);
    int32_t* sums = (int32_t*)(base + o_sums);
    int32_t* order = perm ? perm : (int32_t*)(base + o_order);
    double* xs = (double*)(base + o_xs);
    double* ys = (double*)(base + o_ys);
    double* zs = (double*)(base + o_zs);

    HIP_TRY(ctx, hipMemsetAsync(cnt, 0, (K + 1) * sizeof(int32_t), st));
    const int B = 256;
    int gN = (int)((N + B - 1) / B);
    hipLaunchKernelGGL(k_cell_keys, dim3(gN), dim3(B), 0, st, N, xyz, G, key, cnt);
    hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)ntiles), dim3(SCAN_BLOCK), 0, st, K + 1, cnt, start, sums);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(SCAN_BLOCK), 0, st, (int)ntiles, sums, sums + ntiles);
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)ntiles), dim3(SCAN_BLOCK), 0, st, K + 1, start, sums);
    hipLaunchKernelGGL(k_scatter, dim3(gN), dim3(B), 0, st, N, key, start, cnt, placed);
    hipLaunchKernelGGL(k_place, dim3(gN), dim3(B), 0, st, N, key, start, placed, xyz, order, xs, ys, zs);
    if (idx) {
        // the 27 cells hold about 8.6 n candidates
        const auto kernel = n <= 56 ? k_knn<8> : (n <= 84 ? k_knn<12> : k_knn<18>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)N), dim3(64), 0, st, N, n, G, xs, ys, zs, order, start, idx);
    }
    HIP_TRY(ctx, hipGetLastError());
    return RBFFD_OK;
}

extern "C" int rbffd_knn(rbffd_ctx ctx, int64_t N, const double* xyz, int32_t n, int32_t* idx, int32_t* perm) {
    if (!ctx) return RBFFD_E_ARG;
    if (N < 0 || N > 0x7fffffffLL) return set_error(ctx, RBFFD_E_ARG, "N out of range");
    if (N == 0) return RBFFD_OK;
    if (n < 1 || n > 128 || n > N) return set_error(ctx, RBFFD_E_ARG, "stencil size n=%d invalid for N=%lld", n, (long long)N);
    if (!xyz || (!idx && !perm)) return set_error(ctx, RBFFD_E_ARG, "null pointer");
    return knn_internal(ctx, N, xyz, n, idx, perm);
}
