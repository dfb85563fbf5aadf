// Sparse operator L_X and the method-of-lines time stepper (Sec. 4.2,
// eq. kernel_mol): du_s/dt = D_s L_X u_s + R_s(u), classical RK4.
//
// Layout: sliced ELL with slices of 64 rows (one wavefront), slot-major
// inside a slice: slot k of row r of a slice sits at off + 64 k + r, so the
// loads of the weights and indices of one wavefront are one contiguous run.
// Every row of a surface has exactly n entries (Sec. 4), so a slice holds no
// padding except past a surface's last row.  Rows are in the library's
// spatial order, so the gathered neighbour values are close in memory.  Many
// surfaces (each with its own N and n) form one block-diagonal operator:
// each surface starts on a fresh slice and each slice carries its own n.
// Both precisions store the n - 1 off-diagonal slots of every row in the same
// layout (FP32 and FP64 weights side by side, one index array) and read the
// neighbour values through the slice's halo staged in LDS.  FP64 state uses
// the plain form w_ii u_i + sum_{j != i} w_ij u_j (the diagonal weight kept
// per row), exact for any weights.  FP32 state uses the difference form
// sum_{j != i} w_ij (u_j - u_i) with FP32 weights; it equals L u because the
// rows of L_X sum to zero (constants are reproduced), and it keeps L 1 = 0
// exact in FP32.
//
// One RK4 stage is one kernel: it applies L to the stage input of every
// species with one read of the row, adds the reaction, and writes the next
// stage input and the RK accumulator; stage 4 writes the new state.  The
// steps are captured in a HIP graph and replayed.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <mutex>
#include <cstring>
#include <new>
#include <utility>
#include <vector>

namespace {

constexpr int BLK = 256;

// Element offset, inside a slice of `ns` slots, of slot k of lane r: the first
// 4 (ns / 4) slots go in groups of four with a lane's four slots adjacent (one
// 16-byte load per lane for FP32, two for FP64), the remaining slots one
// 64-element run each.  A slice holds 64 ns elements either way.
__host__ __device__ __forceinline__ int64_t slot_pos(int k, int ns, int r) {
    const int G = ns >> 2;
    return k < 4 * G ? 256 * (int64_t)(k >> 2) + 4 * r + (k & 3) : 256 * (int64_t)G + 64 * (int64_t)(k - 4 * G) + r;
}

// iperm[perm[p]] = p for one surface (perm nullable: identity); iperm starts
// at -1, and a perm entry outside [0, N) sets *bad instead of being written.
__global__ void k_inverse_perm(int64_t N, const int32_t* __restrict__ perm, int32_t* __restrict__ iperm,
                               int* __restrict__ bad) {
    int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int64_t v = perm ? perm[p] : p;
    if (v >= 0 && v < N) iperm[v] = (int32_t)p;
    else *bad = 1;
}

// One 256-thread block per slice of one surface: its slot entries (internal
// row indices), weights in both precisions and halo, i.e. the sorted distinct
// rows the slice's 64 rows read (off-diagonal slots) with every slot entry as
// a position in that list.  Slices with more than OP_HALO_MAX distinct rows
// keep halo = -1 and are read directly.
//
// Thread (r, q) takes slots q, q + 4, ... of row r: four lanes read 16 (index)
// or 32 (weight) bytes of a row, and the block writes 256 consecutive
// elements.  The distinct rows come from a hash table in LDS (at most
// OP_HALO_MAX + 255 entries of HB_SLOTS), are sorted (bitonic, u <= 640), and
// the table then answers where each entry sits.  At N = 2e5, n = 50 a thread
// per row (reads 200 and 400 bytes apart) took 0.76 ms and a sort of all 3136
// entries per slice 0.91 ms; this kernel takes 0.17 ms for both (waits on the
// dependent loads perm -> idx -> iperm).
//
// slice0, off0: first slice of the surface and its slot offset; row0, col0:
// its first internal and first caller row; gperm: internal row -> caller row
// (-1 on padding rows).  A stencil entry outside [0, N), or a row that perm
// does not reach, sets *bad; the slot then points at the row itself with
// weight 0 (the operator is discarded by the caller, but nothing reads out of
// bounds meanwhile).
constexpr int HB_SLOTS = 2048;
static_assert(OP_HALO_MAX + 256 < HB_SLOTS && OP_HALO_MAX <= 1024, "halo hash table");

__device__ __forceinline__ int halo_slot(int32_t j) { return (int)(((uint32_t)j * 2654435761u) >> 21); }

__global__ __launch_bounds__(256) void k_build_slices(int64_t N, int n, int64_t slice0, int64_t off0, int64_t row0,
                                                      int64_t col0, const int32_t* __restrict__ idx,
                                                      const double* __restrict__ w, const int32_t* __restrict__ perm,
                                                      const int32_t* __restrict__ iperm, OpSlice* __restrict__ slices,
                                                      double* __restrict__ wd64, double* __restrict__ w64,
                                                      int32_t* __restrict__ idx32, float* __restrict__ w32,
                                                      uint16_t* __restrict__ lidx, int32_t* __restrict__ halo,
                                                      int32_t* __restrict__ gperm, int* __restrict__ bad) {
    __shared__ int32_t key[HB_SLOTS];
    __shared__ uint16_t pos[HB_SLOTS];
    __shared__ int32_t uniq[1024];
    __shared__ int cnt;
    const int tid = threadIdx.x, r = tid >> 2, q = tid & 3;
    const int64_t sl = blockIdx.x, p = sl * 64 + r;
    const int ns = n - 1, rows = (int)(N - sl * 64 < 64 ? N - sl * 64 : 64);
    const int64_t off = off0 + sl * 64 * ns;
    for (int i = tid; i < HB_SLOTS; i += 256) key[i] = -1;
    if (tid == 0) cnt = 0;
    __syncthreads();
    const bool live = r < rows;
    int64_t i = 0;
    if (live) {
        i = perm ? perm[p] : p;
        if (i < 0 || i >= N || iperm[p] < 0) {  // out of range, or perm misses caller row p
            *bad = 1;
            i = i < 0 || i >= N ? 0 : i;
        }
        if (q == 0) {
            // slot 0 must be the row's own node: the FP32 difference form drops it
            if (idx[i * n] != i) *bad = 1;
            wd64[row0 + p] = w[i * n];
        }
    }
    if (q == 0) gperm[row0 + p] = live ? (int32_t)(col0 + i) : -1;
    for (int k = q; live && k < ns; k += 4) {
        const int32_t c = idx[i * n + 1 + k];
        const int32_t ip = (c >= 0 && c < N) ? iperm[c] : -1;
        const bool ok = ip >= 0;
        if (!ok) *bad = 1;
        const int32_t j = (int32_t)(row0 + (ok ? ip : p));
        const double wk = ok ? w[i * n + 1 + k] : 0.0;
        const int64_t at = off + slot_pos(k, ns, r);
        idx32[at] = j;
        w32[at] = (float)wk;
        w64[at] = wk;
        for (int h = halo_slot(j);; h = (h + 1) & (HB_SLOTS - 1)) {
            const int32_t old = key[h];
            if (old == j) break;
            if (old >= 0) continue;
            // a full list stops the insertions: at most one more per thread gets past this test
            if (*(volatile int*)&cnt > OP_HALO_MAX) break;
            const int32_t was = atomicCAS(&key[h], -1, j);
            if (was == j) break;
            if (was < 0) {
                const int u = atomicAdd(&cnt, 1);
                if (u < 1024) uniq[u] = j;
                break;
            }
        }
    }
    __syncthreads();
    const int u = cnt, H = u <= OP_HALO_MAX ? u : -1;
    if (tid == 0) {
        OpSlice o;
        o.off32 = off;
        o.n = n;
        o.rows = rows;
        o.halo = H;
        o.pad = 0;
        slices[slice0 + sl] = o;
    }
    if (H < 0) return;
    int S = 64;
    while (S < u) S <<= 1;
    for (int t = u + tid; t < S; t += 256) uniq[t] = 0x7fffffff;
    __syncthreads();
    for (int size = 2; size <= S; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = tid; t < S / 2; t += 256) {
                const int lo = 2 * t - (t & (stride - 1)), hi = lo + stride;  // the pair, stride apart
                const int a = uniq[lo], b = uniq[hi];
                if ((a > b) == ((lo & size) == 0)) {
                    uniq[lo] = b;
                    uniq[hi] = a;
                }
            }
            __syncthreads();
        }
    }
    for (int t = tid; t < u; t += 256) {
        const int32_t j = uniq[t];
        halo[(slice0 + sl) * OP_HALO_MAX + t] = j;
        int h = halo_slot(j);
        while (key[h] != j) h = (h + 1) & (HB_SLOTS - 1);
        pos[h] = (uint16_t)t;
    }
    __syncthreads();
    for (int k = q; live && k < ns; k += 4) {
        const int64_t at = off + slot_pos(k, ns, r);
        const int32_t j = idx32[at];  // written by this thread
        int h = halo_slot(j);
        while (key[h] != j) h = (h + 1) & (HB_SLOTS - 1);
        lidx[at] = pos[h];
    }
}

// State lives species-interleaved in internal order: element (p, s) at p*S + s,
// so that one gather fetches every species of a neighbour.
// P internal rows, N caller rows; padding rows (perm -1) hold zero.
template <typename T>
__global__ void k_load_state(int64_t P, int64_t N, int S, const double* __restrict__ in,
                             const int32_t* __restrict__ perm, T* __restrict__ out) {
    int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= P) return;
    const int64_t i = perm[p];
    for (int s = 0; s < S; ++s) out[p * S + s] = i >= 0 ? (T)in[s * N + i] : (T)0;
}

template <typename T>
__global__ void k_store_state(int64_t P, int64_t N, int S, const T* __restrict__ in, const int32_t* __restrict__ perm,
                              double* __restrict__ out) {
    int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= P) return;
    const int64_t i = perm[p];
    if (i < 0) return;
    for (int s = 0; s < S; ++s) out[s * N + i] = (double)in[p * S + s];
}

struct ReactParams {
    double p[5];
};

template <typename T, int R>
__device__ __forceinline__ void reaction(const T (&y)[2], T (&r)[2], const ReactParams& rp) {
    if (R == RBFFD_REACT_SCHNAKENBERG) {
        const T a = (T)rp.p[0], b = (T)rp.p[1], g = (T)rp.p[2];
        const T u2v = y[0] * y[0] * y[1];
        r[0] = g * (a - y[0] + u2v);
        r[1] = g * (b - u2v);
    } else if (R == RBFFD_REACT_TURING) {
        const T al = (T)rp.p[0], be = (T)rp.p[1], ga = (T)rp.p[2], t1 = (T)rp.p[3], t2 = (T)rp.p[4];
        const T u = y[0], v = y[1];
        r[0] = al * u * ((T)1 - t1 * v * v) + v * ((T)1 - t2 * u);
        r[1] = be * v * ((T)1 + al * t1 / be * u * v) + u * (ga + t2 * v);
    } else {
        r[0] = (T)0;
        r[1] = (T)0;
    }
}

struct StageArgs {
    int64_t nslices;
    const OpSlice* slices;
    const uint16_t* lidx;   // halo positions of the slot entries
    const int32_t* halo;    // halo lists (OP_HALO_MAX per slice)
    const double* wd64;     // FP64 path: diagonal weight per internal row
    double D[2];
    double dt;
    ReactParams rp;
    int* nonfinite;         // set to 1 by the last stage when a state value is not finite
    // forcing f_s(t, x_p) = exp(lam t) F[p S + s] (FORCED kernels only): the
    // stage time is t0 + (*steps_done + step_in_launch + c_stage) dt, with
    // *steps_done advanced on the device after each launch sequence
    const void* F;
    double lam, t0, toff;   // toff = (step_in_launch + c_stage), set per launch
    const int64_t* steps_done;
    int mode;               // host: the kernels to use (stage_mode)
};

// Blocks are dispatched round-robin over the 8 XCDs; remap them so that each
// XCD works on one contiguous range of rows (its L2 then holds the part of the
// gathered state those rows touch).
__device__ __forceinline__ int64_t xcd_block() {
    const int64_t nb = gridDim.x, b = blockIdx.x;
    const int64_t x = b & 7, q = nb >> 3, rem = nb & 7;
    return x * q + (x < rem ? x : rem) + (b >> 3);
}

template <typename T, int S>
struct Vec;
template <>
struct Vec<float, 1> { using type = float; };
template <>
struct Vec<float, 2> { using type = float2; };
template <>
struct Vec<double, 1> { using type = double; };
template <>
struct Vec<double, 2> { using type = double2; };

template <typename T, int S>
__device__ __forceinline__ void vload(const T* __restrict__ Y, int64_t j, T (&v)[2]) {
    if constexpr (S == 2) {
        const typename Vec<T, 2>::type t = reinterpret_cast<const typename Vec<T, 2>::type*>(Y)[j];
        v[0] = t.x;
        v[1] = t.y;
    } else {
        v[0] = Y[j];
        v[1] = (T)0;
    }
}
template <typename T, int S>
__device__ __forceinline__ void vstore(T* __restrict__ Y, int64_t j, const T (&v)[2]) {
    if constexpr (S == 2) {
        typename Vec<T, 2>::type t;
        t.x = v[0];
        t.y = v[1];
        reinterpret_cast<typename Vec<T, 2>::type*>(Y)[j] = t;
    } else {
        Y[j] = v[0];
    }
}

// Row of the calling thread: slice and lane.  B / 64 slices per block of B threads.
struct RowPos {
    int64_t p;      // internal row
    int64_t slice;  // -1: past the last slice (the whole wavefront)
    int64_t base;   // element offset of the slice's off-diagonal slots
    int lane;
    int ns;         // slots to read
    int halo;       // halo size, or -1 (direct gathers)
    bool live;
};

template <int B>
__device__ __forceinline__ RowPos row_pos(const StageArgs& a) {
    RowPos rp;
    const int64_t slice = (int64_t)xcd_block() * (B / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    rp.lane = threadIdx.x & 63;
    rp.p = slice * 64 + rp.lane;
    rp.live = false;
    rp.base = 0;
    rp.ns = 0;
    rp.halo = -1;
    rp.slice = -1;
    if (slice >= a.nslices) return rp;
    const OpSlice sl = a.slices[slice];
    rp.slice = slice;
    rp.live = rp.lane < sl.rows;
    rp.base = sl.off32;
    rp.ns = sl.n - 1;
    rp.halo = sl.halo;
    return rp;
}

typedef int i4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));

// The operator's slots are read once per stage.  KEEP: ordinary loads, which
// leave them in the caches (256 MB behind the L2s) for the next stage; else
// non-temporal ones, so that an operator which cannot stay there at least does
// not drive out the state.  STREAM_WIDE: also without reading ahead, for the
// wavefronts that fewer registers allow (stage_mode).
enum { KEEP, STREAM, STREAM_WIDE };
template <int MODE, typename V>
__device__ __forceinline__ V ld(const V* p) {
    if constexpr (MODE == KEEP) return *p;
    else return __builtin_nontemporal_load(p);
}

// four consecutive slots of one lane
template <int MODE>
__device__ __forceinline__ void load4(const int32_t* ix, const float* wx, int (&j)[4], float (&w)[4]) {
    const i4v jv = ld<MODE>(reinterpret_cast<const i4v*>(ix));
    const f4v wv = ld<MODE>(reinterpret_cast<const f4v*>(wx));
    j[0] = jv.x; j[1] = jv.y; j[2] = jv.z; j[3] = jv.w;
    w[0] = wv.x; w[1] = wv.y; w[2] = wv.z; w[3] = wv.w;
}
template <int MODE>
__device__ __forceinline__ void load4(const int32_t* ix, const double* wx, int (&j)[4], double (&w)[4]) {
    const i4v jv = ld<MODE>(reinterpret_cast<const i4v*>(ix));
    const d2v w0 = ld<MODE>(reinterpret_cast<const d2v*>(wx));
    const d2v w1 = ld<MODE>(reinterpret_cast<const d2v*>(wx) + 1);
    j[0] = jv.x; j[1] = jv.y; j[2] = jv.z; j[3] = jv.w;
    w[0] = w0.x; w[1] = w0.y; w[2] = w1.x; w[3] = w1.y;
}

template <typename T, int S>
__device__ __forceinline__ void accumulate(const T* __restrict__ Y, int j, T wk, const T (&yi)[2], T& s0, T& s1) {
    constexpr bool diff = sizeof(T) == 4;
    T y[2];
    vload<T, S>(Y, j, y);
    if (diff) {
        s0 = fma(wk, y[0] - yi[0], s0);
        if (S == 2) s1 = fma(wk, y[1] - yi[1], s1);
    } else {
        s0 = fma(wk, y[0], s0);
        if (S == 2) s1 = fma(wk, y[1], s1);
    }
}

// L applied to the stage input of row rp.p by direct gathers, in slot order.
// FP32: difference form over the n-1 off-diagonal slots; FP64: the diagonal
// term wd u_i, then the off-diagonal slots (plain form).
template <typename T, int S, int MODE>
__device__ __forceinline__ void apply_row(const RowPos& rp, const int32_t* __restrict__ idx,
                                          const T* __restrict__ w, const T* __restrict__ Y, const T (&yi)[2],
                                          T wd, T (&acc)[2]) {
    const int ns = rp.ns;
    const int G = ns >> 2;
    const int32_t* ix = idx + rp.base + 4 * rp.lane;
    const T* wx = w + rp.base + 4 * rp.lane;
    T s0 = wd * yi[0], s1 = wd * yi[1];
    int g = 0;
    for (; g + 2 <= G; g += 2) {  // eight slots in flight
        int j[8];
        T wk[8];
        load4<MODE>(ix + 256 * g, wx + 256 * g, *reinterpret_cast<int(*)[4]>(j), *reinterpret_cast<T(*)[4]>(wk));
        load4<MODE>(ix + 256 * (g + 1), wx + 256 * (g + 1), *reinterpret_cast<int(*)[4]>(j + 4),
              *reinterpret_cast<T(*)[4]>(wk + 4));
#pragma unroll
        for (int t = 0; t < 8; ++t) accumulate<T, S>(Y, j[t], wk[t], yi, s0, s1);
    }
    if (g < G) {
        int j[4];
        T wk[4];
        load4<MODE>(ix + 256 * g, wx + 256 * g, j, wk);
#pragma unroll
        for (int t = 0; t < 4; ++t) accumulate<T, S>(Y, j[t], wk[t], yi, s0, s1);
    }
    const int32_t* ir = idx + rp.base + 256 * G + rp.lane;
    const T* wr = w + rp.base + 256 * G + rp.lane;
    for (int t = 0; t < ns - 4 * G; ++t)
        accumulate<T, S>(Y, ld<MODE>(ir + 64 * t), ld<MODE>(wr + 64 * t), yi,
                         s0, s1);
    acc[0] = s0;
    acc[1] = s1;
}

typedef unsigned short u4v __attribute__((ext_vector_type(4)));

template <typename T, int S>
__device__ __forceinline__ void halo_value(const typename Vec<T, S>::type* ylds, int l, T (&y)[2]) {
    if constexpr (S == 2) {
        const typename Vec<T, 2>::type v = ylds[l];
        y[0] = v.x;
        y[1] = v.y;
    } else {
        y[0] = ylds[l];
        y[1] = (T)0;
    }
}

// four consecutive weights of one lane
template <int MODE>
__device__ __forceinline__ void loadw4(const float* wx, float (&w)[4]) {
    const f4v wv = ld<MODE>(reinterpret_cast<const f4v*>(wx));
    w[0] = wv.x; w[1] = wv.y; w[2] = wv.z; w[3] = wv.w;
}
template <int MODE>
__device__ __forceinline__ void loadw4(const double* wx, double (&w)[4]) {
    const d2v w0 = ld<MODE>(reinterpret_cast<const d2v*>(wx));
    const d2v w1 = ld<MODE>(reinterpret_cast<const d2v*>(wx) + 1);
    w[0] = w0.x; w[1] = w0.y; w[2] = w1.x; w[3] = w1.y;
}

// The n-1 off-diagonal slots with neighbour values from the staged halo, in
// slot order as apply_row.  Up to some 1e5 rows a stage is bound by its chain of
// dependent loads (slice -> halo list -> neighbour values, 0.5-0.8 us each).  So
// the first 384 entries of the halo list are read without waiting for the
// slice; neighbour values, the first sixteen slots and the tail are all in
// flight before the first of them is used; and sixteen slots are read ahead of
// those being summed.  Against reading the halo first and then sixteen slots at
// a time, 1000 FP64 steps at N = 2500, n = 31 took 20.4 -> 15.1 ms (256 entries;
// 384 take 5-10 % less from N = 1e4 to 1e5, where lists are longer than 256).
constexpr int HALO_AHEAD = 6;  // halo entries per lane
static_assert(64 * HALO_AHEAD <= OP_HALO_MAX, "halo lists are OP_HALO_MAX long");
template <typename T>
struct Slots {
    u4v l[4];
    T w[4][4];
};
// Groups past the last are read as the last: a load under a condition would
// make the compiler wait for every load after it as well.
template <typename T, int MODE>
__device__ __forceinline__ void load_slots(const uint16_t* lx, const T* wx, int g, int G, Slots<T>& b) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int at = 256 * (g + q < G ? g + q : G - 1);
        b.l[q] = ld<MODE>(reinterpret_cast<const u4v*>(lx + at));
        loadw4<MODE>(wx + at, b.w[q]);
    }
}

// Y: NV state vectors; conv() makes a neighbour's value of their entries.
template <typename T, int S, int NV, int MODE>
struct RowAhead {
    using V = typename Vec<T, S>::type;
    V y[NV][HALO_AHEAD];
    Slots<T> a;
    uint16_t lt[3];
    T wt[3];

    __device__ __forceinline__ void load(const StageArgs& arg, const RowPos& rp, const T* __restrict__ w,
                                         const T* const (&Y)[NV]) {
        if (MODE == STREAM_WIDE || rp.slice < 0) return;
        const int32_t* h = arg.halo + rp.slice * OP_HALO_MAX + rp.lane;
        int j[HALO_AHEAD];
#pragma unroll
        for (int q = 0; q < HALO_AHEAD; ++q) j[q] = h[64 * q];
        if (rp.halo < 0 || rp.ns == 0) return;
        const int G = rp.ns >> 2, tail = rp.ns & 3;
        const int64_t at = rp.base + (tail ? 256 * G : 0) + rp.lane;
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int64_t k = at + 64 * (t < tail ? t : 0);
            lt[t] = ld<MODE>(arg.lidx + k);
            wt[t] = ld<MODE>(w + k);
        }
        if (G) load_slots<T, MODE>(arg.lidx + rp.base + 4 * rp.lane, w + rp.base + 4 * rp.lane, 0, G, a);
#pragma unroll
        for (int q = 0; q < HALO_AHEAD; ++q) {
            const int64_t k = rp.lane + 64 * q < rp.halo ? j[q] : rp.p;
#pragma unroll
            for (int v = 0; v < NV; ++v) y[v][q] = reinterpret_cast<const V*>(Y[v])[k];
        }
    }
    // every lane of the wavefront; rp.halo >= 0
    template <typename C>
    __device__ __forceinline__ void finish(const StageArgs& arg, const RowPos& rp, const T* __restrict__ w,
                                           const T* const (&Y)[NV], C&& conv, V* yl, const T (&yi)[2], T wd,
                                           T (&acc)[2]) {
        constexpr int first = MODE == STREAM_WIDE ? 0 : HALO_AHEAD;
#pragma unroll
        for (int q = 0; q < first; ++q) {
            if (rp.lane + 64 * q < rp.halo) {
                V e[NV];
#pragma unroll
                for (int v = 0; v < NV; ++v) e[v] = y[v][q];
                yl[rp.lane + 64 * q] = conv(e);
            }
        }
        for (int t = rp.lane + 64 * first; t < rp.halo; t += 64) {
            const int64_t j = arg.halo[rp.slice * OP_HALO_MAX + t];
            V e[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) e[v] = reinterpret_cast<const V*>(Y[v])[j];
            yl[t] = conv(e);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (!rp.live) return;
        constexpr bool diff = sizeof(T) == 4;
        T s0 = wd * yi[0], s1 = wd * yi[1];
        auto acc1 = [&](int l, T wk) {
            T n[2];
            halo_value<T, S>(yl, l, n);
            s0 = fma(wk, diff ? n[0] - yi[0] : n[0], s0);
            if (S == 2) s1 = fma(wk, diff ? n[1] - yi[1] : n[1], s1);
        };
        const int G = rp.ns >> 2, tail = rp.ns & 3;
        auto sum = [&](const Slots<T>& b, int groups) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q < groups) {
                    acc1(b.l[q].x, b.w[q][0]);
                    acc1(b.l[q].y, b.w[q][1]);
                    acc1(b.l[q].z, b.w[q][2]);
                    acc1(b.l[q].w, b.w[q][3]);
                }
            }
        };
        const uint16_t* lx = arg.lidx + rp.base + 4 * rp.lane;
        const T* wx = w + rp.base + 4 * rp.lane;
        int g = 0;
        if constexpr (MODE == STREAM_WIDE) {
            for (; g + 4 <= G; g += 4) {
                load_slots<T, MODE>(lx, wx, g, G, a);
                sum(a, 4);
            }
            if (g < G) {
                load_slots<T, MODE>(lx, wx, g, G, a);
                sum(a, G - g);
            }
            const int64_t at = rp.base + 256 * G + rp.lane;
            for (int t = 0; t < tail; ++t) acc1(ld<MODE>(arg.lidx + at + 64 * t), ld<MODE>(w + at + 64 * t));
            acc[0] = s0;
            acc[1] = s1;
            return;
        }
        Slots<T> b;
        while (g + 8 < G) {
            load_slots<T, MODE>(lx, wx, g + 4, G, b);
            sum(a, 4);
            load_slots<T, MODE>(lx, wx, g + 8, G, a);
            sum(b, 4);
            g += 8;
        }
        if (g + 4 < G) {
            load_slots<T, MODE>(lx, wx, g + 4, G, b);
            sum(a, 4);
            sum(b, G - g - 4);
        } else {
            sum(a, G - g);
        }
#pragma unroll
        for (int t = 0; t < 3; ++t)
            if (t < tail) acc1(lt[t], wt[t]);
        acc[0] = s0;
        acc[1] = s1;
    }
};

// L applied to the stage input of row rp.p: through the staged halo when the
// slice has one, otherwise by direct gathers.  Every lane of the wavefront
// must call this (the halo is loaded cooperatively).
template <typename T, int S, int MODE>
__device__ __forceinline__ void laplacian_row(const StageArgs& a, const RowPos& rp, const int32_t* __restrict__ idx,
                                              const T* __restrict__ w, const T* __restrict__ Y, const T (&yi)[2],
                                              T (&lap)[2]) {
    using V = typename Vec<T, S>::type;
    __shared__ V ylds[OP_HALO_MAX];
    const T* const ys[1] = {Y};
    RowAhead<T, S, 1, MODE> ahead;
    ahead.load(a, rp, w, ys);
    T wd = (T)0;
    if constexpr (sizeof(T) == 8) {
        if (rp.live) wd = ld<MODE>(a.wd64 + rp.p);
    }
    if (rp.halo >= 0) {
        ahead.finish(a, rp, w, ys, [](const V (&e)[1]) { return e[0]; }, ylds, yi, wd, lap);
        return;
    }
    if (rp.live) apply_row<T, S, MODE>(rp, idx, w, Y, yi, wd, lap);
}

// RK4 stage `ST` (0..3), one wavefront per block: blocks of four, on a quarter
// of the CUs, took 6.05 instead of 5.39 ms for 400 FP64 steps at N = 2500 and
// 6.98 instead of 6.16 at N = 10242, two species; the same from N = 1e5 on.
//  Y: stage input; U: state at the start of the step;
// ACC: accumulator; YN: next stage input (stages 0-2) -- stage 3 updates U
// (FP32: YN is then the compensation term of the update).
template <typename T, int S, int R, int ST, bool FORCED, int MODE>
__global__ __launch_bounds__(64) void k_rk4_stage(StageArgs a, const int32_t* __restrict__ idx,
                                                   const T* __restrict__ w, const T* __restrict__ Y,
                                                   T* __restrict__ U, T* __restrict__ ACC, T* __restrict__ YN) {
    const RowPos rp = row_pos<64>(a);
    if (rp.slice < 0) return;  // the whole wavefront
    const int64_t p = rp.p;
    T yi[2] = {0, 0}, u[2], c[2], e[2], f[2], o[2];
    if (rp.live) {  // all that the row needs, before its neighbours are waited for
        vload<T, S>(Y, p, yi);
        vload<T, S>(U, p, u);
        if constexpr (ST > 0) vload<T, S>(ACC, p, c);
        if constexpr (ST == 3 && sizeof(T) == 4) vload<T, S>(YN, p, e);
        if constexpr (FORCED) vload<T, S>(reinterpret_cast<const T*>(a.F), p, f);
    }
    T lap[2];
    laplacian_row<T, S, MODE>(a, rp, idx, w, Y, yi, lap);
    if (!rp.live) return;
    T r[2];
    reaction<T, R>(yi, r, a.rp);
    T k[2];
    k[0] = (T)a.D[0] * lap[0] + r[0];
    k[1] = (T)a.D[1] * lap[1] + r[1];
    if constexpr (FORCED) {
        const double t = a.t0 + ((double)*a.steps_done + a.toff) * a.dt;  // uniform
        const T ef = (T)exp(a.lam * t);
        k[0] = fma(ef, f[0], k[0]);
        k[1] = fma(ef, f[1], k[1]);
    }
    const T dt = (T)a.dt;
    if (ST == 0) {
        o[0] = u[0] + (T)0.5 * dt * k[0];
        o[1] = u[1] + (T)0.5 * dt * k[1];
        vstore<T, S>(ACC, p, k);
        vstore<T, S>(YN, p, o);
    } else if (ST == 1 || ST == 2) {
        const T h = ST == 1 ? (T)0.5 * dt : dt;
        o[0] = u[0] + h * k[0];
        o[1] = u[1] + h * k[1];
        c[0] = c[0] + (T)2 * k[0];
        c[1] = c[1] + (T)2 * k[1];
        vstore<T, S>(ACC, p, c);
        vstore<T, S>(YN, p, o);
    } else {
        if constexpr (sizeof(T) == 4) {
            // FP32 state: compensated (Kahan) update, the running rounding error
            // kept in YN; over 1e4 steps of increments ~1e-4 of the state the
            // plain update drifts by several 1e-5 against FP64
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const T d = dt / (T)6 * (c[q] + k[q]) - e[q];
                const T t = u[q] + d;
                e[q] = (t - u[q]) - d;
                o[q] = t;
            }
            vstore<T, S>(U, p, o);
            vstore<T, S>(YN, p, e);
        } else {
            o[0] = u[0] + dt / (T)6 * (c[0] + k[0]);
            o[1] = u[1] + dt / (T)6 * (c[1] + k[1]);
            vstore<T, S>(U, p, o);
        }
        if (!(isfinite(o[0]) && isfinite(o[1]))) *a.nonfinite = 1;  // every writer stores 1
    }
}

// Device-side step counter of the forced stages, advanced after each launch sequence.
__global__ void k_advance_steps(int64_t* steps_done, int64_t by) { *steps_done += by; }
__global__ void k_set_steps(int64_t* steps_done, int* nonfinite) {
    *steps_done = 0;
    *nonfinite = 0;
}

// one operator application (stage-free): out = L y (reaction-free, D = 1)
template <typename T, int MODE>
__global__ __launch_bounds__(64) void k_apply(StageArgs a, const int32_t* __restrict__ idx, const T* __restrict__ w,
                                               const T* __restrict__ Y, T* __restrict__ out) {
    const RowPos rp = row_pos<64>(a);
    if (rp.slice < 0) return;  // the whole wavefront
    T yi[2] = {0, 0};
    if (rp.live) vload<T, 1>(Y, rp.p, yi);
    T lap[2];
    laplacian_row<T, 1, MODE>(a, rp, idx, w, Y, yi, lap);
    if (rp.live) out[rp.p] = lap[0];
}

// KEEP up to about what the 256 MB cache holds: (slot + index) bytes against
// non-temporal loads, 40 steps each.  FP32: 59 MB 2.38 -> 2.22 ms, 176 MB
// 6.21 -> 5.17, 235 MB 8.06 -> 6.91, 265 MB 9.11 -> 8.59, but 294 MB 9.87 ->
// 10.64, 588 MB 17.6 -> 19.8.  FP64 moves more besides the slots and loses
// later: 49 MB 2.73 -> 2.18 ms, 210 MB 8.32 -> 5.99, 294 MB 11.8 -> 10.8, 490 MB
// 18.5 -> 18.2, 600 MB 24.2 -> 24.5.
// Above that, reading ahead pays for FP32 up to n = 64 (N = 1e6, n = 50: 1-2 %)
// and costs FP32 3 % at n = 101 and FP64 up to 8 % (N = 1e6, n = 70: 22.8 -> 24.6
// ms): more registers, fewer wavefronts, on a launch that memory bounds.
template <typename T>
int stage_mode(int64_t slots, int n) {
    if (slots * (int64_t)(sizeof(T) + sizeof(uint16_t)) <= (int64_t)(sizeof(T) == 4 ? 256 : 512) << 20) return KEEP;
    return sizeof(T) == 4 && n <= 64 ? STREAM : STREAM_WIDE;
}

StageArgs stage_args(rbffd_op op, bool f64) {
    StageArgs a;
    std::memset(&a, 0, sizeof(a));
    a.nslices = op->nslices;
    a.slices = op->slices;
    a.lidx = op->lidx;
    a.halo = op->halo;
    a.wd64 = op->wd64;
    a.mode = f64 ? stage_mode<double>(op->slots, op->n) : stage_mode<float>(op->slots, op->n);
    return a;
}

// Blocks of a stage launch: one slice each.
inline dim3 stage_grid(int64_t nslices) { return dim3((unsigned)nslices); }

// One RK4 step, the i-th of its launch sequence; stage times t_n + c dt with
// c = 0, 1/2, 1/2, 1.
template <typename T, int S, int R, bool FORCED, int MODE>
void enqueue_step(hipStream_t st, StageArgs a, int64_t i, const int32_t* idx, const T* w, T* U, T* ACC, T* Y1,
                  T* Y2, T* COMP) {
    const dim3 g = stage_grid(a.nslices), b(64);
    a.toff = (double)i;
    hipLaunchKernelGGL((k_rk4_stage<T, S, R, 0, FORCED, MODE>), g, b, 0, st, a, idx, w, U, U, ACC, Y1);
    a.toff = (double)i + 0.5;
    hipLaunchKernelGGL((k_rk4_stage<T, S, R, 1, FORCED, MODE>), g, b, 0, st, a, idx, w, Y1, U, ACC, Y2);
    hipLaunchKernelGGL((k_rk4_stage<T, S, R, 2, FORCED, MODE>), g, b, 0, st, a, idx, w, Y2, U, ACC, Y1);
    a.toff = (double)i + 1.0;
    hipLaunchKernelGGL((k_rk4_stage<T, S, R, 3, FORCED, MODE>), g, b, 0, st, a, idx, w, Y1, U, ACC, COMP);
}

template <typename T, bool FORCED, int MODE>
void enqueue_steps_f(hipStream_t st, int S, int R, const StageArgs& a, const int32_t* idx, const T* w, T* U, T* ACC,
                     T* COMP, T* Y1, T* Y2, int64_t steps) {
    for (int64_t i = 0; i < steps; ++i) {
        if (S == 1) {
            enqueue_step<T, 1, RBFFD_REACT_NONE, FORCED, MODE>(st, a, i, idx, w, U, ACC, Y1, Y2, COMP);
        } else if (R == RBFFD_REACT_SCHNAKENBERG) {
            enqueue_step<T, 2, RBFFD_REACT_SCHNAKENBERG, FORCED, MODE>(st, a, i, idx, w, U, ACC, Y1, Y2, COMP);
        } else if (R == RBFFD_REACT_TURING) {
            enqueue_step<T, 2, RBFFD_REACT_TURING, FORCED, MODE>(st, a, i, idx, w, U, ACC, Y1, Y2, COMP);
        } else {
            enqueue_step<T, 2, RBFFD_REACT_NONE, FORCED, MODE>(st, a, i, idx, w, U, ACC, Y1, Y2, COMP);
        }
    }
    // forced stages read the step counter: advance it past this sequence
    if (FORCED) hipLaunchKernelGGL(k_advance_steps, dim3(1), dim3(1), 0, st, const_cast<int64_t*>(a.steps_done), steps);
}

template <typename T, int MODE>
void enqueue_steps_m(hipStream_t st, int S, int R, const StageArgs& a, const int32_t* idx, const T* w, T* U, T* ACC,
                     T* COMP, T* Y1, T* Y2, int64_t steps) {
    if (a.F) enqueue_steps_f<T, true, MODE>(st, S, R, a, idx, w, U, ACC, COMP, Y1, Y2, steps);
    else enqueue_steps_f<T, false, MODE>(st, S, R, a, idx, w, U, ACC, COMP, Y1, Y2, steps);
}

template <typename T>
void enqueue_steps_t(hipStream_t st, int S, int R, const StageArgs& a, const int32_t* idx, const T* w, T* U, T* ACC,
                     T* COMP, T* Y1, T* Y2, int64_t steps) {
    if (a.mode == KEEP) enqueue_steps_m<T, KEEP>(st, S, R, a, idx, w, U, ACC, COMP, Y1, Y2, steps);
    else if (sizeof(T) == 4 && a.mode == STREAM)
        enqueue_steps_m<T, sizeof(T) == 4 ? STREAM : KEEP>(st, S, R, a, idx, w, U, ACC, COMP, Y1, Y2, steps);
    else enqueue_steps_m<T, STREAM_WIDE>(st, S, R, a, idx, w, U, ACC, COMP, Y1, Y2, steps);
}

template <typename T>
void enqueue_apply(hipStream_t st, const StageArgs& a, const int32_t* idx, const T* w, const T* Y, T* out) {
    const dim3 g = stage_grid(a.nslices), b(64);
    if (a.mode == KEEP) hipLaunchKernelGGL((k_apply<T, KEEP>), g, b, 0, st, a, idx, w, Y, out);
    else hipLaunchKernelGGL((k_apply<T, STREAM_WIDE>), g, b, 0, st, a, idx, w, Y, out);
}

// The flag of the stepper's last stage on the host side, allocated on first use.
int ensure_flag(rbffd_op op) {
    if (op->nonfinite_host) return RBFFD_OK;
    if (hipHostMalloc(reinterpret_cast<void**>(&op->nonfinite_host), sizeof(int), hipHostMallocDefault) != hipSuccess) {
        op->nonfinite_host = nullptr;
        return set_error(op->ctx, RBFFD_E_NOMEM, "cannot allocate the host flag");
    }
    return RBFFD_OK;
}

void reset_graph(rbffd_op op) {
    if (op->graph) {
        (void)hipGraphExecDestroy(op->graph);
        op->graph = nullptr;
    }
    op->graph_key_species = -1;
}

void reset_kgraph(rbffd_op op) {
    if (op->kgraph) {
        (void)hipGraphExecDestroy(op->kgraph);
        op->kgraph = nullptr;
    }
    op->kgraph_key = nullptr;
}

// The state workspace: 4 state buffers (U, ACC, Y1, Y2) x 2 species x FP64, and
// the forcing (2 species).
int ensure_work(rbffd_op op) {
    if (op->work.p) return RBFFD_OK;
    const size_t need = 5 * 2 * (size_t)op->P * sizeof(double);
    if (spare_take(op->spare, need, op->work)) return RBFFD_OK;
    return set_error(op->ctx, RBFFD_E_NOMEM, "cannot allocate %zu bytes of state", need);
}

// Build the sliced operator of nsurf surfaces (validated by the callers).  All
// device arrays of the operator but the state workspace are one allocation; the
// inverse permutation is in the context's scratch.  Build, two FP64
// applications and release at N = 2e5, n = 50: 2.9 -> 0.43 ms with the memory of
// an operator destroyed before (also one used on a second context), 3.6 -> 1.3 ms
// for the first of a context and 6.1 -> 1.1 ms for two alive at once, where
// hipMalloc and hipFree add 0.25 ms for each of 64 MB to 1 GB, 0.5 ms above; four
// operators of growing size 11.7 -> 3.5 ms.
int create_op(rbffd_ctx ctx, int nsurf, const rbffd_op_surface* surf, rbffd_op* out) {
    int64_t P = 0, N = 0, slots = 0, maxN = 0, nslices = 0;
    int32_t nmax = 0;
    for (int s = 0; s < nsurf; ++s) {
        const int64_t sl = (surf[s].N + 63) / 64;
        nslices += sl;
        slots += 64 * sl * (surf[s].n - 1);
        P += 64 * sl;
        N += surf[s].N;
        maxN = std::max(maxN, surf[s].N);
        nmax = std::max(nmax, surf[s].n);
    }
    if (P > 0x7fffffffLL) return set_error(ctx, RBFFD_E_ARG, "operator too large: %lld rows", (long long)P);
    int rc = ensure_scratch(ctx, (size_t)maxN * sizeof(int32_t) + 512);
    if (rc) return rc;
    int* bad = (int*)ctx->scratch;
    int32_t* iperm = (int32_t*)((char*)ctx->scratch + 256);
    rbffd_op op = new (std::nothrow) rbffd_op_s();
    if (!op) return set_error(ctx, RBFFD_E_NOMEM, "host allocation failed");
    op->ctx = ctx;
    op->spare = ctx->spare;
    {
        std::lock_guard<std::mutex> lock(op->spare->mu);
        ++op->spare->owners;
    }
    op->N = N;
    op->P = P;
    op->n = nmax;
    op->nsurf = nsurf;
    op->nslices = nslices;
    op->slots = slots;
    size_t bytes = 0;
    auto take = [&](size_t b) {
        const size_t o = bytes;
        bytes += (b + 255) & ~(size_t)255;
        return o;
    };
    const size_t o_sl = take(nslices * sizeof(OpSlice)), o_wd = take(P * sizeof(double));
    const size_t o_w64 = take(slots * sizeof(double)), o_idx = take(slots * sizeof(int32_t));
    const size_t o_w32 = take(slots * sizeof(float)), o_lidx = take(slots * sizeof(uint16_t));
    const size_t o_halo = take(nslices * OP_HALO_MAX * sizeof(int32_t)), o_perm = take(P * sizeof(int32_t));
    const size_t o_cnt = take(sizeof(int64_t) + sizeof(int));
    if (!spare_take(op->spare, bytes, op->slab)) {
        rbffd_op_destroy(op);
        return set_error(ctx, RBFFD_E_NOMEM, "operator allocation failed");
    }
    char* base = (char*)op->slab.p;
    op->slices = (OpSlice*)(base + o_sl);
    op->wd64 = (double*)(base + o_wd);
    op->w64 = (double*)(base + o_w64);
    op->idx32 = (int32_t*)(base + o_idx);
    op->w32 = (float*)(base + o_w32);
    op->lidx = (uint16_t*)(base + o_lidx);
    op->halo = (int32_t*)(base + o_halo);
    op->perm = (int32_t*)(base + o_perm);
    op->counters = base + o_cnt;
    hipStream_t st = ctx->stream;
    hipError_t e = hipMemsetAsync(bad, 0, sizeof(int), st);
    int64_t slice0 = 0, off0 = 0, col0 = 0;
    for (int s = 0; s < nsurf && e == hipSuccess; ++s) {
        const int64_t Ns = surf[s].N, sl = (Ns + 63) / 64;
        const dim3 g((unsigned)((Ns + BLK - 1) / BLK)), b(BLK);
        e = hipMemsetAsync(iperm, 0xff, (size_t)Ns * sizeof(int32_t), st);
        if (e != hipSuccess) break;
        hipLaunchKernelGGL(k_inverse_perm, g, b, 0, st, Ns, surf[s].perm, iperm, bad);
        hipLaunchKernelGGL(k_build_slices, dim3((unsigned)sl), dim3(256), 0, st, Ns, surf[s].n, slice0, off0,
                           64 * slice0, col0, surf[s].idx, surf[s].w, surf[s].perm, iperm, op->slices, op->wd64, op->w64,
                           op->idx32, op->w32, op->lidx, op->halo, op->perm, bad);
        e = hipGetLastError();
        slice0 += sl;
        off0 += 64 * sl * (surf[s].n - 1);
        col0 += Ns;
    }
    int bad_h = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&bad_h, bad, sizeof(int), hipMemcpyDeviceToHost, st);
    const hipError_t e2 = hipStreamSynchronize(st);
    if (e == hipSuccess) e = e2;
    if (e != hipSuccess) {
        rbffd_op_destroy(op);
        return set_error(ctx, RBFFD_E_HIP, "operator build failed: %s", hipGetErrorString(e));
    }
    if (bad_h) {
        rbffd_op_destroy(op);
        return set_error(ctx, RBFFD_E_ARG, "stencil or perm entry outside [0, N) (or perm not a permutation)");
    }
    *out = op;
    return RBFFD_OK;
}

int check_surface(rbffd_ctx ctx, int s, const rbffd_op_surface& d) {
    if (d.N <= 0 || d.N > 0x7fffffffLL) return set_error(ctx, RBFFD_E_ARG, "surface %d: N out of range", s);
    if (d.n < 2 || d.n > 128 || d.n > d.N)
        return set_error(ctx, RBFFD_E_ARG, "surface %d: stencil size n=%d invalid", s, d.n);
    if (!d.idx || !d.w) return set_error(ctx, RBFFD_E_ARG, "surface %d: null pointer", s);
    return RBFFD_OK;
}

}  // namespace

extern "C" int rbffd_op_create(rbffd_ctx ctx, int64_t N, int32_t n, const int32_t* idx, const double* w,
                               const int32_t* perm, rbffd_op* out) {
    if (!ctx || !out) return RBFFD_E_ARG;
    rbffd_op_surface d;
    d.N = N;
    d.n = n;
    d.reserved = 0;
    d.idx = idx;
    d.w = w;
    d.perm = perm;
    if (N <= 0 || N > 0x7fffffffLL) return set_error(ctx, RBFFD_E_ARG, "N out of range");
    if (n < 2 || n > 128 || n > N) return set_error(ctx, RBFFD_E_ARG, "stencil size n=%d invalid", n);
    if (!idx || !w) return set_error(ctx, RBFFD_E_ARG, "null pointer");
    return create_op(ctx, 1, &d, out);
}

extern "C" int rbffd_op_create_batched(rbffd_ctx ctx, int32_t nsurf, const rbffd_op_surface* surf, rbffd_op* out) {
    if (!ctx || !out) return RBFFD_E_ARG;
    if (nsurf < 1 || !surf) return set_error(ctx, RBFFD_E_ARG, "need at least one surface");
    for (int s = 0; s < nsurf; ++s) {
        int rc = check_surface(ctx, s, surf[s]);
        if (rc) return rc;
    }
    return create_op(ctx, nsurf, surf, out);
}

// The whole device is waited for, as by the hipFree of memory that is not kept:
// the operator may have been used on other contexts' streams, or recorded in a
// graph that the caller launched on a stream of its own.
extern "C" int rbffd_op_destroy(rbffd_op op) {
    if (!op) return RBFFD_E_ARG;
    int dev = op->spare->device;
    (void)hipGetDevice(&dev);
    if (dev != op->spare->device) (void)hipSetDevice(op->spare->device);
    const bool idle = hipDeviceSynchronize() == hipSuccess;
    reset_graph(op);
    reset_kgraph(op);
    const SpareMemory::Block blocks[2] = {op->slab, op->work};
    spare_give(op->spare, blocks, idle);
    if (op->impl) (void)hipFree(op->impl);
    if (op->nonfinite_host) (void)hipHostFree(op->nonfinite_host);
    if (dev != op->spare->device) (void)hipSetDevice(dev);
    spare_leave(op->spare, false);
    delete op;
    return RBFFD_OK;
}

extern "C" int rbffd_op_stats(rbffd_op op, int64_t* nslices, int64_t* halo_slices, int64_t* halo_rows,
                              int64_t* halo_entries) {
    if (!op) return RBFFD_E_ARG;
    std::vector<OpSlice> sl((size_t)op->nslices);
    if (!sl.empty()) {
        HIP_TRY(op->ctx, hipStreamSynchronize(op->ctx->stream));
        HIP_TRY(op->ctx, hipMemcpy(sl.data(), op->slices, sl.size() * sizeof(OpSlice), hipMemcpyDeviceToHost));
    }
    int64_t hs = 0, hr = 0, he = 0;
    for (const OpSlice& o : sl)
        if (o.halo >= 0) {
            ++hs;
            hr += o.rows;
            he += o.halo;
        }
    if (nslices) *nslices = op->nslices;
    if (halo_slices) *halo_slices = hs;
    if (halo_rows) *halo_rows = hr;
    if (halo_entries) *halo_entries = he;
    return RBFFD_OK;
}

// ------------------------------------------------------------------------
// Allocation-free operator application.  The internal-order input and output
// vectors live in one fixed device array per GPU (RBFFD_NOALLOC_SCRATCH_BYTES),
// whose device address is looked up once per device when a context is
// created there.  The array's name is a host-side stand-in in host code: only
// the looked-up pointer is ever passed to kernels.
static __device__ __align__(256) unsigned char scratch[RBFFD_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES] = {};
}  // namespace

// Called by rbffd_create with `device` current.
int noalloc_scratch_setup(rbffd_ctx ctx, int device) {
    if (device < 0 || device >= MAX_DEVICES) return set_error(ctx, RBFFD_E_UNSUPPORTED, "device index %d", device);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return RBFFD_OK;
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
        return set_error(ctx, RBFFD_E_HIP, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
    g_scratch_ptr[device] = ptr;
    return RBFFD_OK;
}

extern "C" int rbffd_apply_noalloc(rbffd_ctx ctx, rbffd_op op, int32_t prec, const double* u, double* Lu) {
    if (!ctx || !op || !u || !Lu) return set_error(ctx, RBFFD_E_ARG, "null argument");
    if (prec != RBFFD_F64 && prec != RBFFD_F32) return set_error(ctx, RBFFD_E_ARG, "prec must be F64 or F32");
    const int64_t N = op->N, P = op->P;
    const size_t need = 2 * (size_t)P * (prec == RBFFD_F64 ? sizeof(double) : sizeof(float));
    if (need > (size_t)RBFFD_NOALLOC_SCRATCH_BYTES)
        return set_error(ctx, RBFFD_E_UNSUPPORTED, "operator of %lld padded rows needs %zu bytes of scratch, above the "
                         "%d-byte array of the allocation-free call", (long long)P, need, RBFFD_NOALLOC_SCRATCH_BYTES);
    void* base = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (ctx->device >= 0 && ctx->device < MAX_DEVICES) base = g_scratch_ptr[ctx->device];
    }
    if (!base) return set_error(ctx, RBFFD_E_HIP, "no scratch address for device %d", ctx->device);
    hipStream_t st = ctx->stream;
    const dim3 g((unsigned)((P + BLK - 1) / BLK)), b(BLK);
    StageArgs a = stage_args(op, prec == RBFFD_F64);
    if (prec == RBFFD_F64) {
        double* Y = (double*)base;
        double* out = Y + P;
        hipLaunchKernelGGL(k_load_state<double>, g, b, 0, st, P, N, 1, u, op->perm, Y);
        enqueue_apply<double>(st, a, op->idx32, op->w64, Y, out);
        hipLaunchKernelGGL(k_store_state<double>, g, b, 0, st, P, N, 1, out, op->perm, Lu);
    } else {
        float* Y = (float*)base;
        float* out = Y + P;
        hipLaunchKernelGGL(k_load_state<float>, g, b, 0, st, P, N, 1, u, op->perm, Y);
        enqueue_apply<float>(st, a, op->idx32, op->w32, Y, out);
        hipLaunchKernelGGL(k_store_state<float>, g, b, 0, st, P, N, 1, out, op->perm, Lu);
    }
    HIP_TRY(ctx, hipGetLastError());
    return RBFFD_OK;
}

extern "C" int rbffd_apply(rbffd_ctx ctx, rbffd_op op, int32_t prec, const double* u, double* Lu) {
    if (!ctx || !op || !u || !Lu) return set_error(ctx, RBFFD_E_ARG, "null argument");
    if (prec != RBFFD_F64 && prec != RBFFD_F32) return set_error(ctx, RBFFD_E_ARG, "prec must be F64 or F32");
    op->ctx = ctx;
    const int rc = ensure_work(op);
    if (rc) return rc;
    hipStream_t st = ctx->stream;
    const int64_t N = op->N, P = op->P;
    const dim3 g((unsigned)((P + BLK - 1) / BLK)), b(BLK);
    StageArgs a = stage_args(op, prec == RBFFD_F64);
    if (prec == RBFFD_F64) {
        double* Y = (double*)op->work.p;
        double* out = Y + P;
        hipLaunchKernelGGL(k_load_state<double>, g, b, 0, st, P, N, 1, u, op->perm, Y);
        enqueue_apply<double>(st, a, op->idx32, op->w64, Y, out);
        hipLaunchKernelGGL(k_store_state<double>, g, b, 0, st, P, N, 1, out, op->perm, Lu);
    } else {
        float* Y = (float*)op->work.p;
        float* out = Y + P;
        hipLaunchKernelGGL(k_load_state<float>, g, b, 0, st, P, N, 1, u, op->perm, Y);
        enqueue_apply<float>(st, a, op->idx32, op->w32, Y, out);
        hipLaunchKernelGGL(k_store_state<float>, g, b, 0, st, P, N, 1, out, op->perm, Lu);
    }
    HIP_TRY(ctx, hipGetLastError());
    return RBFFD_OK;
}

namespace {

int step_impl(rbffd_ctx ctx, rbffd_op op, int32_t nspecies, double* state, int32_t prec, const double* D,
              int32_t reaction, const double* params, double dt, int64_t nsteps, int32_t graph_steps, double t0,
              const double* forcing, double lam) {
    if (!ctx || !op || !state || !D) return set_error(ctx, RBFFD_E_ARG, "null argument");
    if (nspecies != 1 && nspecies != 2) return set_error(ctx, RBFFD_E_ARG, "nspecies must be 1 or 2");
    if (prec != RBFFD_F64 && prec != RBFFD_F32) return set_error(ctx, RBFFD_E_ARG, "prec must be F64 or F32");
    if (reaction < 0 || reaction > 2) return set_error(ctx, RBFFD_E_ARG, "unknown reaction %d", reaction);
    if (reaction != RBFFD_REACT_NONE && nspecies != 2)
        return set_error(ctx, RBFFD_E_ARG, "reaction needs two species");
    if (reaction != RBFFD_REACT_NONE && !params) return set_error(ctx, RBFFD_E_ARG, "reaction params required");
    if (!(dt > 0.0)) return set_error(ctx, RBFFD_E_ARG, "dt must be > 0");
    if (nsteps < 0) return set_error(ctx, RBFFD_E_ARG, "nsteps must be >= 0");
    if (graph_steps < 0) return set_error(ctx, RBFFD_E_ARG, "graph_steps must be >= 0");
    if (forcing && !(std::isfinite(t0) && std::isfinite(lam)))
        return set_error(ctx, RBFFD_E_ARG, "t0 and lambda must be finite");
    op->ctx = ctx;
    int rc = ensure_flag(op);
    if (!rc) rc = ensure_work(op);
    if (rc) return rc;
    hipStream_t st = ctx->stream;
    const int64_t N = op->N, P = op->P;
    const dim3 g((unsigned)((P + BLK - 1) / BLK)), b(BLK);
    StageArgs a = stage_args(op, prec == RBFFD_F64);
    a.D[0] = D[0];
    a.D[1] = nspecies == 2 ? D[1] : 0.0;
    a.dt = dt;
    const int np = reaction == RBFFD_REACT_SCHNAKENBERG ? 3 : (reaction == RBFFD_REACT_TURING ? 5 : 0);
    for (int i = 0; i < np; ++i) a.rp.p[i] = params[i];
    int64_t* steps_done = reinterpret_cast<int64_t*>(op->counters);
    int* nonfinite = reinterpret_cast<int*>(reinterpret_cast<char*>(op->counters) + sizeof(int64_t));
    a.nonfinite = nonfinite;
    a.steps_done = steps_done;
    const int G = graph_steps > 0 ? graph_steps : 50;
    const size_t esz = prec == RBFFD_F64 ? sizeof(double) : sizeof(float);
    char* base = (char*)op->work.p;
    void* U = base;
    void* ACC = base + 2 * P * esz;
    void* Y1 = base + 4 * P * esz;
    void* Y2 = base + 6 * P * esz;
    // FP32: compensation of the state update (inside the FP64-sized work area)
    void* COMP = prec == RBFFD_F64 ? nullptr : (void*)(base + 8 * P * esz);
    void* FI = base + 8 * P * sizeof(double);  // forcing in internal order, after the FP64 buffers
    if (forcing) {
        a.F = FI;
        a.lam = lam;
        a.t0 = t0;
    }
    const int32_t* idx = op->idx32;
    const void* w = prec == RBFFD_F64 ? (const void*)op->w64 : (const void*)op->w32;
    // counters are cleared by a kernel (no memset node near the captured graph)
    hipLaunchKernelGGL(k_set_steps, dim3(1), dim3(1), 0, st, steps_done, nonfinite);
    if (prec == RBFFD_F64) {
        hipLaunchKernelGGL(k_load_state<double>, g, b, 0, st, P, N, nspecies, state, op->perm, (double*)U);
        if (forcing) hipLaunchKernelGGL(k_load_state<double>, g, b, 0, st, P, N, nspecies, forcing, op->perm, (double*)FI);
    } else {
        hipLaunchKernelGGL(k_load_state<float>, g, b, 0, st, P, N, nspecies, state, op->perm, (float*)U);
        if (forcing) hipLaunchKernelGGL(k_load_state<float>, g, b, 0, st, P, N, nspecies, forcing, op->perm, (float*)FI);
        HIP_TRY(ctx, hipMemsetAsync(COMP, 0, 2 * (size_t)P * sizeof(float), st));  // outside any captured graph
    }
    HIP_TRY(ctx, hipGetLastError());

    auto enqueue = [&](hipStream_t s, int64_t steps) {
        if (prec == RBFFD_F64)
            enqueue_steps_t<double>(s, nspecies, reaction, a, idx, (const double*)w, (double*)U, (double*)ACC,
                                    nullptr, (double*)Y1, (double*)Y2, steps);
        else
            enqueue_steps_t<float>(s, nspecies, reaction, a, idx, (const float*)w, (float*)U, (float*)ACC,
                                   (float*)COMP, (float*)Y1, (float*)Y2, steps);
    };
    const int64_t reps = nsteps / G;
    const int64_t rest = nsteps % G;
    volatile int* nf_host = reinterpret_cast<volatile int*>(op->nonfinite_host);
    *nf_host = 0;
    bool stopped = false;
    if (reps > 0) {
        const int forced = forcing ? 1 : 0;
        bool same = op->graph && op->graph_key_species == nspecies && op->graph_key_prec == prec &&
                    op->graph_key_react == reaction && op->graph_key_steps == G && op->graph_key_dt == dt &&
                    op->graph_key_D[0] == a.D[0] && op->graph_key_D[1] == a.D[1] &&
                    std::memcmp(op->graph_key_params, a.rp.p, sizeof(a.rp.p)) == 0 &&
                    op->graph_key_forced == forced && (!forced || (op->graph_key_t0 == t0 && op->graph_key_lam == lam));
        if (!same) {
            reset_graph(op);
            hipGraph_t graph;
            HIP_TRY(ctx, hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
            enqueue(st, G);
            hipError_t ce = hipStreamEndCapture(st, &graph);
            if (ce != hipSuccess) return set_error(ctx, RBFFD_E_HIP, "graph capture failed: %s", hipGetErrorString(ce));
            hipError_t ie = hipGraphInstantiate(&op->graph, graph, nullptr, nullptr, 0);
            (void)hipGraphDestroy(graph);
            if (ie != hipSuccess) {
                op->graph = nullptr;
                return set_error(ctx, RBFFD_E_HIP, "graph instantiate failed: %s", hipGetErrorString(ie));
            }
            op->graph_key_species = nspecies;
            op->graph_key_prec = prec;
            op->graph_key_react = reaction;
            op->graph_key_steps = G;
            op->graph_key_dt = dt;
            op->graph_key_D[0] = a.D[0];
            op->graph_key_D[1] = a.D[1];
            std::memcpy(op->graph_key_params, a.rp.p, sizeof(a.rp.p));
            op->graph_key_forced = forced;
            op->graph_key_t0 = t0;
            op->graph_key_lam = lam;
        }
        for (int64_t r = 0; r < reps; ++r) {
            // the flag copied after an earlier replay has already landed: stop on a blow-up
            if (*nf_host) {
                stopped = true;
                break;
            }
            HIP_TRY(ctx, hipGraphLaunch(op->graph, st));
            HIP_TRY(ctx, hipMemcpyAsync(op->nonfinite_host, nonfinite, sizeof(int), hipMemcpyDeviceToHost, st));
        }
    }
    if (rest > 0 && !stopped) enqueue(st, rest);
    if (prec == RBFFD_F64)
        hipLaunchKernelGGL(k_store_state<double>, g, b, 0, st, P, N, nspecies, (const double*)U, op->perm, state);
    else
        hipLaunchKernelGGL(k_store_state<float>, g, b, 0, st, P, N, nspecies, (const float*)U, op->perm, state);
    HIP_TRY(ctx, hipGetLastError());
    HIP_TRY(ctx, hipMemcpyAsync(op->nonfinite_host, nonfinite, sizeof(int), hipMemcpyDeviceToHost, st));
    HIP_TRY(ctx, hipStreamSynchronize(st));
    if (*nf_host)
        return set_error(ctx, RBFFD_E_NONFINITE,
                         "the state became non-finite (steps stopped early; state holds the last values)");
    return RBFFD_OK;
}

}  // namespace

extern "C" int rbffd_step(rbffd_ctx ctx, rbffd_op op, int32_t nspecies, double* state, int32_t prec, const double* D,
                          int32_t reaction, const double* params, double dt, int64_t nsteps, int32_t graph_steps) {
    return step_impl(ctx, op, nspecies, state, prec, D, reaction, params, dt, nsteps, graph_steps, 0.0, nullptr,
                     0.0);
}

extern "C" int rbffd_step_forced(rbffd_ctx ctx, rbffd_op op, int32_t nspecies, double* state, int32_t prec,
                                 const double* D, int32_t reaction, const double* params, double dt, int64_t nsteps,
                                 int32_t graph_steps, double t0, const double* forcing, double lambda) {
    if (!forcing) return set_error(ctx, RBFFD_E_ARG, "forcing is required");
    return step_impl(ctx, op, nspecies, state, prec, D, reaction, params, dt, nsteps, graph_steps, t0, forcing,
                     lambda);
}

// ------------------------------------------------------------------------
// Semi-implicit BDF time stepping (the paper's BDF4 of Sec. 6 for the forced
// diffusion problems and SBDF2 of Sec. 7 for the Turing system): each step
//   sum_{j=0}^{k} a_j u^{n+1-j} = dt (D L u^{n+1} + f(t_{n+1}) + sum_{j=1}^{k} b_j R(u^{n+1-j})),
// i.e. (I - gamma L) u_s^{n+1} = rhs_s / a_0 with gamma = dt D_s / a_0, solved
// per species by unpreconditioned BiCGSTAB, restarted from the true residual
// after a breakdown.  There is no diagonal (Jacobi) scaling on purpose: on
// irregular node sets some stencils give L a positive diagonal entry, so the
// diagonal of I - gamma L passes through zero as dt grows and dividing by it
// wrecks the iteration, while the unscaled system stays well conditioned
// (its eigenvalues have real part >= 1 whenever L's are in the left half
// plane, the stability property of Sec. 5).  Vectors are FP64 in internal
// order, one array per species; every scalar of the iteration stays on the
// device; the host reads the residual norm every few iterations to stop.
namespace {


struct BdfCoef {
    double a[5], b[4];
};

// k-step BDF row a and extrapolation row b (see the oracle's table).
BdfCoef bdf_coef(int k) {
    BdfCoef c;
    std::memset(&c, 0, sizeof(c));
    if (k == 1) {
        c.a[0] = 1.0; c.a[1] = -1.0;
        c.b[0] = 1.0;
    } else if (k == 2) {
        c.a[0] = 1.5; c.a[1] = -2.0; c.a[2] = 0.5;
        c.b[0] = 2.0; c.b[1] = -1.0;
    } else if (k == 3) {
        c.a[0] = 11.0 / 6.0; c.a[1] = -3.0; c.a[2] = 1.5; c.a[3] = -1.0 / 3.0;
        c.b[0] = 3.0; c.b[1] = -3.0; c.b[2] = 1.0;
    } else {
        c.a[0] = 25.0 / 12.0; c.a[1] = -4.0; c.a[2] = 3.0; c.a[3] = -4.0 / 3.0; c.a[4] = 0.25;
        c.b[0] = 4.0; c.b[1] = -6.0; c.b[2] = 4.0; c.b[3] = -1.0;
    }
    return c;
}

// Scalars of one BiCGSTAB solve (device).
struct KrylovScalars {
    double rho, alpha, omega, beta;
    double bb, rr;        // ||b||^2, ||r||^2
    double rr0;           // ||rhat||^2 (the residual at the last start)
    double tol2;          // tol^2
    double gamma;         // the solve's I - gamma L (read by the operator kernel)
    int breakdown;        // rhat (nearly) orthogonal to r, or a zero step
    int done;             // 0 running, 1 converged, 2 restart wanted, 3 non-finite residual
    int iters;            // iterations done since the solve began (restarts not counted)
    int pad;
};

// Iterations of one graph; the host reads the scalars after as many graphs as
// the species' last solve took, and the kernels of iterations after
// convergence (or a breakdown) return at once.
constexpr int KRYLOV_BATCH = 8;
// Block partials that a kernel sums by itself, two loads per thread of a block
// of four wavefronts; with as many slices or fewer the blocks are single
// wavefronts, on four times as many CUs (five steps at N = 10242 6.3 -> 5.7 ms).
// More are first summed to PART_SUMS by a kernel of as many blocks, whose launch
// (2 us) costs less than all of them read by every block of the next kernel
// (summed by one block they cost 5 % of an iteration at N = 1e6).
constexpr int PART_DIRECT = 512;
constexpr int PART_SUMS = 32;
// Slot bytes up to which p and s are formed while they are gathered.  Ten SBDF2
// steps, fused against p and s as passes of their own: 294 MB 89.4 and 90.9 ms,
// 490 MB 146.4 and 144.4 (torus), 153.7 and 151.5 (ellipsoid), 600 MB 203.8 and
// 198.6: an operator that streams from memory drives the vectors out of the
// caches, and the fused kernels gather up to three of them.
constexpr int64_t KRY_FUSED = (int64_t)384 << 20;

struct HistPtrs {
    const double* u[4];   // u^n, u^{n-1}, ... (one species)
    const double* r[4];   // R_s at those states (nullable entries when no reaction)
};

// R(u) for both species of one state (rows in internal order, per-species arrays).
template <int R>
__global__ void k_reaction2(int64_t P, const double* __restrict__ u, const double* __restrict__ v, ReactParams rp,
                            double* __restrict__ ru, double* __restrict__ rv) {
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p >= P) return;
    double y[2] = {u[p], v[p]}, r[2];
    reaction<double, R>(y, r, rp);
    ru[p] = r[0];
    rv[p] = r[1];
}

// L y at row rp.p, neighbour values made by conv() from entries of NV vectors
// (FP64, one species; in slot order).
// load() first, then sum(); every lane of the wavefront takes part in both.
template <int NV, int MODE, int B>
struct LaplacianOf {
    RowAhead<double, 1, NV, MODE> ahead;
    double own[NV];
    double wd;

    __device__ __forceinline__ void load(const StageArgs& a, const RowPos& rp, const double* __restrict__ w,
                                         const double* const (&Y)[NV]) {
        if (rp.live) {
#pragma unroll
            for (int v = 0; v < NV; ++v) own[v] = Y[v][rp.p];
            wd = ld<MODE>(a.wd64 + rp.p);
        }
        ahead.load(a, rp, w, Y);
    }
    template <typename C>
    __device__ __forceinline__ double sum(const StageArgs& a, const RowPos& rp, const int32_t* __restrict__ idx,
                                          const double* __restrict__ w, const double* const (&Y)[NV], double yi,
                                          C&& conv) {
        __shared__ double ylds[B / 64][OP_HALO_MAX];
        const double y2[2] = {yi, 0.0};
        double lap[2] = {0.0, 0.0};
        if (rp.halo >= 0) {
            ahead.finish(a, rp, w, Y, conv, ylds[threadIdx.x >> 6], y2, wd, lap);
            return lap[0];
        }
        if (!rp.live) return 0.0;
        double acc = wd * yi;
#pragma unroll 8
        for (int k = 0; k < rp.ns; ++k) {
            const int64_t at = rp.base + slot_pos(k, rp.ns, rp.lane);
            const int64_t j = idx[at];
            double e[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) e[v] = Y[v][j];
            acc = fma(w[at], conv(e), acc);
        }
        return acc;
    }
};

__device__ __forceinline__ double wave_sum_block(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
// Sums of two values over a block of B = 64 or 256, the same bits in every
// thread (sh: 8 words; a barrier on entry, so that sh may be used again).
template <int B>
__device__ __forceinline__ void block_sum2(double& v0, double& v1, double* sh) {
    v0 = wave_sum_block(v0);
    v1 = wave_sum_block(v1);
    if constexpr (B > 64) {
        __syncthreads();
        if ((threadIdx.x & 63) == 0) {
            sh[2 * (threadIdx.x >> 6)] = v0;
            sh[2 * (threadIdx.x >> 6) + 1] = v1;
        }
        __syncthreads();
        v0 = (sh[0] + sh[2]) + (sh[4] + sh[6]);
        v1 = (sh[1] + sh[3]) + (sh[5] + sh[7]);
    }
}
// Block partials (pairs) summed in a fixed order: deterministic, and the same
// in every block that does it.
// At most PART_DIRECT of them, all loads of a thread in flight at once.
template <int B>
struct FewPartials {
    static constexpr int M = PART_DIRECT / B;
    double2 v[M];
    int count;  // of this thread
    __device__ __forceinline__ FewPartials(const double2* __restrict__ part, int np)
        : count((np - (int)threadIdx.x + B - 1) / B) {
        if (np == 0) return;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            if constexpr (B == 64) {  // no branches: 2 % of an iteration
                v[i] = part[min((int)threadIdx.x + B * i, np - 1)];
            } else {
                v[i] = make_double2(0.0, 0.0);
                if ((int)threadIdx.x + B * i < np) v[i] = part[threadIdx.x + B * i];
            }
        }
    }
    __device__ __forceinline__ void sum(double& d0, double& d1, double* sh) const {
        d0 = d1 = 0.0;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            d0 += B != 64 || i < count ? v[i].x : 0.0;
            d1 += B != 64 || i < count ? v[i].y : 0.0;
        }
        block_sum2<B>(d0, d1, sh);
    }
};
// More of them into PART_SUMS, one range per block.
__global__ __launch_bounds__(256) void k_sum_partials(const double2* __restrict__ part, int np,
                                                      double2* __restrict__ out) {
    __shared__ double sh[8];
    const int per = (np + PART_SUMS - 1) / PART_SUMS, first = blockIdx.x * per, last = min(first + per, np);
    double d0 = 0.0, d1 = 0.0;
    for (int i = first + threadIdx.x; i < last; i += 256) {
        const double2 v = part[i];
        d0 += v.x;
        d1 += v.y;
    }
    block_sum2<256>(d0, d1, sh);
    if (threadIdx.x == 0) out[blockIdx.x] = make_double2(d0, d1);
}

__device__ __forceinline__ int residual_state(const KrylovScalars& k, double rr) {
    if (!(rr <= 1.79e308)) return 3;
    const double lim = k.bb > 0.0 ? k.tol2 * k.bb : k.tol2;
    return rr <= lim ? 1 : 0;
}
// End of an iteration (rr = r.r, rho = rhat.r): converged, non-finite, or else
// beta = (rho' / rho) (alpha / omega) for the next one, unless |rho'| <= 1e-14
// ||rhat|| ||r|| or omega = 0 (breakdown: the host restarts from the true
// residual).
__device__ __forceinline__ void end_iteration(KrylovScalars& k, double rr, double rho) {
    k.iters += 1;
    k.rr = rr;
    k.done = residual_state(k, rr);
    if (k.done) return;
    if (k.breakdown || !(std::fabs(rho) > 1e-14 * std::sqrt(k.rr0 * rr)) || k.omega == 0.0) {
        k.breakdown = 1;
        k.done = 2;
        return;
    }
    k.beta = (rho / k.rho) * (k.alpha / k.omega);
    k.rho = rho;
}

// Start (FIRST: of a step's solve; else after a breakdown): r = rhat = b - (x -
// gamma L x), p = v = 0, partials of b.b and r.r.  FIRST also forms the right
// hand side b = (-sum_{j>=1} a_j u^{n+1-j} + dt sum_j b_j R^{n+1-j} + dt ef F)
// / a_0 and x = u^n.  Padding rows are written as
// zero in every vector, here and below.
template <bool FIRST, int MODE, int B>
__global__ __launch_bounds__(B) void k_kry_start(StageArgs a, const int32_t* __restrict__ idx,
                                                   const double* __restrict__ w, int nk, BdfCoef c, HistPtrs hp,
                                                   const double* __restrict__ F, double ef, double dt, double gamma,
                                                   double* __restrict__ b, double* __restrict__ x,
                                                   double* __restrict__ r, double* __restrict__ rh,
                                                   double* __restrict__ pv, double* __restrict__ v,
                                                   double2* __restrict__ part) {
    __shared__ double sh[8];
    const RowPos rp = row_pos<B>(a);
    const int64_t p = rp.p;
    const double* __restrict__ x0 = FIRST ? hp.u[0] : x;
    const double* const ys[1] = {x0};
    LaplacianOf<1, MODE, B> L;
    L.load(a, rp, w, ys);
    const double yi = rp.live ? L.own[0] : 0.0;
    const double lap = L.sum(a, rp, idx, w, ys, yi, [](const double (&e)[1]) { return e[0]; });
    double bb = 0.0, rr = 0.0;
    if (rp.slice >= 0) {
        double bv = 0.0;
        if constexpr (FIRST) {
            for (int j = 1; j <= nk && rp.live; ++j) {
                bv = fma(-c.a[j], hp.u[j - 1][p], bv);
                if (hp.r[j - 1]) bv = fma(dt * c.b[j - 1], hp.r[j - 1][p], bv);
            }
            if (F && rp.live) bv = fma(dt * ef, F[p], bv);
            bv /= c.a[0];
            b[p] = bv;
            x[p] = yi;
        } else {
            bv = b[p];
        }
        const double rv = bv - fma(-gamma, lap, yi);
        r[p] = rv;
        rh[p] = rv;
        pv[p] = 0.0;
        v[p] = 0.0;
        bb = bv * bv;
        rr = rv * rv;
    }
    block_sum2<B>(bb, rr, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = make_double2(bb, rr);
}
// bb, rr = rr0 = rho = r.r; alpha = omega = 1, tol and gamma stored; iters = 0
// on the first start of a solve; done at once if r already meets tol
__global__ __launch_bounds__(256) void k_kry_begin(const double2* __restrict__ part, int np, KrylovScalars* ks,
                                                   double tol, int first, double gamma) {
    __shared__ double sh[8];
    double d0, d1;
    FewPartials<256>(part, np).sum(d0, d1, sh);
    if (threadIdx.x != 0) return;
    ks->bb = d0;
    ks->rr = ks->rr0 = ks->rho = d1;
    ks->alpha = ks->omega = 1.0;
    ks->beta = 0.0;
    ks->tol2 = tol * tol;
    ks->gamma = gamma;
    ks->breakdown = 0;
    if (first) ks->iters = 0;
    ks->done = residual_state(*ks, d1);
}

// One iteration is three kernels.  What neighbours need of p and s is formed
// from the vectors of the kernel before while it is gathered, so neither is a
// pass of its own; scalars are formed from the block partials by every block
// alike and stored by block 0, in the other of two copies where other blocks
// still read the old one.  What bounds it is the latency of a launch and of its
// dependent loads, and above N = 1e5 the operator's bytes, read twice.  Against
// eleven kernels an iteration and the stage kernels' earlier order of loads: ten
// steps at N = 10242, n = 31 26.4 -> 10.0 ms, five at N = 2500 10.9 -> 4.3 ms,
// five at N = 1e5, n = 50 21.8 -> 11.4 ms, ten at N = 6e5 99.0 -> 89.9 ms.
//
// k_kry_pv: the last iteration's end unless FIRST of a launch sequence (then ks_in is
// final); p' = r + beta (p - omega v), v' = p' - gamma L p', partials rhat.v'
template <bool FIRST, int MODE, int B>
__global__ __launch_bounds__(B) void k_kry_pv(StageArgs a, const int32_t* __restrict__ idx,
                                                const double* __restrict__ w, const double2* __restrict__ part_in,
                                                int np, const KrylovScalars* ks_in, KrylovScalars* ks_out,
                                                const double* __restrict__ r, const double* __restrict__ rh,
                                                const double* __restrict__ pv, const double* __restrict__ v,
                                                double* __restrict__ p_out, double* __restrict__ v_out,
                                                double2* __restrict__ part) {
    __shared__ double sh[8];
    const bool writer = blockIdx.x == 0 && threadIdx.x == 0;
    KrylovScalars k = *ks_in;
    const FewPartials<B> sums(part_in, FIRST ? 0 : np);
    const RowPos rp = row_pos<B>(a);
    const double* const ys[3] = {r, pv, v};
    LaplacianOf<3, MODE, B> L;
    L.load(a, rp, w, ys);
    if constexpr (!FIRST) {
        if (!k.done) {
            double d0, d1;
            sums.sum(d0, d1, sh);
            end_iteration(k, d0, d1);
        }
        if (writer) *ks_out = k;
    }
    if (k.done) return;
    auto val = [&](const double (&e)[3]) { return fma(k.beta, fma(-k.omega, e[2], e[1]), e[0]); };
    const double yi = rp.live ? val(L.own) : 0.0;
    const double lap = L.sum(a, rp, idx, w, ys, yi, val);
    double d = 0.0, z = 0.0;
    if (rp.slice >= 0) {
        const double o = fma(-k.gamma, lap, yi);
        p_out[rp.p] = yi;
        v_out[rp.p] = o;
        d = rh[rp.p] * o;
    }
    block_sum2<B>(d, z, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = make_double2(d, 0.0);
}
// alpha = rho / rhat.v; s = r - alpha v, t = s - gamma L s, partials t.s and t.t
template <int MODE, int B>
__global__ __launch_bounds__(B) void k_kry_st(StageArgs a, const int32_t* __restrict__ idx,
                                                const double* __restrict__ w, const double2* __restrict__ part_in,
                                                int np, KrylovScalars* ks, const double* __restrict__ r,
                                                const double* __restrict__ v, double* __restrict__ sv,
                                                double* __restrict__ tv, double2* __restrict__ part) {
    __shared__ double sh[8];
    const int done = ks->done;
    const double gamma = ks->gamma, rho = ks->rho;
    const FewPartials<B> sums(part_in, np);
    const RowPos rp = row_pos<B>(a);
    const double* const ys[2] = {r, v};
    LaplacianOf<2, MODE, B> L;
    L.load(a, rp, w, ys);
    if (done) return;
    double d0, d1;
    sums.sum(d0, d1, sh);
    const bool broken = d0 == 0.0;
    const double alpha = broken ? 0.0 : rho / d0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {  // no block reads these two here
        ks->alpha = alpha;
        if (broken) ks->breakdown = 1;
    }
    auto val = [&](const double (&e)[2]) { return fma(-alpha, e[1], e[0]); };
    const double yi = rp.live ? val(L.own) : 0.0;
    const double lap = L.sum(a, rp, idx, w, ys, yi, val);
    double ts = 0.0, tt = 0.0;
    if (rp.slice >= 0) {
        const double o = fma(-gamma, lap, yi);
        sv[rp.p] = yi;
        tv[rp.p] = o;
        ts = o * yi;
        tt = o * o;
    }
    block_sum2<B>(ts, tt, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = make_double2(ts, tt);
}
// The two operator kernels above for an operator that streams from memory
// (past KRY_FUSED bytes), where p and s are passes of their own.
template <bool FIRST>
__global__ __launch_bounds__(256) void k_kry_p(int64_t P, const double2* __restrict__ part_in, int np,
                                               const KrylovScalars* ks_in, KrylovScalars* ks_out,
                                               const double* __restrict__ r, const double* __restrict__ pv,
                                               const double* __restrict__ v, double* __restrict__ p_out) {
    __shared__ double sh[8];
    KrylovScalars k = *ks_in;
    if constexpr (!FIRST) {
        const FewPartials<256> sums(part_in, np);
        if (!k.done) {
            double d0, d1;
            sums.sum(d0, d1, sh);
            end_iteration(k, d0, d1);
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) *ks_out = k;
    }
    const int64_t p = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (k.done || p >= P) return;
    p_out[p] = fma(k.beta, fma(-k.omega, v[p], pv[p]), r[p]);
}
__global__ __launch_bounds__(256) void k_kry_s(int64_t P, const double2* __restrict__ part_in, int np,
                                               KrylovScalars* ks, const double* __restrict__ r,
                                               const double* __restrict__ v, double* __restrict__ sv) {
    __shared__ double sh[8];
    if (ks->done) return;
    const double rho = ks->rho;
    const FewPartials<256> sums(part_in, np);
    double d0, d1;
    sums.sum(d0, d1, sh);
    const bool broken = d0 == 0.0;
    const double alpha = broken ? 0.0 : rho / d0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {  // no block reads these two here
        ks->alpha = alpha;
        if (broken) ks->breakdown = 1;
    }
    const int64_t p = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (p < P) sv[p] = fma(-alpha, v[p], r[p]);
}
// out = y - gamma L y, partials of rhat.out (rh given) or of out.y and out.out
__global__ __launch_bounds__(256) void k_kry_av(StageArgs a, const int32_t* __restrict__ idx,
                                                const double* __restrict__ w, const KrylovScalars* ks,
                                                const double* __restrict__ y, const double* __restrict__ rh,
                                                double* __restrict__ out, double2* __restrict__ part) {
    __shared__ double sh[8];
    if (ks->done) return;
    const double gamma = ks->gamma;
    const RowPos rp = row_pos<256>(a);
    const double* const ys[1] = {y};
    LaplacianOf<1, STREAM_WIDE, 256> L;
    L.load(a, rp, w, ys);
    const double yi = rp.live ? L.own[0] : 0.0;
    const double lap = L.sum(a, rp, idx, w, ys, yi, [](const double (&e)[1]) { return e[0]; });
    double d0 = 0.0, d1 = 0.0;
    if (rp.slice >= 0) {
        const double o = fma(-gamma, lap, yi);
        out[rp.p] = o;
        d0 = o * (rh ? rh[rp.p] : yi);
        d1 = rh ? 0.0 : o * o;
    }
    block_sum2<256>(d0, d1, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = make_double2(d0, d1);
}

// omega = t.s / t.t; x += alpha p + omega s, r = s - omega t, partials r.r and rhat.r
template <int B>
__global__ __launch_bounds__(B) void k_kry_xr(int64_t P, const double2* __restrict__ part_in, int np,
                                                KrylovScalars* ks, const double* __restrict__ pv,
                                                const double* __restrict__ sv, const double* __restrict__ tv,
                                                const double* __restrict__ rh, double* __restrict__ x,
                                                double* __restrict__ r, double2* __restrict__ part) {
    __shared__ double sh[8];
    const int done = ks->done;
    const double alpha = ks->alpha;
    const FewPartials<B> sums(part_in, np);
    const int64_t p = blockIdx.x * (int64_t)B + threadIdx.x;
    double s = 0.0, t = 0.0, pi = 0.0, xi = 0.0, h = 0.0;
    if (p < P) {
        s = sv[p];
        t = tv[p];
        pi = pv[p];
        xi = x[p];
        h = rh[p];
    }
    if (done) return;
    double d0, d1;
    sums.sum(d0, d1, sh);
    const double omega = d1 > 0.0 ? d0 / d1 : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) ks->omega = omega;  // no block reads it here
    double rr = 0.0, hr = 0.0;
    if (p < P) {
        x[p] = fma(omega, s, fma(alpha, pi, xi));
        const double q = fma(-omega, t, s);
        r[p] = q;
        rr = q * q;
        hr = h * q;
    }
    block_sum2<B>(rr, hr, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = make_double2(rr, hr);
}
// End of the last iteration of a launch sequence; the scalars move to *ks_out.
__global__ __launch_bounds__(256) void k_kry_end(const double2* __restrict__ part, int np, const KrylovScalars* ks_in,
                                                 KrylovScalars* ks_out) {
    __shared__ double sh[8];
    KrylovScalars k = *ks_in;
    const FewPartials<256> sums(part, np);
    if (!k.done) {
        double d0, d1;
        sums.sum(d0, d1, sh);
        end_iteration(k, d0, d1);
    }
    __syncthreads();
    if (threadIdx.x == 0) *ks_out = k;
}

__global__ void k_copy(int64_t P, const double* __restrict__ src, double* __restrict__ dst) {
    const int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (p < P) dst[p] = src[p];
}

int ensure_impl(rbffd_op op, size_t bytes) {
    if (op->impl_bytes >= bytes) return RBFFD_OK;
    if (op->impl) {
        (void)hipStreamSynchronize(op->ctx->stream);
        reset_kgraph(op);
        (void)hipFree(op->impl);
        op->impl = nullptr;
        op->impl_bytes = 0;
    }
    if (device_alloc(op->spare, &op->impl, bytes) != hipSuccess) {
        return set_error(op->ctx, RBFFD_E_NOMEM, "cannot allocate %zu bytes for the implicit stepper", bytes);
    }
    // Left as it comes: every vector and partial sum is written in full before it
    // is read.  Padding rows of the reaction terms hold R(0, 0), which need not be
    // zero; the solver kernels write them as zero in every vector of a solve and
    // take nothing else from them (rp.live).
    op->impl_bytes = bytes;
    return RBFFD_OK;
}

}  // namespace

extern "C" int rbffd_step_imex(rbffd_ctx ctx, rbffd_op op, int32_t nspecies, double* state, const double* D,
                               int32_t reaction, const double* params, double dt, int64_t nsteps, int32_t order,
                               const double* history, double t0, const double* forcing, double lambda, double tol,
                               int32_t maxit, int64_t* iters_out, double* relres_out) {
    if (!ctx || !op || !state || !D) return set_error(ctx, RBFFD_E_ARG, "null argument");
    if (nspecies != 1 && nspecies != 2) return set_error(ctx, RBFFD_E_ARG, "nspecies must be 1 or 2");
    if (reaction < 0 || reaction > 2) return set_error(ctx, RBFFD_E_ARG, "unknown reaction %d", reaction);
    if (reaction != RBFFD_REACT_NONE && nspecies != 2) return set_error(ctx, RBFFD_E_ARG, "reaction needs two species");
    if (reaction != RBFFD_REACT_NONE && !params) return set_error(ctx, RBFFD_E_ARG, "reaction params required");
    if (!(dt > 0.0)) return set_error(ctx, RBFFD_E_ARG, "dt must be > 0");
    if (nsteps < 0) return set_error(ctx, RBFFD_E_ARG, "nsteps must be >= 0");
    if (order < 1 || order > 4) return set_error(ctx, RBFFD_E_ARG, "order must be 1..4");
    if (!(tol > 0.0) || maxit < 1) return set_error(ctx, RBFFD_E_ARG, "tol must be > 0 and maxit >= 1");
    if (forcing && !(std::isfinite(t0) && std::isfinite(lambda)))
        return set_error(ctx, RBFFD_E_ARG, "t0 and lambda must be finite");
    op->ctx = ctx;
    const int64_t N = op->N, P = op->P;
    const int S = nspecies;
    const bool react = reaction != RBFFD_REACT_NONE;
    // layout: scalars (two copies), summed partials, three sets of block partials;
    // U[s][order], R[s][order] (reaction), F[s], b, x, r, rh, p and v (two each), s, t
    const int nvec = S * order * (react ? 2 : 1) + S + 10;
    const int kblk = op->nslices <= PART_DIRECT ? 64 : 256;  // threads per block of the solver's kernels
    const int nblk = (int)((P + kblk - 1) / kblk);
    constexpr size_t sums_at = 512, parts_at = sums_at + 3 * PART_SUMS * sizeof(double2);
    const size_t head = (parts_at + 3 * (size_t)nblk * sizeof(double2) + 255) & ~(size_t)255;
    const size_t vbytes = (size_t)P * sizeof(double);
    int rc = ensure_impl(op, head + nvec * vbytes);
    if (rc) return rc;
    hipStream_t st = ctx->stream;
    static_assert(2 * sizeof(KrylovScalars) <= sums_at, "scalars");
    KrylovScalars* ks = (KrylovScalars*)op->impl;
    double2* psum = (double2*)((char*)op->impl + sums_at);
    double2* part[3];
    for (int q = 0; q < 3; ++q) part[q] = (double2*)((char*)op->impl + parts_at) + (size_t)q * nblk;
    double* base = (double*)((char*)op->impl + head);
    auto vec = [&](int i) { return base + (size_t)i * P; };
    int vi = 0;
    double* U[2][4] = {};
    double* Rh[2][4] = {};
    for (int s = 0; s < S; ++s)
        for (int j = 0; j < order; ++j) U[s][j] = vec(vi++);
    if (react)
        for (int s = 0; s < S; ++s)
            for (int j = 0; j < order; ++j) Rh[s][j] = vec(vi++);
    double* Fi[2] = {};
    for (int s = 0; s < S; ++s) Fi[s] = vec(vi++);
    double* bvec = vec(vi++);
    double* x = vec(vi++);
    double* r = vec(vi++);
    double* rh = vec(vi++);
    double* pv[2] = {vec(vi), vec(vi + 1)};
    double* v[2] = {vec(vi + 2), vec(vi + 3)};
    double* sv = vec(vi + 4);
    double* tv = vec(vi + 5);
    const dim3 g((unsigned)((P + BLK - 1) / BLK)), b(BLK);
    StageArgs a = stage_args(op, true);
    ReactParams rp;
    std::memset(&rp, 0, sizeof(rp));
    const int np = reaction == RBFFD_REACT_SCHNAKENBERG ? 3 : (reaction == RBFFD_REACT_TURING ? 5 : 0);
    for (int i = 0; i < np; ++i) rp.p[i] = params[i];
    // history: state (and the caller's earlier states, if any) into internal order
    const int have0 = history ? order : 1;
    for (int s = 0; s < S; ++s) {
        hipLaunchKernelGGL(k_load_state<double>, g, b, 0, st, P, N, 1, state + (size_t)s * N, op->perm, U[s][0]);
        for (int j = 1; j < have0; ++j)
            hipLaunchKernelGGL(k_load_state<double>, g, b, 0, st, P, N, 1,
                               history + ((size_t)(j - 1) * S + s) * N, op->perm, U[s][j]);
        if (forcing)
            hipLaunchKernelGGL(k_load_state<double>, g, b, 0, st, P, N, 1, forcing + (size_t)s * N, op->perm, Fi[s]);
    }
    auto eval_reaction = [&](int j) {
        if (!react) return;
        if (reaction == RBFFD_REACT_SCHNAKENBERG)
            hipLaunchKernelGGL(k_reaction2<RBFFD_REACT_SCHNAKENBERG>, g, b, 0, st, P, U[0][j], U[1][j], rp, Rh[0][j],
                               Rh[1][j]);
        else
            hipLaunchKernelGGL(k_reaction2<RBFFD_REACT_TURING>, g, b, 0, st, P, U[0][j], U[1][j], rp, Rh[0][j], Rh[1][j]);
    };
    for (int j = 0; j < have0; ++j) eval_reaction(j);
    HIP_TRY(ctx, hipGetLastError());
    // ring of history slots: slot[j] = index into U/Rh of u^{n-j}
    int slot[4] = {0, 1, 2, 3};
    int have = have0;
    int64_t iters = 0;
    double worst = 0.0;
    int result = RBFFD_OK;
    int expect[2] = {1, 1};  // graphs of the species' last solve
    const dim3 sg(nblk), sb(kblk);
    const bool one = kblk == 64, fused = op->slots * 10 <= KRY_FUSED;
    // the fused kernels keep the slots (512 slices are far below KRY_FUSED), the
    // others do not (ten steps, 490 MB: kept 143.8, not 140.6 ms; ellipsoid 152.7
    // and 144.9)
    const auto start_first = one ? k_kry_start<true, KEEP, 64>
                                 : (fused ? k_kry_start<true, KEEP, 256> : k_kry_start<true, STREAM_WIDE, 256>);
    const auto start_again = one ? k_kry_start<false, KEEP, 64>
                                 : (fused ? k_kry_start<false, KEEP, 256> : k_kry_start<false, STREAM_WIDE, 256>);
    const auto pv_first = one ? k_kry_pv<true, KEEP, 64> : k_kry_pv<true, KEEP, 256>;
    const auto pv_next = one ? k_kry_pv<false, KEEP, 64> : k_kry_pv<false, KEEP, 256>;
    const auto st_kernel = one ? k_kry_st<KEEP, 64> : k_kry_st<KEEP, 256>;
    const auto xr_kernel = one ? k_kry_xr<64> : k_kry_xr<256>;
    // what the next kernel sums: the block partials of set q, or their sum
    const int npart = nblk <= PART_DIRECT ? nblk : PART_SUMS;
    auto summed = [&](int q) -> const double2* {
        if (npart == nblk) return part[q];
        hipLaunchKernelGGL(k_sum_partials, dim3(PART_SUMS), dim3(256), 0, st, part[q], nblk, psum + q * PART_SUMS);
        return psum + q * PART_SUMS;
    };
    for (int64_t n = 0; n < nsteps && result == RBFFD_OK; ++n) {
        const int k = std::min(order, have);
        const BdfCoef c = bdf_coef(k);
        const double t1 = t0 + (double)(n + 1) * dt;
        // the new state goes to the oldest slot (order == k) or the next free one
        const int newslot = have < order ? slot[have] : slot[order - 1];
        for (int s = 0; s < S; ++s) {
            HistPtrs h;
            std::memset(&h, 0, sizeof(h));
            for (int j = 0; j < k; ++j) {
                h.u[j] = U[s][slot[j]];
                h.r[j] = react ? Rh[s][slot[j]] : nullptr;
            }
            const double ef = forcing ? std::exp(lambda * t1) : 0.0;
            const double gamma = dt * D[s] / c.a[0];
            // (re)start from the true residual of x
            auto krylov_start = [&](int first) {
                if (first)
                    hipLaunchKernelGGL(start_first, sg, sb, 0, st, a, op->idx32, op->w64, k, c, h,
                                       forcing ? (const double*)Fi[s] : nullptr, ef, dt, gamma, bvec, x, r, rh, pv[0],
                                       v[0], part[0]);
                else
                    hipLaunchKernelGGL(start_again, sg, sb, 0, st, a, op->idx32, op->w64, k, c, h, nullptr, ef, dt,
                                       gamma, bvec, x, r, rh, pv[0], v[0], part[0]);
                const double2* ps = summed(0);
                hipLaunchKernelGGL(k_kry_begin, dim3(1), dim3(256), 0, st, ps, npart, ks, tol, first, gamma);
            };
            // `count` iterations; every kernel takes its scalars (gamma too) from
            // ks, so the same launches serve every species, step and tolerance.
            // ks[0] holds them before and after.
            auto iterations = [&](int count) {
                int cur = 0;
                const double2* ps = nullptr;
                for (int q = 0; q < count; ++q) {
                    const int from = q & 1, to = 1 - from;
                    if (!fused) {
                        if (q == 0) {
                            hipLaunchKernelGGL(k_kry_p<true>, sg, sb, 0, st, P, nullptr, 0, ks, ks, r, pv[from], v[from],
                                               pv[to]);
                        } else {
                            hipLaunchKernelGGL(k_kry_p<false>, sg, sb, 0, st, P, ps, npart, ks + cur, ks + 1 - cur, r,
                                               pv[from], v[from], pv[to]);
                            cur = 1 - cur;
                        }
                        hipLaunchKernelGGL(k_kry_av, sg, sb, 0, st, a, op->idx32, op->w64, ks + cur, pv[to], rh, v[to],
                                           part[0]);
                        ps = summed(0);
                        hipLaunchKernelGGL(k_kry_s, sg, sb, 0, st, P, ps, npart, ks + cur, r, v[to], sv);
                        hipLaunchKernelGGL(k_kry_av, sg, sb, 0, st, a, op->idx32, op->w64, ks + cur, sv, nullptr, tv,
                                           part[1]);
                        ps = summed(1);
                        hipLaunchKernelGGL(xr_kernel, sg, sb, 0, st, P, ps, npart, ks + cur, pv[to], sv, tv, rh, x, r,
                                           part[2]);
                        ps = summed(2);
                        continue;
                    }
                    if (q == 0) {
                        hipLaunchKernelGGL(pv_first, sg, sb, 0, st, a, op->idx32, op->w64, nullptr, 0, ks, ks, r,
                                           rh, pv[from], v[from], pv[to], v[to], part[0]);
                    } else {
                        hipLaunchKernelGGL(pv_next, sg, sb, 0, st, a, op->idx32, op->w64, ps, npart, ks + cur,
                                           ks + 1 - cur, r, rh, pv[from], v[from], pv[to], v[to], part[0]);
                        cur = 1 - cur;
                    }
                    ps = summed(0);
                    hipLaunchKernelGGL(st_kernel, sg, sb, 0, st, a, op->idx32, op->w64, ps, npart, ks + cur, r, v[to], sv, tv,
                                       part[1]);
                    ps = summed(1);
                    hipLaunchKernelGGL(xr_kernel, sg, sb, 0, st, P, ps, npart, ks + cur, pv[to], sv, tv, rh, x, r,
                                       part[2]);
                    ps = summed(2);
                }
                hipLaunchKernelGGL(k_kry_end, dim3(1), dim3(256), 0, st, ps, npart, ks + cur, ks);
            };
            // KRYLOV_BATCH iterations (an even number: p and v end where they began)
            // from one HIP graph, captured once per operator and vector layout
            auto batch_graph = [&]() -> int {
                if (!op->kgraph || op->kgraph_key != (const void*)x) {
                    reset_kgraph(op);
                    hipGraph_t graph;
                    HIP_TRY(ctx, hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
                    iterations(KRYLOV_BATCH);
                    hipError_t ce = hipStreamEndCapture(st, &graph);
                    if (ce != hipSuccess)
                        return set_error(ctx, RBFFD_E_HIP, "graph capture failed: %s", hipGetErrorString(ce));
                    hipError_t ie = hipGraphInstantiate(&op->kgraph, graph, nullptr, nullptr, 0);
                    (void)hipGraphDestroy(graph);
                    if (ie != hipSuccess) {
                        op->kgraph = nullptr;
                        return set_error(ctx, RBFFD_E_HIP, "graph instantiate failed: %s", hipGetErrorString(ie));
                    }
                    op->kgraph_key = x;
                }
                HIP_TRY(ctx, hipGraphLaunch(op->kgraph, st));
                return RBFFD_OK;
            };
            // initial guess: the current state
            krylov_start(1);
            HIP_TRY(ctx, hipGetLastError());
            bool conv = false;
            double relres = 0.0;
            int restarts = 0, graphs = 0;
            for (;;) {
                // a solve takes about as many graphs as the species' last one
                // did: launch all but one of them (at most seven) unread
                for (bool first = graphs == 0; first && graphs + 1 < expect[s] && graphs < 7 &&
                                               maxit >= (graphs + 1) * KRYLOV_BATCH;
                     ++graphs) {
                    const int rc = batch_graph();
                    if (rc) {
                        result = rc;
                        break;
                    }
                }
                if (result != RBFFD_OK) break;
                KrylovScalars hs;
                HIP_TRY(ctx, hipMemcpyAsync(&hs, ks, sizeof(hs), hipMemcpyDeviceToHost, st));
                HIP_TRY(ctx, hipStreamSynchronize(st));
                relres = hs.bb > 0.0 ? std::sqrt(hs.rr / hs.bb) : std::sqrt(hs.rr);
                if (hs.done == 3 || !std::isfinite(relres)) {
                    result = set_error(ctx, RBFFD_E_NONFINITE, "implicit solve: non-finite residual at step %lld",
                                       (long long)n);
                    break;
                }
                if (hs.done == 1) {
                    conv = true;
                    iters += hs.iters + restarts;
                    break;
                }
                const int used = hs.iters + restarts;
                if (used >= maxit) {
                    iters += used;
                    break;
                }
                if (hs.done == 2) {
                    ++restarts;
                    krylov_start(0);
                } else if (maxit - used >= KRYLOV_BATCH) {
                    const int rc = batch_graph();
                    if (rc) {
                        result = rc;
                        break;
                    }
                    ++graphs;
                } else {
                    iterations(maxit - used);
                }
                HIP_TRY(ctx, hipGetLastError());
            }
            if (result != RBFFD_OK) break;
            expect[s] = graphs;
            worst = std::max(worst, relres);
            hipLaunchKernelGGL(k_copy, g, b, 0, st, P, x, U[s][newslot]);
            if (!conv) {
                result = set_error(ctx, RBFFD_E_NOCONV,
                                   "implicit solve did not reach tol %g in %d iterations (relative residual %g) at "
                                   "step %lld", tol, maxit, relres, (long long)n);
            }
        }
        if (result != RBFFD_OK) break;
        // rotate the history: the new state is u^n from here on, then the
        // previous ones (at most order - 1 of them), then the unused slots
        int ns[4] = {0, 0, 0, 0};
        int q = 0;
        ns[q++] = newslot;
        for (int j = 0; j < std::min(have, order - 1); ++j) ns[q++] = slot[j];
        for (int idx = 0; idx < order && q < order; ++idx) {
            bool used = false;
            for (int j = 0; j < q; ++j) used = used || ns[j] == idx;
            if (!used) ns[q++] = idx;
        }
        for (int j = 0; j < order; ++j) slot[j] = ns[j];
        have = std::min(order, have + 1);
        eval_reaction(slot[0]);
    }
    for (int s = 0; s < S; ++s)
        hipLaunchKernelGGL(k_store_state<double>, g, b, 0, st, P, N, 1, U[s][slot[0]], op->perm, state + (size_t)s * N);
    HIP_TRY(ctx, hipGetLastError());
    HIP_TRY(ctx, hipStreamSynchronize(st));
    if (iters_out) *iters_out = iters;
    if (relres_out) *relres_out = worst;
    return result;
}
