// Learned shape parameter: a 128 -> 128 -> 128 -> 1 ReLU regressor of
// y = log(eps * rho) from the stencil's tangent-plane offsets, with BF16
// matrix-core (MFMA) forward and backward passes and FP32 Adam.
//
// The target is the per-stencil eps that the bisection of Sec. 5
// (eq. target_cond) finds; the network only proposes eps: the weights kernel
// checks kappa_2 at the proposal and falls back to bisection outside the band.
//
// Features (per stencil, centre x_1, unit normal nu, neighbours x_2..x_n):
// offsets d_j = x_j - x_1 in the canonical tangent frame tau_1 ~ Pi (x_2 - x_1)
// (the nearest neighbour), tau_2 = nu x tau_1, scaled by rho = max_j |d_j|:
// f[2(j-2)] = d_j . tau_1 / rho, f[2(j-2)+1] = d_j . tau_2 / rho, zero-padded
// to 128 entries, stored BF16.
//
// Parameters (FP32, this order): W1[128][128] (out, in), b1[128],
// W2[128][128], b2[128], w3[128], b3.  BF16 copies of W1, W2 and the
// transpose of W2 feed the MFMAs.
//
// Every GEMM below is a sum of 16 x 16 output tiles D[r][c] = sum_k A[r][k]
// B[c][k] with both operands K-contiguous; v_mfma_f32_16x16x32_bf16 takes, in
// lane l, A[l%16][8(l/16) .. +7] and B[l%16][8(l/16) .. +7] and returns
// D[4(l/16) + i][l%16], i = 0..3.
#include "common.h"

#include <algorithm>
#include <cmath>

namespace {

constexpr int F = RBFFD_MLP_IN;       // 128
constexpr int H = RBFFD_MLP_HIDDEN;   // 128
constexpr int OFF_W1 = 0;
constexpr int OFF_B1 = OFF_W1 + H * F;
constexpr int OFF_W2 = OFF_B1 + H;
constexpr int OFF_B2 = OFF_W2 + H * H;
constexpr int OFF_W3 = OFF_B2 + H;
constexpr int OFF_B3 = OFF_W3 + H;
static_assert(OFF_B3 + 1 == RBFFD_MLP_PARAMS, "parameter layout");

constexpr int TB = 64;        // a training batch is a multiple of this
constexpr int WG = 256;       // 4 waves
constexpr int TLD = F + 8;    // row stride of the LDS tiles: rows start 4 banks apart

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// float -> bf16, round to nearest even (NaN -> quiet NaN)
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x7fffffu)) return 0x7fc0;
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

__device__ __forceinline__ double first_lane(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

__device__ __forceinline__ uint64_t mix64(uint64_t x) {
    x ^= x >> 30;
    x *= 0xbf58476d1ce4e5b9ull;
    x ^= x >> 27;
    x *= 0x94d049bb133111ebull;
    x ^= x >> 31;
    return x;
}

struct Bf16Params {
    const uint16_t* W1;   // [H][F]
    const uint16_t* W2;   // [H][H]
    const uint16_t* W2T;  // [H][H] transposed
    const float* P;       // FP32 parameters (biases, w3, b3)
};

// One wavefront takes FR samples through the network: their features (rows of
// TLD entries) are in `X`, which the first layer's output then overwrites.
// Returns y of sample 16 (c >> 2) + 4 (l >> 4) + (c & 3), c = l & 15, in the lanes with
// c < 8.  Nothing is shared between wavefronts, so there are no barriers to wait at, and a
// weight fragment serves 32 samples.
constexpr int FR = 32;
__device__ __forceinline__ int sample_of(int l) { return 16 * ((l & 7) >> 2) + 4 * (l >> 4) + (l & 3); }
__device__ __forceinline__ float forward_rows(uint16_t* X, const Bf16Params& prm) {
    const int l = threadIdx.x & 63;
    const int col = l & 15, rq = (l >> 4) * 4, kq = (l >> 4) * 8;
    auto fragments = [&](bf16x8 (&a)[2][4]) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                a[t][q] = *reinterpret_cast<const bf16x8*>(X + (16 * t + col) * TLD + 32 * q + kq);
        }
    };
    // the 32 x 16 outputs ct of a layer with weights w
    auto product = [&](const bf16x8 (&a)[2][4], const uint16_t* w, int ct, floatx4 (&acc)[2]) {
        bf16x8 bf[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            bf[q] = *reinterpret_cast<const bf16x8*>(w + (ct * 16 + col) * F + 32 * q + kq);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            acc[t] = floatx4{0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t][q], bf[q], acc[t], 0, 0, 0);
        }
    };
    bf16x8 a[2][4];
    floatx4 acc[2];
    // ---- layer 1: H1 = relu(X W1^T + b1)
    fragments(a);
    __syncthreads();
#pragma unroll 2
    for (int ct = 0; ct < H / 16; ++ct) {
        const float bb = prm.P[OFF_B1 + ct * 16 + col];
        product(a, prm.W1, ct, acc);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                X[(16 * t + rq + i) * TLD + ct * 16 + col] = f2bf(fmaxf(acc[t][i] + bb, 0.0f));
        }
    }
    __syncthreads();
    // ---- layer 2: H2 = relu(H1 W2^T + b2); layer 3: y = H2 . w3 + b3
    fragments(a);
    float part[2][4] = {};
#pragma unroll 2
    for (int ct = 0; ct < H / 16; ++ct) {
        const float bb = prm.P[OFF_B2 + ct * 16 + col], w3 = prm.P[OFF_W3 + ct * 16 + col];
        product(a, prm.W2, ct, acc);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int i = 0; i < 4; ++i) part[t][i] = fmaf(bf2f(f2bf(fmaxf(acc[t][i] + bb, 0.0f))), w3, part[t][i]);
        }
    }
    float y = 0.0f;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int m = 1; m < 16; m <<= 1) part[t][i] += __shfl_xor(part[t][i], m, 64);
            if (col == 4 * t + i) y = part[t][i];
        }
    }
    return y + prm.P[OFF_B3];
}

__global__ __launch_bounds__(64) void k_mlp(int64_t count, Bf16Params prm, const uint16_t* __restrict__ x,
                                            float* __restrict__ y) {
    __shared__ __attribute__((aligned(16))) uint16_t X[FR * TLD];
    const int l = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * FR;
#pragma unroll
    for (int q = 0; q < FR / 4; ++q) {
        const int b = 4 * q + (l >> 4), k8 = (l & 15) * 8;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (base + b < count) v = *reinterpret_cast<const uint4*>(x + (base + b) * F + k8);
        *reinterpret_cast<uint4*>(X + b * TLD + k8) = v;
    }
    __syncthreads();
    const float v = forward_rows(X, prm);
    const int64_t at = base + sample_of(l);
    if ((l & 15) < 8 && at < count) y[at] = v;
}

// ---- training -------------------------------------------------------------
// A step is two kernels.  k_mlp_backward takes 16 samples per workgroup through
// forward and backward and stores what the weight gradients contract over,
// sample-contiguous; k_mlp_update contracts it, one 16 x 16 block of a weight
// matrix per workgroup, and applies Adam to the entries it owns.  At these
// batches a step is bound by latency, so the first spreads over four times the
// CUs that tiles of 64 reach and has every weight fragment in flight before the
// first matrix product, and the second sums over the batch without atomics (one
// kernel with 33 000 atomic adds per 64 samples, and a separate Adam, took
// 42 us a step at a batch of 4096; these take 9.2 and 6.0 us, 17 us a step).
constexpr int TT = 16;               // samples per workgroup
constexpr int CHUNK = 1 << 15;       // samples per launch: 32 MB of workspace
constexpr int STAT = H + 2;          // per workgroup: dw3, db3, loss

// XT and so on: [tile][128][TT], sample-contiguous; a workgroup of the first
// kernel writes 4 KB in a row of each, a fragment of the second reads two times
// 512 bytes.
struct Chunk {
    uint16_t *XT, *H1T, *G1T, *G2T;
    float* stat;                     // [tile][STAT]
    int64_t ld;                      // samples of the launch, a multiple of 32
};

// One 16 x 16 tile over K = 128 with the B fragments in registers.
__device__ __forceinline__ floatx4 mma_row(const uint16_t* a, const bf16x8 (&bf)[4]) {
    const int l = threadIdx.x & 63;
    floatx4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const bf16x8 av = *reinterpret_cast<const bf16x8*>(a + (l & 15) * TLD + 32 * q + (l >> 4) * 8);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bf[q], acc, 0, 0, 0);
    }
    return acc;
}
__device__ __forceinline__ void load_fragments(const uint16_t* w, bf16x8 (&bf)[4]) {
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        bf[q] = *reinterpret_cast<const bf16x8*>(w + (l & 15) * F + 32 * q + (l >> 4) * 8);
}
__device__ __forceinline__ uint2 pack4(const uint16_t (&h)[4]) {
    return make_uint2((uint32_t)h[0] | (uint32_t)h[1] << 16, (uint32_t)h[2] | (uint32_t)h[3] << 16);
}

// Samples first .. first + ld of the batch; sample s is row s of x, or with a
// seed a hashed row.  Samples past `batch` (the last launch's padding) or rows
// past count are zeros without error.  Wave w has columns 32 w .. 32 w + 31 of
// every layer.
__global__ __launch_bounds__(WG) void k_mlp_backward(int64_t count, int64_t first, int64_t batch, Bf16Params prm,
                                                     const uint16_t* __restrict__ x, const float* __restrict__ target,
                                                     Chunk c, float gscale, uint64_t seed, int64_t step) {
    __shared__ __attribute__((aligned(16))) uint16_t Xs[TT * TLD], H1s[TT * TLD], G2s[TT * TLD];
    __shared__ float ypart[WG / 64][TT], tgs[TT];
    __shared__ bool ins[TT];
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63;
    const int col = l & 15, rq = (l >> 4) * 4;
    bf16x8 w1[2][4], w2[2][4], w2t[2][4];
    float b1[2], b2[2], w3[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int o = 32 * wv + 16 * t;
        load_fragments(prm.W1 + o * F, w1[t]);
        b1[t] = prm.P[OFF_B1 + o + col];
        b2[t] = prm.P[OFF_B2 + o + col];
        w3[t] = prm.P[OFF_W3 + o + col];
    }
    const float b3 = prm.P[OFF_B3];
    {
        const int b = tid >> 4, k8 = (tid & 15) * 8;
        const int64_t smp = first + (int64_t)blockIdx.x * TT + b;
        int64_t rr = smp;
        if (seed != 0)
            rr = (int64_t)(mix64(seed ^ mix64((uint64_t)step * 0x9e3779b97f4a7c15ull + (uint64_t)smp)) %
                           (uint64_t)count);
        const bool in = smp < batch && rr < count;
        uint4 v = make_uint4(0, 0, 0, 0);
        float tg = 0.0f;
        if (in) {
            v = *reinterpret_cast<const uint4*>(x + rr * F + k8);
            tg = target[rr];
        }
        // loads return in order: what is needed last is asked for last
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            load_fragments(prm.W2 + (32 * wv + 16 * t) * H, w2[t]);
            load_fragments(prm.W2T + (32 * wv + 16 * t) * H, w2t[t]);
        }
        if (k8 == 0) {
            tgs[b] = tg;
            ins[b] = in;
        }
        *reinterpret_cast<uint4*>(Xs + b * TLD + k8) = v;
    }
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * TT * H;  // of the tile's arrays
    // ---- layer 1: H1 = relu(X W1^T + b1)
    uint16_t h1[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const floatx4 acc = mma_row(Xs, w1[t]);
        const int o = 32 * wv + 16 * t + col;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h1[t][i] = f2bf(fmaxf(acc[i] + b1[t], 0.0f));
            H1s[(rq + i) * TLD + o] = h1[t][i];
        }
        *reinterpret_cast<uint2*>(c.H1T + t0 + o * TT + rq) = pack4(h1[t]);
    }
    {   // X, sample-contiguous
        const int k = tid >> 1, b0 = (tid & 1) * 8;
        uint32_t v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[q] = (uint32_t)Xs[(b0 + 2 * q) * TLD + k] | (uint32_t)Xs[(b0 + 2 * q + 1) * TLD + k] << 16;
        *reinterpret_cast<uint4*>(c.XT + t0 + k * TT + b0) = make_uint4(v[0], v[1], v[2], v[3]);
    }
    __syncthreads();
    // ---- layer 2: H2 = relu(H1 W2^T + b2); layer 3: y = H2 . w3 + b3
    float h2[2][4], part[4] = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const floatx4 acc = mma_row(H1s, w2[t]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h2[t][i] = bf2f(f2bf(fmaxf(acc[i] + b2[t], 0.0f)));
            part[i] = fmaf(h2[t][i], w3[t], part[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) part[i] += __shfl_xor(part[i], m, 64);
        if (col == 0) ypart[wv][rq + i] = part[i];
    }
    __syncthreads();
    // ---- backward: L = gscale * sum_b (y_b - t_b)^2
    float dy[4], db3 = 0.0f, loss = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int b = rq + i;
        const float y = ((ypart[0][b] + ypart[1][b]) + (ypart[2][b] + ypart[3][b])) + b3;
        const float e = ins[b] ? y - tgs[b] : 0.0f;
        dy[i] = 2.0f * gscale * e;
        db3 += dy[i];
        loss = fmaf(gscale * e, e, loss);
    }
    // dw3, db3 and the loss of the tile; dH2 = dy w3 [H2 > 0]
    float* st = c.stat + (int64_t)blockIdx.x * STAT;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int o = 32 * wv + 16 * t + col;
        float s = 0.0f;
        uint16_t g[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s = fmaf(dy[i], h2[t][i], s);
            g[i] = f2bf(h2[t][i] != 0.0f ? dy[i] * w3[t] : 0.0f);
            G2s[(rq + i) * TLD + o] = g[i];
        }
        *reinterpret_cast<uint2*>(c.G2T + t0 + o * TT + rq) = pack4(g);
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (l < 16) st[o] = s;
    }
    if (wv == 0) {
        db3 += __shfl_xor(db3, 16, 64);
        db3 += __shfl_xor(db3, 32, 64);
        loss += __shfl_xor(loss, 16, 64);
        loss += __shfl_xor(loss, 32, 64);
        if (l == 0) {
            st[H] = db3;
            st[H + 1] = loss;
        }
    }
    __syncthreads();
    // ---- dH1 = (dH2 W2) [H1 > 0]
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const floatx4 acc = mma_row(G2s, w2t[t]);
        uint16_t g[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) g[i] = f2bf(h1[t][i] != 0 ? acc[i] : 0.0f);
        *reinterpret_cast<uint2*>(c.G1T + t0 + (32 * wv + 16 * t + col) * TT + rq) = pack4(g);
    }
}

struct Adam {
    float *P, *M, *V;
    float lr, b1, b2, eps, c1, c2;
    uint16_t *W1, *W2, *W2T;
};
// what becomes of an entry's gradient: + gin (of earlier launches), then
// stored, or with gout null put through Adam
struct Sink {
    const float* gin;
    float* gout;
    Adam a;

    // what take() needs of entry e, read before the sums
    struct Entry {
        float g, p, m, v;
    };
    __device__ __forceinline__ Entry entry(int e) const {
        Entry n = {0.0f, 0.0f, 0.0f, 0.0f};
        if (gin) n.g = gin[e];
        if (!gout) {
            n.p = a.P[e];
            n.m = a.M[e];
            n.v = a.V[e];
        }
        return n;
    }
    __device__ __forceinline__ void take(int e, const Entry& n, float g) const {
        if (gin) g += n.g;
        if (gout) {
            gout[e] = g;
            return;
        }
        const float m = a.b1 * n.m + (1.0f - a.b1) * g;
        const float v = a.b2 * n.v + (1.0f - a.b2) * g * g;
        a.M[e] = m;
        a.V[e] = v;
        const float p = n.p - a.lr * (m * a.c1) / (sqrtf(v * a.c2) + a.eps);
        a.P[e] = p;
        if (e < OFF_B1) a.W1[e - OFF_W1] = f2bf(p);
        if (e >= OFF_W2 && e < OFF_B2) {
            const int q = e - OFF_W2;
            const uint16_t h = f2bf(p);
            a.W2[q] = h;
            a.W2T[(q % H) * H + q / H] = h;
        }
    }
};

// Workgroups 0-63: tiles of dW1[i][k] = sum_b dH1[b][i] X[b][k]; 64-127: of
// dW2[o][i] = sum_b dH2[b][o] H1[b][i]; those of column 0 also the biases, sums
// of the same rows.  128: dw3, db3 and the loss from the tiles' sums.
// Waves take 32 samples in turn, eight of these in flight.
constexpr int UW = 16;               // waves
constexpr int UPDATE_WGS = 2 * (H / 16) * (H / 16) + 1;
__global__ __launch_bounds__(64 * UW) void k_mlp_update(Chunk c, int tiles, Sink sink, float* __restrict__ loss,
                                                        int add_loss) {
    __shared__ float red[UW][256];
    __shared__ float bred[UW][16];
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63;
    if (blockIdx.x == UPDATE_WGS - 1) {
        // thread (g, o): tiles g, g + 7, ... of sum o; 7 x 130 threads
        const int g = tid / STAT, o = tid % STAT;
        const int e = tid < H ? OFF_W3 + tid : OFF_B3;
        Sink::Entry n = {};
        if (tid <= H) n = sink.entry(e);
        float s = 0.0f;
        if (g < 7) {
#pragma unroll 8
            for (int t = g; t < tiles; t += 7) s += c.stat[(int64_t)t * STAT + o];
        }
        float* r = &red[0][0];
        if (g < 7) r[tid] = s;
        __syncthreads();
        if (tid >= STAT) return;
        for (int q = 1; q < 7; ++q) s += r[q * STAT + tid];
        if (tid <= H) sink.take(e, n, s);
        else *loss = add_loss ? *loss + s : s;
        return;
    }
    const int which = blockIdx.x >> 6, rt = (blockIdx.x >> 3) & 7, ct = blockIdx.x & 7;
    const int at = ((l >> 5) * H + (l & 15)) * TT + ((l >> 4) & 1) * 8;
    const uint16_t* A = (which ? c.G2T : c.G1T) + at + rt * 16 * TT;
    const uint16_t* B = (which ? c.H1T : c.XT) + at + ct * 16 * TT;
    int e = -1;  // the thread's entry
    if (tid < 256) e = (which ? OFF_W2 : OFF_W1) + (rt * 16 + tid / 16) * H + ct * 16 + tid % 16;
    else if (ct == 0 && tid < 256 + 16) e = (which ? OFF_B2 : OFF_B1) + rt * 16 + tid - 256;
    Sink::Entry n = {};
    if (e >= 0) n = sink.entry(e);
    const int steps = (int)(c.ld / 32);
    floatx4 acc = {0, 0, 0, 0};
    float rows = 0.0f;
    constexpr int U = 8;
    for (int s0 = wv; s0 < steps; s0 += UW * U) {
        bf16x8 av[U], bv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = min(s0 + UW * u, steps - 1);
            av[u] = *reinterpret_cast<const bf16x8*>(A + 2 * TT * H * (int64_t)s);
            bv[u] = *reinterpret_cast<const bf16x8*>(B + 2 * TT * H * (int64_t)s);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + UW * u < steps) {
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[u], bv[u], acc, 0, 0, 0);
                if (ct == 0) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) rows += (float)av[u][q];
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wv][(4 * (l >> 4) + i) * 16 + (l & 15)] = acc[i];
    if (ct == 0) {
        rows += __shfl_xor(rows, 16, 64);
        rows += __shfl_xor(rows, 32, 64);
        if (l < 16) bred[wv][l] = rows;
    }
    __syncthreads();
    if (e < 0) return;
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < UW; ++q) s += tid < 256 ? red[q][tid] : bred[q][tid - 256];
    sink.take(e, n, s);
}

// BF16 copies of W1, W2 and W2^T from the FP32 parameters
__global__ void k_mlp_convert(const float* __restrict__ P, uint16_t* __restrict__ W1, uint16_t* __restrict__ W2,
                              uint16_t* __restrict__ W2T) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < H * F) W1[e] = f2bf(P[OFF_W1 + e]);
    if (e < H * H) {
        const uint16_t v = f2bf(P[OFF_W2 + e]);
        W2[e] = v;
        W2T[(e % H) * H + e / H] = v;
    }
}

// Features of FG stencils at a time by one wavefront: lane j = stencil slot j
// (n <= 64; 2 (n - 1) <= 126 entries of the F = 128, the rest zero) for what a
// slot needs, lanes 8 u .. 8 u + 7 = stencil u for what a stencil needs once (the
// roots and quotients of its frame: with all lanes at one stencil they were
// most of 500 instructions per stencil).  Stencils beyond N read stencil N - 1.
constexpr int FG = 8;
struct FeatLds {
    double d1[FG][3];  // offset of the nearest neighbour
    double f[FG][8];   // tau_1, tau_2, 1 / rho
};
// slot l (the centre past n) of stencils s0 ..
__device__ __forceinline__ void load_slots(int64_t N, int n, const int32_t* __restrict__ idx, int64_t s0,
                                           int (&j)[FG]) {
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < FG; ++u) {
        const int64_t s = s0 + u < N ? s0 + u : N - 1;
        j[u] = idx[s * n + (l < n ? l : 0)];
    }
}
// Rows of `ld` entries at out, of `rows` stencils; returns rho of stencil u in lanes 8 u + i.
// Indices outside [0, N) read node 0 and make rho NaN (the proposal is then
// unusable and the weights call flags the stencil).
__device__ __forceinline__ double feature_group(int64_t N, int n, const double* __restrict__ xyz,
                                                const double* __restrict__ nrm, const int (&slot)[FG], FeatLds& lds,
                                                uint16_t* out, int ld, int rows) {
    const int l = threadIdx.x & 63, su = l >> 3;
    double dx[FG], dy[FG], dz[FG], r2[FG];
    uint32_t bad = 0;
    int mine = 0;  // centre of stencil su
#pragma unroll
    for (int u = 0; u < FG; ++u) {
        int j = slot[u];
        const bool out_of_range = j < 0 || j >= N;
        if (out_of_range) j = 0;
        if (__ballot(out_of_range)) bad |= 1u << u;
        dx[u] = xyz[3 * (int64_t)j];
        dy[u] = xyz[3 * (int64_t)j + 1];
        dz[u] = xyz[3 * (int64_t)j + 2];
        const int c = __builtin_amdgcn_readfirstlane(j);
        if (su == u) mine = c;
    }
    double nx = nrm[3 * (int64_t)mine], ny = nrm[3 * (int64_t)mine + 1], nz = nrm[3 * (int64_t)mine + 2];
#pragma unroll
    for (int u = 0; u < FG; ++u) {  // lane 0 holds the centre
        dx[u] = l < n ? dx[u] - first_lane(dx[u]) : 0.0;
        dy[u] = l < n ? dy[u] - first_lane(dy[u]) : 0.0;
        dz[u] = l < n ? dz[u] - first_lane(dz[u]) : 0.0;
        r2[u] = (dx[u] * dx[u] + dy[u] * dy[u]) + dz[u] * dz[u];
        if (l == 1) {
            lds.d1[u][0] = dx[u];
            lds.d1[u][1] = dy[u];
            lds.d1[u][2] = dz[u];
        }
    }
    // eight maxima over the lanes at once: halve the stencils a lane holds
    // while they last
    double r4[4], r1[2];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        r4[u] = fmax(l & 32 ? r2[u + 4] : r2[u], __shfl_xor(l & 32 ? r2[u] : r2[u + 4], 32, 64));
#pragma unroll
    for (int u = 0; u < 2; ++u)
        r1[u] = fmax(l & 16 ? r4[u + 2] : r4[u], __shfl_xor(l & 16 ? r4[u] : r4[u + 2], 16, 64));
    double rr = fmax(l & 8 ? r1[1] : r1[0], __shfl_xor(l & 8 ? r1[0] : r1[1], 8, 64));
#pragma unroll
    for (int m = 4; m > 0; m >>= 1) rr = fmax(rr, __shfl_xor(rr, m, 64));
    const double rho = (bad >> su) & 1 ? NAN : sqrt(rr);
    __syncthreads();
    {
        const double nn = sqrt(nx * nx + ny * ny + nz * nz);
        nx /= nn; ny /= nn; nz /= nn;
        // tau_1: the nearest neighbour's offset projected on the tangent plane
        const double ex = lds.d1[su][0], ey = lds.d1[su][1], ez = lds.d1[su][2];
        const double dn = ex * nx + ey * ny + ez * nz;
        double tx = ex - dn * nx, ty = ey - dn * ny, tz = ez - dn * nz;
        double tn = sqrt(tx * tx + ty * ty + tz * tz);
        if (!(tn > 1e-12 * rho)) {  // degenerate: any tangent direction
            const bool ax = fabs(nx) < 0.9;
            tx = ax ? 0.0 : -nz; ty = ax ? nz : 0.0; tz = ax ? -ny : nx;
            tn = sqrt(tx * tx + ty * ty + tz * tz);
        }
        const double ax = tx / tn, ay = ty / tn, az = tz / tn;
        if ((l & 7) == 0) {
            double* f = lds.f[su];
            f[0] = ax; f[1] = ay; f[2] = az;
            f[3] = ny * az - nz * ay; f[4] = nz * ax - nx * az; f[5] = nx * ay - ny * ax;
            f[6] = 1.0 / rho;
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < FG; ++u) {
        const double* f = lds.f[u];
        uint32_t v = 0;
        if (l >= 1 && l < n) {
            const float sv = (float)((dx[u] * f[0] + dy[u] * f[1] + dz[u] * f[2]) * f[6]);
            const float tv = (float)((dx[u] * f[3] + dy[u] * f[4] + dz[u] * f[5]) * f[6]);
            v = (uint32_t)f2bf(sv) | (uint32_t)f2bf(tv) << 16;
        }
        if (u < rows) *reinterpret_cast<uint32_t*>(out + u * ld + 2 * ((l - 1) & 63)) = v;
    }
    __syncthreads();
    return rho;
}

__global__ __launch_bounds__(64) void k_features(int64_t N, int n, const double* __restrict__ xyz,
                                                 const double* __restrict__ nrm, const int32_t* __restrict__ idx,
                                                 uint16_t* __restrict__ feat, double* __restrict__ rho_out) {
    __shared__ FeatLds lds;
    const int64_t s0 = (int64_t)blockIdx.x * FG;
    int j[FG];
    load_slots(N, n, idx, s0, j);
    const int rows = (int)(N - s0 < FG ? N - s0 : FG);
    const double rho = feature_group(N, n, xyz, nrm, j, lds, feat + s0 * F, F, rows);
    const int l = threadIdx.x;
    if (rho_out && (l & 7) == 0 && (l >> 3) < rows) rho_out[s0 + (l >> 3)] = rho;
}

// Features, network and eps = exp(y) / rho of FR stencils per wavefront; the
// features stay in LDS.  Bound by the gathered coordinates: with nodes in
// random order 53 million cache lines come from behind the L2s, 7.5 TB/s.  N =
// 1e6, n = 50: 0.94 ms; features through memory, a network kernel of four
// wavefronts per 64 samples and an exp kernel took 1.35.
__global__ __launch_bounds__(64) void k_predict(int64_t N, int n, const double* __restrict__ xyz,
                                                const double* __restrict__ nrm, const int32_t* __restrict__ idx,
                                                Bf16Params prm, double* __restrict__ eps) {
    __shared__ __attribute__((aligned(16))) uint16_t X[FR * TLD];
    __shared__ FeatLds lds;
    __shared__ double rhos[FR];
    const int l = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * FR;
    int j[FG], next[FG];
    load_slots(N, n, idx, base, next);
    for (int g = 0; g < FR / FG; ++g) {
#pragma unroll
        for (int u = 0; u < FG; ++u) j[u] = next[u];
        if (g + 1 < FR / FG) load_slots(N, n, idx, base + (g + 1) * FG, next);
        const double rho = feature_group(N, n, xyz, nrm, j, lds, X + g * FG * TLD, TLD, FG);
        if ((l & 7) == 0) rhos[g * FG + (l >> 3)] = rho;
    }
    __syncthreads();
    const float y = forward_rows(X, prm);
    const int b = sample_of(l);
    if ((l & 15) < 8 && base + b < N) eps[base + b] = exp((double)y) / rhos[b];
}

struct MlpScratch {
    uint16_t *W1, *W2, *W2T;
};

int mlp_scratch(rbffd_ctx ctx, size_t extra, MlpScratch& ms, char** extra_ptr) {
    const size_t wbytes = (size_t)(H * F + 2 * H * H) * sizeof(uint16_t);
    int rc = ensure_scratch(ctx, wbytes + extra + 512);
    if (rc) return rc;
    char* base = (char*)ctx->scratch;
    ms.W1 = (uint16_t*)base;
    ms.W2 = ms.W1 + H * F;
    ms.W2T = ms.W2 + H * H;
    if (extra_ptr) *extra_ptr = base + ((wbytes + 255) & ~(size_t)255);
    return RBFFD_OK;
}

size_t chunk_bytes(int64_t batch) {
    const size_t ld = (size_t)((std::min<int64_t>(batch, CHUNK) + 31) & ~(int64_t)31);
    return 4 * ld * H * sizeof(uint16_t) + ld / TT * STAT * sizeof(float);
}

// Gradient and loss of one batch, and with a.P set the Adam step (the
// gradient is then only kept between the launches of a batch above CHUNK).
void batch_step(hipStream_t st, int64_t count, int64_t batch, const Bf16Params& p, const uint16_t* feats,
                const float* target, void* work, uint64_t seed, int64_t step, float* grad, float* loss, const Adam& a) {
    for (int64_t first = 0; first < batch; first += CHUNK) {
        const int64_t ns = std::min<int64_t>(batch - first, CHUNK);
        Chunk c;
        c.ld = (ns + 31) & ~(int64_t)31;
        c.XT = (uint16_t*)work;
        c.H1T = c.XT + c.ld * H;
        c.G1T = c.H1T + c.ld * H;
        c.G2T = c.G1T + c.ld * H;
        c.stat = (float*)(c.G2T + c.ld * H);
        const int tiles = (int)(c.ld / TT);
        hipLaunchKernelGGL(k_mlp_backward, dim3(tiles), dim3(WG), 0, st, count, first, batch, p, feats, target, c,
                           1.0f / (float)batch, seed, step);
        Sink sink;
        sink.gin = first ? grad : nullptr;
        sink.gout = a.P && first + ns == batch ? nullptr : grad;
        sink.a = a;
        hipLaunchKernelGGL(k_mlp_update, dim3(UPDATE_WGS), dim3(64 * UW), 0, st, c, tiles, sink, loss, first != 0);
    }
}

void convert(hipStream_t st, const float* P, const MlpScratch& ms) {
    hipLaunchKernelGGL(k_mlp_convert, dim3((H * F + 255) / 256), dim3(256), 0, st, P, ms.W1, ms.W2, ms.W2T);
}

}  // namespace

extern "C" int rbffd_mlp_features(rbffd_ctx ctx, int64_t N, const double* xyz, const double* nrm,
                                  const int32_t* idx, int32_t n, uint16_t* feats, double* rho) {
    if (!ctx) return RBFFD_E_ARG;
    if (N < 0) return set_error(ctx, RBFFD_E_ARG, "N < 0");
    if (N == 0) return RBFFD_OK;
    if (n < 2 || n > 64) return set_error(ctx, RBFFD_E_ARG, "features need 2 <= n <= 64 (one lane per slot)");
    if (!xyz || !nrm || !idx || !feats) return set_error(ctx, RBFFD_E_ARG, "null pointer");
    hipLaunchKernelGGL(k_features, dim3((unsigned)((N + FG - 1) / FG)), dim3(64), 0, ctx->stream, N, n,
                       xyz, nrm, idx, feats, rho);
    HIP_TRY(ctx, hipGetLastError());
    return RBFFD_OK;
}

extern "C" int rbffd_mlp_forward(rbffd_ctx ctx, const float* params, int64_t B, const uint16_t* feats, float* y) {
    if (!ctx) return RBFFD_E_ARG;
    if (B < 0) return set_error(ctx, RBFFD_E_ARG, "B < 0");
    if (B == 0) return RBFFD_OK;
    if (!params || !feats || !y) return set_error(ctx, RBFFD_E_ARG, "null pointer");
    MlpScratch ms;
    int rc = mlp_scratch(ctx, 0, ms, nullptr);
    if (rc) return rc;
    convert(ctx->stream, params, ms);
    Bf16Params p{ms.W1, ms.W2, ms.W2T, params};
    hipLaunchKernelGGL(k_mlp, dim3((unsigned)((B + FR - 1) / FR)), dim3(64), 0, ctx->stream, B, p, feats, y);
    HIP_TRY(ctx, hipGetLastError());
    return RBFFD_OK;
}

extern "C" int rbffd_mlp_grad(rbffd_ctx ctx, const float* params, int64_t B, const uint16_t* feats,
                              const float* target, float* grad, float* loss) {
    if (!ctx) return RBFFD_E_ARG;
    if (B <= 0) return set_error(ctx, RBFFD_E_ARG, "B must be > 0");
    if (!params || !feats || !target || !grad || !loss) return set_error(ctx, RBFFD_E_ARG, "null pointer");
    MlpScratch ms;
    char* extra = nullptr;
    int rc = mlp_scratch(ctx, chunk_bytes(B), ms, &extra);
    if (rc) return rc;
    convert(ctx->stream, params, ms);
    Bf16Params p{ms.W1, ms.W2, ms.W2T, params};
    batch_step(ctx->stream, B, B, p, feats, target, extra, 0, 0, grad, loss, Adam{});
    HIP_TRY(ctx, hipGetLastError());
    return RBFFD_OK;
}

extern "C" int rbffd_mlp_train(rbffd_ctx ctx, float* params, float* adam_m, float* adam_v, int64_t count,
                               const uint16_t* feats, const float* target, const rbffd_train_opts* o,
                               float* loss_per_step) {
    if (!ctx) return RBFFD_E_ARG;
    if (!o || !params || !adam_m || !adam_v || !feats || !target) return set_error(ctx, RBFFD_E_ARG, "null pointer");
    if (count <= 0 || o->batch <= 0 || o->batch % TB != 0 || o->steps < 0)
        return set_error(ctx, RBFFD_E_ARG, "count > 0, batch a positive multiple of %d, steps >= 0 required", TB);
    if (o->seed == 0) return set_error(ctx, RBFFD_E_ARG, "seed must be non-zero");
    MlpScratch ms;
    char* extra = nullptr;
    const size_t gbytes = ((RBFFD_MLP_PARAMS + 1) * sizeof(float) + 255) & ~(size_t)255;  // a gradient and a loss
    int rc = mlp_scratch(ctx, gbytes + chunk_bytes(o->batch), ms, &extra);
    if (rc) return rc;
    float* grad = (float*)extra;
    hipStream_t st = ctx->stream;
    convert(st, params, ms);
    Bf16Params p{ms.W1, ms.W2, ms.W2T, params};
    for (int64_t s = 0; s < o->steps; ++s) {
        const double t = (double)(o->step0 + s + 1);
        const Adam a{params,
                     adam_m,
                     adam_v,
                     (float)o->lr,
                     (float)o->beta1,
                     (float)o->beta2,
                     (float)o->adam_eps,
                     (float)(1.0 / (1.0 - pow(o->beta1, t))),
                     (float)(1.0 / (1.0 - pow(o->beta2, t))),
                     ms.W1,
                     ms.W2,
                     ms.W2T};
        batch_step(st, count, o->batch, p, feats, target, extra + gbytes, o->seed, o->step0 + s, grad,
                   loss_per_step ? loss_per_step + s : grad + RBFFD_MLP_PARAMS, a);
    }
    HIP_TRY(ctx, hipGetLastError());
    return RBFFD_OK;
}

extern "C" int rbffd_predict_eps(rbffd_ctx ctx, const float* params, int64_t N, const double* xyz,
                                 const double* nrm, const int32_t* idx, int32_t n, double* eps) {
    if (!ctx) return RBFFD_E_ARG;
    if (N < 0) return set_error(ctx, RBFFD_E_ARG, "N < 0");
    if (N == 0) return RBFFD_OK;
    if (!params || !xyz || !nrm || !idx || !eps) return set_error(ctx, RBFFD_E_ARG, "null pointer");
    if (n < 2 || n > 64) return set_error(ctx, RBFFD_E_ARG, "features need 2 <= n <= 64 (one lane per slot)");
    MlpScratch ms;
    int rc = mlp_scratch(ctx, 0, ms, nullptr);
    if (rc) return rc;
    hipStream_t st = ctx->stream;
    convert(st, params, ms);
    Bf16Params p{ms.W1, ms.W2, ms.W2T, params};
    hipLaunchKernelGGL(k_predict, dim3((unsigned)((N + FR - 1) / FR)), dim3(64), 0, st, N, n, xyz, nrm, idx, p, eps);
    HIP_TRY(ctx, hipGetLastError());
    return RBFFD_OK;
}
