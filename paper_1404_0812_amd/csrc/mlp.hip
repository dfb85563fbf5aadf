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

constexpr int TB = 64;        // samples per workgroup tile
constexpr int WG = 256;       // 4 waves

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

// One 16x16 output tile over K (multiple of 32): A rows at a (stride lda), B rows at b (stride ldb).
__device__ __forceinline__ void mma_tile(const uint16_t* a, int lda, const uint16_t* b, int ldb, int K,
                                         floatx4& acc) {
    const int l = threadIdx.x & 63;
    const int r = l & 15, kq = (l >> 4) * 8;
    for (int k0 = 0; k0 < K; k0 += 32) {
        const bf16x8 av = *reinterpret_cast<const bf16x8*>(a + (size_t)r * lda + k0 + kq);
        const bf16x8 bv = *reinterpret_cast<const bf16x8*>(b + (size_t)r * ldb + k0 + kq);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc, 0, 0, 0);
    }
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

// Forward over one tile of TB samples: y.
__global__ __launch_bounds__(WG) void k_mlp(int64_t count, Bf16Params prm, const uint16_t* __restrict__ x,
                                            float* __restrict__ y) {
    __shared__ __attribute__((aligned(16))) uint16_t Xs[TB * F];   // [b][k]
    __shared__ __attribute__((aligned(16))) uint16_t H1s[TB * H];  // [b][i]
    __shared__ float ys[TB];
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63;
    const int64_t base = (int64_t)blockIdx.x * TB;
    // ---- load the input tile (zeros beyond count)
    for (int e = tid; e < TB * F / 8; e += WG) {
        const int b = e / (F / 8), k8 = (e % (F / 8)) * 8;
        const int64_t rr = base + b;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (rr < count) v = *reinterpret_cast<const uint4*>(x + rr * F + k8);
        *reinterpret_cast<uint4*>(Xs + b * F + k8) = v;
    }
    __syncthreads();
    const int r0 = wv * 16;              // this wave's 16 sample rows
    const int col = l & 15, rq = (l >> 4) * 4;
    // ---- layer 1: H1 = relu(X W1^T + b1)
    for (int ct = 0; ct < H / 16; ++ct) {
        floatx4 acc = {0, 0, 0, 0};
        mma_tile(Xs + r0 * F, F, prm.W1 + ct * 16 * F, F, F, acc);
        const int o = ct * 16 + col;
        const float bb = prm.P[OFF_B1 + o];
#pragma unroll
        for (int i = 0; i < 4; ++i) H1s[(r0 + rq + i) * H + o] = f2bf(fmaxf(acc[i] + bb, 0.0f));
    }
    __syncthreads();
    // ---- layer 2: H2 = relu(H1 W2^T + b2); layer 3: y = H2 . w3 + b3
    float part[4] = {0, 0, 0, 0};
    for (int ct = 0; ct < H / 16; ++ct) {
        floatx4 acc = {0, 0, 0, 0};
        mma_tile(H1s + r0 * H, H, prm.W2 + ct * 16 * H, H, H, acc);
        const int o = ct * 16 + col;
        const float bb = prm.P[OFF_B2 + o], w3 = prm.P[OFF_W3 + o];
#pragma unroll
        for (int i = 0; i < 4; ++i) part[i] = fmaf(bf2f(f2bf(fmaxf(acc[i] + bb, 0.0f))), w3, part[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) part[i] += __shfl_xor(part[i], m, 64);
    }
    if (col == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) ys[r0 + rq + i] = part[i] + prm.P[OFF_B3];
    }
    __syncthreads();
    if (tid < TB && base + tid < count) y[base + tid] = ys[tid];
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
constexpr int TLD = F + 8;           // row stride of the LDS tiles: rows start 4 banks apart
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

// Features: one wavefront per FEAT_SPW consecutive stencils, lane j = stencil
// slot j (n <= 64; 2 (n - 1) <= 126 entries of the F = 128, the rest zero).  The loads of all of them are issued before any is used (stencils
// beyond N read stencil N - 1 and write nothing), so each wavefront has
// FEAT_SPW round trips to memory in flight instead of one.
constexpr int FEAT_SPW = 4;
__global__ __launch_bounds__(64) void k_features(int64_t N, int n, const double* __restrict__ xyz,
                                                 const double* __restrict__ nrm, const int32_t* __restrict__ idx,
                                                 uint16_t* __restrict__ feat, double* __restrict__ rho_out) {
    __shared__ double t1s[FEAT_SPW][3];
    const int l = threadIdx.x;
    const int64_t s0 = (int64_t)blockIdx.x * FEAT_SPW;
    double dx[FEAT_SPW], dy[FEAT_SPW], dz[FEAT_SPW], nx[FEAT_SPW], ny[FEAT_SPW], nz[FEAT_SPW], rho[FEAT_SPW];
    // indices outside [0, N) read node 0 and make rho NaN (the proposal is then
    // unusable and the weights call flags the stencil)
#pragma unroll
    for (int u = 0; u < FEAT_SPW; ++u) {
        const int64_t s = s0 + u < N ? s0 + u : N - 1;
        int c = idx[s * n];
        bool bad = c < 0 || c >= N;
        if (bad) c = 0;
        int j = l < n ? idx[s * n + l] : c;
        if (j < 0 || j >= N) {
            bad = true;
            j = 0;
        }
        const double cx = xyz[3 * (int64_t)c], cy = xyz[3 * (int64_t)c + 1], cz = xyz[3 * (int64_t)c + 2];
        const double px = xyz[3 * (int64_t)j], py = xyz[3 * (int64_t)j + 1], pz = xyz[3 * (int64_t)j + 2];
        dx[u] = l < n ? px - cx : 0.0;
        dy[u] = l < n ? py - cy : 0.0;
        dz[u] = l < n ? pz - cz : 0.0;
        nx[u] = nrm[3 * (int64_t)c];
        ny[u] = nrm[3 * (int64_t)c + 1];
        nz[u] = nrm[3 * (int64_t)c + 2];
        double r2 = (dx[u] * dx[u] + dy[u] * dy[u]) + dz[u] * dz[u];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) r2 = fmax(r2, __shfl_xor(r2, o, 64));
        const bool any_bad = __ballot(bad) != 0;
        rho[u] = any_bad ? NAN : sqrt(r2);
        const double nn = sqrt(nx[u] * nx[u] + ny[u] * ny[u] + nz[u] * nz[u]);
        nx[u] /= nn; ny[u] /= nn; nz[u] /= nn;
        if (l == 1) {
            // tau_1: the nearest neighbour's offset projected on the tangent plane
            const double dn = dx[u] * nx[u] + dy[u] * ny[u] + dz[u] * nz[u];
            double tx = dx[u] - dn * nx[u], ty = dy[u] - dn * ny[u], tz = dz[u] - dn * nz[u];
            double tn = sqrt(tx * tx + ty * ty + tz * tz);
            if (!(tn > 1e-12 * rho[u])) {  // degenerate: any tangent direction
                const bool ax = fabs(nx[u]) < 0.9;
                tx = ax ? 0.0 : -nz[u]; ty = ax ? nz[u] : 0.0; tz = ax ? -ny[u] : nx[u];
                tn = sqrt(tx * tx + ty * ty + tz * tz);
            }
            t1s[u][0] = tx / tn; t1s[u][1] = ty / tn; t1s[u][2] = tz / tn;
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < FEAT_SPW; ++u) {
        const int64_t s = s0 + u;
        if (s >= N) break;
        const double ax = t1s[u][0], ay = t1s[u][1], az = t1s[u][2];
        const double bx = ny[u] * az - nz[u] * ay, by = nz[u] * ax - nx[u] * az, bz = nx[u] * ay - ny[u] * ax;
        uint16_t* f = feat + s * F;
        if (l >= 1 && l < n) {
            const float sv = (float)((dx[u] * ax + dy[u] * ay + dz[u] * az) / rho[u]);
            const float tv = (float)((dx[u] * bx + dy[u] * by + dz[u] * bz) / rho[u]);
            f[2 * (l - 1)] = f2bf(sv);
            f[2 * (l - 1) + 1] = f2bf(tv);
        }
        for (int k = 2 * (n - 1) + l; k < F; k += 64) f[k] = 0;
        if (l == 0 && rho_out) rho_out[s] = rho[u];
    }
}

__global__ void k_eps_from_y(int64_t N, const float* __restrict__ y, const double* __restrict__ rho,
                             double* __restrict__ eps) {
    const int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (s < N) eps[s] = exp((double)y[s]) / rho[s];
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
    hipLaunchKernelGGL(k_features, dim3((unsigned)((N + FEAT_SPW - 1) / FEAT_SPW)), dim3(64), 0, ctx->stream, N, n,
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
    hipLaunchKernelGGL(k_mlp, dim3((unsigned)((B + TB - 1) / TB)), dim3(WG), 0, ctx->stream, B, p, feats, y);
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
    char* extra = nullptr;
    const size_t fbytes = (size_t)N * F * sizeof(uint16_t);
    const size_t rbytes = (size_t)N * sizeof(double), ybytes = (size_t)N * sizeof(float);
    int rc = mlp_scratch(ctx, fbytes + rbytes + ybytes + 1024, ms, &extra);
    if (rc) return rc;
    uint16_t* feats = (uint16_t*)extra;
    double* rho = (double*)(extra + ((fbytes + 255) & ~(size_t)255));
    float* y = (float*)((char*)rho + ((rbytes + 255) & ~(size_t)255));
    hipStream_t st = ctx->stream;
    hipLaunchKernelGGL(k_features, dim3((unsigned)((N + FEAT_SPW - 1) / FEAT_SPW)), dim3(64), 0, st, N, n, xyz, nrm,
                       idx, feats, rho);
    convert(st, params, ms);
    Bf16Params p{ms.W1, ms.W2, ms.W2T, params};
    hipLaunchKernelGGL(k_mlp, dim3((unsigned)((N + TB - 1) / TB)), dim3(WG), 0, st, N, p, feats, y);
    hipLaunchKernelGGL(k_eps_from_y, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, N, y, rho, eps);
    HIP_TRY(ctx, hipGetLastError());
    return RBFFD_OK;
}
