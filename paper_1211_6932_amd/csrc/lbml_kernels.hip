// lbml_kernels.hip -- gfx950 kernels of the learned droplet initialiser: a
// 4 -> 256 -> 256 -> 256 -> 128 MLP with bf16 matrix-core products (FP32
// accumulation, FP32 master weights, Adam), plus the two profile kernels that
// connect it to the lattice (radial log-density samples <-> density field).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "lbml_launch.hpp"

namespace lbml {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// C[M][N] (FP32, row stride ldc) = sum_k A(m, k) B(k, n) with A(m, k) at
// A[m * sam + k * sak] and B(k, n) at B[k * sbk + n * sbn] (bf16).  One
// wavefront per 16 x 16 tile of C, K consumed 32 at a time by
// v_mfma_f32_16x16x32_bf16 (behind lbml_gemm_bf16 alone: the network's kernels below multiply
// operands in fragment order): lane l holds row (or column) l % 16 and the eight
// consecutive k values 8 (l / 16) .. 8 (l / 16) + 7 of each operand; the
// accumulator holds rows 4 (l / 16) .. 4 (l / 16) + 3 of column l % 16.
// AV / BV: the operand is contiguous in k (sak == 1 / sbk == 1) with 16-byte
// aligned rows, so a lane's eight k values are one 16-byte load; otherwise eight
// 2-byte loads.  Either way the matrix cores see the same values.
// M, N multiples of 16 and K a multiple of 32 (checked by the launcher).
template <bool AV, bool BV>
__global__ __launch_bounds__(256) void gemm_bf16(const __bf16* __restrict__ A, long long sam,
                                                 long long sak, const __bf16* __restrict__ B,
                                                 long long sbk, long long sbn, float* __restrict__ C,
                                                 int ldc, int M, int N, int K)
{
    const int lane = threadIdx.x & 63;
    const int tile = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tiles_n = N / 16;
    if (tile >= (M / 16) * tiles_n) return;
    const int m0 = (tile / tiles_n) * 16, n0 = (tile % tiles_n) * 16;
    const int r = lane & 15, kq = (lane >> 4) * 8;
    const __bf16* arow = A + (long long)(m0 + r) * sam;
    const __bf16* bcol = B + (long long)(n0 + r) * sbn;
    floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = 0; k0 < K; k0 += 32) {
        bf16x8 a, b;
        if constexpr (AV) {
            a = *reinterpret_cast<const bf16x8*>(arow + k0 + kq);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) a[i] = arow[(long long)(k0 + kq + i) * sak];
        }
        if constexpr (BV) {
            b = *reinterpret_cast<const bf16x8*>(bcol + k0 + kq);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) b[i] = bcol[(long long)(k0 + kq + i) * sbk];
        }
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) C[(long long)(m0 + (lane >> 4) * 4 + i) * ldc + n0 + r] = acc[i];
}

// GELU and its derivative from z and e = erf(z / sqrt 2).
__device__ __forceinline__ float gelu_erf(float z) { return erff(z * 0.70710678118654752f); }
__device__ __forceinline__ float gelu(float z, float e) { return 0.5f * z * (1.0f + e); }
__device__ __forceinline__ float gelu_prime(float z, float e)
{
    return 0.5f * (1.0f + e) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

__global__ void fill_zero(unsigned int* __restrict__ p, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// ---------------------------------------------------------------- the network
// A pass over a batch is bound by latency, not by arithmetic (0.33 MFLOP a sample forward)
// or bytes (0.33 MB of bf16 weights), so it is two launches: mlp_pass takes 16 rows of the
// batch per workgroup through every layer, forward and, in training, back to the first
// layer's pre-activation gradients; mlp_grads forms every weight and bias gradient from what
// that left behind and, in a training loop, applies Adam to them on the spot.  512 rows:
// 11.1 + 6.2 us in a training loop, where one launch per operation (32 of them) took 115 us and
// the gaps (159 us a training step, now 21.5 us).
// Products use the matrix cores as gemm_bf16 does (same operand orientation, one accumulator
// over k in steps of 32), whichever launch they are in.

// Layers i = 0 .. 3: inputs (padded), outputs, offset of the weights in the parameter vector
// (the biases follow them).
__device__ constexpr int kLayerIn[4] = {kIn, kHidden, kHidden, kHidden};
__device__ constexpr int kLayerPad[4] = {kInPad, kHidden, kHidden, kHidden};
__device__ constexpr int kLayerOut[4] = {kHidden, kHidden, kHidden, kOut};
constexpr int kMlpThreads = 1024;
constexpr int kMlpLd = kHidden + 8;  // LDS row: 16 rows at 16 bytes fall on different banks

// Every matrix operand is stored in fragment order: element (n, k) of an [..][K] matrix lies
// where the lane that feeds it to a 16 x 16 x 32 product reads it, so that a wavefront's load
// is one stretch of 1 KB (rows of the matrix would give it 64-byte pieces of 16 rows: 7000
// cycles for the 128 KB of a layer; the pass over 512 rows takes 24 us that way, 11.8 us in
// fragment order).
__device__ __forceinline__ long long frag_at(int n, int k, int K)
{
    return ((long long)((n >> 4) * (K >> 5) + (k >> 5)) * 64 + (n & 15) + ((k & 31) >> 3) * 16) * 8 + (k & 7);
}

// Fragments of the right operand for the 16 output columns from n0 on.
template <int K>
__device__ __forceinline__ void load_frags(bf16x8 (&f)[8], const __bf16* __restrict__ W, int n0, int lane)
{
    const bf16x8* from = reinterpret_cast<const bf16x8*>(W) + (long long)(n0 >> 4) * (K / 32) * 64 + lane;
#pragma unroll
    for (int s = 0; s < K / 32; ++s) f[s] = from[64 * s];
}

// The wave's 16 x 16 tile of (LDS rows) x (fragments).
template <int K>
__device__ __forceinline__ floatx4 tile_product(const __bf16 (&A)[16][kMlpLd], const bf16x8 (&f)[8], int lane)
{
    floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < K / 32; ++s) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&A[lane & 15][32 * s + (lane >> 4) * 8]);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, f[s], acc, 0, 0, 0);
    }
    return acc;
}

// R values of one column into the LDS rows and into T (fragments along the batch).
template <int R>
__device__ __forceinline__ void put_column(__bf16 (&A)[16][kMlpLd], __bf16* __restrict__ T, int B, int m0, int col,
                                           int lane, const __bf16 (&v)[R])
{
    const int q = lane >> 4;
#pragma unroll
    for (int j = 0; j < R; ++j) A[4 * q + j][col] = v[j];
    if (T) {
        typedef __bf16 bf16r __attribute__((ext_vector_type(R)));
        bf16r w;
#pragma unroll
        for (int j = 0; j < R; ++j) w[j] = v[j];
        *reinterpret_cast<bf16r*>(T + frag_at(col, m0 + R * q, B)) = w;
    }
}

// One workgroup: 4 R rows of the batch.  A matrix-core tile has 16 rows, four per lane group;
// R of the four are used, because the activation functions (an erf each, on the vector unit)
// cost more than the products: with fewer rows per workgroup more compute units share them.
// Wave w holds output columns 16 w .. 16 w + 15 of every layer, so the pre-activations that
// the backward pass needs stay in its registers; layer inputs and gradients pass between
// waves through LDS; a layer's weights are requested while the layer before is computed.
// TRAIN: the layer inputs (x16, h) and pre-activation gradients dz are written in
// fragments along the batch for mlp_grads, and the workgroup's loss sum.
template <bool TRAIN, int R>
__global__ __launch_bounds__(kMlpThreads) void mlp_pass(MlpArgs a)
{
    __shared__ __align__(16) __bf16 A[2][16][kMlpLd];
    __shared__ float wave_loss[kOut / 16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = blockIdx.x * 4 * R, n0 = wave * 16, col = n0 + (lane & 15), q = lane >> 4;
    const int B = a.B;
    const bool last = wave < kOut / 16;  // has columns of the output layer
    bf16x8 wf[8], wn[8];
    load_frags<kInPad>(wf, a.w[0], n0, lane);
    load_frags<kHidden>(wn, a.w[1], n0, lane);
    // every load the epilogues need is requested here: a load issued after a later layer's
    // weights would have to wait for them (loads return in order)
    float bias[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) bias[i] = i < 3 || last ? a.bias[i][col] : 0.0f;
    const int* idx = a.idx ? a.idx + (long long)a.sc->next * B : nullptr;
    auto source = [&](int m) __attribute__((always_inline)) { return (long long)(idx ? idx[m] : m); };
    if (tid < 4 * R * kInPad) {
        const int m = tid / kInPad, k = tid % kInPad;
        const __bf16 v = static_cast<__bf16>(k < kIn ? (a.x[source(m0 + m) * kIn + k] - a.norm[k]) * a.norm[kIn + k] : 0.0f);
        A[0][4 * (m / R) + m % R][k] = v;
        if (TRAIN && k < kIn) a.xT[frag_at(k, m0 + m, B)] = v;
    }
    // the output layer's base and target, requested long before they are needed
    float yb[R], yt[R];
#pragma unroll
    for (int j = 0; j < R; ++j) yb[j] = yt[j] = 0.0f;
    if (last) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const long long at = source(m0 + R * q + j) * kOut + col;
            if (a.base) yb[j] = a.base[at];
            if (TRAIN) yt[j] = a.target[at];
        }
    }
    __syncthreads();

    float z0[R], z1[R], z2[R], e0[R], e1[R], e2[R];
    // a hidden layer's epilogue: z = c + b, h = bf16(GELU(z)) into the other LDS buffer
    auto hidden = [&](const floatx4 acc, const float b, float (&z)[R], float (&e)[R], const int to, __bf16* hT)
                      __attribute__((always_inline)) {
        __bf16 h[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            z[j] = acc[j] + b;
            e[j] = gelu_erf(z[j]);
            h[j] = static_cast<__bf16>(gelu(z[j], e[j]));
        }
        put_column<R>(A[to], TRAIN ? hT : nullptr, B, m0, col, lane, h);
        __syncthreads();
    };
    hidden(tile_product<kInPad>(A[0], wf, lane), bias[0], z0, e0, 1, a.hT[0]);
    load_frags<kHidden>(wf, a.w[2], n0, lane);
    hidden(tile_product<kHidden>(A[1], wn, lane), bias[1], z1, e1, 0, a.hT[1]);
    if (last) load_frags<kHidden>(wn, a.w[3], n0, lane);
    hidden(tile_product<kHidden>(A[0], wf, lane), bias[2], z2, e2, 1, a.hT[2]);
    if (TRAIN) load_frags<kOut>(wf, a.wt[3], n0, lane);

    float loss = 0.0f;
    if (last) {
        const floatx4 acc = tile_product<kHidden>(A[1], wn, lane);
        const float b = bias[3];
        const float scale = 2.0f / (float)(B * kOut);
        __bf16 dy[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            float z = acc[j] + b;
            if (a.base) z += yb[j];
            if (TRAIN) {
                // dY = bf16(2 (Y - T) / (B N)); loss = mean (Y - T)^2
                const float d = z - yt[j];
                dy[j] = static_cast<__bf16>(scale * d);
                loss += d * d;
            } else {
                a.y[(long long)(m0 + R * q + j) * kOut + col] = z;
            }
        }
        if (TRAIN) {
            put_column<R>(A[0], a.dzT[3], B, m0, col, lane, dy);
            for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
            if (lane == 0) wave_loss[wave] = loss;
        }
    }
    if (!TRAIN) return;
    __syncthreads();
    if (tid == 0) {
        float sum = 0.0f;
        for (int w = 0; w < kOut / 16; ++w) sum += wave_loss[w];
        a.loss_part[blockIdx.x] = sum;
    }

    // dZ_{i-1} = bf16((dZ_i W_i) * GELU'(Z_{i-1}))
    auto back = [&](const floatx4 acc, const float (&z)[R], const float (&e)[R], const int to, __bf16* dzT)
                    __attribute__((always_inline)) {
        __bf16 dz[R];
#pragma unroll
        for (int j = 0; j < R; ++j) dz[j] = static_cast<__bf16>(acc[j] * gelu_prime(z[j], e[j]));
        put_column<R>(A[to], dzT, B, m0, col, lane, dz);
        __syncthreads();
    };
    load_frags<kHidden>(wn, a.wt[2], n0, lane);
    back(tile_product<kOut>(A[0], wf, lane), z2, e2, 1, a.dzT[2]);
    load_frags<kHidden>(wf, a.wt[1], n0, lane);
    back(tile_product<kHidden>(A[1], wn, lane), z1, e1, 0, a.dzT[1]);
    back(tile_product<kHidden>(A[0], wf, lane), z0, e0, 1, a.dzT[0]);

    // the schedule of a training loop: learning rate and bias corrections of this step (FP64
    // running powers of b1, b2, as the host keeps them); mlp_grads counts the step
    if (a.sc && blockIdx.x == 0 && tid == 0) {
        TrainSched* sc = a.sc;
        const int s = sc->next;
        sc->cur = s;
        sc->p1 *= a.b1;
        sc->p2 *= a.b2;
        sc->lr = a.lr[s];
        sc->c1 = (float)(1.0 - sc->p1);
        sc->c2 = (float)(1.0 - sc->p2);
    }
}

// Adam on one FP32 master parameter; returns its new value.  c1, c2: the bias corrections
// 1 - b1^t, 1 - b2^t.
struct AdamState { float p, m, v; };

__device__ __forceinline__ float adam_update(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                                             const AdamState old, float gi, int i, float lr, float b1, float b2,
                                             float eps, float c1, float c2)
{
    const float mi = b1 * old.m + (1.0f - b1) * gi;
    const float vi = b2 * old.v + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = old.p - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    return pi;
}

__global__ void adam(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                     const float* __restrict__ g, int n, float lr, float b1, float b2, float eps, float c1,
                     float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) adam_update(p, m, v, AdamState{p[i], m[i], v[i]}, g[i], i, lr, b1, b2, eps, c1, c2);
}

// Gradients of every parameter from the batch's layer inputs and pre-activation gradients
// (fragments along the batch).  One wavefront per
// 16 x 16 tile of a dW_i = dZ_i^T H_{i-1} (of the first layer's only the four columns of real
// inputs are kept), then wavefronts of 64 bias gradients (sums over the batch in row order), then one
// that sums up the loss.  ADAM: the update of the same parameters, the learning rate and
// bias corrections from the schedule, and both bf16 copies of the weights.
constexpr int kTiles3 = (kOut / 16) * (kHidden / 16), kTiles12 = (kHidden / 16) * (kHidden / 16), kTiles0 = kHidden / 16;
constexpr int kTilesAll = kTiles3 + 2 * kTiles12 + kTiles0;
constexpr int kBiases = 3 * kHidden + kOut;
constexpr int kGradWaves = kTilesAll + kBiases / 64 + 1;
// Steps of 32 rows of the batch in one block of straight code.  Its 96 registers do not hold 16
// steps' operands: the first product waits for eight loads, and about ten are in flight.  Rows
// beyond a multiple of 512 take one step at a time (64 rows 3.6 us, 160 4.4, 480 8.1, 512 8.2,
// 1024 13.8; gradients only).
constexpr int kGradAhead = 16;
constexpr int kBiasAhead = 4;    // the same for the bias gradients
constexpr int kBiasLd = 32 + 8;

template <bool ADAM>
__global__ __launch_bounds__(256) void mlp_grads(GradArgs g)
{
    __shared__ __align__(16) __bf16 sh[4][64][kBiasLd];
    const int lane = threadIdx.x & 63;
    int t = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int B = g.B;
    float lr = 0.0f, c1 = 1.0f, c2 = 1.0f;
    if (ADAM) {
        lr = g.sc->lr;
        c1 = g.sc->c1;
        c2 = g.sc->c2;
    }
    if (t < kTilesAll) {
        const int i = t < kTiles3 ? 3 : t < kTiles3 + kTiles12 ? 2 : t < kTiles3 + 2 * kTiles12 ? 1 : 0;
        t -= i == 3 ? 0 : i == 2 ? kTiles3 : i == 1 ? kTiles3 + kTiles12 : kTiles3 + 2 * kTiles12;
        const int across = i == 0 ? 1 : kHidden / 16;
        const int tm = (t / across) * 16, tn = (t % across) * 16;
        const bf16x8* arow = reinterpret_cast<const bf16x8*>(g.dzT[i] + frag_at(tm, 0, B)) + lane;
        const bf16x8* brow = reinterpret_cast<const bf16x8*>(g.inT[i] + frag_at(tn, 0, B)) + lane;
        // the parameters and moments of this tile, requested with the first operands
        const int c = tn + (lane & 15);
        const bool kept = c < kLayerIn[i];
        const int p0 = g.w_off[i] + (tm + (lane >> 4) * 4) * kLayerIn[i] + c;
        AdamState old[4];
        if (ADAM && kept) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int p = p0 + j * kLayerIn[i];
                old[j] = AdamState{g.theta[p], g.m[p], g.v[p]};
            }
        }
        floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        int k0 = 0;
        for (; k0 + 32 * kGradAhead <= B; k0 += 32 * kGradAhead) {
            bf16x8 x[kGradAhead], y[kGradAhead];
#pragma unroll
            for (int s = 0; s < kGradAhead; ++s) {
                x[s] = arow[2 * k0 + 64 * s];
                y[s] = brow[2 * k0 + 64 * s];
            }
#pragma unroll
            for (int s = 0; s < kGradAhead; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[s], y[s], acc, 0, 0, 0);
        }
        for (; k0 < B; k0 += 32)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(arow[2 * k0], brow[2 * k0], acc, 0, 0, 0);
        if (!kept) return;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = tm + (lane >> 4) * 4 + j;
            const int p = p0 + j * kLayerIn[i];
            g.grad[p] = acc[j];
            if (ADAM) {
                const __bf16 w =
                    static_cast<__bf16>(adam_update(g.theta, g.m, g.v, old[j], acc[j], p, lr, g.b1, g.b2, g.eps, c1, c2));
                g.w[i][frag_at(r, c, kLayerPad[i])] = w;
                if (i > 0) g.wt[i][frag_at(c, r, kLayerOut[i])] = w;
            }
        }
        return;
    }
    t -= kTilesAll;
    if (t < kBiases / 64) {
        const int n = t * 64 + lane;
        const int i = n / kHidden, c = n % kHidden;  // 0 .. 3: three hidden layers, then the output
        const int p = g.w_off[i] + kLayerOut[i] * kLayerIn[i] + c;
        AdamState old{};
        if (ADAM) old = AdamState{g.theta[p], g.m[p], g.v[p]};
        // 32 rows of the batch at a time: the fragments of the 64 columns, turned around in LDS,
        // then added by the column's lane in row order
        const int i64 = (t * 64) / kHidden, c64 = (t * 64) % kHidden;
        const bf16x8* from = reinterpret_cast<const bf16x8*>(g.dzT[i64] + frag_at(c64, 0, B)) + lane;
        __bf16(*turn)[kBiasLd] = sh[threadIdx.x >> 6];
        float acc = 0.0f;
        for (int m = 0; m < B; m += 32 * kBiasAhead) {
            bf16x8 x[kBiasAhead][4];
#pragma unroll
            for (int s = 0; s < kBiasAhead; ++s)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (m + 32 * s < B) x[s][u] = from[(long long)u * (B >> 5) * 64 + 2 * m + 64 * s];
#pragma unroll
            for (int s = 0; s < kBiasAhead; ++s) {
                if (m + 32 * s >= B) break;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    *reinterpret_cast<bf16x8*>(&turn[16 * u + (lane & 15)][(lane >> 4) * 8]) = x[s][u];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bf16x8 w = *reinterpret_cast<const bf16x8*>(&turn[lane][8 * u]);
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc += static_cast<float>(w[j]);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
        g.grad[p] = acc;
        if (ADAM) adam_update(g.theta, g.m, g.v, old, acc, p, lr, g.b1, g.b2, g.eps, c1, c2);
        return;
    }
    if (t == kBiases / 64) {
        float sum = 0.0f;
        for (int q = lane; q < g.parts; q += 64) sum += g.loss_part[q];
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if (lane == 0) {
            const float loss = sum / (float)(B * kOut);
            g.loss[0] = loss;
            if (ADAM) {
                if (g.loss_out) g.loss_out[g.sc->cur] = loss;
                g.sc->next += 1;
            }
        }
    }
}

// flag[0] = 1 if some idx[j], j < n, lies outside [0, rows).
__global__ void check_rows(const int* __restrict__ idx, long long n, int rows, int* __restrict__ flag)
{
    for (long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (long long)gridDim.x * blockDim.x)
        if (idx[j] < 0 || idx[j] >= rows) flag[0] = 1;
}

// bf16 copies of a layer's weights [rows][cols] in fragment order: dst for products over the
// inputs (depth padded to pad) and, unless NULL, dst_t for products over the outputs.
__global__ void to_bf16(const float* __restrict__ src, __bf16* __restrict__ dst, __bf16* __restrict__ dst_t, int rows,
                        int cols, int pad)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * cols) return;
    const int r = i / cols, c = i % cols;
    const __bf16 w = static_cast<__bf16>(src[i]);
    dst[frag_at(r, c, pad)] = w;
    if (dst_t) dst_t[frag_at(c, r, rows)] = w;
}

// ---------------------------------------------------------------- profiles
// Sample radii r_k = R + (k - 63.5) / 2, k = 0..127 (a 64-cell window centred
// on the interface).  A profile L (log densities at r_k) defines the field
// log rho0(d) = (1 - t) L_j + t L_{j+1} with s = (d - r_0) / 0.5 clamped to
// [0, 127], j = min(floor(s), 126), t = s - j, d the minimum-image distance.

__device__ __forceinline__ double min_image(double d, int n)
{
    d = fabs(d);
    return fmin(d, n - d);
}

// Hat coordinates (j, t) of distance d.
__device__ __forceinline__ void hat_of(double d, double r0, int& j, double& t)
{
    double s = (d - r0) * 2.0;
    s = fmin(fmax(s, 0.0), (double)(kOut - 1));
    j = min((int)s, kOut - 2);
    t = s - j;
}

// Least-squares fit, stage 1: the contributions of a pair of rows to the normal equations
// (H^T H) L = H^T log rho: of each sample k the diagonal (k, k), the upper off-diagonal
// (k, k+1) and the right-hand side.  part: [3][(ny + 1) / 2][128] doubles.
// The sites of a row are evaluated once each (one square root and one logarithm), 256 at a
// time, into LDS; then four threads per sample and row each go through a quarter of them, in
// x order, adding the sites whose hat functions reach the sample (a site reaches two samples;
// the weights of the others are zero, without branches).  256 x 256: 152 us when every
// sample's thread evaluated every site of its row, 13 us now.  Two rows per workgroup
// halve what the single workgroup of stage 2 has to read.
constexpr int kFitRows = 2;
constexpr int kFitThreads = 4 * kOut * kFitRows;
constexpr int kFitSites = 256;
constexpr int fit_groups(int ny) { return (ny + kFitRows - 1) / kFitRows; }

// One field's fit; a launch serves up to kFitJobs of them (profile_rows: second grid
// dimension): a field's rows fill half of the chip and its solve one workgroup.  96 fields of
// 256 x 256 after a batched run, moments included: about 5 ms one by one, 4 ms so.
struct FitJob {
    const float* rho;
    double* part;
    float* logrho;
    double cx, cy, r0;
    int nx, ny;
};
constexpr int kFitJobs = 32;
struct FitJobs { FitJob job[kFitJobs]; };  // a kernel argument (at most 4 KB)
static_assert(sizeof(FitJobs) <= 3584, "kernel arguments");

__global__ __launch_bounds__(kFitThreads) void profile_rows(const FitJobs jobs)
{
    const FitJob& job = jobs.job[blockIdx.y];
    const int nx = job.nx, ny = job.ny, groups = fit_groups(ny);
    if ((int)blockIdx.x >= groups) return;
    const float* __restrict__ rho = job.rho;
    double* __restrict__ part = job.part;
    const double cx = job.cx, cy = job.cy, r0 = job.r0;
    __shared__ double st[kFitRows][kFitSites], sv[kFitRows][kFitSites];
    __shared__ int sj[kFitRows][kFitSites];
    __shared__ double sum[4 * kFitRows][3][kOut];
    const int k = threadIdx.x & (kOut - 1), eighth = threadIdx.x / kOut;
    const int which = eighth / 4, quarter = eighth % 4;
    const int in_row = threadIdx.x % (4 * kOut);
    const int y = blockIdx.x * kFitRows + which;
    const double dy = min_image(y - cy, ny);
    const float* row = rho + (long long)y * nx;
    double a = 0.0, e = 0.0, b = 0.0;
    for (int x0 = 0; x0 < nx; x0 += kFitSites) {
        if (in_row < kFitSites) {
            const int x = x0 + in_row;
            int j = -2;  // reaches no sample
            double t = 0.0, v = 0.0;
            if (x < nx && y < ny) {
                const double dx = min_image(x - cx, nx);
                hat_of(sqrt(dx * dx + dy * dy), r0, j, t);
                v = log((double)row[x]);
            }
            sj[which][in_row] = j;
            st[which][in_row] = t;
            sv[which][in_row] = v;
        }
        __syncthreads();
#pragma unroll 8
        for (int q = 0; q < kFitSites / 4; ++q) {
            const int i = quarter * (kFitSites / 4) + q;
            const int j = sj[which][i];
            const double t = st[which][i], u = 1.0 - t;
            const double w = j == k ? u : (j + 1 == k ? t : 0.0);
            const double v = j == k || j + 1 == k ? sv[which][i] : 0.0;
            a += w * w;
            e += j == k ? u * t : 0.0;
            b += w * v;
        }
        __syncthreads();
    }
    sum[eighth][0][k] = a;
    sum[eighth][1][k] = e;
    sum[eighth][2][k] = b;
    __syncthreads();
    if (eighth < 3) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < 4 * kFitRows; ++q) s += sum[q][eighth][k];
        part[((long long)eighth * groups + blockIdx.x) * kOut + k] = s;
    }
}

// Stage 2 (one workgroup): sum the ny records (eight stretches per sample, in order), add
// lam * (graph Laplacian of the sample path), solve the symmetric positive-definite
// tridiagonal system in FP64 and write L as FP32.  The solver is parallel cyclic reduction:
// in each of seven rounds every row eliminates its two neighbours at distance d = 1, 2, 4, ...
// (each round takes Schur complements of a positive-definite matrix, so no pivoting is
// needed).  256 x 256: 82 us with one thread per sample over all rows and one thread solving,
// 8.6 us now.
constexpr int kSolveGroups = 8;
constexpr int kSolveRows = 8;  // rows whose loads are in flight together

__global__ __launch_bounds__(kSolveGroups * kOut) void profile_solve(const FitJobs jobs)
{
    const FitJob& job = jobs.job[blockIdx.x];
    const double* __restrict__ part = job.part;
    float* __restrict__ logrho = job.logrho;
    const int ny = fit_groups(job.ny);  // rows of partials
    __shared__ double sum[kSolveGroups][3][kOut];
    __shared__ double lo[2][kOut], di[2][kOut], up[2][kOut], rh[2][kOut];
    const int k = threadIdx.x & (kOut - 1), group = threadIdx.x / kOut;
    const long long plane = (long long)ny * kOut;
    const int per = (ny + kSolveGroups - 1) / kSolveGroups;
    double a = 0.0, e = 0.0, b = 0.0;
    const int end = min(ny, (group + 1) * per);
    for (int y0 = group * per; y0 < end; y0 += kSolveRows) {
        double va[kSolveRows], ve[kSolveRows], vb[kSolveRows];
#pragma unroll
        for (int q = 0; q < kSolveRows; ++q) {
            const long long o = (long long)(y0 + q) * kOut + k;
            const bool in = y0 + q < end;
            va[q] = in ? part[o] : 0.0;
            ve[q] = in ? part[plane + o] : 0.0;
            vb[q] = in ? part[2 * plane + o] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < kSolveRows; ++q) {
            a += va[q];
            e += ve[q];
            b += vb[q];
        }
    }
    sum[group][0][k] = a;
    sum[group][1][k] = e;
    sum[group][2][k] = b;
    __syncthreads();
    if (group == 0) {
        for (int g = 1; g < kSolveGroups; ++g) {
            a += sum[g][0][k];
            e += sum[g][1][k];
            b += sum[g][2][k];
        }
        if (k > 0) a += kSmooth;
        if (k < kOut - 1) {
            a += kSmooth;
            e -= kSmooth;
        } else {
            e = 0.0;
        }
        di[0][k] = a;
        up[0][k] = e;  // coupling of samples k and k + 1
        rh[0][k] = b;
        if (k == 0) lo[0][0] = 0.0;
        if (k < kOut - 1) lo[0][k + 1] = e;
    }
    __syncthreads();
    int cur = 0;
    for (int d = 1; d < kOut; d *= 2, cur ^= 1) {
        if (group == 0) {
            double l = 0.0, u = 0.0, m = di[cur][k], r = rh[cur][k];
            if (k >= d) {
                const double f = lo[cur][k] / di[cur][k - d];
                l = -f * lo[cur][k - d];
                m -= f * up[cur][k - d];
                r -= f * rh[cur][k - d];
            }
            if (k + d < kOut) {
                const double f = up[cur][k] / di[cur][k + d];
                u = -f * up[cur][k + d];
                m -= f * lo[cur][k + d];
                r -= f * rh[cur][k + d];
            }
            lo[cur ^ 1][k] = l;
            di[cur ^ 1][k] = m;
            up[cur ^ 1][k] = u;
            rh[cur ^ 1][k] = r;
        }
        __syncthreads();
    }
    if (group == 0) logrho[k] = (float)(rh[cur][k] / di[cur][k]);
}

// rho0(x, y) = exp((1 - t) L_j + t L_{j+1}) at the minimum-image distance of
// (x, y) from (cx, cy), for sample radii starting at r.
__device__ __forceinline__ void rho0_site(const float* __restrict__ logrho, double r, double cx, double cy, int nx,
                                          int ny, int x, int y, float* __restrict__ rho0)
{
    const double dx = min_image(x - cx, nx), dy = min_image(y - cy, ny);
    int j;
    double t;
    hat_of(sqrt(dx * dx + dy * dy), r, j, t);
    rho0[(long long)y * nx + x] = (float)exp((1.0 - t) * logrho[j] + t * logrho[j + 1]);
}

__global__ void profile_to_rho0(const float* __restrict__ logrho, double r0, double cx, double cy, int nx, int ny,
                                float* __restrict__ rho0)
{
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x < nx) rho0_site(logrho, r0, cx, cy, nx, ny, x, blockIdx.y, rho0);
}

constexpr int kMassIters = 60;
constexpr double kMaxShift = 8.0;

// Bisection for the outward shift delta in [-8, 8] at which the profile's field has total
// mass `mass` (the mass grows with delta for a profile that falls outwards): 60 halvings,
// delta the middle of the last interval; FP64 site sums in a fixed order.
// out[0] = delta, out[1] = the field's mass at delta.
//
// One level at a time this is a serial chain of 61 sums over the lattice.  A launch of
// mass_round instead evaluates all kMassCands middle points that the next kMassLevels levels
// of the bisection can visit, over the whole chip; the next launch sums up the workgroups'
// partials (every workgroup for itself, in the same order), walks down the levels, and goes
// on from the interval reached.  The interval after every level is that of the plain
// bisection.  256 x 256: 2900 us in one workgroup, 141 us in 18 launches (8.7 us a round).
// The partials live in the output field, which is written last.  Such a round is mostly
// latency, so a launch serves up to kMassJobs profiles (its second grid dimension): the
// starts of 64 droplets of 256 x 256, prediction included, 9.9 ms one by one, 6.9 ms so.
constexpr int kMassLevels = 4;
constexpr int kMassCands = (1 << kMassLevels) - 1;
constexpr int kMassRounds = kMassIters / kMassLevels;
static_assert(kMassRounds * kMassLevels == kMassIters, "whole rounds");
static_assert(kMassLevels == 4, "the sum over a wavefront leaves 16 candidates on 16 lane groups");
constexpr int kMassThreads = 256;
constexpr int kMassBlocks = 256;          // at most; kMassThreads sites each or more
constexpr int kMassStride = kMassCands + 1;

// Interval and partial sums of one round.
struct MassRound {
    double lo, hi;
    double part[1][kMassStride];  // [workgroups][candidates]
};

// One profile's search: its field, its workgroups and the records of even and odd rounds.
struct MassJob {
    const float* logrho;
    double r0, cx, cy, mass;
    int nx, ny, blocks;
    MassRound* rec[2];
    double* out;
    float* rho0;
};
constexpr int kMassJobs = 32;
struct MassJobs { MassJob job[kMassJobs]; };  // a kernel argument (at most 4 KB)
static_assert(sizeof(MassJobs) <= 3584, "kernel arguments");

constexpr size_t mass_round_doubles(int blocks) { return 2 + (size_t)blocks * kMassStride; }

// Middle point of the interval that heap node c (1 = the root) of the bisection tree under
// [lo, hi] halves: the bits of c below the leading one say up (1) or down (0).
__device__ __forceinline__ double mass_node(double lo, double hi, int c)
{
    int bit = 31 - __builtin_clz(c);
    double mid = 0.5 * (lo + hi);
    while (bit-- > 0) {
        if ((c >> bit) & 1) lo = mid;
        else hi = mid;
        mid = 0.5 * (lo + hi);
    }
    return mid;
}

// The field's constant inside the first sample (which = 0) or beyond the last (1): t = 0 in
// interval 0, or t = 1 in the last interval.
__device__ __forceinline__ double end_value(const float* __restrict__ logrho, int which)
{
    const int j = which ? kOut - 2 : 0;
    const double t = which ? 1.0 : 0.0;
    return exp((1.0 - t) * (double)logrho[j] + t * (double)logrho[j + 1]);
}

// The field's value at distance d for sample radii starting at r.
__device__ __forceinline__ double profile_value(const double* __restrict__ L, double d, double r)
{
    int j;
    double t;
    hat_of(d, r, j, t);
    return exp((1.0 - t) * L[j] + t * L[j + 1]);
}

// round 0 .. kMassRounds - 1: candidates of that round; round kMassRounds: the mass at the
// final delta (one candidate), delta to out[0].  Reads the record of the previous round (unused
// in round 0), writes this round's.
__global__ __launch_bounds__(kMassThreads) void mass_round(const MassJobs jobs, int round)
{
    const MassJob& job = jobs.job[blockIdx.y];
    const int blocks = job.blocks;
    if ((int)blockIdx.x >= blocks) return;
    const float* __restrict__ logrho = job.logrho;
    const MassRound* __restrict__ from = job.rec[(round & 1) ^ 1];
    MassRound* __restrict__ to = job.rec[round & 1];
    const double r0 = job.r0, cx = job.cx, cy = job.cy, mass = job.mass;
    const int nx = job.nx, ny = job.ny;
    __shared__ double L[kOut], ends[2], cand[kMassCands], sums[kMassThreads / 16][kMassStride], lohi[2];
    __shared__ double wsum[kMassThreads / 64][kMassStride];
    const int tid = threadIdx.x;
    if (tid < kOut) L[tid] = (double)logrho[tid];
    if (tid < 2) ends[tid] = end_value(logrho, tid);
    if (round == 0) {
        if (tid == 0) {
            lohi[0] = -kMaxShift;
            lohi[1] = kMaxShift;
        }
    } else {
        // sums of the previous round's candidates: 16 threads per stretch of workgroups
        // (all loads of a thread are issued together: read one after the other they would cost
        // a memory latency each)
        constexpr int groups = kMassThreads / 16, per = kMassBlocks / groups;
        const int c = tid & 15, g = tid >> 4;
        double v[per], acc = 0.0;
#pragma unroll
        for (int q = 0; q < per; ++q) v[q] = g + q * groups < blocks ? from->part[g + q * groups][c] : 0.0;
#pragma unroll
        for (int q = 0; q < per; ++q) acc += v[q];
        sums[g][c] = acc;
        __syncthreads();
        if (tid < kMassCands) {
            double m = 0.0;
            for (int q = 0; q < kMassThreads / 16; ++q) m += sums[q][tid];
            cand[tid] = m;
        }
        __syncthreads();
        if (tid == 0) {
            double lo = from->lo, hi = from->hi;
            for (int level = 0, node = 1; level < kMassLevels; ++level) {
                const double mid = 0.5 * (lo + hi);
                const bool up = cand[node - 1] < mass;
                if (up) lo = mid;
                else hi = mid;
                node = 2 * node + (up ? 1 : 0);
            }
            lohi[0] = lo;
            lohi[1] = hi;
        }
    }
    __syncthreads();
    const double lo = lohi[0], hi = lohi[1];
    const int n_cand = round < kMassRounds ? kMassCands : 1;
    if (blockIdx.x == 0 && tid == 0) {
        to->lo = lo;
        to->hi = hi;
        if (round == kMassRounds) job.out[0] = 0.5 * (lo + hi);
    }
    if (tid < n_cand) cand[tid] = r0 + mass_node(lo, hi, tid + 1);
    __syncthreads();
    double acc[kMassStride];
#pragma unroll
    for (int c = 0; c < kMassStride; ++c) acc[c] = 0.0;
    const long long n = (long long)nx * ny;
    for (long long i = (long long)blockIdx.x * kMassThreads + tid; i < n; i += (long long)blocks * kMassThreads) {
        const int x = (int)(i % nx), y = (int)(i / nx);
        const double dx = min_image(x - cx, nx), dy = min_image(y - cy, ny);
        const double d = sqrt(dx * dx + dy * dy);
        // a wavefront wholly beyond the samples, whatever the candidate, needs no exponentials
        const bool outside = __all((d - (r0 + hi)) * 2.0 >= (double)(kOut - 1));
        if (outside || __all((d - (r0 + lo)) * 2.0 <= 0.0)) {
            const double v = ends[outside ? 1 : 0];
#pragma unroll
            for (int c = 0; c < kMassCands; ++c) acc[c] += v;
        } else if (n_cand == 1) {
            acc[0] += profile_value(L, d, cand[0]);
        } else {
#pragma unroll
            for (int c = 0; c < kMassCands; ++c) acc[c] += profile_value(L, d, cand[c]);
        }
    }
    // Sum over the wavefront: in each of four rounds a lane keeps half of its sums and adds the
    // partner's share of them, so that lane groups end up with one candidate each.
    const int lane = tid & 63;
#pragma unroll
    for (int o = 32, m = kMassStride / 2; m >= 1; o >>= 1, m >>= 1) {
        const bool upper = lane & o;
#pragma unroll
        for (int q = 0; q < m; ++q) {
            const double send = upper ? acc[q] : acc[q + m], keep = upper ? acc[q + m] : acc[q];
            acc[q] = keep + __shfl_xor(send, o, 64);
        }
    }
    acc[0] += __shfl_xor(acc[0], 2, 64);
    acc[0] += __shfl_xor(acc[0], 1, 64);
    if ((lane & 3) == 0) wsum[tid >> 6][lane >> 2] = acc[0];
    __syncthreads();
    if (tid < kMassStride) to->part[blockIdx.x][tid] = (wsum[0][tid] + wsum[1][tid]) + (wsum[2][tid] + wsum[3][tid]);
}

// out[1] = the mass of the final round (one wavefront per profile, fixed order).
__global__ __launch_bounds__(64) void mass_final(const MassJobs jobs)
{
    const MassJob& job = jobs.job[blockIdx.x];
    const MassRound* __restrict__ from = job.rec[kMassRounds & 1];
    const int blocks = job.blocks;
    if (blocks == 0) return;  // by mass_small
    double p[kMassBlocks / 64], v = 0.0;
#pragma unroll
    for (int q = 0; q < kMassBlocks / 64; ++q) {
        const int b = threadIdx.x + 64 * q;
        p[q] = b < blocks ? from->part[b][0] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < kMassBlocks / 64; ++q) v += p[q];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (threadIdx.x == 0) job.out[1] = v;
}

// The fields at the shifts found.
__global__ void mass_fields(const MassJobs jobs)
{
    const MassJob& job = jobs.job[blockIdx.z];
    const int x = blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y;
    if (x < job.nx && y < job.ny)
        rho0_site(job.logrho, job.r0 + job.out[0], job.cx, job.cy, job.nx, job.ny, x, y, job.rho0);
}

// The same search by one workgroup per profile in one launch, a level at a time: lattices of
// at most kMassSmall sites, two per thread (32 x 32: 78 us, 33 x 32: 82 us, 45 x 45: 99 us; the rounds above need
// 135 us and more for their launches, 152 us on 33 x 32 and 45 x 45).
constexpr int kMassSmallThreads = 1024;
constexpr int kMassSmallSites = 2;
constexpr int kMassSmall = kMassSmallSites * kMassSmallThreads;

__global__ __launch_bounds__(kMassSmallThreads) void mass_small(const MassJobs jobs)
{
    const MassJob& job = jobs.job[blockIdx.x];
    if (job.blocks > 0) return;  // by mass_round
    const int nx = job.nx, n = job.nx * job.ny;
    const double r0 = job.r0, mass = job.mass;
    __shared__ double L[kOut];
    __shared__ double part[kMassSmallThreads];
    const int tid = threadIdx.x;
    if (tid < kOut) L[tid] = (double)job.logrho[tid];
    double lo = -kMaxShift, hi = kMaxShift;
    double d[kMassSmallSites];
#pragma unroll
    for (int q = 0; q < kMassSmallSites; ++q) {
        const int i = tid + q * kMassSmallThreads;
        const double dx = min_image((i < n ? i % nx : 0) - job.cx, nx), dy = min_image((i < n ? i / nx : 0) - job.cy, job.ny);
        d[q] = sqrt(dx * dx + dy * dy);
    }
    __syncthreads();
    for (int it = 0; it <= kMassIters; ++it) {
        const double delta = 0.5 * (lo + hi);
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < kMassSmallSites; ++q)
            if (tid + q * kMassSmallThreads < n) v += profile_value(L, d[q], r0 + delta);
        part[tid] = v;
        __syncthreads();
        for (int s = kMassSmallThreads / 2; s > 0; s >>= 1) {
            if (tid < s) part[tid] += part[tid + s];
            __syncthreads();
        }
        const double m = part[0];
        if (it == kMassIters) {
            if (tid == 0) {
                job.out[0] = delta;
                job.out[1] = m;
            }
        } else if (m < mass) {
            lo = delta;
        } else {
            hi = delta;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- liquid level
// Bands of a profile around radius R (d_k = (k - 63.5) / 2): inner = samples with
// d_k <= -min(12, R / 2), outer = samples with d_k >= 12.  Inside a relaxed droplet
// the density is the Laplace-shifted liquid density (Sec. IV.A-B); the inner band
// holds it, the outer band the vapour.

constexpr double kBand = 12.0;

// Means of the sample's log density over the two bands, for the workgroup of kOut
// threads that holds one profile (thread k = sample k).  FP64 tree sums in a fixed
// order.  An empty band gives NaN (0 / 0).
__device__ void band_means(double v, double R, double& m_in, double& m_out)
{
    __shared__ double part[4][kOut];
    const int k = threadIdx.x;
    const double d = (k - 63.5) * 0.5;
    const bool in = d <= -fmin(kBand, 0.5 * R);
    const bool out = d >= kBand;
    part[0][k] = in ? v : 0.0;
    part[1][k] = in ? 1.0 : 0.0;
    part[2][k] = out ? v : 0.0;
    part[3][k] = out ? 1.0 : 0.0;
    __syncthreads();
    for (int s = kOut / 2; s > 0; s >>= 1) {
        if (k < s) {
#pragma unroll
            for (int q = 0; q < 4; ++q) part[q][k] += part[q][k + s];
        }
        __syncthreads();
    }
    m_in = part[0][0] / part[1][0];
    m_out = part[2][0] / part[3][0];
    __syncthreads();  // part is reused by the next call
}

// lev[b] = (inner, outer) band means of profile b; R = x[b][2].
__global__ __launch_bounds__(kOut) void profile_levels(const float* __restrict__ L, const float* __restrict__ x,
                                                       double* __restrict__ lev)
{
    const long long b = blockIdx.x;
    const int k = threadIdx.x;
    double m_in, m_out;
    band_means((double)L[b * kOut + k], (double)x[b * kIn + 2], m_in, m_out);
    if (k == 0) {
        lev[2 * b] = m_in;
        lev[2 * b + 1] = m_out;
    }
}

// Profile b pinned to the inner level target[b], in place: with rho = exp(L),
// rho_in / rho_out = exp of the band means and rho* = exp(target),
// rho'_k = rho_out + (rho_k - rho_out) g, g = (rho* - rho_out) / (rho_in - rho_out),
// then rho'_k = rho* on the inner band.  The profile is left as it is when the
// target or g is not finite or some rho'_k <= 0.
__global__ __launch_bounds__(kOut) void profile_anchor(float* __restrict__ L, const float* __restrict__ x,
                                                       const double* __restrict__ target)
{
    const long long b = blockIdx.x;
    const int k = threadIdx.x;
    const double R = (double)x[b * kIn + 2];
    const double v = (double)L[b * kOut + k];
    double m_in, m_out;
    band_means(v, R, m_in, m_out);
    const double lev = target[b];
    const double r_in = exp(m_in), r_out = exp(m_out), r_t = exp(lev);
    const double g = (r_t - r_out) / (r_in - r_out);
    const bool in = (k - 63.5) * 0.5 <= -fmin(kBand, 0.5 * R);
    const double rho = in ? r_t : r_out + (exp(v) - r_out) * g;
    const bool usable = isfinite(lev) && isfinite(g);
    const int bad = __syncthreads_or(!(rho > 0.0));
    if (usable && !bad) L[b * kOut + k] = (float)log(rho);
}

// ---------------------------------------------------------------- launchers

static unsigned grid1(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

hipError_t launch_profile_levels(const float* L, const float* x, int B, double* lev, hipStream_t s)
{
    hipLaunchKernelGGL(profile_levels, dim3(B), dim3(kOut), 0, s, L, x, lev);
    return hipGetLastError();
}

hipError_t launch_profile_anchor(float* L, const float* x, const double* target, int B, hipStream_t s)
{
    hipLaunchKernelGGL(profile_anchor, dim3(B), dim3(kOut), 0, s, L, x, target);
    return hipGetLastError();
}

// An operand that is contiguous in k with 16-byte aligned rows loads eight k values at once.
static bool rows_of_8(const __bf16* P, long long s_row, long long s_k)
{
    return s_k == 1 && s_row % 8 == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0;
}

hipError_t gemm(const __bf16* A, long long sam, long long sak, const __bf16* B, long long sbk, long long sbn,
                float* C, int ldc, int M, int N, int K, hipStream_t s)
{
    if (M % 16 || N % 16 || K % 32 || M <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
    const long long tiles = (long long)(M / 16) * (N / 16);
    const bool av = rows_of_8(A, sam, sak), bv = rows_of_8(B, sbn, sbk);
    auto kern = av ? (bv ? gemm_bf16<true, true> : gemm_bf16<true, false>)
                   : (bv ? gemm_bf16<false, true> : gemm_bf16<false, false>);
    hipLaunchKernelGGL(kern, dim3(grid1(tiles, 4)), dim3(256), 0, s, A, sam, sak, B, sbk, sbn, C, ldc, M, N, K);
    return hipGetLastError();
}

// bytes must be a multiple of 4
hipError_t launch_fill(void* p, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 4;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_zero, dim3(grid1((long long)n, 256)), dim3(256), 0, s, static_cast<unsigned int*>(p), n);
    return hipGetLastError();
}

// Rows per workgroup of the pass: four (one per lane group) up to 1024 rows, where that leaves
// no more workgroups than compute units (512 rows: 11.8 us with 4 rows, 12.6 us with 8, 14.0 us
// with 16); beyond, all 16 of the tile, since every workgroup reads all weights.
int mlp_rows(int B) { return B <= 1024 ? 4 : 16; }

hipError_t launch_mlp_pass(const MlpArgs& a, bool train, hipStream_t s)
{
    if (a.B <= 0 || a.B % (train ? 32 : 16)) return hipErrorInvalidValue;
    const int rows = mlp_rows(a.B);
    const dim3 grid(a.B / rows), block(kMlpThreads);
    if (rows == 16) {
        if (train) hipLaunchKernelGGL((mlp_pass<true, 4>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((mlp_pass<false, 4>), grid, block, 0, s, a);
    } else {
        if (train) hipLaunchKernelGGL((mlp_pass<true, 1>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((mlp_pass<false, 1>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_mlp_grads(const GradArgs& g, bool update, hipStream_t s)
{
    if (g.B <= 0 || g.B % 32) return hipErrorInvalidValue;
    if (update) hipLaunchKernelGGL(mlp_grads<true>, dim3((kGradWaves + 3) / 4), dim3(256), 0, s, g);
    else hipLaunchKernelGGL(mlp_grads<false>, dim3((kGradWaves + 3) / 4), dim3(256), 0, s, g);
    return hipGetLastError();
}

hipError_t launch_adam(float* p, float* m, float* v, const float* g, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2, hipStream_t s)
{
    hipLaunchKernelGGL(adam, dim3(grid1(n, 256)), dim3(256), 0, s, p, m, v, g, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_check_rows(const int* idx, long long n, int rows, int* flag, hipStream_t s)
{
    hipLaunchKernelGGL(check_rows, dim3(256), dim3(256), 0, s, idx, n, rows, flag);
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float* src, __bf16* dst, __bf16* dst_t, int rows, int cols, int pad, hipStream_t s)
{
    hipLaunchKernelGGL(to_bf16, dim3(grid1((long long)rows * cols, 256)), dim3(256), 0, s, src, dst, dst_t, rows, cols,
                       pad);
    return hipGetLastError();
}

hipError_t launch_profiles_extract(const lbml_fit* p, int n, hipStream_t s)
{
    for (int first = 0; first < n; first += kFitJobs) {
        const int count = std::min(kFitJobs, n - first);
        FitJobs jobs{};
        int groups = 0;
        for (int i = 0; i < count; ++i) {
            const lbml_fit& f = p[first + i];
            jobs.job[i] = FitJob{f.rho, static_cast<double*>(f.scratch), f.logrho, f.cx, f.cy, f.R - 0.25 * (kOut - 1),
                                 f.nx, f.ny};
            groups = std::max(groups, fit_groups(f.ny));
        }
        hipLaunchKernelGGL(profile_rows, dim3(groups, count), dim3(kFitThreads), 0, s, jobs);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(profile_solve, dim3(count), dim3(kSolveGroups * kOut), 0, s, jobs);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_profile_extract(const float* rho, int nx, int ny, double cx, double cy, double R, double* part,
                                  float* logrho, hipStream_t s)
{
    const lbml_fit f{rho, cx, cy, R, nx, ny, part, (size_t)3 * ny * kOut * sizeof(double), logrho};
    return launch_profiles_extract(&f, 1, s);
}

// Scratch of the allocation-free profile fit: the [3][ny][128] FP64 row partials for
// ny <= kStaticProfileRows.  Each GPU the library runs on holds its own copy until the
// process ends.  In host code the name `scratch` is only a stand-in for the symbol:
// its device address comes from hipGetSymbolAddress, once per device.
constexpr int kStaticProfileRows = 2048;  // the limit lbml.h states for lbml_profile_extract_noalloc
static __device__ __align__(256) double scratch[3 * kStaticProfileRows * kOut];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Device address of `scratch` on the current device, looked up with that device
// current on the first call and kept per device.
hipError_t static_profile_scratch(double** out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = static_cast<double*>(ptr);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

int static_profile_rows() { return kStaticProfileRows; }

hipError_t launch_profile_extract_static(const float* rho, int nx, int ny, double cx, double cy, double R,
                                         float* logrho, hipStream_t s)
{
    if (ny > kStaticProfileRows) return hipErrorInvalidValue;
    double* part = nullptr;
    const hipError_t e = static_profile_scratch(&part);
    if (e != hipSuccess) return e;
    // profile_rows writes every partial that profile_solve reads: nothing to clear
    return launch_profile_extract(rho, nx, ny, cx, cy, R, part, logrho, s);
}

hipError_t launch_profile_to_rho0(const float* logrho, double R, double cx, double cy, int nx, int ny, float* rho0,
                                  hipStream_t s)
{
    const double r0 = R - 0.25 * (kOut - 1);
    hipLaunchKernelGGL(profile_to_rho0, dim3(grid1(nx, 256), ny), dim3(256), 0, s, logrho, r0, cx, cy, nx, ny, rho0);
    return hipGetLastError();
}

// Up to kMassJobs profiles in one set of launches.
static hipError_t launch_mass_jobs(const lbml_placement* p, int n, hipStream_t s)
{
    MassJobs jobs{};
    int blocks = 0, large = 0, gx = 0, gy = 0;
    for (int i = 0; i < n; ++i) {
        MassJob& job = jobs.job[i];
        const long long sites = (long long)p[i].nx * p[i].ny;
        job = MassJob{p[i].logrho, p[i].R - 0.25 * (kOut - 1), p[i].cx, p[i].cy, p[i].mass, p[i].nx, p[i].ny, 0,
                      {nullptr, nullptr}, p[i].shift, p[i].rho0};
        gx = std::max(gx, (int)grid1(p[i].nx, 256));
        gy = std::max(gy, p[i].ny);
        if (sites <= kMassSmall) continue;  // blocks 0: by mass_small
        // two rounds' records in the output field (8-byte aligned inside it): at most 128
        // doubles and a little per workgroup of at least 256 sites
        job.blocks = (int)std::min<long long>(kMassBlocks, sites / kMassThreads);
        double* base = reinterpret_cast<double*>((reinterpret_cast<uintptr_t>(job.rho0) + 7) / 8 * 8);
        static_assert(2 * (2 + kMassStride) * sizeof(double) + 8 <= kMassThreads * sizeof(float), "records fit in the field");
        job.rec[0] = reinterpret_cast<MassRound*>(base);
        job.rec[1] = reinterpret_cast<MassRound*>(base + mass_round_doubles(job.blocks));
        blocks = std::max(blocks, job.blocks);
        ++large;
    }
    if (large < n) {
        hipLaunchKernelGGL(mass_small, dim3(n), dim3(kMassSmallThreads), 0, s, jobs);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (large > 0) {
        for (int round = 0; round <= kMassRounds; ++round) {
            hipLaunchKernelGGL(mass_round, dim3(blocks, n), dim3(kMassThreads), 0, s, jobs, round);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(mass_final, dim3(n), dim3(64), 0, s, jobs);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(mass_fields, dim3(gx, gy, n), dim3(256), 0, s, jobs);
    return hipGetLastError();
}

hipError_t launch_profiles_to_rho0_mass(const lbml_placement* p, int n, hipStream_t s)
{
    hipError_t e = hipSuccess;
    for (int i = 0; i < n && e == hipSuccess; i += kMassJobs) e = launch_mass_jobs(p + i, std::min(kMassJobs, n - i), s);
    return e;
}

}  // namespace lbml
