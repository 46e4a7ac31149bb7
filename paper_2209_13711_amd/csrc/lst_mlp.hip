// Learned scorer of triplets and quintuplets: MLP 40 -> 64 -> 64 -> 1
// (ReLU, ReLU, logit), one network per object kind.
//
// Inference runs on the gfx950 matrix cores.  A wavefront takes 16
// candidates at a time; layers 1 and 2 are v_mfma_f32_16x16x32_bf16
// products (BF16 operands, FP32 accumulation), the first hidden layer is
// rounded to BF16 (nearest, ties to even) before it feeds the second, and
// the last layer is an FP32 dot product on the vector ALUs (N = 1 would
// waste a matrix tile).  The products are taken as weights x candidates, so
// a lane receives consecutive hidden units of one candidate, which is the
// operand the next layer takes: nothing passes through LDS between layers.
// In the chain the 40 features of a quintuplet are
// computed in registers by the lane that owns it, standardised and written
// straight into the LDS operand tile, so they never travel through HBM.
//
// Training uses the same forward tile (saving the hidden activations, or
// fused into the gradient kernel), a backward pass whose products run on the
// matrix cores in FP32 (v_mfma_f32_16x16x4_f32) per chunk of rows, followed
// by a reduction over the chunks in a fixed order (gradients are bit-for-bit
// deterministic), and Adam on FP32 master weights.
//
// Parameter vector (FP32): W1[64][40] (row = hidden unit), b1[64],
// W2[64][64], b2[64], w3[64], b3.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "lst_access.hpp"
#include "lst_cuts.hpp"

namespace lst {

constexpr int NIN = MLP_NIN, NH = MLP_NH, KP = 64;  // inputs, hidden units, padded K
constexpr int LD = KP + 8;   // LDS row stride in BF16 elements (144 B: conflict-free b128 reads)
constexpr int OFF_W1 = 0, OFF_B1 = NH * NIN, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH;
constexpr int OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NH, NPARAM = OFF_B3 + 1;
static_assert(NPARAM == MLP_NPARAM, "parameter layout");
constexpr int GRAD_CHUNKS = MLP_GRAD_CHUNKS;   // most row chunks of the gradient sums
constexpr int GRAD_FEW = MLP_GRAD_CHUNKS_FEW;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// the caller's hidden-layer arrays are only aligned to their elements: wide
// global accesses that the hardware takes at any address
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));

// float -> BF16 bits, round to nearest even (a NaN stays a quiet NaN)
__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x7fffffu)) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// eight consecutive BF16 values (16 bytes, 16-byte aligned) as an MFMA operand
__device__ __forceinline__ bf16x8 load8(const uint16_t *p)
{
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(p));
}

// Weights in LDS as BF16 [output unit][k] (K zero padded), the rest FP32.
struct alignas(16) MlpW {
    uint16_t w1[NH][LD];
    uint16_t w2[NH][LD];
    float b1[NH], b2[NH], w3[NH];
    float b3;
};

// The weights staged by the block's NT threads: each thread loads its
// elements of each matrix before it converts them, so the loads are in flight
// together rather than one after the other.
template <int NT>
__device__ __forceinline__ void load_weights(const float *P, MlpW &w)
{
    static_assert(NH * KP % NT == 0 && NH * NH == NH * KP, "weight staging");
    constexpr int WPT = NH * KP / NT;
    float a[WPT], b[WPT];
#pragma unroll
    for (int u = 0; u < WPT; ++u) {
        const int i = threadIdx.x + u * NT, o = i / KP, k = i % KP;
        a[u] = k < NIN ? P[OFF_W1 + o * NIN + k] : 0.0f;
        b[u] = P[OFF_W2 + o * NH + k];
    }
#pragma unroll
    for (int u = 0; u < WPT; ++u) {
        const int i = threadIdx.x + u * NT, o = i / KP, k = i % KP;
        w.w1[o][k] = k < NIN ? f2bf(a[u]) : (uint16_t)0;
        w.w2[o][k] = f2bf(b[u]);
    }
    for (int i = threadIdx.x; i < NH; i += blockDim.x) {
        w.b1[i] = P[OFF_B1 + i];
        w.b2[i] = P[OFF_B2 + i];
        w.w3[i] = P[OFF_W3 + i];
    }
    if (threadIdx.x == 0) w.b3 = P[OFF_B3];
}

// orders a wave's LDS writes before later LDS reads by other lanes of the
// same wave (a wave's LDS operations complete in issue order): the operand
// and hidden tiles are wave-private, so no block barrier is needed for them
__device__ __forceinline__ void wave_tile_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Operand layouts of v_mfma_f32_16x16x32_bf16 on a wave64: lane l supplies row
// l%16 of A and column l%16 of B, each with the eight k values 8 (l/16) .. +7
// of the 32-wide k step; lane l receives D rows 4 (l/16) + r, column l%16.
// With A the weights (row = hidden unit) and B the candidates (column =
// candidate), lane l receives units 16 nt + 4 (l/16) + r of candidate l%16.
//
// The second layer takes those units where they are: its k step ks holds the
// units 32 ks .. 32 ks + 31, of which quarter q = l/16 supplies 4 q + j (j < 4)
// and 16 + 4 q + j - 4 (j >= 4).  The order of k inside a step is free as long
// as both operands agree, so its weights are read in that order.
__device__ __forceinline__ bf16x8 layer2_k(const uint16_t *row, int ks, int q)
{
    const uint2 a = *reinterpret_cast<const uint2 *>(row + 32 * ks + 4 * q);
    const uint2 b = *reinterpret_cast<const uint2 *>(row + 32 * ks + 16 + 4 * q);
    return __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, b.x, b.y));
}

// the weights as a wave's operands, kept over its tiles
struct MlpOps {
    bf16x8 w1[4][KP / 32], w2[4][KP / 32];
};

__device__ __forceinline__ MlpOps mlp_ops(const MlpW &w)
{
    const int l = threadIdx.x & 63, c = l & 15, q = l >> 4;
    MlpOps o;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int ks = 0; ks < KP / 32; ++ks) {
            o.w1[nt][ks] = load8(&w.w1[16 * nt + c][32 * ks + 8 * q]);
            o.w2[nt][ks] = layer2_k(w.w2[16 * nt + c], ks, q);
        }
    return o;
}

// ReLU of four hidden units as BF16 (8 bytes)
__device__ __forceinline__ uint2 relu4(const f32x4 &a, const float4 &b)
{
    const float z[4] = {a[0] + b.x, a[1] + b.y, a[2] + b.z, a[3] + b.w};
    uint32_t h[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = f2bf(z[r] > 0.0f ? z[r] : 0.0f);
    return make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
}

// The last layer's sum over the hidden units 16 nt + 4 q + r: a lane adds its
// tiles nt in order for each r (t[r]), then come the 16 sums (q, r) by halves,
// q ^ 2, q ^ 1, r ^ 2, r ^ 1; every lane of a candidate returns it.  Against 64
// bits the layer is 7.7e-8 off like this (of the logits' norm, 1000 to 20,000
// rows), 9.0e-8 to 9.6e-8 with a lane's 16 terms one after the other.  A lane
// sends the sums that its partner keeps, so five values cross the wave and not
// eight; 200,003 rows take 23.1 us with the preparation, 22.7 in the shorter
// order.
__device__ __forceinline__ float logit_sum(const float t[4])
{
    const int l = threadIdx.x & 63;
    const bool hi = l & 32, odd = l & 16;
    float a = hi ? t[2] : t[0], b = hi ? t[3] : t[1];   // r = 0 or 2, 1 or 3
    a += __shfl_xor(hi ? t[0] : t[2], 32, 64);
    b += __shfl_xor(hi ? t[1] : t[3], 32, 64);
    float v = odd ? b : a;
    v += __shfl_xor(odd ? a : b, 16, 64);
    v += __shfl_xor(v, 32, 64);
    v += __shfl_xor(v, 16, 64);
    return v;
}

// Forward of 16 candidates: x[ks] = inputs 32 ks + 8 q .. +7 of candidate l%16.
// Every lane returns the logit of its candidate.  save(nt, h1, h2), when
// given, receives the lane's units 16 nt + 4 q .. +3 of both hidden layers.
template <class F>
__device__ __forceinline__ float mlp_tile(const MlpW &w, const MlpOps &o, const bf16x8 x[KP / 32], F &&save)
{
    const int q = (threadIdx.x & 63) >> 4;
    f32x4 acc[4];
    uint2 h[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        acc[nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < KP / 32; ++ks)
            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o.w1[nt][ks], x[ks], acc[nt], 0, 0, 0);
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
        h[nt] = relu4(acc[nt], *reinterpret_cast<const float4 *>(&w.b1[16 * nt + 4 * q]));
    bf16x8 hk[KP / 32];
#pragma unroll
    for (int ks = 0; ks < KP / 32; ++ks)
        hk[ks] = __builtin_bit_cast(bf16x8, make_uint4(h[2 * ks].x, h[2 * ks].y, h[2 * ks + 1].x, h[2 * ks + 1].y));
    float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // terms of the logit
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        acc[nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < KP / 32; ++ks)
            acc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o.w2[nt][ks], hk[ks], acc[nt], 0, 0, 0);
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const float4 b = *reinterpret_cast<const float4 *>(&w.b2[16 * nt + 4 * q]);
        const float4 c = *reinterpret_cast<const float4 *>(&w.w3[16 * nt + 4 * q]);
        const float z[4] = {acc[nt][0] + b.x, acc[nt][1] + b.y, acc[nt][2] + b.z, acc[nt][3] + b.w};
        const float w3[4] = {c.x, c.y, c.z, c.w};
        float h2[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            h2[r] = z[r] > 0.0f ? z[r] : 0.0f;
            t[r] += h2[r] * w3[r];
        }
        save(nt, h[nt], make_float4(h2[0], h2[1], h2[2], h2[3]));
    }
    return logit_sum(t) + w.b3;
}

// ---------------------------------------------------------------- training forward
// X: [n][KP] BF16 rows (features standardised, zero padded).  A wave takes
// tiles of 16 rows, its operands straight from memory (a row is 128 bytes) and
// the next tile's on their way; few blocks, so that staging the weights (27 KB
// a block) is spread over many tiles.  200,003 rows 12.5-13.7 us (25.6 MB read, 5
// us at the copy rate; the rest is staging and six tiles' latency per wave), 25.2
// us with inputs and hidden layer through LDS and weights staged by 2048
// blocks; 5000 rows with the hidden layers saved 6.2 us, 7.4 before.
constexpr int FWD_BLOCKS = 512;   // two per CU: what its registers allow

template <bool SAVE>
__global__ __launch_bounds__(BLOCK) void k_mlp_forward(const float *P, const uint16_t *X, int64_t n,
                                                       float *logits, uint16_t *h1, float *h2)
{
    __shared__ MlpW w;
    const int l = threadIdx.x & 63, c = l & 15, q = l >> 4;
    const int64_t tiles = (n + 15) / 16, step = (int64_t)gridDim.x * WAVES;
    const int64_t first = (int64_t)blockIdx.x * WAVES + (threadIdx.x >> 6);
    bf16x8 next[KP / 32];
    auto fetch = [&](int64_t tile) {
        const int64_t row = tile * 16 + c;
#pragma unroll
        for (int ks = 0; ks < KP / 32; ++ks) {
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (row < n) v = *reinterpret_cast<const uint4 *>(&X[row * KP + 32 * ks + 8 * q]);
            next[ks] = __builtin_bit_cast(bf16x8, v);
        }
    };
    fetch(first);
    load_weights<BLOCK>(P, w);
    __syncthreads();   // weights staged
    const MlpOps o = mlp_ops(w);
    for (int64_t tile = first; tile < tiles; tile += step) {
        bf16x8 x[KP / 32];
#pragma unroll
        for (int ks = 0; ks < KP / 32; ++ks) x[ks] = next[ks];
        fetch(tile + step);
        const int64_t row = tile * 16 + c;
        const float z = mlp_tile(w, o, x, [&](int nt, const uint2 &a, const float4 &b) {
            if (!SAVE || row >= n) return;
            uint16_t *pa = h1 + row * KP + 16 * nt + 4 * q;
            float *pb = h2 + row * NH + 16 * nt + 4 * q;
            *reinterpret_cast<u32x2_any *>(pa) = u32x2_any{a.x, a.y};
            *reinterpret_cast<f32x4_any *>(pb) = f32x4_any{b.x, b.y, b.z, b.w};
        });
        if (q == 0 && row < n) logits[row] = z;
    }
}

// standardise raw FP32 features [n][40] into BF16 rows of KP (zero padded)
__global__ void k_mlp_prepare(const float *F, const float *mean, const float *istd, int64_t n,
                              uint16_t *X)
{
    const int64_t tot = n * KP;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < tot;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i / KP;
        const int k = (int)(i % KP);
        X[i] = k < NIN ? f2bf((F[r * NIN + k] - mean[k]) * istd[k]) : (uint16_t)0;
    }
}

// the same for 16-byte aligned F and X: eight features per thread, always the
// same eight (the grid's stride is a whole number of rows), so their constants
// are read once.  Bounded by memory: 200,003 rows 13.4 us (57.6 MB, 4.3 TB/s),
// 15.5 us one element per thread.
__global__ __launch_bounds__(BLOCK) void k_mlp_prepare8(const float *F, const float *mean, const float *istd,
                                                        int64_t n, uint16_t *X)
{
    const int k = (threadIdx.x & 7) * 8;
    float m[8], s[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        m[i] = k < NIN ? mean[k + i] : 0.0f;
        s[i] = k < NIN ? istd[k + i] : 0.0f;
    }
    const int64_t stride = (int64_t)gridDim.x * (BLOCK / 8);
    for (int64_t r = (int64_t)blockIdx.x * (BLOCK / 8) + (threadIdx.x >> 3); r < n; r += stride) {
        uint4 out = make_uint4(0u, 0u, 0u, 0u);
        if (k < NIN) {
            const float4 *p = reinterpret_cast<const float4 *>(&F[r * NIN + k]);
            const float4 a = p[0], b = p[1];
            const float f[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            uint32_t u[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) u[i] = f2bf((f[i] - m[i]) * s[i]);
            out = make_uint4(u[0] | (u[1] << 16), u[2] | (u[3] << 16), u[4] | (u[5] << 16), u[6] | (u[7] << 16));
        }
        *reinterpret_cast<uint4 *>(&X[r * KP + k]) = out;
    }
}

// ---------------------------------------------------------------- training backward
// Gradient of the mean BCE-with-logits loss from the row terms
//   g = (sigmoid(z) - y) / n,  dz2 = g w3 [h2 > 0],  dz1 = (dz2 W2) [h1 > 0]
// (W2 the BF16-rounded weights the forward used), summed over the rows:
//   dW1 = dz1^T X, db1 = sum dz1, dW2 = dz2^T h1, db2 = sum dz2,
//   dw3 = h2^T g, db3 = sum g.
// The rows split into at most GRAD_CHUNKS chunks of whole 64-row batches (at
// most GRAD_FEW where the caller's workspace holds no more), one block of
// eight waves per chunk.  In each batch two waves share 16 rows,
// each taking half of the hidden units: their forward (FWD) or the stored
// logits and hidden layers, the row terms into LDS, and dz1 as 16 x 32 x 64
// FP32 matrix products.  The waves then share the 28 16 x 16 tiles of dW1
// (64 x 48, inputs zero padded) and dW2 (64 x 64), each a product over the
// batch's 64 rows; their accumulators stay in registers over the chunk's
// batches.  Products are FP32 matrix-core steps (v_mfma_f32_16x16x4_f32: lane
// l supplies A[l%16][l/16] and B[l/16][l%16], receives D rows 4 (l/16) + r,
// column l%16).  The vector sums are kept per lane over its rows and combined
// in a fixed order at the end.  A block writes its chunk's partial gradient;
// k_mlp_reduce adds the chunks in an order of its own.  Every sum runs in an order
// fixed by n and the most chunks, so the gradient is bit-for-bit reproducible,
// and the forward-fused and the stored-activation variants give the same bits.
//
// Bounded by latency: at 4096 rows 64 blocks run one batch each, a chain of
// loads, small products and barriers.  So eight waves rather than four (two
// per SIMD: the products' and the tiles' chains halve), the batch's rows and
// labels are loaded before the weights, and a row's sigmoid and loss are
// computed once, by one lane.  4096 rows 17.7 -> 13.3 us, 5000 rows (79 blocks
// of one batch instead of 40 of two) 29.0 -> 12.4 us.  Of the 13 us, weights
// and rows to LDS take 2.7, the forward 2, the row terms 0.9, dz1 1.5, the
// tiles 2.8 (their products alone 1.5), the partial sums 1.4.  Step-ordered
// copies of the operands for 16-byte LDS reads made the tiles slower (5.8 us:
// each BF16 operand converted right before its product).
constexpr int GW = 8, GB = GW * 64;    // waves and threads of a block
constexpr int RB = 64;                 // rows per batch of a block: 16 for each pair of waves
constexpr int HT = 2;                  // 16-column tiles of the hidden layer per wave
constexpr int GT = 28;                 // gradient tiles: 12 of dW1, 16 of dW2
constexpr int GT_W = (GT + GW - 1) / GW;   // per wave at most
// row strides of the FP32 row-term tiles: the gradient products read 16
// consecutive columns of 4 consecutive rows per instruction, which a stride of
// 16 banks (mod 64) spreads over distinct banks; dz1 reads 4 consecutive
// columns of 16 rows, which takes a stride of 4 banks, so dz2 is kept in both
constexpr int DS = NH + 16, DR = NH + 4;
static_assert(NIN <= 48 && GB * 8 == RB * KP, "gradient tiles; one 16-byte load per thread stages a batch");

struct alignas(16) SmGrad {
    MlpW w;
    uint16_t x[RB][LD];            // inputs (BF16)
    uint16_t h[RB][LD];            // first hidden layer (BF16)
    float d2[RB][DS], d2r[RB][DR]; // dz2
    float d1[RB][DS];              // dz1; before that, logit terms of the upper hidden half
    float g[RB], y[RB];            // row terms, labels
    float vs[4][3][NH];            // the row groups' db1, db2, dw3
    float gs[4];                   // the row groups' db3
};
static_assert(sizeof(float) * 4 * HT * 4 * 64 <= sizeof(float) * RB * DS, "logit terms fit d1");

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// lane 15 of each row of 16 lanes: the row's sum (DPP row_shr:1,2,4,8; lanes
// outside a shift add zero)
__device__ __forceinline__ float row_sum16(float v)
{
    auto shr = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v += shr(v, std::integral_constant<int, 0x111>{});
    v += shr(v, std::integral_constant<int, 0x112>{});
    v += shr(v, std::integral_constant<int, 0x114>{});
    v += shr(v, std::integral_constant<int, 0x118>{});
    return v;
}

// floats of the backward workspace: the per-row losses, then the partial
// gradients of up to `chunks` chunks
static size_t work_floats(int64_t n, int chunks) { return (size_t)n + (size_t)chunks * NPARAM; }

// rows of the chunk c: [c clen, min((c + 1) clen, n)), clen a multiple of RB
static void grad_chunks(int64_t n, size_t work_bytes, int &nch, int64_t &clen)
{
    const int most = work_bytes >= sizeof(float) * work_floats(n, GRAD_CHUNKS) ? GRAD_CHUNKS : GRAD_FEW;
    int64_t b = (n + RB - 1) / RB;
    if (b < 1) b = 1;
    const int64_t per = (b + most - 1) / most;   // batches of a chunk
    nch = (int)((b + per - 1) / per);
    clen = per * RB;
}

template <bool FWD>
__global__ __launch_bounds__(GB) void k_mlp_grad(const float *P, const uint16_t *X, const uint8_t *y,
                                                 int64_t n, int64_t clen, const float *logits,
                                                 const uint16_t *h1, const float *h2, float *loss_rows,
                                                 float *part)
{
    __shared__ SmGrad sm;
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
    const int rg = w & 3, half = w >> 2;             // 16-row group, half of the hidden units
    const int col = l & 15, q = l >> 4, rl = 16 * rg + col;   // the lane's row of the batch
    const int64_t r0 = (int64_t)blockIdx.x * clen;
    const int64_t r1 = r0 + clen < n ? r0 + clen : n;
    // the batch's inputs (and stored first hidden layer), 16 bytes per thread,
    // zero past the chunk; labels and stored logits one per thread
    const int xr = tid >> 3, xc = (tid & 7) * 8;
    uint4 xv, hv;
    float yv = 0.0f, zv = 0.0f;
    f32x4 h2n[HT];                                   // the lane's row and units of the stored second layer
    const int u0 = 16 * HT * half + 4 * q;           // the lane's first unit
    auto fetch = [&](int64_t b0) {
        xv = hv = make_uint4(0u, 0u, 0u, 0u);
        if (b0 + xr < r1) {
            xv = *reinterpret_cast<const uint4 *>(&X[(b0 + xr) * KP + xc]);
            if (!FWD) hv = *reinterpret_cast<const uint4 *>(&h1[(b0 + xr) * KP + xc]);
        }
        if (tid < RB) {
            const bool live = b0 + tid < r1;
            yv = live && y[b0 + tid] ? 1.0f : 0.0f;
            if (!FWD) zv = live ? logits[b0 + tid] : 0.0f;
        }
        if (!FWD)
#pragma unroll
            for (int i = 0; i < HT; ++i) {
                h2n[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                if (b0 + rl < r1)
                    h2n[i] = *reinterpret_cast<const f32x4_any *>(h2 + (b0 + rl) * NH + u0 + 16 * i);
            }
    };
    fetch(r0);
    load_weights<GB>(P, sm.w);
    f32x4 acc[GT_W];
#pragma unroll
    for (int i = 0; i < GT_W; ++i) acc[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // sums over rows: db1 of the lane's unit 16 (2 half + i) + l%16 (its dz1
    // rows), db2 and dw3 of its units 16 (2 half + i) + 4 q + r (its row), db3
    float sb1[HT] = {0.0f, 0.0f}, sb2[HT][4] = {}, sw3[HT][4] = {}, sg = 0.0f;
    // operands of the wave's gradient tiles: column 16 jt + l%16 of dz1 (dW1)
    // or dz2 (dW2) and column 16 kt + l%16 of the inputs or h1, at row 0
    const float *ta[GT_W];
    const uint16_t *tb[GT_W];
#pragma unroll
    for (int i = 0; i < GT_W; ++i) {
        const int t = w + GW * i < GT ? w + GW * i : GT - 1;
        const bool first = t < 12;
        const int jt = first ? t / 3 : (t - 12) / 4, kt = first ? t % 3 : (t - 12) % 4;
        ta[i] = (first ? &sm.d1[0][0] : &sm.d2[0][0]) + 16 * jt + col;
        tb[i] = (first ? &sm.x[0][0] : &sm.h[0][0]) + 16 * kt + col;
    }
    float4(*sp)[HT][64] = reinterpret_cast<float4(*)[HT][64]>(&sm.d1[0][0]);
    for (int64_t b0 = r0; b0 < r1; b0 += RB) {
        *reinterpret_cast<uint4 *>(&sm.x[xr][xc]) = xv;
        if (!FWD) *reinterpret_cast<uint4 *>(&sm.h[xr][xc]) = hv;
        if (tid < RB) {
            sm.y[tid] = yv;
            if (!FWD) sm.g[tid] = zv;     // the row's logit until its row term replaces it
        }
        float h2v[HT][4];
        if (!FWD)
#pragma unroll
            for (int i = 0; i < HT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) h2v[i][r] = h2n[i][r];
        fetch(b0 + RB);                   // the next batch's rows arrive during this one
        __syncthreads();                  // batch (and, first, weights) in LDS
        float z = 0.0f;
        if (FWD) {
            // mlp_tile's products, each wave its half of the units; the lower
            // half then adds both halves' terms of the logits in mlp_tile's order
            f32x4 a[HT];
#pragma unroll
            for (int i = 0; i < HT; ++i) {
                a[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ks = 0; ks < KP / 32; ++ks)
                    a[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        load8(&sm.w.w1[16 * (HT * half + i) + col][32 * ks + 8 * q]),
                        load8(&sm.x[rl][32 * ks + 8 * q]), a[i], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < HT; ++i)
                *reinterpret_cast<uint2 *>(&sm.h[rl][u0 + 16 * i]) =
                    relu4(a[i], *reinterpret_cast<const float4 *>(&sm.w.b1[u0 + 16 * i]));
            __syncthreads();              // both halves of the hidden layer
            float p[HT][4];
#pragma unroll
            for (int i = 0; i < HT; ++i) {
                a[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ks = 0; ks < KP / 32; ++ks)
                    a[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        layer2_k(sm.w.w2[16 * (HT * half + i) + col], ks, q), layer2_k(sm.h[rl], ks, q), a[i],
                        0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < HT; ++i) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float s = a[i][r] + sm.w.b2[u0 + 16 * i + r];
                    h2v[i][r] = s > 0.0f ? s : 0.0f;
                    p[i][r] = h2v[i][r] * sm.w.w3[u0 + 16 * i + r];
                }
                if (half) sp[rg][i][l] = make_float4(p[i][0], p[i][1], p[i][2], p[i][3]);
            }
            __syncthreads();              // the upper half's terms
            if (!half) {
                float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int i = 0; i < HT; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) t[r] += p[i][r];
#pragma unroll
                for (int i = 0; i < HT; ++i) {
                    const float4 v = sp[rg][i][l];
                    t[0] += v.x;
                    t[1] += v.y;
                    t[2] += v.z;
                    t[3] += v.w;
                }
                z = logit_sum(t) + sm.w.b3;
            }
        }
        // row terms: the first quarter of the lower half takes the group's rows
        if (!half && q == 0) {
            const int64_t row = b0 + rl;
            if (!FWD) z = sm.g[rl];
            const float t = sm.y[rl];
            const bool live = row < r1;
            const float gr = live ? (1.0f / (1.0f + expf(-z)) - t) / (float)n : 0.0f;
            sm.g[rl] = gr;
            sg += gr;
            if (live) loss_rows[row] = (z > 0.0f ? z : 0.0f) - z * t + log1pf(expf(-fabsf(z)));
        }
        __syncthreads();                  // g
        {
            const float gr = sm.g[rl];
#pragma unroll
            for (int i = 0; i < HT; ++i) {
                float dj[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    dj[r] = h2v[i][r] > 0.0f ? gr * sm.w.w3[u0 + 16 * i + r] : 0.0f;
                    sb2[i][r] += dj[r];
                    sw3[i][r] += gr * h2v[i][r];
                }
                const float4 v = make_float4(dj[0], dj[1], dj[2], dj[3]);
                *reinterpret_cast<float4 *>(&sm.d2[rl][u0 + 16 * i]) = v;
                *reinterpret_cast<float4 *>(&sm.d2r[rl][u0 + 16 * i]) = v;
            }
        }
        __syncthreads();                  // dz2 of both halves
        // dz1 (16 x 32) = dz2 (16 x 64) W2 (64 x 32), masked where h1 is zero
        {
            f32x4 d[HT];
#pragma unroll
            for (int i = 0; i < HT; ++i) d[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < NH / 4; ++ks) {
                const float a = sm.d2r[rl][4 * ks + q];
#pragma unroll
                for (int i = 0; i < HT; ++i)
                    d[i] = mfma_f32(a, bf2f(sm.w.w2[4 * ks + q][16 * (HT * half + i) + col]), d[i]);
            }
#pragma unroll
            for (int i = 0; i < HT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int j = 16 * (HT * half + i) + col, row = 16 * rg + 4 * q + r;
                    const float v = sm.h[row][j] != 0 ? d[i][r] : 0.0f;
                    sm.d1[row][j] = v;
                    sb1[i] += v;
                }
        }
        __syncthreads();   // every wave's rows in LDS
        // the wave's gradient tiles t = w + GW i over the batch's 64 rows,
        // four rows per step; the tiles' products of one step are independent
        // (the last waves' fourth tile is not stored)
#pragma unroll 4
        for (int s = 0; s < RB / 4; ++s) {
            const int row = 4 * s + q;
#pragma unroll
            for (int i = 0; i < GT_W; ++i)
                acc[i] = mfma_f32(ta[i][row * DS], bf2f(tb[i][row * LD]), acc[i]);
        }
        __syncthreads();   // the tiles are rewritten by the next batch
    }
    // the chunk's partial gradient
    float *pc = part + (int64_t)blockIdx.x * NPARAM;
#pragma unroll
    for (int i = 0; i < GT_W; ++i) {
        const int t = w + GW * i;
        if (t >= GT) break;
        const bool first = t < 12;
        const int jt = first ? t / 3 : (t - 12) / 4, kt = first ? t % 3 : (t - 12) % 4;
        const int k = 16 * kt + col;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = 16 * jt + 4 * q + r;
            if (first) {
                if (k < NIN) pc[OFF_W1 + j * NIN + k] = acc[i][r];
            } else {
                pc[OFF_W2 + j * NH + k] = acc[i][r];
            }
        }
    }
    // vector sums: the group's 16 rows, then the groups in order
#pragma unroll
    for (int i = 0; i < HT; ++i) {
        float a = sb1[i];
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        if (q == 0) sm.vs[rg][0][16 * (HT * half + i) + col] = a;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float b = row_sum16(sb2[i][r]), c = row_sum16(sw3[i][r]);
            if (col == 15) {
                sm.vs[rg][1][u0 + 16 * i + r] = b;
                sm.vs[rg][2][u0 + 16 * i + r] = c;
            }
        }
    }
    sg = row_sum16(sg);
    if (!half && l == 15) sm.gs[rg] = sg;
    __syncthreads();
    if (tid < 3 * NH) {
        const int v = tid / NH, j = tid % NH;
        float a = 0.0f;
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) a += sm.vs[ww][v][j];
        pc[(v == 0 ? OFF_B1 : v == 1 ? OFF_B2 : OFF_W3) + j] = a;
    } else if (tid == 3 * NH) {
        float a = 0.0f;
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) a += sm.gs[ww];
        pc[OFF_B3] = a;
    }
}

// mean of the per-row losses: one block, fixed-order partials and tree;
// GP_U rows per thread are loaded before they are added
constexpr int GP_U = 16;


__device__ __forceinline__ void loss_body(const float *loss_rows, int64_t n, float *loss)
{
    __shared__ float part[BLOCK];
    float acc = 0.0f;
    // GP_U rows per thread in flight at once, added in row order
    for (int64_t rb = threadIdx.x; rb < n; rb += (int64_t)GP_U * blockDim.x) {
        float v[GP_U];
#pragma unroll
        for (int u = 0; u < GP_U; ++u) {
            const int64_t r = rb + (int64_t)u * blockDim.x;
            v[u] = r < n ? loss_rows[r] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < GP_U; ++u)
            if (rb + (int64_t)u * blockDim.x < n) acc += v[u];
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int s = BLOCK / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = n > 0 ? part[0] / (float)n : 0.0f;
}

// Adam with bias correction; c1 = 1 - beta1^t, c2 = 1 - beta2^t
struct AdamArgs {
    float *m, *v;
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_update(float &p, float &m, float &v, float gr, const AdamArgs &a)
{
    m = a.b1 * m + (1.0f - a.b1) * gr;
    v = a.b2 * v + (1.0f - a.b2) * gr * gr;
    p -= a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
}

__global__ void k_mlp_adam(float *P, const float *grad, AdamArgs a)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= NPARAM) return;
    float q = P[p], m = a.m[p], v = a.v[p];
    adam_update(q, m, v, grad[p], a);
    a.m[p] = m;
    a.v[p] = v;
    P[p] = q;
}

// The end of a backward pass in one launch: grad[p] is the sum of the
// chunks' partials, followed (ADAM) by the Adam update of parameter p with the
// same operations as k_mlp_adam; the block past the parameters takes the mean
// loss (loss_body).  A block takes RD_P parameters: wave w loads chunks w,
// w + 4, ..., all in flight, and adds them in that order; the first wave, its
// optimiser state loaded meanwhile, adds the four sums by pairs.  Against 64
// bits dW1 of 8192 rows is 6.3e-8 off like this, 1.69e-7 with the 128 chunks
// one after the other, 1.22e-7 with 64 chunks of two batches.  Latency bound
// (two loads deep): 3.9 us for 64 or 79 chunks, 4.6 us with one thread loading all
// chunks of a parameter on 28 blocks and the optimiser state after the sum.
constexpr int RD_P = 64;

template <bool ADAM>
__global__ __launch_bounds__(BLOCK) void k_mlp_reduce(const float *part, int nch, float *grad,
                                                      const float *loss_rows, int64_t n, float *loss,
                                                      float *P, AdamArgs a)
{
    if (blockIdx.x == gridDim.x - 1) {
        loss_body(loss_rows, n, loss);
        return;
    }
    __shared__ float s_v[WAVES][RD_P];
    constexpr int PER = GRAD_CHUNKS / WAVES;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, p = blockIdx.x * RD_P + l;
    const bool live = p < NPARAM;
    float m = 0.0f, v = 0.0f, q = 0.0f;
    if (ADAM && w == 0 && live) {
        m = a.m[p];
        v = a.v[p];
        q = P[p];
    }
    float t[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int c = w + WAVES * u;
        t[u] = live && c < nch ? part[(int64_t)c * NPARAM + p] : 0.0f;
    }
    float acc = 0.0f;
#pragma unroll
    for (int u = 0; u < PER; ++u) acc += t[u];   // (past the chunks zeros, which change nothing)
    s_v[w][l] = acc;
    __syncthreads();
    if (w > 0 || !live) return;
    static_assert(WAVES == 4, "four sums");
    acc = (s_v[0][l] + s_v[1][l]) + (s_v[2][l] + s_v[3][l]);
    grad[p] = acc;
    if (ADAM) {
        adam_update(q, m, v, acc, a);
        a.m[p] = m;
        a.v[p] = v;
        P[p] = q;
    }
}

// ---------------------------------------------------------------- scoring in the chain
struct alignas(16) SmScore {
    MlpW w;
    float mean[NIN], istd[NIN];
    uint16_t x[WAVES][64][LD];
    float logit[WAVES][64];
    uint32_t pre[NSH + 1];
};

// Every stored object of one kind (triplets or quintuplets): features in
// registers (lane = object), standardised into the wave's LDS tile, four
// 16-row MFMA tiles per wave, then logit and veto (logit below the
// threshold) stored per object.
template <int KIND>
__global__ __launch_bounds__(BLOCK) void k_mlp_score(EvDev E, Consts K, const float *P,
                                                     const float *mean, const float *istd,
                                                     float threshold)
{
    constexpr int NMD = KIND == OT_T3 ? 3 : 5;
    __shared__ SmScore sm;
    if (upstream_overflow(E)) return;
    const uint32_t n = obj_prefix(E, KIND, sm.pre);
    if (blockIdx.x * (WAVES * 64) >= n) return;   // no rows for this block
    load_weights<BLOCK>(P, sm.w);
    for (int i = threadIdx.x; i < NIN; i += blockDim.x) {
        sm.mean[i] = mean[i];
        sm.istd[i] = istd[i];
    }
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
    for (int k = NIN; k < KP; k += 8)                   // K padding, never rewritten
        *reinterpret_cast<uint4 *>(&sm.x[w][l][k]) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const MlpOps ops = mlp_ops(sm.w);
    for (uint32_t base = blockIdx.x * (WAVES * 64); base < n; base += gridDim.x * (WAVES * 64)) {
        const uint32_t v = base + w * 64 + l;
        const bool live = v < n;
        const int32_t t = live ? obj_at(E, KIND, sm.pre, v) : 0;
        float f[40];
        if (live) {
            MdV Q[NMD];
            MdX X[NMD];
#pragma unroll
            for (int j = 0; j < NMD; ++j) {
                int32_t m;
                if (KIND == OT_T3) m = j == 0 ? E.t3_a[t] : j == 1 ? E.t3_b[t] : E.t3_c[t];
                else m = t5_md(E, t, j);
                Q[j] = load_md(E, m);
                X[j].bend = E.md_bend[m];
                X[j].is2s = E.md_bar[m] >> 1;
            }
            if constexpr (KIND == OT_T3)
                t3_features(K, Q, X, f);
            else
                t5_features(K, Q, X, tri_curv(Q[0], Q[1], Q[2]), tri_curv(Q[2], Q[3], Q[4]), f);
        } else {
#pragma unroll
            for (int k = 0; k < 40; ++k) f[k] = 0.0f;
        }
#pragma unroll
        for (int k = 0; k < NIN; k += 8) {
            uint32_t u[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) u[i] = f2bf((f[k + i] - sm.mean[k + i]) * sm.istd[k + i]);
            *reinterpret_cast<uint4 *>(&sm.x[w][l][k]) = make_uint4(u[0] | (u[1] << 16), u[2] | (u[3] << 16),
                                                                    u[4] | (u[5] << 16), u[6] | (u[7] << 16));
        }
        wave_tile_sync();
#pragma unroll 1
        for (int sub = 0; sub < 4; ++sub) {
            bf16x8 x[KP / 32];
#pragma unroll
            for (int ks = 0; ks < KP / 32; ++ks)
                x[ks] = load8(&sm.x[w][16 * sub + (l & 15)][32 * ks + 8 * (l >> 4)]);
            const float z = mlp_tile(sm.w, ops, x, [](int, const uint2 &, const float4 &) {});
            if (l < 16) sm.logit[w][16 * sub + l] = z;
        }
        wave_tile_sync();
        if (live) {
            const float lg = sm.logit[w][l];
            const uint8_t veto = lg >= threshold ? 0 : 1;
            if (KIND == OT_T3) {
                E.t3_logit[t] = lg;
                E.t3_veto[t] = veto;
            } else {
                E.t5_logit[t] = lg;
                E.t5_veto[t] = veto;
            }
        }
    }
}

// ---------------------------------------------------------------- launchers
static int grid_of(int64_t work, int per_block)
{
    int64_t g = (work + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > GRID_MAX) g = GRID_MAX;
    return (int)g;
}

// Up to GRAD_FEW batches there are no more chunks than that.  Past them a
// workspace of GRAD_FEW chunks is accepted, with two batches per chunk where
// one of GRAD_CHUNKS has one: the backward call 19.9 us against 15.0 at 5000
// rows, 20.4 against 16.2 at 8192.
size_t mlp_workspace_least(int64_t n) { return sizeof(float) * work_floats(n, GRAD_FEW); }

size_t mlp_workspace_bytes(int64_t n)
{
    return sizeof(float) * work_floats(n, n <= (int64_t)GRAD_FEW * RB ? GRAD_FEW : GRAD_CHUNKS);
}

hipError_t mlp_prepare(const float *F, const float *mean, const float *istd, int64_t n, uint16_t *X,
                       hipStream_t s)
{
    if ((((uintptr_t)F | (uintptr_t)X) & 15) == 0)
        hipLaunchKernelGGL(k_mlp_prepare8, dim3(grid_of(n * 8, BLOCK)), dim3(BLOCK), 0, s, F, mean, istd, n, X);
    else
        hipLaunchKernelGGL(k_mlp_prepare, dim3(grid_of(n * KP, BLOCK)), dim3(BLOCK), 0, s, F, mean,
                           istd, n, X);
    return hipGetLastError();
}

hipError_t mlp_forward(const float *P, const uint16_t *X, int64_t n, float *logits, uint16_t *h1,
                       float *h2, hipStream_t s)
{
    const int grid = std::min(grid_of((n + 15) / 16, WAVES), FWD_BLOCKS);
    if (h1)
        hipLaunchKernelGGL(k_mlp_forward<true>, dim3(grid), dim3(BLOCK), 0, s, P, X, n, logits, h1, h2);
    else
        hipLaunchKernelGGL(k_mlp_forward<false>, dim3(grid), dim3(BLOCK), 0, s, P, X, n, logits, h1, h2);
    return hipGetLastError();
}

hipError_t mlp_backward(const float *P, const uint16_t *X, const uint8_t *y, int64_t n,
                        const float *logits, const uint16_t *h1, const float *h2, float *work,
                        size_t work_bytes, float *grad, float *loss, hipStream_t s)
{
    float *lrow = work, *part = work + n;
    int nch;
    int64_t clen;
    grad_chunks(n, work_bytes, nch, clen);
    hipLaunchKernelGGL(k_mlp_grad<false>, dim3(nch), dim3(GB), 0, s, P, X, y, n, clen, logits, h1,
                       h2, lrow, part);
    // the chunk sums and the mean loss in one launch (the loss in the last block)
    hipLaunchKernelGGL(k_mlp_reduce<false>, dim3((NPARAM + RD_P - 1) / RD_P + 1), dim3(BLOCK), 0, s,
                       part, nch, grad, lrow, n, loss, nullptr, AdamArgs{});
    return hipGetLastError();
}

// One Adam step on n rows in two launches, with the same operations in the
// same order as mlp_forward, mlp_backward and mlp_adam one after the other:
// the forward fused with the per-chunk gradient products, then the chunk
// reduction with the Adam update and the mean loss.
hipError_t mlp_train_step(float *P, const uint16_t *X, const uint8_t *y, int64_t n, float *work,
                          size_t work_bytes, float *grad, float *loss, float *m, float *v, float lr,
                          float b1, float b2, float eps, float c1, float c2, hipStream_t s)
{
    float *lrow = work, *part = work + n;
    int nch;
    int64_t clen;
    grad_chunks(n, work_bytes, nch, clen);
    hipLaunchKernelGGL(k_mlp_grad<true>, dim3(nch), dim3(GB), 0, s, P, X, y, n, clen, nullptr,
                       nullptr, nullptr, lrow, part);
    hipLaunchKernelGGL(k_mlp_reduce<true>, dim3((NPARAM + RD_P - 1) / RD_P + 1), dim3(BLOCK), 0, s,
                       part, nch, grad, lrow, n, loss, P, AdamArgs{m, v, lr, b1, b2, eps, c1, c2});
    return hipGetLastError();
}

// ---------------------------------------------------------------- fixed workspace
// Workspace of the backward pass for callers that cannot allocate: one
// file-scope device array, one copy per GPU, held until the process ends.
// In host code the name `scratch` is only a stand-in for the symbol; its
// device address on each GPU comes from hipGetSymbolAddress, taken once per
// device with that device current, and only that address is ever passed on.
static __device__ __align__(256) float scratch[MLP_FIXED_SCRATCH_FLOATS];
static_assert(sizeof(float) * ((size_t)MLP_FIXED_MAX_ROWS + (size_t)GRAD_CHUNKS * NPARAM) <=
                  sizeof(scratch),
              "fixed workspace holds MLP_FIXED_MAX_ROWS rows");

static std::mutex scratch_mu;
static void *scratch_at[MLP_FIXED_MAX_DEVICES];

hipError_t mlp_fixed_scratch(int device, void **out)
{
    *out = nullptr;
    if (device < 0 || device >= MLP_FIXED_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_at[device]) {
        int cur = 0;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if ((e = hipSetDevice(device)) != hipSuccess) return e;
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        const hipError_t back = hipSetDevice(cur);
        if (e != hipSuccess) return e;
        if (back != hipSuccess) return back;
        scratch_at[device] = p;
    }
    *out = scratch_at[device];
    return hipSuccess;
}

hipError_t mlp_adam(float *P, const float *grad, float *m, float *v, float lr, float b1, float b2,
                    float eps, float c1, float c2, hipStream_t s)
{
    hipLaunchKernelGGL(k_mlp_adam, dim3((NPARAM + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, s, P, grad,
                       AdamArgs{m, v, lr, b1, b2, eps, c1, c2});
    return hipGetLastError();
}

hipError_t mlp_score(const EvDev &E, const Consts &K, int kind, const float *P, const float *mean,
                     const float *istd, float threshold, int grid, hipStream_t s)
{
    if (kind == OT_T3)
        hipLaunchKernelGGL(k_mlp_score<OT_T3>, dim3(grid), dim3(BLOCK), 0, s, E, K, P, mean, istd,
                           threshold);
    else
        hipLaunchKernelGGL(k_mlp_score<OT_T5>, dim3(grid), dim3(BLOCK), 0, s, E, K, P, mean, istd,
                           threshold);
    return hipGetLastError();
}

}  // namespace lst
