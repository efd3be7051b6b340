// mlp.hip -- BF16 matrix-core kernels of the flow-map surrogate network.
//
// The surrogate is a fully connected network 64 -> 256 -> 256 -> 256 -> 256 -> 2 with
// the tanh form of GELU after each hidden layer (Hendrycks & Gimpel, 2016).  Weights
// and activations are bfloat16, products accumulate in FP32 on the gfx950 matrix
// cores (v_mfma_f32_32x32x16_bf16), and the optimiser keeps FP32 master weights.
//
// A training step is three kernels: k_train_pass (forward, loss and the gradients of
// every pre-activation, 32 rows a block), k_train_wgrad (the weight gradients, partial
// sums over eight parts of the batch) and k_train_update (their sum, Adam and the
// bfloat16 copies).  Inference is one kernel, k_mlp_fused.
#include "lp_internal.h"

namespace lp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr float kC0 = 0.7978845608028654f;  // sqrt(2/pi)
constexpr float kC1 = 0.044715f;

// GELU(x) and its derivative
__device__ inline void gelu_and_grad(float x, float &g, float &gg)
{
    const float t = tanhf(kC0 * (x + kC1 * x * x * x));
    g = 0.5f * x * (1.f + t);
    gg = 0.5f * (1.f + t) + 0.5f * x * (1.f - t * t) * kC0 * (1.f + 3.f * kC1 * x * x);
}

__device__ inline uint16_t bf16_bits(float f)
{
    uint32_t b = __float_as_uint(f);
    if ((b & 0x7F800000u) == 0x7F800000u && (b & 0x007FFFFFu))
        return (uint16_t)((b >> 16) | 0x40u);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}

// the first nvalid of n values rounded, the rest zero
__global__ void k_to_bf16(const float *x, int64_t nvalid, int64_t n, uint16_t *y)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] = i < nvalid ? bf16_bits(x[i]) : (uint16_t)0;
}

// ---------------------------------------------------------------- fused inference
// The whole network on one tile of 256 rows per block, activations in registers.
// Each layer is computed transposed, H^T = W^T A^T, so the weights are the matrix
// core's A operand (read from LDS, where the block streams them half a layer at a time) and
// the activations its B operand: lane l keeps 8 consecutive features of row
// (l mod 32) for each k-step.  The accumulator of the 32x32x16 product leaves lane
// l with features 8(v/4) + 4(l/32) + (v mod 4) of that row; two permlane32 swaps per
// 32-feature block move each half-wave's missing four features across, which is
// exactly the next layer's B-operand layout.  GELU in the sigmoid form
// x / (1 + exp(-2u)), u = sqrt(2/pi) (x + 0.044715 x^3), on the hardware exp2 and
// reciprocal; bf16 rounding by the round-to-nearest-even convert.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kFusedRows = 256;      // rows per tile: 8 waves x 32
constexpr int kFusedThreads = 512;
constexpr int kStride256 = 256 + 8;  // bf16 per staged weight row of a 256-input layer
constexpr int kStride64 = 64 + 8;    // the same for the 64-input first layer (the 8 bf16 of
                                     // padding put 16 consecutive rows on distinct banks)
constexpr int kHalfRows = 128;       // weight rows (output features) per LDS buffer

__device__ inline float gelu_sigmoid(float x)
{
    constexpr float kLog2e = 1.4426950408889634f;
    const float t = x * x;
    const float m = x * fmaf(t, -2.f * kC0 * kC1 * kLog2e, -2.f * kC0 * kLog2e);
    return x * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(m));
}

__device__ inline uint32_t pack_bf16(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
}

// One step of the network on a wave's 32 rows: the products of one 32-feature output
// block with K inputs (weights from LDS rows of STRIDE bf16 at w, biases at b; the
// accumulator starts from the biases of the features the lane holds and takes the K/16
// products in k order), written beside the epilogue of the block before (prev): GELU
// and bf16 of its 16 values, then the half-wave exchange into the next layer's two
// operands o0, o1 for those 32 features.  Left to itself the compiler issues all the
// products first and the epilogue after them; here the step is cut into one piece per
// product, fenced so that nothing moves across: the weights of the product three
// ahead are read from LDS, the product is issued, and a share of the epilogue follows
// while the matrix core works.  At a layer's first block the previous block is the
// previous layer's last one (CROSS): its outputs are this layer's inputs for k-steps
// K/16 - 2 and K/16 - 1 (o0 and o1 alias in[] there), so those two products come last.
template <int K, int STRIDE, bool PREV, bool CROSS>
__device__ inline f32x16 step(const uint16_t *w, const float *b, int r, int h,
                              const bf16x8 (&in)[16], const f32x16 &prev, bf16x8 &o0,
                              bf16x8 &o1)
{
    constexpr int kSteps = K / 16, kAhead = 3, kLate = CROSS ? 2 : 0, kPer = 16 / kSteps;
    static_assert(!CROSS || PREV, "a layer's first block follows the previous layer's last");
    f32x16 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 v = *reinterpret_cast<const float4 *>(b + 8 * q + 4 * h);
        acc[4 * q + 0] = v.x;
        acc[4 * q + 1] = v.y;
        acc[4 * q + 2] = v.z;
        acc[4 * q + 3] = v.w;
    }
    const uint16_t *wr = w + r * STRIDE + 8 * h;
    bf16x8 wq[kSteps];
#pragma unroll
    for (int i = 0; i < kAhead && i < kSteps; ++i)
        wq[i] = *reinterpret_cast<const bf16x8 *>(wr + 16 * i);
    __builtin_amdgcn_sched_barrier(0);
    float g[16];
    uint32_t P[8];
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        if (i + kAhead < kSteps)
            wq[i + kAhead] = *reinterpret_cast<const bf16x8 *>(wr + 16 * (i + kAhead));
        if (i < kSteps - kLate)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wq[i], in[i], acc, 0, 0, 0);
        if constexpr (PREV) {
#pragma unroll
            for (int v = i * kPer; v < (i + 1) * kPer; ++v) {
                g[v] = gelu_sigmoid(prev[v]);
                if (v & 1)
                    P[v >> 1] = pack_bf16(g[v - 1], g[v]);
                // lanes 32-63 of the first register trade places with lanes 0-31 of the
                // second, once both are packed
                if (v == 7 || v == 15) {
                    const int j0 = v == 7 ? 0 : 4;
#pragma unroll
                    for (int j = j0; j < j0 + 2; ++j) {
                        auto x = __builtin_amdgcn_permlane32_swap(P[j], P[j + 2], false, false);
                        P[j] = x[0];
                        P[j + 2] = x[1];
                    }
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (PREV) {
        o0 = __builtin_bit_cast(bf16x8, u32x4_t{P[0], P[1], P[2], P[3]});
        o1 = __builtin_bit_cast(bf16x8, u32x4_t{P[4], P[5], P[6], P[7]});
    }
    if constexpr (CROSS) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wq[kSteps - 2], o0, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wq[kSteps - 1], o1, acc, 0, 0, 0);
    }
    return acc;
}

typedef __attribute__((address_space(3))) void *lds_ptr_t;

// Rows [0, R) of a row-major [R x K] bf16 matrix at src, loaded straight into LDS rows
// of STRIDE bf16 at dst without passing through registers: K/8 lanes carry a row, 16
// bytes each.  Such a load writes its lanes' 16-byte pieces one after the other from
// one wave-uniform LDS address, so each row is one load with the lanes of the other
// rows switched off.  Row n0 + q of a group of G rows starts 16 q bytes past
// n0 STRIDE*2 + q K*2 (the padding of the rows before it); that shift goes into the
// load's immediate offset, which the hardware adds to the global address as well (the
// lanes' pointers are moved back by it).  The LDS address is then the same for the G
// loads of a group, and their immediates differ, so the compiler can never fold the
// G masked loads into one.  Wave w takes rows w R/8 .. (w + 1) R/8 - 1.  The loads
// count as the wave's vector-memory operations until the data is in LDS.
template <int Q, int G>
__device__ inline void load_row_group(const uint16_t *p, lds_ptr_t d, int g)
{
    if constexpr (Q < G) {
        if (g == Q)
            __builtin_amdgcn_global_load_lds(p, d, 16, 16 * Q, 0);
        load_row_group<Q + 1, G>(p, d, g);
    }
}

template <int R, int K, int STRIDE>
__device__ inline void load_rows_to_lds(uint16_t *dst, const uint16_t *src, int wave, int lane)
{
    constexpr int L = K / 8, G = 64 / L, kPerWave = R / 8;
    static_assert(kPerWave % G == 0, "whole groups of rows per wave");
    static_assert(STRIDE * 2 - K * 2 == 16, "16 bytes of padding per row");
    const int g = lane / L, c = lane % L;
#pragma unroll
    for (int i = 0; i < kPerWave; i += G) {
        const int n0 = wave * kPerWave + i;
        const uint16_t *p = src + (size_t)(n0 + g) * K + c * 8 - 8 * g;
        const lds_ptr_t d = (lds_ptr_t)(reinterpret_cast<char *>(dst) + n0 * STRIDE * 2);
        load_row_group<0, G>(p, d, g);
    }
}

// The wave's own loads into LDS have landed; after the barrier every wave's have, and
// every wave is done reading the buffer that the loads issued next overwrite.
__device__ inline void chunk_sync()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// Weights stream through two LDS buffers in eight chunks per tile: the first layer
// (buffer 0), then each 256-input layer as output features 0-127 (buffer 1) and
// 128-255 (buffer 0), then the output layer (buffer 1).  Each chunk's loads are issued
// one chunk ahead, right after the barrier that frees their buffer, so they run while
// the matrix core works on the other buffer.  Eight chunks per tile keep every
// chunk's buffer the same from tile to tile, so each access names its buffer at
// compile time (and the compiler waits for loads into one buffer only before reading
// that one).
__global__ __launch_bounds__(kFusedThreads) void k_mlp_fused(MlpFusedArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t buf0[kHalfRows * kStride256];
    __shared__ __attribute__((aligned(16))) uint16_t buf1[kHalfRows * kStride256];
    __shared__ __attribute__((aligned(16))) float bl[4 * 256 + 32];
    static_assert(256 * kStride64 <= kHalfRows * kStride256, "first layer fits one buffer");
    const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t ntile = (a.rows + kFusedRows - 1) / kFusedRows;
    for (int c = threadIdx.x; c < 4 * 256 + 32; c += kFusedThreads)
        bl[c] = c < 1024 ? a.bias[c >> 8][c & 255] : a.bias[4][c - 1024];
    load_rows_to_lds<256, 64, kStride64>(buf0, a.WT[0], wave, lane);  // grid <= tiles
    for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
        const int64_t row = tile * kFusedRows + wave * 32 + r;
        const bool live = row < a.rows;
        bf16x8 in[16], out[16];
#pragma unroll
        for (int s = 0; s < 4; ++s)
            in[s] = live ? *reinterpret_cast<const bf16x8 *>(a.X + row * 64 + 16 * s + 8 * h)
                         : bf16x8{};
        chunk_sync();
        load_rows_to_lds<128, 256, kStride256>(buf1, a.WT[1], wave, lane);
        // first layer, 64 inputs, weights in buffer 0
        f32x16 cur = step<64, kStride64, false, false>(buf0, bl, r, h, in, f32x16{}, out[0], out[1]);
#pragma unroll
        for (int nb = 1; nb < 8; ++nb)
            cur = step<64, kStride64, true, false>(buf0 + nb * 32 * kStride64, bl + nb * 32, r, h,
                                                   in, cur, out[2 * nb - 2], out[2 * nb - 1]);
        // 256-input layers: output features 0-127 from buffer 1, 128-255 from buffer 0
#pragma unroll 1
        for (int l = 1; l < 4; ++l) {
            chunk_sync();
            load_rows_to_lds<128, 256, kStride256>(buf0, a.WT[l] + 128 * 256, wave, lane);
            const float *bias = bl + 256 * l;
#pragma unroll
            for (int s = 0; s < 14; ++s)
                in[s] = out[s];
            cur = step<256, kStride256, true, true>(buf1, bias, r, h, in, cur, in[14], in[15]);
#pragma unroll
            for (int nb = 1; nb < 4; ++nb)
                cur = step<256, kStride256, true, false>(buf1 + nb * 32 * kStride256, bias + nb * 32,
                                                         r, h, in, cur, out[2 * nb - 2],
                                                         out[2 * nb - 1]);
            chunk_sync();
            if (l < 3)
                load_rows_to_lds<128, 256, kStride256>(buf1, a.WT[l + 1], wave, lane);
            else
                load_rows_to_lds<32, 256, kStride256>(buf1, a.WT[4], wave, lane);
#pragma unroll
            for (int nb = 4; nb < 8; ++nb)
                cur = step<256, kStride256, true, false>(buf0 + (nb - 4) * 32 * kStride256,
                                                         bias + nb * 32, r, h, in, cur,
                                                         out[2 * nb - 2], out[2 * nb - 1]);
        }
        // output layer, weights in buffer 1; the next tile's first layer goes to buffer 0
        chunk_sync();
        if (tile + gridDim.x < ntile)
            load_rows_to_lds<256, 64, kStride64>(buf0, a.WT[0], wave, lane);
#pragma unroll
        for (int s = 0; s < 14; ++s)
            in[s] = out[s];
        const f32x16 y = step<256, kStride256, true, true>(buf1, bl + 1024, r, h, in, cur, in[14],
                                                           in[15]);
        // outputs 0 and 1 of the row sit in values 0 and 1 of the lower half-wave
        if (live && h == 0) {
            a.Y[row * 2 + 0] = y[0];
            a.Y[row * 2 + 1] = y[1];
        }
    }
}

// ---------------------------------------------------------------- training
// Forward, loss and backward to every pre-activation for 32 rows of the batch, in one
// kernel: the layers one after the other inside a block, so the activations never leave
// it (layer by layer through memory a step was about 35 launches of 4 to 40 us).  Eight
// waves; wave w owns output features 32 w .. 32 w + 31 of every layer, computed
// transposed as in k_mlp_fused: weights (16 fragments straight from L2, each used once
// by the block) are the matrix core's A operand, the layer's inputs its B operand, read
// from LDS where the waves leave them bf16 [row][feature].  The derivatives of the four
// layers' GELU wait in 128 KB of LDS from the forward pass for the backward one, each
// thread reading back what it wrote.  The products take k in increasing order into one
// accumulator per output from zero, the bias is added after them, and values round to
// bf16 where they are handed on, as the layers' definition says, so the gradients of a
// row's pre-activations do not depend on the rows that share its block; the sums over
// rows are k_train_wgrad's, in parts whose number goes with the batch.  32 rows a block
// because the matrix instruction is 32 wide and a batch of 4096 then fills half the CUs;
// what bounds a block is reading the weights (1.1 MB at 64 B per clock, about 8 us).
constexpr int kActStride = kNetHid + 8;  // bf16 per activation row in LDS (no conflicts)

// Two rows' bf16 values of two adjacent features, exchanged between neighbouring lanes
// (rows r and r ^ 1): lane r even gets feature v of rows r, r + 1, lane r odd feature
// v + 1 of rows r - 1, r.
__device__ inline uint32_t pair_rows(uint32_t p, int r)
{
    const uint32_t q = (uint32_t)__builtin_amdgcn_mov_dpp((int)p, 0xB1, 0xF, 0xF, true);
    return (r & 1) ? (q >> 16) | (p & 0xFFFF0000u) : (p & 0xFFFFu) | (q << 16);
}

// One wave's 32 features of 32 rows as bf16: into the LDS rows at act, and feature by
// feature to dst [256][rows].
__device__ inline void put_features(const float g[16], uint16_t *act, uint16_t *dst, int64_t rows,
                                    int64_t row0, int f0, int r, int h)
{
    uint32_t P[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        P[j] = pack_bf16(g[2 * j], g[2 * j + 1]);
    // one lane offset for every store; the rest of the address is the wave's
    const uint32_t at = (uint32_t)(4 * h + (r & 1)) * (uint32_t)rows + (uint32_t)(r & ~1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        *reinterpret_cast<uint2 *>(act + r * kActStride + f0 + 8 * q + 4 * h) =
            uint2{P[2 * q], P[2 * q + 1]};
#pragma unroll
        for (int j = 0; j < 2; ++j)
            *reinterpret_cast<uint32_t *>(dst + (int64_t)(f0 + 8 * q + 2 * j) * rows + row0 + at) =
                pair_rows(P[2 * q + j], r);
    }
}

// The sums over the block's 32 rows of one wave's 32 features, to out[f0 ..]: halves of
// the 16 values trade between lanes until each lane holds one value of 16 rows.
__device__ inline void put_row_sums(const float g[16], float *out, int f0, int r, int h)
{
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
        v[i] = g[i];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int n = 8 >> s, hi = (r >> s) & 1;
#pragma unroll
        for (int i = 0; i < n; ++i) {
            const float keep = hi ? v[i + n] : v[i], give = hi ? v[i] : v[i + n];
            v[i] = keep + __shfl_xor(give, 1 << s, 64);
        }
    }
    const float t = v[0] + __shfl_xor(v[0], 16, 64);
    const int i = 8 * (r & 1) + 4 * ((r >> 1) & 1) + 2 * ((r >> 2) & 1) + ((r >> 3) & 1);
    if (r < 16)
        out[f0 + 8 * (i >> 2) + 4 * h + (i & 3)] = t;
}

template <int LO, int HI>
__device__ inline void load_frags(bf16x8 (&w)[16], const uint16_t *p)
{
#pragma unroll
    for (int i = LO; i < HI; ++i)
        w[i] = *reinterpret_cast<const bf16x8 *>(p + 16 * i);
}

// Products of the wave's fragments with the LDS rows (256 inputs).
__device__ inline f32x16 act_product(const bf16x8 (&w)[16], const uint16_t *act, int r, int h)
{
    f32x16 acc = {};
#pragma unroll
    for (int i = 0; i < 16; ++i)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            w[i], *reinterpret_cast<const bf16x8 *>(act + r * kActStride + 16 * i + 8 * h), acc, 0,
            0, 0);
    return acc;
}

__global__ __launch_bounds__(512) void k_train_pass(TrainArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t act[kTrainRows * kActStride];
    __shared__ float4 grad[4][4][512];  // GELU derivatives [layer][value / 4][thread]
    const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int f0 = 32 * wave;
    const int64_t row0 = (int64_t)blockIdx.x * kTrainRows, row = row0 + r, rows = a.rows;
    bf16x8 w[16], x[4];
    load_frags<0, 4>(w, a.WT[0] + (f0 + r) * kNetIn + 8 * h);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        x[i] = *reinterpret_cast<const bf16x8 *>(a.X + row * kNetIn + 16 * i + 8 * h);
    {  // the input features, transposed: wave w takes features 8 w .. 8 w + 7
        const int f = 8 * wave + 4 * h;
        const uint2 q = *reinterpret_cast<const uint2 *>(a.X + row * kNetIn + f);
        const uint32_t p0 = pair_rows(q.x, r), p1 = pair_rows(q.y, r);
        *reinterpret_cast<uint32_t *>(a.XT + (f + (r & 1)) * rows + row0 + (r & ~1)) = p0;
        *reinterpret_cast<uint32_t *>(a.XT + (f + 2 + (r & 1)) * rows + row0 + (r & ~1)) = p1;
    }
    float g[16];
    f32x16 acc = {};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[i], x[i], acc, 0, 0, 0);
    // The layers share one piece of code (unrolled, a block spent its time fetching 36 KB
    // of instructions, each used once).  The next layer's weights (after the last hidden
    // layer the output layer's 32 rows, two of them outputs, for every wave) are on their
    // way across the GELU.
#pragma unroll 1
    for (int l = 0; l < 4; ++l) {
        float4 bq[4];  // (read before the weights: reads return in order)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            bq[q] = *reinterpret_cast<const float4 *>(a.bias[l] + f0 + 4 * h + 8 * q);
        __builtin_amdgcn_sched_barrier(0);
        load_frags<0, 16>(w, l < 3 ? a.WT[l + 1] + (f0 + r) * kNetHid + 8 * h
                                   : a.WT[4] + r * kNetHid + 8 * h);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 b = bq[q];
            float4 d;
            gelu_and_grad(acc[4 * q + 0] + b.x, g[4 * q + 0], d.x);
            gelu_and_grad(acc[4 * q + 1] + b.y, g[4 * q + 1], d.y);
            gelu_and_grad(acc[4 * q + 2] + b.z, g[4 * q + 2], d.z);
            gelu_and_grad(acc[4 * q + 3] + b.w, g[4 * q + 3], d.w);
            grad[l][q][threadIdx.x] = d;
        }
        if (l)
            __syncthreads();  // every wave has read the layer before
        put_features(g, act, a.HT[l], rows, row0, f0, r, h);
        __syncthreads();
        acc = act_product(w, act, r, h);
    }
    // outputs and their gradient: every wave computes them, so none waits for another
    float d0 = 0.f, d1 = 0.f, loss = 0.f;
    if (h == 0) {  // outputs 0 and 1 of row r are values 0 and 1 of the lower half-wave
        const float2 t = *reinterpret_cast<const float2 *>(a.T + 2 * row);
        const float e0 = (acc[0] + a.bias[4][0]) - t.x, e1 = (acc[1] + a.bias[4][1]) - t.y;
        d0 = e0 * a.inv_b;
        d1 = e1 * a.inv_b;
        loss = 0.5f * e0 * e0 * a.inv_b + 0.5f * e1 * e1 * a.inv_b;
    }
    const uint32_t dq = pack_bf16(d0, d1);  // zero in the upper half-wave, as its k's are
    if (wave == 0) {
        float s0 = d0, s1 = d1;
        for (int off = 16; off > 0; off >>= 1) {
            loss += __shfl_xor(loss, off, 64);
            s0 += __shfl_xor(s0, off, 64);
            s1 += __shfl_xor(s1, off, 64);
        }
        if (lane == 0) {
            a.lpart[blockIdx.x] = loss;
            a.bpart[(int64_t)blockIdx.x * kNetBiases + 4 * kNetHid] = s0;
            a.bpart[(int64_t)blockIdx.x * kNetBiases + 4 * kNetHid + 1] = s1;
        }
        if (h == 0) {
            a.DO[row] = (uint16_t)(dq & 0xFFFFu);
            a.DO[rows + row] = (uint16_t)(dq >> 16);
        }
    }
    // backward: the gradient of layer l's pre-activations from layer l + 1's; the outputs'
    // 30 padding columns are zero, so their product takes the first 16 of 32 k's
    const bf16x8 wo = *reinterpret_cast<const bf16x8 *>(a.Wb[4] + (f0 + r) * kNetOutPad + 8 * h);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
        wo, __builtin_bit_cast(bf16x8, u32x4_t{dq, 0u, 0u, 0u}), f32x16{}, 0, 0, 0);
#pragma unroll 1
    for (int l = 3; l >= 0; --l) {
        if (l)
            load_frags<0, 16>(w, a.Wb[l] + (f0 + r) * kNetHid + 8 * h);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 d = grad[l][q][threadIdx.x];
            g[4 * q + 0] = acc[4 * q + 0] * d.x;
            g[4 * q + 1] = acc[4 * q + 1] * d.y;
            g[4 * q + 2] = acc[4 * q + 2] * d.z;
            g[4 * q + 3] = acc[4 * q + 3] * d.w;
        }
        __syncthreads();  // every wave has read the layer before
        put_features(g, act, a.DT[l], rows, row0, f0, r, h);
        put_row_sums(g, a.bpart + (int64_t)blockIdx.x * kNetBiases + l * kNetHid, f0, r, h);
        if (l == 0)
            break;
        __syncthreads();
        acc = act_product(w, act, r, h);
    }
}

// Weight gradients: dW_l[k][n] = sum over rows of H_l-1[row][k] dZ_l[row][n], a 64 x 64
// tile of one layer (64 x 32 of the output layer) and one part of the batch per block,
// 32 x 32 per wave.  Both operands come feature by feature; 128 rows of the tile's 64 + 64
// features at a time go through LDS, each feature's rows read by 16 neighbouring lanes
// (read straight into the fragments, a load touched 32 cache lines and their lookup was
// the bound: 21.8 us a step of 4096 rows).  The parts are summed by k_train_update in
// order, so a step's gradients are the same from run to run (atomic adds were not).
// Within a part the products of kWgradChain rows make a sum, and these sums the part's, so
// that a large batch's small rows are not lost in one long sum (2^18 rows, most of them
// below half a unit of the large ones' sum: relative error 3.0e-5 in one sum, 2.1e-6 so).
constexpr int kWgradTiles = 4 + 3 * 16 + 4, kWgradRows = 128, kWgradChain = 512;
constexpr int kWgradStride = kWgradRows + 8;  // bf16 per LDS row (no conflicts)

__global__ __launch_bounds__(256) void k_train_wgrad(TrainArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t tile[128 * kWgradStride];
    const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int t = blockIdx.x, l, off = 0, N = kNetHid, ti, tj;
    if (t < 4) {
        l = 0, ti = 0, tj = t;
    } else if (t < 52) {
        t -= 4;
        l = 1 + (t >> 4), ti = (t >> 2) & 3, tj = t & 3;
        off = kNetIn * kNetHid + (l - 1) * kNetHid * kNetHid;
    } else {
        l = 4, ti = t - 52, tj = 0, N = kNetOutPad;
        off = kNetWeights - kNetHid * kNetOutPad;
    }
    const int64_t rows = a.rows, per = (rows / 128 + a.parts - 1) / a.parts * 128;
    const int64_t lo = (int64_t)blockIdx.y * per, hi = lo + per < rows ? lo + per : rows;
    // thread t loads 16 bytes of features t/16 + 16 i: of the inputs (i < 4) and of the
    // gradients (i >= 4; the outputs' gradient has two features, its padding is zero)
    const int f = threadIdx.x >> 4, c = 8 * (threadIdx.x & 15);
    const uint16_t *A = (l == 0 ? a.XT : a.HT[l - 1]) + (int64_t)(64 * ti + f) * rows + c;
    const uint16_t *B = (l < 4 ? a.DT[l] : a.DO) + (int64_t)(64 * tj + f) * rows + c;
    u32x4_t p[8];
    auto load = [&](int64_t k) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = *reinterpret_cast<const u32x4_t *>(A + (int64_t)(16 * i) * rows + k);
            p[4 + i] = u32x4_t{};
            if (l < 4 || f + 16 * i < kNetOut)
                p[4 + i] = *reinterpret_cast<const u32x4_t *>(B + (int64_t)(16 * i) * rows + k);
        }
    };
    const int i0 = 32 * (wave & 1), j0 = 32 * (wave >> 1);
    f32x16 acc = {}, sum = {};
    if (lo < hi)
        load(lo);
    for (int64_t k = lo; k < hi; k += kWgradRows) {
        if (k > lo)
            __syncthreads();  // every wave has read the rows before
#pragma unroll
        for (int i = 0; i < 8; ++i)
            *reinterpret_cast<u32x4_t *>(tile + (16 * i + f) * kWgradStride + c) = p[i];
        __syncthreads();
        if (k + kWgradRows < hi)
            load(k + kWgradRows);
#pragma unroll
        for (int i = 0; i < kWgradRows / 16; ++i)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                *reinterpret_cast<const bf16x8 *>(tile + (i0 + r) * kWgradStride + 16 * i + 8 * h),
                *reinterpret_cast<const bf16x8 *>(tile + (64 + j0 + r) * kWgradStride + 16 * i +
                                                  8 * h),
                acc, 0, 0, 0);
        if ((k - lo) % kWgradChain == kWgradChain - kWgradRows || k + kWgradRows >= hi) {
            sum += acc;
            acc = f32x16{};
        }
    }
    if (64 * tj + j0 >= N)
        return;
    float *out = a.wpart + (int64_t)blockIdx.y * kNetWeights + off;
#pragma unroll
    for (int v = 0; v < 16; ++v)
        out[(64 * ti + i0 + 8 * (v >> 2) + 4 * h + (v & 3)) * N + 64 * tj + j0 + r] = sum[v];
}

__device__ inline float adam_step(float w, float g, float &m, float &v, const UpdateArgs &u)
{
    constexpr float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float mm = b1 * m + (1.f - b1) * g;
    const float vv = b2 * v + (1.f - b2) * g * g;
    m = mm;
    v = vv;
    return w - u.lr * (mm / u.c1) / (sqrtf(vv / u.c2) + eps);
}

// The parameters, a 32 x 32 tile of one layer's weights per block and after those 64
// biases per block: their gradients summed over the partial sums in order and, by MODE,
// applied (Adam, with the bf16 copies W and W^T; the transpose goes through LDS so that
// both are written in runs) or written out packed.  Padding columns stay zero.
constexpr int kUpdateTiles = 16 + 3 * 64 + 8, kUpdateBias = (kNetBiases + 63) / 64;

template <int MODE>
__global__ __launch_bounds__(256) void k_train_update(UpdateArgs u)
{
    constexpr bool kGrad = MODE == kUpAdam || MODE == kUpGrads;
    __shared__ float part[4][64];
    __shared__ uint16_t tr[32][34];
    int t = blockIdx.x;
    if (t >= kUpdateTiles) {  // biases: 64 a block, four threads to each sum
        const int e = (t - kUpdateTiles) * 64 + (threadIdx.x & 63), q = threadIdx.x >> 6;
        float s = 0.f;
        if (kGrad) {
            float c[4] = {0.f, 0.f, 0.f, 0.f};  // (four sums: short, and four reads in flight)
            if (e < kNetBiases)
                for (int k = q; k < u.blocks; k += 16)
#pragma unroll
                    for (int n = 0; n < 4; ++n)
                        c[n] += k + 4 * n < u.blocks
                                    ? u.bpart[(int64_t)(k + 4 * n) * kNetBiases + e]
                                    : 0.f;
            s = (c[0] + c[1]) + (c[2] + c[3]);
            part[q][threadIdx.x & 63] = s;
            __syncthreads();
        }
        if (q == 0 && e < kNetBiases) {
            const int l = e >> 8, j = e & 255;
            const int at = l < 4 ? kNetIn * kNetHid + l * (kNetHid * kNetHid + kNetHid) + j
                                 : kNetParams - kNetOut + j;
            if (kGrad)
                s = (part[0][threadIdx.x] + part[1][threadIdx.x]) +
                    (part[2][threadIdx.x] + part[3][threadIdx.x]);
            if (MODE == kUpAdam)
                u.b[l][j] = adam_step(u.b[l][j], s, u.mb[l][j], u.vb[l][j], u);
            else if (MODE == kUpGrads)
                u.out[at] = s;
            else if (MODE == kUpParams)
                u.out[at] = u.b[l][j];
        }
        if (kGrad && blockIdx.x == gridDim.x - 1 && q == 1 && u.loss) {
            float s1 = 0.f;
            for (int k = threadIdx.x & 63; k < u.blocks; k += 64)
                s1 += u.lpart[k];
            for (int o = 32; o > 0; o >>= 1)
                s1 += __shfl_xor(s1, o, 64);
            if ((threadIdx.x & 63) == 0)
                *u.loss = s1;
        }
        return;
    }
    int l, ti, tj, off, pk;
    if (t < 16) {
        l = 0, ti = t >> 3, tj = t & 7, off = 0, pk = 0;
    } else if (t < 208) {
        t -= 16;
        l = 1 + (t >> 6), ti = (t >> 3) & 7, tj = t & 7;
        off = kNetIn * kNetHid + (l - 1) * kNetHid * kNetHid;
        pk = off + l * kNetHid;
    } else {
        l = 4, ti = t - 208, tj = 0, off = kNetWeights - kNetHid * kNetOutPad;
        pk = off + 4 * kNetHid;
    }
    const int K = l == 0 ? kNetIn : kNetHid, N = l < 4 ? kNetHid : kNetOutPad;
    const int nvalid = l < 4 ? kNetHid : kNetOut;
    const int c = threadIdx.x & 31, j = 32 * tj + c, r0 = threadIdx.x >> 5;
    const bool live = kGrad && j < nvalid;
    // every read of the thread's four weights first (absent parts read the last one)
    float w[4], mm[4], vv[4], q[4][kTrainParts];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int i = (32 * ti + r0 + 8 * n) * N + j;
        w[n] = MODE == kUpGrads ? 0.f : u.W[l][i];
        if (live) {
#pragma unroll
            for (int p = 0; p < kTrainParts; ++p)
                q[n][p] = u.wpart[(int64_t)(p < u.parts ? p : u.parts - 1) * kNetWeights + off + i];
            if (MODE == kUpAdam) {
                mm[n] = u.mW[l][i];
                vv[n] = u.vW[l][i];
            }
        }
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int k = 32 * ti + r0 + 8 * n, i = k * N + j;
        if (live) {
            float g = 0.f;
#pragma unroll
            for (int p = 0; p < kTrainParts; ++p)
                g += p < u.parts ? q[n][p] : 0.f;
            if (MODE == kUpAdam) {
                w[n] = adam_step(w[n], g, mm[n], vv[n], u);
                u.W[l][i] = w[n];
                u.mW[l][i] = mm[n];
                u.vW[l][i] = vv[n];
            } else {
                w[n] = g;
            }
        }
        if (MODE == kUpGrads || MODE == kUpParams) {
            if (j < nvalid)
                u.out[pk + k * nvalid + j] = w[n];
        } else {
            const uint16_t b = bf16_bits(j < nvalid ? w[n] : 0.f);
            u.Wb[l][i] = b;
            tr[c][r0 + 8 * n] = b;
        }
    }
    if (MODE == kUpGrads || MODE == kUpParams)
        return;
    __syncthreads();
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int rr = r0 + 8 * n;
        u.WT[l][(32 * tj + rr) * K + 32 * ti + c] = tr[rr][c];
    }
}

}  // namespace

hipError_t launch_mlp_fused(const MlpFusedArgs &a, hipStream_t s)
{
    if (a.rows <= 0)
        return hipSuccess;
    if (a.rows % 32)
        return hipErrorInvalidValue;
    int cus = 0, dev = 0;
    hipError_t e;
    if ((e = hipGetDevice(&dev)) != hipSuccess ||
        (e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess)
        return e;
    const int64_t ntile = (a.rows + kFusedRows - 1) / kFusedRows;
    const uint32_t grid = (uint32_t)(ntile < cus ? ntile : cus);
    hipLaunchKernelGGL(k_mlp_fused, dim3(grid), dim3(kFusedThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_train_pass(const TrainArgs &a, hipStream_t s)
{
    if (a.rows <= 0 || a.rows % 128 || a.parts < 1 || a.parts > kTrainParts)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_train_pass, dim3((uint32_t)(a.rows / kTrainRows)), dim3(512), 0, s, a);
    hipLaunchKernelGGL(k_train_wgrad, dim3(kWgradTiles, (uint32_t)a.parts), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_train_update(int mode, const UpdateArgs &u, hipStream_t s)
{
    const dim3 grid(kUpdateTiles + kUpdateBias), blk(256);
    switch (mode) {
    case kUpCopies: hipLaunchKernelGGL(k_train_update<kUpCopies>, grid, blk, 0, s, u); break;
    case kUpAdam: hipLaunchKernelGGL(k_train_update<kUpAdam>, grid, blk, 0, s, u); break;
    case kUpGrads: hipLaunchKernelGGL(k_train_update<kUpGrads>, grid, blk, 0, s, u); break;
    case kUpParams: hipLaunchKernelGGL(k_train_update<kUpParams>, grid, blk, 0, s, u); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float *x, int64_t nvalid, int64_t n, uint16_t *y, hipStream_t s)
{
    int64_t b = (n + 255) / 256;
    hipLaunchKernelGGL(k_to_bf16, dim3((uint32_t)(b > 4096 ? 4096 : (b ? b : 1))), dim3(256), 0,
                       s, x, nvalid, n, y);
    return hipGetLastError();
}

}  // namespace lp
