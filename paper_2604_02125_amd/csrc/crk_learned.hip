// crk_learned.hip -- learned troubled-cell indicator for the blending limiter:
// a multilayer perceptron nin -> H -> H -> 1 (ReLU, output alpha_max *
// sigmoid) on the modal energy fractions of rho*p, with BF16 parameters and
// FP32 arithmetic; its training kernels (loss gradient, Adam), the training
// labels (a-posteriori troubled elements) and the inference that replaces the
// modal blending coefficient, falling back to it where the network is not
// trusted.  Parameter vector layout (P values):
//   W1[H][nin], b1[H], W2[H][H], b2[H], W3[H], b3.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <string>

#include "../../include/crk.h"
#include "crk_kernels.hpp"

using namespace crk;

namespace crk {
const char *set_error(crk_status st, const char *msg);
}

namespace {

constexpr int NIN = 16;   // (N+1)^2 features of a degree-3 quadrilateral
constexpr int HID = 64;
constexpr long NPAR = (long)HID * NIN + HID + (long)HID * HID + HID + HID + 1;

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f2bf(float f)
{
    // round to nearest even
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

struct MlpView {
    const uint16_t *W1, *b1, *W2, *b2, *W3, *b3;
};
__device__ __forceinline__ MlpView mlp_view(const uint16_t *th)
{
    MlpView v;
    v.W1 = th;
    v.b1 = v.W1 + HID * NIN;
    v.W2 = v.b1 + HID;
    v.b2 = v.W2 + HID * HID;
    v.W3 = v.b2 + HID;
    v.b3 = v.W3 + HID;
    return v;
}

// ---------------------------------------------------------------- the network on the matrix cores
// Every layer is formed transposed, Y^T = W X^T, for 16 samples at a time.
// In the indicator's tile (mlp_tile) the BF16 weights are the exact A operand,
// and every FP32 activation enters the B operand as the sum of three BF16
// parts (x = hi + mid + lo to within 2^-26 |x|), so each product is exact in
// FP32 and the result is the FP32 network up to the summation order.  The first layer (16 inputs) uses
// v_mfma_f32_16x16x16_bf16, operand layout (lane l, i = 0..3):
// A[l % 16][4 (l / 16) + i], B[4 (l / 16) + i][l % 16],
// D[4 (l / 16) + i][l % 16]; a layer's D is therefore already a B operand of
// the next layer.  The 64-wide layers use the K = 32 form
// v_mfma_f32_16x16x32_bf16 on two 16-row D blocks at a time: a lane's eight
// B values are its four rows of each block, and its eight A values are the
// weights of the same hidden units (whatever hidden unit an operand slot
// carries, A and B carry the same one, so the sum runs over the block pair).
typedef short mx_s4 __attribute__((ext_vector_type(4)));
typedef float mx_f4 __attribute__((ext_vector_type(4)));
typedef __bf16 mx_b8 __attribute__((ext_vector_type(8)));
typedef short mx_s8 __attribute__((ext_vector_type(8)));

// x = hi + mid + lo in BF16 (round to nearest even: the hardware conversion).
// An infinite x is its own hi part with mid = lo = 0, so that it acts as it
// would in FP32 arithmetic.
__device__ __forceinline__ void split3(float x, short &h, short &m, short &l)
{
    const __bf16 bh = (__bf16)x;
    const float fh = (float)bh;
    const float r1 = x == fh ? 0.f : x - fh;
    const __bf16 bm = (__bf16)r1;
    const float r2 = r1 - (float)bm;
    h = __builtin_bit_cast(short, bh);
    m = __builtin_bit_cast(short, bm);
    l = __builtin_bit_cast(short, (__bf16)r2);
}
template <class V>
__device__ __forceinline__ void split3v(const float *x, int n, V &h, V &m, V &l)
{
#pragma unroll
    for (int i = 0; i < n; ++i) {
        short a, b, c;
        split3(x[i], a, b, c);
        h[i] = a;
        m[i] = b;
        l[i] = c;
    }
}

// two 4-value operands of the K = 16 form as one 8-value operand of the
// K = 32 form, reinterpreted as a whole vector (built element by element
// from bit-cast BF16 values, the operand reached the instruction wrongly
// packed with this compiler, although its bits read back unchanged)
__device__ __forceinline__ mx_b8 join8(const mx_s4 &p, const mx_s4 &q)
{
    const mx_s8 t = __builtin_shufflevector(p, q, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(mx_b8, t);
}

// acc + a (bh + bm + bl), the small parts first
__device__ __forceinline__ mx_f4 mfma3(const mx_s4 &a, const mx_s4 &bh, const mx_s4 &bm, const mx_s4 &bl, mx_f4 acc)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, bl, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, bm, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, bh, acc, 0, 0, 0);
}
__device__ __forceinline__ mx_f4 mfma3k32(const mx_b8 &a, const mx_b8 &bh, const mx_b8 &bm, const mx_b8 &bl, mx_f4 acc)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bl, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bm, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bh, acc, 0, 0, 0);
}
constexpr int MX_TILE = 16;
constexpr unsigned MLP_GRID = 2 * 256;   // workgroups of the inference kernels: two wavefronts per SIMD of 256 CUs
static_assert(NIN == 16 && HID == 64, "the tiling below is written for 16 inputs and 64 hidden units");

// The weights a lane holds (col = lane % 16, kq = lane / 16): the A blocks of
// W1 (hidden 16 b + col, inputs 4 kq + i) and W2 (out 16 c + col, hidden units
// of the block pair), and the biases and W3 of the hidden units 16 b + 4 kq + i
// it holds in D.  They stay in registers while a wavefront walks its tiles.
struct MlpRegs {
    mx_s4 A1[4];
    mx_b8 A2[4][2];
    float B1[4][4], B2[4][4], W3[4][4], b3;
};
__device__ __forceinline__ void mlp_load(const MlpView &w, int col, int kq, MlpRegs &r)
{
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        mx_s4 q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r.A1[b][i] = (short)w.W1[(16 * b + col) * NIN + 4 * kq + i];
            r.B1[b][i] = bf2f(w.b1[16 * b + 4 * kq + i]);
            r.B2[b][i] = bf2f(w.b2[16 * b + 4 * kq + i]);
            r.W3[b][i] = bf2f(w.W3[16 * b + 4 * kq + i]);
#pragma unroll
            for (int c = 0; c < 4; ++c) q[c][i] = (short)w.W2[(16 * b + col) * HID + 16 * c + 4 * kq + i];
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) r.A2[b][kb] = join8(q[2 * kb], q[2 * kb + 1]);
    }
    r.b3 = bf2f(w.b3[0]);
}

// The network on the 16 samples of a tile: x = the lane's four inputs
// 4 kq + i of sample col.  Returns z (in all four lanes of the sample).
__device__ __forceinline__ float mlp_tile(const MlpRegs &w, const float *x)
{
    mx_s4 xh, xm, xl;
    split3v(x, 4, xh, xm, xl);
    mx_s4 hh[4], hm[4], hl[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        mx_f4 acc = {0.f, 0.f, 0.f, 0.f};
        acc = mfma3(w.A1[b], xh, xm, xl, acc);
        float h1[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = acc[i] + w.B1[b][i];
            h1[i] = v > 0.f ? v : 0.f;
        }
        split3v(h1, 4, hh[b], hm[b], hl[b]);
    }
    mx_b8 kh[2], km[2], kl[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        kh[kb] = join8(hh[2 * kb], hh[2 * kb + 1]);
        km[kb] = join8(hm[2 * kb], hm[2 * kb + 1]);
        kl[kb] = join8(hl[2 * kb], hl[2 * kb + 1]);
    }
    float z = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        mx_f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) acc = mfma3k32(w.A2[c][kb], kh[kb], km[kb], kl[kb], acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = acc[i] + w.B2[c][i];
            z = fmaf(w.W3[c][i], v > 0.f ? v : 0.f, z);
        }
    }
    z += __shfl_xor(z, 16);
    z += __shfl_xor(z, 32);
    return z + w.b3;
}

// The network on 16 samples bit for bit as FP32 arithmetic with its sums taken
// in index order: v_mfma_f32_16x16x4_f32 adds its four products to the
// accumulator one after the other, each rounded as an FP32 fused
// multiply-add, so a chain of them is the chain of scalar ones.  Operand
// layout (lane l, col = l % 16, kq = l / 16): A[col][kq], B[kq][col],
// D[4 kq + i][col].  Row r of a D block is made hidden unit
// 16 b + 4 (r % 4) + r / 4 (by the A row it is given), so that register i of D
// is unit 16 b + 4 i + kq: the B operand of four units in index order.
struct MlpF32 {
    float A1[4][4], A2[4][16], B1[4][4], B2[4][4];
};
__device__ __forceinline__ void mlp_load_f32(const MlpView &w, int col, int kq, MlpF32 &r)
{
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int row = 16 * b + 4 * (col & 3) + (col >> 2);   // hidden unit of the lane's A row
#pragma unroll
        for (int t = 0; t < 4; ++t) r.A1[b][t] = bf2f(w.W1[row * NIN + 4 * t + kq]);
#pragma unroll
        for (int t = 0; t < 16; ++t) r.A2[b][t] = bf2f(w.W2[row * HID + 4 * t + kq]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r.B1[b][i] = bf2f(w.b1[16 * b + 4 * i + kq]);
            r.B2[b][i] = bf2f(w.b2[16 * b + 4 * i + kq]);
        }
    }
}
// xs[t]: input 4 t + kq of the lane's sample; a1, a2: the sums of both hidden
// layers before the ReLU, register [b][i] of unit 16 b + 4 i + kq
__device__ __forceinline__ void mlp_tile_f32(const MlpF32 &w, const float *xs, mx_f4 *a1, mx_f4 *a2)
{
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        a1[b] = mx_f4{w.B1[b][0], w.B1[b][1], w.B1[b][2], w.B1[b][3]};
        a2[b] = mx_f4{w.B2[b][0], w.B2[b][1], w.B2[b][2], w.B2[b][3]};
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int b = 0; b < 4; ++b) a1[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.A1[b][t], xs[t], a1[b], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const float h = a1[t >> 2][t & 3] > 0.f ? a1[t >> 2][t & 3] : 0.f;   // unit 4 t + kq
#pragma unroll
        for (int b = 0; b < 4; ++b) a2[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.A2[b][t], h, a2[b], 0, 0, 0);
    }
}

// Inference of many samples: a wavefront takes 64 samples in four groups of
// 16.  The output layer, one sum per sample, is formed by one lane per sample
// from the second layer's outputs in LDS (rows of 80: the four rows a store
// touches lie on different banks).
// Bound by the matrix cores' FP32 rate: 80 instructions of 32 cycles per 16
// samples are 85 us for 1 310 720 samples on 1024 SIMDs at 2.4 GHz.  Measured
// there: 144 us (161 without loading the next group ahead and with the
// parameters read two bytes at a time by each lane; 151 with those reads
// alone: each block copies them to LDS first), against 405 us for one lane
// per sample on the vector units with scalar weight loads.  The
// three-part BF16 split of the indicator's tile takes 84 us but rounds
// differently, and these outputs are FP32 sums that callers compare.
constexpr int FW = 64, FROW = FW + 16;
__global__ void __launch_bounds__(256) k_mlp_forward(const uint16_t *theta, const float *x, long n, float alpha_max,
                                                     float *z_out, double *alpha_out)
{
    __shared__ float pool[4][HID * FROW];
    const int lane = threadIdx.x & 63;
    const int col = lane & 15, kq = lane >> 4;
    const long wave = ((long)blockIdx.x * 256 + threadIdx.x) >> 6;
    const long nwaves = ((long)gridDim.x * 256) >> 6;
    const long ntiles = (n + FW - 1) / FW;
    static_assert(sizeof(uint16_t) * NPAR <= sizeof(pool), "the parameters fit the rows");
    uint16_t *th = (uint16_t *)pool[0];               // (before the rows take its place)
    for (int i = threadIdx.x; i < NPAR; i += 256) th[i] = theta[i];
    __syncthreads();
    const MlpView w = mlp_view(th);
    float *h2 = pool[threadIdx.x >> 6];
    MlpF32 r;
    mlp_load_f32(w, col, kq, r);
    const float b3 = bf2f(w.b3[0]);
    const MlpView wg = mlp_view(theta);               // (W3: uniform, scalar loads)
    __syncthreads();
    if (wave >= ntiles) return;                       // uniform per wavefront
    // the lane's inputs of the group of 16 samples that starts at s0 (the
    // next group's are loaded ahead: a group's products hide one round trip)
    float nx[4];
    auto load = [&](long s0) {
        const bool sv = s0 + col < n;
#pragma unroll
        for (int t = 0; t < 4; ++t) nx[t] = sv ? x[(s0 + col) * NIN + 4 * t + kq] : 0.f;
    };
    load(wave * FW);
    for (long tile = wave; tile < ntiles; tile += nwaves) {
        for (int g = 0; g < 4; ++g) {
            float xs[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) xs[t] = nx[t];
            load(g < 3 ? tile * FW + 16 * (g + 1) : (tile + nwaves) * FW);
            mx_f4 a1[4], a2[4];
            mlp_tile_f32(r, xs, a1, a2);
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    h2[(16 * b + 4 * i + kq) * FROW + 16 * g + col] = a2[b][i] > 0.f ? a2[b][i] : 0.f;
        }
        element_sync<64>();
        const long s = tile * FW + lane;
        float z = b3;
#pragma unroll
        for (int k = 0; k < HID; ++k) z = fmaf(bf2f(wg.W3[k]), h2[k * FROW + lane], z);
        if (s < n) {
            if (z_out) z_out[s] = z;
            if (alpha_out) alpha_out[s] = (double)alpha_max / (1.0 + exp(-(double)z));
        }
        element_sync<64>();      // before the next tile overwrites the rows
    }
}

// Gradient of the mean binary cross-entropy of sigmoid(z) against y over n
// samples, in FP32 throughout (v_mfma_f32_16x16x4_f32: fused multiply-adds of
// FP32 operands, so infinities act as in scalar arithmetic).  A workgroup takes
// 64 samples at a time, 16 per wavefront: the forward tile and the
// back-propagated sums D1^T = W2^T D2^T in index order.  The weight gradients
// gW2 = D2 H1^T and gW1 = D1 X^T are products with the 64 samples as the
// contraction, wavefront w taking the rows 16 w ..: there a lane needs several
// samples of one hidden unit where the layers leave four units of one sample,
// so D2, H1, D1, X (and E = dz relu(a2), whose row sums are gW3) pass through
// LDS (rows of GROW values: 16-byte aligned for four-sample loads, successive
// rows four banks apart).  The gradient stays in registers over all of a
// workgroup's samples, which leaves one partial gradient.
// Bound by latency at the usual batch (8192 samples are one pass of 128
// workgroups), so the parameters come through LDS too: read by the lanes of
// each operand straight from memory, two bytes at a time, they took most of
// a 25 us kernel.  Loss and gradient of 200, 8192, 60 000, 300 000 samples:
// 16.3, 18.5, 38, 121 us.  The same products with both operands split in three
// BF16 parts, six products each, took 16.9, 19.5, 41.5, 139: the splitting costs
// more vector instructions than the FP32 matrix rate.  (Vector arithmetic fed
// from LDS, 32 samples per workgroup, and a reduction that walked its partials
// one after the other on 21 workgroups: 23, 85, 529, 2657.)  Relative error
// of the gradient against 64 bits at 8192 samples 5e-8 (2.3e-7 with the serial
// reduction).
constexpr int GWAVES = 4;
constexpr int GS = MX_TILE * GWAVES;   // samples per workgroup and pass
constexpr int GROW = GS + 4;           // LDS row
constexpr int GROWS = 4 * HID + NIN;   // D2, D1, E, H1, X
constexpr int GBLOCKS = 256;           // most workgroups (one per CU)

// four samples (s0 ..) of LDS row r
__device__ __forceinline__ mx_f4 grad_operand(const float *rows, int r, int s0)
{
    return *(const mx_f4 *)(rows + r * GROW + s0);
}

__global__ void __launch_bounds__(64 * GWAVES) k_mlp_grad(const uint16_t *theta, const float *x, const float *y, long n,
                                                          float *partial, float *partial_loss)
{
    __shared__ __align__(16) float pool[GROWS * GROW];
    __shared__ float tail[2][GWAVES];
    static_assert(sizeof(uint16_t) * NPAR <= sizeof(float) * GROWS * GROW, "the parameters fit the rows");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int col = lane & 15, kq = lane >> 4;
    uint16_t *th = (uint16_t *)pool;
    for (int i = tid; i < NPAR; i += 64 * GWAVES) th[i] = theta[i];
    __syncthreads();
    const MlpView w = mlp_view(th);
    MlpF32 r;
    mlp_load_f32(w, col, kq, r);
    float W3[4][4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) W3[b][i] = bf2f(w.W3[16 * b + 4 * i + kq]);
    const float b3 = bf2f(w.b3[0]);
    // W2 transposed, in the same unit order: out 16 b + 4 (col % 4) + col / 4,
    // summed over the units 4 t + kq
    float A2T[4][16];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int t = 0; t < 16; ++t) A2T[b][t] = bf2f(w.W2[(4 * t + kq) * HID + 16 * b + 4 * (col & 3) + (col >> 2)]);
    __syncthreads();                     // the rows take the parameters' place
    float *D2 = pool, *D1 = D2 + HID * GROW, *EE = D1 + HID * GROW, *H1 = EE + HID * GROW, *X = H1 + HID * GROW;
    mx_f4 gW2[4], gW1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < 4; ++b) gW2[b] = mx_f4{0.f, 0.f, 0.f, 0.f};
    float rsum = 0.f, gb3 = 0.f, loss = 0.f;   // rsum: row lane of D2 (wavefront 0), D1 (1), E (2)
    const float inv_n = 1.f / (float)n;
    const int sl = MX_TILE * wv + col;         // sample within the pass
    for (long s0 = (long)blockIdx.x * GS; s0 < n; s0 += (long)gridDim.x * GS) {
        const long s = s0 + sl;
        const bool in = s < n;
        float xs[4];
        mx_f4 a1[4], a2[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) xs[i] = in ? x[s * NIN + 4 * i + kq] : 0.f;
        const float yy = in ? y[s] : 0.f;
        mlp_tile_f32(r, xs, a1, a2);
        float z = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) z = fmaf(W3[c][i], a2[c][i] > 0.f ? a2[c][i] : 0.f, z);
        z += __shfl_xor(z, 16);
        z += __shfl_xor(z, 32);
        z += b3;
        const float sg = 1.f / (1.f + expf(-z));
        const float dz = in ? (sg - yy) * inv_n : 0.f;
        if (kq == 0 && in) {
            // BCE with logits, stable form: log(1 + e^z) - y z
            loss += (z > 0.f ? z + log1pf(expf(-z)) : log1pf(expf(z))) - yy * z;
            gb3 += dz;
        }
        float d2[4][4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 16 * c + 4 * i + kq;
                d2[c][i] = a2[c][i] > 0.f ? dz * W3[c][i] : 0.f;
                D2[row * GROW + sl] = d2[c][i];
                EE[row * GROW + sl] = dz * (a2[c][i] > 0.f ? a2[c][i] : 0.f);
                H1[row * GROW + sl] = a1[c][i] > 0.f ? a1[c][i] : 0.f;
            }
        mx_f4 d1[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) d1[b] = mx_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 16; ++t)
#pragma unroll
            for (int b = 0; b < 4; ++b) d1[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(A2T[b][t], d2[t >> 2][t & 3], d1[b], 0, 0, 0);
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) D1[(16 * b + 4 * i + kq) * GROW + sl] = a1[b][i] > 0.f ? d1[b][i] : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) X[(4 * i + kq) * GROW + sl] = xs[i];
        __syncthreads();
        // this wavefront's 16 rows of both weight gradients, and a row sum per lane
        // (an operand slot of lane group kq carries sample ks + 4 kq + j in A and B alike)
#pragma unroll
        for (int ks = 0; ks < GS; ks += 16) {
            const mx_f4 a = grad_operand(D2, 16 * wv + col, ks + 4 * kq), e = grad_operand(D1, 16 * wv + col, ks + 4 * kq);
            const mx_f4 xo = grad_operand(X, col, ks + 4 * kq);
            mx_f4 h[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) h[b] = grad_operand(H1, 16 * b + col, ks + 4 * kq);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int b = 0; b < 4; ++b) gW2[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], h[b][j], gW2[b], 0, 0, 0);
                gW1 = __builtin_amdgcn_mfma_f32_16x16x4f32(e[j], xo[j], gW1, 0, 0, 0);
            }
        }
        if (wv < 3) {
            const float *row = pool + (wv * HID + lane) * GROW;
            float p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < GS; k += 4)
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] += row[k + i];
            rsum += (p[0] + p[1]) + (p[2] + p[3]);
        }
        __syncthreads();                 // before the next pass overwrites the rows
    }
    float *g = partial + (long)blockIdx.x * NPAR;
    float *oW1 = g, *ob1 = oW1 + HID * NIN, *oW2 = ob1 + HID, *ob2 = oW2 + HID * HID, *oW3 = ob2 + HID, *ob3 = oW3 + HID;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = 16 * wv + 4 * kq + i;
        oW1[row * NIN + col] = gW1[i];
#pragma unroll
        for (int b = 0; b < 4; ++b) oW2[row * HID + 16 * b + col] = gW2[b][i];
    }
    if (wv == 0) ob2[lane] = rsum;
    else if (wv == 1) ob1[lane] = rsum;
    else if (wv == 2) oW3[lane] = rsum;
    // loss and output bias: over the wavefront's 16 samples, then the wavefronts
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) {
        loss += __shfl_xor(loss, m);
        gb3 += __shfl_xor(gb3, m);
    }
    if (lane == 0) {
        tail[0][wv] = loss;
        tail[1][wv] = gb3;
    }
    __syncthreads();
    if (tid == 0) {
        float sl0 = 0.f, sb = 0.f;
#pragma unroll
        for (int k = 0; k < GWAVES; ++k) {
            sl0 += tail[0][k];
            sb += tail[1][k];
        }
        partial_loss[blockIdx.x] = sl0;
        ob3[0] = sb;
    }
}

// Sum of the workgroups' partial gradients in a fixed order.  A workgroup
// takes RCOL consecutive parameters, 256 / RCOL lanes each: every lane adds
// every (256 / RCOL)-th partial (loads in flight together), then a tree.
constexpr int RCOL = 16, RSEG = 256 / RCOL;
__global__ void __launch_bounds__(256) k_mlp_reduce(const float *partial, const float *partial_loss, int nblocks,
                                                    long n_total, float *grad, float *loss)
{
    __shared__ float red[RSEG][RCOL];
    const int c = threadIdx.x % RCOL, g = threadIdx.x / RCOL;
    const long p = (long)blockIdx.x * RCOL + c;
    const float *src = p < NPAR ? partial + p : partial_loss;
    const long stride = p < NPAR ? NPAR : 1;
    float a = 0.f;
    if (p <= NPAR) {
#pragma unroll 4
        for (int b = g; b < nblocks; b += RSEG) a += src[(long)b * stride];
    }
    red[g][c] = a;
    __syncthreads();
    for (int m = RSEG / 2; m > 0; m >>= 1) {
        if (g < m) red[g][c] += red[g + m][c];
        __syncthreads();
    }
    if (g > 0) return;
    if (p < NPAR) grad[p] = red[0][c];
    else if (p == NPAR && loss) *loss = red[0][c] / (float)n_total;
}

__global__ void __launch_bounds__(256) k_adam(long count, float *theta, float *m, float *v, const float *g, float lr,
                                              float b1, float b2, float eps, float c1, float c2, uint16_t *theta_bf16)
{
    const long k = (long)blockIdx.x * 256 + threadIdx.x;
    if (k >= count) return;
    const float gk = g[k];
    const float mk = b1 * m[k] + (1.f - b1) * gk;
    const float vk = b2 * v[k] + (1.f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    const float th = theta[k] - lr * (mk / c1) / (sqrtf(vk / c2) + eps);
    theta[k] = th;
    if (theta_bf16) theta_bf16[k] = f2bf(th);
}

__global__ void __launch_bounds__(256) k_to_bf16(long count, const float *x, uint16_t *y)
{
    const long k = (long)blockIdx.x * 256 + threadIdx.x;
    if (k < count) y[k] = f2bf(x[k]);
}

// Blending coefficient from the network where it is trusted: features inside
// the training range [lo, hi] and a finite output; elsewhere the modal
// coefficient already in alpha_raw stays.  alpha < alpha_min is cut to 0 as
// for the modal indicator.
__global__ void __launch_bounds__(256) k_mlp_alpha(const uint16_t *theta, const float *features, const float *lo,
                                                   const float *hi, long nelem, double alpha_max, double alpha_min,
                                                   double *alpha_raw, const crk::Tables t, int epb, int *tiles)
{
    const int lane = threadIdx.x & 63;
    const int col = lane & 15, kq = lane >> 4;
    const long wave = ((long)blockIdx.x * 256 + threadIdx.x) >> 6;
    const long nwaves = ((long)gridDim.x * 256) >> 6;
    const long ntiles = (nelem + MX_TILE - 1) / MX_TILE;
    if (wave >= ntiles) return;                       // uniform per wavefront
    MlpRegs w;
    mlp_load(mlp_view(theta), col, kq, w);
    float flo[4], fhi[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { flo[i] = lo[4 * kq + i]; fhi[i] = hi[4 * kq + i]; }

    for (long tile = wave; tile < ntiles; tile += nwaves) {
        const long e = tile * MX_TILE + col;
        const bool ev = e < nelem;
        float x[4];
        bool inside = true;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[i] = ev ? features[e * NIN + 4 * kq + i] : 0.f;
            inside &= (x[i] >= flo[i]) && (x[i] <= fhi[i]);
        }
        // all four lanes of an element (col, col + 16, col + 32, col + 48);
        // every lane takes part in both exchanges, whatever its own four say
        int in = inside ? 1 : 0;
        in &= __shfl_xor(in, 16);
        in &= __shfl_xor(in, 32);
        const float z = mlp_tile(w, x);
        if (kq == 0 && ev && in && isfinite(z)) {
            double a = alpha_max / (1.0 + exp(-(double)z));
            if (a < alpha_min) a = 0.0;
            alpha_raw[e] = a;
            // local-phase tile flags of the pipelined step (2D meshes)
            if (tiles != nullptr && a > 0.0) crk::mark_tiles<2>(t, e, epb, tiles);
        }
    }
}

// Troubled-element labels: the unlimited update uh leaves the range of rho or
// p over the element and its face neighbours in un by more than tol
// (relative), or is inadmissible.  One lane per node.
template <typename real, int N>
__global__ void __launch_bounds__(BLOCK) k_labels(const Tables t, const void *un_, const void *uh_, double tol, float *labels)
{
    constexpr int NP = (N + 1) * (N + 1);
    constexpr int EPB = BLOCK / NP;
    __shared__ double red[4][BLOCK];
    __shared__ int bad[BLOCK];
    const int tid = threadIdx.x;
    int le = tid / NP;
    const int node = tid - le * NP;
    const long e = (long)blockIdx.x * EPB + le;
    const bool valid = (le < EPB) && (e < t.nelem);
    if (le >= EPB) le = 0;
    const long es = valid ? e : 0;
    const long E = t.nelem;
    const real *un = (const real *)un_, *uh = (const real *)uh_;
    auto pres = [&](const real *u, long el) {
        const double r = u[((long)0 * E + el) * NP + node], m1 = u[((long)1 * E + el) * NP + node];
        const double m2 = u[((long)2 * E + el) * NP + node], En = u[((long)3 * E + el) * NP + node];
        return (t.gamma - 1.0) * (En - 0.5 * (m1 * m1 + m2 * m2) / r);
    };
    const Nbrs nb = neighbours<2>(t, es);
    long list[5] = {es, nb.n[0][0], nb.n[0][1], nb.n[1][0], nb.n[1][1]};
    double rmin = INFINITY, rmax = -INFINITY, pmin = INFINITY, pmax = -INFINITY;
    for (int k = 0; k < 5; ++k) {
        const double r = un[((long)0 * E + list[k]) * NP + node], p = pres(un, list[k]);
        rmin = fmin(rmin, r);
        rmax = fmax(rmax, r);
        pmin = fmin(pmin, p);
        pmax = fmax(pmax, p);
    }
    red[0][tid] = rmin; red[1][tid] = rmax; red[2][tid] = pmin; red[3][tid] = pmax;
    __syncthreads();
    const int b0 = le * NP;
    for (int q = 0; q < NP; ++q) {
        rmin = fmin(rmin, red[0][b0 + q]);
        rmax = fmax(rmax, red[1][b0 + q]);
        pmin = fmin(pmin, red[2][b0 + q]);
        pmax = fmax(pmax, red[3][b0 + q]);
    }
    int flag = 0;
    for (int v = 0; v < 4; ++v)
        if (!isfinite((double)uh[((long)v * E + es) * NP + node])) flag = 1;
    const double r = uh[((long)0 * E + es) * NP + node], p = pres(uh, es);
    if (!(r > 0.0) || !(p > 0.0)) flag = 1;
    if (r < rmin * (1.0 - tol) || r > rmax * (1.0 + tol)) flag = 1;
    if (p < pmin * (1.0 - tol) || p > pmax * (1.0 + tol)) flag = 1;
    bad[tid] = flag;
    __syncthreads();
    if (!valid || node != 0) return;
    int any = 0;
    for (int q = 0; q < NP; ++q) any |= bad[b0 + q];
    labels[e] = any ? 1.f : 0.f;
}

crk_status hip_err(hipError_t e, const char *where)
{
    std::string m = std::string(where) + ": " + hipGetErrorString(e);
    set_error(CRK_ERR_HIP, m.c_str());
    return CRK_ERR_HIP;
}

crk_status check_shape(int nin, int hidden)
{
    if (nin != NIN || hidden != HID) {
        set_error(CRK_ERR_UNSUPPORTED, "the network is compiled for 16 inputs and 64 hidden units");
        return CRK_ERR_UNSUPPORTED;
    }
    return CRK_OK;
}

inline unsigned blocks(long n, int b) { return (unsigned)((n + b - 1) / b); }

} // namespace

namespace crk {
// used by crk_api.cpp: learned blending coefficients over the modal ones
hipError_t launch_mlp_alpha(const uint16_t *theta, const float *features, const float *lo, const float *hi, long nelem,
                            double alpha_max, double alpha_min, double *alpha_raw, const Tables *t, int *flags,
                            hipStream_t s)
{
    // four wavefronts per workgroup, each walking tiles of 16 elements; at
    // most two wavefronts per SIMD of the 256 CUs (the register budget)
    const long tiles = (nelem + MX_TILE - 1) / MX_TILE;
    long g = (tiles + 3) / 4;
    if (g > (long)MLP_GRID) g = MLP_GRID;
    // flags: local-phase tile flags of the 2D mesh described by *t, or nullptr
    const bool mark = flags != nullptr && t != nullptr;
    const Tables tt = mark ? *t : Tables{};
    const int epb = mark ? tile_block_rt((int)tt.nnode) / (int)tt.nnode : 1;
    hipLaunchKernelGGL(k_mlp_alpha, dim3((unsigned)g), dim3(256), 0, s, theta, features, lo, hi, nelem, alpha_max,
                       alpha_min, alpha_raw, tt, epb, mark ? flags : nullptr);
    return hipGetLastError();
}
hipError_t launch_labels(const Tables &t, int prec, const void *un, const void *uh, double tol, float *labels, hipStream_t s)
{
    const int NP = t.nnode;
    const unsigned g = blocks(t.nelem, BLOCK / NP);
    if (t.dim != 2) return hipErrorInvalidValue;
#define CRK_LAB(R, NN) hipLaunchKernelGGL((k_labels<R, NN>), dim3(g), dim3(BLOCK), 0, s, t, un, uh, tol, labels)
    if (prec == CRK_FP64) {
        switch (t.N) { case 1: CRK_LAB(double, 1); break; case 2: CRK_LAB(double, 2); break;
                       case 3: CRK_LAB(double, 3); break; default: CRK_LAB(double, 4); }
    } else {
        switch (t.N) { case 1: CRK_LAB(float, 1); break; case 2: CRK_LAB(float, 2); break;
                       case 3: CRK_LAB(float, 3); break; default: CRK_LAB(float, 4); }
    }
#undef CRK_LAB
    return hipGetLastError();
}
} // namespace crk

extern "C" {

crk_status crk_mlp_param_count(int nin, int hidden, int64_t *count)
{
    if (!count) { set_error(CRK_ERR_ARG, "null argument"); return CRK_ERR_ARG; }
    crk_status st = check_shape(nin, hidden);
    if (st) return st;
    *count = NPAR;
    return CRK_OK;
}

crk_status crk_mlp_forward(int nin, int hidden, const uint16_t *theta_bf16, const float *x, int64_t n, double alpha_max,
                           float *z, double *alpha, crk_stream stream)
{
    crk_status st = check_shape(nin, hidden);
    if (st) return st;
    if (!theta_bf16 || !x || n < 0) { set_error(CRK_ERR_ARG, "null argument"); return CRK_ERR_ARG; }
    if (n == 0) return CRK_OK;
    // four wavefronts per workgroup, each walking tiles of 64 samples
    unsigned g = blocks(n, 4 * FW);
    if (g > MLP_GRID) g = MLP_GRID;
    hipLaunchKernelGGL(k_mlp_forward, dim3(g), dim3(256), 0, (hipStream_t)stream, theta_bf16, x, (long)n,
                       (float)alpha_max, z, alpha);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? CRK_OK : hip_err(e, "crk_mlp_forward");
}

crk_status crk_mlp_grad_workspace_bytes(int nin, int hidden, int64_t n, size_t *bytes)
{
    crk_status st = check_shape(nin, hidden);
    if (st) return st;
    if (!bytes || n < 0) { set_error(CRK_ERR_ARG, "bad argument"); return CRK_ERR_ARG; }
    // one set per 32 samples: the contract of this entry point and of the check
    // below; the kernel uses one per 64 samples, 256 (5.4 MB) at most
    const long nb = (long)blocks(n, 32);
    *bytes = ((size_t)nb * NPAR * sizeof(float) + 255) / 256 * 256 + (size_t)nb * sizeof(float);
    return CRK_OK;
}

crk_status crk_mlp_loss_grad(int nin, int hidden, const uint16_t *theta_bf16, const float *x, const float *y, int64_t n,
                             float *grad, float *loss, void *workspace, size_t ws_bytes, crk_stream stream)
{
    crk_status st = check_shape(nin, hidden);
    if (st) return st;
    if (!theta_bf16 || !x || !y || !grad || !workspace || n < 1) { set_error(CRK_ERR_ARG, "null argument"); return CRK_ERR_ARG; }
    size_t need = 0;
    crk_mlp_grad_workspace_bytes(nin, hidden, n, &need);
    if (ws_bytes < need) { set_error(CRK_ERR_ARG, "workspace too small"); return CRK_ERR_ARG; }
    unsigned nb = blocks(n, GS);
    if (nb > GBLOCKS) nb = GBLOCKS;
    float *part = (float *)workspace;
    float *pl = (float *)((char *)workspace + ((size_t)nb * NPAR * sizeof(float) + 255) / 256 * 256);
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_mlp_grad, dim3(nb), dim3(64 * GWAVES), 0, s, theta_bf16, x, y, (long)n, part, pl);
    hipLaunchKernelGGL(k_mlp_reduce, dim3(blocks(NPAR + 1, RCOL)), dim3(256), 0, s, (const float *)part,
                       (const float *)pl, (int)nb, (long)n, grad, loss);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? CRK_OK : hip_err(e, "crk_mlp_loss_grad");
}

crk_status crk_mlp_adam(int64_t count, float *theta, float *m, float *v, const float *grad, double lr, double b1,
                        double b2, double eps, int t, uint16_t *theta_bf16, crk_stream stream)
{
    if (!theta || !m || !v || !grad || count < 1 || t < 1) { set_error(CRK_ERR_ARG, "bad argument"); return CRK_ERR_ARG; }
    const float c1 = (float)(1.0 - std::pow(b1, t)), c2 = (float)(1.0 - std::pow(b2, t));
    hipLaunchKernelGGL(k_adam, dim3(blocks(count, 256)), dim3(256), 0, (hipStream_t)stream, (long)count, theta, m, v,
                       grad, (float)lr, (float)b1, (float)b2, (float)eps, c1, c2, theta_bf16);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? CRK_OK : hip_err(e, "crk_mlp_adam");
}

crk_status crk_mlp_to_bf16(int64_t count, const float *theta, uint16_t *theta_bf16, crk_stream stream)
{
    if (!theta || !theta_bf16 || count < 1) { set_error(CRK_ERR_ARG, "bad argument"); return CRK_ERR_ARG; }
    hipLaunchKernelGGL(k_to_bf16, dim3(blocks(count, 256)), dim3(256), 0, (hipStream_t)stream, (long)count, theta,
                       theta_bf16);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? CRK_OK : hip_err(e, "crk_mlp_to_bf16");
}

} // extern "C"
