// mc_train.hip -- training of the delayed-acceptance surrogate on the GPU:
// bfloat16 matrix-core (MFMA) products with float accumulation, float
// master weights and Adam, behind mc_mlp_grad and mc_train_surrogate.
//
// The network (see include/mc.h): eps(phi) = b3 + w3 . bf16(relu(Z2)),
// Z2 = bf16(relu(Z1)) W2 + b2, Z1 = phi W1 + b1, phi the 128 neighbour
// histogram counts of a position.  The training loss of a batch of logged
// moves is mean((eps(phi_new) - eps(phi_old) - dE / l_B)^2); its gradient is
// formed by backpropagation, with the derivative of the bfloat16 rounding
// taken as 1.  Not in the paper: the learned first stage of a two-stage
// Metropolis test whose second stage is the paper's exact dE.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <random>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/mc.h"
#include "mc_internal.hpp"

namespace {

constexpr int kIn = 128, kHid = 128;
constexpr int kNP = MC_DA_NPARAM;
// offsets of the flat parameter vector
constexpr int oW1 = 0, oB1 = oW1 + kIn * kHid, oW2 = oB1 + kHid, oB2 = oW2 + kHid * kHid, oW3 = oB2 + kHid,
              oB3 = oW3 + kHid;
static_assert(oB3 + 1 == kNP, "parameter layout");

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t to_bf16(float v) {
    uint32_t b = __builtin_bit_cast(uint32_t, v);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

// One training step is three launches: rows_kernel (forward, residuals and
// the backward pass down to dZ1, 32 pairs of rows a workgroup, everything
// between the layers in LDS and registers), grads_kernel (the weight
// gradients, the column sums and the loss over all rows) and adam_kernel.
// Every sum keeps one fixed order, whatever the launch: a matrix product
// accumulates its K index in ascending steps of 8 on the matrix cores, a
// column sum runs over 256 strided partial sums and a tree.  Measured, a step
// of 4096 moves: 24 + 22 + 5 us; as sixteen kernels with the activations in
// memory between them and operands read as single bfloat16 values down the
// columns, 2.6 ms.

// Rows of bfloat16 values in LDS are padded to 132 (8-byte reads of 32 rows
// then spread over the banks).
constexpr int kRowPad = kHid + 4;
typedef uint16_t row_t[kRowPad];
static_assert(sizeof(row_t) % 8 == 0, "rows of 8-byte pieces");

// acc[t] += A[32 x 128] B[128 x 32] for two neighbouring column tiles: rows
// row0.. of `a` ([row][k]) and rows col0.., col0 + 32.. of `b` ([column][k]),
// v_mfma_f32_32x32x8bf16_1k (lane l holds A[l % 32][4 (l / 32) + v],
// B[4 (l / 32) + v][l % 32], v = 0..3, and D[8 (r / 4) + 4 (l / 32) + r % 4]
// [l % 32], r = 0..15).
__device__ __forceinline__ void product_32x64(const row_t* a, int row0, const row_t* b, int col0, f32x16 (&acc)[2]) {
    const int lane = threadIdx.x & 63, i = lane & 31, kq = (lane >> 5) * 4;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
#pragma unroll
    for (int k0 = 0; k0 < kHid; k0 += 8) {
        const bf16x4 av = *reinterpret_cast<const bf16x4*>(&a[row0 + i][k0 + kq]);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const bf16x4 bv = *reinterpret_cast<const bf16x4*>(&b[col0 + 32 * t + i][k0 + kq]);
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(av, bv, acc[t], 0, 0, 0);
        }
    }
}

// What rows_kernel leaves for grads_kernel lies in blocks of 32 rows, [R / 32]
// [128 columns][32]: row 8 s + 4 h + v of a block at 16 h + 4 s + v.  That is
// the order in which a lane holds a column of a product (its 16 values go out
// as one run) and in which it wants the operands of the next one over those
// rows (4 steps of it in two 16-byte loads, a wave's loads without gaps).
__device__ __forceinline__ size_t block32(int r, int col) {
    return ((size_t)(r >> 5) * kHid + col) * 32 + (((r >> 2) & 1) * 16 + ((r >> 3) & 3) * 4 + (r & 3));
}

// What rows_kernel reads and leaves for grads_kernel.
struct StepBuffers {
    const float* Pw;                    // working parameters (bfloat16 values)
    const uint16_t *W1t, *W2t, *W2b;    // bfloat16 W1 and W2, [column][k], and W2 as it is
    uint16_t *X, *H1, *H2;              // blocks of rows, bfloat16: input and hidden layers
    uint16_t *dZ2b, *dZ1b;              // blocks of rows, bfloat16
    float *dZ2, *dZ1;                   // blocks of rows
    float *out, *dout, *res;            // [R], [R], [B]
    float* g;
};

struct RowsShared {
    alignas(16) row_t x[64];  // input rows, then H2, then dZ2
    alignas(16) row_t h[64];  // H1, then dZ1
    alignas(16) row_t w1t[kHid], w2t[kHid], w2[kHid];
    float b1[kHid], b2[kHid], w3[kHid];
    float dout[64];
};

// Forward (and, with `back`, backward) of the pairs 32 blockIdx.x ..: rows
// 0..31 of the tile are phi(x_i), rows 32..63 phi(x~_i) of the same moves
// (global rows b and B + b).  feat: packed byte histograms [.][64] words, of
// which pair b is entry idx[b] (idx NULL: b); y[b] = de[idx[b]] * inv_lB (y32
// if given).  Bound: latency of one tile (13 us alone, 24 us for 128 tiles);
// the four waves share it as 2 x 2 blocks of 32 rows by 64 columns.
__global__ void __launch_bounds__(256)
rows_kernel(StepBuffers s, const uint32_t* __restrict__ feat, const int64_t* __restrict__ idx,
            const double* __restrict__ de, double inv_lB, const float* __restrict__ y32, float b3, int B, int back)
{
    __shared__ RowsShared sh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int p0 = blockIdx.x * 32;
    // all loads in flight before the first is used
    constexpr int kPer = kHid * kIn / 8 / 256;
    uint32_t fv[32 * 64 / 256];  // word tid % 64 (counts 4 w .. 4 w + 3) of pairs wave, wave + 4, ...
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int b = p0 + wave + 4 * j;
        fv[j] = feat[(idx ? idx[b] : b) * 64 + lane];
    }
    auto weights = [&](row_t* dst, const uint16_t* src) {
        uint4 v[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) v[j] = reinterpret_cast<const uint4*>(src)[tid + 256 * j];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            uint16_t* to = &dst[(tid + 256 * j) / (kIn / 8)][8 * (tid % (kIn / 8))];
            *reinterpret_cast<uint2*>(to) = make_uint2(v[j].x, v[j].y);
            *reinterpret_cast<uint2*>(to + 4) = make_uint2(v[j].z, v[j].w);
        }
    };
    weights(sh.w1t, s.W1t);
    weights(sh.w2t, s.W2t);
    if (back) weights(sh.w2, s.W2b);
    if (tid < kHid) {
        sh.b1[tid] = s.Pw[oB1 + tid];
        sh.b2[tid] = s.Pw[oB2 + tid];
        sh.w3[tid] = s.Pw[oW3 + tid];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        uint32_t pk[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) pk[q] = to_bf16((float)((fv[j] >> (8 * q)) & 0xFFu));
        *reinterpret_cast<uint2*>(&sh.x[(lane >> 5) * 32 + wave + 4 * j][4 * (lane & 31)]) =
            make_uint2(pk[0] | (pk[1] << 16), pk[2] | (pk[3] << 16));
    }
    __syncthreads();
    const int row0 = 32 * (wave & 1), col0 = 64 * (wave >> 1);
    auto row_of = [&](int r) { return row0 + 8 * (r / 4) + 4 * (lane >> 5) + (r % 4); };
    auto grow_of = [&](int lr) { return (lr < 32 ? p0 : B + p0 - 32) + lr; };
    // this lane's 16 rows of column col to the blocks of rows
    const size_t run0 = block32(grow_of(row0 + 4 * (lane >> 5)), 0);
    auto store_bf16 = [&](uint16_t* dst, int col, const uint32_t (&v)[8]) {
        uint4* to = reinterpret_cast<uint4*>(dst + run0 + 32 * col);
        to[0] = make_uint4(v[0], v[1], v[2], v[3]);
        to[1] = make_uint4(v[4], v[5], v[6], v[7]);
    };
    auto store_f32 = [&](float* dst, int col, const float (&v)[16]) {
        float4* to = reinterpret_cast<float4*>(dst + run0 + 32 * col);
#pragma unroll
        for (int q = 0; q < 4; ++q) to[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    };
    // relu(acc[t] + bias) to the LDS tile and, with `back`, to dst; its mask
    auto relu_rows = [&](const f32x16& a, int col, float bias, row_t* tile, uint16_t* dst) {
        uint32_t on = 0, pk[8];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float z = a[r] + bias;
            on |= (uint32_t)(z > 0.f) << r;
            const uint16_t hb = to_bf16(z > 0.f ? z : 0.f);
            tile[row_of(r)][col] = hb;
            pk[r / 2] = r & 1 ? pk[r / 2] | ((uint32_t)hb << 16) : hb;
        }
        if (back) store_bf16(dst, col, pk);
        return on;
    };
    // gradient rows v to dst, as bfloat16 to dstb and, if given, the LDS tile
    auto grad_rows = [&](const float (&v)[16], int col, float* dst, uint16_t* dstb, row_t* tile) {
        uint32_t pk[8];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint16_t db = to_bf16(v[r]);
            if (tile) tile[row_of(r)][col] = db;
            pk[r / 2] = r & 1 ? pk[r / 2] | ((uint32_t)db << 16) : db;
        }
        store_f32(dst, col, v);
        store_bf16(dstb, col, pk);
    };
    if (back) {
        // the input: column tid / 2, the rows of half tid & 1, of both runs
        const int col = tid >> 1, half = tid & 1;
#pragma unroll
        for (int run = 0; run < 2; ++run) {
            uint32_t pk[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const row_t* from = sh.x + 32 * run + 8 * (q / 2) + 4 * half + 2 * (q & 1);
                pk[q] = (uint32_t)from[0][col] | ((uint32_t)from[1][col] << 16);
            }
            uint4* to = reinterpret_cast<uint4*>(s.X + block32(grow_of(32 * run + 4 * half), col));
            to[0] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
            to[1] = make_uint4(pk[4], pk[5], pk[6], pk[7]);
        }
    }
    f32x16 acc[2];
    uint32_t on1[2], on2[2];  // Z > 0, bit r
    product_32x64(sh.x, row0, sh.w1t, col0, acc);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int col = col0 + 32 * t + (lane & 31);
        on1[t] = relu_rows(acc[t], col, sh.b1[col], sh.h, s.H1);
    }
    __syncthreads();  // (the input rows are no longer needed from here on)
    product_32x64(sh.h, row0, sh.w2t, col0, acc);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int col = col0 + 32 * t + (lane & 31);
        on2[t] = relu_rows(acc[t], col, sh.b2[col], sh.x, s.H2);
    }
    __syncthreads();
    if (wave == 0) {
        // out[r] = b3 + sum_k H2[r][k] w3[k], k ascending; a lane a row
        float o = b3;
#pragma unroll 32
        for (int k = 0; k < kHid; ++k) o = __builtin_fmaf(from_bf16(sh.x[lane][k]), sh.w3[k], o);
        s.out[grow_of(lane)] = o;
        if (back) {
            const float o_new = __shfl(o, 32 + (lane & 31), 64), o_old = __shfl(o, lane & 31, 64);
            const int b = p0 + (lane & 31);
            const float y = y32 ? y32[b] : (float)(de[idx ? idx[b] : b] * inv_lB);
            const float r = o_new - o_old - y;
            const float g = 2.f * r / (float)B;
            const float d = lane < 32 ? -g : g;
            if (lane < 32) s.res[b] = r;
            s.dout[grow_of(lane)] = d;
            sh.dout[lane] = d;
        }
    }
    if (!back) return;
    __syncthreads();
    // dZ2[r][h] = dout[r] w3[h] [Z2 > 0]
    float d[16];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int col = col0 + 32 * t + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) d[r] = ((on2[t] >> r) & 1u) ? sh.dout[row_of(r)] * sh.w3[col] : 0.f;
        grad_rows(d, col, s.dZ2, s.dZ2b, sh.x);
    }
    __syncthreads();
    product_32x64(sh.x, row0, sh.w2, col0, acc);  // dH1 = dZ2 W2^T
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int col = col0 + 32 * t + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) d[r] = ((on1[t] >> r) & 1u) ? acc[t][r] : 0.f;
        grad_rows(d, col, s.dZ1, s.dZ1b, nullptr);
    }
}

// A 32 x 32 tile of C[128 x 128] = A^T B over K = R rows, A and B in blocks
// of 32 rows: one wave, accumulating steps of 8 rows in ascending order (the
// order fixes the sum, so K is not split).  Bound: the chain of dependent
// matrix instructions, 1024 of them in 22 us at R = 8192; the operands travel
// kAhead blocks (4 steps each) ahead, and a tile has a compute unit to itself:
// four tiles on one, 56 us.
constexpr int kAhead = 8;
__device__ __forceinline__ void grad_tile(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, int R, int m0,
                                          int n0, float* __restrict__ C) {
    const int lane = threadIdx.x & 63, i = lane & 31, half = lane >> 5;
    const uint4* a = reinterpret_cast<const uint4*>(A) + (m0 + i) * 4 + 2 * half;
    const uint4* b = reinterpret_cast<const uint4*>(B) + (n0 + i) * 4 + 2 * half;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const int blocks = R / 32;
    uint4 av[kAhead][2], bv[kAhead][2];
    auto load = [&](int q, int k) {  // block k, or the last one again
        const size_t at = (size_t)(k < blocks ? k : blocks - 1) * (kHid * 4);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            av[q][u] = a[at + u];
            bv[q][u] = b[at + u];
        }
    };
    auto steps = [&](int q) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            struct two {
                bf16x4 v[2];
            };
            const two x = __builtin_bit_cast(two, av[q][u]), y = __builtin_bit_cast(two, bv[q][u]);
            acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(x.v[0], y.v[0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(x.v[1], y.v[1], acc, 0, 0, 0);
        }
    };
#pragma unroll
    for (int q = 0; q < kAhead; ++q) load(q, q);
    int k = 0;
    for (; k + kAhead <= blocks; k += kAhead) {
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            steps(q);
            load(q, k + q + kAhead);
        }
    }
#pragma unroll
    for (int q = 0; q < kAhead; ++q)
        if (k + q < blocks) steps(q);
#pragma unroll
    for (int r = 0; r < 16; ++r) C[(m0 + 8 * (r / 4) + 4 * half + (r % 4)) * kHid + n0 + i] = acc[r];
}

// Sum over the 256 threads' values, a tree in thread order.
template <typename T>
__device__ __forceinline__ T block_tree(T v, T* part) {
    part[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
        __syncthreads();
    }
    return part[0];
}

// The gradient over all rows, one launch: blocks 0..31 the 32 tiles of dW2
// = H1^T dZ2 and dW1 = X^T dZ1 (one wave each), then a block per column of the w3, b2 and b1
// gradients, one for b3 and one for the loss mean(res^2) -- the column sums
// run beside the serial matrix chains.
constexpr int kGradTileBlocks = 32, kGradBlocks = kGradTileBlocks + 3 * kHid + 2;
__global__ void __launch_bounds__(256)
grads_kernel(StepBuffers s, int B, double* __restrict__ loss)
{
    __shared__ double part64[256];
    __shared__ float part[256];
    const int R = 2 * B, tid = threadIdx.x;
    int q = blockIdx.x;
    if (q < kGradTileBlocks) {
        if (tid >= 64) return;
        const int m0 = 32 * ((q >> 2) & 3), n0 = 32 * (q & 3);
        if (q < 16)
            grad_tile(s.H1, s.dZ2b, R, m0, n0, s.g + oW2);
        else
            grad_tile(s.X, s.dZ1b, R, m0, n0, s.g + oW1);
        return;
    }
    q -= kGradTileBlocks;
    if (q < 3 * kHid + 1) {
        const int k = q & (kHid - 1), what = q / kHid;
        float acc = 0.f;
        if (what == 0) {
#pragma unroll 8
            for (int r = tid; r < R; r += 256) acc += s.dout[r] * from_bf16(s.H2[block32(r, k)]);
        } else if (what == 3) {
#pragma unroll 8
            for (int r = tid; r < R; r += 256) acc += s.dout[r];
        } else {
            const float* m = what == 1 ? s.dZ2 : s.dZ1;
#pragma unroll 8
            for (int r = tid; r < R; r += 256) acc += m[block32(r, k)];
        }
        const float t = block_tree(acc, part);
        if (tid == 0) s.g[(what == 0 ? oW3 : what == 1 ? oB2 : what == 2 ? oB1 : oB3) + k] = t;
        return;
    }
    double acc = 0.0;
    for (int b = tid; b < B; b += 256) {
        const float r = s.res[b];
        acc += (double)r * (double)r;
    }
    const double t = block_tree(acc, part64);
    if (tid == 0) *loss = t / (double)B;
}

// Parameter t's working copies: the bfloat16 value in float, and in the
// matrices of the hidden layers ([column][k], and W2 also as it is).
__device__ __forceinline__ void store_working(float p, int t, float* Pw, uint16_t* W1t, uint16_t* W2t, uint16_t* W2b) {
    const uint16_t hb = to_bf16(p);
    Pw[t] = from_bf16(hb);
    if (t >= oW1 && t < oB1) {
        const int e = t - oW1;
        W1t[(e % kHid) * kIn + e / kHid] = hb;
    }
    if (t >= oW2 && t < oB2) {
        const int e = t - oW2;
        W2t[(e % kHid) * kHid + e / kHid] = hb;
        W2b[e] = hb;
    }
}

// Adam on the float master weights; refreshes the working copies.
__global__ void adam_kernel(float* __restrict__ P, float* __restrict__ m, float* __restrict__ v,
                            const float* __restrict__ g, int n, float lr, float b1, float b2, float eps, float c1,
                            float c2, float* __restrict__ Pw, uint16_t* __restrict__ W1t, uint16_t* __restrict__ W2t,
                            uint16_t* __restrict__ W2b)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const float gt = g[t];
    const float mt = b1 * m[t] + (1.f - b1) * gt;
    const float vt = b2 * v[t] + (1.f - b2) * gt * gt;
    m[t] = mt;
    v[t] = vt;
    const float p = P[t] - lr * (mt / c1) / (sqrtf(vt / c2) + eps);
    P[t] = p;
    store_working(p, t, Pw, W1t, W2t, W2b);
}

// Working copies from float master weights (bfloat16 values).
__global__ void refresh_kernel(const float* __restrict__ P, int n, float* __restrict__ Pw, uint16_t* __restrict__ W1t,
                               uint16_t* __restrict__ W2t, uint16_t* __restrict__ W2b)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) store_working(P[t], t, Pw, W1t, W2t, W2b);
}

// Device workspace of the network for batches of up to B pairs.
struct Net {
    float *P = nullptr, *Pw = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;
    uint16_t *W1t = nullptr, *W2t = nullptr, *W2b = nullptr;
    uint16_t *X = nullptr, *H1 = nullptr, *H2 = nullptr, *dZ2b = nullptr, *dZ1b = nullptr;
    float *out = nullptr, *dout = nullptr, *res = nullptr, *dZ2 = nullptr, *dZ1 = nullptr, *y = nullptr;
    double* loss = nullptr;
    uint8_t* feat = nullptr;  // staged byte histograms (gradient pass only)
    void* own = nullptr;      // the one allocation behind the pointers, if this object made it
    hipStream_t s = nullptr;

    // every buffer of a batch of B moves (the optimizer's moments only when
    // training; the staged targets and histograms only when not, beside P, so
    // that a pass's inputs go up in one copy), each obtained from
    // take(&pointer, bytes); the loss lies behind g, to come back with it
    template <typename Take>
    static bool layout(Net& n, int B, bool train, Take&& take) {
        const size_t R = 2 * (size_t)B;
        return take(&n.P, 4 * kNP) && (train || (take(&n.y, 4 * (size_t)B) && take(&n.feat, (size_t)B * 2 * kIn))) &&
               take(&n.Pw, 4 * kNP) && (!train || (take(&n.m, 4 * kNP) && take(&n.v, 4 * kNP))) &&
               take(&n.g, 4 * kNP) && take(&n.loss, 8) && take(&n.W1t, 2 * kIn * kHid) && take(&n.W2t, 2 * kHid * kHid) &&
               take(&n.W2b, 2 * kHid * kHid) && take(&n.X, 2 * R * kIn) && take(&n.H1, 2 * R * kHid) &&
               take(&n.H2, 2 * R * kHid) && take(&n.dZ2b, 2 * R * kHid) && take(&n.dZ1b, 2 * R * kHid) &&
               take(&n.out, 4 * R) && take(&n.dout, 4 * R) && take(&n.res, 4 * (size_t)B) &&
               take(&n.dZ2, 4 * R * kHid) && take(&n.dZ1, 4 * R * kHid);
    }
    // bytes of the layout, each buffer rounded up to 256
    static size_t bytes(int B, bool train) {
        Net n;
        size_t at = 0;
        layout(n, B, train, [&](auto**, size_t b) {
            at += (b + 255) & ~(size_t)255;
            return true;
        });
        return at;
    }
    // the buffers carved out of device memory [base, base + cap)
    bool carve(int B, bool train, unsigned char* base, size_t cap) {
        size_t at = 0;
        return layout(*this, B, train, [&](auto** p, size_t b) {
            const size_t a = (b + 255) & ~(size_t)255;
            if (at + a > cap) return false;
            *p = reinterpret_cast<std::remove_reference_t<decltype(*p)>>(base + at);
            at += a;
            return true;
        });
    }
    // ... of an allocation of this object's own
    bool init(int B, bool train, hipStream_t stream) {
        s = stream;
        const size_t cap = bytes(B, train);
        return hipMalloc(&own, cap) == hipSuccess && carve(B, train, (unsigned char*)own, cap);
    }
    ~Net() {
        if (!own) return;
        if (s) (void)hipStreamSynchronize(s);
        (void)hipFree(own);
    }
    // P from host memory (and, of a gradient pass, the staged inputs behind
    // it: `bytes` in all), and the working copies.  The moments are cleared on
    // the stream that uses them: a handle's stream does not wait for the null
    // stream, and a clear need not be done when its call returns
    bool upload_params(const void* p, size_t bytes = 4 * kNP) {
        if (hipMemcpy(P, p, bytes, hipMemcpyHostToDevice) != hipSuccess) return false;
        if (m && hipMemsetAsync(m, 0, 4 * kNP, s) != hipSuccess) return false;
        if (v && hipMemsetAsync(v, 0, 4 * kNP, s) != hipSuccess) return false;
        hipLaunchKernelGGL(refresh_kernel, dim3((kNP + 255) / 256), dim3(256), 0, s, P, kNP, Pw, W1t, W2t, W2b);
        return hipGetLastError() == hipSuccess;
    }
    StepBuffers buffers() const {
        return StepBuffers{Pw, W1t, W2t, W2b, X, H1, H2, dZ2b, dZ1b, dZ2, dZ1, out, dout, res, g};
    }
    // outputs of B moves (pairs idx of the histograms, or all in order)
    void outputs(int B, const uint32_t* f, const int64_t* idx, float b3, float* to) {
        StepBuffers b = buffers();
        b.out = to;
        hipLaunchKernelGGL(rows_kernel, dim3(B / 32), dim3(256), 0, s, b, f, idx, (const double*)nullptr, 0.0,
                           (const float*)nullptr, b3, B, 0);
    }
    // loss (into *l) and gradient (into g) of B moves; targets de[idx] inv_lB,
    // or y where de is NULL
    void gradient(int B, const uint32_t* f, const int64_t* idx, const double* de, double inv_lB, float b3, double* l) {
        hipLaunchKernelGGL(rows_kernel, dim3(B / 32), dim3(256), 0, s, buffers(), f, idx, de, inv_lB,
                           (const float*)(de ? nullptr : y), b3, B, 1);
        hipLaunchKernelGGL(grads_kernel, dim3(kGradBlocks), dim3(256), 0, s, buffers(), B, l);
    }
};

float round_bf16_host(double v) {
    float f = (float)v;
    uint32_t b;
    std::memcpy(&b, &f, 4);
    b += 0x7FFFu + ((b >> 16) & 1u);
    b &= 0xFFFF0000u;
    std::memcpy(&f, &b, 4);
    return f;
}

thread_local std::string g_train_error = "no error";

// Records why a handle-free call failed, for mc_last_error(NULL); returns code.
int noalloc_fail(int code, const std::string& msg) {
    g_train_error = msg;
    mc_internal_note_error(msg.c_str());
    return code;
}

// Bytes of the buffers Net::carve takes for a gradient pass of B moves (each
// piece rounded up to 256 bytes).
constexpr size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }
constexpr size_t grad_pass_bytes(int B) {
    const size_t R = 2 * (size_t)B;
    return 3 * round256(4 * (size_t)kNP) + 3 * round256(2 * kIn * kHid) + 5 * round256(2 * R * kHid) +
           2 * round256(4 * R) + 2 * round256(4 * R * kHid) + 2 * round256(4 * (size_t)B) + round256(8) +
           round256((size_t)B * 2 * kIn);
}

// Largest batch of mc_mlp_grad_noalloc and its device workspace: one
// file-scope array, about 1.75 MB, that every GPU the library runs on holds
// until the process ends.  Host code never names it directly: its device
// address comes from hipGetSymbolAddress, once per device.
constexpr int kNoAllocBatch = MC_NOALLOC_MAX_BATCH;
constexpr size_t kScratchBytes = grad_pass_bytes(kNoAllocBatch);
__device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned char* g_scratch_ptr[kMaxDevices] = {};

// The current device's address of `scratch`, looked up on the device's first
// call; nullptr (and the reason in g_train_error) on failure.
unsigned char* device_scratch() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        g_train_error = "no usable current HIP device";
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            g_train_error = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e);
            return nullptr;
        }
        g_scratch_ptr[dev] = (unsigned char*)p;
    }
    return g_scratch_ptr[dev];
}

// A copy more costs 10 to 18 us, staging the histograms beside the parameters
// a pass of the host over them: 93 us merged against 110 at 256 moves, 158
// against 166 at 1024, 257 against 210 at 4096, 2.2 ms against 1.5 at 65536.
constexpr int kMergedBatch = 1024;

// One gradient pass on host data in the buffers of `net` (params as given,
// p the same in float), on the null stream.
int gradient_pass(Net& net, int batch, const uint8_t* feats, const double* target, const double* params,
                  const std::vector<float>& p, double* loss, double* grad, std::string& err) {
    // P, y and feat as they lie on the device, in one copy; above
    // kMergedBatch moves feat by itself, from where it is
    const size_t y_at = (unsigned char*)net.y - (unsigned char*)net.P, f_at = net.feat - (unsigned char*)net.P;
    const bool merged = batch <= kMergedBatch;
    std::vector<unsigned char> up(merged ? f_at + (size_t)batch * 2 * kIn : f_at);
    std::memcpy(up.data(), p.data(), 4 * kNP);
    float* y = (float*)(up.data() + y_at);
    for (int b = 0; b < batch; ++b) y[b] = (float)target[b];
    if (merged) std::memcpy(up.data() + f_at, feats, (size_t)batch * 2 * kIn);
    if (!net.upload_params(up.data(), up.size()) ||
        (!merged && hipMemcpy(net.feat, feats, (size_t)batch * 2 * kIn, hipMemcpyHostToDevice) != hipSuccess)) {
        err = "input upload failed";
        return MC_E_DEVICE;
    }
    // (byte k of a histogram is byte k & 3 of its word k / 4)
    net.gradient(batch, reinterpret_cast<const uint32_t*>(net.feat), nullptr, nullptr, 0.0, round_bf16_host(params[oB3]),
                 net.loss);
    if (hipDeviceSynchronize() != hipSuccess || hipGetLastError() != hipSuccess) {
        err = "the gradient pass failed on the device";
        return MC_E_DEVICE;
    }
    const size_t l_at = (unsigned char*)net.loss - (unsigned char*)net.g;
    std::vector<unsigned char> down(l_at + sizeof(double));
    if (hipMemcpy(down.data(), net.g, down.size(), hipMemcpyDeviceToHost) != hipSuccess) {
        err = "output download failed";
        return MC_E_DEVICE;
    }
    const float* g = (const float*)down.data();
    double l;
    std::memcpy(&l, down.data() + l_at, sizeof(l));
    if (loss) *loss = l;
    if (grad)
        for (int k = 0; k < kNP; ++k) grad[k] = g[k];
    return MC_OK;
}

}  // namespace

extern "C" {

int mc_mlp_grad(int32_t batch, const uint8_t* feats, const double* target, const double* params, double* loss,
                double* grad) {
    if (batch < 32 || batch % 32 != 0 || !feats || !target || !params)
        return MC_E_ARG;
    std::vector<float> p(kNP);
    for (int k = 0; k < kNP; ++k) {
        if (!std::isfinite(params[k])) return MC_E_ARG;
        p[k] = (float)params[k];
    }
    Net net;
    if (!net.init(batch, false, nullptr)) return MC_E_OOM;
    std::string err;
    return gradient_pass(net, batch, feats, target, params, p, loss, grad, err);
}

int mc_mlp_grad_noalloc(int32_t batch, const uint8_t* feats, const double* target, const double* params,
                        double* loss, double* grad) {
    if (batch < 32 || batch % 32 != 0 || !feats || !target || !params)
        return noalloc_fail(MC_E_ARG, "batch must be a positive multiple of 32, and feats, target and params given");
    if (batch > kNoAllocBatch)
        return noalloc_fail(MC_E_ARG, "batch " + std::to_string(batch) + " exceeds the workspace's " +
                                          std::to_string(kNoAllocBatch) + " moves (MC_NOALLOC_MAX_BATCH)");
    std::vector<float> p(kNP);
    for (int k = 0; k < kNP; ++k) {
        if (!std::isfinite(params[k])) return noalloc_fail(MC_E_ARG, "non-finite parameter");
        p[k] = (float)params[k];
    }
    unsigned char* ws = device_scratch();
    if (!ws) return noalloc_fail(MC_E_DEVICE, g_train_error);
    Net net;
    if (!net.carve(batch, false, ws, kScratchBytes))
        return noalloc_fail(MC_E_STATE, "the buffers of the pass do not fit the workspace");
    std::string err;
    const int rc = gradient_pass(net, batch, feats, target, params, p, loss, grad, err);
    return rc == MC_OK ? MC_OK : noalloc_fail(rc, err);
}

int mc_train_surrogate(mc_handle* h, int32_t chain, int64_t n_moves, int32_t epochs, int32_t batch, double lr,
                       uint64_t seed, const double* params_in, double* params_out, double* loss_out,
                       double* val_loss, double* ref_stage2_reject) {
    if (!h) return MC_E_ARG;
    if (epochs < 1 || batch < 32 || batch % 32 != 0 || !(lr > 0) || !params_out)
        return mc_internal_fail(h, MC_E_ARG, "need epochs >= 1, batch a multiple of 32, lr > 0, params_out");
    MCLogView lg;
    int rc = mc_internal_log(h, chain, &lg);
    if (rc) return rc;
    if (n_moves < 1 || n_moves > lg.cap) return mc_internal_fail(h, MC_E_ARG, "n_moves exceeds the log");
    // usable moves: logged, no conflict, no wall or overlap rejection
    std::vector<uint8_t> flags((size_t)n_moves);
    std::vector<double> de((size_t)n_moves);
    if (hipMemcpy(flags.data(), lg.flags, (size_t)n_moves, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(de.data(), lg.de, 8 * (size_t)n_moves, hipMemcpyDeviceToHost) != hipSuccess)
        return mc_internal_fail(h, MC_E_DEVICE, "log download failed");
    std::vector<int64_t> use;
    for (int64_t k = 0; k < n_moves; ++k)
        if ((flags[k] & 0x80) && !(flags[k] & 0x07)) use.push_back(k);
    if ((int64_t)use.size() < 2 * batch) return mc_internal_fail(h, MC_E_ARG, "too few usable logged moves");
    // the last tenth of the usable moves is held out
    const int64_t n_val = std::max<int64_t>(batch, (int64_t)use.size() / 10) / batch * batch;
    const int64_t n_tr = ((int64_t)use.size() - n_val) / batch * batch;
    std::vector<int64_t> tr(use.begin(), use.begin() + n_tr), va(use.end() - n_val, use.end());
    std::mt19937_64 rng(seed);
    std::vector<float> p(kNP);
    if (params_in) {
        for (int k = 0; k < kNP; ++k) p[k] = (float)params_in[k];
    } else {
        // He initialisation of the weights, zero biases
        std::normal_distribution<double> nd(0.0, 1.0);
        for (int k = 0; k < kNP; ++k) {
            const double sd = k < oB1 ? std::sqrt(2.0 / kIn) : (k >= oW2 && k < oB2) ? std::sqrt(2.0 / kHid)
                              : (k >= oW3 && k < oB3) ? std::sqrt(1.0 / kHid) : 0.0;
            p[k] = (float)(sd * nd(rng));
        }
    }
    Net net;
    if (!net.init(batch, true, lg.stream)) return mc_internal_fail(h, MC_E_OOM, "training workspace");
    // the moves of an epoch in their order, the loss of each of its steps and
    // the outputs of the held-out moves: moved in one piece each, so that
    // the steps follow one another without the host
    const int64_t steps = n_tr / batch;
    struct Held {
        void* p = nullptr;
        hipStream_t s;
        ~Held() {
            if (p) {
                (void)hipStreamSynchronize(s);
                (void)hipFree(p);
            }
        }
    } held{nullptr, lg.stream};
    const size_t order_bytes = round256(8 * (size_t)std::max(n_tr, n_val)), loss_bytes = round256(8 * (size_t)steps);
    if (hipMalloc(&held.p, order_bytes + loss_bytes + 8 * (size_t)n_val) != hipSuccess)
        return mc_internal_fail(h, MC_E_OOM, "training workspace");
    int64_t* d_order = (int64_t*)held.p;
    double* d_loss = (double*)((char*)held.p + order_bytes);
    float* d_out = (float*)((char*)held.p + order_bytes + loss_bytes);
    if (!net.upload_params(p.data())) return mc_internal_fail(h, MC_E_DEVICE, "parameter upload");
    const double inv_lB = lg.lB > 0 ? 1.0 / lg.lB : 1.0;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    float c1 = 1.f, c2 = 1.f;
    std::vector<double> step_loss((size_t)steps);
    for (int e = 0; e < epochs; ++e) {
        std::shuffle(tr.begin(), tr.end(), rng);
        if (hipMemcpyAsync(d_order, tr.data(), 8 * (size_t)n_tr, hipMemcpyHostToDevice, net.s) != hipSuccess)
            return mc_internal_fail(h, MC_E_DEVICE, "index upload");
        for (int64_t k = 0; k < steps; ++k) {
            // b3 cancels in the difference of the two outputs: keep it at its value
            net.gradient(batch, lg.feat, d_order + k * batch, lg.de, inv_lB, 0.f, d_loss + k);
            c1 *= b1;
            c2 *= b2;
            hipLaunchKernelGGL(adam_kernel, dim3((kNP + 255) / 256), dim3(256), 0, net.s, net.P, net.m, net.v, net.g, kNP,
                               (float)lr, b1, b2, eps, 1.f - c1, 1.f - c2, net.Pw, net.W1t, net.W2t, net.W2b);
        }
        // (also before the next epoch's order replaces this one's)
        if (hipMemcpyAsync(step_loss.data(), d_loss, 8 * (size_t)steps, hipMemcpyDeviceToHost, net.s) != hipSuccess ||
            hipStreamSynchronize(net.s) != hipSuccess || hipGetLastError() != hipSuccess)
            return mc_internal_fail(h, MC_E_DEVICE, "training step failed");
        double acc = 0.0;
        for (double l : step_loss) acc += l;
        if (loss_out) loss_out[e] = acc / (double)steps;
    }
    // held-out loss and the stage-2 rejection rate the trained network gives
    // on the held-out moves: sum a1 (1 - a2) / sum a1 with a1 = min(1, e^-dEh)
    // and a2 = min(1, e^-(dE - dEh)) (stage 1 pass probability and stage 2
    // rejection probability of each move)
    double vl = 0.0, s_a1 = 0.0, s_rej = 0.0;
    std::vector<float> outv(2 * (size_t)n_val);
    if (hipMemcpyAsync(d_order, va.data(), 8 * (size_t)n_val, hipMemcpyHostToDevice, net.s) != hipSuccess)
        return mc_internal_fail(h, MC_E_DEVICE, "index upload");
    for (int64_t b0 = 0; b0 < n_val; b0 += batch) net.outputs(batch, lg.feat, d_order + b0, 0.f, d_out + 2 * b0);
    if (hipMemcpyAsync(outv.data(), d_out, 4 * outv.size(), hipMemcpyDeviceToHost, net.s) != hipSuccess ||
        hipStreamSynchronize(net.s) != hipSuccess || hipGetLastError() != hipSuccess)
        return mc_internal_fail(h, MC_E_DEVICE, "evaluation failed");
    for (int64_t b0 = 0; b0 < n_val; b0 += batch) {
        const float* o = outv.data() + 2 * b0;
        for (int b = 0; b < batch; ++b) {
            const double dEh = lg.lB * ((double)o[batch + b] - (double)o[b]);
            const double dE = de[va[b0 + b]];
            const double r = dEh - dE;
            vl += (r * inv_lB) * (r * inv_lB);
            const double a1 = dEh <= 0 ? 1.0 : std::exp(-dEh);
            const double a2 = dE - dEh <= 0 ? 1.0 : std::exp(-(dE - dEh));
            s_a1 += a1;
            s_rej += a1 * (1.0 - a2);
        }
    }
    if (val_loss) *val_loss = vl / (double)n_val;
    if (ref_stage2_reject) *ref_stage2_reject = s_a1 > 0 ? s_rej / s_a1 : 0.0;
    std::vector<float> pf(kNP);
    if (hipMemcpy(pf.data(), net.Pw, 4 * kNP, hipMemcpyDeviceToHost) != hipSuccess)
        return mc_internal_fail(h, MC_E_DEVICE, "parameter download");
    for (int k = 0; k < kNP; ++k) params_out[k] = pf[k];
    return MC_OK;
}

}  // extern "C"
