// Warm-start network of libvrm: a small MLP that predicts, from the offsets of
// an LP's columns, which columns form the optimal basis and their fractions.
//
//   x[128] (32 slots x (dx/h, dy/h), 32 slot masks, q - 2, zero padding)
//     -> 128 (GELU) -> 128 (GELU) -> 64 (32 basis logits, 32 fractions)
//
// Every matrix product runs on the BF16 matrix cores (v_mfma_f32_16x16x32_bf16,
// FP32 accumulation).  Inference is one fused kernel; a training step is two: the
// rows' (forward, loss, backward to the pre-activations) and the parameters' (weight
// gradients over all rows, AdamW).  Master weights and AdamW state are FP32; the
// products read BF16 copies.
#include <hip/hip_runtime.h>

#include "vrm_device.h"
#include "vrm_internal.h"
#include "vrm_mlp.h"

using namespace vrm;

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP32 to BF16, round to nearest even (the conversion instruction of gfx950)
__device__ __forceinline__ uint16_t to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// GELU in its tanh form: z sigma(2u) with u = sqrt(2/pi) (z + 0.044715 z^3)
// (0.5 z (1 + tanh u)); one exponential and one reciprocal
constexpr float kGeluK1 = -2.302208198144325f;    // -2 log2(e) sqrt(2/pi)
constexpr float kGeluK2 = -0.1029432395800235f;   // kGeluK1 * 0.044715
__device__ __forceinline__ float gelu_sigma(float z, float z2)
{
    // exp(-2u) = 2^(z (K1 + K2 z^2)): the factor -2 log2(e) folded into the constants
    const float a = z * __builtin_fmaf(z2, kGeluK2, kGeluK1);
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(a));   // (1 + tanh u) / 2
}
__device__ __forceinline__ float gelu(float z) { return z * gelu_sigma(z, z * z); }
__device__ __forceinline__ float gelu_grad(float z)
{
    const float z2 = z * z;
    const float s = gelu_sigma(z, z2);
    const float du = 0.7978845608028654f + 0.1070322244089003f * z2;
    return s + 2.0f * z * s * (1.0f - s) * du;
}

constexpr int TM = 64, TN = 64, TK = 32, KPAD = 8;

// One 64 x 32 operand tile into LDS as T[i][kk] (i: row of A or column of B, kk
// the k offset), from P(i, k) = P[i * si + k * sk], zeros outside i < ni,
// k < ke.  An operand contiguous in k or in i is read eight elements (16
// bytes) per thread: a run inside the bounds and 16-byte aligned by one
// vector load, else element by element.  Any other layout: one element per load.
__device__ __forceinline__ void stage_tile(uint16_t (*T)[TK + KPAD], const uint16_t* __restrict__ P, long si, long sk,
                                           int i0, int ni, int k0, int ke, int tid)
{
    if (sk == 1) {
        // thread: row tid / 4, k run 8 (tid % 4)
        const int r = tid >> 2, kk = (tid & 3) * 8;
        const int i = i0 + r, k = k0 + kk;
        const uint16_t* src = P + (long)i * si + k;
        uint4 v = {0u, 0u, 0u, 0u};
        if (i < ni && k + 7 < ke && ((uintptr_t)src & 15) == 0) {
            v = *reinterpret_cast<const uint4*>(src);
        } else if (i < ni) {
            uint16_t e[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) e[u] = k + u < ke ? src[u] : (uint16_t)0;
            v = uint4{e[0] | ((uint32_t)e[1] << 16), e[2] | ((uint32_t)e[3] << 16), e[4] | ((uint32_t)e[5] << 16),
                      e[6] | ((uint32_t)e[7] << 16)};
        }
        *reinterpret_cast<uint4*>(&T[r][kk]) = v;
    } else if (si == 1) {
        // thread: k offset tid / 8, rows 8 (tid % 8) .. + 7
        const int kk = tid >> 3, r0 = (tid & 7) * 8;
        const int i = i0 + r0, k = k0 + kk;
        const uint16_t* src = P + (long)k * sk + i;
        uint16_t e[8];
        if (k < ke && i + 7 < ni && ((uintptr_t)src & 15) == 0) {
            const uint4 v = *reinterpret_cast<const uint4*>(src);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                e[2 * u] = (uint16_t)w[u];
                e[2 * u + 1] = (uint16_t)(w[u] >> 16);
            }
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) e[u] = (k < ke && i + u < ni) ? src[u] : (uint16_t)0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) T[r0 + u][kk] = e[u];
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int idx = tid + e * 256;
            const int r = idx >> 5, kk = idx & 31;
            const int i = i0 + r, k = k0 + kk;
            T[r][kk] = (i < ni && k < ke) ? P[(long)i * si + (long)k * sk] : (uint16_t)0;
        }
    }
}

// The stand-alone product of vrm_gemm_bf16 (the network's inference and training have
// kernels of their own): C(m, n) = sum_k A(m, k) B(k, n);  A(m, k) = A[m * sam + k * sak], B(k, n) = B[k * sbk + n * sbn].
// Tile 64 x 64 per block of 4 waves (each 32 x 32 = 2 x 2 MFMA blocks); K in steps of 32.
// gridDim.z > 1 splits K; the partial sums are added atomically.
__global__ __launch_bounds__(256) void k_gemm(int M, int N, int K, const uint16_t* __restrict__ A, long sam, long sak,
                                              const uint16_t* __restrict__ B, long sbk, long sbn, float* C, long ldc,
                                              int kchunk)
{
    __shared__ __attribute__((aligned(16))) uint16_t As[TM][TK + KPAD];
    __shared__ __attribute__((aligned(16))) uint16_t Bs[TN][TK + KPAD];   // stored [n][k]
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
    const int kb = blockIdx.z * kchunk, ke = min(K, kb + kchunk);
    const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = kb; k0 < ke; k0 += TK) {
        // stage A (64 x 32) and B (32 x 64, stored [n][k]): 8 elements per thread each
        stage_tile(As, A, sam, sak, m0, M, k0, ke, tid);
        stage_tile(Bs, B, sbn, sbk, n0, N, k0, ke, tid);
        __syncthreads();
        const int row = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            bf16x8 a = *reinterpret_cast<const bf16x8*>(&As[wm + i * 16 + row][kq]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                bf16x8 b = *reinterpret_cast<const bf16x8*>(&Bs[wn + j * 16 + row][kq]);
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[i][j], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    // epilogue: lane holds rows 4 * (lane / 16) + v, column lane % 16 of each 16 x 16 block
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                int m = m0 + wm + i * 16 + (lane >> 4) * 4 + v;
                int n = n0 + wn + j * 16 + (lane & 15);
                if (m >= M || n >= N) continue;
                float s = acc[i][j][v];
                long o = (long)m * ldc + n;
                if (gridDim.z > 1)
                    atomicAdd(&C[o], s);
                else
                    C[o] = s;
            }
}

__global__ __launch_bounds__(256) void k_to_bf16(int n, const float* __restrict__ in, uint16_t* out)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = to_bf16(in[i]);
}

int nblk(long n) { return (int)((n + 255) / 256); }

// BF16 weights transposed to [n][k] (the B-operand layout of the fused kernel)
constexpr int kOffT1 = 0, kOffT2 = kMlpIn * kMlpHid, kOffT3 = kOffT2 + kMlpHid * kMlpHid;
constexpr int kWtSize = kOffT3 + kMlpHid * kMlpOut;

__global__ __launch_bounds__(256) void k_transpose_w(const uint16_t* __restrict__ wbf, uint16_t* wt)
{
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < kMlpIn * kMlpHid) {
        int k = e / kMlpHid, n = e % kMlpHid;
        wt[kOffT1 + n * kMlpIn + k] = wbf[kOffW1 + e];
        wt[kOffT2 + n * kMlpHid + k] = wbf[kOffW2 + e];
    }
    if (e < kMlpHid * kMlpOut) {
        int k = e / kMlpOut, n = e % kMlpOut;
        wt[kOffT3 + n * kMlpHid + k] = wbf[kOffW3 + e];
    }
}

// Fused inference: each block runs all three layers on tiles of 64 rows; the
// activations stay in LDS and the (L2-resident) transposed weights are read
// from memory as MFMA B operands.  Persistent: blocks loop over tiles; the row
// count may be read on the device.  The inference kernels ask for three waves per SIMD
// (at most 168 VGPRs, no spills): one more wave than the default allocation
// gives hides more of the epilogue's and the loads' latency.
constexpr int FR = 64;               // rows per tile
constexpr int FKP = kMlpHid + 8;     // padded LDS row (bank spread)

// The two hidden layers on the tile in Ta: Ta -> Tb -> Ta (GELU, BF16).
// Wave wv computes all 64 rows x columns [32 wv, 32 wv + 32).
__device__ __forceinline__ void mlp_hidden(uint16_t* Ta, uint16_t* Tb, const uint16_t* __restrict__ wt,
                                           const float* __restrict__ w, int tid)
{
    const int lane = tid & 63, wv = tid >> 6;
    const int row = lane & 15, kq = (lane >> 4) * 8;
    for (int layer = 0; layer < 2; ++layer) {
        const uint16_t* A = layer == 0 ? Ta : Tb;
        uint16_t* O = layer == 0 ? Tb : Ta;
        const uint16_t* Wt = wt + (layer == 0 ? kOffT1 : kOffT2);
        const float* bias = w + (layer == 0 ? kOffB1 : kOffB2);
        f32x4 acc[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k0 = 0; k0 < kMlpHid; k0 += 32) {
            bf16x8 b[2];
#pragma unroll
            for (int j = 0; j < 2; ++j)
                b[j] = *reinterpret_cast<const bf16x8*>(&Wt[(wv * 32 + j * 16 + row) * kMlpHid + k0 + kq]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                bf16x8 a = *reinterpret_cast<const bf16x8*>(&A[(i * 16 + row) * FKP + k0 + kq]);
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[j], acc[i][j], 0, 0, 0);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    int m = i * 16 + (lane >> 4) * 4 + v;
                    int n = wv * 32 + j * 16 + (lane & 15);
                    O[m * FKP + n] = to_bf16(gelu(acc[i][j][v] + bias[n]));
                }
        __syncthreads();
    }
}

// Output columns [n0, n0 + 16) of the last layer for the 64 rows of the tile
// in Ta: lane holds rows i * 16 + 4 (lane / 16) + v, column n0 + lane % 16.
__device__ __forceinline__ void mlp_out16(const uint16_t* Ta, const uint16_t* __restrict__ wt, int n0, int lane,
                                          f32x4 (&acc)[4])
{
    const int row = lane & 15, kq = (lane >> 4) * 8;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k0 = 0; k0 < kMlpHid; k0 += 32) {
        bf16x8 b = *reinterpret_cast<const bf16x8*>(&wt[kOffT3 + (n0 + row) * kMlpHid + k0 + kq]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            bf16x8 a = *reinterpret_cast<const bf16x8*>(&Ta[(i * 16 + row) * FKP + k0 + kq]);
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[i], 0, 0, 0);
        }
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_mlp_infer(int rows, const int* rows_dev, const uint16_t* __restrict__ X,
                                                   const uint16_t* __restrict__ wt, const float* __restrict__ w,
                                                   float* __restrict__ Y)
{
    __shared__ __attribute__((aligned(16))) uint16_t Ta[FR * FKP];
    __shared__ __attribute__((aligned(16))) uint16_t Tb[FR * FKP];
    if (rows_dev) rows = *rows_dev;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int r0 = blockIdx.x * FR; r0 < rows; r0 += gridDim.x * FR) {
        for (int e = tid; e < FR * kMlpIn / 8; e += 256) {
            int r = e / (kMlpIn / 8), c8 = (e % (kMlpIn / 8)) * 8;
            uint4 v = {0u, 0u, 0u, 0u};
            if (r0 + r < rows) v = *reinterpret_cast<const uint4*>(&X[(long)(r0 + r) * kMlpIn + c8]);
            *reinterpret_cast<uint4*>(&Ta[r * FKP + c8]) = v;
        }
        __syncthreads();
        mlp_hidden(Ta, Tb, wt, w, tid);
        // output layer: wave wv computes columns [16 wv, 16 wv + 16)
        f32x4 acc[4];
        mlp_out16(Ta, wt, wv * 16, lane, acc);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                int m = r0 + i * 16 + (lane >> 4) * 4 + v;
                int n = wv * 16 + (lane & 15);
                if (m < rows) Y[(long)m * kMlpOut + n] = acc[i][v] + w[kOffB3 + n];
            }
        __syncthreads();
    }
}

// Inference for the queued small-neighbourhood LPs, with the network input
// built in LDS from their column records (slot s = segment s: exact offset /
// h and mask; q - 2), and only the logits of the eight columns written:
// L[item][8].
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_mlp_infer_small(const int* rows_dev, SmallRec rec, float sc, int q,
                                                         const uint16_t* __restrict__ wt, const float* __restrict__ w,
                                                         float* __restrict__ L)
{
    __shared__ __attribute__((aligned(16))) uint16_t Ta[FR * FKP];
    __shared__ __attribute__((aligned(16))) uint16_t Tb[FR * FKP];
    const int rows = *rows_dev;
    const size_t cap = (size_t)rec.cap;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int r0 = blockIdx.x * FR; r0 < rows; r0 += gridDim.x * FR) {
        for (int e = tid; e < FR * kMlpIn / 8; e += 256) {
            int r = e / (kMlpIn / 8), c8 = (e % (kMlpIn / 8)) * 8;
            *reinterpret_cast<uint4*>(&Ta[r * FKP + c8]) = uint4{0u, 0u, 0u, 0u};
        }
        __syncthreads();
        for (int e = tid; e < FR * VRM_NSEG; e += 256) {
            // consecutive threads take consecutive rows of one segment plane
            const int s = e / FR, r = e % FR;
            const int item = r0 + r;
            if (item < rows) {
                if (rec.pj[s * cap + item] >= 0) {
                    Ta[r * FKP + 2 * s] = to_bf16(rec.off[(4 * s + 0) * cap + item] * sc);
                    Ta[r * FKP + 2 * s + 1] = to_bf16(rec.off[(4 * s + 2) * cap + item] * sc);
                    Ta[r * FKP + 2 * kMlpSlots + s] = 0x3f80;   // 1.0
                }
                if (s == 0) Ta[r * FKP + 3 * kMlpSlots] = q == 3 ? 0x3f80 : 0;
            }
        }
        __syncthreads();
        mlp_hidden(Ta, Tb, wt, w, tid);
        if (wv == 0) {
            f32x4 acc[4];
            mlp_out16(Ta, wt, 0, lane, acc);
            const int n = lane & 15;
            if (n < VRM_NSEG) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        int m = r0 + i * 16 + (lane >> 4) * 4 + v;
                        if (m < rows) L[(long)m * VRM_NSEG + n] = acc[i][v] + w[kOffB3 + n];
                    }
            }
        }
        __syncthreads();
    }
}

// Inference for the queued complete LPs from their column records: the input
// row is built in LDS from the record (slot j < 32 of the nearest-first list:
// offset / h and mask; q - 2), four threads per row, and only the 32 basis
// logits are computed and written: L[item][kMlpSlots].  (Choosing the m
// largest here, at this kernel's occupancy, costs more than a separate pass.)
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_mlp_infer_full(const int* rows_dev, FullRec fr,
                                                        const uint16_t* __restrict__ wt, const float* __restrict__ w,
                                                        float* __restrict__ Lout)
{
    __shared__ __attribute__((aligned(16))) uint16_t Ta[FR * FKP];
    __shared__ __attribute__((aligned(16))) uint16_t Tb[FR * FKP];
    constexpr int LS = kMlpSlots + 1;   // row stride of the logits (staged in Tb)
    static_assert(FR * LS * sizeof(float) <= sizeof(Tb), "the logits fit in the second tile");
    const int rows = *rows_dev;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int rr = tid >> 2, part = tid & 3;   // this thread's row of the tile, its quarter of the slots
    for (int r0 = blockIdx.x * FR; r0 < rows; r0 += gridDim.x * FR) {
        const int r = r0 + rr;
        const int k = r < rows ? fr.kcol[r] : -1;
        {
            float xi = 0.0f, yi = 0.0f;
            if (k > 0) {
                const int t = fr.q_full[r];
                xi = fr.xs[t];
                yi = fr.ys[t];
            }
            const int32_t* rrow = fr.rec + (size_t)r * fr.row;
            uint32_t off[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int j = 8 * part + i;
                uint32_t pr = 0;
                if (j < k) {
                    const int u = (int)((unsigned)rrow[j] >> 6);
                    pr = (uint32_t)to_bf16(((fr.xs[u] - xi) * fr.scale2e) * fr.sc) |
                         ((uint32_t)to_bf16(((fr.ys[u] - yi) * fr.scale2e) * fr.sc) << 16);
                }
                off[i] = pr;
            }
            uint16_t* row = Ta + rr * FKP;
            // elements 16 part .. 16 part + 15: the offset pairs of slots 8 part .. 8 part + 7
            *reinterpret_cast<uint4*>(row + 16 * part) = uint4{off[0], off[1], off[2], off[3]};
            *reinterpret_cast<uint4*>(row + 16 * part + 8) = uint4{off[4], off[5], off[6], off[7]};
            // their masks, then q - 2 (element 3 kMlpSlots) and zero padding
            uint32_t mk[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = 8 * part + 2 * i;
                mk[i] = (j < k ? 0x3f80u : 0u) | ((j + 1 < k ? 0x3f80u : 0u) << 16);
            }
            *reinterpret_cast<uint4*>(row + 2 * kMlpSlots + 8 * part) = uint4{mk[0], mk[1], mk[2], mk[3]};
            *reinterpret_cast<uint4*>(row + 3 * kMlpSlots + 8 * part) =
                uint4{part == 0 && fr.q == 3 ? 0x3f80u : 0u, 0u, 0u, 0u};
        }
        __syncthreads();
        mlp_hidden(Ta, Tb, wt, w, tid);
        // the logits: waves 0 and 1 compute columns [16 wv, 16 wv + 16) of the 64 rows
        float* L = reinterpret_cast<float*>(Tb);
        if (wv < 2) {
            f32x4 acc[4];
            mlp_out16(Ta, wt, wv * 16, lane, acc);
            const int n = wv * 16 + (lane & 15);
            const float b = w[kOffB3 + n];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) L[(i * 16 + (lane >> 4) * 4 + v) * LS + n] = acc[i][v] + b;
        }
        __syncthreads();
        if (r < rows) {
            float4* dst = reinterpret_cast<float4*>(Lout + (size_t)r * kMlpSlots + 8 * part);
            // LS is odd: the row start is not 16-byte aligned in LDS, so the values are read one by one
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = L[rr * LS + 8 * part + i];
            dst[0] = float4{v[0], v[1], v[2], v[3]};
            dst[1] = float4{v[4], v[5], v[6], v[7]};
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- training
// Transposed BF16 operands of the weight gradients, [rows / 32][feature][32 rows]: a
// fragment of 16 features is 1 KB in one piece, its 8 rows per lane one 16-byte load.
constexpr int kRowBlk = 32;
__device__ __forceinline__ size_t t_index(int features, int f, long row)
{
    return ((size_t)(row / kRowBlk) * features + f) * kRowBlk + (size_t)(row % kRowBlk);
}

__device__ __forceinline__ bf16x8 frag(const uint16_t* p) { return *reinterpret_cast<const bf16x8*>(p); }

// Rows kernel: forward pass, loss and the backward pass to the pre-activations for
// tiles of 16 rows.  Wave wv holds columns [32 wv, 32 wv + 32) of the hidden layers and
// [16 wv, 16 wv + 16) of the output.  Masked loss, averaged over rows: BCE-with-logits on
// the basis indicators (output columns below 32) and squared error on the fractions.
// At the trainer's 4096 rows this is bound by latency, one tile per CU: five dependent
// layers.  So a wave keeps its columns of every weight matrix in registers, fetched at
// once at the start (L2; 128 VGPRs), and the tile's activations go from layer to layer
// through LDS; pre-activations stay in registers until the backward pass needs them.
// Before (17 launches: a tiled product per layer and direction, the loss, column sums,
// clears and copies) a step of 4096 rows took 149 us, of 64 rows 85, of 65536 rows 1263;
// now 22.2, 12.5 and 129 us (this kernel 15.5, 10.3 and 71 us of them); rows of normal
// offsets in every slot.  (The trainer's own 4096 rows: 150 us, now 17.9.)  Two workgroups
// per CU (256 VGPRs, 19 of them spilled) measured 23.1 us, 13.5 us and 119 us.
constexpr int kTrainTile = 16;
constexpr int kTrainBlocks = 256;              // one per CU; more rows: loop
constexpr int kBiasCols = 2 * kMlpHid + kMlpOut;
constexpr int DYP = kMlpOut + 8;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1))) void k_train_rows(
    int rows, int tiles, const uint16_t* __restrict__ X, const float* __restrict__ T, const uint16_t* __restrict__ wt,
    const uint16_t* __restrict__ wbf, const float* __restrict__ w, float wf, uint16_t* __restrict__ xt,
    uint16_t* __restrict__ h1t, uint16_t* __restrict__ h2t, uint16_t* __restrict__ dyt, uint16_t* __restrict__ dz2t,
    uint16_t* __restrict__ dz1t, float* __restrict__ bias_part, double* __restrict__ loss_part)
{
    __shared__ __attribute__((aligned(16))) uint16_t Ta[kTrainTile * FKP];   // x, h2, dz2
    __shared__ __attribute__((aligned(16))) uint16_t Tb[kTrainTile * FKP];   // h1
    __shared__ __attribute__((aligned(16))) uint16_t Ty[kTrainTile * DYP];   // dy
    __shared__ double s_loss[4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int row = lane & 15, quad = lane >> 4, kq = quad * 8;
    const bool x_aligned = (reinterpret_cast<uintptr_t>(X) & 15) == 0;
    const float inv = 1.0f / (float)rows;
    bf16x8 w1[4][2], w2[4][2], w3[4], v3[2][2], v2[4][2];
    float b1[2], b2[2], b3;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = wv * 32 + j * 16 + row;
            w1[k][j] = frag(&wt[kOffT1 + n * kMlpIn + 32 * k + kq]);
            w2[k][j] = frag(&wt[kOffT2 + n * kMlpHid + 32 * k + kq]);
            v2[k][j] = frag(&wbf[kOffW2 + n * kMlpHid + 32 * k + kq]);
            if (k < 2) v3[k][j] = frag(&wbf[kOffW3 + n * kMlpOut + 32 * k + kq]);
            if (k == 0) {
                b1[j] = w[kOffB1 + n];
                b2[j] = w[kOffB2 + n];
            }
        }
        w3[k] = frag(&wt[kOffT3 + (wv * 16 + row) * kMlpHid + 32 * k + kq]);
    }
    b3 = w[kOffB3 + wv * 16 + row];
    float s1[2] = {0.0f, 0.0f}, s2[2] = {0.0f, 0.0f}, s3 = 0.0f;   // column sums
    double loss = 0.0;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const long r0 = (long)tile * kTrainTile;
        // the targets of this lane's outputs: rows 4 quad + v, column 16 wv + row
        float y[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const long r = r0 + 4 * quad + v;
            y[v] = r < rows ? T[r * kMlpOut + wv * 16 + row] : 0.0f;
        }
        {
            const int r = tid >> 4, c8 = (tid & 15) * 8;
            uint4 v = {0u, 0u, 0u, 0u};
            if (r0 + r < rows) {
                const uint16_t* src = &X[(r0 + r) * kMlpIn + c8];
                if (x_aligned) {
                    v = *reinterpret_cast<const uint4*>(src);
                } else {
                    uint32_t e[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) e[k] = (uint32_t)src[2 * k] | ((uint32_t)src[2 * k + 1] << 16);
                    v = uint4{e[0], e[1], e[2], e[3]};
                }
            }
            *reinterpret_cast<uint4*>(&Ta[r * FKP + c8]) = v;
        }
        __syncthreads();
        float mask[4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            mask[v] = from_bf16(Ta[(4 * quad + v) * FKP + 2 * kMlpSlots + (wv & 1) * 16 + row]);
        {
            // the tile transposed: eight rows of one input per thread
            const int c = tid & (kMlpIn - 1), o = (tid >> 7) * 8;
            uint32_t e[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                e[k] = (uint32_t)Ta[(o + 2 * k) * FKP + c] | ((uint32_t)Ta[(o + 2 * k + 1) * FKP + c] << 16);
            *reinterpret_cast<uint4*>(&xt[t_index(kMlpIn, c, r0 + o)]) = uint4{e[0], e[1], e[2], e[3]};
        }
        f32x4 z1[2], z2[2];
        // one hidden layer: A -> z (kept), GELU -> O and the transposed copy
        auto hidden = [&](const uint16_t* A, const bf16x8 (&wk)[4][2], const float (&b)[2], f32x4 (&z)[2], uint16_t* O,
                          uint16_t* ot) {
#pragma unroll
            for (int j = 0; j < 2; ++j) z[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bf16x8 a = frag(&A[row * FKP + 32 * k + kq]);
#pragma unroll
                for (int j = 0; j < 2; ++j) z[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, wk[k][j], z[j], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = wv * 32 + j * 16 + row;
                uint16_t e[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    z[j][v] += b[j];
                    e[v] = to_bf16(gelu(z[j][v]));
                    O[(4 * quad + v) * FKP + n] = e[v];
                    if (r0 + 4 * quad + v >= rows) e[v] = 0;
                }
                *reinterpret_cast<uint2*>(&ot[t_index(kMlpHid, n, r0 + 4 * quad)]) =
                    uint2{(uint32_t)e[0] | ((uint32_t)e[1] << 16), (uint32_t)e[2] | ((uint32_t)e[3] << 16)};
            }
            __syncthreads();
        };
        hidden(Ta, w1, b1, z1, Tb, h1t);
        hidden(Tb, w2, b2, z2, Ta, h2t);
        {
            f32x4 p = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(&Ta[row * FKP + 32 * k + kq]), w3[k], p, 0, 0, 0);
            uint16_t e[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float z = p[v] + b3;
                float g;
                if (wv < 2) {
                    const float sp = fmaxf(z, 0.0f) + log1pf(__expf(-fabsf(z)));   // softplus
                    const float sig = 1.0f / (1.0f + __expf(-z));
                    loss += (double)(mask[v] * (sp - y[v] * z) * inv);
                    g = mask[v] * (sig - y[v]) * inv;
                } else {
                    loss += (double)(mask[v] * (wf * (z - y[v]) * (z - y[v])) * inv);
                    g = mask[v] * wf * 2.0f * (z - y[v]) * inv;
                }
                // (no loss from rows past the last: their mask is zero, but the outputs may not be finite)
                if (r0 + 4 * quad + v >= rows) g = 0.0f;
                s3 += g;
                e[v] = to_bf16(g);
                Ty[(4 * quad + v) * DYP + wv * 16 + row] = e[v];
            }
            *reinterpret_cast<uint2*>(&dyt[t_index(kMlpOut, wv * 16 + row, r0 + 4 * quad)]) =
                uint2{(uint32_t)e[0] | ((uint32_t)e[1] << 16), (uint32_t)e[2] | ((uint32_t)e[3] << 16)};
        }
        __syncthreads();
        // d loss / d pre-activation of a hidden layer: (A W^T) gelu'(z)
        auto backward = [&](f32x4 (&d)[2], const f32x4 (&z)[2], float (&sum)[2], uint16_t* O, uint16_t* ot) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = wv * 32 + j * 16 + row;
                uint16_t e[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float g = d[j][v] * gelu_grad(z[j][v]);
                    if (r0 + 4 * quad + v >= rows) g = 0.0f;
                    sum[j] += g;
                    e[v] = to_bf16(g);
                    if (O) O[(4 * quad + v) * FKP + n] = e[v];
                }
                *reinterpret_cast<uint2*>(&ot[t_index(kMlpHid, n, r0 + 4 * quad)]) =
                    uint2{(uint32_t)e[0] | ((uint32_t)e[1] << 16), (uint32_t)e[2] | ((uint32_t)e[3] << 16)};
            }
        };
        f32x4 d[2] = {f32x4{0.0f, 0.0f, 0.0f, 0.0f}, f32x4{0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const bf16x8 a = frag(&Ty[row * DYP + 32 * k + kq]);
#pragma unroll
            for (int j = 0; j < 2; ++j) d[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, v3[k][j], d[j], 0, 0, 0);
        }
        backward(d, z2, s2, Ta, dz2t);
        __syncthreads();
        d[0] = d[1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bf16x8 a = frag(&Ta[row * FKP + 32 * k + kq]);
#pragma unroll
            for (int j = 0; j < 2; ++j) d[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, v2[k][j], d[j], 0, 0, 0);
        }
        backward(d, z1, s1, nullptr, dz1t);
        __syncthreads();   // the next tile overwrites Ta
    }
    // column sums of this workgroup's rows: the four lanes of a column
    auto column = [&](float s) {
        s += __shfl_xor(s, 16, VRM_WAVE);
        return s + __shfl_xor(s, 32, VRM_WAVE);
    };
    float* part = bias_part + (size_t)blockIdx.x * kBiasCols;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const float a = column(s1[j]), b = column(s2[j]);
        if (quad == 0) {
            part[wv * 32 + j * 16 + row] = a;
            part[kMlpHid + wv * 32 + j * 16 + row] = b;
        }
    }
    const float b = column(s3);
    if (quad == 0) part[2 * kMlpHid + wv * 16 + row] = b;
    for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, VRM_WAVE);
    if (lane == 0) s_loss[wv] = loss;
    __syncthreads();
    if (tid == 0) loss_part[blockIdx.x] = s_loss[0] + s_loss[1] + s_loss[2] + s_loss[3];
}

struct AdamW {
    float lr, wd, c1, c2;   // lr 0: no step
    float *w, *m, *v, *grad;
    uint16_t *wbf, *wt;
};

// the gradient of parameter i out, and its step; returns the BF16 weight
__device__ __forceinline__ uint16_t adamw(const AdamW& a, int i, float g)
{
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    if (a.grad) a.grad[i] = g;
    if (!(a.lr > 0.0f)) return 0;
    const float mi = b1 * a.m[i] + (1.0f - b1) * g;
    const float vi = b2 * a.v[i] + (1.0f - b2) * g * g;
    a.m[i] = mi;
    a.v[i] = vi;
    const float mh = mi / a.c1, vh = vi / a.c2;
    const float wi = a.w[i] - a.lr * (mh / (sqrtf(vh) + eps) + a.wd * a.w[i]);
    a.w[i] = wi;
    const uint16_t h = to_bf16(wi);
    a.wbf[i] = h;
    return h;
}

// Parameters kernel.  A workgroup of 16 waves owns a 16 x 16 block of one weight
// matrix: the waves take the row blocks in turn, their sums meet in LDS, and the same
// workgroup makes the parameters' AdamW step: no atomics, no cleared sums, one order of
// additions in every run.  160 workgroups read 32 features each (42 MB of L2 reads at
// 4096 rows, in 6 to 8 us; 61 us at 65536 rows); larger blocks read less but leave more of
// the chip idle.  Five more workgroups sum the bias gradients, the last of them the loss.
constexpr int kTilesW = (kMlpHid / 16) * (kMlpHid / 16), kTilesW3 = (kMlpHid / 16) * (kMlpOut / 16);
__global__ __launch_bounds__(1024) void k_train_params(int nblk32, int parts, const uint16_t* __restrict__ xt,
                                                       const uint16_t* __restrict__ h1t,
                                                       const uint16_t* __restrict__ h2t,
                                                       const uint16_t* __restrict__ dyt,
                                                       const uint16_t* __restrict__ dz2t,
                                                       const uint16_t* __restrict__ dz1t,
                                                       const float* __restrict__ bias_part,
                                                       const double* __restrict__ loss_part, double* loss_out, AdamW a)
{
    static_assert(kMlpIn == kMlpHid, "one tile count for the first two layers");
    __shared__ float red[16][256];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int b = blockIdx.x;
    if (b < 2 * kTilesW + kTilesW3) {
        const int layer = b / kTilesW;   // the third holds fewer tiles
        b -= layer * kTilesW;
        const int nout = layer == 2 ? kMlpOut : kMlpHid;
        const int m0 = b / (nout / 16) * 16, n0 = b % (nout / 16) * 16;
        const uint16_t* A = layer == 0 ? xt : layer == 1 ? h1t : h2t;
        const uint16_t* B = layer == 0 ? dz1t : layer == 1 ? dz2t : dyt;
        const int row = lane & 15, quad = lane >> 4;
        const uint16_t* pa = A + (size_t)(m0 + row) * kRowBlk + quad * 8;
        const uint16_t* pb = B + (size_t)(n0 + row) * kRowBlk + quad * 8;
        const size_t sa = (size_t)kMlpHid * kRowBlk, sb = (size_t)nout * kRowBlk;
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
        for (int k = wv; k < nblk32; k += 16)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(pa + k * sa), frag(pb + k * sb), acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wv][(4 * quad + v) * 16 + row] = acc[v];
        __syncthreads();
        if (tid < 256) {
            float g = 0.0f;
#pragma unroll
            for (int k = 0; k < 16; ++k) g += red[k][tid];
            const int m = m0 + tid / 16, n = n0 + tid % 16;
            const int off = layer == 0 ? kOffW1 : layer == 1 ? kOffW2 : kOffW3;
            const int toff = layer == 0 ? kOffT1 : layer == 1 ? kOffT2 : kOffT3;
            const uint16_t h = adamw(a, off + m * nout + n, g);
            if (a.lr > 0.0f) a.wt[toff + n * kMlpHid + m] = h;
        }
        return;
    }
    b -= 2 * kTilesW + kTilesW3;   // bias columns [64 b, 64 b + 64)
    const int col = 64 * b + lane;
    float s = 0.0f;
#pragma unroll 8
    for (int p = wv; p < parts; p += 16) s += bias_part[(size_t)p * kBiasCols + col];
    red[wv][lane] = s;
    __syncthreads();
    if (tid < 64) {
        float g = 0.0f;
#pragma unroll
        for (int k = 0; k < 16; ++k) g += red[k][lane];
        (void)adamw(a, col < kMlpHid ? kOffB1 + col : col < 2 * kMlpHid ? kOffB2 + col - kMlpHid : kOffB3 + col - 2 * kMlpHid, g);
    } else if (tid < 128 && b == kBiasCols / 64 - 1 && loss_out) {
        double l = 0.0;
        for (int p = lane; p < parts; p += 64) l += loss_part[p];
        for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, VRM_WAVE);
        if (lane == 0) *loss_out = l;
    }
}

}  // namespace

// ----------------------------------------------------------------- host
int vrm_mlp_read_weights(vrm_ctx* c, float* w_dev)
{
    VRM_HIP(hipMemcpyAsync(w_dev, c->mlp->w, sizeof(float) * kMlpParams, hipMemcpyDeviceToDevice, c->stream));
    return VRM_OK;
}

int vrm_mlp_alloc(vrm_ctx* c, int max_rows)
{
    if (c->mlp && c->mlp->max_rows >= max_rows) return VRM_OK;
    MlpState* m = c->mlp;
    void* p;
#define AL(field, bytes)                            \
    VRM_HIP(hipMalloc(&p, (bytes) + 64));           \
    m->field = reinterpret_cast<decltype(m->field)>(p);
    if (!m) {
        m = new MlpState();
        std::memset(m, 0, sizeof(*m));
        AL(w, sizeof(float) * kMlpParams);
        AL(am, sizeof(float) * kMlpParams);
        AL(av, sizeof(float) * kMlpParams);
        AL(wbf, sizeof(uint16_t) * kMlpParams);
        AL(wt, sizeof(uint16_t) * kWtSize);
        AL(loss_part, sizeof(double) * kTrainBlocks);
        AL(bias_part, sizeof(float) * kTrainBlocks * kBiasCols);
        VRM_HIP(hipMemsetAsync(m->w, 0, sizeof(float) * kMlpParams, c->stream));
        VRM_HIP(hipMemsetAsync(m->wbf, 0, sizeof(uint16_t) * kMlpParams, c->stream));
        VRM_HIP(hipMemsetAsync(m->am, 0, sizeof(float) * kMlpParams, c->stream));
        VRM_HIP(hipMemsetAsync(m->av, 0, sizeof(float) * kMlpParams, c->stream));
        c->mlp = m;
    }
    if (max_rows > m->max_rows) {
        uint16_t** bufs[] = {&m->xt, &m->h1t, &m->h2t, &m->dyt, &m->dz2t, &m->dz1t};
        VRM_HIP(hipStreamSynchronize(c->stream));
        m->max_rows = 0;
        for (uint16_t** q : bufs) {
            if (*q) (void)hipFree(*q);
            *q = nullptr;
        }
        // whole blocks of 32 rows
        const size_t R = ((size_t)max_rows + kRowBlk - 1) / kRowBlk * kRowBlk;
        AL(xt, sizeof(uint16_t) * R * kMlpIn);
        AL(h1t, sizeof(uint16_t) * R * kMlpHid);
        AL(h2t, sizeof(uint16_t) * R * kMlpHid);
        AL(dyt, sizeof(uint16_t) * R * kMlpOut);
        AL(dz2t, sizeof(uint16_t) * R * kMlpHid);
        AL(dz1t, sizeof(uint16_t) * R * kMlpHid);
        m->max_rows = max_rows;
    }
#undef AL
    return VRM_OK;
}

void vrm_mlp_free(vrm_ctx* c)
{
    if (!c->mlp) return;
    MlpState* m = c->mlp;
    void* ptrs[] = {m->w, m->am, m->av, m->wbf, m->wt, m->xt, m->h1t, m->h2t, m->dyt, m->dz2t, m->dz1t,
                    m->bias_part, m->loss_part};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    delete m;
    c->mlp = nullptr;
}

int vrm_mlp_set_weights(vrm_ctx* c, const float* w_dev)
{
    MlpState* m = c->mlp;
    VRM_HIP(hipMemcpyAsync(m->w, w_dev, sizeof(float) * kMlpParams, hipMemcpyDeviceToDevice, c->stream));
    hipLaunchKernelGGL(k_to_bf16, dim3(nblk(kMlpParams)), dim3(256), 0, c->stream, kMlpParams, m->w, m->wbf);
    hipLaunchKernelGGL(k_transpose_w, dim3(nblk(kMlpIn * kMlpHid)), dim3(256), 0, c->stream, m->wbf, m->wt);
    VRM_HIP(hipGetLastError());
    VRM_HIP(hipMemsetAsync(m->am, 0, sizeof(float) * kMlpParams, c->stream));
    VRM_HIP(hipMemsetAsync(m->av, 0, sizeof(float) * kMlpParams, c->stream));
    m->step = 0;
    m->loaded = 1;
    return VRM_OK;
}

// fused forward for inference (no intermediate buffers); rows may be an upper bound with rows_dev
int vrm_mlp_infer_small_run(vrm_ctx* c, int rows, const int* rows_dev, const SmallRec& rec, float sc, int q, float* L)
{
    if (rows <= 0) return VRM_OK;
    MlpState* m = c->mlp;
    int tiles = (rows + FR - 1) / FR;
    int grid = tiles < c->tuning.infer_blocks ? tiles : c->tuning.infer_blocks;
    hipLaunchKernelGGL(k_mlp_infer_small, dim3(grid), dim3(256), 0, c->stream, rows_dev, rec, sc, q, m->wt, m->w, L);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

int vrm_mlp_infer_full_run(vrm_ctx* c, int rows, const int* rows_dev, const FullRec& fr, float* L)
{
    if (rows <= 0) return VRM_OK;
    MlpState* m = c->mlp;
    int tiles = (rows + FR - 1) / FR;
    int grid = tiles < c->tuning.infer_blocks ? tiles : c->tuning.infer_blocks;
    hipLaunchKernelGGL(k_mlp_infer_full, dim3(grid), dim3(256), 0, c->stream, rows_dev, fr, m->wt, m->w, L);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

int vrm_mlp_infer_run(vrm_ctx* c, const uint16_t* X, int rows, float* Y, const int* rows_dev)
{
    if (rows <= 0) return VRM_OK;
    MlpState* m = c->mlp;
    int tiles = (rows + FR - 1) / FR;
    int grid = tiles < c->tuning.infer_blocks ? tiles : c->tuning.infer_blocks;
    hipLaunchKernelGGL(k_mlp_infer, dim3(grid), dim3(256), 0, c->stream, rows, rows_dev, X, m->wt, m->w, Y);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

// one AdamW step on the masked BCE + MSE loss of a batch (X, T)
int vrm_mlp_train(vrm_ctx* c, const uint16_t* X, const float* T, int rows, float lr, float wd, float wf,
                  double* loss_out, float* grad_out)
{
    MlpState* m = c->mlp;
    hipStream_t s = c->stream;
    // tiles of 16 rows, an even number of them (the row blocks of 32 are written whole)
    const int nblk32 = (int)(((long)rows + kRowBlk - 1) / kRowBlk);
    const int tiles = nblk32 * (kRowBlk / kTrainTile);
    const int parts = tiles < kTrainBlocks ? tiles : kTrainBlocks;
    hipLaunchKernelGGL(k_train_rows, dim3(parts), dim3(256), 0, s, rows, tiles, X, T, m->wt, m->wbf, m->w, wf, m->xt,
                       m->h1t, m->h2t, m->dyt, m->dz2t, m->dz1t, m->bias_part, m->loss_part);
    AdamW a{lr, wd, 1.0f, 1.0f, m->w, m->am, m->av, grad_out, m->wbf, m->wt};
    if (lr > 0.0f) {
        m->step += 1;
        a.c1 = 1.0f - powf(0.9f, (float)m->step);
        a.c2 = 1.0f - powf(0.999f, (float)m->step);
    }
    hipLaunchKernelGGL(k_train_params, dim3(2 * kTilesW + kTilesW3 + kBiasCols / 64), dim3(1024), 0, s, nblk32, parts,
                       m->xt, m->h1t, m->h2t, m->dyt, m->dz2t, m->dz1t, m->bias_part, m->loss_part, loss_out, a);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}

// plain product for tests: C (FP32, M x N) = A (BF16, M x K, row-major) * B (BF16, K x N, row-major)
int vrm_gemm_test(vrm_ctx* c, const uint16_t* A, const uint16_t* B, float* C, int M, int N, int K, int transA,
                  int transB)
{
    long sam = transA ? 1 : K, sak = transA ? M : 1;
    long sbk = transB ? 1 : N, sbn = transB ? K : 1;
    const int splitk = K >= 1024 ? 8 : 1;
    const int kchunk = splitk > 1 ? ((K + splitk - 1) / splitk + TK - 1) / TK * TK : K;
    hipLaunchKernelGGL(k_gemm, dim3((N + TN - 1) / TN, (M + TM - 1) / TM, (K + kchunk - 1) / kchunk), dim3(256), 0,
                       c->stream, M, N, K, A, sam, sak, B, sbk, sbn, C, (long)N, kchunk);
    VRM_HIP(hipGetLastError());
    return VRM_OK;
}
