// ezo_mlp.hpp -- kernels of the learned self-collision screen: a multilayer
// perceptron dof -> H -> H -> H -> 1 with SiLU activations that predicts a
// configuration's minimum self-collision signed distance from x = q / pi.
//
// Parameters (FP32 master copy, one flat vector):
//   W1[H][D] b1[H] W2[H][H] b2[H] W3[H][H] b3[H] W4[H] b4[1]   (z = W a + b)
// BF16 copies of W2 and W3 feed the MFMA GEMMs (FP32 accumulation); the
// first and last layers (K = dof and N = 1) run on the vector ALUs.
// Activations between layers are BF16; pre-activations kept for the
// backward pass are FP32.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ezo_device.hpp"
#include "ezo_screen.hpp"

namespace ezo {

__device__ __forceinline__ const float* row_ptr(const RowSource& s, int64_t r, int64_t* stride) {
    r += s.rbase;
    int64_t cfg = s.idx ? (int64_t)s.idx[r] : r;
    const float* base = s.q;
    if (s.rows_per_batch > 0) {
        base += (r / s.rows_per_batch) * s.qb;
        cfg = r % s.rows_per_batch;
    }
    *stride = s.sd;
    return base + cfg * s.sn;
}

// Row r of this launch is inactive: past the valid rows, or in a batch
// (edge) whose status is final.
__device__ __forceinline__ bool row_inactive(const RowSource& s, int64_t r, const int* status) {
    if (r >= s.rows) return true;
    return status && s.rows_per_batch > 0 && status[(r + s.rbase) / s.rows_per_batch] >= 0;
}

// Layer 1 on the VALUs: z1 = W1 (q / pi) + b1; h1 = bf16(silu(z1)); z1 kept
// (FP32) when z1out != NULL.  One thread per (row, unit).
__global__ void __launch_bounds__(256) k_mlp_layer1(RowSource src, int64_t rows, int D, int H,
                                                    const float* __restrict__ P, float* __restrict__ z1out,
                                                    __bf16* __restrict__ h1, const int* __restrict__ status) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= rows * H) return;
    const int64_t r = t / H;
    const int i = (int)(t % H);
    if (row_inactive(src, r, status)) {
        if (z1out) z1out[t] = 0.f;
        h1[t] = (__bf16)0.f;
        return;
    }
    const MlpOffsets o = mlp_offsets(D, H);
    int64_t sd;
    const float* x = row_ptr(src, r, &sd);
    float z = P[o.b1 + i];
    for (int j = 0; j < D; ++j) z = fmaf(P[o.W1 + (int64_t)i * D + j], x[j * sd] * kInvPi, z);
    if (z1out) z1out[t] = z;
    h1[t] = (__bf16)siluf(z);
}

// Output layer on the VALUs: y = W4 . h3 + b4, one thread per row.
__global__ void __launch_bounds__(256) k_mlp_out(RowSource src, int64_t rows, int D, int H, const float* __restrict__ P,
                                                 const __bf16* __restrict__ h3, float* __restrict__ y,
                                                 const int* __restrict__ status) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rows || row_inactive(src, r, status)) return;
    const MlpOffsets o = mlp_offsets(D, H);
    const bf16x8* h = reinterpret_cast<const bf16x8*>(h3 + r * H);
    float s = P[o.b4];
    for (int k = 0; k < H / 8; ++k) {
        const bf16x8 v = h[k];
#pragma unroll
        for (int e = 0; e < 8; ++e) s = fmaf(P[o.W4 + 8 * k + e], (float)v[e], s);
    }
    y[r] = s;
}

// ---------------------------------------------------------------------------
// Whole forward pass of rows without batches, H = 64 HB <= 256: persistent
// workgroups of 4 HB waves take 16 RB rows at a time; wave w owns units
// 16 w .. + 15 of every layer and keeps their BF16 weights of both hidden layers
// in registers (64 VGPRs at H = 256), so that a tile reads its inputs and
// writes its outputs only: the activations of one layer go to the next through
// LDS (two buffers).  Products are taken as W h: lane l of a 16x16 result holds
// units 4 (l / 16) .. + 3 of row l % 16, four neighbours of one activation row.
// Layer 1 is v_mfma_f32_16x16x4_f32 started from the bias (a chain of fmaf in
// the order of the inputs); the hidden layers keep K ascending and the bias
// after the sum.  The products of the next 16 rows stand between the activations
// of these, and the next tile passes layer 1 beside this one's layer 3.
// Bound by issue: ten VALU slots an activation, two of them transcendental
// (0.34 ms for 1 M rows at H = 256), and the products (0.14 ms).  1 M rows at
// H = 256: layer, two products and output as launches of their own, activations
// through memory, 2540 us; this 480 us.
// ---------------------------------------------------------------------------
constexpr int kPredU = 1;                // 16-unit tiles per wave (two: 423 us against 345 at H = 192, 473 against 480 at 256)

template <int HB>
__host__ __device__ constexpr size_t predict_lds_bytes(int RB) {
    return sizeof(__bf16) * (size_t)2 * 16 * RB * (64 * HB) + sizeof(float) * (size_t)4 * HB / kPredU * 16 * RB;
}

typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;

// z (+ b) through the activation, rounded to BF16
__device__ __forceinline__ bf16x4 silu4(f32x4 z) {
    bf16x4 h;
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = (__bf16)siluf(z[r]);
    return h;
}
__device__ __forceinline__ bf16x4 silu4(f32x4 z, f32x4 b) {
#pragma unroll
    for (int r = 0; r < 4; ++r) z[r] += b[r];
    return silu4(z);
}

template <int HB, int RB>
__global__ void __launch_bounds__(256 * HB / kPredU, 4)
k_mlp_predict(RowSource src, int D, const float* __restrict__ P, const __bf16* __restrict__ W2b,
              const __bf16* __restrict__ W3b, float* __restrict__ y) {
    constexpr int H = 64 * HB, LD = H, KS = H / 32, R = 16 * RB, U = kPredU, NW = 4 * HB / U;
    extern __shared__ __attribute__((aligned(16))) __bf16 predict_lds[];
    __bf16* const ha = predict_lds;
    __bf16* const hb = ha + R * LD;
    float* const red = reinterpret_cast<float*>(hb + R * LD);        // [NW][R] partial outputs
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, g = lane >> 4, n0 = 16 * U * w;
    const MlpOffsets o = mlp_offsets(D, H);
    // 16-byte chunk j of row r (r % 16 == c) stands at chunk j ^ sc of its row, so
    // that the 16-lane groups of a 128-bit LDS read, which mix two values of g,
    // touch every bank once
    const int sc = HB % 2 ? c >> 1 : c;
    auto at = [&](__bf16* h, int rb, int chunk) { return h + (16 * rb + c) * LD + 8 * (chunk ^ sc); };
    const int wc = (n0 + 4 * g) >> 3, wo = 4 * (g & 1);              // where this lane's results go
    bf16x8 w2[U][KS], w3[U][KS];
    float w1[U][2];
    f32x4 b1[U], b2[U], b3[U], w4[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int n = n0 + 16 * u + c;                               // this lane's unit as a weight row
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            w2[u][k] = *reinterpret_cast<const bf16x8*>(W2b + n * H + 32 * k + 8 * g);
            w3[u][k] = *reinterpret_cast<const bf16x8*>(W3b + n * H + 32 * k + 8 * g);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) w1[u][s] = 4 * s + g < D ? P[o.W1 + n * D + 4 * s + g] : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = n0 + 16 * u + 4 * g + r;                   // the units of its results
            b1[u][r] = P[o.b1 + m];
            b2[u][r] = P[o.b2 + m];
            b3[u][r] = P[o.b3 + m];
            w4[u][r] = P[o.W4 + m];
        }
    }
    const float b4 = P[o.b4];
    const int64_t tiles = (src.rows + R - 1) / R;
    float x[RB][2];
    auto load_x = [&](int64_t t) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int64_t r = t * R + 16 * rb + c;
            const bool ok = r < src.rows;
            const float* q = src.q + (ok ? r : 0) * src.sn + g * src.sd;
#pragma unroll
            for (int s = 0; s < 2; ++s) x[rb][s] = ok && 4 * s + g < D ? q[4 * s * src.sd] : 0.f;
        }
    };
    auto layer1 = [&] {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                f32x4 z = b1[u];
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[u][s], x[rb][s] * kInvPi, z, 0, 0, 0);
                *reinterpret_cast<bf16x4*>(at(ha, rb, wc + 2 * u) + wo) = silu4(z);
            }
    };
    // both unit tiles of a hidden layer for one block of 16 rows
    auto hidden = [&](__bf16* h, const bf16x8 (&wt)[U][KS], int rb, f32x4 (&z)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) z[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(at(h, rb, 4 * k + g));
#pragma unroll
            for (int u = 0; u < U; ++u) z[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[u][k], a, z[u], 0, 0, 0);
        }
    };
    // the matrix unit's work on the next 16 rows between the activations of these
    auto mix = [&](bool next) {
        if (next)
#pragma unroll
            for (int k = 0; k < U * KS; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // one MFMA
                __builtin_amdgcn_sched_group_barrier(0x002, 40 / KS, 0);     // its share of the VALU work
            }
    };
    auto store = [&](int64_t t) {
        for (int r = tid; r < R; r += 64 * NW) {
            float s = b4;
#pragma unroll
            for (int v = 0; v < NW; ++v) s += red[v * R + r];
            if (t * R + r < src.rows) y[t * R + r] = s;
        }
    };
    int64_t t = blockIdx.x, done = -1;
    if (t >= tiles) return;
    load_x(t);
    layer1();
    while (true) {
        const int64_t tn = t + gridDim.x;
        __syncthreads();
        if (done >= 0) store(done);
        if (tn < tiles) load_x(tn);
        f32x4 z[2][U];
        hidden(ha, w2, 0, z[0]);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if (rb + 1 < RB) hidden(ha, w2, rb + 1, z[(rb + 1) & 1]);
#pragma unroll
            for (int u = 0; u < U; ++u)
                *reinterpret_cast<bf16x4*>(at(hb, rb, wc + 2 * u) + wo) = silu4(z[rb & 1][u], b2[u]);
            mix(rb + 1 < RB);
        }
        __syncthreads();
        hidden(hb, w3, 0, z[0]);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            if (rb + 1 < RB) hidden(hb, w3, rb + 1, z[(rb + 1) & 1]);
            float s = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bf16x4 h = silu4(z[rb & 1][u], b3[u]);
#pragma unroll
                for (int r = 0; r < 4; ++r) s = fmaf(w4[u][r], (float)h[r], s);
            }
            mix(rb + 1 < RB);
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (g == 0) red[w * R + 16 * rb + c] = s;
        }
        done = t;
        if (tn >= tiles) break;
        layer1();
        t = tn;
    }
    __syncthreads();
    store(done);
}

// ---------------------------------------------------------------------------
// BF16 MFMA GEMM  C[M][N] = sum_k A(m, k) B(k, n)
// A(m, k) = A[m*sam + k*sak] with AK: sak == 1 (K contiguous) else sam == 1
// (M contiguous); B(k, n) = B[k*sbk + n*sbn] with BK: sbk == 1 else sbn == 1.
// M, N multiples of 64, K a multiple of 32, contiguous runs 16-byte aligned.
// Workgroup: 64x64 output tile, 4 waves of 32x32, each a 2x2 grid of
// v_mfma_f32_16x16x32_bf16.  Staging: every thread loads one 16-byte vector
// of A and one of B per K step (eight consecutive elements along the
// contiguous dimension) into LDS tiles held K-major ([row][k], 8-element
// pad).  Fragment layout (16x16x32): lane l holds A[row l%16][k 8(l/16)..+7],
// B[k 8(l/16)..+7][col l%16] and returns C[rows 4(l/16)..+3][col l%16].
// Split K: blockIdx.z takes K steps [z kc, (z + 1) kc); with gridDim.z > 1
// only GEMM_STORE is allowed and slice z writes C + z M ldc (partial sums,
// reduced by k_sum_slices).  Slices from `slices` on are those of a second
// product A2 B2 of the same shape.
// Epilogues: STORE C = acc (FP32); FWD z = acc + bias[n] -> C (optional),
// Hout = bf16(silu(z)); BWD Hout = bf16(acc * silu'(Z[m][n])).
// ---------------------------------------------------------------------------
enum { GEMM_STORE = 0, GEMM_FWD = 1, GEMM_BWD = 2 };

template <int EPI, bool AK, bool BK>
__global__ void __launch_bounds__(256) k_gemm_bf16(int M, int N, int K, int kc, const __bf16* __restrict__ A,
                                                   int64_t sam, int64_t sak, const __bf16* __restrict__ B,
                                                   int64_t sbk, int64_t sbn, float* __restrict__ C, int64_t ldc,
                                                   const float* __restrict__ bias, __bf16* __restrict__ Hout,
                                                   int64_t ldh, const float* __restrict__ Z, int64_t ldz,
                                                   const int* __restrict__ status, int64_t rows_per_batch,
                                                   int64_t rbase, int slices, const __bf16* __restrict__ A2,
                                                   const __bf16* __restrict__ B2) {
    __shared__ __attribute__((aligned(16))) __bf16 As[64][40];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[64][40];
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    if (m0 >= M || n0 >= N) return;
    // tiles of finished edges are skipped (rows_per_batch is a multiple of 64)
    if (status && rows_per_batch > 0 && status[(m0 + rbase) / rows_per_batch] >= 0) return;
    const bool second = (int)blockIdx.z >= slices;
    if (second) {
        A = A2;
        B = B2;
    }
    const int kb0 = ((int)blockIdx.z - (second ? slices : 0)) * kc, kb1 = min(K, kb0 + kc);
    if (gridDim.z > 1) C += (int64_t)blockIdx.z * M * ldc;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
    // this thread's staging vector: (row, k) of its eight elements
    const int ar = AK ? (tid >> 2) : ((tid & 7) * 8), ak = AK ? ((tid & 3) * 8) : (tid >> 3);
    const int br = BK ? (tid >> 2) : ((tid & 7) * 8), bk = BK ? ((tid & 3) * 8) : (tid >> 3);
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = kb0; k0 < kb1; k0 += 32) {
        const bf16x8 av = *reinterpret_cast<const bf16x8*>(A + (int64_t)(m0 + ar) * sam + (int64_t)(k0 + ak) * sak);
        const bf16x8 bv = *reinterpret_cast<const bf16x8*>(B + (int64_t)(k0 + bk) * sbk + (int64_t)(n0 + br) * sbn);
        if (AK) {
            *reinterpret_cast<bf16x8*>(&As[ar][ak]) = av;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) As[ar + e][ak] = av[e];
        }
        if (BK) {
            *reinterpret_cast<bf16x8*>(&Bs[br][bk]) = bv;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) Bs[br + e][bk] = bv[e];
        }
        __syncthreads();
        bf16x8 a[2], b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const bf16x8*>(&As[wm + 16 * i + (lane & 15)][8 * (lane >> 4)]);
#pragma unroll
        for (int j = 0; j < 2; ++j) b[j] = *reinterpret_cast<const bf16x8*>(&Bs[wn + 16 * j + (lane & 15)][8 * (lane >> 4)]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
                const int n = n0 + wn + 16 * j + (lane & 15);
                const float v = acc[i][j][r];
                if (EPI == GEMM_STORE) {
                    C[(int64_t)m * ldc + n] = v;
                } else if (EPI == GEMM_FWD) {
                    const float z = v + bias[n];
                    if (C) C[(int64_t)m * ldc + n] = z;
                    Hout[(int64_t)m * ldh + n] = (__bf16)siluf(z);
                } else {
                    Hout[(int64_t)m * ldh + n] = (__bf16)(v * silu_gradf(Z[(int64_t)m * ldz + n]));
                }
            }
}

// out[i] = sum_z part[z n + i] (z < slices), a fixed order: deterministic.
__global__ void __launch_bounds__(256) k_sum_slices(const float* __restrict__ part, int slices, int64_t n,
                                                    float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float s = 0.f;
    for (int z = 0; z < slices; ++z) s += part[(int64_t)z * n + i];
    out[i] = s;
}

// ---------------------------------------------------------------------------
// Training pieces
// ---------------------------------------------------------------------------
// Output layer backward for a batch of B rows with targets t (clipped):
// dy = huber'(y - t) / B;  dz3[r][i] = dy W4[i] silu'(z3[r][i]) (BF16);
// row r's Huber loss to row_loss[r] (summed by k_colsum).
__global__ void __launch_bounds__(256) k_mlp_out_back(int64_t B, int D, int H, const float* __restrict__ P,
                                                      const float* __restrict__ y, const float* __restrict__ t,
                                                      const int* __restrict__ tidx, float huber, float clip_lo,
                                                      float clip_hi, const float* __restrict__ z3,
                                                      float* __restrict__ dy_out, __bf16* __restrict__ dz3,
                                                      float* __restrict__ row_loss) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const MlpOffsets o = mlp_offsets(D, H);
    if (q >= B * H) return;
    const int64_t r = q / H;
    const int i = (int)(q % H);
    const float tv = fminf(fmaxf(t[tidx ? tidx[r] : r], clip_lo), clip_hi);
    const float res = y[r] - tv;
    const float g = (fabsf(res) <= huber ? res : (res > 0.f ? huber : -huber)) / (float)B;
    if (i == 0) {
        dy_out[r] = g;
        row_loss[r] = fabsf(res) <= huber ? 0.5f * res * res : huber * (fabsf(res) - 0.5f * huber);
    }
    dz3[q] = (__bf16)(g * P[o.W4 + i] * silu_gradf(z3[q]));
}

// Single-launch batch reductions.  Every block of a group (blockIdx.x) sums
// one slice of rows (blockIdx.y) into part[slice][...]; then the block that
// finishes last in its group (the counter cnt[group] reaches the number of
// slices) adds the slices in slice order -- deterministic, whichever block
// that is -- and resets the counter: cnt[] is zero before and after a launch.
// Called by every thread after its slice sums are written.
__device__ inline bool last_slice(unsigned* cnt) {
    __shared__ int last;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) {
        last = atomicAdd(&cnt[blockIdx.x], 1u) == gridDim.y - 1 ? 1 : 0;
        if (last) cnt[blockIdx.x] = 0u;       // every block of the group has counted
    }
    __syncthreads();
    if (last) __threadfence();
    return last != 0;
}

// sum over the slices z < gridDim.y of part[z stride + i], in slice order;
// the acquire fence in last_slice makes the other blocks' sums visible to
// these plain loads (issued eight at a time)
__device__ inline float sum_slices_of(const float* part, int64_t stride, int64_t i) {
    float tot = 0.f;
    const int nz = (int)gridDim.y;
    int z = 0;
    for (; z + 8 <= nz; z += 8) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(z + u) * stride + i];
#pragma unroll
        for (int u = 0; u < 8; ++u) tot += v[u];
    }
    for (; z < nz; ++z) tot += part[(int64_t)z * stride + i];
    return tot;
}

// Column sums: out[j] = sum_r w[r] X[r][j] (plus out[j] when accumulate),
// j < ncol, w NULL -> 1, X BF16 [B][ncol] or FP32 Xf.  blockIdx.x = a group
// of 64 columns, blockIdx.y = a slice of kColRows rows, four row groups of
// one wave each summed in a fixed order.
constexpr int kColRows = 256;

__global__ void __launch_bounds__(256) k_colsum(int64_t B, int ncol, const float* __restrict__ w,
                                                const __bf16* __restrict__ X, const float* __restrict__ Xf,
                                                float* __restrict__ part, unsigned* __restrict__ cnt,
                                                float* __restrict__ out, int accumulate) {
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + lane;
    const int64_t r0 = (int64_t)blockIdx.y * kColRows, r1 = min(B, r0 + kColRows);
    float s = 0.f;
    if (j < ncol) {
#pragma unroll 8
        for (int64_t r = r0 + g; r < r1; r += 4) {
            const float x = X ? (float)X[r * ncol + j] : Xf[r * ncol + j];
            s = fmaf(w ? w[r] : 1.f, x, s);
        }
    }
    red[g][lane] = s;
    __syncthreads();
    if (g == 0 && j < ncol)
        part[(int64_t)blockIdx.y * ncol + j] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    if (!last_slice(cnt)) return;
    if (g == 0 && j < ncol) {
        const float tot = sum_slices_of(part, ncol, j);
        out[j] = accumulate ? out[j] + tot : tot;
    }
}

// dW1[i][j] = sum_r dz1[r][i] * x[r][j] / pi -> out[i D + j]: one thread
// per (i, j), blockIdx.y = a slice of rs <= kGradW1Rows rows whose inputs
// (x / pi) the block first gathers into LDS, slices summed as in k_colsum.
constexpr int kGradW1Rows = 64;

__global__ void __launch_bounds__(256) k_mlp_grad_w1(RowSource src, int64_t B, int D, int H, int64_t rs,
                                                     const __bf16* __restrict__ dz1, float* __restrict__ part,
                                                     unsigned* __restrict__ cnt, float* __restrict__ out) {
    __shared__ float xs[kGradW1Rows][kMaxDof];
    const int64_t r0 = (int64_t)blockIdx.y * rs, r1 = min(B, r0 + rs);
    const int nr = (int)(r1 - r0);
    for (int q = threadIdx.x; q < nr * D; q += blockDim.x) {
        const int rr = q / D, j = q % D;
        int64_t sd;
        const float* x = row_ptr(src, r0 + rr, &sd);
        xs[rr][j] = x[j * sd] * kInvPi;
    }
    __syncthreads();
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const bool ok = t < H * D;
    if (ok) {
        const int i = t / D, j = t % D;
        float s = 0.f;
#pragma unroll 8
        for (int r = 0; r < nr; ++r) s = fmaf((float)dz1[(r0 + r) * H + i], xs[r][j], s);
        part[(int64_t)blockIdx.y * H * D + t] = s;
    }
    if (!last_slice(cnt)) return;
    if (ok) out[t] = sum_slices_of(part, (int64_t)H * D, t);
}

// ---------------------------------------------------------------------------
// Forward and backward pass of a batch, H = 64 HB <= 256, in one kernel: a
// workgroup of 4 HB waves takes 16 rows through the three layers as
// k_mlp_predict does (wave w: units 16 w .. + 15) and back, with the layers'
// pre-activations in registers.  The weights, also transposed (W3t, W2t), are
// read from L2 for each tile.  To memory go what the weight gradients of the
// hidden layers contract over the batch, h1, h2, d2, d3 (BF16 [B][H]), and each
// workgroup's sums over its rows of everything else: part[workgroup] =
// dW4[H] db3[H] db2[H] db1[H] dW1[H][D] db4 loss.  x[r] is row idx[r] of q.
// Bound by latency at a batch's size (the weights' way from L2 and six barriers
// a tile): 4096 rows at H = 256 took 260 us of kernels in 19 launches, here 31 us
// in this one and 20 in the contraction and the sums' last step.  Two blocks of
// 16 rows a tile do not fit the 128 registers of 16 waves (83 to 177 spilled); of
// one block, 26 registers a lane go to scratch at H = 256, 17 at 192, 4 at 128.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int train_part_floats(int H, int D) { return 4 * H + H * D + 2; }

template <int HB>
__host__ __device__ constexpr size_t train_lds_bytes() {
    return sizeof(__bf16) * (size_t)2 * 16 * 64 * HB + sizeof(float) * (size_t)16 * (4 * HB + kMaxDof);
}

// sum over the 16 lanes of a row
__device__ __forceinline__ float row_sum16(float v) {
    auto add = [](float x, int b) { return x + __int_as_float(b); };
    v = add(v, __builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
    v = add(v, __builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true));
    v = add(v, __builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, true));
    return add(v, __builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, true));
}

template <int HB>
__global__ void __launch_bounds__(256 * HB, 4)
k_mlp_train(const float* __restrict__ q, const int* __restrict__ idx, int64_t B, int D, const float* __restrict__ P,
            const __bf16* __restrict__ W2b, const __bf16* __restrict__ W3b, const __bf16* __restrict__ W2t,
            const __bf16* __restrict__ W3t, const float* __restrict__ target, float huber, float clip_lo, float clip_hi,
            __bf16* __restrict__ h1, __bf16* __restrict__ h2, __bf16* __restrict__ d2, __bf16* __restrict__ d3,
            float* __restrict__ part) {
    constexpr int H = 64 * HB, KS = H / 32, R = 16, NW = 4 * HB;
    extern __shared__ __attribute__((aligned(16))) __bf16 train_lds[];
    __bf16* const la = train_lds;
    __bf16* const lb = la + R * H;
    float* const red = reinterpret_cast<float*>(lb + R * H);         // [NW][R] partial outputs
    float* const xs = red + NW * R;                                  // [R][kMaxDof] q / pi
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, g = lane >> 4, n0 = 16 * w;
    const MlpOffsets o = mlp_offsets(D, H);
    const int sc = HB % 2 ? c >> 1 : c;                              // as in k_mlp_predict
    auto at = [&](__bf16* h, int chunk) { return h + c * H + 8 * (chunk ^ sc); };
    const int m0 = n0 + 4 * g, wc = m0 >> 3, wo = 4 * (g & 1);       // this lane's units of a result
    f32x4 sw4 = {0.f, 0.f, 0.f, 0.f}, s3 = sw4, s2 = sw4, s1 = sw4, sw1 = sw4;
    float sy = 0.f, sl = 0.f;
    // product of 16 rows of W with the tile's rows
    auto product = [&](__bf16* h, const bf16x8 (&wt)[KS]) {
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KS; ++k)
            z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[k], *reinterpret_cast<const bf16x8*>(at(h, 4 * k + g)), z, 0,
                                                        0, 0);
        return z;
    };
    // (`fresh`, zero, keeps the loads inside the tile loop: all four matrices at
    // once do not fit the registers)
    int fresh = 0;
    auto weights = [&](const __bf16* W, bf16x8 (&wt)[KS]) {
        asm volatile("" : "+s"(fresh));
#pragma unroll
        for (int k = 0; k < KS; ++k) wt[k] = *reinterpret_cast<const bf16x8*>(W + fresh + (n0 + c) * H + 32 * k + 8 * g);
    };
    auto four = [&](int64_t off) {
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = P[off + fresh + m0 + r];
        return v;
    };
    auto put = [&](__bf16* l, __bf16* m, int64_t r0, bf16x4 v) {
        *reinterpret_cast<bf16x4*>(at(l, wc) + wo) = v;
        if (m) *reinterpret_cast<bf16x4*>(m + (r0 + c) * H + m0) = v;
    };
    for (int64_t t = blockIdx.x; t * R < B; t += gridDim.x) {
        const int64_t r0 = t * R;
        bf16x8 wt[KS];
        f32x4 z1, z2, z3;
        __syncthreads();                                             // the tile before is done with LDS
        for (int i = tid; i < R * kMaxDof; i += 64 * NW) {
            const int r = i / kMaxDof, j = i % kMaxDof;
            xs[i] = j < D ? q[(int64_t)idx[r0 + r] * D + j] * kInvPi : 0.f;
        }
        weights(W2b, wt);
        float w1[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) w1[s] = 4 * s + g < D ? P[o.W1 + (n0 + c) * D + 4 * s + g] : 0.f;
        __syncthreads();
        const f32x4 b1 = four(o.b1);
        {
            f32x4 z = b1;
#pragma unroll
            for (int s = 0; s < 2; ++s)
                z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[s], xs[c * kMaxDof + 4 * s + g], z, 0, 0, 0);
            z1 = z;
            put(la, h1, r0, silu4(z));
        }
        const f32x4 b2 = four(o.b2);
        __syncthreads();
        {
            z2 = product(la, wt) + b2;
            put(lb, h2, r0, silu4(z2));
        }
        weights(W3b, wt);
        const f32x4 b3 = four(o.b3), w4 = four(o.W4);
        __syncthreads();
        bf16x4 h3;
        {
            z3 = product(lb, wt) + b3;
            h3 = silu4(z3);
            float s = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) s = fmaf(w4[r], (float)h3[r], s);
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (g == 0) red[w * R + c] = s;
        }
        weights(W3t, wt);
        __syncthreads();
        {
            float y = P[o.b4];
#pragma unroll
            for (int v = 0; v < NW; ++v) y += red[v * R + c];
            const float tv = fminf(fmaxf(target[idx[r0 + c]], clip_lo), clip_hi);
            const float res = y - tv;
            const float dy = (fabsf(res) <= huber ? res : (res > 0.f ? huber : -huber)) / (float)B;
            if (w == 0 && g == 0) {
                sy += dy;
                sl += fabsf(res) <= huber ? 0.5f * res * res : huber * (fabsf(res) - 0.5f * huber);
            }
            bf16x4 d;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                d[r] = (__bf16)(dy * w4[r] * silu_gradf(z3[r]));
                s3[r] += (float)d[r];
                sw4[r] = fmaf(dy, (float)h3[r], sw4[r]);
            }
            put(la, d3, r0, d);
        }
        __syncthreads();
        {
            const f32x4 v = product(la, wt);
            bf16x4 d;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                d[r] = (__bf16)(v[r] * silu_gradf(z2[r]));
                s2[r] += (float)d[r];
            }
            put(lb, d2, r0, d);
        }
        weights(W2t, wt);
        __syncthreads();
        {
            const f32x4 v = product(lb, wt);
            bf16x4 d;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                d[r] = (__bf16)(v[r] * silu_gradf(z1[r]));
                s1[r] += (float)d[r];
            }
            put(la, nullptr, r0, d);                             // read back by this wave only, by other lanes
        }
        wave_lds_sync();
        // dW1: this wave's units against the inputs, the rows as K
#pragma unroll
        for (int k = 0; k < R / 4; ++k) {
            const int row = 4 * k + g, rc = row & 15, unit = n0 + c;
            const float a = (float)la[row * H + 8 * ((unit >> 3) ^ (HB % 2 ? rc >> 1 : rc)) + (unit & 7)];
            sw1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a, c < kMaxDof ? xs[row * kMaxDof + (c & 7)] : 0.f, sw1, 0, 0, 0);
        }
    }
    float* const out = part + (int64_t)blockIdx.x * train_part_floats(H, D);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float a = row_sum16(sw4[r]), b = row_sum16(s3[r]), d = row_sum16(s2[r]), e = row_sum16(s1[r]);
        if (c == 0) {
            out[m0 + r] = a;
            out[H + m0 + r] = b;
            out[2 * H + m0 + r] = d;
            out[3 * H + m0 + r] = e;
        }
        if (c < D) out[4 * H + (m0 + r) * D + c] = sw1[r];
    }
    sy = row_sum16(sy);
    sl = row_sum16(sl);
    if (tid == 0) {
        out[4 * H + H * D] = sy;
        out[4 * H + H * D + 1] = sl;
    }
}

// The gradient from k_mlp_train's sums (part[groups][train_part_floats]) and the
// K slices of the hidden layers' products (w: slices of dW3, then of dW2):
// blocks below `nb` take 64 of the sums' columns each, four of their rows side
// by side, the others 256 elements of the products.  Fixed order: deterministic.
__global__ void __launch_bounds__(256) k_mlp_grad_sum(int D, int H, int groups, const float* __restrict__ part,
                                                      int slices, const float* __restrict__ w, int nb,
                                                      float* __restrict__ G, float* __restrict__ loss) {
    const MlpOffsets o = mlp_offsets(D, H);
    const int tid = threadIdx.x, n = train_part_floats(H, D);
    if ((int)blockIdx.x >= nb) {
        const int64_t HH = (int64_t)H * H, i = (int64_t)(blockIdx.x - nb) * 256 + tid;
        if (i >= 2 * HH) return;
        const float* p = w + (i < HH ? 0 : slices * HH) + i % HH;
        float s = 0.f;
        for (int z = 0; z < slices; ++z) s += p[z * HH];
        G[(i < HH ? o.W3 : o.W2) + i % HH] = s;
        return;
    }
    __shared__ float red[4][64];
    const int lane = tid & 63, g = tid >> 6, j = blockIdx.x * 64 + lane;
    float s = 0.f;
    if (j < n) {
#pragma unroll 8
        for (int r = g; r < groups; r += 4) s += part[(int64_t)r * n + j];
    }
    red[g][lane] = s;
    __syncthreads();
    if (g != 0 || j >= n) return;
    s = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    if (j < H) G[o.W4 + j] = s;
    else if (j < 2 * H) G[o.b3 + j - H] = s;
    else if (j < 3 * H) G[o.b2 + j - 2 * H] = s;
    else if (j < 4 * H) G[o.b1 + j - 3 * H] = s;
    else if (j < 4 * H + H * D) G[o.W1 + j - 4 * H] = s;
    else if (j == 4 * H + H * D) G[o.b4] = s;
    else *loss += s;
}

// Adam step with bias correction on the flat parameter vector; refreshes
// the BF16 copies of W2 and W3 (and their transposes where kept).
__global__ void __launch_bounds__(256) k_adam(int64_t n, float* __restrict__ P, const float* __restrict__ G,
                                              float* __restrict__ m, float* __restrict__ v, float lr, float b1,
                                              float b2, float eps, float c1, float c2, int D, int H,
                                              __bf16* __restrict__ W2b, __bf16* __restrict__ W3b,
                                              __bf16* __restrict__ W2t, __bf16* __restrict__ W3t) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const float g = G[k];
    const float mk = b1 * m[k] + (1.f - b1) * g;
    const float vk = b2 * v[k] + (1.f - b2) * g * g;
    m[k] = mk;
    v[k] = vk;
    const float p = P[k] - lr * (mk / c1) / (sqrtf(vk / c2) + eps);
    P[k] = p;
    const MlpOffsets o = mlp_offsets(D, H);
    const bool second = k >= o.W3;
    const int64_t w = k - (second ? o.W3 : o.W2);
    if (w >= 0 && w < (int64_t)H * H) {
        (second ? W3b : W2b)[w] = (__bf16)p;
        __bf16* const t = second ? W3t : W2t;
        if (t) t[w % H * H + w / H] = (__bf16)p;
    }
}

// BF16 copies of W2, W3 from the master parameters.
__global__ void __launch_bounds__(256) k_mlp_cast(int D, int H, const float* __restrict__ P, __bf16* __restrict__ W2b,
                                                  __bf16* __restrict__ W3b, __bf16* __restrict__ W2t,
                                                  __bf16* __restrict__ W3t) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const MlpOffsets o = mlp_offsets(D, H);
    if (k >= (int64_t)H * H) return;
    W2b[k] = (__bf16)P[o.W2 + k];
    W3b[k] = (__bf16)P[o.W3 + k];
    if (W2t) {
        W2t[k % H * H + k / H] = W2b[k];
        W3t[k % H * H + k / H] = W3b[k];
    }
}

__global__ void __launch_bounds__(256) k_fill(float* __restrict__ p, int64_t n, float v) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) p[k] = v;
}

// Counts of {pred >= m} among configurations with target < 0, for a set of
// candidate margins (calibration by bisection on the host).
__global__ void __launch_bounds__(256) k_count_above(int64_t n, const float* __restrict__ pred,
                                                     const float* __restrict__ target, float m,
                                                     unsigned long long* __restrict__ out) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool colliding = r < n && target[r] < 0.f;
    const bool above = colliding && pred[r] >= m;
    const unsigned long long a = __ballot(above), c = __ballot(colliding);
    if ((threadIdx.x & 63) == 0) {
        if (a) atomicAdd(&out[0], (unsigned long long)__popcll(a));
        if (c) atomicAdd(&out[1], (unsigned long long)__popcll(c));
    }
}

}  // namespace ezo
