// mlp_kernels.hip -- kernels of the learned surrogate (gfx950).
//
// The surrogate is a multilayer perceptron 66 -> 512 -> 512 -> 512 -> 2806
// with GELU activations that predicts a coarse 61 x 46 map of a frame: for
// each 20 cm cell, the best exact score among the 5 cm points that a
// re-score of that cell visits.  Its top-64 cells are then re-scored exactly
// at 5 cm.  Weights and
// activations are bfloat16, products accumulate in float32 on the matrix
// cores (v_mfma_f32_16x16x32_bf16); biases, pre-activations, gradients and
// the Adam state are float32.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>

#include "mlp_internal.h"

namespace dpps {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// round to nearest even
__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)((u >> 16) | ((u & 0xFFFFu) ? 0x40u : 0u));
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

__device__ __forceinline__ float gelu_grad(float x)
{
    float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
    float pdf = 0.39894228040143268f * expf(-0.5f * x * x);
    return cdf + x * pdf;
}

// ---------------------------------------------------------------------------
// GEMM: C[M][N] = sum_k A(m, k) B(k, n), bf16 operands, f32 accumulation.
// A(m, k) = A[m*lda + k] when A_K (k contiguous), else A[k*lda + m].
// B(k, n) = B[n*ldb + k] when B_K (k contiguous), else B[k*ldb + n].
// M, N are multiples of 8, K and every K slice multiples of 32.
// Block tile BM x BN (128 x 64 or 64 x 64), K step 64, 256 threads: four
// waves in a 2 x 2 arrangement, each owning a (BM/2) x (BN/2) quarter as
// (BM/32) x (BN/32) MFMA tiles of 16 x 16 (v_mfma_f32_16x16x32_bf16, k
// ascending from 0, so an output element has the same bits whatever the tile).
// The layers are narrow (K = 512 mostly, a few hundred tiles): what bounds
// them is the latency of a K step, not MFMA issue, so a step is 64 deep, goes
// from memory straight into LDS (no registers, no LDS write pass), and the
// next one is in flight while the current one multiplies.  An operand
// that is not k-contiguous (the weight gradients) stays as it lies in memory
// and is transposed by the LDS reads (ds_read_b64_tr_b16).  16-byte chunks
// are permuted within LDS so that a read's lanes spread over the banks.
// K may be split into slices of g.k_slice; with EPI_PARTIAL slice z writes its
// partial product to Cf + z * M * ldc (summed by gemm_reduce).  (Four buffers
// instead of two gained nothing: the waits before LDS reads are not told
// apart by buffer, and two leave room for five workgroups a CU.)
// ---------------------------------------------------------------------------
#define GK 64

// Chunk permutation of row r of an operand tile (BX rows or columns).
// k-contiguous rows are 128 bytes: 8 lanes read the same chunk of 8 rows.
__device__ __forceinline__ int swz_k(int r) { return r & 7; }
// Otherwise row = k: a transposing read takes 32 bytes of rows r0 .. r0 + 3,
// r0 = 8 g for the wave's four groups of 16 lanes.
template <int BX>
__device__ __forceinline__ int swz_x(int r)
{
    return BX == 128 ? (((r & 3) | (((r >> 3) & 1) << 2)) << 1)
                     : ((((r >> 1) & 1) | (((r >> 3) & 1) << 1)) << 1);
}

// One K step of an operand into its LDS tile: each wave instruction moves 64
// chunks of 16 bytes to consecutive LDS addresses; the lane chooses which
// chunk of the matrix lands on its place.  Rows, columns and k past the edge
// are clamped to valid ones (their products are not used).
template <int BX, bool X_K>
__device__ __forceinline__ void load_tile(const uint16_t *__restrict__ src, int ld, int X, int K,
                                          int x0, int k0, uint16_t *tile)
{
    constexpr int CR = X_K ? GK / 8 : BX / 8;  // chunks per LDS row
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int i = 0; i < BX * GK * 2 / 4096; ++i) {
        const int n = i * 4 + w;
        const int row = n * (64 / CR) + l / CR, phys = l % CR;
        const uint16_t *p;
        if (X_K) {
            const int k = min(k0 + (phys ^ swz_k(row)) * 8, K - 8);
            p = src + (size_t)min(x0 + row, X - 1) * ld + k;
        } else {
            const int x = min(x0 + (phys ^ swz_x<BX>(row)) * 8, X - 8);
            p = src + (size_t)min(k0 + row, K - 1) * ld + x;
        }
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void *)p,
            (__attribute__((address_space(3))) void *)(tile + n * 512), 16, 0, 0);
    }
}

// MFMA operand of 16 rows (columns) from x and the 32 k of half kk of the step:
// lane l holds row x + l % 16, k = 32 kk + 8 (l / 16) .. + 7.
template <int BX, bool X_K>
__device__ __forceinline__ bf16x8_t load_frag(const uint16_t *tile, int x, int kk)
{
    const int l = threadIdx.x & 63;
    if (X_K) {
        const int row = x + (l & 15);
        const int phys = (kk * 4 + (l >> 4)) ^ swz_k(row);
        return *(const bf16x8_t *)(tile + row * GK + phys * 8);
    }
    const int row = kk * 32 + (l >> 4) * 8 + ((l & 15) >> 2);
    const int col = x + (l & 3) * 4;
    const uint16_t *p = tile + row * BX + (((col >> 3) ^ swz_x<BX>(row)) * 8 + (col & 4));
    typedef __attribute__((ext_vector_type(4))) short s16x4_t;
    typedef __attribute__((address_space(3))) s16x4_t *lds_t;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)p);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(p + 4 * BX));
    typedef __attribute__((ext_vector_type(8))) short s16x8_t;
    return __builtin_bit_cast(bf16x8_t, (s16x8_t)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Four consecutive outputs from column n of row m (m < M, n + 3 < N).
template <int EPI>
__device__ __forceinline__ void gemm_store(const GemmArgs &g, float *part, int m, int n, f32x4_t v)
{
    const size_t o = (size_t)m * g.ldc + n;
    if (EPI == EPI_BIAS_GELU || EPI == EPI_BIAS) v = v + *(const f32x4_t *)(g.bias + n);
    if (EPI == EPI_BIAS_GELU || EPI == EPI_GELU_GRAD) {
        float z[4] = {v[0], v[1], v[2], v[3]};
        f32x4_t zin = v;
        if (EPI == EPI_GELU_GRAD) zin = *(const f32x4_t *)(g.Zin + o);
        uint16_t h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            h[i] = EPI == EPI_BIAS_GELU ? f2bf(gelu(z[i])) : f2bf(z[i] * gelu_grad(zin[i]));
        if (EPI == EPI_BIAS_GELU && g.Cf) *(f32x4_t *)(g.Cf + o) = v;  // pre-activation
        *(uint2 *)(g.Cb + o) = make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16),
                                          (uint32_t)h[2] | ((uint32_t)h[3] << 16));
        return;
    }
    *(f32x4_t *)((EPI == EPI_PARTIAL ? part : g.Cf) + o) = v;
    if (EPI == EPI_BIAS && g.out && m < g.out_m) {  // the caller's copy, real columns only
        float *p = g.out + (size_t)m * g.ld_out + n;
        if (n + 4 <= g.out_n) {
            __builtin_memcpy(p, &v, sizeof v);
        } else {
            for (int i = 0; i < g.out_n - n; ++i) p[i] = v[i];
        }
    }
}

// LDS of a workgroup: two buffers of each operand.
constexpr int gemm_lds(int BM, int BN) { return 2 * (BM + BN) * GK; }

// Output tile `id` of the (gx column tiles) x (gy row tiles) x (gz K slices) of
// a product.
template <int BM, int BN, bool A_K, bool B_K, int EPI>
__device__ __forceinline__ void gemm_block(const GemmArgs &g, int id, int gx, int gy, int gz,
                                           uint16_t *lds)
{
    constexpr int TM = BM / 32, TN = BN / 32;
    uint16_t *const As = lds, *const Bs = lds + 2 * BM * GK;
    // Workgroups go to the 8 XCDs in turn, each with its own L2: the column
    // tiles of one panel (the rows of a tile, one K slice) are given to one
    // XCD, so that a panel of A is read from memory once and not by all eight.
    int panel = id / gx, n_tile = id % gx;
    const int even = gy * gz / 8 * 8;
    if (id < even * gx) {
        panel = (id / 8) / gx * 8 + id % 8;
        n_tile = (id / 8) % gx;
    }
    const int z = panel / gy;
    const int m0 = (panel - z * gy) * BM, n0 = n_tile * BN;
    const int kb = z * g.k_slice;
    const int ke = min(kb + g.k_slice, g.K);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int wm = (w >> 1) * (BM / 2), wn = (w & 1) * (BN / 2);
    f32x4_t acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    load_tile<BM, A_K>(g.A, g.lda, g.M, g.K, m0, kb, As);
    load_tile<BN, B_K>(g.B, g.ldb, g.N, g.K, n0, kb, Bs);
    int cur = 0;
    for (int k0 = kb; k0 < ke; k0 += GK, cur ^= 1) {
        // this wave's part of the step has landed; after the barrier all of
        // it has, and every wave is done with the other buffer
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const uint16_t *const ta = As + cur * BM * GK, *const tb = Bs + cur * BN * GK;
        bf16x8_t af[2][TM], bfr[2][TN];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
            for (int a = 0; a < TM; ++a) af[kk][a] = load_frag<BM, A_K>(ta, wm + a * 16, kk);
#pragma unroll
            for (int b = 0; b < TN; ++b) bfr[kk][b] = load_frag<BN, B_K>(tb, wn + b * 16, kk);
        }
        if (k0 + GK < ke) {
            load_tile<BM, A_K>(g.A, g.lda, g.M, g.K, m0, k0 + GK, As + (cur ^ 1) * BM * GK);
            load_tile<BN, B_K>(g.B, g.ldb, g.N, g.K, n0, k0 + GK, Bs + (cur ^ 1) * BN * GK);
        }
        // operands swapped: the lane then holds four consecutive columns n of
        // one row m
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            if (kk == 1 && k0 + 32 >= ke) break;  // a last half step
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[kk][b], af[kk][a],
                                                                        acc[a][b], 0, 0, 0);
        }
    }
    float *part = g.Cf + (size_t)z * g.M * g.ldc;
#pragma unroll
    for (int a = 0; a < TM; ++a) {
        const int m = m0 + wm + a * 16 + (l & 15);
        if (m >= g.M) continue;
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            const int n = n0 + wn + b * 16 + (l >> 4) * 4;
            if (n < g.N) gemm_store<EPI>(g, part, m, n, acc[a][b]);
        }
    }
}

template <int BM, int BN, bool A_K, bool B_K, int EPI>
__global__ void __launch_bounds__(256) gemm_kernel(GemmArgs g, int gx, int gy, int gz)
{
    __shared__ __attribute__((aligned(16))) uint16_t lds[gemm_lds(BM, BN)];
    gemm_block<BM, BN, A_K, B_K, EPI>(g, blockIdx.x, gx, gy, gz, lds);
}

// The two products of a backward layer that need only its output gradient, in
// one launch: blocks below nx form the input gradient's tiles (few, with long
// reductions), the others the weight gradient's (split reductions).  Alone
// the former leave most of the chip idle.
__global__ void __launch_bounds__(256) gemm_backward_kernel(GemmArgs gx, GemmArgs gw, int nx,
                                                            int xgx, int xgy, int wgx, int wgy,
                                                            int wgz)
{
    __shared__ __attribute__((aligned(16))) uint16_t lds[gemm_lds(64, 64)];
    if ((int)blockIdx.x < nx)
        gemm_block<64, 64, true, false, EPI_GELU_GRAD>(gx, blockIdx.x, xgx, xgy, 1, lds);
    else
        gemm_block<64, 64, false, false, EPI_PARTIAL>(gw, (int)blockIdx.x - nx, wgx, wgy, wgz, lds);
}

// out[e] = sum over z of part[z][e], in order of z; four elements per thread,
// the slices' loads in flight together.
__global__ void __launch_bounds__(256) gemm_reduce_kernel(const f32x4_t *__restrict__ part,
                                                          int splits, int64_t n4,
                                                          f32x4_t *__restrict__ out)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n4) return;
    f32x4_t s = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int z0 = 0; z0 < splits; z0 += 8) {
        f32x4_t v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (z0 + q < splits) v[q] = part[(size_t)(z0 + q) * n4 + e];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (z0 + q < splits) s = s + v[q];
    }
    out[e] = s;
}

template <int BM, int BN, bool A_K, bool B_K, int EPI>
static void launch_gemm(const GemmArgs &g, int splits, hipStream_t st)
{
    const int gx = (g.N + BN - 1) / BN, gy = (g.M + BM - 1) / BM;
    hipLaunchKernelGGL((gemm_kernel<BM, BN, A_K, B_K, EPI>), dim3(gx * gy * splits), dim3(256), 0, st,
                       g, gx, gy, splits);
}

// Tiles of 64 x 64, or 128 x 64 where that still gives every CU two: the layer
// 4096 x 2816 x 512 takes 25 us with 128 x 64, 29 with 128 x 128 or 64 x 64.
template <bool A_K, bool B_K, int EPI>
static void launch_shape(GemmArgs g, hipStream_t st)
{
    g.k_slice = g.K;
    const int64_t t = (int64_t)((g.M + 127) / 128) * ((g.N + 63) / 64);
    if (t >= 512)
        launch_gemm<128, 64, A_K, B_K, EPI>(g, 1, st);
    else
        launch_gemm<64, 64, A_K, B_K, EPI>(g, 1, st);
}

int gemm_backward(const GemmArgs *x, const GemmArgs &w, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    if ((w.M | w.N) & 7 || w.K & 31 || w.M < 8 || w.N < 8 || w.K < 32 || !w.work) return -1;
    if (x && ((x->M | x->N) & 7 || x->K & 31 || x->M < 8 || x->N < 8 || x->K < 32)) return -1;
    // the weight gradient has few output tiles and a long reduction (the
    // batch): split K into slices of a multiple of 32, partial products into
    // the workspace, then a fixed-order sum
    GemmArgs h = w;
    const int wgx = (w.N + 63) / 64, wgy = (w.M + 63) / 64;
    const int64_t t64 = (int64_t)wgx * wgy, mn = (int64_t)w.M * w.ldc;
    int splits = 1;
    if (t64 < 512 && w.K >= 1024) splits = std::min((int)((512 + t64 - 1) / t64), w.K / 256);
    while (splits > 1 && (int64_t)splits * mn > w.work_elems) --splits;
    h.k_slice = splits > 1 ? ((w.K + splits - 1) / splits + 31) / 32 * 32 : w.K;
    splits = (w.K + h.k_slice - 1) / h.k_slice;
    h.Cf = splits > 1 ? w.work : w.Cf;
    const int nw = wgx * wgy * splits;
    if (x) {
        GemmArgs g = *x;
        g.k_slice = g.K;
        const int xgx = (g.N + 63) / 64, xgy = (g.M + 63) / 64;
        hipLaunchKernelGGL(gemm_backward_kernel, dim3(xgx * xgy + nw), dim3(256), 0, st, g, h,
                           xgx * xgy, xgx, xgy, wgx, wgy, splits);
    } else {
        hipLaunchKernelGGL((gemm_kernel<64, 64, false, false, EPI_PARTIAL>), dim3(nw), dim3(256), 0,
                           st, h, wgx, wgy, splits);
    }
    if (splits > 1)
        hipLaunchKernelGGL(gemm_reduce_kernel, dim3((unsigned)((mn / 4 + 255) / 256)), dim3(256), 0,
                           st, (const f32x4_t *)w.work, splits, mn / 4, (f32x4_t *)w.Cf);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Few-row GEMM for inference on small batches (A and B k-contiguous): one
// wave per 16 x 16 output tile, operands loaded straight from global memory,
// the same v_mfma_f32_16x16x32_bf16 sequence over K (K steps of 32 from 0,
// zero-filled past K) and the same epilogue as gemm_kernel, so each output
// element is computed exactly as gemm_kernel computes it.
#define ROWS_KSTEPS 16   // K <= 512 for the few-row GEMM

template <int EPI>
__global__ void __launch_bounds__(64) gemm_rows_kernel(GemmArgs g)
{
    const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
    const int l = threadIdx.x;
    const int fr = l & 15, fk = (l >> 4) * 8;
    const bool arow = m0 + fr < g.M, brow = n0 + fr < g.N;
    const uint16_t *pa = g.A + (size_t)(m0 + fr) * g.lda + fk;
    const uint16_t *pb = g.B + (size_t)(n0 + fr) * g.ldb + fk;
    // every K step's operands are loaded before the first product
    uint4 va[ROWS_KSTEPS], vb[ROWS_KSTEPS];
#pragma unroll
    for (int s = 0; s < ROWS_KSTEPS; ++s) {
        const int k0 = s * 32;
        const bool kin = k0 + fk < g.K;
        va[s] = make_uint4(0, 0, 0, 0);
        vb[s] = make_uint4(0, 0, 0, 0);
        if (arow && kin) va[s] = *(const uint4 *)(pa + k0);
        if (brow && kin) vb[s] = *(const uint4 *)(pb + k0);
    }
    f32x4_t acc = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < ROWS_KSTEPS; ++s)
        if (s * 32 < g.K)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, va[s]),
                                                          __builtin_bit_cast(bf16x8_t, vb[s]), acc,
                                                          0, 0, 0);
    const int n = n0 + (l & 15);
    if (n >= g.N) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + (l >> 4) * 4 + i;
        if (m >= g.M) continue;
        const float v = acc[i];
        const size_t o = (size_t)m * g.ldc + n;
        if (EPI == EPI_BIAS_GELU) {
            const float z = v + g.bias[n];
            if (g.Cf) g.Cf[o] = z;
            g.Cb[o] = f2bf(gelu(z));
        } else {
            const float z = v + g.bias[n];
            g.Cf[o] = z;
            if (g.out && m < g.out_m && n < g.out_n) g.out[(size_t)m * g.ld_out + n] = z;
        }
    }
}

int gemm_rows(const GemmArgs &g, int epi, void *stream)
{
    if ((g.M | g.N | g.K) & 7 || g.M < 1 || g.K > ROWS_KSTEPS * 32) return -1;
    const dim3 grid((unsigned)((g.N + 15) / 16), (unsigned)((g.M + 15) / 16));
    if (epi == EPI_BIAS_GELU)
        hipLaunchKernelGGL(gemm_rows_kernel<EPI_BIAS_GELU>, grid, dim3(64), 0, (hipStream_t)stream, g);
    else if (epi == EPI_BIAS)
        hipLaunchKernelGGL(gemm_rows_kernel<EPI_BIAS>, grid, dim3(64), 0, (hipStream_t)stream, g);
    else
        return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int gemm(const GemmArgs &g, int epi, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    if ((g.M | g.N) & 7 || g.K & 31 || g.M < 8 || g.N < 8 || g.K < 32) return -1;
    if (epi == EPI_BIAS)
        launch_shape<true, true, EPI_BIAS>(g, st);
    else if (epi == EPI_BIAS_GELU)
        launch_shape<true, true, EPI_BIAS_GELU>(g, st);
    else
        return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ---------------------------------------------------------------------------
// elementwise and reduction kernels
// ---------------------------------------------------------------------------

// Column sums of every layer's dz [M][N] (bias gradients), in two deterministic
// passes over one job list: block (x, y) sums rows [y * COLSUM_ROWS, (y + 1) *
// COLSUM_ROWS) of 256 columns of one layer (lanes = 4 columns, four row phases,
// each phase's 32 loads in flight together, combined in a fixed order) into
// part[y][n]; then each column adds its chunks in order.  One launch per pass
// for all layers: 12 us for what took 8 launches of 8 to 9 us each.
#define COLSUM_ROWS 128
__device__ __forceinline__ int colsum_job(const ColsumJobs &jobs, int cols, int &x)
{
    int j = 0;
    while (j < 3 && x >= jobs.n[j] / cols) x -= jobs.n[j++] / cols;
    return j;
}

__global__ void __launch_bounds__(256) colsum_part_kernel(ColsumJobs jobs, int M)
{
    __shared__ f32x4_t red[4][64];
    int x = blockIdx.x;
    const int j = colsum_job(jobs, 256, x);
    const int c = threadIdx.x & 63, r = threadIdx.x >> 6;
    const int n = x * 256 + 4 * c, N = jobs.n[j];
    const int m0 = blockIdx.y * COLSUM_ROWS;
    const uint16_t *p = jobs.dz[j] + (size_t)(m0 + r) * N + n;
    uint2 v[COLSUM_ROWS / 4];
#pragma unroll
    for (int i = 0; i < COLSUM_ROWS / 4; ++i)
        v[i] = m0 + r + 4 * i < M ? *(const uint2 *)(p + (size_t)(4 * i) * N) : make_uint2(0u, 0u);
    f32x4_t s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < COLSUM_ROWS / 4; ++i) {
        s[0] += bf2f((uint16_t)v[i].x);
        s[1] += bf2f((uint16_t)(v[i].x >> 16));
        s[2] += bf2f((uint16_t)v[i].y);
        s[3] += bf2f((uint16_t)(v[i].y >> 16));
    }
    red[r][c] = s;
    __syncthreads();
    if (r == 0)
        *(f32x4_t *)(jobs.part[j] + (size_t)blockIdx.y * N + n) =
            ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
}

__global__ void __launch_bounds__(64) colsum_final_kernel(ColsumJobs jobs, int chunks)
{
    int x = blockIdx.x;
    const int j = colsum_job(jobs, 64, x);
    const int n = x * 64 + threadIdx.x, N = jobs.n[j];
    float s = 0.0f;
    for (int k0 = 0; k0 < chunks; k0 += 16) {
        float v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q)
            v[q] = k0 + q < chunks ? jobs.part[j][(size_t)(k0 + q) * N + n] : 0.0f;
#pragma unroll
        for (int q = 0; q < 16; ++q)
            if (k0 + q < chunks) s += v[q];
    }
    jobs.db[j][n] = s;
}

// Sums or maxima of NV values over the 256 threads of a block, on every thread:
// the tree v[t] + v[t + 128], then + 64, 32, ... 1, the last six steps by lane
// reads in every wave alike (one barrier; red is free again after the next
// one).
template <int NV, bool MAX>
__device__ __forceinline__ void block_reduce(float (&v)[NV], float (*red)[256])
{
#pragma unroll
    for (int i = 0; i < NV; ++i) red[i][threadIdx.x] = v[i];
    __syncthreads();
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const float a = red[i][l], b = red[i][l + 64], c = red[i][l + 128], d = red[i][l + 192];
        float x = MAX ? fmaxf(fmaxf(a, c), fmaxf(b, d)) : (a + c) + (b + d);
#pragma unroll
        for (int s = 32; s > 0; s >>= 1) {
            const float y = __shfl_down(x, s, 64);
            x = MAX ? fmaxf(x, y) : x + y;
        }
        v[i] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
    }
}

// Training loss of one row (one block per row, 256 threads):
//   sum_c w_c (y_c - t_c)^2 / (rows * outs)        weighted squared error,
//   + ce_weight * CE(softmax(t / tau) || softmax(y / tau)) / rows
// Targets are score maps with infeasible cells (-inf): read as 0 in the
// squared error, excluded from the target distribution of the cross-entropy
// (which ranks the best cells first).  w_c = 1 + pos_weight * t_c.  Writes
// dZ as bf16 (zero in padding) and, per row, the squared-error sum and the
// cross-entropy.  Bound by memory (4096 rows: 92 MB read, 23 written): a
// thread keeps its cells of the row in registers, so predictions and targets
// are read once instead of three times, the target exponentials serve the
// sum and the distribution, and three block reductions take one barrier
// each instead of six with nine.
constexpr int LOSS_PER = TOPK_SORT / 256;  // cells per thread, at most
__global__ void __launch_bounds__(256) loss_kernel(const float *__restrict__ y, int ldy,
                                                   const float *__restrict__ tgt, int ldt, int rows,
                                                   int outs, int rows_pad, int outs_pad,
                                                   float pos_weight, float ce_weight, float tau,
                                                   uint16_t *__restrict__ dz,
                                                   float *__restrict__ partial)
{
    __shared__ float red[3][2][256];
    const int r = blockIdx.x, t0 = threadIdx.x;
    const bool real = r < rows;
    const float itau = 1.0f / tau;
    float yv[LOSS_PER], tv[LOSS_PER], et[LOSS_PER];
    float mx[2] = {-INFINITY, -INFINITY};
#pragma unroll
    for (int i = 0; i < LOSS_PER; ++i) {
        const int n = t0 + 256 * i;
        yv[i] = 0.0f;
        tv[i] = -INFINITY;
        if (real && n < outs) {
            yv[i] = y[(size_t)r * ldy + n];
            tv[i] = tgt[(size_t)r * ldt + n];
        }
    }
    if (real && ce_weight > 0.0f) {
#pragma unroll
        for (int i = 0; i < LOSS_PER; ++i)
            if (t0 + 256 * i < outs) {
                mx[0] = fmaxf(mx[0], yv[i] * itau);
                if (tv[i] > -INFINITY) mx[1] = fmaxf(mx[1], tv[i] * itau);
            }
    }
    block_reduce<2, true>(mx, red[0]);
    const float my = mx[0], mt = mx[1];
    const bool ce = real && ce_weight > 0.0f && mt > -INFINITY;
    float sm[2] = {0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < LOSS_PER; ++i) {
        et[i] = 0.0f;
        if (ce && t0 + 256 * i < outs) {
            sm[0] += expf(yv[i] * itau - my);
            if (tv[i] > -INFINITY) {
                et[i] = expf(tv[i] * itau - mt);
                sm[1] += et[i];
            }
        }
    }
    block_reduce<2, false>(sm, red[1]);
    const float st = sm[1];
    const float lsy = ce ? logf(sm[0]) : 0.0f;
    const float scale = 2.0f / ((float)rows * (float)outs);
    const float cscale = ce_weight * itau / (float)rows;
    float ae[2] = {0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < LOSS_PER; ++i) {
        const int n = t0 + 256 * i;
        if (n >= outs_pad) break;
        float g = 0.0f;
        if (real && n < outs) {
            const float t = tv[i] > -INFINITY ? tv[i] : 0.0f;
            const float wgt = 1.0f + pos_weight * t;
            const float d = yv[i] - t;
            ae[0] += wgt * d * d;
            g = scale * wgt * d;
            if (ce) {
                const float lp = yv[i] * itau - my - lsy;
                const float p = expf(lp);
                const float q = tv[i] > -INFINITY ? et[i] / st : 0.0f;
                ae[1] -= q * lp;
                g += cscale * (p - q);
            }
        }
        dz[(size_t)r * outs_pad + n] = f2bf(g);
    }
    block_reduce<2, false>(ae, red[2]);
    if (threadIdx.x == 0 && r < rows_pad) {
        partial[2 * r] = ae[0];
        partial[2 * r + 1] = ae[1];
    }
}

// Coarse-cell labels from a fine score map (one thread per coarse cell):
// cell (ci, cj) takes the largest score of the fine points
// {4 ci - 2 .. 4 ci + 1} x {4 cj - 2 .. 4 cj + 1} inside the fine lattice
// (the points a re-score of that cell would visit); -inf if none is feasible.
__global__ void pool_kernel(const float *__restrict__ fine, int n_frames, int fnx, int fny,
                            float *__restrict__ coarse, int cnx, int cny)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t per = (int64_t)cnx * cny;
    if (i >= per * n_frames) return;
    const int f = (int)(i / per);
    const int c = (int)(i - (int64_t)f * per);
    const int ci = c % cnx, cj = c / cnx;
    const float *src = fine + (size_t)f * fnx * fny;
    float m = -INFINITY;
    for (int J = max(4 * cj - 2, 0); J <= min(4 * cj + 1, fny - 1); ++J)
        for (int I = max(4 * ci - 2, 0); I <= min(4 * ci + 1, fnx - 1); ++I)
            m = fmaxf(m, src[(size_t)J * fnx + I]);
    coarse[i] = m;
}

// Adam on every parameter tensor (f32 master) of the job list, four elements
// per thread, refreshing the weights' bf16 copies.  Bound by memory (28 + 2
// bytes per parameter, 60 MB); one launch instead of eight.
__global__ void __launch_bounds__(256) adam_kernel(AdamJobs jobs, float lr, float b1, float b2,
                                                   float eps, float c1, float c2)
{
    int x = blockIdx.x, j = 0;
    while (j < ADAM_JOBS - 1 && x >= jobs.blocks[j]) x -= jobs.blocks[j++];
    const AdamJob J = jobs.job[j];
    const int64_t i = ((int64_t)x * 256 + threadIdx.x) * 4;
    if (i >= J.n) return;
    f32x4_t w = *(const f32x4_t *)(J.w + i), m = *(const f32x4_t *)(J.m + i);
    f32x4_t v = *(const f32x4_t *)(J.v + i);
    const f32x4_t g = *(const f32x4_t *)(J.g + i);
    uint16_t h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float gi = g[q] + J.wd * w[q];
        const float mi = b1 * m[q] + (1.0f - b1) * gi;
        const float vi = b2 * v[q] + (1.0f - b2) * gi * gi;
        m[q] = mi;
        v[q] = vi;
        w[q] = w[q] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        h[q] = f2bf(w[q]);
    }
    *(f32x4_t *)(J.m + i) = m;
    *(f32x4_t *)(J.v + i) = v;
    *(f32x4_t *)(J.w + i) = w;
    if (J.wb)
        *(uint2 *)(J.wb + i) = make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16),
                                          (uint32_t)h[2] | ((uint32_t)h[3] << 16));
}

// Parameters between the real layout in pinned host memory (per layer the
// matrix [rows][cols], then the bias [rows]) and the padded device tensors, in
// one pass over the host link; one block per 1024 real elements of a layer's
// matrix or bias.  Copies row by row through pageable memory took 29 ms for
// the 8 MB.
template <bool TO_DEV>
__global__ void __launch_bounds__(256) params_kernel(ParamJobs jobs, float *__restrict__ host)
{
    int x = blockIdx.x, j = 0;
    while (j < ADAM_JOBS - 1 && x >= jobs.blocks[j]) x -= jobs.blocks[j++];
    const ParamJob J = jobs.job[j];
    const unsigned n = (unsigned)J.rows * (unsigned)J.cols;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const unsigned i = (unsigned)x * 1024u + (unsigned)q * 256u + threadIdx.x;
        if (i >= n) return;
        const unsigned r = i / (unsigned)J.cols, c = i - r * (unsigned)J.cols;
        float *const d = J.dev + (size_t)r * J.pitch + c;
        if (TO_DEV)
            *d = host[J.off + i];
        else
            host[J.off + i] = *d;
    }
}

// bf16 copy of a weight matrix.
__global__ void cast_kernel(const float *__restrict__ w, int64_t n, uint16_t *__restrict__ wb)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) wb[i] = f2bf(w[i]);
}

struct FeatureArgs {
    FrameDev *frames;
    dpps_robot *robots;
    dpps_variant *variants;
    uint16_t *x;
    int n_frames, in_pad;
    float inv_hl, inv_hw, inv_v;
};
struct FeatureOneArgs {
    FeatureArgs a;
    OneFrame one;
};

// Feature vector of a frame (one wave per row): teammates with the passer
// first and the rest by distance to the ball, zero-padded to 8 slots; then
// the opponents by distance to the ball in slots 8-15; then the ball.
// Positions are divided by the field's half length / half width, velocities
// by 3.25 m/s.  Columns 66..in_pad-1 are zero; rows >= n_frames are zero.
// Lanes 0-15 rank the team, lanes 16-31 the opponents (ties to the lower
// robot index); the slot table goes through LDS; each lane then writes
// columns l and l + 64 of the row.
// One launch-carried frame (INL) is a kernel of its own: with pointers that
// may lead to either memory, 4096 rows took 17.5 us instead of 5.
__device__ __forceinline__ void feature_row(const FeatureArgs &args, const FrameDev *frames,
                                            const dpps_robot *robots,
                                            const dpps_variant *carried)
{
    const int n_frames = args.n_frames, in_pad = args.in_pad;
    const float inv_hl = args.inv_hl, inv_hw = args.inv_hw, inv_v = args.inv_v;
    __shared__ int slot_robot[16];
    const int f = blockIdx.x;
    const int l = threadIdx.x;
    uint16_t *row = args.x + (size_t)f * in_pad;
    const bool real = f < n_frames;
    FrameDev F;
    if (real) F = frames[f];
    if (carried && real) {  // one frame: its tables for the kernels that follow
        if (l < F.n_team + F.n_opp) args.robots[l] = robots[l];
        if (l < F.n_variants) args.variants[l] = carried[l];
        if (l == 0) args.frames[0] = F;
    }
    if (l < 16) slot_robot[l] = -1;
    __syncthreads();
    if (real) {
        const int side = l >> 4, r = l & 15;
        const int cnt = side == 0 ? F.n_team : F.n_opp;
        const int base = side == 0 ? 0 : F.n_team;
        const bool have = l < 32 && r < cnt;
        float key = INFINITY;
        if (have) {
            const dpps_robot R = robots[F.robot_off + base + r];
            const float dx = R.x - F.ball_x, dy = R.y - F.ball_y;
            key = (side == 0 && r == F.passer) ? -1.0f : dx * dx + dy * dy;
        }
        int rank = 0;
        for (int j = 0; j < 16; ++j) {
            const float kj = __shfl(key, (l & 48) | j, 64);
            rank += (kj < key || (kj == key && j < r)) ? 1 : 0;
        }
        if (have && rank < 8) slot_robot[side * 8 + rank] = base + r;
    }
    __syncthreads();
    for (int c = l; c < in_pad; c += 64) {
        float v = 0.0f;
        if (real && c < 64) {
            const int rb = slot_robot[c >> 2];
            if (rb >= 0) {
                const dpps_robot R = robots[F.robot_off + rb];
                const int comp = c & 3;
                v = comp == 0 ? R.x * inv_hl : comp == 1 ? R.y * inv_hw
                                             : comp == 2 ? R.vx * inv_v : R.vy * inv_v;
            }
        } else if (real && c == 64) {
            v = F.ball_x * inv_hl;
        } else if (real && c == 65) {
            v = F.ball_y * inv_hw;
        }
        row[c] = f2bf(v);
    }
}

__global__ void __launch_bounds__(64) featurize_kernel(FeatureArgs args)
{
    feature_row(args, args.frames, args.robots, nullptr);
}

__global__ void __launch_bounds__(64) featurize_one_kernel(FeatureOneArgs args)
{
    // read from the kernel's arguments in memory (an indexed by-value struct
    // would be copied to scratch)
    typedef const __attribute__((address_space(4))) FeatureOneArgs *KernArgs;
    const OneFrame &one =
        ((const FeatureOneArgs *)(KernArgs)__builtin_amdgcn_kernarg_segment_ptr())->one;
    feature_row(args.a, &one.frame, one.robots, one.variants);
}

// Top-k cells of each frame's predicted map (one 256-thread workgroup per
// frame), ordered by (score, index) descending with ties to the lower index.
// The cells' keys (order-preserving score bits) stay in registers (thread t
// holds cells t, t + 256, ...).  Radix passes of 8 bits narrow down the bin
// of key prefixes that holds the k-th largest key: each pass histograms the
// next digit of the keys in the current bin and picks the digit where the
// count of larger keys reaches k.  Keys above the bin are all taken; once the
// bin holds at most 256 keys, its best ones are found by ranking them
// (composite key: score bits, then the inverted index); a bin of more than
// 256 exactly equal keys gives its lowest indices.  The k winners are
// ordered by their ranks among themselves.
constexpr int TOPK_THREADS = 256;
static_assert(TOPK_MAX <= TOPK_THREADS, "one thread per top-k winner");

// Inclusive prefix sum over the 256 threads of a workgroup (sh: 4 ints):
// DPP row shifts within each row of 16 lanes (lanes without a source add 0),
// the row totals carried by lane reads, then the wave totals through LDS.
template <int N>
__device__ __forceinline__ int row_shr_add(int v)
{
    return v + __builtin_amdgcn_update_dpp(0, v, 0x110 + N, 0xf, 0xf, false);
}

__device__ __forceinline__ int block_scan_256(int v, int *sh)
{
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    v = row_shr_add<1>(v);
    v = row_shr_add<2>(v);
    v = row_shr_add<4>(v);
    v = row_shr_add<8>(v);
    const int r0 = __builtin_amdgcn_readlane(v, 15);
    const int r1 = __builtin_amdgcn_readlane(v, 31);
    const int r2 = __builtin_amdgcn_readlane(v, 47);
    v += (l >= 16 ? r0 : 0) + (l >= 32 ? r1 : 0) + (l >= 48 ? r2 : 0);
    if (l == 63) sh[w] = v;
    __syncthreads();
    int add = 0;
    for (int i = 0; i < w; ++i) add += sh[i];
    __syncthreads();
    return v + add;
}

// Re-score tables of frame f from its top-k cells (the whole workgroup;
// thread t < k holds cell t): each coarse cell (ci, cj) becomes the window
// of fine points {4 ci - 2 .. 4 ci + 1} x {4 cj - 2 .. 4 cj + 1} clipped to
// the fine lattice, one tile per window, and the frame's copy points at
// its k windows.
__device__ void rescore_windows(const RescoreTables &rt, int f, int k, int cell, int *scan_sh)
{
    const FrameDev F = rt.src[f];
    const int t = threadIdx.x;
    int i0 = 0, j0 = 0, nx = 0, ny = 0;
    if (t < k) {
        const int ci = cell % rt.coarse_nx, cj = cell / rt.coarse_nx;
        const int a0 = max(4 * ci - 2, 0), b0 = max(4 * cj - 2, 0);
        const int a1 = min(4 * ci + 1, rt.fine_nx - 1), b1 = min(4 * cj + 1, rt.fine_ny - 1);
        i0 = a0;
        j0 = b0;
        nx = max(a1 - a0 + 1, 0);
        ny = max(b1 - b0 + 1, 0);
    }
    // element offsets: windows in rank order, each with all the frame's variants
    const int incl = block_scan_256(nx * ny, scan_sh);
    if (t < k) {
        WinDev W;
        W.h = rt.fine_h;
        W.i0 = i0;
        W.j0 = j0;
        W.nx = nx;
        W.halfNx = 0.5f * (float)(rt.fine_nx - 1);
        W.halfNy = 0.5f * (float)(rt.fine_ny - 1);
        W.frame = f;
        W.npts = nx * ny;
        W.n_tiles = 1;
        W.elem_base = (incl - nx * ny) * F.n_variants;
        W.out_base = 0;
        rt.wins[(size_t)f * k + t] = W;
        TileDev T;
        T.win = f * k + t;
        T.at = 0;
        rt.tiles[(size_t)f * k + t] = T;
    }
    if (t == 0) {
        FrameDev G = F;
        G.n_windows = k;
        G.win_off = f * k;
        G.tile_begin = f * k;
        G.tile_count = k;
        rt.frames[f] = G;
    }
}

__global__ void __launch_bounds__(TOPK_THREADS) topk_kernel(const float *__restrict__ y, int ldy,
                                                            int n_cells, int k,
                                                            int32_t *__restrict__ out, RescoreTables rt)
{
    constexpr int PER = TOPK_SORT / TOPK_THREADS;
    constexpr int RANK_MAX = TOPK_THREADS;
    __shared__ int hist[256];
    __shared__ int scan_sh[4];
    __shared__ int pick[3];   // digit, keys still to take at it, keys at it
    __shared__ int n_sel, n_cand;
    __shared__ unsigned long long cand[RANK_MAX];
    __shared__ unsigned long long buf[TOPK_MAX];
    __shared__ unsigned long long sorted[TOPK_MAX];
    const int f = blockIdx.x;
    const int t = threadIdx.x;
    const int lane = t & 63;
    uint32_t u[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = j * TOPK_THREADS + t;
        uint32_t b = 0u;
        if (i < n_cells) {
            b = __float_as_uint(y[(size_t)f * ldy + i]);
            b = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
        }
        u[j] = b;
    }
    uint32_t prefix = 0u, pmask = 0u;
    int rem = k, at_T = 0;
    bool ranked = false;
    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        hist[t] = 0;
        __syncthreads();
        // a wave whose counted keys share one digit (typical of the leading
        // digits: sign and exponent) adds them with one atomic
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const bool act = j * TOPK_THREADS + t < n_cells && (u[j] & pmask) == prefix;
            const uint32_t dg = (u[j] >> shift) & 255u;
            const unsigned long long am = __ballot(act);
            if (am == 0ull) continue;
            const int first = __builtin_ctzll(am);
            const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)dg, first);
            if (__ballot(act && dg != d0) == 0ull) {
                if (lane == first) atomicAdd(&hist[d0], (int)__popcll(am));
            } else if (act) {
                atomicAdd(&hist[dg], 1);
            }
        }
        __syncthreads();
        // thread t holds digit 255 - t: the inclusive scan counts the keys
        // whose digit is >= that digit
        const int d = 255 - t;
        const int c = hist[d];
        const int incl = block_scan_256(c, scan_sh);
        const int excl = incl - c;
        if (excl < rem && incl >= rem) {
            pick[0] = d;
            pick[1] = rem - excl;
            pick[2] = c;
        }
        __syncthreads();
        prefix |= (uint32_t)pick[0] << shift;
        pmask |= 255u << shift;
        rem = pick[1];
        at_T = pick[2];
        __syncthreads();
        if (at_T <= RANK_MAX) {
            ranked = true;
            break;
        }
    }
    if (t == 0) {
        n_sel = 0;
        n_cand = 0;
    }
    __syncthreads();
    // keys above the bin are taken, the bin's keys are candidates
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int i = j * TOPK_THREADS + t;
        if (i >= n_cells) continue;
        const uint32_t m = u[j] & pmask;
        const unsigned long long ck =
            ((unsigned long long)u[j] << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)i);
        if (m > prefix)
            buf[atomicAdd(&n_sel, 1)] = ck;
        else if (ranked && m == prefix)
            cand[atomicAdd(&n_cand, 1)] = ck;
    }
    if (!ranked) {
        // more than RANK_MAX keys equal the k-th largest: the rem lowest
        // indices among them, in index order (row j holds indices 256 j + t)
        int before = 0;
        for (int j = 0; j < PER; ++j) {
            const int i = j * TOPK_THREADS + t;
            const int e = (i < n_cells && u[j] == prefix) ? 1 : 0;
            const int incl = block_scan_256(e, scan_sh);
            if (e && before + incl <= rem)
                buf[atomicAdd(&n_sel, 1)] = ((unsigned long long)u[j] << 32) |
                                            (unsigned long long)(0xFFFFFFFFu - (uint32_t)i);
            if (t == TOPK_THREADS - 1) scan_sh[0] = incl;
            __syncthreads();
            before += scan_sh[0];
            __syncthreads();
        }
    }
    __syncthreads();
    if (ranked && t < at_T) {
        // composite keys are unique: the rem highest candidates
        const unsigned long long my = cand[t];
        int r = 0;
        for (int q = 0; q < at_T; ++q) r += cand[q] > my ? 1 : 0;
        if (r < rem) buf[atomicAdd(&n_sel, 1)] = my;
    }
    __syncthreads();
    // the k winners in order: each one's rank among them
    if (t < k) {
        const unsigned long long my = buf[t];
        int r = 0;
        for (int q = 0; q < k; ++q) r += buf[q] > my ? 1 : 0;
        sorted[r] = my;
    }
    __syncthreads();
    int cell = 0;
    if (t < k) {
        cell = (int32_t)(0xFFFFFFFFu - (uint32_t)sorted[t]);
        out[(size_t)f * k + t] = cell;
    }
    if (rt.frames) rescore_windows(rt, f, k, cell, scan_sh);
    if (rt.zero_word && f == 0 && threadIdx.x == 0) *rt.zero_word = 0;
    if (rt.frame_best && threadIdx.x < 2) rt.frame_best[threadIdx.x * gridDim.x + f] = 0u;
}

// host launchers -------------------------------------------------------------

int colsum_chunks(int M) { return (M + COLSUM_ROWS - 1) / COLSUM_ROWS; }

int launch_colsum(const ColsumJobs &jobs, int M, void *st)
{
    const int chunks = colsum_chunks(M);
    int blocks = 0;
    for (int j = 0; j < 4; ++j) {
        if (jobs.n[j] < 256 || jobs.n[j] % 256) return -1;
        blocks += jobs.n[j] / 256;
    }
    if (M < 1) return -1;
    hipLaunchKernelGGL(colsum_part_kernel, dim3(blocks, chunks), dim3(256), 0, (hipStream_t)st, jobs,
                       M);
    hipLaunchKernelGGL(colsum_final_kernel, dim3(4 * blocks), dim3(64), 0, (hipStream_t)st, jobs, chunks);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_loss(const float *y, int ldy, const float *tgt, int ldt, int rows, int outs, int rows_pad,
                int outs_pad, float pos_weight, float ce_weight, float tau, uint16_t *dz,
                float *partial, void *st)
{
    if (outs > outs_pad || outs_pad > LOSS_PER * 256) return -1;
    hipLaunchKernelGGL(loss_kernel, dim3(rows_pad), dim3(256), 0, (hipStream_t)st, y, ldy, tgt, ldt,
                       rows, outs, rows_pad, outs_pad, pos_weight, ce_weight, tau, dz, partial);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_pool(const float *fine, int n_frames, int fnx, int fny, float *coarse, int cnx, int cny,
                void *st)
{
    int64_t n = (int64_t)n_frames * cnx * cny;
    if (n == 0) return 0;
    hipLaunchKernelGGL(pool_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                       (hipStream_t)st, fine, n_frames, fnx, fny, coarse, cnx, cny);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_adam(AdamJobs jobs, float lr, float b1, float b2, float eps, float c1, float c2, void *st)
{
    int blocks = 0;
    for (int j = 0; j < ADAM_JOBS; ++j) {
        if (jobs.job[j].n < 4 || jobs.job[j].n % 4) return -1;
        jobs.blocks[j] = (int)((jobs.job[j].n / 4 + 255) / 256);
        blocks += jobs.blocks[j];
    }
    hipLaunchKernelGGL(adam_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)st, jobs, lr, b1, b2,
                       eps, c1, c2);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_params(ParamJobs jobs, float *host, bool to_dev, void *st)
{
    int blocks = 0;
    for (int j = 0; j < ADAM_JOBS; ++j) {
        if (jobs.job[j].rows < 1 || jobs.job[j].cols < 1) return -1;
        jobs.blocks[j] = (int)(((int64_t)jobs.job[j].rows * jobs.job[j].cols + 1023) / 1024);
        blocks += jobs.blocks[j];
    }
    if (to_dev)
        hipLaunchKernelGGL(params_kernel<true>, dim3(blocks), dim3(256), 0, (hipStream_t)st, jobs, host);
    else
        hipLaunchKernelGGL(params_kernel<false>, dim3(blocks), dim3(256), 0, (hipStream_t)st, jobs, host);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_cast(const float *w, int64_t n, uint16_t *wb, void *st)
{
    hipLaunchKernelGGL(cast_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                       (hipStream_t)st, w, n, wb);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_featurize(FrameDev *frames, dpps_robot *robots, dpps_variant *variants, int n_frames,
                     int rows_pad, int in_pad, float inv_hl, float inv_hw, float inv_v, uint16_t *x,
                     const OneFrame *one, void *st)
{
    if (rows_pad == 0) return 0;
    FeatureArgs a;
    memset(&a, 0, sizeof a);
    a.frames = frames;
    a.robots = robots;
    a.variants = variants;
    a.n_frames = n_frames;
    a.in_pad = in_pad;
    a.inv_hl = inv_hl;
    a.inv_hw = inv_hw;
    a.inv_v = inv_v;
    a.x = x;
    if (one) {
        FeatureOneArgs o;
        o.a = a;
        o.one = *one;
        hipLaunchKernelGGL(featurize_one_kernel, dim3(rows_pad), dim3(64), 0, (hipStream_t)st, o);
    } else {
        hipLaunchKernelGGL(featurize_kernel, dim3(rows_pad), dim3(64), 0, (hipStream_t)st, a);
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_topk(const float *y, int ldy, int n_frames, int n_cells, int k, int32_t *out,
                const RescoreTables *rt, void *st)
{
    if (n_cells > TOPK_SORT || k > n_cells || k > TOPK_MAX) return -1;
    RescoreTables r;
    memset(&r, 0, sizeof r);
    if (rt) r = *rt;
    hipLaunchKernelGGL(topk_kernel, dim3(n_frames), dim3(TOPK_THREADS), 0, (hipStream_t)st, y, ldy,
                       n_cells, k, out, r);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace dpps
