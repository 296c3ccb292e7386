// mlp_internal.h -- internal interface of the surrogate kernels (libdpps).
#pragma once

#include <stdint.h>

#include "dpps_internal.h"

namespace dpps {

enum { EPI_BIAS = 1, EPI_BIAS_GELU = 2, EPI_GELU_GRAD = 3, EPI_PARTIAL = 4 };

#define TOPK_SORT 4096   // most cells per frame for the top-k (>= coarse lattice size)
#define TOPK_MAX 256     // largest k (one workgroup thread per winner)

struct GemmArgs {
    const uint16_t *A;   // bf16
    const uint16_t *B;   // bf16
    int lda, ldb, ldc;
    int M, N, K;
    const float *bias;   // EPI_BIAS, EPI_BIAS_GELU
    const float *Zin;    // EPI_GELU_GRAD: pre-activation, [M][ldc]
    float *Cf;           // f32 output (EPI_BIAS_GELU: may be NULL)
    uint16_t *Cb;        // bf16 output
    float *work;         // workspace of a K split (weight gradients), work_elems floats
    int64_t work_elems;
    int k_slice;         // set by the dispatcher
    float *out;          // EPI_BIAS: a second copy of rows < out_m, columns < out_n (may be NULL)
    int64_t ld_out;
    int out_m, out_n;
};

// A layer's product (A, B k-contiguous; EPI_BIAS or EPI_BIAS_GELU).
int gemm(const GemmArgs &g, int epi, void *stream);
// The two products of a backward layer: x (may be NULL), the input gradient
// (A k-contiguous, B as [k][n]; GELU-gradient epilogue), and w, the weight
// gradient (A as [k][m], B as [k][n]) into w.Cf through the workspace w.work.
int gemm_backward(const GemmArgs *x, const GemmArgs &w, void *stream);
// Inference GEMM of a few rows (A, B k-contiguous; EPI_BIAS or EPI_BIAS_GELU),
// bit-identical per element to gemm(g, epi, stream).
int gemm_rows(const GemmArgs &g, int epi, void *stream);
// Column sums of the layers' output gradients dz [M][n] (n a multiple of 256):
// db; part holds colsum_chunks(M) x n floats.
struct ColsumJobs {
    const uint16_t *dz[4];
    float *db[4];
    float *part[4];
    int n[4];
};
int launch_colsum(const ColsumJobs &jobs, int M, void *st);
int colsum_chunks(int M);
int launch_loss(const float *y, int ldy, const float *tgt, int ldt, int rows, int outs, int rows_pad,
                int outs_pad, float pos_weight, float ce_weight, float tau, uint16_t *dz,
                float *partial, void *st);
int launch_pool(const float *fine, int n_frames, int fnx, int fny, float *coarse, int cnx, int cny,
                void *st);
// One Adam step on a list of tensors (n multiples of 4, 16-byte aligned); wb
// (may be NULL) is refreshed from w.
#define ADAM_JOBS 8
struct AdamJob {
    float *w;
    const float *g;
    float *m, *v;
    uint16_t *wb;
    int64_t n;
    float wd;
};
struct AdamJobs {
    AdamJob job[ADAM_JOBS];
    int blocks[ADAM_JOBS];  // set by the launcher
};
int launch_adam(AdamJobs jobs, float lr, float b1, float b2, float eps, float c1, float c2, void *st);
// Copies of padded device tensors (dev, pitch floats a row) and their real
// rows x cols elements at off in the host's parameter vector (pinned memory).
struct ParamJob {
    float *dev;
    int64_t off;
    int rows, cols, pitch;
};
struct ParamJobs {
    ParamJob job[ADAM_JOBS];
    int blocks[ADAM_JOBS];  // set by the launcher
};
int launch_params(ParamJobs jobs, float *host, bool to_dev, void *st);
int launch_cast(const float *w, int64_t n, uint16_t *wb, void *st);
// one (may be NULL): the only frame, written to frames, robots and variants.
int launch_featurize(FrameDev *frames, dpps_robot *robots, dpps_variant *variants, int n_frames,
                     int rows_pad, int in_pad, float inv_hl, float inv_hw, float inv_v, uint16_t *x,
                     const OneFrame *one, void *st);
// Re-score tables written by the top-k kernel: per frame f, its copy
// frames[f] (n_windows = tile_count = k), k windows and k tiles.
struct RescoreTables {
    const FrameDev *src;
    int coarse_nx, fine_nx, fine_ny;
    float fine_h;
    FrameDev *frames;
    WinDev *wins;
    TileDev *tiles;
    int32_t *zero_word;     // cleared by the kernel (may be NULL)
    uint32_t *frame_best;   // 2 n_frames words cleared by the kernel (may be NULL)
};
// Top-k cells of each frame's map into out [n_frames][k]; with rt, also the
// re-score tables of those cells.
int launch_topk(const float *y, int ldy, int n_frames, int n_cells, int k, int32_t *out,
                const RescoreTables *rt, void *st);

}  // namespace dpps
