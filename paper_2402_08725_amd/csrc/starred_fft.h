// FFT-path data structures shared by the plan (host) and the FFT kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "starred_dense.h"
#include "starred_internal.h"

namespace starred {

constexpr int kFftThreads = 256;
constexpr int kFftTargetElems = 2048;  // complex elements per work group and buffer
constexpr int kFusedThreads = 1024;     // one-launch forward: threads of a work group
constexpr size_t kFusedLdsMax = 150 * 1024;  // one-launch forward: LDS of a work group
constexpr int kFwdFrames = 4;          // spectral product: frames whose loads are issued together
constexpr int kAdjFrames = 2;          // spectral adjoint: frames of a work group (a chunk), default
constexpr int kAdjMaxFrames = 8;       // spectral adjoint: most frames of a chunk
constexpr int kAdjSB = 4;              // spectral adjoint: sources per pass over the rows (M > 1)
constexpr int kAdjSBWide = 8;          // the same with 2-frame chunks and more than kAdjSB sources
constexpr int kAdjSBOne = 16;          // the same with 1-frame chunks (more than kAdjSBWide sources; s < 3)
constexpr int kAdjBlocks = 512;        // spectral adjoint: work groups aimed at per launch
constexpr int kAdjMinRows = 4;         // spectral adjoint: fewest rows of the P grid per thread
constexpr int kAdjMaxRows = 64;        // spectral adjoint: most rows of the P grid per work group
constexpr int kAdjRB = 3;              // spectral adjoint: rows of a thread whose loads are issued together
constexpr int kSumBins = 64;           // chunk-spectrum sums: bins of a work group
constexpr int kSumParts = 4;           // chunk-spectrum sums: runs of chunks per bin (threads)
constexpr int kSumBatch = 16;          // chunk-spectrum sums: loads of a run in flight together
// values of a P x P spectrum in alias order (see starred_fft.hip): s^2 for each bin of the
// Q x (Q/2+1) half plane
__host__ __device__ inline long long alias_bins(int P, int Q) { return (long long)(P / Q) * P * (Q / 2 + 1); }

// A 1-D transform length L = product of radices (4, 2, 3, 5) and the offset of
// its twiddle table e^{-2 pi i m / L}, m < L.
struct FftLen {
    int L;
    int nst;
    int rad[8];
    long long tw_off;
};

// One shape class: frames with the same fine side F, kernel side K and window.
// P is the circular size (P >= F + floor(K/2), a multiple of 2s), Q = P/s.
struct ClassFft {
    int P, Q, F, n, o, K;
    FftLen fP, fQ;
    long long th_off;   // [F][P/2+1]   rows of the h window
    long long hh_off;   // spectrum of the h window, alias order
    long long tab_off;  // [(1 + 2M) P] window and point-source factor tables
    float sscale;       // 1 / (s^2 Q^2)
    int cf_off;         // first entry of this class in the class-ordered frame list
    int ncf;            // number of frames of the class
    int ngch;           // frame chunks of the frequency-domain adjoint
    int gfch;           // frames per chunk
    int ngch_cap;       // chunks the class's gp region holds (its smallest allowed chunks)
    long long gp_off;   // [ngch] summed adjoint spectra of each chunk, alias order (total in chunk 0)
    long long hc_off;   // [F][F] the class's contribution to dL/dh (its window)
    int fused;          // frames of this class take the one-launch forward (spectra fit in LDS)
    int arr;            // spectral adjoint: rows of the Q grid per work group (s rows of the P grid each)
    int nrr;            // spectral adjoint: row ranges (per-frame partial slots)
    int direct;         // the class runs the direct algorithm (the FFT launches skip it)
};

struct FrameFft {
    int cls;
    int pad;
    long long kern_off;  // packed K^2 kernels
    long long s_off;     // kernel spectrum S'', alias order
    long long t_off;     // [n][Q/2+1] row spectra (model / rho)
    long long r_off;     // [Q][Q/2+1] rho_hat
    long long t3_off;    // [P][P/2+1] scratch of the adjoint (and of the kernel transform)
    long long data_off;  // packed n^2
    long long fine_off;  // packed F^2
};

// A group of consecutive lines of one frame (or one class) handled by one work group.
struct LineItem {
    int cls;
    int frame;
    int line0;
    int nl;
};

// A block of output bins of one class and a chunk of that class's frames.
struct SpecItem {
    int cls;
    int f0;
    int nf;
    int bin0;
};

// The transform lengths of the one-launch forward (starred_frame.h): Q = RA RB, and the
// frames NF that a work group takes of a class when frames outnumber the compute units
// (X(Q, RA, RB, NF)): every even 5-smooth length from 16 to 180 but 162, which has no two
// factors up to 16. RA is at least 8, so that the residual's reads come in runs of 32 bytes
// or more. Two frames of 120 or more would need more registers than 1024 threads have (128
// is the exception), or more LDS than there is. 192 has a body for s = 1 without point sources
// (frame_body_frames), the only frames of that length whose plane and tables fit: 300 frames of
// 128^2 207 us on the line passes, 127 with it.
#define STARRED_FRAME_LENGTHS(X) \
    X(16, 8, 2, 4)               \
    X(18, 9, 2, 4)               \
    X(20, 10, 2, 4)              \
    X(24, 12, 2, 4)              \
    X(30, 10, 3, 4)              \
    X(32, 16, 2, 4)              \
    X(36, 12, 3, 4)              \
    X(40, 8, 5, 4)               \
    X(48, 16, 3, 4)              \
    X(50, 10, 5, 4)              \
    X(54, 9, 6, 4)               \
    X(60, 12, 5, 4)              \
    X(64, 16, 4, 4)              \
    X(72, 12, 6, 4)              \
    X(80, 16, 5, 2)              \
    X(90, 10, 9, 2)              \
    X(96, 16, 6, 2)              \
    X(100, 10, 10, 2)            \
    X(108, 12, 9, 2)             \
    X(120, 12, 10, 1)            \
    X(128, 16, 8, 2)             \
    X(144, 16, 9, 1)             \
    X(150, 15, 10, 1)            \
    X(160, 16, 10, 1)            \
    X(180, 15, 12, 1)
constexpr int kFrameMinQ = 16, kFrameMaxQ = 180;
constexpr int kFrameLongQ = 192;

// frames that a work group may take of a class with transform length Q (0: no body);
// several of them only for s = 2 (compile time)
inline int frame_body_frames(int Q, int s)
{
#define STARRED_FRAME_NF(QQ, RA, RB, NF) \
    if (Q == QQ) return s == 2 ? NF : 1;
    STARRED_FRAME_LENGTHS(STARRED_FRAME_NF)
#undef STARRED_FRAME_NF
    return Q == kFrameLongQ && s == 1 ? 1 : 0;
}

// sources whose tables a work group of transform length Q holds: the bodies take 1, 4 or (a loop) M
// of them, the one of kFrameLongQ none
__host__ __device__ constexpr int frame_sources(int M, int Q)
{
    return Q == kFrameLongQ && M == 0 ? 0 : (M <= 1 ? 1 : (M <= 4 ? 4 : M));
}

// bytes of LDS of a work group with `per` frames: their planes of Q/2+1 lines of Q+1
// values, the Q twiddles and the tables of P values (the window's, two per source)
inline size_t frame_lds_bytes(int Q, int P, int M, int per)
{
    return ((size_t)per * (Q / 2 + 1) * (Q + 1) + Q + (size_t)(1 + 2 * frame_sources(M, Q)) * P) * 8;
}

// A work group of the one-launch forward: up to `per` frames of a class.
constexpr int kFrameMax = 4;
struct FrameItem {
    int nf, per;  // frames, and frames the body holds
    int Q, n;
    long long tw_off, tab_off, hh_off;
    int frame[kFrameMax], chi[kFrameMax];  // frame indices and their chi-square slots
    long long s_off[kFrameMax], data_off[kFrameMax], r_off[kFrameMax];
};

// A work group of the frequency-domain adjoint: a chunk of frames and a range of
// rows of one class, with everything the group needs resolved on the host (so
// its loads depend on this item alone).
struct AdjItem {
    int cls;
    int nf;                      // frames in the chunk
    int y0, y1;                  // rows [y0, y1) of the Q grid
    int P, Q;
    int pb;                      // row range index (the per-frame partial slot)
    int pad;
    int fid[kAdjMaxFrames];         // frame indices (-1 past nf)
    long long soff[kAdjMaxFrames];  // kernel spectra S'' (the chunk's first frame again past nf)
    long long roff[kAdjMaxFrames];  // rho_hat (the chunk's first frame again past nf)
    long long tab_off;           // the class's factor tables
    long long gout;              // the chunk's slot in the chunk spectra
};

struct LinePass {
    LineItem *items = nullptr;  // device
    int n_items = 0;
    int aliases = 1;  // k_fold, k_unfold: lines of a column transformed at a time (1 or s)
    size_t lds_bytes = 0;
};

struct FftPlanDev {
    ClassFft *classes = nullptr;
    FrameFft *frames = nullptr;
    int n_classes = 0;
    float2 *tw = nullptr;
    float2 *S = nullptr, *T = nullptr, *T2 = nullptr, *Rh = nullptr, *T3 = nullptr;
    float2 *Th = nullptr, *Hh = nullptr, *tab = nullptr;
    LinePass hrows, hcols, krows, kcols, fcols, frows, rcols;
    // operators on given scenes and residuals (rows in pairs; fold: columns of the Q grid)
    LinePass srows, rrows, arows, fold;
    SpecItem *spec = nullptr;
    int n_spec = 0;
    int *cls_frames = nullptr;
    // frequency-domain adjoint
    int n_frames = 0;
    AdjItem *aspec = nullptr;
    int n_aspec = 0;
    int adj_fc = kAdjFrames;   // frames per chunk of the current items
    int maxpb = 0;           // per-frame partial slots (largest nrr)
    long long total_bins = 0;  // sum over classes of alias_bins
    double *apart = nullptr; // [E][maxpb][1 + 3M]
    float2 *Gp = nullptr;
    float *hcls = nullptr;
    LinePass gcols, grows;
    // loss+gradient forward: frames of fused classes in one launch; the line passes
    // below cover the remaining frames
    SpecItem *spec_lg = nullptr;
    int n_spec_lg = 0;
    FrameItem *frame_items = nullptr;
    int n_frame_items = 0;
    int n_fused = 0;  // frames they cover
    size_t frame_lds = 0;
    LinePass fcols_lg, frows_lg, rcols_lg;
    // every frame, whatever its class runs: the per-frame convolution of rendered
    // scenes (frames with per-frame transforms)
    LinePass srows_x, fold_x, frows_x, arows_x;
};

// Deterministic block sum of one double per thread (NT threads); thread 0 holds it.
template <int NT = kFftThreads>
__device__ __forceinline__ double block_sum_d_fft(double v, double *sh)
{
    #pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0) {
        #pragma unroll
        for (int i = 0; i < NT / 64; ++i) r += sh[i];
    }
    __syncthreads();
    return r;
}

hipError_t fft_prep_kernels(hipStream_t st, const FftPlanDev &d, const float *psf, int s);
// tick: a step counter the launch advances (the first launch of a fused step), or null
// pa, pb: passes of the starlet prior carried by the row and column launches (or null)
hipError_t fft_spectra(hipStream_t st, const FftPlanDev &d, const float *params, int N, int E, int M,
                       float sigma, int *tick = nullptr, DensePiece *pa = nullptr, DensePiece *pb = nullptr);
hipError_t fft_spec_fwd(hipStream_t st, const FftPlanDev &d, const float *params, int N, int E, int M, int s,
                        bool lg = false);
hipError_t fft_model_cols(hipStream_t st, const FftPlanDev &d);
hipError_t fft_model_rows(hipStream_t st, const FftPlanDev &d, const float *data, const float *invvar,
                          double *part_chi, float *model, bool want_rho = true);
hipError_t fft_rho_cols(hipStream_t st, const FftPlanDev &d);
hipError_t fft_scene_adjoint(hipStream_t st, const FftPlanDev &d, const float *resid, int s, float *g);
hipError_t fft_spec_adj(hipStream_t st, const FftPlanDev &d, int M, int s);
hipError_t fft_adj_sums(hipStream_t st, const FftPlanDev &d, int M, double *fsum);
struct FinalArgs;
// dL/dh of the classes: the column inverse alone, and (one class whose window
// is the whole grid) the row inverse that also writes dL/dh, updates h and does
// the evaluation's small reductions in an extra work group
hipError_t fft_grad_h_cols(hipStream_t st, const FftPlanDev &d, DensePiece *pd = nullptr);
// psum (or null): the composite-filter prior's planes after pass D1, summed per pixel instead of reading prior
hipError_t fft_grad_h_rows_final(hipStream_t st, const FftPlanDev &d, const float *prior, const FinalArgs &fin,
                                 const DenseStar *psum = nullptr);
// want_rho: also rho_hat, which the adjoint reads (else the loss alone)
hipError_t fft_fused_fwd(hipStream_t st, const FftPlanDev &d, const float *params, int N, int E, int M, int s,
                         const float *data, const float *invvar, double *part_chi, DensePiece *pc = nullptr,
                         bool want_rho = true);
struct FrameArgs {
    const float2 *tw, *Sp, *Hh, *tab;
    const float *params;
    int N, E, M;
    const float *data, *invvar;
    float2 *Rh;  // null: the loss alone
    double *part_chi;
};

hipError_t launch_frames_s1(hipStream_t st, const FftPlanDev &d, const FrameArgs &g, const DensePiece &dp, size_t lds);
hipError_t launch_frames_s2(hipStream_t st, const FftPlanDev &d, const FrameArgs &g, const DensePiece &dp, size_t lds);
hipError_t launch_frames_s3(hipStream_t st, const FftPlanDev &d, const FrameArgs &g, const DensePiece &dp, size_t lds);
hipError_t fft_model_cols_lg(hipStream_t st, const FftPlanDev &d);
hipError_t fft_model_rows_lg(hipStream_t st, const FftPlanDev &d, const float *data, const float *invvar,
                             double *part_chi, bool want_rho = true);
hipError_t fft_rho_cols_lg(hipStream_t st, const FftPlanDev &d);
hipError_t fft_grad_h_inverse(hipStream_t st, const FftPlanDev &d, DensePiece *pd = nullptr);
hipError_t fft_scene_model(hipStream_t st, const FftPlanDev &d, const float *scene, int s, float *model);
// Frames with per-frame transforms: S_i and D of each frame's rendered scene (fine
// grid, per-frame layout) through its own spectrum, the weighted residual and its
// chi-square partials (one per row group of frows_x), the residuals' row spectra kept for
// the adjoint.
hipError_t fft_xf_forward(hipStream_t st, const FftPlanDev &d, const float *scene, int s, const float *data,
                          const float *invvar, double *part_chi);
// ... and D^T S_i^T of those residuals into g (fine grid, per-frame layout).
hipError_t fft_xf_adjoint(hipStream_t st, const FftPlanDev &d, int s, float *g);

}  // namespace starred
