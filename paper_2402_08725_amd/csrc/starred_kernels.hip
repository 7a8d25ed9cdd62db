// Device kernels of the deconvolution path (Sec. 2.2, Eqs. 8-11) and the shared
// starlet / optimiser kernels, for gfx950 (wave64).
//
// Precision: FP32 arithmetic with FP32 accumulation for every pixel; the
// chi-square and L1 global sums and the small per-frame dot products are
// reduced in FP64 with fixed (deterministic) trees. No floating-point atomics.
#include "starred_internal.h"
#include "starred_fft.h"
#include "starred_finalize.h"

#include <hip/hip_runtime.h>

#include <algorithm>

namespace starred {

// --------------------------------------------------------------------------
// helpers
// --------------------------------------------------------------------------

// Deterministic block sum of one double per thread; result valid in thread 0.
template <int NT>
__device__ __forceinline__ double block_sum_d(double v, double *sh)
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

// --------------------------------------------------------------------------
// Kernel preprocessing (once per set_frames)
// --------------------------------------------------------------------------

// kf[a][psi][t]  = sum_{al,be < s} k(K-1-a+al, K-1-b+be),  b = s t + psi   (flipped, box-folded)
// ka[py][px][al][be] = sf(s(dmin+al) + cp - py, s(dmin+be) + cp - px),
//   sf(T,U) = sum_{al,be < s} k(T-(s-1)+al, U-(s-1)+be)                      (box-folded)
__global__ void k_prep_kernels(const FrameDev *__restrict__ frames, int s,
                               const float *__restrict__ psf, float *__restrict__ kf,
                               float *__restrict__ ka)
{
    const FrameDev fr = frames[blockIdx.x];
    const float *k = psf + fr.kern_off;
    const int K = fr.K, Kp = fr.Kp;
    auto kv = [&](int v, int u) -> float {
        return (v >= 0 && v < K && u >= 0 && u < K) ? k[v * K + u] : 0.0f;
    };
    const int nf = Kp * s * fr.Tpad;
    for (int e = threadIdx.x; e < nf; e += blockDim.x) {
        int t = e % fr.Tpad;
        int psi = (e / fr.Tpad) % s;
        int a = e / (fr.Tpad * s);
        int b = s * t + psi;
        float acc = 0.0f;
        if (b < Kp)
            for (int al = 0; al < s; ++al)
                for (int be = 0; be < s; ++be) acc += kv(K - 1 - a + al, K - 1 - b + be);
        kf[fr.kf_off + e] = acc;
    }
    const int na = s * s * fr.Ar * fr.Bpad;
    for (int e = threadIdx.x; e < na; e += blockDim.x) {
        int be = e % fr.Bpad;
        int al = (e / fr.Bpad) % fr.Ar;
        int ph = e / (fr.Bpad * fr.Ar);
        int py = ph / s, px = ph % s;
        int T = s * (fr.dmin + al) + fr.cp - py;
        int U = s * (fr.dmin + be) + fr.cp - px;
        float acc = 0.0f;
        if (be < fr.Ar && T >= 0 && T < Kp && U >= 0 && U < Kp)
            for (int a2 = 0; a2 < s; ++a2)
                for (int b2 = 0; b2 < s; ++b2) acc += kv(T - (s - 1) + a2, U - (s - 1) + b2);
        ka[fr.ka_off + e] = acc;
    }
}

hipError_t launch_prep_kernels(hipStream_t st, const FrameDev *fr_dev, const FrameDev *, int E,
                               int s, const float *psf, float *kf, float *ka)
{
    if (E <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_prep_kernels, dim3(E), dim3(256), 0, st, fr_dev, s, psf, kf, ka);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// a1: scene rendering f_i = Gamma_i + h[window_i] + sum_k a_ki r_k   (Eq. 9)
// --------------------------------------------------------------------------

// Per-frame transform t_i = (dx, dy, theta): the frame pixel at grid position X
// reads the scene at u = R(theta)(X - C) + C + (dx, dy), C the grid centre. The
// position is formed in FP64 (a few operations per pixel) so that the bilinear
// weights and the Gaussian offsets carry no FP32 rounding of coordinates that
// reach hundreds of pixels.
struct FrameMap {
    double cs, sn, C, dx, dy;
    FrameMap() = default;
    __device__ FrameMap(const float *xf, int i, int N)
    {
        dx = (double)xf[3 * i];
        dy = (double)xf[3 * i + 1];
        sincos((double)xf[3 * i + 2], &sn, &cs);
        C = 0.5 * (double)(N - 1);
    }
    __device__ void map(double X, double Y, double &ux, double &uy) const
    {
        const double vx = X - C, vy = Y - C;
        ux = cs * vx - sn * vy + C + dx;
        uy = sn * vx + cs * vy + C + dy;
    }
};

__device__ __forceinline__ float h_at(const float *__restrict__ h, int N, int X, int Y)
{
    return (X >= 0 && X < N && Y >= 0 && Y < N) ? h[(long long)Y * N + X] : 0.f;
}

// bilinear read of h at (ux, uy) (zero outside the grid) and its partial derivatives
__device__ __forceinline__ float bilerp(const float *__restrict__ h, int N, double ux, double uy, float *gx,
                                       float *gy)
{
    const double fx = floor(ux), fy = floor(uy);
    const int X0 = (int)fx, Y0 = (int)fy;
    const float tx = (float)(ux - fx), ty = (float)(uy - fy);
    const float h00 = h_at(h, N, X0, Y0), h10 = h_at(h, N, X0 + 1, Y0);
    const float h01 = h_at(h, N, X0, Y0 + 1), h11 = h_at(h, N, X0 + 1, Y0 + 1);
    if (gx) {
        *gx = (1.f - ty) * (h10 - h00) + ty * (h11 - h01);
        *gy = (1.f - tx) * (h01 - h00) + tx * (h11 - h10);
    }
    return (1.f - tx) * (1.f - ty) * h00 + tx * (1.f - ty) * h10 + (1.f - tx) * ty * h01 + tx * ty * h11;
}

__global__ void k_render(const FrameDev *__restrict__ frames, int E, int frame0, int N, int M, float sigma,
                         const float *__restrict__ params, float *__restrict__ scene,
                         const int *__restrict__ flist, const float *__restrict__ xf)
{
    const int i = flist ? flist[blockIdx.y] : frame0 + blockIdx.y;
    const FrameDev fr = frames[i];
    const int pix = blockIdx.x * blockDim.x + threadIdx.x;
    __shared__ FrameMap fm;  // (FP64 sine and cosine once per block, not per pixel)
    if (xf) {
        if (threadIdx.x == 0) fm = FrameMap(xf, i, N);
        __syncthreads();
    }
    if (pix >= fr.F * fr.F) return;
    const int y = pix / fr.F, x = pix % fr.F;
    const int Y = y + fr.o, X = x + fr.o;
    const float *h = params;
    const float *a = params + (long long)N * N + E;
    const float *c = a + (long long)E * M;
    double ux = (double)X, uy = (double)Y;
    float v;
    if (xf) {
        fm.map((double)X, (double)Y, ux, uy);
        v = params[(long long)N * N + i] + bilerp(h, N, ux, uy, nullptr, nullptr);
    } else {
        v = params[(long long)N * N + i] + h[(long long)Y * N + X];
    }
    const float inv2s2 = 1.0f / (2.0f * sigma * sigma);
    const float norm = 1.0f / (2.0f * 3.14159265358979f * sigma * sigma);
    for (int k = 0; k < M; ++k) {
        float dx = (float)(ux - (double)c[2 * k]), dy = (float)(uy - (double)c[2 * k + 1]);
        if (fabsf(dx) <= (float)kGaussRadius && fabsf(dy) <= (float)kGaussRadius)
            v += a[(long long)i * M + k] * (norm * expf(-(dx * dx + dy * dy) * inv2s2));
    }
    scene[fr.fine_off + pix] = v;
}

hipError_t launch_render(hipStream_t st, const FrameDev *fr, int E, int Fmax, int N, int M,
                         float sigma, const float *params, float *scene, const int *flist, int nlist,
                         const float *xf)
{
    const int nf = flist ? nlist : E;
    if (nf <= 0) return hipSuccess;
    dim3 grid((Fmax * Fmax + 255) / 256, nf);
    hipLaunchKernelGGL(k_render, grid, dim3(256), 0, st, fr, E, 0, N, M, sigma, params, scene, flist, xf);
    return hipGetLastError();
}

hipError_t launch_render_frame(hipStream_t st, const FrameDev *fr, int E, int i, int F, int N, int M,
                               float sigma, const float *params, float *scene)
{
    dim3 grid((F * F + 255) / 256, 1);
    hipLaunchKernelGGL(k_render, grid, dim3(256), 0, st, fr, E, i, N, M, sigma, params, scene, nullptr, nullptr);
    return hipGetLastError();
}

// ---- one-frame operators of the plain (unfused, per-epoch) baseline ----

// m = D u  (block sum over s x s)
__global__ void k_block_sum(const FrameDev *__restrict__ frames, int i, int s, const float *__restrict__ u,
                            float *__restrict__ m)
{
    const FrameDev fr = frames[i];
    const int pix = blockIdx.x * blockDim.x + threadIdx.x;
    if (pix >= fr.n * fr.n) return;
    const int p = pix / fr.n, q = pix % fr.n;
    const float *uf = u + fr.fine_off;
    float acc = 0.f;
    for (int a = 0; a < s; ++a)
        for (int b = 0; b < s; ++b) acc += uf[(long long)(s * p + a) * fr.F + s * q + b];
    m[fr.data_off + pix] = acc;
}

// rho = w (m - d), chi-square partial of each block
__global__ __launch_bounds__(256) void k_resid(const FrameDev *__restrict__ frames, int i,
                                               const float *__restrict__ m, const float *__restrict__ data,
                                               const float *__restrict__ invvar, float *__restrict__ rho,
                                               double *__restrict__ part)
{
    __shared__ double red[4];
    const FrameDev fr = frames[i];
    const int pix = blockIdx.x * blockDim.x + threadIdx.x;
    double chi = 0.0;
    if (pix < fr.n * fr.n) {
        const long long idx = fr.data_off + pix;
        const float r = m[idx] - data[idx];
        const float w = invvar[idx];
        rho[idx] = w * r;
        chi = 0.5 * (double)w * (double)r * (double)r;
    }
    chi = block_sum_d<256>(chi, red);
    if (threadIdx.x == 0) part[blockIdx.x] = chi;
}

// gh = D^T rho (replicate each data pixel over its s x s block)
__global__ void k_upsample(const FrameDev *__restrict__ frames, int i, int s, const float *__restrict__ rho,
                           float *__restrict__ gh)
{
    const FrameDev fr = frames[i];
    const int pix = blockIdx.x * blockDim.x + threadIdx.x;
    if (pix >= fr.F * fr.F) return;
    const int y = pix / fr.F, x = pix % fr.F;
    gh[fr.fine_off + pix] = rho[fr.data_off + (long long)(y / s) * fr.n + x / s];
}

hipError_t launch_plain_frame_ops(hipStream_t st, int op, const FrameDev *fr, int i, int n, int F, int s,
                                  const float *a, const float *data, const float *invvar, float *out,
                                  double *part)
{
    if (op == 0)
        hipLaunchKernelGGL(k_block_sum, dim3((n * n + 255) / 256), dim3(256), 0, st, fr, i, s, a, out);
    else if (op == 1)
        hipLaunchKernelGGL(k_resid, dim3((n * n + 255) / 256), dim3(256), 0, st, fr, i, a, data, invvar, out, part);
    else
        hipLaunchKernelGGL(k_upsample, dim3((F * F + 255) / 256), dim3(256), 0, st, fr, i, s, a, out);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Register-blocked correlation row: acc[j] += sum_{t < T} tap[t] * pl[j + t],
// j = 0..3, with pl 16-byte aligned in LDS and tap wave-uniform.
// --------------------------------------------------------------------------

__device__ __forceinline__ void corr_row4(const float *__restrict__ pl, const float *__restrict__ tap,
                                          int T, float (&acc)[4])
{
    float4 w0 = *reinterpret_cast<const float4 *>(pl);
    for (int t = 0; t < T; t += 4) {
        const float4 w1 = *reinterpret_cast<const float4 *>(pl + t + 4);
        const float k0 = tap[t], k1 = tap[t + 1], k2 = tap[t + 2], k3 = tap[t + 3];
        acc[0] = fmaf(k0, w0.x, acc[0]);
        acc[1] = fmaf(k0, w0.y, acc[1]);
        acc[2] = fmaf(k0, w0.z, acc[2]);
        acc[3] = fmaf(k0, w0.w, acc[3]);
        acc[0] = fmaf(k1, w0.y, acc[0]);
        acc[1] = fmaf(k1, w0.z, acc[1]);
        acc[2] = fmaf(k1, w0.w, acc[2]);
        acc[3] = fmaf(k1, w1.x, acc[3]);
        acc[0] = fmaf(k2, w0.z, acc[0]);
        acc[1] = fmaf(k2, w0.w, acc[1]);
        acc[2] = fmaf(k2, w1.x, acc[2]);
        acc[3] = fmaf(k2, w1.y, acc[3]);
        acc[0] = fmaf(k3, w0.w, acc[0]);
        acc[1] = fmaf(k3, w1.x, acc[1]);
        acc[2] = fmaf(k3, w1.y, acc[2]);
        acc[3] = fmaf(k3, w1.z, acc[3]);
        w0 = w1;
    }
}

// --------------------------------------------------------------------------
// a2 + a3 + a4: fused S_i, D, residual and chi-square partials (direct)
// --------------------------------------------------------------------------
//
// One work group per (frame, 16 x 32 data-pixel tile). The scene region the
// tile needs is staged in LDS, split into s column planes so that every
// residue class of kernel columns reads consecutive floats; kernel rows are
// streamed in chunks of kFwdCA.
template <int S, bool RESID>
__global__ __launch_bounds__(kFwdThreads) void k_fwd_direct(
    const FrameDev *__restrict__ frames, const Item *__restrict__ items,
    const float *__restrict__ scene, const float *__restrict__ kf, const float *__restrict__ data,
    const float *__restrict__ invvar, float *__restrict__ out, double *__restrict__ part_chi, int n_items)
{
    extern __shared__ float4 lds4[];
    float *lds = reinterpret_cast<float *>(lds4);
    __shared__ double red[kFwdThreads / 64];
    // persistent: the grid walks the (longest-first) item list
    for (int b = blockIdx.x; b < n_items; b += gridDim.x) {
    const Item it = items[b];
    const FrameDev fr = frames[it.frame];
    const int tid = threadIdx.x;
    constexpr int NTX = kFwdTQ / 4;
    const int tx = tid % NTX, ty = tid / NTX;
    const int Kp = fr.Kp, F = fr.F, T = fr.Tpad;
    const int PW = kFwdTQ + T;  // floats per plane row
    const int RW = S * PW;      // floats per region row
    constexpr int ROWS = S * (kFwdTP - 1) + kFwdCA;
    const int A0 = fr.cp - (Kp - 1);
    const int rowF0 = S * it.p0 + A0;
    const int colF0 = S * it.q0 + A0;
    const float *scn = scene + fr.fine_off;
    const float *kfr = kf + fr.kf_off;

    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int a0 = 0; a0 < Kp; a0 += kFwdCA) {
        __syncthreads();
        const int tot = ROWS * RW;
        for (int e = tid; e < tot; e += kFwdThreads) {
            const int r = e / RW, c = e - r * RW;
            const int yy = rowF0 + a0 + r, xx = colF0 + c;
            float v = 0.f;
            if (yy >= 0 && yy < F && xx >= 0 && xx < F) v = scn[yy * F + xx];
            lds[r * RW + (c % S) * PW + c / S] = v;
        }
        __syncthreads();
        const int na = min(kFwdCA, Kp - a0);
        for (int a = 0; a < na; ++a) {
            float racc[4] = {0.f, 0.f, 0.f, 0.f};
            const float *lrow = lds + (S * ty + a) * RW + 4 * tx;
            const float *krow = kfr + (long long)(a0 + a) * S * T;
            #pragma unroll
            for (int psi = 0; psi < S; ++psi) corr_row4(lrow + psi * PW, krow + psi * T, T, racc);
            #pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] += racc[j];
        }
    }

    const int p = it.p0 + ty;
    double chi = 0.0;
    #pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int q = it.q0 + 4 * tx + j;
        if (p < fr.n && q < fr.n) {
            const long long idx = fr.data_off + (long long)p * fr.n + q;
            if (RESID) {
                const float r = acc[j] - data[idx];
                const float w = invvar[idx];
                out[idx] = w * r;
                chi += 0.5 * (double)w * (double)r * (double)r;
            } else {
                out[idx] = acc[j];
            }
        }
    }
    if (RESID) {
        const double tot = block_sum_d<kFwdThreads>(chi, red);
        if (tid == 0) part_chi[it.slot] = tot;
    }
    }
}

size_t fwd_lds_bytes(int s, int Tmax) { return (size_t)(s * (kFwdTP - 1) + kFwdCA) * s * (kFwdTQ + Tmax) * 4; }

int device_cus()
{
    static int n = 0;
    if (n <= 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
    }
    return n;
}

int direct_fwd_groups(int s, int Tmax)
{
    int per = 0;
    const size_t lds = fwd_lds_bytes(s, Tmax);
    hipError_t e = hipErrorInvalidValue;
    if (s == 1) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_fwd_direct<1, true>, kFwdThreads, lds);
    if (s == 2) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_fwd_direct<2, true>, kFwdThreads, lds);
    if (s == 3) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_fwd_direct<3, true>, kFwdThreads, lds);
    if (e != hipSuccess || per < 1) per = 1;
    return per * device_cus();
}

hipError_t launch_fwd_direct(hipStream_t st, int s, const FrameDev *fr, const Item *items,
                             int n_items, int Tmax, const float *scene, const float *kf,
                             const float *data, const float *invvar, float *out, double *part_chi, int groups)
{
    if (n_items <= 0) return hipSuccess;
    const size_t lds = fwd_lds_bytes(s, Tmax);
    const bool resid = (part_chi != nullptr);
    const int grid = (groups > 0 && groups < n_items) ? groups : n_items;
#define FWD_CASE(SS)                                                                               \
    if (s == SS) {                                                                                 \
        if (resid)                                                                                 \
            hipLaunchKernelGGL((k_fwd_direct<SS, true>), dim3(grid), dim3(kFwdThreads), lds, st,    \
                               fr, items, scene, kf, data, invvar, out, part_chi, n_items);        \
        else                                                                                       \
            hipLaunchKernelGGL((k_fwd_direct<SS, false>), dim3(grid), dim3(kFwdThreads), lds,      \
                               st, fr, items, scene, kf, data, invvar, out, part_chi, n_items);    \
        return hipGetLastError();                                                                  \
    }
    FWD_CASE(1)
    FWD_CASE(2)
    FWD_CASE(3)
#undef FWD_CASE
    return hipErrorInvalidValue;
}

// --------------------------------------------------------------------------
// a5: adjoint g_i = S_i^T D^T rho_i, phase by phase (direct)
// --------------------------------------------------------------------------
//
// One work group per (frame, 16 x 32 coarse tile); each of the s^2 phases is a
// stride-1 correlation of rho with the phase kernel, producing the fine pixels
// (s P + py, s Q + px).
template <int S>
__global__ __launch_bounds__(kAdjThreads) void k_adj_direct(
    const FrameDev *__restrict__ frames, const Item *__restrict__ items,
    const float *__restrict__ rho, const float *__restrict__ ka, float *__restrict__ g, int n_items)
{
    extern __shared__ float4 lds4[];
    float *lds = reinterpret_cast<float *>(lds4);
    // persistent: the grid walks the (longest-first) item list
    for (int b = blockIdx.x; b < n_items; b += gridDim.x) {
    if (b != (int)blockIdx.x) __syncthreads();  // the previous item's reads of the tile are done
    const Item it = items[b];
    const FrameDev fr = frames[it.frame];
    const int tid = threadIdx.x;
    constexpr int NTX = kAdjTQ / 4;
    const int tx = tid % NTX, ty = tid / NTX;
    const int n = fr.n, Ar = fr.Ar, Bp = fr.Bpad;
    const int PW = kAdjTQ + Bp;
    const int rows = kAdjTP - 1 + Ar;
    const int r0 = it.p0 + fr.dmin, c0 = it.q0 + fr.dmin;
    const float *rh = rho + fr.data_off;
    for (int e = tid; e < rows * PW; e += kAdjThreads) {
        const int r = e / PW, c = e - r * PW;
        const int yy = r0 + r, xx = c0 + c;
        float v = 0.f;
        if (yy >= 0 && yy < n && xx >= 0 && xx < n) v = rh[yy * n + xx];
        lds[e] = v;
    }
    __syncthreads();
    const int P = it.p0 + ty;
    const float *kfr = ka + fr.ka_off;
    float *gf = g + fr.fine_off;
    for (int py = 0; py < S; ++py)
        for (int px = 0; px < S; ++px) {
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
            const float *kph = kfr + (long long)(py * S + px) * Ar * Bp;
            for (int al = 0; al < Ar; ++al) {
                float racc[4] = {0.f, 0.f, 0.f, 0.f};
                corr_row4(lds + (ty + al) * PW + 4 * tx, kph + (long long)al * Bp, Bp, racc);
                #pragma unroll
                for (int j = 0; j < 4; ++j) acc[j] += racc[j];
            }
            if (P < n) {
                #pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int Q = it.q0 + 4 * tx + j;
                    if (Q < n) gf[(long long)(S * P + py) * fr.F + S * Q + px] = acc[j];
                }
            }
        }
    }
}

size_t adj_lds_bytes(int Ar_max, int Bpad_max) { return (size_t)(kAdjTP - 1 + Ar_max) * (kAdjTQ + Bpad_max) * 4; }

int direct_adj_groups(int s, int Ar_max, int Bpad_max)
{
    int per = 0;
    const size_t lds = adj_lds_bytes(Ar_max, Bpad_max);
    hipError_t e = hipErrorInvalidValue;
    if (s == 1) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_adj_direct<1>, kAdjThreads, lds);
    if (s == 2) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_adj_direct<2>, kAdjThreads, lds);
    if (s == 3) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_adj_direct<3>, kAdjThreads, lds);
    if (e != hipSuccess || per < 1) per = 1;
    return per * device_cus();
}

hipError_t launch_adj_direct(hipStream_t st, int s, const FrameDev *fr, const Item *items,
                             int n_items, int Ar_max, int Bpad_max, const float *rho,
                             const float *ka, float *g, int groups)
{
    if (n_items <= 0) return hipSuccess;
    const size_t lds = adj_lds_bytes(Ar_max, Bpad_max);
    const int grid = (groups > 0 && groups < n_items) ? groups : n_items;
    if (s == 1)
        hipLaunchKernelGGL(k_adj_direct<1>, dim3(grid), dim3(kAdjThreads), lds, st, fr, items, rho, ka, g, n_items);
    else if (s == 2)
        hipLaunchKernelGGL(k_adj_direct<2>, dim3(grid), dim3(kAdjThreads), lds, st, fr, items, rho, ka, g, n_items);
    else if (s == 3)
        hipLaunchKernelGGL(k_adj_direct<3>, dim3(grid), dim3(kAdjThreads), lds, st, fr, items, rho, ka, g, n_items);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// a5: per-frame gradient sums. Block (i, 0): dL/dGamma_i = sum g_i.
// Block (i, 1+k): <g_i, r_k>, <g_i, r_k (X-cx)/sigma^2>, <g_i, r_k (Y-cy)/sigma^2>
// over the +-8 px window of source k.  fsum[i][1+3M].
// --------------------------------------------------------------------------

constexpr int kSumThreads = 256;
constexpr int kSumThreadsXf = 1024;
constexpr int kXfSplit = 4;  // blocks per frame for the transform's gradient (partials added in order)

// Frame sums under a per-frame transform: block 0 dL/dGamma_i; block 1+k the sums of
// g r_k(u) and g r_k(u) (u - c_k)/sigma^2 (scene coordinates u, so dL/dc_k needs no
// rotation); blocks 1+M.. (kXfSplit of them, when gxf is given) dL/d(dx_i, dy_i, theta_i) from
// q(X) = grad h(u) - sum_k a_ik r_k(u) (u - c_k)/sigma^2:  <g, q> and
// <g, q . R'(theta)(X - C)>.
template <int NT>
__device__ void frame_sums_xf(const FrameDev &fr, int i, int by, int E, int N, int M, float sigma,
                              const float *__restrict__ params, const float *__restrict__ gi,
                              double *__restrict__ fsum, const float *__restrict__ xf, double *__restrict__ gxfp,
                              double *red)
{
    const int stride = 1 + 3 * M;
    const int tot = fr.F * fr.F;
    const float *h = params;
    const float *a = params + (long long)N * N + E;
    const float *c = a + (long long)E * M;
    const float inv2s2 = 1.0f / (2.0f * sigma * sigma);
    const float invs2 = 1.0f / (sigma * sigma);
    const float norm = 1.0f / (2.0f * 3.14159265358979f * sigma * sigma);
    __shared__ FrameMap fm;
    if (threadIdx.x == 0) fm = FrameMap(xf, i, N);
    __syncthreads();
    if (by == 0) {
        double acc = 0.0;
        for (int p = threadIdx.x; p < tot; p += NT) acc += (double)gi[p];
        const double sm = block_sum_d<NT>(acc, red);
        if (threadIdx.x == 0) fsum[(long long)i * stride] = sm;
        return;
    }
    if (by <= M) {
        const int k = by - 1;
        const float cx = c[2 * k], cy = c[2 * k + 1];
        // the source's box |u - c| <= R in frame coordinates: around the preimage of
        // c, within R sqrt(2) (+1) on each axis
        const double ex = cx - fm.C - fm.dx, ey = cy - fm.C - fm.dy;
        const double px = fm.cs * ex + fm.sn * ey + fm.C, py = -fm.sn * ex + fm.cs * ey + fm.C;
        const double rad = (double)kGaussRadius * 1.4143 + 1.0;
        const int x_lo = max(fr.o, (int)floor(px - rad)), x_hi = min(fr.o + fr.F - 1, (int)ceil(px + rad));
        const int y_lo = max(fr.o, (int)floor(py - rad)), y_hi = min(fr.o + fr.F - 1, (int)ceil(py + rad));
        const int wx = x_hi - x_lo + 1, wy = y_hi - y_lo + 1;
        double sa = 0.0, sx = 0.0, sy = 0.0;
        if (wx > 0 && wy > 0) {
            for (int e = threadIdx.x; e < wx * wy; e += NT) {
                const int Y = y_lo + e / wx, X = x_lo + e % wx;
                double ux, uy;
                fm.map((double)X, (double)Y, ux, uy);
                const float dx = (float)(ux - (double)cx), dy = (float)(uy - (double)cy);
                if (fabsf(dx) > (float)kGaussRadius || fabsf(dy) > (float)kGaussRadius) continue;
                const float r = norm * expf(-(dx * dx + dy * dy) * inv2s2);
                const float gr = gi[(long long)(Y - fr.o) * fr.F + (X - fr.o)] * r;
                sa += (double)gr;
                sx += (double)(gr * dx * invs2);
                sy += (double)(gr * dy * invs2);
            }
        }
        sa = block_sum_d<NT>(sa, red);
        sx = block_sum_d<NT>(sx, red);
        sy = block_sum_d<NT>(sy, red);
        if (threadIdx.x == 0) {
            fsum[(long long)i * stride + 1 + k] = sa;
            fsum[(long long)i * stride + 1 + M + k] = sx;
            fsum[(long long)i * stride + 1 + 2 * M + k] = sy;
        }
        return;
    }
    // by == 1 + M + sp: the transform's gradient over the frame's pixels sp, sp + NS, ...
    // (in strides of NT), as partials gxfp[i][sp][3] that k_xf_grad_sum adds in order
    const int sp = by - 1 - M;
    double gdx = 0.0, gdy = 0.0, gth = 0.0;
    for (int p = sp * NT + threadIdx.x; p < tot; p += kXfSplit * NT) {
        const double X = (double)(fr.o + p % fr.F), Y = (double)(fr.o + p / fr.F);
        double ux, uy;
        float qx, qy;
        fm.map(X, Y, ux, uy);
        bilerp(h, N, ux, uy, &qx, &qy);
        for (int k = 0; k < M; ++k) {
            const float dx = (float)(ux - (double)c[2 * k]), dy = (float)(uy - (double)c[2 * k + 1]);
            if (fabsf(dx) <= (float)kGaussRadius && fabsf(dy) <= (float)kGaussRadius) {
                const float ar = a[(long long)i * M + k] * norm * expf(-(dx * dx + dy * dy) * inv2s2) * invs2;
                qx -= ar * dx;
                qy -= ar * dy;
            }
        }
        const float gv = gi[p];
        const float vx = (float)(X - fm.C), vy = (float)(Y - fm.C);
        const float cs = (float)fm.cs, sn = (float)fm.sn;
        gdx += (double)(gv * qx);
        gdy += (double)(gv * qy);
        gth += (double)(gv * (qx * (-sn * vx - cs * vy) + qy * (cs * vx - sn * vy)));
    }
    gdx = block_sum_d<NT>(gdx, red);
    gdy = block_sum_d<NT>(gdy, red);
    gth = block_sum_d<NT>(gth, red);
    if (threadIdx.x == 0) {
        double *o = gxfp + ((long long)i * kXfSplit + sp) * 3;
        o[0] = gdx;
        o[1] = gdy;
        o[2] = gth;
    }
}

// dL/d(dx_i, dy_i, theta_i) = the sum of frame i's kXfSplit partials, in order
__global__ void k_xf_grad_sum(int nf, const int *__restrict__ flist, const double *__restrict__ gxfp,
                              float *__restrict__ gxf)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nf * 3) return;
    const int q = e / 3, c = e - 3 * q;
    const int i = flist ? flist[q] : q;
    double acc = 0.0;
    for (int sp = 0; sp < kXfSplit; ++sp) acc += gxfp[((long long)i * kXfSplit + sp) * 3 + c];
    gxf[3 * i + c] = (float)acc;
}

// NT threads per block: kSumThreads, or kSumThreadsXf for frames under transforms
// (whose blocks map and interpolate every pixel: more waves to hide the loads)
template <int NT>
__global__ __launch_bounds__(NT) void k_frame_sums(
    const FrameDev *__restrict__ frames, int E, int frame0, int N, int M, float sigma,
    const float *__restrict__ params, const float *__restrict__ g, double *__restrict__ fsum, int yofs,
    const int *__restrict__ flist, const float *__restrict__ xf, double *__restrict__ gxfp)
{
    __shared__ double red[NT / 64];
    const int i = flist ? flist[blockIdx.x] : frame0 + blockIdx.x;
    const int by = blockIdx.y + yofs;  // yofs = 1: the frame sums of g come from elsewhere
    const FrameDev fr = frames[i];
    const float *gi = g + fr.fine_off;
    const int stride = 1 + 3 * M;
    if (xf) {
        frame_sums_xf<NT>(fr, i, by, E, N, M, sigma, params, gi, fsum, xf, gxfp, red);
        return;
    }
    if (by == 0) {
        double acc = 0.0;
        const int tot = fr.F * fr.F;
        for (int p = threadIdx.x; p < tot; p += NT) acc += (double)gi[p];
        const double s = block_sum_d<NT>(acc, red);
        if (threadIdx.x == 0) fsum[(long long)i * stride] = s;
        return;
    }
    const int k = by - 1;
    const float *c = params + (long long)N * N + E + (long long)E * M;
    const float cx = c[2 * k], cy = c[2 * k + 1];
    const float inv2s2 = 1.0f / (2.0f * sigma * sigma);
    const float invs2 = 1.0f / (sigma * sigma);
    const float norm = 1.0f / (2.0f * 3.14159265358979f * sigma * sigma);
    const int x_lo = max(fr.o, (int)ceilf(cx - kGaussRadius)), x_hi = min(fr.o + fr.F - 1, (int)floorf(cx + kGaussRadius));
    const int y_lo = max(fr.o, (int)ceilf(cy - kGaussRadius)), y_hi = min(fr.o + fr.F - 1, (int)floorf(cy + kGaussRadius));
    const int wx = x_hi - x_lo + 1, wy = y_hi - y_lo + 1;
    double sa = 0.0, sx = 0.0, sy = 0.0;
    if (wx > 0 && wy > 0) {
        for (int e = threadIdx.x; e < wx * wy; e += NT) {
            const int Y = y_lo + e / wx, X = x_lo + e % wx;
            const float dx = (float)X - cx, dy = (float)Y - cy;
            const float r = norm * expf(-(dx * dx + dy * dy) * inv2s2);
            const float gv = gi[(long long)(Y - fr.o) * fr.F + (X - fr.o)];
            const float gr = gv * r;
            sa += (double)gr;
            sx += (double)(gr * dx * invs2);
            sy += (double)(gr * dy * invs2);
        }
    }
    sa = block_sum_d<NT>(sa, red);
    sx = block_sum_d<NT>(sx, red);
    sy = block_sum_d<NT>(sy, red);
    if (threadIdx.x == 0) {
        fsum[(long long)i * stride + 1 + k] = sa;
        fsum[(long long)i * stride + 1 + M + k] = sx;
        fsum[(long long)i * stride + 1 + 2 * M + k] = sy;
    }
}

hipError_t launch_frame_sums(hipStream_t st, const FrameDev *fr, int E, int N, int M, float sigma,
                             const float *params, const float *g, double *fsum, bool with_gamma,
                             const int *flist, int nlist, const float *xf, float *gxf, double *gxfp)
{
    const int nf = flist ? nlist : E;
    if (nf <= 0) return hipSuccess;
    const int yofs = with_gamma ? 0 : 1;
    const bool xgrad = xf && gxf && gxfp;
    const int ny = 1 + M - yofs + (xgrad ? kXfSplit : 0);  // + the transform's gradient blocks
    if (ny <= 0) return hipSuccess;
    if (xf) {
        hipLaunchKernelGGL(k_frame_sums<kSumThreadsXf>, dim3(nf, ny), dim3(kSumThreadsXf), 0, st, fr, E, 0, N, M,
                           sigma, params, g, fsum, yofs, flist, xf, xgrad ? gxfp : nullptr);
        if (xgrad)
            hipLaunchKernelGGL(k_xf_grad_sum, dim3((nf * 3 + 255) / 256), dim3(256), 0, st, nf, flist, gxfp, gxf);
    } else {
        hipLaunchKernelGGL(k_frame_sums<kSumThreads>, dim3(nf, ny), dim3(kSumThreads), 0, st, fr, E, 0, N, M,
                           sigma, params, g, fsum, yofs, flist, xf, nullptr);
    }
    return hipGetLastError();
}

int xf_grad_parts(int E) { return E * kXfSplit * 3; }

hipError_t launch_frame_sums_one(hipStream_t st, const FrameDev *fr, int E, int i, int N, int M, float sigma,
                                 const float *params, const float *g, double *fsum)
{
    hipLaunchKernelGGL(k_frame_sums<kSumThreads>, dim3(1, 1 + M), dim3(kSumThreads), 0, st, fr, E, i, N, M,
                       sigma, params, g, fsum, 0, nullptr, nullptr, nullptr);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// dL/dh = Phi z + sum over frames covering the pixel of g_i (frame order)
// --------------------------------------------------------------------------

constexpr int kFinChunk = 16;   // frames summed by one thread of k_finalize_h_part
constexpr int kFinChunkXf = 4;  // the same for frames under transforms (25 candidates each)

// Two-stage cross-frame sum (frame order within a chunk, then chunk order):
// part[c][Y,X] = sum over frames of chunk c covering (Y,X) of g_i(Y - o_i, X - o_i)
// Transpose of the bilinear read of frame i at grid pixel (PX, PY): the sum of
// g_i(X) times the weight with which frame pixel X read h there, over the frame
// pixels whose transformed position lies within one pixel of (PX, PY) on both axes
// (a gather in a fixed order: the candidates around the preimage of the pixel). Bound by the
// candidates' arithmetic: the weights come from the distances, and a block's frame maps (a sine
// and cosine each) are formed once in LDS; loss and gradient of 100 shifted frames of 64^2
// 217 -> 197 us.
__device__ float transpose_bilerp(const FrameDev &fr, const FrameMap &fm, const float *__restrict__ g, int PX, int PY)
{
    const double ex = (double)PX - fm.C - fm.dx, ey = (double)PY - fm.C - fm.dy;
    const double px = fm.cs * ex + fm.sn * ey + fm.C, py = -fm.sn * ex + fm.cs * ey + fm.C;
    // a frame pixel X reads (PX, PY) when its image u lies in [PX - 1, PX + 1) on both
    // axes, so X - p is the inverse rotation of a vector with components in [-1, 1):
    // within |cos| + |sin| (<= sqrt 2) of p on each axis, at most three candidates each
    const double w = fabs(fm.cs) + fabs(fm.sn) + 1e-9;
    const int xlo = (int)ceil(px - w), xhi = (int)floor(px + w);
    const int ylo = (int)ceil(py - w), yhi = (int)floor(py + w);
    const float *gi = g + fr.fine_off;
    float acc = 0.f;
    for (int Y = ylo; Y <= yhi; ++Y) {
        const int y = Y - fr.o;
        if (y < 0 || y >= fr.F) continue;
        // distances of the row's candidates from the pixel: a step in X moves them by (cos, sin)
        double dx, dy;
        fm.map((double)xlo, (double)Y, dx, dy);
        dx -= (double)PX;
        dy -= (double)PY;
        for (int X = xlo; X <= xhi; ++X, dx += fm.cs, dy += fm.sn) {
            const int x = X - fr.o;
            // the corner weights of the read: 1 - distance, nothing from a pixel away on
            const double wx = 1.0 - fabs(dx), wy = 1.0 - fabs(dy);
            if (x < 0 || x >= fr.F || !(wx > 0.0) || !(wy > 0.0)) continue;
            acc += gi[(long long)y * fr.F + x] * ((float)wx * (float)wy);
        }
    }
    return acc;
}

__global__ void k_finalize_h_part(const FrameDev *__restrict__ frames, int E, int N,
                                  const float *__restrict__ g, float *__restrict__ part,
                                  const int *__restrict__ flist, const float *__restrict__ xf)
{
    const int pix = blockIdx.x * blockDim.x + threadIdx.x;
    const int chunk = xf ? kFinChunkXf : kFinChunk;
    const int i0 = blockIdx.y * chunk, i1 = min(E, i0 + chunk);
    __shared__ FrameMap fm[kFinChunkXf];
    if (xf) {
        if ((int)threadIdx.x < i1 - i0) fm[threadIdx.x] = FrameMap(xf, flist ? flist[i0 + threadIdx.x] : i0 + threadIdx.x, N);
        __syncthreads();
    }
    if (pix >= N * N) return;
    const int Y = pix / N, X = pix % N;
    float acc = 0.f;
    if (xf) {
        for (int q = i0; q < i1; ++q) {
            const int i = flist ? flist[q] : q;
            acc += transpose_bilerp(frames[i], fm[q - i0], g, X, Y);
        }
        part[(long long)blockIdx.y * N * N + pix] = acc;
        return;
    }
    for (int q = i0; q < i1; ++q) {
        const int i = flist ? flist[q] : q;
        const int o = frames[i].o, F = frames[i].F;
        const int y = Y - o, x = X - o;
        if (y >= 0 && y < F && x >= 0 && x < F) acc += g[frames[i].fine_off + (long long)y * F + x];
    }
    part[(long long)blockIdx.y * N * N + pix] = acc;
}

// dL/dh = Phi z + sum of the chunk partials
__global__ void k_finalize_h_sum(int nchunk, int N, const float *__restrict__ part,
                                 const float *__restrict__ prior, float *__restrict__ grad_h)
{
    const int pix = blockIdx.x * blockDim.x + threadIdx.x;
    if (pix >= N * N) return;
    float acc = prior ? prior[pix] : 0.f;
    #pragma unroll 8
    for (int c = 0; c < nchunk; ++c) acc += part[(long long)c * N * N + pix];
    grad_h[pix] = acc;
}

// partial planes the chunked sum needs (frames under transforms take smaller chunks)
int finalize_h_chunks(int E, bool xf)
{
    const int chunk = xf ? kFinChunkXf : kFinChunk;
    return (E + chunk - 1) / chunk;
}

hipError_t launch_finalize_h(hipStream_t st, const FrameDev *fr, int E, int N, const float *g,
                             const float *prior, float *grad_h, float *part, const int *flist, int nlist,
                             const float *xf)
{
    const int nb = (N * N + 255) / 256;
    const int nf = flist ? nlist : E;
    const int nc = finalize_h_chunks(nf, xf != nullptr);
    hipLaunchKernelGGL(k_finalize_h_part, dim3(nb, nc), dim3(256), 0, st, fr, nf, N, g, part, flist, xf);
    hipLaunchKernelGGL(k_finalize_h_sum, dim3(nb), dim3(256), 0, st, nc, N, part, prior, grad_h);
    return hipGetLastError();
}

// Block 0: the small reductions and updates (finalize_small_body). When classes
// is given, blocks 1.. assemble dL/dh of the FFT path: the prior gradient plus the
// window contribution of every shape class, in class order (and update h).
constexpr int kFinThreads = 1024;

// psum.U (or null): the prior's gradient summed per pixel from its per-level planes (its
// passes rode in the step's launches) instead of read from prior
__global__ __launch_bounds__(kFinThreads) void k_finalize_small(FinalArgs fa, const ClassFft *__restrict__ classes,
                                                                int ncls, const float *__restrict__ hcls,
                                                                const float *__restrict__ prior, DenseStar psum)
{
    if (blockIdx.x == 0) {
        finalize_small_body<kFinThreads>(fa);
        return;
    }
    const int N = fa.N;
    const long long NN = (long long)N * N;
    const long long pix = (long long)(blockIdx.x - 1) * kFinThreads + threadIdx.x;
    if (pix >= NN) return;
    float bc1, bc2;
    adam_bias(fa.adam, bc1, bc2);
    const int Y = (int)(pix / N), X = (int)(pix % N);
    float acc = psum.U ? (float)dense_prior_at(psum, pix) : (prior ? prior[pix] : 0.f);
    for (int ci = 0; ci < ncls; ++ci) {
        const ClassFft &c = classes[ci];
        if (c.direct) continue;  // its frames' windows are in prior (the direct path's sum)
        const int y = Y - c.o, x = X - c.o, F = c.F;
        if (y >= 0 && y < F && x >= 0 && x < F) acc += hcls[c.hc_off + (long long)y * F + x];
    }
    finalize_h_pixel(fa.adam, bc1, bc2, pix, acc, fa.grad);
}

hipError_t launch_finalize_small(hipStream_t st, int E, int M, int n_chi, const double *part_chi,
                                 int n_l1, const double *part_l1, double,
                                 const double *fsum, const float *params, int N,
                                 float *grad, double *loss, int *tick, const ClassFft *classes, int ncls,
                                 const float *hcls, const float *prior, const AdamDev &adam, const double *pts,
                                 const DenseStar *psum)
{
    const long long NN = (long long)N * N;
    const int hblocks = (classes && grad) ? (int)((NN + kFinThreads - 1) / kFinThreads) : 0;
    // a fused Adam update needs the h blocks (FFT path) and the gradient
    if (adam.params && (!hblocks || !grad)) return hipErrorInvalidValue;
    FinalArgs fa;
    fa.E = E;
    fa.M = M;
    fa.N = N;
    fa.n_chi = n_chi;
    fa.n_l1 = n_l1;
    fa.part_chi = part_chi;
    fa.part_l1 = part_l1;
    fa.fsum = fsum;
    fa.params = params;
    fa.grad = grad;
    fa.loss = loss;
    fa.tick = tick;
    fa.adam = adam;
    fa.pts = pts;
    hipLaunchKernelGGL(k_finalize_small, dim3(1 + hblocks), dim3(kFinThreads), 0, st, fa, classes, ncls, hcls, prior,
                       psum ? *psum : DenseStar());
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Eq. 11, third term: the point-source image P = sum_k <a_k> r_k on the h grid
// (r_k within +-kGaussRadius of c_k, as in the scene) and the dot products that
// carry its prior's gradient to a and c.
// --------------------------------------------------------------------------

// P_out = P; <a_k> per work group
__global__ __launch_bounds__(256) void k_pts_render(int N, int E, int M, float sigma, const float *__restrict__ params,
                                                     float *__restrict__ P_out)
{
    extern __shared__ float am[];  // <a_k>
    const long long NN = (long long)N * N;
    const float *a = params + NN + E, *c = a + (long long)E * M;
    for (int k = threadIdx.x; k < M; k += blockDim.x) {
        double acc = 0.0;
        for (int i = 0; i < E; ++i) acc += a[(long long)i * M + k];
        am[k] = (float)(acc / E);
    }
    __syncthreads();
    const long long pix = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (pix >= NN) return;
    const int Y = (int)(pix / N), X = (int)(pix % N);
    const float inv2s2 = 1.0f / (2.0f * sigma * sigma), norm = 1.0f / (6.28318530717958647692f * sigma * sigma);
    float v = 0.f;
    for (int k = 0; k < M; ++k) {
        const float dx = (float)X - c[2 * k], dy = (float)Y - c[2 * k + 1];
        if (fabsf(dx) <= kGaussRadius && fabsf(dy) <= kGaussRadius) v += am[k] * norm * expf(-(dx * dx + dy * dy) * inv2s2);
    }
    P_out[pix] = v;
}

hipError_t launch_pts_render(hipStream_t st, int N, int E, int M, float sigma, const float *params,
                             float *P_out)
{
    const long long NN = (long long)N * N;
    hipLaunchKernelGGL(k_pts_render, dim3((unsigned)((NN + 255) / 256)), dim3(256), sizeof(float) * (M > 0 ? M : 1),
                       st, N, E, M, sigma, params, P_out);
    return hipGetLastError();
}

// one work group per source k over the +-kGaussRadius window of r_k, with q = Phi z_P:
// pts[3k] = <q, r_k> / E (added to every dL/da_ik), pts[3k+1..2] = <a_k> <q, dr_k/dc_k>
__global__ __launch_bounds__(256) void k_pts_dots(int N, int E, int M, float sigma, const float *__restrict__ params,
                                                   const float *__restrict__ q, double *__restrict__ pts)
{
    __shared__ double red[256 / 64];
    const int k = blockIdx.x;
    const long long NN = (long long)N * N;
    const float *a = params + NN + E, *c = a + (long long)E * M;
    const float cx = c[2 * k], cy = c[2 * k + 1];
    const int x0 = max(0, (int)ceilf(cx - kGaussRadius)), x1 = min(N - 1, (int)floorf(cx + kGaussRadius));
    const int y0 = max(0, (int)ceilf(cy - kGaussRadius)), y1 = min(N - 1, (int)floorf(cy + kGaussRadius));
    const int w = max(0, x1 - x0 + 1), h = max(0, y1 - y0 + 1);
    const double inv2s2 = 1.0 / (2.0 * (double)sigma * sigma), invs2 = 1.0 / ((double)sigma * sigma);
    const double norm = 1.0 / (6.283185307179586477 * (double)sigma * sigma);
    double sa = 0.0, sx = 0.0, sy = 0.0;
    for (int e = threadIdx.x; e < w * h; e += blockDim.x) {
        const int Y = y0 + e / w, X = x0 + e % w;
        const double dx = (double)X - cx, dy = (double)Y - cy;
        const double r = norm * exp(-(dx * dx + dy * dy) * inv2s2);
        const double qv = q[(long long)Y * N + X];
        sa += qv * r;
        sx += qv * r * dx * invs2;
        sy += qv * r * dy * invs2;
    }
    sa = block_sum_d<256>(sa, red);
    sx = block_sum_d<256>(sx, red);
    sy = block_sum_d<256>(sy, red);
    if (threadIdx.x == 0) {
        double am = 0.0;
        for (int i = 0; i < E; ++i) am += a[(long long)i * M + k];
        am /= E;
        pts[3 * k] = sa / E;
        pts[3 * k + 1] = am * sx;
        pts[3 * k + 2] = am * sy;
    }
}

hipError_t launch_pts_dots(hipStream_t st, int N, int E, int M, float sigma, const float *params, const float *q,
                           double *pts)
{
    if (M <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pts_dots, dim3(M), dim3(256), 0, st, N, E, M, sigma, params, q, pts);
    return hipGetLastError();
}

// App. C images: out[0] = <Gamma> + h + sum_k <a_k> r_k (the epoch average of the
// scene on the h grid), out[1] = h, out[2 + k] = r_k; <a_k>, <Gamma> per work group
__global__ __launch_bounds__(256) void k_pts_images(int N, int E, int M, float sigma, const float *__restrict__ params,
                                                     float *__restrict__ out)
{
    extern __shared__ float am[];  // <a_k>, then <Gamma>
    const long long NN = (long long)N * N;
    const float *G = params + NN, *a = G + E, *c = a + (long long)E * M;
    for (int k = threadIdx.x; k <= M; k += blockDim.x) {
        double acc = 0.0;
        for (int i = 0; i < E; ++i) acc += (k < M) ? a[(long long)i * M + k] : G[i];
        am[k] = (float)(acc / E);
    }
    __syncthreads();
    const long long pix = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (pix >= NN) return;
    const int Y = (int)(pix / N), X = (int)(pix % N);
    const float inv2s2 = 1.0f / (2.0f * sigma * sigma), norm = 1.0f / (6.28318530717958647692f * sigma * sigma);
    float f = am[M] + params[pix];
    for (int k = 0; k < M; ++k) {
        const float dx = (float)X - c[2 * k], dy = (float)Y - c[2 * k + 1];
        float r = 0.f;
        if (fabsf(dx) <= kGaussRadius && fabsf(dy) <= kGaussRadius) r = norm * expf(-(dx * dx + dy * dy) * inv2s2);
        out[(2 + k) * NN + pix] = r;
        f += am[k] * r;
    }
    out[pix] = f;
    out[NN + pix] = params[pix];
}

hipError_t launch_pts_images(hipStream_t st, int N, int E, int M, float sigma, const float *params, float *out)
{
    const long long NN = (long long)N * N;
    hipLaunchKernelGGL(k_pts_images, dim3((unsigned)((NN + 255) / 256)), dim3(256), sizeof(float) * (M + 1), st, N,
                       E, M, sigma, params, out);
    return hipGetLastError();
}

// sums[b] = sum of the n partials of image b (fixed order); am[k] = <a_k>
__global__ __launch_bounds__(256) void k_pts_sums(int B, int n, const double *__restrict__ part, int N, int E, int M,
                                                   const float *__restrict__ params, double *__restrict__ out)
{
    __shared__ double red[256 / 64];
    const int b = blockIdx.x;
    if (b < B) {
        double acc = 0.0;
        for (int i = threadIdx.x; i < n; i += 256) acc += part[(long long)b * n + i];
        acc = block_sum_d<256>(acc, red);
        if (threadIdx.x == 0) out[b] = acc;
        return;
    }
    const int k = b - B;
    const float *a = params + (long long)N * N + E;
    double acc = 0.0;
    for (int i = threadIdx.x; i < E; i += 256) acc += a[(long long)i * M + k];
    acc = block_sum_d<256>(acc, red);
    if (threadIdx.x == 0) out[b] = acc / E;
}

hipError_t launch_pts_sums(hipStream_t st, int B, int n, const double *part, int N, int E, int M, const float *params,
                           double *out)
{
    hipLaunchKernelGGL(k_pts_sums, dim3(B + M), dim3(256), 0, st, B, n, part, N, E, M, params, out);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// a12: Adam update (per-block learning rates)
// --------------------------------------------------------------------------

// The step number lives on the device (d_t) so that a captured graph can run
// consecutive steps: the final reduction kernel of the step advances it, k_adam
// reads it.
__global__ void k_set_int(int *d_t, int v) { *d_t = v; }

// plain device copy, used to calibrate memory-traffic counters
__global__ void k_copy_probe(const float4 *__restrict__ a, float4 *__restrict__ b, long long n4)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (long long)gridDim.x * blockDim.x)
        b[i] = a[i];
}

// Idle lead-in for stage timing: one wave sleeps for a fixed number of
// s_sleep periods (about 3.4 us each at 2.4 GHz) and exits.
__global__ void k_idle(int iters)
{
    for (int i = 0; i < iters; ++i) __builtin_amdgcn_s_sleep(127);
}

hipError_t launch_idle(hipStream_t st, int iters)
{
    hipLaunchKernelGGL(k_idle, dim3(1), dim3(64), 0, st, iters);
    return hipGetLastError();
}

hipError_t launch_copy_probe(hipStream_t st, const float *src, float *dst, long long n)
{
    hipLaunchKernelGGL(k_copy_probe, dim3(2048), dim3(256), 0, st, (const float4 *)src, (float4 *)dst, n / 4);
    return hipGetLastError();
}

__global__ void k_adam(long long P, long long e0, long long e1, long long e2, float lr0, float lr1,
                       float lr2, float lr3, float *__restrict__ params,
                       const float *__restrict__ grad, float *__restrict__ m,
                       float *__restrict__ v, float beta1, float beta2, float eps,
                       const int *__restrict__ d_t, int rule, float eps_root)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P) return;
    const float t = (float)(*d_t);
    const float bc1 = 1.f - powf(beta1, t);
    const float bc2 = 1.f - powf(beta2, t);
    const float lr = i < e0 ? lr0 : (i < e1 ? lr1 : (i < e2 ? lr2 : lr3));
    float pi = params[i], mi = m[i], vi = v[i];
    adam_update(pi, mi, vi, grad[i], lr, beta1, beta2, bc1, bc2, eps, rule == 1, eps_root);
    m[i] = mi;
    v[i] = vi;
    params[i] = pi;
}

hipError_t launch_set_step(hipStream_t st, int *d_t, int value)
{
    hipLaunchKernelGGL(k_set_int, dim3(1), dim3(1), 0, st, d_t, value);
    return hipGetLastError();
}

hipError_t launch_adam(hipStream_t st, long long P, const long long *seg_end, const float *lr,
                       float *params, const float *grad, float *m, float *v, int *d_t, float beta1,
                       float beta2, float eps, int rule, float eps_root)
{
    const int nb = (int)((P + 255) / 256);
    hipLaunchKernelGGL(k_adam, dim3(nb), dim3(256), 0, st, P, seg_end[0], seg_end[1], seg_end[2],
                       lr[0], lr[1], lr[2], lr[3], params, grad, m, v, beta1, beta2, eps, d_t, rule, eps_root);
    return hipGetLastError();
}

__global__ void k_fill(float *p, long long n, float v)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

hipError_t launch_fill(hipStream_t st, float *p, long long n, float v)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

}  // namespace starred
