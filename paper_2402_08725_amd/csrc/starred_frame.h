// The one-launch forward of frames whose Q-grid spectra fit in LDS, for the transform
// lengths Q = RA RB with both factors at most 16: the loss of Eqs. 8-10 and rho_hat, the
// spectrum of the weighted residual that the adjoint reads.
//
// A frame's plane (Q/2+1 lines of stride Q+1) stays in LDS, transformed in place, and every
// length-Q transform is two register DFTs of RA and RB points with one exchange between
// them. Each step reads its inputs where the step before left them and leaves its outputs
// where the next one wants them:
//   product   the s^2 alias terms S'' F of RA bins of a column (global memory), the column's
//             first inverse stage in registers                                      -> LDS
//   columns   second inverse stage                                                  -> LDS
//   rows      first inverse stage, reading pairs of real rows out of the columns     -> LDS
//             second stage: the model in registers; residual, chi-square; the first
//             forward stage on the same registers (it wants the very elements that the
//             inverse stage of the same radix leaves)                                -> LDS
//             second forward stage                                                   -> LDS
//   columns   first forward stage, splitting the row pairs' spectra                   -> LDS
//             second forward stage                                    -> rho_hat (memory)
// A plane is written six times and read eight (three-stage transforms with separate
// re-layouts: 16 and 17). Lanes run over lines wherever LDS is read or written: the odd line
// stride spreads them over all banks; the residual's step runs along the rows instead, so
// that data and weights come in runs of RA consecutive floats.
//
// What bounds it: waits, at the barriers between dependent phases of the one group of 16 waves per
// compute unit and for the product's loads of S''. On 1000 frames of 32^2 .. 128^2 (91 us on the
// supernova workload's data, 78 where data and weights are uniform in [0, 1)) the SIMDs are
// VALU-busy a third of the launch, LDS conflicts take 2 %, and 303 MB move at 3.3 TB/s where a copy
// reaches 5.2. Measured with the former kernel (three-stage transforms, one frame per group, four
// sources' terms whatever M) and with this one: the loss of those frames 201 -> 123 us; eight steps
// of their fit 2175 -> 1772 us; 16 steps over 100 frames of 64^2 (four sources) 1281 -> 1142 us.
//
// A work group of 1024 threads holds one frame or, when there are more frames than compute
// units, NF frames of a class side by side (1024 / NF threads each): a 32^2 frame's plane has
// only 75 RA-point DFTs per stage.
#pragma once

#include "starred_fft.h"
#include "starred_radix.h"

namespace starred {

template <int S, int MS, int RA, int RB, int NF>
__device__ __forceinline__ void frame_body(const FrameItem &f, const FrameArgs &g, float2 *sm, double *red)
{
    constexpr int Q = RA * RB, HQ = Q / 2 + 1, Ls = Q + 1, P = S * Q, NT = kFusedThreads / NF;
    const int slot = NF > 1 ? threadIdx.x / NT : 0, tid = NF > 1 ? threadIdx.x % NT : threadIdx.x;
    // (a slot past the item's frames repeats its first frame and writes nothing)
    const int fs = slot < f.nf ? slot : 0;
    const bool on = slot < f.nf;
    const int i = f.frame[fs], n = f.n, n2 = (n + 1) / 2, M = g.M;
    float2 *A = sm + slot * HQ * Ls;
    float2 *twl = sm + NF * HQ * Ls, *t = twl + Q;
    {
        // the Q twiddles and the factor tables [w | gx_k, gy_k per source], zero past the
        // last source (the product below takes MS sources without a test)
        const float2 *tg = g.tab + f.tab_off;
        for (int e = threadIdx.x; e < Q; e += kFusedThreads) twl[e] = g.tw[f.tw_off + e];
        for (int e = threadIdx.x; e < (1 + 2 * frame_sources(M, Q)) * P; e += kFusedThreads) {
            const int k2 = e / P;  // 0: w, then gx_0, gy_0, gx_1, ...
            t[e] = e < (1 + 2 * M) * P ? tg[e + (k2 > 0 ? (k2 - 1) / 2 * 2 * P : 0)] : make_float2(0.f, 0.f);
        }
    }
    const float2 *Si = g.Sp + f.s_off[fs], *Hc = g.Hh + f.hh_off;
    const float G = g.params[(long long)g.N * g.N + i];
    const float *ai = g.params + (long long)g.N * g.N + g.E + (long long)i * M;
    __syncthreads();
    // ---- the model spectrum: RA bins ky = j + r RB of a column, and their DFT
    if constexpr (MS > 0) {
    constexpr int MR = MS;
    // (the body without sources has no tables for the one that MS = 1 takes with amplitude zero: it
    // reads the window's. Known at compile time: as a value of M it cost every body its constant
    // LDS offsets, 1000 frames of 32^2 .. 128^2 78.4 -> 80.7 us)
    constexpr int tk = Q == kFrameLongQ ? 0 : P;
    for (int it = tid; it < HQ * RB; it += NT) {
        const int j = it / HQ, kx = it - j * HQ;
        float2 wxG[S], px[S][MR];
        #pragma unroll
        for (int b = 0; b < S; ++b) {
            wxG[b] = cscale(t[kx + b * Q], G);
            #pragma unroll
            for (int k = 0; k < MR; ++k)
                px[b][k] = cscale(t[(1 + 2 * k) * tk + kx + b * Q], k < M ? ai[k] : 0.f);
        }
        float2 v[RA];
        #pragma unroll
        for (int r = 0; r < RA; ++r) {
            const int ky = j + r * RB, at = (ky * HQ + kx) * S * S;
            float2 acc = make_float2(0.f, 0.f);
            #pragma unroll
            for (int b = 0; b < S; ++b) {
                float2 h[S], sk[S];
                alias_load<S>(Hc, at + b * S, h);
                alias_load<S>(Si, at + b * S, sk);
                #pragma unroll
                for (int a = 0; a < S; ++a) {
                    const int Ky = ky + a * Q;
                    const float2 wy = t[Ky];
                    float2 F = h[a];
                    F.x = fmaf(wy.x, wxG[b].x, fmaf(-wy.y, wxG[b].y, F.x));
                    F.y = fmaf(wy.x, wxG[b].y, fmaf(wy.y, wxG[b].x, F.y));
                    #pragma unroll
                    for (int k = 0; k < MR; ++k) {
                        const float2 gy = t[(2 + 2 * k) * tk + Ky];
                        F.x = fmaf(gy.x, px[b][k].x, fmaf(-gy.y, px[b][k].y, F.x));
                        F.y = fmaf(gy.x, px[b][k].y, fmaf(gy.y, px[b][k].x, F.y));
                    }
                    acc.x = fmaf(sk[a].x, F.x, fmaf(-sk[a].y, F.y, acc.x));
                    acc.y = fmaf(sk[a].x, F.y, fmaf(sk[a].y, F.x, acc.y));
                }
            }
            v[r] = acc;
            // the loads of two bins (one for s = 3 or several sources) in flight together, no
            // more (registers)
            if (S == 3 || MS > 1 || (r & 1)) __builtin_amdgcn_sched_barrier(0);
        }
        dft<RA, true>(v);
        #pragma unroll
        for (int r = 0; r < RA; ++r) A[kx * Ls + j * RA + r] = v[r];
    }
    } else {
        // many sources: bin by bin (a loop over the sources between the loads and their use
        // leaves no registers for a column's bins), then the first stage on its own
        for (int e = tid; e < HQ * Q; e += NT) {
            const int ky = e / HQ, kx = e - ky * HQ, at = e * S * S;
            float2 F[S][S], sk[S][S];
            #pragma unroll
            for (int b = 0; b < S; ++b) {
                alias_load<S>(Hc, at + b * S, F[b]);
                alias_load<S>(Si, at + b * S, sk[b]);
                #pragma unroll
                for (int a = 0; a < S; ++a) F[b][a] = cadd(F[b][a], cscale(cmul(t[ky + a * Q], t[kx + b * Q]), G));
            }
            for (int k = 0; k < M; ++k) {
                const float2 *tk = t + (1 + 2 * k) * P;
                float2 gx[S], gy[S];
                #pragma unroll
                for (int b = 0; b < S; ++b) {
                    gx[b] = cscale(tk[kx + b * Q], ai[k]);
                    gy[b] = tk[P + ky + b * Q];
                }
                #pragma unroll
                for (int b = 0; b < S; ++b)
                    #pragma unroll
                    for (int a = 0; a < S; ++a) F[b][a] = cadd(F[b][a], cmul(gy[a], gx[b]));
            }
            float2 acc = make_float2(0.f, 0.f);
            #pragma unroll
            for (int b = 0; b < S; ++b)
                #pragma unroll
                for (int a = 0; a < S; ++a) acc = cadd(acc, cmul(sk[b][a], F[b][a]));
            A[kx * Ls + ky] = acc;
        }
        __syncthreads();
        constexpr int KB = (HQ * RB + NT - 1) / NT;
        float2 v[KB][RA];
        #pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int it = tid + q * NT, j = it / HQ, kx = it - j * HQ;
            if (it < HQ * RB) {
                #pragma unroll
                for (int r = 0; r < RA; ++r) v[q][r] = A[kx * Ls + j + r * RB];
                dft<RA, true>(v[q]);
            }
        }
        __syncthreads();
        #pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int it = tid + q * NT, j = it / HQ, kx = it - j * HQ;
            if (it < HQ * RB) {
                #pragma unroll
                for (int r = 0; r < RA; ++r) A[kx * Ls + j * RA + r] = v[q][r];
            }
        }
    }
    __syncthreads();
    // ---- columns, second inverse stage (rows y >= n are not needed)
    {
        constexpr int KB = (HQ * RA + NT - 1) / NT;
        float2 v[KB][RB];
        #pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int it = tid + q * NT, j = it / HQ, kx = it - j * HQ;
            if (it < HQ * RA) {
                #pragma unroll
                for (int r = 0; r < RB; ++r) v[q][r] = A[kx * Ls + j + r * RA];
                #pragma unroll
                for (int r = 1; r < RB; ++r) v[q][r] = cmulc(v[q][r], twl[r * j]);
                dft<RB, true>(v[q]);
            }
        }
        __syncthreads();
        #pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int it = tid + q * NT, j = it / HQ, kx = it - j * HQ;
            if (it < HQ * RA) {
                #pragma unroll
                for (int r = 0; r < RB; ++r)
                    if (j + r * RA < n) A[kx * Ls + j + r * RA] = v[q][r];
            }
        }
    }
    // data and weights of this thread's first residual items, on their way during the rows' first stage
    const float *dp = g.data + f.data_off[fs], *wp = g.invvar + f.data_off[fs];
    float pre[RB][4];
    auto load_data = [&](int it) {
        const int yp = it / RA, j = it - yp * RA;
        #pragma unroll
        for (int r = 0; r < RB; ++r) {
            const int x = j + r * RA;
            const bool va = yp < n2 && x < n, vb = va && 2 * yp + 1 < n;
            const int ia = va ? 2 * yp * n + x : 0, ib = vb ? ia + n : ia;
            pre[r][0] = dp[ia];
            pre[r][1] = wp[ia];
            pre[r][2] = dp[ib];
            pre[r][3] = wp[ib];
        }
    };
    constexpr bool kEarly = Q / 2 * RA <= NT || RB < 8;  // (else there are no registers left for them)
    if (kEarly) load_data(tid);
    __syncthreads();
    // ---- rows in pairs: the inverse of Z = X_2p + i X_2p+1 is x_2p + i x_2p+1 (a missing
    // second row is zero); first stage, out of the columns
    {
        constexpr int KB = (Q / 2 * RB + NT - 1) / NT;
        float2 v[KB][RA];
        int at[KB];
        #pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int it = tid + q * NT, j = it / n2, yp = it - j * n2;
            at[q] = it < n2 * RB ? yp * Ls + j * RA : -1;
            if (at[q] >= 0) {
                const bool two = 2 * yp + 1 < n;
                #pragma unroll
                for (int r = 0; r < RA; ++r) {
                    const int kx = j + r * RB;
                    const bool lo = kx < HQ;
                    const float2 *c = A + (lo ? kx : Q - kx) * Ls + 2 * yp;
                    const float2 xa = c[0];
                    const float2 xb = two ? c[1] : make_float2(0.f, 0.f);
                    v[q][r] = lo ? make_float2(xa.x - xb.y, xa.y + xb.x) : make_float2(xa.x + xb.y, xb.x - xa.y);
                }
                dft<RA, true>(v[q]);
            }
        }
        __syncthreads();
        #pragma unroll
        for (int q = 0; q < KB; ++q)
            if (at[q] >= 0) {
                #pragma unroll
                for (int r = 0; r < RA; ++r) A[at[q] + r] = v[q][r];
            }
    }
    __syncthreads();
    // ---- second inverse stage, the residual, first forward stage
    {
        constexpr int KB = (Q / 2 * RA + NT - 1) / NT;
        float2 v[KB][RB];
        double chi = 0.0;
        #pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int it = tid + q * NT, yp = it / RA, j = it - yp * RA;
            if (q > 0 || !kEarly) load_data(it);
            if (yp < n2) {
                #pragma unroll
                for (int r = 0; r < RB; ++r) v[q][r] = A[yp * Ls + j + r * RA];
                #pragma unroll
                for (int r = 1; r < RB; ++r) v[q][r] = cmulc(v[q][r], twl[r * j]);
                dft<RB, true>(v[q]);
                #pragma unroll
                for (int r = 0; r < RB; ++r) {
                    float va = 0.f, vb = 0.f;
                    if (j + r * RA < n) {
                        const float ra = v[q][r].x - pre[r][0], wa = pre[r][1];
                        va = wa * ra;
                        chi += 0.5 * (double)wa * (double)ra * (double)ra;
                        if (2 * yp + 1 < n) {
                            const float rb = v[q][r].y - pre[r][2], wb = pre[r][3];
                            vb = wb * rb;
                            chi += 0.5 * (double)wb * (double)rb * (double)rb;
                        }
                    }
                    v[q][r] = make_float2(va, vb);
                }
                if (g.Rh) dft<RB, false>(v[q]);
            }
        }
        // the frame's chi-square: wave sums across the barrier, then added in wave order
        #pragma unroll
        for (int off = 32; off > 0; off >>= 1) chi += __shfl_xor(chi, off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = chi;
        __syncthreads();
        if (tid == 0 && on) {
            double tchi = 0.0;
            #pragma unroll
            for (int w = 0; w < NT / 64; ++w) tchi += red[slot * (NT / 64) + w];
            g.part_chi[f.chi[fs]] = tchi;
        }
        if (!g.Rh) return;
        #pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int it = tid + q * NT, yp = it / RA, j = it - yp * RA;
            if (yp < n2) {
                #pragma unroll
                for (int r = 0; r < RB; ++r) A[yp * Ls + j * RB + r] = v[q][r];
            }
        }
    }
    __syncthreads();
    // ---- rows, second forward stage
    {
        constexpr int KB = (Q / 2 * RB + NT - 1) / NT;
        float2 v[KB][RA];
        int at[KB];
        #pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int it = tid + q * NT, j = it / n2, yp = it - j * n2;
            at[q] = it < n2 * RB ? yp * Ls + j : -1;
            if (at[q] >= 0) {
                #pragma unroll
                for (int r = 0; r < RA; ++r) v[q][r] = A[at[q] + r * RB];
                #pragma unroll
                for (int r = 1; r < RA; ++r) v[q][r] = cmul(v[q][r], twl[r * j]);
                dft<RA, false>(v[q]);
            }
        }
        __syncthreads();
        #pragma unroll
        for (int q = 0; q < KB; ++q)
            if (at[q] >= 0) {
                #pragma unroll
                for (int r = 0; r < RA; ++r) A[at[q] + r * RB] = v[q][r];
            }
    }
    __syncthreads();
    // ---- columns, first forward stage: a pair's spectrum Z gives R_2p = (Z(k) + conj Z(-k)) / 2
    // and R_2p+1 = (Z(k) - conj Z(-k)) / 2i; rows y >= n are zero
    {
        constexpr int KB = (HQ * RA + NT - 1) / NT;
        float2 v[KB][RB];
        #pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int it = tid + q * NT, j = it / HQ, kx = it - j * HQ, km = kx == 0 ? 0 : Q - kx;
            if (it < HQ * RA) {
                #pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const int y = j + r * RA;
                    float2 u = make_float2(0.f, 0.f);
                    if (y < n) {
                        const float2 z = A[(y >> 1) * Ls + kx], zm = A[(y >> 1) * Ls + km];
                        u = (y & 1) ? make_float2(0.5f * (z.y + zm.y), 0.5f * (zm.x - z.x))
                                    : make_float2(0.5f * (z.x + zm.x), 0.5f * (z.y - zm.y));
                    }
                    v[q][r] = u;
                }
                dft<RB, false>(v[q]);
            }
        }
        __syncthreads();
        #pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int it = tid + q * NT, j = it / HQ, kx = it - j * HQ;
            if (it < HQ * RA) {
                #pragma unroll
                for (int r = 0; r < RB; ++r) A[kx * Ls + j * RB + r] = v[q][r];
            }
        }
    }
    __syncthreads();
    // ---- columns, second forward stage -> rho_hat
    float2 *R = g.Rh + f.r_off[fs];
    for (int it = tid; it < HQ * RB; it += NT) {
        const int j = it / HQ, kx = it - j * HQ;
        float2 v[RA];
        #pragma unroll
        for (int r = 0; r < RA; ++r) v[r] = A[kx * Ls + j + r * RB];
        #pragma unroll
        for (int r = 1; r < RA; ++r) v[r] = cmul(v[r], twl[r * j]);
        dft<RA, false>(v);
        if (on) {
            #pragma unroll
            for (int r = 0; r < RA; ++r) R[(j + r * RB) * HQ + kx] = v[r];
        }
    }
}

template <int S, int MS>
__global__ __launch_bounds__(kFusedThreads) void k_frame(const FrameItem *__restrict__ items, FrameArgs g, DensePiece dp)
{
    extern __shared__ float2 sm[];
    __shared__ double red[kFusedThreads / 64];
    if (dense_piece_run(dp, sm, red)) return;  // a starlet-prior job carried by this launch
    const FrameItem &f = items[blockIdx.x];
    switch (f.Q * 8 + f.per) {
#define STARRED_FRAME_CASE(QQ, RA, RB, NF)                                      \
    case QQ * 8 + 1: frame_body<S, MS, RA, RB, 1>(f, g, sm, red); break;          \
    case (NF > 1 ? QQ * 8 + NF : -QQ):                                          \
        if constexpr (S == 2 && NF > 1) frame_body<S, MS, RA, RB, NF>(f, g, sm, red); \
        break;
        STARRED_FRAME_LENGTHS(STARRED_FRAME_CASE)
#undef STARRED_FRAME_CASE
    case kFrameLongQ * 8 + 1:
        if constexpr (S == 1 && MS == 1) frame_body<S, MS, 16, 12, 1>(f, g, sm, red);
        break;
    default: break;
    }
}

template <int S>
hipError_t launch_frames(hipStream_t st, const FftPlanDev &d, const FrameArgs &g, const DensePiece &dp, size_t lds)
{
    const int grid = d.n_frame_items + (dp.pass >= 0 ? dp.jobs : 0);
#define STARRED_FRAME_LAUNCH(MS) \
    hipLaunchKernelGGL((k_frame<S, MS>), dim3(grid), dim3(kFusedThreads), lds, st, d.frame_items, g, dp)
    if (g.M <= 1) STARRED_FRAME_LAUNCH(1);
    else if (g.M <= 4 && S < 3) STARRED_FRAME_LAUNCH(4 * (S < 3));
    else STARRED_FRAME_LAUNCH(0);  // (s = 3: four sources' factors take the registers of the nine aliases)
#undef STARRED_FRAME_LAUNCH
    return hipGetLastError();
}

}  // namespace starred
