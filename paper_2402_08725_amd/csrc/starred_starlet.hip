// Launches of the starlet passes (starred_scales.h), and the host side of the
// composite-filter passes that ride in other launches (starred_dense.h).
#include "starred_dense.h"
#include "starred_internal.h"
#include "starred_scales.h"

#include <hip/hip_runtime.h>

#include <vector>

namespace starred {

// The job of a work group: consecutive jobs are neighbouring subimages, which share every line of
// memory their strided pixels lie in, so each of the eight XCDs (work groups go to them in turn)
// takes a run of consecutive jobs and fetches its lines into its own L2 once. 512^2, eight planes, the
// transform: 28.6 us in turn, 24.7 so. Not for short strides (they share few lines: five planes 12.6
// us, 14.0 so) nor above 1024^2, whose planes are larger than the L2s (2048^2: 201 us, 244 so).
constexpr int kStarRuns = 1024;
__device__ __forceinline__ int star_job(const StarArgs &a, int g)
{
    if (a.group(g).D < 8 || a.N > kStarRuns) return blockIdx.x;
    const int n = gridDim.x, x = blockIdx.x & 7, i = blockIdx.x >> 3;
    return x * (n >> 3) + min(x, n & 7) + i;
}

template <class V, int L, int T, int NT>
__global__ __launch_bounds__(NT) void k_star_forward(StarArgs a, int g)
{
    extern __shared__ double lds[];
    __shared__ double red[NT / 64];
    star_forward<V, L, T, NT>(a, g, star_job(a, g), (V *)lds, red);
}

template <class V, int L, int T, int NT>
__global__ __launch_bounds__(NT) void k_star_adjoint(StarArgs a, int g)
{
    extern __shared__ double lds[];
    star_adjoint<V, L, T, NT>(a, g, star_job(a, g), (V *)lds, StarStore{a.out});
}

// J = 1: the only plane is the image itself.
__global__ __launch_bounds__(256) void k_star_plane(StarArgs a)
{
    __shared__ double red[256 / 64];
    const long long NN = (long long)a.N * a.N, pix = (long long)blockIdx.x * 256 + threadIdx.x;
    const int b = blockIdx.y;
    const float lam = b ? a.lam1 : a.lam0;
    double l1 = 0.0;
    if (pix < NN) {
        const float al = a.image(b)[pix];
        if (a.coeffs) a.coeffs[b * NN + pix] = al;
        if (a.W) {
            const float w = a.w_stride ? a.W[pix] : a.W[0];
            if (a.z) a.z[b * NN + pix] = lam * w * (float)((al > 0.f) - (al < 0.f));
            l1 = (double)lam * (double)w * (double)fabsf(al);
        }
    }
    if (a.part_l1) {
        const double s = star_block_sum(l1, red);
        if (threadIdx.x == 0) a.part_l1[(long long)b * gridDim.x + blockIdx.x] = s;
    }
}

__global__ void k_copy(const float *__restrict__ a, float *__restrict__ b, long long n)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = a[i];
}

bool star_fp64(int N, int J) { return N <= kStarSmall && J <= kStarFewPlanes; }

int star_l1_slots(const StarArgs &a)
{
    return a.J == 1 ? (int)(((long long)a.N * a.N + 255) / 256) : a.l1_slots();
}

// tiles of 16 on 512 threads (two waves per SIMD hide more than one); of 32 on 1024, but on 512 for
// one level, whose groups are short (the transform of 512^2 with two planes 4.9 us on 1024, 4.0 on
// 512; of 1024^2 11.3 and 8.5)
constexpr int star_wide_threads(int L) { return L == 1 ? 512 : 1024; }
#define STAR_LAUNCH_WIDE(KERNEL, L)                                                                                 \
    hipLaunchKernelGGL((KERNEL<float, L, kStarTileLarge, star_wide_threads(L)>), grid, dim3(star_wide_threads(L)), \
                       q.lds(), st, a, g)
#define STAR_LAUNCH_L(KERNEL, V, L)                                                             \
    if (q.T == kStarTile)                                                                       \
        hipLaunchKernelGGL((KERNEL<V, L, kStarTile, 512>), grid, dim3(512), q.lds(), st, a, g); \
    else                                                                                        \
        STAR_LAUNCH_WIDE(KERNEL, L)
#define STAR_LAUNCH(KERNEL)                                          \
    do {                                                             \
        const StarArgs::Group q = a.group(g);                        \
        const dim3 grid(a.B * q.jobs());                             \
        switch (q.L + (a.fp64 ? 8 : 0)) {                            \
        case 1: STAR_LAUNCH_L(KERNEL, float, 1); break;              \
        case 2: STAR_LAUNCH_L(KERNEL, float, 2); break;              \
        case 3: STAR_LAUNCH_L(KERNEL, float, 3); break;              \
        case 9: STAR_LAUNCH_L(KERNEL, double, 1); break;             \
        case 10: STAR_LAUNCH_L(KERNEL, double, 2); break;            \
        case 11: STAR_LAUNCH_L(KERNEL, double, 3); break;            \
        default: return hipErrorInvalidValue;                        \
        }                                                            \
    } while (0)

// the passes may be carried by other launches (StarPiece): at most four of them
bool star_rides(const StarArgs &a)
{
    const int n = star_num_groups(a.J);
    return a.fp64 && n > 0 && n <= 2;
}

hipError_t launch_star_forward(hipStream_t st, const StarArgs &a)
{
    if (a.J == 1) {
        hipLaunchKernelGGL(k_star_plane, dim3(star_l1_slots(a), a.B), dim3(256), 0, st, a);
        return hipGetLastError();
    }
    for (int g = 0; g < star_num_groups(a.J); ++g) STAR_LAUNCH(k_star_forward);
    return hipGetLastError();
}

hipError_t launch_star_adjoint(hipStream_t st, const StarArgs &a)
{
    const long long n = (long long)a.B * a.N * a.N;
    if (a.J == 1) {
        hipLaunchKernelGGL(k_copy, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a.z, a.out, n);
        return hipGetLastError();
    }
    for (int g = star_num_groups(a.J) - 1; g >= 0; --g) STAR_LAUNCH(k_star_adjoint);
    return hipGetLastError();
}

// ---- composite filters: LDS, shapes and taps ----

size_t dense_lds_xr(int N, int J, int rx)
{
    return sizeof(double) * ((size_t)rx * (N + 2 * DenseStar::bw(J - 1)) + kDenseXTail);
}

size_t dense_lds_x(int N, int J) { return dense_lds_xr(N, J, dense_rows_per_job(N)); }

size_t dense_lds_y(int J)
{
    return sizeof(double) * (kDenseTile * (size_t)(kDenseTile + 2 * DenseStar::bw(J - 1)) + kDenseYTail);
}

int dense_rows_for(int N, int threads) { return N >= threads ? 1 : threads / N; }

int dense_rows_per_job(int N) { return dense_rows_for(N, kDenseThreads); }

bool dense_fits(int N, int J)
{
    return J >= 2 && J <= kDenseMaxJ - 1 && N <= kDenseMaxN && DenseStar::bw(J - 1) <= N - 1 &&
           dense_lds_y(J) <= kDenseMaxLds && dense_lds_x(N, J) <= kDenseMaxLds;
}

int dense_num_taps(int J) { return J >= 2 ? DenseStar::toff(J) : 0; }

void dense_taps(int J, double *out)
{
    // a_j = h_0 * ... * h_{j-1}, h_l = B3 (1 4 6 4 1)/16 with holes 2^l
    std::vector<double> a{1.0};
    for (int j = 1; j < J; ++j) {
        const int d = 1 << (j - 1);
        std::vector<double> n(a.size() + 4 * d, 0.0);
        const double h[5] = {1.0 / 16, 4.0 / 16, 6.0 / 16, 4.0 / 16, 1.0 / 16};
        for (size_t i = 0; i < a.size(); ++i)
            for (int t = 0; t < 5; ++t) n[i + t * d] += a[i] * h[t];
        a.swap(n);
        for (int i = 0; i < DenseStar::plen(j); ++i) out[DenseStar::toff(j) + i] = i < (int)a.size() ? a[i] : 0.0;
    }
}

}  // namespace starred
