// The starlet transform and its transpose (Eq. 6) in passes of several scales each.
//
// One level of the a-trous cascade filters the whole-sample symmetric extension of the image
// (period 2N - 2) along both axes with B3 at holes d = 2^j, and a symmetric filter keeps that
// extension, so a tile can run several levels on its own if it starts with the extension
// around it: no further mirroring, only a halo of 2 d pixels per level and side. Levels
// l0 .. l0+L-1 have holes that are multiples of D = 2^l0, so they act on each of the D x D
// subimages (y mod D, x mod D) by itself; a job takes a T x T tile of one subimage with a
// halo of H = 2 (2^L - 1) of its own pixels, however large the holes are in the image.
// The transpose runs on the same footing: with E = diag(2, 1, ..., 1, 2) per axis, a level's
// operator satisfies M^T = E^-1 M E, so v = z_j + H_j^T (v - z_j) is, for E v E and E z_j E,
// the same mirror filtering; the factors are exact powers of two.
//
// J planes are J-1 levels, in groups of two and three (one for J = 2): one forward pass per group
// (the coefficients, their subgradient z and the L1 share leave in the pass that forms them, the
// smoothed plane goes on to the next group) and one transposed pass per group, last to first: two
// passes for J <= 4, four for J <= 7, six for J <= 10, where a launch per level made 2 (J - 1) and
// composite filters straight from the image cost hundreds of FP64 operations per pixel. Larger
// groups come last, where subimages are small and every pass reads scattered lines; a group of
// four needs 68 KB and 1024 threads for a tile that is mostly halo, and fills the chip beside an
// evaluation's kernels. Measured, 3 + 4 levels against 2 + 2 + 3: 512^2 with eight planes, transform
// and transpose 56 -> 52 us, loss and gradient of four such frames 176 -> 154; two images of 257^2
// (whose subimages of 33 pixels take four tiles of 32 each) 172 -> 145; and nine planes of 512^2 as
// 3 + 3 + 2 against 3 + 2 + 3: 98 -> 64.
//
// Precision: V is the type of the pixels in a pass and of the planes between the groups.
// FP64 for one or two images up to 256^2 with at most seven planes (prior and transform),
// FP32 beyond (larger grids, eight planes and more, batches of noise fields), where a wide
// tile's LDS traffic bounds the pass.
//
// What bounds a pass: with FP64 tiles of 16 the latency of its loads, barriers and LDS reads
// (1.9 k to 6.4 k filtered pixels per job, five reads and a write each); with FP32 tiles of
// 32 the LDS traffic (14 k filtered pixels for three levels).
#pragma once

#include <hip/hip_runtime.h>

namespace starred {

constexpr int kStarTile = 16;       // FP64 tiles, and FP32 ones of subimages no larger
constexpr int kStarTileLarge = 32;  // FP32 tiles (fewer halo pixels per pixel)
constexpr int kStarSmall = 256;     // grids up to this side ...
constexpr int kStarFewPlanes = 7;   // ... with at most this many planes run in FP64

// levels of the group that starts with `rest` levels to go (two bits each: 1, 2, 3, 2, 2, 3, 2
// for one to seven, then 3)
__host__ __device__ constexpr int star_group_len(int rest) { return (0xFFFFBAE4u >> 2 * rest) & 3; }

__host__ __device__ inline int star_num_groups(int J)
{
    int n = 0;
    for (int l = 0; l < J - 1; ++n) l += star_group_len(J - 1 - l);
    return n;
}

// A batch of B images and where their transform goes. Planes of one image follow each other;
// a null pointer leaves an output out.
struct StarArgs {
    int N = 0, J = 0, B = 0;
    bool fp64 = true;
    const float *img = nullptr;   // image 0
    const float *img1 = nullptr;  // images 1, 2, ...
    const float *W = nullptr;     // weights: per pixel [J][N][N] (w_stride != 0) or per scale [J]
    int w_stride = 0;
    float lam0 = 0.f, lam1 = 0.f;  // weight of image 0 and of the others
    float *coeffs = nullptr;       // [B][J][N][N]
    float *z = nullptr;            // [B][J][N][N] subgradient lambda W sgn(alpha): written, then read
    void *ca = nullptr, *cb = nullptr;  // [B][N][N] planes between the groups
    double *part_l1 = nullptr;     // [B][l1_slots()]
    float *out = nullptr;          // [B][N][N] the transpose of z

    // group g: its first level, its levels, subimages per axis, tile side, tiles per axis
    struct Group {
        int l0, L, D, T, tiles, size;
        __host__ __device__ int jobs() const { return D * D * tiles * tiles; }
        __host__ __device__ int region() const { return T + 4 * ((1 << L) - 1); }
        __host__ __device__ size_t lds() const
        {
            return (size_t)size * 2 * region() * region();
        }
    };
    __host__ __device__ Group group(int g) const
    {
        Group q;
        q.l0 = 0;
        q.L = star_group_len(J - 1);
        for (; g > 0; --g) {
            q.l0 += q.L;
            q.L = star_group_len(J - 1 - q.l0);
        }
        q.D = 1 << q.l0;
        const int side = (N + q.D - 1) / q.D;
        q.T = fp64 || side <= kStarTile ? kStarTile : kStarTileLarge;
        q.tiles = (side + q.T - 1) / q.T;
        q.size = fp64 ? sizeof(double) : sizeof(float);
        return q;
    }
    __host__ __device__ int l1_slots() const  // per image
    {
        int n = 0;
        for (int g = 0; g < star_num_groups(J); ++g) n += group(g).jobs();
        return n;
    }
    __host__ __device__ const float *image(int b) const
    {
        return b == 0 ? img : img1 + (long long)(b - 1) * N * N;
    }
};

// index i of the whole-sample symmetric extension of a line of N >= 2 samples
__device__ __forceinline__ int star_mirror(int i, int N)
{
    i = i < 0 ? -i : i;
    while (i > 2 * (N - 1)) {  // (several periods: small images under wide filters)
        i -= 2 * (N - 1);
    }
    return i > N - 1 ? 2 * (N - 1) - i : i;
}

template <class V>
__device__ __forceinline__ V star_end(int i, int N) { return (i == 0 || i == N - 1) ? V(2) : V(1); }

// B3 = (1 4 6 4 1) / 16 over five samples `step` apart
template <class V>
__device__ __forceinline__ V star_b3(const V *p, int step)
{
    V acc = V(0.0625) * p[-2 * step];
    acc = fma(V(0.25), p[-step], acc);
    acc = fma(V(0.375), p[0], acc);
    acc = fma(V(0.25), p[step], acc);
    return fma(V(0.0625), p[2 * step], acc);
}

// Sum of one double per thread over a work group of any whole number of waves; thread 0's.
__device__ __forceinline__ double star_block_sum(double v, double *sh)
{
    #pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    __syncthreads();
    if (lane == 0) sh[w] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < nw; ++i) r += sh[i];
    __syncthreads();
    return r;
}

// A job's place: image b, subimage (ry, rx), tile origin (ty, tx) in the subimage's pixels.
struct StarJob {
    int b, ry, rx, ty, tx;
    __device__ StarJob(const StarArgs::Group &q, int job)
    {
        const int per = q.jobs(), t2 = q.tiles * q.tiles;
        b = job / per;
        job -= b * per;
        const int cls = job / t2, tile = job - cls * t2;
        ry = cls / q.D;
        rx = cls - ry * q.D;
        ty = tile / q.tiles * q.T;
        tx = tile % q.tiles * q.T;
    }
};

// The passes are compiled for L levels, tiles of T and NT threads: with constant bounds the
// loops unroll, and a thread's LDS reads of several pixels are in flight together (a work
// group has only one to four waves per SIMD to hide their latency). Threads run in rows of
// 16 over the region; the loads of the region go wave by wave along its rows, so that the
// mirrored column of a lane and the mirrored row of a wave are found once.
template <int L, int T>
struct StarShape {
    static constexpr int H = 2 * ((1 << L) - 1), R = T + 2 * H;
};

// region[r][c] <- src(y, x) at the mirrored image positions of the tile and its halo
template <class V, int L, int T, int NT, class Src>
__device__ __forceinline__ void star_stage(const StarArgs &a, const StarArgs::Group &q, const StarJob &j,
                                           V *region, Src src)
{
    constexpr int H = StarShape<L, T>::H, R = StarShape<L, T>::R, NW = NT / 64;
    constexpr int KR = (R + NW - 1) / NW, KC = (R + 63) / 64;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), N = a.N;
    int x[KC];
    #pragma unroll
    for (int k = 0; k < KC; ++k) x[k] = star_mirror(j.rx + q.D * (j.tx + min(lane + 64 * k, R - 1) - H), N);
    V v[KR][KC];
    #pragma unroll
    for (int u = 0; u < KR; ++u) {
        const int y = star_mirror(j.ry + q.D * (j.ty + min(w + u * NW, R - 1) - H), N);
        #pragma unroll
        for (int k = 0; k < KC; ++k) v[u][k] = src(y, x[k]);
    }
    #pragma unroll
    for (int u = 0; u < KR; ++u)
        #pragma unroll
        for (int k = 0; k < KC; ++k)
            if (w + u * NW < R && lane + 64 * k < R) region[(w + u * NW) * R + lane + 64 * k] = v[u][k];
}

// f(r, c, k, ok) over rows [r0, r1) and columns [c0, c1), k the thread's count; a thread past
// the end takes the last row or column once more with ok false (no branches between the
// loads of a thread's pixels)
template <int NT, int r0, int r1, int c0, int c1, class F>
__device__ __forceinline__ void star_each(F f)
{
    constexpr int NY = NT / 16, KR = (r1 - r0 + NY - 1) / NY, KC = (c1 - c0 + 15) / 16;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    #pragma unroll
    for (int u = 0; u < KR; ++u)
        #pragma unroll
        for (int k = 0; k < KC; ++k) {
            const int r = r0 + ty + u * NY, c = c0 + tx + k * 16;
            f(min(r, r1 - 1), min(c, c1 - 1), u * KC + k, r < r1 && c < c1);
        }
}

template <int NT, int r0, int r1, int c0, int c1>
struct StarCount {  // values of star_each's third argument
    static constexpr int n = ((r1 - r0 + NT / 16 - 1) / (NT / 16)) * ((c1 - c0 + 15) / 16);
};

// out = B3 of in along x (or with step e R along y) over rows [r0, r1), columns [c0, c1)
template <class V, int NT, int r0, int r1, int c0, int c1, int R>
__device__ __forceinline__ void star_filter(const V *in, V *out, int step)
{
    V v[StarCount<NT, r0, r1, c0, c1>::n];
    star_each<NT, r0, r1, c0, c1>([&](int r, int c, int k, bool) { v[k] = star_b3(in + r * R + c, step); });
    star_each<NT, r0, r1, c0, c1>([&](int r, int c, int k, bool) { out[r * R + c] = v[k]; });
}

// ---- forward pass ----
template <class V, int L, int T, int NT, int l = 0>
__device__ __forceinline__ void star_forward_level(const StarArgs &a, const StarArgs::Group &q, const StarJob &j,
                                                   bool last, V *cn, float lam, V *region, V *tmp, double &l1)
{
    if constexpr (l < L) {
        constexpr int H = StarShape<L, T>::H, R = StarShape<L, T>::R;
        constexpr int e = 1 << l, lo = 2 * (e - 1), hi = R - lo, in = lo + 2 * e, out = hi - 2 * e;
        const int N = a.N;
        const long long NN = (long long)N * N;
        star_filter<V, NT, lo, hi, in, out, R>(region, tmp, e);
        __syncthreads();
        auto emit = [&](int plane, long long pix, V al) {
            const long long at = ((long long)j.b * a.J + plane) * NN + pix;
            if (a.coeffs) a.coeffs[at] = (float)al;
            if (a.W) {
                const float w = a.w_stride ? a.W[plane * NN + pix] : a.W[plane];
                if (a.z) a.z[at] = lam * w * (float)((al > V(0)) - (al < V(0)));
                l1 += (double)lam * (double)w * fabs((double)al);
            }
        };
        constexpr int K = StarCount<NT, in, out, in, out>::n;
        V was[K], now[K];
        star_each<NT, in, out, in, out>([&](int r, int c, int k, bool) {
            was[k] = region[r * R + c];
            now[k] = star_b3(tmp + r * R + c, e * R);
        });
        star_each<NT, in, out, in, out>([&](int r, int c, int k, bool ok) {
            if (!ok) return;
            region[r * R + c] = now[k];
            const int y = j.ry + q.D * (j.ty + r - H), x = j.rx + q.D * (j.tx + c - H);
            if (r >= H && r < H + T && c >= H && c < H + T && y < N && x < N) {
                const long long pix = (long long)y * N + x;
                emit(q.l0 + l, pix, was[k] - now[k]);
                if (l == L - 1) {
                    if (last) emit(a.J - 1, pix, now[k]);
                    else cn[pix] = now[k];
                }
            }
        });
        __syncthreads();
        star_forward_level<V, L, T, NT, l + 1>(a, q, j, last, cn, lam, region, tmp, l1);
    }
}

template <class V, int L, int T, int NT>
__device__ __forceinline__ void star_forward(const StarArgs &a, int g, int job, V *lds, double *red)
{
    constexpr int R = StarShape<L, T>::R;
    const StarArgs::Group q = a.group(g);
    const StarJob j(q, job);
    const int N = a.N;
    const long long NN = (long long)N * N;
    V *region = lds, *tmp = lds + R * R;
    if (g == 0) {
        const float *im = a.image(j.b);
        star_stage<V, L, T, NT>(a, q, j, region, [&](int y, int x) { return (V)im[y * N + x]; });
    } else {
        const V *c = (const V *)((g & 1) ? a.ca : a.cb) + j.b * NN;
        star_stage<V, L, T, NT>(a, q, j, region, [&](int y, int x) { return c[y * N + x]; });
    }
    __syncthreads();
    const bool last = q.l0 + L == a.J - 1;
    V *cn = last ? nullptr : (V *)((g & 1) ? a.cb : a.ca) + j.b * NN;
    double l1 = 0.0;
    star_forward_level<V, L, T, NT>(a, q, j, last, cn, j.b ? a.lam1 : a.lam0, region, tmp, l1);
    if (a.part_l1) {
        const double s = star_block_sum(l1, red);
        int at = job - j.b * q.jobs();
        for (int k = 0; k < g; ++k) at += a.group(k).jobs();
        if (threadIdx.x == 0) a.part_l1[(long long)j.b * a.l1_slots() + at] = s;
    }
}

// ---- transposed pass (the last group first) ----
// out(pixel, value) takes the transpose's pixels as the first group's pass forms them, each
// pixel once (it may add to what is there)
struct StarStore {
    float *out;
    __device__ void operator()(long long pix, float v) const { out[pix] = v; }
};

template <class V, int L, int T, int NT, class Out, int l = L - 1>
__device__ __forceinline__ void star_adjoint_level(const StarArgs &a, int g, const StarArgs::Group &q, const StarJob &j,
                                                   const float *z, V *region, V *tmp, Out out)
{
    if constexpr (l >= 0) {
        constexpr int H = StarShape<L, T>::H, R = StarShape<L, T>::R;
        // (levels above this one took 2 (2^L - 2^(l+1)) pixels off each side)
        constexpr int e = 1 << l, lo = 2 * ((1 << L) - (2 << l)), hi = R - lo, in = lo + 2 * e, end = hi - 2 * e;
        const int N = a.N;
        const long long NN = (long long)N * N;
        // what joins the filtered value: z_j, less the next level's (on its way during the rows)
        float zl[StarCount<NT, in, end, in, end>::n][2];
        star_each<NT, in, end, in, end>([&](int r, int c, int k, bool) {
            const int y = star_mirror(j.ry + q.D * (j.ty + r - H), N), x = star_mirror(j.rx + q.D * (j.tx + c - H), N);
            const float *p = z + (q.l0 + l) * NN + y * N + x;
            zl[k][0] = p[0];
            zl[k][1] = l > 0 ? p[-NN] : 0.f;
        });
        star_filter<V, NT, lo, hi, in, end, R>(region, tmp, e);
        __syncthreads();
        star_each<NT, in, end, in, end>([&](int r, int c, int k, bool ok) {
            const int y = j.ry + q.D * (j.ty + r - H), x = j.rx + q.D * (j.tx + c - H);
            const V s = star_end<V>(star_mirror(y, N), N) * star_end<V>(star_mirror(x, N), N);
            const V v = fma((V)zl[k][0] - (V)zl[k][1], s, star_b3(tmp + r * R + c, e * R));
            if (l > 0) {
                region[r * R + c] = v;
            } else if (ok && y < N && x < N) {
                const long long pix = (long long)y * N + x;
                if (g > 0) ((V *)((g & 1) ? a.ca : a.cb))[j.b * NN + pix] = v;
                else out(j.b * NN + pix, (float)(v / s));
            }
        });
        __syncthreads();
        star_adjoint_level<V, L, T, NT, Out, l - 1>(a, g, q, j, z, region, tmp, out);
    }
}

template <class V, int L, int T, int NT, class Out>
__device__ __forceinline__ void star_adjoint(const StarArgs &a, int g, int job, V *lds, Out out)
{
    constexpr int R = StarShape<L, T>::R;
    const StarArgs::Group q = a.group(g);
    const StarJob j(q, job);
    const int N = a.N;
    const long long NN = (long long)N * N;
    V *region = lds, *tmp = lds + R * R;
    const bool last = q.l0 + L == a.J - 1;
    const float *z = a.z + (long long)j.b * a.J * NN;
    const float *ztop = z + (q.l0 + L - 1) * NN;
    // E (v - z_top) E, v the plane above the group (held as E v E) or the coarse z
    if (last) {
        const float *zc = z + (a.J - 1) * NN;
        star_stage<V, L, T, NT>(a, q, j, region, [&](int y, int x) {
            const int p = y * N + x;
            return ((V)zc[p] - (V)ztop[p]) * (star_end<V>(y, N) * star_end<V>(x, N));
        });
    } else {
        const V *v = (const V *)((g & 1) ? a.cb : a.ca) + j.b * NN;
        star_stage<V, L, T, NT>(a, q, j, region, [&](int y, int x) {
            const int p = y * N + x;
            return fma(-(V)ztop[p], star_end<V>(y, N) * star_end<V>(x, N), v[p]);
        });
    }
    __syncthreads();
    star_adjoint_level<V, L, T, NT>(a, g, q, j, z, region, tmp, out);
}

// One FP64 pass carried by another launch: its work groups first .. first+jobs-1 run the
// pass's jobs (lds() bytes of dynamic LDS).
struct StarPiece {
    StarArgs a;
    int group = -1;  // -1: none
    bool adjoint = false;
    int first = 0, jobs = 0;
    size_t lds() const { return group < 0 ? 0 : a.group(group).lds(); }
};

// Runs job `job` of a transposed pass, its pixels into out.
template <int NT, class Out>
__device__ __forceinline__ void star_piece_adjoint(const StarPiece &p, int job, void *lds, Out out)
{
    switch (p.a.group(p.group).L) {
    case 1: star_adjoint<double, 1, kStarTile, NT>(p.a, p.group, job, (double *)lds, out); break;
    case 2: star_adjoint<double, 2, kStarTile, NT>(p.a, p.group, job, (double *)lds, out); break;
    default: star_adjoint<double, 3, kStarTile, NT>(p.a, p.group, job, (double *)lds, out); break;
    }
}

// Runs this work group's job when it carries one; true if it did.
template <int NT>
__device__ __forceinline__ bool star_piece_run(const StarPiece &p, void *lds, double *red)
{
    const int job = (int)blockIdx.x - p.first;
    if (p.group < 0 || job < 0 || job >= p.jobs) return false;
    if (p.adjoint) {
        star_piece_adjoint<NT>(p, job, lds, StarStore{p.a.out});
        return true;
    }
    switch (p.a.group(p.group).L) {
    case 1: star_forward<double, 1, kStarTile, NT>(p.a, p.group, job, (double *)lds, red); break;
    case 2: star_forward<double, 2, kStarTile, NT>(p.a, p.group, job, (double *)lds, red); break;
    default: star_forward<double, 3, kStarTile, NT>(p.a, p.group, job, (double *)lds, red); break;
    }
    return true;
}

}  // namespace starred
