// The transposed starlet pass on the host, a thread per work item: how often each pixel of the
// transpose is handed to the pass's functor. Arguments: N J. Prints, for work groups of 256 and of
// 512 threads, the fewest and the most times.
#include <algorithm>
#include <atomic>
#include <barrier>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#define __host__
#define __device__
#define __forceinline__ inline
#define __shared__ static
#define __builtin_amdgcn_readfirstlane(v) (v)
struct Index { unsigned x; };
static thread_local Index threadIdx;
static Index blockIdx, blockDim;
static std::barrier<> *group;
static void __syncthreads() { group->arrive_and_wait(); }
static double __shfl_xor(double v, int, int) { return v; }
using std::fma;
using std::max;
using std::min;

#include "starred_scales.h"

using namespace starred;

struct Count {
    std::atomic<int> *n;
    void operator()(long long pix, float) const { n[pix]++; }
};

template <int NT, int L>
static void pass(const StarArgs &a, int g, Count out)
{
    std::vector<double> lds(a.group(g).lds() / sizeof(double));
    for (int job = 0; job < a.group(g).jobs(); ++job) {
        std::barrier<> bar(NT);
        group = &bar;
        std::vector<std::thread> t;
        for (unsigned i = 0; i < NT; ++i)
            t.emplace_back([&, i] {
                threadIdx.x = i;
                star_adjoint<double, L, kStarTile, NT>(a, g, job, lds.data(), out);
            });
        for (auto &x : t) x.join();
    }
}

template <int NT>
static void count(const StarArgs &a)
{
    std::vector<std::atomic<int>> n(a.N * a.N);
    const Count out{n.data()};
    for (int g = star_num_groups(a.J) - 1; g >= 0; --g) switch (a.group(g).L) {
        case 1: pass<NT, 1>(a, g, out); break;
        case 2: pass<NT, 2>(a, g, out); break;
        default: pass<NT, 3>(a, g, out); break;
        }
    int lo = 1 << 30, hi = 0;
    for (auto &v : n) lo = std::min(lo, v.load()), hi = std::max(hi, v.load());
    printf("%d %d %d\n", NT, lo, hi);
}

int main(int, char **v)
{
    StarArgs a;
    a.N = atoi(v[1]);
    a.J = atoi(v[2]);
    a.B = 1;
    std::vector<float> z((size_t)a.J * a.N * a.N, 1.f);
    std::vector<double> ca(a.N * a.N), cb(a.N * a.N);
    a.z = z.data();
    a.ca = ca.data();
    a.cb = cb.data();
    count<256>(a);
    count<512>(a);
}
