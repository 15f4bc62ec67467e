// hmc_grains.hip -- grains of a spin field: the face-connected clusters of equal spins on the
// periodic lattice, the measure behind the mean grain volume V(t) of the grain-growth law of
// Sec. 6 (V^(2/3) linear in t).
//
// A union-find forest in the label array: a label is the index of a site of the same grain, never larger than
// the site's own, and a site that is its own label is a root.  Each site first points to the start of
// its run of equal spins in x (within its wavefront's 64 sites), a start to its lower neighbour in x, else y, else
// z; labels are then replaced by their roots; every pair of neighbours across whose
// roots still differ is united (the larger root takes the smaller as its label); and the roots are taken again.
// A root is linked only to a smaller one, so the forest ends with one tree a grain whose root is its smallest
// site, whatever the order.  A read that misses another block's latest write sees an older label, an
// ancestor all the same; a union that finds its root linked meanwhile goes on with what it found there.  Every
// walk and every union goes to strictly smaller indices, so all of them end.
//
// Four launches, bound by the latency of the walks, against rounds of neighbour minima until nothing changed with
// a read-back after each (21 of them at 100^3).  A call: grains of 100 sites at 100^3 782 -> 97 us, of 400 sites
// at 200^3 4.9 -> 0.40 ms, one grain of 320^3 2.8 -> 1.0 ms.
#include <numeric>

#include "hmc_device.h"

namespace hmc {

namespace {

__device__ __forceinline__ int32_t label_of(const int32_t* lab, int32_t v)
{
    return __hip_atomic_load(lab + v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int32_t root_of(const int32_t* lab, int32_t v)
{
    for (;;) {
        const int32_t l = label_of(lab, v);
        if (l == v) return v;
        v = l;
    }
}

__device__ __forceinline__ void unite(int32_t* lab, int32_t a, int32_t b)
{
    a = root_of(lab, a);
    b = root_of(lab, b);
    while (a != b) {
        if (a < b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        const int32_t old = atomicMin(lab + a, b);   // a > b
        if (old == a) return;                        // a was a root
        a = root_of(lab, old);                       // linked meanwhile: what it was linked to and b
        b = root_of(lab, b);
    }
}

__global__ __launch_bounds__(256) void k_label_init(const int16_t* __restrict__ spins, int32_t* lab, int K)
{
    const int64_t n3 = (int64_t)K * K * K, KK = (int64_t)K * K;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n3; v += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(v % K), y = (int)((v / K) % K);
        const int16_t s = spins[v];
        const bool on = x > 0 && spins[v - 1] == s;
        // the start of the run of equal spins in x, as far as the wavefront reaches
        const int lane = threadIdx.x & 63;
        const uint64_t starts = __builtin_amdgcn_ballot_w64(!on || lane == 0);
        const int back = lane - (63 - (int)__builtin_clzll(starts & (~0ull >> (63 - lane))));
        int64_t l = v - back;
        if (back == 0) {
            if (on)
                l = v - 1;
            else if (y > 0 && spins[v - K] == s)
                l = v - K;
            else if (v >= KK && spins[v - KK] == s)
                l = v - KK;
        }
        lab[v] = (int32_t)l;
    }
}

// Labels to roots; with COUNT the roots are counted.
template <bool COUNT>
__global__ __launch_bounds__(256) void k_label_roots(int32_t* lab, int64_t n3, unsigned long long* count)
{
    unsigned int n = 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n3; v += (int64_t)gridDim.x * blockDim.x) {
        const int32_t l = lab[v], r = root_of(lab, l);
        if (r != l) lab[v] = r;
        n += r == (int32_t)v;
    }
    if (COUNT) block_count_to(count, n, 1);
}

__global__ __launch_bounds__(256) void k_label_unite(const int16_t* __restrict__ spins, int32_t* lab, int K)
{
    const int64_t n3 = (int64_t)K * K * K, KK = (int64_t)K * K;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n3; v += (int64_t)gridDim.x * blockDim.x) {
        const int x = (int)(v % K), y = (int)((v / K) % K);
        const int16_t s = spins[v];
        const int64_t nb[3] = {x + 1 < K ? v + 1 : v + 1 - K, y + 1 < K ? v + K : v + K - KK,
                               v + KK < n3 ? v + KK : v + KK - n3};
        const int32_t l = lab[v];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (spins[nb[k]] == s) {
                const int32_t m = lab[nb[k]];
                if (m != l) unite(lab, l, m);
            }
    }
}

unsigned grid_of(int64_t n)
{
    const int64_t b = (n + 255) / 256;
    return (unsigned)(b < 8192 ? (b > 0 ? b : 1) : 8192);
}

}  // namespace

hipError_t launch_grain_labels(hmc_ctx_s* c, int rep, int32_t* lab, int64_t* n_grains)
{
    const RepDev& R = c->reps[rep];
    const int64_t n3 = R.n3;
    const unsigned g = grid_of(n3);
    const int16_t* spins = c->d.spins + R.site_off;
    unsigned long long cnt[kCountCopies];
    hipError_t e = hipMemsetAsync(c->d.bonds, 0, sizeof cnt, c->stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_label_init, dim3(g), dim3(256), 0, c->stream, spins, lab, R.K);
    hipLaunchKernelGGL(k_label_roots<false>, dim3(g), dim3(256), 0, c->stream, lab, n3, c->d.bonds);
    hipLaunchKernelGGL(k_label_unite, dim3(g), dim3(256), 0, c->stream, spins, lab, R.K);
    hipLaunchKernelGGL(k_label_roots<true>, dim3(g < 2048 ? g : 2048), dim3(256), 0, c->stream, lab, n3, c->d.bonds);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(cnt, c->d.bonds, sizeof cnt, hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e == hipSuccess) *n_grains = (int64_t)std::accumulate(cnt, cnt + kCountCopies, 0ull);
    return e;
}

}  // namespace hmc
