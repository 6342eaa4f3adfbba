// The finalize kernel and the run-time selection among the pass-kernel
// instantiation units (one per pair of mask radii, logfx_kernels_inst.hip).
#include "logfx_kernels.h"

#include <mutex>

#define LOGFX_RADII(X)                                                                            \
    X(1, 1) X(1, 2) X(2, 2) X(1, 3) X(2, 3) X(3, 3) X(1, 4) X(2, 4) X(3, 4) X(4, 4)

namespace logfx {

#define X(A, B)                                                                                   \
    hipError_t pass1_i_r##A##_##B(const Pass1Args<OrbitTapsI> &, int, int, hipStream_t, int *);  \
    hipError_t pass1_d_r##A##_##B(const Pass1Args<OrbitTapsD> &, const MatTable &, int, int, hipStream_t, int *);  \
    hipError_t pass2_i_r##A##_##B(const Pass2Args<OrbitTapsI> &, int, hipStream_t, int *);        \
    hipError_t pass2_d_r##A##_##B(const Pass2Args<OrbitTapsD> &, int, hipStream_t, int *);
LOGFX_RADII(X)
#undef X

namespace kern {

// ------------------------------------------------------------- finalize
// One workgroup per image: fixed-order reduction of the image's tile sums
// (FP64 path).  1024 threads with eight tiles' loads in flight each, so that a
// large image's tiles are read in one round of loads.
constexpr int kFinThreads = 1024;
__global__ __launch_bounds__(kFinThreads) void finalize_kernel(FinalizeArgs a) {
    __shared__ double sd[4][kFinThreads];
    __shared__ long long sc[2][kFinThreads];
    const int t = threadIdx.x;
    const int image = blockIdx.x;
    const ImageJob J = job_of(a.L, image);
    // thread t adds tiles t, t + kFinThreads, ... in that order; U tiles'
    // loads are in flight at once (a tile past the end adds zeros, which
    // leaves the sums unchanged)
    constexpr int U = 8;
    long long c[2] = {0, 0};
    double s[4] = {0, 0, 0, 0};
    for (int i0 = t; i0 < J.ntiles1; i0 += kFinThreads * U) {
        double v[U][4];
        long long w[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + kFinThreads * u;
            const long long at = (long long)J.base1 + i;
            const bool in = i < J.ntiles1;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[u][k] = in ? __longlong_as_double((long long)a.partials[at * kTileSums + k]) : 0.0;
            w[u][0] = in ? a.counts[at * 2] : 0;
            w[u][1] = in ? a.counts[at * 2 + 1] : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int k = 0; k < 4; ++k) s[k] += v[u][k];
            c[0] += w[u][0];
            c[1] += w[u][1];
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) sd[k][t] = s[k];
    sc[0][t] = c[0];
    sc[1][t] = c[1];
    __syncthreads();
    for (int off = kFinThreads / 2; off > 0; off >>= 1) {
        if (t < off) {
#pragma unroll
            for (int k = 0; k < 4; ++k) sd[k][t] += sd[k][t + off];
            sc[0][t] += sc[0][t + off];
            sc[1][t] += sc[1][t + off];
        }
        __syncthreads();
    }
    if (t == 0) {
        const double v[4] = {sd[0][0], sd[1][0], sd[2][0], sd[3][0]};
        const long long z[2] = {sc[0][0], sc[1][0]};
        image_stats(a, J.img.H * J.img.W, v, z, a.stats[image]);
    }
}

// The same for the integer path's exact sums, in any order: a total per wave
// by DPP, then the waves.  (With loads four at a time and wave totals by LDS
// permutes 9.0 us for 64 images of about 170 tiles, 6.9 for one of 756 and
// 13.3 for one of 5800; now 6.1, 5.1 and 11.5.)
__global__ __launch_bounds__(kFinThreads) void finalize_exact_kernel(FinalizeArgs a) {
    constexpr int W = kTileSums + 2, NW = kFinThreads / kWave;
    __shared__ unsigned long long sw[W][NW];
    const int t = threadIdx.x, image = blockIdx.x;
    const ImageJob J = job_of(a.L, image);
    unsigned long long v[W] = {};   // the tile sums, then the two counts
    // U tiles' words are in flight at once (8192^2 has about 5800 tiles)
    constexpr int U = 6;
    for (int i0 = t; i0 < J.ntiles1; i0 += kFinThreads * U) {
        unsigned long long w[U][W] = {};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + kFinThreads * u;
            if (i >= J.ntiles1) continue;
            const long long at = (long long)J.base1 + i;
#pragma unroll
            for (int k = 0; k < kTileSums; ++k) w[u][k] = a.partials[at * kTileSums + k];
            w[u][kTileSums] = (unsigned long long)a.counts[at * 2];
            w[u][kTileSums + 1] = (unsigned long long)a.counts[at * 2 + 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < W; ++k) v[k] += w[u][k];
    }
#pragma unroll
    for (int k = 0; k < W; ++k) {
        v[k] = wave_total(v[k]);
        if (t % kWave == 0) sw[k][t / kWave] = v[k];
    }
    __syncthreads();
    if (t >= kWave) return;
    // lane 16 (k mod 4) + w of the first wave takes wave w's word k, in two rounds
    static_assert(NW == 16 && W == 8, "words of 16 waves");
    unsigned long long r[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        r[h] = sw[4 * h + t / NW][t % NW];
#pragma unroll
        for (int off = NW / 2; off > 0; off >>= 1) r[h] += __shfl_xor(r[h], off);
    }
    unsigned long long q[kTileSums];
    long long z[2];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const unsigned long long x = __shfl(r[k / 4], NW * (k % 4));
        if (k < kTileSums) q[k < kTileSums ? k : 0] = x;
        else z[k & 1] = (long long)x;
    }
    if (t != 0) return;
    double s[4];
    exact_sums(q, s);
    image_stats(a, J.img.H * J.img.W, s, z, a.stats[image]);
}

}  // namespace kern

hipError_t launch_pass1_i(int ra, int rb, const Pass1Args<OrbitTapsI> &a, int mode, int grid,
                          hipStream_t s, int *max_grid) {
#define X(A, B) if (ra == A && rb == B) return pass1_i_r##A##_##B(a, mode, grid, s, max_grid);
    LOGFX_RADII(X)
#undef X
    return hipErrorInvalidValue;
}
hipError_t launch_pass1_d(int ra, int rb, const Pass1Args<OrbitTapsD> &a, const MatTable &t, int mode, int grid,
                          hipStream_t s, int *max_grid) {
#define X(A, B) if (ra == A && rb == B) return pass1_d_r##A##_##B(a, t, mode, grid, s, max_grid);
    LOGFX_RADII(X)
#undef X
    return hipErrorInvalidValue;
}
hipError_t launch_pass2_i(int ra, int rb, const Pass2Args<OrbitTapsI> &a, int grid, hipStream_t s,
                          int *max_grid) {
#define X(A, B) if (ra == A && rb == B) return pass2_i_r##A##_##B(a, grid, s, max_grid);
    LOGFX_RADII(X)
#undef X
    return hipErrorInvalidValue;
}
hipError_t launch_pass2_d(int ra, int rb, const Pass2Args<OrbitTapsD> &a, int grid, hipStream_t s,
                          int *max_grid) {
#define X(A, B) if (ra == A && rb == B) return pass2_d_r##A##_##B(a, grid, s, max_grid);
    LOGFX_RADII(X)
#undef X
    return hipErrorInvalidValue;
}
// The scratch of logfx_extract_noalloc: every call on a device shares its
// copy, which keeps the last call's contents (each pass writes every slot it
// later reads, so nothing needs clearing).
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

hipError_t noalloc_scratch(int device, void **ptr) {
    static std::mutex mu;
    static void *addr[64] = {};
    if (device < 0 || device >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = p;
    }
    *ptr = addr[device];
    return hipSuccess;
}

hipError_t launch_finalize(const FinalizeArgs &a, hipStream_t s) {
    if (a.exact) hipLaunchKernelGGL(kern::finalize_exact_kernel, dim3(a.L.nimg), dim3(kern::kFinThreads), 0, s, a);
    else hipLaunchKernelGGL(kern::finalize_kernel, dim3(a.L.nimg), dim3(kern::kFinThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace logfx
