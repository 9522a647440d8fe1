// Streaming kernels around the backward sweeps: the V gradient of launches whose sweep stores the node
// gradients, the reduction of the private V-gradient accumulators, and fills.
#pragma once

#include "mrfmp_device.h"

// ---- grad V apart from the sweep (65..128 labels beside mrf_bwd_sweep_chain) --------------------
// Eq. supp-gradient-smoothness: entry (p(lambda), lambda) of the table receives theta_{i-r,i} g(lambda) at
// every replayed update.  Nothing of it depends on the order of the nodes, so where the chain layout has no
// room for the table its helpers store g per node and this streaming pass does the additions: one wavefront
// per node, lanes over lambda, the L x L table of a workgroup in LDS (`ds_add_f64`), added to the workgroup's
// slot at the end.
struct MrfGvParams {
    long long N;
    int L;
    const double *g;         // [N][L]
    const uint8_t *p;        // [N][L] of this direction and iteration
    const float *w;          // [N] edge weights of this direction, or the scalar at w[0] when w_mul == 0
    int w_mul;
    double *gV;              // [gridDim.x][L][L] slots
};

__global__ void __launch_bounds__(512) mrf_bwd_gv_from_g(const MrfGvParams P)
{
    extern __shared__ __align__(16) unsigned char mrf_gvsmem[];
    double *tile = reinterpret_cast<double *>(mrf_gvsmem);
    const int L = P.L;
    for (int e = threadIdx.x; e < L * L; e += blockDim.x) tile[e] = 0.0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const long long wave = (long long)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long nwaves = (long long)gridDim.x * (blockDim.x >> 6);
    for (long long i = wave; i < P.N; i += nwaves) {
        const double wgt = (double)P.w[(size_t)(i * P.w_mul)];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int lam = lane + 64 * s;
            if (lam < L) {
                const double g = P.g[(size_t)i * L + lam];
                if (g != 0.0) {
                    int pv = P.p[(size_t)i * L + lam];
                    pv = pv < L ? pv : L - 1;
                    __hip_atomic_fetch_add(&tile[__mul24(pv, L) + lam], wgt * g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        }
    }
    __syncthreads();
    double *slot = P.gV + (size_t)blockIdx.x * L * L;
    for (int e = threadIdx.x; e < L * L; e += blockDim.x) slot[e] += tile[e];
}

// Reduction of the wavefront-private V-gradient accumulators in a fixed order, two levels:
// first every chunk of `chunk` consecutive slots is summed into its first slot, then the
// chunk heads are summed into the output.
__global__ void __launch_bounds__(256) mrf_reduce_slot_chunks(double *buf, long long n, long long slots, long long chunk)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const long long first = (long long)blockIdx.y * chunk;
    const long long last = first + chunk < slots ? first + chunk : slots;
    double v = 0.0;
    for (long long s = first; s < last; ++s) v = v + buf[(size_t)s * n + e];
    buf[(size_t)first * n + e] = v;
}

__global__ void __launch_bounds__(256) mrf_reduce_slot_heads(const double *buf, float *dst, long long n, long long slots, long long chunk)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    double v = 0.0;
    for (long long s = 0; s < slots; s += chunk) v = v + buf[(size_t)s * n + e];
    dst[e] = (float)v;
}

__global__ void __launch_bounds__(256) mrf_fill_f64(double *dst, long long n, double val)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) dst[e] = val;
}

__global__ void __launch_bounds__(256) mrf_fill_f32(float *dst, long long n, float val)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) dst[e] = val;
}
