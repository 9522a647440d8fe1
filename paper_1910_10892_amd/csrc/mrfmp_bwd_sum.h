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

// Bound by the latency of the loads unless several nodes are in flight per wavefront: with one, 2,048 wavefronts
// took 129 us for the 113 MB of a 256 x 512 grid with 96 labels.
__global__ void __launch_bounds__(512) mrf_bwd_gv_from_g(const MrfGvParams P)
{
    extern __shared__ __align__(16) unsigned char mrf_gvsmem[];
    double *tile = reinterpret_cast<double *>(mrf_gvsmem);
    constexpr int U = 4;                 // nodes in flight per wavefront
    const int L = P.L;
    for (int e = threadIdx.x; e < L * L; e += blockDim.x) tile[e] = 0.0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const long long wave = (long long)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long nwaves = (long long)gridDim.x * (blockDim.x >> 6);
    const int lc0 = lane < L ? lane : 0, lc1 = lane + 64 < L ? lane + 64 : 0;
    for (long long i0 = wave * U; i0 < P.N; i0 += nwaves * U) {
        double g[U][2];
        int pv[U][2];
        float w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long i = i0 + u < P.N ? i0 + u : P.N - 1;
            w[u] = P.w[(size_t)(i * P.w_mul)];
            g[u][0] = P.g[(size_t)i * L + lc0];
            g[u][1] = P.g[(size_t)i * L + lc1];
            pv[u][0] = P.p[(size_t)i * L + lc0];
            pv[u][1] = P.p[(size_t)i * L + lc1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int lam = lane + 64 * s;
                if (lam < L && i0 + u < P.N && g[u][s] != 0.0) {
                    const int pc = pv[u][s] < L ? pv[u][s] : L - 1;
                    __hip_atomic_fetch_add(&tile[__mul24(pc, L) + lam], (double)w[u] * g[u][s], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
    }
    __syncthreads();
    double *slot = P.gV + (size_t)blockIdx.x * L * L;
    for (int e = threadIdx.x; e < L * L; e += blockDim.x)       // (no-return atomics as in mrf_slot_add)
        __hip_atomic_fetch_add(&slot[e], tile[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Reduction of the V-gradient slots in a fixed order.  A workgroup takes ENT entries of the table and 256 / ENT
// threads per entry, which walk the slots in steps of that many, several loads in flight each; their sums meet
// in LDS in thread order.  With up to MRF_SLOTS_ONE_PASS slots one launch with chunk = 1 forms the output; beyond
// that a first launch (grid y = chunks) sums every chunk of `chunk` consecutive slots into its first.
#define MRF_SLOTS_ONE_PASS 512
template <int ENT>
__global__ void __launch_bounds__(256) mrf_reduce_slots(double *buf, float *dst, long long n, long long slots, long long chunk, int heads)
{
    constexpr int SUB = 256 / ENT;
    __shared__ double part[SUB][ENT];
    const int x = threadIdx.x % ENT, sub = threadIdx.x / ENT;
    const long long e = (long long)blockIdx.x * ENT + x;
    // heads: the first slots of the chunks (all slots where chunk is 1); else the slots of chunk blockIdx.y
    const long long first = heads ? 0 : (long long)blockIdx.y * chunk;
    const long long last = heads ? slots : (first + chunk < slots ? first + chunk : slots);
    const long long step = heads ? chunk : 1;
    double v = 0.0;
    if (e < n) {
        const double *at = buf + (size_t)e;
#pragma unroll 8
        for (long long s = first + sub * step; s < last; s += SUB * step) v += at[(size_t)s * n];
    }
    part[sub][x] = v;
    __syncthreads();
    if (sub == 0 && e < n) {
#pragma unroll
        for (int k = 1; k < SUB; ++k) v += part[k][x];
        if (heads) dst[e] = (float)v;
        else buf[(size_t)first * n + e] = v;
    }
}

// What a backward call sets to zero before its sweeps: the edge-weight gradient and the V-gradient slots its
// sweeps add to.
__global__ void __launch_bounds__(256) mrf_bwd_clear(float *gw, long long n_gw, double *slots, long long n_slots)
{
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x, stride = (long long)gridDim.x * blockDim.x;
    for (long long e = t; e < n_gw; e += stride) gw[e] = 0.0f;
    for (long long e = t; e < n_slots; e += stride) slots[e] = 0.0;
}

__global__ void __launch_bounds__(256) mrf_fill_f32(float *dst, long long n, float val)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) dst[e] = val;
}
