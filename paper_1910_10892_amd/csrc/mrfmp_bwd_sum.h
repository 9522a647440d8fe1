// Streaming kernels around the backward sweeps: the pairwise gradients of launches whose sweep stores the node
// gradients, the gradient of per-edge tables, the reduction of the private V-gradient accumulators, and fills.
#pragma once

#include "mrfmp_device.h"

// ---- pairwise gradients apart from the sweep (33..128 labels beside mrf_bwd_sweep_chain) ------------
// Eq. supp-gradient-smoothness and Eq. supp-gradient-edge: at every replayed update, entry (p(lambda), lambda) of the
// table receives theta_{i-r,i} g(lambda), and theta_{i-r,i} receives sum_lambda g(lambda) V(p(lambda), lambda).
// Nothing of them depends on the order of the nodes, so where the chain layout has no room for the tables its
// helpers store g per node and a streaming pass does the rest: lanes over lambda, V and the table in LDS, the table
// added to the workgroup's slot at the end.  Bound by HBM (9 bytes per label); with a single node in flight per
// wavefront it was bound by the latency of the loads, 129 us at 256 x 512, 96 labels.
//   mrf_bwd_pairwise_own     33..64 labels: the wavefronts that add have a table each
//   mrf_bwd_pairwise_shared  65..128 labels: one table, to which all wavefronts add in the order they arrive
struct MrfGvParams {
    long long N;
    int L;
    const double *g;         // [N][L]
    const uint8_t *p;        // [N][L] of this direction and iteration
    const float *w;          // [N] edge weights of this direction, or the scalar at w[0] when w_mul == 0
    int w_mul;
    const float *V;          // [L][L]
    int v_lds;               // V fits in LDS next to the table (it does next to mrf_bwd_pairwise_own's)
    float *gw;               // [N] edge-weight gradient of this direction, accumulated, or NULL
    double *gV;              // [gridDim.x][L][L] slots
};

// V gradient and edge-weight gradient on wavefronts of their own: NA = 4 (49..64 labels) or 8 wavefronts add to tables
// of their own, which a workgroup sums in wavefront order, so the order of every addition is fixed; the others form the
// edge-weight gradient of the same 64 nodes, and find g and p in the cache.  Backward pass, TRWP, 256 x 512, 64 labels, 8
// directions, K = 2: 1.76 ms, 2.15 with both gradients on the four wavefronts (the label sums set the pace), 1.70 with one
// table for sixteen (no fixed order); 37 x 53 nodes 0.304 / 0.411 / 0.286.
template <int NA>
__global__ void __launch_bounds__(1024) mrf_bwd_pairwise_own(const MrfGvParams P)
{
    extern __shared__ __align__(16) unsigned char mrf_gvsmem[];
    double *tabs = reinterpret_cast<double *>(mrf_gvsmem);
    constexpr int CH = 64;                               // nodes of a turn
    constexpr int UA = CH / NA, UG = (CH + 15 - NA) / (16 - NA);      // of which a wavefront has
    const int L = P.L;
    float *vl = reinterpret_cast<float *>(tabs + NA * L * L);
    for (int e = threadIdx.x; e < NA * L * L; e += blockDim.x) tabs[e] = 0.0;
    for (int e = threadIdx.x; e < L * L; e += blockDim.x) vl[e] = P.V[e];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lc = lane < L ? lane : 0;
    if (wv < NA) {
        double *tile = tabs + wv * L * L;
        for (long long i0 = (long long)blockIdx.x * CH + wv * UA; i0 < P.N; i0 += (long long)gridDim.x * CH) {
            double g[UA];
            int pv[UA];
            float w[UA];
#pragma unroll
            for (int u = 0; u < UA; ++u) {
                const long long i = i0 + u < P.N ? i0 + u : P.N - 1;
                w[u] = P.w[(size_t)(i * P.w_mul)];
                g[u] = P.g[(size_t)i * L + lc];
                pv[u] = P.p[(size_t)i * L + lc];
            }
#pragma unroll
            for (int u = 0; u < UA; ++u) {
                const int pc = pv[u] < L ? pv[u] : L - 1;
                if (lane < L && i0 + u < P.N && g[u] != 0.0)
                    __hip_atomic_fetch_add(&tile[__mul24(pc, L) + lc], (double)w[u] * g[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    } else if (P.gw) {
        const int first = (wv - NA) * UG, count = CH - first < UG ? CH - first : UG;
        for (long long i0 = (long long)blockIdx.x * CH + first; count > 0 && i0 < P.N; i0 += (long long)gridDim.x * CH) {
            double g[UG];
            int pv[UG];
#pragma unroll
            for (int u = 0; u < UG; ++u) {
                const long long i = i0 + u < P.N ? i0 + u : P.N - 1;
                g[u] = P.g[(size_t)i * L + lc];
                pv[u] = P.p[(size_t)i * L + lc];
            }
            float mine = 0.0f;           // lane u: edge-weight gradient of node i0 + u
#pragma unroll
            for (int u = 0; u < UG; ++u) {
                const bool live = lane < L && g[u] != 0.0;
                const int pc = pv[u] < L ? pv[u] : L - 1;
                const float v = vl[__mul24(pc, L) + lc];
                const double acc = mrf_wave_sum_f64(live ? g[u] * (double)v : 0.0);
                if (lane == u) mine = (float)acc;
            }
            // one writer per entry and launch: a no-return atomic is a plain accumulate
            if (lane < count && i0 + lane < P.N)
                __hip_atomic_fetch_add(&P.gw[(size_t)(i0 + lane)], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    double *slot = P.gV + (size_t)blockIdx.x * L * L;
    for (int e = threadIdx.x; e < L * L; e += blockDim.x) {     // (no-return atomics as in mrf_slot_add)
        double v = tabs[e];
#pragma unroll
        for (int k = 1; k < NA; ++k) v += tabs[k * L * L + e];
        __hip_atomic_fetch_add(&slot[e], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ void __launch_bounds__(1024) mrf_bwd_pairwise_shared(const MrfGvParams P)
{
    extern __shared__ __align__(16) unsigned char mrf_gvsmem[];
    double *tile = reinterpret_cast<double *>(mrf_gvsmem);
    float *vl = reinterpret_cast<float *>(tile + P.L * P.L);
    constexpr int LP = 2;
    constexpr int U = 4;                 // nodes in flight per wavefront
    const int L = P.L;
    for (int e = threadIdx.x; e < L * L; e += blockDim.x) tile[e] = 0.0;
    if (P.v_lds)
        for (int e = threadIdx.x; e < L * L; e += blockDim.x) vl[e] = P.V[e];
    __syncthreads();
    const float *V = P.v_lds ? vl : P.V;
    const int lane = threadIdx.x & 63;
    const long long wave = (long long)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long nwaves = (long long)gridDim.x * (blockDim.x >> 6);
    int lc[LP];
#pragma unroll
    for (int s = 0; s < LP; ++s) lc[s] = lane + 64 * s < L ? lane + 64 * s : 0;
    for (long long i0 = wave * U; i0 < P.N; i0 += nwaves * U) {
        double g[U][LP];
        int at[U][LP];
        float w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const long long i = i0 + u < P.N ? i0 + u : P.N - 1;
            w[u] = P.w[(size_t)(i * P.w_mul)];
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                g[u][s] = P.g[(size_t)i * L + lc[s]];
                at[u][s] = P.p[(size_t)i * L + lc[s]];
            }
        }
        float mine = 0.0f;               // lane u: edge-weight gradient of node i0 + u
#pragma unroll
        for (int u = 0; u < U; ++u) {
            double acc = 0.0;
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const bool live = lane + 64 * s < L && i0 + u < P.N && g[u][s] != 0.0;
                const int pc = at[u][s] < L ? at[u][s] : L - 1;
                const int e = __mul24(pc, L) + lc[s];
                if (live) __hip_atomic_fetch_add(&tile[e], (double)w[u] * g[u][s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                // (both operands selected: V may be infinite where no update was replayed)
                if (P.gw) acc = __builtin_fma(live ? g[u][s] : 0.0, live ? (double)V[e] : 0.0, acc);
            }
            if (P.gw) {
                acc = mrf_wave_sum_f64(acc);
                if (lane == u) mine = (float)acc;
            }
        }
        // one writer per entry and launch: a no-return atomic is a plain accumulate
        if (P.gw && lane < U && i0 + lane < P.N)
            __hip_atomic_fetch_add(&P.gw[(size_t)(i0 + lane)], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    double *slot = P.gV + (size_t)blockIdx.x * L * L;
    for (int e = threadIdx.x; e < L * L; e += blockDim.x)       // (no-return atomics as in mrf_slot_add)
        __hip_atomic_fetch_add(&slot[e], tile[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- gradient of per-edge tables apart from the sweeps ---------------------------------------------
// Eq. supp-gradient-pairwise: entry (p(lambda), lambda) of an edge's own table receives g(lambda), once per iteration.
// Added in the sweeps, that is a read-modify-write of L scattered entries of every table in every iteration, behind a
// zero fill of all of them.  Here the sweeps store g (one float per label and node), and this pass writes every table
// once: a workgroup takes T neighbouring tables, which are one contiguous range, adds the g of `count` iterations to them
// in LDS (a thread per node and label, iterations one after the other: the order of the additions is that of the sweeps)
// and streams the range out.  With room for less than K iterations of g the passes behind the first one start from what
// is there.  Bound by the bytes of the tables.  256 x 256, 21 labels, 4 directions, K = 3: 118 us for 462 MB; the
// backward pass 693 -> 350 us.
struct MrfEdgeGradParams {
    long long tables;        // R * N
    int L, T;                // labels; tables per workgroup and turn
    int count;               // iterations in g
    const float *g;          // [count][R][N][L], the iteration that was processed first at the front
    const uint8_t *p;        // [R][N][L] of that iteration; the next one lies p_step bytes before it
    long long p_step;
    float *gE;               // [R][N][L][L]
    int accumulate;          // add to what gE holds
};

// VEC: gE and T L L allow accesses of four floats
template <bool VEC>
__global__ void __launch_bounds__(256) mrf_bwd_edge_tables(const MrfEdgeGradParams P)
{
    extern __shared__ __align__(16) float mrf_etile[];
    constexpr int W = VEC ? 4 : 1;
    typedef float vecf __attribute__((ext_vector_type(W)));
    const int L = P.L, LL = L * L, tid = threadIdx.x;
    vecf *tile = reinterpret_cast<vecf *>(mrf_etile);
    const long long turns = (P.tables + P.T - 1) / P.T;
    const size_t slab = (size_t)P.tables * L;
    if (!P.accumulate)
        for (int e = tid; e < P.T * LL / W; e += 256) tile[e] = vecf(0.0f);
    for (long long c = blockIdx.x; c < turns; c += gridDim.x) {
        const long long first = c * P.T;
        const int n = (int)(P.tables - first < P.T ? P.tables - first : P.T);     // tables of this turn
        vecf *out = reinterpret_cast<vecf *>(P.gE + (size_t)first * LL);
        const int whole = n * LL / W;
        if (P.accumulate) {
            __syncthreads();                             // (the turn before this one has left the tile)
            for (int e = tid; e < n * LL; e += 256) mrf_etile[e] = P.gE[(size_t)first * LL + e];
        }
        __syncthreads();
        for (int x = tid; x < n * L; x += 256) {
            const int node = x / L;
            float *col = mrf_etile + node * LL + (x - node * L);
            const float *g = P.g + (size_t)first * L + x;
            const uint8_t *p = P.p + (size_t)first * L + x;
            for (int k = 0; k < P.count; ++k) {
                const int mu = p[-(ptrdiff_t)k * P.p_step];
                col[(mu < L ? mu : L - 1) * L] += g[(size_t)k * slab];
            }
        }
        __syncthreads();
        for (int e = tid; e < whole; e += 256) {
            out[e] = tile[e];
            tile[e] = vecf(0.0f);
        }
        for (int e = whole * W + tid; e < n * LL; e += 256) {                     // (the last turn's ragged end)
            P.gE[(size_t)first * LL + e] = mrf_etile[e];
            mrf_etile[e] = 0.0f;
        }
        // (the next turn's additions wait at its first barrier)
    }
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
// sweeps add to.  Writes the workspace's header as well (mrf_init_header): a launch less.
__global__ void __launch_bounds__(256) mrf_bwd_clear(float *gw, long long n_gw, double *slots, long long n_slots, float *scalar, int *fault, float w)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) { *scalar = w; *fault = 0; }
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x, stride = (long long)gridDim.x * blockDim.x;
    for (long long e = t; e < n_gw; e += stride) gw[e] = 0.0f;
    for (long long e = t; e < n_slots; e += stride) slots[e] = 0.0;
}

__global__ void __launch_bounds__(256) mrf_fill_f32(float *dst, long long n, float val)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) dst[e] = val;
}
