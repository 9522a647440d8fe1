// Backward passes of ISGMR (Alg. 3) and TRWP (Alg. 4): replay of the stored indices p, q
// in reverse scanline order.
//
// One wavefront walks one scanline from its last node back to its first; lanes own labels
// (lambda = lane + 64*s).  Per node: reparametrisation backward through q
// (Eq. supp-isgmr-back-norm), edge-weight gradient (Eq. supp-gradient-edge), V gradient
// (Eq. supp-gradient-smoothness) into an accumulator private to the wavefront, and the
// index scatter s(mu) = sum_{lambda : p(lambda) = mu} g(lambda) through a wavefront-private
// LDS vector.  What the same direction passes on to node i-r stays in registers; nothing
// the sweep reads from memory depends on the previous node, so all of it is prefetched a
// group of D nodes ahead.
//
// A sweep never read-modify-writes message gradients.  It stores s per (direction, node)
// and later sweeps rebuild the gradient of a message from those stores:
//   ISGMR  all directions of an iteration run in one launch; mrf_isgmr_bwd_combine then forms
//          grad theta_i += sum_r s^r_i and grad m^d_i = sum_{r not in {d,d-}} s^r_i.
//   TRWP   directions run one after the other (reverse forward order).  Between two sweeps
//          of direction d every other direction r sweeps exactly once and adds
//          rho_r s^r_i (minus s^r_i if r = d-) to grad m^d_i (Alg. 4 lines 10-11), after
//          which grad m^d is reset; so the sweep of d reads the latest s^r of the other
//          directions and sums them with those coefficients (plus grad c in the first
//          processed iteration).  The sweep of direction 0 also owns grad theta_i.
//
// Precision: tensors in memory are float; the chain a scanline carries from node to node
// (message gradient, its label sum, the scatter sums) and the V-gradient accumulators are
// kept in double, so that rounding does not build up along a scanline.  On this chip
// double adds issue at the same rate as unpacked float adds.
//
// Kernels in this file:
//   mrf_bwd_sweep          one wavefront per scanline (the description above)
//   mrf_bwd_sweep_chain    the node-to-node chain on a wavefront of its own, helper wavefronts
//                          for everything else (launches with few scanlines)
//   mrf_bwd_sweep_split    one wavefront per 64 labels in lock step
//   mrf_bwd_sweep_packed   L <= 32: several scanlines per wavefront, one label per lane; arrays of any size
//   mrf_bwd_sweep_narrow   L <= 32: up to eight scanlines per wavefront, several labels per lane; with five template
//                          parameters the work of a node divided among four wavefronts
//   mrf_isgmr_bwd_combine  ISGMR's sums over directions between two iterations
// Which sweep a launch gets is host arithmetic on the launch shape (dispatch_bwd).
#pragma once

#include "mrfmp_device.h"

struct MrfBwdParams {
    MrfGeom g;
    int r_first, r_count;
    long long blk_begin[MRF_MAXR + 1];     // prefix sums of B*nscan over the launch's directions
    long long total_scanlines;
    int pack_begin[MRF_MAXR + 1];          // mrf_bwd_sweep_narrow: the same in wavefronts, every direction padded to whole ones
    int pack_first;                        // mrf_bwd_sweep_narrow: first of those wavefronts in this launch
    const float *V;
    const float *w;                        // [R][N] edge weights, or one float when w_mul == 0
    int w_mul;
    const uint8_t *p, *q;                  // [R][N][L], [R][N] of this iteration
    // incoming message gradient of direction d at node i = sum_c coefG[d][c] * src_c[i], where
    // src_c = src_base + src_dir[d][c] * src_stride for c < n_src[d]; slot n_src[d] is grad c
    // when use_gc is set
    const float *src_base;
    long long src_stride;
    signed char src_dir[MRF_MAXR][MRF_MAXR];
    signed char n_src[MRF_MAXR];
    float coefG[MRF_MAXR][MRF_MAXR];
    float coefT[MRF_MAXR][MRF_MAXR];       // coefficients of the same sources in grad theta_i
    const float *gc;
    int use_gc;
    float *S;                              // [R][N][L] out: s of direction d at node i-d
    float *gunary;                         // [N][L]
    int unary_dir;                         // direction whose sweep forms grad theta_i, or -1
    int unary_init;                        // grad theta_i is assigned (first iteration) / accumulated
    float *gw;                             // [R][N] or NULL, accumulated over iterations
    double *gV;                            // [slots][L][L] or NULL, one slot per wavefront
    int gv_lds;                            // grad V accumulates in LDS: 1 = a table per wavefront, flushed once per wavefront;
                                           // 2 = one table per workgroup (LDS adds), flushed once into the workgroup's slot
    int v_mode;                            // V for grad w: 0 global, 1 copy in LDS, 2 first row in LDS
    int hot_label;                         // pre-reduce the most popular scatter target (truncated models)
    float carry_scale[MRF_MAXR];           // rho_d (TRWP) or 1 (ISGMR)
    const float *rho_e;                    // [R][N] rho of edge (i-r, i) at node i (TRWP), or NULL: then
                                           // coefG / coefT / carry_scale hold the per-direction values
    float *gE;                             // [R][N][L][L] gradient of per-edge pairwise tables (zeroed by the host,
                                           // accumulated over iterations), or NULL; mrf_bwd_sweep<..., RHOE> only
    int force_plain;                       // the problem has no V: only mrf_bwd_sweep may run
    double *gstore_buf;                    // [N][L] room for gstore (workspace), or NULL
    double *gstore;                        // mrf_bwd_sweep_chain: if not NULL, its helpers store the gradient vector g of
                                           // every node here (0 where no update is replayed) for mrf_bwd_pairwise_*,
                                           // which forms both pairwise gradients from it
    float *gstore32;                       // [R][N][L] the same in float for the gradient of per-edge tables (mrf_bwd_edge_tables)
    int edge;                              // a problem with per-edge tables whose sweeps leave their gradient to that pass:
                                           // no V, no edge-weight gradient
    int *fault;                            // launch-wide word raised when a wait between wavefronts is given up (mrf_wait_turn)
    int spin_limit;                        // microseconds after which a wait is given up
};

#define MRF_BWD_WAVES 4   // wavefronts (= scanlines in flight) per workgroup

// Adds to an entry of a V-gradient slot.  An entry has one writer per launch, so the order of its additions
// is fixed; the no-return atomic keeps the end of a sweep from waiting a memory round trip for every 64 entries
// of the table (7 of them for 21 labels: 5 us of a 14 us launch).
__device__ inline void mrf_slot_add(double *slot, double v)
{
    __hip_atomic_fetch_add(slot, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
#define MRF_CHAIN_MAX_HELPERS 12

// dynamic LDS of mrf_bwd_sweep_chain (host and device agree through these two expressions)
__host__ __device__ constexpr int mrf_bwd_chain_pitch(int LP, bool hot) { return 64 * LP + (hot ? 8 : 0); }
__host__ __device__ inline size_t mrf_bwd_chain_lds_bytes(int LP, int NI, int L, bool hot, bool tables, bool row)
{
    const size_t NR = 2 * (size_t)NI, LL = 64 * (size_t)LP;
    const size_t arrays = sizeof(double) * (NR * (size_t)mrf_bwd_chain_pitch(LP, hot) + NR * LL + (row ? (size_t)L : 0) + (tables ? (size_t)NI * L * L : 0)) +
                          sizeof(int) * (3 * MRF_CHAIN_MAX_HELPERS + 1) + sizeof(float) * (tables ? (size_t)L * L : 0) + sizeof(uint16_t) * NR * LL;
    return (arrays + 7) / 8 * 8 + sizeof(MrfWaitBlock);      // the deadline of the waits sits behind the arrays
}

// LP labels per lane, NS source slots, D prefetch distance, VG: V for the edge-weight
// gradient is gathered from global memory (it fits neither LDS layout), HOT: pre-reduce the
// most popular scatter target, RHOE: the per-edge extras.  TRW coefficients per edge (P.rho_e)
// instead of per direction: what direction c scattered to node i came over the edge (i, i+c)
// and carries that edge's rho.  Gradient of per-edge pairwise tables (P.gE): entry
// (p(lambda), lambda) of the edge's table receives g(lambda) (Eq. supp-gradient-pairwise).
// UNARY = false: no direction of the launch forms grad theta_i (P.unary_dir < 0: ISGMR leaves it to
// mrf_isgmr_bwd_combine), so nothing of it is loaded or kept in registers.
// WAVES: wavefronts per workgroup (more of them share the one V-gradient table of P.gv_lds == 2).
// FULL: the launch has exactly 64 LP labels (the host checks it), so every label test folds away and the
// strides are constants.
template <int LP, int NS, int D, bool VG, bool HOT, bool RHOE = false, bool UNARY = true, int WAVES = MRF_BWD_WAVES, bool FULL = false>
__global__ void __launch_bounds__(64 * WAVES) mrf_bwd_sweep(const MrfBwdParams P)
{
    extern __shared__ __align__(16) unsigned char mrf_bsmem[];
    const int L = FULL ? 64 * LP : P.g.L;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // uniform, and known to be
    double *sbuf = reinterpret_cast<double *>(mrf_bsmem) + wv * 64 * LP;
    double *gvl = reinterpret_cast<double *>(mrf_bsmem) + WAVES * 64 * LP + (P.gv_lds == 1 ? wv * L * L : 0);
    float *vl = reinterpret_cast<float *>(reinterpret_cast<double *>(mrf_bsmem) + WAVES * 64 * LP +
                                          (P.gv_lds == 1 ? WAVES * L * L : (P.gv_lds == 2 ? L * L : 0)));
    const long long slot = (long long)blockIdx.x * WAVES + wv;
    const long long nslots = (long long)gridDim.x * WAVES;
    const long long N = P.g.N;
    double *gVs = P.gV ? P.gV + (size_t)(P.gv_lds == 2 ? (long long)blockIdx.x : slot) * L * L : nullptr;
    const int vzero = mrf_opaque_zero();

    if (P.v_mode == 1)
        for (int e = threadIdx.x; e < L * L; e += blockDim.x) vl[e] = P.V[e];
    else if (P.v_mode == 2)
        for (int e = threadIdx.x; e < L; e += blockDim.x) vl[e] = P.V[e];
    if (gVs && P.gv_lds == 1)
        for (int e = lane; e < L * L; e += 64) gvl[e] = 0.0;
    if (gVs && P.gv_lds == 2)
        for (int e = threadIdx.x; e < L * L; e += blockDim.x) gvl[e] = 0.0;
    __syncthreads();

    for (long long sl = slot; sl < P.total_scanlines; sl += nslots) {
        const int ri = mrf_direction_of(P.blk_begin, P.r_count, sl);
        const int r = P.r_first + ri;
        const unsigned local = (unsigned)(sl - P.blk_begin[ri]);
        const unsigned nsc = (unsigned)P.g.nscan[r];
        const int b = (int)(local / nsc);
        const unsigned t = local - (unsigned)b * nsc;
        const int dh = P.g.dh[r], dw = P.g.dw[r];
        int y0, x0, len;
        mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
        const long long head = ((long long)b * P.g.H + y0) * P.g.W + x0;
        const long long nstep = (long long)dh * P.g.W + dw;
        const double cscale = (double)P.carry_scale[r];
        const bool own_unary = UNARY && (r == P.unary_dir);
        const bool unary_old = own_unary && !P.unary_init;
        const size_t umul = unary_old ? 1 : 0;
        const float *wbase = P.w + (P.w_mul ? (size_t)r * N : 0);
        const uint8_t *pbase = P.p + (size_t)r * N * L;
        const uint8_t *qbase = P.q + (size_t)r * N;

        // source slots; unused ones re-read grad c / the first source with coefficient 0
        const float *src[NS];
        double cG[NS], cT[NS];
        const int nsrc = P.n_src[r];
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            const bool live = c < nsrc;
            const bool isgc = (c == nsrc) && P.use_gc;
            src[c] = live ? P.src_base + (size_t)P.src_dir[r][c] * P.src_stride : P.gc;
            cG[c] = live ? (double)P.coefG[r][c] : (isgc ? 1.0 : 0.0);
            cT[c] = live ? (double)P.coefT[r][c] : (isgc ? 1.0 : 0.0);
        }
        // per-edge rho: where to find the rho of the edge that source slot c used at a node
        const float *rsrc[NS];
        long long rstep[NS];
        double ropp[NS];
        bool rlive[NS];
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            const int sd = (RHOE && c < nsrc) ? P.src_dir[r][c] : r;
            rlive[c] = RHOE && P.rho_e && c < nsrc;
            rsrc[c] = (RHOE && P.rho_e) ? P.rho_e + (size_t)sd * N : nullptr;
            rstep[c] = (long long)P.g.dh[sd] * P.g.W + P.g.dw[sd];
            ropp[c] = (sd == P.g.opp[r]) ? 1.0 : 0.0;
        }

        // the last node of the scanline has no successor in direction r
        {
            const long long last = head + (long long)(len - 1) * nstep;
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const int lam = lane + 64 * s;
                if (lam < L) P.S[((size_t)r * N + last) * L + lam] = 0.0f;
            }
        }

        // prefetch registers: step tt handles node len-1-tt (clamped at the first node)
        float cur[D][NS][LP], nxt[D][NS][LP];
        float ucur[D][UNARY ? LP : 1], unxt[D][UNARY ? LP : 1];       // old grad theta_i (only read when accumulating)
        int pcur[D][LP], pnxt[D][LP];
        int qcur[D], qnxt[D];
        float wcur[D], wnxt[D];
        float rcur[D][NS + 1], rnxt[D][NS + 1];   // RHOE: rho of each source slot's edge, then of this direction's own edge
        auto prefetch = [&](float (&dst)[NS][LP], float (&udst)[UNARY ? LP : 1], int (&pdst)[LP], int &qdst, float &wdst,
                            float (&rdst)[NS + 1], int tt) {
            int n = len - 1 - tt;
            n = n > 0 ? n : 0;
            const long long i = head + (long long)n * nstep;
            if (RHOE && P.rho_e) {
                // (a node without successor in direction c got zeros from that direction: any
                // finite coefficient will do, so the index is only kept inside the array)
#pragma unroll
                for (int c = 0; c < NS; ++c) {
                    long long e = i + rstep[c];
                    e = e < 0 ? 0 : (e > N - 1 ? N - 1 : e);
                    rdst[c] = rsrc[c][(size_t)e + vzero];
                }
                rdst[NS] = P.rho_e[(size_t)r * N + i + vzero];
            }
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const int lam = lane + 64 * s;
                const int lc = lam < L ? lam : 0;
#pragma unroll
                for (int c = 0; c < NS; ++c) dst[c][s] = src[c][(size_t)i * L + lc];
                if constexpr (UNARY) udst[s] = P.gunary[((size_t)i * L + lc) * umul];   // one cached word unless it is needed
                pdst[s] = pbase[(size_t)i * L + lc];
            }
            qdst = qbase[(size_t)i + vzero];
            wdst = wbase[(size_t)(i * P.w_mul) + vzero];
        };
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(cur[u], ucur[u], pcur[u], qcur[u], wcur[u], rcur[u], u);

        double carry[LP];   // what node i+r of this direction passed back to node i
#pragma unroll
        for (int s = 0; s < LP; ++s) { carry[s] = 0.0; sbuf[lane + 64 * s] = 0.0; }
        mrf_wave_lds_fence();

        for (int t0 = 0; t0 < len; t0 += D) {
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(nxt[u], unxt[u], pnxt[u], qnxt[u], wnxt[u], rnxt[u], t0 + D + u);
#pragma unroll
            for (int u = 0; u < D; ++u) {
                // Steps past the first node (last group only) and the first node itself run the
                // same instructions with their stores switched off, so that the loop body has no
                // branches around the prefetched registers.
                const int tt = t0 + u;
                const bool past = tt >= len;
                const int n = past ? 0 : len - 1 - tt;
                const bool update = !past && n > 0;      // node i has a predecessor: replay its update
                const long long i = head + (long long)n * nstep;
                const long long j = i - nstep;
                double cGn[NS], cTn[NS];
#pragma unroll
                for (int c = 0; c < NS; ++c) {
                    // Alg. 4 lines 9-11 with the rho of the edge (i, i+c): rho s to every direction
                    // and to grad theta, minus s to the opposite direction
                    cGn[c] = rlive[c] ? (double)rcur[u][c] - ropp[c] : cG[c];
                    cTn[c] = rlive[c] ? (double)rcur[u][c] : cT[c];
                }
                const double cscale_n = (RHOE && P.rho_e) ? (double)rcur[u][NS] : cscale;
                double g[LP];
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    double acc = carry[s];
#pragma unroll
                    for (int c = 0; c < NS; ++c) acc = __builtin_fma(cGn[c], (double)cur[u][c][s], acc);
                    g[s] = (lane + 64 * s < L) ? acc : 0.0;
                }
                if constexpr (UNARY) if (own_unary) {
                    // grad theta_i: everything every direction passed back to node i
#pragma unroll
                    for (int s = 0; s < LP; ++s) {
                        double accT = carry[s];
#pragma unroll
                        for (int c = 0; c < NS; ++c) accT = __builtin_fma(cTn[c], (double)cur[u][c][s], accT);
                        accT += unary_old ? (double)ucur[u][s] : 0.0;   // (the buffer may hold anything at first)
                        if (!past && lane + 64 * s < L) P.gunary[(size_t)i * L + lane + 64 * s] = (float)accT;
                    }
                }
                int pv[LP];
                double part = 0.0;
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    pv[s] = pcur[u][s] < L ? pcur[u][s] : L - 1;
                    part += g[s];
                }
                // Truncated models send most labels to one source label (the far-field minimiser),
                // which would serialise the LDS adds below.  Guess that label from p at the first
                // and at the last label (one of the two is far from it), take the commoner of the
                // two, and sum its lanes with a DPP tree instead.
                // (Only worth its instructions when the launch is not latency bound or L is large.)
                int hot = -1;
                double hpart = 0.0;
                if (HOT) {
                    const int c0 = __builtin_amdgcn_readlane(pv[0], 0);
                    int c1 = c0;
#pragma unroll
                    for (int s = 0; s < LP; ++s)
                        if (((L - 1) >> 6) == s) c1 = __builtin_amdgcn_readlane(pv[s], (L - 1) & 63);
                    int n0 = 0, n1 = 0;
#pragma unroll
                    for (int s = 0; s < LP; ++s) {
                        const bool vld = lane + 64 * s < L;
                        n0 += __popcll(__ballot(vld && pv[s] == c0));
                        n1 += __popcll(__ballot(vld && pv[s] == c1));
                    }
                    hot = n1 > n0 ? c1 : c0;
#pragma unroll
                    for (int s = 0; s < LP; ++s)
                        if (lane + 64 * s < L && pv[s] == hot) hpart += g[s];
                }
                // back Eq. isgmr-norm: g(q) -= sum_lambda g(lambda)
                double tot, hsum = 0.0;
                int qv = __builtin_amdgcn_readfirstlane(qcur[u]);
                qv = qv < L ? qv : L - 1;
                // HOT: the edge-weight gradient sum_lambda g(lambda) V(p(lambda), lambda) is formed from g
                // before the correction at q, in the same reduction as the two other sums, and corrected
                // by tot V(p(q), q) afterwards
                double gw_sum = 0.0;
                if (HOT) {
                    double wpart = 0.0;
                    float vq = 0.0f;
                    if (P.gw) {
#pragma unroll
                        for (int s = 0; s < LP; ++s) {
                            const int lam = lane + 64 * s;
                            const int dist = pv[s] > lam ? pv[s] - lam : lam - pv[s];
                            const float vv = lam < L ? vl[P.v_mode == 1 ? __mul24(pv[s], L) + lam : dist] : 0.0f;
                            wpart = __builtin_fma(g[s], (double)vv, wpart);       // (g is 0 beyond L)
                            if ((qv >> 6) == s) vq = mrf_readlane_f32(vv, qv & 63);
                        }
                    }
                    mrf_wave_sum3_f64(part, hpart, wpart, tot, hsum, gw_sum);
                    int pq = 0;
#pragma unroll
                    for (int s = 0; s < LP; ++s)
                        if ((qv >> 6) == s) pq = __builtin_amdgcn_readlane(pv[s], qv & 63);
                    if (pq == hot) hsum -= tot;
                    gw_sum = __builtin_fma(-tot, (double)vq, gw_sum);
                } else {
                    tot = mrf_wave_sum_f64(part);
                }
#pragma unroll
                for (int s = 0; s < LP; ++s)
                    if (lane + 64 * s == qv) g[s] = g[s] - tot;

                // index scatter through LDS: s(mu) = sum over lambda with p(lambda) = mu
                // (sbuf was cleared right after the previous step read it)
#pragma unroll
                for (int s = 0; s < LP; ++s)
                    if (lane + 64 * s < L && pv[s] != hot)
                        __hip_atomic_fetch_add(&sbuf[pv[s]], g[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                mrf_wave_lds_fence();
                double sv[LP];
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    sv[s] = sbuf[lane + 64 * s];
                    if (lane + 64 * s == hot) sv[s] += hsum;
                }
                mrf_wave_lds_fence();
#pragma unroll
                for (int s = 0; s < LP; ++s) sbuf[lane + 64 * s] = 0.0;
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int lam = lane + 64 * s;
                    if (update && lam < L) P.S[((size_t)r * N + j) * L + lam] = (float)sv[s];
                    carry[s] = cscale_n * sv[s];
                }

                // pairwise gradients (off the node-to-node chain)
                const double wgt = (double)wcur[u];
                if (HOT && P.gw) {
                    if (update && lane == 0)
                        __hip_atomic_fetch_add(&P.gw[(size_t)r * N + i], (float)gw_sum, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                } else if (P.gw) {
                    double acc = 0.0;
#pragma unroll
                    for (int s = 0; s < LP; ++s) {
                        const int lam = lane + 64 * s;
                        if (lam < L) {
                            float vv;
                            if (VG) {
                                vv = P.V[(size_t)__mul24(pv[s], L) + lam];
                            } else {
                                const int dist = pv[s] > lam ? pv[s] - lam : lam - pv[s];
                                vv = vl[P.v_mode == 1 ? __mul24(pv[s], L) + lam : dist];
                            }
                            acc = __builtin_fma(g[s], (double)vv, acc);
                        }
                    }
                    acc = mrf_wave_sum_f64(acc);
                    // one writer per entry and launch: a no-return atomic is a plain accumulate
                    // that does not make the wavefront wait for the old value
                    if (update && lane == 0)
                        __hip_atomic_fetch_add(&P.gw[(size_t)r * N + i], (float)acc, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                }
                if (RHOE && P.gE) {
                    // one writer per table and launch: plain read-modify-write
#pragma unroll
                    for (int s = 0; s < LP; ++s) {
                        const int lam = lane + 64 * s;
                        if (update && lam < L) {
                            float *e = P.gE + (((size_t)r * N + i) * L + pv[s]) * L + lam;
                            *e = *e + (float)g[s];
                        }
                    }
                }
                if (gVs) {
                    // lane lambda owns column lambda of the wavefront's private accumulator
#pragma unroll
                    for (int s = 0; s < LP; ++s) {
                        const int lam = lane + 64 * s;
                        if (update && lam < L) {
                            if (P.gv_lds == 1) gvl[__mul24(pv[s], L) + lam] = __builtin_fma(wgt, g[s], gvl[__mul24(pv[s], L) + lam]);
                            else if (P.gv_lds == 2) __hip_atomic_fetch_add(&gvl[__mul24(pv[s], L) + lam], wgt * g[s], __ATOMIC_RELAXED,
                                                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                            else __hip_atomic_fetch_add(&gVs[(size_t)__mul24(pv[s], L) + lam], wgt * g[s],
                                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < D; ++u) {
                qcur[u] = qnxt[u];
                wcur[u] = wnxt[u];
#pragma unroll
                for (int c = 0; c <= NS; ++c) rcur[u][c] = rnxt[u][c];
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    if constexpr (UNARY) ucur[u][s] = unxt[u][s];
                    pcur[u][s] = pnxt[u][s];
#pragma unroll
                    for (int c = 0; c < NS; ++c) cur[u][c][s] = nxt[u][c][s];
                }
            }
        }
    }
    if (gVs && P.gv_lds == 1) {
        mrf_wave_lds_fence();
        for (int e = lane; e < L * L; e += 64) mrf_slot_add(&gVs[e], gvl[e]);
    }
    if (P.gv_lds == 2) {
        // (every wavefront of the workgroup arrives here; the slot belongs to this workgroup alone)
        __syncthreads();
        if (gVs)
            for (int e = threadIdx.x; e < L * L; e += blockDim.x) mrf_slot_add(&gVs[e], gvl[e]);
    }
}

// Arguments of mrf_bwd_sweep_chain, laid out by the host so that a wavefront has little to work out before its first
// loads (a launch on a small image is mostly that): per direction of the launch, not of the problem, and the sources as pointers.
struct MrfChainParams {
    int B, H, W, L, w_mul, r_first, r_count;
    long long N;
    int begin[MRF_MAXR + 1];               // prefix sums of B*nscan over the launch's directions
    int dh[MRF_MAXR], dw[MRF_MAXR], nscan[MRF_MAXR];
    float carry_scale[MRF_MAXR];
    // direction ri reads src[ri * src_pitch + c], c < n_src[ri]; cg: coefficient in the message gradient, cd: that in
    // grad theta less cg.  (Twice as long as they can be filled: a kernel reads as many entries as it has slots.)
    int src_pitch, n_src[MRF_MAXR];
    const float *src[2 * MRF_MAXR];
    double cg[2 * MRF_MAXR], cd[2 * MRF_MAXR];
    const float *V, *w;
    const uint8_t *p, *q;
    float *S, *gunary, *gw;
    double *gV, *gstore;
    float *gstore32;
    int unary_dir, unary_init;
    int *fault;
    int spin_limit;
};

// ---- index replay with the node-to-node chain on a wavefront of its own ----------------------
//
// For launches with few scanlines, where the time of a sweep is the length of a scanline
// times the latency of one node step.  Of the work of a node only this depends on the
// previous node: add what it passed back (carry) to the gradient arriving from elsewhere
// (ext), subtract the label sum at q, scatter through p, scale.  The label sum itself does
// not: the scattered vector of a node sums to zero (the reparametrisation took exactly its
// sum off one entry, back Eq. isgmr-norm), hence so does the carry, and the label sum of
// carry + ext is the label sum of ext up to rounding in the last place of a double.  So the
// correction at q can be applied to ext before the carry is known.
//
// A scanline gets 1 + NI wavefronts.  The helpers take the nodes in turn: they load, form
// ext with the correction at q, and publish it with the scatter targets through a ring in LDS
// (stage "pre"), next to a target vector of the node that they have cleared; the chain wavefront
// touches only LDS: per label one add, the scatter, one read, one multiply, and off the way
// to the next node it leaves g in the place of ext; the same helpers later pick up g and the
// scattered vector and do the rest: grad theta (Alg. 4 line 8), the stored s, the edge-weight
// gradient (Eq. supp-gradient-edge) (stage "post").  A helper runs pre(t) then post(t - NI),
// with a ring of 2 NI slots: every slot is free again exactly when its owner comes round to
// it, so only two kinds of wait exist (chain on pre, post on chain), each on a counter that
// only grows.  The chain reads one node ahead; with NI >= 2 no wait can depend on itself:
// post(t - 2 NI), which precedes pre(t) in its helper, needs the chain to have passed step
// t - 2 NI only.
// What a helper knows of a node when it runs pre stays in its registers until post: p, V's
// entries, grad theta less g.  Loads and stores go through buffer views of the image: a lane's
// offset is its label, the node's is a scalar, and what must not be stored gets the offset
// at which the view ends; so a turn is one straight piece of code.  Label sums are formed by
// the matrix unit (mrf_wave_sum_mat_f64).  A helper's turn and the chain's step of a node are 87 vector instructions at
// 96 labels and three sources (counters), where exec-masked stores, 64-bit addresses and sums by DPP took 169: those bounded launches of two
// and more workgroups per compute unit, the chain's own writes (carry, scattered vector, clearing) the others.  256 x 512, 96 labels, TRWP,
// K = 5: 1.66 -> 1.19 ms (65 us for the 269 MB of a launch of 256 scanlines, 4.1 TB/s, 59 us for 226 MB of one of 512); 256 x 256, 256 labels, TRWP, K = 10 4.51 -> 3.16 ms; 283 x 411, 70
// labels, ISGMR, K = 5 1.52 -> 1.22 ms; 32 x 48, 16 labels, ISGMR, K = 5 65 -> 51 us, where half of a launch was the way to its first loads
// (arguments per direction, no 64-bit products, no division for steps of one, loads in front of the preparation of LDS).
//
// GV without VG (L <= 64, as far as LDS has room): the launch also wants the V gradient; every helper keeps an
// accumulator of its own in LDS, lane lambda owning column lambda; their sum goes to the workgroup's slot at the end.
// GV with VG (33..128 labels): there is no room for the tables; the helpers store the gradient vector g of every node
// in P.gstore (0 where no update is replayed) and leave both pairwise gradients to mrf_bwd_pairwise_*, a streaming
// pass that has all of LDS for V and the table.  What is left for a helper is short enough that four of them keep
// up with the chain, so the layout stays ahead to 1,536 scanlines per launch (it did to 512 while the helpers
// gathered from V).
// EDGE (GV and VG, 33..64 labels and fewer): a problem with per-edge tables: the helpers store g in P.gstore32, if that is
// wanted, for mrf_bwd_edge_tables.
// HOT: truncated models send most labels to one source label, and the chain wavefront's LDS adds would queue at that
// one word (64 lanes of one instruction that meet on a word take 170 clocks more than 64 that do not).  The helpers guess it
// (as in mrf_bwd_sweep) and send its lanes to eight words of their own by lane, which leaves next to no queue (9
// clocks); the chain adds the eight up.
// FAR: images whose entries lie beyond 32-bit offsets from the image's first one (more than 2^30, half of that where node
// gradients are stored): every access makes a view of its node's entries alone, by scalar instructions.  TRWP, backward pass, K = 1, against the
// sweeps with 64-bit addresses: 1024 x 16640, 64 labels, two directions 11.5 / 19.6 ms; 512 x 8400, 256 labels 7.4 / 16.1; 512 x 16800, 128
// labels, four directions 16.0 / 40.2, with grad V 36 / 81.  Six helpers; HOT beyond 128 labels and with stored gradients (64 and 128
// labels without: 12.9 -> 11.5, 18.8 -> 16.0 ms).
// SUMS = false: V-gradient tables, but no edge-weight gradient (a learned table with a scalar weight): no V in LDS, no g V, no sum (backward
// pass, 128 x 256, 48 labels, ISGMR, K = 3 0.335 -> 0.272 ms, 37 x 53, 21 labels, TRWP, K = 5 0.215 -> 0.197).  A variant, because a branch in the
// turn took 0.7 % of a learning step that wants both.
template <int LP, int NS, int D, int NI, bool VG, bool GV, bool HOT, bool EDGE = false, bool FAR = false, bool SUMS = true>
__global__ void __launch_bounds__(64 * (1 + NI)) mrf_bwd_sweep_chain(const MrfChainParams P)
{
    static_assert(D == 1 || D == 2, "sets of registers");
    constexpr int NR = 2 * NI;
    constexpr int LL = 64 * LP;
    constexpr int LH = mrf_bwd_chain_pitch(LP, HOT);              // a target vector and, with HOT, the eight words behind it
    static_assert(NI >= 2 && NI <= MRF_CHAIN_MAX_HELPERS && NI % 2 == 0, "helpers per scanline");
    extern __shared__ __align__(16) unsigned char mrf_bsmem[];
    constexpr bool GVT = GV && !VG;          // V-gradient tables in LDS
    constexpr bool GS = GV && VG;            // node gradients stored for mrf_bwd_pairwise_*
    constexpr bool VROW = !VG && !GV;        // first row of V in LDS
    static_assert(!GVT || LP == 1, "V-gradient tables");
    static_assert(SUMS || GVT, "edge-weight gradient");
    static_assert(!EDGE || (GS && !HOT && !FAR), "per-edge tables");
    const int L = P.L;
    // carved in the order of mrf_bwd_chain_lds_bytes
    double *svr = reinterpret_cast<double *>(mrf_bsmem);         // [NR][LH] scatter targets: cleared by pre, chain -> post
    double *er = svr + NR * LH;                                  // [NR][LL] ext, pre -> chain; then g, chain -> post
    double *vd = er + NR * LL;                                   // [L] first row of V (VROW)
    double *gvacc = vd + (VROW ? L : 0);                     // [NI][L*L] V-gradient accumulators (GVT)
    int *pre_done = reinterpret_cast<int *>(gvacc + (GVT ? NI * L * L : 0));   // [MRF_CHAIN_MAX_HELPERS] per helper: last step published
    int *chain_done = pre_done + MRF_CHAIN_MAX_HELPERS;          // last step the chain finished
    int *a_hot = chain_done + 1;                                 // [NR] pre -> chain: most popular scatter target, or -1
    float *vl = reinterpret_cast<float *>(a_hot + 2 * MRF_CHAIN_MAX_HELPERS);   // [L*L] V (GVT)
    uint16_t *tgr = reinterpret_cast<uint16_t *>(vl + (GVT ? L * L : 0));   // [NR][LL] pre -> chain: LDS address of a label's target, less the slot's offset
    typedef __attribute__((address_space(3))) double *mrf_lds_f64;
    const unsigned sv_base = (unsigned)(uintptr_t)(mrf_lds_f64)svr;                 // (0: nothing lies in front of the dynamic LDS)
    MrfWaitBlock &wait_lds = *reinterpret_cast<MrfWaitBlock *>(
        mrf_bsmem + (((unsigned char *)(tgr + NR * LL) - mrf_bsmem) + 7) / 8 * 8);  // for the waits below (mrf_wait_turn)
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // uniform, and known to be

    const int sl = (int)blockIdx.x;        // one scanline per workgroup
    int ri = 0;
    while (ri + 1 < P.r_count && sl >= P.begin[ri + 1]) ++ri;
    const int dh = P.dh[ri], dw = P.dw[ri];
    int b, y0, x0, len;
    unsigned t;
    mrf_geom_order(P.H, P.W, dh, dw, (unsigned)P.nscan[ri], (unsigned)P.B, (unsigned)(sl - P.begin[ri]), b, t);
    mrf_geom_head(P.H, P.W, dh, dw, t, y0, x0, len);

    // LDS, by all wavefronts together; those of the helpers have their first loads under way
    auto prepare = [&]() {
        if (GVT) {
            for (int e = threadIdx.x; SUMS && e < L * L; e += 64 * (1 + NI)) vl[e] = P.V[e];
            for (int e = threadIdx.x; e < NI * L * L; e += 64 * (1 + NI)) gvacc[e] = 0.0;
        } else if (VROW) {
            for (int e = threadIdx.x; e < L; e += 64 * (1 + NI)) vd[e] = (double)P.V[e];
        }
        if (threadIdx.x < MRF_CHAIN_MAX_HELPERS) pre_done[threadIdx.x] = (int)threadIdx.x - NI;
        if (threadIdx.x == 0) { *chain_done = -1; mrf_wait_init(&wait_lds, P.fault, P.spin_limit); }
        __syncthreads();
    };

    if (wv == 0) {
        // ---- the chain: step tt handles node len-1-tt ---------------------------------------
        // One wait per step: the read of the scattered vector.  What the step needs from the
        // ring is read one step ahead.
        __builtin_amdgcn_s_setprio(3);
        const double cscale = (double)P.carry_scale[ri];
        double carry[LP], ext[LP];
        int tg[LP];
        int hot = -1;
        auto await = [&](int u, int tt) {
            int sn;
            int wait_turns = 0;
            do {
                sn = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(&pre_done[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                if (sn < tt) mrf_wait_turn(&wait_lds, wait_turns);
            } while (sn < tt);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        };
        auto entries = [&](int slot) {
            if (HOT) hot = a_hot[slot];
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                ext[s] = er[slot * LL + lane + 64 * s];
                tg[s] = tgr[slot * LL + lane + 64 * s];
            }
        };
        prepare();
        await(0, 0);
        entries(0);
#pragma unroll
        for (int s = 0; s < LP; ++s) carry[s] = 0.0;
        for (int t0 = 0;; t0 += NR) {
#pragma unroll
            for (int u = 0; u < NR; ++u) {          // (unrolled, so that ring addresses are constants)
                const int tt = t0 + u;
                constexpr int rn = NR;
                const int un = (u + 1) % rn;
                const bool last = tt + 1 >= len;
                // index scatter: s(mu) = sum over lambda with p(lambda) = mu (labels past L
                // carry zeros to entries of their own)
                double g[LP];
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    g[s] = carry[s] + ext[s];
                    __hip_atomic_fetch_add((mrf_lds_f64)((unsigned)tg[s] + (unsigned)(u * LH) * 8u), g[s], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                mrf_wave_lds_fence();
                // In one batch behind the scatter: the counter of the next node's helper, then
                // (the LDS queue keeps this order) that node's ring entries, then the scattered
                // vector.  If the counter turns out not to cover the node, its entries are read
                // again after waiting.
                const int flag = __hip_atomic_load(&pre_done[un % NI], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const int hot_now = hot;
                entries(un);
                double sv[LP], hc[8];
#pragma unroll
                for (int s = 0; s < LP; ++s) sv[s] = svr[u * LH + lane + 64 * s];
                if (HOT) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) hc[j] = svr[u * LH + LL + j];
                }
                __builtin_amdgcn_sched_barrier(0);
                // (behind the reads: nobody waits for these)
#pragma unroll
                for (int s = 0; s < LP; ++s) er[u * LL + lane + 64 * s] = g[s];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                // (written by every lane: the same word, and no exec-mask juggling in the step.  LDS executes a
                // wavefront's operations in order: whoever sees the counter sees what was sent before it)
                if (!HOT) __hip_atomic_store(chain_done, tt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (__builtin_expect(!last && __builtin_amdgcn_readfirstlane(flag) < tt + 1, 0)) {
                    await(un % NI, tt + 1);
                    entries(un);
                    __builtin_amdgcn_s_waitcnt(0xC07F);      // (lgkmcnt(0): the way past this branch is counted as if it had not been taken)
                }
                if (HOT) {
                    const double hsum = ((hc[0] + hc[1]) + (hc[2] + hc[3])) + ((hc[4] + hc[5]) + (hc[6] + hc[7]));
#pragma unroll
                    for (int s = 0; s < LP; ++s) {
                        sv[s] += lane + 64 * s == hot_now ? hsum : 0.0;
                        svr[u * LH + lane + 64 * s] = sv[s];
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __hip_atomic_store(chain_done, tt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
#pragma unroll
                for (int s = 0; s < LP; ++s) carry[s] = cscale * sv[s];
                if (last) return;                   // (uniform)
            }
        }
    }

    // ---- helpers ---------------------------------------------------------------------------
    const int jw = wv - 1, r = P.r_first + ri;
    const bool own_unary = (r == P.unary_dir);
    const bool unary_old = own_unary && !P.unary_init;
    // views of the image (the host has checked that they fit 32-bit offsets, or taken FAR); node n of the scanline lies
    // at hn + n * step
    const unsigned HW = (unsigned)P.H * (unsigned)P.W, HWL = HW * (unsigned)L, endb = HWL * 4u;
    const size_t ibn = (size_t)((unsigned)b * HW), ib = ibn * (unsigned)L;
    const size_t dibn = (size_t)(unsigned)r * (unsigned)P.N + ibn, dib = dibn * (unsigned)L;      // in arrays with an image per direction
    const unsigned hn = (unsigned)y0 * (unsigned)P.W + (unsigned)x0, step = (unsigned)(dh * P.W + dw);
    // a lane's offsets; past every view for labels past L
    const unsigned lane4 = 4u * (unsigned)lane;
    const bool in_last = lane + 64 * (LP - 1) < L;
    const unsigned end4 = in_last ? lane4 + 256u * (LP - 1) : MRF_BUF_NONE, end1 = in_last ? (unsigned)lane + 64u * (LP - 1) : MRF_BUF_NONE;
    auto vo = [&](int s) { return s < LP - 1 ? lane4 + 256u * (unsigned)s : end4; };
    auto vp = [&](int s) { return s < LP - 1 ? (unsigned)lane + 64u * (unsigned)s : end1; };
    mrf_buf bs[NS];
    const float *first[NS];                     // FAR: the image in a source
    const int nsrc = P.n_src[ri], src0 = ri * P.src_pitch;
#pragma unroll
    for (int c = 0; c < NS; ++c) {
        first[c] = P.src[src0 + c] + ib;
        bs[c] = mrf_buffer(first[c], c < nsrc ? endb : 0);      // (a slot that is not in use reads zeros)
    }
    // FAR: the n entries of a node alone, or none of them
    auto only = [&](auto *array, size_t entry, unsigned n, bool any) { return mrf_buffer(array + entry, any ? n * (unsigned)sizeof(*array) : 0u); };
    const mrf_buf bp = mrf_buffer(P.p + dib, HWL), bq = mrf_buffer(P.q + dibn, HW);
    const mrf_buf bgo = mrf_buffer(P.gunary + ib, unary_old ? endb : 0);
    const mrf_buf bw = mrf_buffer(P.w + (P.w_mul ? dibn : 0), P.w_mul ? HW * 4u : 4u);
    auto store_f32 = [](mrf_buf bb, unsigned off, unsigned soff, float x) { __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), bb, off, soff, 0); };

    // own steps: tt = jw + it * NI, it = 0 .. T-1; one more turn for the last post
    const int T = len > jw ? (len - jw + NI - 1) / NI : 0;
    struct In {
        float x[NS][LP], gu[LP], w;
        int p[LP], q;
    };
    In in[D];                                   // a turn's loads are issued D turns before it, as soon as its registers are free
    auto prefetch = [&](In &d, int it) {
        int n = len - 1 - (jw + it * NI);
        n = n > 0 ? n : 0;
        const unsigned node = hn + (unsigned)n * step;
        if constexpr (FAR) {
            const size_t e = (size_t)node * (unsigned)L;
            const mrf_buf vgo = only(P.gunary, ib + e, L, unary_old), vp8 = only(P.p, dib + e, L, true);
#pragma unroll
            for (int c = 0; c < NS; ++c) {
                const mrf_buf v = only(first[c], e, L, c < nsrc);
#pragma unroll
                for (int s = 0; s < LP; ++s) d.x[c][s] = mrf_buf_f32s(v, vo(s), 0);
            }
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                d.gu[s] = mrf_buf_f32s(vgo, vo(s), 0);
                d.p[s] = (int)__builtin_amdgcn_raw_buffer_load_b8(vp8, vp(s), 0, 0);
            }
            d.q = (int)__builtin_amdgcn_raw_buffer_load_b8(only(P.q, dibn + node, 1, true), 0, 0, 0);
            d.w = GVT ? mrf_buf_f32s(only(P.w, P.w_mul ? dibn + node : 0, 1, true), 0, 0) : 0.0f;
            return;
        }
        const unsigned ob = node * (unsigned)L * 4u;
#pragma unroll
        for (int s = 0; s < LP; ++s) {
#pragma unroll
            for (int c = 0; c < NS; ++c) d.x[c][s] = mrf_buf_f32s(bs[c], vo(s), ob);
            d.gu[s] = mrf_buf_f32s(bgo, vo(s), ob);
            d.p[s] = (int)__builtin_amdgcn_raw_buffer_load_b8(bp, vp(s), ob >> 2, 0);
        }
        d.q = (int)__builtin_amdgcn_raw_buffer_load_b8(bq, 0, node, 0);
        d.w = GVT ? mrf_buf_f32s(bw, 0, P.w_mul ? node * 4u : 0u) : 0.0f;
    };
#pragma unroll
    for (int v = 0; v < D; ++v) prefetch(in[v], v);
    prepare();
    double cG[NS], cD[NS];
#pragma unroll
    for (int c = 0; c < NS; ++c) { cG[c] = P.cg[src0 + c]; cD[c] = P.cd[src0 + c]; }
    const mrf_buf bgu = mrf_buffer(P.gunary + ib, own_unary ? endb : 0), bS = mrf_buffer(P.S + dib, endb);
    const mrf_buf bgw = mrf_buffer(P.gw + dibn, P.gw ? HW * 4u : 0);
    const mrf_buf bV = mrf_buffer(P.V, (size_t)L * L * 4);
    const mrf_buf bg = mrf_buffer(EDGE ? (const void *)(P.gstore32 + dib) : (const void *)(P.gstore + ib),
                                  EDGE ? (P.gstore32 ? endb : 0) : (P.gstore ? HWL * 8u : 0));
    // the last node of the scanline has no successor in direction r
    if (jw == 0) {
        const unsigned at = hn + (unsigned)(len - 1) * step, last = FAR ? 0u : at * (unsigned)L * 4u;
        const mrf_buf v = FAR ? only(P.S, dib + (size_t)at * (unsigned)L, L, true) : bS;
#pragma unroll
        for (int s = 0; s < LP; ++s) store_f32(v, vo(s), last, 0.0f);
    }

    // what a turn leaves for the next one, where the same node's post stage is
    struct Kept {
        double th[LP];                          // grad theta less g
        float vv[LP];                           // V(p, lambda) (VG)
        int p[LP];
        float w;
    };
    Kept kept = {};
    double *gvl = gvacc + (GVT ? jw * L * L : 0);
    int chain_seen = -1;
    const bool want_w = SUMS && (P.gw || GVT) && !GS;      // (GVT: the host takes SUMS = false without P.gw)

    auto turn = [&](In &in_, int it, auto parity) {
        constexpr int par = decltype(parity)::value;
        const int tt = jw + it * NI;
        Kept now;
        {
            // ---- pre(tt): everything of node len-1-tt that does not need the carry -------
            // (in the last turn there is no such node: what is published then nobody reads)
            const int slot = jw + par * NI;
            double ev[LP], part = 0.0;
            int pc[LP];
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                double e = cG[0] * (double)in_.x[0][s];
#pragma unroll
                for (int c = 1; c < NS; ++c) e = __builtin_fma(cG[c], (double)in_.x[c][s], e);
                ev[s] = e;
                part += e;
                pc[s] = in_.p[s] < L ? in_.p[s] : L - 1;
            }
            // the commoner of p at the first and at the last label: for a truncated model one
            // of the two is far from the far-field minimiser and points to it
            int hot = -1;
            if (HOT) {
                const int c0 = __builtin_amdgcn_readlane(pc[0], 0), c1 = __builtin_amdgcn_readlane(pc[LP - 1], (L - 1) & 63);
                int n0 = 0, n1 = 0;
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int pm = s < LP - 1 || lane + 64 * s < L ? pc[s] : -1;
                    n0 += __popcll(__builtin_amdgcn_ballot_w64(pm == c0));
                    n1 += __popcll(__builtin_amdgcn_ballot_w64(pm == c1));
                }
                hot = n1 > n0 ? c1 : c0;
                a_hot[slot] = hot;              // (by every lane)
            }
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const int lam = lane + 64 * s;
                now.p[s] = pc[s];
                int target = HOT && pc[s] == hot ? LL + (lane & 7) : pc[s];
                if (s == LP - 1) target = lam < L ? target : lam;      // (labels past L: zeros to entries of their own)
                tgr[slot * LL + lam] = (uint16_t)(sv_base + 8u * (unsigned)target);
                svr[slot * LH + lam] = 0.0;
            }
            if (HOT && lane < 8) svr[slot * LH + LL + lane] = 0.0;
            // back Eq. isgmr-norm, on the part of g that is known here: the entry at q loses
            // the label sum
            const double tot = mrf_wave_sum_mat_f64(part);
            const int qv = in_.q < L ? in_.q : L - 1;
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const double corr = lane + 64 * s == qv ? tot : 0.0;
                er[slot * LL + lane + 64 * s] = ev[s] - corr;
                now.th[s] = 0.0;
                if (own_unary) {
                    asm volatile("");            // (a branch, not a selection)
                    double d = corr + (double)in_.gu[s];
#pragma unroll
                    for (int c = 0; c < NS; ++c) d = __builtin_fma(cD[c], (double)in_.x[c][s], d);
                    now.th[s] = d;
                }
                now.vv[s] = 0.0f;
                // (labels past L read p = 0, so their offset stays MRF_BUF_NONE)
                if (VG && !GS) now.vv[s] = mrf_buf_f32s(bV, vo(s) + 4u * (unsigned)__mul24(pc[s], L), 0);
            }
            now.w = in_.w;
            // (LDS keeps a wavefront's operations in order: the counter lands behind the entries)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __hip_atomic_store(&pre_done[jw], tt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        prefetch(in_, it + D);
        {
            // ---- post(tp): what is left of node len-1-tp once the chain has passed --------
            // (in the first turn there is no such node: nothing is stored)
            const int tp = tt - NI;
            int wait_turns = 0;
            while (chain_seen < tp) {
                chain_seen = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(chain_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                if (chain_seen < tp) mrf_wait_turn(&wait_lds, wait_turns);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            const int slot = jw + (1 - par) * NI;
            const int n = len - 1 - tp;
            const bool node = it > 0, update = node && n > 0;      // node i has a predecessor: its update is replayed
            const unsigned on = hn + (unsigned)(FAR && !node ? 0 : n) * step, oi = on * (unsigned)L * 4u;
            const unsigned oj = oi - step * (unsigned)L * 4u;      // node i - r
            const size_t fi = FAR ? (size_t)on * (unsigned)L : 0, fj = FAR ? (size_t)(update ? on - step : on) * (unsigned)L : 0;
            double g[LP], sv[LP], V[LP];
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const int lam = lane + 64 * s;
                sv[s] = svr[slot * LH + lam];
                g[s] = er[slot * LL + lam];
                V[s] = 0.0;
                if (VROW) {
                    unsigned dist;
                    asm("v_sad_u32 %0, %1, %2, 0" : "=v"(dist) : "v"(kept.p[s]), "v"(lam));
                    if (s == LP - 1) dist = lam < L ? dist : 0;
                    V[s] = vd[dist];
                } else if (GVT) {
                    if (SUMS) V[s] = (double)vl[lam < L ? __mul24(kept.p[s], L) + lam : 0];
                } else if (!GS) {
                    V[s] = (double)kept.vv[s];
                }
                if (s == LP - 1) V[s] = in_last ? V[s] : 0.0;
            }
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                if constexpr (FAR) {
                    store_f32(only(P.S, dib + fj, L, update), vo(s), 0, (float)sv[s]);
                    if constexpr (GS) {
                        typedef unsigned u2 __attribute__((ext_vector_type(2)));
                        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, update ? g[s] : 0.0), only(P.gstore, ib + fi, L, node && P.gstore),
                                                              s < LP - 1 || in_last ? 2u * vo(s) : MRF_BUF_NONE, 0, 0);
                    }
                    store_f32(only(P.gunary, ib + fi, L, node && own_unary), vo(s), 0, (float)(g[s] + kept.th[s]));
                    continue;
                }
                store_f32(bS, vo(s), update ? oj : endb, (float)sv[s]);
                if constexpr (EDGE) {
                    store_f32(bg, vo(s), node ? oi : endb, update ? (float)g[s] : 0.0f);
                } else if constexpr (GS) {
                    typedef unsigned u2 __attribute__((ext_vector_type(2)));
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, update ? g[s] : 0.0), bg, s < LP - 1 || in_last ? 2u * vo(s) : MRF_BUF_NONE,
                                                          node ? 2u * oi : 2u * endb, 0);
                }
                store_f32(bgu, vo(s), node ? oi : endb, (float)(g[s] + kept.th[s]));
            }
            if (want_w) {
                double acc = g[0] * V[0];
#pragma unroll
                for (int s = 1; s < LP; ++s) acc = __builtin_fma(g[s], V[s], acc);
                acc = mrf_wave_sum_mat_f64(acc);
                // one writer per entry and launch: a no-return atomic is a plain accumulate
                if constexpr (FAR) mrf_buf_add_f32(only(P.gw, dibn + on, 1, update), lane == 0 ? 0u : MRF_BUF_NONE, (float)acc);
                else __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32((float)acc, bgw, lane == 0 ? 0u : MRF_BUF_NONE, update ? 4u * on : 4u * HW, 0);
            }
            if (GVT && update && lane < L) {
                double *const e = &gvl[__mul24(kept.p[0], L) + lane];
                *e = __builtin_fma((double)kept.w, g[0], *e);
            }
        }
        kept = now;
    };
    if (T > 0) {
        for (int it = 0;; it += 2) {
            turn(in[0], it, std::integral_constant<int, 0>{});
            if (it >= T) break;                 // (uniform)
            turn(in[D - 1], it + 1, std::integral_constant<int, 1>{});
            if (it + 1 >= T) break;
        }
    }
    if (GVT) {
        // one slot per workgroup: the helpers' tables are summed here, in helper order.  (The chain wavefront
        // has ended or will; a barrier waits for the wavefronts that are left.)
        __syncthreads();
        double *gVs = P.gV + (size_t)blockIdx.x * L * L;
        for (int e = (int)threadIdx.x - 64; e < L * L; e += 64 * NI) {
            double v = gvacc[e];
#pragma unroll
            for (int j = 1; j < NI; ++j) v += gvacc[j * L * L + e];
            mrf_slot_add(&gVs[e], v);
        }
    }
}

// ---- index replay, one label per lane, ceil(L/64) wavefronts per scanline --------------------
//
// Same arithmetic as mrf_bwd_sweep for launches with few scanlines and many labels (a lone
// wavefront with 3-4 labels per lane is bound by instruction issue).  Every wavefront owns 64
// labels: it scatters their g into its own copy of the target vector and publishes their sum;
// after one LDS-only barrier each wavefront adds the copies for its own 64 targets in
// wavefront order (fixed order: reproducible), applies the reparametrisation correction
// (the target p(q) loses the label sum) and carries on.  Copies alternate between two sets so
// that one barrier per node is enough; the edge-weight gradient is assembled one node later.
template <int NS, int D, bool VG>
__global__ void __launch_bounds__(256) mrf_bwd_sweep_split(const MrfBwdParams P)
{
    extern __shared__ __align__(16) unsigned char mrf_bsmem[];
    __shared__ double cp[2][4][256];
    __shared__ double psum[2][4];
    __shared__ double gwp[2][4];
    __shared__ int pqs[2];
    float *vl = reinterpret_cast<float *>(mrf_bsmem);
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // uniform, and known to be
    const int NWV = blockDim.x >> 6;
    const int lam = wv * 64 + lane;
    const bool valid = lam < L;
    const int lc = valid ? lam : 0;
    const long long N = P.g.N;
    double *gVs = P.gV ? P.gV + (size_t)blockIdx.x * L * L : nullptr;
    const int vzero = mrf_opaque_zero();

    if (P.v_mode == 1)
        for (int e = threadIdx.x; e < L * L; e += blockDim.x) vl[e] = P.V[e];
    else if (P.v_mode == 2)
        for (int e = threadIdx.x; e < L; e += blockDim.x) vl[e] = P.V[e];
    if (threadIdx.x < 8) { (&psum[0][0])[threadIdx.x] = 0.0; (&gwp[0][0])[threadIdx.x] = 0.0; }

    for (long long sl = blockIdx.x; sl < P.total_scanlines; sl += gridDim.x) {
        const int ri = mrf_direction_of(P.blk_begin, P.r_count, sl);
        const int r = P.r_first + ri;
        const unsigned local = (unsigned)(sl - P.blk_begin[ri]);
        const unsigned nsc = (unsigned)P.g.nscan[r];
        const int b = (int)(local / nsc);
        const unsigned t = local - (unsigned)b * nsc;
        const int dh = P.g.dh[r], dw = P.g.dw[r];
        int y0, x0, len;
        mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
        const long long head = ((long long)b * P.g.H + y0) * P.g.W + x0;
        const long long nstep = (long long)dh * P.g.W + dw;
        const double cscale = (double)P.carry_scale[r];
        const bool own_unary = (r == P.unary_dir);
        const bool unary_old = own_unary && !P.unary_init;
        const size_t umul = unary_old ? 1 : 0;
        const float *wbase = P.w + (P.w_mul ? (size_t)r * N : 0);
        const uint8_t *pbase = P.p + (size_t)r * N * L;
        const uint8_t *qbase = P.q + (size_t)r * N;

        const float *src[NS];
        double cG[NS], cT[NS];
        const int nsrc = P.n_src[r];
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            const bool live = c < nsrc;
            const bool isgc = (c == nsrc) && P.use_gc;
            src[c] = live ? P.src_base + (size_t)P.src_dir[r][c] * P.src_stride : P.gc;
            cG[c] = live ? (double)P.coefG[r][c] : (isgc ? 1.0 : 0.0);
            cT[c] = live ? (double)P.coefT[r][c] : (isgc ? 1.0 : 0.0);
        }

        __syncthreads();                       // previous scanline completely done with the copies
        for (int e = lane; e < 256; e += 64) { cp[0][wv][e] = 0.0; cp[1][wv][e] = 0.0; }
        int pv_prev = 0;                       // where this lane scattered in the previous step
        if (valid) P.S[((size_t)r * N + head + (long long)(len - 1) * nstep) * L + lam] = 0.0f;

        float cur[D][NS], nxt[D][NS];
        float ucur[D], unxt[D];
        int pcur[D], pnxt[D], qcur[D], qnxt[D];
        float wcur[D], wnxt[D];
        auto prefetch = [&](float (&dst)[NS], float &udst, int &pdst, int &qdst, float &wdst, int tt) {
            int n = len - 1 - tt;
            n = n > 0 ? n : 0;
            const long long i = head + (long long)n * nstep;
#pragma unroll
            for (int c = 0; c < NS; ++c) dst[c] = src[c][(size_t)i * L + lc];
            udst = P.gunary[((size_t)i * L + lc) * umul];
            pdst = pbase[(size_t)i * L + lc];
            qdst = qbase[(size_t)i + vzero];
            wdst = wbase[(size_t)(i * P.w_mul) + vzero];
        };
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(cur[u], ucur[u], pcur[u], qcur[u], wcur[u], u);

        double carry = 0.0;
        int par = 0;
        long long gw_node = -1;     // node whose edge-weight gradient parts sit in gwp[par ^ 1]

        for (int t0 = 0; t0 < len; t0 += D) {
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(nxt[u], unxt[u], pnxt[u], qnxt[u], wnxt[u], t0 + D + u);
#pragma unroll
            for (int u = 0; u < D; ++u) {
                const int tt = t0 + u;
                const bool past = tt >= len;
                const int n = past ? 0 : len - 1 - tt;
                const bool update = !past && n > 0;
                const long long i = head + (long long)n * nstep;
                const long long j = i - nstep;

                double g = carry;
#pragma unroll
                for (int c = 0; c < NS; ++c) g = __builtin_fma(cG[c], (double)cur[u][c], g);
                g = valid ? g : 0.0;
                if (own_unary) {
                    double accT = carry;
#pragma unroll
                    for (int c = 0; c < NS; ++c) accT = __builtin_fma(cT[c], (double)cur[u][c], accT);
                    accT += unary_old ? (double)ucur[u] : 0.0;
                    if (!past && valid) P.gunary[(size_t)i * L + lam] = (float)accT;
                }
                const int pv = pcur[u] < L ? pcur[u] : L - 1;
                int qv = __builtin_amdgcn_readfirstlane(qcur[u]);
                qv = qv < L ? qv : L - 1;

                if (valid) __hip_atomic_fetch_add(&cp[par][wv][pv], g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                const double part = mrf_wave_sum_f64(g);
                if (lane == 0) psum[par][wv] = part;
                if (lam == qv) pqs[par] = pv;
                mrf_block_sync_lds();

                // edge-weight gradient of the previous node: parts in wavefront order
                if (P.gw && wv == 0 && lane == 0 && gw_node >= 0) {
                    const double a = ((gwp[par ^ 1][0] + gwp[par ^ 1][1]) + gwp[par ^ 1][2]) + gwp[par ^ 1][3];
                    __hip_atomic_fetch_add(&P.gw[(size_t)r * N + gw_node], (float)a, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                }
                // back Eq. isgmr-norm: g(q) -= sum_lambda g(lambda); the target p(q) loses the sum
                const double tot = ((psum[par][0] + psum[par][1]) + psum[par][2]) + psum[par][3];
                const int pq = pqs[par];
                double sv = 0.0;
#pragma unroll
                for (int w2 = 0; w2 < 4; ++w2)
                    if (w2 < NWV) sv += cp[par][w2][lam];
                if (lam == pq) sv -= tot;
                const double gn = (lam == qv) ? g - tot : g;
                if (update && valid) P.S[((size_t)r * N + j) * L + lam] = (float)sv;
                carry = cscale * sv;
                // own copy of the other set: its readers are past the barrier, clear what was touched
                cp[par ^ 1][wv][pv_prev] = 0.0;
                pv_prev = pv;

                const double wgt = (double)wcur[u];
                if (P.gw) {
                    double acc = 0.0;
                    if (valid) {
                        float vv;
                        if (VG) {
                            vv = P.V[(size_t)__mul24(pv, L) + lam];
                        } else {
                            const int dist = pv > lam ? pv - lam : lam - pv;
                            vv = vl[P.v_mode == 1 ? __mul24(pv, L) + lam : dist];
                        }
                        acc = gn * (double)vv;
                    }
                    acc = mrf_wave_sum_f64(acc);
                    if (lane == 0) gwp[par][wv] = acc;
                    gw_node = update ? i : -1;
                }
                if (gVs && update && valid)
                    __hip_atomic_fetch_add(&gVs[(size_t)__mul24(pv, L) + lam], wgt * gn, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                par ^= 1;
            }
#pragma unroll
            for (int u = 0; u < D; ++u) {
                qcur[u] = qnxt[u];
                wcur[u] = wnxt[u];
                ucur[u] = unxt[u];
                pcur[u] = pnxt[u];
#pragma unroll
                for (int c = 0; c < NS; ++c) cur[u][c] = nxt[u][c];
            }
        }
        if (P.gw) {
            __syncthreads();
            if (wv == 0 && lane == 0 && gw_node >= 0) {
                const double a = ((gwp[par ^ 1][0] + gwp[par ^ 1][1]) + gwp[par ^ 1][2]) + gwp[par ^ 1][3];
                __hip_atomic_fetch_add(&P.gw[(size_t)r * N + gw_node], (float)a, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// ---- index replay for few labels: several scanlines per wavefront ---------------------------
//
// Counterpart of mrf_fwd_sweep_packed: the wavefront is cut into 64/SEG segments of SEG >= L
// lanes, each replaying its own scanline (any direction, any length).  Label sums are DPP
// row sums (plus one swizzle for 32-lane segments), the scatter vector and the V-gradient
// accumulator are per segment in LDS.
// sum over a segment of 21 lanes (three per wavefront, see mrf_seg21_upper): the upper and the lower
// lanes of every row are summed apart, the previous row's upper sum joins this row's lower sum,
// and the upper lanes fetch the result from the row after theirs; a fixed order
__device__ inline double mrf_segment_sum21_f64(double v, int lane)
{
    const bool up = mrf_seg21_upper(lane);
    double u = up ? v : 0.0, lo = up ? 0.0 : v;
    u += mrf_dpp_f64<0xB1>(u);
    lo += mrf_dpp_f64<0xB1>(lo);
    u += mrf_dpp_f64<0x4E>(u);
    lo += mrf_dpp_f64<0x4E>(lo);
    u += mrf_dpp_f64<0x141>(u);
    lo += mrf_dpp_f64<0x141>(lo);
    u += mrf_dpp_f64<0x140>(u);
    lo += mrf_dpp_f64<0x140>(lo);
    const long long ub = __builtin_bit_cast(long long, u);
    // row_bcast:15 into rows 1..3, zero for row 0
    const int plo = __builtin_amdgcn_update_dpp(0, (int)(ub & 0xffffffffLL), 0x142, 0xE, 0xF, false);
    const int phi = __builtin_amdgcn_update_dpp(0, (int)(ub >> 32), 0x142, 0xE, 0xF, false);
    const double full = lo + __builtin_bit_cast(double, ((long long)phi << 32) | (long long)(unsigned)plo);
    const int from = (up ? ((lane & 48) + 16) & 63 : lane) << 2;
    const long long fb = __builtin_bit_cast(long long, full);
    const int rlo = __builtin_amdgcn_ds_bpermute(from, (int)(fb & 0xffffffffLL));
    const int rhi = __builtin_amdgcn_ds_bpermute(from, (int)(fb >> 32));
    return __builtin_bit_cast(double, ((long long)rhi << 32) | (long long)(unsigned)rlo);
}

template <int SEG>
__device__ inline double mrf_segment_sum_f64(double v)
{
    if (SEG == 21) return mrf_segment_sum21_f64(v, (int)(threadIdx.x & 63));
    v += mrf_dpp_f64<0xB1>(v);
    v += mrf_dpp_f64<0x4E>(v);
    v += mrf_dpp_f64<0x141>(v);
    if (SEG == 8) return v;
    v += mrf_dpp_f64<0x140>(v);
    if (SEG == 32) {
        const long long b = __builtin_bit_cast(long long, v);
        const int lo = __builtin_amdgcn_ds_swizzle((int)(b & 0xffffffffLL), 0x401F);
        const int hi = __builtin_amdgcn_ds_swizzle((int)(b >> 32), 0x401F);
        v += __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
    }
    return v;
}

// the value of the segment's first lane (SEG = 8, 16, 32)
template <int SEG>
__device__ inline int mrf_segment_lane0(int v)
{
    v = __builtin_amdgcn_mov_dpp(v, 0x00, 0xF, 0xF, true);                         // quads: their first lane
    const int h = __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);              // row_half_mirror: the other quad of the eight
    const int lane = (int)(threadIdx.x & 63);
    if (SEG == 8) return (lane & 4) ? h : v;
    v = (lane & 4) ? h : v;
    const int m = __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true);              // row_mirror: the other eight of the row
    v = (lane & 8) ? m : v;
    if (SEG == 16) return v;
    const auto x = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    return (int)x[0];                                                              // (rows 0, 2 of v in rows 0 and 1, 2 and 3)
}

// UNARY = false: no direction of the launch forms grad theta_i (ISGMR with its combine passes)
template <int SEG, int NS, int D, bool UNARY = true>
__global__ void __launch_bounds__(64) mrf_bwd_sweep_packed(const MrfBwdParams P)
{
    constexpr int NSEG = 64 / SEG;
    extern __shared__ __align__(16) unsigned char mrf_bsmem[];
    const int L = P.g.L;
    const int lane = threadIdx.x;
    // (three segments of 21 lanes leave lane 63 over: it shadows the last segment and stores nothing)
    const bool lane_on = lane / SEG < NSEG;
    const int seg = lane_on ? lane / SEG : NSEG - 1, lam = lane % SEG;
    const bool valid = lane_on && lam < L;
    const int lc = valid ? lam : 0;
    const long long N = P.g.N;
    double *sbuf = reinterpret_cast<double *>(mrf_bsmem) + seg * SEG;                       // [NSEG][SEG]
    double *gvl = reinterpret_cast<double *>(mrf_bsmem) + NSEG * SEG + (P.gV ? seg * L * L : 0);  // [NSEG][L*L]
    float *vl = reinterpret_cast<float *>(reinterpret_cast<double *>(mrf_bsmem) + NSEG * SEG + (P.gV ? NSEG * L * L : 0));
    double *gVs = P.gV ? P.gV + (size_t)blockIdx.x * L * L : nullptr;      // one slot per workgroup

    for (int e = lane; e < L * L; e += 64) vl[e] = P.V[e];
    if (gVs && lane_on)
        for (int e = lam; e < L * L; e += SEG) gvl[e] = 0.0;
    sbuf[lam] = 0.0;
    __syncthreads();

    const bool any_unary = UNARY && P.unary_dir >= P.r_first && P.unary_dir < P.r_first + P.r_count;
    const long long npacks = (P.total_scanlines + NSEG - 1) / NSEG;
    for (long long pk = blockIdx.x; pk < npacks; pk += gridDim.x) {
        const long long sl = pk * NSEG + seg;
        const bool act_seg = lane_on && sl < P.total_scanlines;

        int r = P.r_first, dh = 0, dw = 1, nsrc = 0;
        unsigned nsc = 1, local = 0;
        float cscale_f = 1.0f;
        int sdir[NS];
        float cGf[NS], cTf[NS];
#pragma unroll
        for (int c = 0; c < NS; ++c) { sdir[c] = 0; cGf[c] = 0.0f; cTf[c] = 0.0f; }
        for (int ri = 0; ri < P.r_count; ++ri) {
            const int rr = P.r_first + ri;
            const bool mine = act_seg && sl >= P.blk_begin[ri] && sl < P.blk_begin[ri + 1];
            if (mine) {
                r = rr; local = (unsigned)(sl - P.blk_begin[ri]); nsc = (unsigned)P.g.nscan[rr]; dh = P.g.dh[rr]; dw = P.g.dw[rr];
                cscale_f = P.carry_scale[rr]; nsrc = P.n_src[rr];
#pragma unroll
                for (int c = 0; c < NS; ++c) { sdir[c] = P.src_dir[rr][c]; cGf[c] = P.coefG[rr][c]; cTf[c] = P.coefT[rr][c]; }
            }
        }
        int y0 = 0, x0 = 0, len = 1;
        long long head = 0;
        if (act_seg) {
            const int b = (int)(local / nsc);
            const unsigned t = local - (unsigned)b * nsc;
            mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
            head = ((long long)b * P.g.H + y0) * P.g.W + x0;
        }
        const long long nstep = (long long)dh * P.g.W + dw;
        const double cscale = (double)cscale_f;
        const bool own_unary = UNARY && act_seg && (r == P.unary_dir);
        const bool unary_old = own_unary && !P.unary_init;
        const size_t umul = unary_old ? 1 : 0;
        const float *wbase = P.w + (P.w_mul ? (size_t)r * N : 0);
        const uint8_t *pbase = P.p + (size_t)r * N * L;
        const uint8_t *qbase = P.q + (size_t)r * N;

        const float *src[NS];
        double cG[NS], cT[NS];
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            const bool live = c < nsrc;
            const bool isgc = (c == nsrc) && P.use_gc;
            src[c] = live ? P.src_base + (size_t)sdir[c] * P.src_stride : P.gc;
            cG[c] = live ? (double)cGf[c] : (isgc ? 1.0 : 0.0);
            cT[c] = live ? (double)cTf[c] : (isgc ? 1.0 : 0.0);
        }
        if (act_seg && valid) P.S[((size_t)r * N + head + (long long)(len - 1) * nstep) * L + lam] = 0.0f;

        int maxlen = 1;
#pragma unroll
        for (int sg = 0; sg < NSEG; ++sg) {
            const int l2 = __builtin_amdgcn_readlane(len, sg * SEG);
            maxlen = l2 > maxlen ? l2 : maxlen;
        }

        float cur[D][NS], nxt[D][NS];
        float ucur[D], unxt[D];
        int pcur[D], pnxt[D], qcur[D], qnxt[D];
        float wcur[D], wnxt[D];
        auto prefetch = [&](float (&dst)[NS], float &udst, int &pdst, int &qdst, float &wdst, int tt) {
            int n = len - 1 - tt;
            n = n > 0 ? n : 0;
            const long long i = head + (long long)n * nstep;
#pragma unroll
            for (int c = 0; c < NS; ++c) dst[c] = src[c][(size_t)i * L + lc];
            if constexpr (UNARY) udst = P.gunary[((size_t)i * L + lc) * umul]; else udst = 0.0f;
            pdst = pbase[(size_t)i * L + lc];
            qdst = qbase[(size_t)i];
            wdst = wbase[(size_t)(i * P.w_mul)];
        };
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(cur[u], ucur[u], pcur[u], qcur[u], wcur[u], u);

        double carry = 0.0;
        for (int t0 = 0; t0 < maxlen; t0 += D) {
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(nxt[u], unxt[u], pnxt[u], qnxt[u], wnxt[u], t0 + D + u);
            // What arrives from elsewhere, and its label sums, for the D nodes of the group at once
            // (independent reductions overlap).  The label sum of g = carry + ext is the label sum
            // of ext: the scattered vector of a node sums to zero, because the reparametrisation took
            // exactly its sum off one entry, hence so does the carry (up to double rounding).
            double ext[D], tot[D];
#pragma unroll
            for (int u = 0; u < D; ++u) {
                double e = 0.0;
#pragma unroll
                for (int c = 0; c < NS; ++c) e = __builtin_fma(cG[c], (double)cur[u][c], e);
                ext[u] = valid ? e : 0.0;
            }
#pragma unroll
            for (int u = 0; u < D; ++u) tot[u] = mrf_segment_sum_f64<SEG>(ext[u]);
#pragma unroll
            for (int u = 0; u < D; ++u) {
                const int tt = t0 + u;
                const bool past = !act_seg || tt >= len;
                const int n = past ? 0 : len - 1 - tt;
                const bool update = !past && n > 0;
                const long long i = head + (long long)n * nstep;
                const long long j = i - nstep;

                double g = valid ? carry + ext[u] : 0.0;
                if constexpr (UNARY) if (any_unary) {        // (uniform) some scanline of this launch forms grad theta
                    double accT = carry;
#pragma unroll
                    for (int c = 0; c < NS; ++c) accT = __builtin_fma(cT[c], (double)cur[u][c], accT);
                    accT += unary_old ? (double)ucur[u] : 0.0;
                    if (own_unary && !past && valid) P.gunary[(size_t)i * L + lam] = (float)accT;
                }
                const int pv = pcur[u] < L ? pcur[u] : L - 1;
                const int qv = qcur[u] < L ? qcur[u] : L - 1;
                // back Eq. isgmr-norm: g(q) -= sum_lambda g(lambda)
                if (lam == qv) g = g - tot[u];

                if (valid) __hip_atomic_fetch_add(&sbuf[pv], g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                mrf_wave_lds_fence();
                const double sv = sbuf[lam];
                mrf_wave_lds_fence();
                sbuf[lam] = 0.0;
                if (update && valid) P.S[((size_t)r * N + j) * L + lam] = (float)sv;
                carry = cscale * sv;

                const double wgt = (double)wcur[u];
                if (P.gw) {
                    double acc = valid ? g * (double)vl[__mul24(pv, L) + lc] : 0.0;
                    acc = mrf_segment_sum_f64<SEG>(acc);
                    if (update && lam == 0)
                        __hip_atomic_fetch_add(&P.gw[(size_t)r * N + i], (float)acc, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                }
                if (gVs && update && valid) gvl[__mul24(pv, L) + lam] = __builtin_fma(wgt, g, gvl[__mul24(pv, L) + lam]);
            }
#pragma unroll
            for (int u = 0; u < D; ++u) {
                qcur[u] = qnxt[u];
                wcur[u] = wnxt[u];
                ucur[u] = unxt[u];
                pcur[u] = pnxt[u];
#pragma unroll
                for (int c = 0; c < NS; ++c) cur[u][c] = nxt[u][c];
            }
        }
    }
    if (gVs) {
        // the segments' tables are summed in segment order
        mrf_wave_lds_fence();
        const double *t0 = reinterpret_cast<double *>(mrf_bsmem) + NSEG * SEG;
        for (int e = lane; e < L * L; e += 64) {
            double v = t0[e];
#pragma unroll
            for (int sg = 1; sg < NSEG; ++sg) v += t0[sg * L * L + e];
            mrf_slot_add(&gVs[e], v);
        }
    }
}

// ---- index replay for few labels: several labels per lane, narrow segments -----------------------
//
// The same replay for launches of up to 32 labels that have scanlines to spare.  A segment of SEG = 8, 16 or
// 32 lanes walks a scanline, a lane owns NL neighbouring labels (NL li, NL li + 1, ...), so a wavefront of 64 / SEG
// scanlines spends its addresses, its reductions over labels (three DPP levels for 8 lanes) and its bookkeeping on
// eight nodes at a time instead of two, and hardly any lane is idle (21 labels: 21 of 24 entries).  Scanlines of one
// wavefront belong to one direction (the host pads every direction to whole wavefronts), so directions, coefficients
// and base addresses are scalars, and an entry is a 32-bit offset into a buffer view (the host checks that N L fits);
// a lane past its scanline's end or without a label has an offset past the view's.
// Per node: everything from memory is prefetched D nodes ahead into one of two register sets that take turns;
// the label sums of D nodes are formed at once (they do not depend on the carry, as in mrf_bwd_sweep_packed); the
// chain is one add per label, the scatter into the segment's row in LDS and its read; the pairwise gradients of
// a node are formed behind the scatter of the next one, while that is under way.
// FULL: L is a multiple of NL, so that a lane's labels are one access of NL floats.
// GV: every wavefront has V-gradient tables of its own in LDS, summed in a fixed order at the end: the order of all
// additions, and with it every bit of the result, is the same in every run.
// GS: a problem with per-edge tables: no V and no edge-weight gradient; the gradient vector g of every node goes to
// P.gstore32 (0 where no update is replayed), if that is wanted, for mrf_bwd_edge_tables.
template <int SEG, int NL>
__host__ __device__ constexpr int mrf_bwd_narrow_row()
{
    // doubles per row of the scatter target: lanes are NL doubles apart, and the rows of a wavefront start on banks
    // that those lanes leave free (24 doubles for three labels per lane, else an odd number for several)
    return (NL == 1 || NL == 3) ? SEG * NL : SEG * NL + 1;
}

// rows of V and of the V-gradient tables have an odd length in LDS (an even one puts a label on the same bank in
// every row); tables start on different banks as the rows above do
__host__ __device__ inline int mrf_bwd_narrow_pitch(int L) { return L | 1; }
template <int SEG, int NL>
__host__ __device__ inline int mrf_bwd_narrow_table(int L)
{
    const int n = L * mrf_bwd_narrow_pitch(L), want = mrf_bwd_narrow_row<SEG, NL>() % 32;
    return n + (want - n % 32 + 32) % 32;
}

// V-gradient tables of one wavefront: one for each of its segments where a workgroup has one wavefront and room (half
// as many from 23 labels on), else as many as leave the workgroup's LDS what it is with one wavefront, at least one.
// Segments that share a table add to it by the lanes of one instruction.  (Backward pass, ISGMR, four wavefronts sharing
// the tables / with tables of their own: 4 x 512 x 512, 21 labels, 4 directions 1.10 / 1.09 ms; 256 x 512, 32 labels, 16
// directions 1.06 / 1.05; TRWP 4 x 512 x 512, 32 labels 1.78 / 1.81)
__host__ __device__ inline int mrf_bwd_narrow_tables(int nseg, int L, int waves)
{
    const int n = (L <= 22 || nseg < 4 ? nseg : nseg / 2) / waves;
    return n > 0 ? n : 1;
}

template <int SEG, int NL, int NS, int D, bool UNARY, bool GV, bool FULL, bool GS = false>
__global__ void __launch_bounds__(256) mrf_bwd_sweep_narrow(const MrfBwdParams P)
{
    constexpr int NSEG = 64 / SEG;
    constexpr int RS = mrf_bwd_narrow_row<SEG, NL>();
    constexpr bool UNIT = NS == 1 && !UNARY;       // ISGMR between its combine passes: one source, coefficients 1
    extern __shared__ __align__(16) unsigned char mrf_bsmem[];
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int waves = (int)(blockDim.x >> 6);
    const int seg = lane / SEG, li = lane % SEG;
    const int lam0 = li * NL;                                 // the lane's first label
    const int ntab = GV ? mrf_bwd_narrow_tables(NSEG, L, waves) : 0, tsize = mrf_bwd_narrow_table<SEG, NL>(L), pitch = mrf_bwd_narrow_pitch(L);
    double *rows = reinterpret_cast<double *>(mrf_bsmem) + wv * (NSEG * RS + 64);            // [waves]{[NSEG][RS], 64 spare}
    double *tabs = reinterpret_cast<double *>(mrf_bsmem) + waves * (NSEG * RS + 64);         // [waves][ntab][tsize]
    float *vl = reinterpret_cast<float *>(tabs + waves * ntab * tsize);                      // [L][pitch] V, then a 0
    double *sb = rows + seg * RS;
    double *spare = rows + NSEG * RS + lane;                  // where a lane with nothing to add adds

    if constexpr (!GS) {
        for (int e = threadIdx.x; e < L * pitch; e += blockDim.x) {
            const int mu = e / pitch, lam = e - mu * pitch;
            vl[e] = lam < L ? P.V[mu * L + lam] : 0.0f;
        }
        if (threadIdx.x == 0) vl[L * pitch] = 0.0f;
    }
    for (int e = threadIdx.x; e < waves * (NSEG * RS + 64 + ntab * tsize); e += blockDim.x) reinterpret_cast<double *>(mrf_bsmem)[e] = 0.0;
    __syncthreads();

    // this wavefront's scanlines: NSEG consecutive ones of direction r
    const int pk = P.pack_first + (int)blockIdx.x * waves + wv;
    int ri = 0;
    while (ri + 1 < P.r_count && pk >= P.pack_begin[ri + 1]) ++ri;
    const int r = P.r_first + ri;
    const unsigned nsc = (unsigned)P.g.nscan[r];
    const unsigned sl = (unsigned)(pk - P.pack_begin[ri]) * NSEG + seg;
    const bool act = pk < P.pack_begin[P.r_count] && sl < (unsigned)P.g.B * nsc;
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0 = 0, x0 = 0, len = 0;
    int last = 0;                                             // the scanline's last node, where the replay starts
    const int nstep = dh * P.g.W + dw;
    if (act) {
        const int b = (int)(sl / nsc);
        mrf_geom_head(P.g.H, P.g.W, dh, dw, sl - (unsigned)b * nsc, y0, x0, len);
        last = (b * P.g.H + y0) * P.g.W + x0 + (len - 1) * nstep;
    }
    int maxlen = 0;
#pragma unroll
    for (int sg = 0; sg < NSEG; ++sg) {
        const int l2 = __builtin_amdgcn_readlane(len, sg * SEG);
        maxlen = l2 > maxlen ? l2 : maxlen;
    }

    const size_t N = (size_t)P.g.N, NL4 = N * L * 4;
    const double cscale = (double)P.carry_scale[r];
    const bool own_unary = UNARY && r == P.unary_dir;
    const unsigned no_store = own_unary ? 0u : MRF_BUF_NONE, no_old = own_unary && !P.unary_init ? 0u : MRF_BUF_NONE;
    const mrf_buf bp = mrf_buffer(P.p + (size_t)r * N * L, N * L), bq = mrf_buffer(P.q + (size_t)r * N, N);
    const mrf_buf bw = mrf_buffer(P.w + (P.w_mul ? (size_t)r * N : 0), P.w_mul ? N * 4 : 4);
    const mrf_buf bs = mrf_buffer(P.S + (size_t)r * N * L, NL4), bu = mrf_buffer(P.gunary, NL4);
    const mrf_buf bgw = mrf_buffer(P.gw ? P.gw + (size_t)r * N : nullptr, P.gw ? N * 4 : 0);
    const mrf_buf bgs = mrf_buffer(GS && P.gstore32 ? P.gstore32 + (size_t)r * N * L : nullptr, GS && P.gstore32 ? NL4 : 0);
    mrf_buf src[NS];
    double cG[NS], cT[NS];
    const int nsrc = P.n_src[r];
#pragma unroll
    for (int c = 0; c < NS; ++c) {
        const bool live = c < nsrc;
        const bool isgc = (c == nsrc) && P.use_gc;
        src[c] = mrf_buffer(live ? P.src_base + (size_t)P.src_dir[r][c] * P.src_stride : P.gc, NL4);
        cG[c] = live ? (double)P.coefG[r][c] : (isgc ? 1.0 : 0.0);
        cT[c] = live ? (double)P.coefT[r][c] : (isgc ? 1.0 : 0.0);
    }

    // accesses of the lane's labels at byte offset `at` of its first one (MRF_BUF_NONE: none of them)
    const bool any = lam0 < L;
    auto load = [&](mrf_buf b, unsigned at, float (&v)[NL]) {
        if constexpr (FULL) {
            mrf_buf_f32xn<NL>(b, at, v);
        } else {
#pragma unroll
            for (int s = 0; s < NL; ++s) v[s] = mrf_buf_f32(b, lam0 + s < L ? at + 4u * s : MRF_BUF_NONE);
        }
    };
    auto store = [&](mrf_buf b, unsigned at, const float (&v)[NL]) {
        if constexpr (FULL) {
            mrf_buf_store_f32xn<NL>(b, at, v);
        } else {
#pragma unroll
            for (int s = 0; s < NL; ++s) mrf_buf_store_f32(b, lam0 + s < L ? at + 4u * s : MRF_BUF_NONE, v[s]);
        }
    };
    // p of the lane's labels: one access of 1, 2 or 4 bytes that stays inside the node's L bytes, and a shift
    constexpr int PB = NL == 1 ? 1 : (NL == 2 ? 2 : 4);
    const int p_at = any ? (lam0 < L - PB ? lam0 : L - PB) : 0, p_shift = any ? 8 * (lam0 - p_at) : 0;
    auto load_p = [&](unsigned at) {
        if constexpr (PB == 1) return (unsigned)mrf_buf_u8(bp, at);
        else if constexpr (PB == 2) return (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(bp, at, 0, 0);
        else return (unsigned)__builtin_amdgcn_raw_buffer_load_b32(bp, at, 0, 0);
    };

    struct In {
        float v[NS][NL];
        float u[UNARY ? NL : 1];         // old grad theta_i (0 unless accumulating)
        unsigned p;
        int q;
        float w;
    };
    In A[D], B[D];
    // The prefetch walks from the last node towards the first and on: what it then loads is another node or nothing,
    // and never used.  Slots without a label load 0.
    unsigned pi = (unsigned)last, pe = (unsigned)last * (unsigned)L;
    const unsigned estep = (unsigned)(nstep * L);
    auto prefetch = [&](In &in) {
        const unsigned at = any ? (pe + (unsigned)lam0) << 2 : MRF_BUF_NONE;
#pragma unroll
        for (int c = 0; c < NS; ++c) load(src[c], at, in.v[c]);
        if constexpr (UNARY) load(bu, no_old ? MRF_BUF_NONE : at, in.u);
        in.p = load_p(any ? pe + (unsigned)p_at : MRF_BUF_NONE);
        in.q = mrf_buf_u8(bq, pi);
        in.w = GV ? mrf_buf_f32(bw, P.w_mul ? pi * 4u : 0u) : 0.0f;
        pe -= estep;
        pi -= (unsigned)nstep;
    };

    // the last node of a scanline has no successor in direction r
    {
        float zero[NL];
#pragma unroll
        for (int s = 0; s < NL; ++s) zero[s] = 0.0f;
        store(bs, act && any ? ((unsigned)last * (unsigned)L + (unsigned)lam0) << 2 : MRF_BUF_NONE, zero);
    }

    // the node whose pairwise gradients are still to be formed
    double gP[NL];
    int pP[NL];
    double wP = 0.0;
    bool updP = false;
#pragma unroll
    for (int s = 0; s < NL; ++s) { gP[s] = 0.0; pP[s] = 0; }
    // edge-weight gradients of a group of D nodes: lane li keeps that of the group's node li, one access adds them all
    static_assert(D <= SEG, "lanes that keep edge-weight gradients");
    float gwkeep = 0.0f;
    int gwleft = 0;                                           // lane's node of the group counts if positive
    unsigned gwat = 0;
    double *tab = tabs + (GV ? (wv * ntab + seg % ntab) * tsize : 0);
    auto pairwise = [&](int slot) {
        int at[NL];
#pragma unroll
        // (where there is no label p is 0, and the 0 behind V is met there: an infinite V[0][0] must not be)
        for (int s = 0; s < NL; ++s) at[s] = __mul24(pP[s], pitch) + ((FULL ? any : lam0 + s < L) ? lam0 + s : L * pitch);
        // (formed whether it is wanted or not: the view of an array that is not there holds nothing)
        double acc = gP[0] * (double)vl[at[0]];
#pragma unroll
        for (int s = 1; s < NL; ++s) acc = __builtin_fma(gP[s], (double)vl[at[s]], acc);     // (g is 0 where there is no label)
        acc = mrf_segment_sum_f64<SEG>(acc);
        gwkeep = li == slot ? (float)acc : gwkeep;
        // one writer per entry and launch: a no-return atomic is a plain accumulate
        if (slot == D - 1) mrf_buf_add_f32(bgw, gwleft > 0 ? gwat : MRF_BUF_NONE, gwkeep);
        if (GV) {
            // (no short-circuit in the conditions: it would become a branch)
#pragma unroll
            for (int s = 0; s < NL; ++s)
                __hip_atomic_fetch_add((int)updP & (int)(FULL ? any : lam0 + s < L) ? &tab[at[s]] : spare, wP * gP[s], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };

    double carry[NL];
#pragma unroll
    for (int s = 0; s < NL; ++s) carry[s] = 0.0;
    unsigned ci = (unsigned)last, ce = (unsigned)last * (unsigned)L + (unsigned)lam0;
    auto group = [&](const In (&in)[D], int t0) {
        double ext[D][NL];
#pragma unroll
        for (int u = 0; u < D; ++u) {
            double part = 0.0;
#pragma unroll
            for (int s = 0; s < NL; ++s) {
                double e = UNIT ? (double)in[u].v[0][s] : cG[0] * (double)in[u].v[0][s];
#pragma unroll
                for (int c = 1; c < NS; ++c) e = __builtin_fma(cG[c], (double)in[u].v[c][s], e);
                ext[u][s] = e;
                part = s == 0 ? e : part + e;
            }
            // back Eq. isgmr-norm: the entry at q loses the label sum
            const double tot = mrf_segment_sum_f64<SEG>(part);
            const int qv = in[u].q < L ? in[u].q : L - 1;
#pragma unroll
            for (int s = 0; s < NL; ++s)
                if (lam0 + s == qv) ext[u][s] -= tot;
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int tt = t0 + u;
            double g[NL];
            int pv[NL];
            if constexpr (UNARY) {
                // grad theta_i: everything every direction passed back to node i
                float out[NL];
#pragma unroll
                for (int s = 0; s < NL; ++s) {
                    double accT = carry[s];
#pragma unroll
                    for (int c = 0; c < NS; ++c) accT = __builtin_fma(cT[c], (double)in[u].v[c][s], accT);
                    out[s] = (float)(accT + (double)in[u].u[s]);
                }
                store(bu, (int)(tt < len) & (int)(any && !no_store) ? ce << 2 : MRF_BUF_NONE, out);
            }
            // Where one label beats all others every lane scatters to it, and LDS would add them one by one (8 lanes
            // on one word take 92 clocks, on words of their own 8): a lane merges its labels that go where its
            // first one goes, and lanes whose first label goes where lane 0's does are summed by DPP for lane 0.
            const unsigned pw = in[u].p >> p_shift;
#pragma unroll
            for (int s = 0; s < NL; ++s) {
                g[s] = carry[s] + ext[u][s];
                const int pr = (int)((pw >> (8 * s)) & 255u);
                pv[s] = pr < L ? pr : L - 1;
            }
            double g0 = g[0];
#pragma unroll
            for (int s = 1; s < NL; ++s) g0 += pv[s] == pv[0] ? g[s] : 0.0;
            const bool common = pv[0] == mrf_segment_lane0<SEG>(pv[0]);
            const double gc0 = mrf_segment_sum_f64<SEG>(common ? g0 : 0.0);
            __hip_atomic_fetch_add((int)!common | (int)(li == 0) ? &sb[pv[0]] : spare, common ? gc0 : g0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
            for (int s = 1; s < NL; ++s)
                __hip_atomic_fetch_add(pv[s] != pv[0] ? &sb[pv[s]] : spare, g[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            mrf_wave_lds_fence();
            double sv[NL];
#pragma unroll
            for (int s = 0; s < NL; ++s) sv[s] = sb[lam0 + s];
            mrf_wave_lds_fence();
#pragma unroll
            for (int s = 0; s < NL; ++s) sb[lam0 + s] = 0.0;
            if constexpr (!GS) pairwise(u == 0 ? D - 1 : u - 1);
            if (u == 0) {
                gwleft = li < D ? len - 1 - t0 - li : 0;
                gwat = (ci - (unsigned)(li * nstep)) << 2;
            }
            const bool update = tt < len - 1;            // node i has a predecessor: replay its update
            if constexpr (GS) {
                float out[NL];
#pragma unroll
                for (int s = 0; s < NL; ++s) out[s] = update ? (float)g[s] : 0.0f;
                store(bgs, (int)(tt < len) & (int)any ? ce << 2 : MRF_BUF_NONE, out);
            }
            ce -= estep;
            {
                float out[NL];
#pragma unroll
                for (int s = 0; s < NL; ++s) out[s] = (float)sv[s];
                store(bs, (int)update & (int)any ? ce << 2 : MRF_BUF_NONE, out);
            }
#pragma unroll
            for (int s = 0; s < NL; ++s) { carry[s] = UNIT ? sv[s] : cscale * sv[s]; gP[s] = g[s]; pP[s] = pv[s]; }
            wP = (double)in[u].w;
            updP = update;
            ci -= (unsigned)nstep;
        }
    };
    if (maxlen > 0) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(A[u]);
        // (as many dropped stores as a group makes: what is in flight when the loop is entered then looks to the
        // compiler like what is in flight when it comes round, else it waits for the newest stores each time)
#pragma unroll
        for (int u = 0; u < D * ((UNARY ? 2 : 1) + (GS ? 1 : 0)) * (FULL ? 1 : NL) + (GS ? 0 : 1); ++u) mrf_buf_store_f32(bs, MRF_BUF_NONE, 0.0f);
        for (int t0 = 0; t0 < maxlen; t0 += 2 * D) {
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(B[u]);
            __builtin_amdgcn_sched_barrier(0);           // (the loads stay in front)
            group(A, t0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(A[u]);
            __builtin_amdgcn_sched_barrier(0);
            group(B, t0 + D);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (!GS) pairwise(D - 1);
    }
    if (GV) {
        __syncthreads();
        double *slot = P.gV + (size_t)blockIdx.x * L * L;
        for (int e = threadIdx.x; e < L * L; e += blockDim.x) {
            const int mu = e / L, at = mu * pitch + (e - mu * L);
            double v = tabs[at];
            for (int k = 1; k < waves * ntab; ++k) v += tabs[k * tsize + at];
            mrf_slot_add(&slot[e], v);
        }
    }
}

// ---- the narrow replay with its work divided among four wavefronts ---------------------------------------
//
// One direction per launch (TRWP) leaves the wavefronts above, eight scanlines each, alone on a quarter of the SIMDs: 4 x 512 x
// 512 is 256 of them, and a node step of theirs is 1,100 clocks.  Here a workgroup of four wavefronts, one per SIMD, walks the
// same scanlines: two take the nodes in turn and do what does not wait for the chain (loads, the gradient arriving from
// elsewhere with the correction at q), one does the chain (add, scatter through LDS, read, the stored s), one what is left (grad
// theta, both pairwise gradients).  Rings in LDS as in mrf_bwd_sweep_chain: ext and p from the first two, the carry that entered a
// node from the chain.  Same operations on the same values in the same order as mrf_bwd_sweep_narrow, but for grad theta: what
// arrives from elsewhere is summed in front of the chain, from the old value on, and the carry is added last (there: the carry first,
// the old value last; both in double, rounded once).
// Every wait is on a counter that only grows: chain on pre, post on chain, pre on post NR steps back.
// Several source arrays; label counts that the lanes' labels divide (the launches that the rule of narrow_lanes gives them).
// Backward pass, 4 x 512 x 512, TRWP, 4 directions, K = 2: 21 labels 1.86 -> 1.42 ms, 16 labels 1.37 -> 1.07, 32 labels 1.82 -> 1.50.  What sets the
// pace now is the chain's 80 instructions and two trips through LDS per node.
template <int SEG, int NL, bool UNARY, bool GV>
__host__ __device__ inline size_t mrf_bwd_narrow_divided_lds(int L)
{
    constexpr int NSEG = 64 / SEG, NR = 8;
    return sizeof(double) * (NSEG * mrf_bwd_narrow_row<SEG, NL>() + 128 + (size_t)(UNARY ? 3 : 2) * NR * NL * 64 +
                             (GV ? (size_t)mrf_bwd_narrow_tables(NSEG, L, 1) * mrf_bwd_narrow_table<SEG, NL>(L) : 0)) +
           sizeof(float) * ((size_t)L * mrf_bwd_narrow_pitch(L) + 1 + 2 * NR * 64 + 8) + sizeof(MrfWaitBlock) + 8;
}

template <int SEG, int NL, int NS, bool UNARY, bool GV>
__global__ void __launch_bounds__(256) mrf_bwd_sweep_narrow(const MrfBwdParams P)
{
    constexpr int NSEG = 64 / SEG, NR = 8, D = NS <= 4 ? 2 : 1;
    constexpr int RS = mrf_bwd_narrow_row<SEG, NL>();
    extern __shared__ __align__(16) unsigned char mrf_bsmem[];
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int seg = lane / SEG, li = lane % SEG;
    const int lam0 = li * NL;                                 // the lane's first label
    const int ntab = GV ? mrf_bwd_narrow_tables(NSEG, L, 1) : 0, tsize = mrf_bwd_narrow_table<SEG, NL>(L), pitch = mrf_bwd_narrow_pitch(L);
    // carved in the order of mrf_bwd_narrow_divided_lds
    double *rows = reinterpret_cast<double *>(mrf_bsmem);     // [NSEG][RS] scatter target, 64 spare, 64 spare of the tables
    double *r_ext = rows + NSEG * RS + 128;                   // [NR][NL][64] pre -> chain, post
    double *r_cin = r_ext + NR * NL * 64;                     // [NR][NL][64] chain -> post
    double *r_all = r_cin + NR * NL * 64;                     // [NR][NL][64] pre -> post: grad theta's part (UNARY)
    double *tabs = r_all + (UNARY ? NR * NL * 64 : 0);        // [ntab][tsize]
    unsigned *r_p = reinterpret_cast<unsigned *>(tabs + ntab * tsize);        // [NR][64]
    float *r_w = reinterpret_cast<float *>(r_p + NR * 64);    // [NR][64]
    int *counters = reinterpret_cast<int *>(r_w + NR * 64);   // pre (two), chain, post: last step done
    float *vl = reinterpret_cast<float *>(counters + 8);      // [L][pitch] V, then a 0
    MrfWaitBlock &wait_lds = *reinterpret_cast<MrfWaitBlock *>(mrf_bsmem + (reinterpret_cast<unsigned char *>(vl + L * pitch + 1) - mrf_bsmem + 7) / 8 * 8);

    for (int e = threadIdx.x; e < L * pitch; e += 256) {
        const int mu = e / pitch, lam = e - mu * pitch;
        vl[e] = lam < L ? P.V[mu * L + lam] : 0.0f;
    }
    for (int e = threadIdx.x; e < NSEG * RS + 128; e += 256) rows[e] = 0.0;
    for (int e = threadIdx.x; e < ntab * tsize; e += 256) tabs[e] = 0.0;
    if (threadIdx.x < 8) counters[threadIdx.x] = -1;
    if (threadIdx.x == 0) { vl[L * pitch] = 0.0f; mrf_wait_init(&wait_lds, P.fault, P.spin_limit); }
    __syncthreads();
    const MrfWaitBlock *const wait_block = &wait_lds;
    int *const pre_done = counters, *const chain_done = counters + 2, *const post_done = counters + 3;
    const auto look = [](int *counter) {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    };
    const auto post = [](int *counter, int n) {               // (written by every lane: the same word)
        __hip_atomic_store(counter, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };

    // this workgroup's scanlines: NSEG consecutive ones of the launch's direction
    const int r = P.r_first;
    const unsigned nsc = (unsigned)P.g.nscan[r];
    const unsigned sl = blockIdx.x * NSEG + seg;
    const bool act = sl < (unsigned)P.g.B * nsc;
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0 = 0, x0 = 0, len = 0;
    int last = 0;                                             // the scanline's last node, where the replay starts
    const int nstep = dh * P.g.W + dw;
    if (act) {
        const int b = (int)(sl / nsc);
        mrf_geom_head(P.g.H, P.g.W, dh, dw, sl - (unsigned)b * nsc, y0, x0, len);
        last = (b * P.g.H + y0) * P.g.W + x0 + (len - 1) * nstep;
    }
    int maxlen = 0;
#pragma unroll
    for (int sg = 0; sg < NSEG; ++sg) {
        const int l2 = __builtin_amdgcn_readlane(len, sg * SEG);
        maxlen = l2 > maxlen ? l2 : maxlen;
    }
    const size_t N = (size_t)P.g.N, NL4 = N * L * 4;
    const unsigned estep = (unsigned)(nstep * L);
    const bool any = lam0 < L;
    unsigned ce = (unsigned)last * (unsigned)L + (unsigned)lam0;      // first entry of the node at hand

    if (wv == 0) {
        // ---- the chain ---------------------------------------------------------------------------------
        __builtin_amdgcn_s_setprio(3);
        const mrf_buf bs = mrf_buffer(P.S + (size_t)r * N * L, NL4);
        double *sb = rows + seg * RS;
        double *spare = rows + NSEG * RS + lane;              // where a lane with nothing to add adds
        const double cscale = (double)P.carry_scale[r];
        float out[NL];
#pragma unroll
        for (int s = 0; s < NL; ++s) out[s] = 0.0f;
        // the last node of a scanline has no successor in direction r
        mrf_buf_store_f32xn<NL>(bs, (int)act & (int)any ? ce << 2 : MRF_BUF_NONE, out);
        if (maxlen == 0) return;
        const auto await = [&](int tt) {
            int turns = 0;
            while (look(&pre_done[tt & 1]) < tt) mrf_wait_turn(wait_block, turns);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        };
        double ext[NL], carry[NL];
        unsigned pk;
        const auto fetch = [&](int slot) {
#pragma unroll
            for (int s = 0; s < NL; ++s) ext[s] = r_ext[(slot * NL + s) * 64 + lane];
            pk = r_p[slot * 64 + lane];
        };
        await(0);
        fetch(0);
#pragma unroll
        for (int s = 0; s < NL; ++s) carry[s] = 0.0;
        for (int tt = 0;;) {
#pragma unroll
            for (int u = 0; u < NR; ++u, ++tt) {              // step tt uses slot u = tt % NR
                double g[NL];
                int pv[NL];
#pragma unroll
                for (int s = 0; s < NL; ++s) {
                    r_cin[(u * NL + s) * 64 + lane] = carry[s];
                    g[s] = carry[s] + ext[s];
                    pv[s] = (int)((pk >> (8 * s)) & 255u);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                post(chain_done, tt);                         // (LDS keeps a wavefront's operations in order)
                // (a lane merges its labels that go where its first one goes, and lanes whose first label goes where lane 0's
                // does are summed by DPP for lane 0: mrf_bwd_sweep_narrow above)
                double g0 = g[0];
#pragma unroll
                for (int s = 1; s < NL; ++s) g0 += pv[s] == pv[0] ? g[s] : 0.0;
                const bool common = pv[0] == mrf_segment_lane0<SEG>(pv[0]);
                const double gc0 = mrf_segment_sum_f64<SEG>(common ? g0 : 0.0);
                __hip_atomic_fetch_add((int)!common | (int)(li == 0) ? &sb[pv[0]] : spare, common ? gc0 : g0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
                for (int s = 1; s < NL; ++s)
                    __hip_atomic_fetch_add(pv[s] != pv[0] ? &sb[pv[s]] : spare, g[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                mrf_wave_lds_fence();
                // in one batch behind the scatter: the counter of the next node's wavefront, then that node's ring entries, then
                // the scattered vector
                const int flag = __hip_atomic_load(&pre_done[(u + 1) & 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                fetch((u + 1) % NR);
                double sv[NL];
#pragma unroll
                for (int s = 0; s < NL; ++s) sv[s] = sb[lam0 + s];
                mrf_wave_lds_fence();
#pragma unroll
                for (int s = 0; s < NL; ++s) {
                    out[s] = (float)sv[s];
                    carry[s] = cscale * sv[s];
                    sb[lam0 + s] = 0.0;
                }
                ce -= estep;
                // node i has a predecessor: replay its update
                mrf_buf_store_f32xn<NL>(bs, (int)(tt < len - 1) & (int)any ? ce << 2 : MRF_BUF_NONE, out);
                if (__builtin_expect(tt + 1 >= maxlen, 0)) return;    // (uniform)
                if (__builtin_expect(__builtin_amdgcn_readfirstlane(flag) < tt + 1, 0)) {
                    await(tt + 1);
                    fetch((u + 1) % NR);
                }
            }
        }
    }

    if (wv <= 2) {
        // ---- pre: step tt of wavefront jw = tt % 2 ----------------------------------------------------------
        const int jw = wv - 1;
        const bool own_unary = UNARY && r == P.unary_dir;
        const unsigned no_old = own_unary && !P.unary_init ? 0u : MRF_BUF_NONE;
        const mrf_buf bp = mrf_buffer(P.p + (size_t)r * N * L, N * L), bq = mrf_buffer(P.q + (size_t)r * N, N);
        const mrf_buf bw = mrf_buffer(P.w + (P.w_mul ? (size_t)r * N : 0), P.w_mul ? N * 4 : 4), bu = mrf_buffer(P.gunary, NL4);
        mrf_buf src[NS];
        double cG[NS], cT[NS];
        const int nsrc = P.n_src[r];
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            const bool live = c < nsrc, isgc = c == nsrc && P.use_gc;
            // (empty slots are empty views: nothing is read for them)
            src[c] = mrf_buffer(live ? P.src_base + (size_t)P.src_dir[r][c] * P.src_stride : P.gc, live || isgc ? NL4 : 0);
            cG[c] = live ? (double)P.coefG[r][c] : (isgc ? 1.0 : 0.0);
            cT[c] = live ? (double)P.coefT[r][c] : (isgc ? 1.0 : 0.0);
        }
        // p of the lane's labels: one access of 1, 2 or 4 bytes that stays inside the node's L bytes, and a shift
        constexpr int PB = NL == 1 ? 1 : (NL == 2 ? 2 : 4);
        const int p_at = any ? (lam0 < L - PB ? lam0 : L - PB) : 0, p_shift = any ? 8 * (lam0 - p_at) : 0;
        const auto load_p = [&](unsigned at) {
            if constexpr (PB == 1) return (unsigned)mrf_buf_u8(bp, at);
            else if constexpr (PB == 2) return (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(bp, at, 0, 0);
            else return (unsigned)__builtin_amdgcn_raw_buffer_load_b32(bp, at, 0, 0);
        };
        struct In {
            float v[NS][NL];
            float u[UNARY ? NL : 1];                          // old grad theta_i (0 unless accumulating)
            unsigned p;
            int q;
            float w;
        };
        In A[D], B[D];
        // (the prefetch walks on past the first node: what it then loads is another node or nothing, and never used)
        unsigned pi = (unsigned)(last - jw * nstep), pe = (unsigned)(last - jw * nstep) * (unsigned)L;
        const auto prefetch = [&](In &in) {
            const unsigned at = any ? (pe + (unsigned)lam0) << 2 : MRF_BUF_NONE;
#pragma unroll
            for (int c = 0; c < NS; ++c) mrf_buf_f32xn<NL>(src[c], at, in.v[c]);
            if constexpr (UNARY) mrf_buf_f32xn<NL>(bu, no_old ? MRF_BUF_NONE : at, in.u);
            in.p = load_p(any ? pe + (unsigned)p_at : MRF_BUF_NONE);
            in.q = mrf_buf_u8(bq, pi);
            in.w = GV ? mrf_buf_f32(bw, P.w_mul ? pi * 4u : 0u) : 0.0f;
            pe -= 2 * estep;
            pi -= (unsigned)(2 * nstep);
        };
        int freed = -1;
        const auto group = [&](const In (&in)[D], int it0) {
#pragma unroll
            for (int u = 0; u < D; ++u) {
                const int tt = jw + 2 * (it0 + u);
                double ext[NL], part = 0.0;
#pragma unroll
                for (int s = 0; s < NL; ++s) {
                    double e = cG[0] * (double)in[u].v[0][s];
#pragma unroll
                    for (int c = 1; c < NS; ++c) e = __builtin_fma(cG[c], (double)in[u].v[c][s], e);
                    ext[s] = e;
                    part = s == 0 ? e : part + e;
                }
                // back Eq. isgmr-norm: the entry at q loses the label sum
                const double tot = mrf_segment_sum_f64<SEG>(part);
                const int qv = in[u].q < L ? in[u].q : L - 1;
                const unsigned pw = in[u].p >> p_shift;
                unsigned pk = 0;
#pragma unroll
                for (int s = 0; s < NL; ++s) {
                    if (lam0 + s == qv) ext[s] -= tot;
                    const unsigned pr = (pw >> (8 * s)) & 255u;
                    pk |= (pr < (unsigned)L ? pr : (unsigned)(L - 1)) << (8 * s);
                }
                double all[NL];
                if constexpr (UNARY) {
                    // grad theta_i: everything every direction passed back to node i, but for the carry
#pragma unroll
                    for (int s = 0; s < NL; ++s) {
                        double a = (double)in[u].u[s];
#pragma unroll
                        for (int c = 0; c < NS; ++c) a = __builtin_fma(cT[c], (double)in[u].v[c][s], a);
                        all[s] = a;
                    }
                }
                if (tt >= maxlen) break;                      // (uniform)
                int turns = 0;
                while (freed < tt - NR) {
                    freed = look(post_done);
                    if (freed < tt - NR) mrf_wait_turn(wait_block, turns);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                const int slot = tt & (NR - 1);
#pragma unroll
                for (int s = 0; s < NL; ++s) {
                    r_ext[(slot * NL + s) * 64 + lane] = ext[s];
                    if constexpr (UNARY) r_all[(slot * NL + s) * 64 + lane] = all[s];
                }
                r_p[slot * 64 + lane] = pk;
                if constexpr (GV) r_w[slot * 64 + lane] = in[u].w;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                post(&pre_done[jw], tt);
            }
        };
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(A[u]);
        for (int it0 = 0; jw + 2 * it0 < maxlen; it0 += 2 * D) {
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(B[u]);
            __builtin_amdgcn_sched_barrier(0);
            group(A, it0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(A[u]);
            __builtin_amdgcn_sched_barrier(0);
            group(B, it0 + D);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        // ---- post ----------------------------------------------------------------------------------------
        const bool own_unary = UNARY && r == P.unary_dir;
        const mrf_buf bu = mrf_buffer(P.gunary, NL4);
        const mrf_buf bgw = mrf_buffer(P.gw ? P.gw + (size_t)r * N : nullptr, P.gw ? N * 4 : 0);
        double *tab = tabs + (GV ? (seg % ntab) * tsize : 0), *spare = rows + NSEG * RS + 64 + lane;
        // edge-weight gradients of eight nodes: lane li < 8 of a segment keeps that of the li-th, one access adds them all
        static_assert(SEG >= 8, "lanes that keep edge-weight gradients");
        float gwkeep = 0.0f;
        int seen = -1;
        for (int tt = 0; tt < maxlen; ++tt) {
            int turns = 0;
            while (seen < tt) {
                seen = look(chain_done);
                if (seen < tt) mrf_wait_turn(wait_block, turns);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            const int slot = tt & (NR - 1);
            double g[NL];
            float out[NL];
            const unsigned pk = r_p[slot * 64 + lane];
            const double w = GV ? (double)r_w[slot * 64 + lane] : 0.0;
#pragma unroll
            for (int s = 0; s < NL; ++s) {
                const double cin = r_cin[(slot * NL + s) * 64 + lane];
                g[s] = cin + r_ext[(slot * NL + s) * 64 + lane];
                if constexpr (UNARY) out[s] = (float)(cin + r_all[(slot * NL + s) * 64 + lane]);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            post(post_done, tt);
            if constexpr (UNARY) mrf_buf_store_f32xn<NL>(bu, (int)(tt < len) & (int)any & (int)own_unary ? ce << 2 : MRF_BUF_NONE, out);
            const bool update = tt < len - 1;                 // node i has a predecessor: its update is replayed
            int at[NL];
#pragma unroll
            // (where there is no label p is 0, and the 0 behind V is met there: an infinite V[0][0] must not be)
            for (int s = 0; s < NL; ++s) at[s] = __mul24((int)((pk >> (8 * s)) & 255u), pitch) + (any ? lam0 + s : L * pitch);
            // (formed whether it is wanted or not: the view of an array that is not there holds nothing)
            double acc = g[0] * (double)vl[any ? at[0] : L * pitch];
#pragma unroll
            for (int s = 1; s < NL; ++s) acc = __builtin_fma(g[s], (double)vl[any ? at[s] : L * pitch], acc);     // (g is 0 where there is no label)
            acc = mrf_segment_sum_f64<SEG>(acc);
            gwkeep = li == (tt & 7) ? (float)acc : gwkeep;
            // one writer per entry and launch: a no-return atomic is a plain accumulate
            if ((tt & 7) == 7 || tt + 1 == maxlen) {
                const int t8 = (tt & ~7) + li;                // this lane's node counts if it has been passed and has a predecessor
                mrf_buf_add_f32(bgw, (int)(li < 8) & (int)(t8 <= tt) & (int)(t8 < len - 1) ? (unsigned)(last - t8 * nstep) << 2 : MRF_BUF_NONE, gwkeep);
            }
            if constexpr (GV) {
                // (no short-circuit in the conditions: it would become a branch)
#pragma unroll
                for (int s = 0; s < NL; ++s)
                    __hip_atomic_fetch_add((int)update & (int)any ? &tab[at[s]] : spare, w * g[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            ce -= estep;
        }
    }
    if constexpr (GV) {
        // (the chain wavefront has ended or will; a barrier waits for the wavefronts that are left)
        __syncthreads();
        double *slot = P.gV + (size_t)blockIdx.x * L * L;
        for (int e = (int)threadIdx.x - 64; e < L * L; e += 192) {
            const int mu = e / L, at = mu * pitch + (e - mu * L);
            double v = tabs[at];
            for (int k = 1; k < ntab; ++k) v += tabs[k * tsize + at];
            mrf_slot_add(&slot[e], v);
        }
    }
}

// ---- the chain layout for up to 32 labels: two scanlines per workgroup -------------------------
//
// mrf_bwd_sweep_chain with the lanes of every wavefront divided as in mrf_bwd_sweep_packed: lanes 0-31 hold
// the labels of one scanline, lanes 32-63 those of the next (one direction per launch, so everything but the
// head and the length of the scanline is shared).  Ring entries are indexed by lane; a scatter target is
// stored as 32 seg + p, so the chain wavefront's step is that of mrf_bwd_sweep_chain unchanged: it neither
// knows nor cares that its 64 entries are two vectors.  A scanline that is shorter than its neighbour gets
// zeros with targets of their own for the steps past its first node, and nothing of those steps is stored.
// For launches of 257 to 1,536 scanlines of up to 32 labels with one direction (TRWP), where the wavefronts of
// mrf_bwd_sweep_narrow would have a SIMD to themselves and do all of a node's work in sequence.
__host__ __device__ inline size_t mrf_bwd_chain_pk_lds_bytes(int NI, int L, bool gv)
{
    const size_t NR = 2 * (size_t)NI, LL = 64;
    const size_t arrays = sizeof(double) * (3 * NR * LL + LL + (gv ? (size_t)2 * L * L : 0)) +
                          sizeof(float) * (NR * LL + (size_t)L * L) + sizeof(int) * (MRF_CHAIN_MAX_HELPERS + 4) + NR * LL;
    return (arrays + 7) / 8 * 8 + sizeof(MrfWaitBlock);
}

template <int NS, int D, int NI, bool GV>
__global__ void __launch_bounds__(64 * (1 + NI)) mrf_bwd_sweep_chain_pk(const MrfBwdParams P)
{
    constexpr int NR = 2 * NI;
    constexpr int LL = 64;
    static_assert(NI >= 2 && NI <= MRF_CHAIN_MAX_HELPERS, "helpers per pair of scanlines");
    extern __shared__ __align__(16) unsigned char mrf_bsmem[];
    const int L = P.g.L;
    // carved in the order of mrf_bwd_chain_pk_lds_bytes
    double *a_ext = reinterpret_cast<double *>(mrf_bsmem);       // [NR][LL] pre -> chain, post
    double *b_cin = a_ext + NR * LL;                             // [NR][LL] chain -> post: carry that entered the node
    double *b_sv = b_cin + NR * LL;                              // [NR][LL]                scattered vector that left it
    double *sbuf = b_sv + NR * LL;                               // [LL] scatter target of the chain
    double *gvacc = sbuf + LL;                                   // [2][L*L] V-gradient tables of the two scanlines (GV): LDS adds by all helpers
    float *a_extT = reinterpret_cast<float *>(gvacc + (GV ? 2 * L * L : 0));   // [NR][LL] pre -> post (grad theta)
    float *vl = a_extT + NR * LL;                                // [L*L] V
    int *pre_done = reinterpret_cast<int *>(vl + L * L);         // [MRF_CHAIN_MAX_HELPERS] per helper: last step published
    int *chain_done = pre_done + MRF_CHAIN_MAX_HELPERS;          // last step the chain finished
    uint8_t *a_p = reinterpret_cast<uint8_t *>(chain_done + 4);  // [NR][LL]
    MrfWaitBlock &wait_lds = *reinterpret_cast<MrfWaitBlock *>(
        mrf_bsmem + ((a_p + NR * LL - mrf_bsmem) + 7) / 8 * 8);
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int seg = lane >> 5, lam = lane & 31;
    const bool valid = lam < L;
    const int lc = valid ? lam : 0;
    const long long N = P.g.N;

    for (int e = threadIdx.x; e < L * L; e += blockDim.x) vl[e] = P.V[e];
    if (GV)
        for (int e = threadIdx.x; e < 2 * L * L; e += blockDim.x) gvacc[e] = 0.0;
    if (threadIdx.x < MRF_CHAIN_MAX_HELPERS) pre_done[threadIdx.x] = (int)threadIdx.x - NI;
    if (threadIdx.x == 0) { *chain_done = -1; mrf_wait_init(&wait_lds, P.fault, P.spin_limit); }
    for (int e = threadIdx.x; e < LL; e += blockDim.x) sbuf[e] = 0.0;
    __syncthreads();

    // one direction per launch; the two scanlines of the workgroup
    const int r = P.r_first;
    const long long sl = (long long)blockIdx.x * 2 + seg;
    const bool act_seg = sl < P.total_scanlines;
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0 = 0, x0 = 0, len = 0;
    long long head = 0;
    if (act_seg) {
        const unsigned nsc = (unsigned)P.g.nscan[r];
        const int b = (int)((unsigned)sl / nsc);
        const unsigned t = (unsigned)sl - (unsigned)b * nsc;
        mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
        head = ((long long)b * P.g.H + y0) * P.g.W + x0;
    }
    const long long nstep = (long long)dh * P.g.W + dw;
    const int len0 = __builtin_amdgcn_readlane(len, 0), len1 = __builtin_amdgcn_readlane(len, 32);
    const int maxlen = len0 > len1 ? len0 : len1;

    if (wv == 0) {
        // ---- the chain: step tt handles node len-1-tt of either scanline (mrf_bwd_sweep_chain's step) ----
        const double cscale = (double)P.carry_scale[r];
        double carry = 0.0, ext;
        int pv;
        auto await = [&](int u, int tt) {
            int sn;
            int wait_turns = 0;
            do {
                sn = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(&pre_done[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                if (sn < tt) mrf_wait_turn(&wait_lds, wait_turns);
            } while (sn < tt);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        };
        if (maxlen > 0) {
            await(0, 0);
            ext = a_ext[lane];
            pv = a_p[lane];
        } else {
            ext = 0.0;
            pv = lane;
        }
        int sb = 0;
        for (int t0 = 0; t0 < maxlen; t0 += NI) {
#pragma unroll
            for (int u = 0; u < NI; ++u) {
                const int tt = t0 + u;
                if (tt < maxlen) {
                    const int slot = sb + u;
                    const int un = (u + 1 == NI) ? 0 : u + 1;
                    const int slotn = (u + 1 == NI) ? (sb == 0 ? NI : 0) : slot + 1;
                    const bool more = tt + 1 < maxlen;
                    const double g = carry + ext;
                    b_cin[slot * LL + lane] = carry;
                    __hip_atomic_fetch_add(&sbuf[pv], g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    mrf_wave_lds_fence();
                    const int flag = __hip_atomic_load(&pre_done[un], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    ext = a_ext[slotn * LL + lane];
                    pv = a_p[slotn * LL + lane];
                    const double sv = sbuf[lane];
                    if (__builtin_expect(more && __builtin_amdgcn_readfirstlane(flag) < tt + 1, 0)) {
                        await(un, tt + 1);
                        ext = a_ext[slotn * LL + lane];
                        pv = a_p[slotn * LL + lane];
                    }
                    // everything this wavefront sent to LDS before the reads above has landed
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                    __builtin_amdgcn_wave_barrier();
                    if (tt > 0)
                        __hip_atomic_store(chain_done, tt - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    sbuf[lane] = 0.0;
                    b_sv[slot * LL + lane] = sv;
                    carry = cscale * sv;
                }
            }
            sb = (sb == 0) ? NI : 0;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) __hip_atomic_store(chain_done, maxlen - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return;
    }

    // ---- helpers ---------------------------------------------------------------------------
    const int jw = wv - 1;
    const bool own_unary = (r == P.unary_dir);
    const bool unary_old = own_unary && !P.unary_init;
    const uint8_t *pbase = P.p + (size_t)r * N * L;
    const uint8_t *qbase = P.q + (size_t)r * N;
    const float *wbase = P.w + (P.w_mul ? (size_t)r * N : 0);

    const float *src[NS];
    double cG[NS], cT[NS];
    const int nsrc = P.n_src[r];
#pragma unroll
    for (int c = 0; c < NS; ++c) {
        const bool live = c < nsrc;
        const bool isgc = (c == nsrc) && P.use_gc;
        src[c] = live ? P.src_base + (size_t)P.src_dir[r][c] * P.src_stride : P.gc;
        cG[c] = live ? (double)P.coefG[r][c] : (isgc ? 1.0 : 0.0);
        cT[c] = live ? (double)P.coefT[r][c] : (isgc ? 1.0 : 0.0);
    }

    // the last node of a scanline has no successor in direction r
    if (jw == 0 && act_seg && valid && len > 0)
        P.S[((size_t)r * N + head + (long long)(len - 1) * nstep) * L + lam] = 0.0f;

    // own steps: tt = jw + it * NI, it = 0 .. T-1; one more turn for the last post
    const int T = maxlen > jw ? (maxlen - jw + NI - 1) / NI : 0;
    float cur[D][NS], nxt[D][NS];
    float ucur[D], unxt[D];
    int pcur[D], pnxt[D], qcur[D], qnxt[D];
    float wcur[D], wnxt[D];                 // edge weight of the node's incoming edge (GV)
    auto prefetch = [&](float (&dst)[NS], float &udst, int &pdst, int &qdst, float &wdst, int it) {
        int n = len - 1 - (jw + it * NI);
        n = n > 0 ? n : 0;
        const long long i = head + (long long)n * nstep;
#pragma unroll
        for (int c = 0; c < NS; ++c) dst[c] = src[c][(size_t)i * L + lc];
        udst = P.gunary[unary_old ? (size_t)i * L + lc : 0];      // one cached word unless it is needed
        pdst = pbase[(size_t)i * L + lc];
        qdst = qbase[(size_t)i];
        wdst = GV ? wbase[(size_t)(i * P.w_mul)] : 0.0f;
    };
    if (T > 0) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(cur[u], ucur[u], pcur[u], qcur[u], wcur[u], u);
    }
    double *gvl = gvacc + (GV ? seg * L * L : 0);
    float wlast = 0.0f;                     // weight of the node whose post stage comes next

    int chain_seen = -1;
    for (int it0 = 0; it0 < T + 1 && T > 0; it0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(nxt[u], unxt[u], pnxt[u], qnxt[u], wnxt[u], it0 + D + u);
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int tt = jw + (it0 + u) * NI;
            if (tt < maxlen) {
                // ---- pre(tt): everything of node len-1-tt that does not need the carry -------
                const int slot = tt % NR;
                const bool live = valid && tt < len;       // (false for the whole of a scanline that has ended)
                double e = 0.0, eT = 0.0;
#pragma unroll
                for (int c = 0; c < NS; ++c) e = __builtin_fma(cG[c], (double)cur[u][c], e);
                if (own_unary) {
#pragma unroll
                    for (int c = 0; c < NS; ++c) eT = __builtin_fma(cT[c], (double)cur[u][c], eT);
                    eT += unary_old ? (double)ucur[u] : 0.0;     // (the buffer may hold anything at first)
                    a_extT[slot * LL + lane] = (float)eT;
                }
                const double ev = live ? e : 0.0;
                // (labels past L and scanlines that have ended scatter their zeros to entries of their own)
                a_p[slot * LL + lane] = (uint8_t)(live ? 32 * seg + (pcur[u] < L ? pcur[u] : L - 1) : lane);
                // back Eq. isgmr-norm, on the part of g that is known here: the entry at q loses the label sum
                const double tot = mrf_segment_sum_f64<32>(ev);
                const int qv = qcur[u] < L ? qcur[u] : L - 1;
                a_ext[slot * LL + lane] = (live && lam == qv) ? ev - tot : ev;
                // (LDS keeps a wavefront's operations in order: the counter lands behind the entries)
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                if (lane == 0) __hip_atomic_store(&pre_done[jw], tt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            const int tp = tt - NI;
            if (tp >= 0 && tp < maxlen) {
                // ---- post(tp): what is left of node len-1-tp once the chain has passed --------
                int wait_turns = 0;
                while (chain_seen < tp) {
                    chain_seen = __builtin_amdgcn_readfirstlane(
                        __hip_atomic_load(chain_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                    if (chain_seen < tp) mrf_wait_turn(&wait_lds, wait_turns);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                const int slot = tp % NR;
                const int n = len - 1 - tp;
                const bool act = valid && n >= 0;        // the node exists
                const bool update = valid && n > 0;      // and has a predecessor: its update is replayed
                const long long i = head + (long long)(n > 0 ? n : 0) * nstep;
                const double cin = b_cin[slot * LL + lane];
                if (own_unary && act) P.gunary[(size_t)i * L + lam] = (float)(cin + (double)a_extT[slot * LL + lane]);
                if (update) P.S[((size_t)r * N + i - nstep) * L + lam] = (float)b_sv[slot * LL + lane];
                if (P.gw || GV) {
                    const double g = cin + a_ext[slot * LL + lane];    // as the chain formed it
                    const int pv = update ? (int)a_p[slot * LL + lane] - 32 * seg : 0;
                    if (P.gw) {
                        double acc = update ? g * (double)vl[__mul24(pv, L) + lam] : 0.0;
                        acc = mrf_segment_sum_f64<32>(acc);
                        // one writer per entry and launch: a no-return atomic is a plain accumulate
                        if (n > 0 && lam == 0)
                            __hip_atomic_fetch_add(&P.gw[(size_t)r * N + i], (float)acc, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
                    }
                    if (GV && update)
                        __hip_atomic_fetch_add(&gvl[__mul24(pv, L) + lam], (double)wlast * g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            wlast = wcur[u];
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            qcur[u] = qnxt[u];
            wcur[u] = wnxt[u];
            ucur[u] = unxt[u];
            pcur[u] = pnxt[u];
#pragma unroll
            for (int c = 0; c < NS; ++c) cur[u][c] = nxt[u][c];
        }
    }
    if (GV) {
        // the two tables, summed, go to the workgroup's slot (the barrier waits for the helpers: the chain
        // wavefront has ended or will)
        __syncthreads();
        double *gVs = P.gV + (size_t)blockIdx.x * L * L;
        for (int e = (int)threadIdx.x - 64; e < L * L; e += 64 * NI) mrf_slot_add(&gVs[e], gvacc[e] + gvacc[L * L + e]);
    }
}

// ISGMR, after the sweeps of iteration k: grad theta_i += sum_r s^r_i, and the gradient of
// m^d (= m-hat^d of iteration k-1) is sum over r not in {d, d-} of s^r_i.
struct MrfCombineParams {
    long long NL;            // N*L
    int R;
    int opp[MRF_MAXR];
    const float *S;          // [R][N][L]
    const float *gc;         // grad c, read when first != 0
    float *gunary;           // [N][L]
    float *ghat;             // [R][N][L] out (next iteration's grad m-hat), NULL on the last; only the slabs of
                             // directions d with canon[d] == d are written
    int canon[MRF_MAXR];     // a direction and its opposite exclude the same pair {d, d-}, so their grad m-hat
                             // is one and the same array: canon[d] = the lower index of the two
    int first;               // first processed iteration: grad theta starts from grad c
    int skip_dir;            // direction whose s does not enter the sums (already added elsewhere), or -1
};

// RT: number of directions rounded up to 4, 8 or 16 (the loops below are unrolled to it);
// VEC: consecutive entries per thread (4 needs N*L divisible by 4 and 16-byte aligned arrays)
template <int RT, int VEC>
__global__ void __launch_bounds__(256) mrf_isgmr_bwd_combine(const MrfCombineParams P)
{
    typedef float vecf __attribute__((ext_vector_type(VEC)));
    const long long stride = (long long)gridDim.x * blockDim.x * VEC;
    for (long long e = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * VEC; e < P.NL; e += stride) {
        // every s^r_i is read once; sums are formed in double, where removing the two excluded
        // directions from the total loses nothing that float storage would keep
        vecf sraw[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r)
            sraw[r] = (r < P.R) ? *reinterpret_cast<const vecf *>(P.S + (size_t)r * P.NL + e) : vecf(0.0f);
        const vecf braw = *reinterpret_cast<const vecf *>((P.first ? P.gc : P.gunary) + e);
        vecf uout;
        vecf gout[RT];
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            double sv[RT];
            double tot = 0.0;
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                sv[r] = (r == P.skip_dir) ? 0.0 : (double)sraw[r][v];
                tot += sv[r];
            }
            uout[v] = (float)((double)braw[v] + tot);
#pragma unroll
            for (int d = 0; d < RT; ++d) {
                double g = tot - sv[d];
#pragma unroll
                for (int r = 0; r < RT; ++r)
                    if (r == P.opp[d]) g -= sv[r];
                gout[d][v] = (float)g;
            }
        }
        *reinterpret_cast<vecf *>(P.gunary + e) = uout;
        if (P.ghat) {
#pragma unroll
            for (int d = 0; d < RT; ++d)
                if (d < P.R && P.canon[d] == d) *reinterpret_cast<vecf *>(P.ghat + (size_t)d * P.NL + e) = gout[d];
        }
    }
}
