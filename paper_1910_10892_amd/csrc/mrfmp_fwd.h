// Forward sweeps of ISGMR (Alg. 1) and TRWP (Alg. 2) and the final aggregation
// (Eq. isgmr-aggregation, Eq. disp), hand-written for gfx950.
//
// Dense sweep kernel: one workgroup walks one scanline, node after node.  The L x L
// min-plus of a node is split over the NW wavefronts of the workgroup by source label mu
// (wavefront w owns MCH consecutive mu); lanes own destination labels lambda
// (lambda = lane + 64*s, s < LP).  The wavefront's slice of V lives in registers for the
// whole sweep; h[mu] (the lambda-independent part of the update) is broadcast from LDS.
// Partial minima meet in LDS once per node (one workgroup barrier per node); every
// wavefront then finishes the node redundantly (merge in ascending mu, argmin over
// lambda, reparametrisation), so no second barrier is needed.
//
// The node-to-node dependence makes a sweep latency bound, so everything that does not
// depend on the previous node (unary, other directions' messages, edge weight) is loaded
// a group of D nodes ahead into a second register set, unconditionally (clamped
// addresses), so that a load is first waited for at least D node steps after its issue.
//
// Kernels in this file, all computing the same update in the same rounding order:
//   mrf_fwd_sweep               dense O(L^2), NW wavefronts per scanline split the source labels
//   mrf_fwd_sweep_sliced        dense, L > 64: the same with the O(L) work of a node divided among the wavefronts
//   mrf_fwd_sweep_halves        dense, 33..128 labels: chunk minima, argmin by a second look at the winning chunk
//   mrf_fwd_sweep_narrow        dense, L <= 32: several scanlines of one direction per wavefront, argmin in two levels
//   mrf_fwd_sweep_packed        the same for launches of few scanlines, the work of a node divided among four wavefronts (five
//                               template parameters), or with 64-bit offsets and scanlines of any direction (six)
//   mrf_fwd_sweep_edge          pairwise potentials given per edge, 33..64 labels
//   mrf_fwd_sweep_edge_groups   the same for up to 32 labels, groups of lanes sharing the source labels
//   mrf_aggregate               final costs and labels
//   mrf_fwd_sweep_window        truncated models: window of 2 TW - 1 source labels per label
//   mrf_fwd_sweep_window_duo    the same with the dependency chain (values) on one wavefront and
//                               index / loader wavefronts beside it, connected by LDS rings
//   mrf_fwd_sweep_window_split  the same, one wavefront per 64 labels in lock step
//   mrf_fwd_sweep_window_squad  value wavefronts per 64 labels, a loader, index wavefronts per node
// Which one a launch gets is host arithmetic on the launch shape (dispatch_fwd).
#pragma once

#include "mrfmp_device.h"

struct MrfFwdParams {
    MrfGeom g;
    int r_first, r_count;                  // directions swept by this launch
    long long blk_begin[MRF_MAXR + 1];     // prefix sums of B*nscan over those directions
    int pack_begin[MRF_MAXR + 1];          // mrf_fwd_sweep_narrow: the same in wavefronts, every direction padded to whole ones
    const float *unary, *V;
    const float *w;                        // [R][N] edge weights, or one float when w_mul == 0
    int w_mul;                             // 1: per-edge weights, 0: the scalar at w[0]
    const float *m_in;                     // [R][N][L] messages read
    float *m_out;                          // [R][N][L] messages written (TRWP: same array)
    uint8_t *p, *q;                        // [R][N][L], [R][N] of this iteration
    float rho[MRF_MAXR];
    const float *rho_e;                    // [R][N] rho of edge (i-r, i) at node i (TRWP), or NULL: then rho[] applies
                                           // (read by mrf_fwd_sweep, mrf_fwd_sweep_window and mrf_fwd_sweep_edge only)
    const float *Te;                       // [R][N][L][L] pairwise potentials per edge (mrf_fwd_sweep_edge), or NULL
    // per swept direction r: the message arrays that enter h, in summation order.  The first
    // n_pre[r] are added before this direction's own running message, the rest after it.
    // (whole words: those come through the scalar cache, a byte takes a vector load from memory that no cache holds yet)
    int src_dir[MRF_MAXR][MRF_MAXR];
    int n_pre[MRF_MAXR], n_src[MRF_MAXR];
    int rm_slot[MRF_MAXR];                 // position of r^- in src_dir[r], or -1 (term absent / still 0)
    int NW;                                // wavefronts per workgroup = ceil(L / MCH)
    int *fault;                            // launch-wide word raised when a wait between wavefronts is given up (mrf_wait_turn)
    int spin_limit;                        // microseconds after which a wait is given up
    int unary_slab[MRF_MAXR];              // direction r reads its lambda-independent start term at
                                           // unary + unary_slab[r] * N * L (0 unless mrf_isgmr_presum prepared them)
    int sgm_std;                           // standard single-pass SGM (Eq. sgm_old): the message carries the node's own
                                           // unary, m^r_i = theta_i + min_mu (m^r_{i-r} + theta_{i-r,i}); mrf_fwd_sweep only
};

// LP: labels per lane; MCH: source labels per wavefront; RMAX: bound on 1 + n_src;
// D: prefetch distance in nodes; TRWP: Eq. trwp (else Eq. isgmr)
template <int LP, int MCH, int RMAX, int D, bool TRWP>
__global__ void __launch_bounds__(64 * ((64 * LP + MCH - 1) / MCH))
mrf_fwd_sweep(const MrfFwdParams P)
{
    extern __shared__ __align__(16) unsigned char mrf_smem[];
    constexpr int NWMAX = (64 * LP + MCH - 1) / MCH;
    constexpr int LPAD = NWMAX * MCH;
    constexpr int SLOTS = 64 * LP;
    const int L = P.g.L, NW = P.NW;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // uniform, and known to be
    float *hbuf = reinterpret_cast<float *>(mrf_smem) + wv * LPAD;          // private to this wavefront
    float2 *part = reinterpret_cast<float2 *>(reinterpret_cast<float *>(mrf_smem) + NWMAX * LPAD);  // [2][NWMAX][SLOTS]

    // workgroup -> (direction r, image b, scanline t)
    const long long blk = blockIdx.x;
    const int ri = mrf_direction_of(P.blk_begin, P.r_count, blk);
    const int r = P.r_first + ri;
    const unsigned local = (unsigned)(blk - P.blk_begin[ri]);
    int b;
    unsigned t;
    mrf_geom_order(P.g.H, P.g.W, P.g.dh[r], P.g.dw[r], (unsigned)P.g.nscan[r], (unsigned)P.g.B, local, b, t);
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0, x0, len;
    mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
    const long long N = P.g.N;
    const long long head = ((long long)b * P.g.H + y0) * P.g.W + x0;
    const long long nstep = (long long)dh * P.g.W + dw;
    const float rho = P.rho[r];
    const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];

    // Sources of h: slot 0 = unary, slot c >= 1 = message array src_dir[r][c-1].  Unused
    // slots read the unary again and enter with factor 0: fma(0, x, v) = v exactly, and
    // fma(1, x, v) = v + x exactly, so the sum below is the plain left-to-right sum of the
    // live terms with this direction's running message inserted after the first n_pre.
    const float *src[RMAX];
    float use[RMAX], carry_at[RMAX + 1], is_rm[RMAX];
    const float vz = mrf_opaque_zero_f();     // keeps the flags below in vector registers
    // standard SGM adds the unary of node i itself after the minimum (Eq. sgm_old): slot 0 then
    // holds theta_i, one node further along the scanline, instead of theta_{i-r}
    const bool sgm_std = !TRWP && P.sgm_std;
    src[0] = P.unary + (size_t)P.unary_slab[r] * N * L + (sgm_std ? nstep * L : 0);
    use[0] = 1.0f;
    is_rm[0] = 0.0f;
#pragma unroll
    for (int c = 1; c < RMAX; ++c) {
        src[c] = (c <= n_src) ? P.m_in + (size_t)P.src_dir[r][c - 1] * N * L : src[0];
        use[c] = ((c <= n_src) ? 1.0f : 0.0f) + vz;
        is_rm[c] = ((c - 1 == rm_slot) ? 1.0f : 0.0f) + vz;
    }
#pragma unroll
    for (int c = 1; c <= RMAX; ++c) carry_at[c] = ((c == n_pre + 1) ? 1.0f : 0.0f) + vz;

    // this wavefront's slice of V: rows mu0 .. mu0+MCH-1, columns = the lane's lambdas
    const int mu0 = wv * MCH;
    float Vr[MCH][LP];
#pragma unroll
    for (int i = 0; i < MCH; ++i)
#pragma unroll
        for (int s = 0; s < LP; ++s) {
            const int mu = mu0 + i, lam = lane + 64 * s;
            Vr[i][s] = (mu < L && lam < L) ? P.V[(size_t)mu * L + lam] : 0.0f;
        }
    // padding of h beyond L, and partial minima of absent wavefronts, can never win a strict '<'
    for (int i = L + lane; i < LPAD; i += 64) hbuf[i] = INFINITY;
    if (NWMAX > 1) {
        for (int i = threadIdx.x; i < 2 * NWMAX * SLOTS; i += blockDim.x) part[i] = make_float2(INFINITY, 0.0f);
        __syncthreads();
    }

    // first node of the scanline: message 0, p = q = 0
    if (wv == 0) {
#pragma unroll
        for (int s = 0; s < LP; ++s) {
            const int lam = lane + 64 * s;
            if (lam < L) {
                // (standard SGM: with nothing before it, the first node's message is its unary)
                P.m_out[((size_t)r * N + head) * L + lam] = sgm_std ? P.unary[(size_t)head * L + lam] : 0.0f;
                P.p[((size_t)r * N + head) * L + lam] = 0;
            }
        }
        if (lane == 0) P.q[(size_t)r * N + head] = 0;
    }

    // Prefetch in groups of D nodes: while the D nodes of one group are processed from the
    // registers `cur`, the inputs of the next group are in flight into `nxt`.
    const int vzero = mrf_opaque_zero();
    const float *wbase = P.w + (P.w_mul ? (size_t)r * N : 0);
    const int lastsrc = len - 2;           // last node that is a predecessor
    float cur[D][RMAX][LP], nxt[D][RMAX][LP];
    float wcur[D], wnxt[D];
    float rcur[D], rnxt[D];                // rho of the edge (i-r, i): per edge if P.rho_e is given
    const float *rbase = P.rho_e ? P.rho_e + (size_t)r * N : nullptr;
    auto prefetch = [&](float (&dst)[RMAX][LP], float &wdst, float &rdst, int nj) {   // inputs of the update nj -> nj+1
        nj = nj < lastsrc ? nj : lastsrc;  // past the end: reload the last one, never used
        const long long j = head + (long long)nj * nstep;
#pragma unroll
        for (int c = 0; c < RMAX; ++c)
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const int lam = lane + 64 * s;
                dst[c][s] = src[c][(size_t)j * L + (lam < L ? lam : 0)];
            }
        wdst = wbase[(size_t)((j + nstep) * P.w_mul) + vzero];
        rdst = rho;
        if (TRWP && rbase) rdst = rbase[(size_t)(j + nstep) + vzero];
    };
    if (len >= 2) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(cur[u], wcur[u], rcur[u], u);
    }

    float carry[LP];   // normalised message of this direction at the previous node
#pragma unroll
    for (int s = 0; s < LP; ++s)
        carry[s] = (sgm_std && lane + 64 * s < L) ? P.unary[(size_t)head * L + lane + 64 * s] : 0.0f;
    int buf = 0, turn = 0;

    for (int n0 = 1; n0 < len; n0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(nxt[u], wnxt[u], rnxt[u], n0 - 1 + D + u);
#pragma unroll
        for (int u = 0; u < D; ++u) {
            // node index of i on the scanline; i-r is node n-1.  The last group may run past
            // the end of the scanline: those steps recompute the last node and store nothing.
            const int nn = n0 + u;
            const bool past = nn >= len;
            const int n = past ? len - 1 : nn;
            const long long i = head + (long long)n * nstep;

            // ---- lambda-independent part h[mu] at node i-r (lane's labels act as mu here) ----
            float a[LP];
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                float v = cur[u][0][s];
                float mrm = 0.0f;
                if (TRWP) {
                    // Eq. trwp: rho (theta_{i-r} + sum_d m^d_{i-r}) - m^{r-}_{i-r}
#pragma unroll
                    for (int c = 1; c < RMAX; ++c) {
                        v = __builtin_fmaf(carry_at[c], carry[s], v);
                        v = __builtin_fmaf(use[c], cur[u][c][s], v);
                        mrm = __builtin_fmaf(is_rm[c], cur[u][c][s], mrm);
                    }
                    v = __builtin_fmaf(carry_at[RMAX], carry[s], v);
                    v = rcur[u] * v;
                    v = v - mrm;
                } else {
                    // Eq. isgmr: theta_{i-r} + sum_{d not in {r, r-}} m^d_{i-r} (what iteration k left), then m-hat^r_{i-r}
#pragma unroll
                    for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(use[c], cur[u][c][s], v);
                    v = v + carry[s];
                    // Eq. sgm_old: the previous message alone (it holds theta_{i-r} already)
                    v = sgm_std ? carry[s] : v;
                }
                a[s] = v;
            }
            const float wgt = wcur[u];

#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const int lam = lane + 64 * s;
                if (lam < L) hbuf[lam] = a[s];
            }
            mrf_wave_lds_fence();

            // ---- min-plus over this wavefront's mu slice, lowest mu on ties ----
            float best[LP];
            int bidx[LP];
#pragma unroll
            for (int s = 0; s < LP; ++s) { best[s] = INFINITY; bidx[s] = 0; }
            // (compares, minima and index selects of the LP label slots go out in blocks that need
            // no wait states: mrf_argmin_step)
            mrf_static_for<MCH / 4>([&](auto q4) {
                constexpr int i4 = 4 * decltype(q4)::value;
                const float4 hv = *reinterpret_cast<const float4 *>(&hbuf[mu0 + i4]);
                const float hq[4] = { hv.x, hv.y, hv.z, hv.w };
                if constexpr (LP == 1) {
                    mrf_argmin_step2<i4>(best[0], bidx[0], __builtin_fmaf(wgt, Vr[i4][0], hq[0]),
                                         __builtin_fmaf(wgt, Vr[i4 + 1][0], hq[1]));
                    mrf_argmin_step2<i4 + 2>(best[0], bidx[0], __builtin_fmaf(wgt, Vr[i4 + 2][0], hq[2]),
                                             __builtin_fmaf(wgt, Vr[i4 + 3][0], hq[3]));
                } else {
                    mrf_static_for<4>([&](auto cc) {
                        constexpr int c = decltype(cc)::value;
                        float dlt[LP];
#pragma unroll
                        for (int s = 0; s < LP; ++s) dlt[s] = __builtin_fmaf(wgt, Vr[i4 + c][s], hq[c]);
                        mrf_argmin_step<i4 + c>(best, bidx, dlt);
                    });
                }
            });

            float tv[LP];
            int tp[LP];
            if (NWMAX > 1) {
                float2 *pb = part + (size_t)buf * NWMAX * SLOTS;
#pragma unroll
                for (int s = 0; s < LP; ++s)
                    pb[wv * SLOTS + lane + 64 * s] = make_float2(best[s], __int_as_float(mu0 + bidx[s]));
                mrf_block_sync_lds();
#pragma unroll
                for (int s = 0; s < LP; ++s) { tv[s] = INFINITY; tp[s] = 0; }
#pragma unroll
                for (int w2 = 0; w2 < NWMAX; ++w2) {
                    float ev[LP];
                    int ei[LP];
#pragma unroll
                    for (int s = 0; s < LP; ++s) {
                        const float2 e = pb[w2 * SLOTS + lane + 64 * s];
                        ev[s] = e.x;
                        ei[s] = __float_as_int(e.y);
                    }
                    mrf_argmin_merge<LP>(tv, tp, ev, ei);
                }
                buf ^= 1;
            } else {
#pragma unroll
                for (int s = 0; s < LP; ++s) { tv[s] = best[s]; tp[s] = bidx[s]; }
            }

            if (sgm_std) {
#pragma unroll
                for (int s = 0; s < LP; ++s) tv[s] = cur[u][0][s] + tv[s];     // theta_i + min_mu (...)
            }
            // ---- q = lowest argmin over lambda, reparametrisation (Eq. isgmr-norm) ----
            float mn = INFINITY;
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                if (lane + 64 * s >= L) tv[s] = INFINITY;
                mn = fminf(mn, tv[s]);
            }
            mn = mrf_wave_min(mn);
            int qidx = -1;
            float tq = mn;
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const unsigned long long bal = __ballot(tv[s] == mn);
                if (qidx < 0 && bal != 0ull) {
                    const int ql = __ffsll((long long)bal) - 1;
                    qidx = 64 * s + ql;
                    tq = mrf_readlane_f32(tv[s], ql);
                }
            }
#pragma unroll
            for (int s = 0; s < LP; ++s) carry[s] = (lane + 64 * s < L) ? tv[s] - tq : 0.0f;

            // ---- outputs of node i (the wavefronts take turns) ----
            if (wv == turn && !past) {
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int lam = lane + 64 * s;
                    if (lam < L) {
                        P.m_out[((size_t)r * N + i) * L + lam] = carry[s];
                        P.p[((size_t)r * N + i) * L + lam] = (uint8_t)tp[s];
                    }
                }
                if (lane == 0) P.q[(size_t)r * N + i] = (uint8_t)qidx;
            }
            turn = (turn + 1 == NW) ? 0 : turn + 1;
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            wcur[u] = wnxt[u];
            rcur[u] = rnxt[u];
#pragma unroll
            for (int c = 0; c < RMAX; ++c)
#pragma unroll
                for (int s = 0; s < LP; ++s) cur[u][c][s] = nxt[u][c][s];
        }
    }
}

// ---- dense sweep, every wavefront owns a slice of the labels ------------------------------------
//
// The same O(L^2) update as mrf_fwd_sweep for more than 64 labels, with the O(L) work of a node
// divided instead of repeated.  Wavefront w holds rows [32 w, 32 w + 32) of V in registers as
// before and evaluates their candidates for all L destination labels; but only these 32 labels
// are also its "home": it alone loads the inputs of h for them, merges the partial results of all
// wavefronts for them, normalises, keeps the running message for them, and stores them.  (In
// mrf_fwd_sweep every wavefront does all of that for all L labels, so that one barrier per node
// suffices; at L = 256 that is a third of its instructions.)  The price is a second barrier per
// node: the minimum over all labels (Eq. isgmr-norm) is the minimum of the wavefronts' home minima,
// exchanged through LDS.  Home labels sit in 32 consecutive lanes of one label slot (lane + 64 s),
// so loads and stores of a wavefront are 128-byte runs.
//   per node:  h(home) -> private LDS copy -> candidates of the 32 source labels for all lambda
//              -> partial (min, argmin) per lambda to LDS -> barrier -> merge at home, home minimum
//              -> LDS -> barrier -> global minimum, q, running message, stores
// Same arithmetic in the same order as mrf_fwd_sweep: results are bit-identical.
template <int LP, int RMAX, int D, bool TRWP>
__global__ void __launch_bounds__(64 * 2 * LP)
mrf_fwd_sweep_sliced(const MrfFwdParams P)
{
    constexpr int MCH = 32;
    constexpr int NWMAX = 2 * LP;
    constexpr int SLOTS = 64 * LP;
    __shared__ __align__(16) float hbuf_all[NWMAX][MCH];         // h of every wavefront's slice (read by its owner only)
    __shared__ float2 part[NWMAX][SLOTS];                        // partial (min, argmin) of wavefront w for label lambda
    __shared__ float2 hmin[NWMAX];                               // home minimum and its label, per wavefront
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    float *hbuf = hbuf_all[wv];

    const long long blk = blockIdx.x;
    const int ri = mrf_direction_of(P.blk_begin, P.r_count, blk);
    const int r = P.r_first + ri;
    const unsigned local = (unsigned)(blk - P.blk_begin[ri]);
    int b;
    unsigned t;
    mrf_geom_order(P.g.H, P.g.W, P.g.dh[r], P.g.dw[r], (unsigned)P.g.nscan[r], (unsigned)P.g.B, local, b, t);
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0, x0, len;
    mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
    const long long N = P.g.N;
    const long long head = ((long long)b * P.g.H + y0) * P.g.W + x0;
    const long long nstep = (long long)dh * P.g.W + dw;
    const float rho = P.rho[r];
    const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];

    // home label of this lane: lanes [32 (w & 1), +32) of the wavefront hold labels 32 w .. 32 w + 31
    const int mu0 = wv * MCH;
    const bool home_lane = (lane >> 5) == (wv & 1);
    const int hl = mu0 + (lane & 31);                 // home label (meaningful in home lanes)
    const bool home = home_lane && hl < L;
    const int hlc = home ? hl : 0;

    const float *src[RMAX];
    float use[RMAX], carry_at[RMAX + 1], is_rm[RMAX];
    const float vz = mrf_opaque_zero_f();
    src[0] = P.unary + (size_t)P.unary_slab[r] * N * L;
    use[0] = 1.0f;
    is_rm[0] = 0.0f;
#pragma unroll
    for (int c = 1; c < RMAX; ++c) {
        src[c] = (c <= n_src) ? P.m_in + (size_t)P.src_dir[r][c - 1] * N * L : src[0];
        use[c] = ((c <= n_src) ? 1.0f : 0.0f) + vz;
        is_rm[c] = ((c - 1 == rm_slot) ? 1.0f : 0.0f) + vz;
    }
#pragma unroll
    for (int c = 1; c <= RMAX; ++c) carry_at[c] = ((c == n_pre + 1) ? 1.0f : 0.0f) + vz;

    // rows mu0 .. mu0 + 31 of V, columns = the lane's destination labels
    float Vr[MCH][LP];
#pragma unroll
    for (int i = 0; i < MCH; ++i)
#pragma unroll
        for (int s = 0; s < LP; ++s) {
            const int mu = mu0 + i, lam = lane + 64 * s;
            Vr[i][s] = (mu < L && lam < L) ? P.V[(size_t)mu * L + lam] : 0.0f;
        }
    // entries of h past L never win a strict '<'; wavefronts that are absent (NW < NWMAX) neither
    if (lane < MCH) hbuf[lane] = INFINITY;
    for (int i = threadIdx.x; i < NWMAX * SLOTS; i += blockDim.x) (&part[0][0])[i] = make_float2(INFINITY, 0.0f);
    if (threadIdx.x < NWMAX) hmin[threadIdx.x] = make_float2(INFINITY, 0.0f);
    __syncthreads();

    // first node of the scanline: message 0, p = q = 0
    if (home) {
        P.m_out[((size_t)r * N + head) * L + hl] = 0.0f;
        P.p[((size_t)r * N + head) * L + hl] = 0;
    }
    if (threadIdx.x == 0) P.q[(size_t)r * N + head] = 0;

    const int vzero = mrf_opaque_zero();
    const float *wbase = P.w + (P.w_mul ? (size_t)r * N : 0);
    const int lastsrc = len - 2;
    float cur[D][RMAX], nxt[D][RMAX];
    float wcur[D], wnxt[D];
    auto prefetch = [&](float (&dst)[RMAX], float &wdst, int nj) {      // inputs of the update nj -> nj + 1
        nj = nj < lastsrc ? nj : lastsrc;
        const long long j = head + (long long)nj * nstep;
#pragma unroll
        for (int c = 0; c < RMAX; ++c) dst[c] = src[c][(size_t)j * L + hlc];
        wdst = wbase[(size_t)((j + nstep) * P.w_mul) + vzero];
    };
    if (len >= 2) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(cur[u], wcur[u], u);
    }

    float carry = 0.0f;        // normalised message of this direction at the previous node, home label

    for (int n0 = 1; n0 < len; n0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(nxt[u], wnxt[u], n0 - 1 + D + u);
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int nn = n0 + u;
            const bool past = nn >= len;
            const int n = past ? len - 1 : nn;
            const long long i = head + (long long)n * nstep;

            // ---- h at node i-r for the home labels (same order of additions as mrf_fwd_sweep) ----
            float v = cur[u][0];
            if (TRWP) {
                float mrm = 0.0f;
#pragma unroll
                for (int c = 1; c < RMAX; ++c) {
                    v = __builtin_fmaf(carry_at[c], carry, v);
                    v = __builtin_fmaf(use[c], cur[u][c], v);
                    mrm = __builtin_fmaf(is_rm[c], cur[u][c], mrm);
                }
                v = __builtin_fmaf(carry_at[RMAX], carry, v);
                v = rho * v;
                v = v - mrm;
            } else {
#pragma unroll
                for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(use[c], cur[u][c], v);
                v = v + carry;
            }
            const float wgt = wcur[u];
            if (home) hbuf[lane & 31] = v;
            mrf_wave_lds_fence();

            // ---- candidates of the 32 source labels of this wavefront, for every lambda ----
            float best[LP];
            int bidx[LP];
#pragma unroll
            for (int s = 0; s < LP; ++s) { best[s] = INFINITY; bidx[s] = 0; }
            // (all of the slice's h in one batch of LDS reads: the registers that the divided loads
            // freed pay for it, and the candidates then run without waiting for LDS)
            float hq[MCH];
#pragma unroll
            for (int i4 = 0; i4 < MCH; i4 += 4) {
                const float4 hv = *reinterpret_cast<const float4 *>(&hbuf[i4]);
                hq[i4] = hv.x; hq[i4 + 1] = hv.y; hq[i4 + 2] = hv.z; hq[i4 + 3] = hv.w;
            }
            mrf_static_for<MCH>([&](auto mm) {
                constexpr int m = decltype(mm)::value;
                float dlt[LP];
#pragma unroll
                for (int s = 0; s < LP; ++s) dlt[s] = __builtin_fmaf(wgt, Vr[m][s], hq[m]);
                mrf_argmin_step<m>(best, bidx, dlt);
            });
#pragma unroll
            for (int s = 0; s < LP; ++s)
                part[wv][lane + 64 * s] = make_float2(best[s], __int_as_float(mu0 + bidx[s]));
            mrf_block_sync_lds();

            // ---- merge at home, in ascending source label: the lowest index survives ----
            float tv = INFINITY;
            int tp = 0;
#pragma unroll
            for (int w2 = 0; w2 < NWMAX; ++w2) {
                const float2 e = part[w2][hlc];
                if (e.x < tv) { tv = e.x; tp = __float_as_int(e.y); }
            }
            if (!home) tv = INFINITY;
            // home minimum and the lowest home label that attains it
            const float lmin = mrf_wave_min(tv);
            const unsigned long long lbal = __ballot(tv == lmin);
            const int llab = mu0 + ((__ffsll((long long)lbal) - 1) & 31);
            if (lane == 0) hmin[wv] = make_float2(lmin, __int_as_float(llab));
            mrf_block_sync_lds();

            // ---- global minimum over the labels, q = lowest label attaining it (Eq. isgmr-norm) ----
            float tq = INFINITY;
            int qidx = 0;
#pragma unroll
            for (int w2 = 0; w2 < NWMAX; ++w2) {
                const float2 e = hmin[w2];
                if (e.x < tq) { tq = e.x; qidx = __float_as_int(e.y); }     // ascending wavefront = ascending label
            }
            carry = home ? tv - tq : 0.0f;

            if (!past) {
                if (home) {
                    P.m_out[((size_t)r * N + i) * L + hl] = carry;
                    P.p[((size_t)r * N + i) * L + hl] = (uint8_t)tp;
                }
                if (threadIdx.x == 0) P.q[(size_t)r * N + i] = (uint8_t)qidx;
            }
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            wcur[u] = wnxt[u];
#pragma unroll
            for (int c = 0; c < RMAX; ++c) cur[u][c] = nxt[u][c];
        }
    }
}

// ---- dense sweep for 33..128 labels: chunk minima, argmin by a second look ----------------------------
//
// The O(L^2) update with fewer instructions per candidate.  A running (minimum, argmin) costs four per candidate
// (fma, compare, minimum, select).  Here eight candidates form their minimum with three-operand minima and only that
// enters the running (minimum, chunk): 15 instructions for eight.  The index inside the winning chunk is found
// afterwards by evaluating its eight candidates once more for the label and comparing with the minimum (the same fma
// on the same operands gives the same bits); V for that comes from a transposed copy in LDS, h from the node's LDS row.
// Wavefront w owns the 32 destination labels 32 w .. 32 w + 31 (as in mrf_fwd_sweep_sliced: it loads, forms h,
// normalises and stores for them); its lower 32 lanes evaluate the first half of the source labels, its upper 32 lanes the
// second half, for the same destination labels, so no lane idles at 96 labels and the two halves meet by one lane
// swap; nothing is merged across wavefronts.  One barrier per node: after it every wavefront reads all of h.
// Where V is non-negative with a zero diagonal (looked at once per workgroup) and the weight is not negative, every
// candidate is >= its h and the one at the smallest h with lambda = mu equals it, so the minimum over lambda that
// Eq. isgmr-norm takes off is the minimum of h, which travels with h; otherwise a second barrier exchanges the minima of
// the new message.  q of a node is assembled behind the next barrier.
// Per node and wavefront at 96 labels about 240 instructions (mrf_fwd_sweep_sliced: 360, two barriers).
template <int NW>
__host__ __device__ constexpr int mrf_fwd_halves_lds() { return NW * 32 * (NW * 32 + 4) * (int)sizeof(float); }

template <int NW, int RMAX, int D, bool TRWP>
__global__ void __launch_bounds__(64 * NW) mrf_fwd_sweep_halves(const MrfFwdParams P)
{
    constexpr int LA = 32 * NW;                   // labels, rounded up
    constexpr int LH = LA / 2;                    // source labels per half
    constexpr int PT = LA + 4;                    // pitch of the transposed table (16-byte rows on different banks)
    constexpr int NCH = LH / 8;                   // chunks per half
    constexpr int none = 256;                     // above any label; as a byte 0, which p and q are where no candidate is below infinity
    extern __shared__ __align__(16) unsigned char mrf_smem[];
    float *vt = reinterpret_cast<float *>(mrf_smem);             // [LA][PT] V transposed: row lambda
    __shared__ __align__(16) float hrow[2][LA];                  // h of the node, by step parity
    __shared__ __align__(16) float hmin_w[2][4];                 // minimum of h per wavefront
    __shared__ __align__(16) float tmin_w[4];                    // minimum of the new message per wavefront (general case)
    __shared__ __align__(16) int q_w[2][4];                      // lowest label that attains the minimum, per wavefront
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int hf = lane >> 5;
    const int lam = 32 * wv + (lane & 31);
    const bool valid = lam < L;
    const int lamc = valid ? lam : 0;

    const long long blk = blockIdx.x;
    const int ri = mrf_direction_of(P.blk_begin, P.r_count, blk);
    const int r = P.r_first + ri;
    const unsigned local = (unsigned)(blk - P.blk_begin[ri]);
    int b;
    unsigned t;
    mrf_geom_order(P.g.H, P.g.W, P.g.dh[r], P.g.dw[r], (unsigned)P.g.nscan[r], (unsigned)P.g.B, local, b, t);
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0, x0, len;
    mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
    const long long N = P.g.N;
    const long long head = ((long long)b * P.g.H + y0) * P.g.W + x0;
    const long long nstep = (long long)dh * P.g.W + dw;
    const float rho = P.rho[r];
    const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];

    // Sources of h in summation order: the unary, then message arrays; unused slots load 0 and enter with factor 0
    // (fma(0, 0, v) = v and fma(1, x, v) = v + x exactly).  r^- once more by itself.  All of them through buffer views:
    // a lane's offset is its label, the node's is a scalar.
    const unsigned NLb = (unsigned)(N * L) * 4u, headb = (unsigned)(head * L) * 4u;
    const mrf_buf bu = mrf_buffer(P.unary + (size_t)__builtin_amdgcn_readfirstlane((int)P.unary_slab[r]) * N * L, NLb);
    const mrf_buf bm = mrf_buffer(P.m_in, (size_t)P.g.R * N * L * 4), bmo = mrf_buffer(P.m_out + (size_t)r * N * L, NLb);
    const mrf_buf bp = mrf_buffer(P.p + (size_t)r * N * L, (size_t)(N * L)), bq = mrf_buffer(P.q + (size_t)r * N, (size_t)N);
    const mrf_buf bw = mrf_buffer(P.w + (P.w_mul ? (size_t)r * N : 0), P.w_mul ? (size_t)N * 4 : 4);
    unsigned slab[RMAX], slab_rm = 0;
    float before[RMAX], after[RMAX];
    const float vz = mrf_opaque_zero_f();
    slab[0] = 0;
#pragma unroll
    for (int c = 1; c < RMAX; ++c) {
        // (uniform as it is; but with plain indices the compiler holds more scalars at once and spills some where there are sixteen arrays)
        slab[c] = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)P.src_dir[r][c <= n_src ? c - 1 : 0] * NLb));
        before[c] = ((c <= n_src && (!TRWP || c <= n_pre)) ? 1.0f : 0.0f) + vz;
        after[c] = ((c <= n_src && TRWP && c > n_pre) ? 1.0f : 0.0f) + vz;
    }
    if (TRWP && rm_slot >= 0) slab_rm = (unsigned)__builtin_amdgcn_readfirstlane((int)((unsigned)P.src_dir[r][rm_slot] * NLb));

    // V: the lane's column of its half's rows in registers, all of it transposed in LDS
    bool plain = true;                             // V >= 0 with a zero diagonal, as far as this lane looks
    float Vr[LH];
#pragma unroll
    for (int i = 0; i < LH; ++i) {
        const int mu = hf * LH + i;
        Vr[i] = (mu < L && valid) ? P.V[(size_t)mu * L + lam] : 0.0f;
        plain = plain && !(Vr[i] < 0.0f) && !(mu == lam && Vr[i] != 0.0f);
        vt[lam * PT + mu] = Vr[i];
    }
    if (threadIdx.x < 8) { (&hmin_w[0][0])[threadIdx.x] = INFINITY; (&q_w[0][0])[threadIdx.x] = none; }
    if (threadIdx.x < 4) tmin_w[threadIdx.x] = INFINITY;
    // sign bit set: some node step may not take the minimum of h for that of the new message
    const int slow = __syncthreads_and(plain ? 1 : 0) != 0 ? 0 : (int)0x80000000;

    const unsigned moff = valid && hf == 0 ? 4u * (unsigned)lam : MRF_BUF_NONE;      // the lower half stores m, the upper one p
    const unsigned poff = valid && hf == 1 ? (unsigned)lam : MRF_BUF_NONE;
    const unsigned qoff = wv == NW - 1 && lane == 0 ? 0u : MRF_BUF_NONE;
    auto store_f32 = [](mrf_buf bb, unsigned off, unsigned soff, float x) { __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), bb, off, soff, 0); };
    auto store_u8 = [](mrf_buf bb, unsigned off, unsigned soff, int x) { __builtin_amdgcn_raw_buffer_store_b8((unsigned char)x, bb, off, soff, 0); };
    // first node of the scanline: message 0, p = q = 0
    store_f32(bmo, moff, headb, 0.0f);
    store_u8(bp, poff, headb >> 2, 0);
    store_u8(bq, qoff, (unsigned)head, 0);
    if (len < 2) return;

    const unsigned lane4 = 4u * (unsigned)lamc;
    unsigned laneof[RMAX];
#pragma unroll
    for (int c = 0; c < RMAX; ++c) laneof[c] = c <= n_src ? lane4 : MRF_BUF_NONE;
    const unsigned laneof_rm = rm_slot >= 0 ? lane4 : MRF_BUF_NONE;
    const unsigned step_lb = (unsigned)((int)nstep * L) * 4u, step_n = (unsigned)(int)nstep;
    struct In {
        float v[RMAX];
        float rm, w;
    };
    In A[D], B[D];
    int pleft = len - 2;                           // the prefetch stays at the last source node, whose further copies are never used
    unsigned pb = headb, pw = (unsigned)head + step_n;
    auto prefetch = [&](In &in) {
        in.v[0] = mrf_buf_f32s(bu, lane4, pb);
#pragma unroll
        for (int c = 1; c < RMAX; ++c) in.v[c] = mrf_buf_f32s(bm, laneof[c], pb + slab[c]);
        in.rm = TRWP ? mrf_buf_f32s(bm, laneof_rm, pb + slab_rm) : 0.0f;
        in.w = mrf_buf_f32s(bw, 0, P.w_mul ? pw * 4u : 0u);
        if (pleft > 0) { pb += step_lb; pw += step_n; }
        --pleft;
    };

    float carry = 0.0f;
    unsigned ob = headb, on = (unsigned)head;      // the node before the one that is formed
    auto group = [&](const In (&in)[D], int n0) {
        float pre[D];
#pragma unroll
        for (int u = 0; u < D; ++u) {
            pre[u] = in[u].v[0];
#pragma unroll
            for (int c = 1; c < RMAX; ++c) pre[u] = __builtin_fmaf(before[c], in[u].v[c], pre[u]);
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int n = n0 + u;
            if (n >= len) break;                   // (uniform)
            const int par = n & 1;
            // ---- h at node i-r for the home labels, its minimum (entries past L hold +inf: they never win) ----
            float v = pre[u] + carry;
            if (TRWP) {
#pragma unroll
                for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(after[c], in[u].v[c], v);
                v = rho * v;
                v = v - in[u].rm;
            }
            v = valid ? v : INFINITY;
            hrow[par][lam] = v;
            hmin_w[par][wv] = mrf_wave_min(v);     // (every lane writes the same word)
            const float wgt = in[u].w;
            mrf_block_sync_lds();

            // all of the half's h and the minima in one batch of LDS reads
            const float *hh = &hrow[par][hf * LH];
            float hq[LH];
#pragma unroll
            for (int i = 0; i < LH; i += 4) {
                const float4 x = *reinterpret_cast<const float4 *>(&hh[i]);
                hq[i] = x.x; hq[i + 1] = x.y; hq[i + 2] = x.z; hq[i + 3] = x.w;
            }
            const float4 h4 = *reinterpret_cast<const float4 *>(&hmin_w[par][0]);
            const int4 qc = *reinterpret_cast<const int4 *>(&q_w[par ^ 1][0]);
            __builtin_amdgcn_sched_barrier(0);

            // ---- chunk minima over the half's source labels ----
            float best = INFINITY;
            int cid = 0;
            mrf_static_for<NCH>([&](auto cc) {
                constexpr int ch = decltype(cc)::value;
                float d[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) d[j] = __builtin_fmaf(wgt, Vr[8 * ch + j], hq[8 * ch + j]);
                // (a running minimum starts below NaN: eight of them in the first chunk must not hide the others)
                const float d67 = ch == 0 ? mrf_min3(d[6], d[7], INFINITY) : mrf_min(d[6], d[7]);
                const float m = mrf_min3(mrf_min3(d[0], d[1], d[2]), mrf_min3(d[3], d[4], d[5]), d67);
                if constexpr (ch == 0) {
                    best = m;
                } else {
                    cid = m < best ? ch : cid;
                    best = mrf_min(best, m);
                }
            });
            // the halves meet: source labels of the lower half come first, so they keep a tie
            const auto bx = __builtin_amdgcn_permlane32_swap(__float_as_uint(best), __float_as_uint(best), false, false);
            const auto cx = __builtin_amdgcn_permlane32_swap((unsigned)cid, (unsigned)cid, false, false);
            const float blo = __uint_as_float(bx[0]), bhi = __uint_as_float(bx[1]);
            const float tv = mrf_min(blo, bhi);
            const float tp = mrf_min3(blo, bhi, FLT_MAX);       // what p looks for: no candidate if none is finite
            const int mu0 = bhi < blo ? LH + 8 * (int)cx[1] : 8 * (int)cx[0];

            // ---- minimum over the labels (Eq. isgmr-norm) ----
            float tq = mrf_min(mrf_min(h4.x, h4.y), mrf_min(h4.z, h4.w));
            if (__builtin_expect((__builtin_amdgcn_readfirstlane(__float_as_int(wgt)) | slow) < 0, 0)) {
                tmin_w[wv] = mrf_wave_min(valid ? tv : INFINITY);
                mrf_block_sync_lds();
                const float4 t4 = *reinterpret_cast<const float4 *>(&tmin_w[0]);
                tq = mrf_min(mrf_min(t4.x, t4.y), mrf_min(t4.z, t4.w));
            }
            carry = tv - tq;
            const unsigned qb = (unsigned)__ballot((int)valid & (int)(tv == tq));
            q_w[par][wv] = qb != 0u ? 32 * wv + __ffs((int)qb) - 1 : none;

            // ---- p: the lowest source label of the winning chunk that attains the minimum, four per half ----
            const int m4 = mu0 + 4 * hf;
            const float4 va = *reinterpret_cast<const float4 *>(&vt[lam * PT + m4]), hv = *reinterpret_cast<const float4 *>(&hrow[par][m4]);
            int pf = none;
            pf = __builtin_fmaf(wgt, va.w, hv.w) == tp ? m4 + 3 : pf;
            pf = __builtin_fmaf(wgt, va.z, hv.z) == tp ? m4 + 2 : pf;
            pf = __builtin_fmaf(wgt, va.y, hv.y) == tp ? m4 + 1 : pf;
            pf = __builtin_fmaf(wgt, va.x, hv.x) == tp ? m4 : pf;
            const auto px = __builtin_amdgcn_permlane32_swap((unsigned)pf, (unsigned)pf, false, false);

            // q of the node before (for the second node: of the first, whose q is 0 again)
            store_u8(bq, qoff, on, n > 1 ? min(min(qc.x, qc.y), min(qc.z, qc.w)) : 0);
            ob += step_lb;
            on += step_n;
            store_f32(bmo, moff, ob, carry);
            store_u8(bp, poff, ob >> 2, (int)min(px[0], px[1]));
        }
    };
#pragma unroll
    for (int u = 0; u < D; ++u) prefetch(A[u]);
    // (dropped stores: what is in flight at the loop's entry then looks like what is in flight when it comes round)
#pragma unroll
    for (int u = 0; u < 3 * D; ++u) store_u8(bq, MRF_BUF_NONE, 0, 0);
    for (int n0 = 1; n0 < len; n0 += 2 * D) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(B[u]);
        __builtin_amdgcn_sched_barrier(0);
        group(A, n0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(A[u]);
        __builtin_amdgcn_sched_barrier(0);
        group(B, n0 + D);
        __builtin_amdgcn_sched_barrier(0);
    }
    mrf_block_sync_lds();
    const int4 qc = *reinterpret_cast<const int4 *>(&q_w[(len - 1) & 1][0]);
    store_u8(bq, qoff, on, min(min(qc.x, qc.y), min(qc.z, qc.w)));
}

// ---- sweep for pairwise potentials given per edge ---------------------------------------------
//
// theta_{i-r,i}(mu,lambda) read from a table of its own per edge, [R][N][L][L] with entry
// (r, i) the edge that arrives at node i (Eq. isgmr / Eq. trwp as written, before the
// decomposition into edge weight times V); for 33..64 labels.  One wavefront per scanline, lanes
// over lambda.  Row mu of a node's table is one coalesced load of L floats; the table is
// fetched in two halves of HALF = 20, 24, 28 or 32 rows into two register sets, each reloaded
// for the next node as soon as the current node is done with it, so that one half is always
// in flight behind the evaluation of the other.  h(mu) comes from the lane that owns mu
// (v_readlane with a constant lane).  The candidate is the plain sum h(mu) + theta(mu,lambda).
template <int HALF, int RMAX, bool TRWP>
__global__ void __launch_bounds__(64)
mrf_fwd_sweep_edge(const MrfFwdParams P)
{
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const bool valid = lane < L;
    const int lamc = valid ? lane : 0;

    const long long blk = blockIdx.x;
    const int ri = mrf_direction_of(P.blk_begin, P.r_count, blk);
    const int r = P.r_first + ri;
    const unsigned local = (unsigned)(blk - P.blk_begin[ri]);
    const unsigned nsc = (unsigned)P.g.nscan[r];
    const int b = (int)(local / nsc);
    const unsigned t = local - (unsigned)b * nsc;
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0, x0, len;
    mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
    const long long N = P.g.N;
    const long long head = ((long long)b * P.g.H + y0) * P.g.W + x0;
    const long long nstep = (long long)dh * P.g.W + dw;
    const float rho = P.rho[r];
    const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];

    // sources of h as in mrf_fwd_sweep: unused slots read the unary with factor 0
    const float *src[RMAX];
    float use[RMAX], carry_at[RMAX + 1], is_rm[RMAX];
    src[0] = P.unary + (size_t)P.unary_slab[r] * N * L;
    use[0] = 1.0f;
    is_rm[0] = 0.0f;
#pragma unroll
    for (int c = 1; c < RMAX; ++c) {
        src[c] = (c <= n_src) ? P.m_in + (size_t)P.src_dir[r][c - 1] * N * L : src[0];
        use[c] = (c <= n_src) ? 1.0f : 0.0f;
        is_rm[c] = (c - 1 == rm_slot) ? 1.0f : 0.0f;
    }
#pragma unroll
    for (int c = 1; c <= RMAX; ++c) carry_at[c] = (c == n_pre + 1) ? 1.0f : 0.0f;

    if (valid) {
        P.m_out[((size_t)r * N + head) * L + lane] = 0.0f;
        P.p[((size_t)r * N + head) * L + lane] = 0;
    }
    if (lane == 0) P.q[(size_t)r * N + head] = 0;
    if (len < 2) return;

    const int vzero = mrf_opaque_zero();
    const float *rbase = P.rho_e ? P.rho_e + (size_t)r * N : nullptr;
    const float *tbase = P.Te + (size_t)r * N * L * L;
    // rows mu0 .. mu0 + HALF - 1 of the table of the edge that arrives at node n of the scanline
    // (rows past L - 1 repeat the last row and are masked at use; a node past the end repeats the last)
    auto load_half = [&](float (&dst)[HALF], int n, int mu0) {
        n = n < len ? n : len - 1;
        const float *tb = tbase + (size_t)(head + (long long)n * nstep) * L * L + lamc;
#pragma unroll
        for (int m = 0; m < HALF; ++m) {
            const int mu = mu0 + m < L ? mu0 + m : L - 1;
            dst[m] = tb[(size_t)mu * L];
        }
    };
    float ta[HALF], tb2[HALF];
    float cur[RMAX], nxt[RMAX];
    float rcur = rho, rnxt = rho;
    auto prefetch = [&](float (&dst)[RMAX], float &rdst, int nj) {      // inputs of the update nj -> nj+1
        nj = nj < len - 2 ? nj : len - 2;
        const long long j = head + (long long)nj * nstep;
#pragma unroll
        for (int c = 0; c < RMAX; ++c) dst[c] = src[c][(size_t)j * L + lamc];
        rdst = rho;
        if (TRWP && rbase) rdst = rbase[(size_t)(j + nstep) + vzero];
    };
    prefetch(cur, rcur, 0);
    load_half(ta, 1, 0);
    load_half(tb2, 1, HALF);

    float carry = 0.0f;
    for (int n = 1; n < len; ++n) {
        prefetch(nxt, rnxt, n);
        const long long i = head + (long long)n * nstep;

        float v = cur[0];
        if (TRWP) {
            float mrm = 0.0f;
#pragma unroll
            for (int c = 1; c < RMAX; ++c) {
                v = __builtin_fmaf(carry_at[c], carry, v);
                v = __builtin_fmaf(use[c], cur[c], v);
                mrm = __builtin_fmaf(is_rm[c], cur[c], mrm);
            }
            v = __builtin_fmaf(carry_at[RMAX], carry, v);
            v = rcur * v;
            v = v - mrm;
        } else {
#pragma unroll
            for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(use[c], cur[c], v);
            v = v + carry;
        }

        // ascending mu with a strict '<': the lowest minimiser survives
        float best = INFINITY;
        int arg = 0;
#pragma unroll
        for (int m = 0; m < HALF; ++m) {
            const float hm = mrf_readlane_f32(v, m);
            const float dl = (m < L) ? hm + ta[m] : INFINITY;
            if (dl < best) { best = dl; arg = m; }
        }
        load_half(ta, n + 1, 0);
#pragma unroll
        for (int m = 0; m < HALF; ++m) {
            const float hm = mrf_readlane_f32(v, (HALF + m) & 63);
            const float dl = (HALF + m < L) ? hm + tb2[m] : INFINITY;
            if (dl < best) { best = dl; arg = HALF + m; }
        }
        load_half(tb2, n + 1, HALF);

        const float tv = valid ? best : INFINITY;
        const float tq = mrf_wave_min(tv);
        const unsigned long long bal = __ballot(tv == tq);
        const int qidx = __ffsll((long long)bal) - 1;
        carry = valid ? tv - tq : 0.0f;
        if (valid) {
            P.m_out[((size_t)r * N + i) * L + lane] = carry;
            P.p[((size_t)r * N + i) * L + lane] = (uint8_t)arg;
        }
        if (lane == 0) P.q[(size_t)r * N + i] = (uint8_t)qidx;

        rcur = rnxt;
#pragma unroll
        for (int c = 0; c < RMAX; ++c) cur[c] = nxt[c];
    }
}

// ---- the same for up to 32 labels ---------------------------------------------------------------
//
// Bound by the bytes of the tables (4 L^2 per node and direction) as long as enough of them are in flight: a launch has a
// wavefront per scanline only, so a wavefront has to keep several nodes' tables on the way, and the counter of loads in
// flight ends at 63.  A table is therefore loaded as it lies in memory, NT = 1..4 accesses of 16 bytes per lane (up to
// eight labels: one of 4), up to seven nodes ahead, and goes through a tile in LDS, from which its rows are read.  (A load
// per pair of rows, four nodes ahead, touches most cache lines twice: 155 us where this takes 131.)
// NG = 64 / SEG groups of SEG lanes (16 up to 16 labels, else 32) hold the same destination labels and group k the source
// labels k HR .. k HR + HR - 1, so no lane idles for want of labels.  Every group forms all of h (same loads, same
// operations) and keeps it in LDS; a lane reads its group's HR entries, finds their lowest argmin, and one or two lane swaps
// join the groups, the lower one first on a tie.  Entries without a source label are h = +inf.  Candidates that are NaN are
// passed over and a label without a finite candidate has p = 0, as in a running argmin that starts from infinity.
// 256 x 256, 21 labels, 4 directions, ISGMR sweep: 273 us with one label per lane and half a table in flight, now 131 (4.2 TB/s
// of tables and messages).
template <int SEG, int HR, int NT, int RMAX, bool TRWP>
__global__ void __launch_bounds__(64)
mrf_fwd_sweep_edge_groups(const MrfFwdParams P)
{
    constexpr int NG = 64 / SEG;
    constexpr int HP = (HR + 3) / 4 * 4;                // LDS row of a group, 16-byte aligned
    // nodes in flight: their loads, and the stores of the nodes between, within the counter's 63
    constexpr int NL = NT > 0 ? NT : 1, D0 = 1 + 63 / (NL + RMAX + 4), D = D0 > 7 ? 7 : D0;
    constexpr int TILE = NT > 0 ? 256 * NT : 64;         // floats
    static_assert(NG == 2 || NG == 4, "lane groups");
    __shared__ __align__(16) float tile[TILE + 256];     // (rows past L end within it: NG HR L <= TILE + 256)
    __shared__ __align__(16) float hrow[NG * HP + 4];       // (the last entry: for lanes without a label to scribble in)
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int lam = lane % SEG, grp = lane / SEG;
    const bool valid = lam < L;
    const unsigned lamc = valid ? (unsigned)lam : 0u;

    const long long blk = blockIdx.x;
    const int ri = mrf_direction_of(P.blk_begin, P.r_count, blk);
    const int r = P.r_first + ri;
    const unsigned local = (unsigned)(blk - P.blk_begin[ri]);
    const unsigned nsc = (unsigned)P.g.nscan[r];
    const int b = __builtin_amdgcn_readfirstlane((int)(local / nsc));
    const unsigned t = local - (unsigned)b * nsc;
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0, x0, len;
    mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
    y0 = __builtin_amdgcn_readfirstlane(y0);              // uniform, and known to be
    x0 = __builtin_amdgcn_readfirstlane(x0);
    len = __builtin_amdgcn_readfirstlane(len);
    const long long N = P.g.N;
    const long long head = ((long long)b * P.g.H + y0) * P.g.W + x0;
    const long long nstep = (long long)dh * P.g.W + dw;
    const float rho = P.rho[r];
    const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];

    // sources of h as in mrf_fwd_sweep: unused slots read the unary with factor 0
    const float *src[RMAX];
    float use[RMAX], carry_at[RMAX + 1], is_rm[RMAX];
    src[0] = P.unary + (size_t)P.unary_slab[r] * N * L;
    use[0] = 1.0f;
    is_rm[0] = 0.0f;
#pragma unroll
    for (int c = 1; c < RMAX; ++c) {
        src[c] = (c <= n_src) ? P.m_in + (size_t)P.src_dir[r][c - 1] * N * L : src[0];
        use[c] = (c <= n_src) ? 1.0f : 0.0f;
        is_rm[c] = (c - 1 == rm_slot) ? 1.0f : 0.0f;
    }
#pragma unroll
    for (int c = 1; c <= RMAX; ++c) carry_at[c] = (c == n_pre + 1) ? 1.0f : 0.0f;

    // Bases of the vectors of the node that is being loaded and of the one that is being stored walk along the scanline by
    // scalar additions.  A node's vectors are views of their own: lanes without a label, and the other groups', store
    // nothing, and behind the scanline's end the views are empty.
    const long long estep = nstep * L;
    const unsigned st4 = grp == 0 && valid ? (unsigned)lam << 2 : MRF_BUF_NONE, st1 = grp == 0 && valid ? (unsigned)lam : MRF_BUF_NONE;
    const unsigned stq = lane == 0 ? 0u : MRF_BUF_NONE;
    float *mo = P.m_out + ((size_t)r * N + head) * L;
    uint8_t *po = P.p + ((size_t)r * N + head) * L, *qo = P.q + (size_t)r * N + head;
    auto store = [&](bool act, float m, int arg, int q) {
        mrf_buf_store_f32(mrf_buffer(mo, act ? (size_t)L * 4 : 0), st4, m);
        mrf_buf_store_u8(mrf_buffer(po, act ? (size_t)L : 0), st1, arg);
        mrf_buf_store_u8(mrf_buffer(qo, act ? (size_t)L : 0), stq, q);       // (lane 0 stores, its first byte)
        mo += estep;
        po += estep;
        qo += nstep;
    };
    store(true, 0.0f, 0, 0);
    if (len < 2) return;

    for (int e = lane; e < NG * HP; e += 64) hrow[e] = INFINITY;       // entries without a source label stay +inf
    const int hslot = valid ? (lam / HR) * HP + lam % HR : NG * HP;
    mrf_wave_lds_fence();

    const int vzero = mrf_opaque_zero();
    // (without a rho per edge the load takes any word: no branch around a load that is prefetched)
    const bool per_edge = TRWP && P.rho_e;
    const float *rb = (per_edge ? P.rho_e + (size_t)r * N : P.unary) + head + nstep;
    const unsigned tsize = (unsigned)(L * L) * 4u;
    // a table as it lies in memory: sixteen bytes per lane and access (up to eight labels: four), the last ones those that
    // end the table; a lane without any keeps to a place of its own behind the tile
    unsigned toff[NL], tput[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        const unsigned at = NT > 0 ? 1024u * k + 16u * lane : 4u * lane;
        const bool live = at < tsize;
        toff[k] = live ? (NT > 0 && at + 16u > tsize ? tsize - 16u : at) : MRF_BUF_NONE;
        tput[k] = live ? toff[k] / 4u : (unsigned)(TILE + 4 * lane);
    }
    struct In {
        float f[NL][4], v[RMAX];
        float rho;
    };
    In in[D];
    // inputs of the update of node n: its edge's table, the vectors of node n - 1 (past the end: the last node again)
    const float *tb = P.Te + ((size_t)r * N + head + nstep) * L * L;
    const long long tstep = estep * L;
#pragma unroll
    for (int c = 0; c < RMAX; ++c) src[c] += (size_t)head * L;
    int ahead = 1;                                       // node that the next prefetch is for
    auto prefetch = [&](In &x) {
        const mrf_buf tv = mrf_buffer(tb, tsize);
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            if constexpr (NT > 0) mrf_buf_f32xn<4>(tv, toff[k], x.f[k]);
            else x.f[k][0] = mrf_buf_f32(tv, toff[k]);
        }
#pragma unroll
        for (int c = 0; c < RMAX; ++c) x.v[c] = src[c][lamc];
        x.rho = TRWP ? rb[vzero] : 1.0f;
        // (a mask instead of a choice, which would become a branch)
        const long long more = ++ahead < len ? -1LL : 0LL;
        const long long tinc = tstep & more, einc = estep & more;
        rb += nstep & more;
        tb += tinc;
#pragma unroll
        for (int c = 0; c < RMAX; ++c) src[c] += einc;
    };
#pragma unroll
    for (int u = 0; u < D; ++u) {
        prefetch(in[u]);
        // (dropped stores: what is in flight at the loop's entry then looks like what is when it comes round)
        for (int x = 0; x < 3; ++x) mrf_buf_store_u8(mrf_buffer(P.q, 1), MRF_BUF_NONE, 0);
        __builtin_amdgcn_sched_barrier(0);
    }

    // the tile holds the table of the node whose rows are read next
    float tr[HR];
    auto put = [&](const In &x) {
#pragma unroll
        for (int k = 0; k < NL; ++k)
#pragma unroll
            for (int c = 0; c < (NT > 0 ? 4 : 1); ++c) tile[tput[k] + c] = x.f[k][c];
    };
    const int trow = valid ? grp * HR * L + lam : 0;
    auto rows = [&]() {
#pragma unroll
        for (int m = 0; m < HR; ++m) tr[m] = tile[trow + m * L];      // (rows past L meet h = +inf)
    };
    for (int e = lane; e < TILE + 256; e += 64) tile[e] = 0.0f;
    mrf_wave_lds_fence();
    put(in[0]);
    mrf_wave_lds_fence();
    rows();
    mrf_wave_lds_fence();

    // lower group's (first) and upper group's value of what a lane holds, in both
    const auto pair = [&](unsigned x, auto upper) {
        if constexpr (decltype(upper)::value) return __builtin_amdgcn_permlane32_swap(x, x, false, false);
        else return __builtin_amdgcn_permlane16_swap(x, x, false, false);
    };
    const auto bits = [](float x) { return __builtin_bit_cast(unsigned, x); };
    const auto real = [](unsigned x) { return __builtin_bit_cast(float, x); };

    // What is left of a node once its message is known (indices and stores) runs in the next node's step, where that
    // waits for h to come back from LDS.
    float dP[HP], bestP = 0.0f, tvP = 0.0f, tqP = 0.0f;
    bool actP = false;
#pragma unroll
    for (int m = 0; m < HP; ++m) dP[m] = 0.0f;
    auto finish = [&]() {
        int arg = 0;
        const float least = mrf_min(bestP, FLT_MAX);                  // (nothing equals it where no candidate is finite)
        mrf_static_for<HP / 4>([&](auto g4) {
            constexpr int m0 = HP - 4 - 4 * decltype(g4)::value;      // from the top down: the lowest index lands last
            mrf_first_equal4<m0>(arg, least, dP[m0], dP[m0 + 1], dP[m0 + 2], dP[m0 + 3]);
        });
        arg += grp * HR;
        // join the groups: a strict '<' keeps the lower group's index on a tie
        float b = least;
        if constexpr (NG == 4) {
            const auto b2 = pair(bits(b), std::false_type{}), a2 = pair((unsigned)arg, std::false_type{});
            arg = real(b2[1]) < real(b2[0]) ? (int)a2[1] : (int)a2[0];
            b = mrf_min(real(b2[0]), real(b2[1]));
        }
        const auto b2 = pair(bits(b), std::true_type{}), a2 = pair((unsigned)arg, std::true_type{});
        arg = real(b2[1]) < real(b2[0]) ? (int)a2[1] : (int)a2[0];
        const unsigned long long bal = __ballot(tvP == tqP);
        store(actP, tvP - tqP, arg, __ffsll((long long)bal) - 1);
    };

    float carry = 0.0f;
    mo -= estep; po -= estep; qo -= nstep;               // (the first turn finishes no node)
    for (int n0 = 1; n0 < len; n0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            float v = in[u].v[0];
            if (TRWP) {
                float mrm = 0.0f;
#pragma unroll
                for (int c = 1; c < RMAX; ++c) {
                    v = __builtin_fmaf(carry_at[c], carry, v);
                    v = __builtin_fmaf(use[c], in[u].v[c], v);
                    mrm = __builtin_fmaf(is_rm[c], in[u].v[c], mrm);
                }
                v = __builtin_fmaf(carry_at[RMAX], carry, v);
                v = (per_edge ? in[u].rho : rho) * v;
                v = v - mrm;
            } else {
#pragma unroll
                for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(use[c], in[u].v[c], v);
                v = v + carry;
            }
            // (the groups write the same values to the same places)
            hrow[hslot] = v;
            mrf_wave_lds_fence();
            float4 hv[HP / 4];
#pragma unroll
            for (int k = 0; k < HP / 4; ++k) hv[k] = *reinterpret_cast<const float4 *>(&hrow[grp * HP + 4 * k]);
            mrf_wave_lds_fence();
            __builtin_amdgcn_sched_barrier(0);
            finish();
            put(in[(u + 1) % D]);
            mrf_wave_lds_fence();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < HP; ++m) {
                const float hm = m % 4 == 0 ? hv[m / 4].x : (m % 4 == 1 ? hv[m / 4].y : (m % 4 == 2 ? hv[m / 4].z : hv[m / 4].w));
                dP[m] = m < HR ? hm + tr[m < HR ? m : 0] : INFINITY;
            }
            rows();
            mrf_wave_lds_fence();
            bestP = mrf_min3(dP[0], dP[1], INFINITY);    // (+inf where every candidate is NaN)
#pragma unroll
            for (int m = 2; m + 1 < HP; m += 2) bestP = mrf_min3(bestP, dP[m], dP[m + 1]);
            float b = bestP;
            if constexpr (NG == 4) {
                const auto b2 = pair(bits(b), std::false_type{});
                b = mrf_min(real(b2[0]), real(b2[1]));
            }
            const auto b2 = pair(bits(b), std::true_type{});
            b = mrf_min(real(b2[0]), real(b2[1]));
            tvP = valid ? b : INFINITY;
            tqP = mrf_wave_min(tvP);                     // (every group holds every label)
            carry = tvP - tqP;
            actP = n0 + u < len;
            __builtin_amdgcn_sched_barrier(0);           // (a node's loads stay together: what is in flight is countable)
            prefetch(in[u]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    finish();
}

// ---- final costs and labels: c_i = theta_i + sum_r m^r_i (direction order), x_i = argmin ----
struct MrfAggParams {
    long long N;
    int L, R;
    int no_unary;        // Eq. isgmr-aggregation-old (standard SGM): c_i = sum_r m^r_i
    const float *unary, *m;
    float *cost;
    uint8_t *labels;     // may be NULL
};

// RT: bound on R (all loads of a node are issued before the first addition)
template <int RT>
__global__ void __launch_bounds__(256) mrf_aggregate(const MrfAggParams P)
{
    const int lane = threadIdx.x & 63;
    const long long wave = (long long)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const long long nwaves = (long long)gridDim.x * (blockDim.x >> 6);
    const int L = P.L;
    for (long long i = wave; i < P.N; i += nwaves) {
        float c[4];
        float mn = INFINITY;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int lam = lane + 64 * s;
            c[s] = INFINITY;
            if (lam < L) {
                float v = P.no_unary ? 0.0f : P.unary[(size_t)i * L + lam];
                float mv[RT];
#pragma unroll
                for (int d = 0; d < RT; ++d)
                    if (d < P.R) mv[d] = P.m[((size_t)d * P.N + i) * L + lam];
#pragma unroll
                for (int d = 0; d < RT; ++d)
                    if (d < P.R) v = v + mv[d];
                c[s] = v;
                P.cost[(size_t)i * L + lam] = v;
            }
            mn = fminf(mn, c[s]);
        }
        if (P.labels) {
            mn = mrf_wave_min(mn);
            int lab = -1;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const unsigned long long bal = __ballot(c[s] == mn);
                if (lab < 0 && bal != 0ull) lab = 64 * s + __ffsll((long long)bal) - 1;
            }
            if (lane == 0) P.labels[i] = (uint8_t)lab;
        }
    }
}

// ---- ISGMR with many directions: what iteration k left at a node, summed once per pair of directions ----
// Eq. isgmr's bracket holds, besides the running message, theta_i + sum over d not in {r, r-} of m^{d,k}_i:
// the same sum for r and for r-, and the same terms in the same order for every node that reads node i.
// One streaming pass per iteration forms it for every pair (2 R + 2 + R vectors moved per node instead of
// R (R - 1) read by the sweeps); the sweeps then read that one vector where they read the unary in the
// first iteration.  The additions are those of the sweeps, left to right in direction order.
struct MrfPresumParams {
    long long NL;            // entries per array
    int R;
    int opp[MRF_MAXR];       // opposite direction, or -1
    const float *unary;      // [N][L]
    const float *m;          // [R][N][L] messages of iteration k
    float *out;              // [R][N][L]: slab d is written for every d with no lower-indexed opposite
};

template <int RT, int VEC>
__global__ void __launch_bounds__(256) mrf_isgmr_presum(const MrfPresumParams P)
{
    typedef float vecf __attribute__((ext_vector_type(VEC)));
    const long long n = P.NL / VEC;
    for (long long e4 = (long long)blockIdx.x * blockDim.x + threadIdx.x; e4 < n; e4 += (long long)gridDim.x * blockDim.x) {
        const long long e = e4 * VEC;
        const vecf th = *reinterpret_cast<const vecf *>(P.unary + e);
        vecf mv[RT];
#pragma unroll
        for (int d = 0; d < RT; ++d)
            if (d < P.R) mv[d] = *reinterpret_cast<const vecf *>(P.m + (size_t)d * P.NL + e);
#pragma unroll
        for (int d = 0; d < RT; ++d) {
            if (d >= P.R) continue;
            const int od = P.opp[d];
            if (od >= 0 && od < d) continue;          // the pair was done at its lower index
            vecf a = th;
#pragma unroll
            for (int c = 0; c < RT; ++c)
                if (c < P.R && c != d && c != od) a = a + mv[c];
            *reinterpret_cast<vecf *>(P.out + (size_t)d * P.NL + e) = a;
        }
    }
}

// ---- fast path: V(mu, lambda) = f(|mu - lambda|) with f non-decreasing and constant (= fT)
// from distance TW on (truncated linear / quadratic models, Sec. 5.1) ------------------------
//
// With a non-negative edge weight every candidate inside the window |mu - lambda| < TW is
// <= g(mu) := fma(w, fT, h(mu)), and every candidate outside it equals g(mu).  Hence
//     min_mu Delta(lambda, mu) = min(W(lambda), gmin),   W = min over the window, gmin = min_mu g,
// and the lowest minimiser is  pW            if W <  gmin
//                              mu_g          if W >  gmin   (mu_g = lowest argmin of g; it is
//                                                            then provably outside the window)
//                              min(pW, mu_g) if W == gmin.
// Values and indices are bit-identical to the dense evaluation; the work per label drops
// from L to 2 TW - 1 candidates.  One wavefront walks one scanline: no workgroup barrier.
// A node with a negative weight falls back to the full loop over mu.
template <int LP, int RMAX, int D, bool TRWP, int TW>
__global__ void __launch_bounds__(64)
mrf_fwd_sweep_window(const MrfFwdParams P)
{
    constexpr int HB = 64 * LP + 2 * TW;          // h with TW entries of padding on both sides
    __shared__ float hpad[HB];
    __shared__ float ftab[TW + 1];
    const int L = P.g.L;
    const int lane = threadIdx.x;

    const long long blk = blockIdx.x;
    const int ri = mrf_direction_of(P.blk_begin, P.r_count, blk);
    const int r = P.r_first + ri;
    const unsigned local = (unsigned)(blk - P.blk_begin[ri]);
    const unsigned nsc = (unsigned)P.g.nscan[r];
    const int b = (int)(local / nsc);
    const unsigned t = local - (unsigned)b * nsc;
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0, x0, len;
    mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
    const long long N = P.g.N;
    const long long head = ((long long)b * P.g.H + y0) * P.g.W + x0;
    const long long nstep = (long long)dh * P.g.W + dw;
    const float rho = P.rho[r];
    const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];

    const float *src[RMAX];
    float use[RMAX], carry_at[RMAX + 1], is_rm[RMAX];
    const float vz = mrf_opaque_zero_f();     // keeps the flags below in vector registers
    src[0] = P.unary + (size_t)P.unary_slab[r] * N * L;
    use[0] = 1.0f;
    is_rm[0] = 0.0f;
#pragma unroll
    for (int c = 1; c < RMAX; ++c) {
        src[c] = (c <= n_src) ? P.m_in + (size_t)P.src_dir[r][c - 1] * N * L : src[0];
        use[c] = ((c <= n_src) ? 1.0f : 0.0f) + vz;
        is_rm[c] = ((c - 1 == rm_slot) ? 1.0f : 0.0f) + vz;
    }
#pragma unroll
    for (int c = 1; c <= RMAX; ++c) carry_at[c] = ((c == n_pre + 1) ? 1.0f : 0.0f) + vz;

    // f(d) = V(0, d) for d < TW, fT = V(0, L-1) (the promise makes every farther entry equal it)
    float f[TW];
#pragma unroll
    for (int d = 0; d < TW; ++d) f[d] = P.V[d < L ? d : L - 1] + vz;
    const float fT = P.V[L - 1] + vz;
    const bool f0zero = (P.V[0] == 0.0f);
    if (lane <= TW) ftab[lane] = lane < TW ? P.V[lane < L ? lane : L - 1] : fT;
    for (int i = lane; i < HB; i += 64) hpad[i] = INFINITY;     // padding never wins a strict '<'
    __syncthreads();
    float *hbuf = hpad + TW;

#pragma unroll
    for (int s = 0; s < LP; ++s) {
        const int lam = lane + 64 * s;
        if (lam < L) {
            P.m_out[((size_t)r * N + head) * L + lam] = 0.0f;
            P.p[((size_t)r * N + head) * L + lam] = 0;
        }
    }
    if (lane == 0) P.q[(size_t)r * N + head] = 0;

    const int vzero = mrf_opaque_zero();
    const float *wbase = P.w + (P.w_mul ? (size_t)r * N : 0);
    const int lastsrc = len - 2;
    float cur[D][RMAX][LP], nxt[D][RMAX][LP];
    float wcur[D], wnxt[D];
    float rcur[D], rnxt[D];                // rho of the edge (i-r, i): per edge if P.rho_e is given
    const float *rbase = P.rho_e ? P.rho_e + (size_t)r * N : nullptr;
    auto prefetch = [&](float (&dst)[RMAX][LP], float &wdst, float &rdst, int nj) {
        nj = nj < lastsrc ? nj : lastsrc;
        const long long j = head + (long long)nj * nstep;
#pragma unroll
        for (int c = 0; c < RMAX; ++c)
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const int lam = lane + 64 * s;
                dst[c][s] = src[c][(size_t)j * L + (lam < L ? lam : 0)];
            }
        wdst = wbase[(size_t)((j + nstep) * P.w_mul) + vzero];
        rdst = rho;
        if (TRWP && rbase) rdst = rbase[(size_t)(j + nstep) + vzero];
    };
    if (len >= 2) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(cur[u], wcur[u], rcur[u], u);
    }

    float carry[LP];
#pragma unroll
    for (int s = 0; s < LP; ++s) carry[s] = 0.0f;

    for (int n0 = 1; n0 < len; n0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(nxt[u], wnxt[u], rnxt[u], n0 - 1 + D + u);
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int nn = n0 + u;
            const bool past = nn >= len;
            const int n = past ? len - 1 : nn;
            const long long i = head + (long long)n * nstep;
            const float wgt = wcur[u];

            float a[LP], gfar[LP];
            float hm = INFINITY;
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                float v = cur[u][0][s];
                float mrm = 0.0f;
                if (TRWP) {
#pragma unroll
                    for (int c = 1; c < RMAX; ++c) {
                        v = __builtin_fmaf(carry_at[c], carry[s], v);
                        v = __builtin_fmaf(use[c], cur[u][c][s], v);
                        mrm = __builtin_fmaf(is_rm[c], cur[u][c][s], mrm);
                    }
                    v = __builtin_fmaf(carry_at[RMAX], carry[s], v);
                    v = rcur[u] * v;
                    v = v - mrm;
                } else {
#pragma unroll
                    for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(use[c], cur[u][c][s], v);
                    v = v + carry[s];
                }
                const int lam = lane + 64 * s;
                if (lam < L) hbuf[lam] = v;
                a[s] = lam < L ? v : INFINITY;
                gfar[s] = lam < L ? __builtin_fmaf(wgt, fT, v) : INFINITY;
                hm = mrf_min(hm, a[s]);
            }
            mrf_wave_lds_fence();

            float tv[LP];
            int tp[LP];
            int qidx = -1;
            float tq;
            // (the weight is wave-uniform: take the branch on a scalar copy of its sign)
            if (__builtin_expect(__builtin_amdgcn_readfirstlane(__float_as_int(wgt)) >= 0, 1)) {
                // One reduction serves the whole node.  g is a non-decreasing function of h, so
                // gmin = fma(w, fT, hmin).  If moreover f(0) = 0, every candidate is >= its h(mu)
                // >= hmin and the candidate (lambda = mu = argmin h) equals hmin, so the minimum
                // over lambda of the new message is hmin itself: q is the lowest label that
                // attains it and no second reduction is needed.
                const float hmin = mrf_wave_min(hm);
                const float gmin = __builtin_fmaf(wgt, fT, hmin);
                int mug = 0;
                bool found = false;
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const unsigned long long bal = __ballot(gfar[s] == gmin);
                    if (!found && bal != 0ull) { found = true; mug = 64 * s + __ffsll((long long)bal) - 1; }
                }
                // window |mu - lambda| < TW, ascending mu
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int lam = lane + 64 * s;
                    float dl[2 * TW - 1];
#pragma unroll
                    for (int o = 0; o < 2 * TW - 1; ++o) {
                        const int dist = o < TW - 1 ? TW - 1 - o : o - (TW - 1);
                        dl[o] = __builtin_fmaf(wgt, f[dist], hbuf[lam + o - (TW - 1)]);
                    }
                    float W = dl[0];
#pragma unroll
                    for (int o = 1; o + 1 < 2 * TW - 1; o += 2) W = mrf_min3(W, dl[o], dl[o + 1]);
                    int po = 2 * TW - 2;
#pragma unroll
                    for (int o = 2 * TW - 3; o >= 0; --o) po = (dl[o] == W) ? o : po;
                    const int pW = lam + po - (TW - 1);
                    const bool wlt = W < gmin, wgt_ = W > gmin;
                    tv[s] = (lam < L) ? (wlt ? W : gmin) : INFINITY;
                    const int tie = pW < mug ? pW : mug;
                    tp[s] = wlt ? pW : (wgt_ ? mug : tie);
                }
                if (__builtin_expect(f0zero, 1)) {
                    tq = hmin;
                } else {
                    float mn = INFINITY;
#pragma unroll
                    for (int s = 0; s < LP; ++s) mn = fminf(mn, tv[s]);
                    tq = mrf_wave_min(mn);
                }
            } else {
                // negative weight: the ordering argument does not hold, evaluate every mu
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int lam = lane + 64 * s;
                    float best = INFINITY;
                    int bi = 0;
                    for (int mu = 0; mu < L; ++mu) {
                        int dist = mu > lam ? mu - lam : lam - mu;
                        dist = dist < TW ? dist : TW;
                        const float dlt = __builtin_fmaf(wgt, ftab[dist], hbuf[mu]);
                        if (dlt < best) { best = dlt; bi = mu; }
                    }
                    tv[s] = (lam < L) ? best : INFINITY;
                    tp[s] = bi;
                }
                float mn = INFINITY;
#pragma unroll
                for (int s = 0; s < LP; ++s) mn = fminf(mn, tv[s]);
                tq = mrf_wave_min(mn);
            }
            mrf_wave_lds_fence();

            // q = lowest label attaining the minimum; reparametrisation (Eq. isgmr-norm)
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const unsigned long long bal = __ballot(tv[s] == tq);
                if (qidx < 0 && bal != 0ull) qidx = 64 * s + __ffsll((long long)bal) - 1;
            }
#pragma unroll
            for (int s = 0; s < LP; ++s) carry[s] = (lane + 64 * s < L) ? tv[s] - tq : 0.0f;

            if (!past) {
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int lam = lane + 64 * s;
                    if (lam < L) {
                        P.m_out[((size_t)r * N + i) * L + lam] = carry[s];
                        P.p[((size_t)r * N + i) * L + lam] = (uint8_t)tp[s];
                    }
                }
                if (lane == 0) P.q[(size_t)r * N + i] = (uint8_t)qidx;
            }
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            wcur[u] = wnxt[u];
            rcur[u] = rnxt[u];
#pragma unroll
            for (int c = 0; c < RMAX; ++c)
#pragma unroll
                for (int s = 0; s < LP; ++s) cur[u][c][s] = nxt[u][c][s];
        }
    }
}

// ---- window sweep with an index wavefront ----------------------------------------------------
//
// Same arithmetic as mrf_fwd_sweep_window, for launches with few scanlines.  Only the VALUES
// of the new message are on the node-to-node dependency chain; the argmin tables p and q and
// every store are not.  Two wavefronts share a scanline: the value wavefront forms h, its
// minimum and the new message and passes h, hmin and the weight through a ring in LDS; the
// index wavefronts follow a little behind, repeat the window evaluation with the index
// bookkeeping (Alg. 1/2: p, q) and store m, p and q.  Both sides evaluate the same
// expressions on the same h, so what is stored equals what the value wavefront carries.
// The index work of a node does not depend on other nodes, so NI index wavefronts take the
// nodes of a scanline in turn (it is somewhat more work per node than the value chain).
// Nobody meets at a barrier: the producer only waits when the ring is full, a consumer when
// its next node is not there yet, and every counter only grows, so all waits end.
//
// LOADER (TRWP with at most three other directions) adds a fourth kind of wavefront in front
// of the value wavefront.  It does the global loads and whatever of h does not need the
// running message: the partial sum theta + (messages of the directions before r), in the
// order Eq. trwp is summed, and the vector of r-.  It hands these, the later directions'
// messages and the weight over through a second ring; the value wavefront then touches LDS
// only, adds the running message and the later directions to the partial sum (same order,
// same roundings), and reads the next node's entries while it reduces the current one.
template <int LP, int RMAX, int D, bool TRWP, int TW, int NI, bool LOADER>
__global__ void __launch_bounds__(64 * ((LOADER ? 2 : 1) + NI))
mrf_fwd_sweep_window_duo(const MrfFwdParams P)
{
    static_assert(!LOADER || (TRWP && RMAX == 4), "loader wavefront: TRWP with up to three other directions");
    constexpr int NW0 = LOADER ? 2 : 1;           // wavefronts in front of the index wavefronts
    constexpr int NRL = 8;                        // slots of the loader's ring (a power of two, >= D)
    constexpr int LL = 64 * LP;
    constexpr int HB = 64 * LP + 2 * TW;          // h with TW entries of padding on both sides
    constexpr int NR = 8;                         // ring slots (a power of two, >= D)
    static_assert(NR >= D && (NR & (NR - 1)) == 0 && NI <= 4, "ring depth");
    constexpr int NT = 64 * (NW0 + NI);
    // One block with the h ring at LDS address 0: the value wavefront's fifteen neighbour reads per
    // label slot then fit the 8-bit offsets of ds_read2_b32 and need no address arithmetic.
    struct Shared {
        float ring[NR][HB];
        alignas(16) float2 ringwh[NR];            // weight and minimum of h (one write of the value wavefront: 256 x 512, 96 labels 2.56 -> 2.54 ms)
        float ftab[TW + 1];
        int produced;                             // last step published
        int loaded;                               // last step the loader has published
        MrfWaitBlock wait;                        // for the waits below (mrf_wait_turn)
        alignas(16) int consumed[4];              // per index wavefront: last step finished
        float lw[NRL];
        alignas(16) float lring[LOADER ? NRL : 1][5][LOADER ? LL : 1];   // partial sum, 3 messages, r- vector
    };
    __shared__ Shared sm;
    auto &ring = sm.ring;
    auto &ringwh = sm.ringwh;
    auto &ftab = sm.ftab;
    int &produced = sm.produced;
    int &loaded = sm.loaded;
    auto &consumed = sm.consumed;
    auto &lw = sm.lw;
    auto &lring = sm.lring;
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool index_wave = wave >= NW0;
    // the wavefronts on the node-to-node chain go first wherever they share a SIMD with the others
    if (!index_wave) __builtin_amdgcn_s_setprio(3);

    const long long blk = blockIdx.x;
    const int ri = mrf_direction_of(P.blk_begin, P.r_count, blk);
    const int r = P.r_first + ri;
    const unsigned local = (unsigned)(blk - P.blk_begin[ri]);
    int b;
    unsigned t;
    mrf_geom_order(P.g.H, P.g.W, P.g.dh[r], P.g.dw[r], (unsigned)P.g.nscan[r], (unsigned)P.g.B, local, b, t);
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0, x0, len;
    mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
    const long long N = P.g.N;
    const long long head = ((long long)b * P.g.H + y0) * P.g.W + x0;
    const long long nstep = (long long)dh * P.g.W + dw;
    const float vz = mrf_opaque_zero_f();     // keeps uniform constants in vector registers

    // f(d) = V(0, d) for d < TW, fT = V(0, L-1) (the promise makes every farther entry equal it)
    float f[TW];
#pragma unroll
    for (int d = 0; d < TW; ++d) f[d] = P.V[d < L ? d : L - 1] + vz;
    const float fT = P.V[L - 1] + vz;
    const bool f0zero = (P.V[0] == 0.0f);
    if ((int)threadIdx.x <= TW) ftab[threadIdx.x] = (int)threadIdx.x < TW ? P.V[(int)threadIdx.x < L ? threadIdx.x : L - 1] : fT;
    // padding and the entries of labels >= L are never written again: they never win a strict '<'
    for (int i = threadIdx.x; i < NR * HB; i += NT) (&ring[0][0])[i] = INFINITY;
    if (threadIdx.x == 0) { produced = 0; loaded = 0; mrf_wait_init(&sm.wait, P.fault, P.spin_limit); }
    const MrfWaitBlock *const wait_block = &sm.wait;
    // index wavefront j takes steps 1 + j, 1 + j + NI, ...; "finished" starts one turn before
    if (threadIdx.x < 4) consumed[threadIdx.x] = (int)threadIdx.x + 1 - NI;
    __syncthreads();

    if (index_wave) {
        // ---- p, q and all stores -----------------------------------------------------------
        const int jw = wave - NW0;
        if (jw == 0) {
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const int lam = lane + 64 * s;
                if (lam < L) {
                    P.m_out[((size_t)r * N + head) * L + lam] = 0.0f;
                    P.p[((size_t)r * N + head) * L + lam] = 0;
                }
            }
            if (lane == 0) P.q[(size_t)r * N + head] = 0;
        }

        // stores relative to the head of the scanline (the host has checked that a node step
        // times L fits 32 bits)
        float *const mrow = P.m_out + ((size_t)r * N + head) * L;
        uint8_t *const prow = P.p + ((size_t)r * N + head) * L;
        uint8_t *const qrow = P.q + (size_t)r * N + head;
        const int istep_l = (int)nstep * L;
        int seen = 0;
        for (int n = 1 + jw; n < len; n += NI) {
            int wait_turns = 0;
            while (seen < n) {
                seen = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(&produced, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                if (seen < n) mrf_wait_turn(wait_block, wait_turns);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            const int slot = n & (NR - 1);
            const float *hbuf = &ring[slot][TW];
            const float2 wh = ringwh[slot];
            const float wgt = wh.x, hmin = wh.y;
            const long long ol = (long long)n * istep_l;
            // the window's h in one batch of LDS reads behind the two words above (entries of labels
            // >= L and the padding hold +inf, so no lane needs a condition)
            float hv[LP][2 * TW - 1];
#pragma unroll
            for (int s = 0; s < LP; ++s)
#pragma unroll
                for (int o = 0; o < 2 * TW - 1; ++o) hv[s][o] = hbuf[lane + 64 * s + o - (TW - 1)];

            float tv[LP];
            int tp[LP];
            float tq;
            // The window evaluation runs for every node, so that the usual case is straight-line
            // code; for a negative weight its results are replaced below.
            {
                const float gmin = __builtin_fmaf(wgt, fT, hmin);
                int mug = 0;
                bool found = false;
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int lam = lane + 64 * s;
                    const float gfar = lam < L ? __builtin_fmaf(wgt, fT, hv[s][TW - 1]) : INFINITY;
                    const unsigned long long bal = __ballot(gfar == gmin);
                    if (!found && bal != 0ull) { found = true; mug = 64 * s + __ffsll((long long)bal) - 1; }
                }
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int lam = lane + 64 * s;
                    float dl[2 * TW - 1];
#pragma unroll
                    for (int o = 0; o < 2 * TW - 1; ++o) {
                        const int dist = o < TW - 1 ? TW - 1 - o : o - (TW - 1);
                        dl[o] = __builtin_fmaf(wgt, f[dist], hv[s][o]);
                    }
                    float W = dl[0];
#pragma unroll
                    for (int o = 1; o + 1 < 2 * TW - 1; o += 2) W = mrf_min3(W, dl[o], dl[o + 1]);
                    int po = 2 * TW - 2;
#pragma unroll
                    for (int o = 2 * TW - 3; o >= 0; --o) po = (dl[o] == W) ? o : po;
                    const int pW = lam + po - (TW - 1);
                    const bool wlt = W < gmin, wgt_ = W > gmin;
                    tv[s] = (lam < L) ? (wlt ? W : gmin) : INFINITY;
                    const int tie = pW < mug ? pW : mug;
                    tp[s] = wlt ? pW : (wgt_ ? mug : tie);
                }
                if (__builtin_expect(f0zero, 1)) {
                    tq = hmin;
                } else {
                    float mn = INFINITY;
#pragma unroll
                    for (int s = 0; s < LP; ++s) mn = fminf(mn, tv[s]);
                    tq = mrf_wave_min(mn);
                }
            }
            if (__builtin_expect(__builtin_amdgcn_readfirstlane(__float_as_int(wgt)) < 0, 0)) {
                // negative weight: the ordering argument does not hold, evaluate every mu
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int lam = lane + 64 * s;
                    float best = INFINITY;
                    int bi = 0;
                    for (int mu = 0; mu < L; ++mu) {
                        int dist = mu > lam ? mu - lam : lam - mu;
                        dist = dist < TW ? dist : TW;
                        const float dlt = __builtin_fmaf(wgt, ftab[dist], hbuf[mu]);
                        if (dlt < best) { best = dlt; bi = mu; }
                    }
                    tv[s] = (lam < L) ? best : INFINITY;
                    tp[s] = bi;
                }
                float mn = INFINITY;
#pragma unroll
                for (int s = 0; s < LP; ++s) mn = fminf(mn, tv[s]);
                tq = mrf_wave_min(mn);
            }
            // this slot has been read: hand it back
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            if (lane == 0) __hip_atomic_store(&consumed[jw], n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);

            int qidx = -1;
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const unsigned long long bal = __ballot(tv[s] == tq);
                if (qidx < 0 && bal != 0ull) qidx = 64 * s + __ffsll((long long)bal) - 1;
            }
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const int lam = lane + 64 * s;
                if (__builtin_expect(lam < L, 1)) {
                    mrow[ol + lam] = tv[s] - tq;
                    prow[ol + lam] = (uint8_t)tp[s];
                }
            }
            if (lane == 0) qrow[(long long)n * nstep] = (uint8_t)qidx;
        }
        return;
    }

    // ---- values: the dependency chain ------------------------------------------------------
    const float rho = P.rho[r];
    const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];
    const float *src[RMAX];
    float use[RMAX], carry_at[RMAX + 1], is_rm[RMAX];
    src[0] = P.unary + (size_t)P.unary_slab[r] * N * L;
    use[0] = 1.0f;
    is_rm[0] = 0.0f;
#pragma unroll
    for (int c = 1; c < RMAX; ++c) {
        src[c] = (c <= n_src) ? P.m_in + (size_t)P.src_dir[r][c - 1] * N * L : src[0];
        use[c] = ((c <= n_src) ? 1.0f : 0.0f) + vz;
        is_rm[c] = ((c - 1 == rm_slot) ? 1.0f : 0.0f) + vz;
    }
#pragma unroll
    for (int c = 1; c <= RMAX; ++c) carry_at[c] = ((c == n_pre + 1) ? 1.0f : 0.0f) + vz;

    const int vzero = mrf_opaque_zero();
    const float *wbase = P.w + (P.w_mul ? (size_t)r * N : 0);
    const int lastsrc = len - 2;
    // addresses relative to the head of the scanline: one 32 x 32 bit product per node (the
    // host has checked that a node step times L fits 32 bits)
    const int step_l = (int)nstep * L;
    const int step_w = (int)nstep * P.w_mul;
    const float *srcb[RMAX];
#pragma unroll
    for (int c = 0; c < RMAX; ++c) srcb[c] = src[c] + (size_t)head * L;
    const float *wb = wbase + (size_t)((head + nstep) * P.w_mul);
    float cur[D][RMAX][LP], nxt[D][RMAX][LP];
    float wcur[D], wnxt[D];
    auto prefetch = [&](float (&dst)[RMAX][LP], float &wdst, int nj) {
        nj = nj < lastsrc ? nj : lastsrc;
        const long long o = (long long)nj * step_l;
#pragma unroll
        for (int c = 0; c < RMAX; ++c)
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                const int lam = lane + 64 * s;
                dst[c][s] = srcb[c][o + (lam < L ? lam : 0)];
            }
        wdst = wb[(long long)nj * step_w + vzero];
    };
    if (LOADER && wave == 1) {
        // ---- loads and the part of h that does not wait for the running message -----------
        float before[RMAX];                   // sources summed before the running message
#pragma unroll
        for (int c = 1; c < RMAX; ++c) before[c] = ((c <= n_pre && c <= n_src) ? 1.0f : 0.0f) + vz;
        if (len >= 2) {
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(cur[u], wcur[u], u);
        }
        int pseen = 0;
        for (int n0 = 1; n0 < len; n0 += D) {
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(nxt[u], wnxt[u], n0 - 1 + D + u);
#pragma unroll
            for (int u = 0; u < D; ++u) {
                const int nn = n0 + u;
                if (nn < len) {
                    // both rings' slots were last used by step nn - NR: the value wavefront, which takes what it finds
                    // here, needs no wait of its own
                    static_assert(NR == NRL, "ring depths");
                    int wait_turns = 0;
                    while (pseen < nn - NR) {
                        int lo = __builtin_amdgcn_readfirstlane(
                            __hip_atomic_load(&consumed[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
#pragma unroll
                        for (int j = 1; j < NI; ++j) {
                            const int cj = __builtin_amdgcn_readfirstlane(
                                __hip_atomic_load(&consumed[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                            lo = cj < lo ? cj : lo;
                        }
                        pseen = lo + NI - 1;
                        if (pseen < nn - NR) mrf_wait_turn(wait_block, wait_turns);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                    const int ls = nn & (NRL - 1);
#pragma unroll
                    for (int s = 0; s < LP; ++s) {
                        float v = cur[u][0][s];
                        float mrm = 0.0f;
#pragma unroll
                        for (int c = 1; c < RMAX; ++c) {
                            v = __builtin_fmaf(before[c], cur[u][c][s], v);
                            mrm = __builtin_fmaf(is_rm[c], cur[u][c][s], mrm);
                            lring[ls][c][lane + 64 * s] = cur[u][c][s];
                        }
                        lring[ls][0][lane + 64 * s] = v;
                        lring[ls][4][lane + 64 * s] = mrm;
                    }
                    if (lane == 0) lw[ls] = wcur[u];
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                    __builtin_amdgcn_wave_barrier();
                    if (lane == 0) __hip_atomic_store(&loaded, nn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
#pragma unroll
            for (int u = 0; u < D; ++u) {
                wcur[u] = wnxt[u];
#pragma unroll
                for (int c = 0; c < RMAX; ++c)
#pragma unroll
                    for (int s = 0; s < LP; ++s) cur[u][c][s] = nxt[u][c][s];
            }
        }
        return;
    }

    float carry[LP];
#pragma unroll
    for (int s = 0; s < LP; ++s) carry[s] = 0.0f;
    int freed = 0;          // every step <= freed is finished (a possibly stale, hence conservative, view)

    if (LOADER) {
        // ---- values, fed by the loader -------------------------------------------------------
        // With two labels per lane a lane holds two ADJACENT labels: its h pair is one 8-byte LDS
        // write, the windows of both labels come out of the same 2 TW + 2 neighbours (TW 8-byte
        // reads instead of 4 TW - 2 single ones), and a ring entry of the loader is one 8-byte read
        // per vector.  The rings are indexed by label, so the other wavefronts keep their own mapping.
        constexpr bool PAIR = LP == 2 && (TW % 2) == 0;
        auto lab = [&](int s) { return PAIR ? 2 * lane + s : lane + 64 * s; };
        auto read_entry = [&](float (&dst)[5][LP], int ls) {
            if constexpr (PAIR) {
#pragma unroll
                for (int c = 0; c < 5; ++c) {
                    const float2 t = *reinterpret_cast<const float2 *>(&lring[ls][c][2 * lane]);
                    dst[c][0] = t.x;
                    dst[c][LP - 1] = t.y;
                }
            } else {
#pragma unroll
                for (int c = 0; c < 5; ++c)
#pragma unroll
                    for (int s = 0; s < LP; ++s) dst[c][s] = lring[ls][c][lane + 64 * s];
            }
        };
        float after[RMAX];                    // sources summed after the running message
#pragma unroll
        for (int c = 1; c < RMAX; ++c) after[c] = ((c > n_pre && c <= n_src) ? 1.0f : 0.0f) + vz;
        auto await_loader = [&](int nn) {
            int sn;
            int wait_turns = 0;
            do {
                sn = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(&loaded, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                if (sn < nn) mrf_wait_turn(wait_block, wait_turns);
            } while (sn < nn);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            return sn;
        };
        float in[5][LP], wgt = 0.0f;
        if (len >= 2) {
            await_loader(1);
            read_entry(in, 1);
            wgt = lw[1];
        }
        if (len < 2) return;
        for (int nn = 1;;) {
#pragma unroll
          for (int u = 1; u <= NR; ++u, ++nn) {   // (unrolled, so that ring addresses are constants)
            const int slot = u & (NR - 1);        // = nn % NR
            float *hbuf = &ring[slot][TW];

            float a[LP];
            float hm = 0.0f;
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                float v = in[0][s] + carry[s];
#pragma unroll
                for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(after[c], in[c][s], v);
                v = rho * v;
                v = v - in[4][s];
                const int lam = lab(s);
                // (lanes past L rewrite the +inf their ring entries hold anyway: no divergence; what
                // they carry from node to node is never looked at)
                a[s] = lam < L ? v : INFINITY;
                if (!PAIR) hbuf[lam] = a[s];
                hm = s == 0 ? a[s] : mrf_min(hm, a[s]);
            }
            if constexpr (PAIR) *reinterpret_cast<float2 *>(&hbuf[2 * lane]) = make_float2(a[0], a[LP - 1]);
            mrf_wave_lds_fence();
            float nb[LP][2 * TW - 1];
            if constexpr (PAIR) {
                // hn[k] = h(2 lane - TW + k), k = 0 .. 2 TW + 1; label 2 lane + s looks at hn[s + 1 ..]
                float hn[2 * TW + 2];
#pragma unroll
                for (int j = 0; j <= TW; ++j) {
                    if (j == TW / 2) {
                        hn[2 * j] = a[0];
                        hn[2 * j + 1] = a[LP - 1];
                    } else {
                        const float2 t = *reinterpret_cast<const float2 *>(&ring[slot][2 * lane + 2 * j]);
                        hn[2 * j] = t.x;
                        hn[2 * j + 1] = t.y;
                    }
                }
#pragma unroll
                for (int s = 0; s < LP; ++s)
#pragma unroll
                    for (int o = 0; o < 2 * TW - 1; ++o) nb[s][o] = hn[o + 1 + s];
            } else {
#pragma unroll
                for (int s = 0; s < LP; ++s)
#pragma unroll
                    for (int o = 0; o < 2 * TW - 1; ++o)
                        nb[s][o] = (o == TW - 1) ? a[s] : hbuf[lane + 64 * s + o - (TW - 1)];
            }
            // the next node's entries, in the same batch of LDS reads; if the loader's counter
            // (read first: the LDS queue keeps the order) does not cover them yet, they are read
            // again after waiting
            const int lsn = (u + 1) & (NRL - 1);
            const int flag = __hip_atomic_load(&loaded, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            float nin[5][LP];
            read_entry(nin, lsn);
            float nwgt = lw[lsn];
            __builtin_amdgcn_sched_barrier(0);    // (the reads are under way while the minimum is formed)
            const float hmin = mrf_wave_min(hm);
            __builtin_amdgcn_sched_barrier(0);
            // LDS executes a wavefront's operations in order: whoever sees the counter also sees the
            // node's ring entries written before it, so no wait is needed in between
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            // (every lane writes the same words: no divergent branch in the node step)
            ringwh[slot] = make_float2(wgt, hmin);
            __hip_atomic_store(&produced, nn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

            float tv[LP];
            float tq;
            // (evaluated for every node, so that the usual case is straight-line code; replaced
            // below for a negative weight)
            {
                const float gmin = __builtin_fmaf(wgt, fT, hmin);
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    // The two candidates at distance d share f(d), and a correctly rounded fma is
                    // non-decreasing in its addend: the smaller of the two comes from the smaller h.
                    float dl[TW];
                    dl[0] = __builtin_fmaf(wgt, f[0], nb[s][TW - 1]);
#pragma unroll
                    for (int d = 1; d < TW; ++d)
                        dl[d] = __builtin_fmaf(wgt, f[d], mrf_min(nb[s][TW - 1 - d], nb[s][TW - 1 + d]));
                    float W = mrf_min(dl[0], gmin);
#pragma unroll
                    for (int d = 1; d + 1 < TW; d += 2) W = mrf_min3(W, dl[d], dl[d + 1]);
                    if ((TW & 1) == 0) W = mrf_min(W, dl[TW - 1]);
                    tv[s] = W;
                }
                if (__builtin_expect(f0zero, 1)) {
                    tq = hmin;
                } else {
                    float mn = INFINITY;
#pragma unroll
                    for (int s = 0; s < LP; ++s) mn = fminf(mn, (lab(s) < L) ? tv[s] : INFINITY);
                    tq = mrf_wave_min(mn);
                }
            }
            if (__builtin_expect(__builtin_amdgcn_readfirstlane(__float_as_int(wgt)) < 0, 0)) {
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int lam = lab(s);
                    float best = INFINITY;
                    for (int mu = 0; mu < L; ++mu) {
                        int dist = mu > lam ? mu - lam : lam - mu;
                        dist = dist < TW ? dist : TW;
                        const float dlt = __builtin_fmaf(wgt, ftab[dist], hbuf[mu]);
                        if (dlt < best) best = dlt;
                    }
                    tv[s] = (lam < L) ? best : INFINITY;
                }
                float mn = INFINITY;
#pragma unroll
                for (int s = 0; s < LP; ++s) mn = fminf(mn, tv[s]);
                tq = mrf_wave_min(mn);
            }
            // the next node's entries were read above with the loader's counter in front of them;
            // looked at only now, so that everything before is one straight block
            if (__builtin_expect(nn + 1 >= len, 0)) return;            // (uniform)
            if (__builtin_expect(__builtin_amdgcn_readfirstlane(flag) < nn + 1, 0)) {
                await_loader(nn + 1);
                read_entry(nin, lsn);
                nwgt = lw[lsn];
            }
#pragma unroll
            for (int s = 0; s < LP; ++s) carry[s] = tv[s] - tq;
            wgt = nwgt;
#pragma unroll
            for (int c = 0; c < 5; ++c)
#pragma unroll
                for (int s = 0; s < LP; ++s) in[c][s] = nin[c][s];
          }
        }
    }

    if (len >= 2) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(cur[u], wcur[u], u);
    }

    for (int n0 = 1; n0 < len; n0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(nxt[u], wnxt[u], n0 - 1 + D + u);
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int nn = n0 + u;
            const bool past = nn >= len;
            const float wgt = wcur[u];
            const int slot = nn & (NR - 1);
            float *hbuf = &ring[slot][TW];

            // the slot was last used by step nn - NR (steps past the end publish nothing
            // and write nothing)
            int wait_turns = 0;
            while (__builtin_expect(!past && freed < nn - NR, 0)) {
                int lo = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(&consumed[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
#pragma unroll
                for (int j = 1; j < NI; ++j) {
                    const int cj = __builtin_amdgcn_readfirstlane(
                        __hip_atomic_load(&consumed[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                    lo = cj < lo ? cj : lo;
                }
                freed = lo + NI - 1;
                if (freed < nn - NR) mrf_wait_turn(wait_block, wait_turns);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");

            float a[LP];
            float hm = 0.0f;
#pragma unroll
            for (int s = 0; s < LP; ++s) {
                float v = cur[u][0][s];
                float mrm = 0.0f;
                if (TRWP) {
#pragma unroll
                    for (int c = 1; c < RMAX; ++c) {
                        v = __builtin_fmaf(carry_at[c], carry[s], v);
                        v = __builtin_fmaf(use[c], cur[u][c][s], v);
                        mrm = __builtin_fmaf(is_rm[c], cur[u][c][s], mrm);
                    }
                    v = __builtin_fmaf(carry_at[RMAX], carry[s], v);
                    v = rho * v;
                    v = v - mrm;
                } else {
#pragma unroll
                    for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(use[c], cur[u][c][s], v);
                    v = v + carry[s];
                }
                const int lam = lane + 64 * s;
                // (lanes past L rewrite the +inf their ring entries hold anyway: no divergence; what
                // they carry from node to node is never looked at)
                a[s] = lam < L ? v : INFINITY;
                if (!past) hbuf[lam] = a[s];
                hm = s == 0 ? a[s] : mrf_min(hm, a[s]);
            }
            // the neighbours' h for the window, requested before the reduction so that the LDS
            // latency passes behind it (the LDS queue keeps the order: writes above, then reads)
            mrf_wave_lds_fence();
            float nb[LP][2 * TW - 1];
#pragma unroll
            for (int s = 0; s < LP; ++s)
#pragma unroll
                for (int o = 0; o < 2 * TW - 1; ++o)
                    nb[s][o] = (o == TW - 1) ? a[s] : hbuf[lane + 64 * s + o - (TW - 1)];
            const float hmin = mrf_wave_min(hm);
            // LDS executes a wavefront's operations in order: whoever sees the counter also sees the
            // node's ring entries written before it, so no wait is needed in between
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            // (every lane writes the same words: no divergent branch in the node step)
            if (!past) {
                ringwh[slot] = make_float2(wgt, hmin);
                __hip_atomic_store(&produced, nn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

            // a past step re-reads the slot of an earlier step: its result is never used
            float tv[LP];
            float tq;
            // (evaluated for every node, so that the usual case is straight-line code; replaced
            // below for a negative weight)
            {
                const float gmin = __builtin_fmaf(wgt, fT, hmin);
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    // The two candidates at distance d share f(d), and a correctly rounded fma is
                    // non-decreasing in its addend: the smaller of the two comes from the smaller h.
                    float dl[TW];
                    dl[0] = __builtin_fmaf(wgt, f[0], nb[s][TW - 1]);
#pragma unroll
                    for (int d = 1; d < TW; ++d)
                        dl[d] = __builtin_fmaf(wgt, f[d], mrf_min(nb[s][TW - 1 - d], nb[s][TW - 1 + d]));
                    float W = mrf_min(dl[0], gmin);
#pragma unroll
                    for (int d = 1; d + 1 < TW; d += 2) W = mrf_min3(W, dl[d], dl[d + 1]);
                    if ((TW & 1) == 0) W = mrf_min(W, dl[TW - 1]);
                    tv[s] = W;
                }
                if (__builtin_expect(f0zero, 1)) {
                    tq = hmin;
                } else {
                    float mn = INFINITY;
#pragma unroll
                    for (int s = 0; s < LP; ++s) mn = fminf(mn, (lane + 64 * s < L) ? tv[s] : INFINITY);
                    tq = mrf_wave_min(mn);
                }
            }
            if (__builtin_expect(__builtin_amdgcn_readfirstlane(__float_as_int(wgt)) < 0, 0)) {
#pragma unroll
                for (int s = 0; s < LP; ++s) {
                    const int lam = lane + 64 * s;
                    float best = INFINITY;
                    for (int mu = 0; mu < L; ++mu) {
                        int dist = mu > lam ? mu - lam : lam - mu;
                        dist = dist < TW ? dist : TW;
                        const float dlt = __builtin_fmaf(wgt, ftab[dist], hbuf[mu]);
                        if (dlt < best) best = dlt;
                    }
                    tv[s] = (lam < L) ? best : INFINITY;
                }
                float mn = INFINITY;
#pragma unroll
                for (int s = 0; s < LP; ++s) mn = fminf(mn, tv[s]);
                tq = mrf_wave_min(mn);
            }
#pragma unroll
            for (int s = 0; s < LP; ++s) carry[s] = tv[s] - tq;
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            wcur[u] = wnxt[u];
#pragma unroll
            for (int c = 0; c < RMAX; ++c)
#pragma unroll
                for (int s = 0; s < LP; ++s) cur[u][c][s] = nxt[u][c][s];
        }
    }
}

// ---- window sweep, one label per lane, ceil(L/64) wavefronts per scanline ------------------
//
// Same arithmetic as mrf_fwd_sweep_window, laid out for launches with few scanlines (TRWP
// sweeps one direction at a time): a lone wavefront issues one instruction every four
// cycles, so the node step is spread over NWV wavefronts that each own 64 labels.  They
// meet once per node: every wavefront publishes its slice of h and its local minimum of h,
// then (after one LDS-only barrier) knows hmin, finds the lowest argmin of g by looking at
// all slices, evaluates its own windows and normalises by hmin without further exchange.
// q is assembled from per-wavefront candidates one node later, after the next barrier.
// Nodes where the single-reduction argument does not apply (negative weight, f(0) != 0)
// take a second barrier.
template <int RMAX, int D, bool TRWP, int TW>
__global__ void __launch_bounds__(256)
mrf_fwd_sweep_window_split(const MrfFwdParams P)
{
    constexpr int HB = 256 + 2 * TW;
    __shared__ float hpad[2][HB];
    __shared__ float ftab[TW + 1];
    __shared__ __align__(16) float hmslot[2][4];     // local minima of h
    __shared__ __align__(16) float tmslot[2][4];     // local minima of the new message (general path)
    __shared__ __align__(16) int qslot[2][4];        // local candidates for q
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // uniform, and known to be
    const int NWV = blockDim.x >> 6;
    const int lam = wv * 64 + lane;
    const bool valid = lam < L;
    const int lamc = valid ? lam : 0;

    const long long blk = blockIdx.x;
    const int ri = mrf_direction_of(P.blk_begin, P.r_count, blk);
    const int r = P.r_first + ri;
    const unsigned local = (unsigned)(blk - P.blk_begin[ri]);
    int b;
    unsigned t;
    mrf_geom_order(P.g.H, P.g.W, P.g.dh[r], P.g.dw[r], (unsigned)P.g.nscan[r], (unsigned)P.g.B, local, b, t);
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0, x0, len;
    mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
    const long long N = P.g.N;
    const long long head = ((long long)b * P.g.H + y0) * P.g.W + x0;
    const long long nstep = (long long)dh * P.g.W + dw;
    const float rho = P.rho[r];
    const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];

    const float *src[RMAX];
    float use[RMAX], carry_at[RMAX + 1], is_rm[RMAX];
    const float vz = mrf_opaque_zero_f();     // keeps the flags below in vector registers
    src[0] = P.unary + (size_t)P.unary_slab[r] * N * L;
    use[0] = 1.0f;
    is_rm[0] = 0.0f;
#pragma unroll
    for (int c = 1; c < RMAX; ++c) {
        src[c] = (c <= n_src) ? P.m_in + (size_t)P.src_dir[r][c - 1] * N * L : src[0];
        use[c] = ((c <= n_src) ? 1.0f : 0.0f) + vz;
        is_rm[c] = ((c - 1 == rm_slot) ? 1.0f : 0.0f) + vz;
    }
#pragma unroll
    for (int c = 1; c <= RMAX; ++c) carry_at[c] = ((c == n_pre + 1) ? 1.0f : 0.0f) + vz;

    float f[TW];
#pragma unroll
    for (int d = 0; d < TW; ++d) f[d] = P.V[d < L ? d : L - 1] + vz;
    const float fT = P.V[L - 1] + vz;
    const bool f0zero = (P.V[0] == 0.0f);
    if (threadIdx.x <= TW) ftab[threadIdx.x] = (int)threadIdx.x < TW ? P.V[(int)threadIdx.x < L ? threadIdx.x : L - 1] : fT;
    for (int i = threadIdx.x; i < 2 * HB; i += blockDim.x) (&hpad[0][0])[i] = INFINITY;
    if (threadIdx.x < 8) {
        (&hmslot[0][0])[threadIdx.x] = INFINITY;
        (&tmslot[0][0])[threadIdx.x] = INFINITY;
        (&qslot[0][0])[threadIdx.x] = -1;
    }
    __syncthreads();

    if (valid) {
        P.m_out[((size_t)r * N + head) * L + lam] = 0.0f;
        P.p[((size_t)r * N + head) * L + lam] = 0;
    }
    if (threadIdx.x == 0) P.q[(size_t)r * N + head] = 0;

    const int vzero = mrf_opaque_zero();
    const float *wbase = P.w + (P.w_mul ? (size_t)r * N : 0);
    const int lastsrc = len - 2;
    float cur[D][RMAX], nxt[D][RMAX];
    float wcur[D], wnxt[D];
    auto prefetch = [&](float (&dst)[RMAX], float &wdst, int nj) {
        nj = nj < lastsrc ? nj : lastsrc;
        const long long j = head + (long long)nj * nstep;
#pragma unroll
        for (int c = 0; c < RMAX; ++c) dst[c] = src[c][(size_t)j * L + lamc];
        wdst = wbase[(size_t)((j + nstep) * P.w_mul) + vzero];
    };
    if (len >= 2) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(cur[u], wcur[u], u);
    }

    float carry = 0.0f;
    int par = 0, qpar = 0;
    long long qnode = -1;      // node whose q is still to be stored (wavefront 0), candidates in qslot[qpar]

    for (int n0 = 1; n0 < len; n0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(nxt[u], wnxt[u], n0 - 1 + D + u);
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int nn = n0 + u;
            const bool past = nn >= len;
            const int n = past ? len - 1 : nn;
            const long long i = head + (long long)n * nstep;
            const float wgt = wcur[u];
            float *hb = &hpad[par][TW];

            float v = cur[u][0];
            if (TRWP) {
                float mrm = 0.0f;
#pragma unroll
                for (int c = 1; c < RMAX; ++c) {
                    v = __builtin_fmaf(carry_at[c], carry, v);
                    v = __builtin_fmaf(use[c], cur[u][c], v);
                    mrm = __builtin_fmaf(is_rm[c], cur[u][c], mrm);
                }
                v = __builtin_fmaf(carry_at[RMAX], carry, v);
                v = rho * v;
                v = v - mrm;
            } else {
#pragma unroll
                for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(use[c], cur[u][c], v);
                v = v + carry;
            }
            if (valid) hb[lam] = v;
            const float hloc = mrf_wave_min(valid ? v : INFINITY);
            if (lane == 0) hmslot[par][wv] = hloc;
            mrf_block_sync_lds();

            // q of the previous node: first wavefront that had a candidate
            if (wv == 0 && qnode >= 0) {
                const int4 qc = *reinterpret_cast<const int4 *>(&qslot[qpar][0]);
                const int qv = qc.x >= 0 ? qc.x : (qc.y >= 0 ? qc.y : (qc.z >= 0 ? qc.z : qc.w));
                if (lane == 0) P.q[(size_t)r * N + qnode] = (uint8_t)qv;
            }

            const float4 hm4 = *reinterpret_cast<const float4 *>(&hmslot[par][0]);
            const float hmin = fminf(fminf(hm4.x, hm4.y), fminf(hm4.z, hm4.w));
            const bool wpos = __builtin_amdgcn_readfirstlane(__float_as_int(wgt)) >= 0;
            float tv;
            int tp;
            if (wpos) {
                const float gmin = __builtin_fmaf(wgt, fT, hmin);
                // lowest argmin of g over all labels: look at every wavefront's slice of h
                int mug = 0;
                bool found = false;
#pragma unroll
                for (int w2 = 0; w2 < 4; ++w2) {
                    if (w2 < NWV) {
                        const float g2 = __builtin_fmaf(wgt, fT, hb[w2 * 64 + lane]);   // padding is +inf
                        const unsigned long long bal = __ballot(g2 == gmin);
                        if (!found && bal != 0ull) { found = true; mug = 64 * w2 + __ffsll((long long)bal) - 1; }
                    }
                }
                float dl[2 * TW - 1];
#pragma unroll
                for (int o = 0; o < 2 * TW - 1; ++o) {
                    const int dist = o < TW - 1 ? TW - 1 - o : o - (TW - 1);
                    dl[o] = __builtin_fmaf(wgt, f[dist], hb[lam + o - (TW - 1)]);
                }
                float W = dl[0];
#pragma unroll
                for (int o = 1; o + 1 < 2 * TW - 1; o += 2) W = mrf_min3(W, dl[o], dl[o + 1]);
                int po = 2 * TW - 2;
#pragma unroll
                for (int o = 2 * TW - 3; o >= 0; --o) po = (dl[o] == W) ? o : po;
                const int pW = lam + po - (TW - 1);
                const bool wlt = W < gmin, wgt_ = W > gmin;
                tv = valid ? (wlt ? W : gmin) : INFINITY;
                const int tie = pW < mug ? pW : mug;
                tp = wlt ? pW : (wgt_ ? mug : tie);
            } else {
                float best = INFINITY;
                int bi = 0;
                for (int mu = 0; mu < L; ++mu) {
                    int dist = mu > lam ? mu - lam : lam - mu;
                    dist = dist < TW ? dist : TW;
                    const float dlt = __builtin_fmaf(wgt, ftab[dist], hb[mu]);
                    if (dlt < best) { best = dlt; bi = mu; }
                }
                tv = valid ? best : INFINITY;
                tp = bi;
            }
            float tq = hmin;
            if (!(wpos && f0zero)) {
                // general case: the minimum of the new message needs its own exchange
                const float tloc = mrf_wave_min(tv);
                if (lane == 0) tmslot[par][wv] = tloc;
                mrf_block_sync_lds();
                const float4 t4 = *reinterpret_cast<const float4 *>(&tmslot[par][0]);
                tq = fminf(fminf(t4.x, t4.y), fminf(t4.z, t4.w));
            }
            const unsigned long long qb = __ballot(tv == tq);
            carry = valid ? tv - tq : 0.0f;

            // steps past the end of the scanline (last group only) leave no trace
            if (!past) {
                if (lane == 0) qslot[par][wv] = qb != 0ull ? wv * 64 + __ffsll((long long)qb) - 1 : -1;
                if (valid) {
                    P.m_out[((size_t)r * N + i) * L + lam] = carry;
                    P.p[((size_t)r * N + i) * L + lam] = (uint8_t)tp;
                }
                qnode = i;
                qpar = par;
            }
            par ^= 1;
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            wcur[u] = wnxt[u];
#pragma unroll
            for (int c = 0; c < RMAX; ++c) cur[u][c] = nxt[u][c];
        }
    }
    // q of the last node
    __syncthreads();
    if (wv == 0 && qnode >= 0) {
        const int4 qc = *reinterpret_cast<const int4 *>(&qslot[qpar][0]);
        const int qv = qc.x >= 0 ? qc.x : (qc.y >= 0 ? qc.y : (qc.z >= 0 ? qc.z : qc.w));
        if (lane == 0) P.q[(size_t)r * N + qnode] = (uint8_t)qv;
    }
}

// ---- window sweep: value wavefronts per 64 labels, a loader and index wavefronts ----------------------
//
// Both ideas above together, for launches of few scanlines: NWV = ceil(L/64) value wavefronts walk the scanline in lock step
// and compute the values of the new message only; of the NI wavefronts beside them the first does all loads and the part
// of h that does not wait for the running message, the others take the nodes in turn and do the argmin tables (all labels
// of a node) and the stores.  What bounds the sweep is the value wavefronts' node step, so
// - the window is shared among the lanes: the four lanes of a quad hold four neighbouring labels, each evaluates a quarter of
//   the distances for all four of them and two exchanges inside the quad leave every lane with its own label's minimum.  A
//   lane then reads 4 TW / 8 neighbours in wide reads instead of 2 TW - 2 single ones (31 reads of a node's 256 labels by
//   every value and index wavefront took a quarter of the node step in LDS bandwidth alone),
// - nothing waits for its own writes, and the wave-wide minimum of h runs while the neighbours are on their way,
// - value wavefronts meet twice without waiting twice: a flag says that a wavefront's h is in the ring (needed for the
//   neighbours), a post carries its minimum (needed behind the window).  The hardware barrier would also wait for the others.
//   Who looks too early looks again, a whole trip through LDS: the wavefronts are some tens of clocks apart, so flags and neighbours
//   are read half way through the minimum and not right behind the own h, and the posts half way through the window
//   (256 x 256, 256 labels, window 16, K = 10 5.48 -> 5.17 ms; window 8, K = 2 1.06 -> 1.00; 200 x 300, 128 labels, 8 directions, K = 2 1.46 ->
//   1.41).
// LDS executes a wavefront's operations in order, so whoever sees a flag, a post or a counter also sees what that wavefront
// wrote before it.  A value wavefront is at most one step ahead of the slowest, whose flag it needs: posts alternate between
// two sets.  The loader fills a slot of the h ring's step once the index wavefronts have left it (NR steps back) and its own
// once the value wavefronts have (NRL steps back); no wait can depend on itself.
// TRWP, 256 x 256, 256 labels, window 16, K = 10: sweeps 8.27 ms with index wavefronts alone beside the values and every neighbour
// read by itself, now 5.2; window 8, K = 2: 1.32 ms (mrf_fwd_sweep_window_duo), now 1.00.  What is left: a part of the step is the
// value wavefronts waiting for each other (K = 2, before the looks were moved: 1.16 ms, 0.93 without looking at flags and posts), the rest
// vector issue: 924 instructions of twelve wavefronts per node are 924 clocks of the four SIMDs.
// (four wavefronts per SIMD with four beside the values, so that two scanlines share a compute unit)
template <int RMAX, int D, bool TRWP, int TW, int NI>
__global__ void __launch_bounds__(64 * (4 + NI), NI <= 4 ? 4 : 3)
mrf_fwd_sweep_window_squad(const MrfFwdParams P)
{
    constexpr int PAD = TW < 4 ? 4 : TW;           // +inf beside the labels
    constexpr int HB = 256 + 2 * PAD;
    constexpr int NR = 8;                          // slots of the rings of h and of the new message
    constexpr int NRL = RMAX <= 4 ? 8 : 4;         // slots of the loader's ring
    constexpr int NX = NI - 1;                     // index wavefronts
    constexpr int NQ = TRWP ? RMAX / 4 : 0;        // TRWP: start term and what is added behind the running message, four by four
    static_assert(NX >= 1 && NX <= 7, "index wavefronts");
    __shared__ __align__(16) float hring[NR][HB];
    __shared__ __align__(16) float tring[NR][256];           // the new message before normalisation
    __shared__ __align__(16) float2 mring[NR];               // minimum of h, of the new message
    __shared__ __align__(16) float4 inq[NQ > 0 ? NQ : 1][NQ > 0 ? NRL : 1][256];
    __shared__ __align__(16) float inr[NRL][256];            // TRWP: message of r^-; ISGMR: start term
    __shared__ float lw[NR];                                 // edge weight
    __shared__ float ftab[TW + 1];
    __shared__ __align__(16) unsigned long long hmx[2][4];   // posts {step, minimum} per value wavefront: of h
    __shared__ __align__(16) unsigned long long tmx[2][4];   // of the new message (general path)
    __shared__ __align__(16) int hflag[4], valued[4], indexed[8];    // last step done, per wavefront
    __shared__ int loaded;
    __shared__ MrfWaitBlock wait_lds;              // for the waits below (mrf_wait_turn)
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int NWV = (int)(blockDim.x >> 6) - NI;   // value wavefronts come first

    const long long blk = blockIdx.x;
    const int ri = mrf_direction_of(P.blk_begin, P.r_count, blk);
    const int r = P.r_first + ri;
    const unsigned local = (unsigned)(blk - P.blk_begin[ri]);
    int b;
    unsigned t;
    mrf_geom_order(P.g.H, P.g.W, P.g.dh[r], P.g.dw[r], (unsigned)P.g.nscan[r], (unsigned)P.g.B, local, b, t);
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    int y0, x0, len;
    mrf_geom_head(P.g.H, P.g.W, dh, dw, t, y0, x0, len);
    len = __builtin_amdgcn_readfirstlane(len);               // uniform, and known to be
    const long long N = P.g.N;
    const long long head = ((long long)__builtin_amdgcn_readfirstlane(b) * P.g.H + __builtin_amdgcn_readfirstlane(y0)) * P.g.W +
                           __builtin_amdgcn_readfirstlane(x0);
    const long long nstep = (long long)dh * P.g.W + dw, estep = nstep * L;

    if ((int)threadIdx.x <= TW) ftab[threadIdx.x] = P.V[(int)threadIdx.x < TW && (int)threadIdx.x < L ? threadIdx.x : L - 1];
    // padding and the entries of labels >= L are never anything else: they never win a strict '<'
    for (int i = threadIdx.x; i < NR * HB; i += blockDim.x) (&hring[0][0])[i] = INFINITY;
    if (threadIdx.x < 8) {
        // wavefronts that are not there have always arrived, with nothing
        const bool here = (int)(threadIdx.x & 3) < NWV;
        const unsigned long long none = here ? 0ull : ((0x7fffffffull << 32) | 0x7f800000ull);
        (&hmx[0][0])[threadIdx.x] = none;
        (&tmx[0][0])[threadIdx.x] = none;
        if (threadIdx.x < 4) { hflag[threadIdx.x] = here ? 0 : 0x7fffffff; valued[threadIdx.x] = here ? 0 : 0x7fffffff; }
        indexed[threadIdx.x] = (int)threadIdx.x < NX ? (int)threadIdx.x + 1 - NX : 0x7fffffff;     // "finished" starts one turn before
    }
    if (threadIdx.x == 0) { loaded = 0; mrf_wait_init(&wait_lds, P.fault, P.spin_limit); }
    const MrfWaitBlock *const wait_block = &wait_lds;
    __syncthreads();
    const auto look = [](const int *counter) {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    };
    const auto look4 = [&](const int *counter) {             // the least of four
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int4 x = *reinterpret_cast<const int4 *>(counter);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        return __builtin_amdgcn_readfirstlane(min(min(x.x, x.y), min(x.z, x.w)));
    };
    const auto post = [](int *counter, int n) {              // (written by every lane: the same word, no exec-mask juggling)
        __hip_atomic_store(counter, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };

    if (wv < NWV) {
        // ---- values: wavefront wv owns labels 64 wv .. 64 wv + 63; step n forms the message of node n ----
        __builtin_amdgcn_s_setprio(3);             // they and the loader go first wherever they share a SIMD with others
        if (len < 2) return;
        constexpr int QD = TW >= 8 ? TW / 4 : 0;   // distances of a lane (TW < 8: all of its own label's)
        const int lam = 64 * wv + lane, quarter = lane & 3, quad = lam & ~3;
        const bool valid = lam < L;
        const float rho = P.rho[r], fT = ftab[TW];
        const bool f0zero = ftab[0] == 0.0f;
        float f[QD > 0 ? QD : TW];
#pragma unroll
        for (int e = 0; e < (QD > 0 ? QD : TW); ++e) f[e] = ftab[QD * quarter + e];
        // (written in place instead of as a function that is inlined, the node step gets two instructions more: 1.5 %)
        const auto run = [&]() {
            float4 q4[NQ > 0 ? NQ : 1];
            float dr, wgt;
            const auto fetch = [&](int ls, int slot) {
#pragma unroll
                for (int k = 0; k < NQ; ++k) q4[k] = inq[k][ls][lam];
                dr = inr[ls][lam];
                wgt = lw[slot];
            };
            const auto arrived = [&]() {
#pragma unroll
                for (int k = 0; k < NQ; ++k) asm volatile("" : : "v"(q4[k].x), "v"(q4[k].y), "v"(q4[k].z), "v"(q4[k].w));
                asm volatile("" : : "v"(dr), "v"(wgt));
            };
            const auto await = [&](int n) {
                int turns = 0;
                while (look(&loaded) < n) mrf_wait_turn(wait_block, turns);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            };
            // posts {step n, x} and returns the least of all wavefronts' x once all have posted step n
            const auto post_min = [&](unsigned long long (&box)[2][4], int n, float x) {
                __hip_atomic_store(&box[n & 1][wv], ((unsigned long long)(unsigned)n << 32) | (unsigned)__float_as_int(x),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            int4 e4[2];                                      // {minimum, step} of wavefronts 0, 1 and of 2, 3
            const auto read_posts = [&](unsigned long long (&box)[2][4], int n) {
#pragma unroll
                for (int k = 0; k < 2; ++k) e4[k] = *reinterpret_cast<const int4 *>(&box[n & 1][2 * k]);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            };
            const auto missing = [&](int n) {
                return __builtin_amdgcn_readfirstlane(min(min(e4[0].y, e4[0].w), min(e4[1].y, e4[1].w))) < n;
            };
            const auto least_post = [&](unsigned long long (&box)[2][4], int n) {
                if (__builtin_expect(missing(n), 0)) {
                    int looks = 0;
                    do {
                        // (the partners are a few instructions apart: look again at once, and at the clock now and then)
                        if ((++looks & 4095) == 0) mrf_wait_check(wait_block);
                        read_posts(box, n);
                    } while (missing(n));
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                return mrf_min(mrf_min(__int_as_float(e4[0].x), __int_as_float(e4[0].z)), mrf_min(__int_as_float(e4[1].x), __int_as_float(e4[1].z)));
            };
            await(1);
            fetch(0, 0);
            arrived();
            float carry = 0.0f;
            for (int n = 1;;) {
#pragma unroll
                for (int u = 0; u < NR; ++u, ++n) {          // step n uses slot u = (n - 1) % NR
                    float v;
                    if constexpr (TRWP) {
                        v = q4[0].x + carry;
#pragma unroll
                        for (int c = 1; c < RMAX; ++c) v = v + (c % 4 == 0 ? q4[c / 4].x : (c % 4 == 1 ? q4[c / 4].y : (c % 4 == 2 ? q4[c / 4].z : q4[c / 4].w)));
                        v = rho * v;
                        v = v - dr;
                    } else {
                        v = dr + carry;
                    }
                    const float w = wgt;
                    v = valid ? v : INFINITY;
                    hring[u][PAD + lam] = v;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    post(&hflag[wv], n);
                    mrf_wave_lds_fence();
                    // the loader's counter and the next node's values; then, in one batch, who has written h and the neighbours
                    float lo[QD > 0 ? QD + 4 : TW], hi[QD > 0 ? QD + 4 : TW];
                    int4 fl;
                    const auto neighbours = [&]() {
                        fl = *reinterpret_cast<const int4 *>(hflag);
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                        if constexpr (QD == 0) {
#pragma unroll
                            for (int d = 0; d < TW; ++d) { lo[d] = hring[u][PAD + lam - d]; hi[d] = hring[u][PAD + lam + d]; }
                        } else if constexpr (QD == 4) {
                            // label quad + s at distance 4 quarter + e: lo[s - e + 4], hi[s + e]
                            const float4 *pl = reinterpret_cast<const float4 *>(&hring[u][PAD + quad - 4 * quarter - 4]);
                            const float4 *ph = reinterpret_cast<const float4 *>(&hring[u][PAD + quad + 4 * quarter]);
#pragma unroll
                            for (int k = 0; k < 2; ++k) {
                                const float4 a = pl[k], c = ph[k];
                                lo[4 * k] = a.x; lo[4 * k + 1] = a.y; lo[4 * k + 2] = a.z; lo[4 * k + 3] = a.w;
                                hi[4 * k] = c.x; hi[4 * k + 1] = c.y; hi[4 * k + 2] = c.z; hi[4 * k + 3] = c.w;
                            }
                        } else {
                            static_assert(QD == 0 || QD == 2 || QD == 4, "window widths");
                            const float2 *pl = reinterpret_cast<const float2 *>(&hring[u][PAD + quad - 2 * quarter - 2]);
                            const float2 *ph = reinterpret_cast<const float2 *>(&hring[u][PAD + quad + 2 * quarter]);
#pragma unroll
                            for (int k = 0; k < 3; ++k) {
                                const float2 a = pl[k], c = ph[k];
                                lo[2 * k] = a.x; lo[2 * k + 1] = a.y;
                                hi[2 * k] = c.x; hi[2 * k + 1] = c.y;
                            }
                        }
                    };
                    const int seen = __hip_atomic_load(&loaded, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    fetch((u + 1) % NRL, (u + 1) % NR);
                    __builtin_amdgcn_sched_barrier(0);
                    float vm = v;
                    mrf_wave_min_first(vm);
                    __builtin_amdgcn_sched_barrier(0);
                    neighbours();
                    __builtin_amdgcn_sched_barrier(0);
                    float hmin = mrf_wave_min_rest(vm);
                    post_min(hmx, n, hmin);
                    __builtin_amdgcn_sched_barrier(0);
                    const auto absent = [&]() { return __builtin_amdgcn_readfirstlane(min(min(fl.x, fl.y), min(fl.z, fl.w))) < n; };
                    if (__builtin_expect(absent(), 0)) {
                        int looks = 0;
                        do {
                            if ((++looks & 4095) == 0) mrf_wait_check(wait_block);
                            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                            neighbours();
                        } while (absent());
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                    // window: the two candidates at a distance share f, and a correctly rounded fma is non-decreasing in its
                    // addend, so the smaller of the two comes from the smaller h
                    float W;
                    if constexpr (QD == 0) {
                        read_posts(hmx, n);
                        __builtin_amdgcn_sched_barrier(0);
                        W = __builtin_fmaf(w, f[0], v);
#pragma unroll
                        for (int d = 1; d < TW; ++d) W = mrf_min(W, __builtin_fmaf(w, f[d], mrf_min(lo[d], hi[d])));
                    } else {
                        float x[4];
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            if (s == 2) {
                                __builtin_amdgcn_sched_barrier(0);
                                read_posts(hmx, n);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                            float dl[QD];
#pragma unroll
                            for (int e = 0; e < QD; ++e) dl[e] = __builtin_fmaf(w, f[e], mrf_min(lo[s - e + QD], hi[s + e]));
                            x[s] = QD == 4 ? mrf_min(mrf_min3(dl[0], dl[1], dl[QD > 2 ? 2 : 0]), dl[QD - 1]) : mrf_min(dl[0], dl[1]);
                        }
                        // every lane keeps two of the four labels and gives two to the lane two further, then one of two
                        const bool up2 = quarter & 2, up1 = quarter & 1;
                        float give0 = up2 ? x[0] : x[2], give1 = up2 ? x[1] : x[3];
                        float keep0 = up2 ? x[2] : x[0], keep1 = up2 ? x[3] : x[1];
                        keep0 = mrf_min(keep0, mrf_dpp_f32<0x4E>(give0));
                        keep1 = mrf_min(keep1, mrf_dpp_f32<0x4E>(give1));
                        const float give = up1 ? keep0 : keep1, keep = up1 ? keep1 : keep0;
                        W = mrf_min(keep, mrf_dpp_f32<0xB1>(give));
                    }
                    hmin = least_post(hmx, n);
                    float tv = mrf_min(W, __builtin_fmaf(w, fT, hmin)), tq = hmin;
                    const bool wneg = __builtin_amdgcn_readfirstlane(__float_as_int(w)) < 0;
                    if (__builtin_expect(wneg, 0)) {
                        // negative weight: the ordering argument does not hold, evaluate every mu
                        float best = INFINITY;
                        for (int mu = 0; mu < L; ++mu) {
                            int dist = mu > lam ? mu - lam : lam - mu;
                            dist = dist < TW ? dist : TW;
                            const float dlt = __builtin_fmaf(w, ftab[dist], hring[u][PAD + mu]);
                            if (dlt < best) best = dlt;
                        }
                        tv = best;
                    }
                    if (__builtin_expect((int)wneg | (int)!f0zero, 0)) {
                        // the minimum of the new message is not that of h
                        tq = mrf_wave_min(valid ? tv : INFINITY);
                        post_min(tmx, n, tq);
                        read_posts(tmx, n);
                        tq = least_post(tmx, n);
                    }
                    carry = tv - tq;
                    arrived();                               // (in front of the writes below, behind which the wait would be for those)
                    tring[u][lam] = tv;
                    mring[u] = make_float2(hmin, tq);        // (every lane and value wavefront writes the same)
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    post(&valued[wv], n);
                    if (n + 1 >= len) return;                // (uniform)
                    if (__builtin_expect(__builtin_amdgcn_readfirstlane(seen) <= n, 0)) {
                        await(n + 1);
                        fetch((u + 1) % NRL, (u + 1) % NR);
                        arrived();
                    }
                }
            }
        };
        run();
        return;
    }

    if (wv == NWV) {
        // ---- loader ------------------------------------------------------------------------------------
        // NLL neighbouring labels per lane and access; the last lane's are the last ones of the node.  Sources of h in
        // summation order; unused slots are empty views (they load 0 and enter with factor 0).
        __builtin_amdgcn_s_setprio(3);
        if (len < 2) return;
        const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];
        const auto run = [&](auto labels) {
            constexpr int NLL = decltype(labels)::value, DL = NLL == 4 ? (D + 1) / 2 : D;      // (the registers of two sets)
            const bool live = NLL * lane < L;
            const int at = live ? (NLL * lane + NLL > L ? L - NLL : NLL * lane) : 0;
            // (views of one image: the host checks that their entries fit)
            const size_t image = (size_t)P.g.H * P.g.W, base = (size_t)__builtin_amdgcn_readfirstlane(b) * image;
            mrf_buf src[RMAX];
            float before[RMAX], after[RMAX], is_rm[RMAX];
            src[0] = mrf_buffer(P.unary + ((size_t)__builtin_amdgcn_readfirstlane((int)P.unary_slab[r]) * N + base) * L, image * L * 4);
#pragma unroll
            for (int c = 1; c < RMAX; ++c) {
                const bool there = c <= n_src;
                src[c] = mrf_buffer(P.m_in + ((size_t)__builtin_amdgcn_readfirstlane(there ? (int)P.src_dir[r][c - 1] : 0) * N + base) * L,
                                    (size_t)(unsigned)__builtin_amdgcn_readfirstlane(there ? 1 : 0) * image * L * 4);
                before[c] = there && (!TRWP || c <= n_pre) ? 1.0f : 0.0f;
                after[c] = there && TRWP && c > n_pre ? 1.0f : 0.0f;
                is_rm[c] = TRWP && c - 1 == rm_slot ? 1.0f : 0.0f;
            }
            const mrf_buf bw = mrf_buffer(P.w + (P.w_mul ? (size_t)r * N + base : 0), P.w_mul ? image * 4 : 4);
            const unsigned first = (unsigned)(head - (long long)base);
            unsigned at4 = live ? (first * (unsigned)L + (unsigned)at) * 4u : MRF_BUF_NONE, w4 = P.w_mul ? (first + (unsigned)(int)nstep) * 4u : 0u;
            const unsigned step4 = live ? (unsigned)(int)estep * 4u : 0u, wstep4 = P.w_mul ? (unsigned)(int)nstep * 4u : 0u;
            struct In {
                float v[RMAX][NLL];
                float w;
            };
            In A[DL], B[DL];
            // (what is loaded past the scanline's end is another node or 0, and never used)
            const auto prefetch = [&](In &in) {
#pragma unroll
                for (int c = 0; c < RMAX; ++c) mrf_buf_f32xn<NLL>(src[c], at4, in.v[c]);
                in.w = mrf_buf_f32(bw, w4);
                at4 += step4;
                w4 += wstep4;
            };
            int freed = 0, left = 0;                         // steps up to these have left the rings
            const auto group = [&](const In (&in)[DL], int n0) {
#pragma unroll
                for (int u = 0; u < DL; ++u) {
                    const int n = n0 + u;
                    float base[NLL], mrm[NLL];
#pragma unroll
                    for (int s = 0; s < NLL; ++s) {
                        base[s] = in[u].v[0][s];
                        mrm[s] = 0.0f;
#pragma unroll
                        for (int c = 1; c < RMAX; ++c) {
                            base[s] = __builtin_fmaf(before[c], in[u].v[c][s], base[s]);
                            if constexpr (TRWP) mrm[s] = __builtin_fmaf(is_rm[c], in[u].v[c][s], mrm[s]);
                        }
                    }
                    if (n >= len) break;                     // (uniform)
                    int turns = 0;
                    while (freed < n - NR) {
                        // the index wavefronts take the steps in turn: behind the slowest one's last step, the others have
                        // finished theirs
                        const int i0 = look4(&indexed[0]), i1 = look4(&indexed[4]);
                        freed = (i0 < i1 ? i0 : i1) + NX - 1;
                        if (freed < n - NR) mrf_wait_turn(wait_block, turns);
                    }
                    while (NRL < NR && left < n - NRL) {
                        left = look4(valued);
                        if (left < n - NRL) mrf_wait_turn(wait_block, turns);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                    const int ls = (n - 1) & (NRL - 1);
                    if (live) {
#pragma unroll
                        for (int s = 0; s < NLL; ++s) {
                            if constexpr (TRWP) {
#pragma unroll
                                for (int k = 0; k < NQ; ++k) {
                                    float a[4];
#pragma unroll
                                    for (int c = 0; c < 4; ++c) a[c] = 4 * k + c == 0 ? base[s] : after[4 * k + c > 0 ? 4 * k + c : 1] * in[u].v[4 * k + c][s];
                                    inq[k][ls][at + s] = make_float4(a[0], a[1], a[2], a[3]);
                                }
                                inr[ls][at + s] = mrm[s];
                            } else {
                                inr[ls][at + s] = base[s];
                            }
                        }
                    }
                    lw[(n - 1) & (NR - 1)] = in[u].w;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    post(&loaded, n);
                }
            };
#pragma unroll
            for (int u = 0; u < DL; ++u) prefetch(A[u]);
            for (int n0 = 1; n0 < len; n0 += 2 * DL) {
#pragma unroll
                for (int u = 0; u < DL; ++u) prefetch(B[u]);
                __builtin_amdgcn_sched_barrier(0);
                group(A, n0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < DL; ++u) prefetch(A[u]);
                __builtin_amdgcn_sched_barrier(0);
                group(B, n0 + DL);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (L <= 128) run(std::integral_constant<int, 2>{});
        else run(std::integral_constant<int, 4>{});
        return;
    }

    // ---- p, q and all stores: index wavefront jw takes steps 1 + jw, 1 + jw + NX, ... -----------------------
    // A lane holds two neighbouring labels, or two pairs 128 labels apart, one after the other.
    const int jw = wv - NWV - 1;
    constexpr int NB = 2 * PAD + 2;                          // neighbours of a pair: labels first - PAD ..
    const int pairs = L > 128 ? 2 : 1;
    const bool whole = L % 2 == 0;                           // a lane has both labels of a pair or none
    float f[TW];
#pragma unroll
    for (int d = 0; d < TW; ++d) f[d] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(ftab[d])));
    const float fT = ftab[TW];
    const auto store = [&](long long i, int pair, float m0, float m1, int p0, int p1) {
        const mrf_buf bm = mrf_buffer(P.m_out + ((size_t)r * N + i) * L, 4 * (size_t)L), bp = mrf_buffer(P.p + ((size_t)r * N + i) * L, (size_t)L);
        const unsigned at = 2u * (unsigned)lane + 128u * (unsigned)pair;      // (offsets of labels past L are past the views)
        if (whole) {
            const float m[2] = { m0, m1 };
            mrf_buf_store_f32xn<2>(bm, 4u * at, m);
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(p0 | p1 << 8), bp, at, 0, 0);
        } else {
            mrf_buf_store_f32(bm, 4u * at, m0);
            mrf_buf_store_f32(bm, 4u * at + 4u, m1);
            mrf_buf_store_u8(bp, at, p0);
            mrf_buf_store_u8(bp, at + 1u, p1);
        }
    };
    const auto store_q = [&](long long i, int q) {
        mrf_buf_store_u8(mrf_buffer(P.q + (size_t)r * N + i, 1), lane == 0 ? 0u : MRF_BUF_NONE, q);
    };
    // the lower of `found` and the lowest label of the pairs' lanes in b0 (their first labels) and b1
    const auto lowest = [&](int found, int pair, unsigned long long b0, unsigned long long b1) {
        const int l0 = (b0 | b1) != 0ull ? __ffsll((long long)(b0 | b1)) - 1 : 64;
        const int at = 128 * pair + 2 * l0 + (int)(1u - (unsigned)((b0 >> (l0 & 63)) & 1ull));
        return l0 < 64 && at < found ? at : found;
    };
    if (jw == 0) {
        for (int s = 0; s < pairs; ++s) store(head, s, 0.0f, 0.0f, 0, 0);
        store_q(head, 0);
    }
    int seen = 0;
    for (int n = 1 + jw; n < len; n += NX) {
        int turns = 0;
        while (seen < n) {
            seen = look4(valued);
            if (seen < n) mrf_wait_turn(wait_block, turns);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        const int slot = (n - 1) & (NR - 1);
        const long long i = head + (long long)n * nstep;
        const float wgt = lw[slot];
        const float2 mm = mring[slot];
        const float hmin = mm.x, tq = mm.y;
        // (a finite minimum of h makes every entry of the message finite)
        const bool positive = (int)(__builtin_amdgcn_readfirstlane(__float_as_int(wgt)) >= 0) &
                              (int)(((unsigned)__builtin_amdgcn_readfirstlane(__float_as_int(hmin)) & 0x7fffffffu) < 0x7f800000u);
        const float gmin = __builtin_fmaf(wgt, fT, hmin);
        // lowest label that attains the far minimum, and the lowest one that attains that of the message
        int mug = L, q = L;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (s >= pairs) break;                           // (uniform)
            const int lam = 2 * lane + 128 * s;
            const float2 h = *reinterpret_cast<const float2 *>(&hring[slot][PAD + lam]), t2 = *reinterpret_cast<const float2 *>(&tring[slot][lam]);
            const bool v0 = lam < L, v1 = lam + 1 < L;
            mug = lowest(mug, s, __ballot((int)v0 & (int)(__builtin_fmaf(wgt, fT, h.x) == gmin)), __ballot((int)v1 & (int)(__builtin_fmaf(wgt, fT, h.y) == gmin)));
            q = lowest(q, s, __ballot((int)v0 & (int)(t2.x == tq)), __ballot((int)v1 & (int)(t2.y == tq)));
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            if (s >= pairs) break;                           // (uniform)
            const int lam = 2 * lane + 128 * s;
            const float2 t2 = *reinterpret_cast<const float2 *>(&tring[slot][lam]);
            const float tv[2] = { t2.x, t2.y };
            int p[2];
            if (__builtin_expect(positive, 1)) {
                float nb[NB];
#pragma unroll
                for (int k = 0; k < NB / 2; ++k) {
                    const float2 x = reinterpret_cast<const float2 *>(&hring[slot][lam])[k];
                    nb[2 * k] = x.x; nb[2 * k + 1] = x.y;
                }
                if (s + 1 == pairs) {
                    // the slot has been read (what follows is in registers): hand it back
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                    post(&indexed[jw], n);
                }
#pragma unroll
                for (int o2 = 0; o2 < 2; ++o2) {
                    // lowest label of the window that attains the value, from the top down; the far minimiser if it does
                    constexpr int C = (2 * TW - 1 + 3) / 4 * 4;
                    float dl[C];
#pragma unroll
                    for (int o = 0; o < C; ++o) {
                        const int d = o < TW - 1 ? TW - 1 - o : o - (TW - 1);
                        dl[o] = o < 2 * TW - 1 ? __builtin_fmaf(wgt, f[d < TW ? d : 0], nb[PAD + o2 + (o < 2 * TW - 1 ? o : 0) - (TW - 1)]) : INFINITY;
                    }
                    int po = 2 * C;
                    mrf_static_for<C / 4>([&](auto g4) {
                        constexpr int o = C - 4 - 4 * decltype(g4)::value;
                        mrf_first_equal4<o>(po, tv[o2], dl[o], dl[o + 1], dl[o + 2], dl[o + 3]);
                    });
                    const int pw = po < 2 * C ? lam + o2 + po - (TW - 1) : L - 1, pg = tv[o2] == gmin ? mug : L - 1;
                    p[o2] = max(min(min(pw, pg), L - 1), 0);
                }
            } else {
                // negative weight, or no finite candidate (p = 0): every mu
#pragma unroll
                for (int o2 = 0; o2 < 2; ++o2) {
                    float best = INFINITY;
                    p[o2] = 0;
                    for (int mu = 0; mu < L; ++mu) {
                        int dist = mu > lam + o2 ? mu - (lam + o2) : lam + o2 - mu;
                        dist = dist < TW ? dist : TW;
                        const float dlt = __builtin_fmaf(wgt, ftab[dist], hring[slot][PAD + mu]);
                        if (dlt < best) { best = dlt; p[o2] = mu; }
                    }
                }
                if (s + 1 == pairs) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                    post(&indexed[jw], n);
                }
            }
            store(i, s, tv[0] - tq, tv[1] - tq, p[0], p[1]);
        }
        store_q(i, q < L ? q : 0);
    }
}

// ---- dense sweep for few labels: several scanlines per wavefront ----------------------------
//
// For L <= 32 a wavefront with one scanline leaves most lanes idle.  Here a wavefront is cut
// into 64/SEG segments of SEG lanes (SEG = 16 or 32 >= L); each segment walks its own
// scanline, possibly of another direction and length than its neighbours, so everything
// that is wave-uniform in the other kernels (node addresses, weight, source flags) is
// per-lane here.  V(.,lambda) sits in SEG registers per lane, h is exchanged through a
// per-segment LDS row, the minimum over labels is a DPP row reduction (plus one swizzle
// for 32-lane segments) and q comes from the segment's slice of a ballot.
__device__ inline float mrf_segment_min21(float v, int lane)
{
    const bool up = mrf_seg21_upper(lane);
    float u = up ? v : INFINITY, lo = up ? INFINITY : v;
    u = mrf_min(u, mrf_dpp_f32<0xB1>(u));
    lo = mrf_min(lo, mrf_dpp_f32<0xB1>(lo));
    u = mrf_min(u, mrf_dpp_f32<0x4E>(u));
    lo = mrf_min(lo, mrf_dpp_f32<0x4E>(lo));
    u = mrf_min(u, mrf_dpp_f32<0x141>(u));
    lo = mrf_min(lo, mrf_dpp_f32<0x141>(lo));
    u = mrf_min(u, mrf_dpp_f32<0x140>(u));
    lo = mrf_min(lo, mrf_dpp_f32<0x140>(lo));
    // rows 1..3: lane 15 of the row before (its upper minimum) joins this row's lower minimum
    const float pu = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        __builtin_bit_cast(int, INFINITY), __builtin_bit_cast(int, u), 0x142 /* row_bcast:15 */, 0xE, 0xF, false));
    const float full = mrf_min(lo, pu);            // the whole segment's minimum, in rows 1..3 (segment = row - 1)
    // upper lanes fetch it from the first lane of the next row; lower lanes hold it already
    const int from = up ? ((lane & 48) + 16) & 63 : lane;
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(from << 2, __builtin_bit_cast(int, full)));
}

template <int SEG>
__device__ inline float mrf_segment_min(float v)
{
    if (SEG == 21) return mrf_segment_min21(v, (int)(threadIdx.x & 63));
    v = mrf_min(v, mrf_dpp_f32<0xB1>(v));
    v = mrf_min(v, mrf_dpp_f32<0x4E>(v));
    v = mrf_min(v, mrf_dpp_f32<0x141>(v));
    v = mrf_min(v, mrf_dpp_f32<0x140>(v));
    if (SEG == 32)   // partner row inside the 32-lane group: swizzle, xor lane id with 16
        v = mrf_min(v, __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F)));
    return v;
}

// The same minimum for 32-lane segments without the trip through the LDS crossbar that the
// swizzle costs: five in-place DPP minima leave the minimum of lanes 0..31 in lane 31 and that of
// lanes 32..63 in lane 63; two v_readlane and a select hand them back.  For the value wavefront
// of latency-bound launches.  All 64 lanes must be active.
__device__ inline float mrf_segment_min32_regs(float v, int lane)
{
    float a, b;
    asm("s_nop 1\n\t"
        "v_min_f32_dpp %2, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_f32_dpp %2, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_f32_dpp %2, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_f32_dpp %2, %2, %2 row_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_f32_dpp %2, %2, %2 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_readlane_b32 %0, %2, 31\n\t"
        "v_readlane_b32 %1, %2, 63"
        : "=s"(a), "=s"(b), "+v"(v));
    return lane < 32 ? a : b;
}

// lowest lane of the caller's segment whose bit is set in a wavefront ballot, as a label
template <int SEG>
__device__ inline int mrf_segment_first(unsigned long long bal, int lane)
{
    if (SEG == 21) {
        const int sh = (lane / 21) * 21;
        return __ffs((int)((unsigned)(bal >> sh) & 0x1FFFFFu)) - 1;
    }
    const unsigned word = lane < 32 ? (unsigned)bal : (unsigned)(bal >> 32);
    const unsigned mine = SEG == 32 ? word : ((word >> (lane & 16)) & 0xFFFFu);
    return __ffs((int)mine) - 1;
}

// MU: source labels evaluated per node, L rounded up to a multiple of four (<= SEG, or 24 for the
// 21-lane segments, whose LDS rows are padded to 28 entries).
// IDX = 1, 2: that many further wavefronts per workgroup take the argmin tables and the stores (as in
// mrf_fwd_sweep_window_duo): the first computes values only and hands each node's h and
// weights over through a ring in LDS.  For launches that leave most issue slots idle, beyond the 32-bit offsets of
// the sweep divided among four wavefronts (below); two, because an index wavefront has more to do per node.
template <int SEG, int MU, int RMAX, int D, bool TRWP, int IDX>
__global__ void __launch_bounds__(64 * (1 + IDX))
mrf_fwd_sweep_packed(const MrfFwdParams P)
{
    static_assert(MU % 4 == 0 && (MU <= SEG || (SEG == 21 && MU == 24)), "source label count");
    constexpr int NSEG = 64 / SEG;                // (three segments of 21 lanes leave lane 63 idle)
    constexpr int NROW = SEG == 21 ? 4 : NSEG;    // LDS rows: the idle lane gets one of its own to scribble in
    constexpr int SEGP = SEG == 21 ? 28 : SEG + 4;   // row stride: 16-byte rows on different banks
    constexpr int NR = IDX ? 8 : 1;               // ring slots (IDX), else the one working row set
    static_assert(NR >= D || !IDX, "ring depth");
    __shared__ __align__(16) float hring[NR][NROW][SEGP];
    __shared__ float wring[NR][64];
    __shared__ int produced;
    __shared__ MrfWaitBlock wait_lds;             // for the waits below (mrf_wait_turn)
    __shared__ int consumed[2];                   // per index wavefront: last step finished
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool index_wave = IDX && wave > 0;
    if (IDX && !index_wave) __builtin_amdgcn_s_setprio(3);      // the value wavefront goes first on a shared SIMD
    const int seg = lane / SEG, lam = lane % SEG;
    const bool valid = lam < L;
    const int lamc = valid ? lam : 0;
    const long long N = P.g.N;
    const long long total = P.blk_begin[P.r_count];
    const long long sl = (long long)blockIdx.x * NSEG + seg;
    const bool act_seg = sl < total && seg < NSEG;

    // per-lane description of the segment's scanline
    int r = P.r_first, dh = 0, dw = 1, n_pre = 0, n_src = 0, rm_slot = -1;
    unsigned nsc = 1, local = 0;
    float rho = 1.0f;
    int sdir[RMAX];
#pragma unroll
    for (int c = 0; c < RMAX; ++c) sdir[c] = 0;
    for (int ri = 0; ri < P.r_count; ++ri) {
        const int rr = P.r_first + ri;
        const bool mine = act_seg && sl >= P.blk_begin[ri] && sl < P.blk_begin[ri + 1];
        if (mine) {
            r = rr; local = (unsigned)(sl - P.blk_begin[ri]); nsc = (unsigned)P.g.nscan[rr]; dh = P.g.dh[rr]; dw = P.g.dw[rr];
            rho = P.rho[rr]; n_pre = P.n_pre[rr]; n_src = P.n_src[rr]; rm_slot = P.rm_slot[rr];
#pragma unroll
            for (int c = 0; c + 1 < RMAX; ++c) sdir[c] = P.src_dir[rr][c];
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
    // Entry offsets walk along the scanline by additions: every lane has a scanline of its own, and a 64-bit
    // product per access and node costs four issue slots each.
    const long long stepL = nstep * L;
    const long long out0 = ((long long)r * N + head) * L + lam;      // entry of the first node in m_out / p
    const long long outq0 = (long long)r * N + head;                 // and in q

    const float *src[RMAX];
    float use[RMAX], carry_at[RMAX + 1], is_rm[RMAX];
    src[0] = P.unary + (size_t)P.unary_slab[r] * N * L;
    use[0] = 1.0f;
    is_rm[0] = 0.0f;
#pragma unroll
    for (int c = 1; c < RMAX; ++c) {
        src[c] = (c <= n_src) ? P.m_in + (size_t)sdir[c - 1] * N * L : src[0];
        use[c] = (c <= n_src) ? 1.0f : 0.0f;
        is_rm[c] = (c - 1 == rm_slot) ? 1.0f : 0.0f;
    }
#pragma unroll
    for (int c = 1; c <= RMAX; ++c) carry_at[c] = (c == n_pre + 1) ? 1.0f : 0.0f;

    float Vr[MU];
#pragma unroll
    for (int mu = 0; mu < MU; ++mu) Vr[mu] = (mu < L && valid) ? P.V[(size_t)mu * L + lam] : 0.0f;
    if (!index_wave) {
#pragma unroll
        for (int sl2 = 0; sl2 < NR; ++sl2) {
            hring[sl2][seg][lam] = INFINITY;      // entries mu >= L stay +inf: they never win
            if (lam < SEGP - SEG) hring[sl2][seg][SEG + lam] = INFINITY;
        }
        if (lane == 0) { produced = 0; consumed[0] = 1 - IDX; consumed[1] = 0; mrf_wait_init(&wait_lds, P.fault, P.spin_limit); }   // "finished" starts one turn before
    }
    const MrfWaitBlock *const wait_block = &wait_lds;
    __syncthreads();

    if ((!IDX || wave == 1) && act_seg && valid) {
        P.m_out[((size_t)r * N + head) * L + lam] = 0.0f;
        P.p[((size_t)r * N + head) * L + lam] = 0;
        if (lam == 0) P.q[(size_t)r * N + head] = 0;
    }

    // longest scanline of the wavefront bounds the loop
    int maxlen = 1;
#pragma unroll
    for (int sg = 0; sg < NSEG; ++sg) {
        const int l2 = __builtin_amdgcn_readlane(len, sg * SEG);
        maxlen = l2 > maxlen ? l2 : maxlen;
    }

    if (index_wave) {
        // ---- p, q and all stores, one node behind or more ----------------------------------
        // index wavefront jw takes steps 1 + jw, 1 + jw + IDX, ...
        const int jw = wave - 1;
        int seen = 0;
        long long io = out0 + (1 + jw) * stepL, iq = outq0 + (1 + jw) * nstep;
        const long long io_step = (IDX > 0 ? IDX : 1) * stepL, iq_step = (IDX > 0 ? IDX : 1) * nstep;
        for (int nn = 1 + jw; nn < maxlen; nn += (IDX > 0 ? IDX : 1), io += io_step, iq += iq_step) {
            int wait_turns = 0;
            while (seen < nn) {
                seen = __builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(&produced, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                if (seen < nn) mrf_wait_turn(wait_block, wait_turns);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
            const int slot = nn & (NR - 1);
            const bool act = act_seg && nn < len;
            const float wgt = wring[slot][lane];
            float dl[MU];
#pragma unroll
            for (int m4 = 0; m4 < MU; m4 += 4) {
                const float4 hv = *reinterpret_cast<const float4 *>(&hring[slot][seg][m4]);
                const float hq[4] = { hv.x, hv.y, hv.z, hv.w };
#pragma unroll
                for (int c = 0; c < 4; ++c) dl[m4 + c] = __builtin_fmaf(wgt, Vr[m4 + c], hq[c]);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            if (lane == 0) __hip_atomic_store(&consumed[jw], nn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            float best = mrf_min(dl[0], dl[1]);
#pragma unroll
            for (int m = 2; m + 1 < MU; m += 2) best = mrf_min3(best, dl[m], dl[m + 1]);
            int bidx = MU - 1;
            mrf_static_for<MU / 4>([&](auto g4) {
                constexpr int m0 = MU - 4 - 4 * decltype(g4)::value;      // groups from the top down
                mrf_first_equal4<m0>(bidx, best, dl[m0], dl[m0 + 1], dl[m0 + 2], dl[m0 + 3]);
            });
            const float tv = valid ? best : INFINITY;
            const float tq = mrf_segment_min<SEG>(tv);
            const int qidx = mrf_segment_first<SEG>(__ballot(tv == tq), lane);
            if (act && valid) {
                P.m_out[io] = tv - tq;
                P.p[io] = (uint8_t)bidx;
                if (lam == 0) P.q[iq] = (uint8_t)qidx;
            }
        }
        return;
    }

    const float *wbase = P.w + (P.w_mul ? (size_t)r * N : 0);
    const int lastsrc = len >= 2 ? len - 2 : 0;
    float cur[D][RMAX], nxt[D][RMAX];
    float wcur[D], wnxt[D];
    // source nodes 0, 1, 2, ... in the order of the calls; past the end: reload the last one, never used
    int pf_n = 0;
    long long pf_off = head * L + lamc;
    long long pf_w = (len >= 2 ? head + nstep : head) * P.w_mul;
    const long long stepW = nstep * P.w_mul;
    auto prefetch = [&](float (&dst)[RMAX], float &wdst) {
#pragma unroll
        for (int c = 0; c < RMAX; ++c) dst[c] = src[c][pf_off];
        wdst = wbase[pf_w];
        const bool more = pf_n < lastsrc;
        pf_off += more ? stepL : 0;
        pf_w += more ? stepW : 0;
        ++pf_n;
    };
#pragma unroll
    for (int u = 0; u < D; ++u) prefetch(cur[u], wcur[u]);
    long long so = out0 + stepL, sq = outq0 + nstep;        // entries of node 1, the first one updated

    float carry = 0.0f;
    int freed = 0;          // every step <= freed has been read by the index wavefront (possibly stale view)
    for (int n0 = 1; n0 < maxlen; n0 += D) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(nxt[u], wnxt[u]);
#pragma unroll
        for (int u = 0; u < D; ++u, so += stepL, sq += nstep) {
            const int nn = n0 + u;
            const bool act = act_seg && nn < len;       // this segment still has a node to update
            const float wgt = wcur[u];

            float v = cur[u][0];
            if (TRWP) {
                float mrm = 0.0f;
#pragma unroll
                for (int c = 1; c < RMAX; ++c) {
                    v = __builtin_fmaf(carry_at[c], carry, v);
                    v = __builtin_fmaf(use[c], cur[u][c], v);
                    mrm = __builtin_fmaf(is_rm[c], cur[u][c], mrm);
                }
                v = __builtin_fmaf(carry_at[RMAX], carry, v);
                v = rho * v;
                v = v - mrm;
            } else {
#pragma unroll
                for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(use[c], cur[u][c], v);
                v = v + carry;
            }
            const int slot = IDX ? (nn & (NR - 1)) : 0;
            if (IDX) {
                // the slot was last used by step nn - NR
                int wait_turns = 0;
                while (__builtin_expect(freed < nn - NR, 0)) {
                    // the index wavefronts take the steps in turn: behind the slowest one's last
                    // step, the others have finished theirs
                    int lo = __builtin_amdgcn_readfirstlane(
                        __hip_atomic_load(&consumed[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                    if (IDX > 1) {
                        const int c1 = __builtin_amdgcn_readfirstlane(
                            __hip_atomic_load(&consumed[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                        lo = c1 < lo ? c1 : lo;
                    }
                    freed = lo + IDX - 1;
                    if (freed < nn - NR) mrf_wait_turn(wait_block, wait_turns);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                }
                wring[slot][lane] = wgt;
            }
            // (lanes past L rewrite the +inf their entries hold anyway: no divergence; what they
            // carry from node to node is never looked at)
            hring[slot][seg][lam] = valid ? v : INFINITY;
            mrf_wave_lds_fence();

            // all candidates, their minimum with three-operand minima, then the lowest index
            // that attains it (scanning downwards, so the lowest survives)
            float dl[MU];
#pragma unroll
            for (int m4 = 0; m4 < MU; m4 += 4) {
                const float4 hv = *reinterpret_cast<const float4 *>(&hring[slot][seg][m4]);
                const float hq[4] = { hv.x, hv.y, hv.z, hv.w };
#pragma unroll
                for (int c = 0; c < 4; ++c) dl[m4 + c] = __builtin_fmaf(wgt, Vr[m4 + c], hq[c]);
            }
            if (IDX) {
                // (LDS keeps a wavefront's operations in order: the counter lands behind the entries)
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                if (lane == 0) __hip_atomic_store(&produced, nn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                mrf_wave_lds_fence();
            }
            float best = mrf_min(dl[0], dl[1]);
#pragma unroll
            for (int m = 2; m + 1 < MU; m += 2) best = mrf_min3(best, dl[m], dl[m + 1]);
            const float tv = valid ? best : INFINITY;
            const float tq = (IDX && SEG == 32) ? mrf_segment_min32_regs(tv, lane) : mrf_segment_min<SEG>(tv);
            carry = tv - tq;
            if (IDX) continue;                    // the index wavefront does the rest

            int bidx = MU - 1;
            mrf_static_for<MU / 4>([&](auto g4) {
                constexpr int m0 = MU - 4 - 4 * decltype(g4)::value;      // groups from the top down
                mrf_first_equal4<m0>(bidx, best, dl[m0], dl[m0 + 1], dl[m0 + 2], dl[m0 + 3]);
            });
            const int qidx = mrf_segment_first<SEG>(__ballot(tv == tq), lane);

            if (act && valid) {
                P.m_out[so] = carry;
                P.p[so] = (uint8_t)bidx;
                if (lam == 0) P.q[sq] = (uint8_t)qidx;
            }
        }
#pragma unroll
        for (int u = 0; u < D; ++u) {
            wcur[u] = wnxt[u];
#pragma unroll
            for (int c = 0; c < RMAX; ++c) cur[u][c] = nxt[u][c];
        }
    }
}

// ---- the packed sweep with its work divided among four wavefronts -------------------------------------
//
// For launches of few labels that do not fill the machine (thumbnails, crops, TRWP's one direction at a time), where the
// time of a sweep is the number of nodes on a scanline times the time of one node step on one wavefront.  A lone wavefront
// issues an instruction every four to five clocks, so what counts is how many instructions stand between two messages, and
// what it waits for:
//   loader   does all global loads, sums what does not depend on the running message, and hands a node over in a ring in LDS
//   values   h, its exchange through LDS, candidates, minimum, normalisation; h and the new message go to the ring
//   index    two of them, taking nodes in turn: the argmin tables (two levels as in mrf_fwd_sweep_narrow) and all stores
// The minimum over the labels of the new message is that of h where V >= 0 with a zero diagonal and the weight is finite and
// not negative (the candidate mu = lambda is h(lambda) itself and no other is smaller), so it is taken while h is on its way
// through LDS; other nodes take it from the message.  Candidates that are NaN are passed over and a label without a finite
// candidate has p = 0, as in a running argmin that starts from infinity.  One scanline per wavefront: NG = 64 / SEG groups of lanes hold the
// same labels and share the source labels (HR each), joined by lane swaps; NG = 1: 64 / SEG scanlines of one direction per
// wavefront, as many as fit.  Directions, factors, counts and base addresses are scalars, an entry is one 32-bit offset
// into buffer views (the host checks that N L fits).
// Every wait is on a counter in LDS that only grows: values on the loader, index on the values, the loader on the index
// wavefronts' step NR nodes back; none can depend on itself.
// A node step of the value wavefront takes 43 (16 labels, one scanline, ISGMR) to 81 instructions (21 labels, three, TRWP) of four to
// five clocks.  With a value wavefront that loads for itself and two index wavefronts, now: 32 x 48, 16 labels, ISGMR, K = 5, forward
// pass 75 -> 58 us; 37 x 53, 21 labels, TRWP, K = 5, 331 -> 254 us; 4 x 512 x 512, 21 labels, TRWP, K = 5, sweeps 4.17 -> 3.3 ms.
template <int SEG, int NG, int MU, int RMAX, bool TRWP>
__global__ void __launch_bounds__(256) mrf_fwd_sweep_packed(const MrfFwdParams P)
{
    constexpr int NSEG = NG > 1 ? 1 : 64 / SEG;   // scanlines per wavefront (three segments of 21 lanes leave lane 63 idle)
    constexpr int NROW = SEG == 21 ? 4 : NSEG;    // LDS rows of h: the idle lane gets one of its own to scribble in
    constexpr int HR = MU / NG;                   // source labels per group of lanes
    constexpr int HP = SEG == 21 ? 28 : SEG + 4;  // row stride: an entry per lane, 16-byte rows on different banks
    constexpr int NCH = HR / 4;                   // groups of four candidates
    constexpr int NR = 8;                         // ring slots
    constexpr int NI = 2;                         // index wavefronts
    constexpr int D = RMAX <= 4 ? 4 : (RMAX == 8 ? 2 : 1);
    constexpr int NQ = TRWP ? RMAX / 4 : 0;       // TRWP: start term and what is added behind the running message, four by four
    static_assert(HR % 4 == 0 && (NG == 1 || NG * SEG == 64), "lane groups");
    __shared__ __align__(16) float hring[NR][NROW][HP];
    __shared__ __align__(16) float4 inq[NQ > 0 ? NQ : 1][NQ > 0 ? NR : 1][64];
    __shared__ __align__(16) float2 ind[NR][64];  // TRWP: message of r^-, weight; ISGMR: start term, weight
    __shared__ float mring[NR][64];
    // Three scanlines per wavefront, which many wavefronts share a SIMD with: the minima of a lane's groups of four candidates
    // go to the index wavefronts as well.  (Else the value wavefront's step is what counts, and they form them again: 37 x 530
    // nodes, 21 labels, TRWP, two scanlines per wavefront 1.36 ms, with the minima handed over 1.48.)
    constexpr int NC = SEG == 21 ? (NCH + 3) / 4 : 0;
    __shared__ __align__(16) float4 cring[NC > 0 ? NC : 1][NC > 0 ? NR : 1][64];     // minima of a lane's groups of four candidates
    __shared__ __align__(16) float vt[SEG][MU + 4];   // V transposed: row lambda
    __shared__ MrfWaitBlock wait_lds;             // for the waits below (mrf_wait_turn)
    __shared__ int loaded, valued, indexed[NI];   // last step finished
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int grp = NG > 1 ? lane / SEG : 0, seg = NG > 1 ? 0 : lane / SEG, lam = lane % SEG;
    const bool valid = lam < L;
    const int lamc = valid ? lam : 0;

    // this wavefront's scanlines: NSEG consecutive ones of direction r
    const int blk = (int)blockIdx.x;
    int ri = 0;
    while (ri + 1 < P.r_count && blk >= P.pack_begin[ri + 1]) ++ri;
    const int r = P.r_first + ri;
    const unsigned nsc = (unsigned)P.g.nscan[r];
    const unsigned sl = (unsigned)(blk - P.pack_begin[ri]) * NSEG + seg;
    const bool act_seg = seg < NSEG && sl < (unsigned)P.g.B * nsc;
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    const int nstep = dh * P.g.W + dw;
    int y0 = 0, x0 = 0, len = 0, head = 0;
    if (act_seg) {
        const int b = sl < nsc ? 0 : (int)(sl / nsc);
        mrf_geom_head(P.g.H, P.g.W, dh, dw, sl - (unsigned)b * nsc, y0, x0, len);
        head = (b * P.g.H + y0) * P.g.W + x0;
    }
    // longest scanline of the wavefront bounds the loops
    int maxlen = 0;
#pragma unroll
    for (int sg = 0; sg < NSEG; ++sg) {
        const int l2 = __builtin_amdgcn_readlane(len, sg * SEG);
        maxlen = l2 > maxlen ? l2 : maxlen;
    }
    const size_t N = (size_t)P.g.N, NL = N * L;
    const unsigned estep = (unsigned)nstep * (unsigned)L;

    if (threadIdx.x == 0) {
        loaded = 0; valued = 0;
        for (int j = 0; j < NI; ++j) indexed[j] = j + 1 - NI;      // "finished" starts one turn before
        mrf_wait_init(&wait_lds, P.fault, P.spin_limit);
    }
    const MrfWaitBlock *const wait_block = &wait_lds;
    const auto look = [](int *counter) {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    };
    const auto post = [](int *counter, int n) {          // (written by every lane: the same word, no exec-mask juggling)
        __hip_atomic_store(counter, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // Everyone but the loader, whose first loads are under way in the meantime, prepares the LDS: entries mu >= L of the rows
    // of h stay +inf (they never win); V transposed, all of a thread's loads in one batch.
    float Vr[HR];                                 // the candidates' column of V
    if (wave != 1) {
        constexpr int NT = 192, IT = (SEG * MU + NT - 1) / NT;
        const int t = wave == 0 ? lane : (int)threadIdx.x - 64;
        float x[IT];
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int e = t + NT * i, l2 = e % SEG, mu = e / SEG;
            x[i] = (mu < L && l2 < L) ? P.V[(size_t)mu * L + l2] : 0.0f;
        }
        for (int e = t; e < NR * NROW * HP; e += NT) (&hring[0][0][0])[e] = INFINITY;
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int e = t + NT * i;
            if (e < SEG * MU) vt[e % SEG][e / SEG] = x[i];
        }
        mrf_block_sync_lds();
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            const float4 x = *reinterpret_cast<const float4 *>(&vt[lam][grp * HR + 4 * k]);
            Vr[4 * k] = x.x; Vr[4 * k + 1] = x.y; Vr[4 * k + 2] = x.z; Vr[4 * k + 3] = x.w;
        }
    }
    const auto bits = [](float x) { return __builtin_bit_cast(unsigned, x); };
    const auto real = [](unsigned x) { return __builtin_bit_cast(float, x); };

    if (wave == 0) {
        // ---- values: step n forms the message of node n ------------------------------------------
        __builtin_amdgcn_s_setprio(3);
        bool plain = true;
#pragma unroll
        for (int m = 0; m < HR; ++m) plain = plain && !(Vr[m] < 0.0f) && !(grp * HR + m == lam && Vr[m] != 0.0f);
        const unsigned long long slow = __all(plain) ? 0ull : ~0ull;
        const float rho = P.rho[r];
        const auto await = [&](int n) {
            int turns = 0;
            while (look(&loaded) < n) mrf_wait_turn(wait_block, turns);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        };
        const auto label_min = [&](float x) {
            if constexpr (NG == 2) return mrf_segment_min32_regs(x, 0);         // (both halves hold every label)
            else if constexpr (SEG == 16) {
                asm("s_nop 1\n\t"
                    "v_min_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
                    "s_nop 1\n\t"
                    "v_min_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
                    "s_nop 1\n\t"
                    "v_min_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                    "s_nop 1\n\t"
                    "v_min_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\t"
                    : "+v"(x));
                return x;
            } else if constexpr (SEG == 32) return mrf_segment_min32_regs(x, lane);
            else return mrf_segment_min<SEG>(x);
        };
        if (maxlen < 2) return;
        float4 q4[NQ > 0 ? NQ : 1];
        float2 d2;
        const auto fetch = [&](int slot) {
#pragma unroll
            for (int k = 0; k < NQ; ++k) q4[k] = inq[k][slot][lane];
            d2 = ind[slot][lane];
        };
        const auto arrived = [&]() {
#pragma unroll
            for (int k = 0; k < NQ; ++k) asm volatile("" : : "v"(q4[k].x), "v"(q4[k].y), "v"(q4[k].z), "v"(q4[k].w));
            asm volatile("" : : "v"(d2.x), "v"(d2.y));
        };
        await(1);
        fetch(0);
        arrived();
        float carry = 0.0f;
        for (int n = 1;;) {
#pragma unroll
            for (int u = 0; u < NR; ++u, ++n) {          // step n uses slot u = (n - 1) % NR
                float v, wgt = d2.y;
                if constexpr (TRWP) {
                    v = q4[0].x + carry;
#pragma unroll
                    for (int c = 1; c < RMAX; ++c) v = v + (c % 4 == 0 ? q4[c / 4].x : (c % 4 == 1 ? q4[c / 4].y : (c % 4 == 2 ? q4[c / 4].z : q4[c / 4].w)));
                    v = rho * v;
                    v = v - d2.x;
                } else {
                    v = d2.x + carry;
                }
                v = valid ? v : INFINITY;
                hring[u][seg][lam] = v;                  // (groups write the same values to the same places)
                mrf_wave_lds_fence();
                float4 hv[NCH];
#pragma unroll
                for (int k = 0; k < NCH; ++k) hv[k] = *reinterpret_cast<const float4 *>(&hring[u][seg][grp * HR + 4 * k]);
                // in the same batch: the loader's counter, then (LDS keeps this order) the next node
                const int seen = __hip_atomic_load(&loaded, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                fetch((u + 1) & (NR - 1));
                __builtin_amdgcn_sched_barrier(0);
                float tq;
                if constexpr (SEG != 21) tq = label_min(v);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (SEG == 21) {
                    // (segments that do not line up with the rows of 16 lanes: a lane has all of h by now)
                    tq = mrf_min3(hv[0].x, hv[0].y, mrf_min(hv[0].z, hv[0].w));
#pragma unroll
                    for (int k = 1; k < NCH; ++k) tq = mrf_min3(mrf_min3(tq, hv[k].x, hv[k].y), hv[k].z, hv[k].w);
                }
                float cm[NCH], best;
#pragma unroll
                for (int k = 0; k < NCH; ++k) {
                    const float e0 = __builtin_fmaf(wgt, Vr[4 * k], hv[k].x), e1 = __builtin_fmaf(wgt, Vr[4 * k + 1], hv[k].y);
                    const float e2 = __builtin_fmaf(wgt, Vr[4 * k + 2], hv[k].z), e3 = __builtin_fmaf(wgt, Vr[4 * k + 3], hv[k].w);
                    if constexpr (NC > 0) {
                        cm[k] = mrf_min(mrf_min3(e0, e1, e2), e3);
                    } else {
                        // (+inf where every candidate is NaN: here, or where the groups are joined)
                        best = k > 0 ? mrf_min3(best, e0, e1) : (NG > 1 ? mrf_min(e0, e1) : mrf_min3(e0, e1, INFINITY));
                        best = mrf_min3(best, e2, e3);
                    }
                }
                if constexpr (NC > 0) {
                    best = cm[0];
#pragma unroll
                    for (int k = 1; k + 1 < NCH; k += 2) best = mrf_min3(best, cm[k], cm[k + 1]);
                    best = mrf_min3(best, cm[NCH - 1], INFINITY);
                }
                if constexpr (NG == 4) {
                    const auto x = __builtin_amdgcn_permlane16_swap(bits(best), bits(best), false, false);
                    best = mrf_min(real(x[0]), real(x[1]));
                }
                if constexpr (NG >= 2) {
                    const auto x = __builtin_amdgcn_permlane32_swap(bits(best), bits(best), false, false);
                    best = mrf_min3(real(x[0]), real(x[1]), INFINITY);
                }
                if (__builtin_expect((__ballot(bits(wgt) >= 0x7f800000u) | slow) != 0, 0)) tq = label_min(valid ? best : INFINITY);
                carry = best - tq;
                // (the next node's values are waited for here, where only reads are under way: behind the writes below the
                // wait would be for those)
                arrived();
                // (what is behind the last group repeats it)
#pragma unroll
                for (int k = 0; k < NC; ++k)
                    cring[k][u][lane] = make_float4(cm[4 * k < NCH ? 4 * k : 0], cm[4 * k + 1 < NCH ? 4 * k + 1 : NCH - 1], cm[4 * k + 2 < NCH ? 4 * k + 2 : NCH - 1],
                                                    cm[4 * k + 3 < NCH ? 4 * k + 3 : NCH - 1]);
                mring[u][lane] = carry;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");      // (LDS keeps a wavefront's operations in order)
                post(&valued, n);
                if (n + 1 >= maxlen) return;             // (uniform)
                if (__builtin_expect(__builtin_amdgcn_readfirstlane(seen) <= n, 0)) {
                    await(n + 1);
                    fetch((u + 1) & (NR - 1));
                    arrived();
                }
            }
        }
    }

    if (wave == 1) {
        // ---- loader ------------------------------------------------------------------------------
        // Sources of h in summation order: the unary, then message arrays; unused slots load 0 and enter with factor 0
        // (fma(0, 0, v) = v and fma(1, x, v) = v + x exactly).  r^- once more by itself.
        __builtin_amdgcn_s_setprio(3);
        const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];
        mrf_buf src[RMAX];
        float before[RMAX], after[RMAX];
        src[0] = mrf_buffer(P.unary + (size_t)__builtin_amdgcn_readfirstlane((int)P.unary_slab[r]) * NL, NL * 4);
#pragma unroll
        for (int c = 1; c < RMAX; ++c) {
            const bool live = c <= n_src;
            const size_t d = (size_t)__builtin_amdgcn_readfirstlane(live ? (int)P.src_dir[r][c - 1] : 0);
            src[c] = mrf_buffer(P.m_in + d * NL, live ? NL * 4 : 0);
            before[c] = live && (!TRWP || c <= n_pre) ? 1.0f : 0.0f;
            after[c] = live && TRWP && c > n_pre ? 1.0f : 0.0f;
        }
        const bool has_rm = TRWP && rm_slot >= 0;
        const mrf_buf brm = mrf_buffer(P.m_in + (size_t)__builtin_amdgcn_readfirstlane(has_rm ? (int)P.src_dir[r][has_rm ? rm_slot : 0] : 0) * NL,
                                       has_rm ? NL * 4 : 0);
        const mrf_buf bw = mrf_buffer(P.w + (P.w_mul ? (size_t)r * N : 0), P.w_mul ? N * 4 : 4);
        struct In {
            float v[RMAX];
            float rm, w;
        };
        In A[D], B[D];
        // (what is loaded past a scanline's end is another node or 0, and never used)
        unsigned pe = ((unsigned)head * (unsigned)L + (unsigned)lamc) << 2;
        unsigned pw = P.w_mul ? (unsigned)(head + nstep) << 2 : 0u;
        const unsigned pe_step = estep << 2, pw_step = P.w_mul ? (unsigned)nstep << 2 : 0u;
        auto prefetch = [&](In &in) {
#pragma unroll
            for (int c = 0; c < RMAX; ++c) in.v[c] = mrf_buf_f32(src[c], pe);
            in.rm = TRWP ? mrf_buf_f32(brm, pe) : 0.0f;
            in.w = mrf_buf_f32(bw, pw);
            pe += pe_step;
            pw += pw_step;
        };
        int freed = 0;                           // steps up to this one have left the ring
        auto group = [&](const In (&in)[D], int n0) {
#pragma unroll
            for (int u = 0; u < D; ++u) {
                const int n = n0 + u;
                float base = in[u].v[0];
#pragma unroll
                for (int c = 1; c < RMAX; ++c) base = __builtin_fmaf(before[c], in[u].v[c], base);
                if (n >= maxlen) break;          // (uniform)
                int turns = 0;
                while (freed < n - NR) {
                    // the index wavefronts take the steps in turn: behind the slowest one's last step, the others have
                    // finished theirs
                    const int i0 = look(&indexed[0]), i1 = look(&indexed[1]);
                    freed = (i0 < i1 ? i0 : i1) + NI - 1;
                    if (freed < n - NR) mrf_wait_turn(wait_block, turns);
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                }
                const int slot = (n - 1) & (NR - 1);
                if constexpr (TRWP) {
                    float a[RMAX];
                    a[0] = base;
#pragma unroll
                    for (int c = 1; c < RMAX; ++c) a[c] = after[c] * in[u].v[c];
#pragma unroll
                    for (int k = 0; k < NQ; ++k) inq[k][slot][lane] = make_float4(a[4 * k], a[4 * k + 1], a[4 * k + 2], a[4 * k + 3]);
                    ind[slot][lane] = make_float2(in[u].rm, in[u].w);
                } else {
                    ind[slot][lane] = make_float2(base, in[u].w);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                post(&loaded, n);
            }
        };
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(A[u]);
        mrf_block_sync_lds();
        for (int n0 = 1; n0 < maxlen; n0 += 2 * D) {
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(B[u]);
            __builtin_amdgcn_sched_barrier(0);
            group(A, n0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < D; ++u) prefetch(A[u]);
            __builtin_amdgcn_sched_barrier(0);
            group(B, n0 + D);
            __builtin_amdgcn_sched_barrier(0);
        }
        return;
    }

    // ---- index: p, q and all stores; wavefront jw takes steps 1 + jw, 1 + jw + NI, ... -------------------
    const int jw = wave - 2;
    const mrf_buf bm = mrf_buffer(P.m_out + (size_t)r * NL, NL * 4), bp = mrf_buffer(P.p + (size_t)r * NL, NL);
    const mrf_buf bq = mrf_buffer(P.q + (size_t)r * N, N);
    const bool mine = act_seg && valid && grp == 0;
    unsigned oe = (unsigned)head * (unsigned)L + (unsigned)lam, on = (unsigned)head;
    if (jw == 0) {
        // first node of the scanline: message 0, p = q = 0
        mrf_buf_store_f32(bm, mine ? oe << 2 : MRF_BUF_NONE, 0.0f);
        mrf_buf_store_u8(bp, mine ? oe : MRF_BUF_NONE, 0);
        mrf_buf_store_u8(bq, mine && lam == 0 ? on : MRF_BUF_NONE, 0);
    }
    const int len_m = mine ? len : 0, len_q = mine && lam == 0 ? len : 0;
    oe += (unsigned)jw * estep;
    on += (unsigned)(jw * nstep);
    int seen = 0;
    oe += estep;
    on += (unsigned)nstep;
    for (int n = 1 + jw; n < maxlen; n += NI) {
        int turns = 0;
        while (seen < n) {
            seen = look(&valued);
            if (seen < n) mrf_wait_turn(wait_block, turns);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        const int slot = (n - 1) & (NR - 1);
        const float wgt = ind[slot][lane].y, m = mring[slot][lane];
        const float *hr = &hring[slot][seg][grp * HR], *vr = &vt[lam][grp * HR];
        // lowest group of four that attains the minimum of all, then the lowest of its candidates, formed once more
        float best = 0.0f;
        int ck = NCH - 1;
        if constexpr (NC > 0) {
            float4 c4[NC];
#pragma unroll
            for (int k = 0; k < NC; ++k) c4[k] = cring[k][slot][lane];
            best = mrf_min(mrf_min3(c4[0].x, c4[0].y, c4[0].z), c4[0].w);
            if constexpr (NC > 1) best = mrf_min(mrf_min3(best, c4[NC - 1].x, c4[NC - 1].y), mrf_min(c4[NC - 1].z, c4[NC - 1].w));
            // (of the repeated ones the lowest index, which is looked at last, is the one that stands)
            if constexpr (NC > 1) mrf_first_equal4<4>(ck, best, c4[NC - 1].x, c4[NC - 1].y, c4[NC - 1].z, c4[NC - 1].w);
            mrf_first_equal4<0>(ck, best, c4[0].x, c4[0].y, c4[0].z, c4[0].w);
        } else if constexpr (NCH > 1) {
            float cm[NCH];
#pragma unroll
            for (int k = 0; k < NCH; ++k) {
                const float4 hk = *reinterpret_cast<const float4 *>(hr + 4 * k);
                const float e0 = __builtin_fmaf(wgt, Vr[4 * k], hk.x), e1 = __builtin_fmaf(wgt, Vr[4 * k + 1], hk.y);
                const float e2 = __builtin_fmaf(wgt, Vr[4 * k + 2], hk.z), e3 = __builtin_fmaf(wgt, Vr[4 * k + 3], hk.w);
                cm[k] = mrf_min(mrf_min3(e0, e1, e2), e3);
            }
            best = cm[0];
#pragma unroll
            for (int k = 1; k + 1 < NCH; k += 2) best = mrf_min3(best, cm[k], cm[k + 1]);
            if constexpr (NCH % 2 == 0) best = mrf_min(best, cm[NCH - 1]);
            // (where there are not four or eight they overlap or repeat: the lowest index wins all the same)
            if constexpr (NCH > 4) mrf_first_equal4<NCH - 4>(ck, best, cm[NCH - 4], cm[NCH - 3], cm[NCH - 2], cm[NCH - 1]);
            mrf_first_equal4<0>(ck, best, cm[0], cm[1], cm[NCH > 2 ? 2 : NCH - 1], cm[NCH > 3 ? 3 : NCH - 1]);
        }
        const float4 va = *reinterpret_cast<const float4 *>(vr + 4 * ck), hv = *reinterpret_cast<const float4 *>(hr + 4 * ck);
        const float d0 = __builtin_fmaf(wgt, va.x, hv.x), d1 = __builtin_fmaf(wgt, va.y, hv.y);
        const float d2 = __builtin_fmaf(wgt, va.z, hv.z), d3 = __builtin_fmaf(wgt, va.w, hv.w);
        if constexpr (NCH == 1) best = mrf_min(mrf_min3(d0, d1, d2), d3);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        post(&indexed[jw], n);
        int arg = 3;
        mrf_first_equal4<0>(arg, best, d0, d1, d2, d3);
        arg += 4 * ck;
        if constexpr (NG > 1) {
            // join the groups: the lower one's index on a tie, never that of a group whose candidates are all NaN
            arg += grp * HR;
            if constexpr (NG == 4) {
                const auto x = __builtin_amdgcn_permlane16_swap(bits(best), bits(best), false, false);
                const auto a = __builtin_amdgcn_permlane16_swap((unsigned)arg, (unsigned)arg, false, false);
                best = mrf_min(real(x[0]), real(x[1]));
                arg = real(x[0]) == best ? (int)a[0] : (int)a[1];
            }
            const auto x = __builtin_amdgcn_permlane32_swap(bits(best), bits(best), false, false);
            const auto a = __builtin_amdgcn_permlane32_swap((unsigned)arg, (unsigned)arg, false, false);
            best = mrf_min(real(x[0]), real(x[1]));
            arg = real(x[0]) == best ? (int)a[0] : (int)a[1];
        }
        arg = best < INFINITY ? arg : 0;                 // (and with that below L: labels past it are +inf)
        // the message is 0 exactly where it attains a finite minimum, NaN where it attains an infinite one
        const unsigned long long least = __ballot((int)valid & (int)!(m > 0.0f));
        const int qidx = mrf_segment_first<SEG>(least, lane);
        mrf_buf_store_f32(bm, n < len_m ? oe << 2 : MRF_BUF_NONE, m);
        mrf_buf_store_u8(bp, n < len_m ? oe : MRF_BUF_NONE, arg);
        mrf_buf_store_u8(bq, n < len_q ? on : MRF_BUF_NONE, qidx);
        oe += NI * estep;
        on += (unsigned)(NI * nstep);
    }
}

// ---- dense sweep for few labels with scanlines to spare: one direction per wavefront ----------------
//
// mrf_fwd_sweep_packed for launches that fill the machine, where the issue of vector instructions bounds the step
// (185 per wavefront and node of the segmentation shape).  Scanlines of one wavefront belong to one direction
// (the host pads every direction to whole wavefronts), so base addresses, factors and source counts are scalars and
// an entry is one 32-bit offset into buffer views (the host checks that N L fits) that walks by one addition; what a
// lane loads past its scanline's end is another node or 0 and never used, and a store that is not wanted has an
// offset past the view's.  The argmin takes two levels: minima of four candidates, the lowest group that attains
// the overall minimum, and that group's four candidates once more (the same fma on the same operands gives the same
// bits) against a transposed copy of V in LDS: 2.6 instructions per candidate instead of 3.5.  Where nothing but the
// start term is read (RMAX = 1: ISGMR's first iteration, and all of them behind mrf_isgmr_presum) no empty slots are.
// Learning steps, K = 5: 4 x 512 x 512, 21 labels, ISGMR 4.32 -> 4.13 ms; 256 x 512, 32 labels, 16 directions 4.17 -> 3.61.
template <int SEG, int MU, int RMAX, int D, bool TRWP>
__global__ void __launch_bounds__(64) mrf_fwd_sweep_narrow(const MrfFwdParams P)
{
    static_assert(MU % 4 == 0 && (MU <= SEG || (SEG == 21 && MU == 24)), "source label count");
    constexpr int NSEG = 64 / SEG;                // (three segments of 21 lanes leave lane 63 idle)
    constexpr int NROW = SEG == 21 ? 4 : NSEG;    // LDS rows: the idle lane gets one of its own to scribble in
    constexpr int SEGP = SEG == 21 ? 28 : SEG + 4;   // row stride: 16-byte rows on different banks
    constexpr int NCH = MU / 4;                   // groups of four candidates
    __shared__ __align__(16) float hrow[NROW][SEGP];
    __shared__ __align__(16) float vt[SEG][MU + 4];  // V transposed: row lambda
    const int L = P.g.L;
    const int lane = threadIdx.x & 63;
    const int seg = lane / SEG, lam = lane % SEG;
    const bool valid = lam < L;
    const int lamc = valid ? lam : 0;

    // this wavefront's scanlines: NSEG consecutive ones of direction r
    const int blk = (int)blockIdx.x;
    int ri = 0;
    while (ri + 1 < P.r_count && blk >= P.pack_begin[ri + 1]) ++ri;
    const int r = P.r_first + ri;
    const unsigned nsc = (unsigned)P.g.nscan[r];
    const unsigned sl = (unsigned)(blk - P.pack_begin[ri]) * NSEG + seg;
    const bool act_seg = seg < NSEG && sl < (unsigned)P.g.B * nsc;
    const int dh = P.g.dh[r], dw = P.g.dw[r];
    const int nstep = dh * P.g.W + dw;
    int y0 = 0, x0 = 0, len = 0, head = 0;
    if (act_seg) {
        const int b = sl < nsc ? 0 : (int)(sl / nsc);
        mrf_geom_head(P.g.H, P.g.W, dh, dw, sl - (unsigned)b * nsc, y0, x0, len);
        head = (b * P.g.H + y0) * P.g.W + x0;
    }
    const float rho = P.rho[r];
    const int n_pre = P.n_pre[r], n_src = P.n_src[r], rm_slot = P.rm_slot[r];

    // Sources of h in summation order: the unary, then message arrays; unused slots load 0 and enter with factor 0
    // (fma(0, 0, v) = v and fma(1, x, v) = v + x exactly).  r^- once more by itself.
    const size_t N = (size_t)P.g.N, NL = N * L;
    mrf_buf src[RMAX];
    float before[RMAX], after[RMAX];
    src[0] = mrf_buffer(P.unary + (size_t)__builtin_amdgcn_readfirstlane((int)P.unary_slab[r]) * NL, NL * 4);
#pragma unroll
    for (int c = 1; c < RMAX; ++c) {
        const bool live = c <= n_src;
        const size_t d = (size_t)__builtin_amdgcn_readfirstlane(live ? (int)P.src_dir[r][c - 1] : 0);
        src[c] = mrf_buffer(P.m_in + d * NL, live ? NL * 4 : 0);
        before[c] = live && (!TRWP || c <= n_pre) ? 1.0f : 0.0f;
        after[c] = live && TRWP && c > n_pre ? 1.0f : 0.0f;
    }
    const bool has_rm = TRWP && rm_slot >= 0;
    const mrf_buf brm = mrf_buffer(P.m_in + (size_t)__builtin_amdgcn_readfirstlane(has_rm ? (int)P.src_dir[r][has_rm ? rm_slot : 0] : 0) * NL,
                                   has_rm ? NL * 4 : 0);
    const mrf_buf bm = mrf_buffer(P.m_out + (size_t)r * NL, NL * 4), bp = mrf_buffer(P.p + (size_t)r * NL, NL);
    const mrf_buf bq = mrf_buffer(P.q + (size_t)r * N, N), bw = mrf_buffer(P.w + (P.w_mul ? (size_t)r * N : 0), P.w_mul ? N * 4 : 4);

    float Vr[MU];
#pragma unroll
    for (int mu = 0; mu < MU; ++mu) {
        Vr[mu] = (mu < L && valid) ? P.V[(size_t)mu * L + lam] : 0.0f;
        vt[lam][mu] = Vr[mu];                     // (every segment writes the same)
    }
    hrow[seg][lam] = INFINITY;                    // entries mu >= L stay +inf: they never win
    if (lam < SEGP - SEG) hrow[seg][SEG + lam] = INFINITY;
    __syncthreads();

    auto store_u8 = [](mrf_buf b, unsigned off, int x) { __builtin_amdgcn_raw_buffer_store_b8((unsigned char)x, b, off, 0, 0); };
    // first node of the scanline: message 0, p = q = 0
    unsigned oe = (unsigned)head * (unsigned)L + (unsigned)lam, on = (unsigned)head;
    {
        const bool st = act_seg && valid;
        mrf_buf_store_f32(bm, st ? oe << 2 : MRF_BUF_NONE, 0.0f);
        store_u8(bp, st ? oe : MRF_BUF_NONE, 0);
        store_u8(bq, st && lam == 0 ? on : MRF_BUF_NONE, 0);
    }
    // longest scanline of the wavefront bounds the loop
    int maxlen = 0;
#pragma unroll
    for (int sg = 0; sg < NSEG; ++sg) {
        const int l2 = __builtin_amdgcn_readlane(len, sg * SEG);
        maxlen = l2 > maxlen ? l2 : maxlen;
    }
    if (maxlen < 2) return;

    const int len_m = valid ? len : 0, len_q = lam == 0 ? len : 0;       // (a segment has lam == 0 only in its first lane)
    const unsigned estep = (unsigned)nstep * (unsigned)L;
    struct In {
        float v[RMAX];
        float rm, w;
    };
    In A[D], B[D];
    unsigned pe = ((unsigned)head * (unsigned)L + (unsigned)lamc) << 2;
    unsigned pw = P.w_mul ? (unsigned)(head + nstep) << 2 : 0u;
    const unsigned pe_step = estep << 2, pw_step = P.w_mul ? (unsigned)nstep << 2 : 0u;
    auto prefetch = [&](In &in) {
#pragma unroll
        for (int c = 0; c < RMAX; ++c) in.v[c] = mrf_buf_f32(src[c], pe);
        in.rm = TRWP ? mrf_buf_f32(brm, pe) : 0.0f;
        in.w = mrf_buf_f32(bw, pw);
        pe += pe_step;
        pw += pw_step;
    };

    float carry = 0.0f;
    auto group = [&](const In (&in)[D], int n0) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int n = n0 + u;
            float v = in[u].v[0];
#pragma unroll
            for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(before[c], in[u].v[c], v);
            v = v + carry;
            if (TRWP) {
#pragma unroll
                for (int c = 1; c < RMAX; ++c) v = __builtin_fmaf(after[c], in[u].v[c], v);
                v = rho * v;
                v = v - in[u].rm;
            }
            const float wgt = in[u].w;
            hrow[seg][lam] = valid ? v : INFINITY;
            mrf_wave_lds_fence();

            // candidates, minima of four, the minimum of all
            float cm[NCH];
#pragma unroll
            for (int k = 0; k < NCH; ++k) {
                const float4 hv = *reinterpret_cast<const float4 *>(&hrow[seg][4 * k]);
                const float d0 = __builtin_fmaf(wgt, Vr[4 * k], hv.x), d1 = __builtin_fmaf(wgt, Vr[4 * k + 1], hv.y);
                const float d2 = __builtin_fmaf(wgt, Vr[4 * k + 2], hv.z), d3 = __builtin_fmaf(wgt, Vr[4 * k + 3], hv.w);
                cm[k] = mrf_min(mrf_min3(d0, d1, d2), d3);
            }
            float best = NCH > 1 ? mrf_min(cm[0], cm[NCH > 1 ? 1 : 0]) : cm[0];
#pragma unroll
            for (int k = 2; k + 1 < NCH; k += 2) best = mrf_min3(best, cm[k], cm[k + 1]);
            if constexpr (NCH > 2 && NCH % 2 == 1) best = mrf_min(best, cm[NCH - 1]);

            const float tv = valid ? best : INFINITY;
            const float tq = mrf_segment_min<SEG>(tv);
            carry = tv - tq;
            const int qidx = mrf_segment_first<SEG>(__ballot(tv == tq), lane);

            // lowest group that attains the minimum (groups overlap or repeat where there are not four or eight:
            // the lowest index wins all the same), then the lowest of its candidates
            int ck = NCH - 1;
            if constexpr (NCH > 4) mrf_first_equal4<NCH - 4>(ck, best, cm[NCH - 4], cm[NCH - 3], cm[NCH - 2], cm[NCH - 1]);
            mrf_first_equal4<0>(ck, best, cm[0], cm[NCH > 1 ? 1 : 0], cm[NCH > 2 ? 2 : NCH - 1], cm[NCH > 3 ? 3 : NCH - 1]);
            const float4 va = *reinterpret_cast<const float4 *>(&vt[lam][4 * ck]), hv = *reinterpret_cast<const float4 *>(&hrow[seg][4 * ck]);
            int pj = 3;
            mrf_first_equal4<0>(pj, best, __builtin_fmaf(wgt, va.x, hv.x), __builtin_fmaf(wgt, va.y, hv.y), __builtin_fmaf(wgt, va.z, hv.z),
                                __builtin_fmaf(wgt, va.w, hv.w));
            mrf_wave_lds_fence();

            oe += estep;
            on += (unsigned)nstep;
            mrf_buf_store_f32(bm, n < len_m ? oe << 2 : MRF_BUF_NONE, carry);
            store_u8(bp, n < len_m ? oe : MRF_BUF_NONE, 4 * ck + pj);
            store_u8(bq, n < len_q ? on : MRF_BUF_NONE, qidx);
        }
    };
#pragma unroll
    for (int u = 0; u < D; ++u) prefetch(A[u]);
    // (dropped stores: what is in flight at the loop's entry then looks like what is in flight when it comes round)
#pragma unroll
    for (int u = 0; u < 3 * D; ++u) store_u8(bq, MRF_BUF_NONE, 0);
    for (int n0 = 1; n0 < maxlen; n0 += 2 * D) {
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(B[u]);
        __builtin_amdgcn_sched_barrier(0);
        group(A, n0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < D; ++u) prefetch(A[u]);
        __builtin_amdgcn_sched_barrier(0);
        group(B, n0 + D);
        __builtin_amdgcn_sched_barrier(0);
    }
}
