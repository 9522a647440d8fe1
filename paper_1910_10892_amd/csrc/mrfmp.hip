// libmrfmp host side: argument checks, workspace layout and launch schedules of the
// ISGMR / TRWP forward and backward passes (Alg. 1-4).  Allocates nothing.
//
// One source, up to nine translation units: compiled as it stands it holds everything; with
// -DMRF_PART=n it holds one part (the list below), so that the build can compile the parts in
// parallel and link them.  The sweep templates of a family are instantiated in one part only.
#include "../../include/mrfmp.h"
#include "mrfmp_device.h"

#ifndef MRF_PART
#define MRF_PART 0
#endif
#define MRF_HAS_FWD (MRF_PART == 0 || MRF_PART == 1)          // forward schedule, per-edge sweep, aggregation
#define MRF_HAS_BWD (MRF_PART == 0 || MRF_PART == 2)          // backward schedule, split sweep, combine pass
#define MRF_HAS_API (MRF_PART == 0 || MRF_PART == 3)          // entry points, heads
#define MRF_HAS_FWD_PACKED (MRF_PART == 0 || MRF_PART == 4)   // packed forward sweep
#define MRF_HAS_FWD_DUO (MRF_PART == 0 || MRF_PART == 5)      // value / index / loader window sweep
#define MRF_HAS_FWD_WINDOW (MRF_PART == 0 || MRF_PART == 6)   // the other window sweeps
#define MRF_HAS_FWD_DENSE (MRF_PART == 0 || MRF_PART == 7)    // dense sweeps
#define MRF_HAS_BWD_CHAIN (MRF_PART == 0 || MRF_PART == 8)    // chain backward sweep
#define MRF_HAS_BWD_PLAIN (MRF_PART == 0 || MRF_PART == 9)    // the other backward sweeps

#if MRF_HAS_FWD || MRF_HAS_FWD_PACKED || MRF_HAS_FWD_DUO || MRF_HAS_FWD_WINDOW || MRF_HAS_FWD_DENSE
#include "mrfmp_fwd.h"
#endif
#if MRF_HAS_BWD || MRF_HAS_BWD_CHAIN || MRF_HAS_BWD_PLAIN
#include "mrfmp_bwd.h"
#endif
#if MRF_HAS_BWD
#include "mrfmp_bwd_sum.h"
#endif
#if MRF_HAS_API
#include "mrfmp_head.h"
#endif

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

namespace mrf_host {

constexpr size_t kAlign = 256;
// private V-gradient accumulators, one per workgroup or wavefront of a sweep: many small ones (flushed from LDS
// once) for few labels, fewer large ones otherwise
inline long long grad_slots(int L) { return L <= 32 ? 16384 : 1024; }

inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

inline int check_problem(const mrf_problem *pr, int algo, bool forward)
{
    if (!pr) return MRF_ERR_NULL_POINTER;
    if (algo != MRF_ISGMR && algo != MRF_TRWP) return MRF_ERR_BAD_ALGORITHM;
    if (pr->B < 1 || pr->H < 1 || pr->W < 1) return MRF_ERR_BAD_SHAPE;
    if (pr->L < 1 || pr->L > MRF_MAX_LABELS) return MRF_ERR_BAD_LABELS;
    if (pr->K < 1) return MRF_ERR_BAD_ITERATIONS;
    // standard SGM is a single pass of the ISGMR sweeps without a backward pass of its own
    if (pr->sgm_standard && (algo != MRF_ISGMR || pr->K != 1 || pr->pairwise_edge)) return MRF_ERR_BAD_ALGORITHM;
    if (pr->R < 1 || pr->R > MRF_MAX_DIRECTIONS) return MRF_ERR_BAD_DIRECTIONS;
    if (!pr->dirs) return MRF_ERR_NULL_POINTER;
    for (int r = 0; r < pr->R; ++r) {
        const int dh = pr->dirs[2 * r], dw = pr->dirs[2 * r + 1];
        if (dh == 0 && dw == 0) return MRF_ERR_BAD_DIRECTIONS;
        for (int d = 0; d < r; ++d)
            if (pr->dirs[2 * d] == dh && pr->dirs[2 * d + 1] == dw) return MRF_ERR_BAD_DIRECTIONS;
    }
    const long long N = (long long)pr->B * pr->H * pr->W;
    if (N > 0x7fffffffLL) return MRF_ERR_BAD_SHAPE;
    if (!pr->pairwise && !pr->pairwise_edge) return MRF_ERR_NULL_POINTER;
    if (pr->pairwise_edge) {
        // one table per edge: few labels only, and no promise about V applies
        if (pr->L > 64) return MRF_ERR_BAD_LABELS;
        if (pr->pairwise_kind != MRF_PAIRWISE_DENSE) return MRF_ERR_BAD_PAIRWISE_KIND;
        if ((long long)pr->R * N * pr->L > 0x7fffffffLL) return MRF_ERR_BAD_SHAPE;
    }
    if (forward && !pr->unary) return MRF_ERR_NULL_POINTER;
    if (algo == MRF_TRWP && !pr->rho && !pr->rho_edge) return MRF_ERR_NULL_POINTER;
    if (pr->pairwise_kind != MRF_PAIRWISE_DENSE && pr->pairwise_kind != MRF_PAIRWISE_TRUNC_LINEAR &&
        pr->pairwise_kind != MRF_PAIRWISE_TRUNC_QUADRATIC && pr->pairwise_kind != MRF_PAIRWISE_DISTANCE)
        return MRF_ERR_BAD_PAIRWISE_KIND;
    if (pr->pairwise_kind != MRF_PAIRWISE_DENSE && !(pr->trunc > 0.0f)) return MRF_ERR_BAD_PAIRWISE_KIND;
    // the window sweeps need V non-decreasing in the label distance: a negative scale turns it round
    if ((pr->pairwise_kind == MRF_PAIRWISE_TRUNC_LINEAR || pr->pairwise_kind == MRF_PAIRWISE_TRUNC_QUADRATIC) &&
        !(pr->scale >= 0.0f)) return MRF_ERR_BAD_PAIRWISE_KIND;
    return MRF_OK;
}

inline void fill_geom(const mrf_problem *pr, MrfGeom &g)
{
    memset(&g, 0, sizeof(g));
    g.B = pr->B; g.H = pr->H; g.W = pr->W; g.L = pr->L; g.R = pr->R;
    g.N = (long long)pr->B * pr->H * pr->W;
    for (int r = 0; r < pr->R; ++r) {
        g.dh[r] = pr->dirs[2 * r];
        g.dw[r] = pr->dirs[2 * r + 1];
    }
    for (int r = 0; r < pr->R; ++r) {
        g.opp[r] = -1;
        for (int d = 0; d < pr->R; ++d)
            if (g.dh[d] == -g.dh[r] && g.dw[d] == -g.dw[r]) g.opp[r] = d;
        g.nscan[r] = (int)mrf_geom_scanlines(g.H, g.W, g.dh[r], g.dw[r]);
    }
}

// nodes of the longest scanline of direction r
inline long long longest_scanline(const MrfGeom &g, int r)
{
    const int ah = mrf_iabs(g.dh[r]), aw = mrf_iabs(g.dw[r]);
    const int down = ah ? (g.H + ah - 1) / ah : INT_MAX, across = aw ? (g.W + aw - 1) / aw : INT_MAX;
    return down < across ? down : across;
}
inline long long longest_scanline(const MrfGeom &g, int r_first, int r_count)
{
    long long most = 0;
    for (int r = r_first; r < r_first + r_count; ++r) {
        const long long n = longest_scanline(g, r);
        most = n > most ? n : most;
    }
    return most;
}

inline size_t msg_bytes(const mrf_problem *pr)
{
    return align_up((size_t)pr->R * pr->B * pr->H * pr->W * pr->L * sizeof(float));
}

inline size_t gradv_bytes(const mrf_problem *pr)
{
    return align_up((size_t)grad_slots(pr->L) * pr->L * pr->L * sizeof(double));
}

// Most scanlines of a launch whose node gradients are stored for mrf_bwd_pairwise_* (33..128 labels, one direction per
// launch), and room for them.  (By shape, directions and algorithm only, so that problems which agree in these can share
// a workspace.)
constexpr long long kApartMost = 1536;
inline size_t gstore_bytes(const mrf_problem *pr, int algo)
{
    if (pr->L <= 32 || pr->L > 128 || (algo == MRF_ISGMR && pr->R > 1)) return 0;
    bool any = false;
    for (int r = 0; r < pr->R; ++r)
        any = any || pr->B * mrf_geom_scanlines(pr->H, pr->W, pr->dirs[2 * r], pr->dirs[2 * r + 1]) <= kApartMost;
    return any ? align_up((size_t)pr->B * pr->H * pr->W * pr->L * sizeof(double)) : 0;
}

// Room for the node gradients that mrf_bwd_edge_tables adds up (per-edge tables): those of all iterations, but no more
// than half of what the tables themselves take.  (A call with less room takes what there is, run_backward.)
inline size_t edge_slab_bytes(const mrf_problem *pr) { return (size_t)pr->R * pr->B * pr->H * pr->W * pr->L * sizeof(float); }
inline size_t edge_grad_bytes(const mrf_problem *pr)
{
    const int most = pr->L / 2 > 1 ? pr->L / 2 : 1;
    return align_up((size_t)(pr->K < most ? pr->K : most) * edge_slab_bytes(pr));
}

// ---- process-global state: defined in the translation unit of the entry points ----------
// tuning knobs (0 = heuristic)
#if MRF_HAS_API
#define MRF_G(decl, init) thread_local decl = init
#else
#define MRF_G(decl, init) extern thread_local decl
#endif
MRF_G(int g_tune_mch, 0);
MRF_G(int g_tune_no_window, 0);
MRF_G(int g_tune_split, 0);      // 0 auto, 1 never, 2 whenever L > 64
MRF_G(int g_tune_pack, 0);       // 0 auto, 1 never, 2 whenever L <= 32
MRF_G(int g_tune_duo, 0);        // 0 auto, 1 never, 2 whenever the window applies
MRF_G(int g_tune_duo_ni, 0);     // index wavefronts per scanline: 0 auto, 1, 2
MRF_G(int g_tune_loader, 0);     // loader wavefront in the window sweep: 0 auto, 1 never, 2 whenever possible
MRF_G(int g_tune_squad, 0);      // loader and index wavefronts next to the split layout: 0 by launch size, 1 never, 2 always
MRF_G(int g_tune_squad_ni, 0);   // how many of both: 0 auto, 4, 8
MRF_G(int g_tune_pack3, 0);      // three scanlines per wavefront for 17..21 labels: 0 by launch size, 1 never, 2 always
MRF_G(int g_tune_isgmr_lazy, 0); // ISGMR backward without a combine pass per iteration (up to 4 directions): 0 auto, 1 never
MRF_G(int g_tune_isgmr_presum, 0); // ISGMR forward with the per-pair sums of the previous iteration formed once: 0 from six directions, 1 never, 2 always
MRF_G(int g_tune_chain_pk, 0);     // chain backward with two scanlines of up to 32 labels per workgroup: 0 by launch size, 1 never, 2 always
MRF_G(int g_tune_gv_apart, 0);     // pairwise gradients of 33..128 labels by a streaming pass behind the chain backward sweep: 0 yes, 1 no
MRF_G(int g_tune_gv_tile, 0);      // V gradient of 33..128 labels in one LDS table per workgroup: 0 yes, 1 no (a slot per wavefront in global memory)
MRF_G(int g_tune_dense_sliced, 0); // dense sweep of 33 and more labels: 0 by launch shape, 1 every wavefront does the whole node, 2 a slice of the labels each, 3 chunk minima
MRF_G(int g_tune_spin_limit, 0); // turns a wait between wavefronts may take: 0 = default
MRF_G(int g_tune_pack_idx, 0);   // packed dense sweep divided among four wavefronts: 0 by launch size, 1 never, 2 always, 3 never and 64-bit offsets,
                                 // 4 always and one scanline per wavefront, 5 always and several, 6 as 3 with two index wavefronts
MRF_G(int g_tune_chain, 0);      // backward sweep with a chain wavefront: 0 auto, 1 never, 2 whenever possible
MRF_G(int g_tune_chain_hot, 0);  // its words for the lanes of the most popular scatter target: 0 auto, 1 never, 2 whenever V is no dense table
MRF_G(int g_tune_chain_ni, 0);   // its helpers per scanline: 0 auto, 2, 4, 6, 8, 12
MRF_G(int g_tune_narrow_divided, 0); // narrow backward sweep divided among four wavefronts: 0 by launch size, 1 never, 2 whenever possible
MRF_G(int g_tune_narrow, 0);     // lanes per scanline of the narrow backward sweep: 0 by launch size, 8, 16, 32; -1: not that sweep
MRF_G(hipEvent_t g_ev_start, nullptr);
MRF_G(hipEvent_t g_ev_stop, nullptr);
#undef MRF_G
#if MRF_HAS_API
thread_local char g_error_detail[256] = "";
thread_local const char *g_last_sweep[2] = {"", ""};      // kernel of the last forward / backward sweep launch
thread_local char g_last_launch[2][160] = {"", ""};       // the same with template arguments and launch shape
#else
extern thread_local char g_error_detail[256];
extern thread_local const char *g_last_sweep[2];
extern thread_local char g_last_launch[2][160];
#endif

// records the kernel of a sweep launch: its name, and "name<template arguments> grid=.. block=.."
inline void note_launch(int backward, const char *name, long long grid, int block, const char *fmt, ...)
    __attribute__((format(printf, 5, 6)));
inline void note_launch(int backward, const char *name, long long grid, int block, const char *fmt, ...)
{
    g_last_sweep[backward] = name;
    char args[96];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(args, sizeof(args), fmt, ap);
    va_end(ap);
    snprintf(g_last_launch[backward], sizeof(g_last_launch[backward]), "%s<%s> grid=%lld block=%d", name, args, grid, block);
}

// Workspace header (the first 256 bytes): float [0] = the scalar edge weight, int at byte 128 = the
// fault word that a wait between wavefronts raises when it runs out (mrf_wait_again).
[[maybe_unused]] constexpr size_t kFaultOffset = 128;
// how long after its start a workgroup may still find one of its wavefronts waiting for another, in microseconds
// (sweeps take milliseconds)
constexpr int kSpinLimit = 4000000;
inline int spin_limit() { return g_tune_spin_limit > 0 ? g_tune_spin_limit : kSpinLimit; }
hipError_t init_header(void *workspace, float w_scalar, hipStream_t st);

// records which call failed and how, for mrf_last_error_detail
inline int hip_fail(hipError_t e, const char *what)
{
    snprintf(g_error_detail, sizeof(g_error_detail), "%s: %s", what, hipGetErrorString(e));
    return MRF_ERR_HIP;
}

inline void mark(hipEvent_t ev, hipStream_t st)
{
    if (g_ev_start && g_ev_stop) (void)hipEventRecord(ev, st);
}

// truncation distance that the forward pass rounds up to one of its window kernels, or 0
inline int window_width(const mrf_problem *pr)
{
    if (g_tune_no_window || pr->pairwise_kind == MRF_PAIRWISE_DENSE) return 0;
    double t = pr->trunc;
    if (pr->pairwise_kind == MRF_PAIRWISE_TRUNC_QUADRATIC) t = sqrt(t);
    if (!(t > 0.0) || t > 16.0) return 0;
    int ti = (int)ceil(t);
    if (ti < 1) ti = 1;
    if (ti >= pr->L) return 0;
    return ti <= 2 ? 2 : (ti <= 4 ? 4 : (ti <= 8 ? 8 : (ti <= 12 ? 12 : 16)));
}

// the schedules and the entry points
hipError_t fill(float *dst, long long n, float v, hipStream_t st);
int run_forward(const mrf_problem *pr, int algo, float *cost, uint8_t *labels, uint8_t *p, uint8_t *q,
                float *messages, void *workspace, size_t workspace_bytes, void *hip_stream);
int run_backward(const mrf_problem *pr, int algo, const float *grad_cost, const uint8_t *p, const uint8_t *q,
                 float *grad_unary, float *grad_w, float *grad_V, void *workspace, size_t workspace_bytes,
                 void *hip_stream);

// launchers of the families, each in the part that instantiates its kernels
#if MRF_HAS_FWD || MRF_HAS_FWD_PACKED || MRF_HAS_FWD_DUO || MRF_HAS_FWD_WINDOW || MRF_HAS_FWD_DENSE
hipError_t run_packed(MrfFwdParams &P, int seg, int algo, int rmax, long long scanlines, hipStream_t st);
hipError_t run_window_duo(MrfFwdParams &P, int algo, int tw, int ni, int ms, long long blocks, hipStream_t st);
hipError_t run_window_loader(MrfFwdParams &P, int tw, long long blocks, hipStream_t st);
hipError_t run_window_split(MrfFwdParams &P, int algo, int tw, int ms, long long blocks, hipStream_t st);
hipError_t run_window_squad(MrfFwdParams &P, int algo, int tw, int ni, int ms, long long blocks, hipStream_t st);
hipError_t run_window(MrfFwdParams &P, int algo, int tw, int ms, long long blocks, hipStream_t st);
hipError_t run_dense(MrfFwdParams &P, int algo, long long blocks, hipStream_t st);
#endif
#if MRF_HAS_BWD || MRF_HAS_BWD_CHAIN || MRF_HAS_BWD_PLAIN
#define MRF_BWD_TILE_WAVES 8
// LDS a workgroup of the chain sweep may take: the whole 160 KB of a compute unit when every
// compute unit gets at most one workgroup, half when two, else the 64 KB any launch may have.
inline size_t chain_lds_cap(long long scanlines)
{
    if (scanlines <= 256) return 156 * 1024;
    if (scanlines <= 512) return 78 * 1024;
    return 64 * 1024;
}

// Whether an image's entries lie beyond what the chain sweep's views reach (node gradients are doubles): then its variant that makes
// a view per access runs, with six helpers.
inline bool chain_far(const MrfGeom &g, bool node_gradients)
{
    return (long long)g.H * g.W * g.L > MRF_BUF_MOST / (node_gradients ? 2 : 1);
}
#define MRF_CHAIN_FAR_HELPERS 6

hipError_t run_bwd_chain(MrfBwdParams &P, int ns, int ni, bool vg, hipStream_t st);
hipError_t run_bwd_chain_pk(MrfBwdParams &P, int ns, int ni, hipStream_t st);
hipError_t run_bwd_packed(MrfBwdParams &P, int seg, int ns, hipStream_t st);
hipError_t run_bwd_narrow(MrfBwdParams &P, int seg, int ns, hipStream_t st);
hipError_t run_bwd_plain(MrfBwdParams &P, int ns, long long blocks, size_t lds, hipStream_t st);
hipError_t run_bwd_tile(MrfBwdParams &P, int ns, long long blocks, size_t lds, hipStream_t st);
#endif

#if MRF_HAS_FWD_PACKED
template <int SEG, int MU>
hipError_t launch_narrow_mu(MrfFwdParams P, int algo, int rmax, hipStream_t st)
{
    constexpr int NSEG = 64 / SEG;
    P.pack_begin[0] = 0;
    for (int ri = 0; ri < P.r_count; ++ri)
        P.pack_begin[ri + 1] = P.pack_begin[ri] + (int)((P.blk_begin[ri + 1] - P.blk_begin[ri] + NSEG - 1) / NSEG);
    const unsigned blocks = (unsigned)P.pack_begin[P.r_count];
    note_launch(0, "mrf_fwd_sweep_narrow", blocks, 64, "%d,%d,%d,%d,%s", SEG, MU, rmax, rmax <= 4 ? 4 : (rmax == 8 ? 2 : 1),
                algo == MRF_TRWP ? "true" : "false");
#define MRF_P(rm, d) \
    if (rmax == rm) { \
        if (algo == MRF_TRWP) hipLaunchKernelGGL((mrf_fwd_sweep_narrow<SEG, MU, rm, d, true>), dim3(blocks), dim3(64), 0, st, P); \
        else hipLaunchKernelGGL((mrf_fwd_sweep_narrow<SEG, MU, rm, d, false>), dim3(blocks), dim3(64), 0, st, P); \
        return hipGetLastError(); \
    }
    MRF_P(1, 4) MRF_P(4, 4) MRF_P(8, 2) MRF_P(16, 1)
#undef MRF_P
    return hipErrorInvalidValue;
}

// the packed sweep divided among four wavefronts
template <int SEG, int NG, int MU>
hipError_t launch_packed_divided(MrfFwdParams P, int algo, int rmax, hipStream_t st)
{
    constexpr int NSEG = NG > 1 ? 1 : 64 / SEG;
    P.pack_begin[0] = 0;
    bool none = algo == MRF_ISGMR;
    for (int ri = 0; ri < P.r_count; ++ri) {
        P.pack_begin[ri + 1] = P.pack_begin[ri] + (int)((P.blk_begin[ri + 1] - P.blk_begin[ri] + NSEG - 1) / NSEG);
        none = none && P.n_src[P.r_first + ri] == 0;
    }
    const unsigned blocks = (unsigned)P.pack_begin[P.r_count];
    if (none) rmax = 1;
    note_launch(0, "mrf_fwd_sweep_packed", blocks, 256, "%d,%d,%d,%d,%s", SEG, NG, MU, rmax, algo == MRF_TRWP ? "true" : "false");
    const dim3 grid(blocks), block(256);
#define MRF_P(rm) \
    if (rmax == rm) { \
        if (algo == MRF_TRWP) hipLaunchKernelGGL((mrf_fwd_sweep_packed<SEG, NG, MU, rm, true>), grid, block, 0, st, P); \
        else hipLaunchKernelGGL((mrf_fwd_sweep_packed<SEG, NG, MU, rm, false>), grid, block, 0, st, P); \
        return hipGetLastError(); \
    }
    MRF_P(4) MRF_P(8) MRF_P(16)
#undef MRF_P
    hipLaunchKernelGGL((mrf_fwd_sweep_packed<SEG, NG, MU, 1, false>), grid, block, 0, st, P);
    return hipGetLastError();
}

template <int SEG, int MU>
hipError_t launch_packed_mu(const MrfFwdParams &P, int algo, int rmax, long long scanlines, hipStream_t st)
{
    const unsigned blocks = (unsigned)((scanlines + 64 / SEG - 1) / (64 / SEG));
    // (few wavefronts in a launch beyond the 32-bit offsets: two further ones per workgroup for the argmin tables and stores)
    const bool idx = g_tune_pack_idx == 6 || (P.g.N * P.g.L > MRF_BUF_MOST && g_tune_pack_idx != 1 && g_tune_pack_idx != 3 &&
                                              (g_tune_pack_idx == 2 || blocks <= 1024));
    // else one wavefront does all: mrf_fwd_sweep_narrow as far as its 32-bit offsets reach
    if (!idx && g_tune_pack_idx != 3 && P.g.N * P.g.L <= MRF_BUF_MOST) {
        bool none = true;
        for (int r = P.r_first; r < P.r_first + P.r_count; ++r) none = none && P.n_src[r] == 0;
        return launch_narrow_mu<SEG, MU>(P, algo, none ? 1 : rmax, st);
    }
    note_launch(0, "mrf_fwd_sweep_packed", blocks, idx ? 192 : 64, "%d,%d,%d,%d,%s,%d", SEG, MU, rmax, rmax == 4 ? 4 : (rmax == 8 ? 2 : 1),
                algo == MRF_TRWP ? "true" : "false", idx ? 2 : 0);
#define MRF_P(rm, d) \
    if (rmax == rm) { \
        if (idx) { \
            if (algo == MRF_TRWP) hipLaunchKernelGGL((mrf_fwd_sweep_packed<SEG, MU, rm, d, true, 2>), dim3(blocks), dim3(192), 0, st, P); \
            else hipLaunchKernelGGL((mrf_fwd_sweep_packed<SEG, MU, rm, d, false, 2>), dim3(blocks), dim3(192), 0, st, P); \
        } else { \
            if (algo == MRF_TRWP) hipLaunchKernelGGL((mrf_fwd_sweep_packed<SEG, MU, rm, d, true, 0>), dim3(blocks), dim3(64), 0, st, P); \
            else hipLaunchKernelGGL((mrf_fwd_sweep_packed<SEG, MU, rm, d, false, 0>), dim3(blocks), dim3(64), 0, st, P); \
        } \
        return hipGetLastError(); \
    }
    MRF_P(4, 4) MRF_P(8, 2) MRF_P(16, 1)
#undef MRF_P
    return hipErrorInvalidValue;
}

// Whether a launch is for the sweep divided among four wavefronts, as far as its 32-bit offsets reach, or for
// mrf_fwd_sweep_narrow (forward pass, divided / narrow, by wavefronts of scanlines):
// - 1,024: TRWP, 4 directions, K = 2: 6 x 512 x 512, 21 labels 1.73 / 2.14 ms, 4 x 512 x 512, 32 labels 1.76 / 2.04, 8 x 512 x 512, 16
//   labels 1.49 / 1.61, 8 labels 1.13 / 1.41; at 1,366 to 1,536 behind: 21 labels 2.86 / 2.62, 32 labels 2.91 / 2.36, 16 labels 2.49 / 2.29
// - ISGMR, 4 directions, K = 3: 1,026 wavefronts (512 x 1024, 21 labels) 0.91 / 1.29, 1,368 0.90 / 0.86; 1,536 with 32 labels 1.16 / 1.36,
//   with 16 0.71 / 0.70
// - eight directions, TRWP: 1,364 wavefronts with 21 labels 1.84 / 2.36, 2,044 with 32 labels 2.40 / 2.68
bool packed_divided(const MrfFwdParams &P, int seg, int algo, int rmax, long long scanlines)
{
    if (P.g.N * P.g.L > MRF_BUF_MOST) return false;
    if (g_tune_pack_idx == 2 || g_tune_pack_idx == 4 || g_tune_pack_idx == 5) return true;
    const long long waves = (scanlines + 64 / seg - 1) / (64 / seg);
    return g_tune_pack_idx == 0 && waves <= (rmax > 4 ? 2048 : (algo == MRF_ISGMR ? 1280 : 1024));
}

// and then, whether a scanline has a wavefront's lanes to itself (forward pass, one / several scanlines per wavefront):
// TRWP, 21 labels, K = 3: 256 scanlines 0.62 / 0.73 ms, 600 1.62 / 1.73, 768 0.75 / 0.80, 1,024 1.61 / 1.53; 16 labels 600 1.16 / 1.30,
// 1,024 1.26 / 1.25; 8 labels, where half of the lanes have no source label, 600 1.30 / 1.19.  ISGMR, all directions in one launch:
// 512 scanlines 0.127 / 0.138 with 16 labels, 1,024 0.178 / 0.160; 320 with 8 labels level
bool packed_one(int L, long long scanlines)
{
    if (g_tune_pack_idx >= 4) return g_tune_pack_idx == 4;
    return scanlines <= (L > 8 ? 768 : 320);
}

template <int SEG>
hipError_t launch_packed(const MrfFwdParams &P, int algo, int rmax, long long scanlines, hipStream_t st)
{
    if (packed_divided(P, SEG, algo, rmax, scanlines)) {
        const bool one = packed_one(P.g.L, scanlines);
        const int mu = (P.g.L + 3) / 4 * 4;
        if constexpr (SEG == 21) return launch_packed_divided<21, 1, 24>(P, algo, rmax, st);
        if constexpr (SEG == 16) {
            if (one) return launch_packed_divided<16, 4, 16>(P, algo, rmax, st);
            if (mu <= 8) return launch_packed_divided<16, 1, 8>(P, algo, rmax, st);
            return mu <= 12 ? launch_packed_divided<16, 1, 12>(P, algo, rmax, st) : launch_packed_divided<16, 1, 16>(P, algo, rmax, st);
        }
        if constexpr (SEG == 32) {
            if (one) return mu <= 24 ? launch_packed_divided<32, 2, 24>(P, algo, rmax, st) : launch_packed_divided<32, 2, 32>(P, algo, rmax, st);
            if (mu <= 24) return mu <= 20 ? launch_packed_divided<32, 1, 20>(P, algo, rmax, st) : launch_packed_divided<32, 1, 24>(P, algo, rmax, st);
            return mu <= 28 ? launch_packed_divided<32, 1, 28>(P, algo, rmax, st) : launch_packed_divided<32, 1, 32>(P, algo, rmax, st);
        }
    }
    // three scanlines of up to 21 labels per wavefront: always 24 source labels
    if constexpr (SEG == 21) {
        return launch_packed_mu<21, 24>(P, algo, rmax, scanlines, st);
    } else {
        // source labels per node: L rounded up to a multiple of four
        const int mu = (P.g.L + 3) / 4 * 4;
        if (mu <= SEG - 12) return launch_packed_mu<SEG, SEG - 12>(P, algo, rmax, scanlines, st);
        if (mu <= SEG - 8) return launch_packed_mu<SEG, SEG - 8>(P, algo, rmax, scanlines, st);
        if (mu <= SEG - 4) return launch_packed_mu<SEG, SEG - 4>(P, algo, rmax, scanlines, st);
        return launch_packed_mu<SEG, SEG>(P, algo, rmax, scanlines, st);
    }
}

hipError_t run_packed(MrfFwdParams &P, int seg, int algo, int rmax, long long scanlines, hipStream_t st)
{
    if (seg == 21) return launch_packed<21>(P, algo, rmax, scanlines, st);
    return seg == 16 ? launch_packed<16>(P, algo, rmax, scanlines, st) : launch_packed<32>(P, algo, rmax, scanlines, st);
}
#endif  // MRF_HAS_FWD_PACKED

#if MRF_HAS_FWD_DUO
template <int LP, int RMAX, int D, int NI>
hipError_t launch_window_duo(const MrfFwdParams &P, int algo, int tw, long long blocks, hipStream_t st)
{
    note_launch(0, "mrf_fwd_sweep_window_duo", blocks, 64 * (1 + NI), "%d,%d,%d,%s,%d,%d,false", LP, RMAX, D,
                algo == MRF_TRWP ? "true" : "false", tw, NI);
#define MRF_W(twv) \
    if (tw == twv) { \
        if (algo == MRF_TRWP) hipLaunchKernelGGL((mrf_fwd_sweep_window_duo<LP, RMAX, D, true, twv, NI, false>), dim3((unsigned)blocks), dim3(64 * (1 + NI)), 0, st, P); \
        else hipLaunchKernelGGL((mrf_fwd_sweep_window_duo<LP, RMAX, D, false, twv, NI, false>), dim3((unsigned)blocks), dim3(64 * (1 + NI)), 0, st, P); \
        return hipGetLastError(); \
    }
    MRF_W(2) MRF_W(4) MRF_W(8) MRF_W(12) MRF_W(16)
#undef MRF_W
    return hipErrorInvalidValue;
}

// value + loader + two index wavefronts (TRWP, up to three other directions)
template <int LP>
hipError_t launch_window_loader(const MrfFwdParams &P, int tw, long long blocks, hipStream_t st)
{
    note_launch(0, "mrf_fwd_sweep_window_duo", blocks, 256, "%d,4,%d,true,%d,2,true", LP, (LP <= 2 ? 4 : 2), tw);
#define MRF_W(twv) \
    if (tw == twv) { \
        hipLaunchKernelGGL((mrf_fwd_sweep_window_duo<LP, 4, (LP <= 2 ? 4 : 2), true, twv, 2, true>), dim3((unsigned)blocks), dim3(256), 0, st, P); \
        return hipGetLastError(); \
    }
    MRF_W(2) MRF_W(4) MRF_W(8) MRF_W(12) MRF_W(16)
#undef MRF_W
    return hipErrorInvalidValue;
}

hipError_t run_window_loader(MrfFwdParams &P, int tw, long long blocks, hipStream_t st)
{
    const int LPw = (P.g.L + 63) / 64;
    if (LPw == 1) return launch_window_loader<1>(P, tw, blocks, st);
    if (LPw == 2) return launch_window_loader<2>(P, tw, blocks, st);
    if (LPw == 3) return launch_window_loader<3>(P, tw, blocks, st);
    return launch_window_loader<4>(P, tw, blocks, st);
}

hipError_t run_window_duo(MrfFwdParams &P, int algo, int tw, int ni, int ms, long long blocks, hipStream_t st)
{
    const int LPw = (P.g.L + 63) / 64;
#define MRF_WCASE(lp) \
    if (LPw == lp && ms + 1 <= 4 && ni == 2) return launch_window_duo<lp, 4, (lp <= 2 ? 4 : 2), 2>(P, algo, tw, blocks, st); \
    if (LPw == lp && ms + 1 <= 4) return launch_window_duo<lp, 4, (lp <= 2 ? 4 : 2), 1>(P, algo, tw, blocks, st); \
    if (LPw == lp && ni == 2) return launch_window_duo<lp, 8, (lp <= 2 ? 2 : 1), 2>(P, algo, tw, blocks, st); \
    if (LPw == lp) return launch_window_duo<lp, 8, (lp <= 2 ? 2 : 1), 1>(P, algo, tw, blocks, st);
    MRF_WCASE(1) MRF_WCASE(2) MRF_WCASE(3) MRF_WCASE(4)
#undef MRF_WCASE
    return hipErrorInvalidValue;
}
#endif  // MRF_HAS_FWD_DUO

#if MRF_HAS_FWD_WINDOW
template <int LP, int RMAX, int D>
hipError_t launch_window(const MrfFwdParams &P, int algo, int tw, long long blocks, hipStream_t st)
{
    note_launch(0, "mrf_fwd_sweep_window", blocks, 64, "%d,%d,%d,%s,%d", LP, RMAX, D, algo == MRF_TRWP ? "true" : "false", tw);
#define MRF_W(twv) \
    if (tw == twv) { \
        if (algo == MRF_TRWP) hipLaunchKernelGGL((mrf_fwd_sweep_window<LP, RMAX, D, true, twv>), dim3((unsigned)blocks), dim3(64), 0, st, P); \
        else hipLaunchKernelGGL((mrf_fwd_sweep_window<LP, RMAX, D, false, twv>), dim3((unsigned)blocks), dim3(64), 0, st, P); \
        return hipGetLastError(); \
    }
    MRF_W(2) MRF_W(4) MRF_W(8) MRF_W(12) MRF_W(16)
#undef MRF_W
    return hipErrorInvalidValue;
}

// ISGMR sweeps that read one array only
template <int LP>
hipError_t launch_window_one(const MrfFwdParams &P, int tw, long long blocks, hipStream_t st)
{
    note_launch(0, "mrf_fwd_sweep_window", blocks, 64, "%d,1,4,false,%d", LP, tw);
#define MRF_W(twv) \
    if (tw == twv) { \
        hipLaunchKernelGGL((mrf_fwd_sweep_window<LP, 1, 4, false, twv>), dim3((unsigned)blocks), dim3(64), 0, st, P); \
        return hipGetLastError(); \
    }
    MRF_W(2) MRF_W(4) MRF_W(8) MRF_W(12) MRF_W(16)
#undef MRF_W
    return hipErrorInvalidValue;
}

// TRWP with nine to sixteen directions: up to fifteen message arrays per update
template <int LP>
hipError_t launch_window_many(const MrfFwdParams &P, int tw, long long blocks, hipStream_t st)
{
    // (prefetch two nodes deep where the registers allow: a node step otherwise waits a whole memory round trip)
    constexpr int D = LP <= 2 ? 2 : 1;
    note_launch(0, "mrf_fwd_sweep_window", blocks, 64, "%d,16,%d,true,%d", LP, D, tw);
#define MRF_W(twv) \
    if (tw == twv) { \
        hipLaunchKernelGGL((mrf_fwd_sweep_window<LP, 16, D, true, twv>), dim3((unsigned)blocks), dim3(64), 0, st, P); \
        return hipGetLastError(); \
    }
    MRF_W(2) MRF_W(4) MRF_W(8) MRF_W(12) MRF_W(16)
#undef MRF_W
    return hipErrorInvalidValue;
}

template <int RMAX, int D>
hipError_t launch_window_split(const MrfFwdParams &P, int algo, int tw, long long blocks, hipStream_t st)
{
    const unsigned threads = 64u * (unsigned)((P.g.L + 63) / 64);
    note_launch(0, "mrf_fwd_sweep_window_split", blocks, (int)threads, "%d,%d,%s,%d", RMAX, D, algo == MRF_TRWP ? "true" : "false", tw);
#define MRF_W(twv) \
    if (tw == twv) { \
        if (algo == MRF_TRWP) hipLaunchKernelGGL((mrf_fwd_sweep_window_split<RMAX, D, true, twv>), dim3((unsigned)blocks), dim3(threads), 0, st, P); \
        else hipLaunchKernelGGL((mrf_fwd_sweep_window_split<RMAX, D, false, twv>), dim3((unsigned)blocks), dim3(threads), 0, st, P); \
        return hipGetLastError(); \
    }
    MRF_W(2) MRF_W(8) MRF_W(16)
#undef MRF_W
    return hipErrorInvalidValue;
}

template <int RMAX, int D>
hipError_t launch_window_squad(const MrfFwdParams &P, int algo, int tw, int ni, long long blocks, hipStream_t st)
{
    const unsigned nwv = (unsigned)((P.g.L + 63) / 64);
    note_launch(0, "mrf_fwd_sweep_window_squad", blocks, (int)(64u * (nwv + ni)), "%d,%d,%s,%d,%d", RMAX, D,
                algo == MRF_TRWP ? "true" : "false", tw, ni);
#define MRF_W(twv, niv) \
    if (tw == twv && ni == niv) { \
        if (algo == MRF_TRWP) hipLaunchKernelGGL((mrf_fwd_sweep_window_squad<RMAX, D, true, twv, niv>), dim3((unsigned)blocks), dim3(64u * (nwv + niv)), 0, st, P); \
        else hipLaunchKernelGGL((mrf_fwd_sweep_window_squad<RMAX, D, false, twv, niv>), dim3((unsigned)blocks), dim3(64u * (nwv + niv)), 0, st, P); \
        return hipGetLastError(); \
    }
    MRF_W(2, 4) MRF_W(8, 4) MRF_W(16, 4) MRF_W(2, 8) MRF_W(8, 8) MRF_W(16, 8)
#undef MRF_W
    return hipErrorInvalidValue;
}

hipError_t run_window_split(MrfFwdParams &P, int algo, int tw, int ms, long long blocks, hipStream_t st)
{
    if (ms + 1 <= 4) return launch_window_split<4, 4>(P, algo, tw, blocks, st);
    return launch_window_split<8, 2>(P, algo, tw, blocks, st);
}

hipError_t run_window_squad(MrfFwdParams &P, int algo, int tw, int ni, int ms, long long blocks, hipStream_t st)
{
    if (ms + 1 <= 4) return launch_window_squad<4, 4>(P, algo, tw, ni, blocks, st);
    return launch_window_squad<8, 2>(P, algo, tw, ni, blocks, st);
}

hipError_t run_window(MrfFwdParams &P, int algo, int tw, int ms, long long blocks, hipStream_t st)
{
    const int LPw = (P.g.L + 63) / 64;
    if (ms + 1 <= 8) {
        P.NW = 1;
        // (nothing but the start term to read: the first iteration of ISGMR, and its later ones after
        // mrf_isgmr_presum; a deeper prefetch fits in the registers the other sources would take)
#define MRF_WCASE(lp) \
        if (LPw == lp && ms == 0 && algo == MRF_ISGMR) return launch_window_one<lp>(P, tw, blocks, st);
        MRF_WCASE(1) MRF_WCASE(2) MRF_WCASE(3) MRF_WCASE(4)
#undef MRF_WCASE
#define MRF_WCASE(lp) \
        if (LPw == lp && ms + 1 <= 4) return launch_window<lp, 4, (lp <= 2 ? 4 : 2)>(P, algo, tw, blocks, st); \
        if (LPw == lp) return launch_window<lp, 8, (lp <= 2 ? 2 : 1)>(P, algo, tw, blocks, st);
        MRF_WCASE(1) MRF_WCASE(2) MRF_WCASE(3) MRF_WCASE(4)
#undef MRF_WCASE
    }
    if (algo == MRF_TRWP && ms + 1 <= 16) {
        P.NW = 1;
        if (LPw == 1) return launch_window_many<1>(P, tw, blocks, st);
        if (LPw == 2) return launch_window_many<2>(P, tw, blocks, st);
        if (LPw == 3) return launch_window_many<3>(P, tw, blocks, st);
        if (LPw == 4) return launch_window_many<4>(P, tw, blocks, st);
    }
    return hipErrorInvalidValue;
}
#endif  // MRF_HAS_FWD_WINDOW

#if MRF_HAS_FWD_DENSE
template <int LP, int MCH, int RMAX, int D>
hipError_t launch_fwd(const MrfFwdParams &P, int algo, long long blocks, hipStream_t st)
{
    note_launch(0, "mrf_fwd_sweep", blocks, 64 * P.NW, "%d,%d,%d,%d,%s", LP, MCH, RMAX, D, algo == MRF_TRWP ? "true" : "false");
    constexpr int NWMAX = (64 * LP + MCH - 1) / MCH;
    const size_t lds = (size_t)NWMAX * NWMAX * MCH * sizeof(float) +
                       (NWMAX > 1 ? (size_t)2 * NWMAX * 64 * LP * sizeof(float2) : 0);
    if (algo == MRF_TRWP)
        hipLaunchKernelGGL((mrf_fwd_sweep<LP, MCH, RMAX, D, true>), dim3((unsigned)blocks), dim3(64 * P.NW), lds, st, P);
    else
        hipLaunchKernelGGL((mrf_fwd_sweep<LP, MCH, RMAX, D, false>), dim3((unsigned)blocks), dim3(64 * P.NW), lds, st, P);
    return hipGetLastError();
}

template <int LP, int RMAX, int D>
hipError_t launch_fwd_sliced(const MrfFwdParams &P, int algo, long long blocks, hipStream_t st)
{
    note_launch(0, "mrf_fwd_sweep_sliced", blocks, 64 * P.NW, "%d,%d,%d,%s", LP, RMAX, D, algo == MRF_TRWP ? "true" : "false");
    if (algo == MRF_TRWP)
        hipLaunchKernelGGL((mrf_fwd_sweep_sliced<LP, RMAX, D, true>), dim3((unsigned)blocks), dim3(64 * P.NW), 0, st, P);
    else
        hipLaunchKernelGGL((mrf_fwd_sweep_sliced<LP, RMAX, D, false>), dim3((unsigned)blocks), dim3(64 * P.NW), 0, st, P);
    return hipGetLastError();
}

template <int NW, int RMAX, int D>
hipError_t launch_fwd_halves(const MrfFwdParams &P, int algo, long long blocks, hipStream_t st)
{
    note_launch(0, "mrf_fwd_sweep_halves", blocks, 64 * NW, "%d,%d,%d,%s", NW, RMAX, D, algo == MRF_TRWP ? "true" : "false");
    constexpr int lds = mrf_fwd_halves_lds<NW>();
#define MRF_H_GO(...) \
    do { \
        if (lds > 64 * 1024) { \
            const hipError_t ea_ = hipFuncSetAttribute(reinterpret_cast<const void *>(&__VA_ARGS__), \
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds); \
            if (ea_ != hipSuccess) return ea_; \
        } \
        hipLaunchKernelGGL((__VA_ARGS__), dim3((unsigned)blocks), dim3(64 * NW), lds, st, P); \
    } while (0)
    if (algo == MRF_TRWP) MRF_H_GO(mrf_fwd_sweep_halves<NW, RMAX, D, true>);
    else MRF_H_GO(mrf_fwd_sweep_halves<NW, RMAX, D, false>);
#undef MRF_H_GO
    return hipGetLastError();
}

// source labels per wavefront: small enough that the slice of V fits in registers, large
// enough that at most 16 wavefronts share a node
// (33..64 labels: four wavefronts of 16 source labels while the launch leaves SIMD slots free, two of 32 from
// 2,048 scanlines on: 512 x 512, 64 labels, ISGMR 2.64 -> 2.02 ms; TRWP on 4 x 512 x 512 11.4 -> 8.2 ms, but on
// 1 x 512 x 512 4.5 against 5.2 ms)
int pick_mch(int L, int LP, bool many_sources, long long blocks)
{
    static const int allowed[4][5] = { {8, 16, 32, 0, 0}, {8, 12, 16, 24, 32}, {16, 24, 32, 48, 0}, {32, 0, 0, 0, 0} };
    int want = g_tune_mch;
    if (want <= 0) want = LP == 1 ? ((L <= 32 || blocks >= 2048) ? 32 : 16) : (LP == 2 ? 24 : 32);
    if (many_sources) want = (LP <= 2) ? (want < 16 ? 16 : (want == 24 || want == 12 ? 16 : want)) : 32;
    int best = 0;
    for (int i = 0; i < 5; ++i) {
        const int m = allowed[LP - 1][i];
        if (m == 0) continue;
        if (many_sources && m != 16 && m != 32) continue;
        if (best == 0 || mrf_iabs(m - want) < mrf_iabs(best - want)) best = m;
    }
    return best;
}

// Whether mrf_fwd_sweep_halves is ahead of the better of the other two dense sweeps (33..128 labels; forward pass, K = 2 unless
// noted, others / halves in ms, or halves over others).  Its node step is the shorter one nearly everywhere, its start the longer one (a
// table in LDS): so on grids with a side of more than 40 the mean length of the launch's scanlines decides, and the longest one where the
// launch lasts about as long as that takes by itself.
// - up to 64 labels, TRWP, up to four arrays, one direction; 16 / 24 / 40 / 64 nodes per scanline: 512 scanlines 1.10 / 1.05 / 1.01 / 1.0;
//   1,024, 36 labels 1.0 / 0.98 / 0.99 / 0.97, 64 labels 0.93 / 0.91 / 0.90 / 0.86; 3,072 1.06 / 1.02 / 0.98 / 0.91; 4,096 1.09 / 1.06 / 1.04 / 0.98.
//   1,536 are as many as the machine holds of it at once: 0.83 / 0.83 / 0.82 / 0.75, with 8 nodes 0.93; 1,792 1.02 / 1.01 / 0.98 / 0.92.  2,048
//   are as many as it holds of the others, which take two wavefronts for each from there on: 1.2 / 1.18 / 1.15 / 1.11; 2,032 and 2,052
//   scanlines of 64 nodes 0.94 and 0.91; 8 x 512 x 512 5.39 / 4.80
// - the same with more arrays, 8 directions, K = 1: 8 x 256 x 256, 40 labels 3.04 / 2.81, 12 x 256 x 256 4.58 / 3.71, 64 labels 4.84 / 4.02, 4 x
//   512 x 512 6.36 / 5.80; 32 x 64 x 64 level; 16 directions 7.71 / 6.74
// - up to 64 labels, ISGMR: 256 x 256, 40 labels 0.461 / 0.386, 384 x 384 0.860 / 0.647, 512 x 512 level, 600 x 600 2.21 / 1.64, 64 labels 2.24 /
//   1.66; images of 48 x 48, 8,064 scanlines 0.95, 8 directions 0.98; 64 images of 20 x 64 level, 8 directions (mean 20) 0.85 / 0.89; 30 of 8 x
//   400 0.67 / 0.56, 8 directions 1.11 / 1.27; 50 of 5 x 41 0.090 / 0.098
// - 65..96 labels: 0.65 to 0.8 from 24 nodes on, at 8 nodes 72 labels level, 96 labels 0.9; 492 columns of 5 nodes 72 labels 1.07, 96 labels
//   0.93, diagonals of 5 x 41 0.114 / 0.178; 50 images of 5 x 41, ISGMR, 8 directions 0.351 / 0.362; 30 of 8 x 400, TRWP, diagonals 2.55 / 1.45
// - 97..128 labels, TRWP: 8 / 16 / 24 / 64 nodes 1.15 / 1.0 / 0.92 / 0.83, whatever the number of scanlines.  ISGMR, where a compute unit holds
//   two workgroups: images of 48 x 48, 960 / 3,072 / 8,064 scanlines 0.91 / 1.02 / 1.03, of 64 x 64 0.89 / 0.97 / 1.0, 8 directions (mean 43) 764 /
//   3,056 / 9,168 scanlines 0.94 / 0.96 / 1.03, of 96 x 96 8,064 scanlines 0.96; 4 of 16 x 1000 2.30 / 1.61, 8 directions 2.41 / 2.86
// On smaller grids as many scanlines as share the cost of its table decide (4 images of 16 x 16, ISGMR, K = 3: 36 labels 44 / 49 us, 128
// labels level; 16 images, TRWP, 36 labels 175 / 193; 28 x 40, K = 3, level up to 64 labels), and 65..96 labels, where the others leave lanes
// idle (28 x 40, 80 labels, TRWP 0.50 / 0.37 ms).
bool chunk_minima_ahead(const MrfFwdParams &P, int algo, int rmax, long long blocks)
{
    const int L = P.g.L;
    const bool trwp = algo == MRF_TRWP;
    if (P.g.H > 40 || P.g.W > 40) {
        const long long nodes = P.g.N * P.r_count, mean = nodes / blocks, longest = longest_scanline(P.g, P.r_first, P.r_count);
        const long long beside = L > 96 ? 256 : (longest > 64 ? 1024 : 512);      // scanlines that the machine sweeps beside the longest
        if (!trwp && longest > 40 && longest * beside >= nodes) return true;
        if (L > 96) return mean >= (trwp ? 16 : (blocks <= 1024 ? 24 : (blocks <= 4096 ? 40 : 56)));
        if (L > 64) return mean >= (trwp ? 5 : 7) || (trwp && blocks >= 4096);
        if (!trwp || rmax > 4) return mean >= 24;
        if (blocks == 2048) return false;
        if (blocks <= 512 || blocks > 3072) return mean >= (blocks <= 512 ? 40 : 48);
        return mean >= (blocks > 1024 && blocks <= 1536 ? 8 : (L > 48 && blocks < 2048 ? 16 : 24));
    }
    const bool middling = blocks > 512 && blocks < 1024;
    if (L <= 64) {
        if (rmax > 4) return blocks > 512;
        if (algo == MRF_TRWP) return L > 48 && middling;
        return blocks > (L > 48 ? 1024 : 2048) && blocks <= 3072;
    }
    if (L <= 96) return !(algo == MRF_TRWP && rmax <= 4 && L <= 72 && middling);
    return (P.g.H > 32 || P.g.W > 32) && (algo == MRF_TRWP || blocks <= 512);
}

hipError_t run_dense(MrfFwdParams &P, int algo, long long blocks, hipStream_t st)
{
    const bool generic = P.rho_e != nullptr;
    const int L = P.g.L;
    const int LP = (L + 63) / 64;
    int max_src = 0;
    for (int r = P.r_first; r < P.r_first + P.r_count; ++r)
        if (P.n_src[r] > max_src) max_src = P.n_src[r];
    const int rmax = (max_src + 1 <= 4) ? 4 : ((max_src + 1 <= 8) ? 8 : 16);
    // 33..128 labels: chunk minima where they are ahead, as far as the 32-bit offsets reach
    const bool halves_fit = L > 32 && L <= 128 && P.g.N * L * P.g.R <= MRF_BUF_MOST && !generic && !P.sgm_std && g_tune_mch == 0;
    if (halves_fit && (g_tune_dense_sliced == 3 || (g_tune_dense_sliced == 0 && chunk_minima_ahead(P, algo, rmax, blocks)))) {
        const int nw = (L + 31) / 32;
        P.NW = nw;
        // 65..96 labels and more than 512 scanlines under way at once (a diagonal's are of any length: nodes by the longest): half the
        // nodes loaded ahead, which leaves registers for four workgroups on a compute unit instead of two.  (Forward pass, TRWP, 96
        // labels, four / two nodes ahead: 3 x 256 x 256, K = 2 2.91 / 2.06 ms, 2 x 256 x 512 3.37 / 2.80, 6 x 256 x 256, K = 1 2.58 / 1.97; eight
        // directions, two / one, 2 x 256 x 512, K = 1 3.58 / 3.01, but 256 x 512, K = 5, whose diagonals are 767 scanlines, half of them short,
        // 10.6 / 10.8.  ISGMR level to 2 % ahead.)
        long long at_once = 0;
        for (int r = P.r_first; r < P.r_first + P.r_count; ++r) at_once += P.g.N / longest_scanline(P.g, r);
        const bool crowded = nw == 3 && at_once > 512;
#define MRF_HCASE(n) \
        if (nw == n && rmax == 4) return launch_fwd_halves<n, 4, 4>(P, algo, blocks, st); \
        if (nw == n && rmax == 8) return launch_fwd_halves<n, 8, 2>(P, algo, blocks, st); \
        if (nw == n && rmax == 16) return launch_fwd_halves<n, 16, 1>(P, algo, blocks, st);
        if (crowded && rmax == 4) return launch_fwd_halves<3, 4, 2>(P, algo, blocks, st);
        if (crowded && rmax == 8) return launch_fwd_halves<3, 8, 1>(P, algo, blocks, st);
        MRF_HCASE(2) MRF_HCASE(3) MRF_HCASE(4)
#undef MRF_HCASE
    }
    // more than 128 labels: every wavefront owns 32 of them (unless a tuning knob or a per-edge variant asks
    // for the sweep in which every wavefront does the O(L) work of the whole node)
    // What follows for 65..128 labels decides where the sweep above is not taken, by its rule, its offsets or knob 16:
    // (where the work outside the candidates is large: many source arrays, or a launch that
    // fills the machine several times over; else three wavefronts of 32 source labels are no faster than four
    // of 24: measured at 96 labels, 256 x 512, per iteration: TRWP with 8 directions 5.70 -> 4.01 ms, with 16
    // 15.1 -> 8.8 ms, ISGMR with 16 directions 4.12 -> 3.74 ms, but TRWP with 4 directions 1.81 -> 1.96 ms)
    // (from 97 labels on the other sweep needs five or six wavefronts of 24 source labels: 256 x 256, 128 labels,
    // ISGMR 3.80 -> 2.03 ms, TRWP 4.1 -> 3.8 ms; at 72 and 80 labels the two are level for ISGMR and this one is
    // behind for TRWP)
    if ((LP >= 3 || (LP == 2 && (g_tune_dense_sliced == 2 || rmax >= 8 || blocks >= 4096 || L > 96))) && !generic && !P.sgm_std && g_tune_mch == 0 && g_tune_dense_sliced != 1) {
        P.NW = (L + 31) / 32;
#define MRF_SCASE(lp) \
        if (LP == lp && rmax == 4) return launch_fwd_sliced<lp, 4, 4>(P, algo, blocks, st); \
        if (LP == lp && rmax == 8) return launch_fwd_sliced<lp, 8, 2>(P, algo, blocks, st); \
        if (LP == lp && rmax == 16) return launch_fwd_sliced<lp, 16, 1>(P, algo, blocks, st);
        MRF_SCASE(2) MRF_SCASE(3) MRF_SCASE(4)
#undef MRF_SCASE
    }
    const int mch = pick_mch(L, LP, rmax > 4, blocks);
    P.NW = (L + mch - 1) / mch;
    // prefetch depth: as deep as the register file allows next to the slice of V
#define MRF_CASE(lp, m) \
    if (LP == lp && mch == m && rmax == 4) return launch_fwd<lp, m, 4, (lp <= 2 ? 4 : 2)>(P, algo, blocks, st);
#define MRF_CASE_MANY(lp, m) \
    if (LP == lp && mch == m && rmax == 8) return launch_fwd<lp, m, 8, (lp <= 2 ? 2 : 1)>(P, algo, blocks, st); \
    if (LP == lp && mch == m && rmax == 16) return launch_fwd<lp, m, 16, 1>(P, algo, blocks, st);
    MRF_CASE(1, 8) MRF_CASE(1, 16) MRF_CASE(1, 32)
    MRF_CASE(2, 8) MRF_CASE(2, 12) MRF_CASE(2, 16) MRF_CASE(2, 24) MRF_CASE(2, 32)
    MRF_CASE(3, 16) MRF_CASE(3, 24) MRF_CASE(3, 32) MRF_CASE(3, 48)
    MRF_CASE(4, 32)
    MRF_CASE_MANY(1, 16) MRF_CASE_MANY(1, 32) MRF_CASE_MANY(2, 16) MRF_CASE_MANY(2, 32)
    MRF_CASE_MANY(3, 32) MRF_CASE_MANY(4, 32)
#undef MRF_CASE
#undef MRF_CASE_MANY
    return hipErrorInvalidValue;
}
#endif  // MRF_HAS_FWD_DENSE

#if MRF_HAS_FWD
// pairwise potentials per edge (L <= 64): more than 32 labels fetch the table in two halves of ceil(L/2) rows
// (rounded up to a multiple of four)
hipError_t launch_edge(const MrfFwdParams &P, int algo, long long blocks, hipStream_t st)
{
    int ms = 0;
    for (int r = P.r_first; r < P.r_first + P.r_count; ++r)
        if (P.n_src[r] > ms) ms = P.n_src[r];
    const int rmax = (ms + 1 <= 4) ? 4 : ((ms + 1 <= 8) ? 8 : 16);
    const int L = P.g.L;
    const dim3 grid((unsigned)blocks), block(64);
    // up to 32 labels: the lanes in groups that share the source labels, in launches of every size (one label per lane and two halves of a
    // table / this, forward pass, K = 2, 4 directions: ISGMR 32 x 48, 5 labels 0.051 / 0.047 ms, 32 labels 0.126 / 0.059; 256 x 256, 8 labels
    // 0.272 / 0.205, 17 labels 0.569 / 0.274; 2 x 256 x 512, 24 labels 1.51 / 1.29, 32 labels 2.24 / 1.95; TRWP 256 x 256, 32 labels 2.54 / 1.02;
    // K = 1, 4 x 512 x 512, 5 labels 1.64 / 1.11)
    if (L <= 32) {
        // (accesses of 1 KB per table: none for up to 8 labels, whose table is one of 256 bytes)
        const int seg = L <= 16 ? 16 : 32, rows = L <= 8 ? 2 : (L <= 16 ? 4 : (L <= 24 ? 12 : 16)), nt = L <= 8 ? 0 : (L * L + 255) / 256;
        note_launch(0, "mrf_fwd_sweep_edge_groups", blocks, 64, "%d,%d,%d,%d,%s", seg, rows, nt, rmax, algo == MRF_TRWP ? "true" : "false");
#define MRF_E(sg, hr, n, rm) \
        if (seg == sg && rows == hr && nt == n && rmax == rm) { \
            if (algo == MRF_TRWP) hipLaunchKernelGGL((mrf_fwd_sweep_edge_groups<sg, hr, n, rm, true>), grid, block, 0, st, P); \
            else hipLaunchKernelGGL((mrf_fwd_sweep_edge_groups<sg, hr, n, rm, false>), grid, block, 0, st, P); \
            return hipGetLastError(); \
        }
#define MRF_EH(sg, hr, n) MRF_E(sg, hr, n, 4) MRF_E(sg, hr, n, 8) MRF_E(sg, hr, n, 16)
        MRF_EH(16, 2, 0) MRF_EH(16, 4, 1) MRF_EH(32, 12, 2) MRF_EH(32, 12, 3) MRF_EH(32, 16, 3) MRF_EH(32, 16, 4)
#undef MRF_EH
#undef MRF_E
    }
    note_launch(0, "mrf_fwd_sweep_edge", blocks, 64, "%d,%d,%s", (L + 7) / 8 * 4, rmax, algo == MRF_TRWP ? "true" : "false");
    if (L > 64) return hipErrorInvalidValue;
#define MRF_E(half, rm) \
    if (L <= 2 * half && rmax == rm) { \
        if (algo == MRF_TRWP) hipLaunchKernelGGL((mrf_fwd_sweep_edge<half, rm, true>), grid, block, 0, st, P); \
        else hipLaunchKernelGGL((mrf_fwd_sweep_edge<half, rm, false>), grid, block, 0, st, P); \
        return hipGetLastError(); \
    }
#define MRF_EH(half) MRF_E(half, 4) MRF_E(half, 8) MRF_E(half, 16)
    MRF_EH(20) MRF_EH(24) MRF_EH(28) MRF_EH(32)
#undef MRF_EH
#undef MRF_E
    return hipErrorInvalidValue;
}

hipError_t dispatch_fwd(MrfFwdParams &P, int algo, int tw, long long blocks, hipStream_t st)
{
    // few labels: several scanlines per wavefront (dense evaluation), unless the launch is so
    // small that it is latency bound and a truncated model can use the shorter window step
    // (up to 16 labels the window templates evaluate 15 candidates, no fewer than the dense step)
    if (P.Te) return launch_edge(P, algo, blocks, st);
    // (TRW coefficients per edge: the two one-wavefront-per-scanline sweeps read them)
    const bool generic = P.rho_e != nullptr;
    if (P.sgm_std) tw = 0;         // standard SGM: the dense sweep is the one that knows it
    if (!P.sgm_std && !generic && P.g.L <= 32 && g_tune_pack != 1 && (g_tune_pack == 2 || tw == 0 || blocks >= 1024 || P.g.L <= 16)) {
        int ms = 0;
        for (int r = P.r_first; r < P.r_first + P.r_count; ++r)
            if (P.n_src[r] > ms) ms = P.n_src[r];
        const int rmax = (ms + 1 <= 4) ? 4 : ((ms + 1 <= 8) ? 8 : 16);
        P.NW = 1;
        // 17..21 labels (the 21 classes of the segmentation shape): three scanlines per wavefront once the
        // launch has wavefronts to spare, else two or one (a latency-bound launch gains nothing from fewer wavefronts:
        // TRWP, 512 x 512 images, K = 3, three / two scanlines per wavefront: 1,024 scanlines 1.64 / 1.53 ms, 1,536 1.69 / 1.80)
        if (P.g.L > 16 && P.g.L <= 21 && g_tune_pack3 != 1 && (g_tune_pack3 == 2 || blocks >= 1280))
            return run_packed(P, 21, algo, rmax, blocks, st);
        return run_packed(P, P.g.L <= 16 ? 16 : 32, algo, rmax, blocks, st);
    }
    if (tw > 0) {
        const int LPw = (P.g.L + 63) / 64;
        int ms = 0;
        for (int r = P.r_first; r < P.r_first + P.r_count; ++r)
            if (P.n_src[r] > ms) ms = P.n_src[r];
        // few scanlines in the launch and many labels: spread each node step over one
        // wavefront per 64 labels
        // (measured with four directions: window 16, 192 or 256 labels, ISGMR with 1,536 to 3,072 scanlines: 2.2
        // against 3.8 ms, 2.6 against 5.4 ms, 5.0 against 7.2 ms, 7.3 against 8.2 ms for the next best layout; window
        // 8, 192 or 256 labels: the value/index pair is ahead)
        const int tws = tw == 4 ? 8 : (tw == 12 ? 16 : tw);      // (these two layouts exist for windows 2, 8 and 16: a wider window is as exact)
        const bool split_ok = !generic && LPw > 1 && g_tune_split != 1 && ms + 1 <= 8;
        const bool split = split_ok && (g_tune_split == 2 || (LPw >= 3 && tws >= 16 && blocks * LPw <= 16384));
        // Those value wavefronts with a loader and index wavefronts beside them (forward pass, against the better of the
        // value/index pair and the split layout):
        // - window 16 (and 12 beyond 128 labels): TRWP 256 x 256, 256 labels, K = 2 1.16 / 1.65 ms with index wavefronts alone beside
        //   them and every neighbour read by itself; K = 1: 600 scanlines 3.06 / 3.32, with 128 labels 2.27 / 2.92, 700 with 200 labels
        //   4.28 / 4.11; ISGMR 512 scanlines, K = 2, 256 labels 0.25 / 0.34, 128 labels 0.16 / 0.20
        // - window 8 beyond 192 labels: TRWP, K = 2, 256 scanlines 1.03 / 1.32, 512 1.76 / 2.17, 600 level; eight directions, K = 1, 655
        //   scanlines 1.75 / 1.95; ISGMR 512 scanlines 0.185 / 0.223, 600 0.335 / 0.320
        // - window 8, 129..192 labels, where the pair has a label slot less: level to 256 scanlines (TRWP, K = 2, 256 x 256: 0.962 / 0.972),
        //   behind beyond (256 and 512 scanlines, 192 labels 1.67 / 1.59; 300 and 600 2.52 / 2.32; ISGMR 512 scanlines, 160 labels 0.187 /
        //   0.165); ahead with more source arrays (eight directions, 160 labels: to 383 scanlines 1.45 / 1.62, to 629 2.95 / 3.14)
        // - window 8, 65..128 labels: behind the pair with its loader (TRWP, up to three source arrays: 0.61 / 0.54), ahead with more
        //   (eight directions: 499 scanlines 1.58 / 1.79, 767 1.32 / 1.17) and for ISGMR to 256 scanlines (65.6 / 68.2 us)
        // (eight beside the values where a scanline has a compute unit to itself and more than 128 labels: 1.16 / 1.36 ms at 256
        // scanlines of 256 labels, but 1.75 / 1.44 at 512 of 96)
        const bool many = ms + 1 > 4;
        const long long squad_max = tw == 16 || (tw == 12 && LPw >= 3) ? 640
                                    : (tw != 8 ? 0 : (LPw >= 3 ? (many ? 656 : (LPw >= 4 ? 512 : 256)) : (many ? 512 : (algo == MRF_ISGMR ? 256 : 0))));
        const bool squad = split_ok && g_tune_squad != 1 && (long long)P.g.H * P.g.W * P.g.L <= MRF_BUF_MOST &&
                           ((g_tune_split == 2 && g_tune_squad == 2) || (g_tune_split == 0 && g_tune_duo == 0 && blocks <= squad_max));
        if (squad) {
            P.NW = LPw;
            const int ni = (g_tune_squad_ni == 4 || g_tune_squad_ni == 8) ? g_tune_squad_ni : (LPw >= 3 && blocks <= 256 ? 8 : 4);
            return run_window_squad(P, algo, tws, ni, ms, blocks, st);
        }
        if (split) {
            P.NW = LPw;
            return run_window_split(P, algo, tws, ms, blocks, st);
        }
        // few scanlines: a second wavefront per scanline takes the argmin tables and the
        // stores off the dependency chain
        // (its addressing wants a node step times L in 32 bits)
        bool step_fits = true;
        for (int r = P.r_first; r < P.r_first + P.r_count; ++r) {
            const long long st = ((long long)mrf_iabs(P.g.dh[r]) * P.g.W + mrf_iabs(P.g.dw[r])) * P.g.L;
            if (st > 0x7fffffffLL) step_fits = false;
        }
        // (a second wavefront per scanline pays while the scanlines alone leave SIMD slots free; measured on
        // square grids with four directions: ISGMR at 2,048 scanlines 1.41 ms with it against 1.52 ms without,
        // at 2,560 scanlines 2.74 against 2.21 ms with 96 labels but 1.27 against 1.37 ms with 40; TRWP at 2,048
        // scanlines 4.92 against 4.32 ms)
        const long long duo_max = algo == MRF_TRWP ? 1536 : (LPw == 1 ? 3072 : 2048);
        const bool duo = !generic && step_fits && g_tune_duo != 1 && (g_tune_duo == 2 || blocks <= duo_max);
        if (ms + 1 <= 8 && duo) {
            P.NW = 1;
            // two index wavefronts while the launch is far from filling the machine
            const int ni = g_tune_duo_ni ? g_tune_duo_ni : (blocks <= 1536 ? 2 : 1);
            // TRWP launches that leave SIMDs idle: a loader wavefront in front of the value wavefront
            if (algo == MRF_TRWP && ms + 1 <= 4 && ni == 2 && g_tune_loader != 1 &&
                (g_tune_loader == 2 || blocks <= 512))
                return run_window_loader(P, tw, blocks, st);
            return run_window_duo(P, algo, tw, ni, ms, blocks, st);
        }
        if (ms + 1 <= 8 || (algo == MRF_TRWP && ms + 1 <= 16)) {
            P.NW = 1;
            return run_window(P, algo, tw, ms, blocks, st);
        }
    }
    return run_dense(P, algo, blocks, st);
}

// Which message arrays enter h at the previous node, in the order they are summed, for the
// sweep of direction r.  live: bit d set if array d holds data (else it is all zero and is
// skipped: adding 0 changes nothing).
void fill_sources(MrfFwdParams &P, int algo, int r, unsigned live)
{
    const int R = P.g.R, rm = P.g.opp[r];
    int n = 0, npre = 0, rmslot = -1;
    for (int d = 0; d < R; ++d) {
        if (d == r || !((live >> d) & 1u)) continue;
        if (algo == MRF_ISGMR && d == rm) continue;       // Eq. isgmr excludes r and r-
        if (algo == MRF_TRWP && d < r) ++npre;            // Eq. trwp sums all d in index order
        if (d == rm) rmslot = n;
        P.src_dir[r][n++] = d;
    }
    P.n_pre[r] = npre;
    P.n_src[r] = n;
    P.rm_slot[r] = rmslot;
}

hipError_t fill(float *dst, long long n, float v, hipStream_t st);

int run_forward(const mrf_problem *pr, int algo, float *cost, uint8_t *labels, uint8_t *p, uint8_t *q,
                float *messages, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    int rc = check_problem(pr, algo, true);
    if (rc != MRF_OK) return rc;
    if (!cost || !p || !q) return MRF_ERR_NULL_POINTER;
    const size_t need = mrf_workspace_bytes(pr, algo, 0);
    if (need > 0 && (!workspace || workspace_bytes < need)) return workspace ? MRF_ERR_WORKSPACE_TOO_SMALL : MRF_ERR_NULL_POINTER;
    hipStream_t st = (hipStream_t)hip_stream;

    MrfFwdParams P;
    memset(&P, 0, sizeof(P));
    fill_geom(pr, P.g);
    const long long N = P.g.N;
    const int R = pr->R, L = pr->L, K = pr->K;
    P.unary = pr->unary; P.V = pr->pairwise;
    for (int r = 0; r < R; ++r) P.rho[r] = (algo == MRF_TRWP && pr->rho) ? pr->rho[r] : 1.0f;
    P.rho_e = (algo == MRF_TRWP) ? pr->rho_edge : nullptr;
    P.Te = pr->pairwise_edge;
    P.sgm_std = pr->sgm_standard ? 1 : 0;

    // workspace: [scalars 256 B][messages A][messages B (ISGMR only)]
    float *scal = (float *)workspace;
    float *bufA = (float *)((char *)workspace + kAlign);
    float *bufB = (float *)((char *)workspace + kAlign + msg_bytes(pr));
    // header: the scalar weight (read through the same vector loads as per-edge weights) and the fault word
    { const hipError_t e_ = init_header(workspace, pr->edge_weight_scalar, st); if (e_ != hipSuccess) return hip_fail(e_, "init_header"); }
    P.fault = (int *)((char *)workspace + kFaultOffset);
    P.spin_limit = spin_limit();
    if (pr->edge_weight) { P.w = pr->edge_weight; P.w_mul = 1; }
    else { P.w = scal; P.w_mul = 0; }
    const size_t pk = (size_t)R * N * L, qk = (size_t)R * N;
    float *final_m = nullptr;
    const int tw = window_width(pr);

    mark(g_ev_start, st);
    if (algo == MRF_ISGMR) {
        // all directions of one iteration in one launch; messages ping-pong between two buffers
        P.r_first = 0; P.r_count = R;
        long long blocks = 0;
        for (int r = 0; r < R; ++r) { P.blk_begin[r] = blocks; blocks += (long long)pr->B * P.g.nscan[r]; }
        P.blk_begin[R] = blocks;
        // Six directions or more: one streaming pass per iteration sums what the previous iteration left at
        // every node, once per pair of opposite directions (mrf_isgmr_presum), and the sweeps read that one
        // array like a unary.  The messages of iteration k - 1 are dead once it has run, so the sweeps write
        // over them and the second buffer holds the sums.
        const long long NL = N * L;
        const bool presum = K > 1 && !pr->sgm_standard && g_tune_isgmr_presum != 1 && (g_tune_isgmr_presum == 2 || R >= 6);
        MrfPresumParams S;
        memset(&S, 0, sizeof(S));
        S.NL = NL; S.R = R; S.unary = pr->unary; S.m = bufA; S.out = bufB;
        for (int r = 0; r < R; ++r) S.opp[r] = P.g.opp[r];
        const bool svec = (NL % 4 == 0) && (((uintptr_t)pr->unary | (uintptr_t)bufA | (uintptr_t)bufB) % 16 == 0);
        long long sblocks = ((svec ? NL / 4 : NL) + 255) / 256;
        if (sblocks > 32768) sblocks = 32768;
        if (sblocks < 1) sblocks = 1;
        for (int k = 0; k < K; ++k) {
            if (presum) {
                P.m_in = bufA; P.m_out = bufA;
                P.unary = (k == 0) ? pr->unary : bufB;
                for (int r = 0; r < R; ++r) {
                    fill_sources(P, algo, r, 0u);
                    P.unary_slab[r] = (int)((k == 0) ? 0 : ((P.g.opp[r] >= 0 && P.g.opp[r] < r) ? P.g.opp[r] : r));
                }
                if (k > 0) {
                    const dim3 sg((unsigned)sblocks), sb(256);
                    if (R <= 8 && svec) hipLaunchKernelGGL((mrf_isgmr_presum<8, 4>), sg, sb, 0, st, S);
                    else if (R <= 8) hipLaunchKernelGGL((mrf_isgmr_presum<8, 1>), sg, sb, 0, st, S);
                    else if (svec) hipLaunchKernelGGL((mrf_isgmr_presum<16, 4>), sg, sb, 0, st, S);
                    else hipLaunchKernelGGL((mrf_isgmr_presum<16, 1>), sg, sb, 0, st, S);
                    { const hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return hip_fail(e_, "hipGetLastError"); }
                }
            } else {
                P.m_in = (k & 1) ? bufB : bufA;      // written by iteration k-1 (unused when k = 0)
                P.m_out = (k & 1) ? bufA : bufB;
                for (int r = 0; r < R; ++r) fill_sources(P, algo, r, k == 0 ? 0u : 0xffffffffu);
            }
            P.p = p + (size_t)k * pk;
            P.q = q + (size_t)k * qk;
            { const hipError_t e_ = dispatch_fwd(P, algo, tw, blocks, st); if (e_ != hipSuccess) return hip_fail(e_, "dispatch_fwd"); }
            if (presum && k > 0) {
                const size_t used = strlen(g_last_launch[0]);
                snprintf(g_last_launch[0] + used, sizeof(g_last_launch[0]) - used, " after mrf_isgmr_presum<%d,%d>", R <= 8 ? 8 : 16, svec ? 4 : 1);
            }
            final_m = P.m_out;
        }
    } else {
        // one launch per (iteration, direction); messages updated in place
        P.m_in = bufA; P.m_out = bufA;
        for (int k = 0; k < K; ++k) {
            for (int r = 0; r < R; ++r) {
                P.r_first = r; P.r_count = 1;
                P.blk_begin[0] = 0;
                const long long blocks = (long long)pr->B * P.g.nscan[r];
                P.blk_begin[1] = blocks;
                // in the first iteration the directions after r have not been written yet: they read as 0
                fill_sources(P, algo, r, k == 0 ? ((1u << r) - 1u) : 0xffffffffu);
                P.p = p + (size_t)k * pk;
                P.q = q + (size_t)k * qk;
                { const hipError_t e_ = dispatch_fwd(P, algo, tw, blocks, st); if (e_ != hipSuccess) return hip_fail(e_, "dispatch_fwd"); }
            }
        }
        final_m = bufA;
    }
    mark(g_ev_stop, st);

    MrfAggParams A;
    A.N = N; A.L = L; A.R = R; A.no_unary = pr->sgm_standard ? 1 : 0;
    A.unary = pr->unary; A.m = final_m; A.cost = cost; A.labels = labels;
    long long ablocks = (N + 3) / 4;
    if (ablocks > 65536) ablocks = 65536;
    if (R <= 4) hipLaunchKernelGGL(mrf_aggregate<4>, dim3((unsigned)ablocks), dim3(256), 0, st, A);
    else if (R <= 8) hipLaunchKernelGGL(mrf_aggregate<8>, dim3((unsigned)ablocks), dim3(256), 0, st, A);
    else hipLaunchKernelGGL(mrf_aggregate<16>, dim3((unsigned)ablocks), dim3(256), 0, st, A);
    { const hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return hip_fail(e_, "hipGetLastError"); }
    if (messages) {
        const hipError_t e_ = hipMemcpyAsync(messages, final_m, pk * sizeof(float), hipMemcpyDeviceToDevice, st);
        if (e_ != hipSuccess) return hip_fail(e_, "hipMemcpyAsync");
    }
    return MRF_OK;
}

#endif  // MRF_HAS_FWD

#if MRF_HAS_BWD_CHAIN
template <int LP, int NS, int D>
hipError_t launch_bwd_chain(const MrfBwdParams &P, int ni, bool vg, hipStream_t st)
{
    const dim3 grid((unsigned)P.total_scanlines);
    const bool gv = P.gV != nullptr;
    const bool edge = P.edge != 0;                        // (per-edge tables: a kernel of its own)
    const bool gs = edge || (LP <= 2 && P.gstore);        // the helpers store the node gradients (no tables, no V)
    if (gs) vg = true;
    const bool hot = P.hot_label && (gs || !((LP == 1 && gv) || vg));
    const bool far = chain_far(P.g, gs && !edge);
    note_launch(1, "mrf_bwd_sweep_chain", P.total_scanlines, 64 * (1 + ni), "%d,%d,%d,%d,%s,%s,%s%s", LP, NS, D, ni,
                (!(LP == 1 && gv) && vg) ? "true" : "false", ((LP == 1 && gv) || gs) ? "true" : "false", hot ? "true" : "false",
                edge ? ",true" : (LP == 1 && gv && !P.gw ? (far ? ",false,true,false" : ",false,false,false") : (far ? ",false,true" : "")));
    if (gv && (LP != 1 || P.total_scanlines > grad_slots(P.g.L))) return hipErrorInvalidValue;
    MrfChainParams C;
    memset(&C, 0, sizeof(C));
    C.B = P.g.B; C.H = P.g.H; C.W = P.g.W; C.L = P.g.L; C.w_mul = P.w_mul; C.r_first = P.r_first; C.r_count = P.r_count; C.N = P.g.N;
    int most = 0;
    for (int ri = 0; ri < P.r_count; ++ri) {
        const int n = P.n_src[P.r_first + ri] + (P.use_gc ? 1 : 0);
        most = n > most ? n : most;
    }
    C.src_pitch = P.r_count == 1 ? MRF_MAXR : most;
    if (most > NS || most * P.r_count > MRF_MAXR) return hipErrorInvalidValue;
    for (int ri = 0; ri < P.r_count; ++ri) {
        const int r = P.r_first + ri, n = P.n_src[r];
        C.begin[ri] = (int)P.blk_begin[ri];
        C.dh[ri] = P.g.dh[r]; C.dw[ri] = P.g.dw[r]; C.nscan[ri] = P.g.nscan[r];
        C.carry_scale[ri] = P.carry_scale[r];
        for (int c = 0; c < n; ++c) {
            const int k = ri * C.src_pitch + c;
            C.src[k] = P.src_base + (size_t)P.src_dir[r][c] * P.src_stride;
            C.cg[k] = (double)P.coefG[r][c];
            C.cd[k] = (double)P.coefT[r][c] - (double)P.coefG[r][c];
        }
        if (P.use_gc) { C.src[ri * C.src_pitch + n] = P.gc; C.cg[ri * C.src_pitch + n] = 1.0; }
        C.n_src[ri] = n + (P.use_gc ? 1 : 0);
    }
    C.begin[P.r_count] = (int)P.blk_begin[P.r_count];
    C.V = P.V; C.w = P.w; C.p = P.p; C.q = P.q; C.S = P.S; C.gunary = P.gunary; C.gw = P.gw; C.gV = P.gV; C.gstore = P.gstore;
    C.gstore32 = P.gstore32; C.unary_dir = P.unary_dir; C.unary_init = P.unary_init; C.fault = P.fault; C.spin_limit = P.spin_limit;
    const size_t lds = mrf_bwd_chain_lds_bytes(LP, ni, P.g.L, hot, gv, !vg && !gv);
    if (lds > chain_lds_cap(P.total_scanlines)) return hipErrorInvalidValue;
    // (more than 64 KB of dynamic LDS has to be announced per kernel)
#define MRF_CH_GO(...) \
    do { \
        if (lds > 64 * 1024) { \
            const hipError_t ea_ = hipFuncSetAttribute(reinterpret_cast<const void *>(&__VA_ARGS__), \
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
            if (ea_ != hipSuccess) return ea_; \
        } \
        hipLaunchKernelGGL((__VA_ARGS__), grid, dim3(64 * (1 + ni)), lds, st, C); \
    } while (0)
    if (far) {
        if constexpr (NS >= 4) {
            if (ni != MRF_CHAIN_FAR_HELPERS || edge) return hipErrorInvalidValue;
            constexpr int n = MRF_CHAIN_FAR_HELPERS;
            if constexpr (LP == 1) {
                if (gv && !P.gw) { MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, false, true, false, false, true, false>); return hipGetLastError(); }
                if (gv) { MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, false, true, false, false, true>); return hipGetLastError(); }
            }
            if constexpr (LP <= 2) {
                if (gs) { MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, true, true, true, false, true>); return hipGetLastError(); }
            }
            if (vg) MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, true, false, false, false, true>);
            else MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, false, false, (LP >= 3), false, true>);
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
#define MRF_CH(n) \
    if (ni == n) { \
        if constexpr (LP == 1 && n >= 4) { \
            if (edge) { \
                MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, true, true, false, true>); \
                return hipGetLastError(); \
            } \
        } \
        if constexpr (LP == 1) { \
            if (gv) { \
                if (P.gw) MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, false, true, false>); \
                else MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, false, true, false, false, false, false>); \
                return hipGetLastError(); \
            } \
        } \
        if constexpr (LP <= 2) { \
            if (gs) { \
                if (hot) MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, true, true, true>); \
                else MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, true, true, false>); \
                return hipGetLastError(); \
            } \
        } \
        if (vg) MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, true, false, false>); \
        else if (P.hot_label) MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, false, false, true>); \
        else MRF_CH_GO(mrf_bwd_sweep_chain<LP, NS, D, n, false, false, false>); \
        return hipGetLastError(); \
    }
    MRF_CH(2) MRF_CH(4) MRF_CH(6) MRF_CH(8) MRF_CH(12)
#undef MRF_CH
#undef MRF_CH_GO
    return hipErrorInvalidValue;
}

hipError_t run_bwd_chain(MrfBwdParams &P, int ns, int ni, bool vg, hipStream_t st)
{
    const int LP = (P.g.L + 63) / 64;
    if (ns == 1 && !P.edge && chain_far(P.g, P.gstore != nullptr)) ns = 4;
#define MRF_CCASE(lp) \
    if (LP == lp && ns == 1) return launch_bwd_chain<lp, 1, (lp <= 2 ? 2 : 1)>(P, ni, vg, st); \
    if (LP == lp && ns == 4) return launch_bwd_chain<lp, 4, (lp <= 2 ? 2 : 1)>(P, ni, vg, st); \
    if (LP == lp && ns == 8) return launch_bwd_chain<lp, 8, 1>(P, ni, vg, st);
    if (LP == 1 && ns == 16) return launch_bwd_chain<1, 16, 1>(P, ni, vg, st);
    if (LP == 2 && ns == 16) return launch_bwd_chain<2, 16, 1>(P, ni, vg, st);
    MRF_CCASE(1) MRF_CCASE(2) MRF_CCASE(3) MRF_CCASE(4)
#undef MRF_CCASE
    return hipErrorInvalidValue;
}
#endif  // MRF_HAS_BWD_CHAIN

#if MRF_HAS_BWD_PLAIN
template <int LP, int NS, int D>
hipError_t launch_bwd(const MrfBwdParams &P, long long blocks, size_t lds, hipStream_t st)
{
    const dim3 grid((unsigned)blocks), block(64 * MRF_BWD_WAVES);
    const bool hot = !(P.rho_e || P.gE) && !(P.gw && P.v_mode == 0) && P.hot_label;
    const bool no_unary = hot && NS == 1 && P.unary_dir < 0;
    note_launch(1, "mrf_bwd_sweep", blocks, 64 * MRF_BWD_WAVES, "%d,%d,%d,%s,%s,%s%s", LP, NS, D,
                (P.gw && P.v_mode == 0) ? "true" : "false", hot ? "true" : "false",
                (P.rho_e || P.gE) ? "true" : "false", no_unary ? ",false" : "");
    if (P.rho_e && P.gw && P.v_mode == 0)
        hipLaunchKernelGGL((mrf_bwd_sweep<LP, NS, D, true, false, true>), grid, block, lds, st, P);
    else if (P.rho_e || P.gE)
        hipLaunchKernelGGL((mrf_bwd_sweep<LP, NS, D, false, false, true>), grid, block, lds, st, P);
    else if (P.gw && P.v_mode == 0)
        hipLaunchKernelGGL((mrf_bwd_sweep<LP, NS, D, true, false>), grid, block, lds, st, P);
    else if (no_unary) {
        if constexpr (NS == 1) {
            if (P.g.L == 64 * LP)
                hipLaunchKernelGGL((mrf_bwd_sweep<LP, NS, D, false, true, false, false, MRF_BWD_WAVES, true>), grid, block, lds, st, P);
            else
                hipLaunchKernelGGL((mrf_bwd_sweep<LP, NS, D, false, true, false, false>), grid, block, lds, st, P);
        }
    } else if (P.hot_label)
        hipLaunchKernelGGL((mrf_bwd_sweep<LP, NS, D, false, true>), grid, block, lds, st, P);
    else
        hipLaunchKernelGGL((mrf_bwd_sweep<LP, NS, D, false, false>), grid, block, lds, st, P);
    return hipGetLastError();
}

// The V gradient in one LDS table per workgroup of MRF_BWD_TILE_WAVES wavefronts (33..128 labels)
template <int LP, int NS, int D>
hipError_t launch_bwd_tile(const MrfBwdParams &P, long long blocks, size_t lds, hipStream_t st)
{
    const dim3 grid((unsigned)blocks), block(64 * MRF_BWD_TILE_WAVES);
    const bool vg = P.gw && P.v_mode == 0;
    note_launch(1, "mrf_bwd_sweep", blocks, 64 * MRF_BWD_TILE_WAVES, "%d,%d,%d,%s,false,false,true,%d", LP, NS, D, vg ? "true" : "false",
                MRF_BWD_TILE_WAVES);
#define MRF_T_GO(...) \
    do { \
        if (lds > 64 * 1024) { \
            const hipError_t ea_ = hipFuncSetAttribute(reinterpret_cast<const void *>(&__VA_ARGS__), \
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
            if (ea_ != hipSuccess) return ea_; \
        } \
        hipLaunchKernelGGL((__VA_ARGS__), grid, block, lds, st, P); \
    } while (0)
    if (vg) MRF_T_GO(mrf_bwd_sweep<LP, NS, D, true, false, false, true, MRF_BWD_TILE_WAVES>);
    else MRF_T_GO(mrf_bwd_sweep<LP, NS, D, false, false, false, true, MRF_BWD_TILE_WAVES>);
#undef MRF_T_GO
    return hipGetLastError();
}

// two scanlines of up to 32 labels per workgroup: chain wavefront + ni helpers
template <int NS, int D>
hipError_t launch_bwd_chain_pk(const MrfBwdParams &P, int ni, hipStream_t st)
{
    const long long blocks = (P.total_scanlines + 1) / 2;
    const bool gv = P.gV != nullptr;
    note_launch(1, "mrf_bwd_sweep_chain_pk", blocks, 64 * (1 + ni), "%d,%d,%d,%s", NS, D, ni, gv ? "true" : "false");
    if (gv && blocks > grad_slots(P.g.L)) return hipErrorInvalidValue;
    const size_t lds = mrf_bwd_chain_pk_lds_bytes(ni, P.g.L, gv);
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(64 * (1 + ni));
#define MRF_PK(n) \
    if (ni == n) { \
        if (gv) hipLaunchKernelGGL((mrf_bwd_sweep_chain_pk<NS, D, n, true>), grid, block, lds, st, P); \
        else hipLaunchKernelGGL((mrf_bwd_sweep_chain_pk<NS, D, n, false>), grid, block, lds, st, P); \
        return hipGetLastError(); \
    }
    MRF_PK(2) MRF_PK(4) MRF_PK(8)
#undef MRF_PK
    return hipErrorInvalidValue;
}

template <int SEG>
hipError_t launch_bwd_packed(const MrfBwdParams &P, int ns, hipStream_t st)
{
    constexpr int NSEG = 64 / SEG;
    const int L = P.g.L;
    long long blocks = (P.total_scanlines + NSEG - 1) / NSEG;
    if (P.gV && blocks > grad_slots(L)) blocks = grad_slots(L);
    note_launch(1, "mrf_bwd_sweep_packed", blocks, 64, "%d,%d,%d", SEG, ns, ns <= 4 ? 4 : (ns == 8 ? 2 : 1));
    const size_t lds = sizeof(double) * (64 + (P.gV ? (size_t)NSEG * L * L : 0)) + sizeof(float) * (size_t)L * L;
    const dim3 grid((unsigned)blocks), block(64);
    if (ns == 1 && P.unary_dir < 0) hipLaunchKernelGGL((mrf_bwd_sweep_packed<SEG, 1, 4, false>), grid, block, lds, st, P);
    else if (ns == 1) hipLaunchKernelGGL((mrf_bwd_sweep_packed<SEG, 1, 4>), grid, block, lds, st, P);
    else if (ns == 4) hipLaunchKernelGGL((mrf_bwd_sweep_packed<SEG, 4, 4>), grid, block, lds, st, P);
    else if (ns == 8) hipLaunchKernelGGL((mrf_bwd_sweep_packed<SEG, 8, 2>), grid, block, lds, st, P);
    else hipLaunchKernelGGL((mrf_bwd_sweep_packed<SEG, 16, 1>), grid, block, lds, st, P);
    return hipGetLastError();
}

hipError_t run_bwd_chain_pk(MrfBwdParams &P, int ns, int ni, hipStream_t st)
{
    if (ns == 1) return launch_bwd_chain_pk<1, 2>(P, ni, st);
    if (ns == 4) return launch_bwd_chain_pk<4, 2>(P, ni, st);
    return launch_bwd_chain_pk<8, 1>(P, ni, st);
}

hipError_t run_bwd_packed(MrfBwdParams &P, int seg, int ns, hipStream_t st)
{
    if (seg == 21) return launch_bwd_packed<21>(P, ns, st);
    return seg == 16 ? launch_bwd_packed<16>(P, ns, st) : launch_bwd_packed<32>(P, ns, st);
}

// the narrow sweep divided among four wavefronts
template <int SEG, int NL>
hipError_t launch_bwd_narrow_divided(MrfBwdParams &P, int ns, long long packs, hipStream_t st)
{
    const int L = P.g.L;
    const bool gv = P.gV != nullptr, unary = P.unary_dir >= 0;
    if (gv && packs > grad_slots(L)) return hipErrorInvalidValue;
    note_launch(1, "mrf_bwd_sweep_narrow", packs, 256, "%d,%d,%d,%s,%s", SEG, NL, ns, unary ? "true" : "false", gv ? "true" : "false");
#define MRF_D_GO(n, un, g) \
    if (ns == n && unary == un && gv == g) { \
        const size_t lds = mrf_bwd_narrow_divided_lds<SEG, NL, un, g>(L); \
        void (*const kernel)(MrfBwdParams) = mrf_bwd_sweep_narrow<SEG, NL, n, un, g>; \
        if (lds > 64 * 1024) { \
            const hipError_t ea_ = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
            if (ea_ != hipSuccess) return ea_; \
        } \
        hipLaunchKernelGGL(kernel, dim3((unsigned)packs), dim3(256), lds, st, static_cast<const MrfBwdParams &>(P)); \
        return hipGetLastError(); \
    }
#define MRF_D(n) MRF_D_GO(n, false, false) MRF_D_GO(n, false, true) MRF_D_GO(n, true, false) MRF_D_GO(n, true, true)
    MRF_D(4) MRF_D(8)
#undef MRF_D
#undef MRF_D_GO
    return hipErrorInvalidValue;
}

template <int SEG, int NL>
hipError_t launch_bwd_narrow(MrfBwdParams &P, int ns, long long packs, hipStream_t st)
{
    // four wavefronts per workgroup share V and a V-gradient slot, but a launch that does not fill the machine
    // spreads its wavefronts over the compute units
    const int waves = packs >= 1024 ? 4 : (packs >= 512 ? 2 : 1);
    const long long blocks = (packs + waves - 1) / waves;
    const int L = P.g.L, nseg = 64 / SEG;
    const bool gv = P.gV != nullptr;
    // a workgroup has a V-gradient slot of its own: what is more than there are slots goes into further launches, which
    // add to the same slots one after the other
    const long long most = gv && blocks > grad_slots(L) ? grad_slots(L) : blocks;
    const size_t lds = sizeof(double) * (size_t)waves * (nseg * mrf_bwd_narrow_row<SEG, NL>() + 64 + (gv ? mrf_bwd_narrow_tables(nseg, L, waves) * mrf_bwd_narrow_table<SEG, NL>(L) : 0)) +
                       sizeof(float) * ((size_t)L * mrf_bwd_narrow_pitch(L) + 1);
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    const dim3 block(64u * (unsigned)waves);
    // (one source, no grad theta and several directions: ISGMR, every coefficient 1)
    const bool unary = ns == 1 ? (P.unary_dir >= 0 || P.r_count == 1) : P.unary_dir >= 0;
    const bool full = L % NL == 0;
#define MRF_N(n, d, un) \
    if (ns == n && unary == un) { \
        for (long long first = 0; first < blocks; first += most) { \
            const dim3 grid((unsigned)(blocks - first < most ? blocks - first : most)); \
            P.pack_first = (int)(first * waves); \
            note_launch(1, "mrf_bwd_sweep_narrow", grid.x, 64 * waves, "%d,%d,%d,%d,%s,%s,%s", SEG, NL, n, d, un ? "true" : "false", \
                        gv ? "true" : "false", full ? "true" : "false"); \
            if (P.edge) { \
                if constexpr (NL == 1 || (SEG == 8 && NL == 3)) { \
                    if (full) hipLaunchKernelGGL((mrf_bwd_sweep_narrow<SEG, NL, n, d, un, false, true, true>), grid, block, lds, st, P); \
                    else return hipErrorInvalidValue; \
                } else return hipErrorInvalidValue; \
            } else if (gv && full) hipLaunchKernelGGL((mrf_bwd_sweep_narrow<SEG, NL, n, d, un, true, true>), grid, block, lds, st, P); \
            else if (gv) hipLaunchKernelGGL((mrf_bwd_sweep_narrow<SEG, NL, n, d, un, true, NL == 1>), grid, block, lds, st, P); \
            else if (full) hipLaunchKernelGGL((mrf_bwd_sweep_narrow<SEG, NL, n, d, un, false, true>), grid, block, lds, st, P); \
            else hipLaunchKernelGGL((mrf_bwd_sweep_narrow<SEG, NL, n, d, un, false, NL == 1>), grid, block, lds, st, P); \
            const hipError_t e_ = hipGetLastError(); \
            if (e_ != hipSuccess) return e_; \
        } \
        return hipSuccess; \
    }
    MRF_N(1, 4, false) MRF_N(1, 4, true) MRF_N(4, 2, false) MRF_N(4, 2, true)
    MRF_N(8, (NL <= 2 ? 2 : 1), false) MRF_N(8, (NL <= 2 ? 2 : 1), true) MRF_N(16, 1, false) MRF_N(16, 1, true)
#undef MRF_N
    return hipErrorInvalidValue;
}

hipError_t run_bwd_narrow(MrfBwdParams &P, int seg, int ns, hipStream_t st)
{
    const int L = P.g.L, nseg = 64 / seg;
    long long packs = 0;
    for (int ri = 0; ri < P.r_count; ++ri) {
        P.pack_begin[ri] = (int)packs;
        packs += ((long long)P.g.B * P.g.nscan[P.r_first + ri] + nseg - 1) / nseg;
    }
    P.pack_begin[P.r_count] = (int)packs;
    const int nl = (L + seg - 1) / seg;
    // the work of a node divided among four wavefronts while the launch leaves SIMDs idle (TRWP, 512 x 512 images, K = 2, one / four
    // wavefronts: 256 wavefronts of scanlines, 21 labels 1.86 / 1.42 ms, 8 labels 1.11 / 0.92; 768 3.44 / 2.91, 1.77 / 1.20; 1,024 of 32 labels
    // 1.82 / 1.50, of 16 labels 1.62 / 1.38; 1,536 of 32 labels 2.30 / 2.41)
    const bool divided = P.r_count == 1 && (ns == 4 || ns == 8) && L % nl == 0 && !P.edge && g_tune_narrow_divided != 1 &&
                         (g_tune_narrow_divided == 2 || packs <= 1024) && !(P.gV && packs > grad_slots(L));
    if (divided && seg == 32 && nl == 1) return launch_bwd_narrow_divided<32, 1>(P, ns, packs, st);
    if (divided && seg == 16 && nl == 1) return launch_bwd_narrow_divided<16, 1>(P, ns, packs, st);
    if (divided && seg == 16 && nl == 2) return launch_bwd_narrow_divided<16, 2>(P, ns, packs, st);
    if (divided && seg == 8 && nl == 1) return launch_bwd_narrow_divided<8, 1>(P, ns, packs, st);
    if (divided && seg == 8 && nl == 3) return launch_bwd_narrow_divided<8, 3>(P, ns, packs, st);
    if (seg == 32 && nl == 1) return launch_bwd_narrow<32, 1>(P, ns, packs, st);
    if (seg == 16 && nl == 1) return launch_bwd_narrow<16, 1>(P, ns, packs, st);
    if (seg == 16 && nl == 2) return launch_bwd_narrow<16, 2>(P, ns, packs, st);
    if (seg == 8 && nl == 1) return launch_bwd_narrow<8, 1>(P, ns, packs, st);
    if (seg == 8 && nl == 2) return launch_bwd_narrow<8, 2>(P, ns, packs, st);
    if (seg == 8 && nl == 3) return launch_bwd_narrow<8, 3>(P, ns, packs, st);
    if (seg == 8 && nl == 4) return launch_bwd_narrow<8, 4>(P, ns, packs, st);
    return hipErrorInvalidValue;
}

hipError_t run_bwd_tile(MrfBwdParams &P, int ns, long long blocks, size_t lds, hipStream_t st)
{
    const int LP = (P.g.L + 63) / 64;
#define MRF_TCASE(lp) \
    if (LP == lp && ns == 1) return launch_bwd_tile<lp, 1, 4>(P, blocks, lds, st); \
    if (LP == lp && ns == 4) return launch_bwd_tile<lp, 4, 4>(P, blocks, lds, st); \
    if (LP == lp && ns == 8) return launch_bwd_tile<lp, 8, 2>(P, blocks, lds, st); \
    if (LP == lp && ns == 16) return launch_bwd_tile<lp, 16, 1>(P, blocks, lds, st);
    MRF_TCASE(1) MRF_TCASE(2)
#undef MRF_TCASE
    return hipErrorInvalidValue;
}

hipError_t run_bwd_plain(MrfBwdParams &P, int ns, long long blocks, size_t lds, hipStream_t st)
{
    const int LP = (P.g.L + 63) / 64;
#define MRF_BCASE(lp) \
    if (LP == lp && ns == 1) return launch_bwd<lp, 1, (lp >= 3 ? 2 : 4)>(P, blocks, lds, st); \
    if (LP == lp && ns == 4) return launch_bwd<lp, 4, (lp <= 2 ? 4 : 2)>(P, blocks, lds, st); \
    if (LP == lp && ns == 8) return launch_bwd<lp, 8, 2>(P, blocks, lds, st); \
    if (LP == lp && ns == 16) return launch_bwd<lp, 16, 1>(P, blocks, lds, st);
    MRF_BCASE(1) MRF_BCASE(2) MRF_BCASE(3) MRF_BCASE(4)
#undef MRF_BCASE
    return hipErrorInvalidValue;
}
#endif  // MRF_HAS_BWD_PLAIN

#if MRF_HAS_BWD
template <int NS, int D>
hipError_t launch_bwd_split(const MrfBwdParams &P, long long blocks, size_t lds, hipStream_t st)
{
    const dim3 grid((unsigned)blocks), block(64u * (unsigned)((P.g.L + 63) / 64));
    note_launch(1, "mrf_bwd_sweep_split", blocks, (int)block.x, "%d,%d,%s", NS, D, (P.gw && P.v_mode == 0) ? "true" : "false");
    if (P.gw && P.v_mode == 0)
        hipLaunchKernelGGL((mrf_bwd_sweep_split<NS, D, true>), grid, block, lds, st, P);
    else
        hipLaunchKernelGGL((mrf_bwd_sweep_split<NS, D, false>), grid, block, lds, st, P);
    return hipGetLastError();
}

// Lanes per scanline of mrf_bwd_sweep_narrow, or 0 where its 32-bit offsets do not reach.  Eight where that leaves
// three labels per lane at most and fills the lanes (backward pass, 4 x 512 x 512, 21 labels, K = 3: ISGMR 1.14 / 1.45 /
// 1.87 ms with 8 / 16 / 32 lanes, TRWP 2.8 / 3.5 / 3.1 ms); two labels per lane are no faster than one (256 x 512, 16
// labels, 16 directions 0.69 ms with 16 lanes, 0.77 with 8), and with four the V-gradient tables of eight scanlines
// crowd LDS (32 labels, 16 directions 1.53 / 1.26 / 1.17 ms; without that gradient 16 lanes are ahead).
// With several source arrays a lane's labels should be one access each: where they do not divide the label count, the
// loads of a node cost more than the idle lanes of a wider segment (TRWP, K = 2, 5 x 512 x 512, 8 directions, 8 / 16 / 32
// lanes: 20 labels 10.6 / 7.1 / 6.7 ms, 23 labels 10.8 / 9.9 / 7.2; 25 labels without grad V 12.5 / 9.1 / 6.7; 9 x 256 x 512,
// 4 directions: 22 labels 2.63 / 2.08 / 2.21, 19 labels 2.54 / 2.49 / 2.41).
int narrow_lanes(const MrfBwdParams &P, int L, int ns)
{
    if (g_tune_narrow < 0 || P.g.N * L > MRF_BUF_MOST) return 0;
    if (g_tune_narrow == 8 || (g_tune_narrow == 16 && L > 8) || (g_tune_narrow == 32 && L > 16)) return g_tune_narrow;
    if (L <= 8) return 8;
    if (L <= 16) return 16;
    if (L <= 24 && (ns == 1 || L % 3 == 0)) return 8;
    if (ns > 1 && L % 2 != 0) return 32;
    return L > 24 && P.gV ? 32 : 16;
}

#define MRF_GV_BLOCKS 256      // workgroups (and slots) of mrf_bwd_pairwise_*

hipError_t dispatch_bwd(MrfBwdParams &P, int pairwise_kind, hipStream_t st)
{
    const int L = P.g.L;
    const int LP = (L + 63) / 64;
    long long blocks = (P.total_scanlines + MRF_BWD_WAVES - 1) / MRF_BWD_WAVES;
    if (P.gV && blocks > grad_slots(L) / MRF_BWD_WAVES) blocks = grad_slots(L) / MRF_BWD_WAVES;
    // LDS: scatter vectors, optional private V-gradient accumulators, optional copy of V
    P.gv_lds = (P.gV && L <= 32) ? 1 : 0;
    // truncated models scatter most labels to one target; pre-reducing it pays when LDS
    // conflicts, not instruction issue, bound the step
    P.hot_label = (pairwise_kind != MRF_PAIRWISE_DENSE && (L > 128 || P.total_scanlines > 1024)) ? 1 : 0;
    P.v_mode = 0;
    if (P.gw) {
        if ((size_t)L * L * sizeof(float) <= 40 * 1024) P.v_mode = 1;
        else if (pairwise_kind != MRF_PAIRWISE_DENSE) P.v_mode = 2;   // promise: V(mu,lambda) = V(0,|mu-lambda|)
    }
    const size_t lds = sizeof(double) * ((size_t)MRF_BWD_WAVES * 64 * LP + (P.gv_lds ? (size_t)MRF_BWD_WAVES * L * L : 0)) +
                       sizeof(float) * (P.v_mode == 1 ? (size_t)L * L : (P.v_mode == 2 ? (size_t)L : 0));
    int need = 0;
    for (int r = P.r_first; r < P.r_first + P.r_count; ++r)
        if (P.n_src[r] + (P.use_gc ? 1 : 0) > need) need = P.n_src[r] + (P.use_gc ? 1 : 0);
    const int ns = need <= 1 ? 1 : (need <= 4 ? 4 : (need <= 8 ? 8 : 16));
    // per-edge tables without a V: the chain layout, or for up to 32 labels and more scanlines the narrow one; either
    // stores the node gradients if they are wanted (run_backward has checked that one of them fits)
    if (P.edge) {
        P.hot_label = 0;
        // (backward pass with the tables' gradient, K = 2, chain / narrow: TRWP, 128 x 128 images, 768 scanlines 8 labels 0.278 / 0.287 ms, 16
        // labels 0.372 / 0.410; 1,024 8 labels 0.372 / 0.294, 16 labels 0.515 / 0.460, 18 labels 0.590 / 0.610, 32 labels 0.863 / 0.900; 1,280 18
        // labels 0.751 / 0.664, 32 labels level.  ISGMR, 1 : 3 images, where the chain stays ahead a little longer: 1,024 scanlines 5 labels
        // 0.138 / 0.203, 32 labels 0.345 / 0.442; 1,280 0.200 / 0.247, 0.541 / 0.613; 1,536 level, 0.710 / 0.816; 2,048 0.355 / 0.313, 1.18 /
        // 1.31.  One line for both.)
        if (L <= 32 && P.total_scanlines > 1024) return run_bwd_narrow(P, L <= 8 || (L <= 24 && L % 3 == 0 && L > 16) ? 8 : (L <= 16 ? 16 : 32), ns, st);
        const int ni = P.total_scanlines <= 256 ? 12 : (P.total_scanlines <= 512 ? 8 : (P.total_scanlines <= 1024 ? 6 : 4));
        return run_bwd_chain(P, ns, ni, true, st);
    }
    // few scanlines: the node-to-node chain on a wavefront of its own, helpers around it
    // (its addressing wants a node step times L in 32 bits, and a variant of its own where an image is beyond that; with the
    // V gradient, L <= 64, room in LDS and a slot per workgroup)
    bool step_fits = true;
    for (int r = P.r_first; r < P.r_first + P.r_count; ++r) {
        const long long stp = ((long long)mrf_iabs(P.g.dh[r]) * P.g.W + mrf_iabs(P.g.dw[r])) * L;
        if (stp > 0x7fffffffLL) step_fits = false;
    }
    const bool gv_any = P.gV != nullptr;
    // 33..128 labels, one direction per launch: the chain layout has no room for V-gradient tables, so its
    // helpers store the node gradients and a streaming pass forms both pairwise gradients (mrf_bwd_pairwise_*)
    // (backward pass per iteration with all gradients, 256 x 512, 8 directions: 96 labels 3.6 -> 1.3 ms, 64 labels 2.1 ->
    // 0.9, 40 labels 1.0 -> 0.75; 16 directions on 128 x 256, 96 labels, 3.8 -> 1.35.  Up to 48 labels a launch of one
    // scanline per compute unit has room for eight helpers with tables of their own: 64 x 96, 40 labels, 4 directions,
    // 0.10 against 0.13 ms)
    const bool gv_apart = gv_any && L > 32 && LP <= 2 && P.gstore_buf && P.r_count == 1 && !P.rho_e && !P.force_plain &&
                          P.total_scanlines <= kApartMost && !(L <= 48 && P.total_scanlines <= 256) && g_tune_gv_apart != 1;
    const bool gv = gv_any && !gv_apart;      // the V gradient inside the sweep that runs
    // as many helpers as keep up with the chain while the machine and the LDS have room
    // (backward pass, ISGMR, 4 directions, K = 3, with 4 / 6 / 8 helpers: 96 labels 512 scanlines 181 / 174 / 167 us, 1,024 604 / 597 /
    // 732, 1,388 924 / 787 / 949, 2,560 2.80 / 2.67 / 3.07 ms; 40 labels 512 112 / 104 / 100 us, 1,388 585 / 520 / 574; 160 labels 512
    // 201 / 183 / 180, 1,388 1.25 / 1.18 / 1.34 ms; 256 labels 512 251 / 237 / 306 us.  TRWP, 256 x 512, 96 labels, K = 5, 256 and 512
    // scanlines, with 6 / 8 / 12 of them 1.50 / 1.28 / 1.31 ms; 256 x 256, 256 labels, K = 10, 256 scanlines 3.18 / 3.17 / 4.44)
    int ni = g_tune_chain_ni ? g_tune_chain_ni
                             : (P.total_scanlines <= 256 ? (LP <= 2 ? 12 : 8) : (P.total_scanlines <= 512 && LP <= 3 ? 8 : 6));
    // (the helpers of many source arrays, and those that leave the pairwise gradients to a later pass: six. 128 x 256, 16
    // directions, 96 labels: 3.1 / 2.7 / 3.0 / 3.6 ms with 4 / 6 / 8 / 12; 256 x 512, 8 directions, 40 labels: 1.75 / 1.50 /
    // 1.66 / 1.80 ms)
    if (!g_tune_chain_ni && gv_apart && (ns == 16 || LP == 1 || P.total_scanlines > 256)) ni = 6;
    if (!g_tune_chain_ni && gv && P.total_scanlines > 384 && ni > 6) ni = 6;   // (the accumulators take LDS)
    const bool vg = P.gw && pairwise_kind == MRF_PAIRWISE_DENSE;
    const bool far = chain_far(P.g, gv_apart);
    if (far) ni = MRF_CHAIN_FAR_HELPERS;
    // truncated models: the lanes that go to the most popular scatter target are kept apart
    const bool chain_hot = far ? !gv && (gv_apart || (!vg && LP >= 3))
                               : (pairwise_kind != MRF_PAIRWISE_DENSE || gv_apart) && !gv && g_tune_chain_hot != 1 &&
                                     (g_tune_chain_hot == 2 || L > 128 || P.total_scanlines > 1024);
    const auto chain_lds = [&](int helpers) { return mrf_bwd_chain_lds_bytes(LP, helpers, L, chain_hot, gv, !vg && !gv_any); };
    while (ni > 2 && (chain_lds(ni) > chain_lds_cap(P.total_scanlines) ||
                      (gv && P.total_scanlines > grad_slots(L)))) ni = (ni == 12) ? 8 : ni - 2;
    // TRW coefficients or pairwise tables per edge: mrf_bwd_sweep handles them (and is the one
    // sweep that never touches V when no edge-weight gradient is asked for)
    const bool generic = P.rho_e != nullptr || P.force_plain;
    const bool chain_fits = !generic && step_fits && !(far && ni != MRF_CHAIN_FAR_HELPERS) && ns <= (LP <= 2 ? 16 : 8) && g_tune_chain != 1 &&
                            (!gv || (LP == 1 && P.total_scanlines <= grad_slots(L))) &&
                            chain_lds(ni) <= chain_lds_cap(P.total_scanlines);
    // (backward pass, chain / the next best layout, truncated models, K = 2.  ISGMR, one source array, 4 directions, 2,048 / 2,304 / 2,560
    // scanlines: 160 labels 1.87 / 1.89, 2.31 / 2.41, 2.87 / 2.77 ms (a dense table ahead by 7 % at 2,560); up to 128 labels ahead to 2,560 (96
    // labels by 5 %); 256 labels 1,536 1.43 / 1.46, 2,048 behind by 16 %.  Label counts that fill the lanes of mrf_bwd_sweep, which has a variant
    // for them: 64 labels 2,304 1.05 / 1.10, 2,560 1.33 / 1.25; 128 labels 1,792 1.04 / 1.06, 2,048 1.37 / 1.26; 192 labels 1,536 1.14 /
    // 1.19, 1,792 1.53 / 1.46, 2,048 2.02 / 1.78.  On long grids most of the scanlines are short and done when the longest still run, so these
    // bounds are by nodes over the longest: 24 x 1026, 128 labels 0.45 / 1.53, 61 x 1168, 192 labels, K = 1 0.39 / 1.19.  Eight directions, whose
    // launch has many short diagonal scanlines, 3,068 / 3,596 / 4,220 (2,048 / 2,400 / 2,816 by the longest): 128 labels 0.693 / 0.696, 0.926 /
    // 0.897, 1.25 / 1.18, 192 labels 0.99 / 0.95 (2,300 by 9 % ahead), 160 labels 0.92 / 1.00, 1.23 / 1.29, level; 96 labels ahead by 15 % at all of them.
    // TRWP, several source arrays: 2,048 scanlines 40 labels 1.55 / 1.77, 96 labels 2.09 / 2.69, 160 labels 2.86 / 3.59, 256
    // labels 4.28 / 4.83; eight directions, 512 scanlines 160 labels 2.53 / 4.71, 256 labels 3.62 / 5.80)
    const long long chain_max = ns >= 4 ? (LP == 1 ? 2560 : 2048)
                                        : (LP == 4 ? 1536 : (P.r_count >= 8 ? (LP <= 2 ? 4224 : 3584) : 2560));
    bool behind = false;
    if (ns == 1 && LP <= 3 && pairwise_kind != MRF_PAIRWISE_DENSE && !P.gV) {
        const bool full = L == 64 * LP;
        const long long most = full && LP == 2 ? 2000 : (full && LP == 3 ? 1536 : 2432);
        behind = (full || LP == 3) && P.g.N * P.r_count > most * longest_scanline(P.g, P.r_first, P.r_count);
    }
    const bool chain = chain_fits && (g_tune_chain == 2 || (P.total_scanlines <= chain_max && !behind));
    // Few labels, one direction per launch (TRWP): the chain layout for one scanline per compute unit, two scanlines
    // around a chain wavefront beyond that, mrf_bwd_sweep_narrow for more than the machine holds that way.  (Backward
    // pass of 256 x 512 grids, 21 labels, 4 directions, K = 3, one / two / four images: 0.83 / 1.35 / 2.15 ms chain,
    // 0.78 / 1.00 / 1.81 ms two scanlines, 2.1 ms narrow; 4 x 512 x 512: 3.4 ms two scanlines, 2.8 ms narrow.  The other label
    // counts, two scanlines / narrow, K = 2: 7 x 256 x 256, 1,792 scanlines, 8 labels 0.95 / 0.59, 16 labels 0.97 / 0.73, 18
    // labels 1.03 / 0.98, 32 labels 1.12 / 1.14.  17, 19 and 23 labels fill no segment: with up to four source arrays 1.59 /
    // 1.80 at 1,640 scanlines, 2.03 / 2.19 at 2,048, 2.42 / 2.95 at 2,560, with eight 4.84 / 4.22 at 1,640)
    const bool fills_none = L > 16 && L <= 24 && L % 2 != 0 && L % 3 != 0;
    // The narrow sweep divided among four wavefronts, which several source arrays take, is ahead earlier.  The machine holds 256
    // workgroups of two scanlines with a compute unit each, 512 with two on each, and the time of a sweep of equal scanlines goes up by
    // a half and by a third where these are full.  (Backward pass, 4 directions, 64 x 64 images, K = 3, two scanlines / divided, at 512,
    // 576, 1,024 and 1,088 scanlines: 5 labels 0.192 / 0.244, 0.299 / 0.247, 0.305 / 0.248, -; 16 labels 0.200 / 0.261, 0.321 / 0.262,
    // 0.324 / 0.271, -; 21 labels 0.209 / 0.353, 0.334 / 0.356, 0.339 / 0.358, 0.464 / 0.359; 32 labels 0.223 / 0.305, 0.356 / 0.330,
    // 0.366 / 0.337, 0.496 / 0.361.  1024 x 1024, 1,024 scanlines, K = 2: 16 labels 2.13 / 1.90, 21 labels 2.23 / 2.73.)
    // The short scanlines of a diagonal direction leave room early (eight directions, 1 x 300 x 300, K = 2, launches of 300 and 599
    // scanlines: 8 labels 0.80 / 0.90, 32 labels 0.90 / 1.05; 512 x 512, 512 and 1,023: 32 labels 1.69 / 1.80; 2 x 256 x 512, 12 labels 1.41 /
    // 1.25).
    const bool divided = (ns == 4 || ns == 8) && P.g.N * L <= MRF_BUF_MOST && g_tune_narrow == 0 && g_tune_narrow_divided != 1;
    const bool even = P.g.dh[P.r_first] == 0 || P.g.dw[P.r_first] == 0;      // (every scanline is as long as the others)
    const long long pk_max = fills_none && ns == 4 ? 2560 : (!divided ? (L <= 8 ? 1024 : 1536)
                                                             : (ns == 4 && even ? (L > 16 && L <= 24 ? 1024 : 512) : (L <= 16 ? 896 : 1280)));
    if (!generic && L <= 32 && P.r_count == 1 && ns <= 8 && g_tune_chain != 1 && g_tune_pack != 2 && g_tune_chain_pk != 1 &&
        (g_tune_chain_pk == 2 || (g_tune_chain != 2 && P.total_scanlines > 256 && P.total_scanlines <= pk_max)) &&
        !(gv_any && (P.total_scanlines + 1) / 2 > grad_slots(L))) {
        // (helpers: 3 x 512 x 512, 16 labels, 8 directions, 1,536 scanlines: 4.3 ms with eight, 5.0 with four; the LDS
        // of a compute unit, which several such workgroups share, sets the pace)
        const int nip = (g_tune_chain_ni == 2 || g_tune_chain_ni == 4 || g_tune_chain_ni == 8) ? g_tune_chain_ni
                                                                                            : (P.total_scanlines <= 1536 ? 8 : 4);
        return run_bwd_chain_pk(P, ns, nip, st);
    }
    // few labels: several scanlines per wavefront, once there are enough of them
    // (all directions in one launch, ISGMR, 1,536 scanlines: 0.47 against 0.56 ms for the chain with 16 labels, 0.63
    // against 0.74 with 32, but 0.66 against 0.59 with 21, where a lane's three labels make the node step long)
    // (without grad V the chain's helpers have less to do: 256 x 512, 4 directions, K = 2, 25 labels 0.38 against 0.40 ms, 31
    // labels 0.38 against 0.43)
    // (and where two scanlines per workgroup have given way to the divided sweep, it is the next: 8 x 128 x 128, 1,024 scanlines,
    // chain / two scanlines / divided: 8 labels 0.447 / 0.315 / 0.274 ms, 16 labels 0.456 / 0.323 / 0.293)
    const long long chain_few = (P.r_count > 1 && L > 16 && (L <= 24 || !gv_any)) ? 1536 : (P.r_count == 1 && divided && pk_max < 1024 ? pk_max : 1024);
    if (!generic && L <= 32 && g_tune_pack != 1 && (g_tune_pack == 2 || P.total_scanlines >= 256) &&
        !(chain && g_tune_pack != 2 && (g_tune_chain == 2 || P.total_scanlines <= chain_few)))
    {
        // three scanlines per wavefront, one label per lane: on request only
        if (L > 16 && L <= 21 && g_tune_pack3 == 2)
            return run_bwd_packed(P, 21, ns, st);
        const int seg = narrow_lanes(P, L, ns);
        if (seg > 0) return run_bwd_narrow(P, seg, ns, st);
        // arrays beyond 32-bit offsets: one label per lane, 64-bit addresses.  (Backward pass, ISGMR with grad V, eight
        // images, 2 directions, K = 1, N L = 1.08e9, against one wavefront per scanline: 20 / 58 ms with 8 labels, 15 / 31
        // with 16, 18 / 25 with 21, 19.5 / 20.5 with 32)
        return run_bwd_packed(P, L <= 16 ? 16 : 32, ns, st);
    }
    if (chain) {
        P.hot_label = chain_hot ? 1 : 0;      // (what its LDS was sized for)
        if (gv_apart) {
            double *const slots = P.gV;
            P.gV = nullptr; P.gstore = P.gstore_buf;
            const hipError_t e = run_bwd_chain(P, ns, ni, vg, st);
            P.gV = slots; P.gstore = nullptr;
            if (e != hipSuccess) return e;
            MrfGvParams G;
            G.N = P.g.N; G.L = L; G.g = P.gstore_buf;
            G.p = P.p + (size_t)P.r_first * P.g.N * L;
            G.w = P.w + (P.w_mul ? (size_t)P.r_first * P.g.N : 0); G.w_mul = P.w_mul;
            G.V = P.V; G.gw = P.gw ? P.gw + (size_t)P.r_first * P.g.N : nullptr;
            G.gV = slots;
            // (up to 64 labels: as many tables, eight or four, as 156 KB hold next to V)
            const size_t vsize = sizeof(float) * (size_t)L * L, tsize = sizeof(double) * (size_t)L * L;
            const int tables = LP == 1 ? (8 * tsize + vsize <= 156 * 1024 ? 8 : 4) : 1;
            G.v_lds = tables * tsize + vsize <= 156 * 1024 ? 1 : 0;
            const size_t glds = tables * tsize + (G.v_lds ? vsize : 0);
            // (a workgroup per compute unit at most.  Its sixteen wavefronts take 64 nodes at a time: one such turn per
            // workgroup while there are few workgroups, then two, so that clearing and flushing the tables does not
            // outweigh the turns.  Backward pass, 8 directions, K = 2, with one / two / four turns: 37 x 53 nodes, 70 labels
            // 0.41 / 0.44 / 0.54 ms; 64 x 96, 96 labels 0.62 / 0.62 / 0.70; 128 x 128, 128 labels 1.21 / 1.07 / 1.10)
            const long long one = (P.g.N + 63) / 64, two = P.g.N / 128;
            long long gblocks = one < 96 ? one : (two > 96 ? two : 96);
            if (gblocks > MRF_GV_BLOCKS) gblocks = MRF_GV_BLOCKS;
            const auto go = [&](void (*kernel)(MrfGvParams)) {
                if (glds > 64 * 1024) {
                    const hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)glds);
                    if (ea != hipSuccess) return ea;
                }
                hipLaunchKernelGGL(kernel, dim3((unsigned)gblocks), dim3(1024), glds, st, G);
                return hipGetLastError();
            };
            if (LP == 1) return tables == 8 ? go(mrf_bwd_pairwise_own<8>) : go(mrf_bwd_pairwise_own<4>);
            return go(mrf_bwd_pairwise_shared);
        }
        return run_bwd_chain(P, ns, ni, vg, st);
    }
    // few scanlines and many labels: one wavefront per 64 labels
    const bool split = !generic && LP >= 3 && g_tune_split != 1 && ns <= 8 &&
                       (g_tune_split == 2 || ((P.total_scanlines < 1024 || (P.total_scanlines == 1024 && LP == 3)) && P.total_scanlines * LP <= 4096));
    if (split) {
        long long sblocks = P.total_scanlines;
        if (P.gV && sblocks > grad_slots(L)) sblocks = grad_slots(L);
        const size_t slds = sizeof(float) * (P.v_mode == 1 ? (size_t)L * L : (P.v_mode == 2 ? (size_t)L : 0));
        P.gv_lds = 0;
        if (ns == 1) return launch_bwd_split<1, 4>(P, sblocks, slds, st);
        if (ns == 4) return launch_bwd_split<4, 4>(P, sblocks, slds, st);
        return launch_bwd_split<8, 2>(P, sblocks, slds, st);
    }
    // the V gradient of 33..128 labels: one table in LDS per workgroup, more wavefronts per workgroup
    if (P.gV && !P.gv_lds && !(P.rho_e || P.gE) && LP <= 2 && g_tune_gv_tile != 1) {
        const size_t tlds = sizeof(double) * ((size_t)MRF_BWD_TILE_WAVES * 64 * LP + (size_t)L * L) +
                            sizeof(float) * (P.v_mode == 1 ? (size_t)L * L : (P.v_mode == 2 ? (size_t)L : 0));
        if (tlds <= 156 * 1024) {
            long long tblocks = (P.total_scanlines + MRF_BWD_TILE_WAVES - 1) / MRF_BWD_TILE_WAVES;
            if (tblocks > grad_slots(L)) tblocks = grad_slots(L);
            P.gv_lds = 2;
            P.hot_label = 0;
            return run_bwd_tile(P, ns, tblocks, tlds, st);
        }
    }
    return run_bwd_plain(P, ns, blocks, lds, st);
}

hipError_t fill(float *dst, long long n, float v, hipStream_t st)
{
    long long blocks = (n + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(mrf_fill_f32, dim3((unsigned)blocks), dim3(256), 0, st, dst, n, v);
    return hipGetLastError();
}

hipError_t launch_edge_tables(const mrf_problem *pr, float *gE, const float *g, const uint8_t *p, int count, bool accumulate, hipStream_t st)
{
    MrfEdgeGradParams E;
    E.L = pr->L;
    E.tables = (long long)pr->R * pr->B * pr->H * pr->W;
    // Up to 32 KB of tables per workgroup, so that five of them share a compute unit and their phases overlap; a multiple of
    // four tables where L L is odd, which keeps every range on a 16-byte boundary.  Four tables of 47, 49, .. 63 labels are
    // more than that (35 to 63.5 KB): four to two workgroups share a compute unit there.
    const int LL = E.L * E.L, unit = LL % 4 ? 4 : 1, fit = 8192 / LL / unit * unit;
    E.T = fit > unit ? fit : unit;
    E.count = count; E.g = g; E.p = p; E.p_step = E.tables * E.L; E.gE = gE; E.accumulate = accumulate ? 1 : 0;
    const long long turns = (E.tables + E.T - 1) / E.T;
    const dim3 grid((unsigned)(turns < 1280 ? turns : 1280)), block(256);
    const size_t lds = sizeof(float) * (size_t)E.T * LL;
    if ((uintptr_t)gE % 16 == 0) hipLaunchKernelGGL(mrf_bwd_edge_tables<true>, grid, block, lds, st, E);
    else hipLaunchKernelGGL(mrf_bwd_edge_tables<false>, grid, block, lds, st, E);
    return hipGetLastError();
}

// Slots that the sweeps of a backward call can add to: a layout has at most one per scanline of a launch (the
// last workgroup of mrf_bwd_sweep may hold up to three wavefronts without one), mrf_bwd_pairwise_* one per workgroup.
long long slots_in_use(const mrf_problem *pr, const MrfGeom &g, int algo)
{
    long long most = 0, all = 0;
    for (int r = 0; r < g.R; ++r) {
        const long long n = (long long)g.B * g.nscan[r];
        all += n;
        if (n > most) most = n;
    }
    long long n = (algo == MRF_ISGMR ? all : most) + MRF_BWD_WAVES - 1;
    if (gstore_bytes(pr, algo) > 0 && n < MRF_GV_BLOCKS) n = MRF_GV_BLOCKS;
    return n < grad_slots(g.L) ? n : grad_slots(g.L);
}

int run_backward(const mrf_problem *pr, int algo, const float *grad_cost, const uint8_t *p, const uint8_t *q,
                 float *grad_unary, float *grad_w, float *grad_V, void *workspace, size_t workspace_bytes,
                 void *hip_stream)
{
    if (pr && pr->sgm_standard) return MRF_ERR_BAD_ALGORITHM;    // (Alg. 3 differentiates the revised update only)
    int rc = check_problem(pr, algo, false);
    if (rc != MRF_OK) return rc;
    if (!grad_cost || !p || !q || !grad_unary) return MRF_ERR_NULL_POINTER;
    // pairwise potentials per edge: grad_V is their gradient [R][B][H][W][L][L]; there are no
    // edge weights to differentiate
    const bool edge_tables = pr->pairwise_edge != nullptr;
    if (edge_tables && grad_w) return MRF_ERR_BAD_PAIRWISE_KIND;
    // (mrf_workspace_bytes asks for more where there are per-edge tables: speed, not a condition)
    const size_t need = kAlign + (algo == MRF_ISGMR ? 2 : 1) * msg_bytes(pr) + gradv_bytes(pr) + gstore_bytes(pr, algo);
    if (!workspace) return MRF_ERR_NULL_POINTER;
    if (workspace_bytes < need) return MRF_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t st = (hipStream_t)hip_stream;

    MrfBwdParams P;
    memset(&P, 0, sizeof(P));
    fill_geom(pr, P.g);
    const long long N = P.g.N;
    const int R = pr->R, L = pr->L, K = pr->K;
    const long long NL = N * L;
    P.V = pr->pairwise;
    P.gw = grad_w;
    P.gc = grad_cost;
    P.gunary = grad_unary;
    P.unary_dir = -1;
    P.rho_e = (algo == MRF_TRWP) ? pr->rho_edge : nullptr;
    const size_t pk = (size_t)R * N * L, qk = (size_t)R * N;

    // workspace: [scalars 256 B][buf0][buf1 (ISGMR only)][V-gradient slots][node gradients for mrf_bwd_pairwise_* (gstore_bytes)]
    char *ws = (char *)workspace;
    float *scal = (float *)ws;
    float *buf0 = (float *)(ws + kAlign);                   // ISGMR: grad m-hat   TRWP: s per direction
    float *buf1 = (float *)(ws + kAlign + msg_bytes(pr));   // ISGMR: s per direction
    double *gvslots = (double *)(ws + kAlign + (algo == MRF_ISGMR ? 2 : 1) * msg_bytes(pr));
    P.fault = (int *)(ws + kFaultOffset);
    P.spin_limit = spin_limit();
    if (pr->edge_weight) { P.w = pr->edge_weight; P.w_mul = 1; }
    else { P.w = scal; P.w_mul = 0; }

    long long slots = 0;
    if (grad_V && !edge_tables) {
        P.gV = gvslots;
        slots = slots_in_use(pr, P.g, algo);
        if (gstore_bytes(pr, algo) > 0) P.gstore_buf = (double *)((char *)gvslots + gradv_bytes(pr));
    }
    if (grad_w || slots > 0) {
        const long long n_gw = grad_w ? (long long)R * N : 0, n_slots = slots * L * L;
        long long blocks = ((n_gw > n_slots ? n_gw : n_slots) + 255) / 256;
        if (blocks > 16384) blocks = 16384;
        hipLaunchKernelGGL(mrf_bwd_clear, dim3((unsigned)blocks), dim3(256), 0, st, grad_w, n_gw, gvslots, n_slots, scal,
                           (int *)(ws + kFaultOffset), pr->edge_weight_scalar);
        const hipError_t e_ = hipGetLastError();
        if (e_ != hipSuccess) return hip_fail(e_, "mrf_bwd_clear");
    } else {
        const hipError_t e_ = init_header(workspace, pr->edge_weight_scalar, st);
        if (e_ != hipSuccess) return hip_fail(e_, "init_header");
    }
    // Per-edge tables: the sweeps store the node gradients of as many iterations as the workspace has room for, and
    // mrf_bwd_edge_tables forms the tables' gradient from them.  mrf_bwd_sweep, which adds to the tables itself, keeps TRW
    // coefficients per edge, arrays beyond the 32-bit offsets of the sweeps that store, and launches of more than 8,192
    // scanlines of 33..64 labels, the most that was measured (backward pass with the tables' gradient, storing / adding: TRWP, 64 x 64
    // images, K = 2, 45 labels 2,560 scanlines 1.79 / 3.03 ms, 8,192 5.95 / 8.50; ISGMR, 64 x 192, 33 labels 2,560 0.46 / 0.74, 8,192 1.36 / 1.79,
    // 64 labels, K = 1, 8,192 2.76 / 3.03).
    long long most = 0, all = 0;
    for (int r = 0; r < R; ++r) {
        const long long n = (long long)pr->B * P.g.nscan[r];
        all += n;
        if (n > most) most = n;
    }
    const long long room = (long long)((workspace_bytes - (size_t)((char *)gvslots - ws)) / edge_slab_bytes(pr));
    const int slabs = (int)(room < K ? room : K);
    P.edge = edge_tables && !P.rho_e && NL <= MRF_BUF_MOST && (!grad_V || slabs > 0) &&
             (L <= 32 || (algo == MRF_ISGMR ? all : most) <= 8192) && g_tune_chain != 1 && g_tune_narrow >= 0;
    float *const edge_g = (float *)gvslots;
    // behind the sweeps of iteration k; P.gstore32 holds where the next iteration's go
    const auto edge_pass = [&](int k) -> hipError_t {
        if (!P.edge || !grad_V) return hipSuccess;
        const int done = (K - 1 - k) % slabs + 1;        // iterations stored since the last pass
        P.gstore32 = edge_g + (size_t)(done % slabs) * R * NL;
        return done == slabs || k == 0 ? launch_edge_tables(pr, grad_V, edge_g, p + (size_t)(k + done - 1) * pk, done, K - 1 - k >= slabs, st) : hipSuccess;
    };
    if (P.edge && grad_V) P.gstore32 = edge_g;
    P.force_plain = edge_tables && !P.edge ? 1 : 0;
    if (edge_tables && grad_V && !P.edge) {
        P.gE = grad_V;
        { const hipError_t e_ = fill(grad_V, (long long)R * N * L * L, 0.0f, st); if (e_ != hipSuccess) return hip_fail(e_, "fill"); }
    }

    mark(g_ev_start, st);
    if (algo == MRF_ISGMR) {
        P.r_first = 0; P.r_count = R;
        long long tot = 0;
        for (int r = 0; r < R; ++r) { P.blk_begin[r] = tot; tot += (long long)pr->B * P.g.nscan[r]; }
        P.blk_begin[R] = tot;
        P.total_scanlines = tot;
        P.S = buf1;
        for (int r = 0; r < R; ++r) {
            // one source: grad m-hat^r itself
            P.n_src[r] = 1; P.src_dir[r][0] = (signed char)r; P.coefG[r][0] = 1.0f; P.coefT[r][0] = 0.0f;
            P.carry_scale[r] = 1.0f;
        }
        MrfCombineParams C;
        memset(&C, 0, sizeof(C));
        C.NL = NL; C.R = R; C.skip_dir = -1;
        for (int r = 0; r < R; ++r) {
            C.opp[r] = P.g.opp[r];
            C.canon[r] = (P.g.opp[r] >= 0 && P.g.opp[r] < r) ? P.g.opp[r] : r;
        }
        C.S = buf1; C.gc = grad_cost; C.gunary = grad_unary;
        long long cblocks = (NL + 255) / 256;
        if (cblocks > 32768) cblocks = 32768;
        // four entries per thread where every array starts on a 16-byte boundary
        const bool cvec = (NL % 4 == 0) && (((uintptr_t)buf0 | (uintptr_t)buf1 | (uintptr_t)grad_cost | (uintptr_t)grad_unary) % 16 == 0);
        long long cblocks4 = (NL / 4 + 255) / 256;
        if (cblocks4 > 32768) cblocks4 = 32768;
        if (cblocks4 < 1) cblocks4 = 1;
        // Up to four directions: no combine pass between iterations.  The sweep of direction d in
        // iteration k reads what the other directions scattered in iteration k + 1 itself (grad m-hat^d =
        // sum over r not in {d, d-} of s^r: at most two arrays, against one array plus the combine's 2 R + 2
        // per node) and the sweep of direction 0 adds all of them, and its own s, to grad theta; one
        // combine pass at the end adds what the other directions scattered in the last sweep.  The s
        // arrays of two iterations alternate between the two buffers.
        // Pays where the pass is bound by its launches (the combine passes are a third of them); on the segmentation shape
        // the sweeps, which are bound by instruction issue and latency, lose more on the extra arrays (2.51 against 1.83 ms) than
        // the combine passes cost.  (On the stereo shape, 256 x 512, 96 labels, it is 1.36 against 1.46 ms: the line could lie higher for the
        // chain layout.)
        const bool lazy = R <= 4 && g_tune_isgmr_lazy != 1 && (g_tune_isgmr_lazy == 2 || NL <= (1LL << 19));
        for (int k = K - 1; lazy && k >= 0; --k) {
            float *s_cur = ((K - 1 - k) & 1) ? buf0 : buf1, *s_prev = ((K - 1 - k) & 1) ? buf1 : buf0;
            P.S = s_cur;
            P.unary_dir = 0;
            P.unary_init = (k == K - 1);
            if (k == K - 1) {
                // back Eq. isgmr-aggregation: every direction's message, and theta, receive grad c
                P.src_base = grad_cost; P.src_stride = 0;
                for (int r = 0; r < R; ++r) { P.n_src[r] = 1; P.src_dir[r][0] = (signed char)r; P.coefG[r][0] = 1.0f; P.coefT[r][0] = 1.0f; }
            } else {
                P.src_base = s_prev; P.src_stride = NL;
                for (int d = 0; d < R; ++d) {
                    int n = 0;
                    for (int r = 0; r < R; ++r) {
                        if (r == d) continue;
                        const bool excluded = (r == P.g.opp[d]);          // Eq. isgmr leaves out r and r-
                        if (excluded && d != 0) continue;
                        P.src_dir[d][n] = (signed char)r;
                        P.coefG[d][n] = excluded ? 0.0f : 1.0f;
                        P.coefT[d][n] = 1.0f;                             // (grad theta: read by direction 0 only)
                        ++n;
                    }
                    P.n_src[d] = (signed char)n;
                }
            }
            P.p = p + (size_t)k * pk;
            P.q = q + (size_t)k * qk;
            { const hipError_t e_ = dispatch_bwd(P, pr->pairwise_kind, st); if (e_ != hipSuccess) return hip_fail(e_, "dispatch_bwd"); }
            { const hipError_t e_ = edge_pass(k); if (e_ != hipSuccess) return hip_fail(e_, "mrf_bwd_edge_tables"); }
            if (k == 0) {
                C.S = s_cur; C.first = 0; C.ghat = nullptr; C.skip_dir = 0;
                const dim3 cg((unsigned)(cvec ? cblocks4 : cblocks)), cb(256);
                if (cvec) hipLaunchKernelGGL((mrf_isgmr_bwd_combine<4, 4>), cg, cb, 0, st, C);
                else hipLaunchKernelGGL((mrf_isgmr_bwd_combine<4, 1>), cg, cb, 0, st, C);
                { const hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return hip_fail(e_, "hipGetLastError"); }
            }
        }
        for (int k = K - 1; !lazy && k >= 0; --k) {
            if (k == K - 1) { P.src_base = grad_cost; P.src_stride = 0; }   // back Eq. isgmr-aggregation
            else { P.src_base = buf0; P.src_stride = NL; }
            // (grad m-hat of a direction and of its opposite are the same sum: one array serves both)
            for (int r = 0; r < R; ++r) P.src_dir[r][0] = (signed char)((k == K - 1) ? r : C.canon[r]);
            P.p = p + (size_t)k * pk;
            P.q = q + (size_t)k * qk;
            { const hipError_t e_ = dispatch_bwd(P, pr->pairwise_kind, st); if (e_ != hipSuccess) return hip_fail(e_, "dispatch_bwd"); }
            { const hipError_t e_ = edge_pass(k); if (e_ != hipSuccess) return hip_fail(e_, "mrf_bwd_edge_tables"); }
            C.first = (k == K - 1);
            C.ghat = (k > 0) ? buf0 : nullptr;
            const dim3 cg((unsigned)(cvec ? cblocks4 : cblocks)), cb(256);
            if (R <= 4 && cvec) hipLaunchKernelGGL((mrf_isgmr_bwd_combine<4, 4>), cg, cb, 0, st, C);
            else if (R <= 4) hipLaunchKernelGGL((mrf_isgmr_bwd_combine<4, 1>), cg, cb, 0, st, C);
            else if (R <= 8 && cvec) hipLaunchKernelGGL((mrf_isgmr_bwd_combine<8, 4>), cg, cb, 0, st, C);
            else if (R <= 8) hipLaunchKernelGGL((mrf_isgmr_bwd_combine<8, 1>), cg, cb, 0, st, C);
            else if (cvec) hipLaunchKernelGGL((mrf_isgmr_bwd_combine<16, 4>), cg, cb, 0, st, C);
            else hipLaunchKernelGGL((mrf_isgmr_bwd_combine<16, 1>), cg, cb, 0, st, C);
            { const hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return hip_fail(e_, "hipGetLastError"); }
        }
    } else {
        P.S = buf0;
        P.src_base = buf0; P.src_stride = NL;
        for (int k = K - 1; k >= 0; --k) {
            for (int d = R - 1; d >= 0; --d) {      // reverse of the forward direction order
                P.r_first = d; P.r_count = 1;
                P.blk_begin[0] = 0;
                P.total_scanlines = (long long)pr->B * P.g.nscan[d];
                P.blk_begin[1] = P.total_scanlines;
                // directions that swept since the last sweep of d: all others, except that in the
                // first processed iteration only those after d have swept at all
                int n = 0;
                for (int r = 0; r < R; ++r) {
                    if (r == d || (k == K - 1 && r < d)) continue;
                    P.src_dir[d][n] = (signed char)r;
                    const float rho_r = pr->rho ? pr->rho[r] : 1.0f;   // (not read when rho_edge is given)
                    P.coefG[d][n] = rho_r - (r == P.g.opp[d] ? 1.0f : 0.0f);
                    P.coefT[d][n] = rho_r;
                    ++n;
                }
                P.n_src[d] = (signed char)n;
                P.carry_scale[d] = pr->rho ? pr->rho[d] : 1.0f;
                P.use_gc = (k == K - 1);
                P.unary_dir = d == 0 ? 0 : -1;         // (the sweep of direction 0 forms grad theta_i)
                P.unary_init = (k == K - 1);
                P.p = p + (size_t)k * pk;
                P.q = q + (size_t)k * qk;
                { const hipError_t e_ = dispatch_bwd(P, pr->pairwise_kind, st); if (e_ != hipSuccess) return hip_fail(e_, "dispatch_bwd"); }
            }
            { const hipError_t e_ = edge_pass(k); if (e_ != hipSuccess) return hip_fail(e_, "mrf_bwd_edge_tables"); }
        }
    }
    mark(g_ev_stop, st);
    if (grad_V && !edge_tables) {
        const long long n = (long long)L * L;
        const long long chunk = slots <= MRF_SLOTS_ONE_PASS ? 1 : 64;
        if (chunk > 1) {
            hipLaunchKernelGGL(mrf_reduce_slots<64>, dim3((unsigned)((n + 63) / 64), (unsigned)((slots + chunk - 1) / chunk)), dim3(256),
                               0, st, gvslots, grad_V, n, slots, chunk, 0);
            const hipError_t e_ = hipGetLastError();
            if (e_ != hipSuccess) return hip_fail(e_, "mrf_reduce_slots");
        }
        hipLaunchKernelGGL(mrf_reduce_slots<16>, dim3((unsigned)((n + 15) / 16)), dim3(256), 0, st, gvslots, grad_V, n, slots, chunk, 1);
        { const hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return hip_fail(e_, "mrf_reduce_slots"); }
    }
    return MRF_OK;
}

#endif  // MRF_HAS_BWD

}  // namespace mrf_host

#if MRF_HAS_API
namespace mrf_host {
hipError_t init_header(void *workspace, float w_scalar, hipStream_t st)
{
    hipLaunchKernelGGL(mrf_init_header, dim3(1), dim3(64), 0, st, (float *)workspace,
                       (int *)((char *)workspace + kFaultOffset), w_scalar);
    return hipGetLastError();
}
}  // namespace mrf_host

using namespace mrf_host;

extern "C" {

size_t mrf_workspace_bytes(const mrf_problem *prob, int algo, int backward)
{
    if (check_problem(prob, algo, false) != MRF_OK) return 0;
    if (!backward) return kAlign + (algo == MRF_ISGMR ? 2 : 1) * msg_bytes(prob);
    size_t grads = gradv_bytes(prob) + gstore_bytes(prob, algo);
    if (prob->pairwise_edge && !(algo == MRF_TRWP && prob->rho_edge) && edge_grad_bytes(prob) > grads) grads = edge_grad_bytes(prob);
    return kAlign + (algo == MRF_ISGMR ? 2 : 1) * msg_bytes(prob) + grads;
}

int mrf_validate(const mrf_problem *prob, int algo) { return check_problem(prob, algo, true); }

int mrf_forward_window(const mrf_problem *prob, int algo)
{
    const int rc = check_problem(prob, algo, false);
    if (rc != MRF_OK) return rc;
    // The window sweeps take up to fifteen message arrays next to the unary for TRWP (any direction set the
    // library accepts) and up to seven for ISGMR, whose sweeps read a single array from six directions on
    // (run_forward); count what an ISGMR launch of the later iterations reads with fewer directions.
    if (algo == MRF_ISGMR && !(prob->R >= 6 && prob->K > 1)) {
        int most = 0;
        for (int r = 0; r < prob->R; ++r) {
            bool has_opp = false;
            for (int d = 0; d < prob->R; ++d)
                if (prob->dirs[2 * d] == -prob->dirs[2 * r] && prob->dirs[2 * d + 1] == -prob->dirs[2 * r + 1]) has_opp = true;
            const int n = prob->R - 1 - (has_opp ? 1 : 0);
            if (n > most) most = n;
        }
        if (most + 1 > 8) return 0;
    }
    return window_width(prob);
}

int mrf_isgmr_forward(const mrf_problem *prob, float *cost, uint8_t *labels, uint8_t *p, uint8_t *q,
                      float *messages, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return run_forward(prob, MRF_ISGMR, cost, labels, p, q, messages, workspace, workspace_bytes, hip_stream);
}

int mrf_trwp_forward(const mrf_problem *prob, float *cost, uint8_t *labels, uint8_t *p, uint8_t *q,
                     float *messages, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return run_forward(prob, MRF_TRWP, cost, labels, p, q, messages, workspace, workspace_bytes, hip_stream);
}

int mrf_isgmr_backward(const mrf_problem *prob, const float *grad_cost, const uint8_t *p, const uint8_t *q,
                       float *grad_unary, float *grad_edge_weight, float *grad_pairwise,
                       void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return run_backward(prob, MRF_ISGMR, grad_cost, p, q, grad_unary, grad_edge_weight, grad_pairwise,
                        workspace, workspace_bytes, hip_stream);
}

int mrf_trwp_backward(const mrf_problem *prob, const float *grad_cost, const uint8_t *p, const uint8_t *q,
                      float *grad_unary, float *grad_edge_weight, float *grad_pairwise,
                      void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return run_backward(prob, MRF_TRWP, grad_cost, p, q, grad_unary, grad_edge_weight, grad_pairwise,
                        workspace, workspace_bytes, hip_stream);
}

int64_t mrf_scanline_count(int32_t H, int32_t W, int32_t dh, int32_t dw)
{
    if (H < 1 || W < 1) return MRF_ERR_BAD_SHAPE;
    if (dh == 0 && dw == 0) return MRF_ERR_BAD_DIRECTIONS;
    return mrf_geom_scanlines(H, W, dh, dw);
}

int mrf_scanline_head(int32_t H, int32_t W, int32_t dh, int32_t dw, int64_t t,
                      int32_t *y0, int32_t *x0, int32_t *len)
{
    if (!y0 || !x0 || !len) return MRF_ERR_NULL_POINTER;
    if (H < 1 || W < 1) return MRF_ERR_BAD_SHAPE;
    if (dh == 0 && dw == 0) return MRF_ERR_BAD_DIRECTIONS;
    if (t < 0 || t >= mrf_geom_scanlines(H, W, dh, dw)) return MRF_ERR_BAD_SHAPE;
    int a, b, c;
    mrf_geom_head(H, W, dh, dw, t, a, b, c);
    *y0 = a; *x0 = b; *len = c;
    return MRF_OK;
}

const char *mrf_strerror(int status)
{
    switch (status) {
    case MRF_OK: return "ok";
    case MRF_ERR_NULL_POINTER: return "a required pointer is NULL";
    case MRF_ERR_BAD_SHAPE: return "B, H, W must be >= 1 and B*H*W < 2^31";
    case MRF_ERR_BAD_LABELS: return "L must be in [1, 256]";
    case MRF_ERR_BAD_ITERATIONS: return "K must be >= 1";
    case MRF_ERR_BAD_DIRECTIONS: return "R must be in [1, 16], steps non-zero and distinct";
    case MRF_ERR_WORKSPACE_TOO_SMALL: return "workspace smaller than mrf_workspace_bytes()";
    case MRF_ERR_BAD_PAIRWISE_KIND: return "unknown pairwise_kind, invalid trunc or negative scale";
    case MRF_ERR_BAD_ALGORITHM: return "algo must be MRF_ISGMR or MRF_TRWP";
    case MRF_ERR_HIP: return "HIP runtime call or kernel launch failed";
    case MRF_ERR_WAIT_EXPIRED: return "a wait between wavefronts of a sweep ran out of its budget: the results of that call are incomplete";
    case MRF_ERR_SCRATCH_LIMIT: return "problem exceeds the fixed scratch of a no-allocation entry point (batch > 64)";
    default: return "unknown status";
    }
}

size_t mrf_energy_workspace_bytes(const mrf_problem *prob)
{
    if (check_problem(prob, MRF_ISGMR, false) != MRF_OK) return 0;
    return sizeof(double) * (size_t)prob->B * MRF_HEAD_BLOCKS;
}

// launches of mrf_energy on `partial`, which holds B * MRF_HEAD_BLOCKS doubles
static int energy_launch(const mrf_problem *prob, const uint8_t *labels, double *energy, double *partial,
                         hipStream_t st)
{
    MrfEnergyParams E;
    memset(&E, 0, sizeof(E));
    fill_geom(prob, E.g);
    E.unary = prob->unary; E.V = prob->pairwise; E.Te = prob->pairwise_edge; E.labels = labels;
    E.partial = partial;
    if (prob->edge_weight) { E.w = prob->edge_weight; E.w_mul = 1; }
    else { E.w = nullptr; E.w_mul = 0; }
    for (int r = 0; r < prob->R; ++r)
        if (E.g.opp[r] < 0 || r < E.g.opp[r]) E.edge_dir[E.n_edge_dir++] = r;
    const long long HW = (long long)prob->H * prob->W;
    long long blocks = (HW + 255) / 256;
    if (blocks > MRF_HEAD_BLOCKS) blocks = MRF_HEAD_BLOCKS;
    E.w_scalar = prob->edge_weight_scalar;
    hipLaunchKernelGGL(mrf_energy_partial, dim3((unsigned)blocks, (unsigned)prob->B), dim3(256), 0, st, E);
    { const hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return hip_fail(e_, "mrf_energy_partial"); }
    hipLaunchKernelGGL(mrf_sum_partials, dim3((unsigned)prob->B), dim3(1024), 0, st, (const double *)E.partial, (int)blocks,
                       energy, (const long long *)nullptr);
    { const hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return hip_fail(e_, "mrf_sum_partials"); }
    return MRF_OK;
}

int mrf_energy(const mrf_problem *prob, const uint8_t *labels, double *energy, void *workspace,
               size_t workspace_bytes, void *hip_stream)
{
    const int rc = check_problem(prob, MRF_ISGMR, true);
    if (rc != MRF_OK) return rc;
    if (!labels || !energy || !workspace) return MRF_ERR_NULL_POINTER;
    if (workspace_bytes < mrf_energy_workspace_bytes(prob)) return MRF_ERR_WORKSPACE_TOO_SMALL;
    return energy_launch(prob, labels, energy, (double *)workspace, (hipStream_t)hip_stream);
}

// ---- mrf_energy for callers that cannot allocate: the partial sums live in a device array of the
// library's own.  Every GPU holds its own copy of the array at its own address; the name below is
// only the host-side handle of the symbol, so host code asks the runtime once per device where the
// copy lives and passes that pointer on.
static __device__ __align__(256) double mrf_energy_scratch[(size_t)MRF_ENERGY_NOALLOC_MAX_BATCH * MRF_HEAD_BLOCKS];
#define MRF_MAX_DEVICES 64
static double *g_energy_scratch_ptr[MRF_MAX_DEVICES];     // per device, set on the first call there

int mrf_energy_noalloc(const mrf_problem *prob, const uint8_t *labels, double *energy, void *hip_stream)
{
    const int rc = check_problem(prob, MRF_ISGMR, true);
    if (rc != MRF_OK) return rc;
    if (!labels || !energy) return MRF_ERR_NULL_POINTER;
    if (prob->B > MRF_ENERGY_NOALLOC_MAX_BATCH) return MRF_ERR_SCRATCH_LIMIT;
    int dev = -1;
    { const hipError_t e_ = hipGetDevice(&dev); if (e_ != hipSuccess) return hip_fail(e_, "hipGetDevice"); }
    if (dev < 0 || dev >= MRF_MAX_DEVICES) return MRF_ERR_SCRATCH_LIMIT;
    if (!g_energy_scratch_ptr[dev]) {
        double *ptr = nullptr;
        const hipError_t e_ = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(mrf_energy_scratch));
        if (e_ != hipSuccess || !ptr) return hip_fail(e_, "hipGetSymbolAddress(mrf_energy_scratch)");
        g_energy_scratch_ptr[dev] = ptr;
    }
    // (every partial sum the second kernel reads is written by the first: nothing has to start at zero)
    return energy_launch(prob, labels, energy, g_energy_scratch_ptr[dev], (hipStream_t)hip_stream);
}

size_t mrf_softmin_l1_workspace_bytes(void)
{
    return kAlign + (sizeof(double) + sizeof(long long)) * MRF_HEAD_BLOCKS;
}

static int softmin_loss(int64_t n_pixels, int32_t L, const float *cost, const float *target, const uint8_t *mask,
                        float *disparity, double *loss, float *grad_cost, double beta, void *workspace,
                        size_t workspace_bytes, void *hip_stream);

int mrf_softmin_l1(int64_t n_pixels, int32_t L, const float *cost, const float *target, const uint8_t *mask,
                   float *disparity, double *loss, float *grad_cost, void *workspace, size_t workspace_bytes,
                   void *hip_stream)
{
    return softmin_loss(n_pixels, L, cost, target, mask, disparity, loss, grad_cost, 0.0, workspace, workspace_bytes,
                        hip_stream);
}

int mrf_softmin_smooth_l1(int64_t n_pixels, int32_t L, const float *cost, const float *target, const uint8_t *mask,
                          float beta, float *disparity, double *loss, float *grad_cost, void *workspace,
                          size_t workspace_bytes, void *hip_stream)
{
    if (!(beta > 0.0f) || !(beta < INFINITY)) return MRF_ERR_BAD_PAIRWISE_KIND;
    return softmin_loss(n_pixels, L, cost, target, mask, disparity, loss, grad_cost, (double)beta, workspace,
                        workspace_bytes, hip_stream);
}

static int softmin_loss(int64_t n_pixels, int32_t L, const float *cost, const float *target, const uint8_t *mask,
                        float *disparity, double *loss, float *grad_cost, double beta, void *workspace,
                        size_t workspace_bytes, void *hip_stream)
{
    if (n_pixels < 1 || n_pixels > 0x7fffffffLL) return MRF_ERR_BAD_SHAPE;
    if (L < 1 || L > MRF_MAX_LABELS) return MRF_ERR_BAD_LABELS;
    if (!cost || !target || !loss || !workspace) return MRF_ERR_NULL_POINTER;
    if (workspace_bytes < mrf_softmin_l1_workspace_bytes()) return MRF_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t st = (hipStream_t)hip_stream;
    MrfLossParams Q;
    memset(&Q, 0, sizeof(Q));
    Q.N = n_pixels; Q.L = L; Q.cost = cost; Q.target = target; Q.mask = mask;
    Q.disparity = disparity; Q.grad_cost = grad_cost; Q.beta = beta;
    Q.count = (long long *)workspace;
    Q.partial = (double *)((char *)workspace + kAlign);
    Q.cpartial = (long long *)((char *)workspace + kAlign + sizeof(double) * MRF_HEAD_BLOCKS);
    if (mask) {
        long long cb = (n_pixels + 255) / 256;
        if (cb > MRF_HEAD_BLOCKS) cb = MRF_HEAD_BLOCKS;
        hipLaunchKernelGGL(mrf_count_mask_partial, dim3((unsigned)cb), dim3(256), 0, st, Q);
        hipLaunchKernelGGL(mrf_count_mask_final, dim3(1), dim3(64), 0, st, Q, (int)cb);
    } else {
        hipLaunchKernelGGL(mrf_set_i64, dim3(1), dim3(64), 0, st, Q.count, (long long)n_pixels);
    }
    { const hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return hip_fail(e_, "mrf_softmin_l1 count"); }
    long long blocks = (n_pixels + 3) / 4;
    if (blocks > MRF_HEAD_BLOCKS) blocks = MRF_HEAD_BLOCKS;
    const int slots = (L + 63) / 64;
    if (slots == 1) hipLaunchKernelGGL(mrf_softmin_l1_kernel<1>, dim3((unsigned)blocks), dim3(256), 0, st, Q);
    else if (slots == 2) hipLaunchKernelGGL(mrf_softmin_l1_kernel<2>, dim3((unsigned)blocks), dim3(256), 0, st, Q);
    else if (slots == 3) hipLaunchKernelGGL(mrf_softmin_l1_kernel<3>, dim3((unsigned)blocks), dim3(256), 0, st, Q);
    else hipLaunchKernelGGL(mrf_softmin_l1_kernel<4>, dim3((unsigned)blocks), dim3(256), 0, st, Q);
    { const hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return hip_fail(e_, "mrf_softmin_l1_kernel"); }
    hipLaunchKernelGGL(mrf_sum_partials, dim3(1), dim3(1024), 0, st, (const double *)Q.partial, (int)blocks, loss,
                       (const long long *)Q.count);
    { const hipError_t e_ = hipGetLastError(); if (e_ != hipSuccess) return hip_fail(e_, "mrf_sum_partials"); }
    return MRF_OK;
}

// Which forward or backward call used this workspace last, did one of its waits between
// wavefronts run out?  Waits for the stream, then reads the fault word of the header.
int mrf_workspace_fault(const void *workspace, void *hip_stream)
{
    if (!workspace) return MRF_ERR_NULL_POINTER;
    hipStream_t st = (hipStream_t)hip_stream;
    { const hipError_t e_ = hipStreamSynchronize(st); if (e_ != hipSuccess) return hip_fail(e_, "hipStreamSynchronize"); }
    int word = 0;
    { const hipError_t e_ = hipMemcpy(&word, (const char *)workspace + kFaultOffset, sizeof(int), hipMemcpyDeviceToHost);
      if (e_ != hipSuccess) return hip_fail(e_, "hipMemcpy"); }
    return word != 0 ? MRF_ERR_WAIT_EXPIRED : MRF_OK;
}

const char *mrf_last_error_detail(void) { return g_error_detail; }

const char *mrf_last_sweep_kernel(int backward) { return g_last_sweep[backward ? 1 : 0]; }

const char *mrf_last_sweep_launch(int backward) { return g_last_launch[backward ? 1 : 0]; }

const char *mrf_version(void) { return "0.3.10"; }

int mrf_set_sweep_events(void *start_event, void *stop_event)
{
    g_ev_start = (hipEvent_t)start_event;
    g_ev_stop = (hipEvent_t)stop_event;
    return MRF_OK;
}

int mrf_tune(int knob, int value)
{
    if (knob == 0) { g_tune_mch = value; return MRF_OK; }
    if (knob == 1) { g_tune_no_window = value; return MRF_OK; }
    if (knob == 2) { g_tune_split = value; return MRF_OK; }
    if (knob == 3) {
        g_tune_narrow = (value == 8 || value == 16 || value == 32) ? value : (value == 3 ? -1 : 0);
        g_tune_pack = g_tune_narrow ? 2 : value;
        return MRF_OK;
    }
    if (knob == 4) { g_tune_duo = value; return MRF_OK; }
    if (knob == 5) { g_tune_duo_ni = (value == 1 || value == 2) ? value : 0; return MRF_OK; }
    if (knob == 6) { g_tune_chain = value; return MRF_OK; }
    if (knob == 12) { g_tune_chain_hot = value; return MRF_OK; }
    if (knob == 8) { g_tune_loader = value; return MRF_OK; }
    if (knob == 9) { g_tune_squad = value; return MRF_OK; }
    if (knob == 11) { g_tune_pack_idx = value; return MRF_OK; }
    if (knob == 10) { g_tune_squad_ni = value; return MRF_OK; }
    if (knob == 13) { g_tune_pack3 = value; return MRF_OK; }
    if (knob == 14) { g_tune_spin_limit = value > 0 ? value : 0; return MRF_OK; }
    if (knob == 15) { g_tune_isgmr_lazy = value; return MRF_OK; }
    if (knob == 16) { g_tune_dense_sliced = value; return MRF_OK; }
    if (knob == 17) { g_tune_isgmr_presum = value; return MRF_OK; }
    if (knob == 18) { g_tune_gv_tile = value; return MRF_OK; }
    if (knob == 19) { g_tune_gv_apart = value; return MRF_OK; }
    if (knob == 20) {
        // (3, 4: by launch size, and the narrow sweep never / whenever possible divided among four wavefronts)
        g_tune_chain_pk = value <= 2 ? value : 0;
        g_tune_narrow_divided = value == 3 ? 1 : (value == 4 ? 2 : 0);
        return MRF_OK;
    }
    if (knob == 7) { g_tune_chain_ni = (value == 2 || value == 4 || value == 6 || value == 8 || value == 12) ? value : 0; return MRF_OK; }
    return MRF_ERR_BAD_ALGORITHM;
}

}  // extern "C"
#endif  // MRF_HAS_API
