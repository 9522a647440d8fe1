"""GPU parity: the HIP path (through the C-ABI library) against the CPU oracle, element by
element, on the same seeded inputs.

Bar: p, q, labels bit-exact (the argmins are decided in float32 on both sides, lowest
index on ties); costs and messages within 1e-5 relative / 1e-4 absolute (they are in fact
expected to be identical: same operations in the same order); gradients within the same
tolerance of the oracle's double instantiation replaying the same indices (the library
carries its sums in double and rounds once on store; the float32 instantiation of the
oracle rounds after every addition and is itself up to about one tolerance away from the
double one on the larger problems -- its distance is printed, not asserted).
"""
import os

import numpy as np
import pytest

from mrf_inputs import DIRS4, DIRS8, DIRS16, make_config, random_problem

pytestmark = pytest.mark.gpu

RTOL, ATOL = 1e-5, 1e-4


def oracle_forward(oracle, pr, threads=False):
    return oracle.forward(pr.algo, pr.unary, pr.pairwise, pr.dirs, pr.K, edge_weight=pr.edge_weight,
                          edge_weight_scalar=pr.edge_weight_scalar, rho=pr.rho, threads=threads,
                          rho_edge=pr.rho_edge)


def oracle_backward(oracle, pr, p, q, dtype=np.float32):
    c = lambda a: None if a is None else a.astype(dtype)
    return oracle.backward(pr.algo, pr.shape, c(pr.pairwise), pr.dirs, pr.K, c(pr.grad_cost), p, q,
                           edge_weight=c(pr.edge_weight), edge_weight_scalar=pr.edge_weight_scalar,
                           rho=pr.rho, dtype=dtype, rho_edge=c(pr.rho_edge))


def check_forward(g, f):
    np.testing.assert_array_equal(g.p, f.p)
    np.testing.assert_array_equal(g.q, f.q)
    np.testing.assert_array_equal(g.labels, f.labels)
    np.testing.assert_allclose(g.messages, f.messages, rtol=RTOL, atol=ATOL)
    np.testing.assert_allclose(g.cost, f.cost, rtol=RTOL, atol=ATOL)


def check_grad(name, got, ref32, ref64):
    """Asserts against the double replay alone; ref32 (the float32 oracle, may be None) only
    adds its own distance to the message."""
    assert np.isfinite(got).all(), name
    e64 = np.abs(got.astype(np.float64) - ref64) / (ATOL + RTOL * np.abs(ref64))
    worst = e64.max() if e64.size else 0.0
    if worst > 1.0:
        e32 = -1.0 if ref32 is None else (np.abs(got.astype(np.float64) - ref32) / (ATOL + RTOL * np.abs(ref32))).max()
        raise AssertionError("%s: worst error/tolerance vs double replay %.3f (vs f32 oracle %.3f)" % (name, worst, e32))


def check_backward(g, b32, b64, want_V=True):
    f = lambda name: None if b32 is None else getattr(b32, name)
    check_grad("grad_unary", g.grad_unary, f("grad_unary"), b64.grad_unary)
    check_grad("grad_edge_weight", g.grad_edge_weight, f("grad_edge_weight"), b64.grad_edge_weight)
    if want_V:
        check_grad("grad_pairwise", g.grad_pairwise, f("grad_pairwise"), b64.grad_pairwise)


def full_check(oracle, pr, threads=False, want_V=True):
    """want_V=False: the caller passes no grad_pairwise buffer (a model whose V has no free
    parameters); the library may then pick other backward kernels."""
    from gpu_harness import run_gpu
    g = run_gpu(pr, want_V=want_V)
    f = oracle_forward(oracle, pr, threads=threads)
    check_forward(g, f)
    b32 = oracle_backward(oracle, pr, f.p, f.q, np.float32)
    b64 = oracle_backward(oracle, pr, f.p, f.q, np.float64)
    check_backward(g, b32, b64, want_V)
    return g


CONFIG_CASES = [
    (1, None, "isgmr", None), (1, None, "trwp", None),
    (2, (24, 40), "trwp", None), (2, (24, 40), "isgmr", None),
    (3, (12, 20), "isgmr", None), (3, (12, 20), "trwp", None),
    (4, (10, 12), "trwp", 3), (4, (10, 12), "isgmr", 2),
    (5, (24, 32), "isgmr", None), (5, (24, 32), "trwp", None),
]


@pytest.mark.parametrize("index,crop,algo,K", CONFIG_CASES)
def test_benchmark_configs_cropped(oracle, index, crop, algo, K):
    print("case config", index, crop, algo, K, flush=True)
    pr = make_config(index, crop=crop, algo=algo, K=K)
    full_check(oracle, pr)


RANDOM_CASES = [
    # seed, algo, B, H, W, L, dirs, K, integer_valued, per_edge
    (1, "isgmr", 1, 5, 7, 1, DIRS4, 2, False, True),
    (2, "trwp", 1, 5, 7, 2, DIRS4, 2, False, True),
    (3, "isgmr", 2, 6, 5, 33, DIRS8, 2, False, True),
    (4, "trwp", 2, 6, 5, 65, DIRS8, 2, False, False),
    (5, "isgmr", 1, 7, 6, 100, DIRS16, 2, False, True),
    (6, "trwp", 1, 7, 6, 129, DIRS16, 2, False, True),
    (7, "isgmr", 1, 4, 9, 200, DIRS4, 3, False, False),
    (8, "trwp", 1, 9, 4, 255, DIRS4, 2, False, True),
    (9, "isgmr", 1, 8, 8, 7, DIRS8, 3, True, True),      # integer data: many ties
    (10, "trwp", 1, 8, 8, 70, DIRS4, 3, True, True),
    (11, "isgmr", 1, 1, 12, 12, DIRS8, 2, False, True),   # one row: vertical/diagonal scanlines have one node
    (12, "trwp", 1, 12, 1, 12, DIRS8, 2, False, True),    # one column
    (13, "isgmr", 1, 6, 6, 16, [(0, 1), (1, 0)], 3, False, True),        # no opposite directions
    (14, "trwp", 1, 6, 6, 16, [(0, 1), (1, 0), (-1, 0)], 3, False, True),
    (15, "trwp", 3, 5, 5, 64, DIRS4, 2, False, True),
    (16, "isgmr", 1, 1, 1, 5, DIRS4, 2, False, True),     # single node: nothing to pass
]


@pytest.mark.parametrize("case", RANDOM_CASES, ids=lambda c: "seed%d" % c[0])
def test_random_shapes(oracle, case):
    print("case random", case[:8], flush=True)
    seed, algo, B, H, W, L, dirs, K, iv, pe = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=pe,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    full_check(oracle, pr)


@pytest.mark.parametrize("algo", ["isgmr", "trwp"])
def test_asymmetric_pairwise(oracle, algo):
    print("case asymmetric", algo, flush=True)
    pr = random_problem(21, algo, 1, 6, 7, 40, DIRS8, 2, symmetric=False)
    full_check(oracle, pr)


@pytest.mark.parametrize("mch", [8, 16, 32])
def test_wavefront_split_does_not_change_results(oracle, mch):
    """The number of source labels per wavefront is a tuning knob; p, q and messages must not
    depend on it."""
    import paper_1910_10892_amd as mrf
    print("case tune", mch, flush=True)
    try:
        assert mrf.mrf_tune(0, mch) == 0
        for L in (48, 96, 130):
            pr = random_problem(30 + L, "trwp", 1, 5, 6, L, DIRS4, 2)
            full_check(oracle, pr)
    finally:
        mrf.mrf_tune(0, 0)


@pytest.mark.parametrize("case", [
    (601, "trwp", 1, 5, 9, 65, DIRS4, 2, False), (602, "isgmr", 2, 4, 7, 96, DIRS8, 2, True),
    (603, "trwp", 1, 6, 5, 130, DIRS8, 2, False), (604, "isgmr", 1, 3, 11, 192, DIRS16, 2, False),
    (605, "trwp", 1, 7, 6, 255, DIRS4, 3, True), (606, "isgmr", 1, 4, 8, 256, DIRS4, 2, False),
    (607, "trwp", 1, 3, 40, 100, [(0, 1), (1, 0), (-1, 0)], 2, False),
], ids=lambda c: "seed%d" % c[0])
def test_dense_sweep_with_a_slice_of_labels_per_wavefront(oracle, case):
    """More than 64 labels, general dense table: the sweep in which every wavefront owns 32 labels
    against the oracle, and bit for bit against the sweep in which every wavefront does the O(L) work
    of the whole node."""
    import paper_1910_10892_amd as mrf
    print("case dense sliced", case[:8], flush=True)
    seed, algo, B, H, W, L, dirs, K, iv = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, symmetric=False,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    try:
        assert mrf.mrf_tune(16, 2) == 0
        a = full_check(oracle, pr, want_V=False)
        assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_sliced"
        assert mrf.mrf_tune(16, 1) == 0
        b = full_check(oracle, pr, want_V=False)
        assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep"
    finally:
        mrf.mrf_tune(16, 0)
    for name in ("p", "q", "labels", "cost", "messages"):
        np.testing.assert_array_equal(getattr(a, name), getattr(b, name), err_msg=name)


HALVES_CASES = [
    # seed, algo, B, H, W, L, dirs, K, integer_valued, V: "plain" (>= 0, zero diagonal) | "mixed signs", some weights negative
    (611, "trwp", 1, 5, 9, 33, DIRS4, 3, False, "plain", False), (612, "isgmr", 2, 4, 7, 64, DIRS8, 2, True, "plain", False),
    (613, "trwp", 1, 6, 5, 65, DIRS8, 2, False, "plain", True), (614, "isgmr", 1, 3, 11, 96, DIRS16, 2, False, "mixed", False),
    (615, "trwp", 1, 7, 6, 97, DIRS4, 3, True, "mixed", True), (616, "isgmr", 1, 4, 8, 128, DIRS4, 2, False, "plain", True),
    (617, "trwp", 1, 1, 40, 127, [(0, 1), (1, 0), (-1, 0)], 2, True, "plain", False), (618, "trwp", 1, 3, 7, 40, DIRS16, 2, True, "plain", False),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", HALVES_CASES, ids=lambda c: "seed%d" % c[0])
def test_dense_sweep_with_chunk_minima(oracle, case):
    """33..128 labels, dense table: the sweep that finds the argmin by a second look at the winning chunk, with
    tables for which the minimum of the new message is that of h and with tables and weights for which it is not,
    ties included; against the oracle and bit for bit against the sweep with a running argmin."""
    import paper_1910_10892_amd as mrf
    seed, algo, B, H, W, L, dirs, K, iv, table, neg = case
    print("case dense halves", case[:6], len(dirs), case[7:], flush=True)
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, symmetric=False, rho=np.linspace(0.3, 0.9, len(dirs)))
    pr.grad_cost = (pr.grad_cost * (0.02 if len(dirs) > 8 else 0.2)).astype(np.float32)
    if table == "plain":
        np.fill_diagonal(pr.pairwise, 0.0)
    else:
        pr.pairwise = (pr.pairwise - np.float32(1.0 if iv else 0.3)).astype(np.float32)
    if neg:
        sign = np.where(np.random.default_rng(seed).random(pr.edge_weight.shape) > 0.2, 1.0, -0.5)
        pr.edge_weight = (pr.edge_weight * sign).astype(np.float32)
    try:
        assert mrf.mrf_tune(16, 3) == 0
        a = full_check(oracle, pr, want_V=False)
        assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_halves", mrf.mrf_last_sweep_launch(False)
        assert mrf.mrf_tune(16, 1) == 0
        b = full_check(oracle, pr, want_V=False)
        assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep"
    finally:
        mrf.mrf_tune(16, 0)
    for name in ("p", "q", "labels", "cost", "messages"):
        np.testing.assert_array_equal(getattr(a, name), getattr(b, name), err_msg=name)


@pytest.mark.gpu
@pytest.mark.parametrize("L", [33, 40, 64, 70, 96, 128])
@pytest.mark.parametrize("algo", ["isgmr", "trwp"])
def test_chunk_minima_where_no_label_is_possible(algo, L):
    """Infinite or NaN unaries for all labels of a pixel, and masks with transitions between equal labels only, make
    messages NaN: the argmins are still labels, those of the sweep with a running argmin."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    for kind in ("infinite", "nan", "masks"):
        print("case no possible label", algo, L, kind, flush=True)
        pr = random_problem(620 + L, algo, 1, 6, 9, L, DIRS8, 2, symmetric=False)
        np.fill_diagonal(pr.pairwise, 0.0)
        if kind == "masks":
            mask = np.random.default_rng(L).random(pr.unary.shape) < 0.3
            mask[..., L // 2] = False
            pr.unary[mask] = np.inf
            pr.pairwise[~np.eye(L, dtype=bool)] = np.inf
        else:
            pr.unary[:, 3, 4, :] = np.inf if kind == "infinite" else np.nan
        try:
            assert mrf.mrf_tune(16, 3) == 0
            a = run_gpu(pr, backward=False)
            assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_halves", mrf.mrf_last_sweep_launch(False)
            assert mrf.mrf_tune(16, 1) == 0
            b = run_gpu(pr, backward=False)
            assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep"
        finally:
            mrf.mrf_tune(16, 0)
        assert a.p.max() < L and a.q.max() < L
        for name in ("p", "q", "labels", "cost", "messages"):
            np.testing.assert_array_equal(getattr(a, name), getattr(b, name), err_msg=name)


@pytest.mark.parametrize("L", [5, 13, 21, 32, 40, 96])
def test_impossible_labels_and_forbidden_transitions(oracle, L):
    """Infinite unaries and infinite entries of V (one label of every pixel and the diagonal stay finite): the argmins of
    the oracle, also where every candidate is infinite."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    pr = random_problem(630 + L, "isgmr", 2, 7, 9, L, DIRS8, 2, symmetric=False)
    rng = np.random.default_rng(L)
    mask = rng.random(pr.unary.shape) < 0.3
    mask[..., L // 2] = False
    pr.unary[mask] = np.inf
    never = rng.random(pr.pairwise.shape) < 0.5
    np.fill_diagonal(never, False)
    pr.pairwise[never] = np.inf
    f = oracle_forward(oracle, pr)
    print("case impossible labels", L, flush=True)
    try:
        assert mrf.mrf_tune(3, 2) == 0 and mrf.mrf_tune(11, 1) == 0 and mrf.mrf_tune(16, 3) == 0
        g = run_gpu(pr, backward=False)
        assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_" + ("narrow" if L <= 32 else "halves")
    finally:
        for knob in (3, 11, 16):
            mrf.mrf_tune(knob, 0)
    for name in ("p", "q", "labels", "cost", "messages"):
        np.testing.assert_array_equal(getattr(g, name), getattr(f, name), err_msg=name)


def not_finite(pr, kind, seed):
    """Writes infinities or NaN into a problem: what the oracle makes of them is a running argmin from infinity, with NaN passed over."""
    rng = np.random.default_rng(seed)
    L = pr.unary.shape[-1]
    if kind == "masks":                       # some labels of every pixel, and transitions, cannot be
        mask = rng.random(pr.unary.shape) < 0.3
        mask[..., L // 2] = False
        pr.unary[mask] = np.inf
        if pr.pairwise_kind == 0:
            never = rng.random(pr.pairwise.shape) < 0.5
            np.fill_diagonal(never, False)
            pr.pairwise[never] = np.inf
    elif kind == "infinite":                  # one pixel without a possible label, in the middle of scanlines
        pr.unary[:, 3, 4, :] = np.inf
    elif kind == "nan":                       # one pixel whose upper labels are not numbers, one with none that is
        pr.unary[:, 3, 4, :L // 2] = np.nan
        pr.unary[:, 2, 6, :] = np.nan
    elif kind == "weight":
        pr.edge_weight[:, :, 2, 5] = np.inf
    return pr


# (masks: TRWP forms 0 x inf and inf - inf from them, so that whole groups of candidates are NaN beside finite ones)
@pytest.mark.parametrize("kind", ["masks", "infinite", "nan", "weight"])
@pytest.mark.parametrize("algo", ["isgmr", "trwp"])
@pytest.mark.parametrize("L", [3, 8, 13, 16, 17, 21, 24, 32])
def test_few_labels_that_are_not_finite_by_the_default_rules(oracle, L, algo, kind):
    """The packed sweep divided among four wavefronts, which small launches get: indices, costs and messages of the oracle where
    labels are impossible, pixels have none, or a weight is infinite; one and several scanlines per wavefront."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    print("case not finite", L, algo, kind, flush=True)
    for zero_diagonal in (True, False):
        pr = random_problem(650 + L, algo, 2, 7, 9, L, DIRS4, 2, symmetric=False, rho=np.linspace(0.3, 0.9, 4))
        if zero_diagonal:
            np.fill_diagonal(pr.pairwise, 0.0)
        not_finite(pr, kind, L)
        with np.errstate(all="ignore"):
            f = oracle_forward(oracle, pr)
        try:
            for knobs in ((0, 0), (4, 0), (5, 0), (2, 2)) if 16 < L <= 21 else ((0, 0), (4, 0), (5, 0)):
                assert mrf.mrf_tune(11, knobs[0]) == 0 and mrf.mrf_tune(13, knobs[1]) == 0
                g = run_gpu(pr, backward=False)
                assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_packed"
                for name in ("p", "q", "cost", "messages"):
                    np.testing.assert_array_equal(getattr(g, name), getattr(f, name), err_msg="%s %s" % (name, knobs))
                some = ~np.isnan(f.cost).any(-1)      # (mrf_aggregate names no label for a pixel whose costs are not numbers)
                np.testing.assert_array_equal(g.labels[some], f.labels[some])
        finally:
            mrf.mrf_tune(11, 0)
            mrf.mrf_tune(13, 0)


@pytest.mark.parametrize("B,H,L,dirs,kernel", [
    (64, 8, 8, DIRS4, "mrf_bwd_sweep_chain_pk"), (65, 8, 8, DIRS4, "mrf_bwd_sweep_narrow"), (128, 8, 16, DIRS4, "mrf_bwd_sweep_narrow"),
    (125, 8, 12, DIRS16, "mrf_bwd_sweep_chain"), (128, 8, 17, DIRS4, "mrf_bwd_sweep_chain_pk"),
    (112, 8, 16, DIRS8, "mrf_bwd_sweep_chain_pk"), (113, 8, 16, DIRS8, "mrf_bwd_sweep_narrow"), (320, 8, 19, DIRS4, "mrf_bwd_sweep_chain_pk"),
    (128, 8, 21, DIRS4, "mrf_bwd_sweep_chain_pk"), (129, 8, 21, DIRS4, "mrf_bwd_sweep_narrow"), (64, 8, 28, DIRS4, "mrf_bwd_sweep_chain_pk"),
    (65, 8, 28, DIRS4, "mrf_bwd_sweep_narrow")])
def test_which_backward_sweep_runs_for_few_labels(oracle, B, H, L, dirs, kernel):
    """Both sides of the bounds between two scanlines per workgroup and the narrow sweep (TRWP; the last launch is that of the first
    direction, B H scanlines): never the chain of one scanline between them (sixteen directions have neither)."""
    import paper_1910_10892_amd as mrf
    print("case which backward sweep", B, H, L, len(dirs), flush=True)
    pr = random_problem(645 + L, "trwp", B, H, 5, L, dirs, 2, symmetric=False, rho=np.linspace(0.3, 0.9, len(dirs)))
    full_check(oracle, pr)
    assert mrf.mrf_last_sweep_kernel(True) == kernel, mrf.mrf_last_sweep_launch(True)


@pytest.mark.parametrize("B,H,W,L,dirs,kernel", [
    (38, 16, 16, 64, DIRS4, "chain"), (39, 16, 16, 64, DIRS4, ""), (40, 16, 16, 63, DIRS4, "chain"), (41, 16, 16, 63, DIRS4, ""),
    (31, 16, 16, 128, DIRS4, "chain"), (32, 16, 16, 128, DIRS4, ""), (40, 16, 16, 127, DIRS4, "chain"), (24, 16, 16, 192, DIRS4, "chain"),
    (25, 16, 16, 192, DIRS4, ""), (38, 16, 16, 191, DIRS4, "chain"), (39, 16, 16, 191, DIRS4, ""), (15, 16, 16, 128, DIRS8, "chain"),
    (16, 16, 16, 128, DIRS8, ""), (12, 16, 16, 192, DIRS8, "chain"), (13, 16, 16, 192, DIRS8, ""), (19, 16, 16, 191, DIRS8, "chain"),
    (20, 16, 16, 191, DIRS8, ""), (2, 4, 500, 192, DIRS4, "chain"), (3, 400, 4, 128, DIRS4, "chain")])
def test_which_backward_sweep_runs_with_one_source(oracle, B, H, W, L, dirs, kernel):
    """ISGMR, truncated model: both sides of the chain layout's bounds, which lie lower for label counts that fill the lanes of the
    sweep that runs beyond, but not on long grids."""
    import paper_1910_10892_amd as mrf
    from mrf_inputs import truncated_linear
    print("case which backward sweep, one source", B, H, W, L, len(dirs), kernel, flush=True)
    pr = random_problem(830 + L, "isgmr", B, H, W, L, dirs, 1)
    pr.pairwise = truncated_linear(L, 4.0, 1.0)
    pr.pairwise_kind, pr.trunc, pr.scale = 1, 4.0, 1.0
    full_check(oracle, pr, want_V=False)
    ran = mrf.mrf_last_sweep_kernel(True)
    assert ran == ("mrf_bwd_sweep_chain" if kernel else "mrf_bwd_sweep"), mrf.mrf_last_sweep_launch(True)


@pytest.mark.parametrize("algo,B,H,W,L,dirs,halves", [
    ("trwp", 1, 40, 6, 64, DIRS4, False), ("trwp", 100, 6, 7, 49, DIRS4, True), ("trwp", 100, 6, 7, 48, DIRS4, False), ("trwp", 171, 6, 7, 64, DIRS4, False),
    ("trwp", 100, 6, 7, 40, DIRS8, True), ("isgmr", 40, 6, 7, 64, DIRS4, True), ("isgmr", 40, 6, 7, 48, DIRS4, False), ("isgmr", 90, 6, 7, 48, DIRS4, True),
    ("isgmr", 130, 6, 7, 64, DIRS4, False), ("trwp", 100, 6, 7, 72, DIRS4, False), ("trwp", 100, 6, 7, 73, DIRS4, True),
    ("trwp", 1, 6, 33, 97, DIRS4, True), ("trwp", 1, 6, 32, 97, DIRS4, False), ("isgmr", 1, 40, 33, 128, DIRS4, True), ("isgmr", 10, 33, 6, 97, DIRS4, False)])
def test_which_dense_sweep_runs(oracle, algo, B, H, W, L, dirs, halves):
    """Both sides of each bound between the sweep with chunk minima and the two others, against the oracle."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    print("case which dense sweep", algo, B, H, W, L, len(dirs), flush=True)
    pr = random_problem(640 + L, algo, B, H, W, L, dirs, 2, symmetric=False, rho=np.linspace(0.3, 0.9, len(dirs)))
    check_forward(run_gpu(pr, backward=False), oracle_forward(oracle, pr))
    assert (mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_halves") == halves, mrf.mrf_last_sweep_launch(False)


@pytest.mark.parametrize("algo,B,H,W,L,dirs,launch", [
    ("trwp", 1, 41, 6, 40, DIRS4, "halves<2,4,4"), ("trwp", 1, 39, 41, 40, DIRS4, ""), ("trwp", 49, 5, 41, 33, DIRS4, ""), ("trwp", 50, 5, 41, 33, DIRS4, ""),
    ("trwp", 9, 24, 57, 40, DIRS4, "halves<2,4,4"), ("trwp", 9, 23, 57, 48, DIRS4, ""), ("trwp", 9, 16, 57, 49, DIRS4, "halves<2,4,4"), ("trwp", 9, 15, 57, 49, DIRS4, ""),
    ("trwp", 25, 8, 41, 36, DIRS4, "halves<2,4,4"), ("trwp", 25, 7, 41, 36, DIRS4, ""), ("trwp", 33, 8, 47, 36, DIRS4, ""),
    ("trwp", 32, 24, 64, 33, DIRS4, ""), ("trwp", 32, 24, 65, 33, DIRS4, "halves<2,4,4"), ("trwp", 64, 24, 49, 33, DIRS4, ""),
    ("trwp", 2, 47, 60, 40, DIRS8, "halves<2,8,2"), ("trwp", 2, 30, 60, 40, DIRS8, ""), ("trwp", 20, 47, 60, 33, DIRS8, "halves<2,8,2"),
    ("isgmr", 60, 5, 41, 64, DIRS4, ""), ("isgmr", 12, 5, 41, 64, DIRS4, "halves<2,4,4"), ("isgmr", 1, 48, 41, 36, DIRS8, "halves<2,4,4"),
    ("isgmr", 3, 41, 6, 100, DIRS8, "halves<4,4,4"), ("isgmr", 6, 41, 6, 100, DIRS8, ""), ("isgmr", 12, 48, 41, 97, DIRS4, "halves<4,4,4"),
    ("isgmr", 7, 48, 41, 97, DIRS8, ""), ("trwp", 1, 16, 41, 128, DIRS4, "halves<4,4,4"), ("trwp", 1, 15, 41, 128, DIRS4, ""),
    ("trwp", 1, 4, 41, 70, DIRS4, ""), ("trwp", 100, 4, 41, 70, DIRS4, "halves<3,4,2"), ("isgmr", 50, 5, 41, 72, DIRS8, ""),
    ("trwp", 12, 5, 42, 70, DIRS4, "halves<3,4,4"), ("trwp", 13, 5, 42, 70, DIRS4, "halves<3,4,2"), ("trwp", 13, 7, 42, 96, DIRS8, "halves<3,8,1"),
    ("isgmr", 2, 41, 70, 80, DIRS8, "halves<3,4,2")])
def test_which_dense_sweep_runs_on_long_scanlines(oracle, algo, B, H, W, L, dirs, launch):
    """The same on grids with a side of more than 40, where the lengths of a launch's scanlines decide, and its two depths of prefetch;
    the last launch of a TRWP pass sweeps the columns or a diagonal."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    print("case long scanlines", algo, B, H, W, L, len(dirs), flush=True)
    pr = random_problem(660 + L, algo, B, H, W, L, dirs, 2, symmetric=False, rho=np.linspace(0.3, 0.9, len(dirs)))
    check_forward(run_gpu(pr, backward=False), oracle_forward(oracle, pr))
    ran = mrf.mrf_last_sweep_launch(False)
    assert launch in ran if launch else "halves" not in ran, ran


PRESUM_CASES = [
    # seed, B, H, W, L, dirs, K, integer_valued, truncated
    (701, 1, 6, 7, 40, DIRS8, 3, False, False), (702, 2, 5, 6, 21, DIRS8, 3, True, False),
    (703, 1, 5, 5, 33, DIRS16, 3, False, False), (704, 1, 7, 9, 96, DIRS8, 3, False, True),
    (705, 1, 6, 8, 192, DIRS16, 2, True, True), (706, 1, 9, 5, 70, DIRS4, 4, False, True),
    (707, 1, 5, 7, 13, ((0, 1), (1, 0), (1, 1)), 3, False, False),      # no direction has its opposite in the set
    (708, 1, 3, 5, 7, ((0, 1), (0, -1), (1, 0)), 3, True, False),       # one pair and a single direction; N L odd
    (709, 1, 12, 11, 130, DIRS8, 2, False, False),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", PRESUM_CASES, ids=lambda c: "seed%d" % c[0])
def test_isgmr_sums_of_the_previous_iteration_formed_once(oracle, case):
    """ISGMR forward where a streaming pass per iteration sums the unary and the previous iteration's
    messages once per pair of opposite directions and the sweeps read that one array (Eq. isgmr):
    against the oracle, and bit for bit against the sweeps that read every array themselves."""
    import paper_1910_10892_amd as mrf
    print("case presum", case[:5], len(case[5]), case[6:], flush=True)
    seed, B, H, W, L, dirs, K, iv, trunc = case
    if trunc:
        pr = truncated_problem(seed, "isgmr", H, W, L, dirs, K, 1, 3.0, iv, "pos")
    else:
        pr = random_problem(seed, "isgmr", B, H, W, L, dirs, K, integer_valued=iv, symmetric=False)
    try:
        assert mrf.mrf_tune(17, 2) == 0
        a = full_check(oracle, pr, want_V=False)
        assert mrf.mrf_tune(17, 1) == 0
        b = full_check(oracle, pr, want_V=False)
    finally:
        mrf.mrf_tune(17, 0)
    for name in ("p", "q", "labels", "cost", "messages"):
        np.testing.assert_array_equal(getattr(a, name), getattr(b, name), err_msg=name)


@pytest.mark.gpu
def test_knobs_and_reports_are_kept_per_thread(oracle):
    """The kernel-choice knobs and the launch reports are the library's only state and belong to the calling
    thread: another thread neither sees this thread's knob nor disturbs its report."""
    import threading
    import paper_1910_10892_amd as mrf
    from gpu_harness import GpuProblem
    pr = make_config(1, algo="isgmr")
    g = GpuProblem(pr)
    seen = {}
    try:
        assert mrf.mrf_tune(3, 1) == 0                    # this thread: never the packed sweep
        g.forward()
        torch_sync = __import__("torch").cuda.synchronize
        torch_sync()
        mine = mrf.mrf_last_sweep_kernel(False)
        assert mine != "mrf_fwd_sweep_packed"

        def other():
            seen["before"] = mrf.mrf_last_sweep_kernel(False)
            g2 = GpuProblem(pr)
            g2.forward()
            torch_sync()
            seen["after"] = mrf.mrf_last_sweep_kernel(False)
        t = threading.Thread(target=other)
        t.start()
        t.join()
        assert seen["before"] == ""                       # nothing launched from that thread yet
        assert seen["after"] == "mrf_fwd_sweep_packed"    # its own default rules, not this thread's knob
        assert mrf.mrf_last_sweep_kernel(False) == mine
    finally:
        mrf.mrf_tune(3, 0)


CHAIN_PK_CASES = [
    # seed, B, H, W, L, dirs, K, integer_valued, per_edge, want_V
    (771, 1, 6, 9, 21, DIRS4, 3, False, True, True), (772, 3, 5, 7, 32, DIRS8, 2, True, True, False),
    (773, 1, 7, 5, 5, ((0, 1), (1, 0), (1, 1)), 2, False, False, True), (774, 1, 1, 13, 17, DIRS4, 2, False, True, True),
    (775, 2, 9, 4, 1, DIRS4, 2, False, True, True), (776, 1, 23, 31, 16, DIRS8, 2, True, True, True),
    (777, 1, 40, 37, 21, DIRS4, 2, False, True, True),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CHAIN_PK_CASES, ids=lambda c: "seed%d" % c[0])
def test_chain_backward_with_two_scanlines_per_workgroup(oracle, case):
    """TRWP with up to 32 labels: the chain layout with two scanlines per workgroup (odd scanline counts,
    diagonal scanlines of unequal length, one-node scanlines, with and without grad_pairwise) against the oracle
    and against the layout the rules would pick."""
    import paper_1910_10892_amd as mrf
    print("case chain pk", case[:5], len(case[5]), case[6:], flush=True)
    seed, B, H, W, L, dirs, K, iv, per_edge, want_V = case
    pr = random_problem(seed, "trwp", B, H, W, L, dirs, K, integer_valued=iv, per_edge=per_edge, symmetric=False,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    pr.grad_cost = (pr.grad_cost * 0.2).astype(np.float32)
    try:
        for ni in (2, 4, 8):
            assert mrf.mrf_tune(20, 2) == 0 and mrf.mrf_tune(7, ni) == 0
            a = full_check(oracle, pr, want_V=want_V)
            assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_chain_pk", mrf.mrf_last_sweep_launch(True)
        assert mrf.mrf_tune(20, 1) == 0 and mrf.mrf_tune(7, 0) == 0
        b = full_check(oracle, pr, want_V=want_V)
        assert mrf.mrf_last_sweep_kernel(True) != "mrf_bwd_sweep_chain_pk"
    finally:
        mrf.mrf_tune(20, 0)
        mrf.mrf_tune(7, 0)
    for name in ("grad_unary", "grad_edge_weight") + (("grad_pairwise",) if want_V else ()):
        check_grad(name + " (two layouts)", getattr(a, name), None, getattr(b, name).astype(np.float64))


FWD_NARROW_CASES = [
    # seed, algo, B, H, W, L, dirs, K, integer_valued, per_edge: label counts around 16, 21 and 32, one and many sources
    (811, "isgmr", 2, 9, 11, 21, DIRS8, 3, True, True), (812, "trwp", 1, 7, 13, 32, DIRS4, 2, True, True),
    (813, "isgmr", 1, 6, 10, 25, DIRS16, 2, False, False), (814, "trwp", 3, 5, 6, 17, DIRS8, 2, False, True),
    (815, "isgmr", 1, 1, 37, 16, DIRS4, 2, True, True), (816, "trwp", 1, 23, 3, 9, ((0, 1), (1, 0), (1, 1)), 3, False, True),
    (817, "trwp", 1, 3, 9, 1, DIRS4, 2, False, True), (818, "trwp", 1, 4, 5, 28, DIRS16, 2, True, True),
    (819, "isgmr", 1, 33, 2, 5, DIRS8, 2, False, True),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", FWD_NARROW_CASES, ids=lambda c: "seed%d" % c[0])
def test_forward_with_one_direction_per_wavefront(oracle, case):
    """Up to 32 labels, one wavefront for several scanlines of a direction, argmin in two levels: ties, negative
    weights, scanline counts that do not fill a wavefront; against the oracle and bit for bit against the sweep
    with one level and 64-bit offsets."""
    import paper_1910_10892_amd as mrf
    print("case narrow forward", case[:6], len(case[6]), case[7:], flush=True)
    seed, algo, B, H, W, L, dirs, K, iv, pe = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=pe, symmetric=False,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    pr.grad_cost = (pr.grad_cost * (0.02 if len(dirs) > 8 else 0.2)).astype(np.float32)
    if pe and seed % 2 == 0:
        sign = np.where(np.random.default_rng(seed).random(pr.edge_weight.shape) > 0.2, 1.0, -0.5)
        pr.edge_weight = (pr.edge_weight * sign).astype(np.float32)
    try:
        assert mrf.mrf_tune(3, 2) == 0
        for three in ((1, 2) if 16 < L <= 21 else (1,)):
            assert mrf.mrf_tune(13, three) == 0 and mrf.mrf_tune(11, 1) == 0
            a = full_check(oracle, pr, want_V=False)
            assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_narrow", mrf.mrf_last_sweep_launch(False)
            assert mrf.mrf_tune(11, 3) == 0
            b = full_check(oracle, pr, want_V=False)
            assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_packed"
            for name in ("p", "q", "labels", "cost", "messages"):
                np.testing.assert_array_equal(getattr(a, name), getattr(b, name), err_msg=name)
    finally:
        for knob in (3, 11, 13):
            mrf.mrf_tune(knob, 0)


NARROW_CASES = [
    # seed, algo, B, H, W, L, dirs, K, integer_valued, per_edge: label counts at the edges of 8-lane segments
    (781, "isgmr", 2, 9, 11, 21, DIRS8, 3, False, True), (782, "trwp", 1, 7, 13, 32, DIRS4, 2, True, True),
    (783, "isgmr", 1, 6, 10, 25, DIRS16, 2, False, False), (784, "trwp", 3, 5, 6, 24, DIRS8, 2, False, True),
    (785, "isgmr", 1, 1, 37, 8, DIRS4, 2, True, True), (786, "trwp", 1, 23, 3, 9, ((0, 1), (1, 0), (1, 1)), 3, False, True),
    (787, "trwp", 1, 3, 9, 1, DIRS4, 2, False, True), (788, "isgmr", 1, 33, 2, 17, DIRS8, 2, False, True),
    (789, "trwp", 1, 4, 5, 16, DIRS16, 2, False, True),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", NARROW_CASES, ids=lambda c: "seed%d" % c[0])
def test_backward_with_several_labels_per_lane(oracle, case):
    """Up to 32 labels, segments of 8, 16 and 32 lanes per scanline: scanline counts that do not fill a
    wavefront, scanlines of unequal length and of one node, with and without grad_pairwise, against the oracle
    and against the one-wavefront sweep."""
    import paper_1910_10892_amd as mrf
    print("case narrow backward", case[:6], len(case[6]), case[7:], flush=True)
    seed, algo, B, H, W, L, dirs, K, iv, pe = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=pe, symmetric=False,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    pr.grad_cost = (pr.grad_cost * (0.02 if len(dirs) > 8 else 0.2)).astype(np.float32)
    got = {}
    try:
        assert mrf.mrf_tune(6, 1) == 0 and mrf.mrf_tune(20, 1) == 0
        for seg in (8, 16, 32):
            for want_V in (True, False):
                assert mrf.mrf_tune(3, seg) == 0
                got[seg, want_V] = full_check(oracle, pr, want_V=want_V)
                assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_narrow", mrf.mrf_last_sweep_launch(True)
        # one label per lane, 64-bit offsets (what takes over where arrays outgrow the views of the narrow sweep)
        assert mrf.mrf_tune(3, 3) == 0
        for want_V in (True, False):
            got[0, want_V] = full_check(oracle, pr, want_V=want_V)
            assert mrf.mrf_last_sweep_launch(True).startswith("mrf_bwd_sweep_packed<%d," % (16 if L <= 16 else 32))
        assert mrf.mrf_tune(3, 1) == 0
        plain = full_check(oracle, pr, want_V=True)
        assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep"
    finally:
        for knob in (3, 6, 20):
            mrf.mrf_tune(knob, 0)
    for (seg, want_V), g in got.items():
        for name in ("grad_unary", "grad_edge_weight") + (("grad_pairwise",) if want_V else ()):
            check_grad("%s (%d lanes)" % (name, seg), getattr(g, name), None, getattr(plain, name).astype(np.float64))


NARROW_WAVES_CASES = [
    # seed, images, L, lanes, block: two and four wavefronts per workgroup, the last one with idle wavefronts
    (801, 75, 5, 8, 64), (802, 301, 5, 8, 128), (803, 153, 13, 16, 128), (804, 303, 16, 16, 256), (805, 601, 23, 8, 256),
    (806, 77, 25, 32, 128), (807, 151, 32, 32, 256), (808, 153, 32, 16, 128), (809, 601, 32, 8, 256),
]


@pytest.mark.parametrize("case", NARROW_WAVES_CASES, ids=lambda c: "seed%d" % c[0])
def test_narrow_backward_with_several_wavefronts_per_workgroup(oracle, case):
    """Batches of small images that take several wavefronts per workgroup: a V, its gradient's slot and the LDS behind
    them shared, with and without grad_pairwise."""
    import paper_1910_10892_amd as mrf
    print("case narrow wavefronts", case, flush=True)
    seed, B, L, lanes, block = case
    pr = random_problem(seed, "isgmr", B, 3, 5, L, DIRS4, 2, symmetric=False)
    try:
        assert mrf.mrf_tune(3, lanes) == 0
        for want_V in (True, False):
            full_check(oracle, pr, want_V=want_V)
            launch = mrf.mrf_last_sweep_launch(True)
            assert launch.startswith("mrf_bwd_sweep_narrow<%d," % lanes) and "block=%d" % block in launch, launch
    finally:
        mrf.mrf_tune(3, 0)


@pytest.mark.parametrize("L,B,want_V,kernel", [
    (17, 1000, True, "chain_pk<4,"), (23, 1280, False, "chain_pk<4,"), (17, 1281, True, "narrow<32,1,4,"), (19, 1300, False, "narrow<32,1,4,"),
    (20, 800, True, "narrow<16,2,4,"), (22, 800, False, "narrow<16,2,4,"), (21, 800, True, "narrow<8,3,4,"),
    (25, 800, False, "narrow<32,1,4,"), (26, 800, False, "narrow<16,2,4,"), (26, 800, True, "narrow<32,1,4,")])
def test_lanes_that_the_label_count_fills(oracle, L, B, want_V, kernel):
    """TRWP launches of more than 1,536 scanlines with several source arrays: the segments whose lanes the label count
    fills, two scanlines per workgroup to 2,560 scanlines where it fills none."""
    import paper_1910_10892_amd as mrf
    print("case lanes filled", L, B, want_V, flush=True)
    pr = random_problem(810 + L, "trwp", B, 2, 3, L, DIRS4, 2, symmetric=False, rho=np.linspace(0.3, 0.9, 4))
    full_check(oracle, pr, want_V=want_V)
    assert mrf.mrf_last_sweep_launch(True).startswith("mrf_bwd_sweep_" + kernel), mrf.mrf_last_sweep_launch(True)


# every segment of the narrow sweep that its lanes' labels fill, up to three and seven source arrays, scanlines of different
# lengths in a workgroup (diagonals, images that fill none), rings that wrap
@pytest.mark.parametrize("case", [(L, lanes, R) for L, lanes in ((1, 8), (5, 8), (8, 8), (9, 16), (16, 16), (18, 8), (21, 8), (24, 8), (20, 16), (32, 16), (17, 32), (23, 32), (32, 32))
                                  for R in (4, 8)], ids=lambda c: "%d_%d_%d" % c)
def test_narrow_backward_divided_among_four_wavefronts(oracle, case):
    """Against the oracle, and against the sweep with one wavefront, which adds the same terms in the same order: the same floats
    but for grad theta, whose sum starts elsewhere."""
    import paper_1910_10892_amd as mrf
    print("case narrow divided", case, flush=True)
    L, lanes, R = case
    B, H, W = (5, 3, 29) if R == 4 else (3, 7, 9)
    pr = random_problem(840 + L, "trwp", B, H, W, L, DIRS8 if R == 8 else DIRS4, 2, symmetric=False, rho=np.linspace(0.3, 0.9, R))
    pr.grad_cost = (pr.grad_cost * 0.2).astype(np.float32)
    try:
        for want_V in (True, False):
            got = []
            for divided in (4, 3):
                assert mrf.mrf_tune(3, lanes) == 0 and mrf.mrf_tune(20, divided) == 0 and mrf.mrf_tune(6, 1) == 0
                got.append(full_check(oracle, pr, want_V=want_V))
                assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_narrow"
                assert ("block=256" in mrf.mrf_last_sweep_launch(True)) == (divided == 4), mrf.mrf_last_sweep_launch(True)
            for name in ("grad_edge_weight",) + (("grad_pairwise",) if want_V else ()):
                np.testing.assert_array_equal(getattr(got[0], name), getattr(got[1], name), err_msg=name)
            np.testing.assert_allclose(got[0].grad_unary, got[1].grad_unary, rtol=1e-6, atol=1e-6)
    finally:
        for k in (3, 6, 20):
            mrf.mrf_tune(k, 0)


MANY_SMALL_IMAGES = [
    # seed, algo, images, L: more workgroups of the narrow sweep than there are V-gradient slots (16,384)
    (791, "isgmr", 6600, 25), (792, "isgmr", 13200, 12), (793, "isgmr", 26400, 5),
]


@pytest.mark.parametrize("case", MANY_SMALL_IMAGES, ids=lambda c: "seed%d" % c[0])
def test_pairwise_gradient_of_more_scanlines_than_slots(oracle, case):
    """Up to 32 labels with grad_pairwise and a batch whose scanlines take more workgroups than the workspace has
    V-gradient slots: the sweep goes into several launches."""
    import paper_1910_10892_amd as mrf
    print("case many small images", case, flush=True)
    seed, algo, B, L = case
    pr = random_problem(seed, algo, B, 2, 2, L, DIRS8, 2, symmetric=False)
    full_check(oracle, pr)
    assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_narrow", mrf.mrf_last_sweep_launch(True)


def test_two_scanlines_per_workgroup_need_a_slot_each(oracle):
    """Chain backward with two scanlines per workgroup on request, for launches with more workgroups than V-gradient
    slots: another sweep takes them."""
    import paper_1910_10892_amd as mrf
    print("case pair layout without slots", flush=True)
    pr = random_problem(794, "trwp", 16500, 2, 2, 6, DIRS4, 2, symmetric=False)
    try:
        assert mrf.mrf_tune(20, 2) == 0
        full_check(oracle, pr)
        assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_narrow", mrf.mrf_last_sweep_launch(True)
        full_check(oracle, pr, want_V=False)
        assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_chain_pk", mrf.mrf_last_sweep_launch(True)
    finally:
        mrf.mrf_tune(20, 0)


@pytest.mark.parametrize("algo,L,H,W", [("isgmr", 8, 1451, 1457), ("trwp", 21, 893, 897)])
def test_backward_of_arrays_beyond_32_bit_offsets(algo, L, H, W):
    """Up to 32 labels, more than 2^30 entries per array: a batch of 64 equal images against one of them (same sums in
    double, other order: a float rounding apart), and the sweep that has 64-bit offsets."""
    import torch
    import paper_1910_10892_amd as mrf
    print("case large batch", algo, L, H, W, flush=True)
    B, K, dirs, dev = 64, 2, ((0, 1), (1, 0)), "cuda:0"
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    rand = lambda *s: torch.rand(s, generator=gen, device=dev)  # noqa: E731
    unary, V, w, gc = rand(1, H, W, L), rand(L, L), rand(2, 1, H, W) + 0.5, rand(1, H, W, L) - 0.5
    code = mrf.MRF_ISGMR if algo == "isgmr" else mrf.MRF_TRWP
    forward = mrf.mrf_isgmr_forward if algo == "isgmr" else mrf.mrf_trwp_forward
    backward = mrf.mrf_isgmr_backward if algo == "isgmr" else mrf.mrf_trwp_backward

    def replay(n, p, q):
        batch = lambda x, axis: x.repeat_interleave(n, dim=axis)  # noqa: E731
        prob = mrf.MrfProblem(None, V, dirs, K, batch(w, 1), rho=(0.4, 0.7), shape=(n, H, W, L))
        g = [torch.empty(s, device=dev) for s in ((n, H, W, L), (2, n, H, W), (L, L))]
        ws = torch.empty(mrf.mrf_workspace_bytes(prob, code, True), dtype=torch.uint8, device=dev)
        backward(prob, batch(gc, 0), batch(p, 2), batch(q, 2), *g, ws)
        return g

    prob = mrf.MrfProblem(unary, V, dirs, K, w, rho=(0.4, 0.7))
    p = torch.empty((K, 2, 1, H, W, L), dtype=torch.uint8, device=dev)
    q = torch.empty((K, 2, 1, H, W), dtype=torch.uint8, device=dev)
    ws = torch.empty(mrf.mrf_workspace_bytes(prob, code, False), dtype=torch.uint8, device=dev)
    forward(prob, torch.empty_like(unary), None, p, q, None, ws)
    one = replay(1, p, q)
    many = replay(B, p, q)
    assert mrf.mrf_last_sweep_launch(True).startswith("mrf_bwd_sweep_packed<%d," % (16 if L <= 16 else 32))
    for b in range(B):
        torch.testing.assert_close(many[0][b], one[0][0], rtol=1e-6, atol=1e-6)
        torch.testing.assert_close(many[1][:, b], one[1][:, 0], rtol=1e-6, atol=1e-6)
    # (a sum of 64 times as many terms, rounded once: the same relative bar as everywhere)
    torch.testing.assert_close(many[2], B * one[2], rtol=RTOL, atol=B * ATOL)


FAR_ROW, FAR_COLUMN = ((0, 1), (0, -1)), ((1, 0), (-1, 0))
FAR_CASES = [
    # H, W, L, dirs, table, grad V: more than 2^30 entries in an image, or half of that with stored node gradients; a kernel each
    (2100, 8200, 64, FAR_ROW, False, False, "<1,4,2,6,false,false,false,false,true>"),
    (8400, 1000, 128, FAR_COLUMN, True, False, "<2,4,2,6,true,false,false,false,true>"),
    (1500, 2900, 255, FAR_ROW + ((0, 2), (0, -2), (0, 3)), False, False, "<4,8,1,6,false,false,true,false,true>"),
    (3000, 1500, 127, FAR_COLUMN, True, True, "<2,4,2,6,true,true,true,false,true>"),
    (1400, 12000, 64, FAR_ROW, True, True, "<1,4,2,6,true,true,true,false,true>"),
    (250, 215000, 20, FAR_ROW, True, True, "<1,4,2,6,false,true,false,false,true>"),
]


@pytest.mark.parametrize("case", FAR_CASES, ids=lambda c: "%dx%d_L%d" % c[:3])
def test_chain_backward_of_images_beyond_32_bit_offsets(case):
    """The chain sweep with a view per access against the sweeps with 64-bit addresses, on indices drawn at random: both sum in
    double and round what they store to float, so a float rounding apart; an entry of grad V sums some 10^5 terms of that error."""
    import torch
    import paper_1910_10892_amd as mrf
    H, W, L, dirs, table, want_V, launch = case
    print("case far image", H, W, L, len(dirs), table, want_V, flush=True)
    R, dev = len(dirs), "cuda:0"
    gen = torch.Generator(device=dev)
    gen.manual_seed(7 + L)
    lab = torch.arange(L, device=dev, dtype=torch.float32)
    V = torch.rand((L, L), generator=gen, device=dev) if table else (lab[:, None] - lab[None, :]).abs().clamp(max=3.0).contiguous()
    w = torch.rand((R, 1, H, W), generator=gen, device=dev) + 0.5
    gc = torch.rand((1, H, W, L), generator=gen, device=dev) - 0.5
    p = torch.randint(0, L, (1, R, 1, H, W, L), generator=gen, device=dev, dtype=torch.uint8)
    q = torch.randint(0, L, (1, R, 1, H, W), generator=gen, device=dev, dtype=torch.uint8)
    kind = {} if table else {"pairwise_kind": 1, "trunc": 3.0, "scale": 1.0}
    prob = mrf.MrfProblem(None, V, dirs, 1, w, rho=np.linspace(0.3, 0.7, R), shape=(1, H, W, L), **kind)
    ws = torch.empty(mrf.mrf_workspace_bytes(prob, mrf.MRF_TRWP, True), dtype=torch.uint8, device=dev)

    def replay():
        g = [torch.full((1, H, W, L), float("nan"), device=dev), torch.full((R, 1, H, W), float("nan"), device=dev),
             torch.full((L, L), float("nan"), device=dev) if want_V else None]
        ws.fill_(0xFF)
        mrf.mrf_trwp_backward(prob, gc, p, q, *g, ws)
        return g, mrf.mrf_last_sweep_launch(True)

    far, ran = replay()
    assert ran.startswith("mrf_bwd_sweep_chain" + launch), ran
    try:
        assert mrf.mrf_tune(6, 1) == 0
        other, ran = replay()
        assert "chain" not in ran, ran
    finally:
        mrf.mrf_tune(6, 0)
    torch.testing.assert_close(far[0], other[0], rtol=RTOL, atol=1e-6)
    torch.testing.assert_close(far[1], other[1], rtol=RTOL, atol=1e-5)
    if want_V:
        torch.testing.assert_close(far[2], other[2], rtol=RTOL, atol=1e-3)


GV_APART_CASES = [
    # seed, B, H, W, L, dirs, K, integer_valued, per_edge
    (751, 1, 6, 9, 96, DIRS4, 3, False, True), (752, 2, 5, 7, 128, DIRS8, 2, True, True),
    (753, 1, 7, 5, 65, ((0, 1), (1, 0), (1, 1)), 2, False, False), (754, 1, 4, 33, 100, DIRS4, 2, False, True),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", GV_APART_CASES, ids=lambda c: "seed%d" % c[0])
def test_pairwise_gradient_added_up_behind_the_chain_sweep(oracle, case):
    """TRWP with 65..128 labels and grad_pairwise: the chain sweep stores the node gradients and a streaming
    pass forms both pairwise gradients (Eq. supp-gradient-smoothness, Eq. supp-gradient-edge); against the oracle, and against the sweep that
    accumulates the table itself."""
    import paper_1910_10892_amd as mrf
    print("case grad V apart", case[:5], len(case[5]), case[6:], flush=True)
    seed, B, H, W, L, dirs, K, iv, per_edge = case
    pr = random_problem(seed, "trwp", B, H, W, L, dirs, K, integer_valued=iv, per_edge=per_edge, symmetric=False,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    pr.grad_cost = (pr.grad_cost * 0.2).astype(np.float32)
    try:
        a = full_check(oracle, pr, want_V=True)
        assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_chain", mrf.mrf_last_sweep_launch(True)
        assert mrf.mrf_tune(19, 1) == 0
        b = full_check(oracle, pr, want_V=True)
        assert mrf.mrf_last_sweep_kernel(True) != "mrf_bwd_sweep_chain"
    finally:
        mrf.mrf_tune(19, 0)
    check_grad("grad_pairwise (two layouts)", a.grad_pairwise, None, b.grad_pairwise.astype(np.float64))


GV_APART_FEW_CASES = [
    # seed, B, H, W, L, dirs, K, kind: 33..64 labels; eight or four tables; sixteen sources; a scatter target with words of its own
    (761, 50, 6, 9, 33, DIRS4, 2, 0), (762, 1, 7, 9, 49, DIRS8, 2, 0), (763, 1, 5, 8, 64, DIRS16, 2, 0), (764, 3, 11, 7, 55, DIRS4, 3, 0),
    (765, 130, 9, 6, 40, DIRS4, 2, 1), (766, 130, 9, 5, 64, DIRS4, 1, 1), (767, 130, 9, 6, 70, DIRS4, 1, 1), (768, 60, 5, 6, 48, DIRS16, 1, 0),
    (769, 1, 5, 7, 96, DIRS16, 2, 0),
]


@pytest.mark.parametrize("case", GV_APART_FEW_CASES, ids=lambda c: "seed%d" % c[0])
def test_pairwise_gradients_from_stored_node_gradients(oracle, case):
    """The same for 33..64 labels, for sixteen directions and for launches that keep the lanes of the most popular scatter
    target apart (truncated models, more than 1,024 scanlines)."""
    import paper_1910_10892_amd as mrf
    print("case node gradients", case[:5], len(case[5]), case[6:], flush=True)
    seed, B, H, W, L, dirs, K, kind = case
    if kind:
        from mrf_inputs import truncated_linear
    pr = random_problem(seed, "trwp", B, H, W, L, dirs, K, symmetric=False, rho=np.linspace(0.3, 0.9, len(dirs)))
    if kind:
        pr.pairwise = truncated_linear(L, 20.0, 0.37)
        pr.pairwise_kind, pr.trunc, pr.scale = 1, 20.0, 0.37
    pr.grad_cost = (pr.grad_cost * (0.02 if len(dirs) > 8 else 0.2)).astype(np.float32)
    a = full_check(oracle, pr)
    launch = mrf.mrf_last_sweep_launch(True)
    assert launch.startswith("mrf_bwd_sweep_chain<%d," % ((L + 63) // 64)) and "true,true,%s" % ("true" if kind else "false") in launch, launch
    try:
        assert mrf.mrf_tune(19, 1) == 0
        b = full_check(oracle, pr)
        assert "true,true," not in mrf.mrf_last_sweep_launch(True)
    finally:
        mrf.mrf_tune(19, 0)
    check_grad("grad_pairwise (two layouts)", a.grad_pairwise, None, b.grad_pairwise.astype(np.float64))


CHAIN_EDGE_CASES = [
    # seed, algo, B, H, W, L, dirs, K, truncated: label counts around 64 per lane slot; scanlines shorter than, as long as and longer
    # than the helpers' ring; one node; images, directions and source slots
    (771, "trwp", 1, 1, 1, 5, DIRS4, 1, False), (772, "trwp", 2, 3, 25, 63, DIRS4, 2, True), (773, "isgmr", 1, 5, 13, 64, DIRS8, 2, True),
    (774, "trwp", 3, 12, 2, 65, DIRS8, 2, True), (775, "isgmr", 1, 24, 7, 128, DIRS4, 2, False), (776, "trwp", 1, 4, 26, 129, DIRS4, 3, True),
    (777, "isgmr", 2, 2, 49, 192, DIRS4, 2, True), (778, "trwp", 1, 7, 11, 193, ((0, 1), (0, -1)), 2, True),
    (779, "trwp", 1, 9, 5, 256, DIRS8, 2, True), (780, "trwp", 1, 5, 30, 37, DIRS16, 1, True),
]


@pytest.mark.parametrize("case", CHAIN_EDGE_CASES, ids=lambda c: "seed%d" % c[0])
def test_chain_backward_with_every_number_of_helpers(oracle, case):
    """The chain sweep with 2 to 12 helpers, with and without the words for the most popular scatter target, against the oracle;
    the number of helpers changes who does a node, not what is done: the same bits."""
    import paper_1910_10892_amd as mrf
    from mrf_inputs import truncated_linear
    print("case chain helpers", case[:6], len(case[6]), case[7:], flush=True)
    seed, algo, B, H, W, L, dirs, K, truncated = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, symmetric=False, rho=np.linspace(0.3, 0.9, len(dirs)))
    if truncated:
        pr.pairwise = truncated_linear(L, 3.0, 0.37)
        pr.pairwise_kind, pr.trunc, pr.scale = 1, 3.0, 0.37
    pr.grad_cost = (pr.grad_cost * (0.02 if len(dirs) > 8 else 0.2)).astype(np.float32)
    try:
        assert mrf.mrf_tune(6, 2) == 0
        for hot in ((1, 2) if truncated else (0,)):
            assert mrf.mrf_tune(12, hot) == 0
            first = None
            for ni in (2, 4, 6, 8, 12):
                assert mrf.mrf_tune(7, ni) == 0
                g = full_check(oracle, pr, want_V=False)
                launch = mrf.mrf_last_sweep_launch(True)
                assert launch.startswith("mrf_bwd_sweep_chain<"), launch
                parts = launch[launch.index("<") + 1:launch.index(">")].split(",")       # LP, NS, D, NI, VG, GV, HOT
                assert parts[3] == str(ni) and parts[6] == ("true" if hot == 2 else "false"), launch
                got = (g.grad_unary, g.grad_edge_weight)
                if first is None:
                    first = got
                assert all(np.array_equal(a, b) for a, b in zip(first, got)), ni
    finally:
        for knob in (6, 7, 12):
            mrf.mrf_tune(knob, 0)


DIAGONAL_ORDER_CASES = [
    # seed, algo, B, H, W, L, truncation (0: dense), forward sweep, backward sweep: diagonals of fewer than 256 scanlines, of one more, of a whole
    # number of runs of 256 and of a remainder; grids higher than wide, wider than high, square, of one row and of one column.  Every sweep
    # that takes its scanlines from mrf_geom_order is among them; mrf_bwd_sweep and mrf_bwd_sweep_split take theirs as they come.
    (781, "trwp", 17, 8, 8, 40, 0, "sweep", "sweep_chain"), (782, "trwp", 257, 1, 3, 70, 0, "sweep_halves", "sweep_chain"),
    (783, "trwp", 32, 9, 8, 100, 6, "sweep_window_squad", "sweep_chain"), (784, "trwp", 40, 6, 9, 70, 6, "sweep_window_duo", "sweep_chain"),
    (785, "isgmr", 33, 7, 10, 40, 0, "sweep", "sweep"), (786, "trwp", 21, 10, 4, 200, 12, "sweep_window_squad", "sweep_split"),
    (787, "trwp", 100, 5, 1, 40, 6, "sweep_window_duo", "sweep_chain"), (788, "isgmr", 30, 6, 5, 200, 12, "sweep_window_split", "sweep"),
    (789, "isgmr", 1, 40, 21, 140, 0, "sweep_sliced", "sweep_split"),
]


@pytest.mark.parametrize("case", DIAGONAL_ORDER_CASES, ids=lambda c: "seed%d" % c[0])
def test_order_of_a_diagonals_scanlines(oracle, case):
    """Every scanline of a diagonal is swept once, whatever run of 256 it falls into (mrf_geom_order)."""
    import paper_1910_10892_amd as mrf
    from mrf_inputs import truncated_linear
    print("case diagonal order", case, flush=True)
    seed, algo, B, H, W, L, trunc, forward, backward = case
    pr = random_problem(seed, algo, B, H, W, L, DIRS8, 2, symmetric=False, rho=np.linspace(0.3, 0.9, 8))
    if trunc:
        pr.pairwise = truncated_linear(L, float(trunc), 0.37)
        pr.pairwise_kind, pr.trunc, pr.scale = 1, float(trunc), 0.37
    pr.grad_cost = (pr.grad_cost * 0.02).astype(np.float32)
    full_check(oracle, pr)
    assert (mrf.mrf_last_sweep_kernel(False), mrf.mrf_last_sweep_kernel(True)) == ("mrf_fwd_" + forward, "mrf_bwd_" + backward)


def test_forbidden_transitions_leave_first_nodes_alone(oracle):
    """Infinite entries of V that no update selects: the edge-weight gradient of nodes without a predecessor stays 0
    (their p is 0, which may point at such an entry)."""
    import paper_1910_10892_amd as mrf
    print("case infinite entries of V", flush=True)
    pr = random_problem(755, "trwp", 1, 6, 9, 70, DIRS4, 2, symmetric=False)
    pr.pairwise[0, 3] = pr.pairwise[0, 66] = np.inf
    g = full_check(oracle, pr)
    assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_chain", mrf.mrf_last_sweep_launch(True)
    assert (g.p[..., 3] != 0)[:, 0, :, :, 1:].all()            # (no update selects a forbidden transition)
    assert (g.grad_edge_weight[0, :, :, 0] == 0).all()


@pytest.mark.parametrize("L", [5, 13, 21, 23, 25, 32])
@pytest.mark.parametrize("algo", ["isgmr", "trwp"])
def test_neighbours_that_must_differ(oracle, algo, L):
    """V with an infinite diagonal (no update selects it): nothing of it reaches a gradient, also where a wavefront
    has lanes without a label."""
    import paper_1910_10892_amd as mrf
    print("case infinite diagonal", algo, L, flush=True)
    pr = random_problem(756 + L, algo, 2, 6, 9, L, DIRS8, 2, symmetric=False)
    np.fill_diagonal(pr.pairwise, np.inf)
    try:
        assert mrf.mrf_tune(3, 2) == 0 and mrf.mrf_tune(6, 1) == 0 and mrf.mrf_tune(20, 1) == 0
        for want_V in (True, False):
            full_check(oracle, pr, want_V=want_V)
            assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_narrow", mrf.mrf_last_sweep_launch(True)
    finally:
        for knob in (3, 6, 20):
            mrf.mrf_tune(knob, 0)


def truncated_problem(seed, algo, H, W, L, dirs, K, kind, trunc, integer_valued, weights):
    """Truncated linear (kind 1) / quadratic (kind 2) pairwise with the kind announced, so the
    library may take its window path.  weights: 'pos' | 'zero_mix' | 'neg_mix'."""
    from mrf_inputs import truncated_linear, truncated_quadratic
    pr = random_problem(seed, algo, 1, H, W, L, dirs, K, integer_valued=integer_valued,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    scale = 1.0 if integer_valued else 0.37
    pr.pairwise = truncated_linear(L, trunc, scale) if kind == 1 else truncated_quadratic(L, trunc, scale)
    pr.pairwise_kind, pr.trunc, pr.scale = kind, float(trunc), float(scale)
    rng = np.random.default_rng(seed + 1000)
    if weights == "zero_mix":
        pr.edge_weight = pr.edge_weight * (rng.random(pr.edge_weight.shape) > 0.3)
    elif weights == "neg_mix":
        pr.edge_weight = pr.edge_weight * np.where(rng.random(pr.edge_weight.shape) > 0.2, 1.0, -0.5)
    pr.edge_weight = pr.edge_weight.astype(np.float32)
    return pr


@pytest.mark.parametrize("kind", ["masks", "infinite", "nan"])
@pytest.mark.parametrize("case", [("isgmr", 96, 200.0, 2, DIRS4), ("trwp", 192, 200.0, 2, DIRS4), ("trwp", 255, 16.0, 1, DIRS4),
                                  ("isgmr", 130, 7.0, 1, DIRS4), ("isgmr", 97, 8.0, 1, DIRS4)], ids=lambda c: "%s_%d" % c[:2])
def test_window_with_loader_and_index_wavefronts_where_labels_are_not_finite(oracle, case, kind):
    """mrf_fwd_sweep_window_squad by the default rules: the indices, costs and messages of the oracle where labels are impossible
    or pixels have none."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    print("case window not finite", case[:4], kind, flush=True)
    algo, L, trunc, pk, dirs = case
    pr = not_finite(truncated_problem(660 + L, algo, 7, 9, L, dirs, 2, pk, trunc, False, "pos"), kind, L)
    with np.errstate(all="ignore"):
        f = oracle_forward(oracle, pr)
    g = run_gpu(pr, backward=False)
    assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_window_squad", mrf.mrf_last_sweep_launch(False)
    for name in ("p", "q", "cost", "messages"):
        np.testing.assert_array_equal(getattr(g, name), getattr(f, name), err_msg=name)
    some = ~np.isnan(f.cost).any(-1)
    np.testing.assert_array_equal(g.labels[some], f.labels[some])


WINDOW_CASES = [
    # seed, algo, H, W, L, dirs, K, kind, trunc, integer_valued, weights
    (41, "trwp", 6, 9, 96, DIRS4, 3, 1, 8.0, False, "pos"),
    (42, "isgmr", 6, 9, 96, DIRS8, 2, 1, 8.0, True, "pos"),        # integer data: ties between window and far field
    (43, "trwp", 5, 7, 40, DIRS4, 3, 1, 2.0, True, "zero_mix"),    # zero weights: every candidate ties
    (44, "isgmr", 5, 7, 70, DIRS4, 2, 2, 200.0, False, "pos"),     # quadratic, window 15
    (45, "trwp", 5, 7, 130, DIRS8, 2, 2, 30.0, True, "neg_mix"),   # negative weights take the full loop
    (46, "isgmr", 4, 6, 200, DIRS4, 2, 1, 1.0, True, "pos"),       # Potts
    (47, "trwp", 4, 6, 17, DIRS4, 2, 1, 16.0, False, "pos"),       # window almost as wide as the label range
    (48, "trwp", 4, 6, 12, DIRS4, 2, 1, 20.0, False, "pos"),       # no truncation inside the range: dense kernel
    (49, "isgmr", 5, 5, 256, DIRS4, 2, 2, 200.0, True, "zero_mix"),
    # scanlines several times longer than the ring between the value and index wavefronts
    (50, "trwp", 3, 41, 96, DIRS4, 2, 1, 8.0, False, "pos"),
    (54, "trwp", 5, 9, 70, DIRS4, 3, 1, 4.0, False, "pos"),          # window 4
    (57, "trwp", 4, 7, 96, DIRS4, 2, 1, 11.0, False, "pos"),         # window 12
    (58, "isgmr", 5, 6, 256, DIRS8, 2, 2, 100.0, True, "zero_mix"),  # quadratic, window 10 -> 12; the 64-label layouts take 16
    (55, "isgmr", 6, 7, 130, DIRS8, 2, 1, 3.0, True, "zero_mix"),
    (56, "trwp", 4, 6, 200, DIRS4, 2, 2, 10.0, True, "pos"),         # quadratic, sqrt(10) -> window 4
    (51, "trwp", 6, 8, 40, DIRS16, 2, 1, 3.0, False, "pos"),       # sixteen directions: fifteen message arrays per update
    (52, "trwp", 5, 9, 200, DIRS16, 2, 2, 60.0, True, "zero_mix"),
    (53, "isgmr", 6, 7, 130, DIRS16, 3, 1, 8.0, True, "pos"),
    (51, "isgmr", 2, 37, 40, DIRS8, 2, 1, 2.0, True, "zero_mix"),
    (52, "trwp", 2, 33, 70, DIRS4, 2, 2, 30.0, True, "neg_mix"),
    (53, "trwp", 1, 12, 40, DIRS8, 2, 1, 2.0, False, "pos"),       # one row: vertical and diagonal scanlines of one node
    (54, "trwp", 5, 6, 96, [(0, 1), (1, 0), (-1, 0)], 3, 1, 8.0, False, "pos"),   # a direction without its opposite
    (55, "isgmr", 6, 1, 33, DIRS4, 2, 1, 4.0, True, "zero_mix"),   # one column
    # 65 .. 128 labels, TRWP: the loader-fed value wavefront holds two adjacent labels per lane
    (56, "trwp", 4, 19, 65, DIRS4, 2, 1, 8.0, False, "pos"),       # one label in the second half of a pair
    (57, "trwp", 5, 13, 75, DIRS4, 3, 1, 2.0, True, "zero_mix"),   # odd label count, narrowest window
    (58, "trwp", 3, 21, 127, DIRS4, 2, 2, 200.0, False, "pos"),    # widest window, last lane half used
    (59, "trwp", 4, 11, 128, DIRS4, 2, 1, 8.0, True, "neg_mix"),   # every lane full; negative weights
    (60, "trwp", 6, 10, 100, [(0, 1), (0, -1), (1, 0)], 3, 2, 30.0, False, "pos"),
    (61, "trwp", 2, 40, 97, DIRS4, 2, 1, 16.0, True, "pos"),
]


@pytest.mark.parametrize("case", WINDOW_CASES, ids=lambda c: "seed%d" % c[0])
def test_window_path_is_exact(oracle, case):
    """Truncated models run through the window kernel; its results must equal the oracle's
    and, bit for bit, those of the dense kernel on the same problem."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    print("case window", case[:5], case[7:], flush=True)
    pr = truncated_problem(*case)
    if len(pr.dirs) > 8:
        # (the backward pass amplifies grad c with every direction and iteration: keep the gradients in the
        # range where the absolute part of the tolerance means something in fp32)
        pr.grad_cost = (pr.grad_cost * 0.05).astype(np.float32)
    got = {}
    try:
        assert mrf.mrf_tune(2, 1) == 0 and mrf.mrf_tune(4, 1) == 0      # one wavefront per scanline
        got["single"] = full_check(oracle, pr)
        if case[0] in (51, 52, 53):     # sixteen directions take the window sweep too
            assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_window", mrf.mrf_last_sweep_launch(False)
        assert mrf.mrf_tune(4, 2) == 0 and mrf.mrf_tune(5, 1) == 0      # value + one index wavefront
        got["pair"] = full_check(oracle, pr)
        assert mrf.mrf_tune(5, 2) == 0 and mrf.mrf_tune(8, 1) == 0      # value + two index wavefronts
        got["trio"] = full_check(oracle, pr)
        assert mrf.mrf_tune(8, 2) == 0                                  # and a loader wavefront (TRWP)
        got["quad"] = full_check(oracle, pr)
        assert mrf.mrf_tune(2, 2) == 0 and mrf.mrf_tune(9, 1) == 0      # one wavefront per 64 labels
        got["split"] = full_check(oracle, pr)
        assert mrf.mrf_tune(9, 2) == 0 and mrf.mrf_tune(10, 4) == 0     # ... for the values, 4 index wavefronts
        got["squad4"] = full_check(oracle, pr)
        assert mrf.mrf_tune(10, 8) == 0
        got["squad8"] = full_check(oracle, pr)
        assert mrf.mrf_tune(1, 1) == 0                                  # dense sweep
        d = run_gpu(pr)
    finally:
        for knob in (1, 2, 4, 5, 8, 9, 10):
            mrf.mrf_tune(knob, 0)
    for layout, g in got.items():
        for name in ("p", "q", "labels", "cost", "messages"):
            np.testing.assert_array_equal(getattr(g, name), getattr(d, name), err_msg="%s %s" % (layout, name))


# label counts around the wavefronts and pairs of labels, odd ones; the widths that share the window among lanes and the one
# that does not; rings that wrap; 3 and 7 source arrays; negative weights, V(0) != 0, integer data
@pytest.mark.parametrize("case", [(L, width, algo, R) for L in (65, 67, 96, 127, 128, 129, 131, 192, 193, 255, 256)
                                  for width, algo, R in ((8, "trwp", 4), (16, "isgmr", 4), (16, "trwp", 8), (2, "trwp", 4))
                                  if R == 4 and width > 2 or L in (67, 129, 256)], ids=lambda c: "%d_%d_%s_%d" % c)
def test_window_sweep_with_loader_value_and_index_wavefronts(oracle, case):
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    print("case squad", case, flush=True)
    L, width, algo, R = case
    for iv, first, sign in ((False, 0.0, 1.0), (True, 0.0, 1.0), (False, 0.0, -0.5), (False, 0.4, 1.0)):
        B, H, W = (2, 3, 21) if R == 4 else (1, 4, 9)
        pr = random_problem(500 + L, algo, B, H, W, L, DIRS8 if R == 8 else DIRS4, 2, integer_valued=iv, per_edge=True, rho=np.linspace(0.3, 0.9, R))
        d = np.abs(np.arange(L)[:, None] - np.arange(L)[None, :]).astype(np.float32)
        pr.pairwise = np.minimum(d, np.float32(width)) if first == 0.0 else np.minimum(d * np.float32(0.3) + np.float32(first), np.float32(0.3 * width + first))
        pr.pairwise_kind, pr.trunc, pr.scale = (1, float(width), 1.0) if first == 0.0 else (3, float(width), 1.0)
        pr.edge_weight = np.abs(pr.edge_weight)
        if sign < 0:
            pr.edge_weight = (pr.edge_weight * np.where(np.random.default_rng(L).random(pr.edge_weight.shape) > 0.2, 1.0, sign)).astype(np.float32)
        f = oracle_forward(oracle, pr)
        try:
            assert mrf.mrf_tune(2, 2) == 0 and mrf.mrf_tune(9, 2) == 0
            for beside in (4, 8):
                assert mrf.mrf_tune(10, beside) == 0
                check_forward(run_gpu(pr, backward=False), f)
                assert mrf.mrf_last_sweep_kernel(False) == "mrf_fwd_sweep_window_squad", mrf.mrf_last_sweep_launch(False)
        finally:
            for k in (2, 9, 10):
                mrf.mrf_tune(k, 0)


# both sides of the bounds of window 8: 129..192 labels to 256 scanlines (656 with more than three source arrays), more labels to 512
@pytest.mark.parametrize("case", [("trwp", 32, 130, 4, True), ("trwp", 33, 130, 4, False), ("isgmr", 8, 192, 4, True), ("isgmr", 9, 192, 4, False),
                                  ("trwp", 64, 193, 4, True), ("trwp", 65, 193, 4, False), ("trwp", 43, 160, 8, True)], ids=lambda c: "%s_%d_%d_%d" % c[:4])
def test_which_window_sweep_runs_for_many_labels(oracle, case):
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    print("case which window sweep", case, flush=True)
    algo, B, L, R, squad = case
    pr = random_problem(670 + L, algo, B, 8, 8, L, DIRS8 if R == 8 else DIRS4, 2, symmetric=False, rho=np.linspace(0.3, 0.9, R))
    pr.pairwise = np.minimum(np.abs(np.arange(L)[:, None] - np.arange(L)[None, :]), 8).astype(np.float32)
    pr.pairwise_kind, pr.trunc, pr.scale = 1, 8.0, 1.0
    check_forward(run_gpu(pr, backward=False), oracle_forward(oracle, pr))
    kernel = mrf.mrf_last_sweep_kernel(False)
    assert kernel == ("mrf_fwd_sweep_window_squad" if squad else "mrf_fwd_sweep_window_duo"), mrf.mrf_last_sweep_launch(False)


CHAIN_CASES = [
    # seed, algo, B, H, W, L, dirs, K, integer_valued, per_edge
    (81, "trwp", 1, 3, 70, 96, DIRS4, 2, False, True),      # scanlines many times the ring
    (82, "isgmr", 1, 2, 45, 40, DIRS8, 2, True, True),
    (83, "trwp", 2, 5, 6, 128, DIRS8, 2, False, False),
    (84, "isgmr", 1, 7, 9, 1, DIRS4, 2, False, True),
    (85, "trwp", 1, 1, 11, 20, DIRS16, 2, True, True),      # one row: most scanlines have one node
    (86, "trwp", 1, 9, 2, 65, [(0, 1), (1, 0), (-1, 0)], 3, False, True),
    (87, "trwp", 1, 4, 30, 200, DIRS4, 2, False, True),     # three and four labels per lane
    (88, "isgmr", 1, 3, 20, 256, DIRS8, 2, True, False),
]


@pytest.mark.parametrize("case", CHAIN_CASES, ids=lambda c: "seed%d" % c[0])
def test_chain_wavefront_backward_layout(oracle, case):
    """Backward sweeps that keep only the node-to-node chain on one wavefront and give the rest
    of a node to 2, 4, 6 or 8 helper wavefronts (chosen for launches with few scanlines when no
    grad_pairwise is asked for): each against the oracle, and against the one-wavefront sweep."""
    import paper_1910_10892_amd as mrf
    print("case chain backward", case[:8], flush=True)
    seed, algo, B, H, W, L, dirs, K, iv, pe = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=pe,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    got = {}
    try:
        assert mrf.mrf_tune(6, 1) == 0
        got[0] = full_check(oracle, pr, want_V=False)
        assert mrf.mrf_tune(6, 2) == 0
        for ni in (2, 4, 6, 8, 12):
            assert mrf.mrf_tune(7, ni) == 0
            got[ni] = full_check(oracle, pr, want_V=False)
    finally:
        mrf.mrf_tune(6, 0)
        mrf.mrf_tune(7, 0)
    for ni in (2, 4, 6, 8, 12):
        for name in ("grad_unary", "grad_edge_weight"):
            np.testing.assert_allclose(getattr(got[ni], name), getattr(got[0], name), rtol=1e-5, atol=1e-4,
                                       err_msg="%d helpers, %s" % (ni, name))


CHAIN_HOT_CASES = [
    # seed, algo, B, H, W, L, dirs, K, kind, trunc, integer_valued
    (101, "trwp", 1, 4, 60, 96, DIRS4, 2, 1, 8.0, False),
    (102, "isgmr", 2, 3, 25, 40, DIRS8, 2, 1, 2.0, True),
    (103, "trwp", 1, 6, 9, 130, DIRS8, 2, 2, 30.0, False),
    (104, "isgmr", 1, 2, 31, 256, DIRS4, 3, 2, 200.0, False),
    (105, "trwp", 1, 5, 5, 2, DIRS4, 2, 1, 1.0, True),
    (106, "trwp", 1, 3, 40, 64, [(0, 1), (0, -1), (1, 1)], 2, 3, 2.0, False),
]


@pytest.mark.parametrize("case", CHAIN_HOT_CASES, ids=lambda c: "seed%d" % c[0])
def test_chain_wavefront_backward_hot_label(oracle, case):
    """The chain layout on truncated models, where most labels scatter to one source label: with
    and without words of their own for that label's lanes, 2 to 12 helpers, against the oracle and
    against each other."""
    import paper_1910_10892_amd as mrf
    from mrf_inputs import truncated_linear, truncated_quadratic, sgm_penalties
    print("case chain backward, hot label", case, flush=True)
    seed, algo, B, H, W, L, dirs, K, kind, trunc, iv = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=True,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    scale = 1.0 if iv else 0.37
    pr.pairwise = (truncated_linear(L, trunc, scale) if kind == 1 else
                   truncated_quadratic(L, trunc, scale) if kind == 2 else sgm_penalties(L, 0.5, 2.0))
    pr.pairwise_kind, pr.trunc, pr.scale = kind, trunc, scale
    got = {}
    try:
        assert mrf.mrf_tune(6, 2) == 0
        for hot in (1, 2):
            for ni in (2, 8, 12):
                assert mrf.mrf_tune(12, hot) == 0 and mrf.mrf_tune(7, ni) == 0
                got[hot, ni] = full_check(oracle, pr, want_V=False)
                assert mrf.mrf_last_sweep_kernel(1) == "mrf_bwd_sweep_chain"
    finally:
        mrf.mrf_tune(6, 0)
        mrf.mrf_tune(7, 0)
        mrf.mrf_tune(12, 0)
    for key in got:
        for name in ("grad_unary", "grad_edge_weight"):
            np.testing.assert_allclose(getattr(got[key], name), getattr(got[1, 2], name), rtol=1e-5, atol=1e-4,
                                       err_msg="%s, %s" % (key, name))


CHAIN_GV_CASES = [
    # seed, algo, B, H, W, L, dirs, K, integer_valued, per_edge
    (91, "trwp", 2, 6, 40, 21, DIRS4, 2, False, True),
    (92, "isgmr", 1, 5, 33, 32, DIRS8, 2, True, True),
    (93, "trwp", 1, 9, 4, 2, DIRS4, 3, False, False),
    (94, "trwp", 1, 1, 13, 17, DIRS8, 2, True, True),       # one row: most scanlines have one node
    (95, "isgmr", 3, 4, 7, 1, DIRS4, 2, False, True),
    (96, "trwp", 1, 5, 30, 48, DIRS4, 2, False, True),      # more than 32 labels: fewer helpers fit
    (97, "isgmr", 1, 4, 21, 64, DIRS4, 2, True, True),
]


@pytest.mark.parametrize("case", CHAIN_GV_CASES, ids=lambda c: "seed%d" % c[0])
def test_chain_wavefront_backward_with_pairwise_gradient(oracle, case):
    """The chain layout when grad_pairwise is asked for (L <= 32: every helper wavefront keeps a
    V-gradient accumulator of its own): 2, 4, 6, 8 helpers against the oracle and against the
    one-wavefront sweep."""
    import paper_1910_10892_amd as mrf
    print("case chain backward with grad V", case[:8], flush=True)
    seed, algo, B, H, W, L, dirs, K, iv, pe = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=pe,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    got = {}
    try:
        assert mrf.mrf_tune(3, 1) == 0
        assert mrf.mrf_tune(6, 1) == 0
        got[0] = full_check(oracle, pr, want_V=True)
        assert mrf.mrf_last_sweep_kernel(1) == "mrf_bwd_sweep"
        assert mrf.mrf_tune(6, 2) == 0
        for ni in (2, 4, 6, 8, 12):
            assert mrf.mrf_tune(7, ni) == 0
            got[ni] = full_check(oracle, pr, want_V=True)
            assert mrf.mrf_last_sweep_kernel(1) == "mrf_bwd_sweep_chain"
    finally:
        mrf.mrf_tune(3, 0)
        mrf.mrf_tune(6, 0)
        mrf.mrf_tune(7, 0)
    for ni in (2, 4, 6, 8, 12):
        for name in ("grad_unary", "grad_edge_weight", "grad_pairwise"):
            np.testing.assert_allclose(getattr(got[ni], name), getattr(got[0], name), rtol=1e-5, atol=1e-4,
                                       err_msg="%d helpers, %s" % (ni, name))


@pytest.mark.parametrize("index,crop,algo,K", [c for c in CONFIG_CASES if c[0] != 5])
def test_benchmark_configs_cropped_without_pairwise_gradient(oracle, index, crop, algo, K):
    """The truncated models have no free parameters in V: run them the way bench.py does."""
    print("case config, no grad_pairwise", index, crop, algo, K, flush=True)
    pr = make_config(index, crop=crop, algo=algo, K=K)
    full_check(oracle, pr, want_V=False)


@pytest.mark.parametrize("algo,K,L,p1,p2", [("isgmr", 1, 64, 0.3, 1.7), ("isgmr", 3, 96, 1.0, 1.0),
                                           ("trwp", 2, 130, 0.5, 2.0)])
def test_sgm_penalties_through_the_window_path(oracle, algo, K, L, p1, p2):
    """The three SGM penalties (Eq. vsgm) announced as a distance function that is constant from
    distance 2 on; K = 1 with ISGMR is the revised single-pass SGM (Eq. sgm).  Window sweep against
    the oracle and, bit for bit, against the dense sweep."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    from mrf_inputs import sgm_penalties
    print("case sgm penalties", algo, K, L, flush=True)
    pr = random_problem(71, algo, 1, 6, 8, L, DIRS8, K, rho=np.linspace(0.3, 0.9, 8))
    pr.pairwise = sgm_penalties(L, p1, p2)
    pr.pairwise_kind, pr.trunc, pr.scale = 3, 2.0, 1.0
    g = full_check(oracle, pr)
    try:
        assert mrf.mrf_tune(1, 1) == 0
        d = run_gpu(pr)
    finally:
        mrf.mrf_tune(1, 0)
    for name in ("p", "q", "labels", "cost", "messages"):
        np.testing.assert_array_equal(getattr(g, name), getattr(d, name), err_msg=name)


@pytest.mark.parametrize("case", [
    (61, "trwp", 1, 6, 7, 200, DIRS4, 3, False, True),
    (62, "isgmr", 1, 5, 6, 256, DIRS8, 2, True, True),
    (63, "trwp", 2, 4, 5, 130, DIRS8, 2, False, False),
    (64, "isgmr", 1, 7, 5, 192, DIRS4, 2, False, True),
], ids=lambda c: "seed%d" % c[0])
def test_multi_wavefront_backward_layout(oracle, case):
    """Backward sweeps with one wavefront per 64 labels (chosen for launches with few scanlines
    and many labels) against the oracle, and identical to the one-wavefront layout."""
    import paper_1910_10892_amd as mrf
    print("case split backward", case[:8], flush=True)
    seed, algo, B, H, W, L, dirs, K, iv, pe = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=pe,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    try:
        assert mrf.mrf_tune(2, 1) == 0
        a = full_check(oracle, pr)
        assert mrf.mrf_tune(2, 2) == 0
        b = full_check(oracle, pr)
    finally:
        mrf.mrf_tune(2, 0)
    for name in ("grad_unary", "grad_edge_weight", "grad_pairwise"):
        np.testing.assert_allclose(getattr(a, name), getattr(b, name), rtol=1e-5, atol=1e-4, err_msg=name)


PACK_CASES = [
    (71, "isgmr", 2, 9, 11, 21, DIRS4, 3, False, True),
    (72, "trwp", 1, 7, 13, 16, DIRS8, 2, True, True),
    (73, "isgmr", 1, 6, 10, 5, DIRS16, 2, False, True),     # 16 directions: scanlines of very different length
    (74, "trwp", 3, 5, 6, 32, DIRS4, 2, False, False),
    (75, "isgmr", 1, 8, 3, 17, DIRS8, 2, True, True),
    (76, "trwp", 1, 3, 9, 1, DIRS4, 2, False, True),
    (77, "isgmr", 2, 13, 17, 21, DIRS8, 2, False, True),    # 21 labels, scanlines of many lengths: packs of three
    (78, "trwp", 1, 10, 7, 20, DIRS4, 3, True, True),
    (79, "isgmr", 1, 5, 64, 18, DIRS4, 2, True, False),
]


@pytest.mark.parametrize("case", PACK_CASES, ids=lambda c: "seed%d" % c[0])
def test_packed_scanlines_layout(oracle, case):
    """For L <= 32 several scanlines share a wavefront; results must not depend on it."""
    import paper_1910_10892_amd as mrf
    print("case packed", case[:8], flush=True)
    seed, algo, B, H, W, L, dirs, K, iv, pe = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=pe,
                        rho=np.linspace(0.3, 0.9, len(dirs)))
    try:
        assert mrf.mrf_tune(3, 1) == 0
        a = full_check(oracle, pr)
        assert mrf.mrf_tune(3, 2) == 0 and mrf.mrf_tune(11, 1) == 0      # packed, one wavefront does all
        b = full_check(oracle, pr)
        assert mrf.mrf_tune(11, 2) == 0                                  # divided among four wavefronts
        c = full_check(oracle, pr)
        more = []
        if 16 < L <= 21:
            # three scanlines per wavefront (segments of 21 lanes), divided and not
            assert mrf.mrf_tune(13, 2) == 0
            more.append(full_check(oracle, pr))
            assert "mrf_fwd_sweep_packed<21," in mrf.mrf_last_sweep_launch(False)
            assert "mrf_bwd_sweep_packed<21," in mrf.mrf_last_sweep_launch(True)
            assert mrf.mrf_tune(11, 1) == 0
            more.append(full_check(oracle, pr))
            more.append(full_check(oracle, pr, want_V=False))
    finally:
        mrf.mrf_tune(3, 0)
        mrf.mrf_tune(11, 0)
        mrf.mrf_tune(13, 0)
    for name in ("p", "q", "labels", "cost", "messages"):
        np.testing.assert_array_equal(getattr(a, name), getattr(b, name), err_msg=name)
        np.testing.assert_array_equal(getattr(a, name), getattr(c, name), err_msg=name)
        for m in more:
            np.testing.assert_array_equal(getattr(a, name), getattr(m, name), err_msg=name)


@pytest.mark.parametrize("case", PACK_CASES, ids=lambda c: "seed%d" % c[0])
def test_packed_scanlines_with_64_bit_offsets(oracle, case):
    """What arrays beyond the 32-bit offsets get, on small ones: one wavefront that does all, and a value wavefront with two index
    wavefronts (launches of few scanlines), also with three scanlines per wavefront; the same bits as mrf_fwd_sweep_narrow."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    print("case packed 64-bit", case[:8], flush=True)
    seed, algo, B, H, W, L, dirs, K, iv, pe = case
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=pe, rho=np.linspace(0.3, 0.9, len(dirs)))
    f = oracle_forward(oracle, pr)
    out = []
    try:
        for form, three in ((1, 1), (3, 1), (6, 1), (3, 2), (6, 2)) if 16 < L <= 21 else ((1, 1), (3, 1), (6, 1)):
            assert mrf.mrf_tune(3, 2) == 0 and mrf.mrf_tune(11, form) == 0 and mrf.mrf_tune(13, three) == 0
            out.append(run_gpu(pr, backward=False))
            check_forward(out[-1], f)
            launch = mrf.mrf_last_sweep_launch(False)
            if form == 1:
                assert launch.startswith("mrf_fwd_sweep_narrow"), launch
            else:
                assert launch.startswith("mrf_fwd_sweep_packed<%d," % (21 if three == 2 else 16 if L <= 16 else 32)), launch
                assert (",2>" if form == 6 else ",0>") in launch, launch
            for name in ("p", "q", "labels", "cost", "messages"):
                np.testing.assert_array_equal(getattr(out[0], name), getattr(out[-1], name), err_msg=name)
    finally:
        for k in (3, 11, 13):
            mrf.mrf_tune(k, 0)


def test_optional_outputs_may_be_null(oracle):
    from gpu_harness import GpuProblem
    import torch
    print("case optional outputs", flush=True)
    for algo in ("isgmr", "trwp"):
        pr = make_config(1, algo=algo, K=2)
        full = GpuProblem(pr)
        full.forward(); full.backward()
        ref = full.results()
        g = GpuProblem(pr, want_messages=False)
        fn = __import__("paper_1910_10892_amd").mrf_isgmr_forward if algo == "isgmr" else \
            __import__("paper_1910_10892_amd").mrf_trwp_forward
        fn(g.prob, g.cost, None, g.p, g.q, None, g.workspace)
        g.backward(want_w=False, want_V=False)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(g.cost.cpu().numpy(), ref.cost)
        np.testing.assert_array_equal(g.p.cpu().numpy(), ref.p)
        # (without grad_pairwise the library may run other backward kernels: same sums, other order)
        np.testing.assert_allclose(g.grad_unary.cpu().numpy(), ref.grad_unary, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("algo,B,H,W,L", [("isgmr", 1, 6, 9, 16), ("trwp", 1, 7, 8, 21), ("trwp", 1, 5, 9, 40), ("isgmr", 1, 6, 5, 48),
                                          ("trwp", 1, 6, 7, 96), ("isgmr", 1, 4, 6, 100), ("trwp", 1, 4, 5, 200), ("trwp", 60, 6, 5, 12)])
@pytest.mark.parametrize("per_edge", [True, False])
def test_each_gradient_alone(oracle, algo, B, H, W, L, per_edge):
    """Every combination of the optional gradients, with a scalar weight and with one per edge, on a workspace that holds garbage
    when the backward pass starts: its header, what the sweeps add to and what nobody asked for."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import GpuProblem
    print("case each gradient alone", algo, B, H, W, L, per_edge, flush=True)
    pr = random_problem(820 + L, algo, B, H, W, L, DIRS4, 2, symmetric=False, per_edge=per_edge, rho=np.linspace(0.3, 0.9, 4))
    pr.grad_cost = (pr.grad_cost * 0.2).astype(np.float32)
    g = GpuProblem(pr)
    g.forward()
    f = g.results(False)
    check_forward(f, oracle_forward(oracle, pr))
    ref = oracle_backward(oracle, pr, f.p, f.q, np.float64)
    for want_w, want_V in ((True, True), (True, False), (False, True), (False, False)):
        for x in (g.grad_unary, g.grad_edge_weight, g.grad_pairwise):
            x.fill_(float("nan"))
        g.workspace.fill_(0xFF)
        g.backward(want_w=want_w, want_V=want_V)
        got = g.results()
        launch = mrf.mrf_last_sweep_launch(True)
        if want_V and launch.startswith("mrf_bwd_sweep_chain<1,") and ",false,true,false" in launch:      # tables in LDS
            assert launch.split(">")[0].endswith(",false,true,false" if want_w else ",false,true,false,false,false,false"), launch
        check_grad("grad_unary", got.grad_unary, None, ref.grad_unary)
        for name, want in (("grad_edge_weight", want_w), ("grad_pairwise", want_V)):
            if want:
                check_grad(name, getattr(got, name), None, getattr(ref, name))
            else:
                assert np.isnan(getattr(got, name)).all(), name


def test_backward_is_reproducible_run_to_run():
    from gpu_harness import GpuProblem
    print("case reproducible", flush=True)
    for idx, crop, algo in ((2, (24, 40), "trwp"), (5, (24, 32), "isgmr")):
        pr = make_config(idx, crop=crop, algo=algo)
        g = GpuProblem(pr)
        g.forward(); g.backward()
        a = g.results()
        g.poison_outputs()
        g.forward(); g.backward()
        b = g.results()
        for name in ("cost", "p", "q", "grad_unary", "grad_edge_weight", "grad_pairwise"):
            np.testing.assert_array_equal(getattr(a, name), getattr(b, name), err_msg=name)


def cancelling_problem(seed, algo, B, H, W, L):
    """Images in pairs with opposite gradients of the costs: every entry of grad_pairwise is a sum that cancels, so what
    is left is the rounding of its additions, which shows any change of their order."""
    pr = random_problem(seed, algo, B, H, W, L, DIRS8, 2, symmetric=False)
    for x in (pr.unary, pr.grad_cost):
        x[B // 2:] = x[:B // 2]
    pr.edge_weight[:, B // 2:] = pr.edge_weight[:, :B // 2]
    pr.grad_cost[B // 2:] *= -1.0
    return pr


def check_reproducible(g):
    """Four backward passes of a problem of the kind above, bit for bit."""
    g.forward()
    runs = []
    for _ in range(4):
        g.workspace.fill_(0xFF)
        g.backward()
        runs.append(g.results())
    assert (runs[0].grad_pairwise != 0).any()                  # (the order matters)
    for r in runs[1:]:
        for name in ("grad_unary", "grad_edge_weight", "grad_pairwise"):
            np.testing.assert_array_equal(getattr(r, name), getattr(runs[0], name), err_msg=name)


@pytest.mark.parametrize("algo,B,L", [("isgmr", 32, 21), ("isgmr", 32, 16), ("isgmr", 16, 32), ("isgmr", 48, 8), ("trwp", 64, 25)])
def test_pairwise_gradient_of_few_labels_is_reproducible(algo, B, L):
    """Launches with several wavefronts per workgroup."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import GpuProblem
    print("case reproducible few labels", algo, B, L, flush=True)
    g = GpuProblem(cancelling_problem(797 + L, algo, B, 24, 32, L))
    try:
        assert mrf.mrf_tune(3, 2) == 0 and mrf.mrf_tune(20, 1) == 0
        check_reproducible(g)
        launch = mrf.mrf_last_sweep_launch(True)
    finally:
        mrf.mrf_tune(3, 0)
        mrf.mrf_tune(20, 0)
    assert launch.startswith("mrf_bwd_sweep_narrow") and int(launch.split("block=")[1].split()[0]) > 64, launch


@pytest.mark.parametrize("L", [33, 40, 46, 50, 64])
def test_pairwise_gradient_behind_the_chain_sweep_is_reproducible(L):
    """33..64 labels, TRWP: the pass behind the chain sweep keeps a table per wavefront (sixteen to four of them)."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import GpuProblem
    print("case reproducible behind the chain", L, flush=True)
    check_reproducible(GpuProblem(cancelling_problem(798 + L, "trwp", 16, 24, 32, L)))
    assert mrf.mrf_last_sweep_launch(True).startswith("mrf_bwd_sweep_chain<1,") and "true,true" in mrf.mrf_last_sweep_launch(True)


def test_waits_between_wavefronts_are_bounded(oracle):
    """The layouts that spread a scanline over several wavefronts give every wait a budget.  With a
    budget of one turn (set from the host) their first unmet wait gives up: every kernel still ends
    normally, and mrf_workspace_fault reports it.  With the default budget the same calls complete
    and report nothing."""
    import torch
    import paper_1910_10892_amd as mrf
    from gpu_harness import GpuProblem
    print("case bounded waits", flush=True)
    cases = [(make_config(2, crop=(24, 40), algo="trwp"), {}),       # value / loader / index wavefronts, chain backward
             (make_config(4, crop=(10, 12), algo="trwp", K=2), {}),  # value wavefronts that meet through LDS, index wavefronts
             (make_config(5, crop=(24, 32), algo="trwp"), {}),       # packed scanlines with index wavefronts
             (make_config(5, crop=(24, 32), algo="trwp"), {20: 2})]  # chain backward with two scanlines per workgroup
    for pr, knobs in cases:
        g = GpuProblem(pr)
        for k, v in knobs.items():
            assert mrf.mrf_tune(k, v) == 0
        try:
            assert mrf.mrf_tune(14, 1) == 0
            g.forward()
            fwd = mrf.mrf_workspace_fault(g.workspace)
            g.backward(want_V=False)
            bwd = mrf.mrf_workspace_fault(g.workspace)
            if knobs:
                assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_chain_pk" and bwd == -11
        finally:
            mrf.mrf_tune(14, 0)
        print("  ", pr.name, mrf.mrf_last_sweep_launch(False), fwd, mrf.mrf_last_sweep_launch(True), bwd, flush=True)
        assert fwd in (0, -11) and bwd in (0, -11)
        assert fwd == -11 or bwd == -11          # these shapes take multi-wavefront layouts: some wait is unmet at first
        # default budget: complete, correct, nothing reported
        g.poison_outputs()
        g.forward()
        assert mrf.mrf_workspace_fault(g.workspace) == 0
        g.backward(want_V=False)
        assert mrf.mrf_workspace_fault(g.workspace) == 0
        got = g.results()
        f = oracle_forward(oracle, pr)
        check_forward(got, f)
        b64 = oracle_backward(oracle, pr, f.p, f.q, np.float64)
        check_grad("grad_unary", got.grad_unary, None, b64.grad_unary)
        for k in knobs:
            mrf.mrf_tune(k, 0)


def test_workspace_too_small_is_an_error_not_a_fault():
    from gpu_harness import GpuProblem
    import paper_1910_10892_amd as mrf
    print("case small workspace", flush=True)
    pr = make_config(1)
    g = GpuProblem(pr)
    small = g.workspace[: 256]
    with pytest.raises(mrf.MrfError) as ei:
        mrf.mrf_isgmr_forward(g.prob, g.cost, g.labels, g.p, g.q, g.messages, small)
    assert ei.value.status == -6


@pytest.mark.parametrize("index,crop,algo", [
    (2, None, "isgmr"),            # stereo shape, all four directions in one launch
    (3, (96, 312), "isgmr"),       # driving-stereo recipe, 1/16 of the area, L = 192, 8 directions
    (4, (64, 64), "trwp"),         # denoising recipe, 1/16 of the area, L = 256
    (5, None, "isgmr"),            # segmentation shape at full size (batch 4, 512 x 512, L = 21)
    (5, None, "trwp"),
])
def test_large_configs(oracle, index, crop, algo):
    """The other benchmark shapes at full size where the oracle finishes in seconds on all host
    threads, else on a centred fraction of the grid with every other parameter unchanged."""
    print("case large config", index, crop, algo, flush=True)
    pr = make_config(index, crop=crop, algo=algo)
    full_check(oracle, pr, threads=True)


def test_full_size_stereo_config_trwp(oracle):
    """The configuration the bench times (TRWP, 256x512, L = 96, K = 5), whole grid, in the
    launch configuration the bench uses (no grad_pairwise buffer: truncated linear V), and once
    more with that buffer; oracle forward on all host threads (bit-identical to one thread,
    asserted in the CPU suite)."""
    from gpu_harness import run_gpu
    print("case full config 2", flush=True)
    pr = make_config(2)
    f = oracle_forward(oracle, pr, threads=True)
    b32 = oracle_backward(oracle, pr, f.p, f.q, np.float32)
    b64 = oracle_backward(oracle, pr, f.p, f.q, np.float64)
    for want_V in (False, True):
        print("  grad_pairwise buffer:", want_V, flush=True)
        g = run_gpu(pr, want_V=want_V)
        check_forward(g, f)
        check_backward(g, b32, b64, want_V)


SGM_STD_CASES = [
    # seed, B, H, W, L, dirs, integer_valued, per_edge, kind (0 dense table, 3 SGM penalties)
    (501, 1, 6, 9, 16, DIRS8, False, True, 3),
    (502, 2, 5, 7, 70, DIRS4, True, True, 3),        # integer data: ties in both argmins
    (503, 1, 4, 6, 130, DIRS16, False, False, 3),
    (504, 1, 7, 5, 21, DIRS8, False, True, 0),       # general dense table
    (505, 1, 1, 9, 200, DIRS4, True, True, 3),       # one row
    (506, 1, 3, 3, 256, DIRS8, False, True, 0),
    (507, 1, 5, 5, 1, DIRS4, False, True, 0),
]


@pytest.mark.parametrize("case", SGM_STD_CASES, ids=lambda c: "seed%d" % c[0])
def test_standard_single_pass_sgm(oracle, case):
    """The standard SGM update (Eq. sgm_old: the message carries the node's own unary) and its
    aggregation (Eq. isgmr-aggregation-old) as a problem flag: forward outputs against the oracle;
    the backward entry points refuse the flag."""
    import torch
    import paper_1910_10892_amd as mrf
    from gpu_harness import GpuProblem
    from mrf_inputs import sgm_penalties
    print("case standard sgm", case, flush=True)
    seed, B, H, W, L, dirs, iv, pe, kind = case
    pr = random_problem(seed, "isgmr", B, H, W, L, dirs, 1, integer_valued=iv, per_edge=pe, symmetric=False)
    if kind == 3:
        pr.pairwise = sgm_penalties(L, 1.0 if iv else 0.3, 2.0 if iv else 1.7)
        pr.pairwise_kind, pr.trunc, pr.scale = 3, 2.0, 1.0
    pr.sgm_standard = True
    g = GpuProblem(pr)
    g.poison_outputs()
    g.forward()
    got = g.results(backward=False)
    f = oracle.sgm_standard_forward(pr.unary, pr.pairwise, pr.dirs, edge_weight=pr.edge_weight,
                                    edge_weight_scalar=pr.edge_weight_scalar)
    check_forward(got, f)
    np.testing.assert_array_equal(got.messages, f.messages)
    np.testing.assert_array_equal(got.cost, f.cost)
    with pytest.raises(mrf.MrfError) as ei:
        g.backward()
    assert ei.value.status == -8
    # more than one iteration has no meaning for a single-pass method
    g.prob.K = 2
    assert mrf.mrf_validate(g.prob, mrf.MRF_ISGMR) == -8


def _progress(msg):
    """Long tests say where they are: on stdout and, where a GPU job's output folder exists, in
    a file there (a run that is silent for minutes is taken for hung)."""
    import os, time
    print(msg, flush=True)
    d = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "gpurun_out")
    if os.path.isdir(d):
        with open(os.path.join(d, "test_progress.log"), "a") as fh:
            fh.write("%s %s\n" % (time.strftime("%H:%M:%S"), msg))


def _full_size_check(oracle, pr, want_V, fwd_launch, bwd_launch):
    """Whole-grid parity in the launch configuration bench.py times: forward element by element
    (oracle forward on all host threads, bit-identical to one thread), gradients against the
    double replay, and the kernel instantiations the launch rules picked."""
    import gc
    import torch
    import paper_1910_10892_amd as mrf
    from gpu_harness import GpuProblem
    g = GpuProblem(pr)
    g.poison_outputs()
    g.forward()
    g.backward(want_V=want_V)
    assert mrf.mrf_workspace_fault(g.workspace) == 0
    assert mrf.mrf_last_sweep_launch(False) == fwd_launch, mrf.mrf_last_sweep_launch(False)
    assert mrf.mrf_last_sweep_launch(True) == bwd_launch, mrf.mrf_last_sweep_launch(True)
    _progress("  GPU done; oracle forward (all host threads)")
    f = oracle_forward(oracle, pr, threads=True)
    _progress("  oracle forward done; comparing")
    for name in ("p", "q", "labels"):
        got = getattr(g, name).cpu().numpy()
        assert np.array_equal(got, getattr(f, name)), name
        del got
    for name in ("messages", "cost"):
        got = getattr(g, name).cpu().numpy()
        ref = getattr(f, name)
        # (identical in fact: same operations in the same order)
        bad = np.abs(got - ref) > ATOL + RTOL * np.abs(ref)
        assert not bad.any(), "%s: %d entries off" % (name, int(bad.sum()))
        del got, bad
    p, q = f.p, f.q
    del f
    gc.collect()
    _progress("  oracle backward (double)")
    b64 = oracle_backward(oracle, pr, p, q, np.float64)
    _progress("  oracle backward done; comparing")
    check_grad("grad_unary", g.grad_unary.cpu().numpy(), None, b64.grad_unary)
    check_grad("grad_edge_weight", g.grad_edge_weight.cpu().numpy(), None, b64.grad_edge_weight)
    if want_V:
        check_grad("grad_pairwise", g.grad_pairwise.cpu().numpy(), None, b64.grad_pairwise)


def test_full_size_driving_stereo_config_isgmr(oracle):
    """The largest benchmark shape whole, as bench.py times it: ISGMR, 384 x 1248, L = 192, 8
    directions, K = 3 -- 9,788 scanlines per launch, message and index arrays beyond 2^31 bytes.
    The first iteration runs the launch with zero messages, the later ones the same launch on the
    per-pair sums that a streaming pass forms from the previous iteration's messages.  (The oracle's share of the test is about 35 s per iteration on 16 host
    threads.)"""
    _progress("case full config 3")
    pr = make_config(3)
    _full_size_check(oracle, pr, False,
                     "mrf_fwd_sweep_window<3,1,4,false,2> grid=9788 block=64 after mrf_isgmr_presum<8,4>",
                     "mrf_bwd_sweep<3,1,2,false,true,false,false> grid=2447 block=256")


def test_full_size_denoising_config_trwp(oracle):
    """The denoising shape whole: TRWP, 256 x 256, L = 256, truncated quadratic, rho = 0.5, in the
    launch configuration of the bench (no grad_pairwise buffer), all K = 10 iterations."""
    _progress("case full config 4")
    pr = make_config(4)
    _full_size_check(oracle, pr, False,
                     "mrf_fwd_sweep_window_squad<4,4,true,16,8> grid=256 block=768",
                     "mrf_bwd_sweep_chain<4,4,1,8,false,false,true> grid=256 block=576")


def test_full_size_denoising_config_dense_sweep(oracle):
    """The same shape through the dense O(L^2) sweep (the launch bench.py times as the dense
    variant of this configuration): K = 2, forward outputs only."""
    import torch
    import paper_1910_10892_amd as mrf
    from gpu_harness import GpuProblem
    _progress("case full config 4, dense sweep (K = 2)")
    pr = make_config(4, K=2)
    pr.pairwise_kind = 0
    g = GpuProblem(pr)
    g.poison_outputs()
    g.forward()
    torch.cuda.synchronize()
    assert mrf.mrf_last_sweep_launch(False) == "mrf_fwd_sweep_sliced<4,4,4,true> grid=256 block=512"
    f = oracle_forward(oracle, pr, threads=True)
    for name in ("p", "q", "labels", "messages", "cost"):
        assert np.array_equal(getattr(g, name).cpu().numpy(), getattr(f, name)), name


def _drawn_problem(seed):
    """A small problem with everything drawn at random: shape, label count (biased towards the
    borders of the kernels' layouts), direction set, iteration count, model and weights."""
    from mrf_inputs import truncated_linear, truncated_quadratic, sgm_penalties
    rng = np.random.default_rng(5000 + seed)
    algo = ("isgmr", "trwp")[int(rng.integers(0, 2))]
    B = int(rng.integers(1, 3))
    H, W = int(rng.integers(1, 11)), int(rng.integers(1, 14))
    L = int(rng.choice([1, 2, 3, 15, 16, 17, 21, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 191, 192, 193, 255, 256]))
    sets = [DIRS4, DIRS8, DIRS16, [(0, 1)], [(1, 0), (-1, 0)], [(0, 1), (0, -1), (1, 1)], [(1, 2), (-1, -2), (0, 1), (2, -1)]]
    dirs = sets[int(rng.integers(0, len(sets)))]
    K = int(rng.integers(1, 4))
    iv = bool(rng.integers(0, 2))
    pe = bool(rng.integers(0, 4) > 0)
    pr = random_problem(6000 + seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=pe,
                        rho=rng.uniform(0.2, 1.0, len(dirs)))
    kind = int(rng.integers(0, 4))
    if kind and L >= 2:
        scale = 1.0 if iv else 0.41
        if kind == 1:
            trunc = float(rng.choice([1.0, 2.0, 3.0, 8.0, 11.0, 16.0, 40.0]))
            pr.pairwise = truncated_linear(L, trunc, scale)
        elif kind == 2:
            trunc = float(rng.choice([1.0, 4.0, 30.0, 200.0]))
            pr.pairwise = truncated_quadratic(L, trunc, scale)
        else:
            trunc = 2.0
            pr.pairwise = sgm_penalties(L, 0.5 if not iv else 1.0, 2.0)
        pr.pairwise_kind, pr.trunc, pr.scale = kind, trunc, scale
        if pr.edge_weight is not None and rng.integers(0, 3) == 0:
            pr.edge_weight = (pr.edge_weight * np.where(rng.random(pr.edge_weight.shape) > 0.15, 1.0, -0.5)).astype(np.float32)
    return pr, bool(rng.integers(0, 2))


# MRF_TEST_EXTRA_SEEDS=n adds n further seeds to each of the three drawn-problem tests (a longer soak)
EXTRA_SEEDS = int(os.environ.get("MRF_TEST_EXTRA_SEEDS", "0"))


@pytest.mark.parametrize("seed", range(150 + EXTRA_SEEDS))
def test_drawn_problems_default_dispatch(oracle, seed):
    """Whatever kernels the launch rules pick for a randomly drawn small problem, with and without
    a grad_pairwise buffer."""
    pr, want_V = _drawn_problem(seed)
    print("case drawn", seed, pr.algo, pr.shape, len(pr.dirs), pr.K, pr.pairwise_kind, pr.trunc, want_V, flush=True)
    # The backward pass is linear in grad c, and with many directions and iterations it amplifies
    # it by orders of magnitude (ISGMR re-injects every message into R - 2 others per iteration).
    # The absolute tolerance only means something for fp32 tensors of moderate size, so grad c is
    # scaled to keep the largest gradient entry near 10.
    f = oracle_forward(oracle, pr)
    b = oracle_backward(oracle, pr, f.p, f.q, np.float64)
    big = max(float(np.abs(b.grad_unary).max()), float(np.abs(b.grad_pairwise).max()),
              float(np.abs(b.grad_edge_weight).max()) if b.grad_edge_weight is not None else 0.0)
    if big > 10.0:
        pr.grad_cost = (pr.grad_cost * np.float32(10.0 / big)).astype(np.float32)
    full_check(oracle, pr, want_V=want_V)


@pytest.mark.parametrize("seed", range(120 + EXTRA_SEEDS))
def test_drawn_problems_forced_layouts(oracle, seed):
    """The same kind of random problems with the kernel-choice knobs drawn at random too, so that
    layouts meet shapes they would not be picked for (the results may not depend on the knobs)."""
    import paper_1910_10892_amd as mrf
    pr, want_V = _drawn_problem(1000 + seed)
    rng = np.random.default_rng(9000 + seed)
    knobs = {2: int(rng.integers(0, 3)), 3: int(rng.integers(0, 3)), 4: int(rng.integers(0, 3)),
             5: int(rng.integers(0, 3)), 6: int(rng.integers(0, 3)), 7: int(rng.choice([0, 2, 4, 6, 8, 12])),
             8: int(rng.integers(0, 3)), 9: int(rng.integers(0, 3)), 10: int(rng.choice([0, 4, 8])),
             11: int(rng.integers(0, 3)), 12: int(rng.integers(0, 3)), 13: int(rng.integers(0, 3)), 15: int(rng.integers(0, 3)), 16: int(rng.integers(0, 3)), 17: int(rng.integers(0, 3)), 18: int(rng.integers(0, 2)), 19: int(rng.integers(0, 2)), 20: int(rng.integers(0, 3))}
    print("case drawn+knobs", seed, pr.algo, pr.shape, len(pr.dirs), pr.K, pr.pairwise_kind, pr.trunc, want_V, knobs,
          flush=True)
    f = oracle_forward(oracle, pr)
    b = oracle_backward(oracle, pr, f.p, f.q, np.float64)
    big = max(float(np.abs(b.grad_unary).max()), float(np.abs(b.grad_pairwise).max()),
              float(np.abs(b.grad_edge_weight).max()) if b.grad_edge_weight is not None else 0.0)
    if big > 10.0:
        pr.grad_cost = (pr.grad_cost * np.float32(10.0 / big)).astype(np.float32)
    try:
        for k, v in knobs.items():
            assert mrf.mrf_tune(k, v) == 0
        full_check(oracle, pr, want_V=want_V)
    finally:
        for k in knobs:
            mrf.mrf_tune(k, 0)


RHO_EDGE_CASES = [
    # seed, B, H, W, L, dirs, K, kind, trunc, integer_valued, per_edge weights
    (201, 2, 6, 9, 21, DIRS4, 2, 0, 0.0, False, True),
    (202, 1, 5, 11, 96, DIRS8, 2, 1, 8.0, False, True),
    (203, 1, 4, 7, 130, DIRS4, 3, 0, 0.0, True, False),
    (204, 1, 3, 9, 200, DIRS4, 2, 2, 30.0, False, True),
    (205, 1, 6, 6, 3, DIRS16, 2, 0, 0.0, False, True),
    (206, 1, 1, 12, 40, [(0, 1), (0, -1), (1, 1)], 2, 3, 2.0, False, True),
    (207, 1, 8, 3, 256, DIRS4, 1, 1, 2.0, True, True),
]


@pytest.mark.parametrize("case", RHO_EDGE_CASES, ids=lambda c: "seed%d" % c[0])
def test_trwp_with_one_rho_per_edge(oracle, case):
    """TRWP with the TRW coefficient of Eq. trwp given per directed edge (an [R,B,H,W] array like
    the edge weights) instead of per direction: forward and backward against the oracle, with and
    without grad_pairwise; and an array that repeats one value per direction gives the forward
    results of the per-direction path bit for bit."""
    from mrf_inputs import truncated_linear, truncated_quadratic, sgm_penalties
    print("case per-edge rho", case, flush=True)
    seed, B, H, W, L, dirs, K, kind, trunc, iv, pe = case
    R = len(dirs)
    pr = random_problem(seed, "trwp", B, H, W, L, dirs, K, integer_valued=iv, per_edge=pe,
                        rho=np.linspace(0.3, 0.9, R))
    if kind:
        scale = 1.0 if iv else 0.37
        pr.pairwise = (truncated_linear(L, trunc, scale) if kind == 1 else
                       truncated_quadratic(L, trunc, scale) if kind == 2 else sgm_penalties(L, 0.5, 2.0))
        pr.pairwise_kind, pr.trunc, pr.scale = kind, trunc, scale
    rng = np.random.default_rng(7000 + seed)
    base = full_check(oracle, pr, want_V=False)
    pr.rho_edge = np.broadcast_to(pr.rho[:, None, None, None], (R, B, H, W)).astype(np.float32).copy()
    same = full_check(oracle, pr, want_V=False)
    for name in ("p", "q", "labels", "cost", "messages"):
        np.testing.assert_array_equal(getattr(base, name), getattr(same, name), err_msg=name)
    np.testing.assert_allclose(same.grad_unary, base.grad_unary, rtol=1e-5, atol=1e-4)
    pr.rho_edge = (rng.integers(1, 4, (R, B, H, W)) / 4.0 if iv else rng.uniform(0.2, 0.9, (R, B, H, W))).astype(np.float32)
    pr.rho = None
    full_check(oracle, pr, want_V=False)
    full_check(oracle, pr, want_V=True)


EDGE_TABLE_CASES = [
    # seed, algo, B, H, W, L, dirs, K, integer_valued
    (301, "isgmr", 2, 5, 7, 21, DIRS4, 2, False),
    (302, "trwp", 1, 6, 5, 21, DIRS4, 3, False),
    (303, "isgmr", 1, 4, 6, 64, DIRS8, 2, False),
    (304, "trwp", 1, 3, 9, 33, DIRS8, 2, True),
    (305, "isgmr", 1, 4, 4, 5, DIRS16, 2, True),
    (306, "trwp", 1, 7, 1, 9, [(1, 0), (-1, 0), (0, 1)], 2, False),
    (307, "trwp", 1, 2, 8, 1, DIRS4, 2, False),
    (308, "isgmr", 1, 3, 5, 16, DIRS4, 1, False),
    (309, "trwp", 1, 3, 5, 17, DIRS4, 2, False),
]


# label counts around the multiples of four and the segments, one scanline per wavefront (knob value 4), several (5), three
# (knob 13); rings that wrap, scanlines of one and two nodes, counts that fill no wavefront; 3, 7 and 15 source arrays
@pytest.mark.gpu
@pytest.mark.parametrize("case", [(L, R, algo) for L in (1, 4, 5, 8, 9, 12, 13, 16, 17, 20, 21, 22, 24, 25, 28, 29, 31, 32)
                                  for R, algo in ((4, "trwp"), (4, "isgmr"), (8, "trwp"), (16, "trwp"), (16, "isgmr"))
                                  if R == 4 or L in (8, 16, 21, 32)], ids=lambda c: "%d_%d_%s" % c)
def test_packed_sweep_divided_among_four_wavefronts(oracle, case):
    """Against the oracle and bit for bit against the sweep with one wavefront: V >= 0 with a zero diagonal (the minimum of h
    is taken for that of the message) and general V with negative weights (it is not), ties."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    print("case divided", case, flush=True)
    L, R, algo = case
    dirs = DIRS16 if R == 16 else DIRS8 if R == 8 else DIRS4
    for plain, iv, (B, H, W) in ((True, False, (2, 3, 37)), (False, False, (1, 7, 19)), (True, True, (1, 1, 12)), (False, True, (3, 5, 2))):
        pr = random_problem(600 + L, algo, B, H, W, L, dirs, 2, integer_valued=iv, per_edge=True, symmetric=False, rho=np.linspace(0.3, 0.9, R))
        if plain:
            pr.pairwise, pr.edge_weight = np.abs(pr.pairwise), np.abs(pr.edge_weight)
            np.fill_diagonal(pr.pairwise, 0.0)
        else:
            sign = np.where(np.random.default_rng(L).random(pr.edge_weight.shape) > 0.1, 1.0, -0.5)
            pr.edge_weight = (pr.edge_weight * sign).astype(np.float32)
        f = oracle_forward(oracle, pr)
        out = []
        try:
            for knobs in ((4, 1), (5, 1), (2, 2), (1, 1)) if 16 < L <= 21 else ((4, 1), (5, 1), (1, 1)):
                assert mrf.mrf_tune(3, 2) == 0 and mrf.mrf_tune(11, knobs[0]) == 0 and mrf.mrf_tune(13, knobs[1]) == 0
                out.append(run_gpu(pr, backward=False))
                check_forward(out[-1], f)
                assert mrf.mrf_last_sweep_kernel(False) == ("mrf_fwd_sweep_narrow" if knobs[0] == 1 else "mrf_fwd_sweep_packed")
                for name in ("p", "q", "labels", "cost", "messages"):
                    np.testing.assert_array_equal(getattr(out[0], name), getattr(out[-1], name), err_msg=name)
        finally:
            for k in (3, 11, 13):
                mrf.mrf_tune(k, 0)


@pytest.mark.parametrize("case", EDGE_TABLE_CASES, ids=lambda c: "seed%d" % c[0])
def test_pairwise_potentials_given_per_edge(oracle, case):
    """Pairwise potentials as one L x L table per directed edge (Eq. isgmr / Eq. trwp as written)
    and the gradient of those tables (Eq. supp-gradient-pairwise): forward and backward against the
    oracle, with and without the table gradient; for TRWP also with one rho per edge."""
    print("case per-edge tables", case, flush=True)
    seed, algo, B, H, W, L, dirs, K, iv = case
    R = len(dirs)
    pr = random_problem(seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=False,
                        rho=np.linspace(0.3, 0.9, R))
    rng = np.random.default_rng(8000 + seed)
    Te = rng.integers(0, 3, (R, B, H, W, L, L)) if iv else rng.random((R, B, H, W, L, L))
    pr.pairwise_edge = Te.astype(np.float32)

    def check(want_V):
        from gpu_harness import run_gpu
        g = run_gpu(pr, want_V=want_V)
        f = oracle.forward(pr.algo, pr.unary, None, pr.dirs, pr.K, rho=pr.rho, rho_edge=pr.rho_edge,
                           pairwise_edge=pr.pairwise_edge)
        check_forward(g, f)
        b = {}
        for dt in (np.float32, np.float64):
            b[dt] = oracle.backward(pr.algo, pr.shape, None, pr.dirs, pr.K, pr.grad_cost.astype(dt), f.p, f.q,
                                    rho=pr.rho, dtype=dt, per_edge_pairwise=True,
                                    rho_edge=None if pr.rho_edge is None else pr.rho_edge.astype(dt))
        check_grad("grad_unary", g.grad_unary, b[np.float32].grad_unary, b[np.float64].grad_unary)
        if want_V:
            check_grad("grad_pairwise_edge", g.grad_pairwise, b[np.float32].grad_pairwise_edge,
                       b[np.float64].grad_pairwise_edge)
        return g

    a = check(True)
    c = check(False)
    np.testing.assert_allclose(c.grad_unary, a.grad_unary, rtol=1e-5, atol=1e-4)
    if algo == "trwp":
        pr.rho_edge = rng.uniform(0.2, 0.9, (R, B, H, W)).astype(np.float32)
        pr.rho = None
        check(True)


# label counts around the sizes of the lane groups and of their shares of the source labels; 4, 8 and 16 directions (up to
# 3, 7 and 15 source arrays); scanlines of 1 to 29 nodes (prefetches past the end)
@pytest.mark.parametrize("case", [(L, R, algo) for L in (2, 7, 8, 9, 13, 16, 17, 20, 24, 25, 29, 32, 33)
                                  for R, algo in ((4, "isgmr"), (4, "trwp"), (8, "trwp"), (16, "trwp"), (16, "isgmr"))
                                  if R == 4 or L in (8, 16, 24, 32)], ids=lambda c: "%d_%d_%s" % c)
def test_per_edge_tables_in_lane_groups(oracle, case):
    """mrf_fwd_sweep_edge_groups: bit for bit the oracle's messages, indices and costs; integer data, so that ties cross the groups."""
    from gpu_harness import run_gpu
    print("case lane groups", case, flush=True)
    L, R, algo = case
    B, H, W = (2, 3, 29) if R == 4 else (1, 7, 13)
    dirs = (DIRS16 if R == 16 else DIRS8 if R == 8 else DIRS4)
    for iv in (False, True):
        pr = random_problem(700 + L, algo, B, H, W, L, dirs, 2, integer_valued=iv, per_edge=False, rho=np.linspace(0.3, 0.9, R))
        rng = np.random.default_rng(9000 + L)
        Te = rng.integers(0, 3, (R, B, H, W, L, L)) if iv else rng.random((R, B, H, W, L, L))
        pr.pairwise_edge = Te.astype(np.float32)
        g = run_gpu(pr, want_V=False)
        check_forward(g, oracle.forward(pr.algo, pr.unary, None, pr.dirs, pr.K, rho=pr.rho, pairwise_edge=pr.pairwise_edge))


@pytest.mark.parametrize("kind", ["masks", "infinite", "nan"])
@pytest.mark.parametrize("algo", ["isgmr", "trwp"])
@pytest.mark.parametrize("L", [3, 8, 13, 16, 17, 24, 25, 32])
def test_per_edge_tables_that_are_not_finite_in_lane_groups(oracle, L, algo, kind):
    """Tables with forbidden transitions, impossible labels and pixels without one: the indices, costs and messages of the oracle."""
    from gpu_harness import run_gpu
    print("case tables not finite", L, algo, kind, flush=True)
    pr = random_problem(680 + L, algo, 2, 7, 9, L, DIRS4, 2, per_edge=False, rho=np.linspace(0.3, 0.9, 4))
    not_finite(pr, kind, L)
    rng = np.random.default_rng(9200 + L)
    pr.pairwise_edge = rng.random((4, 2, 7, 9, L, L)).astype(np.float32)
    if kind != "nan":
        never = rng.random(pr.pairwise_edge.shape) < 0.3
        never[..., np.arange(L), np.arange(L)] = False
        pr.pairwise_edge[never] = np.inf
    with np.errstate(all="ignore"):
        f = oracle.forward(pr.algo, pr.unary, None, pr.dirs, pr.K, rho=pr.rho, pairwise_edge=pr.pairwise_edge)
    g = run_gpu(pr, backward=False)
    for name in ("p", "q", "cost", "messages"):
        np.testing.assert_array_equal(getattr(g, name), getattr(f, name), err_msg=name)
    some = ~np.isnan(f.cost).any(-1)
    np.testing.assert_array_equal(g.labels[some], f.labels[some])


# the sweeps that leave the tables' gradient to a pass of its own: few scanlines (chain) and more than 1,024 (narrow: 8, 16 and
# 32 lanes, three labels per lane), ragged and odd label counts; workspace for one iteration of three (L = 2, 3 on larger
# grids: passes that add to the tables), the least workspace that is accepted, gradients off a 16-byte boundary
@pytest.mark.parametrize("case", [("isgmr", 2, 7, 9, 5, 3), ("trwp", 1, 8, 11, 21, 2), ("isgmr", 1, 6, 5, 64, 2), ("trwp", 1, 5, 6, 45, 1),
                                  ("isgmr", 1, 2, 530, 7, 2), ("isgmr", 1, 2, 530, 13, 2), ("isgmr", 1, 2, 530, 21, 3),
                                  ("isgmr", 1, 2, 530, 23, 2), ("isgmr", 1, 2, 530, 32, 2), ("trwp", 2, 2, 530, 8, 2),
                                  ("trwp", 2, 3, 530, 18, 2), ("trwp", 2, 2, 530, 29, 2),
                                  ("isgmr", 1, 130, 190, 3, 3), ("trwp", 1, 100, 170, 2, 3)], ids=lambda c: "_".join(map(str, c)))
def test_gradient_of_per_edge_tables_in_a_pass_of_its_own(oracle, case):
    import torch
    import paper_1910_10892_amd as mrf
    from gpu_harness import GpuProblem
    print("case table gradient", case, flush=True)
    algo, B, H, W, L, K = case
    pr = random_problem(800 + L, algo, B, H, W, L, DIRS4, K, per_edge=False, rho=np.linspace(0.3, 0.9, 4))
    rng = np.random.default_rng(9100 + L)
    pr.pairwise_edge = rng.random((4, B, H, W, L, L)).astype(np.float32)
    f = oracle.forward(pr.algo, pr.unary, None, pr.dirs, pr.K, rho=pr.rho, pairwise_edge=pr.pairwise_edge)
    b = {dt: oracle.backward(pr.algo, pr.shape, None, pr.dirs, pr.K, pr.grad_cost.astype(dt), f.p, f.q, rho=pr.rho, dtype=dt,
                             per_edge_pairwise=True) for dt in (np.float32, np.float64)}
    for variant in ("as asked for", "least workspace", "off a boundary", "no table gradient"):
        g = GpuProblem(pr)
        if variant == "least workspace":
            plain = mrf.MrfProblem(g.unary, torch.zeros((L, L), device="cuda:0"), pr.dirs, K, rho=pr.rho)
            g.workspace = g.workspace[:mrf.mrf_workspace_bytes(plain, g.algo, True)]
        if variant == "off a boundary":
            g.grad_pairwise = torch.empty(g.grad_pairwise.numel() + 1, device="cuda:0")[1:].view(g.grad_pairwise.shape)
        g.poison_outputs()
        g.forward()
        g.backward(want_V=variant != "no table gradient")
        out = g.results()
        np.testing.assert_array_equal(out.p, f.p)
        check_grad("grad_unary", out.grad_unary, b[np.float32].grad_unary, b[np.float64].grad_unary)
        if variant != "no table gradient":
            if algo == "isgmr" and variant != "least workspace":     # (which may hold no iteration: then the sweep adds to the tables)
                assert mrf.mrf_last_sweep_launch(True).startswith("mrf_bwd_sweep_narrow" if 2 * B * (H + W) > 1024 else "mrf_bwd_sweep_chain")
            check_grad("grad_pairwise_edge", out.grad_pairwise, b[np.float32].grad_pairwise_edge, b[np.float64].grad_pairwise_edge)


# (algo, B, H, W, L, directions, K, iterations whose node gradients the least workspace holds, whether a workgroup of the pass takes
# more than one turn): passes of two and one iterations onto what the first one left, groups that come out even and not; several
# turns in a pass that starts from nothing and in one that does not; 8 and 16 directions on the narrow sweep that stores
@pytest.mark.parametrize("case", [("isgmr", 1, 110, 140, 5, 4, 5, 2, False), ("trwp", 1, 110, 140, 5, 4, 4, 2, False),
                                  ("isgmr", 1, 41, 64, 32, 4, 1, 1, True), ("trwp", 1, 200, 222, 16, 4, 3, 2, True),
                                  ("isgmr", 1, 3, 190, 13, 8, 2, 2, False), ("trwp", 1, 2, 1030, 8, 8, 2, 2, False),
                                  ("isgmr", 1, 3, 150, 21, 16, 2, 2, False), ("trwp", 1, 2, 1030, 18, 16, 2, 2, True)],
                         ids=lambda c: "_".join(map(str, c[:7])))
def test_passes_over_the_gradient_of_per_edge_tables(oracle, case):
    import torch
    import paper_1910_10892_amd as mrf
    from gpu_harness import GpuProblem
    print("case table passes", case, flush=True)
    algo, B, H, W, L, R, K, slabs, turns = case
    dirs = {4: DIRS4, 8: DIRS8, 16: DIRS16}[R]
    pr = random_problem(830 + L, algo, B, H, W, L, dirs, K, per_edge=False, rho=np.linspace(0.3, 0.9, R))
    rng = np.random.default_rng(9400 + L)
    pr.pairwise_edge = rng.random((R, B, H, W, L, L), dtype=np.float32)
    f = oracle.forward(pr.algo, pr.unary, None, pr.dirs, pr.K, rho=pr.rho, pairwise_edge=pr.pairwise_edge)
    b = oracle.backward(pr.algo, pr.shape, None, pr.dirs, pr.K, pr.grad_cost.astype(np.float64), f.p, f.q, rho=pr.rho, dtype=np.float64,
                        per_edge_pairwise=True)
    for variant in ("as asked for", "least workspace"):
        g = GpuProblem(pr)
        if variant == "least workspace":
            plain = mrf.MrfProblem(g.unary, torch.zeros((L, L), device="cuda:0"), pr.dirs, K, rho=pr.rho)
            g.workspace = g.workspace[:mrf.mrf_workspace_bytes(plain, g.algo, True)]
            room = (g.workspace.numel() - mrf.mrf_workspace_bytes(plain, g.algo, False)) // (4 * R * B * H * W * L)
            assert min(room, K) == slabs
        unit = 1 if L % 2 == 0 else 4
        per_turn = max(8192 // (L * L) // unit * unit, unit)
        assert (R * B * H * W > 1280 * per_turn) == turns
        g.poison_outputs()
        g.forward()
        g.backward()
        if R > 4 and algo == "isgmr":                  # (TRWP: the directions across the grid, not the last one swept)
            assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_narrow", mrf.mrf_last_sweep_launch(True)
        out = g.results()
        np.testing.assert_array_equal(out.p, f.p)
        check_grad("grad_unary", out.grad_unary, None, b.grad_unary)
        check_grad("grad_pairwise_edge", out.grad_pairwise, None, b.grad_pairwise_edge)


# chain and narrow layout, TRWP (grad theta formed by one direction per iteration) and ISGMR on small grids (by the first one)
@pytest.mark.parametrize("case", [("trwp", 2, 9, 24, 13), ("trwp", 1, 20, 30, 45), ("isgmr", 2, 12, 14, 21), ("isgmr", 1, 12, 17, 64),
                                  ("trwp", 3, 4, 360, 21), ("isgmr", 1, 2, 530, 8)], ids=lambda c: "_".join(map(str, c)))
@pytest.mark.parametrize("want_V", [True, False])
def test_unary_gradient_of_per_edge_tables_is_rounded_once(oracle, case, want_V):
    """What arrives at theta is summed in double and rounded to float once per pass over it, in every layout: so the layouts
    agree in all bits but where two double sums of other orders, some 2^-50 apart, lie on two sides of a rounding boundary (of
    few floats with few bits between them an exact tie now and then), or cancel to what is left of them (below 2^-40 of the
    largest value, whose last place is 2^-24 of it).  What a scatter array rounds the other way reaches the entries of the scanlines
    through its node that went to the same label: some tens of the 5,616 or more here, one in a hundred at most.  Summed in two
    floats, 1.4 to 14 values in a hundred differ."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    print("case rounded once", case, want_V, flush=True)
    algo, B, H, W, L = case
    pr = random_problem(890 + L, algo, B, H, W, L, DIRS4, 3, per_edge=False, rho=np.linspace(0.3, 0.9, 4))
    pr.pairwise_edge = np.random.default_rng(9300 + L).random((4, B, H, W, L, L)).astype(np.float32)
    a = run_gpu(pr, want_V=want_V)
    assert mrf.mrf_last_sweep_kernel(True) != "mrf_bwd_sweep"
    try:
        assert mrf.mrf_tune(6, 1) == 0
        b = run_gpu(pr, want_V=want_V)
        assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep"
    finally:
        mrf.mrf_tune(6, 0)
    differ = np.count_nonzero(np.abs(a.grad_unary - b.grad_unary) > np.abs(b.grad_unary).max() * 2.0 ** -40)
    assert differ <= a.grad_unary.size // 100, (differ, a.grad_unary.size)


@pytest.mark.parametrize("algo", ["isgmr", "trwp"])
def test_per_edge_tables_of_33_labels_and_many_scanlines(oracle, algo):
    """More than 2,560 scanlines of 33..64 labels in a launch: the chain layout that stores the node gradients."""
    import paper_1910_10892_amd as mrf
    from gpu_harness import run_gpu
    B, H, W, L = (330, 2, 2, 33) if algo == "isgmr" else (1300, 2, 2, 33)
    print("case tables, many scanlines", algo, flush=True)
    pr = random_problem(895, algo, B, H, W, L, DIRS4, 2, per_edge=False, rho=np.linspace(0.3, 0.9, 4))
    pr.pairwise_edge = np.random.default_rng(9500).random((4, B, H, W, L, L), dtype=np.float32)
    f = oracle.forward(pr.algo, pr.unary, None, pr.dirs, pr.K, rho=pr.rho, pairwise_edge=pr.pairwise_edge)
    b = oracle.backward(pr.algo, pr.shape, None, pr.dirs, pr.K, pr.grad_cost.astype(np.float64), f.p, f.q, rho=pr.rho, dtype=np.float64,
                        per_edge_pairwise=True)
    g = run_gpu(pr)
    np.testing.assert_array_equal(g.p, f.p)
    assert mrf.mrf_last_sweep_kernel(True) == "mrf_bwd_sweep_chain", mrf.mrf_last_sweep_launch(True)
    check_grad("grad_unary", g.grad_unary, None, b.grad_unary)
    check_grad("grad_pairwise_edge", g.grad_pairwise, None, b.grad_pairwise_edge)


def test_per_edge_tables_argument_errors():
    import torch
    import paper_1910_10892_amd as mrf
    dev = torch.device("cuda:0")
    L = 70
    z = lambda *s: torch.zeros(s, dtype=torch.float32, device=dev)
    prob = mrf.MrfProblem(z(1, 2, 2, L), None, DIRS4, 1, pairwise_edge=z(4, 1, 2, 2, L, L))
    assert mrf.mrf_workspace_bytes(prob, mrf.MRF_ISGMR, False) == 0          # more than 64 labels
    L = 4
    prob = mrf.MrfProblem(z(1, 2, 2, L), None, DIRS4, 1, pairwise_edge=z(4, 1, 2, 2, L, L))
    ws = torch.empty(max(mrf.mrf_workspace_bytes(prob, mrf.MRF_ISGMR, True), 256), dtype=torch.uint8, device=dev)
    p = torch.zeros((1, 4, 1, 2, 2, L), dtype=torch.uint8, device=dev)
    q = torch.zeros((1, 4, 1, 2, 2), dtype=torch.uint8, device=dev)
    with pytest.raises(mrf.MrfError):      # there are no edge weights to differentiate
        mrf.mrf_isgmr_backward(prob, z(1, 2, 2, L), p, q, z(1, 2, 2, L), z(4, 1, 2, 2), None, ws)


@pytest.mark.parametrize("seed", range(30 + EXTRA_SEEDS))
def test_drawn_medium_problems_forced_layouts(oracle, seed):
    """Random problems whose scanlines are several times longer than the LDS rings of the
    taken-apart layouts (20..69 nodes), with the kernel-choice knobs drawn at random."""
    import paper_1910_10892_amd as mrf
    from mrf_inputs import truncated_linear, truncated_quadratic, sgm_penalties
    rng = np.random.default_rng(77000 + seed)
    algo = ("isgmr", "trwp")[int(rng.integers(0, 2))]
    B, H, W = int(rng.integers(1, 3)), int(rng.integers(20, 70)), int(rng.integers(20, 70))
    L = int(rng.choice([5, 16, 21, 32, 40, 64, 96, 130, 192, 256]))
    dirs = [DIRS4, DIRS8][int(rng.integers(0, 2))]
    K = int(rng.integers(1, 3))
    iv = bool(rng.integers(0, 2))
    pr = random_problem(88000 + seed, algo, B, H, W, L, dirs, K, integer_valued=iv, per_edge=bool(rng.integers(0, 2)),
                        rho=rng.uniform(0.2, 1.0, len(dirs)))
    kind = int(rng.integers(0, 4))
    if kind:
        scale = 1.0 if iv else 0.41
        if kind == 1:
            trunc = float(rng.choice([2.0, 3.0, 8.0, 11.0, 16.0]))
            pr.pairwise = truncated_linear(L, trunc, scale)
        elif kind == 2:
            trunc = float(rng.choice([4.0, 12.0, 30.0, 110.0, 200.0]))
            pr.pairwise = truncated_quadratic(L, trunc, scale)
        else:
            trunc = 2.0
            pr.pairwise = sgm_penalties(L, 0.5 if not iv else 1.0, 2.0)
        pr.pairwise_kind, pr.trunc, pr.scale = kind, trunc, scale
    want_V = bool(rng.integers(0, 2))
    knobs = {2: int(rng.integers(0, 3)), 3: int(rng.integers(0, 3)), 4: int(rng.integers(0, 3)),
             5: int(rng.integers(0, 3)), 6: int(rng.integers(0, 3)), 7: int(rng.choice([0, 2, 4, 6, 8, 12])),
             8: int(rng.integers(0, 3)), 9: int(rng.integers(0, 3)), 10: int(rng.choice([0, 4, 8])),
             11: int(rng.integers(0, 3)), 12: int(rng.integers(0, 3)), 13: int(rng.integers(0, 3)), 15: int(rng.integers(0, 3)), 16: int(rng.integers(0, 3)), 17: int(rng.integers(0, 3)), 18: int(rng.integers(0, 2)), 19: int(rng.integers(0, 2)), 20: int(rng.integers(0, 3))}
    print("case drawn medium", seed, algo, (B, H, W, L), len(dirs), K, kind, want_V, knobs, flush=True)
    f = oracle_forward(oracle, pr, threads=True)
    b = oracle_backward(oracle, pr, f.p, f.q, np.float64)
    big = max(float(np.abs(b.grad_unary).max()), float(np.abs(b.grad_pairwise).max()),
              float(np.abs(b.grad_edge_weight).max()) if b.grad_edge_weight is not None else 0.0)
    if big > 10.0:
        pr.grad_cost = (pr.grad_cost * np.float32(10.0 / big)).astype(np.float32)
    try:
        for k, v in knobs.items():
            assert mrf.mrf_tune(k, v) == 0
        full_check(oracle, pr, threads=True, want_V=want_V)
    finally:
        for k in knobs:
            mrf.mrf_tune(k, 0)
