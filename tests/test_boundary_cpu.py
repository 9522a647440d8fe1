"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every symbol
the header declares, rejects bad problems before touching the device, and its scanline
geometry (Appendix C) enumerates exactly the maximal in-grid chains."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

import paper_1910_10892_amd as mrf
from paper_1910_10892_amd.mrfmp import _CProblem

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "mrfmp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(mrf_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = mrf.load_library()
    names = declared_functions()
    assert {"mrf_isgmr_forward", "mrf_isgmr_backward", "mrf_trwp_forward", "mrf_trwp_backward",
            "mrf_workspace_bytes", "mrf_strerror"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n
    assert mrf.mrf_version().count(".") == 2


def _cprob(**kw):
    dirs = np.array(kw.pop("dirs", [(0, 1), (0, -1), (1, 0), (-1, 0)]), np.int32)
    rho = np.full(len(dirs), 0.5, np.float32)
    c = _CProblem()
    c.B, c.H, c.W, c.L, c.R, c.K = 1, 8, 8, 4, len(dirs), 2
    c.dirs = dirs.ctypes.data
    c.unary = 0x1000      # never dereferenced by the host checks
    c.pairwise = 0x1000
    c.edge_weight = None
    c.edge_weight_scalar = 1.0
    c.rho = rho.ctypes.data
    c.pairwise_kind = 0
    for k, v in kw.items():
        setattr(c, k, v)
    c._keep = (dirs, rho)
    return c


def test_validation_codes_without_gpu():
    lib = mrf.load_library()
    V = lambda c, algo=0: lib.mrf_validate(ctypes.byref(c), algo)
    assert V(_cprob()) == 0
    assert V(_cprob(), 1) == 0
    assert V(_cprob(), 7) == -8
    assert V(_cprob(L=0)) == -3 and V(_cprob(L=257)) == -3
    assert V(_cprob(L=256)) == 0
    assert V(_cprob(K=0)) == -4
    assert V(_cprob(H=0)) == -2
    assert V(_cprob(B=4096, H=1024, W=1024)) == -2
    assert V(_cprob(dirs=[(0, 0)])) == -5
    assert V(_cprob(dirs=[(0, 1), (0, 1)])) == -5
    assert V(_cprob(R=17)) == -5
    assert V(_cprob(unary=None)) == -1
    assert V(_cprob(pairwise=None)) == -1
    assert V(_cprob(rho=None), 1) == -1 and V(_cprob(rho=None), 0) == 0
    assert V(_cprob(rho=None, rho_edge=0x1000), 1) == 0      # per-edge coefficients stand in for rho[]
    assert V(_cprob(pairwise_kind=9)) == -7
    assert V(_cprob(pairwise_kind=1, trunc=0.0)) == -7
    # kinds 1 and 2 promise a non-decreasing function of the label distance: no negative scale
    assert V(_cprob(pairwise_kind=1, trunc=2.0, scale=-1.0)) == -7
    assert V(_cprob(pairwise_kind=2, trunc=2.0, scale=float("nan"))) == -7
    assert V(_cprob(pairwise_kind=1, trunc=2.0, scale=0.0)) == 0
    assert V(_cprob(pairwise_kind=3, trunc=2.0, scale=-1.0)) == 0     # kind 3 does not use scale
    # standard SGM: one pass of the ISGMR sweeps, no TRWP form, no per-edge tables
    assert V(_cprob(sgm_standard=1, K=1)) == 0
    assert V(_cprob(sgm_standard=1, K=2)) == -8
    assert V(_cprob(sgm_standard=1, K=1), 1) == -8
    assert lib.mrf_validate(None, 0) == -1
    for code in range(0, -12, -1):
        assert mrf.mrf_strerror(code) != "unknown status"


def test_forward_kernel_choice_is_host_arithmetic():
    """Truncation distance -> window width (0 = dense sweep); no GPU involved."""
    lib = mrf.load_library()
    W = lambda **kw: lib.mrf_forward_window(ctypes.byref(_cprob(**kw)), 0)
    assert W(L=16, pairwise_kind=1, trunc=4.0) == 4
    assert W(L=16, pairwise_kind=1, trunc=3.0) == 4 and W(L=16, pairwise_kind=1, trunc=4.5) == 8
    assert W(L=96, pairwise_kind=1, trunc=8.0) == 8
    assert W(L=192, pairwise_kind=1, trunc=2.0) == 2
    assert W(L=256, pairwise_kind=2, trunc=200.0) == 16      # ceil(sqrt(200)) = 15
    assert W(L=256, pairwise_kind=2, trunc=100.0) == 12 and W(L=64, pairwise_kind=1, trunc=9.0) == 12
    assert W(L=21, pairwise_kind=0) == 0
    assert W(L=12, pairwise_kind=1, trunc=20.0) == 0          # never truncates inside the label range
    assert W(L=200, pairwise_kind=1, trunc=40.0) == 0         # window wider than the kernel supports
    assert W(L=64, pairwise_kind=3, trunc=2.0) == 2           # SGM penalties: constant from distance 2
    assert W(L=64, pairwise_kind=3, trunc=5.0) == 8
    assert W(L=64, pairwise_kind=4, trunc=2.0) == -7          # unknown kind
    assert W(L=0, pairwise_kind=1, trunc=4.0) == -3
    # any direction set: TRWP sweeps take up to fifteen message arrays, ISGMR sweeps read one array from six
    # directions on
    d8 = [(0, 1), (0, -1), (1, 0), (-1, 0), (1, 1), (-1, -1), (1, -1), (-1, 1)]
    d16 = d8 + [(1, 2), (-1, -2), (2, 1), (-2, -1), (1, -2), (-1, 2), (2, -1), (-2, 1)]
    T = lambda dirs, algo: lib.mrf_forward_window(ctypes.byref(_cprob(dirs=dirs, L=96, pairwise_kind=1, trunc=8.0)), algo)
    assert T(d8, 0) == 8 and T(d8, 1) == 8
    assert T(d8 + [(1, 2)], 0) == 8 and T(d8 + [(1, 2)], 1) == 8
    assert T(d16, 0) == 8 and T(d16, 1) == 8


def test_entry_points_reject_before_any_gpu_work():
    """NULL outputs / short workspaces are reported before a kernel launch is attempted, so
    this runs on a machine without a GPU."""
    lib = mrf.load_library()
    c = _cprob()
    need = lib.mrf_workspace_bytes(ctypes.byref(c), 0, 0)
    assert need >= 2 * 4 * 64 * 4 * 4
    bad = _cprob(L=0)
    assert lib.mrf_workspace_bytes(ctypes.byref(bad), 0, 0) == 0
    fake = ctypes.c_void_p(0x1000)
    for algo, name in ((0, "mrf_isgmr_forward"), (1, "mrf_trwp_forward")):
        f = getattr(lib, name)
        need = lib.mrf_workspace_bytes(ctypes.byref(c), algo, 0)
        assert f(ctypes.byref(c), None, None, fake, fake, None, fake, need, None) == -1
        assert f(ctypes.byref(c), fake, None, fake, fake, None, fake, need - 1, None) == -6
        assert f(ctypes.byref(c), fake, None, fake, fake, None, None, 0, None) == -1
        assert f(ctypes.byref(bad), fake, None, fake, fake, None, fake, need, None) == -3
    for algo, name in ((0, "mrf_isgmr_backward"), (1, "mrf_trwp_backward")):
        f = getattr(lib, name)
        needb = lib.mrf_workspace_bytes(ctypes.byref(c), algo, 1)
        assert f(ctypes.byref(c), None, fake, fake, fake, None, None, fake, needb, None) == -1
        assert f(ctypes.byref(c), fake, fake, fake, fake, None, None, fake, needb - 1, None) == -6


def test_room_for_node_gradients_only_where_a_launch_stores_them():
    """33..128 labels: one direction per launch (TRWP, or a single direction) and few enough scanlines in it."""
    lib = mrf.load_library()

    def room(algo, L, H=64, W=64, **kw):
        c = _cprob(L=L, H=H, W=W, **kw)
        fixed = lib.mrf_workspace_bytes(ctypes.byref(c), algo, 0)
        slots = (16384 if L <= 32 else 1024) * L * L * 8
        return lib.mrf_workspace_bytes(ctypes.byref(c), algo, 1) - fixed - (slots + 255) // 256 * 256

    for L, algo, kw, want in ((64, 1, {}, True), (128, 1, {}, True), (32, 1, {}, False), (129, 1, {}, False), (64, 0, {}, False),
                              (96, 0, {}, False), (64, 0, {"dirs": [(0, 1)]}, True), (64, 1, {"H": 1536, "W": 1536}, True),
                              (64, 1, {"H": 1537, "W": 1537}, False), (64, 1, {"H": 1537, "W": 8}, True)):
        nodes = kw.get("H", 64) * kw.get("W", 64)
        assert room(algo, L, **kw) == (8 * nodes * L if want else 0), (L, algo, kw)


def test_workspace_fault_query_rejects_null():
    lib = mrf.load_library()
    assert lib.mrf_workspace_fault(None, None) == -1
    assert "wait" in mrf.mrf_strerror(-11)
    assert mrf.mrf_tune(14, 5) == 0 and mrf.mrf_tune(14, 0) == 0


def test_every_documented_knob_is_known_and_others_are_refused():
    """mrf_tune: knobs 0..20 as the header lists them; an unknown knob is an error, not a silent no-op."""
    for knob in range(21):
        assert mrf.mrf_tune(knob, 0) == 0, knob
    assert mrf.mrf_tune(21, 0) != 0 and mrf.mrf_tune(-1, 0) != 0
    header = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "mrfmp.h")).read()
    for knob in range(21):
        assert "knob %d:" % knob in header, knob


def test_noalloc_energy_rejects_what_its_scratch_cannot_hold():
    """mrf_energy_noalloc: a batch beyond its fixed device array is an error before any GPU call."""
    lib = mrf.load_library()
    fake = ctypes.c_void_p(0x1000)
    f = lib.mrf_energy_noalloc
    f.restype = ctypes.c_int
    assert f(ctypes.byref(_cprob(B=65)), fake, fake, None) == -10
    assert f(ctypes.byref(_cprob(B=64)), None, fake, None) == -1
    assert f(ctypes.byref(_cprob(L=0)), fake, fake, None) == -3
    assert "scratch" in mrf.mrf_strerror(-10)


@pytest.mark.parametrize("H,W", [(1, 1), (1, 7), (6, 1), (5, 9), (9, 5), (4, 4)])
def test_scanline_geometry_matches_definition(H, W):
    for dh in range(-3, 4):
        for dw in range(-3, 4):
            if dh == 0 and dw == 0:
                continue
            heads = {(y, x) for y in range(H) for x in range(W)
                     if not (0 <= y - dh < H and 0 <= x - dw < W)}
            n = mrf.mrf_scanline_count(H, W, dh, dw)
            assert n == len(heads)
            seen = set()
            covered = 0
            for t in range(n):
                y0, x0, ln = mrf.mrf_scanline_head(H, W, dh, dw, t)
                assert (y0, x0) in heads and (y0, x0) not in seen
                seen.add((y0, x0))
                y, x, k = y0, x0, 0
                while 0 <= y < H and 0 <= x < W:
                    y += dh; x += dw; k += 1
                assert ln == k
                covered += ln
            assert covered == H * W     # each node lies on exactly one scanline
            if abs(dh) == 1 and abs(dw) <= W:
                assert n == W + (H - 1) * abs(dw)      # Eq. supp-wide


def test_scanline_geometry_errors():
    assert mrf.mrf_scanline_count(0, 4, 0, 1) == -2
    assert mrf.mrf_scanline_count(4, 4, 0, 0) == -5
    with pytest.raises(mrf.MrfError):
        mrf.mrf_scanline_head(4, 4, 0, 1, 4)


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures one GPU: any other --gpus ends with a message and a non-zero status before
    anything touches a device."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert res.returncode != 0
    assert "one GPU" in res.stderr and res.stdout.strip() == ""


@pytest.fixture(scope="module")
def scanline_order(tmp_path_factory):
    """mrf_geom_order of the kernels' header as a host function: image and scanline of every place of a direction's launch."""
    d = tmp_path_factory.mktemp("order")
    src, so = d / "order.cpp", d / "order.so"
    src.write_text('#include "mrfmp_device.h"\n'
                   'extern "C" void order(int H, int W, int dh, int dw, unsigned count, unsigned images, int *b, unsigned *t) {\n'
                   '  for (unsigned k = 0; k < count * images; ++k) mrf_geom_order(H, W, dh, dw, count, images, k, b[k], t[k]);\n}\n')
    csrc = os.path.join(ROOT, "paper_1910_10892_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + csrc, str(src), "-o", str(so)],
                   check=True)
    lib = ctypes.CDLL(str(so))

    def order(H, W, dh, dw, images):
        n = mrf.mrf_scanline_count(H, W, dh, dw) * images
        b, t = np.empty(n, np.int32), np.empty(n, np.uint32)
        lib.order(H, W, dh, dw, ctypes.c_uint(n // images), ctypes.c_uint(images), b.ctypes.data_as(ctypes.c_void_p), t.ctypes.data_as(ctypes.c_void_p))
        return b, t

    return order


@pytest.mark.parametrize("images", [1, 2, 3, 17, 64, 257])
def test_a_launch_takes_every_scanline_once_and_those_of_a_diagonal_by_falling_length(scanline_order, images):
    """Whatever run of 256 a scanline falls into; every second run is turned round.  Directions that are no diagonal with a step of
    one come image by image in the order of the geometry."""
    for H, W in [(1, 1), (1, 2), (2, 1), (1, 9), (9, 1), (2, 2), (3, 7), (7, 3), (8, 8), (13, 40), (40, 13), (5, 300), (130, 127)]:
        for dh, dw in [(1, 1), (1, -1), (-1, 1), (-1, -1), (0, 1), (-1, 0), (1, 2), (-2, 1), (2, 2)]:
            if images > 17 and H * W > 100:
                continue
            count = mrf.mrf_scanline_count(H, W, dh, dw)
            b, t = scanline_order(H, W, dh, dw, images)
            place = b.astype(np.int64) * count + t
            np.testing.assert_array_equal(np.sort(place), np.arange(count * images), err_msg=str((H, W, dh, dw)))
            if abs(dh) != 1 or abs(dw) != 1:
                np.testing.assert_array_equal(place, np.arange(count * images))
                continue
            lengths = np.array([mrf.mrf_scanline_head(H, W, dh, dw, int(k))[2] for k in range(count)])[t]
            for first in range(256, len(lengths), 512):
                lengths[first:first + 256] = lengths[first:first + 256][::-1].copy()
            assert (np.diff(lengths) <= 0).all(), (H, W, dh, dw)
