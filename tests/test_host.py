"""Host-side checks of the C-ABI library (no GPU needed)."""
import ctypes
import re
import subprocess
import sys
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]
HEADER = ROOT / "include" / "ascc.h"
LIB = ROOT / "paper_2501_10515_amd" / "libascc.so"


def declared_functions():
    text = HEADER.read_text()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ascc_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_function():
    assert LIB.exists(), "build first: python -m paper_2501_10515_amd.build"
    lib = ctypes.CDLL(str(LIB))
    names = declared_functions()
    assert "ascc_residual" in names and "ascc_build_ints" in names and "ascc_solve" in names
    assert "ascc_update" in names
    for name in names:
        assert hasattr(lib, name), name


def test_binding_covers_the_abi():
    import paper_2501_10515_amd as P

    for name in declared_functions():
        if name in ("ascc_ints_free", "ascc_diis_free", "ascc_ints_shape"):
            continue  # owned by the Ints / Diis wrappers
        if name.startswith("ascc_server_"):
            method = {"create": "__init__", "free": "close", "submit_state": "submit"}.get(
                name[len("ascc_server_"):], name[len("ascc_server_"):])
            assert hasattr(P.Server, method), name
            continue
        assert hasattr(P, name), name


def test_argument_errors_are_reported_not_thrown():
    import paper_2501_10515_amd as P

    with pytest.raises(P.AsccError) as e:
        P.ascc_workspace_bytes(0, 5, 5)
    assert e.value.code == P.ASCC_E_SHAPE
    with pytest.raises(P.AsccError) as e:
        P.ascc_workspace_bytes(2, 5, 5, diis_size=0)
    assert e.value.code == P.ASCC_E_ARG
    lib = P.load_library()
    h = ctypes.c_void_p()
    rc = lib.ascc_build_ints(None, None, 1, 2, 3, 4, 0, 0, None, ctypes.byref(h))
    assert rc == P.ASCC_E_ARG and "device pointers" in P.ascc_last_error()
    assert lib.ascc_residual(None, None, None, None, None, None, None) == P.ASCC_E_ARG
    # the 1-CSF entries reject a hole that is not occupied or a particle that is not virtual
    for hole, particle in [(-1, 3), (2, 3), (0, 1), (0, 5)]:  # no = 2, nv = 3
        h = ctypes.c_void_p(1)
        rc = lib.ascc_build_ints_hbar(None, None, 1, 2, 3, 4, 0, 0, hole, particle, 1, None, ctypes.byref(h))
        assert rc == P.ASCC_E_ARG and "orbital index" in P.ascc_last_error() and not h.value
    rc = lib.ascc_build_ints_hbar(None, None, 1, 2, 3, 4, 0, 0, 1, 2, 1, None, ctypes.byref(h))
    assert rc == P.ASCC_E_ARG and "device pointers" in P.ascc_last_error()
    rc = lib.ascc_build_ints_hbar(None, None, 1, 2, 3, 4, 0, 0, 1, 2, 0, None, ctypes.byref(h))
    assert rc == P.ASCC_E_ARG and "s_sign" in P.ascc_last_error()
    opts = P._lib.Opts(1e-8, 0, 0, 10, 8, 1, 0.0, 0.0, 0)
    res = P._lib.TwoAnsatzResult()
    two = (ctypes.c_void_p * 2)(1, 1)
    rc = lib.ascc_two_ansatz(None, None, 1, 2, 3, 4, 0, 0, 1, 2, 1.0, ctypes.byref(opts), two, two, ctypes.byref(res),
                             None)
    assert rc == P.ASCC_E_ARG and "alpha" in P.ascc_last_error()
    assert lib.ascc_initial_guess(None, None, 2, 3, 0, 2, 1.0, -0.5, None) == P.ASCC_E_ARG


def test_workspace_bytes_scale_with_the_shape():
    import paper_2501_10515_amd as P

    a, d = P.ascc_workspace_bytes(20, 180, 600)
    v = 180
    assert a > 8 * v ** 4  # the full (ac|bd) matrix is part of the integral set
    assert d >= 2 * 8 * 8 * (20 * v + 400 * v * v)


@pytest.mark.parametrize("shapes", [["1,1,1,1", "2,3,8,1", "3,5,12,0", "5,20,60,1", "7,45,37,0"],
                                    ["1,1,1,1,1", "2,3,8,1,1", "3,5,12,0,1", "5,20,60,1,1", "7,45,37,0,1"],
                                    ["20,180,600,1", "40,360,1200,1,1", "30,270,900,0,1", "20,180,600,1,1"],
                                    ["2,3,8,1,0,1", "5,20,60,1,1,2", "7,45,37,0,0,2", "20,180,600,1,1,2",
                                     "40,360,1200,1,1,1"]])
def test_every_launch_stays_in_bounds_dry_run(shapes):
    """The full build / residual / update / solve launch sequence, bounds-checked without a GPU."""
    r = subprocess.run([sys.executable, str(ROOT / "tests" / "dry_run_driver.py"), *shapes], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.count("OK ") == len(shapes)


def _one_of_each(o, v, Q, prec, mode):
    """Bytes of one array of each kind that an integral set works with, without padding."""
    import paper_2501_10515_amd as P

    n, ov, oo, vv = o + v, o * v, o * o, v * v
    To, Tv, packed = o * (o + 1) // 2, v * (v + 1) // 2, mode == P.ASCC_VVVV_PACKED
    factors = Q * (n * n + 4 * ov) + Q * (n * n + n * o + oo + vv)      # B, B_ov, N; what T1 dressing forms
    blocks = (2 * Tv * Tv if packed else vv * vv) + vv * (ov + oo)      # (ac|bd); (kc|bd), (kc|ld)
    ladder = 4 * To * Tv                                                # pair rows of the amplitudes and of the ladder
    doubles = 16 * ov * ov + 2 * oo * oo + oo * (ov + oo)               # rings, assembly; hole-hole ladder; W, Z
    chunk = -(-v // 16) if packed else min(v, max(1, 2**28 // v**3))
    words = factors + blocks + ladder + doubles + 2**23 + max(o, chunk) * v**3
    if prec != P.ASCC_PREC_FP64:  # shadows, four bytes a value
        words += (2 * Tv * Tv + vv * (ov + oo) + 2 * To * Tv + 7 * ov * ov + Q * (3 * ov + oo + vv) + oo * vv + oo * oo) / 2
    return 8 * words


@pytest.mark.parametrize("prec", ["fp64", "bf16x3"])
@pytest.mark.parametrize("o,v,Q", [(4, 36, 120), (5, 20, 60), (8, 72, 240), (12, 108, 360)])
def test_small_packed_sets_take_no_more_than_their_arrays(o, v, Q, prec):
    """A served request is admitted by this size; whole-line rows and alignment are within 1 %."""
    import paper_2501_10515_amd as P

    pc = {"fp64": P.ASCC_PREC_FP64, "bf16x3": P.ASCC_PREC_BF16X3}[prec]
    got = P.ascc_workspace_bytes(o, v, Q, pc, P.ASCC_VVVV_PACKED)[0]
    assert got <= 1.01 * _one_of_each(o, v, Q, pc, P.ASCC_VVVV_PACKED)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("mode", ["full", "packed"])
@pytest.mark.parametrize("o,v,Q", [(30, 15, 120), (60, 30, 270), (100, 10, 300), (256, 4, 700), (256, 100, 1000),
                                   (20, 20, 120), (20, 180, 600)])
def test_sets_with_many_occupied_orbitals_take_no_more_than_their_arrays(o, v, Q, mode, prec):
    """The W/Z pair rows are the largest array of such a set besides the o^4 ones."""
    import paper_2501_10515_amd as P

    pc = {"fp64": P.ASCC_PREC_FP64, "fp32": P.ASCC_PREC_FP32}[prec]
    vm = P.ASCC_VVVV_FULL if mode == "full" else P.ASCC_VVVV_PACKED
    got = P.ascc_workspace_bytes(o, v, Q, pc, vm)[0]
    assert got <= 1.001 * _one_of_each(o, v, Q, pc, vm)


@pytest.mark.parametrize("mode", ["full", "packed"])
@pytest.mark.parametrize("o,v,Q", [(40, 40, 240), (60, 30, 270), (100, 10, 300), (256, 100, 1000), (13, 117, 390), (20, 180, 600)])
def test_a_stacked_state_takes_no_more_than_its_pair_rows_and_ladder(o, v, Q, mode):
    """A batch holds for every state the pair rows of its amplitudes and of its ladder (whole lines of 16 values) and no
    more than another [o][o][v][v]: not the W/Z columns of states with many occupied orbitals, of more than 32 MB."""
    import paper_2501_10515_amd as P

    vm = P.ASCC_VVVV_FULL if mode == "full" else P.ASCC_VVVV_PACKED
    To, ldT, S = o * (o + 1) // 2, -(-v * (v + 1) // 32) * 16, 8
    got = P.ascc_batch_workspace_bytes(o, v, Q, S, 1, vvvv_mode=vm)
    assert got <= S * 8 * (4 * To * ldT + (o * v) ** 2) + 1024


def test_step_summary_of_a_small_set():
    """The ladder and the rings of a small set share a launch with other products: their phases have no intervals."""
    import bench

    run = {"ms_step": 0.2, "steps": 10, "phases": {"dress": (0.3, 10), "df_ints": (0.5, 10), "ring_xz": (0.1, 10)}}
    out = bench.step_summary(run, 1.3e7, 5, 20, "fp64")
    assert out["ms_per_step"] == 0.2 and not [k for k in out if k.startswith(("pp_ladder", "ring_"))]


@pytest.mark.parametrize("prec", ["fp64", "bf16x3"])
def test_ladder_rate_counts_what_its_phase_holds(prec):
    """In FP64 the W/Z rows, [T(o)] x [ov + o^2] sums over T(v) pairs in two halves, are products of the ladder's phase."""
    import bench

    o, v, ms = 20, 180, 4.0
    run = {"ms_step": 12.0, "steps": 1, "phases": {"pp_ladder": (ms, 1)}}
    out = bench.step_summary(run, 1e12, o, v, prec)
    To, Tv = o * (o + 1) // 2, v * (v + 1) // 2
    flops = 2 * (To * Tv**2 + (To - o) * (Tv - v) ** 2)
    if prec == "fp64":
        flops += 2 * 2 * To * Tv * (o * v + o * o)
    assert out["pp_ladder_tflops"] == pytest.approx(flops / (ms * 1e-3) / 1e12, abs=1e-3)
