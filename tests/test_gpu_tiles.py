"""Residuals at sizes around the edges of the contractions' tiles, slices and padded rows, alone and batched."""
import numpy as np
import pytest

from gen.synth_df import make_system, random_amplitudes

pytestmark = pytest.mark.gpu

# FP64: a residual element is a sum of at most about 5000 products of the integrals and amplitudes, each product chain
# rounded a few times: 5000 u = 6e-13 of the largest term, which is no larger than max|R| times five here.
# FP32 and split-BF16x3: as in test_gpu_lowp.py.
REL = {"fp64": 3e-12, "fp32": 2e-6, "bf16x3": 4e-5}


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("mode", ["full", "packed"])
@pytest.mark.parametrize("o,v,Q", [
    (1, 2, 3),     # one pair, rows shorter than a padded line
    (2, 8, 16),    # ov = one stage of K
    (4, 16, 32),   # ov = 64: whole tiles
    (5, 13, 17),   # ov = 65: one row past a tile; T(v) odd
    (8, 12, 33),   # ov = 96, o^2 = 64
    (9, 11, 40),   # ov = 99, T(v) = 66
    (13, 15, 48),  # ov = 195: one 192-row tile and three rows
    (16, 17, 64),  # o^2 = 256, T(o) = 136
    (34, 6, 20),   # three tiles of occupied rows in the dressing
    (52, 4, 24),   # two passes of them
    (66, 3, 81),   # two chunks of fitting indices, the second almost empty
])
def test_tile_edges(o, v, Q, mode, prec):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2501_10515_amd as P
    from oracle import cs_ccsd

    from .gpu_util import dev, gpu_residual, host

    S = 3
    print(f"case o={o} v={v} Q={Q} vvvv={mode} prec={prec}", flush=True)
    B, eps = make_system(o, v, Q, 17, sigma=0.1)
    amps = [random_amplitudes(o, v, 500 + k, 0.05, 0.05) for k in range(S)]
    pc = {"fp64": P.ASCC_PREC_FP64, "fp32": P.ASCC_PREC_FP32, "bf16x3": P.ASCC_PREC_BF16X3}[prec]
    vm = P.ASCC_VVVV_FULL if mode == "full" else P.ASCC_VVVV_PACKED
    ints = P.ascc_build_ints(dev(B), dev(eps), o, precision=pc, vvvv_mode=vm)
    alone = [gpu_residual(P, ints, *a) for a in amps]
    r1, r2 = cs_ccsd.residual(B, np.diag(eps), *amps[0])
    scale = max(np.abs(r1).max(), np.abs(r2).max())
    err = max(np.abs(alone[0][0] - r1).max(), np.abs(alone[0][1] - r2).max())
    print(f"  max|dR| = {err:.3e}  (max|R| = {scale:.3e})", flush=True)
    assert err <= REL[prec] * scale
    # the tiles of a batch are chosen for all its states; its bits are those of each state alone
    P.ascc_batch_reserve(ints, S)
    t1, t2 = [dev(a[0]) for a in amps], [dev(a[1]) for a in amps]
    b1, b2 = [torch.empty_like(t) for t in t1], [torch.empty_like(t) for t in t2]
    e = torch.empty(S, dtype=torch.float64, device="cuda")
    P.ascc_residual_batch(ints, t1, t2, b1, b2, e)
    torch.cuda.synchronize()
    ints.close()
    for k in range(S):
        assert np.array_equal(host(b1[k]), alone[k][0]) and np.array_equal(host(b2[k]), alone[k][1])
        assert float(host(e)[k]) == alone[k][2]


def _grouped_equals_alone(o, v, Q, S, G, prec, mode):
    """Residuals of S states in passes of G, from a workspace of the reported size, against each state alone: the same
    bits."""
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2501_10515_amd as P

    from .gpu_util import dev, gpu_residual, host

    print(f"case o={o} v={v} Q={Q} S={S} G={G} vvvv={mode} prec={prec}", flush=True)
    B, eps = make_system(o, v, Q, 19, sigma=0.1)
    amps = [random_amplitudes(o, v, 600 + k, 0.05, 0.05) for k in range(S)]
    pc = {"fp64": P.ASCC_PREC_FP64, "fp32": P.ASCC_PREC_FP32, "bf16x3": P.ASCC_PREC_BF16X3}[prec]
    vm = P.ASCC_VVVV_FULL if mode == "full" else P.ASCC_VVVV_PACKED
    ints = P.ascc_build_ints(dev(B), dev(eps), o, precision=pc, vvvv_mode=vm)
    nbytes = P.ascc_batch_workspace_bytes(o, v, Q, S, G, precision=pc, vvvv_mode=vm)
    ws = torch.full((nbytes // 8,), float("nan"), dtype=torch.float64, device="cuda")
    P.ascc_batch_reserve_ws(ints, S, G, ws)
    T1, T2 = dev(np.stack([a[0] for a in amps])), dev(np.stack([a[1] for a in amps]))
    R1, R2 = torch.empty_like(T1), torch.empty_like(T2)
    e = torch.empty(S, dtype=torch.float64, device="cuda")
    P.ascc_residual_batch(ints, list(T1), list(T2), list(R1), list(R2), e)
    torch.cuda.synchronize()
    R1, R2, e = host(R1), host(R2), host(e)
    for k in range(S):
        r1, r2, ek = gpu_residual(P, ints, *amps[k])
        assert np.array_equal(R1[k], r1) and np.array_equal(R2[k], r2) and e[k] == ek, f"state {k}"
    ints.close()


@pytest.mark.parametrize("o,v,Q,S,G,prec", [
    # low precision: W/Z in 15 slices, whose partial tiles the scratch holds for 5 states
    (10, 90, 300, 8, 8, "fp32"), (10, 90, 300, 8, 8, "bf16x3"),
    # ... rings in 2 slices, W/Z in 22: partial tiles of one state
    (12, 108, 360, 4, 4, "fp32"), (12, 108, 360, 4, 4, "bf16x3"),
    # hole-hole ladder (300 x 1176 x 300, the pairs as rows of t+-) in 2 slices: partial tiles of 5 states
    (24, 48, 60, 7, 7, "fp64"),
])
def test_slices_do_not_depend_on_the_batch(o, v, Q, S, G, prec):
    _grouped_equals_alone(o, v, Q, S, G, prec, "packed")


EDGES = [(1, 2, 3), (2, 8, 16), (4, 16, 32), (5, 13, 17), (8, 12, 33), (9, 11, 40), (13, 15, 48), (16, 17, 64),
         (34, 6, 20), (52, 4, 24), (66, 3, 81)]  # as in test_tile_edges


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("mode", ["full", "packed"])
@pytest.mark.parametrize("o,v,Q", EDGES)
def test_tile_edges_in_groups(o, v, Q, mode, prec):
    """Every term in passes of three states, the last one of two: launches over operand blocks at these sizes."""
    _grouped_equals_alone(o, v, Q, 5, 3, prec, mode)


@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("o,v,stacks", [
    # the narrow orders (fewer than 128 tiles of 256 x 256): 64 x 64 tiles alone, then 128 x 64, 128 x 128 and 256 x 128
    # ones (split-BF16x3), 64 x 64 with three stages instead of four and 128 x 64 (FP32)
    (12, 60, (4, 8, 12, 16)),
    # the wide orders: 64 x 128, 192 x 256, 256 x 256 and 256 x 128; FP32 64 x 64, 224 x 192, 256 x 256 and 128 x 256
    (24, 126, (2, 3, 4, 8)),
])
def test_every_tile_of_an_order_gives_the_same_bits(o, v, stacks, prec):
    """The ladders of several stacked states take the tiles that fit all their rows, in the order of one state: residuals
    of the first state at the front of growing stacks, and of the last one at their end, against those alone."""
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2501_10515_amd as P

    from .gpu_util import dev

    print(f"case o={o} v={v} states={stacks} prec={prec}", flush=True)
    B, eps = make_system(o, v, 40, 23, sigma=0.1)
    pc = {"fp32": P.ASCC_PREC_FP32, "bf16x3": P.ASCC_PREC_BF16X3}[prec]
    ints = P.ascc_build_ints(dev(B), dev(eps), o, precision=pc, vvvv_mode=P.ASCC_VVVV_PACKED)
    S = max(stacks)
    P.ascc_batch_reserve(ints, S)
    g = torch.Generator(device="cuda").manual_seed(29)
    T1 = 0.05 * torch.randn((S, o, v), dtype=torch.float64, device="cuda", generator=g)
    T2 = 0.05 * torch.randn((S, o, o, v, v), dtype=torch.float64, device="cuda", generator=g)
    T2 = 0.5 * (T2 + T2.permute(0, 2, 1, 4, 3))
    r1, r2 = torch.empty_like(T1), torch.empty_like(T2)
    e = torch.empty(S, dtype=torch.float64, device="cuda")
    for k in {0} | {n - 1 for n in stacks}:
        P.ascc_residual(ints, T1[k], T2[k], r1[k], r2[k], e[k:k + 1])
    R1, R2, E = torch.empty_like(T1), torch.empty_like(T2), torch.empty_like(e)
    for n in stacks:
        P.ascc_residual_batch(ints, list(T1[:n]), list(T2[:n]), list(R1[:n]), list(R2[:n]), E[:n])
        torch.cuda.synchronize()
        for k in (0, n - 1):
            assert torch.equal(R1[k], r1[k]) and torch.equal(R2[k], r2[k]) and E[k] == e[k], (n, k)
    assert float(r2[0].abs().max()) > 1e-2
    ints.close()


@pytest.mark.parametrize("mode", ["full", "packed"])
@pytest.mark.parametrize("o,v,Q", [(40, 39, 60), (64, 9, 30)])  # T(v) = 780: K in slices; T(v) = 45, odd
def test_stacked_states_without_their_wz_columns(o, v, Q, mode):
    """W/Z columns of more than 32 MB: products of their own, with each state and in groups (the last one of one state)."""
    _grouped_equals_alone(o, v, Q, 3, 2, "fp64", mode)
    _grouped_equals_alone(o, v, Q, 2, 1, "fp64", mode)
