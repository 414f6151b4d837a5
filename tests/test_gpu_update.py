"""Jacobi/DIIS updates against the oracle's: one to sixteen stored pairs, one to many blocks, dependent error vectors."""
import numpy as np
import pytest

from gen.synth_df import make_system, random_amplitudes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("o,v,size", [(1, 2, 2), (3, 10, 1), (3, 10, 16), (4, 17, 8), (9, 20, 16)])
def test_updates_with_dependent_vectors(o, v, size):
    """Twenty steps on given residuals, every seventh a repetition of the one before (two equal error vectors: the
    system is singular, the oldest pairs are dropped until one of them is gone).  The residuals are independent random
    vectors, so the accepted systems are conditioned like ten and the coefficients of order one: amplitudes of order
    one agree to some hundred rounding errors, bounded by 1e-12."""
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2501_10515_amd as P
    from oracle.solver import DIIS, denominators

    from .gpu_util import dev, host

    print(f"case o={o} v={v} diis_size={size}", flush=True)
    B, eps = make_system(o, v, 8, 3, sigma=0.1)
    t1, t2 = random_amplitudes(o, v, 4, 0.05, 0.05)
    ints = P.ascc_build_ints(dev(B), dev(eps), o)
    diis = P.ascc_diis_create(ints, size, 1)
    d1, d2 = denominators(eps, o)
    ref = DIIS(size)
    dt1, dt2 = dev(t1), dev(t2)
    stats = torch.empty(8, dtype=torch.float64, device="cuda")
    rng = np.random.default_rng(6)
    for it in range(20):
        if it % 7 != 6:
            r1, r2 = rng.normal(0, 0.01, (o, v)), rng.normal(0, 0.01, (o, o, v, v))
        P.ascc_update(ints, diis, dt1, dt2, dev(r1), dev(r2), dev(np.array([0.5 * it])), stats)
        s1, s2 = r1 / d1, r2 / d2
        t1, t2 = t1 + s1, t2 + s2
        dropped = False
        if it >= 1:
            ref.push(np.concatenate([t1.ravel(), t2.ravel()]), np.concatenate([s1.ravel(), s2.ravel()]))
            n = len(ref.vecs)
            x, _ = ref.extrapolate()
            dropped = len(ref.vecs) < n
            if x is not None:
                t1, t2 = x[: o * v].reshape(o, v), x[o * v:].reshape(o, o, v, v)
        torch.cuda.synchronize()
        st = host(stats)
        assert max(np.abs(host(dt1) - t1).max(), np.abs(host(dt2) - t2).max()) <= 1e-12, it
        assert int(st[4]) == len(ref.vecs) and bool(int(st[5]) & 2) == dropped and not int(st[5]) & 1, it
        assert st[3] == pytest.approx(np.sqrt((r1**2).sum() + (r2**2).sum()), rel=1e-13)
        assert st[2] == max(np.abs(r1).max(), np.abs(r2).max())
        assert st[6] == it and (it == 0 or st[1] == 0.5)
    diis.close()
    ints.close()
