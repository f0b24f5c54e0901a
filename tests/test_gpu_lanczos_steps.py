"""The refresh's Lanczos and its Sturm counts from the fewest to the most steps, and where the
recurrence ends at once (D^-1 A the identity: every later norm is rounding, or zero) or after a
few steps (fewer distinct eigenvalues than steps)."""
import numpy as np
import pytest

import synth
from gpu_util import from_device_bsr, to_device_bsr
from oracle import sa
from oracle import sparse as S
from paper_2606_24748_amd import blkamg as B

pytestmark = pytest.mark.gpu


def matrix(kind, n=90):
    rng = np.random.default_rng(4)
    if kind == "spd":
        rp, ci, v = synth.random_spd_bsr(n, 3, seed=5, max_per_row=9)
        return S.Bsr(n, n, 3, 3, rp.astype(np.int64), ci.astype(np.int64), v)
    one = np.arange(n)
    if kind == "identity":
        return S.Bsr(n, n, 3, 3, np.arange(n + 1), one, 4.0 * np.tile(np.eye(3), (n, 1, 1)))
    if kind == "diagonal":
        q = rng.uniform(-1, 1, (n, 3, 3))
        return S.Bsr(n, n, 3, 3, np.arange(n + 1), one, q @ q.transpose(0, 2, 1) + np.eye(3))
    # pairs of rows [[I, c I], [c I, I]]: eigenvalues 1 - c and 1 + c, c = 0.5
    ci = np.stack([one - one % 2, one - one % 2 + 1], 1).reshape(-1)
    v = np.where((ci == np.repeat(one, 2))[:, None, None], np.eye(3), 0.5 * np.eye(3))
    return S.Bsr(n, n, 3, 3, 2 * np.arange(n + 1), ci, v)


@pytest.mark.parametrize("steps", [2, 3, 33, 64])
@pytest.mark.parametrize("kind,exact", [("spd", None), ("identity", 1.0), ("diagonal", 1.0), ("pairs", 1.5)])
def test_lambda(kind, exact, steps):
    A = matrix(kind)
    rng = np.random.default_rng(6)
    n = A.nbr
    P = S.Bsr(n, 3, 3, 6, np.arange(n + 1), np.arange(n) % 3, rng.uniform(-1, 1, (n, 3, 6)))
    HA, ka = to_device_bsr(A)
    HP, kp = to_device_bsr(P)
    HC = B.ptap_symbolic(HA, HP)
    B.ptap_numeric(HA, HP, HC)
    o = B.blkamg_opts_default()
    o.lanczos_steps = steps
    M = B.amg_hierarchy_create([HA, HC], [HP], o)
    got = float(np.asarray(M.lambdas()).reshape(-1)[0])
    # rounding moves a Ritz value by a few units of the norm's last place per step
    if exact is not None and (kind != "pairs" or steps > 2):
        assert abs(got - exact) <= 1e-12 * exact
    else:
        want, _, _ = sa.lanczos_lambda_max(A, S.block_diag_inverse(A), steps)
        assert abs(got - want) <= 1e-10 * want
