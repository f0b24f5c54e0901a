"""Galerkin symbolic phase where a row's candidates fill its hash set: all columns distinct, all
the same, one below, at and one beyond the longest row kept on the chip (4096 candidates)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import sparse as S  # noqa: E402
from paper_2606_24748_amd import blkamg as B  # noqa: E402
from tests.gpu_util import from_device_bsr, rel2, to_device_bsr  # noqa: E402


# rows of A x blocks of P per row; columns distinct or shared
@pytest.mark.parametrize("na,np_,shared", [(1, 1, False), (5, 13, False), (63, 65, False), (64, 64, False),
                                           (64, 64, True), (17, 241, False), (64, 65, False)])
def test_sets_at_their_limits(na, np_, shared):
    rng = np.random.default_rng(na * 1000 + np_)
    nrow = na + 2
    ncol = np_ if shared else na * np_
    # row 0 of A reaches rows 2.. of P; row 1 is empty; the others hold their diagonal
    a_cols = [np.arange(2, nrow)] + [np.empty(0, int)] + [np.array([i]) for i in range(2, nrow)]
    perm = rng.permutation(ncol)
    p_cols = [np.empty(0, int), np.empty(0, int)]
    p_cols += [np.arange(np_) if shared else np.sort(perm[i * np_:(i + 1) * np_]) for i in range(na)]

    def bsr(cols, nbc, br, bc):
        rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
        ci = np.concatenate(cols).astype(np.int32)
        return S.Bsr(len(cols), nbc, br, bc, rp, ci, rng.uniform(-1, 1, (len(ci), br, bc)))

    A, P = bsr(a_cols, nrow, 3, 3), bsr(p_cols, ncol, 3, 6)
    HA, k1 = to_device_bsr(A)
    HP, k2 = to_device_bsr(P)
    out = []
    for flags in (0, B.PTAP_HOST_SYMBOLIC):
        C = B.ptap_symbolic_ex(HA, HP, flags)
        B.ptap_numeric(HA, HP, C)
        torch.cuda.synchronize()
        out.append((from_device_bsr(C), B.ptap_plan_info(C)))
    (c, i0), (h, i1) = out
    assert i0 == i1
    assert np.array_equal(c.rowptr, h.rowptr) and np.array_equal(c.colidx, h.colidx)
    assert np.array_equal(c.val, h.val)
