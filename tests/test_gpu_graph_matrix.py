"""A batched solve after its matrix was destroyed and another took the handle's place: the
captured iterations are those of the new matrix's arrays."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import numpy as np  # noqa: E402

from paper_2606_24748_amd import blkamg as B  # noqa: E402
from tests.gpu_util import dev, q1_problem  # noqa: E402


def test_solve_with_another_matrix_at_the_same_handle():
    m, i, j, v, A = q1_problem(6, 2)
    rp, ci = dev(A.rowptr.astype(np.int32)), dev(A.colidx.astype(np.int32))
    vals = [dev(A.val), 4.0 * dev(A.val), 16.0 * dev(A.val)]  # all alive throughout

    def matrix(k):
        return B.bsr_create(A.nbr, A.nbc, 3, 3, rp, ci, vals[k])

    H0 = matrix(0)
    M = B.amg_setup(H0, m.coords, m.dirichlet)
    free = np.repeat(~m.dirichlet, 3)
    b = dev(np.random.default_rng(3).uniform(-1, 1, (m.n_dof, 8)) * free[:, None]).reshape(-1)
    x = torch.zeros_like(b)
    got, handles = [], []
    for k in range(3):
        H = matrix(k)
        handles.append(H.h.value)
        assert B.pcg_solve(H, M, b, x, rtol=1e-10, nrhs=8)[0] == B.OK
        got.append(x.clone())
        del H
    print("handles", handles, flush=True)
    # a scaled matrix scales CG's residuals not at all and its solutions by powers of two, exactly
    assert torch.equal(got[1] * 4.0, got[0]) and torch.equal(got[2] * 16.0, got[0])
