"""One-system CG: iteration limits against the oracle's recurrence, a breakdown with a V-cycle
queued ahead, and the next solve after either."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from oracle import solve  # noqa: E402
from paper_2606_24748_amd import blkamg as B  # noqa: E402
from tests.gpu_util import dev, q1_problem, rel2  # noqa: E402


# 3: one partial sum a product; 33: more than 2048 (39,304 rows, 16 rows a workgroup), summed in chunks
@pytest.mark.parametrize("n,maxits", [(3, (1, 2)), (33, (2, 3))])
def test_limits_breakdown_and_next_solve(n, maxits):
    m, i, j, v, A = q1_problem(n, 4)
    plan, HA = B.coo_plan_create(m.n_nodes, m.n_nodes, 3, 3, i, j)
    B.coo_assemble_blocked(plan, dev(v), B.INSERT, HA)
    M = B.amg_setup(HA, m.coords, m.dirichlet)
    H = solve.setup(A, m.coords, m.dirichlet)
    bh = synth.rhs(m, 6)
    b = dev(bh)
    x = torch.empty(m.n_dof, dtype=torch.float64, device="cuda")
    for maxit in maxits:
        xo, it_o, rel_o, ok_o = solve.pcg(A, bh, lambda q: solve.vcycle(H, q), rtol=1e-30, maxit=maxit)
        code, it, rel = B.pcg_solve(HA, M, b, x, rtol=1e-30, maxit=maxit)
        assert (code, it, ok_o) == (B.ENOCONV, it_o, False)
        # rounding of a few products and dots, grown by the V-cycle's condition
        # (192 dofs are solved directly: that residual is itself rounding, below 1e-12)
        assert abs(rel - rel_o) <= 1e-9 * rel_o or max(rel, rel_o) <= 1e-12
        assert rel2(x.cpu().numpy(), xo) <= 1e-9
    code, it, rel = B.pcg_solve(HA, M, b, x, rtol=1e-8)
    ref = x.cpu().numpy()
    assert code == B.OK and rel <= 1e-8
    B.coo_assemble_blocked(plan, dev(-v), B.INSERT, HA)  # p.Ap < 0 with the old hierarchy
    with pytest.raises(B.BlkAmgError) as e:
        B.pcg_solve(HA, M, b, x, rtol=1e-8)
    assert e.value.code == B.EBREAKDOWN
    B.coo_assemble_blocked(plan, dev(v), B.INSERT, HA)
    code2, it2, _ = B.pcg_solve(HA, M, b, x, rtol=1e-8)
    assert code2 == B.OK and it2 == it and np.array_equal(x.cpu().numpy(), ref)
