"""Destroying a handle that owns device memory waits for the device, so a caller may free the
arrays that the handle borrowed; a handle that owns none returns at once."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_24748_amd import blkamg as B  # noqa: E402
from tests.gpu_util import dev, q1_problem  # noqa: E402


@pytest.mark.parametrize("kind", ["bsr", "coo_plan", "fe_plan", "borrowed"])
def test_destroy_waits(kind):
    m, i, j, v, A = q1_problem(3, 1)
    alive = B.coo_plan_create(m.n_nodes, m.n_nodes, 3, 3, i, j)  # the library's memory is kept meanwhile
    rp, ci = dev(A.rowptr.astype("int32")), dev(A.colidx.astype("int32"))
    val = dev(A.val)
    if kind == "bsr":
        h = B.bsr_create(A.nbr, A.nbc, 3, 3, rp, ci, val)
        y = torch.zeros(m.n_dof, dtype=torch.float64, device="cuda")
        B.bsr_spmv_t(h, 1.0, torch.ones_like(y), 0.0, y)  # makes the transposed copy
    elif kind == "borrowed":
        h = B.bsr_create(A.nbr, A.nbc, 3, 3, rp, ci, val)
    elif kind == "coo_plan":
        h, _ = B.coo_plan_create(m.n_nodes, m.n_nodes, 3, 3, i, j)
        del _
    else:
        h = B.fe_ebe_plan_create(alive[1], m.elem_nodes, m.dirichlet)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)  # some 10 to 200 ms, by the clock it counts
    assert not side.query()
    del h
    done = side.query()
    side.synchronize()
    assert done == (kind != "borrowed")
