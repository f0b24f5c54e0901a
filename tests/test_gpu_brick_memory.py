"""Galerkin plan when there is no memory for the brick tables: an allocator that refuses one
request after the other.  The plan then takes the two passes; only the memory these need
themselves is still refused with ENOMEM."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import solve  # noqa: E402
from oracle import sparse as S  # noqa: E402
from paper_2606_24748_amd import blkamg as B  # noqa: E402
from tests.gpu_util import from_device_bsr, q1_problem, rel2, to_device_bsr  # noqa: E402


@pytest.mark.parametrize("dtype", [B.F64, B.F32])
def test_no_memory_for_bricks(dtype, monkeypatch):
    m, i, j, v, A = q1_problem(7, 3)
    P = solve.setup(A, m.coords, m.dirichlet, solve.Options(coarse_eq_limit=10)).levels[0].P
    HA, ka = to_device_bsr(A, dtype)
    HP, kp = to_device_bsr(P, dtype)
    want = S.ptap(from_device_bsr(HA), from_device_bsr(HP))
    B.ptap_symbolic_ex(HA, HP, B.PTAP_SYMMETRIC)  # P's transpose is there from now on
    sizes = []

    def plan(tune, refuse):
        """Sizes requested, and the product (None: ENOMEM), with request number `refuse` refused."""
        sizes.clear()

        def alloc(n, _ctx):
            sizes.append(int(n))
            return None if len(sizes) - 1 == refuse else torch.cuda.caching_allocator_alloc(int(n))

        monkeypatch.setenv("BLKAMG_PTAP_TUNE", tune)
        B.blkamg_set_allocator(alloc, lambda p, n, c: torch.cuda.caching_allocator_delete(p))
        try:
            HC = B.ptap_symbolic_ex(HA, HP, B.PTAP_SYMMETRIC)
            B.ptap_numeric(HA, HP, HC)
            return list(sizes), from_device_bsr(HC)
        except B.BlkAmgError as e:
            assert e.code == B.ENOMEM
            return list(sizes), None
        finally:
            B.blkamg_set_allocator()

    bricks, c0 = plan("ap_sort", -1)
    two, c1 = plan("ap_sort,nobrick", -1)
    first = next(k for k, (a, b) in enumerate(zip(bricks, two)) if a != b)
    assert len(bricks) - first > 20 and c0 is not None and c1 is not None
    tol = {B.F64: 1e-13, B.F32: 2e-5}[dtype]  # as for the mesh products
    assert rel2(c0.val, want.val) <= tol
    assert not (c0.val == c1.val).all()  # the bricks add in another order, so they are on
    for k in range(first, len(bricks)):
        asked, c = plan("ap_sort", k)
        assert c is not None, f"request {k} of {bricks[k]} bytes refused"
        assert (c.val == c1.val).all() and asked[k + 1:] == two[first:]
    assert plan("ap_sort", first - 1)[1] is None
    assert plan("ap_sort,nobrick", len(two) - 1)[1] is None
