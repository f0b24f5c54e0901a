"""The device blocks kept after a hierarchy is destroyed go back to the device on request and
when the caller's allocator finds no memory, with other handles alive and unharmed."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from paper_2606_24748_amd import blkamg as B  # noqa: E402
from tests.gpu_util import dev, q1_problem  # noqa: E402


def test_kept_blocks_go_back():
    m, i, j, v, _ = q1_problem(16, 1)
    plan, HA = B.coo_plan_create(m.n_nodes, m.n_nodes, 3, 3, i, j)
    B.coo_assemble_blocked(plan, dev(v), B.INSERT, HA)
    b = dev(synth.rhs(m, 1))

    def solve():
        M = B.amg_setup(HA, m.coords, m.dirichlet)
        x = torch.zeros(m.n_dof, dtype=torch.float64, device="cuda")
        assert B.pcg_solve(HA, M, b, x, rtol=1e-8)[0] == B.OK
        return x.cpu().numpy()

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    ref = solve()
    B.blkamg_trim()
    base = free()
    solve()
    held = base - free()
    assert held > 8 << 20  # the destroyed hierarchy's buffers (30 MB of A P, A_c and P alone)
    B.blkamg_trim()
    assert base - free() < held / 4
    assert np.array_equal(solve(), ref)
    # an allocator that has no memory until the library gave its own back
    before = free()
    calls = []

    def alloc(n, _ctx):
        calls.append(free())
        return torch.cuda.caching_allocator_alloc(int(n)) if len(calls) > 1 else None

    assert base - before > 8 << 20
    B.blkamg_set_allocator(alloc, lambda p, n, c: torch.cuda.caching_allocator_delete(p))
    try:
        assert free() - before > held / 2  # given back when the allocator was set
        with pytest.raises(B.BlkAmgError) as e:  # nothing kept any more: no second try
            B.coo_plan_create(m.n_nodes, m.n_nodes, 3, 3, i, j)
        assert e.value.code == B.ENOMEM and len(calls) == 1
    finally:
        B.blkamg_set_allocator()
    assert np.array_equal(solve(), ref)
