"""Setups that take the device blocks of destroyed hierarchies: bit for bit the results of the
first ones, also from threads on their own streams at once, with the kept memory bounded."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from paper_2606_24748_amd import blkamg as B  # noqa: E402
from tests.gpu_util import dev, q1_problem  # noqa: E402


@pytest.mark.parametrize("hier", [B.F64, B.F32])
def test_setups_in_kept_blocks(hier):
    def problems():
        out = []
        for n, seed in ((5, 1), (8, 2), (11, 3)):
            m, i, j, v, _ = q1_problem(n, seed)
            plan, HA = B.coo_plan_create(m.n_nodes, m.n_nodes, 3, 3, i, j)
            B.coo_assemble_blocked(plan, dev(v), B.INSERT, HA)
            out.append((m, plan, HA, dev(synth.rhs(m, seed))))
        torch.cuda.synchronize()
        return out

    def solve(prob, stream):
        m, _, HA, b = prob
        with torch.cuda.stream(stream):
            opts = B.blkamg_opts_default()
            opts.hier_dtype = hier
            opts.p_dtype = hier
            M = B.amg_setup(HA, m.coords, m.dirichlet, opts)
            x = torch.zeros(m.n_dof, dtype=torch.float64, device="cuda")
            code, _, _ = B.pcg_solve(HA, M, b, x, rtol=1e-8)
            assert code == B.OK
            del M  # its blocks go to the next setup of either thread
            return x.cpu().numpy()

    own = [problems(), problems()]  # a matrix belongs to one thread
    main = torch.cuda.Stream()
    ref = [solve(q, main) for q in own[0]]
    free0 = torch.cuda.mem_get_info()[0]
    wrong = []

    def work(first):
        try:
            s = torch.cuda.Stream()
            for t in range(9):
                k = (first + t * (first + 1)) % 3
                if not np.array_equal(solve(own[first][k], s), ref[k]):
                    wrong.append((first, t, k))
        except Exception as e:  # reported by the assertion below
            wrong.append((first, repr(e)))

    ts = [threading.Thread(target=work, args=(f,)) for f in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not wrong, wrong
    assert free0 - torch.cuda.mem_get_info()[0] <= (4 << 30) + (1 << 28)
