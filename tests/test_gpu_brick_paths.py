"""Which path a Galerkin plan takes: bricks and the two passes add in different orders, so their
bits differ on random values, and a plan that keeps the two passes gives theirs.  Irregular
patterns in every type, batches cut because their rows of P exceed the LDS, and each refusal."""
import numpy as np
import pytest

import synth
from gpu_util import from_device_bsr, q1_problem, rel2, to_device_bsr
from oracle import solve
from oracle import sparse as S
from paper_2606_24748_amd import blkamg as B
from test_gpu_brick_pieces import clique, ring

pytestmark = pytest.mark.gpu

TOL = {B.F64: 1e-13, B.F32: 2e-5}  # as for the mesh products


def mesh(n, order):
    m, _, _, _, A = q1_problem(n, 3, order=order)
    return A, solve.setup(A, m.coords, m.dirichlet, solve.Options(coarse_eq_limit=10)).levels[0].P


def irregular(rows, cols, a_max, p_max):
    rp, ci, v = synth.random_spd_bsr(rows, 3, seed=rows, max_per_row=a_max)
    prp, pci, pv = synth.random_bsr(rows, cols, 3, 6, seed=cols, max_per_row=p_max)
    return (S.Bsr(rows, rows, 3, 3, rp.astype(np.int64), ci.astype(np.int64), v),
            S.Bsr(rows, cols, 3, 6, prp.astype(np.int64), pci.astype(np.int64), pv))


def wide(rows, cols):
    """Every row of P holds column 0 and three more: one first column, too many coarse blocks."""
    rp, ci, v = synth.random_spd_bsr(rows, 3, seed=1, max_per_row=8)
    rng = np.random.default_rng(2)
    pci = np.concatenate([np.append(0, np.sort(rng.choice(np.arange(1, cols), 3, replace=False))) for _ in range(rows)])
    return (S.Bsr(rows, rows, 3, 3, rp.astype(np.int64), ci.astype(np.int64), v),
            S.Bsr(rows, cols, 3, 6, 4 * np.arange(rows + 1), pci, rng.uniform(-1, 1, (4 * rows, 3, 6))))


CASES = {  # (A, P), bricks in FP64, in FP32
    "mesh_8": (lambda: mesh(8, 1), True, True),
    "mesh_13": (lambda: mesh(13, 1), True, True),
    "irregular_9": (lambda: irregular(500, 9, 40, 3), True, True),
    "irregular_3": (lambda: irregular(64, 3, 30, 2), True, True),
    # 31 (62) rows reach 248 (496) others of two P blocks each: over 355 (711) blocks
    "cut": (lambda: ring(1024, 1.0, 3, np.random.default_rng(7)), True, True),
    "rows_of_300": (lambda: clique(301, 20, np.random.default_rng(8)), False, True),  # 250, 500 A blocks at most
    "rows_of_520": (lambda: clique(521, 20, np.random.default_rng(9)), False, False),
    "wide": (lambda: wide(400, 41), False, False),  # over 128 coarse blocks a brick
    "sparse": (lambda: irregular(90, 80, 6, 1), False, False),  # under four products a coarse block
}


@pytest.mark.parametrize("types", [(B.F64, B.F64), (B.F32, B.F32), (B.F32, B.BF16)])
@pytest.mark.parametrize("name", list(CASES))
def test_path(name, types, monkeypatch):
    make, in_f64, in_f32 = CASES[name]
    A, P = make()
    HA, (_, _, av) = to_device_bsr(A, types[0])
    HP, (_, _, pv) = to_device_bsr(P, types[1])
    monkeypatch.delenv("BLKAMG_PTAP_TUNE", raising=False)
    HC = B.ptap_symbolic_ex(HA, HP, B.PTAP_SYMMETRIC)
    monkeypatch.setenv("BLKAMG_PTAP_TUNE", "ap_sort,nobrick")
    H2 = B.ptap_symbolic_ex(HA, HP, B.PTAP_SYMMETRIC)
    assert B.ptap_plan_info(HC) == B.ptap_plan_info(H2)
    for scale in (1.0, -0.5):
        av.mul_(scale)
        pv.mul_(scale)
        B.bsr_mark_modified(HA)
        B.bsr_mark_modified(HP)
        want = S.ptap(from_device_bsr(HA), from_device_bsr(HP))
        got = []
        for H in (HC, H2):
            B.ptap_numeric(HA, HP, H)
            got.append(from_device_bsr(H).val)
            assert rel2(got[-1], want.val) <= TOL[types[0]]
        assert np.array_equal(*got) != (in_f64 if types[0] == B.F64 else in_f32)
