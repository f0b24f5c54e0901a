"""Dense coarsest solve: the inverse Cholesky factor against numpy at the edges of its
32-dof tiles, alone and in an uneven batch."""
import numpy as np
import pytest
import torch

from gpu_util import dev
from paper_2606_24748_amd import blkamg as B

pytestmark = pytest.mark.gpu


def spd(nodes, seed):
    """Dense SPD matrix of 3 * nodes dofs with eigenvalues between 1 and 100."""
    rng = np.random.default_rng(seed)
    n = 3 * nodes
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    A = (Q * np.geomspace(1.0, 100.0, n)) @ Q.T
    return 0.5 * (A + A.T)


def block_diagonal(mats):
    """The matrices as one BSR of full 3x3-block rows per instance."""
    rp, ci, vals, row0 = [0], [], [], [0]
    for A in mats:
        k = A.shape[0] // 3
        for i in range(k):
            ci.extend(range(row0[-1], row0[-1] + k))
            vals.append(A[3 * i:3 * i + 3].reshape(3, k, 3).transpose(1, 0, 2))
            rp.append(rp[-1] + k)
        row0.append(row0[-1] + k)
    return np.array(rp, np.int32), np.array(ci, np.int32), np.concatenate(vals), np.array(row0, np.int32)


def setup(mats, hier=B.F64):
    rp, ci, v, row0 = block_diagonal(mats)
    nbr = len(rp) - 1
    keep = (dev(rp), dev(ci), dev(v))
    A = B.bsr_create(nbr, nbr, 3, 3, *keep)
    o = B.blkamg_opts_default()
    o.hier_dtype = o.p_dtype = hier
    M = B.amg_setup_batched(A, row0, np.random.default_rng(1).standard_normal((nbr, 3)), None, o)
    return A, M, nbr


@pytest.mark.parametrize("nodes", [1, 10, 11, 21, 22, 32, 43, 64, 75, 118, 333])
@pytest.mark.parametrize("hier", [B.F64, B.F32])
def test_single_matrix(nodes, hier):
    M0 = spd(nodes, nodes)
    if hier == B.F32:
        M0 = M0.astype(np.float32).astype(np.float64)
    A, M, nbr = setup([M0], hier)
    r = np.random.default_rng(7).standard_normal(3 * nbr)
    if hier == B.F32:
        r = r.astype(np.float32).astype(np.float64)
    z = torch.empty(3 * nbr, dtype=torch.float64, device="cuda")
    B.vcycle_apply(M, dev(r), z)
    want = np.linalg.solve(M0, r)
    # Cholesky's backward error is below n eps; condition number 100; FP32 hierarchies
    # round the factor's FP64 result once
    tol = 8 * 3 * nodes * 100 * 2.3e-16 + (6e-8 if hier == B.F32 else 0.0)
    assert np.linalg.norm(z.cpu().numpy() - want) <= tol * np.linalg.norm(want)


def test_uneven_batch_eight_columns():
    sizes = [43, 1, 32, 11, 75, 22]
    mats = [spd(k, 100 + k) for k in sizes]
    A, M, nbr = setup(mats)
    r = np.random.default_rng(8).standard_normal((3 * nbr, 8))
    z = torch.empty(3 * nbr * 8, dtype=torch.float64, device="cuda")
    B.vcycle_apply(M, dev(r.ravel()), z, nrhs=8)
    z = z.cpu().numpy().reshape(-1, 8)
    at = 0
    for k, M0 in zip(sizes, mats):
        want = np.linalg.solve(M0, r[at:at + 3 * k])
        assert np.linalg.norm(z[at:at + 3 * k] - want) <= 8 * 3 * k * 100 * 2.3e-16 * np.linalg.norm(want)
        at += 3 * k


@pytest.mark.parametrize("bad", [0, 31, 32, 100, 128])
def test_non_positive_pivot_is_reported(bad):
    M0 = spd(43, 5)
    M0[bad, bad] = -1.0
    with pytest.raises(B.BlkAmgError) as e:
        setup([M0])
    assert e.value.code == B.ENOTSPD
