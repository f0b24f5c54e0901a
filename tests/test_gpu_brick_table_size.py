"""Galerkin product whose padded brick tables would exceed 32 bits: every row couples 500 nodes
and feeds one coarse block, so 16 places are reserved for each of its products, 2.148e9 in all
for 134 million blocks of A.  Such a plan keeps the two passes, which need no padding."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_24748_amd import blkamg as B  # noqa: E402


def test_tables_beyond_32_bits():
    groups, k = 537, 500
    n = groups * k
    assert 16 * k * n > 2 ** 31 > 16 * k * (n - k)
    rp = torch.arange(n + 1, dtype=torch.int32, device="cuda") * k
    row = torch.arange(n, device="cuda") // k * k
    ci = (row[:, None] + torch.arange(k, device="cuda")).to(torch.int32).reshape(-1).contiguous()
    a = torch.ones(n * k, 3, 3, dtype=torch.float32, device="cuda")
    HA = B.bsr_create(n, n, 3, 3, rp, ci, a)
    g = torch.Generator(device="cuda").manual_seed(3)
    p = torch.randint(-1, 2, (n, 3, 6), generator=g, device="cuda").to(torch.float32)
    prp = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    pci = (torch.arange(n, device="cuda") // k).to(torch.int32)
    HP = B.bsr_create(n, groups, 3, 6, prp, pci, p)
    print(f"symbolic phase, {n * k} blocks of A", flush=True)
    HC = B.ptap_symbolic_ex(HA, HP, B.PTAP_SYMMETRIC)
    assert HC.info()["nnzb"] == groups
    print("product", flush=True)
    B.ptap_numeric(HA, HP, HC)
    # A is all ones: with t the column sums of a group's rows of P, its block is t t^T; whole
    # numbers below 2^24, so FP32 gives them exactly in any order
    t = p.view(groups, k * 3, 6).to(torch.float64).sum(1)
    want = t[:, :, None] * t[:, None, :]
    assert float(want.abs().max()) < 2 ** 24 / 16
    got = HC.arrays()[2].to(torch.float64)
    assert np.array_equal(got.cpu().numpy(), want.cpu().numpy())
