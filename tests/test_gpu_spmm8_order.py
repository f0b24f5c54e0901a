"""Products with eight columns add a row's blocks in the order of one lane per block: block k on
chain k % V of fused multiply-adds, the V chains joined by an xor tree, bit for bit.  The inputs
have half a mantissa, so that every product is exact and numpy's multiply and add is the fused
one.  Row lengths around the multiples of a slot, a chain and the limits of the lane rule."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2606_24748_amd import blkamg as B  # noqa: E402

NP = {B.F64: np.float64, B.F32: np.float32}
SHAPES = [(3, 3), (3, 6), (6, 3), (6, 6)]


def chains(dtype, shape, nb):
    """V of the shape the lane rule picks for rows of nb blocks."""
    f64 = dtype == B.F64
    if nb <= 16:
        return (8 if nb <= 8 else 16) if f64 else 16
    if nb <= 40:
        return 16 if f64 and shape == (6, 6) else 32
    return 64


@pytest.mark.parametrize("dtype", [B.F64, B.F32])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("nb", [1, 4, 7, 8, 9, 16, 17, 27, 32, 33, 40, 41, 62, 64, 65, 121, 130])
def test_order_of_additions(nb, shape, dtype):
    br, bc = shape
    rows, cols, T = 9, max(nb, 5), NP[dtype]
    rng = np.random.default_rng(100 * nb + 10 * br + bc)
    half = 2 ** (26 if dtype == B.F64 else 11)
    draw = lambda *s: (rng.integers(-half, half, s) / half).astype(T)  # noqa: E731
    ci = np.stack([np.sort(rng.choice(cols, nb, replace=False)) for _ in range(rows)]).astype(np.int32)
    a, x = draw(rows, nb, br, bc), draw(cols, bc, 8)
    rp = torch.arange(rows + 1, dtype=torch.int32, device="cuda") * nb
    H = B.bsr_create(rows, cols, br, bc, rp, torch.as_tensor(ci.reshape(-1)).cuda(), torch.as_tensor(a).cuda())
    y = torch.zeros(rows * br * 8, dtype=torch.float64 if dtype == B.F64 else torch.float32, device="cuda")
    B.bsr_spmv(H, 1.0, torch.as_tensor(x.reshape(-1)).cuda(), 0.0, y, 8)
    V = chains(dtype, shape, nb)
    s = np.zeros((V, rows, br, 8), T)
    for k in range(nb):
        for j in range(bc):
            s[k % V] += a[:, k, :, j, None] * x[ci[:, k], j][:, None, :]
    while len(s) > 1:
        s = s[: len(s) // 2] + s[len(s) // 2:]
    assert np.array_equal(y.cpu().numpy().reshape(rows, br, 8), s[0])
