"""Element stiffness stream with eight elements a wave (48 k elements on): the same bits as the
one-element waves give for the elements in shorter calls."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from paper_2606_24748_amd import blkamg as B  # noqa: E402


# the first size of the rule; a last wave of one element; a last wave of five in a ragged workgroup
@pytest.mark.parametrize("count", [48 * 1024, 48 * 1024 + 1, 37**3])
def test_stream_bits_do_not_depend_on_the_wave_size(count):
    m = synth.make_mesh(37, clamp=False, distort=0.2, seed=2)
    lam, mu = synth.lame(*synth.materials(m.n_elem, 9))
    en = torch.as_tensor(m.elem_nodes.astype(np.int32)).cuda()[:count].contiguous()
    X, lam, mu = torch.as_tensor(m.coords).cuda(), torch.as_tensor(lam).cuda()[:count], torch.as_tensor(mu).cuda()[:count]
    got = torch.full((count * 64 + 1, 3, 3), 7.0, dtype=torch.float64, device="cuda")
    B.fe_q1_stream(en, X, lam, mu, got[:-1])
    part = torch.empty((30000 * 64, 3, 3), dtype=torch.float64, device="cuda")
    for a in range(0, count, 30000):
        b = min(count, a + 30000)
        B.fe_q1_stream(en[a:b].contiguous(), X, lam[a:b].contiguous(), mu[a:b].contiguous(), part[: (b - a) * 64])
        assert torch.equal(got[a * 64:b * 64], part[: (b - a) * 64]), a
    assert bool((got[-1] == 7.0).all())
