"""The noise sampler's tiles: frames that fill tiles exactly, leave one element
over or fall short, in short and whole tiles; tiles of one kind of element
(nothing, inversion, rejection), of few rejections (settled at once) and of
many (listed); NaN and negative elements.  The same bits as the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

TILE = 2048
BIG = 1024 * TILE   # whole tiles from here on


def _frame(n, kind, rng):
    lam = np.zeros(n, np.float32)
    if kind == "inversion":
        lam[:] = rng.uniform(0.0, 9.99, n)
    elif kind == "rejection":
        lam[:] = 10.0 ** rng.uniform(1.0, 5.0, n)
    elif kind in ("few", "many"):
        lam[:] = rng.uniform(0.0, 9.99, n) * (rng.uniform(size=n) < 0.5)
        at = rng.uniform(size=n) < (0.02 if kind == "few" else 0.4)
        lam[at] = 10.0 ** rng.uniform(1.0, 3.0, int(at.sum()))
        lam[rng.integers(0, n, 1 + n // 500)] = np.nan
        lam[rng.integers(0, n, 1 + n // 500)] = -4.0
    return lam


@pytest.mark.parametrize("n,kind", [(1, "inversion"), (1, "rejection"), (63, "few"), (256, "zero"), (257, "many"),
                                    (5000, "rejection"), (4999, "inversion"), (BIG - 1, "few"), (BIG, "many"),
                                    (BIG + 1, "few"), (BIG + 2049, "rejection")])
def test_tiles_bit_exact(n, kind):
    import torch
    import paper_2506_03747_amd as nl
    lam = _frame(n, kind, np.random.default_rng(n))
    sn = torch.tensor([0.75], dtype=torch.float64, device="cuda")
    g = torch.from_numpy(lam).cuda()
    out = nl.poisson_noise(g, sn, 77)
    nl.poisson_noise(g, sn, 77, out=g)
    torch.cuda.synchronize()
    want = oracle.poisson_noise(lam, 0.75, 77)
    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert torch.equal(g, out)


@pytest.mark.parametrize("n", [1, 63, 64 * 256, 8 * 1024 * 256 - 1, 8 * 1024 * 256 + 1, 70 * 1024 * 256 + 5])
def test_moments_of_any_length(n):
    """Batches of eight reads per thread, a last one that is partly past the
    end, and counts past the table of reciprocals."""
    import torch
    import paper_2506_03747_amd as nl
    t = torch.rand(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n)) + 0.5
    got = nl.noise_scale(t, 3.0).cpu().numpy()
    d = t.double()
    np.testing.assert_allclose(got[:2], [float(d.mean()), float(d.var(correction=0))], rtol=1e-9, atol=1e-15)
