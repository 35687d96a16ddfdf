"""GPU: channel order and running maxima at the sizes where the work is cut (slices of keys, groups of 64 channels, strips)."""
import numpy as np
import pytest
import torch

from paper_2601_07475_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [16, 64, 80, 1008, 1024, 1040, 2032, 2064, 28672])
@pytest.mark.parametrize("values", ["ties", "equal", "descending"])
def test_order_is_the_stable_ascending_one(K, values):
    rng = np.random.default_rng(K)
    c = {"ties": rng.integers(0, 7, K), "equal": np.full(K, 3), "descending": np.arange(K, 0, -1)}[values].astype(np.float32)
    perm, S, info = B.arcq_calib_select(torch.from_numpy(c).cuda())
    assert np.array_equal(perm.cpu().numpy(), np.argsort(c, kind="stable"))
    raw = int((c > c.max() * np.float32(0.125)).sum())
    assert info[1].item() == raw and S == min(K, -(-raw // 16) * 16)


@pytest.mark.parametrize("M,K", [(1, 16), (3, 528), (33, 1008), (257, 2064)])
def test_maxima_over_batches_that_rise_and_fall(M, K):
    g = torch.Generator(device="cuda").manual_seed(M)
    batches = [torch.randn(M, K, generator=g, device="cuda").half() * f for f in (1.0, 0.25, 8.0, 1.0)]
    colmax = torch.zeros(K, device="cuda")
    for x in batches:
        B.arcq_calib_absmax(x, colmax)
    assert torch.equal(colmax, torch.cat(batches).abs().amax(0).float())
