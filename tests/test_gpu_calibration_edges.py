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


# either side of the size from which a lane ranks a channel against every key; patterns that are no finite value >= 0 still give a permutation
@pytest.mark.parametrize("K", [48, 4112, 8176, 8192, 8208, 14336])
def test_order_of_any_patterns(K):
    rng = np.random.default_rng(K)
    c = rng.choice(np.array([0, 1, 0x3F800000, 0x7F800000, 0x80000000, 0xFFFFFFFE, 0xFFFFFFFF], dtype=np.uint32), K)
    perm, _, _ = B.arcq_calib_select(torch.from_numpy(c.view(np.float32)).cuda())
    assert np.array_equal(perm.cpu().numpy(), np.argsort(c, kind="stable"))


def test_S_reaches_any_host_memory():
    """Page-locked memory takes it from the kernel, other memory from a copy."""
    c = torch.rand(4096, device="cuda")
    perm, info = torch.empty(4096, dtype=torch.int32, device="cuda"), torch.empty(4, dtype=torch.int32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    plain, pinned = torch.full((3,), -1, dtype=torch.int32), torch.full((3,), -1, dtype=torch.int32).pin_memory()
    for host in (plain, pinned, plain[1:], pinned[1:]):
        host.fill_(-1)
        assert B.lib().arcq_calib_select(c.data_ptr(), 4096, perm.data_ptr(), info.data_ptr(), host.data_ptr(), stream) == B.OK
        assert host[0].item() == info[0].item() > 0 and (host[1:] == -1).all()
    assert torch.cuda.current_stream().query()


@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("at", [1, 2, 4])
def test_S_at_any_address(pinned, at):
    c = torch.rand(4096, device="cuda")
    perm, info = torch.empty(4096, dtype=torch.int32, device="cuda"), torch.empty(4, dtype=torch.int32, device="cuda")
    host = torch.full((16,), 0x55, dtype=torch.uint8)
    host = host.pin_memory() if pinned else host
    stream = torch.cuda.current_stream().cuda_stream
    assert B.lib().arcq_calib_select(c.data_ptr(), 4096, perm.data_ptr(), info.data_ptr(), host.data_ptr() + at, stream) == B.OK
    value = host[at:at + 4].numpy().tobytes()
    assert int.from_bytes(value, "little") == info[0].item() > 0
    assert bool((host[:at] == 0x55).all()) and bool((host[at + 4:] == 0x55).all())


def test_select_under_a_default_device():
    c = torch.rand(528, device="cuda")
    perm, S, info = B.arcq_calib_select(c)
    with torch.device("cuda"):
        again, S_again, info_again = B.arcq_calib_select(c)
    assert torch.equal(perm, again) and S == S_again == info[0].item() and torch.equal(info, info_again)


@pytest.mark.parametrize("M,K", [(1, 16), (3, 528), (33, 1008), (257, 2064)])
def test_maxima_over_batches_that_rise_and_fall(M, K):
    g = torch.Generator(device="cuda").manual_seed(M)
    batches = [torch.randn(M, K, generator=g, device="cuda").half() * f for f in (1.0, 0.25, 8.0, 1.0)]
    colmax = torch.zeros(K, device="cuda")
    for x in batches:
        B.arcq_calib_absmax(x, colmax)
    assert torch.equal(colmax, torch.cat(batches).abs().amax(0).float())
