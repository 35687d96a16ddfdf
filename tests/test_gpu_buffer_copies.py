"""Copies into LDS through a buffer descriptor: words at or past the buffer's end arrive as zeros, wherever the scalar offset puts them."""
import pytest
import torch

from paper_2601_07475_amd import binding as B

pytestmark = pytest.mark.gpu


# ends at a lane, inside a lane's words, in the first one; scalar offsets of nothing, below the end and at it
@pytest.mark.parametrize("size,scalar", [(4096, 0), (1024, 0), (512, 0), (500, 0), (4, 0), (0, 0), (2048, 1536), (2048, 1540), (2044, 1600), (2048, 2044),
                                         (2048, 2048), (64, 64), (4, 4)])
@pytest.mark.parametrize("words", [1, 4])
def test_words_past_the_end_arrive_as_zeros(size, scalar, words):
    src = torch.arange(1, 2049, dtype=torch.int32, device="cuda")           # 8192 bytes, all of them mapped: what is past the end shows
    got = B.arcq_probe_buffer_copy(src, size, scalar, words).cpu()
    at = torch.arange(64 * words) + scalar // 4
    assert torch.equal(got[:64 * words], torch.where(at < size // 4, at + 1, 0).int())
    assert bool((got[64 * words:] == B.PROBE_UNTOUCHED - (1 << 32)).all())
