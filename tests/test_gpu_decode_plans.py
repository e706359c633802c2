"""GPU parity of the decode plans: the shapes and counts at which the launch rule changes its variant.

Bar: container and reconstruction equal the CPU oracle's bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2011_09017_amd.workloads import activation

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2011_09017_amd import binding
    binding.lib()
    return binding


def check(gpu, orc, shapes, eb, sub, zero_blocks=0, k=5, p_zero=0.6):
    """One batch call over `shapes`, both directions."""
    xs = [activation(s, k, p_zero, seed=sum(s) + i) for i, s in enumerate(shapes)]
    ctx = gpu.Context(sub=sub, max_numel=sum(x.numel() for x in xs), zero_blocks=zero_blocks)
    bufs, sizes, rc = ctx.compress_batch([x.cuda() for x in xs], [eb] * len(xs))
    assert rc == 0
    outs = [torch.full(s, float("nan"), device="cuda") for s in shapes]
    ctx.decompress_batch(bufs, sizes, shapes, [eb] * len(xs), outs=outs)
    assert ctx.last_status() == 0
    cfg = orc.Config(sub=sub, zero_blocks=zero_blocks)
    for x, s, buf, size, y in zip(xs, shapes, bufs, sizes, outs):
        orc_rc, obuf, osize, _ = orc.compress(x.numpy(), eb, cfg)
        assert orc_rc == 0 and size == osize
        assert np.array_equal(buf[:size].cpu().numpy(), obuf), s
        orc_rc, oy = orc.decompress(obuf, s, eb, cfg)
        assert orc_rc == 0
        assert np.array_equal(y.cpu().numpy().view(np.uint32), oy.view(np.uint32)), s


# planes of two and of seven bands on either side of the count from which a wave takes a plane of its
# own, alone and beside tensors of the other kind
@pytest.mark.parametrize("shapes", [
    [(5, 255, 46, 45)], [(7, 200, 46, 45)], [(10, 255, 113, 110)], [(13, 200, 113, 110)],
    [(10, 255, 46, 45), (3, 5, 7, 7), (2, 3, 200, 190), (1, 64, 56, 56)],
])
def test_shared_planes_or_one_wave_each(gpu, orc, shapes):
    check(gpu, orc, shapes, 1e-2, 32)
