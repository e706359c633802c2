"""GPU parity of the unfused decode's passes along the rows and down the columns.

Bar: the reconstruction equals the CPU oracle's bit for bit.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2011_09017_amd import binding
    binding.lib()
    return binding


# remainders of 64 columns, of a wave's 16 rows, of a workgroup's 128 rows and of a row's steps of 512 elements; rows
# longer than what a tile of the first sweep takes.  Sub-blocks of 64: no fused kernel for these rows
@pytest.mark.parametrize("shape", [
    (1, 1, 1, 3000), (2, 3, 7, 320), (1, 2, 16, 257), (1, 2, 17, 319), (1, 1, 127, 321), (1, 3, 128, 512), (2, 1, 129, 513),
    (1, 2, 256, 577), (1, 1, 257, 1024), (1, 1, 300, 1025), (1, 1, 3, 20000), (3, 1, 1000, 300), (1, 70, 50, 290),
])
@pytest.mark.parametrize("eb", [1e-2, 1e-4])
def test_passes_over_memory(gpu, orc, shape, eb):
    rng = np.random.default_rng(shape[2])
    x = np.maximum(rng.standard_normal(shape).cumsum(-1) * 0.05, 0).astype(np.float32) % 3
    x.reshape(-1)[rng.integers(0, x.size, 20)] = 50
    ctx = gpu.Context(sub=64, max_numel=x.size)
    buf, size, rc = ctx.compress(torch.from_numpy(x).cuda(), eb)
    assert rc >= 0
    cfg = orc.Config(sub=64)
    orc_rc, obuf, osize, _ = orc.compress(x, eb, cfg)
    assert orc_rc == rc and size == osize and np.array_equal(buf[:size].cpu().numpy(), obuf)
    y = ctx.decompress(buf, size, shape, eb)
    orc_rc, oy = orc.decompress(obuf, shape, eb, cfg)
    assert orc_rc == 0
    assert np.array_equal(y.cpu().numpy().view(np.uint32), oy.view(np.uint32))


# either side of the lines from which planes with wide rows take the fused kernel: one and two rounds of bands from
# one plane on, three and four from 192, more from 320; a batch of both kinds
@pytest.mark.parametrize("shapes", [
    [(1, 1, 7, 300)], [(1, 1, 48, 300)], [(1, 3, 24, 512)], [(1, 191, 49, 300)], [(1, 192, 49, 300)], [(1, 192, 96, 300)],
    [(1, 192, 97, 300)], [(1, 319, 33, 500)], [(1, 319, 97, 300)], [(1, 320, 97, 300)], [(2, 2, 20, 400), (1, 4, 300, 400), (3, 8, 30, 30)],
])
@pytest.mark.parametrize("eb", [1e-2, 1e-3])
def test_wide_rows(gpu, orc, shapes, eb):
    rng = np.random.default_rng(len(shapes))
    xs = [np.maximum(rng.standard_normal(s), 0).astype(np.float32) for s in shapes]
    ctx = gpu.Context(sub=32, max_numel=sum(-(-x.size // 4096) * 4096 for x in xs))
    bufs, sizes, rc = ctx.compress_batch([torch.from_numpy(x).cuda() for x in xs], [eb] * len(xs))
    assert rc == 0
    ys = ctx.decompress_batch(bufs, sizes, shapes, [eb] * len(xs))
    cfg = orc.Config(sub=32)
    for x, s, buf, size, y in zip(xs, shapes, bufs, sizes, ys):
        orc_rc, obuf, osize, _ = orc.compress(x, eb, cfg)
        assert orc_rc == 0 and size == osize and np.array_equal(buf[:size].cpu().numpy(), obuf)
        orc_rc, oy = orc.decompress(obuf, s, eb, cfg)
        assert orc_rc == 0
        assert np.array_equal(y.cpu().numpy().view(np.uint32), oy.view(np.uint32))
