"""GPU parity at the edges of the kernels' paths: the shapes, counts and sizes at which a launch rule
changes its variant or a kernel its loop.

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


def check(gpu, orc, shapes, eb, sub, zero_blocks=0, k=5, p_zero=0.6, xs=None):
    """One batch call over `shapes`, both directions."""
    if xs is None:
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


# the same at the lines as they depend on the number of bands: two bands, three, four (a full round), five
@pytest.mark.parametrize("sub", [32, 128])
@pytest.mark.parametrize("shape", [(5, 307, 46, 45), (3, 512, 46, 45), (23, 89, 70, 64), (4, 512, 70, 64), (6, 512, 70, 64),
                                   (8, 512, 70, 90), (8, 512, 86, 70)])
def test_shared_planes_by_their_bands(gpu, orc, shape, sub):
    check(gpu, orc, [shape], 1e-2, sub)


# a few tall planes beside large planes that they take into their launch, and beside more of them than they take
@pytest.mark.parametrize("sub", [32, 128])
@pytest.mark.parametrize("count", [1, 6])
def test_tall_planes_beside_large_ones(gpu, orc, count, sub):
    check(gpu, orc, [(1, 5, 150, 130)] + [(4, 512, 46, 45)] * count + [(3, 50, 14, 14)], 1e-2, sub)


@pytest.mark.parametrize("nsym", [4, 62, 64, 66, 126, 128, 130, 500])
@pytest.mark.parametrize("weights", [(1,), (1, 2, 3, 4, 8), (1, 1, 50, 2000)])
def test_codebook_around_its_window(gpu, orc, nsym, weights):
    """Used symbols around the 64 nodes of either queue that a round of the merge looks at, with counts
    that tie within and across the queues: code lengths and codes of the sequential rule."""
    eb = 1e-2
    _, _, s, _ = orc.constants(eb)
    rng = np.random.default_rng(nsym + len(weights))
    v = np.repeat(np.arange(1, nsym // 2 + 1), rng.choice(weights, nsym // 2))
    rng.shuffle(v)
    d = np.stack([v, -v], axis=1).reshape(-1)                    # (v, -v): the running sums stay small
    d = np.concatenate([d, np.zeros((-d.size) % 64, np.int64)])
    q = np.cumsum(d.reshape(-1, 64), axis=1)
    x = (q.astype(np.float32) * np.float32(s)).reshape(1, -1, 1, 64)
    ctx = gpu.Context(sub=32, max_numel=x.size)
    buf, size, rc = ctx.compress(torch.from_numpy(x).cuda(), eb)
    orc_rc, obuf, osize, st = orc.compress(x, eb, orc.Config(sub=32), want_stages=True)
    assert rc == 0 and orc_rc == 0
    assert np.array_equal(ctx.stage(gpu.CMP_STAGE_LENS).numpy(), st.lens)
    assert size == osize and np.array_equal(buf[:size].cpu().numpy(), obuf)


@pytest.mark.parametrize("chunks", [1, 3, 4, 5, 16, 17])
@pytest.mark.parametrize("extra", [-1, 0, 1])
@pytest.mark.parametrize("zero_blocks", [0, 1])
def test_ranges_of_few_chunks(gpu, orc, chunks, extra, zero_blocks):
    """Tensors that end at or beside the end of a chunk and of a workgroup's range of chunks, alone in a
    call and after another tensor.  Calls as small as these have ranges of four chunks."""
    n = chunks * 4096 + extra
    check(gpu, orc, [(1, 1, 1, n)], 1e-2, 64, zero_blocks, p_zero=0.8)
    check(gpu, orc, [(2, 3, 37, 41), (1, n, 1, 1), (1, 1, 64, 65)], 1e-3, 32, zero_blocks, p_zero=0.8)


@pytest.mark.parametrize("per_range,zero_blocks", [(8, 0), (8, 1), (16, 0), (16, 1)])
def test_ranges_of_8_and_16_chunks(gpu, orc, per_range, zero_blocks):
    """Calls of so many chunks that a range holds 8 or 16 of them: one large tensor, and small ones behind it
    that end inside, at and beside the end of a range."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    fill = 4 * cus * per_range                          # chunks from which on the ranges are that long
    sizes = [4096 * c + extra for c in (1, 3, per_range - 1, per_range, per_range + 1, 2 * per_range) for extra in (-1, 0, 1)]
    xs = [torch.zeros((fill, 64, 8, 8), device="cuda")]         # a chunk per sample
    xs += [activation((1, 1, 1, n), 5, 0.8, seed=n).cuda() for n in sizes]
    xs[0][..., ::7] = 0.3
    ebs = [1e-2] * len(xs)
    ctx = gpu.Context(sub=32, max_numel=sum(x.numel() for x in xs), zero_blocks=zero_blocks)
    bufs, lens, rc = ctx.compress_batch(xs, ebs)
    assert rc == 0
    outs = [torch.full(x.shape, float("nan"), device="cuda") for x in xs]
    ctx.decompress_batch(bufs, lens, [x.shape for x in xs], ebs, outs=outs)
    assert ctx.last_status() == 0
    assert bool(((outs[0] - xs[0]).abs() <= 1e-2).all())
    cfg = orc.Config(sub=32, zero_blocks=zero_blocks)
    for x, buf, size in zip(xs[1:], bufs[1:], lens[1:]):
        orc_rc, obuf, osize, _ = orc.compress(x.cpu().numpy(), 1e-2, cfg)
        assert orc_rc == 0 and size == osize
        assert np.array_equal(buf[:size].cpu().numpy(), obuf), x.shape
    for x, y, buf, size in zip(xs[1:], outs[1:], bufs[1:], lens[1:]):
        orc_rc, oy = orc.decompress(buf[:size].cpu().numpy(), x.shape, 1e-2, cfg)
        assert orc_rc == 0 and np.array_equal(y.cpu().numpy().view(np.uint32), oy.view(np.uint32))


# sub-blocks of 64 and 128 codes, bands decoded by another wave than their own: rows that end inside a
# sub-block, a ragged last sub-block, waves without a band, outliers, planes of every plan, payload
# beyond the staging buffer, sub-blocks without codes
@pytest.mark.parametrize("sub", [64, 128])
@pytest.mark.parametrize("shape,eb,zero_blocks", [
    ((1, 1, 1, 3), 1e-2, 0), ((3, 7, 13, 11), 1e-2, 0), ((2, 41, 28, 29), 1e-2, 1), ((1, 3, 45, 44), 1e-3, 0),
    ((2, 2, 101, 99), 1e-2, 0), ((1, 5, 61, 255), 1e-3, 0), ((29, 200, 47, 45), 2e-2, 0), ((1, 3, 200, 64), 2e-4, 0),
    ((2, 64, 33, 128), 1e-2, 1),
])
def test_pooled_decode(gpu, orc, sub, shape, eb, zero_blocks):
    check(gpu, orc, [shape], eb, sub, zero_blocks, p_zero=0.9 if zero_blocks else 0.5)


# rows wider than four waves in planes larger than a band: shared by the waves of a workgroup up to 512
# columns, with sub-blocks of 32 codes and from a number of planes on, the unfused kernels otherwise
@pytest.mark.parametrize("shape,sub,eb", [
    ((1, 400, 9, 257), 32, 1e-2), ((4, 100, 8, 500), 32, 1e-3), ((1, 192, 17, 512), 32, 1e-2),
    ((1, 192, 4, 513), 32, 1e-2), ((1, 191, 5, 512), 32, 1e-2), ((1, 400, 8, 301), 128, 1e-2),
    ((3, 150, 18, 385), 32, 1e-2), ((1, 3, 40, 700), 32, 1e-2),
])
def test_wide_rows(gpu, orc, shape, sub, eb):
    check(gpu, orc, [shape, (2, 3, 28, 28), (1, 2, 100, 90)], eb, sub, zero_blocks=1 if shape[1] == 150 else 0)


# codebooks on either side of the share of codes past the tables from which every wave decodes its own
# bands (from 2 % of the codes at eb 1e-3 to 0.03 % at 1e-2), and last sub-blocks that another wave than
# the pool's decodes beside it: in the last of two bands, in a band of its own, behind planes of two bands
@pytest.mark.parametrize("sub", [64, 128])
@pytest.mark.parametrize("eb", [1e-3, 1.8e-3, 2.5e-3, 1e-2])
@pytest.mark.parametrize("shape", [(1, 4, 28, 28), (1, 64, 55, 55), (2, 3, 101, 99), (1, 40, 31, 62), (1, 1, 1, 1930),
                                   (1, 2, 9, 7), (1, 2, 38, 37)])
def test_pooled_or_a_wave_each(gpu, orc, shape, eb, sub):
    check(gpu, orc, [shape, (1, 128, 28, 28)], eb, sub)


# bands whose payload exceeds the staging buffer beside bands that fit it, in one workgroup: blocks of rows
# without structure (about ten bits a code) among zeros, in a quarter, a half and three quarters of the tensor
@pytest.mark.parametrize("sub", [32, 64, 128])
@pytest.mark.parametrize("dense", [1, 2, 3])
@pytest.mark.parametrize("shape,block", [((1, 24, 40, 48), 40), ((2, 5, 90, 60), 11), ((1, 50, 17, 13), 150), ((6, 400, 50, 45), 23)])
def test_bands_beyond_the_staging_buffer(gpu, orc, shape, block, dense, sub):
    rng = np.random.default_rng(dense)
    rows = np.arange(int(np.prod(shape[:3])))
    x = rng.uniform(0, 4.5, (rows.size, shape[3])).astype(np.float32)
    x[(rows // block) % 4 >= dense] = 0
    check(gpu, orc, [shape], 1e-2, sub, xs=[torch.from_numpy(x.reshape(shape))])


# wide rows on either side of the counts of planes from which the fused kernel takes them: planes of two rounds
# of bands, of more, and a tensor larger than the memory-side cache
@pytest.mark.parametrize("shape,eb", [
    ((1, 191, 24, 512), 1e-2), ((1, 192, 24, 512), 1e-3), ((1, 447, 45, 400), 1e-2), ((1, 448, 45, 400), 1e-3),
    ((1, 320, 461, 456), 1e-2),
])
def test_wide_rows_from_a_count_of_planes_on(gpu, orc, shape, eb):
    check(gpu, orc, [shape], eb, 32)
