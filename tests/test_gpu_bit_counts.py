"""GPU parity of the packing: bit counts from the first sweep's running counts, and codewords that do
not fit a packing entry.

Bar: the container equals the CPU oracle's byte for byte, the reconstruction bit for bit.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EB = 1e-2
# workgroups of the first sweep that are resident together: a call of up to four chunks each takes runs of that many


def SWEEP_SLOTS():
    return 8 * torch.cuda.get_device_properties(0).multi_processor_count


STEP = float(np.float32(2) * (np.float32(EB) - np.float32(np.ldexp(np.float32(EB), -7))))


@pytest.fixture(scope="module")
def gpu():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2011_09017_amd import binding
    binding.lib()
    return binding


def check(gpu, orc, x, sub, zero_blocks):
    x = np.ascontiguousarray(x, np.float32)
    ctx = gpu.Context(sub=sub, max_numel=x.size, zero_blocks=zero_blocks)
    buf, size, rc = ctx.compress(torch.from_numpy(x).cuda(), EB)
    assert rc == 0
    cfg = orc.Config(sub=sub, zero_blocks=zero_blocks)
    orc_rc, obuf, osize, _ = orc.compress(x, EB, cfg)
    assert orc_rc == 0 and size == osize
    assert np.array_equal(buf[:size].cpu().numpy(), obuf)
    y = ctx.decompress(buf, size, x.shape, EB)
    assert ctx.last_status() == 0
    orc_rc, oy = orc.decompress(obuf, x.shape, EB, cfg)
    assert orc_rc == 0
    assert np.array_equal(y.cpu().numpy().view(np.uint32), oy.view(np.uint32))
    return orc.parse_header(obuf)


# planes of one element: every value is its own residual, so the symbols' counts can be chosen: Fibonacci
# numbers give the longest codes; the rare symbols all in one step, or spread out
@pytest.mark.parametrize("order", ["together", "spread"])
@pytest.mark.parametrize("largest", [100, 500])                 # all symbols have a byte form; most do not
@pytest.mark.parametrize("sub,zero_blocks", [(32, 0), (64, 1), (128, 0)])
def test_codes_longer_than_an_entry(gpu, orc, order, largest, sub, zero_blocks):
    counts = [1, 1]
    while len(counts) < 30:
        counts.append(counts[-1] + counts[-2])
    rng = np.random.default_rng(largest)
    q = rng.permutation(np.arange(-largest, largest + 1))[:len(counts)].astype(np.int64)
    sym = np.repeat(q, counts)
    if order == "spread":
        sym = rng.permutation(sym)
    else:
        sym[:4096] = rng.permutation(sym[:4096])
    h = check(gpu, orc, (sym * STEP).reshape(1, -1, 1, 1), sub, zero_blocks)
    assert h["max_len"] >= 25


# runs of three chunks per workgroup of the first sweep: chunks of bytes, with symbols that have no byte form and
# with outliers in every order; planes of one chunk each, then cut otherwise
@pytest.mark.parametrize("sub,zero_blocks", [(32, 0), (128, 1)])
def test_running_counts(gpu, orc, sub, zero_blocks):
    rng = np.random.default_rng(5)
    planes = 2 * SWEEP_SLOTS() + 204                                 # of one chunk each
    q = np.zeros((1, planes, 64, 64), np.int64)
    kind = rng.integers(0, 4, planes)
    for amplitude, k in ((60, 1), (300, 2), (900, 3)):
        for p in np.nonzero(kind == k)[0]:
            at = rng.integers(0, 4096, 40)
            q[0, p].reshape(-1)[at] = rng.integers(1, amplitude + 1, 40)
    x = q * STEP
    check(gpu, orc, x, sub, zero_blocks)
    cut = planes * 4096 // (37 * 61)
    check(gpu, orc, x.reshape(-1)[:cut * 37 * 61].reshape(1, cut, 37, 61), sub, zero_blocks)


# one symbol that fills every element of runs of eight chunks: a count of 32768, with a byte form and without
@pytest.mark.parametrize("residual", [1, -300])
def test_running_counts_of_full_runs(gpu, orc, residual):
    n = (8 * SWEEP_SLOTS() - 1) * 4096 + 5
    x = np.full((1, n, 1, 1), residual * STEP, np.float32)           # planes of one element
    x[0, ::5000] = 0
    check(gpu, orc, x, 32, 0)


# what include/cmpz.h promises for cmp_create, and two steps of the allocator
def test_scratch_of_a_context(gpu):
    n = 1 << 28
    first = gpu.Context(max_numel=4096)                              # what the runtime sets up on its first use
    first.compress(torch.zeros((1, 1, 64, 64), device="cuda"), EB)
    before = torch.cuda.mem_get_info()[0]
    ctx = gpu.Context(max_numel=n)
    used = before - torch.cuda.mem_get_info()[0]
    ctx.close()
    first.close()
    assert 2 * n < used < 2.51 * n + 2e6 + 2 * (2 << 20)


# rows too wide for the first sweep's tile: its other kernel, runs of four chunks
@pytest.mark.parametrize("sub,zero_blocks", [(32, 0), (32, 1), (128, 1)])
@pytest.mark.parametrize("shape", [(1, 1, 20, 1100), (2, 3, 9, 1501)])
def test_running_counts_wide_rows(gpu, orc, shape, sub, zero_blocks):
    rng = np.random.default_rng(7)
    q = np.where(rng.random(shape) < 0.01, rng.integers(0, 400, shape), 0)
    q[..., : shape[3] // 2] = 0
    check(gpu, orc, q * STEP, sub, zero_blocks)
