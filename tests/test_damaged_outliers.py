"""Containers whose outlier records are damaged are refused, by the fused kernels as by the unfused ones.

The damage is to valid containers of the shapes that every launch of the decoder takes; the CPU oracle
refuses each of them.  No damaged record is ever stored through: an index counts only inside its band.
"""
import numpy as np
import pytest
import torch

from paper_2011_09017_amd.workloads import activation

pytestmark = pytest.mark.gpu

EB = 1e-2
# groups of small planes; large planes shared by a workgroup; a wave per large plane; rows of 257 to 512
# shared by a workgroup; the unfused kernels
SHAPES = [(2, 5, 13, 17), (1, 3, 60, 61), (5, 520, 46, 45), (5, 100, 12, 385), (1, 2, 9, 700)]


def container(shape, sub):
    from paper_2011_09017_amd import binding
    x = activation(shape, 5, 0.5, seed=sum(shape)).numpy()
    flat = x.reshape(-1)
    flat[::max(1, flat.size // 50)] = 40.0                       # outliers all over the tensor
    ctx = binding.Context(sub=sub, max_numel=x.size)
    buf, size, rc = ctx.compress(torch.from_numpy(x).cuda(), EB)
    assert rc == 0
    return ctx, buf[:size].cpu().numpy()


def status(ctx, buf, shape):
    ctx.decompress(torch.from_numpy(buf).cuda(), buf.size, shape, EB)
    return ctx.last_status()


@pytest.mark.parametrize("sub", [32, 128])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("which", ["first", "middle", "last"])
def test_index_beyond_the_tensor(orc, shape, sub, which):
    ctx, good = container(shape, sub)
    h = orc.parse_header(good)
    k = {"first": 0, "middle": h["n_outliers"] // 2, "last": h["n_outliers"] - 1}[which]
    at = h["off_outl_idx"] + 4 * k
    for index in (h["numel"], h["nchunks"] * 4096, 2 ** 32 - 1):
        bad = good.copy()
        bad[at:at + 4] = np.frombuffer(np.uint32(index).tobytes(), np.uint8)
        assert orc.decompress(bad, shape, EB, orc.Config(sub=sub))[0] == orc.E_FORMAT
        assert status(ctx, bad, shape) == orc.E_FORMAT, index
    assert status(ctx, good, shape) == 0


def test_wide_rows_records_of_another_chunk(orc):
    """Rows of 257 to 512 find a band's records by the chunks' counts, where the unfused kernels
    patched every record of the list: counts that deal a record to another chunk are refused."""
    shape = SHAPES[3]
    ctx, good = container(shape, 32)
    h = orc.parse_header(good)
    counts = good[h["off_outl_off"]:h["off_outl_off"] + 4 * (h["nchunks"] + 1)].view("<u4")
    hit = [c for c in range(1, h["nchunks"]) if counts[c - 1] < counts[c] < counts[c + 1]]
    assert hit
    for c in (hit[0], hit[len(hit) // 2], hit[-1]):
        for step in (-1, 1):
            bad = good.copy()
            at = h["off_outl_off"] + 4 * c
            bad[at:at + 4] = np.frombuffer(np.uint32(int(counts[c]) + step).tobytes(), np.uint8)
            assert orc.decompress(bad, shape, EB, orc.Config(sub=32))[0] == orc.E_FORMAT
            assert status(ctx, bad, shape) == orc.E_FORMAT, (c, step)
    assert status(ctx, good, shape) == 0
