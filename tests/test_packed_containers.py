"""Decoding of hand-packed containers: code lengths that only enormous or enormously skewed tensors
produce, packed here around a few thousand codes.

The packer is written from the container's layout alone.  Its containers are read back by the CPU oracle,
and the GPU must return what the oracle returns, bit for bit.
"""
import struct

import numpy as np
import pytest
import torch

EB = 1e-2
RADIUS = 512
SHAPES = [(1, 40, 17, 19), (1, 2, 60, 61)]        # groups of small planes; planes of two bands and more


def pack(lens, sym, shape, sub):
    """A version-1 container without outliers: `sym` coded with the canonical code of `lens`."""
    n, nsub = sym.size, 4096 // sub
    nchunks = (n + 4095) // 4096
    code, prev, words = {}, 0, 0
    for L, k in sorted((int(L), k) for k, L in enumerate(lens) if L):
        words = (words + 1) << (L - prev) if prev else 0
        prev = L
        code[k] = format(words, f"0{L}b")
    sub_bits = np.zeros(nchunks * nsub, np.uint16)
    chunk_off, payload, total_bits = [0], [], 0
    for c in range(nchunks):
        bits = ""
        for j in range(nsub):
            part = sym[c * 4096 + j * sub:min((c + 1) * 4096, c * 4096 + (j + 1) * sub)]
            coded = "".join(code[int(k)] for k in part)
            sub_bits[c * nsub + j] = len(coded)
            bits += coded
        total_bits += len(bits)
        bits += "0" * (-len(bits) % 128)
        payload.append(np.array([int(bits[i:i + 32], 2) for i in range(0, len(bits), 32)], "<u4"))
        chunk_off.append(chunk_off[-1] + len(bits) // 128)

    def up16(b):
        return b + b"\0" * (-len(b) % 16)

    sections = [up16(np.asarray(lens, np.uint8).tobytes()), up16(np.array(chunk_off, "<u4").tobytes()),
                up16(bytes(4 * (nchunks + 1))), up16(sub_bits.tobytes()), np.concatenate(payload).tobytes()]
    off = [256]
    for s in sections:
        off.append(off[-1] + len(s))
    head = bytearray(256)
    head[0:4] = b"CMPZ"
    struct.pack_into("<3I", head, 4, 1, 0, int(np.float32(EB).view(np.uint32)))
    struct.pack_into("<4I", head, 16, *shape)
    struct.pack_into("<Q", head, 32, n)
    struct.pack_into("<4I", head, 40, RADIUS, 4096, sub, 7)
    struct.pack_into("<4I", head, 56, nchunks, 0, 0, int(max(lens)))
    struct.pack_into("<Q", head, 72, total_bits)
    struct.pack_into("<8Q", head, 80, *off, off[-1], off[-1])
    return np.frombuffer(bytes(head) + b"".join(sections), np.uint8).copy()


def deep_codebook(short, deepest):
    """Code lengths 1..short once each, 12 as often as it takes, 13..deepest once each and `deepest`
    once more: a complete code whose codewords past the decoder's first table (11 bits) fill the
    last 2^-short of the code space.  The smallest residuals get the shortest codes."""
    in_order = list(range(1, short + 1)) + [12] * (2 ** (12 - short) - 1) + list(range(13, deepest + 1)) + [deepest]
    assert sum(2 ** (60 - L) for L in in_order) == 2 ** 60
    lens = np.zeros(2 * RADIUS, np.uint8)
    for k, L in enumerate(in_order):
        lens[RADIUS + (k + 1) // 2 * (1 if k % 2 else -1)] = L
    return lens


def deep_symbols(lens, n, seed):
    """Short codes mostly; every codeword past 12 bits twenty times, forty of the 12-bit ones."""
    rng = np.random.default_rng(seed)
    shortest = np.nonzero((lens > 0) & (lens < 12))[0]
    weight = 0.5 ** lens[shortest].astype(np.float64)
    sym = rng.choice(shortest, n, p=weight / weight.sum())
    long = np.concatenate([np.repeat(np.nonzero(lens > 12)[0], 20), rng.choice(np.nonzero(lens == 12)[0], 40)])
    sym[rng.permutation(n)[:long.size]] = rng.permutation(long)
    return sym


def deep_container(orc, shape, short, deepest, sub):
    lens = deep_codebook(short, deepest)
    sym = deep_symbols(lens, int(np.prod(shape)), 100 * short + deepest)
    buf = pack(lens, sym, shape, sub)
    rc, y = orc.decompress(buf, shape, EB, orc.Config(sub=sub))
    assert rc == 0
    return sym, buf, y


@pytest.mark.parametrize("sub", [32, 128])
@pytest.mark.parametrize("short", [3, 9, 11])
def test_packer_against_the_oracle(orc, short, sub):
    for shape in SHAPES:
        sym, buf, y = deep_container(orc, shape, short, 48, sub)
        rc, got, _ = orc.decode_deltas(buf, orc.Config(sub=sub))
        assert rc == 0 and np.array_equal(got, sym)
        q = orc.prefix2d((sym.astype(np.int32) - RADIUS).reshape(-1, *shape[2:]))
        assert np.abs(q).max() < 16384                       # what a compressor's own containers keep to
        _, _, s, _ = orc.constants(EB)
        assert np.array_equal(y.reshape(-1), orc.dequant(q, s).reshape(-1))


@pytest.mark.gpu
@pytest.mark.parametrize("deepest", [33, 34, 35, 36, 48])
@pytest.mark.parametrize("short", range(3, 12))
@pytest.mark.parametrize("sub", [32, 64, 128])
def test_codewords_past_32_bits(orc, sub, short, deepest):
    """The search for codewords that neither decode table resolves begins at length short + 9, looks at
    four lengths at a time and changes its arithmetic at 32 bits: every place in the group of four at
    which that change can fall."""
    from paper_2011_09017_amd import binding
    for shape in SHAPES:
        _, buf, y = deep_container(orc, shape, short, deepest, sub)
        ctx = binding.Context(sub=sub, max_numel=y.size)
        got = ctx.decompress(torch.from_numpy(buf).cuda(), buf.size, shape, EB)
        assert ctx.last_status() == 0
        assert np.array_equal(got.cpu().numpy().view(np.uint32), y.view(np.uint32))
