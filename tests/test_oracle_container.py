"""Pins for chunked bit-packing, the container, and the oracle end to end.

Fixed independently of the oracle: hand-packed bit streams, a hand-computed
whole container, an independent pure-Python decoder of the container written
from the layout description, header-corruption rejection, the error bound of
Section 2.2 and zero preservation of Sections 3.2/4.4 on synthetic activations.
"""
import os
import struct

import numpy as np
import pytest
from hypothesis import assume, given, settings, strategies as st

from paper_2011_09017_amd.workloads import activation

GOLD = os.path.join(os.path.dirname(__file__), "golden")


def align16(v):
    return (v + 15) // 16 * 16


def py_decode(buf, cfg):
    """Independent decoder for the symbol stream: brute-force prefix matching against the
    canonical code table rebuilt from `lens` (dictionary lookup, bit string by bit string)."""
    b = bytes(buf)
    numel, = struct.unpack_from("<Q", b, 32)
    nchunks, = struct.unpack_from("<I", b, 56)
    off_lens, off_co, off_oo, off_sb, off_pl, off_oi, off_ov = struct.unpack_from("<7Q", b, 80)
    nsym = 2 * cfg.radius
    lens = list(b[off_lens:off_lens + nsym])
    table, code, prev = {}, 0, None
    for L, k in sorted((L, k) for k, L in enumerate(lens) if L):
        code = 0 if prev is None else (code + 1) << (L - prev)
        prev = L
        table[format(code, "0%db" % L)] = k
    nsub = cfg.chunk // cfg.sub
    syms = []
    for c in range(nchunks):
        u0, u1 = struct.unpack_from("<2I", b, off_co + 4 * c)
        words = struct.unpack_from("<%dI" % (4 * (u1 - u0)), b, off_pl + 16 * u0)
        bits = "".join(format(w, "032b") for w in words)
        pos = 0
        for j in range(nsub):
            sb, = struct.unpack_from("<H", b, off_sb + 2 * (c * nsub + j))
            n_here = max(0, min(cfg.sub, numel - (c * cfg.chunk + j * cfg.sub)))
            cur, end = "", pos + sb
            got = 0
            p = pos
            while p < end:
                cur += bits[p]; p += 1
                if cur in table:
                    syms.append(table[cur]); cur = ""; got += 1
            assert cur == "" and got == n_here
            pos = end
        assert set(bits[pos:]) <= {"0"}            # padding bits are zero
    return np.array(syms, np.uint16)


def test_hand_computed_2x2_container(orc):
    gold = dict(line.split() for line in open(os.path.join(GOLD, "tiny_container.txt"))
                if line.strip() and not line.startswith("#"))
    eb = np.float32(0.5)
    rc, eb_in, s, r = orc.constants(eb)
    assert float(eb_in) == 127 / 256 and float(s) == 127 / 128
    x = (np.array([[0, 1], [2, 5]], np.float32) * s).reshape(1, 1, 2, 2)
    rc, buf, size, stg = orc.compress(x, eb, want_stages=True)
    assert rc == 0
    assert list(stg.q) == [0, 1, 2, 5]
    assert list(stg.delta) == [0, 1, 2, 2]
    assert list(stg.sym) == [512, 513, 514, 514]
    assert stg.cnt[512] == 1 and stg.cnt[513] == 1 and stg.cnt[514] == 2 and stg.cnt.sum() == 4
    assert (stg.lens[512], stg.lens[513], stg.lens[514]) == (2, 2, 1) and stg.lens.sum() == 5
    assert (stg.codes[514], stg.codes[512], stg.codes[513]) == (0, 0b10, 0b11)
    # the container, written out by hand from the layout
    want = bytearray(int(gold["total_size"]))
    want[0:4] = b"CMPZ"
    struct.pack_into("<3I", want, 4, 1, 0, int(eb.view(np.uint32)))
    struct.pack_into("<4I", want, 16, 1, 1, 2, 2)
    struct.pack_into("<Q", want, 32, 4)
    struct.pack_into("<4I", want, 40, 512, 4096, 128, 7)
    struct.pack_into("<4I", want, 56, 1, int(gold["n_outliers"]), 0, int(gold["max_len"]))
    struct.pack_into("<Q", want, 72, int(gold["total_bits"]))
    off_lens, off_co = 256, 256 + 1024
    off_oo = off_co + 16; off_sb = off_oo + 16; off_pl = off_sb + 64
    off_oi = off_pl + 16
    struct.pack_into("<8Q", want, 80, off_lens, off_co, off_oo, off_sb, off_pl, off_oi, off_oi, off_oi)
    want[off_lens + 512] = 2; want[off_lens + 513] = 2; want[off_lens + 514] = 1
    struct.pack_into("<2I", want, off_co, 0, 1)
    struct.pack_into("<2I", want, off_oo, 0, 0)
    struct.pack_into("<H", want, off_sb, int(gold["sub_bits0"]))
    struct.pack_into("<I", want, off_pl, int(gold["payload_word0"], 16))
    assert size == int(gold["total_size"]) == off_oi
    assert bytes(buf) == bytes(want)
    rc, y = orc.decompress(buf, x.shape, eb)
    assert rc == 0 and np.array_equal(y.view(np.uint32), x.view(np.uint32))


def test_hand_packed_stream_small_chunks(orc):
    """radius 2, chunk 4, sub 2: deltas chosen so that symbols are 2,2,3,1,2,2,2,0(outlier),2,3.
    counts: sym2:6 sym3:2 sym1:1 sym0:1 -> lengths 1,2,3,3 -> codes sym2=0 sym3=10 sym0=110 sym1=111."""
    cfg = orc.Config(radius=2, chunk=4, sub=2, guard_shift=7)
    eb = np.float32(0.5)
    _, _, s, _ = orc.constants(eb)
    d = np.array([0, 0, 1, -1, 0, 0, 0, 5, 0, 1], np.int32)          # one row: W=10, so q = cumsum
    x = (np.cumsum(d).astype(np.float32) * s).reshape(1, 1, 1, 10)
    rc, buf, size, stg = orc.compress(x, eb, cfg, want_stages=True)
    assert rc == 0
    assert list(stg.delta) == list(d)
    assert list(stg.sym) == [2, 2, 3, 1, 2, 2, 2, 0, 2, 3]
    assert list(stg.lens) == [3, 3, 1, 2]
    assert list(stg.codes) == [0b110, 0b111, 0b0, 0b10]
    assert list(stg.outl_idx) == [7] and list(stg.outl_val) == [5]
    h = orc.parse_header(buf)
    assert h["nchunks"] == 3 and h["n_outliers"] == 1 and h["total_bits"] == 6 * 1 + 2 * 2 + 3 + 3
    sb = buf[h["off_sub_bits"]:h["off_sub_bits"] + 12].view("<u2")
    assert list(sb) == [2, 5, 2, 4, 3, 0]
    co = buf[h["off_chunk_off"]:h["off_chunk_off"] + 16].view("<u4")
    oo = buf[h["off_outl_off"]:h["off_outl_off"] + 16].view("<u4")
    assert list(co) == [0, 1, 2, 3] and list(oo) == [0, 0, 1, 1]
    words = [int(buf[h["off_payload"] + 16 * c: h["off_payload"] + 16 * c + 4].view("<u4")[0]) for c in range(3)]
    # chunk0: 0 0 10 111 ; chunk1: 0 0 0 110 ; chunk2: 0 10
    assert words == [0b0010111 << 25, 0b000110 << 26, 0b010 << 29]
    assert list(buf[h["off_outl_idx"]:h["off_outl_idx"] + 4].view("<u4")) == [7]
    assert list(buf[h["off_outl_val"]:h["off_outl_val"] + 4].view("<i4")) == [5]
    assert h["total_size"] == h["off_outl_val"] + 16 == size
    rc, y = orc.decompress(buf, x.shape, eb, cfg)
    assert rc == 0 and np.array_equal(y, x)


CASES = [
    # shape, k, p_zero, eb, cfg kwargs
    ((1, 3, 7, 7), 5, 0.5, 1e-2, {}),
    ((2, 2, 55, 55), 5, 0.5, 1e-3, {}),
    ((1, 5, 33, 19), 3, 0.6, 5e-3, {}),
    ((1, 2, 56, 56), 5, 0.85, 1e-2, {}),
    ((1, 1, 1, 4097), 5, 0.5, 1e-2, {}),
    ((1, 1, 4097, 1), 5, 0.5, 1e-2, {}),
    ((3, 1, 40, 40), 5, 0.5, 1e-3, dict(radius=8)),
    ((3, 1, 40, 40), 5, 0.5, 1e-2, dict(radius=1)),
    ((2, 3, 20, 30), 5, 0.5, 1e-1, dict(chunk=256, sub=32)),
    ((2, 3, 20, 30), 5, 0.5, 1e-2, dict(chunk=64, sub=64)),
]


@pytest.mark.parametrize("shape,k,p_zero,eb,kw", CASES)
def test_roundtrip_properties(orc, shape, k, p_zero, eb, kw):
    cfg = orc.Config(**kw)
    x = activation(shape, k, p_zero, seed=hash(shape) % 1000).numpy()
    rc, buf, size, stg = orc.compress(x, eb, cfg, want_stages=True)
    assert rc == 0 and size == buf.size <= orc.bound(shape, cfg)
    h = orc.parse_header(buf)
    n = x.size
    nsub = cfg.chunk // cfg.sub
    # bit accounting
    sb = buf[h["off_sub_bits"]:h["off_sub_bits"] + 2 * h["nchunks"] * nsub].view("<u2")
    assert int(sb.sum()) == h["total_bits"] == int((stg.cnt.astype(np.uint64) * stg.lens).sum())
    co = buf[h["off_chunk_off"]:h["off_chunk_off"] + 4 * (h["nchunks"] + 1)].view("<u4")
    per_chunk = sb.reshape(h["nchunks"], nsub).sum(axis=1)
    assert np.array_equal(np.diff(co.astype(np.int64)), (per_chunk + 127) // 128)
    assert co[0] == 0 and 16 * int(co[-1]) == h["off_outl_idx"] - h["off_payload"]
    # independent decode of the symbol stream
    assert np.array_equal(py_decode(buf, cfg), stg.sym)
    rc2, sym2, delta2 = orc.decode_deltas(buf, cfg)
    assert rc2 == 0 and np.array_equal(sym2, stg.sym) and np.array_equal(delta2, stg.delta)
    # outliers
    assert h["n_outliers"] == stg.n_outliers == int((stg.sym == 0).sum())
    oo = buf[h["off_outl_off"]:h["off_outl_off"] + 4 * (h["nchunks"] + 1)].view("<u4")
    want_oo = [int((stg.outl_idx < c * cfg.chunk).sum()) for c in range(h["nchunks"] + 1)]
    assert list(oo) == want_oo
    # the guarantee (Section 2.2) and the zero / sign invariants (Sections 3.2, 4.4)
    rc, y = orc.decompress(buf, shape, eb, cfg)
    assert rc == 0
    assert np.abs(y.astype(np.float64) - x.astype(np.float64)).max() <= float(np.float32(eb))
    assert np.all(y[x == 0].view(np.uint32) == 0)
    assert np.all(y >= 0)
    # the re-zero filter of Section 4.4 would change nothing: no value lies strictly inside (0, eb)
    nz = y[y != 0]
    assert nz.size == 0 or np.abs(nz).min() > float(np.float32(eb))
    # recompressing the reconstruction is lossless (quantiser fixed point)
    rc, buf2, _, stg2 = orc.compress(y, eb, cfg, want_stages=True)
    assert np.array_equal(stg2.q, stg.q)
    # determinism
    rc, buf3, _, _ = orc.compress(x, eb, cfg)
    assert np.array_equal(buf3, buf)


def test_outliers_appear_with_small_radius(orc):
    x = activation((3, 1, 40, 40), 5, 0.5, seed=5).numpy()
    rc, buf, size, stg = orc.compress(x, 1e-3, orc.Config(radius=8), want_stages=True)
    assert stg.n_outliers > 100


def test_empty_tensor(orc):
    for shape in [(0, 3, 5, 5), (2, 0, 5, 5), (2, 3, 0, 5), (2, 3, 5, 0)]:
        x = np.zeros(shape, np.float32)
        rc, buf, size, _ = orc.compress(x, 1e-2)
        assert rc == 0 and size == 256 + 1024 + 16 + 16
        h = orc.parse_header(buf)
        assert h["numel"] == 0 and h["nchunks"] == 0 and h["total_bits"] == 0 and h["max_len"] == 0
        rc, y = orc.decompress(buf, shape, 1e-2)
        assert rc == 0 and y.size == 0


def test_all_zero_and_constant_tensors(orc):
    x = np.zeros((2, 2, 9, 9), np.float32)
    rc, buf, size, stg = orc.compress(x, 1e-2, want_stages=True)
    assert stg.max_len == 1 and stg.total_bits == x.size and stg.cnt[512] == x.size
    rc, y = orc.decompress(buf, x.shape, 1e-2)
    assert rc == 0 and np.all(y.view(np.uint32) == 0)
    x[:] = 1.0
    rc, buf, size, stg = orc.compress(x, 1e-2, want_stages=True)
    assert stg.cnt[512] == x.size - 4 and stg.cnt[512 + stg.q[0]] == 4
    rc, y = orc.decompress(buf, x.shape, 1e-2)
    assert np.abs(y - 1.0).max() <= 1e-2


def test_range_warning_and_nospace(orc):
    x = activation((1, 2, 16, 16), seed=1).numpy()
    x[0, 0, 3, 3] = np.inf
    x[0, 1, 5, 5] = np.nan
    rc, buf, size, stg = orc.compress(x, 1e-2, want_stages=True)
    assert rc == orc.W_RANGE and stg.range_events == 2
    assert orc.parse_header(buf)["range_events"] == 2
    rc, y = orc.decompress(buf, x.shape, 1e-2)
    ok = np.isfinite(x)
    assert rc == 0 and np.abs(y[ok] - x[ok]).max() <= 1e-2
    rc, _, need, _ = orc.compress(x, 1e-2, cap=size - 1)
    assert rc == orc.E_NOSPACE and need == size


def test_argument_errors(orc):
    x = np.zeros((1, 1, 4, 4), np.float32)
    assert orc.compress(x, 0.0)[0] == orc.E_ARG
    assert orc.compress(x, float("nan"))[0] == orc.E_ARG
    assert orc.compress(x, 1e-2, orc.Config(radius=0))[0] == orc.E_ARG
    assert orc.compress(x, 1e-2, orc.Config(radius=513))[0] == orc.E_ARG
    assert orc.compress(x, 1e-2, orc.Config(chunk=100, sub=64))[0] == orc.E_ARG
    assert orc.compress(x, 1e-2, shape=(1, 1, -4, 4))[0] == orc.E_ARG
    assert orc.compress(x, 1e-2, shape=(65536, 65536, 1, 1), cap=1024)[0] == orc.E_ARG


U32_FIELDS = ["version", "status", "eb_bits", "radius", "chunk", "sub", "guard_shift", "nchunks",
              "n_outliers", "range_events", "max_len"]
U64_FIELDS = ["numel", "total_bits", "off_lens", "off_chunk_off", "off_outl_off", "off_sub_bits",
              "off_payload", "off_outl_idx", "off_outl_val", "total_size"]


def test_every_single_field_header_corruption_is_rejected(orc):
    shape = (1, 2, 30, 30)
    x = activation(shape, seed=9).numpy()
    x[0, 0, 4, 4] = 200.0                                   # forces an outlier
    rc, buf, size, stg = orc.compress(x, 1e-2, want_stages=True)
    assert rc == 0 and stg.n_outliers > 0
    assert orc.decompress(buf, shape, 1e-2)[0] == 0
    for name in ["magic"] + U32_FIELDS + U64_FIELDS + ["shape0", "shape1", "shape2", "shape3", "tail"]:
        bad = buf.copy()
        if name == "magic":
            bad[0] ^= 1
        elif name == "tail":
            bad[255] = 1
        elif name.startswith("shape"):
            o = orc.HDR["shape"] + 4 * int(name[-1]); bad[o] ^= 1
        elif name == "range_events":
            bad[orc.HDR[name]:orc.HDR[name] + 4] = 255       # > numel
        else:
            bad[orc.HDR[name]] ^= 1
        rc, _ = orc.decompress(bad, shape, 1e-2)
        assert rc in (orc.E_FORMAT, orc.E_MISMATCH), name
    # caller-side mismatches
    assert orc.decompress(buf, (1, 2, 30, 31), 1e-2)[0] in (orc.E_MISMATCH, orc.E_FORMAT)
    assert orc.decompress(buf, shape, 2e-2)[0] == orc.E_MISMATCH
    assert orc.decompress(buf, shape, 1e-2, orc.Config(sub=64))[0] == orc.E_MISMATCH
    assert orc.decompress(buf, shape, 1e-2, size=size - 1)[0] == orc.E_FORMAT
    assert orc.decompress(buf[:100], shape, 1e-2)[0] == orc.E_FORMAT


def test_body_corruptions_are_rejected_not_crashing(orc):
    shape = (1, 2, 30, 30)
    x = activation(shape, seed=9).numpy()
    x[0, 0, 4, 4] = 200.0
    rc, buf, size, _ = orc.compress(x, 1e-2)
    h = orc.parse_header(buf)
    rng = np.random.default_rng(0)
    rejected = 0
    for sect in ["off_lens", "off_chunk_off", "off_outl_off", "off_sub_bits", "off_outl_idx"]:
        for _ in range(20):
            bad = buf.copy()
            o = h[sect] + int(rng.integers(0, 8))
            bad[o] ^= 1 << int(rng.integers(0, 8))
            rc, _ = orc.decompress(bad, shape, 1e-2)
            rejected += rc != 0
    assert rejected >= 90          # metadata flips are caught (a flip in unused lens bytes also is)


@settings(max_examples=25, deadline=None)
@given(st.integers(1, 3), st.integers(1, 3), st.integers(1, 40), st.integers(1, 40),
       st.sampled_from([1e-1, 1e-2, 1e-3]), st.sampled_from([1, 4, 512]), st.integers(0, 1000))
def test_roundtrip_random_shapes(orc, n, c, h, w, eb, radius, seed):
    assume(n * c * h * w >= 2)          # the generator divides by the sample std
    cfg = orc.Config(radius=radius, chunk=256, sub=32)
    x = activation((n, c, h, w), 3, 0.5, seed=seed).numpy()
    assume(np.isfinite(x).all())        # a plane of two elements may be constant after the box filter: no spread to divide by
    rc, buf, size, stg = orc.compress(x, eb, cfg, want_stages=True)
    assert rc == 0
    assert np.array_equal(py_decode(buf, cfg), stg.sym)
    rc, y = orc.decompress(buf, x.shape, eb, cfg)
    assert rc == 0
    assert np.abs(y.astype(np.float64) - x.astype(np.float64)).max() <= float(np.float32(eb))
    assert np.all(y[x == 0].view(np.uint32) == 0)
