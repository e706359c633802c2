"""GPU parity where the kernel that builds the code also finds a tensor's offsets and header (tensors of at
most 128 chunks), and the device-side stack's bookkeeping by the kernels that write and read the containers.

Bar: the container equals the CPU oracle's byte for byte.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EB = 1e-2


@pytest.fixture(scope="module")
def gpu():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2011_09017_amd import binding
    binding.lib()
    return binding


def tensor(shape, seed):
    """a smooth field with rare outliers, and a part with symbols of every size"""
    rng = np.random.default_rng(seed)
    x = (0.02 * rng.standard_normal(shape)).astype(np.float32)
    flat = x.reshape(-1)
    n = flat.size
    flat[n // 2:n // 2 + n // 8] *= 100.0
    flat[rng.integers(0, n, 1 + n // 5000)] = 60.0
    return x


def oracle(orc, x, sub, zero_blocks):
    rc, buf, size, _ = orc.compress(x, EB, orc.Config(sub=sub, zero_blocks=zero_blocks))
    assert rc == 0
    return buf, size


# one element; both sides of a chunk, of a wave's four chunks, of the limit
@pytest.mark.parametrize("sub,zero_blocks", [(32, 0), (128, 1)])
@pytest.mark.parametrize("n", [1, 4096, 4097, 16 * 4096, 16 * 4096 + 1, 65 * 4096 + 5, 128 * 4096 - 1, 128 * 4096, 128 * 4096 + 1,
                               256 * 4096 - 1, 256 * 4096, 256 * 4096 + 1])
def test_sizes(gpu, orc, n, sub, zero_blocks):
    x = tensor((1, 1, 1, n) if n < 200 else (1, n, 1, 1) if n % 16 else (n // 16, 1, 4, 4), n)
    ctx = gpu.Context(sub=sub, max_numel=n, zero_blocks=zero_blocks)
    buf, size, rc = ctx.compress(torch.from_numpy(x).cuda(), EB)
    assert rc == 0
    want, want_size = oracle(orc, x, sub, zero_blocks)
    assert size == want_size and np.array_equal(buf[:size].cpu().numpy(), want)


# all small, and one too large among them
@pytest.mark.parametrize("large", [False, True])
def test_batches(gpu, orc, large):
    shapes = [(2, 3, 20, 20), (1, 70, 61, 61), (1, 1, 1, 1), (3, 128, 28, 29)] + ([(5, 70, 61, 61)] if large else [])
    xs = [tensor(s, k) for k, s in enumerate(shapes)]
    ctx = gpu.Context(sub=32, max_numel=sum(-(-x.size // 4096) * 4096 for x in xs))
    bufs, sizes, rc = ctx.compress_batch([torch.from_numpy(x).cuda() for x in xs], [EB] * len(xs))
    assert rc == 0
    for x, buf, size in zip(xs, bufs, sizes):
        want, want_size = oracle(orc, x, 32, False)
        assert size == want_size and np.array_equal(buf[:size].cpu().numpy(), want)


# pops by launches of fewer and of more workgroups than the stack counts in parts, in and out of order
def test_stack(gpu):
    shapes = [(1, 3, 9, 9), (4, 64, 28, 28), (8, 100, 56, 57), (1, 1, 1, 3), (64, 33, 14, 14)]
    xs = [torch.from_numpy(tensor(s, k)).cuda() for k, s in enumerate(shapes)]
    ctx = gpu.Context(sub=32, max_numel=max(x.numel() for x in xs))
    cap = 1 << 24
    arena = torch.empty(cap, dtype=torch.uint8, device="cuda")
    state = torch.empty(gpu.cmp_arena_state_bytes(len(xs)), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    alone = []
    for x in xs:
        buf, size, _ = ctx.compress(x, EB)
        alone.append((ctx.decompress(buf, size, x.shape, EB), size))
    assert gpu.cmp_arena_init(ctx._h, state.data_ptr(), len(xs), stream) == 0
    for order in ([4, 3, 2, 1, 0], [0, 1, 2, 3, 4], [2, 4, 0, 3, 1]):
        for k, x in enumerate(xs):
            assert gpu.cmp_arena_push(ctx._h, arena.data_ptr(), cap, state.data_ptr(), k, x.data_ptr(), x.shape, EB, stream) == 0
        held = set(range(len(xs)))
        ends = np.cumsum([-(-size // 256) * 256 for _, size in alone])
        for k in order:
            y = torch.empty_like(xs[k])
            assert gpu.cmp_arena_pop(ctx._h, arena.data_ptr(), state.data_ptr(), k, xs[k].shape, EB, y.data_ptr(), stream) == 0
            held.discard(k)
            rc, top, peak, n, failed = gpu.cmp_arena_stats(ctx._h, state.data_ptr(), stream)
            assert rc == 0 and failed == 0 and n == (max(held) + 1 if held else 0)
            assert top == (ends[max(held)] if held else 0) and peak == ends[-1]
            assert torch.equal(y.view(torch.int32), alone[k][0].view(torch.int32))
    assert ctx.last_status() == 0


# the codebook: every count of used symbols around its blocks of 64 and of 256, and weights on both sides of what
# fits a key of 32 bits (2^25), with the same weights many times over
@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 128, 256, 257, 321, 1000])
def test_used_symbols(gpu, orc, n):
    rng = np.random.default_rng(n)
    step = np.float32(2) * (np.float32(EB) - np.float32(np.ldexp(np.float32(EB), -7)))
    counts = rng.choice([1, 2, 3, 5, 8, 13, 40], n)
    q = np.repeat(rng.permutation(np.arange(-(n // 2), n - n // 2)), counts)
    x = (rng.permutation(q) * step).astype(np.float32).reshape(1, -1, 1, 1)
    ctx = gpu.Context(sub=32, max_numel=x.size)
    buf, size, rc = ctx.compress(torch.from_numpy(x).cuda(), EB)
    want, want_size = oracle(orc, x, 32, False)
    assert rc == 0 and size == want_size and np.array_equal(buf[:size].cpu().numpy(), want)


def test_heavy_symbols(gpu, orc):
    step = float(np.float32(2) * (np.float32(EB) - np.float32(np.ldexp(np.float32(EB), -7))))
    x = np.zeros(9 << 22, np.float32)                                # 37.7 M elements, 2^24 and 2^22 of which another value
    x[:1 << 24] = step
    x[1 << 24:(1 << 24) + (1 << 22)] = -step
    x[-3000:] = step * np.random.default_rng(1).integers(-200, 200, 3000)
    x = x.reshape(1, -1, 1, 1)
    ctx = gpu.Context(sub=32, max_numel=x.size)
    buf, size, rc = ctx.compress(torch.from_numpy(x).cuda(), EB)
    want, want_size = oracle(orc, x, 32, False)
    assert rc == 0 and size == want_size and np.array_equal(buf[:size].cpu().numpy(), want)


# no used symbol at all (container version 2, nothing but zeros): the kernel has less to do than with two symbols.  Walking
# links that are not there took 10 us of 33
def test_no_used_symbol_costs_nothing(gpu, orc):
    us = {}
    for used in (0, 2):
        x = np.zeros((1, 1, 64, 64), np.float32)
        if used:
            x[0, 0, 3, 4] = 0.5
        t = torch.from_numpy(x).cuda()
        ctx = gpu.Context(sub=32, max_numel=x.size, zero_blocks=1)
        buf, size, rc = ctx.compress(t, EB)
        want, want_size = oracle(orc, x, 32, 1)
        assert rc == 0 and size == want_size and np.array_equal(buf[:size].cpu().numpy(), want)
        us[used] = float("inf")
        for _ in range(10):
            t0, t1 = torch.cuda.Event(True), torch.cuda.Event(True)
            t0.record()
            for _ in range(30):
                ctx.compress(t, EB, out=buf, sync=False)
            t1.record()
            torch.cuda.synchronize()
            us[used] = min(us[used], t0.elapsed_time(t1) * 1e3 / 30)
    print(us)
    assert us[0] < 1.2 * us[2], us
