"""GPU: the compressor and the pack and merge kernels where they can go wrong: quotients that are exact halves,
infinite ranges, tables at odd addresses, an odd number of row tiles and k tiles, signed zeros."""
import numpy as np
import pytest
import torch

import dz_synth as S
import oracle

pytestmark = pytest.mark.gpu

FORMATS = [(4, 64), (4, 128), (2, 64), (2, 128)]


def _odd(n, dtype, off):
    """A tensor of n values whose first byte is `off` bytes past an aligned address, and its guarded buffer."""
    size = torch.empty(0, dtype=dtype).element_size()
    buf = torch.full((n * size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    return buf[off:off + n * size].view(dtype) if off % size == 0 else None, buf


def _delta(N, K, bits, G):
    """Rows of several kinds: random; multiples of half a grid step, so that most quotients are exact halves;
    subnormal; one with infinities of both signs; signed zeros; equal magnitudes."""
    d = S._normal_f16((N, K), 0.002, S.stream(31, "edges", N, K, bits, G)).numpy().copy()
    top = (1 << bits) - 1
    rng = np.random.default_rng(5)
    half = rng.integers(-top, top + 1, size=K)              # in half steps; the range is exactly `top` steps
    half[::G] = top
    half[1::G] = -top
    d[1] = (half * 0.5 * 2.0 ** -9).astype(np.float16)
    d[2] = (rng.integers(-40, 41, size=K) * 2.0 ** -24).astype(np.float16)
    d[3, 5] = np.inf
    d[3, G + 9] = -np.inf
    d[4] = 0.0
    d[4, ::3] = -0.0
    d[5] = np.where(rng.integers(0, 2, K) > 0, 0.25, -0.25)
    d[6] *= 3e4                                              # ranges that overflow fp16's scale do not occur here, large steps do
    d[7, :] = np.float16(65504)
    d[7, 1::2] = np.float16(-65504)
    return d


@pytest.mark.parametrize("bits,G", FORMATS)
@pytest.mark.parametrize("off", [0, 1])
def test_compress_and_pack_bit_for_bit(dz, bits, G, off):
    N, K = 48, 768                                          # three row tiles, three k tiles: blocks of four tiles end inside
    print(f"case bits={bits} G={G} off={off}", flush=True)
    d = _delta(N, K, bits, G)
    with np.errstate(all="ignore"):
        wc, wi, ws, wz = oracle.compress_.compress(d, bits, G)
    wc = np.where(np.isinf(np.repeat(ws, G // 2, axis=1)), 0, wc)        # an infinite scale: every code is 0
    wz = np.where(np.isinf(ws), np.float16(0), wz)
    dd = torch.from_numpy(d).cuda()
    src = torch.empty(N * K + 8, dtype=torch.float16, device="cuda")[4 * off:4 * off + N * K]    # 8-byte aligned is enough
    src.copy_(dd.view(-1))
    codes, cb = _odd(N * K // 2, torch.uint8, off)
    idx, ib = _odd(N * K // 2, torch.uint8, off)
    scale, sb = _odd(N * K // G, torch.float16, 2 * off)
    zero, zb = _odd(N * K // G, torch.float16, 2 * off)
    with dz.Context(0) as c:
        dz.dz_compress_delta(c.h, src, N, K, bits, G, codes, idx, scale, zero)
        packed = torch.zeros(dz.dz_packed_bytes(N, K, bits, G) + 64, dtype=torch.uint8, device="cuda")
        dz.dz_pack_delta(c.h, codes, idx, scale, zero, N, K, bits, G, packed)
        back = [torch.empty_like(t) for t in (codes, idx, scale, zero)]
        dz.dz_unpack_delta(c.h, packed, N, K, bits, G, *back, None)
        torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy().reshape(wi.shape), wi)
    assert np.array_equal(scale.cpu().numpy().view(np.uint16), ws.view(np.uint16).ravel())
    assert np.array_equal(zero.cpu().numpy().view(np.uint16), wz.view(np.uint16).ravel())
    assert np.array_equal(codes.cpu().numpy().reshape(wc.shape), wc)
    for got, want in zip(back, (codes, idx, scale, zero)):
        assert torch.equal(got.view(torch.uint8), want.view(torch.uint8))
    assert not packed[-64:].any()
    for buf, n in ((cb, N * K // 2), (ib, N * K // 2)):
        assert (buf[:off] == 0xA5).all() and (buf[off + n:] == 0xA5).all()
    for buf, n in ((sb, 2 * N * K // G), (zb, 2 * N * K // G)):
        assert (buf[:2 * off] == 0xA5).all() and (buf[2 * off + n:] == 0xA5).all()


@pytest.mark.parametrize("bits,G", FORMATS)
def test_merge_bit_for_bit(dz, bits, G):
    """f16 of the fp32 sum, element by element; W holds signed zeros, infinities and large values too."""
    N, K = 80, 1280
    print(f"case bits={bits} G={G}", flush=True)
    t = S.make_delta_tables(N, K, bits, G, S.stream(33, "merge", bits, G))
    W = S.make_base(N, K, S.stream(33, "W")).clone()
    W[0, ::2] = -0.0
    W[1, ::7] = float("inf")
    W[2] = 65504.0
    dense = oracle.c.dequant(t.codes.numpy(), t.idx.numpy(), t.scale.numpy(), t.zero.numpy(), bits, G)
    with np.errstate(over="ignore"):
        want = (W.numpy().astype(np.float32) + dense + np.float32(0)).astype(np.float16)
    d = t.to("cuda")
    with dz.Context(0) as c:
        packed = torch.empty(dz.dz_packed_bytes(N, K, bits, G), dtype=torch.uint8, device="cuda")
        dz.dz_pack_delta(c.h, d.codes, d.idx, d.scale, d.zero, N, K, bits, G, packed)
        buf = torch.full(((N + 2) * K,), 7.0, dtype=torch.float16, device="cuda")
        dz.dz_merge_delta(c.h, W.cuda(), packed, N, K, bits, G, buf[K:-K])
        torch.cuda.synchronize()
    got = buf[K:-K].cpu().numpy().reshape(N, K)
    assert np.array_equal(got.view(np.uint16), want.view(np.uint16))
    assert (buf[:K] == 7).all() and (buf[-K:] == 7).all()


@pytest.mark.parametrize("T,N,K,r", [(1, 4, 8, 8), (3, 132, 6152, 64), (5, 1028, 2048, 40)])
def test_lora_reduction_over_lanes_and_waves(dz, T, N, K, r):
    """k that fills one lane, three passes and a rest, and exactly one pass of the four waves."""
    print(f"case T={T} K={K} r={r}", flush=True)
    from dzcase import assert_close
    x = S.make_x(T, K, S.stream(34, "x"))
    A = [S.make_base(r, K, S.stream(34, "A", m), 0.05) for m in range(2)]
    B = [S.make_base(N, r, S.stream(34, "B", m), 0.05) for m in range(2)]
    ids = torch.arange(T, dtype=torch.int32) % 2
    want = oracle.lora.lora_sbmm(x.numpy(), [a.numpy() for a in A], [b.numpy() for b in B], ids.numpy())
    with dz.Context(0) as c:
        out = torch.full((T, N), 7.0, dtype=torch.float16, device="cuda")
        dz.dz_lora_sbmm(c.h, x.cuda(), [a.cuda() for a in A], [b.cuda() for b in B], r, ids.cuda(), out, T, N, K, 0)
        torch.cuda.synchronize()
        assert_close(out, want, "lora")


@pytest.mark.parametrize("bits,G", FORMATS)
def test_compress_takes_a_nan_for_the_largest_magnitude(dz, bits, G):
    """A NaN (quiet or signalling, either sign) is kept, stores code 0 and leaves the rest of its group as it is: the same
    tables as with a value inside the group's range in its place that is the largest of its four."""
    N, K = 16, 512
    print(f"case bits={bits} G={G}", flush=True)
    d = S._normal_f16((N, K), 0.002, S.stream(35, "nan", bits, G)).numpy().copy()
    d[:, 0::G] = 0.02                                        # the range of every group, in its first and third four
    d[:, 8::G] = -0.02
    cols = np.arange(4, K, G) + np.arange(K // G) % 4        # one entry of the second four, each position in turn
    stand = d.copy()
    stand[:, cols] = 0.0175
    d.view(np.uint16)[:, cols] = np.resize(np.array([0x7e00, 0x7d01, 0xfe00, 0xfdff], np.uint16), (N, len(cols)))
    wc, wi, ws, wz = oracle.compress_.compress(stand, bits, G)
    slot = (cols // 4) * 2                                   # the two kept entries of the four that holds the NaN
    at = cols % 4
    wc = wc.copy()
    for s, p in zip(slot, at):
        for j in range(2):
            wc[:, s + j] = np.where(wi[:, s + j] == p, 0, wc[:, s + j])
        assert ((wi[:, s] == p) | (wi[:, s + 1] == p)).all()
    out = [torch.empty(N * n, dtype=t, device="cuda") for n, t in ((K // 2, torch.uint8), (K // 2, torch.uint8),
                                                                   (K // G, torch.float16), (K // G, torch.float16))]
    with dz.Context(0) as c:
        dz.dz_compress_delta(c.h, torch.from_numpy(d).cuda(), N, K, bits, G, *out)
        torch.cuda.synchronize()
    for got, want in zip(out, (wc, wi, ws, wz)):
        got = got.cpu().numpy().reshape(want.shape)
        assert np.array_equal(got.view(np.uint8), np.ascontiguousarray(want).view(np.uint8).reshape(got.view(np.uint8).shape))
