"""GPU: the fused kernel of long segments (base product + 2:4 deltas on more than 64 rows, paper Section 5.1 Eq. (2),
Section 5.2), forced with DZ_OPT_WIDE_TILE = 2, at the edges of its tiles: 256 rows of N, 16 column blocks of 16 requests,
one or two segments a tile, k in tiles of 256 cut into slices of two tiles at least."""
import numpy as np
import pytest
import torch

import dz_synth as S
from dzcase import Case

pytestmark = pytest.mark.gpu


def _ids(lengths, base_rows=0):
    ids = np.concatenate([np.full(n, d, np.int32) for d, n in enumerate(lengths)] + [np.full(base_rows, -1, np.int32)])
    np.random.default_rng(9).shuffle(ids)
    return ids


CASES = [
    # name,           N,    K, bits, G, rows of each delta,              base-only rows
    ("one_k_tile",   256,  256, 4, 128, [256],                            0),
    ("over_a_tile",  272,  512, 4,  64, [257, 1, 15, 16, 17],             0),
    ("under_a_tile",  16, 1280, 2, 128, [240, 0, 255, 241, 33],           1),
    ("pairs",        528, 1024, 2,  64, [128, 128, 129, 127, 31, 225],   17),
    ("base_rows",    240, 2304, 4, 128, [100, 0],                       300),
    ("all_base",     256,  512, 4, 128, [0, 0],                          65),
    ("short",        304, 1024, 4, 128, [3, 1, 2, 0, 5, 1, 1, 60, 9],     4),
]


def _check(out, cs, x, ids, what):
    """Against 64 bits.  The kernel rounds a dequantised value to fp16 (2^-11 relative, 2^-25 among the subnormals), adds 2 K
    products and K / 128 partial sums in fp32 (2^-24 each), and rounds the result once (2^-11, 2^-25 among the subnormals)."""
    xd, W = x.double().numpy(), cs.W.double().numpy()
    y, mag, dmag = xd @ W.T, np.abs(xd) @ np.abs(W).T, np.zeros((cs.T, cs.N))
    for d, dense in enumerate(cs.dense):
        r, dd = np.flatnonzero(ids == d), np.asarray(dense, np.float64)
        y[r] += xd[r] @ dd.T
        dmag[r] = np.abs(xd[r]) @ np.abs(dd).T
    bound = (2.0 ** -11 * np.abs(y) + 2.0 ** -25 * (1 + np.abs(xd).sum(1, keepdims=True)) + 2.0 ** -11 * dmag
             + (2 * cs.K + cs.K / 128) * 2.0 ** -24 * (mag + dmag)) * 1.01
    err = np.abs(out.double().cpu().numpy() - y)
    assert (err <= bound).all(), f"{what}: {np.nanmax(err / bound):.2f} of the bound"


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_tile_edges(dz, case):
    name, N, K, bits, G, lengths, base = case
    print(f"fused {name}", flush=True)
    ids = _ids(lengths, base)
    with dz.Context(0) as c:
        cs = Case(dz, c.h, 31, len(ids), N, K, len(lengths), bits, G, ids)
        for route in (2, 0):                     # the fused kernel, and the narrower one on the same call
            c.set_option(dz.DZ_OPT_WIDE_TILE, route)
            o = cs.out(fill=7.0)
            dz.dz_linear(c.h, cs.dx, cs.dW, cs.packed, cs.dids, o, cs.T, N, K, bits, G)
            assert dz.dz_check(c.h) == dz.DZ_OK
            _check(o, cs, cs.x, ids, f"{name} route {route}")


def test_group_captured_and_replayed_with_other_segments(dz):
    """Projections of different N in one launch; the list of tiles is made on the device, so replays may bring other ids."""
    T, K, D, Ns = 400, 1024, 3, [272, 64, 256]
    print("fused group graph", flush=True)
    with dz.Context(0) as c:
        c.set_option(dz.DZ_OPT_WIDE_TILE, 2)
        cases = [Case(dz, c.h, 60 + p, T, N, K, D, 4, 128, _ids([200, 100, 50], 50)) for p, N in enumerate(Ns)]
        dx, dids, outs = cases[0].dx, cases[0].dids, [cs.out(fill=7.0) for cs in cases]

        def call():
            dz.dz_linear_group(c.h, dx, [cs.dW for cs in cases], [cs.packed for cs in cases], dids, outs, T, Ns, K, 4, 128)

        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call()
        for rep, (lengths, base) in enumerate([([400, 0, 0], 0), ([1, 17, 382], 0), ([0, 0, 0], 400), ([133, 133, 134], 0)]):
            x, ids = S.make_x(T, K, S.stream(90 + rep, "x")), _ids(lengths, base)
            dx.copy_(x)
            dids.copy_(torch.from_numpy(ids))
            for o in outs:
                o.fill_(7.0)
            graph.replay()
            assert dz.dz_check(c.h) == dz.DZ_OK
            for p, cs in enumerate(cases):
                _check(outs[p], cs, x, ids, f"replay {rep} projection {p}")


@pytest.mark.parametrize("bits,G", [(2, 64), (4, 64)])
def test_full_rounds_and_a_sliced_rest(dz, bits, G):
    """More tiles than CUs: whole ones first, then the tiles of the last round cut into slices of k of two and three k tiles."""
    from test_fused_plan import _list
    print(f"fused rounds {bits} {G}", flush=True)
    N, K, lengths = 8192, 1280, [20, 17, 1, 33, 16, 20, 30, 2, 9, 20, 20, 31, 32, 5, 20, 20, 28, 20]
    cus = torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    tiles = N // 256 * int(_list(lengths, 0)[0][0])
    assert tiles > cus and 0 < tiles % cus <= 64
    ids = _ids(lengths)
    with dz.Context(0) as c:
        c.set_option(dz.DZ_OPT_WIDE_TILE, 2)
        cs = Case(dz, c.h, 32, len(ids), N, K, len(lengths), bits, G, ids)
        for rep in range(2):                     # the arrival counters are ready again
            o = cs.out(fill=7.0)
            dz.dz_linear(c.h, cs.dx, cs.dW, cs.packed, cs.dids, o, cs.T, N, K, bits, G)
            assert dz.dz_check(c.h) == dz.DZ_OK
            _check(o, cs, cs.x, ids, f"rounds {rep}")


def test_captured_cold_and_replayed_after_the_workspace_grew(dz):
    """The first call of a context is a captured one: its slices of k fit the partial sums as dz_create made them (128 partial
    tiles; an eager call grows them and may cut finer).  Replays with other segments, before and after that growth."""
    T, N, K, D = 512, 4096, 4096, 2
    print("fused cold capture", flush=True)
    with dz.Context(0) as c:
        c.set_option(dz.DZ_OPT_WIDE_TILE, 2)
        cs = Case(dz, c.h, 33, T, N, K, D, 4, 128, _ids([300, 200], 12))
        dx, dids, o = cs.dx, cs.dids, cs.out(fill=7.0)

        def call():
            dz.dz_linear(c.h, dx, cs.dW, cs.packed, dids, o, T, N, K, 4, 128)

        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call()
        for rep, (lengths, base) in enumerate([([300, 200], 12), ([0, 512], 0), ([17, 1], 494)]):
            x, ids = S.make_x(T, K, S.stream(95 + rep, "x")), _ids(lengths, base)
            dx.copy_(x)
            dids.copy_(torch.from_numpy(ids))
            for what, f in (("replay", graph.replay), ("eager", call)):
                o.fill_(7.0)
                f()
                assert dz.dz_check(c.h) == dz.DZ_OK
                _check(o, cs, x, ids, f"{what} {rep}")


@pytest.mark.parametrize("case", [CASES[1], CASES[4], CASES[6]], ids=lambda c: c[0])
def test_list_of_an_order_that_another_kernel_s_call_made(dz, case):
    name, N, K, bits, G, lengths, base = case
    print(f"fused list {name}", flush=True)
    ids = _ids(lengths, base)
    with dz.Context(0) as c:
        cs = Case(dz, c.h, 34, len(ids), N, K, len(lengths), bits, G, ids)
        c.set_option(dz.DZ_OPT_REUSE_SEGMENTS, 1)
        for route in (0, 2, 0, 2):
            c.set_option(dz.DZ_OPT_WIDE_TILE, route)
            o = cs.out(fill=7.0)
            dz.dz_linear(c.h, cs.dx, cs.dW, cs.packed, cs.dids, o, cs.T, N, K, bits, G)
            assert dz.dz_check(c.h) == dz.DZ_OK
            _check(o, cs, cs.x, ids, f"{name} route {route}")
