"""GPU: the tiled kernels at the edges of their tiles: several projections in one launch whose rows end inside a row
block, batches just over a tile of request rows, few tiles cut into many slices of k, k too short to be cut."""
import pytest
import torch

import oracle
from dzcase import Case, assert_close

pytestmark = pytest.mark.gpu

GROUPS = [
    # T,   K,    D, bits, G,  ids,       N of each projection
    (65,   256,  3, 4, 128, "uniform",  [16, 272]),            # one row past the streaming kernel, one k tile
    (129,  768,  5, 2, 64,  "zipf",     [272, 48, 128, 16]),   # one row in the second tile; three k tiles
    (70,   8192, 3, 4, 64,  "uniform",  [32]),                 # a single tile: sixteen slices of two k tiles
    (200,  4608, 2, 2, 128, "segments", [288, 80]),            # eighteen k tiles in nine slices
    (300,  512,  1, 4, 64,  "segments", [528]),                # every row names the one delta
]


@pytest.mark.parametrize("group", GROUPS, ids=[f"T{g[0]}K{g[1]}" for g in GROUPS])
@pytest.mark.parametrize("idle", [False, True])
def test_group_of_projections_in_one_tiled_launch(dz, group, idle):
    T, K, D, bits, G, ids, Ns = group
    print(f"case T={T} K={K} N={Ns} idle={idle}", flush=True)
    with dz.Context(0) as c:
        cases = [Case(dz, c.h, 50 + p, T, N, K, D, bits, G, ids) for p, N in enumerate(Ns)]
        x, idv = cases[0].x, cases[0].ids.clone()
        if idle:
            idv[::3] = -1
            idv[T - 1] = -1
        dids = idv.cuda()
        for repeat in range(2):                # the arrival counters are back at zero after a call
            outs = [torch.full((T + 2, N), 7.0, dtype=torch.float16, device="cuda") for N in Ns]
            dz.dz_linear_group(c.h, cases[0].dx, [cs.dW for cs in cases], [cs.packed for cs in cases], dids,
                               [o[1:-1] for o in outs], T, Ns, K, bits, G)
            assert dz.dz_check(c.h) == dz.DZ_OK
            for o, cs in zip(outs, cases):
                want = oracle.c.linear(x.numpy(), cs.W.numpy(), cs.dense, idv.numpy())
                assert_close(o[1:-1], want, f"N={cs.N}")
                assert (o[0] == 7).all() and (o[-1] == 7).all()


# sizes that take each tile shape of the base product in turn, whole and in slices of k, with ragged last tiles
# (tests/test_tile_plan.py checks that they do)
BASE = [(65, 16, 256), (65, 16, 1024), (128, 272, 4096), (130, 3088, 2048), (500, 11024, 1024), (1000, 6160, 1024),
        (1000, 8208, 256), (1000, 11024, 256), (1500, 8208, 256), (1500, 11024, 2048), (2049, 272, 2048), (2049, 8208, 1024),
        (161, 1296, 4096), (385, 10960, 1024), (641, 336, 4096), (641, 13072, 256), (641, 13616, 256), (1000, 13104, 256),
        (2049, 2832, 1536), (2049, 6416, 256)]


@pytest.mark.parametrize("T,N,K", BASE)
def test_base_product_tile_shapes(dz, T, N, K):
    """Against torch in fp32: half a unit of fp16 in the last place, 4.9e-4, and the order of the fp32 sums."""
    print(f"case T={T} N={N} K={K}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + N + K)
    x = torch.randn(T, K, generator=gen, device="cuda").half()
    W = (torch.randn(N, K, generator=gen, device="cuda") * 0.02).half()
    want = x.float() @ W.float().t()
    buf = torch.full((T + 2, N), 7.0, dtype=torch.float16, device="cuda")
    with dz.Context(0) as c:
        for repeat in range(2):
            buf[1:-1] = 7.0
            dz.dz_base_gemm(c.h, x, W, buf[1:-1], T, N, K)
            rms = want.pow(2).mean().sqrt()
            off = ((buf[1:-1].float() - want).abs() / torch.maximum(want.abs(), rms)).max().item()
            assert off < 1e-3, off
            assert (buf[0] == 7).all() and (buf[-1] == 7).all()


# several base products in one launch: rows that end inside a row block, the second projection's first block, one k tile
BASE_GROUPS = [(65, [16, 272], 256), (130, [1040, 4096, 80], 2048), (300, [48, 16, 528, 2064], 1536), (777, [5120, 5120], 2048)]


@pytest.mark.parametrize("T,Ns,K", BASE_GROUPS, ids=[f"T{T}P{len(Ns)}K{K}" for T, Ns, K in BASE_GROUPS])
@pytest.mark.parametrize("opts", [{}, {"DZ_OPT_SPLIT_K": 1}, {"DZ_OPT_SPLIT_K": 3}, {"DZ_OPT_WIDE_TILE": 0},
                                  {"DZ_OPT_WIDE_TILE": 0, "DZ_OPT_SPLIT_K": 3}], ids=["default", "whole", "splits3", "narrow", "narrow_splits3"])
def test_group_of_base_products(dz, T, Ns, K, opts):
    """dz_linear_group without deltas.  Against torch in fp32: half a unit of fp16 in the last place, 4.9e-4, and the order of
    the fp32 sums; with the number of k slices given the sums have one order, and the group equals dz_base_gemm bit for bit."""
    print(f"case T={T} N={Ns} K={K} {opts}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + K)
    x = torch.randn(T, K, generator=gen, device="cuda").half()
    W = [(torch.randn(N, K, generator=gen, device="cuda") * 0.02).half() for N in Ns]
    with dz.Context(0) as c:
        for k, v in opts.items():
            c.set_option(getattr(dz, k), v)
        for repeat in range(2):                # the arrival counters are back at zero after a call
            outs = [torch.full((T + 2, N), 7.0, dtype=torch.float16, device="cuda") for N in Ns]
            dz.dz_linear_group(c.h, x, W, [[] for _ in Ns], None, [o[1:-1] for o in outs], T, Ns, K, 4, 128)
            for o, w, N in zip(outs, W, Ns):
                want = x.float() @ w.float().t()
                off = ((o[1:-1].float() - want).abs() / torch.maximum(want.abs(), want.pow(2).mean().sqrt())).max().item()
                assert off < 1e-3, (N, off)
                assert (o[0] == 7).all() and (o[-1] == 7).all()
                if "DZ_OPT_SPLIT_K" in opts:
                    alone = torch.empty(T, N, dtype=torch.float16, device="cuda")
                    dz.dz_base_gemm(c.h, x, w, alone, T, N, K)
                    assert torch.equal(o[1:-1], alone), N


@pytest.mark.parametrize("T,Ns,K", [(777, [5120, 5120], 2048), (300, [11008, 11008], 4096)])
def test_group_of_base_products_goes_to_the_wide_kernel(dz, T, Ns, K):
    """On 256 compute units the wide kernel's 256 x 160 tiles (200 and 172 of them) fill the last round well enough to run
    whole, while the narrower kernel has 280 and 258 tiles and cuts those of its second round into four and eight slices of
    k.  So the default result has the bits of the unsliced one only if it came from the wide kernel."""
    print(f"case T={T} N={Ns} K={K}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn(T, K, generator=gen, device="cuda").half()
    W = [(torch.randn(N, K, generator=gen, device="cuda") * 0.02).half() for N in Ns]
    outs = {}
    for splits in (0, 1):
        with dz.Context(0) as c:
            c.set_option(dz.DZ_OPT_SPLIT_K, splits)
            outs[splits] = [torch.full((T, N), 7.0, dtype=torch.float16, device="cuda") for N in Ns]
            dz.dz_linear_group(c.h, x, W, [[] for _ in Ns], None, outs[splits], T, Ns, K, 4, 128)
            torch.cuda.synchronize()
    for a, b in zip(outs[0], outs[1]):
        assert torch.equal(a, b)
