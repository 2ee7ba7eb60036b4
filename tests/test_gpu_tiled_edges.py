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
BASE = [(65, 16, 256), (65, 16, 1024), (128, 272, 4096), (130, 3088, 2048), (500, 11024, 1024), (1000, 6160, 1024),
        (1000, 8208, 256), (1000, 11024, 256), (1500, 8208, 256), (1500, 11024, 2048), (2049, 272, 2048), (2049, 8208, 1024)]


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
