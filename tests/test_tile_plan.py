"""Host side of the wide kernel of the base product: which tile shape and how many slices of k a call gets (no GPU)."""
import ctypes

from test_gpu_tiled_edges import BASE, BASE_GROUPS

# waves along the rows, row tiles and column blocks of a wave
SHAPES = {(4, 4, 8), (4, 4, 7), (4, 4, 6), (4, 4, 5), (4, 4, 4), (2, 7, 4), (2, 6, 4), (2, 5, 4)}


def _plan(Ns, T, K, cus=256):
    import paper_2312_05215_amd as dz
    out = (ctypes.c_int * 6)()
    dz.lib().dz_tile_plan(len(Ns), (ctypes.c_int * len(Ns))(*Ns), T, K, cus, out)
    return list(out)


def _sides(shape):
    twr, trt, tj = shape
    return twr * trt * 16, 8 // twr * tj * 16


def test_the_base_product_sizes_reach_every_shape_whole_and_sliced():
    whole, sliced, ragged = set(), set(), set()
    for T, N, K in BASE:
        *shape, S, _, _ = _plan([N], T, K)
        shape = tuple(shape)
        (sliced if S > 1 else whole).add(shape)
        rows, cols = _sides(shape)
        if N % rows and T % cols:
            ragged.add((shape, S > 1))
    assert whole == SHAPES and sliced == SHAPES
    assert ragged == {(s, k) for s in SHAPES for k in (False, True)}


def test_plans_cover_the_call():
    """Every tile is whole or sliced, slices are at least two k tiles, their partial tiles fit 64 MB and one round."""
    for T, Ns, K in [(T, [N], K) for T, N, K in BASE] + BASE_GROUPS + [(T, [N] * P, K) for T in (65, 129, 777, 4096)
                                                                     for N in (16, 1040, 28672) for P in (1, 3) for K in (256, 8192)]:
        for cus in (256, 248, 64):
            *shape, S, whole, tiles = _plan(Ns, T, K, cus)
            rows, cols = _sides(shape)
            assert tiles == sum(-(-N // rows) for N in Ns) * -(-T // cols)
            assert tuple(shape) in SHAPES and 0 <= whole <= tiles
            if S == 1:
                assert whole == tiles
            else:
                left = (tiles - whole + 7) // 8 * 8
                assert whole % cus == 0 and left * S <= cus and K // 256 >= 2 * S
                assert left * S * shape[1] * shape[2] * 512 * 16 <= 64 << 20
