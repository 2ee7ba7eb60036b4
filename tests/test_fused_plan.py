"""Host side of the fused kernel of long segments: the list of column tiles that a sort leaves, and the rule that picks the
kernel (no GPU)."""
import ctypes

import numpy as np
import pytest

import fake_hip as F

BLOCKS = 16


def _list(lengths, base):
    import paper_2312_05215_amd as dz
    D, T = len(lengths), int(sum(lengths)) + base
    start = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    most = dz.lib().dz_fused_list(None, T, D, None)
    out = np.full((1 + most + 1, 8), -99, np.int32)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    assert dz.lib().dz_fused_list(ptr(start), T, D, ptr(out)) == most
    assert (out[-1] == -99).all() and out[0, 0] <= most, (lengths, base)
    return out[0], out[1:1 + out[0, 0]], start, T


def _cost(blocks):
    return 11 if blocks < 5 else (blocks + 1) // 2 * 2 + 6


def _vectors():
    yield from ([[n], base] for n in (1, 15, 16, 17, 240, 255, 256, 257, 272, 273, 511, 512, 513, 4097) for base in (0, 1, 300))
    yield from ([[0] * d, base] for d in (1, 2, 128) for base in (1, 65, 5000))
    yield from ([[n] * d, base] for n in (1, 16, 17, 33, 120, 128, 129, 145, 160, 161, 257, 273) for d in (1, 2, 3, 127, 128)
                for base in (0, 17))
    rng = np.random.default_rng(5)
    for i in range(4000):
        D = int(rng.integers(1, 129))
        top = int(2 ** rng.uniform(0, 10.5))
        lengths = rng.integers(0, top + 1, D) * (rng.random(D) < rng.uniform(0.2, 1.0))
        yield [int(n) for n in lengths], int(rng.choice([0, 1, rng.integers(0, 2000)]))


def test_every_row_is_in_one_tile_of_its_delta():
    for lengths, base in _vectors():
        if sum(lengths) + base == 0:
            continue
        head, tiles, start, T = _list(lengths, base)
        D, at, dearest = len(lengths), 0, 0
        for s0, r0, k0, s1, r1, k1, _, _ in tiles.tolist():
            first = (r0 + 31) // 32 * 2 if r1 else (r0 + 15) // 16         # a second segment begins at an even block
            blocks = first + (r1 + 15) // 16
            assert r0 > 0 and r1 >= 0 and blocks <= BLOCKS, (lengths, base)
            dearest = max(dearest, _cost(blocks))
            for s, r, k in ((s0, r0, k0), (s1, r1, k1))[:2 if r1 else 1]:
                assert s == at and 0 <= k <= D, (lengths, base)
                assert start[k] <= s and s + r <= (start[k + 1] if k < D else T), (lengths, base)
                at += r
            assert not (r1 and D in (k0, k1)), (lengths, base)              # rows of the base model share no tile
        assert at == T and head[1] == dearest, (lengths, base)


# name, output sizes, K, D, T, fused
ROUTES = [
    ("13b_qkv", [5120] * 3, 5120, 16, 2048, 1), ("13b_o", [5120], 5120, 16, 2048, 1), ("13b_gate_up", [13824] * 2, 5120, 16, 2048, 1),
    ("13b_down", [5120], 13824, 16, 2048, 1), ("13b_gate", [13824], 5120, 16, 2048, 1),
    ("fewer_than_128_rows_a_delta", [5120] * 3, 5120, 16, 2047, 0),
    ("7b_gate_up", [11008] * 2, 4096, 8, 2048, 1), ("7b_qkv", [4096] * 3, 4096, 8, 2048, 0), ("7b_777", [11008] * 2, 4096, 3, 777, 0),
    ("mixed", [4096], 4096, 8, 200, 0), ("no_delta", [13824] * 2, 5120, 0, 2048, 0),
]


@pytest.mark.parametrize("route", ROUTES, ids=[r[0] for r in ROUTES])
def test_the_rule(route):
    import paper_2312_05215_amd as dz
    _, Ns, K, D, T, fused = route
    assert dz.lib().dz_fused_route(len(Ns), (ctypes.c_int * len(Ns))(*Ns), T, K, D, 256) == fused


def test_the_benchmark_names_the_kernel_that_runs_and_its_traffic():
    import bench
    import dz_synth as S
    cfg = S.config("13b_prefill")
    projs = S.projections_of(cfg)
    for groups, MB in ((S.launch_groups(cfg), 2140), ([[i] for i in range(len(projs))], 1107)):
        launches = [([projs[i][1] for i in g], projs[g[0]][2]) for g in groups]
        kernel = bench.tiled_kernel(launches, cfg.T, cfg.D, 256)
        assert kernel == "fused_kernel"
        traffic, src = bench.profile_traffic(kernel, cfg.name, len(launches))
        assert src == "profiles/fused_kernel_13b_prefill_pmc.txt" and traffic // 10 ** 6 == MB
    both = bench.tiled_kernel([([11008] * 2, 4096), ([4096], 4096)], 2048, 8, 256)
    assert both == "fused_kernel and prefill_kernel"
    assert bench.profile_traffic(both, cfg.name, 4) == (None, None)


def launched():
    """The calls of test_gpu_fused.py and of ROUTES launch the kernel that they are about."""
    data = F.data()
    s = F.Sim()
    for Ns, K, D, T, fused in data["routes"]:
        assert s.linear(Ns, K, D, T) == 0
        assert s.kernels()[-1] == ("fused_kernel" if fused else "prefill_kernel" if D else "tile_kernel"), (Ns, K, D, T)
    for N, K, bits, G, D, T in data["cases"]:
        for tile, kernel in ((2, "fused_kernel"), (0, "prefill_kernel")):
            s.option(F.WIDE_TILE, tile)
            assert s.linear([N], K, D, T, bits, G) == 0
            assert s.kernels() == ["segment_kernel", kernel], (N, K, D, T)
    s.option(F.WIDE_TILE, 2)
    assert s.linear([272, 64, 256], 1024, 3, 400) == 0 and s.kernels()[-1] == "fused_kernel"
    assert s.linear([256], 256, 3, 64) == 0 and s.kernels() == ["stream_kernel"]
    assert s.linear([131072], 8192, 3, 65) == 0 and s.kernels()[-1] == "prefill_kernel"       # W of 2 GiB
    s.option(F.SPLIT_K, 1)
    assert s.linear([256], 256, 3, 65) == 0 and s.kernels()[-1] == "prefill_kernel"


def test_launched(tmp_path):
    from test_gpu_fused import CASES
    cases = [(N, K, bits, G, len(lengths), sum(lengths) + base) for _, N, K, bits, G, lengths, base in CASES]
    F.run(__file__, "launched", tmp_path, dict(routes=[r[1:] for r in ROUTES], cases=cases))


if __name__ == "__main__":
    import sys
    globals()[sys.argv[1]]()
