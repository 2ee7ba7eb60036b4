"""GPU: dz_segment where its runs of requests can go wrong: one wave's run, several, the last one short or empty, more
keys than fit more than one histogram, every request the same key, all idle, indices out of range in a late run."""
import numpy as np
import pytest
import torch

import dz_synth as S
from test_gpu_segment import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [1, 2, 63, 64, 127, 128, 1023, 4000, 8192])
@pytest.mark.parametrize("T", [1, 63, 64, 65, 128, 1023, 1025, 3000])
def test_runs(dz, T, D):
    print(f"case T={T} D={D}", flush=True)
    with dz.Context(0) as c:
        ids = S.ids_uniform(T, D, S.stream(61, "r", T, D)).numpy().copy()
        ids[::5] = -1
        _run(dz, c, ids, D)
        _run(dz, c, np.full(T, D - 1), D)
        _run(dz, c, np.full(T, -1), D)
        assert dz.dz_check(c.h) == dz.DZ_OK
        ids[T - 1] = D
        _run(dz, c, ids, D)
        assert dz.dz_check(c.h) == dz.DZ_ERR_INDEX


def test_a_prefix_sum_over_many_keys_is_shared_by_the_waves(dz):
    """One request over 8192 keys takes less than four calls over one key (a prefix sum walked by one wave alone: seven);
    the best of several runs of back-to-back calls."""
    with dz.Context(0) as c:
        ids = torch.zeros(1, dtype=torch.int32, device="cuda")
        perm = torch.empty(1, dtype=torch.int32, device="cuda")
        best = {}
        for rep in range(6):
            for D in (1, 8192):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                for i in range(51):
                    if i == 1:
                        a.record()
                    dz.dz_segment(c.h, ids, 1, D, None, None, perm)
                b.record()
                torch.cuda.synchronize()
                best[D] = min(best.get(D, 1e9), a.elapsed_time(b) * 20)
        print(f"us a call: {best}", flush=True)
        assert best[8192] < 4 * best[1], best


@pytest.mark.parametrize("T,D", [(1025, 1014), (1025, 1022), (3000, 4091), (128, 8183)])
def test_histograms_that_fill_lds(dz, T, D):
    """Numbers of keys whose histograms leave next to nothing of the 64 KB that a launch may use."""
    print(f"case T={T} D={D}", flush=True)
    with dz.Context(0) as c:
        _run(dz, c, S.ids_uniform(T, D, S.stream(62, "r", T, D)).numpy(), D)
        assert dz.dz_check(c.h) == dz.DZ_OK
