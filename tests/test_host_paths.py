"""What the host side decides for a call, seen on a HIP runtime without a GPU (fake_hip.cpp): sorts, kernels, workspace."""
import sys

import pytest

import fake_hip as F


def captured_orders():
    """DZ_OPT_REUSE_SEGMENTS: an order that a capture recorded has not been made, so neither an eager call nor another
    capture may use it; nor may a graph rely on an order that eager calls make and overwrite."""
    s = F.Sim()
    s.option(F.REUSE_SEGMENTS, 1)
    layer = lambda: (s.linear([4096], 4096, 8, 300), s.linear([64] * 3, 4096, 8, 300))
    s.capture(7)
    assert layer() == (0, 0)
    assert s.kernels() == ["segment_kernel", "prefill_kernel", "prefill_kernel"], "one capture shares one sort"
    s.capture(8)
    assert layer() == (0, 0)
    assert s.kernels() == ["segment_kernel", "prefill_kernel", "prefill_kernel"], "another capture sorts again"
    s.capture(0)
    assert layer() == (0, 0)
    assert s.kernels() == ["segment_kernel", "prefill_kernel", "prefill_kernel"], "an eager call sorts again"
    s.capture(9)
    assert layer() == (0, 0)
    assert s.kernels() == ["segment_kernel", "prefill_kernel", "prefill_kernel"], "a graph sorts for itself"
    s.capture(0)
    # the tile list of the fused kernel: recorded by a capture, asked for by an eager call after one that needed none
    s.option(F.REUSE_SEGMENTS, 1)
    s.option(F.WIDE_TILE, 0)
    assert s.linear([4096], 4096, 8, 2048) == 0
    s.option(F.WIDE_TILE, 2)
    s.capture(10)
    assert s.linear([4096], 4096, 8, 2048) == 0
    s.capture(0)
    s.launches()
    assert s.linear([4096], 4096, 8, 2048) == 0
    assert s.kernels() == ["segment_kernel", "fused_kernel"], "the list has not been made"


def sorts_fit_lds():
    """Static and dynamic LDS of a sort together stay within what a launch may use without an attribute."""
    s, static = F.Sim(), F.static_lds("segment_kernel")
    for D in list(range(130)) + list(range(130, 8193, 11)) + [1014, 1022, 4059, 4091, 5412, 5455, 8118, 8119, 8183, 8192]:
        for T in (1, 65, 1025):
            assert s.segment(T, D) == 0
    for T in (65, 2048, 100000):                # with the tile list of the fused kernel
        for D in (1, 16, 127, 128):
            s.option(F.WIDE_TILE, 2)
            assert s.linear([256], 256, D, T) == 0
    sorts = [l for l in s.launches() if l[0] == "segment_kernel"]
    assert len(sorts) > 2000
    assert max(lds for _, _, lds, _ in sorts) + static <= 65536, (static, max(lds for _, _, lds, _ in sorts))


def memory_is_short():
    """The fused kernel asks for the partial sums it can use, once, and runs with fewer where there is no memory for them."""
    layer = ([5120] * 3, 5120, 16, 2048)
    for K, T, grows in ((5120, 2048, True), (512, 2048, False), (5120, 100, False)):
        s = F.Sim()
        s.option(F.WIDE_TILE, 2)
        before = s.fake.fake_live_bytes()
        assert s.linear([5120] * 3 if T > 100 else [64], K, 16, T) == 0
        assert s.fake.fake_live_bytes() - before == (128 << 20 if grows else 0), K     # (the replaced buffer stays)
    s = F.Sim()
    s.fake.fake_watch(b"fused_kernel", 6)       # the slots it may use
    assert s.linear(*layer) == 0 and s.launches()[-1][::3] == ("fused_kernel", 512)
    s = F.Sim()
    s.room((128 << 20) - 1)
    for _ in range(3):
        assert s.linear(*layer) == 0
        assert s.launches()[-1][::3] == ("fused_kernel", 128)
    assert s.fake.fake_refused() == 1 and s.dz.dz_last_hip_error(s.ctx) == b""
    s = F.Sim()
    s.room(1 << 40)
    s.capture(3)
    assert s.linear(*layer) == 0 and s.launches()[-1][::3] == ("fused_kernel", 128)
    s.capture(0)
    assert s.linear(*layer) == 0 and s.launches()[-1][::3] == ("fused_kernel", 512)
    # a call that cannot do without fails, and leaves the context as it was
    s = F.Sim()
    s.room(0)
    s.option(F.SPLIT_K, 16)
    assert s.linear([11008], 8192, 4, 1024) == -5
    s.option(F.SPLIT_K, 0)
    s.launches()
    assert s.linear([4096], 4096, 4, 100) == 0 and s.kernels() == ["segment_kernel", "prefill_kernel"]


def a_layer_shares_one_sort():
    """DZ_OPT_REUSE_SEGMENTS: one sort serves the calls of a layer, whichever kernels they take and in whichever order; the
    list of the fused kernel is made once, with the sort or from it, and only where a call wants it."""
    s = F.Sim()
    seven_b = [([4096] * 3, 4096, "prefill_kernel"), ([4096], 4096, "prefill_kernel"), ([11008] * 2, 4096, "fused_kernel"),
               ([4096], 11008, "prefill_kernel")]
    for calls, at in ((seven_b + seven_b[2:], 2), (seven_b[2:] + seven_b, 0), (seven_b[:2], 9)):
        s.option(F.REUSE_SEGMENTS, 1)
        for Ns, K, _ in calls:
            assert s.linear(Ns, K, 8, 2048) == 0
        want = [k for _, _, k in calls]
        assert s.kernels() == ["segment_kernel"] + (want if at in (0, 9) else want[:at] + ["fused_list_kernel"] + want[at:])
    # routes that change between the calls: the list of tiles is made when it is first wanted
    s.option(F.REUSE_SEGMENTS, 1)
    for tile, kernels in ((0, ["segment_kernel", "prefill_kernel"]), (2, ["fused_list_kernel", "fused_kernel"]),
                          (0, ["prefill_kernel"]), (2, ["fused_kernel"])):
        s.option(F.WIDE_TILE, tile)
        assert s.linear([4096], 4096, 8, 2048) == 0
        assert s.kernels() == kernels


def growths_are_not_used_up():
    """A context may grow the sorted order from 4096 rows to the most that x can have, the fused kernel's partial sums, and
    the adapters' buffer 44 times.  The partial sums grow once, whatever the sizes of the calls."""
    s, T = F.Sim(), 4097
    s.option(F.WIDE_TILE, 2)
    before = s.fake.fake_live_bytes()
    for N in range(4096, 16384, 256):
        assert s.linear([N], 4096, 1, 512) == 0
    assert s.fake.fake_live_bytes() - before == 128 << 20
    s.option(F.WIDE_TILE, 0)
    while T < 1 << 22:
        assert s.linear([16], 256, 1, T) == 0, T
        T = 2 * T + 1
    rows = 8
    for i in range(45):
        assert s.lora(rows) == 0, i
        rows = rows * 5 // 4 + 1


@pytest.mark.parametrize("scenario", [captured_orders, sorts_fit_lds, memory_is_short, a_layer_shares_one_sort, growths_are_not_used_up], ids=lambda f: f.__name__)
def test_host(scenario, tmp_path):
    F.run(__file__, scenario.__name__, tmp_path)


if __name__ == "__main__":
    globals()[sys.argv[1]]()
