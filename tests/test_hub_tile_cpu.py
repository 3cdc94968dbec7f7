"""Host-side checks of the work items of the Hubbard steps over one triangle."""


def test_items_hold_no_more_tiles_than_a_cluster_has():
    """The launch takes the LDS of its largest item for all of them."""
    from paper_2002_12717_amd import binding
    per = binding.load().hub_tile_per_item
    for ns in range(1, 65):
        for most in (1, 512, 768, 1024, 4096):
            p = per(ns, most)
            assert 1 <= p <= ns * (ns + 1) // 2
            assert p == 1 or (p * ns * ns <= min(most, 1024) and ns < 44)
    assert [per(ns, 4096) for ns in (1, 2, 3, 7, 8, 9, 16, 25, 33, 64)] == [1, 3, 6, 14, 12, 12, 4, 1, 1, 1]


def test_systems_that_take_the_triangle():
    """Clusters below the least size of a closure must not hold the larger part, and
    mixed TPP with more than two neighbours needs 7 x 2^18 elements where clusters of 26
    to 36 sites hold it."""
    import ctypes

    from paper_2002_12717_amd import binding as B
    lib = B.load()
    lib.hub_tile_pays.argtypes = [ctypes.c_int] * 3 + [ctypes.c_longlong] * 3

    def takes(se, mixed, z, sizes):
        small = sum(n ** 4 for n in sizes if n < lib.hub_tile_least(se))
        single = sum(n ** 4 for n in sizes if 26 <= n <= 36)
        return bool(lib.hub_tile_pays(se, mixed, z, sum(n ** 4 for n in sizes), small, single))
    for se in (B.SOA, B.TPH):
        assert takes(se, 0, 2, [2] * 70000) and takes(se, 1, 2, [4] * 5000)
    assert not takes(B.TPP, 0, 2, [7] * 500) and takes(B.TPP, 0, 2, [8] * 300)
    assert not takes(B.DSL, 1, 2, [4] * 5000) and takes(B.DSL, 1, 2, [5] * 2000)
    assert not takes(B.GW, 0, 2, [4] * 5000) and takes(B.GW, 0, 2, [5] * 2000)
    assert takes(B.TPP, 0, 4, [36] + [4] * 1500)            # the larger part is the 36-site cluster
    assert not takes(B.TPP, 0, 4, [36] + [4] * 7000)
    assert not takes(B.TPP, 1, 4, [36]) and takes(B.TPP, 0, 4, [36]) and takes(B.TPP, 1, 2, [36])
    assert takes(B.TPP, 1, 4, [37]) and takes(B.TPP, 1, 4, [32, 32])
    assert takes(B.TPP, 1, 4, [16] * 19) and takes(B.TPP, 1, 4, [25] * 3) and takes(B.DSL, 1, 4, [36])


def test_binding_names_every_step_path():
    import os
    import re

    from paper_2002_12717_amd import binding as B
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    with open(os.path.join(root, "include", "g1g2.h")) as f:
        paths = dict(re.findall(r"G1G2_PATH_(\w+) = (\d+)", f.read()))
    assert {int(v): k.lower() for k, v in paths.items()} == B.PATHS


def test_tuned_batches_count_every_channel():
    """make_batch leaves the choice to the library where it takes slices or the triangle by
    itself: 2^20 elements with the three channels of GW and DSL counted, whatever the
    hoppings."""
    from types import SimpleNamespace

    import numpy as np

    from paper_2002_12717_amd import autotune
    from paper_2002_12717_amd import binding as B
    seen = []
    fake = SimpleNamespace(GW=B.GW, DSL=B.DSL, FP64=B.FP64, HUB_SLICE_KERNEL=B.HUB_SLICE_KERNEL,
                           Batch=lambda *a, flags, **k: seen.append(flags))

    def flags(se, ns, n, h=np.zeros(1)):
        cl = [SimpleNamespace(ns=ns, U=1.0, h0=h, g1=None)] * n
        autotune.make_batch(fake, cl, se, table={"kernel": "triangle"})
        return seen.pop()
    assert flags(B.TPP, 16, 16) == 0 and flags(B.TPP, 16, 15) == B.HUB_SLICE_KERNEL
    for se in (B.GW, B.DSL):
        assert flags(se, 16, 6) == 0 and flags(se, 16, 5) == B.HUB_SLICE_KERNEL
    assert flags(B.TPP, 16, 16, np.full(1, 1j)) == 0
