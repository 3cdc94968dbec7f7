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
    assert [per(ns, 4096) for ns in (1, 2, 3, 9, 16, 25, 33, 64)] == [1, 3, 6, 12, 4, 1, 1, 1]
