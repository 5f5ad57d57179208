"""The settings the autotuner times: every one of them cuts the work differently."""

from paper_1508_00115_amd import tune


def test_no_two_settings_are_the_same_work():
    """tile_cap has no effect on the kernels, so settings may not differ in it alone."""
    seen = [tuple(sorted((k, v) for k, v in s.items() if k != "tile_cap")) for s in tune.DEFAULT_GRID]
    assert len(seen) == len(set(seen)) == 96
