"""The benchmark's count of performed products: which systems go through the subproduct
tree comes from the launches that ran, not from a second statement of the rule, and
the rows of a leaf block are those of the library."""
import os
import re

import bench

HERE = os.path.dirname(os.path.abspath(bench.__file__))


def test_leaf_rows_are_the_library_s():
    with open(os.path.join(HERE, "paper_2505_24256_amd", "csrc", "tree.hpp")) as f:
        assert int(re.search(r"kTreeLeafLog = (\d+);", f.read()).group(1)) == bench.TREE_LEAF_LOG


class _Ran:
    def __init__(self, **launches):
        self.launches = launches

    def timing_get(self, name):
        return self.launches.get(name, 0), 0.0


def test_products_follow_the_launches():
    sizes, R = [31, 961, 9997, 40_000], 30
    quad = {t: R * t * t + t * (t - 1) for t in sizes}
    assert bench._tree_launches(_Ran()) == (0, 0)
    assert bench._tree_launches(_Ran(tree_down=2, tree_sums=1)) == (2, 1)
    assert bench._dots_done(sizes, R, 0, 0) == sum(quad.values())
    # the largest two through the tree, the largest with the power sums as a series
    assert bench._dots_done(sizes, R, 2, 1) == (quad[31] + quad[961] + (R + 1) * 256 * 9997 + (R + 2) * 256 * 40_000)


def test_descent_products_per_series():
    # one level of 512 points: 1.5 * 9 Montgomery products a point for the transforms, 2 pointwise
    assert bench._tree_down_mul32(512, 1) == 512 * 5 * (1.5 * 9 + 2) * 3
    assert bench._tree_down_mul32(512, 7) == 7 * bench._tree_down_mul32(512, 1)


def test_traffic_is_keyed_to_sources_and_system(monkeypatch):
    t, R = bench.TREE_TRAFFIC["system"]
    assert bench._tree_traffic(t + 1, R) is None and bench._tree_traffic(t, R + 1) is None
    monkeypatch.setitem(bench.TREE_TRAFFIC, "sources_sha16", "0" * 16)
    assert bench._tree_traffic(t, R) is None
