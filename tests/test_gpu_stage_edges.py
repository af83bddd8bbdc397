"""The stage kernels at the edges of their paths: node sets of 63 nodes (one wave) and 64
(the workgroup), and stages whose term counts lie around the turns of the one-launch scan
(8 192 each) and the count above which it takes three launches (16 384)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _zr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_24256_amd as zr
    return zr


@pytest.mark.parametrize("degs", [(0, 1, 62), (63, 61, 64), (126, 125, 127)])
def test_node_set_edges(degs):
    zr = _zr()
    polys = [synth.random_poly(synth.make_prime(), 2, d, min(40, (d + 1) ** 2), 50 + d) for d in degs]
    items = [{"deg": [d, d], "box": synth.DeviceBlackBox(f), "seed": 9 + d, "nprobes": 2}
             for d, f in zip(degs, polys)]
    for f, r in zip(polys, zr.reconstruct_batch(polys[0].p, items)):
        assert not isinstance(r, Exception), r
        assert np.array_equal(r[0], f.exps) and np.array_equal(r[1], f.coefs)


@pytest.mark.parametrize("t", [8191, 8192, 8193, 16384, 16385])
def test_scan_edges(t):
    zr = _zr()
    # t distinct prefixes (x1, x2, x3), so that the last stage counts the terms of t lines
    g = np.random.default_rng(t)
    pre = np.stack(np.unravel_index(np.arange(t), (30, 30, 30)), axis=1)
    exps = np.concatenate([pre, g.integers(0, 4, (t, 1))], axis=1).astype(np.uint16)
    p = synth.make_prime()
    f = synth.SparsePoly(p, 4, exps, g.integers(1, p, t, dtype=np.uint64)).sorted()
    e, c = zr.reconstruct(p, [29, 29, 29, 3], synth.DeviceBlackBox(f), seed=t, nprobes=2)
    assert np.array_equal(e, f.exps) and np.array_equal(c, f.coefs)
