"""Unknown degree bounds at sizes where a stage's solves go through the subproduct tree:
the tree and the denominators are made once per stage, however many batches of nodes
the stage takes, and the result is the hidden polynomial.  The second size takes its
denominators from power sums (from 32 768 unknowns on)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def zr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_24256_amd as m
    m.lib()
    m.solve_variant()
    yield m
    m.timing(False)


@pytest.mark.parametrize("deg,terms,least", [([24, 24, 24, 45], 9_000, 5_500), ([36, 36, 36, 60], 70_000, 32_768)])
def test_tree_once_per_stage(zr, deg, terms, least):
    p = synth.make_prime()
    h = synth.random_poly(p, 4, deg, terms, 4242)
    e0 = np.asarray(h.exps)
    assert len(np.unique(e0[:, :3], axis=0)) >= least > 5_000 > len(np.unique(e0[:, :2], axis=0))
    print(f"[gpu-test] unknown degrees {deg}, {terms} terms", flush=True)
    zr.timing(True)
    zr.timing_reset()
    e, c, found = zr.reconstruct_adaptive(p, [80] * 4, synth.DeviceBlackBox(h, nthreads=8), seed=5, confirm=2, nprobes=1)
    launches = {k: zr.timing_get(k)[0] for k in ("tree_up", "tree_sums", "tree_down", "vs_dots")}
    zr.timing(False)
    assert np.array_equal(e, h.exps) and np.array_equal(c, h.coefs)
    assert found == [int(x) for x in e0.max(axis=0)]
    # the last stage's degree exceeds its first batch (the previous degree and two): two batches or three
    assert launches["tree_down"] >= 2
    assert launches["tree_up"] == 1
    assert launches["tree_sums"] == (1 if least >= 32_768 else 0)
