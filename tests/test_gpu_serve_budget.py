"""The server's footprint estimate covers the subproduct tree that a stage's solve goes
through: it is reported, and a further request waits while it does not fit."""
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
    return m


def test_tree_counts_against_the_budget(zr):
    p = synth.make_prime()
    deg, D1 = [126, 126, 30], 31
    big = synth.random_poly(p, 3, deg, 30_000, 611)
    small = synth.random_poly(p, 2, [3, 3], 5, 612)
    t = len(np.unique(np.asarray(big.exps)[:, :2], axis=0))  # unknowns of the last stage's system
    rows = 1 << (t - 1).bit_length()
    # value table, lift, packed rows and sums, skeleton; the next skeleton
    without = 8 * (t * (4 * D1 + 12) + 4 * min(t * D1, 127 * 127 * 31))
    # five residues of the series and of its two products; the children's transforms
    tree = 60 * rows * D1 + 40 * rows * (rows // 256).bit_length()
    print(f"[gpu-test] served t={t}: {without >> 20} MiB without the tree, tree at least {tree >> 20} MiB", flush=True)
    srv = zr.Server(p, hbm_budget=without + tree // 2, max_active=4)
    try:
        one = srv.submit(deg, synth.DeviceBlackBox(big, nthreads=8), seed=3, nprobes=1)
        srv.step()
        srv.step()  # stages 1 and 2; the last one is next
        assert srv.stats()["footprint"] >= without + tree
        two = srv.submit([3, 3], synth.DeviceBlackBox(small), seed=4, nprobes=1)
        srv.step()
        assert srv.stats()["peak_active"] == 1  # the second waited for the first
        for _ in range(3):
            srv.step()
        st, (e, c), _ = srv.poll(one)
        assert st == zr.ZR_OK and np.array_equal(e, big.exps) and np.array_equal(c, big.coefs)
        st, (e, c), _ = srv.poll(two)
        assert st == zr.ZR_OK and np.array_equal(e, small.exps) and np.array_equal(c, small.coefs)
        assert srv.stats()["peak_footprint"] >= without + tree
        assert srv.stats()["footprint"] == 0
    finally:
        srv.close()
