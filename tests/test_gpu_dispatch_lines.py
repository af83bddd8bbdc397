"""Solves on both sides of every line between the staged pass, the pass with scalar rows
and the subproduct tree, of one system and in a batch, bit for bit against the quadratic
pass with one wave per tile."""
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
    yield m
    m.solve_variant()


def _check(zr, t, R):
    import torch
    p = [synth.make_prime(), (1 << 63) - 25, (1 << 61) - 1][(t + R) % 3]
    print(f"[gpu-test] solve t={t} R={R} p={p}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t * 1000 + R)
    mono = torch.randint(1, p, (t,), generator=g, device="cuda")
    rhs = torch.randint(0, p, (R, t), generator=g, device="cuda")
    rhs[0, : t // 2] = p - 1
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = {}
    for variant in ("waves", "producer_consumer"):
        zr.solve_variant(variant)
        out[variant] = torch.full_like(rhs, -1)
        assert zr.lib().zr_vandermonde_solve(p, t, R, mono.data_ptr(), rhs.data_ptr(), out[variant].data_ptr(),
                                             st.data_ptr(), zr._stream(None)) == 0
        torch.cuda.synchronize()
        assert int(st.item()) == 0
    assert torch.equal(out["waves"], out["producer_consumer"])


# tiles of seven (43 and 49 right-hand sides, 127 in three groups), eight and nine values
@pytest.mark.parametrize("t", [1888, 1889, 1951, 2048, 2049])
@pytest.mark.parametrize("R", [43, 49, 50, 57, 63, 99, 127])
def test_staged_and_scalar_rows(zr, t, R):
    _check(zr, t, R)


@pytest.mark.parametrize("t,R", [(2240, 200), (2241, 199), (2241, 200), (2304, 120), (2305, 99), (2305, 100), (2560, 43),
                                 (2561, 42), (2561, 43), (2688, 32), (2689, 31), (2689, 32), (2944, 24), (2945, 23),
                                 (2945, 24), (3072, 63), (3073, 7), (3073, 8), (5499, 7), (5500, 1)])
def test_quadratic_and_tree(zr, t, R):
    _check(zr, t, R)


@pytest.mark.parametrize("sizes,R,repeat", [([699, 700, 701, 1000, 1023, 1024, 1025, 1200, 1535, 513], 60, 8),
                                            ([700], 60, 900), ([8000, 300], 30, 1)])
def test_batch_lines(zr, sizes, R, repeat):
    """Systems around the least size of a batch's tree (700 unknowns, nodes of 1024 rows)
    in numbers that a tree pays for, and one system alone."""
    import torch
    p, ts = synth.make_prime(), sizes * repeat
    print(f"[gpu-test] batch of {len(ts)} systems {sizes}, R={R}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(len(ts))
    so = np.concatenate([[0], np.cumsum(ts)]).astype(np.uint64)
    ro = so * np.uint64(R)
    mono = torch.randint(1, p, (int(so[-1]),), generator=g, device="cuda")
    rhs = torch.randint(0, p, (int(ro[-1]),), generator=g, device="cuda")
    nrhs = np.full(len(ts), R, np.uint32)
    d_so, d_ro = (torch.from_numpy(a.view(np.int64)).cuda() for a in (so, ro))
    out = {}
    for variant in ("waves", "producer_consumer"):
        zr.solve_variant(variant)
        zr.timing(True)
        zr.timing_reset()
        out[variant] = torch.full_like(rhs, -1)
        st = torch.full((len(ts),), 99, dtype=torch.int32, device="cuda")
        assert zr.lib().vandermonde_solve_batch(
            len(ts), p, d_so.data_ptr(), so.ctypes.data, mono.data_ptr(), nrhs.ctypes.data, d_ro.data_ptr(),
            ro.ctypes.data, rhs.data_ptr(), out[variant].data_ptr(), st.data_ptr(), zr._stream(None)) == 0
        torch.cuda.synchronize()
        trees = zr.timing_get("tree_down")[0]
        zr.timing(False)
        assert trees == (1 if variant == "producer_consumer" else 0)
        assert not bool(st.any())
    assert torch.equal(out["waves"], out["producer_consumer"])
