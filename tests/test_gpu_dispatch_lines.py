"""One-system solves on both sides of every line between the staged pass, the pass with
scalar rows and the subproduct tree, bit for bit against the quadratic pass with one
wave per tile."""
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
