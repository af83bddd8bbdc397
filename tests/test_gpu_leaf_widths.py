"""The leaf pass of the subproduct tree at every width of its consumers' tiles beyond one
workgroup per CU (16 384 rows): 8 to 63 right-hand sides take three tiles of up to ten or
seven of up to nine, even or uneven, and 64 two groups.  Bit for bit against the
quadratic pass with one wave per tile."""
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


@pytest.mark.parametrize("R", [8, 11, 17, 27, 30, 31, 33, 35, 36, 38, 41, 42, 43, 46, 49, 50, 51, 53, 55, 56, 57, 60, 63, 64])
def test_leaf_tile_widths(zr, R):
    import torch
    p, t = synth.make_prime(), 16_449
    print(f"[gpu-test] leaf pass t={t} R={R}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(R)
    mono = torch.randint(1, p, (t,), generator=g, device="cuda")
    rhs = torch.randint(0, p, (R, t), generator=g, device="cuda")
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
