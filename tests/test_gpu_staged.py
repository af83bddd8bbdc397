"""GPU parity of the staged producer/consumer pass (systems of at most 3072
unknowns) against the one-wave-per-tile pass, bit for bit, through
zr_vandermonde_solve: chunks and blocks of 16 steps with every kind of remainder,
tiles of one to nine values, idle consumers, more than one group.  Tolerance 0."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("t,R", [(257, 1), (300, 3), (321, 4), (511, 7), (513, 14), (1023, 21), (1025, 29), (1500, 36),
                                 (2047, 43), (2049, 50), (3071, 57), (3072, 63), (3072, 64), (3073, 8), (700, 130)])
def test_staged_equals_waves(t, R):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_24256_amd as zr
    p = (1 << 63) - 25 if t % 2 else synth.make_prime()
    g = torch.Generator(device="cuda").manual_seed(t)
    mono = torch.randint(1, p, (t,), generator=g, device="cuda")
    rhs = torch.randint(0, p, (R, t), generator=g, device="cuda")
    rhs[0] = p - 1
    outs = []
    try:
        for v in ("producer_consumer", "waves"):
            zr.solve_variant(v)
            out = torch.full_like(rhs, -1)
            st = torch.full((1,), 99, dtype=torch.int32, device="cuda")
            assert zr.lib().zr_vandermonde_solve(p, t, R, mono.data_ptr(), rhs.data_ptr(), out.data_ptr(),
                                                 st.data_ptr(), zr._stream(None)) == 0
            torch.cuda.synchronize()
            assert int(st.item()) == 0
            outs.append(out)
    finally:
        zr.solve_variant()
    assert torch.equal(outs[0], outs[1])
