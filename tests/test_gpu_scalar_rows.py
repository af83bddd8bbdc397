"""The producer/consumer pass with scalar rows.  Below 2^21 unknowns most systems go
through the subproduct tree or the staged pass now, so the sizes that tests of
zr_vandermonde_solve name no longer reach it; the no-allocation solve, which never takes the
tree, does beyond 3 072 unknowns, and so does every system above 2^21.

* Right-hand sides from 11 to 127 at sizes that straddle row blocks and chunks, against
  the pass with one wave per tile: three tiles of up to ten, seven even and uneven ones of
  up to nine, with the Horner sum in the producer and without, and two and three groups.
* One system of 2^21 + 1 unknowns, 31 right-hand sides, where the bound on the per-chunk
  state (16 GiB) sets the chunk count and the chunks share their partial-sum slots over
  many launches; checked by the defining property at sampled equations."""
import numpy as np
import pytest

import oracle
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
    m.timing(False)
    m.solve_variant()


@pytest.mark.parametrize("t", [3073, 4097, 6001])
@pytest.mark.parametrize("R", [10, 11, 17, 24, 30, 31, 33, 36, 37, 41, 45, 50, 56, 57, 63, 64, 70, 127])
def test_scalar_rows(zr, t, R):
    import torch
    p = [synth.make_prime(), (1 << 63) - 25, (1 << 61) - 1][(t + R) % 3]
    print(f"[gpu-test] no-allocation solve t={t} R={R} p={p}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(t + R)
    mono = torch.randint(1, p, (t,), generator=g, device="cuda")
    rhs = torch.randint(0, p, (R * t,), generator=g, device="cuda")
    rhs[: t // 2] = p - 1
    want, got = torch.full_like(rhs, -1), torch.full_like(rhs, -1)
    st = torch.full((2,), 99, dtype=torch.int32, device="cuda")
    zr.solve_variant("waves")
    assert zr.lib().zr_vandermonde_solve(p, t, R, mono.data_ptr(), rhs.data_ptr(), want.data_ptr(), st.data_ptr(),
                                         zr._stream(None)) == 0
    zr.solve_variant()
    assert zr.vandermonde_solve_noalloc(p, mono, rhs, got, st[1:], t, R) == 0
    torch.cuda.synchronize()
    assert st.cpu().tolist() == [0, 0]
    assert torch.equal(got, want)


def test_beyond_the_tree(zr):
    p = synth.make_prime()
    t, R = (1 << 21) + 1, 31
    g = synth.SplitMix64(2121)
    m = g.uniform_block(1, p, t)
    assert len(np.unique(m)) == t
    rhs = g.uniform_block(0, p, t * R).reshape(R, t)
    print(f"[gpu-test] solve t={t} R={R} (about 35 s)", flush=True)
    zr.timing(True)
    zr.timing_reset()
    a, st = zr.vandermonde_solve(p, m, rhs)
    launches = {k: zr.timing_get(k)[0] for k in ("tree_down", "vs_dots")}
    zr.timing(False)
    assert st == 0
    assert launches["tree_down"] == 0 and launches["vs_dots"] > 1
    print("[gpu-test] multiply-back at sampled equations", flush=True)
    for j in (0, 17, R - 1):
        for i in (1, 1 + (j * 99_991 + 7) % t, t):
            assert int(oracle.vandermonde_apply(p, m, a[j], i, 1)[0]) == int(rhs[j, i - 1]), (j, i)
