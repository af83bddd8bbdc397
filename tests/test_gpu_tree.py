"""GPU parity of the subproduct-tree solve against the quadratic pass (one wave
per tile), bit for bit, through zr_vandermonde_solve: sizes on both sides of the
leaf blocks (512 rows), the levels (powers of two), the transforms of one
workgroup (4096 points) and of the sizes where the denominators come from power sums
(32 768), right-hand sides from one to more than one group, primes from 65 537
to 2^63 - 25, and singular systems.  Tolerance 0: both compute the same residues."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

PRIMES = [synth.make_prime(), (1 << 63) - 25, (1 << 61) - 1]


@pytest.fixture(scope="module")
def zr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_24256_amd as m
    m.lib()
    yield m
    m.solve_variant()


def _solve(zr, p, mono, rhs, variant):
    import torch
    zr.solve_variant(variant)
    R, t = rhs.shape
    out = torch.full_like(rhs, -1)
    st = torch.full((1,), 99, dtype=torch.int32, device="cuda")
    assert zr.lib().zr_vandermonde_solve(p, t, R, mono.data_ptr(), rhs.data_ptr(), out.data_ptr(), st.data_ptr(),
                                         zr._stream(None)) == 0
    torch.cuda.synchronize()
    return out, int(st.item())


def _system(p, t, R, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    if p < 1 << 20:
        mono = torch.randperm(p - 1, generator=g, device="cuda")[:t].contiguous() + 1
    else:
        mono = torch.randint(1, p, (t,), generator=g, device="cuda")
    rhs = torch.randint(0, p, (R, t), generator=g, device="cuda")
    rhs[0, : t // 2] = p - 1  # the largest residues side by side
    return mono, rhs


@pytest.mark.parametrize("t,R", [(4097, 48), (4608, 46), (4609, 60), (8191, 20), (8192, 16), (8193, 16), (9997, 30),
                                 (10_000, 1), (12_289, 2), (16_384, 10), (16_385, 11), (20_001, 64), (32_767, 3),
                                 (32_768, 62), (32_769, 63), (65_537, 2), (70_000, 20), (131_073, 1)])
def test_tree_equals_quadratic_solve(zr, t, R):
    import torch
    p = PRIMES[t % 3]
    print(f"[gpu-test] tree t={t} R={R} p={p}", flush=True)
    mono, rhs = _system(p, t, R, t)
    got, st = _solve(zr, p, mono, rhs, "producer_consumer")
    want, st0 = _solve(zr, p, mono, rhs, "waves")
    assert st == st0 == 0
    assert torch.equal(got, want)


@pytest.mark.parametrize("t", [9000, 40_000])
def test_tree_small_prime(zr, t):
    import torch
    mono, rhs = _system(65_537, t, 20, 3)
    got, _ = _solve(zr, 65_537, mono, rhs, "producer_consumer")
    want, _ = _solve(zr, 65_537, mono, rhs, "waves")
    assert torch.equal(got, want)


@pytest.mark.parametrize("t", [10_000, 40_000])
@pytest.mark.parametrize("bad", ["repeat", "zero"])
def test_tree_singular(zr, t, bad):
    mono, rhs = _system(PRIMES[0], t, 3, 5)
    mono[t - 7] = mono[11] if bad == "repeat" else 0
    _, st = _solve(zr, PRIMES[0], mono, rhs, "producer_consumer")
    assert st == zr.ZR_ESINGULAR


def test_tree_in_place(zr):
    import torch
    p = PRIMES[0]
    mono, rhs = _system(p, 11_111, 12, 9)
    want, _ = _solve(zr, p, mono, rhs, "waves")
    zr.solve_variant()
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    assert zr.lib().zr_vandermonde_solve(p, 11_111, 12, mono.data_ptr(), rhs.data_ptr(), rhs.data_ptr(),
                                         st.data_ptr(), zr._stream(None)) == 0
    torch.cuda.synchronize()
    assert torch.equal(rhs, want)
