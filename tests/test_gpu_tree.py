"""GPU parity of the subproduct-tree solve against the quadratic pass (one wave
per tile), bit for bit, through zr_vandermonde_solve: sizes on both sides of the
leaf blocks (256 rows), the levels (powers of two), the transforms of one
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


@pytest.mark.parametrize("t,R", [(2561, 37), (3073, 8), (3329, 9), (4097, 48), (4608, 46), (4609, 60), (8191, 20), (8192, 16), (8193, 16), (9997, 30),
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


@pytest.mark.parametrize("graphs", [False, True])
def test_batch_through_one_tree(zr, graphs):
    """Large systems of a batch share one tree per right-hand-side count, small ones keep
    their own path; a singular system does not touch the others."""
    import torch
    p = PRIMES[0]
    shapes = [(20_000, 30), (16_385, 30), (9000, 30), (4097, 30), (1600, 30), (1536, 30), (1535, 30), (700, 30),
              (65, 30), (10, 30), (1, 30), (18_000, 12), (2049, 12), (2048, 12), (5000, 30)]
    sys_ = [_system(p, t, R, i) for i, (t, R) in enumerate(shapes)]
    sys_[-1][0][4999] = sys_[-1][0][3]  # the last one is singular
    so = np.concatenate([[0], np.cumsum([t for t, _ in shapes])]).astype(np.uint64)
    ro = np.concatenate([[0], np.cumsum([t * R for t, R in shapes])]).astype(np.uint64)
    nrhs = np.array([R for _, R in shapes], np.uint32)
    mono = torch.cat([m for m, _ in sys_])
    rhs = torch.cat([v.reshape(-1) for _, v in sys_])
    out = torch.full_like(rhs, -1)
    st = torch.full((len(shapes),), 99, dtype=torch.int32, device="cuda")
    d_so, d_ro = (torch.from_numpy(a.view(np.int64)).cuda() for a in (so, ro))
    zr.solve_variant()
    zr.batch_graphs(graphs)
    try:
        for _ in range(2):
            assert zr.lib().vandermonde_solve_batch(
                len(shapes), p, d_so.data_ptr(), so.ctypes.data, mono.data_ptr(), nrhs.ctypes.data, d_ro.data_ptr(),
                ro.ctypes.data, rhs.data_ptr(), out.data_ptr(), st.data_ptr(), zr._stream(None)) == 0
            torch.cuda.synchronize()
    finally:
        zr.batch_graphs(False)
    assert st.cpu().tolist() == [0] * (len(shapes) - 1) + [zr.ZR_ESINGULAR]
    for i, (t, R) in enumerate(shapes[:-1]):
        want, _ = _solve(zr, p, *sys_[i], "waves")
        assert torch.equal(out[int(ro[i]):int(ro[i + 1])].reshape(R, t), want), (t, R)
