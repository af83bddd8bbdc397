"""Device memory that solves through the subproduct tree take from the allocator, on a
stream of their own (whose cache of blocks starts empty), against what the tree
needs.  Blocks are rounded up to powers of two, so twice the sum bounds them."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
P = synth.make_prime()


@pytest.fixture(scope="module")
def zr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_24256_amd as m
    m.lib()
    m.solve_variant()
    return m


def _rows(t):
    """Rows of the tree's top node: the next power of two."""
    return 1 << max(8, (t - 1).bit_length())


def _transforms(t):
    """Bytes of the transforms kept for one system of t rows: five 4-byte residues of
    2 rows per row and level above the 256-row leaves, once more for the power series."""
    return 40 * _rows(t) * ((_rows(t) // 256).bit_length() - 1 + 1)


def _growth(call):
    """Bytes by which device memory in use grows over call(stream) on a new stream."""
    import torch
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    call(s.cuda_stream)
    torch.cuda.synchronize()
    return before - torch.cuda.mem_get_info()[0]


def _random(t, R, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randint(1, P, (t,), generator=g, device="cuda"),
            torch.randint(0, P, (R * t,), generator=g, device="cuda"))


def test_one_system_leaves_out_the_quadratic_product_tree(zr):
    """A million unknowns, one right-hand side.  The convolution levels' partial sums
    (256 words a row here) belong to the quadratic solve alone."""
    import torch
    t = 1_000_003
    mono, rhs = _random(t, 1, 1)
    out = torch.empty_like(rhs)
    st = torch.zeros(1, dtype=torch.int32, device="cuda")

    def call(s):
        assert zr.lib().zr_vandermonde_solve(P, t, 1, mono.data_ptr(), rhs.data_ptr(), out.data_ptr(), st.data_ptr(),
                                             s) == 0
    got = _growth(call)
    V = _rows(t)
    residues = 2 * 60 * V           # two series (the power sums are one): source and two products, five primes
    twist = 80 * V                  # five primes, both directions, transforms of 2 V points
    leaves = 8 * t * (3 * 8 + 8)    # packed rows (three tiles of 16 words), sums, inverses
    words = 8 * (4 * V + 2 * t + 5 * t)  # polynomials, power sums, series; the base level's buffers
    need = _transforms(t) + residues + twist + leaves + words
    print(f"[gpu-test] one system: {got / 2**20:.0f} MiB taken, {need / 2**20:.0f} MiB needed", flush=True)
    assert int(st.item()) == 0
    assert got <= 2 * need


def test_one_system_keeps_its_series_in_the_output(zr):
    """Many right-hand sides: the workspace is the residues' 640 MB, the transforms and a
    leaf pass of at most 63 right-hand sides, whatever their number."""
    import torch
    t, R = 4_100, 40_000
    mono, rhs = _random(t, R, 2)
    out = torch.empty_like(rhs)
    st = torch.zeros(1, dtype=torch.int32, device="cuda")

    def call(s):
        assert zr.lib().zr_vandermonde_solve(P, t, R, mono.data_ptr(), rhs.data_ptr(), out.data_ptr(), st.data_ptr(),
                                             s) == 0
    got = _growth(call)
    leaves = 8 * t * (10 * 8 + 63 + 32)  # packed rows (ten tiles' worth of 16 words), sums, denominators' chunks
    need = (640 << 20) + _transforms(t) + leaves
    print(f"[gpu-test] {R} right-hand sides: {got / 2**20:.0f} MiB taken, {need / 2**20:.0f} MiB needed, "
          f"right-hand sides {8 * t * R / 2**20:.0f} MiB", flush=True)
    assert int(st.item()) == 0
    assert got <= 2 * need
    # first, middle and last against the same columns alone
    for j in (0, R // 2, R - 1):
        one = torch.empty(t, dtype=torch.int64, device="cuda")
        assert zr.lib().zr_vandermonde_solve(P, t, 1, mono.data_ptr(), rhs[j * t:(j + 1) * t].data_ptr(),
                                             one.data_ptr(), st.data_ptr(), zr._stream(None)) == 0
        torch.cuda.synchronize()
        assert torch.equal(one, out[j * t:(j + 1) * t])


def _batch(zr, shapes, seed):
    """A batch of systems (t, R): (call(stream), systems, solution of each)."""
    import torch
    sys_ = [_random(t, R, seed + i) for i, (t, R) in enumerate(shapes)]
    so = np.concatenate([[0], np.cumsum([t for t, _ in shapes])]).astype(np.uint64)
    ro = np.concatenate([[0], np.cumsum([t * R for t, R in shapes])]).astype(np.uint64)
    nrhs = np.array([R for _, R in shapes], np.uint32)
    mono, rhs = torch.cat([m for m, _ in sys_]), torch.cat([v for _, v in sys_])
    out = torch.full_like(rhs, -1)
    st = torch.full((len(shapes),), 99, dtype=torch.int32, device="cuda")
    d_so, d_ro = (torch.from_numpy(a.view(np.int64)).cuda() for a in (so, ro))

    def call(s):
        assert zr.lib().vandermonde_solve_batch(
            len(shapes), P, d_so.data_ptr(), so.ctypes.data, mono.data_ptr(), nrhs.ctypes.data, d_ro.data_ptr(),
            ro.ctypes.data, rhs.data_ptr(), out.data_ptr(), st.data_ptr(), s) == 0
        torch.cuda.synchronize()
        assert not bool(st.any())
    return call, sys_, lambda i: out[int(ro[i]):int(ro[i + 1])]


def _alone(zr, t, R, mono, rhs):
    import torch
    out = torch.empty_like(rhs)
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    assert zr.lib().zr_vandermonde_solve(P, t, R, mono.data_ptr(), rhs.data_ptr(), out.data_ptr(), st.data_ptr(),
                                         zr._stream(None)) == 0
    torch.cuda.synchronize()
    return out


def test_trees_of_a_batch_share_their_workspace(zr):
    """Six right-hand-side counts are six trees, one after the other: residues and
    transforms of the largest, leaf blocks of all."""
    import torch
    t = 100_003
    shapes = [(t, R) for R in range(26, 32)]
    call, sys_, got_of = _batch(zr, shapes, 50)
    got = _growth(call)
    V = _rows(t)
    residues = 60 * V * 32
    twist = 80 * V
    leaves = sum(t * (4 * 3 * 32 + 8 * (R + 2) + 8 * 11) for t, R in shapes)  # packed rows, sums, polynomials and limbs
    words = 8 * V * (4 + 2 * 5)
    need = residues + _transforms(t) + twist + leaves + words
    print(f"[gpu-test] six trees: {got / 2**20:.0f} MiB taken, {need / 2**20:.0f} MiB needed", flush=True)
    for i in (0, 5):
        assert torch.equal(got_of(i), _alone(zr, t, shapes[i][1], *sys_[i]))
    assert got <= 2 * need


def test_batch_of_several_trees_of_one_count(zr):
    """More rows of one right-hand-side count than one tree holds (2^22): 33 systems whose
    nodes take 2^17 rows each fill one and a part of the next, the small ones follow."""
    import torch
    shapes = [(65_537, 2)] * 33 + [(65_536, 2), (9_000, 2), (3_000, 2)]
    call, sys_, got_of = _batch(zr, shapes, 90)
    call(zr._stream(None))
    for i in (0, 31, 32, 33, 34, 35):
        assert torch.equal(got_of(i), _alone(zr, *shapes[i], *sys_[i])), i
