"""Device memory that solves through the subproduct tree take from the allocator, on a
stream of their own (whose cache of blocks starts empty), against what the tree
needs.  Blocks are rounded up to powers of two, so twice the sum bounds them."""
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
