"""The field inverse on the GPU, through systems of one unknown: a = v / m.  m at
the edges of the field and of the binary Euclid's shifts (powers of two, their
negatives, neighbours of p/2), p from 3 to 2^63 - 25; checked by multiplying back
(tolerance 0)."""
import random

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [3, 5, 65_537, 2_305_843_009_213_693_951, synth.make_prime(), (1 << 63) - 25])
def test_inverse_edges(p):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_24256_amd as zr
    rng = random.Random(p)
    m = {1, 2, p - 1, p - 2, (p - 1) // 2, (p + 1) // 2}
    m |= {(1 << i) % p for i in range(63)} | {p - (1 << i) % p for i in range(63)}
    m |= {rng.randrange(1, p) for _ in range(400)}
    m = [x for x in sorted(m) if 0 < x < p]
    systems = [(np.array([x], np.uint64), np.array([[rng.randrange(p)]], np.uint64)) for x in m]
    out, st = zr.vandermonde_solve_batch(p, systems)
    assert not st.any()
    for x, (_, v), a in zip(m, systems, out):
        assert int(a[0, 0]) * x % p == int(v[0, 0])
