"""The transposed Vandermonde apply of the balanced path, through whole rational
reconstructions whose term counts lie on both sides of its blocks of 128 powers and
256 terms; the result equals the hidden numerator and denominator."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tn,td", [(127, 3), (128, 129), (256, 255), (257, 513), (2, 300)])
def test_apply_block_edges(tn, td):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_24256_amd as zr
    w = synth.rational_workload(3, 14, tn, td, 900 + tn)
    box = synth.DeviceBlackBox(w.num, w.den, nthreads=8)
    (en, cn), (ed, cd) = zr.balanced_reconstruct(w.p, w.deg_num, w.deg_den, box, sched=w.schedule)
    assert np.array_equal(en, w.num.exps) and np.array_equal(cn, w.num.coefs)
    assert np.array_equal(ed, w.den.exps) and np.array_equal(cd, w.den.coefs)
