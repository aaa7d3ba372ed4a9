"""Fractal Fade of W_gate and W_up in one pass of launches (bf16): the histogram's workgroup shares, and the two
matrices in the same memory.  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev
from paper_2511_21089_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2511_21089_amd import binding
    return binding


def bits(t):
    import torch
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


def check_report(thr, kept, rthr, rkept, m):
    for b in range(len(rthr)):
        assert int(kept[b, m]) == rkept[b][m], (b, m)
        if rthr[b][m] is None:
            assert np.isnan(thr[b, m])
        else:                                              # reported as float32, interpolated from the same two values
            assert abs(float(thr[b, m]) - rthr[b][m]) <= 1e-6 * abs(rthr[b][m]) + 1e-30


@pytest.mark.parametrize("widths,sparsity", [
    ([1, 4000, 3, 0, 17], None),                       # one branch holds nearly all: workgroups dealt by size
    ([513, 511], [0.5, 0.999]),                        # a remainder below one group of loads per thread
    ([2], [0.75]),                                     # fewer 16-byte pieces than a workgroup has threads
    ([30] * 64, None),                                 # as many blocks as there can be
])
def test_workgroup_shares(mm, widths, sparsity):
    off = np.concatenate([[0], np.cumsum(widths)]).astype(np.int32)
    rng = np.random.default_rng(len(widths))
    Wg, Wu = (synth.f32_to_bf16_bits((rng.standard_normal((int(off[-1]), 520)) * s).astype(np.float32)) for s in (0.02, 3.0))
    Wg_d, Wu_d = to_dev(Wg), to_dev(Wu)
    thr, kept = mm.mlpmoe_fade(Wg_d, Wu_d, off, sparsity)
    rWg, rWu, rthr, rkept = oracle.fractal_fade(Wg, Wu, off, sparsity)
    assert np.array_equal(bits(Wg_d), rWg) and np.array_equal(bits(Wu_d), rWu)
    for m in range(2):
        check_report(thr, kept, rthr, rkept, m)


def test_one_matrix_given_twice(mm):
    """In the same memory the two are faded one after the other, as two calls would."""
    off, sp = np.array([0, 40, 90], np.int32), [0.3, 0.6]
    W = synth.f32_to_bf16_bits((np.random.default_rng(7).standard_normal((90, 64)) * 0.02).astype(np.float32))
    dev = to_dev(W)
    thr, kept = mm.mlpmoe_fade(dev, dev, off, sp)
    for m in range(2):
        W, _, rthr, rkept = oracle.fractal_fade(W, W, off, sp)
        check_report(thr, kept, [(t[0],) * 2 for t in rthr], [(k[0],) * 2 for k in rkept], m)
    assert np.array_equal(bits(dev), W)
