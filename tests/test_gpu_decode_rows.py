"""The decode kernels for narrow layers and small batches at the edges of their tiles and of the rules that pick them: 4, 8
and 16 output features per workgroup, one and two K groups per MFMA (T = 4 / 5, 8 / 9), widths that end inside a K block,
runs that start and end anywhere in steps of 8, branches that meet inside a tile, float and bf16 results, routing; tables
with odd boundaries and float storage."""
import numpy as np
import pytest

import test_gpu_f32_mfma
import test_gpu_uneven
from gpu_util import check_bf16_flip_aware, flip_terms, run_gpu, run_gpu_with_hidden
from oracle import round_to_bf16
from paper_2511_21089_amd import synth

pytestmark = pytest.mark.gpu

# (d_model, branch widths, branches off, T); run ends are multiples of 8
CASES = [
    (8, [8], [], 1), (8, [8], [], 16), (16, [24, 40], [], 8), (72, [64, 64, 136], [1], 9), (136, [13, 11, 72, 8], [], 5),
    (264, [8, 504, 40, 8], [1], 4), (512, [3, 5, 640, 16], [2], 2), (904, [4864], [], 15), (896, [608] * 8, [2, 5], 8),
    (1024, [1000, 24, 1024], [], 14), (1032, [520, 1528], [], 13), (1536, [2048, 64], [], 9), (1544, [1080], [], 3),
    (2552, [264, 512], [0], 16), (2560, [776], [], 1), (3064, [200, 312], [], 8), (3072, [512], [], 1), (3080, [264, 256], [], 2),
    (4096, [1024], [], 1), (4104, [328, 512], [1], 1),
    (1792, [264], [], 2), (5128, [72], [], 2), (8200, [16, 56], [0], 1),
    (1032, [72, 12296, 24], [0], 3), (1800, [8200], [], 15), (2104, [8, 12480], [0], 9),      # a long K
]


def _layer(case):
    d_model, widths, gone, T = case
    off = np.concatenate([[0], np.cumsum(widths)]).astype(np.int32)
    rng = np.random.default_rng(d_model + T)
    x, Wg, Wu, Wd = synth.random_layer(rng, T, d_model, int(off[-1]), dtype="bf16", w_scale=0.1)
    alpha = rng.uniform(0.8, 1.25, size=len(widths)).astype(np.float32)
    mask = np.ones(len(widths), np.uint8)
    mask[gone] = 0
    for b in gone:                                       # nothing of a pruned branch may reach the result
        Wg[off[b]:off[b + 1]] = Wu[off[b]:off[b + 1]] = 0x7FC0
        Wd[:, off[b]:off[b + 1]] = 0x7FC0
    return x, Wg, Wu, Wd, off, alpha, mask


def _clean(L):
    x, Wg, Wu, Wd, off, alpha, mask = L
    live = np.repeat(mask != 0, np.diff(off))
    return (x, np.where(live[:, None], Wg, 0).astype(np.uint16), np.where(live[:, None], Wu, 0).astype(np.uint16),
            np.where(live[None], Wd, 0).astype(np.uint16), off, alpha, mask)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%d_T%d" % (c[0], sum(c[1]), c[3]))
def test_rows(case):
    L = _layer(case)
    got, H = run_gpu_with_hidden(*L)
    check_bf16_flip_aware(got, H, *_clean(L), label="%s:" % (case,))
    # the bf16 result: the down projection of the stored H (the same as above, bit for bit) up to fp32 summation error and
    # one rounding to bf16, 2^-8 of the value
    got16, H16 = run_gpu_with_hidden(*L, out_bf16=True)
    live = np.repeat(L[6] != 0, np.diff(L[4]))
    assert np.array_equal(H16[:, live], H[:, live])
    f = flip_terms(H16, *_clean(L))
    own = f["H"] @ f["Wd"].T
    assert np.all(np.abs(got16 - own) <= f["sum_err"] + 2.0 ** -8 * (np.abs(own) + f["sum_err"]) + 1e-30)
    assert np.mean(got16 == round_to_bf16(own)) > 0.9 or got16.size < 64


@pytest.mark.parametrize("T", [1, 8, 16])
@pytest.mark.parametrize("d_model", [72, 1280, 3072])
def test_routed_rows(d_model, T):
    """Every token its own branches; all-ones routing has the bits of the plain call (branches are multiples of 64)."""
    L = _layer((d_model, [64, 128, 320, 64], [], T))
    rng = np.random.default_rng(T)
    route = rng.integers(0, 2, size=(T, 4), dtype=np.uint8)
    got, H = run_gpu_with_hidden(*L, route=route)
    check_bf16_flip_aware(got, H, *L, route=route, label="routed %d, T = %d:" % (d_model, T))
    ones, _ = run_gpu_with_hidden(*L, route=np.ones((T, 4), np.uint8))
    plain, _ = run_gpu_with_hidden(*L)
    assert np.array_equal(ones, plain)


SIZES = [(1, 72), (4, 1032), (5, 264), (8, 136), (9, 72), (16, 520), (3, 1544), (12, 1288)]


@pytest.mark.parametrize("T,d_model", SIZES)
@pytest.mark.parametrize("name", sorted(test_gpu_uneven.TABLES))
def test_odd_boundaries(name, T, d_model):
    """Runs that start and end inside a chunk, one run inside a chunk, runs of one neuron; NaN and infinities in every pruned
    branch and in every H that is not written."""
    args = test_gpu_uneven.make(name, T, d_model, seed=T)
    bad = test_gpu_uneven.poison_pruned(args)
    got, H = run_gpu_with_hidden(*bad)
    active = np.repeat(args[6] != 0, np.diff(args[4]))
    assert np.all(np.isnan(H[:, ~active])) and np.all(np.isfinite(got))
    check_bf16_flip_aware(got, H, *args, label="%s T=%d:" % (name, T))
    got16, H16 = run_gpu_with_hidden(*bad, out_bf16=True)
    assert np.array_equal(H16[:, active], H[:, active])
    f = flip_terms(H16, *args)
    own = f["H"] @ f["Wd"].T
    assert np.all(np.abs(got16 - own) <= f["sum_err"] + 2.0 ** -8 * (np.abs(own) + f["sum_err"]) + 1e-30)


@pytest.mark.parametrize("T,d_model", [(1, 68), (4, 1028), (5, 260), (8, 132), (9, 4), (16, 516), (2, 2044), (12, 1284)])
@pytest.mark.parametrize("name", sorted(test_gpu_f32_mfma.TABLES))
def test_float_storage(name, T, d_model):
    args = test_gpu_f32_mfma.make(*test_gpu_f32_mfma.TABLES[name], T, d_model, seed=T)
    test_gpu_f32_mfma.check(run_gpu(*test_gpu_f32_mfma.poison_pruned(args)), *args)
