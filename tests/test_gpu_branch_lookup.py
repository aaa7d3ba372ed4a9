"""The branch (alpha, route bit) of each neuron where a gate+up tile holds more than one branch: boundaries inside a
tile of 8 neurons (decode) and of 32 to 128 (prefill), empty branches, the largest number of branches and of runs.
One d_model per gate+up kernel: x in registers in 2, 4, 8 and 16 blocks, x in LDS, and neither.  Against the oracle."""
import numpy as np
import pytest

from gpu_util import check_bf16_flip_aware, run_gpu_with_hidden
from paper_2511_21089_amd import synth

pytestmark = pytest.mark.gpu

TABLES = {
    "one": ([200], [1]),
    "straddle": ([3, 1, 0, 5, 120, 0, 7, 60, 60], [1, 1, 0, 1, 1, 1, 1, 1, 1]),
    "most_branches": ([1] * 63 + [129], [1] * 64),
    "most_runs": ([8] * 64, [1, 0] * 32),
    "empty_last": ([0, 0, 129, 127, 0, 0], [1, 1, 1, 1, 1, 0]),
}


def layer(name, T, d_model):
    widths, mask = TABLES[name]
    off = np.concatenate([[0], np.cumsum(widths)]).astype(np.int32)
    rng = np.random.default_rng(T + d_model)
    x, Wg, Wu, Wd = synth.random_layer(rng, T, d_model, int(off[-1]), dtype="bf16", w_scale=0.05)
    alpha = np.linspace(0.5, 2.0, len(widths)).astype(np.float32)       # a neighbour's alpha is far outside the bounds
    return x, Wg, Wu, Wd, off, alpha, np.array(mask, np.uint8)


@pytest.mark.parametrize("T,d_model", [(1, 136), (16, 1032), (3, 2056), (16, 4104), (2, 8200), (16, 8200),
                                       (17, 72), (100, 136), (129, 264), (600, 72)])
@pytest.mark.parametrize("name", sorted(TABLES))
def test_branch_lookup(name, T, d_model):
    args = layer(name, T, d_model)
    got, H = run_gpu_with_hidden(*args)
    check_bf16_flip_aware(got, H, *args, label="%s T=%d d_model=%d:" % (name, T, d_model))


@pytest.mark.parametrize("T,d_model", [(5, 136), (16, 8200), (300, 72)])
@pytest.mark.parametrize("name", sorted(TABLES))
def test_branch_lookup_routed(name, T, d_model):
    args = layer(name, T, d_model)
    route = (np.random.default_rng(T).uniform(size=(T, len(args[5]))) < 0.5).astype(np.uint8)
    got, H = run_gpu_with_hidden(*args, route=route)
    check_bf16_flip_aware(got, H, *args, route=route, label="%s routed T=%d d_model=%d:" % (name, T, d_model))
