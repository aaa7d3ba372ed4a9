"""The down projection with K split: the sum of 2 to 32 partial results, around one batch of partial sums and around the
size from which a thread adds two pieces (its second piece past the end included), and the split planned for short K
loops.  Against a float64 product of the stored intermediate; the bf16 result is the float one rounded once."""
import numpy as np
import pytest

from gpu_util import C_SUM, U24, run_gpu_with_hidden, widen
from paper_2511_21089_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2511_21089_amd import binding
    return binding


@pytest.mark.parametrize("T,d_model,d_inter", [
    (1500, 512, 16 * 64), (17, 64, 12 * 64), (33, 72, 32 * 64), (100, 136, 36 * 64), (50, 64, 64 * 64),  # 2, 3, 8, 9,
    (20, 128, 130 * 64),                                                                 # 16 and 32 splits
    (128, 896, 4864), (333, 896, 3656), (600, 896, 4864), (150, 2048, 2048),                             # short K loops
    (2047, 512, 1024), (2048, 512, 1024), (2049, 512, 2048), (1031, 1032, 2048)])                        # around 2^18 pieces
def test_split_sum(mm, T, d_model, d_inter):
    rng = np.random.default_rng(T + d_inter)
    x, Wg, Wu, Wd = synth.random_layer(rng, T, d_model, d_inter, dtype="bf16", w_scale=0.05)
    args = (x, Wg, Wu, Wd, np.array([0, d_inter], np.int32), np.ones(1, np.float32), np.ones(1, np.uint8))
    mm.mlpmoe_profile_enable(16)
    got, H = run_gpu_with_hidden(*args)
    kernels = [name for name, _ in mm.mlpmoe_profile_collect(16)]
    mm.mlpmoe_profile_disable()
    assert "splitk_reduce" in kernels                    # this size is still split
    W = widen(Wd).astype(np.float64)
    bound = C_SUM * U24 * (np.abs(H) @ np.abs(W).T) + 1e-30
    assert np.all(np.abs(got - H @ W.T) <= bound)
    low, _ = run_gpu_with_hidden(*args, out_bf16=True)
    assert np.all(np.abs(low - got) <= 2.0 ** -8 * np.abs(got) + 1e-30)


# Partial sums of at most 16 MiB under a W_down of at most 64 MiB are stored past the L2, through a descriptor of 16 MiB: four
# splits of 2048 x 512 floats end where it ends, four of 1021 x 1016 just below and with tiles that end inside both, five of 1028 x 1048
# are above (tests/test_dispatch_cpu.py checks that the splits are these); 4096 x 8192 is 64 MiB in bf16.
@pytest.mark.parametrize("T,d_model,d_inter", [
    (65, 904, 4864), (129, 1032, 4096), (2048, 512, 2048), (1021, 1016, 2048), (1028, 1048, 4096), (65, 4096, 8192), (65, 4096, 8200)])
def test_partial_sums_around_the_store_limits(mm, T, d_model, d_inter):
    test_split_sum(mm, T, d_model, d_inter)
