"""The routed gate+up projection around full rounds of 256 live tiles: whole tiles, halves and quarters for what is left.
The intermediate of a batch whose tokens all take the same branches equals, bit for bit, the plain forward's with those
branches switched on."""
import numpy as np
import pytest

from gpu_util import C_SUM, U24, run_gpu_with_hidden, widen
from paper_2511_21089_amd import synth

pytestmark = pytest.mark.gpu

WIDTHS = np.array([64, 1, 63, 1, 128, 43]) * 128            # branches of so many tiles of 128 neurons
SUBSETS = {1: [1], 64: [0], 65: [0, 1], 128: [0, 1, 2], 129: [0, 1, 2, 3], 172: [4, 5, 1], 256: [0, 2, 3, 4],
           257: [0, 1, 2, 3, 4], 300: [0, 1, 2, 3, 4, 5]}   # live tiles -> branches


@pytest.mark.parametrize("T", [100, 200])
@pytest.mark.parametrize("tiles", sorted(SUBSETS))
def test_live_tiles(tiles, T):
    assert WIDTHS[SUBSETS[tiles]].sum() == tiles * 128
    off = np.concatenate([[0], np.cumsum(WIDTHS)]).astype(np.int32)
    rng = np.random.default_rng(tiles)
    x, Wg, Wu, Wd = synth.random_layer(rng, T, 64, int(off[-1]), dtype="bf16", w_scale=0.1)
    alpha = rng.uniform(0.8, 1.25, size=6).astype(np.float32)
    on = np.zeros(6, np.uint8)
    on[SUBSETS[tiles]] = 1
    got, H = run_gpu_with_hidden(x, Wg, Wu, Wd, off, alpha, np.ones(6, np.uint8), route=np.tile(on, (T, 1)))
    _, plain = run_gpu_with_hidden(x, Wg, Wu, Wd, off, alpha, on)
    active = np.repeat(on != 0, WIDTHS)
    assert np.array_equal(H[:, active], plain[:, active])
    Hd, W = np.where(active, plain, 0.0), widen(Wd).astype(np.float64)
    assert np.all(np.abs(got - Hd @ W.T) <= C_SUM * U24 * (np.abs(Hd) @ np.abs(W).T) + 1e-30)
