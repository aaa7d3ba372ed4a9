"""The routed gate+up projection around full rounds of 256 live tiles: whole tiles, halves and quarters for what is left.
The intermediate of a batch whose tokens all take the same branches equals, bit for bit, the plain forward's with those
branches switched on."""
import numpy as np
import pytest

from gpu_util import C_SUM, U24, check_bf16_flip_aware, run_gpu_with_hidden, widen
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


@pytest.mark.parametrize("tiles_n", [4096, 4097])
def test_widest_tile_list(tiles_n):
    """More N tiles than 16-bit list entries hold: 4096 tiles of 128 neurons for each of 8 token tiles."""
    off = np.array([0, 64, tiles_n * 64 + 32, tiles_n * 128 - 8, tiles_n * 128], np.int32)
    T, rng = 130, np.random.default_rng(tiles_n)
    x, Wg, Wu, Wd = synth.random_layer(rng, T, 8, int(off[-1]), dtype="bf16", w_scale=0.1)
    alpha, on = rng.uniform(0.8, 1.25, size=4).astype(np.float32), np.array([1, 0, 1, 1], np.uint8)
    route = np.tile(on, (T, 1))
    route[128:, 3] = 0
    got, H = run_gpu_with_hidden(x, Wg, Wu, Wd, off, alpha, np.ones(4, np.uint8), route=route)
    plain_out, plain = run_gpu_with_hidden(x, Wg, Wu, Wd, off, alpha, on)
    active = np.repeat(on != 0, np.diff(off))
    assert np.array_equal(H[:128, active], plain[:128, active])
    assert np.array_equal(H[128:, active][:, :-8], plain[128:, active][:, :-8]) and not H[128:, -8:].any()
    bound = C_SUM * U24 * (np.abs(plain[:, active]) @ np.abs(widen(Wd)[:, active]).T.astype(np.float64))
    assert np.all(np.abs(got - plain_out)[:128] <= 2 * bound[:128])


@pytest.mark.parametrize("T", [100, 128, 129, 256, 300, 700, 2100])
@pytest.mark.parametrize("widths", [[128, 256, 64, 192, 128, 320], [4096, 2048, 8192, 4096], [101, 259, 65, 191, 130, 318]],
                         ids=["small", "rounds", "odd"])
def test_halves_of_token_tiles(widths, T):
    """Halves of 256-token tiles that take other branches than the other half, branches that nobody takes, and halves that take
    nothing: what one half alone needs is computed for it, and the other half's H is 0, not what the workspace held (NaN)."""
    B = len(widths)
    off = np.concatenate([[0], np.cumsum(widths)]).astype(np.int32)
    rng = np.random.default_rng(T + B)
    x, Wg, Wu, Wd = synth.random_layer(rng, T, 64, int(off[-1]), dtype="bf16", w_scale=0.1)
    alpha = rng.uniform(0.8, 1.25, size=B).astype(np.float32)
    route = np.zeros((T, B), np.uint8)
    for lo in range(0, T, 128):
        take = rng.uniform(size=B) < 0.4
        route[lo:lo + 128] = take & (rng.uniform(size=(min(128, T - lo), B)) < 0.9)
    mask = np.ones(B, np.uint8)
    mask[B - 1] = 0
    args = (x, Wg, Wu, Wd, off, alpha, mask)
    got, H = run_gpu_with_hidden(*args, route=route)
    check_bf16_flip_aware(got, H, *args, route=route, label="halves:")
