"""Float storage on the float MFMA kernels (d_model and d_inter multiples of 4): token and feature tails, K tails, runs
that start and end inside a 16-byte chunk, the K split with and without room for its partial sums.  Against float64,
with the error fp32 sums may have and non-finite weights in every pruned branch."""
import numpy as np
import pytest

import oracle
from gpu_util import C_SUM, U24, run_gpu
from paper_2511_21089_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2511_21089_amd import binding
    return binding


TABLES = {
    "even": ([64, 128, 36, 132], [1, 0, 1, 1]),
    "all_on": ([101, 101, 101, 101], [1, 1, 1, 1]),
    "first_k": ([101, 101, 101, 100, 101], [1, 1, 1, 0, 0]),
    "first_off": ([101, 101, 101, 100, 101], [0, 1, 0, 1, 1]),
    "one_chunk": ([1, 1, 1, 1, 9, 130, 5], [0, 1, 0, 1, 0, 1, 0]),
    "no_interior": ([1, 3, 5, 3, 4, 1, 2, 1], [1, 0, 1, 0, 0, 0, 1, 1]),
    "thin": ([1] * 64, [1, 0, 0] * 21 + [1]),
    "tile_edges": ([31, 1, 33, 63, 65, 31], [1, 0, 1, 1, 0, 1]),
}


def make(widths, mask, T, d_model, seed):
    off = np.concatenate([[0], np.cumsum(widths)]).astype(np.int32)
    assert off[-1] % 4 == 0
    rng = np.random.default_rng(seed)
    x, Wg, Wu, Wd = synth.random_layer(rng, T, d_model, int(off[-1]), dtype="f32", w_scale=0.05)
    alpha = rng.uniform(0.8, 1.25, size=len(widths)).astype(np.float32)
    return x, Wg, Wu, Wd, off, alpha, np.array(mask, np.uint8)


def poison_pruned(args):
    x, Wg, Wu, Wd, off, alpha, mask = args
    Wg, Wu, Wd = Wg.copy(), Wu.copy(), Wd.copy()
    for b in np.flatnonzero(mask == 0):
        Wg[off[b]:off[b + 1]] = np.nan
        Wu[off[b]:off[b + 1]] = np.inf
        Wd[:, off[b]:off[b + 1]] = -np.inf
    return x, Wg, Wu, Wd, off, alpha, mask


def check(got, x, Wg, Wu, Wd, off, alpha, mask, floor=1e-30):
    h, g, u, ag, au = oracle.mlpmoe_hidden(x, Wg, Wu, off, alpha, mask, "exact", details=True)
    a = np.repeat(alpha.astype(np.float64) * (mask != 0), np.diff(off))
    sig = 1.0 / (1.0 + np.exp(-g))
    # first-order error of h under the errors of its two fp32 sums, and a few fp32 roundings of h itself
    eg, eu = C_SUM * U24 * ag, C_SUM * U24 * au
    dh = np.abs(a) * (np.abs(sig * (1.0 + g * (1.0 - sig)) * u) * eg + np.abs(g * sig) * eu + eg * eu) + C_SUM * U24 * np.abs(h)
    h = np.where(a != 0, h, 0.0)
    dh = np.where(a != 0, dh, 0.0)
    aWd = np.abs(Wd.astype(np.float64))
    allow = dh @ aWd.T + C_SUM * U24 * (np.abs(h) @ aWd.T)
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - h @ Wd.astype(np.float64).T) <= allow + floor)


@pytest.mark.parametrize("T,d_model", [(1, 68), (17, 4), (64, 96), (65, 132), (300, 64)])
@pytest.mark.parametrize("name", sorted(TABLES))
def test_f32_table(mm, name, T, d_model):
    args = make(*TABLES[name], T, d_model, seed=T)
    got = run_gpu(*poison_pruned(args))
    check(got, *args)


@pytest.mark.parametrize("T", [3, 130])
def test_f32_split_k_and_small_workspace(mm, T):
    import torch
    args = make([1003, 1003, 1003, 1003], [1, 1, 0, 1], T, 64, seed=9)
    bad = poison_pruned(args)
    x, Wg, Wu, Wd, off, alpha, mask = bad
    dev = [torch.from_numpy(a).cuda() for a in (x, Wg, Wu, Wd)]
    full = mm.mlpmoe_workspace_bytes(T, 64, int(off[-1]), 4, 4)
    hidden = (T * mm.mlpmoe_hidden_ld(int(off[-1])) * 4 + 255) // 256 * 256     # float, rows of mlpmoe_hidden_ld
    # a byte short of the room for all partial sums: none are used
    for n in (full, full - 1):
        ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
        out = torch.full((T, 64), float("nan"), dtype=torch.float32, device="cuda")
        mm.mlpmoe_forward_f32_ws(*dev, off, alpha, mask, ws, out=out)
        torch.cuda.synchronize()
        check(out.cpu().numpy(), *args)
    with pytest.raises(mm.MlpMoeError) as ei:
        mm.mlpmoe_forward_f32_ws(*dev, off, alpha, mask, ws[:hidden], out=out)
    assert ei.value.status == mm.ERR_WORKSPACE


@pytest.mark.parametrize("widths,mask,T,d_model", [
    ([2048, 2048], [1, 1], 3, 64),                       # even runs
    ([1003, 1003, 1003, 1003], [1, 1, 0, 1], 130, 68),   # edge chunks, added by the last split
    ([36, 4] * 32, [1, 0] * 32, 17, 64),                 # short runs: more K tiles than the width adds up to
    ([1024, 1024], [1, 1], 100, 896), ([1003, 1003, 1002], [1, 0, 1], 250, 512), ([900] * 4, [1] * 4, 200, 1280),   # splits in groups
])
def test_f32_same_bits_in_any_block(mm, widths, mask, T, d_model):
    """Where the partial sums of a K split are kept, or that there is no room for them, does not show in the result."""
    import torch
    args = make(widths, mask, T, d_model, seed=T)
    x, Wg, Wu, Wd, off, alpha, mask = poison_pruned(args)
    dev = [torch.from_numpy(a).cuda() for a in (x, Wg, Wu, Wd)]
    full = mm.mlpmoe_workspace_bytes(T, d_model, int(off[-1]), len(alpha), 4)
    # bf16 with so many output tiles that nothing is split: the same block but for H
    hidden = [(T * mm.mlpmoe_hidden_ld(int(off[-1])) * e + 255) // 256 * 256 for e in (2, 4)]
    least = mm.mlpmoe_workspace_bytes(T, 1 << 22, int(off[-1]), len(alpha), 2) - hidden[0] + hidden[1]
    assert least < full                                  # K is split
    results = []
    part = T * d_model * 4
    for n in [full, full + 4096, full - 1, (least + full) // 2] + list(range(least, full, part)):
        ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
        out = torch.full((T, d_model), float("nan"), dtype=torch.float32, device="cuda")
        mm.mlpmoe_forward_f32_ws(*dev, off, alpha, mask, ws, out=out)
        torch.cuda.synchronize()
        results.append(out.cpu().numpy())
    check(results[0], *args)
    for r in results[1:]:
        assert np.array_equal(r, results[0])
    status = None
    try:
        mm.mlpmoe_forward_f32_ws(*dev, off, alpha, mask, ws[:least - 1], out=out)
    except mm.MlpMoeError as e:
        status = e.status
    assert status == mm.ERR_WORKSPACE


@pytest.mark.parametrize("T", [31, 32, 97, 128, 129, 250])
@pytest.mark.parametrize("widths,mask", [([4864], [1]), ([1621, 1621, 1622], [1, 0, 1])])
def test_f32_token_tiles(mm, widths, mask, T):
    """Gate+up tiles of 32 tokens (with two and with four K tiles ahead) and of 64, full and partly filled."""
    args = make(widths, mask, T, 72, seed=T)
    check(run_gpu(*poison_pruned(args)), *args)


@pytest.mark.parametrize("T,d_model,widths", [(5, 64, [64, 64]), (70, 132, [129, 129, 258]), (40, 72, [4864])])
def test_f32_infinities(mm, T, d_model, widths):
    """Infinities, NaNs and sums that overflow, in x and in every matrix: each result is the infinity or NaN that float
    arithmetic gives, and everything else what it is without them."""
    x, Wg, Wu, Wd, off, alpha, mask = make(widths, [1] * len(widths), T, d_model, seed=3)
    x[4] *= 1e-30
    clean = [a.copy() for a in (x, Wg, Wu, Wd)]
    x[1, 3], x[2, 5], x[3, 7] = np.inf, np.nan, 3e38
    Wg[10, 7], Wu[20, 9], Wd[4, 11], Wd[6, 13] = 2.0, -np.inf, np.inf, np.nan
    clean[1][10, 7] = 2.0
    got = run_gpu(x, Wg, Wu, Wd, off, alpha, mask)
    a = np.repeat(alpha, np.diff(off))
    with np.errstate(all="ignore"):
        g, u = x @ Wg.T, x @ Wu.T
        ref = (a * (g / (1 + np.exp(-g)) * u)) @ Wd.T
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]) and np.array_equal(np.isinf(got), np.isinf(ref))
    rows, cols = [0, 4], [m for m in range(d_model) if m not in (4, 6)]
    Wu[20, 9], Wd[4, 11], Wd[6, 13] = clean[2][20, 9], clean[3][4, 11], clean[3][6, 13]
    got = run_gpu(x, Wg, Wu, Wd, off, alpha, mask)[rows]
    check(got[:, cols], clean[0][rows], clean[1], clean[2], clean[3][cols], off, alpha, mask)


@pytest.mark.parametrize("T", [70, 256])
@pytest.mark.parametrize("scale", [1e-30, 1e-36, 1e30])
def test_f32_magnitudes(mm, T, scale):
    """Floats of any normal magnitude with all their 24 bits: tiny or huge x against W_gate and W_up the other way round, whose
    products are of order 1, and tiny or huge W_down under results as tiny or huge."""
    x, Wg, Wu, Wd, off, alpha, mask = make([64, 100], [1, 1], T, 64, seed=T)
    up, down = np.float32(scale), np.float32(1 / scale)
    a = (x * up, Wg * down, Wu * down, Wd, off, alpha, mask)
    check(run_gpu(*a), *a)
    a = (x, Wg, Wu, Wd * up, off, alpha, mask)
    check(run_gpu(*a), *a, floor=1e-44)


@pytest.mark.parametrize("n", [4, 8, 896])
def test_f32_error_of_sums(mm, n):
    """Rounding n partial sums, of which the k-th has k / n of the variance of the last, leaves an error of sqrt(n / 6) U24 of a sum (a
    rounding has 1 / 3 U24^2), two chains of half the length (from 17 products on) sqrt(n / 12) U24; g, u and three roundings of h
    itself sqrt(n / 3 / chains + 1) U24 in the 2-norm: 1.5, 1.9 and 12.3 U24.  Short sums show what a product loses, the long one
    the chains."""
    import torch
    T = 256
    args = make([64], [1], T, n, seed=n)
    x, Wg, Wu, Wd, off, alpha, mask = [a * np.float32(20 / n ** 0.5) if i in (1, 2) else a for i, a in enumerate(args)]
    ws = mm.new_workspace(T, n, 64, 1, 4)
    dev = [torch.from_numpy(a).cuda() for a in (x, Wg, Wu, Wd)]
    mm.mlpmoe_forward_f32_ws(*dev, off, alpha, mask, ws)
    torch.cuda.synchronize()
    h = ws[:T * 64 * 4].view(torch.float32).view(T, 64).cpu().numpy().astype(np.float64)
    want = oracle.mlpmoe_hidden(x, Wg, Wu, off, alpha, mask, "exact")
    bound = (n / 3 / (2 if n > 16 else 1) + 1) ** 0.5 * U24
    assert np.linalg.norm(h - want) <= (2 * U24 if n <= 8 else bound) * np.linalg.norm(want)
