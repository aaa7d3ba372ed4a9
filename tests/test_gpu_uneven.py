"""bf16 tables whose branch boundaries are not multiples of 8 (d_model and d_inter are), through the automatic path:
the MFMA kernels with the partial 16-byte chunks at run boundaries added separately.  Against the oracle, H included,
with non-finite weights in every pruned branch."""
import numpy as np
import pytest

from gpu_util import check_bf16_flip_aware, flip_terms, run_gpu, run_gpu_with_hidden
from paper_2511_21089_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2511_21089_amd import binding
    return binding


TABLES = {
    # branch widths, active mask (the widths sum to a multiple of 8)
    "first_k": ([101, 101, 101, 100, 101], [1, 1, 1, 0, 0]),                  # one run, ends inside a chunk
    "first_off": ([101, 101, 101, 100, 101], [0, 1, 0, 1, 1]),                # runs start inside a chunk, one ends the layer
    "one_chunk": ([3, 2, 1, 2, 9, 130, 5], [0, 1, 0, 1, 0, 1, 0]),            # runs inside one chunk, two in the same one
    "no_interior": ([1, 7, 5, 3, 8, 1, 6, 1], [1, 0, 1, 0, 0, 0, 1, 1]),      # nothing but partial chunks
    "thin": ([1] * 64, [1, 0, 0] * 21 + [1]),                                 # 22 runs of one neuron
    "empty": ([0, 129, 0, 127, 0, 64], [1, 1, 1, 0, 1, 1]),                   # empty branches at a boundary
    "all_on": ([129, 255, 1, 127], [1, 1, 1, 1]),                             # one whole run: only the branch table is odd
    "tile_edges": ([127, 2, 127, 257, 63, 64], [1, 0, 1, 1, 0, 1]),           # boundaries around the tile sizes
}


def make(name, T, d_model, seed):
    widths, mask = TABLES[name]
    off = np.concatenate([[0], np.cumsum(widths)]).astype(np.int32)
    assert off[-1] % 8 == 0 and np.any(off % 8)
    rng = np.random.default_rng(seed)
    x, Wg, Wu, Wd = synth.random_layer(rng, T, d_model, int(off[-1]), dtype="bf16", w_scale=0.05)
    alpha = rng.uniform(0.8, 1.25, size=len(widths)).astype(np.float32)
    return x, Wg, Wu, Wd, off, alpha, np.array(mask, np.uint8)


def poison_pruned(args):
    x, Wg, Wu, Wd, off, alpha, mask = args
    Wg, Wu, Wd, alpha = Wg.copy(), Wu.copy(), Wd.copy(), alpha.copy()
    for b in np.flatnonzero(mask == 0):
        Wg[off[b]:off[b + 1]] = 0x7FC0        # NaN
        Wu[off[b]:off[b + 1]] = 0x7F80        # +inf
        Wd[:, off[b]:off[b + 1]] = 0xFF80     # -inf
    return x, Wg, Wu, Wd, off, alpha, mask


@pytest.mark.parametrize("T", [1, 17, 129, 600])
@pytest.mark.parametrize("name", sorted(TABLES))
def test_uneven_table(mm, name, T):
    args = make(name, T, 136 if T != 129 else 264, seed=T)
    bad = poison_pruned(args)
    got, H = run_gpu_with_hidden(*bad)
    off, mask = args[4], args[6]
    active = np.repeat(mask != 0, np.diff(off))
    assert np.all(np.isnan(H[:, ~active]))                       # columns of pruned branches are never written
    assert np.all(np.isfinite(got))
    check_bf16_flip_aware(got, H, *args, label="%s T=%d:" % (name, T))
    assert np.array_equal(run_gpu(*bad), got)                    # the entry point without a workspace argument
    # against the general kernels: no further apart than their stored H and two fp32 summations allow
    gen, Hg = run_gpu_with_hidden(*bad, path=mm.PATH_GENERIC)
    f, fg = flip_terms(H, *args), flip_terms(Hg, *args)
    assert np.all(np.abs(got - gen) <= np.abs(f["H"] - fg["H"]) @ f["aWd"].T + f["sum_err"] + fg["sum_err"] + 1e-30)
    if name == "all_on":
        return                                                   # its one run is aligned: any path takes it
    for p in (mm.PATH_MFMA, mm.PATH_MFMA_SLIM):                  # a forced path keeps its alignment requirement
        with pytest.raises(mm.MlpMoeError) as ei:
            run_gpu(*args, path=p)
        assert ei.value.status == mm.ERR_UNSUPPORTED


@pytest.mark.parametrize("T", [1, 17, 600])
@pytest.mark.parametrize("name", sorted(TABLES))
def test_uneven_table_routed(mm, name, T):
    args = make(name, T, 136, seed=100 + T)
    off, mask = args[4], args[6]
    rng = np.random.default_rng(T)
    route = (rng.uniform(size=(T, len(mask))) < 0.4).astype(np.uint8)
    if T > 256:
        route[:256, ::2] = 0                                     # a token tile nobody of which takes these branches
    route[T // 2] = 0
    got, H = run_gpu_with_hidden(*poison_pruned(args), route=route)
    assert np.all(np.isfinite(got))
    check_bf16_flip_aware(got, H, *args, route=route, label="%s routed T=%d:" % (name, T))
    assert not np.any(got[~np.any(route[:, mask != 0], axis=1)])


def test_uneven_split_k(mm):
    """A long K and few outputs: the K split, whose last part adds the partial chunks."""
    rng = np.random.default_rng(5)
    widths = [1003, 1003, 1003, 1002, 1002, 1003]
    off = np.concatenate([[0], np.cumsum(widths)]).astype(np.int32)
    x, Wg, Wu, Wd = synth.random_layer(rng, 200, 128, int(off[-1]), dtype="bf16")
    args = (x, Wg, Wu, Wd, off, rng.uniform(0.8, 1.25, size=6).astype(np.float32), np.array([1, 1, 0, 1, 1, 0], np.uint8))
    for out_bf16 in (False, True):
        got, H = run_gpu_with_hidden(*poison_pruned(args), out_bf16=out_bf16)
        assert np.all(np.isfinite(got))
        if not out_bf16:
            check_bf16_flip_aware(got, H, *args, label="split K:")
            ref = got
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-30)       # one rounding of the same sums


def test_uneven_silu_far_tail(mm):
    """SiLU(-88) = -5.3e-37: 1 / (1 + exp(88)) is below the smallest normal float, the quotient is not.  Such a gate with a large
    up value counts, on the kernels for odd boundaries as on the general ones."""
    one = {-88: 0xC2B0, 1: 0x3F80, 2 ** 120: 0x7B80}
    for T, route in ((1, None), (300, None), (300, 1)):
        x, Wg, Wu, Wd = (np.zeros(s, np.uint16) for s in ((T, 8), (256, 8), (256, 8), (8, 256)))
        x[:, 0], Wg[:3, 0], Wu[:3, 0], Wd[:, 0] = one[1], one[-88], one[2 ** 120], one[1]
        args = (x, Wg, Wu, Wd, np.array([0, 3, 256], np.int32), np.ones(2, np.float32), np.array([1, 0], np.uint8))
        route = None if route is None else np.ones((T, 2), np.uint8)
        got, H = run_gpu_with_hidden(*args, route=route)
        want = -88.0 / (1.0 + np.exp(88.0)) * 2.0 ** 120            # -0.71
        assert np.all(np.abs(H[:, :3] - want) <= 2.0 ** -8 * abs(want))
        assert np.array_equal(got, np.repeat(H[:, :1], 8, axis=1))
