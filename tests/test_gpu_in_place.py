"""A result stored over x: every kernel that reads x has ended before anything of the result is written, so that the bits are
those of a call with a buffer of its own.  Decode and prefill kernels, float and bf16 results, odd boundaries, routing."""
import numpy as np
import pytest

from paper_2511_21089_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 4, 8, 9, 16, 40])
@pytest.mark.parametrize("kind,d_model,widths", [
    ("f32", 68, [64, 300]), ("f32", 2048, [2051, 2045]), ("bf16", 896, [2048, 2048]), ("bf16", 896, [2051, 2045]),
    ("bf16", 2048, [2048, 512]), ("out_bf16", 896, [2048, 2048]), ("out_bf16", 896, [2051, 2045]), ("routed", 896, [2048, 512])])
def test_in_place(kind, d_model, widths, T):
    import torch
    from gpu_util import to_dev
    from paper_2511_21089_amd import binding as mm
    off = np.concatenate([[0], np.cumsum(widths)]).astype(np.int32)
    alpha, mask = np.array([1.1, 0.9], np.float32), np.ones(2, np.uint8)
    rng = np.random.default_rng(T + d_model)
    x, *W = synth.random_layer(rng, T, d_model, int(off[-1]), dtype="f32" if kind == "f32" else "bf16", w_scale=0.05)
    x, W = to_dev(x), [to_dev(w) for w in W]
    f = {"f32": mm.mlpmoe_forward_f32, "out_bf16": mm.mlpmoe_forward_bf16_out_bf16, "bf16": mm.mlpmoe_forward_bf16,
         "routed": mm.mlpmoe_forward_routed_bf16}[kind]
    more = (torch.ones((T, 2), dtype=torch.uint8, device="cuda"),) if kind == "routed" else ()
    want = f(x, *W, off, alpha, mask, *more).clone()
    over = torch.empty((T, d_model), dtype=want.dtype, device="cuda")
    mine = over.view(-1).view(x.dtype)[-T * d_model:].view(T, d_model)      # bf16 under a float result: its second half
    for _ in range(3):
        mine.copy_(x)
        f(mine, *W, off, alpha, mask, *more, out=over)
        assert torch.equal(over, want)
