"""The encoder's causal attention at the edges of its page classes: histories
on both sides of a page and of a 128-query tile, relative-position tables of
0, 1, 33 and 128 buckets (from LDS) and of 1100 (from memory), head widths 128
and 64, with sharp logits and biases of several units. The second layer's
keys and values and the cross-attention's depend on every attended pair of the
first layer; they are compared with the oracle's as the cache-content test
does (2e-2 of their rms, elementwise). The pool starts as NaN bytes, so
nothing past a history may reach them."""
import numpy as np
import pytest

from paper_2607_28940_amd import inputs as I
from paper_2607_28940_amd.inputs import ModelConfig
from tests.parity_util import DeviceCase, log, oracle_request, tensor_err

pytestmark = pytest.mark.gpu

LENGTHS = [1, 63, 64, 65, 127, 129, 192, 257, 420, 1300]


@pytest.mark.parametrize("R", [0, 1, 33, 128, 1100])
@pytest.mark.parametrize("heads", [2, 4])
def test_causal_attention_pages(oracle_mod, heads, R):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    torch.cuda.set_device(0)
    model = ModelConfig(256, heads, 512, 2, 1, rel_pos_buckets=R)
    n = len(LENGTHS)
    wl = I.custom_workload(model, cfg_id=82, L=LENGTHS, S=[1] * n, C=[1] * n)
    w = I.make_weights(model, ("sharp", "affine"))
    run = DeviceCase(wl, w, fill_byte=0xFF)
    run.build(range(n))
    orc = oracle_mod.Oracle(model, w)
    worst = 0.0
    for r in range(n):
        _, st = oracle_request(orc, wl, r)
        for part, layer, ref in ((0, 1, st["K"][1]), (1, 1, st["V"][1]), (2, 0, st["Kx"][0]), (3, 0, st["Vx"][0])):
            e = tensor_err(run.cache.export(r, part, layer).float().cpu().numpy(), ref)
            worst = max(worst, e)
            assert np.isfinite(e) and e < 2e-2, (LENGTHS[r], part, layer, e)
    log(f"causal pages heads {heads} R {R}: worst {worst:.3e}")
