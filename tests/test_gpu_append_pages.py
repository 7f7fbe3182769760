"""Appends at the edges of the causal page classes: histories of 1 to 9 pages,
the appended events ending inside, at and after a page boundary, 1 to 32 new
events, head widths 64 and 128, relative-position tables of 0 buckets, shorter
than a page, of two pages and the largest that the append kernel holds. Cached
keys and values past the first layer against a rebuild of the whole history on
the staged kernel. Unused pool bytes are NaN."""
import numpy as np
import pytest

from paper_2607_28940_amd import inputs as I
from paper_2607_28940_amd.inputs import ModelConfig
from tests.parity_util import DeviceCase, log

pytestmark = pytest.mark.gpu

LENGTHS = [1, 40, 63, 64, 100, 127, 128, 250, 255, 256, 400, 560]


@pytest.mark.parametrize("R", [0, 1, 33, 128, 256])
@pytest.mark.parametrize("heads", [2, 4])
@pytest.mark.parametrize("new", [1, 17, 32])
def test_append_page_classes(heads, R, new):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    torch.cuda.set_device(0)
    model = ModelConfig(256, heads, 256, 2, 1, rel_pos_buckets=R)
    w = I.make_weights(model, ("sharp", "affine"))
    n = len(LENGTHS)
    wl = I.custom_workload(model, cfg_id=87, L=LENGTHS, S=[1] * n, C=[1] * n, n_append=new)
    inc = DeviceCase(wl, w, fill_byte=0xFF)
    inc.build(range(n))
    inc.append(range(n), 0, new)
    full = DeviceCase(wl, w)
    X = [np.concatenate([I.request_tokens(wl, r, I.STREAM_BEHAVIOR), I.request_tokens(wl, r, I.STREAM_EVENTS)])
         for r in range(n)]
    full.cache.build(list(range(n)), full.dev(np.concatenate(X)), I.offsets([len(x) for x in X]))
    worst = 0.0
    for r in range(n):
        for part, layer in ((0, 1), (1, 1), (2, 0), (3, 0)):
            a = inc.cache.export(r, part, layer).float().cpu().numpy()
            b = full.cache.export(r, part, layer).float().cpu().numpy()
            # two correct results differ by their sums' order (1e-2 of the rms) before
            # each is rounded to bf16, which may then fall on neighbouring values:
            # one unit in the last place, at most 2^-7 of the value
            ulp = np.maximum(np.abs(a), np.abs(b)) / 128
            e = float(np.max(np.maximum(np.abs(a - b) - ulp, 0)) / np.sqrt(np.mean(np.square(b))))
            worst = max(worst, e)
            assert np.all(np.isfinite(a)) and e < 1e-2, (LENGTHS[r], part, layer, e)
    log(f"append {new} heads {heads} R {R}: worst {worst:.3e}")
