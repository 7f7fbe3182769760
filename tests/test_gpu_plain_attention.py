"""The attention kernel of fp32 models and of 32-wide heads at the edges of its
key quarters: histories on both sides of 16, 32, 48 and 64 keys (quarters that
see no key, one, all of theirs), of several pages, and tiles of one query, of
a part of a 16-query group and of more than 64. Scores (cross-attention) and
the second encoder layer's keys (causal attention with relative bias) against
the oracle; unused pool bytes are NaN. Keys elementwise against their rms,
within the bar of the model's type, as the scores."""
import numpy as np
import pytest

from paper_2607_28940_amd import inputs as I
from paper_2607_28940_amd.inputs import ModelConfig
from tests.parity_util import BF16_TOL, FP32_TOL, DeviceCase, check_err, log, oracle_request, score_err, tensor_err

pytestmark = pytest.mark.gpu

LENGTHS = [1, 15, 16, 17, 33, 48, 49, 63, 64, 65, 130, 300]


@pytest.mark.parametrize("dh,dtype", [(32, "f32"), (64, "f32"), (128, "f32"), (32, "bf16")])
def test_plain_attention_edges(oracle_mod, dh, dtype):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    torch.cuda.set_device(0)
    model = ModelConfig(2 * dh if dh > 32 else 128, 2 if dh > 32 else 4, 256, 2, 1, rel_pos_buckets=40, dtype=dtype)
    n = len(LENGTHS)
    wl = I.custom_workload(model, cfg_id=86, L=LENGTHS, S=[r % 3 for r in range(n)],
                           C=[(1, 5, 17, 63, 64, 70)[r % 6] for r in range(n)])
    w = I.make_weights(model, ("sharp", "affine"))
    run = DeviceCase(wl, w, fill_byte=0xFF)
    run.build(range(n))
    scores = run.score(range(n))
    orc = oracle_mod.Oracle(model, w)
    worst = 0.0
    refs = []
    for r in range(n):
        ref, st = oracle_request(orc, wl, r)
        refs.append(ref)
        e = tensor_err(run.cache.export(r, 0, 1).float().cpu().numpy(), st["K"][1])
        worst = max(worst, e)
        assert np.isfinite(e) and e < (FP32_TOL if dtype == "f32" else BF16_TOL), (LENGTHS[r], e)
    err = score_err(np.concatenate(scores), np.concatenate(refs))
    log(f"plain attention d_h {dh} {dtype}: keys {worst:.3e} scores max {err['max']:.3e}")
    check_err(err, FP32_TOL if dtype == "f32" else BF16_TOL)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_plain_attention_independent_of_grid(dtype):
    """32-wide heads: more blocks than CUs take another variant of the kernel
    (two blocks per CU). A user's cached keys and scores are bitwise the same
    alone and among 130 users (4 heads: 520 blocks and more)."""
    import torch
    torch.cuda.set_device(0)
    model = ModelConfig(128, 4, 256, 2, 2, rel_pos_buckets=40, dtype=dtype)
    n, L = 130, [40 + (37 * r) % 200 for r in range(130)]
    wl = I.custom_workload(model, cfg_id=90, L=L, S=[r % 4 for r in range(n)], C=[1 + (7 * r) % 90 for r in range(n)])
    w = I.make_weights(model, ("sharp", "affine"))
    many, one = DeviceCase(wl, w), DeviceCase(wl, w)
    many.build(range(n))
    scores = many.score(range(n))
    for r in (0, 41, 129):
        one.build([r])
        assert np.array_equal(one.score([r])[0], scores[r]), r
        for part in (0, 1):
            assert torch.equal(one.cache.export(r, part, 1), many.cache.export(r, part, 1)), (r, part)
