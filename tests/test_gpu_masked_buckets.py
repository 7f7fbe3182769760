"""Relative-position buckets that mask (minus infinity, or so low that the
biased logit overflows to it) in the encoder's attention, and rows of the
history that are not finite. A bucket may leave a whole page, a key quarter or
a step of the softmax without a visible key before the first visible one."""
import numpy as np
import pytest

from paper_2607_28940_amd import inputs as I
from paper_2607_28940_amd.inputs import ModelConfig
from tests.parity_util import BF16_TOL, FP32_TOL, DeviceCase, log, oracle_request, tensor_err

pytestmark = pytest.mark.gpu

LENGTHS = [1, 17, 40, 64, 100, 300]
REL = 16  # index of "rel" in an encoder layer's tensors


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    torch.cuda.set_device(0)


def _case(model, w, fill_byte=0xFF, n_append=0, L=LENGTHS):
    n = len(L)
    wl = I.custom_workload(model, cfg_id=91, L=L, S=[1] * n, C=[1] * n, n_append=n_append)
    run = DeviceCase(wl, w, fill_byte=fill_byte)
    run.build(range(n))
    return run


@pytest.mark.parametrize("low", [-np.inf, -3e38])
@pytest.mark.parametrize("dh,dtype", [(32, "f32"), (64, "f32"), (128, "f32"), (32, "bf16"), (64, "bf16"), (128, "bf16")])
def test_masked_distances(oracle_mod, dh, dtype, low):
    """Distances 16 to 39 are masked, nearer and farther ones are visible: the
    first keys of queries 16 to 39, and whole key quarters of others, are
    masked. Second-layer keys against the oracle, within the type's bar."""
    model = ModelConfig(2 * dh if dh > 32 else 128, 2 if dh > 32 else 4, 256, 2, 1, rel_pos_buckets=64, dtype=dtype)
    w = I.make_weights(model, ("sharp", "affine"))
    for e in range(model.n_enc_layers):
        w[17 * e + REL] = w[17 * e + REL].copy()
        w[17 * e + REL][:, 16:40] = low
    run = _case(model, w)
    orc = oracle_mod.Oracle(model, w)
    worst = 0.0
    for r in range(len(LENGTHS)):
        _, st = oracle_request(orc, run.wl, r)
        e = tensor_err(run.cache.export(r, 0, 1).float().cpu().numpy(), st["K"][1])
        worst = max(worst, e)
        assert np.isfinite(e) and e < (FP32_TOL if dtype == "f32" else BF16_TOL), (LENGTHS[r], e)
    log(f"masked distances d_h {dh} {dtype} {low}: worst {worst:.3e}")


@pytest.mark.parametrize("low", [-np.inf, -3e38])
@pytest.mark.parametrize("heads", [2, 4])
@pytest.mark.parametrize("R,new", [(33, 0), (33, 9), (1030, 0)])
def test_masked_last_bucket(heads, R, new, low):
    """The last bucket masks every key past a window of R - 1 (histories of several
    pages have pages wholly outside it), with logits of several hundred, whose
    exponentials overflow unless a maximum is taken off. A bias of -1e4 leaves
    nothing of those keys either (e^-1e4 is 0 in fp32), so cached keys and
    values are bitwise the same; histories built whole (staged kernel, tables in
    LDS and in memory) and with 9 events appended (register kernel)."""
    model = ModelConfig(256, heads, 256, 2, 1, rel_pos_buckets=R)
    L = LENGTHS + [1400]
    got = []
    for b in (-1e4, low):
        w = I.make_weights(model, ("sharp", "affine"))
        for e in range(model.n_enc_layers):
            for i in (0, 2):  # Wq, Wk
                w[17 * e + i] = I._round_storage(8 * w[17 * e + i], model.dtype)
            w[17 * e + REL] = w[17 * e + REL].copy()
            w[17 * e + REL][:, -1] = b
        run = _case(model, w, n_append=new, L=L)
        if new:
            run.append(range(len(L)), 0, new)
        got.append([run.cache.export(r, part, layer).float().cpu().numpy() for r in range(len(L))
                    for part, layer in ((0, 1), (1, 1), (2, 0), (3, 0))])
    for a, b in zip(*got):
        assert np.all(np.isfinite(a)) and np.array_equal(a, b)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("dh", [32, 64, 128])
def test_later_rows_do_not_reach_earlier_ones(dh, bad):
    """fp32: a behavior token that is not finite spoils its own row and those
    after it; the rows before it are bitwise as without it (a key that a query
    does not see adds nothing, not zero times its value)."""
    model = ModelConfig(2 * dh, 2, 256, 2, 1, rel_pos_buckets=40, dtype="f32")
    w = I.make_weights(model, ("sharp", "affine"))
    L, at = 150, (20, 77, 149)
    wl = I.custom_workload(model, cfg_id=92, L=[L] * 4, S=[1] * 4, C=[1] * 4)
    run = DeviceCase(wl, w, fill_byte=0xFF)
    X = I.request_tokens(wl, 0, I.STREAM_BEHAVIOR)
    rows = [X] + [X.copy() for _ in at]
    for x, p in zip(rows[1:], at):
        x[p, 3] = bad
    run.cache.build(list(range(4)), run.dev(np.concatenate(rows)), I.offsets([L] * 4))
    for part, layer in ((0, 1), (1, 1), (2, 0), (3, 0)):
        clean = run.cache.export(0, part, layer).float().cpu().numpy()
        assert np.all(np.isfinite(clean))
        for r, p in enumerate(at):
            got = run.cache.export(1 + r, part, layer).float().cpu().numpy()
            assert np.array_equal(got[:p], clean[:p]), (part, layer, p)
            assert not np.all(np.isfinite(got[p])), (part, layer, p)
