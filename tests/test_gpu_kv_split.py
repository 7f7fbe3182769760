"""Decoder cross-attention of small batches: histories of 8 pages and more are
split into parts of at least 4 pages, shorter ones run whole in the same
launch; query counts on both sides of a tile (128) and of a merge block (8).
Scores within the bf16 bar of the oracle, and bitwise the same when the
candidates are reversed (the plan depends on counts and lengths only)."""
import numpy as np
import pytest

from paper_2607_28940_amd import inputs as I
from paper_2607_28940_amd.inputs import ModelConfig
from tests.parity_util import BF16_TOL, DeviceCase, check_err, log, oracle_request, score_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,S,C", [([512], [0], [1]), ([1090, 511, 64], [7, 1, 0], [122, 8, 9]),
                                   ([577, 2050], [64, 3], [193, 126]), ([5000], [5], [700])])
def test_small_batch_split(oracle_mod, L, S, C):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    torch.cuda.set_device(0)
    model = ModelConfig(256, 2, 512, 1, 2, rel_pos_buckets=16)
    wl = I.custom_workload(model, cfg_id=83, L=L, S=S, C=C)
    w = I.make_weights(model, ("sharp", "affine"))
    run = DeviceCase(wl, w, fill_byte=0xFF)
    run.build(range(wl.B))
    base = run.score(range(wl.B))
    orc = oracle_mod.Oracle(model, w)
    o = np.concatenate([oracle_request(orc, wl, r)[0] for r in range(wl.B)])
    err = score_err(np.concatenate(base), o)
    log(f"small-batch split {L}: max err {err['max']:.3e} p99 {err['p99']:.3e}")
    check_err(err, BF16_TOL)
    cand = [I.request_tokens(wl, r, I.STREAM_CANDIDATES)[::-1].copy() for r in range(wl.B)]
    rev = run.score(range(wl.B), cand=cand)
    for r in range(wl.B):
        assert np.array_equal(rev[r], base[r][::-1]), r
