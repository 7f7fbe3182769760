"""Decoder cross-attention of small batches: histories of 32 pages and more are
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
                                   ([577, 2050], [64, 3], [193, 126]), ([5000], [5], [700]), ([2040], [0], [1]),
                                   ([2600, 1985, 511, 64], [7, 1, 0, 2], [122, 8, 9, 5])])
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


def test_short_histories_do_not_depend_on_the_batch():
    """A request of fewer than 32 pages is never split: its scores are bitwise
    the same alone, with a part of its candidates, among few and many other
    users and in workspace-sized passes. From 32 pages on the parts depend on
    the batch; the scores then agree within 1e-2 of their rms (the order of fp32
    sums and the rounding of probabilities to bf16 against another maximum, as
    when an append is compared with a rebuild)."""
    import torch
    torch.cuda.set_device(0)
    model = ModelConfig(256, 2, 512, 1, 2, rel_pos_buckets=16)
    L = [600, 1500, 1984, 470, 2040, 5000]
    n = len(L)
    wl = I.custom_workload(model, cfg_id=89, L=L, S=[5, 0, 33, 2, 7, 3], C=[150, 140, 130, 9, 120, 260])
    run = DeviceCase(wl, I.make_weights(model, ("sharp", "affine")), fill_byte=0xFF)
    run.build(range(n))
    Xs = [I.request_tokens(wl, r, I.STREAM_SERVING) for r in range(n)]
    Xc = [I.request_tokens(wl, r, I.STREAM_CANDIDATES) for r in range(n)]

    def score(ids, cand, **kw):
        s = run.dev(np.concatenate([Xs[i] for i in ids] + [np.zeros((1, model.d_model), np.float32)]))
        so, co = I.offsets([len(Xs[i]) for i in ids]), I.offsets([len(c) for c in cand])
        out = run.cache.score_events(ids, [L[i] for i in ids], s, so, run.dev(np.concatenate(cand)), co, **kw)
        out = out.cpu().numpy().astype(np.float64)
        return [out[co[k]:co[k + 1]] for k in range(len(ids))]

    alone = [score([r], [Xc[r]])[0] for r in range(n)]
    few = score(list(range(n)), Xc)
    many = score(list(range(n)) * 40, Xc * 40)
    need = run.cache.workspace_min_bytes(2, n, I.offsets(wl.S), I.offsets(wl.C))
    passes = score(list(range(n)), Xc, ws_limit=need)
    for r in range(n):
        part = score([r], [Xc[r][-3:]])[0]
        for got, want in ((few[r], alone[r]), (many[r], alone[r]), (many[r + 39 * n], alone[r]), (passes[r], alone[r]),
                          (part, alone[r][-3:])):
            assert np.all(np.isfinite(got))
            if L[r] < 32 * 64 - 63:
                assert np.array_equal(got, want), L[r]
            else:
                assert np.max(np.abs(got - want)) < 1e-2 * np.sqrt(np.mean(np.square(alone[r]))), L[r]
