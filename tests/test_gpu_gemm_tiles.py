"""The projection kernels at the edges of their tiles: one request scored with
its first C candidates, C on both sides of every tile height (32, 64, 128 rows
and the persistent kernel's 256) and at one row, for models whose projections
have 2, 3, 4, 8 and 32 k steps (the ring of stages shorter than its depth, odd,
and longer). Every tile sums an output in the same order, so each score equals,
bitwise, the one of the whole candidate set; that one is checked against the
oracle within the bf16 bar."""
import numpy as np
import pytest

from paper_2607_28940_amd import inputs as I
from paper_2607_28940_amd.inputs import ModelConfig
from tests.parity_util import BF16_TOL, FP32_TOL, DeviceCase, check_err, log, oracle_request, score_err

pytestmark = pytest.mark.gpu

MODELS = {"k2": ModelConfig(128, 2, 256, 1, 1, rel_pos_buckets=16),
          "k3": ModelConfig(192, 3, 256, 1, 2, rel_pos_buckets=16),
          "k4-k6": ModelConfig(256, 2, 384, 1, 2, rel_pos_buckets=16),
          "k8-k32": ModelConfig(512, 8, 2048, 1, 2, rel_pos_buckets=16)}


@pytest.mark.parametrize("name", MODELS)
def test_score_independent_of_tile(oracle_mod, name):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    torch.cuda.set_device(0)
    model = MODELS[name]
    wl = I.custom_workload(model, cfg_id=81, L=[70], S=[3], C=[2600])
    w = I.make_weights(model, ("sharp", "affine"))
    run = DeviceCase(wl, w)
    run.build([0])
    Xc = I.request_tokens(wl, 0, I.STREAM_CANDIDATES)
    base = run.score([0], cand=[Xc])[0]
    assert np.all(np.isfinite(base))
    for C in (1, 28, 29, 30, 60, 61, 62, 125, 126, 253, 254, 600, 1300, 2100):
        assert np.array_equal(run.score([0], cand=[Xc[:C]])[0], base[:C]), C
    n = 300
    err = score_err(base[:n], oracle_request(oracle_mod.Oracle(model, w), wl, 0, cand=Xc[:n])[0])
    log(f"gemm tiles {name}: max err {err['max']:.3e} p99 {err['p99']:.3e}")
    check_err(err, BF16_TOL)


F32 = {"d64": ModelConfig(64, 2, 256, 1, 2, rel_pos_buckets=16, dtype="f32"),
       "d96": ModelConfig(96, 3, 112, 1, 2, rel_pos_buckets=16, dtype="f32")}


@pytest.mark.parametrize("name", F32)
def test_f32_score_independent_of_tile(oracle_mod, name):
    """The fp32 projections: 16x16 outputs per wave and, from 1024 tiles of
    32x32 on, 32x32; column counts that leave waves of a block idle, k of 4, 6
    and 7 chunks. Bitwise independent of the number of rows, and the fp32 bar
    against the oracle (which also covers 8 keys per softmax step on a history
    of 70)."""
    import torch
    torch.cuda.set_device(0)
    model = F32[name]
    wl = I.custom_workload(model, cfg_id=84, L=[70], S=[3], C=[17000])
    w = I.make_weights(model, ("sharp", "affine"))
    run = DeviceCase(wl, w)
    run.build([0])
    Xc = I.request_tokens(wl, 0, I.STREAM_CANDIDATES)
    base = run.score([0], cand=[Xc])[0]
    for C in (1, 12, 13, 14, 29, 30, 61, 300, 4100):
        assert np.array_equal(run.score([0], cand=[Xc[:C]])[0], base[:C]), C
    n = 300
    err = score_err(base[:n], oracle_request(oracle_mod.Oracle(model, w), wl, 0, cand=Xc[:n])[0])
    log(f"f32 gemm tiles {name}: max err {err['max']:.3e}")
    check_err(err, FP32_TOL)


@pytest.mark.parametrize("C", [9000, 33500])
def test_rows_past_the_full_rounds(C):
    """More 256x256 tiles than CUs with a part of a round left over (8 x 36 and
    2 x 131 tiles of the d 512 projections on 256 CUs): the rows past the full
    rounds run in smaller tiles. Same scores, bitwise, as in calls of few rows."""
    import torch
    torch.cuda.set_device(0)
    model = MODELS["k8-k32"]
    wl = I.custom_workload(model, cfg_id=88, L=[70], S=[3], C=[C])
    run = DeviceCase(wl, I.make_weights(model, ("sharp", "affine")))
    run.build([0])
    Xc = I.request_tokens(wl, 0, I.STREAM_CANDIDATES)
    base = run.score([0], cand=[Xc])[0]
    assert np.all(np.isfinite(base))
    for a, b in ((0, 300), (8100, 8300), (C // 2, C // 2 + 1), (max(0, 32768 - 200) if C > 32768 else 8185, C)):
        assert np.array_equal(run.score([0], cand=[Xc[a:b]])[0], base[a:b]), (a, b)


@pytest.mark.parametrize("S,C", [(0, 20000), (33, 20000), (40, 20051)])
def test_pair_kernel(oracle_mod, S, C):
    """Many 128x128 tiles of products that are none of the persistent kernel's
    (N 384 and 1152, K 128 and 384): two blocks per CU. The rows of one array
    and of two, partial last tiles. Bitwise as in calls of few rows, and in
    place as copied; the first scores against the oracle."""
    import torch
    torch.cuda.set_device(0)
    model = ModelConfig(384, 3, 128, 1, 2, rel_pos_buckets=16)
    wl = I.custom_workload(model, cfg_id=93, L=[70], S=[S], C=[C])
    w = I.make_weights(model, ("sharp", "affine"))
    run = DeviceCase(wl, w)
    run.build([0])
    Xc = I.request_tokens(wl, 0, I.STREAM_CANDIDATES)
    base = run.score([0], cand=[Xc])[0]
    assert np.all(np.isfinite(base))
    for a, b in ((0, 300), (C // 2, C // 2 + 130), (C - 200, C)):
        assert np.array_equal(run.score([0], cand=[Xc[a:b]])[0], base[a:b]), (a, b)
    xc = run.dev(np.concatenate([Xc.reshape(-1), np.zeros(1, np.float32)]))
    off = torch.empty_like(xc)[1:]
    off.copy_(xc[:-1])
    xs = run.dev(np.concatenate([I.request_tokens(wl, 0, I.STREAM_SERVING), np.zeros((1, 384), np.float32)]))
    copied = run.cache.score([0], xs, [0, S], off, [0, C]).cpu().numpy().astype(np.float64)
    assert np.array_equal(copied, base)
    err = score_err(base[:200], oracle_request(oracle_mod.Oracle(model, w), wl, 0, cand=Xc[:200])[0])
    log(f"pair kernel S {S} C {C}: max err {err['max']:.3e}")
    check_err(err, BF16_TOL)


@pytest.mark.parametrize("S,C", [(0, 5), (1, 1), (33, 70), (129, 2200)])
@pytest.mark.parametrize("name,model", [("bf16", MODELS["k4-k6"]), ("f32", F32["d64"])])
def test_tokens_in_place_or_copied(name, model, S, C):
    """The first layer reads aligned token arrays where they are (rows of two
    arrays in one product, the serving rows ending inside a tile); tokens one
    element off a 16-byte boundary are copied first. Same scores, bitwise."""
    import torch
    torch.cuda.set_device(0)
    wl = I.custom_workload(model, cfg_id=85, L=[70], S=[S], C=[C])
    run = DeviceCase(wl, I.make_weights(model, ("sharp", "affine")))
    run.build([0])
    xs = run.dev(np.concatenate([I.request_tokens(wl, 0, I.STREAM_SERVING), np.zeros((1, model.d_model), np.float32)]))
    xc = run.dev(I.request_tokens(wl, 0, I.STREAM_CANDIDATES))

    def off(x):
        y = torch.empty(x.numel() + 1, dtype=x.dtype, device=x.device)[1:]
        y.copy_(x.reshape(-1))
        return y
    a = run.cache.score([0], xs, [0, S], xc, [0, C]).cpu().numpy()
    b = run.cache.score([0], off(xs), [0, S], off(xc), [0, C]).cpu().numpy()
    assert np.all(np.isfinite(a)) and np.array_equal(a, b)
