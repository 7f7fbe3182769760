"""The projection kernels at the edges of their tiles: one request scored with
its first C candidates, C on both sides of the tile heights (32, 64, 128 and 256
rows) and at one row, for models whose projections have 2 to 32 k steps. Every
tile sums an output in the same order, so each score equals, bitwise, the one of
the whole candidate set; that one is checked against the oracle within the bf16
bar. Which tile a product takes is the choice of csrc/gemm_plan.h, compiled for
the host here: test_k_steps_of_every_tile says which pairs of tile and k steps
its calls reach."""
import numpy as np
import pytest

from paper_2607_28940_amd import inputs as I
from paper_2607_28940_amd.inputs import ModelConfig
from tests.parity_util import BF16_TOL, FP32_TOL, DeviceCase, check_err, log, oracle_request, score_err
from tests.plan_util import RING_STAGES, Plan

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


# Ring depths are 16, 6, 4, 6 and 4 stages (32x32 to 128x128): k steps fewer than
# half the depth, half, fewer than it, and more than it, odd and even
STEPS = {"k2": (ModelConfig(128, 1, 1088, 1, 1, rel_pos_buckets=16), (20, 900, 2600, 4000, 6000, 8200)),
         "k3": (ModelConfig(192, 3, 384, 1, 1, rel_pos_buckets=16), (130, 300, 900, 8200)),
         "k5": (ModelConfig(256, 2, 320, 1, 1, rel_pos_buckets=16), (20, 900, 2100, 8200)),
         "k7": (ModelConfig(256, 2, 448, 1, 1, rel_pos_buckets=16), (20, 900, 2100, 8200)),
         "k17": (ModelConfig(256, 2, 1088, 1, 1, rel_pos_buckets=16), (34, 900, 1300, 2100, 5000, 8200)),
         "k8": (ModelConfig(512, 4, 2048, 1, 1, rel_pos_buckets=16), (600, 4095, 4096, 4097, 4351, 4352, 4353))}
REACHED = {("32x32", "more, odd"), ("32x32", "fewer"), ("32x64", "more, odd"), ("32x64", "more, even"),
           ("32x64", "half"), ("32x64", "fewer"), ("64x64", "half"), ("64x64", "fewer"), ("64x64", "all"),
           ("64x64", "more, odd"), ("64x64", "more, even"), ("64x128", "more, odd"), ("64x128", "more, even"),
           ("128x128", "half"), ("128x128", "fewer"), ("128x128", "all"), ("128x128", "more, odd"),
           ("128x128", "more, even"), ("persistent", "rows at its tile"), ("persistent", "rows past its tile")}


def _reached(plan):
    seen = set()
    for model, counts in STEPS.values():
        d, F = model.d_model, model.d_ffn
        for C in counts + (max(counts) + 200,):
            for M, N, K in ((C + 3, 3 * d, d), (C, d, d), (C, F, d), (C, d, F)):
                if N % 128 or K % 64:
                    continue
                nk = K // 64
                for t, rows in plan.launches(M, N, K):
                    if t in RING_STAGES:
                        S = RING_STAGES[t]
                        seen.add((t, "half" if nk == S // 2 else "fewer" if nk < S else "all" if nk == S
                                  else "more, odd" if nk % 2 else "more, even"))
                    elif t == "persistent":
                        seen.add((t, "rows at its tile" if rows % 256 == 0 else "rows past its tile"))
    return seen


@pytest.mark.parametrize("name", STEPS)
def test_k_steps_of_every_tile(oracle_mod, tmp_path, name):
    import torch
    torch.cuda.set_device(0)
    assert REACHED <= _reached(Plan(tmp_path)), REACHED - _reached(Plan(tmp_path))
    model, counts = STEPS[name]
    n = max(counts) + 200
    wl = I.custom_workload(model, cfg_id=94, L=[70], S=[3], C=[n])
    w = I.make_weights(model, ("sharp", "affine"))
    run = DeviceCase(wl, w)
    run.build([0])
    Xc = I.request_tokens(wl, 0, I.STREAM_CANDIDATES)
    base = run.score([0], cand=[Xc])[0]
    assert np.all(np.isfinite(base))
    for C in counts:
        assert np.array_equal(run.score([0], cand=[Xc[:C]])[0], base[:C]), C
    err = score_err(base[-200:], oracle_request(oracle_mod.Oracle(model, w), wl, 0, cand=Xc[-200:])[0])
    log(f"k steps {name}: max err {err['max']:.3e}")
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


def test_f32_rows_past_the_grid():
    """fp32 calls of more rows than one launch's grid covers (65535 blocks of 16
    rows) run in row ranges on the same kernel: scores bitwise as in small calls."""
    import torch
    torch.cuda.set_device(0)
    model = F32["d64"]
    C = 16 * 65535 + 1000
    wl = I.custom_workload(model, cfg_id=95, L=[70], S=[3], C=[1])
    run = DeviceCase(wl, I.make_weights(model, ("sharp", "affine")))
    run.build([0])
    xs = run.dev(I.request_tokens(wl, 0, I.STREAM_SERVING))
    xc = torch.randn((C, model.d_model), generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    base = run.cache.score([0], xs, [0, 3], xc, [0, C])
    for a, b in ((0, 300), (16 * 65535 - 200, 16 * 65535 + 200), (C - 300, C)):
        part = run.cache.score([0], xs, [0, 3], xc[a:b].contiguous(), [0, b - a])
        assert torch.isfinite(part).all() and torch.equal(part, base[a:b]), (a, b)
