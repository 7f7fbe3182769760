"""Tile choice of the bf16 products (csrc/gemm_plan.h), compiled for the host:
shapes whose kernel was measured, and bounds of the persistent kernel's share
of the rows."""
import random

import pytest

from tests.plan_util import TILES, Plan


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return Plan(tmp_path_factory.mktemp("plan"))


# (M, N, K): the kernel, and a slower one (us, each launch on operands of its own)
MEASURED = [
    ((66500, 1152, 384), "pair"),        # 130; 128x128 ring 143
    ((33000, 384, 128), "pair"),         # 18.0; 21.3
    ((131200, 384, 384), "pair"),        # 92.6; 102
    ((66500, 640, 640), "pair"),         # 107; 112
    ((50000, 1920, 640), "pair"),        # the pair kernel's own range
    ((33000, 512, 2048), "persistent"),  # 91.3; 107.5
    ((4000, 1536, 512), "persistent"),   # 16.4; 18.1
    ((10240, 2048, 512), "persistent"),  # 30.3; 32.0
    ((24000, 256, 1024), "persistent"),  # 27.5; 30.6
    ((66500, 4096, 1024), "persistent"),
    ((6327, 512, 2048), "128x128"),      # 18.9; pair 29.7, persistent 39.8
    ((3000, 512, 2048), "64x128"),       # 12.7; 128x128 16.2
    ((600, 1024, 1024), "64x64"),        # 6.1; 128x128 10.4, pair 16.0
    ((34, 512, 2048), "32x32"),          # 6.3; 128x128 12.8, pair 25.2
]


@pytest.mark.parametrize("shape,want", MEASURED)
def test_measured_choices(plan, shape, want):
    assert plan.tile(*shape) == want


def test_every_choice_is_possible(plan):
    rng = random.Random(1)
    seen = set()
    for _ in range(20000):
        M, N, K = int(2 ** rng.uniform(0, 18)), 128 * rng.randrange(1, 65), 64 * rng.randrange(1, 129)
        t = plan.tile(M, N, K)
        seen.add(t)
        if t == "persistent":
            assert N % 256 == 0 and K % 128 == 0 and K >= 256 and M >= 2048
            m1 = plan.rows(M, N, K)
            assert 0 < m1 <= M and (m1 == M or m1 % 256 == 0)
    assert seen == set(TILES)


def test_split_rows_stay_on_the_persistent_kernel(plan):
    """The rows split off for full rounds are rows the persistent kernel takes
    (at least 2048): with wide outputs a round has fewer, and a smaller share
    would run on the other kernels though charged as a persistent round."""
    rng = random.Random(2)
    split = 0
    for _ in range(20000):
        M, N, K = int(2 ** rng.uniform(11, 18)), 256 * rng.randrange(1, 65), 128 * rng.randrange(2, 65)
        m1 = plan.rows(M, N, K)
        split += m1 < M
        assert m1 == M or m1 >= 2048, (M, N, K, m1)
    assert split > 500


@pytest.mark.parametrize("M", [1, 300, 5000, 100000])
@pytest.mark.parametrize("N,K", [(131072, 16384), (16384, 131072), (65536, 32768)])
def test_weights_past_2_31_elements(plan, M, N, K):
    """Only the pair kernel addresses the weight with 64 bits."""
    assert N * K >= 2 ** 31 and plan.tile(M, N, K) == "pair"
    assert plan.tile(M, N, K - 128) != "pair" or M > 300
