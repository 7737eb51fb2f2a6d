"""Workspace that a context with a budget has to hold: the small sort's digit
counts take none of their own (they lie where the key arrays are written
later), so a frame of few points fits beside the megabyte of descriptors; and
the call that times its variants takes little more than the others."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_25260_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_25260_amd import lpcc
    lpcc.lib()
    return lpcc


@pytest.mark.parametrize("D,C,nd,n,budget", [(6, 16, 2, 60, 1250000), (10, 16, 3, 60, 1350000),
                                             (12, 16, 4, 60, 1350000), (14, 32, 4, 60, 1450000)])
def test_small_frames_fit_small_budgets(L, D, C, nd, n, budget):
    blob = synth.make_weights(3, C, D, nd)
    m = L.Model(blob, 0)
    xyz = synth.random_cloud(n, D, 31)
    print("D", D, "n", n, flush=True)
    ctx = L.Context(0, hbm_budget=budget)
    assert L.encode_frame(ctx, m, xyz, 8) == O.encode(blob, xyz, 8)
    assert ctx.workspace()[1] <= budget


def test_tuning_large_convolutions_takes_few_descriptors(L):
    """The call that times the variants of its launches holds little more than
    one of a fixed tiling (600000 rows per deep convolution)."""
    D, C, nd, n = 10, 16, 3, 200000
    m = L.Model(synth.make_weights(3, C, D, nd), 0)
    rng = np.random.default_rng(4)
    c = rng.choice(64 ** 3, size=n, replace=False)  # nodes of the fusion depth
    xyz = (np.stack([c // 4096, c // 64 % 64, c % 64], 1) * 16 + rng.integers(0, 16, size=(n, 3))).astype(np.int32)
    held = []
    for tiling in (2, 0):
        print("tiling", tiling, flush=True)
        ctx = L.Context(0)
        ctx.set_tiling(tiling)
        assert len(L.encode_frame(ctx, m, xyz, 8)) > 0
        held.append(ctx.workspace()[1])
    assert held[1] <= held[0] + (512 << 10), held
