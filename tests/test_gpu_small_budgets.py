"""Contexts capped near what a small frame needs: the sort's digit counts take
no memory of their own (they lie where the key arrays are written later), so a
frame of few points fits beside the megabyte of descriptors."""
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
