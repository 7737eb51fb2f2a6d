"""Child convolution under a fixed tiling at the parent counts where its parents
per block change (256 blocks of 128, 256, 512 and 1024): the frequency rows
equal those of an autotuned context, which picks its sizes by time."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("n", [255 * 128, 255 * 128 + 1, 255 * 256 + 1, 255 * 512, 255 * 512 + 1, 255 * 1024 + 1])
@pytest.mark.parametrize("C,zp", [(16, False), (64, True)])
def test_fixed_tiling_at_block_size_edges(L, n, C, zp):
    D, nd = 10, 2  # the child convolution of the deepest depth has n parents, at depth 7
    m = L.Model(synth.make_weights(33 + C, C, D, nd, zero_points=zp), 0)
    rng = np.random.default_rng(n + C)
    c = rng.choice(128 ** 3, size=n, replace=False)
    p = np.stack([c // 128 ** 2, c // 128 % 128, c % 128], 1) * 8
    xyz = (np.concatenate([p, p[::3]]) + rng.integers(0, 8, size=(n + (n + 2) // 3, 3))).astype(np.int32)
    dx = torch.from_numpy(xyz).cuda()
    print("n", n, "C", C, flush=True)
    want = torch.zeros((len(xyz), 256), dtype=torch.int32, device="cuda")
    got = torch.zeros_like(want)
    k = L.level_probs(L.Context(0), m, dx, D - 1, out=want)
    for tiling in (2, 11, 12, 14):
        ctx = L.Context(0)
        ctx.set_tiling(tiling)
        got.zero_()
        torch.cuda.synchronize()
        assert L.level_probs(ctx, m, dx, D - 1, out=got) == k
        assert torch.equal(got[:k], want[:k]), tiling
