"""Launches that only a batch reaches (embedding rows copied from a table, the
block that scans thousands of chunk counts): the streams of a batch equal those
of its frames one by one, and decode to the points."""
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


@pytest.mark.parametrize("C,xfp,cells,cl", [(16, True, 32768, 5), (32, True, 33001, 8), (64, True, 33001, 5), (64, False, 32768, 8)])
def test_batch_equals_frames(L, C, xfp, cells, cl):
    D, nd, nf = 8, 1, 8  # the embedded codes are those of depth 6: `cells` nodes per frame
    m = L.Model(synth.make_weights(70 + C, C, D, nd, xfp=xfp), 0)
    rng = np.random.default_rng(C)
    frames = []
    for _ in range(nf):
        c = rng.choice(64 ** 3, size=cells, replace=False)
        p = np.stack([c // 4096, c // 64 % 64, c % 64], 1) * 4
        frames.append((p + rng.integers(0, 4, size=p.shape)).astype(np.int32))
    print("C", C, "xfp", xfp, "cells", cells, flush=True)
    dev = [torch.from_numpy(f).cuda() for f in frames]
    ctx = L.Context(0)
    outs = [torch.zeros(len(f) * 8 + 65536, dtype=torch.uint8, device="cuda") for f in frames]
    lens, st = L.encode_batch(ctx, m, dev, cl, outs=outs)
    assert st == [0] * nf
    one = L.Context(0)
    for x, o, n in zip(dev, outs, lens):
        assert L.encode_frame(one, m, x, cl) == bytes(o[:n].cpu().numpy())
    decs = [torch.zeros((len(f), 3), dtype=torch.int32, device="cuda") for f in frames]
    nout, st = L.decode_batch(ctx, m, outs, lengths=lens, outs=decs)
    assert st == [0] * nf
    for f, x, n in zip(frames, decs, nout):
        assert np.array_equal(x[:n].cpu().numpy(), f[np.argsort(O.morton(f, D))])
