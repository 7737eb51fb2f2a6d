"""Batches whose headers, payloads and coordinates are moved by one launch per
32 frames: one to 65 frames, streams and outputs at every byte alignment, an
output without room.  Streams and decodes equal the oracle's and nothing
around an output changes."""
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


@pytest.mark.parametrize("nf,base", [(1, 0), (2, 0), (32, 0), (33, 2), (65, 0)])
def test_batches_at_every_alignment(L, nf, base):
    C, D, nd = 16, 6, 2
    blob = synth.make_weights(3, C, D, nd)
    m = L.Model(blob, 0)
    ctx = L.Context(0)
    ctx.set_base_depth(base)
    rng = np.random.default_rng(nf)
    frames = [rng.integers(0, 2 ** D, size=(int(rng.integers(1, 200)), 3)).astype(np.int32) for _ in range(nf)]
    want = [O.encode(blob, f, 5, base=base) for f in frames]
    print("frames", nf, "base", base, flush=True)
    cap = max(len(w) for w in want) + 16
    pool = torch.full(((cap + 64) * nf + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    at = [(cap + 64) * f + f % 17 for f in range(nf)]
    outs = [pool[a:a + cap] for a in at]
    lens, st = L.encode_batch(ctx, m, [torch.from_numpy(f).cuda() for f in frames], 5, outs=outs)
    assert st == [0] * nf
    host = pool.cpu().numpy()
    for a, n, w in zip(at, lens, want):
        assert bytes(host[a:a + n]) == w
    for a, b in zip(at, at[1:]):
        assert (host[a + cap:b] == 0xA5).all()
    decs = [torch.full((len(f) + 1, 3), -7, dtype=torch.int32, device="cuda") for f in frames]
    nout, st = L.decode_batch(ctx, m, outs, lengths=lens, outs=decs)
    assert st == [0] * nf
    for f, x, n in zip(frames, decs, nout):
        u = np.unique(f, axis=0)
        x = x.cpu().numpy()
        assert np.array_equal(x[:n], u[np.argsort(O.morton(u, D))])
        assert (x[len(u):] == -7).all()


def test_output_without_room(L):
    blob = synth.make_weights(3, 16, 6, 2)
    m = L.Model(blob, 0)
    ctx = L.Context(0)
    xyz = np.random.default_rng(1).integers(0, 64, size=(50, 3)).astype(np.int32)
    dx = torch.from_numpy(xyz).cuda()
    out = torch.full((8,), 0xA5, dtype=torch.uint8, device="cuda")
    lens, st = L.encode_batch(ctx, m, [dx, dx], 5, outs=[out[:3], out[4:7]])
    assert all(s != 0 for s in st) and list(lens) == [len(O.encode(blob, xyz, 5))] * 2
    assert (out.cpu().numpy()[[3, 7]] == 0xA5).all()
