"""The memory a server counts for a decode: enough for every base depth, alone
and mixed in one batch (the slot's context is capped at what it was granted),
and no CDF rows of the modelled depths, which a decode does not hold."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_25260_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
D, C, ND = 12, 32, 4


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_25260_amd import lpcc
    lpcc.lib()
    return lpcc


def points(xyz):
    u = np.unique(xyz, axis=0)
    return u[np.argsort(O.morton(u, D))]


def test_decode_bound_counts_what_a_decode_holds(L):
    m = L.Model(synth.make_weights(21, C, D, ND), 0)
    xyz = synth.random_cloud(60000, D, 41)
    ctx = L.Context(0)
    bs = L.encode_frame(ctx, m, xyz, 8)
    largest = int(max(np.frombuffer(bs[16:16 + 4 * D], np.uint32)))
    alone = L.Context(0)
    print("alone", flush=True)
    want = L.decode_frame(alone, m, bs)
    assert np.array_equal(want, points(xyz))
    held, _ = alone.workspace()
    srv = L.Server([m], 0, slots=1, max_batch=1)
    out = np.zeros((len(want), 3), np.int32)
    print("served", flush=True)
    srv.submit(1, 0, np.frombuffer(bs, np.uint8), out)
    srv.drain()
    done, stats = srv.poll(4), srv.stats()
    srv.close()
    assert [d["status"] for d in done] == [0] and np.array_equal(out, want)
    assert held <= stats["bytes_peak"] < held + 256 * largest


@pytest.mark.parametrize("bases", [(0, 0), (7, 7), (0, 3), (7, 1, 0)])
def test_bound_covers_every_base_depth(L, bases):
    """Cubes with many nodes at the base depths; a budget that is exactly the
    largest job's bound still decodes them all."""
    m = L.Model(synth.make_weights(22, C, D, ND), 0)
    ctx = L.Context(0)
    g = np.stack(np.meshgrid(*[np.arange(0, 1 << D, 1 << 7)] * 3, indexing="ij"), -1).reshape(-1, 3)
    streams, want = [], []
    for k, b in enumerate(bases):
        xyz = np.ascontiguousarray(g[np.random.default_rng(k).permutation(len(g))[:20000 + 1000 * k]], np.int32)
        ctx.set_base_depth(b)
        streams.append(np.frombuffer(L.encode_frame(ctx, m, xyz, 8), np.uint8))
        want.append(points(xyz))
    budget = 0
    for rnd in range(2):
        print("bases", bases, "budget", budget, flush=True)
        srv = L.Server([m], 0, slots=1, max_batch=len(bases), hbm_budget=budget)
        outs = [np.zeros((len(w), 3), np.int32) for w in want]
        for s, o in zip(streams, outs):
            srv.submit(1, 0, s, o)
        srv.drain()
        done = srv.poll(8)
        budget = srv.stats()["bytes_peak"]
        srv.close()
        assert sorted(d["status"] for d in done) == [0] * len(bases), done
        for o, w in zip(outs, want):
            assert np.array_equal(o, w)
