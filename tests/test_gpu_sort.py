"""The octree's radix sort at the sizes where its tiles and launches change:
64 tiles of 512 and 2048 keys, one key more, and larger sorts; several frames
in one sort, and key widths whose last digit is short.  A decode of the encoded
stream lists the sorted unique voxels, so it is compared with numpy's."""
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


def morton_sorted(xyz, D):
    u = np.unique(xyz, axis=0).astype(np.uint64)
    m = np.zeros(len(u), np.uint64)
    for b in range(D):
        for a in range(3):
            m |= ((u[:, a] >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b + 2 - a)
    return u[np.argsort(m, kind="stable")].astype(np.int32)


@pytest.mark.parametrize("n", [1, 2, 63, 65, 511, 512, 513, 32767, 32768, 32769, 131072, 131073, 262145])
@pytest.mark.parametrize("D,clustered", [(8, True), (12, False)])
def test_sorted_unique_voxels(L, n, D, clustered):
    m = L.Model(synth.make_weights(11, 16, D, 3), 0)
    ctx = L.Context(0)
    xyz = synth.random_cloud(n, D, n + D, clustered=clustered)
    print("n", n, "D", D, flush=True)
    want = morton_sorted(xyz, D)
    got = L.decode_frame(ctx, m, L.encode_frame(ctx, m, torch.from_numpy(xyz).cuda(), 8))
    assert np.array_equal(got, want)


@pytest.mark.parametrize("sizes", [(5, 0, 1, 700), (20000, 12768), (12768, 20001), (100000, 31072, 1),
                                   (1, 262143), (131073, 131072)])
def test_sorted_per_frame(L, sizes):
    D = 11
    m = L.Model(synth.make_weights(12, 16, D, 3), 0)
    ctx = L.Context(0)
    frames = [synth.random_cloud(n, D, 7 * n + k) for k, n in enumerate(sizes)]
    print("sizes", sizes, flush=True)
    bs, st = L.encode_batch(ctx, m, [torch.from_numpy(f).cuda() for f in frames], 8)
    assert st == [0] * len(sizes)
    got, st = L.decode_batch(ctx, m, bs)
    assert st == [0] * len(sizes)
    for f, g in zip(frames, got):
        assert np.array_equal(g, morton_sorted(f, D)) if len(f) else len(g) == 0
