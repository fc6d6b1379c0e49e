"""Rank counts from bidiagonals at the edges of their variants (tiles of 32, 64, 256 and 512 rows; ragged last tiles,
tall and wide ones), against NumPy's singular values in FP64, and what they leave to the rotations: a tile that is not
finite, tiles above 512 rows."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _symmetric(nr, seed):
    """Decaying singular values in every tile (a smooth kernel), some noise, exactly symmetric complex64."""
    rng = np.random.default_rng(seed)
    x = np.sort(rng.random(nr))
    d = np.abs(x[:, None] - x[None, :])
    a = np.exp(-1j * 40 * d) / (d + 0.02) + 0.5 * (rng.standard_normal((nr, nr)) + 1j * rng.standard_normal((nr, nr)))
    return ((a + a.T) / 2).astype(np.complex64)


def _reference(X, d, eps):
    X = X.astype(np.complex128)
    cut = list(range(0, X.shape[0], d)) + [X.shape[0]]
    sv = {(i, j): np.linalg.svd(X[cut[i]:cut[i + 1], cut[j]:cut[j + 1]], compute_uv=False)
          for i in range(len(cut) - 1) for j in range(i + 1)}
    v0 = max(s[0] for s in sv.values())
    t = eps * v0
    assert min(np.min(np.abs(s - t)) for s in sv.values()) > 1e-10 * v0   # no singular value on the threshold
    k = {ij: int(np.sum(s >= t)) for ij, s in sv.items()}
    n = len(cut) - 1
    return [k[i, j] for i in range(n) for j in range(i)], [k[i, i] for i in range(n)], v0


@pytest.mark.parametrize("nr,d", [(1, 1), (5, 2), (33, 16), (64, 32), (97, 33), (150, 64), (140, 65), (300, 100), (520, 256),
                                  (530, 257), (1024, 512), (600, 560)])
@pytest.mark.parametrize("eps", [0.05, 1e-3])
def test_rank_counts(nr, d, eps):
    import paper_2412_14973_amd as tl
    X = _symmetric(nr, 7 * nr + d)
    ko, kd, v0 = tl.tile_ranks(torch.from_numpy(X).cuda(), d, eps)
    ro, rd, v0r = _reference(X, d, eps)
    assert ko.tolist() == ro and kd.tolist() == rd
    # backward stable reduction: a few n u; the rotations (tiles above 512 rows) stop at 1e-13 per pair, and the
    # rank tests hold them to 1e-12
    assert abs(v0 - v0r) <= (1e-13 if d <= 512 else 1e-12) * v0r


def test_rank_counts_zero_and_nonfinite():
    import paper_2412_14973_amd as tl
    ko, kd, v0 = tl.tile_ranks(torch.zeros(96, 96, dtype=torch.complex64, device="cuda"), 32, 0.01)
    assert v0 == 0.0 and set(ko.tolist()) == set(kd.tolist()) == {32}   # sigma >= 0 holds for all
    # one bad entry: its tile's other columns and all other tiles keep their counts
    X = _symmetric(96, 3)
    ref = _reference(X, 32, 0.05)
    Y = X.copy()
    Y[40, 2] = np.nan
    ko, kd, v0 = tl.tile_ranks(torch.from_numpy(Y).cuda(), 32, 0.05)
    assert kd.tolist() == ref[1] and ko.tolist()[1:] == ref[0][1:] and abs(v0 - ref[2]) <= 1e-12 * ref[2]


@pytest.mark.parametrize("nr,d", [(64, 64), (128, 128), (229, 129), (200, 200), (356, 256), (256, 192)])
@pytest.mark.parametrize("scale", [1.0, 1e-18, 1e18])
def test_rank_counts_in_registers(nr, d, scale):
    """Tiles held in registers whole (to 128 rows) or from the last 128 rows on; squares of the entries' noise near the
    ends of the range of FP64's exponents when they are scaled are not reached."""
    import paper_2412_14973_amd as tl
    X = (_symmetric(nr, 11 * nr + d) * scale).astype(np.complex64)
    ko, kd, v0 = tl.tile_ranks(torch.from_numpy(X).cuda(), d, 0.02)
    ro, rd, v0r = _reference(X, d, 0.02)
    assert ko.tolist() == ro and kd.tolist() == rd and abs(v0 - v0r) <= 1e-13 * v0r


@pytest.mark.parametrize("d", [48, 100, 200])
def test_rank_counts_of_exact_low_rank(d):
    """Rank one, and a tile of one entry: the reflections meet columns that are zero."""
    import paper_2412_14973_amd as tl
    a = np.exp(1j * np.arange(200)).astype(np.complex64)
    X = np.outer(a, a).astype(np.complex64)
    ko, kd, _ = tl.tile_ranks(torch.from_numpy(X).cuda(), d, 0.01)
    assert set(ko.tolist()) <= {1} and set(kd.tolist()) == {1}
    X = np.zeros((200, 200), dtype=np.complex64)
    X[7, 7] = 3j
    ko, kd, v0 = tl.tile_ranks(torch.from_numpy(X).cuda(), d, 0.01)
    assert not np.any(ko) and kd.tolist() == [1] + [0] * (len(kd) - 1) and v0 == 3.0


@pytest.mark.parametrize("nr,cand", [(300, [64, 128, 256]), (300, [100, 40]), (410, [200, 64, 256, 200]), (97, [33, 97]),
                                     (300, [32, 64]), (600, [64, 300])])
@pytest.mark.parametrize("bad", [False, True])
def test_layouts_together_and_one_by_one(nr, cand, bad):
    """All candidates in one pass (33 to 256 rows, room for all), or one after the other in the documented workspace."""
    import ctypes
    import paper_2412_14973_amd as tl
    X = _symmetric(nr, 5 * nr)
    if bad:
        X[3, 1] = X[1, 3] = np.inf
    X = torch.from_numpy(X).cuda()
    d, sizes, ro, rd, ent = tl.choose_layout(X, cand, 0.02)
    lib = tl._lib.load()
    c = np.array(cand, dtype=np.int32)
    ws = tl._ranks_workspace(nr, int(c.max()), X.device)
    ro1, rd1, ent1 = np.zeros(nr * nr, dtype=np.int32), np.zeros(nr, dtype=np.int32), np.zeros(len(cand), dtype=np.int64)
    d1 = ctypes.c_int32()
    tl._lib.check(lib.tlrmdd_choose_layout(tl._ptr(X), nr, c.ctypes.data, len(cand), 0.02, ctypes.byref(d1),
                                           ent1.ctypes.data, ro1.ctypes.data, ro1.size, rd1.ctypes.data, rd1.size,
                                           tl._ptr(ws), ws.numel(), tl._stream()), "choose_layout")
    assert d == d1.value and ent.tolist() == ent1.tolist()
    assert ro.tolist() == ro1[:ro.size].tolist() and rd.tolist() == rd1[:rd.size].tolist()
    ko, kd, _ = tl.tile_ranks(X, d, 0.02)
    assert ro.tolist() == np.maximum(1, ko).tolist()
    assert rd.tolist() == [-1 if k >= (s + 1) // 2 else max(1, k) for k, s in zip(kd.tolist(), sizes.tolist())]


@pytest.mark.parametrize("nr,d", [(1, 1), (33, 16), (64, 32), (97, 33), (64, 64), (300, 100), (356, 256), (530, 257), (600, 560)])
def test_rank_counts_at_the_largest_singular_value(nr, d):
    """eps = 1: v0 counts in its own tile and in no other; where all singular values are alike, all of them do."""
    import paper_2412_14973_amd as tl
    X = _symmetric(nr, 13 * nr + d)
    ko, kd, _ = tl.tile_ranks(torch.from_numpy(X).cuda(), d, 1.0)
    cut = list(range(0, nr, d)) + [nr]
    top = {(i, j): np.linalg.norm(X[cut[i]:cut[i + 1], cut[j]:cut[j + 1]].astype(np.complex128), 2)
           for i in range(len(cut) - 1) for j in range(i + 1)}
    best = max(top.values())
    assert sum(s > (1 - 1e-9) * best for s in top.values()) == 1
    n = len(cut) - 1
    want = {ij: int(s == best) for ij, s in top.items()}
    assert ko.tolist() == [want[i, j] for i in range(n) for j in range(i)] and kd.tolist() == [want[i, i] for i in range(n)]
    ko, kd, v0 = tl.tile_ranks(torch.eye(nr, dtype=torch.complex64, device="cuda") * 2.5, d, 1.0)
    assert not np.any(ko[:n * (n - 1) // 2]) and kd.tolist() == np.diff(cut).tolist() and abs(v0 - 2.5) <= 1e-13


@pytest.mark.parametrize("nr,d", [(64, 32), (128, 64), (200, 100), (400, 200), (600, 300), (1200, 600)])
@pytest.mark.parametrize("scale", [1.0, 1e-30, 1e30])
def test_rank_counts_at_extreme_thresholds(nr, d, scale):
    """Thresholds whose squares leave the range of FP64: none of the values is above, and all but exact zeros are."""
    import paper_2412_14973_amd as tl
    X = torch.eye(nr, dtype=torch.complex64, device="cuda") * scale
    for eps in (1e300, 1e200, 1e160, 1e20, 5.0, 1.5):
        ko, kd, _ = tl.tile_ranks(X, d, eps)
        assert ko.tolist() == [0] and kd.tolist() == [0, 0], eps
    for eps in (1e-250, 1e-190, 1e-155, 1e-110, 1e-60):
        ko, kd, _ = tl.tile_ranks(X, d, eps)
        assert ko.tolist() == [0] and kd.tolist() == [d, d], eps
    ko, kd, _ = tl.tile_ranks(X, d, 0.0)
    assert ko.tolist() == [d] and kd.tolist() == [d, d]
