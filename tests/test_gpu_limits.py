"""Calls at the limits of their buffers: a call that overflows them and is run
again comes out as one that had room from the start."""
import numpy as np
import pytest

from paper_1311_5334_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emt():
    import torch
    assert torch.cuda.is_available()
    from paper_1311_5334_amd import emt as e
    e.load()
    return e


def on_line(g, i, j, r=50):
    """Grains within r of the line through grains i and j (exact)."""
    d = g[j] - g[i]
    c = np.cross(g - g[i], d)
    return int(((c * c).sum(axis=1) <= r * r * int(d @ d)).sum())


def test_seeds_that_overflow_a_large_buffer(emt):
    """The first attempt's buffers hold 2^26 seeds (256 for each of 2^18
    grains), whose mask has too many tiles for a workgroup to add up those
    before its own; none of the call's seeds are taken then, and the call is
    run again."""
    from scipy.spatial import cKDTree
    xyz = synth.make_box_view(31, 140000, (191.0, 191.0, 191.0)).xyz
    tree = cKDTree(xyz.astype(np.float64))
    n_seeds = (tree.count_neighbors(tree, np.sqrt(2500.0 ** 2 - 0.5)) - len(xyz)) // 2
    assert n_seeds > (1 << 26)
    results = []
    with emt.Tracker(device=0, flags=emt.EMT_F_CANDIDATES, min_grains=16) as tr:
        for call in range(2):
            got = tr([xyz])[0]
            assert (tr.stats()["retries"] > 0) == (call == 0)
            cand = tr.candidates(0)
            results.append((got, cand[np.lexsort((cand[:, 1], cand[:, 0]))]))
    (first, c1), (again, c2) = results
    same = np.unique(xyz, axis=0, return_counts=True)[1]
    zero = int((same * (same - 1) // 2).sum())  # pairs of coinciding grains are no seeds
    assert first["n_seeds"] == again["n_seeds"] == n_seeds - zero
    assert len(c1) > 0 and np.array_equal(c1, c2)
    assert first["tracks"].tobytes() == again["tracks"].tobytes()
    assert np.array_equal(first["grains"], again["grains"])
    g = xyz.astype(np.int64)
    listed = {(int(i), int(j)): int(n) for i, j, n in c1}
    rng = np.random.default_rng(1)
    for k in rng.choice(len(c1), min(100, len(c1)), replace=False):
        i, j, n = (int(q) for q in c1[k])
        assert on_line(g, i, j) == n
    for i in rng.choice(len(g), 50, replace=False):
        near = [j for j in tree.query_ball_point(xyz[i], 2400.0) if np.any(xyz[j] != xyz[i])]
        j = int(rng.choice(near))
        a, b = min(int(i), j), max(int(i), j)
        n = on_line(g, a, b)
        assert listed.get((a, b), 0) == (n if n >= 16 else 0)


def test_device_view_longer_than_its_allocation(emt):
    """A device view that runs past the end of its allocation is refused, as a
    copy of it is. (By 12 bytes here, in the allocation's own page, so that they
    are there whatever reads them.)"""
    import ctypes as C
    lib = emt.load()  # (the HIP runtime it is linked to finds hipMalloc)
    lib.hipMalloc.argtypes, lib.hipFree.argtypes = [C.POINTER(C.c_void_p), C.c_size_t], [C.c_void_p]
    p = C.c_void_p()
    assert lib.hipMalloc(C.byref(p), 1200) == 0

    def call(ctx, n):
        v = (emt.EmtViewIn * 1)()
        v[0].xyz = p.value
        v[0].n_grains = n
        return lib.emt_track_views(ctx, v, 1, (emt.EmtViewOut * 1)())

    lib.hipMemset.argtypes = [C.c_void_p, C.c_int, C.c_size_t]
    assert lib.hipMemset(p, 0, 1200) == 0
    with emt.Tracker(device=0, flags=emt.EMT_F_DEVICE_PTRS) as tr:
        assert call(tr.ctx, 100) == emt.EMT_OK
        assert call(tr.ctx, 101) == emt.EMT_EDEVICE
    assert lib.hipFree(p) == 0
