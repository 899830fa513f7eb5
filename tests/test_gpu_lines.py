"""The line grids of the counting kernel against the oracle, at the sizes and
shapes where their rules change: the number of grains from which they are
used, cells too large for packed list words, lists that overflow their share
(a coarser grid then), every face as the long one, a large radius, and the
budgets that leave room for fewer line classes. Everything is compared
exactly (candidates element by element; the fit by tests/parity.py)."""
import numpy as np
import pytest

from oracle import oracle
from paper_1311_5334_amd import synth
from tests.parity import assert_candidates_equal, assert_view_parity

pytestmark = pytest.mark.gpu

FEW = 8192  # grains of a call up to which the binned cells are walked


@pytest.fixture(scope="module")
def emt():
    import torch
    assert torch.cuda.is_available()
    from paper_1311_5334_amd import emt as e
    e.load()
    return e


def check(emt, views, oracle_cfg=None, **cfg):
    oracle_cfg = oracle_cfg or {}
    with emt.Tracker(device=0, flags=emt.EMT_F_CANDIDATES, **cfg) as tr:
        got = tr(views)
        cands = [tr.candidates(v) for v in range(len(views))]
    assert sum(len(c) for c in cands) > 0
    for xyz, g, c in zip(views, got, cands):
        ref = oracle.track_view(xyz, **oracle_cfg)
        assert_candidates_equal(c, ref)
        assert_view_parity(xyz, g, ref)


def moderate(seed, side=205.0, density=4.4):
    return synth.make_density_view(seed, density, side).xyz


def with_lines(seed, n, box, n_lines, per_line):
    """Uniform grains in a box (units) and straight rows of grains across it."""
    rng = np.random.default_rng(seed)
    box = np.asarray(box, np.float64)
    parts = [rng.uniform(0, 1, (n, 3)) * box]
    for _ in range(n_lines):
        p, d = rng.uniform(0.3, 0.7, 3) * box, rng.normal(size=3)
        d /= np.linalg.norm(d)
        t = np.arange(per_line) * 700.0
        row = p + t[:, None] * d
        parts.append(row[np.all((row >= 0) & (row <= box), axis=1)])
    return np.rint(np.concatenate(parts)).astype(np.int32)


@pytest.mark.parametrize("n", [FEW - 1, FEW, FEW + 1])
def test_number_of_grains_that_switches(emt, n):
    xyz = moderate(11)
    assert len(xyz) > n
    check(emt, [xyz[:n]])


@pytest.mark.parametrize("order", [(0, 1, 2), (2, 0, 1), (1, 2, 0)])
def test_every_axis_as_the_short_one(emt, order):
    xyz = np.ascontiguousarray(moderate(12, side=230.0)[:, order])
    check(emt, [xyz, -xyz])


def test_cells_too_large_to_pack(emt):
    # the largest span (2^18 units) in two axes, few grains per volume
    side = float(1 << 18)
    xyz = with_lines(13, 9000, (side, side, 5000.0), 60, 40)
    xyz[0], xyz[1] = (0, 0, 0), (1 << 18, 1 << 18, 5000)
    check(emt, [xyz])


def test_one_plane(emt):
    check(emt, [with_lines(14, 9000, (120000.0, 120000.0, 0.0), 40, 30)])


def test_lists_that_overflow_their_share(emt):
    # a plane lattice of pitch 300 = 3 cells, its grains at a slab's edge and
    # placed so that their rectangles cover 4 x 4 cells of the steepest
    # classes: 16 words a grain, 12 are a class's share
    k = np.arange(95) * 300 + 4
    x, y = np.meshgrid(k, k)
    xyz = np.stack([x.ravel(), y.ravel(), np.zeros(x.size)], axis=1).astype(np.int32)
    xyz = np.concatenate([np.zeros((1, 3), np.int32), xyz])
    check(emt, [xyz], {"R": 700, "n_min": 40}, seed_dist=700, min_grains=40)


def test_views_of_all_kinds_in_one_call(emt):
    check(emt, [moderate(15)[:40], moderate(16), np.zeros((0, 3), np.int32),
                synth.make_density_view(17, 14.0, 100.0).xyz,
                with_lines(18, 2000, (150000.0, 90000.0, 4000.0), 20, 20)])


def test_large_radius(emt):
    xyz = synth.make_density_view(19, 1.1, 420.0).xyz
    assert len(xyz) > FEW
    check(emt, [xyz], {"r": 300, "n_min": 14}, tol_radius=300, min_grains=14)


def test_budgets_with_room_for_fewer_classes(emt):
    xyz = moderate(20)
    assert FEW < len(xyz) <= 2 * FEW
    # from room for every class (about 173 MB) down to the least that is
    # accepted, where three classes are left
    mb = 200
    accepted = []
    while mb > 100:
        try:
            with emt.Tracker(device=0, hbm_budget=mb << 20) as tr:
                tr([xyz])
        except emt.EmtError as e:
            assert e.rc == emt.EMT_ENOMEM
            break
        accepted.append(mb)
        mb -= 1
    assert len(accepted) > 40
    for b in (accepted[0], 150, accepted[-1]):
        check(emt, [xyz], hbm_budget=b << 20)


@pytest.mark.parametrize("copies", [1, 5, 40, 720])
def test_scans_of_every_size(emt, copies):
    """From arrays one workgroup scans to ones whose tile sums take a scan of
    their own (720 views: 2^21 grains in the buffers, 2^23 cells): every copy
    of a view comes out as the oracle has it."""
    xyz = moderate(11)[:1500]
    ref = oracle.track_view(xyz)
    with emt.Tracker(device=0, flags=emt.EMT_F_CANDIDATES) as tr:
        got = tr([xyz] * copies)
        for v in range(copies):
            assert_candidates_equal(tr.candidates(v), ref)
    for g in got:
        assert g["tracks"].tobytes() == got[0]["tracks"].tobytes()
    assert_view_parity(xyz, got[0], ref)


def test_dense_call_after_sparse_ones(emt):
    """The sparse calls leave few grid-wide merge rounds for the next call of
    their size; the dense one's other rounds are the tail's."""
    sparse, dense = moderate(11, density=1.0)[:4000], moderate(12, density=20.0)[:4000]
    with emt.Tracker(device=0, flags=emt.EMT_F_CANDIDATES) as tr:
        for xyz in (dense, sparse, sparse, dense):
            got = tr([xyz])[0]
            ref = oracle.track_view(xyz)
            assert_candidates_equal(tr.candidates(0), ref)
            assert_view_parity(xyz, got, ref)


@pytest.mark.parametrize("n,views", [(700, 14), (1500, 8), (9000, 1)])
def test_path_learned_from_the_call_before(emt, n, views):
    """Small views in a large call, and calls that are over line grids the
    first time and over the binned cells once their seeds are known (and the
    other way round, after a dense call of the same size)."""
    sparse = [moderate(20 + k, side=420.0, density=1.2)[:n] for k in range(views)]
    dense = [moderate(40 + k, side=150.0, density=9.0)[:n] for k in range(views)]
    with emt.Tracker(device=0, flags=emt.EMT_F_CANDIDATES) as tr:
        for batch in (sparse, sparse, dense, dense, sparse):
            got = tr(batch)
            for v in (0, views - 1):
                ref = oracle.track_view(batch[v])
                assert_candidates_equal(tr.candidates(v), ref)
                assert_view_parity(batch[v], got[v], ref)


@pytest.mark.parametrize("n,side", [(3000, 45.0), (9000, 70.0)])
def test_more_seeds_than_an_anchor_stages(emt, n, side):
    """Anchors with more seeds than are put in order before they are written."""
    xyz = synth.make_box_view(5, n, (side, side, side)).xyz
    check(emt, [xyz], dict(n_min=5), min_grains=5)


def steep_lattice():
    """The plane lattice of test_lists_that_overflow_their_share."""
    k = np.arange(95) * 300 + 4
    x, y = np.meshgrid(k, k)
    xyz = np.stack([x.ravel(), y.ravel(), np.zeros(x.size)], axis=1).astype(np.int32)
    return np.concatenate([np.zeros((1, 3), np.int32), xyz])


@pytest.mark.parametrize("view", ["lattice", "plane"])
def test_lists_that_overflow_at_every_budget(emt, view):
    """Every number of line classes that a budget leaves, with lists that
    overflow their share: the least budget that is accepted, and a fine and a
    coarse row of larger ones."""
    if view == "lattice":
        xyz, cfg = steep_lattice(), dict(seed_dist=500, min_grains=60)
        ref = oracle.track_view(xyz, R=500, n_min=60)
        d = np.diff(xyz[np.asarray(ref.cand)[:, :2].astype(int)], axis=1)[:, 0]
        assert (d[:, 0] == d[:, 1]).sum() > 1000  # lines of the steepest slope
    else:
        xyz, cfg = with_lines(14, 9000, (120000.0, 120000.0, 0.0), 40, 30), {}
        ref = oracle.track_view(xyz)
    assert len(ref.cand) > 0

    def run(kb):
        try:
            with emt.Tracker(device=0, flags=emt.EMT_F_CANDIDATES, hbm_budget=kb << 10, **cfg) as tr:
                got = tr([xyz])[0]
                assert_candidates_equal(tr.candidates(0), ref)
                assert_view_parity(xyz, got, ref)
                assert tr.stats()["retries"] == 0
        except emt.EmtError as e:
            assert e.rc == emt.EMT_ENOMEM
            return False
        return True

    refused, accepted = 1 << 10, 400 << 10
    assert run(accepted) and not run(refused)
    while accepted - refused > 32:
        mid = (accepted + refused) // 2
        if run(mid):
            accepted = mid
        else:
            refused = mid
    for more in [64 * k for k in range(24)] + [4 << 10, 12 << 10, 24 << 10, 48 << 10]:
        assert run(accepted + more)


@pytest.mark.parametrize("line", ["200,800,1", "1,1,1", "10,262144,4", "262144,1,2"])
def test_line_grids_of_any_shape(emt, monkeypatch, line):
    monkeypatch.setenv("EMT_LINE", line)
    check(emt, [steep_lattice()], {"R": 700, "n_min": 40}, seed_dist=700, min_grains=40)
    check(emt, [moderate(21), moderate(15)[:2], moderate(15)[:1]])
