"""Kernel variants at the sizes where they can go wrong (edges of tiles,
remainders, the smallest and largest of their ranges), against the oracle."""
import math
import sys

import numpy as np
import pytest

from oracle import pyoracle as O
from paper_2503_13092_amd import synth
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

from paper_2503_13092_amd import ds  # noqa: E402

W = synth.mlp_weights()
G0 = synth.default_geometry()


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def track_states(counts, seed, order):
    """Events of (positive, negative) tracks, their charges interleaved at
    random, all positive first or all negative first; half of the tracks of an
    event come from a few common points, so that close pairs exist."""
    rng = np.random.default_rng(seed)
    cols = {k: [] for k in ("x", "y", "tx", "ty", "q")}
    off = [0]
    for n_pos, n_neg in counts:
        n = n_pos + n_neg
        q = np.concatenate([np.ones(n_pos), -np.ones(n_neg)])
        if order == "random":
            rng.shuffle(q)
        elif order == "negative first":
            q = -q if n_pos == n_neg else q[::-1]
        tx, ty = rng.uniform(-0.25, 0.25, n), rng.uniform(-0.2, 0.2, n)
        x, y = rng.uniform(-800, 800, n), rng.uniform(-700, 700, n)
        zd = rng.choice(rng.uniform(0.0, 2200.0, 4), n)
        common = rng.uniform(0, 1, n) < 0.5
        h = G0["z_ref"] - zd
        x = np.where(common, 0.1 * zd + tx * h + rng.normal(0, 0.3, n), x)
        y = np.where(common, -0.05 * zd + ty * h + rng.normal(0, 0.3, n), y)
        for k, v in zip(cols, (x, y, tx, ty, q / np.exp(rng.uniform(math.log(2), math.log(100), n)))):
            cols[k].append(v)
        off.append(off[-1] + n)
    c = {k: np.concatenate(v).astype(np.float32) for k, v in cols.items()}
    return np.asarray(off, np.int32), c


# 64-row blocks and 32-partner segments of the pair masks and their
# neighbours, one charge missing, one against many, and an event whose masks
# take several panels
COUNTS = [(1, 1), (2, 0), (0, 3), (1, 40), (40, 1), (31, 33), (32, 32), (33, 31), (64, 1), (64, 65), (63, 97),
          (130, 150), (400, 380)]


@pytest.mark.parametrize("block", [64, 256])
@pytest.mark.parametrize("order", ["random", "positive first", "negative first"])
@pytest.mark.parametrize("fp", [0.0, 1.0, -1.0])
def test_vertex_pair_masks_match_oracle(fp, order, block):
    """Every opposite-charge pair that the oracle keeps, in (i, j) order and
    with its values, for straight and curved trajectories (tolerances of
    tests/parity.py: float32 storage of float64 results)."""
    off, c = track_states(COUNTS, seed=3, order=order)
    n, E, cap = len(c["x"]), len(off) - 1, 20000
    b = synth.EventBatch(E, off, c["x"], c["y"], c["tx"], c["ty"], c["q"], np.zeros(4 * E + 1, np.int32),
                         np.zeros(0, np.float32))
    g = dict(G0, fringe_polarity=fp)
    ctx = ds.Context(0, g, W)
    try:
        ds.ds_set_launch(ctx.handle, 1, block, 4, 0)
        ev, tr, vt = ds.DeviceEvents(b), ds.DeviceTracks(n), ds.DeviceVertices(E, cap)
        for k, v in (("x", "x"), ("y", "y"), ("tx", "tx"), ("ty", "ty"), ("qop", "q")):
            getattr(tr, k).copy_(torch.from_numpy(c[v]))
        tr.nhits.fill_(4)
        say(f"[edges] vertex masks: fp {fp}, {order}, block {block}, {n} tracks")
        ds.ds_vertex(ctx.handle, ev, tr, math.inf, vt, ds.DS_MODE_PERSISTENT)
        torch.cuda.synchronize()
        gv = vt.to_numpy()
    finally:
        torch.cuda.synchronize()
        ctx.close()
    st = dict(x=c["x"], y=c["y"], tx=c["tx"], ty=c["ty"], qop=c["q"], nhits=np.full(n, 4, np.int32))
    rv = O.vertex(off, c["q"], st, np.zeros(n), g, math.inf, cap)
    assert rv["count"].sum() > 1000 and gv["overflow"] == rv["overflow"] == 0
    parity.compare_vertices(gv, rv, g["doca_max"])
    for e in range(E):
        k = slice(e * cap, e * cap + int(gv["count"][e]))
        key = gv["i"][k].astype(np.int64) * n + gv["j"][k]
        assert np.all(np.diff(key) > 0), e


@pytest.mark.parametrize("order", [ds.DS_ORDER_INPUT, ds.DS_ORDER_LARGEST_FIRST])
@pytest.mark.parametrize("extra", ["one", -1, 0, 1, 300])
def test_events_taken_once_around_the_grid_size(extra, order):
    """Batches of one event and of one fewer, as many, one more and 300 more
    events than the launch has workgroups: repeated launches, fused and as
    two, are bitwise the per-event launches (each event taken once, the work
    counter back at zero)."""
    grid = torch.cuda.get_device_properties(0).multi_processor_count
    n = 1 if extra == "one" else grid + extra
    cfg = dict(name="small", n_events=n, seed=5, seeds_per_event=12, llp_per_event=4, hits_per_layer=30, zmax=2200.0)
    b = synth.generate(cfg)
    ctx = ds.Context(0, G0, W)
    outs = []
    try:
        ds.ds_set_launch(ctx.handle, 0, 256, 1, 0)
        ds.ds_set_launch(ctx.handle, 1, 64, 1, 0)
        ds.ds_set_event_order(ctx.handle, order)
        ev = ds.DeviceEvents(b)
        for mode, fused in ((ds.DS_MODE_PER_EVENT, 1), (ds.DS_MODE_PERSISTENT, 1), (ds.DS_MODE_PERSISTENT, 0),
                            (ds.DS_MODE_GRAPH, 1), (ds.DS_MODE_GRAPH, 0)):
            ds.ds_set_step_fusion(ctx.handle, fused)
            tr, vt = ds.DeviceTracks(b.n_seeds), ds.DeviceVertices(n, 64)
            say(f"[edges] {n} events over {grid} workgroups, order {order}, mode {mode}, fused {fused}")
            for _ in range(1 if mode == ds.DS_MODE_PER_EVENT else 3):
                for t in (tr.x, tr.nhits, vt.count, vt.x):
                    t.fill_(-7)
                ds.ds_process(ctx.handle, ev, tr, vt, mode, score_max=math.inf)
            torch.cuda.synchronize()
            outs.append((tr.to_numpy(), vt.to_numpy()))
    finally:
        torch.cuda.synchronize()
        ctx.close()
    for t, v in outs[1:]:
        for k in ("x", "y", "tx", "ty", "qop", "chi2", "score", "hits", "nhits", "cand"):
            assert np.array_equal(t[k], outs[0][0][k]), k
        for k in ("count", "i", "j", "x", "y", "z", "doca"):
            assert np.array_equal(v[k], outs[0][1][k]), k


# hits per layer and seeds per event: windows of no, few, more than max_l3 and far more hits (ranked, and cut
# down around the prediction, above 2 max_l3), one lane's worth of seeds to several chunks of them
OCCUPANCIES = [(8, 1), (300, 63), (600, 65), (2400, 40), (4700, 300)]


@pytest.mark.parametrize("hits,seeds", OCCUPANCIES)
@pytest.mark.parametrize("n_closest,max_l3", [((1, 2, 2), 10), ((2, 2, 2), 16), ((1, 1, 0), 3), ((0, 2, 1), 1)])
@pytest.mark.parametrize("algorithm,loose", [(0, False), (0, True), (1, False)])
def test_window_options_match_oracle(algorithm, loose, n_closest, max_l3, hits, seeds):
    """Hits, candidates and track parameters against the oracle (tolerances of
    tests/parity.py) for every way the window search takes: ranked and
    unranked first windows, each number of closest hits, one and two Y sectors."""
    g = dict(synth.default_geometry(loose=loose), n_closest=n_closest, max_l3=max_l3, algorithm=algorithm)
    cfg = dict(name="edges", n_events=4, seed=11 + hits, seeds_per_event=seeds, llp_per_event=min(seeds // 2, 20),
               hits_per_layer=hits, zmax=2200.0)
    b = synth.generate(cfg, geometry=g)
    ref = O.find_tracks(b, g, n_threads=8)
    ctx = ds.Context(0, g, W)
    try:
        for block, bins in ((256, 1024), (64, 64)):
            ds.ds_set_launch(ctx.handle, 0, block, 2, bins)
            ev, tr = ds.DeviceEvents(b), ds.DeviceTracks(b.n_seeds)
            say(f"[edges] algorithm {algorithm}, loose {loose}, {n_closest}, {max_l3}: {hits} hits, {seeds} seeds, "
                f"block {block}")
            ds.ds_find_tracks(ctx.handle, ev, tr, ds.DS_MODE_PERSISTENT, 1)
            torch.cuda.synchronize()
            t = tr.to_numpy()
            # (three hits or triplets per lane are listed for one seed: wide windows and Dv1 in full layers have
            # more than 192, which is flagged and not compared)
            if block == 64 and (loose or algorithm == 1) and hits > 600:
                assert t["flags"] in (0, ds.DS_F_CAPACITY)
                continue
            assert t["flags"] == 0
            parity.compare_tracks(t, ref, min_identical=0.0)
    finally:
        torch.cuda.synchronize()
        ctx.close()


@pytest.mark.parametrize("algorithm", [0, 1])
@pytest.mark.parametrize("events,seeds,hits", [(1, 149, 583), (3, 600, 1100), (40, 30, 3000), (300, 20, 200),
                                               (520, 90, 1500), (1, 1100, 400)])
def test_chosen_launch_shapes_bitwise_equal(events, seeds, hits, algorithm):
    """Launches whose shape the library chooses (512 and 1 024 lanes where few
    events or few resident workgroups leave the chip idle, several wavefronts
    staging a layer, more seeds than a chunk) against 128 lanes and 512 bins
    set by the caller: tracks, candidates and vertices bitwise the same."""
    cfg = dict(name="shapes", n_events=events, seed=events + hits, seeds_per_event=seeds,
               llp_per_event=seeds // 4, hits_per_layer=hits, zmax=2200.0)
    b = synth.generate(cfg)
    outs = []
    for shape in (None, (128, 4, 512)):
        ctx = ds.Context(0, dict(G0, algorithm=algorithm), W)
        try:
            if shape:
                ds.ds_set_launch(ctx.handle, 0, *shape)
            ev, tr, vt = ds.DeviceEvents(b), ds.DeviceTracks(b.n_seeds), ds.DeviceVertices(events, 256)
            say(f"[edges] {events} events, {seeds} seeds, {hits} hits, algorithm {algorithm}, shape {shape}")
            for _ in range(2):
                vt.overflow.zero_()
                ds.ds_process(ctx.handle, ev, tr, vt, ds.DS_MODE_PERSISTENT, score_max=math.inf)
            torch.cuda.synchronize()
            outs.append((tr.to_numpy(), vt.to_numpy()))
        finally:
            torch.cuda.synchronize()
            ctx.close()
    (t0, v0), (t1, v1) = outs
    assert t0["flags"] == t1["flags"] == 0
    for k in ("x", "y", "tx", "ty", "qop", "chi2", "score", "hits", "nhits", "cand"):
        assert np.array_equal(t0[k], t1[k]), k
    for k in ("count", "i", "j", "x", "y", "z", "doca", "overflow"):
        assert np.array_equal(v0[k], v1[k]), k


@pytest.mark.parametrize("loose", [False, True])
@pytest.mark.parametrize("qop_scale,seed_shift", [(1.0, 0.0), (1.4, 0.0), (40.0, 0.0), (1.0, 3e4)])
def test_dv1_map_serves_every_seed(qop_scale, seed_shift, loose):
    """Dv1 where its bit map of UTaX ends: |q/p| up to, around and far beyond
    the windows that are marked in it, wide windows that mark many bins, seeds
    too far out for the float32 look-up, hits beyond the binned range."""
    g = dict(synth.default_geometry(loose=loose), algorithm=1)
    b = synth.generate(dict(name="map", n_events=12, seed=21, seeds_per_event=90, llp_per_event=20,
                            hits_per_layer=250, zmax=2200.0), geometry=g)
    rng = np.random.default_rng(5)
    b.sqop = (b.sqop * qop_scale).astype(np.float32)
    far = rng.uniform(0, 1, b.n_seeds) < 0.3
    b.sx = np.where(far, b.sx + np.float32(seed_shift), b.sx).astype(np.float32)
    out = rng.uniform(0, 1, b.n_hits) < 0.05
    b.hu = np.where(out, b.hu + np.float32(20.0 * 861.0), b.hu).astype(np.float32)
    ref = O.find_tracks(b, g, n_threads=8)
    ctx = ds.Context(0, g, W)
    try:
        for block in (128, 256):
            ds.ds_set_launch(ctx.handle, 0, block, 2, 512)
            ev, tr = ds.DeviceEvents(b), ds.DeviceTracks(b.n_seeds)
            say(f"[edges] Dv1 map: q/p x {qop_scale}, shift {seed_shift}, loose {loose}, block {block}")
            ds.ds_find_tracks(ctx.handle, ev, tr, ds.DS_MODE_PERSISTENT, 1)
            torch.cuda.synchronize()
            t = tr.to_numpy()
            assert t["flags"] == 0
            parity.compare_tracks(t, ref, min_identical=0.0)
    finally:
        torch.cuda.synchronize()
        ctx.close()


@pytest.mark.parametrize("algorithm,extras", [(0, False), (1, False), (0, True)])
@pytest.mark.parametrize("events,seeds,hits,crowd", [(30, 150, 600, 1), (3, 700, 1100, 1), (300, 16, 60, 4),
                                                     (40, 260, 90, 40), (1, 2200, 500, 3)])
def test_clones_killed_in_one_launch(events, seeds, hits, crowd, algorithm, extras):
    """Clone killing inside the fused step (two hash chains per event) against
    the four launches, and against the oracle's pair loop on the tracks as
    found: events of one and of several chunks of seeds, `crowd` copies of each
    seed so that many tracks share all or most of their hits, equal ones too."""
    g = dict(G0, algorithm=algorithm, clone_kill=1)
    b = synth.generate(dict(name="clones", n_events=events, seed=events + seeds, seeds_per_event=seeds,
                            llp_per_event=seeds // 4, hits_per_layer=hits, zmax=2200.0))
    rng = np.random.default_rng(3)
    src = np.arange(b.n_seeds)
    for s0, s1 in zip(b.seed_off[:-1], b.seed_off[1:]):
        src[s0:s1] = s0 + rng.integers(0, max(1, (s1 - s0) // crowd), s1 - s0) if crowd > 1 else src[s0:s1]
    for k in ("sx", "sy", "stx", "sty", "sqop"):
        setattr(b, k, np.ascontiguousarray(getattr(b, k)[src]))
    b.stx = (b.stx + (rng.uniform(0, 1, b.n_seeds) < 0.5) * rng.normal(0, 2e-5, b.n_seeds)).astype(np.float32)
    outs = []
    for fused in (1, 0):
        ctx = ds.Context(0, g, W)
        try:
            ds.ds_set_step_fusion(ctx.handle, fused)
            if extras:
                ds.ds_load_lines(ctx.handle, synth.line_weights())
            ev, tr = ds.DeviceEvents(b), ds.DeviceTracks(b.n_seeds)
            vt = ds.DeviceVertices(events, 256, extras=extras)
            say(f"[edges] clones: {events} events, {seeds} seeds x {crowd}, algorithm {algorithm}, extras {extras}, fused {fused}")
            for _ in range(2):
                vt.overflow.zero_()
                ds.ds_process(ctx.handle, ev, tr, vt, ds.DS_MODE_PERSISTENT, score_max=0.8)
            torch.cuda.synchronize()
            outs.append((tr.to_numpy(), vt.to_numpy()))
            ds.ds_find_tracks(ctx.handle, ev, tr, ds.DS_MODE_PERSISTENT, 0)
            torch.cuda.synchronize()
            found = tr.to_numpy()
        finally:
            torch.cuda.synchronize()
            ctx.close()
    (t0, v0), (t1, v1) = outs
    assert t0["flags"] == t1["flags"] == 0
    for k in ("x", "y", "tx", "ty", "qop", "chi2", "score", "hits", "nhits", "cand"):
        assert np.array_equal(t0[k], t1[k]), k
    assert v0["flags"] == v1["flags"] == 0
    for k in ("count", "i", "j", "x", "y", "z", "doca", "overflow") + (("m_pipi", "m_ppi") if extras else ()):
        assert np.array_equal(v0[k], v1[k]), k
    if extras:   # (lines: the same float32 network on other tiles)
        assert np.max(np.abs(v0["lines"] - v1["lines"])) <= 1e-6
    assert found["flags"] == 0
    killed = O.kill_clones(b.seed_off, found)
    assert crowd == 1 or killed.sum() > 0
    assert np.array_equal(t0["nhits"], np.where(killed > 0, 0, found["nhits"]))
    assert np.array_equal(t0["chi2"], np.where(killed > 0, 0, found["chi2"]))


@pytest.mark.parametrize("step", [0.03125, 0.25])
def test_ties_do_not_depend_on_the_chosen_bins(step):
    """Hits on a grid, so that candidates tie exactly in chi2: a launch that
    takes wider bins than the context's (another workgroup fits) gives the
    tracks of one that takes them as they are."""
    b = synth.generate(dict(name="ties", n_events=600, seed=9, seeds_per_event=150, llp_per_event=30,
                            hits_per_layer=600, zmax=2200.0))
    b.hu = (np.round(b.hu / step) * step).astype(np.float32)
    outs = []
    for shape in (None, (256, 3, 1024)):
        ctx = ds.Context(0, dict(G0, clone_kill=1), W)
        try:
            if shape:
                ds.ds_set_launch(ctx.handle, 0, *shape)
            ev, tr, vt = ds.DeviceEvents(b), ds.DeviceTracks(b.n_seeds), ds.DeviceVertices(b.n_events, 256)
            say(f"[edges] ties on a grid of {step}, shape {shape}")
            ds.ds_process(ctx.handle, ev, tr, vt, ds.DS_MODE_PERSISTENT, score_max=math.inf)
            torch.cuda.synchronize()
            outs.append(tr.to_numpy())
        finally:
            torch.cuda.synchronize()
            ctx.close()
    for k in ("x", "y", "tx", "ty", "qop", "chi2", "score", "hits", "nhits", "cand", "flags"):
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("algorithm,clone_kill", [(0, 0), (1, 0), (0, 1)])
def test_largest_first_classes_bitwise_equal(algorithm, clone_kill):
    """Uneven events in classes of size, a launch each (many events far below
    the largest), against input order: events at the classes' limits and one
    beyond, empty ones, one of the declared size, one with bad offsets."""
    rng = np.random.default_rng(8)
    n = 4700
    b = synth.generate(dict(name="classes", n_events=n, seed=3, seeds_per_event=24, llp_per_event=4,
                            hits_per_layer=110, zmax=2200.0))
    # events merged at random: one to sixteen of them together, then many single ones
    size = np.concatenate([[16, 16, 0, 1], rng.integers(0, 16, 40), np.ones(n, int)])
    keep = np.cumsum(size) <= n
    first = np.concatenate([[0], np.cumsum(size[keep])])
    first[-1] = min(first[-1], n)
    so = b.seed_off[first].astype(np.int32)
    ho = b.hit_off.astype(np.int64)
    per = np.diff(ho).reshape(n, 4)
    order, hit_off = [], [0]
    for e0, e1 in zip(first[:-1], first[1:]):
        for layer in range(4):
            idx = [np.arange(ho[4 * e + layer], ho[4 * e + layer + 1]) for e in range(e0, e1)]
            order += idx
            hit_off.append(hit_off[-1] + int(per[e0:e1, layer].sum()))
    order = np.concatenate(order)
    for k in ("sx", "sy", "stx", "sty", "sqop"):
        setattr(b, k, np.ascontiguousarray(getattr(b, k)[:so[-1]]))
    b.hu = np.ascontiguousarray(b.hu[order])
    if getattr(b, "hit_sector", None) is not None and len(b.hit_sector):
        b.hit_sector = np.ascontiguousarray(b.hit_sector[order])
    b.seed_off, b.hit_off, b.n_events = so, np.asarray(hit_off, np.int32), len(so) - 1
    assert b.n_events >= 4096
    outs = []
    for how in (ds.DS_ORDER_INPUT, ds.DS_ORDER_LARGEST_FIRST):
        ctx = ds.Context(0, dict(G0, algorithm=algorithm, clone_kill=clone_kill), W)
        try:
            ds.ds_set_event_order(ctx.handle, how)
            ev, tr, vt = ds.DeviceEvents(b), ds.DeviceTracks(b.n_seeds), ds.DeviceVertices(b.n_events, 128)
            ev.hit_off[4 * 700 + 2] += 10 ** 6   # (one event's offsets are not monotone)
            say(f"[edges] classes: {b.n_events} events, algorithm {algorithm}, clone_kill {clone_kill}, order {how}")
            for _ in range(3):
                vt.overflow.zero_()
                ds.ds_process(ctx.handle, ev, tr, vt, ds.DS_MODE_PERSISTENT, score_max=math.inf)
            torch.cuda.synchronize()
            outs.append((tr.to_numpy(), vt.to_numpy()))
        finally:
            torch.cuda.synchronize()
            ctx.close()
    (t0, v0), (t1, v1) = outs
    assert t0["flags"] == t1["flags"] == 1   # DS_F_BAD_OFFSETS
    for k in ("x", "y", "tx", "ty", "qop", "chi2", "score", "hits", "nhits", "cand"):
        assert np.array_equal(t0[k], t1[k]), k
    for k in ("count", "i", "j", "x", "y", "z", "doca", "overflow", "flags"):
        assert np.array_equal(v0[k], v1[k]), k
