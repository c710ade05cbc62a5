"""Events and settings at the limits of what the kernels list and sort in LDS:
layers dense enough for more than 128 hits in a seed's sectors, seeds with
more hits than are listed, crowded bins, and the sizes at which calls are
refused."""
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
TRACK_KEYS = ("x", "y", "tx", "ty", "qop", "chi2", "score", "hits", "nhits", "cand")


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def events(n, seeds, hits, seed, geometry=None):
    return synth.generate(dict(name="limits", n_events=n, seed=seed, seeds_per_event=seeds,
                               llp_per_event=min(seeds // 3, 20), hits_per_layer=hits, zmax=2200.0),
                          geometry=geometry or G0)


def find(b, g, shape=(0, 0, 0), repeat=1):
    """ds_find_tracks (scored) of the batch at a launch shape (zeros: the library's choice)."""
    ctx = ds.Context(0, g, W)
    try:
        if any(shape):
            ds.ds_set_launch(ctx.handle, 0, *shape)
        ev, tr = ds.DeviceEvents(b), ds.DeviceTracks(b.n_seeds)
        for _ in range(repeat):
            ds.ds_find_tracks(ctx.handle, ev, tr, ds.DS_MODE_PERSISTENT, 1)
        torch.cuda.synchronize()
        return tr.to_numpy()
    finally:
        torch.cuda.synchronize()
        ctx.close()


@pytest.mark.parametrize("shape", [(0, 0, 0), (64, 0, 0), (256, 0, 0), (512, 0, 0)])
@pytest.mark.parametrize("hits,seeds", [(850, 200), (1500, 700), (3300, 130)])
def test_dv1_seeds_with_more_than_128_utbx_hits(hits, seeds, shape):
    """Two Y sectors hold from about as many UTbX hits as a seed's triplet
    flags (128) to several times as many, in one and in several chunks of
    seeds: tracks of the oracle at every workgroup size."""
    g = dict(G0, algorithm=1)
    b = events(6, seeds, hits, seed=hits + 3, geometry=g)
    ref = O.find_tracks(b, g, n_threads=8)
    say(f"[limits] Dv1, {hits} hits, {seeds} seeds, shape {shape}")
    t = find(b, g, shape, repeat=3)
    assert t["flags"] == 0
    parity.compare_tracks(t, ref, min_identical=0.0)


def first_window_counts(b, g):
    """UTbX hits inside each seed's first window (float64, the method's formula)."""
    z3 = g["z_layer"][3]
    x, y, tx, ty, q = (getattr(b, k).astype(np.float64) for k in ("sx", "sy", "stx", "sty", "sqop"))
    m = x + tx * (z3 - g["z_seed"]) - (y + ty * (z3 - g["z_seed"])) * g["tan_stereo"][3]
    m += g["polarity"] * g["kick"] * q * (g["z_magnet"] - z3)
    half = g["w1_c0"] + g["w1_c1"] * np.abs(q)
    n = np.zeros(b.n_seeds, int)
    for e in range(b.n_events):
        u = np.sort(b.hu[b.hit_off[4 * e + 3]:b.hit_off[4 * e + 4]].astype(np.float64))
        s = slice(b.seed_off[e], b.seed_off[e + 1])
        n[s] = np.searchsorted(u, m[s] + half[s], "right") - np.searchsorted(u, m[s] - half[s], "left")
    return n


@pytest.mark.parametrize("rows", [False, True])
@pytest.mark.parametrize("hits,seeds", [(2400, 40), (2400, 300), (4700, 90)])
def test_truncated_first_windows_leave_other_seeds_alone(hits, seeds, rows):
    """64 lanes list 192 first-window hits of a seed; here windows grow with
    |q/p| until some seeds have two and four times as many.  The batch is
    flagged, and every other seed has the track and the candidate rows that it
    has where all hits are listed (256 lanes: 768)."""
    g = dict(G0, w1_c0=3.0, w1_c1=240.0)
    b = events(8, seeds, hits, seed=hits + seeds, geometry=g)
    n = first_window_counts(b, g)
    whole = n <= 192
    assert 0 < (~whole).sum() < 0.5 * b.n_seeds and n.max() <= 768
    outs = []
    for shape in ((64, 2, 0), (256, 2, 0)):
        say(f"[limits] truncated windows: {hits} hits, {seeds} seeds, rows {rows}, shape {shape}, "
            f"{(~whole).sum()} of {b.n_seeds} beyond 192")
        if not rows:
            outs.append(find(b, g, shape))
            continue
        ctx = ds.Context(0, g, W)
        try:
            ds.ds_set_launch(ctx.handle, 0, *shape)
            r = ds.DeviceCandidates(b.n_seeds, ds.ds_candidate_slots(ctx.handle))
            ds.ds_score_candidates(ctx.handle, ds.DeviceEvents(b), r)
            torch.cuda.synchronize()
            outs.append(r.to_numpy())
        finally:
            torch.cuda.synchronize()
            ctx.close()
    assert outs[0]["flags"] == ds.DS_F_CAPACITY and outs[1]["flags"] == 0
    if not rows:
        for k in TRACK_KEYS:
            assert np.array_equal(outs[0][k][whole], outs[1][k][whole]), k
        parity.compare_tracks(outs[1], O.find_tracks(b, g, n_threads=8), min_identical=0.0)
        return
    whole = whole[np.arange(len(outs[1]["nhits"])) // r.slots]
    full = whole & (outs[1]["nhits"] > 0)
    assert np.array_equal(whole & (outs[0]["nhits"] > 0), full)
    for k in TRACK_KEYS + ("seed",):
        assert np.array_equal(outs[0][k][full], outs[1][k][full]), k


def batch_slice(b, e0, e1):
    s0, s1, h0, h1 = b.seed_off[e0], b.seed_off[e1], b.hit_off[4 * e0], b.hit_off[4 * e1]
    return synth.EventBatch(e1 - e0, b.seed_off[e0:e1 + 1] - s0, *(getattr(b, k)[s0:s1].copy() for k in
                            ("sx", "sy", "stx", "sty", "sqop")), b.hit_off[4 * e0:4 * e1 + 1] - h0, b.hu[h0:h1].copy(),
                            hit_sector=b.hit_sector[h0:h1].copy())


def join(a, b):
    """One batch of two."""
    c = lambda k: np.concatenate([getattr(a, k), getattr(b, k)])
    off = lambda k: np.concatenate([getattr(a, k), getattr(b, k)[1:] + getattr(a, k)[-1]]).astype(np.int32)
    return synth.EventBatch(a.n_events + b.n_events, off("seed_off"), *(c(k) for k in ("sx", "sy", "stx", "sty", "sqop")),
                            off("hit_off"), c("hu"), hit_sector=c("hit_sector"))


@pytest.mark.parametrize("block,hits", [(64, 1200), (0, 3600)])
def test_truncated_dv1_seeds_are_a_function_of_their_event(block, hits):
    """Four wide Y sectors and windows of 10 mm: seeds with more triplets than
    the three per lane that are listed (192, 768) keep the first ones in the
    order of the hits' sectors and indices, whatever else is in the batch,
    whichever workgroup the library takes and whatever its bins."""
    g = dict(synth.default_geometry(loose=True), algorithm=1, n_sectors=4, sector_h=400.0)
    dense, thin = events(3, 150, hits, seed=5, geometry=g), events(700, 12, 40, seed=6, geometry=g)
    ref = find(dense, g, (block or 256, 1, 0))
    say(f"[limits] truncated Dv1 seeds, block {block}, {hits} hits")
    assert ref["flags"] == ds.DS_F_CAPACITY and (ref["nhits"] > 0).mean() > 0.5
    outs = [find(dense, g, (block, 0, 0), repeat=2), find(batch_slice(dense, 0, 1), g, (block, 0, 0)),
            find(join(dense, thin), g, (block, 0, 0)), find(dense, g, (block, 0, 256))]
    for t in outs:
        n = min(dense.n_seeds, len(t["nhits"]))
        assert t["flags"] == ds.DS_F_CAPACITY
        for k in TRACK_KEYS:
            assert np.array_equal(t[k][:n], ref[k][:n]), k


@pytest.mark.parametrize("crowd", ["bins", "more", "edges"])
@pytest.mark.parametrize("block", [0, 512])
def test_crowded_bins_keep_run_order(block, crowd):
    """Bins of many more than 32 UTbX hits, all hits twice (the second copies
    in another place of the run), so that a seed's candidates tie exactly in
    chi2: workgroups whose wavefronts share a layer report the hit that one
    wavefront's placing order gives, every time."""
    g = dict(G0)
    if crowd == "edges":   # a binned range of 100 mm: nearly all hits lie in the two end bins
        g.update(u_min=-50.0, u_max=50.0)
    if crowd == "more":   # and of up to about 256 hits in the inner ones
        g.update(u_min=-300.0, u_max=300.0)
    b = events(6, 150, 1300 if crowd != "more" else 2100, seed=4, geometry=g)
    rng = np.random.default_rng(7)
    hu, off = [], [0]
    for k in range(4 * b.n_events):
        u = b.hu[b.hit_off[k]:b.hit_off[k + 1]]
        hu.append(rng.permutation(np.concatenate([u, u])))
        off.append(off[-1] + 2 * len(u))
    b.hu, b.hit_off, b.hit_sector = np.concatenate(hu), np.asarray(off, np.int32), None
    bins = {"bins": 64, "more": 64, "edges": 1024}[crowd]
    say(f"[limits] crowded bins: {crowd}, block {block}")
    ref = find(b, g, (256, 1, bins))
    assert ref["flags"] == 0 and (ref["nhits"] > 0).mean() > 0.3
    for _ in range(4):
        t = find(b, g, (block, 0, bins), repeat=3)
        for k in TRACK_KEYS + ("flags",):
            assert np.array_equal(t[k], ref[k]), k


def first_triplets_cut(b, g, e, limit):
    """Length of event e's UTbX run up to its only seed's `limit`-th triplet, and whether the seed reaches one
    UTbX sector only."""
    x, y, tx, ty, q = (float(getattr(b, k)[b.seed_off[e]]) for k in ("sx", "sy", "stx", "sty", "sqop"))
    z, zm = g["z_layer"], g["z_magnet"]
    run = lambda L: slice(b.hit_off[4 * e + L], b.hit_off[4 * e + L + 1])
    c = lambda L: x + tx * (z[L] - g["z_seed"]) - (y + ty * (z[L] - g["z_seed"])) * g["tan_stereo"][L]

    def reach(L):
        yl = y + ty * (z[L] - g["z_seed"]) - g["sector_y0"]
        return [int(np.floor((yl + s * g["sector_tol"]) / g["sector_h"])) for s in (-1, 1)]
    (a0, a1), (b0, b1) = reach(0), reach(3)
    u0, s0 = b.hu[run(0)].astype(np.float64), b.hit_sector[run(0)].astype(int)
    u3, s3 = b.hu[run(3)].astype(np.float64), b.hit_sector[run(3)].astype(int)
    u0 = u0[(s0 >= a0) & (s0 <= a1)]
    m = (u3 - c(3)) * (zm - z[0]) / (zm - z[3]) + c(0)
    half = g["w2_c0"] + g["w2_c1"] * abs(q)
    trip = (s3 == b0) & (np.abs(u0[None, :] - m[:, None]) <= half).any(1)
    k = np.nonzero(trip)[0]
    return (int(k[limit - 1]) + 1 if len(k) > limit else len(u3)), b0 == b1, len(k)


@pytest.mark.parametrize("shape,limit,hits", [((64, 0, 0), 192, 1200), ((0, 0, 0), 768, 3600), ((256, 0, 0), 768, 3600)])
def test_truncated_dv1_seeds_keep_the_limit_s_triplets(shape, limit, hits):
    """A seed with more triplets than three per lane has the oracle's track of
    its event cut off behind the last triplet that is listed."""
    g = dict(synth.default_geometry(loose=True), algorithm=1, n_sectors=3, sector_h=1400.0 / 3.0)
    b = events(24, 1, hits, seed=hits, geometry=g)
    say(f"[limits] triplets listed, shape {shape}, {hits} hits")
    t = find(b, g, shape)
    assert t["flags"] == ds.DS_F_CAPACITY
    cut = [first_triplets_cut(b, g, e, limit) for e in range(b.n_events)]
    use = np.array([one for _, one, _ in cut])
    assert use.sum() > 12 and all(n > limit for _, _, n in cut)
    keep = np.ones(b.n_hits, bool)
    for e, (n, _, _) in enumerate(cut):
        keep[b.hit_off[4 * e + 3] + n:b.hit_off[4 * e + 4]] = False
    runs = np.add.reduceat(keep, b.hit_off[:-1])
    c = synth.EventBatch(b.n_events, b.seed_off, b.sx, b.sy, b.stx, b.sty, b.sqop,
                         np.concatenate([[0], np.cumsum(runs)]).astype(np.int32), b.hu[keep], hit_sector=b.hit_sector[keep])
    ref = O.find_tracks(c, g, n_threads=8)
    sub = lambda d: {k: v[use] for k, v in d.items() if isinstance(v, np.ndarray) and len(v) == len(use)}
    parity.compare_tracks(sub(t), sub(ref), min_identical=0.0)


@pytest.mark.parametrize("hits,seeds,half", [(1650, 30, 185.0), (3000, 30, 102.0), (3000, 90, 102.0)])
def test_truncated_first_windows_do_not_depend_on_the_chosen_bins(hits, seeds, half):
    """First windows of about twice the hits that are listed of them (64 lanes:
    192), so that the listing ends among a seed's closest hits: the library's
    bins, wider than the 1 024 asked for where that lets another workgroup in,
    give the tracks of the asked ones."""
    g = dict(G0, w1_c0=half, w1_c1=0.0)
    b = events(24, seeds, hits, seed=hits + seeds, geometry=g)
    say(f"[limits] truncated windows at the chosen bins, {hits} hits, {seeds} seeds")
    ref, t = find(b, g, (64, 0, 1024)), find(b, g, (64, 0, 0))
    assert ref["flags"] == ds.DS_F_CAPACITY and (ref["nhits"] > 0).sum() > 20
    for k in TRACK_KEYS + ("flags",):
        assert np.array_equal(t[k], ref[k]), k


@pytest.mark.parametrize("gap", [4.0, 20.0, 2000.0])
def test_dv1_map_with_a_magnet_point_near_the_last_layer(gap):
    """A magnet point `gap` mm behind UTbX projects a hit to UTaX with a factor
    of up to a hundred, and seeds 15 m out leave the float32 look-up little
    precision: bins of 0.01 mm, windows of one width and few UTaX hits show
    every triplet that it would lose."""
    g = dict(G0, algorithm=1, w2_c0=0.5, w2_c1=0.0, u_min=14995.0, u_max=15005.0)
    g["z_magnet"] = g["z_layer"][3] + gap
    rng = np.random.default_rng(int(gap))
    E, S = 8, 120
    off = np.concatenate([[0], np.cumsum(np.tile([4, 60, 60, 60], E))]).astype(np.int32)
    n = E * S
    f = lambda *a: rng.uniform(*a, n).astype(np.float32)
    seeds = (f(14996.0, 15004.0), f(10.0, 40.0), f(-3e-4, 3e-4), f(-1e-4, 1e-4),
             np.where(rng.uniform(0, 1, n) < 0.5, 1, -1).astype(np.float32) * f(0.02, 0.4))
    b = synth.EventBatch(E, np.arange(0, n + 1, S, dtype=np.int32), *seeds, off,
                         rng.uniform(14995.0, 15005.0, off[-1]).astype(np.float32),
                         hit_sector=np.full(off[-1], 7, np.uint8))   # (heights 0 to 100 mm)
    say(f"[limits] Dv1 map, magnet point {gap} mm behind UTbX")
    ref = O.find_tracks(b, g, n_threads=8)
    assert (ref["nhits"] > 0).sum() > 150
    for shape in ((128, 1, 512), (0, 0, 0)):
        t = find(b, g, shape)
        assert t["flags"] == 0
        parity.compare_tracks(t, ref, min_identical=0.0)


@pytest.mark.parametrize("block,largest", [(64, 5376), (128, 5312), (256, 5120), (512, 4864)])
def test_vertexing_takes_events_up_to_the_same_size(block, largest):
    """The seeds per event that ds_vertex takes at each workgroup size, and one
    more, for which 64 are counted, that it refuses."""
    b = events(2, 6, 20, seed=1)
    ctx = ds.Context(0, G0, W)
    try:
        ds.ds_set_launch(ctx.handle, 1, block, 0, 0)
        tr, vt = ds.DeviceTracks(b.n_seeds), ds.DeviceVertices(b.n_events, 16)
        say(f"[limits] vertexing, block {block}, {largest} seeds declared")
        ds.ds_vertex(ctx.handle, ds.DeviceEvents(b, max_seeds_per_event=largest), tr, 1.0, vt, ds.DS_MODE_PERSISTENT)
        with pytest.raises(ds.DsError, match="DS_E_CAPACITY"):
            ds.ds_vertex(ctx.handle, ds.DeviceEvents(b, max_seeds_per_event=largest + 1), tr, 1.0, vt,
                         ds.DS_MODE_PERSISTENT)
        torch.cuda.synchronize()
        assert vt.to_numpy()["flags"] == 0
    finally:
        torch.cuda.synchronize()
        ctx.close()


@pytest.mark.parametrize("mode", [ds.DS_MODE_PERSISTENT, ds.DS_MODE_GRAPH])
@pytest.mark.parametrize("warm", [False, True])
def test_captured_largest_first_calls_outlive_a_larger_batch(warm, mode):
    """A largest-first call captured into a caller's graph, as the stream's
    first call (nothing may be allocated: it takes input order) and after an
    eager one; then a batch that needs a larger workspace on the same stream,
    and replays among eager work, each bitwise the eager result."""
    b, big = events(300, 20, 60, seed=2), events(2500, 8, 24, seed=3)
    ctx, s = ds.Context(0, G0, W), torch.cuda.Stream()
    try:
        ds.ds_set_event_order(ctx.handle, ds.DS_ORDER_LARGEST_FIRST)
        ev, tr, vt = ds.DeviceEvents(b), ds.DeviceTracks(b.n_seeds), ds.DeviceVertices(b.n_events, 64)
        evb, trb, vtb = ds.DeviceEvents(big), ds.DeviceTracks(big.n_seeds), ds.DeviceVertices(big.n_events, 64)
        step = lambda: ds.ds_process(ctx.handle, ev, tr, vt, mode, score_max=math.inf, stream=s)
        larger = lambda: ds.ds_process(ctx.handle, evb, trb, vtb, mode, score_max=math.inf, stream=s)
        torch.cuda.synchronize()
        if warm:
            step()
            s.synchronize()
        say(f"[limits] capture, mode {mode}, warm {warm}")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            step()
        outs = []
        for k in range(4):
            with torch.cuda.stream(s):
                for t in (tr.x, tr.nhits, vt.count, vt.x):
                    t.fill_(-7)
                vt.overflow.zero_()
                graph.replay()
            s.synchronize()
            outs.append((tr.to_numpy(), vt.to_numpy()))
            larger()
            torch.cuda.synchronize()
        step()
        torch.cuda.synchronize()
        rt, rv = tr.to_numpy(), vt.to_numpy()
        bt = trb.to_numpy()
    finally:
        torch.cuda.synchronize()
        ctx.close()
    assert rt["flags"] == 0 and (rt["nhits"] > 0).any() and bt["flags"] == 0
    parity.compare_tracks(bt, O.find_tracks(big, G0, n_threads=8), min_identical=0.0)
    for t, v in outs:
        for k in TRACK_KEYS:
            assert np.array_equal(t[k], rt[k]), k
        for k in ("count", "i", "j", "x", "y", "z", "doca"):
            assert np.array_equal(v[k], rv[k]), k


@pytest.mark.parametrize("bound", [2**31 - 1, 2**31 - 16, 2**20])
def test_tracking_takes_any_bound_on_the_seeds_of_an_event(bound):
    """Calls that keep no seeds in LDS beyond a chunk take the largest bounds
    that the struct holds; the fused step and the vertexing refuse them."""
    b = events(20, 30, 80, seed=9)
    ref = find(b, G0)
    ctx = ds.Context(0, G0, W)
    try:
        ev, tr, vt = ds.DeviceEvents(b, max_seeds_per_event=bound), ds.DeviceTracks(b.n_seeds), ds.DeviceVertices(20, 8)
        say(f"[limits] {bound} seeds declared")
        ds.ds_find_tracks(ctx.handle, ev, tr, ds.DS_MODE_PERSISTENT, 1)
        r = ds.DeviceCandidates(b.n_seeds, ds.ds_candidate_slots(ctx.handle))
        ds.ds_score_candidates(ctx.handle, ev, r)
        torch.cuda.synchronize()
        t, rows = tr.to_numpy(), r.to_numpy()
        for call in (lambda: ds.ds_process(ctx.handle, ev, tr, vt), lambda: ds.ds_vertex(ctx.handle, ev, tr, 1.0, vt),
                     lambda: ds.ds_kill_clones(ctx.handle, ev, tr)):
            with pytest.raises(ds.DsError, match="DS_E_CAPACITY"):
                call()
    finally:
        torch.cuda.synchronize()
        ctx.close()
    for k in TRACK_KEYS:
        assert np.array_equal(t[k], ref[k]), k
    assert t["flags"] == ref["flags"] == rows["flags"] == 0 and (rows["nhits"] > 0).any()


@pytest.mark.parametrize("what", ["run of 70 000 hits", "bad hit offsets", "bad seed offsets", "non-finite hit"])
def test_skipped_events_are_the_same_in_one_launch_and_in_four(what):
    """Clone killing fused and as four launches on a batch with one event that
    is skipped: the same words are written, the others left alone, and the
    same flags are set."""
    b = events(6, 40, 100, seed=12)
    if what.startswith("run"):   # event 2: 70 000 hits in its first layer
        u = np.random.default_rng(1).uniform(-800, 800, 70000).astype(np.float32)
        b.hu = np.insert(b.hu, b.hit_off[8], u)
        b.hit_off = np.concatenate([b.hit_off[:9], b.hit_off[9:] + 70000]).astype(np.int32)
        b.hit_sector = None
    if what.startswith("non"):
        b.hu[b.hit_off[9] + 3] = np.inf
    outs = []
    for fused in (1, 0):
        ctx = ds.Context(0, dict(G0, clone_kill=1), W)
        try:
            ds.ds_set_step_fusion(ctx.handle, fused)
            ev = ds.DeviceEvents(b, max_hits_per_event=4096)
            if what == "bad hit offsets":
                ev.hit_off[9] = 10**8
            if what == "bad seed offsets":
                ev.seed_off[2] = -5
            tr, vt = ds.DeviceTracks(b.n_seeds), ds.DeviceVertices(b.n_events, 32)
            for t in (tr.x, tr.score, tr.chi2, vt.x):
                t.fill_(7.0)
            vt.count.fill_(-7)
            say(f"[limits] skipped event: {what}, fused {fused}")
            ds.ds_process(ctx.handle, ev, tr, vt, ds.DS_MODE_PERSISTENT, score_max=math.inf)
            torch.cuda.synchronize()
            outs.append((tr.to_numpy(), vt.to_numpy()))
        finally:
            torch.cuda.synchronize()
            ctx.close()
    (t0, v0), (t1, v1) = outs
    assert t0["flags"] != 0
    for k in TRACK_KEYS + ("flags",):
        assert np.array_equal(t0[k], t1[k]), k
    for k in ("count", "i", "j", "x", "y", "z", "doca", "overflow", "flags"):
        assert np.array_equal(v0[k], v1[k]), k


@pytest.mark.parametrize("order", [ds.DS_ORDER_INPUT, ds.DS_ORDER_LARGEST_FIRST])
@pytest.mark.parametrize("n", [60, 700, 4500])
def test_part_of_a_resident_batch(n, order):
    """The first events of longer arrays, whose lengths say nothing of the
    part's occupancy, against the same events as a batch of their own."""
    b = synth.generate(2, n_events=5000, seed=17)
    part = b.subset(np.arange(n))
    outs = []
    for whole in (True, False):
        ctx = ds.Context(0, G0, W)
        try:
            ds.ds_set_event_order(ctx.handle, order)
            src = b if whole else part
            ev, tr, vt = ds.DeviceEvents(src), ds.DeviceTracks(src.n_seeds), ds.DeviceVertices(n, 64)
            ev.struct.n_events = n
            say(f"[limits] part: {n} of {b.n_events} events, whole arrays {whole}, order {order}")
            ds.ds_process(ctx.handle, ev, tr, vt, ds.DS_MODE_PERSISTENT, score_max=math.inf)
            torch.cuda.synchronize()
            outs.append((tr.to_numpy(), vt.to_numpy()))
        finally:
            torch.cuda.synchronize()
            ctx.close()
    (t0, v0), (t1, v1) = outs
    assert t0["flags"] == t1["flags"] == 0
    for k in TRACK_KEYS:
        assert np.array_equal(t0[k][:part.n_seeds], t1[k]), k
    for k in ("count", "i", "j", "x", "y", "z", "doca", "overflow"):
        assert np.array_equal(v0[k], v1[k]), k


def test_launch_settings_are_handed_back():
    """ds_reset_launch takes a context's settings back to those of ds_create,
    whatever was set, and refuses what ds_set_launch refuses as a kernel."""
    ctx = ds.Context(0, G0, W)
    try:
        new = [ds.ds_get_launch(ctx.handle, k) for k in (0, 1)]
        ds.ds_set_launch(ctx.handle, 0, 512, 2, 256)
        ds.ds_set_launch(ctx.handle, 1, 64, 8, 0)
        assert [ds.ds_get_launch(ctx.handle, k) for k in (0, 1)] != new
        for k in (0, 1):
            ds.ds_reset_launch(ctx.handle, k)
        assert [ds.ds_get_launch(ctx.handle, k) for k in (0, 1)] == new
        with pytest.raises(ds.DsError, match="DS_E_ARG"):
            ds.ds_reset_launch(ctx.handle, 2)
    finally:
        ctx.close()


def step(ctx, b, extras, cap=128, static=False, score_max=math.inf, repeat=2):
    ev, tr = ds.DeviceEvents(b), ds.DeviceTracks(b.n_seeds)
    vt = ds.DeviceVertices(b.n_events, cap, extras=extras)
    for _ in range(repeat):
        vt.overflow.zero_()
        if static:
            ds.ds_process_static(ctx.handle, ev, tr, vt, score_max=score_max)
        else:
            ds.ds_process(ctx.handle, ev, tr, vt, ds.DS_MODE_PERSISTENT, score_max=score_max)
    torch.cuda.synchronize()
    return tr.to_numpy(), vt.to_numpy()


def assert_same_step(a, b, extras):
    (t0, v0), (t1, v1) = a, b
    for k in TRACK_KEYS + ("flags",):
        assert np.array_equal(t0[k], t1[k]), k
    for k in ("count", "i", "j", "x", "y", "z", "doca", "overflow", "flags") + (("m_pipi", "m_ppi") if extras else ()):
        assert np.array_equal(v0[k], v1[k]), k
    if extras:   # (the same float32 networks, compiled into another kernel)
        assert np.max(np.abs(v0["lines"] - v1["lines"])) <= 1e-6


@pytest.mark.parametrize("algorithm,extras,fringe", [(1, True, 0.0), (0, False, 1.0), (0, True, -1.0), (1, True, 1.0)])
@pytest.mark.parametrize("seeds,hits", [(150, 500), (700, 900)])
def test_clone_killing_fused_with_every_option(seeds, hits, algorithm, extras, fringe):
    """Clone killing in the fused launch with Dv1, masses and trigger lines
    and curved trajectories together: bitwise the four launches."""
    g = dict(G0, algorithm=algorithm, clone_kill=1, fringe_polarity=fringe)
    b = events(12, seeds, hits, seed=seeds, geometry=g)
    src = np.arange(b.n_seeds)   # (every fourth seed twice in a row)
    src[1::4] = src[0::4][:len(src[1::4])]
    src = np.maximum(src, np.repeat(b.seed_off[:-1], np.diff(b.seed_off)))
    for k in ("sx", "sy", "stx", "sty", "sqop"):
        setattr(b, k, np.ascontiguousarray(getattr(b, k)[src]))
    outs = []
    for fused in (1, 0):
        ctx = ds.Context(0, g, W)
        try:
            ds.ds_load_lines(ctx.handle, synth.line_weights())
            ds.ds_set_step_fusion(ctx.handle, fused)
            say(f"[limits] clones: {seeds} seeds, algorithm {algorithm}, extras {extras}, fringe {fringe}, fused {fused}")
            outs.append(step(ctx, b, extras, score_max=0.7))
        finally:
            torch.cuda.synchronize()
            ctx.close()
    assert outs[0][0]["flags"] == 0 and outs[0][1]["count"].sum() > 10
    assert_same_step(*outs, extras)


@pytest.mark.parametrize("algorithm,clone_kill,extras,static", [(0, 0, True, False), (0, 0, False, True), (1, 1, True, True),
                                                               (1, 0, True, False)])
def test_classes_of_size_with_every_option(algorithm, clone_kill, extras, static):
    """Largest-first batches in classes of size with masses and lines, clones
    killed and through the entry point that allocates nothing: bitwise one
    launch in input order."""
    g = dict(G0, algorithm=algorithm, clone_kill=clone_kill)
    b = synth.generate(2, n_events=4400, seed=23)
    outs = []
    for order in (ds.DS_ORDER_INPUT, ds.DS_ORDER_LARGEST_FIRST):
        ctx = ds.Context(0, g, W)
        try:
            ds.ds_load_lines(ctx.handle, synth.line_weights())
            ds.ds_set_event_order(ctx.handle, order)
            say(f"[limits] classes: algorithm {algorithm}, clones {clone_kill}, extras {extras}, static {static}, order {order}")
            outs.append(step(ctx, b, extras, static=static and order == ds.DS_ORDER_LARGEST_FIRST))
        finally:
            torch.cuda.synchronize()
            ctx.close()
    assert outs[0][0]["flags"] == 0 and outs[0][1]["count"].sum() > 1000
    assert_same_step(*outs, extras)


def former_capacity(hits, seeds, block, bins, algorithm, fused, nsec=14):
    """LDS that decides whether tracking takes events of `hits` and `seeds`, as ds_set_launch's values have
    always decided it: hits and bounds, a lane's seed and three items, 24 bytes per kept track, 6 for its row
    where they do not fit beside the pair buffer."""
    r16 = lambda v: (v + 15) // 16 * 16
    hcap, tcap = max(r16(hits), 16), r16(max(seeds, 1)) if fused else 0
    nbu = max(4, (4 * bins - nsec - 4) // (3 * nsec)) if algorithm else bins
    nb, nb3 = (nsec * nbu + 1, nsec + 1) if algorithm else (bins, bins)
    region = r16(block * 52) + r16(12 * block) + r16(24 * block)
    lds = r16(r16(6 * hcap) + 2 * (3 * nb + nb3 + 1)) + region
    if fused:
        ring = 4
        while ring < 24 * block:
            ring *= 2
        rows = r16(6 * tcap + 4)
        lds += r16(24 * tcap) + (0 if region >= ring + rows else rows)
    return lds


@pytest.mark.parametrize("algorithm", [0, 1])
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("block,bins", [(64, 64), (64, 4096), (192, 512), (256, 1024), (512, 2048)])
def test_tracking_takes_events_up_to_the_same_size(block, bins, fused, algorithm):
    """Largest declared events that tracking and the fused step take, and the
    next that they refuse, at settings of the caller's own."""
    b = events(3, 12, 30, seed=2)
    limit = 160 * 1024 - 256
    ctx = ds.Context(0, dict(G0, algorithm=algorithm), W)
    try:
        ds.ds_set_launch(ctx.handle, 0, block, 0, bins)
        ds.ds_set_launch(ctx.handle, 1, 64, 0, 0)
        tr, vt = ds.DeviceTracks(b.n_seeds), ds.DeviceVertices(3, 8)
        for seeds in (40, 900, 2500):
            most = max(h for h in range(16, 32768, 16) if former_capacity(h, seeds, block, bins, algorithm, fused) <= limit)
            for hits in (most, most + 1):
                say(f"[limits] capacity: {block}, {bins}, fused {fused}, algorithm {algorithm}: {seeds} seeds, {hits} hits")
                ev = ds.DeviceEvents(b, max_seeds_per_event=seeds, max_hits_per_event=hits)
                call = ((lambda: ds.ds_process(ctx.handle, ev, tr, vt, ds.DS_MODE_PERSISTENT, score_max=1.0)) if fused else
                        (lambda: ds.ds_find_tracks(ctx.handle, ev, tr, ds.DS_MODE_PERSISTENT, 1)))
                if hits == most:
                    call()
                    torch.cuda.synchronize()
                    assert tr.to_numpy()["flags"] == 0
                else:
                    with pytest.raises(ds.DsError, match="DS_E_CAPACITY"):
                        call()
    finally:
        torch.cuda.synchronize()
        ctx.close()
