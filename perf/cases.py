"""The workloads that the library's speed is followed on.

Each case is one pass of a user's program through the public entry points: a
batch of synthetic events of a stated occupancy, made on the device from a
seed with the distributions of the package's generator (long-lived particles
decaying before the tracker, ghost seeds, noise hits), and the call or calls
that process it.  ``exact`` repeats the method in float64 with plain torch.
"""
import math

import torch

from paper_2503_13092_amd import autotune, ds, synth

SLOTS = 40          # candidate rows per seed with the default geometry: 10 UTbX hits x 1 x 2 x 2
U_RANGE = 1722.0    # mm covered by the hits' u


# call:      process     ds_process (mode "graph" or "persistent")
#            static      ds_process_static
#            staged      ds_find_tracks, ds_ghost_kill and ds_vertex as calls of their own
#            candidates  ds_score_candidates
# ragged:    occupancies follow a Poisson pile-up around the stated means, as real events do
# all_pairs: every found track is vertexed, not only those the ghost-killer keeps
# bounds:    the caller declares room for the largest event it may ever see, as a server does
_DEFAULT = dict(call="process", mode="graph", events=1, seeds=150, hits=600, ragged=False, algorithm=0, loose=False,
                clone=False, extras=False, fringe=0.0, all_pairs=False, cap=64, cand=True, bounds=False)


def _case(name, **kw):
    return dict(_DEFAULT, name=name, **kw)


def listed():
    return [
        # a server that is asked for one event at a time: the latency floor of a call
        _case("serve_1", mode="persistent", events=1, seeds=149, hits=583, cand=False, bounds=True),
        # what a server admits in one batch at 100 000 events/s: uneven events, room declared for the largest
        _case("serve_64", mode="persistent", events=64, seeds=148, hits=583, ragged=True, cand=False, bounds=True),
        # a small replayed batch of nearly empty events (the package's first configuration)
        _case("tiny_100", events=100, seeds=20, hits=500),
        # the benchmark batch, Dv0 and Dv1
        _case("throughput_10k", events=10000, cand=False),
        _case("throughput_10k_dv1", events=10000, algorithm=1, cand=False),
        # a slice of pile-up events, occupancies spread over more than a factor of ten
        _case("uneven_20k", events=20000, seeds=148, hits=583, ragged=True, cand=False),
        # busy events, every opposite-charge pair of found tracks vertexed
        _case("stress_5k", events=5000, seeds=300, hits=1200, all_pairs=True, cap=1024, cand=False),
        # the fullest events that a workgroup's memory takes
        _case("dense_500", events=500, seeds=300, hits=4800),
        # clone killing switched on
        _case("clones_4k", mode="persistent", events=4000, clone=True),
        # masses and trigger lines of every vertex of the found tracks, curved trajectories, no allocation in the call
        _case("lines_curved_3k", call="static", events=3001, seeds=148, hits=583, ragged=True, extras=True, fringe=1.0,
              all_pairs=True, cap=256),
        # training rows: every candidate of the wide windows, scored
        _case("training_rows_300", call="candidates", events=301, loose=True),
        # the steps as calls of their own, an odd batch
        _case("staged_1111", call="staged", mode="persistent", events=1111, seeds=77, hits=333),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    c = dict(_DEFAULT)
    c["call"] = rng.choice(("process", "process", "process", "static", "staged", "candidates"))
    c["mode"] = rng.choice(("graph", "persistent"))
    c["events"] = log_int(1, 20000)
    c["ragged"] = rng.random() < 0.4
    c["seeds"] = log_int(5, 200 if c["ragged"] else 600)
    c["hits"] = log_int(16, 1300 if c["ragged"] else 4800)
    c["cand"] = rng.random() < 0.5
    if c["call"] == "candidates":
        c["loose"] = rng.random() < 0.5
    else:
        c["algorithm"] = int(rng.random() < 0.35)
        c["clone"] = c["call"] != "staged" and rng.random() < 0.25
        c["extras"] = rng.random() < 0.25
        c["fringe"] = rng.choice((0.0, 0.0, 1.0, -1.0))
        c["all_pairs"] = rng.random() < 0.3
        c["cap"] = 1024 if c["all_pairs"] else 64
    # no more work than the listed cases of its kind: hits, seeds, seed-hit products, pairs, rows
    s, h = c["seeds"], c["hits"]
    most = min(24e6 / (4 * h), 1.5e6 / s)
    if c["algorithm"] == 1:
        most = min(most, 6e8 / (s * h))
    if c["all_pairs"]:
        most = min(most, 3e8 / (s * s * (4 if c["extras"] or c["fringe"] else 1)), 5000)
    if c["call"] == "candidates":
        most = min(most, 45000 / s)
        if c["loose"]:
            most = min(most, 2.5e7 / (s * h))
    c["events"] = max(1, min(c["events"], int(most)))
    return c


# --------------------------------------------------------------------- inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _geometry(case):
    g = synth.default_geometry(loose=bool(case["loose"]))
    g.update(algorithm=int(case["algorithm"]), clone_kill=int(case["clone"]), fringe_polarity=float(case["fringe"]))
    return g


def _gamma(g, qop):
    return -g["fringe_polarity"] * (g["gamma_c0"] + g["gamma_c1"] * qop * 1e-3)


def _events(case, seed):
    """One batch on the device: float32 seeds and hits, int32 offsets, uint8 Y sectors."""
    g, dev = _geometry(case), _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * 7919 + 17)
    f64 = torch.float64
    E = int(case["events"])
    rand = lambda n, lo, hi: lo + (hi - lo) * torch.rand(n, generator=gen, device=dev, dtype=f64)
    randn = lambda n: torch.randn(n, generator=gen, device=dev, dtype=f64)
    sign = lambda n: torch.where(rand(n, 0.0, 1.0) < 0.5, 1.0, -1.0)
    zl, tana = g["z_layer"], g["tan_stereo"]
    zmax = 2500.0 if case["all_pairs"] else 2200.0

    # occupancies
    if case["ragged"]:
        # one mixture of event sizes per case (so that every batch of it holds as many seeds), its events in a
        # random order; the hits follow the event's pile-up
        mix = torch.Generator(device=dev)
        mix.manual_seed(E)
        nu = torch.poisson(torch.full((E,), 5.3, device=dev, dtype=f64), generator=mix)
        n_seed = torch.poisson(nu * (case["seeds"] / 5.3), generator=mix).clamp(5, 600).long()
        order = torch.argsort(rand(E, 0.0, 1.0))
        nu, n_seed = nu[order], n_seed[order]
        n_llp = torch.minimum(rand(E, 0.0, 4.0).long().clamp(max=3), n_seed // 2)
        noise = torch.poisson((nu * (case["hits"] / 5.3)).repeat_interleave(4), generator=gen).long()
        noise = noise.clamp(max=4700 if case["call"] == "candidates" or case["seeds"] > 150 else 4800)
    else:
        n_seed = torch.full((E,), int(case["seeds"]), device=dev)
        n_llp = torch.full((E,), int(case["seeds"]) // 5, device=dev)
        noise = None
    ev = torch.arange(E, device=dev)

    # tracks: the daughters of each decay (opposite charges), then ghosts
    l_ev = ev.repeat_interleave(n_llp)
    g_ev = ev.repeat_interleave(n_seed - 2 * n_llp)
    NL, NG = l_ev.numel(), g_ev.numel()
    two = torch.arange(NL, device=dev).repeat_interleave(2)
    p_tx = torch.cat([rand(NL, -0.25, 0.25)[two], rand(NG, -0.25, 0.25)])
    p_ty = torch.cat([rand(NL, -0.2, 0.2)[two], rand(NG, -0.2, 0.2)])
    zd = torch.cat([rand(NL, 0.0, zmax)[two], rand(NG, 0.0, zmax)])
    q0 = sign(NL)
    ch = torch.cat([torch.stack([q0, -q0], 1).reshape(-1), sign(NG)])
    t_ev = torch.cat([l_ev[two], g_ev])
    NT = t_ev.numel()
    vx, vy = p_tx * zd, p_ty * zd
    qop, x0, tx0, ty = (torch.zeros(NT, device=dev, dtype=f64) for _ in range(4))
    todo = torch.arange(NT, device=dev)
    for _ in range(1000):   # redrawn until inside the acceptance
        m = todo.numel()
        if m == 0:
            break
        q = ch[todo] / torch.exp(rand(m, math.log(2.0), math.log(100.0)))
        a, b = p_tx[todo] + 0.02 * randn(m), p_ty[todo] + 0.02 * randn(m)
        z, gam = zd[todo], _gamma(g, q)
        h = g["z_ref"] - z
        xr, tr = vx[todo] + a * h + gam * h * h, a + 2.0 * gam * h   # state at the UT midpoint
        ok = torch.ones(m, dtype=torch.bool, device=dev)
        for L in range(4):
            inside = ((xr + tr * (zl[L] - g["z_ref"])).abs() < 800.0) & ((vy[todo] + b * (zl[L] - z)).abs() < 700.0)
            ok &= inside | (zl[L] <= z)
        xm = xr + tr * (g["z_magnet"] - g["z_ref"])
        ta = tr + g["polarity"] * g["kick"] * q
        ok &= (xm + ta * (g["z_seed"] - g["z_magnet"])).abs() < 3000.0
        ok &= (vy[todo] + b * (g["z_seed"] - z)).abs() < 2500.0
        k = todo[ok]
        qop[k], x0[k], tx0[k], ty[k] = q[ok], xr[ok], tr[ok], b[ok]
        todo = todo[~ok]
    ta = tx0 + g["polarity"] * g["kick"] * qop
    xs = x0 + tx0 * (g["z_magnet"] - g["z_ref"]) + ta * (g["z_seed"] - g["z_magnet"])
    ys = vy + ty * (g["z_seed"] - zd)
    cols = (xs + 0.1 * randn(NT), ys + 0.1 * randn(NT), ta + 1e-4 * randn(NT), ty + 1e-4 * randn(NT), qop)

    # true hits of the daughters, then noise
    D = 2 * NL
    h_grp, h_u, h_y = [], [], []
    for L in range(4):
        k = torch.arange(D, device=dev)[zd[:D] < zl[L]]
        y = vy[k] + ty[k] * (zl[L] - zd[k])
        h_u.append(x0[k] + tx0[k] * (zl[L] - g["z_ref"]) - y * tana[L] + g["sigma_hit"] * randn(k.numel()))
        h_y.append(y)
        h_grp.append(t_ev[k] * 4 + L)
    if noise is None:
        noise = (int(case["hits"]) - torch.bincount(torch.cat(h_grp), minlength=4 * E)).clamp(min=0)
    n_grp = torch.arange(4 * E, device=dev).repeat_interleave(noise)
    NN = n_grp.numel()
    ny = rand(NN, -700.0, 700.0)
    tan_l = torch.tensor(tana, device=dev, dtype=f64)
    h_u.append(rand(NN, -800.0, 800.0) - ny * tan_l[n_grp % 4])
    h_y.append(ny)
    h_grp.append(n_grp)
    grp, u, y = torch.cat(h_grp), torch.cat(h_u), torch.cat(h_y)
    order = torch.argsort(grp.double() + rand(grp.numel(), 0.0, 1.0))
    grp, u, y = grp[order], u[order], y[order]
    sec = ((y - g["sector_y0"]) / g["sector_h"]).floor().clamp(0, g["n_sectors"] - 1)
    s_order = torch.argsort(t_ev.double() + rand(NT, 0.0, 1.0))
    off = lambda ids, n: torch.cat([torch.zeros(1, device=dev, dtype=torch.long),
                                    torch.bincount(ids, minlength=n).cumsum(0)]).int()
    out = dict(seed_off=off(t_ev, E), hit_off=off(grp, 4 * E), hu=u.float(), hit_sector=sec.to(torch.uint8))
    for k, v in zip(("sx", "sy", "stx", "sty", "sqop"), cols):
        out[k] = v[s_order].float()
    return out


def _batch(inp, E):
    h = {k: v.cpu().numpy() for k, v in inp.items()}
    return synth.EventBatch(E, h["seed_off"], h["sx"], h["sy"], h["stx"], h["sty"], h["sqop"], h["hit_off"], h["hu"],
                            hit_sector=h["hit_sector"])


def _score_max(case, g):
    return math.inf if case["all_pairs"] else g["ghost_threshold"]


def prepare(case, seed):
    E, g = int(case["events"]), _geometry(case)
    batch = _batch(_events(case, seed), E)
    ctx = ds.Context(0, g, synth.mlp_weights())
    autotune.apply_cached(ctx.handle, batch, g["algorithm"])
    bounds = {}
    if case["bounds"]:
        s, h = batch.seeds_per_event(), batch.hits_per_layer().sum(1)
        bounds = dict(max_seeds_per_event=max(512, int(s.max())), max_hits_per_event=max(8192, int(h.max())))
    st = dict(case=case, ctx=ctx, ev=ds.DeviceEvents(batch, **bounds), score_max=_score_max(case, g),
              mode=ds.DS_MODE_GRAPH if case["mode"] == "graph" else ds.DS_MODE_PERSISTENT)
    if case["call"] == "candidates":
        st["rows"] = ds.DeviceCandidates(batch.n_seeds, ds.ds_candidate_slots(ctx.handle))
        return st
    if case["extras"]:
        ds.ds_load_lines(ctx.handle, synth.line_weights())
    st["trk"] = ds.DeviceTracks(batch.n_seeds, with_cand=bool(case["cand"]))
    st["vtx"] = ds.DeviceVertices(E, int(case["cap"]), extras=bool(case["extras"]))
    return st


def run(st):
    case, ctx, ev = st["case"], st["ctx"].handle, st["ev"]
    if case["call"] == "candidates":
        r = st["rows"]
        ds.ds_score_candidates(ctx, ev, r)
        out = {k: getattr(r, k) for k in ("seed", "cand", "nhits", "hits", "x", "y", "tx", "ty", "qop", "chi2", "score")}
        return dict(out, flags=r.flags)
    t, v = st["trk"], st["vtx"]
    if case["call"] == "process":
        ds.ds_process(ctx, ev, t, v, st["mode"], score_max=st["score_max"])
    elif case["call"] == "static":
        ds.ds_process_static(ctx, ev, t, v, score_max=st["score_max"])
    else:
        ds.ds_find_tracks(ctx, ev, t, st["mode"], 0)
        ds.ds_ghost_kill(ctx, ev, t)
        ds.ds_vertex(ctx, ev, t, st["score_max"], v, st["mode"])
    trk = {k: getattr(t, k) for k in ("x", "y", "tx", "ty", "qop", "chi2", "score", "hits", "nhits", "flags")}
    vtx = {k: getattr(v, k) for k in ("count", "i", "j", "x", "y", "z", "doca", "flags")}
    if case["cand"]:
        trk["cand"] = t.cand
    if case["extras"]:
        vtx.update(m_pipi=v.m_pipi, m_ppi=v.m_ppi, lines=v.lines)
    return dict(trk=trk, vtx=vtx)


def work(case):
    """Inputs read once, outputs written once; the arithmetic of the method on
    the mean occupancy (windows' contents from the hit density)."""
    E, s, h = case["events"], case["seeds"], case["hits"]
    S, H = E * s, 4.0 * E * h
    dens = h / U_RANGE
    items = min(10.0, dens * (200.0 if case["loose"] else 6.3) + 0.3)
    if case["algorithm"] == 1:
        items = 1.5 * h / 14.0 * min(1.0, 1.2 * dens / 14.0 * 1.5) + 0.3
    read = 20.0 * S + 4.0 * H + 20.0 * E + (H if case["algorithm"] == 1 else 0.0)
    fits = 156.0 * items * S   # three projections and up to four straight-line fits per UTbX hit
    if case["call"] == "candidates":
        rows = S * min(SLOTS, items * max(1.0, min(4.0, (dens * (20.0 if case["loose"] else 1.1)) ** 2)))
        return dict(bytes=read + 4.0 * S * SLOTS + 56.0 * rows, flops=60.0 * S + fits + 2144.0 * rows)
    found = 0.9 * S
    kept = 0.9 * s if case["all_pairs"] else 0.05 * s
    pairs = E * kept * kept / 4.0
    vert = min(E * case["cap"], 0.03 * pairs)
    out = (52.0 if case["cand"] else 48.0) * S + 4.0 * E + (48.0 if case["extras"] else 24.0) * vert
    flops = 60.0 * S + fits + 2144.0 * found + 17.0 * pairs + (250.0 + (3700.0 if case["extras"] else 0.0)) * vert
    return dict(bytes=read + out, flops=flops)


# ------------------------------------------------------------ float64 reference

def _near(run_key, us, want, m, W, n):
    """The n closest of the sorted hits of run `want` within W of m: distances
    (inf: none), u and sorted position, [items, n] each.  run_key[k] is the run
    of sorted hit k, us its u; hits of a run are contiguous and ascending."""
    big, H = 1e5, us.numel()
    pos = torch.searchsorted(run_key.double() * big + us, want.double() * big + m)
    k = pos[:, None] + torch.arange(-(n + 1), n + 1, device=pos.device)[None, :]
    inb = (k >= 0) & (k < H)
    k = k.clamp(0, max(H - 1, 0))
    u = us[k]
    d = (u - m[:, None]).abs()
    d = torch.where(inb & (run_key[k] == want[:, None]) & (d <= W[:, None]), d, math.inf)
    d, o = torch.sort(d, dim=1, stable=True)
    return d[:, :n], torch.gather(u, 1, o)[:, :n], torch.gather(k, 1, o)[:, :n]


def _candidates(case, g, inp):
    """Every (seed, UTbX hit) item's candidates, generated in blocks of events:
    seed index, rank of the UTbX hit, option indices, hit count, chi2,
    intercept, slope and the four u (nan: no hit), one row per candidate."""
    dev, f64 = inp["hu"].device, torch.float64
    zl, tana = (torch.tensor(g[k], device=dev, dtype=f64) for k in ("z_layer", "tan_stereo"))
    dv1 = g["algorithm"] == 1 and case["call"] != "candidates"
    nsec = int(g["n_sectors"]) if dv1 else 1
    so, ho = inp["seed_off"].long(), inp["hit_off"].long()
    E = so.numel() - 1
    block = max(1, min(E, int(3e8 / max(1.0, case["seeds"] * (case["hits"] / 6.0 if dv1 else 60.0) * 12))))
    zm, zs, z3 = g["z_magnet"], g["z_seed"], zl[3]
    for e0 in range(0, E, block):
        e1 = min(E, e0 + block)
        sa, sb, ha, hb = int(so[e0]), int(so[e1]), int(ho[4 * e0]), int(ho[4 * e1])
        if sa == sb or ha == hb:
            continue
        run_of = torch.arange(4 * (e1 - e0), device=dev).repeat_interleave(ho[4 * e0 + 1:4 * e1 + 1] - ho[4 * e0:4 * e1])
        key = run_of * nsec + (inp["hit_sector"][ha:hb].long() if dv1 else 0)
        u = inp["hu"][ha:hb].double()
        o = torch.argsort(u, stable=True)
        o = o[torch.argsort(key[o], stable=True)]
        us, ks = u[o], key[o]
        start = torch.cat([torch.zeros(1, device=dev, dtype=torch.long),
                           torch.bincount(ks, minlength=4 * (e1 - e0) * nsec).cumsum(0)])
        ev = torch.arange(e1 - e0, device=dev).repeat_interleave(so[e0 + 1:e1 + 1] - so[e0:e1])
        sx, sy, stx, sty, q = (inp[k][sa:sb].double() for k in ("sx", "sy", "stx", "sty", "sqop"))
        yl = sy[:, None] + sty[:, None] * (zl - zs)[None, :]
        c = sx[:, None] + stx[:, None] * (zl - zs)[None, :] - yl * tana[None, :]
        if dv1:
            klo = ((yl - g["sector_tol"] - g["sector_y0"]) / g["sector_h"]).floor()
            khi = ((yl + g["sector_tol"] - g["sector_y0"]) / g["sector_h"]).floor()
            none = (khi < 0) | (klo > nsec - 1)
            klo, khi = klo.clamp(0, nsec - 1).long(), khi.clamp(0, nsec - 1).long()
            khi = torch.where(none, klo - 1, khi)
            r0 = (ev * 4 + 3) * nsec
            first, last = start[r0 + klo[:, 3]], start[r0 + khi[:, 3] + 1]
            n_it = (last - first).clamp(min=0)
            s_i = torch.arange(sb - sa, device=dev).repeat_interleave(n_it)
            base = n_it.cumsum(0) - n_it
            u3 = us[first[s_i] + torch.arange(s_i.numel(), device=dev) - base[s_i]]
            rank = torch.zeros_like(s_i)
        else:
            W1 = g["w1_c0"] + g["w1_c1"] * q.abs()
            m3 = c[:, 3] + g["polarity"] * g["kick"] * q * (zm - z3)
            n3 = int(g["max_l3"])
            d, uu, _ = _near(ks, us, ev * 4 + 3, m3, W1, n3)
            s_i, rank = torch.nonzero(torch.isfinite(d), as_tuple=True)
            u3 = uu[s_i, rank]
        opt = []
        for L in range(3):
            n = int(g["n_closest"][L])
            m = c[s_i, L] + (u3 - c[s_i, 3]) * (zm - zl[L]) / (zm - z3)
            W = (g["w2_c0"] + g["w2_c1"] * q.abs())[s_i]
            want = (ev[s_i] * 4 + L) * nsec
            if dv1:
                da, ua, _ = _near(ks, us, want + klo[s_i, L], m, W, n)
                db, ub, _ = _near(ks, us, want + klo[s_i, L] + 1, m, W, n)
                da = torch.where((khi[s_i, L] >= klo[s_i, L])[:, None], da, math.inf)
                db = torch.where((khi[s_i, L] > klo[s_i, L])[:, None], db, math.inf)
                d, od = torch.sort(torch.cat([da, db], 1), dim=1, stable=True)
                uu = torch.gather(torch.cat([ua, ub], 1), 1, od)
                d, uu = d[:, :n], uu[:, :n]
                if L == 0:   # the axial triplet
                    k = torch.isfinite(d[:, 0])
                    s_i, rank, u3, d, uu = s_i[k], rank[k], u3[k], d[k], uu[k]
            else:
                d, uu, _ = _near(ks, us, want, m, W, n)
            opt.append(torch.where(torch.isfinite(d), uu, math.nan))
        for i0 in range(opt[0].shape[1]):
            for i1 in range(opt[1].shape[1]):
                for i2 in range(opt[2].shape[1]):
                    idx = (i0, i1, i2)
                    uh = torch.stack([opt[0][:, i0], opt[1][:, i1], opt[2][:, i2], u3], 1)
                    has = torch.isfinite(uh)
                    ok = has.sum(1) >= 3
                    ok &= has[:, 0] | has[:, 1]
                    for L in range(3):   # option 0 of an empty layer stands for "no hit"
                        if idx[L] > 0:
                            ok &= has[:, L]
                    k = torch.nonzero(ok)[:, 0]
                    if k.numel() == 0:
                        continue
                    h, s = has[k].double(), s_i[k]
                    rho = torch.where(has[k], uh[k] - c[s], 0.0)
                    dz = (zl - g["z_ref"])[None, :] * h
                    n, sz, szz = h.sum(1), dz.sum(1), (dz * dz).sum(1)
                    sr, szr = rho.sum(1), (dz * rho).sum(1)
                    be = (n * szr - sz * sr) / (n * szz - sz * sz)
                    al = (sr - be * sz) / n
                    res = (rho - al[:, None] - be[:, None] * dz) * h
                    chi2 = (res * res).sum(1) / g["sigma_hit"] ** 2
                    slot = ((rank[k] * opt[0].shape[1] + i0) * opt[1].shape[1] + i1) * opt[2].shape[1] + i2
                    yield sa + s, slot, n, chi2, al, be, uh[k]


def _track(g, inp, s, n, chi2, al, be, uh, W):
    """Track values of fitted candidates in float64, and the score of the network
    on the float32 track that is stored (the network's inputs by definition)."""
    dev, f64 = al.device, torch.float64
    zl, tana = (torch.tensor(g[k], device=dev, dtype=f64) for k in ("z_layer", "tan_stereo"))
    sx, sy, stx, sty, q = (inp[k].double()[s] for k in ("sx", "sy", "stx", "sty", "sqop"))
    dz = g["z_ref"] - g["z_seed"]
    mk = g["polarity"] * g["kick"]
    t = dict(x=sx + stx * dz + al, y=sy + sty * dz, tx=stx + be, ty=sty, qop=-be / mk, chi2=chi2)
    r = {k: v.float().double() for k, v in t.items()}
    yl = r["y"][:, None] + r["ty"][:, None] * (zl - g["z_ref"])[None, :]
    res = uh + yl * tana[None, :] - r["x"][:, None] - r["tx"][:, None] * (zl - g["z_ref"])[None, :]
    res = torch.where(torch.isfinite(uh), res / (5.0 * g["sigma_hit"]), 0.0)
    xm = r["x"] + r["tx"] * (g["z_magnet"] - g["z_ref"]) - sx - stx * (g["z_magnet"] - g["z_seed"])
    f = torch.stack([r["x"] / 1000, r["y"] / 1000, r["tx"] / 0.3, r["ty"] / 0.3, r["qop"] * 2, r["chi2"] / 10,
                     (n - 3.5) * 2, sx / 3000, sy / 3000, stx * 2, sty * 2, q * 2, res[:, 0], res[:, 1], res[:, 2],
                     res[:, 3], xm], 1)
    w = torch.as_tensor(W, device=dev).double()
    W1, b1, W2, b2, W3, b3 = torch.split(w, [544, 32, 512, 16, 16, 1])
    h = torch.relu(f @ W1.view(32, 17).T + b1)
    h = torch.relu(h @ W2.view(16, 32).T + b2)
    t["score"] = torch.sigmoid(h @ W3 + b3)
    return t


def _clones(so, hits, chi2, found):
    """Tracks killed by a better one of their event that shares more than two hits."""
    dead = torch.zeros_like(found)
    S = found.numel()
    n = torch.isfinite(hits).sum(1)
    ev = torch.arange(so.numel() - 1, device=so.device).repeat_interleave(so[1:] - so[:-1])
    step = max(1, int(3e7 / max(1, int((so[1:] - so[:-1]).max()))))
    slot = torch.arange(S, device=so.device)
    for a in range(0, S, step):
        i = slot[a:a + step][found[a:a + step]]
        if i.numel() == 0:
            continue
        cnt = so[ev[i] + 1] - so[ev[i]]
        ii = i.repeat_interleave(cnt)
        jj = so[ev[ii]] + torch.arange(ii.numel(), device=so.device) - (cnt.cumsum(0) - cnt).repeat_interleave(cnt)
        k = found[jj] & (ii != jj)
        ii, jj = ii[k], jj[k]
        k = (hits[ii] == hits[jj]).sum(1) > 2
        ii, jj = ii[k], jj[k]
        better = (n[jj] > n[ii]) | ((n[jj] == n[ii]) & ((chi2[jj] < chi2[ii]) | ((chi2[jj] == chi2[ii]) & (jj < ii))))
        dead[ii[better]] = True
    return dead


def _vertices(case, g, inp, t, keep, cap):
    """Opposite-charge pairs of the kept tracks: point of closest approach after
    three Newton steps from the straight-line start, in (i, j) order."""
    dev, f64 = keep.device, torch.float64
    so = inp["seed_off"].long()
    E = so.numel() - 1
    M = E * cap
    v = {k: torch.zeros(M, device=dev, dtype=f64) for k in ("x", "y", "z", "doca")}
    if case["extras"]:
        v.update(m_pipi=torch.zeros(M, device=dev, dtype=f64), m_ppi=torch.zeros(M, device=dev, dtype=f64),
                 lines=torch.zeros((4, M), device=dev, dtype=f64))
    r = {k: t[k].float().double() for k in ("x", "y", "tx", "ty", "qop")}
    sq = inp["sqop"].double()
    ev_of = torch.arange(E, device=dev).repeat_interleave(so[1:] - so[:-1])
    per = max(1, int(2e7 / max(1, int(((so[1:] - so[:-1]).double() ** 2).mean()) + 1)))
    for e0 in range(0, E, per):
        e1 = min(E, e0 + per)
        s = torch.nonzero(keep[so[e0]:so[e1]])[:, 0] + so[e0]
        if s.numel() < 2:
            continue
        ev = ev_of[s] - e0
        cnt = torch.bincount(ev, minlength=e1 - e0)
        end = cnt.cumsum(0)[ev]
        here = torch.arange(s.numel(), device=dev)
        n = end - here - 1
        a = here.repeat_interleave(n)
        b = torch.arange(a.numel(), device=dev) - (n.cumsum(0) - n)[a] + a + 1
        k = (sq[s[a]] > 0) != (sq[s[b]] > 0)
        a, b = s[a[k]], s[b[k]]
        x1, y1, u1, w1 = (r[k][a] for k in ("x", "y", "tx", "ty"))
        x2, y2, u2, w2 = (r[k][b] for k in ("x", "y", "tx", "ty"))
        g1, g2 = _gamma(g, r["qop"][a]), _gamma(g, r["qop"][b])
        wx, wy = x1 - x2, y1 - y2
        nx, ny, nz = w1 - w2, u2 - u1, u1 * w2 - w1 * u2
        nn = nx * nx + ny * ny + nz * nz
        ok = nn >= 1e-12
        base = wy * nx - wx * ny
        p = -(base + (wx * w2 - wy * u2) * nz) / nn
        q = -(base + (wx * w1 - wy * u1) * nz) / nn
        for _ in range(int(g["newton_iters"])):
            Dx = x1 + u1 * p + g1 * p * p - x2 - u2 * q - g2 * q * q
            Dy, Dz = y1 + w1 * p - y2 - w2 * q, p - q
            a1, a2 = u1 + 2 * g1 * p, u2 + 2 * g2 * q
            f1, f2 = Dx * a1 + Dy * w1 + Dz, -(Dx * a2 + Dy * w2 + Dz)
            h11, h22 = a1 * a1 + w1 * w1 + 1 + 2 * g1 * Dx, a2 * a2 + w2 * w2 + 1 - 2 * g2 * Dx
            h12 = -(a1 * a2 + w1 * w2 + 1)
            det = h11 * h22 - h12 * h12
            ok &= det.abs() >= 1e-12 * (h11 + h22) ** 2
            p, q = p - (h22 * f1 - h12 * f2) / det, q - (h11 * f2 - h12 * f1) / det
        X1, X2, Y1, Y2 = x1 + u1 * p + g1 * p * p, x2 + u2 * q + g2 * q * q, y1 + w1 * p, y2 + w2 * q
        doca = ((X1 - X2) ** 2 + (Y1 - Y2) ** 2 + (p - q) ** 2).sqrt()
        k = torch.nonzero(ok & (doca < g["doca_max"]))[:, 0]
        ek = ev_of[a[k]]
        nk = torch.bincount(ek, minlength=E)
        at = torch.arange(k.numel(), device=dev) - (nk.cumsum(0) - nk)[ek]
        k, at, ek = k[at < cap], at[at < cap], ek[at < cap]
        o = ek * cap + at
        out = dict(x=0.5 * (X1 + X2)[k], y=0.5 * (Y1 + Y2)[k], z=g["z_ref"] + 0.5 * (p + q)[k], doca=doca[k])
        if case["extras"]:
            out.update(_extras(sq[a[k]], sq[b[k]], (u1 + 2 * g1 * p)[k], w1[k], (u2 + 2 * g2 * q)[k], w2[k], out))
        for name, val in out.items():
            v[name][..., o] = val
    return v


def _extras(q1, q2, d1x, d1y, d2x, d2y, v):
    mpi, mpr = 0.13957039, 0.93827209
    p1, p2 = 1 / q1.abs(), 1 / q2.abs()
    k1, k2 = p1 / (d1x ** 2 + d1y ** 2 + 1).sqrt(), p2 / (d2x ** 2 + d2y ** 2 + 1).sqrt()
    Sx, Sy, Sz = k1 * d1x + k2 * d2x, k1 * d1y + k2 * d2y, k1 + k2
    ss = Sx ** 2 + Sy ** 2 + Sz ** 2
    en = lambda p, m: (p ** 2 + m ** 2).sqrt()
    pipi = 1000 * ((en(p1, mpi) + en(p2, mpi)) ** 2 - ss).clamp(min=0).sqrt()
    ep = torch.where(p1 >= p2, en(p1, mpr) + en(p2, mpi), en(p2, mpr) + en(p1, mpi))
    ppi = 1000 * (ep ** 2 - ss).clamp(min=0).sqrt()
    f = torch.stack([p1.log(), p2.log(), d1x / 0.3, d1y / 0.3, d2x / 0.3, d2y / 0.3, v["z"] / 1000,
                     (v["x"] ** 2 + v["y"] ** 2).sqrt() / 100, v["doca"], (pipi - 497.6) / 100, (ppi - 1115.7) / 100,
                     (Sx ** 2 + Sy ** 2).sqrt()], 1)
    w = torch.as_tensor(synth.line_weights(), device=f.device).double().view(4, 449)
    lines = [torch.sigmoid(torch.relu(f @ k[:384].view(32, 12).T + k[384:416]) @ k[416:448] + k[448]) for k in w]
    return dict(m_pipi=pipi, m_ppi=ppi, lines=torch.stack(lines))


def exact(case, seed):
    g, E = _geometry(case), int(case["events"])
    inp = _events(case, seed)
    dev, f64 = inp["hu"].device, torch.float64
    S = inp["sx"].numel()
    W = synth.mlp_weights()
    names = ("x", "y", "tx", "ty", "qop", "chi2", "score")
    if case["call"] == "candidates":
        rows = {k: torch.zeros(max(S * SLOTS, 1), device=dev, dtype=f64) for k in names}
        for s, slot, n, chi2, al, be, uh in _candidates(case, g, inp):
            t = _track(g, inp, s, n, chi2, al, be, uh, W)
            for k in names:
                rows[k][s * SLOTS + slot] = t[k]
        return dict(rows, seed=None, cand=None, nhits=None, hits=None, flags=None)
    # the best candidate of each seed: more hits, then lower chi2, then the first
    best_n = torch.zeros(S, device=dev, dtype=f64)
    best_c, best_a, best_b = (torch.full((S,), math.inf, device=dev, dtype=f64) for _ in range(3))
    best_u = torch.full((S, 4), math.nan, device=dev, dtype=f64)
    for s, slot, n, chi2, al, be, uh in _candidates(case, g, inp):
        top = torch.zeros(S, device=dev, dtype=f64).scatter_reduce_(0, s, n, "amax")
        low = torch.full((S,), math.inf, device=dev, dtype=f64)
        low.scatter_reduce_(0, s, torch.where(n == top[s], chi2, math.inf), "amin")
        k = torch.nonzero((n == top[s]) & (chi2 == low[s]))[:, 0]
        k = k[(n[k] > best_n[s[k]]) | ((n[k] == best_n[s[k]]) & (chi2[k] < best_c[s[k]]))]
        best_n[s[k]], best_c[s[k]], best_a[s[k]], best_b[s[k]], best_u[s[k]] = n[k], chi2[k], al[k], be[k], uh[k]
    found = best_n > 0
    if case["clone"]:
        found = found & ~_clones(inp["seed_off"].long(), best_u, best_c.float(), found)
    s = torch.nonzero(found)[:, 0]
    full = {k: torch.zeros(max(S, 1), device=dev, dtype=f64) for k in names}
    for a in range(0, s.numel(), 1 << 20):
        k = s[a:a + (1 << 20)]
        for name, val in _track(g, inp, k, best_n[k], best_c[k], best_a[k], best_b[k], best_u[k], W).items():
            full[name][k] = val
    keep = found & (full["score"][:S] < _score_max(case, g))
    vtx = _vertices(case, g, inp, full, keep, int(case["cap"]))
    trk = dict(full, hits=None, nhits=None, flags=None)
    if case["cand"]:
        trk["cand"] = None
    return dict(trk=trk, vtx=dict(vtx, count=None, i=None, j=None, flags=None))
