"""Host-only checks of the launch autotuner: the workload signature and the
committed cache of launch settings (the settings the benchmark and the
request loop apply), without a GPU."""
import json
import re

import numpy as np

from paper_2503_13092_amd import autotune, ds, synth


def test_signature_buckets_sizes_by_powers_of_two():
    b = synth.generate(0)   # 100 events x 20 seeds, about 2 000 hits per event
    sig = autotune.signature(b)
    assert re.fullmatch(r"E\d+-S\d+:\d+-H\d+:\d+", sig)
    assert sig.startswith("E7-")          # log2(100) = 6.6 -> 7
    s = np.diff(b.seed_off)
    assert f"-S{round(np.log2(s.mean()))}:{round(np.log2(s.max()))}-" in sig
    # the signature depends on sizes only, not on the values
    b2 = synth.generate(0, seed=99)
    assert autotune.signature(b2) == sig


def test_committed_cache_entries_are_valid_launch_settings():
    cache = autotune.load_cache()
    assert cache, "the package ships a tuned cache"
    for key, entry in cache.items():
        dev, alg, sig = key.split("|")
        assert re.fullmatch(r"gfx\d+-\d+cu", dev), key
        assert alg in ("alg0", "alg1"), key
        assert re.fullmatch(r"E\d+-S\d+:\d+-H\d+:\d+", sig), key
        best = entry["best"]
        assert best["block"] in autotune.SPACE["block"]
        assert best["wg_per_cu"] in autotune.SPACE["wg_per_cu"]
        assert best["bins"] in autotune.SPACE["bins"]
        assert best["order"] in (ds.DS_ORDER_INPUT, ds.DS_ORDER_LARGEST_FIRST)
        assert best["fused"] in (0, 1)
        v = best.get("vertex")
        if v:
            assert v["block"] in autotune.VERTEX_SPACE["block"]
            assert v["wg_per_cu"] in autotune.VERTEX_SPACE["wg_per_cu"]
        # the chosen point was confirmed no slower than the library default
        assert entry["ms"] <= entry["default_ms"] * 1.02
    json.dumps(cache)


def test_benchmark_workloads_have_cache_entries():
    """The three benchmark workloads (throughput, uneven, stress) and the Dv1
    throughput line find their tuned settings by signature."""
    cache = autotune.load_cache()
    sigs = {k.split("|", 1)[1] for k in cache}
    for config, alg in ((1, 0), (2, 0), (4, 0), (1, 1)):
        b = synth.generate(config)
        assert f"alg{alg}|{autotune.signature(b)}" in sigs, (config, alg)


class FakeLibrary:
    """The launch settings of a context as the library keeps them, and step
    times by the settings in force."""

    def __init__(self, ms):
        self.ms, self.launch, self.order, self.fused = ms, {0: [0, 0, 0], 1: [0, 0, 0]}, 0, 1

    def patch(self, monkeypatch):
        for name in ("ds_set_launch", "ds_set_event_order", "ds_set_step_fusion", "ds_process", "ds_vertex"):
            monkeypatch.setattr(ds, name, getattr(self, name))
        monkeypatch.setattr(ds, "ds_reset_launch", self.ds_reset_launch, raising=False)
        monkeypatch.setattr(autotune, "_time", lambda fn, stream, reps: self.ms(self))
        monkeypatch.setattr(autotune, "device_name", lambda: "gfx000-0cu")

    def ds_reset_launch(self, ctx, kernel):
        self.launch[kernel] = [0, 0, 0]

    def ds_set_launch(self, ctx, kernel, block=0, wg_per_cu=0, bins=0):
        self.launch[kernel] = [n or o for n, o in zip((block, wg_per_cu, bins), self.launch[kernel])]

    def ds_set_event_order(self, ctx, order):
        self.order = order

    def ds_set_step_fusion(self, ctx, fused):
        self.fused = fused

    def ds_process(self, *a, **k):
        pass

    ds_vertex = ds_process


def test_a_point_left_to_the_library_is_set_after_any_other(monkeypatch):
    """Cached points of several workloads applied to one context in turn:
    what a point leaves to the library is not what the last one had set."""
    lib = FakeLibrary(lambda l: 1.0)
    lib.patch(monkeypatch)
    autotune.set_point(None, dict(block=256, wg_per_cu=4, bins=512, order=0))
    autotune.set_point(None, dict(block=0, wg_per_cu=0, bins=1024, order=1))
    assert lib.launch[0] == [0, 0, 1024]


def test_the_library_s_own_choice_is_confirmed_like_any_point(monkeypatch):
    """The fastest point, left to the library, is timed again among the last
    candidates and is what the context is left with."""
    import contextlib
    import torch
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: contextlib.nullcontext())
    timed = []

    def ms(lib):
        timed.append(tuple(lib.launch[0]))
        return 1.0 if lib.launch[0][0] == 0 and lib.order == 1 else 2.0

    lib = FakeLibrary(ms)
    lib.patch(monkeypatch)
    b = synth.generate(0, n_events=4)
    e = autotune.autotune(None, b, None, None, None, 0.5, path=None, log=None)
    assert e["best"]["block"] == 0 and e["best"]["order"] == 1 and e["ms"] == 1.0
    assert lib.launch[0][:2] == [0, 0] and lib.order == 1
    assert any(t[0] == 0 for t in timed[-3:])   # (winner, winner unfused, fixed settings)
