"""Events and settings at the limits of what the kernels list and sort in LDS:
layers dense enough for more than 128 hits in a seed's sectors, seeds with
more hits than are listed, crowded bins, and the sizes at which calls are
refused."""
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
