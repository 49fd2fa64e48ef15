"""The way out of results: one launch writes every field of a batch's rows
into page-locked arrays directly, and into ordinary arrays through a ring of
page-locked slots.  Every route must give the bytes of every other one, and
the hit lists of the oracle."""
import ctypes as C

import numpy as np
import pytest

from paper_1702_06359_amd import abi, synth

pytestmark = pytest.mark.gpu
FIELDS = ("par", "cov", "hits", "n_hits", "n_holes", "chi2", "ndof", "status")


def _pinned(shape, dtype):
    import torch
    return torch.zeros(shape, dtype=torch.float64 if dtype == np.float64 else torch.int32, pin_memory=True).numpy()


def _shifted(shape, dtype):
    """Page-locked doubles that start four bytes off their alignment: they have to go through the staging."""
    if dtype != np.float64:
        return _pinned(shape, dtype)
    n = int(np.prod(shape))
    return _pinned((2 * n + 1,), np.int32)[1:].view(np.float64).reshape(shape)


def _equal(got, want):
    for f in FIELDS:
        np.testing.assert_array_equal(getattr(got, f), getattr(want, f), err_msg=f)


# rows at the edges of a tile (64), more events than one launch takes (32), more tiles than it has blocks for one
# wavefront each (256), and more staged bytes than the ring holds (16 MiB; 288 a row)
@pytest.mark.parametrize("sizes", [(1,), (63, 64, 65), (5,) * 33 + (130,), (16384,), (16385, 1), (30000, 40000)])
def test_every_route_gives_the_same_rows(sizes):
    print("case delivery", sizes, flush=True)
    evs = [synth.make_event(n, cfg=31, event=i, noise=0.1) for i, n in enumerate(sizes)]
    with abi.Context(abi.config_from_geometry(synth.Geometry(), max_cands=2)) as ctx:
        hs = ctx.load_events([abi.EventArrays.from_synth(e) for e in evs])

        def outs(empty):
            return [abi.TrackArrays(n, 10, empty=empty) for n in sizes]

        plain, pinned, shifted = outs(None), outs(_pinned), outs(_shifted)
        for o in (plain, pinned, shifted):
            ctx.build_batch(hs, outs=o)
        for a, b, c in zip(plain, pinned, shifted):
            _equal(b, a)
            _equal(c, a)
        for h, a in zip(hs[:3], plain):   # on request, later; a few fields only
            _equal(abi_rows(ctx.fetch_tracks(h, a.n)), a)
            some = abi.TrackArrays(a.n, 10, empty=_pinned)
            some.tracks.par = some.tracks.cov = some.tracks.ndof = None
            abi.check(abi.lib().mkf_fetch_tracks(ctx.h, h, C.byref(some.tracks)))
            for f in FIELDS:
                want = 0 if f in ("par", "cov", "ndof") else getattr(a, f)
                np.testing.assert_array_equal(getattr(some, f), np.broadcast_to(want, getattr(some, f).shape))
    for e, a in zip(evs[:3], plain):
        np.testing.assert_array_equal(a.hits[:, :3], e.seed_hits)
        np.testing.assert_array_equal(a.n_hits, (a.hits >= 0).sum(axis=1))
        np.testing.assert_array_equal(a.ndof, 2 * a.n_hits - 5)


class abi_rows:
    def __init__(self, d):
        self.__dict__.update(d)


@pytest.mark.parametrize("n_layers", [4, 5, 10, 16])
def test_fit_rows_at_every_layer_count(n_layers):
    """The fit stages its result rows where its priors and hit lists were: from four layers (less room than the rows
    take) to sixteen, against the oracle; 200 tracks cross wavefronts and end within one."""
    import oracle
    print("case fit rows", n_layers, flush=True)
    g = synth.Geometry(n_layers=n_layers, radii=tuple(4.0 * (i + 1) for i in range(n_layers)),
                       x0=(0.002,) * n_layers)
    ev = synth.make_event(200, cfg=32, event=n_layers, noise=0.1, geometry=g, pt_range=(1.0, 10.0))
    with abi.Context(abi.config_from_geometry(g, max_cands=2)) as ctx:
        h = ctx.load_event(ev)
        got = ctx.fit_batch([h], [ev.n_seeds])[0]
    ref = oracle.fit(oracle.config(g, max_cands=2), ev.hits, ev.prior_par, ev.prior_cov, ev.truth_hit)
    np.testing.assert_array_equal(got["hits"], ev.truth_hit)
    np.testing.assert_array_equal(got["status"], ref["status"])
    np.testing.assert_array_equal(got["n_hits"] + got["n_holes"], n_layers)
    np.testing.assert_array_equal(got["ndof"], 2 * got["n_hits"] - 5)
    # FP32 over at most 16 layers of about 10^3 roundings of 6e-8 each, adding as their square root; chi2 by
    # differences of positions of 50 cm against 0.01 cm errors: 50 / 0.01 * 6e-8 of a sigma per hit
    np.testing.assert_allclose(got["chi2"], ref["chi2"], rtol=3e-3, atol=3e-3)
    np.testing.assert_allclose(got["par"][:, :3], ref["par"][:, :3], rtol=0, atol=3e-4)


# batches large enough to be built in parts, each delivered by the next part's launch: every lane count (seeds per
# item), blocks of several wavefronts, four layers (a build's LDS below a delivery's), disks, deep layers, and events
# that end within a block of 10,240 rows
@pytest.mark.parametrize("cands,waves,layers,kind", [(6, 1, 10, "barrel"), (8, 2, 10, "barrel"), (1, 4, 4, "barrel"),
                                                     (4, 1, 4, "barrel"), (2, 1, 10, "endcap"), (6, 1, 10, "thick")])
def test_a_build_in_parts_is_the_build_in_one(cands, waves, layers, kind):
    g = synth.Geometry.endcap(layers) if kind == "endcap" else synth.Geometry(
        n_layers=layers, radii=tuple(4.0 * (i + 1) for i in range(layers)), x0=(0.002,) * layers,
        thickness=(0.6,) * layers if kind == "thick" else None)
    sizes = (20481, 1, 30007, 10240)
    print("case parts", cands, waves, layers, kind, flush=True)
    evs = [synth.make_event(n, cfg=33, event=i, noise=0.1, geometry=g) for i, n in enumerate(sizes)]
    with abi.Context(abi.config_from_geometry(g, max_cands=cands)) as ctx:
        ctx.set_tuning(waves_per_block=waves)
        hs = ctx.load_events([abi.EventArrays.from_synth(e) for e in evs])
        one = [abi.TrackArrays(n, layers) for n in sizes]
        ctx.build_batch(hs, flags=abi.BATCH_ASYNC)   # one launch
        for h, o in zip(hs, one):
            abi.check(abi.lib().mkf_fetch_tracks(ctx.h, h, C.byref(o.tracks)))
        for empty in (_pinned, None):
            for _ in range(2):
                parts = [abi.TrackArrays(n, layers, empty=empty) for n in sizes]
                ctx.build_batch(hs, flags=abi.BATCH_REINDEX, outs=parts)
                for a, b in zip(parts, one):
                    _equal(a, b)
