"""What is taken where device memory is short: an event whose index has no room
for the working arrays of the bucketed form is indexed without them, layers
whose counters exceed a block's LDS included, and a served event is admitted
to a budget that holds its inputs, its results in the caller's types, a hit
index and nothing more."""
import contextlib

import numpy as np
import pytest

from paper_1702_06359_amd import abi, synth
from test_gpu_index import check_layer, edge_tolerance, host_bins

pytestmark = pytest.mark.gpu

FIELDS = ("par", "cov", "hits", "n_hits", "n_holes", "chi2", "status", "ndof")


class Capped:
    """Device memory from torch's allocator, refused beyond `cap` bytes in all."""

    def __init__(self, cap=None):
        import torch
        self.cap, self.sizes, self.held = cap, [], {}
        dev = torch.cuda.current_device()
        self.stream = torch.cuda.current_stream(dev).cuda_stream

        def alloc(n, stream, user):
            if self.cap is not None and sum(self.held.values()) + n > self.cap:
                return None
            p = torch.cuda.caching_allocator_alloc(int(n), dev, int(stream or 0))
            self.held[p] = int(n)
            self.sizes.append(int(n))
            return p

        def free(p, stream, user):
            if self.held.pop(int(p), None) is not None:
                torch.cuda.caching_allocator_delete(int(p))

        self.keep = (abi.ALLOC_FN(alloc), abi.FREE_FN(free))
        self.hooks = abi.Allocator()
        self.hooks.alloc, self.hooks.free = self.keep
        self.hooks.user = None


@contextlib.contextmanager
def context(config, memory, monkeypatch, **tuning):
    monkeypatch.setattr(abi, "_torch_hooks", lambda: (memory.hooks, memory.stream, memory.keep))
    with abi.Context(config) as c:
        c.set_tuning(**tuning)
        yield c


# grids and fullest layers: counters that fit a block's LDS (16 and 32 bits wide), and ones that take two, several and
# 32 ranges of it, the last of them ragged
@pytest.mark.parametrize("bins_phi,bins_z,noise", [(2048, 32, 20.0), (1024, 16, 135.0), (2048, 32, 135.0),
                                                   (2047, 51, 135.0), (1024, 1024, 20.0)])
def test_an_index_without_working_arrays(gpu_required, monkeypatch, bins_phi, bins_z, noise):
    print("case index memory", bins_phi, bins_z, noise, flush=True)
    ev = synth.make_event(500, cfg=38, event=1, noise=noise)
    cfg = abi.config_from_geometry(ev.geometry, max_cands=2)
    grid = dict(bins_phi=bins_phi, bins_z=bins_z)
    roomy = Capped()
    with context(cfg, roomy, monkeypatch, **grid) as c:
        h = c.load_event(abi.EventArrays.from_synth(ev))
        want = c.build_batch([h], [500])[0]
        bp, bz = c.index_grid(h)
    data, index = roomy.sizes[:2]
    hits = sum(len(x) for x in ev.hits)
    offsets = 4 * 10 * ((bp * bz + 4) & ~3)
    assert index > offsets + 20 * hits          # the working arrays were there
    tight = Capped(data + offsets + 4 * hits + (64 << 10))
    with context(cfg, tight, monkeypatch, **grid) as c:
        h = c.load_event(abi.EventArrays.from_synth(ev))
        assert tight.sizes[1] < offsets + 256
        for L in range(10):
            off, bin_of, order = c.fetch_index(h, L, len(ev.hits[L]))
            ref, edge = host_bins(ev.hits[L], L, ev.geometry, bp, bz)
            check_layer(off, bin_of, order, ref, edge, edge_tolerance(bp, bz))
        got = c.build_batch([h], [500], flags=abi.BATCH_REINDEX)[0]
    for k in FIELDS:
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)


def test_events_with_and_without_working_arrays_in_one_batch(gpu_required, monkeypatch):
    """One launch of the bucketed form, one of the other for the events left out by it."""
    print("case index memory mixed", flush=True)
    evs = [synth.make_event(400, cfg=39, event=i, noise=n) for i, n in enumerate((165.0, 165.0, 3.0))]
    cfg = abi.config_from_geometry(evs[0].geometry, max_cands=2)
    memory = Capped()
    with context(cfg, memory, monkeypatch) as c:
        hs = [c.load_event(abi.EventArrays.from_synth(evs[0]))]
        memory.cap = sum(memory.held.values()) + memory.sizes[0] + 4 * 10 * 65540 + (64 << 10)
        hs.append(c.load_event(abi.EventArrays.from_synth(evs[1])))
        memory.cap = None
        hs.append(c.load_event(abi.EventArrays.from_synth(evs[2])))
        together = c.build_batch(hs, [400] * 3, flags=abi.BATCH_REINDEX)
        for h, e, t in zip(hs, evs, together):
            for L in (0, 4, 9):
                off, bin_of, order = c.fetch_index(h, L, len(e.hits[L]))
                grid = c.index_grid(h)
                ref, edge = host_bins(e.hits[L], L, e.geometry, *grid)
                check_layer(off, bin_of, order, ref, edge, edge_tolerance(*grid))
    with abi.Context(cfg) as c:
        hs = c.load_events([abi.EventArrays.from_synth(e) for e in evs])
        for a, b in zip(c.build_batch(hs, [400] * 3), together):
            for k in FIELDS:
                np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("cands", [1, 6])
def test_the_per_event_builder_in_the_state_of_full_wavefronts(gpu_required, monkeypatch, cands):
    """A small event spreads its seeds over more wavefronts, of 64 slots each: with room for the slots of full ones
    alone (64 / lanes seeds a wavefront, 4 (31 + 1 + 1 + layers) bytes a slot) it is built in those; with less,
    refused, and built once there is room."""
    print("case builder memory", cands, flush=True)
    n, lanes = 2001, cands
    ev = synth.make_event(n, cfg=41, event=1, noise=0.2)
    cfg = abi.config_from_geometry(ev.geometry, max_cands=cands)
    memory = Capped()
    with context(cfg, memory, monkeypatch) as c:
        h = c.load_event(abi.EventArrays.from_synth(ev))
        want = c.build_batch([h], [n])[0]
        slots = -(-n // (64 // lanes)) * 64
        state = 4 * (31 + 1 + 1 + 10) * slots
        held = sum(memory.held.values())
        memory.cap = held + state - 4096
        with pytest.raises(abi.MkfError) as err:
            c.build(h, n)
        assert err.value.status == abi.E_NOMEM
        for room in (2048, 64 * state):
            memory.cap = held + state + room
            for _ in range(2):
                got = c.build(h, n)
                for k in FIELDS:
                    np.testing.assert_array_equal(got[k], want[k], err_msg=k)
            c.set_tuning(lanes_per_seed=8)      # the state is laid out anew
            memory.cap = None
            c.build(h, n)
            c.set_tuning(lanes_per_seed=lanes)


def _r(n):
    return (n + 255) & ~255


@pytest.mark.parametrize("noise", [20.0, 135.0])
def test_a_served_event_is_admitted_to_a_budget_of_its_results(gpu_required, noise):
    """The budget: hits (16 bytes, and 16 binned), their bins and ranks (4 each), seeds, the FP64 results of a build
    and of a final fit, counts and offsets of the bins, counters and descriptor."""
    print("case serve memory", noise, flush=True)
    n, nl = 500, 10
    ev = synth.make_event(n, cfg=40, event=1, noise=noise)
    hits = sum(len(x) for x in ev.hits)
    with abi.Context(abi.config_from_geometry(ev.geometry, max_cands=2)) as c:
        h = c.load_event(abi.EventArrays.from_synth(ev))
        want = c.build_batch([h], [n])[0]
        bp, bz = c.index_grid(h)
        fields = [16 * hits, 24 * n, 84 * n, 12 * n, 4 * n, 16 * hits, 4 * hits, 4 * hits, 48 * n, 168 * n,
                  4 * nl * n, 4 * n, 4 * n, 8 * n, 4 * n, 48 * n, 168 * n, 8 * n, 4 * n, 4 * n, 40, 768,
                  4 * nl * bp * bz, 4 * nl * ((bp * bz + 4) & ~3)]
        budget = sum(_r(b) for b in fields)
        for room in (budget, 4 * budget):
            c.serve_config(room, max_in_flight=4)
            t, out = c.serve_submit(ev)
            assert t is not None
            c.serve_drain()
            status, _, got = c.serve_poll(t)
            assert status == abi.OK
            for k in FIELDS:
                np.testing.assert_array_equal(got[k], want[k], err_msg=k)
        c.serve_config(budget - hits * 8, max_in_flight=4)
        with pytest.raises(abi.MkfError) as err:
            c.serve_submit(ev)
        assert err.value.status == abi.E_NOMEM
