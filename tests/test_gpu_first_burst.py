"""A new server's first burst goes through page-locked memory that the host has
never touched, where the first touch of every page is slow: several threads
share them, so that neither the submitting thread while it packs nor the
scheduler while it copies results out bears them alone.  And submits from
several threads at once, while those pages are being touched, keep their
inputs."""
import threading
import time

import numpy as np
import pytest

from paper_1702_06359_amd import abi, synth

pytestmark = pytest.mark.gpu

FIELDS = ("par", "cov", "hits", "n_hits", "n_holes", "chi2", "ndof", "status")


def _burst(c, inputs, outs):
    t0 = time.perf_counter()
    tickets = [c.serve_submit(None, ea=ea, out=o)[0] for ea, o in zip(inputs, outs)]
    c.serve_drain()
    t = time.perf_counter() - t0
    for k in tickets:
        assert c.serve_poll(k)[0] == abi.OK
    return t


def _outs(evs):
    outs = [abi.TrackArrays(e.n_seeds, 10) for e in evs]
    for o in outs:
        for f in FIELDS:
            getattr(o, f).fill(1)       # the caller's own pages are there
    return outs


def test_a_first_burst_takes_little_longer_than_the_next(gpu_required):
    """8 events, 60,000 tracks, 39 MB through the staging: the next burst takes about 2 ms, the pages of the first 13
    ms more by two threads in turn, 1 ms by sixteen, and the slabs 1 ms to make.  The best of five servers, so that a
    busy host does not decide; all of them stay open, so that each has memory of its own."""
    evs = [synth.make_event(n, cfg=44, event=i, noise=0.2) for i, n in enumerate((3000, 5000, 6000, 7000, 8000, 9000,
                                                                                 10000, 12000))]
    inputs, outs = [abi.EventArrays.from_synth(e) for e in evs], _outs(evs)
    open_, first, nxt = [], [], []
    try:
        for _ in range(5):
            c = abi.Context(abi.config_from_geometry(synth.Geometry(), max_cands=2))
            open_.append(c)
            h = c.load_event(inputs[0])         # the kernels and the host threads are there
            c.build_batch([h], outs=outs[:1])
            c.serve_config(512 << 20, max_in_flight=16)
            print("case first burst", len(open_), flush=True)
            first.append(_burst(c, inputs, outs))
            nxt.append(min(_burst(c, inputs, outs) for _ in range(4)))
    finally:
        for c in open_:
            c.close()
    print("first", [int(1e6 * t) for t in first], "next", [int(1e6 * t) for t in nxt], flush=True)
    # 2.4-2.8 on three machines; 4.7-5.0 with the pages left to the two threads
    assert min(first) < 3.75 * np.median(nxt)


def test_concurrent_submits_into_new_pages_keep_their_inputs(gpu_required):
    evs = [synth.make_event(1900 + 37 * i, cfg=45, event=i, noise=0.2) for i in range(24)]
    inputs = [abi.EventArrays.from_synth(e) for e in evs]
    with abi.Context(abi.config_from_geometry(synth.Geometry(), max_cands=2)) as c:
        hs = c.load_events(inputs)
        want = c.build_batch(hs, [e.n_seeds for e in evs])
        for rep in range(6):
            c.serve_config(512 << 20, max_in_flight=64)
            print("case concurrent submits", rep, flush=True)
            got, outs = [None] * len(evs), [abi.TrackArrays(e.n_seeds, 10) for e in evs]
            gate = threading.Barrier(6)

            def submit(k):
                gate.wait()
                for i in range(k, len(evs), 6):
                    got[i] = c.serve_submit(None, ea=inputs[i], out=outs[i])[0]

            threads = [threading.Thread(target=submit, args=(k,)) for k in range(6)]
            for t in threads:
                t.start()
            for t in threads:
                t.join()
            c.serve_drain()
            for i, k in enumerate(got):
                status, _, out = c.serve_poll(k)
                assert status == abi.OK
                for f in FIELDS:
                    np.testing.assert_array_equal(out[f], want[i][f], err_msg=f"{i} {f}")
