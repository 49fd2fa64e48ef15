"""The phase timers count the device's work alone: what the host does between
two launches - looking up the arrays of many events, making its staging larger
- belongs to no phase."""
import numpy as np
import pytest

from paper_1702_06359_amd import abi, synth

pytestmark = pytest.mark.gpu

N = 1200    # events of five tracks: a few hundred microseconds on the device, 9,600 output arrays to look up


def _ms(ctx, which, call):
    call()
    ctx.sync()
    best = np.inf
    for _ in range(3):
        ctx.timer_reset()
        call()
        ms, n = ctx.timer_read(which)
        assert n == 1
        best = min(best, ms)
    return best


@pytest.fixture(scope="module")
def many(gpu_required):
    evs = [synth.make_event(5, cfg=35, event=i, noise=0.1) for i in range(8)]
    with abi.Context(abi.config_from_geometry(synth.Geometry(), max_cands=2)) as ctx:
        hs = ctx.load_events([abi.EventArrays.from_synth(evs[i % 8], with_tracks=True) for i in range(N)])
        yield ctx, hs, [5] * N


# the same kernels with and without outputs for the host: the first without a word from the host in between.  Twice
# the time and 50 us are far above what the launches of a delivery take and far below the 9,600 look-ups.
@pytest.mark.parametrize("which,flags", [(1, abi.BATCH_REINDEX), (0, abi.BATCH_REINDEX), (0, abi.BATCH_GRAPH)])
def test_outputs_of_many_events_do_not_lengthen_a_phase(many, which, flags):
    ctx, hs, counts = many
    print("case timers", which, flags, flush=True)
    outs = [abi.TrackArrays(n, 10) for n in counts]
    alone = _ms(ctx, which, lambda: ctx.build_batch(hs, flags=flags | abi.BATCH_ASYNC))
    with_outs = _ms(ctx, which, lambda: ctx.build_batch(hs, flags=flags, outs=outs))
    assert with_outs < 2 * alone + 0.05, (alone, with_outs)


def test_fit_outputs_of_many_events_do_not_lengthen_the_fit(many):
    ctx, hs, counts = many
    print("case timers fit", flush=True)
    alone = _ms(ctx, 2, lambda: ctx.fit_batch(hs))
    with_outs = _ms(ctx, 2, lambda: ctx.fit_batch(hs, counts))
    assert with_outs < 2 * alone + 0.05, (alone, with_outs)


@pytest.mark.parametrize("path", ["build_batch", "fit_batch"])
def test_a_growing_staging_is_no_part_of_a_phase(gpu_required, path):
    """Events loaded one by one leave a staging for one of them: the first call that returns the rows of all of them
    makes it larger (16 MB)."""
    print("case timers staging", path, flush=True)
    n = 4000
    ev = synth.make_event(n, cfg=36, event=1, noise=0.1)
    with abi.Context(abi.config_from_geometry(synth.Geometry(), max_cands=1)) as ctx:
        hs = [ctx.load_event(abi.EventArrays.from_synth(ev, with_tracks=True)) for _ in range(16)]
        if path == "fit_batch":
            alone = _ms(ctx, 2, lambda: ctx.fit_batch(hs))
        else:
            alone = _ms(ctx, 0, lambda: ctx.build_batch(hs))
        ctx.timer_reset()
        if path == "fit_batch":
            ctx.fit_batch(hs, [n] * 16)
            ms, k = ctx.timer_read(2)
        else:
            ctx.build_batch(hs, [n] * 16)
            ms, k = ctx.timer_read(0)
        # the build is in parts and delivers 18 MB of rows on the way (330 us of the host link)
        assert k == 1 and ms < 3 * alone + 0.4, (alone, ms)


def test_a_captured_build_is_not_timed(gpu_required):
    """An asynchronous build captured by the caller: neither the capture nor a replay counts, forty of them (the ring
    of intervals holds 32) leave the capture valid, and the replays build what an eager call builds."""
    import torch
    print("case timers capture", flush=True)
    evs = [synth.make_event(n, cfg=37, event=i, noise=0.1) for i, n in enumerate((700, 300))]
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), abi.Context(abi.config_from_geometry(synth.Geometry(), max_cands=2)) as ctx:
        hs = ctx.load_events([abi.EventArrays.from_synth(e) for e in evs])
        want = ctx.build_batch(hs, [e.n_seeds for e in evs], flags=abi.BATCH_REINDEX)
        ctx.build_batch(hs, flags=abi.BATCH_REINDEX | abi.BATCH_ASYNC)
        ctx.sync()
        ctx.timer_reset()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            for _ in range(40):
                ctx.build_batch(hs, flags=abi.BATCH_REINDEX | abi.BATCH_ASYNC)
        for _ in range(3):
            graph.replay()
            s.synchronize()
            for h, e, w in zip(hs, evs, want):
                got = ctx.fetch_tracks(h, e.n_seeds)
                for k in ("par", "cov", "hits", "chi2", "status"):
                    np.testing.assert_array_equal(got[k], w[k], err_msg=k)
        assert [ctx.timer_read(k)[1] for k in range(3)] == [0, 0, 0]
        ctx.build_batch(hs, flags=abi.BATCH_REINDEX | abi.BATCH_ASYNC)   # queued, then a replay behind it
        graph.replay()
        assert [ctx.timer_read(k)[1] for k in range(3)] == [1, 1, 0]
        one = ctx.timer_read(0)[0]
        ctx.build_batch(hs, flags=abi.BATCH_REINDEX | abi.BATCH_ASYNC)
        assert ctx.timer_read(0)[0] < 3 * one    # a replay's time is 40 builds'
