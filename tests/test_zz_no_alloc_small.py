"""The no-allocation builder on small events loaded one by one, which leave a
page-locked staging far smaller than the results of a batch of them: the call
has to move the rows through what is there.  Page-locked memory is mapped into
the process from the GPU's render node, so an allocation, or a staging freed
and made again, shows in the process's own list of mappings."""
import numpy as np
import pytest

from paper_1702_06359_amd import abi, synth

pytestmark = pytest.mark.gpu

FIELDS = ("par", "cov", "hits", "n_hits", "n_holes", "chi2", "status", "ndof")


def _page_locked():
    with open("/proc/self/maps") as f:
        return [line.split()[0] for line in f if "/dev/dri/" in line or "/dev/kfd" in line]


# events, their tracks: staging below a tile's 64 KB beside results of several MB, of which a slot of the ring holds a
# part of an event's rows or several events; one event alone
@pytest.mark.parametrize("n_events,n_tracks", [(200, 100), (250, 33), (3, 150), (1, 1)])
def test_small_events_loaded_one_by_one(gpu_required, n_events, n_tracks):
    print("case noalloc small", n_events, n_tracks, flush=True)
    base = [synth.make_event(n_tracks, cfg=241, event=i, noise=0.1) for i in range(min(n_events, 8))]
    evs = [base[i % len(base)] for i in range(n_events)]
    counts = [e.n_seeds for e in evs]
    with abi.Context(abi.config_from_geometry(synth.Geometry(), max_cands=2)) as c:
        hs = [c.load_event(e) for e in evs]
        c.build_batch_noalloc(hs, None, flags=abi.BATCH_ASYNC)   # the kernels are loaded
        c.sync()
        before = _page_locked()
        got = c.build_batch_noalloc(hs, counts)
        assert _page_locked() == before
        for a, b in zip(got, c.build_batch(hs, counts)):
            for k in FIELDS:
                np.testing.assert_array_equal(a[k], b[k], err_msg=k)
