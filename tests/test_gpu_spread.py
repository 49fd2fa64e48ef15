"""Seeds per wavefront: a small batch spreads its seeds over more wavefronts
than a large one.  An event built alone, at sizes around a work item's edges,
must give the bits it gives beside events large enough for full wavefronts,
and those of the per-event builder."""
import numpy as np
import pytest

from paper_1702_06359_amd import abi, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cands", [1, 2, 3, 6, 8])
def test_an_event_alone_equals_itself_in_a_full_batch(cands):
    print("case spread", cands, flush=True)
    sizes = (1, 4, 5, 6, 9, 10, 11, 64, 65, 641)
    evs = [synth.make_event(n, cfg=34, event=i, noise=0.3) for i, n in enumerate(sizes)]
    big = [synth.make_event(41000, cfg=34, event=99, noise=0.1)]
    with abi.Context(abi.config_from_geometry(synth.Geometry(), max_cands=cands)) as ctx:
        hs = ctx.load_events([abi.EventArrays.from_synth(e) for e in evs + big])
        together = ctx.build_batch(hs, [e.n_seeds for e in evs + big])
        for h, e, want in zip(hs, evs, together):
            for got in (ctx.build_batch([h], [e.n_seeds])[0], ctx.build(h, e.n_seeds)):
                for f, v in want.items():
                    np.testing.assert_array_equal(got[f], v, err_msg=f"{e.n_seeds} {f}")
