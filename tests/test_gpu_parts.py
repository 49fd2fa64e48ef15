"""Builds in parts, each part's rows delivered by the launch that builds the
next, at every boundary there can be.  The planner decides by a model of the
times, so here it is replaced: in a process of its own, a library loaded before
libmkf.so brings a mkf::plan_parts that ends a part at every block and event
and counts what it was asked.  Against the same batch built by one launch, bit
for bit, and against the oracle at seeds around the boundaries."""
import ctypes as C
import json
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
SIZES = (20481, 1, 30007, 10240)        # eight blocks: a part of one row, events that end within a block
FIELDS = ("par", "cov", "hits", "n_hits", "n_holes", "chi2", "ndof", "status")
# candidates, wavefronts a block, layers, surfaces: every lane count (seeds per item of 64 down to 8), a delivery's LDS
# above and below the build's, blocks of several wavefronts that deliver, and every form of the search
CASES = [(6, 1, 10, "barrel"), (8, 2, 10, "barrel"), (1, 4, 4, "barrel"), (4, 1, 4, "barrel"), (1, 4, 10, "barrel"),
         (6, 4, 10, "barrel"), (2, 1, 10, "endcap"), (6, 1, 10, "endcap"), (1, 4, 7, "endcap"), (6, 1, 10, "thick"),
         (1, 2, 10, "thick"), (6, 1, 16, "barrel")]

STUB = r"""
#include "mkf_runtime.hpp"
static int g_calls, g_parts;
namespace mkf {
std::vector<long long> plan_parts(const std::vector<EventLoad> &loads, const Params &, double)
{
    std::vector<long long> ends;
    long long rows = 0;
    for (const EventLoad &l : loads) {
        for (int b = kSeedBlock; b < l.seeds; b += kSeedBlock) ends.push_back(rows + b);
        rows += l.seeds;
        ends.push_back(rows);
    }
    if ((int)ends.size() > kBuildParts) abort();
    ++g_calls;
    g_parts = (int)ends.size();
    return ends;
}
}
extern "C" int t_calls() { return g_calls; }
extern "C" int t_parts() { return g_parts; }
"""


def _case(stub, cands, waves, layers, kind):
    import oracle
    from paper_1702_06359_amd import abi, synth
    from parity_util import assert_build_parity, compare_build
    from test_gpu_delivery import _pinned, _shifted
    g = synth.Geometry.endcap(layers) if kind == "endcap" else synth.Geometry(
        n_layers=layers, radii=tuple(4.0 * (i + 1) for i in range(layers)), x0=(0.002,) * layers,
        thickness=(0.6,) * layers if kind == "thick" else None)
    evs = [synth.make_event(n, cfg=42, event=i, noise=0.1, geometry=g, pt_range=(1.0, 10.0))
           for i, n in enumerate(SIZES)]
    with abi.Context(abi.config_from_geometry(g, max_cands=cands)) as ctx:
        ctx.set_tuning(waves_per_block=waves)
        hs = ctx.load_events([abi.EventArrays.from_synth(e) for e in evs])
        ctx.build_batch(hs, flags=abi.BATCH_ASYNC)   # one launch
        one = [ctx.fetch_tracks(h, n) for h, n in zip(hs, SIZES)]
        for empty in (_pinned, None, _shifted):
            before = stub.t_calls()
            parts = [abi.TrackArrays(n, layers, empty=empty) for n in SIZES]
            ctx.build_batch(hs, flags=abi.BATCH_REINDEX, outs=parts)
            assert stub.t_calls() == before + 1 and stub.t_parts() == 8
            for a, b in zip(parts, one):
                for f in FIELDS:
                    np.testing.assert_array_equal(getattr(a, f), b[f], err_msg=f)
        some = [abi.TrackArrays(n, layers, empty=_pinned) for n in SIZES]   # the final fit after it, a few fields
        for o in some:
            o.tracks.cov = o.tracks.ndof = o.tracks.n_holes = None
        ctx.build_batch(hs, flags=abi.BATCH_FIT, outs=some)
        for a, b in zip(some, one):
            for f in ("par", "hits", "n_hits", "chi2", "status"):
                np.testing.assert_array_equal(getattr(a, f), b[f], err_msg=f)
    rows = np.array([0, 1, 10238, 10239, 10240, 10241, 20478, 20479, 20480] +
                    list(np.random.default_rng(7).integers(0, SIZES[0], 40)))
    rows = np.unique(rows)
    cfg = oracle.config(g, max_cands=cands)
    ev = evs[0]
    ref = oracle.build_tracks(cfg, ev.hits, ev.seed_par, ev.seed_cov, ev.seed_hits, seed_ids=rows.astype(np.int32),
                              n_threads=8)
    rep = compare_build(one[0], ref, cfg, ev.hits, ev.seed_par, ev.seed_cov, rows=rows)
    assert_build_parity(rep)


def _main(so):
    sys.path[:0] = [HERE, os.path.dirname(HERE)]
    import torch  # noqa: F401
    stub = C.CDLL(so, mode=C.RTLD_GLOBAL | 1)   # lazily bound, before the library
    from paper_1702_06359_amd import abi
    C.CDLL(abi.LIB_PATH, mode=C.RTLD_GLOBAL)
    for case in CASES:
        print("case", case, flush=True)
        try:
            _case(stub, *case)
            said = "ok"
        except AssertionError as e:
            said = ("AssertionError: %s" % e)[:1500]
        print("result " + json.dumps([list(case), said]), flush=True)


@pytest.fixture(scope="module")
def results(gpu_required, tmp_path_factory):
    from paper_1702_06359_amd import build as hip_build
    d = tmp_path_factory.mktemp("parts")
    src, so = d / "stub.cpp", d / "stub.so"
    src.write_text(STUB)
    res = subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                          "-I/opt/rocm/include", "-I", hip_build.CSRC, str(src), "-o", str(so)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    r = subprocess.run([sys.executable, os.path.abspath(__file__), str(so)], capture_output=True, text=True,
                       timeout=100)
    got = [json.loads(line[7:]) for line in r.stdout.splitlines() if line.startswith("result ")]
    return {tuple(c): said for c, said in got}, f"status {r.returncode}: {r.stdout[-300:]} {r.stderr[-1500:]}"


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_a_build_in_parts(results, case):
    by_case, tail = results
    assert by_case.get(case, tail) == "ok"


if __name__ == "__main__":
    _main(sys.argv[1])
