"""A layer of hits, or a run of states, that its first check refuses stays
refused when the search for the first bad value finds none (a caller's array
that changes in between): the load is rejected, and nothing outside the arrays
is read or written.  The checks are replaced by ones that disagree: a library
loaded before libmkf.so brings its own mkf::pack_hits and
mkf::states_in_range."""
import os
import subprocess
import sys

import pytest

from paper_1702_06359_amd import abi, build as hip_build

STUB = r"""
#include "mkf_runtime.hpp"
#include "mkf_pack.hpp"
#include <vector>
namespace mkf {
static bool g_hits, g_states;
bool pack_hits(const double *, size_t n, HitForm, float *) { return !g_hits || n == 1; }
bool states_in_range(const double *, size_t n) { return !g_states || n == 1; }
}
extern "C" int t_pack(int refuse_hits, int refuse_states, int part, char *why_out)
{
    using namespace mkf;
    g_hits = refuse_hits;
    g_states = refuse_states;
    EventShape s;
    s.n_layers = 4;
    s.n_seed_layers = 3;
    s.n_seeds = 5000;
    int32_t n_hits[4] = {9, 8, 7, 6};
    for (int L = 0; L < 4; ++L) s.layer_off[L + 1] = s.layer_off[L] + n_hits[L];
    std::vector<double> h(27, 1.0), par(6 * s.n_seeds, 1.0), cov(21 * s.n_seeds, 1.0);
    std::vector<int32_t> hits(3 * s.n_seeds, 0);
    const double *xyz[4] = {h.data(), h.data(), h.data(), h.data()};
    mkf_event e{};
    e.n_layers = 4;
    e.n_seeds = s.n_seeds;
    e.n_hits = n_hits;
    e.hit_xyz = xyz;
    e.seed_par = par.data();
    e.seed_cov = cov.data();
    e.seed_hits = hits.data();
    std::vector<char> image(event_input_bytes(s) + 256);
    char *at = reinterpret_cast<char *>((reinterpret_cast<uintptr_t>(image.data()) + 255) & ~uintptr_t(255));
    std::string why;
    const mkf_status st = pack_event(&e, s, 0, at, 1, &why, (PackPart)part);
    snprintf(why_out, 200, "%s", why.c_str());
    return st;
}
"""

RUN = r"""
import ctypes as C, sys
try:
    import torch
except ImportError:
    pass
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL | 1)   # lazily bound, before the library
C.CDLL(sys.argv[2], mode=C.RTLD_GLOBAL)
why = C.create_string_buffer(200)
st = stub.t_pack(int(sys.argv[3]), int(sys.argv[4]), int(sys.argv[5]), why)
print("status", st, why.value.decode())
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    if not os.path.exists(abi.LIB_PATH):
        hip_build.build(force=True)
    d = tmp_path_factory.mktemp("refusal")
    src, so = d / "stub.cpp", d / "stub.so"
    src.write_text(STUB)
    res = subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                          "-I/opt/rocm/include", "-I", hip_build.CSRC, str(src), "-o", str(so)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return str(so)


# parts: 0 all inputs, 1 the hits alone, 2 the seeds and tracks
@pytest.mark.parametrize("hits,states,part,said", [(1, 0, 0, "layer 0 hit 0"), (1, 0, 1, "layer 0 hit 0"),
                                                   (0, 1, 0, "seed 0"), (0, 1, 2, "seed 0"), (0, 0, 0, "")])
def test_a_refused_input_stays_refused(stub, hits, states, part, said):
    r = subprocess.run([sys.executable, "-c", RUN, stub, abi.LIB_PATH, str(hits), str(states), str(part)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-500:]
    want = abi.E_INVALID if said else abi.OK
    assert r.stdout.startswith(f"status {want} {said}"), r.stdout
