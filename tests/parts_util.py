"""The parts a batch with host outputs is built in, from the library's own planner (mkf::plan_parts), called through a
few lines of C++ compiled here."""
import ctypes as C
import os
import subprocess

import numpy as np

from paper_1702_06359_amd import abi, build as hip_build

WRAP = r"""
#include "mkf_runtime.hpp"
extern "C" int t_plan(const int *seeds, const int *layer_hits, int n, int geo, int cands, int layers, int seed_layers,
                      double us_per_row, long long *ends)
{
    std::vector<mkf::EventLoad> loads;
    for (int i = 0; i < n; ++i) loads.push_back(mkf::EventLoad{seeds[i], layer_hits[i]});
    mkf::Params P{};
    P.geo = geo;
    P.max_cands = cands;
    P.n_layers = layers;
    P.n_seed_layers = seed_layers;
    const std::vector<long long> e = mkf::plan_parts(loads, P, us_per_row);
    for (size_t k = 0; k < e.size(); ++k) ends[k] = e[k];
    return (int)e.size();
}
extern "C" int t_items(const int *seeds, int n, long long rows, int spi)
{
    std::vector<mkf::EventLoad> loads;
    for (int i = 0; i < n; ++i) loads.push_back(mkf::EventLoad{seeds[i], 0});
    return mkf::items_before(loads, rows, spi);
}
extern "C" int t_spi(int geo, int lanes, long long seeds) { return mkf::seeds_per_item(geo, lanes, seeds); }
extern "C" double t_us_per_row(int layers, int pinned)
{
    double b = 0;
    for (int f = 0; f < mkf::kOutFields; ++f) b += (double)mkf::field_bytes(f, layers);
    return b / (pinned ? mkf::kLinkBytesPerUs : mkf::kCopyBytesPerUs);
}
extern "C" int t_block() { return mkf::kSeedBlock; }
extern "C" int t_most() { return mkf::kBuildParts; }
"""


class Planner:
    def __init__(self, folder):
        if not os.path.exists(abi.LIB_PATH):
            hip_build.build(force=True)
        abi.lib()
        src, so = folder / "plan.cpp", folder / "plan.so"
        src.write_text(WRAP)
        res = subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                              "-I/opt/rocm/include", "-I", hip_build.CSRC, str(src), "-o", str(so), abi.LIB_PATH],
                             capture_output=True, text=True)
        assert res.returncode == 0, res.stderr
        self.L = C.CDLL(str(so))
        self.L.t_plan.argtypes = [C.c_void_p, C.c_void_p] + [C.c_int] * 5 + [C.c_double, C.c_void_p]
        self.L.t_items.argtypes = [C.c_void_p, C.c_int, C.c_longlong, C.c_int]
        self.L.t_spi.argtypes = [C.c_int, C.c_int, C.c_longlong]
        self.L.t_us_per_row.restype = C.c_double
        self.block, self.most = self.L.t_block(), self.L.t_most()

    def ends(self, seeds, layer_hits, geo=0, cands=6, layers=10, seed_layers=3, us_per_row=None, pinned=True):
        s, h = np.asarray(seeds, np.int32), np.asarray(layer_hits, np.int32)
        out = np.zeros(64, np.int64)
        us = self.L.t_us_per_row(layers, int(pinned)) if us_per_row is None else us_per_row
        k = self.L.t_plan(s.ctypes.data, h.ctypes.data, len(s), geo, cands, layers, seed_layers, us, out.ctypes.data)
        return [int(e) for e in out[:k]]

    def items(self, seeds, rows, spi):
        s = np.asarray(seeds, np.int32)
        return self.L.t_items(s.ctypes.data, len(s), rows, spi)
