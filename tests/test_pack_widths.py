"""Host packing of inputs (mkf_pack.cpp): every vector width the host has
must give the bits of the scalar form for every hit form, and the checks must
find a single bad value wherever it stands."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_1702_06359_amd import build as hip_build

WRAP = r"""
#include "mkf_pack.cpp"
using namespace mkf;
template <HitForm F> static bool hits(int w, const double *h, size_t n, float *o)
{
    return w == 2 ? hits_avx512<F>(h, n, o) : w == 1 ? hits_avx2<F>(h, n, o) : hits_body<F>(h, n, o);
}
extern "C" {
int t_width() { return host_width(); }
int t_hits(int w, int form, const double *h, size_t n, float *o)
{
    return form == 0 ? hits<HitForm::kCylinder>(w, h, n, o) : form == 1 ? hits<HitForm::kDisk>(w, h, n, o)
                                                                        : hits<HitForm::kXyz>(w, h, n, o);
}
int t_narrow(int w, const double *s, float *d, size_t n)
{
    return w == 2 ? narrow_avx512(s, d, n) : w == 1 ? narrow_avx2(s, d, n) : narrow_body(s, d, n);
}
int t_states(int w, const double *p, size_t n)
{
    return w == 2 ? states_avx512(p, n) : w == 1 ? states_avx2(p, n) : states_body(p, n);
}
}
"""


@pytest.fixture(scope="module")
def pack(tmp_path_factory):
    d = tmp_path_factory.mktemp("pack")
    src, so = d / "wrap.cpp", d / "wrap.so"
    src.write_text(WRAP)
    res = subprocess.run([hip_build.HIPCC, "-xc++", *hip_build.PACK_FLAGS, "-I", hip_build.CSRC, "-shared", str(src),
                          "-o", str(so)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    L = C.CDLL(str(so))
    L.t_hits.argtypes = [C.c_int, C.c_int, C.c_void_p, C.c_size_t, C.c_void_p]
    L.t_narrow.argtypes = [C.c_int, C.c_void_p, C.c_void_p, C.c_size_t]
    L.t_states.argtypes = [C.c_int, C.c_void_p, C.c_size_t]
    return L


def _widths(pack):
    return range(1, pack.t_width() + 1)


@pytest.mark.parametrize("form", [0, 1, 2])
@pytest.mark.parametrize("n", [1, 3, 7, 8, 31, 32, 33, 1001])
def test_hits_of_every_width_are_the_scalar_bits(pack, form, n):
    rng = np.random.default_rng(n)
    h = np.ascontiguousarray(rng.normal(0, 30, (n, 3)) * 10.0 ** rng.uniform(-3, 3, (n, 1)))
    want = np.zeros((n, 4), np.float32)
    assert pack.t_hits(0, form, h.ctypes.data, n, want.ctypes.data) == 1
    r = np.sqrt(h[:, 0] * h[:, 0] + h[:, 1] * h[:, 1])
    c = {0: (h[:, 0] / r, h[:, 1] / r, h[:, 2], r), 1: (h[:, 0] / r, h[:, 1] / r, r, h[:, 2]),
         2: (h[:, 0], h[:, 1], h[:, 2], 0 * r)}[form]
    np.testing.assert_array_equal(want, np.stack(c, 1).astype(np.float32))
    for w in _widths(pack):
        got = np.zeros((n, 4), np.float32)
        assert pack.t_hits(w, form, h.ctypes.data, n, got.ctypes.data) == 1
        np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))
        for bad in (np.nan, np.inf, -np.inf, 1e39):
            for col in range(3):
                g = h.copy()
                g[n // 2, col] = bad
                assert pack.t_hits(w, form, g.ctypes.data, n, got.ctypes.data) == 0, (w, bad, col)
        g = h.copy()
        g[n - 1, :2] = 0.0      # on the axis
        assert pack.t_hits(w, form, g.ctypes.data, n, got.ctypes.data) == 0


@pytest.mark.parametrize("n", [1, 5, 8, 33, 64, 65, 1000])
def test_values_and_states_of_every_width(pack, n):
    rng = np.random.default_rng(n)
    v = rng.normal(0, 1, 6 * n) * 10.0 ** rng.uniform(-40, 30, 6 * n)
    p = rng.normal(0, 10, (n, 6))
    p[:, 5] = rng.uniform(1e-3, np.pi - 1e-3, n)
    for w in [0, *_widths(pack)]:
        got = np.zeros(6 * n, np.float32)
        assert pack.t_narrow(w, v.ctypes.data, got.ctypes.data, 6 * n) == 1
        np.testing.assert_array_equal(got.view(np.uint32), v.astype(np.float32).view(np.uint32))
        for bad in (np.nan, np.inf, 4e38):
            g = v.copy()
            g[(6 * n) // 2] = bad
            assert pack.t_narrow(w, g.ctypes.data, got.ctypes.data, 6 * n) == 0
        assert pack.t_states(w, p.ctypes.data, n) == 1
        for row, col, bad in ((n - 1, 5, 0.0), (n // 2, 5, np.pi), (0, 5, np.nan)):
            g = p.copy()
            g[row, col] = bad
            assert pack.t_states(w, g.ctypes.data, n) == 0
        g = p.copy()
        g[n - 1, :2] = 0.0
        assert pack.t_states(w, g.ctypes.data, n) == 0
