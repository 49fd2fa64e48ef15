"""The bucketed form of the hit index (few layers of many hits) at its edges:
layers of no hit, of one chunk of 2,048 hits more or less one, of one hit a
bin and of all hits in one bin (a bucket fuller than a block's registers),
grids of a few bins up to 2^20 and ragged ones, beside a layer large enough
that the launch takes this form."""
import numpy as np
import pytest

from paper_1702_06359_amd import abi, synth
from test_gpu_index import check_layer, edge_tolerance, host_bins

pytestmark = pytest.mark.gpu

GRIDS = [(2048, 32), (1, 1), (7, 3), (97, 13), (64, 2), (4096, 256), (1024, 1024)]
COUNTS = (0, 1, 63, 2047, 2048, 2049, 5000, 7000, 20000, 66000)


@pytest.mark.parametrize("bins_phi,bins_z", GRIDS)
def test_bucketed_index_is_the_counting_sort(bins_phi, bins_z):
    rng = np.random.default_rng(bins_phi * 1000 + bins_z)
    g = synth.Geometry()
    hits = []
    for L, n in enumerate(COUNTS):
        phi, z = rng.uniform(-np.pi, np.pi, n), rng.uniform(-1, 1, n) * g.half_z()[L] * 1.1
        if n == 5000:      # one bin holds the whole layer
            phi, z = np.full(n, 0.3), np.full(n, 1.0)
        if n == 7000:      # half of it on the wrap of the azimuth, beyond the grid in z
            phi[::2], z[::2] = np.where(rng.random(3500) < 0.5, np.pi, -np.pi), 1e3
        hits.append(np.stack([g.radii[L] * np.cos(phi), g.radii[L] * np.sin(phi), z], axis=1))
    print("case bucketed index", bins_phi, bins_z, flush=True)
    with abi.Context(abi.config_from_geometry(g)) as c:
        c.set_tuning(bins_phi=bins_phi, bins_z=bins_z)
        h = c.load_event(abi.EventArrays(hits))
        grid = c.index_grid(h)
        for L in range(g.n_layers):
            off, bin_of, order = c.fetch_index(h, L, len(hits[L]))
            ref, edge = host_bins(hits[L], L, g, *grid)
            if COUNTS[L] == 7000:   # the exact wrap may fall on either side of it
                edge = np.where(np.abs(np.abs(np.arctan2(hits[L][:, 1], hits[L][:, 0])) - np.pi) < 1e-5, 0.0, edge)
            check_layer(off, bin_of, order, ref, edge, edge_tolerance(*grid))
