"""Smoothing lengths and neighbour sets of the wave-wide tree search where it
changes course: trees of one step and of several, groups of 8 with a short
last one, and particles with more neighbours in reach than their list holds
(a tight clump at the edge of a coarse particle's support).

Bars: the solve stops at steps of 4 ulp and its sums of about 50 terms round
to about 1e-15 with a slope of order one, so h agrees with the oracle's to
1e-13; neighbour sets are compared on the oracle's h and are exact.
"""
import numpy as np
import pytest
import torch

import oracle
import workloads
from tests.gpu_util import dev, log, unsort

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2302_12727_amd import RT  # noqa: E402


def clump_set(n_side: int, m: int, seed: int) -> np.ndarray:
    """A jittered lattice and m points in a ball of 1/50 of its spacing at a
    cell corner: the lattice particles around reach the whole clump."""
    g = workloads.rng(seed)
    d = g.normal(size=(m, 3))
    d *= (g.uniform(size=(m, 1)) ** (1 / 3) / (50 * n_side)) / np.linalg.norm(d, axis=1, keepdims=True)
    return np.concatenate([workloads.jittered_lattice(n_side, 0.1, seed), 0.5 + d])


@pytest.mark.parametrize("x", [
    workloads.jittered_lattice(5, 0.1, 1),             # 4 leaves, one step of the tree
    workloads.jittered_lattice(13, 0.1, 2)[:2047],     # 64 leaves, one whole step
    workloads.jittered_lattice(13, 0.1, 2)[:2049],     # 65 leaves, two steps
    clump_set(10, 400, 3),
    clump_set(10, 100, 4),                             # reaches cut and drawn out again
], ids=["n125", "n2047", "n2049", "clump", "small clump"])
def test_smoothing_lengths_and_neighbours(x):
    n = x.shape[0]
    geo = oracle.build_geometry(x)
    rt = RT(n, 1)
    perm, h, _, _ = rt.rt_build_cells(dev(x))
    p = perm.cpu().numpy()
    err = float(np.abs(unsort(h.cpu().numpy(), p) / geo.h - 1).max())
    st = rt.rt_get_stats()
    log(f"n={n}: h error {err:.2e}, {st['h_list_overflow']} lists overflowed, "
        f"most gather neighbours {np.diff(geo.gptr).max()}")
    assert err < 1e-13
    if n == 1400:
        # more particles in reach than a list holds, at the root itself too
        assert np.diff(geo.gptr).max() > 128 and st["h_list_overflow"] > 0
    perm, *_ = rt.rt_build_cells(dev(x), dev(geo.h))
    p = perm.cpu().numpy()
    ptr, idx = (t.cpu().numpy() for t in rt.rt_get_neighbours())
    got = p[np.repeat(np.arange(n), np.diff(ptr))].astype(np.int64) * n + p[idx]
    ref = np.repeat(np.arange(n, dtype=np.int64), np.diff(geo.sptr)) * n + geo.sidx
    assert np.array_equal(np.sort(got), np.sort(ref))
    xs = np.ascontiguousarray(x[[0, n // 2, n - 1]] * 0.999 + 0.0005)
    rt.rt_set_sources(dev(xs))
    srcs = oracle.build_sources(geo, xs)
    assert np.abs(rt.rt_get_sources()[3].cpu().numpy() / srcs.h - 1).max() < 1e-13
