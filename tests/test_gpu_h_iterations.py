"""The iteration count and cap of the smoothing-length solve against a model of
the iteration in numpy (start from the leaf box and the Morton window, Newton
steps inside a bracket, doubling until there is one, stop at a step of 4 ulp).

A particle that takes k iterations needs k + 1 evaluations, the last of which
meets the step test: that cap builds and one less is refused.  Evaluations that
the library spends on its candidate lists are not iterations, so it never needs
a larger cap than the model; it may need a smaller one, where a list's end takes
the place of an iterate further from the root.
"""
import numpy as np
import pytest
import torch
from scipy.spatial import cKDTree

import oracle
import workloads
from tests.gpu_util import dev, log, unsort
from tests.test_gpu_search import clump_set

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2302_12727_amd import RT  # noqa: E402
from paper_2302_12727_amd.rt import KAPPA, RTError  # noqa: E402


def model_iterations(xs, eta, kappa=KAPPA):
    """Iterations of every particle; xs in Morton order, unit box."""
    n = xs.shape[0]
    d = xs[None] - xs[:, None]
    d -= np.rint(d)
    r = np.sqrt((d * d).sum(axis=2))
    leaf = np.arange(n) // 32
    ext = np.ones(n)
    for a in range(3):
        lo, hi = (f.reduceat(xs[:, a], np.arange(0, n, 32)) for f in (np.minimum, np.maximum))
        ext *= np.maximum(hi - lo, 1 / 2097152)[leaf]
    h = eta * np.cbrt(ext / np.bincount(leaf)[leaf])
    i = np.arange(n)
    near = np.where((np.abs(i[None] - i[:, None]) <= 16) & (i[None] != i[:, None]), r, np.inf)
    fourth = np.sort(near, axis=1)[:, 3]
    h = np.minimum(np.minimum(h, 0.8 * eta * fourth * 0.94269861348), min(0.25, 0.25 / kappa))
    pref, eta3, eps4 = 16 / np.pi / kappa ** 3, eta ** 3, 4 * 2.0 ** -52
    lo, hi, hcap = np.zeros(n), np.full(n, np.inf), 0.5 / kappa
    its, live = np.zeros(n, dtype=int), np.ones(n, dtype=bool)
    while live.any():
        q = r[live] / (kappa * h[live])[:, None]
        a, b = np.maximum(1 - q, 0), np.maximum(0.5 - q, 0)
        sw = (a ** 3 - 4 * b ** 3).sum(axis=1)
        sdw = ((-3 * a * a + 12 * b * b) * q).sum(axis=1)
        hl, lol, hil = h[live], lo[live], hi[live]
        g, dg = pref * sw - eta3, -pref * sdw / hl
        lol, hil = np.where(g < 0, hl, lol), np.where(g < 0, hil, hl)
        step = np.where(dg > 0, hl - g / np.where(dg > 0, dg, 1), -1.0)
        out = np.where((dg > 0) & (step > hl) & (step < 4 * hl), step, 2 * hl)
        mid = np.where((step > lol) & (step < hil), step, 0.5 * (lol + np.where(np.isinf(hil), 0, hil)))
        open_end = np.isinf(hil)
        new = np.where(open_end, np.minimum(out, hcap), mid)
        done = (g == 0) | (~open_end & ((np.abs(new - hl) <= eps4 * hl)
                                        | ((dg > 0) & (np.abs(step - hl) <= eps4 * hl))
                                        | (hil - lol <= eps4 * hil)))
        assert not (open_end & (hl >= hcap)).any()
        at = np.flatnonzero(live)
        h[at], lo[at], hi[at] = new, lol, hil
        its[at[~done]] += 1
        live[at[done]] = False
        assert its.max() < 200
    return its


def check(x, eta):
    """The context built with the smallest cap, and its Morton order."""
    rt = RT(x.shape[0], 1, eta=eta)
    perm, h, _, _ = rt.rt_build_cells(dev(x))
    model = int(model_iterations(x[perm.cpu().numpy()], eta).max())
    took = rt.rt_get_stats()["h_iter_max"]
    h = h.clone()
    log(f"n={x.shape[0]} eta={eta}: {took} iterations, model {model}")
    assert 1 <= took <= model
    rt.rt_set_h_iterations(took)
    with pytest.raises(RTError, match="RT_ENOCONV"):
        rt.rt_build_cells(dev(x))
    rt.rt_set_h_iterations(took + 1)
    assert torch.equal(rt.rt_build_cells(dev(x))[1], h)
    return rt, perm.cpu().numpy()


@pytest.mark.parametrize("x", [
    workloads.jittered_lattice(13, 0.1, 2),
    workloads.config(4, scale=(1 << 11) / (1 << 24)).x,
    clump_set(10, 100, 4),                      # lists cut and drawn out again
], ids=["lattice", "plummer", "small clump"])
def test_iterations_and_cap(x):
    check(x, 1.2348)


@pytest.mark.parametrize("eta", [1.65, 1.8, 2.2])
@pytest.mark.parametrize("x", [
    workloads.jittered_lattice(13, 0.1, 2),
    clump_set(10, 400, 3),
], ids=["lattice", "clump"])
def test_more_neighbours_than_a_list_holds(x, eta):
    """110 to 260 particles in reach at the root, more than a candidate list's
    120: the iteration as long as the model's all the same, for particles and
    for sources, and h the oracle's (to 1e-13: the solve stops at 4 ulp, its
    sums of up to 700 terms round to about 1e-14 at most)."""
    rt, p = check(x, eta)
    geo = oracle.build_geometry(x, eta=eta)
    err = float(np.abs(unsort(rt.h.cpu().numpy(), p) / geo.h - 1).max())
    xs = np.ascontiguousarray(x[[0, x.shape[0] // 2, x.shape[0] - 1]] * 0.999 + 0.0005)
    rt.rt_set_h_iterations(10)
    rt.rt_set_sources(dev(xs), eta)
    serr = float(np.abs(rt.rt_get_sources()[3].cpu().numpy()
                        / oracle.build_sources(geo, xs, eta).h - 1).max())
    log(f"h error {err:.1e}, of sources {serr:.1e}, most gather neighbours {np.diff(geo.gptr).max()}")
    assert np.diff(geo.gptr).max() > 120
    assert err < 1e-13 and serr < 1e-13


def test_more_dense_groups_than_the_grid():
    """Every point dense, in 12 978 groups of 8: the dense points' kernel runs
    12 288 waves at most, so some take a second group (the last one has 7)."""
    x = workloads.jittered_lattice(47, 0.1, 2)
    rt = RT(x.shape[0], 1, eta=1.8)
    perm, h, _, _ = rt.rt_build_cells(dev(x))
    ref, _ = oracle.solve_h(cKDTree(x, boxsize=1.0), x, 1.8)
    assert rt.rt_get_stats()["h_list_overflow"] == x.shape[0]
    assert np.abs(unsort(h.cpu().numpy(), perm.cpu().numpy()) / ref - 1).max() < 1e-13
