"""Every kernel that the transports choose by the size of the set and its groups,
in its global step and in its ticks, with each solver and surface kind, against
the oracle: all groups of up to 3 in a wave, a block for every group, slices of 3
and 2 of more; 8 or 4 lanes a particle, three waves per SIMD.  The routes are read
from the launch records, so a rule that moves takes a test off its kernel no
longer unseen.

16 000 particles are 250 tiles (the last one whole), 20 000 are 313, 33 000 are
516; the two larger sets end in tiles of 32 and 40 particles.

Bars as in the tests of the single routes: 1e-12 of the neighbourhood's scale in
FP64, 1e-5 in FP32C; photon totals a tenth of that.
"""
import functools

import numpy as np
import pytest
import torch

import oracle
import workloads
from tests.gpu_util import dev, local_err, log, unsort

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2302_12727_amd import RT  # noqa: E402

TOL = {"fp64": 1e-12, "fp32c": 1e-5}
STEPS, TICKS, MAX_BIN = 2, 3, 3
# routes beside the first one; three_waves is GLF's only
ROUTES = {
    ("fp64", 16000): ["whole wide", "one_group", "whole wide", "slices", "one_group three_waves",
                      "one_group three_waves", "slices wide", "slices wide"],
    ("fp64", 20000): ["whole"],
    ("fp64", 33000): ["whole three_waves", "whole", "whole"] + ["slices"] * 5,
    ("fp32c", 16000): ["whole"] + ["one_group"] * 5 + ["slices"] * 2,
    ("fp32c", 33000): ["whole"] * 3 + ["slices"] * 5,
}
NAMES = ["whole", "one_group", "slices", "wide", "three_waves"]
MODES = [(s, a, t) for s in ("glf", "hll") for a in ("hopkins", "ivanova") for t in (False, True)]


@functools.lru_cache(maxsize=None)
def particles(n):
    w = workloads.plummer_workload(n, 8, STEPS, 77, n_src=3, central_source=False)
    geo = oracle.build_geometry(w.x)
    return w, geo, oracle.build_sources(geo, w.xs), oracle.hll_table()


@functools.lru_cache(maxsize=None)
def reference(n, solver, surfaces, ticks):
    """States, pending sums, totals, guard counts and ledgers of 8 groups."""
    w, geo, srcs, tab = particles(n)
    kw = dict(hll=tab if solver == "hll" else None, ivanova=surfaces == "ivanova")
    if ticks:
        U, info = oracle.run_binned(geo, srcs, w.U0, w.L, TICKS, oracle.time_bins(geo, MAX_BIN), **kw)
        acc = info["acc"]
    else:
        U, info = oracle.run(geo, srcs, w.U0, w.L, STEPS, **kw)
        acc = None
    return U, acc, oracle.photon_total(geo, U), info["ledger"]


@pytest.mark.parametrize("precision,n,groups", [(p, n, g + 1) for (p, n), r in ROUTES.items()
                                                for g in range(len(r))])
def test_routes(precision, n, groups):
    w, geo, srcs, tab = particles(n)
    rt = RT(n, groups, precision=precision)
    perm, *_ = rt.rt_build_cells(dev(w.x))
    rt.rt_set_sources(dev(w.xs))
    p = perm.cpu().numpy()
    L = dev(w.L[:, :groups])
    tol, worst = TOL[precision], 0.0
    for solver, surfaces, ticks in MODES:
        rt.rt_set_riemann(solver)
        rt.rt_set_surfaces(surfaces)
        rt.rt_timing(True)
        U = dev(w.U0[p][:, :groups]).to(rt.sdtype)
        Q = torch.zeros(groups, dtype=torch.float64, device="cuda")
        ledger = torch.zeros(groups, dtype=torch.float64, device="cuda")
        acc = torch.zeros(U.shape, dtype=torch.float64, device="cuda")
        if ticks:
            _, cycle = rt.rt_time_bins(MAX_BIN)
            assert cycle > TICKS                # pending sums at the end
            UD = rt.rt_gradient(U)
            for t in range(TICKS):
                rt.rt_tick(U, L, t, UD, acc, photon_total=Q, ledger=ledger)
        else:
            free = torch.empty_like(U)
            for _ in range(STEPS):
                U = rt.step(U, L, photon_total=Q, ledger=ledger, U_unguarded=free)
            assert torch.equal(U[..., 0], free[..., 0].clamp(min=0))
        rt.rt_sync()
        kind = "tick" if ticks else "transport"
        want = set(ROUTES[precision, n][groups - 1].split())
        if solver == "hll":
            want -= {"three_waves"}
        assert {r for r in NAMES if rt.rt_get_timing(f"{kind}/{r}")[1] > 0} == want
        assert rt.rt_get_timing(f"{kind}/{sorted(want)[0]}")[1] == (TICKS if ticks else STEPS)
        ref, pend, Qo, lo = reference(n, solver, surfaces, ticks)
        ref = ref[:, :groups]
        err = local_err(unsort(U.double().cpu().numpy(), p), ref, geo.sptr, geo.sidx)
        assert err < tol, (solver, surfaces, ticks, err)
        worst = max(worst, err)
        assert np.allclose(Q.cpu().numpy(), Qo[:groups], rtol=0.1 * tol, atol=0)
        if ticks:
            got = unsort(acc.cpu().numpy(), p)
            assert np.abs(got).max() > 0
            assert np.abs(got - pend[:, :groups]).max() < tol * np.abs(ref).max() * geo.V.max()
        if precision == "fp64":
            assert np.allclose(ledger.cpu().numpy(), lo[:groups], rtol=1e-10, atol=1e-14)
    log(f"{precision} n={n} G={groups} {ROUTES[precision, n][groups - 1]}: worst local error {worst:.1e}")
