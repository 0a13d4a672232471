"""FP64 transport at the edges of its rules on the number of 64-particle tiles
(8 lanes a particle up to 256 blocks, three waves per SIMD for one group from 513
on, a block for every group of several up to 512, 768 and 1536 blocks) and the
photon totals at the edge of one block's rows (2048 tiles): a step against the
same step, group by group, in a 4-group context, which takes other kernels there
(one group a block of 4 lanes up to 192 tiles, then slices of 2 of 4 lanes).

Groups do not mix, the pair fluxes are the same instructions, and only the order
of the about 50 terms of a sum differs: a relative 50 * 2^-53 = 6e-15 of the
largest state of a neighbourhood, 1e-13 with the cancellation of a flux sum
(|phi| up to c A E / 2 per pair, sum dt A / V of order 10).  Totals are
compensated sums of positive numbers: 1e-15 each, 1e-13 with the difference of
the states.
"""
import pytest
import torch

import workloads
from tests.gpu_util import dev, log

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2302_12727_amd import RT  # noqa: E402


@pytest.mark.parametrize("n,groups,solver,surfaces", [
    (8129, 2, "glf", "hopkins"), (8192, 2, "hll", "ivanova"), (10900, 3, "glf", "hopkins"),
    (10945, 3, "hll", "hopkins"), (16384, 2, "glf", "ivanova"), (16384, 3, "glf", "hopkins"),
    (16385, 3, "glf", "hopkins"), (16383, 1, "hll", "ivanova"), (16321, 2, "hll", "hopkins"),
    (19648, 5, "glf", "hopkins"), (19649, 5, "glf", "hopkins"),
    (32768, 1, "glf", "hopkins"), (32769, 1, "glf", "hopkins"), (33000, 1, "glf", "ivanova"),
    (131072, 1, "glf", "hopkins"), (131073, 2, "glf", "hopkins"),
])
def test_small_and_wide_transports(n, groups, solver, surfaces):
    side = 5
    while side ** 3 < n:
        side += 1
    x = dev(workloads.jittered_lattice(side, 0.1, 7)[:n])
    g = torch.Generator(device="cuda").manual_seed(3)
    U = torch.rand((n, 5, 4), generator=g, device="cuda", dtype=torch.float64)
    U[..., 1:] = 0.5 * (U[..., 1:] - 0.5)
    out, m = [], min(groups, 4)
    for G, cols in ((groups, U[:, :groups]), (4, U[:, :4])):
        rt = RT(n, G)
        rt.rt_build_cells(x)
        rt.rt_set_riemann(solver)
        rt.rt_set_surfaces(surfaces)
        Q = torch.empty(G, dtype=torch.float64, device="cuda")
        ledger = torch.zeros(G, dtype=torch.float64, device="cuda")
        counts = torch.zeros(4, dtype=torch.int64, device="cuda")
        UD = rt.rt_gradient(cols.contiguous())
        V = rt.rt_transport(UD, photon_total=Q, counts=counts, ledger=ledger)
        out.append((V[:, :m], Q[:m], ledger[:m]))
    (a, qa, la), (b, qb, lb) = out
    err = float((a - b).abs().max() / b.abs().max())
    qerr = float(((qa - qb) / qb).abs().max())
    log(f"n={n} G={groups} {solver} {surfaces}: states {err:.1e}, totals {qerr:.1e}")
    assert err < 1e-13 and qerr < 1e-13
    assert float((la - lb).abs().max()) < 1e-13 * float(qb.max())


@pytest.mark.parametrize("n,groups,solver,surfaces", [
    (2000, 2, "glf", "hopkins"), (2000, 3, "hll", "ivanova"), (21824, 3, "glf", "hopkins"),
    (21889, 3, "glf", "hopkins"), (16384, 4, "glf", "ivanova"), (16385, 4, "hll", "hopkins"),
    (19648, 5, "glf", "hopkins"), (19649, 5, "glf", "hopkins"),
])
@pytest.mark.parametrize("ticks", [False, True])
def test_fp32c_groups_keep_their_bits(n, groups, solver, surfaces, ticks):
    """FP32C: a group's sums are formed in one order wherever it runs, pair-once
    up to 3 groups and two-sided above: in a block of its own up to 1024 blocks
    (1536 of more than 4 groups), else with others in one wave.  So it is, bit
    for bit, what it is in a context of one group (up to 3 groups), or of 3
    groups more (above), which crosses those lines elsewhere."""
    side = 5
    while side ** 3 < n:
        side += 1
    x = dev(workloads.jittered_lattice(side, 0.2, 7)[:n])
    g = torch.Generator(device="cuda").manual_seed(3)
    U = torch.rand((n, groups, 4), generator=g, device="cuda", dtype=torch.float64)
    U[..., 1:] = 0.5 * (U[..., 1:] - 0.5)
    U = U.float()
    out = []
    for V in ((U, U[:, :1]) if groups <= 3 else (U, torch.cat([U, U[:, :3]], 1))):
        G = V.shape[1]
        rt = RT(n, G, precision="fp32c")
        rt.rt_build_cells(x)
        rt.rt_set_riemann(solver)
        rt.rt_set_surfaces(surfaces)
        V = V.contiguous().clone()
        if ticks:
            _, cycle = rt.rt_time_bins(3)
            UD = rt.rt_gradient(V)
            acc = torch.zeros(V.shape, dtype=torch.float64, device="cuda")
            for t in range(cycle):
                rt.rt_tick(V, None, t, UD, acc)
        else:
            V = rt.rt_transport(rt.rt_gradient(V))
        out.append(V)
    m = min(groups, out[1].shape[1])
    assert torch.equal(out[0][:, :m], out[1][:, :m])
