"""Gradients of blocks whose neighbour union is over the small capacity, on sets
that are known to reach each path: unions between that capacity and 1024 rows
(staged as larger ones), over 1024 rows too (both those and blocks staged per
pair), and more such blocks than the larger unions serve (all of them per pair).
The number of rows of every block's union is counted from the neighbour lists,
and the routes taken are read from the launch records.

Group by group against a 5-group context, which stages every block per pair:
FP32C sums are formed in one order on every path, so they are equal bit for bit.
FP64: sums of up to 600 terms in two orders differ by 600 * 2^-53 = 7e-14 of the
sum of their magnitudes, at most 2 max|U| / (h E) with the matrix's condition
(about 10 here): 1.5e-12 of the largest record."""
import numpy as np
import pytest
import torch

import workloads
from tests.gpu_util import dev, log

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2302_12727_amd import RT  # noqa: E402

CAPACITY = {("fp64", 2): 880, ("fp64", 3): 640, ("fp64", 4): 512,
            ("fp32c", 2): 880, ("fp32c", 3): 672, ("fp32c", 4): 576}
MOST = {"fp64": 256, "fp32c": 512}              # blocks served by larger unions
SETS = {                                        # positions, eta, routes of 2 to 4 groups
    "lattice": (lambda: workloads.jittered_lattice(17, 0.2, 2), 1.8, {"large", "staged"}),
    "plummer": (lambda: workloads.config(4, scale=(1 << 13) / (1 << 24)).x, 1.5, {"large"}),
    "tight plummer": (lambda: workloads.config(4, scale=(1 << 13) / (1 << 24)).x, 1.6,
                      {"large", "staged"}),
    "many": (lambda: workloads.jittered_lattice(33, 0.2, 2), 2.2, {"staged"}),
}


def union_rows(rt):
    """Distinct gather neighbours and own particles of every 64 particles."""
    ptr, idx = (t.cpu().numpy() for t in rt.rt_get_neighbours())
    _, _, ng = rt.rt_get_geometry()
    ng = ng.cpu().numpy()
    rows = []
    for b in range(0, rt.n, 64):
        own = np.arange(b, min(b + 64, rt.n))
        rows.append(np.unique(np.concatenate([own] + [idx[ptr[i]:ptr[i] + ng[i]] for i in own])).size)
    return np.array(rows)


def routes(rt, name):
    return {r for r in ("large", "staged") if rt.rt_get_timing(f"{name}/{r}")[1] > 0}


@pytest.mark.parametrize("name,ticks", [("lattice", False), ("plummer", False), ("plummer", True),
                                        ("tight plummer", False), ("tight plummer", True),
                                        ("many", False)])
@pytest.mark.parametrize("precision", ["fp64", "fp32c"])
def test_larger_unions(name, ticks, precision):
    make, eta, want = SETS[name]
    x = dev(make())
    n = x.shape[0]
    g = torch.Generator(device="cuda").manual_seed(9)
    U = torch.rand((n, 5, 4), generator=g, device="cuda", dtype=torch.float64) - 0.2
    U = U.to(torch.float64 if precision == "fp64" else torch.float32)
    out = {}
    for G in (5, 2, 3, 4):
        rt = RT(n, G, precision=precision, eta=eta)
        rt.rt_build_cells(x)
        V = U[:, :G].contiguous()
        rt.rt_timing(True)
        if ticks:                               # the records of the particles that end a step
            _, cycle = rt.rt_time_bins(3)
            assert cycle > 1
            UD = torch.zeros((n, G, 16), dtype=V.dtype, device="cuda")
            UD[:, :, :4] = V
            rt.rt_tick(V.clone(), None, 0, UD, torch.zeros(V.shape, dtype=torch.float64, device="cuda"))
            out[G] = UD[:, :, 4:]
            assert bool((out[G] == 0).all(dim=(1, 2)).any()) and bool(out[G].any())
        else:
            out[G] = rt.rt_gradient(V)
        took = routes(rt, "tick" if ticks else "gradient")
        if G == 5:
            rows = union_rows(rt)
            assert not took
            continue
        cap = CAPACITY[precision, G]
        over = int((rows > cap).sum())
        log(f"{name} {precision} G={G}: {over} of {rows.size} unions over {cap} rows, "
            f"{int((rows > 1024).sum())} over 1024; {took}")
        assert rt.rt_get_stats()["union_staged_blocks"] >= over > 0
        assert (over > MOST[precision]) == (name == "many")
        assert (rows > 1024).any() == ("staged" in want)
        assert took == want
        if precision == "fp32c":
            assert torch.equal(out[G], out[5][:, :G])
        else:
            err = float((out[G] - out[5][:, :G]).abs().max() / out[5].abs().max())
            assert err <= 1.5e-12
