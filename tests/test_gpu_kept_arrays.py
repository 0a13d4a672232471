"""The arrays that a context keeps from build to build, over builds that need
longer ones (a clump's neighbour table is several times a lattice's: new arrays),
shorter ones and a few slots more (the same arrays), and over blocks with larger
unions coming and going.  Each build equals that of a new context bit for bit."""
import pytest
import torch

import workloads
from tests.gpu_util import dev, log
from tests.test_gpu_rebuild import outputs
from tests.test_gpu_search import clump_set

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2302_12727_amd import RT  # noqa: E402


@pytest.mark.parametrize("precision,groups", [("fp64", 3), ("fp32c", 4)])
def test_tables_grow_and_are_kept(precision, groups):
    n = 1400
    lattice, other = (dev(workloads.jittered_lattice(12, 0.1, s)[:n]) for s in (5, 6))
    clump = dev(clump_set(10, 400, 3))
    g = torch.Generator(device="cuda").manual_seed(1)
    U = torch.rand((n, groups, 4), generator=g, device="cuda", dtype=torch.float64) * 0.2
    U[..., 0] += 0.8
    U = U.to(torch.float64 if precision == "fp64" else torch.float32)
    rt, slots, held, staged = RT(n, groups, precision=precision), [], [], []
    for x in (lattice, clump, other, clump, lattice):
        got, st = outputs(rt, x, U)
        held.append(rt.rt_get_stats()["device_bytes"])
        fresh, fst = outputs(RT(n, groups, precision=precision), x, U)
        slots.append(st["sell_slots"])
        staged.append(st["union_staged_blocks"])
        assert st == fst
        for a, b in zip(got, fresh):
            assert torch.equal(a, b)
    log(f"{precision} G={groups}: slots {slots}, bytes held {held}, blocks over the capacity {staged}")
    assert slots[1] > 2 * slots[0] and slots[2] < slots[1] and slots[2] != slots[0]
    assert held[1] > held[0] and held[1] == held[2] == held[3] == held[4]
    assert [s > 0 for s in staged] == [False, True, False, True, False]
