"""A context built again for moved particles keeps its arrays: whatever it was
built for before, and on whichever stream, it holds what a new context holds,
bit for bit (longer and shorter neighbour tables, blocks left to the staged
gradient in one build and none in the other)."""
import pytest
import torch

import workloads
from tests.gpu_util import dev, log
from tests.test_gpu_search import clump_set

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2302_12727_amd import RT  # noqa: E402


def outputs(rt, x, U):
    perm, h, V, dt = rt.rt_build_cells(x)
    ptr, idx = rt.rt_get_neighbours()
    Us = U[perm.long()].contiguous()
    UD = rt.rt_gradient(Us)
    out = [perm, h, V, dt, ptr, idx, UD, rt.rt_transport(UD)]
    if rt.precision == "fp64":
        out.append(rt.rt_adjoint(Us, None, Us))
    st = rt.rt_get_stats()
    return [t.clone() for t in out], {k: v for k, v in st.items() if not k.startswith("device")}


@pytest.mark.parametrize("precision,groups", [("fp64", 3), ("fp64", 5), ("fp32c", 4)])
def test_second_build_equals_a_new_context(precision, groups):
    n = 1400
    # 1000 lattice particles about a clump of 400, an even lattice, the first again
    xs = [dev(clump_set(10, 400, 3)), dev(workloads.jittered_lattice(12, 0.1, 5)[:n]),
          dev(clump_set(10, 400, 3))]
    g = torch.Generator(device="cuda").manual_seed(1)
    U = torch.rand((n, groups, 4), generator=g, device="cuda", dtype=torch.float64)
    U = (U * torch.tensor([1.0, 0.2, 0.2, 0.2], device="cuda", dtype=torch.float64))
    U = U.to(torch.float64 if precision == "fp64" else torch.float32)
    again = RT(n, groups, precision=precision)
    other = torch.cuda.Stream()
    for k, x in enumerate(xs):
        fresh, fst = outputs(RT(n, groups, precision=precision), x, U)
        other.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(other if k == 1 else torch.cuda.current_stream()):
            got, gst = outputs(again, x, U)
        torch.cuda.synchronize()
        log(f"{precision} G={groups} build {k}: {gst['sell_slots']} slots, "
            f"{gst['union_staged_blocks']} blocks staged")
        assert gst == fst
        for a, b in zip(got, fresh):
            assert torch.equal(a, b)
