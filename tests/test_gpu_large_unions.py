"""Gradients of blocks whose neighbour union is over the small capacity, staged
as a larger one (up to 1024 rows, a few blocks only) or per pair: group by group
against a 5-group context, which stages every block per pair.

The FP32C sums are formed in one order on every path, so they are equal bit for
bit.  FP64: sums of up to 450 terms in two orders differ by 450 * 2^-53 = 5e-14
of the sum of their magnitudes, which is at most 2 max|U| / (h E) with the
matrix's condition (about 10 here): 1e-12 of the largest record."""
import pytest
import torch

import workloads
from tests.gpu_util import dev, log
from tests.test_gpu_search import clump_set

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2302_12727_amd import RT  # noqa: E402


def sets(name):
    if name == "clump":                         # unions of over 1024 rows too
        return clump_set(10, 400, 3)
    return workloads.config(4, scale=(1 << 14) / (1 << 24)).x


@pytest.mark.parametrize("name", ["clump", "plummer"])
@pytest.mark.parametrize("precision,groups", [("fp64", 2), ("fp64", 3), ("fp64", 4),
                                              ("fp32c", 2), ("fp32c", 3), ("fp32c", 4)])
def test_large_unions(name, precision, groups):
    x = sets(name)
    n = x.shape[0]
    g = torch.Generator(device="cuda").manual_seed(9)
    U = torch.rand((n, 5, 4), generator=g, device="cuda", dtype=torch.float64) - 0.2
    U = U.to(torch.float64 if precision == "fp64" else torch.float32)
    out = []
    for G in (groups, 5):
        rt = RT(n, G, precision=precision)
        rt.rt_build_cells(dev(x))
        out.append(rt.rt_gradient(U[:, :G].contiguous())[:, :groups])
        if G == groups:
            over = rt.rt_get_stats()["union_staged_blocks"]
    a, b = out
    log(f"{name} {precision} G={groups}: {over} blocks over the capacity")
    if precision == "fp32c":
        assert torch.equal(a, b)
    else:
        assert float((a - b).abs().max()) <= 1e-12 * float(b.abs().max())
