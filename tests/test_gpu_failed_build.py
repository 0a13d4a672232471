"""A build that fails after one that succeeded: its context reports no unions and
no task lists of the build before, and builds again afterwards."""
import pytest
import torch

import workloads
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2302_12727_amd import RT  # noqa: E402
from paper_2302_12727_amd.rt import RTError  # noqa: E402

BUILT = ["union_blocks", "union_staged_blocks", "adj_union_blocks", "adj_union_staged_blocks",
         "task_longest", "task_bound"]


def test_failed_build_reports_nothing_of_the_last():
    x = dev(workloads.jittered_lattice(10, 0.1, 3))
    rt = RT(x.shape[0], 3)
    rt.rt_build_cells(x)
    good = rt.rt_get_stats()
    assert good["union_blocks"] > 0 and good["adj_union_blocks"] > 0 and good["task_longest"] > 0
    with pytest.raises(RTError, match="RT_EINVAL"):     # support beyond half the box
        rt.rt_build_cells(x, torch.full((x.shape[0],), 0.5, dtype=torch.float64, device="cuda"))
    bad = rt.rt_get_stats()
    assert [bad[k] for k in BUILT] == [0] * len(BUILT)
    rt.rt_build_cells(x)
    again = rt.rt_get_stats()
    assert [again[k] for k in BUILT] == [good[k] for k in BUILT]
