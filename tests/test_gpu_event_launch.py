"""The event kernel's automatic launch: 4 waves per block while that is at most one block per
CU, then one block per CU whose waves (5 up to a full CU) draw chunks of 64 events from a
counter.  Every quantity is an exact sum, so it must give the bytes of single-wave blocks at
the sizes where its shape changes: one block more than the CUs, the first 5-wave block, the
largest block, a chunk count that no wave count divides, and more events per block than one
stretch between carries."""
import pytest

import workloads as W
from test_gpu_parity import run_schedule

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1503_06182_amd as P
    return P


@pytest.mark.parametrize("name,n", [("dy_z", 2), ("dy_z", 65_536), ("dy_z", 65_537), ("w_plus", 81_921),
                                    ("ww_4l", 196_609), ("ww_had", 196_671), ("w_plus", 1_048_577),
                                    ("ww_had", 1_300_003), ("w_plus", 8_400_001)])
def test_automatic_launch_gives_the_same_bytes(P, name, n):
    cfg = W.config(name)
    assert run_schedule(P, cfg, n, 2) == run_schedule(P, cfg, n, 2, waves_per_block=1, max_blocks=997)
