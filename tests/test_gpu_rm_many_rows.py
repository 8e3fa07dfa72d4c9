"""GPU test of the reward head's backward at the most flat rows that a launch of one
workgroup a row would hold without the workgroups of dw and dbias: the last rows' gradients
are written too."""
import pytest
import torch

from paper_2602_24082_amd import binding as pp
from paper_2602_24082_amd import workload as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def test_rows_up_to_a_launch():
    T, H = (1 << 24) - 1, 8
    pack = wl.make_pack([T - 9], [[4, 5]])
    print(f"rm backward T={T} H={H}", flush=True)
    h, w = torch.ones(T, H, dtype=torch.bfloat16, device=DEV), torch.arange(1, H + 1, device=DEV).bfloat16()
    g = torch.tensor([[0.5, -2.0]], device=DEV)
    dh, dw, db = pp.pp_rm_scores_bwd(pack, h, w, g)
    at = [T - 6, T - 1]
    assert torch.equal(dh[at].float(), g[0][:, None] * w.float())
    dh[at] = 0
    assert int(torch.count_nonzero(dh)) == 0
    assert torch.equal(dw, torch.full((H,), -1.5, device=DEV)) and float(db) == -1.5
