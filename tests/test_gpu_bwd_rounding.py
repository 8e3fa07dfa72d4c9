"""GPU test of the key-major pass's rounding at head size 128: dP is summed first and
delta subtracted from it once, so a sum of small products is not lost against a large
delta.

Two prompt tokens, keys of zeros (S = 0) and lse = 0 make query 1's P exactly 1, dout
of ones and o = (2^24, 3 * 2^16, 0, ...) make its delta D = 2^24 + 3 * 2^16, half way
between two bf16 values.  v_0 holds 0.75 once in every 16 columns, so dP = 6 and dS =
6 - D, which fp32 holds exactly and bf16 rounds to -(2^24 + 2^17); were the products
added one by one to -D, each would be less than half a unit in its last place (2) and
vanish, and the tie -D would round to the even neighbour -(2^24 + 2^18).  q_1 = (1, 0,
...) carries dS to the first element of dK_0."""
import pytest
import torch

from paper_2602_24082_amd import binding as pp
from paper_2602_24082_amd import workload as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("store_ds", [False, True])
def test_delta_is_subtracted_once(store_ds):
    pack, d = wl.make_pack([2], [[]]), 128
    zeros = lambda: torch.zeros(2, 1, d, dtype=torch.bfloat16, device=DEV)
    q, k, v, o, do = (zeros() for _ in range(5))
    q[1, 0, 0] = 1
    v[0, 0, ::16] = 0.75
    o[1, 0, 0], o[1, 0, 1] = 2.0 ** 24, 3 * 2.0 ** 16
    do[1] = 1
    lse = torch.zeros(1, 2, device=DEV)
    _, dk, _ = pp.pp_attn_bwd(pack, q, k, v, o, lse, do, scale=1.0, store_ds=store_ds)
    assert float(dk[0, 0, 0]) == -(2.0 ** 24 + 2.0 ** 17)
