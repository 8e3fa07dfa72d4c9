"""GPU tests of the dK/dV pass on batches that leave compute units idle, whose
long key tiles are cut into several work items with fp32 partial sums: against
the oracle at the attention gradient bar, and the same bits on every run."""
import pytest
import torch

from oracle import pp_oracle as orc
from paper_2602_24082_amd import binding as pp
from paper_2602_24082_amd import workload as wl
from gradcheck import check_grad

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# one row whose first tiles outlast all others; a tile edge, an empty response and
# padding; two rows with the cut tiles in one of them; no head sharing
CASES = [
    ((1100,), [[300, 129]], [0], 128, 8, 2),
    ((640,), [[65, 0, 190]], [33], 64, 16, 4),
    ((1025, 40), [[1, 63], [20, 7]], [0, 5], 128, 4, 1),
    ((1500,), [[200, 100]], [0], 64, 3, 3),
]


@pytest.mark.parametrize("mode", ["plain", "rope", "stored", "fp32"])
@pytest.mark.parametrize("prompts,resps,pad,d,hq,hkv", CASES)
def test_cut_key_tiles_match_oracle(prompts, resps, pad, d, hq, hkv, mode):
    pack = wl.make_pack(prompts, resps, pad=pad)
    print(f"kv split T={pack.total_tokens} d={d} hq={hq} hkv={hkv} {mode}", flush=True)
    dt = torch.float32 if mode == "fp32" else torch.bfloat16
    code = pp.PP_FP32 if mode == "fp32" else pp.PP_BF16
    # the partial sums are the part of the workspace that grows with the cuts
    flat = pack.total_tokens * hq * 8 + (pack.total_tokens * (2 * hq + 2 * hkv) * d * 2 if mode == "fp32" else 0)
    ws = pp.pp_workspace_size(pack, hq, hkv, d, fwd=False, bwd=True, loss=False, dtype=code)[1]
    assert ws > flat + 2 * hkv * 2 * 128 * d * 4
    q, k, v, do = wl.qkv(pack, hq, hkv, d, 900, dt, device="cpu")
    qg, kg, vg, dog = (x.to(DEV) for x in (q, k, v, do))
    args = pack.oracle_args()
    base = 10000.0
    if mode == "rope":
        o, lse, qg, kg = pp.pp_attn_fwd_rope(pack, qg, kg, vg, base)
        run = lambda: pp.pp_attn_bwd_rope(pack, qg, kg, vg, o, lse, dog, base)
    else:
        o, lse = pp.pp_attn_fwd(pack, qg, kg, vg)
        run = lambda: pp.pp_attn_bwd(pack, qg, kg, vg, o, lse, dog, store_ds=mode == "stored")
    got = run()
    # what the kernels attend with: the rotated or given q and k
    qn, kn = qg.double().cpu().numpy(), kg.double().cpu().numpy()
    ref = list(orc.attn_bwd(*args, qn, kn, v.double().numpy(), do.double().numpy()))
    if mode == "rope":
        ref[0], ref[1] = (orc.pack_rope(*args, x, base, inverse=True) for x in ref[:2])
    for name, g, r in zip(("dq", "dk", "dv"), got, ref):
        check_grad(pack, name, g.double().cpu().numpy(), r)
    for a, b in zip(got, run()):
        assert torch.equal(a, b)
