"""GPU test of the timing names of launches that do several jobs: selected by any of its
jobs, such a launch is timed, under that name; with nothing selected each launch is one
entry."""
import pytest
import torch

from paper_2602_24082_amd import binding as pp
from paper_2602_24082_amd import workload as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _calls(what):
    pack = wl.make_pack([9, 4], [[5, 3], [2, 6]])
    T = pack.total_tokens
    if what == "rm":
        h, w = wl.randn((T, 64), 980, torch.float32, DEV), wl.randn((64,), 981, torch.float32, DEV)
        return lambda: pp.pp_rm_scores_bwd(pack, h, w, torch.ones(2, 2, device=DEV))
    if what == "attn_fp32":
        q, k, v, _ = wl.qkv(pack, 4, 2, 64, 982, torch.float32, device=DEV)
        return lambda: pp.pp_attn_fwd(pack, q, k, v)
    x, tok = wl.randn((T, 50), 983, torch.float32, DEV), wl.randint((T,), 50, 984, DEV)
    return lambda: pp.pp_seq_logprob(pack, x, tok, want_tok=True)


@pytest.mark.parametrize("what,names,first", [
    ("rm", ["pp_stage", "pp_rm_dhidden", "pp_rm_dw"], {"pp_stage", "pp_rm_dhidden"}),
    ("attn_fp32", ["pp_stage", "pp_to_bf16", "pp_attn_fwd"], {"pp_stage", "pp_attn_fwd"}),
    ("logprob", ["pp_stage", "pp_fill_zero", "pp_segsum"], {"pp_stage", "pp_logprob_rows", "pp_segsum"})])
def test_names_of_shared_launches(what, names, first):
    call = _calls(what)
    pp.pp_timing_enable(True)
    try:
        for select in [None] + names:
            pp.pp_timing_select([select] if select else None)
            pp.pp_timing_reset()
            call()
            got = pp.pp_timing_get()
            assert set(got) == ({select} if select else first), select
            assert all(n == 1 and ms > 0 for ms, n in got.values())
    finally:
        pp.pp_timing_enable(False)
        pp.pp_timing_select(None)
        pp.pp_timing_reset()
