"""GPU tests of the pinned ring through which self-contained calls stage their plans: a
slot is held until the call's kernels are done, so a long call on one stream must not
stop calls on another, and more calls in flight than there are slots must each read
their own plan."""
import pytest
import torch

from paper_2602_24082_amd import binding as pp
from paper_2602_24082_amd import workload as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def test_a_long_call_holds_no_other_stream():
    long_pack, pack = wl.make_pack([6000] * 24, [[200, 200]] * 24), wl.make_pack([100], [[30, 20]])
    print(f"staging behind a long forward T={long_pack.total_tokens}", flush=True)
    q, k, v, _ = wl.qkv(long_pack, 64, 8, 128, 960, torch.bfloat16, device=DEV)
    x = wl.qkv(pack, 4, 2, 64, 961, torch.bfloat16, device=DEV)[:3]
    a, b = torch.cuda.Stream(device=DEV), torch.cuda.Stream(device=DEV)
    out, lse = torch.empty_like(q), torch.empty(64, long_pack.total_tokens, device=DEV)
    ws = torch.empty(pp.pp_workspace_size(long_pack, 64, 8, 128, bwd=False, loss=False)[0], dtype=torch.uint8, device=DEV)
    want = pp.pp_attn_fwd(pack, *x)
    with torch.cuda.stream(a):  # modules, allocations and pinned memory are there
        pp.pp_attn_fwd(long_pack, q, k, v, out=out, lse=lse, ws=ws)
    with torch.cuda.stream(b):
        got = [pp.pp_attn_fwd(pack, *x) for _ in range(12)]
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(a):
        pp.pp_attn_fwd(long_pack, q, k, v, out=out, lse=lse, ws=ws)
        done.record(a)
    with torch.cuda.stream(b):
        got = [pp.pp_attn_fwd(pack, *x) for _ in range(12)]
    early = not done.query()
    torch.cuda.synchronize()
    assert early, "12 short calls came back only after the long call of another stream had ended"
    for o, l in got:
        assert torch.equal(o, want[0]) and torch.equal(l, want[1])


def test_more_calls_in_flight_than_slots():
    packs = [wl.make_pack([40 + 9 * i], [[5 + i, 20 - i]]) for i in range(8)]
    xs = [wl.qkv(p, 4, 2, 64, 970 + i, torch.bfloat16, device=DEV)[:3] for i, p in enumerate(packs)]
    want = [pp.pp_attn_fwd(p, *x) for p, x in zip(packs, xs)]
    long_pack = wl.make_pack([6000] * 4, [[200, 200]] * 4)
    q, k, v, _ = wl.qkv(long_pack, 32, 8, 128, 962, torch.bfloat16, device=DEV)
    torch.cuda.synchronize()
    print("staging 48 calls in flight", flush=True)
    pp.pp_attn_fwd(long_pack, q, k, v)  # the rest queues up behind it
    got = [pp.pp_attn_fwd(packs[i % 8], *xs[i % 8]) for i in range(48)]
    torch.cuda.synchronize()
    for i, (o, l) in enumerate(got):
        assert torch.equal(o, want[i % 8][0]) and torch.equal(l, want[i % 8][1]), i
