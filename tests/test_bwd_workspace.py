"""The backward's workspace: the part every call needs is linear in the tokens and is
accepted, whatever the batch (so one workspace, sized for the largest batch, serves
smaller ones); the partial sums of cut key tiles and the stored dS are used where there
is room.  Acceptance and sizes on the CPU (a call with a NULL workspace is refused for
its size before its pointer is looked at), modes and results on the GPU."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import pp_oracle as orc
from paper_2602_24082_amd import binding as pp
from paper_2602_24082_amd import workload as wl
from gradcheck import check_grad

MIB = 1 << 20


def _align(n):
    return (n + 255) // 256 * 256


def _accepts(pack, hq, hkv, d, nbytes, dtype=pp.PP_BF16):
    fake = ctypes.c_void_p(256)  # never dereferenced: a NULL workspace is an error
    h = pp._DescHolder(pack)
    st = pp.lib().pp_attn_bwd(h.ref, dtype, hq, hkv, d, 0.0, *[fake] * 9, None, nbytes, None)
    assert pp.STATUS[st] in ("PP_ERR_WORKSPACE_TOO_SMALL", "PP_ERR_INVALID_ARGUMENT")
    plan = ctypes.c_void_p()
    fwd = _align(pp.pp_workspace_size(pack, hq, hkv, d, bwd=False, loss=False, dtype=dtype)[0])
    st2 = pp.lib().pp_plan_create(h.ref, dtype, hq, hkv, d, None, None, fwd + nbytes, None, ctypes.byref(plan))
    assert st2 == st and not plan.value
    return pp.STATUS[st] != "PP_ERR_WORKSPACE_TOO_SMALL"


def _linear_bytes(pack, hq, hkv, d, dtype=pp.PP_BF16):
    """The regions of an uncut recompute backward, counted from the dense mask."""
    T, B = pack.total_tokens, pack.num_rows
    q_tiles = entries = k_tiles = blocks = 0
    for b in range(B):
        n, K = int(pack.row_start[b + 1] - pack.row_start[b]), int(pack.num_resp[b])
        mask = orc.row_mask(n, int(pack.prompt_len[b]), [int(x) for x in pack.resp_off[b, :K]],
                            [int(x) for x in pack.resp_len[b, :K]])
        q_tiles += -(-n // 128)
        k_tiles += -(-n // 128)
        blocks += -(-n // 32)
        for q0 in range(0, n, 128):
            entries += sum(mask[q0:q0 + 128, k0:k0 + 64].any() for k0 in range(0, n, 64))
    copies = 2 * (_align(2 * T * hq * d) + _align(2 * T * hkv * d)) if dtype == pp.PP_FP32 else 0
    return (2 * _align(4 * T) + _align(32 * q_tiles) + _align(8 * entries) + _align(32 * k_tiles) + _align(4 * B)
            + _align(8 * blocks) + _align(4 * T) + _align(4 * d) + 2 * _align(4 * hq * T) + copies)


CUT = [(([1100], [[300, 129]], [0]), 8, 2, 128), (([640], [[65, 0, 190]], [33]), 16, 4, 64),
       (([300], [[60, 40]], [0]), 32, 8, 128), (([1500, 40], [[200, 100], [7, 3]], [0, 0]), 14, 2, 64)]


@pytest.mark.parametrize("dtype", [pp.PP_BF16, pp.PP_FP32])
@pytest.mark.parametrize("rows,hq,hkv,d", CUT)
def test_linear_part_is_enough(rows, hq, hkv, d, dtype):
    pack = wl.make_pack(rows[0], rows[1], pad=rows[2])
    need = _linear_bytes(pack, hq, hkv, d, dtype)
    assert pp.pp_workspace_size(pack, hq, hkv, d, fwd=False, loss=False, dtype=dtype)[1] > need  # has partial sums
    assert _accepts(pack, hq, hkv, d, need, dtype)
    assert not _accepts(pack, hq, hkv, d, need - 1, dtype)


def test_largest_batch_sizes_all():
    """32/8 heads of 128: the workspace of 8 such rows serves 1, 2 and 4 of them."""
    packs = {n: wl.make_pack([1500] * n, [[300, 311]] * n) for n in (1, 2, 4, 8)}
    room = pp.pp_workspace_size(packs[8], 32, 8, 128, fwd=False, loss=False)[1]
    for n, pack in packs.items():
        assert _accepts(pack, 32, 8, 128, room), n


def test_partial_sums_are_bounded():
    """At most 768 tiles of 128 keys of one kv-head, with few records beside them."""
    rng = np.random.default_rng(79)
    seen = 0
    heads = [(32, 8), (56, 8), (28, 4), (14, 2), (8, 1), (8, 8), (64, 64), (40, 40)]
    packs = [wl.make_pack([5183, 20, 30], [[118, 167], [5], [9, 3]]), wl.make_pack([11653], [[200, 300]])]
    for i in range(60):
        B = int(rng.integers(1, 4))
        P = [int(rng.integers(1, int(rng.choice([200, 2000, 9000])))) for _ in range(B)]
        packs.append(wl.make_pack(P, [rng.integers(1, 600, size=int(rng.integers(1, 4))).tolist() for _ in range(B)]))
    for i, pack in enumerate(packs):
        for hq, hkv in heads if i < 2 else [heads[i % len(heads)]]:
            d = 64 if i % 2 else 128
            T = pack.total_tokens
            both = pp.pp_bwd_stored_ds_workspace_size(pack, hq, hkv, d)[0]
            want = pp.pp_workspace_size(pack, hq, hkv, d, fwd=False, loss=False)[1]
            lo, hi = 0, want
            while lo < hi:  # the least that is accepted
                mid = (lo + hi) // 2
                lo, hi = (lo, mid) if _accepts(pack, hq, hkv, d, mid) else (mid + 1, hi)
            assert lo <= want <= lo + 768 * 2 * 128 * d * 4 + 768 * 72 + 768
            assert lo <= 8 * hq * T + 80 * T + 8 * (T // 128 + pack.num_rows) * (T // 64 + 1) + 8192
            assert both > want
            seen += want > lo
    assert seen > 20


def _names(run):
    pp.pp_timing_reset()
    pp.pp_timing_enable(True)
    try:
        out = run()
        return out, set(pp.pp_timing_get())
    finally:
        pp.pp_timing_enable(False)
        pp.pp_timing_reset()


@pytest.mark.gpu
@pytest.mark.parametrize("rows,hq,hkv,d", CUT)
def test_modes_by_room(rows, hq, hkv, d):
    pack = wl.make_pack(rows[0], rows[1], pad=rows[2])
    need = _linear_bytes(pack, hq, hkv, d)
    lean = pp.pp_workspace_size(pack, hq, hkv, d, fwd=False, loss=False)[1]
    both = pp.pp_bwd_stored_ds_workspace_size(pack, hq, hkv, d)[0]
    stored = need + both - lean
    q, k, v, do = wl.qkv(pack, hq, hkv, d, 950, torch.bfloat16, device="cuda:0")
    o, lse = pp.pp_attn_fwd(pack, q, k, v)
    ref = orc.attn_bwd(*pack.oracle_args(), *(x.double().cpu().numpy() for x in (q, k, v, do)))
    fwd = _align(pp.pp_workspace_size(pack, hq, hkv, d, bwd=False, loss=False)[0])
    sums_first = lean >= stored  # the sums are larger than dS: with room for one of them they are taken
    for room, cut, store in ((need, False, False), (min(lean, stored) - 1, False, False), (lean, True, False),
                             (stored, False, True), (max(lean, stored), sums_first, not sums_first),
                             (both - 1, sums_first, not sums_first), (both, True, True)):
        print(f"backward workspace T={pack.total_tokens} d={d} room={room} cut={cut} stored={store}", flush=True)
        ws = torch.full((room + 256,), 0x7f, dtype=torch.uint8, device="cuda:0")
        got, names = _names(lambda: pp.pp_attn_bwd(pack, q, k, v, o, lse, do, ws=ws[:room]))
        assert ("pp_attn_bwd_kv_combine" in names, "pp_attn_bwd_prep" in names) == (cut, store)
        assert (ws[room:] == 0x7f).all()
        for name, g, r in zip(("dq", "dk", "dv"), got, ref):
            check_grad(pack, name, g.double().cpu().numpy(), r)
        plan_ws = torch.empty(fwd + room, dtype=torch.uint8, device="cuda:0")
        plan = pp.pp_plan_create(pack, hq, hkv, d, device="cuda:0", ws=plan_ws)
        for a, b in zip(got, pp.pp_attn_bwd_planned(plan, q, k, v, o, lse, do)):
            assert torch.equal(a, b)
