"""The staging launch's grid: metadata copy, conversions of fp32 inputs and zeros share one
launch, which must stay below 2^32 threads for every batch a call takes (CPU), and a
conversion of more vectors than its blocks have threads is walked in strides (GPU)."""
import ctypes

import pytest
import torch

from paper_2602_24082_amd import binding as pp
from paper_2602_24082_amd import workload as wl

THREADS, CAST_BLOCKS = 256, 1 << 20


def _blocks(nbytes, casts, zeros):
    import host_records
    out = (ctypes.c_int32 * 4)()
    total = host_records.lib().rec_stage_blocks(ctypes.c_int64(nbytes), (ctypes.c_int64 * 4)(*casts), ctypes.c_int64(zeros), out)
    return total, list(out)


@pytest.mark.parametrize("nbytes,casts,zeros", [
    (0, (0, 0, 0, 0), 0), (1, (0, 0, 0, 0), 0), (4097, (1, 1024, 1025, 0), 0), (0, (0, 0, 0, 0), (1 << 31) - 1),
    # a backward of 1.06 million tokens of 64 / 8 heads of 128 in fp32: 19.5e9 values, 4.9e9 threads of 4
    (1 << 27, (1060000 * 64 * 128, 1060000 * 8 * 128, 1060000 * 8 * 128, 1060000 * 64 * 128), 0),
    (1 << 32, (1 << 36, 1 << 36, 1 << 36, 1 << 36), (1 << 31) - 1)])
def test_a_launch_holds_all_of_it(nbytes, casts, zeros):
    total, got = _blocks(nbytes, casts, zeros)
    assert total * THREADS < 1 << 32
    want = [min(-(-(-(-n // 4)) // THREADS), CAST_BLOCKS) for n in casts]
    assert got == want
    assert total == sum(want) + -(-max(nbytes // 16, nbytes % 16) // THREADS) + -(-zeros // THREADS)


@pytest.mark.gpu
def test_conversion_in_strides():
    """Rows of 61 tokens, 1.2e9 query values in fp32 (more than 2^20 blocks of 1024): the
    last rows come out as on their own."""
    n, hq, hkv, d, DEV = 2400, 64, 8, 128, "cuda:0"
    pack, few = wl.make_pack([41] * n, [[12, 8]] * n), wl.make_pack([41] * 3, [[12, 8]] * 3)
    T, t = pack.total_tokens, few.total_tokens
    assert T * hq * d > CAST_BLOCKS * THREADS * 4
    print(f"staging fp32 T={T}", flush=True)
    q = torch.randn(T, hq, d, device=DEV)
    k, v = torch.randn(T, hkv, d, device=DEV), torch.randn(T, hkv, d, device=DEV)
    o, lse = pp.pp_attn_fwd(pack, q, k, v)
    for at in (0, T // 2 // 61 * 61, T - t):
        s = slice(at, at + t)
        o1, lse1 = pp.pp_attn_fwd(few, q[s].contiguous(), k[s].contiguous(), v[s].contiguous())
        assert torch.equal(o[s], o1) and torch.equal(lse[:, s], lse1)
