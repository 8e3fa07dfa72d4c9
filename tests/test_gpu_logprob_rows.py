"""GPU tests of the log-prob kernels' row shapes: vocabularies at the edges of the
register-held shapes (512 x 8, 1024 x 8, 1024 x 19 and, for rows that start on no
16-byte boundary, 1024 x 18 vectors of 16 bytes) and of the form that streams what
1024 x 16 vectors do not hold, rows shorter than a vector, and matrices whose first row is itself off a boundary.
Labels sit on the first and last elements of the rows, where a head or tail element
belongs to one thread.  Against the oracle: the scores in fp32 sums (relative error
a few 1e-6 for 1e5 values, held to 1e-5 of the row's log-prob plus 1e-5), the
gradients as in test_gpu_logprob_bwd.py; and the gathered rows equal the dense ones
bit for bit, whatever boundaries they land on."""
import numpy as np
import pytest
import torch

from oracle import pp_oracle as orc
from paper_2602_24082_amd import binding as pp
from paper_2602_24082_amd import workload as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
RTOL = {torch.float32: 2e-5, torch.bfloat16: 5e-3}
BF, F32 = torch.bfloat16, torch.float32


def _at_offset(x, offset):
    """x on the GPU, contiguous, starting `offset` elements into an allocation."""
    flat = torch.full((x.numel() + offset,), float("nan"), dtype=x.dtype, device=DEV)
    y = flat[offset:].view(x.shape)
    y.copy_(x)
    return y


CASES = [(v, BF, 0) for v in (1, 7, 8, 9, 17, 4097, 32768, 32769, 32776, 65536, 65541, 147457, 147465, 155648, 155656)]
CASES += [(v, F32, 0) for v in (1, 3, 5, 9, 16385, 16388, 32769, 32773, 73729, 73733, 77824, 77828, 131075, 300000)]
CASES += [(4096, BF, 1), (4099, BF, 3), (32776, BF, 7), (4096, F32, 1), (73732, F32, 3)]


@pytest.mark.parametrize("V,dtype,offset", CASES)
def test_row_shapes(V, dtype, offset):
    print(f"logprob rows V={V} {dtype} offset={offset}", flush=True)
    pack = wl.make_pack([3, 1], [[4, 2], [1, 0, 3]], pad=[1, 0])
    T = pack.total_tokens
    logits = wl.randn((T, V), 910, dtype, "cpu", sigma=3.0)
    tokens = wl.randint((T,), V, 911, "cpu")
    edges = [0, V - 1, min(V - 1, 1), max(0, V - 2), min(V - 1, 7), max(0, V - 8)]
    tokens[:T] = torch.tensor([edges[i % len(edges)] if i % 3 else int(tokens[i]) for i in range(T)], dtype=torch.int32)
    dseq = wl.randn((pack.num_rows, pack.max_resp), 912, F32, "cpu")
    lg, tk, ds = _at_offset(logits, offset), tokens.to(DEV), dseq.to(DEV)
    args = pack.oracle_args()
    x = logits.double().numpy()

    seq, tok = pp.pp_seq_logprob(pack, lg, tk, want_tok=True)
    ref_seq, ref_tok = orc.seq_logprob(*args, x, tokens.numpy())
    for got, ref in ((seq, ref_seq), (tok, ref_tok)):
        assert np.abs(got.double().cpu().numpy() - ref).max() <= 1e-5 + 1e-5 * np.abs(ref).max()

    want = orc.seq_logprob_grad(*args, x, tokens.numpy(), dseq.double().numpy())
    dl = _at_offset(torch.full((T, V), float("nan"), dtype=dtype), offset)
    pp.pp_seq_logprob_bwd(pack, lg, tk, ds, dlogits=dl)
    got = dl.double().cpu().numpy()
    gmax = float(dseq.abs().max())
    assert (np.abs(got - want) - RTOL[dtype] * np.abs(want)).max() <= 1e-6 * gmax
    rows = orc.logprob_predicting_rows(*args)
    unused = np.setdiff1d(np.arange(T), rows)
    assert (got[unused] == 0).all()
    dr, ri = pp.pp_seq_logprob_bwd_rows(pack, lg, tk, ds)
    assert ri.cpu().tolist() == rows
    if offset == 0 or V % (16 // lg.element_size()):
        assert torch.equal(dr, dl[ri.long()])
