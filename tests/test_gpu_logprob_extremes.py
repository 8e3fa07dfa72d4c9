"""GPU tests of the log-prob kernels on extreme logits, over every form a row can take
(all elements single ones; register-held; with a head and a tail off the 16-byte
boundaries; longer than the registers): masked entries of -inf or of the type's lowest
value, rows of nothing but the lowest value, the type's largest value, NaN and +inf, on
head and tail elements and in the part that is streamed.  Finite results are held to the
oracle with the bounds of test_gpu_logprob_rows.py; a NaN or +inf anywhere in a
predicting row makes that row's scores and gradient NaN and leaves the other rows alone."""
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
SHAPES = [(5, F32), (9, BF), (4096, F32), (4096, BF), (4099, F32), (4099, BF), (77831, F32), (131072, F32), (155661, BF),
          (163840, BF)]


def _inputs(V, dtype, seed):
    pack = wl.make_pack([3, 1], [[4, 2], [1, 0, 3]], pad=[1, 0])
    x = wl.randn((pack.total_tokens, V), seed, dtype, "cpu", sigma=3.0)
    tokens = wl.randint((pack.total_tokens,), V, seed + 1, "cpu")
    dseq = wl.randn((pack.num_rows, pack.max_resp), seed + 2, F32, "cpu")
    return pack, x, tokens, dseq


def _run(pack, x, tokens, dseq):
    lg, tk, ds = x.to(DEV), tokens.to(DEV), dseq.to(DEV)
    seq, tok = pp.pp_seq_logprob(pack, lg, tk, want_tok=True)
    dl = pp.pp_seq_logprob_bwd(pack, lg, tk, ds)
    dr, ri = pp.pp_seq_logprob_bwd_rows(pack, lg, tk, ds)
    assert torch.equal(dr.view(torch.uint8), dl[ri.long()].view(torch.uint8))
    return seq.double().cpu().numpy(), tok.double().cpu().numpy(), dl.double().cpu().numpy()


@pytest.mark.parametrize("kind", ["neginf_mask", "lowest_mask", "lowest_row", "largest"])
@pytest.mark.parametrize("V,dtype", SHAPES)
def test_finite_results(V, dtype, kind):
    print(f"logprob extremes V={V} {dtype} {kind}", flush=True)
    pack, x, tokens, dseq = _inputs(V, dtype, 930)
    lo, hi = V // 3, max(V // 3 + 1, V // 2)  # what a mask leaves: neither head nor tail
    tokens = lo + tokens % (hi - lo)
    if kind == "neginf_mask":
        x[:, :lo] = -float("inf")
        x[:, hi:] = -float("inf")
    elif kind == "lowest_mask":
        x[:, :lo] = torch.finfo(dtype).min
        x[:, hi:] = torch.finfo(dtype).min
    elif kind == "lowest_row":
        x[:] = torch.finfo(dtype).min
    else:  # its label's log-prob is 0, any other's about -3.4e38
        at = [0, V - 1, lo, V // 2 + 1]
        for t in range(x.shape[0]):
            x[t, at[t % 4]] = torch.finfo(dtype).max
        rows = orc.logprob_predicting_rows(*pack.oracle_args())
        first = {int(pack.row_start[b]) + int(pack.prompt_len[b]) - 1: b for b in range(pack.num_rows)}
        for r in rows:
            if r in first:
                b = first[r]
                for k in range(int(pack.num_resp[b])):
                    tokens[int(pack.row_start[b]) + int(pack.resp_off[b, k])] = at[r % 4]
            tokens[min(r + 1, len(tokens) - 1)] = at[r % 4]
    args, x64 = pack.oracle_args(), x.double().numpy()
    # the same log-probs from logits whose maxima are 0: at 1e38 not even 64 bits hold a row's ln(sum) next to them
    x64 -= x64.max(axis=1, keepdims=True)
    seq, tok, dl = _run(pack, x, tokens, dseq)
    ref_seq, ref_tok = orc.seq_logprob(*args, x64, tokens.numpy())
    assert np.isfinite(ref_tok).all()
    for got, ref in ((seq, ref_seq), (tok, ref_tok)):
        assert np.abs(got - ref).max() <= 1e-5 + 1e-5 * np.abs(ref).max()
    want = orc.seq_logprob_grad(*args, x64, tokens.numpy(), dseq.double().numpy())
    gmax = float(dseq.abs().max())
    assert (np.abs(dl - want) - RTOL[dtype] * np.abs(want)).max() <= 1e-6 * gmax


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("bad", ["nan", "inf"])
@pytest.mark.parametrize("V,dtype", SHAPES)
def test_nan_and_inf_reach_the_row(V, dtype, bad, masked):
    print(f"logprob extremes V={V} {dtype} {bad} masked={masked}", flush=True)
    pack, x, tokens, dseq = _inputs(V, dtype, 940)
    label = V // 2
    tokens[:] = label
    if masked:  # a NaN alone among -inf: no neighbour has a maximum
        keep = x[:, label].clone()
        x[:] = -float("inf")
        x[:, label] = keep
    rows = orc.logprob_predicting_rows(*pack.oracle_args())
    hit = rows[1::2]
    at = [0, V - 1, min(V - 1, 1), max(0, V - 2)]
    for i, r in enumerate(hit):
        x[r, at[i % 4]] = float(bad)
    _, tok, dl = _run(pack, x, tokens, dseq)
    for r in rows:
        assert np.isnan(dl[r]).all() if r in hit else np.isfinite(dl[r]).all(), r
    first = {int(pack.row_start[b]) + int(pack.prompt_len[b]) - 1 for b in range(pack.num_rows)}
    for r in set(rows) - first:  # a response's token is the only one its row predicts
        assert np.isnan(tok[r + 1]) == (r in hit), r
