"""GPU tests of the small kernels at the sizes where their forms change: the pair loss
with its pairs spread over threads (3 to 8 slots a row, several turns of rows) and
plain, and the reward head's backward with vectors or single elements a row and more
slots than one round of loads holds.  Against the oracle; tolerances from the
arithmetic: fp32 sums of n terms (n 2^-24 relative to the terms' magnitudes, held to
2e-6 times their sum of magnitudes) and, for bf16 gradients, one rounding (2^-8)."""
import numpy as np
import pytest
import torch

from oracle import pp_oracle as orc
from paper_2602_24082_amd import binding as pp
from paper_2602_24082_amd import workload as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("K,B", [(2, 5), (3, 1), (3, 86), (4, 42), (4, 43), (8, 9), (8, 10), (8, 300), (9, 7)])
def test_pair_loss_forms(K, B):
    rng = np.random.default_rng(K * 1000 + B)
    num = rng.integers(0, K + 1, size=B).tolist()
    num[B // 2] = K
    pol = (rng.standard_normal((B, K)) * 3).astype(np.float32)
    ref = (rng.standard_normal((B, K)) * 3).astype(np.float32)
    loss, rows, g = pp.pp_dpo_loss(num, torch.from_numpy(pol).to(DEV), torch.from_numpy(ref).to(DEV), 0.5)
    want, want_rows, want_g = orc.pair_loss(num, pol.astype(np.float64), ref.astype(np.float64), 0.5)
    # z is a rounded difference of rounded values: 2^-23 of its terms' magnitudes, up to 12 here
    assert abs(float(loss) - want) <= 5e-6 * max(1.0, abs(want))
    assert np.abs(rows.double().cpu().numpy() - want_rows).max() <= 5e-6 * max(1.0, np.abs(want_rows).max())
    assert np.abs(g.double().cpu().numpy() - want_g).max() <= 5e-6 * max(np.abs(want_g).max(), 1.0 / B)
    assert torch.equal(g, pp.pp_dpo_loss(num, torch.from_numpy(pol).to(DEV), torch.from_numpy(ref).to(DEV), 0.5)[2])


@pytest.mark.parametrize("H,dtype,B,K", [(8, torch.bfloat16, 1, 1), (1001, torch.bfloat16, 3, 2), (4096, torch.bfloat16, 8, 4),
                                         (2056, torch.float32, 13, 5), (257, torch.float32, 33, 4), (3, torch.float32, 1, 3)])
def test_rm_backward_forms(H, dtype, B, K):
    rng = np.random.default_rng(H + B)
    lens = [rng.integers(0, 4, size=int(rng.integers(0, K + 1))).tolist() for _ in range(B)]
    lens[0] = [2] * K
    pack = wl.make_pack(rng.integers(1, 6, size=B).tolist(), lens, pad=rng.integers(0, 3, size=B).tolist())
    print(f"rm H={H} {dtype} slots={B * pack.max_resp} T={pack.total_tokens}", flush=True)
    hidden = wl.randn((pack.total_tokens, H), 920, dtype, "cpu")
    w = wl.randn((H,), 921, dtype, "cpu", sigma=0.1)
    ds = wl.randn((B, pack.max_resp), 922, torch.float32, "cpu")
    args = pack.oracle_args()
    h64, w64 = hidden.double().numpy(), w.double().numpy()
    scores = pp.pp_rm_scores(pack, hidden.to(DEV), w.to(DEV), 0.5)
    want = orc.rm_scores(*args, h64, w64, 0.5)
    mag = 0.5 + np.abs(h64).max() * np.abs(w64).sum()
    assert np.abs(scores.double().cpu().numpy()[:, :want.shape[1]] - want).max() <= 2e-6 * mag
    dh, dw, db = pp.pp_rm_scores_bwd(pack, hidden.to(DEV), w.to(DEV), ds.to(DEV))
    rh, rw, rb = orc.rm_scores_grad(*args, h64, w64, ds.double().numpy())
    rel = 2.0 ** -8 if dtype == torch.bfloat16 else 2e-6
    gsum = np.abs(ds.numpy()).sum()
    assert (np.abs(dh.double().cpu().numpy() - rh) <= rel * np.abs(rh) + 2e-6 * gsum * np.abs(w64).max()).all()
    assert np.abs(dw.double().cpu().numpy() - rw).max() <= 2e-6 * gsum * np.abs(h64).max()
    assert abs(float(db) - rb) <= 2e-6 * gsum
