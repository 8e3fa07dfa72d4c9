"""CPU tests of the workspace sizes that the planner's shortcuts make, against the dense
mask: how many key tiles are listed for all 128-query tiles (a tile in full view, or far
from the tile's own responses, is settled without counting pairs), how many 32 x 32 blocks
of dS the stored mode keeps, and how many log-prob records there are.  Sizes are rounded
to 256 bytes; test_host_plan_records.py holds the records themselves, entry by entry."""
import numpy as np
import pytest

from oracle import pp_oracle as orc
from paper_2602_24082_amd import binding
from paper_2602_24082_amd import workload as wl


def _align(n):
    return (n + 255) // 256 * 256


def _packs(rng):
    B = int(rng.integers(1, 4))
    P = [int(rng.integers(0, int(rng.choice([2, 70, 400])))) for _ in range(B)]
    L = [[0 if rng.random() < 0.15 else int(rng.integers(0, int(rng.choice([4, 50, 300])))) for _ in range(int(rng.integers(0, 6)))]
         for _ in range(B)]
    pad = [int(rng.choice([0, 1, 40, 150])) for _ in range(B)]
    return wl.make_pack(P, L, pad=pad)


def _row_masks(pack):
    offs, lens = pack.resp_off, pack.resp_len
    for b in range(pack.num_rows):
        T, K = int(pack.row_start[b + 1] - pack.row_start[b]), int(pack.num_resp[b])
        yield T, orc.row_mask(T, int(pack.prompt_len[b]), [int(x) for x in offs[b, :K]], [int(x) for x in lens[b, :K]])


# edges of the shortcuts: a prompt or response that ends on a tile, a response that fills
# a query tile, one past either, empty prompts and responses, padding inside a tile
EDGES = [([64], [[64]], [0]), ([128], [[128, 128]], [0]), ([127], [[129, 128]], [1]), ([129], [[0, 0, 127]], [63]),
         ([0], [[300, 5]], [0]), ([0], [[0]], [64]), ([192], [[]], [64]), ([1], [[1] * 8], [0]), ([256], [[1, 255, 256]], [128])]


@pytest.mark.parametrize("case", list(range(len(EDGES))) + ["random"])
def test_listed_tiles_and_blocks(case):
    rng = np.random.default_rng(77)
    packs = [_packs(rng) for _ in range(40)] if case == "random" else [wl.make_pack(*EDGES[case][:2], pad=EDGES[case][2])]
    for pack in packs:
        T, d, hq, hkv = pack.total_tokens, 64, 4, 2
        if T == 0:
            continue
        items = tiles = blocks = 0
        for n, mask in _row_masks(pack):
            items += -(-n // 128)
            for q0 in range(0, n, 128):
                tiles += sum(mask[q0:q0 + 128, k0:k0 + 64].any() for k0 in range(0, n, 64))
            for k0 in range(0, n, 32):
                seen = np.flatnonzero(mask[:, k0:k0 + 32].any(axis=1))
                blocks += max(0, -(-(int(seen[-1]) + 1) // 32) - k0 // 32) if len(seen) else 0
        fwd = binding.pp_workspace_size(pack, hq, hkv, d, bwd=False, loss=False)[0]
        assert fwd == 2 * _align(4 * T) + _align(32 * items) + _align(8 * tiles) + _align(8 * d // 2)
        lean = binding.pp_workspace_size(pack, hq, hkv, d, fwd=False, loss=False)[1]
        stored = binding.pp_bwd_stored_ds_workspace_size(pack, hq, hkv, d)[0]
        assert stored - lean == blocks * hq * 2048


def test_logprob_records():
    rng = np.random.default_rng(78)
    for _ in range(40):
        pack = _packs(rng)
        K = pack.num_resp
        if any(int(pack.prompt_len[b]) == 0 and int(pack.resp_len[b, :int(K[b])].sum()) for b in range(pack.num_rows)):
            continue  # refused: a first token without a predicting position
        rows = len(orc.logprob_predicting_rows(*pack.oracle_args()))
        assert binding.pp_logprob_row_count(pack) == rows
        labels = sum(int(pack.resp_len[b, :int(K[b])].sum()) for b in range(pack.num_rows))
        T, slots = pack.total_tokens, pack.num_rows * pack.max_resp
        size = binding.pp_workspace_size(pack, vocab=10, fwd=False, bwd=False, logprob=True, loss=False)[2]
        assert size == _align(16 * rows) + 2 * _align(4 * labels) + _align(16 * slots) + 2 * _align(4 * T)
