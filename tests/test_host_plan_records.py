"""CPU tests of the planner's records, entry by entry, against the dense mask and the
oracle: every listed key tile and each 32-query block's class, every dK/dV tile's query
range, the cuts as an exact partition of their tiles, the stored dS blocks, the segment
bounds, and the log-prob and reward-head records."""
import numpy as np
import pytest

from oracle import pp_oracle as orc
from paper_2602_24082_amd import workload as wl
import host_records as hr

SKIP, FULL, MASKED, CAUSAL = 0, 1, 2, 3


def _rows(pack):
    """(first flat token, length, prompt, response offsets, lengths, mask) of each row."""
    for b in range(pack.num_rows):
        t0, t1, K = int(pack.row_start[b]), int(pack.row_start[b + 1]), int(pack.num_resp[b])
        off, ln = [int(x) for x in pack.resp_off[b, :K]], [int(x) for x in pack.resp_len[b, :K]]
        P = int(pack.prompt_len[b])
        yield t0, t1 - t0, P, off, ln, orc.row_mask(t1 - t0, P, off, ln)


def _random(rng):
    B = int(rng.integers(1, 4))
    P = [int(rng.integers(0, int(rng.choice([2, 70, 400, 700])))) for _ in range(B)]
    L = [[0 if rng.random() < 0.15 else int(rng.integers(0, int(rng.choice([4, 50, 300]))))
          for _ in range(int(rng.integers(0, 6)))] for _ in range(B)]
    return wl.make_pack(P, L, pad=[int(rng.choice([0, 1, 40, 150])) for _ in range(B)])


# a prompt or response that ends on a tile, a response that fills a query tile, one past
# either, empty prompts and responses, padding inside a tile
EDGES = [([64], [[64]], [0]), ([128], [[128, 128]], [0]), ([127], [[129, 128]], [1]), ([129], [[0, 0, 127]], [63]),
         ([0], [[300, 5]], [0]), ([0], [[0]], [64]), ([192], [[]], [64]), ([1], [[1] * 8], [0]), ([256], [[1, 255, 256]], [128]),
         ([60], [[4, 64, 128, 132]], [0]), ([32], [[32, 0, 64]], [32])]


def _packs(case):
    if case != "random":
        return [wl.make_pack(*EDGES[case][:2], pad=EDGES[case][2])]
    rng = np.random.default_rng(81)
    packs = [_random(rng) for _ in range(30)]
    return [p for p in packs if p.total_tokens]


CASES = list(range(len(EDGES))) + ["random"]


def _class(m, valid_causal):
    """Class of one 32-query block against a key tile of full width, from the mask."""
    if not m.any():
        return SKIP
    if m.all():
        return FULL
    return CAUSAL if (m == valid_causal).all() else MASKED


@pytest.mark.parametrize("which", ["fwd", "dq"])
@pytest.mark.parametrize("case", CASES)
def test_query_tiles(case, which):
    BM, BN = 128, 64
    for pack in _packs(case):
        items, tiles = hr.records(pack, which + "_items"), hr.records(pack, which + "_ktiles")
        by = {(int(i["tok0"]), int(i["q0"])): i for i in items}
        assert len(by) == len(items)
        assert list(items["kt_cnt"]) == sorted(items["kt_cnt"], reverse=True) and items["kt_cnt"].sum() == len(tiles)
        for t0, n, P, off, ln, mask in _rows(pack):
            valid = P + sum(ln)
            for q0 in range(0, n, BM):
                it = by.pop((t0, q0))
                q1 = min(n, q0 + BM)
                assert (it["q_end"], it["P"], it["valid"]) == (q1, P, valid)
                got = tiles[it["kt_off"]:it["kt_off"] + it["kt_cnt"]]
                want = [k0 for k0 in range(0, n, BN) if mask[q0:q1, k0:k0 + BN].any()]
                assert got["k0"].tolist() == want
                for e in got:
                    k0 = int(e["k0"])
                    for w in range(16):
                        a, b = q0 + 32 * w, min(q1, q0 + 32 * w + 32)
                        cls = (int(np.uint32(e["cls"])) >> (2 * w)) & 3
                        if a >= b:
                            assert cls == SKIP
                            continue
                        m = np.zeros((b - a, BN), bool)  # a tile cut short by the row's end has lanes without a key
                        part = mask[a:b, k0:k0 + BN]
                        m[:, :part.shape[1]] = part
                        i, j = np.arange(a, b)[:, None], np.arange(k0, k0 + BN)[None, :]
                        assert cls == _class(m, (j <= i) & (i < valid) & (j < valid)), (k0, w)
        assert not by


@pytest.mark.parametrize("case", CASES)
def test_key_tiles_and_segments(case):
    for pack in _packs(case):
        kv = {(int(i["tok0"]), int(i["k0"])): i for i in hr.records(pack, "kv_items")}
        lo, hi = hr.records(pack, "seg_lo"), hr.records(pack, "seg_hi")
        kb0, panels = hr.records(pack, "row_kb0"), hr.records(pack, "panels")
        next_tile = 0
        for b, (t0, n, P, off, ln, mask) in enumerate(_rows(pack)):
            valid = P + sum(ln)
            for j in range(n):
                seen = np.flatnonzero(mask[:, j])
                assert hi[t0 + j] == (seen[-1] + 1 if len(seen) else 0), j
                start = next((o for o, m in zip(off, ln) if o <= j < o + m), 0 if j < P else -1)
                assert lo[t0 + j] == start, j
            for k0 in range(0, n, 128):
                it = kv.pop((t0, k0))
                seen = np.flatnonzero(mask[:, k0:k0 + 128].any(axis=1))
                assert (it["k_end"], it["valid"], it["row"], it["part"]) == (min(n, k0 + 128), valid, b, -1)
                if len(seen):
                    assert (it["q_begin"], it["q_end"]) == (seen[0], seen[-1] + 1)
                else:
                    assert it["q_begin"] == it["q_end"]
            for kb in range(-(-n // 32)):
                p = panels[kb0[b] + kb]
                seen = np.flatnonzero(mask[:, 32 * kb:32 * kb + 32].any(axis=1))
                want = -(-(int(seen[-1]) + 1) // 32) - kb if len(seen) else 0
                assert (p["off"], p["len"]) == (next_tile, want), (b, kb)
                next_tile += want
        assert not kv


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (14, 2, 64), (8, 1, 64), (12, 12, 128)])
def test_cuts_partition_their_tiles(hq, hkv, d):
    rng = np.random.default_rng(83)
    packs = [wl.make_pack([1500], [[300, 311]]), wl.make_pack([640, 9], [[65, 0, 190], [3]], pad=[33, 0])]
    packs += [p for p in (_random(rng) for _ in range(20)) if p.total_tokens]
    G, cut = hq // hkv, 0
    for pack in packs:
        whole = {(int(i["tok0"]), int(i["k0"])): i for i in hr.records(pack, "kv_items", hq, hkv, d)}
        items, parts, splits = (hr.records(pack, n, hq, hkv, d) for n in ("cut_items", "cut_parts", "cut_splits"))
        if not len(items):
            assert not len(parts) and not len(splits)
            continue
        cut += 1
        assert len(parts) * hkv <= 768 and sorted(parts["slot"]) == list(range(len(parts)))
        pairs = lambda i: G * -(-int(i["q_end"] - i["q_begin"]) // 64)
        length = lambda i: pairs(i) if i["part"] < 0 else int(parts[i["part"]]["n_end"] - parts[i["part"]]["n_begin"])
        assert [length(i) for i in items] == sorted((length(i) for i in items), reverse=True)  # longest first
        assert sorted(i["part"] for i in items if i["part"] >= 0) == list(range(len(parts)))
        by = {}
        for i in items:
            w = whole[int(i["tok0"]), int(i["k0"])]
            assert all(i[f] == w[f] for f in ("k_end", "valid", "q_begin", "q_end", "row"))
            by.setdefault((int(i["tok0"]), int(i["k0"])), []).append(int(i["part"]))
        assert set(by) == set(whole)
        split = {(int(s["tok0"]), int(s["k0"])): s for s in splits}
        for key, ps in by.items():
            if ps == [-1]:
                assert key not in split
                continue
            s = split.pop(key)
            ps.sort()
            assert s["k_end"] == whole[key]["k_end"] and s["parts"] == len(ps) >= 2
            assert [int(parts[p]["slot"]) for p in ps] == list(range(s["slot0"], s["slot0"] + len(ps)))
            ends = [0] + [int(parts[p]["n_end"]) for p in ps]
            assert [int(parts[p]["n_begin"]) for p in ps] == ends[:-1] and ends[-1] == pairs(whole[key])
            assert min(b - a for a, b in zip(ends, ends[1:])) > 0
        assert not split
    assert cut >= 2


def test_logprob_and_reward_records():
    rng = np.random.default_rng(84)
    packs = [wl.make_pack(*e[:2], pad=e[2]) for e in EDGES] + [_random(rng) for _ in range(40)]
    checked = 0
    for pack in packs:
        B, Kmax = pack.num_rows, pack.max_resp
        slot_row, rm_rows, rm_slots = (hr.records(pack, "rm_" + n) for n in ("slot_row", "rows", "slots"))
        want = np.full(B * Kmax, -1)
        for b, (t0, n, P, off, ln, _) in enumerate(_rows(pack)):
            for k, (o, m) in enumerate(zip(off, ln)):
                if m or P:
                    want[b * Kmax + k] = t0 + (o + m - 1 if m else P - 1)
        assert slot_row.tolist() == want.tolist()
        readers = {}
        for s, r in enumerate(want.tolist()):
            if r >= 0:
                readers.setdefault(r, []).append(s)
        assert rm_rows["row"].tolist() == list(readers)
        for r in rm_rows:
            assert rm_slots[r["slot_off"]:r["slot_off"] + r["slot_cnt"]].tolist() == readers[int(r["row"])]
        assert rm_rows["slot_cnt"].sum() == len(rm_slots)

        if any(P == 0 and sum(ln) for _, _, P, _, ln, _ in _rows(pack)):
            continue  # refused: a first token without a predicting position
        checked += 1
        rows, labels, out, item, resp = (hr.records(pack, "lp_" + n) for n in ("rows", "labels", "label_out", "row_item", "resp"))
        assert rows["logit_row"].tolist() == orc.logprob_predicting_rows(*pack.oracle_args())
        predicts = {}  # row -> [(label token, slot)]
        for b, (t0, n, P, off, ln, _) in enumerate(_rows(pack)):
            for k, (o, m) in enumerate(zip(off, ln)):
                for j in range(m):
                    predicts.setdefault(t0 + (P - 1 if j == 0 else o + j - 1), []).append((t0 + o + j, b * Kmax + k))
        assert set(predicts) == set(rows["logit_row"].tolist())
        end = 0
        for i, r in enumerate(rows):
            assert r["label_off"] == end
            end += int(r["label_cnt"])
            s = slice(r["label_off"], end)
            assert list(zip(labels[s].tolist(), out[s].tolist())) == predicts[int(r["logit_row"])]
            assert item[r["logit_row"]] == i
        assert end == len(labels) == len(out) and (item >= 0).sum() == len(rows) and item.min(initial=-1) == -1
        for b, (t0, n, P, off, ln, _) in enumerate(_rows(pack)):
            for k in range(Kmax):
                r = resp[b * Kmax + k]
                assert r["out"] == b * Kmax + k and r["len"] == (ln[k] if k < len(ln) else 0)
                if r["len"]:
                    assert r["tok_begin"] == t0 + off[k]
    assert checked > 30
