// Host side of the preference-packing library: descriptor validation, the
// planner that turns a packed batch (Sec. 3.2) into tile work lists, workspace
// layout, pinned staging of plan metadata, kernel timing and the C ABI entry
// points declared in pp_attn.h.
//
// Validation never touches the GPU, so every error path (and pp_pack_export)
// works on a machine without one.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "../../include/pp_attn.h"
#include "pp_launch.h"
#include "pp_plan.h"

namespace pp {
namespace {

thread_local std::string g_last_error;

pp_status fail(pp_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

pp_status hip_fail(hipError_t e, const char* what) {
  return fail(PP_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

// ---------------------------------------------------------------------------
// Descriptor validation and per-row view
// ---------------------------------------------------------------------------

struct Row {
  int32_t tok0;  // flat start
  int32_t T;     // capacity
  int32_t P;     // prompt length
  int32_t K;     // responses
  int32_t valid; // P + sum L
  const int32_t* off;
  const int32_t* len;
};

struct Batch {
  std::vector<Row> rows;
  int32_t sumT = 0;
  int32_t B = 0;
  int32_t Kmax = 0;
};

pp_status read_desc(const pp_pack_desc* d, Batch* out) {
  if (!d) return fail(PP_ERR_INVALID_ARGUMENT, "desc is NULL");
  if (d->num_rows < 1) return fail(PP_ERR_INVALID_ARGUMENT, "num_rows must be >= 1 (got %d)", d->num_rows);
  if (d->max_resp < 0) return fail(PP_ERR_INVALID_ARGUMENT, "max_resp must be >= 0");
  if (!d->row_start || !d->prompt_len || !d->num_resp)
    return fail(PP_ERR_INVALID_ARGUMENT, "row_start, prompt_len and num_resp must be non-NULL");
  if (d->max_resp > 0 && (!d->resp_off || !d->resp_len))
    return fail(PP_ERR_INVALID_ARGUMENT, "resp_off and resp_len must be non-NULL when max_resp > 0");
  const int B = d->num_rows;
  if (d->row_start[0] != 0) return fail(PP_ERR_BAD_LAYOUT, "row_start[0] must be 0");
  out->rows.resize(B);
  out->B = B;
  out->Kmax = d->max_resp;
  for (int b = 0; b < B; ++b) {
    const int64_t r0 = d->row_start[b], r1 = d->row_start[b + 1];
    if (r1 < r0) return fail(PP_ERR_BAD_LAYOUT, "row_start must be non-decreasing (row %d)", b);
    Row& r = out->rows[b];
    r.tok0 = (int32_t)r0;
    r.T = (int32_t)(r1 - r0);
    r.P = d->prompt_len[b];
    r.K = d->num_resp[b];
    if (r.P < 0) return fail(PP_ERR_BAD_LAYOUT, "prompt_len[%d] < 0", b);
    if (r.K < 0 || r.K > d->max_resp)
      return fail(PP_ERR_BAD_LAYOUT, "num_resp[%d] = %d outside [0, max_resp=%d]", b, r.K, d->max_resp);
    r.off = d->max_resp ? d->resp_off + (int64_t)b * d->max_resp : nullptr;
    r.len = d->max_resp ? d->resp_len + (int64_t)b * d->max_resp : nullptr;
    int64_t pos = r.P;
    for (int k = 0; k < r.K; ++k) {
      if (r.len[k] < 0) return fail(PP_ERR_BAD_LAYOUT, "resp_len[%d,%d] < 0", b, k);
      if (r.off[k] != pos)
        return fail(PP_ERR_BAD_LAYOUT,
                    "responses must follow the prompt contiguously: resp_off[%d,%d] = %d, expected %lld",
                    b, k, r.off[k], (long long)pos);
      pos += r.len[k];
    }
    if (pos > r.T)
      return fail(PP_ERR_BAD_LAYOUT, "row %d: prompt + responses = %lld exceed its %d tokens", b,
                  (long long)pos, r.T);
    r.valid = (int32_t)pos;
  }
  out->sumT = d->row_start[B];
  return PP_OK;
}

pp_status check_heads(int hq, int hkv, int d) {
  if (hq < 1 || hkv < 1) return fail(PP_ERR_INVALID_ARGUMENT, "hq and hkv must be >= 1");
  if (hq % hkv) return fail(PP_ERR_INVALID_ARGUMENT, "hq (%d) must be a multiple of hkv (%d)", hq, hkv);
  if (d != 64 && d != 128) return fail(PP_ERR_UNSUPPORTED, "head_dim %d not supported (64 or 128)", d);
  return PP_OK;
}

pp_status check_dtype(pp_dtype t) {
  if (t != PP_BF16 && t != PP_FP32) return fail(PP_ERR_INVALID_ARGUMENT, "unknown dtype %d", (int)t);
  return PP_OK;
}

// ---------------------------------------------------------------------------
// Exact visible-pair counting on intervals
// ---------------------------------------------------------------------------

inline int64_t overlap(int64_t a0, int64_t a1, int64_t b0, int64_t b1) {
  const int64_t lo = std::max(a0, b0), hi = std::min(a1, b1);
  return hi > lo ? hi - lo : 0;
}

// Segment id: 0 prompt, k+1 response k, -1 padding.
inline int32_t seg_id(const Row& r, int32_t t) {
  if (t < r.P) return 0;
  for (int k = 0; k < r.K; ++k)
    if (r.off[k] <= t && t < r.off[k] + r.len[k]) return k + 1;
  return -1;
}

// sum_{i=a}^{b-1} max(0, min(k1, i+1) - c): the keys in [c, k1) that lie at or
// before query i, summed over a run of queries.
int64_t sum_ramp(int64_t a, int64_t b, int64_t c, int64_t k1) {
  if (b <= a || k1 <= c) return 0;
  int64_t n = 0;
  // x = i + 1 runs over [a+1, b]; x in (c, k1] contributes x - c
  const int64_t lo1 = std::max(a + 1, c + 1), hi1 = std::min(b, k1);
  if (hi1 >= lo1) n += (lo1 - c + hi1 - c) * (hi1 - lo1 + 1) / 2;
  // x in (k1, b] contributes k1 - c
  const int64_t lo2 = std::max(a + 1, k1 + 1);
  if (b >= lo2) n += (b - lo2 + 1) * (k1 - c);
  return n;
}

// Number of visible (query, key) pairs with query in [q0,q1), key in [k0,k1),
// in closed form per segment.  A prompt query i sees keys [0, i]; a query i of
// response k sees [0, P) and [o_k, i]; padding sees nothing.  Responses before
// first_resp must end by q0.
int64_t visible_pairs(const Row& r, int32_t q0, int32_t q1, int32_t k0, int32_t k1, int first_resp = 0) {
  if (k1 <= k0) return 0;
  int64_t n = 0;
  // prompt queries
  {
    const int64_t a = q0, b = std::min(q1, r.P);
    n += sum_ramp(a, b, k0, k1);
  }
  // response queries
  const int64_t kp = overlap(k0, k1, 0, r.P);
  for (int k = first_resp; k < r.K && r.off[k] < q1; ++k) {
    const int64_t o = r.off[k], e = (int64_t)r.off[k] + r.len[k];
    const int64_t a = std::max<int64_t>(q0, o), b = std::min<int64_t>(q1, e);
    if (b <= a) continue;
    n += kp * (b - a) + sum_ramp(a, b, std::max<int64_t>(k0, o), k1);
  }
  return n;
}

// 0 EMPTY, 1 PARTIAL, 2 FULL for the tile clipped to the row.
uint8_t classify_tile(const Row& r, int32_t q0, int32_t q1, int32_t k0, int32_t k1) {
  const int64_t n = visible_pairs(r, q0, q1, k0, k1);
  if (n == 0) return 0;
  if (n == (int64_t)(q1 - q0) * (k1 - k0)) return 2;
  return 1;
}

// ---------------------------------------------------------------------------
// Plans
// ---------------------------------------------------------------------------

struct QPlan {
  std::vector<QTileItem> items;
  std::vector<KTileEntry> ktiles;
};

// Query tiles of BM queries and, for each, the key tiles of BN keys that hold a
// visible pair, with the class of each 32-query block.  Most tiles need no count of
// pairs: a key tile at or before the tile's first query is visible in full if it
// lies in the prompt, or in the one response that holds all the tile's queries, and
// of the keys past the prompt only those from the first response that the tile
// reaches are visible at all, so the walk goes straight there.  The rest (the tile
// that holds the prompt's end, the diagonal, rows' ends) count their pairs.
// (The sizes of one forward of 8 rows, 12656 tokens, planned in 120 us of host time when
// every tile was counted, and in 20 to 25 us now.)
void build_qplan(const Batch& bt, int BM, int BN, QPlan* out) {
  out->items.clear();
  out->ktiles.clear();
  const uint32_t all_full = kWaveFull * 0x55555555u;
  for (int b = 0; b < bt.B; ++b) {
    const Row& r = bt.rows[b];
    int kk = 0;  // first response that ends past the tile's first query
    for (int32_t q0 = 0; q0 < r.T; q0 += BM) {
      QTileItem it{};
      it.tok0 = r.tok0;
      it.q0 = q0;
      it.q_end = std::min(r.T, q0 + BM);
      it.P = r.P;
      it.valid = r.valid;
      it.kt_off = (int32_t)out->ktiles.size();
      it.row = b;
      while (kk < r.K && r.off[kk] + r.len[kk] <= q0) ++kk;
      // first key past the prompt that a query of the tile may see
      const int32_t own = kk < r.K && r.off[kk] < it.q_end ? r.off[kk] : r.T;
      const int32_t own_end = kk < r.K ? r.off[kk] + r.len[kk] : 0;
      const int waves = (it.q_end - q0 + 31) / 32;
      // only keys <= the tile's last query can be visible (causal)
      const int32_t kmax = std::min(it.q_end, r.valid);
      for (int32_t k0 = 0; k0 < kmax; k0 += BN) {
        if (k0 >= r.P && k0 + BN <= own) {
          k0 = own / BN * BN;
          if (k0 >= kmax) break;
        }
        if (k0 + BN <= q0 + 1 && it.q_end <= r.valid &&
            (k0 + BN <= r.P || (k0 >= own && it.q_end <= own_end))) {
          out->ktiles.push_back(KTileEntry{k0, all_full & (waves >= 16 ? ~0u : (1u << (2 * waves)) - 1u)});
          continue;
        }
        const int32_t k1 = std::min(r.T, k0 + BN);
        KTileEntry e{k0, 0u};
        bool any = false;
        for (int w = 0; w < waves; ++w) {
          const int32_t qa = q0 + 32 * w, qb = std::min(it.q_end, qa + 32);
          const int64_t n = visible_pairs(r, qa, qb, k0, k1, kk);
          int cls = kWaveSkip;
          // a key tile cut short by the row's end leaves lanes without a key: masked
          if (n == (int64_t)(qb - qa) * BN) {
            cls = kWaveFull;
          } else if (n > 0) {
            // the visible pairs are exactly the causal ones among real tokens:
            // the mask reduces to j <= i
            const int64_t causal = sum_ramp(qa, std::min(qb, r.valid), k0, std::min(k1, r.valid));
            cls = n == causal ? kWaveCausal : kWaveMasked;
          }
          any = any || n > 0;
          e.cls |= (uint32_t)cls << (2 * w);
        }
        if (any) out->ktiles.push_back(e);
      }
      it.kt_cnt = (int32_t)out->ktiles.size() - it.kt_off;
      out->items.push_back(it);
    }
  }
  // longest-first, so the heaviest tiles start in the first wave of workgroups
  std::stable_sort(out->items.begin(), out->items.end(),
                   [](const QTileItem& a, const QTileItem& b) { return a.kt_cnt > b.kt_cnt; });
}

// One past the last query that sees a key of [k0, k_end), k0 < r.valid: a
// prompt key is seen by every later real token; when the keys lie in
// responses, the last real key's response bounds the range.
int32_t key_tile_q_end(const Row& r, int32_t k0, int32_t k_end) {
  if (k0 < r.P) return r.valid;
  const int32_t last = std::min(k_end, r.valid) - 1;
  int32_t end = r.valid;
  for (int k = 0; k < r.K; ++k)
    if (r.off[k] <= last && last < r.off[k] + r.len[k]) end = r.off[k] + r.len[k];
  return end;
}

// (head, step) pairs of a key tile.
inline int tile_pairs(const KTileItem& t, int G) { return G * ((t.q_end - t.q_begin + kBwdBlockM - 1) / kBwdBlockM); }

// Key tiles of the dK/dV pass, each one work item, longest first.
void build_kplan(const Batch& bt, int BN, std::vector<KTileItem>* out) {
  out->clear();
  for (int b = 0; b < bt.B; ++b) {
    const Row& r = bt.rows[b];
    for (int32_t k0 = 0; k0 < r.T; k0 += BN) {
      KTileItem it{};
      it.tok0 = r.tok0;
      it.k0 = k0;
      it.k_end = std::min(r.T, k0 + BN);
      it.valid = r.valid;
      it.row = b;
      if (k0 >= r.valid) {
        it.q_begin = it.q_end = k0;  // padding keys: nothing sees them
      } else {
        it.q_begin = k0;  // query k0 sees key k0
        it.q_end = key_tile_q_end(r, k0, it.k_end);
      }
      it.part = -1;
      out->push_back(it);
    }
  }
  std::stable_sort(out->begin(), out->end(),
                   [](const KTileItem& a, const KTileItem& b) { return tile_pairs(a, 1) > tile_pairs(b, 1); });
}

// Parts of a tile of n (head, step) pairs when no part may exceed `most`.
inline int split_parts(int n, int most) { return most > 0 && n > most ? (n + most - 1) / most : 1; }

// Finish time, in steps, of one kv-head's items (longest first, each tile of `pairs`
// pairs cut so that no part exceeds `most`; 0: none) on `units` compute units that
// each take the next item when they are free, plus `extra` for every part of a cut
// tile; *n_parts: those parts.  A bound at least `enough` is returned as it is.
struct KPlanSpan {
  // in steps of kBwdBlockM queries (2.0 us at head size 128 with all units busy, 1.5 with few; 1.05 at 64): 1.6 for a
  // workgroup's K/V load and epilogue, 1 more to write a part's fp32 sums
  static constexpr double kItem = 1.6, kPart = 1.0;
  static double cost(int key) { return (key >> 1) + kItem + (key & 1 ? kPart : 0.0); }

  std::vector<int> keys;     // 2 x pairs + part of a cut tile
  std::vector<double> busy;  // min-heap of the units' finish times

  double operator()(const std::vector<int>& pairs, int most, int units, double extra, double enough, int* n_parts) {
    keys.clear();
    *n_parts = 0;
    int64_t sum = 0;
    for (int n : pairs) {
      const int parts = split_parts(n, most);
      if (parts > 1) *n_parts += parts;
      for (int i = 0; i < parts; ++i)
        keys.push_back((int)((int64_t)n * (i + 1) / parts - (int64_t)n * i / parts) * 2 + (parts > 1));
      sum += n;
    }
    const double more = extra * *n_parts;
    const double least = ((double)sum + kItem * (double)keys.size() + kPart * *n_parts) / units + more;
    if (least >= enough) return least;
    std::sort(keys.begin(), keys.end(), std::greater<int>());
    const size_t n = keys.size(), first = std::min(n, (size_t)units);
    double span = 0;
    busy.resize(first);
    for (size_t i = 0; i < first; ++i) span = std::max(span, busy[i] = cost(keys[i]));
    if (n > first) std::make_heap(busy.begin(), busy.end(), std::greater<double>());
    for (size_t i = first; i < n; ++i) {
      // the unit that is free first takes the item: its new time sinks from the top
      const double t = busy[0] + cost(keys[i]);
      span = std::max(span, t);
      size_t at = 0;
      for (size_t c = 1; c < first; c = 2 * at + 1) {
        if (c + 1 < first && busy[c + 1] < busy[c]) ++c;
        if (busy[c] >= t) break;
        busy[at] = busy[c];
        at = c;
      }
      busy[at] = t;
    }
    return span + more;
  }
};

// The dK/dV pass's items with the longest key tiles cut.
struct KvCut {
  std::vector<KTileItem> items;  // longest first; empty: the tiles stay whole
  std::vector<KTilePart> parts;
  std::vector<KTileSplit> splits;
  int slots = 0;
};

// Bytes of one (slot, kv-head)'s partial dK and dV.
inline size_t kv_part_bytes(int d) { return (size_t)2 * kBwdBlockN * d * 4; }

// Cuts the longest key tiles of a batch that leaves compute units idle: with
// few rows a prompt's first tile, which every later query of every head sees,
// outlasts all others (one 8B-shaped row of 2111 tokens: 17 tiles x 8 kv-heads
// on 256 units, the longest 132 steps against 35 a unit on average).  Batches of
// more than 2 workgroups a unit are left alone: cutting their tiles costs more
// in the parts' fixed work than it evens out (measured 0 to 14% slower).  The
// longest part allowed is the one of five that gives the smallest estimate: from
// half as much again as the units' even share, which few tiles exceed, to a third
// of it.  The estimate charges the launch that adds the partial sums 2.5 steps and
// every 46 parts of one kv-head a step more.  That is about twice what the launch
// itself takes for its bytes (400 parts, 52 MB, in 11 us; 432 after 4200 tokens in
// 16), for both head sizes: it stands for all that a further part costs.  A cut has
// to shorten the estimate by a tenth.
//
// On that row the pass took 201 us whole and takes 90 us cut (50 parts of each
// kv-head) and 11 us for the sums; one row of 4200 tokens 417 -> 280 and 16.  Of 60
// batches (1 to 24 rows, 320 to 21600 tokens, three head layouts at each head size),
// each timed whole and at seven cuts from four times the even share to a third, the
// rule's choice was the fastest in 56 and within 1.2% of it in all.
//
// Cuts into more than kMaxKvParts parts (96 MiB of sums at head size 128) are left out.
void split_kplan(const std::vector<KTileItem>& kv, int G, int hkv, KvCut* cut) {
  constexpr double kLaunch = 2.5, kPartsPerStep = 46.0;
  *cut = KvCut();
  if (kv.empty() || (int64_t)kv.size() * hkv > 2 * kComputeUnits) return;
  const int units = std::max(1, kComputeUnits / hkv);
  std::vector<int> pairs;
  int64_t work = 0;
  for (const KTileItem& t : kv) {
    pairs.push_back(tile_pairs(t, G));
    work += pairs.back();
  }
  const int even = (int)((work + units - 1) / units), longest = pairs[0];
  if (longest < 8 || longest <= even) return;  // the units' even share is the longer
  int parts = 0;
  KPlanSpan span_of;
  const double whole = span_of(pairs, 0, units, 0.0, HUGE_VAL, &parts);
  double best = whole;
  int most = 0;
  for (int sixths : {9, 6, 4, 3, 2}) {
    const int m = std::max(4, (even * sixths + 5) / 6);
    const double span = kLaunch + span_of(pairs, m, units, hkv / kPartsPerStep, best - kLaunch, &parts);
    if (span < best && (int64_t)parts * hkv <= kMaxKvParts) {
      best = span;
      most = m;
    }
  }
  if (most == 0 || best > 0.9 * whole) return;
  struct Run {
    int pairs, tile, part;
  };
  std::vector<Run> runs;
  for (size_t j = 0; j < kv.size(); ++j) {
    const KTileItem& t = kv[j];
    const int n = pairs[j], k = split_parts(n, most);
    if (k == 1) {
      runs.push_back({n, (int)j, -1});
      continue;
    }
    cut->splits.push_back(KTileSplit{t.tok0, t.k0, t.k_end, cut->slots, k, 0});
    for (int i = 0; i < k; ++i) {
      const KTilePart p{(int32_t)((int64_t)n * i / k), (int32_t)((int64_t)n * (i + 1) / k), cut->slots++, 0};
      runs.push_back({p.n_end - p.n_begin, (int)j, (int)cut->parts.size()});
      cut->parts.push_back(p);
    }
  }
  std::stable_sort(runs.begin(), runs.end(), [](const Run& a, const Run& b) { return a.pairs > b.pairs; });
  cut->items.reserve(runs.size());
  for (const Run& r : runs) {
    cut->items.push_back(kv[r.tile]);
    cut->items.back().part = r.part;
  }
}

// The per-token arrays below are filled segment by segment: a validated row is
// its prompt [0, P), then its responses back to back from P, then padding.
// seg_lo: row-relative start of the token's segment (0 in the prompt, o_k in
// response k, -1 for padding).
void fill_seg_lo(const Batch& bt, int32_t* o) {
  std::fill(o, o + bt.sumT, -1);
  for (const Row& r : bt.rows) {
    std::fill(o + r.tok0, o + r.tok0 + r.P, 0);
    for (int k = 0; k < r.K; ++k) std::fill(o + r.tok0 + r.off[k], o + r.tok0 + r.off[k] + r.len[k], r.off[k]);
  }
}

// seg_hi: one past the last query that can see key t (row-relative): a prompt key is
// seen by every later real token, a response key only by its own response's
// later tokens (Sec. 3.2), a padding key by nothing.
void fill_seg_hi(const Batch& bt, int32_t* o) {
  std::fill(o, o + bt.sumT, 0);
  for (const Row& r : bt.rows) {
    std::fill(o + r.tok0, o + r.tok0 + r.P, r.valid);
    for (int k = 0; k < r.K; ++k)
      std::fill(o + r.tok0 + r.off[k], o + r.tok0 + r.off[k] + r.len[k], r.off[k] + r.len[k]);
  }
}

// Panels of the stored dS: per row, per 32-key block KB, the query blocks
// KB .. ceil(q_end / 32) - 1, where q_end is one past the last query that sees
// one of the block's keys within its key tile of BN keys (the tile's query
// range clipped to the row's real tokens, and each key's own seg_hi) --
// exactly the 32 x 32 blocks that the key-major pass computes for it --
// numbered consecutively in row and block order.  Returns the tiles per head,
// or -1 if they do not fit 32-bit tile offsets.
int64_t build_ds_panels(const Batch& bt, int BN, std::vector<int32_t>* row_kb0, std::vector<DsPanel>* panels) {
  row_kb0->clear();
  panels->clear();
  int64_t off = 0;
  for (const Row& r : bt.rows) {
    row_kb0->push_back((int32_t)panels->size());
    int kk = 0;  // first response that ends past the block's first key
    for (int32_t kb = 0; kb * 32 < r.T; ++kb) {
      const int32_t k0 = kb * 32 / BN * BN, k_end = std::min(r.T, k0 + BN);
      int32_t q_end = 0;
      if (k0 < r.valid) {
        const int32_t qlim = std::min(key_tile_q_end(r, k0, k_end), r.valid);
        // key j is seen by queries j .. min(qlim, seg_hi(j)) - 1: a prompt key by the
        // most, else the keys of each response in the block
        const int32_t j0 = kb * 32, j1 = std::min(k_end, j0 + 32);
        while (kk < r.K && r.off[kk] + r.len[kk] <= j0) ++kk;
        if (j0 < r.P && std::min(qlim, r.valid) > j0) q_end = std::min(qlim, r.valid);
        for (int k = kk; k < r.K && r.off[k] < j1; ++k) {
          const int32_t first = std::max(j0, r.off[k]), last = std::min(qlim, r.off[k] + r.len[k]);
          if (last > first) q_end = std::max(q_end, last);
        }
      }
      const int32_t len = std::max(0, (q_end + 31) / 32 - kb);
      panels->push_back(DsPanel{(int32_t)off, len});
      off += len;
      if (off > INT32_MAX) return -1;
    }
  }
  return off;
}

// Position ID of row-relative token t (Sec. 3.2: each token keeps the position
// it has in its unpacked sequence): t in the prompt, P + j for token j of a
// response, 0 for padding.
int32_t token_position(const Row& r, int32_t t) {
  const int32_t sid = seg_id(r, t);
  if (sid == 0) return t;
  if (sid > 0) return r.P + (t - r.off[sid - 1]);
  return 0;
}

// Positions: token_position of every token.
void build_positions(const Batch& bt, std::vector<int32_t>* out) {
  out->assign(bt.sumT, 0);
  int32_t* o = out->data();
  for (const Row& r : bt.rows) {
    for (int32_t t = 0; t < r.P; ++t) o[r.tok0 + t] = t;
    for (int k = 0; k < r.K; ++k)
      for (int32_t j = 0; j < r.len[k]; ++j) o[r.tok0 + r.off[k] + j] = r.P + j;
  }
}

// Rotary frequencies base^(-2j/d), j < d/2, in fp64.
void build_inv_freq(int d, float base, std::vector<double>* out) {
  out->resize(d / 2);
  for (int j = 0; j < d / 2; ++j) (*out)[j] = std::pow((double)base, -2.0 * j / d);
}

pp_status check_rope_base(float base) {
  if (!(base > 0.f) || !std::isfinite(base))
    return fail(PP_ERR_INVALID_ARGUMENT, "rope_base must be a finite value > 0, got %g", (double)base);
  return PP_OK;
}

// The log-probs' records, in row and token order: the last prompt position
// predicts the first token of every response, a response's token the next one.
struct LCounts {
  int64_t rows = 0;    // gather records: logit rows that predict a response token
  int64_t labels = 0;  // label tokens
  int64_t resp = 0;    // (row, response) slots
};

LCounts count_lplan(const Batch& bt) {
  LCounts n;
  n.resp = (int64_t)bt.B * bt.Kmax;
  for (const Row& r : bt.rows) {
    int64_t len = 0, some = 0;
    for (int k = 0; k < r.K; ++k) {
      len += r.len[k];
      some += r.len[k] > 0;
    }
    n.labels += len;
    if (some) n.rows += 1 + len - some;
  }
  return n;
}

// labels: flat position of each label token; label_out: its response's slot
// b * K_max + k; row_item: gather record of each flat logit row (-1: predicts
// nothing).  resp, label_out and row_item may be null.
void fill_lplan(const Batch& bt, LogitRowItem* rows, int32_t* labels, RespItem* resp, int32_t* label_out,
                int32_t* row_item) {
  if (row_item) std::fill(row_item, row_item + bt.sumT, -1);
  int32_t n_rows = 0, n_labels = 0;
  auto add_row = [&](int64_t logit_row, int32_t label_cnt) {
    LogitRowItem it{};
    it.logit_row = logit_row;
    it.label_off = n_labels;
    it.label_cnt = label_cnt;
    if (row_item) row_item[logit_row] = n_rows;
    rows[n_rows++] = it;
  };
  auto add_label = [&](int32_t pos, int32_t slot) {
    labels[n_labels] = pos;
    if (label_out) label_out[n_labels] = slot;
    ++n_labels;
  };
  for (int b = 0; b < bt.B; ++b) {
    const Row& r = bt.rows[b];
    int32_t some = 0;
    for (int k = 0; k < r.K; ++k) some += r.len[k] > 0;
    if (some) {
      add_row((int64_t)r.tok0 + r.P - 1, some);
      for (int k = 0; k < r.K; ++k)
        if (r.len[k] > 0) add_label(r.tok0 + r.off[k], b * bt.Kmax + k);
      for (int k = 0; k < r.K; ++k)
        for (int32_t j = 1; j < r.len[k]; ++j) {
          add_row((int64_t)r.tok0 + r.off[k] + j - 1, 1);
          add_label(r.tok0 + r.off[k] + j, b * bt.Kmax + k);
        }
    }
    for (int k = 0; resp && k < bt.Kmax; ++k) {
      RespItem ri{};
      ri.out = b * bt.Kmax + k;
      if (k < r.K) {
        ri.tok_begin = r.tok0 + r.off[k];
        ri.len = r.len[k];
      }
      *resp++ = ri;
    }
  }
}

// ---------------------------------------------------------------------------
// Workspace layout: a metadata prefix copied from the host, then scratch
// ---------------------------------------------------------------------------

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Region {
  size_t off = 0, bytes = 0;
};

struct Layout {
  std::vector<Region> regions;
  size_t meta_bytes = 0;   // host-staged prefix
  size_t total = 0;
  Layout() { regions.reserve(24); }
  size_t add(size_t bytes) {
    Region r;
    r.off = total;
    r.bytes = bytes;
    regions.push_back(r);
    total = align_up(total + bytes);
    return regions.size() - 1;
  }
};

// ---------------------------------------------------------------------------
// Pinned staging ring for plan metadata
// ---------------------------------------------------------------------------

struct StagingSlot {
  void* host = nullptr;       // mapped pinned host memory
  void* dev = nullptr;        // its device address (null: copies go through hipMemcpyAsync)
  size_t cap = 0;
  hipEvent_t done = nullptr;  // recorded on the copy's stream (its device's event)
  bool claimed = false;       // a call is filling it and enqueueing its launches
  bool pending = false;       // done is recorded
  uint64_t used = 0;          // order of the slots' last claims
};

// One ring per device: an event belongs to the device that was current when it
// was created, and a mapped address to the device it was taken for, so slots
// are never shared between devices.  A slot outgrown by a larger image is kept
// (in `retired`) rather than freed: a kernel has read it, and pinned memory is
// only released at unload.
constexpr int kStageSlots = 16;
struct StagingRing {
  StagingSlot slot[kStageSlots];
  uint64_t claims = 0;
  std::vector<void*> retired;
};

std::mutex g_stage_mu;
std::map<int, StagingRing> g_stage;

struct StagingRelease {
  ~StagingRelease() {
    // Only free what is no longer in flight; the runtime may already be down at
    // unload, in which case the OS reclaims the memory.
    for (auto& kv : g_stage) {
      for (auto& s : kv.second.slot) {
        if (s.pending && s.done) hipEventSynchronize(s.done);
        if (s.done) hipEventDestroy(s.done);
        if (s.host) hipHostFree(s.host);
        s = StagingSlot{};
      }
      for (void* h : kv.second.retired) hipHostFree(h);
      kv.second.retired.clear();
    }
  }
} g_stage_release;

// Claims a slot of the ring: the one claimed longest ago if its work is done, else one
// never used, else any whose work is done, else the one claimed longest ago, whose
// work the caller waits for (*wait).  A slot that another stream's long kernels hold is
// passed over, and nobody waits with the ring locked.
StagingSlot* claim_slot(StagingRing& ring, bool* wait) {
  auto done = [](const StagingSlot& s) {
    if (hipEventQuery(s.done) == hipSuccess) return true;
    (void)hipGetLastError();  // not ready (or an error, which the wait will report)
    return false;
  };
  for (;; std::this_thread::yield()) {  // all slots claimed by other threads: they are let go within their calls
    std::lock_guard<std::mutex> lk(g_stage_mu);
    StagingSlot *fresh = nullptr, *oldest = nullptr;
    for (StagingSlot& s : ring.slot) {
      if (s.claimed) continue;
      if (s.pending) oldest = !oldest || s.used < oldest->used ? &s : oldest;
      else if (!fresh) fresh = &s;
    }
    StagingSlot* s = oldest ? oldest : fresh;
    if (!s) continue;
    *wait = oldest && !done(*oldest);
    if (*wait && fresh) s = fresh;
    for (StagingSlot& other : ring.slot) {
      if (!*wait || s == fresh) break;
      if (&other != oldest && !other.claimed && done(other)) {
        s = &other;
        *wait = false;
      }
    }
    if (s == fresh) *wait = false;
    s->claimed = true;
    s->used = ++ring.claims;
    return s;
  }
}

// Stages `bytes` from `src` for device memory `dst` (on the current device,
// whose stream `stream` is) through a pinned slot of that device's ring, then
// calls `launch(dev_src)`, which enqueues the work that needs the data: with a
// mapped slot and a 16-byte aligned `dst`, dev_src is the slot's device address
// and a kernel that `launch` enqueues must copy it into `dst` before any kernel
// reads `dst`; otherwise the data is already on its way by hipMemcpyAsync and
// dev_src is null.  The slot's
// event is recorded after `launch` in every case, so the slot is not reused
// while a kernel may still read it.
template <typename Launch>
pp_status stage_with(void* dst, const void* src, size_t bytes, hipStream_t stream, Launch&& launch) {
  if (bytes == 0) return launch(nullptr);
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice(staging)");
  StagingRing* ring;
  {
    std::lock_guard<std::mutex> lk(g_stage_mu);
    ring = &g_stage[dev];
  }
  bool wait = false;
  StagingSlot& s = *claim_slot(*ring, &wait);
  struct Release {
    StagingSlot& s;
    ~Release() {
      std::lock_guard<std::mutex> lk(g_stage_mu);
      s.claimed = false;
    }
  } release{s};
  if (wait) {
    e = hipEventSynchronize(s.done);
    if (e != hipSuccess) return hip_fail(e, "hipEventSynchronize(staging)");
  }
  s.pending = false;
  if (!s.done) {
    e = hipEventCreateWithFlags(&s.done, hipEventDisableTiming);
    if (e != hipSuccess) return hip_fail(e, "hipEventCreate(staging)");
  }
  if (s.cap < bytes) {
    if (s.host) {
      std::lock_guard<std::mutex> lk(g_stage_mu);
      ring->retired.push_back(s.host);
    }
    s.host = s.dev = nullptr;
    s.cap = 0;
    size_t cap = std::max<size_t>(bytes, 1 << 20);
    // coherent: the copy kernel reads what the host just wrote, never a cached line
    e = hipHostMalloc(&s.host, cap, hipHostMallocMapped | hipHostMallocCoherent);
    if (e != hipSuccess) return hip_fail(e, "hipHostMalloc(staging)");
    s.cap = cap;
    void* d = nullptr;
    if (hipHostGetDevicePointer(&d, s.host, 0) == hipSuccess) s.dev = d;
    else (void)hipGetLastError();  // no mapped address: this slot copies with hipMemcpyAsync
  }
  memcpy(s.host, src, bytes);
  const void* dev_src = nullptr;
  if (s.dev && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
    dev_src = s.dev;
  } else {
    e = hipMemcpyAsync(dst, s.host, bytes, hipMemcpyHostToDevice, stream);
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(plan)");
  }
  const pp_status st = launch(dev_src);
  e = hipEventRecord(s.done, stream);
  if (e != hipSuccess) return hip_fail(e, "hipEventRecord(staging)");
  s.pending = true;
  return st;
}

// Copies `bytes` from `src` into device memory `dst` on `stream` (a copy kernel
// from the mapped slot, or hipMemcpyAsync).
pp_status stage_copy(void* dst, const void* src, size_t bytes, hipStream_t stream) {
  return stage_with(dst, src, bytes, stream, [&](const void* dev_src) -> pp_status {
    if (!dev_src) return PP_OK;
    StageLaunch a;
    a.src = dev_src;
    a.dst = dst;
    a.bytes = bytes;
    hipError_t e = launch_stage(a, stream);
    return e == hipSuccess ? PP_OK : hip_fail(e, "stage_kernel");
  });
}

// Serialises regions into one host image of the metadata prefix.
struct MetaImage {
  std::vector<uint8_t> buf;
  // the region's place in the image, to be filled in
  void* at(const Region& r) {
    if (buf.size() < r.off + r.bytes) {
      buf.resize(r.off + r.bytes);
    }
    return buf.data() + r.off;
  }
  void put(const Region& r, const void* src, size_t bytes) {
    void* dst = at(r);
    if (bytes) memcpy(dst, src, bytes);
  }
};

// ---------------------------------------------------------------------------
// Attention plan + layout
// ---------------------------------------------------------------------------

// bf16 copies of fp32 attention inputs live in the workspace after the plan.
struct CastRegions {
  bool on = false;
  size_t q = 0, k = 0, v = 0, dout = 0;
};

struct FwdPlan {
  QPlan q;
  Layout lay;
  size_t r_seg, r_items, r_kt, r_pos, r_freq;
  CastRegions cast;
};

void plan_fwd(const Batch& bt, pp_dtype dtype, int hq, int hkv, int d, FwdPlan* p) {
  build_qplan(bt, kFwdBlockM, kFwdBlockN, &p->q);
  p->lay = Layout();
  p->r_seg = p->lay.add((size_t)bt.sumT * 4);
  p->r_items = p->lay.add(p->q.items.size() * sizeof(QTileItem));
  p->r_kt = p->lay.add(p->q.ktiles.size() * sizeof(KTileEntry));
  // the rotary variant also stages positions and frequencies (last, so that
  // the plain forward copies only the prefix before them)
  p->r_pos = p->lay.add((size_t)bt.sumT * 4);
  p->r_freq = p->lay.add((size_t)d / 2 * 8);
  p->lay.meta_bytes = p->lay.total;
  if (dtype == PP_FP32) {
    p->cast.on = true;
    p->cast.q = p->lay.add((size_t)bt.sumT * hq * d * 2);
    p->cast.k = p->lay.add((size_t)bt.sumT * hkv * d * 2);
    p->cast.v = p->lay.add((size_t)bt.sumT * hkv * d * 2);
  }
}

// The backward's workspace: its linear part (metadata, per-token scratch, fp32
// callers' bf16 copies), which every call needs, and two regions that it uses if the
// workspace has room: the partial sums of cut key tiles, and last the stored dS
// (hq x ds_tiles tiles of 32 x 32 bf16).  A workspace that holds the linear part and
// the stored dS selects the stored-dS mode, whether or not there is room for the
// partial sums too; a smaller one the recompute mode.  In a batch so small that the
// partial sums are larger than its dS, a workspace with room for one of the two
// takes the partial sums if they fit (the recompute mode's own size must select it).
struct BwdPlan {
  QPlan dq;
  std::vector<KTileItem> kv;  // whole key tiles
  KvCut cut;                  // the same with the longest ones cut, if that pays
  std::vector<int32_t> row_kb0;
  std::vector<DsPanel> panels;
  int64_t ds_tiles = 0;  // per head; -1: the stored mode is not offered
  // workspace bytes without and with the partial sums (the same if no tile is cut)
  size_t lean_total[2], stored_total[2];
  // set for the workspace at hand by settle_bwd
  bool use_cut = false, store_ds = false;
  Layout lay;
  size_t r_seg, r_seg_hi, r_dq_items, r_dq_kt, r_kv_items, r_kv_parts, r_kv_splits, r_row_kb0, r_panels, r_pos, r_freq,
      r_ndelta, r_nlse2, r_kv_sums;
  size_t r_ds = 0;
  CastRegions cast;

  size_t lean_needed() const { return lean_total[0]; }
  size_t lean_wanted() const { return lean_total[1]; }
  size_t stored_wanted() const { return stored_total[1]; }
};

void lay_out_bwd(const Batch& bt, pp_dtype dtype, int hq, int hkv, int d, bool cut, BwdPlan* p) {
  p->use_cut = cut;
  p->cast = CastRegions();
  p->lay = Layout();
  p->r_seg = p->lay.add((size_t)bt.sumT * 4);
  p->r_seg_hi = p->lay.add((size_t)bt.sumT * 4);
  p->r_dq_items = p->lay.add(p->dq.items.size() * sizeof(QTileItem));
  p->r_dq_kt = p->lay.add(p->dq.ktiles.size() * sizeof(KTileEntry));
  p->r_kv_items = p->lay.add((cut ? p->cut.items : p->kv).size() * sizeof(KTileItem));
  p->r_kv_parts = p->lay.add(cut ? p->cut.parts.size() * sizeof(KTilePart) : 0);
  p->r_kv_splits = p->lay.add(cut ? p->cut.splits.size() * sizeof(KTileSplit) : 0);
  p->r_row_kb0 = p->lay.add(p->row_kb0.size() * 4);
  p->r_panels = p->lay.add(p->panels.size() * sizeof(DsPanel));
  p->r_pos = p->lay.add((size_t)bt.sumT * 4);
  p->r_freq = p->lay.add((size_t)d / 2 * 8);
  p->lay.meta_bytes = p->lay.total;
  p->r_ndelta = p->lay.add((size_t)hq * bt.sumT * 4);
  p->r_nlse2 = p->lay.add((size_t)hq * bt.sumT * 4);
  p->r_kv_sums = p->lay.add(cut ? (size_t)p->cut.slots * hkv * kv_part_bytes(d) : 0);
  if (dtype == PP_FP32) {
    p->cast.on = true;
    p->cast.q = p->lay.add((size_t)bt.sumT * hq * d * 2);
    p->cast.k = p->lay.add((size_t)bt.sumT * hkv * d * 2);
    p->cast.v = p->lay.add((size_t)bt.sumT * hkv * d * 2);
    p->cast.dout = p->lay.add((size_t)bt.sumT * hq * d * 2);
  }
  p->lean_total[cut] = p->lay.total;
  if (p->ds_tiles >= 0) p->r_ds = p->lay.add((size_t)p->ds_tiles * hq * 2048);
  p->stored_total[cut] = p->lay.total;
}

void plan_bwd(const Batch& bt, pp_dtype dtype, int hq, int hkv, int d, BwdPlan* p) {
  build_qplan(bt, kDqBlockM, kDqBlockN, &p->dq);
  build_kplan(bt, kBwdBlockN, &p->kv);
  p->ds_tiles = build_ds_panels(bt, kBwdBlockN, &p->row_kb0, &p->panels);
  split_kplan(p->kv, hq / hkv, hkv, &p->cut);
  if (!p->cut.items.empty()) lay_out_bwd(bt, dtype, hq, hkv, d, true, p);
  lay_out_bwd(bt, dtype, hq, hkv, d, false, p);
  if (p->cut.items.empty()) {
    p->lean_total[1] = p->lean_total[0];
    p->stored_total[1] = p->stored_total[0];
  }
}

// Fixes the mode and the layout for a workspace of at least lean_needed() bytes.
void settle_bwd(const Batch& bt, pp_dtype dtype, int hq, int hkv, int d, size_t ws_bytes, BwdPlan* p) {
  const bool sums_only = p->lean_total[1] >= p->stored_total[0] && ws_bytes >= p->lean_total[1] &&
                         ws_bytes < p->stored_total[1];
  p->store_ds = p->ds_tiles >= 0 && ws_bytes >= p->stored_total[0] && !sums_only;
  if (!p->cut.items.empty() && ws_bytes >= (p->store_ds ? p->stored_total[1] : p->lean_total[1]))
    lay_out_bwd(bt, dtype, hq, hkv, d, true, p);
}

// One workspace layout serves the log-prob forward and its backward: the
// backward also stages each label's response slot and, per flat logit row, the
// index of the gather record that reads it (-1 for rows that predict nothing).
struct LogprobPlan {
  LCounts n;
  Layout lay;
  size_t r_rows, r_labels, r_resp, r_label_out, r_row_item, r_tok;
};

void plan_logprob(const Batch& bt, LogprobPlan* p) {
  p->n = count_lplan(bt);
  p->lay = Layout();
  p->r_rows = p->lay.add(p->n.rows * sizeof(LogitRowItem));
  p->r_labels = p->lay.add(p->n.labels * 4);
  p->r_resp = p->lay.add(p->n.resp * sizeof(RespItem));
  p->r_label_out = p->lay.add(p->n.labels * 4);
  p->r_row_item = p->lay.add((size_t)bt.sumT * 4);
  p->lay.meta_bytes = p->lay.total;
  p->r_tok = p->lay.add((size_t)bt.sumT * 4);
}

// The forward's metadata (response records), or the backward's (label slots; dense: each row's record).
void logprob_image(const Batch& bt, const LogprobPlan& p, bool bwd, bool dense, MetaImage* img) {
  const auto& reg = p.lay.regions;
  img->buf.reserve(p.lay.meta_bytes);
  // the last region first: the image has its size before the places are taken
  if (dense) img->at(reg[p.r_row_item]);
  if (bwd) img->at(reg[p.r_label_out]);
  else img->at(reg[p.r_resp]);
  fill_lplan(bt, (LogitRowItem*)img->at(reg[p.r_rows]), (int32_t*)img->at(reg[p.r_labels]),
             bwd ? nullptr : (RespItem*)img->at(reg[p.r_resp]), bwd ? (int32_t*)img->at(reg[p.r_label_out]) : nullptr,
             dense ? (int32_t*)img->at(reg[p.r_row_item]) : nullptr);
}

// Reward-model head: each (row, response) slot's hidden row, and the distinct
// rows with the slots that read them.
struct RmPlan {
  std::vector<int64_t> slot_row;
  std::vector<RmRowSlots> rows;
  std::vector<int32_t> slots;
  Layout lay;
  size_t r_slot_row, r_rows, r_slots, r_row_rec;
};

// The distinct rows come in order of first use, each with its slots in slot order:
// a slot that ends in a response's last token has that row to itself, all empty
// responses of a row share its last prompt token.
void plan_rm(const Batch& bt, RmPlan* p) {
  p->slot_row.assign((size_t)bt.B * bt.Kmax, -1);
  p->rows.clear();
  p->slots.clear();
  for (int b = 0; b < bt.B; ++b) {
    const Row& r = bt.rows[b];
    bool empties = false;  // their record is in
    for (int k = 0; k < r.K; ++k) {
      const int64_t last = r.len[k] > 0 ? (int64_t)r.off[k] + r.len[k] - 1 : (int64_t)r.P - 1;
      if (last < 0) continue;
      p->slot_row[b * bt.Kmax + k] = r.tok0 + last;
      if (r.len[k] == 0 && empties) continue;
      RmRowSlots rec{r.tok0 + last, (int32_t)p->slots.size(), 1};
      p->slots.push_back(b * bt.Kmax + k);
      if (r.len[k] == 0) {
        empties = true;
        for (int j = k + 1; j < r.K; ++j)
          if (r.len[j] == 0) {
            p->slots.push_back(b * bt.Kmax + j);
            ++rec.slot_cnt;
          }
      }
      p->rows.push_back(rec);
    }
  }
  p->lay = Layout();
  p->r_slot_row = p->lay.add(p->slot_row.size() * 8);
  p->r_rows = p->lay.add(p->rows.size() * sizeof(RmRowSlots));
  p->r_slots = p->lay.add(p->slots.size() * 4);
  p->r_row_rec = p->lay.add((size_t)bt.sumT * 4);
  p->lay.meta_bytes = p->lay.total;
}

pp_status check_logprob_layout(const Batch& bt) {
  for (int b = 0; b < bt.B; ++b) {
    const Row& r = bt.rows[b];
    for (int k = 0; k < r.K; ++k)
      if (r.len[k] > 0 && r.P == 0)
        return fail(PP_ERR_BAD_LAYOUT,
                    "row %d has an empty prompt and a non-empty response: its first token has no "
                    "predicting position", b);
  }
  return PP_OK;
}

inline void* at(void* base, const Layout& lay, size_t region) {
  return (uint8_t*)base + lay.regions[region].off;
}

// ---------------------------------------------------------------------------
// Kernel timing
// ---------------------------------------------------------------------------

struct TimingRec {
  const char* name;
  hipEvent_t start, stop;
};

std::mutex g_time_mu;
std::atomic<bool> g_time_on{false};
std::vector<TimingRec> g_time_pending;
std::vector<hipEvent_t> g_event_pool;
struct TimingTotal {
  const char* name;
  double ms;
  int64_t launches;
};
std::vector<TimingTotal> g_time_totals;
std::vector<std::string> g_time_select;  // launch names to time; empty = every launch

bool timing_selected_locked(const char* name) {
  if (g_time_select.empty()) return true;
  for (const auto& n : g_time_select)
    if (n == name) return true;
  return false;
}

hipEvent_t pool_get() {
  if (!g_event_pool.empty()) {
    hipEvent_t e = g_event_pool.back();
    g_event_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

void drain_timing_locked() {
  for (auto& r : g_time_pending) {
    float ms = 0.f;
    // a launch whose events cannot be read (e.g. a failed record) is dropped,
    // not counted as a zero-length launch
    if (hipEventSynchronize(r.stop) != hipSuccess || hipEventElapsedTime(&ms, r.start, r.stop) != hipSuccess) {
      (void)hipGetLastError();
      g_event_pool.push_back(r.start);
      g_event_pool.push_back(r.stop);
      continue;
    }
    bool found = false;
    for (auto& t : g_time_totals)
      if (strcmp(t.name, r.name) == 0) {
        t.ms += ms;
        t.launches += 1;
        found = true;
      }
    if (!found) g_time_totals.push_back({r.name, (double)ms, 1});
    g_event_pool.push_back(r.start);
    g_event_pool.push_back(r.stop);
  }
  g_time_pending.clear();
}

}  // namespace

pp_status report_error(pp_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

pp_status report_hip_error(hipError_t e, const char* what) { return hip_fail(e, what); }

TimingScope::TimingScope(std::initializer_list<const char*> names, hipStream_t stream) : stream_(stream) {
  if (!g_time_on.load(std::memory_order_relaxed)) return;
  std::lock_guard<std::mutex> lk(g_time_mu);
  for (const char* name : names)
    if (!name_ && name && timing_selected_locked(name)) name_ = name;
  if (!name_) return;
  hipEvent_t a = pool_get(), b = pool_get();
  if (!a || !b || hipEventRecord(a, stream) != hipSuccess) {
    (void)hipGetLastError();
    if (a) g_event_pool.push_back(a);
    if (b) g_event_pool.push_back(b);
    return;
  }
  start_ = a;
  stop_ = b;
}

TimingScope::~TimingScope() {
  if (!start_) return;
  std::lock_guard<std::mutex> lk(g_time_mu);
  if (hipEventRecord(stop_, stream_) == hipSuccess) {
    g_time_pending.push_back({name_, start_, stop_});
  } else {
    (void)hipGetLastError();
    g_event_pool.push_back(start_);
    g_event_pool.push_back(stop_);
  }
}

}  // namespace pp

using namespace pp;

// ===========================================================================
// C ABI
// ===========================================================================

extern "C" {

#ifndef PP_BUILD_ID
#define PP_BUILD_ID "unknown"
#endif
int pp_version(void) { return 100; }

const char* pp_build_id(void) { return PP_BUILD_ID; }

const char* pp_status_string(pp_status s) {
  switch (s) {
    case PP_OK: return "ok";
    case PP_ERR_INVALID_ARGUMENT: return "invalid argument";
    case PP_ERR_BAD_LAYOUT: return "bad packed layout";
    case PP_ERR_UNSUPPORTED: return "unsupported";
    case PP_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
    case PP_ERR_HIP: return "HIP error";
    default: break;
  }
  return "unknown status";
}

const char* pp_last_error(void) { return g_last_error.c_str(); }

pp_status pp_workspace_size(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim,
                            int vocab, size_t* fwd, size_t* bwd, size_t* logprob, size_t* loss) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if ((st = check_dtype(dtype)) != PP_OK) return st;
  if (fwd || bwd) {
    st = check_heads(hq, hkv, head_dim);
    if (st != PP_OK) return st;
  }
  if (fwd) {
    FwdPlan p;
    plan_fwd(bt, dtype, hq, hkv, head_dim, &p);
    *fwd = p.lay.total;
  }
  if (bwd) {
    BwdPlan p;
    plan_bwd(bt, dtype, hq, hkv, head_dim, &p);
    *bwd = p.lean_wanted();  // the recompute mode; pp_bwd_stored_ds_workspace_size for the other
  }
  if (logprob) {
    if (vocab < 1) return fail(PP_ERR_INVALID_ARGUMENT, "vocab must be >= 1 for the logprob size");
    st = check_logprob_layout(bt);
    if (st != PP_OK) return st;
    LogprobPlan p;
    plan_logprob(bt, &p);
    *logprob = p.lay.total;
  }
  if (loss) *loss = align_up((size_t)bt.B * 4);
  return PP_OK;
}

}  // extern "C"

namespace pp {
namespace {

// Rotary arguments of the fused attention entry points (null for the plain ones).
struct RopeArgs {
  float base;
  void* q_rot;        // forward: rotated queries out (may be null)
  void* k_rot;        // forward: rotated keys out (required)
};

// The kernels move tensor rows in 16-byte vectors (and DMA them into LDS in
// 16-byte chunks), so every tensor argument must start on a 16-byte boundary.
inline bool aligned16(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15) == 0; }
// workspaces hold metadata records read by scalar loads, doubles and 16-byte
// vectors: they must start on a 256-byte boundary (hipMalloc and torch qualify)
inline bool aligned256(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 255) == 0; }
inline bool aligned4(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 3) == 0; }

pp_status check_fwd_ptrs(int sumT, const void* q, const void* k, const void* v, const void* o, const float* lse,
                         const RopeArgs* rope) {
  if (sumT > 0 && (!q || !k || !v || !o || !lse))
    return fail(PP_ERR_INVALID_ARGUMENT, "q, k, v, o and lse must be non-NULL");
  if (sumT > 0 && rope && !rope->k_rot) return fail(PP_ERR_INVALID_ARGUMENT, "k_rot must be non-NULL");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned4(lse) ||
      (rope && (!aligned16(rope->k_rot) || !aligned16(rope->q_rot))))
    return fail(PP_ERR_INVALID_ARGUMENT, "q, k, v, o (and q_rot, k_rot) must be 16-byte aligned, lse 4-byte aligned");
  return PP_OK;
}

pp_status check_bwd_ptrs(int sumT, const void* q, const void* k, const void* v, const void* o, const float* lse,
                         const void* dout, const void* dq, const void* dk, const void* dv) {
  if (sumT > 0 && (!q || !k || !v || !o || !lse || !dout || !dq || !dk || !dv))
    return fail(PP_ERR_INVALID_ARGUMENT, "q, k, v, o, lse, dout, dq, dk and dv must be non-NULL");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(dout) || !aligned16(dq) ||
      !aligned16(dk) || !aligned16(dv) || !aligned4(lse))
    return fail(PP_ERR_INVALID_ARGUMENT, "q, k, v, o, dout, dq, dk and dv must be 16-byte aligned, lse 4-byte aligned");
  return PP_OK;
}

// The forward's metadata prefix as one host image (rotary positions and
// frequencies included when rope_base is given).
void fwd_image(const Batch& bt, const FwdPlan& p, int head_dim, const double* rope_base, MetaImage* out) {
  MetaImage& img = *out;
  img.buf.reserve(p.lay.meta_bytes);
  fill_seg_lo(bt, (int32_t*)img.at(p.lay.regions[p.r_seg]));
  img.put(p.lay.regions[p.r_items], p.q.items.data(), p.q.items.size() * sizeof(QTileItem));
  img.put(p.lay.regions[p.r_kt], p.q.ktiles.data(), p.q.ktiles.size() * sizeof(KTileEntry));
  std::vector<int32_t> pos;
  std::vector<double> freq;
  if (rope_base) {
    build_positions(bt, &pos);
    build_inv_freq(head_dim, *rope_base, &freq);
    img.put(p.lay.regions[p.r_pos], pos.data(), pos.size() * 4);
    img.put(p.lay.regions[p.r_freq], freq.data(), freq.size() * 8);
  }
}

// What precedes the passes: metadata still to be copied into ws, if any.
StageLaunch stage_of(void* ws, const void* stage_src, size_t stage_bytes) {
  StageLaunch a;
  a.src = stage_src;
  a.dst = ws;
  a.bytes = stage_src ? stage_bytes : 0;
  return a;
}

// Enqueues the forward on metadata already staged in ws, or (stage_src, mapped
// pinned memory) copied there ahead of its kernels.
pp_status fwd_launch(const FwdPlan& p, void* ws, int sumT, pp_dtype dtype, int hq, int hkv, int head_dim,
                     float scale, const void* q, const void* k, const void* v, void* o, float* lse,
                     const RopeArgs* rope, hipStream_t s, const void* stage_src = nullptr, size_t stage_bytes = 0) {
  hipError_t e;
  StageLaunch pre = stage_of(ws, stage_src, stage_bytes);
  const int32_t* d_pos = (const int32_t*)at(ws, p.lay, p.r_pos);
  const double* d_freq = (const double*)at(ws, p.lay, p.r_freq);
  if (rope) {
    // keys are rotated once, in the caller's dtype, into k_rot; the queries are
    // rotated inside the attention kernel
    if ((e = launch_stage(pre, s)) != hipSuccess) return hip_fail(e, "stage_kernel");
    pre = StageLaunch();
    RopeLaunch r{};
    r.x = k;
    r.y = rope->k_rot;
    r.pos = d_pos;
    r.inv_freq = d_freq;
    r.sumT = sumT;
    r.heads = hkv;
    r.head_dim = head_dim;
    r.inverse = false;
    r.dtype = dtype == PP_FP32 ? kFP32 : kBF16;
    if ((e = launch_rope(r, s)) != hipSuccess) return hip_fail(e, "rotary embedding launch");
    k = rope->k_rot;
  }
  if (p.cast.on) {
    // the kernels read bf16: round fp32 inputs once (nearest even)
    void* qb = at(ws, p.lay, p.cast.q);
    void* kb = at(ws, p.lay, p.cast.k);
    void* vb = at(ws, p.lay, p.cast.v);
    pre.cast[0] = {(const float*)q, qb, (int64_t)sumT * hq * head_dim};
    pre.cast[1] = {(const float*)k, kb, (int64_t)sumT * hkv * head_dim};
    pre.cast[2] = {(const float*)v, vb, (int64_t)sumT * hkv * head_dim};
    q = qb;
    k = kb;
    v = vb;
  }
  if ((e = launch_stage(pre, s)) != hipSuccess) return hip_fail(e, "stage_kernel");
  AttnFwdLaunch a{};
  a.q = q;
  a.k = k;
  a.v = v;
  a.o = o;
  a.lse = lse;
  a.items = (const QTileItem*)at(ws, p.lay, p.r_items);
  a.ktiles = (const KTileEntry*)at(ws, p.lay, p.r_kt);
  a.seg_lo = (const int32_t*)at(ws, p.lay, p.r_seg);
  a.n_items = (int)p.q.items.size();
  a.hq = hq;
  a.hkv = hkv;
  a.head_dim = head_dim;
  a.sumT = sumT;
  a.scale = scale > 0.f ? scale : 1.0f / std::sqrt((float)head_dim);
  a.dtype = dtype == PP_FP32 ? kFP32 : kBF16;
  if (rope) {
    a.rope = true;
    a.pos = d_pos;
    a.inv_freq = d_freq;
    a.q_rot = rope->q_rot;
  }
  e = launch_attn_fwd(a, s);
  if (e != hipSuccess) return hip_fail(e, "attention forward launch");
  return PP_OK;
}


pp_status attn_fwd_impl(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim, float scale,
                        const void* q, const void* k, const void* v, void* o, float* lse, const RopeArgs* rope,
                        void* ws, size_t ws_bytes, void* hip_stream) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if ((st = check_heads(hq, hkv, head_dim)) != PP_OK) return st;
  if ((st = check_dtype(dtype)) != PP_OK) return st;
  if (rope && (st = check_rope_base(rope->base)) != PP_OK) return st;
  if ((st = check_fwd_ptrs(bt.sumT, q, k, v, o, lse, rope)) != PP_OK) return st;
  FwdPlan p;
  plan_fwd(bt, dtype, hq, hkv, head_dim, &p);
  if (ws_bytes < p.lay.total)
    return fail(PP_ERR_WORKSPACE_TOO_SMALL, "forward needs %zu workspace bytes, got %zu", p.lay.total,
                ws_bytes);
  if (p.lay.total && !ws) return fail(PP_ERR_INVALID_ARGUMENT, "ws is NULL");
  if (ws && !aligned256(ws)) return fail(PP_ERR_INVALID_ARGUMENT, "ws must be 256-byte aligned");
  if (bt.sumT == 0) return PP_OK;
  MetaImage img;
  const double base = rope ? rope->base : 0.0;
  fwd_image(bt, p, head_dim, rope ? &base : nullptr, &img);
  hipStream_t s = (hipStream_t)hip_stream;
  return stage_with(ws, img.buf.data(), img.buf.size(), s, [&](const void* dev_src) {
    return fwd_launch(p, ws, bt.sumT, dtype, hq, hkv, head_dim, scale, q, k, v, o, lse, rope, s, dev_src,
                      img.buf.size());
  });
}

}  // namespace

pp_status attn_fwd_fixed_scratch(const pp_pack_desc* desc, int hq, int hkv, int head_dim, float scale,
                                 const void* q, const void* k, const void* v, void* o, float* lse,
                                 size_t scratch_cap, pp_status (*get_scratch)(void** ptr), hipStream_t s) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if ((st = check_heads(hq, hkv, head_dim)) != PP_OK) return st;
  if ((st = check_fwd_ptrs(bt.sumT, q, k, v, o, lse, nullptr)) != PP_OK) return st;
  FwdPlan p;
  plan_fwd(bt, PP_BF16, hq, hkv, head_dim, &p);
  if (p.lay.total > scratch_cap)
    return fail(PP_ERR_WORKSPACE_TOO_SMALL,
                "this pack's forward plan needs %zu bytes of scratch; the library's static scratch holds %zu "
                "(use pp_attn_fwd with a workspace)", p.lay.total, scratch_cap);
  if (bt.sumT == 0) return PP_OK;
  void* ws = nullptr;
  if ((st = get_scratch(&ws)) != PP_OK) return st;
  MetaImage img;
  fwd_image(bt, p, head_dim, nullptr, &img);
  // pageable host source: the runtime stages it itself, so nothing is allocated here
  const hipError_t e = hipMemcpyAsync(ws, img.buf.data(), img.buf.size(), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(plan into static scratch)");
  return fwd_launch(p, ws, bt.sumT, PP_BF16, hq, hkv, head_dim, scale, q, k, v, o, lse, nullptr, s);
}

namespace {

// The backward's metadata prefix as one host image.
void bwd_image(const Batch& bt, const BwdPlan& p, int head_dim, const double* rope_base, MetaImage* out) {
  MetaImage& img = *out;
  img.buf.reserve(p.lay.meta_bytes);
  fill_seg_lo(bt, (int32_t*)img.at(p.lay.regions[p.r_seg]));
  fill_seg_hi(bt, (int32_t*)img.at(p.lay.regions[p.r_seg_hi]));
  img.put(p.lay.regions[p.r_dq_items], p.dq.items.data(), p.dq.items.size() * sizeof(QTileItem));
  img.put(p.lay.regions[p.r_dq_kt], p.dq.ktiles.data(), p.dq.ktiles.size() * sizeof(KTileEntry));
  const std::vector<KTileItem>& kv = p.use_cut ? p.cut.items : p.kv;
  img.put(p.lay.regions[p.r_kv_items], kv.data(), kv.size() * sizeof(KTileItem));
  if (p.use_cut) {
    img.put(p.lay.regions[p.r_kv_parts], p.cut.parts.data(), p.cut.parts.size() * sizeof(KTilePart));
    img.put(p.lay.regions[p.r_kv_splits], p.cut.splits.data(), p.cut.splits.size() * sizeof(KTileSplit));
  }
  img.put(p.lay.regions[p.r_row_kb0], p.row_kb0.data(), p.row_kb0.size() * 4);
  img.put(p.lay.regions[p.r_panels], p.panels.data(), p.panels.size() * sizeof(DsPanel));
  std::vector<int32_t> pos;
  std::vector<double> freq;
  if (rope_base) {
    build_positions(bt, &pos);
    build_inv_freq(head_dim, *rope_base, &freq);
    img.put(p.lay.regions[p.r_pos], pos.data(), pos.size() * 4);
    img.put(p.lay.regions[p.r_freq], freq.data(), freq.size() * 8);
  }
}

// Enqueues the backward on metadata already staged in ws, or (stage_src, mapped
// pinned memory) copied there ahead of its kernels.
pp_status bwd_launch(const BwdPlan& p, void* ws, int sumT, pp_dtype dtype, int hq, int hkv, int head_dim,
                     float scale, const void* q, const void* k, const void* v, const void* o,
                     const float* lse, const void* dout, void* dq, void* dk, void* dv, bool rope, hipStream_t s,
                     const void* stage_src = nullptr, size_t stage_bytes = 0) {
  hipError_t e;
  StageLaunch pre = stage_of(ws, stage_src, stage_bytes);
  const void* dout_bf = dout;
  if (p.cast.on) {
    void* qb = at(ws, p.lay, p.cast.q);
    void* kb = at(ws, p.lay, p.cast.k);
    void* vb = at(ws, p.lay, p.cast.v);
    void* db = at(ws, p.lay, p.cast.dout);
    pre.cast[0] = {(const float*)q, qb, (int64_t)sumT * hq * head_dim};
    pre.cast[1] = {(const float*)k, kb, (int64_t)sumT * hkv * head_dim};
    pre.cast[2] = {(const float*)v, vb, (int64_t)sumT * hkv * head_dim};
    pre.cast[3] = {(const float*)dout, db, (int64_t)sumT * hq * head_dim};
    q = qb;
    k = kb;
    v = vb;
    dout_bf = db;
  }
  if ((e = launch_stage(pre, s)) != hipSuccess) return hip_fail(e, "stage_kernel");
  AttnBwdLaunch a{};
  a.q = q;
  a.k = k;
  a.v = v;
  a.o = o;
  a.lse = lse;
  a.dout = dout_bf;
  a.dout_orig = dout;
  a.dq = dq;
  a.dk = dk;
  a.dv = dv;
  a.ndelta = (float*)at(ws, p.lay, p.r_ndelta);
  a.nlse2 = (float*)at(ws, p.lay, p.r_nlse2);
  a.dq_items = (const QTileItem*)at(ws, p.lay, p.r_dq_items);
  a.dq_ktiles = (const KTileEntry*)at(ws, p.lay, p.r_dq_kt);
  a.n_dq_items = (int)p.dq.items.size();
  a.kv_items = (const KTileItem*)at(ws, p.lay, p.r_kv_items);
  a.n_kv_items = (int)(p.use_cut ? p.cut.items : p.kv).size();
  a.kv_parts = (const KTilePart*)at(ws, p.lay, p.r_kv_parts);
  a.kv_splits = (const KTileSplit*)at(ws, p.lay, p.r_kv_splits);
  a.n_kv_splits = p.use_cut ? (int)p.cut.splits.size() : 0;
  a.kv_part = (float*)at(ws, p.lay, p.r_kv_sums);
  a.seg_lo = (const int32_t*)at(ws, p.lay, p.r_seg);
  a.seg_hi = (const int32_t*)at(ws, p.lay, p.r_seg_hi);
  a.hq = hq;
  a.hkv = hkv;
  a.head_dim = head_dim;
  a.sumT = sumT;
  a.scale = scale > 0.f ? scale : 1.0f / std::sqrt((float)head_dim);
  a.dtype = dtype == PP_FP32 ? kFP32 : kBF16;
  if (rope) {
    a.rope = true;
    a.pos = (const int32_t*)at(ws, p.lay, p.r_pos);
    a.inv_freq = (const double*)at(ws, p.lay, p.r_freq);
  }
  if (p.store_ds) {
    a.ds = (__bf16*)at(ws, p.lay, p.r_ds);
    a.row_kb0 = (const int32_t*)at(ws, p.lay, p.r_row_kb0);
    a.kb_panel = (const DsPanel*)at(ws, p.lay, p.r_panels);
    a.ds_tiles = p.ds_tiles;
  }
  e = launch_attn_bwd(a, s);
  if (e != hipSuccess) return hip_fail(e, "attention backward launch");
  return PP_OK;
}


pp_status attn_bwd_impl(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim, float scale,
                        const void* q, const void* k, const void* v, const void* o, const float* lse,
                        const void* dout, void* dq, void* dk, void* dv, const float* rope_base, void* ws,
                        size_t ws_bytes, void* hip_stream) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if ((st = check_heads(hq, hkv, head_dim)) != PP_OK) return st;
  if ((st = check_dtype(dtype)) != PP_OK) return st;
  if (rope_base && (st = check_rope_base(*rope_base)) != PP_OK) return st;
  if ((st = check_bwd_ptrs(bt.sumT, q, k, v, o, lse, dout, dq, dk, dv)) != PP_OK) return st;
  BwdPlan p;
  plan_bwd(bt, dtype, hq, hkv, head_dim, &p);
  if (ws_bytes < p.lean_needed())
    return fail(PP_ERR_WORKSPACE_TOO_SMALL,
                "backward needs %zu workspace bytes (%zu with its partial sums, %zu with the stored dS), got %zu",
                p.lean_needed(), p.lean_wanted(), p.stored_wanted(), ws_bytes);
  settle_bwd(bt, dtype, hq, hkv, head_dim, ws_bytes, &p);
  if (p.lean_needed() && !ws) return fail(PP_ERR_INVALID_ARGUMENT, "ws is NULL");
  if (ws && !aligned256(ws)) return fail(PP_ERR_INVALID_ARGUMENT, "ws must be 256-byte aligned");
  if (bt.sumT == 0) return PP_OK;
  MetaImage img;
  const double base = rope_base ? *rope_base : 0.0;
  bwd_image(bt, p, head_dim, rope_base ? &base : nullptr, &img);
  hipStream_t s = (hipStream_t)hip_stream;
  return stage_with(ws, img.buf.data(), img.buf.size(), s, [&](const void* dev_src) {
    return bwd_launch(p, ws, bt.sumT, dtype, hq, hkv, head_dim, scale, q, k, v, o, lse, dout, dq, dk, dv,
                      rope_base != nullptr, s, dev_src, img.buf.size());
  });
}

// Workspace of pp_rope: positions then frequencies.
struct RopePlan {
  Layout lay;
  size_t r_pos, r_freq;
};

void plan_rope(const Batch& bt, int d, RopePlan* p) {
  p->lay = Layout();
  p->r_pos = p->lay.add((size_t)bt.sumT * 4);
  p->r_freq = p->lay.add((size_t)d / 2 * 8);
  p->lay.meta_bytes = p->lay.total;
}

pp_status check_rope_dim(int d) {
  if (d < 8 || d > 1024 || d % 8)
    return fail(PP_ERR_UNSUPPORTED, "rotary head_dim %d not supported (a multiple of 8 in [8, 1024])", d);
  return PP_OK;
}

}  // namespace
}  // namespace pp

// A staged attention plan: the pack's forward and backward metadata (work
// lists, segment bounds, rotary positions) already in the caller's workspace,
// with the host-side launch summary.  Built once per pack (Sec. 3.2's packing
// is fixed for a training step) and reused by every layer's forward and
// backward, which then enqueue kernels only.
struct pp_plan {
  pp_dtype dtype;
  int hq, hkv, head_dim;
  bool rope;
  int sumT;
  pp::FwdPlan fwd;
  pp::BwdPlan bwd;
  void* ws;        // caller's workspace: forward region first, backward at bwd_off
  size_t bwd_off;
};

namespace pp {
namespace {

pp_status plan_common(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim,
                      const float* rope_base, Batch* bt, pp_plan* p) {
  pp_status st = read_desc(desc, bt);
  if (st != PP_OK) return st;
  if ((st = check_heads(hq, hkv, head_dim)) != PP_OK) return st;
  if ((st = check_dtype(dtype)) != PP_OK) return st;
  if (rope_base && (st = check_rope_base(*rope_base)) != PP_OK) return st;
  p->dtype = dtype;
  p->hq = hq;
  p->hkv = hkv;
  p->head_dim = head_dim;
  p->rope = rope_base != nullptr;
  p->sumT = bt->sumT;
  plan_fwd(*bt, dtype, hq, hkv, head_dim, &p->fwd);
  plan_bwd(*bt, dtype, hq, hkv, head_dim, &p->bwd);
  p->bwd_off = align_up(p->fwd.lay.total);
  return PP_OK;
}

}  // namespace
}  // namespace pp

extern "C" {

pp_status pp_plan_workspace_size(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim,
                                 size_t* bytes) {
  if (!bytes) return fail(PP_ERR_INVALID_ARGUMENT, "bytes is NULL");
  Batch bt;
  pp_plan p{};
  pp_status st = plan_common(desc, dtype, hq, hkv, head_dim, nullptr, &bt, &p);
  if (st != PP_OK) return st;
  *bytes = p.bwd_off + p.bwd.lean_wanted();
  return PP_OK;
}

pp_status pp_bwd_stored_ds_workspace_size(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim,
                                          size_t* bwd, size_t* plan) {
  Batch bt;
  pp_plan p{};
  pp_status st = plan_common(desc, dtype, hq, hkv, head_dim, nullptr, &bt, &p);
  if (st != PP_OK) return st;
  if (p.bwd.ds_tiles < 0)
    return fail(PP_ERR_UNSUPPORTED, "the stored dS of this batch does not fit 32-bit tile offsets");
  if (bwd) *bwd = p.bwd.stored_wanted();
  if (plan) *plan = p.bwd_off + p.bwd.stored_wanted();
  return PP_OK;
}

pp_status pp_plan_create(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim,
                         const float* rope_base, void* ws, size_t ws_bytes, void* hip_stream, pp_plan** plan) {
  if (!plan) return fail(PP_ERR_INVALID_ARGUMENT, "plan is NULL");
  *plan = nullptr;
  pp_plan* p = new (std::nothrow) pp_plan();
  if (!p) return fail(PP_ERR_INVALID_ARGUMENT, "out of host memory for the plan");
  Batch bt;
  pp_status st = plan_common(desc, dtype, hq, hkv, head_dim, rope_base, &bt, p);
  const size_t lean = st == PP_OK ? p->bwd_off + p->bwd.lean_needed() : 0;
  if (st == PP_OK && ws_bytes < lean)
    st = fail(PP_ERR_WORKSPACE_TOO_SMALL,
              "the plan needs %zu workspace bytes (%zu with its partial sums, %zu with the stored dS), got %zu", lean,
              p->bwd_off + p->bwd.lean_wanted(), p->bwd_off + p->bwd.stored_wanted(), ws_bytes);
  if (st == PP_OK) settle_bwd(bt, dtype, hq, hkv, head_dim, ws_bytes - p->bwd_off, &p->bwd);
  if (st == PP_OK && lean && !ws) st = fail(PP_ERR_INVALID_ARGUMENT, "ws is NULL");
  if (st == PP_OK && ws && !aligned256(ws)) st = fail(PP_ERR_INVALID_ARGUMENT, "ws must be 256-byte aligned");
  if (st == PP_OK && bt.sumT > 0) {
    // one image: the forward's metadata at 0, the backward's at bwd_off
    const double base = rope_base ? *rope_base : 0.0;
    MetaImage fi, bi;
    fwd_image(bt, p->fwd, head_dim, rope_base ? &base : nullptr, &fi);
    bwd_image(bt, p->bwd, head_dim, rope_base ? &base : nullptr, &bi);
    std::vector<uint8_t> img(p->bwd_off + bi.buf.size(), 0);
    if (!fi.buf.empty()) memcpy(img.data(), fi.buf.data(), fi.buf.size());
    if (!bi.buf.empty()) memcpy(img.data() + p->bwd_off, bi.buf.data(), bi.buf.size());
    st = stage_copy(ws, img.data(), img.size(), (hipStream_t)hip_stream);
  }
  if (st != PP_OK) {
    delete p;
    return st;
  }
  p->ws = ws;
  *plan = p;
  return PP_OK;
}

pp_status pp_plan_destroy(pp_plan* plan) {
  delete plan;
  return PP_OK;
}

pp_status pp_attn_fwd_planned(const pp_plan* plan, float scale, const void* q, const void* k, const void* v,
                              void* o, float* lse, void* q_rot, void* k_rot, void* hip_stream) {
  if (!plan) return fail(PP_ERR_INVALID_ARGUMENT, "plan is NULL");
  RopeArgs r{0.f, q_rot, k_rot};
  const RopeArgs* rope = plan->rope ? &r : nullptr;
  pp_status st = check_fwd_ptrs(plan->sumT, q, k, v, o, lse, rope);
  if (st != PP_OK) return st;
  if (plan->sumT == 0) return PP_OK;
  return fwd_launch(plan->fwd, plan->ws, plan->sumT, plan->dtype, plan->hq, plan->hkv, plan->head_dim, scale, q, k,
                    v, o, lse, rope, (hipStream_t)hip_stream);
}

pp_status pp_attn_bwd_planned(const pp_plan* plan, float scale, const void* q, const void* k, const void* v,
                              const void* o, const float* lse, const void* dout, void* dq, void* dk, void* dv,
                              void* hip_stream) {
  if (!plan) return fail(PP_ERR_INVALID_ARGUMENT, "plan is NULL");
  pp_status st = check_bwd_ptrs(plan->sumT, q, k, v, o, lse, dout, dq, dk, dv);
  if (st != PP_OK) return st;
  if (plan->sumT == 0) return PP_OK;
  void* ws_b = static_cast<char*>(plan->ws) + plan->bwd_off;
  return bwd_launch(plan->bwd, ws_b, plan->sumT, plan->dtype, plan->hq, plan->hkv, plan->head_dim, scale, q, k, v, o,
                    lse, dout, dq, dk, dv, plan->rope, (hipStream_t)hip_stream);
}

pp_status pp_attn_fwd(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim,
                      float scale, const void* q, const void* k, const void* v, void* o,
                      float* lse, void* ws, size_t ws_bytes, void* hip_stream) {
  return attn_fwd_impl(desc, dtype, hq, hkv, head_dim, scale, q, k, v, o, lse, nullptr, ws, ws_bytes, hip_stream);
}

pp_status pp_attn_bwd(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim,
                      float scale, const void* q, const void* k, const void* v, const void* o,
                      const float* lse, const void* dout, void* dq, void* dk, void* dv, void* ws,
                      size_t ws_bytes, void* hip_stream) {
  return attn_bwd_impl(desc, dtype, hq, hkv, head_dim, scale, q, k, v, o, lse, dout, dq, dk, dv, nullptr, ws,
                       ws_bytes, hip_stream);
}

pp_status pp_attn_fwd_rope(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim,
                           float scale, float rope_base, const void* q, const void* k, const void* v,
                           void* o, float* lse, void* q_rot, void* k_rot, void* ws, size_t ws_bytes,
                           void* hip_stream) {
  RopeArgs r{rope_base, q_rot, k_rot};
  return attn_fwd_impl(desc, dtype, hq, hkv, head_dim, scale, q, k, v, o, lse, &r, ws, ws_bytes, hip_stream);
}

pp_status pp_attn_bwd_rope(const pp_pack_desc* desc, pp_dtype dtype, int hq, int hkv, int head_dim,
                           float scale, float rope_base, const void* q_rot, const void* k_rot,
                           const void* v, const void* o, const float* lse, const void* dout, void* dq,
                           void* dk, void* dv, void* ws, size_t ws_bytes, void* hip_stream) {
  return attn_bwd_impl(desc, dtype, hq, hkv, head_dim, scale, q_rot, k_rot, v, o, lse, dout, dq, dk, dv,
                       &rope_base, ws, ws_bytes, hip_stream);
}

pp_status pp_rope_workspace_size(const pp_pack_desc* desc, int head_dim, size_t* bytes) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if ((st = check_rope_dim(head_dim)) != PP_OK) return st;
  if (!bytes) return fail(PP_ERR_INVALID_ARGUMENT, "bytes is NULL");
  RopePlan p;
  plan_rope(bt, head_dim, &p);
  *bytes = p.lay.total;
  return PP_OK;
}

pp_status pp_rope(const pp_pack_desc* desc, pp_dtype dtype, int heads, int head_dim, float rope_base,
                  int inverse, const void* x, void* y, void* ws, size_t ws_bytes, void* hip_stream) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if ((st = check_dtype(dtype)) != PP_OK) return st;
  if ((st = check_rope_dim(head_dim)) != PP_OK) return st;
  if ((st = check_rope_base(rope_base)) != PP_OK) return st;
  if (heads < 1) return fail(PP_ERR_INVALID_ARGUMENT, "heads must be >= 1");
  if (bt.sumT > 0 && (!x || !y)) return fail(PP_ERR_INVALID_ARGUMENT, "x and y must be non-NULL");
  if (!aligned16(x) || !aligned16(y)) return fail(PP_ERR_INVALID_ARGUMENT, "x and y must be 16-byte aligned");
  RopePlan p;
  plan_rope(bt, head_dim, &p);
  if (ws_bytes < p.lay.total)
    return fail(PP_ERR_WORKSPACE_TOO_SMALL, "rope needs %zu workspace bytes, got %zu", p.lay.total, ws_bytes);
  if (!ws) return fail(PP_ERR_INVALID_ARGUMENT, "ws is NULL");
  if (ws && !aligned256(ws)) return fail(PP_ERR_INVALID_ARGUMENT, "ws must be 256-byte aligned");
  if (bt.sumT == 0) return PP_OK;
  hipStream_t s = (hipStream_t)hip_stream;
  std::vector<int32_t> pos;
  std::vector<double> freq;
  build_positions(bt, &pos);
  build_inv_freq(head_dim, rope_base, &freq);
  MetaImage img;
  img.put(p.lay.regions[p.r_pos], pos.data(), pos.size() * 4);
  img.put(p.lay.regions[p.r_freq], freq.data(), freq.size() * 8);
  if ((st = stage_copy(ws, img.buf.data(), img.buf.size(), s)) != PP_OK) return st;
  RopeLaunch r{};
  r.x = x;
  r.y = y;
  r.pos = (const int32_t*)at(ws, p.lay, p.r_pos);
  r.inv_freq = (const double*)at(ws, p.lay, p.r_freq);
  r.sumT = bt.sumT;
  r.heads = heads;
  r.head_dim = head_dim;
  r.inverse = inverse != 0;
  r.dtype = dtype == PP_FP32 ? kFP32 : kBF16;
  const hipError_t e = launch_rope(r, s);
  if (e != hipSuccess) return hip_fail(e, "rotary embedding launch");
  return PP_OK;
}

pp_status pp_seq_logprob(const pp_pack_desc* desc, pp_dtype logits_dtype, int vocab,
                         const void* logits, const int32_t* tokens, float* seq_logp,
                         float* tok_logp, void* ws, size_t ws_bytes, void* hip_stream) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if ((st = check_dtype(logits_dtype)) != PP_OK) return st;
  if (vocab < 1) return fail(PP_ERR_INVALID_ARGUMENT, "vocab must be >= 1");
  if ((st = check_logprob_layout(bt)) != PP_OK) return st;
  if (bt.Kmax > 0 && !seq_logp) return fail(PP_ERR_INVALID_ARGUMENT, "seq_logp is NULL");
  if (bt.sumT > 0 && (!logits || !tokens))
    return fail(PP_ERR_INVALID_ARGUMENT, "logits and tokens must be non-NULL");
  LogprobPlan p;
  plan_logprob(bt, &p);
  if (ws_bytes < p.lay.total)
    return fail(PP_ERR_WORKSPACE_TOO_SMALL, "logprob needs %zu workspace bytes, got %zu", p.lay.total,
                ws_bytes);
  if (p.lay.total && !ws) return fail(PP_ERR_INVALID_ARGUMENT, "ws is NULL");
  if (ws && !aligned256(ws)) return fail(PP_ERR_INVALID_ARGUMENT, "ws must be 256-byte aligned");
  if (bt.Kmax == 0 && (bt.sumT == 0 || !tok_logp)) return PP_OK;
  hipStream_t s = (hipStream_t)hip_stream;
  MetaImage img;
  logprob_image(bt, p, false, false, &img);
  LogprobLaunch a{};
  a.logits = logits;
  a.tokens = tokens;
  a.tok = tok_logp ? tok_logp : (float*)at(ws, p.lay, p.r_tok);
  a.seq = seq_logp;
  a.rows = (const LogitRowItem*)at(ws, p.lay, p.r_rows);
  a.labels = (const int32_t*)at(ws, p.lay, p.r_labels);
  a.resp = (const RespItem*)at(ws, p.lay, p.r_resp);
  a.n_rows = (int)p.n.rows;
  a.n_resp = (int)p.n.resp;
  a.vocab = vocab;
  a.dtype = logits_dtype == PP_FP32 ? kFP32 : kBF16;
  return stage_with(ws, img.buf.data(), img.buf.size(), s, [&](const void* dev_src) -> pp_status {
    StageLaunch pre = stage_of(ws, dev_src, img.buf.size());
    if (tok_logp) {
      // the caller's per-token output reads 0 off the responses; workspace scratch
      // is only read back at response positions, so it is not cleared
      pre.zero = tok_logp;
      pre.n_zero = bt.sumT;
    }
    hipError_t e = launch_stage(pre, s);
    if (e != hipSuccess) return hip_fail(e, "stage_kernel");
    e = launch_logprob(a, s);
    return e == hipSuccess ? PP_OK : hip_fail(e, "logprob launch");
  });
}

}  // extern "C"

namespace pp {
namespace {

// The log-prob backward, dense (dlogits [sumT, vocab]) or gathered (one row per
// logit row that predicts a response token, [n, vocab], and row_index [n]).
pp_status logprob_bwd_impl(const pp_pack_desc* desc, pp_dtype logits_dtype, int vocab, const void* logits,
                           const int32_t* tokens, const float* dseq, void* dlogits, bool gathered,
                           int32_t* row_index, void* ws, size_t ws_bytes, void* hip_stream) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if ((st = check_dtype(logits_dtype)) != PP_OK) return st;
  if (vocab < 1) return fail(PP_ERR_INVALID_ARGUMENT, "vocab must be >= 1");
  if ((st = check_logprob_layout(bt)) != PP_OK) return st;
  if (bt.Kmax > kMaxRowLabels)
    return fail(PP_ERR_UNSUPPORTED, "the log-prob backward takes at most %d responses per row (max_resp %d)",
                kMaxRowLabels, bt.Kmax);
  if (bt.sumT == 0) return PP_OK;
  LogprobPlan p;
  plan_logprob(bt, &p);
  if (gathered && p.n.rows == 0) return PP_OK;
  if (!logits || !tokens || !dlogits) return fail(PP_ERR_INVALID_ARGUMENT, "logits, tokens and dlogits must be non-NULL");
  if (bt.Kmax > 0 && !dseq) return fail(PP_ERR_INVALID_ARGUMENT, "dseq is NULL");
  if (ws_bytes < p.lay.total)
    return fail(PP_ERR_WORKSPACE_TOO_SMALL, "logprob needs %zu workspace bytes, got %zu", p.lay.total,
                ws_bytes);
  if (!ws) return fail(PP_ERR_INVALID_ARGUMENT, "ws is NULL");
  if (ws && !aligned256(ws)) return fail(PP_ERR_INVALID_ARGUMENT, "ws must be 256-byte aligned");
  hipStream_t s = (hipStream_t)hip_stream;
  MetaImage img;
  logprob_image(bt, p, true, !gathered, &img);
  if ((st = stage_copy(ws, img.buf.data(), img.buf.size(), s)) != PP_OK) return st;
  LogprobBwdLaunch a{};
  a.logits = logits;
  a.tokens = tokens;
  a.dseq = dseq;
  a.dlogits = dlogits;
  a.rows = (const LogitRowItem*)at(ws, p.lay, p.r_rows);
  a.labels = (const int32_t*)at(ws, p.lay, p.r_labels);
  a.label_out = (const int32_t*)at(ws, p.lay, p.r_label_out);
  a.row_item = (const int32_t*)at(ws, p.lay, p.r_row_item);
  a.vocab = vocab;
  a.sumT = bt.sumT;
  a.dtype = logits_dtype == PP_FP32 ? kFP32 : kBF16;
  a.gathered = gathered;
  a.n_rows = (int)p.n.rows;
  a.row_index = row_index;
  hipError_t e = launch_logprob_bwd(a, s);
  if (e != hipSuccess) return hip_fail(e, "logprob backward launch");
  return PP_OK;
}

}  // namespace
}  // namespace pp

extern "C" {

pp_status pp_seq_logprob_bwd(const pp_pack_desc* desc, pp_dtype logits_dtype, int vocab,
                             const void* logits, const int32_t* tokens, const float* dseq,
                             void* dlogits, void* ws, size_t ws_bytes, void* hip_stream) {
  return logprob_bwd_impl(desc, logits_dtype, vocab, logits, tokens, dseq, dlogits, false, nullptr, ws, ws_bytes,
                          hip_stream);
}

pp_status pp_logprob_row_count(const pp_pack_desc* desc, int64_t* n_rows) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if (!n_rows) return fail(PP_ERR_INVALID_ARGUMENT, "n_rows is NULL");
  if ((st = check_logprob_layout(bt)) != PP_OK) return st;
  *n_rows = count_lplan(bt).rows;
  return PP_OK;
}

pp_status pp_seq_logprob_bwd_rows(const pp_pack_desc* desc, pp_dtype logits_dtype, int vocab,
                                  const void* logits, const int32_t* tokens, const float* dseq,
                                  void* dlogits_rows, int32_t* row_index, void* ws, size_t ws_bytes,
                                  void* hip_stream) {
  return logprob_bwd_impl(desc, logits_dtype, vocab, logits, tokens, dseq, dlogits_rows, true, row_index, ws,
                          ws_bytes, hip_stream);
}

pp_status pp_rm_workspace_size(const pp_pack_desc* desc, size_t* bytes) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if (!bytes) return fail(PP_ERR_INVALID_ARGUMENT, "bytes is NULL");
  RmPlan p;
  plan_rm(bt, &p);
  *bytes = p.lay.total;
  return PP_OK;
}

pp_status pp_rm_scores(const pp_pack_desc* desc, pp_dtype dtype, int hidden_dim, const void* hidden,
                       const void* w, float bias, float* scores, void* ws, size_t ws_bytes,
                       void* hip_stream) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if ((st = check_dtype(dtype)) != PP_OK) return st;
  if (hidden_dim < 1) return fail(PP_ERR_INVALID_ARGUMENT, "hidden_dim must be >= 1");
  if (bt.Kmax == 0) return PP_OK;
  if (!scores || !w || (bt.sumT > 0 && !hidden))
    return fail(PP_ERR_INVALID_ARGUMENT, "hidden, w and scores must be non-NULL");
  RmPlan p;
  plan_rm(bt, &p);
  if (ws_bytes < p.lay.total)
    return fail(PP_ERR_WORKSPACE_TOO_SMALL, "rm head needs %zu workspace bytes, got %zu", p.lay.total, ws_bytes);
  if (!ws) return fail(PP_ERR_INVALID_ARGUMENT, "ws is NULL");
  if (ws && !aligned256(ws)) return fail(PP_ERR_INVALID_ARGUMENT, "ws must be 256-byte aligned");
  hipStream_t s = (hipStream_t)hip_stream;
  if ((st = stage_copy(ws, p.slot_row.data(), p.slot_row.size() * 8, s)) != PP_OK) return st;
  RmLaunch a{};
  a.hidden = hidden;
  a.w = w;
  a.bias = bias;
  a.scores = scores;
  a.slot_row = (const int64_t*)at(ws, p.lay, p.r_slot_row);
  a.n_slots = (int)p.slot_row.size();
  a.H = hidden_dim;
  a.dtype = dtype == PP_FP32 ? kFP32 : kBF16;
  hipError_t e = launch_rm_scores(a, s);
  if (e != hipSuccess) return hip_fail(e, "rm scores launch");
  return PP_OK;
}

pp_status pp_rm_scores_bwd(const pp_pack_desc* desc, pp_dtype dtype, int hidden_dim, const void* hidden,
                           const void* w, const float* dscores, void* dhidden, float* dw, float* dbias,
                           void* ws, size_t ws_bytes, void* hip_stream) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if ((st = check_dtype(dtype)) != PP_OK) return st;
  if (hidden_dim < 1) return fail(PP_ERR_INVALID_ARGUMENT, "hidden_dim must be >= 1");
  if (!w || !dw || (bt.sumT > 0 && (!hidden || !dhidden)) || (bt.Kmax > 0 && !dscores))
    return fail(PP_ERR_INVALID_ARGUMENT, "hidden, w, dscores, dhidden and dw must be non-NULL");
  RmPlan p;
  plan_rm(bt, &p);
  if (ws_bytes < p.lay.total)
    return fail(PP_ERR_WORKSPACE_TOO_SMALL, "rm head needs %zu workspace bytes, got %zu", p.lay.total, ws_bytes);
  if (p.lay.total && !ws) return fail(PP_ERR_INVALID_ARGUMENT, "ws is NULL");
  if (ws && !aligned256(ws)) return fail(PP_ERR_INVALID_ARGUMENT, "ws must be 256-byte aligned");
  hipStream_t s = (hipStream_t)hip_stream;
  MetaImage img;
  img.put(p.lay.regions[p.r_slot_row], p.slot_row.data(), p.slot_row.size() * 8);
  img.put(p.lay.regions[p.r_rows], p.rows.data(), p.rows.size() * sizeof(RmRowSlots));
  img.put(p.lay.regions[p.r_slots], p.slots.data(), p.slots.size() * 4);
  int32_t* row_rec = (int32_t*)img.at(p.lay.regions[p.r_row_rec]);
  std::fill(row_rec, row_rec + bt.sumT, -1);
  for (size_t i = 0; i < p.rows.size(); ++i) row_rec[p.rows[i].row] = (int32_t)i;
  if ((st = stage_copy(ws, img.buf.data(), img.buf.size(), s)) != PP_OK) return st;
  RmBwdLaunch a{};
  a.hidden = hidden;
  a.w = w;
  a.dscores = dscores;
  a.dhidden = dhidden;
  a.dw = dw;
  a.dbias = dbias;
  a.slot_row = (const int64_t*)at(ws, p.lay, p.r_slot_row);
  a.rows = (const RmRowSlots*)at(ws, p.lay, p.r_rows);
  a.slots = (const int32_t*)at(ws, p.lay, p.r_slots);
  a.row_rec = (const int32_t*)at(ws, p.lay, p.r_row_rec);
  a.n_slots = (int)p.slot_row.size();
  a.sumT = bt.sumT;
  a.H = hidden_dim;
  a.dtype = dtype == PP_FP32 ? kFP32 : kBF16;
  hipError_t e = launch_rm_bwd(a, s);
  if (e != hipSuccess) return hip_fail(e, "rm backward launch");
  return PP_OK;
}

pp_status pp_dpo_loss(int32_t num_rows, int32_t max_resp, const int32_t* num_resp,
                      const float* logp_pol, const float* logp_ref, float beta, float* loss,
                      float* row_loss, float* dlogp_pol, void* ws, size_t ws_bytes,
                      void* hip_stream) {
  if (num_rows < 1) return fail(PP_ERR_INVALID_ARGUMENT, "num_rows must be >= 1");
  if (max_resp < 0) return fail(PP_ERR_INVALID_ARGUMENT, "max_resp must be >= 0");
  if (!num_resp || !logp_pol || !loss)
    return fail(PP_ERR_INVALID_ARGUMENT, "num_resp, logp_pol and loss must be non-NULL");
  if (!std::isfinite(beta)) return fail(PP_ERR_INVALID_ARGUMENT, "beta must be finite");
  int qualified = 0;
  for (int b = 0; b < num_rows; ++b) {
    if (num_resp[b] < 0 || num_resp[b] > max_resp)
      return fail(PP_ERR_INVALID_ARGUMENT, "num_resp[%d] = %d outside [0, %d]", b, num_resp[b], max_resp);
    if (num_resp[b] >= 2) ++qualified;
  }
  if (qualified == 0) return fail(PP_ERR_INVALID_ARGUMENT, "no row has two responses to compare");
  const size_t need = align_up((size_t)num_rows * 4);
  if (ws_bytes < need)
    return fail(PP_ERR_WORKSPACE_TOO_SMALL, "loss needs %zu workspace bytes, got %zu", need, ws_bytes);
  if (!ws) return fail(PP_ERR_INVALID_ARGUMENT, "ws is NULL");
  if (ws && !aligned256(ws)) return fail(PP_ERR_INVALID_ARGUMENT, "ws must be 256-byte aligned");
  hipStream_t s = (hipStream_t)hip_stream;
  LossLaunch a{};
  if (num_rows <= kLossInlineRows) {
    // few rows: the counts ride in the launch arguments, no copy
    memcpy(a.nr_inline, num_resp, (size_t)num_rows * 4);
    a.num_resp = nullptr;
  } else {
    pp_status st = stage_copy(ws, num_resp, (size_t)num_rows * 4, s);
    if (st != PP_OK) return st;
    a.num_resp = (const int32_t*)ws;
  }
  a.pol = logp_pol;
  a.ref = logp_ref;
  a.beta = beta;
  a.loss = loss;
  a.row_loss = row_loss;
  a.dlogp = dlogp_pol;
  a.B = num_rows;
  a.K_max = max_resp;
  a.n_qualified = qualified;
  hipError_t e = launch_loss(a, s);
  if (e != hipSuccess) return hip_fail(e, "loss launch");
  return PP_OK;
}

pp_status pp_pack_stats(const pp_pack_desc* desc, pp_pack_stats_t* out) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if (!out) return fail(PP_ERR_INVALID_ARGUMENT, "out is NULL");
  pp_pack_stats_t r{};
  auto tri = [](int64_t n) { return n * (n + 1) / 2; };
  double c_pp = 0, c_orig = 0, m_pp = 0, m_orig = 0;
  int64_t n_seq = 0, longest = 0;
  for (const Row& row : bt.rows) {
    const int64_t P = row.P;
    int64_t sum_l = 0, max_l = 0;
    for (int k = 0; k < row.K; ++k) {
      sum_l += row.len[k];
      max_l = std::max<int64_t>(max_l, row.len[k]);
    }
    r.tokens_packed += P + sum_l;
    r.pairs_packed += visible_pairs(row, 0, row.valid, 0, row.valid);
    r.pairs_dense_packed += tri(P + sum_l);
    if (row.K == 0) {
      r.tokens_unpacked += P;
      r.pairs_unpacked += tri(P);
      ++n_seq;
      longest = std::max(longest, P);
      continue;
    }
    ++r.rows_with_responses;
    for (int k = 0; k < row.K; ++k) {
      r.tokens_unpacked += P + row.len[k];
      r.pairs_unpacked += tri(P + row.len[k]);
      ++n_seq;
      longest = std::max<int64_t>(longest, P + row.len[k]);
    }
    const double a = (double)(P + sum_l), b = (double)(P + max_l);
    c_pp += a * a;
    c_orig += row.K * b * b;
    m_pp += a;
    m_orig += row.K * b;
    if (a < std::sqrt((double)row.K) * b) ++r.rows_eq1_cheaper;
  }
  r.tokens_padded = n_seq * longest;
  r.pairs_padded = n_seq * tri(longest);
  r.eq1_cost_ratio = c_orig > 0 ? c_pp / c_orig : 0.0;
  r.eq1_memory_ratio = m_orig > 0 ? m_pp / m_orig : 0.0;
  *out = r;
  return PP_OK;
}

pp_status pp_tile_class_len(const pp_pack_desc* desc, int block_q, int block_k, size_t* len) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if (block_q < 1 || block_k < 1) return fail(PP_ERR_INVALID_ARGUMENT, "block sizes must be >= 1");
  if (!len) return fail(PP_ERR_INVALID_ARGUMENT, "len is NULL");
  size_t n = 0;
  for (const Row& r : bt.rows)
    n += (size_t)((r.T + block_q - 1) / block_q) * ((r.T + block_k - 1) / block_k);
  *len = n;
  return PP_OK;
}

pp_status pp_pack_export(const pp_pack_desc* desc, int block_q, int block_k, int32_t* position_ids,
                         int32_t* segment_ids, uint8_t* tile_class, size_t tile_class_len) {
  Batch bt;
  pp_status st = read_desc(desc, &bt);
  if (st != PP_OK) return st;
  if (tile_class) {
    size_t need = 0;
    if ((st = pp_tile_class_len(desc, block_q, block_k, &need)) != PP_OK) return st;
    if (tile_class_len < need)
      return fail(PP_ERR_INVALID_ARGUMENT, "tile_class needs %zu entries, got %zu", need, tile_class_len);
  }
  size_t tc = 0;
  for (const Row& r : bt.rows) {
    for (int32_t t = 0; t < r.T; ++t) {
      const int32_t sid = seg_id(r, t);
      if (segment_ids) segment_ids[r.tok0 + t] = sid;
      if (position_ids) position_ids[r.tok0 + t] = token_position(r, t);
    }
    if (tile_class) {
      for (int32_t q0 = 0; q0 < r.T; q0 += block_q)
        for (int32_t k0 = 0; k0 < r.T; k0 += block_k)
          tile_class[tc++] = classify_tile(r, q0, std::min(r.T, q0 + block_q), k0, std::min(r.T, k0 + block_k));
    }
  }
  return PP_OK;
}

pp_status pp_timing_enable(int on) {
  g_time_on.store(on != 0);
  return PP_OK;
}

pp_status pp_timing_select(const char* names) {
  std::vector<std::string> sel;
  if (names) {
    const char* c = names;
    while (*c) {
      const char* e = strchr(c, ',');
      const size_t n = e ? (size_t)(e - c) : strlen(c);
      if (n > 0) sel.emplace_back(c, n);
      if (!e) break;
      c = e + 1;
    }
  }
  std::lock_guard<std::mutex> lk(g_time_mu);
  g_time_select.swap(sel);
  return PP_OK;
}

pp_status pp_timing_reset(void) {
  std::lock_guard<std::mutex> lk(g_time_mu);
  drain_timing_locked();
  g_time_totals.clear();
  return PP_OK;
}

int pp_timing_count(void) {
  std::lock_guard<std::mutex> lk(g_time_mu);
  drain_timing_locked();
  return (int)g_time_totals.size();
}

pp_status pp_timing_get(int idx, const char** name, double* total_ms, int64_t* launches) {
  std::lock_guard<std::mutex> lk(g_time_mu);
  drain_timing_locked();
  if (idx < 0 || idx >= (int)g_time_totals.size())
    return fail(PP_ERR_INVALID_ARGUMENT, "timing index %d out of range", idx);
  if (name) *name = g_time_totals[idx].name;
  if (total_ms) *total_ms = g_time_totals[idx].ms;
  if (launches) *launches = g_time_totals[idx].launches;
  return PP_OK;
}

}  // extern "C"
