// Test-only view of the planner: the library's host source with one entry point that
// copies out what a plan holds.  Built by the tests as a library of its own; nothing of it
// is in the product.
#include "../paper_2602_24082_amd/csrc/pp_host.cpp"

namespace {
template <typename T>
int64_t give(const std::vector<T>& v, void* out, int64_t cap) {
  const int64_t n = (int64_t)(v.size() * sizeof(T));
  if (n && n <= cap) memcpy(out, v.data(), n);
  return n;
}
}  // namespace

// Blocks of the staging launch for a copy of `bytes`, four conversions and zeros.
extern "C" int64_t rec_stage_blocks(int64_t bytes, const int64_t* casts, int64_t zeros, int32_t* cast_blocks) {
  StageLaunch a;
  a.bytes = (size_t)bytes;
  for (int c = 0; c < kStageCasts; ++c) a.cast[c].n = casts[c];
  a.n_zero = zeros;
  const StageBlocks nb = stage_blocks(a);
  for (int c = 0; c < kStageCasts; ++c) cast_blocks[c] = nb.cast[c];
  return nb.total;
}

// Record list `what` of a plan, copied into `out` if it fits `cap` bytes; its size in
// bytes, or -1 for a descriptor that is refused.
enum Records {
  kFwdItems, kFwdKtiles, kDqItems, kDqKtiles, kKvItems, kCutItems, kCutParts, kCutSplits, kRowKb0, kPanels, kSegLo, kSegHi,
  kLpRows, kLpLabels, kLpResp, kLpLabelOut, kLpRowItem, kRmSlotRow, kRmRows, kRmSlots
};

extern "C" int64_t rec_list(const pp_pack_desc* desc, int what, int hq, int hkv, int d, void* out, int64_t cap) {
  Batch bt;
  if (read_desc(desc, &bt) != PP_OK) return -1;
  if (what <= kFwdKtiles) {
    FwdPlan p;
    plan_fwd(bt, PP_BF16, hq, hkv, d, &p);
    return what == kFwdItems ? give(p.q.items, out, cap) : give(p.q.ktiles, out, cap);
  }
  if (what <= kPanels) {
    BwdPlan p;
    plan_bwd(bt, PP_BF16, hq, hkv, d, &p);
    switch (what) {
      case kDqItems: return give(p.dq.items, out, cap);
      case kDqKtiles: return give(p.dq.ktiles, out, cap);
      case kKvItems: return give(p.kv, out, cap);
      case kCutItems: return give(p.cut.items, out, cap);
      case kCutParts: return give(p.cut.parts, out, cap);
      case kCutSplits: return give(p.cut.splits, out, cap);
      case kRowKb0: return give(p.row_kb0, out, cap);
      default: return give(p.panels, out, cap);
    }
  }
  if (what <= kSegHi) {
    std::vector<int32_t> v(bt.sumT);
    if (what == kSegLo) fill_seg_lo(bt, v.data());
    else fill_seg_hi(bt, v.data());
    return give(v, out, cap);
  }
  if (what <= kLpRowItem) {
    if (check_logprob_layout(bt) != PP_OK) return -1;
    const LCounts n = count_lplan(bt);
    std::vector<LogitRowItem> rows(n.rows);
    std::vector<int32_t> labels(n.labels), label_out(n.labels), row_item(bt.sumT);
    std::vector<RespItem> resp(n.resp);
    fill_lplan(bt, rows.data(), labels.data(), resp.data(), label_out.data(), row_item.data());
    switch (what) {
      case kLpRows: return give(rows, out, cap);
      case kLpLabels: return give(labels, out, cap);
      case kLpResp: return give(resp, out, cap);
      case kLpLabelOut: return give(label_out, out, cap);
      default: return give(row_item, out, cap);
    }
  }
  RmPlan p;
  plan_rm(bt, &p);
  if (what == kRmSlotRow) return give(p.slot_row, out, cap);
  return what == kRmRows ? give(p.rows, out, cap) : give(p.slots, out, cap);
}
