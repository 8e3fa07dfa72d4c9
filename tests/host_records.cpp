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
