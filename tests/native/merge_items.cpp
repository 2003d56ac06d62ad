// The form of the merge that each item of a plan takes, through the planner: one row per workgroup for items of more
// than 16 splits in few rows, one thread per (row, 4 lanes) for all others, unless those are few.
#include "host.cpp"

#include <cstdio>
#include <cstdlib>

namespace {

struct Wave {
  int q_heads, kv_heads, dim;
  std::vector<int32_t> prefix, chunk;
  int max_splits;
};

// -1: the items of many splits and only they; otherwise whether all items or none take one row per workgroup.
void expect(const char* what, const Wave& w, int wide) {
  const bool latent = w.dim == 576;
  const int B = 64, R = int(w.prefix.size());
  int stride = 1, pages = 0;
  for (int r = 0; r < R; ++r) stride = std::max(stride, (w.prefix[r] + w.chunk[r] + B - 1) / B);
  std::vector<int32_t> table(size_t(R) * stride, -1);
  for (int r = 0; r < R; ++r)
    for (int b = 0; b * B < w.prefix[r] + w.chunk[r]; ++b) table[size_t(r) * stride + b] = pages++;
  const wavepp_attn_shape shape{w.q_heads, w.kv_heads, w.dim, latent ? 512 : w.dim, B, pages, latent, 0.1f};
  const wavepp_batch batch{R, w.prefix.data(), w.chunk.data(), table.data(), stride};
  wavepp_plan* plan = nullptr;
  if (wavepp_attn_plan(&shape, &batch, w.max_splits, &plan) != WAVEPP_OK) {
    fprintf(stderr, "merge_items: %s: %s\n", what, wavepp_last_error());
    exit(1);
  }
  const int items = int(plan->merges.size()), n = plan->num_merge_wide;
  int many = 0, most = 0;
  bool sorted = true;
  for (int i = 0; i < items; ++i) {
    many += plan->merges[i].nsplit > kMergeNarrow;
    most = std::max(most, plan->merges[i].rows);
    if (wide < 0) sorted = sorted && (plan->merges[i].nsplit > kMergeNarrow) == (i < n);
  }
  // the metadata holds the items in the order that the launches take them
  const auto* h = reinterpret_cast<const MetaHeader*>(plan->blob.data());
  const bool stored = h->num_merge == items && (items == 0 || memcmp(plan->blob.data() + plan->off_merges, plan->merges.data(),
                                                                     sizeof(MergeItem) * plan->merges.size()) == 0);
  if (!stored || !sorted || most != plan->merge_rows || n != (wide < 0 ? many : wide ? items : 0)) {
    fprintf(stderr, "merge_items: %s: %d of %d items wide, %d of many splits\n", what, n, items, many);
    exit(1);
  }
  wavepp_plan_destroy(plan);
}

std::vector<int32_t> lens(int first, int n, int rest) {
  std::vector<int32_t> v(size_t(n) + 1, rest);
  v[0] = first;
  return v;
}

}  // namespace

int main() {
  // one request behind a long prefix beside others: few of their rows come along, many have a launch of their own
  // or, behind 17 to 31 splits, decide the form for all
  expect("few other rows", {64, 8, 128, lens(65536, 3, 2500), lens(4, 3, 4), 0}, 1);
  expect("many other rows", {64, 8, 128, lens(65536, 16, 1000), lens(4, 16, 16), 64}, -1);
  expect("many other rows, 20 splits", {64, 8, 128, lens(65536, 16, 1000), lens(4, 16, 16), 20}, 0);
  expect("latent, many other rows", {128, 1, 576, lens(60000, 5, 700), lens(4, 5, 8), 100}, -1);
  // one row an item: what counts is the rows there are, not those that an item may hold
  expect("many items of one row", {16, 16, 128, lens(3000, 40, 1200), lens(1, 40, 1), 24}, 1);
  // many splits of many rows: forced on a large wave
  expect("17 splits of many rows", {32, 8, 128, lens(8000, 3, 8000), lens(1024, 3, 1024), 17}, 0);
  expect("66 splits of many rows", {32, 8, 128, lens(16384, 3, 16384), lens(1024, 3, 1024), 70}, 1);
  expect("66 splits of 64 lanes, many rows", {24, 4, 64, lens(16384, 3, 16384), lens(1024, 3, 1024), 70}, 0);
  // no item of more than 16 splits; no merge at all
  expect("16 splits", {64, 8, 128, lens(16000, 3, 16000), lens(4, 3, 4), 16}, 0);
  expect("no splits", {64, 8, 128, lens(16000, 3, 16000), lens(4, 3, 4), 1}, 0);
  printf("merge_items ok\n");
  return 0;
}
