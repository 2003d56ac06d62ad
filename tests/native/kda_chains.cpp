// Walks the chain list of KDA plans as the kernel's workgroups do (same addresses in the metadata, same steps): every
// (request, head) chain is run once, longest first, and the busiest workgroup is within 4/3 of the best possible
// (Graham's bound for longest-first to the least loaded; 2 % more where the fixed order is kept), of which the even share is a lower bound, and so is k
// times the length of chain 256 (k - 1): of the chains up to it some workgroup has k.
#include "kda_host.cpp"

#include <cstdio>
#include <cstdlib>
#include <random>

namespace {

void check(bool ok, const char* what, int seed) {
  if (ok) return;
  fprintf(stderr, "kda_chains: %s (wave %d)\n", what, seed);
  exit(1);
}

// Returns the busiest workgroup's 64-token blocks.
int64_t walk(const std::vector<int32_t>& lens, int heads, int seed) {
  const int32_t R = int32_t(lens.size());
  std::vector<int32_t> in(lens.size(), -1), out(lens.size());
  std::iota(out.begin(), out.end(), 0);
  const wavepp_kda_shape shape{heads, kKdaDim, kKdaDim, R};
  const wavepp_kda_batch batch{R, lens.data(), in.data(), out.data()};
  wavepp_kda_plan_t* plan = nullptr;
  check(wavepp_kda_plan(&shape, &batch, &plan) == WAVEPP_OK, "plan", seed);
  const unsigned char* base = plan->blob.data();
  check(plan->blob.size() % 16 == 0 && plan->workspace_bytes >= plan->blob.size(), "metadata size", seed);
  const auto* items = reinterpret_cast<const KdaItem*>(base + plan->off_items);
  const int64_t chains = int64_t(plan->items.size()) * heads;
  const int G = int(std::min<int64_t>(chains, kNumCu));
  const int32_t* list = plan->listed ? reinterpret_cast<const int32_t*>(items + plan->items.size()) : nullptr;
  check(!list || (G == kNumCu && reinterpret_cast<const unsigned char*>(list + kNumCu + 1 + chains) <= base + plan->blob.size()),
        "list within the metadata", seed);
  std::vector<char> seen(size_t(chains), 0);
  int64_t busiest = 0, blocks = 0, total = 0, ran = 0;
  for (int w = 0; w < G; ++w) {
    int64_t load = 0, b = 0;
    int32_t last = INT32_MAX;
    for (int round = list ? list[w] : 0;; ++round) {
      if (list && round >= list[w + 1]) break;
      const int c = list ? list[round] : round * G + ((round & 1) ? G - 1 - w : w);
      if (!list && c >= chains) break;
      check(c >= 0 && c < chains && !seen[size_t(c)], "a chain twice or out of range", seed);
      seen[size_t(c)] = 1;
      ++ran;
      const KdaItem& it = items[c / heads];
      check(it.len > 0 && it.len <= last, "longest first", seed);
      last = it.len;
      const int64_t n = (it.len + kKdaBlock - 1) / kKdaBlock;
      load += 2 * n + 1;
      b += n;
    }
    busiest = std::max(busiest, load);
    blocks = std::max(blocks, b);
    total += load;
  }
  check(ran == chains, "every chain", seed);
  int64_t least = (total + kNumCu - 1) / kNumCu;
  for (int64_t k = 1; kNumCu * (k - 1) < chains; ++k) {
    const KdaItem& it = items[kNumCu * (k - 1) / heads];
    least = std::max(least, k * (2 * ((it.len + kKdaBlock - 1) / kKdaBlock) + 1));
  }
  check(chains > kKdaMaxListed || 150 * busiest <= 204 * least, "busiest workgroup", seed);
  wavepp_kda_destroy(plan);
  return blocks;
}

std::vector<int32_t> wave(int longs, int long_len, int shorts, int short_len) {
  std::vector<int32_t> v(size_t(longs), long_len);
  v.insert(v.end(), size_t(shorts), short_len);
  return v;
}

}  // namespace

int main() {
  // one long prompt beside many short ones
  check(walk(wave(1, 16384, 63, 1024), 64, -1) <= 330, "1 x 16,384 + 63 x 1,024, 64 heads", -1);
  check(walk(wave(1, 4096, 63, 512), 32, -2) <= 75, "1 x 4,096 + 63 x 512, 32 heads", -2);
  check(walk(wave(1, 8192, 255, 512), 16, -3) <= 140, "1 x 8,192 + 255 x 512, 16 heads", -3);
  // equal chunks: an even share each, and no list
  check(walk(wave(0, 0, 64, 256), 64, -4) == 64 && walk(wave(0, 0, 4, 4096), 64, -5) == 64, "equal chunks", -4);
  walk(wave(1, 640, 10923, 1), 96, -6);   // more chains than are listed
  std::mt19937 rng(7);
  for (int s = 0; s < 400; ++s) {
    const int heads = int(1 + rng() % 100);
    std::vector<int32_t> lens(1 + rng() % 80);
    const int spread = int(1 + rng() % 13);
    for (auto& n : lens) n = int32_t(rng() % (1u << (rng() % unsigned(spread + 1)))) + int32_t(rng() % 3);
    if (std::count(lens.begin(), lens.end(), 0) == int64_t(lens.size())) lens[0] = 1;
    walk(lens, heads, s);
  }
  printf("kda_chains ok\n");
  return 0;
}
