// Host side of libwavepp_attn: validation, work-list planning, metadata staging and launches.
//
// The plan turns a wave -- per-request spans (request, cached length p_r, chunk length c_r) and
// block tables over a page pool -- into a list of attention work items.  Spans and paging follow
// the paper's problem statement (Preliminaries, "Reuse": ceil(n / B) blocks in non-contiguous
// pages; Pipeline Scheduling: spans of request id, starting token and length, where a position
// that does not match the materialized cache must fail rather than run).
#include "wavepp_attn.h"
#include "internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <mutex>
#include <numeric>
#include <string>
#include <unordered_map>
#include <vector>

using namespace wavepp;

struct wavepp_plan {
  wavepp_attn_shape shape;
  int32_t num_requests = 0;
  int32_t bt_stride = 0;
  int64_t total_tokens = 0;
  uint32_t serial = 0;
  int32_t rows_per_item = 0;
  int32_t kv_tile = 0;
  int32_t max_splits_used = 1;
  int32_t num_real_items = 0;
  std::vector<WorkItem> items;
  std::vector<MergeItem> merges;      // those that merge_wide_kernel takes first
  int32_t num_merge_wide = 0, merge_rows = 0;
  int64_t partial_rows = 0;
  // metadata blob (uploaded as is) and its sub-array offsets
  std::vector<unsigned char> blob;
  size_t off_reqs = 0, off_bt = 0, off_items = 0, off_merges = 0;
  size_t meta_bytes = 0;       // blob size rounded up to 256
  size_t off_opart = 0, off_lpart = 0;
  size_t workspace_bytes = 0;
};

namespace wavepp {
namespace {
thread_local std::string g_last_error;
std::atomic<uint32_t> g_serial{1};
}  // namespace

int set_error(int status, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return status;
}

int set_hip_error(hipError_t e, const char* what) {
  return set_error(WAVEPP_EHIP, "%s: %s", what, hipGetErrorString(e));
}

void clear_error() { g_last_error.clear(); }

const char* last_error_text() { return g_last_error.c_str(); }

uint32_t next_serial() { return g_serial.fetch_add(1); }

// Which plan's metadata each workspace was last given, by the serial of the plan whose upload this
// library enqueued into it.  The entry points that launch kernels consult it before enqueuing
// anything, so a missing or stale upload is an error on the host; the kernels' own serial check
// stays as a second guard (e.g. for a workspace the caller overwrote in between).
namespace {
std::mutex g_ws_mu;
std::unordered_map<uintptr_t, uint32_t> g_ws_serial;
}  // namespace

void note_upload(const void* workspace, uint32_t serial) {
  std::lock_guard<std::mutex> lock(g_ws_mu);
  g_ws_serial[reinterpret_cast<uintptr_t>(workspace)] = serial;
}

int require_upload(const void* workspace, uint32_t serial, const char* upload_fn) {
  uint32_t have = 0;
  bool found = false;
  {
    std::lock_guard<std::mutex> lock(g_ws_mu);
    auto it = g_ws_serial.find(reinterpret_cast<uintptr_t>(workspace));
    if (it != g_ws_serial.end()) {
      found = true;
      have = it->second;
    }
  }
  if (!found)
    return set_error(WAVEPP_EINVAL, "workspace %p holds no uploaded plan: call %s(plan, workspace) first", workspace,
                     upload_fn);
  if (have != serial)
    return set_error(WAVEPP_EINVAL, "workspace %p holds the metadata of another plan (serial %u, this plan %u): call "
                     "%s(plan, workspace) first", workspace, have, serial, upload_fn);
  return WAVEPP_OK;
}

}  // namespace wavepp

namespace {

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

bool supported_shape(const wavepp_attn_shape& s) {
  if (s.page_size != 16 && s.page_size != 64) return false;
  if (s.kv_shared) return s.head_dim_qk == 576 && s.head_dim_v == 512 && s.num_kv_heads == 1;
  return (s.head_dim_qk == 64 && s.head_dim_v == 64) || (s.head_dim_qk == 128 && s.head_dim_v == 128);
}

bool env_flag(const char* name, bool dflt) {
  const char* v = getenv(name);
  if (!v || !*v) return dflt;
  return !(v[0] == '0' || v[0] == 'n' || v[0] == 'N' || v[0] == 'f' || v[0] == 'F');
}

// Estimated cost of an item: rows times the keys they see on average.
double item_cost(const WorkItem& it, int G) {
  double keys = double(it.kv_end - it.kv_begin) - 0.5 * double(it.rows) / double(G);
  return double(it.rows) * std::max(keys, 1.0);
}

// `slots` workgroups that run one item after another, as a min-heap of the times at which they are free.
class SlotClock {
 public:
  explicit SlotClock(int slots) : busy_(size_t(std::max(1, slots)), 0.0) {}
  // the longest-first items of `times`, in order, on empty slots
  SlotClock(int slots, const std::vector<double>& times) : SlotClock(slots) {
    // the first go to a slot each; ascending, they are a heap already
    const size_t n = std::min(times.size(), busy_.size());
    std::reverse_copy(times.begin(), times.begin() + n, busy_.end() - n);
    if (n) longest_ = times[0];
    for (size_t i = n; i < times.size(); ++i) add(times[i]);
  }
  // the next item of `time` goes to the slot that is free first
  void add(double time) {
    const double t = busy_[0] + time;
    longest_ = std::max(longest_, t);
    const size_t n = busy_.size();
    size_t i = 0;
    for (size_t c = 1; c < n; c = 2 * i + 1) {
      if (c + 1 < n && busy_[c + 1] < busy_[c]) ++c;
      if (busy_[c] >= t) break;
      busy_[i] = busy_[c];
      i = c;
    }
    busy_[i] = t;
  }
  double longest() const { return longest_; }

 private:
  std::vector<double> busy_;
  double longest_ = 0.0;
};

// The chip under workgroups of one per CU, the way timings show that it hands them out: in order, in turn over the
// kNumEngines shader engines (8 XCDs of 4), and a workgroup whose engine has no free CU holds up all behind it.
// (260 latent waves' plans follow this to 5 % on average, one queue to 6-7 %, 16 or 64 groups to 5.4-6 %.)
class Dispatch {
 public:
  Dispatch() : free_(kNumCu, 0.0) {}
  void add(double time) {
    constexpr int per = kNumCu / kNumEngines;
    double* f = &free_[size_t(engine_) * per];          // when the engine's CUs are free, in ascending order
    engine_ = engine_ + 1 < kNumEngines ? engine_ + 1 : 0;
    now_ = std::max(now_, f[0]);
    const double t = now_ + time;
    longest_ = std::max(longest_, t);
    int i = 0;
    for (; i + 1 < per && f[i + 1] < t; ++i) f[i] = f[i + 1];
    f[i] = t;
  }
  double longest() const { return longest_; }

 private:
  std::vector<double> free_;
  double now_ = 0.0, longest_ = 0.0;
  int engine_ = 0;
};

// Sorts `order` by `key` (key[i] belongs to order[i]), largest first, equal keys in their order: a radix sort over
// the bytes in which the keys differ.  Some thousand items take a quarter of the time of a comparison sort,
// which mispredicts half its branches.
void sort_descending(std::vector<uint64_t>& key, std::vector<uint32_t>& order) {
  const size_t n = key.size();
  if (n <= 48) {                       // too few to pay for the buckets
    for (size_t i = 1; i < n; ++i) {
      const uint64_t k = key[i];
      const uint32_t o = order[i];
      size_t j = i;
      for (; j > 0 && key[j - 1] < k; --j) {
        key[j] = key[j - 1];
        order[j] = order[j - 1];
      }
      key[j] = k;
      order[j] = o;
    }
    return;
  }
  uint64_t differ = 0;
  for (uint64_t k : key) differ |= k ^ key[0];
  std::vector<uint64_t> key_to(n);
  std::vector<uint32_t> order_to(n);
  for (int shift = 0; shift < 64; shift += 8) {
    if (((differ >> shift) & 255) == 0) continue;
    uint32_t at[257] = {};
    for (uint64_t k : key) ++at[256 - ((k >> shift) & 255)];         // the bucket after the key's own
    for (int b = 0; b < 256; ++b) at[b + 1] += at[b];
    for (size_t i = 0; i < n; ++i) {
      const uint32_t to = at[255 - ((key[i] >> shift) & 255)]++;
      key_to[to] = key[i];
      order_to[to] = order[i];
    }
    key.swap(key_to);
    order.swap(order_to);
  }
}

// Order items heaviest first and spread them over the L2 domains: consecutive workgroup ids go
// round-robin to the kNumXcd domains, so item index k*kNumXcd + x runs on domain x.  Items of one
// (request, KV head), a stream, read the same K/V pages; keeping them on one domain lets its L2 serve the
// re-reads.  With few streams, balance wins and items are placed individually; the same holds where
// whole streams leave some workgroup slots busy much longer than others.
// WAVEPP_STREAM_MAJOR=0 keeps each domain's items in plain heaviest-first order.
// The items of a stream are consecutive in `items`.  `slots` is the number of workgroups the chip runs at a
// time, `overhead` an item's prologue and epilogue in tiles of `kv_tile` keys, `idle` what a tile takes in a
// workgroup whose waves have no rows, of one where all have.
std::vector<WorkItem> order_items(std::vector<WorkItem> items, int G, bool xcd_aware, bool stream_major, int slots,
                                  int kv_tile, double overhead, double idle) {
  const size_t n = items.size();
  typedef std::pair<double, uint32_t> Key;   // (size, index)
  std::vector<double> cost(n);
  std::vector<uint32_t> by_cost(n);          // items, largest cost first, in index order where equal
  {
    std::vector<uint64_t> key(n);
    for (size_t i = 0; i < n; ++i) {
      cost[i] = item_cost(items[i], G);
      memcpy(&key[i], &cost[i], sizeof(double));          // positive doubles sort like their bits
      by_cost[i] = uint32_t(i);
    }
    sort_descending(key, by_cost);
  }
  if (!xcd_aware || n <= 1) {
    std::vector<WorkItem> out;
    out.reserve(n);
    for (uint32_t i : by_cost) out.push_back(items[i]);
    return out;
  }
  std::vector<uint32_t> stream(n), first;      // stream of an item, first item of a stream
  std::vector<Key> by_stream_cost;
  double total = 0.0, biggest = 0.0;
  for (size_t i = 0; i < n; ++i) {
    if (i == 0 || items[i].req != items[i - 1].req || items[i].kv_head != items[i - 1].kv_head) {
      by_stream_cost.push_back(Key(0.0, uint32_t(first.size())));
      first.push_back(uint32_t(i));
    }
    stream[i] = uint32_t(first.size() - 1);
    by_stream_cost.back().first += cost[i];
    total += cost[i];
    biggest = std::max(biggest, by_stream_cost.back().first);
  }
  // Time goes by tiles more than by rows: an item's workgroup runs its key tiles in about the same time however few
  // of its rows are used.
  std::vector<uint64_t> tiles(n);
  double time_sum = 0.0, time_max = 0.0;
  for (size_t i = 0; i < n; ++i) {
    tiles[i] = uint64_t(uint32_t(items[i].kv_end - items[i].kv_begin + kv_tile - 1) / uint32_t(kv_tile));
    time_sum += double(tiles[i]) + overhead;
    time_max = std::max(time_max, double(tiles[i]) + overhead);
  }
  typedef std::vector<std::vector<uint32_t>> Lists;
  // Individual placement: longest first, each to the least loaded domain.  Items of equal time go by cost, that
  // is by their exact key count: a few requests of the same lengths then come in turn and land on a domain
  // each, whose L2 serves their re-reads (8 requests of 131,072 cached tokens on the latent form: 97 % of
  // the reads, against 87 % when each request's equal items are dealt out over all domains).
  auto place = [&](const std::vector<uint32_t>& order, auto time) {
    Lists out(kNumXcd);
    for (auto& l : out) l.reserve(2 * n / kNumXcd);
    Key busy[kNumXcd];                       // least loaded first, in index order where equal
    for (int x = 0; x < kNumXcd; ++x) busy[x] = Key(0.0, uint32_t(x));
    for (uint32_t i : order) {
      out[busy[0].second].push_back(i);
      const Key k(busy[0].first + time(i), busy[0].second);
      int x = 0;
      for (; x + 1 < kNumXcd && busy[x + 1] < k; ++x) busy[x] = busy[x + 1];
      busy[x] = k;
    }
    return out;
  };
  auto place_items = [&] {
    std::vector<uint64_t> key(n);
    std::vector<uint32_t> by_time(by_cost);
    for (size_t i = 0; i < n; ++i) key[i] = tiles[by_cost[i]];
    sort_descending(key, by_time);
    Lists out = place(by_time, [&](uint32_t i) { return double(tiles[i]) + overhead; });
    // In a second round that is not full, the items that share a CU make the difference, and among them their rows:
    // the placement by tiles and one by the time that the rows leave are played through, and the latter is taken
    // where it is more than 9 % shorter.  4 requests of 7-16 K cached and 2-26 new tokens, 64/8 heads, 328 items:
    // 57 us by tiles, 51 by rows too; 22 of 29 K and 1-61, 8/2 heads of 64: 103 and 90.  Nearer than that either can
    // be the slower by 7 %.
    if (idle < 1.0 && n > size_t(slots) && n <= size_t(2) * slots) {
      std::vector<double> time(n);
      for (size_t i = 0; i < n; ++i)
        time[i] = double(tiles[i]) * (idle + (1.0 - idle) * double((items[i].rows + 31) / 32 * 32) / kGqaRowsPerItem) + overhead;
      by_time = by_cost;
      for (size_t i = 0; i < n; ++i) memcpy(&key[i], &time[by_cost[i]], sizeof(double));
      sort_descending(key, by_time);
      Lists by_rows = place(by_time, [&](uint32_t i) { return time[i]; });
      auto play = [&](const Lists& ls) {
        Dispatch chip;
        size_t rounds = 0;
        for (const auto& l : ls) rounds = std::max(rounds, l.size());
        for (size_t k = 0; k < rounds; ++k)
          for (const auto& l : ls) chip.add(k < l.size() ? time[l[k]] : 0.0);
        return chip.longest();
      };
      if (play(by_rows) < 0.91 * play(out)) out = std::move(by_rows);
    }
    return out;
  };
  Lists lists;
  if (first.size() >= size_t(2 * kNumXcd) && biggest <= 0.5 * total / kNumXcd) {
    lists.resize(kNumXcd);
    std::sort(by_stream_cost.begin(), by_stream_cost.end(),
              [](const Key& a, const Key& b) { return a.first > b.first || (a.first == b.first && a.second < b.second); });
    std::vector<int> where(first.size(), 0);
    double load[kNumXcd] = {};
    for (const Key& k : by_stream_cost) {
      const int x = int(std::min_element(load, load + kNumXcd) - load);
      where[k.second] = x;
      load[x] += k.first;
    }
    if (stream_major) {
      // inside a domain, stream by stream (heaviest stream first), each stream's items heaviest
      // first: the items running together on the domain's CUs then mostly belong to one stream and
      // read its tiles at about the same time, so the domain's L2 serves the re-reads
      std::vector<uint32_t> at(first), sorted(n);
      for (uint32_t i : by_cost) sorted[at[stream[i]]++] = i;
      for (const Key& k : by_stream_cost) {
        const size_t end = k.second + 1 < first.size() ? first[k.second + 1] : n;
        lists[where[k.second]].insert(lists[where[k.second]].end(), sorted.begin() + first[k.second], sorted.begin() + end);
      }
    } else {
      for (uint32_t i : by_cost) lists[where[stream[i]]].push_back(i);
    }
    // With few items per slot, the last stream of a domain can run on a few of its slots alone.  Both orders
    // are played through (each domain hands its list to its slots in order); the streams stay together
    // unless that costs more than 5 %, about what the L2's re-reads are worth (2-4 % on long-prefix waves).
    // 12 requests of 0.1-6 K cached and 37-1,500 new tokens, 24/4 heads: 125 tiles against 102, 331 us
    // against 281.
    if (n <= size_t(16) * slots) {
      // the longest domain's time, or the first that is not below `limit`
      auto makespan = [&](const Lists& ls, double limit) {
        double longest = 0.0;
        for (const auto& l : ls) {
          SlotClock clock(slots / kNumXcd);
          for (size_t i = 0; i < l.size() && longest < limit; ++i) {
            clock.add(double(tiles[l[i]]) + overhead);
            longest = std::max(longest, clock.longest());
          }
        }
        return longest;
      };
      const double together = makespan(lists, INFINITY);
      if (std::max(time_max, time_sum / slots) < 0.95 * together) {   // no order is shorter than that
        Lists single = place_items();
        if (makespan(single, 0.95 * together) < 0.95 * together) lists = std::move(single);
      }
    }
  } else {
    lists = place_items();
  }
  size_t longest = 0;
  for (auto& l : lists) longest = std::max(longest, l.size());
  std::vector<WorkItem> out;
  out.reserve(longest * kNumXcd);
  WorkItem pad{};
  pad.part = -1;
  for (size_t k = 0; k < longest; ++k)
    for (int x = 0; x < kNumXcd; ++x) out.push_back(k < lists[x].size() ? items[lists[x][k]] : pad);
  // trim trailing padding
  while (!out.empty() && out.back().rows == 0) out.pop_back();
  return out;
}

// How a wave's key ranges are cut: base item i is split every tps[i] tiles.
struct SplitPlan {
  std::vector<int64_t> tps;
  int64_t pieces = 0;
};

// Modelled time of a wave of pieces, in tiles, each costing its tiles plus `overhead` (queries in, partial out);
// every piece of a split item adds its partial rows to the merge.  The pieces are handed out longest first
// (Dispatch).  Played as one queue in front of 256 CUs, whole pieces with remainders that fit between them look 5-20 %
// better than they run: 8 requests of 7K-100K cached and 3-47 new tokens, 128 heads: 294 pieces 1,445 us, 509
// even ones 1,211.  Over 401 latent waves the plan chosen by this model takes 0.5 % longer than the fastest, by
// the queue 2.7 %.  A plan that cannot beat `best` is not played through.
double split_cost(const std::vector<int64_t>& ntiles, const SplitPlan& sp, double overhead, double merge, double best) {
  const int slots = kNumCu;
  std::vector<uint64_t> len;                 // equal pieces of an item, and its remainder
  std::vector<uint32_t> number;
  len.reserve(2 * ntiles.size());
  number.reserve(2 * ntiles.size());
  double partials = 0.0, sum = 0.0;
  int64_t count = 0;
  uint32_t most = 0;
  for (size_t i = 0; i < ntiles.size(); ++i) {
    const uint32_t n = uint32_t(ntiles[i]), t = uint32_t(sp.tps[i]), whole = n / t, left = n - whole * t;
    if (whole) len.push_back(t), number.push_back(whole);
    if (left) len.push_back(left), number.push_back(1);
    const uint32_t k = whole + (left != 0);
    if (k > 1) partials += double(k);
    count += k;
    sum += double(n);
    most = std::max(most, whole ? t : left);
  }
  const double bound = std::max(double(most) + overhead, (sum + overhead * double(count)) / slots) + merge * partials;
  if (bound >= best) return bound;
  if (count <= slots) return double(most) + overhead + merge * partials;
  sort_descending(len, number);
  Dispatch chip;
  for (size_t i = 0; i < len.size(); ++i)
    for (uint32_t k = 0; k < number[i] && chip.longest() + merge * partials < best; ++k) chip.add(double(len[i]) + overhead);
  return chip.longest() + merge * partials;
}

// Modelled time of a small grouped wave in the 8-wave form (attention and merge, microseconds), its key
// ranges cut evenly into at most `target` items of at least `min_keys` keys: pieces are handed out longest first
// to 256 workgroups that run one at a time, or the wave streams its K/V at about 5.2 TB/s if that takes longer,
// and the partials are written and merged.  The constants are fitted to 1,200 timed waves of 1-16 requests,
// 1K-40K cached tokens and 90-4,000 rows per KV head, 0 to 16 forced splits; the mean error is 4-6 %.  A tile of
// which only some waves have rows takes `idle` of its time plus the rest by the share of active waves.
struct GroupedModel {
  int rows, tile, slots;
  double idle, overhead, tile_us, base_us, part_us_per_mb, merge_us;
};
constexpr GroupedModel kModel128 = {kGqaRowsPerItem, kKvTile, kNumCu, 0.5, 1.0, 2.99, 1.2, 0.55, 2.1};
constexpr GroupedModel kModel64 = {kGqaRowsPerItem, kKvTile, kNumCu, 0.5, 1.0, 2.08, -3.0, 0.53, 6.7};

double grouped_cost(const wavepp_attn_shape& s, const wavepp_batch& b, int64_t target,
                    int64_t min_keys) {
  const GroupedModel& f = s.head_dim_qk == 64 ? kModel64 : kModel128;
  struct Group { int64_t tiles, count, rows; };       // row tiles of one request that see the same key tiles
  const int64_t G = s.num_q_heads / s.num_kv_heads, min_tiles = min_keys / f.tile;
  std::vector<Group> groups;
  double kv_mb = 0.0;
  int64_t longest = 1;
  for (int32_t r = 0; r < b.num_requests; ++r) {
    const int64_t p = b.prefix_lens[r], c = b.chunk_lens[r], rows = c * G;
    if (c == 0) continue;
    const int64_t n = ceil_div(p + c, f.tile);
    longest = std::max(longest, n);
    if (rows / f.rows) groups.push_back({n, rows / f.rows * s.num_kv_heads, f.rows});
    if (rows % f.rows) groups.push_back({n, s.num_kv_heads, rows % f.rows});
    kv_mb += double(p + c) * s.num_kv_heads * s.head_dim_qk * 4e-6;
  }
  auto splits = [&](int64_t n, int64_t T) { return std::max<int64_t>(1, std::min(ceil_div(n, T), n / min_tiles)); };
  auto total = [&](int64_t T) {
    int64_t n = 0;
    for (const Group& g : groups) n += g.count * splits(g.tiles, T);
    return n;
  };
  int64_t lo = std::max<int64_t>(1, min_tiles), hi = std::max(lo, longest);
  if (total(lo) > target) {
    while (hi - lo > 1) {
      const int64_t mid = lo + (hi - lo) / 2;
      if (total(mid) <= target) hi = mid; else lo = mid;
    }
    lo = hi;
  }
  std::vector<std::pair<double, int64_t>> pieces;     // (time in tiles, count)
  double part_mb = 0.0;
  for (const Group& g : groups) {
    const int64_t tps = ceil_div(g.tiles, splits(g.tiles, lo)), S = ceil_div(g.tiles, tps);
    const double w = f.idle + (1.0 - f.idle) * double(ceil_div(g.rows, 32) * 32) / f.rows;
    if (S > 1) {
      pieces.push_back({double(tps) * w + f.overhead, g.count * (S - 1)});
      part_mb += double(g.count * S * g.rows) * s.head_dim_v * 4e-6;
    }
    pieces.push_back({double(g.tiles - tps * (S - 1)) * w + f.overhead, g.count});
  }
  std::sort(pieces.begin(), pieces.end(), std::greater<std::pair<double, int64_t>>());
  std::vector<double> times;
  for (const auto& x : pieces) times.insert(times.end(), size_t(x.second), x.first);
  return std::max(f.tile_us * SlotClock(f.slots, times).longest() + f.base_us, 0.19 * kv_mb) + f.part_us_per_mb * part_mb +
         (part_mb > 0.0 ? f.merge_us : 0.0);
}

// Puts the merge items that take one row per workgroup (merge_wide_kernel) first and returns their number.  That
// form cuts the chain of memory round trips of an item of many splits and pays a workgroup for every row.
// Measured against merge_kernel on all items (attention with the merge, us):
//  - items of more than 16 splits, alone: 87 splits, 16 to 1,024 rows of 128 lanes: 24-45 -> 12-36; 17 to 44
//    splits, up to 1,024 rows: 1-6 less; 4,096 rows: 33 splits the same, 65 3 less; 16,384 rows: 17 splits 6-12
//    more (64 lanes: 65,536 rows 182 -> 229), from 64 splits 7 less.  So up to 64 rows for every split (a
//    workgroup of 512 lanes takes twice the threads: 32), and any number where each group of threads has 8
//    splits to sum.
//  - the other items of such a wave: sent through the same launch they cost about 1 us for 1,500 rows (16,384
//    rows: 122 -> 132), a second launch 2-3 us, which the items of many splits make up from about 32 on.
// The launch has as many workgroups for every item as the item of most rows (`most`) needs; one without a row
// costs about a quarter of one with.
int32_t merge_wide_items(std::vector<MergeItem>& merges, int most, int head_dim_v) {
  int64_t rows = 0, parts = 0;           // rows and partial rows of the items of many splits
  double cost = 0.0, rest = 0.0;         // their workgroups, and those of the others
  for (const MergeItem& m : merges) {
    const double workgroups = 0.75 * m.rows + 0.25 * most;
    if (m.nsplit <= kMergeNarrow) {
      rest += workgroups;
    } else {
      cost += workgroups;
      rows += m.rows;
      parts += int64_t(m.rows) * m.nsplit;
    }
  }
  if (rows == 0) return 0;
  const int threads = head_dim_v == 512 ? 512 : 256, groups = threads / (head_dim_v / 4);
  const double splits = double(parts) / double(rows), width = threads / 256.0;
  if (cost * width > 64.0 * splits && splits < 8.0 * groups) return 0;
  if (rest * width <= 4096.0) return int32_t(merges.size());
  if (splits < 32.0) return 0;
  const auto end = std::stable_partition(merges.begin(), merges.end(),
                                         [](const MergeItem& m) { return m.nsplit > kMergeNarrow; });
  return int32_t(end - merges.begin());
}

}  // namespace

namespace wavepp {

// ---------------------------------------------------------------------------------------------
// Pinned staging for metadata uploads: a small ring of page-locked buffers per device, each
// guarded by an event so a buffer is refilled only after its previous copy has completed.  The
// buffers are coherent and mapped into the device's address space; a copy kernel on the caller's
// stream moves them into the workspace (see launch_upload).
// ---------------------------------------------------------------------------------------------
struct StagingSlot {
  void* host = nullptr;
  void* dev = nullptr;     // the same buffer's device address
  size_t cap = 0;
  hipEvent_t done = nullptr;
  bool pending = false;
};
struct DeviceStaging {
  std::vector<StagingSlot> slots;
  size_t next = 0;
};
std::mutex g_stage_mu;
std::vector<DeviceStaging> g_stage;   // indexed by device id
constexpr int kStageSlots = 8;

int stage_and_copy(const void* src, size_t bytes, void* dst, hipStream_t stream) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return set_hip_error(e, "hipGetDevice");
  std::lock_guard<std::mutex> lock(g_stage_mu);
  if (g_stage.size() <= size_t(dev)) g_stage.resize(dev + 1);
  DeviceStaging& ds = g_stage[dev];
  if (ds.slots.empty()) ds.slots.resize(kStageSlots);
  StagingSlot& s = ds.slots[ds.next];
  ds.next = (ds.next + 1) % ds.slots.size();
  if (!s.done) {
    e = hipEventCreateWithFlags(&s.done, hipEventDisableTiming);
    if (e != hipSuccess) return set_hip_error(e, "hipEventCreateWithFlags");
  }
  if (s.pending) {
    e = hipEventSynchronize(s.done);
    if (e != hipSuccess) return set_hip_error(e, "hipEventSynchronize");
    s.pending = false;
  }
  if (s.cap < bytes) {
    if (s.host) {
      e = hipHostFree(s.host);
      s.host = nullptr;
      s.dev = nullptr;
      s.cap = 0;
      if (e != hipSuccess) return set_hip_error(e, "hipHostFree");
    }
    size_t cap = align_up(std::max<size_t>(bytes, 64 << 10), 4096);
    void* host = nullptr;
    void* mapped = nullptr;
    e = hipHostMalloc(&host, cap, hipHostMallocCoherent | hipHostMallocMapped);
    if (e != hipSuccess) return set_hip_error(e, "hipHostMalloc");
    e = hipHostGetDevicePointer(&mapped, host, 0);
    if (e != hipSuccess) {
      (void)hipHostFree(host);
      return set_hip_error(e, "hipHostGetDevicePointer");
    }
    s.host = host;
    s.dev = mapped;
    s.cap = cap;
  }
  memcpy(s.host, src, bytes);
  e = launch_upload(s.dev, dst, bytes, stream);
  if (e != hipSuccess) return set_hip_error(e, "metadata upload launch");
  e = hipEventRecord(s.done, stream);
  if (e != hipSuccess) return set_hip_error(e, "hipEventRecord");
  s.pending = true;
  return WAVEPP_OK;
}

}  // namespace wavepp

namespace {

int check_workspace(const wavepp_plan* plan, void* ws, size_t ws_bytes) {
  if (!ws) return set_error(WAVEPP_EINVAL, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(ws) % 256) return set_error(WAVEPP_EINVAL, "workspace must be 256-byte aligned");
  if (ws_bytes < plan->workspace_bytes)
    return set_error(WAVEPP_ENOSPACE, "workspace has %zu bytes, plan needs %zu", ws_bytes, plan->workspace_bytes);
  return WAVEPP_OK;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

DevPlan make_dev(const wavepp_plan* plan, void* ws) {
  auto* base = static_cast<unsigned char*>(ws);
  DevPlan d{};
  d.hdr = reinterpret_cast<const MetaHeader*>(base);
  d.reqs = reinterpret_cast<const ReqMeta*>(base + plan->off_reqs);
  d.bt = reinterpret_cast<const int32_t*>(base + plan->off_bt);
  d.items = reinterpret_cast<const WorkItem*>(base + plan->off_items);
  d.merges = reinterpret_cast<const MergeItem*>(base + plan->off_merges);
  d.opart = reinterpret_cast<float*>(base + plan->off_opart);
  d.lpart = reinterpret_cast<float*>(base + plan->off_lpart);
  d.serial = plan->serial;
  d.num_requests = plan->num_requests;
  d.num_items = int32_t(plan->items.size());
  d.num_merge = int32_t(plan->merges.size());
  d.num_merge_wide = plan->num_merge_wide;
  d.merge_rows = plan->merge_rows;
  d.total_tokens = plan->total_tokens;
  d.num_q_heads = plan->shape.num_q_heads;
  d.num_kv_heads = plan->shape.num_kv_heads;
  d.head_dim_qk = plan->shape.head_dim_qk;
  d.head_dim_v = plan->shape.head_dim_v;
  d.page_size = plan->shape.page_size;
  d.kv_shared = plan->shape.kv_shared;
  d.softmax_scale = plan->shape.softmax_scale;
  d.rows_per_item = plan->rows_per_item;
  return d;
}

}  // namespace

extern "C" {

const char* wavepp_status_string(int status) {
  switch (status) {
    case WAVEPP_OK: return "WAVEPP_OK";
    case WAVEPP_EINVAL: return "WAVEPP_EINVAL: invalid argument";
    case WAVEPP_EUNSUPPORTED: return "WAVEPP_EUNSUPPORTED: unsupported shape";
    case WAVEPP_ERANGE: return "WAVEPP_ERANGE: block-table entry outside the page pool";
    case WAVEPP_EALIAS: return "WAVEPP_EALIAS: appended page also referenced elsewhere";
    case WAVEPP_EPOSITION: return "WAVEPP_EPOSITION: span not backed by the block table";
    case WAVEPP_ENOSPACE: return "WAVEPP_ENOSPACE: workspace too small";
    case WAVEPP_EHIP: return "WAVEPP_EHIP: HIP runtime error";
    default: return "unknown wavepp status";
  }
}

const char* wavepp_last_error(void) { return last_error_text(); }

int wavepp_attn_plan(const wavepp_attn_shape* shape, const wavepp_batch* batch, int32_t max_splits,
                     wavepp_plan** out) {
  clear_error();
  if (!shape || !batch || !out) return set_error(WAVEPP_EINVAL, "null argument");
  *out = nullptr;
  const wavepp_attn_shape s = *shape;
  if (s.num_q_heads <= 0 || s.num_kv_heads <= 0 || s.num_pages <= 0 || s.page_size <= 0 ||
      s.head_dim_qk <= 0 || s.head_dim_v <= 0)
    return set_error(WAVEPP_EINVAL, "non-positive shape field");
  if (!(s.softmax_scale > 0.0f) || !std::isfinite(s.softmax_scale))
    return set_error(WAVEPP_EINVAL, "softmax_scale must be positive and finite");
  if (s.num_q_heads % s.num_kv_heads)
    return set_error(WAVEPP_EINVAL, "num_q_heads (%d) is not a multiple of num_kv_heads (%d)", s.num_q_heads,
                s.num_kv_heads);
  if (s.kv_shared != 0 && s.kv_shared != 1) return set_error(WAVEPP_EINVAL, "kv_shared must be 0 or 1");
  if (!supported_shape(s))
    return set_error(WAVEPP_EUNSUPPORTED, "unsupported (head_dim_qk=%d, head_dim_v=%d, page_size=%d, kv_shared=%d, "
                "num_kv_heads=%d)", s.head_dim_qk, s.head_dim_v, s.page_size, s.kv_shared, s.num_kv_heads);
  if (max_splits < 0) return set_error(WAVEPP_EINVAL, "max_splits must be >= 0");
  const int32_t R = batch->num_requests;
  if (R < 0) return set_error(WAVEPP_EINVAL, "num_requests < 0");
  if (R > 0 && (!batch->prefix_lens || !batch->chunk_lens || !batch->block_table))
    return set_error(WAVEPP_EINVAL, "null span or block-table array");
  if (R > 0 && batch->bt_stride <= 0) return set_error(WAVEPP_EINVAL, "bt_stride must be positive");
  const int32_t B = s.page_size, P = s.num_pages, stride = R > 0 ? batch->bt_stride : 0;
  const int G = s.num_q_heads / s.num_kv_heads;

  // --- spans and block tables ------------------------------------------------------------------
  int64_t total = 0;
  std::vector<int32_t> refcount(P, 0);
  for (int32_t r = 0; r < R; ++r) {
    const int64_t p = batch->prefix_lens[r], c = batch->chunk_lens[r];
    if (p < 0 || c < 0) return set_error(WAVEPP_EINVAL, "request %d: negative length (p=%lld, c=%lld)", r, (long long)p,
                                    (long long)c);
    const int64_t n = p + c;
    if (n > INT32_MAX / 2) return set_error(WAVEPP_EINVAL, "request %d: length %lld too large", r, (long long)n);
    if (n > int64_t(stride) * B)
      return set_error(WAVEPP_EPOSITION, "request %d: positions up to %lld but the block table covers %lld", r,
                  (long long)n, (long long)stride * B);
    const int64_t nb = ceil_div(n, B);
    const int32_t* row = batch->block_table + int64_t(r) * stride;
    for (int64_t b = 0; b < nb; ++b) {
      if (row[b] < 0 || row[b] >= P)
        return set_error(WAVEPP_ERANGE, "request %d block %lld: page %d outside [0, %d)", r, (long long)b, row[b], P);
      refcount[row[b]]++;
    }
    total += c;
    if (total > INT32_MAX / 2) return set_error(WAVEPP_EINVAL, "too many tokens in the wave");
  }
  for (int32_t r = 0; r < R; ++r) {
    const int64_t p = batch->prefix_lens[r], c = batch->chunk_lens[r];
    if (c == 0) continue;
    const int32_t* row = batch->block_table + int64_t(r) * stride;
    for (int64_t b = p / B; b < ceil_div(p + c, B); ++b)
      if (refcount[row[b]] != 1)
        return set_error(WAVEPP_EALIAS, "request %d block %lld: page %d receives appended tokens but is referenced %d "
                    "times in the wave", r, (long long)b, row[b], refcount[row[b]]);
  }

  auto plan = new (std::nothrow) wavepp_plan();
  if (!plan) return set_error(WAVEPP_EINVAL, "out of host memory");
  plan->shape = s;
  plan->num_requests = R;
  plan->bt_stride = stride;
  plan->total_tokens = total;
  plan->serial = next_serial();
  const bool mla = s.kv_shared != 0;
  // grouped kernel: 8 waves (256 rows) per workgroup and one workgroup per CU, so that each K/V tile
  // staged in LDS serves 256 rows.  When no (request, KV head) has more than 128 rows (short
  // chunks: the wave is bound by streaming the prefix K/V), half of those waves would idle: the
  // plan then uses 128-row items, run by the 4-wave form of the kernel, two workgroups per CU.
  // WAVEPP_GQA_WAVES=4 or 8 forces one form.
  int64_t max_rows = 0;
  for (int32_t r = 0; r < R; ++r) max_rows = std::max<int64_t>(max_rows, int64_t(batch->chunk_lens[r]) * (s.num_q_heads / s.num_kv_heads));
  const char* gw = getenv("WAVEPP_GQA_WAVES");
  const int gw_n = gw ? atoi(gw) : 0;
  const bool small_rows = gw_n == 4 || (gw_n != 8 && max_rows <= kGqaRowsPerItem / 2);
  const int gqa_rows = small_rows ? kGqaRowsPerItem / 2 : kGqaRowsPerItem;
  const int M = mla ? kMlaRowsPerItem : gqa_rows;
  // keys per tile of the kernel that will run the plan (the 4-wave grouped form uses half tiles);
  // split boundaries fall on whole tiles of it
  const int KT = mla ? kMlaKvTile : (small_rows ? kKvTile / 2 : kKvTile);
  plan->rows_per_item = M;
  plan->kv_tile = KT;

  // --- work items --------------------------------------------------------------------------------
  std::vector<WorkItem> base;
  std::vector<ReqMeta> reqs(R);
  int64_t cu = 0;
  for (int32_t r = 0; r < R; ++r) {
    const int32_t p = batch->prefix_lens[r], c = batch->chunk_lens[r];
    reqs[r] = ReqMeta{p, c, int32_t(cu), int32_t(int64_t(r) * stride)};
    cu += c;
    const int64_t rows_total = int64_t(c) * G;
    for (int32_t g = 0; g < s.num_kv_heads; ++g)
      for (int64_t r0 = 0; r0 < rows_total; r0 += M) {
        WorkItem w{};
        w.req = r;
        w.kv_head = g;
        w.row0 = int32_t(r0);
        w.rows = int32_t(std::min<int64_t>(M, rows_total - r0));
        const int64_t last_tok = (r0 + w.rows - 1) / G;
        w.kv_begin = 0;
        w.kv_end = int32_t(p + last_tok + 1);
        w.part = -1;
        w.split = 0;
        base.push_back(w);
      }
  }
  // key-range splits: forced by max_splits, or chosen so that a small wave still fills the chip,
  // an item's automatic splits sharing its tiles evenly, 1,024 keys (grouped kernel) or 512
  // (latent kernel) each or more; only an item's last split can be shorter.
  // Split a wave with fewer base items than this until it has about that many.  512 items are two
  // workgroups per CU of the 4-wave form, or two rounds of the one-per-CU forms; on the short-chunk
  // waves (c = 16 .. 128) it gave the fastest or within 0.5 % of the fastest split count, against
  // 1,024 items, which cost 2-11 % in the extra partials and merge work.
  // Automatic splits share the wave's tiles out evenly rather than giving every (request, KV head,
  // row tile) the same number of splits: such a wave runs as one round of workgroups and lasts as
  // long as its longest item, so requests with longer prefixes take more splits.
  const int64_t fill_target = 512;
  const int64_t min_split_tiles = (mla ? 512 : 1024) / KT;
  std::vector<int64_t> ntiles(base.size());
  for (size_t i = 0; i < base.size(); ++i) ntiles[i] = ceil_div(base[i].kv_end, KT);
  SplitPlan split{ntiles, int64_t(base.size())};
  if (max_splits >= 1) {
    for (size_t i = 0; i < base.size(); ++i) split.tps[i] = ceil_div(ntiles[i], std::min<int64_t>(max_splits, ntiles[i]));
  } else if (int64_t(base.size()) < fill_target) {
    auto auto_splits = [&](int64_t n, int64_t T) {       // (32-bit divisions: this runs a dozen times an item)
      return std::max<int64_t>(1, std::min(uint32_t(n + T - 1) / uint32_t(T), uint32_t(n) / uint32_t(min_split_tiles)));
    };
    const int64_t longest = base.empty() ? 1 : *std::max_element(ntiles.begin(), ntiles.end());
    // even splits of at most `target` items: the smallest T (no shorter than the minimum) that keeps to it;
    // the number of items does not grow with T, and with T = longest it is base.size() < fill_target
    auto even = [&](int64_t target) {
      auto total = [&](int64_t T) {
        int64_t n = 0;
        for (int64_t t : ntiles) n += auto_splits(t, T);
        return n;
      };
      int64_t lo = std::max<int64_t>(1, min_split_tiles), hi = std::max(lo, longest);
      if (total(lo) > target) {
        while (hi - lo > 1) {
          const int64_t mid = lo + (hi - lo) / 2;
          if (total(mid) <= target) hi = mid; else lo = mid;
        }
        lo = hi;
      }
      SplitPlan sp;
      sp.tps.reserve(ntiles.size());
      for (int64_t t : ntiles) {
        const uint32_t n = uint32_t(t), splits = uint32_t(auto_splits(t, lo)), tps = (n + splits - 1) / splits;
        sp.tps.push_back(tps);
        sp.pieces += (n + tps - 1) / tps;
      }
      return sp;
    };
    // The 8-wave grouped form also runs one workgroup per CU; a wave split to 512 items is two rounds of it.  Its
    // 256 slots are filled once where the model gives that more than 5 %, its mean error: 1.03 to 1.28 times
    // faster wherever it says so on the timed waves (one request of 8K-40K cached tokens, 64/8 heads, 304 rows
    // per KV head: 67.5 us as 352 items, 54.6 as 256), while 256 items always would lose 15 % on average.
    int64_t target = fill_target;
    if (!mla && !small_rows && int64_t(base.size()) < kNumCu && longest >= 2 * min_split_tiles &&
        grouped_cost(s, *batch, kNumCu, 1024) < 0.95 * grouped_cost(s, *batch, fill_target, 1024))
      target = kNumCu;
    split = even(target);
    // The latent form runs one workgroup per CU: 256 slots, not 512, and its partials are four times as wide.
    // For it the alternatives are even splits of at most 256 items, and pieces of about the mean load per
    // slot: whole pieces fill most slots and the items' remainders pair up on the others.  The cheapest by
    // split_cost is taken.  Measured on 12 requests of 4K-16K cached and 1-12 new tokens, 128 heads: 254 us with
    // the 512-item split, 243 with 256 even items.  The overheads are a piece's prologue and epilogue in
    // tiles, and the merge's share of a piece's partial rows at about 5 TB/s.
    if (mla && longest >= 2 * min_split_tiles) {
      const int slots = kNumCu;
      const double overhead = 5.0, merge = 0.015;
      double best = split_cost(ntiles, split, overhead, merge, INFINITY);
      auto consider = [&](SplitPlan sp) {
        if (sp.pieces > fill_target) return;
        const double c = split_cost(ntiles, sp, overhead, merge, best);
        if (c < best) {
          best = c;
          split = std::move(sp);
        }
      };
      if (int64_t(base.size()) < slots) consider(even(slots));
      const int64_t sum = std::accumulate(ntiles.begin(), ntiles.end(), int64_t(0));
      int64_t last = 0;
      for (double f : {1.0, 1.04, 1.08, 1.15, 1.25}) {
        const int64_t T = std::max<int64_t>(min_split_tiles, int64_t(std::ceil(f * double(sum) / slots)));
        if (T == last) continue;
        last = T;
        SplitPlan sp;
        sp.tps.reserve(ntiles.size());
        for (int64_t tiles : ntiles) {
          const uint32_t n = uint32_t(tiles);
          uint32_t t = std::min(uint32_t(T), n), whole = n / t, left = n - whole * t;
          // a remainder below the minimum split length is shared out over the whole pieces, once: the new last piece
          // can be short too (100 tiles: 11 pieces of 9 and one of 1).  Longer pieces until none is short: the
          // same time over 60 waves that it changes, single ones 9 % slower to 3 % faster.
          if (left && left < min_split_tiles) {
            t = (n + whole - 1) / whole;
            whole = n / t;
            left = n - whole * t;
          }
          sp.tps.push_back(t);
          sp.pieces += whole + (left != 0);
        }
        consider(std::move(sp));
      }
    }
  }
  std::vector<WorkItem> items;
  int64_t part_rows = 0;
  int max_used = 1;
  for (size_t bi = 0; bi < base.size(); ++bi) {
    const WorkItem& w = base[bi];
    const int64_t tps = split.tps[bi], S = ceil_div(ntiles[bi], tps);
    if (S == 1) {
      items.push_back(w);
      continue;
    }
    max_used = std::max<int>(max_used, int(S));
    MergeItem m{};
    m.req = w.req;
    m.kv_head = w.kv_head;
    m.row0 = w.row0;
    m.rows = w.rows;
    m.nsplit = int32_t(S);
    m.part = int32_t(part_rows);
    plan->merges.push_back(m);
    for (int64_t si = 0; si < S; ++si) {
      WorkItem x = w;
      x.kv_begin = int32_t(si * tps * KT);
      x.kv_end = int32_t(std::min<int64_t>(w.kv_end, (si + 1) * tps * KT));
      x.part = int32_t(part_rows + si * w.rows);
      x.split = int32_t(si);
      items.push_back(x);
    }
    part_rows += S * w.rows;
    if (part_rows > INT32_MAX / 2) {
      delete plan;
      return set_error(WAVEPP_EINVAL, "split partials too large");
    }
  }
  plan->num_real_items = int32_t(items.size());
  plan->max_splits_used = max_used;
  plan->partial_rows = part_rows;
  for (const MergeItem& m : plan->merges) plan->merge_rows = std::max(plan->merge_rows, m.rows);
  plan->num_merge_wide = merge_wide_items(plan->merges, plan->merge_rows, s.head_dim_v);
  // workgroups per CU: the 4-wave grouped form runs two, or three at head dim 64; the others one
  const int per_cu = small_rows && !mla ? (s.head_dim_qk == 64 ? 3 : 2) : 1;
  plan->items = order_items(std::move(items), G, env_flag("WAVEPP_XCD_ORDER", true),
                            env_flag("WAVEPP_STREAM_MAJOR", true), per_cu * kNumCu, KT, mla ? 5.0 : 1.0, mla || small_rows ? 1.0 : kModel128.idle);
  if (plan->items.size() > size_t(INT32_MAX / 2)) {
    delete plan;
    return set_error(WAVEPP_EINVAL, "too many work items");
  }

  // --- metadata blob -------------------------------------------------------------------------------
  size_t off = align_up(sizeof(MetaHeader), 16);
  plan->off_reqs = off;
  off = align_up(off + sizeof(ReqMeta) * R, 16);
  plan->off_bt = off;
  off = align_up(off + sizeof(int32_t) * size_t(R) * size_t(stride), 16);
  plan->off_items = off;
  off = align_up(off + sizeof(WorkItem) * plan->items.size(), 16);
  plan->off_merges = off;
  off = align_up(off + sizeof(MergeItem) * plan->merges.size(), 16);
  plan->blob.assign(off, 0);
  MetaHeader h{};
  h.magic = kMagic;
  h.serial = plan->serial;
  h.num_requests = R;
  h.num_items = int32_t(plan->items.size());
  h.num_merge = int32_t(plan->merges.size());
  h.bt_stride = stride;
  memcpy(plan->blob.data(), &h, sizeof(h));
  if (R) {
    memcpy(plan->blob.data() + plan->off_reqs, reqs.data(), sizeof(ReqMeta) * R);
    memcpy(plan->blob.data() + plan->off_bt, batch->block_table, sizeof(int32_t) * size_t(R) * size_t(stride));
  }
  if (!plan->items.empty())
    memcpy(plan->blob.data() + plan->off_items, plan->items.data(), sizeof(WorkItem) * plan->items.size());
  if (!plan->merges.empty())
    memcpy(plan->blob.data() + plan->off_merges, plan->merges.data(), sizeof(MergeItem) * plan->merges.size());
  plan->meta_bytes = align_up(off, 256);
  plan->off_opart = plan->meta_bytes;
  plan->off_lpart = align_up(plan->off_opart + sizeof(float) * size_t(part_rows) * size_t(s.head_dim_v), 256);
  plan->workspace_bytes = align_up(plan->off_lpart + sizeof(float) * size_t(part_rows), 256);
  *out = plan;
  return WAVEPP_OK;
}

size_t wavepp_plan_workspace_bytes(const wavepp_plan* plan) { return plan ? plan->workspace_bytes : 0; }

int wavepp_plan_get_info(const wavepp_plan* plan, wavepp_plan_info* info) {
  if (!plan || !info) return set_error(WAVEPP_EINVAL, "null argument");
  info->total_tokens = plan->total_tokens;
  info->num_items = int32_t(plan->items.size());
  info->num_real_items = plan->num_real_items;
  info->num_merge_items = int32_t(plan->merges.size());
  info->max_splits = plan->max_splits_used;
  info->rows_per_item = plan->rows_per_item;
  info->kv_tile = plan->kv_tile;
  info->partial_rows = plan->partial_rows;
  info->metadata_bytes = int64_t(plan->blob.size());
  info->workspace_bytes = int64_t(plan->workspace_bytes);
  return WAVEPP_OK;
}

int wavepp_plan_get_items(const wavepp_plan* plan, int32_t* items, int32_t capacity) {
  if (!plan || (!items && capacity > 0) || capacity < 0) return set_error(WAVEPP_EINVAL, "bad argument");
  const int32_t n = std::min<int32_t>(capacity, int32_t(plan->items.size()));
  for (int32_t i = 0; i < n; ++i) {
    const WorkItem& w = plan->items[i];
    const int32_t v[8] = {w.req, w.kv_head, w.row0, w.rows, w.kv_begin, w.kv_end, w.part, w.split};
    memcpy(items + 8 * int64_t(i), v, sizeof(v));
  }
  return n;
}

int wavepp_attn_plan_upload(const wavepp_plan* plan, void* workspace, size_t ws_bytes, hipStream_t stream) {
  clear_error();
  if (!plan) return set_error(WAVEPP_EINVAL, "plan is NULL");
  int st = check_workspace(plan, workspace, ws_bytes);
  if (st) return st;
  st = stage_and_copy(plan->blob.data(), plan->blob.size(), workspace, stream);
  if (st) return st;
  note_upload(workspace, plan->serial);
  return WAVEPP_OK;
}

int wavepp_attn_append_kv(const wavepp_plan* plan, const void* k_new, const void* v_new, void* k_pool, void* v_pool,
                          void* workspace, size_t ws_bytes, hipStream_t stream) {
  clear_error();
  if (!plan) return set_error(WAVEPP_EINVAL, "plan is NULL");
  int st = check_workspace(plan, workspace, ws_bytes);
  if (st) return st;
  const bool shared = plan->shape.kv_shared != 0;
  if (plan->total_tokens == 0) return WAVEPP_OK;
  st = require_upload(workspace, plan->serial, "wavepp_attn_plan_upload");
  if (st) return st;
  if (!k_new || !k_pool) return set_error(WAVEPP_EINVAL, "k_new / k_pool is NULL");
  if (!shared && (!v_new || !v_pool)) return set_error(WAVEPP_EINVAL, "v_new / v_pool is NULL");
  if (shared && (v_new || v_pool)) return set_error(WAVEPP_EINVAL, "v_new / v_pool must be NULL for a latent cache");
  if (!aligned16(k_new) || !aligned16(k_pool) || (!shared && (!aligned16(v_new) || !aligned16(v_pool))))
    return set_error(WAVEPP_EINVAL, "device buffers must be 16-byte aligned");
  DevPlan d = make_dev(plan, workspace);
  hipError_t e = launch_append(d, k_new, v_new, k_pool, v_pool, stream);
  if (e != hipSuccess) return set_hip_error(e, "append_kv launch");
  return WAVEPP_OK;
}

int wavepp_attn_chunked_prefill(const wavepp_plan* plan, const void* q, const void* k_pool, const void* v_pool,
                                void* out, float* lse, void* workspace, size_t ws_bytes, hipStream_t stream) {
  clear_error();
  if (!plan) return set_error(WAVEPP_EINVAL, "plan is NULL");
  int st = check_workspace(plan, workspace, ws_bytes);
  if (st) return st;
  const bool shared = plan->shape.kv_shared != 0;
  if (plan->total_tokens == 0) return WAVEPP_OK;
  st = require_upload(workspace, plan->serial, "wavepp_attn_plan_upload");
  if (st) return st;
  if (!q || !k_pool || !out) return set_error(WAVEPP_EINVAL, "q / k_pool / out is NULL");
  if (!shared && !v_pool) return set_error(WAVEPP_EINVAL, "v_pool is NULL");
  if (shared && v_pool) return set_error(WAVEPP_EINVAL, "v_pool must be NULL for a latent cache");
  if (!aligned16(q) || !aligned16(k_pool) || !aligned16(out) || (!shared && !aligned16(v_pool)) ||
      (reinterpret_cast<uintptr_t>(lse) & 3))
    return set_error(WAVEPP_EINVAL, "device buffers must be 16-byte aligned (lse 4-byte)");
  DevPlan d = make_dev(plan, workspace);
  hipError_t e = launch_attention(d, q, k_pool, v_pool, out, lse, stream);
  if (e != hipSuccess) return set_hip_error(e, "attention launch");
  if (!plan->merges.empty()) {
    e = launch_merge(d, out, lse, stream);
    if (e != hipSuccess) return set_hip_error(e, "merge launch");
  }
  return WAVEPP_OK;
}

int wavepp_attn_chunked_prefill_noalloc(const wavepp_plan* plan, const void* q, const void* k_new,
                                        const void* v_new, void* k_pool, void* v_pool, void* out, float* lse,
                                        hipStream_t stream) {
  clear_error();
  if (!plan) return set_error(WAVEPP_EINVAL, "plan is NULL");
  if (plan->workspace_bytes > kNoAllocScratchBytes)
    return set_error(WAVEPP_ENOSPACE, "plan needs %zu bytes of scratch, the static scratch holds %zu: plan the wave "
                     "with fewer key-range splits (max_splits) or call wavepp_attn_chunked_prefill with a workspace",
                     plan->workspace_bytes, kNoAllocScratchBytes);
  const bool shared = plan->shape.kv_shared != 0;
  if (plan->total_tokens == 0) return WAVEPP_OK;
  if (!q || !k_pool || !out) return set_error(WAVEPP_EINVAL, "q / k_pool / out is NULL");
  if (!shared && !v_pool) return set_error(WAVEPP_EINVAL, "v_pool is NULL");
  if (shared && (v_pool || v_new)) return set_error(WAVEPP_EINVAL, "v_pool / v_new must be NULL for a latent cache");
  if (k_new && !shared && !v_new) return set_error(WAVEPP_EINVAL, "v_new is NULL while k_new is given");
  if (!k_new && v_new) return set_error(WAVEPP_EINVAL, "v_new is given without k_new");
  if (!aligned16(q) || !aligned16(k_pool) || !aligned16(out) || (!shared && !aligned16(v_pool)) ||
      (k_new && !aligned16(k_new)) || (v_new && !aligned16(v_new)) || (reinterpret_cast<uintptr_t>(lse) & 3))
    return set_error(WAVEPP_EINVAL, "device buffers must be 16-byte aligned (lse 4-byte)");
  void* ws = nullptr;
  hipError_t e = noalloc_scratch(&ws);
  if (e != hipSuccess) return set_hip_error(e, "static scratch address");
  // the plan's metadata into the head of the scratch (from the plan's own host memory: no staging
  // buffer of the library's is involved), then the same kernels as the workspace entry points
  e = hipMemcpyAsync(ws, plan->blob.data(), plan->blob.size(), hipMemcpyHostToDevice, stream);
  if (e != hipSuccess) return set_hip_error(e, "metadata copy into the static scratch");
  DevPlan d = make_dev(plan, ws);
  if (k_new) {
    e = launch_append(d, k_new, v_new, k_pool, v_pool, stream);
    if (e != hipSuccess) return set_hip_error(e, "append_kv launch");
  }
  e = launch_attention(d, q, k_pool, v_pool, out, lse, stream);
  if (e != hipSuccess) return set_hip_error(e, "attention launch");
  if (!plan->merges.empty()) {
    e = launch_merge(d, out, lse, stream);
    if (e != hipSuccess) return set_hip_error(e, "merge launch");
  }
  return WAVEPP_OK;
}

void wavepp_plan_destroy(wavepp_plan* plan) { delete plan; }

}  // extern "C"
