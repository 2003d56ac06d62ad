// Host side of the KDA chunked prefill: validation of the wave, the work list and the launch.
//
// Resume semantics follow the paper's statement that a recurrent layer resumes only from the exact
// state at its prefix boundary (Preliminaries, "Reuse"): each request names the snapshot slot it
// resumes from and the slot that receives its state at the chunk boundary.  Because a wave's
// workgroups run concurrently, a slot written by one request may not be read or written by another.
#include "wavepp_kda.h"
#include "internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <numeric>
#include <vector>

using namespace wavepp;

struct wavepp_kda_plan_s {
  wavepp_kda_shape shape;
  int64_t total_tokens = 0;
  uint32_t serial = 0;
  std::vector<KdaItem> items;
  std::vector<unsigned char> blob;
  size_t off_items = 0;
  bool listed = false;   // each workgroup's chains follow the items
  size_t workspace_bytes = 0;
};

namespace {

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

int check_ws(const wavepp_kda_plan_t* plan, void* ws, size_t ws_bytes) {
  if (!ws) return set_error(WAVEPP_EINVAL, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(ws) % 256) return set_error(WAVEPP_EINVAL, "workspace must be 256-byte aligned");
  if (ws_bytes < plan->workspace_bytes)
    return set_error(WAVEPP_ENOSPACE, "workspace has %zu bytes, plan needs %zu", ws_bytes, plan->workspace_bytes);
  return WAVEPP_OK;
}

// Which of the kernel's kNumCu resident workgroups runs each chain: longest first, each to the workgroup with
// the least work so far, as the hardware hands out workgroups of one chain.  A fixed order that gives every workgroup
// a chain of each round, whatever it has, is 1.3 to 1.5 times slower on waves of one long prompt beside many
// short ones: 1 x 4,096 and 63 x 512 tokens, 32 heads: 120 blocks on the busiest workgroup, 600 us, against 72
// and 438-448; 1 x 8,192 and 255 x 512, 16 heads: 1,220 us against 830-850.  A chain costs its blocks and about
// half a block for its snapshots (16 chains of 4 blocks a workgroup take 411 us, one of 64 blocks 369).
// Empty where the fixed order is as good: at most one chain a workgroup, all of the same number of blocks, or less
// than 2 % between the two (64 requests of 200-312 tokens, 64 heads: 442 us in the fixed order, 444-446 listed);
// and beyond kKdaMaxListed chains, thousands a workgroup, where its imbalance is small but for a chain as long as
// many.  Listing takes about 5 ns a chain.
// The chains of `items` (longest first) come in runs of equal length.  Within a run the workgroups' new loads
// only grow, so the least loaded one is at the head of one of two sorted queues: no heap.  Of equally loaded ones the
// last that was given a chain is first, so that rounds of equal chains alternate in direction like the fixed order (64
// requests of one token, 64 heads: 114 us in the fixed order, 116 listed so, 133 first given first).
std::vector<int32_t> chain_owners(const std::vector<KdaItem>& items, int heads) {
  std::vector<int32_t> owner;
  auto blocks = [&](size_t i) { return int64_t(items[i].len + kKdaBlock - 1) / kKdaBlock; };
  auto cost_of = [&](size_t i) { return 2 * blocks(i) + 1; };         // of a chain of item i, in half blocks
  const int64_t chains = int64_t(items.size()) * heads;
  if (chains <= kNumCu || chains > kKdaMaxListed || blocks(0) == blocks(items.size() - 1)) return owner;
  // the busiest workgroup in the fixed order, against the least that any order can give it
  int64_t fixed[kNumCu] = {}, total = 0, n = 0;
  for (size_t i = 0; i < items.size(); ++i) {
    const int64_t cost = cost_of(i);
    for (int h = 0; h < heads; ++h, ++n) fixed[n / kNumCu & 1 ? kNumCu - 1 - n % kNumCu : n % kNumCu] += cost;
    total += cost * heads;
  }
  const int64_t busiest = *std::max_element(fixed, fixed + kNumCu);
  if (50 * busiest <= 51 * std::max(total / kNumCu, cost_of(0))) return owner;
  owner.resize(size_t(chains));
  typedef std::pair<int64_t, int32_t> Load;           // (work, workgroup)
  std::vector<Load> ready, given, rest;
  given.reserve(size_t(chains));           // (no reallocation while it is read and added to)
  for (int32_t w = 0; w < kNumCu; ++w) ready.push_back(Load(0, w));
  int64_t c = 0;
  for (size_t i = 0, j; i < items.size(); i = j) {
    for (j = i + 1; j < items.size() && blocks(j) == blocks(i);) ++j;
    const int64_t cost = cost_of(i), end = int64_t(j) * heads;
    size_t r = 0, g = 0;
    given.clear();
    while (c < end) {
      const bool old = r < ready.size() && (g == given.size() || ready[r].first <= given[g].first);
      std::vector<Load>& from = old ? ready : given;
      size_t& head = old ? r : g;
      const int64_t load = from[head].first;
      size_t tail = head;
      while (tail < from.size() && from[tail].first == load) ++tail;
      size_t left = tail;
      for (; left > head && c < end; ++c) {
        const int32_t w = from[--left].second;
        owner[size_t(c)] = w;
        given.push_back(Load(load + cost, w));
      }
      // what is left of the equal ones (at the run's end) moves up to the others
      std::move_backward(from.begin() + head, from.begin() + left, from.begin() + tail);
      head = tail - (left - head);
    }
    rest.clear();
    std::merge(ready.begin() + r, ready.end(), given.begin() + g, given.end(), std::back_inserter(rest));
    ready.swap(rest);
  }
  if (50 * busiest <= 51 * ready.back().first) owner.clear();
  return owner;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

extern "C" {

int wavepp_kda_plan(const wavepp_kda_shape* shape, const wavepp_kda_batch* batch, wavepp_kda_plan_t** out) {
  clear_error();
  if (!shape || !batch || !out) return set_error(WAVEPP_EINVAL, "null argument");
  *out = nullptr;
  const wavepp_kda_shape s = *shape;
  if (s.num_heads <= 0 || s.head_dim_k <= 0 || s.head_dim_v <= 0 || s.num_state_slots < 0)
    return set_error(WAVEPP_EINVAL, "non-positive shape field");
  if (s.head_dim_k != kKdaDim || s.head_dim_v != kKdaDim)
    return set_error(WAVEPP_EUNSUPPORTED, "unsupported head dims (d_k=%d, d_v=%d): only %d x %d", s.head_dim_k,
                     s.head_dim_v, kKdaDim, kKdaDim);
  if (int64_t(s.num_heads) * kKdaDim > INT32_MAX / 4) return set_error(WAVEPP_EINVAL, "too many heads");
  const int32_t R = batch->num_requests;
  if (R < 0) return set_error(WAVEPP_EINVAL, "num_requests < 0");
  if (R > 0 && (!batch->chunk_lens || !batch->state_in || !batch->state_out))
    return set_error(WAVEPP_EINVAL, "null chunk_lens / state_in / state_out");

  int64_t total = 0;
  std::vector<int32_t> writer(size_t(s.num_state_slots), -1);
  for (int32_t r = 0; r < R; ++r) {
    const int32_t c = batch->chunk_lens[r];
    if (c < 0) return set_error(WAVEPP_EINVAL, "request %d: negative chunk length %d", r, c);
    total += c;
    if (total > INT32_MAX / 2) return set_error(WAVEPP_EINVAL, "too many tokens in the wave");
    if (c == 0) continue;
    const int32_t si = batch->state_in[r], so = batch->state_out[r];
    if (si < -1 || si >= s.num_state_slots)
      return set_error(WAVEPP_ERANGE, "request %d: state_in %d outside [-1, %d)", r, si, s.num_state_slots);
    if (so < 0 || so >= s.num_state_slots)
      return set_error(WAVEPP_ERANGE, "request %d: state_out %d outside [0, %d)", r, so, s.num_state_slots);
    if (writer[so] >= 0)
      return set_error(WAVEPP_EALIAS, "requests %d and %d both write snapshot slot %d", writer[so], r, so);
    writer[so] = r;
  }
  if (int64_t(total) * s.num_heads > int64_t(INT32_MAX) * 4)
    return set_error(WAVEPP_EINVAL, "wave too large");
  for (int32_t r = 0; r < R; ++r) {
    if (batch->chunk_lens[r] == 0) continue;
    const int32_t si = batch->state_in[r];
    if (si >= 0 && writer[si] >= 0 && writer[si] != r)
      return set_error(WAVEPP_EALIAS, "request %d resumes from slot %d, which request %d writes", r, si, writer[si]);
  }

  auto plan = new (std::nothrow) wavepp_kda_plan_t();
  if (!plan) return set_error(WAVEPP_EINVAL, "out of host memory");
  plan->shape = s;
  plan->total_tokens = total;
  plan->serial = next_serial();
  int64_t cu = 0;
  for (int32_t r = 0; r < R; ++r) {
    const int32_t c = batch->chunk_lens[r];
    if (c > 0) {
      KdaItem it{};
      it.req = r;
      it.cu = int32_t(cu);
      it.len = c;
      it.state_in = batch->state_in[r];
      it.state_out = batch->state_out[r];
      plan->items.push_back(it);
    }
    cu += c;
  }
  // longest chunks first: the order in which chains are given to workgroups
  std::stable_sort(plan->items.begin(), plan->items.end(),
                   [](const KdaItem& a, const KdaItem& b) { return a.len > b.len; });
  if (int64_t(plan->items.size()) * s.num_heads > INT32_MAX / 2) {
    delete plan;
    return set_error(WAVEPP_EINVAL, "too many workgroups");
  }
  plan->off_items = align_up(sizeof(KdaHeader), 16);
  size_t bytes = plan->off_items + sizeof(KdaItem) * plan->items.size();
  std::vector<int32_t> list;
  if (!plan->items.empty()) {
    const std::vector<int32_t> owner = chain_owners(plan->items, s.num_heads);
    if (!owner.empty()) {
      list.assign(kNumCu + 1, 0);
      for (int32_t w : owner) ++list[size_t(w) + 1];
      list[0] = kNumCu + 1;
      for (int w = 0; w < kNumCu; ++w) list[w + 1] += list[w];
      std::vector<int32_t> at(list);
      list.resize(list.size() + owner.size());
      for (size_t c = 0; c < owner.size(); ++c) list[at[owner[c]]++] = int32_t(c);
      plan->listed = true;
      bytes = align_up(bytes + sizeof(int32_t) * list.size(), 16);
    }
  }
  plan->blob.assign(bytes, 0);
  KdaHeader h{};
  h.magic = kKdaMagic;
  h.serial = plan->serial;
  h.num_items = int32_t(plan->items.size());
  h.num_heads = s.num_heads;
  memcpy(plan->blob.data(), &h, sizeof(h));
  if (!plan->items.empty())
    memcpy(plan->blob.data() + plan->off_items, plan->items.data(), sizeof(KdaItem) * plan->items.size());
  if (!list.empty())
    memcpy(plan->blob.data() + plan->off_items + sizeof(KdaItem) * plan->items.size(), list.data(),
           sizeof(int32_t) * list.size());
  plan->workspace_bytes = align_up(plan->blob.size(), 256);
  *out = plan;
  return WAVEPP_OK;
}

size_t wavepp_kda_workspace_bytes(const wavepp_kda_plan_t* plan) { return plan ? plan->workspace_bytes : 0; }

int wavepp_kda_get_info(const wavepp_kda_plan_t* plan, wavepp_kda_info* info) {
  if (!plan || !info) return set_error(WAVEPP_EINVAL, "null argument");
  info->total_tokens = plan->total_tokens;
  info->num_items = int32_t(plan->items.size());
  info->block_tokens = kKdaBlock;
  info->metadata_bytes = int64_t(plan->blob.size());
  info->workspace_bytes = int64_t(plan->workspace_bytes);
  return WAVEPP_OK;
}

int wavepp_kda_upload(const wavepp_kda_plan_t* plan, void* workspace, size_t ws_bytes, hipStream_t stream) {
  clear_error();
  if (!plan) return set_error(WAVEPP_EINVAL, "plan is NULL");
  int st = check_ws(plan, workspace, ws_bytes);
  if (st) return st;
  st = stage_and_copy(plan->blob.data(), plan->blob.size(), workspace, stream);
  if (st) return st;
  note_upload(workspace, plan->serial);
  return WAVEPP_OK;
}

int wavepp_kda_chunked_prefill(const wavepp_kda_plan_t* plan, const void* q, const void* k, const void* v,
                               const float* alpha, const float* beta, float* state_pool, void* out,
                               void* workspace, size_t ws_bytes, hipStream_t stream) {
  clear_error();
  if (!plan) return set_error(WAVEPP_EINVAL, "plan is NULL");
  int st = check_ws(plan, workspace, ws_bytes);
  if (st) return st;
  if (plan->items.empty()) return WAVEPP_OK;
  st = require_upload(workspace, plan->serial, "wavepp_kda_upload");
  if (st) return st;
  if (!q || !k || !v || !alpha || !beta || !state_pool || !out)
    return set_error(WAVEPP_EINVAL, "q / k / v / alpha / beta / state_pool / out is NULL");
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(alpha) || !aligned16(beta) ||
      !aligned16(state_pool) || !aligned16(out))
    return set_error(WAVEPP_EINVAL, "device buffers must be 16-byte aligned");
  KdaDevPlan d{};
  auto* base = static_cast<unsigned char*>(workspace);
  d.hdr = reinterpret_cast<const KdaHeader*>(base);
  d.items = reinterpret_cast<const KdaItem*>(base + plan->off_items);
  d.listed = plan->listed;
  d.serial = plan->serial;
  d.num_items = int32_t(plan->items.size());
  d.num_heads = plan->shape.num_heads;
  hipError_t e = launch_kda_prefill(d, q, k, v, alpha, beta, state_pool, out, stream);
  if (e != hipSuccess) return set_hip_error(e, "kda launch");
  return WAVEPP_OK;
}

void wavepp_kda_destroy(wavepp_kda_plan_t* plan) { delete plan; }

}  // extern "C"
