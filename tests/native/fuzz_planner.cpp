// Random batches through the host planner, built with AddressSanitizer and UBSan by
// tests/test_host_sanitizers.py: every (request, kv head, query row) must get each of its
// visible keys exactly once from the work items, whatever the knobs.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include "efim_internal.h"

using namespace efim;
namespace {

bool same(const Plan& a, const Plan& b) {
  return a.items.size() == b.items.size() && a.merges.size() == b.merges.size() && a.reqs.size() == b.reqs.size() &&
         a.rows_per_item == b.rows_per_item && a.fp8_rows_per_item == b.fp8_rows_per_item &&
         a.max_item_rows == b.max_item_rows && a.partial_rows == b.partial_rows && a.once == b.once &&
         a.rows16 == b.rows16 && a.crowded == b.crowded && a.static_items == b.static_items &&
         a.queued_items == b.queued_items && a.draws == b.draws && a.mean_tiles == b.mean_tiles &&
         a.num_partial_slots == b.num_partial_slots && a.total_bytes == b.total_bytes && a.header_bytes == b.header_bytes &&
         (a.items.empty() || std::memcmp(a.items.data(), b.items.data(), a.items.size() * sizeof(WorkItem)) == 0) &&
         (a.merges.empty() || std::memcmp(a.merges.data(), b.merges.data(), a.merges.size() * sizeof(MergeItem)) == 0);
}

bool fits_static(const Plan& p) { return p.header_bytes <= kStaticListBytes && p.total_bytes <= kStaticPartialBytes; }

// Large compute-heavy steps around what the static call holds: 256 rows where 128 do not fit and 256 do, and only
// there, and only over bf16 caches.
int static_limits(std::mt19937& rng) {
  long held_back = 0, beyond = 0;
  tuning() = Tuning();
  for (int iter = 0; iter < 60; ++iter) {
    const int batch = 400 + rng() % 1600;
    std::vector<int32_t> c(batch), n(batch);
    for (int r = 0; r < batch; ++r) { c[r] = 50 + rng() % 100; n[r] = 150 + rng() % 100; }
    efim_batch_t b{};
    b.batch = batch; b.cached_len = c.data(); b.new_len = n.data();
    b.num_q_heads = 32; b.num_kv_heads = 8; b.head_dim = 128; b.page_size = 16;
    b.max_pages_per_req = 32; b.num_pages = 1 << 24;
    b.block_table = reinterpret_cast<const int32_t*>(0x1000);
    Plan plan, codes, narrow, wide;
    build_plan(&b, 512, &plan);
    build_plan(&b, 512, &codes, true);
    tuning().row_tile = 128; build_plan(&b, 512, &narrow);
    tuning().row_tile = 256; build_plan(&b, 512, &wide);
    tuning().row_tile = 0;
    const bool hold = !fits_static(narrow) && fits_static(wide);
    held_back += hold;
    beyond += !fits_static(wide);
    if (plan.rows_per_item != (hold ? 256 : 128) || codes.rows_per_item != 128 || plan.fp8_rows_per_item != 128) {
      printf("%d requests: tile %d, over codes %d, list %zu / %zu bytes\n", batch, plan.rows_per_item, codes.rows_per_item,
             narrow.header_bytes, wide.header_bytes);
      return 1;
    }
  }
  if (held_back < 5 || beyond < 5) { printf("%ld held back, %ld beyond the limits\n", held_back, beyond); return 1; }
  return 0;
}

}  // namespace

int main() {
  std::mt19937 rng(7);
  long items_total = 0, once_plans = 0, queued_plans = 0, queued_parts = 0, other_tile = 0;
  Plan again;  // built over and over, as the library's cached plan is
  for (int iter = 0; iter < 1200; ++iter) {
    int batch = 1 + rng() % 12;
    std::vector<int32_t> c(batch), n(batch);
    for (int r = 0; r < batch; ++r) {
      int kind = rng() % 6;
      c[r] = kind == 0 ? 0 : (kind == 1 ? rng() % 70 : (kind == 2 ? rng() % 9000 : rng() % 40000));
      n[r] = (rng() % 5 == 0) ? 0 : (rng() % 3 == 0 ? 1 + rng() % 600 : 1 + rng() % 40);
    }
    // two of three batches are short steps: a few tokens per request, few key tiles
    if (iter % 3) {
      const int most = 1 + rng() % 8;
      for (int r = 0; r < batch; ++r) {
        n[r] = rng() % 7 == 0 ? 0 : 1 + rng() % most;
        if (iter % 3 == 1) c[r] %= 700;
      }
    }
    static const int hq[] = {1, 4, 8, 28, 32, 14, 6}, hkv[] = {1, 4, 2, 4, 8, 2, 1};
    int h = rng() % 7;
    // every sixth batch: long ranges of several kv heads and few slots, so that items are left to draw
    const bool queue = iter % 6 == 0;
    if (queue) {
      h = 3 + rng() % 2;
      for (int r = 0; r < batch; ++r) { c[r] = 2500 + rng() % 6000; n[r] = 1 + rng() % 3; }
    }
    efim_batch_t b{};
    b.batch = batch; b.cached_len = c.data(); b.new_len = n.data();
    b.num_q_heads = hq[h]; b.num_kv_heads = hkv[h]; b.head_dim = (rng() & 1) ? 64 : 128;
    b.page_size = 8 << (rng() % 6);
    int maxp = 0; for (int r = 0; r < batch; ++r) maxp = std::max(maxp, (c[r] + n[r] + b.page_size - 1) / b.page_size);
    b.max_pages_per_req = std::max(1, maxp); b.num_pages = 1 << 24;
    b.block_table = reinterpret_cast<const int32_t*>(0x1000);
    static const int splits[] = {-1, -1, 0, 64, 128, 512}; static const int tiles[] = {0, 0, 128, 256};
    tuning().split_kv = splits[rng() % 6];
    if (queue && tuning().split_kv > 0) tuning().split_kv = 64 * (40 + rng() % 30);
    tuning().row_tile = tiles[rng() % 4]; tuning().xcd_grouping = rng() & 1;
    int64_t total = 0;
    int rc = validate_batch(&b, &total);
    if (rc != EFIM_OK) { printf("validate rc %d at iter %d\n", rc, iter); return 1; }
    Plan plan;
    static const int slot_counts[] = {16, 256, 256, 512, 512};
    const int slots = queue ? 16 : slot_counts[rng() % 5];
    const bool fp8 = rng() % 3 == 0;
    build_plan(&b, slots, &plan, fp8);
    build_plan(&b, slots, &again, fp8);
    if (!same(again, plan)) {
      printf("a plan built into a used object differs, iter %d\n", iter);
      return 1;
    }
    // plans of one row tile are the same whatever the caches' format; the bf16 plan names the other one's tile
    Plan other;
    build_plan(&b, slots, &other, !fp8);
    if (other.rows_per_item == plan.rows_per_item ? !same(other, plan) : (fp8 ? plan : other).rows_per_item != plan.fp8_rows_per_item) {
      printf("plans of the two formats, iter %d\n", iter);
      return 1;
    }
    other_tile += other.rows_per_item != plan.rows_per_item;
    // queued items: the end of the list, none of them padding, no two items with keys in common, more draws than items
    const size_t start = (size_t)plan.static_items;
    if (start + plan.queued_items != plan.items.size() || (plan.queued_items == 0) != (plan.draws == 0) ||
        (plan.queued_items > 0 && plan.draws <= plan.queued_items)) {
      printf("queue iter %d: %zu + %d of %zu items, %d draws\n", iter, start, plan.queued_items, plan.items.size(), plan.draws);
      return 1;
    }
    if (plan.queued_items > 0) {
      ++queued_plans;
      queued_parts += !plan.merges.empty();
      for (size_t i = 0; i < plan.items.size(); ++i) {
        const WorkItem& w = plan.items[i];
        if (w.row_count == 0 && i < start) continue;
        bool bad = w.row_count == 0 || w.row_begin != 0;
        for (size_t k = 0; k < i; ++k) {
          const WorkItem& v = plan.items[k];
          bad = bad || (v.row_count > 0 && v.req == w.req && v.kv_head == w.kv_head && v.key_begin < w.key_end && w.key_begin < v.key_end);
        }
        if (bad) { printf("queue iter %d, item %zu\n", iter, i); return 1; }
      }
    }
    items_total += (long)plan.items.size();
    // the kernel that gathers whole ranges at once reads past its buffers if an item has more tiles than it
    // holds, and takes a whole compute unit per item
    if (plan.once) {
      ++once_plans;
      long live = 0;
      bool one_call = true;
      for (int r = 0; r < batch; ++r) one_call = one_call && n[r] >= 1 && n[r] <= kFusedMaxTokens;
      for (const WorkItem& w : plan.items) {
        if (w.row_count == 0) continue;
        ++live;
        if ((w.key_end - w.key_begin + kKeyTile - 1) / kKeyTile > once_tiles(b.head_dim) || w.row_count > once_rows(b.head_dim, one_call)) {
          printf("item too large for its kernel, iter %d\n", iter);
          return 1;
        }
      }
      if (live > slots / 2 || tuning().split_kv >= 0) { printf("whole-range kernel iter %d: %ld items\n", iter, live); return 1; }
    }
    // coverage: every (req, kv head, row) x key range is covered exactly once
    const int g = b.num_q_heads / b.num_kv_heads;
    for (int r = 0; r < batch; ++r) {
      if (n[r] == 0) continue;
      for (int kh = 0; kh < b.num_kv_heads; ++kh) {
        std::vector<int> rows(n[r] * g, 0);
        for (const WorkItem& w : plan.items) {
          if (w.row_count == 0 || w.req != r || w.kv_head != kh) continue;
          if (w.row_begin < 0 || w.row_begin + w.row_count > n[r] * g || w.key_begin < 0 || w.key_end <= w.key_begin) { printf("bad item iter %d\n", iter); return 1; }
          for (int i = 0; i < w.row_count; ++i) {
            int row = w.row_begin + i; int vis = c[r] + row / g + 1;
            int lo = std::min(w.key_begin, vis), hi = std::min(w.key_end, vis);
            rows[row] += hi - lo;
          }
        }
        for (int row = 0; row < n[r] * g; ++row)
          if (rows[row] != c[r] + row / g + 1) { printf("coverage iter %d req %d head %d row %d: %d vs %d\n", iter, r, kh, row, rows[row], c[r] + row / g + 1); return 1; }
      }
    }
  }
  if (once_plans < 50) { printf("only %ld plans for the whole-range kernel\n", once_plans); return 1; }
  if (queued_plans < 50 || queued_parts < 10 || other_tile < 10) {
    printf("%ld plans with queued items, %ld of them with parts, %ld with another tile over codes\n", queued_plans, queued_parts, other_tile);
    return 1;
  }
  if (static_limits(rng)) return 1;
  for (size_t merges = 1; merges < (size_t)kTicketsPerSlot; ++merges) {
    const int shift = ticket_shift(merges);   // counters apart, all in front of the block's last word
    if (((merges - 1) << shift) >= (size_t)kTicketsPerSlot - 1 || (shift < 4 && (merges << (shift + 1)) < (size_t)kTicketsPerSlot)) {
      printf("%zu counters: shift %d\n", merges, shift);
      return 1;
    }
  }
  printf("planner ok, %ld items, %ld plans for the whole-range kernel, %ld with queued items\n", items_total, once_plans, queued_plans);
  return 0;
}
