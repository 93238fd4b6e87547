// Random batches through the host planner, built with AddressSanitizer and UBSan by
// tests/test_host_sanitizers.py: every (request, kv head, query row) must get each of its
// visible keys exactly once from the work items, whatever the knobs.
#include <cstdio>
#include <cstdlib>
#include <random>
#include "efim_internal.h"

using namespace efim;
int main() {
  std::mt19937 rng(7);
  long items_total = 0, once_plans = 0;
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
    efim_batch_t b{};
    b.batch = batch; b.cached_len = c.data(); b.new_len = n.data();
    b.num_q_heads = hq[h]; b.num_kv_heads = hkv[h]; b.head_dim = (rng() & 1) ? 64 : 128;
    b.page_size = 8 << (rng() % 6);
    int maxp = 0; for (int r = 0; r < batch; ++r) maxp = std::max(maxp, (c[r] + n[r] + b.page_size - 1) / b.page_size);
    b.max_pages_per_req = std::max(1, maxp); b.num_pages = 1 << 24;
    b.block_table = reinterpret_cast<const int32_t*>(0x1000);
    static const int splits[] = {-1, -1, 0, 64, 128, 512}; static const int tiles[] = {0, 0, 128, 256};
    tuning().split_kv = splits[rng() % 6]; tuning().row_tile = tiles[rng() % 4]; tuning().xcd_grouping = rng() & 1;
    int64_t total = 0;
    int rc = validate_batch(&b, &total);
    if (rc != EFIM_OK) { printf("validate rc %d at iter %d\n", rc, iter); return 1; }
    Plan plan;
    int slots = (rng() & 1) ? 256 : 512;
    build_plan(&b, slots, &plan);
    build_plan(&b, slots, &again);
    if (again.items.size() != plan.items.size() || again.merges.size() != plan.merges.size() || again.reqs.size() != plan.reqs.size() ||
        again.rows_per_item != plan.rows_per_item || again.max_item_rows != plan.max_item_rows || again.partial_rows != plan.partial_rows ||
        again.once != plan.once || again.rows16 != plan.rows16 || again.crowded != plan.crowded ||
        again.num_partial_slots != plan.num_partial_slots || again.total_bytes != plan.total_bytes ||
        again.header_bytes != plan.header_bytes) {
      printf("a plan built into a used object differs, iter %d\n", iter);
      return 1;
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
  printf("planner ok, %ld items, %ld plans for the whole-range kernel\n", items_total, once_plans);
  return 0;
}
