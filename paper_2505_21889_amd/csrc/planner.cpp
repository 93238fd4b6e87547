// Host-side planner: turns the ragged batch into a list of workgroup-sized work items.
//
// Row space of a (request, kv head) pair: row = token * g + head_in_group with g = Hq/Hkv,
// so rows of one token are adjacent and the causal limit C_r + token + 1 grows with the row.
// A query tile is a run of `rows_per_item` such rows; it needs keys [0, C_r + last_token + 1).
// When there are too few tiles to fill the device, or some are much longer than the average,
// the key range of a tile is cut into chunks (multiples of the 64-key LDS tile) whose partial
// results a merge pass combines in a fixed order.
#include <algorithm>
#include <cstring>
#include <functional>

#include "efim_internal.h"

namespace efim {

Tuning& tuning() {
  static Tuning t;
  return t;
}

int validate_batch(const efim_batch_t* b, int64_t* total_new) {
  if (!b) return EFIM_ERR_INVALID_ARG;
  if (b->batch < 0 || b->num_q_heads <= 0 || b->num_kv_heads <= 0 || b->head_dim <= 0 ||
      b->page_size <= 0 || b->max_pages_per_req < 0 || b->num_pages < 0)
    return EFIM_ERR_INVALID_ARG;
  if (b->num_q_heads % b->num_kv_heads != 0) return EFIM_ERR_INVALID_ARG;
  if (b->head_dim != 64 && b->head_dim != 128) return EFIM_ERR_UNSUPPORTED;
  // pages are powers of two; a 1 KB gather (4 or 8 tokens of one head) must not cross one
  if (b->page_size < kMinPageSize || b->page_size > kMaxPageSize || (b->page_size & (b->page_size - 1)) != 0)
    return EFIM_ERR_UNSUPPORTED;
  if (b->num_q_heads / b->num_kv_heads > 64) return EFIM_ERR_UNSUPPORTED;
  int64_t total = 0;
  if (b->batch > 0) {
    if (!b->cached_len || !b->new_len) return EFIM_ERR_INVALID_ARG;
    for (int r = 0; r < b->batch; ++r) {
      const int64_t c = b->cached_len[r], n = b->new_len[r];
      if (c < 0 || n < 0) return EFIM_ERR_INVALID_ARG;
      if (c + n > (int64_t)1 << 30) return EFIM_ERR_UNSUPPORTED;
      if (n > 0) {
        const int64_t pages = (c + n + b->page_size - 1) / b->page_size;
        if (pages > b->max_pages_per_req || pages > b->num_pages) return EFIM_ERR_INVALID_ARG;
      }
      total += n;
    }
    if (total * b->num_q_heads > (int64_t)1 << 31) return EFIM_ERR_UNSUPPORTED;
    if (total > 0 && !b->block_table) return EFIM_ERR_INVALID_ARG;
  }
  if (total_new) *total_new = total;
  return EFIM_OK;
}

namespace {

struct Tile {
  int32_t req, kv_head, row_begin, row_count, key_end;
  int32_t ktiles;  // ceil(key_end / kKeyTile)
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Query-row tile of a workgroup: 128 rows (each of the 4 waves owns 32; two workgroups per compute unit) or 256 (8
// waves; one workgroup per unit, which gathers a key tile once for twice the rows and two tiles ahead).
// The loops of both do the same work in the same time (8 waves 1.84 us per key tile of a unit, two times 4 waves
// 1.83), so what surrounds them decides.  Two workgroups on a unit cover each other's start and end, and half
// the tile leaves less of a last tile empty and packs better; with long ranges the gathers count and little else
// does.  A compute-heavy step ("compute-heavy": more than the machine balance of about 315 flop per byte, 2.5
// PFLOP/s over 8 TB/s) takes 128 rows up to 32 key tiles in the mean, 64 with head dim 64, and over 8-bit caches
// whenever the workspace that the size query names holds that plan (fp8_plan).  Time with 128 rows over time
// with 256, drawn steps with more than 128 rows per kv head, geometric mean (range): bf16, head dim 128, up to 32
// tiles 0.954 (0.77 .. 1.02, 23 steps), 32 to 40 0.991 (0.95 .. 1.01, 6), 40 to 100 0.997 (0.95 .. 1.11, 9), above 1.009
// (0.94 .. 1.06, 13): past 32 nothing is gained in the mean, and the 256 rows that gather half as often
// stay.  Head dim 64, up to 64 tiles 0.96 (0.87 .. 1.01); 8-bit caches, 9 to 214 tiles, 0.92 (0.80 .. 0.98).
// A step bound by HBM takes 256 rows when it has at least two such tiles per compute unit, which then balance
// over the units without cutting key ranges (no merge pass), and few of its key ranges are read by more
// than one tile (34 requests of 824..1782 + 203..512 tokens, 32/32 heads: 416 / 396 us).
struct RowTile {
  int bf16 = 128, fp8 = 128;  // rows, by the format of the caches
  bool narrowed = false;      // bf16: 128 where the step's size alone says 256
  size_t wide_tiles = 0;      // of 256 rows
};

RowTile choose_row_tile(const efim_batch_t* b, int num_slots) {
  RowTile tile;
  const Tuning& tn = tuning();
  if (tn.row_tile != 0) {
    tile.bf16 = tile.fp8 = tn.row_tile;
    return tile;
  }
  const int g = b->num_q_heads / b->num_kv_heads;
  const int D = b->head_dim;
  const double long_keys = 32.0 * kKeyTile * 128 / D;  // keys a row sees, in the mean over the work
  double flops = 0.0, bytes = 0.0, work = 0.0, work_keys = 0.0, keys = 0.0, keys_read = 0.0;
  int64_t max_rows = 0;
  for (int r = 0; r < b->batch; ++r) {
    const double n = b->new_len[r], c = b->cached_len[r];
    if (n == 0) continue;
    const double seen = c + 0.5 * (n + 1);  // keys a row sees, in the mean
    const int64_t rows = (int64_t)g * b->new_len[r], t = (rows + 255) / 256;
    max_rows = std::max(max_rows, rows);
    flops += 4.0 * D * b->num_q_heads * n * seen;
    bytes += 4.0 * D * ((c + n) * b->num_kv_heads + n * b->num_q_heads);
    work += n * seen;
    work_keys += n * seen * seen;
    keys += c + n;
    keys_read += t * c + n * (t + 1) / 2;
    tile.wide_tiles += (size_t)(b->num_kv_heads * t);
  }
  const bool heavy = max_rows > 128 && flops > 315.0 * bytes;
  if (!heavy && tile.wide_tiles < (size_t)num_slots) return tile;
  tile.narrowed = heavy ? work_keys < long_keys * work : max_rows > 128 && keys_read >= 1.5 * keys;
  tile.bf16 = tile.narrowed ? 128 : 256;
  tile.fp8 = heavy ? 128 : tile.bf16;
  return tile;
}

// Builds the plan with row tiles of M rows.
void build(const efim_batch_t* b, int num_slots, int M, Plan* plan) {
  const int g = b->num_q_heads / b->num_kv_heads;
  const int D = b->head_dim;
  plan->reqs.clear();
  plan->items.clear();
  plan->merges.clear();
  plan->num_partial_slots = 0;
  plan->crowded = false;

  int64_t row = 0;
  int64_t max_rows = 0;
  double keys = 0.0;
  for (int r = 0; r < b->batch; ++r) {
    ReqInfo ri{b->cached_len[r], b->new_len[r], (int32_t)row, 0};
    plan->reqs.push_back(ri);
    row += b->new_len[r];
    max_rows = std::max<int64_t>(max_rows, (int64_t)g * b->new_len[r]);
    if (b->new_len[r] > 0) keys += (double)b->cached_len[r] + b->new_len[r];
  }
  plan->rows_per_item = M;
  if (M == 256) num_slots = std::max(1, num_slots / 2);  // 8-wave workgroups: one per compute unit

  std::vector<Tile> tiles;
  int64_t total_cost = 0;
  int64_t max_cost = 0;
  for (int r = 0; r < b->batch; ++r) {
    const int64_t n = b->new_len[r], c = b->cached_len[r];
    if (n == 0) continue;
    const int64_t rows = n * g;
    for (int h = 0; h < b->num_kv_heads; ++h) {
      for (int64_t r0 = 0; r0 < rows; r0 += M) {
        Tile t;
        t.req = r;
        t.kv_head = h;
        t.row_begin = (int32_t)r0;
        t.row_count = (int32_t)std::min<int64_t>(M, rows - r0);
        const int64_t last_token = (r0 + t.row_count - 1) / g;
        t.key_end = (int32_t)(c + last_token + 1);
        t.ktiles = (t.key_end + kKeyTile - 1) / kKeyTile;
        tiles.push_back(t);
        total_cost += t.ktiles + 4;
        max_cost = std::max<int64_t>(max_cost, t.ktiles + 4);
      }
    }
  }

  // Split policy.  chunk = key tiles per work item (0 = no split).  A workgroup slot's fair
  // share of the whole step is `avg`; a tile much longer than that would finish last, so long
  // tiles are cut into pieces.  Which piece length is best depends on how the pieces pack
  // into the slots (one piece too many costs a whole extra round with most slots idle), so
  // for steps of moderate size the candidates are tried on a model of the device: pieces
  // handed out longest first to `num_slots` slots, a fixed start-up cost per piece.
  const Tuning& tn = tuning();
  constexpr int64_t kStartCost = 4;  // start-up of a work item, in units of one key tile
  auto pieces_of = [&](const Tile& t, int64_t chunk) {
    return (chunk > 0 && 10 * (int64_t)t.ktiles > 13 * chunk) ? (int)((t.ktiles + chunk - 1) / chunk) : 1;
  };
  int64_t chunk = 0;
  if (tn.split_kv > 0) {
    chunk = std::max(1, tn.split_kv / kKeyTile);
  } else if (tn.split_kv < 0 && !tiles.empty()) {
    const double avg = (double)total_cost / std::max(1, num_slots);
    if ((double)max_cost > 1.3 * avg) {
      chunk = (int64_t)std::max(4.0, avg);
      if (tiles.size() <= (size_t)4 * num_slots) {
        // Quick estimate of a candidate: the pieces run in rounds of `num_slots`, a round
        // lasts as long as the longest piece.  The most promising candidates are then played
        // through: pieces handed out longest first, each to the slot that is free first, the
        // step taking as long as the fullest slot.  (A finer model with bandwidth sharing
        // between busy slots was fitted to chunk sweeps on the device and picked worse plans.)
        auto estimate = [&](int64_t c) {
          int64_t pieces = 0, longest = 0;
          for (const Tile& t : tiles) {
            const int n = pieces_of(t, c);
            pieces += n;
            longest = std::max<int64_t>(longest, (t.ktiles + n - 1) / n);
          }
          const int64_t rounds = (pieces + num_slots - 1) / num_slots;
          return rounds * (longest + kStartCost);
        };
        std::vector<int64_t> costs, load;
        auto makespan = [&](int64_t c) {
          costs.clear();
          for (const Tile& t : tiles) {
            const int n = pieces_of(t, c);
            const int64_t per = (t.ktiles + n - 1) / n;
            for (int64_t done = 0; done < t.ktiles; done += per)
              costs.push_back(std::min<int64_t>(per, t.ktiles - done) + kStartCost);
          }
          std::sort(costs.begin(), costs.end(), std::greater<int64_t>());
          load.assign((size_t)num_slots, 0);  // min-heap of slot loads
          auto cmp = std::greater<int64_t>();
          for (int64_t w : costs) {
            std::pop_heap(load.begin(), load.end(), cmp);
            load.back() += w;
            std::push_heap(load.begin(), load.end(), cmp);
          }
          return *std::max_element(load.begin(), load.end());
        };
        const int64_t lo = std::max<int64_t>(4, (int64_t)(0.5 * avg));
        const int64_t hi = std::max<int64_t>(lo, max_cost - kStartCost);
        const int64_t step = std::max<int64_t>(1, (hi - lo) / 64);
        std::vector<std::pair<int64_t, int64_t>> ranked;  // (estimate, candidate)
        for (int64_t c = lo; c <= hi; c += step) ranked.push_back({estimate(c), c});
        std::sort(ranked.begin(), ranked.end());
        int64_t best = makespan(chunk), best_chunk = chunk;
        for (size_t i = 0; i < ranked.size() && i < 6; ++i) {
          const int64_t c = ranked[i].second;
          const int64_t m = makespan(c);
          if (m < best || (m == best && c > best_chunk)) { best = m; best_chunk = c; }
        }
        chunk = best_chunk;
      }
    }
  }

  // Few rows per item and few tiles in all: cut so that every item fits the kernel that gathers its
  // whole range at once, if that makes at most one item per compute unit (that kernel takes the
  // whole LDS of one).  Measured over 94 short steps on either kernel: 0.67 .. 1.007 of the ring's time, 0.89
  // in the mean; with a few tiles per item 0.80 .. 0.95, nothing where the ring had them all in flight too (one
  // request of 8000 keys, 4 heads of 64: 11.8 / 11.7 us; 32/8 heads of 128, 256 items of four tiles: 14.7 / 14.8).  Up
  // to half as many items as units would leave room for a second stream's, but single launches of 129 to 256
  // items are 5 to 20 % slower on the ring (32 requests of 200 keys, 8 layers 89 / 78 us).
  // 8-bit caches with head dim 64 on pages of 8 have no such kernel (their loads span two pages) and run
  // the ring over the same items: ranges of six to eight tiles that would be two parts are one there, which is
  // faster too (8 layers, cut / whole: one request of 330 keys 66.6 / 62.0 us, 16 of 400 71.2 / 66.7, 8 of 500
  // with 16 rows 87.0 / 82.0, two calls, 8 of 400 with 32 rows 123.3 / 116.9).
  // A range that the policy above leaves whole although it does not fit (five
  // tiles of head dim 128) stays whole, and the launch with it on the ring kernel: its fp32 sums go
  // to the output directly, and a cut would put them through binary16 parts, a workspace and, with
  // more than 8 rows, a second launch.  (Speed goes either way.  8 layers, whole / cut: one request of
  // 270 keys with 32 rows per kv head in two calls 120 / 133 us, two of 300 keys with 32 rows 114 / 128;
  // one of 270 keys and one new token in one call, 32/8 heads 80 / 74, eight such 85 / 75.)
  // Head dim 128 with 17 to 32 rows: the sums of eight waves are 128 KB that go through LDS behind the last
  // tile.  The two calls do not gain that back, the step in one call does (its prologue runs on eight
  // waves too), and both have to give the same `out`: only batches that the one call takes.  8 layers,
  // ring / whole range gathered, two calls and one call: 8 requests of 1000 keys, 32 rows 161 / 169 and 152 /
  // 146 us; 25 of 250 keys, 32 rows 129 / 137 and 123 / 114; one of 1000 keys, 32 rows 128 / 131 and 132 / 115;
  // 24 of 250 keys, 28 rows 109 / 114 and 108 / 93.  Head dim 64, 32 rows: 32 of 500 keys 148 / 135 and 127 / 100.
  plan->once = false;
  const bool one_call = std::all_of(b->new_len, b->new_len + b->batch, [](int32_t n) { return n >= 1 && n <= kFusedMaxTokens; });
  if (max_rows <= once_rows(D, one_call) && tn.split_kv < 0) {
    const int64_t most = once_tiles(D), units = M == 256 ? num_slots : num_slots / 2;
    const int64_t cut = chunk > 0 ? std::min(chunk, most) : most;
    int64_t pieces = 0;
    bool fits = true;
    for (const Tile& t : tiles) {
      fits = fits && (t.ktiles <= most || pieces_of(t, chunk) > 1);
      pieces += t.ktiles > most ? (t.ktiles + cut - 1) / cut : 1;
    }
    plan->once = fits && pieces <= units;
    if (plan->once) chunk = cut;
  }
  auto cuts_of = [&](const Tile& t) {
    if (!plan->once) return pieces_of(t, chunk);
    return t.ktiles > once_tiles(D) ? (int)((t.ktiles + chunk - 1) / chunk) : 1;
  };

  struct Pending { WorkItem w; int64_t cost; int64_t group; };
  std::vector<Pending> pend;
  pend.reserve(tiles.size() * 2);
  int64_t slot = 0;
  for (const Tile& t : tiles) {
    const int nsplit = cuts_of(t);
    const int64_t group = (int64_t)t.req * b->num_kv_heads + t.kv_head;
    if (nsplit == 1) {
      WorkItem w{t.req, t.kv_head, t.row_begin, t.row_count, 0, t.key_end, -1, -1};
      pend.push_back({w, t.ktiles + 4, group});
    } else {
      const int per = (t.ktiles + nsplit - 1) / nsplit;  // key tiles per chunk
      MergeItem m{t.req, t.kv_head, t.row_begin, t.row_count, (int32_t)slot, 0, plan->reqs[t.req].row_start, 0};
      int made = 0;
      for (int s = 0; s < nsplit; ++s) {
        const int64_t kb = (int64_t)s * per * kKeyTile;
        if (kb >= t.key_end) break;
        const int64_t ke = std::min<int64_t>(t.key_end, kb + (int64_t)per * kKeyTile);
        WorkItem w{t.req, t.kv_head, t.row_begin, t.row_count, (int32_t)kb, (int32_t)ke,
                   (int32_t)(slot + made), (int32_t)plan->merges.size()};
        pend.push_back({w, (ke - kb + kKeyTile - 1) / kKeyTile + 4, group});
        ++made;
      }
      m.nsplit = made;
      slot += made;
      plan->merges.push_back(m);
    }
  }
  plan->num_partial_slots = slot;

  // Head dim 64, bf16 cache.  Many rows: there are two forms of the kernel, one that leaves room for
  // another 8-wave workgroup on its compute unit (a fourth 4-wave one) and one that runs 2-4 %
  // faster where there is none.  Two on a unit do about 1.15 times the work of one, but either
  // then runs at little more than half speed, and a long one that started late ends late.
  // Measured (us, plain / packed; 32/8 heads unless given).  Two workgroups per unit, items all
  // resident at once: their pairs are fixed and are compared with the plain form's packing --
  // 424 equal items 285 / 259, 512 equal 79.0 / 73.0, 512 of 31..108 tiles 185 / 190, 312 of 40..92
  // tiles 106 / 118.  More items than that are handed out as units fall free: 616 of up to 102
  // tiles, longest 1.4 times an even share 193 / 170, 660 (1.6 times; 4 heads, full misses) 108 /
  // 105, 592 (1.8 times) 98 / 101, 516 (2.0 times) 88 / 97.  Four waves: with up to three items per
  // unit the fourth place stays empty, 488..572 items 1-7 % slower packed; 950..1050 items 6-11 %
  // faster, 1280 equal.  (The short step chooses its number of stages at the same line.)
  if (b->head_dim == 64) {
    const size_t units = (size_t)std::max(1, M == 256 ? num_slots : num_slots / 2), n = pend.size();
    if (M != 256) {
      plan->crowded = n > 3 * units;
    } else if (n > units) {
      constexpr double kTwo = 1.15;
      std::vector<int64_t> cost;
      cost.reserve(n);
      int64_t total = 0;
      for (const Pending& p : pend) {
        cost.push_back(p.cost);
        total += p.cost;
      }
      std::sort(cost.begin(), cost.end(), std::greater<int64_t>());
      if (n > 2 * units) {
        plan->crowded = (double)cost[0] * (double)(2 * units) < 1.7 * (double)total;
      } else {
        double paired = 0;
        std::vector<int64_t> load(cost.begin(), cost.begin() + units);  // ends as a min-heap
        std::make_heap(load.begin(), load.end(), std::greater<int64_t>());
        for (size_t i = 0; i < units; ++i) {
          const double a = (double)cost[i], c = i + units < n ? (double)cost[i + units] : 0.0;
          paired = std::max(paired, 2.0 * c / kTwo + (a - c));
        }
        for (size_t i = units; i < n; ++i) {
          std::pop_heap(load.begin(), load.end(), std::greater<int64_t>());
          load.back() += cost[i];
          std::push_heap(load.begin(), load.end(), std::greater<int64_t>());
        }
        plan->crowded = paired < (double)*std::max_element(load.begin(), load.end());
      }
    }
  }

  // Order: heaviest first.  With XCD grouping, items that read the same K/V (same request and
  // kv head) are given workgroup ids congruent modulo 8, so they run on one XCD and share its
  // L2; the groups are spread over the 8 XCDs by greedy load balancing.
  constexpr int kXcds = 8;
  auto by_cost = [](const Pending& a, const Pending& c) { return a.cost > c.cost; };
  const int64_t ngroups = (int64_t)b->batch * b->num_kv_heads;
  bool group_xcd = tn.xcd_grouping && pend.size() >= (size_t)4 * kXcds;
  if (group_xcd) {
    // only worthwhile when several items share a group
    group_xcd = pend.size() > (size_t)tiles.size() || tiles.size() > (size_t)ngroups;
  }
  if (!group_xcd) {
    std::stable_sort(pend.begin(), pend.end(), by_cost);
    plan->items.reserve(pend.size());
    for (auto& p : pend) plan->items.push_back(p.w);
  } else {
    std::vector<int64_t> gcost(ngroups, 0), gmax(ngroups, 0);
    for (auto& p : pend) {
      gcost[p.group] += p.cost;
      gmax[p.group] = std::max<int64_t>(gmax[p.group], p.cost);
    }
    std::vector<int64_t> order(ngroups);
    for (int64_t i = 0; i < ngroups; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int64_t a, int64_t c) { return gcost[a] > gcost[c]; });
    std::vector<int> gx(ngroups, 0);
    int64_t load[kXcds] = {0};
    for (int64_t gi : order) {
      if (gcost[gi] == 0) continue;
      int best = 0;
      for (int x = 1; x < kXcds; ++x) if (load[x] < load[best]) best = x;
      gx[gi] = best;
      load[best] += gcost[gi];
    }
    // When a (request, kv head) pair has many query tiles (long new sequences), inside one XCD
    // the items run group after group (heaviest group first, and inside a group
    // heaviest item first): the workgroups resident at any time then read the K/V of only one
    // or two (request, kv head) pairs, which fits the 4 MB L2, instead of a slice of all of them.
    // With few query tiles per pair there is little to share and plain heaviest-first order
    // balances better, unless K/V are read twice and more and are larger than the 256 MB cache behind
    // the L2s (34 requests of 824..1782 + 203..512 tokens, 32/32 heads, 920 MB: 466 us heaviest first, 396 by
    // group; 10 requests of which three are full misses, the others one tile per pair: 113 / 117).
    int64_t live_groups = 0;
    for (int64_t gi = 0; gi < ngroups; ++gi) live_groups += gcost[gi] > 0;
    double tile_keys = 0.0;
    for (const Tile& t : tiles) tile_keys += t.key_end;
    const double pair_keys = keys * b->num_kv_heads;
    const bool group_major = (int64_t)tiles.size() >= 4 * std::max<int64_t>(1, live_groups) ||
                             (tile_keys >= 2.0 * pair_keys && pair_keys * 4.0 * D > 256.0 * (1 << 20));
    std::vector<Pending> per[kXcds];
    for (auto& p : pend) per[gx[p.group]].push_back(p);
    size_t longest = 0;
    for (int x = 0; x < kXcds; ++x) {
      if (!group_major) {
        std::stable_sort(per[x].begin(), per[x].end(), by_cost);
        longest = std::max(longest, per[x].size());
        continue;
      }
      // (groups by their LONGEST item first, then by their whole cost: a request with a long
      // cached context and few new rows is a light group of one or two very long items, and an
      // item of 120 key tiles that starts last is a tenth of the whole step on its own)
      std::stable_sort(per[x].begin(), per[x].end(), [&](const Pending& a, const Pending& c) {
        if (a.group != c.group) {
          if (gmax[a.group] != gmax[c.group]) return gmax[a.group] > gmax[c.group];
          if (gcost[a.group] != gcost[c.group]) return gcost[a.group] > gcost[c.group];
          return a.group < c.group;
        }
        return a.cost > c.cost;
      });
      longest = std::max(longest, per[x].size());
    }
    plan->items.reserve(longest * kXcds);
    const WorkItem nothing{0, 0, 0, 0, 0, 0, -1, -1};
    for (size_t k = 0; k < longest; ++k)
      for (int x = 0; x < kXcds; ++x) plan->items.push_back(k < per[x].size() ? per[x][k].w : nothing);
    while (!plan->items.empty() && plan->items.back().row_count == 0) plan->items.pop_back();
  }

  // Items past the ones that start at once can be drawn from a counter by the workgroups that start later (batch calls),
  // longest first, where no two read the same keys.  The dispatcher deals workgroups to the eight XCDs in turn,
  // the same number to each, but an XCD streams up to 10 % faster or slower than another (which ones
  // differs from one set of buffers to the next): bound by HBM, with the second half of the items dealt out, the
  // XCDs ended up to 19 us of 128 apart, drawn 5 of 119.  More workgroups draw than there are items, so that a
  // fast XCD can take more than its share; the others end at once.  us, dealt out / drawn: 16 requests of
  // 1024..4096 + 16..128 tokens, 32/32 heads 141.2 / 137.1; one new token, 46 of 2323..2785 keys 355 / 333, 19 of
  // 3158..10002 368 / 345.  Not where items share keys (28/4 heads, 8..64 new tokens: 117.4 / 122.2): they belong on one XCD.
  // Nor does it pay to cut ranges for it (28/4 heads, one new token, 496 items that all start at once: with a fifth
  // of every range as queued pieces of 6 tiles 69.3 / 71.2, 8-bit cache 34.8 / 38.6).  Head dim 64: twice as
  // many workgroups start at once (four waves: 328 items over codes 20.0 / 24.2 when half of them drew).
  plan->static_items = (int)plan->items.size();
  plan->queued_items = plan->draws = 0;
  int64_t pairs = 0;  // (request, kv head) pairs with work
  for (int r = 0; r < b->batch; ++r) pairs += b->new_len[r] > 0 ? b->num_kv_heads : 0;
  const size_t at_once = (size_t)num_slots * (D == 64 ? 2 : 1);
  plan->mean_tiles = pend.empty() ? 0 : (int)((total_cost - 4 * (int64_t)tiles.size()) / (int64_t)pend.size());
  if ((int64_t)tiles.size() == pairs && !plan->once && tn.xcd_grouping && plan->items.size() > at_once &&
      plan->mean_tiles >= kLongItems) {
    std::vector<WorkItem> rest(plan->items.begin() + at_once, plan->items.end());
    plan->items.resize(at_once);
    rest.erase(std::remove_if(rest.begin(), rest.end(), [](const WorkItem& w) { return w.row_count == 0; }), rest.end());
    std::stable_sort(rest.begin(), rest.end(), [](const WorkItem& a, const WorkItem& c) {
      return a.key_end - a.key_begin > c.key_end - c.key_begin;
    });
    plan->items.insert(plan->items.end(), rest.begin(), rest.end());
    plan->static_items = (int)at_once;
    plan->queued_items = (int)rest.size();
    plan->draws = (plan->queued_items * 3 / 2 + 15) / 8 * 8;
  }

  plan->max_item_rows = 0;
  for (const WorkItem& w : plan->items) plan->max_item_rows = std::max(plan->max_item_rows, (int)w.row_count);
  // Products of 16 rows where no item has more (measured at the kernel).  Not with row tile and ranges both
  // forced: a request of up to 16 rows then gives the same bits alone and beside one of up to 32.
  plan->rows16 = plan->max_item_rows <= 16 && !(tn.row_tile != 0 && tn.split_kv == 0);

  // Layout of the staged header and of the device workspace.
  size_t off = 0;
  plan->off_items = off;
  off = align_up(off + plan->items.size() * sizeof(DevItem), 256);
  plan->off_merges = off;
  off = align_up(off + plan->merges.size() * sizeof(MergeItem), 256);
  plan->header_bytes = off;
  // A partial-result slot holds as many rows as the largest work item has (in steps of 32), not
  // a whole row tile: decode-like steps cut every key range and have a handful of rows per item.
  plan->partial_rows = std::min(M, (plan->max_item_rows + 31) / 32 * 32);
  if (plan->partial_rows < 32) plan->partial_rows = 32;
  const size_t prows = (size_t)plan->partial_rows;
  off = 0;
  plan->off_part_o = off;
  // per row: D binary16 values, then (max, sum, scale, unused) as fp32
  off = align_up(off + (size_t)plan->num_partial_slots * prows * D * sizeof(uint16_t), 256);
  plan->off_part_ml = off;
  off = align_up(off + (size_t)plan->num_partial_slots * prows * 4 * sizeof(float), 256);
  plan->total_bytes = off < 256 ? 256 : off;  // never zero, so callers always pass a real buffer
}

}  // namespace

void build_plan(const efim_batch_t* b, int num_slots, Plan* plan, bool fp8) {
  const RowTile tile = choose_row_tile(b, num_slots);
  plan->fp8_rows_per_item = tile.fp8;
  build(b, num_slots, fp8 ? tile.fp8 : tile.bf16, plan);
  // 128 rows make up to twice the items and other cuts.  Where those outgrow what efim_extend_attention_static (bf16
  // only) holds and 256 rows do not, the step stays at 256: nothing that call takes there is refused.
  auto fits = [](const Plan& p) { return p.header_bytes <= kStaticListBytes && p.total_bytes <= kStaticPartialBytes; };
  if (fp8 || !tile.narrowed || fits(*plan) || tile.wide_tiles * sizeof(DevItem) > kStaticListBytes) return;
  Plan wide;
  wide.fp8_rows_per_item = tile.fp8;
  build(b, num_slots, 256, &wide);
  if (fits(wide)) *plan = std::move(wide);
}

}  // namespace efim
