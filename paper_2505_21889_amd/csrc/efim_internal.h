// Internal declarations shared by the translation units of libefim (host side).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <vector>

#include "efim.h"
#include "efim_debug.h"

namespace efim {

constexpr int kMinPageSize = 8;       // tokens per KV page: a power of two in this range
constexpr int kMaxPageSize = 256;
constexpr int kKeyTile = 64;          // keys staged in LDS per main-loop iteration
constexpr int kWavesPerGroup = 4;     // wavefronts per attention workgroup
// key tiles that the kernel which gathers a whole key range at the start of an item holds (128 KB of bf16 rows)
constexpr int once_tiles(int head_dim) { return head_dim == 128 ? 4 : 8; }
// and the most query rows of an item that it is launched for (reason at the planner's rule); one_call: the
// batch is one that the fused short step takes
constexpr int once_rows(int head_dim, bool one_call) { return head_dim == 128 && !one_call ? 16 : 32; }
constexpr int kMaxRowsPerItem = 256;  // largest query-row tile of one workgroup
constexpr int kStageSlots = 64;       // launch tokens in turn: a token comes round again after this many calls
constexpr int kTicketSlots = kStageSlots;
constexpr int kTicketsPerSlot = 8192; // split query tiles one launch can combine in-kernel, and (the last one) its queue

// log2 of the distance of a launch's arrival counters, in counters: 64 bytes while its block then holds them all in
// front of the queue's, else as far as it does.  Counters of one line are counted up one after another, from whatever
// XCD.  us, all counters of a launch in one line / in lines of their own: one new token, one request of 2344 keys,
// 32 layers 356.5 / 349.9, two of 4290 and 10819 keys, 28/4 heads 14.5 / 13.6, four of 4000..5000 over codes
// 15.7 / 14.6; as a plan object the first 345.0 / 337.5.  128 and 256 bytes are the same as 64.
inline int ticket_shift(size_t merges) {
  int shift = 4;
  while (shift > 0 && (merges << shift) >= (size_t)kTicketsPerSlot) --shift;
  return shift;
}

// Key tiles that the items of a launch have in the mean for its later ones to be drawn (reason at plan_draws).
constexpr int kLongItems = 28;

// Fixed device memory of efim_extend_attention_static: for the work list and for the partial results of split key ranges.
constexpr size_t kStaticListBytes = size_t(2) << 20;
constexpr size_t kStaticPartialBytes = size_t(30) << 20;

// Device-side view of one request.
struct ReqInfo {
  int32_t cached;     // C_r
  int32_t new_len;    // N_r
  int32_t row_start;  // first packed new-token row of the request
  int32_t pad;
};

// Work item as planned: identical fields to efim_work_item_t.
using WorkItem = efim_work_item_t;

// Work item as staged for the device: the planned fields plus what the kernel needs of the
// item's request, so that a workgroup starts with ONE read of the staged work list (the list
// lives in host memory, and every dependent read of it is a trip over the host link).
struct DevItem {
  WorkItem w;
  int32_t cached;     // C_r
  int32_t row_start;  // first packed new-token row of the request
  int32_t pad0, pad1;
};
static_assert(sizeof(DevItem) == 48, "three 16-byte reads");

// One query tile whose key range was split: `nsplit` partial results in consecutive slots.
struct MergeItem {
  int32_t req;
  int32_t kv_head;
  int32_t row_begin;
  int32_t row_count;
  int32_t first_slot;
  int32_t nsplit;
  int32_t row_start;  // first packed new-token row of the request
  int32_t pad1;
};

struct Tuning {
  hipEvent_t ev_start = nullptr;
  hipEvent_t ev_stop = nullptr;
  int split_kv = -1;
  int xcd_grouping = 1;
  int num_slots = 0;
  int row_tile = 0;  // 0 automatic, 128 or 256 forced
  int fused_merge = -1;  // split key ranges combined inside the main kernel: -1 when all items have few rows, 0 never, 1 always
  int device_plan = 1;   // repeated launches of a plan read the work list from a device-resident copy
};
Tuning& tuning();

struct Plan {
  uint64_t id = 0;          // distinct for every plan the cache has built
  int rows_per_item = 128;  // query rows per workgroup tile (32 per wave)
  int fp8_rows_per_item = 128;  // the same in the plan for 8-bit caches: all else equal, plans of one tile are
  int max_item_rows = 0;    // largest row_count of a work item
  int partial_rows = 128;   // rows per partial-result slot of a split key range
  bool once = false;        // few work items of few rows, each short enough for the kernel that gathers a whole range at once
  bool rows16 = false;      // key-parallel kernels: products of 16 rows instead of 32
  bool crowded = false;     // head dim 64: work items crowd the compute units (other forms of the bf16 kernels)
  std::vector<ReqInfo> reqs;
  std::vector<WorkItem> items;
  std::vector<MergeItem> merges;
  // The items from static_items on may be drawn by the workgroups that start later (0 queued items: none are), of
  // which `draws` are launched, more than there are items.  mean_tiles: key tiles of an item, in the mean.
  int static_items = 0, queued_items = 0, draws = 0, mean_tiles = 0;
  int64_t num_partial_slots = 0;
  // byte offsets of the items (as DevItem) and merges inside the staged plan header
  size_t off_items = 0, off_merges = 0, header_bytes = 0;
  // byte offsets of the split-KV partial results inside the device workspace, and its size
  size_t off_part_o = 0, off_part_ml = 0, total_bytes = 0;
};

// Number format of the paged caches: bf16, or E4M3 codes with one scale per tensor
// (value = code value * scale).
struct CacheFormat {
  bool fp8 = false;
  float k_scale = 1.f;
  float v_scale = 1.f;
};

// Validates the host-visible part of a batch. total_new receives T.
int validate_batch(const efim_batch_t* b, int64_t* total_new);

// Whether a launch with a counter draws the plan's queued items.  A draw costs a workgroup 1 to 1.5 us before it can
// start: 16..24 tiles per item 0.8-4.5 % slower drawn (17 requests of 714..1181 +
// 69..230 tokens, 32/32 heads 110 / 115 us), 28 and more 1-7.5 % faster (57 requests of 5319..16384 keys, one new
// token, 32/32 heads 1804 / 1669).  A tile of codes takes half the time, and so the line lies at twice the length there
// (45 requests of 3767..14730 + 8..16 in one call 633 / 617); with at most 16
// rows per item two workgroups share a unit over codes, start at once and gain nothing (27 requests of
// 1649..5713 keys, one new token, 175.2 / 179.0).
inline bool plan_draws(const Plan& plan, bool fp8) {
  return plan.queued_items > 0 && plan.mean_tiles >= (fp8 ? 2 : 1) * kLongItems && !(fp8 && plan.rows16);
}

// Builds the work list. num_slots = number of 4-wave workgroups the device runs concurrently; fp8: for 8-bit caches.
void build_plan(const efim_batch_t* b, int num_slots, Plan* plan, bool fp8 = false);

// Launch of the append kernel: x by y workgroups of 64 * parts << tok_shift threads; a workgroup has `parts` waves
// for each of 1 << tok_shift tokens, a wave kAppendPasses passes of 1024 / head_dim head rows.
constexpr int kAppendThreads = 256;
constexpr int kAppendPasses = 2;
struct AppendShape {
  unsigned x, y;
  int parts, tok_shift;
};
inline AppendShape append_shape(int64_t tokens, int rows, int head_dim) {
  // Usually a workgroup takes the same part of four tokens, and all tokens' first
  // parts go before their second ones.  A large step then reads and writes places far apart
  // at any time, and the workgroup takes all rows of a token (of two or four where a token has
  // two waves or one).  us, parts of four tokens / whole tokens: 28/4 heads of 128, 65536 tokens (604
  // MB) 234 / 216, 32768 106.9 / 105.9, 16384 47.2 / 46.0, 4096 13.3 / 14.5; 32/8 heads of 128, 65536 (805 MB) 299 /
  // 295, 16384 59.8 / 68.9, 2048 8.9 / 9.6; 32/8 heads of 64, 65536 (403 MB) 148 / 155, 32768 64.7 / 78.8.
  constexpr int64_t kWholeTokenBytes = (int64_t)1 << 29;
  constexpr int64_t kMostThreads = ((int64_t)1 << 32) - 1;  // of a launch along x
  const int per_wave = kAppendPasses * (1024 / head_dim);
  const int waves = (rows + per_wave - 1) / per_wave;  // per token
  auto groups_of = [&](int tok_shift) { return (tokens + (1 << tok_shift) - 1) >> tok_shift; };
  if (tokens * rows * head_dim * 2 >= kWholeTokenBytes) {
    const int y = (waves + kAppendThreads / 64 - 1) / (kAppendThreads / 64);
    const int parts = (waves + y - 1) / y;
    const int tok_shift = parts == 1 ? 2 : parts == 2 ? 1 : 0;
    if (groups_of(tok_shift) * (64 * parts << tok_shift) <= kMostThreads)
      return AppendShape{(unsigned)groups_of(tok_shift), (unsigned)y, parts, tok_shift};
  }
  return AppendShape{(unsigned)groups_of(2), (unsigned)waves, 1, 2};
}

// inv_freq: rotary_dim/2 host values; the leading rotary_dim elements of every head row rotate.
int launch_rope_append(const efim_batch_t* b, int64_t total_new, void* q, const void* k_new,
                       const void* v_new, void* k_cache, void* v_cache, const double* inv_freq,
                       int rotary_dim, int interleaved, const CacheFormat& fmt, hipStream_t stream);

// `header` is the device-visible address of the staged plan header (items, merges at
// the plan's offsets); `workspace` holds the split-KV partial results.
// `stage_slot` is the index of the call's launch token (0 .. kStageSlots-1): it selects the
// launch's block of arrival counters.  Negative: no token, split key ranges are combined by the
// second launch.
// `tickets` (optional): DEVICE arrival counters owned by the caller (one per split query tile, ticket_shift apart,
// zero between launches); given, the split key ranges are combined inside the main kernel with these counters and no launch token is needed.
// Without a token items follow the workgroup ids.  `quiet`: the timing hook is not served (a launch that may be
// under graph capture records no events).
int launch_extend_attention(const efim_batch_t* b, const Plan& plan, const char* header, int stage_slot,
                            const void* q, const void* k_cache, const void* v_cache, void* out,
                            float sm_scale, const CacheFormat& fmt, void* workspace, hipStream_t stream,
                            int32_t* tickets = nullptr, bool quiet = false);

// Fused short step (every request has 1 .. kFusedMaxTokens new tokens and at most kFusedMaxRows
// query rows per kv head; the decode step is the case of one token): one launch does the rotary
// embedding, the cache append, the attention and the merge of split key ranges.
// inv_freq / rotary_dim as for launch_rope_append.
constexpr int kFusedMaxRows = 32;    // query rows (new tokens x query heads per kv head) of one request and kv head
constexpr int kFusedMaxTokens = 16;  // new tokens of one request (their rotated K/V rows wait in LDS)
int launch_decode_step(const efim_batch_t* b, const Plan& plan, const char* header, int stage_slot,
                       const void* q, const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                       void* out, const double* inv_freq, int rotary_dim, int interleaved, float sm_scale,
                       const CacheFormat& fmt, void* workspace, hipStream_t stream, int32_t* tickets = nullptr,
                       bool quiet = false);

// Clears `count` 32-bit words at `words` with a kernel (a fill that a captured graph may hold).
int launch_zero_words(int32_t* words, size_t count, hipStream_t stream);

// Whether a plan's split key ranges are combined inside the main kernel (policy and knob).
bool plan_merges_in_kernel(const Plan& plan);

void set_last_hip_error(hipError_t e);

}  // namespace efim
