// efim_extend_attention: causal softmax attention of the new ("inc") tokens over the cached
// prefix+suffix pages plus themselves (EFIM Sec. 1: only the incremental part is computed,
// the rest of the reordered prompt is read from the KV cache).
//
// One workgroup (4 or 8 wavefronts, 32 query rows each) handles one work item: a tile of
// query rows of one (request, kv head) against a range of keys.  Rows are (token,
// head-in-group) pairs so all query heads that share a kv head read its K/V once.  Per
// 64-key tile:
//   * the tile's pages are gathered through the block table straight from HBM into LDS
//     (16 bytes per lane, 1 KB per wave instruction, XOR-swizzled 16-byte chunks), one or
//     two tiles ahead of the one being consumed;
//   * S^T = K Q^T with 32x32x16 bf16 MFMA: every lane ends up with 32 scores of ONE query
//     row, so its reference and sum are per-lane scalars plus one cross-half exchange;
//   * P is rounded to bf16 in registers and is directly the B operand of O^T += V^T P^T;
//     V^T operands come from the row-major V tile through the transposing LDS read;
//   * the three run as a pipeline over 32-key halves, each on another half at any time.
// Accumulation is fp32; partial results of split key ranges are merged by a second kernel or,
// for the decode step, by the workgroup that finishes last.
//
// 8-bit caches (E4M3 codes, one scale per tensor): the gather moves the codes (half the bytes).
// Both operands are read from the landed code tile as they are -- key codes eight at a time
// along the head dimension, value codes through the 8-bit transposing LDS read (eight keys of
// one head-dim element per lane) -- and converted to bf16 operands in registers.  The codes'
// values are exact in bf16; the key scale is folded into the softmax scale and the value
// scale into the final normalisation.
#include <cstddef>
#include <type_traits>

#include "efim_internal.h"
#include "fp8_math.h"
#include "rope_math.h"

namespace efim {
namespace {

// Arrival counters of split query tiles: the workgroup that finishes a tile's last part
// combines the parts.  One block of counters per work-list staging slot, so that launches in
// flight at the same time never share a counter; all zero whenever no launch is running
// (zero-initialised with the module, and the merging workgroup puts its counter back).
// (Aligned, so that which counters share a line does not follow from the size of the code in front of them.)
__device__ __align__(256) int32_t g_tickets[kTicketSlots * kTicketsPerSlot];

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) int i32x2;

#define LDS_PTR(T) __attribute__((address_space(3))) T*

struct AttnParams {
  uint16_t* out;
  // Partial result of one part of a split key range, per query row: the unnormalised output
  // row O as binary16 values O / a with a = max |O| over the row (half the bytes of fp32, on a
  // path that is bound by them; the row's own scale keeps any magnitude in range and the
  // relative error at 2^-11 of the row's largest element), and three fp32 values.
  uint16_t* part_o;  // [slot][rows_per_item][D] binary16 bits
  float* part_ml;    // [slot][rows_per_item][4] = (running max in log2 units, running sum, a, unused)
  int32_t num_q_heads;
  int32_t group;          // Hq / Hkv
  int32_t rows_per_item;  // rows of one partial-result slot
  float scale_log2;       // sm_scale * log2(e) (times the key scale of an 8-bit cache)
  float out_scale;        // 1, or the value scale of an 8-bit cache
  double k_inv;           // 8-bit caches, fused decode step: 1 / scale (code = value / scale)
  double v_inv;
  // --- fused decode step only (one new token per request) ---
  const uint16_t* k_new;  // [B, Hkv, D] raw keys of the new tokens
  const uint16_t* v_new;  // [B, Hkv, D]
  uint16_t* k_cache_w;    // the caches again, writable: the new token's K/V are appended
  uint16_t* v_cache_w;
  const MergeItem* merges;
  int32_t ticket_base;    // first arrival counter of this launch in g_tickets (or in `tickets`),
                          // or -1: the split key ranges are combined by merge_kernel in a second launch
  int32_t ticket_shift;   // counter of merge i: 2^ticket_shift * i behind the first
  int32_t* tickets;       // the caller's arrival counters, or nullptr: the library's own
  int32_t interleaved;    // rotary pairing
  int32_t rotary_dim;     // leading elements of a head row that are rotated
  double inv_freq[64];    // rotation frequency of pair j (rotary_dim / 2 entries)
  int32_t queue_at;       // the counter of drawn items, in g_tickets
  int32_t queued_items;   // items from static_items on are drawn from the queue
  int32_t draws;          // workgroups that draw
};

// The kernel's arguments as they lie in its argument block: each where a struct of them would have it.  The launch
// checks that the kernel's parameters are these.
struct KernelArgs {
  const DevItem* items;
  const int32_t* block_table;
  const uint16_t* q_rows;
  const uint16_t* k_pages;
  const uint16_t* v_pages;
  int32_t max_pages;     // columns of the block table
  int32_t kv_heads;
  int32_t shape;         // heads per group, from bit 8 on the log2 of the page size (tokens per page)
  int32_t static_items;  // the workgroup's item is its id below this
  AttnParams p;
};
constexpr int kFreqAt = offsetof(KernelArgs, p) + offsetof(AttnParams, inv_freq);
static_assert(std::is_standard_layout<KernelArgs>::value && kFreqAt % 4 == 0, "read with 16-byte loads of aligned words");

constexpr float kSlack = 8.f;  // log2 units by which a row max may outgrow its reference

// Plain nested maxima: the compiler turns them into three-operand max instructions itself and,
// unlike for hand-written assembly, inserts the wait states a read of fresh MFMA results needs.
// Sum of sixteen bf16 probabilities (as rounded for the PV product, so the normaliser matches the
// weights the product uses): two-element dot products with ones, one instruction per pair.
__device__ __forceinline__ float sum_pairs(bf16x8 a, bf16x8 b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  float acc = 0.f;
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 0, 1), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 2, 3), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 4, 5), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 6, 7), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 0, 1), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 2, 3), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 4, 5), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(b, b, 6, 7), ones, acc, false);
  return acc;
}

__device__ __forceinline__ float max3(float a, float b, float c) {
  return __builtin_fmaxf(__builtin_fmaxf(a, b), c);
}

// max / sum of a value with the one held by the lane 32 positions away (the two halves of a
// wave hold the two key halves of the same query row): one lane-swap instruction instead of
// a round trip through the LDS crossbar.
__device__ __forceinline__ float cross_half_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// the same between neighbouring quarters (16 lanes) of a wave
__device__ __forceinline__ float cross_quarter_max(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float cross_quarter_sum(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float cross_half_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Maximum over N (16 or 32) neighbouring lanes, in all of them.
template <int N>
__device__ __forceinline__ float row_lanes_max(float v) {
  auto with = [&](auto ctrl) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v = fmaxf(v, with(std::integral_constant<int, 0xB1>{}));   // quad_perm [1, 0, 3, 2]
  v = fmaxf(v, with(std::integral_constant<int, 0x4E>{}));   // quad_perm [2, 3, 0, 1]
  v = fmaxf(v, with(std::integral_constant<int, 0x141>{}));  // row_half_mirror
  v = fmaxf(v, with(std::integral_constant<int, 0x140>{}));  // row_mirror
  if constexpr (N == 32) v = cross_quarter_max(v);
  return v;
}

// Direct HBM -> LDS copy of 16 bytes per lane: lane l's data lands at lds_addr + 16 * l
// (lds_addr, the wave-uniform LDS byte address, travels in M0).  Issued as inline assembly so that the
// compiler does not order LDS reads of OTHER buffers behind it; completion is awaited
// explicitly with s_waitcnt vmcnt before the workgroup barrier that publishes the buffer.
// M0 is a reserved register that cannot be named as a clobber, so every block puts back the
// value it found: whatever the compiler keeps in M0 around the block survives it.
__device__ __forceinline__ void load_to_lds_16(const void* gptr, uint32_t lds_addr) {
  uint32_t saved_m0;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %2, off\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved_m0)
      : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(gptr)
      : "memory");
}

// The same with the address split into a wave-uniform base (scalar registers) and a 32-bit
// per-lane offset: no vector arithmetic on 64-bit addresses in front of the load.
__device__ __forceinline__ void load_to_lds_16(const void* base, uint32_t lane_off, uint32_t lds_addr) {
  uint32_t saved_m0;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %2, %3\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved_m0)
      : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(lane_off), "s"(base)
      : "memory");
}

// Four such loads of consecutive 1 KB pieces: the instruction's offset field moves both the
// global address and the LDS address, so one base and one M0 serve all four.
__device__ __forceinline__ void load_to_lds_4x16(const void* base, uint32_t off0, uint32_t off1, uint32_t off2,
                                                 uint32_t off3, uint32_t lds_addr) {
  uint32_t saved_m0;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %2, %6\n\t"
      "global_load_lds_dwordx4 %3, %6 offset:1024\n\t"
      "global_load_lds_dwordx4 %4, %6 offset:2048\n\t"
      "global_load_lds_dwordx4 %5, %6 offset:3072\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved_m0)
      : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(off0), "v"(off1), "v"(off2), "v"(off3), "s"(base)
      : "memory");
}

__device__ __forceinline__ void load_to_lds_2x16(const void* base, uint32_t off0, uint32_t off1, uint32_t lds_addr) {
  uint32_t saved_m0;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %2, %4\n\t"
      "global_load_lds_dwordx4 %3, %4 offset:1024\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved_m0)
      : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(off0), "v"(off1), "s"(base)
      : "memory");
}

template <int D>
struct Geometry {
  static constexpr int kRowBytes = D * 2;            // one key/value row
  static constexpr int kChunks = D / 8;              // 16-byte chunks per row
  static constexpr int kSteps = D / 16;              // MFMA k-steps over the head dimension
  static constexpr int kDBlocks = D / 32;            // 32-wide blocks of the head dimension
  static constexpr int kTileBytes = kKeyTile * kRowBytes;
  static constexpr int kKeysPerLoad = 1024 / kRowBytes;      // keys moved by one 1 KB wave load
  static constexpr int kLoadsPerMatrix = kTileBytes / 1024;  // wave loads per K (or V) tile
  // chunk swizzles (XOR masks) that spread the K rows read by ds_read_b128 and the V rows
  // read by the transposing read over the LDS banks
  __device__ static int kswz(int row) { return row & (kChunks - 1); }
  __device__ static int vswz(int row) { return (row & (kChunks / 4 - 1)) << 2; }
};

// Two floats as one 8-byte access that is coherent across the whole device.
__device__ __forceinline__ void store_coherent(float* at, float a, float b) {
  const uint64_t bits = (uint64_t)__float_as_uint(a) | ((uint64_t)__float_as_uint(b) << 32);
  __hip_atomic_store(reinterpret_cast<uint64_t*>(at), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_coherent_bits(void* at, uint64_t bits) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(at), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t load_coherent_bits(const void* at) {
  return __hip_atomic_load(reinterpret_cast<const uint64_t*>(at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void load_coherent(const float* at, float* a, float* b) {
  const uint64_t bits = __hip_atomic_load(reinterpret_cast<const uint64_t*>(at), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
  *a = __uint_as_float((uint32_t)bits);
  *b = __uint_as_float((uint32_t)(bits >> 32));
}

// Combines the partial results of a split key range: with M = max_s m_s and
// w_s = 2^(m_s - M):  out = sum_s w_s O_s / sum_s w_s l_s, splits taken in index order
// (O_s = a_s h_s, h_s the stored binary16 row).
// nthreads threads (thread index t) share rows [row_lo, row_hi) of the tile, D/8 threads per
// row with 16 bytes of each part.  The splits are taken GROUP at a time with all their loads issued
// together (one memory round trip per group instead of one per split); a later group rescales
// the running sums.  GROUP does not change the bits of a result as long as it holds all splits.
// COHERENT: the partial results were written by other workgroups of the same launch.
template <int D, int GROUP, bool COHERENT>
__device__ __forceinline__ void merge_rows(const AttnParams& p, const MergeItem& mi, int t,
                                           int nthreads, int row_lo = 0, int row_hi = 1 << 30) {
  typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
  constexpr int E4 = COHERENT ? 1 : 2;  // groups of four elements per thread
  constexpr int VEC = D / (4 * E4);     // threads per row
  const int dv = (t % VEC) * 4 * E4;
  const int g = p.group;
  row_hi = min(row_hi, mi.row_count);
  for (int lr = row_lo + t / VEC; lr < row_hi; lr += nthreads / VEC) {
    float mx = -INFINITY, l = 0.f;
    f32x4 acc[E4];
#pragma unroll
    for (int e = 0; e < E4; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < mi.nsplit; s0 += GROUP) {
      float m[GROUP], ls[GROUP], amax[GROUP];
      uint64_t h[GROUP][E4];
#pragma unroll
      for (int i = 0; i < GROUP; ++i) {
        // splits past the end re-read the last one and get weight zero
        const int s = min(s0 + i, mi.nsplit - 1);
        const int64_t prow = (int64_t)(mi.first_slot + s) * p.rows_per_item + lr;
        if constexpr (COHERENT) {
          float unused;
          load_coherent(p.part_ml + prow * 4, &m[i], &ls[i]);
          load_coherent(p.part_ml + prow * 4 + 2, &amax[i], &unused);
          h[i][0] = load_coherent_bits(p.part_o + prow * D + dv);
        } else {
          const f32x4 mla = *reinterpret_cast<const f32x4*>(p.part_ml + prow * 4);
          m[i] = mla[0];
          ls[i] = mla[1];
          amax[i] = mla[2];
          const u32x4 both = *reinterpret_cast<const u32x4*>(p.part_o + prow * D + dv);
          h[i][0] = (uint64_t)both[0] | ((uint64_t)both[1] << 32);
          h[i][E4 - 1] = (uint64_t)both[2] | ((uint64_t)both[3] << 32);
        }
      }
      float gmx = mx;
#pragma unroll
      for (int i = 0; i < GROUP; ++i) gmx = fmaxf(gmx, m[i]);
      if (s0 > 0) {
        const float back = __builtin_amdgcn_exp2f(mx - gmx);
        l *= back;
#pragma unroll
        for (int e = 0; e < E4; ++e) acc[e] *= back;
      }
      mx = gmx;
#pragma unroll
      for (int i = 0; i < GROUP; ++i) {
        const float w = (s0 + i < mi.nsplit) ? __builtin_amdgcn_exp2f(m[i] - mx) : 0.f;
        // (explicit: left to itself the compiler fused the rescale into the addition in one of the
        // two merges, whose results then differed in the last bit past eight parts)
        l = fmaf(w, ls[i], l);
        const float wa = w * amax[i];
#pragma unroll
        for (int e = 0; e < E4; ++e) {
          const f16x4 hv = __builtin_bit_cast(f16x4, h[i][e]);
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[e][k] = fmaf((float)hv[k], wa, acc[e][k]);
        }
      }
    }
    const float inv = p.out_scale / l;
    const int row = mi.row_begin + lr;
    const int tok = row / g;
    const int hg = row - tok * g;
    uint16_t* dst = p.out + ((int64_t)(mi.row_start + tok) * p.num_q_heads + mi.kv_head * g + hg) * D + dv;
    u32x2 words[E4];
#pragma unroll
    for (int e = 0; e < E4; ++e) {
      bf16x4 o4;
#pragma unroll
      for (int i = 0; i < 4; ++i) o4[i] = (__bf16)(acc[e][i] * inv);
      words[e] = __builtin_bit_cast(u32x2, o4);
    }
    if constexpr (E4 == 1) *reinterpret_cast<u32x2*>(dst) = words[0];
    else *reinterpret_cast<u32x4*>(dst) = u32x4{words[0][0], words[0][1], words[1][0], words[1][1]};
  }
}

// The next queued item for this workgroup, or -1: none is left.  The last of the launch's draws puts the counter back.
__device__ __forceinline__ int draw_item(const AttnParams& p, int static_items, int* s_draw) {
  if (threadIdx.x == 0) {
    int32_t* queue = g_tickets + p.queue_at;
    const int n = __hip_atomic_fetch_add(queue, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n == p.draws - 1) __hip_atomic_store(queue, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_draw = n;
  }
  __syncthreads();
  const int n = __builtin_amdgcn_readfirstlane(*s_draw);
  __syncthreads();  // (the word is part of a tile buffer)
  return n < p.queued_items ? static_items + n : -1;
}

// WAVES wavefronts per workgroup, 32 query rows each; STAGES LDS buffers of one 64-key K/V
// tile each.  Launched are
//   <4 waves, 2 stages>  128 rows, 64 KB LDS with head dim 128, two workgroups per compute unit, which cover each
//                        other's start and end; three stages where a tile is half as large (8-bit caches;
//                        the short step with head dim 64 and many work items);
//   <8 waves, 3 stages>  256 rows, 96 KB LDS with head dim 128, one workgroup per compute unit: each gathered
//                        K/V byte is used by twice as many rows and the gather runs two tiles ahead.
// The planner's rule of the row tile chooses.
//
// FUSED (decode step and other short steps: every request has at most kFusedMaxTokens new
// tokens and at most 32 query rows per kv head, so all rows of a (request, kv head) pair are
// one tile): the kernel also does what efim_rope_append does for those tokens -- q is rotated
// on the way in (global q stays raw); every workgroup rotates the new keys of its pair, patches
// those that fall into its key range into its LDS tiles and stores them, with their values,
// into the paged cache.
//
// KV8: the caches hold E4M3 codes.  The stages then hold code tiles (half the size); the rings
// have three of them in all configurations -- more tiles in flight measured slower, not faster.
//
// KP ("key parallel"): every work item of the launch has at most 32 query rows (decode steps,
// short increments).  One wave would be busy and the others idle: instead waves 0 and 1 (ONCE: all
// eight, in pairs) take all the rows and one 32-key half of a key tile each, with their own running
// max and sums, and their partial results are combined through LDS at the end.  In the four-wave
// kernel the two waves without rows issue all the gathers.
//
// Head dim 64, few rows: a few registers less than the compiler takes by itself let two 8-wave (or
// four 4-wave) workgroups share a compute unit instead of one (or three), without a spill.  The
// same kernel without and with the bound: 64 requests of 4000..7000 + 1..8 tokens, 32/8 heads, one
// launch 143.7 / 137.1 us, 24 requests of 2000..7000 + 4..8 tokens, two calls 47.1 / 42.5 us.
//
// PACK (head dim 64, bf16 cache, many rows): the same for the pipelined kernel, whose plain form
// takes 149 registers (four waves: 151).  With the value product in front of the score product in
// every phase, two key operands in flight instead of four and operand addresses derived from one
// register each it fits 128 without a spill.  Either form does the same arithmetic; Plan::crowded
// chooses.
constexpr int waves_per_simd(int d, int waves, bool fused, bool kv8, bool kp, bool pack) {
  return pack || (d == 64 && kp && !kv8 && (!fused || waves == 8)) ? 4 : 2;
}
//
// P8: 64-byte code rows on pages of 8, the one layout whose 1 KB load spans two pages.
//
// ONCE (key parallel, eight waves): for launches with at most one work item per compute unit, whose
// ranges fit the tile buffers whole (Plan::once).  Such a launch is bound by latency: with a ring
// of two or three buffers and two waves at work the tiles of an item pass one behind the other at
// 0.8 us each.  Here all of them are gathered at the start, each pair of waves takes tiles of its own,
// and the eight waves' sums are combined at the end.  One request of 1000 keys, 32/8 heads 12.2 -> 10.4
// us, 16 requests of 250 keys 10.2 -> 8.2 us, four requests of 300 + 32 tokens, 4 heads of 64, two
// calls 16.8 -> 11.2 us.  An item takes 128 to 160 KB of LDS over bf16 rows (64 to 138 KB over codes), so
// launches on two streams share the device only while their items together are no more than the
// units: two at once, one stream after the other / both, 2 x 64 items 8.3 + 8.3 / 9.5 us, 2 x 128
// 10.8 + 10.8 / 11.8, 2 x 256 10.4 + 11.1 / 17.8 (on the ring 13.7 + 14.8 / 17.3).
//
// R16 (key parallel, no item has more than 16 query rows): products of 16 keys by 16 rows instead of 32 by
// 32.  A 32 x 32 product over one to seven rows spends most of its time, of the softmax and of the
// accumulators on columns that are no rows, and a short step is bound by that chain: one request
// of 2344 keys, 32/8 heads 11.9 -> 11.2 us, 20 requests of 500..3000 keys, 32/32 heads 124.6 -> 118.4 us, 24
// drawn steps 3.4 % in the mean, none slower.  With 17 to 32 rows it would take two column blocks.
template <int D, int WAVES, int STAGES, bool FUSED, bool KV8, bool KP, bool PACK = false, bool P8 = false, bool ONCE = false, bool R16 = false>
__global__ __launch_bounds__(64 * WAVES, ONCE ? 2 : waves_per_simd(D, WAVES, FUSED, KV8, KP, PACK)) void extend_attention_kernel(
    const DevItem* items, const int32_t* block_table, const uint16_t* q_rows, const uint16_t* k_pages, const uint16_t* v_pages,
    const int32_t max_pages, const int32_t kv_heads, const int32_t shape, const int32_t static_items, const AttnParams p) {
  const int g = shape & 0xFF, ps = shape >> 8;  // heads per group (at most 64), log2 of the page size
  static_assert(!ONCE || (KP && WAVES == 8 && STAGES == once_tiles(D) && !P8), "the form for few work items");
  static_assert(!PACK || (D == 64 && !KV8 && !KP), "the packed form is for head dim 64, bf16, many rows");
  static_assert(!P8 || (D == 64 && KV8), "other rows are longer");
  static_assert(KP || !R16, "16 rows are one tile of the key-parallel kernels");
  static_assert(KP || !FUSED, "the decode step has at most 32 rows per tile");
  using G = Geometry<D>;
  // geometry of the gather: rows as they lie in the cache
  constexpr int kGRowBytes = KV8 ? D : 2 * D;
  constexpr int kGChunks = kGRowBytes / 16;
  constexpr int kGTileBytes = kKeyTile * kGRowBytes;
  constexpr int kGKeysPerLoad = 1024 / kGRowBytes;      // keys moved by one 1 KB wave load
  constexpr int kGLoadsPerMatrix = kGTileBytes / 1024;  // wave loads per K (or V) tile
  constexpr int kStageBytes = 2 * kGTileBytes;
  // Buffer s of the ring: K tile at s * kSlotBytes, V tile kVOff behind it.  The pipelined kernels
  // keep all K tiles in front of all V tiles, so that each matrix's buffers lie within the 64 KB
  // that the offset field of an LDS read reaches.
  constexpr int kSlotBytes = KP ? kStageBytes : kGTileBytes;
  constexpr int kVOff = KP ? kGTileBytes : STAGES * kGTileBytes;
  // chunk swizzles of code rows.  Keys: the 8-byte operand reads of 32 consecutive keys spread
  // over all banks.  Values: a 16-lane block of the transposing read touches keys
  // {0..3, 8..11} (or {4..7, 12..15}) of a 16-key group at one 16-byte chunk; bits 0, 1 and 3
  // of the key (D = 128; bits 1 and 3 for the 64-byte rows of D = 64, where two rows share a
  // bank cycle) tell those eight rows apart.
  auto kswz8 = [](int row) { return D == 128 ? (row & 7) : ((row >> 1) & 3); };
  // R16: the block's rows are {0..3, 16..19} + 4 * block, two blocks at a time.
  auto vswz8 = [](int row) {
    if constexpr (R16) return D == 128 ? (((row >> 1) & 3) | (((row >> 4) & 1) << 2)) : (((row >> 2) & 1) | (((row >> 4) & 1) << 1));
    return D == 128 ? ((row & 3) | (((row >> 3) & 1) << 2)) : (((row >> 1) & 1) | (((row >> 3) & 1) << 1));
  };
  // bf16 value rows.  R16: two blocks of four keys at one 32-byte piece are read together
  auto vswz16 = [](int row) { return R16 && D == 128 ? G::vswz(row) ^ (((row >> 2) & 1) << 1) : G::vswz(row); };
  // fused step: the rotated query rows of the tile, then per new token its rotated key and its
  // value as they go into the cache (bf16 rows or code rows) -- behind the tile buffers.  With
  // D = 128 that is 16 KB: two 4-wave workgroups with their 64 KB of tile buffers fill the 160 KB
  // of a compute unit exactly.
  constexpr int kFusedRows = 32;
  constexpr int kTileBufBytes = STAGES * kStageBytes;
  // (8-bit caches: the raw bf16 rows of the new tokens have an area of their own behind that)
  constexpr int kFusedRawBytes = FUSED && KV8 ? kFusedMaxTokens * 2 * 2 * D : 0;
  constexpr int kFusedBytes = FUSED ? kFusedRows * D * 2 + kFusedMaxTokens * 2 * kGRowBytes + kFusedRawBytes : 0;
  // cosines and sines of the new tokens' positions: in the tile buffer that is filled last, or, where
  // all are filled at the start, behind everything else
  constexpr int kTableBytes = FUSED && ONCE ? kFusedMaxTokens * (D / 2) * 16 : 0;
  // key-parallel kernels: where the waves that share the rows leave their sums at the end
  constexpr int kSharers = ONCE ? WAVES : 2;
  constexpr int kMaxRows = R16 ? 16 : 32;
  constexpr int kPitch = D + 4;  // floats from row to row: 16 bytes on, so that 16 rows spread over all banks
  constexpr int kExchangeBytes = KP ? kSharers * kMaxRows * (kPitch + 3) * 4 : 0;
  constexpr int kBufBytes = kTileBufBytes + kFusedBytes + kTableBytes;
  constexpr int kLdsBytes = kBufBytes > kExchangeBytes ? kBufBytes : kExchangeBytes;
  static_assert(STAGES >= 2 && kLdsBytes <= 160 * 1024, "stages must fit the 160 KB LDS");
  // One array, carved by hand.
  __shared__ __attribute__((aligned(1024))) char lds[kLdsBytes];
  char* const stages = lds;
  uint16_t* const s_q = reinterpret_cast<uint16_t*>(lds + kTileBufBytes);
  char* const s_kv = reinterpret_cast<char*>(s_q + kFusedRows * D);  // token j: key row at j * 2 * kGRowBytes, value row behind it
  // raw bf16 rows of the new tokens, key and value row of token j at 2 * j and 2 * j + 1; bf16
  // caches: the same place, rotated where they lie
  uint16_t* const s_raw = reinterpret_cast<uint16_t*>(KV8 ? s_kv + kFusedMaxTokens * 2 * kGRowBytes : s_kv);
  // the "this workgroup merges" flag is only used once the tile buffers are dead
  int* const s_last = reinterpret_cast<int*>(lds);

  // Fused step: the rotation frequency of this thread's pair (thread = (token, pair)), read in the shadow of the work
  // item's load -- behind the gathers it would wait for them.  ONCE: the frequencies go straight from the kernel's
  // arguments to LDS, a copy for each wave, where this wave will put its first tokens' cosines and sines: with one
  // item per compute unit nothing covers the wait for the register, which the compiler puts behind the item.  With
  // many items per unit it is the copies that cost: one new token, 300 requests of 200..400 keys, 32/8 heads 96.8 us
  // with them and 95.3 without, head dim 64 47.2 / 46.3, 298 such over codes 41.1 / 39.4.
  char* const s_table = ONCE ? lds + kTileBufBytes + kFusedBytes : lds + (STAGES - 1) * kStageBytes;
  char* const s_freq = s_table + (threadIdx.x >> 6) * 1024;
  double inv_freq = 0.0;
  if constexpr (FUSED && !ONCE) inv_freq = p.inv_freq[threadIdx.x % (D / 2)];
  if constexpr (FUSED && ONCE) {
    typedef const __attribute__((address_space(4))) char* ArgPtr;
    const ArgPtr freq = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr() + kFreqAt;
    load_to_lds_16((const void*)(uintptr_t)freq, (threadIdx.x & 31u) * 16u, (uint32_t)(uintptr_t)(LDS_PTR(char))s_freq);
  }

  int index = blockIdx.x;
  if constexpr (!ONCE) {  // (there all items start at once)
    if (index >= static_items) {
      index = draw_item(p, static_items, reinterpret_cast<int*>(lds));
      if (index < 0) return;
    }
  }
  const DevItem staged = items[index];
  const WorkItem it = staged.w;
  // (asked for together with the work item, not one after another where they are used)
  if constexpr (FUSED) asm volatile("" ::"s"(p.k_new), "s"(p.v_new), "s"(p.rotary_dim), "s"(p.interleaved));
  asm volatile("" ::"s"(p.num_q_heads), "s"(p.out), "s"(p.part_o), "s"(p.scale_log2), "s"(it.row_count), "s"(staged.cached));
  if (it.row_count == 0) {
    if constexpr (FUSED && ONCE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load into LDS outlives the workgroup
    return;
  }
  struct { int32_t cached, row_start; } rq;
  rq.cached = staged.cached;
  rq.row_start = staged.row_start;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i32 = lane & 31;
  const int hi = lane >> 5;

  const int wave_row0 = KP ? 0 : wave * 32;

  // --- this lane's query row (column of S^T / O^T) ----------------------------------
  const int i16 = lane & 15;
  const int q4 = lane >> 4;
  const int local_row = R16 ? i16 : wave_row0 + i32;
  const bool row_ok = local_row < it.row_count;
  const int row = it.row_begin + local_row;
  const int tok = row / g;
  const int head_in_group = row - tok * g;
  const int n_vis = row_ok ? rq.cached + tok + 1 : 0;  // keys visible to this row
  const int64_t q_off =
      ((int64_t)(rq.row_start + tok) * p.num_q_heads + it.kv_head * g + head_in_group) * D;

  const bool wave_active = wave_row0 < it.row_count;
  const int wave_first_row = it.row_begin + wave_row0;
  const int wave_last_row = it.row_begin + min(it.row_count, wave_row0 + 32) - 1;
  const int wave_min_vis = rq.cached + wave_first_row / g + 1;
  const int wave_max_vis = rq.cached + wave_last_row / g + 1;

  // MFMA B operands of this lane's query row: read here for the plain kernel, after the first
  // gathers have been issued for the fused one (the rotation then overlaps their latency)
  constexpr int kQSteps = R16 ? D / 32 : G::kSteps;  // MFMA steps over the head dimension
  const int q_at = R16 ? 8 * q4 : 8 * hi;            // this lane's eight elements of a step
  bf16x8 qb[kQSteps];
  if constexpr (!FUSED) {
#pragma unroll
    for (int s = 0; s < kQSteps; ++s) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (row_ok) v = *reinterpret_cast<const u32x4*>(q_rows + q_off + (D / kQSteps) * s + q_at);
      qb[s] = __builtin_bit_cast(bf16x8, v);
    }
  }

  f32x16 o[G::kDBlocks];
#pragma unroll
  for (int d = 0; d < G::kDBlocks; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
  f32x4 o16[D / 16];        // R16: head-dim blocks of 16 instead
#pragma unroll
  for (int d = 0; d < D / 16; ++d) o16[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY;  // reference max of the scaled scores (log2 units)
  float l_run = 0.f;        // this lane's share of the running sum

  const int k_begin = it.key_begin;
  const int k_end = it.key_end;
  const int ntiles = (k_end - k_begin + kKeyTile - 1) / kKeyTile;
  const int32_t* bt = block_table + (int64_t)it.req * max_pages;
  const int page_mask = (1 << ps) - 1;
  const int last_page = (k_end - 1) >> ps;

  // Page ids come from the block table through SCALAR loads (constant address space, wave
  // uniform index): they wait on their own counter.  A vector load of page ids inside the tile
  // loop would make the compiler put an s_waitcnt vmcnt(0) in front of its use -- it cannot see
  // how many of the hand-issued gathers are still in flight -- and that wait drains every tile
  // the loop means to keep in flight.
  const int first_page = k_begin >> ps;
  const int first_off = k_begin & page_mask;  // nonzero only for pages larger than a tile
  const auto* btc = (const __attribute__((address_space(4))) int32_t*)(uintptr_t)bt;
  // page id of the page that holds key (k_begin - first_off + rel), rel wave-uniform
  auto page_of = [&](int rel) -> uint32_t {
    return (uint32_t)btc[__builtin_amdgcn_readfirstlane(min(first_page + (rel >> ps), last_page))];
  };
  const int64_t page_bytes = ((int64_t)kv_heads * kGRowBytes) << ps;
  const int64_t head_bytes = ((int64_t)it.kv_head * kGRowBytes) << ps;
  const bool offsets_fit_32 = page_bytes < ((int64_t)1 << 32);  // offsets inside a page, that is
  const int page_loads = (1 << ps) / kGKeysPerLoad;  // 1 KB loads that one page of one head holds
  // Rows of a tile past the end of the key range are fetched from the last key of the range
  // instead: every tile then issues the same number of loads, pages that may not exist are
  // never touched, and LDS only ever holds finite data (the scores of those rows are masked).
  const int64_t last_off = (int64_t)btc[__builtin_amdgcn_readfirstlane(last_page)] * page_bytes + head_bytes +
                           ((k_end - 1) & page_mask) * kGRowBytes;
  // The query loads stay in flight while the first tiles are gathered (the two latencies pass
  // together); they are awaited, with those gathers, in front of the main loop.

  // --- gather of one 64-key tile: the 2 * kLoadsPerMatrix 1 KB loads are dealt to the waves.
  // In the four-wave key-parallel kernel waves 0 and 1 do the products and waves 2 and 3, which
  // have no rows, issue all the loads: per tile the two jobs then overlap instead of adding up.
  constexpr bool kSplitRoles = KP && WAVES == 4;
  constexpr int kIssuers = kSplitRoles ? 2 : WAVES;
  constexpr int kLoadsPerWave = 2 * kGLoadsPerMatrix / kIssuers;
  static_assert(kLoadsPerWave * kIssuers == 2 * kGLoadsPerMatrix, "loads must divide evenly");
  const int issuer = kSplitRoles ? wave - 2 : wave;  // negative: this wave issues no loads
  const int g_key = lane / kGChunks;  // key within one 1 KB load
  const int g_pc = lane % kGChunks;   // physical 16-byte chunk this lane fills
  // LDS byte address of the tile buffers (kept as an integer: the loads take addresses, not
  // pointers)
  const uint32_t lds0 = (uint32_t)(uintptr_t)(LDS_PTR(char))lds;
  // Page ids of this wave's groups of four loads of tile t, fetched ahead of the loop-top wait so
  // that the scalar loads' latency passes behind the barrier.
  constexpr int kGroups4 = kLoadsPerWave % 4 == 0 ? kLoadsPerWave / 4 : 1;
  struct TilePages { uint32_t id[kGroups4]; };
  auto fetch_pages = [&](int t) -> TilePages {
    TilePages tp;
    const int load0 = issuer < 0 ? 0 : issuer * kLoadsPerWave;
    const int idx0 = load0 >= kGLoadsPerMatrix ? load0 - kGLoadsPerMatrix : load0;
#pragma unroll
    for (int g4 = 0; g4 < kGroups4; ++g4) tp.id[g4] = page_of(first_off + t * kKeyTile + (idx0 + 4 * g4) * kGKeysPerLoad);
    return tp;
  };
  auto issue_tile = [&](int t, int stage, const TilePages& pages) {
    if (issuer < 0) return;
    const uint32_t kbuf = lds0 + stage * kSlotBytes;
    const uint32_t vbuf = kbuf + kVOff;
    const int key0 = k_begin + t * kKeyTile;
    const bool full_tile = key0 + kKeyTile <= k_end;  // no row of the tile lies past the key range
    const char* kc = reinterpret_cast<const char*>(k_pages);
    const char* vc = reinterpret_cast<const char*>(v_pages);
    // (not in the eight-wave key-parallel kernel over bf16 caches: measured 1.5-2.5 % slower there
    // -- that kernel is bound by HBM alone, and its loads do better spaced out)
    constexpr bool kGroupedIssue = !(KP && WAVES == 8 && !KV8) || ONCE;
    // The key-parallel kernels of the plain call and ONCE take the last tile of a range the same way: through
    // the general path below they wait for a page lookup in front of each load, one behind the
    // other (one request of 256 + 32 tokens, 4 heads: 7.7 -> 7.2 us).  The other kernels have
    // no registers for it (the decode step's ring spilled: 13.3 -> 13.7 us) or longer ranges.
    constexpr bool kGroupedLast = KP && (!FUSED || ONCE);
    // P8: both page ids of a load come by scalar loads, all of the wave's together, and a lane picks
    // its page's; looked up lane by lane the ids wait on the counter of the gathers and drain the
    // tiles in flight.  64 requests of 4000..7000 + 1..8 tokens, 32/8 heads 116.3 -> 97.5 us.  (A
    // kernel of its own: as a branch it cost the larger pages 1-3 %.)
    if constexpr (P8) {
      static_assert(kGKeysPerLoad == 2 * kMinPageSize && kGLoadsPerMatrix % kLoadsPerWave == 0,
                    "two pages per load, one matrix per wave");
      if (full_tile && offsets_fit_32) {
        const int load0 = issuer * kLoadsPerWave;
        const bool is_v = load0 >= kGLoadsPerMatrix;  // wave-uniform
        const int idx0 = is_v ? load0 - kGLoadsPerMatrix : load0;
        uint32_t id[2 * kLoadsPerWave];
#pragma unroll
        for (int j = 0; j < 2 * kLoadsPerWave; ++j) id[j] = page_of(t * kKeyTile + (2 * idx0 + j) * kMinPageSize);
        const char* mat = (is_v ? vc : kc) + head_bytes + (g_key & (kMinPageSize - 1)) * kGRowBytes;
#pragma unroll
        for (int j = 0; j < kLoadsPerWave; ++j) {
          const int tile_row = (idx0 + j) * kGKeysPerLoad + g_key;
          const int swz = is_v ? vswz8(tile_row) : kswz8(tile_row);
          const uint32_t page = g_key < kMinPageSize ? id[2 * j] : id[2 * j + 1];
          load_to_lds_16(mat + (uint64_t)page * (uint32_t)page_bytes + ((g_pc ^ swz) << 4),
                         (is_v ? vbuf : kbuf) + (idx0 + j) * 1024);
        }
        return;
      }
    }
    if constexpr (!P8 && kGroupedIssue && kGLoadsPerMatrix % kLoadsPerWave == 0) {
      if ((full_tile || kGroupedLast) && offsets_fit_32) {
        // A load never spans two pages: page, head and first row make a wave-uniform base (scalar
        // registers), the lane adds its row and (swizzled) chunk.  This wave's loads are
        // consecutive rows of ONE matrix, so the base is looked up and multiplied out only where
        // a load starts a new page; inside a page the next load is 1 KB further on.
        const int load0 = issuer * kLoadsPerWave;
        const bool is_v = load0 >= kGLoadsPerMatrix;  // wave-uniform
        const int idx0 = is_v ? load0 - kGLoadsPerMatrix : load0;
        const char* mat = is_v ? vc : kc;
        const uint32_t buf = (is_v ? vbuf : kbuf) + idx0 * 1024;
        // GS loads (GS KB of consecutive rows inside one page) at a time: one page lookup, one
        // base, one M0.  PART: rows past the key range take the range's last row instead; a group
        // that lies past it altogether reads the group which holds that row.  (The offset field
        // moves the global address along with the LDS address, so the lane offsets of such rows
        // go backwards: the base lies kBias lower to keep them unsigned.)
        auto grouped = [&](auto gs_c, auto part_c) {
          constexpr int GS = decltype(gs_c)::value;
          constexpr bool PART = decltype(part_c)::value;
          constexpr int kBias = PART ? (GS - 1) * 1024 : 0;
          const int last_row = k_end - 1 - key0;
#pragma unroll
          for (int j = 0; j < kLoadsPerWave; j += GS) {
            int row0 = (idx0 + j) * kGKeysPerLoad;
            const uint32_t page = GS == 4 ? pages.id[j / 4] : page_of(first_off + t * kKeyTile + row0);
            if constexpr (PART) row0 = min(row0, last_row & ~(GS * kGKeysPerLoad - 1));
            const uint32_t in_page = (uint32_t)(key0 + row0) & (uint32_t)page_mask;
            const uint64_t gbase =
                (uint64_t)page * (uint32_t)page_bytes + (uint32_t)head_bytes + in_page * kGRowBytes - kBias;
            uint32_t off[GS];
#pragma unroll
            for (int q = 0; q < GS; ++q) {
              const int tile_row = (idx0 + j + q) * kGKeysPerLoad + g_key;
              const int swz = KV8 ? (is_v ? vswz8(tile_row) : kswz8(tile_row)) : (is_v ? vswz16(tile_row) : G::kswz(tile_row));
              const int src = PART ? (min(tile_row, last_row) - row0) * kGRowBytes + kBias - q * 1024 : g_key * kGRowBytes;
              off[q] = (uint32_t)(src + ((g_pc ^ swz) << 4));
            }
            if constexpr (GS == 4) load_to_lds_4x16(mat + gbase, off[0], off[1], off[2], off[3], buf + j * 1024);
            else load_to_lds_2x16(mat + gbase, off[0], off[1], buf + j * 1024);
          }
        };
        if constexpr (kLoadsPerWave % 4 == 0) {
          if (page_loads >= 4) {
            if (!kGroupedLast || full_tile) grouped(std::integral_constant<int, 4>{}, std::false_type{});
            else if constexpr (kGroupedLast) grouped(std::integral_constant<int, 4>{}, std::true_type{});
            return;
          }
        }
        if constexpr (kLoadsPerWave % 2 == 0) {
          if (page_loads >= 2) {
            if (!kGroupedLast || full_tile) grouped(std::integral_constant<int, 2>{}, std::false_type{});
            else if constexpr (kGroupedLast) grouped(std::integral_constant<int, 2>{}, std::true_type{});
            return;
          }
        }
        if (!kGroupedLast || full_tile) {
          uint64_t base = 0;
#pragma unroll
          for (int j = 0; j < kLoadsPerWave; ++j) {
            const int row0 = (idx0 + j) * kGKeysPerLoad;  // first tile row of this load
            const int tile_row = row0 + g_key;
            const int swz = KV8 ? (is_v ? vswz8(tile_row) : kswz8(tile_row)) : (is_v ? vswz16(tile_row) : G::kswz(tile_row));
            const uint32_t in_page = (uint32_t)(key0 + row0) & (uint32_t)page_mask;
            if (j == 0 || in_page == 0) {
              const uint32_t page = page_of(first_off + t * kKeyTile + row0);
              base = (uint64_t)page * (uint32_t)page_bytes + (uint32_t)head_bytes + in_page * kGRowBytes;
            } else {
              base += 1024;
            }
            load_to_lds_16(mat + base, (uint32_t)(g_key * kGRowBytes + ((g_pc ^ swz) << 4)), buf + j * 1024);
          }
          return;
        }
      }
    }
    // (rolled: this path serves the last tile of a range and a few rare layouts, and is instantiated
    // once per stage; unrolled it was most of the kernel's code.  Not with 64-byte code rows, whose
    // four loads per wave have their page lookups go out together, nor in the eight-wave kernel
    // that takes this path for all tiles.)
    constexpr int kUnroll = kGroupedIssue && kGKeysPerLoad <= kMinPageSize ? 1 : kLoadsPerWave;
#pragma unroll kUnroll
    for (int j = 0; j < kLoadsPerWave; ++j) {
      const int load = issuer * kLoadsPerWave + j;            // 0 .. 2*kGLoadsPerMatrix-1
      const bool is_v = load >= kGLoadsPerMatrix;             // wave-uniform
      const int idx = is_v ? load - kGLoadsPerMatrix : load;
      const int row0 = idx * kGKeysPerLoad;                    // first tile row of this load
      const int tile_row = row0 + g_key;
      const int swz = KV8 ? (is_v ? vswz8(tile_row) : kswz8(tile_row)) : (is_v ? vswz16(tile_row) : G::kswz(tile_row));
      if constexpr (kGKeysPerLoad <= kMinPageSize) {
        if (full_tile) {
          // all rows of the load lie in one page and inside the range
          const int64_t page = page_of(first_off + t * kKeyTile + row0);
          const int64_t base = page * page_bytes + head_bytes + ((key0 + row0) & page_mask) * kGRowBytes;
          load_to_lds_16((is_v ? vc : kc) + base, (uint32_t)(g_key * kGRowBytes + ((g_pc ^ swz) << 4)),
                         (is_v ? vbuf : kbuf) + idx * 1024);
          continue;
        }
      }
      // one load never spans two pages, except for the shortest rows on the smallest pages:
      // then every lane looks its own page up
      int64_t page;
      if constexpr (!P8)
        page = page_of(first_off + t * kKeyTile + row0);
      else
        page = bt[min(first_page + ((first_off + t * kKeyTile + tile_row) >> ps), last_page)];  // per lane
      const int64_t in_off = page * page_bytes + head_bytes + ((key0 + tile_row) & page_mask) * kGRowBytes;
      const int64_t row_off = (key0 + tile_row < k_end) ? in_off : last_off;
      const char* src = (is_v ? vc : kc) + row_off + ((g_pc ^ swz) << 4);
      load_to_lds_16(src, (is_v ? vbuf : kbuf) + idx * 1024);
    }
  };

  // per-lane LDS addresses of the MFMA operands (buffer 0; buffers, key blocks and keys are added
  // as constants, which go into the offset field of the read)
  const int k_swz = G::kswz(i32);
  const int k8_swz = kswz8(i32);  // same for key i32 + 32
  uint32_t k_addr[G::kSteps];
#pragma unroll
  for (int st = 0; st < G::kSteps; ++st)
    k_addr[st] = KV8 ? lds0 + i32 * D + ((st ^ k8_swz) << 4) + 8 * hi
                     : lds0 + i32 * G::kRowBytes + (((2 * st + hi) ^ k_swz) << 4);
  // K operand of key block kb, MFMA step st: 8 consecutive head-dim elements (2 * st + hi) * 8 ..
  // of key kb * 32 + i32 -- 16 bytes of the bf16 tile, or 8 codes that become bf16 in registers
  using KRaw = std::conditional_t<KV8, u32x2, u32x4>;
  auto read_k = [&](uint32_t buf, int kb, int st) -> KRaw {
    // (PACK: bits 5 and 6 of the address belong to the step alone)
    const uint32_t at = PACK ? k_addr[0] ^ (uint32_t)(st << 5) : k_addr[st];
    return *reinterpret_cast<const LDS_PTR(KRaw)>(at + (buf + kb * 32 * kGRowBytes));
  };
  // (the same conversion serves the value operands)
  auto k_operand = [&](KRaw raw) -> bf16x8 {
    if constexpr (KV8) {
      u32x4 v;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        v[2 * j] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[j], 1.0f, false));
        v[2 * j + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[j], 1.0f, true));
      }
      return __builtin_bit_cast(bf16x8, v);
    } else {
      return __builtin_bit_cast(bf16x8, raw);
    }
  };
  // 16-lane block b of the wave reads a 4-key x 16-d patch of V through the transposing
  // read; lane w of the block supplies the address of key w/4, d-offset 4*(w%4) and receives
  // column w of the patch (4 consecutive keys of one d).
  const int blk = lane >> 4;
  const int w16 = lane & 15;
  const int v_key = (blk >> 1) * 4 + (w16 >> 2);            // key inside a 16-key group (+8 for 2nd half)
  const int v_chunk = 2 * (blk & 1) + ((w16 & 3) >> 1);     // 16-byte chunk inside a 32-d block
  const int v_sub = (w16 & 1) * 8;
  const int v_swz = G::vswz(v_key);                         // same for v_key + 8, + 16, ...
  // 8-bit values: a 16-lane block reads an 8-key x 16-d patch of codes; lanes 2e and 2e+1 of the
  // block supply the two 8-byte halves of patch row e, lane w receives column w (one head-dim
  // element, the 8 rows).  The rows are the keys whose probabilities this half of the wave
  // holds in the B operand: {0..3, 8..11} + 4 * (lane / 32) of the 16-key group.
  const int v8_e = w16 >> 1;
  const int v8_key = (v8_e < 4 ? v8_e : v8_e + 4) + (blk >> 1) * 4;
  const int v8_chunk = blk & 1;                             // 16-byte chunk inside a 32-d block
  const int v8_sub = (w16 & 1) * 8;
  const int v8_swz = vswz8(v8_key);                         // same for v8_key + 16, + 32, ...
  // V^T operand of the 16-key group ks4 and head-dim block d: raw LDS data, then as bf16
  using VRaw = KRaw;
  auto& v_operand = k_operand;
  uint32_t v_addr[G::kDBlocks];
#pragma unroll
  for (int d = 0; d < G::kDBlocks; ++d)
    v_addr[d] = KV8 ? lds0 + kVOff + v8_key * D + (((d * 2 + v8_chunk) ^ v8_swz) << 4) + v8_sub
                    : lds0 + kVOff + v_key * G::kRowBytes + v_sub + (((d * 4 + v_chunk) ^ v_swz) << 4);
  auto read_v_raw = [&](uint32_t buf, int ks4, int d) -> VRaw {
    const uint32_t at = (PACK ? v_addr[0] ^ (uint32_t)(d << 6) : v_addr[d]) + (buf + ks4 * 16 * kGRowBytes);
    if constexpr (KV8) {
      return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_PTR(i32x2))(at)));
    } else {
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(at));
      const bf16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(at + 8 * G::kRowBytes));
      return __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };

  // ---- the software pipeline of the kernels with more than 32 query rows per item ----------
  // A half-tile is 32 keys.  While the VALU turns the scores of half h into probabilities, the
  // matrix pipe forms the scores of half h + 1 and adds the value product of half h - 1: the
  // three are independent, so each of a wave's MFMAs has vector instructions to hide behind it
  // and neither pipe waits for the other inside a wave.  Measured on this part: a 32x32x16 MFMA
  // occupies its pipe for 32.4 cycles and the wave's issue slot for four of them, so up to six
  // vector instructions per MFMA are free (an exponential counts as two); with head dim 128 a
  // half needs about four.  With head dim 64 it has half the MFMAs for the same softmax, about
  // eight each: there the vector pipe is the longer one and the matrix pipe hides behind it.
  // Against tiles worked off one phase after the other (scores, softmax, values): 28/4-head step
  // with 8..64 new tokens 131.1 -> 124.6 us (8-bit cache 127.6 -> 121.9 us), 4 x 512 new tokens
  // behind 16384 502 -> 491 us.  Ranges of three to five tiles are too short for it: 28/4 heads, 104
  // items of 3-4 tiles over four layers 79 -> 82 us.
  u32x4 p0[2], p1[2];  // probabilities of an even / odd half as B operands (bf16)
  f32x16 s0, s1;       // raw scores of an even / odd half
  // The reference of a row that has seen no score above minus infinity: so low that any finite
  // score makes an infinite weight, whose half then takes the path that sets the reference.
  constexpr float kNoReference = -3.0e38f;
  float l_half = 0.f;  // row sum of the first half of the tile whose second half is next
  // Two probabilities as a bf16 pair (both operand words and row sums take the rounded values).
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const bf16x2 ones2 = {(__bf16)1.0f, (__bf16)1.0f};
  auto prob = [&](float sc) { return __builtin_amdgcn_exp2f(sc * p.scale_log2 - m_run); };

  // kQk: scores of key half kb of the K tile at ks into sn.  kPv: value product of pp with 32-key
  // half vh of the V tile at vs.  kSm: probabilities of sc into pc and their sum.
  auto phase = [&](auto qk_c, f32x16& sn, uint32_t ks, int kb, auto pv_c, const u32x4 (&pp)[2], uint32_t vs, int vh,
                   auto sm_c, const f32x16& sc, u32x4 (&pc)[2]) __attribute__((always_inline)) -> float {
    constexpr bool kQk = decltype(qk_c)::value, kPv = decltype(pv_c)::value, kSm = decltype(sm_c)::value;
    constexpr int kPvMfma = 2 * G::kDBlocks;
    constexpr int kGroups = G::kSteps + kPvMfma;
    constexpr int kPer = 16 / kGroups;  // score elements turned into probabilities per group
    // Scores first: their K operands are read in front of the phase, the V operands under their
    // MFMAs.  PACK: values first, then fewer registers are live at any point; the last two of
    // their MFMAs and the score MFMAs each cover the read of a K operand two steps ahead.
    constexpr int kAheadK = PACK && kPv ? 2 : G::kSteps;
    constexpr int kFirst = PACK ? kPvMfma : G::kSteps;  // MFMAs of the product that comes first
    KRaw ka[G::kSteps];
    VRaw va[kPvMfma];
    auto load_k = [&](int st) __attribute__((always_inline)) { ka[st] = read_k(ks, kb, st); };
    auto load_v = [&](int j) __attribute__((always_inline)) { va[j] = read_v_raw(vs, vh * 2 + j / G::kDBlocks, j % G::kDBlocks); };
    // (keeps the derived addresses from being formed once and held)
    if constexpr (PACK) asm volatile("" : "+v"(k_addr[0]), "+v"(v_addr[0]));
    if constexpr (kQk && !(PACK && kPv)) {
#pragma unroll
      for (int st = 0; st < G::kSteps; ++st) load_k(st);
    }
    if constexpr (kPv && (PACK || !kQk)) {
#pragma unroll
      for (int j = 0; j < kPvMfma; ++j) load_v(j);
    }
    __builtin_amdgcn_sched_barrier(0);
    float acc = 0.f;
    float pr[kPer > 1 ? kPer : 2];
#pragma unroll
    for (int i = 0; i < kGroups; ++i) {
      const bool scores = (i < kFirst) != PACK;
      const int j = i < kFirst ? i : i - kFirst;
      if (scores) {
        if constexpr (kQk) {
          if (j == 0) {
            f32x16 zero;
#pragma unroll
            for (int r = 0; r < 16; ++r) zero[r] = 0.f;
            sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_operand(ka[j]), qb[j], zero, 0, 0, 0);
          } else {
            sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_operand(ka[j]), qb[j], sn, 0, 0, 0);
          }
          if constexpr (kPv && !PACK) load_v(j);
          if (j + kAheadK < G::kSteps) load_k(j + kAheadK);
        }
      } else if constexpr (kPv) {
        const int d = j % G::kDBlocks;
        o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(va[j]), __builtin_bit_cast(bf16x8, pp[j / G::kDBlocks]),
                                                       o[d], 0, 0, 0);
        if (PACK && kQk && j >= kPvMfma - kAheadK) load_k(j - (kPvMfma - kAheadK));
      }
      if constexpr (kSm) {
#pragma unroll
        for (int e = i * kPer; e < (i + 1) * kPer; ++e) {
          pr[e & 1] = prob(sc[e]);
          if (e & 1) {
            const bf16x2 two = __builtin_convertvector((f32x2){pr[0], pr[1]}, bf16x2);
            pc[e >> 3][(e & 7) >> 1] = __builtin_bit_cast(uint32_t, two);
            // the order of `sum_pairs`; the empty statement keeps each step in its group
            acc = __builtin_amdgcn_fdot2_f32_bf16(two, ones2, acc, false);
            asm volatile("" : "+v"(acc));
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    return acc;
  };
  constexpr auto kYes = std::true_type{};
  constexpr auto kNo = std::false_type{};
  // Causal mask of the half whose first key is key0: element r is key key0 + (r/4)*8 + hi*4 + r%4.
  // Each lane holds one bit per key of the half, and an element takes minus infinity through a bit
  // select: two vector instructions each and no condition register.  A compare whose result a
  // select reads has to stand two wait states in front of it on this target; the compiler keeps
  // that rule for its own instructions (and would turn a plain select here into divergent
  // branches with copies of all sixteen scores) but not inside inline assembly.
  auto mask_half = [&](f32x16& sc, int key0) __attribute__((always_inline)) {
    if (key0 + 32 > wave_min_vis) {
      const int lim = n_vis - key0 - hi * 4;  // visible keys counted from this lane's first key of the half
      // (its last key is number 27, so that a limit of 31 hides nothing)
      const uint32_t hidden = ~0u << min(max(lim, 0), 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)hidden, (r >> 2) * 8 + (r & 3), 1);  // 0 or all ones
        sc[r] = __uint_as_float((m & 0xFF800000u) | (~m & __float_as_uint(sc[r])));
      }
    }
  };
  // maximum of a half's scores of this lane's row, in this lane's half of its elements
  auto half_max = [&](const f32x16& sc) __attribute__((always_inline)) {
    float mx = max3(sc[0], sc[1], sc[2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) mx = max3(mx, sc[r], sc[r + 1]);
    return fmaxf(mx, sc[15]);
  };
  // Moves a row's reference to `m_next` (rows whose reference stays pass m_run: factor one).
  auto move_reference = [&](float m_next) __attribute__((always_inline)) {
    const float f = m_next == m_run ? 1.f : __builtin_amdgcn_exp2f(m_run - m_next);
    l_run *= f;
    l_half *= f;
#pragma unroll
    for (int d = 0; d < G::kDBlocks; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[d][r] *= f;
    m_run = m_next;
  };
  // Behind a half's probabilities: m_run is a reference value, set to the row's maximum over its
  // first tile and moved only by a half whose maximum lies more than 2^kSlack above it, so that
  // probabilities stay below 2^kSlack.  Such a half shows in its sum: no running maximum is formed
  // otherwise.  The first reference is the maximum over all 64 keys of the tile because that
  // makes the largest weight of a short row exactly one: with the maximum over 32 keys the error
  // against 64-bit arithmetic of a step with full misses was 0.7 % larger (relative L2 2.048e-3
  // against 2.033e-3).  A row is moved by its own scores alone, whatever the other rows of the
  // wave hold.
  auto settle = [&](float acc, const f32x16& sc, u32x4 (&pc)[2]) __attribute__((always_inline)) -> float {
    constexpr float kOver = 256.f;  // 2^kSlack; a sum of rounded probabilities is never below its largest one
    if (__any(acc >= kOver)) {
      const float m_new = cross_half_max(half_max(sc)) * p.scale_log2;
      move_reference(m_new > m_run + kSlack ? m_new : m_run);
      u32x4 dummy[2];
      acc = phase(kNo, s0, 0u, 0, kNo, dummy, 0u, 0, kYes, sc, pc);
    }
    return acc;
  };
  // What the bf16 rounding of a half's probabilities dropped, as B operands: with it a
  // probability enters the value product with 16 significant bits.  Used for the (single) tile of
  // a wave whose first row sees very few keys: there the output is a weighted mean of a handful
  // of value rows and can reach magnitude 2-4, where its own bf16 rounding is already 7.8e-3,
  // and the 2^-9 relative rounding of single bf16 weights on top of that would cross the 1e-2
  // error bound.
  // Returns their sum, which goes into the row sum: the normaliser is the sum of the weights the
  // product uses.
  auto dropped = [&](const f32x16& sc, u32x4 (&pl)[2]) __attribute__((always_inline)) -> float {
    float acc = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
      const float a = prob(sc[e]), c = prob(sc[e + 1]);
      const bf16x2 two = __builtin_convertvector((f32x2){a - (float)(__bf16)a, c - (float)(__bf16)c}, bf16x2);
      pl[e >> 3][(e & 7) >> 1] = __builtin_bit_cast(uint32_t, two);
      acc = __builtin_amdgcn_fdot2_f32_bf16(two, ones2, acc, false);
    }
    return acc;
  };

  // One 32-key half (kb = 0 or 1, wave-uniform) of a tile in the key-parallel kernels.  LO: a second
  // pass that adds what the bf16 rounding of the probabilities dropped (see `dropped` above).
  auto compute_half = [&](int t, uint32_t buf, int kb, auto lo_c) __attribute__((always_inline)) {
    constexpr bool LO = decltype(lo_c)::value;
    const int key0 = k_begin + t * kKeyTile + kb * 32;
    f32x16 sc;
    KRaw ka[G::kSteps];
#pragma unroll
    for (int st = 0; st < G::kSteps; ++st) ka[st] = read_k(buf, kb, st);
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[r] = 0.f;
#pragma unroll
    for (int st = 0; st < G::kSteps; ++st)
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_operand(ka[st]), qb[st], sc, 0, 0, 0);
    VRaw va[2][G::kDBlocks];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int d = 0; d < G::kDBlocks; ++d) va[h][d] = read_v_raw(buf, kb * 2 + h, d);
    if (key0 + 32 > wave_min_vis) {
      const int lim = n_vis - key0 - hi * 4;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if ((r >> 2) * 8 + (r & 3) >= lim) sc[r] = -INFINITY;
    }
    if constexpr (!LO) {
      float tmax = max3(sc[0], sc[1], sc[2]);
#pragma unroll
      for (int r = 3; r < 15; r += 2) tmax = max3(tmax, sc[r], sc[r + 1]);
      tmax = cross_half_max(fmaxf(tmax, sc[15]));
      const float m_new = tmax * p.scale_log2;
      const bool grow = m_new > m_run + kSlack;
      if (__any(grow)) {
        // only the rows that outgrew their reference move it: a row's arithmetic then depends
        // on that row's scores alone, whatever the other rows of the wave hold
        const float m_next = grow ? m_new : m_run;
        const float m_safe = (m_next == -INFINITY) ? 0.f : m_next;
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
        l_run *= alpha;
#pragma unroll
        for (int d = 0; d < G::kDBlocks; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
        m_run = m_next;
      }
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
    bf16x8 pb[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float pr = __builtin_amdgcn_exp2f(sc[r] * p.scale_log2 - m_use);
      pb[r >> 3][r & 7] = LO ? (__bf16)(pr - (float)(__bf16)pr) : (__bf16)pr;
    }
    l_run += sum_pairs(pb[0], pb[1]);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int d = 0; d < G::kDBlocks; ++d) {
        o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(va[h][d]), pb[h], o[d], 0, 0, 0);
      }
  };

  // R16.  S^T = K Q^T in two blocks of 16 keys: a lane has keys 16 * kb + 4 * q4 + r of the half and one query
  // row, which is the order in which the value product takes its 32 keys from both operands: eight
  // per lane, {0..3} + 4 * q4 of either block.
  const int k16_swz = KV8 ? kswz8(i16) : G::kswz(i16);  // same for key i16 + 16, + 32, ...
  const int v16_key = KV8 ? 4 * q4 + (v8_e < 4 ? v8_e : v8_e + 12) : 4 * q4 + (w16 >> 2);  // bf16: + 16 for the second block
  const int v16_swz = KV8 ? vswz8(v16_key) : vswz16(v16_key);
  auto compute_half16 = [&](int t, uint32_t buf, int half, auto lo_c) __attribute__((always_inline)) {
    constexpr bool LO = decltype(lo_c)::value;
    const int key0 = k_begin + t * kKeyTile + half * 32;
    const uint32_t at = lds0 + buf + half * 32 * kGRowBytes;
    KRaw ka[2][kQSteps];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int s = 0; s < kQSteps; ++s) {
        const int chunk = KV8 ? 2 * s + (q4 >> 1) : 4 * s + q4;
        ka[kb][s] = *reinterpret_cast<const LDS_PTR(KRaw)>(at + i16 * kGRowBytes + ((chunk ^ k16_swz) << 4) +
                                                           (KV8 ? 8 * (q4 & 1) : 0) + kb * 16 * kGRowBytes);
      }
    f32x4 sc[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      sc[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < kQSteps; ++s)
        sc[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k_operand(ka[kb][s]), qb[s], sc[kb], 0, 0, 0);
    }
    VRaw va[D / 16];
#pragma unroll
    for (int d = 0; d < D / 16; ++d) {
      const uint32_t v_at = at + kVOff + v16_key * kGRowBytes + v_sub;
      if constexpr (KV8) {
        va[d] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_PTR(i32x2))(v_at + ((d ^ v16_swz) << 4))));
      } else {
        const uint32_t c_at = v_at + (((2 * d + ((w16 & 3) >> 1)) ^ v16_swz) << 4);
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(c_at));
        const bf16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_PTR(bf16x4))(c_at + 16 * kGRowBytes));
        va[d] = __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    }
    if (key0 + 32 > wave_min_vis) {
      const int lim = n_vis - key0 - q4 * 4;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (kb * 16 + r >= lim) sc[kb][r] = -INFINITY;
    }
    if constexpr (!LO) {
      float tmax = max3(max3(sc[0][0], sc[0][1], sc[0][2]), sc[0][3], max3(sc[1][0], sc[1][1], sc[1][2]));
      tmax = cross_half_max(cross_quarter_max(fmaxf(tmax, sc[1][3])));
      const float m_new = tmax * p.scale_log2;
      const bool grow = m_new > m_run + kSlack;
      if (__any(grow)) {
        // (as above: a row moves by its own scores alone)
        const float m_next = grow ? m_new : m_run;
        const float m_safe = (m_next == -INFINITY) ? 0.f : m_next;
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
        l_run *= alpha;
#pragma unroll
        for (int d = 0; d < D / 16; ++d)
#pragma unroll
          for (int r = 0; r < 4; ++r) o16[d][r] *= alpha;
        m_run = m_next;
      }
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
    bf16x8 pb;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float pr = __builtin_amdgcn_exp2f(sc[r >> 2][r & 3] * p.scale_log2 - m_use);
      pb[r] = LO ? (__bf16)(pr - (float)(__bf16)pr) : (__bf16)pr;
    }
    float acc = 0.f;
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb, pb, 0, 1), ones2, acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb, pb, 2, 3), ones2, acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb, pb, 4, 5), ones2, acc, false);
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb, pb, 6, 7), ones2, acc, false);
    l_run += acc;
#pragma unroll
    for (int d = 0; d < D / 16; ++d) o16[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v_operand(va[d]), pb, o16[d], 0, 0, 0);
  };
  auto half_of_tile = [&](int t, uint32_t buf, int half, auto lo_c) __attribute__((always_inline)) {
    if constexpr (R16) compute_half16(t, buf, half, lo_c);
    else compute_half(t, buf, half, lo_c);
  };

  // rows with at most this many visible keys get the second (LO) pass over their first tile
  constexpr int kFineKeys = 16;
  const bool fine_wave = k_begin == 0 && wave_min_vis <= kFineKeys;  // wave-uniform
  auto step = [&](int t, uint32_t buf, auto first_c) __attribute__((always_inline)) {
    if (wave < 2 && k_begin + t * kKeyTile + wave * 32 < wave_max_vis) {
      half_of_tile(t, buf, wave, std::false_type{});
      if constexpr (decltype(first_c)::value)
        if (fine_wave && t == 0 && wave == 0) half_of_tile(t, buf, wave, std::true_type{});
    }
  };
  // Loop top for tile t (stage t of the pipelined kernels): the gathers of up to STAGES - 2 later
  // tiles (this wave's newest loads; `last` is the last one it issues) may stay in flight;
  // everything older must have landed.  The barrier publishes tile t and tells that every wave is
  // done with the buffer about to be refilled.
  auto wait_tile = [&](int t, int last) {
    const int later = min(STAGES - 2, last - t);  // tiles issued after t so far
    if (STAGES >= 3 && later == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoadsPerWave) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  static_assert(STAGES <= 3 || ONCE, "wait_tile and the loops below handle two tiles in flight");

  // Pipelined kernels: stage t of the ring holds the keys of tile t and the values of tile t - 1
  // (a tile's scores are formed one tile ahead of its value product); stages 0 .. ntiles.  Each
  // wave gathers rows of one matrix only, so that is a shift of the tile index of the waves that
  // gather values.
  const int shift = (!KP && issuer * kLoadsPerWave >= kGLoadsPerMatrix) ? 1 : 0;
  static_assert(KP || kGLoadsPerMatrix % kLoadsPerWave == 0, "a wave gathers one matrix");
  const int last_stage = ntiles - 1 + shift;
  // Fused step: the raw query rows of the tile and the raw key and value rows of the new tokens go
  // straight to LDS, 1 KB per wave instruction dealt to the waves, ahead of the first gathers:
  // they land first, and their wait leaves the gathers in flight.  The prologue then costs one
  // memory latency and not one each for the gathers, the query and key elements and the values,
  // one behind the other.  Measured per step: one request of 2344 keys, 32/8 heads 15.7 -> 13.3 us;
  // 32 requests of 2048..8192 keys, 28/4 heads 74.9 -> 72.3 us, 8-bit cache 43.7 -> 41.6 us; 16
  // requests of 1024..4096 keys, 32/32 heads 124.9 -> 118.9 us.
  const int n_tok = it.row_count / g;  // fused: all rows of the (request, kv head) pair are in this tile
  if constexpr (FUSED) {
    if constexpr (!ONCE) asm volatile("" ::"v"(inv_freq) : "memory");
    constexpr int kRawChunks = D / 8;            // 16-byte chunks of a bf16 row
    constexpr int kRowsPerLoad = 64 / kRawChunks;
    static_assert(kFusedRows % kRowsPerLoad == 0 && kFusedMaxTokens * 2 % kRowsPerLoad == 0, "loads fill whole areas");
    const int q_loads = (it.row_count + kRowsPerLoad - 1) / kRowsPerLoad;
    const int kv_loads = (2 * n_tok + kRowsPerLoad - 1) / kRowsPerLoad;
    const int c8 = lane % kRawChunks * 8;
    for (int l = wave; l < q_loads + kv_loads; l += WAVES) {
      const uint16_t* src;
      uint32_t dst;
      if (l < q_loads) {
        // (rows past the last are loads of the last one)
        const int r = min(l * kRowsPerLoad + lane / kRawChunks, it.row_count - 1);
        const int tk = r / g;
        src = q_rows + ((int64_t)(rq.row_start + tk) * p.num_q_heads + it.kv_head * g + (r - tk * g)) * D + c8;
        dst = (uint32_t)(uintptr_t)(LDS_PTR(char))s_q + l * 1024;
      } else {
        const int r = min((l - q_loads) * kRowsPerLoad + lane / kRawChunks, 2 * n_tok - 1);
        src = (r & 1 ? p.v_new : p.k_new) + ((int64_t)(rq.row_start + (r >> 1)) * kv_heads + it.kv_head) * D + c8;
        dst = (uint32_t)(uintptr_t)(LDS_PTR(char))s_raw + (l - q_loads) * 1024;
      }
      load_to_lds_16(src, dst);
    }
    if constexpr (ONCE) {
      // the frequencies have landed: all but this wave's raw rows
      static_assert((kFusedRows + 2 * kFusedMaxTokens) / kRowsPerLoad <= 4 * WAVES, "the wait counts that many loads");
      switch ((q_loads + kv_loads - wave + WAVES - 1) / WAVES) {
        case 1: asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); break;
        case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
        case 3: asm volatile("s_waitcnt vmcnt(3)" ::: "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      inv_freq = reinterpret_cast<const double*>(s_freq)[tid % (D / 2)];
    }
  }
  if constexpr (ONCE) {
    // (page ids of all tiles together, one latency, where a page holds the four loads of a wave: bf16 rows of head
    // dim 128 on pages of 16 and more; elsewhere issue_tile looks them up tile by tile)
    TilePages pages[STAGES];
#pragma unroll
    for (int st = 0; st < STAGES; ++st) pages[st] = fetch_pages(min(st, ntiles - 1));
#pragma unroll
    for (int st = 0; st < STAGES; ++st)
      if (st < ntiles) issue_tile(st, st, pages[st]);
  } else {
#pragma unroll
    for (int st = 0; st < STAGES - 1; ++st)
      if (st >= shift && st <= last_stage) issue_tile(st - shift, st, fetch_pages(st - shift));
  }
  // Everything the compiler knows to be loading (the query operands) must have landed before
  // the main loop: inside it the only outstanding vector-memory operations are the gathers,
  // which are awaited by hand.  (vmcnt(0), expcnt/lgkmcnt untouched; the gathers just issued
  // are waited for as well, which the first tiles would do anyway)
  if constexpr (!FUSED) __builtin_amdgcn_s_waitcnt(0x0F70);
  if constexpr (FUSED) {
    // Rotary embedding of the tile's query rows and of the new tokens' keys (token j of the
    // request sits at position C_r + j and is packed row rq.row_start + j), same arithmetic as
    // the stand-alone append kernel.  First the cosines and sines, one task per (token, pair),
    // into the tile buffer that no gather has been issued into yet (the last one; ONCE: an area of their own),
    // while the raw rows are on their way; then one task per (row, pair) over the query rows and the key rows.
    const int rot_half = p.rotary_dim / 2;  // pairs per head row (D/2 when the whole row rotates)
    double* const s_cs = reinterpret_cast<double*>(s_table);  // [token][pair] (cos, sin)
    static_assert(kFusedMaxTokens * (D / 2) * 16 <= (ONCE ? kTableBytes : kStageBytes), "the cos/sin table must fit");
    {
      const int j = tid % (D / 2);
      if (j < rot_half)
        for (int tk = tid / (D / 2); tk < n_tok; tk += 64 * WAVES / (D / 2)) {
          double sn, cs;
          sincos((double)(rq.cached + tk) * inv_freq, &sn, &cs);
          s_cs[(tk * (D / 2) + j) * 2] = cs;
          s_cs[(tk * (D / 2) + j) * 2 + 1] = sn;
        }
    }
    // this wave's raw rows have landed; the gathers issued behind them stay in flight
    static_assert((ONCE ? STAGES : 2) * kLoadsPerWave <= 63, "the wait counts that many tiles");
    if constexpr (ONCE) {
#define EFIM_WAIT_TILES(N) \
  case N: asm volatile("s_waitcnt vmcnt(%0)" ::"n"((N) <= STAGES ? (N) * kLoadsPerWave : 0) : "memory"); break;
      switch (ntiles) {
        EFIM_WAIT_TILES(1) EFIM_WAIT_TILES(2) EFIM_WAIT_TILES(3) EFIM_WAIT_TILES(4)
        EFIM_WAIT_TILES(5) EFIM_WAIT_TILES(6) EFIM_WAIT_TILES(7) EFIM_WAIT_TILES(8)
        default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
#undef EFIM_WAIT_TILES
    } else if (issuer < 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (STAGES >= 3 && ntiles >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kLoadsPerWave) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoadsPerWave) : "memory");
    __syncthreads();
    for (int idx = tid; idx < (it.row_count + n_tok) * (D / 2); idx += 64 * WAVES) {
      const int r = idx / (D / 2), j = idx - r * (D / 2);
      // pair j of the rotated part, or two neighbouring elements behind it (passed through)
      const bool rotate = j < rot_half;
      const int e1 = !rotate ? p.rotary_dim + 2 * (j - rot_half) : (p.interleaved ? 2 * j : j);
      const int e2 = !rotate ? e1 + 1 : (p.interleaved ? 2 * j + 1 : j + rot_half);
      const bool is_key = r >= it.row_count;  // rows behind the query rows: the new tokens' keys
      const int tk = is_key ? r - it.row_count : r / g;
      uint16_t* const row = is_key ? s_raw + tk * 2 * D : s_q + r * D;
      uint32_t y1 = row[e1], y2 = row[e2];
      if (rotate) rotate_pair_bf16(y1, y2, s_cs[(tk * (D / 2) + j) * 2], s_cs[(tk * (D / 2) + j) * 2 + 1], &y1, &y2);
      if (KV8 && is_key) {
        // the key goes into the cache as a code
        uint8_t* krow = reinterpret_cast<uint8_t*>(s_kv + tk * 2 * kGRowBytes);
        krow[e1] = (uint8_t)bf16_bits_to_e4m3(y1, p.k_inv);
        krow[e2] = (uint8_t)bf16_bits_to_e4m3(y2, p.k_inv);
      } else {
        row[e1] = (uint16_t)y1;
        row[e2] = (uint16_t)y2;
      }
    }
    if constexpr (KV8) {
      for (int idx = tid; idx < n_tok * D; idx += 64 * WAVES) {
        const int tk = idx / D, e = idx - tk * D;
        reinterpret_cast<uint8_t*>(s_kv + tk * 2 * kGRowBytes + kGRowBytes)[e] =
            (uint8_t)bf16_bits_to_e4m3(s_raw[(tk * 2 + 1) * D + e], p.v_inv);
      }
    }
    __syncthreads();
  }
  if constexpr (FUSED) {
#pragma unroll
    for (int s = 0; s < kQSteps; ++s) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (row_ok) v = *reinterpret_cast<const u32x4*>(s_q + local_row * D + (D / kQSteps) * s + q_at);
      qb[s] = __builtin_bit_cast(bf16x8, v);
    }
  }
  // Fused step.  Key tiles that reach into the new tokens: their cache slots have not been written
  // yet, so those rows of the landed tile are replaced by the rotated keys / the values
  // from LDS, and the tokens are appended to the paged cache (each position by the one
  // workgroup of its kv head whose key range holds it).  Rows behind the key range,
  // which the gather fetched from the range's last slot, take that token's rows too.
  // True: the tile in buffer `slot` has been written to.
  auto patch_tile = [&](int t, int slot) __attribute__((always_inline)) -> bool {
    const int key0 = k_begin + t * kKeyTile;
    if (k_end <= rq.cached || key0 + kKeyTile <= rq.cached) return false;
    const int prow = max(rq.cached - key0, 0);  // first row of the tile that holds a new token
    constexpr int kPerRow = 2 * kGChunks;  // 16-byte chunks of a key row and a value row
    for (int u = tid; u < (kKeyTile - prow) * kPerRow; u += 64 * WAVES) {
      const int row = prow + u / kPerRow;
      const int w = u % kPerRow;
      const bool is_v = w >= kGChunks;
      const int c = is_v ? w - kGChunks : w;
      const int pos = min(key0 + row, k_end - 1);
      const u32x4 val = *reinterpret_cast<const u32x4*>(s_kv + (pos - rq.cached) * 2 * kGRowBytes +
                                                        (is_v ? kGRowBytes : 0) + c * 16);
      const int swz = KV8 ? (is_v ? vswz8(row) : kswz8(row)) : (is_v ? vswz16(row) : G::kswz(row));
      char* tile = stages + slot * kStageBytes + (is_v ? kGTileBytes : 0);
      *reinterpret_cast<u32x4*>(tile + row * kGRowBytes + ((c ^ swz) << 4)) = val;
      if (key0 + row < k_end) {
        const int64_t page = bt[pos >> ps];
        char* cache = reinterpret_cast<char*>(is_v ? p.v_cache_w : p.k_cache_w);
        *reinterpret_cast<u32x4*>(
            cache + (((page * kv_heads + it.kv_head) << ps) + (pos & page_mask)) * kGRowBytes + c * 16) = val;
      }
    }
    return true;
  };
  // One tile of the unrolled ring: stage s0 (a compile-time constant) holds tile t0 + s0.
  auto ring_step = [&](int t0, auto s0_c) __attribute__((always_inline)) {
    constexpr int s0 = decltype(s0_c)::value;
    {
      const int t = t0 + s0;
      if (t < ntiles) {
        constexpr int kAhead = STAGES - 1;
        const int sl = (s0 + kAhead) % STAGES;  // static after unrolling
        const TilePages pages = fetch_pages(min(t + kAhead, ntiles - 1));
        wait_tile(t, ntiles - 1);
        if (t + kAhead < ntiles) issue_tile(t + kAhead, sl, pages);
        if constexpr (FUSED) {
          if (patch_tile(t, s0)) __syncthreads();
        }
        // (tile 0 is always the first of the unrolled copies)
        step(t, s0 * kSlotBytes, std::bool_constant<s0 == 0>{});
      }
    }
  };
  if constexpr (ONCE) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if constexpr (FUSED) {
      bool patched = false;
      for (int t = max(0, rq.cached - k_begin) / kKeyTile; t < ntiles; ++t) patched |= patch_tile(t, t);
      if (patched) __syncthreads();
    }
    const int half = wave & 1;
    for (int t = wave >> 1; t < ntiles; t += WAVES / 2)
      if (k_begin + t * kKeyTile + half * 32 < wave_max_vis) {
        half_of_tile(t, t * kSlotBytes, half, std::false_type{});
        if (fine_wave && t == 0 && half == 0) half_of_tile(t, 0u, 0, std::true_type{});
      }
  } else if constexpr (KP) {
    for (int t0 = 0; t0 < ntiles; t0 += STAGES) {
      ring_step(t0, std::integral_constant<int, 0>{});
      ring_step(t0, std::integral_constant<int, 1>{});
      if constexpr (STAGES > 2) ring_step(t0, std::integral_constant<int, 2>{});
    }
  } else {
    // key tiles this wave's rows reach into; its pipeline ends there, its gathers go on
    const int n_w = wave_active ? min(ntiles, max(0, (wave_max_vis - k_begin + kKeyTile - 1) / kKeyTile)) : 0;
    // publishes stage t and starts the gather of stage t + STAGES - 1 into `slot`
    auto top = [&](int t, int slot) __attribute__((always_inline)) {
      const int s_new = t + STAGES - 1;
      const TilePages pages = fetch_pages(min(max(s_new - shift, 0), ntiles - 1));
      wait_tile(t, last_stage);
      if (s_new >= shift && s_new <= last_stage) issue_tile(s_new - shift, slot, pages);
    };
    // stage 0: scores of the first tile, probabilities of its first half
    top(0, STAGES - 1);
    if (n_w > 0) {
      constexpr uint32_t ks = 0;
      phase(kYes, s0, ks, 0, kNo, p0, 0u, 0, kNo, s0, p0);
      phase(kYes, s1, ks, 1, kNo, p0, 0u, 0, kNo, s0, p0);
      mask_half(s0, k_begin);
      mask_half(s1, k_begin + 32);
      m_run = cross_half_max(fmaxf(half_max(s0), half_max(s1))) * p.scale_log2;
      if (m_run == -INFINITY) m_run = kNoReference;
      l_half = phase(kNo, s0, 0u, 0, kNo, p0, 0u, 0, kYes, s0, p0);
    }
    auto body = [&](int t, auto slot_c) __attribute__((always_inline)) {
      constexpr int slot = decltype(slot_c)::value;
      top(t, (slot + STAGES - 1) % STAGES);
      constexpr uint32_t ks = slot * kSlotBytes, vs = ks;
      const int key0 = k_begin + t * kKeyTile;
      mask_half(s1, key0 - 32);
      float acc = phase(kYes, s0, ks, 0, kYes, p0, vs, 0, kYes, s1, p1);
      acc = settle(acc, s1, p1);
      l_run += l_half + acc;
      mask_half(s0, key0);
      acc = phase(kYes, s1, ks, 1, kYes, p1, vs, 1, kYes, s0, p0);
      l_half = settle(acc, s0, p0);
    };
    int t = 1;
    while (true) {
      if (t >= n_w) break;
      body(t, std::integral_constant<int, 1 % STAGES>{});
      ++t;
      if (t >= n_w) break;
      body(t, std::integral_constant<int, 2 % STAGES>{});
      ++t;
      if constexpr (STAGES > 2) {
        if (t >= n_w) break;
        body(t, std::integral_constant<int, 3 % STAGES>{});
        ++t;
      }
    }
    if (n_w > 0) {
      // stage n_w: the second half of this wave's last tile and the values of both halves
      const int slot = t % STAGES;
      top(t, (slot + STAGES - 1) % STAGES);
      const uint32_t vs = slot * kSlotBytes;
      mask_half(s1, k_begin + t * kKeyTile - 32);
      const float acc = settle(phase(kNo, s0, 0u, 0, kYes, p0, vs, 0, kYes, s1, p1), s1, p1);
      l_run += l_half + acc;
      phase(kNo, s0, 0u, 0, kYes, p1, vs, 1, kNo, s1, p1);
      if (fine_wave) {
        // (such a wave has one tile only: s0 still holds the scores of its first half)
        u32x4 pl0[2], pl1[2];
        const float lo0 = dropped(s0, pl0), lo1 = dropped(s1, pl1);
        l_run += lo0 + lo1;
        phase(kNo, s0, 0u, 0, kYes, pl0, vs, 0, kNo, s0, pl0);
        phase(kNo, s0, 0u, 0, kYes, pl1, vs, 1, kNo, s1, pl1);
      }
      ++t;
    }
    if (m_run == kNoReference) m_run = -INFINITY;
    for (; t <= ntiles; ++t) top(t, (t + STAGES - 1) % STAGES);
  }

  // --- waves 0 and 1 (ONCE: all eight) shared the rows: they leave their sums in LDS as rows, and all waves
  // combine and write them.  With M = max_w m_w the sums of wave w are rescaled by 2^(m_w - M).
  // Only rows that exist are touched, four elements of a row per thread, and a row leaves as one
  // contiguous piece.  Bound by one wave's instruction stream when wave 0 did it alone, for all 32
  // columns of its accumulators whether they were rows or not: 1.65 us from the last tile to the
  // last store.  One request of 2344 keys, 32/8 heads 13.0 -> 12.2 us; 32 requests of 2048..8192 keys,
  // 28/4 heads 71.4 -> 70.2 us.
  if constexpr (KP) {
    // (no fused multiply-add here: whether the rescaling and the sums below end up fused would
    // depend on how each variant of the kernel is scheduled, and the variants must agree bit
    // for bit)
#pragma clang fp contract(off)
    constexpr int kVec = D / 4;  // threads per row
    float* xo = reinterpret_cast<float*>(lds);      // [sharer][row] x kPitch
    float* xm = xo + kSharers * kMaxRows * kPitch;  // [sharer][row]
    float* xl = xm + kSharers * kMaxRows;           // [sharer][row][2 halves of the wave]
    __syncthreads();  // every wave is done with the tiles
    if (wave < kSharers && row_ok) {
      if constexpr (R16) {
        float* mine = xo + (wave * kMaxRows + i16) * kPitch + q4 * 4;
#pragma unroll
        for (int d = 0; d < D / 16; ++d) *reinterpret_cast<f32x4*>(mine + d * 16) = o16[d];
        if (q4 == 0) xm[wave * kMaxRows + i16] = m_run;
        const float pair = cross_quarter_sum(l_run);
        if ((q4 & 1) == 0) xl[(wave * kMaxRows + i16) * 2 + hi] = pair;
      } else {
        float* mine = xo + (wave * kMaxRows + i32) * kPitch + hi * 4;
#pragma unroll
        for (int d = 0; d < G::kDBlocks; ++d)
#pragma unroll
          for (int rr = 0; rr < 4; ++rr)
            *reinterpret_cast<f32x4*>(mine + d * 32 + rr * 8) =
                f32x4{o[d][rr * 4], o[d][rr * 4 + 1], o[d][rr * 4 + 2], o[d][rr * 4 + 3]};
        if (hi == 0) xm[wave * kMaxRows + i32] = m_run;
        xl[(wave * kMaxRows + i32) * 2 + hi] = l_run;
      }
    }
    __syncthreads();
    // N such pieces of as many rows at a time, so that their latencies pass together.  HALVES (eight sharers, up
    // to 8 rows of head dim 128 or 16 of 64, so that half of the threads would have no row): the halves of a wave
    // take four sharers each (short steps of up to 8 rows 1.5 % faster; where the rows take all threads 4-12 %
    // slower that way).
    auto write_rows = [&](auto n_c, auto halves_c, int first) __attribute__((always_inline)) {
      constexpr int N = decltype(n_c)::value;
      constexpr bool HALVES = decltype(halves_c)::value;
      constexpr int kLanes = HALVES ? 32 : 64;  // lanes of a wave that hold different elements
      constexpr int kMine = HALVES ? kSharers / 2 : kSharers;
      const int w0 = HALVES ? hi * kMine : 0;
      const int piece = wave * kLanes + (HALVES ? i32 : lane);
      const int c = piece % kVec * 4;
      int lr[N];
      float m_all[N], l_tot[N];
      f32x4 v[N];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        lr[i] = first + piece / kVec + i * (kLanes * WAVES / kVec);
        const int at = min(lr[i], it.row_count - 1);
        float m[kMine], a[kMine][2];
        f32x4 ow[kMine];
#pragma unroll
        for (int w = 0; w < kMine; ++w) {
          m[w] = xm[(w0 + w) * kMaxRows + at];
          a[w][0] = xl[((w0 + w) * kMaxRows + at) * 2];
          a[w][1] = xl[((w0 + w) * kMaxRows + at) * 2 + 1];
          ow[w] = *reinterpret_cast<const f32x4*>(xo + ((w0 + w) * kMaxRows + at) * kPitch + c);
        }
        m_all[i] = m[0];
#pragma unroll
        for (int w = 1; w < kMine; ++w) m_all[i] = fmaxf(m_all[i], m[w]);
        if constexpr (HALVES) m_all[i] = cross_half_max(m_all[i]);
        float l0 = 0.f, l1 = 0.f;
#pragma unroll
        for (int w = 0; w < kMine; ++w) {
          const float sc = (m[w] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m[w] - m_all[i]);
          l0 = w == 0 ? a[w][0] * sc : l0 + a[w][0] * sc;
          l1 = w == 0 ? a[w][1] * sc : l1 + a[w][1] * sc;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[i][e] = w == 0 ? ow[w][e] * sc : v[i][e] + ow[w][e] * sc;
        }
        l_tot[i] = l0 + l1;
        if constexpr (HALVES) {
          l_tot[i] = cross_half_sum(l_tot[i]);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[i][e] = cross_half_sum(v[i][e]);
        }
      }
      if (it.partial_slot < 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const float inv = p.out_scale / l_tot[i];
          const int r = it.row_begin + lr[i], tk = r / g;
          bf16x4 out4;
#pragma unroll
          for (int e = 0; e < 4; ++e) out4[e] = (__bf16)(v[i][e] * inv);
          if (lr[i] < it.row_count && (!HALVES || hi == 0))
            *reinterpret_cast<u32x2*>(
                p.out + ((int64_t)(rq.row_start + tk) * p.num_q_heads + it.kv_head * g + (r - tk * g)) * D + c) =
                __builtin_bit_cast(u32x2, out4);
        }
        return;
      }
#pragma unroll
      for (int i = 0; i < N; ++i) {
        // the row's largest magnitude: over the kVec neighbouring lanes that hold it
        const float amax = row_lanes_max<kVec>(
            fmaxf(fmaxf(fabsf(v[i][0]), fabsf(v[i][1])), fmaxf(fabsf(v[i][2]), fabsf(v[i][3]))));
        const float to_unit = amax > 0.f ? 1.f / amax : 0.f;  // (a row without visible keys in this part is all zero)
        typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
        f16x4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = (_Float16)(v[i][e] * to_unit);
        const int64_t prow = (int64_t)it.partial_slot * p.rows_per_item + lr[i];
        if (lr[i] >= it.row_count || (HALVES && hi)) continue;
        if (p.ticket_base >= 0) {
          // device-coherent stores: the workgroup that merges may sit on another XCD
          store_coherent_bits(p.part_o + prow * D + c, __builtin_bit_cast(uint64_t, h));
          if (c == 0) {
            store_coherent(p.part_ml + prow * 4, m_all[i], l_tot[i]);
            store_coherent(p.part_ml + prow * 4 + 2, amax, 0.f);
          }
        } else {
          *reinterpret_cast<uint64_t*>(p.part_o + prow * D + c) = __builtin_bit_cast(uint64_t, h);
          if (c == 0) *reinterpret_cast<f32x4*>(p.part_ml + prow * 4) = f32x4{m_all[i], l_tot[i], amax, 0.f};
        }
      }
    };
    // (The form for four pieces is compiled where a row count reaches it.  Leaving out the one for two as well,
    // where none does, moves the code behind it: one request of 2344 keys, 32 layers 349 -> 355 us.)
    constexpr int kRowsAtOnce = 64 * WAVES / kVec;
    if (ONCE && it.row_count <= kRowsAtOnce / 2) write_rows(std::integral_constant<int, 1>{}, std::bool_constant<ONCE>{}, 0);
    else if (it.row_count <= kRowsAtOnce) write_rows(std::integral_constant<int, 1>{}, std::false_type{}, 0);
    else if (it.row_count <= 2 * kRowsAtOnce) write_rows(std::integral_constant<int, 2>{}, std::false_type{}, 0);
    else if constexpr (kMaxRows > 2 * kRowsAtOnce)
      for (int r0 = 0; r0 < it.row_count; r0 += 4 * kRowsAtOnce) write_rows(std::integral_constant<int, 4>{}, std::false_type{}, r0);
  }

  // --- epilogue ---------------------------------------------------------------------
  if (!KP && wave_active) {
    const float l_tot = cross_half_sum(l_run);
    if (row_ok) {
      if (it.partial_slot < 0) {
        const float inv = p.out_scale / l_tot;
        int64_t out_off = q_off;
        if constexpr (PACK) {
          // formed again (the empty statement hides that it is known): held across the loop it
          // would be spilled
          int r = row;
          asm volatile("" : "+v"(r));
          const int t = r / g;
          out_off = ((int64_t)(rq.row_start + t) * p.num_q_heads + it.kv_head * g + (r - t * g)) * D;
        }
        uint16_t* dst = p.out + out_off;
#pragma unroll
        for (int d = 0; d < G::kDBlocks; ++d)
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)(o[d][rr * 4 + e] * inv);
            *reinterpret_cast<u32x2*>(dst + d * 32 + rr * 8 + hi * 4) = __builtin_bit_cast(u32x2, v);
          }
      } else {
        const int64_t prow = (int64_t)it.partial_slot * p.rows_per_item + local_row;
        uint16_t* dst = p.part_o + prow * D;
        // the row's largest magnitude (this lane holds half of the row, lane +-32 the other half)
        float amax = 0.f;
#pragma unroll
        for (int d = 0; d < G::kDBlocks; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) amax = fmaxf(amax, fabsf(o[d][r]));
        amax = cross_half_max(amax);
        const float to_unit = amax > 0.f ? 1.f / amax : 0.f;  // (a row without visible keys in this part is all zero)
#pragma unroll
        for (int d = 0; d < G::kDBlocks; ++d)
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) {
            typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
            f16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (_Float16)(o[d][rr * 4 + e] * to_unit);
            uint16_t* at = dst + d * 32 + rr * 8 + hi * 4;
            if (p.ticket_base >= 0) {
              // device-coherent stores: the workgroup that merges may sit on another XCD
              store_coherent_bits(at, __builtin_bit_cast(uint64_t, v));
            } else {
              *reinterpret_cast<uint64_t*>(at) = __builtin_bit_cast(uint64_t, v);
            }
          }
        if (hi == 0) {
          if (p.ticket_base >= 0) {
            store_coherent(p.part_ml + prow * 4, m_run, l_tot);
            store_coherent(p.part_ml + prow * 4 + 2, amax, 0.f);
          } else {
            *reinterpret_cast<f32x4*>(p.part_ml + prow * 4) = f32x4{m_run, l_tot, amax, 0.f};
          }
        }
      }
    }
  }
  // Split query tile: every workgroup publishes its partial result and takes a ticket; the one
  // that draws the last ticket finds all partial results visible, combines them and puts the
  // counter back to zero for the next launch.  The partial results travel through
  // device-coherent stores and loads (they bypass the per-XCD caches), so no cache-wide
  // write-back or invalidate is needed: the stores only have to be complete before the ticket
  // is drawn.
  if (it.partial_slot >= 0 && p.ticket_base >= 0) {
    const MergeItem mi = p.merges[it.merge_id];
    int32_t* ticket = (p.tickets ? p.tickets : g_tickets) + p.ticket_base + (it.merge_id << p.ticket_shift);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
    if (tid == 0)
      *s_last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == mi.nsplit - 1;
    __syncthreads();
    if (*s_last) {
      merge_rows<D, 8, true>(p, mi, tid, 64 * WAVES);
      if (tid == 0) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// Bound by the latency of two dependent reads (item, partial results) and by the loads it issues:
// most ranges are cut into two or three parts, so the group of parts read at once follows their
// number.
template <int D>
__global__ __launch_bounds__(256) void merge_kernel(const AttnParams p, const MergeItem* merges) {
  constexpr int ROWS = 256 / (D / 8);  // rows per workgroup
  const MergeItem mi = merges[blockIdx.x];
  // this workgroup's slice of the rows
  const int first = blockIdx.y * ROWS;
  if (first >= mi.row_count) return;
  const int last = min(mi.row_count, first + ROWS);
  if (mi.nsplit <= 2) merge_rows<D, 2, false>(p, mi, threadIdx.x, 256, first, last);
  else if (mi.nsplit <= 4) merge_rows<D, 4, false>(p, mi, threadIdx.x, 256, first, last);
  else merge_rows<D, 8, false>(p, mi, threadIdx.x, 256, first, last);
}

}  // namespace

namespace {

void fill_params(KernelArgs* args, const efim_batch_t* b, const Plan& plan, const char* header, const void* q,
                 const void* k_cache, const void* v_cache, void* out, float sm_scale, const CacheFormat& fmt,
                 char* partials) {
  args->items = reinterpret_cast<const DevItem*>(header + plan.off_items);
  args->block_table = b->block_table;
  args->q_rows = static_cast<const uint16_t*>(q);
  args->k_pages = static_cast<const uint16_t*>(k_cache);
  args->v_pages = static_cast<const uint16_t*>(v_cache);
  args->max_pages = b->max_pages_per_req;
  args->kv_heads = b->num_kv_heads;
  int page_shift = 0;
  while ((1 << page_shift) < b->page_size) ++page_shift;
  args->shape = b->num_q_heads / b->num_kv_heads | page_shift << 8;
  args->static_items = (int32_t)plan.items.size();
  AttnParams* const p = &args->p;
  p->out = static_cast<uint16_t*>(out);
  p->part_o = reinterpret_cast<uint16_t*>(partials + plan.off_part_o);
  p->part_ml = reinterpret_cast<float*>(partials + plan.off_part_ml);
  p->num_q_heads = b->num_q_heads;
  p->group = b->num_q_heads / b->num_kv_heads;
  p->rows_per_item = plan.partial_rows;
  p->scale_log2 = sm_scale * 1.4426950408889634f;
  p->out_scale = 1.f;
  p->k_inv = 1.0 / (double)fmt.k_scale;
  p->v_inv = 1.0 / (double)fmt.v_scale;
  if (fmt.fp8) {
    p->scale_log2 *= fmt.k_scale;
    p->out_scale = fmt.v_scale;
  }
  p->k_new = nullptr;
  p->v_new = nullptr;
  p->k_cache_w = nullptr;
  p->v_cache_w = nullptr;
  p->ticket_base = -1;
  p->ticket_shift = ticket_shift(plan.merges.size());
  p->tickets = nullptr;
  p->queue_at = 0;
  p->queued_items = p->draws = 0;
  p->merges = reinterpret_cast<const MergeItem*>(header + plan.off_merges);
  p->interleaved = 0;
  p->rotary_dim = b->head_dim;
  for (double& f : p->inv_freq) f = 0.0;
}

}  // namespace

namespace {

// Split key ranges are combined inside the main kernel or by merge_kernel in a second launch.
// In-kernel merging sends the partial results through device-coherent (write-through) stores;
// that pays when every tile has very few rows (decode steps of the usual head groupings),
// where it saves a launch, and costs more than the launch as the rows grow, so by default it is used
// when no work item has more than 8 query rows.  4 layers, second launch / in the kernel, us: 16 requests of
// 3000 keys 4 rows 158.4 / 157.0, 8 rows 161.2 / 159.7, 14 rows 99.4 / 99.4 (28/4 heads), 16 rows 167.8 / 169.8, 32
// rows 183.0 / 188.4; two calls 4 rows 173.9 / 172.9, 8 rows 175.0 / 176.2, 16 rows 178.6 / 184.1; four of 4000..5000
// over codes, 4 rows 61.9 / 58.7.  Many parts per range cost the kernel a round of reads for every eight: two requests
// of 2344 keys, ten parts, 4 rows 43.0 / 43.2; head dim 64 gains up to 16 rows with few parts (99.9 / 98.1) and loses
// as much with ten (37.7 / 38.6).
constexpr int kTicketMergeMaxRows = 8;
bool use_tickets(const Plan& plan) {
  const int knob = tuning().fused_merge;
  const bool want = knob < 0 ? plan.max_item_rows <= kTicketMergeMaxRows : knob != 0;
  return want && !plan.merges.empty() && plan.merges.size() < (size_t)kTicketsPerSlot;
}

// Workgroups of a launch; with a launch token, whose block of counters is this launch's alone, the plan's queued items
// may be drawn.  (A plan object's launches have none: a counter in the workspace would be
// shared by launches of one plan that run at the same time, which where no range is cut only read it.  16 requests of
// 1024..4096 keys, one new token, 32/32 heads: 118.0 us as a plan object, 116.2 when it could draw.)
unsigned workgroups(const Plan& plan, bool fp8, int stage_slot, KernelArgs* args) {
  if (stage_slot < 0 || !plan_draws(plan, fp8)) return (unsigned)plan.items.size();
  args->static_items = plan.static_items;
  args->p.queue_at = (stage_slot + 1) * kTicketsPerSlot - 1;
  args->p.queued_items = plan.queued_items;
  args->p.draws = plan.draws;
  return (unsigned)(plan.static_items + plan.draws);
}

__global__ void zero_words_kernel(int32_t* words, size_t count) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) words[i] = 0;
}

// The kernel's arguments.  Those in front of the struct are in scalar registers when a wave starts (the build asks
// for that), so that the work item is the first thing it waits for; the rest is asked for beside the work item.  One
// request of 2344 keys, 32 layers 347 us, without the first 357, without the second 361; 298 requests of 199..408
// keys, head dim 64, over codes 39.4 / 39.6 / 40.6; 32 of 2048..8192, 28/4 heads, 16 layers 1131 / 1135 / 1134.
static_assert(std::is_same<decltype(&extend_attention_kernel<128, 4, 2, true, false, true>),
                           void (*)(decltype(KernelArgs::items), decltype(KernelArgs::block_table), decltype(KernelArgs::q_rows),
                                    decltype(KernelArgs::k_pages), decltype(KernelArgs::v_pages), decltype(KernelArgs::max_pages),
                                    decltype(KernelArgs::kv_heads), decltype(KernelArgs::shape),
                                    decltype(KernelArgs::static_items), decltype(KernelArgs::p))>::value,
              "KernelArgs describes the kernel's parameters");
#define EFIM_ARGS(a) a.items, a.block_table, a.q_rows, a.k_pages, a.v_pages, a.max_pages, a.kv_heads, a.shape, a.static_items, a.p

// Key-parallel kernels: no work item has more than 32 query rows (R16, Plan::rows16: 16), always so for the decode step.
// Four-wave kernels take two stages over bf16 rows and three over 8-bit rows, where a tile is half
// as large.  The short step with head dim 64 takes the third stage with more than three work items
// per compute unit: with two stages three workgroups fit a unit, with three only two, whose
// deeper look-ahead then wins over a third round that is mostly empty.  Measured (us, two stages /
// three): 976 items of 14 tiles 45.3 / 42.4, 1012 of 28 tiles 102.5 / 91.4; up to 520 items two
// are better, 512 of 10 tiles 25.1 / 32.0, 520 of 8 tiles (four layers) 68.7 / 82.8, 320 of 4
// tiles 15.3 / 16.1.  The plain call over the same rows is not faster with three.
template <bool FUSED, bool R16>
void launch_key_parallel(int head_dim, bool wide, bool fp8, bool crowded, bool once, dim3 grid, const KernelArgs& args,
                         hipStream_t stream) {
#define EFIM_KP(DD, WAVES, STAGES, F8, P8, ONCE) \
  extend_attention_kernel<DD, WAVES, STAGES, FUSED, F8, true, false, P8, ONCE, R16><<<grid, 64 * (WAVES), 0, stream>>>(EFIM_ARGS(args))
#define EFIM_KP_FORMS(DD, F8, P8)                            \
  do {                                                       \
    if (wide) EFIM_KP(DD, 8, 3, F8, P8, false);              \
    else EFIM_KP(DD, 4, F8 ? 3 : 2, F8, P8, false);          \
  } while (0)
  const bool two_pages = fp8 && head_dim == 64 && args.shape >> 8 == 3;  // a load spans two pages
  if (two_pages) {
    EFIM_KP_FORMS(64, true, true);
  } else if (once) {
    if (head_dim == 128) {
      if (fp8) EFIM_KP(128, 8, once_tiles(128), true, false, true); else EFIM_KP(128, 8, once_tiles(128), false, false, true);
    } else {
      if (fp8) EFIM_KP(64, 8, once_tiles(64), true, false, true); else EFIM_KP(64, 8, once_tiles(64), false, false, true);
    }
  } else if (head_dim == 128) {
    if (fp8) EFIM_KP_FORMS(128, true, false); else EFIM_KP_FORMS(128, false, false);
  } else if (fp8) {
    EFIM_KP_FORMS(64, true, false);
  } else if (FUSED && crowded && !wide) {
    if constexpr (FUSED) EFIM_KP(64, 4, 3, false, false, false);
  } else {
    EFIM_KP_FORMS(64, false, false);
  }
#undef EFIM_KP_FORMS
#undef EFIM_KP
}

template <bool FUSED>
void launch_kernel(int head_dim, const Plan& plan, bool fp8, dim3 grid, const KernelArgs& args, hipStream_t stream) {
  const bool wide = plan.rows_per_item == 256, crowded = plan.crowded;
  if (FUSED || plan.max_item_rows <= 32) {
    if (plan.rows16) launch_key_parallel<FUSED, true>(head_dim, wide, fp8, crowded, plan.once, grid, args, stream);
    else launch_key_parallel<FUSED, false>(head_dim, wide, fp8, crowded, plan.once, grid, args, stream);
    return;
  }
#define EFIM_PIPE(DD, F8, PACK, P8)                                                                            \
  do {                                                                                                        \
    if (wide) extend_attention_kernel<DD, 8, 3, false, F8, false, PACK, P8><<<grid, 512, 0, stream>>>(EFIM_ARGS(args));       \
    else extend_attention_kernel<DD, 4, F8 ? 3 : 2, false, F8, false, PACK, P8><<<grid, 256, 0, stream>>>(EFIM_ARGS(args));  \
  } while (0)
  if (head_dim == 128) {
    if (fp8) EFIM_PIPE(128, true, false, false); else EFIM_PIPE(128, false, false, false);
  } else if (fp8) {
    if (args.shape >> 8 == 3) EFIM_PIPE(64, true, false, true); else EFIM_PIPE(64, true, false, false);
  } else {
    if (crowded) EFIM_PIPE(64, false, true, false); else EFIM_PIPE(64, false, false, false);
  }
#undef EFIM_PIPE
}

int launch_merge(const efim_batch_t* b, const Plan& plan, const AttnParams& p, hipStream_t stream) {
  const dim3 mgrid((unsigned)plan.merges.size(), (unsigned)((plan.partial_rows * (b->head_dim / 8) + 255) / 256));
  if (b->head_dim == 128) merge_kernel<128><<<mgrid, 256, 0, stream>>>(p, p.merges);
  else merge_kernel<64><<<mgrid, 256, 0, stream>>>(p, p.merges);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_hip_error(e); return EFIM_ERR_LAUNCH; }
  return EFIM_OK;
}

}  // namespace

bool plan_merges_in_kernel(const Plan& plan) { return use_tickets(plan); }

int launch_zero_words(int32_t* words, size_t count, hipStream_t stream) {
  if (count == 0) return EFIM_OK;
  zero_words_kernel<<<dim3((unsigned)((count + 255) / 256)), 256, 0, stream>>>(words, count);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) { set_last_hip_error(e); return EFIM_ERR_LAUNCH; }
  return EFIM_OK;
}

int launch_extend_attention(const efim_batch_t* b, const Plan& plan, const char* header, int stage_slot,
                            const void* q, const void* k_cache, const void* v_cache, void* out,
                            float sm_scale, const CacheFormat& fmt, void* workspace, hipStream_t stream,
                            int32_t* tickets, bool quiet) {
  KernelArgs args;
  AttnParams& p = args.p;
  fill_params(&args, b, plan, header, q, k_cache, v_cache, out, sm_scale, fmt, static_cast<char*>(workspace));
  if (tickets) {
    p.tickets = tickets;
    p.ticket_base = 0;
  } else if (stage_slot >= 0 && use_tickets(plan)) {
    p.ticket_base = stage_slot * kTicketsPerSlot;
  }

  const dim3 grid(workgroups(plan, fmt.fp8, stage_slot, &args));
  Tuning tn = tuning();
  if (quiet) tn.ev_start = tn.ev_stop = nullptr;
  if (tn.ev_start) (void)hipEventRecord(tn.ev_start, stream);
  launch_kernel<false>(b->head_dim, plan, fmt.fp8, grid, args, stream);
  hipError_t e = hipGetLastError();
  if (tn.ev_stop) (void)hipEventRecord(tn.ev_stop, stream);
  if (e != hipSuccess) { set_last_hip_error(e); return EFIM_ERR_LAUNCH; }
  if (!plan.merges.empty() && p.ticket_base < 0) return launch_merge(b, plan, p, stream);
  return EFIM_OK;
}

int launch_decode_step(const efim_batch_t* b, const Plan& plan, const char* header, int stage_slot,
                       const void* q, const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                       void* out, const double* inv_freq, int rotary_dim, int interleaved, float sm_scale,
                       const CacheFormat& fmt, void* workspace, hipStream_t stream, int32_t* tickets, bool quiet) {
  KernelArgs args;
  AttnParams& p = args.p;
  fill_params(&args, b, plan, header, q, k_cache, v_cache, out, sm_scale, fmt, static_cast<char*>(workspace));
  if (tickets) {
    p.tickets = tickets;
    p.ticket_base = 0;
  } else if (stage_slot >= 0 && use_tickets(plan)) {
    p.ticket_base = stage_slot * kTicketsPerSlot;
  }
  p.k_new = static_cast<const uint16_t*>(k_new);
  p.v_new = static_cast<const uint16_t*>(v_new);
  p.k_cache_w = static_cast<uint16_t*>(k_cache);
  p.v_cache_w = static_cast<uint16_t*>(v_cache);
  p.interleaved = interleaved;
  p.rotary_dim = rotary_dim;
  const int D = b->head_dim;
  for (int j = 0; j < rotary_dim / 2; ++j) p.inv_freq[j] = inv_freq[j];

  const dim3 grid(workgroups(plan, fmt.fp8, stage_slot, &args));
  Tuning tn = tuning();
  if (quiet) tn.ev_start = tn.ev_stop = nullptr;
  if (tn.ev_start) (void)hipEventRecord(tn.ev_start, stream);
  launch_kernel<true>(D, plan, fmt.fp8, grid, args, stream);
  hipError_t e = hipGetLastError();
  if (tn.ev_stop) (void)hipEventRecord(tn.ev_stop, stream);
  if (e != hipSuccess) { set_last_hip_error(e); return EFIM_ERR_LAUNCH; }
  if (!plan.merges.empty() && p.ticket_base < 0) return launch_merge(b, plan, p, stream);
  return EFIM_OK;
}

}  // namespace efim
