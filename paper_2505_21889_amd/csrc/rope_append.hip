// efim_rope_append: rotary embedding of the new tokens at their offset positions and
// append of their K/V into the paged cache (EFIM Sec. 1 / Sec. 3.1: the incremental tokens
// come after the cached <P>prefix<S>suffix<M>, so token i of request r sits at position
// C_r + i).  Streaming kernel, bound by HBM bandwidth: 2*(Hq + 2*Hkv)*D*2 bytes per token.
//
// The rotation is done in fp64 and rounded once to bf16 so that the cache contents agree
// bit for bit with a double-precision definition.
//
// KV8 variant: the caches hold E4M3 codes (one byte per element, same [page, head, slot, D]
// layout); the rotated key (after its rounding to bf16) and the value are divided by the
// tensor's scale and rounded to the nearest code on their way out.
#include "efim_internal.h"
#include "fp8_math.h"
#include "rope_math.h"

namespace efim {
namespace {

constexpr int kThreads = kAppendThreads;
constexpr int kPasses = kAppendPasses;
constexpr int kMaxReqPerLaunch = 384;

template <int MAXREQ>
struct RopeArgs {
  double inv_freq[64];            // rotation frequency of pair j (rotary_dim/2 entries)
  int32_t cached[MAXREQ];         // C_r of the requests of this launch
  int32_t row_start[MAXREQ + 1];  // first packed row of each request, and the end
  int32_t nreq;
  int32_t tokens;                 // new tokens of this launch
  int32_t tok_shift;              // log2 of the tokens of a workgroup
  int32_t parts;                  // waves per token in a workgroup
  int32_t req_base;               // index of the first request (block_table row)
  int32_t max_pages;
  int32_t num_q_heads;            // 0 where there are no queries to rotate
  int32_t num_kv_heads;
  int32_t rotary_dim;             // leading elements of a head row that are rotated
  int32_t page_shift;             // log2 of the page size (tokens per page)
  double k_inv;                   // 8-bit caches: 1 / scale (code = value / scale)
  double v_inv;
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// E4M3 codes of eight bf16 values; inv = 1 / (double)scale.
__device__ __forceinline__ u32x2 quantize8(u32x4 x, double inv) {
  float f[8];
  bool nan = false;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    f[2 * t] = bf16_quotient(x[t] << 16, inv);
    f[2 * t + 1] = bf16_quotient(x[t] & 0xFFFF0000u, inv);
    nan |= __builtin_isunordered(f[2 * t], f[2 * t + 1]);
  }
  u32x2 r;
#pragma unroll
  for (int t = 0; t < 2; ++t)
    r[t] = e4m3_pair<true>(f[4 * t + 2], f[4 * t + 3], e4m3_pair<false>(f[4 * t], f[4 * t + 1], 0u));
  if (nan) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
      r[t] = f32_to_e4m3(f[4 * t]) | (f32_to_e4m3(f[4 * t + 1]) << 8) | (f32_to_e4m3(f[4 * t + 2]) << 16) |
             (f32_to_e4m3(f[4 * t + 3]) << 24);
  }
  return r;
}

// Rotates the eight pairs of a unit.  The results go through fp32 two at a time; the one pattern for
// which that could round twice is looked for once per unit (one unit in 4000 has it) and the unit
// then done again value by value.  (With the check and the integer rounding at every value they
// were half of the kernel's instructions.)
template <bool INTERLEAVED>
__device__ __forceinline__ void rotate_units(u32x4& a, u32x4& b, const double (&cs)[8], const double (&sn)[8]) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  uint32_t x1[8], x2[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    // INTERLEAVED: 16 consecutive elements = pairs 0..7, stored (even, odd)
    const uint32_t w = INTERLEAVED ? (t < 4 ? a[t & 3] : b[t & 3]) : a[t >> 1];
    const uint32_t v = INTERLEAVED ? w : b[t >> 1];
    x1[t] = INTERLEAVED || !(t & 1) ? w & 0xFFFFu : w >> 16;
    x2[t] = INTERLEAVED || (t & 1) ? v >> 16 : v & 0xFFFFu;
  }
  float f1[8], f2[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    double y1, y2;
    rotate_pair_f64(x1[t], x2[t], cs[t], sn[t], &y1, &y2);
    f1[t] = (float)y1;
    f2[t] = (float)y2;
  }
  u16x2 off = __builtin_bit_cast(u16x2, off_midpoint(f1[0], f2[0]));
#pragma unroll
  for (int t = 1; t < 8; ++t)
    off = __builtin_elementwise_min(off, __builtin_bit_cast(u16x2, off_midpoint(f1[t], f2[t])));
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    a[t] = INTERLEAVED ? pack_bf16(f1[t], f2[t]) : pack_bf16(f1[2 * t], f1[2 * t + 1]);
    b[t] = INTERLEAVED ? pack_bf16(f1[4 + t], f2[4 + t]) : pack_bf16(f2[2 * t], f2[2 * t + 1]);
  }
  if (off[0] == 0 || off[1] == 0) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      uint32_t y1, y2;
      rotate_pair_bf16(x1[t], x2[t], cs[t], sn[t], &y1, &y2);
      x1[t] = y1;
      x2[t] = y2;
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      a[t] = INTERLEAVED ? x1[t] | (x2[t] << 16) : x1[2 * t] | (x1[2 * t + 1] << 16);
      b[t] = INTERLEAVED ? x1[4 + t] | (x2[4 + t] << 16) : x2[2 * t] | (x2[2 * t + 1] << 16);
    }
  }
}

// A wave takes one token and kPasses passes of 64 / (D / 16) head rows of it (a unit is 16 bytes of one head
// row together with its partner 16 bytes; a lane has the same place in the row in every pass, so that
// it needs the cosines and sines of the same eight pairs).
//
// Up to some ten thousand tokens the kernel is as long as one wave's chain: request of the token, page,
// cosines, rows.  All loads that need no answer of another go out first -- the request table (64
// requests per load, the position found by a ballot), the frequency, the wave's rows -- and the page id
// and the cosines (one pair per lane, exchanged through LDS inside the wave, no barrier) are formed
// while the rows are on their way.  Before, a workgroup searched the table with one dependent load per
// step, evaluated the cosines with one of its four waves and read the rows behind a barrier.  us, before / now,
// passes over the same buffers: 2176 tokens of 16 requests, 32/8 heads 18.6 / 15.0 (other buffers every
// pass); 1113 tokens, 32/32 heads 11.2 / 9.1; 1014 tokens, 28/4 heads 6.7 / 5.5 (5 us of it the host's), 8-bit
// cache 8.7 / 5.8; 87286 tokens, 32/8 heads 419 / 394 = 5.4 TB/s.  One pass per wave is 6-10 % slower
// at 1000 to 2000 tokens, three 0-5 % either way.
template <int D, bool INTERLEAVED, bool KV8, int MAXREQ>
__global__ __launch_bounds__(kThreads) void rope_append_kernel(
    const RopeArgs<MAXREQ> args, uint16_t* __restrict__ q, const uint16_t* __restrict__ k_new,
    const uint16_t* __restrict__ v_new, void* __restrict__ k_cache_raw,
    void* __restrict__ v_cache_raw, const int32_t* __restrict__ block_table) {
#pragma clang fp contract(off)
  constexpr int HALF = D / 2;
  constexpr int UNITS_PER_ROW = D / 16;
  constexpr int ROWS_PER_PASS = 64 / UNITS_PER_ROW;
  __shared__ __attribute__((aligned(16))) double s_cs[kThreads / 64][HALF][2];  // (cos, sin) of the wave's token

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tok = (blockIdx.x << args.tok_shift) + (wave & ((1 << args.tok_shift) - 1));
  if (tok >= args.tokens) return;
  const int part = blockIdx.y * args.parts + (wave >> args.tok_shift);
  const int row = args.row_start[0] + tok;
  const int rot_half = args.rotary_dim / 2;  // pairs per head row (D/2 when the whole row rotates)

  const int nreq = args.nreq;
  int32_t starts[MAXREQ / 64], lens[MAXREQ / 64];
#pragma unroll
  for (int i = 0; i < MAXREQ / 64; ++i) {
    const int r = i * 64 + lane;
    starts[i] = args.row_start[min(r, nreq)];
    lens[i] = args.cached[min(r, nreq - 1)];
  }
  const double freq = args.inv_freq[lane % HALF];

  const int hq = args.num_q_heads, hkv = args.num_kv_heads;
  const int rows_per_tok = hq + 2 * hkv;
  const int cp = lane % UNITS_PER_ROW;
  const bool in_rotary = cp * 16 < args.rotary_dim;
  // element offsets of the unit's two chunks inside the head row: inside the rotated part, for rotate-half
  // the chunk rotary_dim/2 elements further on, for interleaved pairing the next chunk.  Units
  // behind the rotated part (and all of V) are plain copies of two neighbouring chunks.
  const bool apart = !INTERLEAVED && in_rotary;
  const int e0 = apart ? cp * 8 : cp * 16, e1 = apart ? cp * 8 + rot_half : cp * 16 + 8;
  const int hr0 = part * (kPasses * ROWS_PER_PASS) + lane / UNITS_PER_ROW;
  u32x4 a[kPasses], b[kPasses];
#pragma unroll
  for (int i = 0; i < kPasses; ++i) {
    // (0..Hq-1: q heads, then Hkv k heads, then Hkv v heads)
    const int hr = min(hr0 + i * ROWS_PER_PASS, rows_per_tok - 1);
    const uint16_t* src = k_new + ((int64_t)row * hkv + (hr - hq)) * D;
    if (hr < hq) src = q + ((int64_t)row * hq + hr) * D;
    if (hr >= hq + hkv) src = v_new + ((int64_t)row * hkv + (hr - hq - hkv)) * D;
    a[i] = *reinterpret_cast<const u32x4*>(src + e0);
    b[i] = *reinterpret_cast<const u32x4*>(src + e1);
  }

  // request of this row: the last r with row_start[r] <= row
  int req = -1;
#pragma unroll
  for (int i = 0; i < MAXREQ / 64; ++i)
    req += __popcll(__ballot(i * 64 + lane < nreq && starts[i] <= row));
  int pos = 0;
#pragma unroll
  for (int i = 0; i < MAXREQ / 64; ++i)
    if (MAXREQ == 64 || req >> 6 == i)
      pos = __builtin_amdgcn_readlane(lens[i], req & 63) + row - __builtin_amdgcn_readlane(starts[i], req & 63);
  const int32_t page_id = block_table[(int64_t)(args.req_base + req) * args.max_pages + (pos >> args.page_shift)];
  if (lane < rot_half) {
    double s, c;
    sincos((double)pos * freq, &s, &c);
    s_cs[wave][lane][0] = c;
    s_cs[wave][lane][1] = s;
  }
  // (one wave writes and reads: its LDS accesses are in order, the compiler is told by the fence)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  double cs[8], sn[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    cs[t] = s_cs[wave][cp * 8 + t][0];
    sn[t] = s_cs[wave][cp * 8 + t][1];
  }
  // element offset of (page, head 0, slot, 0) in the caches
  const int64_t slot = ((((int64_t)page_id * hkv) << args.page_shift) + (pos & ((1 << args.page_shift) - 1))) * D;

#pragma unroll
  for (int i = 0; i < kPasses; ++i) {
    const int hr = hr0 + i * ROWS_PER_PASS;
    const bool is_q = hr < hq, is_k = !is_q && hr < hq + hkv;
    if (in_rotary && hr < hq + hkv) rotate_units<INTERLEAVED>(a[i], b[i], cs, sn);
    if (hr >= rows_per_tok) continue;
    const int64_t cache_off = slot + (((int64_t)(hr - hq - (is_k ? 0 : hkv)) * D) << args.page_shift);
    if (KV8 && !is_q) {
      uint8_t* row8 = static_cast<uint8_t*>(is_k ? k_cache_raw : v_cache_raw) + cache_off;
      const double inv = is_k ? args.k_inv : args.v_inv;
      *reinterpret_cast<u32x2*>(row8 + e0) = quantize8(a[i], inv);
      *reinterpret_cast<u32x2*>(row8 + e1) = quantize8(b[i], inv);
    } else {
      uint16_t* dst = is_q ? q + ((int64_t)row * hq + hr) * D
                           : static_cast<uint16_t*>(is_k ? k_cache_raw : v_cache_raw) + cache_off;
      *reinterpret_cast<u32x4*>(dst + e0) = a[i];
      *reinterpret_cast<u32x4*>(dst + e1) = b[i];
    }
  }
}

template <int MAXREQ>
int launch_with(const efim_batch_t* b, void* q, const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                const double* inv_freq, int rotary_dim, int interleaved, const CacheFormat& fmt, hipStream_t stream) {
  const int D = b->head_dim;
  RopeArgs<MAXREQ> args;
  for (int j = 0; j < 64; ++j) args.inv_freq[j] = j < rotary_dim / 2 ? inv_freq[j] : 0.0;
  args.rotary_dim = rotary_dim;
  args.page_shift = 0;
  while ((1 << args.page_shift) < b->page_size) ++args.page_shift;
  args.max_pages = b->max_pages_per_req;
  // Keys only: a token has no query rows.  (Skipped one by one they cost waves that load, rotate and drop them: 32/8
  // heads of 128, 16384 tokens 45.7 us against 22.5, 87286 tokens 202 against 139.)
  args.num_q_heads = q ? b->num_q_heads : 0;
  args.num_kv_heads = b->num_kv_heads;
  args.k_inv = 1.0 / (double)fmt.k_scale;
  args.v_inv = 1.0 / (double)fmt.v_scale;

  int64_t row = 0;
  for (int r0 = 0; r0 < b->batch; r0 += MAXREQ) {
    const int n = (b->batch - r0 < MAXREQ) ? b->batch - r0 : MAXREQ;
    const int64_t first = row;
    for (int i = 0; i < n; ++i) {
      args.cached[i] = b->cached_len[r0 + i];
      args.row_start[i] = (int32_t)row;
      row += b->new_len[r0 + i];
    }
    args.row_start[n] = (int32_t)row;
    args.nreq = n;
    args.req_base = r0;
    const int64_t ntok = row - first;
    if (ntok == 0) continue;
    args.tokens = (int32_t)ntok;
    const AppendShape shape = append_shape(ntok, args.num_q_heads + 2 * b->num_kv_heads, D);
    args.parts = shape.parts;
    args.tok_shift = shape.tok_shift;
    const dim3 grid(shape.x, shape.y);
    auto qp = static_cast<uint16_t*>(q);
    auto kn = static_cast<const uint16_t*>(k_new);
    auto vn = static_cast<const uint16_t*>(v_new);
#define EFIM_ROPE_LAUNCH3(DD, IL, F8)                                                                       \
  rope_append_kernel<DD, IL, F8, MAXREQ><<<grid, 64 * args.parts << args.tok_shift, 0, stream>>>(args, qp, kn, vn, k_cache, \
                                                                                                v_cache, b->block_table)
#define EFIM_ROPE_LAUNCH(DD, IL) \
  do { if (fmt.fp8) EFIM_ROPE_LAUNCH3(DD, IL, true); else EFIM_ROPE_LAUNCH3(DD, IL, false); } while (0)
    if (D == 128) {
      if (interleaved) EFIM_ROPE_LAUNCH(128, true); else EFIM_ROPE_LAUNCH(128, false);
    } else {
      if (interleaved) EFIM_ROPE_LAUNCH(64, true); else EFIM_ROPE_LAUNCH(64, false);
    }
#undef EFIM_ROPE_LAUNCH
#undef EFIM_ROPE_LAUNCH3
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_last_hip_error(e); return EFIM_ERR_LAUNCH; }
  }
  return EFIM_OK;
}

}  // namespace

int launch_rope_append(const efim_batch_t* b, int64_t total_new, void* q, const void* k_new,
                       const void* v_new, void* k_cache, void* v_cache, const double* inv_freq,
                       int rotary_dim, int interleaved, const CacheFormat& fmt, hipStream_t stream) {
  (void)total_new;
  auto* launch = b->batch <= 64 ? launch_with<64> : launch_with<kMaxReqPerLaunch>;
  return launch(b, q, k_new, v_new, k_cache, v_cache, inv_freq, rotary_dim, interleaved, fmt, stream);
}

}  // namespace efim
