// Shared between the kernel translation units: kernel arguments, storage types, cross-lane helpers, loads of the
// caches and the walk over a sequence's interval list.
#ifndef SPAN_DEVICE_H_
#define SPAN_DEVICE_H_

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "span_attn.h"
#include "span_internal.h"

namespace spanattn {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kThreads = kWavesPerBlock * 64;
constexpr int kWin = 256;  // rows of a wave whose positions are tabulated at a time (one LDS window)

struct LaunchArgs {
  const void* q;
  const void* k;
  const void* v;
  float* out;
  const int32_t* offsets;
  const int32_t* starts;
  const int32_t* ends;
  const int32_t* ctx_lens;
  const void* k_new;           // append variant: the new token's K / V rows [batch, heads, D], else null
  const void* v_new;
  const int32_t* append_pos;   // append variant: [batch] cache row that receives them
  const int32_t* q_pos;        // few-query variant: [batch] cache position of query token 0 (causal limit), or null
  int32_t* counters;  // [batch*heads] arrival tickets of the slices, counter_stride words apart; zero between calls
  // one slot per workgroup, slot = (first slice row of the sequence + slice) * heads + head:
  float* part_ml;   // [slots, NQ, 2]  (m in log2 units, l)
  float* part_acc;  // [slots, NQ, D]  un-normalised
  int32_t heads, max_len, num_intervals, slice_tokens, num_splits, max_tokens;
  int32_t q_len;                    // query tokens per sequence in q and out ([batch, q_len, heads, D])
  int32_t q_first;                  // matrix kernel: first query token this launch handles
  float scale_log2e;
  int32_t total_slices;             // table mode: entries of `table` in use
  int32_t even;                     // > 0: a sequence's slices share its own token count evenly, `even` positions each at least; 0: slice_tokens each
  int32_t entry_bits;               // table mode: Deal::b_bits | n_bits << 8 | dealt << 16
  int32_t counter_stride;
  int32_t intervals_per_seq;        // mean, in 65536ths, for list_window; -1: no window
  int32_t interleave;               // 1: rows dealt to the waves round-robin (large slices); 0: contiguous quarters
#ifdef SPAN_PHASE_TRACE
  unsigned long long* trace;        // diagnostic build only: [trace_workgroups, kTraceStamps] times of the phases, or null
  size_t trace_workgroups;
#endif
};
// Table mode: blockIdx.y indexes `table` (sequences have different numbers of slices).  The table makes
// the kernel arguments 3 KB larger, which costs about 0.35 us per launch, so calls that do not need it
// (every sequence has the same number of slices) use the plain arguments and a (heads, slices, batch) grid.
struct LaunchArgsTable : LaunchArgs {
  static constexpr bool kHasTable = true;
  static constexpr bool kHasRuns = false;
  uint32_t table[kMaxPlanSlices];   // read by slice_name alone: dealt entries have other fields than pack_slice's, and any order
};
struct LaunchArgsPlain : LaunchArgs {
  static constexpr bool kHasTable = false;
  static constexpr bool kHasRuns = false;
};
// Run mode: blockIdx.y indexes the slices of all sequences, each resolved on the host to its runs of consecutive
// cache positions; the kernel reads no span metadata from device memory.
struct LaunchArgsRuns : LaunchArgs {
  static constexpr bool kHasTable = true;
  static constexpr bool kHasRuns = true;
  RunTables r;
};

// What a table entry names.
struct SliceName {
  int b, split, nsl;  // sequence, slice within it, slices of the sequence
  int y0;             // slot of the sequence's first slice
};
__device__ __forceinline__ SliceName slice_name(const LaunchArgs& a, uint32_t entry, int y) {
  const int bits = a.entry_bits, b_bits = bits & 255, n_bits = bits >> 8 & 255;
  const uint32_t in_n = (1u << n_bits) - 1u;
  const int split = (int)(entry >> b_bits & in_n);
  const int slot = bits >> 16 ? (int)(entry >> (32 - kSlotBits)) : y;
  return SliceName{(int)(entry & ((1u << b_bits) - 1u)), split, (int)(entry >> (b_bits + n_bits) & in_n), slot - split};
}

// Diagnostic build (-DSPAN_PHASE_TRACE): every workgroup reads the constant-rate (100 MHz) clock at the phase
// boundaries named below into registers and thread 0 writes them out when the workgroup ends, so that taking a stamp
// puts no memory operation into the path it measures.  Each stamp names a value that must have been computed before
// the clock is read (the compiler may not move the read ahead of it).  The regular build compiles the stamps away.
// stamps: 0 kernel entry, 10 the sequence's interval range read (device lists), 1 span metadata read and slice known,
// 2 first position table built, 3 first K / V rows consumed, 4 all rows consumed, 5 waves merged in LDS, 6 output row
// stored and acknowledged (one slice per pair), 7 partial state published and acknowledged, 8 ticket returned,
// 9 slices merged, output row stored and acknowledged (last arrival only)
constexpr int kTraceStamps = 16;
#ifdef SPAN_PHASE_TRACE
#define SPAN_TRACE_DECL unsigned long long trace_t[11] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}
#define SPAN_STAMP_AFTER(i, constraint, value)        \
  do {                                                \
    asm volatile("" ::constraint(value) : "memory");  \
    trace_t[i] = wall_clock64();                      \
    asm volatile("" ::: "memory");                    \
  } while (0)
#define SPAN_STAMP_ACKED(i)                                  \
  do {                                                       \
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); \
    trace_t[i] = wall_clock64();                             \
    asm volatile("" ::: "memory");                           \
  } while (0)
#define SPAN_TRACE_FLUSH()                                                                                     \
  do {                                                                                                         \
    const size_t wg_ = (size_t)(blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;                 \
    if (threadIdx.x == 0 && a.trace && wg_ < a.trace_workgroups) {                                             \
      for (int i_ = 0; i_ < 11; ++i_) a.trace[wg_ * kTraceStamps + i_] = trace_t[i_];                          \
    }                                                                                                          \
  } while (0)
#else
#define SPAN_TRACE_DECL \
  do {                  \
  } while (0)
#define SPAN_STAMP_AFTER(i, constraint, value) \
  do {                                         \
  } while (0)
#define SPAN_STAMP_ACKED(i) \
  do {                      \
  } while (0)
#define SPAN_TRACE_FLUSH() \
  do {                     \
  } while (0)
#endif

// matrix kernel, 16-bit types: q stays as stored but for the sign of the score scale; with scale 0 it becomes 0, and what is
// not finite NaN, which is what the scaled scores are.
struct HalfQuery {
  static __device__ __forceinline__ float post_scale(float scale) { return scale == 0.f ? 1.f : fabsf(scale); }
  template <uint32_t kExponent>  // exponent bits of a value
  static __device__ __forceinline__ uint32_t scaled(uint32_t q, float scale) {
    if (__builtin_expect(scale == 0.f, 0)) {
      constexpr uint32_t kNan = kExponent | (kExponent >> 1);
      return ((q & kExponent) == kExponent ? kNan : 0u) | ((q >> 16 & kExponent) == kExponent ? kNan << 16 : 0u);
    }
    return scale < 0.f ? q ^ 0x80008000u : q;
  }
};

// ---- storage types ---------------------------------------------------------------------------------
// unpack: 16 bytes of a row -> fp32 (for the V accumulation).
// The q.k partial product of a lane's 16 bytes never unpacks the 16-bit types: q stays in its stored
// form and v_dot2 multiplies two pairs per instruction into an fp32 sum (products of 16-bit floats are
// exact in fp32); the score scale is applied to the finished dot product (kPostScale).  fp32 rows use
// plain FMAs against a q that was scaled once up front.
struct F32 {
  static constexpr int kBytes = 4, kPerVec = 4;
  static constexpr bool kPostScale = false;
  static constexpr float kWeightScale = 1.f;
  // matrix kernel: the score scale as (what q is multiplied by) x (a positive factor for the finished scores).  The sign and
  // the power of two go into q, exactly, so that a score is not larger than the scaled one; a scale that is 0, denormal or
  // not finite goes there as it is.
  static __device__ __forceinline__ bool plain_scale(float scale) {
    const uint32_t exponent = __builtin_bit_cast(uint32_t, scale) & 0x7f800000u;
    return exponent != 0 && exponent != 0x7f800000u;
  }
  static __device__ __forceinline__ float post_scale(float scale) {
    return plain_scale(scale) ? __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, scale) & 0x007fffffu) | 0x3f800000u) : 1.f;
  }
  static __device__ __forceinline__ uint32_t scale_query(uint32_t q, float scale) {
    const float factor = plain_scale(scale) ? __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, scale) & 0xff800000u) : scale;
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, q) * factor);
  }
  struct Q {
    float f[4];
  };
  static __device__ __forceinline__ void unpack(const u32x4& r, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t w = r[i];  // (bit_cast straight from a vector element reads element 0 every time)
      f[i] = __builtin_bit_cast(float, w);
    }
  }
  static __device__ __forceinline__ bool not_finite(uint32_t w) { return (w & 0x7f800000u) == 0x7f800000u; }  // any value of a dword
  static __device__ __forceinline__ void unpack4(u32x4 r, float* f) { unpack(r, f); }  // four consecutive values
  static __device__ __forceinline__ Q make_q(const u32x4& r, float scale) {
    Q q;
    unpack(r, q.f);
#pragma unroll
    for (int i = 0; i < 4; ++i) q.f[i] *= scale;
    return q;
  }
  static __device__ __forceinline__ float dot(const u32x4& k, const Q& q) {
    float kf[4];
    unpack(k, kf);
    float d = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) d = fmaf(kf[i], q.f[i], d);
    return d;
  }
};
struct F16 : HalfQuery {
  static constexpr int kBytes = 2, kPerVec = 8;
  static constexpr bool kPostScale = true;
  // weights (at most 1) enter the second product of the matrix kernel times 2^15, fp16's largest power of two: the step of
  // a split weight is then 2^-39 of the heaviest row's
  static constexpr float kWeightScale = 32768.f;
  typedef u32x4 Q;
  // C (16x16, fp32) += A (16 x k) * B (k x 16), k = 16 or 32: four / eight 16-bit elements of A and of B per lane
  static __device__ __forceinline__ f32x4 mfma(u32x2 a, u32x2 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, a), __builtin_bit_cast(f16x4, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
  // two weights as kTerms pairs in the storage type: each term is what the ones before it left, rounded (two fp16
  // terms hold 22 bits, three all 24 of an fp32 value, as far as fp16's smallest step allows).  Ahead of two more terms the
  // rounding is towards zero: 11 + 11 bits leave 2 either way, and it is one instruction for the pair.
  template <int kTerms>
  static __device__ __forceinline__ void split(float p0, float p1, uint32_t* terms) {
    float r0 = p0, r1 = p1;
#pragma unroll
    for (int i = 0; i < kTerms; ++i) {
      f16x2 h = {(_Float16)r0, (_Float16)r1};
      if (kTerms == 3 && i < 2) h = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(r0, r1));
      terms[i] = __builtin_bit_cast(uint32_t, h);
      r0 = fmaf((float)h.x, -1.f, r0);
      r1 = fmaf((float)h.y, -1.f, r1);
    }
  }
  static __device__ __forceinline__ void unpack(const u32x4& r, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t w = r[i];
      const f16x2 h = __builtin_bit_cast(f16x2, w);
      f[2 * i] = (float)h.x;
      f[2 * i + 1] = (float)h.y;
    }
  }
  static __device__ __forceinline__ uint32_t scale_query(uint32_t q, float scale) { return scaled<0x7c00u>(q, scale); }
  static __device__ __forceinline__ bool not_finite(uint32_t w) { return (w & 0x7c00u) == 0x7c00u || (w & 0x7c000000u) == 0x7c000000u; }
  static __device__ __forceinline__ void unpack4(u32x2 r, float* f) {
    const f16x4 v = __builtin_bit_cast(f16x4, r);
    for (int i = 0; i < 4; ++i) f[i] = (float)v[i];
  }
  static __device__ __forceinline__ Q make_q(const u32x4& r, float) { return r; }
  static __device__ __forceinline__ float dot(const u32x4& k, const Q& q) {
    float d = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t kw = k[i], qw = q[i];
      d = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, kw), __builtin_bit_cast(f16x2, qw), d, false);
    }
    return d;
  }
};
struct BF16 : HalfQuery {
  static constexpr int kBytes = 2, kPerVec = 8;
  static constexpr bool kPostScale = true;
  static constexpr float kWeightScale = 1.f;
  typedef u32x4 Q;
  static __device__ __forceinline__ f32x4 mfma(u32x2 a, u32x2 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(i16x4, a), __builtin_bit_cast(i16x4, b), c, 0, 0, 0);
  }
  static __device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
  template <int kTerms>  // (three: 24 bits, as many as an fp32 weight has)
  static __device__ __forceinline__ void split(float p0, float p1, uint32_t* terms) {
    float r0 = p0, r1 = p1;
#pragma unroll
    for (int i = 0; i < kTerms; ++i) {
      const bf16x2 h = {(__bf16)r0, (__bf16)r1};
      const uint32_t w = __builtin_bit_cast(uint32_t, h);
      terms[i] = w;
      r0 -= __builtin_bit_cast(float, w << 16);
      r1 -= __builtin_bit_cast(float, w & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ void unpack(const u32x4& r, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t w = r[i];
      f[2 * i] = __builtin_bit_cast(float, w << 16);
      f[2 * i + 1] = __builtin_bit_cast(float, w & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ uint32_t scale_query(uint32_t q, float scale) { return scaled<0x7f80u>(q, scale); }
  static __device__ __forceinline__ bool not_finite(uint32_t w) { return (w & 0x7f80u) == 0x7f80u || (w & 0x7f800000u) == 0x7f800000u; }
  static __device__ __forceinline__ void unpack4(u32x2 r, float* f) {
    const uint32_t v0 = r[0], v1 = r[1];
    f[0] = __builtin_bit_cast(float, v0 << 16);
    f[1] = __builtin_bit_cast(float, v0 & 0xffff0000u);
    f[2] = __builtin_bit_cast(float, v1 << 16);
    f[3] = __builtin_bit_cast(float, v1 & 0xffff0000u);
  }
  static __device__ __forceinline__ Q make_q(const u32x4& r, float) { return r; }
  static __device__ __forceinline__ float dot(const u32x4& k, const Q& q) {
    float d = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t kw = k[i], qw = q[i];
      d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, kw), __builtin_bit_cast(bf16x2, qw), d, false);
    }
    return d;
  }
};

// ---- cross-lane helpers (wave64) ---------------------------------------------------------------
template <int kCtrl>
__device__ __forceinline__ float dpp_f(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), kCtrl, 0xf, 0xf, true));
}
template <int kCtrl>
__device__ __forceinline__ int dpp_i(int x) {
  return __builtin_amdgcn_update_dpp(0, x, kCtrl, 0xf, 0xf, true);
}

// Sum over each aligned group of kLanes lanes (8, 16 or 32); every lane of the group gets the sum.
template <int kLanes>
__device__ __forceinline__ float group_allreduce_sum(float x) {
  x += dpp_f<0xB1>(x);                          // quad_perm [1,0,3,2]
  x += dpp_f<0x4E>(x);                          // quad_perm [2,3,0,1]
  if (kLanes >= 8) x += dpp_f<0x141>(x);        // row_half_mirror
  if (kLanes >= 16) x += dpp_f<0x140>(x);       // row_mirror
  if (kLanes >= 32) x += __shfl_xor(x, 16, 64);
  return x;
}

// Inclusive prefix sum over the 64 lanes.  The rows of 16 are joined by the broadcasts of their last lanes: with a readlane and a select for each
// row, here and in wave_inclusive_max, a scan was some ten instructions longer, in the serial chain ahead of the first rows.  us: 5 x 16 heads x
// ~5000 positions 10.2 -> 10.0; 3 x 12 x ~130 4.97 -> 4.85; 3 x 5 x ~400, 27 tokens 6.12 -> 5.96; 1.006 times over 72 shapes of small calls.
__device__ __forceinline__ int wave_inclusive_scan(int x) {
  x += dpp_i<0x111>(x);  // row_shr:1   (lanes without a source inside their row of 16 add 0)
  x += dpp_i<0x112>(x);  // row_shr:2
  x += dpp_i<0x114>(x);  // row_shr:4
  x += dpp_i<0x118>(x);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15, rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31, rows 2 and 3
  return x;
}

__device__ __forceinline__ int clampi(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

// K / V rows are fetched with raw buffer loads: the descriptor covers exactly one (batch, head) slab,
// so the hardware itself returns zeros for any offset outside it, and the cache policy is explicit.
// Non-temporal (streaming) loads: every row is used once; measured 17 % faster than default-policy loads.
// A wave sends its first batch of row loads, and consumes it, at raised instruction priority and drops back to the
// default for the rest of its rows.  Among waves of equal priority a SIMD issues the oldest first, so without this the
// waves of the workgroups that arrived last on a CU get their first rows only when the earlier ones are nearly done
// (per-workgroup stamps: first rows after 4 us for the first quarter of a launch, after 15-18 us for the last) and
// the launch ends on a thin tail of late starters.  Measured on batch 64 x ~155 positions: 27.67 -> 27.11 us; raising
// the priority for the start-up chain as well, or by progress through the rows, gains less or loses.  One-token
// kernels for 16-bit rows of 128 only, and only launches whose slices hold up to four batches of rows per wave (kBoost
// instances, chosen by the launcher): the passes that serve several tokens lose by it (3 tokens: 31.9 -> 33.6 us), fp32
// rows at the same shape (5 batches) lose 1 %, 16-bit rows of 64 lose 6 %, 9 batches (batch 8 x 300..2000) lose 0.5 %,
// 16 and more gain nothing;
// even the untaken branch in the loop costs the longer streams 0.5 %, hence instances of their own.
#ifndef SPAN_FIRST_BATCH_PRIORITY
#define SPAN_FIRST_BATCH_PRIORITY 3  // (a measurement build sets 0 to time the default arbitration)
#endif
constexpr int kBoostUpToBatches = 4;  // per wave
__device__ __forceinline__ void first_batch_priority(bool first_batch) {
#if SPAN_FIRST_BATCH_PRIORITY > 0
  if (first_batch) __builtin_amdgcn_s_setprio(SPAN_FIRST_BATCH_PRIORITY);
  else __builtin_amdgcn_s_setprio(0);
#else
  (void)first_batch;
#endif
}
#ifndef SPAN_ROW_LOAD_POLICY
#define SPAN_ROW_LOAD_POLICY 2  // (a measurement build overrides it to time the other policies)
#endif
constexpr int kRowLoadPolicy = SPAN_ROW_LOAD_POLICY;  // bit 0 = sc0, bit 1 = nt, bit 4 = sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slab_resource(const void* slab, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(slab), 0, bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 load_row_piece(__amdgpu_buffer_rsrc_t slab, uint32_t byte_off) {
  return __builtin_amdgcn_raw_buffer_load_b128(slab, byte_off, 0, kRowLoadPolicy);
}

// Arrival tickets of a (batch, head) pair's slices.
__device__ __forceinline__ int32_t* ticket_counter(const LaunchArgs& a, size_t bh) { return a.counters + bh * (size_t)a.counter_stride; }

// Device-coherent store of one float that another workgroup reads in the same kernel / load of two that another one wrote.
__device__ __forceinline__ void publish(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x2 observe2(const float* p) {
  return __builtin_bit_cast(f32x2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// The product x, rounded: the compiler must not contract it into the subtraction of the reference that follows.  There the
// product's own rounding would stay behind as an exponent, where for scores of 2^24 and more it is no longer small.
__device__ __forceinline__ float rounded(float x) {
  asm("" : "+v"(x));
  return x;
}

// Both of v_permlane16_swap's (kApart = 16) or v_permlane32_swap's results: lanes 16 (32) apart of `low` and `high` are exchanged, so that
// first + second is, in the lanes with bit kApart clear, the sum over the two of `low`, in the others that of `high`.
struct Swapped {
  float first, second;
};
template <int kApart>
__device__ __forceinline__ Swapped swap_lanes(float low, float high) {
  static_assert(kApart == 16 || kApart == 32, "what the instructions exchange");
  const uint32_t l = __builtin_bit_cast(uint32_t, low), h = __builtin_bit_cast(uint32_t, high);
  uint32_t a, b;
  if constexpr (kApart == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(l, h, false, false);
    a = r[0];
    b = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(l, h, false, false);
    a = r[0];
    b = r[1];
  }
  return Swapped{__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}

// Maximum / sum over the lanes lir, lir + kLanes, lir + 2 kLanes .. of the wave (maximum: kLanes = 8, 16 or 32; sum: 16); every lane gets it.
template <int kLanes>
__device__ __forceinline__ float across_groups_max(float x) {
  if (kLanes <= 8) x = fmaxf(x, dpp_f<0x128>(x));  // row_ror:8
  if (kLanes <= 16) {
    const Swapped s = swap_lanes<16>(x, x);
    x = fmaxf(s.first, s.second);
  }
  const Swapped s = swap_lanes<32>(x, x);
  return fmaxf(s.first, s.second);
}
template <int kLanes>
__device__ __forceinline__ float across_groups_sum(float x) {
  static_assert(kLanes == 16, "what the matrix kernel adds up");
  const Swapped s = swap_lanes<16>(x, x);
  const float y = s.first + s.second;
  const Swapped t = swap_lanes<32>(y, y);
  return t.first + t.second;
}

// The states of a wave's row groups become one.  Lane lir + kLanes i comes with group i's state of columns kPer lir .. + kPer - 1, relative to its
// own m; afterwards m and l are the wave's in every lane, and acc[0 .. kOwn - 1] the wave's sums of the lane's own columns, own_column() on.
// The lanes share the columns' sums out as they are added: half as many with every exchange.
template <int kLanes, int kPer>
struct GroupMerge {
  static constexpr int kOwn = kLanes == 32 ? kPer / 2 : kPer / 4;
  static_assert(kOwn >= 1, "a column per lane at least");
  static __device__ __forceinline__ int own_column(int lane) {
    return kPer * (lane % kLanes) + (lane & 32 ? kPer / 2 : 0) + (kLanes <= 16 && (lane & 16) ? kPer / 4 : 0);
  }
  static __device__ __forceinline__ void merge(float& m, float& l, float* acc) {
    const float all = across_groups_max<kLanes>(m);
    const float f = __builtin_amdgcn_exp2f(m - (all == -INFINITY ? 0.f : all));
    m = all;
    const Swapped fs = swap_lanes<32>(f, f), ls = swap_lanes<32>(l, l);
    l = fmaf(ls.first, fs.first, ls.second * fs.second);
#pragma unroll
    for (int i = 0; i < kPer / 2; ++i) {
      const Swapped s = swap_lanes<32>(acc[i], acc[i + kPer / 2]);
      acc[i] = fmaf(s.first, fs.first, s.second * fs.second);
    }
    if constexpr (kLanes <= 16) {
      const Swapped s = swap_lanes<16>(l, l);
      l = s.first + s.second;
#pragma unroll
      for (int i = 0; i < kPer / 4; ++i) {
        const Swapped s = swap_lanes<16>(acc[i], acc[i + kPer / 4]);
        acc[i] = s.first + s.second;
      }
    }
    if constexpr (kLanes <= 8) {
      l += dpp_f<0x128>(l);  // row_ror:8
#pragma unroll
      for (int i = 0; i < kOwn; ++i) acc[i] += dpp_f<0x128>(acc[i]);
    }
  }
};

// Merge two un-normalised softmax states held in log2 units.
__device__ __forceinline__ void merge_state(float& m, float& l, float* acc, int n, float m2, float l2,
                                            const float* acc2) {
  const float mn = fmaxf(m, m2);
  const float ms = (mn == -INFINITY) ? 0.f : mn;
  const float a = __builtin_amdgcn_exp2f(m - ms), b = __builtin_amdgcn_exp2f(m2 - ms);
  // one rounding order, written out: the compiler may contract x*a + y*b either way round, and every instance of
  // the kernel has to give the same bits
  l = fmaf(l, a, l2 * b);
  for (int i = 0; i < n; ++i) acc[i] = fmaf(acc[i], a, acc2[i] * b);
  m = mn;
}

// The kernel arguments are wanted in registers together: left to itself the compiler fetches some of them only after the
// first have arrived, and each such trip costs some tenths of a microsecond at the head of every call (measured: batch 1 x
// ~560 positions 7.9 -> 7.7 us, 4 workgroups x 80 positions 4.4 -> 4.2 us).
// Returns a.heads, which everything else is computed from, tied to the other arguments of the start-up.  (Not volatile: a
// statement with side effects in front of them would turn the scalar loads of the lists into vector loads.)
__device__ __forceinline__ int heads_with_arguments(const LaunchArgs& a) {
  int heads = a.heads;
  asm("" : "+s"(heads) : "s"(a.q), "s"(a.k), "s"(a.v), "s"(a.offsets), "s"(a.starts), "s"(a.ends), "s"(a.append_pos), "s"(a.q_pos),
      "s"(a.k_new), "s"(a.v_new), "s"(a.max_len), "s"(a.num_intervals), "s"(a.q_len), "s"(a.even), "s"(a.interleave),
      "s"(a.max_tokens), "s"(a.slice_tokens), "s"(a.scale_log2e));
  return heads;
}

// What a call says of sequence b, fetched together as well, where each used to be waited for ahead of the next: a pointer that is
// null reads the list instead (one that is always there), and its value is not used.  With the positions' marks (tabulate_short), us:
// batch 8 x ~560 appended 20.6 -> 20.1; 32 pairs x ~560, 3 tokens 9.5 -> 9.3; 8 x 32 x ~600, 2 tokens 21.3 -> 20.7; 64 x 24 heads x ~150 of 64,
// 20 tokens 45.0 -> 43.8.
struct SequenceWords {
  int first, last;         // span form: its range of the interval lists; dense form: its length, twice
  int append_pos, q_pos;
};
template <bool kDense>
__device__ __forceinline__ SequenceWords sequence_words(const LaunchArgs& a, int b) {
  const int32_t* list = kDense ? a.ctx_lens : a.offsets;
  SequenceWords w;
  w.first = __builtin_amdgcn_readfirstlane(list[b]);
  w.last = kDense ? w.first : __builtin_amdgcn_readfirstlane(list[b + 1]);
  w.append_pos = __builtin_amdgcn_readfirstlane((a.append_pos ? a.append_pos : list)[b]);
  w.q_pos = __builtin_amdgcn_readfirstlane((a.q_pos ? a.q_pos : list)[b]);
  return w;
}
// From here on the words are used (the vector loads of rows that are known from the arguments alone go out before).
__device__ __forceinline__ void arrived(SequenceWords& w) { asm("" : "+s"(w.first) : "s"(w.last), "s"(w.append_pos), "s"(w.q_pos)); }

// Positions of a slice: (n + parts - 1) / parts where a sequence's slices share its positions evenly.  Both sides are below 2^23, which the compiler is told (a third of the instructions).
__device__ __forceinline__ int slice_size(const LaunchArgs& a, int n, int parts) {
  if (a.even == 0) return a.slice_tokens;
  return max((int)(((uint32_t)(n + parts - 1) & 0xffffffu) / ((uint32_t)parts & 0xffffffu)), a.even);
}

// ---- the interval list of a sequence -----------------------------------------------------------------
struct Intervals {
  int count, first;     // intervals first .. first + count - 1 of the lists (scalar)
  int st0, len0, incl0; // this lane's interval of the first 64: start, length (0: none), inclusive prefix sum of the lengths
};
constexpr int kChunkTotals = 256;  // chunks of 64 intervals whose position counts are kept (16384 intervals)
struct IntervalTables {  // LDS of a workgroup
  struct Chunk {         // one wave's copy of up to 64 intervals: exclusive prefix sums and starts
    int pref[64], start[64];
  } chunk[kWavesPerBlock];
  int total[kChunkTotals];    // lists of more than 64 intervals: positions of each chunk
  int wave_sum[kWavesPerBlock];
};

__device__ __forceinline__ Intervals interval_range(const LaunchArgs& a, const SequenceWords& w) {
  const int lo = clampi(w.first, 0, a.num_intervals);
  const int hi = clampi(w.last, lo, a.num_intervals);
  return Intervals{__builtin_amdgcn_readfirstlane(hi - lo), __builtin_amdgcn_readfirstlane(lo), 0, 0, 0};
}

__device__ __forceinline__ int interval_length(const LaunchArgs& a, int i) { return clampi(a.ends[i] - a.starts[i], 0, a.max_len); }

// 64 intervals of the lists around where sequence b's would be if all sequences had as many, fetched next to its range instead of after it:
// a trip to memory less at the head of the call wherever they hold all of the sequence's.  Few-query kernel only: us, lists fetched after their range ->
// so: 15 x 32 heads x ~170, 56 tokens 19.5 -> 18.7; 33 x 8 x 1849, 39 tokens 30.1 -> 29.3; 12 x 32 x ~450, 34 tokens 27.4 -> 26.7; 9 x 5 x ~150 fp32, 22
// tokens 10.7 -> 10.4.  One-token calls gain nothing by it (their longer lists lose 1 %: the wave fetches twice).  Lists of a
// mean beyond the window do without; they lose up to 1 % in the few-query kernel (8 x 12 x ~8900, 2200 intervals each, 19 tokens 87.9 -> 88.6).
// The mean is the arrays' entries per sequence.  Arrays kept with room for more put the window beyond the lists of the later sequences, which are
// then fetched after their range as without it: us, arrays filled, 3 times as long, 12 times (no window): 12 x 32 x ~450, 34 tokens 27.9, 28.1, 28.2; 9 x 5 x ~150 fp32, 22 tokens
// 10.2, 10.6, 10.5; 16 x 16 x ~380 of 64, 9 tokens 7.78, 7.87, 7.88.
constexpr int kNoWindow = 0x7fffffff - 64;  // first of a window that holds nothing
struct ListWindow {
  int first;       // number of lane 0's interval (scalar)
  int start, end;  // this lane's
};
__device__ __forceinline__ ListWindow list_window(const LaunchArgs& a, int b, int lane) {
  const bool none = a.intervals_per_seq < 0;
  const int centre = (b * a.intervals_per_seq + (a.intervals_per_seq >> 1)) >> 16;
  ListWindow w = {none ? kNoWindow : clampi(centre - 32, 0, max(a.num_intervals - 64, 0)), 0, 0};
  if (w.first + lane < a.num_intervals) {
    w.start = a.starts[w.first + lane];
    w.end = a.ends[w.first + lane];
  }
  return w;
}

// The sequence's first 64 intervals into the lanes: one each from lane 0 on ...
__device__ __forceinline__ void fetch_first(const LaunchArgs& a, Intervals& iv, int lane) {
  if (lane < iv.count) {
    iv.st0 = a.starts[iv.first + lane];
    iv.len0 = clampi(a.ends[iv.first + lane] - iv.st0, 0, a.max_len);
  }
}
// ... or where the window has them, with lanes of no length around them.
__device__ __forceinline__ void fetch_first(const LaunchArgs& a, Intervals& iv, const ListWindow& window, int lane) {
  const int ahead = iv.first - window.first;
  if (__builtin_expect(ahead < 0 || ahead + iv.count > 64, 0)) return fetch_first(a, iv, lane);
  iv.st0 = window.start;
  iv.len0 = (uint32_t)(lane - ahead) < (uint32_t)iv.count ? clampi(window.end - window.start, 0, a.max_len) : 0;
}

// Positions of the sequence's list, whose first intervals are in the lanes (fetch_first).  Called by all waves of the workgroup.
// Up to 64 intervals every wave counts for itself and no barrier is met.  Longer lists (a mask in which every token
// decides for itself has an interval per four positions) are a chain of dependent trips to memory if walked chunk by
// chunk, and nothing hides them when few workgroups run: the waves share the chunks, four in flight each, and leave the
// chunks' counts in LDS, where tabulate_positions finds a wave's first chunk.  2 sequences x 14000 positions in 3500
// intervals, 16 heads x 128, bf16: 49.0 -> 30.8 us; one x 4000 in 1000, 32 heads, fp16: 17.1 -> 14.1 us; 32 x 900 (bound by
// the rows): no change.  The long walk is kept out of the straight path: code that is jumped over costs a call of few
// workgroups 0.2 - 0.4 us of instruction fetch.
__device__ __forceinline__ int count_positions(const LaunchArgs& a, Intervals& iv, int wave, int lane, IntervalTables& tab) {
  iv.incl0 = wave_inclusive_scan(iv.len0);
  int n = __builtin_amdgcn_readlane(iv.incl0, 63);
  if (__builtin_expect(iv.count > 64, 0)) {
    const int chunks = (iv.count + 63) / 64;
    if (wave == 0 && lane == 0) tab.total[0] = n;
    int mine = 0;
    constexpr int kInFlight = 4;
    for (int c = 1 + wave; c < chunks; c += kWavesPerBlock * kInFlight) {
      int len[kInFlight];
#pragma unroll
      for (int k = 0; k < kInFlight; ++k) {
        const int i = (c + k * kWavesPerBlock) * 64 + lane;
        len[k] = i < iv.count ? interval_length(a, iv.first + i) : 0;
      }
#pragma unroll
      for (int k = 0; k < kInFlight; ++k) {
        const int total = __builtin_amdgcn_readlane(wave_inclusive_scan(len[k]), 63);
        mine += total;
        if (lane == 0 && c + k * kWavesPerBlock < min(chunks, kChunkTotals)) tab.total[c + k * kWavesPerBlock] = total;
      }
    }
    if (lane == 0) tab.wave_sum[wave] = mine;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWavesPerBlock; ++w) n += __builtin_amdgcn_readfirstlane(tab.wave_sum[w]);
  }
  return n;
}

// The chunk's exclusive prefixes and starts go to the wave's own LDS rows and every lane finds the intervals of its rows:
// virtual token v lies in the last interval whose exclusive prefix is <= v (lanes past the list's end hold the chunk's end
// as prefix and are never chosen).  The wave reads back what it wrote itself (LDS executes a wave's requests in order), so
// there is no block barrier.
template <class RowMap>
__device__ __forceinline__ void place_chunk(const RowMap& vrow, int w0, int wn, int lane, int n_here, int carry, int st, int len,
                                            int incl, int max_len, IntervalTables::Chunk& chunk, int* pos) {
  const int chunk_total = __builtin_amdgcn_readlane(incl, 63);
  chunk.pref[lane] = carry + incl - len;
  chunk.start[lane] = st;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (int r = lane; r < wn; r += 64) {
    const int v = vrow(w0 + r);
    if (v >= carry && v < carry + chunk_total) {
      int idx = 0;
#pragma unroll
      for (int step = 32; step > 0; step >>= 1) {
        const int j = idx + step;
        if (j < n_here && chunk.pref[j] <= v) idx = j;
      }
      const int p = chunk.start[idx] + (v - chunk.pref[idx]);
      pos[r] = clampi(p, 0, max_len - 1);
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// What the lanes of this wave wrote to LDS is read back by others of them (LDS executes a wave's requests in order).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive maximum over the lanes up to each, all values >= 0.
__device__ __forceinline__ int wave_inclusive_max(int x) {
  x = max(x, dpp_i<0x111>(x));
  x = max(x, dpp_i<0x112>(x));
  x = max(x, dpp_i<0x114>(x));
  x = max(x, dpp_i<0x118>(x));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));  // as above; 0 is the neutral element
  return max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
}

// Cache positions of the wave's first rows 0 .. wn - 1 into `pos` for a list of up to 64 intervals, which are still in
// registers from count_positions; row r is virtual token vbase + r + (r / kUnit) * vgap of the sequence (vgap 0, or three units).
// Every interval marks the wave's first row at or after its first token with its number, the largest where several meet; a row's
// interval is the largest mark up to it (an inclusive maximum over the lanes).  Three trips to LDS for 128 rows, where a binary
// search of the prefix sums takes seven for every 64 (place_chunk, which lists of several chunks still use: a chunk holds a few
// of the wave's rows there).
template <int kUnit, int kRows>
__device__ __forceinline__ void tabulate_short(const LaunchArgs& a, const Intervals& iv, int vbase, int vgap, int wn, int wave,
                                               int lane, IntervalTables& tab, int* pos) {
  IntervalTables::Chunk& chunk = tab.chunk[wave];
  const int before = iv.incl0 - iv.len0, x = before - vbase;
  chunk.start[lane] = iv.st0 - before;
  constexpr int kPair = 128;  // rows taken together: two per lane
#pragma unroll
  for (int r0 = 0; r0 < kRows; r0 += kPair) {
    if (r0 < wn) pos[r0 + lane] = pos[r0 + 64 + lane] = 0;
  }
  wave_lds_order();
  const uint32_t ux = (uint32_t)x;
  const uint32_t row = vgap == 0 ? ux : ux / (4u * kUnit) * kUnit + min(ux % (4u * kUnit), (uint32_t)kUnit);
  if (iv.len0 > 0 && (x < 0 || row < (uint32_t)wn))
    __hip_atomic_fetch_max(&pos[x < 0 ? 0u : row], lane + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  wave_lds_order();
  int carry = 1;
  for (int r0 = 0; r0 < wn; r0 += kPair) {
    int m[2], base[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) m[k] = pos[r0 + 64 * k + lane];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      m[k] = max(wave_inclusive_max(m[k]), carry);
      carry = __builtin_amdgcn_readlane(m[k], 63);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) base[k] = chunk.start[m[k] - 1];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int r = r0 + 64 * k + lane;
      pos[r] = clampi(base[k] + vbase + r + r / kUnit * vgap, 0, a.max_len - 1);
    }
  }
  wave_lds_order();
}

// The same for rows w0 .. w0 + wn - 1 and any list: re-reads the intervals, so that nothing stays live across the
// streaming loop.
template <class RowMap>
__device__ __forceinline__ void tabulate_positions(const LaunchArgs& a, const Intervals& iv, const RowMap& vrow, int w0,
                                                   int wn, int wave, int lane, IntervalTables& tab, int* pos) {
  const int vbeg = vrow(w0), vend = vrow(w0 + wn - 1) + 1;
  int c0 = 0, carry = 0;  // first interval of the chunk the walk stands in, positions before it
  if (iv.count > 64) {    // skip the chunks before the window
    const int known = min((iv.count + 63) / 64, kChunkTotals);
    for (int t0 = 0; t0 < known; t0 += 64) {
      const int incl = wave_inclusive_scan(t0 + lane < known ? tab.total[t0 + lane] : 0);
      const int skip = __popcll(__builtin_amdgcn_ballot_w64(t0 + lane < known && carry + incl <= vbeg));
      if (skip > 0) carry += __builtin_amdgcn_readlane(incl, skip - 1);
      c0 = (t0 + skip) * 64;
      if (skip < 64) break;
    }
  }
  int st = 0, len = 0;
  auto load_chunk = [&](int c) {
    st = len = 0;
    if (c + lane < iv.count) {
      st = a.starts[iv.first + c + lane];
      len = clampi(a.ends[iv.first + c + lane] - st, 0, a.max_len);
    }
  };
  load_chunk(c0);
  while (c0 < iv.count) {
    const int incl = wave_inclusive_scan(len), chunk_total = __builtin_amdgcn_readlane(incl, 63);
    const int here = c0, here_carry = carry, here_st = st, here_len = len;
    c0 += 64;
    carry += chunk_total;
    if (carry < vend) load_chunk(c0);  // the next chunk is on its way while this one is searched
    if (carry > vbeg)
      place_chunk(vrow, w0, wn, lane, min(64, iv.count - here), here_carry, here_st, here_len, incl, a.max_len, tab.chunk[wave], pos);
    if (carry >= vend) break;
  }
}

}  // namespace spanattn
#endif
