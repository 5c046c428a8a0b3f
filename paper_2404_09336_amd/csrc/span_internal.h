// Shared between the host-only and the kernel translation units of the library.
#ifndef SPAN_INTERNAL_H_
#define SPAN_INTERNAL_H_

#include <stddef.h>
#include <stdint.h>

#include "span_attn.h"

namespace spanattn {

constexpr int kWavesPerBlock = 4;          // 256 threads per workgroup
constexpr int kMaxSlice = 1 << 22;         // a slice may be a whole sequence (positions are tabulated window by window)
#ifndef SPAN_MIN_SLICE
#define SPAN_MIN_SLICE 128
#endif
constexpr int kMinSlice = SPAN_MIN_SLICE;  // do not cut work finer than this many positions
constexpr int kBoundSlice = 512;           // slices planned from a bound alone hold at most this many positions where a round has room for them
constexpr int kBoundSliceFromBatch = 8;    // ... of batches larger than this (both sides: see plan_partition)
constexpr int kLeastSlice = 64;            // positions of a slice whose size the kernel chooses, see Partition::least_slice
constexpr int kSliceGranule = 16;
constexpr int kUnsplitFromPairs = 512;     // level batches with at least this many (batch, head) pairs are not sliced
#ifndef SPAN_LARGE_SLICE
#define SPAN_LARGE_SLICE 1024
#endif
constexpr int kLargeSlice = SPAN_LARGE_SLICE;  // slices above this size are cut down to it, in several rounds of workgroups
constexpr int kMaxLen = 1 << 22;           // keeps every in-slab byte offset inside 32 bits
#ifndef SPAN_TARGET_WORKGROUPS
#define SPAN_TARGET_WORKGROUPS 2048
#endif
constexpr int64_t kTargetWorkgroups = SPAN_TARGET_WORKGROUPS;  // 256 CUs x 8 resident workgroups

constexpr int kInterleaveFrom = 384;        // slices at least this large deal their rows to the waves round-robin
constexpr int kMaxPlanSlices = 768;        // entries of the slice table passed as kernel argument
constexpr int kMaxPlanBatch = 1024;        // 10 bits of a table entry
constexpr int kMaxPlanSplits = 2047;       // 11 bits of a table entry
constexpr int kMaxQueryTokens = 64;        // few-query variant: query tokens per sequence and call

// Run mode: when the caller also hands in host copies of the span lists, the planner resolves every slice to its
// runs of consecutive cache positions and the runs travel in the kernel arguments (no span metadata is read from
// device memory before the first K row is requested).  Sized so that the arguments stay under 4 KB.
constexpr int kMaxRunSlices = 96;          // slices of all sequences (= grid.y)
constexpr int kMaxRuns = 288;              // runs of all slices
constexpr int kMaxRunSliceRows = 1024;     // rows of one slice: every wave's rows fit one position window

struct RunSlice {      // 16 bytes: one scalar load
  uint32_t entry;      // pack_slice(batch, slice, slices of the sequence), dealt or not
  uint32_t runs_of;    // first run | number of runs << 16
  int32_t rows;        // attended positions of the slice
  int32_t reserved;    // (of a dealt launch: the slice's slot)
};
struct RunTables {
  RunSlice slices[kMaxRunSlices];
  int32_t run[kMaxRuns][2];  // a run covers cache positions [run[.][0], run[.][0] + run[.][1])
};

// Slice table entry (exact mode) as planned: batch index | slice index within the sequence | slices of the sequence.
inline uint32_t pack_slice(uint32_t b, uint32_t split, uint32_t nsl) { return b | (split << 10) | (nsl << 21); }

// A launch whose slices go out in another order than the plan names them (see deal_slices): a table entry then also says which
// slice of the plan it is, which is the slice's slot in the workspace:
// batch index (b_bits) | slice (n_bits) | slices of the sequence (n_bits) | slot (the ten highest bits).
constexpr int kSlotBits = 10;
static_assert(kMaxPlanSlices <= 1 << kSlotBits, "a slot fits an entry");
struct Deal {
  bool dealt = false;            // false: plan order, entries as pack_slice packs them, slot = entry index
  int32_t b_bits = 10, n_bits = 11;
  uint16_t at[kMaxPlanSlices];   // dealt: table index of slice i of the plan
};

struct Partition {
  bool exact;            // slices come from the table; otherwise the grid is (heads, num_splits, batch)
  bool even;             // a sequence's slices share its own token count evenly (needs the caller's counts)
  int32_t least_slice;   // not even: 0, or the kernel shares a sequence's positions evenly between its slices, this many each at least
  int32_t num_splits;    // uniform: KV slices per (batch, head); exact: most slices of any sequence
  int32_t slice_tokens;  // attended positions per slice (exact: upper bound)
  int32_t max_tokens;    // bound on attended positions per sequence
  int32_t total_slices;  // exact: table entries (grid.y); uniform: batch * num_splits
  int32_t queries_per_pass;  // query tokens whose states a slot of the workspace holds (1, 2, 4 or 16)
  int32_t granule;       // exact: sequence b is cut into ceil(n_b / granule) slices,
  int32_t whole;         // ... or stays whole up to so many positions
  bool runs;             // the slices' position runs were resolved on the host (RunTables filled)
};

// Attended positions of every sequence as far as the caller tells them, counted once per call.  Host copies of the span lists, when
// given, are the authority (tokens_per_seq is then not consulted), in every function that plans, so that they all agree.  (Host
// time of a one-token call's plan, walked again by the deal -> once: 8 x 32 heads, 28200 intervals 70 -> 21 us, 32 x 12, 13700 intervals 35 -> 13.)
struct TokenCounts {
  explicit TokenCounts(const span_attn_desc_t* d);
  TokenCounts(const TokenCounts&) = delete;
  TokenCounts& operator=(const TokenCounts&) = delete;
  bool from_lists;
  const int64_t* of;  // [batch], or null where nothing is known

 private:
  int64_t counted_[kMaxPlanBatch];
};

// The planner's rules for short sequences of one and two tokens: whole up to some length, fp32 rows of 128 in half-size slices, short level batches not
// sliced.  kNone is the cut without them, which a workspace sized for longer sequences of the same shape holds where it does not hold half-size
// slices (1 x 32 heads: 266496 bytes for 1000 positions, 150016 for 1025; in slices of kMinSlice 133376 for 1000).  kWhole is for 256 to 511 pairs, where a
// level batch asks for no workspace at all: every sequence up to that length is then left whole.
enum class ShortRules { kApplied, kNone, kWhole };

// Fills `table` (kMaxPlanSlices entries) when the partition is exact; table may be null to only size it.
// `spans`: may be the span form, whose slices of one token are cut finer where only a bound is known (false: the dense entry points, and
// where a workspace does not hold the finer cut).  A descriptor without intervals is a dense call's to every function.
// With `runs` given (span form only) and host copies of the span lists in the descriptor, tries run mode first.
Partition plan_partition(const span_attn_desc_t* d, const TokenCounts& counts, uint32_t* table, RunTables* runs, bool spans,
                         ShortRules rules = ShortRules::kApplied);
inline Partition plan_partition(const span_attn_desc_t* d, uint32_t* table = nullptr, RunTables* runs = nullptr, bool spans = true) {
  return plan_partition(d, TokenCounts(d), table, runs, spans);
}
// The same with the descriptor's workspace: where it does not hold the plan, as ever, the first coarser cut that it holds (not from a bound's finer one, by
// kNone, by kWhole).
Partition plan_for_workspace(const span_attn_desc_t* d, const TokenCounts& counts, uint32_t* table, RunTables* runs, bool spans);

// How a few-query call runs on the matrix cores (span_matrix.hip).  The workspace holds partial states of query tokens: at
// least those of the Partition above, total_slices * queries_per_pass per head, and more where the caller brings them; the
// launches cut the spans into as many slices as that room allows for all the tokens they serve.
struct MatrixPlan {
  int32_t tokens;        // query tokens of one launch (all of the call's unless the caller fixed the number of slices)
  int32_t groups;        // groups of 16 tokens a workgroup serves with one pass over its rows: 1, 2 or 4
  bool table;            // slices from the table.  As planned: sequences with several slices first, so an entry's index is its slot;
                         // whole sequences, which have no slot, in any order.  After a deal only Deal and slice_name can read it.
  bool even;             // as in Partition
  int32_t least_slice;   // as in Partition
  int32_t num_splits;    // as in Partition
  int32_t slice_tokens;  // as in Partition
  int32_t total_slices;  // table entries, or batch * num_splits
  int64_t states;        // token states per head that the slices use
};
// Most groups a workgroup serves: the state of 64 tokens of fp32 rows of 128 does not fit the registers next to a tile.
constexpr int kMatrixMaxGroups(int elt_bytes, int head_dim) { return elt_bytes == 4 && head_dim == 128 ? 2 : 4; }
// Workgroups of the matrix kernel that a CU runs at once, one wave per SIMD each: the most whose registers hold the state, a tile and
// its weights.
constexpr int kMatrixWorkgroupsPerCu(int elt_bytes, int head_dim, int groups) {
  return head_dim == 128 ? (groups == 1 && elt_bytes == 2 ? 4 : 2) : (groups == 1 ? 4 : (groups == 2 ? 3 : 2));
}
bool runs_on_matrix_cores(const span_attn_desc_t* d);
int64_t least_states(const Partition& p);                             // token states per head a call must bring
int64_t most_states(const span_attn_desc_t* d, const Partition& p);   // ... it can use
// False if the call does not run on the matrix cores.  `p` is the call's partition, `states` what the workspace holds per
// head (least_states at least), `table` has kMaxPlanSlices entries.  `two_per_cu`: 512 workgroups whatever fewer would gain, no sequence whole for being
// short; not for a launch, but what a workspace is asked for at least: a shorter call of the shape may want more slices (3 x 5 heads of 64, 16 bits, 3
// tokens, level: 253696 bytes hold the plan for 3013 positions, 285440 also that for 2061).
bool plan_matrix(const span_attn_desc_t* d, const TokenCounts& counts, const Partition& p, int64_t states, MatrixPlan* m, uint32_t* table,
                 bool two_per_cu = false);
inline bool plan_matrix(const span_attn_desc_t* d, const Partition& p, int64_t states, MatrixPlan* m, uint32_t* table) {
  return plan_matrix(d, TokenCounts(d), p, states, m, table);
}
inline bool plan_matrix(const span_attn_desc_t* d, const Partition& p, MatrixPlan* m, uint32_t* table) {
  return plan_matrix(d, p, least_states(p), m, table);
}

// Deals the slices of a plan that cuts its sequences evenly: `entries` holds them in plan order, as pack_slice packs them, and
// is rewritten if the deal is worth it.  `hand_over`: rows that a slice of a sequence with several counts more; `table`: the launch carries
// a table anyway.
void deal_slices(const span_attn_desc_t* d, const TokenCounts& counts, int64_t max_tokens, int32_t total, int32_t hand_over, bool table,
                 uint32_t* entries, Deal* deal);
// The same for what the vector kernels and the matrix kernel launch; a plan without a table may get one.
void deal_partition(const span_attn_desc_t* d, const TokenCounts& counts, Partition* p, uint32_t* table, RunTables* runs, Deal* deal);
inline void deal_partition(const span_attn_desc_t* d, Partition* p, uint32_t* table, RunTables* runs, Deal* deal) {
  deal_partition(d, TokenCounts(d), p, table, runs, deal);
}
void deal_matrix(const span_attn_desc_t* d, const TokenCounts& counts, const Partition& p, MatrixPlan* m, uint32_t* table, Deal* deal);
inline void deal_matrix(const span_attn_desc_t* d, const Partition& p, MatrixPlan* m, uint32_t* table, Deal* deal) {
  deal_matrix(d, TokenCounts(d), p, m, table, deal);
}

int check_desc(const span_attn_desc_t* d);
int32_t query_tokens(const span_attn_desc_t* d);  // q_len of the descriptor, at least 1
size_t workspace_counter_bytes(const span_attn_desc_t* d);
// Words from one pair's ticket counter to the next: the counters' part of the workspace is a multiple of 256 bytes, and few pairs spread over all of it.
// Tickets of one 64-byte line are drawn one after the other, about 10 ns each, and with several hundred workgroups of few pairs a launch waited for them up to 2.5 us.  us, side by
// side -> apart: 2 x 8 heads x ~3200 positions dense of 64 10.8 -> 8.2; 2 x 8 x ~4500 fp32 of 64 19.1 -> 16.2; 3 x 5 x ~600 of 64, 2 tokens 11.2 -> 10.0; 4 x 5 x ~2900
// appended 15.7 -> 14.4; 4 x 5 x 100..1200 fp32 9.6 -> 9.15; 89 shapes of up to 128 pairs 1.01 times on average, most of them with as many lines as before.
int32_t counter_stride(const span_attn_desc_t* d);
size_t workspace_ml_bytes(const span_attn_desc_t* d, int64_t states);
size_t workspace_bytes_for(const span_attn_desc_t* d, int64_t states);
size_t workspace_least_bytes(const span_attn_desc_t* d, const Partition& p);  // with less the call is refused
size_t workspace_bytes(const span_attn_desc_t* d, const TokenCounts& counts, const Partition& p);  // what span_workspace_bytes asks for
inline size_t workspace_bytes(const span_attn_desc_t* d, const Partition& p) { return workspace_bytes(d, TokenCounts(d), p); }
int64_t states_that_fit(const span_attn_desc_t* d, const Partition& p);       // in desc->workspace_bytes (not less than the least)

}  // namespace spanattn
#endif
