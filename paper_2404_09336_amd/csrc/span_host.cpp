// Host-only parts of the span-attention library: span-list validation, work partitioning
// arithmetic and error strings.  No GPU call in this file.
#include <limits.h>

#include <algorithm>
#include <map>
#include <vector>

#include "span_attn.h"
#include "span_internal.h"

extern "C" int span_validate(int32_t batch, int32_t num_intervals, const int32_t* span_offsets,
                             const int32_t* span_starts, const int32_t* span_ends, const int32_t* ctx_lens,
                             int32_t* first_bad_seq, int32_t* first_bad_interval, int64_t* span_tokens_per_seq) {
  if (!span_offsets || !ctx_lens || !first_bad_seq || !first_bad_interval) return SPAN_ERR_NULL;
  if (num_intervals > 0 && (!span_starts || !span_ends)) return SPAN_ERR_NULL;
  if (batch < 0 || num_intervals < 0) return SPAN_ERR_SHAPE;
  *first_bad_seq = -1;
  *first_bad_interval = -1;
  for (int32_t b = 0; b < batch; ++b) {
    const int32_t first = span_offsets[b], last = span_offsets[b + 1];
    auto fail = [&](int code, int32_t interval) {
      *first_bad_seq = b;
      *first_bad_interval = interval;
      return code;
    };
    if (b == 0 && first != 0) return fail(SPAN_BAD_OFFSETS, -1);
    if (last < first || last > num_intervals) return fail(SPAN_BAD_OFFSETS, -1);
    if (last == first) return fail(SPAN_BAD_EMPTY_SPAN, -1);
    int64_t tokens = 0;
    int32_t prev_start = 0, prev_end = 0;
    for (int32_t i = first; i < last; ++i) {
      const int32_t s = span_starts[i], e = span_ends[i], k = i - first;
      if (s < 0 || e > ctx_lens[b]) return fail(SPAN_BAD_RANGE, k);
      if (s >= e) return fail(SPAN_BAD_EMPTY_INTERVAL, k);
      if (k > 0) {
        if (s < prev_start) return fail(SPAN_BAD_UNSORTED, k);
        if (s < prev_end) return fail(SPAN_BAD_OVERLAP, k);
      }
      tokens += (int64_t)e - (int64_t)s;
      prev_start = s;
      prev_end = e;
    }
    if (span_tokens_per_seq) span_tokens_per_seq[b] = tokens;
  }
  return SPAN_OK;
}

namespace spanattn {

int check_desc(const span_attn_desc_t* d) {
  if (!d) return SPAN_ERR_NULL;
  if (d->batch <= 0 || d->heads <= 0 || d->max_len <= 0 || d->max_len > kMaxLen) return SPAN_ERR_SHAPE;
  if (d->head_dim != 64 && d->head_dim != 128) return SPAN_ERR_SHAPE;
  if (d->num_intervals < 0 || d->max_tokens < 0 || d->num_splits < 0) return SPAN_ERR_SHAPE;
  if ((int64_t)d->batch * d->heads > INT_MAX / 2) return SPAN_ERR_SHAPE;
  if (d->batch > 65535) return SPAN_ERR_SHAPE;  // grid z limit
  if (d->dtype != SPAN_F32 && d->dtype != SPAN_F16 && d->dtype != SPAN_BF16) return SPAN_ERR_DTYPE;
  if (d->q_len < 0 || d->q_len > kMaxQueryTokens) return SPAN_ERR_SHAPE;
  return SPAN_OK;
}

int32_t query_tokens(const span_attn_desc_t* d) { return d->q_len > 1 ? d->q_len : 1; }

// Query tokens a slot of the workspace holds (one partial state each): 1, 2, 4, or 16 for 16-bit types with head_dim
// 128 from three tokens on.  Calls on the vector units run as planned with it; those on the matrix cores (three tokens and
// more, some with two) share the states out again, see plan_matrix.
static int32_t queries_per_pass(const span_attn_desc_t* d) {
  const int32_t n = query_tokens(d);
  if (n >= 3 && d->dtype != SPAN_F32 && d->head_dim == 128) return 16;
  return n >= 3 ? 4 : n;
}

// Workgroups of one resident round: the kernel for one query token runs 8 workgroups per CU, the one for two tokens 6
// (their register budgets); the workspace of longer calls is sized for 4.
static int64_t target_workgroups(const span_attn_desc_t* d) {
  const int32_t nq = queries_per_pass(d);
  return nq == 1 ? kTargetWorkgroups : kTargetWorkgroups * (nq == 2 ? 6 : 4) / 8;
}

static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Slices (per head, over all sequences) a call aims at.  The upper end is one resident round of workgroups.  But
// few, large slices beat many small ones as long as the memory system stays busy and a ragged batch can still be
// levelled: a quarter of the wavefront slots saturates HBM, every slice costs its own start-up, and every extra
// slice of a pair a partial state and a ticket.  So: a quarter round, or two slices per sequence on average if
// that is more, never beyond one round.  Measured (batch x attended positions, 32 heads x 128, fp16; this rule
// against always filling the round): 1 x 8000 25.7 vs 30.5 us, 4 x 2000 26.5 vs 28.4, 8 x 200..1600 21.8 vs 23.1,
// 16 x 110..1100 30.0 vs 30.7, 8 x 6000 125.6 vs 130.8; 32 x 4096..16384 is one full round either way.
static int64_t slice_room(const span_attn_desc_t* d) {
  const int64_t round = target_workgroups(d);
  const int64_t most = round / d->heads, least = ceil_div(round / 4, d->heads);
  const int64_t room = std::max<int64_t>(least, 2 * (int64_t)d->batch);
  return std::max<int64_t>(1, std::min(room, most));
}

// Exact mode (the caller knows how many positions each sequence attends).
//
// All workgroups of a launch that fit on the chip at once start together and spend the same first
// microseconds walking the span metadata before any K row is requested; a second round of equal
// workgroups would repeat that dead time, and every extra slice costs a partial state and a ticket.
// So the aim is ONE resident round: the smallest slice size T for which all slices of all sequences,
// times heads, fit into kTargetWorkgroups.  Sequence b gets ceil(n_b / T) slices, which the kernel makes
// equal-sized.  When batch * heads alone exceeds a round, every sequence is one slice.
static int64_t slices_for(int64_t n, int64_t T, int64_t whole) { return n <= std::max<int64_t>(whole, 0) ? 1 : ceil_div(n, T); }

// fp32 rows of 128, one token: slices of half kMinSlice where a call has no more of them than it aims at.  A wave's batch of rows (16 KB with twice the
// loads in flight, see launch_typed) is 16 such rows, and 32 of the others: a slice that fills it is read in one trip.  us, slices of 128 -> of 64: 8 pairs x
// 256 positions 7.15 -> 6.11, x 512 7.58 -> 6.27; 32 pairs x 320 8.0 -> 6.9, x 512 8.4 -> 7.9, x 1000 10.5 -> 10.3; 64 x 400 10.0 -> 9.4, x 512 10.6
// -> 10.7. Slices between 64 and 128 are two batches all the same: 32 pairs, up to 3250 positions planned from a bound 15.8 -> 16.2.
static bool fine_slices(const span_attn_desc_t* d) { return query_tokens(d) == 1 && d->dtype == SPAN_F32 && d->head_dim == 128; }
constexpr int64_t kFineSlice = kMinSlice / 2;

// A sequence of up to so many positions stays in one slice however few the pairs, one or two tokens: two batches of rows a wave take less than the
// hand-over of the slices. us, in two slices -> whole, 256 positions, 8, 32, 96, 160 and 256 pairs: fp16 rows of 128 6.3, 6.4, 7.2, 8.7, 9.9 -> 5.9,
// 6.0, 6.7, 7.2, 8.5, of 64 5.9, 5.75, 6.3, 6.9, 7.6 -> 4.7, 4.7, 5.1, 5.4, 5.9, fp32 of 64 6.1, 6.2, 7.1, 8.5, 9.75 -> 5.7, 5.8, 6.5, 7.0, 8.3; 136
// positions 5.9 -> 4.6, 5.6 -> 4.0, 5.9 -> 4.6 (8 pairs). 320 positions in three: 6.2 -> 7.3, 5.7 -> 6.0, 6.05 -> 7.3 (8 pairs), 11.4 -> 10.3 (256,
// see level below). fp32 rows of 128 up to 128: 256 pairs x 50..100 8.1 -> 7.0; 136 positions, 8 pairs 6.1 -> 5.9, 160 6.1 -> 6.9, 32 pairs 6.3 ->
// 7.4. Two tokens, 256 positions: fp16 of 128 7.8 -> 7.8 (32 pairs), 10.7 -> 8.9 (256); fp32 of 64, 160 positions 7.9 -> 6.6 (32), 256 8.65 -> 8.85.
static int64_t whole_up_to(const span_attn_desc_t* d) {
  if (query_tokens(d) > 2 || (runs_on_matrix_cores(d) && (int64_t)d->batch * d->heads > 256)) return 0;  // (the matrix kernel's: see plan_matrix)
  if (d->dtype == SPAN_F32) return d->head_dim == 128 ? kMinSlice : (query_tokens(d) == 1 ? 256 : 160);
  return 256;
}

// One token: a level batch of at least one workgroup per CU is not sliced up to so many positions (see plan_exact).
static int64_t level_up_to(const span_attn_desc_t* d) {
  const int64_t pairs = (int64_t)d->batch * d->heads;
  if (query_tokens(d) != 1 || pairs < kUnsplitFromPairs / 2) return 0;
  return d->dtype != SPAN_F32 && d->head_dim == 64 ? pairs * 3 / 2 : 768;
}

// Up to so many positions no sequence is sliced, under these rules.
static int64_t unsliced_up_to(const span_attn_desc_t* d, ShortRules rules) {
  if (rules == ShortRules::kApplied) return whole_up_to(d);
  return rules == ShortRules::kWhole && (int64_t)d->batch * d->heads < kUnsplitFromPairs ? level_up_to(d) : 0;
}

static bool plan_exact(const span_attn_desc_t* d, const int64_t* tokens_per_seq, int64_t max_tok, ShortRules rules, Partition* p,
                       uint32_t* table) {
  if (!tokens_per_seq || d->num_splits != 0 || d->batch > kMaxPlanBatch) return false;
  auto tokens = [&](int32_t b) {
    const int64_t n = tokens_per_seq[b];
    return n < 0 ? (int64_t)0 : (n > max_tok ? max_tok : n);
  };
  const bool short_rules = rules == ShortRules::kApplied;
  const int64_t whole = unsliced_up_to(d, rules);
  auto cut = [&](int64_t n, int64_t T) { return slices_for(n, T, whole); };
  auto count = [&](int64_t T) {
    int64_t c = 0;
    for (int32_t b = 0; b < d->batch; ++b) c += cut(tokens(b), T);
    return c;
  };
  int64_t sum = 0, longest = 0;
  for (int32_t b = 0; b < d->batch; ++b) {
    sum += tokens(b);
    if (tokens(b) > longest) longest = tokens(b);
  }
  int64_t room = slice_room(d);  // slices (per head) the call aims at, at most one resident round
  if (room > kMaxPlanSlices) room = kMaxPlanSlices;
  int64_t T = ceil_div(sum, room);
  if (T < kMinSlice) T = short_rules && fine_slices(d) && count(kFineSlice) <= room ? kFineSlice : kMinSlice;
  int64_t total = count(T);
  // A quarter of the chip's wavefront slots (512 workgroups) already keeps the memory system busy, and a
  // pair that is one workgroup needs no partial states and no tickets.  So a batch of at least 512 (batch,
  // head) pairs whose longest sequence is within 35 % of the mean runs unsplit (measured 5-10 % faster than
  // filling the round with slices: batch 16 x 555 tokens +-25 % 30.6 -> 27.9 us, batch 48 x 300 44.6 -> 42.3 us);
  // more ragged batches need the slices to level the work (batch 16, 112..1100 tokens: 30.3 split, 30.9 unsplit).
  // From one workgroup per CU on so do short sequences, one token, if they are level: us, sliced -> whole, fp16 rows of 128: 256 pairs x 400
  // positions 13.4 -> 12.4, x 700 18.7 -> 17.7, x 1000 25.6 -> 28.8; 384 x 448 18.6 -> 17.6, x 700 26.9 -> 25.6, x 1000 38.1 -> 39.4; 448 x 700 31.7
  // -> 27.9; fp32: 256 x 700 33.0 -> 32.6, x 1000 49.7 -> 52.9; fp16 of 64: 256 x 320 8.6 -> 7.4, x 448 9.95 -> 10.15; 320 x 448 11.1 -> 10.6, x 700
  // 14.7 -> 14.9; 448 x 448 13.6 -> 11.6.
  const int64_t pairs = (int64_t)d->batch * d->heads;
  const bool level = (pairs >= kUnsplitFromPairs && longest * 100 * d->batch <= 135 * sum) ||
                     (short_rules && longest <= level_up_to(d) && longest * 100 * d->batch <= 108 * sum);
  if (room < d->batch || level) {  // whole sequences (batch * heads alone exceeds a round, or a level batch)
    T = max_tok > 0 ? max_tok : 1;
    total = count(T);
  } else {
    while (total > room) {  // grow T in proportion to the overshoot (at least one granule) and try again
      const int64_t next = ceil_div(ceil_div(T * total, room), kSliceGranule) * kSliceGranule;
      T = next > T ? next : T + kSliceGranule;
      total = count(T);
    }
    // fits: give back what the proportional step overshot
    for (int i = 0; i < 8 && T - kSliceGranule >= kMinSlice && count(T - kSliceGranule) <= room; ++i)
      T -= kSliceGranule;
    total = count(T);
  }
  // One round cannot always be level: when batch * heads (nearly) fills it, long and short sequences are
  // each one slice.  If the largest slice is then well above the average and large in itself, several
  // rounds of kLargeSlice-sized slices do better: their start-up hides behind the neighbours' streaming and
  // the hardware deals them to whichever CU is free.  (Level plans are left alone: cutting them further
  // only adds partial states; measured 2-4 % slower.)  The slice table bounds the number of slices.
  {
    int64_t largest_now = 1;
    for (int32_t b = 0; b < d->batch; ++b) {
      const int64_t n = tokens(b), per = ceil_div(n, cut(n, T));
      if (per > largest_now) largest_now = per;
    }
    if (largest_now > kLargeSlice && 2 * largest_now * total > 3 * sum) {
      int64_t T2 = kLargeSlice;
      while (T2 < T && count(T2) > kMaxPlanSlices) T2 += kLargeSlice / 4;
      if (T2 < T) {
        T = T2;
        total = count(T);
      }
    }
  }
  int64_t most = 1, least = kMaxPlanSplits + 1, largest = 1;
  for (int32_t b = 0; b < d->batch; ++b) {
    const int64_t n = tokens(b), nsl = cut(n, T);
    if (nsl > most) most = nsl;
    if (nsl < least) least = nsl;
    if (ceil_div(n, nsl) > largest) largest = ceil_div(n, nsl);
  }
  if (most != least) {  // sequences differ in their number of slices: the table is needed, and must fit
    if (total > kMaxPlanSlices || most > kMaxPlanSplits) return false;
    if (table) {
      int32_t y = 0;
      for (int32_t b = 0; b < d->batch; ++b) {
        const int64_t nsl = cut(tokens(b), T);
        for (int64_t s = 0; s < nsl; ++s) table[y++] = pack_slice((uint32_t)b, (uint32_t)s, (uint32_t)nsl);
      }
    }
  } else if (most > 65535) {
    return false;  // grid.y limit of the plain grid
  }
  p->exact = most != least;  // same count for every sequence: a (heads, slices, batch) grid says it all
  p->even = true;
  p->least_slice = 0;
  p->num_splits = (int32_t)most;
  p->slice_tokens = (int32_t)largest;
  p->max_tokens = (int32_t)max_tok;
  p->total_slices = (int32_t)total;
  p->queries_per_pass = queries_per_pass(d);
  p->granule = (int32_t)T;
  p->whole = (int32_t)whole;
  p->runs = false;
  return true;
}

static bool has_host_lists(const span_attn_desc_t* d) {
  return d->host_span_offsets && (d->num_intervals == 0 || (d->host_span_starts && d->host_span_ends));
}

// From the host copies of the span lists the positions are counted with the clamps the kernel applies to the device lists (interval
// indices to [0, num_intervals], lengths to [0, max_len]).
TokenCounts::TokenCounts(const span_attn_desc_t* d) : from_lists(has_host_lists(d) && d->batch <= kMaxPlanBatch), of(d->tokens_per_seq) {
  if (!from_lists) return;
  for (int32_t b = 0; b < d->batch; ++b) {
    const int32_t lo = std::min(std::max(d->host_span_offsets[b], 0), d->num_intervals);
    const int32_t hi = std::min(std::max(d->host_span_offsets[b + 1], lo), d->num_intervals);
    int64_t n = 0;
    for (int32_t i = lo; i < hi; ++i)
      n += std::min<int64_t>(std::max<int64_t>((int64_t)d->host_span_ends[i] - d->host_span_starts[i], 0), d->max_len);
    counted_[b] = n;
  }
  of = counted_;
}

// Run mode: resolves each slice of an exact plan to its runs of consecutive cache positions.  Sequence b has
// n_b attended positions, numbered 0 .. n_b-1 along its interval list, and ceil(n_b / granule) slices (or one) that share
// them evenly (as the kernel cuts them when it walks the device lists itself).  False if the plan does not fit the
// tables or a slice is larger than one position window per wave allows.
static bool plan_runs(const span_attn_desc_t* d, const int64_t* tokens_per_seq, const Partition& p, RunTables* r) {
  if (!p.even || d->batch > kMaxPlanBatch || p.total_slices > kMaxRunSlices) return false;
  int32_t y = 0, nruns = 0;
  for (int32_t b = 0; b < d->batch; ++b) {
    int64_t n = tokens_per_seq[b] < 0 ? 0 : tokens_per_seq[b];
    if (n > p.max_tokens) n = p.max_tokens;
    const int64_t nsl = slices_for(n, p.granule, p.whole), T = ceil_div(n, nsl);
    if (T > kMaxRunSliceRows || nsl > kMaxPlanSplits) return false;
    const int32_t lo = std::min(std::max(d->host_span_offsets[b], 0), d->num_intervals);
    const int32_t hi = std::min(std::max(d->host_span_offsets[b + 1], lo), d->num_intervals);
    int32_t i = lo;        // interval the walk stands in
    int64_t before = 0;    // attended positions of the intervals before it
    for (int64_t s = 0; s < nsl; ++s) {
      if (y >= kMaxRunSlices) return false;
      const int64_t v0 = s * T, v1 = std::min(n, (s + 1) * T);  // the slice owns positions number v0 .. v1-1
      const int32_t first_run = nruns;
      for (int64_t v = v0; v < v1;) {
        int64_t len = 0;
        while (i < hi) {  // skip to the interval that holds position number v
          len = std::min<int64_t>(std::max<int64_t>((int64_t)d->host_span_ends[i] - d->host_span_starts[i], 0), d->max_len);
          if (v < before + len) break;
          before += len;
          ++i;
        }
        if (i >= hi) return false;  // (cannot happen: n was summed over the same list)
        const int64_t take = std::min(v1, before + len) - v;
        if (nruns >= kMaxRuns) return false;
        r->run[nruns][0] = (int32_t)std::min<int64_t>(std::max<int64_t>((int64_t)d->host_span_starts[i] + (v - before), INT32_MIN), INT32_MAX);
        r->run[nruns][1] = (int32_t)take;
        ++nruns;
        v += take;
      }
      r->slices[y].entry = pack_slice((uint32_t)b, (uint32_t)s, (uint32_t)nsl);
      r->slices[y].runs_of = (uint32_t)first_run | ((uint32_t)(nruns - first_run) << 16);
      r->slices[y].rows = (int32_t)(v1 > v0 ? v1 - v0 : 0);
      r->slices[y].reserved = 0;
      ++y;
    }
  }
  return y == p.total_slices;
}

// Uniform mode: every sequence gets the same number of slices, sized from the bound so that a call puts about as many workgroups
// on the chip as slice_room says, never fewer than kMinSlice positions per slice.  The kernel counts every sequence itself and shares
// its positions evenly between its slices (least_slice) - cut at the bound's size, all but the first were short or empty.  us, cut
// at the bound -> shared: 32 x 32 heads x 5..50 % of 4096..16384, bf16 274 -> 236; 16 x 32 x ~560, fp16 38.7 -> 35.7; 20 x 32 x 300..1000
// dense 42.9 -> 38.4; 40 x 16 x 300..900 dense of 64 23.5 -> 22.5.  With kBoundSlice as well (span form): 24 x 12 x 5..50 % of 2000..5000,
// bf16 41.0 -> 31.0 (38.9 shared alone), 16 x 16 x 5..50 % of 1200..4000 fp32 of 64 24.6 -> 19.2 (22.7); slices of up to 256 or 384 win and
// lose 5 % against 512.  Dense contexts, which are less ragged, lose by more slices (8 x 32 x 600..2000 33.4 -> 36.2), and so do up to eight
// sequences whose spans come near the bound, fp16: 4 x 32 x 3000..3100 36.8 -> 38.7, 8 x 16 x 3000..3200 37.3 -> 39.3, 8 x 32 x 1500..1600 35.7 -> 36.5;
// with more they do not (9 x 32 x 1500..1600 41.8, 45.3 in three slices).  It costs small batches far below their bound what it gains large
// ones: 8 x 32 x 5..50 % of 2000..16000 64.3, 44.7 if cut, 4 x 32 x 5..50 % of 4000..16000 35.9 and 29.3.
Partition plan_partition(const span_attn_desc_t* d, const TokenCounts& counts, uint32_t* table, RunTables* runs, bool spans, ShortRules rules) {
  const int64_t max_tok = (d->max_tokens > 0 && d->max_tokens < d->max_len) ? d->max_tokens : d->max_len;
  Partition p;
  if (plan_exact(d, counts.of, max_tok, rules, &p, table)) {
    // Run mode is used where the launch carries a slice table anyway (sequences with different numbers of slices):
    // kernel arguments of that size cost a few tenths of a microsecond per launch, which a batch that needs no
    // table would pay on top (measured: batch 64 x 155 positions, one slice each, 27.7 -> 27.9 us with runs).  Against the table and the
    // device lists, on the same buffers: 10 x 12 heads x ~560, fp16 12.1 -> 11.7, 8 x 32 x ~560 18.0 -> 17.9, 16 x 32 x ~550 30.6 and 30.6, 12 x 32 x ~500,
    // bf16 22.3 -> 22.7, 20 x 16 x ~500 20.65 -> 21.2.  The matrix kernel takes no runs.
    if (counts.from_lists && runs && p.exact && !runs_on_matrix_cores(d)) p.runs = plan_runs(d, counts.of, p, runs);
    return p;
  }
  const int64_t pairs = (int64_t)d->batch * d->heads;
  int64_t splits = d->num_splits > 0 ? d->num_splits : slice_room(d) / d->batch;  // stay within one round
  if (d->num_splits == 0 && spans && d->num_intervals > 0 && query_tokens(d) == 1 && d->batch > kBoundSliceFromBatch) {
    // A bound far above what most sequences attend leaves few large slices for the longest: up to kBoundSlice each.
    const int64_t in_round = target_workgroups(d) / d->heads / d->batch;
    while (splits > 0 && splits < in_round && ceil_div(max_tok, splits) > kBoundSlice) ++splits;
  }
  const int64_t whole = unsliced_up_to(d, rules), fine = slices_for(max_tok, kFineSlice, whole);
  const int64_t most = rules == ShortRules::kApplied && fine_slices(d) && fine <= splits ? fine : slices_for(max_tok, kMinSlice, whole);
  if (d->num_splits == 0 && splits > most) splits = most;
  if (splits > max_tok) splits = max_tok;
  if (splits < 1) splits = 1;
  int64_t slice = ceil_div(ceil_div(max_tok, splits), kSliceGranule) * kSliceGranule;
  if (slice > kMaxSlice) slice = kMaxSlice;
  while (ceil_div(max_tok, slice) > 65535) slice += kSliceGranule;  // grid.y limit
  splits = ceil_div(max_tok, slice);
  p.exact = false;
  p.even = false;
  p.least_slice = d->num_splits == 0 ? kLeastSlice : 0;
  p.num_splits = (int32_t)splits;
  p.slice_tokens = (int32_t)slice;
  p.max_tokens = (int32_t)max_tok;
  p.total_slices = (int32_t)(splits * d->batch);
  p.queries_per_pass = queries_per_pass(d);
  p.granule = (int32_t)slice;
  p.whole = 0;
  p.runs = false;
  return p;
}

// Few-query calls on the matrix cores: all tokens of the call in one launch, a workgroup serving up to 64 of them with
// one pass over its rows.
//
// From three tokens on for every type and head_dim, two tokens see below.  Measured against the passes it replaces (four
// tokens on the vector units, sixteen on the matrix cores, one launch per pass): batch 16 x ~380 positions, 16 heads x 64, fp16, 9 tokens
// 63.9 -> 14.7 us; batch 8 x ~600, 32 heads x 128, fp32, 8 tokens 83.6 -> 39.7 us; 3 tokens, batch 16 x ~370, fp32 49.9 ->
// 45.3 us; batch 16 x ~700, bf16, 32 tokens 96.4 -> 50.1 us; batch 32 x 1000, bf16, 64 tokens 313 -> 130 us.
//
// Slices.  512 workgroups a call (two per CU; no more where no more run at once: a few workgroups in a second round double the time, 43 slices
// per head of 12 heads are 516: us, 43 -> 42: 8 x 12 x ~1800 positions fp32, 6 tokens 54.8 -> 42.3; 24 x 5 x ~1700 fp16, 46 tokens 58.3 -> 49.8; 4 x
// 12 x 300..2800 fp32, 4 tokens 23.5 -> 22.2), but one slice per sequence at least and 1024, 768 or 512 workgroups at most for 16, 32 or 64 tokens a
// workgroup (one resident round of rows of 64; fp32 rows of 128, and 16-bit ones of more than 16 tokens, run two a CU and take up to two): of 256,
// 512, 768 and 1024, 512 is within 3 % of the best or the best at 18 of 20 larger shapes (for smaller ones see one_per_cu_pays); more only pays for itself in partial states, which grow with the
// tokens (batch 16 x ~700, 32 tokens, 16 slices per head against 32: 50.4 and 59.3 us). The slices have to fit the workspace's token states, so
// sequences that stay in one slice, which need no state, come after the others in the table. Groups. A workgroup that serves all tokens reads every
// row once; where the batch has too few (batch, head) pairs to fill the chip that way (fewer than 128 workgroups before slicing), several workgroups
// share a slice's rows through the L2, each for its own tokens: 12 heads x 8, 60 tokens 36.1 us with 64 tokens a workgroup, 29.2 us with 32; 32 pairs
// x 1500 fp32 positions, 30 tokens 38.9 -> 31.1 us; 256 pairs, 24 tokens 22.2 us in two workgroups, 18.9 us in one.
constexpr int32_t kMatrixFromTokens = 3;
// Two tokens: 16-bit rows and few (batch, head) pairs, where the start-up and the hand-over count and the matrix kernel's
// are shorter; many pairs stream better through the vector kernel's 24 waves per CU.  us, vector -> matrix: 64 pairs of 128
// 10.4 -> 9.4 (32 pairs), 20.3 -> 18.0 (192), 23.6 -> 22.4 (256), 28.4 -> 29.2 (384), 33.8 -> 35.7 (512); of 64 20.9 -> 16.3
// (288), 23.8 -> 23.4 (512), 33.7 -> 36.8 (1536); fp32 rows 25.9 -> 26.8 (128), 49.9 -> 54.7 (1024).  (With fp16 weights in two
// terms; the third that they have now costs 1 %.)
constexpr int64_t kMatrixTwoTokenColumns = 32768;  // pairs x head_dim
constexpr int64_t kMatrixWorkgroups = 512;
constexpr int64_t kMatrixPairs = 128;
constexpr int32_t kMatrixMaxFieldSlices = 255;  // slices of a pair when several query blocks share its ticket counter

bool runs_on_matrix_cores(const span_attn_desc_t* d) {
  const int32_t n = query_tokens(d);
  if (n >= kMatrixFromTokens) return true;
  return n == 2 && d->dtype != SPAN_F32 && (int64_t)d->batch * d->heads * d->head_dim <= kMatrixTwoTokenColumns;
}

// Token states per head.  Every sliced call brings those of its Partition (from three tokens on that does not depend on how
// many they are); a few-query call can use more where that pool holds few slices for all its tokens at once (8 sequences x 32
// heads x ~600 positions, 8 tokens, fp32 rows of 128: 44.5 us with the Partition's pool, 39.7 with twice that; 16 x 16 x ~380,
// 9 tokens, fp16 rows of 64: 14.9 and 14.3), up to a whole round of 1024 workgroups and, where the (batch, head) pairs alone
// do not fill the chip, kUnsplitFromPairs workgroups with all tokens of the call.
int64_t least_states(const Partition& p) { return p.num_splits > 1 ? (int64_t)p.total_slices * p.queries_per_pass : 0; }

int64_t most_states(const span_attn_desc_t* d, const Partition& p) {
  const int64_t least = least_states(p);
  if (least == 0 || p.queries_per_pass <= 2 || d->num_splits > 0) return least;
  int64_t slices = target_workgroups(d) / d->heads * p.queries_per_pass;
  if ((int64_t)d->batch * d->heads < kUnsplitFromPairs) slices = std::max(slices, ceil_div(kUnsplitFromPairs, d->heads) * query_tokens(d));
  return std::max(least, std::min<int64_t>(slices, (int64_t)kMaxPlanSlices * p.queries_per_pass));
}

// Workgroups go to the CUs in turns of 256, heads fastest: table entries of a turn.
constexpr int32_t kTurn = 256;  // CUs (a column fits 8 bits)
static int32_t turn_entries(int32_t heads) { return (kTurn + heads / 2) / heads; }

// Slices of a few-query call: one workgroup per CU at most, or the 512 wanted? Where both run at once a second workgroup on a CU costs almost what it
// does, so the plan with one pays (where the lengths are known) unless its largest slice is longer than what the fullest CU gets of the other plan,
// by a factor that is how much better two hide each other's trips. It pays a hand-over's worth more if it cuts nothing. us, up to 512 workgroups ->
// up to 256, level sequences: fp16 rows of 128, 4 tokens: 96 pairs x 300 positions 9.4 -> 9.1, 128 x 512 11.4 -> 11.1, 160 x 256 9.5 -> 8.2, x 400
// 11.5 -> 10.9, x 640 14.5 -> 15.9, 224 x 512 15.4 -> 13.8, 256 x 400 14.4 -> 12.3; 16 tokens: 32 x 1500 12.9 -> 11.1, 128 x 512 12.6 -> 11.6, 160 x
// 512 14.1 -> 13.7, x 1000 21.2 -> 22.9, 224 x 512 17.0 -> 14.3; 32 tokens: 256 x 256 14.9 -> 11.4; 64 tokens: 160 x 256 20.2 -> 15.6, 256 x 400 26.1
// -> 21.7; fp32, 4 tokens: 128 x 512 18.3 -> 17.2, 160 x 300 16.9 -> 16.0, x 512 21.2 -> 22.8, 256 x 400 25.1 -> 22.35; 32 tokens: 160 x 400 28.8 ->
// 30.0; fp16 of 64, 4 tokens: 96 x 512 8.85 -> 8.5, x 640 9.0 -> 9.6, 192 x 512 10.15 -> 9.9; fp32 of 64, whole: 192 x 400 14.4 -> 14.2, x 512 14.9
// -> 16.4, 256 x 400 15.0 -> 13.7, but not cut: 64 x 640 in four 10.4 -> 10.95, 65 x ~800 11.2 -> 11.55. Longer slices gain less, and fewer
// workgroups than five in eight CUs lose (3 workgroups a slice, 48 pairs x ~300, 44 tokens 11.4 -> 12.3): both are left as they were. Where the
// (batch, head) pairs alone are no more than one per CU, a sequence of up to 256 positions (fp32 rows of 64: 192; of 128: 128) stays whole anyway,
// three or four tiles a wave: 256 positions in two slices -> whole, fp16 of 128, 16 tokens: 8 pairs 7.6 -> 7.4, 96 8.4 -> 8.05, 256 12.2 -> 9.4; of
// 64 6.7 -> 5.9, 7.2 -> 6.6, 9.2 -> 7.0; fp32 of 64, 160 positions 8.1 -> 7.6 (8 pairs), 200 8.0 -> 8.9.
struct SliceCost {
  int64_t slices, largest, rows;  // slices, positions of the largest, positions of all
  bool cuts;                      // some sequence has several
};
constexpr int64_t kOnePerCuFrom = 160;  // workgroups
constexpr int64_t kOnePerCuWholeUpTo = 512, kOnePerCuSliceUpTo = 384;  // positions
static bool one_per_cu_pays(const span_attn_desc_t* d, int64_t workgroups_per_slice, const SliceCost& one, const SliceCost& more) {
  constexpr int64_t kStart = 64, kHandOver = 64;  // positions
  if (one.largest > (one.cuts ? kOnePerCuSliceUpTo : kOnePerCuWholeUpTo) || one.slices * workgroups_per_slice < kOnePerCuFrom) return false;
  if (one.cuts && d->dtype == SPAN_F32 && d->head_dim == 64) return false;
  const int64_t percent = d->dtype == SPAN_F32 ? (d->head_dim == 128 ? 95 : 65) : (d->head_dim == 128 ? 110 : 90);
  const int64_t turns = ceil_div(more.slices * workgroups_per_slice, 256), fullest = std::max(more.largest, turns * ceil_div(more.rows, more.slices));
  return one.largest * 100 <= fullest * percent + 100 * (kStart + (!one.cuts && more.cuts ? kHandOver : 0));
}

// False if no plan of up to `most_slices` slices could: known from the lengths alone, without looking for its slices.
static bool one_per_cu_may_pay(int64_t workgroups_per_slice, int64_t most_slices, int64_t longest, int64_t rows) {
  return most_slices * workgroups_per_slice >= kOnePerCuFrom && (longest <= kOnePerCuWholeUpTo || ceil_div(rows, most_slices) <= kOnePerCuSliceUpTo);
}

bool plan_matrix(const span_attn_desc_t* d, const TokenCounts& counts, const Partition& p, int64_t states, MatrixPlan* m, uint32_t* table, bool two_per_cu) {
  int32_t n = query_tokens(d);
  if (!runs_on_matrix_cores(d)) return false;
  const bool sliced = p.num_splits > 1;
  m->states = 0;
  m->tokens = n;
  m->table = false;
  m->even = p.even;
  m->least_slice = p.least_slice;
  m->num_splits = p.num_splits;
  m->slice_tokens = p.slice_tokens;
  m->total_slices = p.total_slices;
  const int32_t elt_bytes = d->dtype == SPAN_F32 ? 4 : 2, max_groups = kMatrixMaxGroups(elt_bytes, d->head_dim);
  auto groups_for = [&](int64_t tokens) { return std::min<int32_t>(max_groups, tokens <= 16 ? 1 : (tokens <= 32 ? 2 : 4)); };
  if (d->num_splits > 0) {  // the caller's number of slices stands: as many tokens a launch as their states fit
    if (sliced && n > p.queries_per_pass) m->tokens = p.queries_per_pass;
    if (sliced) m->states = (int64_t)m->total_slices * m->tokens;
    m->groups = groups_for(m->tokens);
    while ((int64_t)d->batch * ceil_div(m->tokens, 16 * m->groups) > 65535) m->tokens = 16 * m->groups;  // (grid.z limit)
    return true;
  }
  m->groups = groups_for(n);
  const int64_t pairs = (int64_t)d->batch * d->heads;
  auto blocks_for = [&](int32_t groups) { return ceil_div(n, 16 * groups); };
  while (m->groups > 1 && pairs * blocks_for(m->groups) < kMatrixPairs) m->groups /= 2;
  if (d->batch * blocks_for(m->groups) > 65535) m->tokens = n = 16 * m->groups;  // (grid.z limit)
  const int64_t blocks = blocks_for(m->groups);
  const int64_t at_once = (int64_t)kTurn * kMatrixWorkgroupsPerCu(elt_bytes, d->head_dim, m->groups);
  const int64_t most = kTurn * kMatrixWorkgroupsPerCu(2, 64, m->groups) / (d->heads * blocks);
  const int64_t wanted = std::min<int64_t>(ceil_div(kMatrixWorkgroups, d->heads * blocks), two_per_cu ? most : std::max<int64_t>(1, at_once / (d->heads * blocks)));
  const int64_t room = std::max<int64_t>(1, std::min(std::max<int64_t>(wanted, d->batch), most));
  const int64_t whole = two_per_cu || pairs * blocks > kTurn ? 0 : (elt_bytes == 2 ? 256 : (d->head_dim == 64 ? 192 : 0));  // see one_per_cu_pays
  if (!p.even) {  // the counts are not known: every sequence gets the same number of slices
    if (!sliced) return true;
    int64_t splits = std::min<int64_t>(room / d->batch, states / ((int64_t)d->batch * n));
    splits = std::min<int64_t>(std::min<int64_t>(splits, blocks > 1 ? kMatrixMaxFieldSlices : 65535), slices_for(p.max_tokens, kMinSlice, whole));
    if (splits < 1) splits = 1;
    int64_t slice = std::min<int64_t>(ceil_div(ceil_div(p.max_tokens, splits), kSliceGranule) * kSliceGranule, kMaxSlice);
    m->num_splits = (int32_t)ceil_div(p.max_tokens, slice);
    m->slice_tokens = (int32_t)slice;
    m->total_slices = m->num_splits * d->batch;
    if (m->num_splits > 1) m->states = (int64_t)m->total_slices * n;
    return true;
  }
  // (Clamped once and divided in 32 bits, and no second search where the first one's size fits: host time is what a plan costs, every call has one.  us, plan and
  // order of the slices, in 64 bits, clamped each time, searched for up to three times -> so: 8 x 32 heads x 400..700, 8 tokens 1.19 -> 0.75; 30 x 8 x
  // 100..500, 12 tokens 4.0 -> 3.1; 64 x 5 x 300..3000, 20 tokens 12 -> 9; 200 x 2 x 300..3000, 8 tokens 36 -> 25.)
  uint32_t length[kMaxPlanBatch];
  uint32_t longest_of_all = 1;
  int64_t sum = 0;
  for (int32_t b = 0; b < d->batch; ++b) {
    length[b] = (uint32_t)std::min<int64_t>(std::max<int64_t>(counts.of[b], 0), p.max_tokens);
    longest_of_all = std::max(longest_of_all, length[b]);
    sum += length[b];
  }
  auto cut_sequence = [&](int32_t b, int64_t t) { return length[b] <= (uint32_t)whole ? 1u : (length[b] + (uint32_t)t - 1) / (uint32_t)t; };
  // `cap` slices at most, and those of the sequences with several fit the slots
  auto fits = [&](int64_t t, int64_t cap, int64_t room_for) {
    int64_t total = 0, in_slots = 0;
    for (int32_t b = 0; b < d->batch; ++b) {
      const uint32_t s = cut_sequence(b, t);
      if (s > (uint32_t)(blocks > 1 ? kMatrixMaxFieldSlices : kMaxPlanSplits)) return false;
      total += s;
      if (s > 1) in_slots += s;
    }
    return total <= cap && in_slots * n <= room_for;
  };
  int64_t T = std::max<int64_t>(p.max_tokens, 1);
  // smallest slice size from `from` on that fits (the counts fall as it grows); T where none below it does
  auto smallest_fit = [&](int64_t from, int64_t cap, int64_t room_for) {
    int64_t lo = 0, hi = T > from ? ceil_div(T - from, kSliceGranule) : 0;  // in granules above `from`; hi always fits
    while (lo < hi) {
      const int64_t mid = (lo + hi) / 2;
      if (fits(from + mid * kSliceGranule, cap, room_for)) hi = mid;
      else lo = mid + 1;
    }
    return std::min(T, from + hi * kSliceGranule);
  };
  if (sliced) {
    if (room >= d->batch) {
      auto smallest = [&](int64_t cap, int64_t room_for) { return smallest_fit(std::max<int64_t>(kMinSlice, ceil_div(sum, cap)), cap, room_for); };
      const int64_t cap = std::min<int64_t>(room, kMaxPlanSlices), fewer = std::min(cap, kTurn / (d->heads * blocks));
      auto cost = [&](int64_t t) {
        SliceCost c{0, 0, sum, false};
        for (int32_t b = 0; b < d->batch; ++b) {
          const uint32_t s = cut_sequence(b, t);
          c.slices += s;
          c.largest = std::max<int64_t>(c.largest, (length[b] + s - 1) / s);
          c.cuts = c.cuts || s > 1;
        }
        return c;
      };
      // (chosen as with the largest workspace the call can use, so that what span_workspace_bytes asks for is enough for the same plan)
      const int64_t all = most_states(d, p), per_slice = d->heads * blocks;
      int64_t chosen = cap, T_chosen = 0;  // slices at most, and the size that `all` states allow (0: not looked for)
      if (!two_per_cu && fewer >= d->batch && fewer < cap && one_per_cu_may_pay(per_slice, fewer, longest_of_all, sum)) {
        const int64_t T_cap = smallest(cap, all), T_fewer = smallest(fewer, all);
        T_chosen = T_cap;
        if (T_fewer > T_cap && one_per_cu_pays(d, per_slice, cost(T_fewer), cost(T_cap))) {
          chosen = fewer;
          T_chosen = T_fewer;
        }
      }
      // (the smallest that fits more states is the smallest here too if it fits)
      T = T_chosen > 0 && (states >= all || fits(T_chosen, chosen, states)) ? T_chosen : smallest(chosen, states);
    }
    // as in plan_exact: slices well above the average and large in themselves run in several rounds of smaller ones
    int64_t total = 0, largest = 1;
    for (int32_t b = 0; b < d->batch; ++b) {
      const uint32_t s = cut_sequence(b, T);
      total += s;
      largest = std::max<int64_t>(largest, (length[b] + s - 1) / s);
    }
    if (largest > kLargeSlice && 2 * largest * total > 3 * sum) T = smallest_fit(kLargeSlice, kMaxPlanSlices, states);
  }
  int64_t total = 0, longest = 1, most_s = 1, least_s = kMaxPlanSplits + 1;
  for (int32_t b = 0; b < d->batch; ++b) {
    const int64_t s = cut_sequence(b, T);
    total += s;
    if (s > 1) m->states += s * n;
    most_s = std::max(most_s, s);
    least_s = std::min(least_s, s);
    longest = std::max<int64_t>(longest, (length[b] + (uint32_t)s - 1) / (uint32_t)s);
  }
  m->num_splits = (int32_t)most_s;
  m->slice_tokens = (int32_t)longest;
  m->total_slices = (int32_t)total;
  // Whole sequences of unequal length, more workgroups than run at once, in launches that deal_slices does not take: several
  // query blocks, each a grid of its own behind the last, or heads that fill a turn alone.  The longest go first, which is what free CUs
  // should find, and every second turn runs backwards, so that the CUs get long and short ones alike.  us in list order -> so:
  // fp32 rows of 128, 16 x 32 heads x 400..1000 positions, 64 tokens 167.0 -> 159.9; 48 x 16 x 200..900, 48 tokens 212.3 -> 193.1; 36 x 12 x 300..1000, 40
  // tokens 150.2 -> 127.3 (dealt by the rule for one block 146.2); rows of 64, 200..900: 12 x 200, fp16, 8 tokens 61.4 -> 57.6; 8 x 256 fp32, 64 tokens
  // 231.9 -> 223.4; all at once, where the table is all that it adds: 5 x 200, 8 tokens 26.4 -> 26.8, 3 x 300 26.8 -> 27.4.
  const int32_t row = std::max<int32_t>(1, kTurn / d->heads);
  if (most_s == 1 && (blocks > 1 || turn_entries(d->heads) < 2) && d->batch > row && d->batch <= kMaxPlanSlices && pairs * blocks > at_once &&
      longest * 100 * d->batch > 115 * sum) {
    uint64_t by_length[kMaxPlanSlices];  // positions << 16 | sequence
    for (int32_t b = 0; b < d->batch; ++b) by_length[b] = (uint64_t)length[b] << 16 | (uint64_t)b;
    std::sort(by_length, by_length + d->batch, [](uint64_t x, uint64_t y) { return x > y; });
    for (int32_t r = row; r < d->batch; r += 2 * row) std::reverse(by_length + r, by_length + std::min(r + row, d->batch));
    m->table = true;
    for (int32_t y = 0; y < d->batch; ++y) table[y] = pack_slice((uint32_t)(by_length[y] & 0xffff), 0, 1);
  } else if (most_s != least_s) {
    m->table = true;
    int32_t y = 0;
    for (int pass = 0; pass < 2; ++pass) {
      for (int32_t b = 0; b < d->batch; ++b) {
        const int64_t s = cut_sequence(b, T);
        if ((s > 1) != (pass == 0)) continue;
        for (int64_t i = 0; i < s; ++i) table[y++] = pack_slice((uint32_t)b, (uint32_t)i, (uint32_t)s);
      }
    }
  }
  return true;
}

// Workgroups go to the CUs in turns of 256, heads fastest, so with 32 heads the table entries y, y + 8, y + 16, .. run on the same
// CUs, and the launch lasts as long as the CU with the most rows (stamps by CU: its last row is read in step with its rows, correlation 0.7
// to 0.94).  In plan order that is up to 30 % more than the mean (batch 16 x ~550 positions in 31 slices: 1454 rows on a CU, 1105 on
// average).  So: the largest slices first, turn by turn, the largest of each turn to the CUs that have the least so far;
// the smallest slices, which a last, partial turn will hold, are counted ahead.  With more workgroups than run at once the order
// still is one of falling size, which is what free CUs should find.  us in plan order -> dealt, 32 heads x 128 unless said
// otherwise: 32 x ~2700 positions in 64 slices, bf16 230 -> 222; 64 x ~800 121.5 -> 118.4; 40 x 400..2000 dense 127.5 -> 124.3; 32 x ~560, 64
// tokens 117 -> 106; 60 x ~300 of 64, 5 tokens 55.4 -> 53.5; 8 x ~600 fp32, 24 tokens 49.7 -> 47.2; 16 x 16 heads x ~380 of 64, 9
// tokens 14.4 -> 13.9; batch 16 x ~550 31.2 -> 30.2.  The host pays 0.5 us for 30 slices, 1 for 64, 2.5 for 165 (the whole plan
// 1.3 -> 1.9 us, 2.8 -> 3.7, 5.5 -> 8.0).
// In less than two turns of few-query workgroups most CUs hold one, and the hand-over of a slice's states counts as well: as this many
// rows, which puts the slices of cut sequences ahead of short whole ones.  us in plan order -> dealt by rows alone -> with the hand-over:
// fp32, 35 x 8 heads x 60..160 positions, 17 tokens 21.1 -> 24.1 -> 21.4; 25 x 8 x ~150 of 64, 3 tokens 9.05 -> 9.63 -> 9.04; bf16, 25 x 16 x 108..216 of
// 64, two tokens 7.99 -> 8.81 -> 8.38; 41 x 12 x 599..999 fp32 of 64, 47 tokens 95.1 -> 81.3 -> 81.1; 12 x 32 x ~200, 24 tokens 35.1 -> 33.6 -> 33.3;
// the most it costs: bf16, 14 x 16 x ~600, 13 tokens 21.9 -> 20.7 -> 21.1. (64 rows do as well but for 30 x 12 x 60..250, 20 tokens, 25.7 -> 26.9 and
// 25.6 with 128.) Whole sequences, 63 x 8 x 53..268, fp16, 59 tokens 26.5 -> 23.3; 12 x 40 x 345..1151, bf16, 46 tokens 57.6 -> 50.8. One-token
// launches, whose hand-over is a single state, gain nothing by it (geometric mean of 100 shapes 1.000).
constexpr int32_t kHandOverRows = 128;
// A launch whose plan needs no table carries one where that spares the fullest CU 5 % and this many bytes (its share of 0.6 us; the table's
// 3 KB of arguments cost 0.35).  us, without -> with: 64 x 12 heads x 60..200 of 64, 16 tokens 10.5 -> 9.65; 8 x 32 x 500..900, two slices each, two
// tokens 20.0 -> 19.5; 10 x 32 x 300..500, two tokens 16.7 -> 16.2; 64 x 32 x 100..300, one token 35.1 -> 34.4; 60 x 32 x 150..450 of 64, 5 tokens
// 29.9 -> 29.4. Less to spare is left alone: 64 x 144..168 28.4 with and without; 28 x 160 x 200..900 of 64, 8 tokens 111.3, 108.9 with.
constexpr int64_t kDealTableBytes = 16384;

void deal_slices(const span_attn_desc_t* d, const TokenCounts& counts, int64_t max_tokens, int32_t total, int32_t hand_over, bool table,
                 uint32_t* entries, Deal* deal) {
  deal->dealt = false;
  const int32_t columns = turn_entries(d->heads);
  if (columns < 2 || total <= columns || total > kMaxPlanSlices) return;
  // rows of every slice, and what the CUs of a column get in plan order
  uint64_t by_rows[kMaxPlanSlices];  // rows << 16 | slice
  int64_t load[kTurn] = {};
  int64_t all_rows = 0;
  int32_t b_last = 0, most = 1;
  for (int32_t i = 0, column = 0; i < total; ++i, column = column + 1 < columns ? column + 1 : 0) {
    const int32_t b = (int32_t)(entries[i] & 1023u), split = (int32_t)((entries[i] >> 10) & 2047u), nsl = (int32_t)(entries[i] >> 21);
    int32_t rows = (int32_t)std::min<int64_t>(std::max<int64_t>(counts.of[b], 0), max_tokens);
    if (nsl > 1) {
      const int32_t T = (int32_t)(((uint32_t)rows + (uint32_t)nsl - 1) / (uint32_t)nsl);
      rows = std::min(std::max(rows - split * T, 0), T) + hand_over;
    }
    by_rows[i] = (uint64_t)rows << 16 | (uint64_t)i;
    load[column] += rows;
    all_rows += rows;
    b_last = std::max(b_last, b);
    most = std::max(most, nsl);
  }
  const int64_t plain_most = *std::max_element(load, load + columns);
  const int64_t row_bytes = 2 * (int64_t)d->head_dim * (d->dtype == SPAN_F32 ? 4 : 2);
  auto pays = [&](int64_t dealt_most) {
    const int64_t spared = plain_most - dealt_most;
    return spared > 0 && (table || (spared * row_bytes >= kDealTableBytes && spared * 20 >= dealt_most));
  };
  if (!pays(ceil_div(all_rows, columns))) return;  // (not even with the rows shared perfectly)
  int32_t b_bits = 1;
  while (b_last >> b_bits) ++b_bits;
  const int32_t n_bits = (32 - kSlotBits - b_bits) / 2;
  if (most >> n_bits) return;
  std::sort(by_rows, by_rows + total, [](uint64_t x, uint64_t y) { return x > y; });
  const int32_t turns = total / columns, rest = total % columns;  // whole turns, entries of the last one
  uint64_t by_load[kTurn];  // rows so far << 8 | column
  for (int32_t c = 0; c < columns; ++c) by_load[c] = (c < rest ? by_rows[total - 1 - c] >> 16 << 8 : 0) | (uint64_t)c;
  for (int32_t c = 0; c < rest; ++c) deal->at[by_rows[total - 1 - c] & 0xffff] = (uint16_t)(turns * columns + c);
  for (int32_t t = 0; t < turns; ++t) {
    std::sort(by_load, by_load + columns);
    for (int32_t k = 0; k < columns; ++k) {
      const uint64_t s = by_rows[t * columns + k];
      deal->at[s & 0xffff] = (uint16_t)(t * columns + (int32_t)(by_load[k] & 0xff));
      by_load[k] += s >> 16 << 8;
    }
  }
  if (!pays((int64_t)(*std::max_element(by_load, by_load + columns) >> 8))) return;
  if (hand_over > 0) {  // (an estimate: the rows alone must get more level as well)
    int64_t rows_plain[kTurn] = {}, rows_dealt[kTurn] = {};
    for (int32_t k = 0; k < total; ++k) {
      const int32_t i = (int32_t)(by_rows[k] & 0xffff);
      const int64_t rows = (int64_t)(by_rows[k] >> 16) - (entries[i] >> 21 > 1 ? hand_over : 0);
      rows_plain[i % columns] += rows;
      rows_dealt[deal->at[i] % columns] += rows;
    }
    if (*std::max_element(rows_dealt, rows_dealt + columns) >= *std::max_element(rows_plain, rows_plain + columns)) return;
  }
  uint32_t dealt[kMaxPlanSlices];
  for (int32_t i = 0; i < total; ++i)
    dealt[deal->at[i]] = (entries[i] & 1023u) | ((entries[i] >> 10) & 2047u) << b_bits | (entries[i] >> 21) << (b_bits + n_bits) |
                         (uint32_t)i << (32 - kSlotBits);
  std::copy(dealt, dealt + total, entries);
  deal->b_bits = b_bits;
  deal->n_bits = n_bits;
  deal->dealt = true;
}

// Entries of a plan whose sequences all have `slices` slices.
static bool uniform_entries(int32_t batch, int32_t slices, uint32_t* entries) {
  if (batch > kMaxPlanBatch || slices > kMaxPlanSplits || (int64_t)batch * slices > kMaxPlanSlices) return false;
  for (int32_t b = 0; b < batch; ++b) {
    for (int32_t s = 0; s < slices; ++s) entries[b * slices + s] = pack_slice((uint32_t)b, (uint32_t)s, (uint32_t)slices);
  }
  return true;
}

void deal_partition(const span_attn_desc_t* d, const TokenCounts& counts, Partition* p, uint32_t* table, RunTables* runs, Deal* deal) {
  deal->dealt = false;
  if (!p->even || (!p->exact && !uniform_entries(d->batch, p->num_splits, table))) return;
  deal_slices(d, counts, p->max_tokens, p->total_slices, 0, p->exact, table, deal);
  if (!deal->dealt) return;
  p->exact = true;
  if (p->runs) {
    RunSlice slices[kMaxRunSlices];
    for (int32_t i = 0; i < p->total_slices; ++i) {
      slices[deal->at[i]] = runs->slices[i];
      slices[deal->at[i]].reserved = i;
    }
    std::copy(slices, slices + p->total_slices, runs->slices);
  }
}

void deal_matrix(const span_attn_desc_t* d, const TokenCounts& counts, const Partition& p, MatrixPlan* m, uint32_t* table, Deal* deal) {
  deal->dealt = false;
  const bool one_block = m->tokens <= 16 * m->groups;  // (several: see plan_matrix)
  if (!m->even || !one_block || (!m->table && !uniform_entries(d->batch, m->num_splits, table))) return;
  const int32_t hand_over = (int64_t)m->total_slices * d->heads < 2 * kTurn ? kHandOverRows : 0;
  deal_slices(d, counts, p.max_tokens, m->total_slices, hand_over, m->table, table, deal);
  m->table = m->table || deal->dealt;
}

size_t workspace_counter_bytes(const span_attn_desc_t* d) {
  const size_t n = (size_t)d->batch * d->heads * sizeof(int32_t);
  return (n + 255) & ~(size_t)255;
}

int32_t counter_stride(const span_attn_desc_t* d) {
  return (int32_t)(workspace_counter_bytes(d) / sizeof(int32_t) / ((size_t)d->batch * d->heads));
}

size_t workspace_ml_bytes(const span_attn_desc_t* d, int64_t states) {
  const size_t n = (size_t)states * d->heads * 2 * sizeof(float);
  return (n + 255) & ~(size_t)255;
}

size_t workspace_bytes_for(const span_attn_desc_t* d, int64_t states) {
  if (states == 0) return 0;
  return workspace_counter_bytes(d) + workspace_ml_bytes(d, states) + (size_t)states * d->heads * d->head_dim * sizeof(float);
}

size_t workspace_least_bytes(const span_attn_desc_t* d, const Partition& p) { return workspace_bytes_for(d, least_states(p)); }

Partition plan_for_workspace(const span_attn_desc_t* d, const TokenCounts& counts, uint32_t* table, RunTables* runs, bool spans) {
  auto fits = [&](const Partition& p) { return workspace_least_bytes(d, p) <= d->workspace_bytes; };
  Partition p = plan_partition(d, counts, table, runs, spans);
  if (fits(p)) return p;
  for (const ShortRules rules : {ShortRules::kApplied, ShortRules::kNone, ShortRules::kWhole}) {
    for (const bool finer : {true, false}) {
      if (finer && (!spans || rules == ShortRules::kApplied)) continue;  // (is the other one, or the first plan)
      p = plan_partition(d, counts, table, runs, finer, rules);
      if (fits(p)) return p;
    }
  }
  return p;  // (refused: the last is the least demanding)
}

size_t workspace_bytes(const span_attn_desc_t* d, const TokenCounts& counts, const Partition& p) {
  int64_t states = least_states(p);
  const int64_t most = most_states(d, p);
  if (most > states) {  // (a few-query call whose pool may be larger: as much as its plan uses, or the cut that holds shorter calls of the shape)
    MatrixPlan m;
    uint32_t table[kMaxPlanSlices];
    for (const bool two_per_cu : {false, true})
      if (plan_matrix(d, counts, p, most, &m, table, two_per_cu)) states = std::max(states, m.states);
  }
  return workspace_bytes_for(d, states);
}

int64_t states_that_fit(const span_attn_desc_t* d, const Partition& p) {
  const size_t counters = workspace_counter_bytes(d), per_state = (size_t)d->heads * (2 + d->head_dim) * sizeof(float);
  const size_t room = d->workspace_bytes > counters ? d->workspace_bytes - counters : 0;
  int64_t fit = std::min<int64_t>(most_states(d, p), (int64_t)(room / per_state));
  if (fit > 0 && workspace_bytes_for(d, fit) > d->workspace_bytes) --fit;  // (the (m, l) pairs' part is rounded up)
  return std::max(least_states(p), fit);
}

}  // namespace spanattn

extern "C" int span_plan_query(const span_attn_desc_t* desc, span_plan_info_t* info) {
  if (!info) return SPAN_ERR_NULL;
  const int rc = spanattn::check_desc(desc);
  if (rc != SPAN_OK) return rc;
  spanattn::RunTables runs;
  const spanattn::TokenCounts counts(desc);
  const spanattn::Partition p = spanattn::plan_partition(desc, counts, nullptr, &runs, true);
  info->runs_in_arguments = p.runs ? 1 : 0;
  info->queries_per_pass = p.queries_per_pass;
  info->exact = p.even ? 1 : 0;
  info->slice_tokens = p.slice_tokens;
  info->max_splits = p.num_splits;
  info->slice_limit = spanattn::kMaxSlice;
  info->workgroups = (int64_t)p.total_slices * desc->heads;
  info->workspace_bytes = (int64_t)spanattn::workspace_bytes(desc, counts, p);
  return SPAN_OK;
}

extern "C" int span_launch_query(const span_attn_desc_t* desc, span_launch_info_t* info) {
  if (!info) return SPAN_ERR_NULL;
  const int rc = spanattn::check_desc(desc);
  if (rc != SPAN_OK) return rc;
  const spanattn::TokenCounts counts(desc);
  const spanattn::Partition p = desc->workspace ? spanattn::plan_for_workspace(desc, counts, nullptr, nullptr, true)
                                                : spanattn::plan_partition(desc, counts, nullptr, nullptr, true);
  const int64_t states = !desc->workspace ? spanattn::most_states(desc, p) : spanattn::states_that_fit(desc, p);
  const int32_t n = spanattn::query_tokens(desc);
  spanattn::MatrixPlan m;
  uint32_t table[spanattn::kMaxPlanSlices];
  if (spanattn::plan_matrix(desc, counts, p, states, &m, table)) {
    info->matrix_cores = 1;
    info->launches = (n + m.tokens - 1) / m.tokens;
    info->tokens = m.tokens;
    info->max_splits = m.num_splits;
    info->slice_tokens = m.slice_tokens;
    info->query_blocks = (m.tokens + 16 * m.groups - 1) / (16 * m.groups);
    info->workgroups = (int64_t)m.total_slices * desc->heads * info->query_blocks;
    info->partial_states = m.states / m.tokens * n * desc->heads;
  } else {
    info->matrix_cores = 0;
    info->launches = 1;
    info->tokens = n;
    info->max_splits = p.num_splits;
    info->slice_tokens = p.slice_tokens;
    info->query_blocks = 1;
    info->workgroups = (int64_t)p.total_slices * desc->heads;
    info->partial_states = p.num_splits > 1 ? info->workgroups * n : 0;
  }
  return SPAN_OK;
}

extern "C" size_t span_workspace_bytes(const span_attn_desc_t* desc) {
  if (spanattn::check_desc(desc) != SPAN_OK) return 0;
  const spanattn::TokenCounts counts(desc);
  return spanattn::workspace_bytes(desc, counts, spanattn::plan_partition(desc, counts, nullptr, nullptr, true));
}

// ---- blocked encoding (block index + in-block bit mask) <-> interval lists ---------------------------
extern "C" int span_blocks_to_intervals(int32_t batch, int32_t block_size, const int32_t* block_offsets,
                                        const int32_t* block_idx, const uint32_t* block_masks, int32_t capacity,
                                        int32_t* span_offsets, int32_t* span_starts, int32_t* span_ends,
                                        int32_t* needed) {
  if (!block_offsets || !span_offsets || !needed) return SPAN_ERR_NULL;
  if (batch < 0 || capacity < 0 || block_size <= 0 || block_size % 32 != 0) return SPAN_ERR_SHAPE;
  if (capacity > 0 && (!span_starts || !span_ends)) return SPAN_ERR_NULL;
  const int32_t words = block_size / 32;
  int64_t count = 0;  // intervals produced so far (may run past capacity; writes stop at capacity)
  span_offsets[0] = 0;
  *needed = 0;
  for (int32_t b = 0; b < batch; ++b) {
    const int32_t first = block_offsets[b], last = block_offsets[b + 1];
    if ((b == 0 && first != 0) || last < first) return SPAN_BAD_OFFSETS;
    if (last > first && (!block_idx || !block_masks)) return SPAN_ERR_NULL;
    int64_t run_start = -1, run_end = -1;  // open run of attended positions, [run_start, run_end)
    auto close_run = [&]() {
      if (run_start < 0) return;
      if (count < capacity) {
        span_starts[count] = (int32_t)run_start;
        span_ends[count] = (int32_t)run_end;
      }
      ++count;
      run_start = -1;
    };
    for (int32_t j = first; j < last; ++j) {
      if (block_idx[j] < 0) return SPAN_BAD_RANGE;
      if (j > first && block_idx[j] <= block_idx[j - 1]) return SPAN_BAD_UNSORTED;
      const int64_t base = (int64_t)block_idx[j] * block_size;
      if (base + block_size > INT32_MAX) return SPAN_BAD_RANGE;
      for (int32_t w = 0; w < words; ++w) {
        const uint32_t m = block_masks[(size_t)j * words + w];
        for (int32_t t = 0; t < 32; ++t) {
          if (!((m >> t) & 1u)) continue;
          const int64_t pos = base + w * 32 + t;
          if (run_start >= 0 && pos == run_end) {
            ++run_end;
          } else {
            close_run();
            run_start = pos;
            run_end = pos + 1;
          }
        }
      }
    }
    close_run();
    if (count > INT32_MAX) return SPAN_ERR_SHAPE;
    span_offsets[b + 1] = (int32_t)count;
  }
  *needed = (int32_t)count;
  return count > capacity ? SPAN_ERR_CAPACITY : SPAN_OK;
}

extern "C" int span_intervals_to_blocks(int32_t batch, int32_t block_size, const int32_t* span_offsets,
                                        const int32_t* span_starts, const int32_t* span_ends, int32_t capacity,
                                        int32_t* block_offsets, int32_t* block_idx, uint32_t* block_masks,
                                        int32_t* needed) {
  if (!span_offsets || !block_offsets || !needed) return SPAN_ERR_NULL;
  if (batch < 0 || capacity < 0 || block_size <= 0 || block_size % 32 != 0) return SPAN_ERR_SHAPE;
  if (capacity > 0 && (!block_idx || !block_masks)) return SPAN_ERR_NULL;
  const int32_t words = block_size / 32;
  int64_t count = 0;
  block_offsets[0] = 0;
  *needed = 0;
  for (int32_t b = 0; b < batch; ++b) {
    const int32_t first = span_offsets[b], last = span_offsets[b + 1];
    if ((b == 0 && first != 0) || last < first) return SPAN_BAD_OFFSETS;
    if (last > first && (!span_starts || !span_ends)) return SPAN_ERR_NULL;
    std::map<int32_t, std::vector<uint32_t>> touched;  // block index -> mask words, ascending
    for (int32_t i = first; i < last; ++i) {
      const int32_t s = span_starts[i], e = span_ends[i];
      if (s < 0) return SPAN_BAD_RANGE;
      if (s >= e) return SPAN_BAD_EMPTY_INTERVAL;
      for (int64_t blk = s / block_size; blk * block_size < e; ++blk) {
        std::vector<uint32_t>& m = touched[(int32_t)blk];
        if (m.empty()) m.assign(words, 0u);
        const int64_t lo = std::max<int64_t>(s, blk * block_size) - blk * block_size;
        const int64_t hi = std::min<int64_t>(e, (blk + 1) * block_size) - blk * block_size;
        for (int64_t t = lo; t < hi; ++t) m[t / 32] |= 1u << (t % 32);
      }
    }
    for (const auto& kv : touched) {
      if (count < capacity) {
        block_idx[count] = kv.first;
        std::copy(kv.second.begin(), kv.second.end(), block_masks + (size_t)count * words);
      }
      ++count;
    }
    if (count > INT32_MAX) return SPAN_ERR_SHAPE;
    block_offsets[b + 1] = (int32_t)count;
  }
  *needed = (int32_t)count;
  return count > capacity ? SPAN_ERR_CAPACITY : SPAN_OK;
}

// ---- span builder: anchors + references -> sorted disjoint intervals ---------------------------------
extern "C" int span_build(int32_t num_anchors, const int32_t* anchor_starts, const int32_t* anchor_ends,
                          int32_t num_refs, const int32_t* ref_first, const int32_t* ref_last, int32_t prefix_end,
                          int32_t prev_line_start, int32_t cur_line_start, int32_t ctx_len, int32_t capacity,
                          int32_t* out_starts, int32_t* out_ends, int32_t* needed) {
  if (!needed) return SPAN_ERR_NULL;
  if (num_anchors < 0 || num_refs < 0 || capacity < 0 || ctx_len < 0) return SPAN_ERR_SHAPE;
  if (num_anchors > 0 && (!anchor_starts || !anchor_ends)) return SPAN_ERR_NULL;
  if (num_refs > 0 && (!ref_first || !ref_last)) return SPAN_ERR_NULL;
  if (capacity > 0 && (!out_starts || !out_ends)) return SPAN_ERR_NULL;
  *needed = 0;
  auto inside = [&](int32_t p) { return p >= 0 && p <= ctx_len; };
  if (!inside(prefix_end) || !inside(prev_line_start) || !inside(cur_line_start) || prev_line_start > cur_line_start)
    return SPAN_BAD_RANGE;
  std::vector<std::pair<int32_t, int32_t>> ranges;
  ranges.reserve((size_t)num_refs + 3);
  auto add = [&](int32_t s, int32_t e) {
    if (s < e) ranges.emplace_back(s, e);
  };
  add(0, prefix_end);
  add(cur_line_start, ctx_len);
  for (int32_t r = 0; r < num_refs; ++r) {
    if (ref_first[r] == -1) {  // the previous line
      add(prev_line_start, cur_line_start);
      continue;
    }
    if (ref_first[r] < 0 || ref_last[r] >= num_anchors || ref_first[r] > ref_last[r]) return SPAN_BAD_RANGE;
    for (int32_t k = ref_first[r]; k <= ref_last[r]; ++k) {
      if (anchor_starts[k] < 0 || anchor_ends[k] > ctx_len || anchor_starts[k] > anchor_ends[k]) return SPAN_BAD_RANGE;
      add(anchor_starts[k], anchor_ends[k]);
    }
  }
  std::sort(ranges.begin(), ranges.end());
  int64_t count = 0;
  int32_t cur_s = 0, cur_e = -1;  // open interval; cur_e < 0: none
  auto flush = [&]() {
    if (cur_e < 0) return;
    if (count < capacity) {
      out_starts[count] = cur_s;
      out_ends[count] = cur_e;
    }
    ++count;
  };
  for (const auto& r : ranges) {
    if (cur_e >= 0 && r.first <= cur_e) {  // overlapping or touching: extend
      if (r.second > cur_e) cur_e = r.second;
    } else {
      flush();
      cur_s = r.first;
      cur_e = r.second;
    }
  }
  flush();
  *needed = (int32_t)count;
  return count > capacity ? SPAN_ERR_CAPACITY : SPAN_OK;
}

extern "C" const char* span_strerror(int code) {
  switch (code) {
    case SPAN_OK: return "ok";
    case SPAN_ERR_NULL: return "a required pointer is NULL";
    case SPAN_ERR_SHAPE: return "unsupported shape (dims must be positive, head_dim 64 or 128, max_len <= 2^22)";
    case SPAN_ERR_DTYPE: return "unsupported dtype";
    case SPAN_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case SPAN_ERR_HIP: return "a HIP call failed (see span_last_hip_error)";
    case SPAN_ERR_CAPACITY: return "output array too small (needed size reported)";
    case SPAN_ERR_SCRATCH_LIMIT: return "the call needs more scratch than the library's static buffer holds";
    case SPAN_BAD_OFFSETS: return "span_offsets must start at 0, not decrease, and stay within num_intervals";
    case SPAN_BAD_RANGE: return "interval outside [0, ctx_len]";
    case SPAN_BAD_EMPTY_INTERVAL: return "interval with start >= end";
    case SPAN_BAD_OVERLAP: return "interval overlaps the previous one";
    case SPAN_BAD_UNSORTED: return "interval starts before the previous one";
    case SPAN_BAD_EMPTY_SPAN: return "sequence with no interval";
    default: return "unknown code";
  }
}
