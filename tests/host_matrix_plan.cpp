// Randomised check of the few-query launch plan (plan_matrix): every position has an owner, the slots of sequences with
// several slices fit the workspace the call's partition sizes, and the grid and the packed ticket fields stay in range.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "span_internal.h"

#define REQUIRE(c)                                                        \
  do {                                                                    \
    if (!(c)) {                                                           \
      std::printf("%s:%d: %s (case %d)\n", __FILE__, __LINE__, #c, it);   \
      std::abort();                                                       \
    }                                                                     \
  } while (0)

static std::mt19937 rng(20240409);
static int rnd(int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); }

// A workspace of any size from the least that is accepted: the plan's states fit what the launch lays out in it, the size
// asked for gives the plan of an unlimited one, and the least does not depend on the number of tokens from three on.
static void workspaces_of_all_sizes() {
  using namespace spanattn;
  std::vector<uint32_t> base_table(kMaxPlanSlices), table(kMaxPlanSlices);
  int more = 0, fewer_slices = 0;
  for (int it = 0; it < 20000; ++it) {
    span_attn_desc_t d = {};
    d.batch = rnd(1, rnd(0, 2) ? 12 : 60);
    const int heads[] = {1, 3, 8, 16, 32};
    d.heads = heads[rnd(0, 4)];
    d.head_dim = rnd(0, 1) ? 128 : 64;
    d.max_len = rnd(1, 20000);
    d.dtype = rnd(0, 2);
    d.num_intervals = 10;
    d.num_splits = rnd(0, 9) ? 0 : rnd(1, 300);
    d.q_len = rnd(2, 64);
    std::vector<int64_t> tok(d.batch);
    for (auto& t : tok) t = rnd(0, rnd(0, 1) ? d.max_len : (d.max_len + 9) / 10);
    d.tokens_per_seq = rnd(0, 3) ? tok.data() : nullptr;
    const Partition p = plan_partition(&d, base_table.data());
    const size_t least = workspace_least_bytes(&d, p), asked = workspace_bytes(&d, p);
    REQUIRE(least <= asked && (least == 0) == (asked == 0) && (least == 0) == (p.num_splits == 1));
    MatrixPlan full, m;
    if (!plan_matrix(&d, p, most_states(&d, p), &full, table.data())) {
      REQUIRE(least == asked);
      continue;
    }
    if (d.q_len >= 3) {
      span_attn_desc_t other = d;
      other.q_len = rnd(3, 64);
      REQUIRE(workspace_least_bytes(&other, plan_partition(&other, base_table.data())) == least);
    }
    if (least == 0) {
      REQUIRE(full.states == 0 && full.num_splits == 1);
      continue;
    }
    d.workspace_bytes = rnd(0, 3) ? least + (size_t)(rng() % (uint32_t)(asked - least + 1000)) : asked;
    const int64_t states = states_that_fit(&d, p);
    REQUIRE(states >= least_states(p) && workspace_bytes_for(&d, states) <= d.workspace_bytes);
    REQUIRE(plan_matrix(&d, p, states, &m, table.data()) && m.states <= states);
    if (m.num_splits == 1) REQUIRE(m.states == 0);
    if (d.workspace_bytes >= asked) REQUIRE(m.total_slices == full.total_slices && m.num_splits == full.num_splits && m.slice_tokens == full.slice_tokens);
    more += asked > least;
    fewer_slices += m.total_slices < full.total_slices;
  }
  const int it = -2;
  REQUIRE(more > 500 && fewer_slices > 300);
}

int main() {
  using namespace spanattn;
  workspaces_of_all_sizes();
  std::vector<uint32_t> base_table(kMaxPlanSlices);
  int tables = 0, sliced = 0, shared_rows = 0, forced = 0;
  for (int it = 0; it < 40000; ++it) {
    span_attn_desc_t d = {};
    d.batch = rnd(0, 20) ? rnd(1, rnd(0, 2) ? 12 : 80) : rnd(900, 1200);
    const int heads[] = {1, 3, 5, 8, 12, 16, 32, 4000};
    d.heads = heads[rnd(0, 7)];
    d.head_dim = rnd(0, 1) ? 128 : 64;
    d.max_len = rnd(0, 8) ? rnd(1, 20000) : (1 << 22);
    d.dtype = rnd(0, 2);
    d.num_intervals = 10;
    d.max_tokens = rnd(0, 2) ? 0 : rnd(1, d.max_len);
    d.num_splits = rnd(0, 4) ? 0 : rnd(1, 3000);
    d.q_len = rnd(0, 64);
    std::vector<int64_t> tok(d.batch);
    for (auto& t : tok) t = rnd(0, 9) == 0 ? rnd(-5, 0) : rnd(0, rnd(0, 1) ? d.max_len : (d.max_len + 9) / 10);
    d.tokens_per_seq = rnd(0, 3) ? tok.data() : nullptr;
    const Partition p = plan_partition(&d, base_table.data());
    std::vector<uint32_t> table(kMaxPlanSlices);  // its own heap block: a write past the end is caught
    MatrixPlan m;
    const bool used = plan_matrix(&d, p, &m, table.data());
    const bool few_columns = d.dtype != SPAN_F32 && (int64_t)d.batch * d.heads * d.head_dim <= 32768;
    REQUIRE(used == (d.q_len >= 3 || (d.q_len == 2 && few_columns)));
    if (!used) continue;
    const int blocks = (m.tokens + 16 * m.groups - 1) / (16 * m.groups);
    REQUIRE(m.groups == 1 || m.groups == 2 || m.groups == 4);
    REQUIRE(m.tokens >= 1 && m.tokens <= d.q_len && blocks >= 1 && blocks <= 4);
    REQUIRE((int64_t)d.batch * blocks <= 65535 && m.num_splits >= 1 && m.num_splits <= 65535);
    REQUIRE(blocks == 1 || m.num_splits <= 255);
    const int64_t states = p.num_splits > 1 ? (int64_t)p.total_slices * p.queries_per_pass : 0;
    if (m.tokens < d.q_len) {
      ++forced;
      REQUIRE(d.num_splits > 0);
    } else if (d.num_splits == 0) {
      shared_rows += blocks > 1;
    }
    if (m.table) {
      ++tables;
      REQUIRE(m.even && m.total_slices <= kMaxPlanSlices && d.batch <= kMaxPlanBatch);
      std::vector<int> seen(d.batch, 0);
      int slots = 0;
      bool singles = false;
      for (int y = 0; y < m.total_slices;) {
        const int b = table[y] & 1023, n = table[y] >> 21;
        REQUIRE(b < d.batch && !seen[b] && n >= 1 && n <= m.num_splits);
        seen[b] = 1;
        if (n > 1) REQUIRE(!singles);  // sequences with several slices come first: entry index = slot
        singles = singles || n == 1;
        const int64_t want = std::min<int64_t>(std::max<int64_t>(tok[b], 0), p.max_tokens);
        REQUIRE((want + n - 1) / n <= m.slice_tokens);
        for (int s = 0; s < n; ++s, ++y) REQUIRE(y < m.total_slices && table[y] == pack_slice(b, s, n));
        if (n > 1) slots = y;
      }
      for (int s : seen) REQUIRE(s);
      REQUIRE((int64_t)slots * m.tokens <= states);
    } else {
      REQUIRE(m.total_slices == m.num_splits * d.batch);
      REQUIRE(m.even || (int64_t)m.num_splits * m.slice_tokens >= p.max_tokens);
      if (m.num_splits > 1) REQUIRE((int64_t)m.total_slices * m.tokens <= states);
    }
    sliced += m.num_splits > 1;
  }
  const int it = -1;
  REQUIRE(tables > 500 && sliced > 2000 && shared_rows > 500 && forced > 500);  // every kind was exercised
  std::puts("host_matrix_plan: ok");
  return 0;
}
