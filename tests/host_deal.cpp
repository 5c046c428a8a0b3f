// Randomised check of the order in which slices go out (deal_partition, deal_matrix): a dealt table names every slice of the plan
// once, with its own slot, and no column of CUs gets more rows than it would in plan order.
#include <algorithm>
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

using namespace spanattn;
static std::mt19937 rng(20240409);
static int rnd(int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); }

struct Named {
  uint32_t b, split, nsl, slot;
};
static Named named(uint32_t e, const Deal& d) {
  const uint32_t in_n = (1u << d.n_bits) - 1;
  return {e & ((1u << d.b_bits) - 1), e >> d.b_bits & in_n, e >> (d.b_bits + d.n_bits) & in_n, e >> (32 - kSlotBits)};
}

static int64_t most_rows(const std::vector<int64_t>& rows, int heads) {
  const int columns = (256 + heads / 2) / heads;
  std::vector<int64_t> load(columns, 0);
  for (size_t y = 0; y < rows.size(); ++y) load[y % columns] += rows[y];
  return *std::max_element(load.begin(), load.end());
}

int main() {
  int dealt_tables = 0, new_tables = 0, dealt_runs = 0, matrix = 0;
  for (int it = 0; it < 30000; ++it) {
    span_attn_desc_t d = {};
    d.batch = rnd(0, 20) ? rnd(1, 70) : rnd(300, 800);
    const int heads[] = {1, 3, 5, 8, 12, 16, 32, 128, 300};
    d.heads = heads[rnd(0, 8)];
    d.head_dim = rnd(0, 1) ? 128 : 64;
    d.max_len = rnd(0, 8) ? rnd(1, 6000) : (1 << 20);
    d.dtype = rnd(0, 2);
    d.q_len = rnd(0, 1) ? 1 : rnd(2, 64);
    d.max_tokens = rnd(0, 2) ? 0 : rnd(1, d.max_len);
    const int low = rnd(0, d.max_len);
    std::vector<int64_t> tok(d.batch);
    std::vector<int32_t> off(d.batch + 1, 0), st(d.batch, 0), en(d.batch);
    for (int b = 0; b < d.batch; ++b) {
      tok[b] = rnd(0, 30) ? rnd(low, d.max_len) : rnd(-2, 1);
      off[b + 1] = b + 1;
      en[b] = (int32_t)std::max<int64_t>(tok[b], 0);
    }
    d.tokens_per_seq = tok.data();
    if (rnd(0, 1)) {
      d.num_intervals = d.batch;
      d.host_span_offsets = off.data();
      d.host_span_starts = st.data();
      d.host_span_ends = en.data();
    }
    std::vector<uint32_t> table(kMaxPlanSlices);  // its own heap block: a write past the end is caught
    std::vector<RunTables> runs(1);
    Partition p = plan_partition(&d, table.data(), runs.data());
    Deal deal;
    MatrixPlan m;
    int32_t total;
    std::vector<uint32_t> plan;
    std::vector<RunSlice> plan_runs(runs[0].slices, runs[0].slices + kMaxRunSlices);
    bool had_table;
    auto in_plan_order = [&](bool has, int32_t splits) {
      had_table = has;
      plan.clear();
      if (has) plan.assign(table.begin(), table.begin() + total);
      else for (int i = 0; i < total && p.even; ++i) plan.push_back(pack_slice(i / splits, i % splits, splits));
    };
    if (plan_matrix(&d, p, most_states(&d, p), &m, table.data())) {
      total = m.total_slices;
      if (total > 100000) continue;
      in_plan_order(m.table, m.num_splits);
      deal_matrix(&d, p, &m, table.data(), &deal);
      REQUIRE(m.table == (had_table || deal.dealt));
      matrix += deal.dealt;
    } else {
      total = p.total_slices;
      if (total > 100000) continue;
      in_plan_order(p.exact, p.num_splits);
      deal_partition(&d, &p, table.data(), runs.data(), &deal);
      REQUIRE(p.exact == (had_table || deal.dealt));
    }
    if (!deal.dealt) {
      if (had_table) REQUIRE(std::equal(plan.begin(), plan.end(), table.begin()));
      continue;
    }
    REQUIRE(p.even && total <= kMaxPlanSlices && d.heads <= 170);
    ++(had_table ? dealt_tables : new_tables);
    std::vector<int> seen(total, 0);
    std::vector<int64_t> rows(total), plan_rows(total);
    for (int y = 0; y < total; ++y) {
      const Named n = named(table[y], deal);
      REQUIRE(n.slot < (uint32_t)total && !seen[n.slot] && deal.at[n.slot] == y);
      seen[n.slot] = 1;
      REQUIRE(plan[n.slot] == pack_slice(n.b, n.split, n.nsl) && (int)n.b < d.batch && n.split < n.nsl);
      const int64_t tokens = std::min<int64_t>(std::max<int64_t>(tok[n.b], 0), p.max_tokens), T = (tokens + n.nsl - 1) / n.nsl;
      rows[y] = plan_rows[n.slot] = std::min<int64_t>(std::max<int64_t>(tokens - (int64_t)n.split * T, 0), T);
      if (p.runs && d.q_len <= 1) {
        const RunSlice& r = runs[0].slices[y];
        REQUIRE(r.reserved == (int32_t)n.slot && r.entry == plan[n.slot] && r.rows == rows[y] && r.runs_of == plan_runs[n.slot].runs_of);
      }
    }
    dealt_runs += p.runs;
    REQUIRE(most_rows(rows, d.heads) < most_rows(plan_rows, d.heads));
  }
  const int it = -1;
  REQUIRE(dealt_tables > 500 && new_tables > 500 && dealt_runs > 100 && matrix > 500);  // every kind was exercised
  std::puts("host_deal: ok");
  return 0;
}
