// The order in which whole sequences of unequal length go out: every sequence once, and no CU with many more rows than the others.
// Workgroups go to the CUs in turns of 256, heads fastest.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "span_internal.h"

#define REQUIRE(c)                                                                 \
  do {                                                                             \
    if (!(c)) {                                                                    \
      std::printf("%s:%d: %s (%s)\n", __FILE__, __LINE__, #c, name);               \
      std::abort();                                                                \
    }                                                                              \
  } while (0)

using namespace spanattn;

struct Order {
  MatrixPlan plan;
  Deal deal;
  std::vector<int32_t> sequence, split, slices;  // of the table's entries
  double fullest;                                // rows of the fullest column of CUs over the mean, in the first query block
};

static Order order(const char* name, int dtype, int batch, int heads, int head_dim, int least, int most, int tokens) {
  std::mt19937 rng(batch * 1000 + heads);
  span_attn_desc_t d = {};
  d.batch = batch;
  d.heads = heads;
  d.head_dim = head_dim;
  d.dtype = dtype;
  d.max_len = most;
  d.q_len = tokens;
  std::vector<int64_t> counts(batch);
  for (auto& n : counts) n = least + (int)(rng() % (unsigned)(most - least + 1));
  d.tokens_per_seq = counts.data();
  std::vector<uint32_t> table(kMaxPlanSlices);
  const Partition p = plan_partition(&d, table.data());
  Order o;
  REQUIRE(plan_matrix(&d, p, most_states(&d, p), &o.plan, table.data()));
  deal_matrix(&d, p, &o.plan, table.data(), &o.deal);
  const int columns = std::max(1, 256 / heads);
  std::vector<int64_t> load(columns, 0);
  int64_t sum = 0;
  std::vector<int> seen((size_t)batch, 0);
  for (int y = 0; y < o.plan.total_slices; ++y) {
    const uint32_t e = o.plan.table ? table[y] : pack_slice(y / o.plan.num_splits, y % o.plan.num_splits, o.plan.num_splits);
    const uint32_t in_n = (1u << o.deal.n_bits) - 1;
    const int b = e & ((1u << o.deal.b_bits) - 1), split = e >> o.deal.b_bits & in_n, n = e >> (o.deal.b_bits + o.deal.n_bits) & in_n;
    REQUIRE(b < batch && split < n);
    ++seen[b];
    const int64_t T = (counts[b] + n - 1) / n, rows = std::min(std::max<int64_t>(counts[b] - split * T, 0), T);
    load[y % columns] += rows;
    sum += rows;
    o.sequence.push_back(b);
    o.split.push_back(split);
    o.slices.push_back(n);
  }
  for (int y = 0; y < o.plan.total_slices; ++y) REQUIRE(seen[o.sequence[y]] == o.slices[y]);
  o.fullest = (double)*std::max_element(load.begin(), load.end()) * columns / (double)sum;
  std::printf("%-28s slices %d groups %d table %d dealt %d fullest %.3f\n", name, o.plan.total_slices, o.plan.groups, o.plan.table, o.deal.dealt,
              o.fullest);
  return o;
}

// Launches of several query blocks, and those whose heads fill a turn alone.
static void several_blocks() {
  struct Shape {
    const char* name;
    int dtype, batch, heads, head_dim, least, most, tokens;
    double fullest;
  } shapes[] = {{"32x32 two blocks", SPAN_F32, 32, 32, 128, 500, 1000, 64, 1.05}, {"64x16 two blocks", SPAN_F32, 64, 16, 128, 300, 900, 48, 1.06},
                {"16x32 two blocks", SPAN_F32, 16, 32, 128, 400, 1000, 33, 1.08},  {"24x64 two blocks", SPAN_F32, 24, 64, 128, 100, 400, 40, 1.05}};
  for (const Shape& s : shapes) {
    const char* name = s.name;
    const Order o = order(s.name, s.dtype, s.batch, s.heads, s.head_dim, s.least, s.most, s.tokens);
    REQUIRE(o.plan.num_splits == 1 && o.plan.tokens > 16 * o.plan.groups);
    REQUIRE(o.plan.table && o.fullest < s.fullest);
  }
  for (int heads : {192, 256, 300}) {
    const char* name = "heads fill a turn";
    const Order o = order(name, SPAN_F16, 10, heads, 64, 200, 900, 20);
    REQUIRE(o.plan.table && !o.deal.dealt);
  }
  for (int tokens : {64, 8}) {  // lengths almost alike: no table
    const char* name = "level";
    REQUIRE(!order(name, SPAN_F32, 32, tokens == 64 ? 32 : 200, 128, 990, 1000, tokens).plan.table);
  }
}

// Less than two turns of workgroups with more than 16 tokens each.
static void less_than_two_turns() {
  struct Shape {
    const char* name;
    int dtype, batch, heads, head_dim, least, most, tokens;
    double fullest;
  } shapes[] = {{"60x8", SPAN_F16, 60, 8, 128, 53, 268, 59, 1.2}, {"58x8", SPAN_F32, 58, 8, 64, 32, 107, 44, 1.2},
                {"53x8", SPAN_F32, 53, 8, 128, 123, 206, 22, 1.4}, {"41x12", SPAN_F32, 41, 12, 64, 599, 999, 47, 1.2}};
  for (const Shape& s : shapes) {
    const char* name = s.name;
    const Order o = order(s.name, s.dtype, s.batch, s.heads, s.head_dim, s.least, s.most, s.tokens);
    REQUIRE(o.plan.total_slices * s.heads < 512 && o.plan.groups > 1);
    REQUIRE(o.deal.dealt && o.fullest < s.fullest);
  }
  // Short sequences, some of them cut: the cut ones' slices, which have a hand-over ahead of them, go out in the first turn, as in plan order.
  struct Cut {
    int dtype, batch, heads, head_dim, least, most, tokens;
  } cut[] = {{SPAN_F32, 35, 8, 128, 60, 160, 17}, {SPAN_BF16, 25, 15, 64, 108, 190, 2}, {SPAN_F32, 40, 8, 64, 80, 150, 3}};
  for (const Cut& s : cut) {
    const char* name = "short, some cut";
    const Order o = order(name, s.dtype, s.batch, s.heads, s.head_dim, s.least, s.most, s.tokens);
    REQUIRE(o.plan.num_splits == 2 && o.plan.total_slices * s.heads < 512);
    int last_cut = 0, first_whole = o.plan.total_slices;
    for (int y = 0; y < o.plan.total_slices; ++y) {
      if (o.slices[y] > 1) last_cut = y;
      else first_whole = std::min(first_whole, y);
    }
    REQUIRE(last_cut < (256 + s.heads / 2) / s.heads || last_cut < first_whole);
  }
}

// The calls that test_deal.py and test_order.py run on the GPU as dealt ones are.
static bool is_dealt(int dtype, int head_dim, int heads, int tokens, const std::vector<int64_t>& counts, int max_len) {
  span_attn_desc_t d = {};
  d.batch = (int32_t)counts.size();
  d.heads = heads;
  d.head_dim = head_dim;
  d.dtype = dtype;
  d.max_len = max_len;
  d.max_tokens = (int32_t)*std::max_element(counts.begin(), counts.end());
  d.q_len = tokens;
  d.tokens_per_seq = counts.data();
  std::vector<uint32_t> table(kMaxPlanSlices);
  Partition p = plan_partition(&d, table.data());
  MatrixPlan m;
  Deal deal;
  if (plan_matrix(&d, p, most_states(&d, p), &m, table.data())) deal_matrix(&d, p, &m, table.data(), &deal);
  else deal_partition(&d, &p, table.data(), nullptr, &deal);
  return deal.dealt;
}

static void tested_calls_are_dealt() {
  const char* name = "tested calls";
  std::vector<int64_t> many;
  for (int i = 0; i < 30; ++i) many.push_back(200 + 31 * (i % 7));
  const std::vector<std::vector<int64_t>> counts = {{500, 500, 720, 720, 500, 500, 720, 720}, {60, 130, 900, 880, 300, 20, 700, 700, 410, 1}, many};
  struct Call {
    int dtype, head_dim, tokens;
  } calls[] = {{SPAN_F16, 128, 1}, {SPAN_F32, 64, 1}, {SPAN_F32, 128, 2}, {SPAN_BF16, 128, 16}, {SPAN_F16, 64, 9}};
  int dealt = 0;
  for (const auto& n : counts) {
    for (const Call& c : calls) dealt += is_dealt(c.dtype, c.head_dim, 32, c.tokens, n, 1000);
  }
  std::printf("test_deal.py: %d of 15 calls are dealt\n", dealt);
  REQUIRE(dealt == 15);
  struct Other {
    int dtype, head_dim, heads, batch, tokens;
  } others[] = {{SPAN_F16, 128, 8, 60, 59}, {SPAN_F32, 64, 12, 41, 33}, {SPAN_F16, 128, 8, 60, 1}, {SPAN_F32, 64, 5, 90, 2}};
  for (const Other& o : others) {
    std::vector<int64_t> n;
    for (int i = 0; i < o.batch; ++i) n.push_back(60 + 37 * i % 131);
    REQUIRE(is_dealt(o.dtype, o.head_dim, o.heads, o.tokens, n, 200));
  }
}

// The host lists are walked when they are counted and, for the runs of a plan, once more; never for a deal.
static void lists_are_counted_once() {
  for (int tokens : {1, 2, 9, 40}) {
    const char* name = "counted once";
    const int batch = 24, each = 30;
    std::mt19937 rng(9);
    std::vector<int32_t> offsets(1, 0), starts, ends;
    for (int b = 0; b < batch; ++b) {
      for (int i = 0, at = 0; i < each + b; ++i, at += 40) {
        starts.push_back(at);
        ends.push_back(at + 1 + (int32_t)(rng() % 39u));
      }
      offsets.push_back((int32_t)starts.size());
    }
    span_attn_desc_t d = {};
    d.batch = batch;
    d.heads = 32;
    d.head_dim = 128;
    d.dtype = SPAN_F16;
    d.max_len = 4000;
    d.q_len = tokens;
    d.num_intervals = (int32_t)starts.size();
    d.host_span_offsets = offsets.data();
    d.host_span_starts = starts.data();
    d.host_span_ends = ends.data();
    std::vector<uint32_t> table[2];
    Deal deal[2];
    for (int gone : {0, 1}) {
      table[gone].assign(kMaxPlanSlices, 0);
      const TokenCounts counts(&d);
      REQUIRE(counts.from_lists);
      if (gone) std::fill(ends.begin(), ends.end(), 0);  // the lists as they are no longer attend anything
      Partition p = plan_partition(&d, counts, table[gone].data(), nullptr, true);
      MatrixPlan m;
      if (plan_matrix(&d, counts, p, most_states(&d, p), &m, table[gone].data())) deal_matrix(&d, counts, p, &m, table[gone].data(), &deal[gone]);
      else deal_partition(&d, counts, &p, table[gone].data(), nullptr, &deal[gone]);
    }
    REQUIRE(deal[0].dealt && deal[1].dealt && table[0] == table[1]);
  }
}

int main() {
  several_blocks();
  less_than_two_turns();
  lists_are_counted_once();
  tested_calls_are_dealt();
  std::puts("host_order: ok");
  return 0;
}
