// Span-restricted attention for several query tokens of a sequence (the few-query calls, three tokens and more) on
// gfx950's matrix cores: the one place of the decode path that is a dense contraction.
//
// A workgroup of 4 wavefronts takes one slice of a (batch, head) pair's span, as decode_kernel does, and up to 16 G
// query tokens; a call is one launch.  A wave takes its rows in tiles of 16 S rows.  Lane (qi, c4) = (lane % 16,
// lane / 16) plays row / column qi and contraction share c4 of the 16x16 MFMAs:
//   * scores S^T = K Q^T.  Lane (i, c) holds the 16-byte pieces 4 mm + c of K row i and of query row i; both use the
//     same assignment of the head dimension to (MFMA, lane group, element), so K pieces go from the load straight into
//     the operand.  Lane (qi, c4) ends up with the scores of query qi against rows 4 c4 + t of each 16 rows -
//   * outputs O^T = V^T P^T - which is the B operand of the second product (contraction over the tile's rows).  For
//     A = V^T lane (i, c) loads its D / 16 values of rows 4 c + t (whole rows per quarter wave, coalesced) and MFMA e
//     takes element e of each, so lane (qi, c4) accumulates NE = D / 16 x 4 output columns of query qi, and the
//     online-softmax rescaling factor is a per-lane scalar.
//   * 16-bit weights: the fp32 weight enters the second product as kTerms terms of the storage type, each rounding what
//     the ones before left (see weight_terms).  fp32 rows use the fp32 MFMA throughout.
// Bound by memory except for few pairs, where the start-up chain (1 us of list metadata, 2 us to the first rows) and the
// merge count.  Its rounding is that of the vector kernels or less (measured against 64 bits, relative 2-norm: fp32 1.6e-7
// for 1.8e-7, 16-bit rows of 64 1.45e-7 for 1.6e-7, 16-bit rows of 128 1.65e-7 for 1.75e-7).
// K and V are streamed through registers: the next tile's K loads go out as soon as the scores of this one are taken,
// its V loads as soon as the outputs are, so a wave always has loads in flight.  (us with the next tile's loads behind a branch
// and the K lines in halves, as it was -> now: 8 x 32 pairs x ~600 positions of 128, fp16, 2 tokens 22.9 -> 21.5; fp32, 8 tokens
// 37.9 -> 36.2; 64 x 32 x ~155, fp16, 16 tokens 38.0 -> 36.2; 16 x 32 x ~700, bf16, 32 tokens 47.9 -> 45.9; 16 x 16 x ~380 of 64,
// fp16, 9 tokens 13.6 -> 13.1.)
#include "span_device.h"
#include "span_matrix.h"

namespace spanattn {
namespace {

constexpr int kMWin = 512;  // rows of a wave whose positions are tabulated at a time
constexpr uint32_t kNoRow = 0xfffffc00u;  // an offset past every slab (and still so with a piece offset added)

struct MatrixArgs : LaunchArgs {
  int32_t tokens;        // query tokens of this launch: q_first .. q_first + tokens - 1
  int32_t slot_tokens;   // query tokens a slot of the workspace holds
  int32_t batch;
  int32_t query_blocks;  // workgroups per slice, each serving its own 16 G of the tokens
};
struct MatrixArgsPlain : MatrixArgs {
  static constexpr bool kHasTable = false;
};
struct MatrixArgsTable : MatrixArgs {
  static constexpr bool kHasTable = true;
  uint32_t table[kMaxPlanSlices];  // as in LaunchArgsTable
};

// Shape of one instance.
template <class Elt, int D, int G>
struct MatrixShape {
  static constexpr int kRowBytes = D * Elt::kBytes;
  static constexpr int NK = kRowBytes / 64;   // 16-byte pieces of a K row per lane
  static constexpr int NE = D / 16;           // values of a V row per lane
  static constexpr int VW = NE * Elt::kBytes / 4;  // dwords they fill: 2 (16-bit, D = 64), 4, or 8 (fp32, D = 128: two pieces)
  // Groups of 16 rows in a tile.  Two feed the 16x16x32 MFMA of the second product; one keeps 64 tokens inside the
  // register file, and 16 tokens of 16-bit rows of 128 at four waves per SIMD (batch 64 x ~155 positions, 16 tokens: 40.4
  // us against 44.2 with two and three waves).
  static constexpr int S = Elt::kBytes == 4 || G == 4 || (G == 1 && D == 128) ? 1 : 2;
  // Up to 32 tokens of 16-bit rows of 128 have both (kOneGroup): with two groups a tile is 16 KB, and the workgroups of a single
  // round, all asking at once, get their first one late and unevenly; with one the matrix cores do half as much per
  // instruction.  us, two -> one: 512 workgroups, 16 x ~700 positions, bf16, 32 tokens 40.6 -> 39.0, appended 45.6 -> 44.1; in several rounds
  // 64 x 32 pairs x ~220, bf16, 24 tokens 91.9 -> 97.0, 64 x 32 x ~400 fp16, 20 tokens 113.5 -> 119.8.
  static constexpr bool kHasBoth = S == 2 && D == 128;
  // Waves per SIMD.  64 tokens of 16-bit rows of 128 spill 31 (fp16) and 38 (bf16) registers, all of them in the pass for V rows that are
  // not finite (stream_checked).
  static constexpr int kWaves = kMatrixWorkgroupsPerCu(Elt::kBytes, D, G);
};

// Terms of a weight in the storage type.  Three hold all 24 bits of the fp32 weight; bf16 rows need them.  Of fp16 rows the
// calls whose weights met the rows whole before they came to the matrix cores take three (head_dim 64, and two tokens), the
// others the two that their sixteen-token pass had.  The third costs, us with two -> three: 16 x 16 pairs x ~380 positions of
// 64, 9 tokens 14.5 -> 14.8; 16 x 32 x ~560 of 64, 20 tokens 25.8 -> 26.9, 60 tokens 39.8 -> 41.7; 8 x 32 x ~560 of 128, 2
// tokens 22.4 -> 22.4.  For more tokens of 128 it would: 64 x 32 x ~155, 16 tokens 39.9 -> 40.7; 32 x 32 x ~560, 64 tokens
// 115 -> 124.  Weights kept whole on the fp32 MFMA: 16.9, 35.9, 59.2, 25.7, 44.5 and 213.
template <class Elt, int D>
constexpr int weight_terms(bool two_tokens) {
  return std::is_same<Elt, F16>::value && D == 128 && !two_tokens ? 2 : 3;
}

// The value is computed here and not later: the compiler would otherwise sink the additions below the next tile's loads,
// and keep all their operands in registers across them.
__device__ __forceinline__ void pin(f32x4& v) { asm volatile("" : "+v"(v)); }

// `from` of the lane eight further (within its 16) in the lanes of `kBanks` (0x3: lanes 0 - 7 of each 16, 0xc: 8 - 15), `keep` in
// the others.
template <int kBanks>
__device__ __forceinline__ uint32_t swap_half(uint32_t keep, uint32_t from) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)keep, (int)from, 0x128, 0xf, kBanks, false);  // row_ror:8
}

// 16 bytes to / from memory that all XCDs share (sc1: written through, never served from a stale L2 line).
constexpr int kThrough = 16;
__device__ __forceinline__ void publish4(__amdgpu_buffer_rsrc_t slot, uint32_t byte_off, f32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), slot, byte_off, 0, kThrough);
}
__device__ __forceinline__ f32x4 observe4(__amdgpu_buffer_rsrc_t slot, uint32_t byte_off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(slot, byte_off, 0, kThrough));
}

// kShared: several workgroups (query blocks) read the same rows, so the rows are loaded with the default cache policy and
// the later readers find them in the L2; otherwise every row is used once and streams past it.  Inputs that no cache
// holds from call to call: 32 pairs x ~5500 positions, 20 tokens 29.6 -> 25.2 us; 96 pairs x ~900, 60 tokens 30.1 -> 26.5; 32 pairs
// x 1500 fp32, 30 tokens 30.8 -> 28.0; without query blocks it loses (64 x ~155, 16 tokens 39.8 -> 43.7).
// kInStep: ... and wait for all of their loads ahead of a tile's outputs, which keeps the two workgroups of a slice at the same rows, see
// keep_in_step.
enum class Rows { kAlone, kShared, kInStep };
template <class Elt, int D, int G, bool kOneGroup, class Args, Rows kSharing, int kTerms>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(MatrixShape<Elt, D, G>::kWaves, MatrixShape<Elt, D, G>::kWaves))) void matrix_kernel(const Args a) {
  using Shape = MatrixShape<Elt, D, G>;
  constexpr bool kShared = kSharing != Rows::kAlone;
  constexpr int kRowPolicy = kShared ? 0 : kRowLoadPolicy;
  auto load_piece = [](__amdgpu_buffer_rsrc_t slab, uint32_t off) { return __builtin_amdgcn_raw_buffer_load_b128(slab, off, 0, kRowPolicy); };
  constexpr int NK = Shape::NK, NE = Shape::NE, VW = Shape::VW, S = kOneGroup ? 1 : Shape::S;
  constexpr int TR = 16 * S;                 // rows of a tile
  constexpr uint32_t ROWB = Shape::kRowBytes;
  constexpr int NQ = 16 * G;
  constexpr int kPieces = ROWB / 16;
  constexpr int kQRow = ROWB + 16;           // LDS rows of q, padded: operand reads spread over the banks
  constexpr int kAccRow = D + 4;
  constexpr int kAtOnce = G == 4 && D == 128 ? 2 : G;  // groups whose waves' states meet in LDS together (68 KB at most, two workgroups per CU)
  // Groups of rows that K loads alternate between, see load_k.  Rows of one line have nothing to gain from two, and pay for the
  // second set of positions (16 x 16 pairs x ~380, fp16, 9 tokens 14.9 -> 15.1 us), and the fp32 shapes with the most tokens
  // need the registers (8 x 32 x ~600, 24 tokens 50.0 -> 51.1; 16 x 16 x ~600 of 64, 60 tokens 53.1 -> 54.3).  Workgroups that share
  // rows find the second half of a line in the L2 anyway, and gain more from one set less: us, two -> one, fp32 of 64, 32 heads x 6000, 24
  // tokens 31.8 -> 29.9, 4 x 8 x 6000, 64 tokens 52.0 -> 47.7, 2 x 16 x 9000..16000, 32 tokens 62.6 -> 59.4; of 128, 32 x 6000, 64 tokens 85.1 -> 80.2;
  // fp16 of 128, 8 x 12 x 600..2000, 60 tokens 31.6 -> 30.8, bf16, 32 x 5500, 20 tokens 24.8 -> 24.4.
  constexpr int kKSets = NK == 2 || kShared || (Elt::kBytes == 4 && D / 64 * G >= 4) ? 1 : 2;
  constexpr bool kSplitPieces = VW == 8;     // the lane's V values are two pieces half a row apart
  static_assert(kMWin % TR == 0, "tiles do not straddle a window");

  SPAN_TRACE_DECL;
  SPAN_STAMP_AFTER(0, "s", 0);
  const int heads = heads_with_arguments(a);
  const int h = blockIdx.x;
  int b, split, nsl, y0, qb;
  if constexpr (Args::kHasTable) {
    const SliceName e = slice_name(a, a.table[blockIdx.y], (int)blockIdx.y);
    b = e.b;
    split = e.split;
    nsl = e.nsl;
    y0 = e.y0;
    qb = blockIdx.z;
  } else {
    qb = 0;  // grid.z = sequences of block 0, then of block 1, ...
    b = blockIdx.z;
    while (b >= a.batch) {
      b -= a.batch;
      ++qb;
    }
    split = blockIdx.y;
    nsl = a.num_splits;
    y0 = b * nsl;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qi = lane & 15, c4 = lane >> 4;
  const size_t bh = (size_t)b * heads + h;

  struct StreamTables {
    int pos[kWavesPerBlock][kMWin];
    IntervalTables tab;
    unsigned char q[NQ * kQRow] __attribute__((aligned(16)));
  };
  struct WaveStates {  // of kAtOnce groups of 16 tokens
    float acc[kWavesPerBlock][16 * kAtOnce][kAccRow];
  };
  union Overlaid {
    StreamTables st;
    WaveStates ws;
  };
  __shared__ __attribute__((aligned(16))) Overlaid s_u;
  __shared__ __attribute__((aligned(16))) f32x2 s_ml[NQ][kWavesPerBlock];
  __shared__ uint32_t s_ticket;
  auto& s_pos = s_u.st.pos;
  auto& s_q = s_u.st.q;

  // Query token j of this workgroup is row (b, q0 + j, h) of q and out; tokens past the launch's last one are
  // computed from the last real one and never written.
  const int q0 = a.q_first + qb * NQ;
  const int nq_here = min(NQ, a.q_first + a.tokens - q0);
  auto qrow = [&](int j) { return ((size_t)b * a.q_len + (size_t)(q0 + min(j, nq_here - 1))) * heads + h; };

  SequenceWords words = sequence_words<false>(a, b);
  const ListWindow window = list_window(a, b, lane);
  // q goes to LDS (the same for the four waves).  It is fetched here, as are the append form's new rows for the cache
  // (written by the first slice's workgroup, whatever the span holds); both have arrived when the rows' positions are known.
  constexpr int kQLoads = (NQ * kPieces + kThreads - 1) / kThreads;
  const bool append = a.append_pos != nullptr;
  const bool writes_new = append && split == 0;
  u32x4 q_piece[kQLoads], k_piece[kQLoads], v_piece[kQLoads];
#pragma unroll
  for (int i = 0; i < kQLoads; ++i) {
    const int idx = min(tid + i * kThreads, NQ * kPieces - 1);
    const size_t src = qrow(idx / kPieces) * ROWB + 16u * (uint32_t)(idx % kPieces);
    q_piece[i] = *reinterpret_cast<const u32x4*>((const char*)a.q + src);
    if (writes_new) {
      k_piece[i] = *reinterpret_cast<const u32x4*>((const char*)a.k_new + src);
      v_piece[i] = *reinterpret_cast<const u32x4*>((const char*)a.v_new + src);
    }
  }
  // A weight is exp2((score - reference) * post) with the largest unscaled score as reference: the heaviest row's weight is
  // exactly 1 and what is rounded is the distance from it, never the scaled score.  (A rounded scaled reference inside an fma
  // leaves the heaviest row 2^r, r the rounding of the product: for scaled scores from 2^29 on r is no longer small.)
  // post is positive (a hidden row's -Inf stays -Inf); the rest of the scale goes into q: see Elt::scale_query.
  const float post = Elt::post_scale(a.scale_log2e);

  arrived(words);
  // Causal limit: query token j sees no position after lim0 + j.  In the append form the call's tokens sit at
  // positions new0 .. new0 + q_len - 1; those rows come from k_new / v_new, never from the cache.
  // (clamped: any q_pos at or beyond the cache length means "no limit", without overflow)
  const bool limited = a.q_pos != nullptr;
  const int pos0 = limited ? min(words.q_pos, kMaxLen) : 0;
  const int lim0 = limited ? pos0 + q0 : 0x7fffffff;
  const int last_any = limited ? lim0 + nq_here - 1 : 0x7fffffff;
  const int new0 = append ? min(words.append_pos, kMaxLen) : 0x7fffffff;

  Intervals intervals = interval_range(a, words);
  SPAN_STAMP_AFTER(10, "s", intervals.count);
  fetch_first(a, intervals, window, lane);
  int n_total = count_positions(a, intervals, wave, lane, s_u.st.tab);
  n_total = n_total < a.max_tokens ? n_total : a.max_tokens;
  const int T = slice_size(a, n_total, nsl);
  const int slice_begin = split * T;
  const int cnt = __builtin_amdgcn_readfirstlane(clampi(n_total - slice_begin, 0, T));
  SPAN_STAMP_AFTER(1, "s", cnt);

  // How the slice's rows are dealt to the waves (see decode_kernel): contiguous quarters of small slices, tiles
  // round-robin for large ones.
  int nrows, vbase, vgap;
  if (a.interleave) {
    const int units_all = (cnt + TR - 1) / TR;
    const int units = units_all > wave ? (units_all - wave + kWavesPerBlock - 1) / kWavesPerBlock : 0;
    const bool own_last = units > 0 && (wave + (units - 1) * kWavesPerBlock) == units_all - 1;
    nrows = units * TR - (own_last ? units_all * TR - cnt : 0);
    vbase = slice_begin + wave * TR;
    vgap = (kWavesPerBlock - 1) * TR;
  } else {
    const int rpw = (((cnt + kWavesPerBlock - 1) / kWavesPerBlock) + 3) / 4 * 4;
    const int first = min(wave * rpw, cnt);
    nrows = min(first + rpw, cnt) - first;
    vbase = slice_begin + first;
    vgap = 0;
  }
  auto vrow = [&](int r) { return vbase + r + (r / TR) * vgap; };
  if (nrows > 0) {
    if (__builtin_expect(intervals.count <= 64, 1)) tabulate_short<TR, kMWin>(a, intervals, vbase, vgap, min(kMWin, nrows), wave, lane, s_u.st.tab, s_pos[wave]);
    else tabulate_positions(a, intervals, vrow, 0, min(kMWin, nrows), wave, lane, s_u.st.tab, s_pos[wave]);
  }
  SPAN_STAMP_AFTER(2, "s", cnt);

  const uint32_t slab_bytes = (uint32_t)a.max_len * ROWB;
  const __amdgpu_buffer_rsrc_t kslab = slab_resource((const char*)a.k + bh * (size_t)slab_bytes, slab_bytes);
  const __amdgpu_buffer_rsrc_t vslab = slab_resource((const char*)a.v + bh * (size_t)slab_bytes, slab_bytes);
  // new row i of the call (only addressed for positions that the append form brings)
  auto new_row = [&](const void* rows, int i) {
    return (const char*)rows + (((size_t)b * a.q_len + (size_t)i) * heads + h) * ROWB;
  };

  // State of query 16 g + qi in lane (qi, c4).  ref: reference of the weights, the running maximum of the unscaled scores
  // (the same in the four lanes of a query); lsum: this lane's share of their sum; O[g][e][r]: un-normalised output column
  // column(4 c4 + r) + e, times Elt::kWeightScale.
  float ref[G], lsum[G];
  f32x4 O[G][NE];
  // first column of quad u of the values that lane group row i of V^T stands for
  auto column = [&](int i, int u) { return kSplitPieces ? 64 * u + 4 * i : NE * i + 4 * u; };

  u32x4 kr[S][NK];
  uint32_t vr[S][4][VW];

  struct TileRows {         // wave-uniform
    uint32_t ok[S];         // bit i: row 16 s + i takes part
    bool plain;             // every row takes part and every query of the workgroup sees all of them
  };
  // K rows come in loads of eight rows x 128 bytes (kKSets = 2): instructions 2 j and 2 j + 1 bring bytes 128 j .. of rows 0 - 7
  // and 8 - 15, lane (i, c) the 16 bytes c of the line's half i / 8 of row i % 8; order_k puts the halves where the operand wants
  // them.  (Loads of 16 rows x 64 bytes, which are the operand as they come, ask for every line twice: read alone and
  // non-temporal they reach 5.5 TB/s where whole lines reach 6.5.)
  auto load_k = [&](int base, int wn, int ln) {
    const int qi = ln & 15, c4 = ln >> 4;
    TileRows tr;
    tr.plain = true;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      uint32_t off[kKSets];
      bool fresh[kKSets], any_fresh = false;
      int p[kKSets];
      tr.ok[s] = 0;
#pragma unroll
      for (int i = 0; i < kKSets; ++i) {
        constexpr int kRows = 16 / kKSets;
        const int r = base + 16 * s + kRows * i + qi % kRows;
        p[i] = s_pos[wave][r];
        const bool ok = r < wn && p[i] <= last_any;
        tr.ok[s] |= ((uint32_t)__builtin_amdgcn_ballot_w64(ok) & ((1u << kRows) - 1u)) << (kRows * i);
        tr.plain = tr.plain && __builtin_amdgcn_ballot_w64(p[i] > lim0) == 0;
        fresh[i] = ok && p[i] >= new0;
        any_fresh = any_fresh || fresh[i];
        off[i] = ok && !fresh[i] ? (uint32_t)p[i] * ROWB + 64u * (uint32_t)(qi / kRows) + 16u * (uint32_t)c4 : kNoRow;
      }
      tr.plain = tr.plain && tr.ok[s] == 0xffffu;
#pragma unroll
      for (int mm = 0; mm < NK; ++mm) kr[s][mm] = load_piece(kslab, off[mm % kKSets] + 64u * kKSets * (mm / kKSets));
      if (__builtin_amdgcn_ballot_w64(any_fresh) != 0) {  // (rare: the tiles of the call's own tokens)
#pragma unroll
        for (int i = 0; i < kKSets; ++i) {
          if (fresh[i]) {
            const u32x4* src = reinterpret_cast<const u32x4*>(new_row(a.k_new, p[i] - new0)) + 4 * (qi / (16 / kKSets)) + c4;
#pragma unroll
            for (int mm = i; mm < NK; mm += kKSets) kr[s][mm] = src[4 * kKSets * (mm / kKSets)];
          }
        }
      }
    }
    return tr;
  };
  // Afterwards lane (i, c) holds the pieces 4 mm + c of row i: lanes i and i + 8 swap the second line half of row i (first
  // load) for the first half of row i + 8 (second load).
  auto order_k = [&]() {
    if constexpr (kKSets == 2) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int j = 0; j < NK / 2; ++j) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint32_t x = kr[s][2 * j][k], y = kr[s][2 * j + 1][k];
            kr[s][2 * j][k] = swap_half<0xc>(x, y);
            kr[s][2 * j + 1][k] = swap_half<0x3>(y, x);
          }
        }
      }
    }
  };
  auto load_v = [&](int base, const TileRows& tr, int ln) {
    const int qi = ln & 15, c4 = ln >> 4;
    const uint32_t in_row = (kSplitPieces ? 16u : (uint32_t)(VW * 4)) * (uint32_t)qi;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const i32x4 p4 = *reinterpret_cast<const i32x4*>(&s_pos[wave][base + 16 * s + 4 * c4]);
      bool ok[4], any_fresh = false;
      uint32_t off[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        ok[t] = (tr.ok[s] >> (4 * c4 + t)) & 1u;
        any_fresh = any_fresh || (ok[t] && p4[t] >= new0);
        off[t] = ok[t] && p4[t] < new0 ? (uint32_t)p4[t] * ROWB + in_row : kNoRow;
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if constexpr (VW == 2) {
          const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(vslab, off[t], 0, kRowPolicy);
          vr[s][t][0] = w[0];
          vr[s][t][1] = w[1];
        } else {
#pragma unroll
          for (int u = 0; u < VW / 4; ++u) {
            const u32x4 w = load_piece(vslab, off[t] + 256u * u);
#pragma unroll
            for (int k = 0; k < 4; ++k) vr[s][t][4 * u + k] = w[k];
          }
        }
      }
      if (__builtin_amdgcn_ballot_w64(any_fresh) != 0) {  // (rare: the tiles of the call's own tokens)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          if (ok[t] && p4[t] >= new0) {
            const char* src = new_row(a.v_new, p4[t] - new0) + in_row;
#pragma unroll
            for (int k = 0; k < VW; ++k) vr[s][t][k] = *reinterpret_cast<const uint32_t*>(src + 256 * (k / 4) + 4 * (k % 4));
          }
        }
      }
    }
  };

  // Scores of the tile in kr: sc[g][s][t] = query 16 g + qi against row 16 s + 4 c4 + t.  A score is summed in pieces (8
  // products of fp32 values or 32 of 16-bit values, each from zero), not in one long
  // accumulator chain: its rounding goes straight into the weight.
  auto take_scores = [&](f32x4 (&sc)[G][S]) {
    constexpr f32x4 kZero = {0.f, 0.f, 0.f, 0.f};
    order_k();
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const unsigned char* qrow_lds = &s_q[(16 * g + qi) * kQRow + 16 * c4];
      if constexpr (Elt::kBytes == 2) {
#pragma unroll
        for (int s = 0; s < S; ++s) sc[g][s] = kZero;
#pragma unroll
        for (int mm = 0; mm < NK; ++mm) {
          const u32x4 qm = *reinterpret_cast<const u32x4*>(qrow_lds + 64 * mm);
#pragma unroll
          for (int s = 0; s < S; ++s) {
            if constexpr (D == 64 || G < 4) sc[g][s] += Elt::mfma(kr[s][mm], qm, kZero);
            else sc[g][s] = Elt::mfma(kr[s][mm], qm, sc[g][s]);  // (no registers for it)
          }
        }
      } else {
        f32x4 sum[4] = {kZero, kZero, kZero, kZero}, prev[2];
#pragma unroll
        for (int mm = 0; mm < NK; ++mm) {
          const u32x4 qm = *reinterpret_cast<const u32x4*>(qrow_lds + 64 * mm);
          f32x4 piece[2] = {kZero, kZero};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint32_t kw = kr[0][mm][k], qw = qm[k];
            piece[k & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, kw), __builtin_bit_cast(float, qw), piece[k & 1], 0, 0, 0);
          }
          if (mm > 0) sum[(mm - 1) & 3] += prev[0] + prev[1];  // (one piece late: the MFMAs of this one run meanwhile)
          prev[0] = piece[0];
          prev[1] = piece[1];
        }
        sum[(NK - 1) & 3] += prev[0] + prev[1];
        sc[g][0] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
        pin(sc[g][0]);
      }
    }
  };
  // Scores -> weights, and the states' reference and sum; rescales O when the reference moved.
  auto softmax_step = [&](f32x4 (&sc)[G][S], int base, const TileRows& tr) {
    if (!tr.plain) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const i32x4 p4 = *reinterpret_cast<const i32x4*>(&s_pos[wave][base + 16 * s + 4 * c4]);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const bool ok = (tr.ok[s] >> (4 * c4 + t)) & 1u;
          // (no limit: lim0 is the largest int.  Unsigned, as a row that takes no part may be any distance from the limit.)
          const int beyond = (int)((ok ? (uint32_t)p4[t] : 0x7fffffffu) - (uint32_t)lim0);
#pragma unroll
          for (int g = 0; g < G; ++g) sc[g][s][t] = ok && beyond <= 16 * g + qi ? sc[g][s][t] : -INFINITY;
        }
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float mx = -INFINITY;
#pragma unroll
      for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int t = 0; t < 4; ++t) mx = fmaxf(mx, sc[g][s][t]);
      }
      if (__builtin_amdgcn_ballot_w64(mx > ref[g]) != 0) {  // (the maximum settles after the first tiles)
        mx = across_groups_max<16>(mx);
        const float ref_new = fmaxf(ref[g], mx);
        const float ref_safe = ref_new == -INFINITY ? 0.f : ref_new;
        const float alpha = __builtin_amdgcn_exp2f((ref[g] - ref_safe) * post);
        ref[g] = ref_new;
        lsum[g] *= alpha;
#pragma unroll
        for (int e = 0; e < NE; ++e) O[g][e] *= alpha;
      }
      const float ref_safe = ref[g] == -INFINITY ? 0.f : ref[g];
#pragma unroll
      for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int t = 0; t < 4; ++t) sc[g][s][t] = __builtin_amdgcn_exp2f((sc[g][s][t] - ref_safe) * post);
        lsum[g] += (sc[g][s][0] + sc[g][s][1]) + (sc[g][s][2] + sc[g][s][3]);
      }
    }
  };
  // O += V^T P^T with the tile in vr and the weights w.
  auto add_outputs = [&](const f32x4 (&w)[G][S]) {
    if constexpr (Elt::kBytes == 2) {
      uint32_t terms[G][kTerms][2 * S];  // dword 2 s + k: rows 4 c4 + 2 k, + 1 of group s
#pragma unroll
      for (int g = 0; g < G; ++g) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            uint32_t tt[kTerms];
            Elt::template split<kTerms>(w[g][s][2 * k] * Elt::kWeightScale, w[g][s][2 * k + 1] * Elt::kWeightScale, tt);
#pragma unroll
            for (int i = 0; i < kTerms; ++i) terms[g][i][2 * s + k] = tt[i];
          }
        }
      }
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        // element e of the V values, as the pairs (rows 4 c4, + 1), (+ 2, + 3) of each group the MFMA wants
        const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
        uint32_t va[2 * S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          va[2 * s] = __builtin_amdgcn_perm(vr[s][1][e >> 1], vr[s][0][e >> 1], sel);
          va[2 * s + 1] = __builtin_amdgcn_perm(vr[s][3][e >> 1], vr[s][2][e >> 1], sel);
        }
        // (head_dim 64: the tile's own sum first, the running one is rounded once per tile; the smallest terms lead)
        f32x4 part[G];
#pragma unroll
        for (int g = 0; g < G; ++g) part[g] = D == 64 ? f32x4{0.f, 0.f, 0.f, 0.f} : O[g][e];
#pragma unroll
        for (int i = kTerms - 1; i >= 0; --i) {
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const uint32_t* tg = terms[g][i];
            if constexpr (S == 2) part[g] = Elt::mfma(u32x4{va[0], va[1], va[2], va[3]}, u32x4{tg[0], tg[1], tg[2], tg[3]}, part[g]);
            else part[g] = Elt::mfma(u32x2{va[0], va[1]}, u32x2{tg[0], tg[1]}, part[g]);
          }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
          O[g][e] = D == 64 ? O[g][e] + part[g] : part[g];
          if (D == 64) pin(O[g][e]);
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        f32x4 part[G][2];  // the tile's own sums first: the running one is rounded once per tile
#pragma unroll
        for (int g = 0; g < G; ++g) part[g][0] = part[g][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const uint32_t vw = vr[0][t][e];
#pragma unroll
          for (int g = 0; g < G; ++g)
            part[g][t & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, vw), w[g][0][t], part[g][t & 1], 0, 0, 0);
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
          O[g][e] += part[g][0] + part[g][1];
          pin(O[g][e]);
        }
      }
    }
  };
  // The whole pass again, for a cache with V rows that are not finite: those rows are taken out of their tiles and added one
  // at a time on the vector units.  There a row never meets the sums of a query that does not see it, not even with weight
  // zero (0 * Inf), and the fp32 weight meets the V value whole (the terms of a 16-bit weight would turn Inf into
  // Inf + 0 * Inf).  us of the clean call -> with one such row per sequence (with every row taken singly, as it was before):
  // 64 x 32 pairs x 155 positions, 16 tokens, fp16 36 -> 51 (171); 16 x 32 x 700, 32 tokens, bf16 37 -> 60 (623); 8 x 32 x 8192,
  // 16 tokens, bf16 176 -> 291 (2159); 16 x 16 x 380 of 64, 9 tokens, fp16 10 -> 15 (65).
  auto stream_checked = [&]() {
    for (int w0 = 0; w0 < nrows; w0 += kMWin) {
      const int wn = min(kMWin, nrows - w0);
      tabulate_positions(a, intervals, vrow, w0, wn, wave, lane, s_u.st.tab, s_pos[wave]);
#pragma unroll 1
      for (int base = 0; base < wn; base += TR) {
        const TileRows tr = load_k(base, wn, lane);
        load_v(base, tr, lane);
        f32x4 w[G][S];
        take_scores(w);
        softmax_step(w, base, tr);
        uint32_t apart[S];  // bit i: row 16 s + i is not finite (wave-uniform)
#pragma unroll
        for (int s = 0; s < S; ++s) {
          apart[s] = 0;
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            bool wild = false;
#pragma unroll
            for (int k = 0; k < VW; ++k) wild = wild || Elt::not_finite(vr[s][t][k]);
            const uint64_t who = __builtin_amdgcn_ballot_w64(wild);
#pragma unroll
            for (int c = 0; c < 4; ++c) apart[s] |= (who >> (16 * c) & 0xffffu) != 0 ? 1u << (4 * c + t) : 0u;
            if ((who >> (16 * c4) & 0xffffu) != 0) {
#pragma unroll
              for (int k = 0; k < VW; ++k) vr[s][t][k] = 0u;
            }
          }
        }
        add_outputs(w);
#pragma unroll
        for (int s = 0; s < S; ++s) {
#pragma unroll 1
          for (uint32_t todo = apart[s]; todo != 0; todo &= todo - 1) {
            const int i = __builtin_ctz(todo);
            const int p = __builtin_amdgcn_readfirstlane(s_pos[wave][base + 16 * s + i]);
            const __amdgpu_buffer_rsrc_t row = p >= new0 ? slab_resource(new_row(a.v_new, p - new0), ROWB) : vslab;
            const uint32_t row_off = p >= new0 ? 0u : (uint32_t)p * ROWB;
            float wi[G];  // the row's weight for query 16 g + qi: in lane (qi, i / 4), element i % 4
#pragma unroll
            for (int g = 0; g < G; ++g) {
              const float x = (i & 2) != 0 ? ((i & 1) != 0 ? w[g][s][3] : w[g][s][2]) : ((i & 1) != 0 ? w[g][s][1] : w[g][s][0]);
              wi[g] = __shfl(x, 16 * (i >> 2) + qi, 64) * Elt::kWeightScale;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
#pragma unroll
              for (int u = 0; u < NE / 4; ++u) {
                float vf[4];
                const uint32_t off = row_off + (uint32_t)(column(4 * c4 + r, u) * Elt::kBytes);
                if constexpr (Elt::kBytes == 4) Elt::unpack4(load_piece(row, off), vf);
                else Elt::unpack4(__builtin_amdgcn_raw_buffer_load_b64(row, off, 0, kRowPolicy), vf);
#pragma unroll
                for (int g = 0; g < G; ++g) {
                  if (p - lim0 <= 16 * g + qi) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) O[g][4 * u + k][r] = fmaf(wi[g], vf[k], O[g][4 * u + k][r]);
                  }
                }
              }
            }
          }
        }
      }
    }
  };
  auto clear_state = [&]() {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      ref[g] = -INFINITY;
      lsum[g] = 0.f;
#pragma unroll
      for (int e = 0; e < NE; ++e) O[g][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };

#pragma unroll
  for (int i = 0; i < kQLoads; ++i) {
    const int idx = tid + i * kThreads, j = idx / kPieces;
    const uint32_t piece = 16u * (uint32_t)(idx % kPieces);
    if (NQ * kPieces % kThreads != 0 && idx >= NQ * kPieces) continue;
    for (int k = 0; k < 4; ++k) q_piece[i][k] = Elt::scale_query(q_piece[i][k], a.scale_log2e);
    *reinterpret_cast<u32x4*>(&s_q[j * kQRow + piece]) = q_piece[i];
    if (writes_new && j < nq_here) {
      const int p = new0 + q0 + j;
      if (p >= 0 && p < a.max_len) {
        const size_t row = (bh * (size_t)a.max_len + (size_t)p) * ROWB + piece;
        *reinterpret_cast<u32x4*>((char*)a.k + row) = k_piece[i];
        *reinterpret_cast<u32x4*>((char*)a.v + row) = v_piece[i];
      }
    }
  }
  TileRows cur = {};
  if (nrows > 0) {
    cur = load_k(0, min(kMWin, nrows), lane);
    load_v(0, cur, lane);
  }
  __syncthreads();  // q is in LDS
  clear_state();
  for (int w0 = 0; w0 < nrows; w0 += kMWin) {
    const int wn = min(kMWin, nrows - w0);
    if (__builtin_expect(w0 > 0, 0)) {
      // The lane's addresses are computed here and not ahead of the loop, where the compiler would move them: kept across the tiles they
      // cost registers that 32 tokens of 16-bit rows of 64 and of fp32 rows of 128 do not have (2 to 5 spilled, and with them the set-up
      // of scratch memory for every wave; now none).  us, with the spills -> without: 64 x 12 heads x 200..500 of 64, bf16, 32 tokens 22.1 -> 21.0, level ones of ~490, fp16 25.5 -> 23.6; 16 x 32 x
      // 400..800, fp16, 20 tokens 20.6 -> 19.3; 8 x 32 x ~600 fp32 of 128, 24 tokens 44.2 -> 43.8.
      int ln = 16 * c4 + qi;
      asm volatile("" : "+v"(ln));
      tabulate_positions(a, intervals, vrow, w0, wn, wave, ln, s_u.st.tab, s_pos[wave]);
      cur = load_k(0, wn, ln);
      load_v(0, cur, ln);
    }
    // (the window's last tile apart: with the next tile's loads behind a branch the compiler could not count them, and would
    // wait for all of them ahead of this tile's outputs)
    int base = 0;
    for (; base + TR < wn; base += TR) {
      f32x4 sc[G][S];
      take_scores(sc);
      const TileRows next = load_k(base + TR, wn, lane);
      softmax_step(sc, base, cur);
      if constexpr (kSharing == Rows::kInStep) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
      add_outputs(sc);
      load_v(base + TR, next, lane);
      cur = next;
#ifdef SPAN_PHASE_TRACE
      if (w0 == 0 && base == 0) SPAN_STAMP_AFTER(3, "v", lsum[0]);
#endif
      // (the scheduler must not pull the next iteration's work up into this one: the registers would not suffice)
      asm volatile("" ::"v"(lsum[0]) : "memory");
    }
    f32x4 sc[G][S];
    take_scores(sc);
    softmax_step(sc, base, cur);
    add_outputs(sc);
#ifdef SPAN_PHASE_TRACE
    if (w0 == 0 && base == 0) SPAN_STAMP_AFTER(3, "v", lsum[0]);
#endif
  }
  {
    float z[4] = {0.f, 0.f, 0.f, 0.f};  // stay 0 unless some output is Inf or NaN
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int e = 0; e < NE; ++e) {
#pragma unroll
        for (int r = 0; r < 4; ++r) z[r] = fmaf(O[g][e][r], 0.f, z[r]);
      }
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64((z[0] + z[1]) + (z[2] + z[3]) != 0.f) != 0, 0)) {
      clear_state();
      stream_checked();
    }
  }
  SPAN_STAMP_AFTER(4, "v", O[0][0][0] + lsum[0]);

  // ---- the waves' states are merged in LDS, the tokens of kAtOnce groups together -----------------------
  // (What counts here are a wave's own instructions, about five cycles each, and trips to LDS: as few rounds as LDS allows, and a
  // thread stays with one token, whose weights it works out once.  us with 16 tokens a round, weights worked out for every quad of
  // columns and slices merged one after the other -> so: 16 x 8 heads x ~600 positions, bf16, 28 tokens, up to 5 slices 23.9 -> 19.5; 6 x 32 x ~400 of 64, fp16,
  // 62 tokens 21.5 -> 19.1; 2 x 5 x 500..5000, 48 tokens, 22 slices 25.3 -> 21.7; 45 x 32 x ~130, bf16, 60 tokens, whole sequences 78.6 -> 72.9; 16 x 32 x ~700,
  // 32 tokens 39.8 -> 38.9; 64 x 32 x ~155, fp16, 16 tokens 35.5 -> 35.1; 55 shapes of 2 to 64 tokens 1.052 times on average, none slower by 1 %.)
  // (The lane is found again: kept from the start it would cost the tiles a register, where they have none.)
  const int lane_here = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), thread = 64 * wave + lane_here;
  const int qn = lane_here & 15, cn = lane_here >> 4;  // qi and c4
#pragma unroll
  for (int g = 0; g < G; ++g) {  // the four lanes of a query hold the weights of disjoint rows
    lsum[g] = across_groups_sum<16>(lsum[g]) * Elt::kWeightScale;
    if (cn == 0) s_ml[16 * g + qn][wave] = f32x2{ref[g], lsum[g]};
  }
  // Of 16 kAtOnce tokens a thread finishes `part`'s quads of columns of token `mine`: columns 4 (part + kPerToken i) .. + 3.
  constexpr int kPerToken = kThreads / (16 * kAtOnce), kQuads = D / 4 / kPerToken;
  static_assert(kQuads >= 1, "a quad per thread at least");
  const int mine = thread / kPerToken, part = thread % kPerToken;
  const bool direct = nsl == 1;
  const size_t slot_floats = (size_t)a.slot_tokens * D;
  const size_t slot0 = (size_t)y0 * heads + h, my_slot = slot0 + (size_t)split * heads;
  const uint32_t q_in_slot = (uint32_t)(q0 - a.q_first);
  auto acc_slot = [&](size_t slot) { return slab_resource(a.part_acc + slot * slot_floats, (uint32_t)(slot_floats * 4)); };
  auto ml_slot = [&](size_t slot) { return slab_resource(a.part_ml + slot * (size_t)a.slot_tokens * 2, (uint32_t)a.slot_tokens * 8u); };
  auto store_row = [&](int token, float L, const f32x4 (&o)[kQuads]) {
    const float sum = L != 0.f ? L : 1.f;
    float* row = a.out + qrow(token) * D + 4 * part;
#pragma unroll
    for (int i = 0; i < kQuads; ++i) *reinterpret_cast<f32x4*>(row + 4 * kPerToken * i) = f32x4{o[i][0] / sum, o[i][1] / sum, o[i][2] / sum, o[i][3] / sum};
  };
#pragma unroll
  for (int g0 = 0; g0 < G; g0 += kAtOnce) {
    if (16 * g0 >= nq_here) break;  // (workgroup-uniform: groups without a real token)
    __syncthreads();  // the (reference, sum) pairs are in LDS; the streaming tables, or the states of the groups before, are no longer read
#pragma unroll
    for (int g = g0; g < g0 + kAtOnce; ++g) {
      if (16 * g + qn < nq_here) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
          for (int u = 0; u < NE / 4; ++u)
            *reinterpret_cast<f32x4*>(&s_u.ws.acc[wave][16 * (g - g0) + qn][column(4 * cn + r, u)]) =
                f32x4{O[g][4 * u][r], O[g][4 * u + 1][r], O[g][4 * u + 2][r], O[g][4 * u + 3][r]};
        }
      }
    }
    const int token = 16 * g0 + mine;
    float weight[kWavesPerBlock], M = -INFINITY, L = 0.f;
    {
      f32x2 ml[kWavesPerBlock];
#pragma unroll
      for (int w = 0; w < kWavesPerBlock; ++w) ml[w] = s_ml[token][w];
#pragma unroll
      for (int w = 0; w < kWavesPerBlock; ++w)
        if (ml[w][1] != 0.f) M = fmaxf(M, ml[w][0]);  // (a NaN sum counts: it has to reach the output)
#pragma unroll
      for (int w = 0; w < kWavesPerBlock; ++w) {  // (a wave without rows for the token: weight 0, states 0)
        weight[w] = ml[w][1] != 0.f ? __builtin_amdgcn_exp2f((ml[w][0] - M) * post) : 0.f;
        L = fmaf(weight[w], ml[w][1], L);
      }
    }
    __syncthreads();
    if (token < nq_here) {
      f32x4 o[kQuads];
#pragma unroll
      for (int i = 0; i < kQuads; ++i) {
        o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) {
          const f32x4 ow = *reinterpret_cast<const f32x4*>(&s_u.ws.acc[w][mine][4 * (part + kPerToken * i)]);
#pragma unroll
          for (int k = 0; k < 4; ++k) o[i][k] = fmaf(weight[w], ow[k], o[i][k]);
        }
      }
      if (direct) {
        store_row(token, L, o);
      } else {
        const uint32_t at = q_in_slot + (uint32_t)token;
        const __amdgpu_buffer_rsrc_t slot = acc_slot(my_slot);
#pragma unroll
        for (int i = 0; i < kQuads; ++i) publish4(slot, (at * D + (uint32_t)(4 * (part + kPerToken * i))) * 4u, o[i]);
        if (part == 0) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, f32x2{M, L}), ml_slot(my_slot), at * 8u, 0, kThrough);
      }
    }
  }
  SPAN_STAMP_ACKED(6);
  if (direct) {
    SPAN_TRACE_FLUSH();
    return;
  }

  // ---- several slices: the workgroup that arrives last for (b, h) and these tokens merges them all ------------
  // (the hand-over of decode_kernel, step 5).  With several query blocks each has 8 bits of the pair's counter.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // my published stores are acknowledged
  __syncthreads();
  SPAN_STAMP_AFTER(7, "s", 0);
  const int field = a.query_blocks > 1 ? 8 * qb : 0;
  const uint32_t field_mask = a.query_blocks > 1 ? 0xffu : 0xffffffffu;
  if (thread == 0)
    s_ticket = (uint32_t)__hip_atomic_fetch_add(ticket_counter(a, bh), (int)(1u << field), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  SPAN_STAMP_AFTER(8, "v", s_ticket);
  if (((s_ticket >> field) & field_mask) != (uint32_t)(nsl - 1)) {
    SPAN_TRACE_FLUSH();
    return;
  }
  // Slices are merged several at a time: all their states are asked for together and their weights worked out ahead of the sums.  A
  // state costs its instructions whether it is there or not, so up to four slices are merged by code for four (us, by that for eight ->
  // so: 8 x 32 heads x ~300 positions, fp16, 20 tokens 13.8 -> 12.4; 9 x 12 x ~600 of 64, 37 tokens 15.2 -> 14.3; 48 shapes of 2 to 64 tokens 1.027
  // times on average, none slower by 1 %).
  auto merge = [&](int token, auto at_once) {
    constexpr int kMerge = decltype(at_once)::value;
    const uint32_t at = q_in_slot + (uint32_t)token;
    f32x4 o[kQuads];
#pragma unroll
    for (int i = 0; i < kQuads; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float M = -INFINITY, L = 0.f;
    for (int s0 = 0; s0 < nsl; s0 += kMerge) {
      f32x2 ml[kMerge];
      f32x4 os[kMerge][kQuads];
#pragma unroll
      for (int k = 0; k < kMerge; ++k) {
        const size_t slot = slot0 + (size_t)min(s0 + k, nsl - 1) * heads;  // (past the end: a slot that exists, unused)
        ml[k] = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(ml_slot(slot), at * 8u, 0, kThrough));
        const __amdgpu_buffer_rsrc_t states = acc_slot(slot);
#pragma unroll
        for (int i = 0; i < kQuads; ++i) os[k][i] = observe4(states, (at * D + (uint32_t)(4 * (part + kPerToken * i))) * 4u);
      }
      const float before = M;
#pragma unroll
      for (int k = 0; k < kMerge; ++k) {
        if (s0 + k >= nsl) ml[k][1] = 0.f;
        if (ml[k][1] != 0.f) M = fmaxf(M, ml[k][0]);
      }
      const float safe = M == -INFINITY ? 0.f : M;
      if (s0 > 0) {
        const float old = __builtin_amdgcn_exp2f((before - safe) * post);
        L *= old;
#pragma unroll
        for (int i = 0; i < kQuads; ++i) o[i] *= old;
      }
#pragma unroll
      for (int k = 0; k < kMerge; ++k) {
        if (s0 + k < nsl) {
          const float w = ml[k][1] != 0.f ? __builtin_amdgcn_exp2f((ml[k][0] - safe) * post) : 0.f;  // (weight 0: states 0)
          L = fmaf(w, ml[k][1], L);
#pragma unroll
          for (int i = 0; i < kQuads; ++i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) o[i][c] = fmaf(w, os[k][i][c], o[i][c]);
          }
        }
      }
    }
    store_row(token, L, o);
  };
#pragma unroll 1
  for (int g0 = 0; g0 < G; g0 += kAtOnce) {
    const int token = 16 * g0 + mine;
    if (token < nq_here) {
      if (nsl <= 4) merge(token, std::integral_constant<int, 4>{});
      else merge(token, std::integral_constant<int, 8>{});
    }
  }
  // leave this block's part of the ticket counter ready for the next call
  if (thread == 0) __hip_atomic_fetch_add(ticket_counter(a, bh), (int)(0u - ((uint32_t)nsl << field)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  SPAN_STAMP_ACKED(9);
  SPAN_TRACE_FLUSH();
}

constexpr int64_t kOneRoundOfTwo = 512;  // workgroups, two per CU

// Two workgroups of 16 tokens of rows of 128 that share a slice find each other's rows in their XCD's L2 as long as neither runs ahead.  With the next
// tile's loads counted they drift, the further the longer the slice, and from 400 KB of rows a slice on that costs more than it gains.
// They have to be on one XCD (workgroups go to the eight in turn) and to run at once.  us with the loads counted -> in step:
// fp32, 6 x 16 heads x 9000..12000 positions, 20 tokens 353.6 -> 313.7, 7 x 16 x 3000..4000, 17 tokens 126.5 -> 118.8, 2 x 16 x 9000..12000, 32 tokens 107.8 ->
// 101.6, slices of 450 KB 36.5 -> 35.7, of 180 25.8 -> 26.9; 16 bits, 6 x 16 x 9000..12000 129.2 -> 120.8, slices of 450 KB 18.8 -> 17.9, of 340 30.35 -> 30.9.  Not so
// with four workgroups a slice (151.5 -> 156.8), on different XCDs (3 x 5 69.0 -> 73.2), more of them than run at once (2 x 24 fp32 82.5 -> 84.4), rows
// of 64, or 32 tokens a workgroup (6 x 16 fp32, 40 tokens 113 -> 117).
bool keep_in_step(int64_t of_a_block, int blocks, int per_cu, int64_t slice_bytes) {
  return blocks == 2 && of_a_block % 8 == 0 && of_a_block * blocks <= 256 * per_cu && slice_bytes >= 400000;
}

template <class Elt, int D, int G>
void launch_shape(const LaunchArgs& base, const MatrixPlan& p, const uint32_t* table, int batch, int q_first, int tokens, hipStream_t stream) {
  const int blocks = (tokens + 16 * G - 1) / (16 * G);
  auto fill = [&](MatrixArgs& m) {
    static_cast<LaunchArgs&>(m) = base;
    m.q_first = q_first;
    m.tokens = tokens;
    m.slot_tokens = p.tokens;
    m.batch = batch;
    m.query_blocks = blocks;
    m.num_splits = p.num_splits;
    m.slice_tokens = p.slice_tokens;
    m.total_slices = p.total_slices;
    m.even = p.even ? 1 : p.least_slice;
    m.interleave = p.slice_tokens >= kInterleaveFrom ? 1 : 0;
  };
  auto start_tiled = [&](auto one_group, auto rows, auto two_tokens) {
    constexpr bool kOneGroup = decltype(one_group)::value;
    constexpr Rows kSharing = decltype(rows)::value;
    constexpr int kTerms = weight_terms<Elt, D>(decltype(two_tokens)::value);
    if (p.table) {
      MatrixArgsTable m;
      fill(m);
      for (int i = 0; i < p.total_slices; ++i) m.table[i] = table[i];
      hipLaunchKernelGGL((matrix_kernel<Elt, D, G, kOneGroup, MatrixArgsTable, kSharing, kTerms>),
                         dim3((unsigned)base.heads, (unsigned)p.total_slices, (unsigned)blocks), dim3(kThreads), 0, stream, m);
    } else {
      MatrixArgsPlain m;
      fill(m);
      hipLaunchKernelGGL((matrix_kernel<Elt, D, G, kOneGroup, MatrixArgsPlain, kSharing, kTerms>),
                         dim3((unsigned)base.heads, (unsigned)p.num_splits, (unsigned)(batch * blocks)), dim3(kThreads), 0, stream, m);
    }
  };
  const int64_t of_a_block = (int64_t)base.heads * (p.table ? p.total_slices : (int64_t)p.num_splits * batch);  // workgroups
  auto start = [&](auto rows, auto two_tokens) {
    if constexpr (MatrixShape<Elt, D, G>::kHasBoth) {
      if (of_a_block * blocks <= kOneRoundOfTwo) return start_tiled(std::true_type{}, rows, two_tokens);
    }
    start_tiled(std::false_type{}, rows, two_tokens);
  };
  constexpr std::integral_constant<Rows, Rows::kAlone> alone{};
  if constexpr (G < 4) {  // (64 tokens are a call's most: one block)
    if constexpr (G == 1 && D == 128) {
      if (keep_in_step(of_a_block, blocks, MatrixShape<Elt, D, G>::kWaves, (int64_t)p.slice_tokens * 2 * MatrixShape<Elt, D, G>::kRowBytes))
        return start(std::integral_constant<Rows, Rows::kInStep>{}, std::false_type{});
    }
    if (blocks > 1) return start(std::integral_constant<Rows, Rows::kShared>{}, std::false_type{});
  }
  if constexpr (G == 1) {
    if (base.q_len == 2) return start(alone, std::true_type{});
  }
  start(alone, std::false_type{});
}

template <class Elt, int D>
void launch_groups(const LaunchArgs& base, const MatrixPlan& p, const uint32_t* table, int batch, int q_first, int tokens, hipStream_t stream) {
  if (p.groups == 1) launch_shape<Elt, D, 1>(base, p, table, batch, q_first, tokens, stream);
  else if (p.groups == 2 || kMatrixMaxGroups(Elt::kBytes, D) == 2) launch_shape<Elt, D, 2>(base, p, table, batch, q_first, tokens, stream);
  else if constexpr (kMatrixMaxGroups(Elt::kBytes, D) == 4) launch_shape<Elt, D, 4>(base, p, table, batch, q_first, tokens, stream);
}

}  // namespace

hipError_t launch_matrix(const LaunchArgs& base, int dtype, int head_dim, const MatrixPlan& p, const uint32_t* table,
                         int batch, hipStream_t stream) {
  for (int first = 0; first < base.q_len; first += p.tokens) {
    const int tokens = base.q_len - first < p.tokens ? base.q_len - first : p.tokens;
    const bool d128 = head_dim == 128;
    if (dtype == SPAN_F32) {
      if (d128) launch_groups<F32, 128>(base, p, table, batch, first, tokens, stream);
      else launch_groups<F32, 64>(base, p, table, batch, first, tokens, stream);
    } else if (dtype == SPAN_F16) {
      if (d128) launch_groups<F16, 128>(base, p, table, batch, first, tokens, stream);
      else launch_groups<F16, 64>(base, p, table, batch, first, tokens, stream);
    } else {
      if (d128) launch_groups<BF16, 128>(base, p, table, batch, first, tokens, stream);
      else launch_groups<BF16, 64>(base, p, table, batch, first, tokens, stream);
    }
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

}  // namespace spanattn
