// Span-restricted single-query (decode) attention for gfx950: the kernel and the C entry points that launch it.
//
// What is computed: for every (batch b, head h), softmax over the scores of the positions in the
// sequence's span only, times the matching V rows (paper Sec. 2.2 eqs. (4)-(6) for one query row,
// restricted to the span as in Sec. 3.3).  The paper's own kernel visits fixed-size blocks that
// touch the span and masks inside them (Algorithm 1); here the span is a list of half-open position
// intervals, so exactly the rows inside the intervals are read and no mask exists.
//
// Mapping to the machine (single-query decode is a GEMV: one multiply-add per loaded element, so
// the kernel is bound by HBM and uses no matrix cores):
//   * grid = (heads, KV slices, batch).  A sequence's span is flattened into a virtual token index
//     0..n_b-1 (prefix sums of the interval lengths) and cut into slices; the host sizes the slices so
//     that one launch fills the chip about once (2048 workgroups), however large that makes a slice.
//     When the caller passes the per-sequence token counts, every sequence is cut into equal slices of
//     about the same size as everyone else's; if the sequences then differ in their number of slices the
//     grid becomes (heads, all slices of all sequences) and a table in the kernel arguments names each
//     slice's sequence, so ragged batches leave no idle workgroup.
//   * a workgroup is 4 wavefronts; each wavefront takes its share of the slice's rows (a contiguous
//     quarter, or every fourth 1 KiB unit of a large slice) and is independent of the others until the
//     final merge - it even builds its own part of the virtual-token -> position table (256 rows at a
//     time), so no barrier sits in front of the first K load.
//   * one 64-lane buffer load fetches 1 KiB = whole rows: D*sizeof(elt)/16 lanes per row, each lane a
//     128-bit piece, non-temporal.  The q.k dot product is finished with DPP adds inside those lanes;
//     every row group of a wavefront carries its own online-softmax state (m, l, acc), merged by
//     log-sum-exp at the end: first across row groups (lane exchanges), then across wavefronts (LDS), then
//     - only if the (batch, head) pair has more than one slice - across slices: every workgroup
//     publishes its state and takes a ticket; the one that arrives last for its pair merges them all,
//     so the whole call is a single launch.
//   * the append entry points also write the new token's K / V row into the cache; within that launch
//     the row is taken from the arguments, never read back from the cache.
//   * two query tokens of a sequence are (for many pairs or fp32 rows) served with one pass over the span's rows (template argument NQ):
//     per-token softmax states in registers, each token under its own causal limit.  Three and more run on the
//     matrix cores (span_matrix.hip).
#include <mutex>

#include "span_device.h"
#include "span_matrix.h"

namespace spanattn {
namespace {

// ---- the streaming kernel ------------------------------------------------------------------------
// NQ query tokens per sequence are served by one pass over the span's rows (NQ = 1: the decode step proper).
// The register budget is 64 per lane for one query (8 waves per SIMD) and 80 for two (6); 128 (4) where a wave has twice the loads
// in flight.
enum class Stream { kDefault, kBoost, kWide };  // see launch_typed
constexpr int waves_per_simd(int nq, Stream stream) { return stream == Stream::kWide ? 4 : (nq == 1 ? 8 : 6); }

template <class Elt, int D, bool kDense, int U, int NQ, class Args, Stream kStream = Stream::kDefault>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(waves_per_simd(NQ, kStream), waves_per_simd(NQ, kStream)))) void
decode_kernel(const Args a) {
  constexpr bool kBoost = kStream == Stream::kBoost;
  constexpr int EPL = Elt::kPerVec;        // elements per lane (one 128-bit piece)
  constexpr int LPR = D / EPL;             // lanes per row
  constexpr int RPL = 64 / LPR;            // rows per wave-wide load
  constexpr uint32_t ROWB = D * Elt::kBytes;
  static_assert(LPR == 8 || LPR == 16 || LPR == 32, "row must span 8, 16 or 32 lanes");

  // heads vary fastest: consecutive workgroups go to different XCDs, and the 'is this slice empty'
  // answer is the same for all heads of a (batch, slice), so full and empty slices spread evenly
  SPAN_TRACE_DECL;
  SPAN_STAMP_AFTER(0, "s", 0);
  const int heads = heads_with_arguments(a);
  const int h = blockIdx.x;
  int b, split, nsl, y0;  // sequence, slice within it, slices of the sequence, first slice row of the sequence
  if constexpr (Args::kHasTable) {
    if constexpr (Args::kHasRuns) {
      const uint32_t e = a.r.slices[blockIdx.y].entry;
      b = e & 1023u;
      split = (e >> 10) & 2047u;
      nsl = e >> 21;
      y0 = (a.entry_bits >> 16 ? a.r.slices[blockIdx.y].reserved : (int)blockIdx.y) - split;
    } else {
      const SliceName e = slice_name(a, a.table[blockIdx.y], (int)blockIdx.y);
      b = e.b;
      split = e.split;
      nsl = e.nsl;
      y0 = e.y0;
    }
  } else {
    b = blockIdx.z;
    split = blockIdx.y;
    nsl = a.num_splits;
    y0 = b * nsl;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // in a scalar register: what derives from it stays scalar
  const int grp = lane / LPR, lir = lane % LPR;
  const size_t bh = (size_t)b * heads + h;

  // Append variant.  Every lane fetches its piece of the new token's K / V row right away (the latency
  // hides behind the metadata chain).  The row is written into the cache by the first slice's workgroup
  // of each (batch, head) and, in this launch, never read back from the cache: the wave that meets
  // position new_pos in its rows takes it from the copy parked in LDS instead, so the kernel has no race.
  // With several query tokens (NQ > 1) every token brings a row, for positions append_pos[b] + token; they are
  // handled with the rows that only some tokens of the pass see (below) and new_pos stays unused.
  const bool append_many = NQ > 1 && a.append_pos != nullptr;
  // Run mode reads nothing of the lists (its launches are promised not to), so no null pointer is replaced by them, and what is given is
  // waited for where it is used.
  SequenceWords words = {};
  if constexpr (!Args::kHasRuns) words = sequence_words<kDense>(a, b);
  auto append_position = [&]() { return Args::kHasRuns ? a.append_pos[b] : words.append_pos; };
  auto query_position = [&]() { return Args::kHasRuns ? a.q_pos[b] : words.q_pos; };
  u32x4 kn_raw = {0u, 0u, 0u, 0u}, vn_raw = {0u, 0u, 0u, 0u};
  if (NQ == 1 && a.append_pos) {
    kn_raw = *reinterpret_cast<const u32x4*>((const char*)a.k_new + bh * ROWB + (uint32_t)lir * 16u);
    vn_raw = *reinterpret_cast<const u32x4*>((const char*)a.v_new + bh * ROWB + (uint32_t)lir * 16u);
  }

  __shared__ int s_pos[kWavesPerBlock][kWin];
  __shared__ IntervalTables s_tab;
  __shared__ __attribute__((aligned(16))) float s_acc[kWavesPerBlock][NQ][D];
  __shared__ u32x4 s_new[NQ == 1 ? kWavesPerBlock : 1][2][LPR];  // append variant: the new K / V row, parked until its owner needs it
  __shared__ f32x2 s_ml[kWavesPerBlock][NQ];
  __shared__ int s_ticket;
#ifdef SPAN_STAGE_LDS
  __shared__ u32x4 s_stage[kWavesPerBlock][2][U][64];  // measurement build: U K tiles and U V tiles of 1 KiB per wave
#endif

  // Query token j is row (b, j, h) of q and out.  (a.q_len is NQ; with the constant in its place the compiler's order costs
  // batch 64 x ~155 positions 0.8 us of 27.0.)
  auto qrow = [&](int j) { return ((size_t)b * a.q_len + (size_t)j) * heads + h; };
  // q pieces of this lane.  Scores carry the factor scale*log2(e), so that exp() becomes exp2(): fp32 q is
  // multiplied by it here, 16-bit q stays as stored and the finished dot product is multiplied instead.
  typename Elt::Q qv[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    const u32x4 qr = *reinterpret_cast<const u32x4*>((const char*)a.q + qrow(j) * ROWB + (uint32_t)lir * 16u);
    qv[j] = Elt::make_q(qr, a.scale_log2e);
  }
  const float post = Elt::kPostScale ? a.scale_log2e : 1.f;
  if constexpr (!Args::kHasRuns) arrived(words);
  const int new_pos = (NQ == 1 && a.append_pos) ? append_position() : -2;  // -2 matches no position
  // Causal limit (few-query variant): query token j sees no position after its own, q_pos[b] + j.
  int lim[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j)  // (clamped: any q_pos at or beyond the cache length means "no limit", without overflow)
    lim[j] = a.q_pos ? min(query_position(), kMaxLen) + j : 0x7fffffff;

  // ---- step 1: how many attended positions does the sequence have, which are mine ----------------
  int n_total;
  Intervals intervals = {0, 0, 0, 0, 0};
  if constexpr (Args::kHasRuns) {
    n_total = 0;  // the slice's rows come from the arguments, see below
  } else if (kDense) {
    n_total = clampi(words.first, 0, a.max_len);
  } else {
    intervals = interval_range(a, words);
    SPAN_STAMP_AFTER(10, "s", intervals.count);
    fetch_first(a, intervals, lane);
    n_total = count_positions(a, intervals, wave, lane, s_tab);
  }
  n_total = n_total < a.max_tokens ? n_total : a.max_tokens;
  int slice_begin, cnt;
  if constexpr (Args::kHasRuns) {  // rows are numbered within the slice
    slice_begin = 0;
    cnt = clampi(a.r.slices[blockIdx.y].rows, 0, kMaxRunSliceRows);
  } else {
    const int T = slice_size(a, n_total, nsl);
    slice_begin = split * T;
    cnt = __builtin_amdgcn_readfirstlane(clampi(n_total - slice_begin, 0, T));
  }
  SPAN_STAMP_AFTER(1, "s", cnt);

  // State of this slice once its waves are merged, un-normalised, m in log2 units: thread t < D holds output column t.
  const int t = tid % D;
  const bool owns = tid < D;
  float M[NQ], L[NQ], o[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    M[j] = -INFINITY;
    L[j] = 0.f;
    o[j] = 0.f;
  }
  // A wave's state goes to LDS, and thread t < D makes one of the four.
  auto leave_state = [&](auto shape, int j, float wave_m, float wave_l, const float* wave_acc) {
    using Shape = decltype(shape);
    float* to = &s_acc[wave][j][Shape::own_column(lane)];
    if constexpr (Shape::kOwn == 2) *reinterpret_cast<f32x2*>(to) = f32x2{wave_acc[0], wave_acc[1]};
    else to[0] = wave_acc[0];
    if (lane == 0) s_ml[wave][j] = f32x2{wave_m, wave_l};
  };
  auto merge_waves = [&]() {
    if (tid < D) {
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        float top = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) top = fmaxf(top, s_ml[w][j][0]);
        const float safe = top == -INFINITY ? 0.f : top;  // (a wave without rows: -Inf, weight 0, sums 0)
        float sum = 0.f, out = 0.f;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) {
          const float wgt = __builtin_amdgcn_exp2f(s_ml[w][j][0] - safe);
          sum = fmaf(wgt, s_ml[w][j][1], sum);
          out = fmaf(wgt, s_acc[w][j][tid], out);
        }
        M[j] = top;
        L[j] = sum;
        o[j] = out;
      }
    }
  };
  // Append variant: the first slice's workgroup writes the new row into the cache, whatever the span holds.
  if (NQ == 1 && a.append_pos && split == 0 && wave == 0 && lane < LPR && new_pos >= 0 && new_pos < a.max_len) {
    const size_t row = (bh * (size_t)a.max_len + (size_t)new_pos) * ROWB + (uint32_t)lir * 16u;
    *reinterpret_cast<u32x4*>((char*)a.k + row) = kn_raw;
    *reinterpret_cast<u32x4*>((char*)a.v + row) = vn_raw;
  }
  if constexpr (NQ > 1) {  // the new tokens' rows, one token per wave
    if (append_many && split == 0 && lane < LPR) {
      for (int i = wave; i < NQ; i += kWavesPerBlock) {
        const int pos_i = min(append_position(), kMaxLen) + i;
        if (pos_i >= 0 && pos_i < a.max_len) {
          const size_t src = qrow(i) * ROWB + (uint32_t)lir * 16u;
          const size_t row = (bh * (size_t)a.max_len + (size_t)pos_i) * ROWB + (uint32_t)lir * 16u;
          *reinterpret_cast<u32x4*>((char*)a.k + row) = *reinterpret_cast<const u32x4*>((const char*)a.k_new + src);
          *reinterpret_cast<u32x4*>((char*)a.v + row) = *reinterpret_cast<const u32x4*>((const char*)a.v_new + src);
        }
      }
    }
  }
  if (cnt > 0) {  // same decision in all 4 waves
  // How the slice's rows are dealt to the 4 waves.  My rows are numbered r = 0..nrows-1; row r is
  // virtual token vrow(r) of the sequence.
  //  * small slices: contiguous quarters (RPL-aligned), four short sequential streams;
  //  * large slices (a.interleave): units of RPL rows (one load instruction, 1 KiB) dealt round-robin,
  //    wave w owns units w, w+4, ...  The workgroup then reads one window that moves through the slice.
  //    Quarters of a large slice are a multiple of the memory-channel interleave apart, so the four
  //    streams (and those of the neighbouring heads, a power-of-two slab stride away) pile onto the same
  //    channels: measured 6.1 -> 6.8 TB/s on batch 64 x 1024 cached tokens when dealing round-robin,
  //    while slices of 100-170 rows are 2-4 % faster with quarters.
  int nrows, vbase, vgap;  // row r is virtual token vbase + r + (r / RPL) * vgap: one formula, no branch where rows are named
  if (a.interleave) {
    const int units_all = (cnt + RPL - 1) / RPL;
    const int units = units_all > wave ? (units_all - wave + kWavesPerBlock - 1) / kWavesPerBlock : 0;
    const bool own_last = units > 0 && (wave + (units - 1) * kWavesPerBlock) == units_all - 1;
    nrows = units * RPL - (own_last ? units_all * RPL - cnt : 0);
    vbase = slice_begin + wave * RPL;
    vgap = (kWavesPerBlock - 1) * RPL;
  } else {
    const int rpw = (((cnt + kWavesPerBlock - 1) / kWavesPerBlock) + RPL - 1) / RPL * RPL;
    const int first = min(wave * rpw, cnt);
    nrows = min(first + rpw, cnt) - first;
    vbase = slice_begin + first;
    vgap = 0;
  }
  auto vrow = [&](int r) { return vbase + r + (r / RPL) * vgap; };

  // ---- steps 2 and 3, one window of kWin rows at a time -----------------------------------------
  const uint32_t slab_bytes = (uint32_t)a.max_len * ROWB;
  const __amdgpu_buffer_rsrc_t kslab = slab_resource((const char*)a.k + bh * (size_t)slab_bytes, slab_bytes);
  const __amdgpu_buffer_rsrc_t vslab = slab_resource((const char*)a.v + bh * (size_t)slab_bytes, slab_bytes);
  const uint32_t lane_off = (uint32_t)lir * 16u;

  float m[NQ], l[NQ];
  float acc[NQ][EPL];
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    m[j] = -INFINITY;
    l[j] = 0.f;
#pragma unroll
    for (int i = 0; i < EPL; ++i) acc[j][i] = 0.f;
  }
  if (NQ == 1 && a.append_pos && lane < LPR) {  // park the new row in LDS (frees the registers)
    s_new[wave][0][lane] = kn_raw;
    s_new[wave][1][lane] = vn_raw;
  }

  // ---- step 2: virtual token -> KV position (span path only) -----------------------------------------
  if constexpr (Args::kHasRuns) {
    // Run mode: the slice is a short list of runs [start, start + len) in the kernel arguments.  Row number v of
    // the slice lies in the last run whose rows-before count is <= v; a wave has at most kWin rows (the host
    // checked the slice size), four per lane, and walks the runs with scalar loads - no LDS search, and no
    // vector memory access ahead of the first K row.
    const uint32_t ro = a.r.slices[blockIdx.y].runs_of;
    const int run0 = min((int)(ro & 0xffffu), kMaxRuns), nrun = min((int)(ro >> 16), kMaxRuns - run0);
    int v[kWin / 64], p[kWin / 64];
#pragma unroll
    for (int k = 0; k < kWin / 64; ++k) {
      v[k] = vrow(lane + 64 * k);
      p[k] = 0;
    }
    int before = 0;
    constexpr int kRunBatch = 8;  // runs fetched together: their scalar loads are all in flight before the first is used
    for (int j0 = 0; j0 < nrun; j0 += kRunBatch) {
      int st[kRunBatch], ln[kRunBatch];
#pragma unroll
      for (int i = 0; i < kRunBatch; ++i) {
        const int idx = min(run0 + j0 + i, kMaxRuns - 1);
        st[i] = a.r.run[idx][0];
        ln[i] = a.r.run[idx][1];
      }
#pragma unroll
      for (int i = 0; i < kRunBatch; ++i) {
        const bool live = j0 + i < nrun;
#pragma unroll
        for (int k = 0; k < kWin / 64; ++k) p[k] = (live && v[k] >= before) ? st[i] + (v[k] - before) : p[k];
        before += live ? ln[i] : 0;
      }
    }
#pragma unroll
    for (int k = 0; k < kWin / 64; ++k)
      if (lane + 64 * k < nrows) s_pos[wave][lane + 64 * k] = clampi(p[k], 0, a.max_len - 1);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    if (!kDense && nrows > 0 && __builtin_expect(intervals.count <= 64, 1)) tabulate_short<RPL, kWin>(a, intervals, vbase, vgap, min(kWin, nrows), wave, lane, s_tab, s_pos[wave]);
  }
  SPAN_STAMP_AFTER(2, "v", lane_off);

  for (int w0 = 0; w0 < nrows; w0 += kWin) {
  const int wn = min(kWin, nrows - w0);  // rows w0 .. w0+wn-1 of mine
  if constexpr (!Args::kHasRuns) {
    if (!kDense && __builtin_expect(w0 > 0 || intervals.count > 64, 0)) tabulate_positions(a, intervals, vrow, w0, wn, wave, lane, s_tab, s_pos[wave]);
  }

  if (NQ == 1 && a.append_pos) {  // is the appended row one of the window's rows?  Then row group 0 takes it in now.
    bool mine = false;
    for (int r = lane; r < wn; r += 64) mine = mine || (kDense ? vrow(w0 + r) : s_pos[wave][r]) == new_pos;
    if (__builtin_amdgcn_ballot_w64(mine) != 0) {  // wave-uniform
      float vf[EPL];
      Elt::unpack(s_new[wave][1][lir], vf);
      const float d = rounded(group_allreduce_sum<LPR>(Elt::dot(s_new[wave][0][lir], qv[0])) * post);
      if (grp == 0) {
        const float l_one = 1.f;
        merge_state(m[0], l[0], acc[0], EPL, d, l_one, vf);
      }
    }
  }

  // Passes of two tokens: the span rows between the first and the last token's causal limit (at most NQ - 1
  // positions of a sequence) are seen by the later tokens only.  The streaming loop below serves the rows every
  // token of the pass sees; these few are taken in here, one at a time, each into the states of exactly the
  // tokens that see it - a hidden row never meets a token's sums, not even with weight zero (0 * Inf).
  // In the append form the pass's own tokens sit at exactly these positions and at the first token's own: their
  // rows are not in the cache yet for this launch and come from k_new / v_new instead.
  if constexpr (NQ > 1) {
    if (a.q_pos) {
      const int first_here = lim[0] + (append_many ? 0 : 1);  // first position the streaming loop leaves out
      for (int r0 = 0; r0 < wn; r0 += 64) {
        const int p = r0 + lane < wn ? s_pos[wave][r0 + lane] : -1;
        uint64_t todo = __builtin_amdgcn_ballot_w64(p >= first_here && p <= lim[NQ - 1]);
        while (todo != 0) {  // wave-uniform
          const int pb = __builtin_amdgcn_readlane(p, __builtin_ctzll(todo));
          todo &= todo - 1;
          u32x4 kb, vb;  // every row group fetches the same row
          if (append_many) {
            const int i = pb - lim[0];  // the token that brought this row
            const size_t src = qrow(i) * ROWB + lane_off;
            kb = *reinterpret_cast<const u32x4*>((const char*)a.k_new + src);
            vb = *reinterpret_cast<const u32x4*>((const char*)a.v_new + src);
          } else {
            const uint32_t off = (uint32_t)pb * ROWB + lane_off;
            kb = load_row_piece(kslab, off);
            vb = load_row_piece(vslab, off);
          }
          float vf[EPL];
          Elt::unpack(vb, vf);
#pragma unroll
          for (int j = 0; j < NQ; ++j) {
            const float d = rounded(group_allreduce_sum<LPR>(Elt::dot(kb, qv[j])) * post);
            if (pb <= lim[j] && grp == 0) {
              const float l_one = 1.f;
              merge_state(m[j], l[j], acc[j], EPL, d, l_one, vf);
            }
          }
        }
      }
    }
  }

  // ---- step 3: stream the window's K and V rows, online softmax per row group -------------------
  for (int base = 0; base < wn; base += RPL * U) {
    if constexpr (kBoost) {  // (wave-uniform: set at the first batch, reset at the second)
      if (w0 + base <= RPL * U) first_batch_priority(w0 + base == 0);
    }
    u32x4 kr[U], vr[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = base + u * RPL + grp;
      const int p = kDense ? vrow(w0 + min(r, wn - 1)) : s_pos[wave][min(r, wn - 1)];
      // Rows that take no part are not fetched at all: a row group past the window's end, the appended row
      // (not in the cache yet for this launch; its owner added it above), and span rows after the causal
      // limit of the first query token of the pass (masked positions have no influence, whatever the cache
      // holds there: Sec. 2.2, mask paragraph; the few rows that only later tokens of the pass see were
      // taken in above).  They request an offset past the slab instead, for which the buffer hardware
      // returns zeros, and get no weight.
      ok[u] = r < wn && p != new_pos && p <= lim[0] && !(append_many && p == lim[0]);
      const uint32_t off = ok[u] ? (uint32_t)p * ROWB + lane_off : 0xfffffff0u;
#ifdef SPAN_STAGE_LDS
      // measurement build: the same rows staged through LDS (direct-to-LDS loads, lane i's 16 bytes land in slot i)
#if defined(__HIP_DEVICE_COMPILE__)  // (the host pass has no LDS address space to type-check the builtin against)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(kslab, &s_stage[wave][0][u][0], 16, off, 0, 0, kRowLoadPolicy);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(vslab, &s_stage[wave][1][u][0], 16, off, 0, 0, kRowLoadPolicy);
#endif
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the tiles are in LDS
#pragma unroll
    for (int u = 0; u < U; ++u) {
      kr[u] = s_stage[wave][0][u][lane];
      vr[u] = s_stage[wave][1][u][lane];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read out before the next iteration's loads overwrite them
    {
#else
      kr[u] = load_row_piece(kslab, off);
      vr[u] = load_row_piece(vslab, off);
#endif
    }
    float w[NQ][U];  // scores first, then softmax weights
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        const float d = group_allreduce_sum<LPR>(Elt::dot(kr[u], qv[j])) * post;
        w[j][u] = ok[u] ? d : -INFINITY;
      }
    }
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      float mx = -INFINITY;
#pragma unroll
      for (int u = 0; u < U; ++u) mx = fmaxf(mx, w[j][u]);
      const float m_new = fmaxf(m[j], mx);
      const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m[j] - m_safe);
      l[j] *= alpha;
#pragma unroll
      for (int i = 0; i < EPL; ++i) acc[j][i] *= alpha;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        w[j][u] = __builtin_amdgcn_exp2f(w[j][u] - m_safe);
        l[j] += w[j][u];
      }
      m[j] = m_new;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float vf[EPL];
      Elt::unpack(vr[u], vf);
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
#pragma unroll
        for (int i = 0; i < EPL; ++i) acc[j][i] = fmaf(w[j][u], vf[i], acc[j][i]);
      }
    }
#ifdef SPAN_PHASE_TRACE
    if (w0 == 0 && base == 0) SPAN_STAMP_AFTER(3, "v", acc[0][0]);
#endif
  }
  }  // windows
  SPAN_STAMP_AFTER(4, "v", acc[0][0]);

  // ---- step 4: merge row groups (lane exchanges), then waves (LDS) --------------------------------
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    GroupMerge<LPR, EPL>::merge(m[j], l[j], acc[j]);
    leave_state(GroupMerge<LPR, EPL>{}, j, m[j], l[j], acc[j]);
  }
  __syncthreads();
  merge_waves();
  }  // cnt > 0
  SPAN_STAMP_AFTER(5, "v", o[0]);

  // Output column t of an un-normalised state.  (A sum that is NaN, of a visible row whose score is NaN or +Inf, is none of an empty one's: it
  // reaches the output, here and through the slices below, however the sequence is cut.)
  auto store_rows = [&](const float* ll, const float* oo) {
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      a.out[qrow(j) * D + t] = ll[j] != 0.f ? oo[j] / ll[j] : 0.f;
    }
  };

  if (nsl == 1) {  // one slice for this (batch, head): this workgroup owns the output row
    if (owns) store_rows(L, o);
    SPAN_STAMP_ACKED(6);
    SPAN_TRACE_FLUSH();
    return;
  }

  // ---- step 5: several slices.  Publish this slice's state; the workgroup that arrives last for
  // (b, h) merges all of them by log-sum-exp and writes the output row (no second kernel launch).
  //
  // Cross-workgroup hand-over without cache-wide fences: the states are written and read with
  // device-scope relaxed atomics (write-through / cache-bypassing accesses, each coherent on its own),
  // the writer waits for its stores to be acknowledged before the ticket is taken, and the reader
  // only starts after its own ticket came back.  A device-scope fence would write back and
  // invalidate the whole L2 of the XCD for every workgroup, which costs far more than the merge.
  // state of slice s of (b, h) lives in slot (y0 + s) * heads + h
  const size_t H = (size_t)heads;
  const size_t my_slot = (size_t)(y0 + split) * H + h;
  if (owns) {
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      if (cnt > 0) publish(&a.part_acc[(my_slot * NQ + j) * D + t], o[j]);
      if (t == 0) {
        publish(&a.part_ml[(my_slot * NQ + j) * 2], M[j]);
        publish(&a.part_ml[(my_slot * NQ + j) * 2 + 1], L[j]);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // my published stores are acknowledged
  }
  __syncthreads();
  SPAN_STAMP_AFTER(7, "s", 0);
  if (tid == 0) s_ticket = __hip_atomic_fetch_add(ticket_counter(a, bh), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  SPAN_STAMP_AFTER(8, "v", s_ticket);
  if (s_ticket != nsl - 1) {
    SPAN_TRACE_FLUSH();
    return;
  }

  // The slices are dealt to groups of D / 4 threads, four columns each: a group merges its slices, then the groups are merged as the row
  // groups of a slice are.  What counts is the workgroup's own instructions, about five cycles each for a wave alone.  us, each column
  // by two threads, slice after slice, and row groups merged whole in every lane (GroupMerge) -> so: 1 x 12 heads x ~2500 positions dense, 20 slices 8.3 -> 7.3;
  // 5 x 32 x ~80 of 64 6.9 -> 6.2; 1 x 16 x ~760 6.8 -> 6.3; 5 x 32 x ~530 12.2 -> 11.5; 20 x 32 x ~600 39.8 -> 39.2; 71 shapes 1.045 times on average,
  // none slower.
  constexpr int kColThreads = D / 4, kGroups = kThreads / kColThreads;
  const int part = tid / kColThreads, col = 4 * (tid % kColThreads);
  const size_t slot0 = (size_t)y0 * H + h;  // slice s of this (b, h) is slot0 + s * H
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    float mm = -INFINITY, ll = 0.f, oo[4] = {0.f, 0.f, 0.f, 0.f};
    auto merge_slices = [&](auto at_once) {  // so many of the group's slices, all of whose states are asked for together
      constexpr int kBatch = decltype(at_once)::value;
      for (int s0 = part; s0 < nsl; s0 += kGroups * kBatch) {
        f32x2 ml[kBatch], lo[kBatch], hi[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
          const size_t state = (slot0 + (size_t)min(s0 + k * kGroups, nsl - 1) * H) * NQ + j;  // (past the end: a slot that exists, unused)
          ml[k] = observe2(&a.part_ml[state * 2]);
          lo[k] = observe2(&a.part_acc[state * D + col]);
          hi[k] = observe2(&a.part_acc[state * D + col + 2]);
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
          if (s0 + k * kGroups < nsl && ml[k][1] != 0.f) {  // (an empty slice's sums are never written)
            const float oo2[4] = {lo[k][0], lo[k][1], hi[k][0], hi[k][1]};
            merge_state(mm, ll, oo, 4, ml[k][0], ml[k][1], oo2);
          }
        }
      }
    };
    if (nsl <= kGroups) merge_slices(std::integral_constant<int, 1>{});
    else merge_slices(std::integral_constant<int, 4>{});
    GroupMerge<kColThreads, 4>::merge(mm, ll, oo);
    leave_state(GroupMerge<kColThreads, 4>{}, j, mm, ll, oo);
  }
  __syncthreads();
  merge_waves();
  if (owns) store_rows(L, o);
  // leave the ticket counter ready for the next call (same device-coherent access path as the tickets)
  if (tid == 0) __hip_atomic_store(ticket_counter(a, bh), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  SPAN_STAMP_ACKED(9);
  SPAN_TRACE_FLUSH();
}

// Zeroes n 32-bit words (a plain kernel, so that the call can also be recorded into a HIP graph).
__global__ __launch_bounds__(256) void zero_words_kernel(uint32_t* p, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// One wave per sequence: the span gains the positions after the ones just appended (see span_advance).  Bound by its chain
// of trips to memory (arguments, list range, list): the lanes read 64 intervals at a time, where one thread per sequence
// walked them one after the other (alone in a graph, us: 8 sequences of 10 intervals 2.4 -> 2.2, 64 of 10 2.7 -> 2.2, 4 of 700
// 77 -> 4.0).
__global__ __launch_bounds__(64) void advance_kernel(int max_len, int num_intervals, int count, const int32_t* offsets,
                                                     const int32_t* starts, int32_t* ends, int32_t* append_pos, int32_t* ctx_lens) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const int p = append_pos[b];
  const int lo = clampi(offsets[b], 0, num_intervals), hi = clampi(offsets[b + 1], lo, num_intervals);
  const int ctx = ctx_lens ? ctx_lens[b] : 0;
  if (p < 0 || (long long)p + 2 * (long long)count > (long long)max_len) return;
  const int next = p + count;  // first position of the next step's tokens; they take next .. next + count - 1
  int grow = -1;        // interval that ends right after the appended tokens (the last one that does)
  bool taken = false;   // some of the next positions are already inside an interval
  for (int i0 = lo; i0 < hi; i0 += 64) {
    const bool here = i0 + lane < hi;
    const int st = here ? starts[i0 + lane] : 0, en = here ? ends[i0 + lane] : 0;
    const uint64_t closes = __builtin_amdgcn_ballot_w64(st < en && en == next);
    if (closes != 0) grow = i0 + 63 - __builtin_clzll(closes);
    taken = taken || __builtin_amdgcn_ballot_w64(st < en && st < next + count && next < en) != 0;
  }
  if (lane == 0) {
    if (grow >= 0 && !taken) ends[grow] = next + count;
    append_pos[b] = next;
    if (ctx_lens) ctx_lens[b] = ctx + count;
  }
}

thread_local int g_last_hip_error = 0;
#ifdef SPAN_PHASE_TRACE
unsigned long long* g_trace = nullptr;  // set by span_debug_set_trace
size_t g_trace_workgroups = 0;
#endif

// ---- scratch owned by the library, for span_decode_attn_static ---------------------------------------
// One array per GPU the library runs on, resident until the process ends.  `scratch` is only a host-side
// handle here: host code never passes it to a kernel or a copy, it asks the runtime once per device where
// that device's copy lives and uses that address from then on.
static __device__ __align__(256) unsigned char scratch[SPAN_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device, null until first asked

// Address of the current device's scratch array; resolves it on the first call for that device.
int static_scratch(void** ptr) {
  int dev = -1;
  hipError_t err = hipGetDevice(&dev);
  if (err == hipSuccess && (dev < 0 || dev >= kMaxDevices)) err = hipErrorInvalidDevice;
  if (err == hipSuccess) {
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
      void* p = nullptr;
      err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (err == hipSuccess && (!p || ((uintptr_t)p & 255u))) err = hipErrorInvalidSymbol;
      if (err == hipSuccess) g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
  }
  if (err != hipSuccess) {
    g_last_hip_error = (int)err;
    return SPAN_ERR_HIP;
  }
  return SPAN_OK;
}

// Twice the loads in flight (kWide), for launches of few workgroups with little to read: nothing but the trips to memory bounds
// them, and a slice of the planner's smallest size is then one batch per wave instead of two.  us, default -> wide: one request of ~560 positions,
// 32 heads x 128, fp16, appended 8.20 -> 7.65, of 64 7.61 -> 7.09; 2 x 12 x ~560 of 64 7.60 -> 7.06; 6 x 8 x 200..250 of 64 7.14 -> 6.62; 4 x 5 x 100..250 fp16
// 7.01 -> 6.57; 2 x 16 x ~400 fp32 of 64 8.07 -> 7.69; 4 workgroups x 80 positions 4.17 -> 3.88; 12 x 5 heads x ~1000 11.5 -> 10.8, of 64 9.66 -> 9.28.
// The line, dense calls, default over wide (more: wide is faster): one batch of rows of 128 bytes 1.04 - 1.14 up to 512 workgroups, of 256 bytes
// 1.03 - 1.09 up to one workgroup per CU, 0.98 - 1.04 up to two; two batches, which fp32 rows of 128 have at the planner's smallest size,
// 1.02 - 1.11 up to 240 workgroups, 1.00 at 256, but 0.93 - 0.97 with 288 to 384 (7 x 16 heads x 276..346 10.0 -> 10.8 us): there the rate of the
// memory counts and it costs the resident waves (64 x ~155: 27.8 -> 30.6; dense rows of 64, 576 workgroups x 250 positions 15.1 -> 15.65).
constexpr int64_t kWideUpToWorkgroups = 512;       // slices of one (wide) batch of rows per wave
constexpr int64_t kWideTwiceUpToWorkgroups = 256;  // of two

// How the grid names its slices.
enum class GridMode { kPlain, kTable, kRuns };

template <class Elt, int D, bool kDense, int NQ>
int launch_typed(const LaunchArgsTable& a, const RunTables* runs, GridMode mode, int batch, hipStream_t stream) {
  // K loads (and as many V loads) a wave has in flight before it consumes the first: 4 KiB + 4 KiB, but
  // never more than 16 rows (with 128-byte rows that is 2 instructions of 8 rows); half of that when
  // several query tokens share the registers
  constexpr int kRowsPerLoad = 64 / (D / Elt::kPerVec);
#ifdef SPAN_IN_FLIGHT
  constexpr int kInFlight = SPAN_IN_FLIGHT;
#else
  constexpr int kInFlight = (kRowsPerLoad >= 8 ? 2 : 4) / (NQ > 1 ? 2 : 1);
#endif
  // short slices of 16-bit rows, one token: the instances that send a wave's first batch at raised priority
  constexpr bool kCanBoost = NQ == 1 && Elt::kBytes == 2 && D == 128 && SPAN_FIRST_BATCH_PRIORITY > 0;
  const bool boost = kCanBoost && a.slice_tokens <= kBoostUpToBatches * kWavesPerBlock * kRowsPerLoad * kInFlight;
  // few workgroups with little to read, one token: twice the loads in flight
  constexpr bool kCanWiden = NQ == 1;
  const int64_t workgroups = (int64_t)a.heads * (mode == GridMode::kPlain ? (int64_t)a.num_splits * batch : a.total_slices);
  constexpr int kWideRows = kWavesPerBlock * kRowsPerLoad * 2 * kInFlight;  // of a slice
  const bool wide = kCanWiden && workgroups <= (a.slice_tokens <= kWideRows ? kWideUpToWorkgroups : kWideTwiceUpToWorkgroups) &&
                    a.slice_tokens <= 2 * kWideRows;
  auto start = [&](const auto& args, dim3 grid) {
    using Args = std::decay_t<decltype(args)>;
    if constexpr (kCanWiden) {
      if (wide) {
        hipLaunchKernelGGL((decode_kernel<Elt, D, kDense, 2 * kInFlight, NQ, Args, Stream::kWide>), grid, dim3(kThreads), 0, stream, args);
        return;
      }
    }
    if constexpr (kCanBoost) {
      if (boost) {
        hipLaunchKernelGGL((decode_kernel<Elt, D, kDense, kInFlight, NQ, Args, Stream::kBoost>), grid, dim3(kThreads), 0, stream, args);
        return;
      }
    }
    hipLaunchKernelGGL((decode_kernel<Elt, D, kDense, kInFlight, NQ, Args>), grid, dim3(kThreads), 0, stream, args);
  };
  if (mode == GridMode::kRuns) {
    if constexpr (!kDense) {
      LaunchArgsRuns ra;
      static_cast<LaunchArgs&>(ra) = static_cast<const LaunchArgs&>(a);
      ra.r = *runs;
      start(ra, dim3((unsigned)a.heads, (unsigned)a.total_slices, 1u));
    } else {
      return SPAN_ERR_SHAPE;  // (not reachable: the dense form never plans runs)
    }
  } else if (mode == GridMode::kTable) {
    start(a, dim3((unsigned)a.heads, (unsigned)a.total_slices, 1u));
  } else {
    LaunchArgsPlain plain;
    static_cast<LaunchArgs&>(plain) = static_cast<const LaunchArgs&>(a);
    start(plain, dim3((unsigned)a.heads, (unsigned)a.num_splits, (unsigned)batch));
  }
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) {
    g_last_hip_error = (int)err;
    return SPAN_ERR_HIP;
  }
  return SPAN_OK;
}

template <class Elt, int D, bool kDense>
int launch_queries(const LaunchArgsTable& a, const RunTables* runs, int nq, GridMode mode, int batch,
                   hipStream_t stream) {
  if constexpr (!kDense) {  // the few-query variant exists for the span form only
    if (nq == 2) return launch_typed<Elt, D, false, 2>(a, runs, mode, batch, stream);
    if (nq != 1) return SPAN_ERR_SHAPE;  // (not reachable: three tokens and more run on the matrix cores)
  }
  return launch_typed<Elt, D, kDense, 1>(a, runs, mode, batch, stream);
}

int32_t entry_bits(const Deal& deal) { return deal.b_bits | deal.n_bits << 8 | (deal.dealt ? 1 << 16 : 0); }

// The dense form, planned from a bound: up to here slices of a fixed size (as many sequences then have empty slices, which end at once).
// us, fixed -> shared: 8 x 32 heads x 600..2000 32.7 -> 33.3, 4 x 32 x 1000..2000 fp32 33.5 -> 34.5, 4 x 16 x 300..1500 of 64 8.62 -> 8.90; but 16 x 16 x
// 200..900 of 64 12.4 -> 12.0, 2 x 32 x 2000..8000 30.3 -> 29.4; more pairs: 20 x 12 x 333..1000 of 64 13.1 (at 240 pairs) -> 12.8, 12 x 32 x 1200..3000
// 70.1 -> 67.2, 20 x 32 x 300..1000 42.9 -> 38.4.
constexpr int64_t kDenseFixedUpToPairs = 256;

template <bool kDense>
int launch(const span_attn_desc_t* d, const void* q, const void* k, const void* v, const int32_t* offsets,
           const int32_t* starts, const int32_t* ends, const int32_t* ctx_lens, float scale, float* out,
           const void* k_new = nullptr, const void* v_new = nullptr, const int32_t* append_pos = nullptr,
           const int32_t* q_pos = nullptr, bool few_query = false) {
  const int rc = check_desc(d);
  if (rc != SPAN_OK) return rc;
  if (query_tokens(d) > 1 && !few_query) return SPAN_ERR_SHAPE;  // only span_decode_attn_multi takes several
  if (!q || !k || !v || !out) return SPAN_ERR_NULL;
  if (kDense ? !ctx_lens : (!offsets || (d->num_intervals > 0 && (!starts || !ends)))) return SPAN_ERR_NULL;
  LaunchArgsTable a;
  RunTables runs;
  span_attn_desc_t own;
  if (kDense && (d->host_span_offsets || d->host_span_starts || d->host_span_ends)) {
    own = *d;  // span lists mean nothing to the dense form
    own.host_span_offsets = own.host_span_starts = own.host_span_ends = nullptr;
    d = &own;
  }
  const TokenCounts counts(d);
  Partition p = plan_for_workspace(d, counts, a.table, kDense ? nullptr : &runs, !kDense);
  const size_t need = workspace_least_bytes(d, p);
  if (need > 0 && (!d->workspace || ((uintptr_t)d->workspace & 255u) || d->workspace_bytes < need))
    return SPAN_ERR_WORKSPACE;
  const int64_t states = need ? states_that_fit(d, p) : 0;

  a.q = q;
  a.k = k;
  a.v = v;
  a.out = out;
  a.offsets = offsets;
  a.starts = starts;
  a.ends = ends;
  a.ctx_lens = ctx_lens;
  a.k_new = k_new;
  a.v_new = v_new;
  a.append_pos = append_pos;
  a.q_pos = q_pos;
  a.q_len = query_tokens(d);
  a.counters = need ? (int32_t*)d->workspace : nullptr;
  a.part_ml = need ? (float*)((char*)d->workspace + workspace_counter_bytes(d)) : nullptr;
  a.part_acc = need ? (float*)((char*)d->workspace + workspace_counter_bytes(d) + workspace_ml_bytes(d, states)) : nullptr;
  a.counter_stride = counter_stride(d);
  a.heads = d->heads;
  a.max_len = d->max_len;
  a.num_intervals = d->num_intervals;
  // (a mean beyond the window's 64 would be fetched for nothing, and the kernel multiplies it by the batch in 31 bits)
  a.intervals_per_seq = d->num_intervals <= 0x7fff && d->num_intervals <= 64 * (int64_t)d->batch ? d->num_intervals * 65536 / d->batch : -1;
  a.slice_tokens = p.slice_tokens;
  a.num_splits = p.num_splits;
  a.max_tokens = p.max_tokens;
  a.even = p.even ? 1 : p.least_slice;
  a.interleave = p.slice_tokens >= kInterleaveFrom ? 1 : 0;
  a.scale_log2e = scale * 1.4426950408889634f;
#ifdef SPAN_PHASE_TRACE
  a.trace = g_trace;
  a.trace_workgroups = g_trace_workgroups;
#endif
  hipStream_t stream = (hipStream_t)d->stream;

  Deal deal;
  MatrixPlan mp;
  if (!kDense && plan_matrix(d, counts, p, states, &mp, a.table)) {
    deal_matrix(d, counts, p, &mp, a.table, &deal);
    a.entry_bits = entry_bits(deal);
    const hipError_t err = launch_matrix(a, d->dtype, d->head_dim, mp, a.table, d->batch, stream);
    if (err != hipSuccess) {
      g_last_hip_error = (int)err;
      return SPAN_ERR_HIP;
    }
    return SPAN_OK;
  }

  if (kDense && (int64_t)d->batch * d->heads <= kDenseFixedUpToPairs) a.even = p.even ? 1 : 0;
  deal_partition(d, counts, &p, a.table, &runs, &deal);
  a.entry_bits = entry_bits(deal);
  a.total_slices = p.total_slices;
  const GridMode mode = p.runs ? GridMode::kRuns : (p.exact ? GridMode::kTable : GridMode::kPlain);
  const bool d128 = d->head_dim == 128;
  const int nq = a.q_len;
  switch (d->dtype) {
    case SPAN_F32:
      return d128 ? launch_queries<F32, 128, kDense>(a, &runs, nq, mode, d->batch, stream)
                  : launch_queries<F32, 64, kDense>(a, &runs, nq, mode, d->batch, stream);
    case SPAN_F16:
      return d128 ? launch_queries<F16, 128, kDense>(a, &runs, nq, mode, d->batch, stream)
                  : launch_queries<F16, 64, kDense>(a, &runs, nq, mode, d->batch, stream);
    default:
      return d128 ? launch_queries<BF16, 128, kDense>(a, &runs, nq, mode, d->batch, stream)
                  : launch_queries<BF16, 64, kDense>(a, &runs, nq, mode, d->batch, stream);
  }
}

}  // namespace
}  // namespace spanattn

extern "C" int span_decode_attn(const span_attn_desc_t* desc, const void* q, const void* k_cache,
                                const void* v_cache, const int32_t* span_offsets, const int32_t* span_starts,
                                const int32_t* span_ends, const int32_t* ctx_lens, float scale, float* out) {
  (void)ctx_lens;
  return spanattn::launch<false>(desc, q, k_cache, v_cache, span_offsets, span_starts, span_ends, nullptr, scale, out);
}

extern "C" int span_decode_attn_static(const span_attn_desc_t* desc, const void* q, const void* k_cache,
                                       const void* v_cache, const int32_t* span_offsets, const int32_t* span_starts,
                                       const int32_t* span_ends, const int32_t* ctx_lens, float scale, float* out) {
  (void)ctx_lens;
  const int rc = spanattn::check_desc(desc);
  if (rc != SPAN_OK) return rc;
  span_attn_desc_t d = *desc;
  d.workspace = nullptr;
  d.workspace_bytes = 0;
  size_t need;
  {
    const spanattn::TokenCounts counts(&d);
    need = spanattn::workspace_bytes(&d, counts, spanattn::plan_partition(&d, counts, nullptr, nullptr, true));
  }
  if (need > SPAN_STATIC_SCRATCH_BYTES) return SPAN_ERR_SCRATCH_LIMIT;
  if (need > 0) {
    void* ptr = nullptr;
    const int src = spanattn::static_scratch(&ptr);
    if (src != SPAN_OK) return src;
    d.workspace = ptr;
    d.workspace_bytes = SPAN_STATIC_SCRATCH_BYTES;
    // the array keeps what the last call (of any shape) left: the tickets of this call's pairs start at zero
    const size_t words = spanattn::workspace_counter_bytes(&d) / sizeof(uint32_t);
    hipLaunchKernelGGL(spanattn::zero_words_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0,
                       (hipStream_t)d.stream, (uint32_t*)ptr, words);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
      spanattn::g_last_hip_error = (int)err;
      return SPAN_ERR_HIP;
    }
  }
  return spanattn::launch<false>(&d, q, k_cache, v_cache, span_offsets, span_starts, span_ends, nullptr, scale, out);
}

extern "C" int span_decode_attn_multi(const span_attn_desc_t* desc, const void* q, const void* k_cache,
                                      const void* v_cache, const int32_t* span_offsets, const int32_t* span_starts,
                                      const int32_t* span_ends, const int32_t* q_pos, float scale, float* out) {
  return spanattn::launch<false>(desc, q, k_cache, v_cache, span_offsets, span_starts, span_ends, nullptr, scale, out,
                                 nullptr, nullptr, nullptr, q_pos, true);
}

extern "C" int dense_decode_attn(const span_attn_desc_t* desc, const void* q, const void* k_cache,
                                 const void* v_cache, const int32_t* ctx_lens, float scale, float* out) {
  return spanattn::launch<true>(desc, q, k_cache, v_cache, nullptr, nullptr, nullptr, ctx_lens, scale, out);
}

extern "C" int span_decode_attn_append(const span_attn_desc_t* desc, const void* q, const void* k_new, const void* v_new,
                                       void* k_cache, void* v_cache, const int32_t* append_pos,
                                       const int32_t* span_offsets, const int32_t* span_starts,
                                       const int32_t* span_ends, float scale, float* out) {
  if (!k_new || !v_new || !append_pos) return SPAN_ERR_NULL;
  return spanattn::launch<false>(desc, q, k_cache, v_cache, span_offsets, span_starts, span_ends, nullptr, scale, out,
                                 k_new, v_new, append_pos);
}

extern "C" int span_decode_attn_multi_append(const span_attn_desc_t* desc, const void* q, const void* k_new,
                                             const void* v_new, void* k_cache, void* v_cache,
                                             const int32_t* append_pos, const int32_t* span_offsets,
                                             const int32_t* span_starts, const int32_t* span_ends, float scale,
                                             float* out) {
  if (!k_new || !v_new || !append_pos) return SPAN_ERR_NULL;
  return spanattn::launch<false>(desc, q, k_cache, v_cache, span_offsets, span_starts, span_ends, nullptr, scale, out,
                                 k_new, v_new, append_pos, append_pos, true);
}

extern "C" int dense_decode_attn_append(const span_attn_desc_t* desc, const void* q, const void* k_new, const void* v_new,
                                        void* k_cache, void* v_cache, const int32_t* append_pos,
                                        const int32_t* ctx_lens, float scale, float* out) {
  if (!k_new || !v_new || !append_pos) return SPAN_ERR_NULL;
  return spanattn::launch<true>(desc, q, k_cache, v_cache, nullptr, nullptr, nullptr, ctx_lens, scale, out, k_new,
                                v_new, append_pos);
}

extern "C" int span_advance(const span_attn_desc_t* desc, const int32_t* span_offsets, const int32_t* span_starts,
                            int32_t* span_ends, int32_t* append_pos, int32_t* ctx_lens) {
  const int rc = spanattn::check_desc(desc);
  if (rc != SPAN_OK) return rc;
  if (!span_offsets || !append_pos || (desc->num_intervals > 0 && (!span_starts || !span_ends))) return SPAN_ERR_NULL;
  hipLaunchKernelGGL(spanattn::advance_kernel, dim3((unsigned)desc->batch), dim3(64), 0, (hipStream_t)desc->stream,
                     desc->max_len, desc->num_intervals, spanattn::query_tokens(desc), span_offsets, span_starts, span_ends,
                     append_pos, ctx_lens);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) {
    spanattn::g_last_hip_error = (int)err;
    return SPAN_ERR_HIP;
  }
  return SPAN_OK;
}

extern "C" int span_workspace_init(const span_attn_desc_t* desc) {
  const int rc = spanattn::check_desc(desc);
  if (rc != SPAN_OK) return rc;
  const spanattn::Partition p = spanattn::plan_for_workspace(desc, spanattn::TokenCounts(desc), nullptr, nullptr, true);
  const size_t need = spanattn::workspace_least_bytes(desc, p);
  if (need == 0) return SPAN_OK;
  if (!desc->workspace || ((uintptr_t)desc->workspace & 255u) || desc->workspace_bytes < need) return SPAN_ERR_WORKSPACE;
  const size_t words = spanattn::workspace_counter_bytes(desc) / sizeof(uint32_t);
  hipLaunchKernelGGL(spanattn::zero_words_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0,
                     (hipStream_t)desc->stream, (uint32_t*)desc->workspace, words);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) {
    spanattn::g_last_hip_error = (int)err;
    return SPAN_ERR_HIP;
  }
  return SPAN_OK;
}

extern "C" int span_last_hip_error(void) { return spanattn::g_last_hip_error; }

#ifdef SPAN_PHASE_TRACE
// Diagnostic build only: device buffer of workgroups * 16 64-bit words that every later launch stamps (null = off);
// workgroups of a launch beyond `workgroups` leave no stamp.
extern "C" void span_debug_set_trace(void* device_words, size_t workgroups) {
  spanattn::g_trace = (unsigned long long*)device_words;
  spanattn::g_trace_workgroups = device_words ? workgroups : 0;
}
#endif
