// Approximate scores from the 1-bit key cache (Alg. 1 step 2) over many workgroups per unit; first kernel of the fused step.
// How a wavefront scores a pair block: fier_score_dev.h.
#include <type_traits>

#include "fier_dev.h"
#include "fier_kernels.h"
#include "fier_quant_dev.h"
#include "fier_score_dev.h"

namespace fier {

constexpr int kScoreMaxBpw = 13;  // pair blocks per wavefront at most (the launcher keeps to it)

// grid (units * (n_x [+ 1 if HIST])), n_x = ceil(max_ctx / (256 bpw)), block 256: scoring workgroup x of a unit
// owns 4 bpw consecutive pair blocks, wave w the blocks 4 bpw x + w, + 4, + 8, ...  The launcher picks bpw so that the whole grid is
// resident at once: the per-workgroup prologue (q, R) and epilogue (histogram flush, arrival) are then paid once.
//
// HIST (first kernel of the fused step): every score is also counted in an equal-width histogram of kSelBins
// bins over [-R, R], R = sum_c |q_c| * absmax_c >= |score| -- a bound known before any score exists, so that
// scoring and histogramming are one pass.  The workgroup's LDS histogram is added to the unit's histogram in
// memory with device atomics and the workgroup is done: nobody waits or counts arrivals here; the threshold
// kernel reads the merged histogram (and clears it for the next call).
// The extra workgroup of a unit performs the decode-stage append (Sec. 3.1) when k_new is given: its four wavefronts share the
// tokens of the group the new row falls in (eight each of 32-token groups, 32 and up to twice 32 of longer ones), exchange their minima
// and maxima through lscore across a barrier that all four reach, and re-quantize and score their tokens straight from registers; wavefront
// 0 writes the new K/V rows and the group's (s, z).  The other workgroups leave those tokens alone.  The bound R uses the absmax of before the
// append (every workgroup must bin with the same R); the new group's contribution is handed to the last kernel
// of the step through `newmax`.  A score outside [-R, R] simply lands in the outermost bin.
// LONG: quantization groups longer than 32 tokens.  (Separate variants: the long groups' append takes more registers, and
// in one kernel with the other cost the 32-token groups their fifth workgroup per CU: 56 -> 60 us at 32 units x 128k.)
//   The bound asks for six workgroups per CU with 32-token groups (69 to 77 registers; us per step at five / six / seven: 32 units
// x 128k 55.0 / 53.3 / 53.6, 128 ragged units up to 64k 96.9 / 96.7 / 97.2, three such layers 266.6 / 265.6 / 265.2, 32 x 32k
// 32.0 / 32.1 / 31.9), with longer ones for four from two query heads per kv head on: asked for five the compiler puts 8 to 20 bytes
// per lane into scratch at five, seven and eight heads, asked for four it needs 88 to 96 registers up to seven heads (five workgroups fit
// all the same) and 101 at eight.  us per step, fp16, 97 registers at two to seven heads / now, g = 128: 4 heads 28.1 / 27.9 at 8
// units x 32k, 35.8 / 34.6 at 32 x 32k, 55.5 / 53.7 at 32 x 128k, 56.7 / 55.9 at 128 ragged units up to 30k; 6 heads 30.4 / 29.9,
// 38.0 / 36.8 and 59.1 / 58.2 at the first, second and last; 7 heads 58.4 / 56.3 at 32 x 128k.
template <int DT, int NREP, bool HIST, bool STREAM, bool LONG, class LAYERS>
__global__ __launch_bounds__(256, HIST ? (!LONG ? 6 : NREP == 1 ? 5 : 4) : 1) void score_kernel(const uint4* kbits, const uint4* kmeta,
                                                    const float* __restrict__ kabsmax, const uint16_t* __restrict__ q,
                                                    const int32_t* __restrict__ seq_lens, int extra,
                                                    float* __restrict__ scores, UnitCtl* __restrict__ ctl,
                                                    uint32_t* __restrict__ ghist, const int32_t* __restrict__ budgets,
                                                    int max_budget, uint32_t* __restrict__ K, uint32_t* __restrict__ V,
                                                    const uint32_t* __restrict__ k_new,
                                                    const uint32_t* __restrict__ v_new, float* __restrict__ newmax,
                                                    int n_kv_heads, int max_ctx, int bpw, int group_shift, int n_x, KvLayout lay,
                                                    const LAYERS lb) {
  __shared__ uint32_t lhist[HIST ? kSelBins : 1];
  __shared__ __attribute__((aligned(16))) unsigned char a_lds[4 * kAWave];
  // The workgroup's scores wait here and leave as one contiguous burst at the end: stores interleaved block by block
  // with the loads make the memory turn around between reading and writing all the time.
  __shared__ __attribute__((aligned(16))) float lscore[kScoreMaxBpw * 4 * kPair];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  // Workgroups are dispatched in the order of their index.  HIST: the first `units` workgroups are the appending
  // ones (theirs is the longest chain of dependent loads: started last, they would end the kernel
  // late), then n_x scoring workgroups per unit, a unit's ranges next to each other.
  const int n_units = (int)gridDim.x / (n_x + (HIST ? 1 : 0));
  const bool append_wg = HIST && __builtin_expect((int)blockIdx.x < n_units, 0);  // its code out of the others' way
  const int wid = (int)blockIdx.x - (HIST ? n_units : 0);
  const int unit = append_wg ? (int)blockIdx.x : wid / n_x;
  int range = append_wg ? -1 : wid - unit * n_x;
  if constexpr (std::is_same<LAYERS, LayerBatch>::value)
    if (!append_wg) range = turned_wg(range, n_x, (uint32_t)unit, 256u);
  const int b = unit / n_kv_heads;
  if constexpr (std::is_same<LAYERS, LayerBatch>::value) {  // this workgroup's layer
    const int z = (int)blockIdx.z;
    const LayerShift at = lb.at[z];
    const int64_t ws = lb.ws_shift(z);
    kbits = shifted(kbits, at.kbits);
    kmeta = shifted(kmeta, at.kmeta);
    kabsmax = shifted(kabsmax, at.kabsmax);
    seq_lens = shifted(seq_lens, at.seq_lens);
    K = shifted(K, at.k);
    V = shifted(V, at.v);
    lay.table = lay.table ? shifted(lay.table, at.table) : nullptr;
    scores = shifted(scores, ws);
    ctl = shifted(ctl, ws);
    ghist = shifted(ghist, ws);
    newmax = shifted(newmax, ws);
    const size_t zu = (size_t)z * n_units;
    q += zu * NREP * kD;
    if (k_new != nullptr) {
      k_new += zu * (kD / 2);
      v_new += zu * (kD / 2);
    }
  }
  const uint16_t* qb = q + (size_t)unit * NREP * kD;
  // The appending wavefronts' chain of dependent loads is the longest in the kernel: what it needs and what does
  // not depend on the sequence length (the new rows, their lanes' query values) leaves before anything else.
  uint32_t kn = 0, vn = 0, qpair[NREP];
#pragma unroll
  for (int r = 0; r < NREP; ++r) qpair[r] = 0;
  if (__builtin_expect(append_wg, 0) && k_new != nullptr) {
    kn = k_new[(size_t)unit * (kD / 2) + lane];
    vn = v_new[(size_t)unit * (kD / 2) + lane];
#pragma unroll
    for (int r = 0; r < NREP; ++r) qpair[r] = reinterpret_cast<const uint32_t*>(qb + r * kD)[lane];
  }
  int Lold = seq_lens[b];
  Lold = Lold < 0 ? 0 : (Lold > max_ctx ? max_ctx : Lold);
  const bool app = HIST && k_new != nullptr && Lold < max_ctx;  // this unit receives a new row in this step
  int L = HIST ? Lold + (app ? 1 : 0) : Lold + extra;
  L = L > max_ctx ? max_ctx : L;
  const int gshift = LONG ? group_shift : 0;
  const int gsize = kG << gshift;  // tokens per quantization group: 32, 64, 128 or 256
  const int tail_start = app ? (Lold / gsize) * gsize : L;  // tokens from here on are scored by the appending workgroup
  if (__builtin_expect(append_wg, 0)) {
    if (!app) return;
  } else {
    // range 0 of a unit always runs so that an empty unit still gets its control block written
    if (range * (4 * kPair) * bpw >= L && !(HIST && range == 0)) return;
  }
  // ... and the rows of the group the new token falls in as soon as the length is known (longer groups than 32: each of
  // the four wavefronts its chunk)
  uint32_t tail_rows[LONG ? kG : kTailRows];
  int tail_t0 = 0, tail_ntok = 0;
  if (HIST && __builtin_expect(append_wg, 0)) {
    tail_t0 = tail_start;
    tail_ntok = Lold - tail_start + 1;
    if constexpr (LONG) append_load_chunk(K, lay.rows_of(unit), tail_t0, tail_ntok, wave, kn, lane, tail_rows);
    else tail_load(K, lay.rows_of(unit), tail_t0, tail_ntok, wave, lane, tail_rows);
  }
  const int n_groups = max_ctx / gsize;
  const int row = lane >> 4, n = lane & 15;
  const int gsel = row >> 1;  // the group of the pair block whose (s, z) this row of lanes holds
  const int hsel = row & 1;   // the 64-channel half it holds
  FIER_PROF(0, HIST && unit == 0 && range == 3)
  if (HIST) { FIER_PROF_WG(0) }
  FIER_PROF(7, HIST && unit == 0 && append_wg)

  // ---- first block's loads go out before anything else (their addresses do not depend on q) ----------------
  const int P0 = range * (4 * bpw) + wave;  // this wave's blocks: P0, P0 + 4, ...
  const int lim = L < tail_start ? L : tail_start;  // tokens below this are scored by the scoring workgroups
  const bool scoring = !append_wg && P0 * kPair < lim;
  const uint32_t* __restrict__ bits_u = reinterpret_cast<const uint32_t*>(kbits) + (size_t)unit * max_ctx * 4;
  const uint4* __restrict__ meta_u = kmeta + (size_t)unit * n_groups * (kD / 4);
  // lane l loads the whole 16-byte code word of token l of the block (one contiguous 1 KiB request per wavefront);
  // the lane's (s, z) quad of block P is at meta_u[((2 P + gsel) >> gshift) * 32 + 16 hsel + n]: half-block
  // 2 P + gsel (32 tokens) lies in group (2 P + gsel) >> gshift
  // (wavefronts that score nothing load the unit's first block: with the first loads under a branch the compiler moved their
  // results to other registers behind it, and so waited for them before it issued the query's loads)
  const int Pl = scoring ? P0 : 0;
  const uint4* const pb = reinterpret_cast<const uint4*>(bits_u) + ((size_t)Pl * kPair + lane);
  const uint4* const pm = meta_u + ((size_t)((2 * Pl + gsel) >> gshift) * 32 + 16 * hsel + n);
  const int pm_step = 256 >> gshift;  // uint4 per block step: a wave's next block is 4 blocks = 8 half-blocks on
  // blocks of this wave that hold tokens to score: P0, P0 + 4, ... below ceil(lim / 64), at most bpw; only the
  // last of them can be a partial one
  int nb = scoring ? ((lim + kPair - 1) / kPair - P0 + 3) / 4 : 0;
  nb = nb > bpw ? bpw : nb;
  // block P0 + 4 i of this wave; past the wave's last block the last one is fetched again (unconditional loads
  // keep the count of outstanding requests the same on every path)
  auto fetch = [&](uint32_t (&w)[4], uint4& m, int i) {
    i = i < nb ? i : nb - 1;
    i = i < 0 ? 0 : i;
    // STREAM: the codes and metadata are read once per step and, from a size on, are better kept out of the caches
    // (see the launcher)
    const uint4 v = STREAM ? load_stream(pb + (size_t)i * (4 * kPair)) : pb[(size_t)i * (4 * kPair)];
    w[0] = v.x;
    w[1] = v.y;
    w[2] = v.z;
    w[3] = v.w;
    m = STREAM ? load_stream(pm + (size_t)i * pm_step) : pm[(size_t)i * pm_step];
  };
  uint32_t w_cur[4];
  uint4 m_cur;
  fetch(w_cur, m_cur, 0);
  __builtin_amdgcn_sched_barrier(0);

  // ---- the lane's 4 query channels c = 64 hsel + 4 n + e, summed over the query heads of this kv head ------
  float qs[4];
  float R = 0.f, hscale = 0.f;
  {
#pragma unroll
    for (int e = 0; e < 4; ++e) qs[e] = 0.f;
#pragma unroll
    for (int r = 0; r < NREP; ++r) {
      const uint2 qq = *reinterpret_cast<const uint2*>(qb + r * kD + 64 * hsel + 4 * n);
      qs[0] += lo16f<DT>(qq.x);
      qs[1] += hi16f<DT>(qq.x);
      qs[2] += lo16f<DT>(qq.y);
      qs[3] += hi16f<DT>(qq.y);
    }
    if (HIST) {
      const float4 am = *reinterpret_cast<const float4*>(kabsmax + (size_t)unit * kD + 64 * hsel + 4 * n);
      float rpart = fabsf(qs[0]) * am.x;
      rpart += fabsf(qs[1]) * am.y;
      rpart += fabsf(qs[2]) * am.z;
      rpart += fabsf(qs[3]) * am.w;
      rpart = row_allsum(rpart);   // this half of the channels
      rpart += swap_rows(rpart);   // both halves
      // lane 0's sum is taken so that R is bit-identical in every lane, wave and workgroup (the binning must be
      // the same function everywhere)
      R = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(rpart)));
      hscale = sel_scale(R, kSelBins);
      for (int i = tid; i < kSelBins; i += 256) lhist[i] = 0;
      __syncthreads();
    }
  }

  FIER_PROF(1, HIST && unit == 0 && range == 3)
  if (__builtin_expect(append_wg, 0)) {
    if constexpr (HIST) {
      if constexpr (!LONG) {
        static_assert(kAWave >= kTailLds && sizeof(lscore) >= 4 * 64 * sizeof(float4), "scratch of the appending workgroup");
        const int t0 = tail_t0, ntok = tail_ntok;
        uint4 mine;
        const GroupScale gs = append_row_short<DT>(
            K, V, lay.rows_of(unit), const_cast<uint32_t*>(reinterpret_cast<const uint32_t*>(kbits)),
            const_cast<uint32_t*>(reinterpret_cast<const uint32_t*>(kmeta)), unit, Lold, max_ctx, kn, vn, lane, wave, tail_rows,
            reinterpret_cast<float4*>(lscore), mine);
        if (wave == 0) {
          newmax[(size_t)unit * kD + 2 * lane] = gs.amax0();
          newmax[(size_t)unit * kD + 2 * lane + 1] = gs.amax1();
        }
        if (wave * kTailRows < ntok) {
          float q0 = 0.f, q1 = 0.f;
#pragma unroll
          for (int r = 0; r < NREP; ++r) {
            q0 += lo16f<DT>(qpair[r]);
            q1 += hi16f<DT>(qpair[r]);
          }
          // this workgroup scores nothing else: the weights take the operands' place
          const float sc = tail_scores8(mine, wave, q0, q1, gs, a_lds + wave * kAWave);
          const int tok = wave * kTailRows + lane;
          if (lane < kTailRows && tok < ntok) {
            scores[(size_t)unit * max_ctx + t0 + tok] = sc;
            atomicAdd(&lhist[sel_bin(sc, R, hscale, kSelBins)], 1u);
          }
        }
      }
      if constexpr (LONG) {
        // Groups of 64, 128 or 256 tokens: all four wavefronts, 32 tokens at a time; a chunk is scored as soon as its
        // code words exist.
        static_assert(kAWave >= kTailLds && sizeof(lscore) >= 4 * 64 * sizeof(float4), "scratch of the appending workgroup");
        float q0 = 0.f, q1 = 0.f;
#pragma unroll
        for (int r = 0; r < NREP; ++r) {
          q0 += lo16f<DT>(qpair[r]);
          q1 += hi16f<DT>(qpair[r]);
        }
        const int t0 = tail_t0, ntok = tail_ntok;
        const GroupScale gs = append_row_long<DT>(
            K, V, lay.rows_of(unit), const_cast<uint32_t*>(reinterpret_cast<const uint32_t*>(kbits)),
            const_cast<uint32_t*>(reinterpret_cast<const uint32_t*>(kmeta)), unit, Lold, max_ctx, 1 << gshift, kn, vn, lane,
            wave, tail_rows, reinterpret_cast<float4*>(lscore), [&](int c, const uint4& mine, const GroupScale& g) {
              const float sc = tail_scores(mine, c & 1, q0, q1, g, a_lds + wave * kAWave);
              const int tok = (c >> 1) * kPair + lane;  // within the group
              if (tok < ntok && lane >> 5 == (c & 1)) {
                scores[(size_t)unit * max_ctx + t0 + tok] = sc;
                atomicAdd(&lhist[sel_bin(sc, R, hscale, kSelBins)], 1u);
              }
            });
        if (wave == 0) {
          newmax[(size_t)unit * kD + 2 * lane] = gs.amax0();
          newmax[(size_t)unit * kD + 2 * lane + 1] = gs.amax1();
        }
      }
    }
  }

  if (scoring) {
    BlockScorer<DT> scorer;
    scorer.init(qs, a_lds + wave * kAWave);

    // full_tag: every token of the block is below `lim`.  The store and the count are then unmasked, so the number
    // of memory operations in flight is the same on every path and the wait for the next block's loads can leave
    // this block's store outstanding -- with a masked store the compiler has to wait for everything, and the
    // store's acknowledgement (it is the last operation issued) lands on the critical path of every iteration.
    auto score_block = [&](auto full_tag, int it) {
      constexpr bool FULL = decltype(full_tag)::value;
      const int P = P0 + 4 * it;
      const float sc = scorer.score(w_cur, m_cur);
      const int tok = P * kPair + lane;
      lscore[(wave + 4 * it) * kPair + lane] = sc;
      if (HIST && (FULL || tok < lim)) atomicAdd(&lhist[sel_bin(sc, R, hscale, kSelBins)], 1u);
    };
    for (int it = 0; it + 1 < nb; ++it) {
      uint32_t w_nxt[4];
      uint4 m_nxt;
      fetch(w_nxt, m_nxt, it + 1);  // the next block is on its way while this one is scored
      score_block(std::true_type(), it);
#pragma unroll
      for (int t = 0; t < 4; ++t) w_cur[t] = w_nxt[t];
      m_cur = m_nxt;
    }
    score_block(std::false_type(), nb - 1);  // the wave's last block may be a partial one
  }

  // ---- the workgroup's scores: tokens [tok_wg, min(tok_wg + 256 bpw, lim)) in one go ------------------------------
  if (!append_wg) {
    __syncthreads();
    const int tok_wg = range * (4 * kPair) * bpw;
    int n_wg = lim - tok_wg;
    n_wg = n_wg > 4 * kPair * bpw ? 4 * kPair * bpw : n_wg;
    float* __restrict__ dst = scores + (size_t)unit * max_ctx + tok_wg;  // tok_wg is a multiple of 256: 16-byte aligned
    for (int i = 4 * tid; i < n_wg; i += 4 * 256) {
      const float4 v4 = *reinterpret_cast<const float4*>(lscore + i);
      if (i + 3 < n_wg) {
        if constexpr (HIST) {
          // the step's second kernel reads them once, after this kernel has ended: stored with the streaming hint
          // (0.5 us per step at the 64k and 128k shapes, nothing at the others)
          typedef float f4_t __attribute__((ext_vector_type(4)));
          __builtin_nontemporal_store(f4_t{v4.x, v4.y, v4.z, v4.w}, reinterpret_cast<f4_t*>(dst + i));
        } else {
          *reinterpret_cast<float4*>(dst + i) = v4;
        }
      } else {
        dst[i] = v4.x;
        if (i + 1 < n_wg) dst[i + 1] = v4.y;
        if (i + 2 < n_wg) dst[i + 2] = v4.z;
      }
    }
  }
  FIER_PROF(2, HIST && unit == 0 && range == 3)
  FIER_PROF(8, HIST && unit == 0 && append_wg)
  if constexpr (HIST) {
    __syncthreads();
    uint32_t* __restrict__ gh = ghist + (size_t)unit * kSelBins;
    for (int i = tid; i < kSelBins; i += 256) {
      const uint32_t c = lhist[i];
      if (c) atomicAdd(&gh[i], c);
    }
    // the bound the scores were binned with, for the kernels that follow (range 0 of a unit always runs)
    if (range == 0 && tid == 0) {
      UnitCtl* c = &ctl[unit];
      c->R = R;
      c->scale = hscale;
    }
    FIER_PROF(3, unit == 0 && range == 3)
    FIER_PROF_WG(1)
  }
}

// Compiled in parts, FIER_SCORE_PART = DT, next to the rest of this file.
template <int DT, bool HIST>
hipError_t launch_score_dt(KvLayout lay, int n_rep, const uint32_t* kbits, const uint32_t* kmeta, const float* kabsmax,
                                  const void* q, const int32_t* seq_lens, int extra, float* scores,
                                  const StepBuffers* sb, const int32_t* budgets, int max_budget, void* K, void* V,
                                  const void* k_new, const void* v_new, int units, int n_kv_heads, int max_ctx,
                                  int group_size, const LayerBatch& lb, hipStream_t st) {
  const int gshift = group_size == 256 ? 3 : group_size == 128 ? 2 : group_size == 64 ? 1 : 0;
  // Blocks per wavefront.  The smallest that lets every workgroup be resident at once (256 CUs; the registers
  // allow 6 workgroups per CU for the fused kernel, 5 at longer groups -- 4 with 8 query heads per kv head --, 8 for the
  // score-only one), at least 4: prologue (q, R) and epilogue (histogram flush) are then paid once.  Beyond 12 the grid is cut into several rounds of shorter
  // workgroups instead: a workgroup's lifetime bounds the ragged end of the kernel, and in a batch of unequal
  // contexts (the host cannot see the lengths) the short units' workgroups exit at once and the dispatcher
  // backfills the machine with the long units' -- with one round, a few long units would stream alone at one
  // block in flight per wavefront.  Strides of a power of two between the workgroups' streams are avoided (they
  // collide in the memory channels: measured 8 vs 7 or 9, 16 vs 13).
  const int n_blocks = (max_ctx + kPair - 1) / kPair;
  const int all_units = units * lb.n;  // of all layers of the launch
  const int wg_slots = HIST ? 256 * (gshift ? 5 : 6) - all_units : 256 * 8;
  const int per_unit = wg_slots / all_units > 0 ? wg_slots / all_units : 1;
  int bpw = (n_blocks + 4 * per_unit - 1) / (4 * per_unit);
  bpw = bpw < 4 ? 4 : bpw;
  const int rounds = (bpw + 11) / 12;
  bpw = (bpw + rounds - 1) / rounds;
  if (bpw >= 8 && (bpw & (bpw - 1)) == 0) ++bpw;
  if (bpw > kScoreMaxBpw) return hipErrorInvalidValue;  // cannot happen: at most 12, + 1
  int n_x = (n_blocks + 4 * bpw - 1) / (4 * bpw);  // scoring workgroups per unit
  // Workgroups go round-robin to the eight XCDs: with n_x a multiple of four the same ranges of all units are on one or two of
  // them, and of unequal contexts the ranges with tokens are few.  Hence one more, empty workgroup per unit where there are several
  // sequences.  (Several layers: turned_wg.)  us per step: 54 sequences of up to 22k, 5 units each, n_x = 8, 66.0 / 58.9; 21 of up to
  // 44k in 88k, 8 units, 4 heads, n_x = 16, 135.8 / 111.2; over 551 random ragged shapes with such n_x .99 (.75 to 1.04), equal ones
  // 1.00; the score-only launch of one sequence of 65k, 8 units, lost 0.9 of 38.4.
  if (HIST && lb.n == 1 && units > n_kv_heads && n_x % 4 == 0) ++n_x;
  dim3 grid((unsigned)units * (unsigned)(n_x + (HIST ? 1 : 0)), 1, (unsigned)lb.n);
  // Streaming hint on the loads of the codes and their metadata (read once per step).  Measured with the step
  // rotating over 12 layer caches, this kernel alone, us without / with it: 32 units x 128k 34.4 / 30.6, 32 x 64k
  // 19.2 / 16.5, the ragged 128-unit batch 34.5 / 31.5 (whole steps: 62.2 / 61.5, 32.6 / 31.9, 102.3 / 100.7);
  // shapes of 32 units x 32k and below lost 0.2-0.4 us per step with it.  Hence from 64 MB per launch.
  const bool stream = (long)all_units * max_ctx * 32 >= (64L << 20);
#define FIER_SCORE_ARGS                                                                                            \
  (const uint4*)kbits, (const uint4*)kmeta, kabsmax, (const uint16_t*)q, seq_lens, extra, scores,                  \
      sb ? sb->ctl : nullptr, sb ? sb->hist : nullptr, budgets, max_budget, (uint32_t*)K, (uint32_t*)V,            \
      (const uint32_t*)k_new, (const uint32_t*)v_new, sb ? sb->newmax : nullptr, n_kv_heads, max_ctx, bpw, gshift, \
      n_x, lay
  auto launch = [&](auto long_tag, auto rep_tag) {
    constexpr bool LONG = decltype(long_tag)::value;  // without HIST nothing is appended: any group size
    constexpr int R = decltype(rep_tag)::value;
    if constexpr (HIST)
      if (lb.n > 1) {
        if (stream) score_kernel<DT, R, HIST, true, LONG, LayerBatch><<<grid, 256, 0, st>>>(FIER_SCORE_ARGS, lb);
        else score_kernel<DT, R, HIST, false, LONG, LayerBatch><<<grid, 256, 0, st>>>(FIER_SCORE_ARGS, lb);
        return;
      }
    if (stream) score_kernel<DT, R, HIST, true, LONG, OneLayer><<<grid, 256, 0, st>>>(FIER_SCORE_ARGS, OneLayer());
    else score_kernel<DT, R, HIST, false, LONG, OneLayer><<<grid, 256, 0, st>>>(FIER_SCORE_ARGS, OneLayer());
  };
#define FIER_SCORE_CASE(R)                                                                                         \
  case R:                                                                                                          \
    if constexpr (HIST) {                                                                                          \
      if (gshift) launch(std::true_type(), std::integral_constant<int, R>());                                      \
      else launch(std::false_type(), std::integral_constant<int, R>());                                            \
    } else {                                                                                                       \
      launch(std::true_type(), std::integral_constant<int, R>());                                                  \
    }                                                                                                              \
    break;
  switch (n_rep) {
    FIER_SCORE_CASE(1)
    FIER_SCORE_CASE(2)
    FIER_SCORE_CASE(3)
    FIER_SCORE_CASE(4)
    FIER_SCORE_CASE(5)
    FIER_SCORE_CASE(6)
    FIER_SCORE_CASE(7)
    FIER_SCORE_CASE(8)
    default:
      return hipErrorInvalidValue;
  }
#undef FIER_SCORE_CASE
#undef FIER_SCORE_ARGS
  return hipGetLastError();
}

#define FIER_SCORE_INSTANCE(WORD, DT, HIST)                                                                          \
  WORD template hipError_t launch_score_dt<DT, HIST>(                                                               \
      KvLayout, int, const uint32_t*, const uint32_t*, const float*, const void*, const int32_t*, int, float*,      \
      const StepBuffers*, const int32_t*, int, void*, void*, const void*, const void*, int, int, int, int,          \
      const LayerBatch&, hipStream_t);
#ifdef FIER_SCORE_PART
FIER_SCORE_INSTANCE(, FIER_SCORE_PART, true)
FIER_SCORE_INSTANCE(, FIER_SCORE_PART, false)
#else
FIER_SCORE_INSTANCE(extern, DT_F16, true)
FIER_SCORE_INSTANCE(extern, DT_F16, false)
FIER_SCORE_INSTANCE(extern, DT_BF16, true)
FIER_SCORE_INSTANCE(extern, DT_BF16, false)

hipError_t launch_score(int dtype, KvLayout lay, int n_rep, const uint32_t* kbits, const uint32_t* kmeta, const float* kabsmax,
                        const void* q, const int32_t* seq_lens, int extra, float* scores, const StepBuffers* sb,
                        const int32_t* budgets, int max_budget, void* K, void* V, const void* k_new,
                        const void* v_new, int units, int n_kv_heads, int max_ctx, int group_size, const LayerBatch& lb,
                        hipStream_t st) {
  if (sb) {
    if (dtype == DT_F16)
      return launch_score_dt<DT_F16, true>(lay, n_rep, kbits, kmeta, kabsmax, q, seq_lens, extra, scores, sb, budgets,
                                           max_budget, K, V, k_new, v_new, units, n_kv_heads, max_ctx, group_size, lb, st);
    return launch_score_dt<DT_BF16, true>(lay, n_rep, kbits, kmeta, kabsmax, q, seq_lens, extra, scores, sb, budgets,
                                          max_budget, K, V, k_new, v_new, units, n_kv_heads, max_ctx, group_size, lb, st);
  }
  if (dtype == DT_F16)
    return launch_score_dt<DT_F16, false>(lay, n_rep, kbits, kmeta, kabsmax, q, seq_lens, extra, scores, nullptr, nullptr,
                                          0, nullptr, nullptr, nullptr, nullptr, units, n_kv_heads, max_ctx, group_size, lb, st);
  return launch_score_dt<DT_BF16, false>(lay, n_rep, kbits, kmeta, kabsmax, q, seq_lens, extra, scores, nullptr, nullptr, 0,
                                         nullptr, nullptr, nullptr, nullptr, units, n_kv_heads, max_ctx, group_size, lb, st);
}
#endif  // FIER_SCORE_PART

}  // namespace fier
