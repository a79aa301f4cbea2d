// The whole decode step of a unit (append, score, top-B, attention: Alg. 1 with the append of Sec. 3.1) by ONE workgroup,
// for short contexts: the units of one layer or of several (blockIdx.y) side by side, one launch.
//
// The scores of a unit fit LDS, so nothing of the step leaves the workgroup: no histogram in memory, no candidates, threshold
// word or partials handed over, no second launch, no merge.  In order:
//   1. the tail group is re-quantized with the new row and scored from registers, a wavefront per eight tokens; the
//      wavefronts score pair blocks (BlockScorer); every score is binned into an LDS histogram over [-R, R];
//   2. one scan finds the threshold bin; its members (about 1 % of the tokens) are ranked against each other, a wavefront
//      per candidate, 64 comparisons per instruction (beyond kUnitCand members: the radix selection over LDS);
//   3. the selected tokens are listed in ascending order (LDS, and idx_out), a thread owning consecutive tokens;
//   4. the wavefronts gather the rows (attend_rows / attend_rows_mfma), their states meet in LDS, the output is written.
// The control block, the rows per range and the scores are left in the workspace as the two-kernel form leaves them, the
// scores by a call's last layer only.
#include "fier_attn_dev.h"
#include "fier_dev.h"
#include "fier_kernels.h"
#include "fier_quant_dev.h"
#include "fier_score_dev.h"
#include "fier_select_dev.h"

namespace fier {

constexpr int kUnitCand = 512;  // threshold-bin members ranked pairwise
constexpr int kUnitMaxCtx = 16384;
[[maybe_unused]] constexpr uint32_t kUnitFixedLds = kSelBins * 4 + kUnitCand * 8 + kUnitMaxCtx / 64 * 4 + kUnitMaxCtx / kRangeTokens * 4 + 128;
constexpr int kUnitAhead = 3;   // pair blocks in flight per wavefront

// LDS of a workgroup of nw wavefronts beyond its fixed arrays, bytes from the start: scores and the scorers' operands, whose
// place the partials take later; the row list; the minima and maxima the tail's wavefronts exchange.
struct UnitLds {
  uint32_t operands, rows, exchange, bytes;
};
inline UnitLds unit_lds(int nw, int n_rep, int max_ctx, int max_budget) {
  UnitLds l;
  l.operands = (uint32_t)max_ctx * 4;
  const uint32_t scoring = l.operands + (uint32_t)nw * kAWave, partials = (uint32_t)(n_rep * (nw * 160 + 10)) * 4;
  l.rows = ((scoring > partials ? scoring : partials) + 15) / 16 * 16;
  l.exchange = l.rows + ((uint32_t)max_budget * 2 + 15) / 16 * 16;
  l.bytes = l.exchange + (uint32_t)nw * 64 * 16;
  return l;
}

struct UnitArgs {
  const uint4* kbits;
  const uint4* kmeta;
  float* kabsmax;
  uint32_t* K;
  uint32_t* V;
  const uint16_t* q;
  const uint32_t* k_new;  // nullptr: nothing is appended
  const uint32_t* v_new;
  const int32_t* seq_lens;
  const int32_t* budgets;
  float* out;
  int32_t* idx_out;    // nullptr: no index list
  int32_t* count_out;  // nullptr: no counts
  // of the call's last layer's part of the workspace
  UnitCtl* ctl;
  uint32_t* hist;
  uint32_t* sel_cnt;
  float* scores;
  const float* newmax;
  int max_budget, batch, n_kv_heads, max_ctx, gshift, range_tokens;
  float scale_log2e;
  int by_length;  // the longest sequences first
  int scored;     // phase 2 of the step: scores, histogram, R and newmax are in the workspace (every layer's part)
  KvLayout lay;
  UnitLds lds;
};

// The bin that holds the want-th largest score of a histogram in LDS and the number of scores above it; every wavefront finds
// it for itself (a lane owns eight bins), which costs less than the barriers of a scan over the workgroup.
__device__ __forceinline__ void find_bin_wave(const uint32_t* hist, uint32_t want, int& bin, uint32_t& above) {
  static_assert(kSelBins == 512, "eight bins per lane");
  const int lane = threadIdx.x & 63;
  const uint4 lo = *reinterpret_cast<const uint4*>(hist + kSelBins - 8 - 8 * lane);
  const uint4 hi = *reinterpret_cast<const uint4*>(hist + kSelBins - 4 - 8 * lane);
  const uint32_t cnt[8] = {hi.w, hi.z, hi.y, hi.x, lo.w, lo.z, lo.y, lo.x};  // descending bins
  uint32_t sum = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) sum += cnt[k];
  uint32_t before = wave_incl_scan_u32(sum, lane) - sum;
  const int owner = __builtin_ctzll(__ballot(before < want && want <= before + sum) | (1ull << 63));
  int at = 0;
  uint32_t ab = before;
#pragma unroll
  for (int k = 0; k < 7; ++k) {  // past the bins that end before the want-th
    const bool past = at == k && ab + cnt[k] < want;
    at += past;
    ab += past ? cnt[k] : 0u;
  }
  bin = __builtin_amdgcn_readlane(kSelBins - 1 - 8 * lane - at, owner);
  above = (uint32_t)__builtin_amdgcn_readlane((int)ab, owner);
}

// grid (kv heads, layers, batch), block 64 NW.
template <int DT, int NREP, int NW, bool STREAM>
__global__ __launch_bounds__(64 * NW, 4) void unit_step_kernel(UnitArgs a, const LayerBatch lb) {
  constexpr int NT = 64 * NW;
  constexpr int kPitch = NW * 160 + 10;  // floats per head of the partials
  // Tokens of the tail group per wavefront.  With two workgroups per CU the other one fills the gaps of the chain and what counts
  // is its instructions (16 layers of 64 ragged paged units up to 8k 95.4 us, 97.9 with eight tokens a wavefront).
  constexpr int CH = NW == 16 ? kTailRows : kG;
  extern __shared__ __attribute__((aligned(16))) unsigned char arena[];
  __shared__ __attribute__((aligned(16))) uint32_t hist[kSelBins];
  __shared__ unsigned long long cand[kUnitCand];
  __shared__ uint32_t scan_tmp[NW];
  __shared__ uint32_t bound[kUnitMaxCtx / kRangeTokens];  // selected tokens before each range
  __shared__ uint32_t res[2];
  __shared__ uint32_t n_cand;
  __shared__ int32_t lblk[kUnitMaxCtx / 64];
  float* const scores = reinterpret_cast<float*>(arena);
  uint16_t* const rows = reinterpret_cast<uint16_t*>(arena + a.lds.rows);

  FIER_PROF_WG(0)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int z = (int)blockIdx.y, h = (int)blockIdx.x;
  const int n_units = a.batch * a.n_kv_heads;
  const bool last_layer = z == lb.n - 1;
  if (lb.n > 1) {  // this workgroup's layer
    const LayerShift at = lb.at[z];
    a.kbits = shifted(a.kbits, at.kbits);
    a.kmeta = shifted(a.kmeta, at.kmeta);
    a.kabsmax = shifted(a.kabsmax, at.kabsmax);
    a.K = shifted(a.K, at.k);
    a.V = shifted(a.V, at.v);
    a.seq_lens = shifted(a.seq_lens, at.seq_lens);
    a.lay.table = a.lay.table ? shifted(a.lay.table, at.table) : nullptr;
    const size_t zu = (size_t)z * n_units;
    a.q += zu * NREP * kD;
    if (a.k_new) {
      a.k_new += zu * (kD / 2);
      a.v_new += zu * (kD / 2);
    }
    a.out += zu * NREP * kD;
    if (a.idx_out) a.idx_out += zu * a.max_budget;
    if (a.count_out) a.count_out += zu;
    if (a.scored) {
      const int64_t ws = lb.ws_shift(z);
      a.ctl = shifted(a.ctl, ws);
      a.hist = shifted(a.hist, ws);
      a.sel_cnt = shifted(a.sel_cnt, ws);
      a.scores = shifted(a.scores, ws);
      a.newmax = shifted(a.newmax, ws);
    }
  }
  const int max_ctx = a.max_ctx;
  // Grids beyond the resident one: the sequences in the order of their lengths, so that the last workgroups to start
  // are the shortest ones.
  int b = (int)blockIdx.z, Lold;
  if (a.by_length) {  // at most 64 sequences
    const int len = lane < a.batch ? a.seq_lens[lane] : INT32_MIN;
    int before = 0;
    for (int j = 0; j < a.batch; ++j) {
      const int o = __builtin_amdgcn_readlane(len, j);
      before += o > len || (o == len && j < lane);
    }
    b = __builtin_ctzll(__ballot(lane < a.batch && before == (int)blockIdx.z));
    Lold = __builtin_amdgcn_readlane(len, b);
  } else {
    Lold = a.seq_lens[b];
  }
  const int unit = b * a.n_kv_heads + h;
  Lold = Lold < 0 ? 0 : (Lold > max_ctx ? max_ctx : Lold);
  const bool app = a.k_new != nullptr && Lold < max_ctx;
  const int n = Lold + (app ? 1 : 0);
  int B = a.budgets[b];
  const KvRows kv = a.lay.rows_of(unit);
  if (kv.blocks)
    for (int i = tid; i < a.lay.blocks_per_seq; i += NT) lblk[i] = kv.blocks[i];
  for (int i = tid; i < kSelBins; i += NT) hist[i] = 0;

  float R, hscale;
  float amax_lo = 0.f, amax_hi = 0.f;  // bounds of the re-quantized group (wavefront 0: channels 2 lane, 2 lane + 1)
  UnitCtl* const c = &a.ctl[unit];
  if (!a.scored) {
    // ---- 1. append and score --------------------------------------------------------------------------------------------
    const uint16_t* qb = a.q + (size_t)unit * NREP * kD;
    const int gsize = kG << a.gshift, t0 = Lold & ~(gsize - 1), ntok = Lold - t0 + 1;  // the tail group with the new row
    // its chunks of CH tokens, to the end of the group (32 tokens) or of the last pair block that holds one; wavefront w has
    // the chunks w, w + NW, ...; one that has the whole group for itself scores nothing else
    const int chunks = app ? (a.gshift ? (ntok + kPair - 1) / kPair * (kPair / CH) : kG / CH) : 0;
    const int first = chunks == 1 ? 1 : 0, n_waves = NW - first, P0 = wave - first;
    const int tail_start = app ? t0 : n;
    const int n_blocks = (tail_start + kPair - 1) / kPair;  // pair blocks P0, P0 + n_waves, ... are this wavefront's
    const int nb = P0 >= 0 && P0 < n_blocks ? (n_blocks - P0 + n_waves - 1) / n_waves : 0;
    uint32_t kn = 0, vn = 0, trow[CH], qpair[NREP];
    if (wave < chunks) {
      kn = a.k_new[(size_t)unit * (kD / 2) + lane];
      vn = a.v_new[(size_t)unit * (kD / 2) + lane];
#pragma unroll
      for (int r = 0; r < NREP; ++r) qpair[r] = reinterpret_cast<const uint32_t*>(qb + r * kD)[lane];
      tail_load(a.K, kv, t0, ntok, wave, lane, trow);
    }
    const int row = lane >> 4, m16 = lane & 15, gsel = row >> 1, hsel = row & 1;
    const uint4* const pb = a.kbits + ((size_t)unit * max_ctx + (size_t)(P0 > 0 ? P0 : 0) * kPair + lane);
    const uint4* const meta_u = a.kmeta + (size_t)unit * (max_ctx >> (5 + a.gshift)) * (kD / 4) + 16 * hsel + m16;
    uint32_t w[kUnitAhead][4];
    uint4 m[kUnitAhead];
    auto fetch = [&](uint32_t (&ww)[4], uint4& mm, int i) {
      i = i < nb ? i : nb - 1;
      const uint4* p = pb + (size_t)i * n_waves * kPair;
      const uint4* q4 = meta_u + (size_t)((2 * (P0 + i * n_waves) + gsel) >> a.gshift) * 32;
      const uint4 v = STREAM ? load_stream(p) : *p;
      ww[0] = v.x;
      ww[1] = v.y;
      ww[2] = v.z;
      ww[3] = v.w;
      mm = STREAM ? load_stream(q4) : *q4;
    };
    if (nb > 0) {
#pragma unroll
      for (int d = 0; d < kUnitAhead; ++d) fetch(w[d], m[d], d);
    }
    float qs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < NREP; ++r) {
      const uint2 qq = *reinterpret_cast<const uint2*>(qb + r * kD + 64 * hsel + 4 * m16);
      qs[0] += lo16f<DT>(qq.x);
      qs[1] += hi16f<DT>(qq.x);
      qs[2] += lo16f<DT>(qq.y);
      qs[3] += hi16f<DT>(qq.y);
    }
    {
      // the bound of the scores, from before the append: as in the score kernel, the same in every wavefront
      const float4 am = *reinterpret_cast<const float4*>(a.kabsmax + (size_t)unit * kD + 64 * hsel + 4 * m16);
      float rpart = fabsf(qs[0]) * am.x;
      rpart += fabsf(qs[1]) * am.y;
      rpart += fabsf(qs[2]) * am.z;
      rpart += fabsf(qs[3]) * am.w;
      rpart = row_allsum(rpart);
      rpart += swap_rows(rpart);
      R = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(rpart)));
      hscale = sel_scale(R, kSelBins);
    }
    __syncthreads();  // the histogram is clear; the loads above are on their way
    FIER_PROF_WG(1)
    float4* const exchange = reinterpret_cast<float4*>(arena + a.lds.exchange);
    unsigned char* const operands = arena + a.lds.operands + wave * kAWave;
    if (wave < chunks) {
      MinMax mm = tail_minmax_start<DT>(trow, ntok, wave, kn, a.gshift != 0);
      tail_minmax<DT>(mm, trow, ntok, wave, kn);
      for (int c = wave + NW; c * CH < ntok; c += NW) {
        uint32_t r[CH];
        tail_load(a.K, kv, t0, ntok, c, lane, r);
        tail_minmax<DT>(mm, r, ntok, c, kn);
      }
      exchange[wave * 64 + lane] = make_float4(mm.mn0, mm.mx0, mm.mn1, mm.mx1);
    }
    if (chunks > 1) __syncthreads();
    if (wave < chunks) {
      const GroupScale gs = group_scale<DT>(tail_join(exchange, chunks < NW ? chunks : NW, lane));
      uint2* const meta = reinterpret_cast<uint2*>(const_cast<uint32_t*>(reinterpret_cast<const uint32_t*>(a.kmeta)) +
                             ((size_t)unit * (max_ctx >> (5 + a.gshift)) + (size_t)(t0 >> (5 + a.gshift))) * kD) + lane;
      uint4* const bits = const_cast<uint4*>(a.kbits) + (size_t)unit * max_ctx + t0;
      if (wave == 0) {
        a.K[kv.row(Lold) * (kD / 2) + lane] = kn;
        a.V[kv.row(Lold) * (kD / 2) + lane] = vn;
        *meta = make_uint2(gs.s0 | (gs.z0 << 16), gs.s1 | (gs.z1 << 16));
        amax_lo = gs.amax0();
        amax_hi = gs.amax1();
        if (a.gshift == 0 && (t0 & kG) == 0 && ntok == 1) {  // opens a pair block: its second group holds no token yet
          if (lane >= kG) bits[lane] = make_uint4(0, 0, 0, 0);
          meta[kD / 2] = make_uint2(0, 0);
        }
      }
      float q0 = 0.f, q1 = 0.f;
#pragma unroll
      for (int r = 0; r < NREP; ++r) {
        q0 += lo16f<DT>(qpair[r]);
        q1 += hi16f<DT>(qpair[r]);
      }
#pragma unroll 1
      for (int c = wave;;) {
        const uint4 mine = tail_codes<DT>(trow, ntok, c, kn, gs, lane);
        if (lane / CH == c % (kPair / CH)) bits[c * CH / kPair * kPair + lane] = mine;
        if (c * CH < ntok) {
          float sc;
          if constexpr (CH == kG) sc = tail_scores(mine, c & 1, q0, q1, gs, operands);
          else sc = tail_scores8(mine, c & 7, q0, q1, gs, operands);
          const int tok = c * CH + lane;
          if (lane < CH && tok < ntok) {
            scores[t0 + tok] = sc;
            atomicAdd(&hist[sel_bin(sc, R, hscale, kSelBins)], 1u);
          }
        }
        c += NW;
        if (c >= chunks) break;
        tail_load(a.K, kv, t0, ntok, c, lane, trow);
      }
    }
    FIER_PROF_WG(2)
    if (nb > 0) {
      BlockScorer<DT> scorer;
      scorer.init(qs, operands);
      auto one = [&](uint32_t (&ww)[4], const uint4& mq, int i) {
        const float sc = scorer.score(ww, mq);
        const int tok = (P0 + i * n_waves) * kPair + lane;
        if (tok < tail_start) {
          scores[tok] = sc;
          atomicAdd(&hist[sel_bin(sc, R, hscale, kSelBins)], 1u);
        }
      };
      for (int i = 0; i < nb; i += kUnitAhead) {
#pragma unroll
        for (int d = 0; d < kUnitAhead; ++d)
          if (i + d < nb) {
            one(w[d], m[d], i + d);
            fetch(w[d], m[d], i + d + kUnitAhead);
          }
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the appended rows, before other wavefronts gather them
  } else {
    R = c->R;
    hscale = c->scale;
    const float* __restrict__ s = a.scores + (size_t)unit * max_ctx;
    __syncthreads();
    for (int i = tid; i < n; i += NT) {
      const float sc = s[i];
      scores[i] = sc;
      atomicAdd(&hist[sel_bin(sc, R, hscale, kSelBins)], 1u);
    }
    if (wave == 0 && app) {
      amax_lo = a.newmax[(size_t)unit * kD + 2 * lane];
      amax_hi = a.newmax[(size_t)unit * kD + 2 * lane + 1];
    }
    uint32_t* __restrict__ gh = a.hist + (size_t)unit * kSelBins;
    for (int i = tid; i < kSelBins; i += NT) gh[i] = 0;
  }
  B = B > a.max_budget ? a.max_budget : B;
  B = B > n ? n : B;
  B = B < 0 ? 0 : B;
  if (tid == 0) n_cand = 0;
  __syncthreads();  // scores, histogram
  FIER_PROF_WG(3)
  if (app && wave == 0) {  // every wavefront has read the bounds; non-negative floats order like their bit patterns
    uint32_t* slot = reinterpret_cast<uint32_t*>(a.kabsmax + (size_t)unit * kD) + 2 * lane;
    if (amax_lo >= 0.f) atomicMax(slot, __float_as_uint(amax_lo));
    if (amax_hi >= 0.f) atomicMax(slot + 1, __float_as_uint(amax_hi));
  }
  GatherQuery<NREP> qr;
  qr.load(reinterpret_cast<const uint4*>(a.q) + (size_t)unit * NREP * (kD / 8));

  // ---- 2. the threshold bin, and the exact threshold among its members -------------------------------------------------------
  const bool need_threshold = B > 0 && B < n;
  int tbin = B >= n ? -1 : kSelBins;  // everything / nothing is selected by bin alone
  uint32_t above = 0;
  if (need_threshold) find_bin_wave(hist, (uint32_t)B, tbin, above);
  const uint32_t in_bin = need_threshold ? hist[tbin] : 0u;
  // a thread owns `own` consecutive tokens: a power of two from 4 to 32
  int own = 4;
  while (own * NT < n) own *= 2;
  const int i0 = tid * own;
  uint32_t dmask = 0, cmask = 0;
  {
    const float from = (float)tbin, to = (float)(tbin + 1);  // sel_bin without its conversion
    for (int j = 0; j < own; j += 4) {
      if (i0 + j >= n) break;
      const float4 v4 = *reinterpret_cast<const float4*>(scores + i0 + j);
      const float vv[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float x = fminf(fmaxf((vv[k] + R) * hscale, 0.0f), (float)(kSelBins - 1));
        const bool ok = i0 + j + k < n;
        dmask |= ok && x >= to ? 1u << (j + k) : 0u;
        cmask |= ok && x >= from && x < to ? 1u << (j + k) : 0u;
      }
    }
  }
  uint32_t T = 0;
  int32_t idxT = -1;
  if (need_threshold) {
    const uint32_t want = (uint32_t)B - above;  // >= 1 of them are selected, larger key first, equal keys by lower index
    if (in_bin <= (uint32_t)kUnitCand) {
      for (uint32_t mb = cmask; __ballot(mb != 0u); mb &= mb - 1u) {  // one atomic per wavefront and round
        const unsigned long long has = __ballot(mb != 0u);
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&n_cand, (uint32_t)__builtin_popcountll(has));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) +
             __builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u));
        if (mb) {
          const int t = i0 + __builtin_ctz(mb);
          cand[at] = ((unsigned long long)score_key(scores[t]) << 32) | (uint32_t)~t;
        }
      }
      __syncthreads();
      if (in_bin <= 128u) {
        const unsigned long long c0 = (uint32_t)lane < in_bin ? cand[lane] : 0ull;
        const unsigned long long c1 = (uint32_t)lane + 64u < in_bin ? cand[lane + 64] : 0ull;
        for (uint32_t k = wave; k < in_bin; k += NW) {
          const unsigned long long from = k < 64u ? c0 : c1;
          const unsigned long long me =
              ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(from >> 32), (int)(k & 63u)) << 32) |
              (uint32_t)__builtin_amdgcn_readlane((int)from, (int)(k & 63u));
          const int rank = __builtin_popcountll(__ballot(c0 > me)) + __builtin_popcountll(__ballot(c1 > me));
          if ((uint32_t)rank == want - 1u && lane == 0) {
            res[0] = (uint32_t)(me >> 32);
            res[1] = ~(uint32_t)me;
          }
        }
      } else {
        for (uint32_t k = wave; k < in_bin; k += NW) {
          const unsigned long long me = cand[k];
          uint32_t rank = 0;
          for (uint32_t j = 0; j < in_bin; j += 64)
            rank += (uint32_t)__builtin_popcountll(__ballot(j + lane < in_bin && cand[j + lane < in_bin ? j + lane : 0] > me));
          if (rank == want - 1u && lane == 0) {
            res[0] = (uint32_t)(me >> 32);
            res[1] = ~(uint32_t)me;
          }
        }
      }
      __syncthreads();
      T = res[0];
      idxT = (int32_t)res[1];
    } else {
      __syncthreads();
      stream_select<NT>([&](int k) { return scores[k]; }, n, tbin, R, hscale, want, reinterpret_cast<uint32_t*>(cand),
                        scan_tmp, res, nullptr, T, idxT);
      __syncthreads();
    }
  }

  FIER_PROF_WG(4)
  // ---- 3. the selection, in token order ---------------------------------------------------------------------------------------
  for (uint32_t mb = cmask; mb; mb &= mb - 1u) {
    const int j = __builtin_ctz(mb);
    const uint32_t key = score_key(scores[i0 + j]);
    if (key > T || (key == T && i0 + j <= idxT)) dmask |= 1u << j;
  }
  const uint32_t n_sel = (uint32_t)B;
  uint32_t pos;
  {
    const uint32_t cnt = (uint32_t)__builtin_popcount(dmask), incl = wave_incl_scan_u32(cnt, lane);
    if (lane == 63) scan_tmp[wave] = incl;
    __syncthreads();
    const uint32_t of_wave = lane < NW ? scan_tmp[lane] : 0u;
    pos = (uint32_t)__builtin_amdgcn_readlane((int)(wave_incl_scan_u32(of_wave, lane) - of_wave), wave) + incl - cnt;
  }
  if (i0 % kRangeTokens == 0 && i0 < kUnitMaxCtx) bound[i0 / kRangeTokens] = pos;
  for (uint32_t mb = dmask; mb; mb &= mb - 1u) {
    const int t = i0 + __builtin_ctz(mb);
    rows[pos] = (uint16_t)t;
    if (a.idx_out) a.idx_out[(size_t)unit * a.max_budget + pos] = t;
    ++pos;
  }
  if (!a.scored && last_layer) {
    float* __restrict__ dst = a.scores + (size_t)unit * max_ctx;
    for (int i = 4 * tid; i < n; i += 4 * NT) {
      const float4 v4 = *reinterpret_cast<const float4*>(scores + i);
      if (i + 3 < n) {
        *reinterpret_cast<float4*>(dst + i) = v4;
      } else {
        dst[i] = v4.x;
        if (i + 1 < n) dst[i + 1] = v4.y;
        if (i + 2 < n) dst[i + 2] = v4.z;
      }
    }
  }
  __syncthreads();  // the row list, the positions at the ranges' ends
  if (a.scored || last_layer) {  // for the index-list kernel
    if (tid == 0) {
      c->R = R;
      c->scale = hscale;
      c->tbin = tbin;
      c->above = above;
      c->budget = B;
      c->T = T;
      c->idxT = idxT;
    }
    const int per = a.range_tokens / kRangeTokens;
    if (tid * a.range_tokens < n) {
      const uint32_t to = (tid + 1) * a.range_tokens < n ? bound[(tid + 1) * per] : n_sel;
      a.sel_cnt[(size_t)unit * ((max_ctx + a.range_tokens - 1) / a.range_tokens) + tid] = to - bound[tid * per];
    }
  }
  if (a.count_out && tid == 0) a.count_out[unit] = B;

  FIER_PROF_WG(5)
  // ---- 4. attention over the selected rows --------------------------------------------------------------------------------------
  GatherState<NREP> st;
  st.init();
  auto row_of = [&](int j) {
    const int t = (int)rows[j];
    return kv.blocks ? (size_t)lblk[t >> kv.shift] * kv.block_stride + kv.base + (size_t)(t & kv.mask) : kv.base + (size_t)t;
  };
  const uint4* const K4 = reinterpret_cast<const uint4*>(a.K);
  const uint4* const V4 = reinterpret_cast<const uint4*>(a.V);
  if constexpr (NREP >= 3)
    attend_rows_mfma<DT, NREP, false, false, STREAM, NW>(K4, V4, qr, row_of, 0, (int)n_sel, a.scale_log2e, st);
  else
    attend_rows<DT, NREP, false, STREAM, NW>(K4, V4, qr.c, row_of, 0, (int)n_sel, a.scale_log2e, st);
  FIER_PROF_WG(6)
  float* const sh = reinterpret_cast<float*>(arena);
  wave_partials<DT, NREP, kPitch>(st, sh);  // nobody reads the scores any more: a barrier has followed the last read
  __syncthreads();
  // a wavefront folds 64 channels of a head: the wavefronts' weights one per lane
  for (int o0 = wave * 64; o0 < NREP * kD; o0 += NT) {
    const int r = o0 / kD, ch = (o0 + lane) % kD;
    const float* src = sh + r * kPitch;
    const float2 ml = *reinterpret_cast<const float2*>(src + (lane < NW ? lane : 0) * 160 + 8);
    const float ms = lane < NW ? ml.x : -INFINITY;
    const float M = wave_allmax_f(ms);
    const float wgt = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - M);
    const float l = wave_allsum_f(lane < NW ? wgt * ml.y : 0.f);
    float acc = 0.f;
#pragma unroll
    for (int k = 0; k < NW; ++k)
      acc += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wgt), k)) * src[(ch >> 3) * 10 + k * 160 + (ch & 7)];
    a.out[(size_t)unit * NREP * kD + o0 + lane] = l > 0.f ? acc / l : 0.f;
  }
  FIER_PROF_WG(7)
}

// Compiled in parts, FIER_UNIT_PART = 2 (NW == 16) + DT, next to the rest of this file.
template <int DT, int NW>
hipError_t launch_unit_step_dt(const UnitArgs& a, int n_rep, bool stream, const LayerBatch& lb, hipStream_t st) {
  const dim3 grid((unsigned)a.n_kv_heads, (unsigned)lb.n, (unsigned)a.batch);
#define FIER_UNIT_CASE(R)                                                                                 \
  case R:                                                                                                 \
    if (stream) unit_step_kernel<DT, R, NW, true><<<grid, 64 * NW, a.lds.bytes, st>>>(a, lb);             \
    else unit_step_kernel<DT, R, NW, false><<<grid, 64 * NW, a.lds.bytes, st>>>(a, lb);                   \
    break;
  switch (n_rep) {
    FIER_UNIT_CASE(1)
    FIER_UNIT_CASE(2)
    FIER_UNIT_CASE(3)
    FIER_UNIT_CASE(4)
    FIER_UNIT_CASE(5)
    FIER_UNIT_CASE(6)
    FIER_UNIT_CASE(7)
    FIER_UNIT_CASE(8)
    default:
      return hipErrorInvalidValue;
  }
#undef FIER_UNIT_CASE
  return hipGetLastError();
}

#define FIER_UNIT_INSTANCE(WORD, DT, NW) \
  WORD template hipError_t launch_unit_step_dt<DT, NW>(const UnitArgs&, int, bool, const LayerBatch&, hipStream_t);
#ifdef FIER_UNIT_PART
FIER_UNIT_INSTANCE(, FIER_UNIT_PART & 1, (FIER_UNIT_PART >> 1) != 0 ? 16 : 8)
#else
FIER_UNIT_INSTANCE(extern, DT_F16, 8)
FIER_UNIT_INSTANCE(extern, DT_F16, 16)
FIER_UNIT_INSTANCE(extern, DT_BF16, 8)
FIER_UNIT_INSTANCE(extern, DT_BF16, 16)

// Wavefronts per unit where the step of `layers` layers of `units` units takes this kernel, else 0.  It is bound by what one
// CU does with a unit: about 2.4 us per 1000 tokens scored and 110 of them gathered, on top of 7 us, where the two-kernel form
// takes 20 us for small calls whatever the context and is bound by memory for large ones.  us per layer, two kernels / 16
// wavefronts / 8, budget 11 %:
//   8 units       1k 17.2 / 10.0 / 9.4   2k 18.7 / 11.6 / 12.1   4k 19.4 / 15.8 / 19.1   8k 20.2 / 25.0 / 32.6
//   128 units     1k 19.7 / 11.3 / 10.8  2k 22.3 / 15.7 / 16.9   4k 24.8 / 21.8 / 26.1   8k 33.1 / 35.4 / 45.6
//   256, 4 heads  1k 22.8 / 14.0 / 13.4  4k 35.1 / 29.2 / 31.0   8k 52.1 / 45.5 / 51.8   16k 79.8 / 81.9 / 98.0
//   512, 4 heads  1k 29.9 / 27.0 / 17.8  4k 54.9 / 55.8 / 43.6   8k 83.7 / 86.9 / 73.3
//   16 layers of 64 ragged paged units up to 8k, 4 heads  126 / - / 93-95 per call of all 16
// Hence up to 256 workgroups 16 wavefronts, to a number of tokens and rows that grows with the share of the GPU in use; beyond, 8
// wavefronts (two workgroups per CU), with three heads or more to 12000.
//   One or two heads: the gather is on the vector units here, past 64 workgroups a row counts twice (25 % budgets: 128 units x 6.4k 37.8 / 43.7, 104 x
// 5.2k 36.2 / 40.4), and the two-kernel form has five workgroups per CU, so that up to 1280 short units are one round of it where
// this kernel needs two or three.  Of several layers it clears the parts first, so this kernel is worth more there.  Its time over
// that of two kernels, equal contexts, mean / worst of 5 to 570 random shapes each:
//   workgroups                 257-320    -384       -512       -640       -768      -1024      -1280      -1536      -2048      -3072
//   one layer, to 4000         .77/0.99  .77/0.97   .76/0.92  1.03/1.24  1.02/1.16  1.03/1.24  1.14/1.44   .90/0.98  1.01/1.13  1.03/1.13
//     4000 to 8000            1.03/1.12  .94/1.04   .88/1.00  1.13/1.29  1.09/1.18  1.03/1.07  1.07/1.14   .92/0.96  1.00/1.09
//     8000 to 12000           1.15/1.22 1.04/1.12   .97/1.08
//   several layers, to 4000    .65/0.85  .64/0.84   .63/0.88   .86/1.07   .85/1.04   .85/1.00   .97/1.23   .80/0.93   .89/1.03   .95/1.12
//     4000 to 8000             .86/0.98  .81/0.93   .75/0.89   .99/1.14   .95/1.04   .91/1.02  1.00/1.13   .89/0.99   .96/1.05   .97/1.09
//     8000 to 12000            .94/1.09  .89/1.03   .85/0.99
// One layer therefore takes it up to 512 and from 1281 to 1536 workgroups, several up to 1024 and from 1281 to 2048, four and more up
// to 3072 (at 1025 to 1280 and 2049 to 3072, 6039 shapes of 4 / 8 / 16 layers: .92 / .91 / .90, 50 of them more than 1.07, 1.14 at
// worst, half of those 50 with contexts below 300; 184 of 2 / 3 layers: .97 / .95).  Calls that want the index list, another launch
// there, keep the larger limits (66 shapes past these .91, 1.12 at worst).
//   Against the two kernels as they were before this kernel: three heads and more, 4900 random shapes that take it (1 to 8 layers, 1 to
// 2000 units, budgets of 3 to 25 %) .54 to .71 of the time by their number of workgroups, 1 of them more than 1.07 (1.09); one and two
// heads, 5800 shapes past 200 workgroups .785, 14 of them more than 1.07 (1.12 at worst; 283 and 1.32 with the larger limits for all).
int unit_form(int units, int layers, int n_rep, int max_budget, int max_ctx, bool with_index_list) {
  if (max_ctx > kUnitMaxCtx) return 0;
  const int64_t grid = (int64_t)units * layers;
  const int64_t work = n_rep <= 2 && grid > 64 ? (max_ctx + 2 * (int64_t)max_budget) * 10 / 11 : (int64_t)max_ctx + max_budget;
  const int nw = grid <= 256 ? 16 : 8;
  int64_t limit = 12000;
  if (grid <= 64) limit = 5500;
  else if (grid <= 256) limit = 5500 + (grid - 64) * 40;
  else if (n_rep <= 2) {
    const bool filled = grid <= 1024 ? layers > 1 : grid > 1280 && grid <= (layers > 1 ? 2048 : 1536);
    if (with_index_list) limit = grid <= 512 ? 12000 : 8000;
    else if (grid <= 512) limit = layers > 1 ? 8000 + (grid - 256) * 16 : 4000 + (grid - 256) * 31;
    else limit = filled || (layers >= 4 && grid <= 3072) ? 8000 : 0;
  }
  if (work > limit) return 0;
  return unit_lds(nw, n_rep, max_ctx, max_budget).bytes + kUnitFixedLds <= (nw == 16 ? 160u : 80u) * 1024u ? nw : 0;
}

hipError_t launch_unit_step(int nw, int dtype, KvLayout lay, int n_rep, const uint32_t* kbits, const uint32_t* kmeta,
                            float* kabsmax, const void* q, const int32_t* seq_lens, const StepBuffers& sb,
                            const int32_t* budgets, int max_budget, float sm_scale, void* K, void* V, const void* k_new,
                            const void* v_new, float* out, int32_t* idx_out, int32_t* count_out, int batch, int n_kv_heads,
                            int max_ctx, int group_size, int range_tokens, bool scored, const LayerBatch& lb,
                            hipStream_t st) {
  UnitArgs a;
  a.kbits = (const uint4*)kbits;
  a.kmeta = (const uint4*)kmeta;
  a.kabsmax = kabsmax;
  a.K = (uint32_t*)K;
  a.V = (uint32_t*)V;
  a.q = (const uint16_t*)q;
  a.k_new = (const uint32_t*)k_new;
  a.v_new = (const uint32_t*)v_new;
  a.seq_lens = seq_lens;
  a.budgets = budgets;
  a.out = out;
  a.idx_out = idx_out;
  a.count_out = count_out;
  a.ctl = sb.ctl;
  a.hist = sb.hist;
  a.sel_cnt = sb.sel_cnt;
  a.scores = sb.scores;
  a.newmax = sb.newmax;
  a.max_budget = max_budget;
  a.batch = batch;
  a.n_kv_heads = n_kv_heads;
  a.max_ctx = max_ctx;
  a.gshift = group_size == 256 ? 3 : group_size == 128 ? 2 : group_size == 64 ? 1 : 0;
  a.range_tokens = range_tokens;
  a.scale_log2e = sm_scale * 1.4426950408889634f;
  const long grid = (long)batch * n_kv_heads * lb.n;
  a.by_length = batch > 1 && batch <= 64 && grid > 256L * (16 / nw);  // at four wavefronts per SIMD
  a.scored = scored;
  a.lay = lay;
  a.lds = unit_lds(nw, n_rep, max_ctx, max_budget);
  const bool stream = grid * max_budget * (2 * kD * 2) >= (8L << 20);  // as the other gathers
  if (dtype == DT_F16)
    return (nw == 16 ? launch_unit_step_dt<DT_F16, 16> : launch_unit_step_dt<DT_F16, 8>)(a, n_rep, stream, lb, st);
  return (nw == 16 ? launch_unit_step_dt<DT_BF16, 16> : launch_unit_step_dt<DT_BF16, 8>)(a, n_rep, stream, lb, st);
}
#endif  // FIER_UNIT_PART

}  // namespace fier
