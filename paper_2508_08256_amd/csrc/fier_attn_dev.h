// Device functions of the attention kernels (Alg. 1 step 4): the gather loops over a row list, the per-workgroup
// partial (m, l, o) store and the merge of a unit's partials.  Shared by the stand-alone attention kernel
// (fier_attn.hip) and the fused decode step (fier_step.hip).
#pragma once

#include <type_traits>

#include "fier_dev.h"
#include "fier_kernels.h"

namespace fier {

constexpr int kAttnUnroll = 2;                  // rows per 16-lane row per iteration

// Running softmax state of one 16-lane row of a wavefront, per query head: lane cn holds channels 8cn..8cn+7.
template <int NREP>
struct AttnState {
  float m[NREP], l[NREP], o[NREP][8];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int r = 0; r < NREP; ++r) {
      m[r] = -INFINITY;
      l[r] = 0.f;
#pragma unroll
      for (int c = 0; c < 8; ++c) o[r][c] = 0.f;
    }
  }
};

// A row_of that cannot place an entry (an index outside the cache in a caller's list) returns this; the entry is
// then skipped: it gets no weight.
constexpr size_t kNoRow = ~(size_t)0;



// Attend over entries [start, end) of a row list; row_of(j) gives the row of entry j in the K / V arrays (the
// callers map a token to its row: contiguous, or through the block table), or kNoRow if CHECKED and the entry
// is to be skipped (safe_row is then read in its place and masked).  The workgroup's lane rows (4 per wavefront) take entries round-robin in batches of kAttnUnroll.  Calls may follow each other
// on the same state: the running softmax simply continues.  NW: wavefronts of the workgroup.
template <int DT, int NREP, bool CHECKED = false, bool STREAM = false, int NW = 4, class RowOf>
__device__ __forceinline__ void attend_rows(const uint4* __restrict__ K, const uint4* __restrict__ V,
                                            const uint4 (&qr)[NREP], RowOf row_of, int start, int end,
                                            float scale_log2e, AttnState<NREP>& st, size_t safe_row = 0) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rs = lane >> 4, cn = lane & 15;
  for (int i0 = start + wave * (4 * kAttnUnroll); i0 < end; i0 += NW * 4 * kAttnUnroll) {
    uint4 kk[kAttnUnroll], vv[kAttnUnroll];
    bool valid[kAttnUnroll];
#pragma unroll
    for (int u = 0; u < kAttnUnroll; ++u) {
      const int j = i0 + u * 4 + rs;
      valid[u] = j < end;
      size_t r = row_of(valid[u] ? j : start);
      if (CHECKED) {
        valid[u] = valid[u] && r != kNoRow;
        r = r == kNoRow ? safe_row : r;
      }
      const size_t ro = r * (kD / 8) + cn;
      kk[u] = STREAM ? load_stream(K + ro) : K[ro];
      vv[u] = STREAM ? load_stream(V + ro) : V[ro];
    }
#pragma unroll
    for (int r = 0; r < NREP; ++r) {
      float logit[kAttnUnroll];
      float mx = st.m[r];
#pragma unroll
      for (int u = 0; u < kAttnUnroll; ++u) {
        float d = dot2<DT>(kk[u].x, qr[r].x, 0.f);
        d = dot2<DT>(kk[u].y, qr[r].y, d);
        d = dot2<DT>(kk[u].z, qr[r].z, d);
        d = dot2<DT>(kk[u].w, qr[r].w, d);
        d = row_allsum(d);
        logit[u] = valid[u] ? d * scale_log2e : -INFINITY;
        mx = fmaxf(mx, logit[u]);
      }
      const float mref = mx == -INFINITY ? 0.f : mx;
      const float alpha = __builtin_amdgcn_exp2f(st.m[r] - mref);
      float p[kAttnUnroll], psum = 0.f;
#pragma unroll
      for (int u = 0; u < kAttnUnroll; ++u) {
        p[u] = __builtin_amdgcn_exp2f(logit[u] - mref);
        psum += p[u];
      }
      st.m[r] = mx;
      st.l[r] = st.l[r] * alpha + psum;
#pragma unroll
      for (int c = 0; c < 8; ++c) st.o[r][c] *= alpha;
#pragma unroll
      for (int u = 0; u < kAttnUnroll; ++u) {
        const uint32_t vw[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          st.o[r][2 * c] += p[u] * lo16f<DT>(vw[c]);
          st.o[r][2 * c + 1] += p[u] * hi16f<DT>(vw[c]);
        }
      }
    }
  }
}

typedef float floatx4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

template <int DT>
__device__ __forceinline__ floatx4_t mfma_16x16x32(const uint4& a, const uint4& b, floatx4_t c) {
  if (DT == DT_F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0,
                                                  0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                 0, 0, 0);
}

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((ext_vector_type(4)));
template <int DT>
__device__ __forceinline__ floatx4_t mfma_16x16x16(uint2 a, uint2 b, floatx4_t c) {
  if (DT == DT_F16)
    return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(half4_t, a), __builtin_bit_cast(half4_t, b), c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4_t, a), __builtin_bit_cast(short4_t, b), c, 0, 0, 0);
}

// LDS floats per query head of store_partials: [wave][channel chunk][o[8], m, l].  650 and not 640: the matrix-core
// state's writes of all heads go out together, 16 lanes and a head pitch of a multiple of 64 words would meet in a bank.
constexpr int kPartialFloats = 4 * 16 * 10 + 10;

// ---- three to eight query heads per kv head: both products on the matrix cores -------------------------------------------
// Per wavefront and tile of 16 gathered rows:
//   S = K q^T   (rows = tokens, columns = query heads): four v_mfma_f32_16x16x32.  A = the K rows as they lie in memory
//     (lane (n, kq) loads channels 32c + 8kq .. + 7 of row n), B = the queries.  Lane (n, kq) is left with the logits of
//     tokens 4kq .. 4kq + 3 for column n -- which is the B operand of the second product as it stands;
//   O^T += V^T P^T (rows = channels, columns = heads): eight v_mfma_f32_16x16x16.  Lane (n, kq) loads channels 8n .. 8n + 7
//     of the V rows of tokens 4kq .. 4kq + 3 (a row is 16 lanes, 256 contiguous bytes); the four tokens of one of its
//     channels, two byte permutations, are the lane's A operand of the product over channels 8m + c, m = 0..15.
// So nothing crosses lanes but the maximum over the four lane rows, and each lane keeps 32 of its column's 128 outputs.
// The probabilities are three operands in the V type, p = hi + mid + lo: with bf16 (8 bits each) all 24 bits of p; with fp16 (11 each,
// p scaled by 2^15) all of them down to 2^-16 of the wavefront's running maximum, below that to the format's last place, an error of
// at most 2^-39 of the maximum per row (2^-38 from six heads on).  The 16 columns have room for the parts: column n is part n / kCols of head n % kCols,
// kCols = NREP up to five heads; from six on hi and mid take the columns and lo, half of it each, a second product into the
// same sums.
//   Before, P.V ran on the vector ALUs, 32 V elements and 32 x 4 multiply-adds of each lane per tile and head group behind an
// exchange of p through LDS: about 350 vector instructions per tile at four heads (115 now), 141 to 157 registers at four
// or five heads and 182 to 206 at six to eight, i.e. three or two workgroups per CU instead of four.
template <int NREP>
struct MfmaState {
  static constexpr int kCols = NREP <= 5 ? NREP : 8;
  float m, l;      // running maximum of the lane's column (the same in its four lanes), its own tokens' part of the sum
  floatx4_t o[8];  // o[c][i]: channel 8 (4 kq + i) + c of the lane's column
  __device__ __forceinline__ void init() {
    m = -INFINITY;
    l = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) o[c] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
};

// The running state of a gather and what it needs of the queries, by the number of query heads per kv head.
template <int NREP>
using GatherState = std::conditional_t<(NREP >= 3), MfmaState<NREP>, AttnState<NREP>>;
template <int NREP>
struct GatherQuery {
  uint4 c[NREP >= 3 ? 4 : NREP];
  // q_unit: the unit's NREP query rows
  __device__ __forceinline__ void load(const uint4* __restrict__ q_unit) {
    const int n = threadIdx.x & 15, kq = threadIdx.x >> 4 & 3;
    if constexpr (NREP >= 3) {
      constexpr int kCols = MfmaState<NREP>::kCols;
      const int h = n % kCols;
#pragma unroll
      for (int k = 0; k < 4; ++k) c[k] = q_unit[(size_t)(h < NREP ? h : 0) * (kD / 8) + 4 * k + kq];
    } else {
#pragma unroll
      for (int r = 0; r < NREP; ++r) c[r] = q_unit[(size_t)r * (kD / 8) + n];
    }
  }
};

// The largest value among the four lanes with the same lane % 16.
__device__ __forceinline__ float rows_allmax(float x) {
  typedef unsigned int u2_t __attribute__((ext_vector_type(2)));
  const u2_t a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const u2_t b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// x without its leading bits (mask: those of the part's format), exactly; x for mask 0
__device__ __forceinline__ float drop_part(float x, uint32_t mask) { return x - __uint_as_float(__float_as_uint(x) & mask); }
// Four non-negative values, each cut off to the format's leading bits, as an operand.
template <int DT>
__device__ __forceinline__ uint2 pack_part(const float (&x)[4]) {
  if (DT == DT_F16)  // rounds towards zero
    return make_uint2(__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(x[0], x[1])),
                      __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(x[2], x[3])));
  return make_uint2(__builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]), 0x07060302u),
                    __builtin_amdgcn_perm(__float_as_uint(x[3]), __float_as_uint(x[2]), 0x07060302u));
}

constexpr float kLargeLogit = 0x1p22f;  // below it a logit's rounding error is at most 1/8 and a weight at most 1.1
// As attend_rows, for three to eight query heads per kv head.  STREAM_V: the V rows with the streaming hint (the K rows, which
// are loaded in four pieces per row, keep plain loads in gathers).
template <int DT, int NREP, bool CHECKED = false, bool STREAM = false, bool STREAM_V = STREAM, int NW = 4, class RowOf>
__device__ __forceinline__ void attend_rows_mfma(const uint4* __restrict__ K, const uint4* __restrict__ V,
                                                 const GatherQuery<NREP>& q, RowOf row_of, int start, int end,
                                                 float scale_log2e, MfmaState<NREP>& st, size_t safe_row = 0) {
  static_assert(NREP >= 3 && NREP <= 8, "heads per kv head");
  constexpr int kCols = MfmaState<NREP>::kCols;
  constexpr uint32_t kLead = DT == DT_F16 ? 0xffffe000u : 0xffff0000u;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 15, kq = lane >> 4;
  const int part = n / kCols;
  const uint32_t cut1 = part >= 1 ? kLead : 0u, cut2 = part >= 2 ? kLead : 0u;
  bool large = __ballot(st.m != -INFINITY && fabsf(st.m) >= kLargeLogit) != 0ull;  // some column's maximum
  for (int j0 = start + wave * 16; j0 < end; j0 += NW * 16) {
    uint4 kk[4], vv[4];
    size_t rk = row_of(j0 + n < end ? j0 + n : start);
    if (CHECKED) rk = rk == kNoRow ? safe_row : rk;
    rk *= (kD / 8);
#pragma unroll
    for (int c = 0; c < 4; ++c) kk[c] = STREAM ? load_stream(K + rk + 4 * c + kq) : K[rk + 4 * c + kq];
    bool valid[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int jv = j0 + 4 * kq + u;
      valid[u] = jv < end;
      size_t rv = row_of(valid[u] ? jv : start);
      if (CHECKED) {
        valid[u] = valid[u] && rv != kNoRow;
        rv = rv == kNoRow ? safe_row : rv;
      }
      vv[u] = STREAM_V ? load_stream(V + rv * (kD / 8) + n) : V[rv * (kD / 8) + n];
    }
    floatx4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 4; ++c) s = mfma_16x16x32<DT>(kk[c], q.c[c], s);
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = valid[i] ? s[i] * scale_log2e : -INFINITY;
    const float mx = fmaxf(st.m, rows_allmax(fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3]))));
    const float mref = mx == -INFINITY ? 0.f : mx;
    const float alpha = __builtin_amdgcn_exp2f(st.m - mref);
    if (__ballot(alpha != 1.0f)) {  // the maxima settle after a few tiles
#pragma unroll
      for (int c = 0; c < 8; ++c) st.o[c] *= alpha;
      large = __ballot(fabsf(mref) >= kLargeLogit) != 0ull;
    }
    // The weights take the scaled logit unrounded, which is the more accurate while logits are small: its distance from the
    // rounded maximum then is, for the largest one, that one's rounding error, which from 2^24 on moves the largest weight itself
    // away from 1 by powers of two.  Large logits are rounded as their maximum is: no weight above 1, the largest one 1.
    float e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = fmaf(s[i], scale_log2e, -mref);
    if (__builtin_expect(large, 0)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) e[i] = fabsf(mref) >= kLargeLogit ? p[i] - mref : e[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = valid[i] ? __builtin_amdgcn_exp2f(e[i]) : 0.f;
    st.l = st.l * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
    st.m = mx;
    uint2 pb, pb_lo;
    float lo[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = DT == DT_F16 ? p[i] * 0x1p15f : p[i];  // the small ones stay normal fp16 numbers
      p[i] = drop_part(drop_part(x, cut1), cut2);
      if (kCols == 8) lo[i] = 0.5f * drop_part(drop_part(x, kLead), kLead);
    }
    pb = pack_part<DT>(p);
    if constexpr (kCols == 8) pb_lo = pack_part<DT>(lo);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      auto word = [&](int u) { return c < 2 ? vv[u].x : (c < 4 ? vv[u].y : (c < 6 ? vv[u].z : vv[u].w)); };
      const uint32_t sel = c & 1 ? 0x07060302u : 0x05040100u;
      const uint2 va = make_uint2(__builtin_amdgcn_perm(word(1), word(0), sel), __builtin_amdgcn_perm(word(3), word(2), sel));
      st.o[c] = mfma_16x16x16<DT>(va, pb, st.o[c]);
      if constexpr (kCols == 8) st.o[c] = mfma_16x16x16<DT>(va, pb_lo, st.o[c]);
    }
  }
}

// The sum over the four lanes with the same lane % 16 (lanes 16 apart first), by exchanges between registers: no LDS crossbar.
__device__ __forceinline__ float rows_allsum(float x) {
  typedef unsigned int u2_t __attribute__((ext_vector_type(2)));
  const u2_t a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const u2_t b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// value of lane i + N of the row of 16 lanes (0 past its end)
template <int N>
__device__ __forceinline__ float row_from(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x100 + N, 0xf, 0xf, true));
}

// The wavefront's state into LDS, sh + head * PITCH: [wave][channel chunk of 8][o[8], m, l].
template <int DT, int NREP, int PITCH = kPartialFloats>
__device__ __forceinline__ void wave_partials(const AttnState<NREP>& st, float* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rs = lane >> 4, cn = lane & 15;
#pragma unroll
  for (int r = 0; r < NREP; ++r) {
    const float M = rows_allmax(st.m[r]);
    const float w = st.m[r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(st.m[r] - M);
    const float l = rows_allsum(st.l[r] * w);
    float o[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) o[c] = rows_allsum(st.o[r][c] * w);
    if (rs == 0) {
      float* dst = sh + r * PITCH + (wave * 16 + cn) * 10;
#pragma unroll
      for (int c = 0; c < 8; ++c) dst[c] = o[c];
      dst[8] = M;
      dst[9] = l;
    }
  }
}
template <int DT, int NREP, int PITCH = kPartialFloats>
__device__ __forceinline__ void wave_partials(const MfmaState<NREP>& st, float* sh) {
  constexpr int kCols = MfmaState<NREP>::kCols;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = lane & 15, kq = lane >> 4;
  const float l = rows_allsum(st.l);
  float* dst = sh + n * PITCH + (wave * 16 + 4 * kq) * 10;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float o[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {  // hi + mid + lo
      o[c] = st.o[c][i] + row_from<kCols>(st.o[c][i]);
      if (kCols <= 5) o[c] += row_from<2 * kCols <= 10 ? 2 * kCols : 10>(st.o[c][i]);
      if (DT == DT_F16) o[c] *= 0x1p-15f;
    }
    if (n < NREP) {
#pragma unroll
      for (int c = 0; c < 8; c += 2) *reinterpret_cast<float2*>(dst + i * 10 + c) = make_float2(o[c], o[c + 1]);
      *reinterpret_cast<float2*>(dst + i * 10 + 8) = make_float2(st.m, l);
    }
  }
}

// Combine the wavefronts' states of the workgroup per query head and write one partial (m, l, o[128]) per head into slot
// `slot` of the unit's partial arrays.  A wavefront's lanes are folded first (wave_partials), so that only one state per
// wavefront and head goes through LDS and all heads share one barrier.
// sh: NREP * kPartialFloats floats.  Contains barriers: every thread of the workgroup calls it.
// mark: the slot's l goes out as -(l + 1) (l >= 0, so the sign is free): a workgroup of the step records that way that
// its partial lacks its threshold-bin rows (merge_heads takes such a slot with its true l).
template <int DT, int NREP, bool COHERENT>
__device__ __forceinline__ void store_partials(const GatherState<NREP>& st, float* sh, int unit, int n_slots, int slot,
                                               float* __restrict__ po, float* __restrict__ pm,
                                               float* __restrict__ pl, bool mark = false) {
  const int tid = threadIdx.x;
  __syncthreads();  // sh may still be read as something else by a slower wavefront
  wave_partials<DT, NREP>(st, sh);
  __syncthreads();
  // thread -> (head parity, channel): threads 0..127 take the even heads, 128..255 the odd ones
  const int ch = tid & 127, chunk = ch >> 3, e = ch & 7;
  for (int r = tid >> 7; r < NREP; r += 2) {
    const float* src = sh + r * kPartialFloats + chunk * 10;
    float M = -INFINITY;
#pragma unroll
    for (int wv = 0; wv < 4; ++wv) M = fmaxf(M, src[wv * 160 + 8]);
    float acc = 0.f, lsum = 0.f;
#pragma unroll
    for (int wv = 0; wv < 4; ++wv) {
      const float ms = src[wv * 160 + 8];
      const float w = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - M);
      acc += w * src[wv * 160 + e];
      lsum += w * src[wv * 160 + 9];
    }
    const size_t ps = ((size_t)unit * NREP + r) * n_slots + slot;
    if (COHERENT) {  // read back by another workgroup of this kernel
      store_coherent(&po[ps * kD + ch], acc);
      if (ch == 0) {
        store_coherent(&pm[ps], M);
        store_coherent(&pl[ps], mark ? -(lsum + 1.f) : lsum);
      }
    } else {
      po[ps * kD + ch] = acc;
      if (ch == 0) {
        pm[ps] = M;
        pl[ps] = mark ? -(lsum + 1.f) : lsum;
      }
    }
  }
}

__device__ __forceinline__ float wave_allsum_f(float x) {
  return rows_allsum(row_allsum(x));
}
__device__ __forceinline__ float wave_allmax_f(float x) {
  x = fmaxf(x, row_ror<8>(x));
  x = fmaxf(x, row_ror<4>(x));
  x = fmaxf(x, row_ror<2>(x));
  x = fmaxf(x, row_ror<1>(x));
  return rows_allmax(x);
}

// Merge the partial slots [0, n_used) of all NREP query heads of a unit into out[NREP][128].  256 threads form
// four groups of 64 (thread k of a group owns channels 2k, 2k+1).  Each group folds the slots s = sub, sub + GPH,
// ... of one head with a running maximum, 32 or 40 slots per batch: their (m, l) sit one per lane and reach the other
// lanes as scalars, the independent 8-byte loads of o are in flight together, so that the round trips
// to memory overlap; with fewer than four heads several groups share a head and meet in LDS.
// A slot stored with a mark (l < 0, see store_partials) counts with its true l.
// sh: 4 * 130 floats.  Has barriers.
template <int NREP>
__device__ __forceinline__ void merge_heads(const float* __restrict__ po, const float* __restrict__ pm,
                                            const float* __restrict__ pl, int unit, int n_slots, int n_used,
                                            float* sh, float* __restrict__ out_unit) {
  constexpr int GPH = NREP == 1 ? 4 : (NREP == 2 ? 2 : 1);  // groups per head
  constexpr int BATCH = GPH == 1 ? 40 : 32;                 // slots per batch and group (a 128k context has 33)
  constexpr int HPP = 4 / GPH;                              // heads per pass
  const int tid = threadIdx.x, lane = tid & 63;
  const int k2 = lane * 2, g = tid >> 6;
#pragma unroll 1
  for (int h0 = 0; h0 < NREP; h0 += HPP) {
    const int h = h0 + g / GPH, sub = g % GPH;
    const bool head_ok = h < NREP;  // the same for the whole wavefront
    const size_t base = ((size_t)unit * NREP + (head_ok ? h : 0)) * n_slots;
    float M = -INFINITY, acc0 = 0.f, acc1 = 0.f, lsum = 0.f;
    for (int s0 = sub; s0 < n_used && head_ok; s0 += GPH * BATCH) {
      // (m, l) of the batch's slots live one per lane; every lane loads its two channels of all the slots
      const int sj = s0 + GPH * lane;
      const bool okj = lane < BATCH && sj < n_used;
      const float mj = okj ? load_coherent(&pm[base + sj]) : -INFINITY;
      float lj = okj ? load_coherent(&pl[base + sj]) : 0.f;
      unsigned long long os[BATCH];
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        const int s = s0 + GPH * k;
        os[k] = load_coherent(reinterpret_cast<const unsigned long long*>(&po[(base + (s < n_used ? s : s0)) * kD + k2]));
      }
      if (NREP == 2) __builtin_amdgcn_sched_barrier(0);  // without it 14 registers spill
      lj = lj < 0.f ? -lj - 1.f : lj;
      const float mx = fmaxf(M, wave_allmax_f(mj));
      const float mref = mx == -INFINITY ? 0.f : mx;
      const float alpha = __builtin_amdgcn_exp2f(M - mref);
      const float wj = __builtin_amdgcn_exp2f(mj - mref);  // 0 for an empty slot
      acc0 *= alpha;
      acc1 *= alpha;
      lsum = lsum * alpha + wave_allsum_f(wj * lj);
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wj), k));
        acc0 += w * __uint_as_float((uint32_t)os[k]);
        acc1 += w * __uint_as_float((uint32_t)(os[k] >> 32));
      }
      M = mx;
    }
    __syncthreads();
    sh[g * 130 + k2] = acc0;
    sh[g * 130 + k2 + 1] = acc1;
    if (k2 == 0) {
      sh[g * 130 + 128] = lsum;
      sh[g * 130 + 129] = M;
    }
    __syncthreads();
    for (int o = tid; o < HPP * kD; o += 256) {
      const int hh = o / kD, c = o % kD;
      if (h0 + hh < NREP) {
        float mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < GPH; ++j) mx = fmaxf(mx, sh[(hh * GPH + j) * 130 + 129]);
        const float mref = mx == -INFINITY ? 0.f : mx;
        float l = 0.f, a = 0.f;
#pragma unroll
        for (int j = 0; j < GPH; ++j) {
          const float w = __builtin_amdgcn_exp2f(sh[(hh * GPH + j) * 130 + 129] - mref);
          l += w * sh[(hh * GPH + j) * 130 + 128];
          a += w * sh[(hh * GPH + j) * 130 + c];
        }
        out_unit[(size_t)(h0 + hh) * kD + c] = l > 0.f ? a / l : 0.f;
      }
    }
  }
}

}  // namespace fier
