// Scores of one pair block (64 tokens) by one wavefront, on the matrix cores (Alg. 1 step 2): shared by the score kernel and
// the kernel that does a unit's whole step.
//   score[j] = sum_c q_c * (z[G(j)][c] + bit[j][c] * s[G(j)][c]),  q = sum of the unit's query heads.
//
// The contraction over the 128 channels runs on the matrix cores as an int8 product
// (v_mfma_i32_16x16x64_i8), one wavefront per pair block (64 tokens = groups 2P and 2P+1) at a time:
//   * B operand = the codes.  A byte with a single bit k set IS the integer 2^k (bit 7: -128), so one v_and of a
//     code word with 0x01010101 << k yields four B elements: 8 vector ops expand 32 codes.  Lane (n, kq) of the
//     wavefront owns word kq of token n of a 16-token tile, which is exactly the B layout (k = 16 kq + 0..15);
//     the words arrive as one 16-byte load per token and are put into that order by four lane-row swaps;
//   * A operand = the weights.  w = q_c s_c (binary32 product), divided by its bit's power of two and turned
//     into a 31-bit fixed-point number relative to the largest |w| of its own group (the scale is a power of
//     two, found per group with a DPP max), then cut into four signed bytes: F = d0 + 2^8 d1 + 2^16 d2 + 2^24 d3.
//     The four digits are four rows of A.  The rows are built once per pair block by the lanes that hold the
//     group's (s, z) and reach the A layout through 1.3 KiB of LDS per wavefront;
//   * the digit rows are read back as two A operands, one with the digits in rows 0-3 / 8-11 and zeros elsewhere
//     for the first tile of each group, one with them in rows 4-7 / 12-15 for the second tile: both tiles of a
//     group accumulate into one 16x16 result that holds tile t in rows 4t..4t+3, the rows lane row t receives.
//     Lane l ends up with the four digit sums of token l of the block, recombines them in binary32 and adds
//     base[G] = sum_c q_c z[G][c];
//   * the integer accumulation is exact; the only rounding is the fixed-point step of the weights,
//     <= 2^(k-1) * 2^-30 * 2 max_c|w_c| per channel, about 4e-6 max|w| in the worst case over 128 channels.
//
// Channel bookkeeping.  Row r = lane / 16 works for group g = r / 2 and channel half h = r % 2; lane n of the row
// loads (s, z) of channels c = 64h + 4n + e, e = 0..3, as one 16-byte request.  Channel c sits in code word
// kq = h + 2(e & 1) at bit i = 2n + (e >> 1), i.e. byte y = i / 8, bit k = i % 8: MFMA j = k / 4, B register
// r = k % 4, contraction index K = 16 kq + 4r + y.
#pragma once

#include "fier_dev.h"
#include "fier_quant_dev.h"

namespace fier {

typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

// LDS image of one wavefront's A operand: [j (K half)][group][digit][64 bytes], a zero row per j, padded so that
// the (group, j) sub-blocks start in different banks.
constexpr int kADigit = 64;
constexpr int kAGroup = 320;
constexpr int kAZeroRow = 576;
constexpr int kAPlane = 672;
constexpr int kAWave = 2 * kAPlane;

__device__ __forceinline__ float wave_allsum(float x) {
  x = row_allsum(x);
  x += __shfl_xor(x, 16, 64);
  x += __shfl_xor(x, 32, 64);
  return x;
}

// value of the lane 16 away (rows 0 <-> 1, 2 <-> 3)
__device__ __forceinline__ float swap_rows(float x) {
  return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(x), 0x401f));  // bit mode: xor 16
}
// max over the 16 lanes of a row of non-negative floats, as unsigned integers (their bit patterns order alike)
template <int N>
__device__ __forceinline__ uint32_t row_ror_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x120 + N, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t row_allmax_u32(uint32_t x) {
  x = max(x, row_ror_u32<8>(x));
  x = max(x, row_ror_u32<4>(x));
  x = max(x, row_ror_u32<2>(x));
  x = max(x, row_ror_u32<1>(x));
  return x;
}

// Scores of tokens an append has just quantized, from their code words: the weights q_c s_c of a token's set bits plus base =
// sum_c q_c z_c.  q0, q1: q_c of channels c = 2 lane, 2 lane + 1.  The 128 bits are added up 16 at a time and these eight sums
// in pairs, the same in both functions: tail_scores8 has a lane per (16 bits, token) of eight tokens, tail_scores a lane per
// (half of the bits, token) of 32.  Bit i of word d is channel 64 (d & 1) + 2 i + (d >> 1).  lds: kTailLds bytes, the wavefront's.
constexpr int kTailPitch = 20;  // floats per 16 weights: eight lanes' reads fall in different banks
constexpr int kTailLds = 8 * kTailPitch * 4 + 8 * 16;
__device__ __forceinline__ float tail_weights(float q0, float q1, const GroupScale& g, float* wl) {
  const int lane = threadIdx.x & 63;
  float* w = wl + (lane >> 4) * kTailPitch + (lane & 15);
  w[0] = q0 * g.sf0;
  w[4 * kTailPitch] = q1 * g.sf1;
  return wave_allsum(fmaf(q1, g.zf1, q0 * g.zf0));
}
__device__ __forceinline__ float tail_sum16(uint32_t bits, const float* w) {
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < 16; i += 4) {
    const float4 w4 = *reinterpret_cast<const float4*>(w + i);
    acc += (bits >> i & 1u) ? w4.x : 0.f;
    acc += (bits >> (i + 1) & 1u) ? w4.y : 0.f;
    acc += (bits >> (i + 2) & 1u) ? w4.z : 0.f;
    acc += (bits >> (i + 3) & 1u) ? w4.w : 0.f;
  }
  return acc;
}
__device__ __forceinline__ float sum_swap32(float x) {
  const u32x2_t s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
// Lane 8 c + t holds token t's word; every lane gets the score of token lane % 8.
__device__ __forceinline__ float tail_scores8(const uint4& mine, int c, float q0, float q1, const GroupScale& g, unsigned char* lds) {
  const int lane = threadIdx.x & 63;
  float* wl = reinterpret_cast<float*>(lds);
  unsigned char* words = lds + 8 * kTailPitch * 4;
  const float base = tail_weights(q0, q1, g, wl);
  if (lane >> 3 == c) reinterpret_cast<uint4*>(words)[lane & 7] = mine;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const uint32_t bits = *reinterpret_cast<const uint16_t*>(words + 16 * (lane & 7) + 2 * (lane >> 3));
  float acc = tail_sum16(bits, wl + (lane >> 3) * kTailPitch);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // reads done before what comes into their place
  acc += row_ror<8>(acc);
  const u32x2_t s = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc), __float_as_uint(acc), false, false);
  return sum_swap32(__uint_as_float(s[0]) + __uint_as_float(s[1])) + base;
}
// Lane 32 half + t holds token t's word; every lane gets the score of token lane % 32.
__device__ __forceinline__ float tail_scores(const uint4& mine, int half, float q0, float q1, const GroupScale& g, unsigned char* lds) {
  const int lane = threadIdx.x & 63;
  float* wl = reinterpret_cast<float*>(lds);
  const float base = tail_weights(q0, q1, g, wl);
  const u32x2_t a = __builtin_amdgcn_permlane32_swap(mine.x, mine.z, false, false);
  const u32x2_t b = __builtin_amdgcn_permlane32_swap(mine.y, mine.w, false, false);
  const uint32_t w0 = half ? a[1] : a[0], w1 = half ? b[1] : b[0];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const float* w = wl + 4 * kTailPitch * (lane >> 5);
  float s0 = tail_sum16(w0, w) + tail_sum16(w0 >> 16, w + kTailPitch);
  asm volatile("" : "+v"(s0));  // a word's weights at a time
  const float s1 = tail_sum16(w1, w + 2 * kTailPitch) + tail_sum16(w1 >> 16, w + 3 * kTailPitch);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // reads done before what comes into their place
  return sum_swap32(s0 + s1) + base;
}

// One wavefront's scorer.  a_lds: its kAWave bytes of LDS.
template <int DT>
struct BlockScorer {
  float qs[4];  // the lane's 4 query channels c = 64 hsel + 4 n + e, summed over the query heads of the unit's kv head
  float qk[4];  // q_c divided by the integer its code bit stands for in B
  int a_wr[4];  // LDS byte offset of digit 0 of channel e
  int a_even, a_odd;
  unsigned char* a_lds;

  __device__ __forceinline__ void init(const float (&q)[4], unsigned char* lds) {
    const int lane = threadIdx.x & 63, row = lane >> 4, n = lane & 15;
    const int gsel = row >> 1;  // the group of the pair block whose (s, z) this row of lanes holds
    const int hsel = row & 1;   // the 64-channel half it holds
    a_lds = lds;
#pragma unroll
    for (int e = 0; e < 4; ++e) qs[e] = q[e];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int kq_c = hsel + 2 * (e & 1);
      const int i_c = 2 * n + (e >> 1);
      const int y = i_c >> 3, k = i_c & 7;
      // 2^-k, negative for k = 7 (a byte with only bit 7 set is -128)
      const float inv_bit = __uint_as_float(((uint32_t)(127 - k) << 23) | (k == 7 ? 0x80000000u : 0u));
      qk[e] = qs[e] * inv_bit;
      a_wr[e] = (k >> 2) * kAPlane + gsel * kAGroup + 16 * kq_c + 4 * (k & 3) + y;
    }
    // Two A operands.  "Even" serves the first tile of each group and carries the digits of the first group in
    // rows 0-3, of the second in rows 8-11; "odd" serves the second tiles with the same digits in rows 4-7 and
    // 12-15; all other rows read the zero row.  The two tiles of a group then accumulate into one 16x16 result
    // that holds tile t in rows 4t..4t+3, the rows lane row t receives.
    if (lane < 32) *reinterpret_cast<uint32_t*>(a_lds + (lane >> 4) * kAPlane + kAZeroRow + 4 * n) = 0u;
    const int a_real = (n >> 3) * kAGroup + (n & 3) * kADigit;
    a_even = ((n & 4) ? kAZeroRow : a_real) + 16 * row;
    a_odd = ((n & 4) ? a_real : kAZeroRow) + 16 * row;
  }

  // w_cur: lane l holds the code word of token l of the block; m_cur: the lane's (s, z) quad, of group gsel, channels c.
  // Returns the score of token l in lane l.
  __device__ __forceinline__ float score(uint32_t (&w_cur)[4], const uint4& m_cur) const {
    const int gsel = (threadIdx.x & 63) >> 5;
    // The B layout wants, in lane (row r, n), word r of the tokens 16 t + n, t = 0..3; the load left word d of
    // token 16 r + n in register d: a 4x4 transpose between register index and lane row, two swap stages.
    {
      const u32x2_t a = __builtin_amdgcn_permlane32_swap(w_cur[0], w_cur[2], false, false);
      const u32x2_t b = __builtin_amdgcn_permlane32_swap(w_cur[1], w_cur[3], false, false);
      const u32x2_t c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
      const u32x2_t d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
      w_cur[0] = c[0];
      w_cur[1] = c[1];
      w_cur[2] = d[0];
      w_cur[3] = d[1];
    }

    // ---- this row's weights -> fixed point relative to the group's largest -> digit rows in LDS ----------
    const uint32_t mw[4] = {m_cur.x, m_cur.y, m_cur.z, m_cur.w};
    float wv[4];
    float basep = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      wv[e] = qk[e] * lo16f<DT>(mw[e]);
      basep += qs[e] * hi16f<DT>(mw[e]);
    }
    uint32_t mx = __float_as_uint(fmaxf(fmaxf(fabsf(wv[0]), fabsf(wv[1])), fmaxf(fabsf(wv[2]), fabsf(wv[3]))));
    mx = row_allmax_u32(mx);
    mx = max(mx, (uint32_t)__builtin_amdgcn_ds_swizzle((int)mx, 0x401f));  // over all 128 channels of the group
    // max|w| < 2^(ex - 126), ex its biased exponent: scale = 2^(156 - ex) keeps |w * scale| < 2^30
    uint32_t exb = mx & 0x7f800000u;
    exb = exb < (29u << 23) ? (29u << 23) : exb;
    const float scale = __uint_as_float(0x8d800000u - exb);      // (283 - ex) << 23
    const float inv_scale = __uint_as_float(exb - (29u << 23));  // 2^(ex - 156); 0 when the group carries nothing
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int F = (int)rintf(wv[e] * scale);
      // signed digits: the bytes of (F + 0x808080) ^ 0x808080, the top one as it is
      const uint32_t X = ((uint32_t)F + 0x00808080u) ^ 0x00808080u;
      unsigned char* dst = a_lds + a_wr[e];
      dst[0] = (unsigned char)X;
      dst[kADigit] = (unsigned char)(X >> 8);
      dst[2 * kADigit] = (unsigned char)(X >> 16);
      dst[3 * kADigit] = (unsigned char)(X >> 24);
    }
    float base = row_allsum(basep);
    base += swap_rows(base);  // every lane of rows 2g, 2g + 1: base of group g
    // the writes above come from other lanes of this same wavefront: LDS operations of a wavefront complete
    // in order, the fences keep the compiler from moving the reads above them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    // ---- 4 tiles x 2 K-halves ----------------------------------------------------------------------------
    const i32x4_t ae0 = *reinterpret_cast<const i32x4_t*>(a_lds + a_even);
    const i32x4_t ae1 = *reinterpret_cast<const i32x4_t*>(a_lds + a_even + kAPlane);
    const i32x4_t ao0 = *reinterpret_cast<const i32x4_t*>(a_lds + a_odd);
    const i32x4_t ao1 = *reinterpret_cast<const i32x4_t*>(a_lds + a_odd + kAPlane);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // reads done before the next block's writes
    i32x4_t acc[2];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      i32x4_t b[2][2];  // [tile of the group][K half]
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          b[u][0][r] = (int)(w_cur[2 * g + u] & (0x01010101u << r));
          b[u][1][r] = (int)(w_cur[2 * g + u] & (0x01010101u << (4 + r)));
        }
      acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ae0, b[0][0], i32x4_t{0, 0, 0, 0}, 0, 0, 0);
      acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ae1, b[0][1], acc[g], 0, 0, 0);
      acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ao0, b[1][0], acc[g], 0, 0, 0);
      acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ao1, b[1][1], acc[g], 0, 0, 0);
    }
    // lane l = 16 row + n is token l of the block: its digit sums are registers 0..3 of its group's result
    const i32x4_t dg = gsel ? acc[1] : acc[0];
    float f = (float)dg[0];
    f = fmaf((float)dg[1], 256.0f, f);
    f = fmaf((float)dg[2], 65536.0f, f);
    f = fmaf((float)dg[3], 16777216.0f, f);
    return fmaf(f, inv_scale, base);
  }
};

}  // namespace fier
