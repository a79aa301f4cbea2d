// The 1-bit group quantizer as a device function, shared by the bulk quantizer, the append kernel and the
// fused decode step (Alg. 1 step 1; Eq. 5 read as round-to-nearest, Sec. 3.3).
#pragma once

#include <type_traits>

#include "fier_dev.h"
#include "fier_kernels.h"

namespace fier {

// ---- the decision arithmetic, in one place (binary32, no contraction) --------------------------------------------
// z = min (-0 -> +0);  s = RN_dtype(max - z), held at the largest finite value;  bit = 2 * (k - z) >= s.
struct MinMax {  // running min / max of the lane's two channels over the tokens seen so far
  float mn0, mx0, mn1, mx1;
};
template <int DT>
__device__ __forceinline__ void minmax_first(MinMax& m, uint32_t row) {
  m.mn0 = m.mx0 = lo16f<DT>(row);
  m.mn1 = m.mx1 = hi16f<DT>(row);
}
template <int DT>
__device__ __forceinline__ void minmax_update(MinMax& m, uint32_t row, bool present) {
  const float a = lo16f<DT>(row), b = hi16f<DT>(row);
  m.mn0 = (present && a < m.mn0) ? a : m.mn0;
  m.mx0 = (present && a > m.mx0) ? a : m.mx0;
  m.mn1 = (present && b < m.mn1) ? b : m.mn1;
  m.mx1 = (present && b > m.mx1) ? b : m.mx1;
}
struct GroupScale {  // (s, z) of the lane's two channels: stored words and the same as binary32
  uint32_t s0, z0, s1, z1;
  float sf0, zf0, sf1, zf1;
  // max(|z|, |z + s|): the larger reconstruction level in magnitude
  __device__ __forceinline__ float amax0() const { return fmaxf(fabsf(zf0), fabsf(zf0 + sf0)); }
  __device__ __forceinline__ float amax1() const { return fmaxf(fabsf(zf1), fabsf(zf1 + sf1)); }
};
template <int DT>
__device__ __forceinline__ GroupScale group_scale(MinMax m) {
#pragma clang fp contract(off)
  const float cap = DT == DT_F16 ? 65504.0f : 3.3895313892515355e38f;
  if (m.mn0 == 0.0f) m.mn0 = 0.0f;
  if (m.mn1 == 0.0f) m.mn1 = 0.0f;
  float d0 = m.mx0 - m.mn0;
  float d1 = m.mx1 - m.mn1;
  d0 = d0 > cap ? cap : d0;
  d1 = d1 > cap ? cap : d1;
  if (d0 == 0.0f) d0 = 0.0f;
  if (d1 == 0.0f) d1 = 0.0f;
  GroupScale g;
  g.s0 = f2w<DT>(d0), g.s1 = f2w<DT>(d1);
  g.z0 = f2w<DT>(m.mn0), g.z1 = f2w<DT>(m.mn1);
  g.sf0 = w2f<DT>(g.s0), g.sf1 = w2f<DT>(g.s1);
  g.zf0 = w2f<DT>(g.z0), g.zf1 = w2f<DT>(g.z1);
  return g;
}
// f(T), f(T + 1), ... below n, at most N, n the same in every lane: one scalar branch for all that are not there.  (Nested
// and not a loop with an early exit, which the compiler does not always unroll.)
template <int T, int N, class F>
__device__ __forceinline__ void first_rows(int n, F&& f) {
  if constexpr (T < N) {
    if (T < n) {
      f(std::integral_constant<int, T>());
      first_rows<T + 1, N>(n, f);
    }
  }
}

// Code of row t of a group, into lane lane_base + t.
template <int DT>
__device__ __forceinline__ void code_row(uint32_t r, int t, const GroupScale& g, int lane, int lane_base, uint4& mine) {
#pragma clang fp contract(off)
  const float a = lo16f<DT>(r) - g.zf0;
  const float b = hi16f<DT>(r) - g.zf1;
  const bool c0 = a + a >= g.sf0, c1 = b + b >= g.sf1;
  const uint64_t even = __ballot(c0);
  const uint64_t odd = __ballot(c1);
  if (lane == lane_base + t)
    mine = make_uint4((uint32_t)even, (uint32_t)(even >> 32), (uint32_t)odd, (uint32_t)(odd >> 32));
}
// Codes of up to 32 rows (tokens 0..ntok-1 present) under scale g.  Lane lane_base + t receives the 128-bit code word of
// token t in `mine`.  An empty statement that "produces" the next row and `mine`: the next row's compares cannot start before
// this row's ballots have been used up.  Left to itself the compiler makes the ballots of all 32 rows first, and 64 of them
// do not fit the scalar registers (they were spilled to vector lanes and read back).
template <int DT>
__device__ __forceinline__ void code_rows(const uint32_t (&rows)[kG], int ntok, const GroupScale& g, int lane,
                                          int lane_base, uint4& mine) {
  uint32_t r = rows[0];
#pragma unroll
  for (int t = 0; t < kG; ++t) {
    // ntok is the same in every lane: a row that is not there costs one scalar branch
    if (t < ntok) code_row<DT>(r, t, g, lane, lane_base, mine);
    if (t + 1 < kG) {
      r = rows[t + 1];
      asm volatile("" : "+v"(r), "+v"(mine.x), "+v"(mine.y), "+v"(mine.z), "+v"(mine.w));
    }
  }
}

// Quantize one 32-token group (ntok in [1, 32] tokens present) for the lane's two channels.
// rows[t] holds the packed pair (channel 2l in the low half) of token t; entries t >= ntok are ignored.
// Lane lane_base + t receives the 128-bit code word of token t in `mine` (zero for tokens not present):
// x, y = even channels 0..62 / 64..126 (bit i = channel 2i, 64 + 2i), z, w = odd channels likewise.
template <int DT>
__device__ __forceinline__ GroupScale quantize_group(const uint32_t (&rows)[kG], int ntok, int lane, int lane_base,
                                                     uint4& mine) {
  MinMax m;
  minmax_first<DT>(m, rows[0]);
  first_rows<1, kG>(ntok, [&](auto t) { minmax_update<DT>(m, rows[t], true); });
  const GroupScale g = group_scale<DT>(m);
  code_rows<DT>(rows, ntok, g, lane, lane_base, mine);
  return g;
}

// Groups of g = 32 ns tokens, ns in {2, 4, 8}: the group's rows do not fit the registers, so they are read twice
// (min / max, then codes), 32 rows at a time.  row_at(t) returns the packed pair of token t of the group (t < ntok).
// Pass 1 returns the scale; pass 2 is code_rows per 32-token chunk, driven by the caller.
template <int DT, class RowAt>
__device__ __forceinline__ GroupScale long_group_scale(RowAt row_at, int ntok) {
  MinMax m;
  minmax_first<DT>(m, row_at(0));
  for (int c0 = 0; c0 < ntok; c0 += kG) {
    uint32_t rows[kG];
#pragma unroll
    for (int t = 0; t < kG; ++t) rows[t] = row_at(c0 + t < ntok ? c0 + t : 0);
#pragma unroll
    for (int t = 0; t < kG; ++t) minmax_update<DT>(m, rows[t], c0 + t < ntok);
  }
  return group_scale<DT>(m);
}

// kabsmax[u][c] >= |dequantized key| of every token quantized so far: raised with an integer max on the bit
// pattern (non-negative floats order like unsigned integers); a plain read filters most of the atomics.
__device__ __forceinline__ void raise_absmax(float* __restrict__ slot, float a) {
  if (a > *reinterpret_cast<volatile float*>(slot)) atomicMax(reinterpret_cast<unsigned int*>(slot), __float_as_uint(a));
}

// ---- the group an appended row falls in, eight tokens per wavefront ------------------------------------------------------------
// The group's re-quantization is a chain of dependent steps at the start of every decode step, on its critical path (one
// wavefront for the whole group of 32: steps of 8 units x 16k, 4 heads, took 23.7 us with 24 tokens in it and 24.8 with 32, now
// 22.0, where one with a single token takes 21.2): a
// wavefront to every kTailRows tokens (chunk c; N in the functions below), minima and maxima through LDS.  t0: the group's first token, ntok: its tokens
// with the new one, which comes from registers (kn, token ntok - 1: never the row the append writes).
constexpr int kTailRows = 8;
// The rows of the chunk that the cache holds; zeros past them.
template <int N>
__device__ __forceinline__ void tail_load(const uint32_t* __restrict__ K, const KvRows kv, int t0, int ntok, int c, int lane,
                                          uint32_t (&rows)[N]) {
  const uint32_t* src = K + (kv.row(t0) + (size_t)(c * N)) * (kD / 2) + lane;  // a group lies inside one block
#pragma unroll
  for (int t = 0; t < N; ++t) rows[t] = 0;
  first_rows<0, N>(ntok - 1 - c * N, [&](auto t) { rows[t] = src[(size_t)t * (kD / 2)]; });
}
// Its minima and maxima joined to m, the new row with them if it is the chunk's.
template <int DT, int N>
__device__ __forceinline__ void tail_minmax(MinMax& m, const uint32_t (&rows)[N], int ntok, int c, uint32_t kn) {
  const int old = ntok - 1 - c * N;
  first_rows<0, N>(old, [&](auto t) { minmax_update<DT>(m, rows[t], true); });
  if (old >= 0 && old < N) minmax_update<DT>(m, kn, true);
}
// What a wavefront starts from: with 32-token groups the first one from the group's first row, else infinities.
template <int DT, int N>
__device__ __forceinline__ MinMax tail_minmax_start(const uint32_t (&rows)[N], int ntok, int c, uint32_t kn, bool long_group) {
  MinMax m = {INFINITY, -INFINITY, INFINITY, -INFINITY};
  if (!long_group && c == 0) minmax_first<DT>(m, ntok > 1 ? rows[0] : kn);
  return m;
}
// Of all wavefronts, in their order; n of them have stored theirs, 64 a wavefront.
__device__ __forceinline__ MinMax tail_join(const float4* xch, int n, int lane) {
  const float4 f = xch[lane];
  MinMax m = {f.x, f.y, f.z, f.w};
  for (int w = 1; w < n; ++w) {
    const float4 o = xch[w * 64 + lane];
    m.mn0 = o.x < m.mn0 ? o.x : m.mn0;
    m.mx0 = o.y > m.mx0 ? o.y : m.mx0;
    m.mn1 = o.z < m.mn1 ? o.z : m.mn1;
    m.mx1 = o.w > m.mx1 ? o.w : m.mx1;
  }
  return m;
}
// Its codes: lane (N c + t) % 64 receives the code word of token N c + t of the group.
template <int DT, int N>
__device__ __forceinline__ uint4 tail_codes(const uint32_t (&rows)[N], int ntok, int c, uint32_t kn, const GroupScale& g,
                                            int lane) {
  const int old = ntok - 1 - c * N, base = c * N & (kPair - 1);
  uint4 mine = make_uint4(0, 0, 0, 0);
  first_rows<0, N>(old, [&](auto t) {
    uint32_t r = rows[t];  // see code_rows
    asm volatile("" : "+v"(r), "+v"(mine.x), "+v"(mine.y), "+v"(mine.z), "+v"(mine.w));
    code_row<DT>(r, t, g, lane, base, mine);
  });
  if (old >= 0 && old < N) code_row<DT>(kn, old, g, lane, base, mine);
  return mine;
}

// Row L of a unit appended by four wavefronts, 32-token groups (lane = channel pair): the K/V rows written, the group the row
// falls in re-derived from the rows present, its code words and (s, z) stored.  rows: chunk `wave`, from tail_load (which may
// run well before: the loads are the long part of the chain).  xch: 256 float4 in LDS.  Returns the group's scale; mine: the
// code words of the wavefront's tokens in lanes 8 wave ...  Has a barrier.
template <int DT>
__device__ __forceinline__ GroupScale append_row_short(uint32_t* __restrict__ K, uint32_t* __restrict__ V, const KvRows kv,
                                                       uint32_t* __restrict__ kbits, uint32_t* __restrict__ kmeta, int unit,
                                                       int L, int max_ctx, uint32_t kn, uint32_t vn, int lane, int wave,
                                                       const uint32_t (&rows)[kTailRows], float4* xch, uint4& mine) {
  const int n_groups = max_ctx / kG, Gi = L / kG, t0 = Gi * kG, ntok = L - t0 + 1;
  MinMax m = tail_minmax_start<DT>(rows, ntok, wave, kn, false);
  tail_minmax<DT>(m, rows, ntok, wave, kn);
  xch[wave * 64 + lane] = make_float4(m.mn0, m.mx0, m.mn1, m.mx1);
  if (wave == 0) {
    K[kv.row(L) * (kD / 2) + lane] = kn;
    V[kv.row(L) * (kD / 2) + lane] = vn;
  }
  __syncthreads();
  const GroupScale gs = group_scale<DT>(tail_join(xch, 4, lane));
  mine = tail_codes<DT>(rows, ntok, wave, kn, gs, lane);
  const bool opens_pair_block = (Gi & 1) == 0 && ntok == 1;  // its second group holds no token yet
  uint4* bdst = reinterpret_cast<uint4*>(kbits) + (size_t)unit * max_ctx + t0;
  if (lane >> 3 == wave || (opens_pair_block && wave == 0 && lane >= kG)) bdst[lane] = mine;
  if (wave == 0) {
    uint2* mdst = reinterpret_cast<uint2*>(kmeta + ((size_t)unit * n_groups + Gi) * kD) + lane;
    *mdst = make_uint2(gs.s0 | (gs.z0 << 16), gs.s1 | (gs.z1 << 16));
    if (opens_pair_block) mdst[kD / 2] = make_uint2(0, 0);
  }
  return gs;
}

// The same for groups of g = 32 ns tokens (ns in {2, 4, 8}), by a workgroup of four wavefronts: wavefront w takes the
// group's 32-token chunks w and w + 4 (the second one only at g = 256).  Latency bound, a chain of dependent steps at the
// start of every decode step: one wavefront that read the group twice, 32 rows at a time, made the first kernel of the
// step 15.8 us at 16 units x 20k tokens and g = 128, and two such layers per call 42.2 us; this way they take 37.5.
//
// The rows of chunk c of the tail group (t0 its first token, ntok tokens with the new one), zeros past the end.
__device__ __forceinline__ void append_load_chunk(const uint32_t* __restrict__ K, const KvRows kv, int t0, int ntok, int c,
                                                  uint32_t kn, int lane, uint32_t (&rows)[kG]) {
  const uint32_t* src = K + kv.row(t0) * (kD / 2) + lane;  // a group lies inside one block
  const int first = c * kG;
#pragma unroll
  for (int t = 0; t < kG; ++t) {
    // rows before the new one come from memory (never the row the append writes)
    const uint32_t r = first + t < ntok - 1 ? src[(size_t)(first + t) * (kD / 2)] : 0u;
    rows[t] = first + t == ntok - 1 ? kn : r;
  }
}

// rows: chunk `wave`, from append_load_chunk.  xch: 256 float4 in LDS.  Every pair block of the group that holds a token
// gets its code words rewritten; on_chunk(c, mine, gs) is called for each of the wavefront's chunks that holds a token,
// `mine` the code word of token t0 + 64 (c >> 1) + lane in the lanes of the chunk's half.  Called by all four wavefronts.
template <int DT, class OnChunk>
__device__ __forceinline__ GroupScale append_row_long(uint32_t* __restrict__ K, uint32_t* __restrict__ V,
                                                      const KvRows kv, uint32_t* __restrict__ kbits,
                                                      uint32_t* __restrict__ kmeta, int unit, int L, int max_ctx, int ns,
                                                      uint32_t kn, uint32_t vn, int lane, int wave,
                                                      uint32_t (&rows)[kG], float4* xch, OnChunk on_chunk) {
  const int g = kG * ns;
  const int n_groups = max_ctx / g;
  const int Gi = L / g, t0 = Gi * g, ntok = L - t0 + 1;
  if (wave == 0) {
    K[kv.row(L) * (kD / 2) + lane] = kn;
    V[kv.row(L) * (kD / 2) + lane] = vn;
  }
  // the number of tokens is the same in every lane: a row that is not there costs a scalar branch
  MinMax m = {INFINITY, -INFINITY, INFINITY, -INFINITY};
  const int n_first = ntok - wave * kG;
#pragma unroll
  for (int t = 0; t < kG; ++t)
    if (t < n_first) minmax_update<DT>(m, rows[t], true);
  const int n_second = ntok - (wave + 4) * kG;
  if (n_second > 0) {  // eight at a time: they are read again to be coded, the registers hold the first chunk
    const uint32_t* src = K + kv.row(t0) * (kD / 2) + lane;
    const int first = (wave + 4) * kG;
#pragma unroll 1
    for (int t1 = 0; t1 < kG; t1 += 8) {
      uint32_t r[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) r[t] = first + t1 + t < ntok - 1 ? src[(size_t)(first + t1 + t) * (kD / 2)] : kn;
#pragma unroll
      for (int t = 0; t < 8; ++t) minmax_update<DT>(m, r[t], true);  // past the end: the new row once more
    }
  }
  xch[wave * 64 + lane] = make_float4(m.mn0, m.mx0, m.mn1, m.mx1);
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float4 o = xch[w * 64 + lane];
    m.mn0 = fminf(m.mn0, o.x), m.mx0 = fmaxf(m.mx0, o.y), m.mn1 = fminf(m.mn1, o.z), m.mx1 = fmaxf(m.mx1, o.w);
  }
  const GroupScale gs = group_scale<DT>(m);
  if (wave == 0) {
    uint2* mdst = reinterpret_cast<uint2*>(kmeta + ((size_t)unit * n_groups + Gi) * kD) + lane;
    *mdst = make_uint2(gs.s0 | (gs.z0 << 16), gs.s1 | (gs.z1 << 16));
  }
  uint4* bdst = reinterpret_cast<uint4*>(kbits) + (size_t)unit * max_ctx + t0;
#pragma unroll 1
  for (int c = wave;;) {
    int nt = ntok - c * kG;
    nt = nt > kG ? kG : nt;
    uint4 mine = make_uint4(0, 0, 0, 0);
    // Where the lane stands in the chunk, unknown to the compiler: it made the 32 row numbers and the 32 masks of lanes before the
    // loop, 32 vector registers and 64 scalar ones, which spilled into a 97th vector register (score kernel, two to six heads).
    int at = lane - (c & 1) * kG;
    asm volatile("" : "+v"(at));
    code_rows<DT>(rows, nt, gs, at, 0, mine);
    if (c < ns && (c >> 1) * kPair < ntok && lane >> 5 == (c & 1)) bdst[(c >> 1) * kPair + lane] = mine;
    if (nt > 0) on_chunk(c, mine, gs);
    c += 4;
    if (c >= ns) break;
    append_load_chunk(K, kv, t0, ntok, c, kn, lane, rows);
  }
  return gs;
}

}  // namespace fier
