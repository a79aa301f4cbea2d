// 1-bit group quantizer of the key cache (Alg. 1 step 1; Eq. 5 read as round-to-nearest, Sec. 3.3)
// and the decode-stage append of Sec. 3.1.
//
// The packed layout is token-major (16 bytes per token) while min / max run along the tokens of a channel.  The bulk
// kernel keeps a pair block (64 tokens) in one wavefront's registers, 16 bytes = 8 channels of one token per lane and
// load; the tail and append kernels, one wavefront per unit, hold a channel pair per lane and transpose by ballots.
//
// The decision arithmetic is fixed so that any implementation of the same definition produces the
// same bits:  z = min (an input value, -0 -> +0);  s = RN_dtype(f32(max) - f32(z)), held at the
// largest finite value;  bit = 2*(f32(k) - f32(z)) >= f32(s);  all in binary32, no contraction.
#include "fier_dev.h"
#include "fier_kernels.h"
#include "fier_quant_dev.h"

#pragma clang fp contract(off)

namespace fier {

typedef short short2_t __attribute__((ext_vector_type(2)));

// Both 16-bit floats of a word as signed integers that order like the floats (sign-magnitude -> two's
// complement; the map is its own inverse).  Minimum and maximum of finite values can then be taken two channels
// at a time with packed integer instructions, for fp16 and bf16 alike; -0 sorts below +0, which the
// canonicalisation of zeros in group_scale makes immaterial.
__device__ __forceinline__ short2_t order_keys(uint32_t pair) {
  const short2_t v = __builtin_bit_cast(short2_t, pair);
  return v ^ ((v >> 15) & (short)0x7fff);
}

// One wavefront, g = 32: the unit's last pair block when it is partial (1 to 63 tokens present).
template <int DT>
__device__ __forceinline__ void quantize_tail_short(const uint32_t* __restrict__ K, uint32_t* __restrict__ kbits,
                                                    uint32_t* __restrict__ kmeta, float* __restrict__ kabsmax,
                                                    const int32_t* __restrict__ seq_lens, int n_kv_heads, int max_ctx,
                                                    const KvLayout& lay, const int unit, const int lane) {
  int L = seq_lens[unit / n_kv_heads];
  L = L < 0 ? 0 : (L > max_ctx ? max_ctx : L);
  const int P = L / kPair;
  if (P * kPair >= L) return;
  const int n_groups = max_ctx / kG;
  uint4 mine = make_uint4(0, 0, 0, 0);
  float amax0 = 0.f, amax1 = 0.f;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int t0 = P * kPair + h * kG;
    int ntok = L - t0;
    ntok = ntok > kG ? kG : ntok;
    uint32_t meta0 = 0, meta1 = 0;
    if (ntok > 0) {
      uint32_t rows[kG];
      const uint32_t* src = K + lay.rows_of(unit).row(t0) * (kD / 2) + lane;
#pragma unroll
      for (int t = 0; t < kG; ++t) rows[t] = src[(size_t)(t < ntok ? t : 0) * (kD / 2)];
      const GroupScale gs = quantize_group<DT>(rows, ntok, lane, h * kG, mine);
      meta0 = gs.s0 | (gs.z0 << 16);
      meta1 = gs.s1 | (gs.z1 << 16);
      amax0 = fmaxf(amax0, gs.amax0());
      amax1 = fmaxf(amax1, gs.amax1());
    }
    uint2* mdst = reinterpret_cast<uint2*>(kmeta + ((size_t)unit * n_groups + 2 * P + h) * kD) + lane;
    *mdst = make_uint2(meta0, meta1);
  }
  reinterpret_cast<uint4*>(kbits)[(size_t)unit * max_ctx + P * kPair + lane] = mine;
  raise_absmax(kabsmax + (size_t)unit * kD + 2 * lane, amax0);
  raise_absmax(kabsmax + (size_t)unit * kD + 2 * lane + 1, amax1);
}

// One wavefront, g = 32 ns with ns in {2, 4, 8}: the unit's last group when it is partial.  Its rows are read twice
// (min / max, then codes), 32 at a time.
template <int DT>
__device__ __forceinline__ void quantize_tail_long(const uint32_t* __restrict__ K, uint32_t* __restrict__ kbits,
                                                   uint32_t* __restrict__ kmeta, float* __restrict__ kabsmax,
                                                   const int32_t* __restrict__ seq_lens, int n_kv_heads, int max_ctx,
                                                   int ns, const KvLayout& lay, const int unit, const int lane) {
  const int g = kG * ns;
  int L = seq_lens[unit / n_kv_heads];
  L = L < 0 ? 0 : (L > max_ctx ? max_ctx : L);
  const int Gi = L / g;
  const int t0 = Gi * g;
  if (t0 >= L) return;
  const int ntok = L - t0;
  const int n_groups = max_ctx / g;
  const uint32_t* src = K + lay.rows_of(unit).row(t0) * (kD / 2) + lane;
  auto row_at = [&](int t) { return src[(size_t)t * (kD / 2)]; };
  const GroupScale gs = long_group_scale<DT>(row_at, ntok);
  uint2* mdst = reinterpret_cast<uint2*>(kmeta + ((size_t)unit * n_groups + Gi) * kD) + lane;
  *mdst = make_uint2(gs.s0 | (gs.z0 << 16), gs.s1 | (gs.z1 << 16));
  for (int pb = 0; pb * kPair < ntok; ++pb) {
    uint4 mine = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c0 = pb * kPair + h * kG;
      int nt = ntok - c0;
      nt = nt > kG ? kG : nt;
      if (nt > 0) {
        uint32_t rows[kG];
#pragma unroll
        for (int t = 0; t < kG; ++t) rows[t] = row_at(c0 + t < ntok ? c0 + t : 0);
        code_rows<DT>(rows, nt, gs, lane, h * kG, mine);
      }
    }
    reinterpret_cast<uint4*>(kbits)[(size_t)unit * max_ctx + t0 + pb * kPair + lane] = mine;
  }
  raise_absmax(kabsmax + (size_t)unit * kD + 2 * lane, gs.amax0());
  raise_absmax(kabsmax + (size_t)unit * kD + 2 * lane + 1, gs.amax1());
}

template <int DT, int NS>
__device__ __forceinline__ void quantize_tail(const uint32_t* __restrict__ K, uint32_t* __restrict__ kbits,
                                              uint32_t* __restrict__ kmeta, float* __restrict__ kabsmax,
                                              const int32_t* __restrict__ seq_lens, int n_kv_heads, int max_ctx,
                                              const KvLayout& lay, const int unit, const int lane) {
  if constexpr (NS == 1)
    quantize_tail_short<DT>(K, kbits, kmeta, kabsmax, seq_lens, n_kv_heads, max_ctx, lay, unit, lane);
  else
    quantize_tail_long<DT>(K, kbits, kmeta, kabsmax, seq_lens, n_kv_heads, max_ctx, NS, lay, unit, lane);
}

// The same word by word for one 16-bit float; keys order like the floats, -0 (key -1) just below +0 (key 0).
__device__ __forceinline__ int order_key(uint32_t w16) {
  const int v = (int)(int16_t)w16;
  return v ^ ((v >> 15) & 0x7fff);
}
__device__ __forceinline__ uint32_t key_word(int key) { return (uint32_t)(key ^ ((key >> 15) & 0x7fff)) & 0xffffu; }

// The decision "bit = 2 (k - z) >= s" as a threshold on k.  Its left side, two binary32 operations, never falls as k
// grows, so the 16-bit values that get a 1 are those from some smallest one on: its key is returned.  It is the first
// 16-bit value at or above the midpoint z + s / 2 unless a binary32 rounding moves a neighbour across; that is checked
// with the definition itself, and where it fails (never seen on real data; e.g. bf16 values 2^-30 around a midpoint at
// 0) the threshold is searched for.
template <int DT>
__device__ __forceinline__ int code_threshold(float z, float s) {
#pragma clang fp contract(off)
  auto one = [&](int key) {
    const float d = w2f<DT>(key_word(key)) - z;
    return d + d >= s;
  };
  const float mid = z + 0.5f * s;
  const uint32_t w = f2w<DT>(mid);
  int key = order_key(w);
  key += w2f<DT>(w) < mid ? 1 : 0;
  key = key == 0 ? -1 : key;  // -0 equals +0
  const bool good = one(key) && !one(key - 1);
  if (__any(!good)) {
    constexpr int kMaxKey = DT == DT_F16 ? 0x7bff : 0x7f7f;  // the largest finite value: it gets a 1
    int lo = ~kMaxKey - 1, hi = kMaxKey;                     // below the lowest finite value; that one has key ~kMaxKey
#pragma unroll 1
    for (int i = 0; i < 16; ++i) {  // fewer than 2^16 values in between
      const int m = (lo + hi) >> 1;
      const bool move = hi - lo > 1;
      const bool o = one(m);
      hi = move && o ? m : hi;
      lo = move && !o ? m : lo;
    }
    key = good ? key : hi;
  }
  return key;
}

// What the coding pass needs of a row's dword: operands of min / max, and a word whose sign bits say "below threshold".
// fp16: the packed half-precision instructions on the values themselves (exact: a min / max picks an input, and a sum
// rounds to a value of the exact sum's sign, denormals included).  bf16 has none: integer ones on the ordered keys.
//   min / max go down a lane's tokens; for fp16 they are written as the instruction, because the builtin adds a quieting
// of signalling NaNs to every operand.  The compiler does not count such a statement as a vector instruction when it
// places the two wait states that a permlane swap needs after a write of its operands: settle() goes between the two, and
// the minima and maxima between swaps (cross_min / cross_max) are the builtin.
template <int DT>
struct Pair16 {
  static __device__ __forceinline__ uint32_t prepare(uint32_t w) {
    return DT == DT_F16 ? w : __builtin_bit_cast(uint32_t, order_keys(w));
  }
  static __device__ __forceinline__ uint32_t words(uint32_t p) { return prepare(p); }  // the map is its own inverse
  static __device__ __forceinline__ uint32_t min(uint32_t a, uint32_t b) {
    if constexpr (DT == DT_F16) {
      uint32_t d;
      asm("v_pk_min_f16 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
      return d;
    } else {
      return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(short2_t, a), __builtin_bit_cast(short2_t, b)));
    }
  }
  static __device__ __forceinline__ uint32_t max(uint32_t a, uint32_t b) {
    if constexpr (DT == DT_F16) {
      uint32_t d;
      asm("v_pk_max_f16 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
      return d;
    } else {
      return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(short2_t, a), __builtin_bit_cast(short2_t, b)));
    }
  }
  static __device__ __forceinline__ void settle(uint32_t (&mn)[4], uint32_t (&mx)[4]) {
    if constexpr (DT == DT_F16)
      asm volatile("s_nop 1" : "+v"(mn[0]), "+v"(mn[1]), "+v"(mn[2]), "+v"(mn[3]), "+v"(mx[0]), "+v"(mx[1]), "+v"(mx[2]), "+v"(mx[3]));
  }
  static __device__ __forceinline__ uint32_t cross_min(uint32_t a, uint32_t b) {
    if constexpr (DT == DT_F16)
      return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(half2_t, a), __builtin_bit_cast(half2_t, b)));
    else
      return min(a, b);
  }
  static __device__ __forceinline__ uint32_t cross_max(uint32_t a, uint32_t b) {
    if constexpr (DT == DT_F16)
      return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(half2_t, a), __builtin_bit_cast(half2_t, b)));
    else
      return max(a, b);
  }
  // fp16: the negated threshold, +0 for a threshold of -0 (then -0 and +0 both add up to +0: not below); bf16: its key
  static __device__ __forceinline__ uint32_t threshold(float z0, float s0, float z1, float s1) {
    const int k0 = code_threshold<DT>(z0, s0), k1 = code_threshold<DT>(z1, s1);
    if constexpr (DT == DT_F16)
      return (key_word(k0) | key_word(k1) << 16) ^ 0x80008000u;
    else
      return ((uint32_t)k0 & 0xffffu) | (uint32_t)k1 << 16;
  }
  static __device__ __forceinline__ uint32_t below(uint32_t p, uint32_t thr) {  // sign bits of the halves
    if constexpr (DT == DT_F16)
      return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, p) + __builtin_bit_cast(half2_t, thr));
    else
      return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(short2_t, p), __builtin_bit_cast(short2_t, thr)));
  }
};

typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
// Lane rows of 16.  swap16: {rows a0 b0 a2 b2, rows a1 b1 a3 b3}; swap32: {rows a0 a1 b0 b1, rows a2 a3 b2 b3}.
__device__ __forceinline__ u32x2_t swap16(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_permlane16_swap(a, b, false, false);
}
__device__ __forceinline__ u32x2_t swap32(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_permlane32_swap(a, b, false, false);
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}
// v: nibble t belongs to token t.  Returns, in lane m of each 8 lanes, token m's nibbles of all 8 lanes, lane order.
__device__ __forceinline__ uint32_t transpose_nibbles(uint32_t v, uint32_t sel4, uint32_t sel2, uint32_t rot1, uint32_t keep1) {
  uint32_t o = dpp_u32<0x1b>(dpp_u32<0x141>(v));  // lane ^ 4 = (lane ^ 7) ^ 3: half-row mirror, quad reversal
  v = __builtin_amdgcn_perm(o, v, sel4);          // halves
  o = dpp_u32<0x4e>(v);                           // lane ^ 2
  v = __builtin_amdgcn_perm(o, v, sel2);          // bytes
  o = dpp_u32<0xb1>(v);                           // lane ^ 1
  o = __builtin_amdgcn_alignbit(o, o, rot1);      // nibbles
  return (v & keep1) | (o & ~keep1);
}

// Whole groups, and the partial one at a unit's end.  Grid units * (1 + n_x), n_x >= ceil(n_pairs / (4 bpw)), block 256.
// The first `units` workgroups do the units' partial groups (one wavefront, the longest chain of dependent loads:
// started last it would end the kernel late, and as a kernel of its own it took 4 to 17 us after this one); then wave w
// of workgroup x of a unit owns the pair blocks 4 bpw x + w, + 4, + 8, ...; NS = group size / 32.
//   A pair block sits in 64 registers: load i of lane (row r, n) brings channels 8n .. 8n + 7 of token 16 r + i.  Minima
// and maxima are taken two channels per instruction, first down the lane's 16 tokens, then across the lane rows that
// share a group (NS = 1: rows 0, 1 and rows 2, 3; else all four; NS = 4, 8: also across the 2 / 4 neighbouring
// wavefronts of the group, through LDS, one barrier per block -- every row is read exactly once).  Each exchange halves
// the channels a lane looks after, so the scales are computed once per group and channel.  The bit is the sign of
// (value - threshold), see code_threshold; 16 tokens' signs make four registers, and a transposition of nibbles over 8
// lanes leaves every lane with the code word of its own token: one coalesced 1 KiB store.  As soon as a row has been
// coded its registers receive the row of the wave's next block.
//   What bounds it: HBM, 302 MB in 57 us (5.3 TB/s) at 32 units x 32k tokens.  The version before, which held a channel
// pair per lane and made each row's two ballots into a code word, took 71 us there, 50 of them the issue of 27 vector
// instructions per row; this one issues 9 (fp16) and 12 (bf16).  32 x 128k: 284 -> 230 us; 32 ragged units up to 24k at
// g = 128: 74 -> 35.  128 registers keep four workgroups on a CU.
template <int DT, int NS>
__global__ __launch_bounds__(256, 4) void quantize_kernel(const uint32_t* __restrict__ K, uint32_t* __restrict__ kbits,
                                                       uint32_t* __restrict__ kmeta, float* __restrict__ kabsmax,
                                                       const int32_t* __restrict__ seq_lens, int units, int n_kv_heads,
                                                       int max_ctx, int bpw, int n_x, KvLayout lay) {
  using P16 = Pair16<DT>;
  constexpr int kWavesPerGroup = NS >= 4 ? NS / 2 : 1;
  __shared__ uint2 xch[2][4][64];  // [iteration parity][wavefront][lane]: packed (min, max), NS >= 4 only
  const int lane = threadIdx.x & 63;
  // the wavefront's number as a scalar: everything derived from it (addresses, branches) is then uniform for the
  // compiler too
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if ((int)blockIdx.x < units) {
    if (wave == 0) quantize_tail<DT, NS>(K, kbits, kmeta, kabsmax, seq_lens, n_kv_heads, max_ctx, lay, (int)blockIdx.x, lane);
    return;
  }
  const int wid = (int)blockIdx.x - units;
  const int unit = wid / n_x;
  const int base = (wid - unit * n_x) * (4 * bpw);
  int L = seq_lens[unit / n_kv_heads];
  L = L < 0 ? 0 : (L > max_ctx ? max_ctx : L);
  // pair blocks that consist of whole groups
  const int n_full = NS == 1 ? L / kPair : (L / (kG * NS)) * (NS / 2);
  if (base >= n_full) return;
  const int n_groups = max_ctx / (kG * NS);
  const KvRows kv = lay.rows_of(unit);
  const int r = lane >> 4, n = lane & 15;
  // row i of the lane: uniform block address + the lane's offset + 256 i
  const char* const K1 = reinterpret_cast<const char*>(K);
  uint32_t voff = (uint32_t)(16 * r * kD * 2 + 16 * n);
  auto row_at = [&](const char* block, int i) {
    return load_stream(reinterpret_cast<const uint4*>(block + voff + i * (kD * 2)));
  };
  const uint32_t sel4 = (lane & 4) ? 0x03020706u : 0x05040100u;  // byte selectors: 0-3 own, 4-7 the other lane's
  const uint32_t sel2 = (lane & 2) ? 0x03070105u : 0x06020400u;
  const uint32_t rot1 = (lane & 1) ? 4u : 28u, keep1 = (lane & 1) ? 0xf0f0f0f0u : 0x0f0f0f0fu;
  const bool upper = (lane & 8) != 0;
  uint4 rows[16];
  if (base + wave < n_full) {
    const char* const block = K1 + kv.row((base + wave) * kPair) * (kD * 2);
#pragma unroll
    for (int i = 0; i < 16; ++i) rows[i] = row_at(block, i);
  }
  float amax[4] = {0.f, 0.f, 0.f, 0.f};
  for (int it = 0; it < bpw; ++it) {
    if (base + 4 * it >= n_full) break;  // the same for the whole workgroup
    const int P = base + 4 * it + wave;
    const bool active = P < n_full;  // the wavefronts of one group are active together
    uint32_t mn[4], mx[4];
    if (active) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        rows[i] = make_uint4(P16::prepare(rows[i].x), P16::prepare(rows[i].y), P16::prepare(rows[i].z), P16::prepare(rows[i].w));
        const uint32_t v[4] = {rows[i].x, rows[i].y, rows[i].z, rows[i].w};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          mn[w] = i ? P16::min(mn[w], v[w]) : v[w];
          mx[w] = i ? P16::max(mx[w], v[w]) : v[w];
        }
      }
      P16::settle(mn, mx);
      // rows 0 | 1 and 2 | 3 together: even rows keep the lane's dwords 0, 1, odd rows dwords 2, 3
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const u32x2_t a = swap16(mn[w], mn[w + 2]), b = swap16(mx[w], mx[w + 2]);
        mn[w] = P16::cross_min(a[0], a[1]);
        mx[w] = P16::cross_max(b[0], b[1]);
      }
      if constexpr (NS >= 2) {  // all four rows: rows 0, 1 keep the first of these, rows 2, 3 the second
        const u32x2_t a = swap32(mn[0], mn[1]), b = swap32(mx[0], mx[1]);
        mn[0] = P16::cross_min(a[0], a[1]);
        mx[0] = P16::cross_max(b[0], b[1]);
      }
    }
    if constexpr (NS >= 4) {
      if (active) xch[it & 1][wave][lane] = make_uint2(mn[0], mx[0]);
      __syncthreads();  // the buffer of the other parity is rewritten only after the next barrier
      if (active) {
        const int first = wave & ~(kWavesPerGroup - 1);
#pragma unroll
        for (int k = 1; k < kWavesPerGroup; ++k) {
          const uint2 o = xch[it & 1][first + ((wave + k) & (kWavesPerGroup - 1))][lane];
          mn[0] = P16::cross_min(mn[0], o.x);
          mx[0] = P16::cross_max(mx[0], o.y);
        }
      }
    }
    if (!active) continue;
    // (s, z) and threshold of the channel pairs this lane looks after
    constexpr int kOwn = NS == 1 ? 2 : 1;
    uint32_t thr_own[kOwn], meta[2 * kOwn];
#pragma unroll
    for (int w = 0; w < kOwn; ++w) {
      const uint32_t mnw = P16::words(mn[w]), mxw = P16::words(mx[w]);
      MinMax m;
      m.mn0 = lo16f<DT>(mnw), m.mn1 = hi16f<DT>(mnw);
      m.mx0 = lo16f<DT>(mxw), m.mx1 = hi16f<DT>(mxw);
      const GroupScale g = group_scale<DT>(m);
      meta[2 * w] = g.s0 | (g.z0 << 16);
      meta[2 * w + 1] = g.s1 | (g.z1 << 16);
      amax[2 * w] = fmaxf(amax[2 * w], fmaxf(fabsf(g.zf0), fabsf(g.zf0 + g.sf0)));
      amax[2 * w + 1] = fmaxf(amax[2 * w + 1], fmaxf(fabsf(g.zf1), fabsf(g.zf1 + g.sf1)));
      thr_own[w] = P16::threshold(g.zf0, g.sf0, g.zf1, g.sf1);
    }
    // ... back to all lanes of the group
    uint32_t thr[4];
    {
      u32x2_t half;  // dwords 0 | 2 and 1 | 3 by row parity
      if constexpr (NS == 1)
        half = u32x2_t{thr_own[0], thr_own[1]};
      else
        half = swap32(thr_own[0], thr_own[0]);
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        const u32x2_t t = swap16(half[w], half[w]);
        thr[w] = t[0];
        thr[w + 2] = t[1];
      }
    }
    // codes; the row's registers then take the row of the wave's next block
    const bool more = it + 1 < bpw && P + 4 < n_full;
    const char* const block = K1 + kv.row((more ? P + 4 : P) * kPair) * (kD * 2);
    uint32_t acc[4];  // 4 tokens each: nibble t of the low (high) half = the even (odd) channels' signs of token t
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[j] = 0;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const uint4 v = rows[4 * j + t];
        const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));
          acc[j] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(ushort2_t, acc[j]) >> (unsigned short)1);
          acc[j] |= P16::below(d[w], thr[w]) & 0x80008000u;
        }
      }
      // An empty statement that "produces" the offset from the finished signs: these loads cannot start before the rows
      // whose registers they take have been used up (hoisted, they doubled the registers: 182 instead of 128).
      asm volatile("" : "+v"(acc[j]), "+v"(voff));
      if (more) {
#pragma unroll
        for (int t = 0; t < 4; ++t) rows[4 * j + t] = row_at(block, 4 * j + t);
      }
    }
    // even / odd nibbles of tokens 0-7 and 8-15, transposed over the 8 lanes of a channel half
    const uint32_t e0 = transpose_nibbles(~__builtin_amdgcn_perm(acc[1], acc[0], 0x05040100u), sel4, sel2, rot1, keep1);
    const uint32_t o0 = transpose_nibbles(~__builtin_amdgcn_perm(acc[1], acc[0], 0x07060302u), sel4, sel2, rot1, keep1);
    const uint32_t e1 = transpose_nibbles(~__builtin_amdgcn_perm(acc[3], acc[2], 0x05040100u), sel4, sel2, rot1, keep1);
    const uint32_t o1 = transpose_nibbles(~__builtin_amdgcn_perm(acc[3], acc[2], 0x07060302u), sel4, sel2, rot1, keep1);
    // lanes 0-7 of a row hold the lower 64 channels of tokens 0-7 and 8-15, lanes 8-15 the upper ones: each keeps the
    // token of its own number and sends the other
    const uint32_t re = dpp_u32<0x128>(upper ? e0 : e1), ro = dpp_u32<0x128>(upper ? o0 : o1);  // lane ^ 8
    reinterpret_cast<uint4*>(kbits)[(size_t)unit * max_ctx + P * kPair + lane] =
        make_uint4(upper ? re : e0, upper ? e1 : re, upper ? ro : o0, upper ? o1 : ro);
    if constexpr (NS == 1) {
      uint4* mdst = reinterpret_cast<uint4*>(kmeta + ((size_t)unit * n_groups + 2 * P + (r >> 1)) * kD + 8 * n + 4 * (r & 1));
      *mdst = make_uint4(meta[0], meta[1], meta[2], meta[3]);
    } else if ((P & (kWavesPerGroup - 1)) == 0) {  // the group's first wavefront
      uint2* mdst = reinterpret_cast<uint2*>(kmeta + ((size_t)unit * n_groups + P / (NS / 2)) * kD + 8 * n + 4 * (r & 1) + 2 * (r >> 1));
      *mdst = make_uint2(meta[0], meta[1]);
    }
  }
  if constexpr (NS == 1) {  // lanes 32 apart look after the same four channels: two each
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const u32x2_t a = swap32(__float_as_uint(amax[w]), __float_as_uint(amax[w + 2]));
      amax[w] = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    }
  }
  // the workgroup's bound in one update per channel: the updates of a unit's workgroups meet on the same 512 bytes
  __shared__ float2 amax_sh[4][kD / 2];
  amax_sh[wave][4 * n + 2 * (r & 1) + (r >> 1)] = make_float2(amax[0], amax[1]);
  __syncthreads();
  if (threadIdx.x < kD) {
    const float* const a = reinterpret_cast<const float*>(amax_sh) + threadIdx.x;
    raise_absmax(kabsmax + (size_t)unit * kD + threadIdx.x, fmaxf(fmaxf(a[0], a[kD]), fmaxf(a[2 * kD], a[3 * kD])));
  }
}

__global__ void zero_absmax_kernel(float* __restrict__ kabsmax, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) kabsmax[i] = 0.f;
}

// grid (units), block 256.  Writes the new K/V rows at position L = seq_len and re-derives the group that row falls in from
// the rows present (the new row comes from registers).
template <int DT, bool LONG>
__global__ __launch_bounds__(256) void append_kernel(uint32_t* __restrict__ K, uint32_t* __restrict__ V,
                                                     uint32_t* __restrict__ kbits, uint32_t* __restrict__ kmeta,
                                                     float* __restrict__ kabsmax, const int32_t* __restrict__ seq_lens,
                                                     const uint32_t* __restrict__ k_new, const uint32_t* __restrict__ v_new,
                                                     int n_kv_heads, int max_ctx, int ns, KvLayout lay) {
  __shared__ float4 xch[4 * 64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = blockIdx.x;
  const int L = seq_lens[unit / n_kv_heads];
  if (L < 0 || L >= max_ctx) return;
  const uint32_t kn = k_new[(size_t)unit * (kD / 2) + lane];
  const uint32_t vn = v_new[(size_t)unit * (kD / 2) + lane];
  const int t0 = L / (kG * ns) * (kG * ns), ntok = L - t0 + 1;
  uint32_t rows[LONG ? kG : kTailRows];
  GroupScale gs;
  if constexpr (!LONG) {
    uint4 mine;
    tail_load(K, lay.rows_of(unit), t0, ntok, wave, lane, rows);
    gs = append_row_short<DT>(K, V, lay.rows_of(unit), kbits, kmeta, unit, L, max_ctx, kn, vn, lane, wave, rows, xch, mine);
  } else {
    append_load_chunk(K, lay.rows_of(unit), t0, ntok, wave, kn, lane, rows);
    gs = append_row_long<DT>(K, V, lay.rows_of(unit), kbits, kmeta, unit, L, max_ctx, ns, kn, vn, lane, wave, rows, xch,
                             [](int, const uint4&, const GroupScale&) {});
  }
  if (wave != 0) return;
  raise_absmax(kabsmax + (size_t)unit * kD + 2 * lane, gs.amax0());
  raise_absmax(kabsmax + (size_t)unit * kD + 2 * lane + 1, gs.amax1());
}

template <int DT>
static void launch_quantize_dt(KvLayout lay, const uint32_t* K, uint32_t* kbits, uint32_t* kmeta, float* kabsmax,
                               const int32_t* seq_lens, int units, int n_kv_heads, int max_ctx, int ns, int bpw, int n_x,
                               hipStream_t st) {
  const dim3 grid((unsigned)units * (unsigned)(1 + n_x));
#define FIER_Q_CASE(NS)                                                                                               \
  quantize_kernel<DT, NS><<<grid, 256, 0, st>>>(K, kbits, kmeta, kabsmax, seq_lens, units, n_kv_heads, max_ctx, bpw, \
                                                n_x, lay)
  switch (ns) {
    case 1: FIER_Q_CASE(1); break;
    case 2: FIER_Q_CASE(2); break;
    case 4: FIER_Q_CASE(4); break;
    default: FIER_Q_CASE(8); break;
  }
#undef FIER_Q_CASE
}

hipError_t launch_quantize(int dtype, KvLayout lay, const void* K, uint32_t* kbits, uint32_t* kmeta, float* kabsmax,
                           const int32_t* seq_lens, int units, int n_kv_heads, int max_ctx, int group_size,
                           hipStream_t st) {
  zero_absmax_kernel<<<(units * kD + 255) / 256, 256, 0, st>>>(kabsmax, units * kD);
  const int ns = group_size / kG;
  const int n_pairs = max_ctx / kPair;
  // Pair blocks per wavefront: the most of 1, 2, 4 that still leaves a resident round of workgroups (256 CUs x 4).
  // Measured (us at 1 / 2 / 3 / 4 / 6 / 9): 8 units x 4k 9.8 / 10.9 / 13.5 / 16.0 / 20.4 / 26.6, 32 ragged units up to
  // 12k 23.5 / 27.5 / 29.5 / 30.1 / 40.5 / 46.0, 8 x 32k 26.9 / 25.8 / 26.1 / 29.8 / 33.3 / 46.4, 32 ragged units up to
  // 24k at g = 128 - / 34.5 / 40.4 / 39.7 / 41.5 / 53.8, 32 x 32k - / 59.3 / 59.8 / 57.6 / 60.0 / 60.6, 32 x 128k 412 /
  // 267 / 239 / 230 / 236 / 246, 128 ragged units up to 64k 306 / 265 / 272 / 273 / 283 / 288.
  const long blocks = (long)n_pairs * units;
  const int bpw = blocks >= 4L * 4 * 1024 ? 4 : blocks >= 4L * 2 * 1024 ? 2 : 1;
  // An odd number per unit: where only the first tokens of a large capacity are there, the workgroups with work lie n_x
  // apart, and workgroups go round-robin to the 8 XCDs and their CUs: at a multiple of 8 one XCD did everything.  512
  // units of 1000 tokens in 65536 rows: 331 us at n_x = 64, 55 at 65; 128 ragged units up to 64k 279 / 259.
  const int n_x = (n_pairs + 4 * bpw - 1) / (4 * bpw) | 1;
  if (dtype == DT_F16)
    launch_quantize_dt<DT_F16>(lay, (const uint32_t*)K, kbits, kmeta, kabsmax, seq_lens, units, n_kv_heads, max_ctx, ns,
                               bpw, n_x, st);
  else
    launch_quantize_dt<DT_BF16>(lay, (const uint32_t*)K, kbits, kmeta, kabsmax, seq_lens, units, n_kv_heads, max_ctx,
                                ns, bpw, n_x, st);
  return hipGetLastError();
}

hipError_t launch_append(int dtype, KvLayout lay, void* K, void* V, uint32_t* kbits, uint32_t* kmeta, float* kabsmax,
                         const int32_t* seq_lens, const void* k_new, const void* v_new, int units, int n_kv_heads,
                         int max_ctx, int group_size, hipStream_t st) {
  const int ns = group_size / kG;
#define FIER_APPEND(DT, LONG)                                                                                       \
  append_kernel<DT, LONG><<<units, 256, 0, st>>>((uint32_t*)K, (uint32_t*)V, kbits, kmeta, kabsmax,                  \
                                                             seq_lens, (const uint32_t*)k_new,                      \
                                                             (const uint32_t*)v_new, n_kv_heads, max_ctx, ns, lay)
  if (dtype == DT_F16) {
    if (ns == 1) FIER_APPEND(DT_F16, false);
    else FIER_APPEND(DT_F16, true);
  } else {
    if (ns == 1) FIER_APPEND(DT_BF16, false);
    else FIER_APPEND(DT_BF16, true);
  }
#undef FIER_APPEND
  return hipGetLastError();
}

}  // namespace fier
