// Quantization side of libqaq: tile build (append / requantize), width selection,
// canonical export, dequantization, accounting.  Compiled with FP contraction off:
// the fp32 operation order of the encoder and decoder is part of the contract
// (one rounding per operation, round to nearest even).
#include "qaq_internal.h"
#include <type_traits>

namespace {

constexpr int kThreads = 256;

template <int D>
struct TileLds {
  uint8_t stage[QAQ_TT][D];            // one code per (position, channel), at the token's width
  uint32_t mm[QAQ_TT];                 // fp16 min | fp16 max << 16, by position
  uint8_t oidx[QAQ_TT][QAQ_MAX_NO2];   // outlier channels, by position
  uint16_t oval[QAQ_TT][QAQ_MAX_NO2];  // outlier fp16 values
  uint8_t bits[QAQ_TT];
  uint16_t slot_of_pos[QAQ_TT];
};

__device__ __forceinline__ float h2f(uint16_t b) { return __half2float(__ushort_as_half(b)); }
__device__ __forceinline__ uint16_t f2h(float f) { return __half_as_ushort(__float2half_rn(f)); }

__device__ __forceinline__ uint32_t rd_field(const uint8_t* base, QaqFieldPos p, uint32_t mask) {
  return (*(const uint32_t*)(base + p.byte_off) >> p.shift) & mask;
}

// Code of (slot, channel d) as stored for this tile side.
template <int D>
__device__ __forceinline__ uint32_t load_code(int side, const uint8_t* base, const QaqCounts& c, uint32_t r2,
                                              uint32_t r1, uint32_t r4, uint32_t r8, uint32_t r1b, int slot, int d) {
  const int n32 = c.n32();
  if (slot >= c.first1()) {
    const int i1 = slot - c.first1();
    return side == 0 ? rd_field(base, qaq_k_field(r1b, 1, i1, d, D), 1u) : rd_field(base, qaq_v_field(r1b, 1, i1, d, D), 1u);
  }
  if (slot < n32) {
    uint32_t f = side == 0 ? rd_field(base, qaq_k_field(r2, 2, slot, d, D), 3u)
                           : rd_field(base, qaq_v_field(r2, 2, slot, d, D), 3u);
    if (slot < c.n3) {
      uint32_t lo = side == 0 ? rd_field(base, qaq_k_field(r1, 1, slot, d, D), 1u)
                              : rd_field(base, qaq_v_field(r1, 1, slot, d, D), 1u);
      return f * 2u + lo;
    }
    return f;
  }
  if (slot < n32 + c.n4) {
    int i4 = slot - n32;
    return side == 0 ? rd_field(base, qaq_k_field(r4, 4, i4, d, D), 15u)
                     : rd_field(base, qaq_v_field(r4, 4, i4, d, D), 15u);
  }
  int i8 = slot - n32 - c.n4;
  if (side == 0) return rd_field(base, qaq_k_field(r8, 8, i8, d, D), 255u) ^ 0x80u;
  return base[r8 + (uint32_t)i8 * D + d];
}

// Bring a stored tile side into LDS, indexed by position.
template <int D>
__device__ void tile_load(const QaqView& v, int side, int b, int h, int tile, int n_tok, TileLds<D>& L) {
  const int tid = threadIdx.x;
  const QaqCounts c = qaq_load_counts(v, side, b, h, tile, n_tok);
  uint32_t r2, r1, r4, r8, r1b;
  if (side == 0) { QaqKRegions r = qaq_k_regions(c, D); r2 = r.r2; r1 = r.r1; r4 = r.r4; r8 = r.r8; r1b = r.r1b; }
  else { QaqVRegions r = qaq_v_regions(c, D); r2 = r.r2; r1 = r.r1; r4 = r.r4; r8 = r.r8; r1b = r.r1b; }
  if (tid < n_tok) {
    const int s = tid;
    const size_t gi = qaq_slot_index(v, b, h, tile, s);
    const int pos = v.perm[side][gi];
    L.mm[pos] = v.mm[side][gi];
    L.slot_of_pos[pos] = (uint16_t)s;
    L.bits[pos] = (uint8_t)c.bits_of_slot(s);
    for (int k = 0; k < v.no2 && !v.csr; ++k) {
      L.oidx[pos][k] = v.oidx[side][gi * v.no2 + k];
      L.oval[pos][k] = v.oval[side][gi * v.no2 + k];
    }
  }
  if (v.csr && tid < n_tok) {       // variable-length side store: by position; unused places of the row = channel 255
    const size_t pi = qaq_slot_index(v, b, h, tile, tid);
    const size_t pool0 = qaq_slot_index(v, b, h, tile, 0) * (size_t)v.no2;
    const int cnt = v.ocnt[side][pi], st = v.ostart[side][pi];
    for (int k = 0; k < v.no2; ++k) {
      L.oidx[tid][k] = k < cnt ? v.oidx[side][pool0 + st + k] : (uint8_t)0xffu;
      L.oval[tid][k] = k < cnt ? v.oval[side][pool0 + st + k] : (uint16_t)0;
    }
  }
  __syncthreads();
  const uint8_t* base = qaq_tile_codes(v, side, b, h, tile);
  for (int e = tid; e < n_tok * D; e += kThreads) {
    const int pos = e / D, d = e % D;
    L.stage[pos][d] = (uint8_t)load_code<D>(side, base, c, r2, r1, r4, r8, r1b, L.slot_of_pos[pos], d);
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------------
// Tile build (append / requantize): a tile side is written as a whole.  Codes travel through LDS as one byte per
// (position, channel), a token's code in the upper bits of its byte; both directions between that staging form and the
// stored code planes work on whole 32-bit words: shifts and masks take four codes along, and the token-transposed value
// planes go through 4x4 byte transposes in registers.
// ---------------------------------------------------------------------------------
template <int D, int MAXO = QAQ_MAX_NO2>   // MAXO: outlier entries held per token (2 in the common one-per-end build)
struct BuildLds {
  static constexpr int SROW = D / 4 + 1;   // dwords per staged row; the odd stride spreads rows over the banks
  uint32_t stage[(QAQ_TT + 1) * SROW];     // byte d of row pos = code of channel d (the last row: nobody's)
  uint32_t mm[QAQ_TT];                     // fp16 min | fp16 max << 16, by position
  uint8_t oidx[QAQ_TT][MAXO];              // outlier channels, by position
  uint16_t oval[QAQ_TT][MAXO];             // outlier fp16 values
  uint8_t bits_old[QAQ_TT];                // widths, by position
  uint8_t order[QAQ_TT];                   // positions to encode; later the position of the token that holds a slot
  alignas(16) uint16_t row_of_slot[QAQ_TT];      // byte offset of the staged row of the token that holds a slot
  alignas(16) uint16_t row_of_old[QAQ_TT];       // ... that held it before
  int wave_cnt[QAQ_NCLASS][4];
  int wave_enc[4];
  float wave_bound[4];
  float wave_bound2[4];
  int wave_ocnt[4];                        // variable-length side store: entries of the new tokens per wavefront
  int wave_wide[4];                        // widenings asked for, per wavefront
};

__device__ __forceinline__ int lanes_below(unsigned long long mask) {     // set bits of `mask` below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// rows of four bytes <-> columns of four bytes: t[k] byte j = w[j] byte k
__device__ __forceinline__ void transpose4(const uint32_t (&w)[4], uint32_t (&t)[4]) {
  const uint32_t a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);   // w0.b0 w1.b0 w0.b1 w1.b1
  const uint32_t b = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);   // w0.b2 w1.b2 w0.b3 w1.b3
  const uint32_t c = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
  const uint32_t d = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
  t[0] = __builtin_amdgcn_perm(c, a, 0x05040100u);
  t[1] = __builtin_amdgcn_perm(c, a, 0x07060302u);
  t[2] = __builtin_amdgcn_perm(d, b, 0x05040100u);
  t[3] = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, true);      // (within quads every lane has a source)
}
// Reductions over the four consecutive lanes (one quad) that share a token; every lane
// of the quad ends up with the result.
__device__ __forceinline__ uint32_t quad_umax(uint32_t x) {
  uint32_t y = dpp_u<0xB1>(x); x = x > y ? x : y;      // quad_perm [1,0,3,2]
  y = dpp_u<0x4E>(x); return x > y ? x : y;            // quad_perm [2,3,0,1]
}
__device__ __forceinline__ uint32_t quad_umin(uint32_t x) {
  uint32_t y = dpp_u<0xB1>(x); x = x < y ? x : y;
  y = dpp_u<0x4E>(x); return x < y ? x : y;
}
// Integers that order like the fp16 numbers (both zeros the same): on the bit patterns, two at a time: per 16-bit half,
// 0x8000 + magnitude for a positive number, 0x8000 - magnitude for a negative one (both zeros
// give 0x8000).  Shifted into the upper half of a word such a key leaves 16 low bits for the
// channel number.
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef short ss2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t order_keys_pair(uint32_t two_halves) {
  const us2 b = __builtin_bit_cast(us2, two_halves);
  const us2 sg = __builtin_bit_cast(us2, __builtin_bit_cast(ss2, b) >> (ss2)15);    // 0xffff where negative
  const us2 mag = b & (us2)0x7fffu;
  const us2 t = (mag ^ sg) - sg;                                                      // +-magnitude, two's complement
  return __builtin_bit_cast(uint32_t, (us2)(t + (us2)0x8000u));
}
// ... and as signed 16-bit numbers (magnitude, or minus magnitude), for the packed maximum and minimum
__device__ __forceinline__ ss2 signed_keys_pair(uint32_t two_halves) {
  const ss2 b = __builtin_bit_cast(ss2, two_halves);
  const ss2 sg = b >> (ss2)15;
  return ((b & (ss2)0x7fff) ^ sg) - sg;
}
__device__ __forceinline__ ss2 pk_max(ss2 a, ss2 b) { return __builtin_elementwise_max(a, b); }
__device__ __forceinline__ ss2 pk_min(ss2 a, ss2 b) { return __builtin_elementwise_min(a, b); }
__device__ __forceinline__ uint32_t signed_key_bits(int key) { return (uint32_t)(key < 0 ? 0x8000 - key : key); }   // fp16 bits (of +0 for a zero)
// maximum, minimum in one instruction: of a NaN and a number the number, as fmaxf, but without its test for signalling NaNs
__device__ __forceinline__ float vmaxf(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float vminf(float a, float b) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// Larger and smaller of two pairs of fp16, one instruction (of a NaN and a number the number); `pk_hmaximum`: the NaN.
__device__ __forceinline__ uint32_t pk_hmax(uint32_t a, uint32_t b) { uint32_t r; asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b)); return r; }
__device__ __forceinline__ uint32_t pk_hmin(uint32_t a, uint32_t b) { uint32_t r; asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b)); return r; }
__device__ __forceinline__ uint32_t pk_hmaximum(uint32_t a, uint32_t b, uint32_t c) { uint32_t r; asm("v_pk_maximum3_f16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c)); return r; }
__device__ __forceinline__ uint32_t halves_swapped(uint32_t x) { return __builtin_amdgcn_alignbit(x, x, 16u); }
// An element of a pair of fp16 less a float, rounded once (the fp16 number is exact in fp32): one instruction
__device__ __forceinline__ float half_minus(uint32_t pair, bool upper, float x) {
  float r;
  if (upper) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(pair), "v"(x));
  else asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(pair), "v"(x));
  return r;
}
// floor of eight numbers, clamped to [0, 255], as the bytes of two words.  v_cvt_pk_u8_f32 rounds as the mode register
// says and saturates: rounding toward zero for the eight of them takes the place of eight floors (below zero both give 0).
__device__ __forceinline__ void floor_bytes(const float (&x)[8], uint32_t& w0, uint32_t& w1) {
  asm("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 3\n\t"
      "v_cvt_pk_u8_f32 %0, %2, 0, 0\n\t"
      "v_cvt_pk_u8_f32 %1, %6, 0, 0\n\t"
      "v_cvt_pk_u8_f32 %0, %3, 1, %0\n\t"
      "v_cvt_pk_u8_f32 %1, %7, 1, %1\n\t"
      "v_cvt_pk_u8_f32 %0, %4, 2, %0\n\t"
      "v_cvt_pk_u8_f32 %1, %8, 2, %1\n\t"
      "v_cvt_pk_u8_f32 %0, %5, 3, %0\n\t"
      "v_cvt_pk_u8_f32 %1, %9, 3, %1\n\t"
      "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0"
      : "=&v"(w0), "=&v"(w1)
      : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]));
}
// value of a key made from order_keys_pair (upper 16 bits; the low bits carry a channel number)
__device__ __forceinline__ float key16_value(uint32_t key) {
  const uint32_t k = key >> 16;
  const uint32_t hb = k >= 0x8000u ? k - 0x8000u : ((0x8000u - k) | 0x8000u);
  return h2f((uint16_t)hb);
}

// ---------------------------------------------------------------------------------
// Encoder for one token vector, run by the four lanes of a quad; lane c holds the 8-channel
// chunks c, c+4, c+8, ... (a quad reads 64 contiguous bytes per load).  Outliers
// (Section 4.2): the n_o largest, then the n_o smallest of the rest, ties to the lower
// channel; [min,max] over what remains; then the midpoint quantizer of Section 4.1:
// code = clamp(floor((x-min)*2^B/range)), always at eight bits: a narrower code is its upper bits.
//
// Bound by vector instructions: a bulk build spends four fifths of its on the search and the codes.  So the search works
// on pairs of fp16 values and looks for the channels afterwards (193 instructions for a quad's lane with 32 elements; 228 with a
// sweep over all words for each channel, 282 on integer keys, 395 with the channel in the low bits of 32-bit keys), and a code takes three instructions, not six.  Figures:
// see fresh_tile.
// ---------------------------------------------------------------------------------
template <int D, bool ONE>   // ONE: exactly one outlier per end (the common case) has its own, shorter search
struct TokenEncoder {
  static constexpr int NCH = D / 32;          // 16-byte chunks per lane
  static constexpr int EPL = 8 * NCH;         // elements per lane

  __device__ static __forceinline__ uint32_t half_bits(const uint4 (&raw)[NCH], int i, int e) {
    const uint32_t w = e < 2 ? raw[i].x : e < 4 ? raw[i].y : e < 6 ? raw[i].z : raw[i].w;
    return (w >> (16 * (e & 1))) & 0xffffu;
  }
  __device__ static __forceinline__ int channel(int c, int i, int e) { return 32 * i + 8 * c + e; }

  // fp16 bits of the outlier on channel ch (held by this lane), whose value is `val`
  __device__ static __forceinline__ uint16_t outlier_bits(const uint4 (&raw)[NCH], int c, int ch, float val) {
    uint32_t hv = f2h(val);
    if (val == 0.0f) {   // the key does not keep the sign of a zero: take the stored bits
#pragma unroll
      for (int i = 0; i < NCH; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (channel(c, i, e) == ch) hv = half_bits(raw, i, e);
    }
    return (uint16_t)hv;
  }

  // The pair of values `pair` (both halves the same) among the words x: the lowest channel that holds it, over the quad;
  // 255 or more if none does
  template <typename WORD>
  __device__ static __forceinline__ uint32_t first_channel(WORD word, int c, uint32_t pair, us2 one) {
    constexpr uint32_t ALL = (1u << (4 * NCH)) - 1u;
    uint32_t misses = 0u;                   // per word one bit of each half, the first word's in bit 4 NCH - 1 of it
#pragma unroll
    for (int j = 0; j < 4 * NCH; ++j)
      asm("v_lshl_or_b32 %0, %1, 1, %2" : "=v"(misses) : "v"(misses), "v"(__builtin_elementwise_min(__builtin_bit_cast(us2, word(j) ^ pair), one)));
    const uint32_t hits = misses ^ (ALL * 0x10001u);
    const uint32_t e_lo = 2u * (uint32_t)__builtin_clz((hits << 16) | 1u), e_hi = 2u * (uint32_t)__builtin_clz(hits | 1u) + 1u;
    const uint32_t e = (e_lo < e_hi ? e_lo : e_hi) - 2u * (16u - 4 * NCH);
    const uint32_t ch = ((e & ~7u) << 2) + (uint32_t)(8 * c) + (e & 7u);
    return quad_umin(e < (uint32_t)EPL ? ch : 0xffu);
  }
  __device__ static __forceinline__ uint32_t word_of(const uint4 (&raw)[NCH], int j) {
    return (j & 3) == 0 ? raw[j >> 2].x : (j & 3) == 1 ? raw[j >> 2].y : (j & 3) == 2 ? raw[j >> 2].z : raw[j >> 2].w;
  }

  // The same where `pair` is the extreme of the whole token and ext[i] that of chunk i in each half (SMALLEST: which extreme):
  // by halving, since the extreme of the first half of what is left tells whether it is there.  47 instructions an end at
  // 128 channels where the sweep over all words takes 60.
  template <bool SMALLEST>
  __device__ static __forceinline__ uint32_t channel_of_end(const uint4 (&raw)[NCH], const uint32_t (&ext)[NCH], int c, uint32_t pair) {
    auto further = [](uint32_t a, uint32_t b) { return SMALLEST ? pk_hmin(a, b) : pk_hmax(a, b); };
    auto has = [&](uint32_t m) {
      const uint32_t x = m ^ pair;
      const us2 z = __builtin_elementwise_min(__builtin_bit_cast(us2, x), __builtin_bit_cast(us2, halves_swapped(x)));
      return z.x == 0;
    };
    uint32_t w[8], e = 0u, first = ext[0];
    if constexpr (NCH == 4) {
      const bool in = has(further(ext[0], ext[1]));
#pragma unroll
      for (int j = 0; j < 8; ++j) w[j] = in ? word_of(raw, j) : word_of(raw, 8 + j);
      first = in ? ext[0] : ext[2];
      e = in ? 0u : 16u;
    } else {
      static_assert(NCH == 2, "chunks per lane");
#pragma unroll
      for (int j = 0; j < 8; ++j) w[j] = word_of(raw, j);
    }
    bool in = has(first);
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = in ? w[j] : w[4 + j];
    e += in ? 0u : 8u;
    in = has(further(w[0], w[1]));
    w[0] = in ? w[0] : w[2]; w[1] = in ? w[1] : w[3];
    e += in ? 0u : 4u;
    in = has(w[0]);
    w[0] = (in ? w[0] : w[1]) ^ pair;
    e += in ? 0u : 2u;
    const bool low = (w[0] & 0xffffu) == 0u, high = w[0] < 0x10000u;
    e += low ? 0u : 1u;
    const uint32_t ch = ((e & ~7u) << 2) + (uint32_t)(8 * c) + (e & 7u);
    return quad_umin(low || high ? ch : 0xffu);
  }

  // One outlier per end: the largest and the smallest value of a token and the runners-up.  The two largest and the two
  // smallest come from four words at a time, sorted as pairs (ten instructions for eight elements) and merged into the
  // running ones; then over the halves of the words and the lanes of the quad (there the largest and minus the smallest
  // in one word); the channels are looked up afterwards.  On the fp16 values themselves where the ends are ordinary
  // numbers; where an end is a zero (two bit patterns) or not finite, or a value is not a number, on integer keys.
  __device__ static __forceinline__ void ends_of_token(const uint4 (&raw)[NCH], int c, uint8_t* oidx_row, uint16_t* oval_row, float& mn, float& mx, bool& finite) {
    uint32_t ones = 0x10001u;
    asm("" : "+s"(ones));              // (known to be ones, the minimum with them becomes two compares and two selects)
    const us2 one = __builtin_bit_cast(us2, ones);
    uint32_t A1 = 0u, A2 = 0u, B1 = 0u, B2 = 0u, any = 0u;      // (any: the largest, or a NaN if there is one)
    uint32_t hi[NCH], lo[NCH];                                  // of each chunk
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const uint32_t x = raw[i].x, y = raw[i].y, z = raw[i].z, w = raw[i].w;
      const uint32_t h0 = pk_hmax(x, y), l0 = pk_hmin(x, y), h1 = pk_hmax(z, w), l1 = pk_hmin(z, w);
      const uint32_t s3 = pk_hmax(h0, h1), s0 = pk_hmin(l0, l1), m0 = pk_hmin(h0, h1), m1 = pk_hmax(l0, l1);
      const uint32_t s2 = pk_hmax(m0, m1), s1 = pk_hmin(m0, m1);
      hi[i] = s3; lo[i] = s0;
      if (i == 0) { A1 = s3; A2 = s2; B1 = s0; B2 = s1; any = pk_hmaximum(x, y, z); any = pk_hmaximum(any, w, w); }
      else {
        A2 = pk_hmax(pk_hmin(A1, s3), pk_hmax(A2, s2)); A1 = pk_hmax(A1, s3);
        B2 = pk_hmin(pk_hmax(B1, s0), pk_hmin(B2, s1)); B1 = pk_hmin(B1, s0);
        any = pk_hmaximum(any, x, y); any = pk_hmaximum(any, z, w);
      }
    }
    const uint32_t As = halves_swapped(A1), Bs = halves_swapped(B1);
    A2 = pk_hmax(pk_hmin(A1, As), pk_hmax(A2, halves_swapped(A2)));
    B2 = pk_hmin(pk_hmax(B1, Bs), pk_hmin(B2, halves_swapped(B2)));
    B1 = pk_hmin(B1, Bs);
    any = pk_hmaximum(any, any, halves_swapped(any));
    uint32_t e1 = __builtin_amdgcn_perm(B1, any, 0x05040100u) ^ 0x80000000u;
    uint32_t e2 = __builtin_amdgcn_perm(B2, A2, 0x05040100u) ^ 0x80000000u;
#pragma unroll
    for (int step = 0; step < 2; ++step) {
      const uint32_t y1 = step ? dpp_u<0x4E>(e1) : dpp_u<0xB1>(e1), y2 = step ? dpp_u<0x4E>(e2) : dpp_u<0xB1>(e2);
      e2 = pk_hmax(pk_hmin(e1, y1), pk_hmax(e2, y2));
      e1 = pk_hmaximum(e1, y1, y1);
    }
    const us2 mag = __builtin_bit_cast(us2, e1 & 0x7fff7fffu) - one;              // magnitudes of the ends, less one
    const us2 most = __builtin_elementwise_max(mag, mag.yx);
    uint32_t ch_top, ch_bot, v_top, v_bot;
    if (__ballot(most.x >= 0x7bffu) == 0ull) {
      const uint32_t top_pair = __builtin_amdgcn_perm(0u, e1, 0x01000100u), bot_pair = __builtin_amdgcn_perm(0u, e1, 0x03020302u) ^ 0x80008000u;
      ch_top = channel_of_end<false>(raw, hi, c, top_pair);
      ch_bot = channel_of_end<true>(raw, lo, c, bot_pair);
      // the smallest of the rest is the overall smallest unless that is the top element itself: all values are equal
      // then, and it is the second of them
      if (top_pair == bot_pair) ch_bot = 1u;
      v_top = e1 & 0xffffu; v_bot = (e1 >> 16) ^ 0x8000u;
      // what remains: its largest value is the runner-up of the largest, its smallest of the smallest (equal values make
      // the choice of element moot; a zero without its sign)
      mx = h2f((uint16_t)(e2 & 0xffffu)) + 0.0f; mn = h2f((uint16_t)((e2 >> 16) ^ 0x8000u)) + 0.0f;
      finite = true;
    } else {
      ends_by_keys(raw, c, one, ch_top, ch_bot, v_top, v_bot, mn, mx, finite);
    }
    if (c == 0) {          // the side store's row, by channel
      const bool first = ch_top < ch_bot;
      *(uint16_t*)oidx_row = (uint16_t)(first ? ch_top | (ch_bot << 8) : ch_bot | (ch_top << 8));
      *(uint32_t*)oval_row = first ? v_top | (v_bot << 16) : v_bot | (v_top << 16);
    }
  }
  // The same for any bit patterns, on signed 16-bit keys (signed_keys_pair)
  __device__ static __forceinline__ void ends_by_keys(const uint4 (&raw)[NCH], int c, us2 one, uint32_t& ch_top, uint32_t& ch_bot, uint32_t& v_top, uint32_t& v_bot,
                                                      float& mn, float& mx, bool& finite) {
    ss2 A1, A2;      // largest and runner-up; in the upper half, of the numbers with their signs changed
    A1 = A2 = (ss2)(short)-0x8000;
#pragma unroll 1
    for (int j = 0; j < 4 * NCH; ++j) {
      uint32_t w = 0u;
#pragma unroll
      for (int i = 0; i < 4 * NCH; ++i) w = i == j ? word_of(raw, i) : w;
      const ss2 k = signed_keys_pair(w);
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const ss2 x = hf ? ss2{k.y, (short)-k.y} : ss2{k.x, (short)-k.x};
        A2 = pk_max(pk_min(A1, x), A2); A1 = pk_max(A1, x);
      }
    }
#pragma unroll
    for (int step = 0; step < 2; ++step) {
      const uint32_t e1 = __builtin_bit_cast(uint32_t, A1), e2 = __builtin_bit_cast(uint32_t, A2);
      const ss2 y1 = __builtin_bit_cast(ss2, step ? dpp_u<0x4E>(e1) : dpp_u<0xB1>(e1)), y2 = __builtin_bit_cast(ss2, step ? dpp_u<0x4E>(e2) : dpp_u<0xB1>(e2));
      A2 = pk_max(pk_min(A1, y1), pk_max(A2, y2)); A1 = pk_max(A1, y1);
    }
    const int top = A1.x, bot = -A1.y;
    finite = top < 0x7c00 && bot > -0x7c00;
    const uint32_t top_pair = __builtin_amdgcn_perm(0u, (uint32_t)top, 0x01000100u), bot_pair = __builtin_amdgcn_perm(0u, (uint32_t)bot, 0x01000100u);
    auto word = [&](int j) { return __builtin_bit_cast(uint32_t, signed_keys_pair(word_of(raw, j))); };
    ch_top = first_channel(word, c, top_pair, one);
    ch_bot = top == bot ? 1u : first_channel(word, c, bot_pair, one);
    // (the key does not keep the sign of a zero: the bits as they are stored)
    v_top = v_bot = 0u;
#pragma unroll
    for (int i = 0; i < NCH; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (channel(c, i, e) == (int)ch_top) v_top = half_bits(raw, i, e);
        if (channel(c, i, e) == (int)ch_bot) v_bot = half_bits(raw, i, e);
      }
    v_top = quad_umax(v_top); v_bot = quad_umax(v_bot);
    mx = h2f((uint16_t)signed_key_bits(A2.x)); mn = h2f((uint16_t)signed_key_bits(-A2.y));
  }

  // Any number of outliers: the largest, then the smallest of the rest, each found over the quad (keys as in ends_by_keys;
  // kx, kn: of the elements that are left, a taken one at the far end).  The loops over words stay short of registers: 32
  // keys for each end made this form take 177 of them, two wavefronts per SIMD.
  __device__ static __forceinline__ void outliers_one_by_one(const uint4 (&raw)[NCH], int c, us2 one, int n_o, float thr_lo, float thr_hi,
                                                             uint8_t* oidx_row, uint16_t* oval_row, float& mn, float& mx) {
    constexpr int W = 4 * NCH;
    ss2 kx[W], kn[W];
#pragma unroll
    for (int j = 0; j < W; ++j) kx[j] = kn[j] = signed_keys_pair(word_of(raw, j));
    auto largest = [&]() -> int {
      ss2 m = kx[0];
#pragma unroll
      for (int j = 1; j < W; ++j) m = pk_max(m, kx[j]);
      m = pk_max(m, m.yx);
      m = pk_max(m, __builtin_bit_cast(ss2, dpp_u<0xB1>(__builtin_bit_cast(uint32_t, m))));
      return pk_max(m, __builtin_bit_cast(ss2, dpp_u<0x4E>(__builtin_bit_cast(uint32_t, m)))).x;
    };
    auto smallest = [&]() -> int {
      ss2 m = kn[0];
#pragma unroll
      for (int j = 1; j < W; ++j) m = pk_min(m, kn[j]);
      m = pk_min(m, m.yx);
      m = pk_min(m, __builtin_bit_cast(ss2, dpp_u<0xB1>(__builtin_bit_cast(uint32_t, m))));
      return pk_min(m, __builtin_bit_cast(ss2, dpp_u<0x4E>(__builtin_bit_cast(uint32_t, m)))).x;
    };
    int n_rec = 0;
#pragma unroll 1
    for (int end = 0; end < 2; ++end) {
      bool alive = true;                   // the same for the four lanes of a quad
#pragma unroll 1
      for (int k = 0; k < n_o; ++k) {
        const int M = end == 0 ? largest() : smallest();
        const float val = h2f((uint16_t)signed_key_bits(M));
        alive = alive && (end == 0 ? val > thr_hi : val < thr_lo);
        if (__ballot(alive) == 0ull) break;
        const uint32_t pair = __builtin_amdgcn_perm(0u, (uint32_t)M, 0x01000100u);
        const uint32_t ch = first_channel([&](int j) { return __builtin_bit_cast(uint32_t, end == 0 ? kx[j] : kn[j]); }, c, pair, one);
        const bool mine = alive && ((ch >> 3) & 3u) == (uint32_t)c;
        const uint32_t at = (ch >> 5) * 4u + ((ch >> 1) & 3u);
        const uint32_t half = mine ? (ch & 1u ? 0xffff0000u : 0xffffu) : 0u;
#pragma unroll
        for (int j = 0; j < W; ++j) {
          const uint32_t m = at == (uint32_t)j ? half : 0u;
          kx[j] = __builtin_bit_cast(ss2, (__builtin_bit_cast(uint32_t, kx[j]) & ~m) | (0x80008000u & m));
          kn[j] = __builtin_bit_cast(ss2, (__builtin_bit_cast(uint32_t, kn[j]) & ~m) | (0x7fff7fffu & m));
        }
        if (mine) { oidx_row[n_rec] = (uint8_t)ch; oval_row[n_rec] = outlier_bits(raw, c, (int)ch, val); }
        n_rec += alive ? 1 : 0;
      }
    }
    if (c == 0)
      for (int k = n_rec; k < 2 * n_o; ++k) { oidx_row[k] = 0xffu; oval_row[k] = 0; }
    mx = h2f((uint16_t)signed_key_bits(largest())); mn = h2f((uint16_t)signed_key_bits(smallest()));
  }

  // Outliers by thresholds, where no token of the wavefront has more of them at an end than are kept and no value is not a
  // number (else nothing is done and the result is false): every value outside is one, in any order, the rest is [min, max].
  __device__ static __forceinline__ bool passing_thresholds(const uint4 (&raw)[NCH], int c, us2 one, int n_o, float thr_lo, float thr_hi,
                                                            uint8_t* oidx_row, uint16_t* oval_row, float& mn, float& mx) {
    constexpr int W = 4 * NCH;
    // the thresholds as keys: of the largest fp16 number not above thr_hi, the smallest not below thr_lo
    const uint32_t hb = f2h(thr_hi), lb = f2h(thr_lo);
    const int key_hi = (int)signed_keys_pair(hb).x - (h2f((uint16_t)hb) > thr_hi ? 1 : 0), key_lo = (int)signed_keys_pair(lb).x + (h2f((uint16_t)lb) < thr_lo ? 1 : 0);
    const ss2 hi = {(short)key_hi, (short)key_hi}, lo = {(short)key_lo, (short)key_lo};
    uint32_t any = raw[0].x, hits = 0u;        // (hits, values outside: per word a bit for each half, the first word's in bit W - 1)
    ss2 most = {-0x8000, -0x8000}, least = {0x7fff, 0x7fff};
    uint32_t n_top = 0u;
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const ss2 k = signed_keys_pair(word_of(raw, j));
      if (j & 1) any = pk_hmaximum(any, word_of(raw, j), word_of(raw, j - 1));
      // one where the clamped value differs from the value
      const uint32_t over = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(us2, __builtin_bit_cast(uint32_t, pk_max(k, hi)) ^ __builtin_bit_cast(uint32_t, hi)), one));
      const uint32_t under = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(us2, __builtin_bit_cast(uint32_t, pk_min(k, lo)) ^ __builtin_bit_cast(uint32_t, lo)), one));
      const uint32_t out = over | under;
      n_top += over;
      asm("v_lshl_or_b32 %0, %1, 1, %2" : "=v"(hits) : "v"(hits), "v"(out));
      const ss2 mask = (ss2)0 - __builtin_bit_cast(ss2, out);
      const uint32_t m = __builtin_bit_cast(uint32_t, mask), kw = __builtin_bit_cast(uint32_t, k);
      most = pk_max(most, __builtin_bit_cast(ss2, (kw & ~m) | (0x80008000u & m)));
      least = pk_min(least, __builtin_bit_cast(ss2, (kw & ~m) | (0x7fff7fffu & m)));
    }
    const int top = (int)((n_top & 0xffffu) + (n_top >> 16)), all = __popc(hits);
    auto quad_sum = [](int x) { x += (int)dpp_u<0xB1>((uint32_t)x); return x + (int)dpp_u<0x4E>((uint32_t)x); };
    const int counts = quad_sum(top | (all << 16)), q_top = counts & 0xffff, q_all = counts >> 16;
    any = pk_hmaximum(any, halves_swapped(any), any);
    const bool nan = (any & 0x7fffu) > 0x7c00u;
    if (__ballot(nan || q_top > n_o || q_all - q_top > n_o) != 0ull) return false;
    most = pk_max(most, most.yx); least = pk_min(least, least.yx);
#pragma unroll
    for (int step = 0; step < 2; ++step) {
      const uint32_t a = __builtin_bit_cast(uint32_t, most), b = __builtin_bit_cast(uint32_t, least);
      most = pk_max(most, __builtin_bit_cast(ss2, step ? dpp_u<0x4E>(a) : dpp_u<0xB1>(a)));
      least = pk_min(least, __builtin_bit_cast(ss2, step ? dpp_u<0x4E>(b) : dpp_u<0xB1>(b)));
    }
    mx = h2f((uint16_t)signed_key_bits(most.x)); mn = h2f((uint16_t)signed_key_bits(least.x));
    // the row: unused places first, then every lane's entries behind those of the lanes before it
    if (c == 0)
      for (int k = q_all; k < 2 * n_o; ++k) { oidx_row[k] = 0xffu; oval_row[k] = 0; }
    const int x1 = (int)dpp_u<0xB1>((uint32_t)all), x2 = (int)dpp_u<0x4E>((uint32_t)all), x3 = (int)dpp_u<0x1B>((uint32_t)all);     // of lanes c^1, c^2, c^3
    int at = (c & 1 ? x1 : 0) + (c & 2 ? x2 + x3 : 0);
    while (hits) {
      const int bit = 31 - __builtin_clz(hits);
      hits &= ~(1u << bit);
      const int hf = bit >> 4, w = W - 1 - (bit & 15);
      uint32_t x = 0u;
#pragma unroll
      for (int j = 0; j < W; ++j) x = w == j ? word_of(raw, j) : x;
      oidx_row[at] = (uint8_t)(32 * (w >> 2) + 8 * c + 2 * (w & 3) + hf);
      oval_row[at] = (uint16_t)(x >> (16 * hf));
      ++at;
    }
    return true;
  }

  // thr_lo, thr_hi: an outlier must lie below thr_lo resp. above thr_hi (+inf, -inf: the count
  // rule, every candidate passes); a side stops at its first candidate that does not, and the
  // rows of the side store are filled from the front, the rest marked unused (channel 255)
  __device__ static __forceinline__ void run(const uint4 (&raw)[NCH], int c, bool fresh, int n_o, uint32_t* mm_pos,
                                             uint8_t* oidx_row, uint16_t* oval_row, uint32_t* stage_row,
                                             float thr_lo = INFINITY, float thr_hi = -INFINITY) {
    float mn, mx;
    bool finite = false;      // all values known to be
    if (fresh) {
      if constexpr (ONE) {
        ends_of_token(raw, c, oidx_row, oval_row, mn, mx, finite);
      } else {
        uint32_t ones = 0x10001u;
        asm("" : "+s"(ones));              // (see ends_of_token)
        const us2 one = __builtin_bit_cast(us2, ones);
        if (thr_lo == INFINITY || !passing_thresholds(raw, c, one, n_o, thr_lo, thr_hi, oidx_row, oval_row, mn, mx))
          outliers_one_by_one(raw, c, one, n_o, thr_lo, thr_hi, oidx_row, oval_row, mn, mx);
      }
      if (c == 0) *mm_pos = (uint32_t)f2h(mn) | ((uint32_t)f2h(mx) << 16);
    } else {
      const uint32_t m = *mm_pos;
      mn = h2f((uint16_t)(m & 0xffffu));
      mx = h2f((uint16_t)(m >> 16));
    }
    const float range = mx - mn;
    const float inv = range > 0.0f ? 256.0f / range : 0.0f;   // an empty range gives code 0 everywhere
    // (the byte conversion's own clamp is the quantizer's at eight bits, but for a NaN, whose code is the top one)
    const bool clamps = __ballot(!finite) != 0ull;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t w = e < 2 ? raw[i].x : e < 4 ? raw[i].y : e < 6 ? raw[i].z : raw[i].w;
        const float diff = half_minus(w, e & 1, mn);
        x[e] = diff * inv;
      }
      if (clamps) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = vminf(x[e], 255.0f);
      }
      uint32_t w0, w1;
      floor_bytes(x, w0, w1);
      stage_row[2 * (4 * i + c)] = w0;
      stage_row[2 * (4 * i + c) + 1] = w1;
    }
  }
};

// ---------------------------------------------------------------------------------
// Widenings asked for in a tile side: every wavefront leaves its count in LDS (`per_wave`,
// four entries); after the next barrier add_widenings, called by one thread, adds them to the
// tile side's own counters (kind 0 = refused for want of the unquantized copy, 1 = served).
// A tile side is only ever written by the workgroup that owns it, so no atomics are needed;
// the accounting kernel sums the counters.
__device__ __forceinline__ void note_widenings(int* per_wave, bool wider, int tid) {
  const unsigned long long bal = __ballot(wider);
  if ((tid & 63) == 0) per_wave[tid >> 6] = __popcll(bal);
}
__device__ __forceinline__ void add_widenings(const QaqView& v, size_t tile_side, const int* per_wave, bool served) {
  const int n = per_wave[0] + per_wave[1] + per_wave[2] + per_wave[3];
  if (n) v.refused[tile_side * 2 + (served ? 1 : 0)] += (unsigned int)n;
}

// What both forms of the build have in common, for one position's thread.
// Width by the rules of Section 4.1: the narrowest that satisfies lhs <= threshold * 2^B, else the widest
__device__ __forceinline__ int rule_width(const QaqRuleArgs& ru, float lhs, float thr) {
  int w = ru.bit_set[ru.nbits - 1];
  for (int i = ru.nbits - 1; i >= 0; --i)
    if (lhs <= ldexpf(thr, ru.bit_set[i])) w = ru.bit_set[i];
  return w;
}
// Side store's row of a fresh token: order by channel (the one-per-end encoder leaves it so)
__device__ __forceinline__ void sort_side_store(uint8_t* idx, uint16_t* val, int no2) {
  for (int i = 1; i < no2; ++i) {
    const uint8_t ki = idx[i];
    const uint16_t vi = val[i];
    int j = i - 1;
    while (j >= 0 && idx[j] > ki) { idx[j + 1] = idx[j]; val[j + 1] = val[j]; --j; }
    idx[j + 1] = ki;
    val[j + 1] = vi;
  }
}
// Values: what the attention kernel needs as the fixed-point range of a tile -- the largest per-token step range/2^B (a 3-bit
// code is split into planes, the upper one weighs twice the step) and the largest magnitude an outlier correction (stored value
// minus reconstruction) can have
__device__ __forceinline__ float value_bound(int bits, float mn, float mx, const uint8_t* idx, const uint16_t* val, int no2) {
  const float range = mx - mn;
  float bnd = ldexpf(range, bits == 3 ? -2 : -bits);
  for (int k = 0; k < no2; ++k) {
    if (idx[k] == 0xffu) continue;        // (variable-length side store: an unused place)
    const float ov = h2f(val[k]);
    bnd = fmaxf(bnd, fmaxf(fabsf(ov - mx), fabsf(ov - mn)) + range);
  }
  return bnd;
}
// Keys: thresholds for which the token keeps its width (Section 4.1 key rule as the comparison range <= threshold * 2^B): a token
// at width B widens below range / 2^B and narrows from range / 2^B' on, B' the next narrower width; the power-of-two scalings are exact
__device__ __forceinline__ void key_interval(const QaqRuleArgs& ru, int bits, float range, float& lo, float& hi) {
  int narrower = 0;
  for (int i = 0; i < ru.nbits; ++i)
    if (ru.bit_set[i] < bits) narrower = ru.bit_set[i];
  if (bits < ru.bit_set[ru.nbits - 1]) lo = ldexpf(range, -bits);
  if (narrower > 0) hi = ldexpf(range, -narrower);
}
// Variable-length side store: the entries of the new tokens (positions n_before .. n_after - 1) go behind the tile's last one, in
// position order (a prefix sum of their counts)
template <int D, int MAXO>
__device__ __forceinline__ void put_new_runs(const QaqView& v, int side, size_t gi0, int n_before, int n_after, BuildLds<D, MAXO>& L, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
  const size_t pool0 = gi0 * (size_t)v.no2;
  const bool fresh = tid >= n_before && tid < n_after;
  int cnt = 0;
  if (fresh)
    for (int k = 0; k < v.no2; ++k) cnt += L.oidx[tid][k] != 0xffu;
  int inc = cnt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == 63) L.wave_ocnt[wave] = inc;
  __syncthreads();
  int start = inc - cnt;
  for (int w = 0; w < wave; ++w) start += L.wave_ocnt[w];
  if (n_before > 0) start += (int)v.ostart[side][gi0 + n_before - 1] + (int)v.ocnt[side][gi0 + n_before - 1];
  if (fresh) {
    v.ostart[side][gi0 + tid] = (uint16_t)start;
    v.ocnt[side][gi0 + tid] = (uint8_t)cnt;
    for (int k = 0; k < cnt; ++k) {          // the row is sorted by channel, unused places last
      v.oidx[side][pool0 + start + k] = L.oidx[tid][k];
      v.oval[side][pool0 + start + k] = L.oval[tid][k];
    }
  }
}
// Class counts and bounds of a tile side (one thread; per wavefront: the value bound, or the ends of the key interval)
__device__ __forceinline__ void put_tile_summary(const QaqView& v, int side, size_t tile_id, const QaqCounts& cn, const float* bound, const float* bound2) {
  uint16_t* cp = v.counts + (tile_id * 2 + side) * 4;
  cp[QC3] = (uint16_t)cn.n3; cp[QC2] = (uint16_t)cn.n2; cp[QC4] = (uint16_t)cn.n4; cp[QC8] = (uint16_t)cn.n8;
  const float most = fmaxf(fmaxf(bound[0], bound[1]), fmaxf(bound[2], bound[3]));
  if (side == 1) v.vbound[tile_id] = most;
  else ((float2*)v.kthr)[tile_id] = make_float2(most, fminf(fminf(bound2[0], bound2[1]), fminf(bound2[2], bound2[3])));
}

// ---------------------------------------------------------------------------------
// A tile side that held nothing (bulk appends, prompt encoding, the first token of a tile).  Every token is encoded at
// eight bits, so the stored fields of every class are the same upper bits of a staged byte and the planes are put together
// by shifts that take all tokens of a word along (top_fields), one 4x4 byte transpose per four channels of 16 values; there is
// nothing to keep, to read back or to compare with, so none of the general path's bookkeeping.
//
// Bound by vector instructions (the search and the codes, see TokenEncoder), then by the fp16 rows it reads.  Vector instructions
// per wavefront 3240 -> 2600 by the encoder, -> 2020 by this form (through the general path before): 2 x 32 heads x 12001
// tokens 167 -> 140 -> 109 us = 4.2 TB/s, 16 x 8 heads x 8192 216 -> 143, 8 x 32 heads x 4096 at eight bits, in three chunks,
// 229 -> 197 -> 187.
// ---------------------------------------------------------------------------------

// FW upper bits below bit 8 - SKIP of the bytes of N = 8 / FW words -> fields of one word, the first word's lowest
template <int FW, int SKIP, int N>
__device__ __forceinline__ uint32_t top_fields(const uint32_t (&w)[N]) {
  constexpr uint32_t M = 0x01010101u * (((1u << FW) - 1u) << (8 - FW));
  uint32_t x = w[0] << SKIP;
#pragma unroll
  for (int i = 1; i < N; ++i) x = ((x >> FW) & ~M) | ((w[i] << SKIP) & M);
  return x;      // (what a shift brings in from the next byte is replaced in the same step; N steps replace every bit)
}

template <int D, int MAXO, bool HAS1>
__device__ __forceinline__ void pack_fresh(int side, uint8_t* base, const QaqCounts& c, const BuildLds<D, MAXO>& L, int tid) {
  constexpr int NQ = D / 16, KS = D / 64;
  const int n32 = c.n32();
  const uint8_t* const staged = (const uint8_t*)L.stage;
  auto row_of = [&](int slot) { return (const uint32_t*)(staged + L.row_of_slot[slot]); };
  if (side == 0) {
    const QaqKRegions r = qaq_k_regions(c, D);
    auto slice = [&](const uint32_t* row, int q) { return row + (16 * (q % KS) + 4 * (q / KS)); };
    for (int it = tid; it < n32 * (D / 64); it += kThreads) {          // four slices of a token: 16 bytes
      const uint32_t* row = row_of(it / (D / 64));
      const int q0 = 4 * (it % (D / 64));
      uint32_t o[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t* p = slice(row, q0 + k);
        const uint32_t w[4] = {p[0], p[1], p[2], p[3]};
        o[k] = top_fields<2, 0>(w);
      }
      *(uint4*)(base + r.r2 + 16u * (uint32_t)it) = make_uint4(o[0], o[1], o[2], o[3]);
    }
    auto low_word = [&](const uint32_t* row, int jj, auto skip) {      // slices 2 jj and 2 jj + 1, one bit each
      const uint32_t *p = slice(row, 2 * jj), *p1 = slice(row, 2 * jj + 1);
      const uint32_t w[8] = {p[0], p[1], p[2], p[3], p1[0], p1[1], p1[2], p1[3]};
      return top_fields<1, decltype(skip)::value>(w);
    };
    for (int it = tid; it < c.n3 * (D / 32); it += kThreads)
      *(uint32_t*)(base + r.r1 + 4u * (uint32_t)it) = low_word(row_of(it / (D / 32)), it % (D / 32), std::integral_constant<int, 2>{});
    for (int it = tid; it < c.n4 * (D / 32); it += kThreads) {         // two slices: 16 bytes
      const uint32_t* row = row_of(n32 + it / (D / 32));
      const uint32_t *p = slice(row, 2 * (it % (D / 32))), *p1 = slice(row, 2 * (it % (D / 32)) + 1);
      const uint32_t a[2] = {p[0], p[1]}, b[2] = {p[2], p[3]}, a1[2] = {p1[0], p1[1]}, b1[2] = {p1[2], p1[3]};
      *(uint4*)(base + r.r4 + 16u * (uint32_t)it) = make_uint4(top_fields<4, 0>(a), top_fields<4, 0>(b), top_fields<4, 0>(a1), top_fields<4, 0>(b1));
    }
    for (int it = tid; it < c.n8 * NQ; it += kThreads) {
      const uint32_t* p = slice(row_of(n32 + c.n4 + it / NQ), it % NQ);
      *(uint4*)(base + r.r8 + 16u * (uint32_t)it) = make_uint4(p[0] ^ 0x80808080u, p[1] ^ 0x80808080u, p[2] ^ 0x80808080u, p[3] ^ 0x80808080u);
    }
    for (int it = tid; HAS1 && it < c.n1 * (D / 32); it += kThreads)
      *(uint32_t*)(base + r.r1b + 4u * (uint32_t)it) = low_word(row_of(c.first1() + it / (D / 32)), it % (D / 32), std::integral_constant<int, 0>{});
    return;
  }
  // values: fields of slots past the end of a region are whatever those slots hold (no reader looks at them)
  const QaqVRegions r = qaq_v_regions(c, D);
  for (int it = tid; it < ((n32 + 15) / 16) * (D / 4); it += kThreads) {
    const int u = it / (D / 4), c4 = it % (D / 4), cg = c4 >> 2;
    const uint4* offs = (const uint4*)&L.row_of_slot[16 * u];
    const uint4 oa = offs[0], ob = offs[1];
    const uint32_t off[8] = {oa.x, oa.y, oa.z, oa.w, ob.x, ob.y, ob.z, ob.w};
    uint32_t w[16], m[4], o[4];
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] = *(const uint32_t*)(staged + ((off[i >> 1] >> (16 * (i & 1))) & 0xffffu) + 4 * c4);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t x[4] = {w[j], w[4 + j], w[8 + j], w[12 + j]};
      m[j] = top_fields<2, 0>(x);
    }
    transpose4(m, o);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      *(uint32_t*)(base + r.r2 + (uint32_t)u * (4 * D) + 4u * (uint32_t)((4 * (c4 & 3) + k) * (D / 16) + cg)) = o[k];
  }
  auto low_units = [&](uint32_t region, int first, int n, auto skip) {      // one bit of every token of units of 16 slots
    for (int it = tid; it < ((n + 15) / 16) * (D / 8); it += kThreads) {
      const int u = it / (D / 8), rest = it % (D / 8), cgp = rest >> 2, n4 = rest & 3;
      uint32_t m[4], o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t x[8];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const uint32_t* row = row_of(min(first + 16 * u + 4 * v + j, QAQ_TT - 1)) + (8 * cgp + n4);
          x[v] = row[0]; x[4 + v] = row[4];
        }
        m[j] = top_fields<1, decltype(skip)::value>(x);
      }
      transpose4(m, o);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        *(uint32_t*)(base + region + (uint32_t)u * (2 * D) + 4u * (uint32_t)((4 * n4 + k) * (D / 32) + cgp)) = o[k];
    }
  };
  low_units(r.r1, 0, c.n3, std::integral_constant<int, 2>{});
  for (int it = tid; it < ((c.n4 + 7) / 8) * (D / 4); it += kThreads) {
    const int hu = it / (D / 4), c4 = it % (D / 4), cg = c4 >> 2;
    uint32_t m[4], o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int s0 = n32 + 8 * hu + j;
      const uint32_t x[2] = {row_of(min(s0, QAQ_TT - 1))[c4], row_of(min(s0 + 4, QAQ_TT - 1))[c4]};
      m[j] = top_fields<4, 0>(x);
    }
    transpose4(m, o);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      *(uint32_t*)(base + r.r4 + (uint32_t)hu * (4 * D) + 4u * (uint32_t)((4 * (c4 & 3) + k) * (D / 16) + cg)) = o[k];
  }
  for (int it = tid; it < c.n8 * (D / 16); it += kThreads) {
    const uint32_t* p = row_of(n32 + c.n4 + it / (D / 16)) + 4 * (it % (D / 16));
    *(uint4*)(base + r.r8 + 16u * (uint32_t)it) = make_uint4(p[0], p[1], p[2], p[3]);
  }
  if (HAS1) low_units(r.r1b, c.first1(), c.n1, std::integral_constant<int, 0>{});
}

// ---- what a fresh tile side and one that is written anew as a whole have in common ----
// Slots by class, in position order inside a class (thread t: position t, its class or -1).  Afterwards, behind a barrier,
// row_of_slot holds the staged rows' byte offsets and `order` the positions, by slot; slots past the last token: row 0.
template <int D, int MAXO, bool HAS1>
__device__ __forceinline__ void sort_slots(int cls, QaqCounts& cn, BuildLds<D, MAXO>& L, int tid) {
  constexpr int NC = HAS1 ? QAQ_NCLASS : 4, ROW = 4 * BuildLds<D, MAXO>::SROW;
  const int lane = tid & 63, wave = tid >> 6;
  int rank = 0;
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const unsigned long long bal = __ballot(cls == k);
    if (lane == 0) L.wave_cnt[k][wave] = __popcll(bal);
    rank = cls == k ? lanes_below(bal) : rank;
  }
  L.row_of_slot[tid] = 0;
  __syncthreads();
  int m[QAQ_NCLASS];
  m[QC1] = 0;
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) { const int x = __builtin_amdgcn_readfirstlane(L.wave_cnt[k][w]); before += w < wave ? x : 0; all += x; }
    m[k] = all;
    rank += cls == k ? before : 0;
  }
  cn.n3 = m[QC3]; cn.n2 = m[QC2]; cn.n4 = m[QC4]; cn.n8 = m[QC8]; cn.n1 = m[QC1];
  if (cls >= 0) {
    const int sl = cn.start(cls) + rank;
    L.row_of_slot[sl] = (uint16_t)(tid * ROW);
    L.order[sl] = (uint8_t)tid;
  }
}
// Metadata in slot order, the tile's summary, the code planes (positions n_before .. n - 1 are new)
template <int D, bool ONE, bool HAS1>
__device__ __forceinline__ void put_sorted(const QaqView& v, int side, int bh, int tile, int n_before, int n, const QaqCounts& cn, BuildLds<D, ONE ? 2 : QAQ_MAX_NO2>& L, int tid) {
  constexpr int MAXO = ONE ? 2 : QAQ_MAX_NO2;
  const bool csr = !ONE && v.csr;
  const int b = bh / v.Hkv, h = bh % v.Hkv;
  const size_t gi0 = qaq_slot_index(v, b, h, tile, 0);
  if (tid < n) {
    const int p = L.order[tid];
    v.mm[side][gi0 + tid] = L.mm[p];
    v.perm[side][gi0 + tid] = (uint8_t)p;
    if (ONE) {
      *(uint16_t*)(v.oidx[side] + (gi0 + tid) * 2) = *(const uint16_t*)L.oidx[p];
      *(uint32_t*)(v.oval[side] + (gi0 + tid) * 2) = *(const uint32_t*)L.oval[p];
    } else {
      for (int k = 0; k < v.no2 && !csr; ++k) {
        v.oidx[side][(gi0 + tid) * v.no2 + k] = L.oidx[p][k];
        v.oval[side][(gi0 + tid) * v.no2 + k] = L.oval[p][k];
      }
    }
  }
  if (csr && n > n_before) put_new_runs<D, MAXO>(v, side, gi0, n_before, n, L, tid);
  if (tid == 0) put_tile_summary(v, side, qaq_bh(v, b, h) * v.NT + tile, cn, L.wave_bound, L.wave_bound2);
  pack_fresh<D, MAXO, HAS1>(side, qaq_tile_codes(v, side, b, h, tile), cn, L, tid);
}

// All stored codes of a tile side -> staged bytes, a code in the upper bits of its byte (what is below it is left to
// chance: a token's width never grows here).
template <int D, int MAXO, bool HAS1>
__device__ __forceinline__ void unpack_all(int side, const uint8_t* base, const QaqCounts& c, BuildLds<D, MAXO>& L, int tid) {
  constexpr int NQ = D / 16, KS = D / 64;
  const int n32 = c.n32();
  uint8_t* const staged = (uint8_t*)L.stage;
  constexpr uint32_t LOW = 0x20202020u;
  if (side == 0) {
    const QaqKRegions r = qaq_k_regions(c, D);
    auto slice = [&](int slot, int q) { return (uint32_t*)(staged + L.row_of_old[slot]) + (16 * (q % KS) + 4 * (q / KS)); };
#pragma unroll 2
    for (int it = tid; it < n32 * NQ; it += kThreads) {
      const int s = it / NQ, q = it % NQ;
      const uint32_t w2 = *(const uint32_t*)(base + (r.r2 + 4u * (uint32_t)it));
      const uint32_t w1 = *(const uint32_t*)(base + (s < c.n3 ? r.r1 + (uint32_t)s * (D / 8) + 4u * (uint32_t)(q >> 1) : r.r2)) >> (4 * (q & 1));
      uint32_t* row = slice(s, q);
#pragma unroll
      for (int v = 0; v < 4; ++v) row[v] = ((w2 << (6 - 2 * v)) & ~LOW) | ((w1 << (5 - v)) & LOW);
    }
    for (int it = tid; it < c.n4 * NQ; it += kThreads) {
      const uint2 w = *(const uint2*)(base + (r.r4 + 8u * (uint32_t)it));
      uint32_t* row = slice(n32 + it / NQ, it % NQ);
      row[0] = w.x << 4; row[1] = w.x; row[2] = w.y << 4; row[3] = w.y;
    }
    for (int it = tid; it < c.n8 * NQ; it += kThreads) {
      const uint4 w = *(const uint4*)(base + (r.r8 + 16u * (uint32_t)it));
      uint32_t* row = slice(n32 + c.n4 + it / NQ, it % NQ);
      row[0] = w.x ^ 0x80808080u; row[1] = w.y ^ 0x80808080u; row[2] = w.z ^ 0x80808080u; row[3] = w.w ^ 0x80808080u;
    }
    for (int it = tid; HAS1 && it < c.n1 * NQ; it += kThreads) {
      const int s = it / NQ, q = it % NQ;
      const uint32_t w = *(const uint32_t*)(base + (r.r1b + (uint32_t)s * (D / 8) + 4u * (uint32_t)(q >> 1))) >> (4 * (q & 1));
      uint32_t* row = slice(c.first1() + s, q);
#pragma unroll
      for (int v = 0; v < 4; ++v) row[v] = w << (7 - v);
    }
    return;
  }
  const QaqVRegions r = qaq_v_regions(c, D);
  auto words = [&](uint32_t at, int stride, uint32_t (&m)[4]) {      // four channels' words -> per token of a group of four
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = *(const uint32_t*)(base + (at + (uint32_t)(4 * k * stride)));
    transpose4(w, m);
  };
  for (int it = tid; it < ((n32 + 15) / 16) * (D / 4); it += kThreads) {
    const int u = it / (D / 4), c4 = it % (D / 4), cg = c4 >> 2, n0 = 4 * (c4 & 3);
    const uint4* offs = (const uint4*)&L.row_of_old[16 * u];
    const uint4 oa = offs[0], ob = offs[1];
    const uint32_t off[8] = {oa.x, oa.y, oa.z, oa.w, ob.x, ob.y, ob.z, ob.w};
    uint32_t m[4], l[4] = {0u, 0u, 0u, 0u};
    words(r.r2 + (uint32_t)u * (4 * D) + 4u * (uint32_t)(n0 * (D / 16) + cg), D / 16, m);
    if (16 * u < c.n3) {
      words(r.r1 + (uint32_t)u * (2 * D) + 4u * (uint32_t)(n0 * (D / 32) + (cg >> 1)), D / 32, l);
#pragma unroll
      for (int j = 0; j < 4; ++j) l[j] >>= 4 * (cg & 1);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {            // token 4 v + j of the unit
      const int j = i & 3, v = i >> 2;
      if (16 * u + i < n32) *(uint32_t*)(staged + ((off[i >> 1] >> (16 * (i & 1))) & 0xffffu) + 4 * c4) = ((m[j] << (6 - 2 * v)) & ~LOW) | ((l[j] << (5 - v)) & LOW);
    }
  }
  for (int it = tid; it < ((c.n4 + 7) / 8) * (D / 4); it += kThreads) {
    const int hu = it / (D / 4), c4 = it % (D / 4);
    uint32_t m[4];
    words(r.r4 + (uint32_t)hu * (4 * D) + 4u * (uint32_t)(4 * (c4 & 3) * (D / 16) + (c4 >> 2)), D / 16, m);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (8 * hu + i < c.n4) *(uint32_t*)(staged + L.row_of_old[n32 + 8 * hu + i] + 4 * c4) = i < 4 ? m[i & 3] << 4 : m[i & 3];
  }
  for (int it = tid; it < c.n8 * (D / 16); it += kThreads) {
    const uint4 w = *(const uint4*)(base + (r.r8 + 16u * (uint32_t)it));
    uint32_t* row = (uint32_t*)(staged + L.row_of_old[n32 + c.n4 + it / (D / 16)]) + 4 * (it % (D / 16));
    row[0] = w.x; row[1] = w.y; row[2] = w.z; row[3] = w.w;
  }
  for (int it = tid; HAS1 && it < ((c.n1 + 15) / 16) * (D / 4); it += kThreads) {
    const int u = it / (D / 4), c4 = it % (D / 4), cg = c4 >> 2;
    uint32_t m[4];
    words(r.r1b + (uint32_t)u * (2 * D) + 4u * (uint32_t)(4 * (c4 & 3) * (D / 32) + (cg >> 1)), D / 32, m);
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (16 * u + i < c.n1) *(uint32_t*)(staged + L.row_of_old[c.first1() + 16 * u + i] + 4 * c4) = (m[i & 3] >> (4 * (cg & 1))) << (7 - (i >> 2));
  }
}

template <int D, bool ONE, bool HAS1>
__device__ __forceinline__ void fresh_tile(const QaqBuildArgs& a, BuildLds<D, ONE ? 2 : QAQ_MAX_NO2>& L, const int bh, const int tile, const int side, const int tid) {
  constexpr int MAXO = ONE ? 2 : QAQ_MAX_NO2, ROW = 4 * BuildLds<D, MAXO>::SROW;
  typedef TokenEncoder<D, ONE> Enc;
  const QaqView& v = a.v;
  const QaqRuleArgs& ru = a.rule;
  const bool csr = !ONE && v.csr;
  const int lane = tid & 63, wave = tid >> 6;
  const int b = bh / v.Hkv, h = bh % v.Hkv, t0 = tile * QAQ_TT;
  const int len_before = qaq_seq_len(v, b, a.len_before), n_new0 = t0 - len_before;      // (position 0 is new token n_new0)
  const int n = min(qaq_seq_len(v, b, a.len_after) - t0, QAQ_TT);
  const size_t gi0 = qaq_slot_index(v, b, h, tile, 0);

  // encode: a quad of lanes per token, 64 tokens per pass, the next pass's rows requested before the current one's are used
  const uint8_t* const rows = (const uint8_t*)a.newx[side] + ((long long)bh * a.n_new + n_new0) * (2 * D);
  uint8_t* const put = a.orig_put[side] ? (uint8_t*)a.orig_put[side] + ((long long)bh * a.orig_tokens + t0) * (2 * D) : nullptr;
  const float thr_lo = csr ? v.othr[(side * v.Hkv + h) * 2] : INFINITY, thr_hi = csr ? v.othr[(side * v.Hkv + h) * 2 + 1] : -INFINITY;
  constexpr int TPP = kThreads / 4;
  const int NP = (n + TPP - 1) / TPP, c = tid & 3, gt = tid >> 2;
  auto fetch = [&](int pass, uint4 (&raw)[Enc::NCH]) {
    const int p = pass * TPP + gt;
    const uint32_t at = (uint32_t)min(p, n - 1) * (2 * D) + 16u * (uint32_t)c;
#pragma unroll
    for (int i = 0; i < Enc::NCH; ++i) {        // read once: streaming loads
      const u32x4 t = __builtin_nontemporal_load((const u32x4*)(rows + (at + 64 * i)));
      raw[i] = make_uint4(t.x, t.y, t.z, t.w);
    }
    if (put && p < n) {                         // keep the unquantized token for later widening
#pragma unroll
      for (int i = 0; i < Enc::NCH; ++i) *(uint4*)(put + (at + 64 * i)) = raw[i];
    }
  };
  auto encode = [&](int pass, const uint4 (&raw)[Enc::NCH]) {
    const int p = pass * TPP + gt;
    if (p < n) Enc::run(raw, c, true, v.no2 / 2, &L.mm[p], L.oidx[p], L.oval[p], (uint32_t*)((uint8_t*)L.stage + p * ROW), thr_lo, thr_hi);
  };
  uint4 cur[Enc::NCH], nxt[Enc::NCH];
  fetch(0, cur);
  // the window's part of the value rule (thread t: position t), or the widths given
  float pred = 0.0f;
  int bits = a.widest;
  if (a.mode >= 2 && side == 1 && tid < n) {
    const int t = t0 + tid;
    const size_t ri = qaq_bh(v, b, h) * v.Tmax + t;
    float s = 0.0f;
    if (a.mode == 2)
      for (int g = 0; g < ru.G; ++g) s = fmaxf(s, ru.scores[((size_t)b * v.Hq + (h * ru.G + g)) * ru.score_stride + t]);
    s = qaq_ring_value(v, s);
    pred = qaq_window_max_compact(v, qaq_rows_covering(v, ru.row_len, b, t), ru.new_row, ri, s);
    if (a.mode == 2) qaq_ring_store(v, (size_t)ru.new_row * ((size_t)v.B * v.Hkv * v.Tmax) + ri, s);
  } else if (a.mode == 0 && a.newbits[side] && tid < n) {
    bits = a.newbits[side][(size_t)bh * a.n_new + (n_new0 + tid)];
  }
#pragma unroll 1
  for (int pass = 0; pass < NP; ++pass) {
    if (pass + 1 < NP) fetch(pass + 1, nxt);
    encode(pass, cur);
#pragma unroll
    for (int i = 0; i < Enc::NCH; ++i) cur[i] = nxt[i];
  }
  __syncthreads();

  // widths, the tile's bounds, classes (thread t: position t)
  int cls = -1;
  {
    float bnd = 0.0f, lo = 0.0f, hi = INFINITY;
    if (tid < n) {
      const uint32_t m = L.mm[tid];
      const float mn = h2f((uint16_t)(m & 0xffffu)), mx = h2f((uint16_t)(m >> 16)), range = mx - mn;
      if (a.mode >= 2) {
        bits = rule_width(ru, side == 0 ? range : range * pred, side == 0 ? qaq_tau_k(ru, v, b, h) : qaq_c_v(ru, v, b));
        if (ru.out_bits[side]) ru.out_bits[side][(a.mode == 2 ? (size_t)bh * a.len_after + t0 : (size_t)bh * a.n_new + n_new0) + tid] = (uint8_t)bits;
      }
      v.tags[side][gi0 + tid] = (uint8_t)bits;
      cls = qaq_class_of_bits(bits);
      if (!ONE) sort_side_store(L.oidx[tid], L.oval[tid], v.no2);
      if (side == 1) bnd = value_bound(bits, mn, mx, L.oidx[tid], L.oval[tid], v.no2);
      else key_interval(ru, bits, range, lo, hi);
    }
    if (side == 1) {
      bnd = wave_max(bnd);
      if (lane == 0) L.wave_bound[wave] = bnd;
    } else {
      lo = wave_max(lo); hi = wave_min(hi);
      if (lane == 0) { L.wave_bound[wave] = lo; L.wave_bound2[wave] = hi; }
    }
  }
  QaqCounts cn;
  sort_slots<D, MAXO, HAS1>(cls, cn, L, tid);
  __syncthreads();
  put_sorted<D, ONE, HAS1>(v, side, bh, tile, 0, n, cn, L, tid);
}

// HAS1: the width set contains 1 (five classes); without it the fifth class costs nothing.
// One tile side (unit bh, tile, side) that holds tokens: appends to it, moves its tokens to other widths.  tid: the thread
// (an argument: see k_build_listed).
//
// A side with nothing to do is left after its widths are known.  Any other is read into LDS and written anew in the manner
// of a fresh one, with the tokens that are new or widen encoded in between.  Moving only the tokens that change (the
// decode-step kernel's way, with few registers) was not worth its bookkeeping here: 8 x 32 heads x 4000 tokens, 0.5 % of the
// tokens changed 93 -> 74 us, 5 % 154 -> 102, half of them 198 -> 106, all 225 -> 122; two outliers per end 157 -> 95 ... 392 -> 161.
template <int D, bool ONE, bool HAS1>
__device__ __forceinline__ void build_tile(const QaqBuildArgs& a, BuildLds<D, ONE ? 2 : QAQ_MAX_NO2>& L, const int bh, const int tile, const int side, const int tid) {
  constexpr int MAXO = ONE ? 2 : QAQ_MAX_NO2, ROW = 4 * BuildLds<D, MAXO>::SROW;
  typedef TokenEncoder<D, ONE> Enc;
  const QaqView& v = a.v;
  const QaqRuleArgs& ru = a.rule;
  const bool csr = !ONE && v.csr;     // (the one-per-end build never has the variable-length side store)
  const int lane = tid & 63, wave = tid >> 6;
  const int b = bh / v.Hkv, h = bh % v.Hkv;
  const int t0 = tile * QAQ_TT;
  const int len_before = qaq_seq_len(v, b, a.len_before), len_after = qaq_seq_len(v, b, a.len_after);   // of this sequence
  const int n_before = min(max(len_before - t0, 0), QAQ_TT);
  const int n_after = min(max(len_after - t0, 0), QAQ_TT);

  if (a.mode == 1 && a.newbits[side] == nullptr) return;   // requantize: nothing to do for this side
  // an append, where sequences differ in length: the grid starts at the shortest sequence's open
  // tile, which a longer sequence may have filled already
  if ((a.mode == 0 || a.mode == 3) && n_before == n_after) return;

  // decode-step update, key side: the rule compares a token's range with one threshold per
  // (T, head); the tile keeps, from when it was built, the interval of thresholds for which
  // none of its tokens changes width, so a tile with nothing to do costs one 8-byte load
  const size_t tile_id = qaq_bh(v, b, h) * v.NT + tile;
  if (a.mode == 2 && side == 0 && n_before == n_after && !ru.out_bits[0]) {
    const float2 keep = ((const float2*)v.kthr)[tile_id];
    const float tau = qaq_tau_k(ru, v, b, h);
    if (tau >= keep.x && tau < keep.y) return;
  }

  // everything whose address is known up front is requested in one go: the slot-order metadata, and what the
  // widths come from (for a requantize the widths themselves)
  const uint8_t* const base = qaq_tile_codes(v, side, b, h, tile);
  QaqCounts c_old = qaq_load_counts(v, side, b, h, tile, n_before);
  if (!HAS1) c_old.n1 = 0;
  const size_t gi0 = qaq_slot_index(v, b, h, tile, 0);
  const bool cached = tid < n_before, fresh = tid >= n_before && tid < n_after;
  int pos_old = 0;
  uint32_t mm_old = 0;
  uint8_t oi_old[MAXO];
  uint16_t ov_old[MAXO];
  if (cached) {
    pos_old = v.perm[side][gi0 + tid];
    mm_old = v.mm[side][gi0 + tid];
#pragma unroll
    for (int k = 0; k < MAXO; ++k)
      if (k < v.no2 && !csr) { oi_old[k] = v.oidx[side][(gi0 + tid) * v.no2 + k]; ov_old[k] = v.oval[side][(gi0 + tid) * v.no2 + k]; }
  }
  // the inputs of the width rules that are indexed by position (this step's scores, the window rows); the value side
  // keeps the window (an append by the rules, mode 3, takes the window as it stands and writes no row)
  float pred = 0.0f;
  int oldb = 0, want = a.widest;        // of position tid: width so far, width asked for
  if (side == 1 && ((a.mode == 2 && tid < n_after) || (a.mode == 3 && fresh))) {
    const int t = t0 + tid;
    const size_t ring_row = (size_t)v.B * v.Hkv * v.Tmax;
    const size_t ri = qaq_bh(v, b, h) * v.Tmax + t;
    // (the scores row by row, the window's rows at once, in the compact form: the decode-step kernel's
    // form with its variants by row count makes this kernel call its helpers out of line)
    float s = 0.0f;
    if (a.mode == 2)
      for (int g = 0; g < ru.G; ++g) s = fmaxf(s, ru.scores[((size_t)b * v.Hq + (h * ru.G + g)) * ru.score_stride + t]);
    s = qaq_ring_value(v, s);
    pred = qaq_window_max_compact(v, qaq_rows_covering(v, ru.row_len, b, t), ru.new_row, ri, s);
    if (a.mode == 2) qaq_ring_store(v, (size_t)ru.new_row * ring_row + ri, s);
  }
  if (a.mode == 1 && cached) {
    oldb = v.tags[side][gi0 + tid];
    want = a.newbits[side][(size_t)bh * a.len_before + t0 + tid];
  } else if (a.mode == 0 && fresh && a.newbits[side]) {
    want = a.newbits[side][(size_t)bh * a.n_new + (t0 + tid - len_before)];
  }
  const bool served = a.orig[side] != nullptr;
  bool wider = false, changed = false;
  if (a.mode == 1) {
    // no token of the tile changes: leave it alone
    wider = cached && want > oldb;
    changed = cached && (want < oldb || (wider && served));
    note_widenings(L.wave_wide, wider, tid);
    const bool any = __syncthreads_or(changed ? 1 : 0) != 0;
    if (tid == 0) add_widenings(v, tile_id * 2 + side, L.wave_wide, served);
    if (!any) return;
  }

  // metadata by position
  if (cached) {
    L.mm[pos_old] = mm_old;
    L.row_of_old[tid] = (uint16_t)pos_old;       // (the position until it is known which rows are encoded)
    L.bits_old[pos_old] = (uint8_t)(HAS1 ? c_old.bits_of_slot(tid) : c_old.bits_of_slot4(tid));
#pragma unroll
    for (int k = 0; k < MAXO; ++k)
      if (k < v.no2 && !csr) { L.oidx[pos_old][k] = oi_old[k]; L.oval[pos_old][k] = ov_old[k]; }
  }
  // variable-length side store: the tile's pool is in position order and a token's entries never
  // move; thread `tid` fetches those of position tid (unused places of its row: channel 255)
  if (csr && cached) {
    const size_t pool0 = gi0 * (size_t)v.no2;
    const int cnt = v.ocnt[side][gi0 + tid], st = v.ostart[side][gi0 + tid];
#pragma unroll
    for (int k = 0; k < MAXO; ++k) {
      const bool have = k < cnt;
      L.oidx[tid][k] = have ? v.oidx[side][pool0 + st + k] : (uint8_t)0xffu;
      L.oval[tid][k] = have ? v.oval[side][pool0 + st + k] : (uint16_t)0;
    }
  }
  __syncthreads();

  // decode-step update: widths of the cached positions by the rules; the tile is left alone
  // if none of them moves and the new token is not in it
  auto ruled_width = [&](uint32_t m) {
    const float range = h2f((uint16_t)(m >> 16)) - h2f((uint16_t)(m & 0xffffu));
    return rule_width(ru, side == 0 ? range : range * pred, side == 0 ? qaq_tau_k(ru, v, b, h) : qaq_c_v(ru, v, b));
  };
  if (cached) oldb = L.bits_old[tid];
  if (a.mode == 2) {
    if (cached) {
      want = ruled_width(L.mm[tid]);
      if (ru.out_bits[side]) ru.out_bits[side][(size_t)bh * a.len_after + t0 + tid] = (uint8_t)want;
    }
    wider = cached && want > oldb;
    changed = cached && (want < oldb || (wider && served));
    note_widenings(L.wave_wide, wider, tid);
    const bool any = __syncthreads_or(changed ? 1 : 0) != 0;
    if (tid == 0) add_widenings(v, tile_id * 2 + side, L.wave_wide, served);
    if (!any && n_before == n_after) return;
  }

  // width of every position (appends leave the cached tokens at theirs; a new token's by the rules follows from its
  // range); whether it is encoded: new tokens, and cached ones that widen from the unquantized copy
  int bits = cached && !changed ? oldb : want;
  const bool enc = fresh || (changed && wider);
  const unsigned long long enc_bal = __ballot(enc);
  if (lane == 0) L.wave_enc[wave] = __popcll(enc_bal);
  __syncthreads();
  // encode: a quad of lanes per token, 64 tokens per pass, the positions gathered into a list so that they fill
  // the passes densely; the rows of the next pass are requested before the current pass is computed
  const int n_enc = L.wave_enc[0] + L.wave_enc[1] + L.wave_enc[2] + L.wave_enc[3];
  {
    int off = 0;
    for (int w = 0; w < wave; ++w) off += L.wave_enc[w];
    if (enc) L.order[off + lanes_below(enc_bal)] = (uint8_t)tid;
  }
  // staged rows by old slot (what is encoded is not staged from its old code); the widths' place now says who is encoded
  L.bits_old[tid] = enc ? 1 : 0;
  __syncthreads();
  {
    const int p = cached ? (int)L.row_of_old[tid] : QAQ_TT;
    L.row_of_old[tid] = (uint16_t)((p < QAQ_TT && !L.bits_old[p] ? p : QAQ_TT) * ROW);
  }
  if (n_enc > 0) {                           // uniform: every thread has the same sum
    const float thr_lo = csr ? v.othr[(side * v.Hkv + h) * 2] : INFINITY;
    const float thr_hi = csr ? v.othr[(side * v.Hkv + h) * 2 + 1] : -INFINITY;
    constexpr int TPP = kThreads / 4;     // tokens per pass
    const int NP = (n_enc + TPP - 1) / TPP;
    const int c = tid & 3, gt = tid >> 2;
    auto position = [&](int pass) { return (int)L.order[min(pass * TPP + gt, QAQ_TT - 1)]; };
    // rows by position of this tile (the new tokens' first row is that of position n_before)
    const uint8_t* const new_rows = (const uint8_t*)a.newx[side] + ((long long)bh * a.n_new + (t0 - len_before)) * (2 * D);
    const uint8_t* const old_rows = (const uint8_t*)a.orig[side] + ((long long)bh * a.orig_tokens + t0) * (2 * D);
    uint8_t* const put_rows = a.orig_put[side] ? (uint8_t*)a.orig_put[side] + ((long long)bh * a.orig_tokens + t0) * (2 * D) : nullptr;
    auto fetch = [&](int pass, uint4 (&raw)[Enc::NCH]) -> int {   // 0 = nothing to do, 1 = fresh, 2 = widen
      if (pass >= NP || pass * TPP + gt >= n_enc) return 0;
      const int p = position(pass);
      const bool is_new = p >= n_before;
      const uint32_t at = (uint32_t)p * (2 * D) + 16u * (uint32_t)c;
      const uint8_t* src = (is_new ? new_rows : old_rows) + at;
#pragma unroll
      for (int i = 0; i < Enc::NCH; ++i) {      // read once: streaming loads
        const u32x4 t = __builtin_nontemporal_load((const u32x4*)(src + 64 * i));
        raw[i] = make_uint4(t.x, t.y, t.z, t.w);
      }
      if (is_new && put_rows) {            // keep the unquantized token for later widening
#pragma unroll
        for (int i = 0; i < Enc::NCH; ++i) *(uint4*)(put_rows + at + 64 * i) = raw[i];
      }
      return is_new ? 1 : 2;
    };
    uint4 cur[Enc::NCH], nxt[Enc::NCH];
    int kind = fetch(0, cur);
#pragma unroll 1
    for (int pass = 0; pass < NP; ++pass) {
      const int kind_next = fetch(pass + 1, nxt);
      if (kind) {                          // whole quads drop out together
        const int p = position(pass);
        Enc::run(cur, c, kind == 1, v.no2 / 2, &L.mm[p], L.oidx[p], L.oval[p], (uint32_t*)((uint8_t*)L.stage + p * ROW), thr_lo, thr_hi);
      }
#pragma unroll
      for (int i = 0; i < Enc::NCH; ++i) cur[i] = nxt[i];
      kind = kind_next;
    }
    __syncthreads();
  }

  // the width of a new token by the rules, the tile's bounds, classes
  int cls = -1;
  {
    float bnd = 0.0f, lo = 0.0f, hi = INFINITY;
    if (tid < n_after) {
      const uint32_t m = L.mm[tid];
      const float mn = h2f((uint16_t)(m & 0xffffu)), mx = h2f((uint16_t)(m >> 16));
      if (fresh && a.mode >= 2) {
        bits = ruled_width(m);
        if (ru.out_bits[side]) ru.out_bits[side][(a.mode == 2 ? (size_t)bh * a.len_after + t0 : (size_t)bh * a.n_new + (t0 - len_before)) + tid] = (uint8_t)bits;
      }
      if (fresh || changed) v.tags[side][gi0 + tid] = (uint8_t)bits;
      cls = qaq_class_of_bits(bits);
      if (!ONE && fresh) sort_side_store(L.oidx[tid], L.oval[tid], v.no2);
      if (side == 1) bnd = value_bound(bits, mn, mx, L.oidx[tid], L.oval[tid], v.no2);
      else key_interval(ru, bits, mx - mn, lo, hi);
    }
    if (side == 1) {
      bnd = wave_max(bnd);
      if (lane == 0) L.wave_bound[wave] = bnd;
    } else {
      lo = wave_max(lo); hi = wave_min(hi);
      if (lane == 0) { L.wave_bound[wave] = lo; L.wave_bound2[wave] = hi; }
    }
  }
  QaqCounts cn;
  sort_slots<D, MAXO, HAS1>(cls, cn, L, tid);
  // (with every token of the side encoded there is nothing to keep: 8 x 32 heads x 4000 tokens all widened 214 us with the old
  // codes read all the same, 176 without; 198 when only moved tokens were handled)
  if (n_enc < n_after) unpack_all<D, MAXO, HAS1>(side, base, c_old, L, tid);
  __syncthreads();
  put_sorted<D, ONE, HAS1>(v, side, bh, tile, n_before, n_after, cn, L, tid);
}

// Grid (units, tiles, 2 sides) -- heads are the fastest grid dimension: with tiles fastest and a
// tile count that is a multiple of eight, every die would see the same two tile indices of every
// head, which ran 30 % slower.
template <int D, bool ONE, bool HAS1>
__global__ __launch_bounds__(kThreads, (D == 64 && ONE ? 7 : 1)) void k_build(QaqBuildArgs a) {      // (the narrow form at 75 registers without a bound: six wavefronts per SIMD)
  qaq_request_arguments<0, offsetof(QaqBuildArgs, rule) + offsetof(QaqRuleArgs, c_v)>();
  __shared__ BuildLds<D, ONE ? 2 : QAQ_MAX_NO2> L;
  const int tile = a.tile0 + (int)blockIdx.y, t0 = tile * QAQ_TT, b = (int)blockIdx.x / a.v.Hkv;
  if (qaq_seq_len(a.v, b, a.len_after) <= t0) return;
  if (qaq_seq_len(a.v, b, a.len_before) <= t0) fresh_tile<D, ONE, HAS1>(a, L, (int)blockIdx.x, tile, (int)blockIdx.z, (int)threadIdx.x);
  else build_tile<D, ONE, HAS1>(a, L, (int)blockIdx.x, tile, (int)blockIdx.z, (int)threadIdx.x);
}

// The same for a list of tile sides (a.todo: entries (unit * NT + tile) * 2 + side, a.todo_count[0] of
// them, both in device memory): a one-dimensional grid whose workgroups share out the entries.  The last
// workgroup to finish leaves the list empty for the next step, whichever step that is (a captured run of
// steps may be replayed from its start); a workgroup that starts after that had no entry anyway.
//
// Bound by the workgroups in flight, i.e. by registers: left to itself the compiler keeps everything that
// follows from the thread or from the kernel's arguments in registers across the loop (142-247 of them when that was tried).
// So each round takes the thread's index and the arguments as if they were new: 80 | 108 registers at 64 channels, 119 | 168 at
// 128 (one outlier per end | other forms, which keep up to 21 scalars in lanes of vector registers), no scratch.  With the
// grid of launch_update, a step of 8 x 32 heads x 4000 tokens that hands half of the sides over takes 145-159 us (274-306 when
// the general build moved token by token; 64 channels 115-120, 202-216 then).
template <int D, bool ONE>
constexpr int listed_per_cu() { return D == 128 ? (ONE ? 4 : 3) : (ONE ? 5 : 4); }      // workgroups a compute unit takes
template <int D, bool ONE, bool HAS1>
__global__ __launch_bounds__(kThreads, (listed_per_cu<D, ONE>())) void k_build_listed(QaqBuildArgs a) {
  __shared__ BuildLds<D, ONE ? 2 : QAQ_MAX_NO2> L;
  const uint32_t n = *a.todo_count;
  if (blockIdx.x >= n) return;
  qaq_request_arguments<0, offsetof(QaqBuildArgs, rule) + offsetof(QaqRuleArgs, c_v)>();
#pragma unroll 1
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const uint32_t e = a.todo[i];
    const QaqBuildArgs* args = qaq_arguments_anew<QaqBuildArgs>();
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    build_tile<D, ONE, HAS1>(*args, L, (int)((e >> 1) / (uint32_t)args->v.NT), (int)((e >> 1) % (uint32_t)args->v.NT), (int)(e & 1u), tid);
    __syncthreads();        // the next tile side reuses the staging memory
  }
  // (every wavefront of a workgroup with entries has read the count: there was a barrier since)
  if (threadIdx.x == 0 && atomicAdd(&a.todo_count[2], 1u) + 1u == min(n, gridDim.x)) {
    a.todo_count[0] = 0u; a.todo_count[1] = n; a.todo_count[2] = 0u;
  }
}

// ---------------------------------------------------------------------------------
// Decode-step update (Section 4.2 "Integration in text generation process": the part of a step
// after the attention).  Same result as build_tile in mode 2, built for what a decode step does to
// a tile: a few tokens change width, one token is appended to the last tile, everything else stays.
//
// Two wavefronts per tile side, two tokens per lane (k_update), where the value sides fill the chip; where they do not,
// four, one token per lane (k_update_few).  What bounds the update is the chain of dependent
// steps of a tile side -- metadata, widths, codes of the tokens that move, read-modify-write of the words
// they go to -- and the instructions spent on all 256 tokens of a tile to move the dozen that change.  Half
// as many wavefronts as tokens / 64 evaluate what is uniform over the tile half as often and leave room for
// sixteen tile sides per compute unit (10 KB of LDS, 64 registers), so that all value sides of a 4096-token
// layer of 256 heads are in flight at once.
//
// A tile side with nothing to do is left after one 8-byte load (keys) or after the rules.  Slots are
// re-assigned so that as few tokens move as possible: a token keeps its index inside its class's
// region.  A region whose start moves (a class count before it crossed a multiple of 16) is copied as
// a whole, 16 bytes per lane, up to kMaxCopy bytes of them; only the codes of the tokens that change
// class, are squeezed out or arrive go through LDS.  Tile sides in which more tokens move than the launch
// has staging memory for (a hyper-parameter that jumped) are handed to the general kernel through a list.
//
// Measured, kernel trace, against four wavefronts per tile side with one token per lane: 8 x 32 heads x 4096 tokens
// 42.1 -> 33.4 us, 16 x 8 heads x 8192 with 8 query heads each 39.3 -> 32.0, 8 heads x 512 tokens 11.9 -> 11.4; with
// outliers by thresholds (the general kernel until then) 3 x 16 heads x 2500 34 -> 15.9.  Of that the slots were 10 us,
// 580 scalar instructions per wavefront for masks class by class; as compares per lane and one list of free slots: 33.4 -> 30.
// Vector and scalar instructions fill two thirds of the issue slots each.  With indices in 32 bits, the window's rows without
// a look at their ends where all cover the tile, one load of scores where a KV head has one query head and class counts in pairs a
// wavefront has 15 % fewer scalar ones (517 -> 438), compute units are busy 7 % less, and 24 steps of a small model take 436 instead of 453 us.
// With the taken slots worked out from the old ones (not marked in LDS behind a barrier), 2- and 3-bit slots without a look at the
// rest, the moved tokens' slots beside the gathering of their codes and every value region from another wavefront on, 8 x 32 heads x
// 4096 tokens 29.4 -> 27.7 us, 16 x 8 x 8192 29.0 -> 27.8 (kernel trace).
//
// Where a compute unit has few tile sides, an instruction that waits for the one before it takes eight cycles and nothing
// else fills them: a side's way is its instructions and some five trips to memory.  Four wavefronts halve what a lane does for
// the tile; two of them look at the window, the last one encodes the appended token, whose row is asked for with everything else.
// Two | four wavefronts, kernel trace: 8 heads x 512 tokens of 64 channels 9.7 | 7.9 us, 6 x 12 heads of 336 to 1901 tokens
// with the copies in host memory 16.1 | 12.0, outliers by thresholds, 3 x 16 x 2500, 15.4 | 11.3.
// ---------------------------------------------------------------------------------
constexpr int kMaxCopy = 8192;
// Four wavefronts per tile side up to this many value sides per compute unit, where two have become as fast.  (Vector registers, 55 to 58,
// would let eight sides of four wavefronts live on a compute unit; scalar ones, 112 and 16 for the trap handler of a SIMD's 800, let six.
// With 96, by a launch bound of seven or asked for, seven live: where there are seven a step takes 6 % less, with up to three 1 % more,
// and 4 x 32 heads of 3400, 3300, 1400 and 400 tokens 7 % more, 29.9 -> 32.1 us.)  Eight steps with their prompt, us, two | four: 5 (2 x 32 heads x 4100 tokens) 351.3 | 343.2, 6 (3 x 32 x 4000) 411.8 | 399.9,
// 7 (4 x 32 x 3500 of 64 channels) 352.9 | 347.6, 8 (4 x 32 x 4000) 454.4 | 455.3, the same with spiked values 467.7 | 470.7.
constexpr int kUpdFew = 7;
constexpr int kUpdResident = 16;    // tile sides a compute unit takes: two wavefronts of at most 64 registers each

// Beside this block a tile side has LDS for the codes of `a.max_moved` tokens (dynamic, sized at launch): that many
// staged rows, then a list word and a [min, max] for each.  Before any code is gathered the space holds, by position,
// the value side's predicted scores and (variable-length side store) largest | smallest outlier << 16.
template <int D, int NW>
struct UpdLds {
  // keys: byte d of a staged row = channel d; values: byte n*(D/16) + g = channel 16*g + n, the order of a unit's words
  static constexpr int SROW = D / 4 + 1;   // dwords per staged row (odd stride: rows spread over the banks)
  static constexpr int PER_TOKEN = 4 * SROW + 8;
  uint8_t m_of_slot[QAQ_TT];               // by new slot: index in the moved list
  uint8_t freeslot[QAQ_TT];                // the slots no token keeps, in order, those of every 64 slots in 64 places of their own
  unsigned long long same[QAQ_TT / 64];    // bit by old slot: the cached token there stays in its class
  uint32_t mask2[16], mask4[32], mask1b[16];   // value side: slots to write per unit of 16 (2-bit fields, 1-bit tokens) or half-unit of 8 (4-bit)
  unsigned long long written[QAQ_TT / 64 + 1];   // ... bit by slot
  uint32_t newrow[D / 4];                  // the appended token: its codes at the widest width, byte d = channel d
  uint32_t new_oi[2], new_ov[4];           // ... outlier channels, outlier values
  uint32_t new_mm;
  int new_no;                              // ... outliers (variable-length side store)
  int w_cls[NW][3];                        // per wavefront: tokens of a class, two counts per word
  int w_any[NW], w_wide[NW], w_moved[NW];
  int first_free[QAQ_NCLASS];              // per class: free slots before its first one among its 64 | which 64 << 8
  float w_bnd[NW], w_lo[NW], w_hi[NW];
  uint8_t units[NW][32];                   // ... units with words to write
};

// unsigned wavefront reductions, as wave_max.  (The appended token is a chain of one per outlier and two more, and the side
// that receives it has the longest way to go.  By shuffles through LDS, six round trips each, generating with outliers by
// thresholds, 3 x 16 heads x 2500 tokens, took 291 us, so 283.6.)
__device__ __forceinline__ uint32_t wave_umax(uint32_t x) {
  asm volatile(QAQ_DPP_STEP("v_max_u32_dpp", "quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_max_u32_dpp", "quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_max_u32_dpp", "row_half_mirror row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_max_u32_dpp", "row_mirror row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_max_u32_dpp", "row_bcast:15 row_mask:0xa bank_mask:0xf")
               QAQ_DPP_STEP("v_max_u32_dpp", "row_bcast:31 row_mask:0xc bank_mask:0xf")
               "s_nop 1"
               : "+v"(x));
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ uint32_t wave_umin(uint32_t x) {
  asm volatile(QAQ_DPP_STEP("v_min_u32_dpp", "quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_min_u32_dpp", "quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_min_u32_dpp", "row_half_mirror row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_min_u32_dpp", "row_mirror row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_min_u32_dpp", "row_bcast:15 row_mask:0xa bank_mask:0xf")
               QAQ_DPP_STEP("v_min_u32_dpp", "row_bcast:31 row_mask:0xc bank_mask:0xf")
               "s_nop 1"
               : "+v"(x));
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
__device__ __forceinline__ uint16_t key16_bits(uint32_t key) {     // fp16 bits of a key made by order_keys_pair (upper half)
  const uint32_t k = key >> 16;
  return (uint16_t)(k >= 0x8000u ? k - 0x8000u : ((0x8000u - k) | 0x8000u));
}
__device__ __forceinline__ uint32_t width_mask(int bits) { return 0x01010101u * ((1u << bits) - 1u); }

// The window's part of the value rule (Section 4.2) for two consecutive positions of one lane: largest
// score over this step's row (the maximum over the G query heads, rounded to what the window stores:
// `s`) and the window's rows.  As qaq_predicted, with loads of two elements (rows start at any multiple of
// the element: the loads are written as copies, so the compiler knows the alignment), all in flight
// together: W rows are read whatever the window's length (1, 3, 5 or 8: what it has not is row 0 again).
// ri0: index inside a ring row that p0 >= 0 (the lane's first position) counts from, row0: the same of the scores; lim[r]:
// positions from there on that row r covers.
struct Two { float x[2]; };
template <int W, typename RAW>
__device__ __forceinline__ void predicted2_w(const QaqView& v, const int (&lim)[QAQ_MAX_WINDOW], int skip, size_t ri0, int p0,
                                             const Two (&g)[4], float (&s)[2], float (&m)[2]) {
  const size_t ring_row = (size_t)v.B * v.Hkv * v.Tmax;
  struct R2 { RAW x[2]; } raw[W];
#pragma unroll
  for (int r = 0; r < W; ++r)
    __builtin_memcpy(&raw[r], (const uint8_t*)((const RAW*)v.ring + (size_t)(r < v.window && r != skip ? r : 0) * ring_row + ri0) + (uint32_t)(p0 * (int)sizeof(RAW)), sizeof(R2));
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    s[e] = qaq_ring_value(v, vmaxf(vmaxf(vmaxf(s[e], g[0].x[e]), vmaxf(g[1].x[e], g[2].x[e])), g[3].x[e]));
    m[e] = s[e];
  }
#pragma unroll
  for (int r = 0; r < W; ++r) {
    const int end = r < v.window && r != skip ? lim[r] : 0;
    float xs[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float x = sizeof(RAW) == 4 ? __uint_as_float((uint32_t)raw[r].x[e])
                    : v.ring_half == 1 ? h2f((uint16_t)raw[r].x[e]) : __uint_as_float((uint32_t)raw[r].x[e] << 16);
      xs[e] = x;
    }
    if (end >= QAQ_TT) {                                    // (uniform; what a row does not cover is left out)
      m[0] = vmaxf(m[0], xs[0]); m[1] = vmaxf(m[1], xs[1]);
    } else if (end > 0) {
      m[0] = vmaxf(m[0], p0 < end ? xs[0] : 0.0f); m[1] = vmaxf(m[1], p0 + 1 < end ? xs[1] : 0.0f);
    }
  }
}
template <typename RAW>
__device__ __forceinline__ void predicted2_t(const QaqView& v, const int (&lim)[QAQ_MAX_WINDOW], int skip, size_t ri0, int p0,
                                             const Two (&g)[4], float (&s)[2], float (&m)[2]) {
  if (v.window == 1) predicted2_w<1, RAW>(v, lim, skip, ri0, p0, g, s, m);
  else if (v.window <= 3) predicted2_w<3, RAW>(v, lim, skip, ri0, p0, g, s, m);
  else if (v.window <= 5) predicted2_w<5, RAW>(v, lim, skip, ri0, p0, g, s, m);
  else predicted2_w<8, RAW>(v, lim, skip, ri0, p0, g, s, m);
}
__device__ __forceinline__ void predicted2(const QaqView& v, const int (&lim)[QAQ_MAX_WINDOW], int skip, size_t ri0, int p0,
                                           const float* row0, int G, size_t stride, float (&s)[2], float (&m)[2]) {
  Two g[4];
  s[0] = s[1] = 0.0f;                                       // probabilities: >= 0
#pragma unroll 1
  for (int g0 = 4; g0 < G; g0 += 4) {                       // query heads beyond the first four
#pragma unroll
    for (int j = 0; j < 4; ++j) __builtin_memcpy(&g[j], (const uint8_t*)(row0 + (size_t)min(g0 + j, G - 1) * stride) + (uint32_t)(4 * p0), sizeof(Two));
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 2; ++e) s[e] = vmaxf(s[e], g[j].x[e]);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) __builtin_memcpy(&g[j], (const uint8_t*)(row0 + (size_t)min(j, G - 1) * stride) + (uint32_t)(4 * p0), sizeof(Two));
  if (v.ring_half) predicted2_t<uint16_t>(v, lim, skip, ri0, p0, g, s, m);
  else predicted2_t<uint32_t>(v, lim, skip, ri0, p0, g, s, m);
}

// The same for a tile that every row of the window covers -- all but the last one, once the window is full --: no row has
// an end to look at, and with one query head per KV head the row of scores is one load.  ring: the ring at the tile's first
// position.  A row that the window has not, or that this step's row replaces, is another one that counts.
template <int W, int GB, typename RAW>
__device__ __forceinline__ void predicted_full_w(const QaqView& v, int skip, const RAW* ring, size_t ring_row, int p0,
                                                 const float* row0, int G, size_t stride, float (&s)[2], float (&m)[2]) {
  struct R2 { RAW x[2]; } raw[W > 1 ? W - 1 : 1];
  const int other = skip == 0 ? 1 : 0;
#pragma unroll
  for (int r = 1; r < W; ++r) {                              // the rows behind `skip`, round the ring
    int at = skip + r;
    at -= at >= v.window ? v.window : 0;
    if (W == 3 || W == 8) at = r < v.window ? at : other;    // (these take windows of two, and of six and seven rows)
    __builtin_memcpy(&raw[r - 1], (const uint8_t*)(ring + (size_t)at * ring_row) + (uint32_t)(p0 * (int)sizeof(RAW)), sizeof(R2));
  }
  Two g[GB];
  s[0] = s[1] = 0.0f;                                        // probabilities: >= 0
#pragma unroll 1
  for (int g0 = GB; g0 < G; g0 += GB) {                      // query heads beyond the first GB
#pragma unroll
    for (int j = 0; j < GB; ++j) __builtin_memcpy(&g[j], (const uint8_t*)(row0 + (size_t)min(g0 + j, G - 1) * stride) + (uint32_t)(4 * p0), sizeof(Two));
#pragma unroll
    for (int j = 0; j < GB; ++j)
#pragma unroll
      for (int e = 0; e < 2; ++e) s[e] = vmaxf(s[e], g[j].x[e]);
  }
#pragma unroll
  for (int j = 0; j < GB; ++j) __builtin_memcpy(&g[j], (const uint8_t*)(row0 + (size_t)min(j, G - 1) * stride) + (uint32_t)(4 * p0), sizeof(Two));
#pragma unroll
  for (int e = 0; e < 2; ++e) {
#pragma unroll
    for (int j = 0; j < GB; ++j) s[e] = vmaxf(s[e], g[j].x[e]);
    s[e] = qaq_ring_value(v, s[e]);
    m[e] = s[e];
#pragma unroll
    for (int r = 1; r < W; ++r) {
      const RAW x = raw[r - 1].x[e];
      m[e] = vmaxf(m[e], sizeof(RAW) == 4 ? __uint_as_float((uint32_t)x) : v.ring_half == 1 ? h2f((uint16_t)x) : __uint_as_float((uint32_t)x << 16));
    }
  }
}
template <int GB, typename RAW>
__device__ __forceinline__ void predicted_full_t(const QaqView& v, int skip, size_t ri0, size_t ring_row, int p0,
                                                 const float* row0, int G, size_t stride, float (&s)[2], float (&m)[2]) {
  const RAW* ring = (const RAW*)v.ring + ri0;
  if (v.window == 1) predicted_full_w<1, GB, RAW>(v, skip, ring, ring_row, p0, row0, G, stride, s, m);
  else if (v.window <= 3) predicted_full_w<3, GB, RAW>(v, skip, ring, ring_row, p0, row0, G, stride, s, m);
  else if (v.window == 4) predicted_full_w<4, GB, RAW>(v, skip, ring, ring_row, p0, row0, G, stride, s, m);
  else if (v.window == 5) predicted_full_w<5, GB, RAW>(v, skip, ring, ring_row, p0, row0, G, stride, s, m);
  else predicted_full_w<8, GB, RAW>(v, skip, ring, ring_row, p0, row0, G, stride, s, m);
}
__device__ __forceinline__ void predicted_full(const QaqView& v, int skip, size_t ri0, size_t ring_row, int p0,
                                               const float* row0, int G, size_t stride, float (&s)[2], float (&m)[2]) {
  if (v.ring_half) {
    if (G == 1) predicted_full_t<1, uint16_t>(v, skip, ri0, ring_row, p0, row0, 1, stride, s, m);
    else predicted_full_t<4, uint16_t>(v, skip, ri0, ring_row, p0, row0, G, stride, s, m);
  } else {
    if (G == 1) predicted_full_t<1, uint32_t>(v, skip, ri0, ring_row, p0, row0, 1, stride, s, m);
    else predicted_full_t<4, uint32_t>(v, skip, ri0, ring_row, p0, row0, G, stride, s, m);
  }
}

// class of a slot (the classes are numbered in slot order), width of a class: no branches
template <bool HAS1>
__device__ __forceinline__ int class_at(const QaqCounts& c, int slot) {
  const int k = (slot >= c.n3 ? 1 : 0) + (slot >= c.n32() ? 1 : 0) + (slot >= c.n32() + c.n4 ? 1 : 0);
  return HAS1 ? k + (slot >= c.first1() ? 1 : 0) : k;
}
static_assert(QC3 == 0 && QC2 == 1 && QC4 == 2 && QC8 == 3 && QC1 == 4, "classes are numbered in slot order");
__device__ __forceinline__ int bits_of_class(int k) { return (int)((0x18423u >> (4 * k)) & 15u); }
template <bool HAS1>
__device__ __forceinline__ int class_start(const QaqCounts& c, int k) {        // slot less index inside the region
  const int n32 = c.n32(), first8 = n32 + c.n4, first1 = first8 + c.n8;
  int r = k == QC4 ? n32 : 0;
  r = k == QC8 ? first8 : r;
  if (HAS1) r = k == QC1 ? first1 : r;
  return r;
}

// Value side: the fields of the slots to write are put into the words as they are stored (a word holds
// one channel of up to 16 tokens; a word of a unit that did not exist starts from zero).  BF: field
// width; `masks`: slots to write per unit of 16 (BF 4: of 8) from slot0 on, those from n_slots on left out; `n3`: slots
// below it hold 3-bit codes (BF 2: their upper bits are wanted).  Each wavefront lists the units with
// work and takes every NW-th group of them from `wave` on (the regions start with different wavefronts: a trip to memory
// each), the words of a batch requested together.
template <int D, int BF, int NW>
__device__ __forceinline__ void put_units(int wave, uint8_t* region, const uint32_t* masks, int units_old, int n_slots, int slot0, int n3, const uint32_t* stage, UpdLds<D, NW>& L) {
  constexpr int LPU = BF == 1 ? D / 8 : D / 4;       // lanes per unit, four consecutive words each
  constexpr int UPW = 64 / LPU, U = NW > 2 && UPW > 2 ? 1 : 2, SPU = BF == 4 ? 8 : 16;
  constexpr uint32_t UB = BF == 1 ? 2 * D : 4 * D;
  const int lane = threadIdx.x & 63, own = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  auto mask_of = [&](int u) {
    const int n = min(max(n_slots - SPU * u, 0), SPU);
    return masks[u] & ((1u << n) - 1u);
  };
  const int n_units = (n_slots + SPU - 1) / SPU;      // at most 16 (BF 4: 32)
  const unsigned long long work = __ballot(lane < n_units && mask_of(min(lane, 256 / SPU - 1)) != 0u);
  const int nu = __popcll(work);
  if (nu == 0) return;
  if ((work >> lane) & 1ull) L.units[own][lanes_below(work)] = (uint8_t)lane;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (the wavefront's own list)
  const int sub = lane / LPU, c = lane % LPU;
#pragma unroll 1
  for (int i0 = wave * UPW * U; i0 < nu; i0 += NW * UPW * U) {
    u32x4 o[U];
    int un[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      un[k] = L.units[own][min(i0 + k * UPW + sub, nu - 1)];
      o[k] = *(const u32x4*)(region + (uint32_t)(un[k] * (int)UB + 16 * c));
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      if (i0 + k * UPW + sub >= nu) continue;
      uint32_t msk = mask_of(un[k]);
      if (un[k] >= units_old) o[k] = (u32x4)0u;
      while (msk) {
        const int i = __ffs(msk) - 1;
        msk &= msk - 1;
        const int sl = slot0 + SPU * un[k] + i;
        const uint32_t* row = &stage[(int)L.m_of_slot[sl] * UpdLds<D, NW>::SROW];
        if (BF == 1) {
          const uint32_t w0 = row[2 * c], w1 = row[2 * c + 1];      // word e: bytes 2*e and 2*e + 1 of the pair
          const int bp = 8 * (i & 3) + (i >> 2);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t x = (e < 2 ? w0 : w1) >> (16 * (e & 1));
            o[k][e] = (o[k][e] & ~(0x11u << bp)) | (((x & 1u) | ((x >> 4) & 0x10u)) << bp);
          }
        } else {
          constexpr uint32_t FM = BF == 2 ? 3u : 15u;
          const uint32_t w = row[c] >> (BF == 2 && sl < n3 ? 1 : 0);
          const int bp = 8 * (i & 3) + BF * (i >> 2);
#pragma unroll
          for (int e = 0; e < 4; ++e) o[k][e] = (o[k][e] & ~(FM << bp)) | (((w >> (8 * e)) & FM) << bp);
        }
      }
      *(u32x4*)(region + (uint32_t)(un[k] * (int)UB + 16 * c)) = o[k];
    }
  }
}

// ONE: one outlier per end in the fixed-length side store; else any count, or the variable-length store.
// HAS1: the width set contains 1.
// NW: wavefronts per tile side, two or four.
template <int D, bool ONE, bool HAS1, int NW>
__device__ __forceinline__ void update_side(const QaqBuildArgs& a) {
  // (and the key thresholds of the first 128 heads)
  qaq_request_arguments<0, offsetof(QaqBuildArgs, rule) + offsetof(QaqRuleArgs, tau_k) + 128 * sizeof(float)>();
  __shared__ UpdLds<D, NW> L;
  extern __shared__ uint32_t stage[];        // [max_moved][SROW], then the moved list
  constexpr int SROW = UpdLds<D, NW>::SROW, NQ = D / 16, KS = D / 64, NT = 64 * NW, J = QAQ_TT / NT, NC = HAS1 ? QAQ_NCLASS : 4;
  constexpr int NOI = ONE ? 1 : 4;          // words of outlier values per token, pairs of outlier channels
  uint32_t* const mv = stage + a.max_moved * SROW;      // moved list: token | new slot << 8 | position << 16 | old width << 24 | new width << 28
  uint32_t* const mv_mm = mv + a.max_moved;             // ... fp16 min | max << 16
  float* const pred = (float*)stage;                    // value side, until the codes are gathered: predicted scores
  uint32_t* const oext_at = stage + QAQ_TT;             // ... extremes of the outliers
  const QaqView& v = a.v;
  const QaqRuleArgs& ru = a.rule;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), tok0 = 64 * J * wave + lane;
  // (indices in 32 bits: a tile takes tens of kilobytes of the arena.  The KV head and the sequence only where they are asked for)
  const int bh = blockIdx.x;
  // Value sides first: nearly every one of them has work (a token's predicted score moves every step), most key sides leave after
  // one load and fill in behind.  Where not all sides are in flight at once, the tile that receives the token (of the
  // longest sequence) before all others: its sides have the longest way to go, and the key side was started last, 18-23 us
  // after the first ones at 8 x 32 heads x 4096 tokens, and waited for.
  int tile = blockIdx.y, side = 1 - (int)blockIdx.z;
  if (a.open_first) {
    const int n = (int)gridDim.y, open = a.len_before / QAQ_TT, at = tile + n * (int)blockIdx.z;      // 0 .. 2 n - 1
    const int r = at - 2, t = r < n - 1 ? r : r - (n - 1);
    side = at < 2 ? 1 - at : r < n - 1 ? 1 : 0;
    tile = at < 2 ? open : t + (t >= open ? 1 : 0);
  }
  const int t0 = tile * QAQ_TT;
  const int shorter = v.ragged ? v.shortfall[bh / v.Hkv] : 0;      // than the longest sequence
  const int len_before = max(a.len_before - shorter, 0), len_after = max(a.len_after - shorter, 0);   // of this sequence
  const int n_before = min(max(len_before - t0, 0), QAQ_TT);
  const int n_after = min(max(len_after - t0, 0), QAQ_TT);
  if (bh == 0 && blockIdx.y == 0 && blockIdx.z == 0 && tid == 0) a.todo_count[1] = 0u;      // (k_build_listed, if it has entries, leaves their number)
  if (n_after == 0) return;
  const bool csr = !ONE && v.csr;
  const int no2 = ONE ? 2 : v.no2;
  const bool has_new = n_after > n_before;           // the appended token is position n_before of this tile
  const uint32_t tile_id = (uint32_t)bh * (uint32_t)v.NT + (uint32_t)tile;
  // keys: the tile recorded, when it was built, the interval of thresholds for which none of its
  // tokens changes width (one 8-byte load decides)
  if (side == 0 && !has_new && !ru.out_bits[0]) {
    const float2 keep = ((const float2*)v.kthr)[tile_id];
    const float tau = ru.tau_k[v.ragged ? bh : bh % v.Hkv];
    if (tau >= keep.x && tau < keep.y) return;
  }

  // ---- everything whose address is known up front ------------------------------------------------
  uint8_t* base = v.codes[side] + (size_t)tile_id * v.cap[side];
  const uint2 counts_raw = *(const uint2*)(v.counts + ((size_t)tile_id * 2 + side) * 4);
  const size_t gi0 = (size_t)tile_id * QAQ_TT;      // (units follow one another in whole tiles)
  // the appended token's row, two channels per lane (where there is none, what is read anyway: no load behind a branch.  Two
  // wavefronts have no register for it until it is used)
  auto new_row = [&](bool some) { return (some ? (const uint32_t*)(a.newx[side] + (size_t)(uint32_t)(bh * a.n_new) * D) : v.mm[side] + gi0)[min(lane, D / 2 - 1)]; };
  uint32_t new_w = 0u;
  if (NW > 2) new_w = new_row(has_new);
  // token tok0 + 64*j: the cached token in that old slot, or (== n_before) the appended one
  uint32_t mm[J], oi[J], ov[J];      // (oi, ov: ONE; else the side store is read again for the tokens that move)
  uint32_t oext[J];                  // value side, not ONE: largest | smallest outlier << 16
  int pos[J];
  float thr_lo = INFINITY, thr_hi = -INFINITY;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const uint32_t s = (uint32_t)min(tok0 + 64 * j, max(n_before - 1, 0));
    mm[j] = *(const uint32_t*)((const uint8_t*)(v.mm[side] + gi0) + 4u * s);       // (uniform base, 32-bit lane offset)
    pos[j] = *(v.perm[side] + gi0 + s);
    oi[j] = ov[j] = 0u;
    oext[j] = 0xffffffffu;
    if (ONE) {
      oi[j] = *(const uint16_t*)(v.oidx[side] + gi0 * 2 + 2u * s);
      ov[j] = *(const uint32_t*)((const uint8_t*)(v.oval[side] + gi0 * 2) + 4u * s);
    }
  }
  auto thresholds = [&] {
    const float* t = v.othr + (side * v.Hkv + bh % v.Hkv) * 2;
    thr_lo = t[0]; thr_hi = t[1];
  };
  if (NW > 2 && csr) thresholds();
  if (!ONE && !csr && side == 1 && no2 > 0) {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const size_t at = (gi0 + min(tok0 + 64 * j, max(n_before - 1, 0))) * no2;
      const uint32_t* p = (const uint32_t*)(v.oval[1] + at);
      const uint16_t* pi = (const uint16_t*)(v.oidx[1] + at);
      uint32_t x[NOI], xi[NOI];
#pragma unroll
      for (int k = 0; k < NOI; ++k) { x[k] = p[min(k, no2 / 2 - 1)]; xi[k] = pi[min(k, no2 / 2 - 1)]; }
      float hi = -INFINITY, lo = INFINITY;
      bool some = false;
#pragma unroll
      for (int k = 0; k < 2 * NOI; ++k) {
        const float f = h2f((uint16_t)(x[k >> 1] >> (16 * (k & 1))));
        const bool used = ((xi[k >> 1] >> (8 * (k & 1))) & 0xffu) != 0xffu;
        hi = fmaxf(hi, used ? f : -INFINITY); lo = fminf(lo, used ? f : INFINITY);
        some |= used;
      }
      oext[j] = some ? (uint32_t)f2h(hi) | ((uint32_t)f2h(lo) << 16) : 0xffffffffu;
    }
  }
  if (side == 1 && (NW == 2 || wave < 2)) {      // the window (Section 4.2), this step's row stored: two positions per lane of two wavefronts
    const size_t ring_row = (size_t)((uint32_t)gridDim.x * (uint32_t)v.NT) * QAQ_TT;
    const size_t ri0 = gi0;
    const float* row0 = ru.scores + (size_t)(uint32_t)(bh * ru.G) * ru.score_stride + t0;
    if (t0 + QAQ_TT <= ru.rows_full - shorter) {
      float s[2], m[2];
      predicted_full(v, ru.new_row, ri0, ring_row, 2 * tid, row0, ru.G, ru.score_stride, s, m);
      if (v.ring_half == 0) {
        __builtin_memcpy((uint8_t*)((float*)v.ring + (size_t)ru.new_row * ring_row + ri0) + (uint32_t)(8 * tid), s, 8);
      } else {
        uint16_t hs[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) hs[e] = v.ring_half == 1 ? f2h(s[e]) : qaq_bf16_bits(s[e]);
        __builtin_memcpy((uint8_t*)((uint16_t*)v.ring + (size_t)ru.new_row * ring_row + ri0) + (uint32_t)(4 * tid), hs, 4);
      }
      pred[2 * tid] = m[0]; pred[2 * tid + 1] = m[1];
    } else if (len_after >= 2) {
      int lim[QAQ_MAX_WINDOW];
#pragma unroll
      for (int r = 0; r < QAQ_MAX_WINDOW; ++r) lim[r] = max(ru.row_len[r] - shorter, 0) - t0;
      // (the lane that the tile's end falls into reads one position further down: the one before it is
      // another lane's as well, and gets the same value from both)
      // (lane offsets are unsigned: in a tile with one token everything counts from the position before it)
      const int p0 = min(2 * tid, n_after - 2), back = n_after < 2 ? 1 : 0;
#pragma unroll
      for (int r = 0; r < QAQ_MAX_WINDOW; ++r) lim[r] += back;
      float s[2], m[2];
      predicted2(v, lim, ru.new_row, ri0 - back, p0 + back, row0 - back, ru.G, ru.score_stride, s, m);
      if (2 * tid < n_after) {
        const size_t ro = (size_t)ru.new_row * ring_row + ri0 + p0;
        if (p0 >= 0) {
          if (v.ring_half == 0) {
            __builtin_memcpy((uint8_t*)((float*)v.ring + (size_t)ru.new_row * ring_row + ri0) + (uint32_t)(4 * p0), s, 8);
          } else {
            uint16_t hs[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) hs[e] = v.ring_half == 1 ? f2h(s[e]) : qaq_bf16_bits(s[e]);
            __builtin_memcpy((uint16_t*)v.ring + ro, hs, 4);
          }
          pred[p0] = m[0]; pred[p0 + 1] = m[1];
        } else {               // a tile with one token: the position before it is another tile's
          qaq_ring_store(v, ro + 1, s[1]);
          pred[0] = m[1];
        }
      }
    } else if (tid == 0) {          // a sequence of one token
      float s = 0.0f;
      for (int g = 0; g < ru.G; ++g) s = fmaxf(s, row0[(size_t)g * ru.score_stride]);
      s = qaq_ring_value(v, s);
      pred[0] = qaq_window_max_compact(v, qaq_rows_covering(v, ru.row_len, bh / v.Hkv, t0), ru.new_row, ri0, s);
      qaq_ring_store(v, (size_t)ru.new_row * ring_row + ri0, s);
    }
  }
  if (csr && side == 1) {
      // outliers by thresholds: the extremes of every position's run in the tile's pool
      const size_t pool0 = gi0 * (size_t)no2;
      int cnt[J], st[J], most = 0;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int p = min(tok0 + 64 * j, max(n_before - 1, 0));
        cnt[j] = v.ocnt[1][gi0 + p];
        st[j] = v.ostart[1][gi0 + p];
      }
#pragma unroll
      for (int j = 0; j < J; ++j) { if (tok0 + 64 * j >= n_before) cnt[j] = 0; most = max(most, cnt[j]); }
      float hi[J], lo[J];
#pragma unroll
      for (int j = 0; j < J; ++j) { hi[j] = -INFINITY; lo[j] = INFINITY; }
#pragma unroll 1
      for (int k0 = 0; k0 < QAQ_MAX_NO2 && __ballot(most > k0) != 0ull; k0 += 4) {
        uint16_t x[J][4];
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
          for (int k = 0; k < 4; ++k) x[j][k] = v.oval[1][pool0 + (cnt[j] > 0 ? st[j] + min(k0 + k, cnt[j] - 1) : 0)];
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
          for (int k = 0; k < 4; ++k) { const float f = h2f(x[j][k]); hi[j] = fmaxf(hi[j], f); lo[j] = fminf(lo[j], f); }
      }
#pragma unroll
      for (int j = 0; j < J; ++j)
        if (tok0 + 64 * j < n_before) oext_at[tok0 + 64 * j] = cnt[j] > 0 ? (uint32_t)f2h(hi[j]) | ((uint32_t)f2h(lo[j]) << 16) : 0xffffffffu;
  }

  // ---- the appended token: outliers, range, codes at the widest width (Section 4.2 "Outliers",
  // Section 4.1 quantizer), by the last wavefront, two channels per lane --------------------------------
  if (has_new && wave == NW - 1) {
    int new_no = 0;              // outliers found (the variable-length store: as many as pass the thresholds)
    const bool act = 2 * lane < D;
    if (NW == 2) new_w = new_row(true);
    const uint32_t w = act ? new_w : 0u;
    if (act && a.orig_put[side]) ((uint32_t*)(a.orig_put[side] + ((size_t)bh * a.orig_tokens + len_before) * D))[lane] = w;
    const uint32_t kk = order_keys_pair(w);
    const int ch0 = 2 * lane, ch1 = 2 * lane + 1;
    const uint32_t k0 = kk << 16, k1 = kk & 0xffff0000u;
    bool in0 = act, in1 = act;
    if (NW == 2 && csr) thresholds();
    // the largest values, lowest channel first; then the smallest of the rest, lowest channel first; the
    // one in lane k is the k-th found
    uint32_t my_ch = 0xffu, my_val = 0u;
#pragma unroll 1
    for (int end = 0; end < 2; ++end)
#pragma unroll 1
      for (int k = 0; k < no2 / 2; ++k) {
        const uint32_t M = end == 0 ? wave_umax(max(in0 ? k0 | (uint32_t)(127 - ch0) : 0u, in1 ? k1 | (uint32_t)(127 - ch1) : 0u))
                                    : wave_umin(min(in0 ? k0 | (uint32_t)ch0 : 0xffffffffu, in1 ? k1 | (uint32_t)ch1 : 0xffffffffu));
        const int ch = end == 0 ? 127 - (int)(M & 127u) : (int)(M & 127u);
        if (!ONE) {               // (the count rule's thresholds are infinite: what no number passes is left out as in a bulk build)
          const float val = key16_value(M);
          if (!(end == 0 ? val > thr_hi : val < thr_lo)) break;
        }
        const uint32_t wc = (uint32_t)__builtin_amdgcn_readlane((int)w, ch >> 1);
        if (lane == new_no) { my_ch = (uint32_t)ch; my_val = (wc >> (16 * (ch & 1))) & 0xffffu; }
        in0 = in0 && ch0 != ch;
        in1 = in1 && ch1 != ch;
        ++new_no;
      }
    // [min, max] of what remains
    const uint32_t A2 = wave_umax(max(in0 ? k0 : 0u, in1 ? k1 : 0u));
    const uint32_t B2 = wave_umin(min(in0 ? k0 : 0xffffffffu, in1 ? k1 : 0xffffffffu));
    const uint32_t mn_b = key16_bits(B2), mx_b = key16_bits(A2);
    const float mn = h2f((uint16_t)mn_b), mx = h2f((uint16_t)mx_b);
    const float range = mx - mn;
    const float levels = (float)(1 << a.widest);
    const float inv = range > 0.0f ? levels / range : 0.0f;
    const float top_code = levels - 1.0f;
    uint32_t cw = 0u;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float diff = h2f((uint16_t)(w >> (16 * e))) - mn;
      const float prod = diff * inv;
      cw = __builtin_amdgcn_cvt_pk_u8_f32(fminf(floorf(prod), top_code), e, cw);
    }
    if (act) ((uint16_t*)L.newrow)[lane] = (uint16_t)cw;
    if (lane == 0) { L.new_mm = mn_b | (mx_b << 16); L.new_no = new_no; }
    // the side store is ordered by channel (unused places last)
    int rank = 0;
#pragma unroll
    for (int k = 0; k < 2 * NOI; ++k) {
      const uint32_t ck = (uint32_t)__builtin_amdgcn_readlane((int)my_ch, k);
      rank += ck < my_ch || (ck == my_ch && k < lane) ? 1 : 0;
    }
    if (lane < 2 * NOI) { ((uint8_t*)L.new_oi)[rank] = (uint8_t)my_ch; ((uint16_t*)L.new_ov)[rank] = (uint16_t)my_val; }
    if (!ONE && side == 1 && lane == 0) {
      float hi = -INFINITY, lo = INFINITY;
      for (int k = 0; k < new_no; ++k) { const float f = h2f(((const uint16_t*)L.new_ov)[k]); hi = fmaxf(hi, f); lo = fminf(lo, f); }
      oext_at[n_before] = new_no > 0 ? (uint32_t)f2h(hi) | ((uint32_t)f2h(lo) << 16) : 0xffffffffu;
    }
  }
  __syncthreads();
  QaqCounts c_old;
  c_old.n3 = c_old.n2 = c_old.n4 = c_old.n8 = c_old.n1 = 0;
  if (n_before > 0) {
    const uint32_t c01 = (uint32_t)__builtin_amdgcn_readfirstlane((int)counts_raw.x), c23 = (uint32_t)__builtin_amdgcn_readfirstlane((int)counts_raw.y);
    static_assert(QC3 == 0 && QC2 == 1 && QC4 == 2 && QC8 == 3, "order of the stored counts");
    c_old.n3 = (int)(c01 & 0xffffu); c_old.n2 = (int)(c01 >> 16); c_old.n4 = (int)(c23 & 0xffffu); c_old.n8 = (int)(c23 >> 16);
    if (HAS1) c_old.n1 = n_before - (c_old.n3 + c_old.n2 + c_old.n4 + c_old.n8);
  }

  // ---- widths by the rules of Section 4.1 -----------------------------------------------------------
  const float thr = side == 0 ? ru.tau_k[v.ragged ? bh : bh % v.Hkv] : ru.c_v[v.ragged ? bh / v.Hkv : 0];
  float thr_b[NC];             // (entries past the last width repeat it)
  int wc[NC];                  // width | class << 4
#pragma unroll
  for (int i = 0; i < NC; ++i) { thr_b[i] = ldexpf(thr, ru.bit_set[i]); wc[i] = ru.width_class[i]; }
  const bool served = a.orig[side] != nullptr;
  int cls[J];                  // class after this step, -1: no token
  unsigned long long same_cls[J];   // cached tokens that stay in their class
  int nb[J], ob[J];
  float bnd = 0.0f, lo = 0.0f, hi = INFINITY;
  unsigned long long any = 0ull;
  int n_wide = 0;
  unsigned long long bal_cls[NC][J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int tok = tok0 + 64 * j;
    const bool live = tok < n_after, is_new = has_new && tok == n_before;
    if (is_new) {
      mm[j] = L.new_mm;
      pos[j] = n_before;
      oi[j] = L.new_oi[0] & 0xffffu; ov[j] = L.new_ov[0];
    }
    const float mnf = h2f((uint16_t)(mm[j] & 0xffffu)), mxf = h2f((uint16_t)(mm[j] >> 16));
    const float range = mxf - mnf;
    const float lhs = side == 0 ? range : range * pred[pos[j]];
    int rc = wc[NC - 1];
#pragma unroll
    for (int i = NC - 1; i >= 0; --i) rc = lhs <= thr_b[i] ? wc[i] : rc;
    const int req = rc & 15;
    if (ru.out_bits[side] && live) ru.out_bits[side][(size_t)bh * a.len_after + t0 + pos[j]] = (uint8_t)req;
    const int oc = class_at<HAS1>(c_old, tok);
    ob[j] = bits_of_class(oc);
    ob[j] = is_new ? a.widest : ob[j];                  // encoded at the widest width; narrowing drops low bits
    const bool wider = live & !is_new & (req > ob[j]);
    nb[j] = (wider & !served) ? ob[j] : req;
    n_wide += __popcll(__ballot(wider));
    any |= __ballot(live & (is_new | (nb[j] != ob[j])));
    cls[j] = (wider & !served) ? oc : rc >> 4;
    cls[j] = live ? cls[j] : -1;
    same_cls[j] = __ballot((tok < n_before) & (cls[j] == oc));
#pragma unroll
    for (int c = 0; c < NC; ++c) bal_cls[c][j] = __ballot(cls[j] == c);
    // what the attention kernel and the next step's skip test need of the tile
    if (side == 1) {
      float bt = ldexpf(range, nb[j] == 3 ? -2 : -nb[j]);
      uint32_t x = ONE ? ov[j] : oext[j];           // two numbers the tile's largest correction is between
      if (!ONE && (csr || is_new)) x = oext_at[pos[j]];
      const float o1 = h2f((uint16_t)(x & 0xffffu)), o0 = h2f((uint16_t)(x >> 16));
      const float bo = fmaxf(fmaxf(fabsf(o1 - mxf), fabsf(o1 - mnf)), fmaxf(fabsf(o0 - mxf), fabsf(o0 - mnf))) + range;
      if (ONE || x != 0xffffffffu) bt = fmaxf(bt, bo);
      if (live) bnd = fmaxf(bnd, bt);
    } else if (live) {
      int narrower = 0;
#pragma unroll
      for (int i = 0; i < NC; ++i)
        if (ru.bit_set[i] < nb[j]) narrower = ru.bit_set[i];
      if (nb[j] < ru.bit_set[NC - 1]) lo = fmaxf(lo, ldexpf(range, -nb[j]));
      if (narrower > 0) hi = fminf(hi, ldexpf(range, -narrower));
    }
  }
  if (side == 1) bnd = wave_max(bnd);
  else { lo = wave_max(lo); hi = wave_min(hi); }
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < J; ++j) L.same[J * wave + j] = same_cls[j];
#pragma unroll
    for (int c = 0; c < (NC + 1) / 2; ++c) {             // two counts per word
      int n = 0;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        n += __popcll(bal_cls[2 * c][j]);
        if (2 * c + 1 < NC) n += __popcll(bal_cls[2 * c + 1 < NC ? 2 * c + 1 : 0][j]) << 16;
      }
      L.w_cls[wave][c] = n;
    }
    L.w_any[wave] = any != 0ull; L.w_wide[wave] = n_wide;
    L.w_bnd[wave] = bnd; L.w_lo[wave] = lo; L.w_hi[wave] = hi;
  }
  __syncthreads();
  int all_wide = 0, some = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) { all_wide += L.w_wide[w]; some |= L.w_any[w]; }
  if (!some) {          // nothing moves and nothing is appended
    if (tid == 0 && all_wide) v.refused[((size_t)tile_id * 2 + side) * 2 + (served ? 1 : 0)] += (unsigned int)all_wide;
    return;
  }
  auto all_waves = [&](int c) {
    int n = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) n += L.w_cls[w][c];
    return __builtin_amdgcn_readfirstlane(n);
  };
  QaqCounts cn;
  {
    const int n01 = all_waves(0), n23 = all_waves(1);
    cn.n3 = n01 & 0xffff; cn.n2 = n01 >> 16; cn.n4 = n23 & 0xffff; cn.n8 = n23 >> 16;
    cn.n1 = HAS1 ? all_waves(2) : 0;
  }

  // ---- regions.  A token's codes sit at an index inside its class's region (2- and 3-bit tokens: the
  // slot; the others: the slot less the class's first one).  The 2-bit fields start the tile side; another
  // region's start moves when the space before it changes.  What it holds for the tokens that stay is then
  // copied, region by region as long as the copies are small; the tokens of one that is not copied are
  // written again like any other moved token. -----------------------------------------------------------
  const int n32o = c_old.n32(), n32n = cn.n32();
  uint32_t r_old[QAQ_NCLASS], r_new[QAQ_NCLASS];
  int cp_end[QAQ_NCLASS];       // 16-byte pieces to copy, summed up to and including the class's region
  uint32_t lost = 0u;           // bit c: the region of class c moved and is not copied
  {
    if (side == 0) {
      const QaqKRegions r0 = qaq_k_regions(c_old, D), r1 = qaq_k_regions(cn, D);
      r_old[QC3] = r0.r1; r_old[QC2] = r0.r2; r_old[QC4] = r0.r4; r_old[QC8] = r0.r8; r_old[QC1] = r0.r1b;
      r_new[QC3] = r1.r1; r_new[QC2] = r1.r2; r_new[QC4] = r1.r4; r_new[QC8] = r1.r8; r_new[QC1] = r1.r1b;
    } else {
      const QaqVRegions r0 = qaq_v_regions(c_old, D), r1 = qaq_v_regions(cn, D);
      r_old[QC3] = r0.r1; r_old[QC2] = r0.r2; r_old[QC4] = r0.r4; r_old[QC8] = r0.r8; r_old[QC1] = r0.r1b;
      r_new[QC3] = r1.r1; r_new[QC2] = r1.r2; r_new[QC4] = r1.r4; r_new[QC8] = r1.r8; r_new[QC1] = r1.r1b;
    }
    const int n3 = min(c_old.n3, cn.n3), n4 = min(c_old.n4, cn.n4), n8 = min(c_old.n8, cn.n8), n1 = min(c_old.n1, cn.n1);
    int bytes[QAQ_NCLASS];     // (keys: records; values: whole units; both within what the region is sized for)
    bytes[QC2] = 0;
    bytes[QC3] = side == 0 ? (n3 * (D / 8) + 15) & ~15 : ((n3 + 15) / 16) * (2 * D);
    bytes[QC4] = side == 0 ? n4 * (D / 2) : ((n4 + 7) / 8) * (4 * D);
    bytes[QC8] = n8 * D;
    bytes[QC1] = side == 0 ? (n1 * (D / 8) + 15) & ~15 : ((n1 + 15) / 16) * (2 * D);
    int sum = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const bool moved = r_old[c] != r_new[c] && bytes[c] > 0;
      const bool fits = sum + bytes[c] <= kMaxCopy;
      if (moved && !fits) lost |= 1u << c;
      if (moved && fits) sum += bytes[c];
      cp_end[c] = sum >> 4;
    }
  }

  // ---- slots: a cached token that stays in its class keeps its index if the region still reaches it; the others --
  // tokens that change class, tokens squeezed out, the appended one -- take the free slots of their class in order.
  // Which old slots can be kept follows from the class counts alone, and which of a class's new slots are then taken from
  // the old slots they were; free slots are in class order as they are, so they make one list, and only the tokens that
  // move ask where their class begins in it. ------------------------------------------------------------------------
  const int shift4 = n32n - n32o, shift8 = shift4 + cn.n4 - c_old.n4, shift1 = shift8 + cn.n8 - c_old.n8;     // new slot less old slot of a kept token
  auto kept_end = [&](int c, int first, int n_old, int n_new) { return (lost >> c) & 1u ? first : first + min(n_old, n_new); };
  const int f8 = n32o + c_old.n4, f1 = f8 + c_old.n8;
  const int e3 = kept_end(QC3, 0, c_old.n3, cn.n3), s2 = max(cn.n3, c_old.n3), e2 = min(n32o, n32n);
  const int e4 = kept_end(QC4, n32o, c_old.n4, cn.n4), e8 = kept_end(QC8, f8, c_old.n8, cn.n8), e1 = kept_end(QC1, f1, c_old.n1, cn.n1);
  // What is left to write of a token, in one register: position, slot (of a token that moves: its place among the wavefront's
  // that do), width, old width, and whether it moves or its place changes, whether its width does, whether it moves.
  uint32_t left[J];
  constexpr uint32_t kMoves = 1u << 20, kRetag = 1u << 21, kNeeds = 1u << 22;
  unsigned long long need_bal[J];
  int moved_here = 0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int at = J * wave + j, tok = tok0 + 64 * j;      // (tokens 64*at .. +63, and the slots of these numbers)
    const unsigned long long live_bal = __ballot(tok < n_after);
    unsigned long long free_bal;
    int to = tok;
    const bool narrow = 64 * at + 64 <= e2;
    if (narrow) {                   // (scalar) 2- and 3-bit tokens before and after: what is kept stays where it is
      need_bal[j] = free_bal = live_bal & ~(same_cls[j] & __ballot((tok < e3) | (tok >= s2)));
    } else {
      bool can = (tok < e3) | ((tok >= s2) & (tok < e2)) | ((tok >= n32o) & (tok < e4)) | ((tok >= f8) & (tok < e8));
      if (HAS1) can |= (tok >= f1) & (tok < e1);
      to = tok + (tok >= n32o ? shift4 : 0);
      to = tok >= f8 ? tok + shift8 : to;
      if (HAS1) to = tok >= f1 ? tok + shift1 : to;
      need_bal[j] = live_bal & ~(same_cls[j] & __ballot(can));
      // the same place as a new slot: its class, and whether the old slot that class would have kept there was kept
      const int k = class_at<HAS1>(cn, tok);
      int from = tok - (k == QC4 ? shift4 : k == QC8 ? shift8 : HAS1 && k == QC1 ? shift1 : 0);
      const int k0 = k == QC3 ? 0 : k == QC2 ? s2 : k == QC4 ? n32o : !HAS1 || k == QC8 ? f8 : f1;
      const int k1 = k == QC3 ? e3 : k == QC2 ? e2 : k == QC4 ? e4 : !HAS1 || k == QC8 ? e8 : e1;
      const bool inside = (from >= k0) & (from < k1);
      from = inside ? from : 0;
      const bool taken = inside & (((((const uint32_t*)L.same)[from >> 5] >> (from & 31)) & 1u) != 0u);
      free_bal = __ballot(!taken) & live_bal;
    }
    const int below = lanes_below(free_bal);
    if ((free_bal >> lane) & 1ull) L.freeslot[64 * at + below] = (uint8_t)tok;
    if (tok == cn.n3) L.first_free[QC2] = below | (at << 8);      // (a class that has no slot is never asked for)
    if (!narrow && ((tok == n32n) | (tok == n32n + cn.n4) | (HAS1 && tok == cn.first1()))) {
      const int x = below | (at << 8);
      if (tok == n32n) L.first_free[QC4] = x;
      if (tok == n32n + cn.n4) L.first_free[QC8] = x;
      if (HAS1 && tok == cn.first1()) L.first_free[QC1] = x;
    }
    // every free slot is taken by a token that moves: the slots to write
    if (lane == 0) L.written[at] = free_bal;
    const bool live = tok < n_after, need = ((need_bal[j] >> lane) & 1ull) != 0ull, is_new = has_new & (tok == n_before);
    if (need) to = moved_here + lanes_below(need_bal[j]);
    left[j] = (uint32_t)pos[j] | ((uint32_t)(to & 0xff) << 8) | ((uint32_t)nb[j] << 16) | ((uint32_t)ob[j] << 24) |
              ((live & ((to != tok) | need)) ? kMoves : 0u) | ((live & ((nb[j] != ob[j]) | is_new)) ? kRetag : 0u) | (need ? kNeeds : 0u);
    moved_here += __popcll(need_bal[j]);
  }
  if (lane == 0) L.w_moved[wave] = moved_here;
  if (tid == 0) L.written[QAQ_TT / 64] = 0ull;
  __syncthreads();
  int n_moved = 0, moved0 = 0;          // tokens that move; ... of the wavefronts before this one
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const int n = __builtin_amdgcn_readfirstlane(L.w_moved[w]);
    moved0 += w < wave ? n : 0;
    n_moved += n;
  }
  if (n_moved > a.max_moved) {
    // nothing of the cache has been written yet (the window row and the width outputs are the same
    // numbers when the general kernel writes them again)
    if (tid == 0) a.todo[atomicAdd(a.todo_count, 1u)] = (uint32_t)(tile_id * 2 + side);
    return;
  }
#pragma unroll
  for (int j = 0; j < J; ++j)
    if (left[j] & kNeeds) {
      const int at = moved0 + (int)((left[j] >> 8) & 0xffu);
      mv[at] = (uint32_t)(tok0 + 64 * j) | ((left[j] & 0xffu) << 16) | (left[j] & 0xf000000u) | ((left[j] << 12) & 0xf0000000u);
      mv_mm[at] = mm[j];
    }
  __syncthreads();
  // (what follows up to the next barrier does not look at the moved tokens' slots)
  if (wave == 0) {            // the moved tokens' slots, a token per lane
    int free_to[3], sum = 0;               // free slots among the first 64, 128, 192
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const uint2 m = *(const uint2*)&L.written[i];
      sum += __builtin_popcount(__builtin_amdgcn_readfirstlane((int)m.x)) + __builtin_popcount(__builtin_amdgcn_readfirstlane((int)m.y));
      free_to[i] = sum;
    }
    int used[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) used[c] = 0;
#pragma unroll 1
    for (int m0 = 0; m0 < n_moved; m0 += 64) {
      const bool live = m0 + lane < n_moved;
      const int m = min(m0 + lane, n_moved - 1);
      const int c = live ? qaq_class_of_bits((int)(mv[m] >> 28)) : -1;
      int rank = 0;
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        const unsigned long long bal = __ballot(c == k);
        rank = c == k ? used[k] + lanes_below(bal) : rank;
        used[k] += __popcll(bal);
      }
      const int x = c > 0 ? L.first_free[c] : 0, i = x >> 8;
      const int f = rank + (x & 255) + (i == 0 ? 0 : i == 1 ? free_to[0] : i == 2 ? free_to[1] : free_to[2]);
      const int of = f < free_to[0] ? 0 : f < free_to[1] ? 64 - free_to[0] : f < free_to[2] ? 128 - free_to[1] : 192 - free_to[2];
      if (live) {
        const int slot = L.freeslot[f + of];
        ((uint8_t*)&mv[m])[1] = (uint8_t)slot;
        L.m_of_slot[slot] = (uint8_t)m;
      }
    }
  }
  if (side == 1 && wave == NW - 1) {     // value side: which slots are written, by unit of the region they are in
    auto slots_from = [&](int first) -> uint32_t {       // slots [first, first + 16) of those to write
      const uint32_t* p = (const uint32_t*)L.written + (min(first, QAQ_TT) >> 5);
      return __builtin_amdgcn_alignbit(p[1], p[0], (uint32_t)first & 31u) & 0xffffu;
    };
    if (lane < 16) L.mask2[lane] = slots_from(16 * lane);
    else if (lane < 48) L.mask4[lane - 16] = slots_from(n32n + 8 * (lane - 16)) & 0xffu;
    else if (HAS1) L.mask1b[lane - 48] = slots_from(cn.first1() + 16 * (lane - 48));
  }
  // ---- codes of the moved tokens -> LDS, at the new width: sixteen channels per work item --------------------
  // (all loads of an item without a condition, so that they are in flight together: the class selects addresses,
  // shifts and masks.  Four channels per item cost as many instructions per item.)
  {
    constexpr int LPT = D / 16;
    const int n_items = n_moved * LPT;
    const int new_tok = has_new ? n_before : QAQ_TT;
    // sixteen values of the unquantized copy at the token's [min, max] (Section 4.2 "Integration"), four codes per word
    auto encode16 = [&](const u32x4& x0, const u32x4& x1, uint32_t m2, int n_b, uint32_t (&codes)[4]) {
      const float mn = h2f((uint16_t)(m2 & 0xffffu)), mx = h2f((uint16_t)(m2 >> 16));
      const float rg = mx - mn;
      const float levels = (float)(1 << n_b);
      const float inv = rg > 0.0f ? levels / rg : 0.0f;
      const float top_code = levels - 1.0f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        codes[k] = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t hw = k < 2 ? x0[2 * k + (e >> 1)] : x1[2 * (k - 2) + (e >> 1)];
          const float diff = h2f((uint16_t)(hw >> (16 * (e & 1)))) - mn;
          const float prod = diff * inv;
          codes[k] = __builtin_amdgcn_cvt_pk_u8_f32(fminf(floorf(prod), top_code), e, codes[k]);
        }
      }
    };
    auto gather = [&](auto side_c) {
      constexpr int SD = decltype(side_c)::value;
#pragma unroll 1
      for (int it = tid < 64 ? tid + NT - 64 : tid - 64; it < n_items; it += NT) {      // (the first wavefront is still at the slots)
        int c = it % LPT;
        asm volatile("" : "+v"(c));        // (nothing that follows from it is worth a register across the loop)
        const int m = it / LPT;
        const uint32_t e = mv[m];
        const int tok = (int)(e & 0xffu), o_b = (int)((e >> 24) & 15u), n_b = (int)(e >> 28), p = (int)((e >> 16) & 0xffu);
        const int slot = min(tok, max(n_before - 1, 0));                 // (the appended token has no old codes: any in-range address)
        const bool fresh = tok == new_tok, wide = n_b > o_b && !fresh;
        const int k = class_at<HAS1>(c_old, slot), idx = slot - class_start<HAS1>(c_old, k);
        const bool f3 = k == QC3, f8 = k == QC8, f1 = HAS1 && k == QC1, f4 = k == QC4;
        const int drop = o_b - n_b;
        const uint32_t keep_bits = width_mask(n_b);
        uint32_t codes[4];
        if constexpr (SD == 0) {
          // keys: slice c of the record, channels 64*ks + 16*g ..: one word, two or four, and for a 3-bit token half a
          // word of low bits; of the copy's row 32 bytes
          const int ch0 = 64 * (c % KS) + 16 * (c / KS);
          uint32_t ro = k <= QC2 ? 0u : r_old[QC8];
          ro = f4 ? r_old[QC4] : ro;
          if (HAS1) ro = f1 ? r_old[QC1] : ro;
          const int s8 = (int)((0x30122u >> (4 * k)) & 15u);           // 8 >> s8 bits per channel
          const uint32_t at = ro + (uint32_t)idx * ((uint32_t)D >> s8) + ((uint32_t)(16 * c) >> s8 & ~3u);
          const uint32_t lo_at = f3 ? r_old[QC3] + (uint32_t)slot * (D / 8) + 4u * (uint32_t)(c >> 1) : at;
          const uint32_t st1 = f4 || f8 ? 4u : 0u, st2 = f8 ? 4u : 0u;
          uint32_t w[4];
          w[0] = *(const uint32_t*)(base + at);
          w[1] = *(const uint32_t*)(base + (at + st1));
          w[2] = *(const uint32_t*)(base + (at + 2u * st2));
          w[3] = *(const uint32_t*)(base + (at + 3u * st2));
          uint32_t low = *(const uint32_t*)(base + lo_at);
          u32x4 x0 = (u32x4)0u, x1 = (u32x4)0u;
          if (wide) {
            const u32x4* src = (const u32x4*)(a.orig[0] + ((size_t)bh * a.orig_tokens + (t0 + p)) * D + ch0);
            x0 = src[0]; x1 = src[1];
          }
          if (fresh) {
#pragma unroll
            for (int q = 0; q < 4; ++q) codes[q] = (L.newrow[ch0 / 4 + q] >> drop) & keep_bits;
          } else if (wide) {
            encode16(x0, x1, mv_mm[m], n_b, codes);
          } else {
            if (HAS1 && f1) low = w[0];
            low >>= 4 * (c & 1);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              uint32_t x = f8 ? w[q] ^ 0x80808080u : f4 ? (w[q >> 1] >> (4 * (q & 1))) & 0x0f0f0f0fu : (w[0] >> (2 * q)) & 0x03030303u;
              const uint32_t lb = (low >> q) & 0x01010101u;
              if (f3) x = (x << 1) | lb;
              if (HAS1 && f1) x = lb;
              codes[q] = (x >> drop) & keep_bits;
            }
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) stage[m * SROW + ch0 / 4 + q] = codes[q];
        } else {
          // values: words 16*c .. 16*c+15 of the token's unit, a channel each, and for a 3-bit token eight words of low
          // bits, two channels each; of an 8-bit row or of the copy's row the channels 16*c ..
          const int us = f4 ? 3 : 4, u = idx >> us, i = idx - (u << us);
          const uint32_t lo = (uint32_t)u * (2u * D) + 32u * (uint32_t)c;
          uint32_t at = (uint32_t)u * (4u * D) + 64u * (uint32_t)c + (f4 ? r_old[QC4] : 0u);
          at = f8 ? r_old[QC8] + (uint32_t)idx * D + 16u * (uint32_t)c : at;
          const uint32_t lo_at = HAS1 && f1 ? r_old[QC1] + lo : f3 ? r_old[QC3] + lo : at & ~31u;
          if (HAS1) at = f1 ? lo_at : at;
          const bool unit = !f8 && !f1;
          u32x4 w[4], l[2];
          w[0] = *(const u32x4*)(base + at);
          w[1] = *(const u32x4*)(base + (at + (unit ? 16u : 0u)));
          w[2] = *(const u32x4*)(base + (at + (unit ? 32u : 0u)));
          w[3] = *(const u32x4*)(base + (at + (unit ? 48u : 0u)));
          l[0] = *(const u32x4*)(base + lo_at);
          l[1] = *(const u32x4*)(base + (lo_at + (f3 || f1 ? 16u : 0u)));
          if (wide) {
            const u32x4* src = (const u32x4*)(a.orig[1] + ((size_t)bh * a.orig_tokens + (t0 + p)) * D + 16 * c);
            w[0] = src[0]; w[1] = src[1];
          }
          uint8_t* row = (uint8_t*)&stage[m * SROW];
          if (fresh || wide || f8) {             // by channel: channel 16*c + n goes to byte n*(D/16) + c
            if (fresh) {
#pragma unroll
              for (int q = 0; q < 4; ++q) codes[q] = (L.newrow[4 * c + q] >> drop) & keep_bits;
            } else if (wide) {
              encode16(w[0], w[1], mv_mm[m], n_b, codes);
            } else {
#pragma unroll
              for (int q = 0; q < 4; ++q) codes[q] = (w[0][q] >> drop) & keep_bits;
            }
#pragma unroll
            for (int n = 0; n < 16; ++n) row[n * (D / 16) + c] = (uint8_t)(codes[n >> 2] >> (8 * (n & 3)));
          } else {
            const int sh = 8 * (i & 3) + (f4 ? 4 : 2) * (i >> 2), shl = 8 * (i & 3) + (i >> 2);
            const uint32_t msk = f4 ? 15u : 3u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              uint32_t x = 0u;
#pragma unroll
              for (int n = 0; n < 4; ++n) x |= ((w[q][n] >> sh) & msk) << (8 * n);
              if (f3 || f1) {                       // bits 0 and 4 of a word: two channels
                const uint32_t l0 = l[q >> 1][2 * (q & 1)] >> shl, l1 = l[q >> 1][2 * (q & 1) + 1] >> shl;
                const uint32_t lb = (l0 & 1u) | ((l0 << 4) & 0x100u) | ((l1 << 16) & 0x10000u) | ((l1 << 20) & 0x1000000u);
                x = f1 ? lb : (x << 1) | lb;
              }
              stage[m * SROW + 4 * c + q] = (x >> drop) & keep_bits;
            }
          }
        }
      }
    };
    if (side == 0) gather(std::integral_constant<int, 0>{});
    else gather(std::integral_constant<int, 1>{});
  }

  // ---- regions that start elsewhere: read as a whole, then written.  (Asked for before the moved tokens' codes by four
  // wavefronts: no difference) ------------------------------------------------------------------------------
  const int n_cp = cp_end[NC - 1];
  if (n_cp > 0) {
    constexpr int CP = kMaxCopy / (16 * NT);
    u32x4 x[CP];
    uint32_t dst[CP];
#pragma unroll
    for (int k = 0; k < CP; ++k) {
      const int i = min(NT * k + tid, n_cp - 1);
      uint32_t so = 0u, d = 0u;
#pragma unroll
      for (int c = NC - 1; c >= 0; --c)          // the class whose share holds piece i
        if (i < cp_end[c]) {
          const uint32_t first = 16u * (uint32_t)(i - (c > 0 ? cp_end[c > 0 ? c - 1 : 0] : 0));
          so = r_old[c] + first; d = r_new[c] + first;
        }
      dst[k] = d;
      x[k] = *(const u32x4*)(base + so);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();           // old and new places may overlap: everything read before anything is written
#pragma unroll
    for (int k = 0; k < CP; ++k)
      if (NT * k + tid < n_cp) *(u32x4*)(base + dst[k]) = x[k];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // ... and written before words of it are read again
  }
  uint32_t oi_mv[J][NOI], ov_mv[J][NOI];
  if (!ONE && !csr) {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int tok = tok0 + 64 * j;
      const size_t gi = gi0 + min(tok, max(n_before - 1, 0));
      if (left[j] & kMoves) {
#pragma unroll
        for (int k = 0; k < NOI; ++k)
          if (2 * k < no2) {
            oi_mv[j][k] = tok == n_before ? ((const uint16_t*)L.new_oi)[k] : *(const uint16_t*)(v.oidx[side] + gi * no2 + 2 * k);
            ov_mv[j][k] = tok == n_before ? L.new_ov[k] : *(const uint32_t*)(v.oval[side] + gi * no2 + 2 * k);
          }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < J; ++j) asm volatile("" :: "v"(oi[j]), "v"(ov[j]));      // (the side store's too)
  __syncthreads();      // every read of the old layout is done

  // ---- metadata: tokens whose slot changed (moved ones, and tokens behind a moved class border),
  // widths by position, class counts, the tile's bounds ------------------------------------------------
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int p = (int)(left[j] & 0xffu);
    if (left[j] & kMoves) {
      uint32_t slot = (left[j] >> 8) & 0xffu;
      if (left[j] & kNeeds) slot = (mv[moved0 + slot] >> 8) & 0xffu;
      const size_t gi = gi0 + slot;
      v.mm[side][gi] = mm[j];
      v.perm[side][gi] = (uint8_t)p;
      if (ONE) {
        *(uint16_t*)(v.oidx[side] + gi * 2) = (uint16_t)oi[j];
        *(uint32_t*)(v.oval[side] + gi * 2) = ov[j];
      } else {
#pragma unroll
        for (int k = 0; k < NOI; ++k)
          if (!csr && 2 * k < no2) {
            *(uint16_t*)(v.oidx[side] + gi * no2 + 2 * k) = (uint16_t)oi_mv[j][k];
            *(uint32_t*)(v.oval[side] + gi * no2 + 2 * k) = ov_mv[j][k];
          }
      }
    }
    if (left[j] & kRetag) v.tags[side][gi0 + p] = (uint8_t)((left[j] >> 16) & 15u);
  }
  if (csr && has_new) {        // the appended token's run goes behind the tile's last one
    const size_t pool0 = gi0 * (size_t)no2;
    const int st = n_before > 0 ? (int)v.ostart[side][gi0 + n_before - 1] + (int)v.ocnt[side][gi0 + n_before - 1] : 0;
    const int new_no = L.new_no;
    if (tid == 0) { v.ostart[side][gi0 + n_before] = (uint16_t)st; v.ocnt[side][gi0 + n_before] = (uint8_t)new_no; }
    if (tid < new_no) {
      v.oidx[side][pool0 + st + tid] = ((const uint8_t*)L.new_oi)[tid];
      v.oval[side][pool0 + st + tid] = ((const uint16_t*)L.new_ov)[tid];
    }
  }
  if (tid == 0) {
    uint16_t* cp = v.counts + (((size_t)tile_id * 2 + side) * 4);
    cp[QC3] = (uint16_t)cn.n3; cp[QC2] = (uint16_t)cn.n2; cp[QC4] = (uint16_t)cn.n4; cp[QC8] = (uint16_t)cn.n8;
    float b = L.w_bnd[0], l = L.w_lo[0], h = L.w_hi[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) { b = fmaxf(b, L.w_bnd[w]); l = fmaxf(l, L.w_lo[w]); h = fminf(h, L.w_hi[w]); }
    if (side == 1) v.vbound[tile_id] = b;
    else ((float2*)v.kthr)[tile_id] = make_float2(l, h);
    if (all_wide) v.refused[((size_t)tile_id * 2 + side) * 2 + (served ? 1 : 0)] += (unsigned int)all_wide;
  }

  // ---- codes of the moved tokens -> their new places ----------------------------------------------------
  if (side == 0) {
    for (int it = tid; it < n_moved * NQ; it += NT) {
      const int m = it / NQ, q = it % NQ;
      const uint32_t e = mv[m];
      const int sl = (int)((e >> 8) & 0xffu), n_b = (int)(e >> 28);
      const uint32_t* row = &stage[m * SROW + 16 * (q % KS) + 4 * (q / KS)];
      const uint32_t* row1 = &stage[m * SROW + 16 * ((q | 1) % KS) + 4 * ((q | 1) / KS)];       // slices q and q+1 of 1-bit fields share a word
      if (n_b <= 3) {
        if (!HAS1 || n_b > 1) {
          const int sh = n_b == 3 ? 1 : 0;
          uint32_t w = 0;
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) w |= ((row[vq] >> sh) & 0x03030303u) << (2 * vq);
          *(uint32_t*)(base + r_new[QC2] + (uint32_t)sl * (D / 4) + 4u * (uint32_t)q) = w;
        }
        if (n_b != 2 && !(q & 1)) {
          uint32_t w1 = 0;
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) w1 |= ((row[vq] & 0x01010101u) << vq) | ((row1[vq] & 0x01010101u) << (4 + vq));
          const uint32_t at = HAS1 && n_b == 1 ? r_new[QC1] + (uint32_t)(sl - cn.first1()) * (D / 8) : r_new[QC3] + (uint32_t)sl * (D / 8);
          *(uint32_t*)(base + at + 4u * (uint32_t)(q >> 1)) = w1;
        }
      } else if (n_b == 4) {
        const uint2 w = make_uint2((row[0] & 0x0f0f0f0fu) | ((row[1] & 0x0f0f0f0fu) << 4), (row[2] & 0x0f0f0f0fu) | ((row[3] & 0x0f0f0f0fu) << 4));
        *(uint2*)(base + r_new[QC4] + (uint32_t)(sl - n32n) * (D / 2) + 8u * (uint32_t)q) = w;
      } else {
        *(uint4*)(base + r_new[QC8] + (uint32_t)(sl - n32n - cn.n4) * D + 16u * (uint32_t)q) =
            make_uint4(row[0] ^ 0x80808080u, row[1] ^ 0x80808080u, row[2] ^ 0x80808080u, row[3] ^ 0x80808080u);
      }
    }
    return;
  }
  // value side: the words of the units with slots to write
  // (the slots that are written were marked before the codes were gathered: barriers since)
  auto old_units = [&](int c, int n) { return (lost >> c) & 1u ? 0 : n; };
  auto from = [&](int w) { return (wave + w) & (NW - 1); };
  if (n32n > 0) put_units<D, 2>(wave, base + r_new[QC2], L.mask2, (n32o + 15) / 16, n32n, 0, cn.n3, stage, L);
  if (cn.n3 > 0) put_units<D, 1>(from(1), base + r_new[QC3], L.mask2, old_units(QC3, (min(c_old.n3, cn.n3) + 15) / 16), cn.n3, 0, 0, stage, L);
  if (cn.n4 > 0) put_units<D, 4>(from(2), base + r_new[QC4], L.mask4, old_units(QC4, (min(c_old.n4, cn.n4) + 7) / 8), cn.n4, n32n, 0, stage, L);
  if (HAS1 && cn.n1 > 0) put_units<D, 1>(from(3), base + r_new[QC1], L.mask1b, old_units(QC1, (min(c_old.n1, cn.n1) + 15) / 16), cn.n1, cn.first1(), 0, stage, L);
  if (cn.n8 > 0)
    for (int it = tid; it < n_moved * (D / 16); it += NT) {        // 8-bit tokens: token-major bytes, 16 per item
      const int m = it / (D / 16), dq = 4 * (it % (D / 16));
      const uint32_t e = mv[m];
      if ((e >> 28) != 8u) continue;
      const int sl = (int)((e >> 8) & 0xffu);
      const uint8_t* row = (const uint8_t*)&stage[m * SROW] + (dq >> 2);      // channel group dq / 4
      uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int n = 0; n < 16; ++n) w[n >> 2] |= (uint32_t)row[n * (D / 16)] << (8 * (n & 3));
      *(uint4*)(base + r_new[QC8] + (uint32_t)(sl - n32n - cn.n4) * D + 4u * (uint32_t)dq) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

template <int D, bool ONE, bool HAS1>
__global__ __launch_bounds__(128, 8) void k_update(QaqBuildArgs a) { update_side<D, ONE, HAS1, 2>(a); }
template <int D, bool ONE, bool HAS1>
__global__ __launch_bounds__(256, 4) void k_update_few(QaqBuildArgs a) { update_side<D, ONE, HAS1, 4>(a); }

// ---------------------------------------------------------------------------------
// Width selection (Section 4.1 bit rules written as comparisons, Section 4.2 window).
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_select(QaqSelectArgs a) {
  qaq_request_arguments<0, offsetof(QaqSelectArgs, tau_k)>();
  __shared__ float rk[QAQ_TT], rv[QAQ_TT];
  const QaqView& v = a.v;
  const int tid = threadIdx.x;
  const int tile = blockIdx.x, bh = blockIdx.y, b = bh / v.Hkv, h = bh % v.Hkv;
  const int t0 = tile * QAQ_TT;
  const int n_tok = min(qaq_seq_len(v, b, a.len) - t0, QAQ_TT);
  if (n_tok <= 0) return;
  // all loads first (slot-order ranges, this step's scores, the window rows), one barrier,
  // then the comparisons
  const int t = t0 + tid;
  const size_t ring_row = (size_t)v.B * v.Hkv * v.Tmax;
  const size_t ri = qaq_bh(v, b, h) * v.Tmax + t;
  float pred = 0.0f;
  if (tid < n_tok) {
    const size_t gi = qaq_slot_index(v, b, h, tile, tid);
    const uint32_t mk = v.mm[0][gi], mv = v.mm[1][gi];
    const int pk = v.perm[0][gi], pv = v.perm[1][gi];
    float s;
    const uint32_t covered = qaq_rows_covering(v, a.row_len, b, t);
    pred = a.scores ? qaq_predicted<true>(v, covered, a.new_row, ri, t, a.scores, (size_t)b * v.Hq + h * a.G, a.G, (size_t)a.len, &s)
                    : qaq_predicted<false>(v, covered, -1, ri, t, nullptr, 0, 0, 0, &s);
    if (a.scores) qaq_ring_store(v, (size_t)a.new_row * ring_row + ri, s);
    rk[pk] = h2f((uint16_t)(mk >> 16)) - h2f((uint16_t)(mk & 0xffffu));
    rv[pv] = h2f((uint16_t)(mv >> 16)) - h2f((uint16_t)(mv & 0xffffu));
  }
  __syncthreads();
  if (tid >= n_tok) return;
  const float tau = a.tau_k[v.ragged ? b * v.Hkv + h : h];
  const float c_v = a.c_v[v.ragged ? b : 0];
  const float lhs_v = rv[tid] * pred;
  int bk = a.bit_set[a.nbits - 1], bv = a.bit_set[a.nbits - 1];
  for (int i = a.nbits - 1; i >= 0; --i) {
    const int bb = a.bit_set[i];
    if (rk[tid] <= ldexpf(tau, bb)) bk = bb;
    if (lhs_v <= ldexpf(c_v, bb)) bv = bb;
  }
  a.out_bits[0][(size_t)bh * a.len + t] = (uint8_t)bk;
  a.out_bits[1][(size_t)bh * a.len + t] = (uint8_t)bv;
}

// ---------------------------------------------------------------------------------
// Canonical export (tests, export; not on the decode path) and dequantization.
// ---------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kThreads) void k_export(QaqExportArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  TileLds<D>& L = *reinterpret_cast<TileLds<D>*>(smem_raw);
  const QaqView& v = a.v;
  const int tid = threadIdx.x;
  const int tile = blockIdx.x, bh = blockIdx.y, b = bh / v.Hkv, h = bh % v.Hkv;
  const int t0 = tile * QAQ_TT;
  const int n_tok = min(qaq_seq_len(v, b, a.len) - t0, QAQ_TT);
  if (n_tok <= 0) return;
  tile_load<D>(v, a.side, b, h, tile, n_tok, L);
  if (tid < n_tok) {
    const size_t o = (size_t)bh * a.len + t0 + tid;
    if (a.bits) a.bits[o] = L.bits[tid];
    if (a.minmax) { a.minmax[2 * o] = (uint16_t)(L.mm[tid] & 0xffffu); a.minmax[2 * o + 1] = (uint16_t)(L.mm[tid] >> 16); }
    for (int k = 0; k < v.no2; ++k) {
      if (a.oidx) a.oidx[o * v.no2 + k] = L.oidx[tid][k];
      if (a.oval) a.oval[o * v.no2 + k] = L.oval[tid][k];
    }
  }
  if (a.codes) {
    for (int e = tid; e < n_tok * D; e += kThreads) {
      const int pos = e / D, k = e % D;
      const int bits = L.bits[pos];
      uint32_t byte = 0;
      if (k < D * bits / 8) {
        for (int j = 0; j < 8; ++j) {
          const int gb = 8 * k + j;
          const int d = gb / bits, bit = gb % bits;
          byte |= ((L.stage[pos][d] >> bit) & 1u) << j;
        }
      }
      a.codes[((size_t)bh * a.len + t0 + pos) * D + k] = (uint8_t)byte;
    }
  }
}

// Dequantization.  Bound by the fp16 rows it writes (2 D bytes per token side against D b / 8 read), so
// everything is arranged for whole-line traffic: a work item is eight channels of a token, D/8 lanes
// write one row's 2 D consecutive bytes with 16-byte stores, and codes are read in the words they are
// stored in and spread four at a time by masks, not code by code.  Keys: slot order, an item's word
// belongs to the token alone.  Values: an item is (unit of 16 tokens, eight channels) -- eight words, each
// one channel of the 16 tokens, turned into rows by 4x4 byte transposes; the D/8 lanes of a unit read its
// 4 D bytes between them.
// The stores want wavefronts in flight more than long ones: loops are not unrolled, so that 64 registers (72 where a token has
// more than two outliers) let 32 (28) of them live on a compute unit; unrolled they took 104 and half as many did.
// 8 sequences x 32 heads x 4096 tokens x 128 channels, all 8-bit (805 MB): 1232 us code by code through an LDS staging
// tile, 209 us (3.8 TB/s; a 4 GiB copy: 4.85) with whole words at 16 wavefronts, 175 (4.6) at 32; widths of mean 2.5 / 2.1
// (615 MB) 203 -> 101; 64 channels, mean 4 / 3, 112 -> 68; three outliers per end 250 -> 174.

// eight codes (one per byte, channels in order) -> eight fp16 values, with the outliers among these channels
// put in: ch0 = first channel, NO2 outlier entries per token (idx: one byte each, 0xff = unused)
template <int NO2>
struct DequantToken {
  float scale, mn;
  uint32_t idx[(NO2 + 3) / 4 > 0 ? (NO2 + 3) / 4 : 1];
  uint32_t val[(NO2 + 1) / 2 > 0 ? (NO2 + 1) / 2 : 1];
  __device__ __forceinline__ uint4 eight(uint32_t lo, uint32_t hi, int ch0) const {
    uint32_t h[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t w = j < 2 ? lo : hi;
      const float c0 = (float)((w >> (16 * (j & 1))) & 0xffu) + 0.5f, c1 = (float)((w >> (16 * (j & 1) + 8)) & 0xffu) + 0.5f;
      const float p0 = c0 * scale, p1 = c1 * scale;
      h[j] = (uint32_t)f2h(p0 + mn) | ((uint32_t)f2h(p1 + mn) << 16);
    }
#pragma unroll
    for (int k = 0; k < NO2; ++k) {
      const int rel = (int)((idx[k >> 2] >> (8 * (k & 3))) & 0xffu) - ch0;
      if ((unsigned)rel < 8u) {
        const uint32_t ov = (val[k >> 1] >> (16 * (k & 1))) & 0xffffu;
        const uint32_t m = rel & 1 ? 0xffff0000u : 0xffffu, x = ov | (ov << 16);
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = (rel >> 1) == j ? ((h[j] & ~m) | (x & m)) : h[j];
      }
    }
    return make_uint4(h[0], h[1], h[2], h[3]);
  }
};

// NO2: outlier entries per token: 0, 2, or up to 8 (the run-time count v.no2; also the variable-length store)
template <int D, int NO2>
__global__ __launch_bounds__(kThreads, (NO2 > 2 ? 6 : 8)) void k_dequant(QaqDequantArgs a) {
  constexpr int NI = NO2 ? (NO2 + 3) / 4 : 1, NV = NO2 ? (NO2 + 1) / 2 : 1;
  constexpr int LPT = D / 8, KS = D / 64;
  __shared__ float s_scale[QAQ_TT], s_mn[QAQ_TT];
  __shared__ int s_row[QAQ_TT];                  // by slot: output row, -1 = outside [t0, t1)
  __shared__ uint32_t s_idx[NI][QAQ_TT], s_val[NV][QAQ_TT];
  const QaqView& v = a.v;
  const int tid = threadIdx.x;
  // heads fastest, then tiles (see k_build)
  const int bh = blockIdx.x, b = bh / v.Hkv, h = bh % v.Hkv;
  const int tile = a.t0 / QAQ_TT + blockIdx.y;
  const int side = blockIdx.z;
  if (a.out[side] == nullptr) return;
  const int t0 = tile * QAQ_TT;
  const int n_tok = min(qaq_seq_len(v, b, a.len) - t0, QAQ_TT);
  if (n_tok <= 0) return;
  const QaqCounts c = qaq_load_counts(v, side, b, h, tile, n_tok);
  if (tid < n_tok) {
    const size_t gi = qaq_slot_index(v, b, h, tile, tid);
    const int pos = v.perm[side][gi];
    const uint32_t mm = v.mm[side][gi];
    uint32_t ix[NI], vx[NV];
#pragma unroll
    for (int k = 0; k < NI; ++k) ix[k] = 0xffffffffu;
#pragma unroll
    for (int k = 0; k < NV; ++k) vx[k] = 0u;
    if constexpr (NO2 == 2) {
      ix[0] = *(const uint16_t*)(v.oidx[side] + gi * 2) | 0xffff0000u;
      vx[0] = *(const uint32_t*)(v.oval[side] + gi * 2);
    } else if constexpr (NO2 > 2) {
      size_t e0 = gi * v.no2;
      int cnt = v.no2;
      if (v.csr) {
        const size_t g0 = qaq_slot_index(v, b, h, tile, 0);
        cnt = v.ocnt[side][g0 + pos];
        e0 = g0 * v.no2 + v.ostart[side][g0 + pos];
      }
#pragma unroll
      for (int k = 0; k < NO2; ++k)
        if (k < cnt) {
          ix[k >> 2] = (ix[k >> 2] & ~(0xffu << (8 * (k & 3)))) | ((uint32_t)v.oidx[side][e0 + k] << (8 * (k & 3)));
          vx[k >> 1] |= (uint32_t)v.oval[side][e0 + k] << (16 * (k & 1));
        }
    }
    const float mn = h2f((uint16_t)(mm & 0xffffu)), mx = h2f((uint16_t)(mm >> 16));
    s_scale[tid] = ldexpf(mx - mn, -c.bits_of_slot(tid));
    s_mn[tid] = mn;
    const int t = t0 + pos;
    s_row[tid] = t >= a.t0 && t < a.t1 ? t - a.t0 : -1;
#pragma unroll
    for (int k = 0; k < NI; ++k) s_idx[k][tid] = ix[k];
#pragma unroll
    for (int k = 0; k < NV; ++k) s_val[k][tid] = vx[k];
  }
  __syncthreads();
  const uint8_t* base = qaq_tile_codes(v, side, b, h, tile);
  __half* out = a.out[side] + (size_t)bh * (a.t1 - a.t0) * D;
  auto put = [&](int slot, int ch0, uint32_t lo, uint32_t hi) {
    const int row = s_row[slot];
    if (row < 0) return;
    DequantToken<NO2> tk;
    tk.scale = s_scale[slot]; tk.mn = s_mn[slot];
#pragma unroll
    for (int k = 0; k < NI; ++k) tk.idx[k] = s_idx[k][slot];
#pragma unroll
    for (int k = 0; k < NV; ++k) tk.val[k] = s_val[k][slot];
    const uint4 x = tk.eight(lo, hi, ch0);
    // (the output may start at any fp16: the type says so, and it still is one 16-byte store)
    typedef uint32_t u32x4_of_halves __attribute__((ext_vector_type(4), aligned(2)));
    const u32x4_of_halves xv = {x.x, x.y, x.z, x.w};
    __builtin_nontemporal_store(xv, (u32x4_of_halves*)(out + (size_t)row * D + ch0));      // written once, read by somebody else
  };
  const int n32 = c.n32(), first8 = n32 + c.n4, first1 = c.first1();
  if (side == 0) {
    const QaqKRegions r = qaq_k_regions(c, D);
#pragma unroll 1
    for (int it = tid; it < n_tok * LPT; it += kThreads) {
      const int s = it / LPT, c8 = it % LPT;           // channels 8 c8 .. +7: half `hf` of slice q
      const int hf = c8 & 1, q = ((c8 >> 1) & 3) * KS + (c8 >> 3);
      uint32_t lo, hi;
      if (s < n32) {
        const uint32_t w = *(const uint32_t*)(base + r.r2 + (uint32_t)s * (D / 4) + 4u * (uint32_t)q) >> (4 * hf);
        lo = w & 0x03030303u; hi = (w >> 2) & 0x03030303u;
        if (s < c.n3) {
          const uint32_t l = *(const uint32_t*)(base + r.r1 + (uint32_t)s * (D / 8) + 4u * (uint32_t)(q >> 1)) >> (4 * (q & 1) + 2 * hf);
          lo = (lo << 1) | (l & 0x01010101u); hi = (hi << 1) | ((l >> 1) & 0x01010101u);
        }
      } else if (s < first8) {
        const uint32_t w = *(const uint32_t*)(base + r.r4 + (uint32_t)(s - n32) * (D / 2) + 4u * (uint32_t)(2 * q + hf));
        lo = w & 0x0f0f0f0fu; hi = (w >> 4) & 0x0f0f0f0fu;
      } else if (s < first1) {
        const uint2 w = *(const uint2*)(base + r.r8 + (uint32_t)(s - first8) * D + 16u * (uint32_t)q + 8u * (uint32_t)hf);
        lo = w.x ^ 0x80808080u; hi = w.y ^ 0x80808080u;
      } else {
        const uint32_t l = *(const uint32_t*)(base + r.r1b + (uint32_t)(s - first1) * (D / 8) + 4u * (uint32_t)(q >> 1)) >> (4 * (q & 1) + 2 * hf);
        lo = l & 0x01010101u; hi = (l >> 1) & 0x01010101u;
      }
      put(s, 8 * c8, lo, hi);
    }
    return;
  }
  const QaqVRegions r = qaq_v_regions(c, D);
  // the 2-bit field units (and the low bits of the 3-bit tokens among them)
  for (int it = tid; it < ((n32 + 15) / 16) * LPT; it += kThreads) {
    const int u = it / LPT, c8 = it % LPT, cg = c8 >> 1, n0 = 8 * (c8 & 1);     // channels 16 cg + n0 .. +7
    uint32_t w[8], l[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) w[k] = *(const uint32_t*)(base + r.r2 + (uint32_t)u * (4 * D) + 4u * (uint32_t)((n0 + k) * (D / 16) + cg));
    const bool low = 16 * u < c.n3;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      l[k] = low ? *(const uint32_t*)(base + r.r1 + (uint32_t)u * (2 * D) + 4u * (uint32_t)((n0 + k) * (D / 32) + (cg >> 1))) >> (4 * (cg & 1)) : 0u;
#pragma unroll 1
    for (int vq = 0; vq < 4; ++vq) {
      uint32_t x[4], tl[4], th[4], ll[4], lh[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = (w[k] >> (2 * vq)) & 0x03030303u;
      transpose4(x, tl);
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = (w[4 + k] >> (2 * vq)) & 0x03030303u;
      transpose4(x, th);
      if (low) {
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = (l[k] >> vq) & 0x01010101u;
        transpose4(x, ll);
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = (l[4 + k] >> vq) & 0x01010101u;
        transpose4(x, lh);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int s = 16 * u + 4 * vq + j;
        if (s >= n32) break;
        uint32_t lo = tl[j], hi = th[j];
        if (s < c.n3) { lo = (lo << 1) | ll[j]; hi = (hi << 1) | lh[j]; }
        put(s, 8 * c8, lo, hi);
      }
    }
  }
  for (int it = tid; it < ((c.n4 + 7) / 8) * LPT; it += kThreads) {
    const int hu = it / LPT, c8 = it % LPT, cg = c8 >> 1, n0 = 8 * (c8 & 1);
    uint32_t w[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) w[k] = *(const uint32_t*)(base + r.r4 + (uint32_t)hu * (4 * D) + 4u * (uint32_t)((n0 + k) * (D / 16) + cg));
#pragma unroll 1
    for (int vq = 0; vq < 2; ++vq) {
      uint32_t x[4], tl[4], th[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = (w[k] >> (4 * vq)) & 0x0f0f0f0fu;
      transpose4(x, tl);
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = (w[4 + k] >> (4 * vq)) & 0x0f0f0f0fu;
      transpose4(x, th);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i4 = 8 * hu + 4 * vq + j;
        if (i4 < c.n4) put(n32 + i4, 8 * c8, tl[j], th[j]);
      }
    }
  }
#pragma unroll 1
  for (int it = tid; it < c.n8 * LPT; it += kThreads) {        // token-major bytes
    const int i8 = it / LPT, c8 = it % LPT;
    const uint2 w = *(const uint2*)(base + r.r8 + (uint32_t)i8 * D + 8u * (uint32_t)c8);
    put(first8 + i8, 8 * c8, w.x, w.y);
  }
  for (int it = tid; it < ((c.n1 + 15) / 16) * LPT; it += kThreads) {
    const int u = it / LPT, c8 = it % LPT, cg = c8 >> 1, n0 = 8 * (c8 & 1);
    uint32_t l[8];
#pragma unroll
    for (int k = 0; k < 8; ++k)
      l[k] = *(const uint32_t*)(base + r.r1b + (uint32_t)u * (2 * D) + 4u * (uint32_t)((n0 + k) * (D / 32) + (cg >> 1))) >> (4 * (cg & 1));
#pragma unroll 1
    for (int vq = 0; vq < 4; ++vq) {
      uint32_t x[4], tl[4], th[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = (l[k] >> vq) & 0x01010101u;
      transpose4(x, tl);
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = (l[4 + k] >> vq) & 0x01010101u;
      transpose4(x, th);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i1 = 16 * u + 4 * vq + j;
        if (i1 < c.n1) put(first1 + i1, 8 * c8, tl[j], th[j]);
      }
    }
  }
}

// ---------------------------------------------------------------------------------
// Accounting.
// statbuf: [0..3] hist K (2,3,4,8), [4..7] hist V, [8] layout code bytes, [9] meta bytes,
// [10], [11] 1-bit token-heads K, V, [12], [13] widenings refused / served since the cache was made
// ---------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_stats(QaqView v, int len) {
  __shared__ unsigned long long acc[14];
  const int tid = threadIdx.x;
  if (tid < 14) acc[tid] = 0;
  __syncthreads();
  const int ntile = (len + QAQ_TT - 1) / QAQ_TT;
  const long long total = (long long)v.B * v.Hkv * ntile * 2;
  unsigned long long loc[14] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (long long i = (long long)blockIdx.x * kThreads + tid; i < total; i += (long long)gridDim.x * kThreads) {
    const int side = (int)(i & 1);
    const long long j = i >> 1;
    const int tile = (int)(j % ntile);
    const int bh = (int)(j / ntile);
    const int n_tok = min(qaq_seq_len(v, bh / v.Hkv, len) - tile * QAQ_TT, QAQ_TT);
    if (n_tok <= 0) continue;      // past the end of a shorter sequence
    const QaqCounts c = qaq_load_counts(v, side, bh / v.Hkv, bh % v.Hkv, tile, n_tok);
    loc[side * 4 + 0] += c.n2; loc[side * 4 + 1] += c.n3; loc[side * 4 + 2] += c.n4; loc[side * 4 + 3] += c.n8;
    loc[10 + side] += c.n1;

    // bytes a scan reads: key records one by one, value planes in whole units
    loc[8] += side == 0 ? (unsigned long long)c.n32() * (v.D / 4) + (c.n3 + c.n1) * (v.D / 8) + c.n4 * (v.D / 2) + c.n8 * v.D
                        : qaq_v_regions(c, v.D).end;
    if (!v.csr) loc[9] += (unsigned long long)c.total() * (4 + 1 + 3 * v.no2);
    else {   // min/max, order byte, (offset, count), and the entries the tile's pool holds
      const size_t pl = qaq_slot_index(v, bh / v.Hkv, bh % v.Hkv, tile, c.total() - 1);
      loc[9] += (unsigned long long)c.total() * (4 + 1 + 3) + 3ull * ((unsigned)v.ostart[side][pl] + (unsigned)v.ocnt[side][pl]);
    }
  }
  // widenings: every tile side the cache has room for (a cache that was reset keeps its history)
  const long long sides = (long long)v.B * v.Hkv * v.NT * 2;
  for (long long i = (long long)blockIdx.x * kThreads + tid; i < sides; i += (long long)gridDim.x * kThreads) {
    loc[12] += v.refused[2 * i]; loc[13] += v.refused[2 * i + 1];
  }
  for (int k = 0; k < 14; ++k) if (loc[k]) atomicAdd(&acc[k], loc[k]);
  __syncthreads();
  if (tid < 14 && acc[tid]) atomicAdd((unsigned long long*)&v.statbuf[tid], acc[tid]);
}

__global__ void k_init(QaqView v) {
  const size_t n = (size_t)v.B * v.Hkv * v.NT * 2 * 4;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) v.counts[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x < 32) v.statbuf[threadIdx.x] = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < (size_t)v.B * v.Hkv * v.NT * 4; i += (size_t)gridDim.x * blockDim.x) v.refused[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x < 3) v.todo_count[threadIdx.x] = 0;
}

__global__ void k_clear_stats(QaqView v) {
  if (threadIdx.x < 32) v.statbuf[threadIdx.x] = 0;
}

}  // namespace

hipError_t qaq_launch_init(const QaqView& v, hipStream_t s) {
  hipLaunchKernelGGL(k_init, dim3(64), dim3(256), 0, s, v);
  return hipGetLastError();
}

hipError_t qaq_launch_build(const QaqBuildArgs& a, int ntiles, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  dim3 grid(a.v.B * a.v.Hkv, ntiles, 2);
  const bool one = a.v.no2 == 2 && !a.v.csr;      // (the one-per-end search has no threshold test)
  if (a.v.D == 128) {
    if (a.v.has1) {
      if (one) hipLaunchKernelGGL((k_build<128, true, true>), grid, dim3(kThreads), 0, s, a);
      else hipLaunchKernelGGL((k_build<128, false, true>), grid, dim3(kThreads), 0, s, a);
    } else {
      if (one) hipLaunchKernelGGL((k_build<128, true, false>), grid, dim3(kThreads), 0, s, a);
      else hipLaunchKernelGGL((k_build<128, false, false>), grid, dim3(kThreads), 0, s, a);
    }
  } else {
    if (a.v.has1) {
      if (one) hipLaunchKernelGGL((k_build<64, true, true>), grid, dim3(kThreads), 0, s, a);
      else hipLaunchKernelGGL((k_build<64, false, true>), grid, dim3(kThreads), 0, s, a);
    } else {
      if (one) hipLaunchKernelGGL((k_build<64, true, false>), grid, dim3(kThreads), 0, s, a);
      else hipLaunchKernelGGL((k_build<64, false, false>), grid, dim3(kThreads), 0, s, a);
    }
  }
  return hipGetLastError();
}

template <int D, bool ONE, bool HAS1>
static hipError_t launch_update(const QaqBuildArgs& a_in, int ntiles, float moving, bool* whole, hipStream_t s) {
  QaqBuildArgs a = a_in;
  const long long sides = (long long)a.v.B * a.v.Hkv * ntiles * 2;
  // LDS for moved tokens: what is left of a compute unit's 160 KB when all value sides are resident at once (the key
  // sides, few of which have work, take the places that become free), from a sixteenth -- 64 tokens of 128 channels, 120
  // of 64 -- up to a whole tile, which leaves nothing for the general kernel to do (a batch of six with unequal prompts,
  // 72 heads in all: 20.4 + 13.8 us with staging for 60 tokens and the second launch, 17.4 us without)
  constexpr int lds = 160 * 1024, grain = 1280;       // (LDS is handed out 1280 bytes at a time)
  constexpr int least = (lds / kUpdResident / grain * grain - (int)sizeof(UpdLds<D, 2>)) / UpdLds<D, 2>::PER_TOKEN;
  static_assert(least == (D == 128 ? 64 : 120), "the figures above and those at expected_moves");
  static_assert(least * UpdLds<D, 2>::PER_TOKEN >= 2 * QAQ_TT * 4, "the space also holds two words per position before any code is staged");
  const int cus = qaq_compute_units();
  const long long resident = (sides / 2 + cus - 1) / cus;
  const bool few = resident <= kUpdFew;
  const int room = lds / (int)(resident < kUpdResident ? resident : kUpdResident) / grain * grain - (int)(few ? sizeof(UpdLds<D, 4>) : sizeof(UpdLds<D, 2>));
  a.max_moved = room / UpdLds<D, 2>::PER_TOKEN;
  a.open_first = sides > (long long)kUpdResident * cus;
  if (a.max_moved > QAQ_TT) a.max_moved = QAQ_TT;
  *whole = a.max_moved < QAQ_TT && moving * QAQ_TT >= (float)a.max_moved;
  if (*whole) return qaq_launch_build(a_in, ntiles, s);
  const size_t staging = (size_t)a.max_moved * UpdLds<D, 2>::PER_TOKEN;
  if (few) hipLaunchKernelGGL((k_update_few<D, ONE, HAS1>), dim3(a.v.B * a.v.Hkv, ntiles, 2), dim3(256), staging, s, a);
  else hipLaunchKernelGGL((k_update<D, ONE, HAS1>), dim3(a.v.B * a.v.Hkv, ntiles, 2), dim3(128), staging, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.max_moved == QAQ_TT) return e;
  // The tile sides it handed over (their number is only known on the device): as many workgroups as a compute unit holds
  // at the kernel's registers and LDS.  An empty list costs the same with 512 and with 1536 of them (4.6 us, the launch).
  const long long most = (long long)listed_per_cu<D, ONE>() * cus;
  hipLaunchKernelGGL((k_build_listed<D, ONE, HAS1>), dim3((unsigned)(sides < most ? sides : most)), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t qaq_launch_update(const QaqBuildArgs& a, int ntiles, float moving, bool* whole, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  const bool one = a.v.no2 == 2 && !a.v.csr;
  if (a.v.D == 128) {
    if (a.v.has1) return one ? launch_update<128, true, true>(a, ntiles, moving, whole, s) : launch_update<128, false, true>(a, ntiles, moving, whole, s);
    return one ? launch_update<128, true, false>(a, ntiles, moving, whole, s) : launch_update<128, false, false>(a, ntiles, moving, whole, s);
  }
  if (a.v.has1) return one ? launch_update<64, true, true>(a, ntiles, moving, whole, s) : launch_update<64, false, true>(a, ntiles, moving, whole, s);
  return one ? launch_update<64, true, false>(a, ntiles, moving, whole, s) : launch_update<64, false, false>(a, ntiles, moving, whole, s);
}

hipError_t qaq_launch_select(const QaqSelectArgs& a, hipStream_t s) {
  const int ntile = (a.len + QAQ_TT - 1) / QAQ_TT;
  if (ntile <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_select, dim3(ntile, a.v.B * a.v.Hkv), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t qaq_launch_export(const QaqExportArgs& a, hipStream_t s) {
  const int ntile = (a.len + QAQ_TT - 1) / QAQ_TT;
  if (ntile <= 0) return hipSuccess;
  dim3 grid(ntile, a.v.B * a.v.Hkv);
  if (a.v.D == 128) hipLaunchKernelGGL(k_export<128>, grid, dim3(kThreads), sizeof(TileLds<128>), s, a);
  else hipLaunchKernelGGL(k_export<64>, grid, dim3(kThreads), sizeof(TileLds<64>), s, a);
  return hipGetLastError();
}

hipError_t qaq_launch_dequant(const QaqDequantArgs& a, hipStream_t s) {
  if (a.t1 <= a.t0) return hipSuccess;
  const int tile_lo = a.t0 / QAQ_TT, tile_hi = (a.t1 - 1) / QAQ_TT;
  const dim3 grid(a.v.B * a.v.Hkv, tile_hi - tile_lo + 1, 2), block(kThreads);
  const int no2 = a.v.csr ? QAQ_MAX_NO2 : a.v.no2;
  if (a.v.D == 128) {
    if (no2 == 2) hipLaunchKernelGGL((k_dequant<128, 2>), grid, block, 0, s, a);
    else if (no2 == 0) hipLaunchKernelGGL((k_dequant<128, 0>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_dequant<128, QAQ_MAX_NO2>), grid, block, 0, s, a);
  } else {
    if (no2 == 2) hipLaunchKernelGGL((k_dequant<64, 2>), grid, block, 0, s, a);
    else if (no2 == 0) hipLaunchKernelGGL((k_dequant<64, 0>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_dequant<64, QAQ_MAX_NO2>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

hipError_t qaq_launch_stats(const QaqView& v, int len, hipStream_t s) {
  hipLaunchKernelGGL(k_clear_stats, dim3(1), dim3(64), 0, s, v);
  hipLaunchKernelGGL(k_stats, dim3(64), dim3(kThreads), 0, s, v, len);
  return hipGetLastError();
}
