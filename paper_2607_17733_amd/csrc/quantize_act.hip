// quantize_act.hip -- online MXINT quantization of bf16 activation rows.
//
// MXSens (arXiv 2607.17733) Section 2 and Section 4.1: every 32-element
// block of the permuted row gets one shared exponent E = floor(log2 max|x|)
// + 127 and mantissas of its own width m in {4, 6, 8} (or 3, stored as 2q in
// the 4-bit layout).
//
// Work decomposition.  A workgroup owns R consecutive rows (1 to 64, by the
// number of rows and CUs) and stages them in LDS, so the permutation becomes
// an LDS gather (entries outside [0, K) take the zero padding after the row).
// The (row, padded block) items come in chunks of 64, a wave each, that never
// straddle two segments, so a wave runs the code of one width.  Lanes run
// over rows fastest, so the rows of a block write contiguous runs of the
// operand tiles (whole 128-byte lines at R = 8), and consecutive workgroups
// run on one XCD, whose L2 then completes every line of the tile.  The same
// kernel packs the weights (a row is a weight column): 14336 x 4096 in 37 us
// (155 MB), where a workgroup per row with a quarter block per thread took
// 173.
//
// Arithmetic.  The block maximum is taken on the integer |bf16| patterns (two
// per register); the mantissas are computed in fp32, where every step is
// exact: x * 2^-s scales an 8-bit significand by a power of two, rint and the
// clamp act on integers below 2^8.  The packed row is assembled from the
// integers' low bytes, four elements per register.  The operand image uses the
// gfx950 scaled FP6/FP8 conversions (the values are exact in the target format,
// so they never round).
#include "mxq_device.h"
#include "mxq_internal.h"
#include <algorithm>
#include <atomic>

namespace mxq {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned v6u __attribute__((ext_vector_type(6)));
typedef short v2s __attribute__((ext_vector_type(2)));
typedef unsigned short v2us __attribute__((ext_vector_type(2)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kMaxThreads = 1024;
constexpr int kRowPad = 8;              // zero bf16 elements after each staged row

// A block of 32 values kept as its even and odd elements (the register
// layout the FP6 conversion takes).
struct Blk {
  v16f e, o;
  __device__ float operator[](int t) const { return (t & 1) ? o[t >> 1] : e[t >> 1]; }
};

// 32 values / div as FP6 e3m2 codes, element t at bits 6t of 24 bytes (the
// conversion interleaves its two 16-element inputs).
__device__ inline v6u to_e3m2(const Blk &v, float div) {
  return __builtin_amdgcn_cvt_scalef32_2xpk16_bf6_f32(v.e, v.o, div);
}

// Elements 16h..16h+15 / div as FP8 e4m3 codes, one byte each.
__device__ inline u4 to_e4m3(const Blk &v, int h, float div) {
  u4 r;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const int t = 16 * h + 4 * d;
    v2s z = {0, 0};
    z = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(z, v[t], v[t + 1], div, false);
    z = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(z, v[t + 2], v[t + 3], div, true);
    r[d] = ((uint32_t)(uint16_t)z[1] << 16) | (uint16_t)z[0];
  }
  return r;
}

// Low bytes of the integers of elements t0, t0+step, t0+2step, t0+3step.
__device__ inline uint32_t byte_lanes(const Blk &v, int t0, int step) {
  return ((uint32_t)(int)v[t0] & 255u) | (((uint32_t)(int)v[t0 + step] & 255u) << 8) |
         (((uint32_t)(int)v[t0 + 2 * step] & 255u) << 16) |
         ((uint32_t)(int)v[t0 + 3 * step] << 24);
}

// Two's-complement nibbles of elements t0..t0+7 (element t0+t at bits 4t):
// byte j takes element t0+2j in its low and t0+2j+1 in its high nibble.
__device__ inline uint32_t nibbles8(const Blk &v, int t0) {
  const uint32_t ev = byte_lanes(v, t0, 2), od = byte_lanes(v, t0 + 1, 2);
  return (ev & 0x0F0F0F0Fu) | ((od & 0x0F0F0F0Fu) << 4);
}

// Two's-complement bytes of elements t0..t0+3.
__device__ inline uint32_t bytes4(const Blk &v, int t0) { return byte_lanes(v, t0, 1); }

// Top-bit word d of a 6-bit block (canonical packed layout): byte j holds
// the signed top two bits (bits 4-5) of elements 16d+2j, 16d+2j+1,
// 16d+8+2j, 16d+9+2j in bits 6-7, 4-5, 2-3, 0-1.
__device__ inline uint32_t top_word(const Blk &v, int d) {
  const uint32_t a = byte_lanes(v, 16 * d, 2), b = byte_lanes(v, 16 * d + 1, 2);
  const uint32_t c = byte_lanes(v, 16 * d + 8, 2), e = byte_lanes(v, 16 * d + 9, 2);
  return ((a & 0x30303030u) << 2) | (b & 0x30303030u) | ((c & 0x30303030u) >> 2) |
         ((e & 0x30303030u) >> 4);
}

// The 3-bit two's-complement codes of the 32 elements, element t at bits 3t
// of 96 bits (canonical packed row).
__device__ inline void pack3(const Blk &v, uint32_t *w) {
  w[0] = w[1] = w[2] = 0;
#pragma unroll
  for (int t = 0; t < 32; ++t) {
    const uint32_t c = (uint32_t)(int)v[t] & 7u;
    const int b = 3 * t;
    w[b >> 5] |= c << (b & 31);
    if ((b & 31) > 29) w[(b >> 5) + 1] |= c >> (32 - (b & 31));
  }
}

// Where padded block rem of segment SEG goes: its step, position in the
// step, its block of the width map, and the step's offset in a 16-row tile
// of the operand image and its scale group and byte.  The segment is a
// compile-time constant, so every per-segment quantity is a constant index
// into the width map's geometry.
struct ItemGeo {
  int s, rem, pos, b;
  bool pad;
  int step_off, group, byte;
};
template <int SEG>
__device__ inline ItemGeo item_geo_seg(const LGeo &lg, int rem) {
  ItemGeo g;
  constexpr int two = SEG < 2 ? 2 : 1;               // log2 blocks per step
  const int k = rem >> two;
  g.s = SEG;
  g.rem = rem;
  g.pos = rem & ((1 << two) - 1);
  g.pad = rem >= lg.nb[SEG];
  g.b = lg.b0[SEG] + rem;
  constexpr int sb = kLanes * a_lane_bytes(0);       // 3/4/6-bit step bytes
  int before = 0;
#pragma unroll
  for (int i = 0; i < SEG; ++i) before += lg.S[i];
  g.step_off = before * sb + k * (SEG == 3 ? kLanes * a_lane_bytes(3) : sb);
  g.group = lg.G0[SEG] + (k >> 2);
  g.byte = k & (kGroupSteps - 1);
  return g;
}
// The items of a row group in chunks of 64 (a wave each), every chunk inside
// one segment, so that a wave runs one segment's code: W[s] chunks hold the
// padded blocks of segment s of the group's 2^lg rows.
struct Chunks {
  int W[kSegs], total;
  __device__ Chunks(const LGeo &lg, int lg_rows) {
    total = 0;
#pragma unroll
    for (int s = 0; s < kSegs; ++s) {
      W[s] = (((lg.S[s] * (s < 2 ? 4 : 2)) << lg_rows) + 63) >> 6;
      total += W[s];
    }
  }
};

// What a launch writes: the GEMMs' operand image of activations, packed rows,
// or the weight layout (the row is a weight column).
enum { kModeImage, kModeRows, kModeWeights };
// Where the rows come from: as they are, RMS-normalised, SiLU(gate) * up.
enum { kProdNone, kProdRms, kProdSwiglu };

// Block `pos` of step (segment SEG, padded block rem) of weight column `row`:
// its codes in the layout both GEMMs read (LGeo in mxq_device.h) and its
// scale bytes.  v holds the block's mantissas, Eu its exponent.  The FP6
// codes s|k are the e3m2 codes of q / 16 (linear in k, so the scaled
// conversion writes them; adding +0 first gives a zero mantissa the sign 0).
template <int SEG, bool FULL>
__device__ inline void store_weights(const QuantArgs &q, const LGeo &lg, const ItemGeo &g,
                                     int64_t row, Blk &v, uint32_t Eu) {
  constexpr int CB = w_chunk_bytes(SEG, FULL);
  const int k = g.rem >> (SEG < 2 ? 2 : 1);          // step within the segment
  const int n = (int)(row & (kWCols - 1)) >> 4, c = (int)row & 15;
  uint8_t *chunk = q.mant + (row / kWCols) * q.w_super + w_seg_base<SEG, FULL>(lg) +
                   ((int64_t)k * kWSlabs + n) * CB;
  uint8_t *scl = q.exp + (row / kWCols) * q.w_super_sc + (int64_t)g.group * 2048 + n;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    v.e[i] += 0.f;
    v.o[i] += 0.f;
  }
  const int l = 16 * g.pos + c;
  if (SEG <= 1) {
    const v6u w = to_e3m2(v, 16.f);
    const uint32_t d[6] = {w[0], w[1], w[2], w[3], w[4], w[5]};
    uint32_t x[4];
    if (SEG == 0 && !FULL) {
      fold3(d, x);
      *(u2 *)(chunk + 8 * l) = u2{x[0], x[1]};
      *(uint32_t *)(chunk + 512 + 4 * l) = x[2];
    } else if (SEG == 1 && FULL) {
      *(u4 *)(chunk + 16 * l) = u4{d[0], d[1], d[2], d[3]};
      *(u2 *)(chunk + 1024 + 8 * l) = u2{d[4], d[5]};
    } else {
      fold4(d, x);
      *(u4 *)(chunk + 16 * l) = u4{x[0], x[1], x[2], x[3]};
    }
    scl[32 * l + 8 * g.byte] = (uint8_t)Eu;
  } else if (SEG == 2) {
    // |q| = 8h + l, both planes with q's sign
    Blk h, lo;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      h.e[i] = truncf(v.e[i] * 0.125f);
      h.o[i] = truncf(v.o[i] * 0.125f);
      lo.e[i] = copysignf(fmaf(h.e[i], -8.f, v.e[i]), v.e[i]);
      lo.o[i] = copysignf(fmaf(h.o[i], -8.f, v.o[i]), v.o[i]);
    }
    const v6u wl = to_e3m2(lo, 16.f), wh = to_e3m2(h, 16.f);
    const uint32_t dl[6] = {wl[0], wl[1], wl[2], wl[3], wl[4], wl[5]};
    uint32_t x[4];
    fold4(dl, x);
    *(u4 *)(chunk + 16 * l) = u4{x[0], x[1], x[2], x[3]};
    if (FULL) {
      const uint32_t dh[6] = {wh[0], wh[1], wh[2], wh[3], wh[4], wh[5]};
      fold4(dh, x);
      *(u4 *)(chunk + 512 + 16 * l) = u4{x[0], x[1], x[2], x[3]};
    } else {
      // the high plane's magnitudes only: the sign is the low plane's
      const uint32_t dh[6] = {wh[0] & kF2Q0, wh[1] & kF2Q1, wh[2] & kF2Q2,
                              wh[3] & kF2Q0, wh[4] & kF2Q1, wh[5] & kF2Q2};
      fold2(dh, x);
      *(u2 *)(chunk + 512 + 8 * l) = u2{x[0], x[1]};
    }
  } else {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      u4 w;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        uint32_t b = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          b |= w_code8((int)v[16 * j + 4 * d + i], FULL) << (8 * i);
        w[d] = b;
      }
      *(u4 *)(chunk + 32 * l + 16 * j) = w;
    }
  }
  if (SEG >= 2) {
    scl[32 * (32 * g.pos + c) + 8 * g.byte] = (uint8_t)Eu;
    scl[32 * (32 * g.pos + 16 + c) + 8 * g.byte] = (uint8_t)Eu;
  }
  // the unused scale bytes of a segment's short last group
  if (g.rem == 0) {
    const int S = lg.S[SEG], G0 = lg.G0[SEG];
    for (int kk = S; kk < (S + kGroupSteps - 1) / kGroupSteps * kGroupSteps; ++kk) {
      uint8_t *z = q.exp + (row / kWCols) * q.w_super_sc +
                   (int64_t)(G0 + kk / kGroupSteps) * 2048 + 8 * (kk % kGroupSteps) + n;
      for (int gg = 0; gg < 4; ++gg) z[32 * (16 * gg + c)] = 0;
    }
  }
}

// One (row, padded block) item: gather, quantize, write what MODE names.  sr
// is the row, in LDS followed by zero padding (or, with the identity
// permutation, in global memory).
template <bool RNA, int MODE, int SEG>
__device__ inline void quantize_item(const QuantArgs &q, const LGeo &lg, const ItemGeo &g,
                                     int64_t row, const uint8_t *sr) {
  constexpr int s = SEG;
  constexpr int m = s == 0 ? 3 : s == 1 ? 4 : s == 2 ? 6 : 8;
  const int rem = g.rem, pos = g.pos, b = g.b;
  const bool pad = g.pad;

  // gather: pr[i] holds elements 2i (low half) and 2i+1 (high half)
  uint32_t pr[16];
  const int p0 = b * kBlock;
  if (pad) {
#pragma unroll
    for (int i = 0; i < 16; ++i) pr[i] = 0;
  } else if (!q.perm) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const u4 d = *(const u4 *)(sr + 2 * (p0 + 8 * u));
#pragma unroll
      for (int k = 0; k < 4; ++k) pr[4 * u + k] = d[k];
    }
  } else {
    // entries outside [0, K) take the zero after the row
    const unsigned K = (unsigned)q.K;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int4 e = *(const int4 *)(q.perm + b * kBlock + 4 * u);
      v2us x, y;
      x.x = *(const uint16_t *)(sr + 2 * min((unsigned)e.x, K));
      x.y = *(const uint16_t *)(sr + 2 * min((unsigned)e.y, K));
      y.x = *(const uint16_t *)(sr + 2 * min((unsigned)e.z, K));
      y.y = *(const uint16_t *)(sr + 2 * min((unsigned)e.w, K));
      pr[2 * u] = __builtin_bit_cast(uint32_t, x);
      pr[2 * u + 1] = __builtin_bit_cast(uint32_t, y);
    }
  }

  // block exponent from the integer maximum of |bits|, two lanes at a time
  v2us mx = {0, 0};
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t a = pr[i] & 0x7FFF7FFFu;
    mx = __builtin_elementwise_max(mx, __builtin_bit_cast(v2us, a));
  }
  const uint32_t amax = mx.x > mx.y ? mx.x : mx.y;
  const int E = block_exponent(amax);

  // mantissas as exact integer-valued floats: rint(x * 2^(127 + m - 2 - E)),
  // clamped; a block holding Inf or NaN (E = 255) quantizes to zeros, so
  // its values are replaced by zeros first
  if (E == 255) {
#pragma unroll
    for (int i = 0; i < 16; ++i) pr[i] = 0;
  }
  Blk v;
  {
    constexpr float qmax = (float)((1 << (m - 1)) - 1);
    const float qmin = q.full_clamp ? -(qmax + 1.f) : -qmax;
    const int sh = 127 + m - 2 - E;
#pragma unroll
    for (int u = 0; u < 32; ++u) {
      const uint32_t bits = (u & 1) ? (pr[u >> 1] & 0xFFFF0000u) : (pr[u >> 1] << 16);
      float y = ldexpf(__uint_as_float(bits), sh);
      if (RNA) {
        const float tr = truncf(y);
        y = fabsf(y - tr) >= 0.5f ? tr + copysignf(1.f, y) : tr;
      } else {
        y = rintf(y);
      }
      y = __builtin_amdgcn_fmed3f(y, qmin, qmax);
      if (u & 1) v.o[u >> 1] = y; else v.e[u >> 1] = y;
    }
  }
  const uint32_t Eu = pad ? 0u : (uint32_t)E;

  if (MODE == kModeRows) {
    if (pad) return;
    q.exp[row * q.out_erb + b] = (uint8_t)E;
    // the block's offset in the packed row: 12, 16, 24 or 32 bytes per block
    const int64_t aoff = s == 0 ? 12LL * b
                       : s == 1 ? 12LL * q.n3 + 16LL * (b - q.n3)
                       : s == 2 ? 12LL * q.n3 + 16LL * (q.n4 - q.n3) + 24LL * (b - q.n4)
                                : 12LL * q.n3 + 16LL * (q.n4 - q.n3) + 24LL * q.n6 +
                                      32LL * (b - q.n4 - q.n6);
    uint8_t *p = q.mant + row * q.out_rb + aoff;
    if (m == 3) {
      uint32_t w[3];
      pack3(v, w);
      *(uint32_t *)p = w[0];
      *(uint32_t *)(p + 4) = w[1];
      *(uint32_t *)(p + 8) = w[2];
    } else if (m == 4) {
      *(u4 *)p = u4{nibbles8(v, 0), nibbles8(v, 8), nibbles8(v, 16), nibbles8(v, 24)};
    } else if (m == 6) {
      *(u2 *)p = u2{nibbles8(v, 0), nibbles8(v, 8)};
      *(u2 *)(p + 8) = u2{nibbles8(v, 16), nibbles8(v, 24)};
      *(u2 *)(p + 16) = u2{top_word(v, 0), top_word(v, 1)};
    } else {
#pragma unroll
      for (int d = 0; d < 4; ++d)
        *(u2 *)(p + 8 * d) = u2{bytes4(v, 8 * d), bytes4(v, 8 * d + 4)};
    }
    return;
  }
  if (MODE == kModeWeights) {
    if (q.full_clamp) store_weights<SEG, true>(q, lg, g, row, v, Eu);
    else store_weights<SEG, false>(q, lg, g, row, v, Eu);
    return;
  }

  // operand image (16-row tiles) and its scale words
  const int r = (int)(row & (kATileRows - 1));
  uint8_t *stp = q.img + (row >> 4) * q.a_tile + g.step_off;
  uint8_t *scw = q.img_exp + (row >> 4) * q.a_tile_sc + g.group * 256 + g.byte;
  if (s <= 1) {
    // E3M2 codes of q (4-bit) or of 2q (3-bit)
    if (s == 0) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        v.e[i] *= 2.f;
        v.o[i] *= 2.f;
      }
    }
    const int l = 16 * pos + r;
    const v6u c = to_e3m2(v, 1.f);
    *(u2 *)(stp + 24 * l) = u2{c[0], c[1]};
    *(u2 *)(stp + 24 * l + 8) = u2{c[2], c[3]};
    *(u2 *)(stp + 24 * l + 16) = u2{c[4], c[5]};
    scw[4 * l] = (uint8_t)Eu;
  } else {
    // digits q = base h + l: the high digits first, then the low digits in
    // the same registers (h is dead once its codes are formed)
    Blk d;
    constexpr float f = s == 2 ? 0.125f : 0.0625f, base = s == 2 ? 8.f : 16.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      d.e[i] = floorf(v.e[i] * f);
      d.o[i] = floorf(v.o[i] * f);
    }
    if (s == 2) {
      // lane groups 2 pos (high plane h/2) and 2 pos + 1 (low plane l/16)
      const int lh = 16 * (2 * pos) + r, ll = lh + 16;
      const v6u ch = to_e3m2(d, 2.f);
      *(u2 *)(stp + 24 * lh) = u2{ch[0], ch[1]};
      *(u2 *)(stp + 24 * lh + 8) = u2{ch[2], ch[3]};
      *(u2 *)(stp + 24 * lh + 16) = u2{ch[4], ch[5]};
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        d.e[i] = fmaf(d.e[i], -base, v.e[i]);
        d.o[i] = fmaf(d.o[i], -base, v.o[i]);
      }
      const v6u cl = to_e3m2(d, 16.f);
      *(u2 *)(stp + 24 * ll) = u2{cl[0], cl[1]};
      *(u2 *)(stp + 24 * ll + 8) = u2{cl[2], cl[3]};
      *(u2 *)(stp + 24 * ll + 16) = u2{cl[4], cl[5]};
    } else {
      // E4M3 2h and l/8; lane group 2 plane + half holds elements
      // 16 half..16 half + 15 of the plane, at byte 16 pos
#pragma unroll
      for (int e = 0; e < 2; ++e)
        *(u4 *)(stp + 32 * (16 * e + r) + 16 * pos) = to_e4m3(d, e, 0.5f);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        d.e[i] = fmaf(d.e[i], -base, v.e[i]);
        d.o[i] = fmaf(d.o[i], -base, v.o[i]);
      }
#pragma unroll
      for (int e = 0; e < 2; ++e)
        *(u4 *)(stp + 32 * (16 * (2 + e) + r) + 16 * pos) = to_e4m3(d, e, 8.f);
    }
    scw[4 * (16 * (2 * pos) + r)] = (uint8_t)Eu;
    scw[4 * (16 * (2 * pos + 1) + r)] = (uint8_t)Eu;
  }
  // the unused scale bytes of a segment's short last group
  if (rem == 0) {
    const int S = lg.S[s], G0 = lg.G0[s];
    for (int k = S; k < (S + kGroupSteps - 1) / kGroupSteps * kGroupSteps; ++k) {
      uint8_t *z = q.img_exp + (row >> 4) * q.a_tile_sc +
                   (int64_t)(G0 + k / kGroupSteps) * 256 + k % kGroupSteps;
      for (int g = 0; g < 4; ++g) z[4 * (16 * g + r)] = 0;
    }
  }
}

// Item `i` of segment SEG: block i >> lg_rows of row i mod 2^lg_rows.
template <bool RNA, int MODE, int SEG>
__device__ inline void quantize_chunk(const QuantArgs &q, const LGeo &lg, int i, int64_t r0,
                                      const uint8_t *rows, int rowB) {
  const int rem = i >> q.lg_rows, lr = i & ((1 << q.lg_rows) - 1);
  const int64_t row = r0 + lr;
  if (rem >= lg.S[SEG] * (SEG < 2 ? 4 : 2) || row >= q.out_rows) return;
  quantize_item<RNA, MODE, SEG>(q, lg, item_geo_seg<SEG>(lg, rem), row, rows + lr * rowB);
}

__device__ inline float bf16f(uint32_t b) { return __uint_as_float(b << 16); }

// float32 -> bf16 bits, round to nearest even (gfx950 converts a pair per
// instruction; a NaN stays a NaN)
__device__ inline uint32_t to_bf16(float f) {
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}

// e^t in float32, evaluated the same way on every machine: the Cody-Waite
// reduction t = k ln2 + r (ln2 split in two so that k * LN2_HI is exact)
// and the Taylor polynomial of e^r to degree 7 (|r| <= ln2 / 2), every
// operation rounded on its own (no fused multiply-add); then 2^k exactly.
__device__ inline float exp32(float t) {
#pragma clang fp contract(off)
  constexpr float kInvLn2 = __builtin_bit_cast(float, 0x3FB8AA3Bu);
  constexpr float kLn2Hi = __builtin_bit_cast(float, 0x3F317200u);
  constexpr float kLn2Lo = __builtin_bit_cast(float, 0x35BFBE8Eu);
  t = fminf(fmaxf(t, -120.f), 120.f);
  const float k = rintf(t * kInvLn2);
  const float r = (t - k * kLn2Hi) - k * kLn2Lo;
  float p = __builtin_bit_cast(float, 0x39500D01u);                  // 1/7!
  p = p * r + __builtin_bit_cast(float, 0x3AB60B61u);                // 1/6!
  p = p * r + __builtin_bit_cast(float, 0x3C088889u);                // 1/5!
  p = p * r + __builtin_bit_cast(float, 0x3D2AAAABu);                // 1/4!
  p = p * r + __builtin_bit_cast(float, 0x3E2AAAABu);                // 1/3!
  p = p * r + 0.5f;
  p = p * r + 1.f;
  p = p * r + 1.f;
  return ldexpf(p, (int)k);
}

// bf16 bits of bf16(silu(g)) * u (float32 product, nearest-even), with
// silu(g) = g / (1 + e^-g) (the producer of the down projection's input)
__device__ inline uint32_t swiglu1(uint32_t g, uint32_t u) {
#pragma clang fp contract(off)
  const float gf = bf16f(g);
  const float s = gf != gf ? __builtin_nanf("") : gf / (1.f + exp32(-gf));
  return to_bf16(bf16f(to_bf16(s)) * bf16f(u));
}

// silu(g) by the hardware exponential and reciprocal, for |g| <= 80: at most
// kSiluUlp float32 units from swiglu1's (over every bf16 gate).  g * kC is
// exact (8 + 16 significant bits); the rest of log2(e) enters as the factor
// 2^(-g c) = 1 - g c ln 2.
constexpr int kSiluUlp = 3;
__device__ inline float silu_fast(float g) {
  constexpr float kC = 47274.f / 32768.f;              // log2(e) to 16 bits
  constexpr float kR = -4.8885e-6f;                    // -(log2(e) - kC) ln 2
  float e = __builtin_amdgcn_exp2f(g * -kC);
  e = fmaf(e, g * kR, e);
  return g * __builtin_amdgcn_rcpf(1.f + e);
}

// Eight elements of swiglu1.  Its float32 silu is rounded to bf16, so the
// fast silu gives the same bits unless a rounding boundary lies within its
// error: vectors with such an element, or with a gate beyond the fast range
// (NaN and infinities among them), are evaluated as defined (about 5 % of the
// waves take that branch for one or more lanes).
__device__ inline u4 swiglu8(u4 g, u4 u) {
  float s[8];
  u4 o;
  uint32_t gm = 0, near = 0xFFFFu;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    s[2 * j] = silu_fast(__uint_as_float(g[j] << 16));
    s[2 * j + 1] = silu_fast(__uint_as_float(g[j] & 0xFFFF0000u));
    gm = max(gm, max((g[j] << 16) & 0x7FFF0000u, g[j] & 0x7FFF0000u));
#pragma unroll
    for (int k = 0; k < 2; ++k)
      near = min(near, (__float_as_uint(s[2 * j + k]) - (0x8000u - kSiluUlp)) & 0xFFFFu);
  }
  if (gm > 0x42A00000u || near <= 2 * kSiluUlp) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      o[j] = swiglu1(g[j] & 0xFFFFu, u[j] & 0xFFFFu) | (swiglu1(g[j] >> 16, u[j] >> 16) << 16);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float a = bf16f(to_bf16(s[2 * j])) * __uint_as_float(u[j] << 16);
      const float b = bf16f(to_bf16(s[2 * j + 1])) * __uint_as_float(u[j] & 0xFFFF0000u);
      o[j] = to_bf16(a) | (to_bf16(b) << 16);
    }
  }
  return o;
}

// RMS normalisation of the R staged rows, in place (the fused producer of
// the quantizer; Appendix A.2 keeps normalisation in 16-bit floating
// point): per row, ms = sum of x^2 / K in float64 (each 32-element block
// in order, then the blocks in order), r = float32(1 / sqrt(ms + eps)),
// then y = bf16(g * bf16(x * r)) with float32 products.
__device__ void rms_normalise(const QuantArgs &q, uint8_t *smem, int R, int rowB, int t,
                              int nthr, int64_t r0) {
  const int K = (int)q.K, nbk = K / kBlock;
  double *part = (double *)(smem + R * rowB);
  // (an odd count of sums per row, and lanes over rows first: a wave's reads of
  // the rows, and the rows' serial sums below, then lie in distinct banks: 2048 x
  // 4096 15.3 -> 14.7 us)
  const int pst = nbk | 1;
  float *rr = (float *)(part + R * pst);
  for (int it = t; it < R * nbk; it += nthr) {
    const int lr = it & (R - 1), b = it >> q.lg_rows;
    const u4 *xr = (const u4 *)(smem + lr * rowB + 64 * b);
    double sum = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const u4 d = xr[u];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double lo = (double)bf16f(d[j] & 0xFFFFu), hi = (double)bf16f(d[j] >> 16);
        sum += lo * lo;
        sum += hi * hi;
      }
    }
    part[lr * pst + b] = sum;
  }
  __syncthreads();
  if (t < R) {
    // the block sums in order; loaded sixteen at a time so that only the
    // additions form the dependent chain
    const double *pp = part + t * pst;
    double acc = 0.0;
    int b = 0;
    for (; b + 16 <= nbk; b += 16) {
      double v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = pp[b + u];
#pragma unroll
      for (int u = 0; u < 16; ++u) acc += v[u];
    }
    for (; b < nbk; ++b) acc += pp[b];
    // the zero rows past the input (operand-image padding) stay zero, also
    // with eps = 0
    rr[t] = r0 + t < q.src_rows ? (float)(1.0 / sqrt(acc / (double)K + (double)q.eps)) : 0.f;
  }
  __syncthreads();
  const int cpr = K / 8;                                 // 8-element chunks per row
  for (int c = t; c < R * cpr; c += nthr) {
    const int lr = c / cpr, k0 = (c - lr * cpr) * 8;
    u4 *xp = (u4 *)(smem + lr * rowB + 2 * k0);
    const u4 d = *xp;
    const u4 gv = *(const u4 *)(q.gain + k0);
    const float r = rr[lr];
    u4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t h0 = to_bf16(bf16f(d[j] & 0xFFFFu) * r), h1 = to_bf16(bf16f(d[j] >> 16) * r);
      const uint32_t y0 = to_bf16(bf16f(gv[j] & 0xFFFFu) * bf16f(h0));
      const uint32_t y1 = to_bf16(bf16f(gv[j] >> 16) * bf16f(h1));
      o[j] = y0 | (y1 << 16);
    }
    *xp = o;
  }
  __syncthreads();
}

// bf16(silu(g)) of every gate with 2^-14 <= |g| < 2^7 (21 binades of 128
// values, positive and negative in turn), as swiglu1 defines it: entry
// rotl16(g) - kSiluLo.
constexpr int kSiluLo = 2 * (113 << 7), kSiluN = 2 * (21 << 7);

__device__ inline uint32_t rotl16(uint32_t g) { return ((g << 1) | (g >> 15)) & 0xFFFFu; }

// Eight elements of swiglu1, the silu from the table in LDS.  A vector with a
// gate outside the table is evaluated as defined.
__device__ inline u4 swiglu8_table(const uint16_t *tab, u4 g, u4 u) {
  u4 o;
  bool in = true;
  uint32_t s[8];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const v2us x = __builtin_bit_cast(v2us, (uint32_t)g[j]);
    const v2us i = (v2us)((x << 1) | (x >> 15)) - (unsigned short)kSiluLo;
    in = in && i.x < kSiluN && i.y < kSiluN;
    s[2 * j] = tab[min((int)i.x, kSiluN - 1)];
    s[2 * j + 1] = tab[min((int)i.y, kSiluN - 1)];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j)
    o[j] = to_bf16(bf16f(s[2 * j]) * __uint_as_float(u[j] << 16)) |
           (to_bf16(bf16f(s[2 * j + 1]) * __uint_as_float(u[j] & 0xFFFF0000u)) << 16);
  if (!in) o = swiglu8(g, u);
  return o;
}

template <bool RNA, int MODE, int PROD>
__global__ __launch_bounds__(kMaxThreads) void quantize_act_kernel(QuantArgs q) {
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int t = threadIdx.x;
  const int nthr = blockDim.x;
  const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), nwaves = nthr >> 6;
  const int K = (int)q.K;
  const int rowB = 2 * (K + kRowPad);                // staged row stride (bytes)
  const int lgR = q.lg_rows;
  const int R = 1 << lgR;
  // XCD-aware order: consecutive row groups (whole operand tiles) stay on one
  // XCD, so its L2 completes every line of the tile.
  const int64_t nwg = gridDim.x;
  int64_t w0 = blockIdx.x;
  if ((nwg & 7) == 0) w0 = (w0 & 7) * (nwg >> 3) + (w0 >> 3);

  const int rms = PROD == kProdRms ? R * (8 * (K / kBlock | 1) + 4) : 0;
  uint16_t *silu = nullptr;
  if (PROD == kProdSwiglu && q.silu_table) {
    silu = (uint16_t *)(smem + ((R * rowB + rms + 15) & ~15));
    for (int i = t; i < kSiluN; i += nthr) {
      const uint32_t e = (uint32_t)(i + kSiluLo);
      silu[i] = (uint16_t)swiglu1(((e >> 1) | (e << 15)) & 0xFFFFu, 0x3F80u);
    }
    __syncthreads();
  }
  for (int lr = t; lr < R; lr += nthr) *(u4 *)(smem + lr * rowB + 2 * K) = u4{0u, 0u, 0u, 0u};

  // With SiLU * up a workgroup takes every nwg-th row group, so that its table
  // serves them all; else one.  The groups that run at one time are adjacent:
  // with a contiguous range each, a line of a tile was written at different
  // times, in parts that left the L2 one by one (M = 4096, K = 14336: 92 -> 82 us;
  // M = 2048, K = 65536, all 8-bit 342 -> 218).
  const int64_t groups = PROD == kProdSwiglu ? (q.out_rows + R - 1) >> lgR : w0 + 1;
  for (int64_t grp = w0; grp < groups; grp += nwg) {
    const int64_t r0 = grp << lgR;
    // the geometry is formed per group (an opaque zero): held over the loop
    // its scalars would spill
    int z = 0;
    if (PROD == kProdSwiglu) asm volatile("" : "+s"(z));
    const LGeo lg(q.n3 + z, q.n4 + z, q.n6 + z, q.n8 + z);
    const Chunks ch(lg, lgR);
    // Stage the rows.  Each thread issues a batch of loads before it stores
    // any of them, so the batch costs one memory latency instead of one per
    // load.
    constexpr int kBatch = 8;
    if (PROD != kProdSwiglu && q.vec16 && K % 512 == 0 && R * q.ld * 2 <= 0x7fffffff) {
      // Rows of whole 1 KB pieces go straight into LDS (direct-to-LDS loads,
      // one piece per wave instruction), all in flight until the wait before the
      // barrier below.  Rows past the source's end read zeros: the buffer
      // resource ends at its last row.
      const int64_t live = q.src_rows > r0 ? q.src_rows - r0 : 0;
      const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
          (void *)(q.src + r0 * q.ld), 0, (int)min(live * q.ld * 2, (int64_t)0x7fffffff),
          0x00020000);
      const int per_row = K / 512;
      int lr = wave / per_row, j = wave - lr * per_row;
      const int dl = nwaves / per_row, dj = nwaves - dl * per_row;
      while (lr < R) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void *)(smem + lr * rowB + j * 1024),
                                                 16, lane * 16, (int)(lr * q.ld * 2) + j * 1024, 0,
                                                 0);
        lr += dl;
        j += dj;
        if (j >= per_row) {
          j -= per_row;
          ++lr;
        }
      }
    } else if (PROD == kProdSwiglu && q.vec16) {
      // gate and up vectors: a batch of both in flight, then their products
      constexpr int kPairs = 4;
      const int vpr = K / 8, nv = R * vpr;
      const int dq = nthr / vpr, dr = nthr - dq * vpr;
      int lr = t / vpr, c = t - lr * vpr;
      for (int v0 = t; v0 < nv; v0 += nthr * kPairs) {
        u4 g[kPairs], u[kPairs];
        int off[kPairs];
#pragma unroll
        for (int k = 0; k < kPairs; ++k) {
          off[k] = lr * rowB + 16 * c;
          g[k] = u[k] = u4{0u, 0u, 0u, 0u};
          if (v0 + k * nthr < nv && r0 + lr < q.src_rows) {
            const int64_t src = (r0 + lr) * q.ld + 8 * c;
            g[k] = *(const u4 *)(q.src + src);
            u[k] = *(const u4 *)(q.src2 + src);
          }
          c += dr;
          lr += dq;
          if (c >= vpr) {
            c -= vpr;
            ++lr;
          }
        }
#pragma unroll
        for (int k = 0; k < kPairs; ++k)
          if (v0 + k * nthr < nv)
            *(u4 *)(smem + off[k]) = silu ? swiglu8_table(silu, g[k], u[k]) : swiglu8(g[k], u[k]);
      }
    } else if (q.vec16) {
      // vector v = lr * vpr + c, advanced by nthr without dividing per load
      const int vpr = K / 8, nv = R * vpr;
      const int dq = nthr / vpr, dr = nthr - dq * vpr;
      int lr0 = t / vpr, c0 = t - lr0 * vpr;
      for (int v0 = t; v0 < nv; v0 += nthr * kBatch) {
        u4 d[kBatch];
        int lrk[kBatch], ck[kBatch];
        int lr = lr0, c = c0;
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
          lrk[k] = lr;
          ck[k] = c;
          if (v0 + k * nthr < nv) {
            if (r0 + lr < q.src_rows)
              d[k] = *(const u4 *)(q.src + (r0 + lr) * q.ld + 8 * c);
            else
              d[k] = u4{0u, 0u, 0u, 0u};
          }
          c += dr;
          lr += dq;
          if (c >= vpr) {
            c -= vpr;
            ++lr;
          }
        }
        lr0 = lr;
        c0 = c;
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
          if (v0 + k * nthr < nv) *(u4 *)(smem + lrk[k] * rowB + 16 * ck[k]) = d[k];
      }
    } else {
      for (int lr = 0; lr < R; ++lr) {
        const bool live = r0 + lr < q.src_rows;
        const uint16_t *src = q.src + (r0 + lr) * q.ld;
        for (int c = t; c < K; c += nthr) {
          uint32_t v = live ? src[c] : 0u;
          if (PROD == kProdSwiglu && live) v = swiglu1(v, q.src2[(r0 + lr) * q.ld + c]);
          *(uint16_t *)(smem + lr * rowB + 2 * c) = (uint16_t)v;
        }
      }
    }
    // the direct-to-LDS loads are complete before the workgroup meets
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (PROD == kProdRms) rms_normalise(q, smem, R, rowB, t, nthr, r0);

    // the widest segments first: their items take longest
    for (int wc = wave; wc < ch.total; wc += nwaves) {
      int x = wc;
      if (x < ch.W[3])
        quantize_chunk<RNA, MODE, 3>(q, lg, 64 * x + lane, r0, smem, rowB);
      else if ((x -= ch.W[3]) < ch.W[2])
        quantize_chunk<RNA, MODE, 2>(q, lg, 64 * x + lane, r0, smem, rowB);
      else if ((x -= ch.W[2]) < ch.W[1])
        quantize_chunk<RNA, MODE, 1>(q, lg, 64 * x + lane, r0, smem, rowB);
      else
        quantize_chunk<RNA, MODE, 0>(q, lg, 64 * (x - ch.W[1]) + lane, r0, smem, rowB);
    }
    // zero the padding of the packed and exponent rows
    if (MODE == kModeRows)
      for (int lr = t; lr < R; lr += nthr) {
        const int64_t row = r0 + lr;
        if (row < q.src_rows) {
          for (int64_t z = q.row_used; z < q.canon_rb; ++z) q.mant[row * q.out_rb + z] = 0;
          for (int64_t z = q.n4 + q.n6 + q.n8; z < q.canon_erb; ++z)
            q.exp[row * q.out_erb + z] = 0;
        }
      }
    if (PROD != kProdSwiglu) break;
    if (grp + nwg < groups) __syncthreads();               // the rows are consumed
  }
}

// Packed rows of the identity permutation (the KV cache): a block's 64 bytes
// are contiguous, so a lane reads its block itself and nothing is staged.
// Lanes run over the blocks of a row, then over rows: the reads and the packed
// rows are contiguous over a wave.
constexpr int kRowsThreads = 256;

template <bool RNA>
__global__ __launch_bounds__(kRowsThreads) void quantize_rows_kernel(QuantArgs q) {
  const LGeo lg(q.n3, q.n4, q.n6, q.n8);
  const int nb = (int)(q.K / kBlock);
  const int64_t it = (int64_t)blockIdx.x * kRowsThreads + threadIdx.x;
  const int64_t row = it / nb;
  const int b = (int)(it - row * nb);
  if (row >= q.src_rows) return;
  const uint8_t *sr = (const uint8_t *)(q.src + row * q.ld);
  if (b < lg.b0[1])
    quantize_item<RNA, kModeRows, 0>(q, lg, item_geo_seg<0>(lg, b), row, sr);
  else if (b < lg.b0[2])
    quantize_item<RNA, kModeRows, 1>(q, lg, item_geo_seg<1>(lg, b - lg.b0[1]), row, sr);
  else if (b < lg.b0[3])
    quantize_item<RNA, kModeRows, 2>(q, lg, item_geo_seg<2>(lg, b - lg.b0[2]), row, sr);
  else
    quantize_item<RNA, kModeRows, 3>(q, lg, item_geo_seg<3>(lg, b - lg.b0[3]), row, sr);
  if (b == 0) {
    for (int64_t z = q.row_used; z < q.canon_rb; z += 4)
      *(uint32_t *)(q.mant + row * q.out_rb + z) = 0;
    int64_t z = nb;
    for (; z & 3; ++z) q.exp[row * q.out_erb + z] = 0;
    for (; z < q.canon_erb; z += 4) *(uint32_t *)(q.exp + row * q.out_erb + z) = 0;
  }
}

}  // namespace

// Bytes per staged row: the row and its zero padding, plus with RMS
// normalisation its block sums and its 1/rms.
static int64_t row_lds(int64_t K, bool rmsnorm) {
  return 2 * (K + kRowPad) + (rmsnorm ? 8 * (K / kBlock | 1) + 4 : 0);
}

// Row groups: R rows (a power of two) and T threads per workgroup.  While one
// workgroup per CU covers the rows, R is the least that does (more workgroups
// of fewer rows leave each a shorter chain) and a wave takes one chunk; beyond
// that two workgroups share a CU, so that one stages rows while the other
// computes.  Measured, us: M = 1, K = 4096: R = 1 4.3, R = 8 6.5; M = 333: R =
// 1 / 2 / 4 / 8 5.2 / 4.8 / 5.6 / 6.8; M = 4096: 1024 threads and one
// workgroup per CU 17.6, two of 512 13.1.
struct RowGroups {
  int lg, threads, per_cu;
};
static RowGroups row_groups(const QuantArgs &a, int cus) {
  const int64_t row = row_lds(a.K, a.rmsnorm != 0), extra = a.swiglu ? 2 * kSiluN : 0;
  auto fits = [&](int lg, int n) { return n * ((row << lg) + 16 + extra) <= kMaxLds; };
  const LGeo g(a.n3, a.n4, a.n6, a.n8);
  auto waves = [&](int lg) {
    int w = 0;
    for (int s = 0; s < kSegs; ++s) w += (((g.S[s] * (s < 2 ? 4 : 2)) << lg) + 63) / 64;
    return w;
  };
  constexpr int kMaxWaves = kMaxThreads / 64;
  auto one = [&](int lg) { return RowGroups{lg, 64 * std::min(waves(lg), kMaxWaves), 1}; };
  for (int lg = 0; lg <= 6 && fits(lg, 1) && waves(lg) <= 2 * kMaxWaves; ++lg)
    if (((a.out_rows - 1) >> lg) + 1 <= cus) return one(lg);
  int lg = 0;
  while (lg < 6 && fits(lg + 1, 2) && waves(lg + 1) <= kMaxWaves + 2) ++lg;
  if (!fits(lg, 2)) return one(0);
  // SiLU * up of long rows: its tables and arithmetic outweigh the overlap
  // (K = 14336, M = 4096: 4 rows and 1024 threads, one per CU, 82 us, 2 rows
  // and 512 threads, two per CU, 86 us)
  if (a.swiglu && lg <= 1 && fits(lg + 1, 1)) return RowGroups{lg + 1, kMaxThreads, 1};
  // Permuted rows of which two workgroups of one fit a CU, but no two of two: the
  // gather outweighs the overlap, and two rows share its column numbers (M = 4096,
  // 4-6-8, K = 20480 96 -> 74 us, K = 28672 134 -> 105; the kernel with a table of
  // them 80 and 143).  Not with RMS normalisation (177, 189).  All 6-bit images
  // from the next length on (K = 14336 69 -> 62, table 65; 4-6-8 52.5, 54.5).
  if (a.perm && !a.rmsnorm && fits(lg + 1, 1) &&
      (lg == 0 || (lg == 1 && !a.weights && !a.write_rows && 2 * g.S[2] > g.nsteps)))
    return RowGroups{lg + 1, kMaxThreads, 1};
  return RowGroups{lg, 64 * std::min(waves(lg), kMaxWaves / 2), 2};
}

template <int MODE, int PROD>
static hipError_t go_quantize(const QuantArgs &a, int64_t grid, int threads, int64_t lds,
                              hipStream_t stream) {
  const auto fn = a.ties_away ? quantize_act_kernel<true, MODE, PROD>
                              : quantize_act_kernel<false, MODE, PROD>;
  // the LDS limit, once per kernel and device
  static std::atomic<uint64_t> raised[2] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = -1;
  std::atomic<uint64_t> &mask = raised[a.ties_away != 0];
  if (dev < 0 || dev > 63 || !(mask.load(std::memory_order_relaxed) >> dev & 1)) {
    if (hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)kMaxLds) == hipSuccess && dev >= 0 && dev <= 63)
      mask.fetch_or(uint64_t(1) << dev, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(threads), (size_t)lds, stream, a);
  return hipGetLastError();
}

int64_t quantize_act_lds(int64_t K, bool rmsnorm) { return row_lds(K, rmsnorm); }

hipError_t launch_quantize_act(const QuantArgs &args, hipStream_t stream) {
  QuantArgs a = args;
  if (a.out_rows <= 0) return hipSuccess;
  if (a.write_rows && !a.perm && a.vec16) {
    const int64_t wg = (a.src_rows * (a.K / kBlock) + kRowsThreads - 1) / kRowsThreads;
    hipLaunchKernelGGL(a.ties_away ? quantize_rows_kernel<true> : quantize_rows_kernel<false>,
                       dim3((unsigned)wg), dim3(kRowsThreads), 0, stream, a);
    return hipGetLastError();
  }
  const int cus = device_cu_count();
  const RowGroups rg = row_groups(a, cus);
  a.lg_rows = rg.lg;
  const int64_t groups = ((a.out_rows - 1) >> rg.lg) + 1;
  // the silu table pays from six times its own size in elements
  const int64_t grid = a.swiglu ? std::min<int64_t>(groups, (int64_t)rg.per_cu * cus) : groups;
  int64_t lds = ((row_lds(a.K, a.rmsnorm != 0) << rg.lg) + 15) & ~15;
  a.silu_table = a.swiglu && a.vec16 && ((groups / grid * a.K) << rg.lg) >= 6 * kSiluN &&
                 lds + 2 * kSiluN <= kMaxLds;
  if (a.silu_table) lds += 2 * kSiluN;
  if (lds > kMaxLds) return hipErrorInvalidValue;
  if (a.weights) return go_quantize<kModeWeights, kProdNone>(a, grid, rg.threads, lds, stream);
  if (a.write_rows) return go_quantize<kModeRows, kProdNone>(a, grid, rg.threads, lds, stream);
  if (a.rmsnorm) return go_quantize<kModeImage, kProdRms>(a, grid, rg.threads, lds, stream);
  if (a.swiglu) return go_quantize<kModeImage, kProdSwiglu>(a, grid, rg.threads, lds, stream);
  return go_quantize<kModeImage, kProdNone>(a, grid, rg.threads, lds, stream);
}

}  // namespace mxq
