// attn.hip -- decode attention over an MXINT KV cache.
//
// MXSens (arXiv 2607.17733), Appendix A.2: the KV cache is quantized to
// MXINT (32-element blocks along the head dimension, 4 to 8 bits each) and
// attention reads it.  One new token per sequence attends to the T cached
// tokens of its sequence: per query head h (KV head h / G, G = Hq / Hkv),
// s_t = (q_h . K_t) * scale, p = softmax(s), o_h = sum_t p_t V_t, with K_t
// and V_t dequantized block by block, value = q * 2^(E - 127 - (m - 2)).
//
// The caches are the activation quantizer's packed rows (row (b * T + t) *
// Hkv + h, D = 128 values in four blocks) and exponent rows.  The token range
// of a (sequence, KV head) is split over workgroups so that a small batch
// still fills the GPU; the four waves of a workgroup take chunks of 32 tokens
// in turn, the next chunk's rows in flight while the current one is computed.
//
// Both products run on the bf16 matrix cores (16x16x32, float32
// accumulation).  A dequantized value q * 2^k with |q| <= 128 is exact in
// bf16, and so is a bf16 query element, so every product is exact:
//   scores  S[token][head]: a lane dequantizes 8 elements of its token's row
//           per product; the order of the 128 elements over the products is
//           free, as the query operand takes the same;
//   values  O[head][d] += P . V, where the float32 probabilities are split
//           into three bf16 terms whose sum is the float32 value, so the
//           weights are those of a float32 softmax.
// What bounds the kernel is the vector work of the dequantization, so it is
// done once per element, row by row for K and for V alike: 4-bit mantissas
// become sign-magnitude bytes, eight at a time, whose FP8 (e4m3) value is
// linear (k 2^-9), and the scaled conversion writes two bf16 values per
// instruction, the block scale included: 13 instructions for 8 elements.  K
// goes straight to the product; V goes to LDS as bf16 rows and comes back
// through the transposing LDS read.
// A lane of the score product's output holds one head and four tokens of
// each 16-token half, and the same lane supplies that head's probabilities
// to the value product, its eight tokens being the product's reduction slots
// (the V operand takes its tokens in the same slots).  The softmax is online
// against a reference m per head that is raised (and the sums rescaled) only
// when a score passes it by more than kSlack: the probabilities are then up to
// e^kSlack instead of 1, which costs float32 no precision.  It would cost
// range: from the first block of E >= 224 on, a wave keeps m the largest score
// (below that, sums of 2^31 / e^kSlack such tokens stay finite).  Waves, then splits,
// are merged in a fixed order, so results do not depend on timing.  Each
// width mix of the four blocks is its own instance, so block offsets and
// widths are compile-time constants.
//
// 16 sequences, 8 KV heads, 4096 tokens, with the merge, over caches not yet
// read (with a per-element dequantization of V gathered byte by byte): widths
// 4/4/6/8 40.4 us (49.6), all 4-bit 32.7 (40.6), all 8-bit 44.1 (47.1), all
// 3-bit 32.6 (142).
#include <algorithm>
#include <mutex>

#include "mxq_internal.h"

namespace mxq {

// Per-split partial results of the allocation-free entry point: one array
// per GPU, resident until the process ends.  In host code `scratch` names a
// host-side stand-in, not device memory; its device address comes from
// hipGetSymbolAddress, once per device, with that device current.
static __device__ __align__(256) float scratch[kAttnStaticWorkBytes / sizeof(float)];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch_ptr[kMaxDevices] = {};

}  // namespace

hipError_t attn_static_scratch(float **ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = (float *)p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

namespace {

typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s4 lds_s4;

constexpr int kD = 128;
// Waves of a workgroup (two workgroups per CU).  Eight leave each so few
// chunks that starting and merging cost more than they hide: 16 x 4096 tokens
// all 4-bit 28.5 against 25.8 us.
constexpr int kWaves = 4;
constexpr int kMaxG = 16;
constexpr int kChunk = 32;         // tokens per wave step: the value product's reduction
constexpr float kSlack = 4.f;
// LDS row of a token's 128 bf16 values, padded by 8 banks: the rows of 8
// lanes' 16-byte writes, and of 8 quads' transposing reads, lie in distinct banks
constexpr int kVRow = 2 * kD + 32;

// The four blocks of a cache row (head dimension 128): N3 3-bit, N4 4-bit,
// N6 6-bit and N8 8-bit blocks, in that order.  Rows of one width are read a
// block per lane (lane group g: block g, product j: elements 8j ..), others
// eight elements of each block (product j: block j, lane group g: elements
// 8g ..), so that all lanes run one width's code.
template <int N3, int N4, int N6, int N8>
struct Geo {
  static constexpr bool kUniform = N3 == 4 || N4 == 4 || N6 == 4 || N8 == 4;
  static constexpr bool kBig = N3 < 4;       // blocks wider than 3 bits
  static constexpr int width(int b) {
    return b < N3 ? 3 : b < N3 + N4 ? 4 : b < N3 + N4 + N6 ? 6 : 8;
  }
  static constexpr int off(int b) { return b == 0 ? 0 : off(b - 1) + 4 * width(b - 1); }
  static constexpr int kRow = (off(4) + 15) / 16 * 16;
  // dwords a lane holds of product j's elements, and their start
  static constexpr int words(int j) {
    return kUniform ? (j == 0 ? width(0) : 0) : width(j) == 4 ? 1 : 2;
  }
  static constexpr int start(int j) { return j == 0 ? 0 : start(j - 1) + words(j - 1); }
  static constexpr int kWords = start(4);
  // mixed rows are staged in LDS, in 16-byte pieces; the row stride keeps 16
  // lanes' accesses in distinct banks
  static constexpr int kVec = kRow / 16;
  static constexpr int kLds = kUniform ? 0 : (kRow + 31) / 32 * 32 + 16;
  static constexpr int kPieces = kChunk * kVec;
  static constexpr int kPer = (kPieces + 63) / 64;
};

// A lane's share of one token's row: its packed words and the row's four
// block exponents.
template <class Gm>
struct Raw {
  uint32_t w[Gm::kWords];
  uint32_t ex;
};

template <class Gm, int J>
__device__ inline void load_block(const uint8_t *row, int g, Raw<Gm> &r) {
  constexpr int M = Gm::width(J), S = Gm::start(J);
  const uint8_t *p = row + Gm::off(J);
  if constexpr (M == 4) {
    r.w[S] = *(const uint32_t *)(p + 4 * g);
  } else if constexpr (M == 6) {
    r.w[S] = *(const uint32_t *)(p + 4 * g);
    r.w[S + 1] = *(const uint32_t *)(p + 16 + 4 * (g >> 1));
  } else if constexpr (M == 8) {
    r.w[S] = *(const uint32_t *)(p + 8 * g);
    r.w[S + 1] = *(const uint32_t *)(p + 8 * g + 4);
  } else {
    // bytes 3g .. 3g + 2 of the block's 12
    const int o = (3 * g) & ~3;
    r.w[S] = *(const uint32_t *)(p + o);
    r.w[S + 1] = *(const uint32_t *)(p + (o < 8 ? o + 4 : 8));
  }
}

template <class Gm>
__device__ inline void load_raw(const uint8_t *row, int g, Raw<Gm> &r) {
  if constexpr (Gm::kUniform) {
    constexpr int M = Gm::width(0);
    const uint8_t *p = row + 4 * M * g;
    if constexpr (M == 4 || M == 8) {
#pragma unroll
      for (int i = 0; i < M / 4; ++i) {
        const u4 d = *(const u4 *)(p + 16 * i);
#pragma unroll
        for (int k = 0; k < 4; ++k) r.w[4 * i + k] = d[k];
      }
    } else {
#pragma unroll
      for (int i = 0; i < M; ++i) r.w[i] = *(const uint32_t *)(p + 4 * i);
    }
  } else {
    load_block<Gm, 0>(row, g, r);
    load_block<Gm, 1>(row, g, r);
    load_block<Gm, 2>(row, g, r);
    load_block<Gm, 3>(row, g, r);
  }
}

// (a & m) | (b & ~m) for m = 0x0F0F0F0F; the mask is opaque to the compiler,
// which would split a constant one into two instructions.
__device__ inline uint32_t low_nibbles_else(uint32_t a, uint32_t b) {
  uint32_t m;
  asm("s_mov_b32 %0, 0x0f0f0f0f" : "=s"(m));
  return (a & m) | (b & ~m);
}

__device__ inline bf8 to_bf8(const float (&x)[8]) {
  bf8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r[j] = (__bf16)x[j];      // exact: at most 8 significant bits
  return r;
}

// The largest exponent whose scale keeps an M-bit block's dequantization inside
// the float range: the FP8 conversion of a 4-bit block takes 2^(E - 127 - 2 + 9),
// and the offset of 6- and 8-bit blocks is -2^(E - 127 + 1).  Beyond it the block
// is dequantized at this exponent and scaled again (big_blocks).
constexpr int max_exp(int m) { return m == 3 ? 255 : m == 4 ? 247 : 253; }

// Element of slot i of a lane's eight: 4- and 6-bit blocks yield the even
// elements, then the odd ones.
__host__ __device__ constexpr int slot_elem(int m, int i) {
  return m != 4 && m != 6 ? i : i < 4 ? 2 * i : 2 * (i - 4) + 1;
}

// Product J's eight elements of a row, dequantized (in slot order).
template <class Gm, int J>
__device__ inline bf8 dequant(const Raw<Gm> &r, int g) {
  constexpr int M = Gm::width(J), S = Gm::start(J);
  const int E = (int)__builtin_amdgcn_ubfe(r.ex, Gm::kUniform ? 8 * g : 8 * J, 8);
  if constexpr (M == 4) {
    const uint32_t w = r.w[Gm::kUniform ? J : S];
    // two's complement nibbles -> sign bits and magnitudes 0..8
    const uint32_t sg = w & 0x88888888u, one = sg >> 3;
    const uint32_t mag = (w ^ ((one << 4) - one)) + one;
    const uint32_t ev = low_nibbles_else(mag, sg << 4), od = low_nibbles_else(mag >> 4, sg);
    const float sc = __uint_as_float((uint32_t)(min(E, max_exp(4)) + 7) << 23);
    bf2 v[4];
    v[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(ev, sc, false);
    v[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(ev, sc, true);
    v[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(od, sc, false);
    v[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(od, sc, true);
    return bf8{v[0][0], v[0][1], v[1][0], v[1][1], v[2][0], v[2][1], v[3][0], v[3][1]};
  } else {
    const float sc = __builtin_amdgcn_ldexpf(1.f, (M == 3 ? E : min(E, max_exp(M))) - 127 - (M - 2));
    float x[8];
    if constexpr (M == 3) {
      uint32_t w;
      if constexpr (Gm::kUniform) {
        constexpr int b = 24 * J, lo = b >> 5, sh = b & 31;
        w = r.w[lo] >> sh;
        if constexpr (sh > 8) w |= r.w[lo + 1] << (32 - sh);
      } else {
        w = __builtin_amdgcn_alignbit(r.w[S + 1], r.w[S], 8 * ((3 * g) & 3));
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = (float)(int)__builtin_amdgcn_sbfe((int)w, 3 * j, 3) * sc;
    } else {
      // bytes of q + 2^(M - 1); u sc - 2^(M - 1) sc is exact, in one rounding
      // (both terms are finite up to max_exp)
      uint32_t b0, b1;
      if constexpr (M == 8) {
        b0 = r.w[Gm::kUniform ? 2 * J : S] ^ 0x80808080u;
        b1 = r.w[Gm::kUniform ? 2 * J + 1 : S + 1] ^ 0x80808080u;
      } else {
        // byte j of the top word: bits 7:6 and 5:4 (3:2 and 1:0 in the odd
        // halves) are the top bits of elements 2j and 2j + 1
        const uint32_t w = r.w[Gm::kUniform ? J : S];
        const uint32_t tw = r.w[Gm::kUniform ? 4 + (J >> 1) : S + 1]
                            << (Gm::kUniform ? 4 * (J & 1) : 4 * (g & 1));
        b0 = low_nibbles_else(w, (tw >> 2) & 0x30303030u) ^ 0x20202020u;
        b1 = low_nibbles_else(w >> 4, tw & 0x30303030u) ^ 0x20202020u;
      }
      const float off = sc * -(float)(1 << (M - 1));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        x[j] = fmaf((float)((b0 >> (8 * j)) & 255u), sc, off);
        x[4 + j] = fmaf((float)((b1 >> (8 * j)) & 255u), sc, off);
      }
    }
    return to_bf8(x);
  }
}

// Whether a block of a row has its top three exponent bits set (E >= 224): it
// may pass max_exp, or, as V, leave the sums no room for kSlack.
__device__ inline bool has_big(uint32_t ex) {
  return (ex & (ex << 1) & (ex << 2) & 0x80808080u) != 0;
}

// The rest of such blocks' scales.  E = 255 is no exception: the quantizer
// writes zero mantissas with it, which stay zeros.
template <class Gm>
__device__ inline void big_blocks(const Raw<Gm> &r, int g, bf8 (&v)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int m = Gm::width(j);
    if (m == 3) continue;
    const int E = (int)((r.ex >> (8 * (Gm::kUniform ? g : j))) & 255u);
    const float f = __builtin_amdgcn_ldexpf(1.f, max(E - max_exp(m), 0));
#pragma unroll
    for (int i = 0; i < 8; ++i) v[j][i] = (__bf16)((float)v[j][i] * f);
  }
}

template <class Gm>
__device__ inline void dequant_row(const Raw<Gm> &r, int g, bool big, bf8 (&v)[4]) {
  v[0] = dequant<Gm, 0>(r, g);
  v[1] = dequant<Gm, 1>(r, g);
  v[2] = dequant<Gm, 2>(r, g);
  v[3] = dequant<Gm, 3>(r, g);
  if (Gm::kBig && big) big_blocks(r, g, v);
}

// e^d for d <= kSlack: 2^t with t = d log2 e, and what t lost in rounding (d -
// t ln 2, which the median keeps finite for d = -inf) as a first-order factor;
// a NaN stays.
__device__ inline float exp_f(float d) {
  const float t = d * 1.44269504f;
  const float e = __builtin_amdgcn_exp2f(t);
  return fmaf(e, __builtin_amdgcn_fmed3f(fmaf(t, -0.693147181f, d), -1.f, 1.f), e);
}

__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// DUP (at most 8 heads per KV head): the score product's columns 8..15 repeat
// the heads, and a column takes the 16 tokens of one half of the chunk only,
// so that every lane's softmax work counts; the two columns of a head are
// merged at the end like waves.
template <int N3, int N4, int N6, int N8, bool DUP>
__global__ __launch_bounds__(64 * kWaves, 2)
void attn_decode_kernel(AttnArgs a) {
  using Gm = Geo<N3, N4, N6, N8>;
  // A wave's LDS: the dequantized V rows.  Staged mixed rows lie in the same
  // place, K's at its start and V's at its end: K is consumed first, and the
  // first half of V's rows ends before the staged V rows begin.
  constexpr int kStage = kChunk * kVRow;
  static_assert(Gm::kLds <= kVRow / 2, "staged rows");
  constexpr int kMerge = kWaves * kMaxG * kD * 4;
  constexpr int kPool = kWaves * kStage > kMerge ? kWaves * kStage : kMerge;
  __shared__ __attribute__((aligned(16))) uint8_t pool[kPool];
  __shared__ uint32_t xs[kWaves][2][kChunk];               // exponent dwords of K, V rows
  __shared__ float mm[kWaves][kMaxG], ml[kWaves][kMaxG], mf[kWaves][kMaxG];
  const int t = threadIdx.x, lane = t & 63, g = lane >> 4, n = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int nw = blockDim.x >> 6;                          // at most kWaves
  const int G = a.G;
  constexpr int kVals = DUP ? 4 : 8;                       // probabilities per lane and chunk
  const int head = DUP ? n & 7 : n;                        // of lane column n
  const bool lower = !DUP || n < 8;
  const float ninf = -__builtin_inff();
  // The KV heads of a (sequence, split) share cache lines: they run on one XCD
  // (XCD x has the workgroups x, x + 8, ... of the dispatch, and takes a
  // contiguous range of the (sequence, split, head) list).
  const uint32_t Hkv = (uint32_t)a.Hkv, total = gridDim.x * gridDim.y;
  const uint32_t id = blockIdx.y * gridDim.x + blockIdx.x;
  const uint32_t x = id & 7, per = total >> 3, extra = total & 7;
  const uint32_t pos = x * per + min(x, extra) + (id >> 3);
  const int unit = (int)(pos / Hkv), kvh = (int)(pos - (uint32_t)unit * Hkv);
  const int b = unit / a.splits, split = unit - b * a.splits;
  uint8_t *vs = pool + wave * kStage;

  // the score product's Q operand: head n of the group (columns past the last
  // head repeat it), the elements of product j in slot order.  No branch, so
  // that the first rows are loaded before Q arrives: 1 x 4096 tokens, 64 heads
  // 11.15 -> 10.8 us.
  const uint32_t sign = a.scale < 0.f ? 0x80008000u : 0u;
  bf8 qop[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e0 = Gm::kUniform ? 32 * g + 8 * j : 32 * j + 8 * g;
    u4 x = *(const u4 *)(a.q + ((int64_t)b * a.Hq + (int64_t)kvh * G + min(head, G - 1)) * kD + e0);
    x ^= u4{sign, sign, sign, sign};
    const bf8 y = __builtin_bit_cast(bf8, x);
#pragma unroll
    for (int i = 0; i < 8; ++i) qop[j][i] = y[slot_elem(Gm::width(j), i)];
  }

  const int64_t t0 = (int64_t)split * a.tokens_per_split;
  const int64_t t1 = t0 + a.tokens_per_split < a.T ? t0 + a.tokens_per_split : a.T;
  const float scale = fabsf(a.scale);                      // its sign is in Q
  float run_m = ninf, run_l = 0.f;                         // column n; this lane's tokens
  float ref = 0.f;                                         // run_m, once finite
  float top = ninf, slack = kSlack;                        // the lane's largest score (unscaled)
  f4 o[8];                                                 // columns 4g + r, value 16 dt + n
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) o[dt] = (f4){0.f, 0.f, 0.f, 0.f};

  // Rows past the end are the chunk's last token (weight 0).
  Raw<Gm> rk[2], rv[2];                                    // (mixed rows: in LDS until used)
  u4 pk[Gm::kPer], pv[Gm::kPer];
  uint32_t px = 0;
  uint8_t *const ks = vs, *const ws = vs + kChunk * (kVRow - Gm::kLds);
  const int64_t step = a.Hkv * Gm::kRow, xstep = a.Hkv * a.exp_bytes;   // per token
  const int64_t first = (int64_t)b * a.T * a.Hkv + kvh;
  auto fetch = [&](int64_t c) __attribute__((always_inline)) {
    const int last = (int)(t1 - c < kChunk ? t1 - c : kChunk) - 1;
    const uint8_t *kc = a.k_mant + first * Gm::kRow + c * step;
    const uint8_t *vc = a.v_mant + first * Gm::kRow + c * step;
    if constexpr (Gm::kUniform) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const uint32_t off = (uint32_t)min(16 * mt + n, last) * (uint32_t)step;
        load_raw<Gm>(kc + off, g, rk[mt]);
        load_raw<Gm>(vc + off, g, rv[mt]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < Gm::kPer; ++i) {
        const int pc = min(i * 64 + lane, Gm::kPieces - 1);
        const int r = pc / Gm::kVec, cc = pc % Gm::kVec;
        const uint32_t off = (uint32_t)min(r, last) * (uint32_t)step + 16 * cc;
        pk[i] = *(const u4 *)(kc + off);
        pv[i] = *(const u4 *)(vc + off);
      }
    }
    px = *(const uint32_t *)((lane < 32 ? a.k_exp : a.v_exp) + first * a.exp_bytes + c * xstep +
                             (uint32_t)min(lane & 31, last) * (uint32_t)xstep);
  };
  if (t0 + kChunk * wave < t1) fetch(t0 + kChunk * wave);

  for (int64_t c0 = t0 + kChunk * wave; c0 < t1; c0 += kChunk * nw) {
    const int nt = (int)(t1 - c0 < kChunk ? t1 - c0 : kChunk);
    wave_sync();                                           // the previous chunk is consumed
    if constexpr (!Gm::kUniform) {
#pragma unroll
      for (int i = 0; i < Gm::kPer; ++i) {
        const int pc = i * 64 + lane;
        if (pc < Gm::kPieces) {
          const int r = pc / Gm::kVec, cc = pc % Gm::kVec;
          *(u4 *)(ks + r * Gm::kLds + 16 * cc) = pk[i];
          *(u4 *)(ws + r * Gm::kLds + 16 * cc) = pv[i];
        }
      }
    }
    xs[wave][lane >> 5][lane & 31] = px;
    const bool big = __any(has_big(px));
    if (big) slack = 0.f;                                  // for the rest of the wave's tokens
    wave_sync();
    if constexpr (!Gm::kUniform) {
      if (c0 + kChunk * nw < t1) fetch(c0 + kChunk * nw);
    }
    // scores: tokens 16 mt + 4 g + r of head n
    f4 sacc[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      bf8 v[4];
      if constexpr (!Gm::kUniform) load_raw<Gm>(ks + (16 * mt + n) * Gm::kLds, g, rk[mt]);
      rk[mt].ex = xs[wave][0][16 * mt + n];
      dequant_row(rk[mt], g, big, v);
      f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[j], qop[j], acc, 0, 0, 0);
      sacc[mt] = acc;
    }
    wave_sync();                                           // K's staged rows are consumed
    // V rows to LDS, in slot order
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      bf8 v[4];
      if constexpr (!Gm::kUniform) load_raw<Gm>(ws + (16 * mt + n) * Gm::kLds, g, rv[mt]);
      rv[mt].ex = xs[wave][1][16 * mt + n];
      dequant_row(rv[mt], g, big, v);
      uint8_t *vr = vs + (16 * mt + n) * kVRow;
      if (mt == 1) wave_sync();                            // V's staged rows are consumed
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *(bf8 *)(vr + 2 * (Gm::kUniform ? 32 * g + 8 * j : 32 * j + 8 * g)) = v[j];
    }
    if constexpr (Gm::kUniform) {
      if (c0 + kChunk * nw < t1) fetch(c0 + kChunk * nw);
    }
    wave_sync();

    // online softmax; value i of this lane is token tok(i) of the chunk
    auto tok = [&](int i) __attribute__((always_inline)) {
      return (DUP ? (lower ? 0 : 16) : 16 * (i >> 2)) + 4 * g + (i & 3);
    };
    float p[kVals];
#pragma unroll
    for (int i = 0; i < kVals; ++i)
      p[i] = !DUP ? sacc[i >> 2][i & 3] : lower ? sacc[0][i] : sacc[1][i];
    if (nt < kChunk) {
#pragma unroll
      for (int i = 0; i < kVals; ++i)
        if (tok(i) >= nt) p[i] = ninf;
    }
#pragma unroll
    for (int i = 0; i < kVals; ++i) top = fmaxf(top, p[i]);
    float cm = top == ninf ? ninf : top * scale;
    if (__any(cm > run_m + slack || run_m == ninf)) {
      cm = fmaxf(cm, __shfl_xor(cm, 16));
      cm = fmaxf(cm, __shfl_xor(cm, 32));
      const float nm = fmaxf(run_m, cm);
      const float alpha = run_m == ninf ? 0.f : exp_f(run_m - nm);
      run_l *= alpha;
      run_m = nm;
      ref = nm == ninf ? 0.f : nm;                         // scores of -inf weigh 0
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float ah = __shfl(alpha, 4 * g + r);         // column 4g + r lives in lane 4g + r
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) o[dt][r] *= ah;
      }
    }
    // the probabilities, as three bf16 terms summing to the float32 value
    float e[kVals];
#pragma unroll
    for (int i = 0; i < kVals; ++i) e[i] = exp_f(fmaf(p[i], scale, -ref));
    if (nt < kChunk) {
#pragma unroll
      for (int i = 0; i < kVals; ++i)
        if (tok(i) >= nt) e[i] = 0.f;
    }
    uint32_t pw[3][4];
#pragma unroll
    for (int i = 0; i < kVals / 2; ++i) {
      float x0 = e[2 * i], x1 = e[2 * i + 1];
      run_l += x0 + x1;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const bf2 h = {(__bf16)x0, (__bf16)x1};
        pw[k][i] = __builtin_bit_cast(uint32_t, h);
        x0 -= __uint_as_float(pw[k][i] << 16);
        x1 -= __uint_as_float(pw[k][i] & 0xFFFF0000u);
      }
    }
    bf8 pt[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      u4 x;
      if constexpr (DUP)                                   // the other half's slots weigh 0
        x = lower ? u4{pw[k][0], pw[k][1], 0u, 0u} : u4{0u, 0u, pw[k][0], pw[k][1]};
      else
        x = u4{pw[k][0], pw[k][1], pw[k][2], pw[k][3]};
      pt[k] = __builtin_bit_cast(bf8, x);
    }
    // values: the V operand takes the lane's tokens in the same slots
    const uint8_t *vp = vs + (4 * g + (n >> 2)) * kVRow + 8 * (n & 3);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(vp + 32 * dt));
      const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4 *)(vp + 32 * dt + 16 * kVRow));
      const bf8 v = __builtin_bit_cast(bf8, (s8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
      for (int k = 0; k < 3; ++k)
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pt[k], v, o[dt], 0, 0, 0);
    }
  }
  run_l += __shfl_xor(run_l, 16);
  run_l += __shfl_xor(run_l, 32);

  // Merge the waves (and a head's two columns) in order: every (wave, column)
  // gets its weight against the head's largest reference, each wave writes its
  // weighted outputs (over the V rows), and those are added up.
  constexpr int kCols = DUP ? 2 : 1, kStride = kMaxG / kCols;   // a head's columns, and their distance
  if (g == 0) {
    mm[wave][n] = run_m;
    ml[wave][n] = run_l;
  }
  __syncthreads();
  for (int i = t; i < kMaxG * nw; i += 64 * nw) {
    const int w = i / kMaxG, c = i % kMaxG;
    float M = ninf;
#pragma unroll
    for (int v = 0; v < kWaves; ++v)
      if (v < nw) M = fmaxf(M, fmaxf(mm[v][c], mm[v][c ^ (kMaxG - kStride)]));
    // without a score above -inf: nothing (or a NaN, which stays)
    mf[w][c] = mm[w][c] == ninf ? ml[w][c] : exp_f(mm[w][c] - M);
  }
  __syncthreads();
  float *mo = (float *)pool;                               // [kWaves][kMaxG][kD]
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = 4 * g + r;
    if (c % kStride < G) {
      const float f = mf[wave][c];
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) {
        const int d = 16 * dt + (n & 8) + slot_elem(Gm::width(dt >> 1), n & 7);
        mo[(wave * kMaxG + c) * kD + d] = f == 0.f ? 0.f : o[dt][r] * f;
      }
    }
  }
  __syncthreads();
  float *part = a.work + (((int64_t)b * a.Hkv + kvh) * a.splits + split) * G * (kD + 2);
  for (int i = t; i < G * kD / 4; i += 64 * nw) {
    const int h = i / (kD / 4), d = 4 * (i % (kD / 4));
    f4 O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
#pragma unroll
      for (int c = 0; c < kCols; ++c)
        if (w < nw) O += *(const f4 *)(mo + (w * kMaxG + h + c * kStride) * kD + d);
    float *po = part + h * (kD + 2) + 2 + d;
    *(f2 *)po = f2{O[0], O[1]};
    *(f2 *)(po + 2) = f2{O[2], O[3]};
  }
  if (t < G) {
    float M = ninf, L = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
#pragma unroll
      for (int c = 0; c < kCols; ++c)
        if (w < nw) {
          const int k = t + c * kStride;
          M = fmaxf(M, mm[w][k]);
          L += mf[w][k] == 0.f ? 0.f : ml[w][k] * mf[w][k];
        }
    // (finite: the merge of the splits takes differences)
    part[t * (kD + 2)] = fmaxf(M, -__FLT_MAX__);
    part[t * (kD + 2) + 1] = L;
  }
}

// o[b][h] = the splits' partials merged in a fixed order.  Groups of LPG lanes
// (four values each, from column 4 LPG blockIdx.z) take every kGroups-th split,
// BATCH splits' loads in flight together, so that kGroups * BATCH splits cost
// one memory latency; then the groups are merged pairwise (one after the other
// their rounding was the largest part of the result's: 1 x 1777 tokens 1.57e-7
// from 64 bits, pairwise 1.35e-7).
constexpr int kCombThreads = 256;

template <int LPG, int BATCH>
__global__ __launch_bounds__(kCombThreads) void attn_combine_kernel(AttnArgs a) {
  constexpr int kGroups = kCombThreads / LPG, kCols = 4 * LPG;
  __shared__ __attribute__((aligned(16))) float po[kGroups][kCols];
  __shared__ float pm[kGroups], pl[kGroups];
  const int t = threadIdx.x, d = 4 * (t % LPG), grp = t / LPG, h = blockIdx.x, b = blockIdx.y;
  const int c0 = kCols * blockIdx.z;
  const int G = a.G, kvh = h / G, g = h - kvh * G, S = a.splits;
  const float *base = a.work + (((int64_t)b * a.Hkv + kvh) * S * G + g) * (kD + 2);
  const int64_t stride = (int64_t)G * (kD + 2);
  const float ninf = -__builtin_inff();
  float M = ninf, L = 0.f;
  f4 O = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = grp; s0 < S; s0 += kGroups * BATCH) {
    f2 ml[BATCH], o0[BATCH], o1[BATCH];
    float nm = M;
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const float *p = base + min(s0 + kGroups * u, S - 1) * stride;
      ml[u] = *(const f2 *)p;
      o0[u] = *(const f2 *)(p + 2 + c0 + d);
      o1[u] = *(const f2 *)(p + 4 + c0 + d);
    }
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      if (s0 + kGroups * u < S) nm = fmaxf(nm, ml[u][0]);
    const float f0 = M == ninf ? 0.f : expf(M - nm);
    L *= f0;
    O *= f0;
    M = nm;
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      if (s0 + kGroups * u < S) {
        const float f = expf(ml[u][0] - nm);
        L += ml[u][1] * f;
        O += f4{o0[u][0], o0[u][1], o1[u][0], o1[u][1]} * f;
      }
  }
  *(f4 *)(po[grp] + d) = O;
  if (t % LPG == 0) {
    pm[grp] = M;
    pl[grp] = L;
  }
  __syncthreads();
  if (t >= kCols) return;
  // a lane per group: its weight (0 for a group that had no split)
  const int lane = t & 63;
  const float m = lane < kGroups ? pm[lane] : ninf;
  float Mx = m;
#pragma unroll
  for (int o = 1; o < kGroups; o *= 2) Mx = fmaxf(Mx, __shfl_xor(Mx, o));
  const float w = m == ninf ? 0.f : expf(m - Mx);
  float Ls[kGroups], Os[kGroups];
#pragma unroll
  for (int k = 0; k < kGroups; ++k) {
    const float f = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), k));
    Ls[k] = pl[k] * f;
    Os[k] = po[k][t] * f;
  }
#pragma unroll
  for (int n = kGroups / 2; n > 0; n /= 2)
#pragma unroll
    for (int k = 0; k < n; ++k) {
      Ls[k] += Ls[k + n];
      Os[k] += Os[k + n];
    }
  a.o[((int64_t)b * a.Hq + h) * kD + c0 + t] = Os[0] / Ls[0];
}

template <int N3, int N4, int N6, int N8>
void launch_t(const AttnArgs &a, hipStream_t s) {
  // one wave per 32 tokens of a split, at most kWaves
  const int64_t w = std::min<int64_t>((a.tokens_per_split + kChunk - 1) / kChunk, kWaves);
  const auto fn = a.G <= kMaxG / 2 ? attn_decode_kernel<N3, N4, N6, N8, true>
                                   : attn_decode_kernel<N3, N4, N6, N8, false>;
  // (a dispatch holds fewer than 2^32 threads per dimension)
  hipLaunchKernelGGL(fn, dim3((unsigned)(a.splits * a.Hkv), (unsigned)a.B),
                     dim3((unsigned)(64 * w)), 0, s, a);
}

// The kernel for a row's width mix, code = 125 n3 + 25 n4 + 5 n6 + n8 (the
// 35 mixes of four blocks).
template <int C>
bool dispatch(int code, const AttnArgs &a, hipStream_t s) {
  constexpr int n3 = C / 125, n4 = C / 25 % 5, n6 = C / 5 % 5, n8 = C % 5;
  if constexpr (n3 + n4 + n6 + n8 == 4) {
    if (code == C) {
      launch_t<n3, n4, n6, n8>(a, s);
      return true;
    }
  }
  if constexpr (C > 0) {
    return dispatch<C - 1>(code, a, s);
  } else {
    return false;
  }
}

}  // namespace

int64_t attn_tokens_per_split(int64_t B, int64_t Hkv, int64_t T) {
  // about 512 workgroups, whole multiples of 64 tokens
  const int64_t chunks = (T + 63) / 64;
  int64_t s = (512 + B * Hkv - 1) / (B * Hkv);
  if (s > chunks) s = chunks;
  if (s < 1) s = 1;
  return (chunks + s - 1) / s * 64;
}

hipError_t launch_attn_decode(const AttnArgs &a, hipStream_t s) {
  const int n3 = a.n3, n4 = a.n4 - a.n3;
  if (n3 < 0 || n4 < 0 || n3 + n4 + a.n6 + a.n8 != 4) return hipErrorInvalidValue;
  if (!dispatch<500>(125 * n3 + 25 * n4 + 5 * a.n6 + a.n8, a, s)) return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // The splits in one memory latency, with few loads per lane for few splits;
  // many splits come with few heads, whose columns go to several workgroups.
  // Main kernel and merge, us, over caches not yet read (<32, 8> alone served
  // all before): 16 x 4096 tokens, 64 heads (4 splits) <32, 2> 31.8, <16, 4>
  // 32.3, <32, 8> 32.6; 1 x 1777, 64 heads (28) 10.5, 9.9, 10.2; 1 x 4096, 64
  // heads (64) 13.3, 11.3, 11.5, <8, 8> 11.8; 2 x 9000, 5 heads (141) <16, 4>
  // 11.9, <8, 8> 11.1, <32, 8> 13.1; 1 x 32768, one head (512) 16.1, 12.3, 19.5.
  auto merge = [&](auto fn, int parts) {
    hipLaunchKernelGGL(fn, dim3((unsigned)a.Hq, (unsigned)a.B, (unsigned)parts),
                       dim3(kCombThreads), 0, s, a);
  };
  if (a.splits <= 16) merge(attn_combine_kernel<32, 2>, 1);
  else if (a.splits <= 64) merge(attn_combine_kernel<16, 4>, 2);
  else merge(attn_combine_kernel<8, 8>, 4);
  return hipGetLastError();
}

}  // namespace mxq
