// Prefill write of a layer's compressed cache (W1), the decode-time append of one
// token (W3: a bf16 tail write, or on the 32nd token the quantisation of the
// completed group with W1's block quantiser), and the test-only dequantiser.
//
// An anchor layer stores, per (sequence, KV head), its keys and values — after an
// optional eviction gather (KV-Kaizen §3, long context: the evictor runs on the
// same cache and the ratios multiply) — quantised by the table's scheme
// (App. C.3: grouped asymmetric KIVI32, or the paper's symmetric per-row SYMROW),
// or as bf16 at b = 16 (§2.2: a b = 16 GQA layer is the uncompressed cache).
// The layout written is the one documented in include/kvk.h.
//
// One wave writes the keys or the values of one 32-token block of one stream at d_h 128,
// of two at d_h 64 (half a wave each), without barriers.  Lane (q, tg) holds channels 8q .. 8q+7 of the eight
// tokens 16 (n/4) + 4 tg + n%4, n = 0..7: its loads are 16 bytes and a row's lanes
// read it whole, the 8 channels of a token are a chunk of the K layout and the 8
// tokens of a channel a chunk of the V layout, so every code word is formed in one
// lane's registers.  Group minima and maxima are in-lane trees finished by lane
// swaps.  The part is put together in the wave's LDS slot, in its output order, and
// leaves with 16-byte stores of contiguous kilobytes.  The kernel is specialised per
// head width, bit-width, scheme and input type.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "kvk_device.h"
#include "kvk_internal.h"

using namespace kvkd;

namespace {

// Sequences of a per-sequence batch one write launch serves (those whose plan gives
// the layer the same bit-width), and each one's region.
constexpr int kWriteSeqs = 64;

struct CompressArgs {
  const void* k;
  const void* v;
  const int32_t* keep;
  uint8_t* region;
  int64_t block_bytes;
  int64_t stream_bytes;
  int32_t in_f32;
  int32_t n_tokens;
  int32_t n_stored;
  int32_t nbf;      // full blocks written
  int32_t nb_cap;   // full-block capacity (tail block sits after it)
  int32_t D;
  int32_t bits;
  int32_t qs;       // kvk_qscheme
  // Per-sequence batches (n_seq > 0): the launch's streams are the Hkv streams of
  // sequences seq_of[0 .. n_seq), whose regions start seq_region[j] bytes after
  // `region`; the inputs stay indexed by the batch's sequence.  n_seq = 0: one table.
  int32_t n_seq, Hkv;
  int32_t n_streams;  // of the launch
  int32_t seq_of[kWriteSeqs];
  int64_t seq_region[kWriteSeqs];
};

#pragma clang fp contract(off)

// ---------------------------------------------------------------------------
// The lanes of a block and their rows
// ---------------------------------------------------------------------------

template <int D>
struct Lanes {
  static constexpr int kQ = D / 8;              // lanes of a row
  static constexpr int kPerBlock = 4 * kQ;      // lanes of a block: the wave, or half of it
  static constexpr int kBlocks = 64 / kPerBlock;  // blocks of a wave
};

// x, opaque to the compiler: what is derived from it is computed again rather than
// kept in registers from an earlier phase.
__device__ __forceinline__ int renewed(int x) {
  asm("" : "+v"(x));
  return x;
}

// Token of row n in the lanes of token set tg.
__device__ __forceinline__ int row_token(int n, int tg) { return 16 * (n >> 2) + 4 * tg + (n & 3); }

__device__ __forceinline__ u4v pack_bf16(f4 lo, f4 hi) {
  u4v r;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const float x0 = p < 2 ? lo[2 * p] : hi[2 * p - 4], x1 = p < 2 ? lo[2 * p + 1] : hi[2 * p - 3];
    r[p] = (uint32_t)f32_to_bf16_bits(x0) | ((uint32_t)f32_to_bf16_bits(x1) << 16);
  }
  return r;
}

// A lane's eight rows of eight channels, as loaded: bf16 packed, or fp32.  NT: loaded
// non-temporally.  Not fp32 rows: a row's lanes read it with two loads, each half of
// every line, and the second then misses (d_h 128, 4 x 8 KV heads x 8192 tokens, int8:
// 72 -> 55 us with plain loads, 76 -> 64 with inputs that rotate over 1 GiB; d_h 64, 39
// -> 30 and 43 -> 34).
template <bool F32>
struct Rows;
template <>
struct Rows<false> {
  u4v w[8];
  template <bool NT>
  __device__ __forceinline__ void load(const void* base, int64_t e, int n) {
    const u4v* p = reinterpret_cast<const u4v*>(static_cast<const uint16_t*>(base) + e);
    if constexpr (NT) w[n] = __builtin_nontemporal_load(p);
    else w[n] = *p;
  }
  __device__ __forceinline__ float get(int n, int c) const {
    const uint32_t x = w[n][c >> 1];
    return __uint_as_float(c & 1 ? x & 0xffff0000u : x << 16);
  }
  __device__ __forceinline__ u4v bf16(int n) const { return w[n]; }
  // Forget the conversions of an earlier pass over the rows (64 registers if kept), or
  // keep the common ones of two branches in each.
  __device__ __forceinline__ void renew() {
#pragma unroll
    for (int n = 0; n < 8; ++n)
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        uint32_t x = w[n][p];
        asm("" : "+v"(x));
        w[n][p] = x;
      }
  }
};
template <>
struct Rows<true> {
  f4 lo[8], hi[8];
  template <bool NT>
  __device__ __forceinline__ void load(const void* base, int64_t e, int n) {
    const f4* p = reinterpret_cast<const f4*>(static_cast<const float*>(base) + e);
    lo[n] = p[0];
    hi[n] = p[1];
  }
  __device__ __forceinline__ float get(int n, int c) const { return c < 4 ? lo[n][c] : hi[n][c - 4]; }
  __device__ __forceinline__ u4v bf16(int n) const { return pack_bf16(lo[n], hi[n]); }
  __device__ __forceinline__ void renew() {}
};

// Minima and maxima, which the compiler forms as v_min3 / v_max3 trees.  A quiet NaN
// operand is skipped (a signalling one, which no arithmetic gives, can hide the operands
// before it).  Written as fminf / fmaxf and not as the instructions in asm: the results
// meet lane swaps and DPP reads, which need two wait states after a vector write, and the
// compiler counts those only for instructions that it sees.
template <class F>
__device__ __forceinline__ float min8(F x) {
  return fminf(fminf(fminf(fminf(fminf(x(0), x(1)), x(2)), x(3)), x(4)), fminf(fminf(x(5), x(6)), x(7)));
}
template <class F>
__device__ __forceinline__ float max8v(F x) {
  return fmaxf(fmaxf(fmaxf(fmaxf(fmaxf(x(0), x(1)), x(2)), x(3)), x(4)), fmaxf(fmaxf(x(5), x(6)), x(7)));
}
// Largest |x| of eight values, 0 where all are NaN.
template <class F>
__device__ __forceinline__ float amax8(F x) {
  return fmaxf(max8v([&](int i) { return fabsf(x(i)); }), 0.0f);
}

// ---------------------------------------------------------------------------
// Quantisers
// ---------------------------------------------------------------------------

// Scale, reciprocal and zero of one grouped-asymmetric group: s, z the fp16 values
// (App. C.3) and y = 1/s to an ulp; s = y = 0 stands for the groups whose codes are 0
// whatever the value (s zero, or beyond fp16: infinite).  (mx - mn) / levels is
// rounded correctly by one residual step on the product with the constant's
// reciprocal: the residual is exact (levels has 8 bits), and the quotient's distance
// from a rounding boundary exceeds the step's error (as in Coder::quotient).
struct Group {
  float s, y, z;
  uint32_t sz;  // the stored pair: scale in the low half, zero in the high half
};
template <int BITS>
__device__ __forceinline__ Group make_group(float mn, float mx) {
  constexpr float levels = (float)((1 << BITS) - 1), inv = 1.0f / levels;
  const float d = mx - mn;
  const float q = fminf(d * inv, 3.402823466e38f);
  const float sc = __builtin_fmaf(__builtin_fmaf(-levels, q, d), inv, q);
  const _Float16 s16 = (_Float16)sc, z16 = (_Float16)mn;
  Group g;
  const float s = (float)s16;
  g.z = (float)z16;
  g.sz = (uint32_t)bitcast<uint16_t>(s16) | ((uint32_t)bitcast<uint16_t>(z16) << 16);
  const bool live = s > 0.0f && s < __builtin_huge_valf();
  g.s = live ? s : 0.0f;
  g.y = live ? __builtin_amdgcn_rcpf(s) : 0.0f;
  return g;
}

// 1.5 * 2^23: adding it rounds to the nearest integer (ties to even) into the low bits.
constexpr float kRound = 12582912.0f;

// The code of x in a grouped-asymmetric group, in the low bits of the result (the bits
// above hold kRound's).  fp32 (x - z) / s correctly rounded, then rounded to an
// integer and clamped.  The division: q = a y is within 2 ulp of a / s; r = a - s q is
// exact in one fma (s has 11 significant bits); q + r y differs from a / s by under
// 2^-44 relative before its rounding, and a / s lies no closer than 2^-36 to a
// rounding boundary (a - s m is a whole number of units of a 36-bit product), so the
// result is the correctly rounded quotient: 4 operations in place of the compiler's
// 11.  The bound at 512 only matters when a is infinite (z beyond fp16): it keeps the
// residual infinite instead of NaN.  A NaN (any NaN input) gives code 0.
template <int BITS>
__device__ __forceinline__ uint32_t group_code(float x, float s, float y, float z) {
  constexpr float levels = (float)((1 << BITS) - 1);
  const float a = x - z;
  const float q = fminf(a * y, 512.0f);
  const float t = __builtin_fmaf(__builtin_fmaf(-s, q, a), y, q);
  return __float_as_uint(__builtin_amdgcn_fmed3f(t, 0.0f, levels) + kRound);
}

// One symmetric row: the stored bf16 scale; s and y = 1/s of the row scaled by f, a
// power of two that keeps both away from the denormals; the clamp (0 where the scale
// is zero).  s = y = 0 for an infinite scale: finite values get code 0.
struct Row {
  float s, y, f, hi;
  uint16_t bits;
};
template <int BITS>
__device__ __forceinline__ Row make_row(float am) {
  constexpr float q = (float)((1 << (BITS - 1)) - 1);
  Row r;
  r.bits = f32_to_bf16_bits(am / q);
  const float s = bf16_to_f32(r.bits);
  r.f = s < 0x1p-60f ? 0x1p64f : (s > 0x1p60f ? 0x1p-64f : 1.0f);
  const bool live = s > 0.0f && s < __builtin_huge_valf();
  r.s = live ? s * r.f : 0.0f;
  r.y = live ? __builtin_amdgcn_rcpf(r.s) : 0.0f;
  r.hi = s != 0.0f ? q : 0.0f;
  return r;
}
// The stored code of x in a symmetric row (as group_code: s has 8 significant bits).
template <int BITS>
__device__ __forceinline__ uint32_t row_code(float x, const Row& r) {
  const float a = x * r.f;
  const float q = a * r.y;
  const float t = __builtin_fmaf(__builtin_fmaf(-r.s, q, a), r.y, q);
  return __float_as_uint(__builtin_amdgcn_fmed3f(t, -r.hi, r.hi) + (kRound + (float)(1 << (BITS - 1))));
}

// Eight codes (low bits of b) as a chunk, to the chunk's place at byte `at` of a part.
// b = 2: the chunk's two bytes sit in the word it shares with its neighbour.
template <int BITS>
__device__ __forceinline__ void store_chunk(uint8_t* part, int at, const uint32_t (&b)[8]) {
  if constexpr (BITS == 8) {
    u2v w;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t lo = __builtin_amdgcn_perm(b[4 * h + 1], b[4 * h], 0x0c0c0400u);
      const uint32_t hi = __builtin_amdgcn_perm(b[4 * h + 3], b[4 * h + 2], 0x04000c0cu);
      w[h] = lo | hi;
    }
    *reinterpret_cast<u2v*>(part + at) = w;
  } else {
    // slot s at bit 16 (s%2) + BITS (s/2): the high bits of the shifted terms fall
    // above bit 22 and are dropped with the upper halves
    uint32_t lo = b[0], hi = b[1];
#pragma unroll
    for (int p = 1; p < 4; ++p) {
      lo |= b[2 * p] << (BITS * p);
      hi |= b[2 * p + 1] << (BITS * p);
    }
    if constexpr (BITS == 4) {
      *reinterpret_cast<uint32_t*>(part + at) = __builtin_amdgcn_perm(hi, lo, 0x05040100u);
    } else {
      part[at] = (uint8_t)lo;
      part[at + 2] = (uint8_t)hi;
    }
  }
}

// Byte of the K chunk (token t, channels 8q..8q+7) in the K codes of a block and of the V
// chunk (channel c, token set tg) in its V codes, by the share layout of kvk.h.
template <int D, int BITS>
__device__ __forceinline__ int k_chunk_byte(int t, int q) {
  const int j = q >> 2, lam = 16 * (q & 3) + (t & 15), tile = 2 * D * BITS * (t >> 4);
  constexpr int P = D * BITS / 32;
  if constexpr (BITS == 2) return tile + share_byte(P, lam, 4 * (j >> 1)) + (j & 1);
  return tile + share_byte(P, lam, BITS * j);
}
template <int D, int BITS>
__device__ __forceinline__ int v_chunk_byte(int c, int tg) {
  const int m = c >> 4, lam = 16 * tg + (c & 15);
  constexpr int P = D * BITS / 16;
  if constexpr (BITS == 2) return share_byte(P, lam, 4 * (m >> 1)) + (m & 1);
  return share_byte(P, lam, BITS * m);
}

// Reduction over the token sets of one channel's minimum or maximum, all lanes ending
// with it (d_h 64: the sets are 8 and 16 lanes apart).
__device__ __forceinline__ float sets_min64(float x) {
  x = fminf(x, dpp<0x128>(x));  // row_ror:8
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fminf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float sets_max64(float x) {
  x = fmaxf(x, dpp<0x128>(x));
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}

struct Pair {
  float a, b;
};
__device__ __forceinline__ Pair swap16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ Pair swap32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
// x of the four 16-lane rows to every lane: row r's value in out[r].
__device__ __forceinline__ void gather_rows(float x, float (&out)[4]) {
  const Pair h = swap32(x, x);  // rows 0, 1 twice; rows 2, 3 twice
  const Pair l = swap16(h.a, h.a), u = swap16(h.b, h.b);
  out[0] = l.a;
  out[1] = l.b;
  out[2] = u.a;
  out[3] = u.b;
}

// KIVI32 key metadata: every lane's eight channel groups, and the stored pairs into
// kmeta (fp16 scale[D] then zero[D]).
template <int D, int BITS, class R>
__device__ __forceinline__ void kivi_key_groups(const R& rows, int q, int tg, uint16_t* kmeta, float (&s)[8],
                                                float (&y)[8], float (&z)[8]) {
  float mn[8], mx[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    mn[c] = min8([&](int n) { return rows.get(n, c); });
    mx[c] = max8v([&](int n) { return rows.get(n, c); });
  }
  if constexpr (D == 128) {
    // the token sets are the four 16-lane rows: each swap finishes half of two
    // channels' reductions, so that row tg ends with the channels
    // k + 2 (tg / 2) + 4 (tg % 2), k = 0, 1, forms their groups, and the rows share them
    float rn[4], rx[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const Pair a = swap16(mn[k], mn[k + 4]), b = swap16(mx[k], mx[k + 4]);
      rn[k] = fminf(a.a, a.b);
      rx[k] = fmaxf(b.a, b.b);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const Pair a = swap32(rn[k], rn[k + 2]), b = swap32(rx[k], rx[k + 2]);
      const Group g = make_group<BITS>(fminf(a.a, a.b), fmaxf(b.a, b.b));
      const int c = 8 * q + k + 2 * (tg >> 1) + 4 * (tg & 1);
      kmeta[c] = (uint16_t)g.sz;
      kmeta[D + c] = (uint16_t)(g.sz >> 16);
      float t[4];
      constexpr int kOf[4] = {0, 4, 2, 6};
      gather_rows(g.s, t);
#pragma unroll
      for (int r = 0; r < 4; ++r) s[k + kOf[r]] = t[r];
      gather_rows(g.y, t);
#pragma unroll
      for (int r = 0; r < 4; ++r) y[k + kOf[r]] = t[r];
      gather_rows(g.z, t);
#pragma unroll
      for (int r = 0; r < 4; ++r) z[k + kOf[r]] = t[r];
    }
  } else {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const Group g = make_group<BITS>(sets_min64(mn[c]), sets_max64(mx[c]));
      if (tg == 0) {
        kmeta[8 * q + c] = (uint16_t)g.sz;
        kmeta[D + 8 * q + c] = (uint16_t)(g.sz >> 16);
      }
      s[c] = g.s;
      y[c] = g.y;
      z[c] = g.z;
    }
  }
}

// Per-token groups of N lanes (32 channels: 4; 64: 8), every lane's eight tokens: the
// stored pairs in sz.
template <int BITS, int N, class R>
__device__ __forceinline__ void token_groups(const R& rows, int q, float (&s)[8], float (&y)[8], float (&z)[8],
                                             uint32_t (&sz)[8]) {
  float mn[8], mx[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    mn[n] = min8([&](int c) { return rows.get(n, c); });
    mx[n] = max8v([&](int c) { return rows.get(n, c); });
  }
  if constexpr (N == 4) {
    // a quad's lane finishes two of the eight tokens (2 k + q%2 + (q/2)%2 * 4) and the
    // others take the results from it
    const bool o1 = q & 1, o2 = q & 2;
    float an[4], ax[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      an[k] = fminf(o1 ? mn[2 * k + 1] : mn[2 * k], dpp<kQuadXor1>(o1 ? mn[2 * k] : mn[2 * k + 1]));
      ax[k] = fmaxf(o1 ? mx[2 * k + 1] : mx[2 * k], dpp<kQuadXor1>(o1 ? mx[2 * k] : mx[2 * k + 1]));
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const float bn = fminf(o2 ? an[k + 2] : an[k], dpp<kQuadXor2>(o2 ? an[k] : an[k + 2]));
      const float bx = fmaxf(o2 ? ax[k + 2] : ax[k], dpp<kQuadXor2>(o2 ? ax[k] : ax[k + 2]));
      const Group g = make_group<BITS>(bn, bx);
      const float szf = __uint_as_float(g.sz);
#define KVK_FROM_QUAD(E, CTRL) \
  { \
    constexpr int n = (E & 1) + 2 * (E >> 1) * 2; \
    s[2 * k + n] = dpp<CTRL>(g.s); \
    y[2 * k + n] = dpp<CTRL>(g.y); \
    z[2 * k + n] = dpp<CTRL>(g.z); \
    sz[2 * k + n] = __float_as_uint(dpp<CTRL>(szf)); \
  }
      KVK_FROM_QUAD(0, 0x00) KVK_FROM_QUAD(1, 0x55) KVK_FROM_QUAD(2, 0xAA) KVK_FROM_QUAD(3, 0xFF)
#undef KVK_FROM_QUAD
    }
  } else {
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      float a = mn[n], b = mx[n];
      a = fminf(a, dpp<kQuadXor1>(a));
      b = fmaxf(b, dpp<kQuadXor1>(b));
      a = fminf(a, dpp<kQuadXor2>(a));
      b = fmaxf(b, dpp<kQuadXor2>(b));
      a = fminf(a, dpp<kHalfRowMirror>(a));
      b = fmaxf(b, dpp<kHalfRowMirror>(b));
      const Group g = make_group<BITS>(a, b);
      s[n] = g.s;
      y[n] = g.y;
      z[n] = g.z;
      sz[n] = g.sz;
    }
  }
}

__device__ __forceinline__ u4v low_halves(const uint32_t (&x)[8]) {
  u4v r;
#pragma unroll
  for (int p = 0; p < 4; ++p) r[p] = __builtin_amdgcn_perm(x[2 * p + 1], x[2 * p], 0x05040100u);
  return r;
}
__device__ __forceinline__ u4v high_halves(const uint32_t (&x)[8]) {
  u4v r;
#pragma unroll
  for (int p = 0; p < 4; ++p) r[p] = __builtin_amdgcn_perm(x[2 * p + 1], x[2 * p], 0x07060302u);
  return r;
}

// Keys of a block into their LDS image: the codes, then the metadata.
template <int D, int BITS, int QS, class R>
__device__ __forceinline__ void quant_keys(R& rows, int q, int tg, uint8_t* img) {
  tg = renewed(tg);
  rows.renew();
  uint8_t* meta = img + 4 * D * BITS;
  float s[8], y[8], z[8];
  if constexpr (QS == kQsKivi) {
    kivi_key_groups<D, BITS>(rows, q, tg, reinterpret_cast<uint16_t*>(meta), s, y, z);
  } else if constexpr (QS == kQsG64) {
    uint32_t sz[8];
    token_groups<BITS, 8>(rows, q, s, y, z, sz);
    if (q % 8 == 0) {  // fp16 index ((tau*4 + kg)*NG*2 + g*2 + w)*4 + e
      const u4v sc = low_halves(sz), ze = high_halves(sz);
#pragma unroll
      for (int tau = 0; tau < 2; ++tau) {
        u4v* m4 = reinterpret_cast<u4v*>(meta + 16 * ((tau * 4 + tg) * (D / 64) + q / 8));
        *m4 = u4v{sc[2 * tau], sc[2 * tau + 1], ze[2 * tau], ze[2 * tau + 1]};
      }
    }
  }
  rows.renew();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    uint32_t b[8];
    const int t = row_token(n, tg);
    if constexpr (QS == kQsSym) {
      float am = amax8([&](int c) { return rows.get(n, c); });
      am = D == 128 ? max16(am) : max8(am);
      const Row r = make_row<BITS>(am);
      if (q == 0) reinterpret_cast<uint16_t*>(meta)[t] = r.bits;
#pragma unroll
      for (int c = 0; c < 8; ++c) b[c] = row_code<BITS>(rows.get(n, c), r);
    } else {
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int g = QS == kQsKivi ? c : n;
        b[c] = group_code<BITS>(rows.get(n, c), s[g], y[g], z[g]);
      }
    }
    store_chunk<BITS>(img, k_chunk_byte<D, BITS>(t, q), b);
    __builtin_amdgcn_sched_barrier(0);  // chunk after chunk: interleaved ones spill
  }
}

// Values of a block, likewise.
template <int D, int BITS, int QS, class R>
__device__ __forceinline__ void quant_values(R& rows, int q, int tg, uint8_t* img) {
  tg = renewed(tg);
  rows.renew();
  uint8_t* meta = img + 4 * D * BITS;
  if constexpr (QS == kQsSym) {
    Row r[8];
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      float am = amax8([&](int c) { return rows.get(n, c); });
      am = D == 128 ? max16(am) : max8(am);
      r[n] = make_row<BITS>(am);
      if (q == 0) reinterpret_cast<uint16_t*>(meta)[row_token(n, tg)] = r[n].bits;
    }
    rows.renew();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      uint32_t b[8];
#pragma unroll
      for (int n = 0; n < 8; ++n) b[n] = row_code<BITS>(rows.get(n, c), r[n]);
      store_chunk<BITS>(img, v_chunk_byte<D, BITS>(8 * q + c, tg), b);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    constexpr int GL = QS == kQsKivi ? 4 : 8;  // lanes of a group
    float s[8], y[8], z[8];
    uint32_t sz[8];
    token_groups<BITS, GL>(rows, q, s, y, z, sz);
    if (q % GL == 0) {  // fp16 index ((g*2 + w)*4 + kg)*8 + s
      u4v* m4 = reinterpret_cast<u4v*>(meta) + 8 * (q / GL) + tg;
      m4[0] = low_halves(sz);
      m4[4] = high_halves(sz);
    }
    rows.renew();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      uint32_t b[8];
#pragma unroll
      for (int n = 0; n < 8; ++n) b[n] = group_code<BITS>(rows.get(n, c), s[n], y[n], z[n]);
      store_chunk<BITS>(img, v_chunk_byte<D, BITS>(8 * q + c, tg), b);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// bf16 K part (64 D bytes) of a block into LDS: a lane's row is a 16-byte piece.
template <int D, class R>
__device__ __forceinline__ void bf16_keys(const R& rows, int q, int tg, uint8_t* img) {
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    const int t = row_token(n, tg);
    *reinterpret_cast<u4v*>(img + 32 * D * (t >> 4) + 1024 * (q >> 2) + 16 * (16 * (q & 3) + (t & 15))) = rows.bf16(n);
  }
}
// bf16 V part (64 D bytes): a channel's eight tokens are a 16-byte piece.
template <int D, class R>
__device__ __forceinline__ void bf16_values(const R& rows, int q, int tg, uint8_t* img) {
  u4v w[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) w[n] = rows.bf16(n);
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    u4v o;
#pragma unroll
    for (int p = 0; p < 4; ++p)
      o[p] = __builtin_amdgcn_perm(w[2 * p + 1][c >> 1], w[2 * p][c >> 1], c & 1 ? 0x07060302u : 0x05040100u);
    const int ch = 8 * q + c;
    *reinterpret_cast<u4v*>(img + 1024 * (ch >> 4) + 16 * (16 * tg + (ch & 15))) = o;
  }
}

// Order a wave's LDS accesses (one wave's run in order; this keeps the compiler's
// order and waits for the writes).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Bytes of the K (or V) codes and of the K (or V) metadata of a quantised block, which
// holds K codes, V codes, K metadata, V metadata; and of the LDS image of a part.
template <int D, int BITS>
constexpr int kCodeBytes = 4 * D * BITS;
template <int D, int QS>
constexpr int kMetaBytes = QS == kQsKivi ? 4 * D : (QS == kQsSym ? 64 : 2 * D);
template <int D, int BITS, int QS>
constexpr int kImageBytes =
    BITS == 16 || kCodeBytes<D, BITS> + kMetaBytes<D, QS> < 64 * D ? 64 * D : kCodeBytes<D, BITS> + kMetaBytes<D, QS>;

// The LDS image of part `part` (0 K, 1 V) to its places in the block at `out`, by the
// lanes of the block: a bf16 part, or codes and metadata.
template <int D>
__device__ __forceinline__ void copy_bf16_part(const uint8_t* img, uint8_t* out, int part, int l) {
  wave_lds_fence();
  for (int o = 16 * l; o < 64 * D; o += 16 * Lanes<D>::kPerBlock)
    __builtin_nontemporal_store(*reinterpret_cast<const u4v*>(img + o),
                                reinterpret_cast<u4v*>(out + 64 * D * part + o));
}
template <int D, int BITS, int QS>
__device__ __forceinline__ void copy_quant_part(const uint8_t* img, uint8_t* out, int part, int l) {
  constexpr int cb = kCodeBytes<D, BITS>, mb = kMetaBytes<D, QS>;
  wave_lds_fence();
  for (int o = 16 * l; o < cb + mb; o += 16 * Lanes<D>::kPerBlock) {
    const int to = o < cb ? cb * part + o : 2 * cb + mb * part + (o - cb);
    __builtin_nontemporal_store(*reinterpret_cast<const u4v*>(img + o), reinterpret_cast<u4v*>(out + to));
  }
}

// The input elements of a lane's rows: stored tokens tok0 .. (none past `last`), through
// the keep list under eviction.
template <int D>
__device__ __forceinline__ void row_elements(const CompressArgs& a, int in_stream, int tok0, int last, int q, int tg,
                                             int64_t (&e)[8]) {
  int pos[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    pos[n] = tok0 + row_token(n, tg);
    pos[n] = pos[n] < last ? pos[n] : last;
  }
  if (a.keep) {
    const int32_t* keep = a.keep + (int64_t)in_stream * a.n_stored;
#pragma unroll
    for (int n = 0; n < 8; ++n) pos[n] = keep[pos[n]];
#pragma unroll
    for (int n = 0; n < 8; ++n) pos[n] = pos[n] < 0 ? 0 : (pos[n] >= a.n_tokens ? a.n_tokens - 1 : pos[n]);
  }
#pragma unroll
  for (int n = 0; n < 8; ++n) e[n] = ((int64_t)in_stream * a.n_tokens + pos[n]) * D + 8 * q;
}

// Waves of a workgroup.  One: a launch of few blocks spreads over the CUs, and a short one
// lasts as long as its fullest CU (one token of 8 KV heads, d_h 128: 2.5 us; two waves
// 2.8, four 3.6; 4 x 4 KV heads x 2000 tokens of d_h 64, int8: 6.0, 7.4 and 8.5).  Two for
// bf16 rows at d_h 128: 4 x 8 KV heads x 8192 tokens, int8, 35.9 us, with one 37.0.
template <int D, bool F32>
constexpr int kWriteWaves = D == 128 && !F32 ? 2 : 1;

// One wave writes the keys or the values of one 32-token block of one stream (two at d_h
// 64), with BITS-bit codes (or bf16 at BITS = 16; a stream's tail block is always bf16).
// Not both in one wave: its chain of loads, codes and stores is what a small launch takes
// (8 KV heads x 256 tokens, d_h 128, int8: 6.1 -> 4.1 us; d_h 64 7.5 -> 5.5), and the
// registers of one part leave room for as many loads in flight on a full GPU (14B mixed
// stack, 32 anchors: 1150 -> 1121 us).
//
// Bound: HBM and the vector units about equally (d_h 128, KIVI32: about 14 vector
// operations per value; the input is read and the codes are written once).
//
// Loads are non-temporal where bf16 rows are quantised (14B mixed stack, 32 anchors: 1264
// -> 1170 us), not where they are copied: inputs still in the last-level cache take 41.5 us
// at d_h 128 (4 x 8 KV heads x 8192 tokens) against 45.7, others 49.3 against 47.7.
template <int D, int BITS, int QS, bool F32>
__global__ __launch_bounds__((64 * kWriteWaves<D, F32>), F32 ? 3 : 4) void compress_kernel(CompressArgs a) {
  using L = Lanes<D>;
  constexpr int kWaves = kWriteWaves<D, F32>;
  constexpr bool kNt = !F32 && BITS != 16;
  constexpr int kImg = kImageBytes<D, BITS, QS>;
  __shared__ __align__(16) uint8_t img_all[kWaves * L::kBlocks * kImg];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = lane % L::kPerBlock, q = l % L::kQ, tg = l / L::kQ, sub = lane / L::kPerBlock;
  const int nblk = a.nbf + 1;
  const uint32_t gw = blockIdx.x * kWaves + wave, id = (gw >> 1) * L::kBlocks + sub;
  const int part = gw & 1;  // 0: keys, 1: values
  if (id >= (uint32_t)a.n_streams * nblk) return;
  const int stream = id / (uint32_t)nblk;  // of the launch
  const int blk = id - (uint32_t)stream * nblk;
  const bool tail = blk == a.nbf;
  const int tok0 = blk * 32;
  int in_stream = stream;               // of the inputs
  uint8_t* sbase = a.region + (int64_t)stream * a.stream_bytes;
  if (a.n_seq > 0) {
    const int j = stream / a.Hkv, h = stream - j * a.Hkv;
    in_stream = a.seq_of[j] * a.Hkv + h;
    sbase = a.region + a.seq_region[j] + (int64_t)h * a.stream_bytes;
  }

  uint8_t* img = img_all + (wave * L::kBlocks + sub) * kImg;
  uint8_t* out = sbase + (tail ? (int64_t)a.nb_cap * a.block_bytes : (int64_t)blk * a.block_bytes);
  const void* in = part ? a.v : a.k;
  Rows<F32> rows;
  int64_t e[8];
  if (BITS == 16 || tail) {
    row_elements<D>(a, in_stream, tok0, tail ? a.n_stored - 1 : tok0 + 31, q, tg, e);
#pragma unroll
    for (int n = 0; n < 8; ++n) rows.template load<kNt>(in, e[n], n);
    const int ntok = tail ? a.n_stored - tok0 : 32;  // valid tokens of this block; zeros after them
    Rows<false> r;
#pragma unroll
    for (int n = 0; n < 8; ++n) r.w[n] = row_token(n, tg) < ntok ? rows.bf16(n) : u4v{0, 0, 0, 0};
    if (part == 0) bf16_keys<D>(r, q, tg, img);
    else bf16_values<D>(r, q, tg, img);
    copy_bf16_part<D>(img, out, part, l);
    return;
  }
  if constexpr (BITS != 16) {
    row_elements<D>(a, in_stream, tok0, tok0 + 31, q, tg, e);
#pragma unroll
    for (int n = 0; n < 8; ++n) rows.template load<kNt>(in, e[n], n);
    if (part == 0) quant_keys<D, BITS, QS>(rows, q, tg, img);
    else quant_values<D, BITS, QS>(rows, q, tg, img);
    copy_quant_part<D, BITS, QS>(img, out, part, l);
  }
}

// Decode-time append of one token to every anchor of a layer range.
struct AppendItem {
  int64_t region;        // byte offset of the anchor's region (of one sequence's streams) in the arena
  int32_t stream_bytes;
  int32_t block_bytes;
  int32_t bits;
  int32_t row;           // the anchor's row in the new-token input (layer - layer_begin)
  int32_t s0;            // input stream (b * Hkv + kvh) of the item's first stream
  int32_t pad;
};

// Items per launch: kernel arguments are limited to 4 KiB.
constexpr int kAppendItems = 120;

struct AppendArgs {
  const void* k;         // [rows][B][Hkv][D] new keys
  const void* v;         // [rows][B][Hkv][D] new values
  uint8_t* arena;
  int32_t in_f32;
  int32_t pos;           // stored tokens before the call: the new token's position
  int32_t nb_cap;
  int32_t n_streams;     // streams per item: B * Hkv, or Hkv under per-sequence plans
  int64_t row_stride;    // elements between the rows of consecutive layers in k and v
  AppendItem items[kAppendItems];
};
static_assert(sizeof(AppendArgs) <= 4096, "kernel arguments");

__device__ __forceinline__ uint16_t new_token_bf16(const void* p, int64_t e, int in_f32) {
  return in_f32 ? f32_to_bf16_bits(static_cast<const float*>(p)[e]) : static_cast<const uint16_t*>(p)[e];
}

// The new token to slot pos % 32 of the bf16 tail block of every stream: one
// thread per (stream, channel), grid (streams * D / 256, anchors).
template <int D>
__global__ __launch_bounds__(256) void tail_write_kernel(AppendArgs a) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= a.n_streams * D) return;
  const int sidx = idx / D, c = idx % D, t = a.pos & 31;
  const AppendItem& it = a.items[blockIdx.y];
  uint8_t* tailb = a.arena + it.region + (int64_t)sidx * it.stream_bytes + (int64_t)a.nb_cap * it.block_bytes;
  const int64_t e = (int64_t)it.row * a.row_stride + (int64_t)(it.s0 + sidx) * D + c;
  *reinterpret_cast<uint16_t*>(tailb + k_bf16_byte(D, t, c)) = new_token_bf16(a.k, e, a.in_f32);
  *reinterpret_cast<uint16_t*>(tailb + v_bf16_byte(D, t, c)) = new_token_bf16(a.v, e, a.in_f32);
}

// The token that fills the tail (pos % 32 == 31) completes a 32-token group: a wave for
// the keys and one for the values of each (stream, anchor), of two streams at d_h 64,
// quantise the tail's bf16 values plus the new token (rounded to bf16) into full block
// pos / 32, exactly as the prefill write quantises a block.  The tail is then empty (its
// stale slots are never read).
template <int D, int QS>
__global__ __launch_bounds__(128) void group_write_kernel(AppendArgs a) {
  using L = Lanes<D>;
  constexpr int kImg = kImageBytes<D, 8, QS>;
  __shared__ __align__(16) uint8_t img_all[2 * L::kBlocks * kImg];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = lane % L::kPerBlock, q = l % L::kQ, tg = l / L::kQ, sub = lane / L::kPerBlock;
  const int part = wave;  // 0: keys, 1: values
  const int sidx = blockIdx.x * L::kBlocks + sub;
  if (sidx >= a.n_streams) return;
  const AppendItem& it = a.items[blockIdx.y];
  uint8_t* base = a.arena + it.region + (int64_t)sidx * it.stream_bytes;
  const uint8_t* tailb = base + (int64_t)a.nb_cap * it.block_bytes;
  const int64_t e0 = (int64_t)it.row * a.row_stride + (int64_t)(it.s0 + sidx) * D + 8 * q;
  // the tail block's pieces are the lane's rows (K) and its channels' tokens (V)
  Rows<false> rows;
  if (part == 0) {
#pragma unroll
    for (int n = 0; n < 8; ++n)
      rows.w[n] = *reinterpret_cast<const u4v*>(tailb + k_bf16_byte(D, row_token(n, tg), 8 * q));
  } else {
    u4v vc[8];
#pragma unroll
    for (int n = 0; n < 8; ++n)
      vc[n] = *reinterpret_cast<const u4v*>(tailb + 64 * D + share_byte(D, 16 * tg + ((8 * q + n) & 15), q >> 1 << 4));
#pragma unroll
    for (int n = 0; n < 8; ++n)
#pragma unroll
      for (int p = 0; p < 4; ++p)
        rows.w[n][p] = __builtin_amdgcn_perm(vc[2 * p + 1][n >> 1], vc[2 * p][n >> 1], n & 1 ? 0x07060302u : 0x05040100u);
  }
  if (tg == 3) {  // row 7 is token 31: the new one in place of a stale slot
    const void* in = part ? a.v : a.k;
    if (a.in_f32) {
      Rows<true> x;
      x.load<false>(in, e0, 0);
      rows.w[7] = x.bf16(0);
    } else {
      rows.load<false>(in, e0, 7);
    }
  }
  uint8_t* img = img_all + (wave * L::kBlocks + sub) * kImg;
  uint8_t* out = base + (int64_t)(a.pos >> 5) * it.block_bytes;
  if (it.bits == 16) {
    if (part == 0) bf16_keys<D>(rows, q, tg, img);
    else bf16_values<D>(rows, q, tg, img);
    copy_bf16_part<D>(img, out, part, l);
    return;
  }
#define KVK_GROUP_BITS(B) \
  { \
    if (part == 0) quant_keys<D, B, QS>(rows, q, tg, img); \
    else quant_values<D, B, QS>(rows, q, tg, img); \
    copy_quant_part<D, B, QS>(img, out, part, l); \
  }
  if (it.bits == 8) KVK_GROUP_BITS(8)
  else if (it.bits == 4) KVK_GROUP_BITS(4)
  else KVK_GROUP_BITS(2)
#undef KVK_GROUP_BITS
}

// Test-only dequantiser: one thread per (stream, token, channel).
template <int D>
__global__ __launch_bounds__(256) void dequant_kernel(const uint8_t* region, int64_t stream_bytes,
                                                      int64_t block_bytes, int nb_cap, int n_stored,
                                                      int n_streams, int bits, int qs, float* kout,
                                                      float* vout) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t total = (int64_t)n_streams * n_stored * D;
  if (idx >= total) return;
  const int c = (int)(idx % D);
  const int64_t st = idx / D;
  const int tok = (int)(st % n_stored);
  const int stream = (int)(st / n_stored);
  const int blk = tok >> 5, t = tok & 31;
  const int nbf = n_stored >> 5;
  const uint8_t* base = region + (int64_t)stream * stream_bytes;
  float kv, vv;
  if (blk >= nbf || bits == 16) {
    const uint8_t* b = base + (blk >= nbf ? (int64_t)nb_cap * block_bytes : (int64_t)blk * block_bytes);
    kv = bf16_to_f32(*reinterpret_cast<const uint16_t*>(b + k_bf16_byte(D, t, c)));
    vv = bf16_to_f32(*reinterpret_cast<const uint16_t*>(b + v_bf16_byte(D, t, c)));
  } else {
    const uint8_t* b = base + (int64_t)blk * block_bytes;
    const uint32_t* w = reinterpret_cast<const uint32_t*>(b);
    const uint32_t mask = (1u << bits) - 1u;
    const int64_t kb = k_code_bit(D, bits, t, c), vb = v_code_bit(D, bits, t, c);
    const uint32_t uk = (w[kb >> 5] >> (kb & 31)) & mask;
    const uint32_t uv = (w[vb >> 5] >> (vb & 31)) & mask;
    const uint16_t* meta = reinterpret_cast<const uint16_t*>(b + 8LL * D * bits);
    if (qs == KVK_Q_GROUP64) {
      const int g = c >> 6, ng = D / 64;
      const int ki = (((t >> 4) * 4 + ((t >> 2) & 3)) * ng * 2 + g * 2) * 4 + (t & 3);
      kv = fmaf((float)uk, f16_bits_to_f32(meta[ki]), f16_bits_to_f32(meta[ki + 4]));
      vv = fmaf((float)uv, f16_bits_to_f32(meta[D + v_meta_index(t, g, 0)]),
                f16_bits_to_f32(meta[D + v_meta_index(t, g, 1)]));
    } else if (qs == KVK_Q_KIVI32) {
      kv = fmaf((float)uk, f16_bits_to_f32(meta[c]), f16_bits_to_f32(meta[D + c]));
      const int g = c >> 5;
      vv = fmaf((float)uv, f16_bits_to_f32(meta[2 * D + v_meta_index(t, g, 0)]),
                f16_bits_to_f32(meta[2 * D + v_meta_index(t, g, 1)]));
    } else {
      const int off = 1 << (bits - 1);
      kv = (float)((int)uk - off) * bf16_to_f32(meta[t]);
      vv = (float)((int)uv - off) * bf16_to_f32(meta[32 + t]);
    }
  }
  kout[idx] = kv;
  vout[idx] = vv;
}

}  // namespace

using namespace kvk;

// One W1 launch over `nstreams` streams of the arguments' layout.
template <int D, int BITS, int QS>
static void launch_w1_kernel(const CompressArgs& a, hipStream_t stream) {
  const auto launch = [&](auto f32) {
    constexpr bool F32 = decltype(f32)::value;
    constexpr int waves = kWriteWaves<D, F32>, blocks = Lanes<D>::kBlocks;
    const int64_t all = 2 * (((int64_t)a.n_streams * (a.nbf + 1) + blocks - 1) / blocks);  // keys and values
    const unsigned grid = (unsigned)((all + waves - 1) / waves);
    hipLaunchKernelGGL((compress_kernel<D, BITS, QS, F32>), dim3(grid), dim3(64 * waves), 0, stream, a);
  };
  if (a.in_f32) launch(std::true_type{});
  else launch(std::false_type{});
}
template <int D, int QS>
static bool launch_w1_bits(const CompressArgs& a, hipStream_t stream) {
  switch (a.bits) {
    case 16: launch_w1_kernel<D, 16, 0>(a, stream); return true;
    case 8: launch_w1_kernel<D, 8, QS>(a, stream); return true;
    case 4: launch_w1_kernel<D, 4, QS>(a, stream); return true;
    case 2: launch_w1_kernel<D, 2, QS>(a, stream); return true;
  }
  return false;
}
template <int D>
static bool launch_w1_scheme(const CompressArgs& a, hipStream_t stream) {
  return a.qs == KVK_Q_KIVI32 ? launch_w1_bits<D, kQsKivi>(a, stream)
                              : (a.qs == KVK_Q_SYMROW ? launch_w1_bits<D, kQsSym>(a, stream)
                                                      : launch_w1_bits<D, kQsG64>(a, stream));
}
static kvk_status launch_w1(CompressArgs& a, int64_t nstreams, hipStream_t stream) {
  if (nstreams * (a.nbf + 1) > 0x7fffffffLL) return fail(KVK_ERR_UNSUPPORTED, "grid too large");
  a.n_streams = (int32_t)nstreams;
  const bool launched = a.D == 128 ? launch_w1_scheme<128>(a, stream) : a.D == 64 && launch_w1_scheme<64>(a, stream);
  if (!launched) return fail(KVK_ERR_UNSUPPORTED, "no write kernel for d_h %d, %d bits", a.D, a.bits);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(KVK_ERR_DEVICE, "compress launch: %s", hipGetErrorString(e));
  return KVK_OK;
}

extern "C" kvk_status kvk_compress_layer(const kvk_table* t, int32_t layer, const void* k, const void* v,
                                         int32_t in_dtype, int32_t n_tokens, const int32_t* keep_idx,
                                         void* arena, hipStream_t stream) {
  if (!t) return fail(KVK_ERR_INVALID, "kvk_compress_layer: NULL table");
  const kvk_dims& d = t->d;
  if (layer < 0 || layer >= d.n_layers) return fail(KVK_ERR_INVALID, "layer %d out of range", layer);
  if (t->plan[layer].inherit) return KVK_OK;  // an inheriting layer writes nothing (§2.1)
  if (!k || !v || !arena) return fail(KVK_ERR_INVALID, "kvk_compress_layer: NULL buffer");
  if (in_dtype != KVK_BF16 && in_dtype != KVK_F32) return fail(KVK_ERR_INVALID, "in_dtype %d", in_dtype);
  if (n_tokens < 1 || n_tokens > d.max_tokens)
    return fail(KVK_ERR_INVALID, "n_tokens %d outside 1..max_tokens (%d)", n_tokens, d.max_tokens);
  const bool evict = d.keep_tokens > 0;
  if (evict && !keep_idx) return fail(KVK_ERR_INVALID, "the table evicts: keep_idx is required");
  if (!evict && keep_idx) return fail(KVK_ERR_INVALID, "the table does not evict: keep_idx must be NULL");
  if (evict && n_tokens < d.keep_tokens)
    return fail(KVK_ERR_INVALID, "n_tokens %d < keep_tokens %d", n_tokens, d.keep_tokens);
  if ((reinterpret_cast<uintptr_t>(arena) & 15) || (reinterpret_cast<uintptr_t>(k) & 15) ||
      (reinterpret_cast<uintptr_t>(v) & 15))
    return fail(KVK_ERR_INVALID, "misaligned buffer (16-byte alignment required)");
  if (kvk_status st = check_gpu_buffers({k, v, keep_idx, arena}, "kvk_compress_layer")) return st;
  if (!t->seq.empty()) {  // per-sequence plans: each sequence's own table and arena
    // The inputs stay indexed by the batch's sequence (GQA: K and V [B][Hkv][n][d_h];
    // MLA: latent [B][n][r] and positional key [B][n][d_R]).
    if (d.kind != KVK_MLA) {
      // One launch per bit-width for the sequences whose plans store the layer at it
      // (each sequence still written exactly as its one-sequence table writes it).
      for (const int bits : {16, 8, 4, 2}) {
        CompressArgs a;
        a.k = k;
        a.v = v;
        a.keep = keep_idx;
        a.region = static_cast<uint8_t*>(arena);
        a.in_f32 = in_dtype == KVK_F32;
        a.n_tokens = n_tokens;
        a.n_stored = evict ? d.keep_tokens : n_tokens;
        a.nbf = a.n_stored / KVK_GROUP;
        a.nb_cap = t->nb_cap;
        a.D = d.head_dim;
        a.bits = bits;
        a.qs = d.qscheme;
        a.Hkv = d.n_kv_heads;
        a.n_seq = 0;
        for (int b = 0; b < d.batch; ++b) {
          const kvk_table* s = t->seq[b];
          if (s->plan[layer].inherit || s->bits[layer] != bits) continue;
          a.block_bytes = s->block_bytes[layer];      // equal for every sequence at this bit-width
          a.stream_bytes = s->info.stream_bytes[layer];
          a.seq_of[a.n_seq] = b;
          a.seq_region[a.n_seq] = t->seq_base[b] + s->info.layer_offset[layer];
          if (++a.n_seq == kWriteSeqs) {
            const kvk_status st = launch_w1(a, (int64_t)a.n_seq * d.n_kv_heads, stream);
            if (st != KVK_OK) return st;
            a.n_seq = 0;
          }
        }
        if (a.n_seq > 0) {
          const kvk_status st = launch_w1(a, (int64_t)a.n_seq * d.n_kv_heads, stream);
          if (st != KVK_OK) return st;
        }
      }
      return KVK_OK;
    }
    return mla_compress_layer_batched(t, layer, k, v, in_dtype, n_tokens, keep_idx, arena, stream);
  }
  if (d.kind == KVK_MLA)
    return mla_compress_layer(t, layer, k, v, in_dtype, n_tokens, keep_idx, arena, stream);

  CompressArgs a;
  a.k = k;
  a.v = v;
  a.keep = keep_idx;
  a.region = static_cast<uint8_t*>(arena) + t->info.layer_offset[layer];
  a.block_bytes = t->block_bytes[layer];
  a.stream_bytes = t->info.stream_bytes[layer];
  a.in_f32 = in_dtype == KVK_F32;
  a.n_tokens = n_tokens;
  a.n_stored = evict ? d.keep_tokens : n_tokens;
  a.nbf = a.n_stored / KVK_GROUP;
  a.nb_cap = t->nb_cap;
  a.D = d.head_dim;
  a.bits = t->bits[layer];
  a.qs = d.qscheme;
  a.n_seq = 0;
  a.Hkv = d.n_kv_heads;
  return launch_w1(a, (int64_t)d.batch * d.n_kv_heads, stream);
}

static kvk_status append_gqa(const kvk_table* t, int32_t l0, int32_t l1, const void* k, const void* v,
                             int32_t in_dtype, int32_t n_stored, void* arena, hipStream_t stream);

extern "C" kvk_status kvk_compress_layer_project(const kvk_table* t, int32_t layer, const void* x,
                                                 const void* w_dkv, int32_t d_model, const void* k_rope,
                                                 int32_t n_tokens, const int32_t* keep_idx, void* arena,
                                                 void* latent_out, hipStream_t stream) {
  if (!t) return fail(KVK_ERR_INVALID, "kvk_compress_layer_project: NULL table");
  const kvk_dims& d = t->d;
  if (d.kind != KVK_MLA) return fail(KVK_ERR_INVALID, "kvk_compress_layer_project: an MLA table is required");
  if (layer < 0 || layer >= d.n_layers) return fail(KVK_ERR_INVALID, "layer %d out of range", layer);
  const bool per_seq = !t->seq.empty();
  if (per_seq && latent_out)
    return fail(KVK_ERR_INVALID, "kvk_compress_layer_project: latent_out must be NULL for per-sequence tables");
  if (!per_seq && t->plan[layer].inherit) return KVK_OK;  // an inheriting layer writes nothing (§2.1)
  if (!x || !w_dkv || !k_rope || !arena) return fail(KVK_ERR_INVALID, "kvk_compress_layer_project: NULL buffer");
  if (d_model < 32 || d_model % 32)
    return fail(KVK_ERR_INVALID, "d_model %d: a positive multiple of 32", d_model);
  if (n_tokens < 1 || n_tokens > d.max_tokens)
    return fail(KVK_ERR_INVALID, "n_tokens %d outside 1..max_tokens (%d)", n_tokens, d.max_tokens);
  const bool evict = d.keep_tokens > 0;
  if (evict && !keep_idx) return fail(KVK_ERR_INVALID, "the table evicts: keep_idx is required");
  if (!evict && keep_idx) return fail(KVK_ERR_INVALID, "the table does not evict: keep_idx must be NULL");
  if (evict && n_tokens < d.keep_tokens)
    return fail(KVK_ERR_INVALID, "n_tokens %d < keep_tokens %d", n_tokens, d.keep_tokens);
  if ((reinterpret_cast<uintptr_t>(arena) & 15) || (reinterpret_cast<uintptr_t>(x) & 15) ||
      (reinterpret_cast<uintptr_t>(w_dkv) & 15) || (reinterpret_cast<uintptr_t>(k_rope) & 15) ||
      (reinterpret_cast<uintptr_t>(latent_out) & 15))
    return fail(KVK_ERR_INVALID, "misaligned buffer (16-byte alignment required)");
  if (kvk_status st = check_gpu_buffers({x, w_dkv, k_rope, keep_idx, arena, latent_out}, "kvk_compress_layer_project"))
    return st;
  if (per_seq)  // each sequence's own table and arena, the inputs indexed by the batch's sequence
    return mla_compress_layer_project_batched(t, layer, x, w_dkv, d_model, k_rope, n_tokens, keep_idx, arena, stream);
  return mla_compress_layer_project(t, layer, x, w_dkv, d_model, k_rope, n_tokens, keep_idx, arena, latent_out,
                                    stream);
}

extern "C" kvk_status kvk_append_token(const kvk_table* t, int32_t l0, int32_t l1, const void* k, const void* v,
                                       int32_t in_dtype, int32_t n_stored, void* arena, hipStream_t stream) {
  if (!t) return fail(KVK_ERR_INVALID, "kvk_append_token: NULL table");
  const kvk_dims& d = t->d;
  if (l0 < 0 || l1 > d.n_layers || l0 >= l1)
    return fail(KVK_ERR_INVALID, "layer range [%d, %d) invalid for %d layers", l0, l1, d.n_layers);
  if (!k || !v || !arena) return fail(KVK_ERR_INVALID, "kvk_append_token: NULL buffer");
  if (in_dtype != KVK_BF16 && in_dtype != KVK_F32) return fail(KVK_ERR_INVALID, "in_dtype %d", in_dtype);
  if (n_stored < 0 || n_stored >= t->cap)
    return fail(KVK_ERR_INVALID, "n_stored %d: the stream holds at most %d tokens", n_stored, t->cap);
  if ((reinterpret_cast<uintptr_t>(arena) & 15) || (reinterpret_cast<uintptr_t>(k) & 15) ||
      (reinterpret_cast<uintptr_t>(v) & 15))
    return fail(KVK_ERR_INVALID, "misaligned buffer (16-byte alignment required)");
  bool stores = false;  // an anchor in the range (of some sequence's plan)
  for (size_t i = 0; i < (t->seq.empty() ? 1 : t->seq.size()); ++i)
    for (int l = l0; l < l1; ++l) stores |= !(t->seq.empty() ? t : t->seq[i])->plan[l].inherit;
  if (!stores) return KVK_OK;  // only inheritors: nothing is stored
  if (kvk_status st = check_gpu_buffers({k, v, arena}, "kvk_append_token")) return st;
  if (d.kind == KVK_MLA) return mla_append_token(t, l0, l1, k, v, in_dtype, n_stored, arena, stream);
  return append_gqa(t, l0, l1, k, v, in_dtype, n_stored, arena, stream);
}

// One item per (anchor layer) of a shared plan, over all B * Hkv streams; under
// per-sequence plans one per (sequence, anchor layer of its plan), over its Hkv
// streams.  Launched in groups of up to kAppendItems items.
static kvk_status append_gqa(const kvk_table* t, int32_t l0, int32_t l1, const void* k, const void* v,
                             int32_t in_dtype, int32_t n_stored, void* arena, hipStream_t stream) {
  const kvk_dims& d = t->d;
  const bool per_seq = !t->seq.empty();
  std::vector<AppendItem> items;
  for (int b = 0; b < (per_seq ? d.batch : 1); ++b) {
    const kvk_table* st = per_seq ? t->seq[b] : t;
    const int64_t base = per_seq ? t->seq_base[b] : 0;
    for (int l = l0; l < l1; ++l) {
      if (st->plan[l].inherit) continue;  // an inheriting layer stores nothing (§2.1)
      AppendItem it;
      it.region = base + st->info.layer_offset[l];
      it.stream_bytes = (int32_t)st->info.stream_bytes[l];
      it.block_bytes = (int32_t)st->block_bytes[l];
      it.bits = st->bits[l];
      it.row = l - l0;
      it.s0 = per_seq ? b * d.n_kv_heads : 0;
      it.pad = 0;
      items.push_back(it);
    }
  }
  AppendArgs a;
  a.k = k;
  a.v = v;
  a.arena = static_cast<uint8_t*>(arena);
  a.in_f32 = in_dtype == KVK_F32;
  a.pos = n_stored;
  a.nb_cap = t->nb_cap;
  a.n_streams = per_seq ? d.n_kv_heads : d.batch * d.n_kv_heads;
  a.row_stride = (int64_t)d.batch * d.n_kv_heads * d.head_dim;
  const int qs = d.qscheme;
  const dim3 b3(256);
  for (size_t i0 = 0; i0 < items.size(); i0 += kAppendItems) {
    const int n = (int)std::min<size_t>(kAppendItems, items.size() - i0);
    std::copy(items.begin() + i0, items.begin() + i0 + n, a.items);
    if (n_stored % KVK_GROUP != KVK_GROUP - 1) {
      const dim3 g3((unsigned)((a.n_streams * d.head_dim + 255) / 256), (unsigned)n);
      if (d.head_dim == 128) hipLaunchKernelGGL(tail_write_kernel<128>, g3, b3, 0, stream, a);
      else hipLaunchKernelGGL(tail_write_kernel<64>, g3, b3, 0, stream, a);
    } else {
      const int per_wg = d.head_dim == 128 ? 1 : 2;  // streams of a workgroup
      const dim3 g3((unsigned)((a.n_streams + per_wg - 1) / per_wg), (unsigned)n), b2(128);
      if (d.head_dim == 128) {
        if (qs == KVK_Q_KIVI32) hipLaunchKernelGGL((group_write_kernel<128, kQsKivi>), g3, b2, 0, stream, a);
        else if (qs == KVK_Q_GROUP64) hipLaunchKernelGGL((group_write_kernel<128, kQsG64>), g3, b2, 0, stream, a);
        else hipLaunchKernelGGL((group_write_kernel<128, kQsSym>), g3, b2, 0, stream, a);
      } else {
        if (qs == KVK_Q_KIVI32) hipLaunchKernelGGL((group_write_kernel<64, kQsKivi>), g3, b2, 0, stream, a);
        else if (qs == KVK_Q_GROUP64) hipLaunchKernelGGL((group_write_kernel<64, kQsG64>), g3, b2, 0, stream, a);
        else hipLaunchKernelGGL((group_write_kernel<64, kQsSym>), g3, b2, 0, stream, a);
      }
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(KVK_ERR_DEVICE, "append launch: %s", hipGetErrorString(e));
  }
  return KVK_OK;
}

extern "C" kvk_status kvk_debug_dequantize(const kvk_table* t, int32_t layer, int32_t n_stored,
                                           const void* arena, float* k_out, float* v_out,
                                           hipStream_t stream) {
  if (!t) return fail(KVK_ERR_INVALID, "kvk_debug_dequantize: NULL table");
  const kvk_dims& d = t->d;
  if (layer < 0 || layer >= d.n_layers) return fail(KVK_ERR_INVALID, "layer %d out of range", layer);
  if (!arena || !k_out || !v_out) return fail(KVK_ERR_INVALID, "NULL buffer");
  if (n_stored < 0 || n_stored > t->cap)
    return fail(KVK_ERR_INVALID, "n_stored %d outside 0..%d", n_stored, t->cap);
  if (n_stored == 0) return KVK_OK;
  if (kvk_status st = check_gpu_buffers({arena, k_out, v_out}, "kvk_debug_dequantize")) return st;
  if (d.kind == KVK_MLA && !t->seq.empty()) {
    // sequence b's values at b n_stored r (latent, rows of its own kept width) and
    // b n_stored d_R (positional key)
    for (int b = 0; b < d.batch; ++b) {
      const kvk_status st = mla_debug_dequantize(t->seq[b], layer, n_stored,
                                                 static_cast<const uint8_t*>(arena) + t->seq_base[b],
                                                 k_out + (int64_t)b * n_stored * d.latent_dim,
                                                 v_out + (int64_t)b * n_stored * d.rope_dim, stream);
      if (st != KVK_OK) return st;
    }
    return KVK_OK;
  }
  if (d.kind == KVK_MLA) return mla_debug_dequantize(t, layer, n_stored, arena, k_out, v_out, stream);
  if (!t->seq.empty()) {
    const int64_t per = (int64_t)d.n_kv_heads * n_stored * d.head_dim;
    for (int b = 0; b < d.batch; ++b) {
      const kvk_status st = kvk_debug_dequantize(t->seq[b], layer, n_stored,
                                                 static_cast<const uint8_t*>(arena) + t->seq_base[b],
                                                 k_out + b * per, v_out + b * per, stream);
      if (st != KVK_OK) return st;
    }
    return KVK_OK;
  }
  const int a = t->info.anchor_of[layer];
  const uint8_t* region = static_cast<const uint8_t*>(arena) + t->info.layer_offset[a];
  const int nstreams = d.batch * d.n_kv_heads;
  const int64_t total = (int64_t)nstreams * n_stored * d.head_dim;
  const int64_t grid = (total + 255) / 256;
  if (grid > 0x7fffffffLL) return fail(KVK_ERR_UNSUPPORTED, "grid too large");
  const int qs = d.qscheme;
  if (d.head_dim == 128)
    hipLaunchKernelGGL(dequant_kernel<128>, dim3((unsigned)grid), dim3(256), 0, stream, region,
                       t->info.stream_bytes[a], t->block_bytes[a], t->nb_cap, n_stored, nstreams,
                       t->bits[a], qs, k_out, v_out);
  else
    hipLaunchKernelGGL(dequant_kernel<64>, dim3((unsigned)grid), dim3(256), 0, stream, region,
                       t->info.stream_bytes[a], t->block_bytes[a], t->nb_cap, n_stored, nstreams,
                       t->bits[a], qs, k_out, v_out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(KVK_ERR_DEVICE, "dequantise launch: %s", hipGetErrorString(e));
  return KVK_OK;
}
