// quant.hip -- quantize + pack of prompt tokens (Alg. 1, Eq. 7), the fp16 tail
// append and the block close of generated tokens (Alg. 2), for gfx950.
//
// One workgroup (256 threads) builds one 64-slot record of one pool of one
// (sequence, layer, kv head) unit.  Four lanes own one token row (consecutive
// lanes, or for the rotating bases lanes 16 apart): quarter q loads channels
// [32q, 32q+32).  Codes go to LDS, then each thread packs
// whole segments (Sec. 4.1 mixed-radix symbols) into the LDS body with atomic
// ORs, and the record is written with 16-byte stores.
#include <hip/hip_fp16.h>

#include <type_traits>

#include "semkv_internal.h"

namespace semkv {
namespace {

constexpr int kPitch = 132;             // LDS row pitch of the code arrays (bytes)
constexpr int kMaxBodyWords = 3072 / 4; // largest body: L = 8

__device__ inline float h2f(uint16_t b) { return __half2float(__ushort_as_half(b)); }
__device__ inline uint16_t f2h(float f) { return __half_as_ushort(__float2half_rn(f)); }
// fp16 bits with +-inf replaced by +-65504, the largest finite binary16: the
// two parameters of a group stay finite for finite input, and the codes are
// taken against the stored (saturated) pair
__device__ inline uint16_t sat16(uint16_t h) {
  return (h & 0x7FFFu) == 0x7C00u ? uint16_t((h & 0x8000u) | 0x7BFFu) : h;
}

// Correctly rounded fp32 square root of a >= 0.  The hardware result is within
// one ulp; the neighbour whose rounding interval holds sqrt(a) is chosen by
// comparing a with the squared interval ends, which are exact in double (a
// 25-bit midpoint squares to at most 50 bits).  sqrt is never exactly halfway
// between two floats, so no tie arises.
__device__ inline float sqrt_rn(float a) {
  float r = __builtin_sqrtf(a);
  if (!(a > 0.0f) || !(a < INFINITY)) return r;
  const double ad = double(a);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float dn = __uint_as_float(__float_as_uint(r) - 1u), up = __uint_as_float(__float_as_uint(r) + 1u);
    const double lo = 0.5 * (double(dn) + double(r)), hi = 0.5 * (double(r) + double(up));
    if (ad < lo * lo) r = dn;
    else if (ad >= hi * hi) r = up;
  }
  return r;
}

// fp16 of the correctly rounded fp32 square root of a >= 0: the hardware's
// root is within one ulp, so only where its neighbours two ulps away round to
// different fp16 values (one row in two thousand) is the exact root needed.
__device__ inline uint16_t sqrt_f16(float a) {
  const float r = __builtin_amdgcn_sqrtf(a);
  const uint32_t b = __float_as_uint(r);
  const uint16_t lo = f2h(__uint_as_float(b - 2u)), hi = f2h(__uint_as_float(b + 2u));
  if (lo == hi && b > 2u) return lo;         // a = 0, infinities and NaN take the exact way
  return f2h(sqrt_rn(a));
}

// The value of lane (this lane xor 1) or xor 2: exact DPP moves within a quad at full VALU rate.  Every lane has a
// source lane, so the move needs no prior value (none to materialize, and the
// compiler may fold the move into the add that uses it).
template <int CTRL>
__device__ inline float quad_mov(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E;

// Minimum and maximum of a row quarter (32 fp16 values), two values at a time
// and NaN if any is one: the quarter's finiteness comes with them.
typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
__device__ inline void quarter_range(const uint32_t d[16], float& mn, float& mx) {
  h16x2 a = __builtin_bit_cast(h16x2, d[0]), b = a;
#pragma unroll
  for (int i = 1; i < 15; i += 2) {
    const h16x2 x = __builtin_bit_cast(h16x2, d[i]), y = __builtin_bit_cast(h16x2, d[i + 1]);
    a = __builtin_elementwise_minimum(__builtin_elementwise_minimum(a, x), y);
    b = __builtin_elementwise_maximum(__builtin_elementwise_maximum(b, x), y);
  }
  const h16x2 z = __builtin_bit_cast(h16x2, d[15]);
  a = __builtin_elementwise_minimum(a, z);
  b = __builtin_elementwise_maximum(b, z);
  mn = float(__builtin_elementwise_minimum(a.x, a.y));
  mx = float(__builtin_elementwise_maximum(b.x, b.y));
}

// Asymmetric affine quantizer (Sec. 4.1) of one row quarter; the min/max of a
// group of G channels is combined over the G/32 lanes holding it.  Returns
// {scale, zero} as fp16 bits (low half = scale).
template <int L>
__device__ uint32_t affine_quarter(const uint32_t d[16], int G, uint32_t code[8], bool& nonfinite) {
  float x[32];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    x[2 * i] = h2f(uint16_t(d[i] & 0xFFFFu));
    x[2 * i + 1] = h2f(uint16_t(d[i] >> 16));
  }
  float mn, mx;
  quarter_range(d, mn, mx);
  const bool odd = !(mn > -INFINITY && mx < INFINITY);       // an infinity or a NaN (which both carry)
  nonfinite |= odd;
  if (odd) {                                                  // the range of the other values
    mn = mx = x[0];
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      mn = fminf(mn, x[i]);
      mx = fmaxf(mx, x[i]);
    }
  }
  if (G >= 64) {
    mn = fminf(mn, quad_mov<kQuadXor1>(mn));
    mx = fmaxf(mx, quad_mov<kQuadXor1>(mx));
  }
  if (G >= 128) {
    mn = fminf(mn, quad_mov<kQuadXor2>(mn));
    mx = fmaxf(mx, quad_mov<kQuadXor2>(mx));
  }
  float zero = mn + 0.0f;                               // -0 -> +0
  uint16_t s16 = f2h(__fdiv_rn(mx - mn, float(L - 1)));
  // only 2 levels can overflow: (max - min) / 1 reaches 131008, while for
  // L >= 3 the quotient is at most 65504
  if constexpr (L == 2) s16 = sat16(s16);
  float sf = h2f(s16);
  float inv = sf == 0.0f ? 0.0f : __fdiv_rn(1.0f, sf);
  // clamp to [0, L-1] (NaN -> 0), then one convert-and-insert per code: the
  // convert rounds to nearest even, and with integer bounds clamping before
  // rounding gives the code rounding before clamping gives
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    uint32_t w = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float c = fminf(fmaxf((x[4 * k + e] - zero) * inv, 0.0f), float(L - 1));
      w = __builtin_amdgcn_cvt_pk_u8_f32(c, e, w);
    }
    code[k] = w;
  }
  return uint32_t(s16) | (uint32_t(f2h(zero)) << 16);
}

// H diag(sign) x of one row quarter (the dequantizer's layout: a row's
// quarters in the four lanes of a quad): sign flip, then the unnormalized
// Walsh-Hadamard transform, stages 1..16 inside the lane and 32, 64 across
// the lanes of the row's quad.
__device__ inline void rotate_quarter(const float x[32], int q, uint32_t sbits, float u[32]) {
#pragma unroll
  for (int i = 0; i < 32; ++i) u[i] = __uint_as_float(__float_as_uint(x[i]) ^ ((sbits << (31 - i)) & 0x80000000u));
#pragma unroll
  for (int h = 1; h < 32; h <<= 1)
#pragma unroll
    for (int i = 0; i < 32; ++i)
      if (!(i & h)) {
        float p = u[i], r = u[i + h];
        u[i] = p + r;
        u[i + h] = p - r;
      }
  // cross-lane stages: the upper lane of a pair takes o - u = o + (-u), the
  // lower u + o = o + u (IEEE addition commutes; -u is a sign flip)
  const uint32_t f1 = (q & 1) ? 0x80000000u : 0u, f2 = (q & 2) ? 0x80000000u : 0u;
#pragma unroll
  for (int i = 0; i < 32; ++i) {                         // h = 32: partner lane q ^ 1
    const float o = quad_mov<kQuadXor1>(u[i]);
    u[i] = o + __uint_as_float(__float_as_uint(u[i]) ^ f1);
  }
#pragma unroll
  for (int i = 0; i < 32; ++i) {                         // h = 64: partner lane q ^ 2
    const float o = quad_mov<kQuadXor2>(u[i]);
    u[i] = o + __uint_as_float(__float_as_uint(u[i]) ^ f2);
  }
}

// ---- rows of the rotating bases while they are quantized
// A token row sits in the lanes l, l + 16, l + 32, l + 48 of a wave: lane
// quarter q = lane / 16 loads channels [32 q, 32 q + 32).  The two stages that
// cross lanes then swap 16-lane rows between two registers
// (v_permlane16_swap, v_permlane32_swap): one register gets both lower halves,
// the other both upper ones, and a butterfly is an add and a subtract with no
// sign flips and no wait states, 1.5 instructions per value and stage; a
// quad's lane exchange by DPP took two and the wait states of its hazards.
// The lanes then hold other channels than they loaded (rot_channel).
// Bound by vector instructions (tq: the VALU issues one per 3.4 cycles, about
// what four waves reach).  With the signs applied to packed fp16 pairs, the
// norm's tree by the same swaps, thresholds as clamped multiply-adds and the
// finiteness check on one rotated value, ranking and quantizing 131072 tokens
// of 8 layers at 4/3 levels went from 1.52 to 1.28 ms, 3 x 10007 tokens of the
// rotated affine base from 305 to 289 us.
// The swaps are written in place (the compiler's own intrinsic copied both
// registers first, 2 moves a swap) and four at a time behind the two wait
// states that a swap needs after a vector write of its registers.  Called with
// the row's four lanes active.
__device__ inline void swap16(float& a, float& b) {          // a: both even rows of 16, b: both odd ones
  __asm__("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ inline void swap32(float& a, float& b) {          // a: both lower halves of 32, b: both upper ones
  __asm__("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ inline void swap16x4(float& a0, float& b0, float& a1, float& b1, float& a2, float& b2, float& a3, float& b3) {
  __asm__("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3\n\t"
          "v_permlane16_swap_b32 %4, %5\n\tv_permlane16_swap_b32 %6, %7"
          : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1), "+v"(a2), "+v"(b2), "+v"(a3), "+v"(b3));
}
__device__ inline void swap32x4(float& a0, float& b0, float& a1, float& b1, float& a2, float& b2, float& a3, float& b3) {
  __asm__("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\tv_permlane32_swap_b32 %2, %3\n\t"
          "v_permlane32_swap_b32 %4, %5\n\tv_permlane32_swap_b32 %6, %7"
          : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1), "+v"(a2), "+v"(b2), "+v"(a3), "+v"(b3));
}
__device__ inline void swap16x2(float& a0, float& b0, float& a1, float& b1) {
  __asm__("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3" : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1));
}
__device__ inline void swap32x2(float& a0, float& b0, float& a1, float& b1) {
  __asm__("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\tv_permlane32_swap_b32 %2, %3" : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1));
}
// the value of f over the four lanes of a row, in all of them
template <class F>
__device__ inline float row_reduce(float v, F f) {
  float w = v;
  swap16(v, w);
  v = f(v, w);
  w = v;
  swap32(v, w);
  return f(v, w);
}

// Sign masks of a row quarter's 16 fp16 pairs.
__device__ inline void sign_masks(uint32_t sbits, uint32_t m[16]) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const uint32_t t = i < 8 ? sbits << (15 - 2 * i) : sbits >> (2 * i - 15);   // bits 2i, 2i + 1 at 15, 16
    m[i] = (t & 0x8000u) | ((t << 15) & 0x80000000u);
  }
}

// diag(sign) x of a row quarter as fp32 (zeros for a row that is not there)
__device__ inline void load_signed(const uint16_t* src, bool valid, const uint32_t m[16], float x[32]) {
  const uint4* p = reinterpret_cast<const uint4*>(src);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint4 w = valid ? p[k] : make_uint4(0u, 0u, 0u, 0u);
    const uint32_t d[4] = {w.x ^ m[4 * k], w.y ^ m[4 * k + 1], w.z ^ m[4 * k + 2], w.w ^ m[4 * k + 3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[8 * k + 2 * e] = h2f(uint16_t(d[e] & 0xFFFFu));
      x[8 * k + 2 * e + 1] = h2f(uint16_t(d[e] >> 16));
    }
  }
}

// H x of the row, stages 1..16 inside the lane, 32 and 64 across its lanes,
// each as lower + upper and lower - upper.  Register 16 q0 + 8 q1 + i then holds
// channel rot_channel(lane) + 64 q1 + 32 q0 + i.
__device__ inline int rot_channel(int lane) { return (lane & 16) + ((lane & 32) >> 2); }
__device__ inline void rotate_row(float u[32]) {
#pragma unroll
  for (int h = 1; h < 32; h <<= 1)
#pragma unroll
    for (int i = 0; i < 32; ++i)
      if (!(i & h)) {
        const float p = u[i], r = u[i + h];
        u[i] = p + r;
        u[i + h] = p - r;
      }
#pragma unroll
  for (int i = 0; i < 16; i += 4) {                          // h = 32: lane quarters 0-1, 2-3
    swap16x4(u[i], u[i + 16], u[i + 1], u[i + 17], u[i + 2], u[i + 18], u[i + 3], u[i + 19]);
#pragma unroll
    for (int k = i; k < i + 4; ++k) {
      const float p = u[k], r = u[k + 16];
      u[k] = p + r;
      u[k + 16] = p - r;
    }
  }
#pragma unroll
  for (int g = 0; g < 32; g += 16)
#pragma unroll
    for (int i = g; i < g + 8; i += 4) {                     // h = 64: lane halves
      swap32x4(u[i], u[i + 8], u[i + 1], u[i + 9], u[i + 2], u[i + 10], u[i + 3], u[i + 11]);
#pragma unroll
      for (int k = i; k < i + 4; ++k) {
        const float p = u[k], r = u[k + 8];
        u[k] = p + r;
        u[k + 8] = p - r;
      }
    }
}

// The row norm's square: the squares summed by the fixed pairwise tree
// (channels 64 apart, then 32, 16, ..., 1), in every lane of the row.
__device__ inline float row_square_sum(const float x[32]) {
  float a[16];
#pragma unroll
  for (int m = 0; m < 16; m += 4) {                          // 64: i = 2 m + lane half
    float q[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) q[k] = x[2 * m + k] * x[2 * m + k];
    swap32x4(q[0], q[1], q[2], q[3], q[4], q[5], q[6], q[7]);
#pragma unroll
    for (int k = 0; k < 4; ++k) a[m + k] = q[2 * k] + q[2 * k + 1];
  }
#pragma unroll
  for (int m = 0; m < 8; m += 4) {                           // 32: i = 4 m + 2 (odd row) + lane half
    swap16x4(a[2 * m], a[2 * m + 1], a[2 * m + 2], a[2 * m + 3], a[2 * m + 4], a[2 * m + 5], a[2 * m + 6], a[2 * m + 7]);
#pragma unroll
    for (int k = 0; k < 4; ++k) a[m + k] = a[2 * (m + k)] + a[2 * (m + k) + 1];
  }
#pragma unroll
  for (int h = 4; h >= 1; h >>= 1)                           // 16, 8, 4
#pragma unroll
    for (int m = 0; m < h; ++m) a[m] = a[m] + a[m + h];
  return row_reduce(a[0], [](float p, float r) { return p + r; });   // 2, 1
}

// TurboQuant-MSE base (Sec. 4.9) of one row (signed, not yet rotated, in u):
// the row norm, one fp16 scalar, and Lloyd-Max threshold codes of the rotated
// row.  A threshold's step is one clamped multiply-add: (u - t) 2^64 is 0 or
// below where u <= t, and at least 1 where u > t (u and t differ by at least
// 2^-49: u is a multiple of 2^-24, t has 24 significant bits and is 0 or at
// least 2^-26).  Returns rho bits.
template <int L>
__device__ uint16_t tq_row(float u[32], const float* tau, uint32_t code[8]) {
  uint16_t r16 = sqrt_f16(row_square_sum(u));
  if ((r16 & 0x7FFFu) == 0x7C00u) r16 = 0x7BFFu;       // saturate to 65504
  rotate_row(u);
  const float rf = h2f(r16);
  constexpr float kBig = 18446744073709551616.0f;      // 2^64
  float thr[L - 1];
#pragma unroll
  for (int k = 0; k < L - 1; ++k) thr[k] = -(rf * tau[k]) * kBig;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    uint32_t w = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float c = 0.0f;
#pragma unroll
      for (int t = 0; t < L - 1; ++t) {
        float f;
        __asm__("v_fma_f32 %0, %1, %2, %3 clamp" : "=v"(f) : "v"(u[4 * k + e]), "s"(kBig), "v"(thr[t]));
        c = t == 0 ? f : c + f;
      }
      w = __builtin_amdgcn_cvt_pk_u8_f32(c, e, w);
    }
    code[k] = w;
  }
  return r16;
}

// The reductions f and g of a row's NG values of v and of w, one value a group:
// lane quarter q is left with those of group q % NG (NG = 1: every lane).  The
// swaps halve the values held as they fold the row, so four groups take 6 swaps
// (each group folded over the row by itself: 16).
template <int NG, class F, class E>
__device__ inline void row_reduce_groups(float (&v)[NG], float (&w)[NG], F f, E g, float& rv, float& rw) {
  if constexpr (NG == 4) {
    swap16x4(v[0], v[1], v[2], v[3], w[0], w[1], w[2], w[3]);
    float a = f(v[0], v[1]), b = f(v[2], v[3]), c = g(w[0], w[1]), d = g(w[2], w[3]);
    swap32x2(a, b, c, d);
    rv = f(a, b), rw = g(c, d);
  } else {
    float a, c;
    if constexpr (NG == 2) {
      swap16x2(v[0], v[1], w[0], w[1]);
      a = f(v[0], v[1]), c = g(w[0], w[1]);
    } else {
      float b = a = v[0], d = c = w[0];
      swap16x2(a, b, c, d);
      a = f(a, b), c = g(c, d);
    }
    float b = a, d = c;
    swap32x2(a, b, c, d);
    rv = f(a, b), rw = g(c, d);
  }
}
// The way back: x and y of group q % NG, held by lane quarter q, in every lane
// of the row as xs[group] and ys[group].
template <int NG>
__device__ inline void row_spread_groups(float x, float y, float (&xs)[NG], float (&ys)[NG]) {
  if constexpr (NG == 4) {
    float a = x, b = x, c = y, d = y;
    swap32x2(a, b, c, d);                    // a, c: of quarters 0 and 1, in both halves; b, d: of 2 and 3
    xs[0] = xs[1] = a, xs[2] = xs[3] = b;
    ys[0] = ys[1] = c, ys[2] = ys[3] = d;
    swap16x4(xs[0], xs[1], xs[2], xs[3], ys[0], ys[1], ys[2], ys[3]);
  } else if constexpr (NG == 2) {
    xs[0] = xs[1] = x, ys[0] = ys[1] = y;
    swap16x2(xs[0], xs[1], ys[0], ys[1]);
  } else {
    xs[0] = x, ys[0] = y;
  }
}

// Affine quantizer of the rotated row (Sec. 4.1 with its Hadamard rotation):
// y = H diag(sign) x / 16 (the division is exact), then per group of G
// rotated coordinates zero = fp16(min y) (-0 stored as +0) and scale =
// fp16(max(0, (max y - zero) / (L-1))), each saturated at +-65504, codes
// against the stored pair.  u: H diag(sign) x.  Returns {scale, zero} of the
// lane quarter's group (q % (128 / G)) as fp16 bits (low half = scale).
// Every lane holds channels of every group, but works out the parameters of
// one and gets the others' by swaps: two IEEE divisions a row and lane.  With
// every group's parameters in every lane (eight divisions at G = 32), packing
// 16 x 4096 tokens of a layer at 6/5 levels took 127 us at G = 32 and 110 at
// 64, now 100 and 97 (100 at 128).
template <int L, int G>
__device__ inline uint32_t rot_affine_row(const float u[32], uint32_t code[8]) {
  constexpr int NG = 128 / G;
  float mn[NG], mx[NG];
#pragma unroll
  for (int i = 0; i < NG; ++i) mn[i] = INFINITY, mx[i] = -INFINITY;
  // registers 16 q0 + 8 q1 + i, i < 8, are of group (64 q1 + 32 q0) / G
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const int g = (64 * ((i >> 3) & 1) + 32 * (i >> 4)) / G;
    mn[g] = fminf(mn[g], u[i]);
    mx[g] = fmaxf(mx[g], u[i]);
  }
  float lo, hi;
  row_reduce_groups<NG>(mn, mx, [](float p, float r) { return fminf(p, r); }, [](float p, float r) { return fmaxf(p, r); }, lo, hi);
  // the exact 1/16 of the extremes; of the values in the code's subtraction
  lo *= 0.0625f;
  hi *= 0.0625f;
  // rotated coordinates reach 128 * 65504 / 16 in magnitude: both parameters
  // saturate at +-65504
  uint16_t z16 = sat16(f2h(lo));
  z16 = z16 == 0x8000u ? uint16_t(0) : z16;
  const float z = h2f(z16);
  const float s32 = __fdiv_rn(hi - z, float(L - 1));
  const uint16_t s16 = sat16(f2h(s32 > 0.0f ? s32 : 0.0f));
  const float sf = h2f(s16);
  float zero[NG], inv[NG];
  row_spread_groups<NG>(z, sf == 0.0f ? 0.0f : __fdiv_rn(1.0f, sf), zero, inv);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int g = (64 * ((k >> 1) & 1) + 32 * (k >> 2)) / G;
    uint32_t w = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {                         // clamp, then round in the convert
      const float c = fminf(fmaxf(fmaf(u[4 * k + e], 0.0625f, -zero[g]) * inv[g], 0.0f), float(L - 1));
      w = __builtin_amdgcn_cvt_pk_u8_f32(c, e, w);
    }
    code[k] = w;
  }
  return uint32_t(s16) | (uint32_t(z16) << 16);
}

// The row and the quarter of it that a thread of the workgroup holds while
// quantizing: neighbouring lanes for the unrotated base, lanes 16 apart for
// the rotating ones.
template <int BASE>
__device__ inline int row_of_thread(int tid) { return BASE == 0 ? tid >> 2 : (tid >> 6) * 16 + (tid & 15); }
template <int BASE>
__device__ inline int quarter_of_thread(int tid) { return BASE == 0 ? tid & 3 : (tid >> 4) & 3; }

// Quantize a row's K or V: every thread of the row writes its codes to the
// row of the code array (zeros for a row that is not there) and the metadata
// of its share of the groups.  m: the rotating bases' sign masks.  bad: a value
// was not finite.  GC: the rotated affine base's group size, 0 to read it from g.
// Returns the tq base's norm (fp16 bits).
template <int BASE, int L, int GC>
__device__ uint16_t quantize_row(const PoolGeom& g, const uint16_t* src, bool valid, int q, const uint32_t m[16],
                             const float* tau, uint8_t* codes, uint8_t* meta_dst, int slot, bool& bad) {
  if constexpr (BASE == 0) {
    uint32_t d[16], code[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint4 p = valid ? reinterpret_cast<const uint4*>(src)[k] : make_uint4(0u, 0u, 0u, 0u);
      d[4 * k] = p.x, d[4 * k + 1] = p.y, d[4 * k + 2] = p.z, d[4 * k + 3] = p.w;
    }
    const uint32_t w = affine_quarter<L>(d, g.G, code, bad);
    const int per = g.G / 32;
    if (q % per == 0) reinterpret_cast<uint32_t*>(meta_dst)[(q / per) * kSlots + slot] = valid ? w : 0u;
    uint32_t* dst = reinterpret_cast<uint32_t*>(codes + 32 * q);
#pragma unroll
    for (int i = 0; i < 8; ++i) dst[i] = valid ? code[i] : 0u;
    return 0;
  } else {
    float u[32];
    uint32_t code[8];
    uint16_t r = 0;
    load_signed(src, valid, m, u);
    if constexpr (BASE == 1) {
      r = tq_row<L>(u, tau, code);
      if (q == 0) reinterpret_cast<uint16_t*>(meta_dst)[slot] = valid ? r : uint16_t(0);
    } else {
      rotate_row(u);
      auto affine = [&](auto GI) {
        constexpr int G = decltype(GI)::value;
        const uint32_t w = rot_affine_row<L, G>(u, code);
        if (q < 128 / G) reinterpret_cast<uint32_t*>(meta_dst)[q * kSlots + slot] = valid ? w : 0u;
      };
      if constexpr (GC != 0) affine(std::integral_constant<int, GC>{});
      else if (g.G == 128) affine(std::integral_constant<int, 128>{});
      else if (g.G == 64) affine(std::integral_constant<int, 64>{});
      else affine(std::integral_constant<int, 32>{});
    }
    // an infinity or a NaN of the row reaches every rotated coordinate, and
    // finite rows stay finite (128 * 65504)
    bad |= (__float_as_uint(u[0]) & 0x7F800000u) == 0x7F800000u;
    uint32_t* dst = reinterpret_cast<uint32_t*>(codes + rot_channel(int(threadIdx.x) & 63));
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int q0 = k >> 2, q1 = (k >> 1) & 1;
      dst[(64 * q1 + 32 * q0) / 4 + (k & 1)] = valid ? code[k] : 0u;
    }
    return r;
  }
}

// K's and V's row quarters of a tq row.  A norm that is a NaN is stored with the
// row's own sign rather than the sign mask's: the row is read again where it is
// reported as not finite, which brings all four of its lanes there, so nothing
// is held in registers, and no branch is taken, for other rows.
template <int L>
__device__ inline void quantize_tq_rows(const PoolGeom& g, const uint16_t* k, const uint16_t* v, bool valid, int q, const uint32_t m[16],
                                        const float* tau, uint8_t* ck, uint8_t* cv, uint8_t* meta, int slot) {
  const uint16_t* const src[2] = {k, v};
  uint16_t norm[2];
  bool bad = false;
#pragma unroll
  for (int kv = 0; kv < 2; ++kv)
    norm[kv] = quantize_row<1, L, 0>(g, src[kv], valid, q, m, tau, kv ? cv : ck, meta + kv * g.meta_bytes, slot, bad);
  if (!(bad && valid)) return;
  atomicOr(g.status, 2);
  for (int kv = 0; kv < 2; ++kv) {
    if ((norm[kv] & 0x7FFFu) <= 0x7C00u) continue;
    const uint32_t plain[16] = {};
    float x[32];
    load_signed(src[kv], true, plain, x);
    const uint16_t r = sqrt_f16(row_square_sum(x));
    if (q == 0) reinterpret_cast<uint16_t*>(meta + kv * g.meta_bytes)[slot] = r;
  }
}

// Symbol of ND codes of base L at bytes O.. of a row of codes: dword reads and
// four digits per dot product (L^3 fits a byte up to 6 levels; 7 levels take
// the digits one by one).  Codes past ND meet zero weights.  With a byte read
// and a multiply-add per code of K instead, and the affine range one fp32 value
// at a time with a finiteness check of its own, ranking and quantizing 32768
// tokens of 32 layers took 961 us instead of 936, and 131072 tokens of 8
// layers on the tq base 1278 instead of 1257.
template <int L, int O, int ND>
__device__ __forceinline__ uint32_t row_symbol(const uint32_t* row) {
  constexpr int sh = O & 3, n1 = (sh + ND + 3) / 4;                    // dwords the codes span
  const uint32_t d0 = row[O / 4], d1 = n1 > 1 ? row[O / 4 + 1] : 0u, d2 = n1 > 2 ? row[O / 4 + 2] : 0u;
  const uint32_t c03 = sh ? __builtin_amdgcn_alignbyte(d1, d0, sh) : d0;
  constexpr uint32_t w03 = 1u | (ND > 1 ? uint32_t(L) << 8 : 0u) | (ND > 2 ? uint32_t(L * L) << 16 : 0u) |
                           (ND > 3 ? uint32_t(L * L * L) << 24 : 0u);
  uint32_t v = __builtin_amdgcn_udot4(c03, w03, 0u, false);
  if constexpr (ND > 4) {
    const uint32_t c47 = sh ? __builtin_amdgcn_alignbyte(d2, d1, sh) : d1;
    constexpr uint32_t L4 = uint32_t(L) * L * L * L;
    if constexpr (L4 < 256u) {               // 2 and 3 levels
      constexpr uint32_t w47 = L4 | (ND > 5 ? L4 * L << 8 : 0u) | (ND > 6 ? L4 * L * L << 16 : 0u) | (ND > 7 ? L4 * L * L * L << 24 : 0u);
      v = __builtin_amdgcn_udot4(c47, w47, v, false);
    } else {                                 // 6 levels: one more code
      v += __umul24(c47 & 255u, L4);
    }
  }
  return v;
}

// OR the bits of one segment into an LDS body.  The segment holds symbols
// p = j, j+4, ... of a line of NV codes: code p*n+i of the line is at
// codes[(p*n+i)*stride].  J is compile-time: the symbols' widths and bit
// positions are constants, the line's offset is applied by one funnel shift
// per word.  ROW: the line is a row of codes (stride 1, 4-byte aligned).
template <int L, int NV, int NL, bool ROW, int J, int K = 0>
__device__ __forceinline__ void row_symbols(const uint32_t* row, uint32_t (&v)[16]) {
  constexpr SegTable<L, NV, NL> t{};
  if constexpr (K < 16) {
    if constexpr (t.width[J][K] > 0) v[K] = row_symbol<L, sym_digits(L) * (J + 4 * K), t.ndig[J][K]>(row);
    row_symbols<L, NV, NL, ROW, J, K + 1>(row, v);
  }
}
template <int L, int NV, int NL, bool ROW, int J>
__device__ __forceinline__ void pack_segment_j(const uint8_t* codes, int stride, int line, uint32_t* body) {
  constexpr int n = sym_digits(L);
  constexpr SegTable<L, NV, NL> t{};
  constexpr int BITS = t.bits[J];
  constexpr int NWD = (BITS + 31) / 32 + 1;             // words, one spare for the shift
  uint32_t w[NWD];
#pragma unroll
  for (int k = 0; k < NWD; ++k) w[k] = 0u;
  int nb = 0;
  constexpr bool DOT = ROW && L != 7;
  uint32_t sym[16];
  if constexpr (DOT) row_symbols<L, NV, NL, ROW, J>(reinterpret_cast<const uint32_t*>(codes), sym);
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int wd = t.width[J][k], nd = t.ndig[J][k];
    if (wd > 0) {
      const int p = J + 4 * k;
      uint32_t v = 0;
      if constexpr (DOT) {
        v = sym[k];
      } else {
#pragma unroll
        for (int i = n - 1; i >= 0; --i)
          if (i < nd) v = v * L + codes[(n * p + i) * stride];
      }
      w[nb >> 5] |= v << (nb & 31);
      if ((nb & 31) + wd > 32) w[(nb >> 5) + 1] |= v >> (32 - (nb & 31));
      nb += wd;
    }
  }
  const int off = t.start[J] + line * BITS;
  const int w0 = off >> 5, sh = off & 31;
#pragma unroll
  for (int k = 0; k < NWD; ++k) {
    const uint32_t lo = k ? w[k - 1] : 0u;
    const uint32_t o = sh ? __builtin_amdgcn_alignbit(w[k], lo, 32 - sh) : w[k];
    if (32 * k < sh + BITS && o) atomicOr(&body[w0 + k], o);
  }
}

template <int L, int NV, int NL, bool ROW>
__device__ __forceinline__ void pack_segment(const uint8_t* codes, int stride, int line, int j, uint32_t* body) {
  switch (j) {                                          // j is the same for a whole wave
    case 0: pack_segment_j<L, NV, NL, ROW, 0>(codes, stride, line, body); break;
    case 1: pack_segment_j<L, NV, NL, ROW, 1>(codes, stride, line, body); break;
    case 2: pack_segment_j<L, NV, NL, ROW, 2>(codes, stride, line, body); break;
    default: pack_segment_j<L, NV, NL, ROW, 3>(codes, stride, line, body); break;
  }
}

// Decode one segment of an LDS body back into codes (used to extend a
// partially filled record when a generation block closes).
template <int L, int NV, int NL>
__device__ void unpack_segment(const uint32_t* body, int line, int j, uint8_t* codes, int stride) {
  constexpr int n = sym_digits(L);
  constexpr int S = num_syms(L, NV);
  constexpr SegTable<L, NV, NL> t{};
  int off = pick4(j, t.start[0], t.start[1], t.start[2], t.start[3]) +
            line * pick4(j, t.bits[0], t.bits[1], t.bits[2], t.bits[3]);
#pragma unroll
  for (int k = 0; 4 * k < S; ++k) {
    const int p = j + 4 * k;
    const int w = pick4(j, t.width[0][k], t.width[1][k], t.width[2][k], t.width[3][k]);
    const int nd = pick4(j, t.ndig[0][k], t.ndig[1][k], t.ndig[2][k], t.ndig[3][k]);
    if (w > 0) {
      int wd = off >> 5, sh = off & 31;
      uint64_t pair = uint64_t(body[wd]) | (uint64_t(body[wd + 1]) << 32);
      uint32_t v = uint32_t(pair >> sh) & ((1u << w) - 1u);
#pragma unroll
      for (int i = 0; i < n; ++i)
        if (i < nd) {
          codes[(n * p + i) * stride] = uint8_t(v % L);
          v /= L;
        }
      off += w;
    }
  }
}

template <int L>
__device__ __forceinline__ void pack_record(const uint8_t* ck, const uint8_t* cv, uint32_t* bk, uint32_t* bv) {
  int tid = threadIdx.x;
  pack_segment<L, kD, kSlots, true>(ck + (tid & 63) * kPitch, 1, tid & 63, tid >> 6, bk);
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    int s = tid + 256 * e;
    pack_segment<L, kSlots, kD, false>(cv + (s & 127), kPitch, s & 127, s >> 7, bv);
  }
}

__device__ void store_bodies(uint8_t* rec, const uint32_t* bk, const uint32_t* bv, int tb) {
  const uint4* sk = reinterpret_cast<const uint4*>(bk);
  const uint4* sv = reinterpret_cast<const uint4*>(bv);
  uint4* dk = reinterpret_cast<uint4*>(rec);
  uint4* dv = reinterpret_cast<uint4*>(rec + tb);
  for (int i = threadIdx.x; i < tb / 16; i += 256) {
    dk[i] = sk[i];
    dv[i] = sv[i];
  }
}

struct Lds {
  alignas(16) uint8_t ck[kSlots * kPitch];
  alignas(16) uint8_t cv[kSlots * kPitch];
  alignas(16) uint32_t bk[kMaxBodyWords + 8];
  alignas(16) uint32_t bv[kMaxBodyWords + 8];
};

template <int BASE, int L, int GC>
__device__ void prefill_record(const QuantArgs& a, Lds& s, int pool, int tile, int b, int l, int h) {
  const PoolGeom& g = a.g;
  const int tid = threadIdx.x, r = row_of_thread<BASE>(tid), q = quarter_of_thread<BASE>(tid);
  int64_t slot = int64_t(tile) * kSlots + r;
  bool valid = slot < a.n_pool[pool];
  int tok = valid ? a.idx[pool][int64_t(b) * a.n_pool[pool] + slot] : 0;
  uint32_t m[16];
  if constexpr (BASE != 0) sign_masks(g.signs[(int64_t(l) * g.n_kv_heads + h) * 4 + q], m);
  if (tok < 0 || tok >= a.T) {             // a slot list not produced by semkv_rank
    if (valid) atomicOr(g.status, 4);
    tok = 0;
  }
  constexpr int tb = tile_bytes(L);
  uint8_t* rec = g.pools + unit_offset(g, b, l, h) + (pool ? g.lo_offset : 0) + int64_t(tile) * g.rec_bytes[pool];
  for (int i = tid; i < kMaxBodyWords + 8; i += 256) s.bk[i] = s.bv[i] = 0u;
  bool bad = false;
  const int64_t base_off = int64_t(l) * a.sL + int64_t(b) * a.sB + int64_t(h) * a.sH + int64_t(tok) * a.sT + 32 * q;
  if constexpr (BASE == 1) {
    quantize_tq_rows<L>(g, a.K + base_off, a.V + base_off, valid, q, m, g.tau[pool], s.ck + r * kPitch, s.cv + r * kPitch, rec + 2 * tb, r);
  } else {
#pragma unroll
    for (int kv = 0; kv < 2; ++kv)
      quantize_row<BASE, L, GC>(g, (kv ? a.V : a.K) + base_off, valid, q, m, g.tau[pool], (kv ? s.cv : s.ck) + r * kPitch,
                                rec + 2 * tb + kv * g.meta_bytes, r, bad);
  }
  if (bad && valid) atomicOr(g.status, 2);
  __syncthreads();
  pack_record<L>(s.ck, s.cv, s.bk, s.bv);
  __syncthreads();
  store_bodies(rec, s.bk, s.bv, tb);
}

// The rotated affine base has a kernel per group size (GC): with the size read
// at run time, the branches on it kept V's loads behind K's work, and 3 x 5003
// tokens of a layer at 6/5 levels and G = 128 took 23.4 us instead of 22.2.
template <int BASE, int LH, int LL, int GC>
__global__ __launch_bounds__(256) void quantize_pack_kernel(QuantArgs a) {
  __shared__ Lds s;
  int tile = blockIdx.x, pool = blockIdx.y & 1, h = blockIdx.y >> 1;
  int b = blockIdx.z / a.n_layers_launched, l = a.layer0 + blockIdx.z % a.n_layers_launched;
  if (int64_t(tile) * kSlots >= a.n_pool[pool]) return;
  if (pool == 0) prefill_record<BASE, LH, GC>(a, s, 0, tile, b, l, h);
  else prefill_record<BASE, LL, GC>(a, s, 1, tile, b, l, h);
}

// ---------------------------------------------------------------- close --

template <int BASE, int L>
__device__ void close_record(const CloseArgs& a, Lds& s, const int* row_of, int m, int pool,
                             int tile, int b, int l, int h) {
  const PoolGeom& g = a.g;
  const int tid = threadIdx.x, r = row_of_thread<BASE>(tid), q = quarter_of_thread<BASE>(tid);
  constexpr int tb = tile_bytes(L);
  uint8_t* rec = g.pools + unit_offset(g, b, l, h) + (pool ? g.lo_offset : 0) + int64_t(tile) * g.rec_bytes[pool];
  int64_t first = int64_t(tile) * kSlots;
  int64_t n0 = a.n0[pool];
  // existing rows of this record are unpacked; the rest start at code 0
  for (int i = tid; i < kMaxBodyWords + 8; i += 256) s.bk[i] = s.bv[i] = 0u;
  __syncthreads();
  if (first < n0) {
    const uint32_t* gk = reinterpret_cast<const uint32_t*>(rec);
    const uint32_t* gv = reinterpret_cast<const uint32_t*>(rec + tb);
    for (int i = tid; i < tb / 4; i += 256) {
      s.bk[i] = gk[i];
      s.bv[i] = gv[i];
    }
  }
  __syncthreads();
  unpack_segment<L, kD, kSlots>(s.bk, tid & 63, tid >> 6, s.ck + (tid & 63) * kPitch, 1);
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    int sg = tid + 256 * e;
    unpack_segment<L, kSlots, kD>(s.bv, sg & 127, sg >> 7, s.cv + (sg & 127), kPitch);
  }
  __syncthreads();
  int64_t slot = first + r;
  bool fresh = slot >= n0;                 // slots written by this close
  bool valid = fresh && slot < n0 + m;
  int row = valid ? row_of[slot - n0] : 0;
  bool bad = false;
  if (fresh) {
    const uint16_t* src = a.tail + ((((int64_t(b) * g.n_layers + l) * g.n_kv_heads + h) * 2) * kSlots + row) * kD + 32 * q;
    uint32_t m[16];
    if constexpr (BASE != 0) sign_masks(g.signs[(int64_t(l) * g.n_kv_heads + h) * 4 + q], m);
    if constexpr (BASE == 1) {
      quantize_tq_rows<L>(g, src, src + kSlots * kD, valid, q, m, g.tau[pool], s.ck + r * kPitch, s.cv + r * kPitch, rec + 2 * tb, r);
    } else {
#pragma unroll
      for (int kv = 0; kv < 2; ++kv)
        quantize_row<BASE, L, 0>(g, src + kv * kSlots * kD, valid, q, m, g.tau[pool], (kv ? s.cv : s.ck) + r * kPitch,
                                 rec + 2 * tb + kv * g.meta_bytes, r, bad);
    }
  }
  if (bad && valid) atomicOr(g.status, 2);
  __syncthreads();
  for (int i = tid; i < kMaxBodyWords + 8; i += 256) s.bk[i] = s.bv[i] = 0u;
  __syncthreads();
  pack_record<L>(s.ck, s.cv, s.bk, s.bv);
  __syncthreads();
  store_bodies(rec, s.bk, s.bv, tb);
}

template <int BASE, int LH, int LL>
__global__ __launch_bounds__(256) void close_kernel(CloseArgs a) {
  __shared__ Lds s;
  __shared__ float sc[kSlots];
  __shared__ int cls[kSlots], row_of[2][kSlots];
  int tid = threadIdx.x;
  int pool = blockIdx.y & 1, h = blockIdx.y >> 1;
  int b = blockIdx.z / a.g.n_layers, l = blockIdx.z % a.g.n_layers;
  if (tid < a.n) {
    float v = a.tail_scores[int64_t(b) * kSlots + tid];
    sc[tid] = v == 0.0f ? 0.0f : v;
    if (isnan(v)) atomicOr(a.g.status, 1);
  }
  __syncthreads();
  if (tid < a.n) {                         // rank inside the block (Alg. 2)
    float v = sc[tid];
    int rank = 0;
    for (int j = 0; j < a.n; ++j) rank += (sc[j] > v || (sc[j] == v && j < tid)) ? 1 : 0;
    cls[tid] = rank < a.k_hi ? 0 : 1;
  }
  __syncthreads();
  if (tid < a.n) {
    int c = cls[tid], pos = 0;
    for (int j = 0; j < tid; ++j) pos += cls[j] == c ? 1 : 0;
    row_of[c][pos] = tid;
    if (c == 0 && pool == 0 && h == 0 && l == 0 && blockIdx.x == 0) {
      int64_t t = a.pos0 + tid;
      atomicOr(&a.flags[int64_t(b) * a.flag_words + (t >> 5)], 1u << (t & 31));
    }
  }
  __syncthreads();
  int m = pool == 0 ? a.k_hi : a.n - a.k_hi;
  int64_t n0 = a.n0[pool];
  int64_t tile = n0 / kSlots + blockIdx.x;
  if (m == 0 || tile > (n0 + m - 1) / kSlots) return;
  if (pool == 0) close_record<BASE, LH>(a, s, row_of[0], m, 0, int(tile), b, l, h);
  else close_record<BASE, LL>(a, s, row_of[1], m, 1, int(tile), b, l, h);
}

// ------------------------------------------------------------ dequant --

// The values one record holds, as decode attention sees them: affine
// x = fmaf(c, scale, zero); rotated affine x = sign . H y / 8 with y the
// affine value; tq x = sign . H (rho mu[c]) / 128.  One workgroup per record:
// the bodies are unpacked into LDS as for a block close, four lanes per slot.
template <int BASE, int L>
__device__ void dequant_record(const DequantArgs& a, Lds& s, int pool, int tile, int b, int h) {
  const PoolGeom& g = a.g;
  const int tid = threadIdx.x, r = tid >> 2, q = tid & 3;
  constexpr int tb = tile_bytes(L);
  const uint8_t* rec = g.pools + unit_offset(g, b, a.layer, h) + (pool ? g.lo_offset : 0) +
                       int64_t(tile) * g.rec_bytes[pool];
  for (int i = tid; i < kMaxBodyWords + 8; i += 256) s.bk[i] = s.bv[i] = 0u;
  __syncthreads();
  const uint32_t* gk = reinterpret_cast<const uint32_t*>(rec);
  const uint32_t* gv = reinterpret_cast<const uint32_t*>(rec + tb);
  for (int i = tid; i < tb / 4; i += 256) {
    s.bk[i] = gk[i];
    s.bv[i] = gv[i];
  }
  __syncthreads();
  unpack_segment<L, kD, kSlots>(s.bk, tid & 63, tid >> 6, s.ck + (tid & 63) * kPitch, 1);
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int sg = tid + 256 * e;
    unpack_segment<L, kSlots, kD>(s.bv, sg & 127, sg >> 7, s.cv + (sg & 127), kPitch);
  }
  __syncthreads();
  const int64_t slot = int64_t(tile) * kSlots + r;
  const bool valid = slot < a.n_rows[pool];
  const int64_t N = a.n_rows[0] + a.n_rows[1];
  const int64_t row = (pool ? a.n_rows[0] : 0) + slot;
  const uint32_t sbits = BASE != 0 ? g.signs[(int64_t(a.layer) * g.n_kv_heads + h) * 4 + q] : 0u;
#pragma unroll
  for (int kv = 0; kv < 2; ++kv) {
    const uint8_t* c = (kv ? s.cv : s.ck) + r * kPitch + 32 * q;
    const uint8_t* meta = rec + 2 * tb + kv * g.meta_bytes;
    float x[32];
    if (BASE != 1) {
      const uint32_t m = reinterpret_cast<const uint32_t*>(meta)[((32 * q) / g.G) * kSlots + r];
      const float sc = h2f(uint16_t(m & 0xFFFFu)), z = h2f(uint16_t(m >> 16));
#pragma unroll
      for (int i = 0; i < 32; ++i) x[i] = fmaf(float(c[i]), sc, z);
    } else {
      const float rho = h2f(reinterpret_cast<const uint16_t*>(meta)[r]);
      const float* mu = a.mu[pool];
#pragma unroll
      for (int i = 0; i < 32; ++i) x[i] = rho * mu[c[i] < L ? c[i] : 0];
    }
    if (BASE != 0) {                       // sign . H x, scaled back
      float u[32];
      rotate_quarter(x, q, 0u, u);
      const float k = BASE == 2 ? 0.125f : 1.0f / 128.0f;
#pragma unroll
      for (int i = 0; i < 32; ++i) x[i] = ((sbits >> i) & 1u) ? -u[i] * k : u[i] * k;
    }
    float* dst = (kv ? a.v_hat : a.k_hat) + ((int64_t(b) * g.n_kv_heads + h) * N + row) * kD + 32 * q;
    if (valid) {
#pragma unroll
      for (int i = 0; i < 32; i += 4) *reinterpret_cast<float4*>(dst + i) = make_float4(x[i], x[i + 1], x[i + 2], x[i + 3]);
    }
  }
}

template <int BASE, int LH, int LL>
__global__ __launch_bounds__(256) void dequant_kernel(DequantArgs a) {
  __shared__ Lds s;
  const int tile = blockIdx.x, pool = blockIdx.y & 1, h = blockIdx.y >> 1, b = blockIdx.z;
  if (int64_t(tile) * kSlots >= a.n_rows[pool]) return;
  if (pool == 0) dequant_record<BASE, LH>(a, s, 0, tile, b, h);
  else dequant_record<BASE, LL>(a, s, 1, tile, b, h);
}

__global__ void append_kernel(AppendArgs a) {
  // one block per (layer, b, kv head); 64 threads copy K and V rows
  int z = blockIdx.x;
  int h = z % a.n_kv_heads;
  int b = (z / a.n_kv_heads) % a.batch;
  int li = z / (a.n_kv_heads * a.batch);
  int l = a.layer0 + li;
  const uint32_t* k = reinterpret_cast<const uint32_t*>(a.k + ((int64_t(li) * a.batch + b) * a.n_kv_heads + h) * kD);
  const uint32_t* v = reinterpret_cast<const uint32_t*>(a.v + ((int64_t(li) * a.batch + b) * a.n_kv_heads + h) * kD);
  uint32_t* dst = reinterpret_cast<uint32_t*>(a.tail + ((((int64_t(b) * a.n_layers + l) * a.n_kv_heads + h) * 2) * kSlots + a.slot) * kD);
  int t = threadIdx.x;
  dst[t] = k[t];
  dst[kSlots * kD / 2 + t] = v[t];
}

template <int BASE, int LH, int LL>
int launch_qp(const QuantArgs& a, hipStream_t st) {
  dim3 grid(a.max_tiles, 2 * a.g.n_kv_heads, a.g.batch * a.n_layers_launched);
  if constexpr (BASE != 2) {
    hipLaunchKernelGGL((quantize_pack_kernel<BASE, LH, LL, 0>), grid, dim3(256), 0, st, a);
  } else {
    // metadata finer than a row only at 6/5 and 5/4 levels
    constexpr bool FINE = LH == LL + 1 && (LL == 5 || LL == 4);
    if (a.g.G == 128) hipLaunchKernelGGL((quantize_pack_kernel<BASE, LH, LL, 128>), grid, dim3(256), 0, st, a);
    else if (FINE && a.g.G == 64) hipLaunchKernelGGL((quantize_pack_kernel<BASE, LH, LL, FINE ? 64 : 128>), grid, dim3(256), 0, st, a);
    else if (FINE && a.g.G == 32) hipLaunchKernelGGL((quantize_pack_kernel<BASE, LH, LL, FINE ? 32 : 128>), grid, dim3(256), 0, st, a);
    else return -2;
  }
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

template <int BASE, int LH, int LL>
int launch_dq(const DequantArgs& a, hipStream_t st) {
  const int64_t mt = ((a.n_rows[0] > a.n_rows[1] ? a.n_rows[0] : a.n_rows[1]) + kSlots - 1) / kSlots;
  dim3 grid(unsigned(mt), 2 * a.g.n_kv_heads, a.g.batch);
  hipLaunchKernelGGL((dequant_kernel<BASE, LH, LL>), grid, dim3(256), 0, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

template <int BASE, int LH, int LL>
int launch_cl(const CloseArgs& a, hipStream_t st) {
  dim3 grid(2, 2 * a.g.n_kv_heads, a.g.batch * a.g.n_layers);
  hipLaunchKernelGGL((close_kernel<BASE, LH, LL>), grid, dim3(256), 0, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

}  // namespace

#define SEMKV_DISPATCH_LEVELS(BASE, LH, LL, FN, ...)                                  \
  if (BASE == 0 && LH == 6 && LL == 5) return FN<0, 6, 5>(__VA_ARGS__);              \
  if (BASE == 0 && LH == 5 && LL == 4) return FN<0, 5, 4>(__VA_ARGS__);              \
  if (BASE == 0 && LH == 6 && LL == 4) return FN<0, 6, 4>(__VA_ARGS__);              \
  if (BASE == 0 && LH == 4 && LL == 3) return FN<0, 4, 3>(__VA_ARGS__);              \
  if (BASE == 0 && LH == 5 && LL == 3) return FN<0, 5, 3>(__VA_ARGS__);              \
  if (BASE == 0 && LH == 6 && LL == 3) return FN<0, 6, 3>(__VA_ARGS__);              \
  if (BASE == 1 && LH == 4 && LL == 3) return FN<1, 4, 3>(__VA_ARGS__);              \
  if (BASE == 2 && LH == 6 && LL == 5) return FN<2, 6, 5>(__VA_ARGS__);              \
  if (BASE == 2 && LH == 5 && LL == 4) return FN<2, 5, 4>(__VA_ARGS__);              \
  if (BASE == 0 && LH == 8 && LL == 7) return FN<0, 8, 7>(__VA_ARGS__);              \
  if (BASE == 0 && LH == 7 && LL == 6) return FN<0, 7, 6>(__VA_ARGS__);              \
  if (BASE == 0 && LH == 3 && LL == 2) return FN<0, 3, 2>(__VA_ARGS__);              \
  if (BASE == 2 && LH == 8 && LL == 7) return FN<2, 8, 7>(__VA_ARGS__);              \
  if (BASE == 2 && LH == 7 && LL == 6) return FN<2, 7, 6>(__VA_ARGS__);              \
  if (BASE == 2 && LH == 3 && LL == 2) return FN<2, 3, 2>(__VA_ARGS__);              \
  return -2;

int launch_quantize(const QuantArgs& a, hipStream_t s) {
  SEMKV_DISPATCH_LEVELS(a.g.base, a.g.L[0], a.g.L[1], launch_qp, a, s)
}

int launch_close(const CloseArgs& a, hipStream_t s) {
  SEMKV_DISPATCH_LEVELS(a.g.base, a.g.L[0], a.g.L[1], launch_cl, a, s)
}

int launch_dequant(const DequantArgs& a, hipStream_t s) {
  SEMKV_DISPATCH_LEVELS(a.g.base, a.g.L[0], a.g.L[1], launch_dq, a, s)
}

int launch_append(const AppendArgs& a, hipStream_t s) {
  dim3 grid(a.n_layers_launched * a.batch * a.n_kv_heads);
  hipLaunchKernelGGL(append_kernel, grid, dim3(64), 0, s, a);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

}  // namespace semkv
