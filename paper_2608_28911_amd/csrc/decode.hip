// decode.hip -- split-K GQA decode attention over the mixed-precision cache
// (the decoding consumer of SemKV, Sec. 3.1 and Alg. 1), for gfx950.
//
// Work split: a (sequence, kv head) unit's tiles -- its high pool, then its
// low pool -- are dealt to nsplit workgroups of NW waves (nsplit chosen by the
// host so that the whole grid is resident at once): tile u goes to wave slot
// u mod (nsplit NW), slot v = w nsplit + s being wave w of workgroup s.  Every
// wave thus gets an even share of the (costlier) high-precision tiles, first
// in its sequence, and keeps its own online-softmax state for the 4 query
// heads of the kv head.  Each lane loads the segments it decodes from memory
// straight into its registers, a record ahead; only a record's metadata goes
// through LDS.  (With whole records staged in LDS the staging writes, the
// unaligned segment reads and their bank conflicts were a third of the LDS
// cycles, 518 a record at batch 16, and LDS was active 61 % of the time; now
// 301 and 42 %.  A segment's registers are loaded again as soon as it is
// decoded, which keeps a wave's loads spread over its record: all at the
// record's top, batch 1 at 32768 tokens took 13.8 us a launch instead of 13.2
// and tq at 131072 25.1 instead of 24.0.  The staged form against this one, in
// a graph on one box, us a launch: batch 16 at 16384 tokens 46.5 -> 40.9, batch
// 4 at 32768 with a tail 30.5 -> 27.1, tq at 131072 25.5 -> 23.3, batch 1 at
// 32768 14.0 -> 12.7, 2048 tokens 10.1 -> 9.9.  The prologue is longer for it,
// 3.0 us instead of 2.4 until the operands are ready (tq 3.4 instead of 3.0),
// but no wait for the first record follows, which ends at 5.5 instead of 6.3.
// What is left is mostly the launch's fixed part -- 2.6 us to launch, 3.0 of
// prologue, 4 of merge -- and memory: at batch 16 the records stream at about
// 5.6 TB/s.)
// Products run on the int8 matrix cores
// (v_mfma_i32_16x16x64_i8), exact in their integer sums.  Per record:
//   scores  C[16 rows (head, byte) x 16 tokens] += A B: A holds the query of
//           head h as a fixed-point integer qi = rint(q 2^e) (|qi| < 2^20, e
//           per head and metadata group) split into three bytes, one per row,
//           restricted to one metadata group; B the base-L digits of 16
//           tokens as bytes, decoded from the packed K symbols through LDS
//           tables (one dword of digit bytes per entry).  The affine
//           dequantization x = s c + z is folded out:
//           q.x = s (q.c) + z (sum q) per group.
//   softmax online, base 2; unnormalized p, rescaled when the maximum moves.
//   values  C[16 rows (head, byte) x 16 channels] += A[16 x 64 tokens]
//           B[64 tokens x 16 channels] with A the weights p * s as 21-bit
//           integers (one power-of-2 scale per head, three bytes in three
//           rows) and B the V digits (V symbols run along tokens).  The
//           integer sums run across records and are folded into float sums
//           only when the running maximum moves or a record's weights would
//           not fit the scale.
// The last run also takes the fp16 tail of generated tokens.  The waves'
// states merge in LDS into one partial per workgroup; the last workgroup of a
// unit to finish merges the partials (log-sum-exp) and, for the rotated bases
// (TurboQuant-MSE, and the affine base under its Hadamard rotation), applies
// the inverse random-sign Hadamard rotation.
// Bases: 0 affine, 1 TurboQuant-MSE, 2 affine of the rotated row.  Bases 0
// and 2 share the affine levels and metadata; bases 1 and 2 score against the
// rotated query H diag(sign) q and accumulate values in the rotated domain.
#include <hip/hip_fp16.h>

#include <stddef.h>

#include <type_traits>

#include "semkv_internal.h"

namespace semkv {

// ---- tracing build only (-DSEMKV_TIMELINE, libsemkv_timeline.so): lane 0 of
// every wave of the first kTimelineWGs workgroups of a launch records the
// constant 100 MHz clock at the ends of the kernel's phases (event ids below);
// a later launch overwrites the stamps.  The product library compiles every
// stamp to nothing.
#ifdef SEMKV_TIMELINE
constexpr int kTimelineWGs = 4096, kTimelineWaves = 16, kTimelineEvents = 32;
__device__ unsigned long long g_timeline[kTimelineWGs * kTimelineWaves * kTimelineEvents];
__device__ inline void timeline_stamp(int ev) {
  const int wg = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  if ((threadIdx.x & 63) == 0 && wg < kTimelineWGs)
    g_timeline[(wg * kTimelineWaves + (threadIdx.x >> 6)) * kTimelineEvents + ev] = wall_clock64();
}
// slots 14 and 15 of a wave hold counts, kept in the wave's state and
// written once (a read-modify-write of memory in the record loop would wait
// for the loads in flight)
__device__ inline void timeline_put(int ev, unsigned long long v) {
  const int wg = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  if ((threadIdx.x & 63) == 0 && wg < kTimelineWGs)
    g_timeline[(wg * kTimelineWaves + (threadIdx.x >> 6)) * kTimelineEvents + ev] = v;
}
#define SEMKV_STAMP(ev) timeline_stamp(ev)
#else
#define SEMKV_STAMP(ev) ((void)0)
#endif
// the stamps inside the prologue and the first record (16..21) delay what they
// measure: compiled in only with -DSEMKV_TIMELINE_FINE as well
#if defined(SEMKV_TIMELINE) && defined(SEMKV_TIMELINE_FINE)
#define SEMKV_STAMP_FINE(ev) SEMKV_STAMP(ev)
#else
#define SEMKV_STAMP_FINE(ev) ((void)0)
#endif
// 0 start, 1 tables and query operands built, 2 the wave's state set up,
// 3..7 the wave's 1st..5th record done (a 6th and later overwrite 7), 8 the
// first record's arithmetic done, 16..18 inside the first record: its metadata
// in LDS, scores done, softmax and flush done, 19..21 in
// the prologue: tables written, query value in hand, query runs done,
// 9 the wave's records done, 10 workgroup partial merged, 11 partial stored,
// 12 split counter taken, 13 the last workgroup's merge done; counts: 14 the
// wave's value-sum flushes, 15 its records (both cleared at the wave's start)

namespace {

typedef int32_t int4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kRsqrtD = 0.08838834764831845f;   // 1 / sqrt(128)

// f(0), ..., f(N-1) with compile-time indices
template <int N, class F, int I = 0>
__device__ __forceinline__ void static_for(F f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, F, I + 1>(f);
  }
}

// ------------------------------------------------------------ traits ----

__host__ __device__ constexpr int ipow(int b, int e) {
  int r = 1;
  for (int i = 0; i < e; ++i) r *= b;
  return r;
}

__host__ __device__ constexpr int gcd_of(int a, int b) { return b == 0 ? a : gcd_of(b, a % b); }

// Chunk layout: an MFMA operand gives each lane 16 byte slots; a chunk fills
// them with SPC symbols of STRIDE slots each; slot_digit / slot_plane give the
// code a slot holds (-1: a zero pad slot).  4-level codes of the tq base take
// two slots, their low and high bit (the Lloyd-Max levels are affine in those
// bits).
template <int BASE, int L>
struct Traits {
  static constexpr int n = sym_digits(L);
  static constexpr int P = (BASE == 1 && L == 4) ? 2 : 1;   // MFMA slots per code
  static constexpr int STRIDE = (L == 5 || L == 8 || (L == 4 && BASE != 1)) ? 4 : 8;
  static constexpr int SPC = 16 / STRIDE;
  static constexpr int EDW = STRIDE / 4;                     // operand dwords per symbol
  static constexpr int SK = num_syms(L, kD), SV = num_syms(L, kSlots);
  static constexpr int NSK = (SK + 3) / 4, NSV = (SV + 3) / 4;
  static constexpr int NCK = (NSK + SPC - 1) / SPC, NCV = (NSV + SPC - 1) / SPC;
  static constexpr int W = width_of(L, n);
  static constexpr int TB = tile_bytes(L);
  static constexpr int KSEGW = (NSK * W + 31) / 32;          // normalized dwords of a K segment
  static constexpr int VSEGW = (NSV * W + 31) / 32;
  // decode table: symbol -> operand dwords of digit bytes.  L = 6 splits a
  // symbol into s mod 1296 (4 codes, one table dword) and s div 1296 (the
  // fifth code, which is its own operand dword: no table); L = 7 into s mod
  // 2401 (4 codes) and s div 2401 (3 codes), one table dword each.
  static constexpr bool SPLIT = L == 6 || L == 7;
  static constexpr int DIV = L == 6 ? 1296 : L == 7 ? 2401 : 1;  // the split's divisor
  static constexpr int TED = SPLIT ? 1 : EDW;                // dwords per table entry
  static constexpr int NENT = L == 6 ? DIV : SPLIT ? DIV + ipow(L, n) / DIV : ipow(L, n);   // entries
  static constexpr int LUTDW = NENT * TED;                   // dwords of one copy
};

template <int BASE, int L>
__host__ __device__ constexpr int slot_digit(int w) {
  return (BASE == 1 && L == 4) ? w / 2
       : L == 6 ? (w < 5 ? w : -1)
       : L == 5 ? (w < 3 ? w : -1)
       : L == 3 ? (w < 5 ? w : -1)
       : L == 7 ? (w < 7 ? w : -1)
       : L == 8 ? (w < 2 ? w : -1)
       : w;                                                  // affine L = 4, L = 2
}
template <int BASE, int L>
__host__ __device__ constexpr int slot_plane(int w) { return (BASE == 1 && L == 4) ? w % 2 : 0; }
// the slot (within a symbol's STRIDE slots) of code d, plane 0: the inverse
// of slot_digit / slot_plane
template <int BASE, int L>
__host__ __device__ constexpr int digit_slot(int d) {
  return (BASE == 1 && L == 4) ? 2 * d : d;
}
template <int BASE, int L>
__host__ __device__ constexpr bool digit_slot_inverts() {
  for (int d = 0; d < sym_digits(L); ++d) {
    const int w = digit_slot<BASE, L>(d);
    if (w < 0 || w >= 8 || slot_digit<BASE, L>(w) != d || slot_plane<BASE, L>(w) != 0) return false;
  }
  return true;
}
static_assert(digit_slot_inverts<0, 6>() && digit_slot_inverts<0, 5>() && digit_slot_inverts<0, 4>() &&
              digit_slot_inverts<0, 3>() && digit_slot_inverts<1, 4>() && digit_slot_inverts<1, 3>() &&
              digit_slot_inverts<0, 2>() && digit_slot_inverts<0, 7>() && digit_slot_inverts<0, 8>(), "slots");

__device__ inline uint32_t mulhi24(uint32_t a, uint32_t b) {
  return uint32_t((uint64_t(a & 0xFFFFFFu) * uint64_t(b & 0xFFFFFFu)) >> 32);
}

// a * b + c on 24-bit signed a, b: one full-rate v_mad_i32_i24 (left to
// itself the compiler widens this to a 64-bit multiply-add)
__device__ inline uint32_t mad_i24(uint32_t a, int b, uint32_t c) {
  uint32_t r;
  __asm__("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b), "v"(c));
  return r;
}

// ------------------------------------------------------ decode tables ----

// Dword K of table entry E: the digit bytes of operand slots 4K .. 4K+3 of
// symbol value E (L = 6: entry E < 1296 gives the four codes of s mod 1296 ->
// slots 0-3; slot 4 holds s div 1296 itself).
template <int BASE, int L, int K>
__host__ __device__ constexpr uint32_t entry_dword(uint32_t E) {
  using Tr = Traits<BASE, L>;
  if constexpr (L == 6) {
    return (E % 6) | ((E / 6 % 6) << 8) | ((E / 36 % 6) << 16) | ((E / 216) << 24);
  } else if constexpr (L == 7) {                             // s mod 2401: 4 codes; s div 2401: 3 codes
    const bool hi = E >= 2401;
    const uint32_t v = hi ? E - 2401 : E;
    return (v % 7) | ((v / 7 % 7) << 8) | ((v / 49 % 7) << 16) | (hi ? 0u : (v / 343) << 24);
  } else {
    uint32_t w = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int wsl = 4 * K + j, dg = slot_digit<BASE, L>(wsl);
      if (dg >= 0) {
        const uint32_t p = uint32_t(ipow(L, dg)), c = E / p - (E / (p * L)) * L;
        const uint32_t d = slot_plane<BASE, L>(wsl) ? (c >> 1) : (Tr::P == 2 ? (c & 1u) : c);
        w |= d << (8 * j);
      }
    }
    return w;
  }
}

// the digits a table entry gives, checked against plain base-L arithmetic
// (L = 6: the four codes of s mod 1296; L = 7: the entries of both parts,
// which cover every symbol through s mod 2401 and s div 2401)
template <int BASE, int L>
__host__ __device__ constexpr bool entries_match_digits() {
  using Tr = Traits<BASE, L>;
  const int nent = Tr::NENT;
  for (int E = 0; E < nent; ++E) {
    for (int w = 0; w < Tr::STRIDE; ++w) {
      uint32_t byte = 0, want = 0;
      if (L == 6) {
        // entries are s mod 1296: four codes in slots 0-3 (slot 4, the
        // quotient, is not tabled)
        if (w >= 4) continue;
        byte = (entry_dword<BASE, L, 0>(uint32_t(E)) >> (8 * w)) & 0xFFu;
        int c = E;
        for (int t = 0; t < w; ++t) c /= L;
        want = uint32_t(c % L);
      } else if (Tr::SPLIT) {
        // the low part's entry gives the first four digits of base 7 in
        // slots 0-3, the high part's the rest from slot 4 on
        const bool hi = w >= 4;
        if (hi != (E >= Tr::DIV)) continue;
        byte = (entry_dword<BASE, L, 0>(uint32_t(E)) >> (8 * (w % 4))) & 0xFFu;
        const int v = hi ? E - Tr::DIV : E, first = 4;
        const int dg = slot_digit<BASE, L>(w) - (hi ? first : 0);
        if (slot_digit<BASE, L>(w) >= 0) {
          int c = v;
          for (int t = 0; t < dg; ++t) c /= L;
          want = uint32_t(c % L);
        }
      } else {
        const uint32_t dw = w < 4 ? entry_dword<BASE, L, 0>(uint32_t(E)) : entry_dword<BASE, L, 1>(uint32_t(E));
        byte = (dw >> (8 * (w % 4))) & 0xFFu;
        const int dg = slot_digit<BASE, L>(w);
        if (dg >= 0) {
          int c = E;
          for (int t = 0; t < dg; ++t) c /= L;
          c %= L;
          want = slot_plane<BASE, L>(w) ? uint32_t(c >> 1) : (Tr::P == 2 ? uint32_t(c & 1) : uint32_t(c));
        }
      }
      if (byte != want) return false;
    }
  }
  return true;
}
static_assert(entries_match_digits<0, 6>() && entries_match_digits<0, 5>() && entries_match_digits<0, 4>() &&
              entries_match_digits<0, 3>() && entries_match_digits<1, 4>() && entries_match_digits<1, 3>() &&
              entries_match_digits<0, 2>() && entries_match_digits<0, 7>() && entries_match_digits<0, 8>(), "tables");

// A pool's decode table and the places of its weights, made by the compiler
// and read from memory by every workgroup: made by the workgroup instead, the
// table took 110 of a launch's ~530 prologue instructions per wave.
//  lut:  the table's dwords, entry after entry (one copy)
//  pvw:  per lane (n, r): where the weights of tokens 16 blk + n, blk = 0..3,
//        land in the weight operands (value group 0, plane 0, row 4r)
constexpr int kLaneGroup = 16 * 16 + 16;                     // bytes per lane group of the weight operands
template <int BASE, int L>
struct PoolConst {
  using Tr = Traits<BASE, L>;
  // pvw is read 16 bytes at a time, lut up to 8
  alignas(16) uint32_t lut[Tr::LUTDW];
  alignas(16) uint32_t pvw[64][4];
  constexpr PoolConst() : lut(), pvw() {
    for (int e = 0; e < Tr::NENT; ++e) {
      lut[e * Tr::TED] = entry_dword<BASE, L, 0>(uint32_t(e));
      if (Tr::TED == 2) lut[e * Tr::TED + Tr::TED - 1] = entry_dword<BASE, L, 1>(uint32_t(e));
    }
    for (int lane = 0; lane < 64; ++lane)
      for (int blk = 0; blk < 4; ++blk) {
        const int t = 16 * blk + lane % 16, p = t / Tr::n, d = t % Tr::n, k = p / 4;
        pvw[lane][blk] = uint32_t((k / Tr::SPC) * 4 * kLaneGroup + p % 4 * kLaneGroup + 64 * (lane / 16) +
                                  k % Tr::SPC * Tr::STRIDE + digit_slot<BASE, L>(d));
      }
  }
};
template <int BASE, int L>
__device__ const PoolConst<BASE, L> kPoolConst{};
template <int BASE, int L>
constexpr bool pool_const_aligned() {
  using C = PoolConst<BASE, L>;
  return alignof(C) >= 16 && offsetof(C, lut) % 16 == 0 && offsetof(C, pvw) % 16 == 0 && sizeof(C::pvw[0]) == 16;
}
static_assert(pool_const_aligned<0, 2>() && pool_const_aligned<0, 3>() && pool_const_aligned<0, 4>() &&
              pool_const_aligned<0, 5>() && pool_const_aligned<0, 6>() && pool_const_aligned<0, 7>() &&
              pool_const_aligned<0, 8>() && pool_const_aligned<1, 3>() && pool_const_aligned<1, 4>(), "vector loads");

// 16-byte piece q of the replicated LDS table (entry e of replica r at entry
// slot e R + r; R >= 4, so a piece lies in one entry, repeated)
template <int BASE, int L, int R>
__device__ inline uint4 lut_piece(uint32_t q) {
  using Tr = Traits<BASE, L>;
  static_assert(R >= 4 && (R & (R - 1)) == 0, "replicas");
  const uint32_t* t = kPoolConst<BASE, L>.lut;
  if constexpr (Tr::TED == 1) {
    const uint32_t x = t[(4 * q) / R];
    return make_uint4(x, x, x, x);
  } else {
    const uint2 x = *reinterpret_cast<const uint2*>(t + 2 * ((2 * q) / R));
    return make_uint4(x.x, x.y, x.x, x.y);
  }
}

// Bits [OFF, OFF+W) of a normalized segment moved to bit S; the bits around
// them are junk (the caller masks them off).
template <int OFF, int W, int S, int NW>
__device__ inline uint32_t field_at(const uint32_t (&seg)[NW]) {
  constexpr int w = OFF / 32, sh = OFF % 32;
  if constexpr (sh + W <= 32) {
    if constexpr (sh >= S) return sh == S ? seg[w] : seg[w] >> (sh - S);
    else return seg[w] << (S - sh);
  } else {
    static_assert(sh >= S, "field position");
    return __builtin_amdgcn_alignbit(seg[w + 1], seg[w], sh - S);
  }
}

// (a << s) | c and (a & b) | c as single instructions (the compiler turns the
// OR of disjoint bits into an add and re-associates the table's base address
// into it, which costs an instruction per symbol)
__device__ inline uint32_t lshl_or(uint32_t a, int s, uint32_t c) {
  uint32_t r;
  __asm__("v_lshl_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(s), "v"(c));
  return r;
}
__device__ inline uint32_t and_or(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  __asm__("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// (symbol K of a segment) << S | lbase; a symbol past the line's last is 0.
// FULL has bit K set when symbol K has the full width in every segment (its
// lane mask is then a constant).
template <int BASE, int L, int S, uint32_t FULL, int K, int NW, int NS>
__device__ inline uint32_t sym_addr(const uint32_t (&seg)[NW], const uint32_t (&maskS)[NS], uint32_t lbase) {
  using Tr = Traits<BASE, L>;
  if constexpr (K >= NS) {
    return lbase;
  } else {
    constexpr int OFF = K * Tr::W, sh = OFF % 32;
    if constexpr (((FULL >> K) & 1u) && sh + Tr::W <= 32)
      return lshl_or((seg[OFF / 32] >> sh) & ((1u << Tr::W) - 1u), S, lbase);
    else
      return and_or(field_at<OFF, Tr::W, S, NW>(seg), maskS[K], lbase);
  }
}

// bit K set when symbol K of a line of NVALS codes has the full width in all
// four segments
template <int L, int NVALS, int NLINES>
__host__ __device__ constexpr uint32_t full_symbols() {
  constexpr SegTable<L, NVALS, NLINES> t{};
  uint32_t f = 0;
  for (int k = 0; k < 16; ++k) {
    bool all = true;
    for (int j = 0; j < 4; ++j) all = all && t.width[j][k] == width_of(L, sym_digits(L));
    if (all) f |= 1u << k;
  }
  return f;
}

// A lane's view of its pool's LDS tables: entry e of its replica is at byte
// (e << S) + lbase of t; for L = 7 the s div 2401 part starts at hbase.
struct LutRef {
  const uint8_t* t;
  uint32_t lbase, hbase;
};

__host__ __device__ constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x / 2); }

// floor(v / 1296) for v < 6^5 as the high word of x * M with x = (v << S) + b,
// b < 2^S a multiple of 4 (the lane's replica offset): the least M above
// 2^(32-S) / 1296 that is exact for every v at both ends of b (x * M does not
// decrease with b), found at compile time.
__host__ __device__ constexpr bool magic1296_ok(int S, uint64_t M) {
  if (M >= (1u << 24) || (7775u << S) + (1u << S) >= (1u << 24)) return false;
  const uint64_t bmax = (1u << S) - 4;
  for (uint64_t v = 0; v < 7776; ++v)
    if (((v << S) * M) >> 32 != v / 1296 || (((v << S) + bmax) * M) >> 32 != v / 1296) return false;
  return true;
}
__host__ __device__ constexpr uint32_t magic1296(int S) {
  const uint64_t m0 = ((uint64_t(1) << (32 - S)) + 1295) / 1296;
  for (uint64_t M = m0; M < m0 + 64; ++M)
    if (magic1296_ok(S, M)) return uint32_t(M);
  return 0u;
}

// floor(v / 2401) for v < 7^7 as the high word of v * 1788825 (v and the
// multiplier fit 24 bits).  floor(v M / 2^32) does not decrease with v, so it
// is exact everywhere when it is exact on both sides of every multiple of 2401.
constexpr uint32_t kMagic2401 = 1788825u;
__host__ __device__ constexpr bool magic2401_exact() {
  if (kMagic2401 >= (1u << 24) || 823542u >= (1u << 24)) return false;
  for (uint64_t k = 1; k <= 343; ++k) {
    const uint64_t below = 2401 * k - 1, at = 2401 * k;
    if ((below * kMagic2401) >> 32 != k - 1) return false;
    if (at < 823543 && (at * kMagic2401) >> 32 != k) return false;
  }
  return true;
}
static_assert(magic2401_exact(), "7-level digit split");

// operand dwords of 7-level symbol K: the s mod 2401 and s div 2401 entries
template <int BASE, int S, uint32_t FULL, int K, int NW, int NS>
__device__ inline uint2 l7_symbol(const uint32_t (&seg)[NW], const uint32_t (&maskS)[NS], const LutRef& lr) {
  const uint32_t x = sym_addr<BASE, 7, S, FULL, K, NW, NS>(seg, maskS, 0u);   // v << S
  const uint32_t hi = mulhi24(x >> S, kMagic2401);                           // v div 2401
  const uint32_t lo = mad_i24(hi, -(2401 << S), x) + lr.lbase;                // ((v mod 2401) << S) + lbase
  return make_uint2(*reinterpret_cast<const uint32_t*>(lr.t + lo),
                    *reinterpret_cast<const uint32_t*>(lr.t + ((hi << S) + lr.hbase)));
}

// operand dwords of 6-level symbol K: the s mod 1296 entry (codes 0-3) and
// s div 1296 (code 4, a value below 6: its own operand dword)
template <int BASE, int S, uint32_t FULL, int K, int NW, int NS>
__device__ inline uint2 l6_symbol(const uint32_t (&seg)[NW], const uint32_t (&maskS)[NS], const LutRef& lr) {
  constexpr uint32_t M = magic1296(S);
  static_assert(M != 0, "digit split");
  const uint32_t x = sym_addr<BASE, 6, S, FULL, K, NW, NS>(seg, maskS, lr.lbase);   // (v << S) + lbase
  const uint32_t hi = mulhi24(x, M);                                                // v div 1296
  const uint32_t lo = mad_i24(hi, -(1296 << S), x);                                 // ((v mod 1296) << S) + lbase
  return make_uint2(*reinterpret_cast<const uint32_t*>(lr.t + lo), hi);
}

// Operand dwords of symbol slot K of a segment.  A slot past the longest
// segment (K >= NS, known at compile time) holds no symbol in any lane: its
// digits are zero and no table is read.  Slots of lanes whose segment is one
// symbol shorter read table entry 0 (all digits zero) through a zero mask.
template <int BASE, int L, int S, uint32_t FULL, int K, int NW, int NS>
__device__ inline uint32_t sym_dword(const uint32_t (&seg)[NW], const uint32_t (&maskS)[NS], const LutRef& lr) {
  if constexpr (K >= NS) return 0u;
  else return *reinterpret_cast<const uint32_t*>(lr.t + sym_addr<BASE, L, S, FULL, K, NW, NS>(seg, maskS, lr.lbase));
}
template <int BASE, int L, int S, uint32_t FULL, int K, int NW, int NS>
__device__ inline uint2 sym_dword2(const uint32_t (&seg)[NW], const uint32_t (&maskS)[NS], const LutRef& lr) {
  if constexpr (K >= NS) return make_uint2(0u, 0u);
  else return *reinterpret_cast<const uint2*>(lr.t + sym_addr<BASE, L, S, FULL, K, NW, NS>(seg, maskS, lr.lbase));
}

// MFMA operand of chunk C of a segment (symbols SPC*C ..), read from the tables
template <int BASE, int L, int S, uint32_t FULL, int C, int NW, int NS>
__device__ inline int4v chunk_operand(const uint32_t (&seg)[NW], const uint32_t (&maskS)[NS], const LutRef& lr) {
  using Tr = Traits<BASE, L>;
  uint4v r;
  if constexpr (L == 6 || L == 7) {
    uint2 p0 = make_uint2(0u, 0u), p1 = make_uint2(0u, 0u);
    if constexpr (L == 6) {
      if constexpr (2 * C < NS) p0 = l6_symbol<BASE, S, FULL, 2 * C, NW, NS>(seg, maskS, lr);
      if constexpr (2 * C + 1 < NS) p1 = l6_symbol<BASE, S, FULL, 2 * C + 1, NW, NS>(seg, maskS, lr);
    } else {
      if constexpr (2 * C < NS) p0 = l7_symbol<BASE, S, FULL, 2 * C, NW, NS>(seg, maskS, lr);
      if constexpr (2 * C + 1 < NS) p1 = l7_symbol<BASE, S, FULL, 2 * C + 1, NW, NS>(seg, maskS, lr);
    }
    r = uint4v{p0.x, p0.y, p1.x, p1.y};
  } else if constexpr (Tr::SPC == 4) {
    r = uint4v{sym_dword<BASE, L, S, FULL, 4 * C, NW, NS>(seg, maskS, lr),
               sym_dword<BASE, L, S, FULL, 4 * C + 1, NW, NS>(seg, maskS, lr),
               sym_dword<BASE, L, S, FULL, 4 * C + 2, NW, NS>(seg, maskS, lr),
               sym_dword<BASE, L, S, FULL, 4 * C + 3, NW, NS>(seg, maskS, lr)};
  } else {
    const uint2 a = sym_dword2<BASE, L, S, FULL, 2 * C, NW, NS>(seg, maskS, lr);
    const uint2 b = sym_dword2<BASE, L, S, FULL, 2 * C + 1, NW, NS>(seg, maskS, lr);
    r = uint4v{a.x, a.y, b.x, b.y};
  }
  return __builtin_bit_cast(int4v, r);
}

// MFMA operands of all NC chunks of a segment: every table read is issued
// before the first product needs one (LDS returns them in order)
template <int BASE, int L, int S, uint32_t FULL, int NW, int NS, int NC>
__device__ inline void chunk_operands(const uint32_t (&seg)[NW], const uint32_t (&maskS)[NS], const LutRef& lr,
                                      int4v (&A)[NC]) {
  static_assert(NC <= 4, "chunks");
#define SEMKV_O(C) if constexpr (C < NC) A[C] = chunk_operand<BASE, L, S, FULL, C, NW, NS>(seg, maskS, lr);
  SEMKV_O(0) SEMKV_O(1) SEMKV_O(2) SEMKV_O(3)
#undef SEMKV_O
}

// masks of the symbols of segment j (zero past the line's last symbol)
template <int L, int NVALS, int NLINES, int NS>
__device__ inline void segment_masks(int j, uint32_t (&mask)[NS]) {
  constexpr SegTable<L, NVALS, NLINES> t{};
#pragma unroll
  for (int k = 0; k < NS; ++k)
    mask[k] = pick4(j, (1u << t.width[0][k]) - 1u, (1u << t.width[1][k]) - 1u,
                    (1u << t.width[2][k]) - 1u, (1u << t.width[3][k]) - 1u);
}

// dwords that hold any line's segment, from the dword of its first bit on
template <int L, int NVALS, int NLINES>
__host__ __device__ constexpr int seg_dwords() {
  constexpr SegTable<L, NVALS, NLINES> t{};
  int most = 0;
  for (int j = 0; j < 4; ++j)
    for (int line = 0; line < NLINES; ++line) {
      const int n = ((t.start[j] + line * t.bits[j]) % 32 + t.bits[j] + 31) / 32;
      most = n > most ? n : most;
    }
  return most;
}

__device__ inline float hf(uint16_t b) { return __half2float(__ushort_as_half(b)); }

template <int BASE, int L, int G>
struct Geo {
  using Tr = Traits<BASE, L>;
  static constexpr int MB = meta_bytes(BASE, G);
  static constexpr int RB = 2 * Tr::TB + 2 * MB;
  static constexpr int KLD = seg_dwords<L, kD, kSlots>(), VLD = seg_dwords<L, kSlots, kD>();   // dwords of a segment
  static constexpr int NML = (2 * MB + 1023) / 1024;         // 1 KB metadata pieces per record
  static constexpr int NG = BASE != 1 ? kD / G : 1;          // score products per chunk (query groups)
  static constexpr int NGV = BASE != 1 ? kD / G : 1;         // value groups
  static constexpr int NPL = Tr::P;                          // value planes (tq, 4 levels: 2)
  // Score products: a chunk covers CCH consecutive channels, a query group GQ,
  // so only the (group, chunk) pairs that share a channel are not all zero
  // (G = 32: 5 of 12 at 5 levels, 7 of 16 at 6).  Pairs are numbered along the
  // channels; pair_at is the number of the pair that holds channel c: the
  // chunk and group edges at or below c, each once.
  static constexpr int CCH = 4 * Tr::SPC * Tr::n, GQ = BASE != 1 ? G : kD;
  static constexpr int BOTH = CCH / gcd_of(CCH, GQ) * GQ;     // both have an edge at its multiples
  __host__ __device__ static constexpr int pair_at(int c) { return c / CCH + c / GQ - c / BOTH; }
  static constexpr int NPAIR = pair_at(kD - 1) + 1;
  static constexpr bool pair_used(int g, int ch) { return ch * CCH < (g + 1) * GQ && g * GQ < (ch + 1) * CCH; }
  static constexpr int pair_of(int g, int ch) { return pair_at(g * GQ > ch * CCH ? g * GQ : ch * CCH); }
  // int8 weights of one wave and one value group at a time, in value
  // A-operand order: [chunk][lane group][row][16 slots], so a lane reads a
  // chunk's operand at once.  Row 4h + s holds byte s of head h's weights;
  // rows 4h + 3, pad slots and slots past token 63 are never written and
  // stay zero.
  // lane groups 272 bytes apart (16 rows of 16 slots, then 16 bytes of pad):
  // the byte writes of consecutive symbols, which sit in consecutive lane
  // groups, land in different LDS banks rather than all in one
  static constexpr int KGS = kLaneGroup;                     // bytes per lane group
  static constexpr int CHB = 4 * KGS;                        // bytes per chunk
  static constexpr int PV = Tr::NCV * CHB;                   // bytes per wave
  static_assert(RB % 16 == 0, "record pieces");
};

// the pairs in use are numbered 0, 1, ... without gaps, and every channel's
// pair is the one of its chunk and group
template <class Ge, int NCK, int NG>
__host__ __device__ constexpr bool pairs_numbered() {
  int n = 0;
  for (int g = 0; g < NG; ++g)
    for (int ch = 0; ch < NCK; ++ch)
      if (Ge::pair_used(g, ch)) n += Ge::pair_of(g, ch) < Ge::NPAIR ? 1 : 1000;
  for (int c = 0; c < kD; ++c)
    if (!Ge::pair_used(c / Ge::GQ, c / Ge::CCH) || Ge::pair_of(c / Ge::GQ, c / Ge::CCH) != Ge::pair_at(c)) return false;
  return n == Ge::NPAIR;
}

template <int CTRL>
__device__ inline float dpp(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
// reductions over the 16 lanes of a row (row_ror 8, 4, 2, 1).  The maximum
// is four DPP maxima written out: fmaxf of a DPP move costs three
// instructions a step (the move, a quieting max of the moved value that the
// IEEE-mode maxNum contract asks of an operand not known to be canonical, the
// max), and the values here are never NaN.  Every DPP read of a register
// written by the VALU instruction just before it needs two wait states, which
// the compiler does not insert around inline assembly: hence the s_nop 1
// before each (and after the last, for a DPP read that may follow).
// Called with the whole wave active.
__device__ inline float row_max16(float x) {
  float r;
  __asm__("s_nop 1\n\t"
          "v_max_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
          "s_nop 1\n\t"
          "v_max_f32_dpp %0, %0, %0 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
          "s_nop 1\n\t"
          "v_max_f32_dpp %0, %0, %0 row_ror:2 row_mask:0xf bank_mask:0xf\n\t"
          "s_nop 1\n\t"
          "v_max_f32_dpp %0, %0, %0 row_ror:1 row_mask:0xf bank_mask:0xf\n\t"
          "s_nop 1"
          : "=&v"(r) : "v"(x));
  return r;
}
// max of four values that are never NaN (no quieting of operands)
__device__ inline float max4(float a, float b, float c, float d) {
  float r;
  __asm__("v_max3_f32 %0, %1, %2, %3\n\t"
          "v_max_f32 %0, %0, %4"
          : "=&v"(r) : "v"(a), "v"(b), "v"(c), "v"(d));
  return r;
}
__device__ inline float row_sum16(float x) {
  x += dpp<0x128>(x);
  x += dpp<0x124>(x);
  x += dpp<0x122>(x);
  return x + dpp<0x121>(x);
}

// normalized segment of NW dwords from the ND dwords that hold it, the first
// bit at bit `sh` (its low 5 bits) of the first
template <int NW, int ND>
__device__ inline void normalize(const uint32_t* d, int sh, uint32_t (&seg)[NW]) {
#pragma unroll
  for (int k = 0; k < NW; ++k) seg[k] = __builtin_amdgcn_alignbit(k + 1 < ND ? d[k + 1] : 0u, k < ND ? d[k] : 0u, sh);
}

// ------------------------------------------------------- kernel layout ----

template <int BASE, int LH, int LL, int G>
struct Plan {
  using GH = Geo<BASE, LH, G>;
  using GL = Geo<BASE, LL, G>;
  static constexpr int KLD = GH::KLD > GL::KLD ? GH::KLD : GL::KLD, VLD = GH::VLD > GL::VLD ? GH::VLD : GL::VLD;
  static constexpr int NML = GH::NML;
  static constexpr int MSTAGE = 2 * GH::MB;                 // bytes of a record's metadata
  static constexpr int PV = GH::PV > GL::PV ? GH::PV : GL::PV;
  static constexpr int NGV = GH::NGV;
  static constexpr int NG = GH::NG;
  static constexpr int NPAIRS = GH::NPAIR + GL::NPAIR;       // score operands of both pools
  static_assert(GH::NGV == GL::NGV, "pools share the value groups");
  static_assert(pairs_numbered<GH, Traits<BASE, LH>::NCK, GH::NG>() && pairs_numbered<GL, Traits<BASE, LL>::NCK, GL::NG>(), "pairs");
  // LDS of a workgroup of nw waves with rh / rl table replicas (the Shared
  // layout below, with margin)
  static constexpr int lds_bytes(int nw, int rh, int rl) {
    return nw * (MSTAGE + PV + 256) + (Traits<BASE, LH>::LUTDW * rh + Traits<BASE, LL>::LUTDW * rl) * 4 +
           (GH::NPAIR + GL::NPAIR) * 64 * 16 + 4 * kD * 4 + 2080 + 3104 + 640;
  }
  // 2 waves per SIMD, one workgroup per compute unit, one thread per (head,
  // channel) of the query and the output: every level pair fits
  static constexpr int NW = kDecodeWaves;
  static_assert(NW * 64 == 4 * kD && lds_bytes(NW, 4, 4) <= 160 * 1024, "workgroup");
  static constexpr int NT = 64 * NW;
  // table replicas per pool: the most that fit, the low pool (the larger
  // share of the tokens) first (32 dword replicas: a conflict-free lookup of
  // any entries)
  // (the 7-level tables, 2744 entries, keep 4 replicas: 44 KB; the 6-level
  // table, 1296 entries, at most 8: 41 KB)
  static constexpr int cap(int L) { return L == 7 ? 4 : L == 6 ? 8 : 32; }
  static constexpr int pick_replicas(bool hi) {
    constexpr int opts[8][2] = {{32, 32}, {16, 32}, {8, 32}, {16, 16}, {8, 16}, {8, 8}, {4, 8}, {4, 4}};
    for (const auto& o : opts) {
      const int rh = o[0] < cap(LH) ? o[0] : cap(LH), rl = o[1] < cap(LL) ? o[1] : cap(LL);
      if (lds_bytes(NW, rh, rl) <= 160 * 1024) return hi ? rh : rl;
    }
    return 0;
  }
  static constexpr int RH = pick_replicas(true), RL = pick_replicas(false);
  static_assert(RH >= 4 && RL >= 4, "LDS");
  // table entries are 2^SH, 2^SL bytes apart
  static constexpr int SH = ilog2(RH * Traits<BASE, LH>::TED * 4), SL = ilog2(RL * Traits<BASE, LL>::TED * 4);
  static_assert((1 << SH) == RH * Traits<BASE, LH>::TED * 4 && (1 << SL) == RL * Traits<BASE, LL>::TED * 4, "entry stride");
  static constexpr int LUTH = Traits<BASE, LH>::LUTDW * RH;  // dwords of the high-pool tables
  static constexpr int LUTL = Traits<BASE, LL>::LUTDW * RL;
};

struct Fin { float m[4], l[4]; float o[4][kD]; };             // one wave's state, merged form
struct TailScratch { float lg[4][kSlots]; float mx[4], sum[4]; float o[4][kD]; };

// A wave's current record in registers: the dwords of its lanes' four K
// segments and eight V segments, and the metadata on its way to LDS.
template <class PL>
struct Record {
  uint32_t k[4][PL::KLD], v[8][PL::VLD];
  uint4 m[PL::NML];
};

template <class PL>
struct Shared {
  // decode tables (high pool, low pool) first: their offsets fit the 16-bit
  // immediate offset of an LDS read, so a lookup needs no base add
  alignas(16) uint32_t lut[PL::LUTH + PL::LUTL];
  alignas(16) uint8_t meta[PL::NW][PL::MSTAGE];              // per wave: the record's metadata
  alignas(16) uint8_t pv[PL::NW][PL::PV];                    // per wave int8 weights, later its Fin
  float qorig[4][kD];                                        // query as given (fp16 tail)
  Fin tfin;                                                  // the fp16 tail's state
  TailScratch ts;
  alignas(16) uint4 aq[PL::NPAIRS][64];                      // score A operands: pool, (group, chunk) pair, lane
  float zpart[4][4];                                         // per head: sums of q over 32-channel runs
  float qmax[4][4];                                          // per head: max |q| over 32-channel runs
  float qsc[2][4][4], zws[2][4][4];                          // per pool, head and group: score scale, zero-point term
  float zc[PL::NW][4][4];                                    // per wave, head, group: sum p * zero
  int last;
};

template <class PL>
__device__ inline Fin* wave_fin(Shared<PL>& sm, int w) {
  static_assert(PL::PV >= int(sizeof(Fin)) && PL::PV % 16 == 0, "state in the weight array");
  return reinterpret_cast<Fin*>(sm.pv[w]);
}

template <int NGV>
struct WaveState {
  float m, l, z[NGV];
  float qw, qwi;     // scale of the int8 weights (a power of 2) and its inverse
  float of[8];       // flushed value sums, channel 16 cb + n of head r
  int4v cv[8];       // integer value sums since the last flush, rows (head, byte)
#ifdef SEMKV_TIMELINE
  int nrec = 0, nflush = 0;   // tracing build: records and flushes of the wave
#endif
};

// the integer q . codes of one head from its three byte rows
__device__ inline float comb3(const int4v& c) {
  return fmaf(float(c[0]), 16384.0f, fmaf(float(c[1]), 128.0f, float(c[2])));
}
// the same for one product of a score: |row 0| < 2^16, |row 1| < 2^17, so
// the integer sum stays below 2^31
// bits [OFF, OFF+7) of x as one instruction (left to itself the compiler
// emits a shift and a mask).  Its operand must not come straight from a
// matrix instruction: the compiler does not insert the wait states a read of
// an MFMA result needs before inline assembly.
template <int OFF>
__device__ inline uint32_t bits7(uint32_t x) {
  uint32_t r;
  __asm__("v_bfe_u32 %0, %1, %2, 7" : "=v"(r) : "v"(x), "i"(OFF));
  return r;
}
__device__ inline float comb3_score(const int4v& c) {
  // two shift-adds; the empty statement keeps the compiler from re-associating
  // them into two shifts and a three-way add
  int t = (c[0] << 7) + c[1];
  __asm__("" : "+v"(t));
  return float((t << 7) + c[2]);
}

// ------------------------------------------------------- record loads ----

// Where a lane's segments of a record of one pool begin: byte offsets of the
// first two blocks' dwords, the bytes from a block to the next but one, and the
// bit within (32 lines are a whole number of dwords, so blocks two apart share
// it).
struct LaneGeo {
  int kb[2], vb[2], kstep, vstep;            // what a load needs
  int ksh[2], vsh[2];                        // what the extraction needs
};

// What a lane's geometry needs of the segments of one body, in scalars: bits
// of a line's segment j in byte j of `bits`, and the bits of the segments
// before it as j b0 less byte j of `less`.
struct SegScalars {
  uint32_t bits, less;
  int b0;
};
template <int L, int NV, int NL>
__host__ __device__ constexpr SegScalars seg_scalars() {
  constexpr SegTable<L, NV, NL> t{};
  SegScalars s{0u, 0u, t.bits[0]};
  for (int j = 0; j < 4; ++j) {
    s.bits |= uint32_t(t.bits[j]) << (8 * j);
    s.less |= uint32_t(j * t.bits[0] - t.start[j] / NL) << (8 * j);
  }
  return s;
}
template <int L, int NV, int NL>
__host__ __device__ constexpr bool seg_scalars_ok() {
  constexpr SegTable<L, NV, NL> t{};
  for (int j = 0; j < 4; ++j) {
    const int less = j * t.bits[0] - t.start[j] / NL;
    if (t.bits[j] < 0 || t.bits[j] > 255 || less < 0 || less > 255 || t.start[j] % NL != 0) return false;
  }
  return true;
}

// the lane's geometry in the high (hi) or low pool: hi is the same for the
// whole wave, so the pool's constants are scalar selects (about 35 vector
// instructions; every wave pays them before its first record's loads)
template <int BASE, int LH, int LL>
__device__ inline LaneGeo lane_geo(bool hi, int lane) {
  static_assert(seg_scalars_ok<LH, kD, kSlots>() && seg_scalars_ok<LL, kD, kSlots>() && seg_scalars_ok<LH, kSlots, kD>() &&
                seg_scalars_ok<LL, kSlots, kD>(), "segment scalars");
  constexpr SegScalars kH = seg_scalars<LH, kD, kSlots>(), kL = seg_scalars<LL, kD, kSlots>();
  constexpr SegScalars vH = seg_scalars<LH, kSlots, kD>(), vL = seg_scalars<LL, kSlots, kD>();
  const uint32_t n = lane & 15, j = lane >> 4;
  // first bit of line n's segment j, and the bits of one line of it
  auto first = [&](uint32_t bits, uint32_t less, int b0, int lines, int& lb) {
    lb = int(__builtin_amdgcn_ubfe(bits, 8 * j, 8));
    return int(__umul24(j, b0) - __builtin_amdgcn_ubfe(less, 8 * j, 8)) * lines + int(__umul24(n, lb));
  };
  int kbits, vbits;
  const int k0 = first(hi ? kH.bits : kL.bits, hi ? kH.less : kL.less, hi ? kH.b0 : kL.b0, kSlots, kbits);
  const int v0 = first(hi ? vH.bits : vL.bits, hi ? vH.less : vL.less, hi ? vH.b0 : vL.b0, kD, vbits) +
                 8 * (hi ? tile_bytes(LH) : tile_bytes(LL));
  LaneGeo g;
  g.ksh[0] = k0;
  g.ksh[1] = k0 + 16 * kbits;
  g.vsh[0] = v0;
  g.vsh[1] = v0 + 16 * vbits;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    g.kb[i] = (g.ksh[i] >> 3) & ~3;
    g.vb[i] = (g.vsh[i] >> 3) & ~3;
  }
  g.kstep = 4 * kbits;
  g.vstep = 4 * vbits;
  return g;
}

template <int N>
__device__ inline void load_dwords(__amdgpu_buffer_rsrc_t rs, int off, uint32_t* r) {
  if constexpr (N >= 4) {
    const uint4v x = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
    r[0] = x.x, r[1] = x.y, r[2] = x.z, r[3] = x.w;
    load_dwords<N - 4>(rs, off + 16, r + 4);
  } else if constexpr (N == 3) {
    const auto x = __builtin_amdgcn_raw_buffer_load_b96(rs, off, 0, 0);
    r[0] = x[0], r[1] = x[1], r[2] = x[2];
  } else if constexpr (N == 2) {
    const auto x = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
    r[0] = x[0], r[1] = x[1];
  } else if constexpr (N == 1) {
    r[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
  }
}

// Loads of a record straight into the registers that use it: each lane the
// dwords of its own segments, through a buffer descriptor bounded by the
// record's size (what a load reads past its end is 0, without memory traffic).
// Every record takes the same loads, whichever its pool; with `any` false (no
// record is left) they are bounded by 0 bytes and read nothing.
template <int BASE, int LH, int LL, int G, class PL>
struct RecordSource {
  __amdgpu_buffer_rsrc_t rs;
  int meta;
  __device__ inline RecordSource(const PoolGeom& g, const uint8_t* unit, int tile, int nt0, bool any) {
    const bool hi = tile < nt0;
    const uint8_t* rec = hi ? unit + int64_t(tile) * PL::GH::RB : unit + g.lo_offset + int64_t(tile - nt0) * PL::GL::RB;
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(rec), 0, !any ? 0 : hi ? PL::GH::RB : PL::GL::RB, kBufferWord3);
    meta = hi ? 2 * tile_bytes(LH) : 2 * tile_bytes(LL);
  }
  __device__ inline void k(const LaneGeo& lg, int i, Record<PL>& r) const {
    load_dwords<PL::KLD>(rs, lg.kb[i & 1] + (i >> 1) * lg.kstep, r.k[i]);
  }
  __device__ inline void m(int lane, Record<PL>& r) const {
#pragma unroll
    for (int i = 0; i < PL::NML; ++i) {
      const uint4v x = __builtin_amdgcn_raw_buffer_load_b128(rs, meta + i * 1024 + lane * 16, 0, 0);
      r.m[i] = make_uint4(x.x, x.y, x.z, x.w);
    }
  }
  __device__ inline void v(const LaneGeo& lg, int i, Record<PL>& r) const {
    load_dwords<PL::VLD>(rs, lg.vb[i & 1] + (i >> 1) * lg.vstep, r.v[i]);
  }
};

// Per head, of the query x (affine) or the rotated query (bases 1, 2) held by one
// thread per (head, channel) -- whole waves, 64 channels of one head each:
// sums over aligned runs of 32 channels (the zero-point terms) and the
// largest magnitude of each such run (the fixed-point scale).
template <class PL>
__device__ inline void query_runs(float x, int h, int c, Shared<PL>& sm) {
  const float sx = row_sum16(x), ax = row_max16(fabsf(x));
  const float s0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sx), 0));
  const float s1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sx), 16));
  const float s2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sx), 32));
  const float s3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sx), 48));
  const float a0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ax), 0));
  const float a1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ax), 16));
  const float a2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ax), 32));
  const float a3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ax), 48));
  if ((c & 31) == 0) {
    sm.zpart[h][c / 32] = (c & 32) ? s2 + s3 : s0 + s1;
    sm.qmax[h][c / 32] = (c & 32) ? fmaxf(a2, a3) : fmaxf(a0, a1);
  }
}

// sum of head h's query over query group g, and the exponent e of its fixed-
// point form: the largest magnitude a pool's operands hold (the tq plane
// weights included), times 2^e, lies in [2^19, 2^20)
template <int BASE, int G, class PL>
__device__ inline float query_sum(const Shared<PL>& sm, int h, int g) {
  constexpr int GQ = BASE != 1 ? G : kD;
  float z = 0.0f;
#pragma unroll
  for (int k = 0; k < GQ / 32; ++k) z += sm.zpart[h][g * GQ / 32 + k];
  return z;
}
template <int BASE, int L, int G, class PL>
__device__ inline int query_exp(const Shared<PL>& sm, const float* mu, int h, int g) {
  constexpr int GQ = BASE != 1 ? G : kD;
  float mx = 0.0f;
#pragma unroll
  for (int k = 0; k < GQ / 32; ++k) mx = fmaxf(mx, sm.qmax[h][g * GQ / 32 + k]);
  mx *= BASE != 1 || L == 3 ? 1.0f : mu[2] + mu[3];        // tq, 4 levels: mu2 + mu3 > mu3 - mu2 > 0
  const int E = __builtin_amdgcn_frexp_expf(mx);          // mx = f 2^E, f in [0.5, 1)
  return mx >= 1e-30f ? 20 - E : 0;
}

// Constants of one pool's scores and weights.  tq: mu = -m, 0, m (L = 3) or
// -b, -a, a, b (L = 4), affine in a code's bit planes.  Rotated affine: k =
// sign . H y / 8 with y = s c + z the affine value of the rotated coordinates,
// so q . k = (H sign . q) . y / 8, and the values are summed as y / 8 in the
// rotated domain (powers of 2: exact).
template <int BASE, int L>
struct Scale {
  static constexpr float kR = BASE == 2 ? 0.125f : 1.0f;
  static constexpr float kScore = kLog2e * kRsqrtD * kR;
  float cS, cZ, wP[2];
  __device__ explicit Scale(const float* mu)
      : cS(BASE != 1 ? 1.0f : (L == 3 ? mu[2] / 128.0f : 1.0f / 128.0f)),
        cZ(BASE != 1 ? 0.0f : (L == 3 ? -mu[2] / 128.0f : -mu[3] / 128.0f)),
        wP{BASE != 1 ? 1.0f : (L == 3 ? 1.0f : mu[3] - mu[2]), BASE != 1 ? 1.0f : (L == 3 ? 1.0f : mu[2] + mu[3])} {}
};

// the three bytes of channel c's integer, plane pl, to their places in one pool's operands
template <int BASE, int L, int G, int POOL, class PL>
__device__ inline void scatter_bytes(Shared<PL>& sm, int qi, int h, int c, int pl) {
  using Tr = Traits<BASE, L>;
  using Ge = Geo<BASE, L, G>;
  const int p = c / Tr::n, d = c - p * Tr::n, kg = p & 3, sk = p >> 2;
  uint8_t* dst = reinterpret_cast<uint8_t*>(&sm.aq[(POOL ? PL::GH::NPAIR : 0) + Ge::pair_at(c)][kg * 16 + 4 * h]) +
                 (sk % Tr::SPC) * Tr::STRIDE + digit_slot<BASE, L>(d) + pl;
  dst[0] = uint8_t(qi >> 14);
  dst[16] = uint8_t((qi >> 7) & 0x7F);
  dst[32] = uint8_t(qi & 0x7F);
}
// Score A operands of both pools, by the threads that hold the query x (affine)
// or the rotated query (bases 1, 2), one per (head h, channel c).  Lane (row m
// = 4h + s, kg), (group, chunk) pair, slot holds byte s of qi = rint(x 2^e)
// (tq: of the plane-weighted x) at the channel the slot addresses, |qi| <
// 2^20, e per head and group.  qi splits as 2^14 b0 + 2^7 b1 + b2 (b0 signed,
// b1, b2 in [0, 127]), so a product sums the exact integer qi . codes in three
// rows.  Each thread makes its channel's integer once and writes its three
// bytes to the one place each has; pad slots and rows 4h + 3 are zero before
// the call.  Gathering, one thread per operand of 16 slots, repeated the
// rounding for every slot, byte and group: at G = 32 and 2048 tokens it took
// 2.1 us of a 12.1 us launch (the scatter: 0.75), at G = 128 0.75 us (0.45).
// The group's first thread also leaves the score scale 2^-e and the
// zero-point term (the sum of q) of its head and group.
template <int BASE, int LH, int LL, int G, class PL>
__device__ inline void scatter_query(const DecodeArgs& a, Shared<PL>& sm, float x, int h, int c) {
  constexpr int GQ = PL::GH::GQ;
  const int g = c / GQ;
  if constexpr (BASE != 1) {                 // the same integers and scales in both pools
    const int e = query_exp<BASE, LH, G>(sm, a.mu[0], h, g);
    const float z = query_sum<BASE, G>(sm, h, g);
    const int qi = int(rintf(ldexpf(x, e)));
    scatter_bytes<BASE, LH, G, 0>(sm, qi, h, c, 0);
    scatter_bytes<BASE, LL, G, 1>(sm, qi, h, c, 0);
    if (c % GQ == 0) {
      const float k = Scale<BASE, LH>::kScore;
      sm.qsc[0][h][g] = sm.qsc[1][h][g] = ldexpf(k, -e);
      sm.zws[0][h][g] = sm.zws[1][h][g] = z * k;
    }
  } else {
    auto pool = [&](auto I) {
      constexpr int POOL = I.value, L = POOL ? LL : LH;
      using Sc = Scale<BASE, L>;
      const Sc k(a.mu[POOL]);
      const int e = query_exp<BASE, L, G>(sm, a.mu[POOL], h, g);
#pragma unroll
      for (int pl = 0; pl < Traits<BASE, L>::P; ++pl)
        scatter_bytes<BASE, L, G, POOL>(sm, int(rintf(ldexpf(k.wP[pl] * x, e))), h, c, pl);
      if (c % GQ == 0) {
        sm.qsc[POOL][h][g] = ldexpf(Sc::kScore * k.cS, -e);
        sm.zws[POOL][h][g] = query_sum<BASE, G>(sm, h, g) * (Sc::kScore * k.cZ);
      }
    };
    static_for<2>(pool);
  }
}

// ---------------------------------------------------- one pool's records ----

template <int BASE, int LH, int LL, int G, int POOL, class PL>
__device__ void run_pool(const DecodeArgs& a, Shared<PL>& sm, WaveState<PL::NGV>& st, const uint8_t* unit,
                         int nt0, int first, int stride, int i0, int i1, int count, Record<PL>& R, LaneGeo& geo, uint4& pvwq) {
  constexpr int L = POOL ? LL : LH;
  using Tr = Traits<BASE, L>;
  using Ge = Geo<BASE, L, G>;
  constexpr int NG = Ge::NG, NGV = Ge::NGV;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 15, r = lane >> 4, kg = r;
  uint8_t* kmeta = sm.meta[wave];
  const uint8_t* vmeta = kmeta + Ge::MB;
  const Scale<BASE, L> sc(a.mu[POOL]);
  constexpr float kR = Scale<BASE, L>::kR;

  // ---- score A operands (built once per workgroup): in registers for one
  // query group, else read per product
  constexpr int A0 = POOL ? PL::GH::NPAIR : 0;
  auto aq = [&](int pair) {
    const uint4 v = sm.aq[A0 + pair][lane];
    return __builtin_bit_cast(int4v, uint4v{v.x, v.y, v.z, v.w});
  };
  int4v Aq[NG == 1 ? Tr::NCK : 1];
  if constexpr (NG == 1) {
#pragma unroll
    for (int c = 0; c < Tr::NCK; ++c) Aq[c] = aq(c);
  }
  // tables: the lane's replica; entries 2^S bytes apart
  constexpr int NR = POOL ? PL::RL : PL::RH;
  constexpr int S = POOL ? PL::SL : PL::SH;
  constexpr uint32_t KFULL = full_symbols<L, kD, kSlots>(), VFULL = full_symbols<L, kSlots, kD>();
  const uint32_t lb = uint32_t((lane & (NR - 1)) * Tr::TED * 4);
  const LutRef lut{reinterpret_cast<const uint8_t*>(sm.lut + (POOL ? PL::LUTH : 0)), lb, lb + (uint32_t(Tr::DIV) << S)};
  uint32_t kmask[Tr::NSK], vmask[Tr::NSV];
  segment_masks<L, kD, kSlots>(kg, kmask);
  segment_masks<L, kSlots, kD>(kg, vmask);
#pragma unroll
  for (int k = 0; k < Tr::NSK; ++k) kmask[k] <<= S;
#pragma unroll
  for (int k = 0; k < Tr::NSV; ++k) vmask[k] <<= S;
  // softmax lanes: where token 16 blk + n of each block lands in the weight
  // operands (value group 0, plane 0, row 4r)
  if (POOL == 1 && i0 > 0) {
    geo = lane_geo<BASE, LH, LL>(false, lane);
    pvwq = *reinterpret_cast<const uint4*>(kPoolConst<BASE, L>.pvw[lane]);
  }
  const uint32_t pvwr[4] = {pvwq.x, pvwq.y, pvwq.z, pvwq.w};
  // softmax lanes: token n of each 16-token block, head r.  Per query group
  // of head r, times the softmax scale: the sum of q (zero-point term) and
  // 2^-e (the fixed-point query's scale); tq folds its level offsets in
  float zwsK[NG], qscK[NG];
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    zwsK[i] = sm.zws[POOL][r][i];
    qscK[i] = sm.qsc[POOL][r][i];
  }
  // the weight operands' pad slots and unused rows are zero: cleared by the
  // prologue, and again where the low pool's layout follows the high pool's
  uint8_t* pvw = sm.pv[wave];
  static_assert(Ge::PV % 16 == 0, "weight array pieces");
  if (POOL == 1 && i0 > 0)
    for (int i = lane; i < Ge::PV / 16; i += 64) reinterpret_cast<uint4*>(pvw)[i] = make_uint4(0u, 0u, 0u, 0u);
  const int64_t nrows = a.n_rows[POOL];

  for (int it = i0; it < i1; ++it) {
    const int tile = first + stride * it;
    // each segment leaves its load registers when it is decoded, and the next
    // record's load takes them (the empty statements keep the extraction
    // before the load: sunk below it, it would need registers of its own)
    const RecordSource<BASE, LH, LL, G, PL> next(a.g, unit, tile + stride, nt0, it + 1 < count);
    if (POOL == 0 && it + 1 == i1) {         // the next one is the low pool's: its places, this one's bits
      const int k0 = geo.ksh[0], k1 = geo.ksh[1], v0 = geo.vsh[0], v1 = geo.vsh[1];
      geo = lane_geo<BASE, LH, LL>(false, lane);
      geo.ksh[0] = k0, geo.ksh[1] = k1, geo.vsh[0] = v0, geo.vsh[1] = v1;
    }
    auto k_segment = [&](int i, uint32_t (&seg)[Tr::KSEGW]) {
      normalize<Tr::KSEGW, Ge::KLD>(R.k[i], geo.ksh[i & 1], seg);
#pragma unroll
      for (int k = 0; k < Tr::KSEGW; ++k) __asm__ volatile("" : "+v"(seg[k]));
      next.k(geo, i, R);
    };
    auto v_segment = [&](int i, uint32_t (&seg)[Tr::VSEGW]) {
      normalize<Tr::VSEGW, Ge::VLD>(R.v[i], geo.vsh[i & 1], seg);
#pragma unroll
      for (int k = 0; k < Tr::VSEGW; ++k) __asm__ volatile("" : "+v"(seg[k]));
      next.v(geo, i, R);
    };
#pragma unroll
    for (int i = 0; i < PL::NML; ++i)
      if (PL::MSTAGE % 1024 == 0 || lane * 16 < PL::MSTAGE) *reinterpret_cast<uint4*>(kmeta + i * 1024 + lane * 16) = R.m[i];
    next.m(lane, R);
    if (it == 0) SEMKV_STAMP_FINE(16);
    const int ptile = POOL ? tile - nt0 : tile;
    const int nvalid = nrows - int64_t(ptile) * kSlots < kSlots ? int(nrows - int64_t(ptile) * kSlots) : kSlots;

    // ---- scores: C[(h, byte)][token] = q_h bytes . codes; lane holds token n, head r
    float lg[4];
    // metadata written above by other lanes of this wave
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    constexpr int NKM = BASE != 1 ? NG : 1, NVM = BASE != 1 ? NGV : 1;
    uint32_t km[4][NKM], vm[4][NVM];
    auto load_km = [&](int blk) {
      const int t = 16 * blk + n;
#pragma unroll
      for (int i = 0; i < NKM; ++i)
        km[blk][i] = BASE != 1 ? *reinterpret_cast<const uint32_t*>(kmeta + (i * kSlots + t) * 4)
                               : uint32_t(*reinterpret_cast<const uint16_t*>(kmeta + t * 2));
    };
    // one metadata word a token: all read here; several: a block's keys' words
    // with its products, the values' after the scores
    auto load_vm = [&]() {
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) {
        const int t = 16 * blk + n;
#pragma unroll
        for (int i = 0; i < NVM; ++i)
          vm[blk][i] = BASE != 1 ? *reinterpret_cast<const uint32_t*>(vmeta + (i * kSlots + t) * 4)
                                 : uint32_t(*reinterpret_cast<const uint16_t*>(vmeta + t * 2));
      }
    };
    if constexpr (NVM == 1) {
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) load_km(blk);
      load_vm();
    }
    // the score of token 16 blk + n from its products, one per query group,
    // in the softmax's base-2 scale: (q . c) 2^-e s + z (sum q) per group
    // (tq: rho ((q . c) 2^-e cS + cZ sum q)); masked tokens are set apart
    auto score = [&](int blk, const int4v (&acc)[NG]) {
      float x;
      if constexpr (BASE != 1) {
        x = hf(km[blk][0] >> 16) * zwsK[0];
#pragma unroll
        for (int i = 1; i < NG; ++i) x = fmaf(hf(km[blk][i] >> 16), zwsK[i], x);
#pragma unroll
        for (int i = 0; i < NG; ++i) x = fmaf(comb3_score(acc[i]) * qscK[i], hf(km[blk][i] & 0xFFFFu), x);
      } else {
        x = fmaf(comb3_score(acc[0]), qscK[0], zwsK[0]) * hf(uint16_t(km[blk][0]));
      }
      return x;
    };
    // software pipeline: the next block's table reads are in flight during
    // the current block's products
    int4v Bk[2][Tr::NCK];
    auto k_operands = [&](int i, int4v (&B)[Tr::NCK]) {
      uint32_t seg[Tr::KSEGW];
      k_segment(i, seg);
      chunk_operands<BASE, L, S, KFULL, Tr::KSEGW, Tr::NSK, Tr::NCK>(seg, kmask, lut, B);
    };
    auto v_operands = [&](int i, int4v (&B)[Tr::NCV]) {
      uint32_t seg[Tr::VSEGW];
      v_segment(i, seg);
      chunk_operands<BASE, L, S, VFULL, Tr::VSEGW, Tr::NSV, Tr::NCV>(seg, vmask, lut, B);
    };
    k_operands(0, Bk[0]);
    constexpr bool DEFER = NG == 1;          // score arithmetic after the first value segment's table reads are issued
    int4v acck[DEFER ? 4 : 1][NG];
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
      if constexpr (NVM > 1) load_km(blk);
      if (blk + 1 < 4) k_operands(blk + 1, Bk[(blk + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      int4v acc[NG];
      static_for<NG>([&](auto I) {
        constexpr int i = I.value;
        acc[i] = int4v{0, 0, 0, 0};
        static_for<Tr::NCK>([&](auto C) {
          constexpr int ch = C.value;
          if constexpr (Ge::pair_used(i, ch)) {              // else chunk ch holds no channel of group i
            int4v A;
            constexpr int pair = Ge::pair_of(i, ch);
            if constexpr (NG == 1) A = Aq[ch];
            else A = aq(pair);
            acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, Bk[blk & 1][ch], acc[i], 0, 0, 0);
          }
        });
      });
      if constexpr (DEFER) {
#pragma unroll
        for (int i = 0; i < NG; ++i) acck[blk][i] = acc[i];
      } else {
        lg[blk] = score(blk, acc);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // the first value operands do not depend on the softmax: their LDS round
    // trip overlaps it
    if constexpr (NVM > 1) load_vm();
    int4v Bv[2][Tr::NCV];
    v_operands(0, Bv[0]);
    if constexpr (DEFER) {
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) lg[blk] = score(blk, acck[blk]);
    }
    if (nvalid < kSlots) {                   // the pool's last record: slots past its rows
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) lg[blk] = 16 * blk + n < nvalid ? lg[blk] : -INFINITY;
    }
    if (it == 0) SEMKV_STAMP_FINE(17);
    // ---- online softmax (base 2) for head r over this record's 64 tokens,
    // rescaled lazily: the reference maximum st.m moves only when a score
    // passes it by more than 8 (weights up to 2^8 fit the fixed-point range),
    // or on the wave's first record
    const float mt = row_max16(max4(lg[0], lg[1], lg[2], lg[3]));
    const bool grow = !(mt <= st.m + 8.0f);
    const float m_new = grow ? mt : st.m;
    const float alpha = grow ? __builtin_amdgcn_exp2f(st.m - m_new) : 1.0f;
    st.m = m_new;
    float lsum = 0.0f, wmax = 0.0f;
    float wv[4][NGV][Ge::NPL];               // value weights of the lane's tokens
    float zadd[NGV];
#pragma unroll
    for (int i = 0; i < NGV; ++i) zadd[i] = 0.0f;
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
      const float p = __builtin_amdgcn_exp2f(lg[blk] - m_new);   // 0 for masked tokens
      lsum += p;
      if constexpr (BASE != 1) {
        const float pr = p * kR;
#pragma unroll
        for (int i = 0; i < NGV; ++i) {
          const uint32_t m = vm[blk][i];
          wv[blk][i][0] = pr * hf(m & 0xFFFFu);
          wmax = fmaxf(wmax, wv[blk][i][0]);
          zadd[i] = fmaf(pr, hf(m >> 16), zadd[i]);
        }
      } else {
        const float rho = hf(uint16_t(vm[blk][0]));
#pragma unroll
        for (int pl = 0; pl < Ge::NPL; ++pl) {
          wv[blk][0][pl] = p * rho * sc.cS * sc.wP[pl];
          wmax = fmaxf(wmax, wv[blk][0][pl]);
        }
        zadd[0] = fmaf(p * rho, sc.cZ, zadd[0]);
      }
    }
    // ---- the integer value sums hold weights of one scale and one reference
    // maximum: fold them into the float sums when the maximum moves or this
    // record's weights would not fit 21 bits (their rounding stays below
    // 2^21 - 1, so the top byte stays below 128), and re-pick the scale
    const bool flush = grow || wmax * st.qw >= 2097151.0f;
#ifdef SEMKV_TIMELINE
    st.nrec += 1;
#endif
    if (__builtin_amdgcn_ballot_w64(flush) != 0) {
#ifdef SEMKV_TIMELINE
      st.nflush += 1;
#endif
      wmax = row_max16(wmax);
      st.l *= alpha;
#pragma unroll
      for (int i = 0; i < NGV; ++i) st.z[i] *= alpha;
#pragma unroll
      for (int cb = 0; cb < 8; ++cb) {
        st.of[cb] = (st.of[cb] + comb3(st.cv[cb]) * st.qwi) * alpha;
        st.cv[cb] = int4v{0, 0, 0, 0};
      }
      const int E = __builtin_amdgcn_frexp_expf(wmax);          // wmax = f 2^E, f in [0.5, 1)
      const int e = wmax >= 1e-30f ? 19 - E : 100;
      st.qw = ldexpf(1.0f, e);
      st.qwi = ldexpf(1.0f, -e);
    }
    st.l += lsum;
#pragma unroll
    for (int i = 0; i < NGV; ++i) st.z[i] += zadd[i];
    if (it == 0) SEMKV_STAMP_FINE(18);

    // ---- values: C[(h, byte)][channel] += weights (tokens) x V codes, one
    // value group's int8 weights (byte s of rint(w qw) in row 4r + s) at a time
    int4v Aw[Tr::NCV];
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) {
      constexpr int CPG = BASE != 1 ? G / 16 : 8;          // channel blocks per value group
      if (cb % CPG == 0) {
        const int gv = cb / CPG;
#pragma unroll
        for (int blk = 0; blk < 4; ++blk)
#pragma unroll
          for (int pl = 0; pl < Ge::NPL; ++pl) {
            // the integer nearest w qw (< 2^21 - 1) in the low mantissa bits
            // of w qw + 1.5 2^23 (one rounding of the exact sum)
            const uint32_t q = __float_as_uint(fmaf(wv[blk][gv][pl], st.qw, 12582912.0f));
            uint8_t* w = pvw + pvwr[blk] + pl;
            w[0] = uint8_t(bits7<14>(q));
            w[16] = uint8_t(bits7<7>(q));
            w[32] = uint8_t(bits7<0>(q));
          }
        // weights written above by other lanes of this wave are read below
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int c = 0; c < Tr::NCV; ++c) {
          const uint4 v = *reinterpret_cast<const uint4*>(pvw + c * Ge::CHB + kg * Ge::KGS + n * 16);
          Aw[c] = __builtin_bit_cast(int4v, uint4v{v.x, v.y, v.z, v.w});
        }
      }
      if (cb + 1 < 8) v_operands(cb + 1, Bv[(cb + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < Tr::NCV; ++c) st.cv[cb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(Aw[c], Bv[cb & 1][c], st.cv[cb], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
#ifdef SEMKV_TIMELINE
    if (it == 0) SEMKV_STAMP(8);
#endif
    SEMKV_STAMP(3 + (it < 4 ? it : 4));
  }
}

// A wave's state in merged form: sums over the tokens of a row, the integer
// value sums folded in, the zero-point term added.  Lane (n, r) holds head r
// at channels 16 cb + n.
template <int BASE, int G, class PL>
__device__ void wave_finish(Shared<PL>& sm, WaveState<PL::NGV>& st) {
  constexpr int NGV = PL::NGV;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 15, r = lane >> 4;
  st.l = row_sum16(st.l);
#pragma unroll
  for (int i = 0; i < NGV; ++i) st.z[i] = row_sum16(st.z[i]);
  if (n == 0) {
#pragma unroll
    for (int i = 0; i < NGV; ++i) sm.zc[wave][r][i] = st.z[i];
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  Fin* f = wave_fin(sm, wave);
  if (n == 0) {
    f->m[r] = st.m;
    f->l[r] = st.l;
  }
#pragma unroll
  for (int cb = 0; cb < 8; ++cb) {
    const int ch = 16 * cb + n;
    f->o[r][ch] = st.of[cb] + comb3(st.cv[cb]) * st.qwi + sm.zc[wave][r][BASE != 1 ? ch / G : 0];
  }
}

// Partials cross workgroups (and XCDs, whose L2 caches are not coherent with
// each other): they are written with agent-scope atomic stores and read with
// the same coherent cache policy (sc1), so neither side needs a cache
// write-back or invalidate.
__device__ inline void st_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}


// The unnormalized Walsh-Hadamard transform H x of the 4 rows of 128 values
// held one per thread of the workgroup (thread t: row t >> 7, entry t & 127).
// Stages 1..32 pair lanes of one wave (DPP quad permutes for 1 and 2, lane
// exchanges for the rest); stage 64 pairs the two waves of a row through the
// LDS buffer xch.  Each stage computes the lower entry as lower + upper and the
// upper as lower - upper, the radix-2 butterflies in the usual order.  Every
// thread of the workgroup calls it; xch is free again when it returns.
__device__ inline float fwht_rows(float x, float (*xch)[kD]) {
  const int tid = threadIdx.x, lane = tid & 63;
  float p = dpp<0xB1>(x);                                  // lane ^ 1
  x = (lane & 1) ? p - x : x + p;
  p = dpp<0x4E>(x);                                        // lane ^ 2
  x = (lane & 2) ? p - x : x + p;
#pragma unroll
  for (int hs = 4; hs < 64; hs <<= 1) {
    p = __shfl_xor(x, hs);
    x = (lane & hs) ? p - x : x + p;
  }
  xch[tid >> 7][tid & 127] = x;
  __syncthreads();
  p = xch[tid >> 7][(tid & 127) ^ 64];
  x = (tid & 64) ? p - x : x + p;
  __syncthreads();
  return x;
}

// fp16 tail of generated tokens (1 to 64 rows): its attention state goes to
// sm.tfin.  Runs after the workgroup's records, when the decode tables and the
// query operands are free: the K and V tails are staged in the table area
// (both in one round trip), then every thread works:
// 8 threads per row for the scores, one wave per head for the softmax, one
// thread per (head, channel) for the values.
template <int BASE, class PL>
__device__ void tail_split(const DecodeArgs& a, Shared<PL>& sm, int b, int layer, int kvh) {
  static_assert(sizeof(sm.lut) >= 2 * kSlots * kD * 2, "tail staging");
  static_assert(PL::NT == 4 * kD, "one thread per (head, channel)");
  const PoolGeom& g = a.g;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nt = a.n_tail;
  TailScratch& ts = sm.ts;
  const uint16_t* kt = a.tail + ((((int64_t(b) * g.n_layers + layer) * g.n_kv_heads + kvh) * 2) * kSlots) * kD;
  const uint16_t* vt = kt + kSlots * kD;
  uint4* kl = reinterpret_cast<uint4*>(sm.lut);             // [64 rows][16 pieces of 8 fp16]
  uint4* vl = kl + kSlots * kD / 8;
  {
    // piece i (8 channels of row i / 16); the two pieces of a thread: i0, i1
    const int i0 = tid, i1 = tid + PL::NT;
    const bool in0 = (i0 >> 4) < nt, in1 = (i1 >> 4) < nt;
    uint4 ka = make_uint4(0u, 0u, 0u, 0u), kb = ka, va = ka, vb2 = ka;
    if (in0) {
      ka = reinterpret_cast<const uint4*>(kt)[i0];
      va = reinterpret_cast<const uint4*>(vt)[i0];
    }
    if (in1) {
      kb = reinterpret_cast<const uint4*>(kt)[i1];
      vb2 = reinterpret_cast<const uint4*>(vt)[i1];
    }
    if (in0) {
      kl[i0] = ka;
      vl[i0] = va;
    }
    if (in1) {
      kl[i1] = kb;
      vl[i1] = vb2;
    }
  }
  __syncthreads();
  // scores: thread (row t, channel block j of 16) sums its block for the 4
  // heads; the 8 threads of a row are 8 neighbouring lanes (scalars only:
  // small arrays here would be placed in memory)
  {
    const int t = tid >> 3, j = tid & 7;
    uint4 k0 = make_uint4(0u, 0u, 0u, 0u), k1 = k0;
    if (t < nt) {
      k0 = kl[t * 16 + 2 * j];
      k1 = kl[t * 16 + 2 * j + 1];
    }
    auto dot4 = [](const float* q, uint32_t w0, uint32_t w1, float x) {
      const float4 qv = *reinterpret_cast<const float4*>(q);
      x = fmaf(qv.x, hf(uint16_t(w0 & 0xFFFFu)), x);
      x = fmaf(qv.y, hf(uint16_t(w0 >> 16)), x);
      x = fmaf(qv.z, hf(uint16_t(w1 & 0xFFFFu)), x);
      return fmaf(qv.w, hf(uint16_t(w1 >> 16)), x);
    };
    auto dot16 = [&](int h) {
      const float* q = &sm.qorig[h][16 * j];
      float x = dot4(q, k0.x, k0.y, 0.0f);
      x = dot4(q + 4, k0.z, k0.w, x);
      x = dot4(q + 8, k1.x, k1.y, x);
      return dot4(q + 12, k1.z, k1.w, x);
    };
    float d0 = dot16(0), d1 = dot16(1), d2 = dot16(2), d3 = dot16(3);
#pragma unroll
    for (int m = 1; m < 8; m <<= 1) {
      d0 += __shfl_xor(d0, m);
      d1 += __shfl_xor(d1, m);
      d2 += __shfl_xor(d2, m);
      d3 += __shfl_xor(d3, m);
    }
    if (t < nt && j == 0) {
      constexpr float sc = kLog2e * kRsqrtD;
      ts.lg[0][t] = d0 * sc;
      ts.lg[1][t] = d1 * sc;
      ts.lg[2][t] = d2 * sc;
      ts.lg[3][t] = d3 * sc;
    }
  }
  __syncthreads();
  // softmax: wave h takes head h, lane t token t
  if (wave < 4) {
    const float x = lane < nt ? ts.lg[wave][lane] : -INFINITY;
    float M = x;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) M = fmaxf(M, __shfl_xor(M, m));
    const float p = lane < nt ? __builtin_amdgcn_exp2f(x - M) : 0.0f;
    float ssum = p;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) ssum += __shfl_xor(ssum, m);
    if (lane < nt) ts.lg[wave][lane] = p;
    if (lane == 0) {
      ts.mx[wave] = M;
      ts.sum[wave] = ssum;
    }
  }
  __syncthreads();
  const int h = tid >> 7, c = tid & 127;
  const uint16_t* vrow = reinterpret_cast<const uint16_t*>(vl);
  float o = 0.0f;
  for (int t = 0; t < nt; ++t) o = fmaf(ts.lg[h][t], hf(vrow[t * kD + c]), o);
  if (BASE != 0) {                           // into the rotated domain: H (sign . o) / 128
    const uint32_t* sw = g.signs + (int64_t(layer) * g.n_kv_heads + kvh) * 4;
    o = ((sw[c >> 5] >> (c & 31)) & 1u) ? -o : o;
    o = fwht_rows(o, ts.o) * (1.0f / 128.0f);
  }
  sm.tfin.o[h][c] = o;
  if (c == 0) {
    sm.tfin.m[h] = ts.mx[h];
    sm.tfin.l[h] = ts.sum[h];
  }
}

// Merge of the partials of one (layer, sequence, kv head), run by the last
// workgroup to finish: log-sum-exp over the partials, then for the rotated
// bases the inverse rotation o = sign . H o_rot.  vb indexes the launch's
// (layer, sequence) pairs: partials, counters, queries and outputs.
template <int BASE, class PL>
__device__ void merge_splits(const DecodeArgs& a, Shared<PL>& sm, int vb, int layer, int kvh) {
  const int tid = threadIdx.x;
  const int ns = a.nsplit;
  const float* unit = a.ws + (int64_t(vb) * a.g.n_kv_heads + kvh) * ns * 4 * kPartial;
  // thread (head h, quarter q, channel quad cq) takes the splits s = q, q+4,
  // ... with 16-byte loads at the coherent level (cache policy sc1, as the
  // agent-scope loads), then the four quarters merge in LDS
  const int h = tid >> 7, q = (tid >> 5) & 3, cq = tid & 31;
  // the sign of this thread's output channel (rotated bases), loaded first
  const uint32_t sbits = BASE != 0 ? a.g.signs[(int64_t(layer) * a.g.n_kv_heads + kvh) * 4 + ((tid & 127) >> 5)] : 0u;
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(unit), 0, ns * 4 * kPartial * 4, kBufferWord3);
  constexpr int kCoherent = 16;              // sc1
  constexpr int kBatch = 8;
  float M = -INFINITY, Lsum = 0.0f;
  float4v o = float4v{0, 0, 0, 0};
  for (int s0 = q; s0 < ns; s0 += 4 * kBatch) {
    float mv[kBatch], lv[kBatch];
    float4v x[kBatch];
    // all loads issued at once, unconditionally (one round trip): a split
    // past the last reads zeros through the buffer descriptor and is given
    // m = -inf afterwards
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int sp = s0 + 4 * k;
      const int off = (sp * 4 + h) * kPartial * 4;
      const auto ml = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, kCoherent);
      mv[k] = __uint_as_float(ml[0]);
      lv[k] = __uint_as_float(ml[1]);
      x[k] = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16 + 16 * cq, 0, kCoherent));
    }
#pragma unroll
    for (int k = 0; k < kBatch; ++k) mv[k] = s0 + 4 * k < ns ? mv[k] : -INFINITY;
    float Mn = M;
#pragma unroll
    for (int k = 0; k < kBatch; ++k) Mn = fmaxf(Mn, mv[k]);
    const float keep = M == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(M - Mn);
    Lsum *= keep;
    o *= keep;
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const float sc = mv[k] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mv[k] - Mn);
      Lsum += lv[k] * sc;
      o += x[k] * sc;
    }
    M = Mn;
  }
  struct Quarters { float m[4][4], l[4][4]; float4v o[4][4][32]; };
  static_assert(sizeof(Quarters) <= sizeof(sm.pv), "merge scratch");
  Quarters& qs = *reinterpret_cast<Quarters*>(&sm.pv[0][0]);
  if (cq == 0) {
    qs.m[h][q] = M;
    qs.l[h][q] = Lsum;
  }
  qs.o[h][q][cq] = o;
  __syncthreads();
  const int c = tid & 127;
  float Mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < 4; ++k) Mx = fmaxf(Mx, qs.m[h][k]);
  float L = 0.0f, O = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float sc = qs.m[h][k] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(qs.m[h][k] - Mx);
    L += qs.l[h][k] * sc;
    O += qs.o[h][k][c >> 2][c & 3] * sc;
  }
  float r = O / L;
  if (BASE != 0) {
    r = fwht_rows(r, sm.ts.o);
    r = ((sbits >> (c & 31)) & 1u) ? -r : r;
  }
  a.out[((int64_t(vb) * a.g.n_kv_heads + kvh) * 4 + h) * kD + c] = r;
}

template <int BASE, int LH, int LL, int G>
__global__ __launch_bounds__((Plan<BASE, LH, LL, G>::NT)) void decode_kernel(DecodeArgs a) {
  using PL = Plan<BASE, LH, LL, G>;
  constexpr int NW = PL::NW, NT = PL::NT;
  __shared__ Shared<PL> sm;
  static_assert(sizeof(Shared<PL>) <= 160 * 1024, "LDS");
  // blockIdx.z = (layer of the launch) x batch + sequence: an all-layers
  // launch covers n_layers_launched layers from a.layer
  const int split = blockIdx.x, kvh = blockIdx.y, vb = blockIdx.z;
  const int li = a.n_layers_launched > 1 ? vb / a.g.batch : 0, b = vb - li * a.g.batch, layer = a.layer + li;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const PoolGeom& g = a.g;
  SEMKV_STAMP(0);

  // ---- the query first (the longest wait of the prologue), one (head,
  // channel) per thread, so no branch forces a wait on the load
  const int h = tid >> 7, c = tid & 127;
  const uint16_t qbits = a.q[((int64_t(vb) * g.n_kv_heads * 4) + kvh * 4 + h) * kD + c];
  // rotated bases: the sign word of this thread's channel, in flight with the query
  const uint32_t qsign = BASE != 0 ? g.signs[(int64_t(layer) * g.n_kv_heads + kvh) * 4 + (c >> 5)] : 0u;

  // ---- fused append (Alg. 2): the workgroup that attends over the fp16 tail
  // first stores this layer's new K/V row in it, as its last row (read back
  // by the same workgroup after the barriers below); placed before the record
  // loads, so that its wait covers the query load only
  if (a.k_new != nullptr && split == a.nsplit - 1 && tid < 2 * kD / 2) {
    const int kv = tid >> 6, w = tid & 63;                // 64 dwords each of K and V
    const uint32_t* src = reinterpret_cast<const uint32_t*>((kv ? a.v_new : a.k_new) + (int64_t(b) * g.n_kv_heads + kvh) * kD);
    uint32_t* dst = reinterpret_cast<uint32_t*>(
        a.tail + ((((int64_t(b) * g.n_layers + layer) * g.n_kv_heads + kvh) * 2 + kv) * kSlots + (a.n_tail - 1)) * kD);
    dst[w] = src[w];
  }

  // ---- decode tables, from memory (before the record's loads, so that they
  // are not waited for with it)
  constexpr int NTH = (PL::LUTH / 4 + NT - 1) / NT, NTL = (PL::LUTL / 4 + NT - 1) / NT;
  uint4 th[NTH], tl[NTL];
  // the operands' pad slots and unused rows are zero
  for (int i = tid; i < PL::NPAIRS * 64; i += NT) (&sm.aq[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
  for (int i = tid; i < int(sizeof(sm.pv)) / 16; i += NT) reinterpret_cast<uint4*>(&sm.pv[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
  for (int k = 0; k < NTH; ++k) th[k] = lut_piece<BASE, LH, PL::RH>(tid + k * NT < PL::LUTH / 4 ? tid + k * NT : 0);
#pragma unroll
  for (int k = 0; k < NTL; ++k) tl[k] = lut_piece<BASE, LL, PL::RL>(tid + k * NT < PL::LUTL / 4 ? tid + k * NT : 0);
  // ---- this wave's tiles: first, first + stride, ... (high pool first),
  // and the first of them in flight (a wave without records loads tile 0,
  // unused)
  const int nt0 = a.tiles[0], stride = a.nsplit * NW;
  const int first = wave * a.nsplit + split;
  const int count = a.full[1] + (first < a.left[1] ? 1 : 0), nhi = a.full[0] + (first < a.left[0] ? 1 : 0);
  const uint8_t* unit = g.pools + unit_offset(g, b, layer, kvh);
  const int tile0 = count > 0 ? first : 0;
  // where the softmax lanes' weights go in the wave's first pool
  uint4 pvwq = *reinterpret_cast<const uint4*>(nhi > 0 ? kPoolConst<BASE, LH>.pvw[lane] : kPoolConst<BASE, LL>.pvw[lane]);
  LaneGeo geo = {};
  if (count > 0) geo = lane_geo<BASE, LH, LL>(tile0 < nt0, lane);
  Record<PL> R;
  {
    const RecordSource<BASE, LH, LL, G, PL> rec(g, unit, tile0, nt0, count > 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) rec.k(geo, i, R);
    rec.m(lane, R);
#pragma unroll
    for (int i = 0; i < 8; ++i) rec.v(geo, i, R);
  }

  {
    uint4* d = reinterpret_cast<uint4*>(sm.lut);
#pragma unroll
    for (int k = 0; k < NTH; ++k)
      if (tid + k * NT < PL::LUTH / 4) d[tid + k * NT] = th[k];
#pragma unroll
    for (int k = 0; k < NTL; ++k)
      if (tid + k * NT < PL::LUTL / 4) d[PL::LUTH / 4 + tid + k * NT] = tl[k];
  }
  SEMKV_STAMP_FINE(19);
  float xq = hf(qbits);
  sm.qorig[h][c] = xq;
  if (BASE != 0) xq = ((qsign >> (c & 31)) & 1u) ? -xq : xq;
  SEMKV_STAMP_FINE(20);
  if (BASE != 0) xq = fwht_rows(xq, sm.ts.o);    // rotate: H (sign . q)
  query_runs(xq, h, c, sm);                      // the query the scores use: its runs
  SEMKV_STAMP_FINE(21);
  __syncthreads();
  scatter_query<BASE, LH, LL, G>(a, sm, xq, h, c);
  __syncthreads();
  SEMKV_STAMP(1);

  // ---- this wave's records
  WaveState<PL::NGV> st;
  st.m = -INFINITY;
  st.l = 0.0f;
#pragma unroll
  for (int i = 0; i < PL::NGV; ++i) st.z[i] = 0.0f;
  st.qw = st.qwi = 1.0f;
#pragma unroll
  for (int cb = 0; cb < 8; ++cb) {
    st.of[cb] = 0.0f;
    st.cv[cb] = int4v{0, 0, 0, 0};
  }
  SEMKV_STAMP(2);
  if (nhi > 0) run_pool<BASE, LH, LL, G, 0>(a, sm, st, unit, nt0, first, stride, 0, nhi, count, R, geo, pvwq);
  if (count > nhi) run_pool<BASE, LH, LL, G, 1>(a, sm, st, unit, nt0, first, stride, nhi, count, count, R, geo, pvwq);
  SEMKV_STAMP(9);
#ifdef SEMKV_TIMELINE
  timeline_put(14, uint32_t(st.nflush));
  timeline_put(15, uint32_t(st.nrec));
#endif
  wave_finish<BASE, G>(sm, st);
  __syncthreads();
  const bool tail = split == a.nsplit - 1 && a.n_tail > 0;
  if (tail) {
    tail_split<BASE>(a, sm, b, layer, kvh);
    __syncthreads();
  }

  // ---- workgroup partial: merge of the waves' (and the tail's) states
  SEMKV_STAMP(10);
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < NW; ++w) M = fmaxf(M, wave_fin(sm, w)->m[h]);
  if (tail) M = fmaxf(M, sm.tfin.m[h]);
  float Lsum = 0.0f, o = 0.0f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const Fin* f = wave_fin(sm, w);
    const float sc = f->m[h] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(f->m[h] - M);
    Lsum += f->l[h] * sc;
    o += f->o[h][c] * sc;
  }
  if (tail) {
    const float sc = sm.tfin.m[h] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(sm.tfin.m[h] - M);
    Lsum += sm.tfin.l[h] * sc;
    o += sm.tfin.o[h][c] * sc;
  }
  float* dst = a.ws + ((int64_t(vb) * g.n_kv_heads + kvh) * a.nsplit + split) * 4 * kPartial + h * kPartial;
  if (c == 0) {
    st_agent(dst, M);
    st_agent(dst + 1, Lsum);
  }
  st_agent(dst + 4 + c, o);
  // every thread's partial stores are complete (at the coherent level) before
  // the workgroup's counter increment; the last workgroup reads them after it
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  SEMKV_STAMP(11);
  if (tid == 0) {
    uint32_t* ctr = a.counters + (vb * g.n_kv_heads + kvh) * kCounterStride;
    const uint32_t old = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sm.last = old == uint32_t(a.nsplit - 1);
    if (sm.last) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  SEMKV_STAMP(12);
  if (!sm.last) return;
  merge_splits<BASE>(a, sm, vb, layer, kvh);
#ifdef SEMKV_TIMELINE
  __syncthreads();
  SEMKV_STAMP(13);
#endif
}

template <int BASE, int LH, int LL, int G>
int occupancy() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, decode_kernel<BASE, LH, LL, G>, Plan<BASE, LH, LL, G>::NT, 0) != hipSuccess)
    return 1;
  return n > 0 ? n : 1;
}

template <int BASE, int LH, int LL, int G>
int launch_g(const DecodeArgs& a, hipStream_t st) {
  using PL = Plan<BASE, LH, LL, G>;
  // slot s of stride = nsplit x NW holds tiles s, s + stride, ...: their
  // number, all and of the high pool, without a division in every wave
  DecodeArgs d = a;
  const int stride = a.nsplit * PL::NW;
  d.tiles[0] = int((a.n_rows[0] + kSlots - 1) / kSlots);
  d.tiles[1] = d.tiles[0] + int((a.n_rows[1] + kSlots - 1) / kSlots);
  for (int i = 0; i < 2; ++i) {
    d.full[i] = d.tiles[i] / stride;
    d.left[i] = d.tiles[i] % stride;
  }
  dim3 grid(a.nsplit, a.g.n_kv_heads, a.g.batch * a.n_layers_launched);
  hipLaunchKernelGGL((decode_kernel<BASE, LH, LL, G>), grid, dim3(PL::NT), 0, st, d);
  return hipGetLastError() == hipSuccess ? 0 : -5;
}

template <int BASE, int LH, int LL>
int launch_dec(const DecodeArgs& a, hipStream_t st) {
  if constexpr (BASE == 1) {
    return launch_g<BASE, LH, LL, 128>(a, st);
  } else {
    if (a.g.G == 128) return launch_g<BASE, LH, LL, 128>(a, st);
    if (a.g.G == 64) return launch_g<BASE, LH, LL, 64>(a, st);
    return launch_g<BASE, LH, LL, 32>(a, st);
  }
}

template <int BASE, int LH, int LL>
int occ_dec(int G) {
  if constexpr (BASE == 1) {
    return occupancy<BASE, LH, LL, 128>();
  } else {
    if (G == 128) return occupancy<BASE, LH, LL, 128>();
    if (G == 64) return occupancy<BASE, LH, LL, 64>();
    return occupancy<BASE, LH, LL, 32>();
  }
}

}  // namespace

int launch_decode(const DecodeArgs& a, hipStream_t s) {
  const int B = a.g.base, LH = a.g.L[0], LL = a.g.L[1];
  if (B == 0 && LH == 6 && LL == 5) return launch_dec<0, 6, 5>(a, s);
  if (B == 0 && LH == 5 && LL == 4) return launch_dec<0, 5, 4>(a, s);
  if (B == 0 && LH == 6 && LL == 4) return launch_dec<0, 6, 4>(a, s);
  if (B == 0 && LH == 4 && LL == 3) return launch_dec<0, 4, 3>(a, s);
  if (B == 0 && LH == 5 && LL == 3) return launch_dec<0, 5, 3>(a, s);
  if (B == 0 && LH == 6 && LL == 3) return launch_dec<0, 6, 3>(a, s);
  if (B == 1 && LH == 4 && LL == 3) return launch_dec<1, 4, 3>(a, s);
  if (B == 2 && LH == 6 && LL == 5) return launch_dec<2, 6, 5>(a, s);
  if (B == 2 && LH == 5 && LL == 4) return launch_dec<2, 5, 4>(a, s);
  // the rest of the level grid (uniform sweeps, Sec. 4.2): metadata per row only
  if (a.g.G == 128) {
    if (B == 0 && LH == 8 && LL == 7) return launch_g<0, 8, 7, 128>(a, s);
    if (B == 0 && LH == 7 && LL == 6) return launch_g<0, 7, 6, 128>(a, s);
    if (B == 0 && LH == 3 && LL == 2) return launch_g<0, 3, 2, 128>(a, s);
    if (B == 2 && LH == 8 && LL == 7) return launch_g<2, 8, 7, 128>(a, s);
    if (B == 2 && LH == 7 && LL == 6) return launch_g<2, 7, 6, 128>(a, s);
    if (B == 2 && LH == 3 && LL == 2) return launch_g<2, 3, 2, 128>(a, s);
  }
  return -2;
}

int decode_blocks_per_cu(int base, int LH, int LL, int G) {
  if (base == 0 && LH == 6 && LL == 5) return occ_dec<0, 6, 5>(G);
  if (base == 0 && LH == 5 && LL == 4) return occ_dec<0, 5, 4>(G);
  if (base == 0 && LH == 6 && LL == 4) return occ_dec<0, 6, 4>(G);
  if (base == 0 && LH == 4 && LL == 3) return occ_dec<0, 4, 3>(G);
  if (base == 0 && LH == 5 && LL == 3) return occ_dec<0, 5, 3>(G);
  if (base == 0 && LH == 6 && LL == 3) return occ_dec<0, 6, 3>(G);
  if (base == 1 && LH == 4 && LL == 3) return occ_dec<1, 4, 3>(G);
  if (base == 2 && LH == 6 && LL == 5) return occ_dec<2, 6, 5>(G);
  if (base == 2 && LH == 5 && LL == 4) return occ_dec<2, 5, 4>(G);
  if (G == 128) {
    if (base == 0 && LH == 8 && LL == 7) return occupancy<0, 8, 7, 128>();
    if (base == 0 && LH == 7 && LL == 6) return occupancy<0, 7, 6, 128>();
    if (base == 0 && LH == 3 && LL == 2) return occupancy<0, 3, 2, 128>();
    if (base == 2 && LH == 8 && LL == 7) return occupancy<2, 8, 7, 128>();
    if (base == 2 && LH == 7 && LL == 6) return occupancy<2, 7, 6, 128>();
    if (base == 2 && LH == 3 && LL == 2) return occupancy<2, 3, 2, 128>();
  }
  return 1;
}


}  // namespace semkv

#ifdef SEMKV_TIMELINE
#include "semkv.h"
#include "semkv_timeline.h"
extern "C" int semkv_timeline_read(void* host, size_t bytes) {
  if (host == nullptr || bytes != sizeof(semkv::g_timeline)) return SEMKV_EINVAL;
  return hipMemcpyFromSymbol(host, HIP_SYMBOL(semkv::g_timeline), bytes) == hipSuccess ? SEMKV_OK : SEMKV_EHIP;
}
#endif
