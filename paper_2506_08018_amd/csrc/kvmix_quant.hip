// Quantize-and-pack, dequantize (test helper) and window-append kernels for gfx950.
//
// Paper Sec. 3.2.1 (Keys grouped per channel, Values per token), Sec. 3.2.2 (group-wise
// min/max quantizer, steps 1-4, 3-bit block of 11 with q_max = 3 for its 11th element),
// Sec. 3.4 item 1 (quantize and append into the historical cache in one kernel).
//
// Built with -ffp-contract=off: the code arithmetic is specified operation by operation
// (fp32 subtract, IEEE divide, round-half-even) so that codes are reproducible bit for bit.
#include <type_traits>
#include "kvmix_common.hpp"

namespace kvmix {

namespace {

template <int BITS>
__device__ __forceinline__ float step_of(float s, int i) {
  if (BITS == 3 && (i == 10 || i == 21)) return (s * 7.0f) / 3.0f;  // same range over q_max = 3
  return s;
}

template <int BITS>
__device__ __forceinline__ int qmax_of(int i) {
  if (BITS == 3 && (i == 10 || i == 21)) return 3;
  return (1 << BITS) - 1;
}

// value of lane (l ^ 1) / (l ^ 2) of each quad (every source lane exists: the last argument lets the move fold into the OR that uses it)
__device__ __forceinline__ uint32_t quad_x1(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true); }
__device__ __forceinline__ uint32_t quad_x2(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true); }
// value of lane (l ^ 4): of a row of 16, by a mirror of its halves of 8 (l ^ 7), then of quads (l ^ 3)
__device__ __forceinline__ uint32_t lane_x4(uint32_t v) {
  const int m = __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);
  return (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x1B, 0xf, 0xf, true);
}

// Codes travel as "biased codes": the bit pattern of the float 1.5 * 2^23 + code, i.e. kBias + code. Adding
// 1.5 * 2^23 to a value in [0, 2^22) rounds it to an integer (ties to even) in one operation and leaves that
// integer in the low mantissa bits; the low 16 bits of kBias are zero.
constexpr float kMagic = 12582912.0f;
constexpr uint32_t kBias = 0x4B400000u;

// range / q_max, correctly rounded: a product with the rounded reciprocal, its exact remainder and one correction. Equal to the IEEE
// quotient for 3, 7 and 15 at every fp32 significand (tried one by one in tests/test_quantizer_division.py); a range of fp16 numbers is far
// from the ends of the exponent range.
template <int BITS>
__device__ __forceinline__ float over_qmax(float range) {
  if constexpr (BITS == 1) return range;
  constexpr float kQ = (float)((1 << BITS) - 1), kInv = 1.0f / kQ;
  const float q = range * kInv;
  return __builtin_fmaf(__builtin_fmaf(-kQ, q, range), kInv, q);
}

// Scale, minimum and bracketing reciprocal steps of one group from its extremes (fp32 images of fp16 values).
struct GroupParams { float mn, s, inv_lo, inv_hi, inv2_lo, inv2_hi; bool slow; uint16_t scale_h, zero_h; };
template <int BITS>
__device__ __forceinline__ GroupParams group_params(float mn, float mx) {
  GroupParams g;
  if (mn == 0.0f) mn = 0.0f;                      // -0 -> +0
  float range = mx - mn;
  if (range == 0.0f) range = 0.0f;                // a zero-range group stores scale +0 whatever the signs of its zeros
  const bool infinite = range == __builtin_inff();       // (outside what the entry points promise anything for: scale infinity, codes 0)
  const float s32 = infinite ? range : over_qmax<BITS>(range);
  // round-to-nearest-even; a 1-bit step (the range itself) beyond the fp16 range is stored as the largest fp16 number
  const half_t sh = (half_t)(BITS == 1 ? fminf(s32, 65504.0f) : s32);
  g.mn = mn;
  g.s = (float)sh;
  g.scale_h = __builtin_bit_cast(uint16_t, sh);
  g.zero_h = __builtin_bit_cast(uint16_t, (half_t)mn);
  // 1 / s_i bracketed from below and above by 2^-19 relative: far more than the errors of the hardware
  // reciprocal (1 ulp), of the products below and of the fp32 rounding of the true quotient taken together
  // (under 2^-21). 0 for a zero scale: every product, hence every code, is then 0.
  const float inv = g.s != 0.0f ? __builtin_amdgcn_rcpf(g.s) : 0.0f;
  g.inv_lo = inv * (1.0f - 0x1p-19f);
  g.inv_hi = inv * (1.0f + 0x1p-19f);
  g.inv2_lo = g.inv_lo * (3.0f / 7.0f);          // the step s * 7 / 3 of the two 2-bit elements of a 3-bit group
  g.inv2_hi = g.inv_hi * (3.0f / 7.0f);
  // Only when the stored scale is a rounded image of range / q_max to fp16's full precision is every quotient
  // at most q_max * (1 + 2^-11) and the upper clip idle. A subnormal scale (rounded with a larger relative error)
  // or a saturated 1-bit scale sends the whole group down the path that clips.
  g.slow = (g.s != 0.0f && g.s < 0x1p-14f) || (BITS == 1 && g.s >= 65504.0f) || infinite;
  return g;
}

// Extremes of 32 fp16 numbers per half, 16 pairs from one source and 16 from another or 32 of one: three operands at a time. The
// instructions hand a NaN on, unlike the ones that take two operands: nan says that there is one (the group then goes the slow way,
// with the extremes of the others).
__device__ __forceinline__ uint32_t min3(uint32_t a, uint32_t b, uint32_t c) { uint32_t r; asm("v_pk_minimum3_f16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c)); return r; }
__device__ __forceinline__ uint32_t max3(uint32_t a, uint32_t b, uint32_t c) { uint32_t r; asm("v_pk_maximum3_f16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c)); return r; }
template <int N>
__device__ __forceinline__ void extremes(const uint32_t (&x)[N], half2_t& mn, half2_t& mx, bool& nan) {
  uint32_t lo = min3(x[0], x[1], x[2]), hi = max3(x[0], x[1], x[2]);
#pragma unroll
  for (int i = 3; i < N; i += 2) {
    lo = min3(lo, x[i], x[i + 1 < N ? i + 1 : i]);
    hi = max3(hi, x[i], x[i + 1 < N ? i + 1 : i]);
  }
  mn = __builtin_bit_cast(half2_t, lo);
  mx = __builtin_bit_cast(half2_t, hi);
  nan = !(mx[0] == mx[0] && mx[1] == mx[1]);
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(nan) != 0, 0)) {
    mn = mx = __builtin_bit_cast(half2_t, x[0]);
#pragma unroll
    for (int i = 1; i < N; i++) {
      mn = __builtin_elementwise_min(mn, __builtin_bit_cast(half2_t, x[i]));
      mx = __builtin_elementwise_max(mx, __builtin_bit_cast(half2_t, x[i]));
    }
  }
}

// code = clamp(rint((x - mn) / s_i)) with the IEEE quotient rounded to fp32 first. The quotient q lies strictly
// between (x - mn) * inv_lo and (x - mn) * inv_hi, and so does its fp32 image; rounding to an integer is
// monotone, so when both products round to the same integer (each with the single rounding of a fused
// multiply-add onto kMagic), that integer is the code. x >= mn always, and the upper clip is idle but for the groups marked slow.
// The other cases, the quotient within 2^-18 relative of k + 1/2, are in practice exact ties (fp16 inputs over an fp16 step: one
// element in 4000, so that one batch of 1024 in five has one): resolve_tie recognises those by the exact remainder d - (k + 1/2) s,
// which a fused multiply-add gives without rounding, and takes the even one of k and k + 1. What is left, next to never, is compared with
// the two ends of the range of quotients that fp32 rounds to k + 1/2 (settle). No division: when every tie went through one, the
// divisions took a quarter of the time of a tile.
// d: x - mn in fp32; i: index of the element inside its group. All return biased codes.
template <int BITS> constexpr bool two_bit(int i) { return BITS == 3 && (i == 10 || i == 21); }
template <int BITS>
__device__ __forceinline__ uint32_t code_below(float d, const GroupParams& g, int i) {
  return __builtin_bit_cast(uint32_t, __builtin_fmaf(d, two_bit<BITS>(i) ? g.inv2_lo : g.inv_lo, kMagic));
}
template <int BITS>
__device__ __forceinline__ uint32_t code_above(float d, const GroupParams& g, int i) {
  return __builtin_bit_cast(uint32_t, __builtin_fmaf(d, two_bit<BITS>(i) ? g.inv2_hi : g.inv_hi, kMagic));
}
// An element of which the lanes in `near` are next to k + 1/2 (lo the code below): bit `at` of open is set where it is no exact tie.
// (The step of a 2-bit element of a 3-bit group is itself rounded: its remainder does not tell.)
template <int BITS>
__device__ __forceinline__ uint32_t resolve_tie(uint32_t lo, float d, const GroupParams& g, int i, int at, bool near, uint32_t& open) {
  const float rest = __builtin_fmaf((__builtin_bit_cast(float, lo) - kMagic) + 0.5f, -g.s, d);
  open |= near & (two_bit<BITS>(i) | (rest != 0.0f)) ? 1u << at : 0u;
  return lo + (near ? lo & 1u : 0u);
}
// x - mn in fp32 of the low / high half of a pair of fp16 numbers: x * 1 - mn, rounded once like the subtraction, with the conversion in
// the same instruction
template <int HALF>
__device__ __forceinline__ float diff(uint32_t pair, float mn) {
  float d;
  if constexpr (HALF == 0) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,0]" : "=v"(d) : "v"(pair), "v"(mn));
  else asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d) : "v"(pair), "v"(mn));
  return d;
}
// fp32 rounds a quotient to h = k + 1/2 when it is at most half a unit in the last place of h away (half that below h = 1/2, where the
// spacing changes); the ends times the step have at most 49 bits, so that the comparisons in 64 bits are exact.
__device__ __forceinline__ uint32_t settle(float d, float inv_lo, float step) {
  const uint32_t lo = __builtin_bit_cast(uint32_t, __builtin_fmaf(d, inv_lo, kMagic));
  const float h = (__builtin_bit_cast(float, lo) - kMagic) + 0.5f;
  const double half = (double)__builtin_bit_cast(float, __builtin_bit_cast(uint32_t, h) & 0x7f800000u) * 0x1p-24;
  const double s = (double)step;
  uint32_t code = lo + (lo & 1u);
  if ((double)d > s * ((double)h + half)) code = lo + 1u;
  if ((double)d < s * ((double)h - (h == 0.5f ? 0.5 * half : half))) code = lo;
  return code;
}
// A lane's batch of 16 elements: code[at], of element first + at of the group g0 (Values), whose fp16 number is half at % 2 of
// pair[at / 2], or of element first + at % 8 of g0 or g1 (Keys), half at / 8 of pair[at % 8]. open: the elements to compare with
// the ends of the range; one per lane and round, next to never.
// Index inside its group of element `at` of a batch that begins with `first`. Two Value waves to a tile (HALF 0, 1): channels 8
// HALF .. + 7, then 16 further.
template <bool KEYS, int HALF> __device__ __forceinline__ constexpr int element_of(int first, int at) {
  return KEYS ? first + (at & 7) : HALF < 0 ? first + (at & 15) : 8 * HALF + (at & 7) + 16 * (at >> 3 & 1);
}
template <int BITS, bool KEYS, int HALF>
__device__ __forceinline__ void settle_open(uint32_t (&code)[16], const uint32_t (&pair)[8], const GroupParams& g0, const GroupParams& g1, int first, uint32_t open) {
  const float mn0 = g0.mn, mn1 = g1.mn, s0 = g0.s, s1 = g1.s, inv0 = g0.inv_lo, inv1 = g1.inv_lo, inv2_0 = g0.inv2_lo, inv2_1 = g1.inv2_lo;
#pragma unroll 1
  while (__builtin_amdgcn_ballot_w64(open != 0) != 0) {
    const int at = open ? __builtin_ctz(open) : 31;       // 31: no element
    open &= open - 1u;
    uint32_t x = 0;
#pragma unroll
    for (int n = 0; n < 8; n++) {
      x = (KEYS ? at & 7 : at >> 1) == n ? pair[n] : x;
      asm("" : "+v"(x));          // (a chain of selects: recognised as an indexed array it would move to memory)
    }
    const int half = KEYS ? at >> 3 & 1 : at & 1, i = element_of<KEYS, HALF>(first, at);
    const float mn = KEYS && half ? mn1 : mn0, s = KEYS && half ? s1 : s0;
    const bool two = BITS == 3 && (i == 10 || i == 21);
    const float inv = two ? (KEYS && half ? inv2_1 : inv2_0) : (KEYS && half ? inv1 : inv0);
    const float d = (float)__builtin_bit_cast(half_t, (uint16_t)(x >> (16 * half))) - mn;
    const uint32_t c = settle(d, inv, two ? (s * 7.0f) / 3.0f : s);
#pragma unroll
    for (int n = 0; n < 16; n++) {
      code[n] = n == at ? c : code[n];
      asm("" : "+v"(code[n]));
    }
  }
}
// The codes of a batch. The comparison of the two products of an element is a mask of the wave's lanes in scalar registers: only elements
// that some lane has next to k + 1/2 are looked at again.
template <int BITS, bool KEYS, int HALF>
__device__ __forceinline__ void quantize_batch(uint32_t (&code)[16], const uint32_t (&pair)[8], const GroupParams& g0, const GroupParams& g1, int first, uint64_t slow) {
  auto element = [&](int at) { return element_of<KEYS, HALF>(first, at); };
  auto group = [&](int at) -> const GroupParams& { return KEYS && at >= 8 ? g1 : g0; };
  auto d = [&](int at) {
    const uint32_t x = pair[KEYS ? at & 7 : at >> 1];
    const float mn = group(at).mn;
    return (KEYS ? at >= 8 : at & 1) ? diff<1>(x, mn) : diff<0>(x, mn);
  };
  uint64_t near[16], any = slow;
#pragma unroll
  for (int at = 0; at < 16; at++) {
    const float v = d(at);
    code[at] = code_below<BITS>(v, group(at), element(at));
    near[at] = __builtin_amdgcn_ballot_w64(code[at] != code_above<BITS>(v, group(at), element(at)));
    any |= near[at];
  }
  if (__builtin_expect(any != 0, 0)) {
    uint32_t open = 0;
#pragma unroll
    for (int at = 0; at < 16; at++)
      if (near[at] != 0) code[at] = resolve_tie<BITS>(code[at], d(at), group(at), element(at), at, __builtin_amdgcn_inverse_ballot_w64(near[at]), open);
    settle_open<BITS, KEYS, HALF>(code, pair, g0, g1, first, open);
    if (slow != 0) {      // clip (and nothing but code 0 for what is not a number)
#pragma unroll
      for (int at = 0; at < 16; at++) {
        const uint32_t top = kBias + (uint32_t)qmax_of<BITS>(element(at)), c = code[at] < top ? code[at] : top;
        code[at] = (code[at] & 0x7fffffffu) > 0x7f800000u ? kBias : c;
      }
    }
  }
}

// Number of 32-bit word accumulators a lane fills for one code section before the lanes of its quad are combined: words i = 0..15
// (half of them where two waves share a section) of its (kq, j) column group; 4-bit sections have two chunks. 1-bit sections
// consist of the bit plane alone (the `hi` words below, stored at the start of the section).
template <int BITS, int SPLIT> constexpr int acc_words() { return (BITS == 4 ? 32 : 16) / SPLIT; }

// Final step of every wave: `w` holds, in every lane of a quad (q = lane & 3), the complete words
// i = 0..15 (per chunk) of column group (kq, j), or 8 of them from i0 on; lane q has a quarter of them to deliver. `hi` (3- and 1-bit)
// holds the high-plane words, complete in both lanes j and j^1; the even-j lanes deliver them.
// A word of which only the bytes of `mask` are this launch's to write (PARTIAL: Values that leave the window token by token share
// their words with the neighbouring tokens' codes, which are already in place or still to come). A token's are whole halves of a
// word, and whole bytes of a plane word (BYTES): stored as such, nothing is read. (Words were read and written back: the read
// waited for memory at the end of the kernel.)
template <bool PARTIAL, bool BYTES>
__device__ __forceinline__ void put_word(uint32_t* p, uint32_t v, uint32_t mask) {
  if (!PARTIAL || mask == 0xFFFFFFFFu) {
    *p = v;
  } else if constexpr (BYTES) {
    uint8_t* at = reinterpret_cast<uint8_t*>(p);
#pragma unroll
    for (int i = 0; i < 4; i++)
      if (mask >> (8 * i) & 1u) at[i] = (uint8_t)(v >> (8 * i));
  } else {
    uint16_t* at = reinterpret_cast<uint16_t*>(p);
    if (mask & 1u) at[0] = (uint16_t)v;
    if (mask >> 16) at[1] = (uint16_t)(v >> 16);
  }
}

// Words of a section from the wave: lane q of a quad has those of columns i = 4q .. 4q+3. To the section itself where other launches'
// bits share the words (PARTIAL), otherwise to the wave's image of the section in LDS.
template <int BITS, bool PARTIAL, int SPLIT>
__device__ __forceinline__ void put_words(uint32_t* sec, const uint32_t (&w)[acc_words<BITS, SPLIT>()], const uint32_t (&hi)[16 / SPLIT],
                                          int kq, int j, int q, int i0, uint32_t wmask = 0xFFFFFFFFu, uint32_t hmask = 0xFFFFFFFFu) {
  constexpr int kChunks = BITS == 4 ? 2 : BITS == 1 ? 0 : 1;
  constexpr int kPlane = BITS == 1 ? 0 : 256;     // first word of the 1-bit plane
  constexpr int kWords = 16 / SPLIT, kEach = kWords / 4;
#pragma unroll
  for (int c = 0; c < kChunks; c++)
#pragma unroll
    for (int n = 0; n < kEach; n++) {
      const uint32_t* x = &w[kWords * c + n];
      const uint32_t v = q == 0 ? x[0] : q == 1 ? x[kEach] : q == 2 ? x[2 * kEach] : x[3 * kEach];
      put_word<PARTIAL, false>(sec + 256 * c + 4 * (16 * kq + i0 + kEach * q + n) + j, v, wmask);
    }
  if constexpr (BITS == 3 || BITS == 1) {
    if ((j & 1) == 0) {
#pragma unroll
      for (int n = 0; n < kEach; n++) {
        const uint32_t v = q == 0 ? hi[n] : q == 1 ? hi[kEach + n] : q == 2 ? hi[2 * kEach + n] : hi[3 * kEach + n];
        put_word<PARTIAL, true>(sec + kPlane + 2 * (16 * kq + i0 + kEach * q + n) + (j >> 1), v, hmask);
      }
    }
  }
}
// orders the wave's own LDS writes before its following LDS reads (LDS executes a wave's operations in order; this pins the compiler)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Which accesses of a launch go past the caches (see launch_quantize_pack).
enum Stream { kCached, kStreamOut, kStreamBoth };
// the section from its image, 16 (bit plane: 8) bytes per lane and instruction
template <Stream S, typename T>
__device__ __forceinline__ void put(T* p, T v) {
  if constexpr (S != kCached) __builtin_nontemporal_store(v, p);
  else *p = v;
}
template <int BITS, Stream S>
__device__ __forceinline__ void store_section(uint32_t* sec, const uint32_t* image, int lane) {
  constexpr int kChunks = BITS == 4 ? 2 : BITS == 1 ? 0 : 1;
#pragma unroll
  for (int c = 0; c < kChunks; c++) put<S>(reinterpret_cast<u32x4_t*>(sec) + 64 * c + lane, reinterpret_cast<const u32x4_t*>(image)[64 * c + lane]);
  if constexpr (BITS == 3 || BITS == 1) {
    constexpr int kPlane = BITS == 1 ? 0 : 256;
    put<S>(reinterpret_cast<u32x2_t*>(sec + kPlane) + lane, reinterpret_cast<const u32x2_t*>(image + kPlane)[lane]);
  }
}

template <Stream S, typename T>
__device__ __forceinline__ T load_row(const uint16_t* p) {
  const T* t = reinterpret_cast<const T*>(p);
  return S == kStreamBoth ? __builtin_nontemporal_load(t) : *t;
}

// One workgroup of two waves (SPLIT = 1) or four (SPLIT = 2) quantizes and packs one (unit, 32-token tile). Two: wave 0 the Key
// tile, wave 1 the Value tile, each for itself. A lane owns what ends up in the same words: lane = 16*kq + 4*j + q.
//   Key wave:   q = ks; channels d0 = 32*ks + 8*kq + 2*j and d0 + 1 over the 32 tokens (two groups); a word
//               (l = 16*kq + i, j) gets its fields of slot ks + 4*m from this lane, the other ks from the quad.
//   Value wave: q = g;  tokens 8*kq + 2*j and + 1, channels 32*g .. 32*g + 31 (two groups); a word gets its
//               fields of slots 2*g, 2*g + 1 from this lane, the other blocks from the quad.
// The lanes of a quad OR their partial words together (DPP), the 1-bit plane of 3-bit codes also across the
// two j of a word; each lane then has a quarter of the words.
// Memory sees whole rows and whole sections: Key rows are 4 bytes per lane; Value rows 16 bytes per lane, four rows per
// instruction, handed to their lanes through LDS; finished words go through LDS to a store of 1 KB per instruction, and so does the
// metadata of the two waves (8 bytes of every 16 each). What a variant that only loads and stores takes for 31 488 tiles of 2/2
// bit, its accesses past the caches: 98 us with the metadata in its pieces, 93 this way (111 with Value rows in pieces of 16 bytes
// and words stored one by one). The whole kernel: 112.9 us before, with divisions for ties, 90.7 now (a large copy's rate); 8 096
// tiles of 3/4 bit 38.8 and 32.2, about 700 vector instructions per wave and tile (21 us of issue) that only partly overlap the
// loads when a place sees four tiles.
//
// PARTIAL: ageing with separate fronts for Keys and Values. The Key wave works on the tiles [k_tile_a, k_tile_b)
// only; the Value wave writes the codes and metadata of the tokens [v_tok_a, v_tok_b) only: the halves and bytes of words that are
// theirs (put_word), without reading the words. Every row comes from the ring, everything is written in place. With four waves a tile
// (below) the exchange is a barrier all the same: Key waves that leave early pass it first.
//
// SPLIT = 2: two waves for the Keys (16 tokens each) and two for the Values (channels 8 h .. 8 h + 7 and 16 + 8 h .. of every block
// of 32). Each has half of a section's words; the two exchange the extremes of their halves of the groups through LDS. A lane has
// 32 elements instead of 64, one after the other: of the 3.5 us (4.6 at most, where exact ties are settled) that a tile alone took
// in two waves from its start to its last store, the parameters of the groups were 0.45, the codes 1.05 (with ties 2.3) and the
// words 0.4.
template <int KB, int VB, bool PARTIAL, int SPLIT, Stream S>
__device__ __forceinline__ void quantize_tile(const uint16_t* k_in, const uint16_t* v_in, int64_t tok, int64_t unit_b, int64_t unit_h, uint32_t* packed,
                                              int n_tiles, int n_ring, const QuantArgs& a) {
  constexpr int kWords = 16 / SPLIT;           // words of a column group, per wave
  __shared__ __attribute__((aligned(16))) uint32_t s_key[512];             // the Key section's image
  __shared__ __attribute__((aligned(16))) uint32_t s_value[kTile * kD / 2];   // the Value rows, then the Value section's image
  __shared__ __attribute__((aligned(16))) uint32_t s_meta[kMetaWords];
  __shared__ __attribute__((aligned(16))) u32x4_t s_extremes[SPLIT == 2 ? 4 : 1][SPLIT == 2 ? kWave : 1];
  // (read together: where they are used it would be one read after the other)
  if constexpr (PARTIAL)
    asm volatile("" ::"s"(a.ring_w0), "s"(a.W_cap), "s"(a.tile0), "s"(a.Hkv), "s"(a.k_tile_a), "s"(a.k_tile_b), "s"(a.v_tok_a), "s"(a.v_tok_b), "s"(a.tiles_cap));
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int side = wave / SPLIT, part = wave % SPLIT;      // side: 0 Keys, 1 Values
  const int kq = lane >> 4, j = (lane >> 2) & 3, q = lane & 3;
  const int tile_in = blockIdx.x, jh = blockIdx.y, b = blockIdx.z;   // no integer division at the start of a short kernel
  const uint16_t* in = (side ? v_in : k_in) + b * unit_b + jh * unit_h;
  // Input row i (of those that stay in the window) to its ring slot: rows 16 bytes per lane, four at a time. from: ring slot, counted from
  // ring_w0, of the first of 32 slots; the slots [lo, hi) of them are this workgroup's to fill.
  auto copy_rows = [&](int from, int lo, int hi) {
    uint16_t* ring_w = (side ? a.v_ring_w : a.k_ring_w) + (size_t)(b * a.Hkv + jh) * a.W_cap * kD;
    u32x4_t x[8 / SPLIT];
    int at[8 / SPLIT];
#pragma unroll
    for (int n = 0; n < 8 / SPLIT; n++) {
      const int rel = from + 4 * (n * SPLIT + part) + (lane >> 4);
      int i = rel - a.copy_at;
      if (i < 0) i += a.W_cap;
      at[n] = -1;
      if (rel >= lo && rel < hi && i < a.n_copy) {
        const int slot = a.ring_w0 + rel;
        at[n] = slot >= a.W_cap ? slot - a.W_cap : slot;
        x[n] = *reinterpret_cast<const u32x4_t*>(in + (int64_t)(a.copy_row + i) * tok + 8 * (lane & 15));
      }
    }
#pragma unroll
    for (int n = 0; n < 8 / SPLIT; n++)
      if (at[n] >= 0) *reinterpret_cast<u32x4_t*>(ring_w + (size_t)at[n] * kD + 8 * (lane & 15)) = x[n];
  };
  if constexpr (!PARTIAL) {
    if (tile_in >= n_tiles) {       // window rows that land in slots which no tile of the launch reads
      copy_rows((tile_in - n_tiles + a.copy_tile0) * kTile, a.n_read, a.W_cap);
      return;
    }
  }
  // orders LDS accesses of the two waves that share a side (all four pass it)
  auto exchange = [&](u32x4_t mine) {
    s_extremes[wave % (SPLIT == 2 ? 4 : 1)][lane % (SPLIT == 2 ? kWave : 1)] = mine;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    return s_extremes[(wave ^ 1) % (SPLIT == 2 ? 4 : 1)][lane % (SPLIT == 2 ? kWave : 1)];
  };
  if constexpr (PARTIAL) {
    const int tile_abs = a.tile0 + tile_in;
    if (side == 0 && (tile_abs < a.k_tile_a || tile_abs >= a.k_tile_b)) {        // the Keys of this tile are not in the launch
      if constexpr (SPLIT == 2) exchange(u32x4_t{0, 0, 0, 0});
      return;
    }
  }
  // The tile's rows: the first n_old from ring slots, the rest from the input. Slots of one tile never wrap (everything is in steps of 32),
  // so either part is a base and a stride. (PARTIAL: the input is the ring, its first row the one in slot 0.)
  const int n_old = PARTIAL ? 0 : n_ring - tile_in * kTile;
  const uint16_t* new_rows = in - (int64_t)n_old * tok;           // row t of the tile, t >= n_old, at new_rows + t * tok
  const uint16_t* old_rows = nullptr;
  if constexpr (PARTIAL) {
    int slot0 = a.ring_w0 + tile_in * kTile;
    while (slot0 >= a.W_cap) slot0 -= a.W_cap;        // (the launch may span more rows than the ring has slots; only rows of live tokens are read)
    new_rows = in + (int64_t)slot0 * kD;
  } else if (n_old > 0) {
    int slot0 = a.ring_w0 + tile_in * kTile;
    if (slot0 >= a.W_cap) slot0 -= a.W_cap;
    old_rows = (side ? a.v_ring : a.k_ring) + ((int64_t)(b * a.Hkv + jh) * a.W_cap + slot0) * kD;
  }
  // a tile all of one kind, the usual case
  const bool whole = PARTIAL || n_old >= kTile || n_old <= 0;
  const uint16_t* rows = !PARTIAL && n_old > 0 ? old_rows : new_rows;
  const int64_t stride = PARTIAL || n_old > 0 ? kD : tok;
  // what the end of the kernel needs, read while the rows are on their way
  auto read_rest = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!PARTIAL) asm volatile("" ::"s"(a.Hkv), "s"(a.tiles_cap), "s"(a.n_read));
    __builtin_amdgcn_sched_barrier(0);
  };
  // (packed: of the launch's first tile)
  auto record = [&]() { return packed + ((size_t)(b * a.Hkv + jh) * a.tiles_cap + (size_t)tile_in) * record_words(KB, VB); };
  uint32_t hi[kWords];
#pragma unroll
  for (int i = 0; i < kWords; i++) hi[i] = 0;

  if (side == 0) {
    constexpr int kTokens = kTile / SPLIT;           // of this wave: kTokens * part ..
    const int d0 = 32 * q + 8 * kq + 2 * j;
    uint32_t xw[kTokens];                            // (x[tau][d0], x[tau][d0 + 1])
    if (whole) {
      const uint16_t* row = rows + kTokens * part * stride;
#pragma unroll
      for (int t = 0; t < kTokens; t++) { xw[t] = load_row<S, uint32_t>(row + d0); row += stride; }
    } else {
#pragma unroll
      for (int n = 0; n < kTokens; n++) {
        const int t = kTokens * part + n;
        xw[n] = load_row<kCached, uint32_t>((t < n_old ? old_rows + t * kD : new_rows + t * tok) + d0);
      }
    }
    read_rest();
    half2_t mn2, mx2;
    bool nan;
    extremes(xw, mn2, mx2, nan);
    if constexpr (SPLIT == 2) {
      const u32x4_t other = exchange(u32x4_t{__builtin_bit_cast(uint32_t, mn2), __builtin_bit_cast(uint32_t, mx2), 0, 0});
      const uint32_t omn = other[0], omx = other[1];       // (copies: a bit cast applied to the element itself reads element 0)
      mn2 = __builtin_elementwise_min(mn2, __builtin_bit_cast(half2_t, omn));
      mx2 = __builtin_elementwise_max(mx2, __builtin_bit_cast(half2_t, omx));
    }
    const GroupParams g0 = group_params<KB>((float)mn2[0], (float)mx2[0]);
    const GroupParams g1 = group_params<KB>((float)mn2[1], (float)mx2[1]);
    const uint64_t slow = __builtin_amdgcn_ballot_w64(g0.slow || g1.slow || nan);
    uint32_t* rec = PARTIAL ? record() : nullptr;
    // metadata word 4*(d0/2) + f: scale pair (f = 0), minimum pair (f = 1)
    if (part == 0)
      *reinterpret_cast<u32x2_t*>((PARTIAL ? rec : s_meta) + 4 * (d0 >> 1)) =
          u32x2_t{(uint32_t)g0.scale_h | ((uint32_t)g1.scale_h << 16), (uint32_t)g0.zero_h | ((uint32_t)g1.zero_h << 16)};
    uint32_t w[acc_words<KB, SPLIT>()];
#pragma unroll
    for (int i = 0; i < acc_words<KB, SPLIT>(); i++) w[i] = 0;
    auto codes = [&](auto first) {       // first: the wave's first token
#pragma unroll
      for (int t0 = 0; t0 < kTokens; t0 += 8) {
        uint32_t bc[16];                               // biased codes: the lane's first channel, then its second
        const uint32_t pairs[8] = {xw[t0], xw[t0 + 1], xw[t0 + 2], xw[t0 + 3], xw[t0 + 4], xw[t0 + 5], xw[t0 + 6], xw[t0 + 7]};
        quantize_batch<KB, true, -1>(bc, pairs, g0, g1, decltype(first)::value + t0, slow);
        // tokens t0 + n and t0 + 4 + n are the two token halves m of the same word of the column group
#pragma unroll
        for (int n = 0; n < 4; n++) {
          const int i = 4 * (t0 >> 3) + n;
          // the codes of the two channels side by side: the low halves of the biased codes are the codes
          const uint32_t p0 = __builtin_amdgcn_perm(bc[8 + n], bc[n], 0x05040100u), p1 = __builtin_amdgcn_perm(bc[12 + n], bc[4 + n], 0x05040100u);
          if constexpr (KB == 1) {
            hi[i] = (p0 | (p1 << 1)) << (8 * (j & 1) + 2 * q);           // the code is the plane's bit
          } else if constexpr (KB == 4) {
            w[i] = p0 << (4 * q);                                        // chunk m, field ks
            w[kWords + i] = p1 << (4 * q);
          } else {
            const uint32_t both = p0 | (p1 << 8);                        // slots ks + 4*m
            if constexpr (KB == 2) {
              w[i] = both << (2 * q);
            } else {
              w[i] = (both & 0x03030303u) << (2 * q);
              const uint32_t top = (both >> 2) & 0x01010101u;
              hi[i] = ((top | (top >> 7)) & 0x00030003u) << (8 * (j & 1) + 2 * q);
            }
          }
        }
      }
    };
    // (only 3-bit groups have elements that differ from the others)
    if (SPLIT == 2 && KB == 3 && part) codes(std::integral_constant<int, kTokens>{});
    else codes(std::integral_constant<int, 0>{});
#pragma unroll
    for (int i = 0; i < acc_words<KB, SPLIT>(); i++) { w[i] |= quad_x1(w[i]); w[i] |= quad_x2(w[i]); }
    if constexpr (KB == 3 || KB == 1) {
#pragma unroll
      for (int i = 0; i < kWords; i++) { hi[i] |= quad_x1(hi[i]); hi[i] |= quad_x2(hi[i]); hi[i] |= lane_x4(hi[i]); }
    }
    put_words<KB, false, SPLIT>(PARTIAL ? rec + kMetaWords : s_key, w, hi, kq, j, q, kWords * part);
  } else {
    const int tau0 = 8 * kq + 2 * j;
    // PARTIAL: which of the lane's two tokens, and of the two of lane j ^ 1, are among those that leave now
    auto leaves = [&](int tau) { const int t = (a.tile0 + tile_in) * kTile + tau; return !PARTIAL || (t >= a.v_tok_a && t < a.v_tok_b); };
    const bool mine[2] = {leaves(tau0), leaves(tau0 + 1)};
    // Rows to LDS, pieces of 16 bytes: the whole row, or (two waves) every second piece. Piece p of row t lies at p ^ (t/2 % 4) of
    // its row in LDS: the 16 lanes that read together (4 rows, 4 pieces) then find theirs in distinct banks (two waves: two at a
    // time)
    constexpr int kPieces = 16 / SPLIT, kRows = kWave / kPieces;      // of a row; rows per instruction
    uint32_t* area = s_value + part * (kTile * kPieces * 4);
    {
      const int r4 = lane / kPieces, c = lane % kPieces, piece = SPLIT == 2 ? 2 * c + part : c;
      u32x4_t x[kPieces / 2];
      if constexpr (PARTIAL) {
        // Rows of tokens that stay are not read: beyond the resource's end a load returns zeros. (With a branch around each load
        // the rows were once waited for one after the other.)
        const uint64_t base = reinterpret_cast<uint64_t>(rows);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base), hi32 = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
        const __amdgpu_buffer_rsrc_t tile = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uint64_t)hi32 << 32) | lo), 0, kTile * kD * 2, 0x00020000);
#pragma unroll
        for (int n = 0; n < kPieces / 2; n++) {
          const int t = kRows * n + r4;
          x[n] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(tile, leaves(t) ? 2 * kD * t + 16 * piece : 0x40000000, 0, 0));
        }
      } else if (whole) {
        const uint16_t* row = rows + r4 * stride + 8 * piece;
#pragma unroll
        for (int n = 0; n < kPieces / 2; n++) {
          x[n] = load_row<S, u32x4_t>(row);
          row += kRows * stride;
        }
      } else {
#pragma unroll
        for (int n = 0; n < kPieces / 2; n++) {
          const int t = kRows * n + r4;
          x[n] = load_row<kCached, u32x4_t>((t < n_old ? old_rows + t * kD : new_rows + t * tok) + 8 * piece);
        }
      }
      read_rest();
#pragma unroll
      for (int n = 0; n < kPieces / 2; n++) {
        const int t = kRows * n + r4;
        *reinterpret_cast<u32x4_t*>(area + 4 * kPieces * t + 4 * (c ^ ((t >> 1) & 3))) = x[n];
      }
      wave_lds_fence();
    }
    constexpr int kOwn = 4 / SPLIT;                  // pieces of a group of this wave
    // rows tau0, tau0 + 1: channels 32*q .. 32*q + 31 (two waves: 8*part .. + 7 and 16 + 8*part .. of them)
    u32x4_t xr[2][kOwn];
#pragma unroll
    for (int hh = 0; hh < 2; hh++)
#pragma unroll
      for (int c = 0; c < kOwn; c++) xr[hh][c] = *reinterpret_cast<const u32x4_t*>(area + 4 * kPieces * (tau0 + hh) + 4 * ((kOwn * q + c) ^ j));
    const uint32_t wmask = (mine[0] ? 0x0000FFFFu : 0u) | (mine[1] ? 0xFFFF0000u : 0u);
    // a plane word holds the pairs j (even, bits 0-7 and 16-23) and j + 1 (bits 8-15 and 24-31); the even lane stores it
    uint32_t hmask = (mine[0] ? 0x000000FFu : 0u) | (mine[1] ? 0x00FF0000u : 0u);
    if constexpr (PARTIAL) hmask |= (leaves(tau0 + 2) ? 0x0000FF00u : 0u) | (leaves(tau0 + 3) ? 0xFF000000u : 0u);
    else hmask = 0xFFFFFFFFu;
    half2_t mn2[2], mx2[2];
    bool nan[2];
#pragma unroll
    for (int hh = 0; hh < 2; hh++) {
      uint32_t x[4 * kOwn];
#pragma unroll
      for (int e = 0; e < 4 * kOwn; e++) x[e] = xr[hh][e >> 2][e & 3];
      extremes(x, mn2[hh], mx2[hh], nan[hh]);
    }
    if constexpr (SPLIT == 2) {
      const u32x4_t other = exchange(u32x4_t{__builtin_bit_cast(uint32_t, mn2[0]), __builtin_bit_cast(uint32_t, mx2[0]),
                                             __builtin_bit_cast(uint32_t, mn2[1]), __builtin_bit_cast(uint32_t, mx2[1])});
#pragma unroll
      for (int hh = 0; hh < 2; hh++) {
        const uint32_t omn = other[2 * hh], omx = other[2 * hh + 1];
        mn2[hh] = __builtin_elementwise_min(mn2[hh], __builtin_bit_cast(half2_t, omn));
        mx2[hh] = __builtin_elementwise_max(mx2[hh], __builtin_bit_cast(half2_t, omx));
      }
    }
    GroupParams gp[2];
    uint64_t slow[2];
#pragma unroll
    for (int hh = 0; hh < 2; hh++) {
      const float mn = fminf((float)mn2[hh][0], (float)mn2[hh][1]), mx = fmaxf((float)mx2[hh][0], (float)mx2[hh][1]);
      gp[hh] = group_params<VB>(mn, mx);
      slow[hh] = __builtin_amdgcn_ballot_w64(gp[hh].slow || nan[hh]);
    }
    uint32_t* rec = PARTIAL ? record() : nullptr;
    // metadata word 4*(16*g + tau0/2) + f: scale pair (f = 2), minimum pair (f = 3)
    if (part == 0) {
      const uint32_t sc2 = (uint32_t)gp[0].scale_h | ((uint32_t)gp[1].scale_h << 16), zp2 = (uint32_t)gp[0].zero_h | ((uint32_t)gp[1].zero_h << 16);
      uint32_t* mp = (PARTIAL ? rec : s_meta) + 4 * (16 * q + (tau0 >> 1)) + 2;
      if constexpr (!PARTIAL) {
        *reinterpret_cast<u32x2_t*>(mp) = u32x2_t{sc2, zp2};
      } else {
        put_word<true, false>(mp, sc2, wmask);
        put_word<true, false>(mp + 1, zp2, wmask);
      }
    }
    // partial words with the lane-independent shifts first: one token's fields (slot parity e/16), then the two tokens side by side
    constexpr int kField = VB == 4 || VB == 3 ? 4 : 2;          // (3-bit codes: taken apart into planes afterwards)
    uint32_t pw[2][kWords];
    auto codes = [&](auto half) {
      constexpr int HALF = decltype(half)::value;
#pragma unroll
      for (int hh = 0; hh < 2; hh++)
#pragma unroll
        for (int e0 = 0; e0 < 32 / SPLIT; e0 += 16) {
          uint32_t bc[16];                               // biased codes
          uint32_t pairs[8];
#pragma unroll
          for (int n = 0; n < 8; n++) pairs[n] = xr[hh][(e0 >> 3) + (n >> 2)][n & 3];
          quantize_batch<VB, false, HALF>(bc, pairs, gp[hh], gp[hh], e0, slow[hh]);
#pragma unroll
          for (int n = 0; n < 16; n++) {
            const int i = n % kWords, slot = (e0 + n) / kWords;
            // (the bias lies above bit 16 and stays there)
            pw[hh][i] = slot == 0 ? bc[n] : (bc[n] << kField) + pw[hh][i];
          }
        }
    };
    if constexpr (SPLIT == 1) codes(std::integral_constant<int, -1>{});
    else if (VB == 3 && part) codes(std::integral_constant<int, 1>{});
    else codes(std::integral_constant<int, 0>{});
    uint32_t ph[kWords];
#pragma unroll
    for (int i = 0; i < kWords; i++) {
      const uint32_t both = __builtin_amdgcn_perm(pw[1][i], pw[0][i], 0x05040100u);       // the low halves side by side
      pw[0][i] = both;
      ph[i] = both;
      if constexpr (VB == 3) {
        pw[0][i] = (both & 0x00030003u) | ((both >> 2) & 0x000C000Cu);
        ph[i] = ((both >> 2) & 0x00010001u) | ((both >> 4) & 0x00040004u);
      }
    }
    uint32_t w[acc_words<VB, SPLIT>()];
    if constexpr (VB == 4) {
      // slot 2*g + sp: chunk g/2, field 2*(g%2) + sp; the chunk's words are complete after the pair (g, g^1)
#pragma unroll
      for (int i = 0; i < kWords; i++) {
        uint32_t v = pw[0][i] << (8 * (q & 1));
        v |= quad_x1(v);
        const uint32_t other = quad_x2(v);            // the other chunk's words, from lane g ^ 2
        w[i] = (q & 2) ? other : v;                  // chunk 0
        w[kWords + i] = (q & 2) ? v : other;         // chunk 1
      }
    } else {
#pragma unroll
      for (int i = 0; i < kWords; i++) {
        w[i] = pw[0][i] << (4 * q);
        w[i] |= quad_x1(w[i]); w[i] |= quad_x2(w[i]);
      }
      if constexpr (VB == 3 || VB == 1) {
        // bit plane: bit 16*hh + 8*(j%2) + 2*(slot%4) + slot/4 with slot = 2*g + sp
#pragma unroll
        for (int i = 0; i < kWords; i++) {
          hi[i] = ph[i] << (8 * (j & 1) + 4 * (q & 1) + (q >> 1));
          hi[i] |= quad_x1(hi[i]); hi[i] |= quad_x2(hi[i]); hi[i] |= lane_x4(hi[i]);
        }
      }
    }
    if constexpr (PARTIAL) {
      put_words<VB, true, SPLIT>(rec + kMetaWords + tile_words(KB), w, hi, kq, j, q, kWords * part, wmask, hmask);
    } else {
      wave_lds_fence();      // (the rows in this area have been read; by the other wave too: exchange)
      put_words<VB, false, SPLIT>(s_value, w, hi, kq, j, q, kWords * part);
    }
  }
  if constexpr (!PARTIAL) {
    __syncthreads();         // the metadata of both sides, and the side's own section, are in LDS
    uint32_t* rec = record();
    if (part == 0) {
      if (side == 0) store_section<KB, S>(rec + kMetaWords, s_key, lane);
      else store_section<VB, S>(rec + kMetaWords + tile_words(KB), s_value, lane);
    }
    if (part == SPLIT - 1) put<S>(reinterpret_cast<u32x2_t*>(rec) + 64 * side + lane, reinterpret_cast<const u32x2_t*>(s_meta)[64 * side + lane]);
    // New rows that land in slots this tile was read from (all waves have their rows: the barrier): this workgroup fills those.
    if (tile_in * kTile < a.n_read) copy_rows(tile_in * kTile, 0, a.n_read);
  }
}

// Four waves: small launches. The parameters in front of `a` are preloaded into scalar registers (build.py): what the first
// requests need where all rows are rows of the input. (Read from memory in turn, they let the first request out 0.85 us after the
// start.)
typedef int64_t i64x2_t __attribute__((ext_vector_type(2)));
template <int KB, int VB, bool PARTIAL, Stream S>
__global__ __launch_bounds__(256, 4) void quantize_pack_kernel(const uint16_t* k, const uint16_t* v, i64x2_t strides, int64_t unit_h, uint32_t* packed,
                                                               u32x2_t counts, QuantArgs a) {
  quantize_tile<KB, VB, PARTIAL, 2, S>(k, v, strides[0], strides[1], unit_h, packed, (int)counts[0], (int)counts[1], a);
}
// Two waves: large launches, to which preloading (0.3 us in front of a launch) gives nothing.
template <int KB, int VB, bool PARTIAL, Stream S>
__global__ __launch_bounds__(128, 4) void quantize_pack_many_kernel(QuantArgs a) {
  quantize_tile<KB, VB, PARTIAL, 1, S>(a.k, a.v, a.tok, a.unit_b, a.unit_h, a.packed + (size_t)a.tile0 * record_words(KB, VB), a.n_tiles, a.n_ring, a);
}

// x = code * s_i + min, evaluated in fp32 (multiply, then add), of the first n_tokens tokens of every unit.
__global__ __launch_bounds__(256) void dequant_kernel(DequantArgs a) {
  const int u = blockIdx.y, tile_i = blockIdx.x;
  const uint32_t* rec = a.packed + ((size_t)u * a.tiles_cap + tile_i) * record_words(a.k_bits, a.v_bits);
  for (int e = threadIdx.x; e < kTile * kD; e += blockDim.x) {
    const int tau = e / kD, d = e % kD;
    const int t = tile_i * kTile + tau;
    if (t < a.n_tokens) a.out[((size_t)u * a.n_tokens + t) * kD + d] = dequant_elem(rec, a.k_bits, a.v_bits, a.which, tau, d);
  }
}

// New tokens of every unit into consecutive ring slots of the two fp16 windows (one full row each). The arguments are not preloaded
// here: that costs a launch 0.3 us (one token for 256 units: 1.95 and 2.15 us), and there is nothing in these kernels to hide it.
// Few rows, bound by the launch, and rows that don't begin at multiples of 16 bytes (full-precision layers take any): a workgroup
// per unit and token.
__global__ __launch_bounds__(128) void append_kernel(AppendArgs a) {
  const int u = blockIdx.x, i = blockIdx.y, d = threadIdx.x;
  const int64_t src = (int64_t)(u / a.Hkv) * a.batch + (int64_t)(u % a.Hkv) * a.head + (int64_t)i * a.tok + d;
  const size_t dst = ((size_t)u * a.W_cap + (a.slot + i) % a.W_cap) * kD + d;
  a.k_win[dst] = a.k_new[src];
  a.v_win[dst] = a.v_new[src];
}
// More of them, bound by memory: 16 bytes per lane, a workgroup takes 4 kv heads of a token. 300 tokens for 512 units 63 -> 24 us,
// 31 for 2048 units 19.9 -> 8.8, 300 for 8 units 2.57 -> 2.15; below 1024 rows it is no faster (one token for 256 units 1.94 and
// 1.98 us).
constexpr int kAppendHeads = 4;
__global__ __launch_bounds__(32 * kAppendHeads) void append_many_kernel(AppendArgs a) {
  const int row = threadIdx.x >> 4, piece = threadIdx.x & 15;
  const int i = blockIdx.x, b = blockIdx.y, j = blockIdx.z * kAppendHeads + (row >> 1);
  if (j >= a.Hkv) return;
  int slot = a.slot + i;      // (no more tokens than slots)
  if (slot >= a.W_cap) slot -= a.W_cap;
  const uint16_t* src = (row & 1 ? a.v_new : a.k_new) + b * a.batch + j * a.head + i * a.tok + 8 * piece;
  uint16_t* dst = (row & 1 ? a.v_win : a.k_win) + ((size_t)(b * a.Hkv + j) * a.W_cap + slot) * kD + 8 * piece;
  *reinterpret_cast<u32x4_t*>(dst) = *reinterpret_cast<const u32x4_t*>(src);
}

// Load-only pass over a buffer in the launch shape of the attention kernel (one workgroup per contiguous span,
// 16 bytes per lane and load, non-temporal policy, four loads in flight per lane): the rate a kernel of this
// shape can reach on the machine at hand when it does nothing but read.
__global__ __launch_bounds__(768) void stream_read_kernel(const u32x4_t* buf, size_t n16, uint32_t* sink) {
  const size_t per_wg = (n16 + gridDim.x - 1) / gridDim.x;
  const size_t begin = (size_t)blockIdx.x * per_wg;
  const size_t end = begin + per_wg < n16 ? begin + per_wg : n16;
  const size_t step = blockDim.x;
  u32x4_t acc = {0, 0, 0, 0};
  size_t i = begin + threadIdx.x;
  for (; i + 3 * step < end; i += 4 * step) {
    const u32x4_t a = __builtin_nontemporal_load(buf + i), b = __builtin_nontemporal_load(buf + i + step);
    const u32x4_t c = __builtin_nontemporal_load(buf + i + 2 * step), d = __builtin_nontemporal_load(buf + i + 3 * step);
    acc |= (a ^ b) | (c ^ d);
  }
  for (; i < end; i += step) acc |= __builtin_nontemporal_load(buf + i);
  // never true for real data in all four words at once: keeps the loads alive without a store per lane
  if ((acc[0] & acc[1] & acc[2] & acc[3]) == 0xFFFFFFFFu && sink) sink[0] = 1u;
}

// Four waves to a tile or two: with four the chain from a tile's rows to its record is half as long, and more waves hide each
// other's; with two each row is requested by one wave only, and the work that both waves of a side do (extremes met through LDS,
// parameters) is done once. Time of two waves over that of four, all pairs of widths, records past the caches from 2048 tiles on:
//   tiles         512        2048       4096       6144       8192       12 288     16 384
//   no 3 bit      1.16-1.25  1.06-1.11  1.05-1.08  1.04-1.06  1.03-1.05  1.01-1.03  1.00-1.03
//   a 3-bit side  1.13-1.25  1.00-1.02  1.00-1.02  0.97-1.00  0.96-0.98  0.94-0.97  0.92-0.96
// (2/2 bit 5.2 and 4.4 us, 9.4 and 8.8, ..., 44.7 and 44.7; 3/4 bit 6.1 and 5.0, 10.4 and 10.5, ..., 49.3 and 51.7.) More tiles are
// also loaded past the caches, where four waves lose (31 488 tiles at 2/2 bit 91 and 105 us). 8 tiles: 4.1 and 3.5 us (2/2 bit), 4.8
// and 3.8 (3/4). Ageing with the fronts apart, without and with a 3-bit side: 512 tiles 1.14-1.24 and 1.16-1.19, 4096 1.08-1.11 and
// 1.03-1.04, 6144 1.06-1.10 and 0.97-0.99; one Value token for each of 256 units 4.3 and 3.4 us (2/2 bit).
template <int KB, int VB, bool PARTIAL>
hipError_t launch_qp(const QuantArgs& a, dim3 grid, Stream stream, size_t tiles, hipStream_t s) {
  auto run_four = [&](auto kernel) {
    return launch(kernel, grid, 4 * kWave, s, a.k, a.v, i64x2_t{a.tok, a.unit_b}, a.unit_h, a.packed + (size_t)a.tile0 * record_words(KB, VB),
                  u32x2_t{(uint32_t)a.n_tiles, (uint32_t)a.n_ring}, a);
  };
  auto run_two = [&](auto kernel) { return launch(kernel, grid, 2 * kWave, s, a); };
  const bool four = tiles <= (PARTIAL || KB == 3 || VB == 3 ? 4096 : 8192);
  if constexpr (PARTIAL) return four ? run_four(quantize_pack_kernel<KB, VB, true, kCached>) : run_two(quantize_pack_many_kernel<KB, VB, true, kCached>);
  if constexpr (!PARTIAL) {
    if (stream == kCached) return run_four(quantize_pack_kernel<KB, VB, false, kCached>);          // (fewer than 2048 tiles)
    if (stream == kStreamOut)
      return four ? run_four(quantize_pack_kernel<KB, VB, false, kStreamOut>) : run_two(quantize_pack_many_kernel<KB, VB, false, kStreamOut>);
    return run_two(quantize_pack_many_kernel<KB, VB, false, kStreamBoth>);
  }
}

// The bit pairs the library accepts: every pair of 1..4 (a 16-bit side never reaches the quantizer).
template <bool PARTIAL>
hipError_t launch_bits(const QuantArgs& a, int k_bits, int v_bits, int n_tiles, int units, hipStream_t s) {
  if (n_tiles == 0 || units == 0) return hipSuccess;
  const dim3 grid(n_tiles + (PARTIAL ? 0 : a.copy_tiles), a.Hkv, units / a.Hkv);
  // Rows are loaded past the caches where a launch reads more than the memory-side cache (256 MB) can still hold of what was
  // written last. A variant that only loads and stores, 256 units of 44, 60, 76, 92, 123 tiles (16 KB each): cached 31.4, 42.3, 61.6, 76.4,
  // 101.9 us, past the caches 33.7, 45.7, 57.4, 69.3, 92.9. Records are stored past them but for the few tiles of a decode step, which are
  // read next. (The same variant, 2048 tiles: 5.8 us with cached stores, 5.1 without; 15 360: 43.8, 42.3; the whole kernel with 512
  // tiles: 6.6, 7.0.)
  const size_t tiles = (size_t)n_tiles * units;
  const Stream streaming = tiles * (2 * kTile * kD * 2) > ((size_t)256 << 20) ? kStreamBoth : tiles >= 2048 ? kStreamOut : kCached;
  switch (k_bits * 10 + v_bits) {
    case 11: return launch_qp<1, 1, PARTIAL>(a, grid, streaming, tiles, s);
    case 12: return launch_qp<1, 2, PARTIAL>(a, grid, streaming, tiles, s);
    case 13: return launch_qp<1, 3, PARTIAL>(a, grid, streaming, tiles, s);
    case 14: return launch_qp<1, 4, PARTIAL>(a, grid, streaming, tiles, s);
    case 21: return launch_qp<2, 1, PARTIAL>(a, grid, streaming, tiles, s);
    case 22: return launch_qp<2, 2, PARTIAL>(a, grid, streaming, tiles, s);
    case 23: return launch_qp<2, 3, PARTIAL>(a, grid, streaming, tiles, s);
    case 24: return launch_qp<2, 4, PARTIAL>(a, grid, streaming, tiles, s);
    case 31: return launch_qp<3, 1, PARTIAL>(a, grid, streaming, tiles, s);
    case 32: return launch_qp<3, 2, PARTIAL>(a, grid, streaming, tiles, s);
    case 33: return launch_qp<3, 3, PARTIAL>(a, grid, streaming, tiles, s);
    case 34: return launch_qp<3, 4, PARTIAL>(a, grid, streaming, tiles, s);
    case 41: return launch_qp<4, 1, PARTIAL>(a, grid, streaming, tiles, s);
    case 42: return launch_qp<4, 2, PARTIAL>(a, grid, streaming, tiles, s);
    case 43: return launch_qp<4, 3, PARTIAL>(a, grid, streaming, tiles, s);
    case 44: return launch_qp<4, 4, PARTIAL>(a, grid, streaming, tiles, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_quantize_pack(QuantArgs a, int k_bits, int v_bits, int n_tiles, int units, hipStream_t s) {
  a.n_tiles = n_tiles;
  return launch_bits<false>(a, k_bits, v_bits, n_tiles, units, s);
}

hipError_t launch_quantize_fronts(const QuantArgs& a, int k_bits, int v_bits, int n_tiles, int units, hipStream_t s) {
  return launch_bits<true>(a, k_bits, v_bits, n_tiles, units, s);
}

hipError_t launch_dequant(const DequantArgs& a, int units, hipStream_t s) {
  if (a.n_tokens == 0 || units == 0) return hipSuccess;
  dequant_kernel<<<dim3((a.n_tokens + kTile - 1) / kTile, units), 256, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t launch_stream_read(const void* buf, size_t bytes, int workgroups, int threads, uint32_t* sink, hipStream_t s) {
  if (bytes < 16 || workgroups < 1) return hipSuccess;
  stream_read_kernel<<<workgroups, threads, 0, s>>>(reinterpret_cast<const u32x4_t*>(buf), bytes / 16, sink);
  return hipGetLastError();
}

hipError_t launch_append(const AppendArgs& a, hipStream_t s) {
  if (a.n == 0 || a.units == 0) return hipSuccess;
  const bool aligned = ((reinterpret_cast<uintptr_t>(a.k_new) | reinterpret_cast<uintptr_t>(a.v_new)) & 15u) == 0 &&
                       a.tok % 8 == 0 && a.head % 8 == 0 && a.batch % 8 == 0;
  if (aligned && (int64_t)a.units * a.n > 1024)
    return launch(append_many_kernel, dim3(a.n, a.units / a.Hkv, (a.Hkv + kAppendHeads - 1) / kAppendHeads), 32 * kAppendHeads, s, a);
  return launch(append_kernel, dim3(a.units, a.n), 128, s, a);
}

}  // namespace kvmix
