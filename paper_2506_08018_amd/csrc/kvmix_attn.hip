// Fused decode attention over the packed mixed-bit KV cache plus the fp16 recent window (gfx950).
//
// Paper Sec. 3.4 item 2 (dequantize on the fly while multiplying, never materialize fp16 K/V),
// Sec. 3.2.2 step 4 (x = q*s + min), Sec. 3.3 (recent tokens stay in full precision).
//
// Formulation. For one kv head and one 32-token tile
//   score[t][h] = sum_d code[t][d] * (q[h][d]*s[d])  +  sum_d q[h][d]*z[d]
//   out[d][h]  += sum_t code[t][d] * (p[t][h]*s[t][g(d)])  +  sum_t p[t][h]*z[t][g(d)]
// Both code sums are 16x16x32 fp16 MFMAs whose A operand is the packed word ANDed with a mask: a 1/2/4-bit field left in place
// inside a zero fp16 pattern is the subnormal code * 2^(pos-24), exact, and MFMA honours subnormal inputs (3-bit codes are a 2-bit
// plane plus a 1-bit plane). The scale factors ride in the B operand, split into an fp16 (hi, lo) pair held in two MFMA columns so
// that the products stay exact to ~22 bits; the up-to-8 query heads of the group use columns 0..7 (hi) and 8..15 (lo). Groups of 16
// heads and more run in blocks of 8, or in blocks of 16: a head per column, with hi and lo as two instructions on the same
// accumulators. The fp16 window runs on MFMAs with plain fp16 operands; so do the zero-point sums for groups of 4 query heads and
// more, while groups of 1 or 2 heads take them (and the softmax denominator) on the vector unit, where they are cheaper than matrix
// instructions with mostly empty columns.
//
// Data movement. Every byte of a tile record is loaded from HBM once, by one lane (16 B of
// metadata and 16 B of every 1 KiB of codes per lane); a wave has one tile in flight while the
// other waves of its SIMD compute (two or three in flight measured no faster at full load). The scale-folded
// B operands are computed cooperatively (each lane two values per head) and redistributed
// through a wave-private LDS area (8 and 16 heads: by every lane for itself, from scales in that area), so no barrier is
// needed inside the main loop. Window Value rows go from memory straight into the same area.
// Softmax is online, per wave, with a lazily raised reference maximum; waves of a workgroup
// take tiles from a shared counter and merge through LDS (without a barrier when the unit is not
// split: the last wave to deliver combines); splits of one unit merge through a workspace, the
// last arriving workgroup writes the output. Tiles between a Key front and a Value front (one side in a record, the
// other in the ring) are taken by the same waves in the same launch.
#include <type_traits>
#include "kvmix_common.hpp"

namespace kvmix {

namespace {

// Waves per workgroup; this file is compiled once for each of the two forms (the launch picks one, see attn_waves in kvmix_api.hip),
// each without and with tiles between two fronts.
// 12 waves, one workgroup per CU: 168 registers per lane. 8 waves: 128 registers, two workgroups per CU.
constexpr int kNW = KVMIX_WAVES;
constexpr bool kMixed = KVMIX_MIXED;     // with tiles between a Key front and a Value front
constexpr int kMergeBatch = 32;          // splits whose partials the merging workgroup requests together (one round trip)
// Reference of the running softmax (log2 units): numerators 2^(score - reference) are kept at or below 2^kRefCap;
// when a score would exceed that, the reference is raised to (that score - kRefCap + 4), which leaves room for
// scores 16 times larger before the next raise. Numerators are large on purpose: they and their products with
// the Value scales travel as fp16 pairs whose absolute resolution is 2^-25, and the thousands of low-weight
// tokens of a long context sit near that floor; with numerators up to 2^6 instead of 1 the floor is 64 times
// lower relative to the sums. The price is the range: a Value group scale must stay below 2^16 / 2^6 = 1024.
constexpr float kRefCap = 6.0f;
constexpr float kRefMargin = 4.0f - kRefCap;

typedef float float2_t __attribute__((ext_vector_type(2)));

// 2^x by the hardware instruction alone (results below 2^-126 flush to zero, which is harmless here)
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float4_t mfma16(half8_t a, half8_t b, float4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
// value of lane (l ^ 8) within each row of 16 lanes
__device__ __forceinline__ float ror8(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xf, 0xf, false));
}
__device__ __forceinline__ half8_t as_half8(u32x4_t v) { return __builtin_bit_cast(half8_t, v); }
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp_f(float v) {   // lanes without a source (or outside ROW_MASK) read 0
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, false));
}
// sum over the 16 lanes of each row; every lane of the row gets it
__device__ __forceinline__ float row_sum(float v) {
  v += dpp_f<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_f<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_f<0x141>(v);   // row_half_mirror
  v += dpp_f<0x140>(v);   // row_mirror
  return v;
}
// maximum over the 16 lanes of each row; every lane of the row gets it
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, dpp_f<0xB1>(v));
  v = fmaxf(v, dpp_f<0x4E>(v));
  v = fmaxf(v, dpp_f<0x141>(v));
  v = fmaxf(v, dpp_f<0x140>(v));
  return v;
}
// sum over the 64 lanes of the wave as a wave-uniform value
__device__ __forceinline__ float wave_sum(float v) {
  v = row_sum(v);
  v += dpp_f<0x142, 0xA>(v);   // row_bcast:15 -> rows 1 and 3 add the sum of the row before
  v += dpp_f<0x143, 0xC>(v);   // row_bcast:31 -> rows 2 and 3 add the sum of rows 0..1
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ float wave_max(float v) {   // rare path: plain butterflies
  v = fmaxf(v, __shfl_xor(v, 1)); v = fmaxf(v, __shfl_xor(v, 2)); v = fmaxf(v, __shfl_xor(v, 4));
  v = fmaxf(v, __shfl_xor(v, 8)); v = fmaxf(v, __shfl_xor(v, 16)); v = fmaxf(v, __shfl_xor(v, 32));
  return v;
}
__device__ __forceinline__ float uniform_lane(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
// orders the wave's own LDS writes before its following LDS reads (LDS executes a wave's
// operations in order; this only pins the compiler)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bit position (inside a 16-bit half, after the unpack shift) of the field that feeds slot `s`
// (0..3 = slot % 4): the MFMA sees code * 2^(pos - 24). Fields are moved as high in the fp16 mantissa
// as they fit: the matrix core aligns the products of one dot product to their largest nominal
// exponent (that of a subnormal is fixed) and truncates below its window, so a code sitting in the
// lowest mantissa bits loses product bits (measured: ~1e-5 relative at position 0, exact from 6 up).
template <int BITS> __device__ __forceinline__ constexpr int field_pos(int s) { return BITS == 4 ? 4 * (s & 1) + 2 : BITS == 1 ? 2 * s + 4 : 2 * s + 2; }

// The codes of a tile between two fronts: multiplied up to the fp16 number code * 2^-7, a normal one, whatever the field. Of
// products of subnormal operands the matrix core drops low bits (see above): where a field lies low, that is more than everything
// else takes from a result. These tiles used to be summed in fp32 on the vector unit, and their error against 64 bits stays what it
// was. 1000 tokens, all Keys in the ring and all Values packed at 2, 3, 4 bit, outputs that are not the fp16 rounding of the result
// in 64 bits: 0.1 to 0.3 % on the vector unit, 8, 5 and 4 % with the fields as they are (an error of 4e-5, 2e-5, 1e-5 of the result
// next to the rounding's 2.1e-4), 0.2 to 0.7 % this way (5e-7).
constexpr int kExactPos = 17;
template <int BITS> __device__ __forceinline__ half8_t exact_codes(half8_t fields, int s) {
  const half_t up = (half_t)__builtin_ldexpf(1.0f, kExactPos - field_pos<BITS>(s));
  return fields * half8_t{up, up, up, up, up, up, up, up};
}

// ---- A operands from packed words. wa = word << 2, wb = word >> 6 (slots 0..3 / 4..7 of each half).
// 2-bit plane (also the low plane of 3-bit): slot field from bits 2*slot to bits 2*(slot%4) + 2.
__device__ __forceinline__ half8_t unpack2(const u32x4_t& wa, const u32x4_t& wb, int slot) {
  const uint32_t mask = 0x00030003u << (2 * (slot & 3) + 2);
  const u32x4_t src = (slot & 4) ? wb : wa;
  return as_half8(src & mask);
}
// 4-bit: 8 words (two chunks of 4), slot -> chunk slot/4, field slot%4 from bits 4*field to 4*(field%2) + 2.
__device__ __forceinline__ half8_t unpack4(const u32x4_t& wa, const u32x4_t& wb, int field) {
  const uint32_t mask = 0x000F000Fu << (4 * (field & 1) + 2);
  const u32x4_t src = (field & 2) ? wb : wa;
  return as_half8(src & mask);
}
// 1-bit high plane of 3-bit codes: 2 words; word j/2 holds, for pair j, bit 8*(j%2) + 2*(slot%4) + slot/4.
// hs[v] = plane shifted so that variant v = 2*(j%2) + slot/4 has its bits at 2*(slot%4) + 4, two above
// the low plane's field (bit 10, the lowest exponent bit, continues the subnormal scale: 2^-14).
__device__ __forceinline__ half8_t unpack1(const u32x2_t (&hs)[4], int slot) {
  const uint32_t mask = 0x00010001u << (2 * (slot & 3) + 4);
  const int hi = slot >> 2;
  u32x4_t r;
  r[0] = hs[0 + hi][0] & mask;   // j = 0: word 0, variant (0, hi)
  r[1] = hs[2 + hi][0] & mask;   // j = 1: word 0, variant (1, hi)
  r[2] = hs[0 + hi][1] & mask;   // j = 2: word 1
  r[3] = hs[2 + hi][1] & mask;   // j = 3: word 1
  return as_half8(r);
}
__device__ __forceinline__ void shift_hi_plane(const u32x2_t& h, u32x2_t (&hs)[4]) {
  hs[0] = h << 4;   // (j%2 = 0, slot/4 = 0): source bit 2*s     -> 2*s + 4
  hs[1] = h << 3;   // (0, 1):                 source bit 2*s + 1 -> 2*s + 4
  hs[2] = h >> 4;   // (1, 0):                 source bit 2*s + 8 -> 2*s + 4
  hs[3] = h >> 5;   // (1, 1):                 source bit 2*s + 9 -> 2*s + 4
}

// Tile loads are buffer loads: a unit's array is one buffer resource (scalar registers), the tile's
// byte offset a scalar operand and the lane's offset one 32-bit vector register, so a load costs no
// address arithmetic. Reads beyond the resource's size return zero instead of faulting.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  // the base is wave-uniform by construction; saying so keeps the descriptor in scalar registers
  const uint64_t v = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  void* ub = reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ub, 0, (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}
// Cache policy of the tile loads: non-temporal. Every record is read once per launch; marked as streaming it
// does not displace other lines on its way through the caches (measured: 1.5 us less per launch on the
// Llama-2-7B-shaped workload).
constexpr int kStreaming = 2;
__device__ __forceinline__ u32x4_t buf_load16(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, kStreaming));
}
__device__ __forceinline__ u32x2_t buf_load8(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, kStreaming));
}

// 16 bytes per lane from memory into LDS: lane l's go to dst + 16 l (dst: wave-uniform). Counted like a load, waited for
// explicitly before the LDS is read.
__device__ __forceinline__ void buf_load_to_lds16(rsrc_t r, uint32_t voff, uint32_t soff, void* dst) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, (int)voff, (int)soff, 0, kStreaming);
}
// Transposing read: of a group of 16 lanes, lane i passes the address of 4 halves of row i / 4 (columns 4 (i % 4) .. +3) and gets column i
// of the four rows. Two of them, four rows (1 KiB) apart: 8 consecutive rows of the lane's column.
__device__ __forceinline__ half8_t read_transposed(const char* lds, int off) {
  typedef short short4_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) short4_t* lds4_t;
  const short4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(lds + off));
  const short4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(lds + off + 4 * kD * 2));
  return __builtin_bit_cast(half8_t, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The lane's share of one packed tile as loaded (Raw) and prepared for unpacking (Codes).
template <int BITS> struct Raw;
template <> struct Raw<1> {     // the bit plane alone: 8 bytes per lane
  u32x2_t h;
  __device__ __forceinline__ void load(rsrc_t r, uint32_t soff, uint32_t, uint32_t l8) { h = buf_load8(r, l8, soff); }
};
template <> struct Raw<2> {
  u32x4_t w;
  __device__ __forceinline__ void load(rsrc_t r, uint32_t soff, uint32_t l16, uint32_t) { w = buf_load16(r, l16, soff); }
};
template <> struct Raw<3> {
  u32x4_t w; u32x2_t h;
  __device__ __forceinline__ void load(rsrc_t r, uint32_t soff, uint32_t l16, uint32_t l8) {
    w = buf_load16(r, l16, soff);
    h = buf_load8(r, l8, soff + 1024u);
  }
};
template <> struct Raw<4> {
  u32x4_t w[2];
  __device__ __forceinline__ void load(rsrc_t r, uint32_t soff, uint32_t l16, uint32_t) {
    w[0] = buf_load16(r, l16, soff);
    w[1] = buf_load16(r, l16, soff + 1024u);
  }
};
template <int BITS> struct Codes;
template <> struct Codes<1> {
  u32x2_t hs[4];
  __device__ __forceinline__ explicit Codes(const Raw<1>& r) { shift_hi_plane(r.h, hs); }
  __device__ __forceinline__ half8_t lo(int slot) const { return unpack1(hs, slot); }
};
template <> struct Codes<2> {
  u32x4_t wa, wb;
  __device__ __forceinline__ explicit Codes(const Raw<2>& r) : wa(r.w << 2), wb(r.w >> 6) {}
  __device__ __forceinline__ half8_t lo(int slot) const { return unpack2(wa, wb, slot); }
};
template <> struct Codes<3> {
  u32x4_t wa, wb; u32x2_t hs[4];
  __device__ __forceinline__ explicit Codes(const Raw<3>& r) : wa(r.w << 2), wb(r.w >> 6) { shift_hi_plane(r.h, hs); }
  // the 2-bit field with the plane's bit right above it: one 3-bit field, the subnormal (or, with the bit at
  // position 10, smallest normal) fp16 number code * 2^(pos - 24)
  __device__ __forceinline__ half8_t lo(int slot) const {
    return as_half8(__builtin_bit_cast(u32x4_t, unpack2(wa, wb, slot)) | __builtin_bit_cast(u32x4_t, unpack1(hs, slot)));
  }
};
template <> struct Codes<4> {
  u32x4_t wa[2], wb[2];
  __device__ __forceinline__ explicit Codes(const Raw<4>& r) { wa[0] = r.w[0] << 2; wa[1] = r.w[1] << 2; wb[0] = r.w[0] >> 6; wb[1] = r.w[1] >> 6; }
  __device__ __forceinline__ half8_t lo(int slot) const { return unpack4(wa[slot >> 2], wb[slot >> 2], slot & 3); }
};

// One tile in flight: the lane's 16 bytes of metadata (Key scale pair, Key minimum pair, Value scale
// pair, Value minimum pair) and its share of the two code sections. The record of a tile is contiguous
// in memory, so a tile is three to five full-width loads from one stream.
template <int KB, int VB> struct Stage {
  u32x4_t meta;
  Raw<KB> kc; Raw<VB> vc;
  // rec: buffer resource over the unit's records; t: tile index inside the unit (wave-uniform)
  // l16: 16 * lane
  __device__ __forceinline__ void load(rsrc_t rec, int t, uint32_t l16) {
    const uint32_t l8 = l16 >> 1;
    const uint32_t soff = (uint32_t)t * (uint32_t)(record_words(KB, VB) * 4);
    meta = buf_load16(rec, l16, soff);
    kc.load(rec, soff + (uint32_t)(kMetaWords * 4), l16, l8);
    vc.load(rec, soff + (uint32_t)((kMetaWords + tile_words(KB)) * 4), l16, l8);
  }
};

// Groups whose split partials tell of themselves: a word is zero until it has been stored (see the split merge).
template <int G> constexpr bool kTagged = G <= 4;
constexpr int kMaxTries = 1 << 16;      // a round trip to memory each
__device__ __forceinline__ float not_zero(float v) { return v == 0.0f ? -0.0f : v; }
__device__ __forceinline__ void st_agent2(uint64_t* p, float2_t v) {
  const float a = not_zero(v[0]), b = not_zero(v[1]);
  __hip_atomic_store(p, (uint64_t)__builtin_bit_cast(uint32_t, a) | (uint64_t)__builtin_bit_cast(uint32_t, b) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// 8 bytes past the caches of the XCD, as an agent-scope load reads them (sc1)
constexpr int kAgent = 16;
__device__ __forceinline__ u32x2_t ld_agent2(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, kAgent));
}
__device__ __forceinline__ void st_agent2_zero(rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{0, 0}, r, (int)voff, (int)soff, kAgent);
}
// workgroup barrier that orders LDS accesses but waits for no access to memory
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ half2_t as_half2(uint32_t v) { return __builtin_bit_cast(half2_t, v); }
__device__ __forceinline__ uint32_t as_u32(half2_t v) { return __builtin_bit_cast(uint32_t, v); }
// Product of two fp16 pairs as packed fp16 pairs (hi, lo) with hi + lo == a * b to ~21 bits: hi is the product
// rounded to fp16 (one packed multiply), lo the residual of the exact product against that same register (one
// packed fused multiply-add; the residual of an fp16 product is itself an fp16 number unless it falls below
// 2^-24, where it is off by at most 2^-25 absolute).
__device__ __forceinline__ void mul_split(half2_t a, half2_t b, uint32_t& hi, uint32_t& lo) {
  const half2_t h = a * b;
  const half2_t l = __builtin_elementwise_fma(a, b, -h);
  hi = as_u32(h);
  lo = as_u32(l);
}
// fp32 pair -> packed fp16 pairs (hi, lo) with hi + lo == x to ~22 bits.
// The hi parts come from the truncating packed conversion, an intrinsic of its own: written as a plain
// cast, the multiply that produced x may get fused into one of the two uses of the hi part only, and the
// stored hi part and the one the lo part refers to then differ by a double rounding.
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t& hi, uint32_t& lo) {
  const half2_t hv = __builtin_bit_cast(half2_t, __builtin_amdgcn_cvt_pkrtz(x0, x1));
  const half_t l0 = (half_t)(x0 - (float)hv[0]), l1 = (half_t)(x1 - (float)hv[1]);
  const half2_t lv = {l0, l1};
  hi = __builtin_bit_cast(uint32_t, hv);
  lo = __builtin_bit_cast(uint32_t, lv);
}
// fp32 pair -> packed fp16 pairs, hi rounded to nearest, lo what the rounding left (rounded): the remainder is taken with the fp16
// number as it is, without a conversion back (a tile of 16 heads: 16 vector instructions of 255 less).
__device__ __forceinline__ void split_nearest(float x0, float x1, uint32_t& hi, uint32_t& lo) {
  const half2_t hv = __builtin_convertvector(float2_t{x0, x1}, half2_t);
  hi = as_u32(hv);
  float r0, r1;       // (the exponentials behind x0 and x1 have passed the conversion above: nothing here reads them too early)
  asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r0) : "v"(hi), "v"(x0));
  asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r1) : "v"(hi), "v"(x1));
  const half2_t lv = __builtin_convertvector(float2_t{r0, r1}, half2_t);
  lo = as_u32(lv);
}
__device__ __forceinline__ half_t split_part(float x, bool lo_part) {
  const half2_t hv = __builtin_bit_cast(half2_t, __builtin_amdgcn_cvt_pkrtz(x, 0.0f));
  const half_t hi = hv[0];
  const half_t lo = (half_t)(x - (float)hi);
  return lo_part ? lo : hi;
}
__device__ __forceinline__ float lo_half(uint32_t v) { return (float)__builtin_bit_cast(half_t, (uint16_t)(v & 0xffffu)); }
__device__ __forceinline__ float hi_half(uint32_t v) { return (float)__builtin_bit_cast(half_t, (uint16_t)(v >> 16)); }

// Wave-private LDS exchange area.
// A matrix operand (16 columns x 128 reduction positions, or x 32 for one channel block of the Values) is kept in the order in
// which a wave reads it: piece P = 4 * ks + kq (8 reduction positions) holds 16 bytes per operand row, rows 0 .. G-1 the hi parts of
// the heads, rows G .. 2G-1 the lo parts (an immediate offset apart, so that one two-address LDS write stores both). The head's place is
// XORed with P % 4 from 4 heads on: the 4 bytes per lane of a write then fall into distinct banks, and so do the 16 bytes
// per lane of a read (measured: 4.5 cycles per read of 1 KiB, 8.4 with operand rows 272 bytes apart; with 4 or 8 heads the
// exchange area was what bound the packed loop).
// Up to 4 heads leave columns idle; nothing they compute is stored. Their lanes read 16 bytes of zeros that every step has at the
// same offset from its start: with the heads' operands repeated in them instead the matrix core takes more power and the clock goes
// down in a run of launches (4 heads: 2.13 GHz, 2.23 with zeros; 1 head: 2.21, 2.28). 8 layers of 128 units x 8200 tokens, 4 heads:
// 208.5 us repeated, 204.3 with zeros; 16 layers of 256 units x 4100 tokens, 1 head: 354.2, 351.9.
// The Key side of a tile is done with its part before the Value side writes its own, so the two share memory (the
// wave's LDS operations run in order; a fence between the steps pins the compiler): 16 waves per CU fit.
// With 1 or 2 heads the few rows are kept whole, 320 bytes apart: the lanes of one row read the same 16 bytes, and a write is
// contiguous.
template <int G> struct Operand {
  static constexpr bool kPieces = G >= 4;
  static constexpr int kPiece = kPieces ? 32 * G : 16;        // bytes from a row's 8 reduction positions to its next 8
  static constexpr int kRow = kPieces ? 16 : 320;             // bytes from a head to the next
  static constexpr bool kIdle = G <= 4;                       // there are columns not in use
  static constexpr int kStep = 4 * kPiece + (kPieces && kIdle ? 16 : 0);      // bytes per ks (Keys) or channel block (Values)
  static constexpr int kLo = kRow * G;                        // from a head's hi part to its lo part
  static constexpr int kZeroAt = kPieces ? 4 * kPiece : 2 * G * kRow;         // the zeros of step 0: behind its pieces, or behind the rows
  static constexpr int kBytes = kPieces ? 4 * kStep : 2 * G * kRow + 3 * kStep + 16;
  // byte offset of the 4 bytes (reduction positions 2l, 2l+1 of the whole operand) that lane l writes for head hh
  static __device__ __forceinline__ int write_at(int l, int hh) { return (l >> 4) * kStep + ((l >> 2) & 3) * kPiece + 4 * (l & 3) + kRow * (hh ^ (kPieces ? (l >> 2) & 3 : 0)); }
  // byte offset of the 16 bytes that a lane (column of head h, part) reads as k-quarter kq of step 0
  static __device__ __forceinline__ int read_at(int kq, int h, bool lo) { return kq * kPiece + kRow * (h ^ (kPieces ? kq : 0)) + (lo ? kLo : 0); }
};
// Groups of 8 heads: the 16 columns are all in use, and every lane folds the scales into its own operand instead (the
// scales of the tile go through LDS, not the products: 2 bytes per position instead of 32): the two-address writes of the
// products took half of the LDS time, which bound the loop.
template <int G> constexpr bool kOwnOperand = G >= 8;
// Blocks of 16 heads, one head per column: see process_wide.
template <int G> constexpr bool kWide = G == 16;
template <int G> struct __attribute__((aligned(16))) WaveLds {
  static constexpr int kOpBytes = kOwnOperand<G> ? kD * 2 : Operand<G>::kBytes;
  struct Key {
    char op[kOpBytes];            // scale-folded query (own operand: the Key scales [channel])
    uint16_t zk[kD];              // Key zero-points of the tile [channel]
  };
  struct Value {
    char op[kOpBytes];               // scale-folded numerators (own operand: the Value scales [block][token])
    // scores of the tile [row][token] (rows: head h hi 2h, lo 2h + 1). Pitch 144 B: the rows are written 16 bytes per lane by
    // the 16 columns at once, and with a pitch of 128 B all rows would start in the same banks (measured: the two
    // stores of a tile took as long as all its other LDS traffic)
    float s[kWide<G> ? 1 : 2 * G][kTile + 4];
    char pq[kWide<G> ? 16 : Operand<G>::kStep];      // softmax numerators as two fp16 terms, an operand of 32 positions
    uint16_t zv[4][kTile];           // Value zero-points [channel block][token]
  };
  union { Key k; Value v; };
};

template <int G, int NW> struct MergeLds {        // per-wave reference maximum and sum of numerators of every head
  float m[NW][G];
  float l[NW][G];
};

// MIXED: Keys and Values age at fronts of their own (blocks of 1, 2, 4 and 16 heads); the tiles between the fronts have one side in
// a record and the other in the ring. Two kinds of tile share a half with the window tiles and are worked on with them, two with
// the packed ones:
//   Value front ahead: Keys from the ring, Values from the record (with the packed tiles); where the front stands inside a tile, the tokens
//     behind it are a window tile of which only they count.
//   Key front ahead: Keys from the record, Values from the ring (with the window tiles); the tokens before a front inside a tile are a
//     packed tile of which only they count.
// In a launch of their own on the vector unit these tiles took 13 us (14 tiles per unit of 128, 256 units, 1 head) next to 28 for
// the rest; a decode step of two such layers, with its appends and flushes, went from 103 us to 80.4, of two layers of 64 units x
// 3000 tokens and 8 heads from 103 to 47.
// The parameters in front of `a` (fields of it, see the first lines) are the 14 words that a workgroup finds in its scalar
// registers when it starts (they are preloaded: build.py): what a wave needs for its query and its first packed tile. Read from
// memory, three reads in a row as the code comes to them, they kept the first requests back: 24 units x 4 heads, 6 splits 7.28 ->
// 6.97 us per launch, 8 units x 8 heads x 2000 tokens 7.35 -> 6.99, 32 units x 1 head, 3 splits 6.06 -> 5.90; all read together at
// the start 7.24, 7.20, 6.11. Few parameters: each costs the host's launch some 15 ns.
template <int KB, int VB, int G, int NW, bool MIXED>
__global__ __launch_bounds__(NW * kWave, NW == 12 ? 3 : 4) void decode_attn_kernel(
    const uint16_t* q, const uint32_t* packed, u32x4_t shares, u32x4_t items, u32x2_t heads, AttnArgs a) {
  constexpr int kWaves = NW;
  constexpr int kThreads = kWaves * kWave;
  // per wave: the exchange area of the packed tiles; before that, the staging area in which a window tile's
  // Value rows (token-major in memory) are turned into matrix-core operands (8 consecutive tokens per lane)
  // and, once the wave has worked through its tiles, its result (a wave's memory is its own: a wave that is
  // done never waits for the others)
  union __attribute__((aligned(256))) WaveArea { WaveLds<G> x; uint16_t t[kTile][kD]; float o[G][kD + 16]; };   // result rows 64 bytes apart modulo a pass over the banks
  __shared__ WaveArea s_wave[kWaves];
  __shared__ MergeLds<G, NW> R;
  __shared__ int s_next;   // next unclaimed packed tile of this workgroup
  __shared__ int s_done;   // waves that have delivered their result

  a.q = q; a.packed = packed;
  a.n_splits = (int)shares[0]; a.win_each = (int)shares[1]; a.win_extra = (int)shares[2]; a.win_tiles = (int)shares[3];
  a.items_q = (int)items[0]; a.items_r = (int)items[1]; a.tiles_cap = (int)items[2]; a.n_w = (int)items[3];
  a.G = (int)heads[0]; a.head_blocks = (int)heads[1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // said to be uniform: what depends on it alone lives in scalar registers
  const int col = lane & 15, kq = lane >> 4;         // MFMA column / row index, k-quarter
  const int h = col & (G - 1);                       // head of the column (columns past the used ones repeat them)
  const bool lo_part = !kWide<G> && col >= 8;
  const bool col_valid = (col & 7) < G;              // the column's results are stored
  const int sp = blockIdx.x, u = blockIdx.y;
  // Query groups of more than 8 heads run as blocks of 8 or 16 heads in workgroups of their own (grid z): the blocks
  // of a unit read the same records and window rows at about the same time, so a tile comes from HBM once and from
  // the caches after that. uo numbers the (unit, head block) pairs; blocks of 8: rows uo*8 .. uo*8+7 of q and out.
  // Blocks of 16: the last one of a group may be partly empty; its idle columns repeat the group's last head.
  const int uo = u * a.head_blocks + (int)blockIdx.z;
  const int head0 = kWide<G> ? (int)blockIdx.z * G : 0;              // first head of the block inside the unit's group
  const int n_heads = kWide<G> ? (a.G - head0 < G ? a.G - head0 : G) : G;
  WaveLds<G>& L = s_wave[wave].x;
  uint16_t (&T)[kTile][kD] = s_wave[wave].t;
  const int row = 2 * h + (lo_part ? 1 : 0);         // score row of this lane's column
  const int op_read = Operand<G>::kIdle && !col_valid ? Operand<G>::kZeroAt : Operand<G>::read_at(kq, h, lo_part);

  // Work of this split: of the window's live tiles (numbered by age) those with index sp, sp + n_splits, ..., so that every split
  // carries its share of them, and a contiguous range of packed tiles. The first a.win_extra splits have one window tile more than
  // the others and a.win_tiles packed tiles less. (Quotient and remainder come from the host: the start of a launch is
  // latency-bound and integer division takes hundreds of instructions here.)
  const int extra = sp < a.win_extra ? sp : a.win_extra;
  const int p_begin = sp * a.items_q + (sp < a.items_r ? sp : a.items_r) - extra * a.win_tiles;
  const int p_end = p_begin + a.items_q + (sp < a.items_r ? 1 : 0) - (sp < a.win_extra ? a.win_tiles : 0);
  const int n_win = a.win_each + (sp < a.win_extra ? 1 : 0);

  // ---- the query and the wave's first tile are requested before anything else is done.
  // Packed tiles are claimed from a workgroup counter; the first claims are static (wave order).
  const size_t row0 = kWide<G> ? (size_t)u * a.G + head0 : (size_t)uo * G;      // first of the block's rows of q and out
  const uint16_t* qbase = a.q + row0 * kD;   // heads of unit u = (b, j) are rows (b*Hkv + j)*G .. +G-1 of q and out
  half8_t qB[4];       // plain q as B operand: the column's head (hi and lo columns alike, zero in columns not in use)
  constexpr bool kLateQuery = MIXED && G == 4 && VB == 4;      // (next to the tiles between two fronts there are no registers for it: read in front of the packed ones)
  uint32_t qraw[G];    // q of channels (2*lane, 2*lane+1) of every head (not needed where the lanes make their own operands)
  // loaded by the hi columns in use only (a load's cost at the start of a launch is its active lanes), copied to the lo columns later;
  // groups of 1 or 2 heads use it for window tiles only, and the other waves' requests are better spent on their first tiles (16 layers of
  // 256 units: 356.4 us with, 352.9 us without)
  const bool needs_q = MIXED || G > 2 || wave < a.win_each + (sp < a.win_extra ? 1 : 0);
#pragma unroll
  for (int ks = 0; ks < 4; ks++) {
    qB[ks] = half8_t{0, 0, 0, 0, 0, 0, 0, 0};
    if (needs_q && col < G) qB[ks] = *reinterpret_cast<const half8_t*>(qbase + (col < n_heads ? col : n_heads - 1) * kD + 32 * ks + 8 * kq);
  }
  auto copy_q_to_lo = [&]() {
    if constexpr (kWide<G>) return;
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      u32x4_t v = __builtin_bit_cast(u32x4_t, qB[ks]);
#pragma unroll
      for (int i = 0; i < 4; i++) { const int w = (int)v[i]; v[i] = (uint32_t)__builtin_amdgcn_update_dpp(w, w, 0x128, 0xf, 0xc, false); }   // row_ror:8 into lanes 8..15
      qB[ks] = as_half8(v);
    }
  };
#pragma unroll
  for (int hh = 0; hh < G; hh++) qraw[hh] = kOwnOperand<G> || kLateQuery ? 0u : reinterpret_cast<const uint32_t*>(qbase + hh * kD)[lane];

  constexpr uint32_t kRecBytes = (uint32_t)(record_words(KB, VB) * 4);
  const rsrc_t up = make_rsrc(reinterpret_cast<const char*>(a.packed) + (size_t)u * a.tiles_cap * kRecBytes, (uint32_t)a.tiles_cap * kRecBytes);
  const int n_early = n_win < kWaves ? kWaves - n_win : 0;      // waves n_win .. kWaves-1 start on packed tiles
  const bool has_packed = p_end > p_begin;
  const bool early = wave >= n_win;
  // (written before the first load into LDS is issued: the compiler lets an LDS write wait for those)
  if (tid == 0) { s_next = p_begin + n_early; s_done = 0; }
  Stage<KB, VB> st;
  int it = p_end;
  uint32_t lane16 = 16u * lane;
  asm volatile("" : "+v"(lane16));     // kept in a register of its own: computed again it would land in one that a pending load fills, and wait

  // Window tile r (by age) of the unit: the Key rows as MFMA A operands (rows = tokens), the Value rows straight into the
  // wave's staging area (loads that write LDS: no registers are held while they are under way, which lets a wave fit
  // into 128 registers). The Value rows are requested when the Key rows have arrived: requested together they delay the
  // first packed tiles (16 layers of 256 units: 364 us, 360.5 us this way).
  // Fused append: the newest token of the unit is not in the window arrays yet. The wave that takes its tile reads
  // that one row from k_new / v_new instead of the ring, treats it like any other row of the tile (the host
  // counts it in n_w) and stores it into the ring for the steps to come.
  const int new_tau = a.new_slot & 31;
  auto win_slot = [&](int r) { int wi = a.w0_tile + r; wi = wi >= a.ring_tiles ? wi - a.ring_tiles : wi; return wi * kTile; };   // first slot of the tile
  // Whether a window tile is the new token's (wave-uniform). Not to be asked of a tile between two fronts: in a full ring the new
  // token may share the ring tile of the oldest Values, in rows before theirs.
  auto win_new = [&](int slot0) { return a.new_slot >= 0 && slot0 == (a.new_slot & ~31); };
  struct WinKeys { half8_t r[2][4]; };
  // live: tokens of the tile (from its first row on) that are there, at least one; has_new: the new token is the last of them
  auto win_load_k = [&](int slot0, int live, bool has_new, int lane, WinKeys& w) {
    const int col = lane & 15, kq = lane >> 4;
    const uint16_t* kw = a.k_win + ((size_t)u * a.W_cap + slot0) * kD;
    const uint16_t* kn = a.k_new + (size_t)u * kD;
#pragma unroll
    for (int m = 0; m < 2; m++) {
      const int tau = 8 * (col >> 2) + 4 * m + (col & 3);   // row `col` of M-tile m
      // a slot past the live tokens is not read: its lanes take the tile's first row instead (live, and already on its
      // way: a cache hit; k_new where the new token is that row), whose products the softmax mask discards
      const int tau_r = tau < live ? tau : 0;
      const uint16_t* rowp = (has_new && tau_r == new_tau) ? kn : kw + (size_t)tau_r * kD;
#pragma unroll
      for (int ks = 0; ks < 4; ks++) w.r[m][ks] = *reinterpret_cast<const half8_t*>(rowp + 32 * ks + 8 * kq);
    }
  };
  // Value rows 4j .. 4j+3 per instruction, 16 bytes per lane in lane order: chunk c (8 channels) of row t goes to chunk
  // c ^ swizzle(t) of its row, so that the transposing reads below find their 8 rows x 32 bytes in distinct banks.
  auto swizzle = [](int t) { return 2 * ((t & 3) + 4 * ((t >> 3) & 1)); };
  auto win_load_v = [&](int slot0, int live, bool has_new, int lo, int lane) {      // rows from lo on (0 but for tiles between two fronts)
    const int col = lane & 15, kq = lane >> 4;
    // The resource spans the tile's rows that are live and in the ring (a new token is the last live row of its tile and not in
    // the ring yet). Rows beyond it are not read: their lanes write zeros, which meet a weight of zero (a dead slot may hold infinities
    // and NaN). A resource over the tile: a ring may be larger than 32-bit offsets reach.
    const int n_rows = has_new ? new_tau : live < kTile ? live : kTile;
    const rsrc_t rows = make_rsrc(a.v_win + ((size_t)u * a.W_cap + slot0) * kD, (uint32_t)n_rows * (kD * 2));
#pragma unroll
    for (int j = 0; j < 8; j++)
      buf_load_to_lds16(rows, (MIXED && 4 * j + kq < lo ? 0x40000000u : 0u) + 256u * (4 * j + kq) + 16u * (col ^ (2 * kq) ^ ((j & 2) ? 8 : 0)), 0, &T[4 * j][0]);
  };
  // the append itself, one row of each side, 16 lanes each: requested with the tile, then stored into the ring and (the
  // Value row) into the staging area
  auto append_load = [&](bool has_new) {
    u32x4_t x = {0, 0, 0, 0};
    if (has_new && lane < 32) x = *reinterpret_cast<const u32x4_t*>((lane >= 16 ? a.v_new : a.k_new) + (size_t)u * kD + 8 * col);
    return x;
  };
  auto append_stage = [&](const u32x4_t& x) {
    if (lane >= 16 && lane < 32) *reinterpret_cast<u32x4_t*>(&T[new_tau][8 * (col ^ swizzle(new_tau))]) = x;
  };
  auto append_store = [&](const u32x4_t& x) {
    if (lane < 32) *reinterpret_cast<u32x4_t*>((lane >= 16 ? a.v_win_w : a.k_win_w) + ((size_t)u * a.W_cap + a.new_slot) * kD + 8 * col) = x;
  };
  // The only workgroup barrier before the results are merged: the counters are set. It must not wait for the
  // loads just requested (a full __syncthreads would): LDS serves a wave's operations in order, so waiting for
  // the wave's LDS operations before the barrier is all that the two counter writes need. Both kinds of wave pass a barrier
  // of their own code path: what a wave has requested before it stays in registers of that path alone.
  auto start_barrier = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");   // no memory access of the code below moves above the barrier
  };

  // q of the lane's two channels, prescaled so that code products of all four channel blocks come out in the
  // same unit: the field of block ks sits at bit field_pos(ks), the query is scaled by 2^(field_pos(0) - field_pos(ks))
  // (exact in fp16 for |q| >= 2^-8; smaller values lose bits far below anything the scores resolve)
  constexpr int kPos0 = field_pos<KB>(0);
  const half_t pre = (half_t)__builtin_ldexpf(1.0f, kPos0 - field_pos<KB>(lane >> 4));
  half2_t qh[G];
#pragma unroll
  for (int hh = 0; hh < G; hh++) qh[hh] = as_half2(qraw[hh]) * half2_t{pre, pre};
  // plain query of step ks, prescaled likewise (lanes that make their own operands; computed anew for every tile: 12 more registers
  // around the loop do not fit, and with the power of two on the Key scales instead small scales would lose bits)
  auto q_scaled = [&](int ks) {
    const int e = kPos0 - field_pos<KB>(ks);
    if (e == 0) return qB[ks];
    const half_t f = (half_t)__builtin_ldexpf(1.0f, e);
    uint32_t w = as_u32(half2_t{f, f});
    asm volatile("" : "+s"(w));
    const half2_t f2 = as_half2(w);
    return qB[ks] * half8_t{f2[0], f2[1], f2[0], f2[1], f2[0], f2[1], f2[0], f2[1]};
  };
  // zero outside the lo columns
  const uint32_t lo_mask = lo_part ? 0xFFFFFFFFu : 0u;
  auto lo_only = [&](half8_t v, uint32_t signs = 0) {      // signs: 0x80008000 for the negative
    u32x4_t w = __builtin_bit_cast(u32x4_t, v);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      uint32_t t = (w[i] ^ signs) & lo_mask;
      asm("" : "+v"(t));      // (a sign taken off the result is an operand modifier then, not a bit operation on the masked word)
      w[i] = t;
    }
    return as_half8(w);
  };

  const half8_t zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  const half8_t ones8 = {1, 1, 1, 1, 1, 1, 1, 1};
  const float c_code = a.scale_log2 * __builtin_ldexpf(1.0f, 24 - kPos0);   // code products carry 2^(field_pos(0) - 24)
  const float c_plain = a.scale_log2;

  float4_t acc[8];
  float4_t accZ = {0, 0, 0, 0};
#pragma unroll
  for (int m = 0; m < 8; m++) acc[m] = float4_t{0, 0, 0, 0};
  float mref = -INFINITY;

  // online softmax of the lane's 8 tokens (8*kq + e of the tile, column col). The score of token e is
  // s[e]*c + z (log2 domain) summed over the hi and lo columns; z is zero in lo columns. Raises the
  // reference if needed (rescaling the accumulators) and returns the numerators 2^(score - reference).
  // raises the per-column reference to cover mx (log2-domain upper estimate of the tile's scores,
  // identical in all lanes of a column pair) and rescales the accumulators accordingly
  auto raise_reference = [&](float mx) {
    if (__any(mx > mref + kRefCap)) {
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mnew = mx > mref + kRefCap ? mx + kRefMargin : mref;
      const float f = (mnew == mref) ? 1.0f : fast_exp2(mref - mnew);
      mref = mnew;
      accZ *= f;
#pragma unroll
      for (int m = 0; m < 8; m++) acc[m] *= f;
    }
  };
  // (No inline assembly here: an instruction that reads what the matrix core writes has to wait for it, and only the compiler's own
  // are made to.)
  auto max8 = [](const float (&s)[8]) {
    float mx = fmaxf(fmaxf(s[0], s[1]), s[2]);
    mx = fmaxf(fmaxf(mx, s[3]), s[4]);
    mx = fmaxf(fmaxf(mx, s[5]), s[6]);
    return fmaxf(mx, s[7]);
  };

  // claiming a tile: the counter update is issued early (lane 0) and its result taken after the tile in
  // between has been worked on, so that the LDS round trip is not waited for
  auto grab_issue = [&]() -> int {
    int t = 0;
    if (lane == 0) t = __hip_atomic_fetch_add(&s_next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return t;
  };
  auto grab_take = [](int t) -> int { return __builtin_amdgcn_readfirstlane(t); };
  auto grab = [&]() -> int { return grab_take(grab_issue()); };

  constexpr bool kSmall = G <= 2;
  // A window tile once the scores of its tokens are there (x[e] * c + z, log2 domain, in both columns of a head; tokens that do not count:
  // -infinity) and its Value rows requested: online softmax, sums.
  auto absorb_window = [&](const float (&x)[8], float c, auto z, int ln, bool has_new, const u32x4_t& appended) {
    float p[8];
    constexpr bool kPlain = !std::is_same_v<decltype(z), float>;     // no z
    if constexpr (kPlain) raise_reference(max8(x) * c);
    else raise_reference(max8(x) * c + z);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      if constexpr (kPlain) p[e] = fast_exp2(x[e] * c - mref);
      else p[e] = fast_exp2(x[e] * c + (z - mref));
    }
    half8_t PB, PL;                                      // (blocks of 16: both parts in every column)
#pragma unroll
    for (int e = 0; e < 8; e++) { PB[e] = split_part(p[e], lo_part); if constexpr (kWide<G>) PL[e] = split_part(p[e], true); }
    accZ = mfma16(col >= 4 ? ones8 : zero8, PB, accZ);   // rows 4..15 accumulate the sum of numerators
    if constexpr (kWide<G>) accZ = mfma16(col >= 4 ? ones8 : zero8, PL, accZ);
    __builtin_amdgcn_sched_barrier(0);       // (not in front of the numerators)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the Value rows are in the staging area
    if (has_new) append_stage(appended);
    wave_lds_fence();
    // lane's part of the transposing reads: rows 8*kq + col/4 (+ 4), channels 4 * (col % 4) .. +3 of a block of 16
    const int cc = ln & 15, k4 = ln >> 4;
    const int t_off = (8 * k4 + (cc >> 2)) * (kD * 2) + ((((cc & 3) >> 1) ^ (2 * (cc >> 2) + 8 * (k4 & 1))) << 4) + 8 * (cc & 1);
#pragma unroll
    for (int m = 0; m < 8; m++) {
      const half8_t Avm = read_transposed(reinterpret_cast<const char*>(&T[0][0]), t_off ^ (m << 5));
      float4_t t = mfma16(Avm, PB, float4_t{0, 0, 0, 0});
      if constexpr (kWide<G>) t = mfma16(Avm, PL, t);
      if constexpr (VB == 3) {   // the final 7/3 step factor of channels 10 / 21 applies to codes only
#pragma unroll
        for (int r4 = 0; r4 < 4; r4++) {
          const int dd = 16 * (m & 1) + 4 * kq + r4;
          if (dd == 10 || dd == 21) t[r4] *= (3.0f / 7.0f);
        }
      }
      acc[m] += t * __builtin_ldexpf(1.0f, field_pos<VB>(m & 3) - 24);
      if (m & 1) __builtin_amdgcn_sched_barrier(0);      // (reads of all eight blocks hoisted together do not fit the registers)
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the staging area has been read: it is free again
  };

  auto op_write = [&](int hh) { return Operand<G>::write_at(lane, hh); };
  // the zeros of the idle columns (nothing but window rows and results is ever written to these places)
  auto zero_idle = [&]() {
    if constexpr (Operand<G>::kIdle) {
      if (lane < 4) *reinterpret_cast<u32x4_t*>(&L.k.op[Operand<G>::kZeroAt + lane * Operand<G>::kStep]) = u32x4_t{0, 0, 0, 0};
      if constexpr (Operand<G>::kPieces) {
        if (lane == 4) *reinterpret_cast<u32x4_t*>(&L.v.pq[Operand<G>::kZeroAt]) = u32x4_t{0, 0, 0, 0};
      }
      wave_lds_fence();
    }
  };
  // Key sides of a packed tile: code sums S of the lane's tokens (8*kq + 4*m + r) and column, zero-point terms zt.
  // EXACT (a tile between two fronts): codes as normal numbers and the query as it is; the sums come out in the same unit.
  const float kExactKeys = __builtin_ldexpf(1.0f, kPos0 - kExactPos);
  auto key_operand = [](auto exact, const Codes<KB>& kc, int slot) { return decltype(exact)::value ? exact_codes<KB>(kc.lo(slot), slot & 3) : kc.lo(slot); };
  auto keys_small = [&](auto exact, const u32x4_t& meta, const Raw<KB>& kr, float4_t (&S)[2], float (&zt)[G]) {
    constexpr bool EXACT = decltype(exact)::value;
    // Lane owns channels 2*lane, 2*lane+1: scale-folded query to LDS, zero-point term by dot product
    const half2_t s2 = as_half2(meta[0]);
    const uint32_t kz_pair = meta[1];   // a copy: a bit cast applied to the vector element itself reads element 0
#pragma unroll
    for (int hh = 0; hh < G; hh++) {
      uint32_t hi, lo;
      mul_split(EXACT ? as_half2(qraw[hh]) : qh[hh], s2, hi, lo);
      *reinterpret_cast<uint32_t*>(&L.k.op[op_write(hh)]) = hi;
      *reinterpret_cast<uint32_t*>(&L.k.op[op_write(hh) + Operand<G>::kLo]) = lo;
      const float zp = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, qraw[hh]), __builtin_bit_cast(half2_t, kz_pair), 0.0f, false);
      zt[hh] = wave_sum(zp) * c_plain;
    }
    wave_lds_fence();
    const Codes<KB> kc(kr);
    half8_t Bk[4];
#pragma unroll
    for (int ks = 0; ks < 4; ks++) Bk[ks] = *reinterpret_cast<const half8_t*>(&L.k.op[op_read + ks * Operand<G>::kStep]);
    S[0] = float4_t{0, 0, 0, 0}; S[1] = float4_t{0, 0, 0, 0};
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
      for (int ks = 0; ks < 4; ks++) S[m] = mfma16(key_operand(exact, kc, ks + 4 * m), Bk[ks], S[m]);
    if constexpr (EXACT) { S[0] *= kExactKeys; S[1] *= kExactKeys; }
    if constexpr (KB == 3) {   // tokens 10 and 21 of the group step by s*7/3
      if (kq == 1) S[0][2] *= (7.0f / 3.0f);
      if (kq == 2) S[1][1] *= (7.0f / 3.0f);
    }
  };
  // Groups of 4 heads (the others only compile these).
  auto keys_large = [&](auto exact, const u32x4_t& meta, const Raw<KB>& kr, float4_t (&S)[2], float& zt) {
    if constexpr (G != 4) return;
    constexpr bool EXACT = decltype(exact)::value;
    half2_t qx[G];        // (as it is, the query is read again: no registers for it around the loop)
#pragma unroll
    for (int hh = 0; hh < G; hh++) qx[hh] = EXACT ? as_half2(reinterpret_cast<const uint32_t*>(qbase + hh * kD)[lane]) : qh[hh];
    // Cooperative operand preparation: lane owns channels 2*lane, 2*lane+1.
    const half2_t s2 = as_half2(meta[0]);
#pragma unroll
    for (int hh = 0; hh < G; hh++) {
      uint32_t hi, lo;
      mul_split(qx[hh], s2, hi, lo);
      *reinterpret_cast<uint32_t*>(&L.k.op[op_write(hh)]) = hi;
      *reinterpret_cast<uint32_t*>(&L.k.op[op_write(hh) + Operand<G>::kLo]) = lo;
    }
    reinterpret_cast<uint32_t*>(&L.k.zk[0])[lane] = meta[1];
    wave_lds_fence();
    const Codes<KB> kc(kr);
    half8_t Bk[4];
    float4_t Sz = {0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      const half8_t z8 = *reinterpret_cast<const half8_t*>(&L.k.zk[32 * ks + 8 * kq]);
      Sz = mfma16(z8, qB[ks], Sz);     // every A row is the zero-point vector
      Bk[ks] = *reinterpret_cast<const half8_t*>(&L.k.op[op_read + ks * Operand<G>::kStep]);
    }
    S[0] = float4_t{0, 0, 0, 0}; S[1] = float4_t{0, 0, 0, 0};
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
      for (int ks = 0; ks < 4; ks++) S[m] = mfma16(key_operand(exact, kc, ks + 4 * m), Bk[ks], S[m]);
    if constexpr (EXACT) { S[0] *= kExactKeys; S[1] *= kExactKeys; }
    if constexpr (KB == 3) {   // tokens 10 and 21 of the group step by s*7/3
      if (kq == 1) S[0][2] *= (7.0f / 3.0f);
      if (kq == 2) S[1][1] *= (7.0f / 3.0f);
    }
    zt = Sz[0] * c_plain;
  };
  auto keys_wide = [&](auto exact, const u32x4_t& meta, const Raw<KB>& kr, float4_t (&S)[2], float& zt) {
    if constexpr (!kWide<G>) return;
    constexpr bool EXACT = decltype(exact)::value;
    reinterpret_cast<uint32_t*>(L.k.op)[lane] = meta[0];
    reinterpret_cast<uint32_t*>(&L.k.zk[0])[lane] = meta[1];
    wave_lds_fence();
    const Codes<KB> kc(kr);
    float4_t Sz = {0, 0, 0, 0};
    S[0] = float4_t{0, 0, 0, 0}; S[1] = float4_t{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      const half8_t z8 = *reinterpret_cast<const half8_t*>(&L.k.zk[32 * ks + 8 * kq]);
      const half8_t s8 = *reinterpret_cast<const half8_t*>(&L.k.op[64 * ks + 16 * kq]);
      Sz = mfma16(z8, qB[ks], Sz);       // every A row is the zero-point vector
      const half8_t qp = EXACT ? qB[ks] : q_scaled(ks), hi = qp * s8, lo = __builtin_elementwise_fma(qp, s8, -hi);
#pragma unroll
      for (int m = 0; m < 2; m++) {
        const half8_t c = key_operand(exact, kc, ks + 4 * m);
        S[m] = mfma16(c, hi, S[m]);
        S[m] = mfma16(c, lo, S[m]);
      }
    }
    if constexpr (EXACT) { S[0] *= kExactKeys; S[1] *= kExactKeys; }
    if constexpr (KB == 3) {   // tokens 10 and 21 of the group step by s*7/3
      if (kq == 1) S[0][2] *= (7.0f / 3.0f);
      if (kq == 2) S[1][1] *= (7.0f / 3.0f);
    }
    zt = Sz[0] * c_plain;
  };
  // Tiles between the fronts whose Values come from the record: dealt out like the window tiles, the waves without one of those first.
  const int n_rec = !MIXED ? 0 : a.m_ahead ? a.m_tiles : a.m_front > a.m_first * kTile ? 1 : 0;
  const int first_rec = sp + (kWaves - 1 - wave) * a.n_splits;
  // 4 heads (and 1 head with 4/3 bit): a wave that has some requests its first packed tile after them. Held in registers meanwhile,
  // the tile made 13 of the 16 kernels spill, and scratch memory alone costs a launch 2 to 3 us (128 units x 4 heads x 4000 tokens,
  // 3/4 bit, 800 Keys and 400 Values in fp16: 36.4 us, 20.9 this way; 2/4 bit 24.9, 19.8). The others have the registers, and lose
  // 3 to 13 % when the tile comes late.
  constexpr bool kLateTile = MIXED && (G == 4 || (G == 1 && KB == 4 && VB == 3));
  const bool late_tile = kLateTile && first_rec < n_rec;
  // ---- fp16 window tiles: taken round-robin by the waves before the packed stream.
  // Past the end a wave re-reads the last tile (cache hit) and skips its work: the load stream and the
  // loop body stay uniform, which keeps the outstanding-load accounting exact.
  const int live_tiles = (a.n_w + kTile - 1) / kTile;
  // ring slot of tile j between the fronts
  auto mixed_slot = [&](int j) { int wi = a.m_ring + j; wi = wi >= a.ring_tiles ? wi - a.ring_tiles : wi; return wi * kTile; };
  if (!early) {
    int r = sp + wave * a.n_splits;                      // < the number of live tiles, since wave < n_win
    const int r_step = kWaves * a.n_splits;
    int left = (n_win - wave + kWaves - 1) / kWaves;     // tiles of this wave
    for (int begin = 1; left > 0; left--, r += r_step) {
      asm volatile("" : "+s"(begin));     // (keeps the first pass from being compiled a second time: the code is read cold at the start of a launch)
      int slot0, live, lo = 0;
      if (!MIXED || r < live_tiles) {
        slot0 = win_slot(r);
        live = a.n_w - r * kTile;
      } else {
        const int j = a.m_ahead ? a.m_tiles - 1 : r - live_tiles, t0 = (a.m_first + j) * kTile;
        slot0 = mixed_slot(j);
        live = a.m_end - t0;
        lo = a.m_front - t0;
      }
      // the lane number as a value of this iteration: addresses derived from it are not kept in registers around the loop
      int ln = lane;
      asm volatile("" : "+v"(ln));
      if constexpr (MIXED) {
        if (r >= live_tiles && !a.m_ahead) {      // Keys from the record
          const uint32_t soff = (uint32_t)(a.m_first + r - live_tiles) * kRecBytes;
          const u32x4_t meta = buf_load16(up, lane16, soff);
          Raw<KB> kr;
          kr.load(up, soff + (uint32_t)(kMetaWords * 4), lane16, lane16 >> 1);
          __builtin_amdgcn_sched_barrier(0);
          if (begin) start_barrier();
          __builtin_amdgcn_sched_barrier(0);
          if (begin) copy_q_to_lo();
          begin = 0;
          zero_idle();
          float4_t S[2];
          float z = 0.0f;
          if constexpr (kSmall) {
            float zt[G];
            keys_small(std::true_type{}, meta, kr, S, zt);
#pragma unroll
            for (int hh = 0; hh < G; hh++) z = h == hh ? zt[hh] : z;
          } else if constexpr (kWide<G>) {
            keys_wide(std::true_type{}, meta, kr, S, z);
          } else {
            float zt;
            keys_large(std::true_type{}, meta, kr, S, zt);
            const float other = ror8(zt);
            z = lo_part ? other : zt;
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (the exchange area is about to take the Value rows)
          win_load_v(slot0, live, false, lo, ln);
          float x[8];
#pragma unroll
          for (int m = 0; m < 2; m++)
#pragma unroll
            for (int r4 = 0; r4 < 4; r4++) {
              const float sum = kWide<G> ? S[m][r4] : S[m][r4] + ror8(S[m][r4]);
              x[4 * m + r4] = 8 * kq + 4 * m + r4 >= lo ? sum : -INFINITY;
            }
          absorb_window(x, c_code, z, ln, false, u32x4_t{0, 0, 0, 0});
          continue;
        }
      }
      WinKeys wk;
      const bool has_new = (!MIXED || r < live_tiles) && win_new(slot0);
      win_load_k(slot0, live, has_new, ln, wk);
      const u32x4_t appended = append_load(has_new);
      __builtin_amdgcn_sched_barrier(0);      // (matrix instructions moved up here would wait for their rows in front of the barrier)
      if (begin) start_barrier();
      __builtin_amdgcn_sched_barrier(0);
      if (begin) copy_q_to_lo();
      begin = 0;
      float4_t S[2] = {float4_t{0, 0, 0, 0}, float4_t{0, 0, 0, 0}};
#pragma unroll
      for (int m = 0; m < 2; m++)
#pragma unroll
        for (int ks = 0; ks < 4; ks++) S[m] = mfma16(wk.r[m][ks], qB[ks], S[m]);
      win_load_v(slot0, live, has_new, lo, ln);
      float x[8];
#pragma unroll
      for (int m = 0; m < 2; m++)
#pragma unroll
        for (int r4 = 0; r4 < 4; r4++) {
          const int tau = 8 * kq + 4 * m + r4;
          x[4 * m + r4] = tau < live && (!MIXED || tau >= lo) ? S[m][r4] : -INFINITY;
        }
      absorb_window(x, c_plain, std::false_type{}, ln, has_new, appended);
      if (has_new) append_store(appended);                 // (after the reads: those would wait for a store in front of them)
    }
    if (has_packed) {   // claim the first packed tile now
      it = grab();
      if (!late_tile) st.load(up, it < p_end ? it : p_end - 1, lane16);
    }
  }
  // (a condition of its own: as the else of the one above it would be laid out in front of it, and the loads above would then wait
  // for the query, behind which the registers they share with the tile become free)
  int early_s = __builtin_amdgcn_readfirstlane(early ? 1 : 0);
  asm volatile("" : "+s"(early_s));
  if (early_s) {
    it = p_begin + (wave - n_win);
    if (has_packed && !late_tile) st.load(up, it < p_end ? it : p_end - 1, lane16);
    __builtin_amdgcn_sched_barrier(0);
    start_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kOwnOperand<G>) copy_q_to_lo();      // (smaller groups use the lo columns for window tiles only)
  }

  // ---- small query groups (G <= 2): the matrix core's columns are nearly empty, so the per-tile extras
  // (Key zero-point term, Value zero-point term, sum of numerators) are cheaper on the vector unit:
  // a packed dot product plus a wave reduction, and per-lane running sums reduced once at the end.
  float lwin = 0.0f;            // window tiles' sum of numerators of the lane's column (hi + lo)
  float lacc[G], zacc[G];       // running sum of numerators / of numerator * Value minimum over the lane's tokens
  float mref_u[G];              // reference of head hh, the same value in every lane
  if constexpr (kSmall) {
    lwin = __shfl(accZ[0], 16 + col);
    lwin += ror8(lwin);
#pragma unroll
    for (int hh = 0; hh < G; hh++) {
      lacc[hh] = 0.0f; zacc[hh] = 0.0f;
      mref_u[hh] = uniform_lane(mref, hh);
    }
  }
  const float inv_c_code = 1.0f / c_code;

  // sums: code or plain products of the tile's tokens in the columns' rows of L.v.s, scores sum * c + zt; tokens from `limit` on (MIXED)
  // do not count
  auto scores_out = [&](const float4_t (&S)[2]) {
    if (col_valid) {
      *reinterpret_cast<float4_t*>(&L.v.s[row][8 * kq]) = S[0];
      *reinterpret_cast<float4_t*>(&L.v.s[row][8 * kq + 4]) = S[1];
    }
  };
  // Adds the products of the codes of block m (16 channels) and the lanes' operands: hi, and lo where that is an operand of its own.
  auto add_values = [&](auto exact, const Codes<VB>& vc, int m, half8_t hi, auto... lo) {
    if constexpr (decltype(exact)::value) {
      const half8_t c = exact_codes<VB>(vc.lo(m), m & 3);
      float4_t t = mfma16(c, hi, float4_t{0, 0, 0, 0});
      ((t = mfma16(c, lo, t)), ...);
      acc[m] += t * __builtin_ldexpf(1.0f, field_pos<VB>(m & 3) - kExactPos);
    } else {
      const half8_t c = vc.lo(m);
      acc[m] = mfma16(c, hi, acc[m]);
      ((acc[m] = mfma16(c, lo, acc[m])), ...);
    }
  };
  auto values_small = [&](auto exact, const u32x4_t& meta, const Raw<VB>& vr, float c, float inv_c, const float (&zt)[G], int limit) {
    wave_lds_fence();
    // -- Value side. Lane (tp, g) owns tokens (2*tp, 2*tp+1) of channel block g.
    {
      const int tp = lane & 15;
      const float s0 = lo_half(meta[2]), s1 = hi_half(meta[2]);
      const float z0 = lo_half(meta[3]), z1 = hi_half(meta[3]);
      float sum0[G], sum1[G];
      bool over = false;
#pragma unroll
      for (int hh = 0; hh < G; hh++) {
        const float2_t sh = *reinterpret_cast<const float2_t*>(&L.v.s[2 * hh][2 * tp]);
        const float2_t sl = *reinterpret_cast<const float2_t*>(&L.v.s[2 * hh + 1][2 * tp]);
        sum0[hh] = 2 * tp < limit ? sh[0] + sl[0] : -INFINITY;
        sum1[hh] = 2 * tp + 1 < limit ? sh[1] + sl[1] : -INFINITY;
        // score = sum * c + zt; it exceeds what the reference allows iff sum > (reference + cap - zt) / c
        over |= fmaxf(sum0[hh], sum1[hh]) > (mref_u[hh] + kRefCap - zt[hh]) * inv_c;
      }
      if (__any(over)) {   // rare: raise the reference of the heads that need it and rescale what was accumulated
#pragma unroll
        for (int hh = 0; hh < G; hh++) {
          const float mx = wave_max(fmaxf(sum0[hh], sum1[hh])) * c + zt[hh];
          if (mx > mref_u[hh] + kRefCap) {          // wave-uniform
            const float mnew = mx + kRefMargin;
            const float f = fast_exp2(mref_u[hh] - mnew);      // 0 for the first tile (reference -inf)
            mref_u[hh] = mnew;
            lacc[hh] *= f; zacc[hh] *= f;
            if (h == hh) {                // the lanes of this head's columns
              mref = mnew;
              lwin *= f;
#pragma unroll
              for (int m = 0; m < 8; m++) acc[m] *= f;
            }
          }
        }
      }
#pragma unroll
      for (int hh = 0; hh < G; hh++) {
        const float off = zt[hh] - mref_u[hh];
        const float p0 = fast_exp2(sum0[hh] * c + off);
        const float p1 = fast_exp2(sum1[hh] * c + off);
        lacc[hh] += p0 + p1;
        zacc[hh] += p0 * z0 + p1 * z1;
        uint32_t hi, lo;
        split_pair(p0 * s0, p1 * s1, hi, lo);
        *reinterpret_cast<uint32_t*>(&L.v.op[op_write(hh)]) = hi;          // lane 16 g + tp: positions 2 tp, 2 tp + 1 of block g
        *reinterpret_cast<uint32_t*>(&L.v.op[op_write(hh) + Operand<G>::kLo]) = lo;
      }
    }
    wave_lds_fence();
    {
      const Codes<VB> vc(vr);
      half8_t Bv[4];
#pragma unroll
      for (int g = 0; g < 4; g++) Bv[g] = *reinterpret_cast<const half8_t*>(&L.v.op[op_read + g * Operand<G>::kStep]);
#pragma unroll
      for (int m = 0; m < 8; m++) add_values(exact, vc, m, Bv[m >> 1]);
    }
    wave_lds_fence();   // the next tile's operand writes come after these reads
  };
  auto process_small = [&](const Stage<KB, VB>& st) {
    float4_t S[2];
    float zt[G];
    keys_small(std::false_type{}, st.meta, st.kc, S, zt);
    scores_out(S);
    values_small(std::false_type{}, st.meta, st.vc, c_code, inv_c_code, zt, kTile);
  };

  auto values_large = [&](auto exact, const u32x4_t& meta, const Raw<VB>& vr, float (&x)[8], float c, float zt) {
    if constexpr (G != 4) return;
    // Reference maximum from the hi column (the lo column changes a score by < 2^-10 of its size, which a
    // reference does not need); lo lanes take their partner's value so that a column pair stays in step.
    float mx = max8(x) * c + zt;
    const float mx_partner = ror8(mx);        // cross-lane read outside any divergent branch: all lanes must take part
    mx = lo_part ? mx_partner : mx;
    raise_reference(mx);
    // log2-domain scores against the reference; the zero-point term and the reference enter through the hi column
    const float off_col = lo_part ? 0.0f : zt - mref;
#pragma unroll
    for (int e = 0; e < 8; e++) x[e] = x[e] * c + off_col;

    // -- Value side. Scores to LDS; lane (tp, g) then owns tokens (2*tp, 2*tp+1) of channel block g.
    if (col_valid) {
      *reinterpret_cast<float4_t*>(&L.v.s[row][8 * kq]) = float4_t{x[0], x[1], x[2], x[3]};
      *reinterpret_cast<float4_t*>(&L.v.s[row][8 * kq + 4]) = float4_t{x[4], x[5], x[6], x[7]};
    }
    wave_lds_fence();
    // The four lane groups g would all compute the same numerators; instead group g finishes those of head g and hands them to the
    // others through LDS as two fp16 terms (the rounded value and what the rounding left over: together ~22 bits, the same pair
    // enters the Value sums, the zero-point sums and the denominator).
    {
      const int tp = lane & 15, hh = lane >> 4;
      // (both reads are issued before the first write: the compiler does not move LDS reads across LDS writes through pointers of the same
      // type, and one read at a time costs an LDS round trip each)
      const float2_t sh = *reinterpret_cast<const float2_t*>(&L.v.s[2 * hh][2 * tp]);
      const float2_t sl = *reinterpret_cast<const float2_t*>(&L.v.s[2 * hh + 1][2 * tp]);
      // leading terms rounded to nearest: they are multiplied on their own below, and a truncated leading term
      // whose remainder's product falls below the fp16 range would bias the sums (plain casts are safe here:
      // the values come out of the exponential instruction, nothing can be fused into the conversions)
      const float p0 = fast_exp2(sh[0] + sl[0]), p1 = fast_exp2(sh[1] + sl[1]);
      uint32_t hv, lv;
      split_nearest(p0, p1, hv, lv);
      const int at = Operand<G>::write_at(tp, hh);
      *reinterpret_cast<uint32_t*>(&L.v.pq[at]) = hv;
      *reinterpret_cast<uint32_t*>(&L.v.pq[at + Operand<G>::kLo]) = lv;
      reinterpret_cast<uint32_t*>(&L.v.zv[0][0])[lane] = meta[3];
    }
    wave_lds_fence();
    half8_t Bv[4];
    // plain numerators: the column's own row
    const half8_t PB = *reinterpret_cast<const half8_t*>(&L.v.pq[op_read]);
    {
      const int tp = lane & 15;
      const half2_t s2 = as_half2(meta[2]);
      uint32_t pw[G], dw[G];
#pragma unroll
      for (int hh = 0; hh < G; hh++) {
        const int at = Operand<G>::write_at(tp, hh);
        pw[hh] = *reinterpret_cast<const uint32_t*>(&L.v.pq[at]);
        dw[hh] = *reinterpret_cast<const uint32_t*>(&L.v.pq[at + Operand<G>::kLo]);
      }
#pragma unroll
      for (int hh = 0; hh < G; hh++) {
        const half2_t p2 = as_half2(pw[hh]), d2 = as_half2(dw[hh]);
        // (p2 + d2) * s2: exact product of the leading term in two parts, the small term's product folded into the second
        const half2_t hv = p2 * s2;
        const half2_t lv = __builtin_elementwise_fma(d2, s2, __builtin_elementwise_fma(p2, s2, -hv));
        *reinterpret_cast<uint32_t*>(&L.v.op[op_write(hh)]) = as_u32(hv);
        *reinterpret_cast<uint32_t*>(&L.v.op[op_write(hh) + Operand<G>::kLo]) = as_u32(lv);
      }
      wave_lds_fence();
#pragma unroll
      for (int g = 0; g < 4; g++) Bv[g] = *reinterpret_cast<const half8_t*>(&L.v.op[op_read + g * Operand<G>::kStep]);
    }
    {
      const Codes<VB> vc(vr);
      // zero-point term: A rows 0..3 carry the zero-points of channel blocks 0..3, rows 4..15 are ones
      // and accumulate the sum of the numerators
      half8_t z8 = ones8;
      if (col < 4) z8 = *reinterpret_cast<const half8_t*>(&L.v.zv[col][8 * kq]);
      accZ = mfma16(z8, PB, accZ);
#pragma unroll
      for (int m = 0; m < 8; m++) add_values(exact, vc, m, Bv[m >> 1]);
    }
    wave_lds_fence();   // the next tile's operand writes come after these reads
  };
  auto process_large = [&](const Stage<KB, VB>& st) {
    if constexpr (G != 4) return;
    float4_t S[2];
    float zt, x[8];
    keys_large(std::false_type{}, st.meta, st.kc, S, zt);
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
      for (int r = 0; r < 4; r++) x[4 * m + r] = S[m][r];
    values_large(std::false_type{}, st.meta, st.vc, x, c_code, zt);
  };
  // Blocks of 8 heads: every lane folds the scales into its own operands. In one piece: cut in two like the one for 4 heads, 4 of
  // its forms with 8 waves spill.
  auto process_own = [&](const Stage<KB, VB>& st) {
    if constexpr (!kOwnOperand<G> || kWide<G>) return;
    // -- Key side
    {
      reinterpret_cast<uint32_t*>(L.k.op)[lane] = st.meta[0];
      reinterpret_cast<uint32_t*>(&L.k.zk[0])[lane] = st.meta[1];
    }
    wave_lds_fence();
    float x[8], zt;
    {
      const Codes<KB> kc(st.kc);
      half8_t Bk[4];
      float4_t Sz = {0, 0, 0, 0};
#pragma unroll
      for (int ks = 0; ks < 4; ks++) {
        const half8_t z8 = *reinterpret_cast<const half8_t*>(&L.k.zk[32 * ks + 8 * kq]);
        Sz = mfma16(z8, qB[ks], Sz);     // every A row is the zero-point vector
        const half8_t s8 = *reinterpret_cast<const half8_t*>(&L.k.op[64 * ks + 16 * kq]);
        const half8_t qp = q_scaled(ks);
        Bk[ks] = __builtin_elementwise_fma(qp, s8, -lo_only(qp * s8));
      }
      float4_t S[2] = {float4_t{0, 0, 0, 0}, float4_t{0, 0, 0, 0}};
#pragma unroll
      for (int m = 0; m < 2; m++)
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
          S[m] = mfma16(kc.lo(ks + 4 * m), Bk[ks], S[m]);
        }
      if constexpr (KB == 3) {   // tokens 10 and 21 of the group step by s*7/3
        if (kq == 1) S[0][2] *= (7.0f / 3.0f);
        if (kq == 2) S[1][1] *= (7.0f / 3.0f);
      }
      zt = Sz[0] * c_plain;
#pragma unroll
      for (int m = 0; m < 2; m++)
#pragma unroll
        for (int r = 0; r < 4; r++) x[4 * m + r] = S[m][r];
    }
    // Reference maximum from the hi column (the lo column changes a score by < 2^-10 of its size, which a
    // reference does not need); lo lanes take their partner's value so that a column pair stays in step.
    float mx = max8(x) * c_code + zt;
    const float mx_partner = ror8(mx);        // cross-lane read outside any divergent branch: all lanes must take part
    mx = lo_part ? mx_partner : mx;
    raise_reference(mx);
    // log2-domain scores against the reference; the zero-point term and the reference enter through the hi column
    const float off_col = lo_part ? 0.0f : zt - mref;
#pragma unroll
    for (int e = 0; e < 8; e++) x[e] = x[e] * c_code + off_col;

    // -- Value side. Scores to LDS; lane (tp, g) then owns tokens (2*tp, 2*tp+1) of channel block g.
    if (col_valid) {
      *reinterpret_cast<float4_t*>(&L.v.s[row][8 * kq]) = float4_t{x[0], x[1], x[2], x[3]};
      *reinterpret_cast<float4_t*>(&L.v.s[row][8 * kq + 4]) = float4_t{x[4], x[5], x[6], x[7]};
    }
    wave_lds_fence();
    // The four lane groups g would all compute the same numerators; instead group g finishes those of the
    // heads 4k + g only and hands them to the others through LDS as two fp16 terms (the rounded value and what
    // the rounding left over: together ~22 bits, the same pair enters the Value sums, the zero-point sums and
    // the denominator).
    {
      const int tp = lane & 15, g = lane >> 4;
      // (all reads of a step are issued before its first write: the compiler does not move LDS reads across LDS
      // writes through pointers of the same type, and one read at a time costs an LDS round trip each)
      constexpr int kShare = G / 4 > 0 ? G / 4 : 1;   // (only used with 8 heads)
      float2_t sh[kShare], sl[kShare];
#pragma unroll
      for (int k = 0; k < G / 4; k++) {
        const int hh = 4 * k + g;                                  // differs between the lane groups
        sh[k] = *reinterpret_cast<const float2_t*>(&L.v.s[2 * hh][2 * tp]);
        sl[k] = *reinterpret_cast<const float2_t*>(&L.v.s[2 * hh + 1][2 * tp]);
      }
#pragma unroll
      for (int k = 0; k < G / 4; k++) {
        const int hh = 4 * k + g;
        // leading terms rounded to nearest: they are multiplied on their own below, and a truncated leading term
        // whose remainder's product falls below the fp16 range would bias the sums (plain casts are safe here:
        // the values come out of the exponential instruction, nothing can be fused into the conversions)
        const float p0 = fast_exp2(sh[k][0] + sl[k][0]), p1 = fast_exp2(sh[k][1] + sl[k][1]);
        uint32_t hv, lv;
        split_nearest(p0, p1, hv, lv);
        const int at = Operand<G>::write_at(tp, hh);
        *reinterpret_cast<uint32_t*>(&L.v.pq[at]) = hv;
        *reinterpret_cast<uint32_t*>(&L.v.pq[at + Operand<G>::kLo]) = lv;
      }
      reinterpret_cast<uint32_t*>(&L.v.zv[0][0])[lane] = st.meta[3];
      reinterpret_cast<uint32_t*>(L.v.op)[lane] = st.meta[2];
    }
    wave_lds_fence();
    half8_t Bv[4];
    // plain numerators: the column's own row
    const half8_t PB = *reinterpret_cast<const half8_t*>(&L.v.pq[op_read]);
    // hi columns: the rounded products p * s; lo columns: what the rounding left, and the small terms' products
    const half8_t p8 = *reinterpret_cast<const half8_t*>(&L.v.pq[Operand<G>::read_at(kq, h, false)]);
    const half8_t nx = lo_only(p8, 0x80008000u), dx = lo_only(PB);
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const half8_t s8 = *reinterpret_cast<const half8_t*>(&L.v.op[64 * g + 16 * kq]);
      Bv[g] = __builtin_elementwise_fma(dx, s8, __builtin_elementwise_fma(p8, s8, nx * s8));
    }
    {
      const Codes<VB> vc(st.vc);
      // zero-point term: A rows 0..3 carry the zero-points of channel blocks 0..3, rows 4..15 are ones
      // and accumulate the sum of the numerators
      half8_t z8 = ones8;
      if (col < 4) z8 = *reinterpret_cast<const half8_t*>(&L.v.zv[col][8 * kq]);
      accZ = mfma16(z8, PB, accZ);
#pragma unroll
      for (int m = 0; m < 8; m++) {
        acc[m] = mfma16(vc.lo(m), Bv[m >> 1], acc[m]);
      }
    }
    wave_lds_fence();   // the next tile's operand writes come after these reads
  };
  // Blocks of 16 heads (of groups of 16 and more, multi-query attention): a column is a head, the hi and lo parts are two matrix
  // instructions on the same accumulators. The scores come out with a lane holding 8 tokens of its head, which are the tokens of
  // its operand for the Values: softmax, numerators and operands stay in the lane, only the tile's scales and minima go through
  // LDS, and the codes are cut out once for 16 heads. Bound by instruction issue: about 240 vector and 38 matrix instructions per
  // tile and wave (255 with masks and numerator splits written out: 27 us at 72 heads x 32 sequences of 4096 tokens, and 22.8 with
  // these and the head-wise tail; blocks of 8 took 49).
  auto values_wide = [&](auto exact, const u32x4_t& meta, const Raw<VB>& vr, float (&x)[8], float c, float zt) {
    if constexpr (!kWide<G>) return;
    raise_reference(max8(x) * c + zt);
    const float off = zt - mref;
#pragma unroll
    for (int e = 0; e < 8; e++) x[e] = fast_exp2(x[e] * c + off);       // the numerators of tokens 8*kq + e
    reinterpret_cast<uint32_t*>(L.v.op)[lane] = meta[2];
    reinterpret_cast<uint32_t*>(&L.v.zv[0][0])[lane] = meta[3];
    wave_lds_fence();
    u32x4_t pw, rw;       // numerators as two fp16 terms: rounded to nearest, and the rest
#pragma unroll
    for (int e = 0; e < 4; e++) { uint32_t hv, lv; split_nearest(x[2 * e], x[2 * e + 1], hv, lv); pw[e] = hv; rw[e] = lv; }
    const half8_t P = as_half8(pw), R8 = as_half8(rw);
    // zero-point term: A rows 0..3 carry the zero-points of channel blocks 0..3, rows 4..15 are ones
    // and accumulate the sum of the numerators
    half8_t z8 = ones8;
    if (col < 4) z8 = *reinterpret_cast<const half8_t*>(&L.v.zv[col][8 * kq]);
    accZ = mfma16(z8, P, accZ);
    accZ = mfma16(z8, R8, accZ);
    const Codes<VB> vc(vr);
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const half8_t s8 = *reinterpret_cast<const half8_t*>(&L.v.op[64 * g + 16 * kq]);
      const half8_t hi = P * s8;
      const half8_t lo = __builtin_elementwise_fma(R8, s8, __builtin_elementwise_fma(P, s8, -hi));
#pragma unroll
      for (int m = 2 * g; m < 2 * g + 2; m++) add_values(exact, vc, m, hi, lo);
    }
    wave_lds_fence();   // the next tile's scales come after these reads
  };
  auto process_wide = [&](const Stage<KB, VB>& st) {
    if constexpr (!kWide<G>) return;
    float4_t S[2];
    float zt, x[8];
    keys_wide(std::false_type{}, st.meta, st.kc, S, zt);
#pragma unroll
    for (int m = 0; m < 2; m++)
#pragma unroll
      for (int r = 0; r < 4; r++) x[4 * m + r] = S[m][r];
    values_wide(std::false_type{}, st.meta, st.vc, x, c_code, zt);
  };
  auto process = [&](const Stage<KB, VB>& st) {
    if constexpr (kWide<G>) process_wide(st);
    else if constexpr (kSmall) process_small(st);
    else if constexpr (kOwnOperand<G>) process_own(st);
    else process_large(st);
  };

  if constexpr (MIXED) if (first_rec < n_rec) {
    zero_idle();
    for (int j = first_rec; j < n_rec; j += kWaves * a.n_splits) {
      const uint32_t soff = (uint32_t)(a.m_first + j) * kRecBytes;
      const int t0 = (a.m_first + j) * kTile;
      const int n_tok = (a.m_front < a.m_end ? a.m_front : a.m_end) - t0;        // tokens with a packed Value
      const int limit = n_tok < kTile ? n_tok : kTile;
      u32x4_t meta = buf_load16(up, lane16, soff);
      Raw<VB> vr;
      vr.load(up, soff + (uint32_t)((kMetaWords + tile_words(KB)) * 4), lane16, lane16 >> 1);
      float4_t S[2];
      float zts[G], ztl = 0.0f, c = c_code, inv_c = inv_c_code;
      if (a.m_ahead) {
        WinKeys wk;
        win_load_k(mixed_slot(j), a.m_end - t0, false, lane, wk);
        S[0] = float4_t{0, 0, 0, 0}; S[1] = float4_t{0, 0, 0, 0};
#pragma unroll
        for (int m = 0; m < 2; m++) {
#pragma unroll
          for (int ks = 0; ks < 4; ks++) S[m] = mfma16(wk.r[m][ks], qB[ks], S[m]);
#pragma unroll
          for (int e = 0; e < 4; e++) S[m][e] = lo_part ? 0.0f : S[m][e];
        }
#pragma unroll
        for (int hh = 0; hh < G; hh++) zts[hh] = 0.0f;
        c = c_plain;
        inv_c = 1.0f / c_plain;
      } else {
        Raw<KB> kr;
        kr.load(up, soff + (uint32_t)(kMetaWords * 4), lane16, lane16 >> 1);
        if constexpr (kSmall) keys_small(std::true_type{}, meta, kr, S, zts);
        else if constexpr (kWide<G>) keys_wide(std::true_type{}, meta, kr, S, ztl);
        else keys_large(std::true_type{}, meta, kr, S, ztl);
      }
      // what the record holds for tokens without a packed Value is not defined
      const int tp = lane & 15;
      const uint32_t keep = (2 * tp < limit ? 0x0000FFFFu : 0u) | (2 * tp + 1 < limit ? 0xFFFF0000u : 0u);
      meta[2] &= keep; meta[3] &= keep;
      if constexpr (kSmall) {
        scores_out(S);
        values_small(std::true_type{}, meta, vr, c, inv_c, zts, limit);
      } else {
        float x[8];
#pragma unroll
        for (int m = 0; m < 2; m++)
#pragma unroll
          for (int e = 0; e < 4; e++) x[4 * m + e] = 8 * kq + 4 * m + e < limit || lo_part ? S[m][e] : -INFINITY;
        if constexpr (kWide<G>) values_wide(std::true_type{}, meta, vr, x, c, ztl);
        else values_large(std::true_type{}, meta, vr, x, c, ztl);
      }
    }
    if constexpr (kLateTile) {
      Stage<KB, VB> first;       // (not st itself: what it holds without a packed tile would be kept)
      if (has_packed) first.load(up, it < p_end ? it : p_end - 1, lane16);
      st = first;
    }
  }

  if (has_packed) {
    if constexpr (kLateQuery) {
#pragma unroll
      for (int hh = 0; hh < G; hh++) qh[hh] = as_half2(reinterpret_cast<const uint32_t*>(qbase + hh * kD)[lane]) * half2_t{pre, pre};
    }
    zero_idle();
    // Two workgroups share a compute unit: of the waves that can issue a SIMD takes the oldest, so that the workgroup that came first
    // ran ahead and the other one was left with half of the unit's waves at the end (8 heads, 512 units of 126 tiles: first
    // workgroups done at 41 us, second ones at 51). With a.even a wave starts at the highest priority and takes one step down with
    // the first tile it claims past half of the workgroup's tiles, then past half of those that were left at that claim, twice: the
    // workgroup behind goes first, and both end together. After its tiles a wave has the lowest: results and merge don't hold up the
    // neighbour's tiles (kept at the level of its last claim, 512 units of 30 tiles took 17.8 us with 8 heads and 18.4 with 16; 17.5
    // and 17.7; at 126 tiles the same within 1 %. The level from the number of the claimed tile alone, several steps at once: 17.6 and
    // 18.3.)
    int prio = 0, next_at = p_end;
    if constexpr (kWaves == 8) {
      if (a.even && p_end - p_begin > 12) {      // (a handful of tiles, 32 units of 8: 6.2 us without, 6.4 with)
        prio = 3;
        next_at = p_begin + ((p_end - p_begin) >> 1);
        __builtin_amdgcn_s_setprio(3);
      }
    }
    while (it < p_end) {
      const int ticket = grab_issue();
      if constexpr (kWaves == 8) {
        if (it >= next_at) {
          prio--;
          next_at = prio > 0 ? it + ((p_end - it) >> 1) : p_end;
          if (prio == 2) __builtin_amdgcn_s_setprio(2);
          else if (prio == 1) __builtin_amdgcn_s_setprio(1);
          else __builtin_amdgcn_s_setprio(0);
        }
      }
      process(st);
      it = grab_take(ticket);
      st.load(up, it < p_end ? it : p_end - 1, lane16);
    }
    if constexpr (kWaves == 8) __builtin_amdgcn_s_setprio(0);
  }

  {
  // Where the packed loop has no register to spare, lane and thread number are made anew here (elsewhere the values at hand are
  // better: 0.17 us per launch of 32 units x 8 splits).
  constexpr bool kAnew = G == 4 && (MIXED ? KB == 3 && VB <= 2 : kWaves == 8 && ((KB >= 3 && VB >= 3) || (KB == 4 && VB == 2)));
  int lane = threadIdx.x & 63;
  if constexpr (kAnew) {
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(lane));
    __builtin_assume(lane >= 0 && lane < kWave);
  }
  const int tid = kAnew ? wave * kWave + lane : (int)threadIdx.x, col = lane & 15, kq = lane >> 4;
  // ---- per-wave result (into the wave's own area, whose exchange contents are no longer needed): undo the
  // field scaling, add hi and lo columns, add the zero-point term.
  // accZ: lanes with kq == 0 hold the zero-point sums of channel blocks 0..3, lanes with kq >= 1 the
  // sum of numerators (any register).
  float zsum[4];
  float lsum;
  if constexpr (kSmall) {
    // running sums: the lanes of row 0 cover all tokens once (numerators), the lanes of row g hold the
    // zero-point sums of channel block g; hi lanes take the whole term, lo lanes nothing
    lsum = lwin;
#pragma unroll
    for (int g = 0; g < 4; g++) zsum[g] = 0.0f;
#pragma unroll
    for (int hh = 0; hh < G; hh++) {
      const float lr = row_sum(lacc[hh]), zr = row_sum(zacc[hh]);
      const bool mine = col == hh;
      const float lt = uniform_lane(lr, 0);   // cross-lane reads stay outside divergent code: the source lane must be active
      lsum += mine ? lt : 0.0f;
#pragma unroll
      for (int g = 0; g < 4; g++) { const float t = uniform_lane(zr, 16 * g); zsum[g] = mine ? t : zsum[g]; }
    }
  } else {
#pragma unroll
    for (int g = 0; g < 4; g++) zsum[g] = __shfl(accZ[g], col);
    lsum = __shfl(accZ[0], 16 + col);
    if constexpr (!kWide<G>) lsum += ror8(lsum);
  }
#pragma unroll
  for (int m = 0; m < 8; m++) {
    const float sc = __builtin_ldexpf(1.0f, 24 - field_pos<VB>(m & 3));
    float4_t o4;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      float v = acc[m][r] * sc;
      if (VB == 3) {   // channels 10 and 21 of each block of 32 step by s*7/3
        const int dd = 16 * (m & 1) + 4 * kq + r;
        if (dd == 10 || dd == 21) v *= (7.0f / 3.0f);
      }
      v += zsum[m >> 1];
      o4[r] = kWide<G> ? v : v + ror8(v);
    }
    if (col < G) *reinterpret_cast<float4_t*>(&s_wave[wave].o[col][16 * m + 4 * kq]) = o4;   // channels 16m + 4kq .. +3
  }
  if (col < G && kq == 0) { R.m[wave][col] = mref; R.l[wave][col] = lsum; }

  // Wave w combines the waves' results of heads w, w + kWaves, ... of the block, a lane two channels: the weights 2^(m_w - M) once
  // per head (lane w holds the w-th), handed out as scalars.
  constexpr int kHeads = (G + kWaves - 1) / kWaves;       // heads per wave
  auto combine_head = [&](int hh, float2_t& ml, float2_t& O) {
    const float mw = lane < kWaves ? R.m[lane < kWaves ? lane : 0][hh] : -INFINITY, lw = lane < kWaves ? R.l[lane < kWaves ? lane : 0][hh] : 0.0f;
    float2_t o[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; w++) o[w] = *reinterpret_cast<const float2_t*>(&s_wave[w].o[hh][2 * lane]);
    const float M = uniform_lane(row_max(mw), 0);
    const float fw = (mw == -INFINITY) ? 0.0f : fast_exp2(mw - M);
    ml = float2_t{M, uniform_lane(row_sum(lw * fw), 0)};
    O = float2_t{0, 0};
#pragma unroll
    for (int w = 0; w < kWaves; w++) O += o[w] * uniform_lane(fw, w);
  };
  uint16_t* outp = a.out + row0 * kD;
  // partial of split s, head hh of the block: [unit][block][split][head of the block] (blocks of 16: [unit][split][head of the group])
  const size_t part0 = kWide<G> ? (size_t)u * a.n_splits * a.G + head0 : (size_t)uo * a.n_splits * G;
  const int part_step = kWide<G> ? a.G : G;
  auto part_at = [&](int s, int hh) { return a.part + (part0 + (size_t)s * part_step + hh) * (kD + 2); };
  auto put_out = [&](int hh, const float2_t& O, float Lsum) {
    const half2_t v = {(half_t)(O[0] / Lsum), (half_t)(O[1] / Lsum)};
    reinterpret_cast<uint32_t*>(outp + hh * kD)[lane] = as_u32(v);
  };

  if (a.n_splits == 1) {
    if constexpr (G <= 2) {
      // No barrier: a wave delivers its result and leaves; the last one to deliver combines them.
      // (LDS serves a wave's operations in order, so its results are in place before its count.)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      int done = 0;
      if (lane == 0) done = __hip_atomic_fetch_add(&s_done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      done = __builtin_amdgcn_readfirstlane(done);
      if (done != kWaves - 1) return;
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
      for (int hh = 0; hh < G; hh++) {
        float2_t ml, O;
        combine_head(hh, ml, O);
        put_out(hh, O, ml[1]);
      }
    } else {
      lds_barrier();
#pragma unroll
      for (int k = 0; k < kHeads; k++) {
        const int hh = wave + k * kWaves;
        float2_t ml, O;
        if (hh < n_heads) {
          combine_head(hh, ml, O);
          put_out(hh, O, ml[1]);
        }
      }
    }
    return;
  }

  // ---- split merge: every workgroup stores its partial, the last one of the unit to arrive combines them. Partials are stored and
  // loaded with agent scope, which the hardware keeps coherent per access across the XCDs' L2s: stores are written through to the
  // level that all XCDs share, loads miss the XCD's own, no cache-wide flush is needed.
  // Larger groups: a wave waits until its stores have completed; after a barrier the arrival is counted. Groups of up to 4 heads:
  // partials that tell of themselves. Every word of the partials is zero before and after a call; a split stores its words as
  // anything but zero (a zero as minus zero). The arrival is counted, by a wave of its own, before the partial is even combined:
  // the count is on its way meanwhile, and no store is waited for. The workgroup that arrives last knows that every other one of
  // the unit has its results and stores them without waiting for anything; it takes a partial when all of its words read as other
  // than zero. Stores that wait for nothing and a count that is back when they are issued, instead of stores, their
  // acknowledgement, a barrier and the count in a row: 32 units of 3 splits (one small layer) 6.37 -> 5.85 us, 24 units of 6 splits
  // and 4 heads 8.2 -> 7.6, 32 units of 8 splits 10.4 -> 9.6, 128 of 2 splits 24.9 -> 24.5; no change for 8 units of 32 splits, 66
  // KB to read and to zero for the one workgroup. Groups of 8 heads have no wave to spare for the count, and twice the words to
  // zero.
  static_assert(!kTagged<G> || G < kWaves);
  lds_barrier();          // the waves' results are in LDS
  uint32_t prev = 0;
  if constexpr (kTagged<G>) {
    if (tid == kThreads - 1) prev = __hip_atomic_fetch_add(&a.counters[uo * a.counter_stride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
#pragma unroll
  for (int k = 0; k < kHeads; k++) {
    const int hh = wave + k * kWaves;
    if (hh < n_heads) {
      float2_t ml, O;
      combine_head(hh, ml, O);
      uint64_t* row = reinterpret_cast<uint64_t*>(part_at(sp, hh));
      if (lane == 0) st_agent2(row, ml);
      st_agent2(row + 1 + lane, O);
    }
  }
  if constexpr (kTagged<G>) {
    if (tid == kThreads - 1) s_done = prev == (uint32_t)a.n_splits - 1u;   // reused as the "last workgroup" flag
    lds_barrier();
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's partial stores have completed ...
    __syncthreads();                                     // ... and so have those of all waves, before the arrival is counted
    if (tid == 0) {
      prev = __hip_atomic_fetch_add(&a.counters[uo * a.counter_stride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_done = prev == (uint32_t)a.n_splits - 1u;
    }
    __syncthreads();
  }
  if (!s_done) return;
  // The loads of all heads of a wave and up to kBatch parts are under way together, without a branch around each; parts past the
  // last one are read as the last one and weigh nothing. (Blocks of 16 heads used to take four round trips: 32 units x 72 heads, 3
  // splits, 27.5 -> 22.8 us per launch; 4 x 16 heads 12.0 -> 9.9; 8 units of 8 heads 10.1 -> 8.4.)
  const uint32_t part_bytes = (uint32_t)(part_step * (kD + 2) * sizeof(float));
  // hd: first head of the wave (every kWaves-th from there on); the splits from s_first on, a batch every s_step
  auto merge = [&](auto batch, int hd, int s_first, int s_step, auto put) {
    constexpr int kBatch = decltype(batch)::value;
    float M[kHeads], Lsum[kHeads];
    float2_t O[kHeads];
#pragma unroll
    for (int k = 0; k < kHeads; k++) { M[k] = -INFINITY; Lsum[k] = 0.0f; O[k] = float2_t{0, 0}; }
    for (int s0 = s_first; s0 < a.n_splits; s0 += s_step) {
      const int n = a.n_splits - s0 < kBatch ? a.n_splits - s0 : kBatch;       // >= 1
      u32x2_t ml[kHeads], os[kHeads][kBatch];
      // where the rows begin, one after the other by addition (with a product and a choice for each, launches of 8 and more heads
      // took 0 to 1.5 % longer)
      uint32_t at[kBatch];
      {
        const uint32_t last = (uint32_t)(s0 + n - 1) * part_bytes;
        at[0] = (uint32_t)s0 * part_bytes;
#pragma unroll
        for (int i = 1; i < kBatch; i++) {
          at[i] = at[i - 1] + part_bytes < last ? at[i - 1] + part_bytes : last;
          asm("" : "+s"(at[i]));
        }
      }
      // (tagged) The last arrival waits for stores that nothing holds up. The bound is for a counter that was not zero to begin
      // with, with which another arrival may count as the last; even then the missing workgroups are on their way. (Partials that
      // were not zero are taken for what they say.)
      for (int tries = 0;; tries++) {
        asm volatile("" ::: "memory");        // (to the compiler these loads see the same memory every time otherwise)
        uint32_t least = 1;
#pragma unroll
        for (int k = 0; k < kHeads; k++) {
          const int hh = hd + k * kWaves < n_heads ? hd + k * kWaves : n_heads - 1;
          const rsrc_t rows = make_rsrc(part_at(0, hh), (uint32_t)(a.n_splits - 1) * part_bytes + (kD + 2) * 4u);
          ml[k] = ld_agent2(rows, (uint32_t)(s0 + (lane < n ? lane : n - 1)) * part_bytes, 0);
#pragma unroll
          for (int i = 0; i < kBatch; i++) os[k][i] = ld_agent2(rows, 8u + 8u * lane, at[i]);
        }
        if constexpr (!kTagged<G>) break;
#pragma unroll
        for (int k = 0; k < kHeads; k++) {
          least = ml[k][0] < ml[k][1] ? ml[k][0] : ml[k][1];
#pragma unroll
          for (int i = 0; i < kBatch; i++) {
            least = os[k][i][0] < least ? os[k][i][0] : least;
            least = os[k][i][1] < least ? os[k][i][1] : least;
          }
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(least == 0u) == 0, 1)) break;
        // In vain: NaN as this batch's sum of numerators, so that the head comes out as NaN and not as a number without some of its
        // tokens. (Marking the counter as well, for later calls, costs every launch of 4 heads 0.1 us of 7 to 16.)
        if (__builtin_expect(tries == kMaxTries, 0)) { ml[0][1] = 0x7FC00000u; break; }
      }
      if constexpr (kTagged<G>) {
        if (s0 + s_step >= a.n_splits) lds_barrier();      // the wave has all of its rows: the waves that don't merge zero them
      }
#pragma unroll
      for (int k = 0; k < kHeads; k++) {
        const uint32_t mb = ml[k][0], lb = ml[k][1];      // (copies: a bit cast applied to an element itself reads element 0)
        const float mk = lane < n ? __builtin_bit_cast(float, mb) : -INFINITY, lk = __builtin_bit_cast(float, lb);
        // weights 2^(m_k - M) once per wave (lane i holds the i-th), handed out as scalars; cross-lane reads stay outside divergent code
        const float mrow = row_max(mk);
        float Mn = fmaxf(M[k], uniform_lane(mrow, 0));
        if constexpr (kBatch > 16) Mn = fmaxf(Mn, uniform_lane(mrow, 16));
        const float fold = (M[k] == -INFINITY) ? 0.0f : fast_exp2(M[k] - Mn);
        const float fk = (mk == -INFINITY) ? 0.0f : fast_exp2(mk - Mn);
        const float lrow = row_sum(lk * fk);
        Lsum[k] = Lsum[k] * fold + uniform_lane(lrow, 0);
        if constexpr (kBatch > 16) Lsum[k] += uniform_lane(lrow, 16);
        O[k] *= fold;
#pragma unroll
        for (int i = 0; i < kBatch; i++) {
          const uint32_t o0 = os[k][i][0], o1 = os[k][i][1];
          O[k] += float2_t{__builtin_bit_cast(float, o0), __builtin_bit_cast(float, o1)} * uniform_lane(fk, i);
        }
        M[k] = Mn;
      }
    }
#pragma unroll
    for (int k = 0; k < kHeads; k++)
      if (hd + k * kWaves < n_heads) put(hd + k * kWaves, O[k], Lsum[k], M[k]);
  };
  auto to_out = [&](int hh, const float2_t& O, float Lsum, float) { put_out(hh, O, Lsum); };
  if constexpr (kTagged<G>) {
    constexpr int kBatch = kWaves == 8 && G == 4 ? 16 : kMergeBatch;      // (4 heads, 8 waves: 32 do not fit the registers)
    // Many splits of 1 or 2 heads: 16 partials of one head to a wave, then the waves' sums like the waves' results before. (When
    // one wave took both batches of its head, with the zeros of the first in front of the second's loads, 4 units of 1 head in 50
    // splits took 9.0 us per launch; 7.4 now. With 32 splits and 4 heads two waves of 16 are slower than one of 32, 13.0 us against
    // 12.3, and the longer code costs the short launches 1 %.)
    constexpr int kRows = kWaves / G;      // x 16: at least 64
    const int rows = G == 4 || a.n_splits <= kBatch ? 1 : (a.n_splits + 15) / 16 < kRows ? (a.n_splits + 15) / 16 : kRows;
    const int merging = rows * G;      // waves
    if (wave >= merging) lds_barrier();
    else if (a.n_splits <= 8) merge(std::integral_constant<int, 8>{}, wave, 0, 8, to_out);
    else if (G == 4 || rows == 1) merge(std::integral_constant<int, kBatch>{}, wave, 0, kBatch, to_out);
    else if constexpr (G < 4) {
      const int hd = wave % G, row = wave / G;
      merge(std::integral_constant<int, 16>{}, hd, 16 * row, 16 * kRows, [&](int hh, const float2_t& O, float Lsum, float M) {
        if (lane == 0) { R.m[row][hh] = M; R.l[row][hh] = Lsum; }
        *reinterpret_cast<float2_t*>(&s_wave[row].o[hh][2 * lane]) = O;
      });
    }
    // Nobody else reads the unit's partials: zero again, the splits' rows one after the other, by the waves that don't merge while
    // the others sum up (by the merging waves where all of them merge). Zeroed by the merging waves ahead of their sums, whose
    // stores alone took 1.1 us then (behind the sums 0.1 us more), and now: 8 units of 4 heads, 32 splits 12.0 -> 11.4 us per
    // launch, 1 unit, 64 splits 16.4 -> 15.4; 8 units of 1 head, 8 splits 6.53 -> 6.38; 32 units, 3 splits 5.87 -> 5.77.
    if (wave >= merging || merging == kWaves) {
      const int first = merging == kWaves ? 0 : merging;
      const uint32_t bytes = (uint32_t)a.n_splits * part_bytes;          // a multiple of 8
      const rsrc_t all = make_rsrc(part_at(0, 0), bytes);
      for (uint32_t at = 16u * ((uint32_t)(wave - first) * kWave + lane); at + 16u <= bytes; at += 16u * kWave * (uint32_t)(kWaves - first))
        __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{0, 0, 0, 0}, all, (int)at, 0, kAgent);
      if ((bytes & 8u) && wave == first && lane == 0) st_agent2_zero(all, bytes - 8u, 0);
    }
    if constexpr (G < 4) if (rows > 1) {
      if (wave >= rows) {       // rows of no partial
        if (lane < G) { R.m[wave][lane] = -INFINITY; R.l[wave][lane] = 0.0f; }
#pragma unroll
        for (int hh = 0; hh < G; hh++) *reinterpret_cast<float2_t*>(&s_wave[wave].o[hh][2 * lane]) = float2_t{0, 0};
      }
      lds_barrier();
      if (wave < G) {
        float2_t ml, O;
        combine_head(wave, ml, O);
        put_out(wave, O, ml[1]);
      }
    }
  } else if (wave < n_heads) {
    if (a.n_splits <= 8) merge(std::integral_constant<int, 8>{}, wave, 0, 8, to_out);
    else {
      constexpr int kBatch = kHeads > 1 ? 16 : kMergeBatch;      // (32 do not fit the registers)
      merge(std::integral_constant<int, kBatch>{}, wave, 0, kBatch, to_out);
    }
  }
  if (tid == 0) __hip_atomic_store(&a.counters[uo * a.counter_stride], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <int KB, int VB>
hipError_t launch_g(const AttnArgs& a, int G, dim3 grid, hipStream_t s) {
  hipError_t e = hipErrorInvalidValue;
  auto run = [&](auto kernel) {
    const uint32_t u[10] = {(uint32_t)a.n_splits, (uint32_t)a.win_each, (uint32_t)a.win_extra, (uint32_t)a.win_tiles, (uint32_t)a.items_q, (uint32_t)a.items_r,
                            (uint32_t)a.tiles_cap, (uint32_t)a.n_w, (uint32_t)a.G, (uint32_t)a.head_blocks};
    u32x4_t shares = {u[0], u[1], u[2], u[3]}, items = {u[4], u[5], u[6], u[7]};
    u32x2_t heads = {u[8], u[9]};
    e = launch(kernel, grid, kNW * kWave, s, a.q, a.packed, shares, items, heads, a);
  };
  switch (G) {
    case 1: run(decode_attn_kernel<KB, VB, 1, kNW, kMixed>); break;
    case 2: run(decode_attn_kernel<KB, VB, 2, kNW, kMixed>); break;
    case 4: run(decode_attn_kernel<KB, VB, 4, kNW, kMixed>); break;
#if !KVMIX_MIXED
    case 8:
      // (a block of 8 heads with 3- or 4-bit Values has 12 waves: attn_waves)
      if constexpr (kNW == 12 || VB < 3) { run(decode_attn_kernel<KB, VB, 8, kNW, kMixed>); break; }
      else break;
#endif
#if KVMIX_WAVES == 8 || KVMIX_MIXED
    case 16: run(decode_attn_kernel<KB, VB, 16, kNW, kMixed>); break;
#endif
  }
  return e;
}

}  // namespace

template <>
hipError_t launch_decode_attn<kNW, kMixed>(const AttnArgs& a, int k_bits, int v_bits, int block, int units, hipStream_t s) {
  const dim3 grid(a.n_splits, units, a.head_blocks);
  switch (k_bits * 10 + v_bits) {
    case 11: return launch_g<1, 1>(a, block, grid, s);
    case 12: return launch_g<1, 2>(a, block, grid, s);
    case 13: return launch_g<1, 3>(a, block, grid, s);
    case 14: return launch_g<1, 4>(a, block, grid, s);
    case 21: return launch_g<2, 1>(a, block, grid, s);
    case 31: return launch_g<3, 1>(a, block, grid, s);
    case 41: return launch_g<4, 1>(a, block, grid, s);
    case 22: return launch_g<2, 2>(a, block, grid, s);
    case 23: return launch_g<2, 3>(a, block, grid, s);
    case 24: return launch_g<2, 4>(a, block, grid, s);
    case 32: return launch_g<3, 2>(a, block, grid, s);
    case 33: return launch_g<3, 3>(a, block, grid, s);
    case 34: return launch_g<3, 4>(a, block, grid, s);
    case 42: return launch_g<4, 2>(a, block, grid, s);
    case 43: return launch_g<4, 3>(a, block, grid, s);
    case 44: return launch_g<4, 4>(a, block, grid, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace kvmix
