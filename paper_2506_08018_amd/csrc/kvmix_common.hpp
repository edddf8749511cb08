// Shared definitions of the KVmix HIP library (gfx950). Not used by the CPU oracle.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include "../../include/kvmix.h"

namespace kvmix {

constexpr int kD = 128;        // head dimension
constexpr int kTile = 32;      // tokens per tile = Key group length = Value group width
constexpr int kWave = 64;

typedef _Float16 half_t;
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__host__ __device__ constexpr int tile_words(int bits) { return 128 * bits; }  // 32 x 128 codes
// A tile record: 256 metadata words, then the Key code section, then the Value code section.
constexpr int kMetaWords = 256;
__host__ __device__ constexpr int record_words(int k_bits, int v_bits) { return kMetaWords + tile_words(k_bits) + tile_words(v_bits); }
// 16-bit index, inside a record, of the metadata halves (f = 0 scale, 1 minimum)
__host__ __device__ constexpr int key_meta_half(int d, int f) { return 2 * (4 * (d >> 1) + f) + (d & 1); }
__host__ __device__ constexpr int value_meta_half(int tau, int g, int f) { return 2 * (4 * (16 * g + (tau >> 1)) + 2 + f) + (tau & 1); }

// Position of a code inside its tile (layout statement: include/kvmix.h).
// (l, j, hh, slot): 16-byte column, word in column, 16-bit half, slot in half.
struct CodePos { int word, bit, hword, hbit; };

__host__ __device__ inline CodePos pos_from_slots(int bits, int l, int j, int hh, int slot) {
  CodePos p;
  p.hword = -1; p.hbit = 0;
  if (bits == 1) {
    p.word = 2 * l + (j >> 1);
    p.bit = 16 * hh + 8 * (j & 1) + 2 * (slot & 3) + (slot >> 2);
    return p;
  }
  if (bits == 4) {
    p.word = 256 * (slot >> 2) + 4 * l + j;
    p.bit = 16 * hh + 4 * (slot & 3);
    return p;
  }
  p.word = 4 * l + j;
  p.bit = 16 * hh + 2 * slot;
  if (bits == 3) {
    p.hword = 256 + 2 * l + (j >> 1);
    p.hbit = 16 * hh + 8 * (j & 1) + 2 * (slot & 3) + (slot >> 2);
  }
  return p;
}

// Token / channel held by (column l, word j, half hh, slot) of a Key or Value tile.
__host__ __device__ inline void key_td(int l, int j, int hh, int slot, int& tau, int& d) {
  const int i = l & 15, kq = l >> 4, ks = slot & 3, m = slot >> 2;
  d = 32 * ks + 8 * kq + 2 * j + hh;
  tau = 8 * (i >> 2) + 4 * m + (i & 3);
}
__host__ __device__ inline void value_td(int l, int j, int hh, int slot, int& tau, int& d) {
  const int i = l & 15, kq = l >> 4;
  d = 16 * slot + i;
  tau = 8 * kq + 2 * j + hh;
}

// x = code * s_i + min (Sec. 3.2.2 step 4) of token tau, channel d of a tile record, in fp32 (multiply, then add);
// which = 0 Key, 1 Value. The straightforward form, for the helper kernels that are not bound by it.
__device__ inline float dequant_elem(const uint32_t* rec, int k_bits, int v_bits, int which, int tau, int d) {
  const uint16_t* meta = reinterpret_cast<const uint16_t*>(rec);
  const int bits = which ? v_bits : k_bits;
  const uint32_t* words = rec + kMetaWords + (which ? tile_words(k_bits) : 0);
  int l, j, hh, slot, gi, ms, mz;
  if (which == 0) {
    const int ks = d / 32, kq = (d % 32) / 8, m = (tau % 8) / 4, i = 4 * (tau / 8) + tau % 4;
    l = 16 * kq + i; j = (d % 8) / 2; hh = d % 2; slot = ks + 4 * m;
    ms = key_meta_half(d, 0); mz = key_meta_half(d, 1); gi = tau;
  } else {
    l = 16 * (tau / 8) + d % 16; j = (tau % 8) / 2; hh = tau % 2; slot = d / 16;
    ms = value_meta_half(tau, d / 32, 0); mz = value_meta_half(tau, d / 32, 1); gi = d % 32;
  }
  const CodePos p = pos_from_slots(bits, l, j, hh, slot);
  int code;
  if (bits == 3) code = ((words[p.word] >> p.bit) & 3u) + 4 * ((words[p.hword] >> p.hbit) & 1u);
  else code = (words[p.word] >> p.bit) & ((1u << bits) - 1u);
  const float s = (float)__builtin_bit_cast(half_t, meta[ms]);
  const float mn = (float)__builtin_bit_cast(half_t, meta[mz]);
  const float si = (bits == 3 && (gi == 10 || gi == 21)) ? (s * 7.0f) / 3.0f : s;
  const float prod = (float)code * si;
  return prod + mn;
}

// Launch descriptors filled by the C-ABI layer (host) and passed by value.
struct QuantArgs {
  // The token sequence that is quantized: its rows [0, n_ring) are the ring slots (ring_w0 + r) % W_cap of the two
  // fp16 windows ([units][W_cap][128]), every later row r is row r - n_ring of the input. Tile t takes rows
  // 32 t .. 32 t + 31.
  const uint16_t* k; const uint16_t* v;
  int64_t tok, unit_b, unit_h;                  // strides of both inputs (channel stride 1)
  const uint16_t* k_ring; const uint16_t* v_ring;
  int n_ring, ring_w0, W_cap;
  uint32_t* packed;
  int tiles_cap;   // tiles per unit in the packed cache
  int tile0;       // first destination tile
  int Hkv;
  // Input rows that stay in the window (an appending launch only): row copy_row + i, i = 0 .. n_copy - 1, goes to the ring slot
  // that lies copy_at + i slots behind ring_w0, around the ring. The slots [0, n_read) behind ring_w0 are also read by tiles of the
  // launch: the workgroup of the tile in question fills those, once it has its rows. The others are filled by copy_tiles workgroups
  // from n_tiles on, 32 slots each, from slot 32 copy_tile0 on.
  int n_tiles, n_copy, copy_row, copy_at, n_read, copy_tile0, copy_tiles;
  uint16_t* k_ring_w; uint16_t* v_ring_w;
  // Ageing with separate fronts (every row comes from the ring, which is the input then; row r of the launch is token 32*tile0 +
  // r): the Key side is written for the destination tiles [k_tile_a, k_tile_b) only, the Value side for the tokens [v_tok_a,
  // v_tok_b) only; everything else in the records is left as it is.
  int k_tile_a, k_tile_b, v_tok_a, v_tok_b;
};

struct DequantArgs {
  const uint32_t* packed;
  float* out; int tiles_cap; int n_tokens; int k_bits; int v_bits; int which;   // out: [units][n_tokens][128]
};

struct AppendArgs {
  const uint16_t* k_new; const uint16_t* v_new;   // element (b, j, i, d) at b*batch + j*head + i*tok + d
  int64_t tok, head, batch;
  uint16_t* k_win; uint16_t* v_win;
  int W_cap; int slot; int n; int units; int Hkv;   // tokens i = 0..n-1 go to ring slots (slot + i) % W_cap
};

struct AttnArgs {
  const uint16_t* q;
  const uint32_t* packed;
  const uint16_t* k_win; const uint16_t* v_win;
  // fused append: the newest token of every unit ([units][128] each) is not in the window arrays yet but counted
  // in n_w; the wave that takes the window tile of ring slot new_slot reads it from here and stores it
  const uint16_t* k_new; const uint16_t* v_new;
  int n_splits;
  // window tiles with live tokens: win_each per split, one more for the first win_extra splits
  int win_each, win_extra;
  // packed tiles: (packed tiles + win_extra * win_tiles) divided by n_splits, quotient and remainder; the splits with a
  // window tile more than the others take win_tiles packed tiles less
  int items_q, items_r, win_tiles;
  int tiles_cap, W_cap, n_w;
  int ring_tiles, w0_tile;       // W_cap / 32; ring tile that holds the oldest window token
  int new_slot;           // -1: nothing to append
  int G;                  // query heads per kv head
  int head_blocks;        // workgroups per (split, unit): grid z
  float scale_log2;       // softmax_scale * log2(e)
  int counter_stride;
  uint16_t* out;
  uint16_t* k_win_w; uint16_t* v_win_w;
  float* part;            // partials: [units][n_splits][G][kD + 2]
  uint32_t* counters;     // arrival counters (zero before and after every call), one per (unit, head block), counter_stride words apart
  // Tiles between two fronts (MIXED): tiles [m_first, m_first + m_tiles), tokens up to m_end;
  // m_front: the Value front; m_ahead: it is ahead of the Key front; m_ring: ring tile of tile m_first. The window tiles above are dealt
  // out together with those of them whose Values come from the ring.
  int m_first, m_tiles, m_end, m_front, m_ring;
  bool m_ahead;
  bool even;              // the workgroups that share a compute unit keep pace with each other (8 waves)
};

// A launch by hipLaunchKernel itself, without the configuration that <<<>>> pushes and pops (host time of a decode step of one
// launch 5.6 -> 5.3 us, with the preloaded parameters as few as they can be: passed one by one, 13 of them, it was 5.8).
template <typename... Params, typename... Args>
hipError_t launch(void (*kernel)(Params...), dim3 grid, int threads, hipStream_t s, const Args&... args) {
  static_assert((std::is_same_v<Params, Args> && ...), "an argument of its own type for each parameter");
  void* pointers[] = {const_cast<void*>(static_cast<const void*>(&args))...};
  const hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3(threads), pointers, 0, s);
  if (e != hipSuccess) (void)hipGetLastError();      // reported by the caller's status, not by a later call
  return e;
}

// over n_tiles tiles (and the window rows that a.n_copy names)
hipError_t launch_quantize_pack(QuantArgs a, int k_bits, int v_bits,
                                int n_tiles, int units, hipStream_t s);
hipError_t launch_quantize_fronts(const QuantArgs& a, int k_bits, int v_bits,
                                  int n_tiles, int units, hipStream_t s);
hipError_t launch_dequant(const DequantArgs& a, int units, hipStream_t s);
hipError_t launch_append(const AppendArgs& a, hipStream_t s);
hipError_t launch_stream_read(const void* buf, size_t bytes, int workgroups, int threads, uint32_t* sink, hipStream_t s);
// WAVES: waves per workgroup, 8 or 12 (blocks of 16 heads: 8). MIXED: with the tiles between two fronts (blocks of 1, 2, 4 and 16
// heads, 12 waves). block: query heads per workgroup (1, 2, 4, 8 or 16); a unit's group of a.G heads takes (a.G + block - 1) /
// block workgroups per split.
template <int WAVES, bool MIXED>
hipError_t launch_decode_attn(const AttnArgs& a, int k_bits, int v_bits, int block, int units, hipStream_t s);
template <> hipError_t launch_decode_attn<8, false>(const AttnArgs& a, int k_bits, int v_bits, int block, int units, hipStream_t s);
template <> hipError_t launch_decode_attn<12, false>(const AttnArgs& a, int k_bits, int v_bits, int block, int units, hipStream_t s);
template <> hipError_t launch_decode_attn<12, true>(const AttnArgs& a, int k_bits, int v_bits, int block, int units, hipStream_t s);

}  // namespace kvmix
