// C-ABI entry points of libkvmix: host-side validation and launch plumbing only.
// Contract and layout: include/kvmix.h.
#include <atomic>
#include <cmath>
#include <mutex>
#include "kvmix_common.hpp"

using namespace kvmix;

namespace {

std::atomic<int> g_last_hip_error{0};

constexpr int kMaxDevices = 64;

// Compute units of the current device, asked once per device (0 when the query fails).
int num_cus() {
  static std::atomic<int> cached[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) return 0;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

int hip_fail(hipError_t e) {
  g_last_hip_error.store((int)e);
  return KVMIX_ERR_HIP;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_shape_cfg(const kvmix_shape* sh, const kvmix_layer_cfg* cfg) {
  if (!sh || !cfg) return KVMIX_ERR_NULL;
  if (sh->group != kTile) return KVMIX_ERR_BAD_GROUP;
  if (sh->D != kD || sh->B < 1 || sh->Hkv < 1 || sh->Hq < 1 || sh->Hq % sh->Hkv) return KVMIX_ERR_BAD_SHAPE;
  const int G = sh->Hq / sh->Hkv;
  if (G != 1 && G != 2 && G != 4 && (G % 8 != 0 || G > 512)) return KVMIX_ERR_BAD_SHAPE;
  if ((long long)sh->B * sh->Hkv > 65535) return KVMIX_ERR_BAD_SHAPE;
  const int kb = cfg->k_bits, vb = cfg->v_bits;
  if (kb == 16 || vb == 16) {
    if (kb != 16 || vb != 16) return KVMIX_ERR_BAD_BITS;
  } else if (kb < 1 || kb > 4 || vb < 1 || vb > 4) {
    return KVMIX_ERR_BAD_BITS;
  }
  if (cfg->window != -1 && (cfg->window < 0 || cfg->window % kTile)) return KVMIX_ERR_BAD_SHAPE;
  return KVMIX_OK;
}

// ring slot of token t (both windows)
int slot_of(const kvmix_layer_cache* c, long long t) {
  long long s = (c->w0 + t - c->n_q) % c->W_cap;
  return (int)(s < 0 ? s + c->W_cap : s);
}
// tokens that live in the ring: from the older of the two fronts to the newest
int ring_tokens(const kvmix_layer_cache* c) { return c->n_w + (c->v_lead < 0 ? -c->v_lead : 0); }

int check_cache(const kvmix_layer_cfg* cfg, const kvmix_layer_cache* c, bool need_packed) {
  if (!c) return KVMIX_ERR_NULL;
  if (c->T_cap < 0 || c->T_cap % kTile || c->W_cap < kTile || c->W_cap % kTile) return KVMIX_ERR_BAD_SHAPE;
  if (c->n_q < 0 || c->n_q % kTile || c->n_q > c->T_cap) return KVMIX_ERR_BAD_SHAPE;
  if (c->n_w < 0 || c->n_w > c->W_cap || c->w0 < 0 || c->w0 >= c->W_cap || c->w0 % kTile) return KVMIX_ERR_BAD_SHAPE;
  if (c->v_lead > c->n_w || (long long)c->n_q + c->v_lead < 0 || (long long)c->n_w - c->v_lead > c->W_cap || (long long)c->n_q + c->v_lead > c->T_cap)
    return KVMIX_ERR_BAD_SHAPE;
  if (c->v_lead != 0 && cfg->k_bits == 16) return KVMIX_ERR_BAD_BITS;
  if (!c->k_win || !c->v_win) return KVMIX_ERR_NULL;
  if (!aligned16(c->k_win) || !aligned16(c->v_win)) return KVMIX_ERR_ALIGN;
  if (cfg->k_bits == 16) return c->n_q == 0 ? KVMIX_OK : KVMIX_ERR_BAD_BITS;
  if (need_packed || c->n_q > 0) {
    if (!c->packed) return KVMIX_ERR_NULL;
    if (!aligned16(c->packed)) return KVMIX_ERR_ALIGN;
    // a unit's records are addressed with 32-bit byte offsets
    if ((long long)(c->T_cap / kTile) * record_words(cfg->k_bits, cfg->v_bits) * 4 > 0x7fffffffLL) return KVMIX_ERR_BAD_SHAPE;
  }
  return KVMIX_OK;
}

// (unit, block of at most 8 query heads) pairs: each is one workgroup per split (blocks of 16 heads: at least half as many)
int out_units(const kvmix_shape* sh) {
  const int G = sh->Hq / sh->Hkv;
  return sh->B * sh->Hkv * (G > 8 ? G / 8 : 1);
}

int max_splits(const kvmix_shape* sh) {
  const int units = out_units(sh);
  int s = 512 / units;
  if (s < 8) s = 8;
  if (s > 64) s = 64;
  return s;
}

size_t counters_bytes(int units) { return (((size_t)units * 4 + 255) / 256) * 256; }

void fill_quant_dst(QuantArgs& a, const kvmix_layer_cache* c) {
  a.packed = c->packed;
  a.tiles_cap = c->T_cap / kTile;
}

}  // namespace

extern "C" {

int kvmix_version(void) { return 1; }

const char* kvmix_strerror(int status) {
  switch (status) {
    case KVMIX_OK: return "ok";
    case KVMIX_ERR_NULL: return "null pointer";
    case KVMIX_ERR_BAD_BITS: return "unsupported bit-width";
    case KVMIX_ERR_BAD_GROUP: return "unsupported group size";
    case KVMIX_ERR_BAD_SHAPE: return "unsupported shape or count";
    case KVMIX_ERR_ALIGN: return "misaligned pointer or stride";
    case KVMIX_ERR_WORKSPACE: return "workspace too small";
    case KVMIX_ERR_HIP: return "HIP error";
  }
  return "unknown status";
}

int kvmix_last_hip_error(void) { return g_last_hip_error.load(); }

int kvmix_cache_bytes(const kvmix_shape* sh, const kvmix_layer_cfg* cfg, int T_cap, int W_cap,
                      size_t* packed_b, size_t* win_b) {
  const int st = check_shape_cfg(sh, cfg);
  if (st) return st;
  if (T_cap < 0 || T_cap % kTile || W_cap < kTile || W_cap % kTile) return KVMIX_ERR_BAD_SHAPE;
  const size_t units = (size_t)sh->B * sh->Hkv, tiles = (size_t)T_cap / kTile;
  const bool packed = cfg->k_bits != 16;
  if (packed_b) *packed_b = packed ? units * tiles * record_words(cfg->k_bits, cfg->v_bits) * 4 : 0;
  if (win_b) *win_b = units * (size_t)W_cap * kD * 2;
  return KVMIX_OK;
}

int kvmix_workspace_bytes(const kvmix_shape* sh, int T_max, size_t* bytes) {
  kvmix_layer_cfg cfg = {2, 2, 0};
  const int st = check_shape_cfg(sh, &cfg);
  if (st) return st;
  if (!bytes) return KVMIX_ERR_NULL;
  if (T_max < 0) return KVMIX_ERR_BAD_SHAPE;
  const size_t units = (size_t)sh->B * sh->Hkv, G = (size_t)(sh->Hq / sh->Hkv);
  *bytes = counters_bytes(out_units(sh)) + units * (size_t)(max_splits(sh) + 1) * G * (kD + 2) * sizeof(float);
  return KVMIX_OK;
}

int kvmix_quantize_pack(const kvmix_shape* sh, const kvmix_layer_cfg* cfg, const uint16_t* k_fp16, const uint16_t* v_fp16,
                        int64_t token_stride, int64_t head_stride, int64_t batch_stride, int n_tokens, int t0,
                        const kvmix_layer_cache* c, void* stream) {
  int st = check_shape_cfg(sh, cfg);
  if (st) return st;
  if (cfg->k_bits == 16) return KVMIX_ERR_BAD_BITS;
  if (!k_fp16 || !v_fp16) return KVMIX_ERR_NULL;
  st = check_cache(cfg, c, true);
  if (st) return st;
  if (n_tokens < 0 || n_tokens % kTile || t0 < 0 || t0 % kTile || (long long)t0 + n_tokens > c->T_cap) return KVMIX_ERR_BAD_SHAPE;
  if (!aligned16(k_fp16) || !aligned16(v_fp16) || token_stride % 8 || head_stride % 8 || batch_stride % 8 || token_stride < kD)
    return KVMIX_ERR_ALIGN;
  QuantArgs a{};
  a.k = k_fp16; a.v = v_fp16;
  a.tok = token_stride; a.unit_b = batch_stride; a.unit_h = head_stride;
  a.n_ring = 0; a.W_cap = 1;
  fill_quant_dst(a, c);
  a.tile0 = t0 / kTile;
  a.Hkv = sh->Hkv;
  const hipError_t e = launch_quantize_pack(a, cfg->k_bits, cfg->v_bits, n_tokens / kTile, sh->B * sh->Hkv, (hipStream_t)stream);
  return e == hipSuccess ? KVMIX_OK : hip_fail(e);
}

int kvmix_append_tokens(const kvmix_shape* sh, const kvmix_layer_cfg* cfg, const uint16_t* k_new, const uint16_t* v_new,
                        int64_t token_stride, int64_t head_stride, int64_t batch_stride, int n_tokens,
                        kvmix_layer_cache* c, void* stream) {
  int st = check_shape_cfg(sh, cfg);
  if (st) return st;
  if (!k_new || !v_new) return KVMIX_ERR_NULL;
  const bool packed = cfg->k_bits != 16;
  st = check_cache(cfg, c, packed);
  if (st) return st;
  if (n_tokens < 0) return KVMIX_ERR_BAD_SHAPE;
  if (token_stride < kD || head_stride < 0 || batch_stride < 0) return KVMIX_ERR_ALIGN;
  if (packed && (!aligned16(k_new) || !aligned16(v_new) || token_stride % 8 || head_stride % 8 || batch_stride % 8)) return KVMIX_ERR_ALIGN;
  const bool ageing = packed && cfg->window >= 0;    // this call flushes; otherwise it only fills the ring
  if (ageing && c->v_lead != 0) return KVMIX_ERR_BAD_SHAPE;
  if (ageing && c->W_cap < cfg->window + kTile) return KVMIX_ERR_BAD_SHAPE;
  // dry run of the counters: nothing is launched unless everything fits
  {
    long long n_q = c->n_q, n_w = c->n_w;
    if (ring_tokens(c) >= c->W_cap && n_tokens > 0) return KVMIX_ERR_BAD_SHAPE;
    if (!ageing) {
      if ((long long)ring_tokens(c) + n_tokens > c->W_cap) return KVMIX_ERR_BAD_SHAPE;
    } else {
      if (n_w >= cfg->window + kTile && n_tokens > 0) return KVMIX_ERR_BAD_SHAPE;   // a flush is overdue: not a state this library leaves
      const long long flushes = (n_w + n_tokens) >= cfg->window + kTile ? (n_w + n_tokens - cfg->window) / kTile : 0;
      if (n_q + flushes * kTile > c->T_cap) return KVMIX_ERR_BAD_SHAPE;
    }
  }
  if (n_tokens == 0) return KVMIX_OK;
  const int units = sh->B * sh->Hkv, W = c->W_cap;
  // The old window tokens followed by the new ones form one sequence of m rows; its first 32 F rows leave for the
  // packed part (F tiles, from the ring or straight from the input: a token that is flushed within this call never
  // passes through the ring), the rest is the new window. The quantizer's launch over the F tiles also copies the
  // surviving new rows into their ring slots: those that land in the slot of an old row by the workgroup that reads this old row.
  // (A prompt of 32 700 tokens for 8 units: 42.0 us in two launches, 38.8 in one.)
  const long long m = (long long)c->n_w + n_tokens;
  const int F = ageing && m >= cfg->window + kTile ? (int)((m - cfg->window) / kTile) : 0;
  const long long first_kept = (long long)F * kTile;                       // first row of the sequence that stays in the window
  const int i0 = first_kept > c->n_w ? (int)(first_kept - c->n_w) : 0;      // first new token that stays
  const int n_copy = n_tokens - i0;                                         // at most W: what stays fits the ring
  const int copy_at = (int)((c->n_w + (long long)i0) % W);                  // where it goes, counted from slot w0
  if (F > 0) {
    QuantArgs a{};
    a.n_copy = n_copy; a.copy_row = i0; a.copy_at = copy_at;
    a.k_ring_w = c->k_win; a.v_ring_w = c->v_win;
    // slots [0, n_read) are read by tiles; the rows go to [copy_at, end) and, around the ring, [0, end - W)
    const int n_read = (int)(first_kept < c->n_w ? first_kept : c->n_w), end = copy_at + n_copy;
    a.n_read = copy_at < n_read || end > W ? n_read : 0;
    // slots outside [0, n_read): from copy_at on (or from n_read on, where the rows begin inside it or go around)
    int first = copy_at, last = end < W ? end : W;
    if (end - W > n_read || first < n_read) first = n_read;
    a.copy_tile0 = first / kTile;
    a.copy_tiles = n_copy > 0 && last > first ? (last + kTile - 1) / kTile - a.copy_tile0 : 0;
    a.k = k_new; a.v = v_new;
    a.tok = token_stride; a.unit_b = batch_stride; a.unit_h = head_stride;
    a.k_ring = c->k_win; a.v_ring = c->v_win; a.n_ring = c->n_w; a.ring_w0 = c->w0; a.W_cap = W;
    fill_quant_dst(a, c);
    a.tile0 = c->n_q / kTile;
    a.Hkv = sh->Hkv;
    const hipError_t e = launch_quantize_pack(a, cfg->k_bits, cfg->v_bits, F, units, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e);
  } else {
    AppendArgs ap{};
    ap.k_new = k_new; ap.v_new = v_new;
    ap.tok = token_stride; ap.head = head_stride; ap.batch = batch_stride;
    ap.k_win = c->k_win; ap.v_win = c->v_win;
    ap.W_cap = W; ap.slot = (c->w0 + copy_at) % W; ap.n = n_copy; ap.units = units; ap.Hkv = sh->Hkv;
    const hipError_t e = launch_append(ap, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e);
  }
  c->n_q += F * kTile;
  c->w0 = (int)((c->w0 + first_kept) % W);
  c->n_w = (int)(m - first_kept);
  return KVMIX_OK;
}

int kvmix_append(const kvmix_shape* sh, const kvmix_layer_cfg* cfg, const uint16_t* k_new, const uint16_t* v_new,
                 kvmix_layer_cache* c, void* stream) {
  if (!sh) return KVMIX_ERR_NULL;
  return kvmix_append_tokens(sh, cfg, k_new, v_new, kD, kD, (int64_t)sh->Hkv * kD, 1, c, stream);
}

}  // extern "C"

namespace {

// Everything an attention launch needs, filled by plan_attention after all host-side checks have passed.
// `mixed`: the fronts of Keys and Values differ.
struct AttnPlan { AttnArgs a; int kb, vb, G, block, units, waves; bool mixed; };

constexpr int kWindowTileCost = 3;   // packed tiles that take a wave as long as one window tile

size_t split_workspace_bytes(int units, int n_parts, int G) {
  return counters_bytes(units * (G > 8 ? G / 8 : 1)) + (size_t)units * n_parts * G * (kD + 2) * sizeof(float);
}

// How an attention call divides the n = n_q + n_w tokens of a cache whose Value front is n_q + v_lead:
// tiles [0, packed_tiles) have Keys and Values packed, tokens [32 packed_tiles, t_a) are the mixed range, tokens
// [t_a, n) are window tokens of both (t_a is a multiple of 32 unless it equals n).
struct Fronts { int packed_tiles; long long t_a; int n_w_eff, w0_eff; bool mixed; };
Fronts fronts_of(const kvmix_layer_cache* c, int n_w) {
  Fronts f;
  const long long n = (long long)c->n_q + n_w, n_qv = (long long)c->n_q + c->v_lead;
  if (c->v_lead == 0) {
    f.packed_tiles = c->n_q / kTile; f.t_a = c->n_q; f.n_w_eff = n_w; f.w0_eff = c->w0; f.mixed = false;
    return f;
  }
  const long long lo = n_qv < c->n_q ? n_qv : c->n_q, hi = n_qv < c->n_q ? c->n_q : n_qv;
  f.packed_tiles = (int)(lo / kTile);
  long long t_a = (hi + kTile - 1) / kTile * kTile;
  if (t_a > n) t_a = n;
  f.t_a = t_a;
  f.n_w_eff = (int)(n - t_a);
  f.w0_eff = f.n_w_eff > 0 ? slot_of(c, t_a) : 0;
  f.mixed = true;
  return f;
}

// Waves per workgroup of the attention kernel. 12 waves fill a compute unit with one workgroup, 8 leave room for two. Launches that
// need more workgroups than there are compute units run 8: twice the workgroups are resident, so that one's start and merge overlap
// another's stream (512 units of 128 tiles, 8 heads: 53.2 us against 54.1; 1 head, 600 units of 36: 23.3 against 25.9; 2048 of 20:
// 38.9 against 50.6). With at most one workgroup per compute unit the 4 more waves pay when each has many tiles to stream (1 head,
// 256 units of 128 tiles: 20.5 us against 23.2; 32 tiles: 10.3 against 10.6), and cost in start and merge when there are few (9
// tiles: 7.7 us against 7.5); from 16 to 24 tiles the two are within 2 % (16: 8.5 and 8.5). 8 heads with 3- or 4-bit Values do not
// fit the 128 registers of the 8-wave form (spilling: 93 us where 12 waves take 62; as half a block of 16: plan_attention).
int attn_waves(long long workgroups, int n_tiles, int n_splits, int block, int v_bits, int cus) {
  if (block > 8) return 8;
  if (block == 8 && (v_bits == 3 || v_bits == 4)) return 12;
  return workgroups > (cus > 0 ? cus : 256) || n_tiles <= 20 * n_splits ? 8 : 12;
}

// Groups of 16 heads and more run in blocks of 16 or of 8 heads. A block of 16 takes less work per head, a block of 8 has the
// shorter chain per tile and half the outputs to combine and to merge. Modelled times of a launch in us, for tiles of 2/2 bit;
// fixed parts and merging splits besides the tiles. Blocks of 16: workgroups that share a compute unit share its rate, and the
// second one starts late. A tile of 3/4 bit counts as 1.3 (8 x 48 heads over 8000 tokens: 16.3 us in blocks of 8, 14.3 in blocks of
// 16), a window tile as 2.4. Fitted to 1 x 72 heads over 8000 tokens (1, 4, 8, 16, 32 splits: 42.7, 15.9, 12.2, 11.0, 12.2 us in
// blocks of 16; 36.9, 14.8, 11.0, 9.6, 12.7 in blocks of 8), 16 x 48 over 4000 (2, 4, 5, 6, 8: 18.2, 13.6, 12.8, 16.0, 15.2; 16.7
// in blocks of 8, 2 splits), 32 x 48 over 2000 (1, 2, 4: 15.7, 13.3, 15.0; 15.4 in blocks of 8, unsplit), 64 x 16 over 1000 (2, 3,
// 4, 5: 10.7, 10.1, 9.5, 12.1; 10.3 in blocks of 8, 2 splits), 1 x 16 over 1000 (1, 4: 8.9, 7.9; 8.9, 7.3), 32 x 72 over 4000 (1 to
// 4: 29.5, 29.8, 24.0, 28.2).
double tile_work(int packed_tiles, int window_tiles, int k_bits, int v_bits) {
  return packed_tiles * (1.0 + 0.1 * (k_bits + v_bits - 4)) + 2.4 * window_tiles;
}
double cost_of_16(double sharing, double work, int s) {
  return s == 1 ? 5.0 + 0.16 * sharing * work : 7.6 + 2.2 * (sharing - 1.0) + 0.155 * sharing * work / s + 0.12 * s;
}
double cost_of_8(double work, int s) {      // one workgroup per compute unit
  return s == 1 ? 6.0 + 0.122 * work : 7.0 + 0.122 * work / s + 0.08 * s;
}
double sharing_of(int workgroups, int s, int cus) { return (double)(((long long)workgroups * s + cus - 1) / cus); }
// Split count of a launch in blocks of 16 heads, at least 6 tiles per split: the smallest modelled time, all tiles alike (weighted, 32 x 72
// heads over 2000 full-precision tokens got 3 splits and took 27.6 us instead of 26.7, measured before the merge became head-wise)
int wide_splits(int workgroups, int n_items, int s_max, int cus) {
  int best_s = 1;
  double best = 0.0;
  for (int s = 1; s == 1 || (s <= s_max && s * 6 <= n_items); s++) {
    const double c = cost_of_16(sharing_of(workgroups, s, cus), n_items, s);
    if (s == 1 || c < best) { best = c; best_s = s; }
  }
  return best_s;
}

// Validates an attention call against the cache state `c` (window count n_w) and fills the launch descriptor;
// launches nothing. With k_new / v_new the newest token of every unit is taken from there (ring slot new_slot,
// counted in n_w) and stored into the window by the kernel.
int plan_attention(const kvmix_shape* sh, const kvmix_layer_cfg* cfg, const uint16_t* q, const kvmix_layer_cache* c, int n_w,
                   const uint16_t* k_new, const uint16_t* v_new, int new_slot,
                   float softmax_scale, uint16_t* out, void* workspace, size_t workspace_bytes, int n_splits, AttnPlan* plan) {
  int st = check_shape_cfg(sh, cfg);
  if (st) return st;
  if (!q || !out) return KVMIX_ERR_NULL;
  if (!aligned16(q) || !aligned16(out)) return KVMIX_ERR_ALIGN;
  st = check_cache(cfg, c, false);
  if (st) return st;
  if (c->n_q + n_w < 1 || n_w < 0 || n_w > c->W_cap || (long long)n_w - (c->v_lead < 0 ? c->v_lead : 0) > c->W_cap) return KVMIX_ERR_BAD_SHAPE;
  const int units = sh->B * sh->Hkv, G = sh->Hq / sh->Hkv;
  const Fronts fr = fronts_of(c, n_w);
  // With the whole ring: the split count, and what a workspace is refused by, do not change as the window fills.
  const int n_items = c->W_cap / kTile + fr.packed_tiles;
  // What there is to do: the ring may be mostly empty.
  const int live_tiles = fr.packed_tiles + (fr.n_w_eff + kTile - 1) / kTile;
  if (n_splits < 0 || n_splits > max_splits(sh)) return KVMIX_ERR_BAD_SHAPE;
  const bool any_splits = n_splits == 0;
  const int cus = num_cus();
  if (any_splits) {
    // The launch is taken to run in rounds of `cus` workgroups. A round costs a fixed part (start, merge of the waves, partial and
    // arrival: about what 48 tiles take) plus the tiles of one split; take the split count with the smallest rounds x (48 + tiles
    // per split), at least 8 tiles each. (Twice as many workgroups of 8 waves fit the card; the count is also what a workspace is
    // refused or accepted by, and 128 units of 256 tiles take 24.4 us with 4 splits of 8 waves, 23.8 with 2 of 12.)
    if (cus == 0) return hip_fail(hipErrorInvalidDevice);
    const int ou = out_units(sh);
    int s_max = n_items / 8;
    if (s_max > max_splits(sh)) s_max = max_splits(sh);
    double best = 0.0, unsplit = 0.0;
    n_splits = 1;
    for (int s = 1; s <= s_max || s == 1; s++) {
      const double rounds = (double)(((long long)ou * s + cus - 1) / cus);
      const double cost = rounds * (48.0 + (double)n_items / s);
      if (s == 1) unsplit = cost;
      if (s == 1 || cost < best) { best = cost; n_splits = s; }
    }
    // an unsplit launch has no partials to write and merge, which the model leaves out: it wins a near tie
    // (288 workgroups of 8 heads over 4096 tokens: 51 us unsplit, 55 us with 2 splits, modelled 352 against 336)
    if (unsplit <= 1.06 * best) n_splits = 1;
  }
  if (n_splits > n_items) n_splits = n_items;
  // 4 heads: no more than the 32 splits whose partials one wave merges in two batches at most, until a split of the full count
  // would have 24 tiles less than one of 32, about where the two meet (32 and 64 splits, 1 unit, 2/2 bit: 16 000 tokens 8.6 and
  // 10.0 us, 40 000 11.2 and 11.6, 48 000 12.0 and 11.6, 64 000 13.8 and 12.0; 3/4 bit 40 000 12.3 and 12.3, 48 000 13.1 and 12.2;
  // 4 units, 2/2 bit: 40 000 11.6 and 12.6, 48 000 12.4 and 12.6, 64 000 14.2 and 13.1). A workspace is refused or accepted by the
  // full count all the same.
  const int n_counted = n_splits;
  if (any_splits && G == 4 && n_splits > 32 && (double)n_items * (1.0 / 32 - 1.0 / n_splits) < 24.0) n_splits = 32;
  // Two workgroups of 8 waves to a compute unit, at one pace, take a round's fixed part once (62 tiles' worth for the two) and
  // leave fewer compute units empty: a split launch that has one workgroup at most for each goes to a count that makes it more
  // than one but at most two, where that is modelled 8 % better (split launches cost another 12 tiles). Measured, old time over
  // new, at 2/2 bit with 1, 2, 4, 8 heads:
  //   2 -> 5 splits (86 to 102 units)  119 tiles 1.03-1.06 (8 heads 1.01), 253 tiles 1.02-1.10, 1.08-1.13, 1.14-1.15, 1.06-1.07
  //   3 -> 7 splits (65 to 73 units)   378 tiles 0.99-1.02, 1.03-1.06, 1.08-1.09, 1.03-1.04; 1003 tiles 0.98-1.03, 1.02-1.11, 1.17, 1.10-1.12
  //   4 -> 9 splits (52 to 56 units)   1003 tiles 0.97-1.03, 1.00-1.04, 1.10-1.12, 0.96-0.98
  // so from 2 splits with any of them and from 3 with 2 heads and more. The wider the codes, the nearer a launch is to what memory
  // gives either way: with 1 head up to 4 bits of Key and Value together (from 2 splits at 5 bits 0.99-1.18, at 6 0.98-1.09),
  // otherwise up to 5 (0.99-1.23; at 6 bits 0.94-1.17). Only with a workspace that holds these partials; it is refused or accepted
  // by the count above. 8 heads with 3- or 4-bit Values have 12 waves there.
  // An unsplit launch stays unsplit: it leaves the workspace alone, so that calls that overlap may hand over the same one, or
  // one that is not zero (129 to 170 units in 3 splits would take 3 to 13 % less: 160 units of 94 tiles, 4 heads, 16.7 and 14.9 us).
  bool paired = false;
  if (any_splits && (n_splits == 2 || (n_splits == 3 && G > 1)) && (long long)units * n_splits <= cus && !fr.mixed && G <= 8 &&
      cfg->k_bits + cfg->v_bits <= (G > 1 ? 5 : 4) && !(G == 8 && cfg->v_bits >= 3)) {
    const double as_is = 60.0 + (double)live_tiles / n_splits;
    int s = 2 * cus / units;
    if (s > max_splits(sh)) s = max_splits(sh);
    if (s > live_tiles / 8) s = live_tiles / 8;
    if (s > n_splits && (long long)units * s > cus && 62.0 + 2.0 * live_tiles / s < 0.92 * as_is &&
        workspace_bytes >= split_workspace_bytes(units, s, G)) {
      n_splits = s;
      paired = true;
    }
  }
  int block = G;
  if (G > 8 || (G == 8 && fr.mixed)) {
    // (With the fronts apart 8 heads are half a block of 16: a block of 16 takes a tile in about the time of a block of 8.)
    // Blocks of 8 heads where a launch of them has at most one workgroup per compute unit (see above: the faster ones at equal split
    // counts), blocks of 16 otherwise.
    block = !fr.mixed && cus > 0 && (long long)out_units(sh) * n_splits <= cus ? 8 : 16;
    if (any_splits) {
      // The count above is that of blocks of 8, and it is what a workspace is refused or accepted by. A workspace that also holds
      // the partials of the count that suits blocks of 16 gets those where they are modelled to be faster, or within 2 % (4 x 48
      // heads over 32 000 tokens, modelled alike: 22.8 us in blocks of 8, 20.8 in blocks of 16). At equal counts blocks of 8 it is
      // (64 x 16 heads over 300 tokens, unsplit: 7.8 us per launch, 8.6 in blocks of 16).
      const double work = tile_work(fr.packed_tiles, (fr.n_w_eff + kTile - 1) / kTile, cfg->k_bits, cfg->v_bits);
      const int wide = units * ((G + 15) / 16), n = wide_splits(wide, n_items, max_splits(sh), cus);
      auto fits = [&](int splits) {
        const int parts = splits + (fr.mixed ? 1 : 0);
        return parts == 1 || (workspace && aligned16(workspace) && workspace_bytes >= split_workspace_bytes(units, parts, G));
      };
      if (fits(n) && fits(n_splits) && (block == 16 || (n != n_splits && cost_of_16(sharing_of(wide, n, cus), work, n) < 1.02 * cost_of_8(work, n_splits)))) { n_splits = n; block = 16; }
    }
  }
  // 8 heads with 3- or 4-bit Values do not fit the 8-wave form of a block of 8 (attn_waves); as half a block of 16 they do. Where
  // there are more workgroups than compute units, two of 8 waves side by side then beat one of 12 after the other, by more the more
  // of a round stays empty. Times of 12 waves over those of 8, all four Key widths with 3- and 4-bit Values: 512 units of 300 tokens
  // 1.18-1.23, 1000 1.13-1.16, 2000 1.09-1.15, 4070 1.04-1.08 (3/4 bit 58.1 -> 54.6 us), 5000 1.04-1.07; 320 units x 4000 1.06-1.16;
  // 800 x 600 1.26-1.29; 1600 x 2000 1.10-1.13; 1040 x 3000 1.04-1.07; in splits, 136 units x 2000 in 2 and 3 1.13-1.15 and
  // 1.20-1.21, 384 x 4800 in 2 1.06-1.08. A tile takes a little longer that way: long contexts stay with 12 waves (2/4 bit, 512 x
  // 8000 tokens 101.4 in 12 waves, 103.5; 768 x 4000 83.0, 84.6).
  // Relative error against 64 bits (the rounding to fp16 alone is 2.07e-4), mean over these eight widths and 300 to 4000 tokens of
  // N(0,1): 2.0821e-4 in 12 waves, 2.0821e-4. Nearly uniform weights over 4000 tokens, whose outputs are small next to what they are
  // the sum of: 2.0756e-4 and 2.0772e-4 (both terms of an operand meet in one accumulator, as in every block of 16).
  const int tiles_each = (live_tiles + n_splits - 1) / n_splits;      // of a workgroup
  if (block == 8 && G == 8 && (cfg->v_bits == 3 || cfg->v_bits == 4)) {
    const long long workgroups = (long long)units * n_splits;
    if (cus > 0 && workgroups > cus && tiles_each <= (workgroups <= 2 * cus ? 160 : 96)) block = 16;
  }
  AttnArgs a{};
  // (With the fronts apart a workspace is refused or accepted as if the tokens between them had a partial of their own.)
  const int n_parts = (G <= 4 || paired ? n_counted : n_splits) + (fr.mixed ? 1 : 0);
  if (n_parts > 1) {
    if (!workspace) return KVMIX_ERR_NULL;
    if (!aligned16(workspace)) return KVMIX_ERR_ALIGN;
    if (workspace_bytes < split_workspace_bytes(units, n_parts, G)) return KVMIX_ERR_WORKSPACE;
    a.counters = reinterpret_cast<uint32_t*>(workspace);
    a.part = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) + counters_bytes(out_units(sh)));
  }
  // The counters' 256 bytes (at least) are shared out evenly: splits that arrive together then meet on fewer cache lines
  // (8 units x 32 splits, whose 256 arrivals queued up on one line for 1.3 us on average)
  a.counter_stride = 1;
  while (a.counter_stride * 2 * out_units(sh) <= 64) a.counter_stride *= 2;
  a.q = q; a.out = out; a.G = G;
  a.packed = c->packed;
  a.k_win = c->k_win; a.v_win = c->v_win;
  a.k_new = k_new; a.v_new = v_new; a.k_win_w = c->k_win; a.v_win_w = c->v_win; a.new_slot = new_slot;
  a.tiles_cap = c->T_cap / kTile; a.W_cap = c->W_cap; a.n_w = fr.n_w_eff;
  a.ring_tiles = c->W_cap / kTile; a.w0_tile = fr.w0_eff / kTile;
  a.n_splits = n_splits;
  int live = (fr.n_w_eff + kTile - 1) / kTile;
  if (fr.mixed) {
    a.m_first = fr.packed_tiles; a.m_tiles = (int)((fr.t_a + kTile - 1) / kTile) - fr.packed_tiles;
    a.m_end = (int)fr.t_a; a.m_front = c->n_q + c->v_lead; a.m_ahead = c->v_lead > 0;
    a.m_ring = slot_of(c, (long long)fr.packed_tiles * kTile) / kTile;
    live += !a.m_ahead ? a.m_tiles : a.m_front < a.m_end ? 1 : 0;
  }
  a.win_each = live / n_splits; a.win_extra = live % n_splits;
  a.win_tiles = kWindowTileCost < fr.packed_tiles / n_splits ? kWindowTileCost : fr.packed_tiles / n_splits;
  a.items_q = (fr.packed_tiles + a.win_extra * a.win_tiles) / n_splits;
  a.items_r = (fr.packed_tiles + a.win_extra * a.win_tiles) % n_splits;
  const float scale = softmax_scale > 0.0f ? softmax_scale : 1.0f / std::sqrt((float)kD);
  a.scale_log2 = scale * 1.4426950408889634f;
  plan->a = a;
  plan->kb = cfg->k_bits == 16 ? 2 : cfg->k_bits;
  plan->vb = cfg->v_bits == 16 ? 2 : cfg->v_bits;
  plan->G = G; plan->units = units;
  plan->block = block;
  plan->a.head_blocks = (G + block - 1) / block;
  // (with the fronts apart always 12: those kernels do not fit the registers of 8 waves)
  plan->waves = fr.mixed ? 12 : attn_waves((long long)out_units(sh) * n_splits, live + fr.packed_tiles, n_splits, plan->block, plan->vb, cus);
  plan->mixed = fr.mixed;
  // Workgroups of 8 waves that are all resident at once, two to a compute unit, keep pace with each other (8 heads, 512 units of
  // 4070 tokens: 2/2 bit 48.3 -> 45.6 us, 3/2 bit 57.8 -> 54.5; 320 units 43.1 -> 40.1; 4 heads 38.7 -> 37.2; 1 head, 320 units
  // 27.4 -> 26.5; 16 heads 49.7 -> 47.9). With more of them than that it is better that some end early and make room (768
  // workgroups of 128 tiles: 75.9 us as they come, 83.7 at one pace).
  const long long workgroups = (long long)units * n_splits * ((G + block - 1) / block);
  plan->a.even = plan->waves == 8 && workgroups > cus && workgroups <= 2 * cus;
  // with the append inside the launch the new token must be a window token of the main launch
  if (fr.mixed && new_slot >= 0 && fr.n_w_eff < 1) return KVMIX_ERR_BAD_SHAPE;
  return KVMIX_OK;
}

int launch_plan(const AttnPlan& p, void* stream) {
  const hipError_t e = p.mixed        ? launch_decode_attn<12, true>(p.a, p.kb, p.vb, p.block, p.units, (hipStream_t)stream)
                       : p.waves == 8 ? launch_decode_attn<8, false>(p.a, p.kb, p.vb, p.block, p.units, (hipStream_t)stream)
                                      : launch_decode_attn<12, false>(p.a, p.kb, p.vb, p.block, p.units, (hipStream_t)stream);
  return e == hipSuccess ? KVMIX_OK : hip_fail(e);
}

// ---- split workspace of kvmix_decode_attn_static: a fixed array in device memory, one copy per GPU. Its arrival counters have a
// place of their own, the same for every shape: calls of different shapes follow each other without the array being cleared, and a counter
// must never lie where another shape leaves partials. A split call has at least two partials of 520 bytes per head, so that what
// fits kScratchBytes has no more than this many counters (at most one per head).
constexpr size_t kScratchBytes = KVMIX_STATIC_SCRATCH_BYTES;
constexpr size_t kScratchCounterBytes = 16384;
static_assert(kScratchCounterBytes / sizeof(uint32_t) >= kScratchBytes / (2 * (kD + 2) * sizeof(float)), "counters of every shape that fits");
// Partials of groups of up to 4 heads are zero between calls, those of larger groups are left as they are: each kind has a place of
// its own.
static __device__ __align__(256) unsigned char scratch[kScratchCounterBytes + 2 * kScratchBytes];
// In host code the array's name is only a handle; its address on a device comes from hipGetSymbolAddress,
// asked once per device with that device current. Each GPU holds its own copy at its own address.
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

__global__ void clear_words_kernel(uint32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// Address of the current device's copy of `scratch`. The first call on a device also clears the arrival counters and the partials behind
// them on `stream`, ahead of the first launch that uses them; afterwards every attention launch leaves them zero again.
int scratch_address(void** ptr, hipStream_t stream) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e);
  if (dev < 0 || dev >= kMaxDevices) return hip_fail(hipErrorInvalidDevice);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e);
    if (!p) return hip_fail(hipErrorInvalidSymbol);
    constexpr int kWords = (int)((kScratchCounterBytes + kScratchBytes) / 4);
    clear_words_kernel<<<kWords / 256, 256, 0, stream>>>(reinterpret_cast<uint32_t*>(p), kWords);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e);
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return KVMIX_OK;
}

}  // namespace

extern "C" {

int kvmix_decode_attn(const kvmix_shape* sh, const kvmix_layer_cfg* cfg, const uint16_t* q, const kvmix_layer_cache* c,
                      float softmax_scale, uint16_t* out, void* workspace, size_t workspace_bytes, int n_splits, void* stream) {
  const int st0 = check_shape_cfg(sh, cfg);   // before the cache struct is looked at
  if (st0) return st0;
  if (!q || !out) return KVMIX_ERR_NULL;
  if (!aligned16(q) || !aligned16(out)) return KVMIX_ERR_ALIGN;
  if (!c) return KVMIX_ERR_NULL;
  AttnPlan plan;
  const int st = plan_attention(sh, cfg, q, c, c->n_w, nullptr, nullptr, -1, softmax_scale, out, workspace, workspace_bytes, n_splits, &plan);
  return st ? st : launch_plan(plan, stream);
}

int kvmix_decode_attn_static(const kvmix_shape* sh, const kvmix_layer_cfg* cfg, const uint16_t* q, const kvmix_layer_cache* c,
                             float softmax_scale, uint16_t* out, int n_splits, void* stream) {
  const int st0 = check_shape_cfg(sh, cfg);
  if (st0) return st0;
  if (!q || !out) return KVMIX_ERR_NULL;
  if (!aligned16(q) || !aligned16(out)) return KVMIX_ERR_ALIGN;
  if (!c) return KVMIX_ERR_NULL;
  AttnPlan plan;
  // First pass with a workspace of the array's size at a dummy aligned address: settles the split count and runs every check.
  int st = plan_attention(sh, cfg, q, c, c->n_w, nullptr, nullptr, -1, softmax_scale, out, reinterpret_cast<void*>(256), kScratchBytes, n_splits, &plan);
  if (st) return st;
  if (plan.a.n_splits > 1) {
    void* ptr = nullptr;
    st = scratch_address(&ptr, (hipStream_t)stream);
    if (st) return st;
    plan.a.counters = reinterpret_cast<uint32_t*>(ptr);
    plan.a.part = reinterpret_cast<float*>(reinterpret_cast<char*>(ptr) + kScratchCounterBytes + (plan.G <= 4 ? 0 : kScratchBytes));
  } else {
    plan.a.counters = nullptr; plan.a.part = nullptr;
  }
  return launch_plan(plan, stream);
}

int kvmix_decode_step(const kvmix_shape* sh, const kvmix_layer_cfg* cfg, const uint16_t* k_new, const uint16_t* v_new,
                      const uint16_t* q, kvmix_layer_cache* c, float softmax_scale, uint16_t* out,
                      void* workspace, size_t workspace_bytes, int n_splits, void* stream) {
  int st = check_shape_cfg(sh, cfg);
  if (st) return st;
  if (!k_new || !v_new || !c) return KVMIX_ERR_NULL;
  AttnPlan plan;
  const bool flush = cfg->k_bits != 16 && cfg->window >= 0 && c->n_w + 1 == cfg->window + kTile;
  if (cfg->k_bits != 16 && cfg->window >= 0 && c->v_lead != 0) return KVMIX_ERR_BAD_SHAPE;   // fixed-window ageing needs one front
  if (flush) {
    // The 32 oldest window tokens move to the packed part before the attention reads them. Every check is made
    // first, the attention's against the counters as the flush will leave them, so that a failing call launches
    // nothing and leaves the counters alone.
    st = check_cache(cfg, c, true);
    if (st) return st;
    if (c->n_q + kTile > c->T_cap || c->W_cap < cfg->window + kTile) return KVMIX_ERR_BAD_SHAPE;
    if (!aligned16(k_new) || !aligned16(v_new)) return KVMIX_ERR_ALIGN;
    kvmix_layer_cache after = *c;
    after.n_q += kTile; after.n_w = c->n_w + 1 - kTile; after.w0 = (c->w0 + kTile) % c->W_cap;
    if (cfg->window >= kTile) {
      // The new token is not among the 32 oldest: quantize-and-pack them straight from the ring (one launch), then
      // the attention launch with the append inside, as on every other step.
      const int slot = (c->w0 + c->n_w) % c->W_cap;
      st = plan_attention(sh, cfg, q, &after, after.n_w, k_new, v_new, slot, softmax_scale, out, workspace, workspace_bytes, n_splits, &plan);
      if (st) return st;
      const int W = c->W_cap;
      QuantArgs qa{};
      // (the tile's slots do not wrap: its rows are rows of an input with the ring's strides)
      qa.k = c->k_win + (size_t)c->w0 * kD; qa.v = c->v_win + (size_t)c->w0 * kD;
      qa.tok = kD; qa.unit_h = (int64_t)W * kD; qa.unit_b = qa.unit_h * sh->Hkv;
      qa.n_ring = 0; qa.W_cap = W;
      fill_quant_dst(qa, c);
      qa.tile0 = c->n_q / kTile;
      qa.Hkv = sh->Hkv;
      const hipError_t e = launch_quantize_pack(qa, cfg->k_bits, cfg->v_bits, 1, sh->B * sh->Hkv, (hipStream_t)stream);
      if (e != hipSuccess) return hip_fail(e);
      c->n_q = after.n_q; c->w0 = after.w0; c->n_w = after.n_w - 1;   // the flush is done; the append follows
      st = launch_plan(plan, stream);
      if (st) return st;
      c->n_w += 1;
      return KVMIX_OK;
    }
    // window length 0: the new token is itself among the 32 that are flushed; append, quantize-pack, attention
    st = plan_attention(sh, cfg, q, &after, after.n_w, nullptr, nullptr, -1, softmax_scale, out, workspace, workspace_bytes, n_splits, &plan);
    if (st) return st;
    st = kvmix_append(sh, cfg, k_new, v_new, c, stream);
    if (st) return st;
    return launch_plan(plan, stream);
  }
  st = check_cache(cfg, c, cfg->k_bits != 16);
  if (st) return st;
  if (ring_tokens(c) >= c->W_cap) return KVMIX_ERR_BAD_SHAPE;
  if (cfg->k_bits != 16 && c->W_cap < cfg->window + kTile) return KVMIX_ERR_BAD_SHAPE;
  if (!aligned16(k_new) || !aligned16(v_new)) return KVMIX_ERR_ALIGN;
  if (c->v_lead != 0 && fronts_of(c, c->n_w + 1).t_a > (long long)c->n_q + c->n_w) {
    // The new token shares its tile with the younger front: it belongs to the range between the fronts, whose ring rows the launch
    // reads from the ring. Plan against the counters as the append will leave them, append, then the attention launch.
    kvmix_layer_cache after = *c;
    after.n_w += 1;
    st = plan_attention(sh, cfg, q, &after, after.n_w, nullptr, nullptr, -1, softmax_scale, out, workspace, workspace_bytes, n_splits, &plan);
    if (st) return st;
    st = kvmix_append(sh, cfg, k_new, v_new, c, stream);
    if (st) return st;
    return launch_plan(plan, stream);
  }
  const int slot = (c->w0 + c->n_w) % c->W_cap;
  // the kernel's window count includes the new token: it is read from k_new / v_new in place of its ring row (and stored)
  st = plan_attention(sh, cfg, q, c, c->n_w + 1, k_new, v_new, slot, softmax_scale, out, workspace, workspace_bytes, n_splits, &plan);
  if (st) return st;
  st = launch_plan(plan, stream);
  if (st) return st;
  c->n_w += 1;
  return KVMIX_OK;
}

int kvmix_rpc_next(double r_k, double r_v, int current_k, int current_v, int* num_k, int* num_v) {
  if (!num_k || !num_v) return KVMIX_ERR_NULL;
  if (!(r_k >= 0.0 && r_k <= 1.0) || !(r_v >= 0.0 && r_v <= 1.0) || current_k < 0 || current_v < 0) return KVMIX_ERR_BAD_SHAPE;
  *num_k = (int)std::floor(r_k * (double)current_k);
  *num_v = (int)std::floor(r_v * (double)current_v);
  return KVMIX_OK;
}

int kvmix_flush(const kvmix_shape* sh, const kvmix_layer_cfg* cfg, kvmix_layer_cache* c, int keep_k, int keep_v, void* stream) {
  int st = check_shape_cfg(sh, cfg);
  if (st) return st;
  if (cfg->k_bits == 16) return KVMIX_ERR_BAD_BITS;
  st = check_cache(cfg, c, true);
  if (st) return st;
  if (keep_k < 0 || keep_v < 0) return KVMIX_ERR_BAD_SHAPE;
  const long long n = (long long)c->n_q + c->n_w, n_qv = (long long)c->n_q + c->v_lead;
  long long nk = n - keep_k, nv = n - keep_v;
  if (nk < 0) nk = 0;
  nk -= nk % kTile;
  if (nk < c->n_q) nk = c->n_q;
  if (nv < n_qv) nv = n_qv;
  if (nk > c->T_cap || nv > c->T_cap) return KVMIX_ERR_BAD_SHAPE;
  const bool k_moves = nk > c->n_q, v_moves = nv > n_qv;
  if (!k_moves && !v_moves) return KVMIX_OK;
  // one launch over the tiles that either side touches
  long long first = k_moves ? c->n_q / kTile : n_qv / kTile, last = k_moves ? nk / kTile : (nv + kTile - 1) / kTile;
  if (v_moves) {
    if (n_qv / kTile < first) first = n_qv / kTile;
    if ((nv + kTile - 1) / kTile > last) last = (nv + kTile - 1) / kTile;
  }
  QuantArgs a{};
  a.k = c->k_win; a.v = c->v_win; a.W_cap = c->W_cap;
  a.tok = kD; a.unit_h = (int64_t)c->W_cap * kD; a.unit_b = a.unit_h * sh->Hkv;
  a.ring_w0 = slot_of(c, first * kTile);
  fill_quant_dst(a, c);
  a.tile0 = (int)first;
  a.Hkv = sh->Hkv;
  a.k_tile_a = c->n_q / kTile; a.k_tile_b = (int)(nk / kTile);
  a.v_tok_a = (int)n_qv; a.v_tok_b = (int)nv;
  const hipError_t e = launch_quantize_fronts(a, cfg->k_bits, cfg->v_bits, (int)(last - first), sh->B * sh->Hkv, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(e);
  c->w0 = slot_of(c, nk);
  c->n_q = (int)nk;
  c->n_w = (int)(n - nk);
  c->v_lead = (int)(nv - nk);
  return KVMIX_OK;
}

int kvmix_stream_read(const void* buf, size_t bytes, int workgroups, int threads, void* sink, void* stream) {
  if (!buf) return KVMIX_ERR_NULL;
  if (!aligned16(buf)) return KVMIX_ERR_ALIGN;
  if (workgroups < 1 || workgroups > 65535 || threads < 64 || threads > 768 || threads % 64) return KVMIX_ERR_BAD_SHAPE;
  const hipError_t e = launch_stream_read(buf, bytes, workgroups, threads, reinterpret_cast<uint32_t*>(sink), (hipStream_t)stream);
  return e == hipSuccess ? KVMIX_OK : hip_fail(e);
}

int kvmix_dequant(const kvmix_shape* sh, const kvmix_layer_cfg* cfg, const kvmix_layer_cache* c, int which, float* out, void* stream) {
  int st = check_shape_cfg(sh, cfg);
  if (st) return st;
  if (cfg->k_bits == 16) return KVMIX_ERR_BAD_BITS;
  if (!out) return KVMIX_ERR_NULL;
  if (which != 0 && which != 1) return KVMIX_ERR_BAD_SHAPE;
  st = check_cache(cfg, c, true);
  if (st) return st;
  DequantArgs a{};
  a.packed = c->packed;
  a.out = out; a.tiles_cap = c->T_cap / kTile; a.n_tokens = c->n_q + (which ? c->v_lead : 0);
  a.k_bits = cfg->k_bits; a.v_bits = cfg->v_bits; a.which = which;
  const hipError_t e = launch_dequant(a, sh->B * sh->Hkv, (hipStream_t)stream);
  return e == hipSuccess ? KVMIX_OK : hip_fail(e);
}

}  // extern "C"
