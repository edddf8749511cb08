// The host side of the attention calls without a GPU: kvmix_decode_attn with the launches taken down instead of made, on a device of
// 256 compute units. One call per input line (B Hkv G k_bits v_bits n_q n_w W_cap v_lead workspace n_splits; workspace in bytes,
// -1: kvmix_workspace_bytes, 0: none), one line out: status, splits, waves, heads per block, workgroups keep pace, workspace used.
#include "../paper_2506_08018_amd/csrc/kvmix_api.hip"
#include <cstdio>

namespace {
AttnArgs seen;
int seen_waves, seen_block;
}  // namespace

namespace kvmix {
hipError_t launch_quantize_pack(QuantArgs, int, int, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_quantize_fronts(const QuantArgs&, int, int, int, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_append(const AppendArgs&, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_dequant(const DequantArgs&, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_stream_read(const void*, size_t, int, int, uint32_t*, hipStream_t) { return hipErrorUnknown; }
hipError_t note(const AttnArgs& a, int waves, int block) { seen = a; seen_waves = waves; seen_block = block; return hipSuccess; }
template <> hipError_t launch_decode_attn<8, false>(const AttnArgs& a, int, int, int block, int, hipStream_t) { return note(a, 8, block); }
template <> hipError_t launch_decode_attn<12, false>(const AttnArgs& a, int, int, int block, int, hipStream_t) { return note(a, 12, block); }
template <> hipError_t launch_decode_attn<12, true>(const AttnArgs& a, int, int, int block, int, hipStream_t) { return note(a, 12, block); }
}  // namespace kvmix

extern "C" hipError_t hipGetDevice(int* device) { *device = 0; return hipSuccess; }
extern "C" hipError_t hipDeviceGetAttribute(int* value, hipDeviceAttribute_t, int) { *value = 256; return hipSuccess; }

int main() {
  int B, Hkv, G, kb, vb, n_q, n_w, W, lead, splits;
  long ws;
  while (scanf("%d %d %d %d %d %d %d %d %d %ld %d", &B, &Hkv, &G, &kb, &vb, &n_q, &n_w, &W, &lead, &ws, &splits) == 11) {
    const kvmix_shape sh{B, Hkv * G, Hkv, kD, kTile};
    const kvmix_layer_cfg cfg{kb, vb, -1};
    uint16_t* p = reinterpret_cast<uint16_t*>(4096);      // never followed
    const kvmix_layer_cache c{reinterpret_cast<uint32_t*>(p), p, p, n_q + W, W, n_q, n_w, 0, lead};
    size_t bytes = 0;
    kvmix_workspace_bytes(&sh, n_q + W, &bytes);
    if (ws >= 0) bytes = (size_t)ws;
    const int st = kvmix_decode_attn(&sh, &cfg, p, &c, 0.0f, p, ws == 0 ? nullptr : p, bytes, splits, nullptr);
    if (st) printf("%d 0 0 0 0 0\n", st);
    else printf("0 %d %d %d %d %d\n", seen.n_splits, seen_waves, seen_block, (int)seen.even, (int)(seen.n_splits > 1 && seen.counters != nullptr));
  }
}
