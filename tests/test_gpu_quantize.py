"""GPU parity: kvmix_quantize_pack / kvmix_dequant vs the oracle, bit-exact on codes, scales and zero-points."""
import numpy as np
import pytest

import kvmix_synth as synth
from gpu_common import assert_cache_equal, bits_of, make_pair, u16

pytestmark = pytest.mark.gpu

COMBOS = [(kb, vb) for kb in (1, 2, 3, 4) for vb in (1, 2, 3, 4)]      # every pair the launch tables instantiate


@pytest.mark.parametrize("kb,vb", COMBOS)
def test_quantize_pack_bit_exact(kb, vb):
    print(f"case quantize_pack kb={kb} vb={vb}", flush=True)
    q, k, v, rc, gc, shape, cfg = make_pair(2, 4, 2, 32 * 7 + 32, 32, kb, vb, seed=100 + kb * 10 + vb)
    assert gc.n_q == rc.n_q == 32 * 7
    assert_cache_equal(rc, gc)


def adversarial_kv(seed, B, Hkv, T):
    """Groups the quantizer has to get exactly right: constant, two-valued, full fp16 range, subnormal,
    signed zeros, exact ties."""
    rng = np.random.default_rng(seed)
    k = rng.standard_normal((B, Hkv, T, 128)).astype(np.float32)
    v = rng.standard_normal((B, Hkv, T, 128)).astype(np.float32)
    for a in (k, v):
        a[:, :, 0:32, 0:32] = 1.25                                   # constant (both axes)
        a[:, :, 32:64, :] = np.where(rng.random((B, Hkv, 32, 128)) < 0.5, -3.0, 5.0)
        a[:, :, 64:96, 0:64] = rng.choice([-65504.0, 65504.0, 0.0, 1.0], (B, Hkv, 32, 64))
        a[:, :, 64:96, 64:128] = rng.uniform(-6e-5, 6e-5, (B, Hkv, 32, 64))   # fp16 subnormals
        a[:, :, 96:128, :] = rng.integers(0, 16, (B, Hkv, 32, 128)) * 0.5      # many exact ties
        a[:, :, 128:160, :] = np.where(rng.random((B, Hkv, 32, 128)) < 0.5, -0.0, 0.0)
        a[:, :, 128:160, ::7] = 2.0 ** -20
        a[:, :, 160:192, :] *= 1000.0
    return k.astype(np.float16), v.astype(np.float16)


@pytest.mark.parametrize("kb,vb", [(2, 2), (3, 3), (4, 4), (1, 1), (1, 4), (3, 1)])   # 1 bit: ranges beyond fp16 store the largest fp16 step
def test_quantize_pack_adversarial_groups(kb, vb):
    print(f"case adversarial kb={kb} vb={vb}", flush=True)
    B, Hkv, T = 1, 2, 256
    k, v = adversarial_kv(7, B, Hkv, T)
    q = np.zeros((B, Hkv, 128), np.float16)
    _, _, _, rc, gc, shape, cfg = make_pair(B, Hkv, Hkv, T + 32, 32, kb, vb, q_k_v=(q, np.concatenate([k, k[:, :, :32]], 2), np.concatenate([v, v[:, :, :32]], 2)))
    assert_cache_equal(rc, gc)


@pytest.mark.parametrize("kb,vb,units,tiles", [
    (2, 2, 128, 64), (2, 2, 128, 65),       # 8192 tiles, the most for four waves to a tile, and one tile per unit more
    (4, 1, 128, 64), (1, 4, 128, 65), (4, 4, 128, 65), (1, 1, 128, 65),
    (3, 4, 64, 64), (3, 4, 64, 65),         # 3-bit groups: 4096
    (4, 3, 64, 64), (2, 3, 64, 65), (3, 3, 64, 65), (1, 3, 64, 64),
    (2, 4, 64, 31), (2, 4, 64, 32),         # around 2048 tiles: records past the caches from there on
])
def test_quantize_pack_wave_forms(kb, vb, units, tiles):
    print(f"case wave forms kb={kb} vb={vb} units={units} tiles={tiles}", flush=True)
    B, Hkv, T = units // 8, 8, 32 * tiles
    k, v = adversarial_kv(17, 1, Hkv, T)
    k, v = (np.concatenate([np.roll(a, 32 * b, axis=2) for b in range(B)]) for a in (k, v))
    q = np.zeros((B, Hkv, 128), np.float16)
    window = lambda a: np.concatenate([a, a[:, :, :32]], 2)
    _, _, _, rc, gc, shape, cfg = make_pair(B, Hkv, Hkv, T + 32, 32, kb, vb, q_k_v=(q, window(k), window(v)))
    assert gc.n_q == T
    assert_cache_equal(rc, gc)


def near_tie_groups(rng, n_groups, q_max):
    """Groups of 32 fp16 values [mn, mx, x ...] whose quotients (x - mn) / s (s = the group's stored step) lie within
    a few 10^-6 relative of k + 1/2 without being ties: inside and just outside the band in which a kernel that
    brackets the quotient has to fall back on the division. A minimum of small magnitude next to a range of order
    one gives x - mn a fine grid, so such quotients exist (about one per group among all fp16 x).
    (Inputs only: the expected codes come from the oracle.) Returns the groups and the number of near-tie elements."""
    out = np.zeros((n_groups, 32), np.float16)
    pos = np.arange(1, 0x7C00, dtype=np.uint16).view(np.float16)              # every positive finite fp16 number
    n_near = 0
    for g in range(n_groups):
        mn = np.float16(rng.uniform(-1.0, 1.0) * 2.0 ** rng.integers(-12, -6))
        mx = np.float16(rng.uniform(0.25, 16.0))
        rng32 = np.float32(mx) - np.float32(mn)
        s = np.float64(np.float16(rng32 / np.float32(q_max)))
        x = pos[pos < mx]
        d32 = (x.astype(np.float32) - np.float32(mn)).astype(np.float64)
        t = d32 / s
        d = np.abs(t - np.floor(t) - 0.5)
        near = x[(d > 0) & (d < 8e-6 * np.maximum(t, 1.0)) & (t < q_max + 0.4)]
        pick = rng.permutation(near)[:30]
        n_near += len(pick)
        fill = rng.choice(x, 30 - len(pick)) if len(pick) < 30 else np.zeros(0, np.float16)
        out[g] = np.concatenate([[mn, mx], pick, fill]).astype(np.float16)
    return out, n_near


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_quantize_pack_near_tie_quotients(bits):
    print(f"case near-tie quotients bits={bits}", flush=True)
    B, Hkv, T = 1, 2, 128
    rng = np.random.default_rng(40 + bits)
    q_max = (1 << bits) - 1
    vg, n_v = near_tie_groups(rng, B * Hkv * T * 4, q_max)
    vg = vg.reshape(B, Hkv, T, 4, 32)
    v = vg.reshape(B, Hkv, T, 128)                                           # Values: a group is 32 channels of a token
    kg, n_k = near_tie_groups(rng, B * Hkv * (T // 32) * 128, q_max)
    kg = kg.reshape(B, Hkv, T // 32, 128, 32)
    assert n_v > 50 and n_k > 50, (n_v, n_k)      # the inputs do hold such quotients
    k = np.ascontiguousarray(kg.transpose(0, 1, 2, 4, 3)).reshape(B, Hkv, T, 128)   # Keys: 32 tokens of a channel
    q = np.zeros((B, Hkv, 128), np.float16)
    pad_k, pad_v = k[:, :, :32], v[:, :, :32]                                 # the window tokens make_pair leaves unpacked
    _, _, _, rc, gc, shape, cfg = make_pair(B, Hkv, Hkv, T + 32, 32, bits, bits,
                                            q_k_v=(q, np.concatenate([k, pad_k], 2), np.concatenate([v, pad_v], 2)))
    assert gc.n_q == rc.n_q == T
    assert_cache_equal(rc, gc)


@pytest.mark.parametrize("kb,vb", [(3, 3), (2, 3), (3, 4), (1, 2)])
def test_quantize_pack_ties(kb, vb):
    """Groups full of exact ties at the plain step and, in elements 10 and 21, at the step of the 2-bit elements of a 3-bit group (itself
    rounded to fp32 unless the scale is a multiple of 3), their neighbours one fp16 number away, and tiny ranges with a subnormal
    scale: codes that the bracket leaves open, bit for bit as the oracle has them."""
    print(f"case ties kb={kb} vb={vb}", flush=True)
    B, Hkv, T = 1, 2, 160
    rng = np.random.default_rng(70 + 10 * kb + vb)

    def groups(n, bits):
        q_max = (1 << bits) - 1
        out = np.zeros((n, 32), np.float16)
        for g in range(n):
            s = np.float16(rng.choice([3 * 2.0 ** -6, 2.0 ** -4, rng.uniform(0.01, 2.0), 2.0 ** -20]))
            step = np.full(32, float(s))
            if bits == 3:
                step[[10, 21]] = np.float32(np.float32(s) * np.float32(7)) / np.float32(3)
            top = np.full(32, q_max)
            if bits == 3:
                top[[10, 21]] = 3
            x = (rng.integers(0, top) + 0.5) * step
            x = x.astype(np.float16)
            x = np.where(rng.random(32) < 0.25, np.nextafter(x, np.float16(rng.choice([-1, 9]))), x).astype(np.float16)
            ends = [e for e in rng.permutation(32) if e not in (10, 21)][:2]
            x[ends[0]], x[ends[1]] = 0, np.float16(float(s) * q_max)
            out[g] = np.clip(x, 0, x[ends[1]])
        return out

    v = groups(B * Hkv * T * 4, vb).reshape(B, Hkv, T, 128)
    kg = groups(B * Hkv * (T // 32) * 128, kb).reshape(B, Hkv, T // 32, 128, 32)
    k = np.ascontiguousarray(kg.transpose(0, 1, 2, 4, 3)).reshape(B, Hkv, T, 128)
    q = np.zeros((B, Hkv, 128), np.float16)
    _, _, _, rc, gc, shape, cfg = make_pair(B, Hkv, Hkv, T + 32, 32, kb, vb,
                                            q_k_v=(q, np.concatenate([k, k[:, :, :32]], 2), np.concatenate([v, v[:, :, :32]], 2)))
    assert gc.n_q == rc.n_q == T
    assert_cache_equal(rc, gc)


def test_quantize_pack_offsets_and_strides():
    """Writing at a token offset into a larger cache, from a strided (sliced) source."""
    import torch
    import paper_2506_08018_amd as kv
    from oracle.kvmix_ref import RefCache
    B, Hkv, T = 2, 2, 192
    q, k, v = synth.gen_layer_numpy(5, 0, B, Hkv, Hkv, T)
    rc = RefCache(B, Hkv, Hkv, 3, 4, 32, 256, 64)
    shape, cfg = kv.Shape(B, Hkv, Hkv), kv.LayerCfg(3, 4, 32)
    gc = kv.LayerCache(shape, cfg, 256, 64)
    kt, vt = torch.from_numpy(k).cuda(), torch.from_numpy(v).cuda()
    for (a, b_) in ((0, 64), (64, 160), (160, 192)):
        print(f"case offsets chunk {a}:{b_}", flush=True)
        assert rc.quantize_pack(u16(k[:, :, a:b_]), u16(v[:, :, a:b_])) == 0
        kv.quantize_pack(shape, cfg, kt[:, :, a:b_], vt[:, :, a:b_], gc)   # non-contiguous views: strides passed through
    torch.cuda.synchronize()
    assert gc.n_q == rc.n_q == 192
    assert_cache_equal(rc, gc)


@pytest.mark.parametrize("kb,vb", [(2, 4), (3, 2), (4, 3)])
def test_dequant_matches_oracle(kb, vb):
    import torch
    import paper_2506_08018_amd as kv
    print(f"case dequant kb={kb} vb={vb}", flush=True)
    q, k, v, rc, gc, shape, cfg = make_pair(1, 2, 2, 160, 32, kb, vb, seed=9)
    for which in (0, 1):
        out = torch.zeros((shape.units, gc.n_q, 128), dtype=torch.float32, device="cuda")
        kv.dequant(shape, cfg, gc, which, out)
        got = out.cpu().numpy().astype(np.float64)
        want = rc.dequant(which)
        assert np.all(np.abs(got - want) <= 2.0 ** -22 * (np.abs(want) + np.abs(got) + 1e-30) + 2.0 ** -22 * 70.0)


def test_error_returns_launch_nothing():
    import torch
    import paper_2506_08018_amd as kv
    shape, cfg = kv.Shape(1, 2, 2), kv.LayerCfg(2, 2, 32)
    gc = kv.LayerCache(shape, cfg, 64, 64)
    k = torch.zeros((1, 2, 48, 128), dtype=torch.float16, device="cuda")
    with pytest.raises(kv.KVMixError) as e:
        kv.quantize_pack(shape, cfg, k, k, gc)
    assert e.value.status == -4
    k = torch.zeros((1, 2, 96, 128), dtype=torch.float16, device="cuda")
    with pytest.raises(kv.KVMixError) as e:
        kv.quantize_pack(shape, cfg, k, k, gc)
    assert e.value.status == -4
    with pytest.raises(kv.KVMixError) as e:
        kv.quantize_pack(shape, kv.LayerCfg(5, 2, 32), k[:, :, :32], k[:, :, :32], gc)
    assert e.value.status == -2
    with pytest.raises(kv.KVMixError) as e:
        kv.quantize_pack(kv.Shape(1, 2, 2, 64, 32), cfg, k[:, :, :32], k[:, :, :32], gc)
    assert e.value.status == -4
    with pytest.raises(kv.KVMixError) as e:
        kv.quantize_pack(kv.Shape(1, 2, 2, 128, 64), cfg, k[:, :, :32], k[:, :, :32], gc)
    assert e.value.status == -3
    assert gc.n_q == 0 and not bits_of(gc.packed, np.uint32).any()
