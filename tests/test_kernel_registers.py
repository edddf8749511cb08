"""The built library: no attention kernel keeps registers in scratch memory (read from the kernel descriptors' metadata, no GPU needed)."""
import os
import re
import struct
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2506_08018_amd", "libkvmix.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def device_code_objects(blob):
    """The gfx950 code objects of every offload bundle linked into the library."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + name_len]
            p += 24 + name_len
            if b"gfx950" in name and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(magic, p)


def test_no_kernel_spills(tmp_path):
    """A launch with scratch memory costs 2 to 3 us more, whatever it keeps there; the kernels for tiles between two fronts and 4 heads once did."""
    n = {}
    for i, code in enumerate(device_code_objects(open(LIB, "rb").read())):
        path = tmp_path / f"{i}.co"
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in notes.split(".agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
            spilled = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
            scratch = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", kernel).group(1))
            n[name] = (spilled, scratch)
    assert sum("decode_attn_kernel" in k for k in n) > 100 and sum("quantize_pack_kernel" in k for k in n) >= 16, len(n)
    assert {k: v for k, v in n.items() if v != (0, 0)} == {}
