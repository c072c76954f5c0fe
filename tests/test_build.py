"""What the compiler made of the kernels, from the metadata in the built library (host only)."""
import os
import re
import struct
import subprocess

import paper_2406_15486_amd as sa

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


def _kernels(path, tmp):
    """Metadata of every kernel in the library's gfx950 code objects, by mangled name."""
    data = open(path, "rb").read()
    found = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.start()
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            offset, size, n = struct.unpack_from("<QQQ", data, p)
            target, p = data[p + 24:p + 24 + n], p + 24 + n
            if b"gfx950" not in target or size == 0:
                continue
            obj = tmp / f"{len(found)}.co"
            obj.write_bytes(data[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
            fields = {}
            for key, value in re.findall(r"^\s*(?:- )?\.(\w+):\s+(\S+)$", notes, re.M):
                fields[key] = value
                if key == "wavefront_size":          # the last field of a kernel
                    found[fields["symbol"]], fields = fields, {}
    return found


def test_no_kernel_spills(tmp_path):
    """No scratch, no spilled vector register, no scalar register kept in a vector lane: the attention kernels use up to
    252 registers and lose several times what a spill looks like it costs, in the middle of their loops."""
    kernels = _kernels(sa.lib_path(), tmp_path)
    assert sum("flash_kernel" in name for name in kernels) >= 10 and any("select_kernel" in name for name in kernels)
    for name, k in kernels.items():
        assert (k["private_segment_fixed_size"], k["vgpr_spill_count"], k["sgpr_spill_count"]) == ("0", "0", "0"), (name, k)
        assert int(k["vgpr_count"]) <= (128 if "12flash_kernelILi1E" in name else 256), (name, k["vgpr_count"])
