"""The token kernels' scratch memory, from the metadata of the built library.
The runtime allocates it behind the caller's workspace, a stack for every lane
that a queue may run, so the kernels keep (nearly) everything in registers:
none in the held-out kernels, at most 64 bytes a lane in fold-in's and 96 in the
z-step's.  The long lists' variants at 4 waves a SIMD (128 registers), taken where
that measured faster, may have up to 288."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1704_03581_amd", "libpulda.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _kernels(tmp_path):
    """{mangled kernel name: scratch bytes a lane} of the library's gfx950 code."""
    data = open(LIB, "rb").read()
    out = {}
    for n, m in enumerate(re.finditer(MAGIC, data)):
        at = m.start() + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" not in name or size == 0:
                continue
            path = tmp_path / f"code{n}.o"
            path.write_bytes(data[m.start() + off:m.start() + off + size])
            text = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for k in re.finditer(r"\.name:\s+(_Z\S+)(.*?)\.private_segment_fixed_size:\s+(\d+)", text, re.S):
                out[k.group(1)] = int(k.group(3))
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_token_kernels_scratch(tmp_path):
    kernels = _kernels(tmp_path)
    limits = [("ltr_kernel", 0), ("foldin_step_kernel", 64), ("z_step_kernel", 96), ("z_lane_kernel", 0)]
    seen = dict.fromkeys([k for k, _ in limits], 0)
    for name, size in kernels.items():
        for part, limit in limits:
            if part in name:
                seen[part] += 1
                four = re.search(r"ILi64E.*Li4E|ltr_kernelILi32ELi4E", name) is not None
                assert size <= (288 if four else limit), (name, size)
    assert all(seen.values()), seen
