"""What the kernels of the built library ask for, from the metadata of its code objects."""
import re
import struct
import subprocess

import pytest

from paper_2602_11562_amd import binding

READELF = "/opt/rocm/lib/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """{kernel's mangled name: bytes of scratch a lane}"""
    data, path, out = open(binding.LIB_PATH, "rb").read(), tmp_path_factory.mktemp("objects") / "code.o", {}
    for start in (m.start() for m in re.finditer(re.escape(BUNDLE), data)):      # one bundle a source
        at = start + len(BUNDLE) + 8
        for _ in range(struct.unpack_from("<Q", data, at - 8)[0]):
            offset, size, name = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + name]
            at += 24 + name
            if not size or b"gfx950" not in triple:
                continue
            path.write_bytes(data[start + offset:start + offset + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            names = re.findall(r"^    \.name:\s+(\S+)", notes, re.M)
            sizes = re.findall(r"^    \.private_segment_fixed_size:\s+(\d+)", notes, re.M)
            assert len(names) == len(sizes)
            out.update(zip(names, map(int, sizes)))
    return out


def test_tiled_gsta_spills_nowhere(scratch):
    kernels = {k: n for k, n in scratch.items() if "gsta_tiled_kernel" in k}
    assert len(kernels) > 50
    assert not {k for k, n in kernels.items() if n}
