"""LDS of the projections around a separate GSTA pass: what the built kernels declare against what their layout reaches."""
import os
import re
import subprocess

import pytest

from paper_2602_11562_amd import build


@pytest.fixture(scope="module")
def declared(tmp_path_factory):
    """{kernel's mangled name: bytes of LDS}, from the device assembly of the source as the library is built."""
    out = str(tmp_path_factory.mktemp("project") / "gsta_project.s")
    r = subprocess.run([build._hipcc(), *build.HIPCC_FLAGS, "--offload-device-only", "-S", "-o", out,
                        os.path.join(build.CSRC, "gsta_project.hip")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = open(out).read()
    return {m[1]: int(m[2]) for m in
            re.finditer(r"\.amdhsa_kernel (\S+)\n\s*\.amdhsa_group_segment_fixed_size (\d+)", text)}


def _parts(d, n):
    """Bytes up to the last place of the first n bf16 parts of 16 pairs' vectors: rows unpadded at d = 128; at d = 64 of pitch
    d + 8, the second and third part 16 and 32 rows and another 64 and 160 values behind the first."""
    if d == 128:
        return 2 * 16 * d * n
    return 2 * ((n - 1) * 16 * (d + 8) + (0, 64, 160)[n - 1] + 15 * (d + 8) + d)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kernel", ["gsta_r_kernel", "gsta_out_kernel"])
def test_declared_lds_holds_every_place(declared, kernel, d):
    lds, = [n for name, n in declared.items() if f"{kernel}ILi{d}E" in name]
    patches = d // 16 * 32 * d                             # a wave's 16 columns of a matrix
    need = patches + (_parts(d, 1) + _parts(d, 3) if kernel == "gsta_r_kernel" else 2 * _parts(d, 3))
    assert lds >= need
