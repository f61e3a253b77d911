"""Registers and LDS of the built kernels, from the code object's own notes:
what the launch rules count on for workgroups sharing a compute unit."""
import re
import struct
import subprocess

import pytest
import yaml

from paper_2609_15030_amd.build import LIB

CU_LDS, SIMD_VGPRS, SIMDS = 160 * 1024, 512, 4


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled name without arguments: metadata} of the gfx950 code object
    inside the built library."""
    blob = open(LIB, "rb").read()
    at = blob.index(b"__CLANG_OFFLOAD_BUNDLE__")
    n, = struct.unpack_from("<Q", blob, at + 24)
    pos, code = at + 32, None
    for _ in range(n):
        off, size, tlen = struct.unpack_from("<QQQ", blob, pos)
        if b"gfx950" in blob[pos + 24:pos + 24 + tlen]:
            code = blob[at + off:at + off + size]
        pos += 24 + tlen
    path = tmp_path_factory.mktemp("co") / "gfx950.co"
    path.write_bytes(code)
    notes = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", str(path)], check=True,
                           capture_output=True, text=True).stdout
    meta = yaml.safe_load(notes[notes.index("---"):notes.index("...")])["amdhsa.kernels"]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in meta), check=True, capture_output=True,
                           text=True).stdout.split("\n")
    short = lambda s: re.sub(r"^(void )?la::", "", s.split("(")[0])
    return {short(s): k for s, k in zip(names, meta)}


def workgroups_per_cu(k):
    waves = k[".max_flat_workgroup_size"] // 64
    lds = k[".group_segment_fixed_size"]
    by_regs = SIMDS * (SIMD_VGPRS // (-(-k[".vgpr_count"] // 8) * 8)) // waves
    return min(by_regs, CU_LDS // lds if lds else by_regs)


@pytest.mark.parametrize("dk,dv,least", [(128, 128, 2), (128, 64, 2), (64, 128, 3), (64, 64, 3)])
def test_narrow_segment_maps_share_a_cu(kernels, dk, dv, least):
    """A 64-column map workgroup has two scan waves for a CU's four SIMDs: with
    one workgroup per CU half of the SIMDs would run none."""
    assert workgroups_per_cu(kernels[f"gdr_xscan_kernel<{dk}, {dv}, 2, 64>"]) >= least
