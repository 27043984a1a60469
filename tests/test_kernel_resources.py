"""Registers of the compiled kernels, from the code objects' own metadata: no
kernel keeps values in scratch memory or in lanes of other registers. A kernel
that outgrows its registers still gives right results, only slower, so nothing
else here would notice.
"""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2608_29291_amd", "libce_router.so")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
AMDGPU = 224  # e_machine


def code_objects(data):
    """The gfx950 ELF images inside the library's offload bundles."""
    at = 0
    while (at := data.find(b"\x7fELF", at + 1)) > 0:
        if struct.unpack_from("<H", data, at + 18)[0] == AMDGPU:
            shoff, = struct.unpack_from("<Q", data, at + 40)
            size, n = struct.unpack_from("<HH", data, at + 58)
            yield data[at:at + shoff + size * n]


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(LIB) or not os.path.exists(READELF):
        pytest.skip("library or llvm-readelf missing")
    d = tmp_path_factory.mktemp("co")
    out = {}
    for i, co in enumerate(code_objects(open(LIB, "rb").read())):
        p = d / f"{i}.co"
        p.write_bytes(co)
        r = subprocess.run([READELF, "--notes", str(p)], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        for k in r.stdout.split("\n  - .agpr_count:")[1:]:
            f = dict(re.findall(r"^\s+\.(\w+):\s+(\S+)$", k, flags=re.M))
            out[f["symbol"]] = f
    return out


def test_every_kernel_is_seen(kernels):
    names = " ".join(kernels)
    for part in ("score_kernel", "score_tile_kernel", "ffn_gemm_pp2_kernel", "ffn_mid_kernel", "ffn_few_kernel",
                 "attention_kernel", "attention_decode_kernel"):
        assert part in names, part


# scalars that a kernel keeps in lanes of a vector register outside its loops
SCALARS = {"select_kernel": 4, "score_tile_kernelILi64ELi64E": 21}


def test_no_spills(kernels):
    bad = {}
    for n, f in kernels.items():
        allowed = max([v for k, v in SCALARS.items() if k in n], default=0)
        if f["vgpr_spill_count"] != "0" or f["private_segment_fixed_size"] != "0" or int(f["sgpr_spill_count"]) > allowed:
            bad[n] = f["sgpr_spill_count"], f["vgpr_spill_count"], f["private_segment_fixed_size"]
    assert not bad, bad
