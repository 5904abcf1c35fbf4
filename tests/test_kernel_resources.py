"""How many wavefronts of the gather kernels, the resident slab and the LayerNorm-side transposition a SIMD holds, from the
compiler's resource report: registers decide it, and a kernel that needs a few more than its share loses a whole workgroup per CU,
or cannot be launched.  The report is that of the library's own launch files, so that every kernel named here is one that the
library launches.  None of the kernels in them may spill, but where it says so.  No GPU."""
import os
import re
import subprocess

import pytest

from paper_2203_05016_amd import build as lib_build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCES = ["launch_gather_f16.hip", "launch_gather_conv_f16.hip", "launch_gather_stride2_f16.hip"]

# (V, columns of a tile, wavefronts of a workgroup that split a tile - 0: whole tiles of shared weights -, result,
# geometry) -> wavefronts per SIMD
WANTED = {
    (32, 64, 1, "16", "GeomLinearBuf"): 4,
    (64, 64, 1, "16", "GeomLinearBuf"): 4,
    (64, 64, 1, "f32", "GeomLinearBuf"): 4,
    (128, 64, 1, "16", "GeomLinearBuf"): 2,
    (64, 64, 2, "f32", "GeomLinearBuf"): 4,
    (128, 64, 2, "16", "GeomRows"): 2,
    (64, 64, 1, "16", "GeomConvRuns<false>"): 4,
    (64, 64, 2, "16", "GeomConvRuns<false>"): 4,
    (64, 64, 4, "16", "GeomConvRuns<false>"): 4,
    (64, 64, 4, "f32", "GeomConvRuns<true>"): 4,
    (128, 64, 2, "16", "GeomConvRuns<false>"): 2,
    (128, 64, 4, "16", "GeomConvRuns<true>"): 2,
}
for _geom in ("GeomLinearBuf", "GeomRows"):
    for _out in ("16", "f32"):
        # weights shared through the LDS
        for _V, _waves in ((16, 4), (32, 4), (64, 3), (128, 2)):
            WANTED[(_V, 64, 0, _out, _geom)] = _waves
        for _V in (16, 32, 64):
            WANTED[(_V, 128, 0, _out, _geom)] = 2
        # 128 columns, and their steps shared by 2 and 4
        for _V, _waves in ((16, 3), (32, 3), (64, 2)):
            WANTED[(_V, 128, 1, _out, _geom)] = _waves
        for _V, _waves in ((16, 3), (32, 2), (64, 2)):
            WANTED[(_V, 128, 2, _out, _geom)] = _waves
            WANTED[(_V, 128, 4, _out, _geom)] = _waves
for _geom in ("GeomConvRuns<false>", "GeomConvRuns<true>", "GeomQuads", "GeomNarrow", "GeomLinear<true>", "GeomLinear<false>"):
    for _out in ("16", "f32"):
        WANTED[(32, 128, 1, _out, _geom)] = 3
        WANTED[(64, 128, 1, _out, _geom)] = 2
for _V, _waves in ((16, 3), (32, 4), (64, 3), (128, 2)):
    for _split in (1, 2, 4, 8):
        WANTED[(_V, 64, _split, "16", "GeomConvRuns2")] = _waves
    if _V < 128:
        WANTED[(_V, 128, 1, "16", "GeomConvRuns2")] = 2
for _geom in ("GeomLinear<true>", "GeomLinear<false>"):
    WANTED[(64, 64, 1, "16", _geom)] = WANTED[(64, 64, 1, "f32", _geom)] = 4


def _kernels(sources):
    """(mangled name, wavefronts per SIMD, spilled registers) of every kernel of the sources"""
    jobs = [subprocess.Popen([HIPCC, "-x", "hip", "-c", os.path.join(lib_build.CSRC, source), "-o", os.devnull, "--offload-device-only",
                              "-Rpass-analysis=kernel-resource-usage"] + lib_build.FLAGS,
                             stdout=subprocess.PIPE, stderr=subprocess.STDOUT) for source in sources]
    for job in jobs:
        text = job.communicate(timeout=600)[0].decode()
        assert job.returncode == 0, text[-2000:]
        for part in text.split("Function Name: ")[1:]:
            yield (part.split()[0], int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", part).group(1)),
                   int(re.search(r"VGPRs Spill: (\d+)", part).group(1)))


def _report():
    found = {}
    for name, waves, spill in _kernels(SOURCES):
        m = re.search(r"gather_kernelILi(\d+)ELi(\d+)ELi\d+E(f|DF16_)NS_(\d+)([A-Za-z0-9]+?)(ILb([01])EE)?ELb\dELi(\d+)EEE", name)
        if m:
            geom = m.group(5) + ("" if m.group(7) is None else "<%s>" % ("true" if m.group(7) == "1" else "false"))
            key = (int(m.group(1)), int(m.group(2)), int(m.group(8)), "f32" if m.group(3) == "f" else "16", geom)
            assert key not in found, key
            found[key] = (waves, spill)
    return found


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_gather_kernels_keep_their_residency():
    found = _report()
    assert not set(WANTED) - set(found), set(WANTED) - set(found)
    short = {key: (found[key], want) for key, want in WANTED.items() if found[key][0] < want}
    assert not short, short
    spilled = {key: value for key, value in found.items() if value[1]}
    assert not spilled, spilled


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_resident_kernels_can_be_launched_and_do_not_spill():
    """A workgroup of 16 wavefronts needs 4 per SIMD to exist at all, and two of 8 (V <= 32) to share a CU; V >= 64 has 8 per CU."""
    seen = set()
    for name, waves, spill in _kernels(["launch_resident_f16.hip", "launch_resident_conv_f16.hip"]):
        m = re.search(r"slab_kernel_residentILi(\d+)ELi(\d+)E", name)
        assert m and spill == 0 and waves >= (4 if int(m.group(1)) <= 32 else 2), (name, waves, spill)
        seen.add((int(m.group(1)), int(m.group(2))))
    assert seen == {(16, 8), (16, 16), (32, 8), (32, 16), (64, 8), (128, 8)}


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_layernorm_kernels_can_be_launched():
    """Workgroups of 16 wavefronts: 4 per SIMD (the streaming kernel's 8 wavefronts: 2).  One spilled register in the kernels that hold 4096
    features of two tokens, in 64 registers; none in the others."""
    seen = set()
    for name, waves, spill in _kernels(["layernorm_transpose.hip"]):
        kind = re.search(r"layernorm_transpose_(few|resident|register|kernel)", name).group(1)
        assert spill <= (1 if kind == "register" else 0) and waves >= (2 if kind == "kernel" else 4), (name, waves, spill)
        seen.add(kind)
    assert seen == {"few", "resident", "register", "kernel"}
