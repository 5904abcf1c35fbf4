"""How many wavefronts of the gather kernels a SIMD holds, from the compiler's resource report: registers
decide it, and a kernel that needs a few more than its share loses a whole workgroup per CU.  Nothing may
spill.  No GPU."""
import os
import re
import subprocess

import pytest

from paper_2203_05016_amd import build as lib_build

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# (V, columns of a tile, wavefronts of a workgroup that split a tile, result, geometry) -> wavefronts per SIMD
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


def _report():
    r = subprocess.run([HIPCC, "-x", "hip", "-c", os.path.join(HERE, "kernel_resources.hip"), "-o", os.devnull,
                        "--offload-device-only", "-Rpass-analysis=kernel-resource-usage"] + lib_build.FLAGS,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=300)
    text = r.stdout.decode()
    assert r.returncode == 0, text[-2000:]
    found = {}
    for part in text.split("Function Name: ")[1:]:
        name = part.split()[0]
        m = re.search(r"gather_kernelILi(\d+)ELi(\d+)ELi\d+ELi\d+E(f|DF16_)NS_\d+([A-Za-z]+)(ILb([01])EE)?ELb\dELi(\d+)EEE", name)
        if m:
            geom = m.group(4) + ("" if m.group(6) is None else "<%s>" % ("true" if m.group(6) == "1" else "false"))
            key = (int(m.group(1)), int(m.group(2)), int(m.group(7)), "f32" if m.group(3) == "f" else "16", geom)
            found[key] = (int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", part).group(1)),
                          int(re.search(r"VGPRs Spill: (\d+)", part).group(1)))
    return found


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_gather_kernels_keep_their_residency():
    found = _report()
    assert set(found) == set(WANTED)
    for key, want in WANTED.items():
        waves, spilled = found[key]
        assert spilled == 0, (key, spilled)
        assert waves >= want, (key, waves, want)
