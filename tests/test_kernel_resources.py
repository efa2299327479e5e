"""What the compiler gives the kernels whose measured rates depend on it, read from its resource remarks (no GPU needed):
wavefronts per SIMD as the launch bounds ask for, and no more registers spilled to memory than when they were measured, which
no parity test would notice."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# kernel (mangled name contains): wavefronts per SIMD at least, spilled vector registers at most.  k_pack* code a chunk by
# workgroups of 8 wavefronts with 33 KB of LDS, of which 4 fit a compute unit: 8 per SIMD, from fp32 rows (16 registers per
# array more) 4.
LIMITS = {"k_pack_keys": (8, 34), "6k_packILi1ELb0": (8, 10), "6k_packILi2ELb0": (8, 10), "6k_packILi0ELb0": (4, 0),
          "6k_packILi0ELb1": (4, 0), "6k_packILi1ELb1": (4, 0), "6k_packILi2ELb1": (4, 0), "7kb_packILi0": (4, 0), "7kb_packILi1": (8, 10), "7kb_packILi2": (8, 10)}
# The calls in one launch: workgroups of 8 wavefronts that wait for each other, and the host counts on two of them per compute
# unit being resident: 4 per SIMD.  Several blobs in binary64: 64 registers hold the running values.
ONE_LAUNCH = {"lc_encode.hip": {"12k_encode_oneILi%dE" % t: (4, 0) for t in range(3)},
              "lc_decode_one.hip": {"12k_decode_oneILi%dELb%dE" % (t, many): (4, 20 if t == 3 and many else 0) for t in range(4) for many in range(2)}}


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("source", ["lc_encode.hip", "lc_decode_one.hip"])
def test_wavefronts_per_simd_and_spills(tmp_path, source):
    from paper_2009_13003_amd import build
    flags = [f for f in build.FLAGS if f != "-shared"]
    res = subprocess.run(["hipcc"] + flags + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", "-o",
                                              str(tmp_path / "out.o"), os.path.join(build.CSRC, source)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    found = {}
    for b in re.split(r"remark: Function Name: ", res.stderr)[1:]:
        occ, spill = re.search(r"Occupancy \[waves/SIMD\]: (\d+)", b), re.search(r"VGPRs Spill: (\d+)", b)
        if occ and spill:
            found[b.split()[0]] = (int(occ.group(1)), int(spill.group(1)))
    limits = dict(LIMITS if source == "lc_encode.hip" else {}, **ONE_LAUNCH[source])
    for name, (occupancy, spills) in limits.items():
        match = [v for k, v in found.items() if name in k]
        assert len(match) == 1, (name, sorted(found))
        assert match[0][0] >= occupancy and match[0][1] <= spills, (name, match)
