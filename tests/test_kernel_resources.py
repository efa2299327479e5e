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


# The kernels of lc_decode.hip, which takes minutes to compile, and the batch's count, read from the library as built: vector registers
# at most (512 a SIMD: 168 leave room for 3 wavefronts, 128 for 4) and how many are spilled.
BUILT = {"8k_decodeILi%dELb0E" % t: (256 if t == 3 else 168, 0) for t in range(4)}
BUILT.update({"9kb_decodeILi%dE" % t: (168, 0) for t in range(3)})
# (kb_hist: two workgroups of 8 wavefronts per compute unit stay, three of fp32 come and go, or four)
BUILT.update({"7kb_histILi%dELb%dELb%dE" % (t, stay, short): (64 if short or (t and not stay) else 128 if stay else 85, 0)
              for t in range(3) for stay, short in ((0, 0), (1, 0), (0, 1))})
BUILT.update({"14k_decode_fusedILi%dELb%dELi%dE" % (n, longs, t): (128 if n <= 2 or (n, longs, t) == (3, 1, 0) else 168 if n <= 5 else 256, 0)
              for n in range(1, 9) for longs in range(2) for t in range(3)})
# (of 2 to 4 blobs of 8 symbols two workgroups share a compute unit; fp32 rows of 3 and 4 spill a few)
BUILT.update({"14k_decode_pairsILi%dELb0ELi%dE" % (n, t): (128 if n <= 4 else 256, {3: 2, 4: 6}.get(n, 0) if t == 0 else 0) for n in range(2, 9) for t in range(3)})
BUILT.update({"14k_decode_pairsILi%dELb1ELi%dE" % (n, t): (256, 0) for n in range(2, 5) for t in range(3)})


def registers_of(library, folder):
    """Kernel name -> (vector registers, spilled ones), from the notes of the library's code objects for the GPU."""
    import struct
    data, at, found = open(library, "rb").read(), 0, {}
    while True:
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)
        if at < 0:
            return found
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            offset, size, name = struct.unpack_from("<QQQ", data, entry)
            if size and b"gfx950" in data[entry + 24:entry + 24 + name]:
                with open(str(folder / "code"), "wb") as f:
                    f.write(data[at + offset:at + offset + size])
                notes = subprocess.run([os.path.join(ROCM, "llvm", "bin", "llvm-readelf"), "--notes", str(folder / "code")], capture_output=True, text=True).stdout
                for kernel in re.split(r"\n  - \.agpr_count", notes)[1:]:
                    field = lambda k: re.search(r"\.%s:\s+(\S+)" % k, kernel).group(1)
                    found[field("name")] = (int(field("vgpr_count")), int(field("vgpr_spill_count")))
            entry += 24 + name
        at += 24


ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(not os.path.exists(os.path.join(ROCM, "llvm", "bin", "llvm-readelf")), reason="needs llvm-readelf")
def test_registers_of_the_library_as_built(tmp_path):
    from paper_2009_13003_amd import build
    if not os.path.exists(build.LIB):
        build.build_library()
    found = registers_of(build.LIB, tmp_path)
    assert len(found) > 100, sorted(found)
    for name, (registers, spills) in BUILT.items():
        match = [v for k, v in found.items() if name in k]
        assert len(match) == 1, (name, sorted(found))
        assert match[0][0] <= registers and match[0][1] <= spills, (name, match)
