"""Registers of the built kernels, read from the metadata of the code objects in
libhuge.so.  The step's kernels live on the rows that their waves have in
flight and on what fits beside them, so a variant must not lose a wave per SIMD
(512 registers, given out eight at a time) unnoticed."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2307_14490_amd as P

LIB = os.path.join(os.path.dirname(P.__file__), "libhuge.so")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
FILT = shutil.which("c++filt") or "/opt/rocm/llvm/bin/llvm-cxxfilt"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled name: (VGPRs, bytes of scratch per thread)} of every kernel."""
    if not os.path.exists(READELF) or not os.path.exists(FILT):
        pytest.skip("no llvm-readelf or c++filt")
    P.load()  # builds the library if there is none
    data = open(LIB, "rb").read()
    magic, out = b"__CLANG_OFFLOAD_BUNDLE__", {}
    at = data.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n if n < 16 else 0):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name and size:
                f = tmp_path_factory.mktemp("co") / "k.co"
                f.write_bytes(data[at + off:at + off + size])
                notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True,
                                       text=True).stdout
                for k in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
                    get = lambda key: re.search(r"\." + key + r":\s+(\S+)", k).group(1)  # noqa: E731
                    out[get("symbol")] = (int(get("vgpr_count")),
                                          int(get("private_segment_fixed_size")))
        at = data.find(magic, at + 1)
    assert out
    names = subprocess.run([FILT], input="\n".join(s.removesuffix(".kd") for s in out),
                           capture_output=True, text=True).stdout.split("\n")
    return {n.replace("huge::", ""): v for n, v in zip(names, out.values())}


def waves(vgprs):
    return min(8, 512 // (-(-vgprs // 8) * 8))


# Waves per SIMD of k_fused_step by policy, table type, chunks or units per
# lane and negatives in flight (full: their number is K); 5 for float and 4 for
# bf16 tables where not listed (the least over the lanes per row).
LEAST = {
    ("PairIO", "bf16", 1, 8, False): 3, ("PairIO", "bf16", 1, 8, True): 3,
    ("PairIO", "bf16", 2, 5, True): 3, ("PairIO", "bf16", 2, 6, True): 3,
    ("PairIO", "bf16", 2, 8, False): 2, ("PairIO", "bf16", 2, 8, True): 2,
    ("RowIO", "bf16", 3, 8, False): 3, ("RowIO", "bf16", 3, 8, True): 3,
    ("RowIO", "bf16", 4, 5, True): 3, ("RowIO", "bf16", 4, 6, True): 3,
    ("RowIO", "bf16", 4, 8, False): 3, ("RowIO", "bf16", 4, 8, True): 2,
    ("RowIO", "f32", 1, 8, False): 4, ("RowIO", "f32", 2, 5, True): 4,
    ("RowIO", "f32", 2, 6, True): 4, ("RowIO", "f32", 2, 8, False): 3,
    ("RowIO", "f32", 2, 8, True): 3, ("RowIO", "f32", 3, 4, True): 4,
    ("RowIO", "f32", 3, 5, True): 4, ("RowIO", "f32", 3, 6, True): 3,
    ("RowIO", "f32", 3, 8, False): 2, ("RowIO", "f32", 3, 8, True): 2,
    ("RowIO", "f32", 4, 2, False): 4, ("RowIO", "f32", 4, 3, True): 4,
    ("RowIO", "f32", 4, 4, True): 3, ("RowIO", "f32", 4, 5, True): 3,
    ("RowIO", "f32", 4, 6, True): 2, ("RowIO", "f32", 4, 8, False): 2,
    ("RowIO", "f32", 4, 8, True): 2,
}


def test_fused_step_keeps_its_waves(kernels):
    seen, lost = 0, []
    for name, (vgprs, scratch) in kernels.items():
        m = re.search(r"k_fused_step<(\d+), (\d+), (true|false), (\w+)<(\d+), (\d+), "
                      r"(unsigned short|float)>", name)
        if m is None:
            continue
        lanes, nb, full = int(m[1]), int(m[2]), m[3] == "true"
        if not full and nb not in (2, 8):
            continue  # K = 1, 7 and above 8 are the counts that are no block's
        kind = "bf16" if m[7] == "unsigned short" else "f32"
        want = LEAST.get((m[4], kind, int(m[6]), nb, full), 5 if kind == "f32" else 4)
        if m[4] == "PairIO" and m[6] == "1" and nb == 8 and lanes >= 16 and full:
            want = 4
        if m[4] == "PairIO" and m[6] == "1" and nb == 8 and lanes <= 8 and not full:
            want = 4
        seen += 1
        if waves(vgprs) < want or scratch:
            lost.append((name[:90], vgprs, scratch, want))
    assert seen > 200 and not lost, lost


def test_fused_step_leaves_room_for_the_preparation(kernels):
    """The block of five negatives, the paper's count: 88 registers at five waves
    and 104 at four leave 72 and 96 to a wave of the next batch's preparation."""
    for name, (vgprs, _) in kernels.items():
        m = re.search(r"k_fused_step<(\d+), 5, true, (\w+)<\d+, 1, (unsigned short|float)>", name)
        if m is not None:
            assert vgprs <= (88 if m[3] == "float" else 104), name[:90]


def test_preparation_fits_beside_the_fused_step(kernels):
    """Nothing that runs beside it takes more than the 72 registers left, or keeps
    any in memory."""
    seen = 0
    for name, (vgprs, scratch) in kernels.items():
        m = re.search(r"k_(group|radix_pass)<(?:true|false|\d+), 256>|k_(sample|tile_scan)\(", name)
        if m is not None:
            seen += 1
            assert vgprs <= (72 if m[1] == "group" else 64) and scratch == 0, name[:90]
    assert seen == 7
