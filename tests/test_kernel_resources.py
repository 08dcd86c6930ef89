"""Registers of the built kernels, read from the library's own code object
(no GPU): the direct J/K primitive-lane kernels that serve long FP64 lists
hold the recursion's values in all of a lane's registers, so what else is
kept there goes to scratch memory and is paid for in every primitive quartet.

The bounds are the scratch bytes a lane of these kernels when each block is
one wave and the Boys function is the eight-term Taylor sum (measured: the
(dd|ds) kernel of 20 waters moves 2.1 GB a launch with 180 bytes, 3.2 GB with
232)."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel symbol: {metadata key: value}} of every device code object in the library."""
    from paper_2406_03121_amd import build as hipbuild
    if not os.path.exists(hipbuild.LIB):
        hipbuild.build()
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    data = open(hipbuild.LIB, "rb").read()
    out = {}
    tmp = tmp_path_factory.mktemp("co")
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" not in name or not size:
                continue
            f = tmp / "obj"
            f.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
            for entry in re.split(r"\n\s+- \.a", notes):
                sym = re.search(r"\.symbol:\s+'?(\S+?)\.kd'?\s", entry)
                if sym:
                    out[sym[1]] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\b", entry)}
        at = data.find(MAGIC, at + 1)
    return out


# (la, lb, lc, ld), scratch bytes a lane
@pytest.mark.parametrize("l,scratch", [((2, 2, 2, 1), 20), ((2, 2, 2, 0), 180), ((2, 1, 2, 1), 260), ((2, 2, 1, 1), 240),
                                       ((2, 1, 1, 1), 20), ((2, 2, 1, 0), 0), ((1, 1, 1, 1), 0)])
def test_primitive_lane_scratch(kernels, l, scratch):
    dims = r"k_planeI\w*?ClassDimsI" + "".join(f"Li{x}E" for x in l) + "E"
    mode_jk = r"E?Li2EdLi1E"
    found = [(s, m) for s, m in kernels.items() if re.search(dims + mode_jk, s)]
    assert len(found) == 1, [s for s in kernels if "k_plane" in s][:5]
    assert found[0][1]["private_segment_fixed_size"] <= scratch
    # two waves a SIMD, but for (dd|dp)
    if l != (2, 2, 2, 1):
        assert found[0][1]["vgpr_count"] <= 256
