"""LDS of the filter kernels, as the compiler records it beside each kernel of the
built library: how many blocks a CU holds depends on it, so it is held where it
was measured."""
import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def lds(tmp_path_factory):
    """Static LDS bytes by kernel name (mangled)."""
    from paper_2204_06204_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2204_06204_amd.build import build
        build()
    data = open(_lib.LIB_PATH, "rb").read()
    out = {}
    for at in (m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)):
        pos = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, name_len = struct.unpack_from("<QQQ", data, pos)
            if size and b"gfx950" in data[pos + 24:pos + 24 + name_len]:
                obj = tmp_path_factory.mktemp("co") / "kernels.o"
                obj.write_bytes(data[at + off:at + off + size])
                notes = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
                for m in re.finditer(r"\.group_segment_fixed_size: (\d+).*?\.name:\s+(\S+)", notes, re.S):
                    out[m[2]] = int(m[1])
            pos += 24 + name_len
    assert out
    return out


def _kernel(lds, name, args):
    """The one kernel `name` whose mangled template arguments are `args`."""
    found = [v for k, v in lds.items() if f"{len(name)}{name}I{args}E" in k]
    assert len(found) == 1, (name, args)
    return found[0]


@pytest.mark.parametrize("t", ["f", "d"])
def test_identity_filter_stages_nothing(lds, t):
    """A filter without neighbours has its values in registers: beside the sum's
    few words (16 waves' values) it needs no LDS."""
    assert _kernel(lds, "k_filter_z", f"{t}Li0ELb0E") <= 16 * 8 + 16


@pytest.mark.parametrize("radius", [0, 1])
@pytest.mark.parametrize("t", ["f", "d"])
def test_filter_step_lds(lds, t, radius):
    """The fused filter and step: no more LDS than before it also wrote records
    (30,840 bytes: five blocks of four waves on a CU)."""
    assert _kernel(lds, "k_filter_z", f"{t}Li{radius}ELb1E") <= 30840
