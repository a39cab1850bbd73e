"""Properties of the device code in the built librtn.so that its sources cannot state to the compiler."""
import os
import re
import struct
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_1912_02057_amd import build

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """The library's code objects, one per source with kernels, as files."""
    if not os.path.exists(build.LIB):
        build.build_lib()
    d, out, at = open(build.LIB, "rb").read(), [], -1
    while (at := d.find(MAGIC, at + 1)) >= 0:
        n, q = struct.unpack_from("<Q", d, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", d, q)
            if b"gfx950" in d[q + 24:q + 24 + idlen]:
                out.append(str(tmp_path_factory.mktemp("co") / "code.o"))
                with open(out[-1], "wb") as f:
                    f.write(d[at + off:at + off + size])
            q += 24 + idlen
    assert len(out) >= 10
    return out


def _scalars(operand):
    m = re.fullmatch(r"s(\d+)|s\[(\d+):(\d+)\]", operand)
    if not m:
        return set()
    return {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))


def _direct_loads(obj):
    """(instruction, wait states since M0 was written, least wait states since a vector instruction wrote one of its
    scalar registers) of every load to LDS; None where nothing did within 8 instructions."""
    asm = subprocess.run([LLVM + "/llvm-objdump", "-d", "--no-show-raw-insn", obj], check=True, stdout=subprocess.PIPE, text=True).stdout
    lines = asm.split("\n")
    found = []
    for i, line in enumerate(lines):
        if "load_lds" not in line and " lds" not in line:
            continue
        text = line.split("//")[0].strip()
        used = set().union(*[_scalars(t) for t in re.split(r"[ ,]+", text)[1:]])
        waits, m0, vec = 0, None, None
        for prev in reversed(lines[max(0, i - 8):i]):
            t = re.split(r"[ ,]+", prev.split("//")[0].strip())
            if len(t) < 1 or not t[0] or t[0].endswith(":"):
                break
            if t[0].startswith("s_") and len(t) > 1:
                if t[1] == "m0" and m0 is None:
                    m0 = waits
                used -= _scalars(t[1])
            elif t[0].startswith("v_") and len(t) > 1:
                dst = _scalars(t[1]) if t[0].startswith("v_cmp") else _scalars(t[1]) | (_scalars(t[2]) if "_co" in t[0] else set())
                if dst & used and vec is None:
                    vec = waits
            waits += int(t[1], 0) + 1 if t[0] == "s_nop" else 1
        found.append((text, m0, vec))
    return found


def test_direct_loads_have_their_wait_states(objects):
    """gfx9: one wait state between a scalar write of M0 and a load to LDS, five between a vector instruction's write of a
    scalar register and a load that reads it.  The compiler does not look into the statements that hold these loads."""
    with ThreadPoolExecutor(8) as ex:
        loads = [l for found in ex.map(_direct_loads, objects) for l in found]
    assert len(loads) > 1000
    assert not [l for l in loads if l[1] is None or l[1] < 1][:5]
    assert not [l for l in loads if l[2] is not None and l[2] < 5][:5]


def _kernels(obj):
    """name -> (vector registers, bytes of scratch) from the object's metadata"""
    notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", obj], check=True, stdout=subprocess.PIPE, text=True).stdout
    field = lambda text, key: int(re.search(r"\.%s:\s+(\d+)" % key, text)[1])
    return {re.search(r"\.name:\s+(_Z\S+)", k)[1]: (field(k, "vgpr_count"), field(k, "private_segment_fixed_size"))
            for k in re.split(r"\n  - \.agpr_count|\n  - \.args", notes)[1:] if re.search(r"\.name:\s+_Z", k)}


def test_gathering_weight_only_conv_has_two_blocks_per_cu(objects):
    """Its 64 x 64 form has blocks of 16 waves and LDS for two of them: 64 registers a lane, without scratch."""
    found = {n: v for obj in objects for n, v in _kernels(obj).items() if re.search(r"k_wconvILi64ELi64ELi2ELi2ELi4ELi\d+ELi0ELi2ELi64E", n)}
    assert len(found) == 2
    assert all(vgprs <= 64 and scratch == 0 for vgprs, scratch in found.values()), found
