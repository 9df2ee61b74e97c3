"""What the compiler made of the kernels in the built library, from the metadata of its code objects: kernels whose
state outgrows the registers keep it in scratch memory, and nothing but their time shows it."""
import os
import re
import subprocess

import pytest

from paper_2508_19740_amd import build as hip_build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled kernel name: (registers, spilled registers)} of every kernel of the library."""
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf is not installed")
    with open(hip_build.LIB, "rb") as f:
        blob = f.read()
    tmp = tmp_path_factory.mktemp("code")
    found = {}
    for at in (m.start() for m in re.finditer(MAGIC, blob)):
        n = int.from_bytes(blob[at + 24:at + 32], "little")       # entries: offset, size, length of the name, name
        p = at + 32
        for _ in range(n):
            off, size, ln = (int.from_bytes(blob[p + 8 * i:p + 8 * i + 8], "little") for i in range(3))
            name, p = blob[p + 24:p + 24 + ln], p + 24 + ln
            if b"gfx950" not in name:
                continue
            path = tmp / f"{at}.elf"
            path.write_bytes(blob[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for k in re.split(r"\n  - \.", notes)[1:]:
                k = "." + k
                get = {key: re.search(rf"\.{key}:\s+(\S+)", k) for key in ("symbol", "vgpr_count", "vgpr_spill_count")}
                if all(get.values()):
                    found[get["symbol"][1].strip("'\"").removesuffix(".kd")] = (int(get["vgpr_count"][1]), int(get["vgpr_spill_count"][1]))
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout.split("\n")
    return dict(zip(names, found.values()))


def test_score_kernels_keep_their_state_in_registers(kernels):
    """Every supported pair of code length and group, every width it is run with.  A few dozen registers in
    scratch cost less than the width gains (measured up to 38); from about 50 on the narrower kernel is faster."""
    spilled = {}
    pairs = set()
    for name, (_, spill) in kernels.items():
        m = re.search(r"score_kernel<(\d+), (\d+), [^>]*>", name)
        if m:
            pairs.add((int(m[1]), int(m[2])))
            spilled[m[0]] = spill
    assert pairs == {(w, g) for w in range(1, 17) for g in range(1, 9)} | {(32, 1), (32, 2)}
    assert {k: v for k, v in spilled.items() if v > 40} == {}
    assert {k: v for k, v in spilled.items() if ", 512, 2>" in k and v} == {}      # that width exists for its registers
