"""Registers of the built kernels, from the code objects' own metadata (no GPU): the
batched kernels that launches are sized for keep the waves per SIMD that the sizing
assumes, and the batched query of hands of up to five fingers keeps nothing in scratch
memory."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2511_07418_amd", "liblg.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
OBJCOPY = "/opt/rocm/llvm/bin/llvm-objcopy"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> (vector registers, scratch bytes per lane) of every kernel of the library"""
    if not os.path.exists(LIB) or not os.path.exists(READELF) or not shutil.which("c++filt"):
        pytest.skip("no built library or no ELF tools")
    d = tmp_path_factory.mktemp("co")
    fat = str(d / "fat")
    subprocess.run([OBJCOPY, "--dump-section", ".hip_fatbin=" + fat, LIB, str(d / "rest")], check=True)
    data = open(fat, "rb").read()
    at = [m.start() for m in re.finditer(b"\x7fELF\x02\x01\x01", data)] + [len(data)]
    out = {}
    for i, (a, b) in enumerate(zip(at, at[1:])):
        co = str(d / f"co{i}")
        open(co, "wb").write(data[a:b])
        notes = subprocess.run([READELF, "--notes", co], capture_output=True, text=True).stdout
        for block in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.symbol:\s+'?(\S+?)\.kd", block)
            if name:
                out[name[1]] = (int(re.search(r"\.vgpr_count:\s+(\d+)", block)[1]),
                                int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", block)[1]))
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True).stdout.splitlines()
    return {n.split("(")[0].removeprefix("void "): v for n, v in zip(names, out.values())}


def test_penetration_keeps_four_waves_per_simd(kernels):
    found = {n: v for n, v in kernels.items() if n.startswith("lg::k_penetrate")}
    assert len(found) == 4, sorted(kernels)
    assert all(v[0] <= 128 for v in found.values()), found


def test_batched_query_uses_no_scratch_up_to_five_fingers(kernels):
    found = {n: v for n, v in kernels.items() if re.match(r"lg::k_query_batch<\d, [345], ", n)}
    assert len(found) == 12, sorted(kernels)
    assert all(v[1] == 0 and v[0] <= 64 for v in found.values()), found
