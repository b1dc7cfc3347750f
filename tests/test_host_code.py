"""Properties of the device code in libkperf.so, from the metadata that the compiler leaves in it (no GPU needed)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def kernels(tmp_path):
    """{mangled name: bytes of scratch memory per lane} of every kernel in the library."""
    lib = os.path.join(ROOT, "paper_2505_21661_amd", "libkperf.so")
    if not os.path.exists(lib):
        from paper_2505_21661_amd import build as kbuild

        kbuild.build()
    data = open(lib, "rb").read()
    found = {}
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        end = data.find(b"\x7fELF", at + 1)
        path = tmp_path / "code.o"
        path.write_bytes(data[at:end if end >= 0 else len(data)])
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True).stdout
        for entry in notes.split("- .agpr_count:")[1:]:
            found[re.search(r"\.name: +(\S+)", entry).group(1)] = int(re.search(r"\.private_segment_fixed_size: +(\d+)", entry).group(1))
        at = end
    return found


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_replay_kernels_hold_their_state_in_registers(tmp_path):
    """The bounds on hardware waves per SIMD leave every replay kernel the vector registers that it needs."""
    found = {k: v for k, v in kernels(tmp_path).items() if "kp_waits_main" in k or "kp_pairs_main" in k}
    assert len(found) == 10, found
    assert not any(found.values()), found
