"""What the gfx950 code of the built library has to contain where no run can be relied on to show it missing
(no GPU needed: the code objects are taken out of libkperf.so and disassembled)."""
import glob
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def reduce_functions(tmp_path_factory):
    """{mangled name: instructions} of the LDS-resident statistics decoder's code object."""
    import paper_2505_21661_amd as kp
    from paper_2505_21661_amd import build as kbuild

    if not os.path.exists(kp.binding.LIB_PATH):
        kbuild.build()
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    where = tmp_path_factory.mktemp("code")
    lib = shutil.copy(kp.binding.LIB_PATH, where)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=where, check=True, stdout=subprocess.DEVNULL)
    out = {}
    for path in glob.glob(str(where / "*gfx950")):
        if b"kp_reduce_main" not in open(path, "rb").read():
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", path], check=True,
                              capture_output=True, text=True).stdout
        for name, body in re.findall(r"^<(\w+)>:\n(.*?)(?=^<\w+>:|\Z)", text, flags=re.S | re.M):
            out[name] = [line.split("//")[0].strip() for line in body.splitlines() if line.strip()]
    return out


def counted_forms(functions):
    """The decoder kernels that count their workgroups: a release to the other workgroups (the write-back of the
    L2 cache) is only there."""
    return {n: c for n, c in functions.items() if "kp_reduce_main" in n and any(i.startswith("buffer_wbl2") for i in c)}


def test_every_wave_waits_for_its_atomics_before_its_workgroup_is_counted(reduce_functions):
    """The barrier ahead of the count does not wait for global memory, and the count's release only waits for the
    wave that counts: each wave has to wait for its own atomics on the statistics block in front of the barrier."""
    forms = counted_forms(reduce_functions)
    assert forms, "no counted form of the decoder found"
    multi_wave = 0
    for name, code in forms.items():
        release = next(k for k, i in enumerate(code) if i.startswith("buffer_wbl2"))
        atomics = [k for k in range(release) if code[k].startswith("global_atomic")]
        assert atomics, name
        barriers = [k for k in range(atomics[-1], release) if code[k].startswith("s_barrier")]
        multi_wave += bool(barriers)
        upto = barriers[0] if barriers else release  # (one wave needs no barrier)
        waits = [i for i in code[atomics[-1]:upto] if i.startswith("s_waitcnt") and "vmcnt(0)" in i]
        assert waits or not barriers, f"{name}: atomics in flight at the barrier before the count"
    assert multi_wave >= 2, sorted(forms)
