"""What a call of libkperf.so launches, found out without a GPU: run(calls) answers each call with its status and
its launches.  The library is loaded in a child process over tests/fake_hip.c in place of the HIP runtime."""
import ctypes
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUFFER = 0x10000000  # stands for any device buffer; never read or written


def libraries(tmp_path, lib=None):
    """Paths of the stand-in for the HIP runtime and of libkperf.so, both built if need be."""
    if lib is None:
        lib = os.path.join(ROOT, "paper_2505_21661_amd", "libkperf.so")
        if not os.path.exists(lib):
            from paper_2505_21661_amd import build as kbuild

            kbuild.build()
    fake = os.path.join(str(tmp_path), "libfake_hip.so")
    if not os.path.exists(fake):
        subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", fake, os.path.join(ROOT, "tests", "fake_hip.c")])
    return fake, lib


def run(calls, tmp_path, lib=None):
    """calls: dicts with "fn", and "trace" (n_wg, waves, regions, cap) or "args"; "device" (index, CUs, resident
    workgroups per CU).  Returns [(status, [(kernel, grid, block, dynamic LDS)])]."""
    fake, lib = libraries(tmp_path, lib)
    done = subprocess.run([sys.executable, os.path.abspath(__file__), fake, lib], input=json.dumps(calls), text=True,
                          capture_output=True, timeout=120)
    assert done.returncode == 0, (done.returncode, done.stderr[-2000:])
    return [(status, [tuple(x) for x in launches]) for status, launches in json.loads(done.stdout)]


class Hdr(ctypes.Structure):
    _fields_ = [(n, ctypes.c_uint32) for n in ("magic", "version", "n_wg", "waves", "n_regions", "cap_wave", "rec_cost", "flags")]
    _fields_ += [("pad", ctypes.c_uint32 * 8)]


def _child(fake_path, lib_path):
    fake = ctypes.CDLL(fake_path, mode=ctypes.RTLD_GLOBAL)
    fake.fake_launch.restype = ctypes.c_char_p
    lib = ctypes.CDLL(lib_path)
    p = lambda v: ctypes.c_void_p(v)  # noqa: E731
    out = []
    for call in json.loads(sys.stdin.read()):
        fake.fake_device(*call.get("device", (0, 256, 1)))
        fake.fake_forget()
        if "trace" in call:
            n_wg, waves, regions, cap = call["trace"]
            hdr = Hdr(0x4652504B, 1, n_wg, waves, regions, cap, 20, 0)
            status = getattr(lib, call["fn"])(p(BUFFER), ctypes.c_size_t(n_wg * waves * cap), ctypes.byref(hdr), p(BUFFER), None)
        elif call["fn"] == "kp_gemm_instrumented":
            m, n, k, mask, cap = call["args"]
            status = lib.kp_gemm_instrumented(p(BUFFER), p(BUFFER), p(BUFFER), m, n, k, ctypes.c_uint32(mask), p(BUFFER),
                                              ctypes.c_size_t(cap), None)
        elif call["fn"] == "kp_stages_critical":
            n_wg, regions, iterations = call["args"]
            status = lib.kp_stages_critical(p(BUFFER), n_wg, regions, iterations, p(BUFFER), None)
        else:
            raise ValueError(call["fn"])
        launches = []
        for i in range(fake.fake_launches()):
            grid, block, lds = ctypes.c_uint32(), ctypes.c_uint32(), ctypes.c_uint64()
            name = fake.fake_launch(i, ctypes.byref(grid), ctypes.byref(block), ctypes.byref(lds)).decode()
            launches.append((name, grid.value, block.value, lds.value))
        out.append((status, launches))
    print(json.dumps(out))


if __name__ == "__main__":
    _child(*sys.argv[1:])
