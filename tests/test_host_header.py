"""How the header of a trace in device memory gets to the host, over tests/fake_hip.c (no GPU needed): the host memory that
its kernel writes to, from the first call to a device reset, with threads that come and go."""
import ctypes
import json
import os
import subprocess
import sys
import threading

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COUNTS = ("kernels", "copies", "allocations", "frees", "stray_writes", "unguarded")


def run(what, tmp_path):
    from tests import fake_hip

    fake, lib = fake_hip.libraries(tmp_path)
    done = subprocess.run([sys.executable, os.path.abspath(__file__), fake, lib, what], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, (done.returncode, done.stderr[-2000:])
    return json.loads(done.stdout)


def test_a_thread_that_ends_makes_no_call_of_the_runtime(tmp_path):
    """One allocation serves all threads; nothing is freed behind a thread's back, where it could wait for kernels or
    break another thread's capture, and the allocation is made where a capture allows it."""
    got = run("threads", tmp_path)
    assert got["status"] == [0] * 40
    assert got["kernels"] == 40 and got["copies"] == 0
    assert got["allocations"] == 1 and got["frees"] == 0 and got["unguarded"] == 0


def test_after_a_device_reset_the_memory_is_allocated_anew(tmp_path):
    """Neither the kernel nor the host touches memory that the reset took back."""
    got = run("reset", tmp_path)
    assert got["status"] == [0, 0, 0, 0] and got["kernels"] == 4
    assert got["stray_writes"] == 0 and got["allocations"] == 1


def test_a_kernel_that_did_not_run_is_named(tmp_path):
    got = run("silent", tmp_path)
    assert all(s != 0 for s in got["status"][:3]) and "no error" not in got["error"] and "did not run" in got["error"]
    assert got["status"][3:] == [0, 0] and got["kernels"] == 5  # other places serve the calls behind


def test_without_a_place_the_header_is_copied(tmp_path):
    """Places that a kernel may still write to stay taken; with none left the header comes by the runtime's copy."""
    got = run("exhausted", tmp_path)
    assert all(s != 0 for s in got["status"][:-3]) and got["status"][-3:] == [0, 0, 0]
    assert got["copies"] == 3 and got["allocations"] == 1


def _child(fake_path, lib_path, what):
    from fake_hip import BUFFER, Hdr

    fake = ctypes.CDLL(fake_path, mode=ctypes.RTLD_GLOBAL)
    lib = ctypes.CDLL(lib_path)
    lib.kp_last_error.restype = ctypes.c_char_p
    hdr = Hdr(0x4652504B, 1, 6, 4, 3, 128, 20, 0)
    fake.fake_header(ctypes.byref(hdr))

    def call(status):
        p = ctypes.c_void_p(BUFFER)
        status.append(lib.kp_trace_reduce(p, ctypes.c_size_t(6 * 4 * 128), p, None))

    status, error = [], ""
    if what == "threads":
        for _ in range(10):
            batch = [threading.Thread(target=call, args=(status,)) for _ in range(4)]
            for t in batch:
                t.start()
            for t in batch:
                t.join()
    elif what == "reset":
        for _ in range(2):
            call(status)
            call(status)
            if len(status) == 2:
                fake.fake_reset()
    elif what == "silent":
        fake.fake_silent(1)
        for _ in range(3):
            call(status)
        error = lib.kp_last_error().decode()
        fake.fake_silent(0)
        call(status)
        call(status)
    elif what == "exhausted":
        fake.fake_silent(1)
        for _ in range(32):
            call(status)
        fake.fake_silent(0)
        for _ in range(3):
            call(status)
    out = {"status": status, "error": error}
    out.update((name, fake.fake_count(i)) for i, name in enumerate(COUNTS))
    print(json.dumps(out))


if __name__ == "__main__":
    _child(*sys.argv[1:])
