"""Properties of the built device code, from the metadata that the compiler leaves in libkperf.so, and of the binding, both without a GPU."""
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
    assert len(found) == 14, found  # five forms of the wait kernel, nine of the timeline kernel
    assert not any(found.values()), found


@pytest.mark.parametrize("raw_lookup", [True, False])
def test_a_call_without_a_stream_takes_torchs_current_one(monkeypatch, raw_lookup):
    """With torch's lookup of the bare handle, and by its public interface where a torch does not have that."""
    torch = pytest.importorskip("torch")
    from paper_2505_21661_amd import binding

    class Stream:
        cuda_stream = 0x5000

    monkeypatch.setattr(torch.cuda, "init", lambda: None)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 0x4000 + device, raising=False)
    if not raw_lookup:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    monkeypatch.setattr(binding, "_current_stream", None, raising=False)
    assert binding._stream(None) == (0x4003 if raw_lookup else 0x5000)
    assert binding._stream(None) == (0x4003 if raw_lookup else 0x5000)
    assert binding._stream(7) == 7 and binding._stream(Stream) == 0x5000


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_every_kernel_of_the_statistics_is_taken_by_some_geometry(tmp_path):
    """Either side of the lines in the numbers of workgroups and regions, all waves and ring sizes."""
    from tests import fake_hip

    calls = [{"fn": "kp_trace_reduce_hdr", "trace": (n_wg, waves, regions, 1 << log2)} for n_wg in (1, 257, 401, 1401, 2600)
             for waves in range(1, 17) for regions in (1, 8, 9, 16, 17, 32, 33, 64, 65, 128) for log2 in range(1, 20)]
    taken = {x[0] for _, launches in fake_hip.run(calls, tmp_path) for x in launches}
    built = {k for k in kernels(tmp_path) if "kp_reduce" in k}
    assert built and built == taken, built ^ taken
