"""Host emulation of the probe pass's inner loops: a wave of probe_window (groups
of one to four hashes) and probe_single, cut out of bloom.hip and compiled by
g++ against the stand-in for the HIP device runtime of tests/emu (64 threads in
step), with AddressSanitizer and UBSan, against a direct query: filters that
LDS holds whole, in part and hardly, one to thirteen hashes, both layouts,
ragged windows, overflowing queues, the sender's selection; and the rule that
picks the group.  Host code only: no GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2102_03112_amd", "csrc")
EMU = os.path.join(ROOT, "tests", "emu")


def _between(text, start, end):
    a = text.index(start)
    return text[a:text.index(end, a)]


@pytest.fixture(scope="module")
def emulator(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("probe_emu")
    src = open(os.path.join(CSRC, "bloom.hip")).read()
    (d / "ext_sizes.inc").write_text(_between(src, "constexpr uint32_t PB_THREADS", "// The filter a tile is probed"))
    (d / "ext_groups.inc").write_text(_between(src, "// A tensor's filter as the probe", "// The receiver's dense output starts"))
    (d / "ext_windows.inc").write_text(_between(src, "// One window: the indices", "// A wave's window: ns steps"))
    exe = d / "probe_emu"
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-DEMU_WAVE_IN_STEP", f"-I{d}", f"-I{EMU}", f"-I{CSRC}", "-o", str(exe),
           os.path.join(EMU, "probe_emu.cpp"), os.path.join(EMU, "emu_rt.cpp"), "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return str(exe)


@pytest.mark.parametrize("layout", [0, 1], ids=["standard", "partitioned"])
@pytest.mark.parametrize("k", [1, 2, 3, 7, 13])
def test_probe_window_on_the_host(emulator, k, layout):
    r = subprocess.run([emulator, str(k), str(layout)], capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert r.stdout.startswith("OK"), r.stdout
