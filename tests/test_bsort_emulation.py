"""Host emulation of the bucket sort: k_bsort_split, k_bsort_deal and
k_bsort_bucket, cut out of valuefit.hip and compiled by g++ against the stand-in
for the HIP device runtime of tests/emu, with AddressSanitizer and UBSan.  Ranks
and sorted values are compared with a stable sort.  A store past a list of too
full bins, a barrier that some threads never reach or a wrong order fails the
test.  Host code only: no GPU."""
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
    d = tmp_path_factory.mktemp("bsort_emu")
    src = open(os.path.join(CSRC, "valuefit.hip")).read()
    (d / "ext_stile.inc").write_text(_between(src, "__device__ __forceinline__ uint32_t tensor_of_stile", "// Before the"))
    (d / "ext_bsort.inc").write_text(_between(src, "constexpr uint32_t BS_THREADS", "hipError_t launch_sort"))
    exe = d / "bsort_emu"
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           f"-I{d}", f"-I{EMU}", f"-I{CSRC}", "-o", str(exe), os.path.join(EMU, "bsort_emu.cpp"),
           os.path.join(EMU, "emu_rt.cpp"), "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return str(exe)


CAP = 4096  # a bucket's room; a mean bucket holds 1024

CASES = [
    # kind, then planned and actual values of each tensor
    ("normal", [(1, 1), (10, 0), (63, 63), (CAP, CAP), (6000, 5000)]),
    ("equal", [(CAP, CAP), (9000, 9000)]),
    ("coarse", [(CAP, CAP), (9000, 9000)]),  # several bins too full at once
    ("ulps", [(CAP, CAP), (20_000, 20_000)]),  # one bin cut into 30 too full ones
    ("signs", [(CAP, 4000)]),
    ("nested", [(160, 160), (CAP, CAP)]),
    ("normal", [(700, CAP + 1), (300, 300)]),  # planned as one bucket, and more values than its room
]


@pytest.mark.parametrize("kind,sizes", CASES, ids=[f"{k}-{s[0][1]}" for k, s in CASES])
def test_bucket_sort_on_the_host(emulator, kind, sizes):
    args = [str(x) for s in sizes for x in s]
    r = subprocess.run([emulator, kind, *args], capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert r.stdout.startswith("OK"), r.stdout
