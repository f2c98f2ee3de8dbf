"""Host code under sanitizers, on the CPU.

* The oracle (oracle/hps_oracle.cpp) is built with gcc's AddressSanitizer and
  UndefinedBehaviorSanitizer and the whole oracle test file runs against that build in a child
  process (the sanitizer runtime has to be loaded before the interpreter starts).
* The host side of the HIP library is built with -fsanitize=undefined in trap mode (this
  image ships no clang sanitizer runtime, so undefined behaviour ends the process instead of
  being reported, and there is no AddressSanitizer for it) and the C ABI's argument checks
  (tests/test_abi.py: calls that return before anything touches a GPU) run against that build.
* The clamping of bags' offsets (csrc/pool.hpp), compiled for the host the same way, is given offsets of every kind.
"""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run_pytest(test_file, env_extra):
    env = dict(os.environ)
    env.update(env_extra)
    res = subprocess.run([sys.executable, "-m", "pytest", os.path.join(ROOT, "tests", test_file), "-x", "-q",
                          "-p", "no:cacheprovider"], cwd=ROOT, env=env, stdout=subprocess.PIPE,
                         stderr=subprocess.STDOUT, text=True, timeout=600)
    return res.returncode, res.stdout


def test_oracle_under_address_and_undefined_behaviour_sanitizers(tmp_path):
    gxx = shutil.which("g++")
    asan = subprocess.run(["gcc", "-print-file-name=libasan.so"], stdout=subprocess.PIPE, text=True).stdout.strip()
    if not gxx or not os.path.isabs(asan) or not os.path.exists(asan):
        pytest.skip("no g++ / libasan here")
    lib = str(tmp_path / "libhps_oracle_san.so")
    subprocess.check_call([gxx, "-O1", "-g", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared",
                           "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-o", lib,
                           os.path.join(ROOT, "oracle", "hps_oracle.cpp")])
    preload = asan + (":" + os.environ["LD_PRELOAD"] if os.environ.get("LD_PRELOAD") else "")
    rc, out = _run_pytest("test_oracle.py", {"HPS_ORACLE_LIB": lib, "LD_PRELOAD": preload,
                                             "ASAN_OPTIONS": "detect_leaks=0"})
    assert rc == 0 and "AddressSanitizer" not in out and "runtime error" not in out, out[-4000:]


def test_abi_argument_checks_with_undefined_behaviour_traps(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc here")
    lib = str(tmp_path / "libhps_ubsan.so")
    res = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-shared", "-fPIC",
                          "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fsanitize-trap=undefined",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-o", lib,
                          os.path.join(ROOT, "paper_2003_05622_amd", "csrc", "hps.hip")],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-4000:]
    rc, out = _run_pytest("test_abi.py", {"HPS_LIB": lib})
    assert rc == 0, out[-4000:]


BAGS = r"""
#include "pool.hpp"
#include <climits>
#include <cstdio>
using namespace hps;
int main() {
  const u32 sizes[] = {0u, 1u, 7u, 4096u, (1u << 30) - 1};
  for (u32 n : sizes) {
    const i32 m = (i32)n;
    const i32 some[] = {INT_MIN, INT_MIN + 1, -8, -1, 0, 1, 5, 4095, 4096, m - 1, m, m + 1, m + 8, INT_MAX - 8, INT_MAX - 7, INT_MAX - 1, INT_MAX};
    for (i32 a : some)
      for (i32 b : some) {
        const i32 offsets[2] = {a, b};
        const BagRange r = load_bag(offsets, 0, 1, n);
        i32 turns = 0;                       // (as the kernel goes through a bag; a long one's first turns)
        bool inside = true, last = false;
        for (i32 i0 = r.lo; !last && turns < 4; i0 += kPoolInFlight, ++turns) {
          last = i0 + kPoolInFlight >= r.hi;
          for (int j = 0; j < kPoolInFlight; ++j) inside = inside && (!(i0 + j < r.hi) || (i0 + j >= 0 && i0 + j < m));
        }
        const bool proper = a >= 0 && a <= b && b <= m;
        if (!inside || r.lo < 0 || r.hi < r.lo || r.hi > m || (proper && (r.lo != a || r.hi != b))) { std::printf("%u: %d %d\n", n, a, b); return 1; }
      }
  }
  const i32 offsets[2] = {3, 4};
  const BagRange none = load_bag(offsets, 1, 1, 10);
  std::puts(none.lo == 0 && none.hi == 0 ? "bags ok" : "a bag beyond the last");
  return 0;
}
"""


def test_bag_ranges_stay_inside_whatever_the_offsets(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc here")
    (tmp_path / "bags.hip").write_text(BAGS)
    exe = str(tmp_path / "bags")
    res = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17",
                          "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fsanitize-trap=undefined",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                          "-I", os.path.join(ROOT, "paper_2003_05622_amd", "csrc"), "-o", exe, str(tmp_path / "bags.hip")],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-4000:]
    res = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert res.returncode == 0 and "bags ok" in res.stdout, (res.returncode, res.stdout[-4000:])
