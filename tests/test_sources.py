"""Rules that the kernel sources keep, checked without a GPU."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_08061_amd", "csrc")


def sources():
    return {f: open(os.path.join(CSRC, f)).read() for f in sorted(os.listdir(CSRC))}


def test_wave_barriers_are_fences():
    """Lanes that exchange data through LDS without a workgroup barrier do so over a fence: a
    bare wave barrier orders no memory access."""
    for name, text in sources().items():
        helper = re.search(r"void wave_lds_fence\(\) \{.*?\n\}", text, re.S)
        rest = text.replace(helper.group(0), "") if helper else text
        assert "__builtin_amdgcn_wave_barrier" not in rest, name
        if helper:
            assert "__builtin_amdgcn_fence(__ATOMIC_ACQ_REL" in helper.group(0)
    assert "wave_lds_fence()" in sources()["luna_map_backward.hip"]


def test_past_end_offset_leaves_room():
    """The buffer offset that reads as 0 is one shared constant, and the offsets that a load
    adds to it (a second 16-byte piece at most) stay within an int."""
    found = {n: re.findall(r"0x7fff[0-9a-f]{4}", t) for n, t in sources().items()}
    others = {"0x7fff7fff", "0x7fffffff"}  # (all but the sign bits of a bf16 pair; the largest grid)
    values = {(n, v) for n, vs in found.items() for v in vs if v not in others}
    assert len(values) == 1, values
    (name, value), = values
    assert name == "luna_device.hpp" and f"constexpr int kPastEnd = {value};" in sources()[name]
    assert int(value, 16) + 64 < 2 ** 31


ALLOW_LDS = r"""
#include "luna_kernels.hpp"
#include <cstdio>
static int device = 0, calls = 0, fails = 0;
extern "C" hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) {
  ++calls;
  return fails-- > 0 ? hipErrorInvalidValue : hipSuccess;
}
static void one() {}
static void two() {}
int main() {
  int bad = 0;
  auto expect = [&](hipError_t e, hipError_t want, int n) {
    if (e != want || calls != n) printf("status %d calls %d, wanted %d and %d\n", e, calls, want, n), ++bad;
  };
  fails = 1;
  expect(luna::allow_lds<one>(1 << 17), hipErrorInvalidValue, 1);  // a failure is not kept
  expect(luna::allow_lds<one>(1 << 17), hipSuccess, 2);
  expect(luna::allow_lds<one>(1 << 17), hipSuccess, 2);  // a success is
  expect(luna::allow_lds<two>(1 << 17), hipSuccess, 3);  // for each kernel
  device = 3;
  expect(luna::allow_lds<one>(1 << 17), hipSuccess, 4);  // and each device
  expect(luna::allow_lds<one>(1 << 17), hipSuccess, 4);
  device = 64;
  expect(luna::allow_lds<one>(1 << 17), hipSuccess, 5);
  expect(luna::allow_lds<one>(1 << 17), hipSuccess, 6);
  return bad;
}
"""


def test_dynamic_lds_is_asked_of_every_device(tmp_path):
    """The attribute that lets a kernel take more than 64 KiB of dynamic LDS, against stand-ins
    for the two runtime calls; no launcher sets it by itself."""
    for name, text in sources().items():
        assert "hipFuncSetAttribute" not in text or name == "luna_kernels.hpp", name
    src, exe = tmp_path / "allow_lds.cpp", tmp_path / "allow_lds"
    src.write_text(ALLOW_LDS)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include", str(src), "-o",
                    str(exe)], check=True)
    p = subprocess.run([str(exe)], capture_output=True, text=True)
    assert p.returncode == 0, p.stdout
