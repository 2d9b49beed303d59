"""Rules that the kernel sources keep, checked without a GPU."""
import os
import re

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
