"""What the compiler made of the kernels: instructions this GPU does not run as the compiler means them.

`v_subrev_u32_dpp d, a, b` is meant as b - moved(a).  The GPU returns moved(b) - a: the move across lanes
goes to the operand that a reversed instruction takes first.  The compiler makes it from any x - moved(y).
"""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = "/opt/rocm/llvm/bin"
REVERSED_MOVE = re.compile(r"\bv_\w*rev_\w*_dpp\b")


def device_objects(fatbin: bytes):
    """The gfx950 code objects of a .hip_fatbin section: offload bundles one behind the other."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = fatbin.find(magic)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", fatbin, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", fatbin, p)
            name = fatbin[p + 24:p + 24 + n].decode()
            p += 24 + n
            if name.endswith("gfx950") and size:
                yield fatbin[at + offset:at + offset + size]
        at = fatbin.find(magic, at + len(magic))


def disassembled(elf: str, tmp) -> str:
    section = str(tmp / "fatbin")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={section}", elf,
                    str(tmp / "rest")], check=True, capture_output=True)
    text = []
    for i, code in enumerate(device_objects(open(section, "rb").read())):
        obj = tmp / f"code{i}.o"
        obj.write_bytes(code)
        text.append(subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", str(obj)],
                                   check=True, capture_output=True, text=True).stdout)
    return "\n".join(text)


def test_no_lane_move_inside_a_reversed_instruction(tmp_path):
    from paper_2604_00317_amd import binding as B
    B.load_library()
    text = disassembled(B.LIB_PATH, tmp_path)
    assert text.count("s_endpgm") > 100 and "v_sub_u32_dpp" in text      # the kernels are there
    assert REVERSED_MOVE.findall(text) == []


def test_words_between_patches_reach_the_l2_or_pass_it(tmp_path):
    """What is stored for readers on the same XCD is written through to its L2 (sc0), what others read goes
    past it (sc1), loads go past the L1 (sc1); a second store to a place leaves the first one alone."""
    from paper_2604_00317_amd import build
    src = tmp_path / "probe.hip"
    src.write_text('#include "patch_kernel.hpp"\n'
                   "using namespace nimble::patch;\n"
                   "__global__ void near_words(double *o, double a, double b) "
                   "{ put_word(o, a, 0u, true); put_word(o, b, 1u, true); }\n"
                   "__global__ void far_words(double *o, double a, double b) "
                   "{ put_word(o, a, 0u); put_word(o, b, 1u); }\n"
                   "__global__ void reads(double *o, unsigned long long *r) { *r = get_word(o); }\n")
    r = subprocess.run(["/opt/rocm/bin/hipcc", *build.FLAGS, f"-I{build.CSRC}", "-S",
                        "--cuda-device-only", "-o", "-", str(src)], check=True,
                       capture_output=True, text=True)
    code = {}
    for name in ("near_words", "far_words", "reads"):
        body = re.search(rf"^_Z\d+{name}\w*:(.*?)s_endpgm", r.stdout, re.M | re.S).group(1)
        code[name] = [line.split() for line in body.splitlines() if "global_" in line]
    assert [(c[0], c[-1]) for c in code["near_words"]] == [("global_store_dwordx2", "sc0")] * 2
    assert [(c[0], c[-1]) for c in code["far_words"]] == [("global_store_dwordx2", "sc1")] * 2
    assert (code["reads"][0][0], code["reads"][0][-1]) == ("global_load_dwordx2", "sc1")


@pytest.mark.parametrize("expr,bad", [("nimble::dpp_less_i32<0x121>(v, x)", False),
                                      ("x - nimble::dpp_i32<0x121>(v)", True)])
def test_the_subtraction_helper_keeps_the_move_in_front(tmp_path, expr, bad):
    """The helper's form, and the one that the check above is there to find."""
    from paper_2604_00317_amd import build
    src = tmp_path / "probe.hip"
    src.write_text('#include "wave_ops.hpp"\n'
                   "__global__ void k(int *o) { int v = o[threadIdx.x], x = o[64 + threadIdx.x];\n"
                   f"  o[threadIdx.x] = {expr}; }}\n")
    r = subprocess.run(["/opt/rocm/bin/hipcc", *build.FLAGS, f"-I{build.CSRC}", "-S",
                        "--cuda-device-only", "-o", "-", str(src)], check=True,
                       capture_output=True, text=True)
    assert bool(REVERSED_MOVE.search(r.stdout)) == bad
