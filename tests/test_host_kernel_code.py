"""What the compiler made of the kernels: the gfx950 code in the built library, read with the
toolchain's own tools.  No GPU."""
import os
import re
import struct
import subprocess

import pytest

from paper_2005_05758_amd import build

LLVM = "/opt/rocm/llvm/bin/"
pytestmark = pytest.mark.skipif(not os.path.exists(LLVM + "llvm-readelf"), reason="no LLVM tools")


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """Paths of the gfx950 code objects bundled in the library, one per source file."""
    if not os.path.exists(build.LIB):
        build.build()
    d = tmp_path_factory.mktemp("code")
    fat = str(d / "fat.bin")
    subprocess.run(["objcopy", "--dump-section", ".hip_fatbin=" + fat, build.LIB, str(d / "copy.so")], check=True)
    data = open(fat, "rb").read()
    magic, paths = b"__CLANG_OFFLOAD_BUNDLE__", []
    for at in (m.start() for m in re.finditer(magic, data)):
        pos = at + len(magic)
        n, = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + length].decode()
            pos += 24 + length
            if triple.startswith("hip") and size:
                assert "gfx950" in triple
                paths.append(str(d / f"{len(paths)}.co"))
                with open(paths[-1], "wb") as f:
                    f.write(data[at + off:at + off + size])
    assert paths
    return paths


def _demangled(names):
    out = subprocess.run(["c++filt"], input="\n".join(names), text=True, stdout=subprocess.PIPE, check=True).stdout.split("\n")
    return [re.sub(r"\(.*", "", o).replace("void csb::", "") for o in out[:len(names)]]


def _notes(paths):
    """{kernel: (bytes of scratch per lane, vector registers)}"""
    found = []
    for p in paths:
        text = subprocess.run([LLVM + "llvm-readelf", "--notes", p], text=True, stdout=subprocess.PIPE, check=True).stdout
        for entry in re.split(r"\n  - \.", text)[1:]:
            name = re.search(r"\.?name: +(_Z\S+)", entry)
            numbers = [re.search(r"\." + k + r": +(\d+)", entry) for k in ("private_segment_fixed_size", "vgpr_count")]
            if name and all(numbers):
                found.append((name.group(1), tuple(int(n.group(1)) for n in numbers)))
    return dict(zip(_demangled([n for n, _ in found]), [v for _, v in found]))


def test_batched_products_use_no_scratch(code_objects):
    """The loops of the batched products count the loads in flight: a spilled register is one more."""
    scratch = {k: v[0] for k, v in _notes(code_objects).items() if k.startswith("spmm_")}
    assert sum(k.startswith("spmm_reg_multi_kernel<true, 16, 2") for k in scratch) == 3      # the widest two-source forms
    assert {k: s for k, s in scratch.items() if s} == {}


def test_16_row_products_of_16_bit_leave_room_for_two_workgroups(code_objects):
    """Two workgroups of 16 wavefronts share a CU where a wavefront takes at most 64 of the 512 registers
    of a lane: the products of 16 rows by 64 right-hand sides in 16 bits."""
    registers = {k: v[1] for k, v in _notes(code_objects).items() if re.match(r"spmm_reg16_kernel<16, 1, [12], 1>", k)}
    assert len(registers) == 2 and all(v <= 64 for v in registers.values()), registers


@pytest.fixture(scope="module")
def code(code_objects):
    """{kernel: its instructions}"""
    found = {}
    for p in code_objects:
        text = subprocess.run([LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", p], text=True, stdout=subprocess.PIPE, check=True).stdout
        parts = re.split(r"\n[0-9a-f]+ <(\S+)>:\n", text)
        found.update(zip(_demangled(parts[1::2]), parts[2::2]))
    return found


def test_several_products_per_launch_load_no_arguments_per_lane(code):
    """The kernels that take several products find a product's pointers and strides among their
    arguments; a lane that chooses between two sources must choose between registers.  Their loads
    are those of the kernel that takes one product."""
    loads = {k: len(re.findall(r"\t(?:global|flat|buffer)_load_", c)) for k, c in code.items() if re.match(r"spmm_(reg_)?(multi_)?kernel<", k)}
    multi = [k for k in loads if "multi_" in k]
    assert len(multi) == len(loads) - len(multi) == 56              # 20 of the general form, 36 of the register form
    assert {k: loads[k] for k in multi if loads[k] != loads[k.replace("multi_", "")]} == {}


def test_input_offsets_are_unsigned(code):
    """A batched product's input may be 4 GiB long: the byte offset of a row, a 24-bit product, is
    neither extended with its sign nor shifted as a signed number."""
    wrong = {}
    for k, c in code.items():
        if not k.startswith("spmm_"):
            continue
        products = set()
        for line in c.split("\n"):
            arith = re.match(r"\tv_ashrrev_i32\w* v\d+, \d+, (v\d+)", line)
            if arith and arith.group(1) in products:
                wrong[k] = wrong.get(k, 0) + 1
            written = re.match(r"\t(?:v|global|buffer|ds)_\w+ (v\d+),", line)
            if written:
                (products.add if line.startswith("\tv_mul_u32_u24") else products.discard)(written.group(1))
    assert sum(k.startswith("spmm_") for k in code) > 90 and wrong == {}
