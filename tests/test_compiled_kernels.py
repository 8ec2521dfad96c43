"""What the compiler made of the kernels: registers and scratch memory from the notes in the built library's code objects
(host-only, no GPU needed).  Plans count on so many workgroups per compute unit, and no test of results sees that fewer fit."""
import struct
import subprocess

import pytest

from paper_1912_05234_amd import binding
from paper_1912_05234_amd import build

msgpack = pytest.importorskip("msgpack")
REGISTERS = 512  # of a SIMD's lane, shared by its waves in groups of eight


def notes(elf):
    """Contents of the AMDGPU metadata notes of a code object."""
    assert elf[:4] == b"\x7fELF"
    offset, size, count = struct.unpack_from("<Q", elf, 0x28)[0], *struct.unpack_from("<HH", elf, 0x3A)
    for k in range(count):
        kind, at, length = struct.unpack_from("<4xI16xQQ", elf, offset + k * size)
        end = at + length
        while kind == 7 and at < end:  # SHT_NOTE
            name, desc, tag = struct.unpack_from("<III", elf, at)
            body = at + 12 + (name + 3) // 4 * 4
            if tag == 32:  # NT_AMDGPU_METADATA
                yield msgpack.unpackb(elf[body:body + desc])
            at = body + (desc + 3) // 4 * 4


def kernels():
    """{demangled name without arguments: its metadata} of every kernel in the library."""
    binding.lib()
    blob, magic, found = open(build.LIB, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", []
    at = blob.find(magic)
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", blob, at + 24)[0]):
            start, size, length = struct.unpack_from("<QQQ", blob, entry)
            target = blob[entry + 24:entry + 24 + length]
            if size and b"gfx950" in target:
                for note in notes(blob[at + start:at + start + size]):
                    found += note["amdhsa.kernels"]
            entry += 24 + length
        at = blob.find(magic, at + 1)
    plain = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True, check=True)
    names = [n.replace("(anonymous namespace)::", "").split("(")[0].removeprefix("void ") for n in plain.stdout.splitlines()]
    return dict(zip(names, found))


KERNELS = kernels()


def form(name):
    """Template arguments of a kernel as numbers."""
    return [int(v) if v.isdigit() else v == "true" for v in name[name.index("<") + 1:-1].split(", ")]


def resident(kernel):
    """Workgroups of four waves that a compute unit's registers hold."""
    return REGISTERS // (-(-kernel[".vgpr_count"] // 8) * 8)


WGRAD = sorted(n for n in KERNELS if n.startswith("cnn::tile::wgrad_kernel<"))


def test_every_form_of_the_weight_gradient_is_there():
    assert len(WGRAD) >= 40


@pytest.mark.parametrize("name", WGRAD)
def test_weight_gradient_forms_fit_as_often_as_plans_count_on(name):
    """512 / (4 nt mt + 3 nt + 60) workgroups, at most four (cnn_ops.hip), four registers a row tile more with rounded operands.
    Before the bound on the registers eight and six tap tiles of two row tiles held one workgroup less than that, and calls
    planned for three ran a second turn: 9770 images 2 -> 23, 8 x 21, 7 x 7 42 -> 55 us."""
    nt, mt, rounded, _ = form(name)
    wanted = min(4, REGISTERS // (4 * nt * mt + 3 * nt + 60 + 4 * mt * rounded))
    assert resident(KERNELS[name]) >= wanted
    assert KERNELS[name][".private_segment_fixed_size"] == 0, "scratch memory"


@pytest.mark.parametrize("name", ["train_epoch_kernel", "train_group_kernel<false>", "train_group_kernel<true>", "train_kernel<true>",
                                  "forward_group_kernel<false>", "forward_kernel<false>", "reduce_update_kernel<32>"])
def test_kernels_of_the_network_keep_everything_in_registers(name):
    """(train_kernel<false> does not: three registers, 16 bytes, accounted for in its measured traffic.)  The device-side epoch loop
    held thirty weights of the output layer in registers from its table loads on, and spilled seven."""
    assert KERNELS[name][".private_segment_fixed_size"] == 0 and KERNELS[name][".vgpr_spill_count"] == 0
