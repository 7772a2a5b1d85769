"""Registers of kernels that run at their limit, from the metadata of the
gfx950 code objects in the built library: the two-tile Hamiltonian pass and
the adjoint pass of plans the pair kernel does not take keep their amplitudes
in registers (ten spilled cost a 4x4 product 5%)."""
import os
import struct
import subprocess

import pytest

from paper_2108_13410_amd import build

msgpack = pytest.importorskip("msgpack")


def _code_objects(lib):
    """The gfx950 ELF images of every offload bundle in the library."""
    data = open(lib, "rb").read()
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        if count > 16:  # (the magic as a string constant)
            at += 24
            continue
        for _ in range(count):
            off, size, idl = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + idl]
            p += 24 + idl
            if b"gfx950" in target and size:
                yield data[at + off:at + off + size]
        at = p


def _kernels(elf):
    """Kernel records of the AMDGPU metadata note of an ELF image."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    entsize, num = struct.unpack_from("<HH", elf, 58)
    for i in range(num):
        kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
        if kind != 7:  # SHT_NOTE
            continue
        off, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 24)
        end = off + size
        while off < end:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, off)
            desc = off + 12 + (namesz + 3) // 4 * 4
            if ntype == 32:  # NT_AMDGPU_METADATA
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            off = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(build.LIB):
        build.build()
    recs = [k for elf in _code_objects(build.LIB) for k in _kernels(elf)]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in recs), capture_output=True, text=True,
                           check=True).stdout.split("\n")
    short = [n.replace("z2h::", "").replace("(anonymous namespace)::", "").replace("void ", "") for n in names]
    out = {n.split("(")[0]: k for n, k in zip(short, recs)}
    assert len(out) > 100
    return out


@pytest.mark.parametrize("split,limit", [("false", 0), ("true", 2)])
def test_hamiltonian_two_tiles_in_registers(kernels, split, limit):
    assert kernels[f"ham_kernel<double, 4, true, {split}>"][".vgpr_spill_count"] <= limit


@pytest.mark.parametrize("R,NL", [(3, 1), (3, 2), (3, 3), (3, 4), (4, 1), (4, 2), (4, 3)])
def test_adjoint_in_registers(kernels, R, NL):
    k = kernels[f"adj_kernel<double, {R}, {NL}>"]
    assert k[".vgpr_spill_count"] == 0
    assert k[".vgpr_count"] <= (128 if R == 3 else 256)  # four waves a SIMD, two


def test_one_workgroup_states_share_a_cu(kernels):
    """12 qubits, four waves a workgroup: two workgroups a CU (their LDS is
    checked where it is laid out)."""
    for real, ex in (("float", 2), ("double", 1)):
        k = kernels[f"resident_kernel<Shape<4, 2, 0, 11>, {real}, {ex}>"]
        assert k[".vgpr_count"] + k.get(".agpr_count", 0) <= 256


def test_small_state_gates_apart():
    """The tile pass of large circuits alone with its own kind: beside the
    small states' kernel, the same instructions took 3% to 4% longer."""
    objs = [elf for elf in _code_objects(build.LIB) if any("fused_kernel" in k[".name"] for k in _kernels(elf))]
    assert len(objs) == 1 and not any("fine_kernel" in k[".name"] for k in _kernels(objs[0]))
