"""What the compiler made of the kernels: registers and scratch memory, read from the metadata of the built library.

No kernel may spill vector registers.  The persistent kernels are written to fit their budget (128 registers in the
16-wave forms) exactly, and a change that costs them one register shows nowhere else: the results stay right, and the
spilled value, often a weight that has just been requested, is waited for in every phase."""
import os
import re
import struct
import subprocess

import pytest

import paper_2306_16601_amd as sp
from paper_2306_16601_amd import build as B

msgpack = pytest.importorskip("msgpack")


def _code_objects(path):
    """The gfx950 ELF images in the library's offload bundles (one bundle per translation unit)."""
    data, magic = open(path, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length] and size:
                yield data[at + offset:at + offset + size]
            p += 24 + length
        at = data.find(magic, at + 24)


def _kernels(elf):
    """Kernel descriptions of the AMDGPU metadata note (type 32)."""
    table, = struct.unpack_from("<Q", elf, 40)
    entry, sections = struct.unpack_from("<HH", elf, 58)
    for k in range(sections):
        at = table + k * entry
        kind, = struct.unpack_from("<I", elf, at + 4)
        p, size = struct.unpack_from("<QQ", elf, at + 24)
        end = p + size
        while kind == 7 and p < end:
            name, desc, note = struct.unpack_from("<III", elf, p)
            p += 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[p:p + desc]).get("amdhsa.kernels", [])
            p += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    sp.lib()
    return [k for elf in _code_objects(sp.binding.LIB_PATH) for k in _kernels(elf) if "rowtile" in k[".name"]]


def test_no_kernel_spills_vector_registers(kernels):
    assert len(kernels) > 400
    spilled = {k[".name"]: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in kernels
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled, spilled


def test_the_base_name_is_that_of_every_kernel(kernels):
    """A profiler's filter on spmm_kernel_name() shows all that spmm_run launches, and nothing else of the library."""
    name = sp.spmm_kernel_name()
    assert all(re.match(r"_ZN4spmm\d+" + name, k[".name"]) for k in kernels)
    others = [k[".name"] for elf in _code_objects(sp.binding.LIB_PATH) for k in _kernels(elf) if "rowtile" not in k[".name"]]
    assert others and not any(name in n for n in others)


def test_resident_kernels_leave_room_for_a_second_workgroup(kernels):
    """128 registers: two workgroups of 8 waves on a CU, with Sum and without.  (Pairs of row tiles, R = 2: one.)"""
    seen = 0
    for k in kernels:
        m = re.search(r"simpleILi(\d+)ELi8ELi1ELi\d+ELi(\d+)E", k[".name"])
        if m:
            seen += 1
            assert k[".vgpr_count"] <= 128, k[".name"]
    assert seen == 33


HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
@pytest.mark.parametrize("waves, slots", [(8, 8), (12, 4), (8, 4)])
def test_weight_requests_of_int32_outputs_wait_for_no_stores(tmp_path, waves, slots):
    """The loader-wave kernels store int32 accumulators as they are, and must not wait for those stores before they
    request the next phase's weights: no more full waits in the code than with binary32 outputs."""
    waits = []
    for out in ("SPMM_OUT_S32", "SPMM_OUT_F32"):
        src, asm = tmp_path / (out + ".hip"), tmp_path / (out + ".s")
        src.write_text('#include "spmm_kernels.h"\nnamespace spmm { template __global__ void spmm_rowtile_mfma_fed<128, %d, 4, %d, %s, 0>'
                       "(const KernelArgs); }\n" % (waves, slots, out))
        subprocess.run([HIPCC, *B.HIPCC_FLAGS, "-x", "hip", "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True,
                       capture_output=True)
        waits.append(len(re.findall(r"s_waitcnt vmcnt\(0\)\s", asm.read_text())))
    assert waits[0] <= waits[1], waits


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
@pytest.mark.parametrize("kernel", ["simple<16, 8, 1", "simple<32, 8, 1", "simple<64, 8, 1", "simple<64, 8, 2", "slab<16, 8"])
def test_a_table_costs_the_resident_kernels_no_loops_over_lanes(tmp_path, kernel):
    """The weights come through a buffer resource, the same in all lanes.  Where the compiler cannot tell, it reads the resource
    lane by lane, in a loop around each load: the kernels with a table must have no more of that than those without, and read
    the bounds that it is made of by scalar loads as they do."""
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text('#include "spmm_kernels.h"\nnamespace spmm {\n' + "".join(
        "template __global__ void spmm_rowtile_mfma_%s, SPMM_OUT_U8, %s>(const KernelArgs);\n" % (kernel, post)
        for post in ("SPMM_POST_NONE", "SPMM_POST_GELU")) + "}\n")
    subprocess.run([HIPCC, *B.HIPCC_FLAGS, "-x", "hip", "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True, capture_output=True)
    plain, table = (re.split(r"^; -- End function|^\s*\.end_amdhsa_kernel", k, flags=re.M)[0]
                    for k in re.split(r"^\s*\.globl\s+_ZN4spmm", asm.read_text(), flags=re.M)[1:3])
    lanes, scalar = ([len(re.findall(op, k)) for k in (plain, table)] for op in (r"\bv_readfirstlane_b32\b", r"\bs_load_dword"))
    assert lanes[1] <= lanes[0] + 8, lanes
    assert scalar[1] >= scalar[0], scalar


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
@pytest.mark.parametrize("kernel, passes", [("simple<16, 8, 1", 4), ("simple<32, 8, 1", 8), ("simple<64, 8, 1", 8), ("slab<16, 8", 8)])
def test_rounds_of_k_request_their_activations_together(tmp_path, kernel, passes):
    """A request for each pass of activation rows where K is resident, and as many for K in rounds (and rows too far apart for one
    32-bit offset), not one that every pass waits for; beside them one where a single pass holds K, and one for rows beyond the
    offsets of a pass.  (The compiler joins the requests that the starts for other numbers of passes share.)"""
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text('#include "spmm_kernels.h"\nnamespace spmm { template __global__ void spmm_rowtile_mfma_%s, SPMM_OUT_S32, 0>'
                   "(const KernelArgs); }\n" % kernel)
    subprocess.run([HIPCC, *B.HIPCC_FLAGS, "-x", "hip", "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True, capture_output=True)
    requests = len(re.findall(r"\bglobal_load_dwordx4\b", asm.read_text()))
    assert requests >= 2 * passes + 2, requests
