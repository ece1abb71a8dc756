"""What the compiler made of the prefill's kernels, read from the built library: registers, spills and loops over lanes that a
change of their prologue once brought in without any result changing.  CPU only."""
import os
import re
import shutil
import subprocess

import msgpack
import pytest

from paper_2509_18467_amd import build, lawcat

OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects():
    """The gfx950 code objects (ELF images) inside the library, one per translation unit."""
    blob = open(lawcat.LIB_PATH, "rb").read()
    at = blob.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC)
        n, p = int.from_bytes(blob[p:p + 8], "little"), p + 8
        for _ in range(n):
            offset, size, idlen = (int.from_bytes(blob[p + 8 * i:p + 8 * i + 8], "little") for i in range(3))
            if b"gfx950" in blob[p + 24:p + 24 + idlen]:
                yield blob[at + offset:at + offset + size]
            p += 24 + idlen
        at = blob.find(MAGIC, p)


@pytest.fixture(scope="module")
def kernels():
    """Metadata of every kernel, under its demangled name without arguments."""
    found = {}
    for image in code_objects():
        # the note of the code object: name size 7, description size, type 32 (metadata), "AMDGPU"
        m = re.search(rb"\x07\0\0\0(....)\x20\0\0\0AMDGPU\0\0", image, re.S)
        if m is None:
            continue
        meta = msgpack.unpackb(image[m.end():m.end() + int.from_bytes(m.group(1), "little")], strict_map_key=False)
        found.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
    assert found
    return found


def chunk(kernels, d, heads, mode, output=True):
    name = f"gla_chunk_kernelILi{d}ELi{heads}ELi{mode}ELb{int(output)}E"
    one, = [k for n, k in kernels.items() if name in n]
    return one


def launch_lds(d, heads, mode, tmp_path):
    """The LDS that the output pass is launched with, from the header that the launch takes it from."""
    source, program = tmp_path / "lds.hip", tmp_path / "lds"
    source.write_text('#include "gla_chunk_impl.h"\n#include <cstdio>\n'
                      f'int main() {{ printf("%d", lawcat::chunk::Kernel<{d}, {heads}, {mode}, true>::G::kBytes); }}\n')
    subprocess.run([build.HIPCC, "--offload-host-only", "-std=c++17", "-I", build.CSRC, str(source), "-o", str(program)], check=True)
    return int(subprocess.run([str(program)], check=True, capture_output=True, text=True).stdout)


# (modes: 0 = queries and keys as they are, 1 = conv, 2 = conv and 1 + ELU)
@pytest.mark.parametrize("heads", [1, 2])
def test_three_workgroups_a_compute_unit(kernels, heads, tmp_path):
    """Head dim 64, few query heads, no conv: 512 registers a lane of a SIMD, in granules of 8, for three waves, and 160 KB of LDS, in
    pieces of 1280 bytes, for three workgroups."""
    assert chunk(kernels, 64, heads, 0)[".vgpr_count"] <= 168
    assert 3 * -(-launch_lds(64, heads, 0, tmp_path) // 1280) * 1280 <= 160 * 1024


# (three registers at head dim 64 are the price of three workgroups, see three_share)
@pytest.mark.parametrize("d,heads,mode,most", [(128, 1, 0, 0), (128, 1, 1, 0), (128, 1, 2, 0), (128, 2, 0, 0), (128, 2, 1, 0), (128, 2, 2, 0),
                                               (64, 1, 0, 0), (64, 2, 0, 3)])
def test_spills(kernels, d, heads, mode, most):
    assert chunk(kernels, d, heads, mode)[".vgpr_spill_count"] <= most


@pytest.mark.parametrize("heads", [1, 2, 4])
@pytest.mark.parametrize("mode", [1, 2])
def test_two_workgroups_a_compute_unit(kernels, heads, mode):
    """Head dim 128, four waves: half of a lane's 512 registers of a SIMD, no spills (18, from LDS addresses kept over the loop, cost what
    a seventh of the form's gain is)."""
    one, = [k for n, k in kernels.items() if f"gla_wide_kernelILi{heads}ELi{mode}E" in n]
    assert one[".vgpr_count"] <= 256 and one[".vgpr_spill_count"] == 0 and one[".private_segment_fixed_size"] == 0


@pytest.mark.parametrize("heads,most", [(1, 200), (2, 204), (4, 212)])
def test_walk_of_fp32_storage_reads_operands_as_it_uses_them(kernels, heads, most):
    """Head dim 64: none are held in registers ahead of their use, which is the slower way there (203, 217 and 255 registers)."""
    one, = [k for n, k in kernels.items() if f"gla_walk_kernelIfLi64ELi{heads}E" in n]
    assert one[".vgpr_count"] <= most


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_uniform_descriptors(tmp_path):
    """No load of the prefill's kernels looks for lanes with equal descriptors: that takes four v_readfirstlane per load, hundreds a
    kernel where the workgroup's sequence and segment are not known to be uniform, about a dozen otherwise."""
    seen = 0
    for i, image in enumerate(code_objects()):
        if b"gla_chunk_kernel" not in image:
            continue
        path = tmp_path / f"{i}.o"
        path.write_bytes(image)
        text = subprocess.run([OBJDUMP, "-d", str(path)], check=True, capture_output=True, text=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S*gla_(?:chunk|wide)_kernel\S*)>:\n(.*?)(?=^\S|\Z)", text, re.S | re.M):
            seen += 1
            assert body.count("v_readfirstlane_b32") < 40, name
    assert seen >= 30
