"""What the built kernels take of a compute unit's registers, read from the code
objects of librac.so: no kernel spills to memory, and those whose wavefronts a
SIMD is a matter of their speed keep that number."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

import paper_2608_04991_amd as rac

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> (vector registers, registers spilled to memory)"""
    if not os.path.exists(rac.library_path()):
        pytest.fail("librac.so is not built; run __graft_entry__.build()")
    tmp = str(tmp_path_factory.mktemp("code"))
    run = lambda *a: subprocess.run(a, check=True, capture_output=True, text=True).stdout
    run(f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={tmp}/fat", rac.library_path(), f"{tmp}/rest")
    data = open(f"{tmp}/fat", "rb").read()
    starts = [m.start() for m in re.finditer(MAGIC, data)]
    out = {}
    for i, (a, b) in enumerate(zip(starts, starts[1:] + [len(data)])):
        part = f"{tmp}/{i}"
        open(part, "wb").write(data[a:b])
        run(f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
            f"--input={part}", f"--output={part}.elf")
        for note in run(f"{LLVM}/llvm-readelf", "--notes", part + ".elf").split("  - .agpr_count")[1:]:
            field = lambda k: re.search(rf"\.{k}:\s+(\S+)", note).group(1)
            out[field("name")] = int(field("vgpr_count")), int(field("vgpr_spill_count"))
    plain = subprocess.run(["c++filt"], input="\n".join(out), text=True, capture_output=True, check=True).stdout
    return {re.sub(r"\(anonymous namespace\)::|^void ", "", p).split("(")[0]: v
            for p, v in zip(plain.splitlines(), out.values())}


def waves_per_simd(vgprs: int) -> int:
    return min(8, 512 // (-(-vgprs // 8) * 8))


def test_no_kernel_spills(kernels):
    assert len(kernels) > 200
    assert [n for n, (_, spilled) in kernels.items() if spilled] == []


@pytest.mark.parametrize("pattern,count,waves", [
    # the per-token chunk encode (step tables) at 4 bits: 106 registers, four
    # wavefronts, made 4962 x 2432 with k = 8 take 66 us instead of 40
    (r"rac_encode_kernel<4, [34], [34], 1, false>", 4, 5),
    # a decode holds eight: a resident workgroup's rows are counted on that
    (r"rac_decode_kernel<.*", 24, 8)])
def test_wavefronts_per_simd(kernels, pattern, count, waves):
    hit = {n: v for n, (v, _) in kernels.items() if re.fullmatch(pattern, n)}
    assert len(hit) == count
    assert {n: waves_per_simd(v) for n, v in hit.items()} == dict.fromkeys(hit, waves)
