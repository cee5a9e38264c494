"""What the compiler made of kernels whose speed hangs on it: read from the code objects of the built library.  Runs without a GPU."""
import os
import re
import struct
import subprocess

import pytest

from paper_2507_00217_amd import build

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The library's gfx950 code objects, one per translation unit with kernels, as files."""
    if not os.path.exists(build.LIB):
        build.build(verbose=False)
    blob, d, paths, at = open(build.LIB, "rb").read(), tmp_path_factory.mktemp("co"), [], 0
    while (at := blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        n, p = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", blob, p)
            if blob[p + 24:p + 24 + tlen].endswith(b"gfx950") and size:
                paths.append(d / f"{len(paths)}.co")
                paths[-1].write_bytes(blob[at + off:at + off + size])
            p += 24 + tlen
        at += 24
    assert paths
    return paths


@pytest.fixture(scope="module")
def resources(code_objects):
    """kernel -> {vgpr_count, vgpr_spill_count, private_segment_fixed_size}"""
    out = {}
    for path in code_objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in text.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel)[1]
            out[name] = {k: int(re.search(rf"\.{k}:\s+(\d+)", kernel)[1]) for k in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size")}
    return out


def test_two_forward_workgroups_of_head_dim_64_fit_a_compute_unit(resources):
    """8 wavefronts each, so four to a SIMD: 512 / 4 registers, none spilled."""
    found = {n: r for n, r in resources.items() if re.search(r"attn_fwd_kernelILi64ELi512E", n)}
    assert len(found) == 2, sorted(resources)
    for n, r in found.items():
        assert r["vgpr_count"] <= 128 and r["vgpr_spill_count"] == 0 and r["private_segment_fixed_size"] == 0, (n, r)


def test_two_column_sum_workgroups_fit_a_compute_unit(resources):
    """16 wavefronts each, so eight to a SIMD: 512 / 8 registers."""
    (found,) = [r for n, r in resources.items() if "col_sum_kernel" in n]
    assert found["vgpr_count"] <= 64


def test_loading_wavefronts_wait_by_count(code_objects):
    """The loops of the wavefronts that only load (loads to LDS and a barrier, no MFMA): the one wait for loads in them is the counted one
    that leaves later tiles outstanding."""
    seen = 0
    for path in code_objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        for func in re.split(r"\n(?=[0-9a-f]{16} <)", text):
            name = re.search(r"<(\S+)>:", func)
            if not name or not re.search(r"gemm_(quarter|tiny|mid|wgrad_small)_kernel", name[1]):
                continue
            code = [(int(a, 16), i.strip()) for i, a in re.findall(r"^\s+(.+?)\s*// ([0-9A-F]+):", func, re.M)]
            at, loops = {a: n for n, (a, _) in enumerate(code)}, []
            for n, (a, ins) in enumerate(code):
                jump = re.match(r"s_(?:cbranch_\w+|branch) (\d+)", ins)
                if jump and int(jump[1]) >= 1 << 15:                              # a 16-bit count of words, negative: back
                    first = at[a + 4 + 4 * (int(jump[1]) - (1 << 16))]
                    body = [x for _, x in code[first:n]]
                    if any(x.startswith("buffer_load") and x.endswith("lds") for x in body) and any(x == "s_barrier" for x in body):
                        loops.append(body)
            if not loops:
                continue
            body = min(loops, key=len)
            if any(x.startswith("v_mfma") for x in body):                         # its own wavefronts load: no such loop
                continue
            waits = [x for x in body if x.startswith("s_waitcnt") and "vmcnt" in x]
            assert len(waits) == 1 and re.search(r"vmcnt\([1-9]", waits[0]), (name[1], waits)
            seen += 1
    assert seen >= 30


# (kernel's tile, loads of one K tile per thread that loads, K tiles ahead)
RINGS = [(r"gemm_quarter_kernelILb[01]ELi\dELi4ELi4E", 8, 4), (r"gemm_tiny_kernelILb[01]ELi\dELi0ELi4E", 4, 8), (r"gemm_tiny_kernelILb[01]ELi\dELi1ELi4E", 6, 4),
         (r"gemm_mid_kernelILb[01]ELi\dELi0E", 5, 4), (r"gemm_mid_kernelILb[01]ELi\dELi[12]E", 10, 2), (r"gemm_mid_kernelILb[01]ELi\dELi3E", 3, 8)]


@pytest.mark.parametrize("kernel,loads,ahead", RINGS)
def test_a_short_reduction_starts_with_its_first_tile(code_objects, kernel, loads, ahead):
    """A reduction of no more K tiles than the ring holds ahead is loaded whole before the first barrier; that waits for the first tile only: of
    `ahead` tiles all but one may be outstanding (a count that no other wait of the loading wavefronts has), and so for fewer tiles."""
    found = 0
    for path in code_objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True, check=True).stdout
        for func in re.split(r"\n(?=[0-9a-f]{16} <)", text):
            name = re.search(r"<(\S+)>:", func)
            if name and re.search(kernel, name[1]):
                waits = {int(n) for n in re.findall(r"s_waitcnt vmcnt\((\d+)\)", func)}
                assert waits >= {n * loads for n in range(1, ahead)}, (name[1], sorted(waits))
                found += 1
    assert found
