"""What the compiler made of the FP32 force and jerk kernels, read from the library built
here: properties that a run cannot show, or shows only as lost time."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIBPATH = os.path.join(ROOT, "paper_1406_4254_amd", "libetics.so")
LLVM = os.environ.get("ETICS_LLVM", "/opt/rocm/llvm/bin")

pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-objdump")),
                                reason="needs ROCm's llvm-objdump")


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects of the library, extracted into a folder of their own."""
    if not os.path.exists(LIBPATH):
        from paper_1406_4254_amd import build
        build.build()
    d = tmp_path_factory.mktemp("code")
    os.symlink(LIBPATH, d / "lib.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", "lib.so"], cwd=d, check=True,
                   capture_output=True)
    found = sorted(str(p) for p in d.iterdir() if p.name.endswith("gfx950"))
    assert found
    return found


def kernels(path, pattern):
    """Names of a code object's kernels that match."""
    out = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "-s", "--wide", path], check=True,
                         capture_output=True, text=True).stdout
    names = {line.split()[-1] for line in out.splitlines() if " FUNC " in line}
    return sorted(n for n in names if re.search(pattern, n))


def test_coefficient_loads_are_range_checked(code_objects):
    """The FP32 force and jerk kernels ask for coefficients past the last ones and leave the
    answer to the range check of their buffer descriptor, which compares the vector and the
    instruction's offset with the array's size: no load may carry its position in the scalar
    offset, which is not compared."""
    loads = 0
    for path in code_objects:
        names = kernels(path, r"scf_(force|jerk)(_batched)?_kernelIf")
        if not names:
            continue
        out = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", "--mcpu=gfx950",
                              "--disassemble-symbols=" + ",".join(names), path], check=True, capture_output=True,
                             text=True).stdout
        for line in out.splitlines():
            m = re.match(r"\s+buffer_load_\w+ [av]\S+, v\d+, s\[\d+:\d+\], (\S+)(.*)", line)
            if not m:
                assert "buffer_load" not in line, line
                continue
            loads += 1
            assert m.group(1) == "0" and "offen" in m.group(2), line
    assert loads > 1000


# bytes of scratch a lane that the FP32 jerk kernels may use, by lmax bucket (else none): where
# a wavefront more on each SIMD measured faster than the registers it costs
SCRATCH = {"scf_jerk_kernel": {6: 64, 10: 32, 12: 128}, "scf_jerk_batched_kernel": {10: 64, 12: 448}}


def kernel_notes(code_objects, pattern):
    """The compiler's notes on every kernel whose name matches, with the match."""
    for path in code_objects:
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", path], check=True, capture_output=True,
                               text=True).stdout
        for block in re.split(r"\n  - \.", notes):
            m = re.search(r"\.name:\s+_ZN5etics\d+" + pattern, block)
            if m:
                yield m, {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\n", block)}


def test_jerk_kernels_keep_their_registers(code_objects):
    """The FP32 jerk kernels once held most of their values in scratch (1300 bytes a lane at the
    largest cutoffs), which made the single-system call slower than vector FMAs."""
    seen = 0
    for m, note in kernel_notes(code_objects, r"(scf_jerk_kernel|scf_jerk_batched_kernel)IfLi(\d+)E"):
        seen += 1
        assert note["private_segment_fixed_size"] <= SCRATCH[m.group(1)].get(int(m.group(2)), 0), m.group(0)
    assert seen == 14


def test_fp64_jerk_keeps_its_constants(code_objects):
    """The FP64 jerk kernels have no loop over points out of which their constants could be moved
    (they went to vector lanes, up to 1100 of them)."""
    found = list(kernel_notes(code_objects, r"scf_jerk(_batched)?_kernelIdLi\d+E"))
    assert len(found) == 14
    for m, note in found:
        assert note["sgpr_spill_count"] == 0, m.group(0)
