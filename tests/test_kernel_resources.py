"""Wavefronts that fit a SIMD beside each other, from the register counts in the
built library's kernel metadata (CPU only): a SIMD of gfx950 has 512 vector
registers a lane, handed out in eights, to at most eight waves."""
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


def waves(vgprs: int) -> int:
    return min(8, 512 // (-(-vgprs // 8) * 8))


@pytest.fixture(scope="module")
def vgprs(tmp_path_factory):
    """Vector registers of every kernel of the library, by demangled name."""
    from paper_1810_11685_amd import build as B
    if shutil.which("c++filt") is None or not all(os.path.exists(f"{LLVM}/{t}") for t in ("llvm-objcopy", "llvm-readelf")):
        pytest.skip("LLVM tools not found")
    if not os.path.exists(B.LIB):
        pytest.skip("library not built")
    d = tmp_path_factory.mktemp("fatbin")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={d}/fat", B.LIB, f"{d}/rest"], check=True)
    data = (d / "fat").read_bytes()
    at = [m.start() for m in re.finditer(b"\x7fELF", data)] + [len(data)]
    counts = {}
    for k in range(len(at) - 1):
        (d / "elf").write_bytes(data[at[k]:at[k + 1]])
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", f"{d}/elf"], capture_output=True, text=True).stdout
        for m in re.finditer(r"\.symbol:\s+(\S+)\.kd.*?\.vgpr_count:\s+(\d+)", notes, re.S):
            counts[m[1]] = int(m[2])
    names = subprocess.run(["c++filt"], input="\n".join(counts), capture_output=True, text=True).stdout
    out = dict(zip(names.split("\n"), counts.values()))
    assert len(out) == len(counts) > 100
    return out


def test_kernels_for_several_lengths_keep_their_waves(vgprs):
    """The pass kernels without a length of their own (launches over several
    lengths, and grids of 8 to 24 points): the radix 6 and 12 stages of the
    longer lengths do not set their register count."""
    # row modes by number: 0 F1, 1 F2, 2 F2L, 3 F3, 4 A1, 6 A2, 7 A3; 8, 9: one field in, out
    seen = 0
    for name, v in vgprs.items():
        m = re.match(r"void qpat::(row|col)_kernel<(\d+|true|false), (\d+|true|false), 0, false>", name)
        if not m:
            continue
        if m[1] == "col":
            least = 5
        else:
            mode = int(m[2])
            least = 8 if mode in (8, 9) else 4 if mode in (0, 1, 2, 3, 4, 6, 7) else None
        if least:
            seen += 1
            assert waves(v) >= least, (name, v)
    assert seen == 12 + 2 * 9


def test_no_kernels_that_no_launch_takes(vgprs):
    """Fused row kernels on global twiddles exist for the plans with radix-8 ends
    alone: with radix-4 ends (48, 96, 128, 1024) the launch refuses them."""
    fused = {m[1] for n in vgprs if (m := re.match(r"void qpat::row_kernel<(?:33|38), true, (\d+), true>", n))}
    assert fused == {"64", "192", "256", "384", "512", "768"}
