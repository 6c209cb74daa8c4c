"""What the compiled device code has to hold whatever order the compiler
finds for it, read from the assembly that hipcc writes for gfx950 (built here,
no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2608_06411_amd import build as B


@pytest.fixture(scope="module")
def gemm_asm(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "gemm.s")
    flags = [f for f in B.COMMON if f != "-fPIC"]
    subprocess.run([B.hipcc(), *flags, *B.DEVICE_FLAGS, "-x", "hip", "--cuda-device-only", "-S",
                    os.path.join(B.CSRC, "gemm.hip"), "-o", out], check=True, capture_output=True)
    return open(out).read()


def _blocks(asm, kernel):
    """The kernel's basic blocks as lists of lines."""
    body = re.search(rf"^{kernel}:.*?^\.Lfunc_end", asm, re.M | re.S).group(0)
    return [b.splitlines() for b in re.split(r"^\.LBB\w+:", body, flags=re.M)]


def test_row_norm_reads_are_waited_for(gemm_asm):
    """The row norms read half-tiles of A that the next phase's direct loads
    overwrite, so every such read is followed, in its own block and before
    any barrier, by a wait that the source states (between the assembler's
    inline-asm marks), not one that only the use of its value brings."""
    kernel = r"_ZN4mapk12_GLOBAL__N_115gemm_big_kernelILb1ELi256EEEvNS_9GemmBatchE"
    seen = 0
    for block in _blocks(gemm_asm, kernel):
        reads = [i for i, x in enumerate(block) if "ds_read_b128" in x]
        squares = [i for i, x in enumerate(block) if re.search(r"v_fma\w*_f32\w*\s+(v\d+), (v\d+), \2\b", x)]
        if not reads or not squares or any("mfma" in x for x in block):
            continue
        inline = False
        waited = None
        for i, x in enumerate(block[reads[0]:]):
            inline = inline and "#ASMEND" not in x or "#ASMSTART" in x
            if "s_barrier" in x:
                break
            if inline and "lgkmcnt(0)" in x:
                waited = reads[0] + i
        assert waited is not None and waited > reads[-1], "\n".join(block)
        seen += 1
    assert seen >= 4  # two blocks of rows in each half of A at least
