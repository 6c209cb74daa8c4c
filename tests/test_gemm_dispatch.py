"""The host's choice of a GEMM kernel, asked through a small program linked
against the built library: which problem lists it accepts for the direct-load
kernels (nothing is launched, no GPU needed)."""
import os
import subprocess

import pytest

from paper_2608_06411_amd import build as B

PROBE = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "internal.h"
using namespace mapk;

// K ksplit kchunk offset: one bf16 problem of 300 x 200 whose B starts `offset` bytes past a 16-byte boundary.
// cosine B N D: which kernel takes the upper triangle of B cosine matrices.
int main(int argc, char** argv) {
  if (argc == 5 && !strcmp(argv[1], "cosine")) {
    GemmBatch g;
    memset(&g, 0, sizeof(g));
    GemmProblem& p = g.p[0];
    p.batch = atoi(argv[2]);
    p.M = p.N = p.ldc = atoi(argv[3]);
    p.K = p.lda = p.ldb = atoi(argv[4]);
    p.strideA = p.strideB = (long long)p.N * p.K;
    p.epi = EPI_COSINE;
    p.triangular = 1;
    p.A = p.B = reinterpret_cast<const void*>(0x10000);
    g.count = 1;
    gemm_finalize(g);
    const char* name = "staged";
    if (gemm_big_tiles(MAP_BF16, g)) name = "big";
    else if (gemm_small_tiles(MAP_BF16, g)) name = "small";
    else if (gemm_direct_loads(MAP_BF16, g)) name = "128";
    printf("%s\n", name);
    return 0;
  }
  for (int i = 1; i + 3 < argc; i += 4) {
    GemmBatch g;
    memset(&g, 0, sizeof(g));
    GemmProblem& p = g.p[0];
    p.M = 300;
    p.N = 200;
    p.K = p.lda = p.ldb = atoi(argv[i]);
    p.ldc = 200;
    p.batch = 1;
    p.ksplit = atoi(argv[i + 1]);
    p.kchunk = atoi(argv[i + 2]);
    p.epi = p.ksplit > 1 ? EPI_PARTIAL : EPI_BIAS;
    p.A = reinterpret_cast<const void*>(0x10000);
    p.B = reinterpret_cast<const void*>(0x20000 + atoi(argv[i + 3]));
    p.C = reinterpret_cast<void*>(0x30000);
    g.count = 1;
    gemm_finalize(g);
    printf("%d\n", gemm_direct_loads(MAP_BF16, g) ? 1 : 0);
  }
}
"""


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    if not os.path.exists(B.LIB):
        pytest.fail("libmap.so is not built (run python -m paper_2608_06411_amd.build)")
    d = tmp_path_factory.mktemp("probe")
    src, exe = str(d / "probe.cpp"), str(d / "probe")
    with open(src, "w") as f:
        f.write(PROBE)
    subprocess.run([B.hipcc(), "-std=c++17", "-I", B.INCLUDE, "-I", B.CSRC, "-x", "hip", "--offload-host-only", src,
                    "-x", "none", B.LIB, f"-Wl,-rpath,{os.path.dirname(B.LIB)}", "-o", exe], check=True, capture_output=True)
    return lambda *args: subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True).stdout.split()


@pytest.fixture(scope="module")
def direct_loads(probe):
    return lambda *problems: [v == "1" for v in probe(*[v for p in problems for v in p])]


@pytest.mark.parametrize("B,N,D,kernel", [
    (16, 1000, 256, "big"), (20, 769, 512, "big"), (16, 1000, 1152, "big"),
    (1, 65, 256, "small"), (3, 33, 512, "small"), (2, 128, 768, "small"), (1, 1408, 256, "small"), (3, 700, 320, "small"),
    (1, 1409, 256, "128"), (1, 1500, 1088, "128"), (2, 1500, 1152, "128"), (1, 1500, 320, "128"), (1, 1500, 640, "128"),
    (2, 1500, 192, "staged"),
])
def test_cosine_sizes_reach_their_kernel(probe, B, N, D, kernel):
    """The sizes that the GPU tests take for each kernel's edges run there (on
    256 compute units, what the host assumes without a GPU)."""
    assert probe("cosine", B, N, D) == [kernel]


def test_k_ranges(direct_loads):
    """A split product runs on direct loads only if every K range has the four
    slices of 64 that the kernel loads before its first step; a shorter last
    range would be read past its rows."""
    cases = [(K, ks, chunk, 0) for K in range(256, 2049, 64) for chunk in (256, 512, 768) for ks in (2, 3, 4, 5)]
    got = direct_loads(*cases)
    for (K, ks, chunk, _), ok in zip(cases, got):
        assert ok == (K - (ks - 1) * chunk >= 256), (K, ks, chunk)
    cases = [(K, ks, 0, 0) for K in range(256, 2049, 64) for ks in (1, 2, 3, 4)]
    for (K, ks, _, _), ok in zip(cases, direct_loads(*cases)):
        assert ok == (ks == 1 or K % (256 * ks) == 0), (K, ks)


def test_slices_and_alignment(direct_loads):
    assert direct_loads((192, 1, 0, 0), (256, 1, 0, 0), (320, 1, 0, 0), (328, 1, 0, 0)) == [False, True, True, False]
    assert direct_loads((512, 1, 0, 2), (512, 1, 0, 8), (512, 2, 256, 2), (512, 1, 0, 16)) == [False, False, False, True]
