"""Segments of the two-level binning's pair lists at the end of the 32-bit range:
the pairs that the kernels' steps of 64 take are each segment's own, and every
walk ends.  (The bounds are a host function too: a small host program prints
them.)"""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]

PROGRAM = """
#include "nxs_internal.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4) {
    auto u = [&](int k) { return (uint32_t)strtoul(argv[i + k], nullptr, 10); };
    const nxs::PairRange r = nxs::segment_pairs(u(0), u(1), u(2), u(3));
    printf("%u %u\\n", r.first, r.n);
  }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    hipcc = shutil.which("hipcc")
    if not hipcc:
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("segments")
    (d / "s.hip").write_text(PROGRAM)
    subprocess.run([hipcc, "-std=c++17", "--offload-host-only", f"-I{ROOT}/include",
                    f"-I{ROOT}/paper_2603_02887_amd/csrc", str(d / "s.hip"), "-o", str(d / "s")],
                   check=True)
    return d / "s"


@pytest.mark.parametrize("shift", [6, 8, 10])
@pytest.mark.parametrize("begin,end", [
    (0, 1), (5, 5 + 1024), (2**32 - 2 - 3000, 2**32 - 2), (2**32 - 2 - 64, 2**32 - 2),
    (2**32 - 1026, 2**32 - 257), (2**31 - 7, 2**31 + 4001)])
def test_every_pair_once(program, begin, end, shift):
    segs = -(-(end - begin) // (1 << shift))
    args = [str(v) for k in range(segs) for v in (begin, end, k, shift)]
    out = subprocess.run([str(program), *args], check=True, capture_output=True, text=True)
    at = begin
    for line in out.stdout.split("\n")[:segs]:
        first, n = map(int, line.split())
        assert first == at and 0 < n <= 1 << shift
        at += n
    assert at == end
