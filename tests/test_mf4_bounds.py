"""The matrix-core helper refuses a chunk past the operand's blocks, or an
operator column past its last, when the kernel is compiled; before, the
products were left out and the accumulator returned as it was."""

import os
import subprocess

import pytest

from paper_2401_06132_amd import build

SOURCE = """
#include "mf4.h"
extern "C" __global__ void k(float* o, const float* i) {
  fr::mf4v c = {0, 0, 0, 0}, d[2] = {c, c};
#pragma unroll
  for (int j = 0; j < 4; ++j) c = fr::mf4<%d>(i[threadIdx.x], i[64 + j], c, j + %d);
  fr::Mf4Op<2, 6> op;
  op.load(i, threadIdx.x);
  op.col(%d, i[threadIdx.x], d);
  o[threadIdx.x] = c[0] + d[0][1] + d[1][2];
}
"""


@pytest.mark.parametrize("cbsz,first,col,ok", [(4, 12, 5, True), (4, 13, 5, False), (3, 4, 0, True), (3, 5, 0, False),
                                               (3, 0, 6, False), (4, -1, 0, False)])
def test_chunk_bounds(tmp_path, cbsz, first, col, ok):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src = tmp_path / "k.hip"
    src.write_text(SOURCE % (cbsz, first, col))
    r = subprocess.run([build.HIPCC] + build.COMMON + build.DEVICE + ["--cuda-device-only", "-c", str(src), "-o",
                                                                     str(tmp_path / "k.o")], capture_output=True, text=True)
    assert (r.returncode == 0) == ok, r.stderr
    assert ok or "mf4: the chunk" in r.stderr, r.stderr
