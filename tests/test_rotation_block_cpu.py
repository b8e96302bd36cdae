"""Rotation layers of the register passes: the assembly made for each number of
register bits works on the elements that a thread has, and on no others. Compiled
here from the kernels' own header; nothing is run.
"""
import re
import subprocess

import pytest

from paper_2011_13524_amd import build as B

SOURCE = """
#include "tile_reg.h"
using namespace qsv;
extern "C" __global__ void layer(%(t)s* p, const cx<%(t)s>* coef, unsigned rot) {
  cx<%(t)s> v[1 << %(rb)d];
  for (int i = 0; i < (1 << %(rb)d); ++i) v[i] = {p[2 * i], p[2 * i + 1]};
  rot_layer<%(t)s, %(rb)d>(v, rot, coef);
  for (int i = 0; i < (1 << %(rb)d); ++i) p[2 * i] = v[i].re, p[2 * i + 1] = v[i].im;
}
"""


@pytest.mark.parametrize("t", ["float", "double"])
@pytest.mark.parametrize("rb", [3, 4, 5])
def test_a_rotation_layer_has_the_products_of_its_elements(t, rb, tmp_path):
    src = tmp_path / "layer.hip"
    src.write_text(SOURCE % {"t": t, "rb": rb})
    out = tmp_path / "layer.s"
    flags = [f for f in B.CFLAGS if f != "-fPIC"]
    subprocess.run([B.HIPCC, *flags, "-I" + B.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True,
                   capture_output=True, timeout=300)
    # per register bit and axis (X, Y), three products for each of the 2^rb
    # real components of the pairs' first members
    fmas = len(re.findall(r"\bv_fmac?_f(?:32|64)\b", out.read_text()))
    assert fmas == rb * 2 * 3 * (1 << rb)
