"""What the compiler makes of kernels, read from their assembly (gfx950, compiled here).  Kernels that ask for the next turn's rows ahead: the
turn's arithmetic lies between the loads and the first wait for them (loads return in order, so that one touch of a value loaded last would
wait for all of them).  Half-precision pieces: every one made once."""
import os
import re
import subprocess

import pytest

from paper_2507_03840_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no compiler")


def kernels(source, tmp):
    out = str(tmp / (os.path.basename(source) + ".s"))
    subprocess.run([build.HIPCC, *build.FLAGS, "-w", "-S", "--cuda-device-only", source, "-o", out], cwd=build.CSRC, check=True,
                   stderr=subprocess.DEVNULL)
    found, name = {}, None
    for line in open(out):
        line = line.split(";")[0].strip()
        if re.match(r"_Z\w+:$", line):
            name, found[line[:-1]] = line[:-1], []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and line and not line.startswith("."):
            found[name].append(line)
    return found


def arithmetic_before_wait(code):
    """Vector instructions between the last load to LDS and the next wait for loads."""
    last = max(i for i, s in enumerate(code) if s.startswith("global_load_lds"))
    n = 0
    for s in code[last:]:
        if s.startswith("s_waitcnt") and "vmcnt" in s:
            break
        n += s.startswith("v_")
    return n


# an edge of lmax 1 takes more than 100 vector instructions in any of the kernels, one of lmax 4 about 1,000
@pytest.mark.parametrize("source,kernel,instances", [("tp_bins.hip", "tp_bins_kernel", 12), ("readout_adjoint.hip", "ra_bins_kernel", 16),
                                                     ("readout_adjoint.hip", "ra_edges_kernel", 16)])
def test_rows_of_the_next_turn(tmp_path, source, kernel, instances):
    code = {k: v for k, v in kernels(source, tmp_path).items() if kernel in k}
    assert len(code) == instances
    for name, lines in code.items():
        print(name, arithmetic_before_wait(lines))
        assert arithmetic_before_wait(lines) > 100, name
        assert not any(s.startswith("scratch_") for s in lines), name


@pytest.mark.parametrize("values,scale", [("a[8 * i + q]", "s"), ("a[8 * i + q]", "1.0f"), ("a[8 * i + q] * b[8 * i + q]", "s"),
                                          ("a[8 * i + q] * b[8 * i + q]", "1.0f")])
def test_pieces_are_made_once(tmp_path, values, scale):
    """sgh_cut8: eight values take sixteen roundings to half precision; one more, and a remainder is that of another high piece."""
    source = tmp_path / "cut.hip"
    source.write_text(f'''
#include "{build.CSRC}/egnn_internal.h"
#include "{build.CSRC}/stream_gemm.h"
__global__ void cut(const float* a, const float* b, uint4* out, float s) {{
  const int i = threadIdx.x;
  float x[8];
  for (int q = 0; q < 8; ++q) x[q] = {values};
  sgh_cut8(x, {scale}, out[2 * i], out[2 * i + 1]);
}}''')
    (lines,) = kernels(str(source), tmp_path).values()
    ops = [s.split()[0] for s in lines]
    one = sum(o.startswith(("v_fma_mixlo_f16", "v_fma_mixhi_f16", "v_cvt_f16_f32")) for o in ops)
    two = sum(o.startswith("v_cvt_pk") and "f16_f32" in o for o in ops)
    assert one + 2 * two == 16
