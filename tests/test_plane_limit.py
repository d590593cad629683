"""Which kernels a context takes by the size of an angle's plane of intensities: the
wave-group kernels address it by 32-bit byte offsets, so planes of more than 4 GiB go to the
thread-per-cell kernels (64-bit), and gas feedback, which only the wave-group kernels have, is
refused for them.  Host code only: the rule is asked of the library's own context set-up."""
import os
import subprocess

import numpy as np
import pytest

from paper_1403_6126_amd import rt

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "rt_internal.hpp"
int main(int argc, char **argv) {
  const double mu[6] = {0.5, 0, 0, -0.5, 0, 0}, w[2] = {0.5, 0.5};
  for (int i = 1; i + 1 < argc; i += 2) {
    rt_grid g = {1, {atoi(argv[i]), 1, 1}, {1.0, 1.0, 1.0}, {{0, 0}, {0, 0}, {0, 0}}};
    rt_angles a = {2, mu, w};
    rt_params p = {1.0, 1.0, 5.0 / 3.0, 1.0, atoi(argv[i + 1]), 0u, 0.0, 0, 0.0};
    rt_ctx c;
    const int st = rtk::ctx_init_host(&g, &a, &p, &c);
    printf("%d %d %lld\n", st, c.shape.waves, rtk::ctx_step_blocks(&c, true));
  }
}
"""


def test_planes_beyond_32_bit_offsets_run_per_cell(tmp_path):
    src = tmp_path / "shape.hip"
    src.write_text(SRC)
    exe = tmp_path / "shape"
    lib = os.path.dirname(rt.LIB_PATH)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-std=c++17", "-O1",
                    "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-w", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(lib, "csrc"), str(src), "-L", lib, "-l:librt.so",
                    f"-Wl,-rpath,{lib}", "-o", str(exe)], check=True)
    cases = [(n, p) for p, lim in ((rt.RT_FP64, 2**29), (rt.RT_FP32_MIXED, 2**30))
             for n in (2**28, lim - 1, lim, lim + 1, 2**31 - 1)]
    out = subprocess.run([str(exe)] + [str(x) for c in cases for x in c], check=True,
                         capture_output=True, text=True).stdout.split()
    rows = np.array(out, dtype=np.int64).reshape(-1, 3)
    for (n, p), (st, waves, blocks) in zip(cases, rows):
        fits = n * (4 if p == rt.RT_FP32_MIXED else 8) <= 2**32
        assert st == rt.RT_OK and (waves > 0) == fits, (n, p, waves)
        assert blocks == -(-n // (64 if fits else 256)), (n, p, blocks)


@pytest.mark.parametrize("precision,n", [(rt.RT_FP64, 2**29 + 1), (rt.RT_FP32_MIXED, 2**30 + 1)])
def test_feedback_needs_planes_of_4_gib(precision, n):
    mu, w = rt.rt_quadrature(rt.RT_QUAD_GAUSS_LEGENDRE, 2)
    g = rt.make_grid(1, (n, 1, 1), (1.0, 1.0, 1.0), ((0, 0),) * 3)
    p = rt.make_params(1.0, 1.0, 5 / 3, 1.0, precision, rt.RT_GAS_FEEDBACK)
    with pytest.raises(rt.RTError) as ei:
        rt.rt_create(g, mu, w, p)
    assert ei.value.status == rt.RT_EUNSUPPORTED
