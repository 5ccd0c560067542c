"""fp64 -> fp16 of the small tensors (dq_common.h): one rounding, ties to even, saturating at the fp16
range, compared on the CPU with numpy's conversion over every fp16 value's neighbourhood, the rounding
boundaries between them, subnormals, values beyond fp32 and the non-finite ones."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "dq_common.h"
int main() {   // stdin: doubles; stdout: per value the saturated bits, the plain bits, the flag
  double x;
  while (fread(&x, sizeof x, 1, stdin) == 1) {
    bool sat = false;
    const uint16_t out[3] = {dq::f64_to_f16_rne(x, true, &sat), dq::f64_to_f16_rne(x, false, nullptr), (uint16_t)sat};
    fwrite(out, sizeof out, 1, stdout);
  }
}
"""


def test_one_rounding_to_fp16(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no ROCm compiler here")
    src, exe = tmp_path / "round.hip", str(tmp_path / "round")
    src.write_text(PROGRAM)
    run = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xarch_host", "-mf16c", "-Xclang", "-target-feature",
                          "-Xclang", "-packed-fp32-ops",
                          "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2405_12591_amd", "csrc"),
                          str(src), "-o", exe], capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-2000:]
    halves = np.arange(0x7C00, dtype=np.uint16).view(np.float16).astype(np.float64)
    ties = (halves[:-1] + halves[1:]) / 2                      # exact in fp64
    x = np.concatenate([halves, ties, np.nextafter(ties, np.inf), np.nextafter(ties, 0), ties * (1 + 2.0 ** -30),
                        [65519.999999, 65520.0, 65536.0, 1e39, 1e300, np.inf, 1e-39, 1e-46, 5e-324, 2.0 ** -25, 0.0],
                        np.random.default_rng(1).standard_normal(4096) * 10.0 ** np.random.default_rng(2).uniform(-9, 6, 4096)])
    x = np.concatenate([x, -x, [np.nan]])
    out = subprocess.run([exe], input=x.tobytes(), capture_output=True, check=True).stdout
    sat, plain, flag = np.frombuffer(out, np.uint16).reshape(-1, 3).T
    with np.errstate(over="ignore"):
        want = x.astype(np.float16)
    beyond = np.abs(x) >= 65520
    assert np.array_equal(flag != 0, beyond)
    clipped = np.where(beyond, np.copysign(np.float16(65504), x).astype(np.float16), want)
    for got, ref in ((plain, want), (sat, clipped)):
        g = got.view(np.float16)
        assert np.isnan(g[-1]) and np.array_equal(got[:-1], ref[:-1].view(np.uint16)), x[:-1][got[:-1] != ref[:-1].view(np.uint16)][:8]
