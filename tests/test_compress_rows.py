"""Which of the caller's rows a compression call may read (dq_unit.h), on the CPU: the rows of a block come as an address and a
number, and over all blocks of a call these are exactly the valid rows of the sequences that are not skipped; a block with
nothing to do has no address.  The number of blocks with something to do, by which the eigen-solver's launch chooses, is theirs."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <vector>
#include "dq_unit.h"
int main() {   // stdin: B, H, t_new, T_b, d, NB, n_valid given, blk_idx, n_valid; stdout: per unit slot, nv, 1 + row of X (0: null), live blocks of its sequence
  int p[7];
  while (fread(p, sizeof p, 1, stdin) == 1) {
    std::vector<int32_t> first(p[0]), valid(p[0]);
    if (fread(first.data(), 4, p[0], stdin) != (size_t)p[0] || fread(valid.data(), 4, p[0], stdin) != (size_t)p[0]) return 1;
    const dq_format f = {4, p[4], p[4], p[4] / 8, 8, p[3], 1, 0, 1};
    const dq::Geometry g = dq::make_geometry(f, p[1], p[5]);
    const long rows = (long)p[0] * p[1] * p[2];
    std::vector<uint16_t> k(rows * p[4]), v(rows * p[4]);
    const dq::CompressJob job = {k.data(), v.data(), p[2], (p[2] + p[3] - 1) / p[3], first.data(), p[6] ? valid.data() : nullptr, 0, 0, p[0]};
    for (int u = 0; u < 2 * p[0] * p[1] * job.n_blocks; ++u) {
      const dq::UnitRef r = dq::unit_ref(g, job, u);
      const long at = r.X ? r.X - (r.which ? v.data() : k.data()) : -p[4];
      if (at % p[4]) return 2;
      const int out[4] = {r.slot, r.nv, (int)(at / p[4]) + 1, dq::live_blocks(g, job, r.b)};
      fwrite(out, sizeof out, 1, stdout);
    }
  }
}
"""


def test_a_block_reads_the_valid_rows_of_sequences_that_are_not_skipped(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no ROCm compiler here")
    src, exe = tmp_path / "rows.hip", str(tmp_path / "rows")
    src.write_text(PROGRAM)
    run = subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                          "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2405_12591_amd", "csrc"),
                          str(src), "-o", exe], capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-2000:]
    rng = np.random.default_rng(1)
    for _ in range(60):
        b, h, tb, d = int(rng.integers(1, 5)), int(rng.integers(1, 4)), int(rng.choice([128, 256])), int(rng.choice([64, 128]))
        t_new = int(rng.choice([1, tb - 1, tb, tb + 1, int(rng.integers(1, 5 * tb))]))
        n_blocks, given = -(-t_new // tb), int(rng.integers(0, 2))
        nb = n_blocks + int(rng.integers(0, 2))
        first = rng.integers(-1, nb + 1, b).astype(np.int32)
        valid = np.array([rng.choice([-1, 0, 1, t_new, t_new + 3, int(rng.integers(0, t_new + 1))]) for _ in range(b)], np.int32)
        data = np.array([b, h, t_new, tb, d, nb, given], np.int32).tobytes() + first.tobytes() + valid.tobytes()
        out = np.frombuffer(subprocess.run([exe], input=data, capture_output=True, check=True).stdout, np.int32).reshape(b, h, n_blocks, 2, 4)
        for i in range(b):
            rows = min(max(int(valid[i]), 0), t_new) if given else t_new
            for j in range(n_blocks):
                nv = min(max(rows - j * tb, 0), tb)
                live = first[i] >= 0 and first[i] + j < nb and nv > 0
                for hd in range(h):
                    row = (i * h + hd) * t_new + j * tb
                    want = (first[i] + j, nv, 1 + row) if live else (-1, nv, 0)
                    assert (out[i, hd, j, :, :3] == want).all(), (t_new, tb, first, valid, given, i, hd, j, out[i, hd, j], want)
            assert (out[i, :, :, :, 3] == (out[i, 0, :, 0, 0] >= 0).sum()).all(), (t_new, tb, first, valid, given, i)
