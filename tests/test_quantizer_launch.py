"""The quantisers' threads per row and the kernel that is launched for them agree, and cover the row: every row length, on the CPU."""
import os
import subprocess

import pytest

from paper_2603_08185_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")

SOURCE = """
#include "%s/serq_device.h"
#include <cstdio>
int main() {
  for (int nchunk = 8; nchunk <= 131072 / 8; nchunk += 8)
    for (long long M : {1, 256, 257, 384, 385, 512, 513, 4096})
      for (auto kind : {serq::Quantizer::kPlain, serq::Quantizer::kGated, serq::Quantizer::kAsym}) {
        const int threads = serq::quantizer_threads(kind, nchunk, M);
        const int per = (nchunk + threads - 1) / threads;
        int kt = 0, nc = -1;
#define LAUNCH(KT, NC) (kt = KT, nc = NC)
        SERQ_QUANTIZER_LAUNCH(threads, per, LAUNCH);
        if (kt != threads || (nc > 0 ? nc < per : nc < 0 || nchunk <= 4096) || kt %% 64 || kt > 1024) {
          printf("nchunk %%d, M %%lld: %%d threads, %%d pieces, kernel of %%d x %%d", nchunk, M, threads, per, kt, nc);
          return 1;
        }
      }
  return 0;
}
"""


def test_every_row_length_has_its_kernel(tmp_path):
    src, exe = tmp_path / "t.hip", tmp_path / "t"
    src.write_text(SOURCE % build.CSRC)
    subprocess.run([HIPCC, "--cuda-host-only", "-std=c++17", "-O1", "-w", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
