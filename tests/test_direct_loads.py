"""The direct global -> LDS load by four lanes (dma64), where not all lanes are active: it takes those of the first four that are, and
the lanes that go on behind it are the ones that came.  The machine code, run lane by lane on the CPU."""
import os
import struct
import subprocess

import numpy as np
import pytest

from paper_2603_08185_amd import build
from tests import _isa

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")

SOURCE = """
#include "%s/serq_device.h"
namespace serq {
struct P { const uint8_t* src; int first; };
__global__ void kernel(const P p) {
  __shared__ uint8_t lds[2048];
  const int l = threadIdx.x;
  if (l >= p.first) {
    dma64(p.src, 16u * l, lds_addr(lds));
    dma16(p.src, 16u * l, lds_addr(lds) + 1024);
  }
  asm volatile("s_waitcnt vmcnt(0)\\n\\ts_barrier" ::: "memory");
}
}
"""


@pytest.mark.parametrize("first", [0, 1, 3, 40])
def test_four_lane_load_keeps_the_active_lanes(first, tmp_path):
    src, out = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(SOURCE % build.CSRC)
    subprocess.run([HIPCC, *build.FLAGS, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True)
    text = out.read_text()
    lines = next(v for k, v in _isa.kernels(text).items() if "kernel" in k)
    buf = {"src": (0x7F0000000000, 1024)}
    wave = _isa.Wave(_isa.program(lines), struct.pack("<Qi", buf["src"][0], first) + bytes(20), 0, 0, buf, 2048)
    loads = [set(np.flatnonzero(ld.off != np.uint64(_isa.M64))) for ld in wave.run()]
    active = set(range(first, 64))
    four = active & set(range(4))
    assert loads == ([four] if four else []) + [active]                   # (a load by no lane at all brings nothing)
    assert wave.st["exec"] == _isa.M64
