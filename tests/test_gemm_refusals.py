"""Product launches that a tile cannot carry out are refused on the host, before anything is launched.
CPU only: a small program calls the library's launcher with such descriptors."""

import os
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]
PKG = ROOT / "paper_1312_1549_amd"
ROCM = Path(os.environ.get("ROCM_PATH", "/opt/rocm"))

PROGRAM = r"""
#include <cstdio>
#include "omm_internal.h"
using namespace omm;
int main() {
  // pair rows or a symmetric result together with planes, FP64 small tiles and a staged BF16 one
  int bad = 0;
  for (int tile = 0; tile < gemm_num_tiles(); ++tile)
    for (int pair = 0; pair < 2; ++pair) {
      GemmDesc d{CF64, T_F64, T_F64, T_F64, T_F64, KC, KC, tile, 1};
      if (!gemm_supported(d)) continue;
      if (pair && tile < 7) continue;  // the staged tiles rotate the planes in a pass of their own
      GemmOp op{};
      op.M = 16; op.N = 16; op.nseg = 1; op.K[0] = 16;
      op.lda[0] = op.ldb[0] = op.ldc = op.ldp = 16;
      op.Chi = &op;
      if (pair) op.pair_rows = 16; else op.tri = 1;
      const int e = (int)gemm_launch(d, &op, 1, nullptr, nullptr, 0, nullptr);
      std::printf("tile %d %s: %d\n", tile, pair ? "pair" : "tri", e);
      bad += e != (int)hipErrorInvalidValue;
    }
  return bad;
}
"""


def test_planes_of_symmetric_and_paired_products_are_refused(tmp_path):
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("checked without a GPU, so that nothing could be launched")
    src, exe = tmp_path / "refusals.cpp", tmp_path / "refusals"
    src.write_text(PROGRAM)
    lib = PKG / "libomm.so"
    if not lib.exists():
        from paper_1312_1549_amd.build import build

        build()
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{PKG / 'csrc'}", f"-I{ROCM / 'include'}",
                    str(src), str(lib), f"-L{ROCM / 'lib'}", "-lamdhip64", f"-Wl,-rpath,{PKG}:{ROCM / 'lib'}",
                    "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "tile 7 pair" in run.stdout and "tile 0 tri" in run.stdout, run.stdout
