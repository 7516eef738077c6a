"""The bf16 GEMM's launch plans, from the planner's own code compiled for the host alone (CPU only)."""
import os
import subprocess

import pytest

from paper_2608_22646_amd import build

PROGRAM = r"""
#include "%s"
#include <cstdio>
namespace dllm { int device_cu_count() { return 256; } }
using namespace dllm;
int main() {
  // a K split of a q/k/v or SwiGLU GEMM goes to a kernel with partial sums for them: none of the 256-row tiles
  for (int K : {256, 512, 1024, 3584, 4096, 12288, 18944})
    for (int N = 256; N <= 49152; N += 256)
      for (int M : {1, 17, 32, 33, 64, 65, 96, 127, 128, 129, 160, 300, 512, 1095, 8192})
        for (int epi : {EPI_QKV_ROPE, EPI_SWIGLU}) {
          const Plan p = plan(M, N, K, epi);
          if (p.bm == 256 && p.split > 1) printf("plan %%d %%d %%d %%d: split %%d\n", M, N, K, epi, p.split);
        }
  GemmArgs g{};
  g.M = 4096;
  g.N = 512;
  g.K = 512;
  for (int which = 0; which < 4; ++which) try {
      if (which == 0) launch_tile16<TileL, EPI_SWIGLU>(g, 2, nullptr);
      if (which == 1) launch_tile16<TileL, EPI_QKV_ROPE>(g, 2, nullptr);
      if (which == 2) launch_tile16<TileM, EPI_SWIGLU>(g, 2, nullptr);
      if (which == 3) launch_tile16<TileM, EPI_QKV_ROPE>(g, 2, nullptr);
      puts("launched");
    } catch (const HipError& e) {
      puts(e.what());
    }
}
"""


@pytest.fixture(scope="module")
def output(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.hip", d / "plan"
    src.write_text(PROGRAM % os.path.join(build.CSRC, "k_gemm_bf16.hip"))
    # host code only: the kernels are not compiled, so their code object is missing at link time
    subprocess.run([build.hipcc(), "--cuda-host-only", f"--offload-arch={build.ARCH}", "-O1", "-std=c++17", "-w",
                    "-x", "hip", str(src), "-o", str(exe), "-Wl,--unresolved-symbols=ignore-all"], check=True, timeout=300)
    # no GPU is shown to it: a launch that is not refused fails on the host
    env = dict(os.environ, HIP_VISIBLE_DEVICES="", ROCR_VISIBLE_DEVICES="")
    return subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=120, env=env).stdout.split("\n")


def test_256_row_tiles_split_k_for_residuals_only(output):
    assert not [l for l in output if l.startswith("plan")]
    refused = [l for l in output if l and not l.startswith("plan")]
    assert len(refused) == 4 and all("K split" in l for l in refused), refused
