"""Streaming products refuse more rows than they have a kernel for: they must say so, not
return K splits that nothing wrote.  Links the built object of skinny.hip into a host
program; a refusal comes before any GPU call, so none is needed."""
import os
import subprocess

from paper_2609_09338_amd import build

PROGRAM = r"""
#include <cstdio>
#include "internal.h"
int main() {
  osp::GemvArgs a{};
  a.N = 1024;
  a.Kd = 1024;
  struct { osp::SrcKind src; int rows; } refused[] = {
    {osp::SRC_TAPS, 65}, {osp::SRC_TAPS, 96}, {osp::SRC_SWIGLU, 65}, {osp::SRC_ATTN, 80}, {osp::SRC_PREP, 97}, {osp::SRC_PREP, 4096}};
  for (auto& r : refused) {
    a.max_rows = r.rows;
    std::printf("%d\n", osp::launch_skinny(r.src, a, nullptr));
  }
  a.max_rows = 97;
  std::printf("%d\n", osp::launch_lm_head(a, osp::lm_head_plan(4096, 256), false, nullptr) ? 1 : 0);
}
"""


def test_streaming_products_refuse_more_rows_than_they_take(tmp_path):
    obj = os.path.join(build.BUILD, "skinny.o")
    if not os.path.exists(obj):
        build.build(verbose=False)
    main, exe = tmp_path / "main.cpp", tmp_path / "refuse"
    main.write_text(PROGRAM)
    cmd = [build.hipcc(), "-x", "hip"] + build.flags(False) + ["-c", str(main), "-o", str(tmp_path / "main.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([build.hipcc(), f"--offload-arch={build.ARCH}", str(tmp_path / "main.o"), obj, "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.split() == ["0"] * 7, (out.returncode, out.stdout, out.stderr)
