"""Rules of the matrix-core products' launches on the host: what a kernel does not take must
be refused, before any GPU call (so none is needed).  Links built objects into host programs."""
import os
import subprocess

from paper_2609_09338_amd import build

STREAMING = r"""
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


TILED = r"""
#include <cstdio>
#include "internal.h"
int main() {
  alignas(256) static char mem[1024];
  osp::GemvArgs a{};
  a.N = 1024;
  a.max_rows = 200;
  auto say = [&](osp::SrcKind src, long rows) { std::printf("%d\n", osp::gemm_rows_supported(src, a, rows) ? 1 : 0); };
  // taps of 3 x 4096 columns, weights beside them
  a.taps = mem;
  a.w0 = mem + 256;
  a.ldt = a.Kd = 12288;
  say(osp::SRC_TAPS, 200);                       // taken
  say(osp::SRC_TAPS, 87381);                     // the last that a 31-bit byte offset reaches
  say(osp::SRC_TAPS, 87382);
  a.taps = mem + 2;
  say(osp::SRC_TAPS, 200);
  a.taps = mem + 8;
  say(osp::SRC_TAPS, 200);
  a.taps = mem;
  a.w0 = mem + 258;
  say(osp::SRC_TAPS, 200);
  a.w0 = mem + 256;
  a.ldt = a.Kd = 600;                            // not whole 32-column steps
  say(osp::SRC_TAPS, 200);
  // prepared rows
  a.taps = nullptr;
  a.Kd = a.ld_xa = 1024;
  say(osp::SRC_PREP, 200);                       // taken
  a.w1 = mem + 512;
  say(osp::SRC_PREP, 200);                       // taken
  a.w1 = mem + 516;
  say(osp::SRC_PREP, 200);
  a.w1 = nullptr;
  a.max_rows = 128;
  say(osp::SRC_PREP, 128);
}
"""


def _run(tmp_path, program, name):
    obj = os.path.join(build.BUILD, name)
    if not os.path.exists(obj):
        build.build(verbose=False)
    main, exe = tmp_path / "main.cpp", tmp_path / "rule"
    main.write_text(program)
    cmd = [build.hipcc(), "-x", "hip"] + build.flags(False) + ["-c", str(main), "-o", str(tmp_path / "main.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([build.hipcc(), f"--offload-arch={build.ARCH}", str(tmp_path / "main.o"), obj, "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, (out.returncode, out.stdout, out.stderr)
    return out.stdout.split()


def test_streaming_products_refuse_more_rows_than_they_take(tmp_path):
    """They must not return K splits that nothing wrote."""
    assert _run(tmp_path, STREAMING, "skinny.o") == ["0"] * 7


def test_tiled_products_take_what_their_copies_reach(tmp_path):
    """Copies into LDS move 16 aligned bytes at 31-bit offsets."""
    assert _run(tmp_path, TILED, "gemm_rows.o") == list("11000001100")
