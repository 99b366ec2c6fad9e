"""The waits of the three-stage tiled products (gemm_rows.hip, blocks of 256 rows), read
from the gfx950 assembly of the source as the library builds it: past each of the loop's
barriers the next copies overwrite the stage that the step before has read, so a wavefront
may only arrive there with its LDS reads done (lgkmcnt(0)) and with no more copies
outstanding than the step requests (vmcnt(CP)).  Compiles for the GPU, needs none."""
import os
import re
import subprocess

import pytest

from paper_2609_09338_amd import build


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    out = tmp_path_factory.mktemp("isa") / "gemm_rows.lst"
    cmd = [build.hipcc()] + build.flags(False) + ["--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm_rows.hip"),
                                                  "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out.read_text()


def _kernels(text):
    """{(source, epilogue, row tiles): its instructions} of k_gemm_rows<source, epilogue, row tiles>."""
    found = {}
    for m in re.finditer(r"^(_ZN3osp11k_gemm_rowsILi(\d+)ELi(\d+)ELi(\d+)E\w+):(.*?)^\s*\.end_amdhsa_kernel", text, re.S | re.M):
        code = [line.split(";")[0].strip() for line in m.group(5).splitlines()]
        found[tuple(int(x) for x in m.group(2, 3, 4))] = [x for x in code if x and not x.startswith(".")]
    return found


def test_loop_barriers_wait_for_reads_and_copies(listing):
    wide = {k: v for k, v in _kernels(listing).items() if k[2] == 4}
    assert len(wide) == 3
    for (src, epi, _), code in wide.items():
        at = [i for i, x in enumerate(code) if x == "s_barrier"]
        assert len(at) == 3, (src, epi)
        copies = sum(x.endswith(" lds") for x in code[at[0]:at[1]])      # a step's
        for i in at:
            # back from the barrier to its wait: no LDS read may be issued in between
            for x in reversed(code[:i]):
                assert not x.startswith("ds_"), (src, epi, x)
                if x.startswith("s_waitcnt"):
                    break
            assert f"vmcnt({copies})" in x and "lgkmcnt(0)" in x, (src, epi, x)
