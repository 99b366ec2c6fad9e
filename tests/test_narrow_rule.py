"""When an ingest runs its last layer for the used rows alone (csrc/narrow.h), on the host:
never where nothing is dropped, never for fewer rows than were measured to pay, and monotone
in the rows."""
import os
import subprocess

import pytest

from paper_2609_09338_amd import build

PROGRAM = r"""
#include <cstdio>
#include "narrow.h"
int main() {
  osprey_config c{};
  int dtype, d, nq, hd, ffn;
  long rows, keep;
  while (std::scanf("%d %d %d %d %d %ld %ld", &dtype, &d, &nq, &hd, &ffn, &rows, &keep) == 7) {
    c.dtype = dtype; c.d_model = d; c.n_q_heads = nq; c.head_dim = hd; c.d_ffn = ffn;
    std::printf("%d\n", osp::narrow_pays(c, rows, keep) ? 1 : 0);
  }
}
"""
F32, BF16 = 0, 1
D256, D1024, D2560, F1024 = (F32, 256, 4, 64, 1024), (BF16, 1024, 16, 128, 3072), (BF16, 2560, 32, 128, 9728), (F32, 1024, 16, 128, 3072)


@pytest.fixture(scope="module")
def pays(tmp_path_factory):
    d = tmp_path_factory.mktemp("narrow")
    (d / "main.cpp").write_text(PROGRAM)
    exe = str(d / "rule")
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, "-I", os.path.join(build.ROOT, "include"), str(d / "main.cpp"),
                    "-o", exe], check=True)

    def ask(queries):
        text = "\n".join(" ".join(map(str, (*body, rows, keep))) for body, rows, keep in queries)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
        return [x == "1" for x in out]
    return ask


def test_dtype_values():
    from paper_2609_09338_amd import _lib as L
    assert (L.OSPREY_F32, L.OSPREY_BF16) == (F32, BF16)


def test_nothing_to_drop_is_never_narrowed(pays):
    q = [(body, keep, keep) for body in (D256, D1024, D2560, F1024) for keep in (1, 16, 64, 65, 96, 128, 256)]
    assert not any(pays(q))


def test_more_rows_never_turn_it_off(pays):
    for body in (D256, D1024, D2560, F1024):
        for keep in (1, 3, 8, 64, 65, 128, 256):
            got = pays([(body, rows, keep) for rows in range(keep, 16 * keep + 200)])
            assert got == sorted(got) and got[-1]


@pytest.mark.parametrize("body,rows,keep,want", [
    (D1024, 65, 1, True), (D1024, 64, 1, False), (D1024, 128, 64, False), (D1024, 192, 64, True), (D1024, 96, 96, False),
    (D1024, 288, 96, False), (D1024, 384, 96, True), (D2560, 128, 64, True), (D2560, 192, 96, False), (D2560, 288, 96, True),
    (D256, 128, 1, True), (D256, 15, 1, False), (D256, 16, 2, True), (D256, 16, 4, False), (D256, 32, 8, False),
    (F1024, 24, 4, True), (F1024, 24, 8, False), (F1024, 32, 8, True), (F1024, 24, 16, False)])
def test_measured_cases(pays, body, rows, keep, want):
    assert pays([(body, rows, keep)]) == [want]
