"""How batch norm's sums cover a tensor (csrc/bn_shape.h, host arithmetic): the lines between one and two slices of channels, on the side
where the measurements beside them put a shape; and that every row and channel is covered whatever the shape."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_1901_06773_amd", "csrc")
MAIN = """
#include <cstdio>
#include "bn_shape.h"
int main() {
  long rows; int c, v, es, back, stores;
  while (std::scanf("%ld %d %d %d %d %d", &rows, &c, &v, &es, &back, &stores) == 6) {
    const acc::SumShape s = acc::bn_sum_shape(rows, c, v, es, back, stores);
    std::printf("%d %d %d %d %d %d\\n", s.tpr, s.rpi, s.col_slices, s.slabs, acc::bn_stores_early(rows, c, es, false), acc::bn_stores_early(rows, c, es, true));
  }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    d = tmp_path_factory.mktemp("bn_shape")
    (d / "main.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")])

    def ask(cases):
        text = "".join(" ".join(str(int(x)) for x in c) + "\n" for c in cases)
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True)
        assert not out.stderr
        return [tuple(int(x) for x in line.split()) for line in out.stdout.splitlines()]
    return ask


# rows, channels, bytes of a value, backward (2: storing the masked gradient), slices of channels; four channels per thread
@pytest.mark.parametrize("rows,c,es,back,slices", [
    (2000, 128, 4, 0, 1), (2000, 128, 4, 1, 1), (2000, 132, 4, 1, 1), (784, 132, 4, 1, 1),     # slabs are not fewer with two
    (8036, 128, 4, 0, 2), (16384, 128, 4, 1, 2), (4096, 256, 4, 0, 2), (4096, 256, 4, 1, 2), (3600, 132, 4, 1, 2),
    (2000, 132, 2, 1, 1), (8036, 200, 2, 0, 2), (8036, 200, 2, 1, 2),
    (12544, 200, 2, 0, 1), (12544, 200, 2, 1, 1), (16384, 132, 2, 1, 1), (12544, 256, 2, 1, 1),  # one slice would take the finishing launch
    (12544, 200, 4, 0, 2), (12544, 200, 4, 1, 1), (14500, 252, 4, 1, 1), (16384, 132, 4, 1, 1),
    (12544, 256, 4, 0, 2), (12544, 256, 4, 1, 2), (16384, 256, 4, 2, 2), (13000, 160, 4, 1, 2), (16384, 192, 4, 1, 2), (16384, 192, 4, 2, 1),
    (14500, 224, 4, 2, 1), (8036, 192, 4, 2, 2),
    (16385, 256, 4, 0, 1), (8036, 124, 4, 0, 1), (8036, 260, 4, 0, 2),
])
def test_slices_of_channels(shapes, rows, c, es, back, slices):
    assert shapes([(rows, c, 4, es, back > 0, back == 2)])[0][2] == slices


# the pass that stores as it sums: no slice of a few threads beside one of 64
@pytest.mark.parametrize("rows,c,es,tpr", [(12544, 260, 4, 33), (25088, 264, 4, 33), (25088, 320, 4, 40), (12544, 384, 4, 48), (25088, 512, 4, 64), (16384, 300, 2, 38)])
def test_slices_of_like_width_where_gradients_are_stored(shapes, rows, c, es, tpr):
    assert shapes([(rows, c, 4, es, 1, 1)])[0][0] == tpr
    assert shapes([(rows, c, 4, es, 1, 0)])[0][0] == 64


# rows, channels, channels per thread, bytes of a value, backward (2: storing the masked gradient), slabs
@pytest.mark.parametrize("rows,c,v,es,back,slabs", [
    (1568, 2048, 4, 4, 2, 98), (1568, 2048, 4, 4, 1, 96), (25088, 256, 8, 2, 2, 784), (25088, 256, 8, 2, 1, 768), (25088, 256, 8, 2, 0, 768),
    (28672, 256, 8, 2, 2, 896), (28673, 256, 8, 2, 2, 768), (65536, 256, 8, 2, 0, 768), (65537, 256, 8, 2, 0, 1024), (65537, 256, 8, 2, 1, 1024),
    (200704, 512, 8, 2, 2, 768), (200704, 512, 8, 2, 0, 1024), (12544, 2048, 4, 2, 0, 128), (12544, 2048, 4, 2, 2, 96),
    (200704, 64, 4, 4, 0, 768), (200704, 64, 4, 4, 1, 768), (200704, 64, 4, 4, 2, 768),
])
def test_three_or_four_workgroups_per_compute_unit(shapes, rows, c, v, es, back, slabs):
    assert shapes([(rows, c, v, es, back > 0, back == 2)])[0][3] == slabs


# alone / in an iteration
@pytest.mark.parametrize("rows,c,es,alone,step", [
    (8036, 1024, 4, True, False), (32144, 512, 4, True, False), (128576, 256, 4, True, True), (25088, 1024, 4, True, True),
    (8036, 1024, 2, True, True), (1023, 1024, 4, False, False), (1023, 1024, 2, False, False),
])
def test_where_the_sums_store_the_masked_gradient(shapes, rows, c, es, alone, step):
    assert shapes([(rows, c, 4, es, 1, 1)])[0][4:] == (alone, step)


def test_everything_is_covered(shapes):
    cases = [(rows, c, v, es, back > 0, back == 2) for rows in (1, 3, 49, 513, 2048, 4097, 9999, 16384, 16385, 200704, 1 << 31)
             for c in (4, 8, 64, 124, 128, 132, 200, 252, 256, 260, 264, 320, 512, 516, 2048, 65536) for v, es in ((4, 4), (4, 2), (8, 2))
             for back in (0, 1, 2) if c % v == 0]
    for (rows, c, v, es, back, stores), (tpr, rpi, cols, slabs, _, _) in zip(cases, shapes(cases)):
        assert 1 <= tpr <= 64 and tpr * rpi <= 256 and rpi >= 1
        assert cols * tpr * v >= c > (cols - 1) * tpr * v              # no slice without channels
        assert 1 <= slabs <= 1024 and slabs * cols <= max(1024, cols)
