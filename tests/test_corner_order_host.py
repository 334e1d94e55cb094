"""The corner turn's order of workgroups, where both were timed (no GPU needed): corner_order.h is
compiled with g++ and has to pick the faster one."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_05341_amd", "csrc")
HARNESS = r"""
#include "corner_order.h"
#include <stdio.h>
int main() {
  int bits, nc, tc;
  long ns, in_pitch, out;
  while (scanf("%d %d %ld %ld %ld %d", &bits, &nc, &ns, &in_pitch, &out, &tc) == 6)
    printf("%d\n", (int)dd::corner_runs(bits, nc, ns, in_pitch, (uint64_t)out, tc));
}
"""
# (bits, channels, samples, us by runs, us in order of time tiles), rows padded to 16 bytes
TIMES = [
    (32, 16384, 5000, 154.7, 137.9), (32, 8192, 5000, 67.1, 63.4), (32, 1024, 100000, 166.0, 158.0),
    (16, 16384, 5000, 71.6, 64.7), (16, 4096, 9522, 25.8, 23.3), (16, 128, 200000, 16.0, 14.5),
    (8, 32768, 1994, 28.1, 24.5), (8, 8192, 20000, 69.0, 65.9), (8, 64, 2152448, 63.3, 54.7), (8, 4096, 136192, 94.0, 88.0),
    (4, 16384, 8300, 39.8, 34.6), (4, 32768, 2002, 27.0, 22.3), (4, 256, 271658, 26.7, 24.1), (4, 8192, 14388, 38.9, 35.7),
    (32, 3000, 70002, 360.3, 609.6), (32, 64, 6357532, 661.6, 1326.4), (32, 4096, 119498, 720.0, 815.1),
    (16, 257, 125636, 19.2, 29.2), (16, 512, 357442, 171.3, 256.1), (16, 16384, 26540, 384.5, 423.4),
    (8, 1024, 2318480, 977.1, 2006.2), (8, 4096, 781250, 1308.0, 1808.0), (8, 1000, 100002, 29.0, 41.5),
    (8, 8192, 40002, 151.0, 173.0), (8, 4096, 253562 // 128 * 128, 383.7, 415.6),
    (4, 257, 231424, 22.9, 31.1), (4, 3000, 82732, 63.4, 77.6), (4, 512, 255994, 35.9, 41.7), (4, 4096, 441676, 1099.0, 1285.0),
]


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("corner_order")
    (d / "h.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(d / "h.cpp"), "-o", str(d / "h")], check=True)
    return str(d / "h")


def test_order_is_the_faster_one(exe):
    def pitch(n, bits):
        return ((n * bits + 7) // 8 + 15) // 16 * 16

    tile = {4: 256, 8: 256, 16: 128, 32: 64}
    text = "\n".join("%d %d %d %d %d %d" % (b, nc, ns, pitch(nc, b), pitch(ns, b), tile[b]) for b, nc, ns, _, _ in TIMES)
    got = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
    assert len(got) == len(TIMES)
    for g, row in zip(got, TIMES):
        assert (g == "1") == (row[3] < row[4]), row
