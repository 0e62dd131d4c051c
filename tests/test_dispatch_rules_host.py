"""The rules that share a call out over the chip, evaluated on the host: the library's own objects are linked into a small
program that prints what the launchers decide.  No GPU is used."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2104_10949_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <string.h>
#include "prf.h"
int main(int argc, char** argv) {
    unsigned long long a[4];
    char what[16];
    while (scanf("%15s %llu %llu", what, a, a + 1) == 3) {
        const cg::PrfSplit s = cg::prf_split(a[0], a[1]);
        printf("%llu %u %u\n", (unsigned long long)s.blocks, s.waves, s.per_wg);
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    """rules(what, rows of numbers) -> rows of numbers printed by the program"""
    from paper_2104_10949_amd import build as b
    objects = [os.path.join(CSRC, o) for _, o, _ in b.UNITS]
    if not all(os.path.exists(o) for o in objects):
        b.build()
    d = tmp_path_factory.mktemp("rules")
    src, exe = str(d / "rules.cpp"), str(d / "rules")
    with open(src, "w") as f:
        f.write(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), src, *objects, "-L", os.path.join(rocm, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.join(rocm, "lib"), "-o", exe], check=True)

    def ask(what, rows):
        text = "".join(what + " " + " ".join(str(v) for v in r) + "\n" for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]

    return ask


def test_prf_runs_are_even_over_the_compute_units(rules):
    """One workgroup runs per compute unit, so the slowest of 256 takes ceil(blocks / 256) runs of per_wg chunks: within
    5 % of an even share for long calls, and never more than a workgroup's constants have room for."""
    full = 256 * 2044 * 128   # words of one full run per compute unit
    cases = [(f, n) for f in (0, 1, 127, 130, 2 ** 40 + 77)
             for n in (1, 2, 128, 129, 32768, 262144, 300001, 1 << 20, 5000000, 1 << 26, full - 128, full, full + 128, 70000000,
                       int(1.5 * full), 2 * full + 5, 140000000, int(2.5 * full), 1 << 28, 1 << 30, (1 << 33) + 12345)]
    for (first, n), (blocks, waves, per_wg) in zip(cases, rules("prf", cases)):
        chunks = (first + n - 1) // 128 - first // 128 + 1
        assert (blocks - 1) * per_wg < chunks <= blocks * per_wg < 2 ** 62, (first, n)
        assert 1 <= per_wg <= 2044 and blocks < 2 ** 31, (first, n)
        assert waves == 16, (first, n)   # short calls too: they are little more than the fill of the tables
        slowest = -(-blocks // 256) * per_wg
        assert slowest <= max(1.05 * chunks / 256, chunks / 256 + 1), (first, n, blocks, per_wg)
