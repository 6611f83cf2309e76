"""Arithmetic that the launcher hands to the kernels, compiled for the host from the launcher's own header and checked here."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_22804_amd", "csrc")
SOURCE = r"""
#include <cstdio>
#include "mor_launch.h"
using namespace mor;
// A shift by the width of the shifted value or more is undefined: the de-quantize kernel shifts columns in 32 bits, rows in 64.
static bool shifts() {
    const int64_t dims[] = {1, 7, 8, 63, 64, 65, 120, 127, 128, 129, 200, 4096, 65536, 4194296};
    for (int gran = kGranTensor; gran <= kGranBlock64; ++gran)
        for (int64_t rows : dims)
            for (int64_t cols : dims) {
                const StatsGeom g = make_geom(gran, rows, cols);
                const int c32 = block_shift(g.pc, cols, 32), r64 = block_shift(g.pr, rows, 64);
                if (c32 < 0 || c32 > 31 || r64 < 0 || r64 > 63) return false;
                const int64_t some[] = {0, 1, 62, 63, 64, 65, 127, 128, 129, rows - 1, cols - 1};
                for (int64_t i : some) {
                    if (i >= 0 && i < cols && (int64_t)((uint32_t)i >> c32) != i / g.pc) return false;
                    if (i >= 0 && i < rows && (i >> r64) != i / g.pr) return false;
                }
            }
    return true;
}
// n / d from the reciprocal, at the ends of its range and around multiples of d.
static bool reciprocals() {
    for (int64_t d = 1; d < 0x7FFFFFFF; d += d < 3000 ? 1 : d / 7 + 1) {
        uint32_t mul, shift;
        recip_of(d, &mul, &shift);
        for (int64_t k = 0; k < 0x7FFFFFFF; k += k < 8 * d ? d : 0x7FFFFFFF / 5)
            for (int64_t n = k - 2; n <= k + 2; ++n) {
                if (n < 0 || n >= 0x7FFFFFFF) continue;
                const uint32_t q = (uint32_t)(((uint64_t)(2u * (uint32_t)n) * mul) >> 32) >> shift;
                if ((int64_t)q != n / d) return false;
            }
    }
    return true;
}
// Several large operands without a proof get more workgroups for their copies than one does; small ones and proven ones do not.
static bool copy_budget() {
    const int64_t mb = 1 << 20;
    return scope_copy_budget(0, 0) == 1024 && scope_copy_budget(1, 224 * mb) == 1024 && scope_copy_budget(2, 224 * mb) == 2048 &&
           scope_copy_budget(12, 960 * mb) == 4096 && scope_copy_budget(12, 100 * mb) == 1600 && scope_copy_budget(64, mb) == 1024;
}
int main() {
    printf("shifts=%d reciprocals=%d copy_budget=%d\n", shifts(), reciprocals(), copy_budget());
    return 0;
}
"""


@pytest.fixture(scope="module")
def answers(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.cpp", d / "rules"
    src.write_text(SOURCE)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    return dict(kv.split("=") for kv in out.split())


@pytest.mark.parametrize("rule", ["shifts", "reciprocals", "copy_budget"])
def test_rule(answers, rule):
    assert answers[rule] == "1"
