"""The planning programme's row counters (csrc/wm_plan_rows.hpp) compiled for the
host and run at the ends of chains of up to 2^31 - 1 rows, the most that 32-bit
offsets allow: every row is in exactly one batch, the loop ends, a shorter chain
of the same wave has no rows left, and no stored batch reaches past its chain."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_04178_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#define __host__
#define __device__
#include "wm_plan_rows.hpp"
using namespace wm;
#define CHECK(x) do { if (!(x)) { std::printf("L=%d: %s\n", L, #x); return 1; } } while (0)
int main(int, char** v)
{
    const int32_t L = (int32_t)std::atol(v[1]);
    PlanRows rows(L), beside(5);
    const uint32_t first = L > 64 ? (uint32_t)(L - 64) & ~15u : 0u;   // the last batches
    rows.at = beside.at = first;
    int64_t seen = 0;
    int batches = 0;
    for (; rows.more(); rows.next(), beside.next()) {
        CHECK(++batches <= 6);
        CHECK(rows.left() == (int64_t)L - (int64_t)rows.at && rows.left() > 0);
        CHECK(beside.left() == (rows.at >= 5u ? 0 : 5 - (int32_t)rows.at));
        for (int k = 0; k < kPlanBatch; ++k) seen += k < rows.left();
    }
    CHECK(rows.left() == 0 && seen == (int64_t)L - first);
    // backwards over the same rows, as the cut lengths are followed
    int64_t next = L;
    for (int32_t w0 = last_batch(L); w0 >= (int32_t)first; w0 -= kPlanBatch) {
        int64_t n = 0;
        for (int r = 0; r < kPlanBatch; ++r) n += r < L - w0;
        CHECK((int64_t)w0 + n == next);
        CHECK(batch_stored(w0, L) == ((int64_t)w0 + kPlanBatch < (int64_t)L));
        next = w0;
    }
    CHECK(next == (L > 0 ? (int64_t)first : 0));
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    src, exe = str(d / "rows.cpp"), str(d / "rows")
    open(src, "w").write(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O0", "-ftrapv", "-Wall", "-I", CSRC, src, "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("L", [0, 1, 15, 16, 17, 64, 2 ** 31 - 33, 2 ** 31 - 32, 2 ** 31 - 17, 2 ** 31 - 16,
                               2 ** 31 - 15, 2 ** 31 - 2, 2 ** 31 - 1])
def test_plan_row_counters(program, L):
    r = subprocess.run([program, str(L)], capture_output=True, text=True, timeout=10)
    assert r.returncode == 0, r.stdout
