"""The rules that cut a call's work into shares (csrc/wm_shares.hpp), compiled for
the host and checked over their ranges."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_04178_amd", "csrc")


def _build(tmp, name, body):
    src, exe = str(tmp / f"{name}.cpp"), str(tmp / name)
    open(src, "w").write("#include <cstdio>\n#include <cstdlib>\n#include \"wm_shares.hpp\"\nusing namespace wm;\n"
                         "int main(int, char** v)\n{\n" + body + "\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ftrapv", "-Wall", "-I", CSRC, src, "-o", exe], check=True)
    return lambda *a: [int(x) for x in subprocess.run([exe] + [str(x) for x in a], capture_output=True, text=True,
                                                      timeout=10, check=True).stdout.split()]


@pytest.mark.parametrize("n,avg", [(1, 1), (1000, 52), (1 << 15, 52), (1 << 16, 52), (1 << 16, 6), (1 << 14, 196),
                                   (2 ** 31 - 1, 1), (40000, 0)])
def test_tile_runs(tmp_path, n, avg):
    # waves of a 256-CU device at 24 per CU
    run = _build(tmp_path, "run", 'std::printf("%lld", (long long)tile_run(std::atoll(v[1]), std::atoll(v[2]), '
                                  "std::atoll(v[3]), std::atoi(v[4])));")
    one = run(n, n * avg, 6144, 1)[0]
    assert one >= max(1, -(-n // 6144))              # the waves hold every shape
    for gm in (2, 4, 8):
        per = run(n, n * avg, 6144, gm)[0]
        assert 1 <= per <= one
        # no shorter than three rounds of 64 candidates unless the runs of gm = 1 are
        assert per >= min(one, 192 // avg if avg else one)


def test_sweep_clears_flags(tmp_path):
    f = _build(tmp_path, "clears", 'std::printf("%d", (int)sweep_clears_flags(std::atoi(v[1]), std::atoll(v[2]), '
                                   "std::atoi(v[3])));")
    for block in (64, 128, 256, 512):
        assert f(1, 0, block) == [1] and f(1, 64 * block, block) == [1]
        assert f(1, 64 * block + 1, block) == [0] and f(1, 1 << 25, block) == [0]
        assert f(2, 1, block) == [0]
