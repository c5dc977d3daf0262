"""The split of the weight gradient's row sum for every row count of a training step up to 200,000 rows and some far
larger: no more splits than the workspace holds partial products for, and every row in one of them.  Runs the library's
own rule (csrc/mlp_split.h) on the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "mlp_split.h"
#include <cstdio>
int main() {
    int bad = 0;
    auto check = [&](int64_t rows) {
        const ri::Gw2Split s = ri::gw2_split(rows);
        const bool ok = s.splits >= 1 && s.splits <= ri::GW2_SPLITS && s.per >= 64 && s.per % 16 == 0 &&
                        4 * s.per * s.splits >= rows && 4 * s.per * (s.splits - 1) < rows;
        if (!ok && bad++ < 10) std::printf("rows %lld: per %lld splits %d\n", (long long)rows, (long long)s.per, s.splits);
    };
    for (int64_t n = 1; n <= 200000; ++n) {
        check((n + 31) / 32 * 32);
        check((n + 63) / 64 * 64);
    }
    for (int64_t n = 1 << 20; n < (int64_t(1) << 33); n = n * 3 / 2 + 1) check((n + 63) / 64 * 64);
    return bad != 0;
}
"""


def test_row_sum_splits_fit_their_workspace(tmp_path):
    src, exe = tmp_path / "split.cpp", tmp_path / "split"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2407_19614_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
