"""LDS of the workgroup sums in the h passes against the launch shapes that
the tuner and its cache can pick (half, default and double the pencils)."""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1610_07522_amd", "csrc")

FACT = {int(n): (int(r1), int(r2)) for n, r1, r2 in re.findall(
    r"struct Fact<(\d+)>\s*\{\s*static constexpr int R1 = (\d+), R2 = (\d+);",
    open(os.path.join(CSRC, "sky_common.h")).read())}


def shapes(n, value_bytes):
    """Threads per workgroup of every pencil count that launch_apply_h takes."""
    r1, r2 = FACT[n]
    rt = max(r1, r2)
    d = 64 if rt == 4 else 32

    def ok(lp):
        return (n * n % lp == 0 and rt * lp <= 1024 and
                lp * (2 * r1 * (r2 + 1) + 1) * value_bytes <= 96 * 1024)

    return sorted({rt * lp for lp in (d // 2, d, 2 * d) if lp == d or ok(lp)})


@pytest.mark.parametrize("value_bytes", [8, 16])
@pytest.mark.parametrize("n", sorted(FACT))
def test_h_pass_sums_have_an_entry_per_wave(n, value_bytes):
    src = open(os.path.join(CSRC, "k_grid.hip")).read()
    body = src[src.index("k_h_pass(const cpx<T>*"):]
    extent = re.search(r"__shared__ double red\[(.*?)\];", body).group(1)
    rule = re.search(r"int waves_of_threads\(int threads\) \{ return (.*?); \}", src)
    for threads in shapes(n, value_bytes):
        entries = extent
        if rule:
            entries = entries.replace("waves_of_threads(C::THREADS)", f"({rule.group(1)})")
        entries = eval(entries.replace("/", "//"), {"threads": threads})
        assert entries >= -(-threads // 64), (n, threads)
