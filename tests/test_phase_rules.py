"""Which phases the dispatch sends along the line, against what the launch's
32-bit index can walk; asked of the built library, on the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2606_27086_amd")

PROGRAM = r"""
#include "smx_internal.h"
#include <cstdio>
#include <cstdlib>

int main(int argc, char **argv) // objective, then lengths: per length whether on the line, workgroups
{
    for (int i = 2; i < argc; ++i) {
        smx::PertParams pp{};
        pp.obj = std::atoi(argv[1]);
        pp.B = 1;
        pp.n = std::atoll(argv[i]);
        std::printf("%d %d %d\n", (int)smx::phase_on_line(pp), smx::phase_grid(pp), smx::kTrialBlock);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                           os.path.join(PKG, "csrc"), "-o", str(d / "rules"), str(d / "rules.cpp"),
                           os.path.join(PKG, "libsmx.so"), "-Wl,-rpath," + PKG, "-L/opt/rocm/lib", "-lamdhip64"])

    def ask(obj, lengths):
        out = subprocess.check_output([str(d / "rules"), str(obj), *map(str, lengths)], text=True)
        return [tuple(map(int, line.split())) for line in out.split("\n") if line]

    return ask


@pytest.mark.parametrize("obj", [1, 4])  # squared norm, L1
def test_line_phase_index_stays_in_32_bits(rules, obj):
    """A launch on the line steps an int by workgroups x threads: from any
    entry it visits, the next step must still be an int."""
    last = 2 ** 31 - 1
    lengths = [1, 8193, 131072, 131073, 10 ** 8, last - 600000, last - 524288, last - 524287, last - 1, last]
    for n, (line, grid, block) in zip(lengths, rules(obj, lengths)):
        if line:
            assert (n - 1) + grid * block <= last, n
    assert rules(obj, [8193])[0][0] == 1
