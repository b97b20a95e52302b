"""The rules that send a perturbation phase to its kernels, asked of the built
library on the host: the line form against what its 32-bit index can walk, and
the tiles of the TV phase."""
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


def _compile(d, text):
    (d / "rules.cpp").write_text(text)
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                           os.path.join(PKG, "csrc"), "-o", str(d / "rules"), str(d / "rules.cpp"),
                           os.path.join(PKG, "libsmx.so"), "-Wl,-rpath," + PKG, "-L/opt/rocm/lib", "-lamdhip64"])


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    _compile(d, PROGRAM)

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


@pytest.mark.parametrize("B,rows,cols,grid", [
    (1, 64, 64, 16), (1, 1000, 1000, 3969),
    (32, 64, 64, 16), (8, 128, 128, 64), (2, 256, 256, 256), (4, 33, 21, 6),    # up to 512 (tile, slice) pairs
    (32, 80, 64, 160), (16, 81, 90, 246), (8, 130, 130, 297), (2, 257, 250, 272), (32, 256, 256, 256),
])
def test_tv_tiles_by_resident_workgroups(tv_grid, B, rows, cols, grid):
    """16 x 16 tiles, a workgroup a slice, while all (tile, slice) pairs are
    resident at once; beyond, whole lines in tiles halved until there are 256."""
    assert tv_grid(B, rows, cols) == grid


@pytest.fixture(scope="module")
def tv_grid(tmp_path_factory):
    d = tmp_path_factory.mktemp("tv")
    body = PROGRAM[:PROGRAM.index("int main")] + r"""
int main(int, char **argv)
{
    smx::PertParams pp{};
    pp.obj = 2;
    pp.B = std::atoi(argv[1]);
    pp.tv_rows = std::atoi(argv[2]);
    pp.tv_cols = std::atoi(argv[3]);
    pp.n = (long long)pp.tv_rows * pp.tv_cols;
    std::printf("%d\n", smx::phase_grid(pp));
    return 0;
}
"""
    _compile(d, body)
    return lambda B, r, c: int(subprocess.check_output([str(d / "rules"), str(B), str(r), str(c)], text=True))
