"""The order of a one-workgroup phase's reads, writes and barriers, run on the
host: the loop of csrc/phase_rounds.h with a thread a wave, against a schedule
that holds every wave but the first before each of its reads of shared state
until wave 0 waits at its next barrier or has left.  Whatever wave 0 writes
before a barrier is then seen by a read that no barrier orders before it.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "phase_rounds.h"
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <thread>
#include <vector>

constexpr int W = 4;
std::mutex mu;
std::condition_variable cv;
int at_barrier = 0, ended = 0, generation = 0;
bool first_waits = false, first_gone = false;
thread_local int wave;
thread_local int barriers, sums;

void barrier()
{
    std::unique_lock<std::mutex> lk(mu);
    ++barriers;
    const int g = generation;
    if (wave == 0) first_waits = true;
    cv.notify_all();
    if (++at_barrier + ended == W) { // a wave that has ended counts as arrived, as the hardware's barrier has it
        at_barrier = 0;
        ++generation;
        first_waits = false;
        cv.notify_all();
    } else {
        cv.wait(lk, [&] { return generation != g; });
    }
}

void leave()
{
    std::unique_lock<std::mutex> lk(mu);
    if (wave == 0) first_gone = true;
    if (at_barrier + ++ended == W && at_barrier) {
        at_barrier = 0;
        ++generation;
        first_waits = false;
    }
    cv.notify_all();
}

struct Shared { // a word of LDS
    int v = 0;
    Shared &operator=(int x)
    {
        std::lock_guard<std::mutex> lk(mu);
        v = x;
        return *this;
    }
    operator int()
    {
        std::unique_lock<std::mutex> lk(mu);
        if (wave != 0) cv.wait(lk, [] { return first_waits || first_gone; });
        return v;
    }
} todo, phase;

std::vector<int> script; // what decide() returns, 0 last
size_t next_round = 0;

int decide()
{
    const int n = script[next_round++];
    if (n == 0) phase = 0; // the phase is over
    return n;
}
void sum(int)
{
    ++sums;
    barrier();
}

// the planted mistake: the loop goes by the phase's state, read at its head
void by_state()
{
    while (phase) {
        if (wave == 0) todo = decide();
        barrier();
        const int n = todo;
        if (n > 0) sum(n);
        barrier();
    }
}

int main(int argc, char **argv)
{
    const bool planted = std::atoi(argv[1]) != 0;
    for (int i = 2; i < argc; ++i) script.push_back(std::atoi(argv[i]));
    script.push_back(0);
    phase.v = 1;
    std::vector<std::thread> t;
    int b[W], s[W];
    for (int w = 0; w < W; ++w)
        t.emplace_back([&, w] {
            wave = w;
            if (planted) by_state();
            else smx::phase_rounds(wave == 0, todo, decide, sum, barrier);
            b[w] = barriers;
            s[w] = sums;
            leave();
        });
    for (auto &x : t) x.join();
    for (int w = 0; w < W; ++w) std::printf("%d %d\n", b[w], s[w]);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("rounds")
    (d / "rounds.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-D__device__=", "-I",
                           os.path.join(ROOT, "paper_2606_27086_amd", "csrc"), "-o", str(d / "rounds"),
                           str(d / "rounds.cpp")])
    return str(d / "rounds")


def waves(program, planted, script):
    out = subprocess.run([program, str(int(planted)), *map(str, script)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0
    return [tuple(map(int, line.split())) for line in out.stdout.split("\n") if line]


@pytest.mark.parametrize("script", [[], [8], [8, 8, 3], [1, 8, 8, 8, 8]])
def test_every_wave_takes_the_same_rounds(program, script):
    """No rounds to sum, one, several: each wave passes the barriers the first
    one passes (one and those of the sums for each round, one to end)."""
    assert waves(program, False, script) == [(3 * len(script) + 1, len(script))] * 4


@pytest.mark.parametrize("script", [[], [8, 8]])
def test_the_schedule_shows_a_late_read(program, script):
    """A loop that goes by the state wave 0 writes loses the late waves."""
    got = waves(program, True, script)
    assert any(g != got[0] for g in got[1:]), got
