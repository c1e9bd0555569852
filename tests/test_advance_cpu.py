"""How a call of n steps is split into launches (csrc/advance.hpp), compiled
for the host: a captured graph is replayed whenever its steps remain, also
after calls that left the populations in the other buffer, and launches of
two steps never go past a guard poll."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "advance.hpp"
// argv: graph steps, poll interval, steps of the calls; two steps a launch.
// Per call: replays, launches, polls, steps taken, buffer at the end.
int main(int argc, char** argv) {
  const int graph = atoi(argv[1]), every = atoi(argv[2]);
  int cur = 0;
  for (int i = 3; i < argc; ++i) {
    int replays = 0, launches = 0, polls = 0, taken = 0, since = 0;
    const int st = mlf::advance(
        atoi(argv[i]), every, graph, [&](long left) { return left >= 2 ? 2 : 1; },
        [&]() { ++replays; taken += graph; since += graph; return 0; },
        [&](int n) {
          ++launches; cur ^= 1; taken += n; since += n;
          return every > 0 && since > every ? 7 : 0;  // went past a poll
        },
        [&]() { ++polls; since = 0; return 0; });
    if (st) return st;
    printf("%d %d %d %d %d\n", replays, launches, polls, taken, cur);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("advance")
    (d / "main.cpp").write_text(SOURCE)
    exe = str(d / "main")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2409_16659_amd", "csrc"),
                    "-o", exe, str(d / "main.cpp")], check=True)
    return exe


def _run(program, graph, every, calls):
    r = subprocess.run([program, str(graph), str(every), *map(str, calls)], capture_output=True, text=True, check=True)
    return [tuple(map(int, line.split())) for line in r.stdout.splitlines()]


@pytest.mark.parametrize("every", [0, 4, 5])
@pytest.mark.parametrize("calls", [[2, 8, 8, 8], [1, 8, 8], [3, 20, 8, 5, 16], [8, 2, 2, 8, 6, 9]])
def test_graph_is_replayed_whenever_its_steps_remain(program, every, calls):
    for n, (replays, launches, _, taken, _) in zip(calls, _run(program, 8, every, calls)):
        assert taken == n
        assert replays == n // 8
        assert (launches == 0) == (n % 8 == 0)


def test_launches_end_at_guard_polls(program):
    for every in (1, 2, 3, 7):
        for n, (replays, launches, polls, taken, _) in zip((1, 6, 15), _run(program, 0, every, (1, 6, 15))):
            assert (replays, taken) == (0, n)
            assert polls == (n - 1) // every
            full, rest = divmod(n, every)
            assert launches == full * ((every + 1) // 2) + (rest + 1) // 2
