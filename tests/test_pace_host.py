"""How far a blocking solve enqueues ahead of the device (csrc/pace.hpp), on the CPU:
the loop of the blocking solve, two quanta in flight and one read at a time, on
residuals whose course is known."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_15411_amd", "csrc")

HARNESS = r"""
#include "pace.hpp"
#include <cstdio>
#include <cstdlib>
#include <deque>
// args: tol every warm eta1 rate max_iter long_iter; prints iterations done, enqueued, reads
int main(int, char** v) {
  const double tol = atof(v[1]), eta1 = atof(v[4]), rate = atof(v[5]);
  const int every = atoi(v[2]), warm = atoi(v[3]), max_iter = atoi(v[6]);
  cbs::Pace pace(tol, every, warm != 0, atoi(v[7]) != 0);
  std::deque<int> flight;   // last iteration of each quantum in flight
  int enqueued = 0, read = 0, reads = 0, done = 0, iter = 0;
  double eta = eta1 / rate;
  while (!done) {
    while (flight.size() < 2 && enqueued < max_iter) {
      int q = pace.next(enqueued - read);
      if (q == 0) break;
      if (q < 0 || q > every) return 2;
      if (q > max_iter - enqueued) q = max_iter - enqueued;
      flight.push_back(enqueued += q);
    }
    if (flight.empty()) return 3;   // nothing to wait for: the solve would not end
    while (!done && iter < flight.front()) {
      ++iter;
      eta *= rate;
      done = eta <= tol || iter >= max_iter;
    }
    flight.pop_front();
    ++reads;
    read = iter;
    pace.read(iter, eta);
  }
  printf("%d %d %d\n", iter, enqueued, reads);
  return 0;
}
"""


@pytest.fixture(scope="module")
def pace(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("pace")
    (d / "h.cpp").write_text(HARNESS)
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                        str(d / "h.cpp"), "-o", str(d / "h")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(tol, every, warm, eta1, rate, max_iter=100000, long_iter=False):
        r = subprocess.run([str(d / "h"), repr(tol), str(every), str(int(warm)), repr(eta1),
                            repr(rate), str(max_iter), str(int(long_iter))],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.returncode
        return tuple(int(x) for x in r.stdout.split())
    return run


@pytest.mark.parametrize("every", [1, 3, 10, 20, 64])
@pytest.mark.parametrize("n", [1, 2, 5, 11, 20, 39, 41, 63, 150, 871])
@pytest.mark.parametrize("warm", [False, True])
def test_converging_solves_leave_little_behind(pace, every, n, warm):
    """A residual that falls steadily to tol at iteration n: past it there is less
    than a quarter of a quantum (one quantum while a cold start has shown fewer
    than two residuals), not two quanta."""
    rate = 1e-4 ** (1.0 / n) * 0.999999
    done, enqueued, reads = pace(1e-4, every, warm, rate, rate)
    assert done == n
    least = max(1, every // 4)
    unknown = 2 * least if warm else 2 * every
    assert enqueued - n < (every if not warm and n <= unknown else least + 1)
    # a quantum stays check_every iterations long while the end is far
    assert reads <= -(-n // every) + (5 if n > unknown else 3)


@pytest.mark.parametrize("every", [1, 10, 20, 64])
@pytest.mark.parametrize("n", [45, 63, 150, 160, 871])
def test_long_iterations_end_on_the_spot(pace, every, n):
    """Where an iteration outlasts a reading the last ones are enqueued one by one:
    at most one behind a steady residual, and few reads for it."""
    if n <= 2 * every:
        pytest.skip("fewer than two residuals read")
    rate = 1e-4 ** (1.0 / n) * 0.999999
    done, enqueued, reads = pace(1e-4, every, False, rate, rate, long_iter=True)
    assert done == n and enqueued - n <= 1
    assert reads <= -(-n // every) + 3


@pytest.mark.parametrize("tol,rate", [(0.0, 0.9), (0.0, 1.0), (1e-4, 1.0), (1e-4, 1.001)])
def test_solves_that_do_not_converge_keep_two_quanta(pace, tol, rate):
    """tol = 0, a stalled and a growing residual: max_iter iterations in quanta of
    check_every, none more."""
    done, enqueued, reads = pace(tol, 10, False, 1.0, rate, 237)
    assert (done, enqueued, reads) == (237, 237, 24)


def test_a_residual_that_slows_down_is_not_polled_every_iteration(pace):
    """An estimate that keeps falling short costs a read per quarter quantum at most."""
    done, enqueued, reads = pace(1e-4, 20, False, 1.0, 0.9999, 200000)
    assert done == 92099 or abs(done - 92099) < 3
    assert enqueued - done <= 6 and reads < done // 20 + 10
