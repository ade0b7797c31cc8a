"""The host threads of a pass over a batch (csrc/host_team.h), compiled for the CPU: phases stay in step, an exception of
one thread ends the others' waits and reaches the caller, and threads that wait long do not burn processor time."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1611_03404_amd", "csrc")

MAIN = r"""
#include "host_team.h"
#include <chrono>
#include <cstdio>
#include <cstring>
#include <ctime>
#include <new>
using namespace celeste;
#define NEED(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main(int argc, char** argv) {
  if (!std::strcmp(argv[1], "phases")) {
    for (int rep = 0; rep < 50; ++rep)
      for (int nt : {1, 2, 3, 7, TEAM_MAX}) {
        std::vector<int> sum(TEAM_MAX, 0), seen(TEAM_MAX, 0);
        team(nt, [&](int t, int n, Barrier& bar) {
          for (int phase = 0; phase < 20; ++phase) {
            sum[t] += phase;
            bar.wait();
            int all = 0;
            for (int k = 0; k < n; ++k) all += sum[k];
            if (all == n * phase * (phase + 1) / 2) ++seen[t];
            bar.wait();
          }
        });
        for (int t = 0; t < nt; ++t) NEED(seen[t] == 20);
      }
    const auto first = [](int64_t n, int64_t at) { return first_failure(n, 100, [&](int64_t i) { return i < at; }); };
    for (int64_t n : {1, 2047, 4096, 100000}) NEED(first(n, n) == n && first(n, n / 2) == n / 2 && first(n, 0) == 0);
    return 0;
  }
  if (!std::strcmp(argv[1], "throw")) {
    for (int who : {0, 1, 3})
      for (int barriers : {0, 1, 2}) {
        bool caught = false;
        try {
          team(4, [&](int t, int, Barrier& bar) {
            for (int k = 0; k < barriers; ++k) bar.wait();
            if (t == who) throw std::bad_alloc();
            bar.wait();
          });
        } catch (const std::bad_alloc&) {
          caught = true;
        }
        NEED(caught);
      }
    return 0;
  }
  // "idle": three threads wait 0.4 s for the fourth
  const std::clock_t c = std::clock();
  team(4, [&](int t, int, Barrier& bar) {
    if (t == 0) std::this_thread::sleep_for(std::chrono::milliseconds(400));
    bar.wait();
  });
  const double used = double(std::clock() - c) / CLOCKS_PER_SEC;
  std::printf("processor time %.3f s\n", used);
  NEED(used < 0.2);
  return 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("team")
    (d / "main.cpp").write_text(MAIN)
    out = str(d / "team")
    subprocess.run([cxx, "-std=c++17", "-O2", "-pthread", "-I", CSRC, str(d / "main.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("what", ["phases", "throw", "idle"])
def test_team(exe, what):
    r = subprocess.run([exe, what], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
