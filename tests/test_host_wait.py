"""The host's wait for records in mapped memory (csrc/ilh_wait.h), compiled for the CPU and driven by a
scripted stream: the records, or the mark that their producer was given up, may become visible only
after the stream reports completion, and each ends the wait with its own outcome."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_16424_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "ilh_wait.h"
// argv: milliseconds after which the stream is done, the records arrive, the mark arrives (-1: never), and
// what the query then reports
int main(int, char** a) {
  using clock = std::chrono::steady_clock;
  const auto t0 = clock::now();
  auto after = [&](const char* ms) {
    return std::atof(ms) >= 0 && clock::now() - t0 >= std::chrono::duration<double, std::milli>(std::atof(ms));
  };
  const ilh::Waited w = ilh::wait_records([&] { return after(a[2]); }, [&] { return after(a[3]); },
                                          [&] { return after(a[1]) ? std::atoi(a[4]) : 0; });
  std::printf("%d\n", (int)w);
}
"""

ARRIVED, GIVEN_UP, MISSING, _, FAILED = range(5)


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("wait")
    (d / "wait.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(d / "wait.cpp"), "-o", str(d / "wait")], check=True)
    return str(d / "wait")


# the stream is done after 2 ms in the trailing cases: its first query after that starts the grace time
@pytest.mark.parametrize("done,records,mark,query,outcome", [
    ("-1", "0", "-1", "1", ARRIVED),
    ("-1", "20", "-1", "1", ARRIVED),
    ("-1", "-1", "20", "1", GIVEN_UP),
    ("2", "6", "-1", "1", ARRIVED),
    ("2", "-1", "6", "1", GIVEN_UP),
    ("2", "-1", "-1", "1", MISSING),
    ("2", "-1", "-1", "7", FAILED),
])
def test_outcome(program, done, records, mark, query, outcome):
    r = subprocess.run([program, done, records, mark, query], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and int(r.stdout) == outcome
