"""Host loops on several threads: an exception in a thread, and threads that
cannot be started, end neither the process nor the loop's account of itself."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1505_04340_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <sys/resource.h>
#include "slr_threads.h"

static long resident_limit() {   // address space in use
  long pages = 0;
  FILE *f = std::fopen("/proc/self/statm", "r");
  if (!f || std::fscanf(f, "%ld", &pages) != 1) std::exit(3);
  std::fclose(f);
  return pages * 4096;
}

int main(int argc, char **argv) {
  const bool few = argc > 1 && !std::strcmp(argv[1], "few");
  if (few) {   // no room for another stack
    const rlim_t n = (rlim_t)resident_limit() + (1 << 20);
    const rlimit r{n, n};
    if (setrlimit(RLIMIT_AS, &r)) return 4;
  }
  std::atomic<int> done{0};
  if (!slr::run_parallel(1000, 8, [&](int) { ++done; }) || done != 1000) return 5;
  done = 0;
  if (slr::run_parallel(1000, 8, [&](int i) { if (i == 17) throw std::bad_alloc(); ++done; }) || done > 999) return 6;
  if (!slr::run_parallel(0, 8, [&](int) { std::abort(); })) return 7;
  std::puts("ok");
  return 0;
}
"""


def test_exceptions_and_missing_threads(tmp_path):
    src = tmp_path / "t.cpp"
    src.write_text(MAIN)
    exe = str(tmp_path / "t")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", exe])
    for mode in ("many", "few"):
        r = subprocess.run([exe, mode], capture_output=True, text=True, timeout=60)
        assert (r.returncode, r.stdout.strip()) == (0, "ok"), (mode, r)
