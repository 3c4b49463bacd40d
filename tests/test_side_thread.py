"""The thread that enqueues the depth network beside the worker
(csrc/side_thread.h), compiled for the host with g++: both tasks run at once,
either one's error reaches the caller, and a process that can start no thread
runs them in turn instead of ending."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2604_27441_amd", "csrc", "side_thread.h")

PROGRAM = r"""
#include "%s"
#include <sys/resource.h>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#define CHECK(x) do { if (!(x)) { printf("line %%d: %%s\n", __LINE__, #x); return 1; } } while (0)

int main(int argc, char** argv) {
  const bool limited = argc > 1 && !strcmp(argv[1], "limited");
  if (limited) {  // no address space for another stack
    rlimit l;
    getrlimit(RLIMIT_AS, &l);
    FILE* f = fopen("/proc/self/statm", "r");
    long pages = 0;
    CHECK(f && fscanf(f, "%%ld", &pages) == 1);
    fclose(f);
    l.rlim_cur = pages * 4096 + (1 << 20);
    CHECK(setrlimit(RLIMIT_AS, &l) == 0);
  }
  revo::SideThread t;
  std::atomic<int> inits{0}, calls{0};
  CHECK(t.start([&] { ++inits; }) == !limited);
  for (int i = 0; i < 1000; ++i) {
    CHECK(t.run([&] { ++calls; return 0; }, [&] { ++calls; return 0; }) == 0);
    CHECK(calls == 2 * (i + 1));
    CHECK(t.run([&] { return 0; }, [&] { return -5; }) == -5);
    CHECK(t.run([&] { return -7; }, [&] { return 0; }) == -7);
    CHECK(t.run([&] { return -7; }, [&] { return -5; }) == -5);
  }
  CHECK(inits == !limited);
  if (!limited) {
    // each task waits for the other to have begun
    std::atomic<int> begun{0};
    auto meet = [&] { ++begun; while (begun < 2) std::this_thread::yield(); return 0; };
    CHECK(t.run(meet, meet) == 0);
  }
  t.stop();
  t.stop();
  CHECK(t.run([&] { return 0; }, [&] { return -5; }) == -5);  // stopped: in turn
  puts("ok");
  return 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("side")
    (d / "t.cpp").write_text(PROGRAM % HEADER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    str(d / "t.cpp"), "-o", str(d / "t")], check=True)
    return str(d / "t")


@pytest.mark.parametrize("mode", ["threads", "limited"])
def test_two_tasks(exe, mode):
    r = subprocess.run([exe, mode], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout, r.stderr)
