"""Function attributes belong to a device: the large dynamic LDS of a kernel is asked for on every device that
it runs on, not on the first one alone."""
import glob
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1601_06767_amd", "csrc")

PROGRAM = r"""
#include <cassert>
#include <thread>
#include <vector>
#include "per_device.h"
enum Status { kOk = 0, kBad = 1 };
int main() {
  gw::OncePerDevice done;
  int calls = 0;
  auto good = [&] { ++calls; return kOk; };
  assert(done.run(0, good) == kOk && calls == 1);
  assert(done.run(0, good) == kOk && calls == 1);    // known
  assert(done.run(3, [&] { ++calls; return kBad; }) == kBad && calls == 2);
  assert(done.run(3, good) == kOk && calls == 3);    // another device, and again after a failure
  assert(done.run(3, good) == kOk && calls == 3);
  for (int i = 0; i < 2; ++i) assert(done.run(64, good) == kOk && calls == 4 + i);   // beyond the bits: each time
  gw::OncePerDevice shared;
  std::atomic<int> sets{0};
  std::vector<std::thread> t;
  for (int i = 0; i < 8; ++i)
    t.emplace_back([&, i] { assert(shared.run(i % 2, [&] { ++sets; return kOk; }) == kOk); });
  for (auto& x : t) x.join();
  assert(sets >= 2);
  const int before = sets;
  for (int d = 0; d < 2; ++d) shared.run(d, [&] { ++sets; return kOk; });
  assert(sets == before);
}
"""


def test_set_up_runs_once_on_every_device(tmp_path):
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    subprocess.run([str(exe)], check=True, timeout=60)


def test_every_function_attribute_is_set_per_device():
    for path in glob.glob(os.path.join(CSRC, "*")):
        text = open(path).read()
        n = text.count("hipFuncSetAttribute")
        assert n == (1 if os.path.basename(path) == "internal.h" else 0), path
