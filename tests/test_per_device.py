"""What is asked of a device once is asked of every device, and again after a failure: the helper (a C++ program with
devices that are made up), and that every launch that needs more LDS goes through it."""
import os
import subprocess

from paper_2605_09877_amd import build

PROGRAM = r"""
#include <cassert>
#include <initializer_list>
#include "per_device.h"
enum Err { kOk = 0, kLost, kRefused };
int main() {
  kvm::OncePerDevice<Err> once, other;
  int device = 0, asked = 0;
  Err where = kOk, answer = kOk;
  auto call = [&](kvm::OncePerDevice<Err> &o) {
    return o([&](int *d) { *d = device; return where; }, [&] { ++asked; return answer; });
  };
  answer = kRefused;                                   // a failure is reported and not kept
  assert(call(once) == kRefused && asked == 1);
  answer = kOk;
  assert(call(once) == kOk && asked == 2);
  assert(call(once) == kOk && asked == 2);             // what was granted is
  device = 1;                                          // by that device alone
  answer = kRefused;
  assert(call(once) == kRefused && asked == 3);
  answer = kOk;
  assert(call(once) == kOk && asked == 4 && call(once) == kOk && asked == 4);
  device = 0;
  assert(call(once) == kOk && asked == 4);
  assert(call(other) == kOk && asked == 5);            // and for that thing
  where = kLost;
  assert(call(once) == kLost && asked == 5);
  where = kOk;
  for (int d : {63, 64, 1000, -1}) {                   // beyond the ones remembered: every time
    device = d;
    const int before = asked;
    assert(call(once) == kOk && call(once) == kOk && asked == before + (d == 63 ? 1 : 2));
  }
}
"""


def test_every_device_is_asked_and_failures_are_not_kept(tmp_path):
    src, exe = tmp_path / "once.cpp", tmp_path / "once"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    subprocess.run([str(exe)], check=True, timeout=60)


def test_lds_is_asked_for_in_one_place():
    uses = {}
    for name in sorted(os.listdir(build.CSRC)):
        with open(os.path.join(build.CSRC, name)) as f:
            uses[name] = f.read().count("hipFuncSetAttribute")
    assert {name for name, n in uses.items() if n} == {"kvm_internal.h"}, uses
