"""Host-side device bookkeeping of the launchers (csrc/device.h), compiled for the CPU with the system compiler."""
import os
import re

from host_cpp import CSRC, compile_cpp, run


ONCE = r"""
#include <chrono>
#include <cstdio>
#include <thread>
#include "device.h"
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s\n", #x); return 1; } } while (0)
int main() {
  // a second thread arrives while the first is still setting: it may not go on before a set has been completed
  ppll::OncePerDevice once;
  std::atomic<bool> entered{false}, second_back{false};
  std::atomic<int> completed{0};
  std::thread first([&] {
    once(0, [&] {
      entered = true;
      for (int i = 0; i < 2000 && !second_back; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(1));
      ++completed;
      return 0;
    });
  });
  while (!entered) std::this_thread::yield();
  const int status = once(0, [&] { ++completed; return 0; });
  const int completed_before_second_went_on = completed;
  second_back = true;
  first.join();
  CHECK(status == 0 && completed_before_second_went_on >= 1);
  // done: not set again; another device on its own; a failure is reported and tried again
  int calls = 0;
  CHECK(once(0, [&] { ++calls; return 0; }) == 0 && calls == 0);
  CHECK(once(1, [&] { ++calls; return 7; }) == 7 && calls == 1);
  CHECK(once(1, [&] { ++calls; return 0; }) == 0 && calls == 2);
  CHECK(once(1, [&] { ++calls; return 0; }) == 0 && calls == 2);
  // devices beyond the table are set every time
  for (int dev : {-1, ppll::MAX_DEVICES}) {
    calls = 0;
    once(dev, [&] { ++calls; return 0; });
    once(dev, [&] { ++calls; return 0; });
    CHECK(calls == 2);
  }
  return 0;
}
"""


def test_a_kernel_attribute_counts_as_raised_only_once_it_is(tmp_path):
    run(compile_cpp(tmp_path, ONCE))


PER_DEVICE = r"""
#include <cstdio>
#include "device.h"
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s\n", #x); return 1; } } while (0)
int main() {
  ppll::PerDevice units;
  int asked = 0;
  for (int i = 0; i < 3; ++i) CHECK(units(0, [&] { ++asked; return 256; }) == 256);
  CHECK(asked == 1);
  CHECK(units(1, [&] { return 0; }) == 0);          // no answer: asked again
  CHECK(units(1, [&] { return 304; }) == 304);
  CHECK(units(0, [&] { return 1; }) == 256);
  CHECK(units(ppll::MAX_DEVICES, [&] { return 2; }) == 2 && units(ppll::MAX_DEVICES, [&] { return 3; }) == 3);
  return 0;
}
"""


def test_a_device_is_asked_for_its_compute_units_once(tmp_path):
    run(compile_cpp(tmp_path, PER_DEVICE))
    asking = [f for f in os.listdir(CSRC) if "hipDeviceAttributeMultiprocessorCount" in open(os.path.join(CSRC, f)).read()]
    assert asking == ["k_dispatch.hip"]


def test_the_lds_attribute_is_raised_in_one_place_to_a_size_of_the_kernel_alone():
    places, raised = [], []
    for f in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, f)).read()
        places += [f] * text.count("hipFuncSetAttribute(")
        raised += [(f, m) for m in re.findall(r"raise_lds\(\(const void\*\)[^;]*?, (?:\(int\))?([^;]*), \w+(?:\[\d\])?\)\)?;", text)]
    assert places == ["k_dispatch.hip"]
    # a size handed to the launch at hand is called lds; the matrix-core attention's is a function of its template argument
    assert len(raised) >= 15
    assert {f for f, m in raised if m == "lds"} <= {"k_attn_mfma.hip"}, raised


def test_a_bare_barrier_is_a_barrier_for_the_compiler_too():
    # the builtin orders execution only; pipe::barrier() holds the accesses on either side of it in place
    ordered = 'asm volatile("" ::: "memory");\n  __builtin_amdgcn_s_barrier();\n  asm volatile("" ::: "memory");\n'
    bare = []
    for f in sorted(os.listdir(CSRC)):
        if os.path.isfile(os.path.join(CSRC, f)):
            text = open(os.path.join(CSRC, f)).read()
            bare += [f] * (text.count("__builtin_amdgcn_s_barrier()") - text.count(ordered))
    assert bare == []
