"""The gate that keeps apart the sections of several streams whose workgroups wait for one another (csrc/section_gate.h), compiled
with the host compiler against a runtime that writes down what it is asked for."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <atomic>
#include <chrono>
#include <string>
#include <thread>
#include "paper_1802_07170_amd/csrc/section_gate.h"
static std::string said, order = "..";
static bool broken = false;
struct Rt {
  using Event = int; using Stream = int;
  static bool record(Event e, Stream st) { if (broken) return false; said += "R" + std::to_string(st) + "." + std::to_string(e) + " "; return true; }
  static void wait(Stream st, Event e) { said += "W" + std::to_string(st) + "." + std::to_string(e) + " "; }
  static void finish(Event e) { said += "F" + std::to_string(e) + " "; }
};
using Gate = cmt::SectionGate<Rt>;
static int check(const char* what, const char* want) {
  const bool ok = said == want;
  if (!ok) printf("%s: %s (expected %s)\n", what, said.c_str(), want);
  said.clear();
  return ok ? 0 : 1;
}
int main(int argc, char** argv) {
  Gate g;
  Gate::Client a, b, c, d;
  a.alone = 1; a.shared = 2; b.alone = 3; b.shared = 4; c.alone = 5; c.shared = 6; d.alone = 7; d.shared = 8;
  auto in = [&](Gate::Client& who, int stream, bool alone) { g.enter(who, stream, alone); g.leave(who, stream, alone); };
  const std::string what = argv[1];
  %s
  printf("no such case\n");
  return 1;
}
"""

CASES = {
    # one client's sections follow each other on its stream
    "one client": ("in(a, 7, 1); in(a, 7, 0); in(a, 7, 1);", "R7.1 R7.2 R7.1 "),
    "two streams": ("in(a, 7, 1); in(b, 8, 1); in(a, 7, 1);", "R7.1 W8.1 R8.3 W7.3 R7.1 "),
    # one value for two streams: hipStreamPerThread of two threads, or a new stream in a destroyed one's place
    "one handle value": ("in(a, 7, 1); in(b, 7, 1);", "R7.1 W7.1 R7.3 "),
    # sections that may share the chip do not wait for one another ...
    "shared": ("in(a, 7, 0); in(b, 8, 0); in(c, 9, 0); in(a, 7, 0);", "R7.2 R8.4 R9.6 R7.2 "),
    # ... but for the last one that ran alone, and the next one alone waits for each of them, once
    "shared after alone": ("in(a, 7, 1); in(b, 8, 0); in(c, 9, 0);", "R7.1 W8.1 R8.4 W9.1 R9.6 "),
    "alone after shared": ("in(a, 7, 0); in(b, 8, 0); in(a, 7, 0); in(c, 9, 1); in(d, 6, 1);", "R7.2 R8.4 R7.2 W9.2 W9.4 R9.5 W6.5 R6.7 "),
    "own shared one before alone": ("in(a, 7, 0); in(b, 8, 0); in(a, 7, 1); in(b, 8, 0);", "R7.2 R8.4 W7.4 R7.1 W8.1 R8.4 "),
    # an end that could not be recorded: the ones before it are still waited for
    "not recorded": ("in(a, 7, 0); broken = true; in(b, 8, 1); broken = false; in(c, 9, 1);", "R7.2 W8.2 W9.2 R9.5 "),
    # a client that goes is waited for, and then by nobody
    "gone": ("in(a, 7, 1); in(a, 7, 0); g.add(a, 7); g.add(b, 8); if (g.crowded(b)) g.remove(a); if (!g.crowded(b)) in(b, 7, 1);", "R7.1 R7.2 F2 F1 R7.3 "),
    # several clients on one stream follow each other: nobody there has a use for shorter sections
    "crowded": ("g.add(a, 7); g.add(b, 7); if (!g.crowded(a) && !g.crowded(b)) said += 'n'; g.add(c, 8); for (auto* p : {&a, &b, &c}) if (g.crowded(*p)) said += 'y'; "
                "g.remove(a); if (g.crowded(b)) said += 'y';", "nyyyF2 F1 y"),
    # on the host: two shared sections open at once; one alone is enqueued when both are closed, and before a third
    "order on the host": ("""
      g.enter(a, 7, false); g.enter(b, 8, false);
      std::atomic<int> n{0};
      std::thread t1([&] { g.enter(c, 9, true); order[n++] = 'C'; g.leave(c, 9, true); });
      std::this_thread::sleep_for(std::chrono::milliseconds(100));
      std::thread t2([&] { g.enter(d, 6, false); order[n++] = 'D'; g.leave(d, 6, false); });
      std::this_thread::sleep_for(std::chrono::milliseconds(100));
      if (n != 0) { printf("not kept out\\n"); return 1; }
      g.leave(a, 7, false); g.leave(b, 8, false);
      t1.join(); t2.join();
      said = order;""", "CD"),
}


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("gate")
    cases = "".join(f'if (what == "{k}") {{ {code} return check("{k}", "{want}"); }}\n' for k, (code, want) in CASES.items())
    (d / "gate.cpp").write_text(PROGRAM.replace("  %s\n", cases))
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-pthread", f"-I{ROOT}", str(d / "gate.cpp"), "-o", str(d / "gate")], check=True)
    return str(d / "gate")


@pytest.mark.parametrize("case", CASES)
def test_who_waits_for_whom(exe, case):
    r = subprocess.run([exe, case], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
