"""The gate that keeps apart the sections of several streams whose workgroups wait for one another (csrc/section_gate.h), compiled
with the host compiler against a runtime that writes down what it is asked for."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <string.h>
#include <string>
#include "paper_1802_07170_amd/csrc/section_gate.h"
static std::string said;
struct Rt {
  using Event = int; using Stream = int;
  static bool record(Event e, Stream st) { said += "R" + std::to_string(st) + "." + std::to_string(e) + " "; return true; }
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
  Gate::Client a{1}, b{2};
  const std::string what = argv[1];
  %s
  printf("no such case\n");
  return 1;
}
"""

CASES = {
    # one client's sections follow each other on its stream
    "alone": ("g.enter(a, 7); g.leave(a, 7); g.enter(a, 7); g.leave(a, 7);", "R7.1 R7.1 "),
    "two streams": ("g.enter(a, 7); g.leave(a, 7); g.enter(b, 8); g.leave(b, 8); g.enter(a, 7); g.leave(a, 7);", "R7.1 W8.1 R8.2 W7.2 R7.1 "),
    # one value for two streams: hipStreamPerThread of two threads, or a new stream in a destroyed one's place
    "one handle value": ("g.enter(a, 7); g.leave(a, 7); g.enter(b, 7); g.leave(b, 7);", "R7.1 W7.1 R7.2 "),
    # a client that goes is waited for, and then by nobody
    "gone": ("g.enter(a, 7); g.leave(a, 7); g.remove(a); g.enter(b, 7); g.leave(b, 7);", "R7.1 F1 R7.2 "),
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
