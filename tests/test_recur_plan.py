"""The shapes of the whole-recurrence kernels (csrc/recur_plan.h, compiled with the host compiler): workgroups that wait for one
another come in groups small enough that the launches a process can have in flight always finish on 256 CUs."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "paper_1802_07170_amd/csrc/recur_plan.h"
int main() {
  using namespace cmt;
  static_assert(SEQ_QUEUES * (SEQ_MAX_GROUP - 1) < 256, "four incomplete groups leave a CU free");
  for (int Hh = 8; Hh <= 1024; Hh += 8)                 // (the bottom layer's directions have half the hidden size)
    for (int prec = 0; prec < 2; ++prec)
      for (int ndir = 1; ndir <= 2; ++ndir)
        for (int Bp = 16; Bp <= 4096; Bp += Bp < 512 ? 16 : 512)
          for (int bwd = 0; bwd < 2; ++bwd) {
            const SeqPlan p = bwd ? seq_bwd_plan(prec, ndir, Bp, Hh) : seq_fwd_plan(prec, ndir, Bp, Hh);
            const int units = (bwd ? 16 : 4) * p.rt, k = bwd ? 4 * Hh : Hh;
            const bool ok = p.group <= SEQ_MAX_GROUP && p.group * units >= Hh && (p.group - 1) * units < Hh &&
                            p.ks * p.nk * 32 >= k && p.groups * p.bt * 16 >= ndir * Bp && p.ks + p.ne <= 16 && p.lk < p.nk &&
                            (prec || p.bt == 1 || p.nk < 4) && (!bwd || 4 * p.rt % p.ne == 0);
            if (!ok) { printf("%d %d %d %d %d: group %d\n", Hh, prec, ndir, Bp, bwd, p.group); return 1; }
          }
  return 0;
}
"""


def test_groups_that_wait_for_one_another_are_small_enough(tmp_path):
    src = tmp_path / "plan.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "plan"
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", f"-I{ROOT}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


PITCH_PROGRAM = r"""
#include "paper_1802_07170_amd/csrc/row_pitch.h"
int main() {
  using namespace cmt;
  int bad = 0;
  for (int H = 16; H <= 1024; H += 16)
    for (int E = 8; E <= 1024; E += 8)
      for (int prec = 0; prec < 2; ++prec) {
        const RowPitch p = row_pitch(prec, E, H, true), q = row_pitch(prec, E, H, false);
        const bool copies = prec && H % 32 == 0;         // what api.hip's layout makes fragment-major copies of
        const bool fed = copies && E % 32 == 0, bottom = copies && (E + H) % 16 == 0;
        bad += (p.states != ACT_PAD && !fed) + (p.gates_bottom != ACT_PAD && !bottom) + (p.gates != ACT_PAD && !copies);
        bad += H == 1024 && E == 1024 && prec && (p.states != ACT_PAD_LINES || p.gates != ACT_PAD_LINES || p.gates_bottom != ACT_PAD_LINES);
        bad += q.states != ACT_PAD || q.gates != ACT_PAD || q.gates_bottom != ACT_PAD;
      }
  return bad != 0;
}
"""


def test_rows_that_a_position_reads_are_never_padded_to_whole_lines(tmp_path):
    """Whole cache lines only for rows of which the kernels of a position read fragment-major copies."""
    src = tmp_path / "pitch.cpp"
    src.write_text(PITCH_PROGRAM)
    exe = tmp_path / "pitch"
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", f"-I{ROOT}", str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
