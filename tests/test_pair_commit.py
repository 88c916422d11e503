"""A transition's table updates beside its data (csrc/pair_commit.h), built with
the host compiler: a tile of the pair that reads the table entry, and the freed
block, at any point between the committing workgroup's accesses finds the
pair's blocks."""

import os
import shutil
import subprocess

import pytest

from paper_2609_33536_amd import build

SOURCE = r"""
#include <cstdio>
#include <vector>
#include "pair_commit.h"

struct State { int entry, freed; };
// The committing workgroup: its writes make the states that other tiles can see.
struct Committer {
  std::vector<State>& states;
  int load_entry() { return states.back().entry; }
  int load_freed() { std::puts("the committing workgroup read freed"); return -7; }
  void store_freed(int v) { states.push_back({states.back().entry, v}); }
  void store_entry(int v) { states.push_back({v, states.back().freed}); }
};
// Another tile: its accesses see the state at the points given for them.
struct Tile {
  const std::vector<State>& states;
  const size_t entry_at, freed_at;
  int load_entry() { return states[entry_at].entry; }
  int load_freed() { return states[freed_at].freed; }
  void store_freed(int) { std::puts("another tile wrote freed"); }
  void store_entry(int) { std::puts("another tile wrote the entry"); }
};

int main() {
  int bad = 0, late = 0;
  const int nb = 10;
#ifdef ENTRY_FIRST   // a committer in the wrong order, which the walk has to find
  const bool entry_first = true;
#else
  const bool entry_first = false;
#endif
  for (int b0 : {-1, 0, 3, 9, 10})
    for (int e : {-1, 0, 4, 9, 10})
      for (int stale : {-1, 0, 7, 12345678}) {   // what freed[i] held before the call
        if (b0 == e && b0 >= 0 && b0 < nb) continue;   // (not a TARGET pair)
        std::vector<State> states{{e, stale}};
        Committer c{states};
        int got = -5;
        if (entry_first) c.store_entry(b0), states[0].entry = e;
        const bool valid = b0 >= 0 && b0 < nb && e >= 0 && e < nb;
        bool ok = true;
        if (entry_first) c.store_freed(e), ok = valid;
        else ok = ekv::demotion_block(c, true, b0, nb, got);
        if (!entry_first && (ok != valid || (ok && got != e) || states.back().freed != (valid ? e : -1))) ++bad;
        if (ok && !entry_first) c.store_entry(b0);
        if (!entry_first && states.back().entry != (valid ? b0 : e)) ++bad;
        for (size_t p = 0; p < states.size(); ++p)
          for (size_t q = p; q < states.size(); ++q) {
            Tile t{states, p, q};
            int b1 = -5;
            const bool on = ekv::demotion_block(t, false, b0, nb, b1);
            if (on != valid || (on && b1 != e)) ++bad;
            late += on && states[p].entry == b0;
          }
      }
  // refinement: before the update the entry is the packed block, after it the new one
  for (int bp : {-1, 0, 9, 10})
    for (int e : {-1, 0, 9, 10})
      for (int bq : {-1, 0, 5, 10}) {
        std::vector<State> states{{e, 0}};
        Committer c{states};
        const bool ok = ekv::refinement_ok(c, bp, bq, nb);
        if (ok != (bp >= 0 && bp < nb && e >= 0 && e < nb && bq >= 0 && bq < nb)) ++bad;
        if (ok) c.store_entry(bq);
        for (size_t p = 0; p < states.size(); ++p) {
          Tile t{states, p, p};
          if (ekv::refinement_ok(t, bp, bq, nb) != ok) ++bad;
        }
      }
  std::printf("bad %d late %d\n", bad, late);
}
"""


def _run(tmp_path, *flags):
    gxx = shutil.which("g++")
    if not gxx or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers missing")
    (tmp_path / "model.cpp").write_text(SOURCE)
    for cmd in ([gxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{build.CSRC}", *flags,
                 "model.cpp", "-o", "model"], ["./model"]):
        p = subprocess.run(cmd, cwd=tmp_path, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert p.returncode == 0, p.stdout[-3000:]
    words = p.stdout.split()
    assert len(words) == 4, p.stdout
    return int(words[1]), int(words[3])


def test_tiles_find_their_blocks_at_every_point(tmp_path):
    bad, late = _run(tmp_path)
    assert bad == 0 and late == 28   # 7 valid (b0, entry) x 4 stale values x the one state after the update


def test_the_walk_finds_an_entry_written_before_the_freed_block(tmp_path):
    assert _run(tmp_path, "-DENTRY_FIRST")[0] > 0
