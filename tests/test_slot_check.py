"""A cell's check at the end of its phase, on the CPU: chains move disks between one-disk slots with unchecked stores, as
the event loops do (a bin change empties the old slot and writes the new one's centre, meta word and index; a rejected
chain is undone, latest move first).  Every disk has its slot at the end, and no undo started from an empty one, exactly
if no move went to a slot that held another disk, whatever came after it."""
import os
import subprocess

import pytest

from paper_1409_6948_amd import build as B

MODEL = r"""
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>
#include "ec_internal.h"

struct Move { int from, to; double old; };

int main(int argc, char** argv) {
  const int disks = std::atoi(argv[1]), slots = std::atoi(argv[2]), reject = std::atoi(argv[3]), bump = std::atoi(argv[4]);
  std::mt19937 rng(7 + 13 * disks + slots);
  auto draw = [&](int n) { return (int)(rng() % (unsigned)n); };
  int wrong = 0, hit = 0, clean = 0;
  for (int trial = 0; trial < 20000; ++trial) {
    std::vector<double> pos(slots, std::nan(""));
    std::vector<uint32_t> meta(slots, 0xFFFFFFFFu);
    std::vector<int> own_loc(disks);
    double next = 1.0;
    for (int k = 0; k < disks; ++k) {
      int s;
      do s = draw(slots); while (!std::isnan(pos[s]));
      pos[s] = next++; meta[s] = (uint32_t)k; own_loc[k] = s;
    }
    bool taken = false;  // some move went to a slot that held another disk
    bool kept = true;
    const int chains = 1 + draw(6);
    for (int c = 0; c < chains; ++c) {
      int k = draw(disks), at = own_loc[k];
      std::vector<Move> log;
      const int events = 1 + draw(6);
      for (int e = 0; e < events; ++e) {
        // the moved centre's bin: mostly an empty one or its own, now and then another disk's
        int to = draw(slots);
        if (!std::isnan(pos[to]) && to != at && draw(100) >= bump) to = at;
        if (to != at && !std::isnan(pos[to])) taken = true;
        log.push_back({at, to, pos[at]});
        const double v = std::isnan(pos[at]) ? pos[at] : next++;
        if (to != at) { pos[at] = std::nan(""); meta[to] = (uint32_t)k; own_loc[k] = to; }
        pos[to] = v;
        // the disk it hits goes on
        std::vector<int> held;
        for (int s = 0; s < slots; ++s) if (!std::isnan(pos[s]) && s != to) held.push_back(s);
        if (held.empty()) break;
        at = held[draw((int)held.size())];
        k = (int)meta[at];
      }
      if (reject && draw(2)) {
        for (int u = (int)log.size() - 1; u >= 0; --u) {
          kept = kept && !std::isnan(pos[log[u].to]);
          if (log[u].to != log[u].from) {
            const uint32_t mv = meta[log[u].to];
            pos[log[u].to] = std::nan(""); meta[log[u].from] = mv; own_loc[(int)mv] = log[u].from;
          }
          pos[log[u].from] = log[u].old;
        }
      }
    }
    for (int k = 0; k < disks; ++k) kept = kept && ec::slot_kept(meta[own_loc[k]], (uint32_t)k, pos[own_loc[k]]);
    (taken ? hit : clean) += 1;
    wrong += kept == taken;
  }
  std::printf("%d %d %d\n", wrong, hit, clean);
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("slots")
    (d / "model.cpp").write_text(MODEL)
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", B.CSRC, "-I", "/opt/rocm/include",
                        "-o", str(d / "model"), str(d / "model.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return str(d / "model")


@pytest.mark.parametrize("disks,slots", [(2, 3), (2, 9), (5, 9), (12, 30)])
@pytest.mark.parametrize("reject", [0, 1])
def test_a_taken_slot_is_always_seen(model, disks, slots, reject):
    r = subprocess.run([model, str(disks), str(slots), str(reject), "6"], capture_output=True, text=True, timeout=60)
    wrong, hit, clean = map(int, r.stdout.split())
    assert hit > 1000 and clean > 1000
    assert wrong == 0


def test_the_cell_kernel_looks():
    text = open(os.path.join(B.CSRC, "ec_kernels.hip")).read()
    a, b = text.index("void phase_cell("), text.index("// ---- write back: old position + local displacement")
    assert "slot_kept(" in text[a:b]
