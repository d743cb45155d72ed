"""The rule by which helpers of the batched solve take slices, on the CPU: a leader that publishes
one job after the other, takes back what no helper claimed in time and reuses its vectors, and a
helper that is held up at any of its memory accesses while the leader goes on."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <cstdio>
#include "team_claim.h"

// the shared record, with two fields of the job in place of its vectors
struct Team { int64_t job = 0; int a = 0, b = 0, claim[3] = {}, done[3] = {}; };

// the leader, one memory access per step. Slices 1 .. helpers(e) of job e go to helpers.
struct Leader {
  Team& T;
  int epoch = 0, phase = 0, slice = 1, polls = 0;
  static int helpers(int e) { return e < 2 ? 0 : (e < 4 ? 1 : 2); }  // one joins at 2, one at 4
  void step() {
    switch (phase) {
      case 0: ++epoch; T.a = epoch; phase = 1; break;
      case 1: T.b = epoch; phase = 2; break;
      case 2: T.job = team::job_word(epoch, helpers(epoch) + 1); slice = 1; polls = 0; phase = 3; break;
      case 3:
        if (slice > helpers(epoch)) { phase = 0; break; }
        if (T.done[slice] == epoch) { ++slice; polls = 0; break; }
        if (++polls < 2) break;  // the time a helper has
        int* p = &T.claim[slice];
        if (team::claim(epoch, [=] { return *p; }, [=](int& cur, int to) {
              if (*p != cur) { cur = *p; return false; }
              *p = to;
              return true;
            })) { ++slice; polls = 0; }
        break;
    }
  }
  bool serving(int e, int h) const { return epoch == e && phase == 3 && slice <= h; }
};

// helper h looks at one job; before access i the leader takes sched[i] steps
int run(int h, const int* sched, long* worked) {
  Team T;
  Leader L{T};
  int at = 0;
  auto hold = [&] { for (int q = sched[at++]; q > 0; --q) L.step(); };
  hold();
  const int64_t word = T.job;
  const int e = team::job_epoch(word);
  if (e == 0 || h >= team::job_slices(word)) return 0;
  hold();
  const int a = T.a;
  hold();
  const int b = T.b;
  int* p = &T.claim[h];
  int tries = 0;
  if (!team::claim(e, [&] { hold(); return *p; }, [&](int& cur, int to) {
        if (tries++ == 0) hold();
        if (*p != cur) { cur = *p; return false; }
        *p = to;
        return true;
      })) return 0;
  if (!L.serving(e, h)) return 1;            // the leader has moved on
  if (a != e || b != e) return 2;            // fields of another job
  for (int q = 0; q < 40; ++q) L.step();     // however long the slice takes
  if (!L.serving(e, h)) return 3;            // the leader did not wait
  T.done[h] = e;
  ++*worked;
  return 0;
}

int main() {
  long worked = 0, runs = 0;
  int s[5];
  for (int h = 1; h <= 2; ++h)
    for (s[0] = 0; s[0] < 40; ++s[0])
      for (s[1] = 0; s[1] < 14; ++s[1])
        for (s[2] = 0; s[2] < 14; ++s[2])
          for (s[3] = 0; s[3] < 14; ++s[3])
            for (s[4] = 0; s[4] < 14; ++s[4], ++runs) {
              const int bad = run(h, s, &worked);
              if (bad) {
                std::printf("fault %d: helper %d held up for %d %d %d %d %d steps\n", bad, h, s[0], s[1], s[2], s[3], s[4]);
                return 1;
              }
            }
  std::printf("%ld schedules, %ld slices\n", runs, worked);
  return worked > 0 ? 0 : 2;  // schedules in which the helper was in time
}
"""


def test_a_claimed_slice_is_of_the_job_the_leader_waits_for(tmp_path):
    src = tmp_path / "claims.cpp"
    src.write_text(HARNESS)
    exe = tmp_path / "claims"
    inc = os.path.join(ROOT, "paper_2405_05865_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", inc, "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
