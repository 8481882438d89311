"""Which resident solves may share a device (csrc/resident_gate.h), compiled for
the CPU: every set of solves that could meet there fits, and solves that fit
do not wait for each other."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_20418_amd", "csrc")


def run_cpp(tmp_path, body):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include <random>\n#include <vector>\n'
                   '#include "resident_gate.h"\nusing namespace maze;\n'
                   '#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\\n", __LINE__, #x);'
                   ' std::exit(1); } } while (0)\n' + body)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


def test_solves_that_can_meet_fit_together(tmp_path):
    run_cpp(tmp_path, """
struct S {
  int place;
  long long id;
  uint64_t lane;
  int need, cap;
  unsigned after;  // live ones it follows
};
int main() {
  std::mt19937 rng(7);
  for (int round = 0; round < 400; ++round) {
    GateLedger led;
    std::vector<S> live;
    for (int k = 0; k < 60; ++k) {
      if (live.size() < 9 && (live.empty() || rng() % 3)) {
        S s{};
        s.lane = 1 + rng() % 6;
        s.cap = rng() % 3 ? 4 * (2 + (int)(rng() % 4)) : 0;
        s.need = 1 + (int)(rng() % 9);
        const uint32_t wait = led.waits(s.lane, s.need, s.cap);
        for (size_t i = 0; i < live.size(); ++i)
          if ((wait >> live[i].place & 1) || live[i].lane == s.lane) s.after |= 1u << i | live[i].after;
        s.place = led.free_place();
        s.id = led.add(s.place, s.lane, s.need, s.cap, wait);
        live.push_back(s);
      } else if (!live.empty()) {  // one that follows no live one ends
        for (size_t t = 0, i = rng() % live.size(); t < live.size(); ++t, i = (i + 1) % live.size()) {
          if (live[i].after) continue;
          led.remove(live[i].place, live[i].id);
          if (rng() % 2) led.remove(live[i].place, live[i].id);
          live.erase(live.begin() + (long)i);
          for (S& o : live)
            o.after = (o.after & ((1u << i) - 1)) | ((o.after >> 1) & ~((1u << i) - 1));
          break;
        }
      }
      for (unsigned m = 1; m < 1u << live.size(); ++m) {  // every set that can meet
        int sum = 0, cap = 1 << 30, n = 0;
        bool meet = true;
        for (size_t i = 0; i < live.size(); ++i)
          if (m >> i & 1) {
            meet = meet && !(live[i].after & m);
            sum += live[i].need;
            cap = live[i].cap < cap ? live[i].cap : cap;
            ++n;
          }
        CHECK(!meet || n == 1 || sum <= cap);
      }
    }
  }
  return 0;
}
""")


def test_small_solves_meet_and_large_ones_take_turns(tmp_path):
    run_cpp(tmp_path, """
int main() {
  CHECK(gate_need(32, 256) == 1 && gate_need(33, 256) == 2 && gate_need(256, 256) == 8);
  CHECK(gate_need(5, 4) == 5 && gate_cap(1) == 0 && gate_cap(2) == 8);
  GateLedger led;
  // a call that was late to see its solve's end leaves the place's next solve in
  const long long a = led.add(0, 1, 8, 0, 0);
  led.remove(0, a);
  const long long b = led.add(0, 2, 8, 0, 0);
  led.remove(0, a);
  CHECK(led.holds(0, b) && !led.holds(0, a));
  led.remove(0, b);
  CHECK(led.oldest() < 0);
  long long id[GateLedger::kMax];
  for (int i = 0; i < 8; ++i) {  // 32^3: 32 workgroups, two to a CU
    CHECK(led.waits(10 + i, 1, 8) == 0);
    CHECK(led.free_place() == i);
    id[i] = led.add(i, 10 + i, 1, 8, 0);
  }
  CHECK(led.waits(30, 1, 8) == 1);       // a ninth waits for the first of them alone
  CHECK(led.waits(31, 8, 0) == 0xff);    // 128^3 waits for all
  CHECK(led.waits(12, 8, 0) == 0xfb);    // that of its own stream ends before it anyway
  CHECK(!led.waiting());
  led.add(8, 30, 1, 8, 1);
  CHECK(led.waiting());
  led.remove(3, id[3]);
  CHECK(led.waiting());
  led.remove(0, id[0]);                  // the one it waits for
  CHECK(!led.waiting());
  while (led.free_place() >= 0) led.add(led.free_place(), 99, 1, 8, 0);
  CHECK(led.oldest() == 1);
  return 0;
}
""")
