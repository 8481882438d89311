// Which resident solves of a process may share a device. Plain bookkeeping,
// for the library and for tests on the host.
//
// The workgroups of a resident solve wait for each other, so solves on the
// device at the same time must all find places whatever order their workgroups
// are dispatched in. Workgroups go to the XCDs and, within one, to the shader
// engines in turn, so a solve of nwg workgroups needs up to ceil(nwg /
// engines) places on each engine (`need`). An engine of 8 CUs has 8 * per
// places where a CU holds per workgroups of the solve, and solves share a
// device while their needs together come to at most half the places of the
// one with the fewest (`cap`): the other half is for CUs and registers that
// are divided unevenly. A solve with one workgroup to a CU (cap 0) runs alone.
//
// A solve that has to wait is queued behind the end of the others on the
// device, one at a time: streams share a few hardware queues, and a queue that
// waits holds up its other streams. (Eight threads with 64^3 mixed sessions:
// 3010 steps/s with every waiting solve queued, 5170 with four threads.) Calls
// after it wait on the host.
#pragma once

#include <cstdint>

namespace maze {

constexpr int kEngineCus = 8;

inline int gate_need(int nwg, int cus) {
  const int engines = cus >= kEngineCus ? cus / kEngineCus : 1;
  return (nwg + engines - 1) / engines;
}
inline int gate_cap(int per) { return per >= 2 ? kEngineCus * per / 2 : 0; }

// The solves queued and not known to have ended.
struct GateLedger {
  static constexpr int kMax = 32;
  struct Solve {
    long long id = 0;   // 0: free; later solves have larger ones
    uint64_t lane = 0;  // its stream: solves of one stream follow each other
    int need = 0, cap = 0;
    uint32_t behind = 0;  // places of the solves it waits for
  };
  static_assert(kMax <= 32, "one bit a place");
  Solve at[kMax];
  long long last = 0;

  int oldest() const {
    int o = -1;
    for (int i = 0; i < kMax; ++i)
      if (at[i].id && (o < 0 || at[i].id < at[o].id)) o = i;
    return o;
  }
  int free_place() const {
    for (int i = 0; i < kMax; ++i)
      if (!at[i].id) return i;
    return -1;
  }
  // Places of the solves whose end a new one has to wait for. The newest ones
  // stay beside it, as far as they fit together.
  uint32_t waits(uint64_t lane, int need, int cap) const {
    int sum = need, room = cap;
    long long before = last + 1;
    uint32_t behind = 0;
    for (;;) {
      int n = -1;
      for (int i = 0; i < kMax; ++i)
        if (at[i].id && at[i].id < before && (n < 0 || at[i].id > at[n].id)) n = i;
      if (n < 0) return behind;
      before = at[n].id;
      if (at[n].lane == lane) continue;
      const int r = room < at[n].cap ? room : at[n].cap;
      if (sum + at[n].need <= r) {
        sum += at[n].need;
        room = r;
      } else {
        behind |= 1u << n;
      }
    }
  }
  // Whether a solve is queued behind others.
  bool waiting() const {
    for (const Solve& s : at)
      if (s.id && s.behind) return true;
    return false;
  }
  // Returns the solve's id.
  long long add(int place, uint64_t lane, int need, int cap, uint32_t behind) {
    at[place] = {++last, lane, need, cap, behind};
    return last;
  }
  bool holds(int place, long long id) const { return at[place].id == id; }
  // The end of solve `id`. Another call may have seen it before and its place
  // may be a later solve's by now, which stays.
  void remove(int place, long long id) {
    if (!holds(place, id)) return;
    at[place].id = 0;
    for (Solve& s : at) s.behind &= ~(1u << place);
  }
};

}  // namespace maze
