// Teams of workgroups that wait for each other: how a launch of the single-read scoring kernel is laid out, and when its waits
// are safe next to other launches.  Plain C++: the rule is checked on the host against a model of the device.
//
// A workgroup waits only for the others of its team, and it draws its place in a team when it starts.  Places are drawn from one
// counter or from two, and the teams of a counter fill up one after the other; so of a launch at most one team per counter is on the device in
// part.  A team that is there whole needs nobody else: it ends, and its places come free, as they do when other kernels
// end.  A place that comes free lets a workgroup in that waits for one, which completes a team or brings one nearer to that.  Only if parts of
// teams held every place would none come free, and they cannot while
//     (places that the parts of one launch may hold) x (such launches at a time)  <  places of the device.
// Launches at a time: a stream's launches follow one another and streams share the process's hardware queues, HW_QUEUES of
// them.  So streams that have queues of their own (confined to some compute units, or of another priority) take no part in this: they get
// the two-pass kernels, which wait for nobody.
#ifndef LAQ_TEAM_H
#define LAQ_TEAM_H

#include <stdint.h>

#include <algorithm>

namespace laq {

constexpr int HW_QUEUES = 4;               // of normal priority, HIP's own number

// Whether a stream goes through the queues that are counted, and may use every compute unit (mask: a bit for each).
inline bool stream_counted(const uint32_t* mask, int cus, int priority) {
  int open = 0;
  for (int i = 0; i < cus; ++i) open += mask[i / 32] >> (i % 32) & 1;
  return open == cus && priority == 0;
}

struct TeamPlan {
  int T;                                   // workgroups per team
  int n_teams;                             // team t takes heads t, t + n_teams, ...
  int early;                               // the workgroups with the lowest numbers that draw from the first counter (whole teams of them)
};

// Places that the parts of a launch's teams may hold.
inline int places_of_parts(int T, int counters) { return counters * (T - 1); }
inline bool parts_leave_a_place(int T, int counters, int resident) {
  return (long long)places_of_parts(T, counters) * HW_QUEUES < resident;
}
// Whether teams of this length are safe in ordinary launches: with one counter at least.
inline bool ordinary_team(int T, int resident) { return parts_leave_a_place(T, 1, resident); }
// Two counters are the faster ones (see drawn_place()) and are taken where they are safe too, and where the rule does not hold anyway.
inline int counters_of(int T, int resident) { return parts_leave_a_place(T, 2, resident) || !ordinary_team(T, resident) ? 2 : 1; }

// false: the device does not hold a team of this length
inline bool plan_teams(int n_heads, int T, int resident, TeamPlan* out) {
  if (resident <= 0 || T > resident) return false;
  out->T = T;
  out->n_teams = std::min(resident / T, n_heads);
  out->early = (counters_of(T, resident) == 2 ? std::min(out->n_teams, resident / 2 / T) : out->n_teams) * T;
  return true;
}

}  // namespace laq

#endif  // LAQ_TEAM_H
