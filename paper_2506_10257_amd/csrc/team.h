// Meetings of a team of workgroups (eig_steps.hip) and what the launch after it
// makes of them.  Plain C++, so that a test on the CPU can run the same rules in
// every order of events.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define RPCA_HD __host__ __device__
#else
#define RPCA_HD
#endif

namespace rpca {

// One workgroup's part of a meeting that is complete once `all` arrivals are
// counted: true when it may go on.  A workgroup whose time is over says so
// (lose) and leaves, and every other one leaves at this meeting or a later one.
// They need not all leave at the same one: a workgroup that arrives after
// another has left still completes the count.  So what a launch wrote stands
// only by steps_stand.
template <typename Ctl>
RPCA_HD inline bool meet_team(Ctl& c, unsigned all) {
  c.arrive();
  while (c.arrived() < all) {
    if (c.lost()) return false;
    if (c.late()) {
      c.lose();
      return false;
    }
  }
  return true;
}

// Whether the steps' projector of iteration `next` stands, asked by the next
// launch: every workgroup has ended, so `lost` is final, and if none of them
// left early each has written its blocks.
RPCA_HD inline bool steps_stand(uint32_t lost, int32_t booked, int32_t next) {
  return lost == 0 && booked == next;
}

}  // namespace rpca
