// How many rounds of a pointer-jumping loop the host enqueues. Plain C++, so
// that a host program can check the bounds against a model of the loops.
#pragma once
#include <stdint.h>

namespace ce {

// Links climbed per pointer-jumping round: a round makes links HOPS + 1 times
// as long, so a path of k rows takes log(k) / log(5) rounds; a launch costs
// about as much as the four extra reads (19 rounds of one link each took 85 us
// at 7e4 rows).
constexpr int HOPS = 4;

// Rounds after which every row on a path of up to `links` links, the first of
// them followed before the rounds, has ARRIVED at the end: the loop looks at
// the node that it comes to, and a link is (HOPS + 1)^r long after r rounds.
constexpr int rounds_to_arrive(int64_t links) {
  int r = 0;
  for (int64_t reach = 1; reach < links; reach *= HOPS + 1) r++;
  return r;
}

// Rounds after which every row has SEEN that it is at the end: the loop keeps
// a row until its HOPS reads of a round show it a node that points to itself,
// so round r is a row's last if HOPS links of the length before it reach the
// end: HOPS * (HOPS + 1)^(r - 1).
constexpr int rounds_to_confirm(int64_t links) {
  int r = 1;
  for (int64_t reach = HOPS; reach < links; reach *= HOPS + 1) r++;
  return r;
}

}  // namespace ce
