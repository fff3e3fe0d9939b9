// mc_queue.h -- the protocol of the spike id queue in LDS between the poller of
// a workgroup and the wavefronts that deliver (see mc_persist.hip).
//
// Ids have running positions (modulo 2^32): [0, tail) have been put in, [0,
// head) claimed, and position q lies in slot q mod the number of slots.  The
// poller knows only how many ids have been delivered, in whatever order, so a
// slot is protected by one fact: an unclaimed position is at or beyond the head,
// no more ids than the head says can have been delivered, and the poller stays
// within its room.  A claimed position has no such protection (wavefronts
// that claimed later ids may deliver them first), so an id is read before the
// exchange that claims it: if the exchange finds the head where it was, the
// slots read were still those of unclaimed positions.
//
// Templates over the operations, so that the same code runs in the kernel and
// in a model that tries every order of the operations on the host.
#pragma once
#include "mc_common.h"

namespace mc {

// Claims some of the ids before `tail`: a short queue is shared out in rounds
// of `per`, a long one evenly among `nw` wavefronts, at most 64 at a time.
// q.head() loads the head, q.read(h) the ids from position h on, q.take(h, to)
// moves the head from h to `to` and returns the head it found.  Returns how
// many of the ids read last are claimed (0: none left).
template <class Q>
MC_HD unsigned claim_ids(Q& q, unsigned tail, unsigned per, unsigned nw) {
  unsigned h = q.head();                      // (may be past the tail by now)
  while ((int)(tail - h) > 0) {
    const unsigned avail = tail - h, even = avail / nw;
    unsigned want = per > even ? per : even;
    want = want < 64u ? want : 64u;
    want = want < avail ? want : avail;
    q.read(h);
    const unsigned found = q.take(h, h + want);
    if (found == h) return want;
    h = found;
  }
  return 0;
}

// Ids the poller may put in beyond `tail` when `gone` have been delivered.
MC_HD unsigned queue_room(unsigned capacity, unsigned tail, unsigned gone) { return capacity - (tail - gone); }

}  // namespace mc
