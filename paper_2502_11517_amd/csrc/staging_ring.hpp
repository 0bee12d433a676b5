// The pinned staging slots of a handle go round; one is written again only after the work that reads it has completed.
// That is recorded once per half of the ring, behind its last slot: an event is a packet on the stream.  A call holds
// at most one slot.  One that ends in an error without giving its slot back may have enqueued work that reads it: the
// slot is taken again after the stream has drained, and the half still closes with a recorded event.
#pragma once

namespace pasta {

template <int N> struct StagingRing {
  static_assert(N % 2 == 0, "two halves");
  int next = 0;
  bool open = false;  // slot `next` has been taken and not been given back
  bool used[2] = {};

  // wait(half): until the event of that half; drain(): until everything enqueued so far.  Both false on failure.
  template <class Wait, class Drain> bool take(int* slot, Wait wait, Drain drain) {
    if (open) {
      if (!drain()) return false;
    } else if (next % (N / 2) == 0 && used[next / (N / 2)] && !wait(next / (N / 2))) {
      return false;
    }
    open = true;
    *slot = next;
    return true;
  }
  template <class Record> bool give(Record record) {  // the work that reads the slot has been enqueued
    if (next % (N / 2) == N / 2 - 1) {
      if (!record(next / (N / 2))) return false;
      used[next / (N / 2)] = true;
    }
    next = (next + 1) % N;
    open = false;
    return true;
  }
};

}  // namespace pasta
