// Which resident launches of one GPU may run side by side.
//
// The blocks of a resident launch wait for each other on the GPU, so launches that run together must have at
// most a block per CU in total: with more, each would hold some of the places the other waits for.  A new launch
// waits (on its stream, for events) for enough of the earlier ones.
#pragma once

#include <algorithm>

namespace dd {

// The newest resident launch of each stream that may still run, oldest first.  An entry counts for everything that may
// run until its event: its own blocks, or those of what it waits for that has no entry of its own any more (the
// stream's launch before it, an entry taken out to make room).  Entries that are waited for stay: what comes later may
// still meet them.  So of any launches that run together, the newest saw all others listed and found room beside them.
template <class Stream, class Event>
struct ResFlights {
  struct Entry {
    Stream stream;
    Event end;
    int blocks;
  };
  static constexpr int kMost = 32;
  Entry e[kMost];
  int n = 0;

  // Before a launch of `blocks` blocks is queued on `st`; add() follows with the value returned.  done(event): known to
  // be over; wait(event): the stream waits for it; drop(event): not needed any more.
  template <class Done, class Wait, class Drop>
  int admit(Stream st, int blocks, int cus, Done&& done, Wait&& wait, Drop&& drop) {
    int mine = 0;      // blocks that may run before this launch and have no entry
    const auto remove = [&](int i) {
      drop(e[i].end);
      for (int j = i + 1; j < n; ++j) e[j - 1] = e[j];
      --n;
    };
    for (int i = 0; i < n;) {
      const bool own = e[i].stream == st, over = done(e[i].end);
      if (own && !over) mine += e[i].blocks;
      if (own || over) remove(i);
      else ++i;
    }
    if (n == kMost) {
      wait(e[0].end);
      mine += e[0].blocks;
      remove(0);
    }
    // the newest ones that leave room run beside this launch, all before them are waited for
    int room = cus - blocks, first = n;
    while (first > 0 && room >= e[first - 1].blocks) room -= e[--first].blocks;
    for (int i = 0; i < first; ++i) wait(e[i].end);
    return std::min(std::max(mine, blocks), cus);
  }
  void add(Stream st, Event end, int blocks) { e[n++] = Entry{st, end, blocks}; }
};

}  // namespace dd
