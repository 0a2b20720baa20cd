// When a plan's start ranges come from a sample of the starts (plain C++: the
// CPU tests read it too).
#pragma once

#include <algorithm>

namespace hpop {

// A start outside its sampled range costs the build twice, every start read
// costs it about a tenth more. So after a miss the same records are read in
// full, and new ones are sampled again: at once after the first miss, and after
// each further one in a row only past 1, 3, 7 .. 63 more sets of records. A
// sample that held ends the row. One odd set thus costs its own build, and a
// program whose records always miss one more build in 64.
struct RangeChoice {
  bool exact = false;  // the present records: read every start
  int wait = 0;        // sets of records to read in full before the next sample
  int row = 0;         // the wait after one more miss
  void missed() {
    exact = true;
    wait = row;
    row = std::min(63, 2 * row + 1);
  }
  void held() { row = 0; }
  void new_records() {
    if (!exact) return;
    if (wait > 0) --wait;
    else exact = false;
  }
};

}  // namespace hpop
