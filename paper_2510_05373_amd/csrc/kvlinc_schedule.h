// The order in which a decode launch walks the groups of a sequence: integer arithmetic, the same on the host.
#pragma once

#include <hip/hip_runtime.h>

namespace kvlinc {

constexpr int kWaves = 4;  // of a streaming workgroup

// Time is cut into rounds of 4 n_splits slots, slot(round, wave, split) = 4 n_splits round + n_splits wave +
// n_splits - 1 - split; the groups 0, 1, 2, ... go to the slots in order, except that the four waves of split 0 sit out the
// first `skip` rounds: a share of the window each is their work for that time.  Consecutive groups thus go to different
// workgroups, and every split gets the same share whatever the length.
// The first group of the other splits' waves is the same with any number of skipped rounds.
struct GroupOrder {
  int slots, off, skip, wave;
  __host__ __device__ GroupOrder(int n_splits, int split, int wave_, int skip_)
      : slots(kWaves * n_splits), off(wave_ * n_splits + n_splits - 1 - split), skip(skip_), wave(wave_) {}
  __host__ __device__ int group(int round) const { return round * slots + off - (round < skip ? kWaves * round + wave : kWaves * skip); }
};

// Rounds that split 0 sits out, from the groups of the longest sequence that a launch is made for.  A share of the window takes about
// as long as two groups of 2 bits, or one of 4: two rounds at 2 bits, but one where the second would make that sequence a round
// longer, ceil((count + 8) / slots) > ceil((count + 4) / slots).  Decode launches of equal lengths and two splits or more, the one
// round in the time of the two: 0.97 where two make it longer (118 shapes; 0.86 to 1.04), 1.01 to 1.02 where they do not (887).
// At 4 bits, 16 sequences of 8k tokens: 39.1 us a step with two, 37.4 with one.
// (The host's to say: from each sequence's own counter in the kernel, with the first record requested again where the guess was
// wrong, launches of two splits or more took 1.006 of the time of two rounds always, those with the longer schedules included.)
inline int window_rounds(int count, int n_splits, int bits) {
  if (bits != 2) return 1;
  return n_splits > 1 && (count + 7) % (kWaves * n_splits) < kWaves ? 1 : 2;
}

}  // namespace kvlinc
