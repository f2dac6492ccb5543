// Host build of the integer arithmetic that the decode kernel's workgroups share (see test_decode_schedule.py).
#include "kvlinc_schedule.h"

extern "C" {

int window_rounds(int count, int n_splits, int bits) { return kvlinc::window_rounds(count, n_splits, bits); }

int group_of_round(int n_splits, int split, int wave, int skip, int round) { return kvlinc::GroupOrder(n_splits, split, wave, skip).group(round); }

}  // extern "C"
