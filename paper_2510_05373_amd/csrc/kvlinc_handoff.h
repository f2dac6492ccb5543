// Who merges the partial results of a (sequence, kv head): the counter that the workgroups of a decode launch arrive at, and what they
// make of it.  Counter: add(n) returns the number before, look() the present one, pause() lets some time pass.
#pragma once

#include <hip/hip_runtime.h>

namespace kvlinc {

// What arrives at a (sequence, kv head): its streaming workgroups, 1 each, and those of the correction, kCorrArrival each.
// Who merges: the streaming workgroup that completes the streaming ones, if the correction is complete; otherwise, where the launch
// says that the correction is awaited -- its workgroups are the first of the grid --, the same workgroup, which looks at the
// counter until it is, up to `looks` times; or else the correction workgroup that completes the count.  A streaming workgroup
// that gives up leaves kGaveUp in the counter: whoever adds to it last, it or the correction, sees the other and merges.
// The single split of a sequence keeps its result where the correction is awaited and looks before it arrives; if that gives up it
// arrives with the mark and looks no more.  (A sequence of one split without a correction, or that finds it complete, does not
// arrive at all.)
// Whoever merges is the last to touch the counter, and clears it.
constexpr int kCorrArrival = 64, kGaveUp = 1 << 16;
__host__ __device__ inline int streams_arrived(int count) { return count & (kCorrArrival - 1); }
__host__ __device__ inline int parts_arrived(int count) { return (count & (kGaveUp - 1)) / kCorrArrival; }

template <class Counter>
__host__ __device__ inline bool await_parts(Counter& counter, int n_parts, int looks) {
  for (int i = 0; i < looks; ++i) {
    if (parts_arrived(counter.look()) == n_parts) return true;
    counter.pause();
  }
  return false;
}

// Arrival of a streaming workgroup.  Returns whether it merges.
template <class Counter>
__host__ __device__ inline bool stream_arrives(Counter& counter, int n_splits, int n_parts, bool awaited, bool gave_up, int looks) {
  const int before = counter.add(gave_up ? 1 + kGaveUp : 1);
  if (streams_arrived(before) != n_splits - 1) return false;
  if (parts_arrived(before) == n_parts) return true;
  if (!awaited || gave_up) return false;
  return await_parts(counter, n_parts, looks) || parts_arrived(counter.add(kGaveUp)) == n_parts;
}

// Whether the correction workgroup that added kCorrArrival to `before` merges.
__host__ __device__ inline bool correction_merges(int before, int n_splits, int n_parts, bool awaited) {
  return parts_arrived(before) == n_parts - 1 && streams_arrived(before) == n_splits && (!awaited || before >= kGaveUp);
}

}  // namespace kvlinc
