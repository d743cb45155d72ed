// Who computes a slice of a team job of the batched solve: the words that the leader and the
// helpers exchange. Plain C++ over the caller's atomics, so the rule can be checked on the host.
//
// The leader numbers its jobs 1, 2, ... (epochs). It prepares the fields of job e + 1 only when
// every slice of job e is done or claimed by itself. So a helper may use what it read of job e
// if, after reading it, it claims one of that job's slices:
//   - claims only go forward. A helper that was held up between reading job e and claiming finds
//     the leader's claim of e, or of a later job, and leaves the slice alone. (A rule that only
//     refuses an equal number lets it overwrite a later claim and compute the old job into
//     vectors that the leader has moved on from.)
//   - the number of slices is part of the published word. Read beside it, it may already be the
//     next job's, and a helper that joined in between would claim a slice that job e has not.
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define MSP_TEAM_FN __device__ __forceinline__
#else
#define MSP_TEAM_FN inline
#endif

namespace team {

MSP_TEAM_FN int64_t job_word(int epoch, int nslice) { return ((int64_t)epoch << 32) | (uint32_t)nslice; }
MSP_TEAM_FN int job_epoch(int64_t w) { return (int)(w >> 32); }
MSP_TEAM_FN int job_slices(int64_t w) { return (int)(uint32_t)w; }

// load(): the slice's last claim. cas(cur, e): exchange cur for e, or load cur. True if the
// caller now has the slice for job e.
template <class Load, class Cas>
MSP_TEAM_FN bool claim(int e, Load load, Cas cas) {
  int cur = load();
  while (cur < e)
    if (cas(cur, e)) return true;
  return false;
}

}  // namespace team
