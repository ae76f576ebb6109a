// The rule by which a wait inside a persistent kernel ends: plain C++, for the kernels and for a host test.
#pragma once

#ifdef __HIP__
#define MDI_HOST_DEVICE __host__ __device__
#else
#define MDI_HOST_DEVICE
#endif

namespace mdi {

// How often a waiting thread looks whether its workgroup has given up elsewhere (a power of two): often enough that the
// waits after a failed one cost nothing against `limit`, seldom enough that an ordinary wait - a few polls - never does.
constexpr int kPollsPerLook = 64;

// Called after a poll that found nothing, with the number of such polls so far.  True: ask again.  False: stop waiting,
// either because another wait of the workgroup has expired - failed() -, or because this one just has, which
// give_up() then records.
template <typename Failed, typename GiveUp>
MDI_HOST_DEVICE inline bool may_poll_again(int& polls, int limit, const Failed& failed, const GiveUp& give_up) {
  if ((++polls & (kPollsPerLook - 1)) == 0 && failed()) return false;
  if (polls <= limit) return true;
  give_up();
  return false;
}

}  // namespace mdi
