// The limit of a device-side wait that polls: it ends with a time-out when the
// poller has seen no progress for `limit` ticks of the device wall clock, not
// when the launch has lasted that long, so a long launch that keeps moving is
// never given up. Plain C++ (no device headers).
#pragma once

#ifdef __HIPCC__
#define SPTRSV_HD __host__ __device__ __forceinline__
#else
#define SPTRSV_HD inline
#endif

struct WaitLimit {
  unsigned long long since;  // the clock when the poller was last known to move
  bool moved;                // it has moved since

  // Called now and then with the clock: whether the wait is over its limit. The
  // first look after a movement restarts it.
  SPTRSV_HD bool expired(unsigned long long now, unsigned long long limit) {
    if (moved) {
      since = now;
      moved = false;
    }
    return now - since > limit;
  }
};
