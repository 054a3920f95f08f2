// The host's wait for records that a kernel leaves in mapped host memory.  Plain C++, no HIP: the
// stream query is the caller's.
#pragma once

#include <immintrin.h>

#include <chrono>

namespace ilh {

enum class Waited {
  Arrived,   // the records are there
  GivenUp,   // the work that would have stored them says that it was given up
  Missing,   // the stream is done and neither came
  TimedOut,  // two minutes passed
  Failed     // the query reported an error
};

// arrived(): the records are complete; given_up(): their producer marked itself as given up; query(): the
// state of the stream (0: at work, 1: done, anything else: an error).  The query is asked once a
// millisecond only: it costs the stream a marker, and an ordinary wait is far shorter.
template <typename A, typename G, typename Q>
Waited wait_records(A&& arrived, G&& given_up, Q&& query) {
  using clock = std::chrono::steady_clock;
  const auto t0 = clock::now();
  auto asked = t0;
  for (unsigned spins = 1; !arrived(); ++spins) {
    _mm_pause();
    if (given_up()) return Waited::GivenUp;
    if ((spins & 1023) != 0) continue;
    const auto now = clock::now();
    if (now - asked < std::chrono::milliseconds(1)) continue;
    asked = now;
    const int q = query();
    if (q != 0 && q != 1) return Waited::Failed;
    if (q == 1) {
      // host-mapped stores, of the records and of the mark, can trail the completion that the stream
      // reports: 10 ms more
      while (!arrived() && !given_up() && clock::now() - now < std::chrono::milliseconds(10)) _mm_pause();
      return arrived() ? Waited::Arrived : given_up() ? Waited::GivenUp : Waited::Missing;
    }
    if (now - t0 > std::chrono::seconds(120)) return Waited::TimedOut;
  }
  return Waited::Arrived;
}

}  // namespace ilh
