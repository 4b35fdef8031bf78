// How a workgroup of the serving ring takes its next unit or closes the launch
// (team_ring.hip), over any memory M:
//
//   uint64_t head()               the claim counter; its value has arrived on return
//   uint32_t tail()               units published
//   uint32_t unit(uint32_t i)     unit i (slot | rank << 16)
//   bool stop()                   the host asks an idle launch to leave
//   bool cas(uint64_t h, uint64_t to)   the claim counter h -> to
//
// The counter's top bit closes the launch.  It may be closed only where no
// system is partly claimed, since the rest of that system's team would wait for
// workgroups that no longer come.  Hence the order of the loads: the tail read
// after the head covers every unit claimed before it, so a head at or past it is
// the end of a system, and the compare-and-swap holds only if no unit has been
// claimed since.  (A tail read before the head can be older than the claims
// that the head counts, and a half-claimed system then looks like none.)
#pragma once

#include <cstdint>

#if defined(__HIP__)
#define CB_HD __host__ __device__ __forceinline__
#else
#define CB_HD inline
#endif

namespace cb {

constexpr uint64_t kRingClosed = UINT64_C(1) << 63;
constexpr int kClaimClosed = -1;   // the launch takes nothing any more
constexpr int kClaimNothing = -2;  // nothing is published that is not claimed
constexpr int kClaimAgain = -3;    // another workgroup was faster

// A unit (>= 0) or one of the above.  leave: close the launch where that is
// possible (it is old); idle: close it if there is nothing to take.
template <class M>
CB_HD int claim_step(M& m, bool leave, bool idle) {
    const uint64_t h = m.head();
    if (h & kRingClosed) return kClaimClosed;
    const bool work = (int32_t)(m.tail() - (uint32_t)h) > 0;
    const uint32_t unit = work ? m.unit((uint32_t)h) : 0u;
    const bool first = (unit >> 16) == 0;  // the first of its system
    if (work && !(leave && first)) return m.cas(h, h + 1) ? (int)unit : kClaimAgain;
    if (!leave && !idle && !m.stop()) return kClaimNothing;
    return m.cas(h, h | kRingClosed) ? kClaimClosed : kClaimAgain;
}

}  // namespace cb
