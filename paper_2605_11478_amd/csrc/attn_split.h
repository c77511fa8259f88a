// Equal contiguous ranges of attention work units (32- or 128-token pieces of
// all groups laid end to end) over wavefronts or workgroups.
#ifndef FIBQ_ATTN_SPLIT_H
#define FIBQ_ATTN_SPLIT_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fibq {
namespace dev {

// The first unit of wavefront w of `waves`: w units / waves, from the quotient
// and remainder of units by waves.  All of this is in 32 bits (units < 2^31,
// waves < 2^16): a 64-bit division is 0.5 KB of code, and a small call's time
// is mostly instruction fetches (a merge kernel of 50 KB took 34 us for 63
// records, of 5 KB 4 us; attn_k4.hip's main kernel 14.4 us at 21 KB, 11.4 at 15).
struct Split {
  uint32_t units, q, r, waves, upg;
};
__host__ __device__ __forceinline__ uint32_t first_unit(uint32_t w, const Split& s) {
  return w * s.q + w * s.r / s.waves;
}

// the wavefront whose unit range [first_unit(w), first_unit(w + 1)) holds u
__device__ __forceinline__ uint32_t wave_of(uint32_t u, const Split& s) {
  // (the float estimate is off by less than 0.1, and rounded down)
  uint32_t w = (uint32_t)((float)u * ((float)s.waves / (float)s.units));
  w = w > 0 ? w - 1 : 0;
  while (first_unit(w + 1, s) <= u) ++w;
  return w;
}

inline Split make_split(int64_t units, uint32_t waves, int upg) {
  return Split{(uint32_t)units, (uint32_t)(units / waves), (uint32_t)(units % waves), waves,
               (uint32_t)upg};
}

}  // namespace dev
}  // namespace fibq

#endif
