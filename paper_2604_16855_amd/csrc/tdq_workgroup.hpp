// What one thread finds out for its whole workgroup.  No other header, so that a host program can run it with threads
// as wavefronts.
#pragma once

namespace tdq {

// Thread 0 finds out whether it is so, every thread gets the answer.  *flag, a word of LDS, may be written again as
// soon as this returns: the second barrier waits for the wavefronts that are late to read it.
template <typename F>
__device__ __forceinline__ bool known_to_all(unsigned* flag, F&& is_so) {
  if (threadIdx.x == 0) *flag = is_so() ? 1u : 0u;
  __syncthreads();
  const bool so = *flag != 0u;
  __syncthreads();
  return so;
}

}  // namespace tdq
