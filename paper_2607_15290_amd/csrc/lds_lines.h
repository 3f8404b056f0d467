// DFTs along lines that lie in LDS, for the kernels that keep a whole column
// or grid there (plane.hip, grid2d.hip).
#pragma once
#include "fft_core.h"

namespace llg {

// All nlines lines of the block, DFT of length N in direction DIR by NT
// threads.  Lines are spread over the lanes first.  in(line, pos) and
// out(line, pos, value) move a value; at(line, pos) is its LDS slot.  The
// line's values are all read before any of its slots is written.  tws: stride
// of the length-N table in tw.
template <typename T, int N, int DIR, int NT, class At, class In, class Out>
__device__ __forceinline__ void lds_lines(int nlines, const cx<T>* __restrict__ tw, int tws, At&& at, In&& in,
                                          Out&& out) {
  constexpr int P = plan_p(N), TPL = N / P, L = NT / TPL;
  const int ln = threadIdx.x % L, t = threadIdx.x / L;
  for (int l0 = 0; l0 < nlines; l0 += L) {  // the same trips for every thread (barriers inside)
    const bool on = t < TPL && l0 + ln < nlines;
    const int line = on ? l0 + ln : 0;
    cx<T> v[P];
    if (on) {
#pragma unroll
      for (int q = 0; q < P; ++q) v[in_slot<N>(q)] = in(line, t + TPL * q);
    }
    auto acc = [&](int pos) -> cx<T>& { return at(line, pos); };
    line_fft<T, N, DIR>(v, t, acc, tw, tws, on);
    __syncthreads();  // a later stage's reads before the values are replaced
    if (on) {
#pragma unroll
      for (int s = 0; s < P; ++s) out(line, t + TPL * out_q<N>(s), v[s]);
    }
  }
  __syncthreads();
}

}  // namespace llg
