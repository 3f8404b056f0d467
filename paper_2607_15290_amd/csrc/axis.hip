// Axis passes of the spectral pipeline (DFTs along y or z, see
// pipeline_kernels.h).  Dispatches the runtime axis length to a kernel
// instantiation.
#include "llg_internal.h"
#include "pipeline_kernels.h"

namespace llg {

// Passes with fewer wide blocks than this (one per CU) take the narrow shape:
// 256^2 7.65 -> 5.98 us, 512^2 8.8 -> 7.7.  Above it the two are the same within
// the noise: solves at 64^3 (448 wide blocks) 3.162 ms narrow, 3.170 wide; 80^3
// 3.565 and 3.560; 96 x 64 x 48 2.92 and 2.97, runs of one side 1% apart.
#ifndef LLG_AXIS_NARROW_BLOCKS
#define LLG_AXIS_NARROW_BLOCKS 256
#endif

template <typename T, int N, bool NARROW>
static void axis_launch(const Ctx& c, int axis, int mode, const SymArgs& sym, cx<T>* spec, const cx<T>* tw,
                        hipStream_t st) {
  using C = AxisCfg<T, N, NARROW>;
  const dim3 grid((unsigned)((c.geom.cs + C::W - 1) / C::W), (unsigned)(axis == 1 ? c.nz : c.ny));
  const dim3 block(C::W * C::TPL);
  switch (mode) {
    case 0: hipLaunchKernelGGL((k_axis<T, N, 0, NARROW>), grid, block, 0, st, spec, c.geom, axis, sym, tw); break;
    case 1: hipLaunchKernelGGL((k_axis<T, N, 1, NARROW>), grid, block, 0, st, spec, c.geom, axis, sym, tw); break;
    default: hipLaunchKernelGGL((k_axis<T, N, 2, NARROW>), grid, block, 0, st, spec, c.geom, axis, sym, tw); break;
  }
}

template <typename T, int N>
static hipError_t axis_n(const Ctx& c, int axis, int mode, const SymArgs& sym, cx<T>* spec, hipStream_t st) {
  constexpr int W = AxisCfg<T, N, false>::W;
  const long long blocks = (long long)((c.geom.cs + W - 1) / W) * (axis == 1 ? c.nz : c.ny);
  const cx<T>* tw;
  if constexpr (std::is_same<T, double>::value) tw = c.tw_d[axis];
  else tw = c.tw_f[axis];
  const double bytes = 2.0 * c.geom.cs * double(c.ny) * c.nz * 2 * sizeof(T);
  ProfScope ps(c.prof, st, mode == 0 ? KK_AXIS_FWD : (mode == 1 ? KK_AXIS_INV : KK_AXIS_FUSED), bytes);
  if constexpr (AxisCfg<T, N, true>::W < W) {
    if (blocks < LLG_AXIS_NARROW_BLOCKS) {
      axis_launch<T, N, true>(c, axis, mode, sym, spec, tw, st);
      return hipGetLastError();
    }
  }
  axis_launch<T, N, false>(c, axis, mode, sym, spec, tw, st);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_axis(const Ctx& c, int axis, int mode, const SymArgs& sym, cx<T>* spec, hipStream_t st) {
  const int n = axis == 1 ? c.ny : c.nz;
  switch (n) {
#define LLG_CASE(v) \
  case v: return axis_n<T, v>(c, axis, mode, sym, spec, st);
    LLG_FOR_AXIS(LLG_CASE)
#undef LLG_CASE
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_axis<double>(const Ctx&, int, int, const SymArgs&, cx<double>*, hipStream_t);
template hipError_t launch_axis<float>(const Ctx&, int, int, const SymArgs&, cx<float>*, hipStream_t);

}  // namespace llg
