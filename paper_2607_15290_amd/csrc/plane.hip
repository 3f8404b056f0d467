// The axis passes of a small 3-D grid in one kernel.
//
// k_plane: one block per spectral column, whose ny x nz values stay in LDS
// from the forward DFTs along y through z, the Fourier multiplier and the
// inverse DFTs back to y.  As three passes (y forward, z fused, y inverse)
// the column is read and written three times, and on small grids each launch
// costs its 3-4 us whatever it moves.  A block reads one value of each row
// (16 or 8 bytes of a 128-byte line), so each XCD takes a contiguous range of
// columns and finds its neighbours' lines in its L2.
#include "lds_lines.h"
#include "llg_internal.h"
#include "pipeline_kernels.h"

namespace llg {

// Lengths along y and z that the kernel takes (at run time).
#define LLG_FOR_PLANE(X) X(4) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32)
constexpr int kPlaneThreads = 256;
// LDS line stride: odd, so that lanes on neighbouring lines hit different banks
__host__ __device__ constexpr int plane_stride(int ny) { return ny + 1 - ny % 2; }

template <typename T, int DIR, class At, class In, class Out>
__device__ __forceinline__ void plane_axis(int n, int nlines, const cx<T>* __restrict__ tw, At&& at, In&& in,
                                           Out&& out) {
  switch (n) {  // plane_ok: n is one of them
#define LLG_CASE(v) \
  case v: lds_lines<T, v, DIR, kPlaneThreads>(nlines, tw, 1, at, in, out); break;
    LLG_FOR_PLANE(LLG_CASE)
#undef LLG_CASE
  }
}

template <typename T>
__global__ __launch_bounds__(kPlaneThreads) void k_plane(cx<T>* __restrict__ spec, SpecGeom g, SymArgs sym,
                                                         const cx<T>* __restrict__ twy,
                                                         const cx<T>* __restrict__ twz) {
  extern __shared__ double plane_lds[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(plane_lds);
  const unsigned nb = gridDim.x, xcd = blockIdx.x % 8, per = nb / 8, rem = nb % 8;
  const int col = int((xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + blockIdx.x / 8);
  const int ny = g.ny, nz = g.nz, sy = plane_stride(ny);
  cx<T>* base = spec + col;
  const auto row = [&](int y, int z) -> cx<T>& { return base[(long long)(y + ny * z) * g.rs]; };
  const auto at_y = [&](int z, int y) -> cx<T>& { return lds[z * sy + y]; };  // line z along y
  const auto at_z = [&](int y, int z) -> cx<T>& { return lds[z * sy + y]; };  // line y along z
  plane_axis<T, -1>(
      ny, nz, twy, at_y, [&](int z, int y) { return row(y, z); }, [&](int z, int y, cx<T> v) { at_y(z, y) = v; });
  const double xx = sym.cx * (col % (g.nh + 1));
  plane_axis<T, -1>(
      nz, ny, twz, at_z, [&](int y, int z) { return at_z(y, z); },
      [&](int y, int z, cx<T> v) {
        const double yy = sym.cy * (y < ny / 2 ? y : y - ny), zz = sym.cz * (z < nz / 2 ? z : z - nz);
        double mult = sym.a + sym.b * (xx * xx + yy * yy + zz * zz);
        mult = sym.invert ? sym.inv_ng / mult : sym.inv_ng * mult;
        at_z(y, z) = cscale(v, T(mult));
      });
  plane_axis<T, 1>(
      nz, ny, twz, at_z, [&](int y, int z) { return at_z(y, z); }, [&](int y, int z, cx<T> v) { at_z(y, z) = v; });
  plane_axis<T, 1>(
      ny, nz, twy, at_y, [&](int z, int y) { return at_y(z, y); }, [&](int z, int y, cx<T> v) { row(y, z) = v; });
}

namespace {
bool plane_length(int n) {
#define LLG_EQ(v) || n == v
  return false LLG_FOR_PLANE(LLG_EQ);
#undef LLG_EQ
}
template <typename T>
size_t plane_bytes(const Ctx& c) {
  return sizeof(cx<T>) * size_t(c.nz) * plane_stride(c.ny);
}
}  // namespace

// Largest column: 24 x 24 in float64, 32 x 32 in float32.  Solves against the
// three passes: 16^3 0.94 -> 0.84 ms, 24^3 1.03 -> 0.97, 32^3 (17 KB) 0.94 ->
// 0.99; 48^3 3.52 -> 3.80 (the kernel 18 us, the passes 15): the block's four
// sets of lines follow each other on one CU, so it wins only where a launch
// costs more than they do.
constexpr size_t kPlaneBytes = 10240;
template <typename T>
bool plane_ok(const Ctx& c) {
  return c.dim == 3 && plane_length(c.ny) && plane_length(c.nz) && plane_bytes<T>(c) <= kPlaneBytes;
}

template <typename T>
hipError_t launch_plane(const Ctx& c, const SymArgs& sym, cx<T>* spec, hipStream_t st) {
  if (!plane_ok<T>(c)) return hipErrorInvalidValue;
  const cx<T>*twy, *twz;
  if constexpr (std::is_same<T, double>::value) twy = c.tw_d[1], twz = c.tw_d[2];
  else twy = c.tw_f[1], twz = c.tw_f[2];
  ProfScope ps(c.prof, st, KK_AXIS_FUSED, 2.0 * c.geom.cs * double(c.ny) * c.nz * sizeof(cx<T>));
  hipLaunchKernelGGL((k_plane<T>), dim3(unsigned(c.geom.cs)), dim3(kPlaneThreads), plane_bytes<T>(c), st, spec,
                     c.geom, sym, twy, twz);
  return hipGetLastError();
}

template bool plane_ok<double>(const Ctx&);
template bool plane_ok<float>(const Ctx&);
template hipError_t launch_plane<double>(const Ctx&, const SymArgs&, cx<double>*, hipStream_t);
template hipError_t launch_plane<float>(const Ctx&, const SymArgs&, cx<float>*, hipStream_t);

}  // namespace llg
