// A whole pipeline of a small 2-D grid in one kernel.
//
// k_grid2d: one block holds the three half spectra of the grid in LDS from the
// prologue to the epilogue.  As three passes (x forward, y, x inverse) such a
// grid is three launches of 3.5-5 us each that move a few kilobytes; here the
// planes are read and written once and barriers separate the passes.  Bound by
// the latency of that chain on one CU: at 32^2 in float64 10.4 us (the three
// passes 11.1, and a launch costs the host about 3 more), M^{-1} x 15.7 ->
// 10.6 us a call.
//   512 threads: with 1024 the registers of the 16- to 24-point DFTs do not
//   fit (32^2 12.3 us, 24^2 14.5 against 9.3).
//   The twiddles are read where they are used: copied to LDS first the kernel
//   is 1-8% slower, they hit the L1.
#include "lds_lines.h"
#include "llg_internal.h"
#include "pipeline_kernels.h"

namespace llg {

#define LLG_FOR_GRID_X(X) X(2) X(3) X(4) X(5) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32)
#define LLG_FOR_GRID_Y(X) X(4) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64)
constexpr int kGridThreads = 512;
// LDS row stride of nh + 1 columns: odd, so that lanes on neighbouring rows
// hit different banks
__host__ __device__ constexpr int grid_stride(int nh) { return nh + 1 + nh % 2; }

template <typename T, int DIR, class At, class In, class Out>
__device__ __forceinline__ void grid_x(int nh, int nlines, const cx<T>* __restrict__ tw, At&& at, In&& in, Out&& out) {
  switch (nh) {  // grid2d_ok: nh is one of them
#define LLG_CASE(v) \
  case v: lds_lines<T, v, DIR, kGridThreads>(nlines, tw, 2, at, in, out); break;
    LLG_FOR_GRID_X(LLG_CASE)
#undef LLG_CASE
  }
}
template <typename T, int DIR, class At, class In, class Out>
__device__ __forceinline__ void grid_y(int n, int nlines, const cx<T>* __restrict__ tw, At&& at, In&& in, Out&& out) {
  switch (n) {
#define LLG_CASE(v) \
  case v: lds_lines<T, v, DIR, kGridThreads>(nlines, tw, 1, at, in, out); break;
    LLG_FOR_GRID_Y(LLG_CASE)
#undef LLG_CASE
  }
}

// The epilogues that the kernel takes, with the prologue each is used with: the
// operators in both precisions, the right-hand side, the solvers' other
// operators and the Laplacian in float64.  Not EPI_FUSED: with and without
// Arnoldi products it has to give the same bits.
#define LLG_FOR_GRID_EPI(X)                                                                   \
  X(EPI_APPLY, PRO_COPY3) X(EPI_APPLY_T, PRO_M2T) X(EPI_MATVEC, PRO_COPY3) X(EPI_MATVEC_T, PRO_COPY3)
#define LLG_FOR_GRID_EPI_F64(X)                                                               \
  X(EPI_STORE3, PRO_COPY3) X(EPI_RHS, PRO_COPY3) X(EPI_JT, PRO_COPY3) X(EPI_APPLY_SYM, PRO_COPY3) \
  X(EPI_FUSED_SYM, PRO_SMINUS)

template <typename T, int EPI>
__device__ __forceinline__ void grid_epilogue(const PipeIO<T, T, T>& io, const NodalArgs& na, long long i,
                                              const cx<T> (&fz)[3]) {
  EpiRaw<T, T, T, EPI> raw;
  epilogue_load<false, T, T, T, EPI>(io, na, i, raw);
  T o0[4], o1[4];
  const T F0[3] = {fz[0].x, fz[1].x, fz[2].x}, F1[3] = {fz[0].y, fz[1].y, fz[2].y};
  epilogue_compute<T, T, T, EPI>(raw, 0, F0, na, o0);
  epilogue_compute<T, T, T, EPI>(raw, 1, F1, na, o1);
  if constexpr (EPI == EPI_RHS) {
    if (io.out_f) {
#pragma unroll
      for (int f = 0; f < 3; ++f) store2<false>(io.out_f + f * io.ng + i, fz[f].x, fz[f].y);
    }
  }
  constexpr int NOUT = EPI == EPI_STORE3 ? 3 : 4;
#pragma unroll
  for (int f = 0; f < NOUT; ++f) store2<false>(io.out + f * io.ng + i, o0[f], o1[f]);
}

template <typename T>
__global__ __launch_bounds__(kGridThreads) void k_grid2d(PipeIO<T, T, T> io, int pro, int epi, SpecGeom g, SymArgs sym,
                                                         NodalArgs na, const cx<T>* __restrict__ twx,
                                                         const cx<T>* __restrict__ twy) {
  extern __shared__ double grid_lds[];
  constexpr bool kF64 = std::is_same<T, double>::value;
  cx<T>* lds = reinterpret_cast<cx<T>*>(grid_lds);
  const int tid = threadIdx.x, ny = g.ny, nh = g.nh, sx = grid_stride(nh), npair = nh * ny;
  // rows (f, y) of nh + 1 values: node pairs, then the half spectrum along x
  const auto at_x = [&](int row, int k) -> cx<T>& { return lds[row * sx + k]; };
  for (int e = tid; e < npair; e += kGridThreads) {
    const long long i = 2 * e;
    cx<T> u[3];
    const auto fill = [&](auto p) {
      constexpr int PRO = decltype(p)::value;
      ProRaw<T, T, PRO> raw;
      prologue_load<false, T, T, PRO>(io.in, io.m, io.ng, i, raw);
      prologue_compute<T, T, PRO>(raw, na, u);
    };
    if (pro == PRO_COPY3) fill(std::integral_constant<int, PRO_COPY3>{});
    else if (pro == PRO_M2T) fill(std::integral_constant<int, PRO_M2T>{});
    else if constexpr (kF64) fill(std::integral_constant<int, PRO_SMINUS>{});
    const int y = e / nh, xp = e - y * nh;
#pragma unroll
    for (int f = 0; f < 3; ++f) at_x(f * ny + y, xp) = u[f];
  }
  __syncthreads();
  const auto load_x = [&](int row, int k) { return at_x(row, k); };
  const auto store_x = [&](int row, int k, cx<T> v) { at_x(row, k) = v; };
  grid_x<T, -1>(nh, 3 * ny, twx, at_x, load_x, store_x);
  // split step in place: U[k] and U[nh - k] both come from Z[k] and Z[nh - k]
  const int half = nh / 2 + 1;
  for (int e = tid; e < 3 * ny * half; e += kGridThreads) {
    const int row = e / half, k = e - row * half, k2 = nh - k;
    const cx<T> za = at_x(row, k), zb = at_x(row, k == 0 ? 0 : k2);
    const auto split = [&](cx<T> a, cx<T> bc, int kk) {
      const cx<T> b{bc.x, -bc.y};
      const cx<T> E{T(0.5) * (a.x + b.x), T(0.5) * (a.y + b.y)};
      const cx<T> O{T(0.5) * (a.y - b.y), T(-0.5) * (a.x - b.x)};
      return cadd(E, cmul(twx[kk], O));
    };
    at_x(row, k) = split(za, zb, k);
    if (k2 != k) at_x(row, k2) = split(zb, za, k2);
  }
  __syncthreads();
  // lines along y: column (f, k)
  const int ncol = 3 * (nh + 1);
  const auto at_y = [&](int col, int y) -> cx<T>& {
    const int f = (col > nh) + (col > 2 * nh + 1);
    return lds[(f * ny + y) * sx + col - f * (nh + 1)];
  };
  const auto load_y = [&](int col, int y) { return at_y(col, y); };
  grid_y<T, -1>(ny, ncol, twy, at_y, load_y, [&](int col, int y, cx<T> v) {
    const int f = (col > nh) + (col > 2 * nh + 1);
    const double xx = sym.cx * (col - f * (nh + 1)), yy = sym.cy * (y < ny / 2 ? y : y - ny);
    double mult = sym.a + sym.b * (xx * xx + yy * yy);
    mult = sym.invert ? sym.inv_ng / mult : sym.inv_ng * mult;
    at_y(col, y) = cscale(v, T(mult));
  });
  grid_y<T, 1>(ny, ncol, twy, at_y, load_y, [&](int col, int y, cx<T> v) { at_y(col, y) = v; });
  grid_x<T, 1>(
      nh, 3 * ny, twx, at_x,
      [&](int row, int k) {
        const cx<T> a = at_x(row, k), bc = at_x(row, nh - k);
        const cx<T> e{a.x + bc.x, a.y - bc.y};
        const cx<T> d{a.x - bc.x, a.y + bc.y};
        const cx<T> o = cmulc(d, twx[k]);
        return cx<T>{e.x - o.y, e.y + o.x};
      },
      store_x);
  for (int e = tid; e < npair; e += kGridThreads) {
    const int y = e / nh, xp = e - y * nh;
    const cx<T> fz[3] = {at_x(y, xp), at_x(ny + y, xp), at_x(2 * ny + y, xp)};
#define LLG_CASE(E, P) \
  case E: grid_epilogue<T, E>(io, na, 2 * e, fz); break;
    switch (epi) { LLG_FOR_GRID_EPI(LLG_CASE) }
    if constexpr (kF64) {
      switch (epi) { LLG_FOR_GRID_EPI_F64(LLG_CASE) }
    }
#undef LLG_CASE
  }
}

namespace {
bool grid_length(int nh, int ny) {
#define LLG_EQ(v) || nh == v
  const bool x = false LLG_FOR_GRID_X(LLG_EQ);
#undef LLG_EQ
#define LLG_EQ(v) || ny == v
  return x && (false LLG_FOR_GRID_Y(LLG_EQ));
#undef LLG_EQ
}
template <typename T>
bool grid_modes(int pro, int epi) {
#define LLG_EQ(E, P) || (epi == E && pro == P)
  if (std::is_same<T, double>::value && (false LLG_FOR_GRID_EPI_F64(LLG_EQ))) return true;
  return false LLG_FOR_GRID_EPI(LLG_EQ);
#undef LLG_EQ
}
}  // namespace

// Largest grid: 1280 nodes in float64, 2560 in float32.  M^{-1} x, three passes
// against one kernel: float64 24^2 15.6 -> 9.3 us, 32^2 15.8 -> 10.6, 48 x 32
// 15.6 -> 13.4 (but 13.3 us of GPU time against 12.9), 48^2 15.6 -> 17.7, 64^2
// 14.6 -> 27.5; float32 32^2 15.6 -> 8.7, 48^2 15.7 -> 12.8, 64 x 48
// transposed 15.4 -> 16.9, 64^2 15.7 -> 18.6.  The passes of a solve's Arnoldi
// steps stay three kernels: their last one reads the whole basis, which needs
// many CUs.
constexpr size_t kGridBytes = 10240;
template <typename T>
bool grid2d_ok(const Ctx& c, int pro, int epi) {
  return c.dim == 2 && size_t(c.ng) * sizeof(T) <= kGridBytes && grid_length(c.geom.nh, c.ny) &&
         grid_modes<T>(pro, epi);
}

template <typename T>
hipError_t launch_grid2d(const Ctx& c, int pro, int epi, const SymArgs& sym, const NodalArgs& na,
                         const PipeIO<T, T, T>& io, hipStream_t st) {
  if (!grid2d_ok<T>(c, pro, epi) || io.rhs) return hipErrorInvalidValue;
  const cx<T>*twx, *twy;
  if constexpr (std::is_same<T, double>::value) twx = c.tw_d[0], twy = c.tw_d[1];
  else twx = c.tw_f[0], twy = c.tw_f[1];
  const size_t bytes = sizeof(cx<T>) * 3 * size_t(c.ny) * grid_stride(c.geom.nh);
  ProfScope ps(c.prof, st, KK_XINV, 14.0 * double(c.ng) * sizeof(T));
  hipLaunchKernelGGL((k_grid2d<T>), dim3(1), dim3(kGridThreads), bytes, st, io, pro, epi, c.geom, sym, na, twx, twy);
  return hipGetLastError();
}

#define LLG_GRID(T)                                                                                            \
  template bool grid2d_ok<T>(const Ctx&, int, int);                                                            \
  template hipError_t launch_grid2d<T>(const Ctx&, int, int, const SymArgs&, const NodalArgs&,                 \
                                       const PipeIO<T, T, T>&, hipStream_t);
LLG_GRID(double)
LLG_GRID(float)
#undef LLG_GRID

}  // namespace llg
