// Lower-order field pipeline (float64).
//
// The linear part of the effective field, exchange + periodic demagnetization
// + uniaxial anisotropy, is one symmetric 3x3 Fourier multiplier (FieldArgs in
// pipeline.h): the anisotropy matrix 2K e e^T is constant in space, so it
// commutes with the DFT.  Unlike the scalar multipliers of the Krylov
// operators it couples the three components, so the last axis pass takes the
// same columns of all three half spectra in one block:
//   2D: x-forward, y (forward, multiplier, inverse), x-inverse
//   3D: x-forward, y-forward, z (forward, multiplier, inverse), y-inverse, x-inverse
// The pipeline runs once per Picard iteration (right-hand side), per energy
// or diagnostic evaluation, and per adjoint Krylov iteration when the
// lower-order field is present; the forward Krylov operators do not use it.
#include "pipeline_run.h"

namespace llg {

// Columns of one half spectrum per block (three times as many in all).
__host__ __device__ constexpr int field_wk(int n) { return n >= 256 ? 4 : 8; }

// k_axis_field: lines along y or z of field_wk(N) columns of the three
// components: forward DFT, multiplier, inverse DFT.  After the forward DFT
// every value goes to LDS once, and each thread reads the three components of
// its positions.  As passes of their own (forward, multiplier, inverse) this
// moved the spectra three times: 76 us at 192 x 160 x 96 against 53 us.
// Row segments are not aligned to cache lines (a half spectrum has nh + 1
// columns), so each XCD takes a contiguous range of blocks and finds the
// other half of a line in its L2.
template <int N>
__global__ __launch_bounds__(3 * field_wk(N) * (N / plan_p(axis_plan_key(8, N)))) void k_axis_field(
    cx<double>* __restrict__ spec, SpecGeom g, int axis, FieldArgs fa, const cx<double>* __restrict__ tw) {
  using T = double;
  constexpr int KEY = axis_plan_key(8, N), P = plan_p(KEY), TPL = N / P, WK = field_wk(N), W = 3 * WK;
  __shared__ cx<T> lds[N * (W + 1)];
  const int c = threadIdx.x % W, t = threadIdx.x / W;
  const int comp = c / WK, kc = c % WK;
  const unsigned nb = gridDim.x * gridDim.y, lin = blockIdx.x + gridDim.x * blockIdx.y;
  const unsigned xcd = lin % 8, per = nb / 8, rem = nb % 8;
  const unsigned logical = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + lin / 8;
  const int kx = int(logical % gridDim.x) * WK + kc, outer = int(logical / gridDim.x);
  const long long sp = axis == 1 ? g.rs : (long long)g.rs * g.ny;
  const long long so = axis == 1 ? (long long)g.rs * g.ny : g.rs;
  const bool valid = kx <= g.nh;
  cx<T>* base = spec + outer * so + (valid ? comp * (g.nh + 1) + kx : 0);
  cx<T> v[P];
#pragma unroll
  for (int q = 0; q < P; ++q) v[in_slot<KEY>(q)] = base[(t + TPL * q) * sp];
  if (!valid) {
#pragma unroll
    for (int q = 0; q < P; ++q) v[q] = cx<T>{T(0), T(0)};
  }
  cx<T>* col_lds = lds + c;
  auto acc = [col_lds](int pos) -> cx<T>& { return col_lds[pos * (W + 1)]; };
  line_fft<T, KEY, -1>(v, t, acc, tw, 1);
  __syncthreads();
#pragma unroll
  for (int s = 0; s < P; ++s) acc(t + TPL * out_q<KEY>(s)) = v[s];
  __syncthreads();
  const double xx = fa.cx * kx;
  const double dx = kx == g.nh ? 0.0 : xx;  // derivative wave vector: Nyquist entries are zero
  const double e[3] = {fa.e0, fa.e1, fa.e2};
  cx<T> w[P];
#pragma unroll
  for (int s = 0; s < P; ++s) {
    const int q = out_q<KEY>(s), kp = t + TPL * q;
    const int ka = kp < N / 2 ? kp : kp - N;
    const int ko = axis == 1 ? 0 : (outer < g.ny / 2 ? outer : outer - g.ny);
    const int ky = axis == 1 ? ka : ko, kz = axis == 1 ? 0 : ka;
    const double yy = fa.cy * ky, zz = axis == 1 ? 0.0 : fa.cz * kz;
    const double s2 = xx * xx + yy * yy + zz * zz;
    const double dw[3] = {dx, ky == -g.ny / 2 ? 0.0 : yy, kz == -g.nz / 2 ? 0.0 : zz};
    const double qd = s2 > 0.0 ? fa.s_dm / s2 : 0.0;
    const double d = fa.s_id + fa.s_ex * s2;
    const cx<T>* row = lds + kp * (W + 1) + kc;
    const cx<T> u0 = row[0], u1 = row[WK], u2 = row[2 * WK];
    const double wu_r = dw[0] * u0.x + dw[1] * u1.x + dw[2] * u2.x;
    const double wu_i = dw[0] * u0.y + dw[1] * u1.y + dw[2] * u2.y;
    const double eu_r = e[0] * u0.x + e[1] * u1.x + e[2] * u2.x;
    const double eu_i = e[0] * u0.y + e[1] * u1.y + e[2] * u2.y;
    const double wc = comp == 0 ? dw[0] : (comp == 1 ? dw[1] : dw[2]);
    const double ec = comp == 0 ? e[0] : (comp == 1 ? e[1] : e[2]);
    const double re = d * v[s].x + qd * wc * wu_r + fa.s_an * ec * eu_r;
    const double im = d * v[s].y + qd * wc * wu_i + fa.s_an * ec * eu_i;
    w[in_slot<KEY>(q)] = cx<T>{re * fa.inv_ng, im * fa.inv_ng};
  }
  line_fft<T, KEY, 1>(w, t, acc, tw, 1);
  if (valid) {
#pragma unroll
    for (int s = 0; s < P; ++s) base[(t + TPL * out_q<KEY>(s)) * sp] = w[s];
  }
}

template <int N>
static hipError_t axis_field_n(const Ctx& c, int axis, const FieldArgs& fa, hipStream_t st) {
  constexpr int W = 3 * field_wk(N), TPL = N / plan_p(axis_plan_key(8, N));
  const dim3 grid((unsigned)((c.geom.nh + field_wk(N)) / field_wk(N)), (unsigned)(axis == 1 ? c.nz : c.ny));
  ProfScope ps(c.prof, st, KK_FIELD3, 2.0 * c.geom.cs * double(c.ny) * c.nz * sizeof(cx<double>));
  hipLaunchKernelGGL((k_axis_field<N>), grid, dim3(W * TPL), 0, st, reinterpret_cast<cx<double>*>(c.spec), c.geom,
                     axis, fa, c.tw_d[axis]);
  return hipGetLastError();
}

static hipError_t launch_axis_field(const Ctx& c, int axis, const FieldArgs& fa, hipStream_t st) {
  switch (axis == 1 ? c.ny : c.nz) {
#define LLG_CASE(v) \
  case v: return axis_field_n<v>(c, axis, fa, st);
    LLG_FOR_AXIS(LLG_CASE)
#undef LLG_CASE
    default: return hipErrorInvalidValue;
  }
}

template <int NH>
static hipError_t field_nh(const Ctx& c, const FieldArgs& fa, int epi, const NodalArgs& na,
                           const PipeIO<double, double, double>& io, hipStream_t st) {
  using T = double;
  launch_xfwd<T, T, T, NH, PRO_COPY3>(c, na, io, st);
  cx<T>* spec = reinterpret_cast<cx<T>*>(c.spec);
  const SymArgs none{};
  hipError_t e;
  if (c.dim == 2) {
    if ((e = launch_axis_field(c, 1, fa, st)) != hipSuccess) return e;
  } else {
    if ((e = launch_axis<T>(c, 1, 0, none, spec, st)) != hipSuccess) return e;
    if ((e = launch_axis_field(c, 2, fa, st)) != hipSuccess) return e;
    if ((e = launch_axis<T>(c, 1, 1, none, spec, st)) != hipSuccess) return e;
  }
  switch (epi) {
    case EPI_STORE3: launch_xinv<T, T, T, NH, EPI_STORE3>(c, na, io, st); break;
    case EPI_RHS: launch_xinv<T, T, T, NH, EPI_RHS>(c, na, io, st); break;
    case EPI_ADDF: launch_xinv<T, T, T, NH, EPI_ADDF>(c, na, io, st); break;
    case EPI_JT: launch_xinv<T, T, T, NH, EPI_JT>(c, na, io, st); break;
    case EPI_ENERGY: launch_xinv<T, T, T, NH, EPI_ENERGY>(c, na, io, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t run_field(const Ctx& c, const FieldArgs& fa, int epi, const NodalArgs& na,
                     const PipeIO<double, double, double>& io, hipStream_t st) {
  switch (c.geom.nh) {
#define LLG_CASE(n) \
  case n: return field_nh<n>(c, fa, epi, na, io, st);
    LLG_FOR_NH(LLG_CASE)
#undef LLG_CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace llg
