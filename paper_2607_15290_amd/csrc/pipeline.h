// Spectral pipeline: layout, argument blocks, prologue / epilogue modes.
//
// A pipeline applies one real, even Fourier multiplier to three real grid
// planes ("filtered fields") and combines the result node by node with other
// planes.  Every operator of the hot path is such a pipeline:
//
//   matvec      A x         : filtered v with a + b|xi|^2, a = alpha,
//                             b = theta k C_hat (Sec. 2.4, eq. "saddle point
//                             system"), epilogue adds m x v + m r, -m.v
//   apply       M^{-1} p    : filtered p_v with 1/(alpha + lambda + b|xi|^2)
//                             (Algorithm 1), epilogue = closed-form 4x4
//                             nodal inverse (eq. "inverse S")
//   apply^T     M^{-T} p    : prologue = transposed nodal inverse, then
//                             Algorithm 1
//   fused       M^{-1} A x  : M2^{-1}[x + M1^{-1}((calS - lambda I) x)], an
//                             identity because A = M1 + calS - lambda I
//   adjoint     J^T M^{-T} y: [I + (N - lambda I) M1^{-1}] M2^{-T} y, N = J^T -
//                             calH node-wise (the midpoint Jacobian, no
//                             lower-order field); right preconditioning
//   rhs         C_hat Delta_N m + (1+alpha^2) h (Sec. 2.4, eq. "total system")
//
// Grid planes are SoA, node index i = x + nx (y + ny z).  Between passes the
// three filtered fields live in one complex spectral buffer: each (y, z) row
// holds three half spectra (kx = 0..nx/2) back to back, 3 (nx/2+1) complex
// values, padded to a row stride rs that is a multiple of 16 elements.
#pragma once
#include "fft_core.h"

namespace llg {

// Line lengths with kernel instantiations: half-lengths nx/2 of the x passes
// and lengths of the y / z passes (plans in fft_core.h).
#define LLG_FOR_NH_LO(X) X(2) X(3) X(4) X(5) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32)
#define LLG_FOR_NH_HI(X) X(40) X(48) X(64) X(80) X(96) X(128) X(160) X(192) X(256)
#define LLG_FOR_NH(X) LLG_FOR_NH_LO(X) LLG_FOR_NH_HI(X)
constexpr int kNhLoMax = 32;  // the pipelines of the two halves are separate translation units
#define LLG_FOR_AXIS(X) \
  X(4) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64) X(80) X(96) X(128) X(160) X(192) \
  X(256) X(320) X(384) X(512)

// FFT plan key of the x passes for elements of elem_bytes bytes and half-length
// nh: the float64 passes at nh = 128, 256 take the finer plan (fewer points
// per thread, half the LDS per block; see kPlanFine).
__host__ __device__ constexpr int x_plan_key(int elem_bytes, int nh) {
  return (elem_bytes == 8 && (nh == 128 || nh == 256)) ? (nh | kPlanFine) : nh;
}

// Launch shapes of the x passes (rows = x lines per block).  Wide: 192 threads
// that each hold a part of a line of one of the three fields; streams best
// when there are several blocks per CU.  Mid and small: 256 threads, some of
// which only load, store and reduce, on the rows that hold about 256 or 64
// node pairs, so that grids of few rows still reach every CU.
enum XShape : int { X_WIDE = 0, X_MID = 1, X_SMALL = 2 };
__host__ __device__ constexpr int x_lx(int elem_bytes, int nh, int shape) {
  const int tpl = nh / plan_p(x_plan_key(elem_bytes, nh));
  if (shape == X_WIDE) return 64 / tpl;
  const int pairs = shape == X_MID ? 256 : 64, most = 64 / tpl;
  const int lx = nh >= pairs ? 1 : pairs / nh;
  return lx < most ? lx : most;
}
inline unsigned x_blocks(int elem_bytes, int nh, long long lines, int shape) {
  const int lx = x_lx(elem_bytes, nh, shape);
  return unsigned((lines + lx - 1) / lx);
}
// Shape of the x passes on a grid: wide above LLG_X_WIDE_BLOCKS wide blocks
// (one per CU), otherwise the mid shape if it gives a block to nearly every
// CU.  Solves (float64, left float32 form; blocks in brackets) on both sides:
//  * wide line at 640: 160 x 96 x 80 (480 wide) 6044 -> 6695 us, 4476 -> 4349:
//    bound by bytes, and 36 of the mid shape's 256 threads hold a part of a
//    line; 96^3 (576) 4896 -> 4926, 3826 -> 3657; 128 x 64 x 48 (384) 2533 ->
//    2354, 2149 -> 1900;
//  * wide line at 128, which leaves CUs idle: 512^2 (256 wide in float64, 128
//    in float32) 1634 -> 1834, 1298 -> 1324; 64^3 (256) 1878 -> 1987, 1545 ->
//    1683; 80^3 (200) 3176 -> 3462, 2673 -> 2871;
//  * mid line at 100: 256^2 (128 mid) 747 -> 822, 870 -> 907; 80 x 40 x 24
//    (160) 1178 -> 1053, 1359 -> 1281;
//  * mid line at 300: 48^3 (231) 1104 -> 1425, 1250 -> 1279; 80 x 40 x 32 (214)
//    1127 -> 1441, 1298 -> 1373; 128 x 24 x 32 (192) 1037 -> 1084, 1042 -> 1052.
#ifndef LLG_X_WIDE_BLOCKS
#define LLG_X_WIDE_BLOCKS 256
#endif
#ifndef LLG_X_MID_BLOCKS
#define LLG_X_MID_BLOCKS 192
#endif
inline int x_shape(int elem_bytes, int nh, long long lines) {
  if (x_blocks(elem_bytes, nh, lines, X_WIDE) > LLG_X_WIDE_BLOCKS) return X_WIDE;
  return x_blocks(elem_bytes, nh, lines, X_MID) >= LLG_X_MID_BLOCKS ? X_MID : X_SMALL;
}

// Whether the x-forward pass of a shape can carry a riding reduction
// (RideReduce).  The branch costs the wide passes of large grids, which never
// take it, 1.1 us of 403 in the float32 M^{-1} x at 256^3, so it is left out
// there: a wide pass of few enough nodes (kRideMaxBlocks) has lines of at
// most 16 nodes.
__host__ __device__ constexpr bool x_rides(int nh, int shape) { return shape != X_WIDE || nh <= 8; }

// FFT plan key of the y / z passes: with LLG_AXIS_FINE_F64 the float64
// passes at N = 256 take the finer plan as well.
#ifndef LLG_AXIS_FINE_F64
#define LLG_AXIS_FINE_F64 0
#endif
__host__ __device__ constexpr int axis_plan_key(int elem_bytes, int n) {
  return (LLG_AXIS_FINE_F64 && elem_bytes == 8 && n == 256) ? (n | kPlanFine) : n;
}

inline bool nh_supported(int n) {
#define LLG_EQ(v) || n == v
  return false LLG_FOR_NH(LLG_EQ);
}
inline bool axis_supported(int n) { return false LLG_FOR_AXIS(LLG_EQ); }
#undef LLG_EQ

struct SpecGeom {
  int nx, ny, nz, nh;  // nh = nx / 2
  int cs;              // 3 (nh + 1) valid columns per row
  int rs;              // row stride in complex elements
  long long ng;        // nodes
};

struct SymArgs {
  double a, b;           // multiplier a + b |xi|^2 (or its inverse)
  double cx, cy, cz;     // 2 pi / L per axis
  double inv_ng;         // 1 / N_g
  int invert;            // 1: use 1 / (a + b |xi|^2)
};

struct NodalArgs {
  double lam;            // HSS shift lambda
  double hs;             // 1 + alpha^2 (field scaling)
  double chat;           // C_hat
  double hu0, hu1, hu2;  // uniform applied field
  double half_k;         // k / 2 (adjoint operator)
  const double* hfield;  // optional spatial field (3 planes) or null
};

enum ProMode : int {
  PRO_NONE = -1,   // no x-forward pass: the spectral buffer already holds the
                   // filtered fields' x spectra (left by k_xfwd_upd)
  PRO_COPY3 = 0,   // u = in[0..2]
  PRO_SMINUS = 1,  // u = m x v + m r - lambda v  (first half of the fused op)
  PRO_M2T = 2,     // u = ((lambda I + S~) p)_v / (lambda^2 + |m|^2)
};

enum EpiMode : int {
  EPI_STORE3 = 0,    // out[0..2] = F
  EPI_APPLY = 1,     // out = M2^{-1} (F, p_r / lambda)
  EPI_APPLY_T = 2,   // out = (F, ((lambda I + S~) p)_r / (lambda d))
  EPI_MATVEC = 3,    // out = (F + m x v + m r, -m.v)
  EPI_MATVEC_T = 4,  // out = (F - m x v - m r, m.v)
  EPI_FUSED = 5,     // out = M2^{-1} (x + (F, (-m.v - lambda r) / lambda))
  EPI_RHS = 6,       // out = (-C_hat F + (1+alpha^2) h, 0)
  EPI_JT = 7,        // out = J^T mu of the midpoint residual (adjoint), F = H mu_v
  EPI_APPLY_SYM = 8, // out = (F, p_r / lambda): (lambda I + calH)^{-1} p alone
  EPI_FUSED_SYM = 9, // out = x + (F, (-m.v - lambda r) / lambda): (lambda I + calH)^{-1} A x
  EPI_ADDF = 10,     // out = (aux_v - (1+alpha^2) F, 0): right-hand side with the lower-order field
  EPI_ENERGY = 11,   // no output: per-block partial sums of chat/2 m.F - m.h (discrete energy density)
  EPI_JT_RIGHT = 12, // out = J^T M^{-T} y of the midpoint adjoint, right-preconditioned (one pipeline,
                     // prologue PRO_M2T on m = m_half, F = (calH + lambda I)^{-1} of the prologue)
};

// Symmetric 3x3 Fourier multiplier of the lower-order field pipeline:
//   M(xi) = (s_id + s_ex |xi|^2) I + s_dm xi~ xi~^T / |xi|^2 + s_an e e^T,
// xi~ = xi with the Nyquist entry of each axis set to zero (spectral first
// derivative of real data), the demagnetizing term zero at xi = 0.  With
// s_id = 0, s_ex = cexc, s_dm = demag, s_an = -2K the output is minus the
// linear part of the effective field (exchange, periodic demagnetization of
// Sec. 2.2, uniaxial anisotropy of Sec. 2.1).
struct FieldArgs {
  double s_id, s_ex, s_dm, s_an;
  double e0, e1, e2;   // easy axis
  double cx, cy, cz;   // 2 pi / L per axis
  double inv_ng;
};

// Pointers of one pipeline call.  "in" planes feed the prologue (and are
// re-read by epilogues that need x or p); "m" is the magnetization the
// nodal blocks are built on.
template <typename T, typename TIn, typename TOut>
struct PipeIO {
  const TIn* in;     // 4 planes (x or p), or 3 planes for PRO_COPY3 + EPI_STORE3/RHS
  const T* m;        // 3 planes (may be null for modes that do not use it)
  TOut* out;         // 4 planes (3 for EPI_STORE3)
  long long ng;
  const T* aux_v;    // EPI_JT, EPI_JT_RIGHT: forward velocity v (3 planes)
  const T* aux_r;    // EPI_JT, EPI_JT_RIGHT: forward multiplier (1 plane)
  // Residual form: when rhs is set, the pipeline writes out = rhs - (operator
  // output) and each x-inverse block stores the partial sum of squares of its
  // outputs at red[blockIdx.x].  EPI_ENERGY writes no output and stores the
  // block's partial sum of the energy density at red[blockIdx.x].
  const TOut* rhs = nullptr;
  double* red = nullptr;
  // EPI_RHS: when set, the filtered fields F = (-Delta_N) in (3 planes) are
  // stored here as well.
  T* out_f = nullptr;
};

// Results of a reduction for the host (device side of await_post): the values
// go to their slots of the mapped host mirror, n_also further values are
// copied there, and once every block's values are visible the last block sets
// the host flag to seq.  The host polls the flag: no event or copy enters the
// stream, and the wait ends as soon as the values arrive.
struct Post {
  double* mirror = nullptr;  // device address of the mirror slots of out
  const double* also = nullptr;
  double* also_mirror = nullptr;
  int n_also = 0;
  unsigned* count = nullptr;
  unsigned long long* flag = nullptr;  // null: nothing to post
  unsigned long long seq = 0;
};
// A reduction (nv rows of nb block partials, value-major, into out and the
// Post) that rides in the next x-forward pass as its last block: on small grids
// it takes the place of a launch of its own between two passes.
struct RideReduce {
  const double* part = nullptr;
  int nb = 0, nv = 0;  // nv = 0: nothing rides
  double* out = nullptr;
  Post post;
};
// Most update blocks of a pass whose reduction rides: the one block that sums
// them ends with the pass around it up to there.  With the line at 500 blocks
// float64 solves at 384^2 (576) 1232 -> 1307 us, 512^2 (1024) 1597 -> 1657, 64^3
// (1024) 1880 -> 1919; at 4400 64 x 64 x 80 (1280) 2397 -> 2315, 128 x 64 x 48
// (1536) 2632 -> 2556, 80^3 (2016) 3179 -> 3206, 128 x 128 x 64 (4096) 5368 ->
// 5464.
constexpr int kRideMaxBlocks = 1100;

// Arnoldi inner products taken by an x-inverse pass on its own output (the
// precision form's matvec): with basis directions u_0 at u0 and u_i at
// U1 + (i - 1) ld (1 <= i < nv), each block stores the partial sums of
// u_i . out over its nodes at partial[i * gridDim.x + blockIdx.x].
constexpr int kBasisDotsMax = 32;
struct BasisDots {
  const double* u0 = nullptr;
  const double* U1 = nullptr;
  long long ld = 0;
  int nv = 0;
  double* partial = nullptr;
  double* out = nullptr;  // when set, the reduced products go here instead of the caller's default
  // Deferred reduction (small grids): when defer is set and the pass has few
  // enough blocks (kDeferMaxSums), it leaves its block partials at defer
  // (value-major) instead of reducing them and stores its block count at
  // *defer_nb; otherwise it reduces as usual (products at out) and stores 0.
  // The Arnoldi update pass reduces deferred partials.
  double* defer = nullptr;
  int* defer_nb = nullptr;
  const RideReduce* ride = nullptr;  // reduction carried by the operator's x-forward pass
};
// Products are left for deferred reduction when the partials per value times
// the blocks of the update pass, each of which sums them all, are at most this
// (512^2: 512 x 1024).  With the line at 2^18 float64 solves at 512^2 1597 ->
// 1566 us and 64^3 (2^19) 1880 -> 1827, the precision forms within 1%; at 2^21
// 96 x 64 x 48 (2^19.4) 1899 -> 1992, 80 x 64 x 64 (2^19.8) 2071 -> 2222, 96 x
// 64 x 64 (2^20.3) 2450 -> 2675, the precision forms 0.3-2.6% slower.
constexpr long long kDeferMaxSums = 1 << 19;

// Delayed-CGS2 pass 2 of Arnoldi step j carried by the first x pass of the
// operator of step j + 1 (k_xfwd_upd): with basis directions u_0 at u0 and
// u_q at U1 + (q - 1) ld, the pass forms
//   u_new = (w - sum_{q <= j} gamma_q u_q) * inv_beta
// node by node, stores it at unew (the next basis direction), feeds it to
// the operator's prologue, and leaves the block partials of u_q . u_new
// (q <= j) and u_new . u_new at partial[q * gridDim.x + blockIdx.x],
// q = 0 .. j + 1.
struct UpdFirst {
  const double* u0 = nullptr;
  const double* U1 = nullptr;
  long long ld = 0;
  int j = 0;
  const double* gamma = nullptr;  // j + 1 coefficients (device)
  const double* p = nullptr;      // pass-1 products (posted to the host with the new ones)
  double inv_beta = 0;
  double* unew = nullptr;         // must not alias w or a basis column 0..j
  double* partial = nullptr;
};

}  // namespace llg
