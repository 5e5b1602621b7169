// Axis-pass kernel: the directional spectral sub-step of the split step.
//
// One launch processes every pencil of the grid along one axis j and applies
//   PROP: v <- F_j^-1 ( m(k_j) * F_j v )         (S(s, L_j) with m = exp(-i alpha k_j^2 s)/N_j,
//                                                  or a spectral derivative with m = i k_j / N_j)
//   FWD : v <- scale * F_j v        (natural frequency order out)
//   INV : v <- scale * F_j^-1 v     (natural frequency order in, unnormalised inverse)
//   TURN: v <- S_2 P S_1 v, S_1 and S_2 two propagator sub-steps along the same axis and P
//         the pointwise sub-step between them (see below)
// with optional pointwise prologues (the nonlinear sub-step S(dt, N), its adjoint) fused in
// front of the transform, and passes that only sum what they transform.
//
// Transform structure (time-evolution section: each S(s, L_j) is exact in Fourier space):
// N = R_0 R_1 ... R_{S-1}; T threads per pencil each hold E = N/T points in registers.
// Forward stages are decimation-in-frequency butterflies done in registers, with an
// LDS exchange between stages; after the last stage position p holds the coefficient
// of the digit-reversed frequency.  PROP multiplies there by a table already stored in
// that order and runs the exact inverse (conjugate-twiddle DIT) stages in reverse, so
// no reordering pass is ever needed.  W pencils share one workgroup; for the strided
// axes (y, z) the W pencils are x-adjacent so each global access is a W*S-byte row.
//
// TURN: the linear sub-steps of one time step commute, so a run may take the axes of its
// steps in alternating order (x y z | z y x | x y z ...).  Then the last sub-step of one
// step, the nonlinear rotation and the first sub-step of the next act on the same
// pencils and run in one pass, without psi leaving the registers in between: a step
// reads and writes psi twice instead of three times (once for two axes or with the
// xy-plane pass).
//
// Table layouts (built on the host for the schedule in use): every table load of one
// instruction reads consecutive entries across the lanes, so it costs a few vector-L1
// requests instead of one per lane.
//   multiplier / k^2: the entry of position g*R_last + r is stored at r*(N/R_last) + g
//                     (g = t + T*j runs over the lanes of one load)
//   twiddles        : stage s keeps W_{R_s M_s}^{lo k} at TWOFF(s) + (k-1)*M_s + lo
#pragma once

#include "gp_device.h"

namespace gpk {

// global-memory pointers: accesses through them are global (not flat) instructions,
// which count on the vector-memory counter only (the qualifier is for the device
// compilation pass; the host pass only checks the kernel bodies)
#if defined(__HIP_DEVICE_COMPILE__)
#define GPK_GLOBAL __attribute__((address_space(1)))
#else
#define GPK_GLOBAL
#endif
template <class X>
__device__ __forceinline__ const GPK_GLOBAL X* gptr(const void* p) { return (const GPK_GLOBAL X*)p; }
template <class X>
__device__ __forceinline__ GPK_GLOBAL X* gptr_mut(void* p) { return (GPK_GLOBAL X*)p; }

// A table pointer the compiler cannot tell from another: two sub-steps in one kernel read
// their twiddles from the same table, and keeping a stage's 15 to 31 entries from the first
// for the second costs 60 to 120 registers a lane (1024 points: spills to scratch memory).
__device__ __forceinline__ const void* reload(const void* p) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+s"(p));
#endif
  return p;
}

// Keeps the operations that make these values ahead of the next in_order's.
template <class Real>
__device__ __forceinline__ void in_order(double& acc, cplx<Real>& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(acc), "+v"(v.x), "+v"(v.y));
#endif
}

enum PassKind { CONTIG = 0, STRIDED = 1 };
enum PassMode { PROP = 0, FWD = 1, INV = 2, TURN = 3 };
// pointwise work fused in front of the transform (PRO_DERIV: none; the multiplier is that
// of a spectral derivative, i k_j / N_j, and sum k_j^2 |F_j v|^2 is accumulated for the
// kinetic energy;
// PRO_ARGLE: none, but turn the derivative after the inverse transform into the
// explicit part of the imaginary-time step and that into its transform, stored in lane
// order; PRO_MULT3: none, but multiply the
// forward transform by the separable 3-D propagator m_x(k_x) m_y(k_y) m_z(k_z) before
// it is stored -- the last forward pass of the literal 3-D form)
// PRO_HESS (FWD): J = Im sum_j conj(F_j) d F_j along the axis, F_j the three fields in, aux, aux2.
// Lane order: the coefficients along an axis as the lanes hold them after the forward stages,
// the entry of table index li at li.  Between passes that agree on the schedule it needs no
// reordering exchange, and it is as coalesced as the natural order.  PRO_LANE (FWD, INV): such
// output, such input.  PRO_SOLVE (FWD): the diagonal solve of the imaginary-time step and the
// inverse transform after the forward one.  PRO_LANE_D (INV): PRO_LANE, and the derivative
// along the axis from the same coefficients.
// In a TURN pass: the work between its two sub-steps (PRO_NL, PRO_ADJ_NL, or PRO_TAPE:
// store the state there as well, then rotate it).  PRO_SWAP: none; the pass exchanges the
// two outer axes of the layout (see pencil_pair).  PRO_ENERGY (FWD): sums only, nothing is
// stored: k_j^2 |F_j v|^2 and, where point_partial is given, |v|^2 and (|v|^2 - 1)^2.
// PRO_POWER, PRO_VPOWER (FWD): power sums only, sum over the tile's pencils of |F_j f|^2 per
// frequency, f = |v|^2 - 1 or the velocity 2 alpha Im(conj(v) d_j v)/|v|^2 along the axis,
// whose derivative is taken in the same pass; PRO_VPOWER also sums f^2 (point_partial).
enum Prologue { PRO_NONE = 0, PRO_NL = 1, PRO_ADJ_NL = 2, PRO_DERIV = 4, PRO_ARGLE = 5, PRO_MULT3 = 6,
                PRO_TAPE = 7, PRO_SWAP = 8, PRO_ENERGY = 9, PRO_POWER = 10, PRO_VPOWER = 11,
                PRO_LANE = 12, PRO_SOLVE = 13, PRO_LANE_D = 14, PRO_HESS = 15 };

// per-run pointers of a grouped (ensemble) launch: run = blockIdx.y
struct RunPtrs {
  const void* in;
  void* out;
  const void* mult;
  const void* mult2;       // turning passes: the multipliers of the second sub-step
  double nl_coef;
};

struct PassArgs {
  const RunPtrs* batch;    // grouped launch over runs of one size, or null
  const void* in;          // input field (complex, working precision)
  void* out;               // output field (may equal in)
  const void* mult;        // PROP: multiplier in lane order (N_j FP64 complex entries)
  const void* mult2;       // TURN: multiplier of the second sub-step
  const void* tw;          // per-stage twiddles W_{R M}^{lo k} (Tab<Real> entries, layout above)
  const void* aux;         // PRO_ADJ_NL, PRO_ARGLE: the state phi at the same points;
                           // PRO_MULT3: m_x in natural frequency order (FP64 complex)
  const void* aux2;        // PRO_ARGLE: d phi / dx and d phi / dy at the same points;
  const void* aux3;        // PRO_MULT3: m_y and m_z
                           // PRO_SOLVE: k_x^2 and k_z^2 in lane order (aux, aux2)
  void* tape;              // PRO_TAPE: where the state between the sub-steps is stored;
                           // PRO_SOLVE: the transform of phi, in and out; PRO_LANE_D: d_j v
  const void* vel;         // PRO_ARGLE: velocity planes v_x, v_y, v_z (Real, one field each)
  double q4a;              // PRO_ARGLE: 1 / (4 alpha); PRO_SOLVE: dtau alpha / 2 (nl_coef: dtau)
  const double* ksq;       // k_j^2 in position order (kinetic accumulation)
  double* kin_partial;     // per-workgroup partial sum of k_j^2 |F_j v|^2 (or null)
  double* point_partial;   // PRO_ENERGY: per-workgroup sums of |v|^2, then of (|v|^2 - 1)^2, or null
  double nl_coef;          // beta * dt of the nonlinear prologue
  double scale;            // FWD/INV output scale
  long npencils;           // number of pencils along this axis
  long inner, outer;       // pencil p starts at (p / inner) * outer + (p % inner)
  long es;                 // element stride along the axis
  int axis;                // PRO_MULT3: the pass's axis (0 x, 1 y, 2 z) ...
  int nx, ny;              // ... and the grid's x and y lengths (PRO_SWAP: ny = nz)
};

template <int N_, int T_, int W_, int R0, int R1, int R2>
struct Sched {
  static constexpr int N = N_, T = T_, W = W_, E = N_ / T_;
  static constexpr int NS = (R0 > 1) + (R1 > 1) + (R2 > 1);
  static constexpr int rad(int s) { return s == 0 ? R0 : s == 1 ? R1 : R2; }
  // product of the radices after stage s (the digit weight of stage s)
  static constexpr int M(int s) { int m = 1; for (int i = s + 1; i < NS; ++i) m *= rad(i); return m; }
  // product of the radices before stage s (the frequency weight of stage s)
  static constexpr int K(int s) { int k = 1; for (int i = 0; i < s; ++i) k *= rad(i); return k; }
  // twiddle sub-table of stage s: entries W_{R M}^{lo k} at (k-1)*M(s) + lo, stages with
  // M(s) > 1 stored one after another
  static constexpr int TWOFF(int s) {
    int o = 0;
    for (int i = 0; i < s; ++i) if (M(i) > 1) o += (rad(i) - 1) * M(i);
    return o;
  }
  static constexpr bool valid() {
    if (T * E != N) return false;
    int p = 1;
    for (int s = 0; s < NS; ++s) { if (E % rad(s)) return false; p *= rad(s); }
    return p == N;
  }
  static_assert(valid(), "inconsistent FFT schedule");
  static constexpr int THREADS = T * W;
  static constexpr int RL = rad(NS > 0 ? NS - 1 : 0);     // radix of the last stage
};

// Lanes of one pencil in the contiguous mapping: TL consecutive lanes on one pencil
// (a 128-byte segment, or the whole pencil when it is shorter).
template <class S, int SZ>
constexpr int lanes_per_pencil() { return (S::T * SZ <= 128) ? S::T : 128 / SZ; }

// Smallest pitch >= n, in points of SZ bytes, that sets the rows of one LDS cycle
// apart by whole lane groups.  The LDS serves 128 bytes per cycle (16 lanes of a
// 64-bit access, 8 of a 128-bit one); with TL lanes per row, 128/(SZ TL) rows share a
// cycle and a pitch of TL modulo 128/SZ points puts each row on its own banks.  With
// one row per cycle the pitch is kept at 128 B modulo 256 B.
template <int SZ>
constexpr int row_pitch(int n, int TL) {
  int c = n;
  if (128 % SZ != 0) return c;
  const int slots = 128 / SZ;
  if (TL < slots) {
    while (c % slots != TL % slots) ++c;
  } else {
    while (c % (2 * slots) != slots) ++c;
  }
  return c;
}

// LDS layout of the stage exchanges (SZ = bytes per element).
//   CONTIG  [col][pos + pos/RL + pad]: one pad element every RL positions spreads the
//           stride-RL accesses of the last stage over the banks; the column pitch
//           (row_pitch) gives the pencils that share an LDS cycle different banks.
//   STRIDED [pos + pos/RL][col]: one pad row every RL rows, for the same reason.
template <class S, int SZ, int KIND>
struct Lds {
  static constexpr int PADN = S::N + S::N / S::RL;
  static constexpr int cpitch() { return row_pitch<SZ>(PADN, lanes_per_pencil<S, SZ>()); }
  static constexpr int CP = cpitch();
  static constexpr int ELEMS = (S::NS > 1) ? (KIND == CONTIG ? S::W * CP : PADN * S::W) : 1;
  static __device__ __forceinline__ int addr(int pos, int col) {
    if constexpr (KIND == CONTIG) return col * CP + pos + pos / S::RL;
    else return (pos + pos / S::RL) * S::W + col;
  }
};

// position held by register (j + B*r) of thread t at stage s
template <class S, int s>
__device__ __forceinline__ int stage_pos(int t, int j, int r) {
  constexpr int Ms = S::M(s);
  constexpr int Ls = S::rad(s) * Ms;
  const int g = t + S::T * j;
  return (g / Ms) * Ls + r * Ms + (g % Ms);
}

// position of natural frequency k (digit-reversal of the DIF output order)
template <class S>
__host__ __device__ constexpr int freq_pos(int k) {
  int p = 0;
  for (int s = 0; s < S::NS; ++s) p += ((k / S::K(s)) % S::rad(s)) * S::M(s);
  return p;
}

template <class Real, class S, int KIND>
__device__ __forceinline__ int lds_addr(int pos, int col) {
  return Lds<S, (int)sizeof(cplx<Real>), KIND>::addr(pos, col);
}

// layout ids for exchanges: 0..NS-1 = stage layouts, -1 = natural frequency layout
template <class Real, class S, int KIND, int L>
__device__ __forceinline__ void put(cplx<Real>* lds, const cplx<Real>* v, int t, int col) {
  if constexpr (L < 0) {
#pragma unroll
    for (int e = 0; e < S::E; ++e) lds[lds_addr<Real, S, KIND>(freq_pos<S>(t + S::T * e), col)] = v[e];
  } else {
    constexpr int B = S::E / S::rad(L);
#pragma unroll
    for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
      for (int j = 0; j < B; ++j) lds[lds_addr<Real, S, KIND>(stage_pos<S, L>(t, j, r), col)] = v[j + B * r];
  }
}
template <class Real, class S, int KIND, int L>
__device__ __forceinline__ void get(const cplx<Real>* lds, cplx<Real>* v, int t, int col) {
  if constexpr (L < 0) {
#pragma unroll
    for (int e = 0; e < S::E; ++e) v[e] = lds[lds_addr<Real, S, KIND>(freq_pos<S>(t + S::T * e), col)];
  } else {
    constexpr int B = S::E / S::rad(L);
#pragma unroll
    for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
      for (int j = 0; j < B; ++j) v[j + B * r] = lds[lds_addr<Real, S, KIND>(stage_pos<S, L>(t, j, r), col)];
  }
}

template <class Real, class S, int KIND, int FROM, int TO>
__device__ __forceinline__ void exchange(cplx<Real>* lds, cplx<Real>* v, int t, int col) {
  __syncthreads();                          // previous readers of lds are done
  put<Real, S, KIND, FROM>(lds, v, t, col);
  __syncthreads();
  get<Real, S, KIND, TO>(lds, v, t, col);
}

// table entry i (32-bit index from the uniform table base; P is a global-memory or
// an LDS pointer)
template <class P>
__device__ __forceinline__ auto tab_at(P t, int i) {
  return t[(unsigned)i];
}

// forward DIF stage s: butterfly over digit s, then twiddle W_{L_s}^{lo*k}
template <class Real, class S, int s, class P>
__device__ __forceinline__ void fwd_stage(cplx<Real>* v, int t, P tw) {
  constexpr int R = S::rad(s), B = S::E / R, Ms = S::M(s);
#pragma unroll
  for (int j = 0; j < B; ++j) {
    cplx<Real> x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = v[j + B * r];
    Dft<R, -1, Real>::run(x);
    if constexpr (Ms > 1) {
      const int lo = (t + S::T * j) % Ms;
#pragma unroll
      for (int k = 1; k < R; ++k) x[k] = tmul(x[k], tab_at(tw, S::TWOFF(s) + (k - 1) * Ms + lo));
    }
#pragma unroll
    for (int k = 0; k < R; ++k) v[j + B * k] = x[k];
  }
}

// inverse of fwd_stage (up to the factor R): conjugate twiddle, then inverse butterfly
template <class Real, class S, int s, class P>
__device__ __forceinline__ void inv_stage(cplx<Real>* v, int t, P tw) {
  constexpr int R = S::rad(s), B = S::E / R, Ms = S::M(s);
#pragma unroll
  for (int j = 0; j < B; ++j) {
    cplx<Real> x[R];
#pragma unroll
    for (int k = 0; k < R; ++k) x[k] = v[j + B * k];
    if constexpr (Ms > 1) {
      const int lo = (t + S::T * j) % Ms;
#pragma unroll
      for (int k = 1; k < R; ++k) x[k] = tmulc(x[k], tab_at(tw, S::TWOFF(s) + (k - 1) * Ms + lo));
    }
    Dft<R, +1, Real>::run(x);
#pragma unroll
    for (int r = 0; r < R; ++r) v[j + B * r] = x[r];
  }
}

template <class Real, class S, int KIND, int s, class P>
__device__ __forceinline__ void forward_all(cplx<Real>* v, cplx<Real>* lds, int t, int col, P tw) {
  fwd_stage<Real, S, s, P>(v, t, tw);
  if constexpr (s + 1 < S::NS) {
    exchange<Real, S, KIND, s, s + 1>(lds, v, t, col);
    forward_all<Real, S, KIND, s + 1, P>(v, lds, t, col, tw);
  }
}

template <class Real, class S, int KIND, int s, class P>
__device__ __forceinline__ void inverse_all(cplx<Real>* v, cplx<Real>* lds, int t, int col, P tw) {
  inv_stage<Real, S, s, P>(v, t, tw);
  if constexpr (s > 0) {
    exchange<Real, S, KIND, s, s - 1>(lds, v, t, col);
    inverse_all<Real, S, KIND, s - 1, P>(v, lds, t, col, tw);
  }
}

// Complex64 tiles of whole contiguous pencils move between global memory and the
// lanes through the LDS exchange buffer with 16-byte accesses: unit u of the tile
// (u = tid + THREADS i) holds points 2q, 2q+1 of tile pencil u / (N/2), so one load or
// store instruction of a wavefront covers 1 KB of one pencil, against four 128-byte
// pieces of four pencils with one point per lane.  `pencil(pc)` is the element offset
// of tile pencil pc.  Complex128 points are 16 bytes already and move directly.
template <class S>
constexpr bool wide_io() { return S::NS > 1 && S::N % 2 == 0 && S::E % 2 == 0; }

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <class S, class F>
__device__ __forceinline__ void load_tile_wide(cplx<float>* v, cplx<float>* lds, const void* in, F pencil,
                                               int t, int col) {
  using L = Lds<S, 8, CONTIG>;
  constexpr int HN = S::N / 2, U = S::E / 2;
  const auto src = gptr<cplx<float>>(in);
  f32x4 r[U];
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const int u = (int)threadIdx.x + S::THREADS * i, pc = u / HN, q = u % HN;
    r[i] = *(const GPK_GLOBAL f32x4*)(src + pencil(pc) + 2 * q);
  }
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const int u = (int)threadIdx.x + S::THREADS * i, pc = u / HN, q = u % HN;
    lds[L::addr(2 * q, pc)] = mk(r[i].x, r[i].y);
    lds[L::addr(2 * q + 1, pc)] = mk(r[i].z, r[i].w);
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < S::E; ++e) v[e] = lds[L::addr(t + S::T * e, col)];
}

template <class S, class F>
__device__ __forceinline__ void store_tile_wide(const cplx<float>* v, cplx<float>* lds, void* out, F pencil,
                                                int t, int col) {
  using L = Lds<S, 8, CONTIG>;
  constexpr int HN = S::N / 2, U = S::E / 2;
  const auto dst = gptr_mut<cplx<float>>(out);
  __syncthreads();                          // the last exchange has been read
#pragma unroll
  for (int e = 0; e < S::E; ++e) lds[L::addr(t + S::T * e, col)] = v[e];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const int u = (int)threadIdx.x + S::THREADS * i, pc = u / HN, q = u % HN;
    const cplx<float> p0 = lds[L::addr(2 * q, pc)], p1 = lds[L::addr(2 * q + 1, pc)];
    *(GPK_GLOBAL f32x4*)(dst + pencil(pc) + 2 * q) = f32x4{p0.x, p0.y, p1.x, p1.y};
  }
}

// PRO_SWAP (x passes of grids with n = ny = nz, n even): pencil (z, y) is written where
// pencil (y, z) was and the reverse, in place, so the layout goes from [z][y][x] to
// [y][z][x] and back with the next such pass.  The axis that then has the stride nx can be
// transformed with rows that lie nx points apart instead of nx ny: at 1024^3 complex64 every
// row of a z tile falls in a memory page of its own and the turning pass takes 10.6 ms,
// against 7.0 with the y stride, while this pass still moves whole contiguous pencils.
// A tile holds W / 2 pairs {(i, j), (j, i)}, i <= j (a pencil of the diagonal fills both
// places, with equal bytes), which it has read completely before it writes.  Pairs
// are counted along row i together with row n - 1 - i, n + 1 pairs for the two.
__device__ __forceinline__ void pencil_pair(unsigned u, unsigned n, unsigned& i, unsigned& j) {
  const unsigned r = u / (n + 1), c = u % (n + 1);
  if (c < n - r) { i = r; j = r + c; }
  else { i = n - 1 - r; j = i + (c - (n - r)); }
}

// nonlinear sub-step S(dt, N): v <- v exp(-i beta (|v|^2 - 1) dt), in the working precision.
// SMALL: the angle is known to be within the short series' range.
template <bool SMALL>
__device__ __forceinline__ cplx<double> nl_rotate(cplx<double> v, double coef) {
  GPK_AS_WRITTEN
  double s, c;
  const double a = -coef * (cabs2(v) - 1.0);
  if constexpr (SMALL) sincos_small(a, &s, &c);
  else sincos_rot(a, &s, &c);
  return cmul(v, mk(c, s));
}
// FP32: v + v (cos a - 1 + i sin a), see sincos_m1; the small correction is formed
// first, so the result carries one rounding at the size of v
template <bool SMALL>
__device__ __forceinline__ cplx<float> nl_rotate(cplx<float> v, double coef) {
  GPK_AS_WRITTEN
  float s, cm1;
  const float a = -float(coef) * (cabs2(v) - 1.0f);
  if constexpr (SMALL) sincos_m1_small(a, &s, &cm1);
  else sincos_m1(a, &s, &cm1);
  const float dx = fmaf(v.x, cm1, -v.y * s), dy = fmaf(v.y, cm1, v.x * s);
  return mk(v.x + dx, v.y + dy);
}

// adjoint of the linearised nonlinear sub-step at phi:
//   lam <- conj(u) lam + 2 beta dt Im(conj(lam) u phi) phi,  u = exp(-i beta (|phi|^2-1) dt)
template <bool SMALL, class Real>
__device__ __forceinline__ cplx<Real> nl_adjoint(cplx<Real> lam, cplx<Real> phi, Real coef) {
  GPK_AS_WRITTEN
  Real s, c;
  const Real a = -coef * (cabs2(phi) - Real(1));
  if constexpr (SMALL) sincos_small(a, &s, &c);
  else sincos_rot(a, &s, &c);
  const cplx<Real> u = mk(c, s);
  const cplx<Real> up = cmul(u, phi);
  const Real im = fmadd(lam.x, up.y, -(lam.y * up.x));  // Im(conj(lam) * up)
  const cplx<Real> r = cmulc(lam, u);                    // conj(u) lam
  const Real f = Real(2) * coef * im;
  return mk(fmadd(f, phi.x, r.x), fmadd(f, phi.y, r.y));
}

// The rotations of all points a lane holds.  One branch for the lane: within the short
// series (kSmallAngle, which covers the time steps of the method's workloads) straight code
// for all points.  A lane with a larger angle takes the general routine point after point
// in a rolled loop that turns the register array by one place, and its wavefront both paths.
// (Unrolled with the general routine at every point, its code was 35 KB of a 43 KB
// kernel at 256 points complex128, 45 of 65 KB at 1024 points complex64, beside a
// 64 KB instruction cache that two compute units share: the turning pass took 13.7 ms
// at 1024^3 where the plain pass takes 3.6.)
template <class Real>
__device__ __forceinline__ bool angle_small(cplx<Real> v, Real coef) {
  GPK_AS_WRITTEN
  return fabs(coef * (cabs2(v) - Real(1))) <= Real(kSmallAngle);    // false for a NaN
}
template <int E, class Real>
__device__ __forceinline__ void rotate_points(cplx<Real>* v, double coef) {
  bool small = true;
#pragma unroll
  for (int e = 0; e < E; ++e) small = small && angle_small(v[e], Real(coef));
  if (small) {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = nl_rotate<true>(v[e], coef);
  } else {
#pragma unroll 1
    for (int i = 0; i < E; ++i) {
      const cplx<Real> x = nl_rotate<false>(v[0], coef);
#pragma unroll
      for (int e = 0; e + 1 < E; ++e) v[e] = v[e + 1];
      v[E - 1] = x;
    }
  }
}
// the same for the adjoint at the states phi
template <int E, class Real>
__device__ __forceinline__ void rotate_adjoint(cplx<Real>* v, cplx<Real>* phi, Real coef) {
  bool small = true;
#pragma unroll
  for (int e = 0; e < E; ++e) small = small && angle_small(phi[e], coef);
  if (small) {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = nl_adjoint<true>(v[e], phi[e], coef);
  } else {
#pragma unroll 1
    for (int i = 0; i < E; ++i) {
      const cplx<Real> x = nl_adjoint<false>(v[0], phi[0], coef);
#pragma unroll
      for (int e = 0; e + 1 < E; ++e) { v[e] = v[e + 1]; phi[e] = phi[e + 1]; }
      v[E - 1] = x;
    }
  }
}

template <class Real, class S, int KIND, int MODE, int PRO>
__global__ __launch_bounds__(S::THREADS) void axis_pass(PassArgs a) {
  using C = cplx<Real>;
  constexpr int T = S::T, W = S::W, E = S::E;
  // (power sums use the buffer for a double per point of the tile)
  constexpr bool POWER = PRO == PRO_POWER || PRO == PRO_VPOWER;
  constexpr int EXCH = Lds<S, (int)sizeof(C), KIND>::ELEMS, SUMS = S::N * W * 8 / (int)sizeof(C);
  __shared__ C lds[POWER && SUMS > EXCH ? SUMS : EXCH];
  __shared__ double red[S::THREADS / 64 + 1];

  if (a.batch) {                          // uniform per workgroup
    const RunPtrs r = a.batch[blockIdx.y];
    a.in = r.in; a.out = r.out; a.mult = r.mult; a.mult2 = r.mult2; a.nl_coef = r.nl_coef;
  }
  if constexpr (MODE == FWD && PRO == PRO_NONE) {
    if (!a.batch) {                       // fields that follow one another in memory
      const long skip = (long)blockIdx.y * a.npencils * S::N * (long)sizeof(C);
      a.in = (const char*)a.in + skip;
      a.out = (char*)a.out + skip;
    }
  }
  const int tid = threadIdx.x;
  int t, col;
  if constexpr (KIND == CONTIG) {
    // TL consecutive points of one pencil form a 128-byte segment; a wavefront
    // covers several pencils per load instruction (spreads requests over channels)
    constexpr int TL = lanes_per_pencil<S, (int)sizeof(C)>();
    t = tid % TL + TL * (tid / (TL * W));
    col = (tid / TL) % W;
  } else {
    col = tid % W;
    t = tid / W;
  }
  // XCD-aware tile order: workgroups are dispatched round-robin over the 8 XCDs;
  // give each XCD a contiguous run of tiles so tiles that share cache lines meet
  // in the same L2.
  const unsigned G = gridDim.x, b = blockIdx.x;
  const unsigned nfull = G / 8, rem = G % 8, xcd = b % 8;
  const long tile = (long)xcd * nfull + (xcd < rem ? xcd : rem) + b / 8;
  const long es = a.es;
  const long estep = (long)T * es * (long)sizeof(C);
  const auto tw = gptr<Tab<Real>>(a.tw);
  const auto mult = gptr<cplx<double>>(a.mult);     // FP64 multipliers for both precisions

  // Addressing: element e of this lane in tile tl sits at
  //   bbase + e*T*es   (uniform: first pencil of the tile, scalar registers)
  // + loff             (per lane, < 2^32 bytes for every supported shape)
  // so each access is a scalar-base + 32-bit-offset load or store.
  // A lane past the last pencil (ragged last tile) takes the last pencil: it loads,
  // transforms and stores exactly what that pencil's own lanes do, so every load and
  // store is issued unconditionally (no branch around memory instructions) and the
  // duplicate stores write equal bytes.
  struct Where { long bbase; unsigned loff; bool active; long pstart; };
  auto where = [&](long tl) {
    Where w;
    const long p = tl * W + col;
    w.active = p < a.npencils;
    const long pp = w.active ? p : a.npencils - 1;
    // pencil indices are below 2^20 for every supported shape: 32-bit division
    // (no 64-bit division subroutine with its branches)
    const unsigned inner = (unsigned)a.inner, q0 = (unsigned)(tl * W), q = (unsigned)pp;
    w.bbase = (long)(q0 / inner) * a.outer + (long)(q0 % inner);
    w.pstart = (long)(q / inner) * a.outer + (long)(q % inner);
    w.loff = (unsigned)(((long)(q / inner) * a.outer + (long)(q % inner) - w.bbase + (long)t * es) * (long)sizeof(C));
    return w;
  };
  auto load = [&](C* v, const Where& w, const void* from) {
    const auto inb = gptr<char>(from) + w.bbase * (long)sizeof(C);
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = *(const GPK_GLOBAL C*)(inb + e * estep + w.loff);
  };

  // the same addresses in lane order: register j + B r holds entry t + T j + r N/R_last
  auto lane_off = [&](int r, int j) { return (long)(T * j + r * (S::N / S::RL)) * es * (long)sizeof(C); };
  auto load_lane = [&](C* v, const void* from, const Where& w) {
    constexpr int L = S::NS - 1, B = E / S::rad(L);
    const auto inb = gptr<char>(from) + w.bbase * (long)sizeof(C);
#pragma unroll
    for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
      for (int j = 0; j < B; ++j) v[j + B * r] = *(const GPK_GLOBAL C*)(inb + lane_off(r, j) + w.loff);
  };
  auto store_lane = [&](const C* v, void* to, const Where& w) {
    constexpr int L = S::NS - 1, B = E / S::rad(L);
    const auto outb = gptr_mut<char>(to) + w.bbase * (long)sizeof(C);
#pragma unroll
    for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
      for (int j = 0; j < B; ++j) *(GPK_GLOBAL C*)(outb + lane_off(r, j) + w.loff) = v[j + B * r];
  };
  auto store = [&](const C* v, void* to, const Where& w) {
    const auto outb = gptr_mut<char>(to) + w.bbase * (long)sizeof(C);
#pragma unroll
    for (int e = 0; e < E; ++e) *(GPK_GLOBAL C*)(outb + e * estep + w.loff) = v[e];
  };

  // x pencils of complex64 propagator passes: whole tiles of contiguous pencils,
  // moved with 16-byte accesses (a pencil past the last one takes the last one, as
  // the lanes do, so the duplicate stores write equal bytes)
  constexpr bool WIDE = sizeof(Real) == 4 && KIND == CONTIG && (MODE == PROP || MODE == TURN) &&
                        (PRO == PRO_NONE || PRO == PRO_NL || PRO == PRO_SWAP || PRO == PRO_DERIV) && wide_io<S>();
  // first point of pencil pc of the tile, as it is read and as it is written
  auto swap_pencil = [&](int pc, bool written) {
    const unsigned n = (unsigned)a.ny, last = n * (n + 1) / 2 - 1;
    const unsigned u = (unsigned)tile * (W / 2) + (unsigned)pc / 2;
    unsigned i, j;
    pencil_pair(u < last ? u : last, n, i, j);
    return (long)((((pc & 1) != 0) != written) ? j * n + i : i * n + j) * S::N;
  };
  auto tile_pencil = [&](int pc) {
    if constexpr (PRO == PRO_SWAP) return swap_pencil(pc, false);
    const long p = tile * W + pc;
    return (p < a.npencils ? p : a.npencils - 1) * (long)S::N;
  };
  auto out_pencil = [&](int pc) {
    if constexpr (PRO == PRO_SWAP) return swap_pencil(pc, true);
    else return tile_pencil(pc);
  };

  // nonlinear sub-step (or its adjoint) on the points the lane holds
  auto rotate = [&](C* v, const Where& cur) {
    if constexpr (PRO == PRO_NL || PRO == PRO_TAPE) {
      rotate_points<E>(v, a.nl_coef);
    } else if constexpr (PRO == PRO_ADJ_NL) {
      // a few points at a time: the tape's points beside all of the lane's own do not fit
      // the registers
      constexpr int CH = E % 4 == 0 ? 4 : E % 3 == 0 ? 3 : E % 2 == 0 ? 2 : 1;
      const auto phib = gptr<char>(a.aux) + cur.bbase * (long)sizeof(C);
#pragma unroll
      for (int e0 = 0; e0 < E; e0 += CH) {
        C f[CH];
#pragma unroll
        for (int e = 0; e < CH; ++e) f[e] = *(const GPK_GLOBAL C*)(phib + (e0 + e) * estep + cur.loff);
        rotate_adjoint<CH>(v + e0, f, Real(a.nl_coef));
      }
    }
  };

  double kin_acc = 0.0;
  // transform one tile held in v (prologue, transform, multiplier, inverse) and store it
  auto process = [&](C* v, const Where& cur) {
    if constexpr (MODE == PROP || MODE == FWD) {
      if constexpr (PRO == PRO_NL || PRO == PRO_ADJ_NL) {
        rotate(v, cur);
      }
    }

    if constexpr (MODE == INV) {
      if constexpr (S::NS > 1) exchange<Real, S, KIND, -1, S::NS - 1>(lds, v, t, col);
      inverse_all<Real, S, KIND, S::NS - 1>(v, lds, t, col, tw);
      const Real sc = Real(a.scale);
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = cscale(v[e], sc);
    } else if constexpr (MODE == TURN) {
      constexpr int L = S::NS - 1, B = E / S::rad(L);
      auto substep = [&](const void* table) {
        const auto tw = gptr<Tab<Real>>(reload(a.tw));
        const auto m = gptr<cplx<double>>(table);
        forward_all<Real, S, KIND, 0>(v, lds, t, col, tw);
#pragma unroll
        for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
          for (int j = 0; j < B; ++j)
            v[j + B * r] = pmul(v[j + B * r], tab_at(m, r * (S::N / S::rad(L)) + t + T * j));
        inverse_all<Real, S, KIND, L>(v, lds, t, col, tw);
      };
      substep(a.mult);
      if constexpr (PRO == PRO_TAPE) {
        const auto tb = gptr_mut<char>(a.tape) + cur.bbase * (long)sizeof(C);
#pragma unroll
        for (int e = 0; e < E; ++e) *(GPK_GLOBAL C*)(tb + e * estep + cur.loff) = v[e];
      }
      rotate(v, cur);
      substep(a.mult2);
    } else {
      forward_all<Real, S, KIND, 0>(v, lds, t, col, tw);
      constexpr int L = S::NS - 1;
      constexpr int B = E / S::rad(L);
      if constexpr (MODE == PROP) {
        if constexpr (PRO == PRO_DERIV) {
          // i k/N F_j v; the energy sum_k k^2 |F_j v|^2 is N^2 times the sum of its squares,
          // plus the Nyquist coefficient, which the derivative leaves out
          constexpr int P = freq_pos<S>(S::N / 2), RL = S::RL, G = P / RL;
          // With 24 points a lane or more the squares are summed a point at a time before the
          // next table entry is taken (in_order): left to the scheduler, the sums fall behind
          // and the FP64 products of all points wait in registers (512 points complex64: 306
          // registers, one wavefront per SIMD, 1.22 ms a pass at 512^3 against 0.75).
          double acc = 0.0;
#pragma unroll
          for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
            for (int j = 0; j < B; ++j) {
              const double k = gptr<double>(a.mult)[(unsigned)(2 * (r * (S::N / S::rad(L)) + t + T * j) + 1)];
              const double x = v[j + B * r].x, y = v[j + B * r].y;
              if (S::N % 2 == 0 && r == P % RL && j == G / T && t == G % T) acc += 0.25 * (x * x + y * y);
              const double re = -y * k, im = x * k;
              acc = fma(re, re, fma(im, im, acc));
              v[j + B * r] = mk(Real(re), Real(im));
              if constexpr (E >= 24) in_order(acc, v[j + B * r]);
            }
          if (cur.active) kin_acc = acc * ((double)S::N * S::N);
        } else {
#pragma unroll
          for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
            for (int j = 0; j < B; ++j)
              v[j + B * r] = pmul(v[j + B * r], tab_at(mult, r * (S::N / S::rad(L)) + t + T * j));
        }
        inverse_all<Real, S, KIND, L>(v, lds, t, col, tw);
        if constexpr (PRO == PRO_ARGLE) {
          // v holds d phi / dz (this pass is the z derivative); replace it by the explicit
          // part of the imaginary-time step at the same points:
          //   n = -i v.grad phi + (beta - |v|^2/(4 alpha) - beta |phi|^2) phi
          const long ntot = a.npencils * (long)S::N;
          const auto vel = gptr<Real>(a.vel);
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const long idx = cur.bbase + (long)((e * estep + cur.loff) / (long)sizeof(C));
            const C f = gptr<C>(a.aux)[idx], gx = gptr<C>(a.aux2)[idx], gy = gptr<C>(a.aux3)[idx];
            const double ux = vel[idx], uy = vel[ntot + idx], uz = vel[2 * ntot + idx];
            const double gr = ux * gx.x + uy * gy.x + uz * v[e].x, gi = ux * gx.y + uy * gy.y + uz * v[e].y;
            const double pr = f.x, pi = f.y;
            const double c = a.nl_coef - (ux * ux + uy * uy + uz * uz) * a.q4a - a.nl_coef * (pr * pr + pi * pi);
            v[e] = mk(Real(gi + c * pr), Real(-gr + c * pi));
          }
          const auto tw2 = gptr<Tab<Real>>(reload(a.tw));
          forward_all<Real, S, KIND, 0>(v, lds, t, col, tw2);
          store_lane(v, a.out, cur);
          return;
        }
      } else {  // FWD: reorder to natural frequency order
        if constexpr (S::NS > 1) exchange<Real, S, KIND, L, -1>(lds, v, t, col);
        const Real sc = Real(a.scale);
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = cscale(v[e], sc);
        if constexpr (PRO == PRO_MULT3) {
          // v[e] holds frequency t + T e of the pencil starting at point cur.pstart;
          // the factors multiply in the order (m_x m_y) m_z, in FP64
          const auto mx = gptr<cplx<double>>(a.aux), my = gptr<cplx<double>>(a.aux2),
                     mz = gptr<cplx<double>>(a.aux3);
          const long nxy = (long)a.nx * a.ny;
          const int ix = (int)(cur.pstart % a.nx), iy = (int)((cur.pstart / a.nx) % a.ny),
                    iz = (int)(cur.pstart / nxy);
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const int f = t + T * e;
            const cplx<double> m = cmul(cmul(mx[a.axis == 0 ? f : ix], my[a.axis == 1 ? f : iy]),
                                        mz[a.axis == 2 ? f : iz]);
            v[e] = pmul(v[e], m);
          }
        }
      }
    }

    if constexpr (WIDE) {
      store_tile_wide<S>(v, lds, a.out, out_pencil, t, col);
    } else if constexpr (PRO == PRO_SWAP) {
      const auto dst = gptr_mut<C>(a.out) + out_pencil(col) + t;
#pragma unroll
      for (int e = 0; e < E; ++e) dst[T * e] = v[e];
    } else {
      store(v, a.out, cur);
    }
  };

  // fixed-order sum over the workgroup (wave butterfly, then waves in order), in thread 0
  auto block_sum = [&](double acc) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    __syncthreads();
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    double s = 0.0;
    if (tid == 0)
      for (int w = 0; w < S::THREADS / 64 + (S::THREADS % 64 ? 1 : 0); ++w) s += red[w];
    return s;
  };

  C v[E];
  const Where w = where(tile);
  if constexpr (PRO == PRO_HESS) {
    // Bound by registers and exchanges: three derivatives of the points a lane holds, their
    // products with the undifferentiated points summed here.  128^3 complex128: 6 derivative
    // passes and 6 passes that summed their products through memory took 268 us, these three
    // take 92 us (256 VGPRs at 16 points a lane, no scratch memory).
    constexpr int L = S::NS - 1, B = E / S::rad(L);
    Real J[E];
#pragma unroll
    for (int e = 0; e < E; ++e) J[e] = Real(0);
#pragma unroll 1
    for (int j = 0; j < 3; ++j) {
      const void* f = j == 0 ? a.in : j == 1 ? a.aux : a.aux2;
      load(v, w, f);
      const auto tw1 = gptr<Tab<Real>>(reload(a.tw));
      const void* table = reload(a.mult);
      forward_all<Real, S, KIND, 0>(v, lds, t, col, tw1);
#pragma unroll
      for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
        for (int i = 0; i < B; ++i) {
          const double k = gptr<double>(table)[(unsigned)(2 * (r * (S::N / S::rad(L)) + t + T * i) + 1)];
          const C x = v[i + B * r];
          v[i + B * r] = mk(Real(-(double)x.y * k), Real((double)x.x * k));
        }
      inverse_all<Real, S, KIND, L>(v, lds, t, col, tw1);
      const auto inb = gptr<char>(f) + w.bbase * (long)sizeof(C);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const C x = *(const GPK_GLOBAL C*)(inb + e * estep + w.loff);    // again, from the cache
        J[e] = Real((double)J[e] + ((double)x.x * (double)v[e].y - (double)x.y * (double)v[e].x));
      }
    }
    const auto outb = gptr_mut<char>(a.out) + w.bbase * (long)sizeof(Real);
#pragma unroll
    for (int e = 0; e < E; ++e) *(GPK_GLOBAL Real*)(outb + (e * estep + (long)w.loff) / 2) = J[e];
    return;
  }
  if constexpr (PRO == PRO_LANE && MODE == FWD) {
    load(v, w, a.in);
    forward_all<Real, S, KIND, 0>(v, lds, t, col, tw);
    store_lane(v, a.out, w);
    return;
  }
  if constexpr (PRO == PRO_LANE && MODE == INV) {
    load_lane(v, a.in, w);
    inverse_all<Real, S, KIND, S::NS - 1>(v, lds, t, col, tw);
    store(v, a.out, w);
    return;
  }
  if constexpr (PRO == PRO_LANE_D) {
    constexpr int L = S::NS - 1, B = E / S::rad(L);
    load_lane(v, a.in, w);
    inverse_all<Real, S, KIND, L>(v, lds, t, col, tw);
    store(v, a.out, w);
    // the coefficients again (from the cache), times i k: the derivative table holds k/N
    load_lane(v, reload(a.in), w);
#pragma unroll
    for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const double k = (double)S::N * gptr<double>(a.mult)[(unsigned)(2 * (r * (S::N / S::rad(L)) + t + T * j) + 1)];
        const C x = v[j + B * r];
        v[j + B * r] = mk(Real(-k * (double)x.y), Real(k * (double)x.x));
      }
    const auto tw2 = gptr<Tab<Real>>(reload(a.tw));
    inverse_all<Real, S, KIND, L>(v, lds, t, col, tw2);
    store(v, a.tape, w);
    return;
  }
  if constexpr (PRO == PRO_SOLVE) {
    // P <- ((1 - h k^2) P + dtau Q)/(1 + h k^2), h = dtau alpha / 2, Q the transform of the
    // explicit part, all in lane order (a y pass: pencil (z, x)); then P/N^3 back along y
    constexpr int L = S::NS - 1, B = E / S::rad(L);
    load(v, w, a.in);
    forward_all<Real, S, KIND, 0>(v, lds, t, col, tw);
    const unsigned nx = (unsigned)a.inner, p = (unsigned)(w.pstart / a.outer) * nx + (unsigned)(w.pstart % a.outer);
    const double kxz = gptr<double>(a.aux)[p % nx] + gptr<double>(a.aux2)[p / nx];
    const auto pb = gptr_mut<char>(a.tape) + w.bbase * (long)sizeof(C);
#pragma unroll
    for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const double hk = a.q4a * (kxz + gptr<double>(a.ksq)[(unsigned)(r * (S::N / S::rad(L)) + t + T * j)]);
        const double num = 1.0 - hk, den = 1.0 / (1.0 + hk);
        const auto at = (GPK_GLOBAL C*)(pb + lane_off(r, j) + w.loff);
        const C f = *at, q = v[j + B * r];
        const double re = (num * (double)f.x + a.nl_coef * (double)q.x) * den;
        const double im = (num * (double)f.y + a.nl_coef * (double)q.y) * den;
        *at = mk(Real(re), Real(im));
        v[j + B * r] = mk(Real(re * a.scale), Real(im * a.scale));
      }
    const auto tw2 = gptr<Tab<Real>>(reload(a.tw));
    inverse_all<Real, S, KIND, L>(v, lds, t, col, tw2);
    store(v, a.out, w);
    return;
  }
  if constexpr (POWER) {
    constexpr int L = S::NS - 1, B = E / S::rad(L), RL = S::RL;
    load(v, w, a.in);
    if constexpr (PRO == PRO_POWER) {
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = mk(cabs2(v[e]) - Real(1), Real(0));
    } else {
      forward_all<Real, S, KIND, 0>(v, lds, t, col, tw);
#pragma unroll
      for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
        for (int j = 0; j < B; ++j)
          v[j + B * r] = pmul(v[j + B * r], tab_at(mult, r * (S::N / S::rad(L)) + t + T * j));
      inverse_all<Real, S, KIND, L>(v, lds, t, col, tw);
      // the points again (from the cache: beside the derivatives they do not fit the registers)
      const auto inb = gptr<char>(reload(a.in)) + w.bbase * (long)sizeof(C);
      double v2 = 0.0;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const C p = *(const GPK_GLOBAL C*)(inb + e * estep + w.loff);
        const double pr = p.x, pi = p.y, rho = pr * pr + pi * pi;
        const double f = rho > 0.0 ? a.scale / rho : 0.0;
        const double vel = f * (pr * (double)v[e].y - pi * (double)v[e].x);
        v2 += vel * vel;
        v[e] = mk(Real(vel), Real(0));
      }
      const double s = block_sum(w.active ? v2 : 0.0);
      if (tid == 0) gptr_mut<double>(a.point_partial)[blockIdx.x] = s;
    }
    const auto tw2 = gptr<Tab<Real>>(reload(a.tw));
    forward_all<Real, S, KIND, 0>(v, lds, t, col, tw2);
    // |F f|^2 of every pencil to LDS, row = position, the columns of a row turned by the
    // position's group and, in the sums, by the frequency, so that lanes meet in no bank
    double* sums = reinterpret_cast<double*>(lds);
    __syncthreads();                        // the last exchange has been read
#pragma unroll
    for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const double x = v[j + B * r].x, y = v[j + B * r].y;
        const int g = t + T * j;
        sums[(g * RL + r) * W + (col + g) % W] = w.active ? x * x + y * y : 0.0;
      }
    __syncthreads();
    for (int k = tid; k < S::N; k += S::THREADS) {
      const double* row = sums + freq_pos<S>(k) * W;
      double s = 0.0;
      for (int c = 0; c < W; ++c) s += row[(c + k) % W];
      gptr_mut<double>(a.kin_partial)[(long)blockIdx.x * S::N + k] = s;
    }
    return;
  }
  if constexpr (PRO == PRO_ENERGY) {
    load(v, w, a.in);
    Neu rho_acc, int_acc;
    if (a.point_partial && w.active) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const double x = v[e].x, y = v[e].y, rho = x * x + y * y;
        rho_acc.add(rho);
        int_acc.add((rho - 1.0) * (rho - 1.0));
      }
    }
    forward_all<Real, S, KIND, 0>(v, lds, t, col, tw);
    constexpr int L = S::NS - 1, B = E / S::rad(L);
#pragma unroll
    for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const C x = v[j + B * r];
        kin_acc += gptr<double>(a.ksq)[(unsigned)(r * (S::N / S::rad(L)) + t + T * j)] *
                   ((double)x.x * x.x + (double)x.y * x.y);
      }
    if (!w.active) kin_acc = 0.0;
    const long at = (long)blockIdx.y * gridDim.x + blockIdx.x, all = (long)gridDim.y * gridDim.x;
    const double k = block_sum(kin_acc);
    if (tid == 0) gptr_mut<double>(a.kin_partial)[at] = k;
    if (a.point_partial) {
      const double r = block_sum(rho_acc.val()), q = block_sum(int_acc.val());
      if (tid == 0) { gptr_mut<double>(a.point_partial)[at] = r; gptr_mut<double>(a.point_partial)[all + at] = q; }
    }
    return;
  }
  if constexpr (WIDE) load_tile_wide<S>(v, lds, a.in, tile_pencil, t, col);
  else if constexpr (PRO == PRO_SWAP) {
    const auto src = gptr<C>(a.in) + tile_pencil(col) + t;
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = src[T * e];
  } else load(v, w, a.in);
  process(v, w);

  if constexpr (PRO == PRO_DERIV) {
    const double s = block_sum(kin_acc);
    if (tid == 0) gptr_mut<double>(a.kin_partial)[blockIdx.x] = s;
  }
}

// launcher signature shared by every instantiation
using PassLauncher = void (*)(const PassArgs&, unsigned grid, unsigned runs, hipStream_t stream);

template <class Real, class S, int KIND, int MODE, int PRO>
void launch_pass(const PassArgs& a, unsigned grid, unsigned runs, hipStream_t stream) {
  hipLaunchKernelGGL((axis_pass<Real, S, KIND, MODE, PRO>), dim3(grid, runs), dim3(S::THREADS), 0, stream, a);
}

// kernel variants compiled for every schedule
enum Variant { V_PROP = 0, V_PROP_NL, V_PROP_ADJ, V_DERIV, V_FWD, V_INV, V_PROP_ARGLE, V_FWD_MULT3,
               V_TURN, V_TURN_TAPE, V_TURN_ADJ, V_PROP_SWAP, V_ENERGY, V_POWER, V_VPOWER,
               V_FWD_LANE, V_INV_LANE, V_INV_LANE_D, V_SOLVE, V_HESS, V_COUNT };

}  // namespace gpk
