// xy-plane pass: the two in-plane sub-steps S(s, L_x) S(s, L_y) of the split step
// (time-evolution section; the axes commute, so the x and y factors may be applied
// together) on one z-plane per workgroup, reading and writing psi once.
//
// The plane (N x N points, N <= 128 for complex64, <= 64 for complex128) is small
// enough to stay on chip: the rows are loaded from global memory and transformed
// with the row (contiguous) mapping of the axis pass, written to LDS in natural
// order, read back as columns and transformed with the column (strided) mapping,
// then stored.  The transform stages, tables and the nonlinear prologue are those of
// the axis pass (same schedule type, W = N).
//
// TURN: the plane's sub-steps end one time step and begin the next (gp_pass.h), rows,
// columns, nonlinear rotation, columns, rows in one launch.  With the z pass turning
// as well, a step is one sweep of psi and one launch.
#pragma once

#include "gp_pass.h"

namespace gpk {

struct PlaneArgs {
  const RunPtrs* batch;    // grouped launch over runs of one size, or null
  const void* in;
  void* out;
  const void* mult;        // FP64 complex multipliers in the plane schedule's lane order (x and
                           // y share them: one length, one alpha)
  const void* mult2;       // TURN: multipliers of the second time step
  const void* tw;          // per-stage twiddles of the plane schedule (Tab<Real>)
  double nl_coef;          // beta * dt for the fused nonlinear rotation
};

constexpr int cmax(int a, int b) { return a > b ? a : b; }

template <class Real, class S, int MODE, int PRO>
__global__ __launch_bounds__(S::THREADS) void plane_pass(PlaneArgs a) {
  static_assert(S::W == S::N && S::NS > 1, "a plane workgroup holds all N rows; the stage exchanges order its LDS use");
  using C = cplx<Real>;
  constexpr int N = S::N, T = S::T, E = S::E;
  // plane row pitch in LDS: rows that share an LDS cycle in the row-major write get
  // their own banks (the column reads take consecutive points of one row)
  constexpr int SZ = (int)sizeof(C), TL = lanes_per_pencil<S, SZ>();
  constexpr int P = (TL < 128 / SZ) ? row_pitch<SZ>(N, TL) : N + 1;
  constexpr int L = S::NS - 1, B = E / S::rad(L);
  constexpr int EX = Lds<S, (int)sizeof(C), CONTIG>::ELEMS, EY = Lds<S, (int)sizeof(C), STRIDED>::ELEMS;
  // one buffer serves the row exchanges, the plane and the column exchanges in turn
  __shared__ C lds[cmax(cmax(EX, EY), N * P)];

  if (a.batch) {                          // uniform per workgroup
    const RunPtrs r = a.batch[blockIdx.y];
    a.in = r.in; a.out = r.out; a.mult = r.mult; a.mult2 = r.mult2; a.nl_coef = r.nl_coef;
  }
  const int tid = threadIdx.x;
  const long base = (long)blockIdx.x * N * N;   // first point of this z-plane
  // lane (tr, row) of the row mapping, lane (tc, col) of the column mapping
  const int tr = tid % TL + TL * (tid / (TL * N)), row = (tid / TL) % N;
  const int tc = tid / N, col = tid % N;
  C v[E];

  auto rotate = [&] { rotate_points<E>(v, a.nl_coef); };
  auto multiply = [&](const void* table, int t) {
    const auto m = gptr<cplx<double>>(table);
#pragma unroll
    for (int r = 0; r < S::rad(L); ++r)
#pragma unroll
      for (int j = 0; j < B; ++j) v[j + B * r] = pmul(v[j + B * r], m[(unsigned)(r * (N / S::rad(L)) + t + T * j)]);
  };
  auto rows = [&](const void* table) {    // S(s, L_x)
    const auto tw = gptr<Tab<Real>>(reload(a.tw));
    forward_all<Real, S, CONTIG, 0>(v, lds, tr, row, tw);
    multiply(table, tr);
    inverse_all<Real, S, CONTIG, L>(v, lds, tr, row, tw);
  };
  auto columns = [&](const void* table) { // S(s, L_y)
    const auto tw = gptr<Tab<Real>>(reload(a.tw));
    // the first exchange starts with a barrier: every read of the plane is done by then
    forward_all<Real, S, STRIDED, 0>(v, lds, tc, col, tw);
    multiply(table, tc);
    inverse_all<Real, S, STRIDED, L>(v, lds, tc, col, tw);
  };

  const auto src = gptr<C>(a.in) + base + (long)row * N + tr;
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = src[T * e];
  if constexpr (MODE == PROP && PRO == PRO_NL) rotate();
  rows(a.mult);
  __syncthreads();                         // the last row exchange has been read
#pragma unroll
  for (int e = 0; e < E; ++e) lds[row * P + tr + T * e] = v[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = lds[(tc + T * e) * P + col];
  if constexpr (MODE == PROP) {
    columns(a.mult);
    const auto dst = gptr_mut<C>(a.out) + base + col;
#pragma unroll
    for (int e = 0; e < E; ++e) dst[(long)(tc + T * e) * N] = v[e];
  } else {
    columns(a.mult);
    rotate();
    columns(a.mult2);
    __syncthreads();                       // the last column exchange has been read
#pragma unroll
    for (int e = 0; e < E; ++e) lds[(tc + T * e) * P + col] = v[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = lds[row * P + tr + T * e];
    rows(a.mult2);
    const auto dst = gptr_mut<C>(a.out) + base + (long)row * N + tr;
#pragma unroll
    for (int e = 0; e < E; ++e) dst[T * e] = v[e];
  }
}

using PlaneLauncher = void (*)(const PlaneArgs&, unsigned planes, unsigned runs, hipStream_t stream);

template <class Real, class S, int MODE, int PRO>
void launch_plane(const PlaneArgs& a, unsigned planes, unsigned runs, hipStream_t stream) {
  hipLaunchKernelGGL((plane_pass<Real, S, MODE, PRO>), dim3(planes, runs), dim3(S::THREADS), 0, stream, a);
}

}  // namespace gpk
