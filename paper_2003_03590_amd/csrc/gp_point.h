// Launch wrappers of the pointwise and reduction kernels (gp_point.hip).
#pragma once

#include "gp_registry.h"

namespace gpk {

void launch_init_phase(int prec, const double* theta, void* psi, long n, hipStream_t st);
void launch_nonlinear(int prec, void* psi, long n, double coef, hipStream_t st);
void launch_scale_copy(int prec, const void* in, void* out, long n, double scale, hipStream_t st);
void launch_mult3(int prec, void* f, int nx, int ny, int nz, const void* mx, const void* my, const void* mz,
                  hipStream_t st);
void launch_diag_fields(int prec, const void* psi, void* f0, void* f1, void* f2, void* f3, long n, double alpha,
                        double* partial, unsigned blocks, hipStream_t st);
void launch_spectral(int prec, const void* F0, const void* F1, const void* F2, const void* F3, int nx, int ny, int nz,
                     double alpha, double beta, int nshell, unsigned blocks, double* bins, hipStream_t st);
// out[0] = max over the field of |a - b|^2 (partial: blocks doubles)
void launch_sup_diff2(int prec, const void* a, const void* b, long n, double* partial, unsigned blocks, double* out,
                      hipStream_t st);
// psum, pmax: `blocks` doubles each (sum and max of |w|^2 per block)
void launch_mach_partials(int prec, const void* psi, const void* d0, const void* d1, const void* d2, long n,
                          double alpha, double* psum, double* pmax, unsigned blocks, hipStream_t st);
void launch_segmax(const double* in, long len, double* out, hipStream_t st);
// every point of f <- re + i im
void launch_fill(int prec, void* f, long n, double re, double im, hipStream_t st);
void launch_copy16(const void* src, void* dst, long bytes, hipStream_t st);   // bytes: a multiple of 8
// helicity stages (see the kernels for the packing of real fields into states)
// partial: blocks doubles (sum |grad psi|^2)
void launch_hel_pack(int prec, const void* psi, const void* d0, const void* d1, const void* d2, void* s3, void* s4,
                     void* s5, long n, double alpha, double* partial, unsigned blocks, hipStream_t st);
void launch_hel_omega(int prec, const void* t3, const void* t4, const void* t5, void* s6, void* s7, long n,
                      hipStream_t st);
// Jx, Jy, Jz: real fields; s0 .. s3: the packed v and v_reg for the spectra (null: none wanted);
// g2_sum: device, one double (sum |grad psi|^2); partial: 2 * blocks doubles
void launch_hel_vreg(int prec, const void* psi, const void* d0, const void* d1, const void* d2, const void* Jx,
                     const void* Jy, const void* Jz, const void* w01, const void* w2, void* s0, void* s1, void* s2,
                     void* s3, long n, double alpha, const double* g2_sum, double* partial, unsigned blocks,
                     hipStream_t st);
// bins: blocks * 2 * nshell doubles
void launch_hel_spectral(int prec, const void* V01, const void* V2, const void* R01, const void* R2, const void* O01,
                         const void* O2, int nx, int ny, int nz, int nshell, unsigned blocks, double* bins, hipStream_t st);
// out[3][nj/2] per-axis structure functions from pk[3][nj]
void launch_structure_axes(const double* pk, int nj, double ntot, double* out, hipStream_t st);
void launch_segsum(const double* in, long len, int nseg, double* out, hipStream_t st);
// segment sums of several quantities: quantity q holds, for each of m runs, len[q] numbers
// from in + first[q] on; out[q][run] (len 0: the sum is 0)
struct SegLens { long first[5], len[5]; };
void launch_segsums(const double* in, const SegLens& s, unsigned m, double* out, hipStream_t st);
// out[chunk][cols]: sums of the columns of in[rows][cols] over `chunks` runs of rows
unsigned colsum_chunks(long rows);                      // 1 .. 16
void launch_colsum(const double* in, long rows, int cols, unsigned chunks, double* out, hipStream_t st);
// the reductions of the diagnostics in one launch: red[0..4] = the five segment sums of one run,
// red[5] = a sixth over in6[0 .. len6), red[6 ..] = column sums of bins[rows][cols] by chunks
void launch_diag_reduce(const double* in, const SegLens& s, const double* in6, long len6, const double* bins, long rows,
                        int cols, unsigned chunks, double* red, hipStream_t st);
// energies and spectra from red (bin sums still by chunks); out may be pinned host memory
void launch_finalize_diag(const double* red, unsigned chunks, double w0, double w1, double w2, int nshell, double alpha,
                          double beta, double ntot, double* out, hipStream_t st);
void launch_loss_fields(int prec, const void* psi, const void* d0, const void* d1, const void* d2, void* f0,
                        void* f1, long n, double alpha, hipStream_t st);
void launch_loss_spectral(int prec, void* F0, void* F1, int nx, int ny, int nz, int smin, int smax,
                          double* partial, unsigned blocks, hipStream_t st);
void launch_loss_lambda1(int prec, const void* psi, void* d0, void* d1, void* d2, const void* G0, const void* G1,
                         void* lam, long n, double alpha, hipStream_t st);
void launch_loss_lambda2(int prec, void* lam, const void* e0, const void* e1, const void* e2, long n,
                         hipStream_t st);
void launch_phase_grad(int prec, const void* psi0, const void* lam0, double* out, long n, hipStream_t st);
void launch_argle_explicit(int prec, const void* phi, const void* dx, const void* dy, const void* dz, const void* v,
                           void* out, long n, double alpha, double beta, hipStream_t st);
void launch_argle_solve(int prec, void* P, const void* Q, int nx, int ny, int nz, double a, double dtau, double inv_n,
                        hipStream_t st);
void launch_argle_energy(int prec, const void* phi, const void* dx, const void* dy, const void* dz, const void* v,
                         long n, double alpha, double beta, double* partial, unsigned blocks, hipStream_t st);
// table: npairs * 3 * max(nx, ny, nz) doubles of scratch memory; far: core width, a radius or a
// separation above kFarRing
constexpr double kFarRing = 100.0;
void launch_init_rvr(int prec, const void* pairs, void* table, int npairs, double xi, double a1, double a2, double b1,
                     bool far, int nx, int ny, int nz, void* psi, hipStream_t st);
size_t ringpar_bytes();
void launch_structure_final(const double* pk, int nj, double ntot, double* out, hipStream_t st);

}  // namespace gpk
