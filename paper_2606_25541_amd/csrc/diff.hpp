// Differential PSFD operator with a z-PML (the comparison solver of the
// preconditioner study) and its background-field and full-domain solves.
#pragma once
#include "engine.hpp"

struct psfd_diff_plan;

namespace psfd {

Status diff_create(const psfd_diff_problem& p, psfd_diff_plan*& out);
void diff_destroy(psfd_diff_plan* p);
// y = A x (precond PSFD_PRECOND_NONE) or D A x (PSFD_PRECOND_DAMPING); deps: the
// contrast planes [ncz][ny][nx], x, y: [3][nz_ext][ny][nx], all of dtype
Status diff_apply(psfd_diff_plan* p, const void* deps, const void* x, void* y, int dtype, int precond, hipStream_t s);
Status diff_solve(psfd_diff_plan* p, const void* deps, void* e, void* orders, const psfd_opts* opts, int precond,
                  psfd_info* info, hipStream_t s);

// ---- kernels with compile-time shapes (k_diffz.hip) --------------------------
// Transverse FFT of planes: in, out [planes][ny][nx]. Forward: planes 0 .. 3 pe - 1,
// and, launched with 3 ncz planes more, the spectra of V x (V = k0sq deps) of the
// contrast planes into `aux`, [3][ncz][ny][nx]. Inverse with deps: out
// = IFFT in - V x on the contrast planes.
struct DiffPlaneArgs {
  const void* in;
  void* out;
  const void* deps;  // [ncz][ny][nx], or null
  void* aux;         // forward: receives the spectra of V x; inverse: x, the operand of V x (read)
  int pe, zc0, ncz;
  double k0sq;
  const void* tw;    // twiddles of every length (length n at offset n)
};
// curl curl - k_bg^2 of the field w [3][pe][ny][nx] in the transverse spectrum, in
// place, times 1 / (Nx Ny); damp: minus the spectrum vx [3][ncz][ny][nx] of V x on
// the contrast planes, and times the spectral damping.
struct DiffZcolArgs {
  int nx, ny;
  void* w;
  const void* vx;
  int zc0, ncz;
  const double *kx, *ky, *zt;  // zt: kappa_d [pe], kappa [pe], 1 / s(z) [pe] (complex)
  double kbg2;
  const void* tw;
};
template <class T> bool diff_ct_shape(int nx, int ny, int pe);
template <class T, bool INV>
bool launch_diff_plane(const DiffPlaneArgs& a, int nx, int ny, int nplanes, hipStream_t s);
template <class T>
bool launch_diff_zcol(const DiffZcolArgs& a, int pe, bool damp, hipStream_t s);

}  // namespace psfd
