// Host-driven restarted GMRES (Saad & Schultz): classical Gram-Schmidt with the
// projections and ||w||^2 from one launch and the new norm by Pythagoras (a
// second pass where the update leaves less than `cancel` of the norm, its norm by
// Pythagoras from its own projections too), Givens rotations and the small
// triangular solve on the host. Reductions run in a fixed order (block partials,
// then one wavefront per sum), so a solve is deterministic.
//
// The norm by difference is off by eps / (2 c^2), c what a pass leaves of the norm.
// One pass is trusted for c >= `cancel`. After a second pass c is near 1 again
// unless w lies in the span of the basis to rounding (twice is enough: Giraud,
// Langou, Rozloznik, van den Eshof 2005), and then hn is rounding noise of the
// first pass or 0 however it is formed: the rotation takes |g_(j+1)| below any
// tolerance, the cycle ends, and the restart's residual b - A x decides.
//
// A step runs on the device alone: the step kernel sums the partials, forms the
// norm and scale the update takes, and writes them to mapped host memory; the
// launches of a second pass test its flag and return at once where it is not
// needed. The host issues the next step's apply before it waits for a step's
// scalars, so that the device never waits for the host's rotations; that apply is
// dropped where the step ends the cycle. On a 32 x 32 x 16 isolated FP64 solve a step
// took about 165 us of which its kernels were 45 (copies down and up, two waits and
// their wake-ups); with the three launches of k_gm_pass it takes about 40,
// 2.6 -> 0.79 ms the solve.
#include "gmres_host.hpp"

#include <algorithm>
#include <cmath>
#include <complex>
#include <type_traits>
#include <vector>

namespace psfd {

namespace {

constexpr int KB = 256;      // threads per block
constexpr double ETA_MIXED = 1e-4;
// Vectors up to this length (4 values per thread of GM_BLOCKS blocks) take a
// Gram-Schmidt pass in one launch (k_gm_pass); beyond, 256 blocks are too few
// for the memory and the separate kernels' blocks are as many as the vector needs
// (a step at 98304 values 67.2 -> 63.6 us, at 196608 98.6 -> 97.4, at 786432 207 -> 208).
constexpr long long GM_SHORT = 4LL * GM_BLOCKS * KB;

#define GMCHK(call)                                    \
  do {                                                 \
    hipError_t e_ = (call);                            \
    if (e_ != hipSuccess) return hip_status(e_, #call); \
  } while (0)

Status bad(int code, const char* m) {
  Status s;
  s.code = code;
  s.msg = m;
  return s;
}

// part[i * GM_BLOCKS + blk] = sum over the block's chunk of conj(V_i) w, i < nv
// (FP64 accumulation); a block takes four vectors, which share its reads of w.
// second: only where the step kernel asked for a second pass
template <class T>
__global__ void __launch_bounds__(KB) k_gm_dots(const T* __restrict__ V, long long stride, int nv,
                                                const T* __restrict__ w, long long n, double2* __restrict__ part,
                                                const GmScalars* __restrict__ sc, bool second) {
  __shared__ double2 red[4][KB / 64];
  if (second && !sc->cancel) return;
  const int i0 = blockIdx.y * 4, tid = threadIdx.x;
  const T* v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = V + min(i0 + q, nv - 1) * stride;
  double2 acc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = make_double2(0.0, 0.0);
  for (long long e = (long long)blockIdx.x * KB + tid; e < n; e += (long long)GM_BLOCKS * KB) {
    const double2 c = to_d(w[e]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double2 a = to_d(v[q][e]);
      acc[q].x += a.x * c.x + a.y * c.y;
      acc[q].y += a.x * c.y - a.y * c.x;
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    acc[q] = make_double2(lane_sum(acc[q].x), lane_sum(acc[q].y));
    if ((tid & 63) == 0) red[q][tid >> 6] = acc[q];
  }
  __syncthreads();
  if (tid < 4 && i0 + tid < nv) {
    double2 t = red[tid][0];
#pragma unroll
    for (int k = 1; k < KB / 64; ++k) t = cadd(t, red[tid][k]);
    part[(long long)(i0 + tid) * GM_BLOCKS + blockIdx.x] = t;
  }
}

// The nv sums of the partials into h (LDS), one wavefront each in a fixed order;
// every thread of the block of NT calls it, a barrier follows.
template <int NT> PSFD_D void gm_sums(const double2* __restrict__ part, int nv, double2* h) {
  const int lane = threadIdx.x & 63;
#pragma unroll 2
  for (int i = threadIdx.x >> 6; i < nv; i += NT / 64) {
    double2 p[GM_BLOCKS / 64];
#pragma unroll
    for (int k = 0; k < GM_BLOCKS / 64; ++k) p[k] = part[(long long)i * GM_BLOCKS + lane + 64 * k];
    double2 t = p[0];
#pragma unroll
    for (int k = 1; k < GM_BLOCKS / 64; ++k) t = cadd(t, p[k]);
    t = make_double2(lane_sum(t.x), lane_sum(t.y));
    if (lane == 0) h[i] = t;
  }
}

// ||w||^2 before a pass is h[nv - 1], the projections are the others: the norm
// after it by Pythagoras
PSFD_D double gm_norm(const double2* h, int nv) {
  const double w2 = h[nv - 1].x;
  double p2 = 0.0;
  for (int i = 0; i < nv - 1; ++i) p2 += h[i].x * h[i].x + h[i].y * h[i].y;
  const double d2 = w2 - p2;
  return d2 == d2 ? sqrt(fmax(d2, 0.0)) : d2;  // (fmax would drop a NaN)
}
PSFD_D double gm_inv(double hn) { return hn > 0.0 ? 1.0 / hn : 1.0; }
PSFD_D bool gm_cancel(double hn, double w2, double cancel) { return !(hn >= cancel * sqrt(fmax(w2, 0.0))); }

// What a pass leaves in GmScalars; what the host reads also goes to mapped host
// memory. NT threads of one block.
template <int NT>
PSFD_D void gm_publish(const double2* h, int nv, double hn, double cancel, GmScalars* dev, GmScalars* host,
                       bool second) {
  for (int i = threadIdx.x; i < nv; i += NT) {
    if (second) {
      dev->h2[i] = h[i];
      host->h[i] = cadd(dev->h[i], h[i]);
    } else {
      dev->h[i] = host->h[i] = h[i];
    }
  }
  if (threadIdx.x == 0) {
    dev->hn = host->hn = hn;
    dev->inv = gm_inv(hn);
    if (!second) {
      const double w2 = h[nv - 1].x;
      dev->w2 = host->w2 = w2;
      dev->cancel = gm_cancel(hn, w2, cancel);
    }
  }
}

// One block: the sums of the partials, then hn, inv and (first pass) cancel as in
// GmScalars.
__global__ void __launch_bounds__(1024) k_gm_step(const double2* __restrict__ part, int nv, double cancel,
                                                  GmScalars* dev, GmScalars* host, bool second) {
  __shared__ double2 h[GM_MAX + 2];
  if (second && !dev->cancel) return;
  gm_sums<1024>(part, nv, h);
  __syncthreads();
  const double hn = threadIdx.x == 0 ? gm_norm(h, nv) : 0.0;
  gm_publish<1024>(h, nv, hn, cancel, dev, host, second);
}

// A Gram-Schmidt pass of a short vector in one launch of GM_BLOCKS blocks: every
// block sums the projection partials itself (part; nv vectors and ||w||^2), updates
// its elements of w, and in the first pass, where a second one follows, forms that
// one's partials (part2) from the elements it has just written. With k_gm_dots in
// front a step then takes three launches beside the apply where dots, step and
// update of both passes take six, each 3 to 6 us of latency on the timeline
// whatever its work: a 32 x 32 x 16 FP64 isolated solve 914 -> 787 us,
// 64 x 64 x 16 mixed 71 -> 68 us a step. Element
// and partial order are those of the separate kernels.
template <class T, bool SECOND>
__global__ void __launch_bounds__(KB) k_gm_pass(T* __restrict__ w, const T* __restrict__ V, long long stride, int nv,
                                                long long n, const double2* __restrict__ part,
                                                double2* __restrict__ part2, double cancel, GmScalars* dev,
                                                GmScalars* host) {
  __shared__ double2 h[GM_MAX + 2], red[4][KB / 64];
  __shared__ double hns;
  if (SECOND && !dev->cancel) return;
  const int tid = threadIdx.x;
  const long long e0 = (long long)blockIdx.x * KB + tid, step = (long long)GM_BLOCKS * KB;
  gm_sums<KB>(part, nv + 1, h);
  __syncthreads();
  if (tid == 0) hns = gm_norm(h, nv + 1);
  __syncthreads();
  const double hn = hns;
  const bool more = !SECOND && gm_cancel(hn, h[nv].x, cancel);
  const double inv = more ? 1.0 : gm_inv(hn);
  if (blockIdx.x == 0) gm_publish<KB>(h, nv + 1, hn, cancel, dev, host, SECOND);
  for (long long e = e0; e < n; e += step) {
    double2 acc = to_d(w[e]);
#pragma unroll 4
    for (int i = 0; i < nv; ++i) {
      const double2 c = h[i], v = to_d(V[i * stride + e]);
      acc.x -= c.x * v.x - c.y * v.y;
      acc.y -= c.x * v.y + c.y * v.x;
    }
    w[e] = from_d<T>(cscale(acc, inv));
  }
  if (!more) return;
  for (int i0 = 0; i0 <= nv; i0 += 4) {
    const T* v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = i0 + q < nv ? V + (i0 + q) * stride : w;
    double2 acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = make_double2(0.0, 0.0);
    for (long long e = e0; e < n; e += step) {
      const double2 c = to_d(w[e]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double2 a = to_d(v[q][e]);
        acc[q].x += a.x * c.x + a.y * c.y;
        acc[q].y += a.x * c.y - a.y * c.x;
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      acc[q] = make_double2(lane_sum(acc[q].x), lane_sum(acc[q].y));
      if ((tid & 63) == 0) red[q][tid >> 6] = acc[q];
    }
    __syncthreads();
    if (tid < 4 && i0 + tid <= nv) {
      double2 t = red[tid][0];
#pragma unroll
      for (int k = 1; k < KB / 64; ++k) t = cadd(t, red[tid][k]);
      part2[(long long)(i0 + tid) * GM_BLOCKS + blockIdx.x] = t;
    }
    __syncthreads();
  }
}

// w = (w - sum_{i < nv} h_i V_i) inv (in FP64, stored in w's type), h and inv from
// the step kernel. The first pass leaves the scale to the second where one follows.
template <class T, bool SECOND>
__global__ void __launch_bounds__(KB) k_gm_update(T* __restrict__ w, const T* __restrict__ V, long long stride,
                                                  const GmScalars* __restrict__ sc, int nv, long long n) {
  const bool cancel = sc->cancel != 0;
  if (SECOND && !cancel) return;
  const long long e = (long long)blockIdx.x * KB + threadIdx.x;
  if (e >= n) return;
  double2 acc = to_d(w[e]);
#pragma unroll 4
  for (int i = 0; i < nv; ++i) {
    const double2 c = SECOND ? sc->h2[i] : sc->h[i], v = to_d(V[i * stride + e]);
    acc.x -= c.x * v.x - c.y * v.y;
    acc.y -= c.x * v.y + c.y * v.x;
  }
  w[e] = from_d<T>(cscale(acc, !SECOND && cancel ? 1.0 : sc->inv));
}

// x += sum_{i < nv} coef_i V_i
struct GmCoefs { double2 c[GM_MAX]; };
template <class T>
__global__ void __launch_bounds__(KB) k_gm_axpys(double2* __restrict__ x, const T* __restrict__ V, long long stride,
                                                 GmCoefs coef, int nv, long long n) {
  const long long e = (long long)blockIdx.x * KB + threadIdx.x;
  if (e >= n) return;
  double2 acc = x[e];
#pragma unroll 4
  for (int i = 0; i < nv; ++i) {
    const double2 c = coef.c[i], v = to_d(V[i * stride + e]);
    acc.x += c.x * v.x - c.y * v.y;
    acc.y += c.x * v.y + c.y * v.x;
  }
  x[e] = acc;
}

// r = b - ax and the partials of ||r||^2 (ax null: r = b)
__global__ void __launch_bounds__(KB) k_gm_resid(const double2* __restrict__ b, const double2* __restrict__ ax,
                                                 double2* __restrict__ r, long long n, double2* __restrict__ part) {
  __shared__ double red[KB / 64];
  const int tid = threadIdx.x;
  double acc = 0.0;
  for (long long e = (long long)blockIdx.x * KB + tid; e < n; e += (long long)GM_BLOCKS * KB) {
    const double2 v = ax ? csub(b[e], ax[e]) : b[e];
    r[e] = v;
    acc += cabs2(v);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double t = red[0];
#pragma unroll
    for (int k = 1; k < KB / 64; ++k) t += red[k];
    part[blockIdx.x] = make_double2(t, 0.0);
  }
}

// out = a inv in out's type, inv from the step kernel
template <class TO>
__global__ void __launch_bounds__(KB) k_gm_scale(const double2* __restrict__ a, const GmScalars* __restrict__ dev,
                                                 TO* __restrict__ out, long long n) {
  const long long e = (long long)blockIdx.x * KB + threadIdx.x;
  if (e < n) out[e] = from_d<TO>(cscale(a[e], dev->inv));
}

template <class T>
Status gmres_t(long long n, const ApplyFn& A, const double2* B, double2* X, const HostGmres& o, psfd_info& inf,
               GmresWs& ws, hipStream_t s) {
  typedef std::complex<double> cd;
  const bool f32 = sizeof(T) == 8;
  const int m = o.m;
  // basis, A x and residual in one allocation
  void* mem = nullptr;
  struct Free {
    void*& q;
    ~Free() { if (q) (void)hipFree(q); }
  } fr{mem};
  const size_t vbytes = ((size_t)(m + 1) * n * sizeof(T) + 255) / 256 * 256;
  GMCHK(hipMalloc(&mem, vbytes + 2 * (size_t)n * sizeof(double2)));
  T* V = (T*)mem;
  double2* w64 = (double2*)((char*)mem + vbytes);
  double2* r64 = w64 + n;
  const unsigned g1 = (unsigned)((n + KB - 1) / KB);
  const int dt = f32 ? PSFD_C64 : PSFD_C128;
  const volatile GmScalars* hs = ws.host;
  // the sums V_i^H w, i < nv (the last: w itself), what the step kernel makes of
  // them, and the scalars' event
  double2* part2 = ws.part + GM_BLOCKS * (GM_MAX + 2);
  auto proj = [&](int nv, const T* w, bool second) {
    hipLaunchKernelGGL(k_gm_dots<T>, dim3(GM_BLOCKS, (nv + 3) / 4), dim3(KB), 0, s, (const T*)V, n, nv, w, n, ws.part,
                       (const GmScalars*)ws.dev, second);
  };
  auto dots = [&](int nv, const T* w, bool second) {
    proj(nv, w, second);
    hipLaunchKernelGGL(k_gm_step, dim3(1), dim3(1024), 0, s, ws.part, nv, o.cancel, ws.dev, ws.dhost, second);
  };
  // ev marks the scalars of the launches so far
  auto mark = [&]() -> Status {
    GMCHK(hipGetLastError());
    GMCHK(hipEventRecord(ws.ev, s));
    return Status();
  };
  auto wait = [&]() -> Status {
    GMCHK(hipEventSynchronize(ws.ev));
    return Status();
  };
  // r64 = b - ax, its norm, and v_0 = r64 / ||r64|| issued behind it
  auto residual = [&](const double2* ax, double& beta) -> Status {
    Status st;
    hipLaunchKernelGGL(k_gm_resid, dim3(GM_BLOCKS), dim3(KB), 0, s, B, ax, r64, n, ws.part);
    hipLaunchKernelGGL(k_gm_step, dim3(1), dim3(1024), 0, s, ws.part, 1, 0.0, ws.dev, ws.dhost, false);
    if (!(st = mark()).ok()) return st;
    hipLaunchKernelGGL(k_gm_scale<T>, dim3(g1), dim3(KB), 0, s, (const double2*)r64, (const GmScalars*)ws.dev, V, n);
    if (!(st = wait()).ok()) return st;
    beta = std::sqrt(std::max((double)hs->w2, 0.0));
    if (!std::isfinite((double)hs->w2)) beta = hs->w2;
    return Status();
  };
  Status st;
  double bnorm = 0.0;
  if (!(st = residual(nullptr, bnorm)).ok()) return st;
  if (!std::isfinite(bnorm)) return bad(PSFD_ERR_NONFINITE, "right-hand side is not finite");
  if (bnorm == 0.0) {
    GMCHK(hipMemsetAsync(X, 0, n * sizeof(double2), s));
    GMCHK(hipStreamSynchronize(s));
    inf.status = PSFD_OK;
    inf.rel_residual = 0.0;
    return Status();
  }
  double beta = bnorm, rel = 1.0;
  if (o.warm) {
    // r = b - A x0
    if (!(st = A(X, w64, PSFD_C128, s)).ok()) return st;
    if (!(st = residual(w64, beta)).ok()) return st;
    rel = beta / bnorm;
    if (!std::isfinite(rel)) return bad(PSFD_ERR_NONFINITE, "non-finite residual");
    inf.rel_residual = rel;
    if (rel <= o.rtol) {
      inf.status = PSFD_OK;
      GMCHK(hipStreamSynchronize(s));
      return Status();
    }
  } else {
    GMCHK(hipMemsetAsync(X, 0, n * sizeof(double2), s));
  }
  std::vector<cd> H((size_t)(m + 1) * m), g(m + 1), sn(m), y(m);
  std::vector<double> cs(m);
  auto Hij = [&](int i, int j) -> cd& { return H[(size_t)i * m + j]; };
  while (inf.iters < o.max_iters) {
    ++inf.cycles;
    std::fill(H.begin(), H.end(), cd(0.0));
    std::fill(g.begin(), g.end(), cd(0.0));
    g[0] = beta;
    const double stop = std::max(o.rtol * bnorm, f32 ? ETA_MIXED * beta : 0.0);
    int k = 0;
    bool ahead = false;  // A v_j has been issued
    for (int j = 0; j < m && inf.iters < o.max_iters; ++j) {
      // w = A v_j straight into slot j + 1; one launch gives V_{0..j}^H w and
      // ||w||^2; the norm after the update follows from Pythagoras, and a
      // cancellation (norm ratio below cancel) takes a second pass
      T* wj = V + (j + 1) * n;
      if (!ahead && !(st = A(V + j * n, wj, dt, s)).ok()) return st;
      if (n <= GM_SHORT) {
        proj(j + 2, wj, false);
        hipLaunchKernelGGL((k_gm_pass<T, false>), dim3(GM_BLOCKS), dim3(KB), 0, s, wj, (const T*)V, n, j + 1, n,
                           (const double2*)ws.part, part2, o.cancel, ws.dev, ws.dhost);
        hipLaunchKernelGGL((k_gm_pass<T, true>), dim3(GM_BLOCKS), dim3(KB), 0, s, wj, (const T*)V, n, j + 1, n,
                           (const double2*)part2, ws.part, o.cancel, ws.dev, ws.dhost);
        if (!(st = mark()).ok()) return st;
      } else {
        dots(j + 2, wj, false);
        hipLaunchKernelGGL((k_gm_update<T, false>), dim3(g1), dim3(KB), 0, s, wj, (const T*)V, n,
                           (const GmScalars*)ws.dev, j + 1, n);
        dots(j + 2, wj, true);
        if (!(st = mark()).ok()) return st;
        hipLaunchKernelGGL((k_gm_update<T, true>), dim3(g1), dim3(KB), 0, s, wj, (const T*)V, n,
                           (const GmScalars*)ws.dev, j + 1, n);
      }
      ahead = j + 1 < m && inf.iters + 1 < o.max_iters;
      if (ahead && !(st = A(wj, wj + n, dt, s)).ok()) return st;
      if (!(st = wait()).ok()) return st;
      const double w2 = hs->w2, hn = hs->hn;
      for (int i = 0; i <= j; ++i) Hij(i, j) = cd(hs->h[i].x, hs->h[i].y);
      if (!std::isfinite(hn) || !std::isfinite(w2)) return bad(PSFD_ERR_NONFINITE, "non-finite Krylov vector");
      Hij(j + 1, j) = hn;
      ++inf.iters;
      k = j + 1;
      for (int i = 0; i < j; ++i) {  // previous rotations
        const cd a = Hij(i, j), c2 = Hij(i + 1, j);
        Hij(i, j) = cs[i] * a + sn[i] * c2;
        Hij(i + 1, j) = -std::conj(sn[i]) * a + cs[i] * c2;
      }
      const cd a = Hij(j, j);
      const double bb = hn, r = std::sqrt(std::norm(a) + bb * bb);
      if (r == 0.0) { cs[j] = 1.0; sn[j] = 0.0; }
      else if (std::abs(a) == 0.0) { cs[j] = 0.0; sn[j] = 1.0; }
      else { cs[j] = std::abs(a) / r; sn[j] = (a / std::abs(a)) * bb / r; }
      Hij(j, j) = cs[j] * a + sn[j] * bb;
      Hij(j + 1, j) = 0.0;
      g[j + 1] = -std::conj(sn[j]) * g[j];
      g[j] = cs[j] * g[j];
      if (std::abs(g[j + 1]) <= stop || hn == 0.0) break;
    }
    for (int i = k - 1; i >= 0; --i) {  // back substitution
      cd acc = g[i];
      for (int l = i + 1; l < k; ++l) acc -= Hij(i, l) * y[l];
      y[i] = acc / Hij(i, i);
    }
    GmCoefs yk;
    for (int i = 0; i < k; ++i) yk.c[i] = make_double2(y[i].real(), y[i].imag());
    hipLaunchKernelGGL(k_gm_axpys<T>, dim3(g1), dim3(KB), 0, s, X, (const T*)V, n, yk, k, n);
    // FP64 residual r = b - A x
    if (!(st = A(X, w64, PSFD_C128, s)).ok()) return st;
    if (!(st = residual(w64, beta)).ok()) return st;
    rel = beta / bnorm;
    if (!std::isfinite(rel)) return bad(PSFD_ERR_NONFINITE, "non-finite residual");
    if (rel <= o.rtol) { inf.status = PSFD_OK; break; }
  }
  inf.rel_residual = rel;
  inf.mono_residual = rel;
  GMCHK(hipGetLastError());
  GMCHK(hipStreamSynchronize(s));
  return Status();
}

}  // namespace

GmresWs::~GmresWs() {
  if (part) (void)hipFree(part);
  if (dev) (void)hipFree(dev);
  if (host) (void)hipHostFree(host);
  if (ev) (void)hipEventDestroy(ev);
}

static Status ws_ready(GmresWs& w) {
  if (!w.part) GMCHK(hipMalloc((void**)&w.part, 2 * sizeof(double2) * GM_BLOCKS * (GM_MAX + 2)));
  if (!w.dev) GMCHK(hipMalloc((void**)&w.dev, sizeof(GmScalars)));
  if (!w.host) {
    GMCHK(hipHostMalloc((void**)&w.host, sizeof(GmScalars), hipHostMallocCoherent | hipHostMallocMapped));
    GMCHK(hipHostGetDevicePointer((void**)&w.dhost, w.host, 0));
  }
  if (!w.ev) GMCHK(hipEventCreateWithFlags(&w.ev, hipEventDisableTiming));
  return Status();
}

Status gmres_host(long long n, const ApplyFn& A, const double2* b, double2* x, const HostGmres& o, psfd_info& info,
                  GmresWs& ws, hipStream_t s) {
  if (!(o.rtol > 0.0) || o.m < 1 || o.m > GM_MAX || o.max_iters < 1)
    return bad(PSFD_ERR_INVALID_ARG, "need rtol > 0, 1 <= restart <= 64, max_iters >= 1");
  if (o.precision != PSFD_FP64 && o.precision != PSFD_MIXED)
    return bad(PSFD_ERR_INVALID_ARG, "precision must be PSFD_FP64 or PSFD_MIXED");
  info.status = PSFD_NOT_CONVERGED;
  Status st = ws_ready(ws);
  if (!st.ok()) return st;
  return o.precision == PSFD_MIXED ? gmres_t<float2>(n, A, b, x, o, info, ws, s)
                                   : gmres_t<double2>(n, A, b, x, o, info, ws, s);
}

}  // namespace psfd
