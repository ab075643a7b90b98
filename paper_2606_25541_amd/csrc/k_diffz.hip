// Kernels of one apply of the differential operator with compile-time shapes:
//   k_diff_plane   2-D FFT of the planes (16 .. 128 a side), forward with the
//                  spectrum of V x beside that of x, or inverse with y -= V x;
//   k_diff_zcol    curl curl - k_bg^2 along z in the transverse spectrum (64 .. 1024
//                  planes), with the spectrum of V x taken off and the spectral
//                  damping applied in the same pass.
// One apply is three launches, with or without the damping:
//   y = IFFT_xy C FFT_xy x - V x,   D y = IFFT_xy D_z (C FFT_xy x - FFT_xy V x).
// (The run-time kernels take four and seven: V x as a pass of its own, and the
// damping as another forward transform, pencil and inverse.) Whole apply, before
// and after: 32 x 32 x 256 FP32 damped 97 -> 32.0 us, 64 x 64 x 128 FP64 undamped
// 70.7 -> 43.8, 16 x 32 x 128 FP32 undamped 39.0 -> 17. The FP64 case moves 160 MB
// (3.7 TB/s); the small ones are bound by the serial chain of a column's transforms
// and by launches.
#include "diff.hpp"
#include "fft_lds.hpp"
#include "regfft.hpp"

namespace psfd {

namespace {

// -------------------------------------------------------------------------
// Planes: one per block, 8 values per thread (4 on 256-value planes), rows then
// columns through LDS, the last column pass in registers (see k_plane).
// -------------------------------------------------------------------------
template <int LNX, int LNY> struct DpShape {
  static constexpr int NX = 1 << LNX, NY = 1 << LNY, N = NX * NY, P = NX + 1;
  static constexpr int NT = N / 8 >= 64 ? N / 8 : 64, KT = N / NT, LKT = KT == 8 ? 3 : 2;
  static constexpr int LRL = (LNY - 1) % LKT + 1, RL = 1 << LRL, PL = NY / RL, TS = NT / NX, NBL = KT / RL;
  static constexpr int ELEMS = NY * P + NX + NY;
  static_assert(NT * KT == N && NT % NX == 0 && PL == TS * NBL && (1 << LKT) == KT, "plane split");
};

template <class T, bool INV, int LNX, int LNY>
__global__ void __launch_bounds__((DpShape<LNX, LNY>::NT)) k_diff_plane(DiffPlaneArgs a) {
  typedef DpShape<LNX, LNY> S;
  typedef typename real_of<T>::type R;
  constexpr int N = S::N, NX = S::NX, NY = S::NY, P = S::P, NT = S::NT, KT = S::KT;
  extern __shared__ double2 smem_d[];
  T* lds = reinterpret_cast<T*>(smem_d);
  T* twx = lds + NY * P;
  T* twy = twx + NX;
  const int tid = threadIdx.x, np = 3 * a.pe;
  // forward: planes np + c ncz + k carry V x of contrast plane k
  int plane = blockIdx.x, kc = -1;
  if (INV) {
    const int k = plane % a.pe - a.zc0;
    if (k >= 0 && k < a.ncz && a.deps) kc = k;
  } else if (plane >= np) {
    const int q = plane - np;
    kc = q % a.ncz;
    plane = q / a.ncz * a.pe + a.zc0 + kc;
  }
  const T* in = (const T*)a.in + (long long)plane * N;
  const T* tg = (const T*)a.tw;
  T va[KT], vb[KT], xa[INV ? KT : 1];
#pragma unroll
  for (int k = 0; k < KT; ++k) va[k] = in[tid + k * NT];
  if (kc >= 0) {
    const T* dp = (const T*)a.deps + (long long)kc * N;
#pragma unroll
    for (int k = 0; k < KT; ++k) vb[k] = dp[tid + k * NT];
    if constexpr (INV) {
      const T* xp = (const T*)a.aux + (long long)plane * N;
#pragma unroll
      for (int k = 0; k < KT; ++k) xa[k] = xp[tid + k * NT];
    }
  }
  if (tid < NX) twx[tid] = tg[NX + tid];
  for (int i = tid; i < NY; i += NT) twy[i] = tg[NY + i];
  if constexpr (!INV) {
    if (kc >= 0) {
#pragma unroll
      for (int k = 0; k < KT; ++k) va[k] = cscale(cmul(vb[k], va[k]), (R)a.k0sq);
    }
  }
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const int i = tid + k * NT;
    lds[(i >> LNX) * P + (i & (NX - 1))] = va[k];
  }
  __syncthreads();
  typedef FftCT<LNX, NY, P, 1, NT> Rows;
  typedef FftCT<LNY, NX, 1, P, NT> Cols;
  lds_fft_tab<T, INV, true, KT, Rows, false, false, S::LKT>(lds, Rows(), twx, tid);
  T res[KT];
  lds_fft_tab_regout<T, INV, true, KT, Cols, false, S::LKT>(lds, Cols(), twy, tid, res);
  // butterfly i, output j: row (tid / nx + TS i) + PL j, plane element
  // tid + (i + NBL j) NT, one of the thread's own loaded ones
  T* out = !INV && kc >= 0 ? (T*)a.aux + (long long)((int)blockIdx.x - np) * N : (T*)a.out + (long long)blockIdx.x * N;
#pragma unroll
  for (int i = 0; i < S::NBL; ++i)
#pragma unroll
    for (int j = 0; j < S::RL; ++j) {
      const int k = i + S::NBL * j;
      T v = res[i * S::RL + j];
      if constexpr (INV) {
        if (kc >= 0) v = csub(v, cscale(cmul(vb[k], xa[INV ? k : 0]), (R)a.k0sq));
      }
      out[tid + k * NT] = v;
    }
}

// -------------------------------------------------------------------------
// z columns. A sequence (component, column) of N planes lives in TH = N / R1
// threads, thread t holding planes t + TH j (j < R1). Its DFT is one register DFT
// over j, an exchange through LDS, and the TH-point transform over t of every
// residue k1: a second register DFT where TH <= R1, else two with another exchange.
// The inverse goes back the same way, in place, to the same planes.
// -------------------------------------------------------------------------
template <class T, int N, int LB, int R1> struct ZF {
  static constexpr int TH = N / R1, E = R1;
  static constexpr bool L3 = TH > R1;
  static constexpr int K = L3 ? 1 : R1 / TH;       // two passes: residues per thread
  static constexpr int SK = L3 ? TH / 8 : 1;       // L3: TH = SK * 8, t = t0 + SK t1
  static constexpr int NM = R1 * SK / TH;          // L3: middle butterflies (radix 8) per thread
  static constexpr int NC = L3 ? R1 * 8 / TH : 1;  // L3: last butterflies (radix SK) per thread
  static_assert(!L3 || (SK <= 8 && NM >= 1 && NC >= 1 && NM * 8 == R1 && NC * SK == R1), "z column passes");
  // LDS position of (k1, t): rows of TH with a pad per row (L3: per SK), so that the
  // lanes of a pass (LB columns by consecutive t, or by consecutive k1 or t1) meet
  // distinct banks
  static constexpr int ROW = L3 ? (TH + TH / SK) * LB : TH * LB + LB;
  static constexpr int ELEMS = R1 * ROW;
  PSFD_D static int at(int k1, int t) { return k1 * ROW + (L3 ? t + t / SK : t) * LB; }
  // wavenumber index (0 .. N - 1) of register e of a spectrum
  PSFD_D static int freq(int t, int e) {
    if constexpr (L3) {
      const int b = t + TH * (e / SK);
      return (b >> 3) + R1 * ((b & 7) + 8 * (e % SK));
    } else {
      return t + TH * (e / TH) + R1 * (e % TH);
    }
  }
  // u: planes t + TH j -> spectrum; every thread of the block calls it (act: whether
  // its sequence takes part), after a pass that may still read buf
  PSFD_D static void fwd(T (&u)[E], T* buf, const T* tw, int t, bool act) {
    __syncthreads();
    if (act) {
      dft_r<T, R1, false>(u);
#pragma unroll
      for (int k = 0; k < R1; ++k) {
        if (L3 && k > 0) u[k] = cmul(u[k], tw[t * k]);
        buf[at(k, t)] = u[k];
      }
    }
    __syncthreads();
    if constexpr (!L3) {
      if (act) {
#pragma unroll
        for (int i = 0; i < K; ++i) {
          const int k1 = t + TH * i;
#pragma unroll
          for (int s = 0; s < TH; ++s) {
            T x = buf[at(k1, s)];
            if (s > 0) x = cmul(x, tw[s * k1]);
            u[i * TH + s] = x;
          }
          dft_r<T, TH, false>(u + i * TH);
        }
      }
    } else {
      if (act) {
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          const int b = t + TH * i, k1 = b / SK, t0 = b % SK;
          T v[8];
#pragma unroll
          for (int s = 0; s < 8; ++s) v[s] = buf[at(k1, t0 + SK * s)];
          dft_r<T, 8, false>(v);
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            if (s > 0) v[s] = cmul(v[s], tw[R1 * t0 * s]);
            buf[at(k1, t0 + SK * s)] = v[s];
          }
        }
      }
      __syncthreads();
      if (act) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int b = t + TH * i, k1 = b >> 3, m1 = b & 7;
#pragma unroll
          for (int s = 0; s < SK; ++s) u[i * SK + s] = buf[at(k1, s + SK * m1)];
          dft_r<T, SK, false>(u + i * SK);
        }
      }
    }
  }
  // spectrum -> planes t + TH j (unnormalised), from the registers fwd left
  PSFD_D static void inv(T (&u)[E], T* buf, const T* tw, int t, bool act) {
    if constexpr (!L3) {
      if (act) {
#pragma unroll
        for (int i = 0; i < K; ++i) {
          const int k1 = t + TH * i;
          dft_r<T, TH, true>(u + i * TH);
#pragma unroll
          for (int s = 0; s < TH; ++s) {
            T x = u[i * TH + s];
            if (s > 0) x = cmulc(x, tw[s * k1]);
            buf[at(k1, s)] = x;
          }
        }
      }
      __syncthreads();
    } else {
      if (act) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int b = t + TH * i, k1 = b >> 3, m1 = b & 7;
          dft_r<T, SK, true>(u + i * SK);
#pragma unroll
          for (int s = 0; s < SK; ++s) buf[at(k1, s + SK * m1)] = u[i * SK + s];
        }
      }
      __syncthreads();
      if (act) {
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          const int b = t + TH * i, k1 = b / SK, t0 = b % SK;
          T v[8];
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            v[s] = buf[at(k1, t0 + SK * s)];
            if (s > 0) v[s] = cmulc(v[s], tw[R1 * t0 * s]);
          }
          dft_r<T, 8, true>(v);
#pragma unroll
          for (int s = 0; s < 8; ++s) buf[at(k1, t0 + SK * s)] = v[s];
        }
      }
      __syncthreads();
    }
    if (act) {
#pragma unroll
      for (int k = 0; k < R1; ++k) {
        u[k] = buf[at(k, t)];
        if (L3 && k > 0) u[k] = cmulc(u[k], tw[t * k]);
      }
      dft_r<T, R1, true>(u);
#pragma unroll
      for (int k = 0; k < R1; ++k) pin(u[k]);
    }
  }
};

template <class T> PSFD_D T times_i(T a, typename real_of<T>::type k) {  // i k a
  T r;
  r.x = -k * a.y;
  r.y = k * a.x;
  return r;
}

// A block takes LB adjacent kx of one ky in three groups of LB TH threads, group g
// holding component g. Groups x and y form the z derivatives of u_x and u_y, then
// of c_y and c_x (c = curl u); each also reads the components its own result
// needs, and group z takes c_x and c_y through LDS. Three groups instead of one
// thread per column and plane residue, because the small transverse grids of
// these solves leave the chip short of wavefronts and the transforms of one
// thread form a serial chain.
// The values of planes (component c, t + TH j) are read from memory again where
// they are needed next instead of held (FP64: they do not fit).
template <class T, int N, int LB, int R1> struct ZcolShape {
  typedef ZF<T, N, LB, R1> F;
  static constexpr int GT = LB * F::TH, NT = 3 * GT;
  static constexpr int LDS = (3 * F::ELEMS + 2 * N) * (int)sizeof(T);  // buffers, twiddles, 1 / s(z)
  static_assert(GT % 64 == 0 && NT <= 1024 && LDS <= 160 * 1024, "z column split");
};

template <class T, int N, int LB, int R1, bool DAMP>
__global__ void __launch_bounds__((ZcolShape<T, N, LB, R1>::NT)) k_diff_zcol(DiffZcolArgs a) {
  typedef ZcolShape<T, N, LB, R1> S;
  typedef ZF<T, N, LB, R1> F;
  typedef typename real_of<T>::type R;
  constexpr int E = F::E, TH = F::TH;
  extern __shared__ double2 smem_d[];
  T* bufs = reinterpret_cast<T*>(smem_d);
  T* tw = bufs + 3 * F::ELEMS;
  T* inv_s = tw + N;
  const int tid = threadIdx.x, g = tid / S::GT, r = tid - g * S::GT, col = r % LB, t = r / LB;
  const int nblk = a.nx / LB, ky = blockIdx.x / nblk, kx = (blockIdx.x - ky * nblk) * LB + col;
  T* buf = bufs + g * F::ELEMS + col;
  // component c, plane t + TH j of the thread's column: lane offset go, scalar at(c, j)
  const unsigned plane = (unsigned)(a.nx * a.ny) * (unsigned)sizeof(T);
  const LaneBuf w(a.w, 3u * N * plane);
  const unsigned go = (unsigned)t * plane + (unsigned)(ky * a.nx + kx) * (unsigned)sizeof(T);
  // the group's component is uniform over its wavefronts
  const int gu = __builtin_amdgcn_readfirstlane(g);
  auto at = [&](int c, int j) { return (unsigned)(c * N + TH * j) * plane; };
  T u[E];
#pragma unroll
  for (int j = 0; j < E; ++j) w.load(u[j], go, at(gu, j));
  const T* tg = (const T*)a.tw + N;
  const double2* sg = reinterpret_cast<const double2*>(a.zt + 2 * N);
  for (int i = tid; i < N; i += S::NT) {
    tw[i] = tg[i];
    inv_s[i] = from_d<T>(sg[i]);
  }
  const double kxd = a.kx[kx], kyd = a.ky[ky], dk = a.zt[N + 1];  // kappa_l = l dk
  const R kxv = (R)kxd, kyv = (R)kyd, kb2 = (R)a.kbg2;
  const bool xy = g < 2;
  // i kappa_l / N on the spectrum (the z-Nyquist derivative is zero)
  auto deriv = [&]() {
    F::fwd(u, buf, tw, t, xy);
    if (xy) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int l = F::freq(t, e), ls = l < N / 2 ? l : l - N;
        u[e] = times_i(u[e], (R)((l == N / 2 ? 0.0 : (double)ls * dk) * (1.0 / N)));
      }
    }
    F::inv(u, buf, tw, t, xy);
    if (xy) {
#pragma unroll
      for (int j = 0; j < E; ++j) u[j] = cmul(u[j], inv_s[t + TH * j]);
    }
  };
  deriv();
  // group x: c_y = D u_x - i kx u_z; group y: c_x = i ky u_z - D u_y
  if (xy) {
    const R k = g == 0 ? -kxv : kyv, sd = g == 0 ? (R)1 : (R)-1;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      T z;
      w.load(z, go, at(2, j));
      u[j] = cadd(cscale(u[j], sd), times_i(z, k));
    }
  }
  // group z: (curl c)_z - k_bg^2 u_z = i kx c_y - i ky c_x - k_bg^2 u_z
  __syncthreads();
  if (xy) {
#pragma unroll
    for (int j = 0; j < E; ++j) buf[(t + TH * j) * LB] = u[j];
  }
  __syncthreads();
  if (!xy) {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const T cy = bufs[(t + TH * j) * LB + col], cx = bufs[F::ELEMS + (t + TH * j) * LB + col];
      u[j] = csub(csub(times_i(cy, kxv), times_i(cx, kyv)), cscale(u[j], kb2));
    }
  }
  deriv();
  // group x: i ky c_z - D c_y - k_bg^2 u_x; group y: D c_x - i kx c_z - k_bg^2 u_y;
  // c_z = i kx u_y - i ky u_x
  if (xy) {
    const R k = g == 0 ? kyv : -kxv, sd = g == 0 ? (R)-1 : (R)1;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      T ux, uy;
      w.load(ux, go, at(0, j));
      w.load(uy, go, at(1, j));
      const T cz = csub(times_i(uy, kxv), times_i(ux, kyv));
      u[j] = csub(cadd(cscale(u[j], sd), times_i(cz, k)), cscale(g == 0 ? ux : uy, kb2));
    }
  }
  const R inv_t = (R)(1.0 / ((double)a.nx * a.ny));
  R sc = inv_t;
  if constexpr (DAMP) {
    // the spectrum of V x on the contrast planes
    const LaneBuf vx(a.vx, 3u * (unsigned)a.ncz * plane);
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const int k = t + TH * j - a.zc0;
      if (k >= 0 && k < a.ncz) {
        T v;
        vx.load(v, (unsigned)k * plane + (unsigned)(ky * a.nx + kx) * (unsigned)sizeof(T), (unsigned)(gu * a.ncz) * plane);
        u[j] = csub(u[j], v);
      }
    }
    F::fwd(u, buf, tw, t, true);
    const double kt2 = kxd * kxd + kyd * kyd;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int l = F::freq(t, e);
      const double kap = (double)(l < N / 2 ? l : l - N) * dk, k2 = kt2 + kap * kap;
      u[e] = cscale(u[e], (R)((k2 > a.kbg2 ? a.kbg2 / k2 : 1.0) * (1.0 / N)));
    }
    F::inv(u, buf, tw, t, true);
  } else {
    __syncthreads();  // every group has read what the others overwrite
  }
#pragma unroll
  for (int j = 0; j < E; ++j) w.store(cscale(u[j], sc), go, at(gu, j));
}

}  // namespace

// Which shapes take these kernels: planes of 16 .. 128 a side of at most 8192
// FP32 or 4096 FP64 values, z lengths 64 .. 1024, and at least the columns of a block.
template <class T> static constexpr int zcol_lb(int n) {
  return n <= 128 ? 8 : n == 1024 && sizeof(T) == 16 ? 2 : 4;
}
// 16 planes per thread instead of 8 (32 x 32 x 512 FP64 damped 62.2 -> 55.4 us with 8,
// 64 x 64 x 512 FP64 damped 229 -> 205, FP32 148 -> 127, 64 x 64 x 128 FP64 47.1 -> 45.1,
// 32 x 32 x 256 FP32 damped 34.4 -> 32.9): only FP64 with damping at 256 planes in more
// than 512 blocks, whose two exchanges and 97 registers then bound it
// (64 x 64 x 256 105 us with 16, 111 with 8; 32 x 64, 512 blocks, 55.8 and 53.0).
template <class T> static constexpr bool zcol_wide(int n) { return sizeof(T) == 16 && n == 256; }
template <class T> static constexpr bool dplane_fits(int lx, int ly) {
  return lx >= 4 && lx <= 7 && ly >= 4 && ly <= 7 && lx + ly <= (sizeof(T) == 8 ? 13 : 12);
}
template <class T> bool diff_ct_shape(int nx, int ny, int pe) {
  return dplane_fits<T>(ilog2i(nx), ilog2i(ny)) && pe >= 64 && pe <= 1024;
}
template bool diff_ct_shape<float2>(int, int, int);
template bool diff_ct_shape<double2>(int, int, int);

template <class K, class A> static void run(K kern, int nblk, int nt, int lds, hipStream_t s, const A& args) {
  if (lds > 65536) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  hipLaunchKernelGGL(kern, dim3((unsigned)nblk), dim3(nt), (size_t)lds, s, args);
}

template <class T, bool INV>
bool launch_diff_plane(const DiffPlaneArgs& a, int nx, int ny, int nplanes, hipStream_t s) {
  bool done = false;
  auto shape = [&](auto lx, auto ly) {
    constexpr int LX = decltype(lx)::value, LY = decltype(ly)::value;
    if constexpr (dplane_fits<T>(LX, LY)) {
      if (nx != 1 << LX || ny != 1 << LY) return;
      typedef DpShape<LX, LY> S;
      run(k_diff_plane<T, INV, LX, LY>, nplanes, S::NT, S::ELEMS * (int)sizeof(T), s, a);
      done = true;
    }
  };
  auto rows = [&](auto ly) {
    shape(std::integral_constant<int, 4>(), ly);
    shape(std::integral_constant<int, 5>(), ly);
    shape(std::integral_constant<int, 6>(), ly);
    shape(std::integral_constant<int, 7>(), ly);
  };
  rows(std::integral_constant<int, 4>());
  rows(std::integral_constant<int, 5>());
  rows(std::integral_constant<int, 6>());
  rows(std::integral_constant<int, 7>());
  return done;
}
template bool launch_diff_plane<float2, false>(const DiffPlaneArgs&, int, int, int, hipStream_t);
template bool launch_diff_plane<float2, true>(const DiffPlaneArgs&, int, int, int, hipStream_t);
template bool launch_diff_plane<double2, false>(const DiffPlaneArgs&, int, int, int, hipStream_t);
template bool launch_diff_plane<double2, true>(const DiffPlaneArgs&, int, int, int, hipStream_t);

template <class T>
bool launch_diff_zcol(const DiffZcolArgs& a, int pe, bool damp, hipStream_t s) {
  auto go = [&](auto n) {
    constexpr int N = decltype(n)::value, LB = zcol_lb<T>(N);
    const int nblk = a.ny * (a.nx / LB);
    auto one = [&](auto r) {
      constexpr int R1 = decltype(r)::value;
      typedef ZcolShape<T, N, LB, R1> S;
      if (damp) run(k_diff_zcol<T, N, LB, R1, true>, nblk, S::NT, S::LDS, s, a);
      else run(k_diff_zcol<T, N, LB, R1, false>, nblk, S::NT, S::LDS, s, a);
    };
    // 8 planes per thread, which gives a column twice the wavefronts of 16 and each
    // half the chain, for one more exchange (N = 1024 has no such split). One kind
    // is faster with 16: see zcol_wide.
    if constexpr (zcol_wide<T>(N)) {
      if (damp && nblk > 512) {
        one(std::integral_constant<int, 16>());
        return true;
      }
    }
    one(std::integral_constant<int, N == 1024 ? 16 : 8>());
    return true;
  };
  switch (pe) {
    case 64: return go(std::integral_constant<int, 64>());
    case 128: return go(std::integral_constant<int, 128>());
    case 256: return go(std::integral_constant<int, 256>());
    case 512: return go(std::integral_constant<int, 512>());
    case 1024: return go(std::integral_constant<int, 1024>());
  }
  return false;
}
template bool launch_diff_zcol<float2>(const DiffZcolArgs&, int, bool, hipStream_t);
template bool launch_diff_zcol<double2>(const DiffZcolArgs&, int, bool, hipStream_t);

}  // namespace psfd
