// Quarter-plane kernels (operator apply): the transverse transform of an
// ny x nx plane split four ways over y. Block q of a plane takes the rows
// y = 4 r + q (r < ny / 4), transforms them along x (nx points) and along r
// (ny / 4 points), and stores the quarter spectrum times its twiddle,
// Y'_q(ky', kx) = W_ny^(q ky') Y_q(ky', kx), ky' < ny / 4. The full spectrum is
// the radix-4 decimation-in-time combine
//   X(ky' + (ny / 4) m, kx) = sum_q W4^(q m) Y'_q(ky', kx),
// a twiddle-free 4-point DFT that the z-pencil kernel takes on load. Back the
// same way: the pencil stores Z'_q = sum_m W4^(-q m) X(ky' + (ny / 4) m), and
// block q multiplies by W_ny^(-q ky') and transforms along r and x back to the
// rows y = 4 r + q.
//
// Why four blocks per plane. On 128 x 128 planes they keep every CU busy with
// three resident blocks whose loads and FFT passes overlap (768 blocks at 192
// planes); one block per plane leaves 64 of 256 CUs idle and runs each CU's
// load, transform and store one after the other. A 256 x 256 FP32 quarter is
// one block per CU, and the transform is one pass through HBM where row and
// column strips take two. On smaller and rectangular planes a stage is bound
// by the latency of one block's load - transform - store chain and by idle CUs
// (48 planes at 256 x 64 x 16): a quarter of the work per block in four times
// the blocks shortens that chain.
// Layout between the kernels, per plane: the four quarter spectra interleaved
// in pieces of four values, (q, ky', kx) at qp_index<nx>(ky', kx, q), so that
// the 16 values a pencil block takes at one (component, z) are contiguous.
#pragma once
#include <cstdio>
#include <cstdlib>

#include "kernels.hpp"
#include "fft_lds.hpp"

namespace psfd {

// Threads and values per thread of a block. FP32: 16 values on the planes of
// 4096 and more values per quarter (rows of 128 by radix 16 and 8, of 256 by
// 16 and 16), FP64 and the smaller planes 8; at least one thread per column and
// one wavefront. No pass takes a radix above the values of a thread.
template <class T, int LNX, int LNY> struct QpShape {
  static constexpr int NX = 1 << LNX, NY = 1 << LNY, ROWS = NY / 4, ELEM = ROWS * NX;
  static constexpr int KW = sizeof(T) == 8 && ELEM >= 4096 ? 16 : 8;
  static constexpr int N0 = ELEM / KW > NX ? ELEM / KW : NX;
  static constexpr int NT = N0 > 64 ? N0 : 64, KT = ELEM / NT;
  static constexpr int LKT = KT == 16 ? 4 : KT == 8 ? 3 : KT == 4 ? 2 : 1;
  static constexpr int LRM_ROWS = LKT, LRM_COLS = LKT < 3 ? LKT : 3;
  static constexpr int LRL = (LNY - 3) % LRM_COLS + 1, RL = 1 << LRL;  // last column pass: radix RL
  static constexpr size_t lds() { return ((size_t)ROWS * (NX + 1) + NX + (NX == NY ? 1 : 2) * ROWS) * sizeof(T); }
  static_assert(KT * NT == ELEM && NT % NX == 0 && (1 << LKT) == KT && ROWS <= NT && RL <= KT, "quarter-plane split");
};

template <int NX> PSFD_D int qp_index(int kyq, int kx, int q) { return kyq * (4 * NX) + (kx >> 2) * 16 + 4 * q + (kx & 3); }

template <class T, bool INV, int LD, int ST, int LNX, int LNY>
__global__ void __launch_bounds__((QpShape<T, LNX, LNY>::NT)) k_qplane(TileArgs a) {
  typedef QpShape<T, LNX, LNY> S;
  constexpr int NX = S::NX, NY = S::NY, QR = S::ROWS, P = NX + 1, NT = S::NT, KT = S::KT, TS = NT / NX;
  constexpr int PN = NX * NY;
  static_assert(!INV || LD == LD_PLAIN, "inverse: plain load");
  static_assert(INV || (LD == LD_VX && ST == ST_PLAIN), "forward: contrast multiply, plain store");
  extern __shared__ double2 smem_d[];
  T* lds = reinterpret_cast<T*>(smem_d);
  T* twx = lds + QR * P;  // W_nx^k, k < nx
  T* twr = twx + NX;      // W_(ny/4)^k, k < ny / 4
  T* twq = twr + QR;      // W_ny^(q k), k < ny / 4 (square planes: in twx)
  const int b = blockIdx.y;
  if (a.active && !a.active[b]) return;
  // block order: with 8 | nz, XCD x (= hw mod 8) takes the planes z = x mod 8 of
  // all three components and their four quarters, so the three blocks that read
  // one contrast plane share an L2, and so do the four that write (or read) one
  // 128-byte line of the layout
  int plane, q;
  {
    const int hw = blockIdx.x;
    if ((a.nz & 7) == 0) {
      const int xc = hw & 7, i = hw >> 3, t = i >> 2, c = t % 3, zz = t / 3;
      q = i & 3;
      plane = c * a.nz + xc + 8 * zz;
    } else {
      plane = hw >> 2;
      q = hw & 3;
    }
  }
  const int z = plane % a.nz;
  const long long poff = (long long)plane * PN;
  const int tid = threadIdx.x;
  typedef typename real_of<T>::type R;
  const T* twg = reinterpret_cast<const T*>(a.tw);
  const T tw0 = twg[NX + (tid & (NX - 1))];
  const T tw1 = twg[QR + (tid & (QR - 1))];
  T tw2;
  if constexpr (NX != NY) tw2 = twg[NY + q * (tid & (QR - 1))];
  // the twiddle loads ahead of the data loads: their LDS writes wait for them alone
  __builtin_amdgcn_sched_barrier(0);
  const T* in = vref<T>(a.in, b) + poff;
  const T* vol = INV ? nullptr : vref<T>(a.vol, b) + (long long)z * PN;
  const T* aux = ST == ST_AXPBY ? vref<T>(a.aux, b) + poff : nullptr;
  // the column transform's last pass (radix RL, stride PL = ny / 4 / RL)
  // leaves its results in registers: butterfly i of the thread (column
  // s = tid mod nx, index t = tid / nx + TS i) forms rows r = t + PL j of
  // that column
  constexpr int RL = S::RL, PL = QR / RL, NBL = KT / RL;
  static_assert(PL == TS * NBL && NBL * RL == KT, "quarter-plane last column pass");
  T va[KT], vb[INV ? 1 : KT], xa[ST == ST_AXPBY ? KT : 1];
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const int i = tid + k * NT, r = i >> LNX, x = i & (NX - 1);
    if constexpr (!INV) {
      va[k] = in[(4 * r + q) * NX + x];
      vb[k] = vol[(4 * r + q) * NX + x];
    } else {
      va[k] = in[qp_index<NX>(r, x, q)];
    }
  }
  if constexpr (ST == ST_AXPBY) {
#pragma unroll
    for (int i = 0; i < NBL; ++i)
#pragma unroll
      for (int j = 0; j < RL; ++j) {
        const int r = (tid >> LNX) + TS * i + PL * j, x = tid & (NX - 1);
        xa[i * RL + j] = aux[(4 * r + q) * NX + x];
      }
  }
  const double* tab = a.tab + (long long)b * a.tab_stride;
  R ks = (R)1;
  if constexpr (!INV) ks = (R)tab[TS_K0SQ] * (a.in_scale ? (R)a.in_scale[(long long)b * a.scale_stride] : (R)1);
  if (tid < NX) twx[tid] = tw0;
  if (tid < QR) twr[tid] = tw1;
  if constexpr (NX != NY)
    if (tid < QR) twq[tid] = tw2;
  auto wq = [&](int r) { return NX == NY ? twx[q * r] : twq[r]; };
  // the inverse multiplies by W_ny^(-q ky') on the way into LDS
  if constexpr (INV) __syncthreads();
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const int i = tid + k * NT, r = i >> LNX;
    T v;
    if constexpr (INV) v = cmulc(va[k], wq(r));
    else v = cscale(cmul(vb[k], va[k]), ks);
    lds[r * P + (i & (NX - 1))] = v;
  }
  __syncthreads();
  typedef FftCT<LNX, QR, P, 1, NT> Rows;      // ny / 4 rows of nx points
  typedef FftCT<LNY - 2, NX, 1, P, NT> Cols;  // nx columns of ny / 4 points
  lds_fft_tab<T, INV, true, KT, Rows, false, false, S::LRM_ROWS>(lds, Rows(), twx, tid);
  T res[KT];
  lds_fft_tab_regout<T, INV, true, KT, Cols, false, S::LRM_COLS>(lds, Cols(), twr, tid, res);
  T* out = vref<T>(a.out, b) + poff;
  const R al = (R)a.alpha, ga = (R)a.gamma;
#pragma unroll
  for (int i = 0; i < NBL; ++i)
#pragma unroll
    for (int j = 0; j < RL; ++j) {
      const int r = (tid >> LNX) + TS * i + PL * j, x = tid & (NX - 1);
      T v = res[i * RL + j];
      if constexpr (!INV) {
        out[qp_index<NX>(r, x, q)] = cmul(v, wq(r));
      } else {
        if constexpr (ST == ST_AXPBY) {
          const T xv = xa[ST == ST_AXPBY ? i * RL + j : 0];
          v.x = al * xv.x + ga * v.x;
          v.y = al * xv.y + ga * v.y;
        }
        out[(4 * r + q) * NX + x] = v;
      }
    }
}

// Whether a plane takes the quarter kernels: both sides 16 .. 256 and 1024 or
// more values (below, a quarter leaves a thread fewer than 4 values and its
// passes radix 2), at most 16384 FP32 or 8192 FP64 values per quarter (132 KB
// of LDS; a 256 x 256 FP64 quarter would need twice that). Whole apply, quarter
// planes against one block (or row and column strips) per plane, with the
// compile-time pencils: 32 x 32 x 32 FP64 20.5 -> 16.1 us, 256 x 64 x 16 FP32
// 46.8 -> 25.7, 64 x 128 x 16 FP32 36.6 -> 19.2, 64 x 32 x 64 FP32 24.6 -> 18.1,
// 128 x 32 x 64 FP32 30.4 -> 22.0, 64 x 64 x 32 FP32 20.7 -> 19.2, 128 x 128 x 64
// FP64 137 -> 105, 256 x 256 x 64 FP32 243 -> 221.
constexpr bool qplane_fits(int lnx, int lny, size_t esz) {
  return lnx >= 4 && lnx <= 8 && lny >= 4 && lny <= 8 && lnx + lny >= 10 && lnx + lny - 2 <= (esz == 8 ? 14 : 13);
}

template <class T, bool INV, int LD, int ST>
void launch_qplane(const TileArgs& a, int nplanes, int nbatch, hipStream_t s) {
  auto go = [&](auto kern, int nt, size_t l) {
    if (l > 65536)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)l);
    hipLaunchKernelGGL(kern, dim3(4 * nplanes, nbatch), dim3(nt), l, s, a);
  };
  bool done = false;
  if (!a.gv.st && nplanes == 3 * a.nz) {
    auto shape = [&](auto lx, auto ly) {
      constexpr int LX = decltype(lx)::value, LY = decltype(ly)::value;
      if constexpr (qplane_fits(LX, LY, sizeof(T))) {
        if (a.nx != 1 << LX || a.ny != 1 << LY) return;
        typedef QpShape<T, LX, LY> S;
        go(k_qplane<T, INV, LD, ST, LX, LY>, S::NT, S::lds());
        done = true;
      }
    };
    auto rows = [&](auto ly) {
      shape(std::integral_constant<int, 4>(), ly);
      shape(std::integral_constant<int, 5>(), ly);
      shape(std::integral_constant<int, 6>(), ly);
      shape(std::integral_constant<int, 7>(), ly);
      shape(std::integral_constant<int, 8>(), ly);
    };
    rows(std::integral_constant<int, 4>());
    rows(std::integral_constant<int, 5>());
    rows(std::integral_constant<int, 6>());
    rows(std::integral_constant<int, 7>());
    rows(std::integral_constant<int, 8>());
  }
  if (!done) {
    std::fprintf(stderr, "psfd: internal error: quarter-plane launch on an unsupported shape\n");
    std::abort();
  }
}

}  // namespace psfd
