// Quarter-plane kernels (operator apply and Arnoldi steps): the transverse transform of an
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
#include "krylov.hpp"
#include "givens.hpp"
#include "fft_lds.hpp"
#include "regfft.hpp"

namespace psfd {

// Threads and values per thread of a block. FP32: 16 values on quarters of more
// than 4096 values (256 x 256: 1024 threads), 4 at 1024 (256 threads shorten the
// chain that bounds them: 64 x 64 x 32 apply 18.9 -> 18.0 us against 8), else 8. At
// 4096 values 16 above 32 planes (WIDE), where the blocks are enough to fill the
// chip, 8 up to there; 8 against 16 values: apply 256 x 64 x 16 26.9 against 28.2 us,
// 128 x 128 x 16 23.8 against 25.1, 128 x 128 x 32 36.3 against 36.6, 256 x 64 x 64 53.3
// against 52.4; with the Gram-Schmidt work a step at 128 x 128 x 8 41.3 against 43.1,
// at 32 planes 66.3 alike, at 64 105.7 against 103.7 (the plain apply of 128 x 128 x 64
// is level). FP64: 8. At least one thread per column and one wavefront. No pass
// takes a radix above the values of a thread.
template <class T, int LNX, int LNY, bool WIDE> struct QpShape {
  static constexpr int NX = 1 << LNX, NY = 1 << LNY, ROWS = NY / 4, ELEM = ROWS * NX;
  static constexpr int KW = sizeof(T) == 16 ? 8 : ELEM >= (WIDE ? 4096 : 8192) ? 16 : ELEM == 1024 ? 4 : 8;
  static constexpr int N0 = ELEM / KW > NX ? ELEM / KW : NX;
  static constexpr int NT = N0 > 64 ? N0 : 64, KT = ELEM / NT;
  static constexpr int LKT = KT == 16 ? 4 : KT == 8 ? 3 : KT == 4 ? 2 : 1;
  static constexpr int LRM_ROWS = LKT, LRM_COLS = LKT < 3 ? LKT : 3;
  static constexpr int LRL = (LNY - 3) % LRM_COLS + 1, RL = 1 << LRL;  // last column pass: radix RL
  // projection partials a lane of the update requests at once: all 12 of the wide
  // shapes (768 partials at 64 planes; in two rounds of 6 the second waits for the
  // first, 16 x 128 x 128 x 64 1909 -> 1880 us a step), else 6 (all at 32 planes; 12
  // cost registers: 256 x 256 spills, 423 -> 444, four 64 x 64 x 64 116.8 -> 117.9)
  static constexpr int DU = WIDE ? 12 : 6;
  static constexpr size_t lds() { return ((size_t)ROWS * (NX + 1) + NX + (NX == NY ? 1 : 2) * ROWS) * sizeof(T); }
  static_assert(KT * NT == ELEM && NT % NX == 0 && (1 << LKT) == KT && ROWS <= NT && RL <= KT, "quarter-plane split");
};

template <int NX> PSFD_D int qp_index(int kyq, int kx, int q) { return kyq * (4 * NX) + (kx >> 2) * 16 + 4 * q + (kx & 3); }

// ---- Gram-Schmidt work of an Arnoldi step inside the transverse kernels -------
// The forward kernel of a step also does the update of the column before, the
// inverse one the projections of the vector it writes: a block owns the same
// values of every basis slot, element k of a thread at lane + k 4 NT values from
// the plane's start in both directions, so a slot is read once per kernel and
// the new vector not again. Bound by the slot reads on large planes and by the
// block's chain (partials - sum - slots - transform) and the launch itself on
// 64 x 64 ones; four blocks per plane overlap those chains. Mean over the columns
// of GMRES(8), against one block per plane carrying the same work: 128 x 128 x 64
// forward 36.4 -> 31.3 us, inverse 31.5 -> 28.0; 64 x 64 x 32 10.6 -> 9.4 and 9.9 ->
// 8.0. Whole Arnoldi step: 128 x 128 x 64 112.7 -> 103.1 us, 128 x 128 x 16 72 -> 54,
// 64 x 64 x 32 36.5 -> 31.7; shapes that ran separate projection and update passes:
// 64 x 128 x 32 72.6 -> 40.9, 256 x 64 x 32 101 -> 64, 256 x 256 x 64 509 -> 407.
//
// The slots are read in groups of G whose loads are issued together (slots past
// the last are empty buffers, which load nothing). Two of 4 values per thread,
// else one: more in flight costs registers, and with them resident blocks, which
// hide the chains better (64 x 64 x 32, groups of 8 / 4 / 2 / 1: 33.9 / 32.7 / 31.7 /
// 31.6 us a step, eight instances 119.6 / 114.5 / 110.6 / 111.8).
// With nt the slots are read past the caches: where the slots of the instances
// that run exceed them (qp_past_caches; the limit is the launch's).
template <class S> constexpr int qp_group() { return S::KT == 4 ? 2 : 1; }

template <class S, class T, int KT, int G>
PSFD_D void qp_slots(const T* V, long long ldv, bool nt, int i0, int cnt, unsigned lane, T (&p)[G][KT]) {
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const LaneBuf s(V + (long long)min(i0 + g, cnt - 1) * ldv, i0 + g < cnt ? S::NX * S::NY * (int)sizeof(T) : 0);
    if (nt) {
#pragma unroll
      for (int k = 0; k < KT; ++k) s.load_nt(p[g][k], lane, k * 4 * S::NT * (int)sizeof(T));
    } else {
#pragma unroll
      for (int k = 0; k < KT; ++k) s.load(p[g][k], lane, k * 4 * S::NT * (int)sizeof(T));
    }
  }
}

// Whether the slots are read past the caches: mode 2 counts the launch's running
// instances (their flags in `active`; the same answer in every lane).
PSFD_D bool qp_past_caches(int mode, int cached, const int* active) {
  if (mode < 2) return mode != 0;
  const int nb = gridDim.y, lane = threadIdx.x & 63;
  int n = 0;
  for (int i = 0; i < nb; i += 64) n += __popcll(__ballot(i + lane < nb && active[min(i + lane, nb - 1)] != 0));
  return n > cached;
}

// The Gram-Schmidt update of column cnt - 1 on this block's values wv of slot
// cnt, in place: w - sum_{i<cnt} h_i s_i slot_i, stored back to the slot; this
// block's ||slot||^2 goes to part[pidx]. h_i = s_i <slot_i, w> from the projection
// partials, summed by every block in one fixed order (dots_total), so all get the
// same coefficients bit for bit; block 0 stores h and ||w||^2 before the update
// for the Givens step.
template <class S, class T, int KT>
PSFD_D void qp_update(const TileArgs& a, int cnt, T (&wv)[KT], const LaneBuf& slot, unsigned lane, int b,
                      int pidx, long long poff) {
  constexpr int NT = S::NT, NW = NT / 64, G = qp_group<S>();
  typedef typename real_of<T>::type R;
  __shared__ T hc[MAXM];
  __shared__ double nred[NW];
  const UpdateTask& u = a.up;
  const int tid = threadIdx.x, wave = tid >> 6;
  GState& St = u.st[b];
  const T* sb = reinterpret_cast<const T*>(u.V) + (long long)b * u.bsv + poff;
  const double2* pb = u.dpart + (long long)b * PSTR * u.nblk;
  const bool nt = qp_past_caches(u.nt, u.cached, a.active);
  T p[G][KT];
  qp_slots<S>(sb, u.ldv, nt, 0, cnt, lane, p);
  for (int i = wave; i <= cnt; i += NW) {
    const double sc = St.sc[i];
    const double2 t = dots_total<S::DU>(pb + (long long)i * u.nblk, u.nblk);
    if ((tid & 63) == 0) {
      if (i < cnt) {
        hc[i] = from_d<T>(cscale(t, sc * sc));
        if (pidx == 0) St.h[i] = cscale(t, sc);
      } else if (pidx == 0) {
        St.wn2_in = t.x;  // value cnt is ||w||^2
      }
    }
  }
  __syncthreads();
  for (int i0 = 0; i0 < cnt; i0 += G) {
    if (i0 > 0) qp_slots<S>(sb, u.ldv, nt, i0, cnt, lane, p);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (i0 + g < cnt) {
        const T h = hc[i0 + g];
#pragma unroll
        for (int k = 0; k < KT; ++k) {
          wv[k].x -= h.x * p[g][k].x - h.y * p[g][k].y;
          wv[k].y -= h.x * p[g][k].y + h.y * p[g][k].x;
        }
      }
    }
  }
  R nn = 0;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    slot.store(wv[k], lane, k * 4 * NT * (int)sizeof(T));
    nn += wv[k].x * wv[k].x + wv[k].y * wv[k].y;
  }
  nn = lane_sum(nn);
  if ((tid & 63) == 0) nred[wave] = (double)nn;
  __syncthreads();
  if (tid == 0) {
    double t = nred[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) t += nred[w];
    u.part[(long long)b * (12 * a.nz) + pidx] = make_double2(t, 0.0);
  }
}

// Gram-Schmidt projections of this block's values wv of the new Arnoldi vector:
// partial <slot_i, w> for i < cnt and ||w||^2, summed in the vector precision
// within a wavefront and in FP64 across the wavefronts in a fixed order, stored
// as partial pidx of nblk (indices no block owns get zeros). p holds the first
// group of slots (qp_slots before the transform).
template <class S, class T, int KT, int G>
PSFD_D void qp_dots(const TileArgs& a, bool nt, int cnt, const T (&wv)[KT], T (&p)[G][KT], const T* sb, unsigned lane, int b,
                    int pidx) {
  constexpr int NW = S::NT / 64;
  static_assert(S::lds() >= (size_t)PSTR * NW * sizeof(double2), "partials fit the block's LDS");
  extern __shared__ double2 smem_d[];
  double2* red = smem_d;  // [PSTR][NW]; the plane's LDS is free after the barrier
  const DotTask& d = a.dt;
  const int tid = threadIdx.x, wave = tid >> 6;
  __syncthreads();
  for (int i0 = 0; i0 < cnt; i0 += G) {
    if (i0 > 0) qp_slots<S>(sb, d.ldv, nt, i0, cnt, lane, p);
    // all G sums side by side (zeros for the slots past the last)
    T acc[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      acc[g] = cmake<T>(0, 0);
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        acc[g].x += p[g][k].x * wv[k].x + p[g][k].y * wv[k].y;
        acc[g].y += p[g][k].x * wv[k].y - p[g][k].y * wv[k].x;
      }
      acc[g] = cmake<T>(lane_sum(acc[g].x), lane_sum(acc[g].y));
    }
    if ((tid & 63) == 0) {
#pragma unroll
      for (int g = 0; g < G; ++g)
        if (i0 + g < cnt) red[(i0 + g) * NW + wave] = to_d(acc[g]);
    }
  }
  typename real_of<T>::type nn = 0;
#pragma unroll
  for (int k = 0; k < KT; ++k) nn += wv[k].x * wv[k].x + wv[k].y * wv[k].y;
  nn = lane_sum(nn);
  if ((tid & 63) == 0) red[cnt * NW + wave] = make_double2((double)nn, 0.0);
  __syncthreads();
  if (tid <= cnt) {
    double2 t = red[tid * NW];
#pragma unroll
    for (int w = 1; w < NW; ++w) t = cadd(t, red[tid * NW + w]);
    double2* pp = d.part + ((long long)b * PSTR + tid) * d.nblk;
    pp[pidx] = t;
    for (int i = pidx + 12 * a.nz; i < d.nblk; i += 12 * a.nz) pp[i] = make_double2(0, 0);
  }
  // the update of this column is now pending (read by the next step's kernels)
  if (pidx == 0 && tid == 0) d.st[b].pend = 1;
}

template <class T, bool INV, int LD, int ST, int LNX, int LNY, bool WIDE>
__global__ void __launch_bounds__((QpShape<T, LNX, LNY, WIDE>::NT)) k_qplane(TileArgs a) {
  typedef QpShape<T, LNX, LNY, WIDE> S;
  constexpr int NX = S::NX, NY = S::NY, QR = S::ROWS, P = NX + 1, NT = S::NT, KT = S::KT, TS = NT / NX;
  constexpr int PN = NX * NY;
  static_assert(!INV || LD == LD_PLAIN, "inverse: plain load");
  constexpr bool UPD = LD == LD_UPD_VX || LD == LD_UPD_SLOT;  // Gram-Schmidt update on load
  constexpr bool DOTS = ST == ST_DOTS;
  constexpr bool GIV = LD == LD_VX_GIV;  // with the pending Givens step
  static_assert(INV || ((LD == LD_VX || GIV || UPD) && ST == ST_PLAIN), "forward: contrast multiply, plain store");
  extern __shared__ double2 smem_d[];
  T* lds = reinterpret_cast<T*>(smem_d);
  T* twx = lds + QR * P;  // W_nx^k, k < nx
  T* twr = twx + NX;      // W_(ny/4)^k, k < ny / 4
  T* twq = twr + QR;      // W_ny^(q k), k < ny / 4 (square planes: in twx)
  const int b = blockIdx.y;
  // the Givens step of the column before in the extra last block of the grid; the
  // others scale the input by the norm they sum from the same partials, bitwise the
  // task's (as a launch of its own it costs a step more: GMRES(8)
  // 128 x 128 x 16 FP64 96.0 -> 92.6 us, 64 x 64 x 8 FP64 48.5 -> 46.2, 64 x 64 x 16
  // mixed 35.6 -> 33.1, 128 x 128 x 64 FP64 at restart 30 467 -> 462.5)
  if constexpr (GIV) {
    if (blockIdx.x == gridDim.x - 1) {
      givens_task<NT>(a.gv.st, a.gv.run, a.gv.part, a.gv.nblk, b);
      return;
    }
  }
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
  // the update of column cnt - 1 on slot cnt; per instance (up.j < 0) only with a
  // pending update, and at up.j = 0 not at all: then the plain scaled load of the
  // slot (by S.inv_norm, as LD_VX with in_scale)
  int cnt = 0;
  bool upd = LD == LD_UPD_VX;
  if constexpr (UPD) cnt = a.up.j;
  if constexpr (LD == LD_UPD_SLOT) {
    if (a.up.j >= 0) {
      upd = cnt > 0;
    } else {
      const GState& St = a.up.st[b];
      const int pend = St.pend, js = St.j;
      upd = pend != 0;
      cnt = __builtin_amdgcn_readfirstlane(js + 1);
      in = reinterpret_cast<const T*>(a.up.V) + (long long)b * a.up.bsv + (long long)(upd ? js + 1 : js) * a.up.ldv +
           poff;
    }
  }
  const T* vol = INV ? nullptr : vref<T>(a.vol, b) + (long long)z * PN;
  const T* aux = ST == ST_AXPBY ? vref<T>(a.aux, b) + poff : nullptr;
  // the column transform's last pass (radix RL, stride PL = ny / 4 / RL)
  // leaves its results in registers: butterfly i of the thread (column
  // s = tid mod nx, index t = tid / nx + TS i) forms rows r = t + PL j of
  // that column
  constexpr int RL = S::RL, PL = QR / RL, NBL = KT / RL;
  static_assert(PL == TS * NBL && NBL * RL == KT, "quarter-plane last column pass");
  T va[KT], vb[INV ? 1 : KT], xa[ST == ST_AXPBY ? KT : 1];
  const unsigned lane = ((4 * (tid >> LNX) + q) * NX + (tid & (NX - 1))) * (unsigned)sizeof(T);
  if constexpr (UPD) {
    const LaneBuf slot(in, PN * (unsigned)sizeof(T));
#pragma unroll
    for (int k = 0; k < KT; ++k) slot.load(va[k], lane, k * 4 * NT * (int)sizeof(T));
    const LaneBuf vbuf(vol, PN * (unsigned)sizeof(T));
    constexpr bool VB0 = KT < 16;  // ahead of the slots where the registers allow it
#pragma unroll
    for (int k = 0; k < KT && VB0; ++k) vbuf.load(vb[k], lane, k * 4 * NT * (int)sizeof(T));
    if (LD == LD_UPD_VX || upd) qp_update<S>(a, cnt, va, slot, lane, b, 4 * plane + q, poff);
#pragma unroll
    for (int k = 0; k < KT && !VB0; ++k) vbuf.load(vb[k], lane, k * 4 * NT * (int)sizeof(T));
  } else
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
  // the first group of basis slots, on its way during the transform
  constexpr int G = qp_group<S>();
  T p[DOTS ? G : 1][DOTS ? KT : 1];
  const T* sb = nullptr;
  bool nt = false;
  if constexpr (DOTS) {
    nt = qp_past_caches(a.dt.nt, a.dt.cached, a.active);
    sb = reinterpret_cast<const T*>(a.dt.V) + (long long)b * a.dt.bsv + poff;
    cnt = a.dt.jh + 1;
    if (a.dt.jh < 0) cnt = __builtin_amdgcn_readfirstlane(a.dt.st[b].j) + 1;
    qp_slots<S>(sb, a.dt.ldv, nt, 0, cnt, lane, p);
  }
  const double* tab = a.tab + (long long)b * a.tab_stride;
  R ks = (R)1;
  // LD_UPD_*: an updated vector enters unscaled (the pencil kernel scales it)
  if constexpr (UPD) ks = (R)tab[TS_K0SQ] * (LD == LD_UPD_SLOT && !upd ? (R)a.up.st[b].inv_norm : (R)1);
  else if constexpr (GIV)
    ks = (R)tab[TS_K0SQ] * (R)inv_norm_of(norm_from_partials<NT>(a.gv.part + (long long)b * a.gv.nblk, a.gv.nblk));
  else if constexpr (!INV) ks = (R)tab[TS_K0SQ] * (a.in_scale ? (R)a.in_scale[(long long)b * a.scale_stride] : (R)1);
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
        if constexpr (DOTS) va[i + NBL * j] = v;  // row 4 r + q: element k = i + NBL j of the thread
      }
    }
  if constexpr (DOTS) qp_dots<S>(a, nt, cnt, va, p, sb, lane, b, 4 * plane + q);
}

// Whether a plane takes the quarter kernels: both sides 16 .. 256 and 1024 or
// more values (below, a quarter leaves a thread fewer than 4 values and its
// passes radix 2), at most 16384 FP32 or 8192 FP64 values per quarter (132 KB
// of LDS; a 256 x 256 FP64 quarter would need twice that). Whole apply, quarter
// planes against one block (or row and column strips) per plane, with the
// compile-time pencils: 32 x 32 x 32 FP64 20.5 -> 16.1 us, 256 x 64 x 16 FP32
// 46.8 -> 24.0, 64 x 128 x 16 FP32 36.6 -> 19.2, 64 x 32 x 64 FP32 24.6 -> 18.1,
// 128 x 32 x 64 FP32 30.4 -> 22.0, 64 x 64 x 32 FP32 20.7 -> 17.7, 128 x 128 x 64
// FP64 137 -> 105, 256 x 256 x 64 FP32 243 -> 221.
constexpr bool qplane_fits(int lnx, int lny, size_t esz) {
  return lnx >= 4 && lnx <= 8 && lny >= 4 && lny <= 8 && lnx + lny >= 10 && lnx + lny - 2 <= (esz == 8 ? 14 : 13);
}

// Whether the quarter kernels of a plane also carry the Gram-Schmidt work of an
// Arnoldi step: FP32 (mixed precision's inner solves), 4096 and more values per
// plane. Every block of the update sums all 12 nz partials of each projection, so
// on smaller planes that sum would outweigh the block's own values; they keep
// the separate passes.
constexpr bool qplane_gs_fits(int lnx, int lny, size_t esz) {
  return esz == 8 && qplane_fits(lnx, lny, esz) && lnx + lny >= 12;
}

template <class T, bool INV, int LD, int ST>
void launch_qplane(const TileArgs& a, int nplanes, int nbatch, hipStream_t s) {
  constexpr bool GIV = LD == LD_VX_GIV;
  auto go = [&](auto kern, int nt, size_t l) {
    if (l > 65536)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)l);
    hipLaunchKernelGGL(kern, dim3(4 * nplanes + (GIV ? 1 : 0), nbatch), dim3(nt), l, s, a);
  };
  bool done = false;
  if ((a.gv.st != nullptr) == GIV && nplanes == 3 * a.nz) {
    auto shape = [&](auto lx, auto ly) {
      constexpr int LX = decltype(lx)::value, LY = decltype(ly)::value;
      constexpr bool GS = ST == ST_DOTS || LD == LD_UPD_VX || LD == LD_UPD_SLOT;
      if constexpr (GS ? qplane_gs_fits(LX, LY, sizeof(T)) : qplane_fits(LX, LY, sizeof(T))) {
        if (a.nx != 1 << LX || a.ny != 1 << LY) return;
        // the 16-value split by the shape alone, so that a solve takes the same
        // arithmetic by itself, in a batch and in a server's slot
        constexpr bool W = sizeof(T) == 8 && LX + LY == 14;
        auto split = [&](auto wide) {
          constexpr bool WIDE = decltype(wide)::value;
          typedef QpShape<T, LX, LY, WIDE> S;
          go(k_qplane<T, INV, LD, ST, LX, LY, WIDE>, S::NT, S::lds());
        };
        if (W && a.nz > 32) split(std::bool_constant<W>());
        else split(std::false_type());
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
