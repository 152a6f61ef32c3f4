// Matrix-free local part of H_hat: the tensor-structured multivector product
// that the paper names as future work (Sec. VI), for 2-component spinors.
//
// Per cell e and column n the product of the cell operator of eqn:FEHlocEl with
// the gathered, M_D^{-1/2}-scaled spinor u = (u_up, u_dn) is evaluated without
// forming the cell matrix:
//   1. U = (B (x) B (x) B)^T u        values at the quadrature points (3 passes)
//   2. W = w_q J [(V + |k|^2/2) U + (B_xc . sigma) U]          pointwise
//   3. for each direction d: G_d = D_d U (collocation derivative along d),
//        W += D_d^T (w_q J G_d / 2) - i k_d w_q J G_d
//   4. y = (B (x) B (x) B) W            back to the nodes (3 passes)
// and y, scaled by M_D^{-1/2}, is added into the output rows of the cell's nodes.
// B[a][q] = l_a(x_q) is the 1-D GLL-node Lagrange basis at the quadrature points
// and D_d = (2/h_d) Dq with Dq[q][r] = l~_r'(x_q) the derivative of the Lagrange
// basis on the quadrature points.  With n_q = p + 1 points per direction both
// are exact for the degree-p fields of the cell, so the result equals the
// product with the assembled cell matrices (kinetic K, mass, k-gradient C,
// potential and field matrices) up to rounding: same quadrature, different
// order of summation.  Work per cell and column is 9 line contractions of
// n_p^4 complex-by-real multiply-adds per spin in FP64 at k = 0 (12 with the k-term
// and in FP32), against 4 (2 n_p^3)^2 for the dense cell product, and no cell
// matrices are stored.
//
// FP64, or FP32 (mixed precision: tables, quadrature data, LDS fields and
// arithmetic in FP32, rows converted on gather and added into the FP64 output).
//
// Launch: one workgroup of 256 (FP64) or 512 (FP32) threads per (cell of one
// colour, chunk of CW columns).  Both spins of CW columns live in two LDS buffers of
// n_p^3 complex values per field; each thread owns one line (along the pass direction)
// of one (column, spin) field, keeps it in registers and writes the contracted
// line, so every LDS value read feeds n_p multiply-adds.  Within a colour no
// two cells share a node, so the scatter is a plain read-add-write.  Or one launch for
// all cells, which writes the products out cell by cell (ye).
#include <functional>

#include "mfma.h"
#include "sumfact.h"

namespace chfsi {

namespace {

template <class T> struct MfT;
template <> struct MfT<double> {
  typedef double2 C2;
  typedef double4 Q4;
  static constexpr int NT = 256;
};
template <> struct MfT<float> {
  typedef float2 C2;
  typedef float4 Q4;
  static constexpr int NT = 512;
};

struct MfMesh {
  int nx, ny;               // cells along x, y
  int Nx, Ny, Nz, Nxy;      // nodes
};
// waves per SIMD that the registers are limited for: what the LDS lets share a CU, as
// far as the registers do not spill much (FP64 at n_p = 6 and five waves: 54 ms for
// an adjoint that takes 42 at four)
template <class T>
constexpr int mf_waves(int NP) { return sizeof(T) == 8 ? (NP <= 6 ? 4 : NP == 8 ? 2 : 3) : (NP <= 7 ? 6 : 3); }
// columns per workgroup: the same LDS bytes in both precisions
template <class T>
constexpr int mf_cw(int NP) { return sizeof(T) == 8 ? sf_cols(NP) : 2 * sf_cols(NP); }

// Kinetic and k-gradient terms of one line u along direction d, added into w:
//   w += a_d Dq^T (wJ Dq u) - i b_d wJ Dq u,
// a_d = (2/h_d)^2 / 2, b_d = k_d (2/h_d), wJ = wl w1[q] with wl = J times the two
// weights held fixed along the line.  FP64: wl comes out of the first term, which is
// one contraction with K = Dq^T diag(w1) Dq (eoK) instead of two (with the second
// term, K and Dq: two as before).  FP32 keeps Dq and Dq^T: their rounded tables hold
// the identities listed in mf_prepare, and the kinetic weights a_d wJ come per point
// from kin (formed in FP64 and rounded once), since products of the shared 1-D
// weights rounded in FP32 would bias the operator the same way in every cell.
template <class T, int NP, bool KT>
__device__ __forceinline__ void grad_line(const T* __restrict__ eoDf, const T* __restrict__ eoDb,
                                          const T* __restrict__ eoK, const T* __restrict__ w1, T wl, T a_d, T b_d,
                                          const T* __restrict__ kin, const typename MfT<T>::C2 (&u)[NP],
                                          typename MfT<T>::C2 (&w)[NP]) {
  typedef typename MfT<T>::C2 C2;
  if constexpr (sizeof(T) == 8 && !KT) {
    const T c = a_d * wl;
    sf_eo_each<T, NP, false>(eoK, u, [&](int r, C2 v) {
      w[r] = C2{fma(c, v.x, w[r].x), fma(c, v.y, w[r].y)};
      if (r >= NP / 2) __builtin_amdgcn_sched_barrier(0);   // (one pair's sums at a time in registers)
    });
  } else if constexpr (sizeof(T) == 8) {
    C2 g[NP], dw[NP];
    sf_eo<T, NP, false>(eoK, u, dw);
    const T c = a_d * wl;
#pragma unroll
    for (int r = 0; r < NP; ++r) w[r] = C2{fma(c, dw[r].x, w[r].x), fma(c, dw[r].y, w[r].y)};
    // (the barriers keep the two contractions' registers apart)
    __builtin_amdgcn_sched_barrier(0);
    sf_eo<T, NP, true>(eoDf, u, g);
#pragma unroll
    for (int r = 0; r < NP; ++r) {        // -i b wJ g = b wJ g.y - i b wJ g.x
      const T s = b_d * wl * w1[r];
      w[r].x = fma(s, g[r].y, w[r].x);
      w[r].y = fma(-s, g[r].x, w[r].y);
    }
    __builtin_amdgcn_sched_barrier(0);
  } else {
    C2 g[NP], fk[NP];
    sf_eo<T, NP, true>(eoDf, u, g);
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const T k = kin[q * NP * NP];
      fk[q] = C2{k * g[q].x, k * g[q].y};
    }
    sf_eo_each<T, NP, true>(eoDb, fk, [&](int r, C2 v) { w[r] = C2{w[r].x + v.x, w[r].y + v.y}; });
    if constexpr (KT) {
#pragma unroll
      for (int r = 0; r < NP; ++r) {
        const T s = b_d * wl * w1[r];
        w[r].x = fma(s, g[r].y, w[r].x);
        w[r].y = fma(-s, g[r].x, w[r].y);
      }
    }
  }
}

// Lines of a pass along y: groups of 8 lanes share one z, so that the lanes of a
// 128-bit LDS access hit distinct banks (consecutive lines of n_p = 6, 7 overlap by
// the pitch of a plane: conflicts per LDS cycle 0.37 with them, 0.34 so, at n_p = 7); other
// orders keep consecutive lines.
template <int NP>
constexpr int mf_ypitch() { return NP == 6 || NP == 7 ? 8 : NP; }

// Points between neighbouring x-lines in LDS: n_p = 8 would put every line of an x pass
// on the same banks (degree-6 filter, k = 0, FP64, 128 columns on 8^3 cells: 10.2 against
// 10.4 ms).
template <int NP>
constexpr int mf_pitch() { return NP == 8 ? 9 : NP; }

// Phase 3 in two parts, the x-lines of each spin by themselves (each thread reads the other
// spin's values from LDS), instead of both spins' lines in one thread.  Together saves
// a pass over the LDS, but takes the registers of four lines and half the threads (a
// quarter of them at n_p >= 8).  With the k-term that never pays: against together,
// FP64 degree-6 filter, 128 columns: p = 5, 14^3 cells 17.3 and 17.8 ms, p = 6, 12^3
// 17.8 and 18.4, p = 7, 8^3 9.9 and 11.8, p = 8, 8^3 17.7 and 20.0; FP32, p = 6, 15.9 and
// 17.5.  At k = 0 it pays for n_p = 8 (9.9 and 10.4, FP32 8.3 and 9.2) and in FP32 for 7 (15.8
// and 16.2), not elsewhere (FP64 p = 6 17.7 and 17.3, p = 8 18.9 and 17.7).
template <class T, int NP, bool KT>
constexpr bool mf_split() { return KT || NP == 8 || (sizeof(T) == 4 && NP == 7); }

// tab: [B: NP*NP][Dq: NP*NP][w: NP][even-odd tables of B, B^T, Dq, Dq^T, K], qd:
// [E][x][y + NP z] of (wJ V, wJ Bx, wJ By, wJ Bz), kin: [3][point on the line][line],
// all in the arithmetic type T.  Both run along the lines' index first, so that the
// lanes of a load share cache lines (point after point along x, every lane was on a
// line of its own, and the lookups cost more than the rows').
//
// One workgroup per work item (cell of the colour, chunk of CW columns); items
// are cell major and consecutive items run on one XCD (workgroup b on XCD b % 8),
// so the column chunks of a cell share its rows in that XCD's L2.  Seven phases,
// a thread owning one line in each:
//   1. z-lines of x gathered, B            5. + kinetic z, then B^T along z
//   2. y: B                                6. B^T along y
//   3. x: B -> U; potential, kinetic x     7. B^T along x, y scattered
//   4. + kinetic y
// (phase 3 takes the x-lines of both spins together or one by one, see mf_split).
// Nothing saturates: the vector units (36 % busy), the requests of 32-byte row
// pieces to L2 (42 % of one per clock and channel), the LDS and the waits for rows (41 %
// of the wave cycles; p = 6, k = 0, FP64) each take a share at the three workgroups per
// CU that 44 KB of LDS allow, so each is kept short: one contraction per kinetic term
// (FP64), one 64-bit multiplication per line's addresses, quadrature data in the order of the lanes, the old values of the
// output rows loaded right after phase 3 and used in phase 7, barriers that order
// LDS only.  Per colour launch of 512 cells, p = 6, 128 columns: 0.73 -> 0.61 ms; filter
// of 16^3 cells, degree 24: 225 -> 205 ms.
// Slower here (whole filter, 16^3 cells): the y and z kinetic terms carried along the
// interpolation as one more field (five phases, 11 contractions for 9, a fifth of
// the LDS traffic less) 217 ms, the spins of phase 3 in neighbouring lanes 207 ms, x
// and z exchanged 207 ms; field pitches without bank conflicts changed nothing.
template <class T, int NP, bool KT>
__global__ __launch_bounds__(MfT<T>::NT, mf_waves<T>(NP)) void mf_apply_kernel(
    const T* __restrict__ tab, const typename MfT<T>::Q4* __restrict__ qd, const MfMesh mesh,
    const int32_t* __restrict__ cells, int total, int n_chunks, const double* __restrict__ minv_sqrt,
    const double2* __restrict__ X, int64_t ldx, double2* __restrict__ Y, int64_t ldy, int n_vec, double alpha,
    T J, T half_k2, T a0, T a1, T a2, T b0, T b1, T b2, const T* __restrict__ kin,
    const double* __restrict__ alpha_d, typename MfT<T>::C2* __restrict__ ye) {
  typedef typename MfT<T>::C2 C2;
  typedef typename MfT<T>::Q4 Q4;
  constexpr int NT = MfT<T>::NT;
  constexpr int CW = mf_cw<T>(NP);
  constexpr int N2 = NP * NP, N3 = N2 * NP;
  constexpr int YP = mf_ypitch<NP>(), NY = YP * NP;
  constexpr int SY = mf_pitch<NP>(), SZ = SY * NP, SF = SZ * NP;   // point (x, y, z): x + SY y + SZ z
  static_assert(2 * CW * N2 <= NT, "one edge task per thread");
  extern __shared__ double2 mf_sm_raw[];
  C2* bufU = reinterpret_cast<C2*>(mf_sm_raw);   // [CW][2][SF]
  C2* bufW = bufU + CW * 2 * SF;
  T* w2 = reinterpret_cast<T*>(bufW + CW * 2 * SF);  // [N2] J w_a w_b
  const T* w1 = tab + 2 * N2;
  const T* eoBf = tab + 2 * N2 + NP;
  const T* eoBb = eoBf + sf_eo_size(NP);
  const T* eoDf = eoBb + sf_eo_size(NP);
  const T* eoDb = eoDf + sf_eo_size(NP);
  const T* eoK = eoDb + sf_eo_size(NP);
  const int tid = threadIdx.x;

  const int per_xcd = (total + 7) / 8;
  const int item = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (item >= total) return;
  // edge task: column fastest, then spin, then the line, so that neighbouring
  // lanes read one row
  const bool edge = tid < 2 * CW * N2;
  const int tc = tid % CW, ts = (tid / CW) % 2, tl = tid / (2 * CW);
  const int ta = tl % NP, tb = tl / NP;          // the line's two fixed indices
  const int tf = (tc * 2 + ts) * SF;
  const int e = cells ? cells[item / n_chunks] : item / n_chunks;
  const int col = (item % n_chunks) * CW + tc;
  const int cx = e % mesh.nx, cyz = e / mesh.nx;
  const int cy = cyz % mesh.ny, cz = cyz / mesh.ny;
  const bool ok = edge && col < n_vec;
  // nodes of a line along d: the first, and a step that wraps at the line's end
  // where the cell is the last of its row (uniform over the workgroup)
  const int fx = cx * (NP - 1), fy = cy * (NP - 1), fz = cz * (NP - 1);
  const auto wrap = [](int i, int n) { return i >= n ? i - n : i; };
  const int last_x = fx + NP - 1 == mesh.Nx ? -fx : NP - 1;
  const int last_z = fz + NP - 1 == mesh.Nz ? -fz : NP - 1;

  // 1. gather M^{-1/2} x along the task's z-line (addresses clamped in bounds)
  if (edge) {
    const int cc = ok ? col : 0;
    const int I0 = wrap(fx + ta, mesh.Nx) + mesh.Nx * wrap(fy + tb, mesh.Ny) + mesh.Nxy * fz;
    const double2* __restrict__ x0 = X + ((2 * (int64_t)I0 + ts) * ldx + cc);
    const int64_t zs = 2 * mesh.Nxy * ldx;
    double xs[NP];
    double2 xr[NP];
#pragma unroll
    for (int z = 0; z < NP; ++z) {
      const int k = z == NP - 1 ? last_z : z;
      xs[z] = minv_sqrt[I0 + mesh.Nxy * k];
      xr[z] = x0[zs * k];
    }
    if (tid < N2) w2[tid] = J * w1[tid % NP] * w1[tid / NP];
    C2 u[NP], r[NP];
#pragma unroll
    for (int z = 0; z < NP; ++z) {
      const double f = ok ? xs[z] : 0.0;
      u[z] = C2{(T)(f * xr[z].x), (T)(f * xr[z].y)};
    }
    sf_eo<T, NP, false>(eoBf, u, r);
#pragma unroll
    for (int o = 0; o < NP; ++o) bufU[tf + ta + SY * tb + o * SZ] = r[o];
  }
  lds_barrier();

  // a line of a y phase: field and first point; false for the lanes that pad a group
  const auto yline = [&](int t, int& f, int& l) {
    const int g = t % NY, fi = t / NY, x = g % YP, z = g / YP;
    l = x + NP * z;
    f = fi * SF + x + z * SZ;
    return x < NP;
  };
  // 2. y
  for (int t = tid; t < NY * 2 * CW; t += NT) {
    int p, l;
    if (!yline(t, p, l)) continue;
    C2 v[NP], r[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) v[j] = bufU[p + j * SY];
    sf_eo<T, NP, false>(eoBf, v, r);
#pragma unroll
    for (int o = 0; o < NP; ++o) bufU[p + o * SY] = r[o];
  }
  lds_barrier();

  // 3. x-lines: U, potential and field, kinetic x
  if constexpr (mf_split<T, NP, KT>()) {
    for (int t = tid; t < N2 * 2 * CW; t += NT) {
      const int l = t % N2, base = (t / N2) * SF + l * SY;
      C2 v[NP], r[NP];
#pragma unroll
      for (int j = 0; j < NP; ++j) v[j] = bufU[base + j];
      sf_eo<T, NP, false>(eoBf, v, r);
#pragma unroll
      for (int o = 0; o < NP; ++o) bufU[base + o] = r[o];
    }
    lds_barrier();
    for (int t = tid; t < N2 * 2 * CW; t += NT) {
      const int l = t % N2, f = t / N2, base = f * SF + l * SY, other = (f ^ 1) * SF + l * SY;
      const Q4* __restrict__ dq = qd + (size_t)e * N3 + l;
      const T wl = w2[l], sg = (f & 1) ? (T)-1 : (T)1;
      C2 u[NP], s[NP];
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        u[q] = bufU[base + q];
        // up:   (s + Bz) u0 + (Bx - i By) u1;  down: (s - Bz) u1 + (Bx + i By) u0
        const C2 o = bufU[other + q];
        const Q4 d = dq[q * N2];
        const T sv = (KT ? d.x + half_k2 * (wl * w1[q]) : d.x) + sg * d.w, dz = sg * d.z;
        s[q].x = sv * u[q].x + d.y * o.x + dz * o.y;
        s[q].y = sv * u[q].y + d.y * o.y - dz * o.x;
      }
      grad_line<T, NP, KT>(eoDf, eoDb, eoK, w1, wl, a0, b0, kin + l, u, s);
#pragma unroll
      for (int q = 0; q < NP; ++q) bufW[base + q] = s[q];
    }
  } else {
    for (int t = tid; t < N2 * CW; t += NT) {
      const int l = t % N2, base = (t / N2) * 2 * SF + l * SY;
      const Q4* __restrict__ dq = qd + (size_t)e * N3 + l;
      const T wl = w2[l];
      C2 u0[NP], u1[NP], s0[NP], s1[NP];
      {
        C2 v[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) v[j] = bufU[base + j];
        sf_eo<T, NP, false>(eoBf, v, u0);
#pragma unroll
        for (int j = 0; j < NP; ++j) v[j] = bufU[base + SF + j];
        sf_eo<T, NP, false>(eoBf, v, u1);
      }
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        bufU[base + q] = u0[q];
        bufU[base + SF + q] = u1[q];
        // up:   (s + Bz) u0 + (Bx - i By) u1;  down: (s - Bz) u1 + (Bx + i By) u0
        const Q4 d = dq[q * N2];
        const T s = d.x;
        s0[q].x = (s + d.w) * u0[q].x + d.y * u1[q].x + d.z * u1[q].y;
        s0[q].y = (s + d.w) * u0[q].y + d.y * u1[q].y - d.z * u1[q].x;
        s1[q].x = (s - d.w) * u1[q].x + d.y * u0[q].x - d.z * u0[q].y;
        s1[q].y = (s - d.w) * u1[q].y + d.y * u0[q].y + d.z * u0[q].x;
      }
      grad_line<T, NP, KT>(eoDf, eoDb, eoK, w1, wl, a0, b0, kin + l, u0, s0);
      grad_line<T, NP, KT>(eoDf, eoDb, eoK, w1, wl, a0, b0, kin + l, u1, s1);
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        bufW[base + q] = s0[q];
        bufW[base + SF + q] = s1[q];
      }
    }
  }

  // the output rows of phase 7's x-line, in flight while the next phases run
  const int I7 = fx + mesh.Nx * wrap(fy + ta, mesh.Ny) + mesh.Nxy * wrap(fz + tb, mesh.Nz);
  double2* __restrict__ y0 = Y + ((2 * (int64_t)I7 + ts) * ldy + col);
  // (FP64; in FP32, with the k-term from n_p = 7 on, and at n_p = 9 their registers cost
  // more: p = 6, k != 0, 128 columns on 12^3 cells 2.50 ms with them, 2.42 without; p = 5
  // 1.80 and 1.85; p = 8, k = 0, degree-6 filter on 8^3 18.5 and 17.9)
  constexpr bool kEarly = sizeof(T) == 8 && NP <= (KT ? 6 : 8);
  double2 yo[NP];
  if (kEarly && ok && !ye) {
#pragma unroll
    for (int o = 0; o < NP; ++o) yo[o] = y0[2 * ldy * (o == NP - 1 ? last_x : o)];
  }
  lds_barrier();

  // 4. kinetic y
  for (int t = tid; t < NY * 2 * CW; t += NT) {
    int p, l;
    if (!yline(t, p, l)) continue;
    C2 u[NP], w[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) u[j] = bufU[p + j * SY];
#pragma unroll
    for (int j = 0; j < NP; ++j) w[j] = bufW[p + j * SY];
    grad_line<T, NP, KT>(eoDf, eoDb, eoK, w1, w2[l], a1, b1, kin + N3 + l, u, w);
#pragma unroll
    for (int j = 0; j < NP; ++j) bufW[p + j * SY] = w[j];
  }
  lds_barrier();

  // 5. kinetic z; W is then complete, and goes back along z
  for (int t = tid; t < N2 * 2 * CW; t += NT) {
    const int l = t % N2, base = (t / N2) * SF + l % NP + SY * (l / NP);
    C2 u[NP], w[NP], r[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) u[j] = bufU[base + j * SZ];
#pragma unroll
    for (int j = 0; j < NP; ++j) w[j] = bufW[base + j * SZ];
    grad_line<T, NP, KT>(eoDf, eoDb, eoK, w1, w2[l], a2, b2, kin + 2 * N3 + l, u, w);
    sf_eo<T, NP, false>(eoBb, w, r);
#pragma unroll
    for (int j = 0; j < NP; ++j) bufW[base + j * SZ] = r[j];
  }
  lds_barrier();

  // 6. back along y
  for (int t = tid; t < NY * 2 * CW; t += NT) {
    int p, l;
    if (!yline(t, p, l)) continue;
    C2 v[NP], r[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) v[j] = bufW[p + j * SY];
    sf_eo<T, NP, false>(eoBb, v, r);
#pragma unroll
    for (int o = 0; o < NP; ++o) bufW[p + o * SY] = r[o];
  }
  lds_barrier();

  // 7. back along x, then Y[rows] += alpha M^{-1/2} y
  if (ok) {
    C2 v[NP], y[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) v[j] = bufW[tf + tl * SY + j];
    sf_eo<T, NP, false>(eoBb, v, y);
    if (ye) {                             // all cells in one launch: gathered by the caller
      C2* __restrict__ yr = ye + (((size_t)e * N3 + tl * NP) * 2 + ts) * n_vec + col;
#pragma unroll
      for (int o = 0; o < NP; ++o) yr[(size_t)2 * n_vec * o] = y[o];
      return;
    }
    const double al = alpha_d ? *alpha_d : alpha;
    if (!kEarly) {
#pragma unroll
      for (int o = 0; o < NP; ++o) yo[o] = y0[2 * ldy * (o == NP - 1 ? last_x : o)];
    }
#pragma unroll
    for (int o = 0; o < NP; ++o) {
      const int k = o == NP - 1 ? last_x : o;
      const double sc = al * minv_sqrt[I7 + k];
      y0[2 * ldy * k] = double2{fma(sc, (double)y[o].x, yo[o].x), fma(sc, (double)y[o].y, yo[o].y)};
    }
  }
}

// qd[e][x][y + nq z] = w_q J (V, Bx, By, Bz), in FP64 and FP32
__global__ void mf_qdata_kernel(const double* __restrict__ V, const double* __restrict__ B,
                                const double* __restrict__ w1, double J, int nq, int64_t n_points,
                                double4* __restrict__ qd, float4* __restrict__ qd32) {
  const int nq3 = nq * nq * nq;
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n_points;
       p += (int64_t)gridDim.x * blockDim.x) {
    const int q = (int)(p % nq3);
    const double wj = J * w1[q % nq] * w1[(q / nq) % nq] * w1[q / (nq * nq)];
    const double4 v = double4{wj * V[p], wj * B[3 * p], wj * B[3 * p + 1], wj * B[3 * p + 2]};
    const int64_t o = p - q + (q % nq) * (nq * nq) + q / nq;
    qd[o] = v;
    qd32[o] = float4{(float)v.x, (float)v.y, (float)v.z, (float)v.w};
  }
}

template <class T, int NP, bool KT>
void launch_mf_t(chfsi_ctx* c, const KPoint& kp, const double2* X, int64_t ldx, double2* W, int64_t ldw, int n_vec,
                 double alpha, const double* alpha_d, void* ye) {
  typedef typename MfT<T>::C2 C2;
  typedef typename MfT<T>::Q4 Q4;
  constexpr int CW = mf_cw<T>(NP);
  const size_t sh = 2 * (size_t)CW * 2 * mf_pitch<NP>() * NP * NP * sizeof(C2) + NP * NP * sizeof(T);
  const MfMesh mesh{c->nc[0], c->nc[1], c->Nd[0], c->Nd[1], c->Nd[2], c->Nd[0] * c->Nd[1]};
  const int n_chunks = cdiv(n_vec, CW);
  T a[3], b[3];
  for (int d = 0; d < 3; ++d) {
    const double sd = 2.0 / c->h[d];
    a[d] = (T)(0.5 * sd * sd);
    b[d] = (T)(kp.k[d] * sd);
  }
  const T half_k2 = (T)(0.5 * (kp.k[0] * kp.k[0] + kp.k[1] * kp.k[1] + kp.k[2] * kp.k[2]));
  const T* tab = nullptr;
  const Q4* qd = nullptr;
  const T* kin = nullptr;    // FP32 only (FP64 forms the weights in the kernel)
  if constexpr (sizeof(T) == 8) {
    tab = c->mf_tab.ptr;
    qd = reinterpret_cast<const Q4*>(c->mf_qd.ptr);
    kin = tab;
  } else {
    tab = c->mf_tab32.ptr;
    qd = reinterpret_cast<const Q4*>(c->mf_qd32.ptr);
    kin = c->mf_kin32.ptr;
  }
  const double np3 = (double)NP * NP * NP;
  for (int k = 0; k < (ye ? 1 : c->n_colours); ++k) {
    const int n_in = ye ? c->n_cells : c->colour_off[k + 1] - c->colour_off[k];
    if (n_in == 0) continue;
    const int64_t total = (int64_t)n_in * n_chunks;
    CHFSI_CHECK(total < (int64_t)1 << 30, CHFSI_EINVAL, "matrix-free apply: too many work items");
    // algorithmic flops of the dense cell product (the filter's count), flops of the
    // kernel's line contractions taken as dense, 9 or 12 per spin (the even-odd form
    // issues about half of those multiply-adds), and the rows moved
    const double n2 = 2.0 * c->nloc;
    const double flops = 8.0 * n2 * n2 * n_vec * n_in;
    const double exec = (sizeof(T) == 8 && !KT ? 72.0 : 96.0) * np3 * NP * (double)n_vec * n_in;
    const double bytes = (double)n_in * 3.0 * c->nloc * 2.0 * n_vec * sizeof(double2);
    StageTimer tm(c, sizeof(T) == 8 ? CHFSI_STAGE_CELL_FP64 : CHFSI_STAGE_CELL_FP32, flops, exec, bytes);
    const int grid = (int)(8 * ((total + 7) / 8));
    hipLaunchKernelGGL((mf_apply_kernel<T, NP, KT>), dim3(grid), dim3(MfT<T>::NT), sh, c->stream, tab, qd,
                       mesh, ye ? nullptr : c->colour_cells.ptr + c->colour_off[k], (int)total, n_chunks,
                       c->minv_sqrt.ptr, X, ldx, W, ldw, n_vec, alpha, (T)c->J, half_k2, a[0], a[1], a[2], b[0],
                       b[1], b[2], kin, alpha_d, (C2*)ye);
    LAUNCH_CHECK();
  }
}

template <int NP>
void launch_mf_np(chfsi_ctx* c, const KPoint& kp, bool fp64, const double2* X, int64_t ldx, double2* W, int64_t ldw,
                  int n_vec, double alpha, const double* alpha_d, void* ye) {
  if (fp64) {
    if (kp.gamma) launch_mf_t<double, NP, false>(c, kp, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye);
    else launch_mf_t<double, NP, true>(c, kp, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye);
  } else {
    if (kp.gamma) launch_mf_t<float, NP, false>(c, kp, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye);
    else launch_mf_t<float, NP, true>(c, kp, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye);
  }
}

}  // namespace

bool mf_supported(const chfsi_ctx* c) { return c->nq == c->np1 && c->np1 >= 2 && c->np1 <= 9; }

int64_t mf_items_per_cell(const chfsi_ctx* c, int n_vec, bool fp64) {
  return cdiv(n_vec, fp64 ? mf_cw<double>(c->np1) : mf_cw<float>(c->np1));
}

void mf_prepare(chfsi_ctx* c) {
  CHFSI_CHECK(mf_supported(c), CHFSI_EINVAL, "matrix-free apply needs n_q = p + 1 and 1 <= p <= 8");
  const int n = c->np1;
  std::vector<double> Bq, Dlag;
  lagrange_on(c->ref.xq, c->ref.xq, Bq, Dlag);   // Dlag[r][q] = l~_r'(x_q)
  std::vector<double> tab(2 * n * n + n);
  for (int a = 0; a < n; ++a)
    for (int q = 0; q < n; ++q) tab[a * n + q] = c->ref.B[(size_t)a * c->nq + q];
  for (int q = 0; q < n; ++q)
    for (int r = 0; r < n; ++r) tab[n * n + q * n + r] = Dlag[(size_t)r * n + q];
  for (int q = 0; q < n; ++q) tab[2 * n * n + q] = c->ref.wq[q];
  // even-odd tables of B (nodes -> points), B^T, Dq (G = Dq U), Dq^T and K, each as
  // out[o] = sum_i M[i][o] in[i]
  const int h = n / 2, es = 2 * h * h + 2 * h + 1;
  auto Bm = [&](int i, int o) { return tab[i * n + o]; };
  auto Dm = [&](int q, int r) { return tab[n * n + q * n + r]; };
  auto eo = [&](const std::function<double(int, int)>& M, bool skew) {
    double big = 0.0, dev = 0.0;
    for (int i = 0; i < n; ++i)
      for (int o = 0; o < n; ++o) {
        big = std::max(big, std::fabs(M(i, o)));
        dev = std::max(dev, std::fabs(M(n - 1 - i, n - 1 - o) - (skew ? -1.0 : 1.0) * M(i, o)));
      }
    CHFSI_CHECK(dev <= 1e-12 * std::max(1.0, big), CHFSI_EINVAL, "quadrature rule is not symmetric");
    std::vector<double> t(es, 0.0);
    for (int i = 0; i < h; ++i)
      for (int o = 0; o < h; ++o) {
        t[i * h + o] = 0.5 * (M(i, o) + M(i, n - 1 - o));
        t[h * h + i * h + o] = 0.5 * (M(i, o) - M(i, n - 1 - o));
      }
    if (n % 2) {
      for (int o = 0; o < h; ++o) t[2 * h * h + o] = M(h, o);
      for (int i = 0; i < h; ++i) t[2 * h * h + h + i] = M(i, h);
      t[2 * h * h + 2 * h] = M(h, h);
    }
    tab.insert(tab.end(), t.begin(), t.end());
  };
  eo([&](int i, int o) { return Bm(i, o); }, false);
  eo([&](int i, int o) { return Bm(o, i); }, false);
  eo([&](int i, int o) { return Dm(o, i); }, true);
  eo([&](int i, int o) { return Dm(i, o); }, true);
  // K = Dq^T diag(w) Dq (centrosymmetric, for a symmetric rule), summed in extended
  // precision; the closing entry of each sum over a constant's image is re-formed
  // so that K maps constants to zero as Dq does
  const int k0 = (int)tab.size();
  eo([&](int i, int o) {
    long double k = 0.0;
    for (int q = 0; q < n; ++q) k += (long double)c->ref.wq[q] * Dm(q, i) * Dm(q, o);
    return (double)k;
  }, false);
  for (int o = 0; o < h; ++o) {
    long double sum = 0.0;                 // 2 sum_i A[i][o] + M[h][o] = 0
    for (int i = 0; i < h - (n % 2 == 0); ++i) sum += tab[k0 + i * h + o];
    if (n % 2) tab[k0 + 2 * h * h + o] = (double)(-2.0L * sum);
    else tab[k0 + (h - 1) * h + o] = (double)-sum;
  }
  if (n % 2) {
    long double sum = 0.0;                 // 2 sum_i M[i][h] + M[h][h] = 0
    for (int i = 0; i < h; ++i) sum += tab[k0 + 2 * h * h + h + i];
    tab[k0 + 2 * h * h + 2 * h] = (double)(-2.0L * sum);
  }
  std::vector<float> tab32(tab.begin(), tab.end());
  // The FP32 tables keep identities of the exact ones, so that rounding them does
  // not perturb every cell the same way: the interpolation reproduces constants
  // and linear functions (sum_a l_a = 1, sum_a xi_a l_a(x) = x) and the
  // collocation derivative maps them to 0 and 1.  In each sum the closing entry
  // is re-formed in FP64 from the rounded others.  The tables of the transposed
  // contractions are then taken from the rounded forward ones (for a
  // centrosymmetric M the even-odd blocks of M^T are those of M transposed; for a
  // skew one the two blocks also swap), so that the FP32 operator keeps the exact
  // adjoint structure of the FP64 one.
  {
    const int b0 = 2 * n * n + n, bb0 = b0 + es, d0 = b0 + 2 * es, db0 = b0 + 3 * es;
    const std::vector<double>& xi = c->ref.xi;   // GLL nodes (input of B)
    const std::vector<double>& xq = c->ref.xq;   // quadrature points (output of B, input of Dq)
    auto Af = [&](int t0, int i, int o) -> float& { return tab32[t0 + i * h + o]; };
    auto Cf = [&](int t0, int i, int o) -> float& { return tab32[t0 + h * h + i * h + o]; };
    for (int o = 0; o < h; ++o) {
      // B: constants (sum of the A column and the middle row) and linear functions (C column)
      double sa = 0.0, sc = 0.0, da = 0.0, dc = 0.0;
      for (int i = 0; i < h; ++i) {
        if (!(n % 2 == 0 && i == h - 1)) sa += Af(b0, i, o);
        if (i > 0) sc += Cf(b0, i, o) * xi[i];
        if (i > 0) da += Af(d0, i, o) * xq[i];
        if (!(n % 2 == 0 && i == h - 1)) dc += Cf(d0, i, o);
      }
      if (n % 2) {
        tab32[b0 + 2 * h * h + o] = (float)(1.0 - 2.0 * sa);
        tab32[d0 + 2 * h * h + o] = (float)(-2.0 * dc);
      } else {
        Af(b0, h - 1, o) = (float)(0.5 - sa);
        Cf(d0, h - 1, o) = (float)(-dc);
      }
      Cf(b0, 0, o) = (float)((0.5 * xq[o] - sc) / xi[0]);
      Af(d0, 0, o) = (float)((0.5 - da) / xq[0]);
    }
    if (n % 2) {
      double sm = 0.0, dm = 0.0;
      for (int i = 0; i < h; ++i) sm += tab32[b0 + 2 * h * h + h + i];
      tab32[b0 + 2 * h * h + 2 * h] = (float)(1.0 - 2.0 * sm);
      for (int i = 1; i < h; ++i) dm += tab32[d0 + 2 * h * h + h + i] * xq[i];
      tab32[d0 + 2 * h * h + h] = (float)((0.5 - dm) / xq[0]);
      tab32[d0 + 2 * h * h + 2 * h] = 0.0f;
    }
    for (int i = 0; i < h; ++i)
      for (int o = 0; o < h; ++o) {
        Af(bb0, i, o) = Af(b0, o, i);
        Cf(bb0, i, o) = Cf(b0, o, i);
        Af(db0, i, o) = Cf(d0, o, i);
        Cf(db0, i, o) = Af(d0, o, i);
      }
    if (n % 2) {
      for (int k = 0; k < h; ++k) {
        tab32[bb0 + 2 * h * h + k] = tab32[b0 + 2 * h * h + h + k];
        tab32[bb0 + 2 * h * h + h + k] = tab32[b0 + 2 * h * h + k];
        tab32[db0 + 2 * h * h + k] = tab32[d0 + 2 * h * h + h + k];
        tab32[db0 + 2 * h * h + h + k] = tab32[d0 + 2 * h * h + k];
      }
      tab32[bb0 + 2 * h * h + 2 * h] = tab32[b0 + 2 * h * h + 2 * h];
      tab32[db0 + 2 * h * h + 2 * h] = 0.0f;
    }
  }
  // FP32 kinetic weights per direction, point i on the line and line l:
  // (2/h_d)^2 / 2 * J w_x w_y w_z
  const int n2 = n * n, n3 = n2 * n;
  std::vector<float> kin32(3 * (size_t)n3);
  for (int d = 0; d < 3; ++d) {
    const double sd = 2.0 / c->h[d];
    for (int i = 0; i < n; ++i)
      for (int l = 0; l < n2; ++l) {
        const int a = l % n, b = l / n;      // the other two indices, in the order x, y, z
        const int x = d == 0 ? i : a, y = d == 0 ? a : d == 1 ? i : b, z = d == 2 ? i : b;
        kin32[(size_t)d * n3 + i * n2 + l] =
            (float)(0.5 * sd * sd * c->J * c->ref.wq[x] * c->ref.wq[y] * c->ref.wq[z]);
      }
  }
  c->mf_tab.upload(tab.data(), tab.size(), c->stream);
  c->mf_tab32.upload(tab32.data(), tab32.size(), c->stream);
  c->mf_kin32.upload(kin32.data(), kin32.size(), c->stream);
  CHFSI_HIP(hipStreamSynchronize(c->stream));   // the host tables go out of scope
}

void mf_set_local(chfsi_ctx* c, const double* V, const double* B) {
  if (c->mf_tab.n == 0) mf_prepare(c);
  const int64_t n_points = (int64_t)c->n_cells * c->nq3;
  c->mf_qd.alloc((size_t)n_points * 4);
  c->mf_qd32.alloc((size_t)n_points * 4);
  hipLaunchKernelGGL(mf_qdata_kernel, dim3((unsigned)std::min<int64_t>(cdiv(n_points, 256), 8192)), dim3(256), 0,
                     c->stream, V, B, c->mf_tab.ptr + 2 * c->np1 * c->np1, c->J, c->nq, n_points, reinterpret_cast<double4*>(c->mf_qd.ptr),
                     reinterpret_cast<float4*>(c->mf_qd32.ptr));
  LAUNCH_CHECK();
  CHFSI_HIP(hipStreamSynchronize(c->stream));
  c->mf_gen = c->gen;
}

void launch_mf_products(chfsi_ctx* c, const KPoint& kp, int prec, const double2* X, int64_t ldx, double2* W,
                        int64_t ldw, int n_vec, double alpha, const double* alpha_d, void* ye) {
  const bool fp64 = prec != CHFSI_PREC_MIXED;
  switch (c->np1) {
    case 2: launch_mf_np<2>(c, kp, fp64, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye); break;
    case 3: launch_mf_np<3>(c, kp, fp64, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye); break;
    case 4: launch_mf_np<4>(c, kp, fp64, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye); break;
    case 5: launch_mf_np<5>(c, kp, fp64, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye); break;
    case 6: launch_mf_np<6>(c, kp, fp64, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye); break;
    case 7: launch_mf_np<7>(c, kp, fp64, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye); break;
    case 8: launch_mf_np<8>(c, kp, fp64, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye); break;
    case 9: launch_mf_np<9>(c, kp, fp64, X, ldx, W, ldw, n_vec, alpha, alpha_d, ye); break;
    default: throw Error{CHFSI_EINVAL, "matrix-free apply: unsupported p"};
  }
}

}  // namespace chfsi
