// Cell-level operator: setup of the Pauli-form cell matrices and the fused
// gather / MFMA cell product / scatter-add kernels (Sec. IV.B, the
// cell-level dense products of the FE matrix-multivector product), per
// colour for one operator, for all its cells with the products written out, or as a
// persistent grid over a batch.
//
// Cell operator storage ("Pauli form"): the spinor cell matrix of
// eqn:FEHlocEl with the k-terms of eqn:FEHloc is, with every term scaled by
// M_D^{-1/2} on both sides,
//   [[A + Bz + iS, Bx - iBy], [Bx + iBy, A - Bz + iS]]
// with A = kinetic + |k|^2/2 mass + V-weighted mass and B_d the B_d-weighted
// masses (real symmetric) and S the skew-symmetrised k-gradient term (real
// antisymmetric, zero at Gamma).  Each cell stores the real matrices
// Pu = A + Bz - Bx - By, Pd = A - Bz - Bx - By, Bx, By (and S when k != 0)
// instead of the complex
// 2n x 2n matrix: half the bytes, and 8 instead of 16 real MFMAs per complex
// multiply-add block at Gamma (the sum of four rank-one spin terms below).
// Matrices are stored pre-tiled in MFMA A-operand order: [cell][row block of
// 16][k-step of 4], each tile [64 lanes][Pu, Pd, Bx, By] (one 16- or two 16-byte
// loads per lane) and then [64 lanes] of S.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"
#include "mfma.h"

namespace chfsi {

// ============================================================================
// Cell operator setup
// ============================================================================
// One block per (cell, row block of 16).  Weighted masses by quadrature,
//   M_f[i][j] = sum_q w_q J f(r_q) N_i(r_q) N_j(r_q),  N_i = l_ax l_ay l_az,
// for f in {V, Bx, By, Bz}; then the scaled Pauli-form matrices, in FP64 and FP32.
// The sums are factorised over the directions and shared by the rows of the block:
//   G[bz][qx, qy]      = sum_qz l_az l_bz f     once per az of the block
//   H[by, bz][qx]      = sum_qy l_ay l_by G     once per pair (ay, az), at most `group`
//                                               pairs at a time (what LDS holds)
//   M[i][j]            = sum_qx l_ax l_bx H     one entry per thread, rows fastest
// about 0.2 M multiply-adds per block of n_p = 7 where point by point they are 7.5 M,
// and the entries are written in the tiles' order, 32 bytes a lane side by side (one
// thread per column wrote every lane to a line of its own: 1.12 ms).  512 cells,
// p = 5, one k-point: 2.43 ms and 0.25 ms for the FP32 copy before, 0.34 ms for both.
__global__ __launch_bounds__(256) void cell_setup_kernel(
    const double* __restrict__ V, const double* __restrict__ B, const double* __restrict__ U0,
    const double* __restrict__ Sk, const double* __restrict__ minv_sqrt,
    const int32_t* __restrict__ cell_nodes, const double* __restrict__ B1,
    const double* __restrict__ wq1, double J, int np1, int nq, int nloc, int nrb, int nkb, int nmat,
    int group, double* __restrict__ out, float* __restrict__ out32) {
  extern __shared__ double smem[];
  const int nq2 = nq * nq, nq3 = nq2 * nq, np2 = np1 * np1;
  double4* sW = reinterpret_cast<double4*>(smem);   // [nq3] weighted (V, Bx, By, Bz)
  double4* sG = sW + nq3;                           // [np1][nq2]
  double4* sH = sG + (size_t)np1 * nq2;             // [group][np2][nq]
  double* sB1 = reinterpret_cast<double*>(sH + (size_t)group * np2 * nq);   // [np1][nq]
  double* sS = sB1 + np1 * nq;                      // [nloc] M^{-1/2} at the cell's nodes
  const int e = blockIdx.x, rb = blockIdx.y, tid = threadIdx.x;
  for (int q = tid; q < nq3; q += 256) {
    const int qx = q % nq, qy = (q / nq) % nq, qz = q / nq2;
    const double wJ = wq1[qx] * wq1[qy] * wq1[qz] * J;
    const size_t p = (size_t)e * nq3 + q;
    sW[q] = double4{wJ * V[p], wJ * B[3 * p], wJ * B[3 * p + 1], wJ * B[3 * p + 2]};
  }
  for (int t = tid; t < np1 * nq; t += 256) sB1[t] = B1[t];
  for (int a = tid; a < nloc; a += 256) sS[a] = minv_sqrt[cell_nodes[(size_t)e * nloc + a]];
  const int i_begin = rb * 16, i_last = min(i_begin + 16, nloc) - 1, npad = nkb * 4;
  const size_t base = ((size_t)e * nrb + rb) * nkb * nmat * 64;
  const auto acc4 = [](double4& s, double w, const double4& v) {
    s.x = fma(w, v.x, s.x);
    s.y = fma(w, v.y, s.y);
    s.z = fma(w, v.z, s.z);
    s.w = fma(w, v.w, s.w);
  };
  const int pair_end = i_last / np1 + 1;            // pairs ay + np1 az of the block's rows
  int az_g = -1;                                    // az of sG
  for (int p0 = i_begin / np1; p0 < pair_end; p0 += group) {
    const int p1 = min(p0 + group, pair_end);
    for (int p = p0; p < p1; ++p) {
      const int ay = p % np1, az = p / np1;
      __syncthreads();                    // the tables are filled; sG and sH are read
      if (az != az_g) {
        for (int t = tid; t < np1 * nq2; t += 256) {
          const int bz = t / nq2, qxy = t - bz * nq2;
          double4 s = {0.0, 0.0, 0.0, 0.0};
          for (int qz = 0; qz < nq; ++qz) acc4(s, sB1[az * nq + qz] * sB1[bz * nq + qz], sW[qxy + nq2 * qz]);
          sG[t] = s;
        }
        az_g = az;
        __syncthreads();
      }
      double4* h = sH + (size_t)(p - p0) * np2 * nq;
      for (int t = tid; t < np2 * nq; t += 256) {
        const int bzy = t / nq, qx = t - bzy * nq, by = bzy % np1, bz = bzy / np1;
        double4 s = {0.0, 0.0, 0.0, 0.0};
        for (int qy = 0; qy < nq; ++qy)
          acc4(s, sB1[ay * nq + qy] * sB1[by * nq + qy], sG[bz * nq2 + nq * qy + qx]);
        h[t] = s;
      }
    }
    __syncthreads();
    for (int t = tid; t < 16 * npad; t += 256) {
      const int j = t >> 4, i = i_begin + (t & 15), pi = i / np1;
      const bool valid = i < nloc && j < nloc;
      if (valid ? pi < p0 || pi >= p1 : p0 != i_begin / np1) continue;   // (padding: with the first group)
      double4 m = {0.0, 0.0, 0.0, 0.0};
      double sk = 0.0;
      if (valid) {
        const int ax = i - pi * np1, bzy = j / np1, bx = j - bzy * np1;
        const double4* h = sH + ((size_t)(pi - p0) * np2 + bzy) * nq;
        for (int qx = 0; qx < nq; ++qx) acc4(m, sB1[ax * nq + qx] * sB1[bx * nq + qx], h[qx]);
        const double s = sS[i] * sS[j];
        const double a0 = U0[(size_t)i * nloc + j] + m.x;
        m = double4{s * (a0 + m.w - m.y - m.z), s * (a0 - m.w - m.y - m.z), s * m.y, s * m.z};
        if (nmat > 4) sk = s * Sk[(size_t)i * nloc + j];
      }
      const int lane = t & 63;
      const size_t o = base + (size_t)(t >> 6) * nmat * 64;
      *reinterpret_cast<double4*>(out + o + lane * 4) = m;
      *reinterpret_cast<float4*>(out32 + o + lane * 4) = float4{(float)m.x, (float)m.y, (float)m.z, (float)m.w};
      if (nmat > 4) {
        out[o + 256 + lane] = sk;
        out32[o + 256 + lane] = (float)sk;
      }
    }
  }
}

// Cell operators of one k-point from the fields; U0 and S of the k-point are in kp.
void launch_cell_setup(chfsi_ctx* c, KPoint& kp, const double* V, const double* B) {
  const size_t per_cell = (size_t)c->nrb * c->nkb * kp.nmat * 64;
  kp.cell64.alloc(per_cell * c->n_cells);
  kp.cell32.alloc(per_cell * c->n_cells);
  if (c->ref_b1.n == 0) {
    c->ref_b1.upload(c->ref.B.data(), c->ref.B.size(), c->stream);
    c->ref_wq.upload(c->ref.wq.data(), c->ref.wq.size(), c->stream);
  }
  const int np1 = c->np1, nq = c->nq;
  // pairs (ay, az) of a block at a time: all (16 rows cross at most 15 / n_p + 2), or as
  // many as 128 KB of LDS hold (one always fits, at n_p = 9 and n_q = 12)
  const size_t fixed = (size_t)(c->nq3 + np1 * nq * nq) * sizeof(double4) +
                       (size_t)(np1 * nq + c->nloc) * sizeof(double);
  const size_t per = (size_t)np1 * np1 * nq * sizeof(double4);
  const size_t fit = fixed < 128 * 1024 ? (128 * 1024 - fixed) / per : 0;
  const int group = (int)std::max<size_t>(1, std::min<size_t>(15 / np1 + 2, fit));
  const size_t sh = fixed + group * per;
  dim3 grid(c->n_cells, c->nrb);
  hipLaunchKernelGGL(cell_setup_kernel, grid, dim3(256), sh, c->stream, V, B, kp.U0.ptr, kp.S.ptr, c->minv_sqrt.ptr,
                     c->cell_nodes.ptr, c->ref_b1.ptr, c->ref_wq.ptr, c->J, np1, nq, c->nloc, c->nrb, c->nkb,
                     kp.nmat, group, kp.cell64.ptr, kp.cell32.ptr);
  LAUNCH_CHECK();
}

// ============================================================================
// Fused gather / cell product / scatter-add, one launch per colour (or all cells)
// ============================================================================
// Block = 2 (row blocks) x WC (column groups) waves of 16 rows x 16*CB columns:
// block tile 32 local rows x BN = 16*CB*WC columns of one cell.  K loop over
// the cell's local nodes in stages of 8 nodes: the gathered spinor rows (u, d) =
// (X_up, X_dn) are staged in LDS as complex pairs, double-buffered, with the
// next stage's global loads issued before the current stage's MFMAs.  Each wave
// reads its A fragments straight from the pre-tiled cell operator.  The spin
// structure is a sum of four rank-one terms,
//   A + B.sigma = Pu |up><up| + Pd |dn><dn| + Bx |1,1><1,1| + By |1,i><1,i|
//   Pu = A + Bz - Bx - By,  Pd = A - Bz - Bx - By,
// so that per 4-node k-step and 16-column block 8 real products do
//   yu = Pu u,  yd = Pd d,  tx = Bx (u + d),  ty = By (u - i d)     (+ S: 4 more)
//   Y_up = yu + tx + ty,    Y_dn = yd + tx + i ty
// instead of the 12 of the products entry by entry.  The MFMAs bound the kernel
// (matrix units 74 % busy, 64 % of the wave cycles wait for issue), so the four extra
// accumulators and the additions on the fragments are paid for.  FP64 filter of 128 columns on 8^3
// cells, p = 6, degree 24: 97.2 -> 74.0 ms; with FP32 products and the k-term, 200
// columns on 10^3 cells, p = 5, degree 16: 80.5 -> 68.7 ms.
template <class T> struct CellC2;
template <> struct CellC2<double> { typedef double2 type; };
template <> struct CellC2<float> { typedef float2 type; };

// Shape of a tile of 32 TW columns (TW = 1, 2, 4): column groups of waves and
// 16-column blocks per wave.  FP64: one block per wave up to 64 columns (eight
// waves, 128 VGPRs, 16 waves per CU; two blocks per wave leave 8 per CU and run
// 4 % slower); FP32: two (its accumulators are half as wide, 4 % faster than one).
template <class T, int TW> constexpr int cell_wc() { return sizeof(T) == 8 ? (TW == 1 ? 2 : 4) : (TW == 4 ? 4 : 2); }
template <class T, int TW> constexpr int cell_cb() { return 2 * TW / cell_wc<T, TW>(); }
template <class T, int TW> constexpr int cell_threads() { return 128 * cell_wc<T, TW>(); }
// waves per SIMD that the registers are limited for
template <class T, int TW> constexpr int cell_min_waves() { return sizeof(T) == 8 && cell_cb<T, TW>() > 1 ? 2 : 4; }

template <class T, int TW>
struct CellSmem {
  static constexpr int BN = 32 * TW;
  static constexpr int BK = 8;
  static constexpr int PAD = 2;
  typename CellC2<T>::type sB[2][2][BK][BN + PAD];      // [buffer][spin][node][column]
  int32_t sNode[(kMaxP + 1) * (kMaxP + 1) * (kMaxP + 1)];
};

// One block tile of the fused gather / cell product / scatter-add for cell e,
// row tile rt (two 16-row blocks) and column tile ct.  Starts and ends with
// the block synchronised, so it can be called repeatedly by a persistent block.
template <class T, int TW, bool HAS_S>
__device__ __forceinline__ void cell_tile(CellSmem<T, TW>& sm, const T* __restrict__ cm,
                                          const int32_t* __restrict__ cell_nodes, int e, int rt, int ct,
                                          int nloc, int nrb, int nkb, int nmat,
                                          const double2* __restrict__ X, int64_t ldx,
                                          double2* __restrict__ W, int64_t ldw, int n_vec, double alpha,
                                          typename CellC2<T>::type* __restrict__ ye) {
  typedef typename Vec4<T>::type V4;
  typedef typename CellC2<T>::type C2;
  constexpr int CB = cell_cb<T, TW>();
  constexpr int NT = cell_threads<T, TW>();
  constexpr int BN = 32 * TW;
  constexpr int BK = 8;
  constexpr int NPRE = (BK * 2 * BN) / NT;
  auto& sB = sm.sB;
  auto& sNode = sm.sNode;
  __syncthreads();                        // previous tile's LDS reads are done

  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int wr = wave & 1, wc = wave >> 1;
  const int rb = rt * 2 + wr;
  const bool row_active = rb < nrb;
  // an inactive row block (odd nrb) computes on the last valid block and skips the epilogue,
  // so the stage loop below has no branches and loads overlap the MFMAs
  const int rb_eff = row_active ? rb : nrb - 1;
  const int col0 = ct * BN;
  // waves past the last column only stage and wait (a block of 130 columns costs 144, not 192)
  const bool cols_active = col0 + wc * (CB * 16) < n_vec;

  for (int i = tid; i < nloc; i += NT) sNode[i] = cell_nodes[(size_t)e * nloc + i];
  __syncthreads();

  V4 acc[CB][8];                          // yu, yd, tx, ty: real and imaginary parts
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[cb][k] = V4{0, 0, 0, 0};

  const T* Abase = cm + ((size_t)(e * nrb + rb_eff) * nkb) * nmat * 64;
  const int nstage = nkb / 2;
  double2 pre[NPRE];
  V4 aC[2], aN[2];                        // Pu, Pd, Bx, By of the stage's two k-steps
  T sC[2], sN[2];

  // per-thread constants of the gather: (k node, spin, column) of each prefetch slot
  int g_kk[NPRE], g_sp[NPRE], g_col[NPRE];
  bool g_cv[NPRE];
#pragma unroll
  for (int j = 0; j < NPRE; ++j) {
    const int idx = tid + NT * j;
    g_col[j] = idx % BN;
    g_sp[j] = (idx / BN) & 1;
    g_kk[j] = idx / (2 * BN);
    g_cv[j] = col0 + g_col[j] < n_vec;
  }
  const int gcol_max = n_vec - 1;

  auto gload = [&](int s) {
#pragma unroll
    for (int j = 0; j < NPRE; ++j) {
      const int knode = s * BK + g_kk[j];
      const bool valid = g_cv[j] && knode < nloc;
      const int kn = knode < nloc ? knode : 0;                    // in-bounds address always
      const int gcol = min(col0 + g_col[j], gcol_max);
      const double2 v = X[(2 * (int64_t)sNode[kn] + g_sp[j]) * ldx + gcol];
      pre[j] = valid ? v : double2{0.0, 0.0};
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int j = 0; j < NPRE; ++j) sB[buf][g_sp[j]][g_kk[j]][g_col[j]] = C2{(T)pre[j].x, (T)pre[j].y};
  };
  // tile of one k-step: [64 lanes][Pu, Pd, Bx, By], then [64 lanes] of S
  auto aload = [&](int s, V4 (&dst)[2], T (&ds)[2]) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const T* Ap = Abase + (size_t)(s * 2 + kk) * nmat * 64;
      dst[kk] = *reinterpret_cast<const V4*>(Ap + lane * 4);
      ds[kk] = HAS_S ? Ap[256 + lane] : (T)0;
    }
  };

  gload(0);
  lstore(0);
  if (!cols_active) {
    __syncthreads();
    for (int s = 0; s < nstage; ++s) {
      gload(s + 1 < nstage ? s + 1 : s);
      lstore((s & 1) ^ 1);
      __syncthreads();
    }
    return;                               // (no barrier follows inside the tile)
  }
  aload(0, aC, sC);
  __syncthreads();
  for (int s = 0; s < nstage; ++s) {
    const int buf = s & 1;
    const int sn = s + 1 < nstage ? s + 1 : s;      // the last stage reloads itself (unused)
    gload(sn);
    aload(sn, aN, sN);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const T pu = aC[kk][0], pd = aC[kk][1], bx = aC[kk][2], by = aC[kk][3];
      const T sv = sC[kk], nsv = -sC[kk];
      const int krow = kk * 4 + (lane >> 4);
      C2 u[CB], d[CB];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const int col = wc * (CB * 16) + cb * 16 + (lane & 15);
        u[cb] = sB[buf][0][krow][col];
        d[cb] = sB[buf][1][krow][col];
      }
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        acc[cb][0] = mfma(pu, u[cb].x, acc[cb][0]);
        acc[cb][1] = mfma(pu, u[cb].y, acc[cb][1]);
        acc[cb][2] = mfma(pd, d[cb].x, acc[cb][2]);
        acc[cb][3] = mfma(pd, d[cb].y, acc[cb][3]);
      }
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        acc[cb][4] = mfma(bx, u[cb].x + d[cb].x, acc[cb][4]);
        acc[cb][5] = mfma(bx, u[cb].y + d[cb].y, acc[cb][5]);
        acc[cb][6] = mfma(by, u[cb].x + d[cb].y, acc[cb][6]);
        acc[cb][7] = mfma(by, u[cb].y - d[cb].x, acc[cb][7]);
      }
      if (HAS_S) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          acc[cb][0] = mfma(nsv, u[cb].y, acc[cb][0]);
          acc[cb][1] = mfma(sv, u[cb].x, acc[cb][1]);
          acc[cb][2] = mfma(nsv, d[cb].y, acc[cb][2]);
          acc[cb][3] = mfma(sv, d[cb].x, acc[cb][3]);
        }
      }
    }
    lstore(buf ^ 1);       // the other buffer was last read before the previous barrier
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      aC[kk] = aN[kk];
      sC[kk] = sN[kk];
    }
  }

  if (!row_active) return;                // (no barrier follows inside the tile)
  // epilogue: lane holds rows acc_row(lane, j), column lane%16 of each 16x16 tile
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int rl = rb * 16 + acc_row<T>(lane, j);
    if (rl >= nloc) continue;
    const int64_t node = sNode[rl];
    double2* w0 = W + (2 * node) * ldw;
    double2* w1 = W + (2 * node + 1) * ldw;
    C2* ye0 = ye + ((size_t)e * nloc + rl) * 2 * n_vec;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const int gcol = col0 + wc * (CB * 16) + cb * 16 + (lane & 15);
      if (gcol >= n_vec) continue;
      const T tx = acc[cb][4][j], ti = acc[cb][5][j], yx = acc[cb][6][j], yi = acc[cb][7][j];
      const C2 y0 = {acc[cb][0][j] + (tx + yx), acc[cb][1][j] + (ti + yi)};
      const C2 y1 = {acc[cb][2][j] + (tx - yi), acc[cb][3][j] + (ti + yx)};
      if (ye) {
        ye0[gcol] = y0;
        ye0[n_vec + gcol] = y1;
        continue;
      }
      double2 o0 = w0[gcol], o1 = w1[gcol];
      o0.x = fma(alpha, (double)y0.x, o0.x);
      o0.y = fma(alpha, (double)y0.y, o0.y);
      o1.x = fma(alpha, (double)y1.x, o1.x);
      o1.y = fma(alpha, (double)y1.y, o1.y);
      w0[gcol] = o0;
      w1[gcol] = o1;
    }
  }
}

template <class T, int TW, bool HAS_S>
__global__ __launch_bounds__((cell_threads<T, TW>()), (cell_min_waves<T, TW>())) void cell_apply_kernel(
    const T* __restrict__ cm, const int32_t* __restrict__ cell_nodes,
    const int32_t* __restrict__ cells, int nloc, int nrb, int nkb, int nmat, int n_rowtiles,
    int n_coltiles, int n_work, const double2* __restrict__ X, int64_t ldx, double2* __restrict__ W,
    int64_t ldw, int n_vec, double alpha, typename CellC2<T>::type* __restrict__ ye) {
  __shared__ CellSmem<T, TW> sm;
  // Workgroups are dispatched round-robin over the 8 XCDs; remap so that each
  // XCD gets a contiguous range of (cell, row tile, column tile) work and the
  // row tiles of one cell share that XCD's L2 for the gathered rows.
  const int per_xcd = (n_work + 7) / 8;
  const int bid = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if (bid >= n_work) return;              // uniform over the block, before any barrier
  const int ct = bid % n_coltiles;
  const int rt = (bid / n_coltiles) % n_rowtiles;
  const int ci = bid / (n_coltiles * n_rowtiles);
  cell_tile<T, TW, HAS_S>(sm, cm, cell_nodes, cells ? cells[ci] : ci, rt, ct, nloc, nrb, nkb, nmat, X, ldx, W, ldw,
                          n_vec, alpha, ye);
}

// Batched form: one persistent grid walks a static list of (task, cell, row
// tile, column tile) items across many independent operators (k-points, systems):
// those of one colour phase, or all cells of small tasks (into their ye).  Items were
// ordered on the host so that item i runs on XCD i % 8 and the row tiles of a cell
// share an XCD.
template <class T, int TW, bool HAS_S>
__global__ __launch_bounds__((cell_threads<T, TW>()), (cell_min_waves<T, TW>())) void cell_batch_kernel(const BatchTaskArgs tasks,
                                                         const int4* __restrict__ items, int n_items,
                                                         const double* __restrict__ alpha, int src) {
  __shared__ CellSmem<T, TW> sm;
  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    const int4 w = items[it];
    if (w.x < 0) continue;                // padding item (uniform over the block)
    const BatchTaskDev& t = tasks.t[w.x];
    const T* cm = sizeof(T) == 8 ? (const T*)t.cm64 : (const T*)t.cm32;
    cell_tile<T, TW, HAS_S>(sm, cm, t.cell_nodes, w.y, w.z, w.w, t.nloc, t.nrb, t.nkb, t.nmat, t.buf[src],
                            t.ld[src], t.buf[src ^ 1], t.ld[src ^ 1], t.n_vec, alpha[w.x],
                            (typename CellC2<T>::type*)t.ye);
  }
}

template <class T, int TW, bool HAS_S>
static void launch_cells(chfsi_ctx* c, const T* cm, int nmat, const double2* X, int64_t ldx,
                         double2* W, int64_t ldw, int n_vec, double alpha, void* ye = nullptr) {
  const int BN = 32 * TW;
  const int n_rowtiles = cdiv(c->nrb, 2);
  const int n_coltiles = cdiv(n_vec, BN);
  for (int k = 0; k < (ye ? 1 : c->n_colours); ++k) {
    const int n_in = ye ? c->n_cells : c->colour_off[k + 1] - c->colour_off[k];
    if (n_in == 0) continue;
    const int nblk = n_in * n_rowtiles * n_coltiles;
    const double n2 = 2.0 * c->nloc;
    const double flops = 8.0 * n2 * n2 * n_vec * n_in;
    // issued MFMA flops: per cell nrb row blocks x the 16-column blocks of the waves that
    // have a column, each nkb k-steps of (8 | 12) MFMAs of 16x16x4 (2048 flops)
    const int col_blocks = cdiv(n_vec, 16 * cell_cb<T, TW>()) * cell_cb<T, TW>();
    const double exec = (double)n_in * c->nrb * col_blocks * c->nkb * (HAS_S ? 12 : 8) * 2048.0;
    const double bytes = (double)n_in * ((double)nmat * c->nloc * c->nloc * sizeof(T) +
                                         3.0 * c->nloc * 2.0 * n_vec * sizeof(double2));
    StageTimer tm(c, sizeof(T) == 8 ? CHFSI_STAGE_CELL_FP64 : CHFSI_STAGE_CELL_FP32, flops, exec, bytes);
    const int grid = 8 * ((nblk + 7) / 8);
    hipLaunchKernelGGL((cell_apply_kernel<T, TW, HAS_S>), dim3(grid), dim3((cell_threads<T, TW>())), 0, c->stream, cm,
                       c->cell_nodes.ptr, ye ? nullptr : c->colour_cells.ptr + c->colour_off[k], c->nloc, c->nrb,
                       c->nkb, nmat, n_rowtiles, n_coltiles, nblk, X, ldx, W, ldw, n_vec, alpha,
                       (typename CellC2<T>::type*)ye);
    LAUNCH_CHECK();
  }
}

// 64-column tiles for every block wider than 32: at p = 5..6 they run 1-4 %
// faster than 128-column tiles in both precisions (four workgroups per CU
// instead of one hide the epilogue and barrier latencies; the two column tiles
// of a cell read its operator through the same L2).  The per-column arithmetic
// does not depend on the tile width, so results are bitwise the same.
static int cell_tile_width(int n_vec) { return n_vec > 32 ? 2 : 1; }

int64_t cell_items_per_cell(const chfsi_ctx* c, int n_vec) {
  return (int64_t)cdiv(c->nrb, 2) * cdiv(n_vec, 32 * cell_tile_width(n_vec));
}

template <class T, bool HAS_S>
static void launch_cells_cb(chfsi_ctx* c, const T* cm, int nmat, const double2* X, int64_t ldx,
                            double2* W, int64_t ldw, int n_vec, double alpha, void* ye) {
  if (cell_tile_width(n_vec) == 2)
    launch_cells<T, 2, HAS_S>(c, cm, nmat, X, ldx, W, ldw, n_vec, alpha, ye);
  else
    launch_cells<T, 1, HAS_S>(c, cm, nmat, X, ldx, W, ldw, n_vec, alpha, ye);
}

// Local (cell) part of H_hat: W += alpha * sum_e R_e^T H_e R_e X colour by colour,
// or the products of all cells to ye.
void launch_cell_products(chfsi_ctx* c, KPoint& kp, int prec, const double2* X, int64_t ldx, double2* W,
                          int64_t ldw, int n_vec, double alpha, void* ye) {
  if (prec == CHFSI_PREC_MIXED) {
    if (kp.gamma) launch_cells_cb<float, false>(c, kp.cell32.ptr, kp.nmat, X, ldx, W, ldw, n_vec, alpha, ye);
    else launch_cells_cb<float, true>(c, kp.cell32.ptr, kp.nmat, X, ldx, W, ldw, n_vec, alpha, ye);
  } else {
    if (kp.gamma) launch_cells_cb<double, false>(c, kp.cell64.ptr, kp.nmat, X, ldx, W, ldw, n_vec, alpha, ye);
    else launch_cells_cb<double, true>(c, kp.cell64.ptr, kp.nmat, X, ldx, W, ldw, n_vec, alpha, ye);
  }
}

// ---------------------------------------------------------------- batched form
template <class T, int TW, bool HAS_S>
static void launch_batch_t(hipStream_t s, const BatchTaskArgs& tasks, const int4* items, int n_items,
                           const double* alpha, int src, int grid) {
  hipLaunchKernelGGL((cell_batch_kernel<T, TW, HAS_S>), dim3(grid), dim3((cell_threads<T, TW>())), 0, s, tasks, items, n_items, alpha,
                     src);
  LAUNCH_CHECK();
}

template <class T, bool HAS_S>
static void launch_batch_cb(hipStream_t s, int CB, const BatchTaskArgs& tasks, const int4* items, int n_items,
                            const double* alpha, int src, int grid) {
  if (CB == 4)
    launch_batch_t<T, 4, HAS_S>(s, tasks, items, n_items, alpha, src, grid);
  else if (CB == 2)
    launch_batch_t<T, 2, HAS_S>(s, tasks, items, n_items, alpha, src, grid);
  else
    launch_batch_t<T, 1, HAS_S>(s, tasks, items, n_items, alpha, src, grid);
}

void launch_cell_batch(hipStream_t s, bool fp64, int CB, bool has_s, const BatchTaskArgs& tasks, const int4* items,
                       int n_items, const double* alpha, int src, int grid) {
  if (fp64) {
    if (has_s) launch_batch_cb<double, true>(s, CB, tasks, items, n_items, alpha, src, grid);
    else launch_batch_cb<double, false>(s, CB, tasks, items, n_items, alpha, src, grid);
  } else {
    if (has_s) launch_batch_cb<float, true>(s, CB, tasks, items, n_items, alpha, src, grid);
    else launch_batch_cb<float, false>(s, CB, tasks, items, n_items, alpha, src, grid);
  }
}

template <class T, int TW, bool HAS_S>
static int occ_t() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, cell_batch_kernel<T, TW, HAS_S>, (cell_threads<T, TW>()), 0) != hipSuccess) n = 1;
  return std::max(1, n);
}

int cell_batch_blocks_per_cu(bool fp64, int CB, bool has_s) {
  if (fp64) {
    if (has_s) return CB == 4 ? occ_t<double, 4, true>() : CB == 2 ? occ_t<double, 2, true>() : occ_t<double, 1, true>();
    return CB == 4 ? occ_t<double, 4, false>() : CB == 2 ? occ_t<double, 2, false>() : occ_t<double, 1, false>();
  }
  if (has_s) return CB == 4 ? occ_t<float, 4, true>() : CB == 2 ? occ_t<float, 2, true>() : occ_t<float, 1, true>();
  return CB == 4 ? occ_t<float, 4, false>() : CB == 2 ? occ_t<float, 2, false>() : occ_t<float, 1, false>();
}

template <class T, bool HAS_S>
static void cells_with_cb(chfsi_ctx* c, int CB, const T* cm, int nmat, const double2* X, int64_t ldx, double2* W,
                          int64_t ldw, int n_vec) {
  if (CB == 4) launch_cells<T, 4, HAS_S>(c, cm, nmat, X, ldx, W, ldw, n_vec, 1.0);
  else if (CB == 2) launch_cells<T, 2, HAS_S>(c, cm, nmat, X, ldx, W, ldw, n_vec, 1.0);
  else launch_cells<T, 1, HAS_S>(c, cm, nmat, X, ldx, W, ldw, n_vec, 1.0);
}

// Mean time (ms) of the cell stage of one apply with column tiles of 32*CB.
double time_cell_stage(chfsi_ctx* c, KPoint& kp, int CB, int prec, const double2* X, int64_t ldx, double2* W,
                       int64_t ldw, int n_vec, int reps) {
  const bool was = c->stats_on;
  c->stats_on = false;
  hipEvent_t e0, e1;
  CHFSI_HIP(hipEventCreate(&e0));
  CHFSI_HIP(hipEventCreate(&e1));
  auto run = [&]() {
    if (prec == CHFSI_PREC_MIXED) {
      if (kp.gamma) cells_with_cb<float, false>(c, CB, kp.cell32.ptr, kp.nmat, X, ldx, W, ldw, n_vec);
      else cells_with_cb<float, true>(c, CB, kp.cell32.ptr, kp.nmat, X, ldx, W, ldw, n_vec);
    } else {
      if (kp.gamma) cells_with_cb<double, false>(c, CB, kp.cell64.ptr, kp.nmat, X, ldx, W, ldw, n_vec);
      else cells_with_cb<double, true>(c, CB, kp.cell64.ptr, kp.nmat, X, ldx, W, ldw, n_vec);
    }
  };
  run();                                   // warm
  CHFSI_HIP(hipEventRecord(e0, c->stream));
  for (int r = 0; r < reps; ++r) run();
  CHFSI_HIP(hipEventRecord(e1, c->stream));
  CHFSI_HIP(hipEventSynchronize(e1));
  float ms = 0.f;
  CHFSI_HIP(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  c->stats_on = was;
  return ms / reps;
}

}  // namespace chfsi
