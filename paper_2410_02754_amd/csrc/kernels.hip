// Device kernels and their launchers for gfx950 (CDNA4, wave64).
//
// Operator action (Sec. IV.B, "FE discretized matrix multivector product"):
// extraction X_e = R_e X, cell products H_e X_e, nonlocal projector terms,
// assembly Y = sum_e R_e^T Y_e.  The four steps run as
//   1. the projector contraction C_a = P_a^H X and the coupling C'_a = Delta_a C_a
//      (eqn:FEHnloc),
//   2. an initialisation pass over the nodes: the recurrence terms (beta W + gamma X)
//      and the back-product P_a C'_a,
//   3. one launch per cell colour of the fused gather / cell product / scatter-add
//      kernel; cells of one colour share no node, so the read-add-write of the
//      epilogue needs no atomics and the result is bitwise reproducible.
// Small applies run step 3 first, for all cells in one launch that writes the cells'
// products (ye), and step 2 adds those of each node in the colour order
// (products_scratch_bytes).
//
// The cell products live in cell.hip and matfree.hip; this file holds the
// element-wise, nonlocal, adjoint and dense-block kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.h"
#include "mfma.h"
#include "sumfact.h"

namespace chfsi {

// ============================================================================
// Element-wise passes
// ============================================================================
__global__ void axpby_rows_kernel(double2* __restrict__ W, int64_t ldw, const double2* __restrict__ X,
                                  int64_t ldx, int64_t rows, int n_vec, double beta, double gamma) {
  const int64_t total = rows * n_vec;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / n_vec;
    const int n = (int)(t - r * n_vec);
    double2 w = {0.0, 0.0};
    if (beta != 0.0) {
      w = W[r * ldw + n];
      w.x *= beta;
      w.y *= beta;
    }
    if (gamma != 0.0) {
      const double2 x = X[r * ldx + n];
      w.x += gamma * x.x;
      w.y += gamma * x.y;
    }
    W[r * ldw + n] = w;
  }
}

void launch_axpby_rows(chfsi_ctx* c, double2* W, int64_t ldw, const double2* X, int64_t ldx,
                       int64_t rows, int n_vec, double beta, double gamma) {
  const int64_t total = rows * n_vec;
  StageTimer tm(c, CHFSI_STAGE_AXPY, 0.0, 0.0,
                (double)total * sizeof(double2) * (1.0 + (beta != 0.0) + (gamma != 0.0)));
  const int blocks = (int)std::min<int64_t>(cdiv(total, 256), 8192);
  hipLaunchKernelGGL(axpby_rows_kernel, dim3(std::max(blocks, 1)), dim3(256), 0, c->stream, W, ldw, X,
                     ldx, rows, n_vec, beta, gamma);
  LAUNCH_CHECK();
}

__global__ void copy_rows_kernel(double2* __restrict__ D, int64_t ldd, const double2* __restrict__ S,
                                 int64_t lds, int64_t rows, int n_vec) {
  const int64_t total = rows * n_vec;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / n_vec;
    const int n = (int)(t - r * n_vec);
    D[r * ldd + n] = S[r * lds + n];
  }
}

void launch_copy_rows(chfsi_ctx* c, double2* dst, int64_t ldd, const double2* src, int64_t lds,
                      int64_t rows, int n_vec) {
  const int64_t total = rows * n_vec;
  const int blocks = (int)std::min<int64_t>(cdiv(total, 256), 8192);
  hipLaunchKernelGGL(copy_rows_kernel, dim3(std::max(blocks, 1)), dim3(256), 0, c->stream, dst, ldd, src,
                     lds, rows, n_vec);
  LAUNCH_CHECK();
}

// ============================================================================
// Nonlocal projector terms (eqn:FEHnloc in the cell form of Sec. IV.B)
// ============================================================================
template <class T> struct C2;
template <> struct C2<double> { typedef double2 type; };
template <> struct C2<float> { typedef float2 type; };

constexpr int kMaxPj = 9;

// 16-column blocks per wave of the contraction and initialisation kernels: one
// in FP64 (fewer registers, more resident waves to cover the row loads), two in FP32.
template <class T>
constexpr int nl_col_blocks() { return sizeof(T) == 8 ? 1 : 2; }

// Contraction partials, one wave per (chunk of an atom's support, 16- or
// 32-column tile): partial[chunk][2 chi + s][n] = sum_j conj(P[j][chi]) X[2 node_j + s][n].
// Done as 16x16x4 MFMAs: row = projector index chi (n_pj <= 9 of the 16 rows
// used), k = four support entries per step, column = 16 of the tile's columns;
// sixteen entries' operands are loaded before their MFMAs are issued.
// REALP: the projector values are real (Gamma point), two real MFMAs per step.
// PACK (complex values, n_pj <= 8): rows 0-7 carry the real parts and rows
// 8-15 the imaginary parts of the projectors, so one MFMA against Re x and one
// against Im x replace the four of the plain complex step, and
//   Re c = (p_r x_r)[chi] + (p_i x_i)[chi + 8],  Im c = (p_r x_i)[chi] - (p_i x_r)[chi + 8];
// row chi + 8 is accumulator register j + 2 of the same lane (FP64) or register
// j of the lane 32 above (FP32).
// A chunk is cut into nsub parts (partial[chunk * nsub + part]) where whole
// chunks are too few waves to fill the GPU: a wave walks its entries 16 at a
// time, each step a trip to memory, so 512 entries of a narrow block are a chain
// of 32 trips that eight parts cut to four.
template <class T>
struct NlContractArgs {
  const typename C2<T>::type* proj;
  const int32_t *sup_node, *chunk_atom, *chunk_begin, *chunk_end, *chunk_order, *atom_npj;
  int max_pj, nsub, n_work, n_coltiles;
  const double2* X;
  int64_t ldx;
  int n_vec;
  typename C2<T>::type* partial;
};

template <class T, bool REALP, bool PACK>
__device__ __forceinline__ void nl_contract_wave(const NlContractArgs<T>& g, int wid) {
  typedef typename C2<T>::type CT;
  typedef typename Vec4<T>::type V4;
  static_assert(!PACK || !REALP, "packed rows: complex projector values only");
  constexpr int U = 4;                    // k-steps per batch
  constexpr int NCB = nl_col_blocks<T>();
  const CT* __restrict__ proj = g.proj;
  const double2* __restrict__ X = g.X;
  const int32_t* __restrict__ sup_node = g.sup_node;
  const int64_t ldx = g.ldx;
  const int n_vec = g.n_vec, max_pj = g.max_pj;
  const int lane = threadIdx.x & 63;
  const int kl = lane >> 4, il = lane & 15;
  const int oi = wid / (g.n_coltiles * g.nsub), rem = wid - oi * g.n_coltiles * g.nsub;
  const int sub = rem / g.n_coltiles, ct = rem - sub * g.n_coltiles;
  const int ch = g.chunk_order[oi];
  const int a = g.chunk_atom[ch], cb0 = g.chunk_begin[ch], ce0 = g.chunk_end[ch];
  const int part = ((ce0 - cb0 + g.nsub - 1) / g.nsub + 15) / 16 * 16;   // whole batches per part
  const int b = cb0 + sub * part, e = min(ce0, b + part);                // b >= e: an empty part
  const int npj = g.atom_npj[a];
  const int chi = PACK ? (il & 7) : il;   // projector of this lane's A row
  int col[NCB];
  bool cv[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    col[cb] = ct * 16 * NCB + cb * 16 + il;
    cv[cb] = col[cb] < n_vec;
    if (!cv[cb]) col[cb] = n_vec - 1;     // clamped: loads stay in bounds
  }
  V4 cr[2][NCB], ci[2][NCB];              // [spin][16-column block]
#pragma unroll
  for (int sp = 0; sp < 2; ++sp)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) cr[sp][cb] = ci[sp][cb] = V4{0, 0, 0, 0};
  // Entry 4 u + kl of a batch is this lane's k index of step u.  All loads of a batch
  // are issued before its first use and without branches: the node numbers were
  // fetched with the batch before, unused rows (chi >= npj) and columns read in
  // bounds and are never stored.  Only the last, partial batch is masked (TAIL: its
  // missing entries repeat the last one with both factors zeroed).
  const int chi_c = min(chi, max_pj - 1);
  int nd[U];
  auto nodes = [&](int j0) {
#pragma unroll
    for (int u = 0; u < U; ++u) nd[u] = sup_node[min(j0 + 4 * u + kl, e - 1)];
  };
  auto batch = [&](int j0, auto tail) {
    constexpr bool TAIL = decltype(tail)::value;
    CT pv[U];
    double2 xv[U][2][NCB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = TAIL ? min(j0 + 4 * u + kl, e - 1) : j0 + 4 * u + kl;
      pv[u] = proj[(size_t)j * max_pj + chi_c];
      const double2* __restrict__ xr = X + 2 * (int64_t)nd[u] * ldx;
#pragma unroll
      for (int sp = 0; sp < 2; ++sp)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) xv[u][sp][cb] = xr[sp * ldx + col[cb]];
    }
    if (!TAIL) nodes(j0 + 4 * U);
    __builtin_amdgcn_sched_barrier(0);    // (the scheduler would pair loads and uses to save registers)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (TAIL) {
        const bool jv = j0 + 4 * u + kl < e;
        pv[u] = CT{jv ? pv[u].x : (T)0, jv ? pv[u].y : (T)0};
#pragma unroll
        for (int sp = 0; sp < 2; ++sp)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            xv[u][sp][cb].x = jv ? xv[u][sp][cb].x : 0.0;
            xv[u][sp][cb].y = jv ? xv[u][sp][cb].y : 0.0;
          }
      }
      if constexpr (PACK) {
        const T av = il < 8 ? pv[u].x : pv[u].y;
#pragma unroll
        for (int sp = 0; sp < 2; ++sp)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            cr[sp][cb] = mfma(av, (T)xv[u][sp][cb].x, cr[sp][cb]);   // [p_r; p_i] x_r
            ci[sp][cb] = mfma(av, (T)xv[u][sp][cb].y, ci[sp][cb]);   // [p_r; p_i] x_i
          }
      } else {
        const T pr = pv[u].x, pi = pv[u].y, npi = -pv[u].y;
#pragma unroll
        for (int sp = 0; sp < 2; ++sp)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            const T xr = (T)xv[u][sp][cb].x, xi = (T)xv[u][sp][cb].y;
            cr[sp][cb] = mfma(pr, xr, cr[sp][cb]);      // conj(p) x
            if (!REALP) cr[sp][cb] = mfma(pi, xi, cr[sp][cb]);
            ci[sp][cb] = mfma(pr, xi, ci[sp][cb]);
            if (!REALP) ci[sp][cb] = mfma(npi, xr, ci[sp][cb]);
          }
      }
    }
  };
  if (b < e) {                            // (an empty part stores zeros)
    nodes(b);
    int j0 = b;
    for (; j0 + 4 * U <= e; j0 += 4 * U) batch(j0, std::false_type{});
    if (j0 < e) batch(j0, std::true_type{});
  }
  CT* out = g.partial + ((size_t)ch * g.nsub + sub) * 2 * max_pj * n_vec;
  if constexpr (PACK) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (sizeof(T) == 8 && j >= 2) break;                       // FP64: rows 8-15
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
          // row x + 8: same lane (FP64) or the lane 32 above (FP32; every lane shuffles)
          T hr, hi;
          if constexpr (sizeof(T) == 8) {
            hr = cr[sp][cb][j + 2];
            hi = ci[sp][cb][j + 2];
          } else {
            hr = __shfl_down(cr[sp][cb][j], 32);
            hi = __shfl_down(ci[sp][cb][j], 32);
          }
          const int x = acc_row<T>(lane, j);
          if (x >= 8 || x >= npj || !cv[cb]) continue;             // FP32: lanes 32-63 hold rows 8-15
          CT v;
          v.x = cr[sp][cb][j] + hi;
          v.y = ci[sp][cb][j] - hr;
          out[(size_t)(2 * x + sp) * n_vec + col[cb]] = v;
        }
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int x = acc_row<T>(lane, j);
      if (x >= npj) continue;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        if (!cv[cb]) continue;
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
          CT v;
          v.x = cr[sp][cb][j];
          v.y = ci[sp][cb][j];
          out[(size_t)(2 * x + sp) * n_vec + col[cb]] = v;
        }
      }
    }
  }
}

// The same for a block of one column: 64 entries at a time, one per lane, and the sums
// over the lanes by halving (32 lanes keep one half of the values, 32 the other, and
// so on), so that four projectors take 17 exchanges.  The matrix-unit form loads each
// x sixteen times over, 12 wave loads for 16 entries against 6 for 64: 16 atoms,
// 250000 rows 39 -> 19 us.
template <class T, bool REALP>
__device__ __forceinline__ void nl_contract_one(const NlContractArgs<T>& g, int wid) {
  typedef typename C2<T>::type CT;
  const int lane = threadIdx.x & 63, max_pj = g.max_pj;
  const int oi = wid / g.nsub, sub = wid - oi * g.nsub;
  const int ch = g.chunk_order[oi];
  const int a = g.chunk_atom[ch], cb0 = g.chunk_begin[ch], ce0 = g.chunk_end[ch];
  const int part = ((ce0 - cb0 + g.nsub - 1) / g.nsub + 15) / 16 * 16;   // as in the block form
  const int b = cb0 + sub * part, e = min(ce0, b + part);
  const int npj = g.atom_npj[a];
  T s[kMaxPj][4];                         // [chi][spin][re, im]
#pragma unroll
  for (int x = 0; x < kMaxPj; ++x) s[x][0] = s[x][1] = s[x][2] = s[x][3] = (T)0;
  for (int j = b + lane; j < e; j += 64) {
    const double2* __restrict__ xr = g.X + 2 * (int64_t)g.sup_node[j] * g.ldx;
    const CT* __restrict__ pr = g.proj + (size_t)j * max_pj;
    CT pv[kMaxPj];
#pragma unroll
    for (int x = 0; x < kMaxPj; ++x)
      if (x < npj) pv[x] = pr[x];
    const double2 u = xr[0], d = xr[g.ldx];
    const T v[4] = {(T)u.x, (T)u.y, (T)d.x, (T)d.y};
#pragma unroll
    for (int x = 0; x < kMaxPj; ++x)
      if (x < npj) {
#pragma unroll
        for (int sp = 0; sp < 2; ++sp) {
          s[x][2 * sp] += pv[x].x * v[2 * sp];
          s[x][2 * sp + 1] += pv[x].x * v[2 * sp + 1];
          if (!REALP) {
            s[x][2 * sp] += pv[x].y * v[2 * sp + 1];
            s[x][2 * sp + 1] -= pv[x].y * v[2 * sp];
          }
        }
      }
  }
  T* out = reinterpret_cast<T*>(g.partial + ((size_t)ch * g.nsub + sub) * 2 * max_pj);
#pragma unroll
  for (int x0 = 0; x0 < kMaxPj; x0 += 4) {
    if (x0 >= npj) break;
    T v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = x0 + k / 4 < kMaxPj ? s[x0 + k / 4 < kMaxPj ? x0 + k / 4 : 0][k % 4] : (T)0;
#pragma unroll
    for (int h = 8, d = 32; h > 0; h /= 2, d /= 2) {
      const bool up = lane & d;
#pragma unroll
      for (int k = 0; k < h; ++k) {
        const T keep = up ? v[k + h] : v[k], send = up ? v[k] : v[k + h];
        v[k] = keep + __shfl_xor(send, d);
      }
    }
    v[0] += __shfl_xor(v[0], 2);
    v[0] += __shfl_xor(v[0], 1);
    // lane bits 5..2, the highest first, are the value's index
    const int k = lane >> 2;
    if ((lane & 3) == 0 && x0 + k / 4 < npj) out[4 * x0 + k] = v[0];
  }
}

template <class T, bool REALP>
__global__ __launch_bounds__(256) void nl_contract_one_kernel(const NlContractArgs<T> g) {
  const int wid = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (wid < g.n_work) nl_contract_one<T, REALP>(g, wid);
}

template <class T, bool REALP, bool PACK = false>
__global__ __launch_bounds__(256) void nl_contract_kernel(const NlContractArgs<T> g) {
  // each XCD takes a contiguous range of the (window, atom)-ordered chunks, so the
  // chunks of different atoms over the same rows meet in that XCD's L2
  const int per_xcd = (int)((gridDim.x + 7) / 8);
  const int bid = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  const int wid = __builtin_amdgcn_readfirstlane(bid * 4 + (int)(threadIdx.x >> 6));
  if (wid >= g.n_work) return;            // no barrier in this kernel
  nl_contract_wave<T, REALP, PACK>(g, wid);
}

// Coefficients of one atom and COLS columns: the sum over the atom's parts,
//   C[r][n] = sum_part partial[part][r][n],
// and the coupling C'[r][n] = alpha sum_r' Delta[r][r'] C[r'][n] (r = 2 chi + spin).
// 256 / COLS threads per column take every (256 / COLS)th part (in a fixed order),
// meet by lane exchange and in LDS, and each then forms its rows of C'.  Serial
// chains of loads set its time, so the columns of a workgroup are few where the
// atoms and columns alone give few workgroups (coef_cols).  alpha_d (device, or
// null) overrides alpha at run time (graph replays with new filter bounds).
template <class T>
struct NlCoefArgs {
  const typename C2<T>::type* partial;
  const int32_t *atom_chunk0, *atom_npj;
  const double2* delta;
  int max_pj, nsub, n_part, col0, n_vec;      // the parts hold n_part columns: columns col0 .. of C'
  double alpha;
  const double* alpha_d;
  typename C2<T>::type* Cp;
};

template <class T>
struct NlCoefSmem {
  typename C2<T>::type w[4][2 * kMaxPj * 16];
  typename C2<T>::type c[2 * kMaxPj * 16];
};

template <class T, int COLS>
__device__ __forceinline__ void nl_coef_block(NlCoefSmem<T>& sm, const NlCoefArgs<T>& g, int a, int ctile) {
  typedef typename C2<T>::type CT;
  constexpr int SLOTS = 256 / COLS;
  const int tid = threadIdx.x, il = tid % COLS, slot = tid / COLS, wave = tid >> 6;
  const int col = ctile * COLS + il;
  const int mr = 2 * g.max_pj, nr = 2 * g.atom_npj[a];
  const int p0 = g.atom_chunk0[a] * g.nsub, p1 = g.atom_chunk0[a + 1] * g.nsub;
  const CT* __restrict__ part = g.partial + min(col, g.n_part - 1);
  T sr[2 * kMaxPj], si[2 * kMaxPj];
#pragma unroll
  for (int r = 0; r < 2 * kMaxPj; ++r) sr[r] = si[r] = (T)0;
  for (int p = p0 + slot; p < p1; p += SLOTS) {
    CT v[2 * kMaxPj];
#pragma unroll
    for (int r = 0; r < 2 * kMaxPj; ++r)
      if (r < nr) v[r] = part[((size_t)p * mr + r) * g.n_part];
#pragma unroll
    for (int r = 0; r < 2 * kMaxPj; ++r)
      if (r < nr) {
        sr[r] += v[r].x;
        si[r] += v[r].y;
      }
  }
#pragma unroll
  for (int r = 0; r < 2 * kMaxPj; ++r) {
#pragma unroll
    for (int d = COLS; d < 64; d *= 2) {
      sr[r] += __shfl_xor(sr[r], d);
      si[r] += __shfl_xor(si[r], d);
    }
    if ((tid & 63) < COLS) {
      CT o;
      o.x = sr[r];
      o.y = si[r];
      sm.w[wave][r * COLS + il] = o;
    }
  }
  __syncthreads();
  for (int e = tid; e < nr * COLS; e += 256) {
    CT o;
    o.x = (sm.w[0][e].x + sm.w[1][e].x) + (sm.w[2][e].x + sm.w[3][e].x);
    o.y = (sm.w[0][e].y + sm.w[1][e].y) + (sm.w[2][e].y + sm.w[3][e].y);
    sm.c[e] = o;
  }
  __syncthreads();
  const double alpha = g.alpha_d ? *g.alpha_d : g.alpha;
  for (int r = slot; r < nr; r += SLOTS) {
    T xr = 0, xi = 0;
    for (int q = 0; q < nr; ++q) {
      const double2 d = g.delta[((size_t)a * mr + r) * mr + q];
      const CT c = sm.c[q * COLS + il];
      xr += (T)d.x * c.x - (T)d.y * c.y;
      xi += (T)d.x * c.y + (T)d.y * c.x;
    }
    if (col < g.n_part) {
      CT o;
      o.x = (T)alpha * xr;
      o.y = (T)alpha * xi;
      g.Cp[((size_t)a * mr + r) * g.n_vec + g.col0 + col] = o;
    }
  }
}

template <class T, int COLS>
__global__ __launch_bounds__(256) void nl_coef_kernel(const NlCoefArgs<T> g) {
  __shared__ NlCoefSmem<T> sm;
  nl_coef_block<T, COLS>(sm, g, blockIdx.x, blockIdx.y);
}

// Recurrence initialisation fused with the nonlocal back-product, one wave per
// (run of kNlRun = 16 consecutive global nodes, 16- or 32-column tile):
//   W[2I+s][n] = beta Wold[2I+s][n] + gamma X[2I+s][n] + rscale[n] Rs[2I+s][n]
//               + sum_{atoms a at I} sum_chi P[entry(a, I)][chi] C'[a][2 chi + s][n]
// For each atom meeting the run, the back-product is the complex product of the
// run's 16 x n_pj projector block with the n_pj x (16 | 32) coefficient tile, done as
// 16x16x4 MFMAs (k = projector index, padded to a multiple of 4; nodes of the run
// outside the atom's support contribute zero rows).  All operands of an atom are
// loaded before its MFMAs; each coefficient row is read once per run.  W and
// Wold are not read without the beta term, X without the gamma term, Rs without
// the residual term (FL: which terms are present).  REALP: real projector values
// (Gamma point), two real MFMAs per step instead of four.  bg_d (device, or null)
// overrides (beta, gamma) at run time; FL still selects which terms are read.
// GATHER: the cell products were written cell by cell (ye[cell][local node][spin][n])
// and every node adds alpha (msc: alpha M^{-1/2}) times the values of the up to
// eight cells that hold it, in the colour order of the assembly: bit for bit the
// sum that the per-colour launches leave.  The cells of a node follow from its
// position in the mesh.
constexpr int kInitBeta = 1, kInitGamma = 2, kInitRs = 4;

struct MeshShape {
  int p, np1, nx, ny, nz, Nx, Ny;       // degree, cells and nodes per direction
};

template <class T>
struct InitArgs {
  const typename C2<T>::type* proj;
  const int32_t *run_off, *pair_atom, *pair_ent, *atom_npj;
  int max_pj, has_nl;
  const typename C2<T>::type* Cp;
  const double2* X;
  int64_t ldx;
  double2* W;
  int64_t ldw;
  const double2* Wold;
  int64_t ldo;
  const double2* Rs;
  int64_t ldr;
  const double* rscale;
  int64_t n_nodes;
  int n_work, n_coltiles, n_vec;
  double beta, gamma, alpha;
  const double *bg_d, *alpha_d;
  const typename C2<T>::type* ye;
  const double* msc;
  MeshShape mesh;
};

// The cells along one direction that hold node coordinate i, in colour order, as
// their part of the row of ye: cell * cell_rows + local index * loc_rows; returns
// how many (1 or 2).
__device__ __forceinline__ int dir_rows(int i, int p, int n, int cell_rows, int loc_rows, int (&row)[2]) {
  const int c = i / p, a = i - c * p;
  row[0] = row[1] = c * cell_rows + a * loc_rows;
  if (a != 0) return 1;
  const int l = c == 0 ? n - 1 : c - 1;               // the cell that ends at this node
  const int kc = (n % 2 != 0 && c == n - 1) ? 2 : c % 2, kl = (n % 2 != 0 && l == n - 1) ? 2 : l % 2;
  row[kl < kc ? 0 : 1] = l * cell_rows + p * loc_rows;
  return 2;
}

template <class T, int FL, bool REALP, bool GATHER>
__device__ __forceinline__ void init_nl_wave(const InitArgs<T>& g, int wid) {
  typedef typename C2<T>::type CT;
  typedef typename Vec4<T>::type V4;
  static_assert(kNlRun == 16, "one MFMA row block per run");
  double beta = g.beta, gamma = g.gamma;
  if (g.bg_d) {
    beta = g.bg_d[0];
    gamma = g.bg_d[1];
  }
  constexpr int KS = (kMaxPj + 3) / 4;    // k-steps per atom
  constexpr int NCB = nl_col_blocks<T>();
  const double2* __restrict__ X = g.X;
  const double2* Wold = g.Wold;
  double2* W = g.W;
  const double2* __restrict__ Rs = g.Rs;
  const double* __restrict__ rscale = g.rscale;
  const CT* __restrict__ proj = g.proj;
  const int64_t ldx = g.ldx, ldw = g.ldw, ldo = g.ldo, ldr = g.ldr, n_nodes = g.n_nodes;
  const int n_vec = g.n_vec, max_pj = g.max_pj;
  const int run = wid / g.n_coltiles, ct = wid - run * g.n_coltiles;
  const int lane = threadIdx.x & 63;
  const int kl = lane >> 4, il = lane & 15;
  int col[NCB];
  bool cv[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    col[cb] = ct * 16 * NCB + cb * 16 + il;
    cv[cb] = col[cb] < n_vec;
    if (!cv[cb]) col[cb] = n_vec - 1;     // clamped: loads stay in bounds
  }
  V4 dr[2][NCB], di[2][NCB];              // [spin][16-column block]
  // FP64: the recurrence terms start the accumulators, so that their loads are in
  // flight while the projector back-product runs (lane element j of an
  // accumulator is node acc_row(lane, j) of the run, column col[cb])
  constexpr bool kPre = sizeof(T) == 8;
  const int64_t node0 = (int64_t)run * kNlRun;
#pragma unroll
  for (int sp = 0; sp < 2; ++sp)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      dr[sp][cb] = di[sp][cb] = V4{0, 0, 0, 0};
      if constexpr (kPre) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int64_t node = node0 + acc_row<T>(lane, j);
          const int64_t row = 2 * (node < n_nodes ? node : n_nodes - 1) + sp;
          const int c = col[cb];
          double tr = 0.0, ti = 0.0;
          if (FL & kInitBeta) {
            const double2 o = Wold[row * ldo + c];
            tr += beta * o.x;
            ti += beta * o.y;
          }
          if (FL & kInitGamma) {
            const double2 xv = X[row * ldx + c];
            tr += gamma * xv.x;
            ti += gamma * xv.y;
          }
          if (FL & kInitRs) {
            const double2 rv = Rs[row * ldr + c];
            const double sc = rscale[c];
            tr += sc * rv.x;
            ti += sc * rv.y;
          }
          dr[sp][cb][j] = (T)tr;
          di[sp][cb][j] = (T)ti;
        }
      }
    }
  if (g.has_nl) {
    const int p0 = g.run_off[run], p1 = g.run_off[run + 1];
    for (int pr = p0; pr < p1; ++pr) {
      const int a = g.pair_atom[pr];
      const int npj = g.atom_npj[a];
      const int ent = g.pair_ent[(size_t)pr * kNlRun + il];    // A row = node il of the run
      const CT* __restrict__ cpa = g.Cp + (size_t)a * 2 * max_pj * n_vec;
      CT pa[KS];
      CT bv[KS][2][NCB];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int x = 4 * ks + kl;                               // projector index of this lane
        const bool xv = x < npj;
        pa[ks] = (xv && ent >= 0) ? proj[(size_t)ent * max_pj + x] : CT{(T)0, (T)0};
        const int xr = xv ? x : 0;
#pragma unroll
        for (int sp = 0; sp < 2; ++sp)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            const CT v = cpa[(size_t)(2 * xr + sp) * n_vec + col[cb]];
            bv[ks][sp][cb] = (xv && cv[cb]) ? v : CT{(T)0, (T)0};
          }
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (4 * ks >= npj) break;                                // wave-uniform
        const T nai = -pa[ks].y;
#pragma unroll
        for (int sp = 0; sp < 2; ++sp)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            dr[sp][cb] = mfma(pa[ks].x, bv[ks][sp][cb].x, dr[sp][cb]);
            if (!REALP) dr[sp][cb] = mfma(nai, bv[ks][sp][cb].y, dr[sp][cb]);
            di[sp][cb] = mfma(pa[ks].x, bv[ks][sp][cb].y, di[sp][cb]);
            if (!REALP) di[sp][cb] = mfma(pa[ks].y, bv[ks][sp][cb].x, di[sp][cb]);
          }
      }
    }
  }
  // lane holds nodes acc_row(lane, j) of the run, columns col[cb]; every load of
  // the epilogue is issued unconditionally (clamped rows) and only the stores
  // are predicated
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t node = node0 + acc_row<T>(lane, j);
    const bool nv = node < n_nodes;
    const int64_t nodec = nv ? node : n_nodes - 1;
    double2 v[NCB][2];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int sp = 0; sp < 2; ++sp) {
        const int64_t row = 2 * nodec + sp;
        const int c = col[cb];
        double2 t = {(double)dr[sp][cb][j], (double)di[sp][cb][j]};
        if constexpr (kPre) {
          v[cb][sp] = t;
          continue;
        }
        if (FL & kInitBeta) {
          const double2 o = Wold[row * ldo + c];
          t.x += beta * o.x;
          t.y += beta * o.y;
        }
        if (FL & kInitGamma) {
          const double2 xv = X[row * ldx + c];
          t.x += gamma * xv.x;
          t.y += gamma * xv.y;
        }
        if (FL & kInitRs) {
          const double2 rv = Rs[row * ldr + c];
          const double sc = rscale[c];
          t.x += sc * rv.x;
          t.y += sc * rv.y;
        }
        v[cb][sp] = t;
      }
    if constexpr (GATHER) {
      const MeshShape& ms = g.mesh;
      const int nd = (int)nodec, nloc = ms.np1 * ms.np1 * ms.np1;
      const double alpha = g.alpha_d ? *g.alpha_d : g.alpha;
      const double sc = g.msc ? alpha * g.msc[nd] : alpha;
      const int iyz = nd / ms.Nx, ix = nd - iyz * ms.Nx;
      const int iz = iyz / ms.Ny, iy = iyz - iz * ms.Ny;
      int rx[2], ry[2], rz[2];
      const int kx = dir_rows(ix, ms.p, ms.nx, nloc, 1, rx);
      const int ky = dir_rows(iy, ms.p, ms.ny, nloc * ms.nx, ms.np1, ry);
      const int kz = dir_rows(iz, ms.p, ms.nz, nloc * ms.nx * ms.ny, ms.np1 * ms.np1, rz);
#pragma unroll
      for (int z = 0; z < 2; ++z)
#pragma unroll
        for (int y = 0; y < 2; ++y)
          if (z < kz && y < ky) {
#pragma unroll
            for (int x = 0; x < 2; ++x)
              if (x < kx) {
                const CT* __restrict__ yr = g.ye + (size_t)(rx[x] + ry[y] + rz[z]) * 2 * n_vec;
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                  for (int sp = 0; sp < 2; ++sp) {
                    const CT yv = yr[(size_t)sp * n_vec + col[cb]];
                    v[cb][sp].x = fma(sc, (double)yv.x, v[cb][sp].x);
                    v[cb][sp].y = fma(sc, (double)yv.y, v[cb][sp].y);
                  }
              }
          }
    }
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int sp = 0; sp < 2; ++sp)
        if (nv && cv[cb]) W[(2 * node + sp) * ldw + col[cb]] = v[cb][sp];
  }
}

// The same for a block of one column, on the vector units: lane = (half of the run's
// atoms, node, spin), the halves meet by lane exchange.  The matrix-unit form spends
// 15 of 16 columns of every load on copies: 16 atoms, 250000 rows 40 -> 23 us.
template <class T>
__device__ __forceinline__ void init_one(const InitArgs<T>& g, int wid, int fl, bool realp) {
  typedef typename C2<T>::type CT;
  const int lane = threadIdx.x & 63, half = lane >> 5, il = (lane & 31) >> 1, sp = lane & 1;
  const int64_t node = (int64_t)wid * kNlRun + il;
  const bool nv = node < g.n_nodes;
  const int64_t nd = nv ? node : g.n_nodes - 1, row = 2 * nd + sp;
  const double beta = g.bg_d ? g.bg_d[0] : g.beta, gamma = g.bg_d ? g.bg_d[1] : g.gamma;
  double2 o = {0.0, 0.0}, xv = {0.0, 0.0}, rv = {0.0, 0.0};
  if (fl & kInitBeta) o = g.Wold[row * g.ldo];
  if (fl & kInitGamma) xv = g.X[row * g.ldx];
  if (fl & kInitRs) rv = g.Rs[row * g.ldr];
  CT s = {(T)0, (T)0};
  if (g.has_nl) {
    const int p1 = g.run_off[wid + 1];
    int pr = g.run_off[wid] + half;
    int a = pr < p1 ? g.pair_atom[pr] : 0, ent = pr < p1 ? g.pair_ent[(size_t)pr * kNlRun + il] : -1;
    for (; pr < p1; pr += 2) {
      const int npj = g.atom_npj[a];
      const CT* __restrict__ cp = g.Cp + (size_t)a * 2 * g.max_pj + sp;
      const CT* __restrict__ pp = g.proj + (size_t)(ent < 0 ? 0 : ent) * g.max_pj;
      const bool in = ent >= 0;
      CT pv[kMaxPj], cv[kMaxPj];
#pragma unroll
      for (int x = 0; x < kMaxPj; ++x)
        if (x < npj) {
          pv[x] = pp[x];
          cv[x] = cp[2 * x];
        }
      if (pr + 2 < p1) {                  // the next atom, with these in flight
        a = g.pair_atom[pr + 2];
        ent = g.pair_ent[(size_t)(pr + 2) * kNlRun + il];
      }
      if (in)
#pragma unroll
        for (int x = 0; x < kMaxPj; ++x)
          if (x < npj) {
            s.x += pv[x].x * cv[x].x;
            s.y += pv[x].x * cv[x].y;
            if (!realp) {
              s.x -= pv[x].y * cv[x].y;
              s.y += pv[x].y * cv[x].x;
            }
          }
    }
    s.x += __shfl_xor(s.x, 32);
    s.y += __shfl_xor(s.y, 32);
  }
  if (half != 0) return;
  double2 t = {(double)s.x, (double)s.y};
  if (fl & kInitBeta) {
    t.x += beta * o.x;
    t.y += beta * o.y;
  }
  if (fl & kInitGamma) {
    t.x += gamma * xv.x;
    t.y += gamma * xv.y;
  }
  if (fl & kInitRs) {
    t.x += g.rscale[0] * rv.x;
    t.y += g.rscale[0] * rv.y;
  }
  if (g.ye) {                             // as in the block form
    const MeshShape& ms = g.mesh;
    const int n = (int)nd, nloc = ms.np1 * ms.np1 * ms.np1;
    const double alpha = g.alpha_d ? *g.alpha_d : g.alpha;
    const double sc = g.msc ? alpha * g.msc[n] : alpha;
    const int iyz = n / ms.Nx, ix = n - iyz * ms.Nx;
    const int iz = iyz / ms.Ny, iy = iyz - iz * ms.Ny;
    int rx[2], ry[2], rz[2];
    const int kx = dir_rows(ix, ms.p, ms.nx, nloc, 1, rx);
    const int ky = dir_rows(iy, ms.p, ms.ny, nloc * ms.nx, ms.np1, ry);
    const int kz = dir_rows(iz, ms.p, ms.nz, nloc * ms.nx * ms.ny, ms.np1 * ms.np1, rz);
    CT yv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {         // all in flight (x fastest; absent ones repeat another)
      const int x = (k & 1) < kx ? k & 1 : 0, y = (k >> 1 & 1) < ky ? k >> 1 & 1 : 0, z = k >> 2 < kz ? k >> 2 : 0;
      yv[k] = g.ye[(size_t)(rx[x] + ry[y] + rz[z]) * 2 + sp];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if ((k & 1) < kx && (k >> 1 & 1) < ky && k >> 2 < kz) {
        t.x = fma(sc, (double)yv[k].x, t.x);
        t.y = fma(sc, (double)yv[k].y, t.y);
      }
  }
  if (nv) g.W[row * g.ldw] = t;
}

template <class T>
__global__ __launch_bounds__(256) void init_one_kernel(const InitArgs<T> g, int fl, int realp) {
  const int wid = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (wid < g.n_work) init_one<T>(g, wid, fl, realp);
}

template <class T, int FL, bool REALP, bool GATHER>
__global__ __launch_bounds__(256) void init_nl_kernel(const InitArgs<T> g) {
  const int wid = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (wid >= g.n_work) return;            // no barrier in this kernel
  init_nl_wave<T, FL, REALP, GATHER>(g, wid);
}

// the packed complex contraction applies (at most 8 projectors per atom)
static bool pack_rows(const NonlocalK& nl) { return nl.max_pj <= 8; }

// Parts per chunk of the contraction: enough waves for the GPU (16384 = 16 per
// SIMD; above that whole chunks are the better work items, since each part writes
// its own rows of partial sums), and 64 entries or more in a full chunk's part.  A
// function of the whole block's width, so that a contraction over column groups
// splits alike; whole chunks where the parts of a column would not fit the fixed
// scratch that takes the whole ones.
static int nl_parts(const NonlocalK& nl, int n_vec) {
  const int64_t waves = (int64_t)std::max(1, nl.n_chunks) * cdiv(n_vec, 16);
  const int s = (int)std::max<int64_t>(1, std::min<int64_t>(kNlChunk / 64, 16384 / waves));
  const size_t mr = 2 * nl.max_pj;
  const size_t need = ((size_t)nl.n_chunks * s * mr + (size_t)nl.n_atoms * mr * n_vec) * sizeof(double2);
  return need <= (size_t)CHFSI_NOALLOC_SCRATCH_BYTES ? s : 1;
}

// Rows of partial sums per projector row: parts times columns, or what a narrower block in
// more parts takes, so that scratch grown for one block serves every narrower one (under
// stream capture it cannot grow).  Widths of one 16-column tile count share their parts.
static size_t nl_partial_rows(const NonlocalK& nl, int n_vec) {
  size_t m = (size_t)nl_parts(nl, n_vec) * n_vec;
  for (int w = 16; w < n_vec && (int64_t)nl.n_chunks * (w / 16) <= 8192; w += 16)     // (beyond: whole chunks)
    m = std::max(m, (size_t)nl_parts(nl, w) * w);
  return m * nl.n_chunks;
}

// Columns per workgroup of the coefficient kernel.  A function of the whole block's
// width, so that column groups sum alike: 1 where columns are one or two (16 atoms of
// about 970 parts: 48 us with 16, 13 with 1), 4 where an atom has more than 64 parts
// and the workgroups still fit the GPU at once (4 atoms, 128 columns, about 130 parts
// each: 50 against 31 us), else 16 (32 tasks of 2 atoms with about 32 parts: 8.9
// against 12.1 us with 4).
static int coef_cols(const NonlocalK& nl, int n_vec) {
  if (n_vec <= 2) return 1;
  const int64_t parts = (int64_t)nl.n_chunks * nl_parts(nl, n_vec);
  return parts > 64 * (int64_t)nl.n_atoms && (int64_t)nl.n_atoms * cdiv(n_vec, 4) <= 1024 ? 4 : 16;
}

template <class T>
static NlContractArgs<T> contract_args(const NonlocalK& nl, const typename C2<T>::type* proj, const double2* X,
                                       int64_t ldx, int n_vec, int nsub, typename C2<T>::type* partial) {
  NlContractArgs<T> g;
  g.proj = proj;
  g.sup_node = nl.sup_node.ptr;
  g.chunk_atom = nl.chunk_atom.ptr;
  g.chunk_begin = nl.chunk_begin.ptr;
  g.chunk_end = nl.chunk_end.ptr;
  g.chunk_order = nl.chunk_order.ptr;
  g.atom_npj = nl.atom_npj.ptr;
  g.max_pj = nl.max_pj;
  g.nsub = nsub;
  g.n_coltiles = cdiv(n_vec, 16 * nl_col_blocks<T>());
  const int64_t work = (int64_t)nl.n_chunks * nsub * g.n_coltiles;
  CHFSI_CHECK(work < (int64_t)1 << 30, CHFSI_EINVAL, "nonlocal contraction: too many work items");
  g.n_work = (int)work;
  g.X = X;
  g.ldx = ldx;
  g.n_vec = n_vec;
  g.partial = partial;
  return g;
}

// Work of the stages, as the timers count it
struct StageWork {
  double flops, bytes;
};
static StageWork nonlocal_work(const NonlocalK& nl, int n_vec, size_t elem) {
  StageWork w{0.0, (double)nl.n_entries * (2.0 * n_vec * sizeof(double2) + nl.max_pj * elem)};
  for (const auto& at : nl.atoms)
    w.flops += 2.0 * 8.0 * at.n_sup * at.n_pj * 2.0 * n_vec + 8.0 * 4.0 * at.n_pj * at.n_pj * n_vec;
  return w;
}
// terms: recurrence terms read, beside the rows written; ye_elem: bytes of a gathered
// cell product (0: none are)
static StageWork init_work(const chfsi_ctx* c, const NonlocalK* nl, int n_vec, int terms, size_t ye_elem) {
  return StageWork{nl ? 8.0 * 2.0 * nl->n_entries * nl->max_pj * n_vec : 0.0,
                   2.0 * (double)c->n_nodes * n_vec * sizeof(double2) * (1.0 + terms) +
                       2.0 * (double)c->n_cells * c->nloc * n_vec * ye_elem};
}

// Nonlocal coefficients C' = alpha Delta P^H X for every atom; returns the
// device array [n_atoms][2 max_pj][n_vec] (in the scratch buffer), or null.
// Scratch: the caller's buffer (scratch, at least nonlocal_scratch_bytes(nl,
// n_vec) bytes) or the context's growable buffer.  alpha_d as in nl_coef_kernel.
template <class T>
static const typename C2<T>::type* nonlocal_coeffs(chfsi_ctx* c, NonlocalK& nl,
                                                   const typename C2<T>::type* proj, const double2* X,
                                                   int64_t ldx, int n_vec, double alpha,
                                                   const double* alpha_d = nullptr, void* scratch = nullptr) {
  typedef typename C2<T>::type CT;
  if (nl.n_atoms == 0 || nl.n_entries == 0) return nullptr;
  const int mr = 2 * nl.max_pj;
  const int nsub = nl_parts(nl, n_vec);
  const size_t n_cp = (size_t)nl.n_atoms * mr * n_vec;
  int group = n_vec;                      // columns per contraction launch
  if (!scratch && c->nl_fixed) {
    // fixed buffer: whole coefficient arrays, then as many columns of
    // partials per contraction launch as fit (the caller checked that one does)
    const size_t per_col = (size_t)nl.n_chunks * nsub * mr * sizeof(CT);
    const size_t head = n_cp * sizeof(CT);
    CHFSI_CHECK(c->nl_fixed_bytes >= head + per_col, CHFSI_EINVAL, "fixed nonlocal scratch too small");
    group = (int)std::min<size_t>(n_vec, (c->nl_fixed_bytes - head) / per_col);
    scratch = c->nl_fixed;
  } else if (!scratch) {
    const size_t bytes = (nl_partial_rows(nl, n_vec) * mr + n_cp) * sizeof(CT);
    c->scratch.alloc((bytes + sizeof(double) - 1) / sizeof(double));
    scratch = c->scratch.ptr;
  }
  CT* Cp = reinterpret_cast<CT*>(scratch);
  CT* partial = Cp + n_cp;
  const StageWork nw = nonlocal_work(nl, n_vec, sizeof(CT));
  StageTimer tm(c, CHFSI_STAGE_NONLOCAL, nw.flops, nw.flops, nw.bytes);
  for (int c0 = 0; c0 < n_vec; c0 += group) {
    const int gc = std::min(group, n_vec - c0);
    const NlContractArgs<T> ca = contract_args<T>(nl, proj, X + c0, ldx, gc, nsub, partial);
    const dim3 cgrid(8 * cdiv(cdiv(ca.n_work, 4), 8));
    if (n_vec == 1 && nl.real_proj)
      hipLaunchKernelGGL((nl_contract_one_kernel<T, true>), cgrid, dim3(256), 0, c->stream, ca);
    else if (n_vec == 1)
      hipLaunchKernelGGL((nl_contract_one_kernel<T, false>), cgrid, dim3(256), 0, c->stream, ca);
    else if (nl.real_proj)
      hipLaunchKernelGGL((nl_contract_kernel<T, true>), cgrid, dim3(256), 0, c->stream, ca);
    else if (pack_rows(nl))
      hipLaunchKernelGGL((nl_contract_kernel<T, false, true>), cgrid, dim3(256), 0, c->stream, ca);
    else
      hipLaunchKernelGGL((nl_contract_kernel<T, false>), cgrid, dim3(256), 0, c->stream, ca);
    LAUNCH_CHECK();
    const NlCoefArgs<T> co{partial, nl.atom_chunk0.ptr, nl.atom_npj.ptr, nl.delta.ptr, nl.max_pj, nsub,
                           gc,      c0,                 n_vec,           alpha,        alpha_d,   Cp};
    const int cols = coef_cols(nl, n_vec);
    const dim3 fgrid(nl.n_atoms, cdiv(gc, cols));
    if (cols == 1) hipLaunchKernelGGL((nl_coef_kernel<T, 1>), fgrid, dim3(256), 0, c->stream, co);
    else if (cols == 4) hipLaunchKernelGGL((nl_coef_kernel<T, 4>), fgrid, dim3(256), 0, c->stream, co);
    else hipLaunchKernelGGL((nl_coef_kernel<T, 16>), fgrid, dim3(256), 0, c->stream, co);
    LAUNCH_CHECK();
  }
  return Cp;
}

static MeshShape mesh_shape(const chfsi_ctx* c) {
  return MeshShape{c->p, c->np1, c->nc[0], c->nc[1], c->nc[2], c->Nd[0], c->Nd[1]};
}

template <class T>
static InitArgs<T> init_args(chfsi_ctx* c, NonlocalK& nl, const typename C2<T>::type* proj,
                             const typename C2<T>::type* Cp, const double2* X, int64_t ldx, double2* W, int64_t ldw,
                             const double2* Wold, int64_t ldo, int n_vec, double beta, double gamma) {
  const bool has = Cp != nullptr;
  InitArgs<T> g{};
  g.proj = proj;
  g.run_off = has ? nl.run_off.ptr : nullptr;
  g.pair_atom = has ? nl.pair_atom.ptr : nullptr;
  g.pair_ent = has ? nl.pair_ent.ptr : nullptr;
  g.atom_npj = has ? nl.atom_npj.ptr : nullptr;
  g.max_pj = nl.max_pj;
  g.has_nl = has;
  g.Cp = Cp;
  g.X = X;
  g.ldx = ldx;
  g.W = W;
  g.ldw = ldw;
  g.Wold = Wold;
  g.ldo = ldo;
  g.n_nodes = c->n_nodes;
  g.n_coltiles = cdiv(n_vec, 16 * nl_col_blocks<T>());
  g.n_work = (int)((c->n_nodes + kNlRun - 1) / kNlRun * g.n_coltiles);
  g.n_vec = n_vec;
  g.beta = beta;
  g.gamma = gamma;
  g.mesh = mesh_shape(c);
  return g;
}

template <class T>
static void launch_init(chfsi_ctx* c, const InitArgs<T>& g, const NonlocalK& nl) {
  const bool realp = g.has_nl && nl.real_proj;
  const StageWork iw = init_work(c, g.has_nl ? &nl : nullptr, g.n_vec, (g.beta != 0.0) + (g.gamma != 0.0),
                                 g.ye ? 2 * sizeof(T) : 0);
  StageTimer tm(c, CHFSI_STAGE_AXPY, iw.flops, 0.0, iw.bytes);
  const int fl = (g.beta != 0.0 ? kInitBeta : 0) | (g.gamma != 0.0 ? kInitGamma : 0) | (g.Rs ? kInitRs : 0);
  const dim3 grid(cdiv(g.n_work, 4)), blk(256);
  if (g.n_vec == 1) {
    hipLaunchKernelGGL((init_one_kernel<T>), grid, blk, 0, c->stream, g, fl, realp ? 1 : 0);
    LAUNCH_CHECK();
    return;
  }
#define INIT_NL_LAUNCH(F, RP, GA) hipLaunchKernelGGL((init_nl_kernel<T, F, RP, GA>), grid, blk, 0, c->stream, g)
#define INIT_NL_CASE(F)                     \
  case F:                                   \
    if (realp && g.ye)                      \
      INIT_NL_LAUNCH(F, true, true);        \
    else if (realp)                         \
      INIT_NL_LAUNCH(F, true, false);       \
    else if (g.ye)                          \
      INIT_NL_LAUNCH(F, false, true);       \
    else                                    \
      INIT_NL_LAUNCH(F, false, false);      \
    break;
  switch (fl) {
    INIT_NL_CASE(0)
    INIT_NL_CASE(1)
    INIT_NL_CASE(2)
    INIT_NL_CASE(3)
    INIT_NL_CASE(4)
    INIT_NL_CASE(5)
    INIT_NL_CASE(6)
    default:
    INIT_NL_CASE(7)
  }
#undef INIT_NL_CASE
#undef INIT_NL_LAUNCH
  LAUNCH_CHECK();
}

// Where the cell products of one apply go.  Per-colour launches add them into
// the output; each needs enough workgroups, or its tail (and at the 27 colours of
// an odd mesh the number of launches) sets the time.  Otherwise one launch over all
// cells writes them to ye, and the initialisation pass gathers them: the same
// sums to the bit.  The line is drawn at kYeWork workgroups per colour on the mean
// and kYeMax bytes of ye.  Filters by colours and by cells: 3^3 cells, p = 4, one
// apply of 32 columns 500 and 47 us; 9^3, p = 5 (27 colours), matrix-free, 130
// columns 23.5 and 18.8 ms; 8^3, p = 5, matrix-free adjoint, 128 columns (4096
// workgroups per colour) 46.2 and 43.2 ms; 8^3, p = 6, cell matrices, 128 columns
// 72.6 and 68.8 ms; 16^3, p = 6, matrix-free, 128 columns (32768 per colour) 226
// and 233 ms.
constexpr int64_t kYeWork = 8192;
constexpr size_t kYeMax = (size_t)2 << 30;

size_t products_scratch_bytes(const chfsi_ctx* c, int n_vec, bool fp64) {
  const int64_t per_cell = c->form == CHFSI_FORM_MATRIX_FREE ? mf_items_per_cell(c, n_vec, fp64)
                                                             : cell_items_per_cell(c, n_vec);
  const size_t bytes = (size_t)c->n_cells * c->nloc * 2 * n_vec * (fp64 ? sizeof(double2) : sizeof(float2));
  return per_cell * c->n_cells <= kYeWork * c->n_colours && bytes <= kYeMax ? bytes : 0;
}

// The context's ye for this apply, or null: per-colour launches (which also serve
// where nothing may be allocated, the fixed-scratch filter).  Under stream capture
// always null: a graph would keep ye's address, and a wider apply after the capture
// moves ye.  (The default stream cannot be captured.)
static void* ye_for_call(chfsi_ctx* c, int n_vec, bool fp64) {
  const size_t bytes = c->nl_fixed ? 0 : products_scratch_bytes(c, n_vec, fp64);
  if (bytes == 0) return nullptr;
  if (c->stream) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    CHFSI_HIP(hipStreamIsCapturing(c->stream, &st));
    if (st != hipStreamCaptureStatusNone) return nullptr;
  }
  return c->ye.get(bytes);
}

template <class T>
static void apply_t(chfsi_ctx* c, KPoint& kp, const typename C2<T>::type* proj, const double2* X, int64_t ldx,
                    double2* W, int64_t ldw, const double2* Wold, int64_t ldo, int n_vec, int prec, double alpha,
                    double beta, double gamma, const double2* Rs, int64_t ldr, const double* rscale) {
  typedef typename C2<T>::type CT;
  const bool mf = c->form == CHFSI_FORM_MATRIX_FREE;
  const CT* Cp = nonlocal_coeffs<T>(c, kp.nl, proj, X, ldx, n_vec, alpha);
  InitArgs<T> g = init_args<T>(c, kp.nl, proj, Cp, X, ldx, W, ldw, Wold, ldo, n_vec, beta, gamma);
  g.Rs = Rs;
  g.ldr = ldr;
  g.rscale = rscale;
  CT* ye = static_cast<CT*>(ye_for_call(c, n_vec, sizeof(T) == 8));
  if (ye) {
    g.ye = ye;
    g.alpha = alpha;
    g.msc = mf ? c->minv_sqrt.ptr : nullptr;
    if (mf) launch_mf_products(c, kp, prec, X, ldx, nullptr, 0, n_vec, 1.0, nullptr, ye);
    else launch_cell_products(c, kp, prec, X, ldx, nullptr, 0, n_vec, 1.0, ye);
    launch_init<T>(c, g, kp.nl);
    return;
  }
  launch_init<T>(c, g, kp.nl);
  if (mf) launch_mf_products(c, kp, prec, X, ldx, W, ldw, n_vec, alpha);
  else launch_cell_products(c, kp, prec, X, ldx, W, ldw, n_vec, alpha);
}

void apply_H3(chfsi_ctx* c, KPoint& kp, const double2* X, int64_t ldx, double2* W, int64_t ldw,
              const double2* Wold, int64_t ldo, int n_vec, int prec, double alpha, double beta, double gamma,
              const double2* Rs, int64_t ldr, const double* rscale) {
  if (prec == CHFSI_PREC_MIXED)
    apply_t<float>(c, kp, kp.nl.proj32.ptr, X, ldx, W, ldw, Wold, ldo, n_vec, prec, alpha, beta, gamma, Rs, ldr,
                   rscale);
  else
    apply_t<double>(c, kp, kp.nl.proj.ptr, X, ldx, W, ldw, Wold, ldo, n_vec, prec, alpha, beta, gamma, Rs, ldr,
                    rscale);
}

void apply_H2(chfsi_ctx* c, KPoint& kp, const double2* X, int64_t ldx, double2* W, int64_t ldw,
              const double2* Wold, int64_t ldo, int n_vec, int prec, double alpha, double beta,
              double gamma) {
  apply_H3(c, kp, X, ldx, W, ldw, Wold, ldo, n_vec, prec, alpha, beta, gamma, nullptr, 0, nullptr);
}

// Y[r][n] = a[n] Y[r][n] + b[n] X[r][n]   (per-column scalars on the device)
__global__ void cols_axpby_kernel(double2* __restrict__ Y, int64_t ldy, const double2* __restrict__ X, int64_t ldx,
                                  int64_t rows, int n_vec, const double* __restrict__ a, const double* __restrict__ b) {
  const int64_t total = rows * n_vec;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / n_vec;
    const int n = (int)(t - r * n_vec);
    const double2 y = Y[r * ldy + n], x = X[r * ldx + n];
    Y[r * ldy + n] = double2{a[n] * y.x + b[n] * x.x, a[n] * y.y + b[n] * x.y};
  }
}

void launch_cols_axpby(chfsi_ctx* c, double2* Y, int64_t ldy, const double2* X, int64_t ldx, int64_t rows,
                       int n_vec, const double* a_d, const double* b_d) {
  const int64_t total = rows * n_vec;
  const int blocks = (int)std::min<int64_t>(cdiv(total, 256), 8192);
  StageTimer tm(c, CHFSI_STAGE_AXPY, 0.0, 0.0, 3.0 * (double)total * sizeof(double2));
  hipLaunchKernelGGL(cols_axpby_kernel, dim3(std::max(blocks, 1)), dim3(256), 0, c->stream, Y, ldy, X, ldx, rows,
                     n_vec, a_d, b_d);
  LAUNCH_CHECK();
}

void apply_H(chfsi_ctx* c, KPoint& kp, const double2* X, int64_t ldx, double2* W, int64_t ldw,
             int n_vec, int prec, double alpha, double beta, double gamma) {
  apply_H2(c, kp, X, ldx, W, ldw, W, ldw, n_vec, prec, alpha, beta, gamma);
}

// ---------------------------------------------------------------- batched support
template <class T>
static void nonlocal_init_t(chfsi_ctx* c, KPoint& kp, const typename C2<T>::type* proj, const double2* X, int64_t ldx,
                            double2* W, int64_t ldw, int n_vec, double alpha, double beta, double gamma,
                            const double* alpha_d, const double* bg_d, void* scratch) {
  const typename C2<T>::type* Cp = nonlocal_coeffs<T>(c, kp.nl, proj, X, ldx, n_vec, alpha, alpha_d, scratch);
  InitArgs<T> g = init_args<T>(c, kp.nl, proj, Cp, X, ldx, W, ldw, W, ldw, n_vec, beta, gamma);
  g.bg_d = bg_d;
  launch_init<T>(c, g, kp.nl);
}

void apply_nonlocal_init(chfsi_ctx* c, KPoint& kp, const double2* X, int64_t ldx, double2* W, int64_t ldw,
                         int n_vec, int prec, double alpha, double beta, double gamma, const double* alpha_d,
                         const double* bg_d, void* scratch) {
  if (prec == CHFSI_PREC_MIXED)
    nonlocal_init_t<float>(c, kp, kp.nl.proj32.ptr, X, ldx, W, ldw, n_vec, alpha, beta, gamma, alpha_d, bg_d, scratch);
  else
    nonlocal_init_t<double>(c, kp, kp.nl.proj.ptr, X, ldx, W, ldw, n_vec, alpha, beta, gamma, alpha_d, bg_d, scratch);
}

// ---- Small tasks of a batch: one launch per stage of an apply for all of them.  Per
// task the same waves and blocks as in an apply by cells (bit for bit); a table gives
// each workgroup its task and block, and the tasks' arguments are in device memory.
template <class T>
struct BatchNl {
  NlContractArgs<T> c;
  NlCoefArgs<T> f;
  InitArgs<T> i;
  double2* buf[2];
  int64_t ld[2];
  int64_t rows;
  int index;                              // in the recurrence coefficient tables
  int has_nl, realp, pack, n_atoms, coef_cols, coef_tiles;
};
constexpr int kBatchCopy = 4096;          // elements per workgroup of the copy

// A pointer read from memory, as one to device memory (else its accesses are flat).
template <class P>
__device__ __forceinline__ P* global_ptr(P* p) {
  return (P*)(__attribute__((address_space(1))) P*)p;
}

template <class T>
__global__ __launch_bounds__(256) void batch_contract_kernel(const BatchNl<T>* __restrict__ tasks,
                                                             const int2* __restrict__ map, int src) {
  const int2 w = map[blockIdx.x];
  const BatchNl<T>& t = tasks[w.x];
  const int wid = __builtin_amdgcn_readfirstlane(w.y * 4 + (int)(threadIdx.x >> 6));
  if (wid >= t.c.n_work) return;      // no barrier in this kernel
  NlContractArgs<T> g = t.c;
  g.proj = global_ptr(g.proj);
  g.sup_node = global_ptr(g.sup_node);
  g.chunk_atom = global_ptr(g.chunk_atom);
  g.chunk_begin = global_ptr(g.chunk_begin);
  g.chunk_end = global_ptr(g.chunk_end);
  g.chunk_order = global_ptr(g.chunk_order);
  g.atom_npj = global_ptr(g.atom_npj);
  g.partial = global_ptr(g.partial);
  g.X = global_ptr(t.buf[src]);
  g.ldx = t.ld[src];
  if (t.realp) nl_contract_wave<T, true, false>(g, wid);
  else if (t.pack) nl_contract_wave<T, false, true>(g, wid);
  else nl_contract_wave<T, false, false>(g, wid);
}

template <class T>
__global__ __launch_bounds__(256) void batch_coef_kernel(const BatchNl<T>* __restrict__ tasks,
                                                         const int2* __restrict__ map,
                                                         const double* __restrict__ alpha) {
  __shared__ NlCoefSmem<T> sm;
  const int2 w = map[blockIdx.x];
  const BatchNl<T>& t = tasks[w.x];
  NlCoefArgs<T> g = t.f;
  g.partial = global_ptr(g.partial);
  g.atom_chunk0 = global_ptr(g.atom_chunk0);
  g.atom_npj = global_ptr(g.atom_npj);
  g.delta = global_ptr(g.delta);
  g.Cp = global_ptr(g.Cp);
  g.alpha_d = alpha + t.index;
  const int a = w.y / t.coef_tiles, ct = w.y % t.coef_tiles;
  if (t.coef_cols == 1) nl_coef_block<T, 1>(sm, g, a, ct);
  else if (t.coef_cols == 4) nl_coef_block<T, 4>(sm, g, a, ct);
  else nl_coef_block<T, 16>(sm, g, a, ct);
}

template <class T, int FL>
__global__ __launch_bounds__(256) void batch_init_kernel(const BatchNl<T>* __restrict__ tasks,
                                                         const int2* __restrict__ map, int src,
                                                         const double* __restrict__ alpha,
                                                         const double* __restrict__ bg) {
  const int2 w = map[blockIdx.x];
  const BatchNl<T>& t = tasks[w.x];
  const int wid = __builtin_amdgcn_readfirstlane(w.y * 4 + (int)(threadIdx.x >> 6));
  if (wid >= t.i.n_work) return;          // no barrier in this kernel
  InitArgs<T> g = t.i;
  g.proj = global_ptr(g.proj);
  g.run_off = global_ptr(g.run_off);
  g.pair_atom = global_ptr(g.pair_atom);
  g.pair_ent = global_ptr(g.pair_ent);
  g.atom_npj = global_ptr(g.atom_npj);
  g.Cp = global_ptr(g.Cp);
  g.ye = global_ptr(g.ye);
  if (g.msc) g.msc = global_ptr(g.msc);
  g.X = global_ptr(t.buf[src]);
  g.ldx = t.ld[src];
  g.W = global_ptr(t.buf[src ^ 1]);
  g.ldw = t.ld[src ^ 1];
  g.Wold = g.W;
  g.ldo = g.ldw;
  g.alpha_d = alpha + t.index;
  g.bg_d = bg + 2 * t.index;
  if (t.realp) init_nl_wave<T, FL, true, true>(g, wid);
  else init_nl_wave<T, FL, false, true>(g, wid);
}

__global__ __launch_bounds__(256) void batch_copy_kernel(const BatchNl<double>* __restrict__ tasks,
                                                         const int2* __restrict__ map) {
  const int2 w = map[blockIdx.x];
  const BatchNl<double>& t = tasks[w.x];
  double2* d = global_ptr(t.buf[0]);
  const double2* s = global_ptr(t.buf[1]);
  const int n_vec = t.i.n_vec;
  const int64_t i0 = (int64_t)w.y * kBatchCopy, total = t.rows * n_vec;
  const int64_t i1 = i0 + kBatchCopy < total ? i0 + kBatchCopy : total;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) {
    const int64_t r = i / n_vec, n = i - r * n_vec;
    d[r * t.ld[0] + n] = s[r * t.ld[1] + n];
  }
}

// (task, block of the task) of each workgroup of a launch
struct BatchMap {
  std::vector<int2> h;
  DevBuf<int2> d;
  int n = 0;
  void add(int task, int64_t blocks) {
    for (int64_t i = 0; i < blocks; ++i) h.push_back(int2{task, (int)i});
  }
  void upload(hipStream_t s) {
    n = (int)h.size();
    if (n > 0) d.upload(h.data(), h.size(), s);
  }
};
template <class T>
struct BatchStage {
  std::vector<BatchNl<T>> h;
  DevBuf<BatchNl<T>> d;
  BatchMap contract, coef, init;
  void add(const BatchNl<T>& b) {
    const int t = (int)h.size();
    h.push_back(b);
    if (b.has_nl) {
      contract.add(t, cdiv(b.c.n_work, 4));
      coef.add(t, (int64_t)b.n_atoms * b.coef_tiles);
    }
    init.add(t, cdiv(b.i.n_work, 4));
  }
  void upload(hipStream_t s) {
    d.upload(h.data(), h.size(), s);
    contract.upload(s);
    coef.upload(s);
    init.upload(s);
  }
};
// one context's part of the joint launches, for its stage timers
struct BatchShare {
  chfsi_ctx* ctx;
  StageWork nl[2], init[2][2];            // [precision: FP32, FP64], [step: the first, later ones][precision]
};
struct BatchSmall::Impl {
  BatchStage<double> s64;
  BatchStage<float> s32;
  BatchMap copy;
  std::vector<BatchShare> shares;
  // The timers of the contexts that record: the launches' time goes to all contexts by
  // their flops (nonlocal) or bytes (init).
  typedef std::vector<std::unique_ptr<StageTimer>> Timers;
  Timers time(bool nonlocal, bool first, bool fp64) const {
    Timers t;
    const int stage = nonlocal ? CHFSI_STAGE_NONLOCAL : CHFSI_STAGE_AXPY;
    double total = 0.0;
    for (const auto& s : shares) total += nonlocal ? s.nl[fp64].flops : s.init[!first][fp64].bytes;
    for (const auto& s : shares) {
      const StageWork& w = nonlocal ? s.nl[fp64] : s.init[!first][fp64];
      const double part = nonlocal ? w.flops : w.bytes;
      if (s.ctx->stats_on && part > 0.0)
        t.emplace_back(new StageTimer(s.ctx, stage, w.flops, nonlocal ? w.flops : 0.0, w.bytes, part / total));
    }
    return t;
  }
};

template <class T>
static BatchNl<T> batch_nl(const SmallTask& s, const typename C2<T>::type* proj) {
  typedef typename C2<T>::type CT;
  chfsi_ctx* c = s.ctx;
  NonlocalK& nl = s.kp->nl;
  BatchNl<T> b{};
  b.buf[0] = s.buf[0];
  b.buf[1] = s.buf[1];
  b.ld[0] = s.ld[0];
  b.ld[1] = s.ld[1];
  b.rows = 2 * c->n_nodes;
  b.index = s.index;
  b.has_nl = nl.n_atoms != 0 && nl.n_entries != 0;
  CT* Cp = nullptr;
  if (b.has_nl) {
    const int nsub = nl_parts(nl, s.n_vec);
    Cp = reinterpret_cast<CT*>(s.nl_scratch);
    CT* partial = Cp + (size_t)nl.n_atoms * 2 * nl.max_pj * s.n_vec;
    b.c = contract_args<T>(nl, proj, nullptr, 0, s.n_vec, nsub, partial);
    b.f = NlCoefArgs<T>{partial, nl.atom_chunk0.ptr, nl.atom_npj.ptr, nl.delta.ptr, nl.max_pj, nsub,
                        s.n_vec, 0,                  s.n_vec,         1.0,          nullptr,   Cp};
    b.realp = nl.real_proj;
    b.pack = pack_rows(nl);
    b.n_atoms = nl.n_atoms;
    b.coef_cols = coef_cols(nl, s.n_vec);
    b.coef_tiles = cdiv(s.n_vec, b.coef_cols);
  }
  b.i = init_args<T>(c, nl, proj, Cp, nullptr, 0, nullptr, 0, nullptr, 0, s.n_vec, 1.0, 1.0);
  b.i.ye = reinterpret_cast<const CT*>(s.ye);
  b.i.msc = c->form == CHFSI_FORM_MATRIX_FREE ? c->minv_sqrt.ptr : nullptr;
  return b;
}

BatchSmall::BatchSmall(const std::vector<SmallTask>& tasks, hipStream_t stream) : impl_(new Impl) {
  Impl& m = *impl_;
  for (size_t t = 0; t < tasks.size(); ++t) {
    const SmallTask& s = tasks[t];
    m.s64.add(batch_nl<double>(s, s.kp->nl.proj.ptr));
    m.s32.add(batch_nl<float>(s, s.kp->nl.proj32.ptr));
    m.copy.add((int)t, (2 * s.ctx->n_nodes * s.n_vec + kBatchCopy - 1) / kBatchCopy);
    auto sh = std::find_if(m.shares.begin(), m.shares.end(), [&](const BatchShare& x) { return x.ctx == s.ctx; });
    if (sh == m.shares.end()) sh = m.shares.insert(sh, BatchShare{s.ctx, {}, {}});
    const NonlocalK& nl = s.kp->nl;
    const bool has = nl.n_atoms != 0 && nl.n_entries != 0;
    const auto add = [](StageWork& a, const StageWork& b) {
      a.flops += b.flops;
      a.bytes += b.bytes;
    };
    for (int k = 0; k < 2; ++k) {
      if (has) add(sh->nl[k], nonlocal_work(nl, s.n_vec, k ? sizeof(double2) : sizeof(float2)));
      for (int later = 0; later < 2; ++later)
        add(sh->init[later][k],
            init_work(s.ctx, has ? &nl : nullptr, s.n_vec, 1 + later, k ? sizeof(double2) : sizeof(float2)));
    }
  }
  m.s64.upload(stream);
  m.s32.upload(stream);
  m.copy.upload(stream);
  CHFSI_HIP(hipStreamSynchronize(stream));   // the host arrays have been read
}

BatchSmall::~BatchSmall() = default;

template <class T>
static void batch_nonlocal(hipStream_t s, const BatchStage<T>& b, int src, const double* alpha) {
  if (b.contract.n == 0) return;          // no task has atoms
  hipLaunchKernelGGL((batch_contract_kernel<T>), dim3(b.contract.n), dim3(256), 0, s, b.d.ptr, b.contract.d.ptr, src);
  LAUNCH_CHECK();
  hipLaunchKernelGGL((batch_coef_kernel<T>), dim3(b.coef.n), dim3(256), 0, s, b.d.ptr, b.coef.d.ptr, alpha);
  LAUNCH_CHECK();
}

void BatchSmall::nonlocal(hipStream_t s, bool fp64, int src, const double* alpha) {
  const auto tm = impl_->time(true, false, fp64);
  if (fp64) batch_nonlocal(s, impl_->s64, src, alpha);
  else batch_nonlocal(s, impl_->s32, src, alpha);
}

template <class T>
static void batch_init(hipStream_t s, const BatchStage<T>& b, int src, bool first, const double* alpha,
                       const double* bg) {
  if (first)
    hipLaunchKernelGGL((batch_init_kernel<T, kInitGamma>), dim3(b.init.n), dim3(256), 0, s, b.d.ptr, b.init.d.ptr, src,
                       alpha, bg);
  else
    hipLaunchKernelGGL((batch_init_kernel<T, kInitBeta | kInitGamma>), dim3(b.init.n), dim3(256), 0, s, b.d.ptr,
                       b.init.d.ptr, src, alpha, bg);
  LAUNCH_CHECK();
}

void BatchSmall::init(hipStream_t s, bool fp64, int src, bool first, const double* alpha, const double* bg) {
  const auto tm = impl_->time(false, first, fp64);
  if (fp64) batch_init(s, impl_->s64, src, first, alpha, bg);
  else batch_init(s, impl_->s32, src, first, alpha, bg);
}

void BatchSmall::copy_back(hipStream_t s) {
  hipLaunchKernelGGL(batch_copy_kernel, dim3(impl_->copy.n), dim3(256), 0, s, impl_->s64.d.ptr, impl_->copy.d.ptr);
  LAUNCH_CHECK();
}

size_t nonlocal_scratch_bytes_min(const KPoint& kp, int n_vec) {
  const NonlocalK& nl = kp.nl;
  if (nl.n_atoms == 0 || nl.n_entries == 0) return 0;
  const size_t mr = 2 * nl.max_pj;
  return ((size_t)nl.n_chunks * mr + 2 * (size_t)nl.n_atoms * mr * n_vec) * sizeof(double2);
}

size_t nonlocal_scratch_bytes(const KPoint& kp, int n_vec) {
  const NonlocalK& nl = kp.nl;
  if (nl.n_atoms == 0 || nl.n_entries == 0) return 0;
  const size_t mr = 2 * nl.max_pj;
  const size_t n = nl_partial_rows(nl, n_vec) * mr + (size_t)nl.n_atoms * mr * n_vec;
  return n * sizeof(double2);  // the larger of the two precisions
}

// ============================================================================
// Adjoint: fields at the quadrature points and their cross densities
// ============================================================================
// One block per (cell, group of columns).  For CC columns at a time, the
// M^{-1/2}-scaled cell rows of L and Y (both spins) are gathered into LDS and
// interpolated to the quadrature points by sum factorisation over x, y, z
// (N_i = l_ax l_ay l_az); each thread then owns up to four points and
// accumulates, over the group's columns,
//   Re l^H y,  Re l^H sigma_x y,  Re l^H sigma_y y,  Re l^H sigma_z y,
// written (times w_q J) to partial[group][cell][point][4]; a second kernel adds
// the groups in a fixed order into dV, dB.
constexpr int kCdMaxQ = 4;   // points per thread: nq^3 <= 1024
// NS = 4 streams (L up, L down, Y up, Y down), or NS = 2 when L = Y (densities:
// the block is gathered and interpolated once).  colw: per-column weights (the
// occupations) or null; wJ: multiply by w_q J (the adjoint pairing) or not (the
// densities themselves).
template <int NS>
__global__ __launch_bounds__(256) void cross_density_kernel(
    const double2* __restrict__ L, int64_t ldl, const double2* __restrict__ Y, int64_t ldy, int n_vec,
    const int32_t* __restrict__ cell_nodes, const double* __restrict__ minv_sqrt,
    const double* __restrict__ B1, const double* __restrict__ wq1, double J, int np1, int nq, int nloc,
    int maxsz, int CC, int cols_per_group, const double* __restrict__ colw, int wJ,
    double* __restrict__ partial) {
  extern __shared__ double2 sm[];
  double2* bufA = sm;                               // [CC*NS][maxsz]
  double2* bufB = sm + (size_t)CC * NS * maxsz;     // [CC*NS][maxsz]
  double* sBt = reinterpret_cast<double*>(bufB + (size_t)CC * NS * maxsz);   // [np1][nq]
  const int e = blockIdx.x, g = blockIdx.y, tid = threadIdx.x;
  const int nq3 = nq * nq * nq;
  const int c_begin = g * cols_per_group, c_end = min(n_vec, c_begin + cols_per_group);
  for (int t = tid; t < np1 * nq; t += 256) sBt[t] = B1[t];
  double acc[kCdMaxQ][4];
#pragma unroll
  for (int i = 0; i < kCdMaxQ; ++i) acc[i][0] = acc[i][1] = acc[i][2] = acc[i][3] = 0.0;
  const int32_t* nodes = cell_nodes + (size_t)e * nloc;
  for (int n0 = c_begin; n0 < c_end; n0 += CC) {
    // gather: stream s = 2 * operand + spin
    for (int t = tid; t < CC * NS * nloc; t += 256) {
      const int i = t % nloc, s = (t / nloc) % NS, cc = t / (NS * nloc);
      const int col = n0 + cc;
      double2 v = {0.0, 0.0};
      if (col < c_end) {
        const int64_t I = nodes[i];
        const int64_t r = 2 * I + (s & 1);
        const double sc = minv_sqrt[I];
        const double2 z = (s < 2) ? L[r * ldl + col] : Y[r * ldy + col];
        v.x = sc * z.x;
        v.y = sc * z.y;
      }
      bufA[(size_t)(cc * NS + s) * maxsz + i] = v;
    }
    __syncthreads();
    // x: T1[qx + nq (ay + np az)] = sum_ax l_ax(qx) Z[ax + np (ay + np az)]
    for (int t = tid; t < CC * NS * nq * np1 * np1; t += 256) {
      const int o = t % (nq * np1 * np1), st = t / (nq * np1 * np1);
      const int qx = o % nq, rest = o / nq;
      const double2* in = bufA + (size_t)st * maxsz + rest * np1;
      double2 v = {0.0, 0.0};
      for (int ax = 0; ax < np1; ++ax) {
        const double b = sBt[ax * nq + qx];
        v.x += b * in[ax].x;
        v.y += b * in[ax].y;
      }
      bufB[(size_t)st * maxsz + o] = v;
    }
    __syncthreads();
    // y: T2[qx + nq (qy + nq az)] = sum_ay l_ay(qy) T1[qx + nq (ay + np az)]
    for (int t = tid; t < CC * NS * nq * nq * np1; t += 256) {
      const int o = t % (nq * nq * np1), st = t / (nq * nq * np1);
      const int qx = o % nq, qy = (o / nq) % nq, az = o / (nq * nq);
      const double2* in = bufB + (size_t)st * maxsz;
      double2 v = {0.0, 0.0};
      for (int ay = 0; ay < np1; ++ay) {
        const double b = sBt[ay * nq + qy];
        const double2 z = in[qx + nq * (ay + np1 * az)];
        v.x += b * z.x;
        v.y += b * z.y;
      }
      bufA[(size_t)st * maxsz + o] = v;
    }
    __syncthreads();
    // z: Zq[qx + nq (qy + nq qz)] = sum_az l_az(qz) T2[qx + nq (qy + nq az)]
    for (int t = tid; t < CC * NS * nq3; t += 256) {
      const int o = t % nq3, st = t / nq3;
      const int qxy = o % (nq * nq), qz = o / (nq * nq);
      const double2* in = bufA + (size_t)st * maxsz;
      double2 v = {0.0, 0.0};
      for (int az = 0; az < np1; ++az) {
        const double b = sBt[az * nq + qz];
        const double2 z = in[qxy + nq * nq * az];
        v.x += b * z.x;
        v.y += b * z.y;
      }
      bufB[(size_t)st * maxsz + o] = v;
    }
    __syncthreads();
#pragma unroll
    for (int qi = 0; qi < kCdMaxQ; ++qi) {
      const int q = tid + 256 * qi;
      if (q >= nq3) continue;
      for (int cc = 0; cc < CC; ++cc) {
        if (n0 + cc >= c_end) break;
        const double cw = colw ? colw[n0 + cc] : 1.0;
        const double2 l0 = bufB[(size_t)(cc * NS + 0) * maxsz + q], l1 = bufB[(size_t)(cc * NS + 1) * maxsz + q];
        const double2 y0 = bufB[(size_t)(cc * NS + NS - 2) * maxsz + q];
        const double2 y1 = bufB[(size_t)(cc * NS + NS - 1) * maxsz + q];
        // conj(l_a) y_b = (lr - i li)(yr + i yi)
        const double r00 = l0.x * y0.x + l0.y * y0.y, i00 = l0.x * y0.y - l0.y * y0.x;
        const double r11 = l1.x * y1.x + l1.y * y1.y, i11 = l1.x * y1.y - l1.y * y1.x;
        const double r01 = l0.x * y1.x + l0.y * y1.y, i01 = l0.x * y1.y - l0.y * y1.x;
        const double r10 = l1.x * y0.x + l1.y * y0.y, i10 = l1.x * y0.y - l1.y * y0.x;
        (void)i00;
        (void)i11;
        acc[qi][0] += cw * (r00 + r11);   // 1
        acc[qi][1] += cw * (r01 + r10);   // sigma_x
        acc[qi][2] += cw * (i01 - i10);   // sigma_y: Re(conj(l0)(-i y1) + conj(l1)(i y0))
        acc[qi][3] += cw * (r00 - r11);   // sigma_z
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int qi = 0; qi < kCdMaxQ; ++qi) {
    const int q = tid + 256 * qi;
    if (q >= nq3) continue;
    const int qx = q % nq, qy = (q / nq) % nq, qz = q / (nq * nq);
    const double w = wJ ? wq1[qx] * wq1[qy] * wq1[qz] * J : 1.0;
    double* out = partial + (((size_t)g * gridDim.x + e) * nq3 + q) * 4;
#pragma unroll
    for (int d = 0; d < 4; ++d) out[d] = w * acc[qi][d];
  }
}

// dV[e][q] += alpha sum_g partial[g][e][q][0], dB[e][q][d] += alpha sum_g partial[g][e][q][1 + d]
__global__ void cross_density_reduce_kernel(const double* __restrict__ partial, int64_t n_points, int n_groups,
                                            double alpha, double* __restrict__ dV, double* __restrict__ dB) {
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n_points;
       p += (int64_t)gridDim.x * blockDim.x) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int g = 0; g < n_groups; ++g)
#pragma unroll
      for (int d = 0; d < 4; ++d) s[d] += partial[((size_t)g * n_points + p) * 4 + d];
    dV[p] += alpha * s[0];
#pragma unroll
    for (int d = 0; d < 3; ++d) dB[p * 3 + d] += alpha * s[1 + d];
  }
}

// The same sums with n_q = n_p by sum factorisation.  A workgroup of 512
// threads owns one cell and a group of columns, and walks the group in chunks of
// CW columns of NS streams (NF = NS CW = 8 fields, one LDS buffer of n_p^3
// complex values per field: 44 KB at n_p = 7, two workgroups per CU).  Per chunk
// each thread loads the z-lines of its (column, stream, line) tasks straight into
// registers (column fastest, so neighbouring lanes read one row), interpolates
// along z there, and the y and x passes run in place in LDS; the next chunk's
// z-lines are loaded while the current chunk runs its LDS phases (LDS-only
// barriers).  tab = the matrix-free tables [B][Dq][w][even-odd tables].
// The n_groups column groups are interleaved (group g takes the chunks g,
// g + n_groups, ...) and n_groups is a multiple of the chunks that share a
// 128-byte row line, so the groups of one cell, neighbouring work items on one
// XCD, read the pieces of each line at the same time.  Work item bid -> column
// group bid % n_groups, cell order[bid / n_groups] (the densities' tiled order).
constexpr int kQfThreads = 512;
constexpr int qf_fields(int) { return 8; }

template <int NP, int NS>
__global__ __launch_bounds__(kQfThreads) void qfield_sf_kernel(
    const double2* __restrict__ L, int64_t ldl, const double2* __restrict__ Y, int64_t ldy, int n_vec,
    const int32_t* __restrict__ cell_nodes, const double* __restrict__ minv_sqrt, const double* __restrict__ tab,
    double J, int n_cells, int n_groups, const int32_t* __restrict__ order, const double* __restrict__ colw,
    int wJ, double* __restrict__ partial) {
  constexpr int NT = kQfThreads;
  constexpr int NF = qf_fields(NP), CW = NF / NS;
  constexpr int N2 = NP * NP, N3 = N2 * NP;
  constexpr int NTASK = NF * N2, TPT = (NTASK + NT - 1) / NT;
  constexpr int QPT = (N3 + NT - 1) / NT;
  extern __shared__ double2 qf_sm[];
  double2* buf = qf_sm;                 // [CW][NS][N3]
  const double* w1 = tab + 2 * N2;
  const double* eoBf = tab + 2 * N2 + NP;    // even-odd table of B (sf_eo)
  const int total = n_cells * n_groups;
  const int per_xcd = (total + 7) / 8;
  const int bid = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (bid >= total) return;
  const int g = bid % n_groups, e = order[bid / n_groups], tid = threadIdx.x;
  const int c_end = n_vec, c_step = CW * n_groups;
  const int32_t* nodes = cell_nodes + (size_t)e * N3;

  // the thread's tasks: (column offset c, stream s = 2 operand + spin, z-line l);
  // row pointers and M^{-1/2} factors are fixed over the chunks
  const double2* row[TPT][NP];
  double sc[TPT][NP];
  int tcol[TPT];
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    const int t = min(tid + NT * k, NTASK - 1);
    const int c = t % CW, s = (t / CW) % NS, l = t / (CW * NS);
    tcol[k] = c;
#pragma unroll
    for (int z = 0; z < NP; ++z) {
      const int64_t I = nodes[l + z * N2];
      const int64_t r = 2 * I + (s & 1);
      row[k][z] = (s < 2) ? L + r * ldl : Y + r * ldy;
      sc[k][z] = minv_sqrt[I];
    }
  }
  double2 zv[TPT][NP];
#pragma unroll
  for (int k = 0; k < TPT; ++k)
#pragma unroll
    for (int z = 0; z < NP; ++z) zv[k][z] = row[k][z][min(g * CW + tcol[k], c_end - 1)];

  double acc[QPT][4];
#pragma unroll
  for (int j = 0; j < QPT; ++j) acc[j][0] = acc[j][1] = acc[j][2] = acc[j][3] = 0.0;
  for (int n0 = g * CW; n0 < c_end; n0 += c_step) {
    double cwv[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) cwv[c] = (n0 + c < c_end) ? (colw ? colw[n0 + c] : 1.0) : 0.0;
    // interpolation along z in registers (zero past the last column)
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
      const int t = tid + NT * k;
      if (t >= NTASK) break;
      const int c = t % CW, s = (t / CW) % NS, l = t / (CW * NS);
      const bool ok = n0 + c < c_end;
      double2 u[NP];
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const double f = ok ? sc[k][i] : 0.0;
        u[i] = double2{f * zv[k][i].x, f * zv[k][i].y};
      }
      double2* out = buf + (c * NS + s) * N3 + l;
      double2 r[NP];
      sf_eo<double, NP, false>(eoBf, u, r);
#pragma unroll
      for (int o = 0; o < NP; ++o) out[o * N2] = r[o];
    }
    if (n0 + c_step < c_end) {
#pragma unroll
      for (int k = 0; k < TPT; ++k)
#pragma unroll
        for (int z = 0; z < NP; ++z) zv[k][z] = row[k][z][min(n0 + c_step + tcol[k], c_end - 1)];
    }
    lds_barrier();
    sf_line_pass<NP, NF, 1, NT>(eoBf, buf, buf);
    lds_barrier();
    sf_line_pass<NP, NF, 0, NT>(eoBf, buf, buf);
    lds_barrier();
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
      const int q = tid + NT * j;
      if (q >= N3) continue;
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const double cw = cwv[c];
        const double2 l0 = buf[(c * NS + 0) * N3 + q], l1 = buf[(c * NS + 1) * N3 + q];
        const double2 y0 = buf[(c * NS + NS - 2) * N3 + q], y1 = buf[(c * NS + NS - 1) * N3 + q];
        const double r00 = l0.x * y0.x + l0.y * y0.y;
        const double r11 = l1.x * y1.x + l1.y * y1.y;
        const double r01 = l0.x * y1.x + l0.y * y1.y, i01 = l0.x * y1.y - l0.y * y1.x;
        const double r10 = l1.x * y0.x + l1.y * y0.y, i10 = l1.x * y0.y - l1.y * y0.x;
        acc[j][0] += cw * (r00 + r11);
        acc[j][1] += cw * (r01 + r10);
        acc[j][2] += cw * (i01 - i10);
        acc[j][3] += cw * (r00 - r11);
      }
    }
    lds_barrier();   // the next chunk overwrites the buffer
  }
#pragma unroll
  for (int j = 0; j < QPT; ++j) {
    const int q = tid + NT * j;
    if (q >= N3) continue;
    const double w = wJ ? J * w1[q % NP] * w1[(q / NP) % NP] * w1[q / N2] : 1.0;
    double* out = partial + (((size_t)g * n_cells + e) * N3 + q) * 4;
#pragma unroll
    for (int d = 0; d < 4; ++d) out[d] = w * acc[j][d];
  }
}

// Densities (one operand, two spins) with n_q = n_p: a workgroup of 512 threads
// owns one cell and one of n_groups interleaved column groups (group g takes the
// chunks of DC = 4 columns g, g + n_groups, ...) and walks it chunk by chunk,
// both spins at once (8 LDS fields of n_p^3 values, 44 KB at n_p = 7).  A
// chunk's z-line loads cover 4 consecutive columns of a row, half a 128-byte
// line: the group holding the other half is the neighbouring work item, which
// runs at the same time on the same XCD, so each line is fetched once.
// M^{-1/2} at the cell's nodes sits in LDS, so the kernel stays within 128
// VGPRs at n_p <= 7 and two workgroups share a CU.  The LDS fields are padded
// (den_px, den_fp: x extent and field gap per n_p) so that the eight lanes of
// a 128-bit LDS access hit distinct banks in the line passes (at n_p = 7 the
// compact layout puts two lanes of every eight on one bank in the y pass).  The next chunk's z-lines are
// loaded while the current one runs its LDS phases (LDS-only barriers).  Work
// item bid -> column group bid % n_groups, cell order[bid / n_groups] (4x4x4
// tiles of cells, tile after tile; each XCD takes a contiguous range, so the
// workgroups resident on an XCD hold a compact block of cells and their shared
// face nodes meet in its L2).  Output as qfield_sf_kernel (no quadrature weights).
constexpr int kDenCols = 4;
constexpr int kDenTile = 4;
constexpr int den_px(int NP) { return NP <= 3 ? NP : NP <= 6 ? 7 : 9; }
constexpr int den_fp(int NP) {
  return NP == 2 ? 1 : NP == 4 ? 1 : NP == 5 ? 6 : NP == 6 ? 11 : NP == 8 ? 1 : NP == 9 ? 6 : 0;
}
constexpr int den_field(int NP) { return den_px(NP) * NP * NP + den_fp(NP); }

template <int NP>
__global__ __launch_bounds__(kQfThreads) void density_sf_kernel(
    const double2* __restrict__ X, int64_t ldx, int n_vec, const int32_t* __restrict__ cell_nodes,
    const int32_t* __restrict__ order, const double* __restrict__ minv_sqrt, const double* __restrict__ tab,
    int n_cells, int n_groups, const double* __restrict__ colw, double* __restrict__ partial) {
  constexpr int NT = kQfThreads, DC = kDenCols, NF = 2 * DC;
  constexpr int N2 = NP * NP, N3 = N2 * NP;
  constexpr int NTASK = NF * N2, TPT = (NTASK + NT - 1) / NT;
  constexpr int QPT = (N3 + NT - 1) / NT;
  constexpr int SY = den_px(NP), SZ = SY * NP, SF = den_field(NP);
  static_assert(SY >= NP && (NP - 1) * (1 + SY + SZ) < SF, "padded field layout overlaps");
  extern __shared__ double2 den_sm[];
  double2* buf = den_sm;                                    // [DC][2 spins][SF]
  double* ssc = reinterpret_cast<double*>(buf + NF * SF);   // [N3] M^{-1/2} at the cell's nodes
  const double* eoBf = tab + 2 * N2 + NP;
  const int total = n_cells * n_groups;
  const int per_xcd = (total + 7) / 8;
  const int bid = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (bid >= total) return;
  const int g = bid % n_groups, e = order[bid / n_groups], tid = threadIdx.x;
  const int c_end = n_vec, c_step = DC * n_groups;
  const int32_t* nodes = cell_nodes + (size_t)e * N3;
  for (int i = tid; i < N3; i += NT) ssc[i] = minv_sqrt[nodes[i]];

  // the thread's z-line tasks: column offset c fastest, then the spin, then the line
  int32_t nd[TPT][NP];
#pragma unroll
  for (int k = 0; k < TPT; ++k) {
    const int t = min(tid + NT * k, NTASK - 1);
    const int l = t / NF;
#pragma unroll
    for (int z = 0; z < NP; ++z) nd[k][z] = nodes[l + z * N2];
  }
  auto zload = [&](int n0, double2 (&zv)[TPT][NP]) {
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
      const int t = min(tid + NT * k, NTASK - 1);
      const int col = min(n0 + t % DC, c_end - 1);
      const int sp = (t / DC) & 1;
#pragma unroll
      for (int z = 0; z < NP; ++z) zv[k][z] = X[(2 * (int64_t)nd[k][z] + sp) * ldx + col];
    }
  };
  double2 zv[TPT][NP];
  zload(g * DC, zv);
  double acc[QPT][4];
#pragma unroll
  for (int j = 0; j < QPT; ++j) acc[j][0] = acc[j][1] = acc[j][2] = acc[j][3] = 0.0;
  lds_barrier();                          // ssc is written
  for (int n0 = g * DC; n0 < c_end; n0 += c_step) {
    // z interpolation in registers (zero past the last column) into LDS
#pragma unroll
    for (int k = 0; k < TPT; ++k) {
      const int t = tid + NT * k;
      if (t >= NTASK) break;
      const int c = t % DC, sp = (t / DC) & 1, l = t / NF;
      const bool ok = n0 + c < c_end;
      double2 u[NP];
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const double f = ok ? ssc[l + i * N2] : 0.0;
        u[i] = double2{f * zv[k][i].x, f * zv[k][i].y};
      }
      double2* out = buf + (2 * c + sp) * SF + (l % NP) + (l / NP) * SY;
      double2 r[NP];
      sf_eo<double, NP, false>(eoBf, u, r);
#pragma unroll
      for (int o = 0; o < NP; ++o) out[o * SZ] = r[o];
    }
    if (n0 + c_step < c_end) zload(n0 + c_step, zv);
    lds_barrier();
    sf_line_pass<NP, NF, 1, NT, double, SY, SZ, SF>(eoBf, buf, buf);
    lds_barrier();
    sf_line_pass<NP, NF, 0, NT, double, SY, SZ, SF>(eoBf, buf, buf);
    lds_barrier();
#pragma unroll
    for (int j = 0; j < QPT; ++j) {
      const int q = tid + NT * j;
      if (q >= N3) continue;
      const int pq = (q % NP) + ((q / NP) % NP) * SY + (q / N2) * SZ;
#pragma unroll
      for (int c = 0; c < DC; ++c) {
        const double cw = (n0 + c < c_end) ? (colw ? colw[n0 + c] : 1.0) : 0.0;
        const double2 u0 = buf[(2 * c) * SF + pq], u1 = buf[(2 * c + 1) * SF + pq];
        const double r00 = u0.x * u0.x + u0.y * u0.y;
        const double r11 = u1.x * u1.x + u1.y * u1.y;
        const double r01 = u0.x * u1.x + u0.y * u1.y, i01 = u0.x * u1.y - u0.y * u1.x;
        acc[j][0] += cw * (r00 + r11);
        acc[j][1] += cw * (2.0 * r01);       // u^H sigma_x u
        acc[j][2] += cw * (2.0 * i01);       // u^H sigma_y u
        acc[j][3] += cw * (r00 - r11);       // u^H sigma_z u
      }
    }
    lds_barrier();   // the next round overwrites the buffer
  }
#pragma unroll
  for (int j = 0; j < QPT; ++j) {
    const int q = tid + NT * j;
    if (q >= N3) continue;
    double* out = partial + (((size_t)g * n_cells + e) * N3 + q) * 4;
#pragma unroll
    for (int d = 0; d < 4; ++d) out[d] = acc[j][d];
  }
}

// The cell order of density_sf_kernel: tiles of kDenTile^3 cells (ragged at
// the edges), tile after tile, cells within a tile x fastest.
static void den_order_prepare(chfsi_ctx* c) {
  if (c->den_order.ptr && c->den_order.n == (size_t)c->n_cells) return;
  constexpr int T = kDenTile;
  std::vector<int32_t> ord;
  ord.reserve(c->n_cells);
  const int nx = c->nc[0], ny = c->nc[1], nz = c->nc[2];
  for (int tz = 0; tz < nz; tz += T)
    for (int ty = 0; ty < ny; ty += T)
      for (int tx = 0; tx < nx; tx += T)
        for (int z = tz; z < std::min(nz, tz + T); ++z)
          for (int y = ty; y < std::min(ny, ty + T); ++y)
            for (int x = tx; x < std::min(nx, tx + T); ++x) ord.push_back(x + nx * (y + ny * z));
  CHFSI_CHECK((int64_t)ord.size() == c->n_cells, CHFSI_EINVAL, "densities: cell order does not cover the mesh");
  c->den_order.release();
  c->den_order.upload(ord.data(), ord.size(), c->stream);
  CHFSI_HIP(hipStreamSynchronize(c->stream));   // the host vector ends here
}

template <int NP>
static void launch_density_sf(chfsi_ctx* c, const double2* X, int64_t ldx, int n_vec, const double* colw,
                              double* rho, double* mag) {
  constexpr int DC = kDenCols;
  constexpr int N3 = NP * NP * NP;
  const size_t sh = (size_t)2 * DC * den_field(NP) * sizeof(double2) + (size_t)N3 * sizeof(double);
  if (c->mf_tab.n == 0) mf_prepare(c);
  den_order_prepare(c);
  // at least two groups (the two halves of each 128-byte row line), more on
  // small meshes to fill the GPU; every group holds at least one chunk
  const int n_chunks = cdiv(n_vec, DC);
  const int want = std::max(2, cdiv(4096, std::max(1, c->n_cells)));
  const int groups = std::max(1, std::min(n_chunks, want));
  const int64_t n_points = (int64_t)c->n_cells * c->nq3;
  c->cd_partial.alloc((size_t)groups * n_points * 4);
  const int64_t total = (int64_t)c->n_cells * groups;
  CHFSI_CHECK(total < (int64_t)1 << 30, CHFSI_EINVAL, "densities: too many work items");
  StageTimer tm(c, CHFSI_STAGE_AXPY, 0.0, 0.0, (double)c->n_cells * c->nloc * 2.0 * n_vec * sizeof(double2));
  hipLaunchKernelGGL((density_sf_kernel<NP>), dim3((unsigned)(8 * ((total + 7) / 8))), dim3(kQfThreads), sh,
                     c->stream, X, ldx, n_vec, c->cell_nodes.ptr, c->den_order.ptr, c->minv_sqrt.ptr,
                     c->mf_tab.ptr, c->n_cells, groups, colw, c->cd_partial.ptr);
  LAUNCH_CHECK();
  hipLaunchKernelGGL(cross_density_reduce_kernel, dim3((unsigned)std::min<int64_t>(cdiv(n_points, 256), 4096)),
                     dim3(256), 0, c->stream, c->cd_partial.ptr, n_points, groups, 1.0, rho, mag);
  LAUNCH_CHECK();
}

template <int NP, int NS>
static void launch_qfield_sf(chfsi_ctx* c, const double2* L, int64_t ldl, const double2* Y, int64_t ldy,
                             int n_vec, const double* colw, int wJ, double alpha, double* dV, double* dB) {
  constexpr int CW = qf_fields(NP) / NS;
  const size_t sh = (size_t)qf_fields(NP) * NP * NP * NP * sizeof(double2);
  if (c->mf_tab.n == 0) mf_prepare(c);
  den_order_prepare(c);
  // a multiple of the chunks that share a 128-byte row line (8 complex values),
  // at least 4096 work items where the columns allow; each group holds a chunk
  constexpr int LQ = 8 / CW > 1 ? 8 / CW : 1;
  const int n_chunks = cdiv(n_vec, CW);
  const int want = LQ * cdiv(std::max(1, cdiv(4096, std::max(1, c->n_cells))), LQ);
  const int groups = std::max(1, std::min(n_chunks, want));
  const int64_t n_points = (int64_t)c->n_cells * c->nq3;
  c->cd_partial.alloc((size_t)groups * n_points * 4);
  const int64_t total = (int64_t)c->n_cells * groups;
  CHFSI_CHECK(total < (int64_t)1 << 30, CHFSI_EINVAL, "quadrature-point fields: too many work items");
  StageTimer tm(c, CHFSI_STAGE_AXPY, 0.0, 0.0, (double)NS / 2 * c->n_cells * c->nloc * 2.0 * n_vec * sizeof(double2));
  hipLaunchKernelGGL((qfield_sf_kernel<NP, NS>), dim3((unsigned)(8 * ((total + 7) / 8))), dim3(kQfThreads), sh,
                     c->stream, L, ldl, Y, ldy, n_vec, c->cell_nodes.ptr, c->minv_sqrt.ptr, c->mf_tab.ptr, c->J,
                     c->n_cells, groups, c->den_order.ptr, colw, wJ, c->cd_partial.ptr);
  LAUNCH_CHECK();
  hipLaunchKernelGGL(cross_density_reduce_kernel, dim3((unsigned)std::min<int64_t>(cdiv(n_points, 256), 4096)),
                     dim3(256), 0, c->stream, c->cd_partial.ptr, n_points, groups, alpha, dV, dB);
  LAUNCH_CHECK();
}

// n_q = n_p: sum-factorised line passes; otherwise the general kernel below.
template <int NS>
static bool qfield_fast(chfsi_ctx* c, const double2* L, int64_t ldl, const double2* Y, int64_t ldy, int n_vec,
                        const double* colw, int wJ, double alpha, double* dV, double* dB) {
  if (c->nq != c->np1) return false;
  switch (c->np1) {
    case 2: launch_qfield_sf<2, NS>(c, L, ldl, Y, ldy, n_vec, colw, wJ, alpha, dV, dB); return true;
    case 3: launch_qfield_sf<3, NS>(c, L, ldl, Y, ldy, n_vec, colw, wJ, alpha, dV, dB); return true;
    case 4: launch_qfield_sf<4, NS>(c, L, ldl, Y, ldy, n_vec, colw, wJ, alpha, dV, dB); return true;
    case 5: launch_qfield_sf<5, NS>(c, L, ldl, Y, ldy, n_vec, colw, wJ, alpha, dV, dB); return true;
    case 6: launch_qfield_sf<6, NS>(c, L, ldl, Y, ldy, n_vec, colw, wJ, alpha, dV, dB); return true;
    case 7: launch_qfield_sf<7, NS>(c, L, ldl, Y, ldy, n_vec, colw, wJ, alpha, dV, dB); return true;
    case 8: launch_qfield_sf<8, NS>(c, L, ldl, Y, ldy, n_vec, colw, wJ, alpha, dV, dB); return true;
    case 9: launch_qfield_sf<9, NS>(c, L, ldl, Y, ldy, n_vec, colw, wJ, alpha, dV, dB); return true;
    default: return false;
  }
}

// Shared launcher: partial sums per (cell, column group), then the fixed-order
// group reduction adding alpha * (sums) into (dV, dB).
template <int NS>
static void launch_cross_density(chfsi_ctx* c, const double2* L, int64_t ldl, const double2* Y, int64_t ldy,
                                 int n_vec, const double* colw, int wJ, double alpha, double* dV, double* dB) {
  if (qfield_fast<NS>(c, L, ldl, Y, ldy, n_vec, colw, wJ, alpha, dV, dB)) return;
  const int np1 = c->np1, nq = c->nq;
  const int maxsz = std::max(std::max(c->nloc, nq * np1 * np1), std::max(nq * nq * np1, c->nq3));
  CHFSI_CHECK(c->nq3 <= 256 * kCdMaxQ, CHFSI_EINVAL, "quadrature-point fields support n_q <= 10");
  const size_t per_cc = 2 * NS * (size_t)maxsz * sizeof(double2);
  const size_t budget = 128 * 1024;
  const int CC = (int)std::max<size_t>(1, std::min<size_t>(4, budget / per_cc));
  const size_t sh = CC * per_cc + np1 * nq * sizeof(double);
  CHFSI_CHECK(sh <= 160 * 1024, CHFSI_EINVAL, "quadrature-point fields: cell too large for LDS");
  if (c->ref_b1.n == 0) {
    c->ref_b1.upload(c->ref.B.data(), c->ref.B.size(), c->stream);
    c->ref_wq.upload(c->ref.wq.data(), c->ref.wq.size(), c->stream);
  }
  // column groups: enough (cell, group) blocks to fill the GPU, whole CC chunks each
  const int max_groups = std::max(1, cdiv(n_vec, CC));
  const int want = std::max(1, cdiv(4096, std::max(1, c->n_cells)));
  int groups = std::min(max_groups, want);
  const int cpg = CC * cdiv(cdiv(n_vec, groups), CC);
  groups = cdiv(n_vec, cpg);
  const int64_t n_points = (int64_t)c->n_cells * c->nq3;
  c->cd_partial.alloc((size_t)groups * n_points * 4);
  StageTimer tm(c, CHFSI_STAGE_AXPY, 0.0, 0.0, (double)NS / 2 * c->n_cells * c->nloc * 2.0 * n_vec * sizeof(double2));
  hipLaunchKernelGGL(cross_density_kernel<NS>, dim3(c->n_cells, groups), dim3(256), sh, c->stream, L, ldl, Y,
                     ldy, n_vec, c->cell_nodes.ptr, c->minv_sqrt.ptr, c->ref_b1.ptr, c->ref_wq.ptr, c->J, np1, nq,
                     c->nloc, maxsz, CC, cpg, colw, wJ, c->cd_partial.ptr);
  LAUNCH_CHECK();
  hipLaunchKernelGGL(cross_density_reduce_kernel, dim3((unsigned)std::min<int64_t>(cdiv(n_points, 256), 4096)),
                     dim3(256), 0, c->stream, c->cd_partial.ptr, n_points, groups, alpha, dV, dB);
  LAUNCH_CHECK();
}

void cross_density(chfsi_ctx* c, const double2* L, int64_t ldl, const double2* Y, int64_t ldy, int n_vec,
                   double alpha, double* dV, double* dB) {
  launch_cross_density<4>(c, L, ldl, Y, ldy, n_vec, nullptr, 1, alpha, dV, dB);
}

void densities(chfsi_ctx* c, const double2* X, int64_t ldx, int n_vec, const double* occ_d, double* rho,
               double* mag) {
  if (c->nq == c->np1) {
    switch (c->np1) {
      case 2: launch_density_sf<2>(c, X, ldx, n_vec, occ_d, rho, mag); return;
      case 3: launch_density_sf<3>(c, X, ldx, n_vec, occ_d, rho, mag); return;
      case 4: launch_density_sf<4>(c, X, ldx, n_vec, occ_d, rho, mag); return;
      case 5: launch_density_sf<5>(c, X, ldx, n_vec, occ_d, rho, mag); return;
      case 6: launch_density_sf<6>(c, X, ldx, n_vec, occ_d, rho, mag); return;
      case 7: launch_density_sf<7>(c, X, ldx, n_vec, occ_d, rho, mag); return;
      case 8: launch_density_sf<8>(c, X, ldx, n_vec, occ_d, rho, mag); return;
      case 9: launch_density_sf<9>(c, X, ldx, n_vec, occ_d, rho, mag); return;
      default: break;
    }
  }
  launch_cross_density<2>(c, X, ldx, X, ldx, n_vec, occ_d, 0, 1.0, rho, mag);
}

// ============================================================================
// Dense tall-skinny products (FP64 MFMA) for CholGS and Rayleigh-Ritz
// ============================================================================
// Both products run on one LDS-staged tile engine: workgroup tile 64 x 64
// complex outputs, 4 waves of 32 x 32 (2 x 2 blocks of 16 x 16, 4 real MFMAs
// per complex block and k-step of 4), k staged through LDS in double-buffered
// stages of 8, k-major ([k][m] and [k][n]) so that every fragment read is 16
// consecutive complex values.  The next stage's global loads are issued before
// the current stage's MFMAs.  Bound by the FP64 matrix rate: the tile's size only
// sets the cache reads per MFMA, and against 128 x 64 less of it lies above the
// diagonal of a triangular product and three or four workgroups fit a CU, so that
// fewer rows still fill the GPU.  On 432000 rows x 384 columns: Gram product 5.9 ->
// 5.0 ms (matrix units 77 % busy), triangular rotation 8.4 (with the copies of its
// panels) -> 5.0 ms; 250000 x 256: Gram 2.4 -> 1.4, full rotation 2.7 either way.
constexpr int kGM = 64, kGN = 64, kGK = 8, kGPad = 2;   // pad: k rows 4 apart on other banks
constexpr int kGSlots = 1024;    // workgroups of one round: 4 on each of 256 CUs

// MB: 16-row blocks per wave (2: the tile of 64 rows)
template <int MB = 2>
struct GemmSmem {
  double2 a[2][kGK][32 * MB + kGPad];
  double2 b[2][kGK][kGN + kGPad];
};

// Tile t of an n x n product; triangular: the tiles (i, j <= i) row by row
// (whole products: any height of tile)
__device__ __forceinline__ int2 gram_tile(int t, int n, int lower) {
  if (!lower) {
    const int nt = (n + kGN - 1) / kGN;
    return int2{t / nt, t % nt};
  }
  int i = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while (i * (i + 1) / 2 > t) --i;
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  return int2{i, t - i * (i + 1) / 2};
}

// acc[mb][nb] (re, im) += op(A) B over one LDS stage; CONJ: op(A) = conj(A)
template <bool CONJ, int MB>
__device__ __forceinline__ void gemm_stage(const GemmSmem<MB>& sm, int buf, int wm, int wn, int lane, d4 (&cr)[MB][2],
                                           d4 (&ci)[MB][2]) {
  const int kl = lane >> 4, il = lane & 15;
#pragma unroll
  for (int ks = 0; ks < kGK / 4; ++ks) {
    double2 fa[MB], fb[2];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) fa[mb] = sm.a[buf][ks * 4 + kl][wm * (16 * MB) + mb * 16 + il];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) fb[nb] = sm.b[buf][ks * 4 + kl][wn * 32 + nb * 16 + il];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const double ar = fa[mb].x, ai = CONJ ? -fa[mb].y : fa[mb].y, nai = -ai;
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        cr[mb][nb] = mfma(ar, fb[nb].x, cr[mb][nb]);
        cr[mb][nb] = mfma(nai, fb[nb].y, cr[mb][nb]);
        ci[mb][nb] = mfma(ar, fb[nb].y, ci[mb][nb]);
        ci[mb][nb] = mfma(ai, fb[nb].x, ci[mb][nb]);
      }
    }
  }
}

// Partial S = X^H Y over row ranges, lower-triangle tiles only when asked.
// Work item = (tile, row range g), the items of one range consecutive on one XCD,
// so the tiles reading the same rows share that XCD's L2.  partial[g] holds the
// range's n x n sum.  A wave whose block lies above the diagonal of a triangular
// product has nothing to do but its share of the staging.
template <int MB>
__global__ __launch_bounds__(256, MB == 2 ? 4 : 2) void gram_kernel(const double2* __restrict__ X, int64_t ldx,
                                                      const double2* __restrict__ Y, int64_t ldy, int64_t rows,
                                                      int n, int64_t range_rows, int n_groups, int n_tiles,
                                                      int lower, double2* __restrict__ partial) {
  __shared__ GemmSmem<MB> sm;
  const int n_work = n_tiles * n_groups;
  const int per_xcd = (int)((gridDim.x + 7) / 8);
  const int bid = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if (bid >= n_work) return;              // uniform over the block, before any barrier
  const int g = bid / n_tiles;
  const int2 tl = gram_tile(bid - g * n_tiles, n, lower);
  const int i0 = tl.x * (32 * MB), j0 = tl.y * kGN;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave & 1, wn = wave >> 1;
  const bool busy = !lower || i0 + (wm + 1) * (16 * MB) - 1 >= j0 + wn * 32;
  // staging map: 8 rows x 32 MB or 64 columns of the operands, MB or 2 per thread, columns
  // (tid & 31) + 32 u, so each LDS store writes 32 consecutive elements of a row
  // (no bank conflicts) and each load reads 512 B
  const int sk = tid >> 5, sc = tid & 31;
  d4 cr[MB][2], ci[MB][2];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) cr[mb][nb] = ci[mb][nb] = d4{0, 0, 0, 0};
  double2 pa[MB], pb[2];
  const int64_t r_begin = g * range_rows;
  const int64_t r_end = r_begin + range_rows < rows ? r_begin + range_rows : rows;
  auto gload = [&](int64_t r0) {
    const int64_t r = r0 + sk;
    const bool rv = r < r_end;
    const double2* xp = X + (rv ? r : 0) * ldx;
    const double2* yp = Y + (rv ? r : 0) * ldy;
#pragma unroll
    for (int u = 0; u < MB; ++u) {
      const int c = i0 + sc + 32 * u;
      pa[u] = (rv && c < n) ? xp[c] : double2{0.0, 0.0};
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int d = j0 + sc + 32 * u;
      pb[u] = (rv && d < n) ? yp[d] : double2{0.0, 0.0};
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int u = 0; u < MB; ++u) sm.a[buf][sk][sc + 32 * u] = pa[u];
#pragma unroll
    for (int u = 0; u < 2; ++u) sm.b[buf][sk][sc + 32 * u] = pb[u];
  };
  const int nst = (int)((r_end - r_begin + kGK - 1) / kGK);
  gload(r_begin);
  lstore(0);
  __syncthreads();
  for (int st = 0; st < nst; ++st) {
    const int buf = st & 1;
    const bool more = st + 1 < nst;
    if (more) gload(r_begin + (int64_t)(st + 1) * kGK);
    if (busy) gemm_stage<true, MB>(sm, buf, wm, wn, lane, cr, ci);
    if (more) lstore(buf ^ 1);            // that buffer was last read before the previous barrier
    __syncthreads();
  }
  double2* out = partial + (size_t)g * n * n;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int ri = i0 + wm * (16 * MB) + mb * 16 + acc_row<double>(lane, j);
        const int cj = j0 + wn * 32 + nb * 16 + (lane & 15);
        if (ri < n && cj < n) out[(size_t)ri * n + cj] = double2{cr[mb][nb][j], ci[mb][nb][j]};
      }
}

// S[i][j] = sum over ranges of partial[g][i][j] for the (i, j) of the tiles; one
// workgroup takes four rows of a tile (one element per thread: one workgroup per
// tile left the GPU idle, 353 -> 13 us at n = 384)
__global__ __launch_bounds__(256) void gram_reduce_kernel(const double2* __restrict__ partial, int n_groups, int n,
                                                          int lower, double2* __restrict__ S) {
  const int2 tl = gram_tile(blockIdx.x, n, lower);
  const int i = tl.x * kGM + blockIdx.y * 4 + (threadIdx.x >> 6), j = tl.y * kGN + (threadIdx.x & 63);
  if (i >= n || j >= n) return;
  const double2* p = partial + (size_t)i * n + j;
  const size_t nn = (size_t)n * n;
  double2 s = {0.0, 0.0};
#pragma unroll 8
  for (int g = 0; g < n_groups; ++g) {
    const double2 v = p[g * nn];
    s.x += v.x;
    s.y += v.y;
  }
  S[(size_t)i * n + j] = s;
}

// Tiles and row ranges of a Gram product.  Ranges: one round of workgroups, cut at whole
// stages; past half a round of tiles the count of at most four that fills its rounds best.
// Whole products of many columns take tiles of 128 rows, 2 workgroups on a CU, where the
// columns past n and the last round's idle places do not undo a twentieth less per element
// (a quarter less LDS traffic per MFMA): on 432000 rows 600 columns 23.0 against 24.5 ms,
// 1000 59.0 and 62.2, but 800, seven tiles of 128 for 6.25, 41.6 with tiles of 64.
// Triangular products would lose more above the diagonal.
static GramShape gram_ranges(int64_t rows, int64_t tiles, int64_t slots) {
  GramShape g;
  const auto fill = [&](int64_t k) { return (double)(tiles * k) / (double)((tiles * k + slots - 1) / slots * slots); };
  int64_t groups = std::max<int64_t>(1, slots / tiles);
  if (groups == 1)
    for (int64_t k = 2; k <= 4; ++k)
      if (fill(k) > 1.05 * fill(groups)) groups = k;
  groups = std::min<int64_t>(groups, std::max<int64_t>(1, rows / 64));
  g.high = false;
  g.tiles = tiles;
  g.range_rows = (cdiv(rows, groups) + kGK - 1) / kGK * kGK;
  g.groups = std::max(1, cdiv(rows, g.range_rows));
  g.cost = (double)tiles / fill(g.groups);
  return g;
}

GramShape gram_shape(int64_t rows, int n, bool lower_only) {
  const int64_t nt = cdiv(n, kGM);
  const GramShape g = gram_ranges(rows, lower_only ? nt * (nt + 1) / 2 : nt * nt, kGSlots);
  if (lower_only || n < 512) return g;
  GramShape h = gram_ranges(rows, cdiv(n, 2 * kGM) * nt, kGSlots / 2);
  h.high = true;
  return 2.0 * 0.95 * h.cost < g.cost ? h : g;
}

// S = X^H Y on the device (its lower triangle): in c->scratch, which is grown for
// `extra` doubles behind it
double2* gram_device(chfsi_ctx* c, const double2* X, int64_t ldx, const double2* Y, int64_t ldy, int64_t rows, int n,
                     bool lower_only, size_t extra) {
  const GramShape g = gram_shape(rows, n, lower_only);
  const size_t nn = (size_t)n * n;
  CHFSI_CHECK(g.tiles * g.groups < (int64_t)1 << 30, CHFSI_EINVAL, "Gram product: too many columns");
  c->scratch.alloc(2 * nn * (g.groups + 1) + extra);
  double2* partial = reinterpret_cast<double2*>(c->scratch.ptr);
  double2* Sd = partial + g.groups * nn;
  StageTimer tm(c, CHFSI_STAGE_GRAM, 8.0 * (double)rows * n * n * (lower_only ? 0.5 : 1.0),
                8.0 * (double)rows * kGM * kGN * g.tiles * (g.high ? 2 : 1), 2.0 * (double)rows * n * sizeof(double2));
  const int64_t n_work = g.tiles * g.groups;
  const dim3 grid(8 * cdiv(n_work, 8));
  if (g.high)
    hipLaunchKernelGGL(gram_kernel<4>, grid, dim3(256), 0, c->stream, X, ldx, Y, ldy, rows, n, g.range_rows, g.groups,
                       (int)g.tiles, 0, partial);
  else
    hipLaunchKernelGGL(gram_kernel<2>, grid, dim3(256), 0, c->stream, X, ldx, Y, ldy, rows, n, g.range_rows, g.groups,
                       (int)g.tiles, lower_only ? 1 : 0, partial);
  LAUNCH_CHECK();
  const int nt = cdiv(n, kGN);
  hipLaunchKernelGGL(gram_reduce_kernel, dim3(lower_only ? nt * (nt + 1) / 2 : nt * nt, kGM / 4), dim3(256), 0, c->stream,
                     partial, g.groups, n, lower_only ? 1 : 0, Sd);
  LAUNCH_CHECK();
  return Sd;
}

void gram(chfsi_ctx* c, const double2* X, int64_t ldx, const double2* Y, int64_t ldy, int64_t rows,
          int n, std::vector<cplx>& S, bool lower_only) {
  const double2* Sd = gram_device(c, X, ldx, Y, ldy, rows, n, lower_only, 0);
  std::vector<double2> h((size_t)n * n);
  CHFSI_HIP(hipMemcpyAsync(h.data(), Sd, (size_t)n * n * sizeof(double2), hipMemcpyDeviceToHost, c->stream));
  CHFSI_HIP(hipStreamSynchronize(c->stream));
  S.resize((size_t)n * n);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) {
      if (lower_only && j > i)
        S[(size_t)i * n + j] = std::conj(cplx(h[(size_t)j * n + i].x, h[(size_t)j * n + i].y));
      else
        S[(size_t)i * n + j] = cplx(h[(size_t)i * n + j].x, h[(size_t)i * n + j].y);
    }
}

// One 64 x 64 tile of P Q: rows r0.. of P (valid below prow), columns j0.., k below
// kend, into X.  trim: the tile crosses Q's diagonal, a wave's k range ends at its
// own last column.
__device__ __forceinline__ void rotate_tile(GemmSmem<>& sm, const double2* P, int64_t ldp, int64_t r0, int64_t prow,
                                            const double2* __restrict__ Q, int n, int j0, int kend, int trim,
                                            double2* X, int64_t ldx) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave & 1, wn = wave >> 1;
  // staging map: A 64 rows x 8 k (rows (tid >> 3) + 32 u: eight lanes read the 128
  // bytes of a row, and the k-major stores of 16 lanes hit all banks once), B 8 rows
  // of Q x 64 columns (columns (tid & 31) + 32 u)
  const int am = tid >> 3, ak = tid & 7;
  const int bk = tid >> 5, bn = tid & 31;
  const double2* pp = P + (r0 + am) * ldp + ak;
  const int64_t pstep = 32 * ldp;
  const double2* qp = Q + (size_t)bk * n + j0 + bn;
  const int64_t qstep = (int64_t)kGK * n;
  const int my_end = trim ? j0 + wn * 32 + 32 : kend;
  d4 cr[2][2], ci[2][2];
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) cr[mb][nb] = ci[mb][nb] = d4{0, 0, 0, 0};
  double2 pa[2], pb[2];
  auto gload = [&](int k0) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      pa[u] = (r0 + am + 32 * u < prow && k0 + ak < kend) ? pp[u * pstep] : double2{0.0, 0.0};
      pb[u] = (k0 + bk < kend && j0 + bn + 32 * u < n) ? qp[32 * u] : double2{0.0, 0.0};
    }
    pp += kGK;
    qp += qstep;
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      sm.a[buf][ak][am + 32 * u] = pa[u];
      sm.b[buf][bk][bn + 32 * u] = pb[u];
    }
  };
  const int nst = (kend + kGK - 1) / kGK;
  gload(0);
  lstore(0);
  __syncthreads();
  for (int st = 0; st < nst; ++st) {
    const int buf = st & 1;
    const bool more = st + 1 < nst;
    if (more) gload((st + 1) * kGK);
    if (st * kGK < my_end) gemm_stage<false, 2>(sm, buf, wm, wn, lane, cr, ci);
    if (more) lstore(buf ^ 1);
    __syncthreads();                      // the last one: every read of P and sm is done
  }
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t r = r0 + wm * 32 + mb * 16 + acc_row<double>(lane, j);
        const int cj = j0 + wn * 32 + nb * 16 + (lane & 15);
        if (r < prow && cj < n) X[r * ldx + cj] = double2{cr[mb][nb][j], ci[mb][nb][j]};
      }
}

// X[r][:] = P[r][:] Q over a row panel P (a copy of those rows of X).  Work item =
// (row tile, column tile), the column tiles of one row tile on one XCD, so that they read
// its panel rows through one L2.  UPPER (Q upper triangular): a column tile's k range ends
// with it; an XCD takes its row tiles' last column tiles first, the long ranges before the
// short ones.
template <bool UPPER>
__global__ __launch_bounds__(256, 4) void rotate_kernel(const double2* __restrict__ P, int n, int64_t prow,
                                                        const double2* __restrict__ Q, double2* __restrict__ X,
                                                        int64_t ldx, int n_rt, int n_ct) {
  __shared__ GemmSmem<> sm;
  const int xcd = (int)(blockIdx.x % 8), i = (int)(blockIdx.x / 8);
  int rt, ct;
  if (UPPER) {
    const int per_rt = (n_rt + 7) / 8;
    rt = xcd * per_rt + i % per_rt;
    ct = n_ct - 1 - i / per_rt;
  } else {
    const int bid = xcd * (int)((gridDim.x + 7) / 8) + i;
    rt = bid / n_ct;
    ct = bid - rt * n_ct;
  }
  if (rt >= n_rt || ct < 0) return;       // uniform over the block, before any barrier
  const int kend = UPPER && (ct + 1) * kGN < n ? (ct + 1) * kGN : n;
  rotate_tile(sm, P, n, (int64_t)rt * kGM, prow, Q, n, ct * kGN, kend, UPPER, X, ldx);
}

// X <- X Q in place, Q upper triangular: a workgroup owns 64 rows and takes its
// column tiles from the last to the first.  A tile reads columns up to its own last
// one and writes its own, which no later tile reads, so no copy of X is made.  Three
// workgroups per CU: at four it spills (5.4 against 5.0 ms on 432000 x 384).
__global__ __launch_bounds__(256, 3) void rotate_upper_kernel(double2* X, int64_t ldx, int64_t rows, int n,
                                                              const double2* __restrict__ Q) {
  __shared__ GemmSmem<> sm;
  for (int j0 = (n - 1) / kGN * kGN; j0 >= 0; j0 -= kGN) {
    const int kend = j0 + kGN < n ? j0 + kGN : n;
    rotate_tile(sm, X, ldx, (int64_t)blockIdx.x * kGM, rows, Q, n, j0, kend, 1, X, ldx);
  }
}

// In place a triangular rotation has a workgroup per 64 rows, each walking all column
// tiles; fewer than there are CUs leave the GPU idle, and the copy of the rows costs less
// than that: 54 row tiles, 1000 columns 1.34 ms in place and 0.35 by panels; 128, 384: 0.22
// and 0.12, 128 columns 0.038 and 0.035; 182, 512: 0.37 and 0.29; 215, 800: 0.95 and 0.81,
// 128 columns 0.040 and 0.045; 250, 384: 0.22 and 0.26, 512: 0.38 and 0.35; 432, 384: 0.37
// and 0.43.
static bool rotate_by_panels(int64_t rows, int n, bool upper) {
  return !upper || (n > kGN && cdiv(rows, kGM) <= (n <= 2 * kGN ? 128 : 216));
}

// Rows of a panel: whole rounds of workgroups within 128 MiB of copied rows
static int64_t rotate_panel_rows(int64_t rows, int n) {
  const int64_t n_ct = cdiv(n, kGN);
  const int64_t cap = std::max<int64_t>(1, ((int64_t)1 << 27) / ((int64_t)n * 16) / kGM);   // row tiles
  const int64_t rounds = cap * n_ct / kGSlots;
  const int64_t rt = rounds > 0 ? std::max<int64_t>(1, rounds * kGSlots / n_ct) : cap;
  return std::min<int64_t>(rt, cdiv(rows, kGM)) * kGM;
}

// Doubles of the n x n matrix of a rotation and the panel behind it
size_t rotation_doubles(int64_t rows, int n, bool upper) {
  return ((rotate_by_panels(rows, n, upper) ? (size_t)rotate_panel_rows(rows, n) * n : 0) + (size_t)n * n) * 2;
}

// Room for the n x n matrix of rotate_device
double2* rotation_matrix(chfsi_ctx* c, int64_t rows, int n, bool upper) {
  c->panel.alloc(rotation_doubles(rows, n, upper));
  return reinterpret_cast<double2*>(c->panel.ptr);
}

void rotate_device(chfsi_ctx* c, double2* X, int64_t ldx, int64_t rows, int n, const double2* Qd, bool upper) {
  const bool panels = rotate_by_panels(rows, n, upper);
  StageTimer tm(c, CHFSI_STAGE_ROTATE, 8.0 * (double)rows * n * n * (upper ? 0.5 : 1.0),
                8.0 * (double)rows * n * n * (upper ? 0.5 : 1.0), (panels ? 4.0 : 2.0) * (double)rows * n * sizeof(double2));
  if (!panels) {
    hipLaunchKernelGGL(rotate_upper_kernel, dim3(cdiv(rows, kGM)), dim3(256), 0, c->stream, X, ldx, rows, n, Qd);
    LAUNCH_CHECK();
    return;
  }
  double2* P = reinterpret_cast<double2*>(c->panel.ptr) + (size_t)n * n;
  const int64_t prow = rotate_panel_rows(rows, n);
  for (int64_t r0 = 0; r0 < rows; r0 += prow) {
    const int64_t pr = std::min(prow, rows - r0);
    launch_copy_rows(c, P, n, X + r0 * ldx, ldx, pr, n);
    const int n_rt = cdiv(pr, kGM), n_ct = cdiv(n, kGN);
    if (upper)
      hipLaunchKernelGGL(rotate_kernel<true>, dim3(8 * cdiv(n_rt, 8) * n_ct), dim3(256), 0, c->stream, P, n, pr, Qd,
                         X + r0 * ldx, ldx, n_rt, n_ct);
    else
      hipLaunchKernelGGL(rotate_kernel<false>, dim3(8 * cdiv((int64_t)n_rt * n_ct, 8)), dim3(256), 0, c->stream, P, n,
                         pr, Qd, X + r0 * ldx, ldx, n_rt, n_ct);
    LAUNCH_CHECK();
  }
}

void rotate_inplace(chfsi_ctx* c, double2* X, int64_t ldx, int64_t rows, int n, const std::vector<cplx>& Q,
                    bool upper) {
  double2* Qd = rotation_matrix(c, rows, n, upper);
  std::vector<double2> qh((size_t)n * n);
  for (size_t i = 0; i < qh.size(); ++i) qh[i] = double2{Q[i].real(), Q[i].imag()};
  CHFSI_HIP(hipMemcpyAsync(Qd, qh.data(), qh.size() * sizeof(double2), hipMemcpyHostToDevice, c->stream));
  rotate_device(c, X, ldx, rows, n, Qd, upper);
  CHFSI_HIP(hipStreamSynchronize(c->stream));   // qh leaves scope
}

// ============================================================================
// Cholesky factor of the Gram matrix and the rotation it gives (CholGS)
// ============================================================================
// S' = D S D with D = diag(S)^{-1/2}, S' = L L^H, R = D L^{-H}, all in blocks of 32
// columns, on the device, so that nothing but the column of a failed pivot comes to
// the host before X R.  On the host with 16 threads this was 3.65 ms at n = 384 and
// the copies to and fro; the launches below take 0.62 ms (0.16 at n = 96, 2.0 at
// 1000).  A launch per block column of the factor and one for the inverse; bound by
// the chain of 32 pivots in each diagonal block (37 us per block, and 128 us for the
// inverse), not by the n^3 work.
constexpr int kCB = 32, kCPad = 2;         // block; pad as in the tile engine
typedef double2 CholTile[kCB][kCB + kCPad];

// info: [0] the matrix has a non-finite element, [1] first column without a
// positive diagonal, [2] first failed pivot (n: none)
__global__ __launch_bounds__(256) void chol_scale_kernel(const double2* __restrict__ S, int n, double* __restrict__ dsc,
                                                         double2* __restrict__ R, int* __restrict__ info) {
  const int i = blockIdx.x;
  const double si = S[(size_t)i * n + i].x;
  const double di = 1.0 / sqrt(si);
  if (threadIdx.x == 0) {
    dsc[i] = di;
    if (!(si > 0.0)) atomicMin(&info[1], i);
  }
  bool bad = false;
  for (int j = threadIdx.x; j < n; j += 256) {
    R[(size_t)i * n + j] = double2{0.0, 0.0};
    if (j > i) continue;
    const double2 v = S[(size_t)i * n + j];
    bad |= !isfinite(v.x) || !isfinite(v.y);
  }
  if (bad) atomicOr(&info[0], 1);
}

// A = D S D (lower triangle) into A
__global__ __launch_bounds__(256) void chol_apply_scale_kernel(const double2* __restrict__ S, int n,
                                                               const double* __restrict__ dsc,
                                                               double2* __restrict__ A) {
  const int i = blockIdx.x;
  const double di = dsc[i];
  for (int j = threadIdx.x; j <= i; j += 256) {
    const double2 v = S[(size_t)i * n + j];
    const double w = di * dsc[j];
    A[(size_t)i * n + j] = double2{v.x * w, v.y * w};
  }
}

// t <- the 32 x 32 block (bi, bj) of A (zero outside the matrix; outside the lower
// triangle too, with an identity on a diagonal past n)
__device__ __forceinline__ void chol_load(CholTile& t, const double2* __restrict__ A, int n, int bi, int bj) {
  for (int e = threadIdx.x; e < kCB * kCB; e += 256) {
    const int r = e / kCB, c = e % kCB, i = bi * kCB + r, j = bj * kCB + c;
    double2 v = {0.0, 0.0};
    if (i < n && j < n && j <= i) v = A[(size_t)i * n + j];
    else if (i == j) v.x = 1.0;
    t[r][c] = v;
  }
}

// acc of this wave's 16 x 16 quarter += P Q^H (HERM) or P Q over 32 columns
template <bool HERM>
__device__ __forceinline__ void chol_gemm(const CholTile& P, const CholTile& Q, d4& cr, d4& ci) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = (wave & 1) * 16 + (lane & 15), c = (wave >> 1) * 16 + (lane & 15), kl = lane >> 4;
#pragma unroll
  for (int ks = 0; ks < kCB / 4; ++ks) {
    const double2 a = P[r][4 * ks + kl];
    double2 b = HERM ? Q[c][4 * ks + kl] : Q[4 * ks + kl][c];
    if (HERM) b.y = -b.y;
    cr = mfma(a.x, b.x, cr);
    ci = mfma(a.x, b.y, ci);
    cr = mfma(-a.y, b.y, cr);
    ci = mfma(a.y, b.x, ci);
  }
}

// Factor of the diagonal block b in t and its inverse, by elimination of [t | I]:
// 256 threads, two barriers a column (the quotients of the column, the rest).  Products of
// quotients (a_ik / d_k) conj(a_jk), not of scaled columns, so that two equal columns of
// one block leave a pivot of exactly zero (in different blocks the pivot is a rounding,
// of either sign: L_jp = A_jp L_pp^{-H} rounds).
__device__ __forceinline__ void chol_factor(CholTile& t, CholTile& m, int n, int b, double2* __restrict__ L,
                                            double2* __restrict__ invd, int* __restrict__ info) {
  __shared__ double2 quot[kCB];
  for (int e = threadIdx.x; e < kCB * kCB; e += 256) m[e / kCB][e % kCB] = double2{e / kCB == e % kCB ? 1.0 : 0.0, 0.0};
  __syncthreads();
  for (int k = 0; k < kCB; ++k) {
    const double d = t[k][k].x;
    if (threadIdx.x == 0 && (!(d > 0.0) || !isfinite(d))) atomicMin(&info[2], b * kCB + k);
    if (threadIdx.x > k && threadIdx.x < kCB) {
      const double2 a = t[threadIdx.x][k];
      quot[threadIdx.x] = double2{a.x / d, a.y / d};
    }
    __syncthreads();
    // columns k+1.. of t below the diagonal, and columns 0..k of m
    for (int e = threadIdx.x; e < (kCB - 1 - k) * kCB; e += 256) {
      const int i = k + 1 + e / kCB, c = e % kCB;
      const double qx = quot[i].x, qy = quot[i].y;
      if (c <= k) {
        const double2 w = m[k][c];
        m[i][c].x -= qx * w.x - qy * w.y;
        m[i][c].y -= qx * w.y + qy * w.x;
      } else if (c <= i) {
        const double2 w = t[c][k];
        t[i][c].x -= qx * w.x + qy * w.y;
        t[i][c].y -= qy * w.x - qx * w.y;
      }
    }
    __syncthreads();
  }
  // rows and columns scaled by the pivots' roots
  for (int e = threadIdx.x; e < kCB * kCB; e += 256) {
    const int r = e / kCB, c = e % kCB, i = b * kCB + r, j = b * kCB + c;
    const double lr = sqrt(t[r][r].x), lc = sqrt(t[c][c].x);
    double2 v = t[r][c], w = m[r][c];
    if (c > r) v = w = double2{0.0, 0.0};
    else if (c == r) v = double2{lr, 0.0};
    else v = double2{v.x / lc, v.y / lc};
    w = double2{w.x / lr, w.y / lr};
    if (i < n && j < n) L[(size_t)i * n + j] = v;
    invd[(size_t)b * kCB * kCB + e] = w;
  }
}

__global__ __launch_bounds__(256) void chol_first_kernel(const double2* __restrict__ A, int n, double2* __restrict__ L,
                                                         double2* __restrict__ invd, int* __restrict__ info) {
  __shared__ CholTile t, m;
  chol_load(t, A, n, 0, 0);
  __syncthreads();
  chol_factor(t, m, n, 0, L, invd, info);
}

// Block column p eliminated: workgroup (i, j), p < j <= i, takes
// L_ip = A_ip L_pp^{-H}, L_jp alike, A_ij -= L_ip L_jp^H; the workgroups of column
// p + 1 also write their L_ip, and that of its diagonal factors the block.
__global__ __launch_bounds__(256) void chol_step_kernel(double2* __restrict__ A, int n, int p, double2* __restrict__ L,
                                                        double2* __restrict__ invd, int* __restrict__ info) {
  __shared__ CholTile t, m, u;
  int i = (int)((sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);
  while (i * (i + 1) / 2 > (int)blockIdx.x) --i;
  while ((i + 1) * (i + 2) / 2 <= (int)blockIdx.x) ++i;
  const int j = p + 1 + (int)blockIdx.x - i * (i + 1) / 2;
  i += p + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = (wave & 1) * 16, c0 = (wave >> 1) * 16 + (lane & 15);
  for (int e = threadIdx.x; e < kCB * kCB; e += 256) u[e / kCB][e % kCB] = invd[(size_t)p * kCB * kCB + e];
  chol_load(t, A, n, i, p);
  chol_load(m, A, n, j, p);
  __syncthreads();
  d4 lr{0, 0, 0, 0}, li{0, 0, 0, 0}, mr{0, 0, 0, 0}, mi{0, 0, 0, 0};
  chol_gemm<true>(t, u, lr, li);
  chol_gemm<true>(m, u, mr, mi);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = r0 + acc_row<double>(lane, q);
    t[r][c0] = double2{lr[q], li[q]};
    m[r][c0] = double2{mr[q], mi[q]};
    const int gi = i * kCB + r;
    if (j == p + 1 && gi < n) L[(size_t)gi * n + p * kCB + c0] = double2{lr[q], li[q]};
  }
  __syncthreads();
  d4 ar{0, 0, 0, 0}, ai{0, 0, 0, 0};
  chol_gemm<true>(t, m, ar, ai);
  chol_load(u, A, n, i, j);
  __syncthreads();
  const bool next = i == p + 1;           // its diagonal block: j = i
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = r0 + acc_row<double>(lane, q);
    const int gi = i * kCB + r, gj = j * kCB + c0;
    const double2 v = {u[r][c0].x - ar[q], u[r][c0].y - ai[q]};
    if (next) u[r][c0] = v;
    else if (gi < n && gj <= gi) A[(size_t)gi * n + gj] = v;
  }
  if (!next) return;                      // uniform over the block
  __syncthreads();
  chol_factor(u, m, n, i, L, invd, info);
}

// Block column j of X = L^{-1}, from the diagonal down: X_ij = -L_ii^{-1} sum_k L_ik X_kj,
// and R = D X^H.  The column's own blocks are read back from X (this workgroup's
// stores, behind barriers).
__global__ __launch_bounds__(256) void chol_inverse_kernel(const double2* __restrict__ L, int n,
                                                           const double2* __restrict__ invd,
                                                           const double* __restrict__ dsc, double2* X,
                                                           double2* __restrict__ R) {
  __shared__ CholTile t, m;
  const int j = blockIdx.x, nb = (n + kCB - 1) / kCB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = (wave & 1) * 16, c0 = (wave >> 1) * 16 + (lane & 15);
  const auto store = [&](int i, const CholTile& v) {
    for (int e = threadIdx.x; e < kCB * kCB; e += 256) {
      const int r = e / kCB, c = e % kCB, gi = i * kCB + r, gj = j * kCB + c;
      if (gi < n && gj < n) X[(size_t)gi * n + gj] = v[r][c];
    }
    for (int e = threadIdx.x; e < kCB * kCB; e += 256) {
      const int c = e / kCB, r = e % kCB, gi = i * kCB + r, gj = j * kCB + c;
      if (gi < n && gj < n) R[(size_t)gj * n + gi] = double2{dsc[gj] * v[r][c].x, -(dsc[gj] * v[r][c].y)};
    }
  };
  const auto diag = [&](CholTile& v, int b) {
    for (int e = threadIdx.x; e < kCB * kCB; e += 256) v[e / kCB][e % kCB] = invd[(size_t)b * kCB * kCB + e];
  };
  diag(t, j);
  __syncthreads();
  store(j, t);
  __syncthreads();
  constexpr int kPer = kCB * kCB / 256;
  for (int i = j + 1; i < nb; ++i) {
    d4 sr{0, 0, 0, 0}, si{0, 0, 0, 0};
    double2 pl[kPer], px[kPer];
    const auto gload = [&](int k) {       // L_ik and X_kj (k < i <= nb - 1: whole blocks of columns)
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        const int f = threadIdx.x + 256 * e, r = f / kCB, c = f % kCB;
        const int gi = i * kCB + r, gj = j * kCB + c;
        pl[e] = gi < n ? L[(size_t)gi * n + k * kCB + c] : double2{0.0, 0.0};
        px[e] = gj < n ? X[(size_t)(k * kCB + r) * n + gj] : double2{0.0, 0.0};
      }
    };
    gload(j);
    for (int k = j; k < i; ++k) {
      __syncthreads();                    // the last products have read t and m
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        const int f = threadIdx.x + 256 * e;
        t[f / kCB][f % kCB] = pl[e];
        m[f / kCB][f % kCB] = px[e];
      }
      __syncthreads();
      if (k + 1 < i) gload(k + 1);
      chol_gemm<false>(t, m, sr, si);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) m[r0 + acc_row<double>(lane, q)][c0] = double2{-sr[q], -si[q]};
    diag(t, i);
    __syncthreads();
    d4 xr{0, 0, 0, 0}, xi{0, 0, 0, 0};
    chol_gemm<false>(t, m, xr, xi);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) m[r0 + acc_row<double>(lane, q)][c0] = double2{xr[q], xi[q]};
    __syncthreads();
    store(i, m);
    __syncthreads();
  }
}

// Device memory of chol_rotation behind the Gram matrix, in doubles: A (later the
// inverse), L, the diagonal blocks' inverses, the scales, info
size_t chol_extra(int n) {
  const size_t nb = cdiv(n, kCB);
  return 4 * (size_t)n * n + 2 * nb * kCB * kCB + n + 4;
}

// R (device) from the Gram matrix Sd, whose `chol_extra` follows it; the columns of a
// failure, or n, in info (host): see chol_scale_kernel
void chol_rotation(chfsi_ctx* c, double2* Sd, int n, double2* R, int (&info)[3]) {
  const size_t nn = (size_t)n * n;
  const int nb = cdiv(n, kCB);
  double2 *A = Sd + nn, *L = A + nn, *invd = L + nn;
  double* dsc = reinterpret_cast<double*>(invd + (size_t)nb * kCB * kCB);
  int* info_d = reinterpret_cast<int*>(dsc + n);
  const int none[3] = {0, n, n};
  CHFSI_HIP(hipMemcpyAsync(info_d, none, sizeof none, hipMemcpyHostToDevice, c->stream));
  hipStream_t s = c->stream;
  hipLaunchKernelGGL(chol_scale_kernel, dim3(n), dim3(256), 0, s, Sd, n, dsc, R, info_d);
  LAUNCH_CHECK();
  hipLaunchKernelGGL(chol_apply_scale_kernel, dim3(n), dim3(256), 0, s, Sd, n, dsc, A);
  LAUNCH_CHECK();
  hipLaunchKernelGGL(chol_first_kernel, dim3(1), dim3(256), 0, s, A, n, L, invd, info_d);
  LAUNCH_CHECK();
  for (int p = 0; p + 1 < nb; ++p) {
    const int r = nb - 1 - p;
    hipLaunchKernelGGL(chol_step_kernel, dim3(r * (r + 1) / 2), dim3(256), 0, s, A, n, p, L, invd, info_d);
    LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(chol_inverse_kernel, dim3(nb), dim3(256), 0, s, L, n, invd, dsc, A, R);
  LAUNCH_CHECK();
  CHFSI_HIP(hipMemcpyAsync(info, info_d, sizeof none, hipMemcpyDeviceToHost, s));
  CHFSI_HIP(hipStreamSynchronize(s));
}

// ============================================================================
// Reductions with a fixed grid (deterministic order)
// ============================================================================
constexpr int kRedGroups = 256;

__global__ __launch_bounds__(256) void resid_kernel(const double2* __restrict__ W, int64_t ldw,
                                                    const double2* __restrict__ X, int64_t ldx,
                                                    int64_t rows, int n, const double* __restrict__ theta,
                                                    double* __restrict__ partial) {
  __shared__ double red[256];
  const int g = blockIdx.x;
  const int col = blockIdx.y * 64 + (threadIdx.x & 63);
  const int lr = threadIdx.x >> 6;
  double s = 0.0;
  if (col < n) {
    const double th = theta[col];
    for (int64_t r = (int64_t)g * 4 + lr; r < rows; r += (int64_t)kRedGroups * 4) {
      const double2 w = W[r * ldw + col], x = X[r * ldx + col];
      const double dr = w.x - th * x.x, di = w.y - th * x.y;
      s += dr * dr + di * di;
    }
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x < 64 && col < n)
    partial[(size_t)g * n + col] = ((red[threadIdx.x] + red[threadIdx.x + 64]) + red[threadIdx.x + 128]) +
                                   red[threadIdx.x + 192];
}

void column_resid_norms(chfsi_ctx* c, const double2* W, int64_t ldw, const double2* X, int64_t ldx,
                        int64_t rows, int n, const double* theta, double* out) {
  c->scratch.alloc((size_t)kRedGroups * n + n);
  double* part = c->scratch.ptr;
  double* th = part + (size_t)kRedGroups * n;
  CHFSI_HIP(hipMemcpyAsync(th, theta, n * sizeof(double), hipMemcpyHostToDevice, c->stream));
  hipLaunchKernelGGL(resid_kernel, dim3(kRedGroups, cdiv(n, 64)), dim3(256), 0, c->stream, W, ldw, X, ldx,
                     rows, n, th, part);
  LAUNCH_CHECK();
  std::vector<double> h((size_t)kRedGroups * n);
  CHFSI_HIP(hipMemcpyAsync(h.data(), part, h.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  CHFSI_HIP(hipStreamSynchronize(c->stream));
  for (int j = 0; j < n; ++j) {
    double s = 0.0;
    for (int g = 0; g < kRedGroups; ++g) s += h[(size_t)g * n + j];
    out[j] = std::sqrt(s);
  }
}

__global__ __launch_bounds__(256) void dot_kernel(const double2* __restrict__ x, const double2* __restrict__ y,
                                                  int64_t rows, double* __restrict__ partial) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t r = blockIdx.x * 256 + threadIdx.x; r < rows; r += (int64_t)kRedGroups * 256)
    s += x[r].x * y[r].x + x[r].y * y[r].y;
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// ---- Lanczos recurrence with its scalars on the device: a step's kernels sum the
// partial products they need themselves, so that no step waits for the host.
// sc: alpha_j at [0, steps), |w_j| at [steps, 2 steps), |v_0| at [2 steps].
__device__ __forceinline__ double red_sum(const double* __restrict__ partial, double* red) {
  red[threadIdx.x] = partial[threadIdx.x];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double s = red[0];
  __syncthreads();                        // red is free again
  return s;
}
static_assert(kRedGroups == 256, "red_sum takes one partial sum per thread");

// w <- w - alpha v - |w_{j-1}| vp (vp: none at j = 0), alpha from its partial sums,
// and the partial sums of |w|^2
__global__ __launch_bounds__(256) void lanczos_update_kernel(double2* __restrict__ w, const double2* __restrict__ v,
                                                             const double2* __restrict__ vp, int64_t rows,
                                                             const double* __restrict__ dots, int j, int steps,
                                                             double* __restrict__ sc, double* __restrict__ norms) {
  __shared__ double red[256];
  const double alpha = red_sum(dots, red);
  const double beta = j > 0 ? sc[steps + j - 1] : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) sc[j] = alpha;
  double s = 0.0;
  for (int64_t r = blockIdx.x * 256 + threadIdx.x; r < rows; r += (int64_t)kRedGroups * 256) {
    double2 x = w[r];
    const double2 y = v[r];
    x.x -= alpha * y.x;
    x.y -= alpha * y.y;
    if (j > 0) {
      const double2 z = vp[r];
      x.x -= beta * z.x;
      x.y -= beta * z.y;
    }
    w[r] = x;
    s += x.x * x.x + x.y * x.y;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) norms[blockIdx.x] = red[0];
}

// v <- w / |w| from the partial sums of |w|^2 (zero where that is not positive); the
// norm to out
__global__ __launch_bounds__(256) void lanczos_scale_kernel(double2* __restrict__ v, const double2* __restrict__ w,
                                                            int64_t rows, const double* __restrict__ norms,
                                                            double* __restrict__ out) {
  __shared__ double red[256];
  const double nrm = sqrt(red_sum(norms, red));
  const bool pos = nrm > 0.0;
  const double f = 1.0 / nrm;
  if (blockIdx.x == 0 && threadIdx.x == 0) *out = nrm;
  for (int64_t r = blockIdx.x * 256 + threadIdx.x; r < rows; r += (int64_t)kRedGroups * 256) {
    const double2 x = w[r];
    v[r] = pos ? double2{f * x.x, f * x.y} : double2{0.0, 0.0};
  }
}

// alpha_j and |w_j| of up to `steps` steps from v0 (those up to the first |w_j| that is
// not positive), and |v0|.  20 steps on 250000 rows with 16 atoms were 4.0 ms with two
// trips to the host and five vector kernels a step, 2.4 ms with these three and the
// narrower coefficient tiles, 1.6 ms with the one-column product; the product with H is 68 of a step's 82 us.
void lanczos_steps(chfsi_ctx* c, KPoint& kp, const double2* v0, int steps, double& n0, std::vector<double>& al,
                   std::vector<double>& bn) {
  const int64_t rows = 2 * c->n_nodes;
  const size_t n_sc = 2 * (size_t)steps + 1;
  c->lanczos.alloc((size_t)6 * rows + 2 * kRedGroups + n_sc);
  double2* v = reinterpret_cast<double2*>(c->lanczos.ptr);
  double2 *w = v + rows, *vp = w + rows;
  double* dots = reinterpret_cast<double*>(vp + rows);
  double *norms = dots + kRedGroups, *sc = norms + kRedGroups;
  hipStream_t s = c->stream;
  const auto dot = [&](const double2* x, const double2* y, double* out) {
    hipLaunchKernelGGL(dot_kernel, dim3(kRedGroups), dim3(256), 0, s, x, y, rows, out);
    LAUNCH_CHECK();
  };
  std::vector<double> h(n_sc);
  dot(v0, v0, norms);
  hipLaunchKernelGGL(lanczos_scale_kernel, dim3(kRedGroups), dim3(256), 0, s, v, v0, rows, norms, sc + 2 * steps);
  LAUNCH_CHECK();
  constexpr int kLook = 32;               // steps between the host's looks at a breakdown
  int done = 0;
  bool ended = false;
  while (done < steps && !ended) {
    const int j1 = std::min(steps, done + kLook);
    for (int j = done; j < j1; ++j) {
      apply_H(c, kp, v, 1, w, 1, 1, CHFSI_PREC_FP64, 1.0, 0.0, 0.0);
      dot(v, w, dots);
      hipLaunchKernelGGL(lanczos_update_kernel, dim3(kRedGroups), dim3(256), 0, s, w, v, vp, rows, dots, j, steps, sc,
                         norms);
      LAUNCH_CHECK();
      std::swap(vp, v);                   // vp <- v
      hipLaunchKernelGGL(lanczos_scale_kernel, dim3(kRedGroups), dim3(256), 0, s, v, w, rows, norms, sc + steps + j);
      LAUNCH_CHECK();
    }
    CHFSI_HIP(hipMemcpyAsync(h.data(), sc, n_sc * sizeof(double), hipMemcpyDeviceToHost, s));
    CHFSI_HIP(hipStreamSynchronize(s));
    n0 = h[2 * steps];
    if (!(n0 > 0.0 && std::isfinite(n0))) return;
    for (int j = done; j < j1 && !ended; ++j) {
      al.push_back(h[j]);
      bn.push_back(h[steps + j]);
      ended = !(h[steps + j] > 0.0);
    }
    done = j1;
  }
}

// ============================================================================
// Seeded fill (SplitMix64, counter form) and finiteness check
// ============================================================================
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t i) {
  uint64_t z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__global__ void fill_random_kernel(double2* __restrict__ X, int64_t n_rows, int n_vec, int64_t ld,
                                   uint64_t seed, int64_t row0, int col0, int64_t ntc) {
  const int64_t total = n_rows * n_vec;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / n_vec;
    const int n = (int)(t - r * n_vec);
    const uint64_t j = (uint64_t)(row0 + r) * (uint64_t)ntc + (uint64_t)(col0 + n);
    const double ur = (double)(splitmix64_at(seed, 2 * j) >> 11) * (1.0 / 9007199254740992.0);
    const double ui = (double)(splitmix64_at(seed, 2 * j + 1) >> 11) * (1.0 / 9007199254740992.0);
    X[r * ld + n] = double2{2.0 * ur - 1.0, 2.0 * ui - 1.0};
  }
}

void launch_fill_random(chfsi_ctx* c, double2* X, int64_t n_rows, int n_vec, int64_t ld, uint64_t seed,
                        int64_t row0, int col0, int64_t ntc) {
  const int64_t total = n_rows * n_vec;
  const int blocks = (int)std::min<int64_t>(cdiv(total, 256), 8192);
  hipLaunchKernelGGL(fill_random_kernel, dim3(std::max(blocks, 1)), dim3(256), 0, c->stream, X, n_rows,
                     n_vec, ld, seed, row0, col0, ntc);
  LAUNCH_CHECK();
}

__global__ void zero_int_kernel(int* __restrict__ f) { f[0] = f[1] = 0; }

__global__ void nonfinite_kernel(const double* __restrict__ p, int64_t n, const double* __restrict__ q, int64_t m,
                                 int* __restrict__ flag) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x, i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  for (int64_t i = i0; i < n; i += step)
    if (!isfinite(p[i])) flag[0] = 1;
  for (int64_t i = i0; i < m; i += step)
    if (!isfinite(q[i])) flag[1] = 1;
}

int check_finite2(chfsi_ctx* c, const double* p, int64_t n, const double* q, int64_t m) {
  c->scratch.alloc(1);
  int* flag = reinterpret_cast<int*>(c->scratch.ptr);
  hipLaunchKernelGGL(zero_int_kernel, dim3(1), dim3(1), 0, c->stream, flag);
  LAUNCH_CHECK();
  const int blocks = (int)std::min<int64_t>(cdiv(std::max(n, m), 256), 4096);
  hipLaunchKernelGGL(nonfinite_kernel, dim3(std::max(blocks, 1)), dim3(256), 0, c->stream, p, n, q, m, flag);
  LAUNCH_CHECK();
  int h[2] = {0, 0};
  CHFSI_HIP(hipMemcpyAsync(h, flag, sizeof(h), hipMemcpyDeviceToHost, c->stream));
  CHFSI_HIP(hipStreamSynchronize(c->stream));
  return (h[0] ? 1 : 0) | (h[1] ? 2 : 0);
}

}  // namespace chfsi
