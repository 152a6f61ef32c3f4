// Scalar fields of the self-consistent loop (Sec. III.B: the fixed-point map
// and its density mixing; Sec. IV.A: the two-grid start).
//
// Fields live at the cell quadrature points ([E][nq^3], the order of
// chfsi_quad_points) or at the global nodes ([M]).  The FE scalar operator
// A = K_s + kappa^2 M_c (K_s = int grad N_I . grad N_J, M_c = int N_I N_J) has
// the same tensor-product cell matrix in every cell of the uniform mesh, so the
// assembled operator is a sum of Kronecker products of assembled 1-D matrices, whose
// rows reach p nodes to either side: its action and its diagonal come from
// two 1-D row tables, node by node, without assembly.  Screened Poisson problems
// (kappa^2 - lap) u = g are solved in the FE space by conjugate gradients
// preconditioned with the diagonal of A.  Sums have a fixed order (bitwise
// reproducible).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "internal.h"
#include "mfma.h"

namespace chfsi {

namespace {
constexpr int kFieldRed = 256;      // fixed reduction grid (deterministic order)

// The mesh and 1-D tables of the scalar kernels.
struct ScalMesh {
  int p, np1, nq, nx, ny, nz, Nx, Ny, Nz;
  const double* B;      // [np1][nq] Lagrange basis at the quadrature points
  const double* wq;     // [nq] weights
  const double* rows;   // [2][p][2p + 1]: rows of the assembled 1-D stiffness and mass of the
                        // nodes a = 0 .. p-1 of a cell, over the nodes -p .. p of the cell's frame
  double J, sx, sy, sz; // A = J (sx S M M + sy M S M + sz M M S + kappa^2 M M M), s_d = (2/h_d)^2
};

// Sum of the 256 threads' values, to every thread, in a fixed order.
__device__ __forceinline__ double block_sum(double v, double* sm) {
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) v += __shfl_xor(v, k);
  __syncthreads();                        // sm is free
  if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
  __syncthreads();
  return (sm[0] + sm[1]) + (sm[2] + sm[3]);
}
// NS such sums at once: the 256 threads' v[k], to every thread in v[k]
template <int NS>
__device__ __forceinline__ void block_sums(double (&v)[NS], double* sm) {
#pragma unroll
  for (int k = 32; k > 0; k >>= 1)
#pragma unroll
    for (int i = 0; i < NS; ++i) v[i] += __shfl_xor(v[i], k);
  __syncthreads();                        // sm is free
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int i = 0; i < NS; ++i) sm[4 * i + (threadIdx.x >> 6)] = v[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NS; ++i) v[i] = (sm[4 * i] + sm[4 * i + 1]) + (sm[4 * i + 2] + sm[4 * i + 3]);
}

// ---- Conjugate gradients, two kernels per step, scalars on the device.  A step was
// a fill, a launch per colour, ten vector kernels and three round trips to the host
// (about 130 us on 4^3 cells, p = 4); these two take 9.4 us.  red: [kCgDots][stride]
// partial sums (p.Ap; r.r and r.z of even and odd steps; b.b), a part per workgroup,
// then the state: the number of steps when r.r reached the tolerance, or -1.
// Up to kCgParts workgroups, eight per CU: with one per CU large meshes of low order
// waited for each other's trips to memory (128 steps: p = 3, 48^3 cells 121 ms, now 40;
// p = 6, 16^3 17.6 and 10.4).
constexpr int kCgDots = 6, kCgPq = 0, kCgRr = 1, kCgRz = 3, kCgBb = 5, kCgParts = 2048;
// Where part i of dot k lies, and this thread's share of the n parts.  Up to 256 of them
// (MANY = false) a fixed stride and one part per thread: with the run's stride and the
// loop small meshes took 1 to 2 % longer (128 steps: 3^3 cells, p = 4 1.755 ms and 1.725;
// 4^3, p = 4 1.747 and 1.716, p = 7 2.772 and 2.731).
template <bool MANY>
__device__ __forceinline__ int cg_at(int stride, int k, int i) {
  return k * (MANY ? stride : 256) + i;
}
template <bool MANY>
__device__ __forceinline__ double cg_part(const double* __restrict__ red, int stride, int k, int n) {
  double s = (int)threadIdx.x < n ? red[cg_at<MANY>(stride, k, threadIdx.x)] : 0.0;
  if constexpr (MANY)
    for (int i = threadIdx.x + 256; i < n; i += 256) s += red[cg_at<MANY>(stride, k, i)];
  return s;
}

// 1 / diag(A) at node (ax, ay, az) of a cell's frame (a < p in each direction)
__device__ __forceinline__ double inv_diag(const ScalMesh& m, double kappa2, int ax, int ay, int az) {
  const int w = 2 * m.p + 1, c = m.p;     // the diagonal entry of row a is at column p + a
  const double* S = m.rows;
  const double* M = m.rows + m.p * w;
  const double mx = M[ax * w + c + ax], my = M[ay * w + c + ay], mz = M[az * w + c + az];
  const double s = m.sx * S[ax * w + c + ax] * my * mz + m.sy * mx * S[ay * w + c + ay] * mz +
                   m.sz * mx * my * S[az * w + c + az] + kappa2 * (mx * my * mz);
  return 1.0 / (m.J * s);
}

// r = b, u = 0, z = r / diag(A); partial b.b (= r.r) and r.z
template <bool MANY>
__global__ __launch_bounds__(256) void cg_start_kernel(const ScalMesh m, double kappa2, int64_t n,
                                                       const double* __restrict__ b, double* __restrict__ u,
                                                       double* __restrict__ r, double* __restrict__ z, int stride,
                                                       double* __restrict__ red) {
  __shared__ double sm[4];
  double rr = 0.0, rz = 0.0;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int iyz = (int)(i / m.Nx), ix = (int)(i - (int64_t)iyz * m.Nx);
    const double ri = b[i], zi = inv_diag(m, kappa2, ix % m.p, (iyz % m.Ny) % m.p, (iyz / m.Ny) % m.p) * ri;
    u[i] = 0.0;
    r[i] = ri;
    z[i] = zi;
    rr += ri * ri;
    rz += ri * zi;
  }
  rr = block_sum(rr, sm);
  rz = block_sum(rz, sm);
  if (threadIdx.x == 0) {
    red[cg_at<MANY>(stride, kCgRr, blockIdx.x)] = rr;
    red[cg_at<MANY>(stride, kCgBb, blockIdx.x)] = rr;
    red[cg_at<MANY>(stride, kCgRz, blockIdx.x)] = rz;
    if (blockIdx.x == 0) red[cg_at<MANY>(stride, kCgDots, 0)] = -1.0;
  }
}

// Head of step `it`: the state and the sums it needs, asked for ...
struct CgHead {
  double state, d[4];
};
template <bool MANY>
__device__ __forceinline__ CgHead cg_ask(const double* __restrict__ red, int stride, int n_part, int it) {
  const int odd = it & 1;
  return CgHead{red[cg_at<MANY>(stride, kCgDots, 0)],
                {cg_part<MANY>(red, stride, kCgRr + odd, n_part), cg_part<MANY>(red, stride, kCgBb, n_part),
                 cg_part<MANY>(red, stride, kCgRz + odd, n_part),
                 it > 0 ? cg_part<MANY>(red, stride, kCgRz + 1 - odd, n_part) : 0.0}};
}
// ... and beta from them, or false if the iteration has ended (a step before, or now)
template <bool MANY>
__device__ __forceinline__ bool cg_go(CgHead& h, double* sm, double* __restrict__ red, int stride, int it, double tol,
                                      double& beta) {
  block_sums(h.d, sm);
  if (h.state >= 0.0) return false;
  const double rr = h.d[0], bb = h.d[1];
  if (bb == 0.0 || (it > 0 && sqrt(rr) / sqrt(bb) <= tol)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) red[cg_at<MANY>(stride, kCgDots, 0)] = (double)it;
    return false;
  }
  beta = it == 0 ? 0.0 : h.d[2] / h.d[3];
  return true;
}

// Step `it`, first half: stops everything once r.r is small enough, else
// p = z + beta p (into the other buffer), q = A p, partial p.q.  A workgroup takes the
// nodes owned by a cell (local index < p in each direction): the frame of
// (2p + 1)^3 nodes around them is read into LDS and contracted with the row tables
// along z, y and x; the mass and stiffness parts that the other directions need go
// along, scaled at the end.  On a small mesh a step is a chain of trips to memory: the
// state, the partial sums and the first cell's frame are all asked for at once
// (5.9 us on 4^3 cells, p = 4, and the update 3.5; 8.8 and 4.1 one after the other).
template <int P, bool MANY>
__global__ __launch_bounds__(256) void cg_apply_kernel(const ScalMesh m, double kappa2, int64_t n, int n_part,
                                                       int it, double tol, const double* __restrict__ z,
                                                       const double* __restrict__ p_old, double* __restrict__ p_new,
                                                       double* __restrict__ q, int stride,
                                                       double* __restrict__ red) {
  extern __shared__ double fsm[];
  __shared__ double sm[16];
  constexpr int p = P, w = 2 * p + 1, w3 = w * w * w;
  constexpr int kCgPre = w3 <= 1024 ? (w3 + 255) / 256 : 4;       // frame values per thread fetched ahead
  CgHead head = cg_ask<MANY>(red, stride, n_part, it);
  const auto node = [&](int e, int t) {   // frame entry t of cell e
    const int cx = e % m.nx, cyz = e / m.nx, cy = cyz % m.ny, cz = cyz / m.ny;
    const int fx = t % w, fy = (t / w) % w, fz = t / (w * w);
    int ix = cx * p + fx - p, iy = cy * p + fy - p, iz = cz * p + fz - p;
    ix = ix < 0 ? ix + m.Nx : ix >= m.Nx ? ix - m.Nx : ix;
    iy = iy < 0 ? iy + m.Ny : iy >= m.Ny ? iy - m.Ny : iy;
    iz = iz < 0 ? iz + m.Nz : iz >= m.Nz ? iz - m.Nz : iz;
    return ix + (int64_t)m.Nx * (iy + (int64_t)m.Ny * iz);
  };
  double zf[kCgPre], pf[kCgPre];
#pragma unroll
  for (int k = 0; k < kCgPre; ++k) {
    const int t = threadIdx.x + 256 * k;
    const int64_t I = node(blockIdx.x, t < w3 ? t : 0);
    zf[k] = z[I];
    pf[k] = it > 0 ? p_old[I] : 0.0;
  }
  double* sR = fsm;                       // [2][p][w] row tables
  double* sX = sR + 2 * p * w;            // [w][w][w] frame (x fastest), then [2][w (y)][w (x)][p (z)] ...
  double* sM = sX + w3;                   // [p][w][w] mass part along z, then [p][p][w]
  double* sS = sM + p * w * w;            // stiffness part, likewise
  for (int t = threadIdx.x; t < 2 * p * w; t += 256) sR[t] = m.rows[t];
  double beta;
  if (!cg_go<MANY>(head, sm, red, stride, it, tol, beta)) return;
  const double* rS = sR;
  const double* rM = sR + p * w;
  double pq = 0.0;
  for (int e = blockIdx.x; e < (int)n; e += gridDim.x) {
    const bool first = e == (int)blockIdx.x;
    if (!first) __syncthreads();          // the last cell's sX is read
    const auto put = [&](int t, double zv, double pv) {
      const double v = it == 0 ? zv : fma(beta, pv, zv);
      const int fx = t % w, fy = (t / w) % w, fz = t / (w * w);
      sX[t] = v;
      if (fx >= p && fx < 2 * p && fy >= p && fy < 2 * p && fz >= p && fz < 2 * p) p_new[node(e, t)] = v;
    };
    if (first) {
#pragma unroll
      for (int k = 0; k < kCgPre; ++k)
        if ((int)threadIdx.x + 256 * k < w3) put(threadIdx.x + 256 * k, zf[k], pf[k]);
    }
    for (int t = threadIdx.x + (first ? 256 * kCgPre : 0); t < w3; t += 256) {
      const int64_t I = node(e, t);
      put(t, z[I], it > 0 ? p_old[I] : 0.0);
    }
    __syncthreads();
    double own[2];                        // the values of this thread's own nodes
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int t = min((int)threadIdx.x + 256 * k, p * p * p - 1), a = t % p, bc = t / p;
      own[k] = sX[p + a + w * (p + bc % p + w * (p + bc / p))];
    }
    for (int t = threadIdx.x; t < p * w * w; t += 256) {          // along z: M, S
      const int xy = t % (w * w), a = t / (w * w);
      double vm = 0.0, vs = 0.0;
#pragma unroll
      for (int j = 0; j < w; ++j) {
        if (j < p && a > 0) continue;     // (rows a > 0 stay in the cell)
        const double x = sX[xy + w * w * j];
        vm = fma(rM[a * w + j], x, vm);
        vs = fma(rS[a * w + j], x, vs);
      }
      sM[t] = vm;
      sS[t] = vs;
    }
    __syncthreads();
    double* tA = sX;                      // [p z][p y][w x]: M M
    double* tB = sX + p * p * w;          // sy S M + sz M S (+ kappa^2 M M)
    for (int t = threadIdx.x; t < p * p * w; t += 256) {          // along y
      const int x = t % w, a = (t / w) % p, c = t / (w * p);
      double mm = 0.0, sm_ = 0.0, ms = 0.0;
#pragma unroll
      for (int j = 0; j < w; ++j) {
        if (j < p && a > 0) continue;
        const double vm = sM[(c * w + j) * w + x], vs = sS[(c * w + j) * w + x];
        mm = fma(rM[a * w + j], vm, mm);
        sm_ = fma(rS[a * w + j], vm, sm_);
        ms = fma(rM[a * w + j], vs, ms);
      }
      tA[t] = mm;
      tB[t] = m.sy * sm_ + m.sz * ms + kappa2 * mm;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2; ++k) {                                 // along x (p^3 <= 512)
      const int t = threadIdx.x + 256 * k;
      if (t >= p * p * p) break;
      const int a = t % p, bc = t / p;
      double v = 0.0, vs = 0.0;
#pragma unroll
      for (int j = 0; j < w; ++j) {
        if (j < p && a > 0) continue;
        v = fma(rM[a * w + j], tB[bc * w + j], v);
        vs = fma(rS[a * w + j], tA[bc * w + j], vs);
      }
      const int cx = e % m.nx, cyz = e / m.nx, cy = cyz % m.ny, cz = cyz / m.ny;
      const int64_t I = cx * p + a + (int64_t)m.Nx * (cy * p + bc % p + (int64_t)m.Ny * (cz * p + bc / p));
      const double y = m.J * fma(m.sx, vs, v);
      q[I] = y;
      pq = fma(own[k], y, pq);
    }
  }
  pq = block_sum(pq, sm);
  if (threadIdx.x == 0) red[cg_at<MANY>(stride, kCgPq, blockIdx.x)] = pq;
}

// The same first half for orders 1 and 2, a thread per node: its row of A reaches 27 to
// 125 nodes, read through the caches, where a workgroup per cell would have one or eight
// nodes to share its barriers: 128 steps on 64^3 cells with p = 1 4 and 34 ms, p = 2 36
// and 51; on 16^3 with p = 2 3.3 and 2.9.  From p = 3 a node reads too many.
template <int P, bool MANY>
__global__ __launch_bounds__(256) void cg_apply_node_kernel(const ScalMesh m, double kappa2, int64_t n, int n_part,
                                                            int it, double tol, const double* __restrict__ z,
                                                            const double* __restrict__ p_old,
                                                            double* __restrict__ p_new, double* __restrict__ q,
                                                            int stride, double* __restrict__ red) {
  __shared__ double sm[16];
  constexpr int w = 2 * P + 1;
  __shared__ double sR[2 * P * w];
  for (int t = threadIdx.x; t < 2 * P * w; t += 256) sR[t] = m.rows[t];
  CgHead head = cg_ask<MANY>(red, stride, n_part, it);
  double beta;
  if (!cg_go<MANY>(head, sm, red, stride, it, tol, beta)) return;   // (its barriers order sR)
  double pq = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int iyz = (int)(i / m.Nx), ix = (int)(i - (int64_t)iyz * m.Nx), iz = iyz / m.Ny, iy = iyz - iz * m.Ny;
    const int a = ix % P, b = iy % P, c = iz % P;
    // rows of the three directions: entry j at node offset j - P from the cell's first node
    const double *Sx = sR + a * w, *Sy = sR + b * w, *Sz = sR + c * w;
    const double *Mx = Sx + P * w, *My = Sy + P * w, *Mz = Sz + P * w;
    int off[w];
#pragma unroll
    for (int j = 0; j < w; ++j) {
      const int x = ix - a + j - P;
      off[j] = x < 0 ? x + m.Nx : x >= m.Nx ? x - m.Nx : x;
    }
    double y = 0.0, own = 0.0;
#pragma unroll
    for (int jz = 0; jz < w; ++jz) {
      if (jz < P && c > 0) continue;      // (rows a > 0 stay in the cell)
      int kz = iz - c + jz - P;
      kz = kz < 0 ? kz + m.Nz : kz >= m.Nz ? kz - m.Nz : kz;
#pragma unroll
      for (int jy = 0; jy < w; ++jy) {
        if (jy < P && b > 0) continue;
        int ky = iy - b + jy - P;
        ky = ky < 0 ? ky + m.Ny : ky >= m.Ny ? ky - m.Ny : ky;
        const int64_t r0 = (int64_t)m.Nx * (ky + (int64_t)m.Ny * kz);
        double vs = 0.0, vm = 0.0;
#pragma unroll
        for (int j = 0; j < w; ++j) {     // (entries left of the cell are zero in rows a > 0)
          double v = z[r0 + off[j]];
          if (it > 0) v = fma(beta, p_old[r0 + off[j]], v);
          vs = fma(Sx[j], v, vs);
          vm = fma(Mx[j], v, vm);
          if (jz == P + c && jy == P + b && j == P + a) own = v;
        }
        const double mm = My[jy] * Mz[jz];
        y = fma(m.sx * mm, vs, y);
        y = fma(m.sy * Sy[jy] * Mz[jz] + m.sz * My[jy] * Sz[jz] + kappa2 * mm, vm, y);
      }
    }
    y *= m.J;
    p_new[i] = own;
    q[i] = y;
    pq = fma(own, y, pq);
  }
  pq = block_sum(pq, sm);
  if (threadIdx.x == 0) red[cg_at<MANY>(stride, kCgPq, blockIdx.x)] = pq;
}

// Second half: u += alpha p, r -= alpha q, z = r / diag(A); partial r.r, r.z for the next step
template <bool MANY>
__global__ __launch_bounds__(256) void cg_update_kernel(const ScalMesh m, double kappa2, int64_t n, int n_part,
                                                        int n_pq, int it, const double* __restrict__ p,
                                                        const double* __restrict__ q, double* __restrict__ u,
                                                        double* __restrict__ r, double* __restrict__ z, int stride,
                                                        double* __restrict__ red) {
  __shared__ double sm[8];
  const int odd = it & 1;
  const double state = red[cg_at<MANY>(stride, kCgDots, 0)];
  double d[2] = {cg_part<MANY>(red, stride, kCgRz + odd, n_part), cg_part<MANY>(red, stride, kCgPq, n_pq)};
  const int64_t i0 = blockIdx.x * (int64_t)256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
  // this thread's first values, asked for with the sums
  const int64_t ic = i0 < n ? i0 : n - 1;
  double pv = p[ic], qv = q[ic], uv = u[ic], rv = r[ic];
  block_sums(d, sm);
  if (state >= 0.0) return;
  const double al = d[0] / d[1];
  double s[2] = {0.0, 0.0};
  for (int64_t i = i0; i < n; i += step) {
    if (i != i0) {
      pv = p[i];
      qv = q[i];
      uv = u[i];
      rv = r[i];
    }
    const int iyz = (int)(i / m.Nx), ix = (int)(i - (int64_t)iyz * m.Nx);
    u[i] = fma(al, pv, uv);
    const double ri = fma(-al, qv, rv);
    const double zi = inv_diag(m, kappa2, ix % m.p, (iyz % m.Ny) % m.p, (iyz / m.Ny) % m.p) * ri;
    r[i] = ri;
    z[i] = zi;
    s[0] += ri * ri;
    s[1] += ri * zi;
  }
  block_sums(s, sm);
  if (threadIdx.x == 0) {
    red[cg_at<MANY>(stride, kCgRr + 1 - odd, blockIdx.x)] = s[0];
    red[cg_at<MANY>(stride, kCgRz + 1 - odd, blockIdx.x)] = s[1];
  }
}

// One direction of a tensor contraction in LDS: out[.. o ..] = sum_i T(i, o) in[.. i ..]
// with n_in values in, n_out out along the direction, inner values before it and outer after.
template <class F>
__device__ __forceinline__ void contract_dir(const double* in, double* out, int inner, int n_in, int n_out, int outer,
                                             F T) {
  for (int t = threadIdx.x; t < inner * n_out * outer; t += 256) {
    const int i0 = t % inner, o = (t / inner) % n_out, k = t / (inner * n_out);
    double s = 0.0;
    for (int i = 0; i < n_in; ++i) s = fma(T(i, o), in[i0 + inner * (i + n_in * k)], s);
    out[t] = s;
  }
  __syncthreads();
}

// be[e][i] = sum_q N_i(r_q) w_q J g[e][q], the cells' parts of the right-hand side
__global__ __launch_bounds__(256) void scal_project_kernel(const ScalMesh m, int buf, const double* __restrict__ g,
                                                           double* __restrict__ be) {
  extern __shared__ double fsm[];
  const int nq = m.nq, np = m.np1, nq3 = nq * nq * nq, nloc = np * np * np, e = blockIdx.x;
  double* sB = fsm;                       // [np1][nq]
  double* a = sB + np * nq;
  double* b = a + buf;
  for (int t = threadIdx.x; t < np * nq; t += 256) sB[t] = m.B[t];
  for (int t = threadIdx.x; t < nq3; t += 256)
    a[t] = m.wq[t % nq] * m.wq[(t / nq) % nq] * m.wq[t / (nq * nq)] * m.J * g[(size_t)e * nq3 + t];
  __syncthreads();
  const auto T = [&](int q, int i) { return sB[i * nq + q]; };
  contract_dir(a, b, nq * nq, nq, np, 1, T);
  contract_dir(b, a, nq, nq, np, np, T);
  contract_dir(a, b, 1, nq, np, np * np, T);
  for (int t = threadIdx.x; t < nloc; t += 256) be[(size_t)e * nloc + t] = b[t];
}

// b[I] = scale times the sum of be over the cells that hold node I (fixed order)
__global__ __launch_bounds__(256) void scal_gather_kernel(const ScalMesh m, int64_t n, double scale,
                                                          const double* __restrict__ be, double* __restrict__ b) {
  const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (i >= n) return;
  const int ix = (int)(i % m.Nx), iy = (int)((i / m.Nx) % m.Ny), iz = (int)(i / ((int64_t)m.Nx * m.Ny));
  const int nloc = m.np1 * m.np1 * m.np1;
  double s = 0.0;
  for (int k = 0; k < 8; ++k) {
    // (k & 1) etc.: the cell that ends at this node instead of the one it lies in
    int cx = ix / m.p, ax = ix - cx * m.p, cy = iy / m.p, ay = iy - cy * m.p, cz = iz / m.p, az = iz - cz * m.p;
    if ((k & 1) && ax != 0) continue;
    if ((k & 2) && ay != 0) continue;
    if ((k & 4) && az != 0) continue;
    if (k & 1) ax = m.p, cx = cx == 0 ? m.nx - 1 : cx - 1;
    if (k & 2) ay = m.p, cy = cy == 0 ? m.ny - 1 : cy - 1;
    if (k & 4) az = m.p, cz = cz == 0 ? m.nz - 1 : cz - 1;
    s += be[(size_t)(cx + m.nx * (cy + m.ny * cz)) * nloc + ax + m.np1 * (ay + m.np1 * az)];
  }
  b[i] = scale * s;
}

// out[e][q] = sum_i N_i(r_q) u[I(e, i)]
__global__ __launch_bounds__(256) void scal_interp_kernel(const ScalMesh m, int buf,
                                                          const int32_t* __restrict__ cell_nodes,
                                                          const double* __restrict__ u, double* __restrict__ out) {
  extern __shared__ double fsm[];
  const int nq = m.nq, np = m.np1, nq3 = nq * nq * nq, nloc = np * np * np, e = blockIdx.x;
  double* sB = fsm;
  double* a = sB + np * nq;
  double* b = a + buf;
  for (int t = threadIdx.x; t < np * nq; t += 256) sB[t] = m.B[t];
  for (int t = threadIdx.x; t < nloc; t += 256) a[t] = u[cell_nodes[(size_t)e * nloc + t]];
  __syncthreads();
  const auto T = [&](int i, int q) { return sB[i * nq + q]; };
  contract_dir(a, b, np * np, np, nq, 1, T);
  contract_dir(b, a, np, np, nq, nq, T);
  contract_dir(a, b, 1, np, nq, nq * nq, T);
  for (int t = threadIdx.x; t < nq3; t += 256) out[(size_t)e * nq3 + t] = b[t];
}

// partial[g] = sum over this group's strided range of x[i] * y[i] * (w ? w[i % nw] : 1)
__global__ __launch_bounds__(256) void wdot_kernel(const double* __restrict__ x, const double* __restrict__ y,
                                                   const double* __restrict__ w, int64_t nw, int64_t n,
                                                   double* __restrict__ partial) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)kFieldRed * 256) {
    const double t = x[i] * (y ? y[i] : 1.0);
    s += w ? t * w[i % nw] : t;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int k = 128; k > 0; k >>= 1) {
    if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// y = a x + b y (y may be null: y = a x written to out)
__global__ void axpby_kernel(int64_t n, double a, const double* __restrict__ x, double b, const double* y,
                             double* out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = a * x[i] + (y ? b * y[i] : 0.0);
}

__global__ void fill_kernel(int64_t n, double v, double* __restrict__ out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = v;
}

// LSDA (Dirac) exchange under the locally collinear substitution
// rho_up,dn = (rho +- |m|)/2: v_s = -(6/pi)^(1/3) rho_s^(1/3),
// V = (v_up + v_dn)/2, B = (v_up - v_dn)/2 m/|m|  (B = 0 where m = 0)
__global__ void exchange_kernel(int64_t n, const double* __restrict__ rho, const double* __restrict__ m,
                                const double* __restrict__ vadd, const double* __restrict__ badd,
                                double* __restrict__ V, double* __restrict__ B) {
  const double cx = cbrt(6.0 / M_PI);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const double mx = m[3 * i], my = m[3 * i + 1], mz = m[3 * i + 2];
    const double ma = sqrt(mx * mx + my * my + mz * mz);
    const double ru = fmax(0.5 * (rho[i] + ma), 0.0), rd = fmax(0.5 * (rho[i] - ma), 0.0);
    const double vu = -cx * cbrt(ru), vd = -cx * cbrt(rd);
    V[i] = 0.5 * (vu + vd) + (vadd ? vadd[i] : 0.0);
    const double f = ma > 0.0 ? 0.5 * (vu - vd) / ma : 0.0;
    B[3 * i] = f * mx + (badd ? badd[3 * i] : 0.0);
    B[3 * i + 1] = f * my + (badd ? badd[3 * i + 1] : 0.0);
    B[3 * i + 2] = f * mz + (badd ? badd[3 * i + 2] : 0.0);
  }
}

// two-grid transfer: every fine node takes the coarse field of its canonical cell
// (the cell where its local index is below p in each direction), through the
// coarse Lagrange basis at the fine GLL nodes: Yf = M_f^{1/2} T (M_c^{-1/2} Yc)
__global__ __launch_bounds__(256) void block_interp_kernel(
    const double2* __restrict__ Yc, int64_t ldc, double2* __restrict__ Yf, int64_t ldf, int n_vec,
    const double* __restrict__ T /*[npc][npf]*/, const int32_t* __restrict__ cnodes_c, const double* __restrict__ ms_c,
    const double* __restrict__ ms_f, int pf, int npc, int ncx, int ncy, int nfx, int nfy, int64_t n_fine) {
  const int64_t total = n_fine * n_vec;
  const int nlc = npc * npc * npc;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t I = t / n_vec;
    const int col = (int)(t - I * n_vec);
    const int ix = (int)(I % nfx), iy = (int)((I / nfx) % nfy), iz = (int)(I / ((int64_t)nfx * nfy));
    const int cx = ix / pf, cy = iy / pf, cz = iz / pf;
    const int ax = ix - cx * pf, ay = iy - cy * pf, az = iz - cz * pf;
    const int32_t* nd = cnodes_c + (size_t)(cx + ncx * (cy + ncy * cz)) * nlc;
    const int npf = pf + 1;
    double2 s0 = {0.0, 0.0}, s1 = {0.0, 0.0};
    for (int k = 0; k < npc; ++k) {
      const double tz = T[k * npf + az];
      for (int j = 0; j < npc; ++j) {
        const double tyz = tz * T[j * npf + ay];
        for (int i = 0; i < npc; ++i) {
          const double w = tyz * T[i * npf + ax];
          const int64_t J = nd[i + npc * (j + npc * k)];
          const double sc = w * ms_c[J];
          const double2 u0 = Yc[(2 * J) * ldc + col], u1 = Yc[(2 * J + 1) * ldc + col];
          s0.x += sc * u0.x;
          s0.y += sc * u0.y;
          s1.x += sc * u1.x;
          s1.y += sc * u1.y;
        }
      }
    }
    const double f = 1.0 / ms_f[I];
    Yf[(2 * I) * ldf + col] = double2{f * s0.x, f * s0.y};
    Yf[(2 * I + 1) * ldf + col] = double2{f * s1.x, f * s1.y};
  }
}

int grid_for(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(cdiv(n, 256), 8192)); }
}  // namespace

// ---------------------------------------------------------------- host side
struct FieldOps {
  DevBuf<double> rows;     // row tables of the assembled 1-D stiffness and mass (ScalMesh)
  DevBuf<double> wJ;       // [nq3] w_q J
  DevBuf<double> wJ3;      // [3 nq3] w_q J repeated per vector component
  DevBuf<double> ones;     // [max(M, E nq3)] ones
  DevBuf<double> md;       // [M] lumped mass M_D
  DevBuf<double> gq;       // [E nq3] a field at the quadrature points
  DevBuf<double> red;      // reduction partials (and the CG's sums and state)
  DevBuf<double> be;       // [E][nloc] cells' parts of a nodal right-hand side
  DevBuf<double> v[7];     // u, r, z, p (two), q = A p, b
  ScalMesh mesh;
  double md_sum = 0.0;
  bool ready = false;
};

static void fill(chfsi_ctx* c, int64_t n, double v, double* out);
static void axpby(chfsi_ctx* c, int64_t n, double a, const double* x, double b, const double* y, double* out);

static FieldOps& fops(chfsi_ctx* c) {
  if (!c->fields) c->fields = std::make_shared<FieldOps>();
  FieldOps& f = *c->fields;
  if (!f.ready) {
    for (auto* b : {&f.wJ, &f.wJ3, &f.ones, &f.md, &f.gq, &f.red, &f.be, &f.rows}) b->spare = &c->ye;
    for (auto& b : f.v) b.spare = &c->ye;
    const int n = c->np1, nq = c->nq, nloc = c->nloc, nq3 = c->nq3;
    std::vector<double> wJ(nq3);
    // rows a = 0 .. p-1 of the assembled 1-D matrices over the nodes -p .. p: node 0 is
    // shared with the cell before (its last row), the others lie inside the cell
    const int p = c->p, w = 2 * p + 1;
    std::vector<double> rows((size_t)2 * p * w, 0.0);
    for (int k = 0; k < 2; ++k) {
      const std::vector<double>& T = k == 0 ? c->ref.D : c->ref.B;
      for (int a = 0; a < n; ++a)
        for (int b = 0; b < n; ++b) {
          double v = 0.0;
          for (int q = 0; q < nq; ++q) v += c->ref.wq[q] * T[a * nq + q] * T[b * nq + q];
          if (a < p) rows[((size_t)k * p + a) * w + p + b] += v;
          else rows[(size_t)k * p * w + b] += v;      // node p of the cell before = node 0
        }
    }
    for (int q = 0; q < nq3; ++q)
      wJ[q] = c->ref.wq[q % nq] * c->ref.wq[(q / nq) % nq] * c->ref.wq[q / (nq * nq)] * c->J;
    std::vector<double> wJ3((size_t)3 * nq3), md(c->n_nodes);
    for (int q = 0; q < nq3; ++q) wJ3[3 * q] = wJ3[3 * q + 1] = wJ3[3 * q + 2] = wJ[q];
    f.md_sum = 0.0;
    for (int64_t i = 0; i < c->n_nodes; ++i) {
      md[i] = 1.0 / (c->minv_sqrt_h[i] * c->minv_sqrt_h[i]);
      f.md_sum += md[i];
    }
    const int64_t np = (int64_t)c->n_cells * nq3;
    f.rows.upload(rows.data(), rows.size(), c->stream);
    if (c->ref_b1.n == 0) {
      c->ref_b1.upload(c->ref.B.data(), c->ref.B.size(), c->stream);
      c->ref_wq.upload(c->ref.wq.data(), c->ref.wq.size(), c->stream);
    }
    f.wJ.upload(wJ.data(), wJ.size(), c->stream);
    f.wJ3.upload(wJ3.data(), wJ3.size(), c->stream);
    f.md.upload(md.data(), md.size(), c->stream);
    f.ones.alloc(std::max<int64_t>(c->n_nodes, np));
    fill(c, std::max<int64_t>(c->n_nodes, np), 1.0, f.ones.ptr);
    f.gq.alloc(np);
    f.red.alloc(kCgDots * kCgParts + 1);
    f.be.alloc((size_t)c->n_cells * nloc);
    f.mesh = ScalMesh{p, n, nq, c->nc[0], c->nc[1], c->nc[2], c->Nd[0], c->Nd[1], c->Nd[2], c->ref_b1.ptr,
                      c->ref_wq.ptr, f.rows.ptr, c->J, 4.0 / (c->h[0] * c->h[0]), 4.0 / (c->h[1] * c->h[1]),
                      4.0 / (c->h[2] * c->h[2])};
    for (auto& b : f.v) b.alloc(c->n_nodes);
    CHFSI_HIP(hipStreamSynchronize(c->stream));
    f.ready = true;
  }
  return f;
}

// sum_i x_i y_i (w_{i mod nw}); fixed grid, partials summed on the host in order
static double wdot(chfsi_ctx* c, FieldOps& f, const double* x, const double* y, const double* w, int64_t nw,
                   int64_t n) {
  hipLaunchKernelGGL(wdot_kernel, dim3(kFieldRed), dim3(256), 0, c->stream, x, y, w, nw, n, f.red.ptr);
  LAUNCH_CHECK();
  double h[kFieldRed];
  CHFSI_HIP(hipMemcpyAsync(h, f.red.ptr, sizeof(h), hipMemcpyDeviceToHost, c->stream));
  CHFSI_HIP(hipStreamSynchronize(c->stream));
  double s = 0.0;
  for (int g = 0; g < kFieldRed; ++g) s += h[g];
  return s;
}

static void axpby(chfsi_ctx* c, int64_t n, double a, const double* x, double b, const double* y, double* out) {
  hipLaunchKernelGGL(axpby_kernel, dim3(grid_for(n)), dim3(256), 0, c->stream, n, a, x, b, y, out);
  LAUNCH_CHECK();
}

static void fill(chfsi_ctx* c, int64_t n, double v, double* out) {
  hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(256), 0, c->stream, n, v, out);
  LAUNCH_CHECK();
}

static int scal_buf(const chfsi_ctx* c) {        // largest stage of a cell's contractions
  const int n = std::max(c->np1, c->nq);
  return n * n * n;
}

// b = scale int N_I g (nodal, overwritten)
static void scal_project(chfsi_ctx* c, FieldOps& f, double scale, const double* g, double* b) {
  const int buf = scal_buf(c);
  const size_t sh = (size_t)(c->np1 * c->nq + 2 * buf) * sizeof(double);
  hipLaunchKernelGGL(scal_project_kernel, dim3(c->n_cells), dim3(256), sh, c->stream, f.mesh, buf, g, f.be.ptr);
  LAUNCH_CHECK();
  hipLaunchKernelGGL(scal_gather_kernel, dim3(cdiv(c->n_nodes, 256)), dim3(256), 0, c->stream, f.mesh, c->n_nodes,
                     scale, f.be.ptr, b);
  LAUNCH_CHECK();
}

static void scal_interp(chfsi_ctx* c, FieldOps& f, const double* u, double* out) {
  const int buf = scal_buf(c);
  const size_t sh = (size_t)(c->np1 * c->nq + 2 * buf) * sizeof(double);
  hipLaunchKernelGGL(scal_interp_kernel, dim3(c->n_cells), dim3(256), sh, c->stream, f.mesh, buf,
                     c->cell_nodes.ptr, u, out);
  LAUNCH_CHECK();
}

// The kernels of order p (see cg_at)
struct CgKernels {
  decltype(&cg_start_kernel<true>) start;
  decltype(&cg_apply_kernel<3, true>) apply;
  decltype(&cg_update_kernel<true>) update;
};
template <bool MANY>
static CgKernels cg_kernels(int p) {
  static constexpr decltype(&cg_apply_kernel<3, MANY>) kApply[] = {
      cg_apply_node_kernel<1, MANY>, cg_apply_node_kernel<2, MANY>, cg_apply_kernel<3, MANY>, cg_apply_kernel<4, MANY>,
      cg_apply_kernel<5, MANY>,      cg_apply_kernel<6, MANY>,      cg_apply_kernel<7, MANY>, cg_apply_kernel<8, MANY>};
  static_assert(sizeof kApply / sizeof *kApply == kMaxP, "one per order");
  return {cg_start_kernel<MANY>, kApply[p - 1], cg_update_kernel<MANY>};
}

// A u = b by CG preconditioned with diag(A)^{-1}, A = K_s + kappa2 M_c; b is v[6]; u
// returned in v[0].  Stops when ||r|| <= tol ||b||.  Returns the iteration count
// (negative if max_iter hit).  The host looks every kCgBatch steps; the steps issued
// past the end return at once.
static int pcg(chfsi_ctx* c, FieldOps& f, double kappa2, double tol, int max_iter, double* rel_out) {
  constexpr int kCgBatch = 16;
  const int64_t n = c->n_nodes;
  double *u = f.v[0].ptr, *r = f.v[1].ptr, *z = f.v[2].ptr, *q = f.v[5].ptr, *b = f.v[6].ptr;
  double* pp[2] = {f.v[3].ptr, f.v[4].ptr};
  const int p = c->p, w = 2 * p + 1;
  // a thread per node or, from p = 3 on, a workgroup per cell
  const bool by_node = p <= 2;
  const int n_part = std::min(kCgParts, cdiv(n, 256));
  const int n_pq = by_node ? n_part : std::min(kCgParts, c->n_cells);
  const bool many = std::max(n_part, n_pq) > 256;
  const int stride = many ? std::max(n_part, n_pq) : 256;
  const size_t sh = by_node ? 0 : (size_t)(2 * p * w + w * w * w + 2 * p * w * w) * sizeof(double);
  const CgKernels k = many ? cg_kernels<true>(p) : cg_kernels<false>(p);
  hipLaunchKernelGGL(k.start, dim3(n_part), dim3(256), 0, c->stream, f.mesh, kappa2, n, b, u, r, z, stride, f.red.ptr);
  LAUNCH_CHECK();
  std::vector<double> h((size_t)kCgDots * stride + 1);
  for (int it = 0;;) {
    const int end = std::min(max_iter, it + kCgBatch);
    for (; it < end; ++it) {
      hipLaunchKernelGGL(k.apply, dim3(n_pq), dim3(256), sh, c->stream, f.mesh, kappa2,
                         by_node ? n : c->n_cells, n_part, it, tol, z, pp[1 - (it & 1)], pp[it & 1], q, stride,
                         f.red.ptr);
      LAUNCH_CHECK();
      hipLaunchKernelGGL(k.update, dim3(n_part), dim3(256), 0, c->stream, f.mesh, kappa2, n, n_part, n_pq, it,
                         pp[it & 1], q, u, r, z, stride, f.red.ptr);
      LAUNCH_CHECK();
    }
    CHFSI_HIP(hipMemcpyAsync(h.data(), f.red.ptr, h.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    CHFSI_HIP(hipStreamSynchronize(c->stream));
    const double state = h.back();
    const int done = state >= 0.0 ? (int)state : it;
    double rr = 0.0, bb = 0.0;
    for (int g = 0; g < n_part; ++g) {
      rr += h[(size_t)(kCgRr + (done & 1)) * stride + g];
      bb += h[(size_t)kCgBb * stride + g];
    }
    const double rel = bb == 0.0 ? 0.0 : std::sqrt(rr) / std::sqrt(bb);
    if (state < 0.0 && it < max_iter) continue;
    if (rel_out) *rel_out = rel;
    return state >= 0.0 || rel <= tol ? done : -done;
  }
}

double field_integral(chfsi_ctx* c, const double* g) {
  FieldOps& f = fops(c);
  return wdot(c, f, g, nullptr, f.wJ.ptr, c->nq3, (int64_t)c->n_cells * c->nq3);
}

double field_inner(chfsi_ctx* c, const double* r1, const double* m1, const double* r2, const double* m2) {
  FieldOps& f = fops(c);
  const int64_t np = (int64_t)c->n_cells * c->nq3;
  double s = wdot(c, f, r1, r2, f.wJ.ptr, c->nq3, np);
  if (m1 && m2) s += wdot(c, f, m1, m2, f.wJ3.ptr, 3 * c->nq3, 3 * np);
  return 0.5 * s;
}

// (kappa^2 - lap) u = scale g in the FE space, u at the quadrature points (u may
// alias g).  kappa2 == 0: the periodic problem with g - mean(g), u of zero
// lumped-mass mean.  Returns the CG iteration count (negative: not converged).
int screened_poisson(chfsi_ctx* c, double kappa2, double scale, const double* g, double* u_q, double tol,
                     int max_iter, double* rel) {
  FieldOps& f = fops(c);
  const int64_t np = (int64_t)c->n_cells * c->nq3;
  const double vol = c->box[0] * c->box[1] * c->box[2];
  const double* src = g;
  if (kappa2 == 0.0) {
    const double gbar = field_integral(c, g) / vol;
    axpby(c, np, 1.0, g, -gbar, f.ones.ptr, f.gq.ptr);          // g - mean(g)
    src = f.gq.ptr;
  }
  scal_project(c, f, scale, src, f.v[6].ptr);
  if (kappa2 == 0.0) {
    // the right-hand side's roundoff component along the constants (the null space)
    const double bm = wdot(c, f, f.v[6].ptr, nullptr, nullptr, 1, c->n_nodes) / (double)c->n_nodes;
    axpby(c, c->n_nodes, 1.0, f.v[6].ptr, -bm, f.ones.ptr, f.v[6].ptr);
  }
  const int it = pcg(c, f, kappa2, tol, max_iter, rel);
  if (kappa2 == 0.0) {
    const double mean = wdot(c, f, f.v[0].ptr, f.md.ptr, nullptr, 1, c->n_nodes) / f.md_sum;
    axpby(c, c->n_nodes, 1.0, f.v[0].ptr, -mean, f.ones.ptr, f.v[0].ptr);
  }
  scal_interp(c, f, f.v[0].ptr, u_q);
  CHFSI_HIP(hipStreamSynchronize(c->stream));
  return it;
}

void launch_exchange(chfsi_ctx* c, int64_t n_points, const double* rho, const double* m, const double* vadd,
                     const double* badd, double* V, double* B) {
  hipLaunchKernelGGL(exchange_kernel, dim3(grid_for(n_points)), dim3(256), 0, c->stream, n_points, rho, m, vadd,
                     badd, V, B);
  LAUNCH_CHECK();
}

void field_axpby(chfsi_ctx* c, int64_t n, double a, const double* x, double b, const double* y, double* out) {
  axpby(c, n, a, x, b, y, out);
}

void field_fill(chfsi_ctx* c, int64_t n, double v, double* out) { fill(c, n, v, out); }

void interpolate_block(chfsi_ctx* cc, chfsi_ctx* cf, const double2* Yc, int64_t ldc, double2* Yf, int64_t ldf,
                       int n_vec) {
  std::vector<double> T, D;
  lagrange_on(cc->ref.xi, cf->ref.xi, T, D);      // T[i][a] = l_i^{p-1}(xi_a^p)
  DevBuf<double> Td;
  Td.upload(T.data(), T.size(), cf->stream);
  const int64_t total = cf->n_nodes * n_vec;
  hipLaunchKernelGGL(block_interp_kernel, dim3(grid_for(total)), dim3(256), 0, cf->stream, Yc, ldc, Yf, ldf, n_vec,
                     Td.ptr, cc->cell_nodes.ptr, cc->minv_sqrt.ptr, cf->minv_sqrt.ptr, cf->p, cc->np1, cc->nc[0],
                     cc->nc[1], cf->Nd[0], cf->Nd[1], cf->n_nodes);
  LAUNCH_CHECK();
  CHFSI_HIP(hipStreamSynchronize(cf->stream));
}

}  // namespace chfsi
