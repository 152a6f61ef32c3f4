// Hermitian eigendecomposition on the host for the T x T projected problems of
// the Rayleigh-Ritz step (Sec. III.B.2), T <= a few thousand: Householder
// reduction to a Hermitian tridiagonal matrix (Golub and Van Loan, Sec. 8.3), a
// diagonal phase change that makes it real, then the implicit QL iteration with
// shifts on the real tridiagonal (Bowdler, Martin, Reinsch and Wilkinson, 1968),
// accumulating the rotations, and back-transformation by blocks of reflectors in
// the compact WY form I - Y T Y^H (Schreiber and Van Loan, 1989).
// All matrices are row-major std::vector<cplx> of size n*n.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <functional>
#include <memory>
#include <numeric>
#include <thread>

#include "internal.h"

namespace chfsi {

// Fixed set of worker threads for the O(n^3) loops below.  run(f) calls f(t, nt)
// on every worker t (the caller is worker 0) and returns when all are done; the
// workers spin briefly, then yield, between calls, so the many short parallel
// phases of one factorisation pay no thread start-up.
class Pool {
 public:
  explicit Pool(size_t work) {
    nt_ = (int)std::min<unsigned>(16u, std::max(1u, std::thread::hardware_concurrency()));
    if (work < ((size_t)1 << 16)) nt_ = 1;
    for (int t = 1; t < nt_; ++t) th_.emplace_back([this, t]() { loop(t); });
  }
  ~Pool() {
    stop_.store(true);
    gen_.fetch_add(1);
    for (auto& x : th_) x.join();
  }
  int size() const { return nt_; }
  void run(const std::function<void(int, int)>& f) {
    if (nt_ == 1) {
      f(0, 1);
      return;
    }
    f_ = &f;
    done_.store(0);
    gen_.fetch_add(1, std::memory_order_release);
    f(0, nt_);
    for (int spin = 0; done_.load(std::memory_order_acquire) != nt_ - 1; ++spin)
      if (spin > 4096) std::this_thread::yield();
  }
  // [lo, hi) share of n items for worker t of nt
  static void range(int n, int t, int nt, int& lo, int& hi) {
    lo = (int)((int64_t)n * t / nt);
    hi = (int)((int64_t)n * (t + 1) / nt);
  }

 private:
  void loop(int t) {
    unsigned seen = 0;
    while (true) {
      unsigned g;
      for (int spin = 0; (g = gen_.load(std::memory_order_acquire)) == seen; ++spin)
        if (spin > 4096) std::this_thread::yield();
      seen = g;
      if (stop_.load()) return;
      (*f_)(t, nt_);
      done_.fetch_add(1, std::memory_order_acq_rel);
    }
  }
  int nt_ = 1;
  std::vector<std::thread> th_;
  std::atomic<unsigned> gen_{0};
  std::atomic<int> done_{0};
  std::atomic<bool> stop_{false};
  const std::function<void(int, int)>* f_ = nullptr;
};

// Inner loops, compiled twice: for processors with AVX2 and FMA and for any (chosen
// at run time).  Complex numbers are interleaved (re, im), a vector holds two.
typedef double v4 __attribute__((vector_size(32), aligned(8), may_alias));

#define CHFSI_DENSE_KERNELS(NAME, ATTR)                                                                               \
  struct NAME {                                                                                                       \
    /* A -= (a + i b) conj(q) + (e + i f) conj(v); out = sum of the new A times x */                                  \
    ATTR static void update_dot(double* __restrict__ A, int n2, const double* q, const double* v, const double* x,    \
                                double a, double b, double e, double f, double* out) {                                \
      const v4 a4 = {a, -a, a, -a}, e4 = {e, -e, e, -e};                                                              \
      v4 s1[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}}, s2[2] = {{0, 0, 0, 0}, {0, 0, 0, 0}};                                  \
      int j = 0;                                                                                                      \
      for (; j + 8 <= n2; j += 8)                                                                                     \
        for (int u = 0; u < 2; ++u) {                                                                                 \
          const int k = j + 4 * u;                                                                                    \
          const v4 qk = *(const v4*)(q + k), vk = *(const v4*)(v + k), xk = *(const v4*)(x + k);                      \
          const v4 y = *(const v4*)(A + k) - (a4 * qk + b * __builtin_shufflevector(qk, qk, 1, 0, 3, 2) + e4 * vk +   \
                                              f * __builtin_shufflevector(vk, vk, 1, 0, 3, 2));                       \
          *(v4*)(A + k) = y;                                                                                          \
          s1[u] += y * __builtin_shufflevector(xk, xk, 0, 0, 2, 2);                                                   \
          s2[u] += y * __builtin_shufflevector(xk, xk, 1, 1, 3, 3);                                                   \
        }                                                                                                             \
      const v4 t1 = s1[0] + s1[1], t2 = s2[0] + s2[1];                                                                \
      double r1 = t1[0] + t1[2], i1 = t1[1] + t1[3], r2 = t2[0] + t2[2], i2 = t2[1] + t2[3];                          \
      for (; j < n2; j += 2) {                                                                                        \
        const double yr = A[j] - (a * q[j] + b * q[j + 1] + e * v[j] + f * v[j + 1]);                                 \
        const double yi = A[j + 1] - (b * q[j] - a * q[j + 1] + f * v[j] - e * v[j + 1]);                             \
        A[j] = yr;                                                                                                    \
        A[j + 1] = yi;                                                                                                \
        r1 += yr * x[j];                                                                                              \
        i1 += yi * x[j];                                                                                              \
        r2 += yr * x[j + 1];                                                                                          \
        i2 += yi * x[j + 1];                                                                                          \
      }                                                                                                               \
      out[0] = r1 - i2;                                                                                               \
      out[1] = i1 + r2;                                                                                               \
    }                                                                                                                 \
    /* y += (ar + i ai) x over n2 doubles */                                                                          \
    ATTR static void caxpy(double* __restrict__ y, const double* __restrict__ x, double ar, double ai, int n2) {      \
      const v4 w = {-ai, ai, -ai, ai};                                                                                \
      int j = 0;                                                                                                      \
      for (; j + 4 <= n2; j += 4) {                                                                                   \
        const v4 u = *(const v4*)(x + j);                                                                             \
        *(v4*)(y + j) += ar * u + w * __builtin_shufflevector(u, u, 1, 0, 3, 2);                                      \
      }                                                                                                               \
      for (; j < n2; j += 2) {                                                                                        \
        y[j] += ar * x[j] - ai * x[j + 1];                                                                            \
        y[j + 1] += ar * x[j + 1] + ai * x[j];                                                                        \
      }                                                                                                               \
    }                                                                                                                 \
    /* a chain of len rotations of rows (i, i + 1), i = m - 1 down, on eight columns */                               \
    ATTR static void rotate8(double* Z, int m, int len, const double* rc, const double* rs) {                         \
      double* z = Z + (size_t)m * 8;                                                                                  \
      v4 c0 = *(const v4*)z, c1 = *(const v4*)(z + 4);                                                                \
      for (int r = 0; r < len; ++r) {                                                                                 \
        double* up = z - 8;                                                                                           \
        const v4 a0 = *(const v4*)up, a1 = *(const v4*)(up + 4);                                                      \
        *(v4*)z = rs[r] * a0 + rc[r] * c0;                                                                            \
        *(v4*)(z + 4) = rs[r] * a1 + rc[r] * c1;                                                                      \
        c0 = rc[r] * a0 - rs[r] * c0;                                                                                 \
        c1 = rc[r] * a1 - rs[r] * c1;                                                                                 \
        z = up;                                                                                                       \
      }                                                                                                               \
      *(v4*)z = c0;                                                                                                   \
      *(v4*)(z + 4) = c1;                                                                                             \
    }                                                                                                                 \
  };
CHFSI_DENSE_KERNELS(DenseAny, )
CHFSI_DENSE_KERNELS(DenseAvx2, __attribute__((target("avx2,fma"))))
#undef CHFSI_DENSE_KERNELS

struct DenseOps {
  decltype(&DenseAny::update_dot) update_dot;
  decltype(&DenseAny::caxpy) caxpy;
  decltype(&DenseAny::rotate8) rotate8;
};
static DenseOps dense_ops() {
  if (__builtin_cpu_supports("avx2") && __builtin_cpu_supports("fma"))
    return {DenseAvx2::update_dot, DenseAvx2::caxpy, DenseAvx2::rotate8};
  return {DenseAny::update_dot, DenseAny::caxpy, DenseAny::rotate8};
}

// sqrt(f^2 + g^2); hypot only where the squares could leave the range
static inline double hyp(double f, double g) {
  const double s = f * f + g * g;
  return s > 1e-280 && s < 1e280 ? std::sqrt(s) : std::hypot(f, g);
}

// The rotations of the QL iteration on their way from the thread that finds them to
// those that apply them, a chain (of rows (i, i + 1), i = m - 1 .. m - len) at a time.
// When the room is used up the producer waits until every consumer has taken all.
class RotQueue {
 public:
  // consumers: those at work beside the producer (0: one afterwards; the room grows)
  RotQueue(int n, int consumers) : taken_(std::max(1, consumers)), alone_(consumers == 0) {
    cap_ = std::max<size_t>(n, std::min<size_t>((size_t)1 << 20, 4 * (size_t)n * n + 1024));
    rc_.reset(new double[cap_]);
    rs_.reset(new double[cap_]);
    chains_.reserve(cap_);
  }
  // room for a chain of at most n rotations
  void open(int n) {
    if (used_ + n <= cap_) return;
    if (alone_) {
      for (auto* a : {&rc_, &rs_}) {
        std::unique_ptr<double[]> b(new double[2 * cap_]);
        std::copy(a->get(), a->get() + used_, b.get());
        *a = std::move(b);
      }
      cap_ *= 2;
      return;
    }
    const int64_t all = published_.load(std::memory_order_relaxed);
    for (auto& t : taken_)
      for (int spin = 0; t.v.load(std::memory_order_acquire) < all; ++spin)
        if (spin > 4096) std::this_thread::yield();
    used_ = 0;
    chains_.clear();
    base_ = all;
  }
  void push(double c, double s) {
    rc_[used_ + len_] = c;
    rs_[used_ + len_] = s;
    ++len_;
  }
  void close(int m) {
    if (len_ == 0) return;
    chains_.push_back({m, len_, used_});
    used_ += len_;
    len_ = 0;
    published_.fetch_add(1, std::memory_order_release);
  }
  void finish() { finished_.store(true, std::memory_order_release); }
  // f(m, len, c, s) for every chain in order, until the producer has finished
  template <class F>
  void consume(int who, F f) {
    for (int64_t g = 0;;) {
      int64_t p;
      for (int spin = 0; (p = published_.load(std::memory_order_acquire)) == g; ++spin) {
        if (finished_.load(std::memory_order_acquire) && published_.load(std::memory_order_acquire) == g) return;
        if (spin > 4096) std::this_thread::yield();
      }
      for (; g < p; ++g) {
        const Chain& c = chains_.data()[g - base_];
        f(c.m, c.len, &rc_[c.off], &rs_[c.off]);
      }
      taken_[who].v.store(g, std::memory_order_release);
    }
  }

 private:
  struct Chain {
    int m, len;
    size_t off;
  };
  struct alignas(64) Count {
    std::atomic<int64_t> v{0};
    Count() = default;
    Count(const Count& o) : v(o.v.load()) {}
    Count& operator=(const Count& o) {
      v.store(o.v.load());
      return *this;
    }
  };
  size_t cap_, used_ = 0;
  int len_ = 0;
  int64_t base_ = 0;
  std::unique_ptr<double[]> rc_, rs_;
  std::vector<Chain> chains_;   // with consumers beside the producer it never outgrows its first room
  std::vector<Count> taken_;
  const bool alone_;
  std::atomic<int64_t> published_{0};
  std::atomic<bool> finished_{false};
};

// Implicit QL on the real symmetric tridiagonal (d, e), e[i] couples i, i+1: the
// eigenvalues in d.  out: takes the rotations, in order, or null.
static void tridiag_ql(std::vector<double>& d, std::vector<double>& e, int n, RotQueue* out) {
  if (n == 0) return;
  e.resize(n);
  e[n - 1] = 0.0;
  for (int l = 0; l < n; ++l) {
    int iter = 0;
    while (true) {
      int m = l;
      for (; m < n - 1; ++m) {
        const double dd = std::fabs(d[m]) + std::fabs(d[m + 1]);
        if (std::fabs(e[m]) <= 1e-16 * dd) break;
      }
      if (m == l) break;
      if (++iter > 200) break;
      double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
      double r = std::hypot(g, 1.0);
      g = d[m] - d[l] + e[l] / (g + std::copysign(r, g));
      double s = 1.0, c = 1.0, p = 0.0;
      int i = m - 1;
      bool deflated = false;
      if (out) out->open(n);
      for (; i >= l; --i) {
        double f = s * e[i], b = c * e[i];
        r = hyp(f, g);
        e[i + 1] = r;
        if (r == 0.0) {
          d[i + 1] -= p;
          e[m] = 0.0;
          deflated = true;
          break;
        }
        s = f / r;
        c = g / r;
        g = d[i + 1] - p;
        r = (d[i] - g) * s + 2.0 * c * b;
        p = s * r;
        d[i + 1] = g + p;
        g = c * r - b;
        if (out) out->push(c, s);
      }
      if (out) out->close(m);
      if (deflated) continue;
      d[l] -= p;
      e[l] = g;
      e[m] = 0.0;
    }
  }
}

// The same with eigenvector i in row i of Z, in blocks of eight columns ([block][n][8],
// so that a block stays in the first cache), from the identity.  The rotations only act
// on Z: the first worker finds them, the others apply them as they come, each to its
// own blocks (alone: afterwards).  Along a chain the updated row i is the next
// rotation's row i+1 and stays in registers.
static void tridiag_vectors(std::vector<double>& d, std::vector<double>& e, std::vector<double>& Z, int n, Pool& pool,
                            const DenseOps& ops) {
  const int consumers = std::max(1, pool.size() - 1), blocks = (n + 7) / 8;
  Z.resize((size_t)blocks * n * 8);
  RotQueue q(n, pool.size() - 1);
  const auto apply = [&](int who) {
    int lo, hi;
    Pool::range(blocks, who, consumers, lo, hi);
    for (int b = lo; b < hi; ++b)
      for (int u = 0; u < 8 && 8 * b + u < n; ++u) Z[((size_t)b * n + 8 * b + u) * 8 + u] = 1.0;
    q.consume(who, [&](int m, int len, const double* rc, const double* rs) {
      for (int b = lo; b < hi; ++b) ops.rotate8(&Z[(size_t)b * n * 8], m, len, rc, rs);
    });
  };
  if (pool.size() > 1) {
    pool.run([&](int t, int) {
      if (t > 0) {
        apply(t - 1);
        return;
      }
      tridiag_ql(d, e, n, &q);
      q.finish();
    });
    return;
  }
  tridiag_ql(d, e, n, &q);
  q.finish();
  apply(0);
}

// One pass over the trailing block per reflector: the update of the one before and the
// product with the new vector, every row by the same thread throughout.  Bound by the
// threads' meetings and the vectors they pass, and in the QL iteration by its chain of
// square roots and quotients.  16 threads, n = 256: reduction 3.0 -> 1.6 ms (two passes
// before, and column k read across all rows), QL with its rotations 2.5 -> 1.9,
// back-transformation 2.2 -> 0.6, in all 7.8 -> 4.4 ms; n = 512 33 -> 14 ms.
void hermitian_eig(const std::vector<cplx>& Ain, int n, std::vector<double>& w, std::vector<cplx>& V) {
  Pool pool((size_t)n * n * n);
  const DenseOps ops = dense_ops();
  std::vector<cplx> A = Ain;
  // use the lower triangle; make A exactly Hermitian from it
  for (int i = 0; i < n; ++i) {
    A[(size_t)i * n + i] = A[(size_t)i * n + i].real();
    for (int j = 0; j < i; ++j) A[(size_t)j * n + i] = std::conj(A[(size_t)i * n + j]);
  }
  std::vector<std::vector<cplx>> vs(std::max(0, n - 2));
  std::vector<cplx> offd(std::max(0, n - 1), 0.0);
  std::vector<double> d(n), e(std::max(1, n));
  // the pending update A -= 2 (v q^H + q v^H), v the vector of the reflector before, and
  // the new vector x: two buffers in turn, so that v is in the threads' caches already
  std::vector<cplx> buf[2] = {std::vector<cplx>(n, 0.0), std::vector<cplx>(n, 0.0)}, q(n, 0.0), p(n);
  const auto row = [&](int i, int from, const std::vector<cplx>& v, const std::vector<cplx>& x, cplx* out) {
    ops.update_dot(reinterpret_cast<double*>(&A[(size_t)i * n + from]), 2 * (n - from),
                   reinterpret_cast<const double*>(&q[from]), reinterpret_cast<const double*>(&v[from]),
                   reinterpret_cast<const double*>(&x[from]), 2.0 * v[i].real(), 2.0 * v[i].imag(), 2.0 * q[i].real(),
                   2.0 * q[i].imag(), reinterpret_cast<double*>(out));
  };
  cplx unused;
  for (int k = 0; k + 2 < n; ++k) {
    std::vector<cplx>&v = buf[(k & 1) ^ 1], &x = buf[k & 1];
    row(k, k, v, x, &unused);
    d[k] = A[(size_t)k * n + k].real();
    const int m = n - k - 1;               // size of the trailing block
    const cplx* Ak = &A[(size_t)k * n];
    double xn2 = 0.0;
    for (int i = k + 1; i < n; ++i) {
      x[i] = std::conj(Ak[i]);             // column k
      xn2 += std::norm(x[i]);
    }
    const double xn = std::sqrt(xn2);
    if (xn != 0.0) {
      const cplx x0 = x[k + 1];
      const cplx phase = (std::abs(x0) > 0.0) ? x0 / std::abs(x0) : cplx(1.0, 0.0);
      const cplx alpha = -phase * xn;
      x[k + 1] -= alpha;
      double vn = 0.0;
      for (int i = k + 1; i < n; ++i) vn += std::norm(x[i]);
      vn = std::sqrt(vn);
      for (int i = k + 1; i < n; ++i) x[i] /= vn;
      offd[k] = alpha;
      vs[k].assign(x.begin() + k + 1, x.end());
    }                                      // (else x = 0: the pass only updates)
    const auto pass = [&](int t, int nt) {
      // rows by eights, so that no two threads write one line of p
      for (int b = (k + 1) / 8; 8 * b < n; ++b) {
        if (b % nt != t) continue;
        for (int i = std::max(k + 1, 8 * b); i < std::min(n, 8 * b + 8); ++i) row(i, k + 1, v, x, &p[i]);
      }
    };
    if ((size_t)m * m > 8192) pool.run(pass);
    else pass(0, 1);
    // the new pending update: rho = x^H p, q = p - rho x
    double rho = 0.0;
    for (int i = k + 1; i < n; ++i) rho += x[i].real() * p[i].real() + x[i].imag() * p[i].imag();
    for (int i = k + 1; i < n; ++i) q[i] = cplx(p[i].real() - rho * x[i].real(), p[i].imag() - rho * x[i].imag());
  }
  for (int i = std::max(0, n - 2); i < n; ++i) {
    row(i, std::max(0, n - 2), buf[(n & 1) ^ 1], buf[n & 1], &unused);    // the last x was buf[(n - 3) & 1]
    d[i] = A[(size_t)i * n + i].real();
  }
  if (n >= 2) offd[n - 2] = A[(size_t)(n - 1) * n + n - 2];
  // phases phi_0 = 1, phi_{k+1} = phi_k e_k / |e_k| make the tridiagonal real
  std::vector<cplx> phi(n, 1.0);
  for (int k = 0; k + 1 < n; ++k) {
    const double a = std::abs(offd[k]);
    e[k] = a;
    phi[k + 1] = (a > 0.0) ? phi[k] * offd[k] / a : phi[k];
  }
  std::vector<double> Z;
  tridiag_vectors(d, e, Z, n, pool, ops);
  // sort ascending
  std::vector<int> order(n);
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return d[a] < d[b]; });
  w.resize(n);
  // V[:, j] = Q (phi .* z_order[j])
  V.resize((size_t)n * n);
  for (int j = 0; j < n; ++j) w[j] = d[order[j]];
  // Q = H_0 H_1 ... H_{n-3} applied to V, H_k = I - 2 v_k v_k^H (v_k unit, nonzero
  // from row k+1).  The reflectors go in blocks of kWY consecutive ones, each block
  // H_k1 ... H_k2 = I - Y T Y^H (compact WY form: Y = [v_k1 .. v_k2], T upper
  // triangular, T_ii = 2, T[0:i, i] = -2 T[0:i, 0:i] (Y[:, 0:i]^H v_i)), applied as
  // V_sub -= Y (T (Y^H V_sub)), last block first; each worker takes its own range of
  // columns (the columns are independent).
  constexpr int kWY = 32;
  const int nref = std::max(0, n - 2);
  struct Blk {
    int k1, k2;                 // reflectors k1..k2
    std::vector<cplx> Y;        // [m1][nb], rows k1+1 .. n-1 (zero above each v's start)
    std::vector<cplx> T;        // [nb][nb] upper
  };
  std::vector<Blk> blks((nref + kWY - 1) / kWY);
  const auto build = [&](Blk& B, int k1) {
    B.k1 = k1;
    B.k2 = std::min(nref, k1 + kWY) - 1;
    const int nb = B.k2 - B.k1 + 1, m1 = n - k1 - 1;
    B.Y.assign((size_t)m1 * nb, 0.0);
    for (int j = 0; j < nb; ++j) {
      const auto& v = vs[k1 + j];
      if (v.empty()) continue;
      for (size_t i = 0; i < v.size(); ++i) B.Y[(size_t)(j + i) * nb + j] = v[i];   // v_k starts at row k+1
    }
    B.T.assign((size_t)nb * nb, 0.0);
    std::vector<cplx> g(nb);
    for (int i = 0; i < nb; ++i) {
      if (vs[k1 + i].empty()) continue;      // H = I: zero column of Y, T_ii = 0
      // g[0:i] = Y[:, 0:i]^H v_i
      std::fill(g.begin(), g.end(), 0.0);
      for (int r = i; r < m1; ++r) {
        const cplx* Yr = &B.Y[(size_t)r * nb];
        const double a = Yr[i].real(), b = Yr[i].imag();
        for (int j = 0; j < i; ++j)
          g[j] += cplx(Yr[j].real() * a + Yr[j].imag() * b, Yr[j].real() * b - Yr[j].imag() * a);
      }
      for (int j = 0; j < i; ++j) {
        cplx acc = 0.0;
        for (int l = j; l < i; ++l) acc += B.T[(size_t)j * nb + l] * g[l];
        B.T[(size_t)j * nb + i] = -2.0 * acc;
      }
      B.T[(size_t)i * nb + i] = 2.0;
    }
  };
  pool.run([&](int t, int nt) {
    for (size_t b = t; b < blks.size(); b += nt) build(blks[b], (int)b * kWY);
  });
  pool.run([&](int t, int nt) {
    int lo, hi;
    Pool::range(n, t, nt, lo, hi);
    if (lo >= hi) return;
    const int nc = hi - lo, w2 = 2 * nc;
    // this worker's columns together (rows of V are a multiple of the cache's period apart)
    std::vector<cplx> U((size_t)n * nc);
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < nc; ++j)
        U[(size_t)i * nc + j] = phi[i] * Z[((size_t)(i / 8) * n + order[lo + j]) * 8 + i % 8];
    std::vector<double> W((size_t)kWY * w2), W2((size_t)kWY * w2);
    for (int bi = (int)blks.size() - 1; bi >= 0; --bi) {
      const Blk& B = blks[bi];
      const int nb = B.k2 - B.k1 + 1, m1 = n - B.k1 - 1, r0 = B.k1 + 1;
      // W = Y^H V_sub (interleaved re, im)
      std::fill(W.begin(), W.begin() + (size_t)nb * w2, 0.0);
      for (int r = 0; r < m1; ++r) {
        const double* __restrict__ Vr = reinterpret_cast<const double*>(&U[(size_t)(r0 + r) * nc]);
        const cplx* Yr = &B.Y[(size_t)r * nb];
        const int jmax = std::min(nb, r + 1);      // v_{k1+j} starts at row j of the block
        for (int j = 0; j < jmax; ++j) ops.caxpy(&W[(size_t)j * w2], Vr, Yr[j].real(), -Yr[j].imag(), w2);
      }
      // W2 = T W
      for (int j = 0; j < nb; ++j) {
        double* __restrict__ W2j = &W2[(size_t)j * w2];
        std::fill(W2j, W2j + w2, 0.0);
        for (int l = j; l < nb; ++l) {
          const cplx tl = B.T[(size_t)j * nb + l];
          ops.caxpy(W2j, &W[(size_t)l * w2], tl.real(), tl.imag(), w2);
        }
      }
      // V_sub -= Y W2
      for (int r = 0; r < m1; ++r) {
        double* __restrict__ Vr = reinterpret_cast<double*>(&U[(size_t)(r0 + r) * nc]);
        const cplx* Yr = &B.Y[(size_t)r * nb];
        const int jmax = std::min(nb, r + 1);
        for (int j = 0; j < jmax; ++j) ops.caxpy(Vr, &W2[(size_t)j * w2], -Yr[j].real(), -Yr[j].imag(), w2);
      }
    }
    for (int i = 0; i < n; ++i) std::copy(&U[(size_t)i * nc], &U[(size_t)i * nc] + nc, &V[(size_t)i * n + lo]);
  });
}

void tridiag_eigvals(std::vector<double> d, std::vector<double> e, std::vector<double>& w) {
  const int n = (int)d.size();
  tridiag_ql(d, e, n, nullptr);
  std::sort(d.begin(), d.end());
  w = d;
}

}  // namespace chfsi
