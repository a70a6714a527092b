// One-sided (Hestenes) Jacobi SVD in FP64 and the truncated-SVD
// pseudo-inverse used to solve the KIFMM matching equations (Methods, Fast
// multipole method: the equivalent densities are found by matching
// check-surface potentials and solving the resulting linear systems).
//
// Column pairs are rotated until every pair is orthogonal to working
// precision; the column norms are then the singular values.  The
// pseudo-inverse keeps singular values above tau * s_max.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <map>
#include <thread>
#include <vector>

// Host functions built for AVX2 as well, chosen at run time (this file also
// passes through the device compiler, which knows no such targets).
#ifdef __HIP_DEVICE_COMPILE__
#define HOST_CLONES
#else
#define HOST_CLONES __attribute__((target_clones("avx2", "default")))
#endif

namespace fmm {

// C (m x p, ldc) = A (m x k, lda) * B (k x p, ldb), four rows of C at a time
// (each row of B read once for the four); every element of C is the sum over
// k in ascending order.  No clone may contract to fused multiply-adds: the
// operators' bits must not depend on the machine.
HOST_CLONES void matmul_rect(int m, int k, int p, const double *A, int lda, const double *B, int ldb, double *C, int ldc) {
  for (int i = 0; i < m; i += 4) {
    const int rows = std::min(4, m - i);
    for (int r = 0; r < rows; ++r) std::fill(C + (size_t)(i + r) * ldc, C + (size_t)(i + r) * ldc + p, 0.0);
    const double *a0 = A + (size_t)i * lda, *a1 = a0 + (rows > 1 ? lda : 0), *a2 = a0 + (rows > 2 ? 2 * (size_t)lda : 0),
                 *a3 = a0 + (rows > 3 ? 3 * (size_t)lda : 0);
    double *__restrict__ c0 = C + (size_t)i * ldc;
    if (rows == 4) {
      double *__restrict__ c1 = c0 + ldc, *__restrict__ c2 = c1 + ldc, *__restrict__ c3 = c2 + ldc;
      for (int kk = 0; kk < k; ++kk) {
        const double *__restrict__ b = B + (size_t)kk * ldb;
        const double x0 = a0[kk], x1 = a1[kk], x2 = a2[kk], x3 = a3[kk];
        for (int j = 0; j < p; ++j) {
          const double y = b[j];
          c0[j] += x0 * y;
          c1[j] += x1 * y;
          c2[j] += x2 * y;
          c3[j] += x3 * y;
        }
      }
    } else {
      for (int r = 0; r < rows; ++r) {
        const double *a = A + (size_t)(i + r) * lda;
        double *__restrict__ c = C + (size_t)(i + r) * ldc;
        for (int kk = 0; kk < k; ++kk) {
          const double x = a[kk];
          const double *__restrict__ b = B + (size_t)kk * ldb;
          for (int j = 0; j < p; ++j) c[j] += x * b[j];
        }
      }
    }
  }
}

// Threads of one SVD meet at a barrier after every round of rotations.
struct SpinBarrier {
  explicit SpinBarrier(int n) : n_(n) {}
  void wait() {
    const int g = gen_.load(std::memory_order_acquire);
    if (count_.fetch_add(1, std::memory_order_acq_rel) + 1 == n_) {
      count_.store(0, std::memory_order_relaxed);
      gen_.fetch_add(1, std::memory_order_acq_rel);
    } else {
      while (gen_.load(std::memory_order_acquire) == g) std::this_thread::yield();
    }
  }
  std::atomic<int> count_{0}, gen_{0};
  const int n_;
};

// A: m x n row-major (m >= n).  Returns U (m x n, row-major), s (n), V (n x n,
// row-major) with A = U diag(s) V^T, s unsorted.  Each sweep visits every
// column pair once in the round-robin order (n - 1 rounds of disjoint pairs,
// a dummy column when n is odd); the pairs of a round are independent and
// are shared by `nthreads` threads, each pair rotated by the same arithmetic
// whichever thread takes it, so the result does not depend on the thread
// count.
static void jacobi_svd(int m, int n, const double *A, std::vector<double> &U,
                       std::vector<double> &s, std::vector<double> &V, int nthreads) {
  // work column-major for contiguous column access
  std::vector<double> a((size_t)m * n), v((size_t)n * n, 0.0);
  for (int i = 0; i < m; ++i)
    for (int j = 0; j < n; ++j) a[(size_t)j * m + i] = A[(size_t)i * n + j];
  for (int j = 0; j < n; ++j) v[(size_t)j * n + j] = 1.0;
  std::vector<double> nrm(n);
  for (int j = 0; j < n; ++j) {
    double t = 0;
    const double *c = &a[(size_t)j * m];
    for (int i = 0; i < m; ++i) t += c[i] * c[i];
    nrm[j] = t;
  }
  const double eps = 1e-15;
  const int N = n + (n & 1);  // with a dummy column when n is odd
  auto rotate = [&](int p, int q) -> int {
    double *cp = &a[(size_t)p * m], *cq = &a[(size_t)q * m];
    const double alpha = nrm[p], beta = nrm[q];
    double gamma = 0;
    for (int i = 0; i < m; ++i) gamma += cp[i] * cq[i];
    if (std::fabs(gamma) <= eps * std::sqrt(alpha * beta) || gamma == 0.0) return 0;
    const double zeta = (beta - alpha) / (2.0 * gamma);
    const double t = (zeta >= 0 ? 1.0 : -1.0) / (std::fabs(zeta) + std::sqrt(1.0 + zeta * zeta));
    const double c = 1.0 / std::sqrt(1.0 + t * t), sn = c * t;
    double np = 0, nq = 0;
    for (int i = 0; i < m; ++i) {
      const double x = cp[i], y = cq[i];
      const double xn = c * x - sn * y, yn = sn * x + c * y;
      cp[i] = xn;
      cq[i] = yn;
      np += xn * xn;
      nq += yn * yn;
    }
    nrm[p] = np;
    nrm[q] = nq;
    double *vp = &v[(size_t)p * n], *vq = &v[(size_t)q * n];
    for (int i = 0; i < n; ++i) {
      const double x = vp[i], y = vq[i];
      vp[i] = c * x - sn * y;
      vq[i] = sn * x + c * y;
    }
    return 1;
  };
  // pair k of round r (circle method over N columns)
  auto pair_of = [&](int r, int k, int &p, int &q) {
    int x = (r + k) % (N - 1), y = (r - k + N - 1) % (N - 1);
    if (k == 0) y = N - 1;
    p = std::min(x, y);
    q = std::max(x, y);
  };
  const int nth = std::max(1, std::min(nthreads, N / 2));
  SpinBarrier bar(nth);
  std::vector<int> rot(nth, 0);
  std::atomic<bool> done{false};
  auto worker = [&](int tid) {
    for (int sweep = 0; sweep < 60; ++sweep) {
      rot[tid] = 0;
      for (int r = 0; r < N - 1; ++r) {
        for (int k = tid; k < N / 2; k += nth) {
          int p, q;
          pair_of(r, k, p, q);
          if (q < n) rot[tid] += rotate(p, q);
        }
        bar.wait();
      }
      if (tid == 0) {
        int total = 0;
        for (int t = 0; t < nth; ++t) total += rot[t];
        done.store(total == 0, std::memory_order_release);
      }
      bar.wait();
      if (done.load(std::memory_order_acquire)) break;
      bar.wait();  // every thread has read `done` before the next sweep resets its count
    }
  };
  if (N >= 2) {
    std::vector<std::thread> th;
    for (int t = 1; t < nth; ++t) th.emplace_back(worker, t);
    worker(0);
    for (auto &t : th) t.join();
  }
  s.assign(n, 0.0);
  U.assign((size_t)m * n, 0.0);
  V.assign((size_t)n * n, 0.0);
  for (int j = 0; j < n; ++j) {
    double t = 0;
    const double *c = &a[(size_t)j * m];
    for (int i = 0; i < m; ++i) t += c[i] * c[i];
    s[j] = std::sqrt(t);
    for (int i = 0; i < m; ++i) U[(size_t)i * n + j] = s[j] > 0 ? c[i] / s[j] : 0.0;
    for (int i = 0; i < n; ++i) V[(size_t)i * n + j] = v[(size_t)j * n + i];
  }
}

// Truncated SVD factors of A (n x n): singular values above tau * s_max,
// sorted in decreasing order, are kept (rank r).  UT (n x n, row-major) gets
// U^T in its first r rows and zeros below; VS (n x n, row-major) gets
// V diag(1/s) in its first r columns and zeros to the right, so that
// pinv(A) = VS * UT.  Returns r.
int tsvd_factors(int n, const double *A, double tau, double *UT, double *VS, int nthreads) {
  std::vector<double> U, s, V;
  jacobi_svd(n, n, A, U, s, V, nthreads);
  std::vector<int> order(n);
  for (int j = 0; j < n; ++j) order[j] = j;
  std::sort(order.begin(), order.end(), [&](int a, int b) { return s[a] > s[b]; });
  const double smax = n ? s[order[0]] : 0.0;
  int r = 0;
  while (r < n && s[order[r]] > tau * smax) ++r;
  std::fill(UT, UT + (size_t)n * n, 0.0);
  std::fill(VS, VS + (size_t)n * n, 0.0);
  for (int k = 0; k < r; ++k) {
    const int j = order[k];
    for (int i = 0; i < n; ++i) {
      UT[(size_t)k * n + i] = U[(size_t)i * n + j];
      VS[(size_t)i * n + k] = V[(size_t)i * n + j] / s[j];
    }
  }
  return r;
}

// The same factors for a matrix A between two surfaces that are both the grid
// `grid` (n x 3, symmetric under x -> -x, y -> -y, z -> -z) about one centre,
// with a radial kernel: A commutes with the three reflections, so it is block
// diagonal in vectors even or odd in each coordinate, and every singular
// vector can be taken from one of the eight classes.  code[k] (bit 2: odd in
// x, bit 1: y, bit 0: z) is the class of column k: reflecting the axes in
// mask m multiplies it by (-1)^popcount(code[k] & m), which lets one operator
// serve every reflected offset.  Returns r, the number of singular values
// above tau * s_max (over all classes); their columns fill 16-wide blocks of
// one class each where that takes no more than ceil(r / 16) blocks, so that an
// operator between reflection-symmetric boxes has whole zero tiles.  Columns
// left empty are zero, with code 255.  UT is ldv x n and VS n x ldv, ldv = n
// rounded up to 16.  Each class holds about n / 8
// vectors, so its SVD costs 1/512 of the whole one.
int tsvd_factors_parity(int n, const double *grid, const double *A, double tau, double *UT, double *VS, int ldv,
                        unsigned char *code) {
  auto find = [&](double x, double y, double z) {
    for (int i = 0; i < n; ++i)
      if (std::fabs(grid[3 * i] - x) < 1e-9 && std::fabs(grid[3 * i + 1] - y) < 1e-9 &&
          std::fabs(grid[3 * i + 2] - z) < 1e-9)
        return i;
    return -1;
  };
  // one representative per orbit (all coordinates >= 0) and its eight images
  std::vector<std::vector<int>> orbit;
  for (int i = 0; i < n; ++i) {
    const double *g = grid + 3 * i;
    if (g[0] < -1e-9 || g[1] < -1e-9 || g[2] < -1e-9) continue;
    std::vector<int> im(8);
    for (int m = 0; m < 8; ++m)
      im[m] = find(m & 4 ? -g[0] : g[0], m & 2 ? -g[1] : g[1], m & 1 ? -g[2] : g[2]);
    orbit.push_back(im);
  }
  struct Val { double s; int cls, col; };
  std::vector<Val> vals;
  std::vector<std::vector<double>> QU(8), QV(8);  // per class: n x nc, columns of U and V
  std::vector<int> nc(8, 0);
  std::vector<double> B, U, s, V;
  for (int c = 0; c < 8; ++c) {
    // orthonormal basis of the class: one vector per orbit that carries it,
    // with equal weights up to sign on the orbit's points
    std::vector<std::vector<std::pair<int, double>>> Q;
    for (const std::vector<int> &im : orbit) {
      std::map<int, double> v;
      for (int f = 0; f < 8; ++f) v[im[f]] += (__builtin_popcount(c & f) & 1) ? -1.0 : 1.0;
      double t = 0;
      for (const auto &e : v) t += e.second * e.second;
      if (t < 0.5) continue;
      Q.emplace_back();
      for (const auto &e : v) Q.back().push_back({e.first, e.second / std::sqrt(t)});
    }
    const int m = (int)Q.size();
    nc[c] = m;
    if (m == 0) continue;
    B.assign((size_t)m * m, 0.0);
    for (int a = 0; a < m; ++a)
      for (const auto &x : Q[a])
        for (int b = 0; b < m; ++b)
          for (const auto &y : Q[b]) B[(size_t)a * m + b] += x.second * A[(size_t)x.first * n + y.first] * y.second;
    jacobi_svd(m, m, B.data(), U, s, V, 1);
    QU[c].assign((size_t)n * m, 0.0);
    QV[c].assign((size_t)n * m, 0.0);
    for (int a = 0; a < m; ++a)
      for (const auto &x : Q[a])
        for (int k = 0; k < m; ++k) {
          QU[c][(size_t)x.first * m + k] += x.second * U[(size_t)a * m + k];
          QV[c][(size_t)x.first * m + k] += x.second * V[(size_t)a * m + k];
        }
    for (int k = 0; k < m; ++k) vals.push_back({s[k], c, k});
  }
  double smax = 0;
  for (const Val &v : vals) smax = std::max(smax, v.s);
  std::sort(vals.begin(), vals.end(), [](const Val &a, const Val &b) { return a.cls != b.cls ? a.cls < b.cls : a.s > b.s; });
  // columns by 16: whole blocks of one class first; the classes' remainders
  // share blocks (first fit, largest first), split over blocks only where
  // that would take more blocks than there are columns for
  std::vector<std::vector<int>> kept(8), block;
  std::vector<std::pair<int, std::vector<int>>> rest;
  int r = 0;
  for (int i = 0; i < (int)vals.size(); ++i)
    if (vals[i].s > tau * smax) { kept[vals[i].cls].push_back(i); ++r; }
  for (const std::vector<int> &k : kept) {
    size_t i = 0;
    for (; i + 16 <= k.size(); i += 16) block.emplace_back(k.begin() + i, k.begin() + i + 16);
    if (i < k.size()) rest.push_back({-(int)(k.size() - i), std::vector<int>(k.begin() + i, k.end())});
  }
  std::stable_sort(rest.begin(), rest.end(), [](const auto &a, const auto &b) { return a.first < b.first; });
  const size_t full = block.size(), want = (size_t)(r + 15) / 16;
  for (const auto &g : rest) {
    size_t b = full;
    while (b < block.size() && block[b].size() + g.second.size() > 16) ++b;
    if (b == block.size()) block.emplace_back();
    block[b].insert(block[b].end(), g.second.begin(), g.second.end());
  }
  if (block.size() > want) {
    block.resize(full);
    for (const auto &g : rest)
      for (int i : g.second) {
        if (block.size() == full || block.back().size() == 16) block.emplace_back();
        block.back().push_back(i);
      }
  }
  std::fill(UT, UT + (size_t)ldv * n, 0.0);
  std::fill(VS, VS + (size_t)n * ldv, 0.0);
  std::fill(code, code + 16 * want, (unsigned char)255);
  for (size_t b = 0; b < block.size(); ++b)
    for (size_t j = 0; j < block[b].size(); ++j) {
      const Val &v = vals[block[b][j]];
      const int m = nc[v.cls];
      const size_t k = 16 * b + j;
      for (int i = 0; i < n; ++i) {
        UT[k * n + i] = QU[v.cls][(size_t)i * m + v.col];
        VS[(size_t)i * ldv + k] = QV[v.cls][(size_t)i * m + v.col] / v.s;
      }
      code[k] = (unsigned char)v.cls;
    }
  return r;
}

// Low-rank split of A (rows x cols, row-major): with A = U S V^T and the k
// singular values above tau * s_max kept (decreasing order),
// L = U_k S_k^{1/2} (rows x k, row-major, leading dimension ldl) and
// R = S_k^{1/2} V_k^T (k x cols, row-major, leading dimension ldr), so that
// A ~ L R.  Returns k (0 for a zero matrix).
int tsvd_split(int rows, int cols, const double *A, double tau, double *L, int ldl, double *R, int ldr) {
  // the one-sided Jacobi SVD wants at least as many rows as columns: work on
  // the transpose when A is wide
  const bool tr = rows < cols;
  const int m = tr ? cols : rows, n = tr ? rows : cols;
  std::vector<double> B((size_t)m * n);
  for (int i = 0; i < rows; ++i)
    for (int j = 0; j < cols; ++j) {
      if (tr) B[(size_t)j * n + i] = A[(size_t)i * cols + j];
      else B[(size_t)i * n + j] = A[(size_t)i * cols + j];
    }
  std::vector<double> U, s, V;
  jacobi_svd(m, n, B.data(), U, s, V, 1);
  std::vector<int> order(n);
  for (int j = 0; j < n; ++j) order[j] = j;
  std::sort(order.begin(), order.end(), [&](int a, int b) { return s[a] > s[b]; });
  const double smax = n ? s[order[0]] : 0.0;
  int k = 0;
  while (k < n && s[order[k]] > tau * smax && s[order[k]] > 0.0) ++k;
  // B = U S V^T (m x n); A = B or B^T
  for (int c = 0; c < k; ++c) {
    const int j = order[c];
    const double h = std::sqrt(s[j]);
    for (int i = 0; i < rows; ++i) L[(size_t)i * ldl + c] = h * (tr ? V[(size_t)i * n + j] : U[(size_t)i * n + j]);
    for (int i = 0; i < cols; ++i) R[(size_t)c * ldr + i] = h * (tr ? U[(size_t)i * n + j] : V[(size_t)i * n + j]);
  }
  return k;
}

// out (n x n row-major) = pinv(A) with singular values <= tau * s_max dropped.
void pinv_tsvd(int n, const double *A, double tau, double *out) {
  std::vector<double> U, s, V;
  jacobi_svd(n, n, A, U, s, V, 1);
  double smax = 0;
  for (double x : s) smax = std::max(smax, x);
  std::vector<double> sinv(n, 0.0);
  for (int j = 0; j < n; ++j)
    if (s[j] > tau * smax) sinv[j] = 1.0 / s[j];
  // out = V diag(sinv) U^T
  for (int i = 0; i < n; ++i)
    for (int k = 0; k < n; ++k) {
      double t = 0;
      for (int j = 0; j < n; ++j) t += V[(size_t)i * n + j] * sinv[j] * U[(size_t)k * n + j];
      out[(size_t)i * n + k] = t;
    }
}

}  // namespace fmm
