// Small dense Hermitian problems of the subspace iteration, one workgroup per
// matrix (nb <= 64), entirely on the device so that an outer iteration needs no
// host round trip and can be recorded in a hipGraph.
//
// Eigenproblems: cyclic two-sided Jacobi with the round-robin (tournament)
// ordering, nb/2 disjoint rotations per round applied in parallel; a complex
// rotation [[c, sigma], [-conj(sigma), c]] annihilates one 2x2 Hermitian block.
// Converges quadratically to full FP64 accuracy.
//
//   heev_kernel, mode 0:  A -> eigenvalues ascending + eigenvectors Q[v][w]
//   heev_kernel, mode 1 (orthonormaliser of a Gram matrix G):  T with X T
//         orthonormal.  A Gram matrix that is provably well conditioned takes
//         the Cholesky factor of its scaled form, D G D = L L^H, T = D L^-H; any
//         other the eigen-decomposition (SVQB), D G D = U diag(lambda) U^H,
//         T = D U diag(lambda)^-1/2, with D = diag(G)^-1/2.
//   rr_kernel (Rayleigh-Ritz step):  S^H M S -> eigenvalues and T = S Q
//
// Why Cholesky first: a filtered block of nearly converged Ritz vectors has a
// Gram matrix near the identity.  Its eigenvalues cluster at 1, so the
// eigenvectors are an arbitrary dense mixture of the block: Jacobi needed 9-12
// sweeps to find them, and the projected matrix S^H M S, dense in that basis,
// another 9-12.  The triangular factor is nb short steps and stays near the
// identity, so S^H M S is nearly diagonal and Jacobi ends in a few sweeps.
//
// Also: the control kernel that turns Ritz values and residuals into the
// convergence flags and the next Chebyshev filter coefficients.
#include "hkp_internal.h"

namespace hkp {

namespace {

constexpr int kNBP = HKP_NB_MAX;   // padded size (even)
constexpr int kMaxItems = 3;       // work items of a thread in a Jacobi round

struct Rot {
  double c, sr, si;   // cos, sigma = sin e^{i phi}
  int p, q;
};

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}

// Threads of a Jacobi workgroup on n players (even): one work item each where that
// fits (n (n / 2) slices of V and the pair blocks on and above the diagonal).  What
// bounds a round is its chain (rotation parameters, barrier, update, barrier); idle
// waves would only lengthen the barriers.
__host__ __device__ inline int jacobi_threads(int n) {
  const int h = n / 2, items = h * (h + 1) / 2 + n * h;
  const int t = (items + 63) / 64 * 64;
  return t > 1024 ? 1024 : t;
}

// Eigen-decomposition of the Hermitian n x n matrix in a (n even, LDS, row length
// NBP + 1): its diagonal becomes the eigenvalues, v (set to I here) the
// eigenvectors.  rel_only: rotate by the relative test alone, else also ignore
// entries below 1e-3 eps of the Frobenius norm (a diagonal that may be ~0).
template <int NBP>
__device__ __forceinline__ void jacobi(double2 (*a)[NBP + 1], double2 (*v)[NBP + 1], Rot* rot,
                                       int n, bool rel_only, double frob, int* any_rot) {
  const int tid = threadIdx.x, nt = blockDim.x;
  const int h = n / 2, nup = h * (h + 1) / 2, m = n - 1;
  for (int t = tid; t < n * n; t += nt) {
    const int i = t / n, j = t - i * n;
    v[i][j] = make_double2(i == j ? 1.0 : 0.0, 0.0);
    if (i == j) a[i][i].y = 0.0;
  }
  // this thread's items, fixed for every round: pair blocks (P <= Q), row by row, then
  // the (row, pair) slices of V
  int item[kMaxItems];   // P << 8 | Q, or 1 << 16 | row << 8 | pair; -1: none
#pragma unroll
  for (int u = 0; u < kMaxItems; ++u) {
    const int t = tid + u * nt;
    item[u] = -1;
    if (t < nup) {
      int P = 0, rem = t;
      while (rem >= h - P) {
        rem -= h - P;
        ++P;
      }
      item[u] = (P << 8) | (P + rem);
    } else if (t < nup + n * h) {
      const int w = t - nup, i = w / h;
      item[u] = (1 << 16) | (i << 8) | (w - i * h);
    }
  }
  const double eps = 2.220446049250313e-16;
  const double thr = rel_only ? 0.0 : 1e-3 * eps * frob;
  const double thr2 = thr * thr, eps2 = 0.25 * eps * eps;
  // pair `tid` of round 0 (the tournament's players move on by one each round and
  // are back at the start after n - 1 rounds)
  int pa = tid == 0 ? m : tid, pb = tid == 0 ? 0 : m - tid;
  __syncthreads();
  for (int sweep = 0; sweep < 40; ++sweep) {
    if (tid == 0) *any_rot = 0;
    __syncthreads();
    for (int round = 0; round < m; ++round) {
      if (tid < h) {
        // rotation parameters: with r = sqrt(d^2 + 4 |apq|^2), d = aqq - app,
        // c^2 = (1 + |d| / r) / 2 and sin = sgn(d) |apq| / (r c); two reciprocal
        // square roots in the chain instead of three roots and three divisions
        const int p = pa < pb ? pa : pb, q = pa < pb ? pb : pa;
        const double app = a[p][p].x, aqq = a[q][q].x;
        const double2 apq = a[p][q];
        const double m2 = fma(apq.x, apq.x, apq.y * apq.y);
        Rot r;
        r.p = p;
        r.q = q;
        r.c = 1.0;
        r.sr = r.si = 0.0;
        if (m2 > eps2 * fabs(app * aqq) && m2 > thr2) {
          const double d = aqq - app;
          const double ri = rsqrt(fma(d, d, 4.0 * m2));
          const double c2 = fma(0.5 * fabs(d), ri, 0.5);
          const double ci = rsqrt(c2);
          const double f = (d >= 0.0 ? ri : -ri) * ci;
          r.c = c2 * ci;
          r.sr = apq.x * f;
          r.si = apq.y * f;
          *any_rot = 1;
        }
        rot[tid] = r;
        if (tid != 0) pa = pa + 1 == m ? 0 : pa + 1;
        pb = pb + 1 == m ? 0 : pb + 1;
      }
      __syncthreads();
      // A <- N^H A N and V <- V N with N block diagonal over the pairs: every 2x2
      // block of A (pair P rows, pair Q columns) with P <= Q and every (row, pair)
      // slice of V is owned by one thread, so one phase updates everything in place;
      // the block (Q, P) is written as the conjugate transpose of (P, Q), which
      // keeps A exactly Hermitian
#pragma unroll
      for (int u = 0; u < kMaxItems; ++u) {
        if (item[u] < 0) continue;
        const int hi = (item[u] >> 8) & 255, lo = item[u] & 255;
        const Rot rq = rot[lo];
        const double2 sg = make_double2(rq.sr, rq.si), sgc = make_double2(rq.sr, -rq.si);
        const bool qz = rq.sr == 0.0 && rq.si == 0.0;
        if (item[u] >> 16) {
          if (qz) continue;
          const double2 xp = v[hi][rq.p], xq = v[hi][rq.q];
          const double2 u0 = cmul(sgc, xq), u1 = cmul(sg, xp);
          v[hi][rq.p] = make_double2(fma(rq.c, xp.x, -u0.x), fma(rq.c, xp.y, -u0.y));
          v[hi][rq.q] = make_double2(fma(rq.c, xq.x, u1.x), fma(rq.c, xq.y, u1.y));
          continue;
        }
        const Rot rp = rot[hi];
        const bool pz = rp.sr == 0.0 && rp.si == 0.0;
        if (pz && qz) continue;
        double2 a00 = a[rp.p][rq.p], a01 = a[rp.p][rq.q];
        double2 a10 = a[rp.q][rq.p], a11 = a[rp.q][rq.q];
        if (!qz) {   // columns: p <- c p - conj(sigma) q, q <- sigma p + c q
          const double2 e01 = cmul(sgc, a01), e11 = cmul(sgc, a11);
          const double2 e00 = cmul(sg, a00), e10 = cmul(sg, a10);
          a00 = make_double2(fma(rq.c, a00.x, -e01.x), fma(rq.c, a00.y, -e01.y));
          a01 = make_double2(fma(rq.c, a01.x, e00.x), fma(rq.c, a01.y, e00.y));
          a10 = make_double2(fma(rq.c, a10.x, -e11.x), fma(rq.c, a10.y, -e11.y));
          a11 = make_double2(fma(rq.c, a11.x, e10.x), fma(rq.c, a11.y, e10.y));
        }
        if (!pz) {   // rows: p <- c p - sigma q, q <- conj(sigma) p + c q
          const double2 tg = make_double2(rp.sr, rp.si), tgc = make_double2(rp.sr, -rp.si);
          const double2 e10 = cmul(tg, a10), e11 = cmul(tg, a11);
          const double2 e00 = cmul(tgc, a00), e01 = cmul(tgc, a01);
          a00 = make_double2(fma(rp.c, a00.x, -e10.x), fma(rp.c, a00.y, -e10.y));
          a01 = make_double2(fma(rp.c, a01.x, -e11.x), fma(rp.c, a01.y, -e11.y));
          a10 = make_double2(fma(rp.c, a10.x, e00.x), fma(rp.c, a10.y, e00.y));
          a11 = make_double2(fma(rp.c, a11.x, e01.x), fma(rp.c, a11.y, e01.y));
        }
        if (hi == lo) {
          // the rotated pair itself: annihilated entry exactly zero, real diagonal
          a01 = make_double2(0, 0);
          a10 = make_double2(0, 0);
          a00.y = 0.0;
          a11.y = 0.0;
        }
        a[rp.p][rq.p] = a00;
        a[rp.p][rq.q] = a01;
        a[rp.q][rq.p] = a10;
        a[rp.q][rq.q] = a11;
        if (hi != lo) {
          a[rq.p][rp.p] = make_double2(a00.x, -a00.y);
          a[rq.q][rp.p] = make_double2(a01.x, -a01.y);
          a[rq.p][rp.q] = make_double2(a10.x, -a10.y);
          a[rq.q][rp.q] = make_double2(a11.x, -a11.y);
        }
      }
      __syncthreads();
    }
    const int go = *any_rot;
    __syncthreads();
    if (!go) break;
  }
}

// sum over the workgroup, the same value in every thread (red: one double a wave)
__device__ __forceinline__ double block_sum(double f, double* red) {
  for (int off = 32; off > 0; off >>= 1) f += __shfl_down(f, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = f;
  __syncthreads();
  double t = 0.0;
  for (int k = 0; k < (int)((blockDim.x + 63) >> 6); ++k) t += red[k];
  __syncthreads();
  return t;
}

template <int NBP>
__device__ __forceinline__ double frobenius(double2 (*a)[NBP + 1], int n, double* red) {
  double f = 0.0;
  for (int t = threadIdx.x; t < n * n; t += blockDim.x) {
    const double2 x = a[t / n][t % n];
    f += x.x * x.x + x.y * x.y;
  }
  return sqrt(block_sum(f, red));
}

// eigenvalues (the diagonal of a) to lam, their ascending order (stable in index) to rank
template <int NBP>
__device__ __forceinline__ void rank_eigenvalues(double2 (*a)[NBP + 1], int n, int nb,
                                                 double* lam, int* rank) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) lam[i] = a[i][i].x;
  __syncthreads();
  for (int i = threadIdx.x; i < nb; i += blockDim.x) {
    int rk = 0;
    const double li = lam[i];
    for (int j = 0; j < nb; ++j) {
      const double lj = lam[j];
      rk += (lj < li) || (lj == li && j < i);
    }
    rank[i] = rk;
  }
  __syncthreads();
}

// Cholesky factor and the inverse of its unit-triangular part, together: A = L diag(d) L^H
// (A, Hermitian with unit diagonal, in a's lower triangle, destroyed), W = L^-1 into
// v's lower triangle, rd = 1 / d.  Step k updates every (i, j <= i), i > k, once: the
// remaining matrix for j > k, row i of W for j <= k; it reads column k of a and row k
// of v, which it does not write, so one barrier per step.  True if every pivot is
// positive and lambda_max / lambda_min <= 1e4 is certain, from lambda_max <= |A|_F and
// 1 / lambda_min <= |diag(d)^-1/2 W|_F^2 (the line below which one pass of either
// orthonormaliser leaves an error of at most 1e4 eps).
template <int NBP>
__device__ __forceinline__ bool cholesky(double2 (*a)[NBP + 1], double2 (*v)[NBP + 1], double* rd,
                                         int n, double frob, double* red, int* bad) {
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int t = tid; t < n * n; t += nt) {
    const int i = t / n, j = t - i * n;
    v[i][j] = make_double2(i == j ? 1.0 : 0.0, 0.0);
  }
  if (tid == 0) {
    *bad = !(a[0][0].x > 0.0);
    rd[0] = 1.0 / a[0][0].x;
  }
  const int nlow = n * (n + 1) / 2;
  __syncthreads();
  for (int k = 0; k + 1 < n; ++k) {
    for (int t = tid; t < nlow; t += nt) {
      // row i of the lower triangle holds entries i (i + 1) / 2 .. i (i + 3) / 2
      int i = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
      if (i * (i + 1) / 2 > t) --i;
      if ((i + 1) * (i + 2) / 2 <= t) ++i;
      if (i <= k) continue;
      const int j = t - i * (i + 1) / 2;
      const double r = rd[k];
      const double2 aik = a[i][k];
      const double2 l = make_double2(aik.x * r, aik.y * r);
      if (j > k) {
        const double2 ajk = a[j][k];
        const double2 p = cmul(l, make_double2(ajk.x, -ajk.y));
        double2 x = make_double2(a[i][j].x - p.x, a[i][j].y - p.y);
        if (i == j) x.y = 0.0;
        a[i][j] = x;
        if (i == k + 1) {   // (k + 1, k + 1): the next pivot
          if (!(x.x > 0.0)) *bad = 1;
          rd[k + 1] = 1.0 / x.x;
        }
      } else {
        const double2 p = cmul(l, v[k][j]);
        v[i][j] = make_double2(v[i][j].x - p.x, v[i][j].y - p.y);
      }
    }
    __syncthreads();
  }
  double f = 0.0;
  for (int t = tid; t < n * n; t += nt) {
    const int i = t / n, j = t - i * n;
    if (j <= i) f += (v[i][j].x * v[i][j].x + v[i][j].y * v[i][j].y) * rd[i];
  }
  const double inv = block_sum(f, red);
  return !*bad && inv * frob <= 1e4;
}

// Launched with jacobi_threads() threads; bound by latency (one workgroup per matrix).
// Orthonormaliser, 40 x 40 matrices of a mixed solve of the 256 x 48 x 48 double dot:
// 528 us with SVQB, 33 us with the Cholesky factor.
__global__ void __launch_bounds__(1024)
heev_kernel(double* A, int nb, long long mat_stride, double* evals, double* out, int mode,
            int* status, const int* active, int* again) {
  __shared__ double2 a[kNBP][kNBP + 1];
  __shared__ double2 v[kNBP][kNBP + 1];
  __shared__ Rot rot[kNBP / 2];
  __shared__ double dscale[kNBP];
  __shared__ double lam[kNBP];
  __shared__ int rank[kNBP];
  __shared__ double red[16];
  __shared__ int flag;

  const int b = blockIdx.x;
  if (active && !active[b]) {
    if (again && threadIdx.x == 0) again[b] = 0;
    return;
  }
  const int tid = threadIdx.x, nt = blockDim.x;
  const int n = nb + (nb & 1);      // even number of players; the pad is decoupled
  const double2* Ab = reinterpret_cast<const double2*>(A + 2 * (long long)b * mat_stride);
  double* ev = evals + (long long)b * nb;
  double2* Ob = reinterpret_cast<double2*>(out + 2 * (long long)b * mat_stride);

  // load A; in mode 1 scaled to unit diagonal
  auto load = [&]() {
    for (int t = tid; t < n * n; t += nt) {
      const int i = t / n, j = t - i * n;
      double2 x = make_double2(0, 0);
      if (i < nb && j < nb) x = Ab[(long long)i * nb + j];
      a[i][j] = x;
    }
    __syncthreads();
    if (mode != 1) return;
    for (int i = tid; i < n; i += nt) {
      const double d = i < nb ? a[i][i].x : 1.0;
      dscale[i] = d > 0.0 ? 1.0 / sqrt(d) : 0.0;
    }
    __syncthreads();
    for (int t = tid; t < n * n; t += nt) {
      const int i = t / n, j = t - i * n;
      const double s = dscale[i] * dscale[j];
      a[i][j].x *= s;
      a[i][j].y *= s;
      if (i == j) a[i][j].y = 0.0;
    }
    __syncthreads();
  };
  load();
  const double frob = frobenius<kNBP>(a, n, red);
  if (mode == 1) {
    if (cholesky<kNBP>(a, v, lam, nb, frob, red, &flag)) {
      // T = D L^-H: column c is the conjugate of row c of L^-1 = diag(d)^-1/2 W
      for (int t = tid; t < nb * nb; t += nt) {
        const int r = t / nb, c = t - r * nb;
        double2 x = make_double2(0, 0);
        if (r <= c) {
          const double s = dscale[r] * sqrt(lam[c]);
          x = make_double2(v[c][r].x * s, -v[c][r].y * s);
        }
        Ob[t] = x;
      }
      if (again && tid == 0) again[b] = 0;
      return;
    }
    __syncthreads();
    load();
  }
  jacobi<kNBP>(a, v, rot, n, mode == 1, frob, &flag);
  rank_eigenvalues<kNBP>(a, n, nb, lam, rank);
  if (mode == 0) {
    for (int i = tid; i < nb; i += nt) ev[rank[i]] = lam[i];
    for (int t = tid; t < nb * nb; t += nt) {
      const int r = t / nb, c = t % nb;   // component r of eigenvector c
      Ob[(long long)r * nb + rank[c]] = v[r][c];
    }
  } else {
    // T[:, k] = D U[:, k] / sqrt(lambda_k) with a floor on tiny lambda
    double lmax = 0.0;
    for (int i = 0; i < nb; ++i) lmax = fmax(lmax, lam[i]);
    const double floor_ = lmax * 1e-15;
    int bad = 0;
    for (int i = tid; i < nb; i += nt) {
      ev[rank[i]] = lam[i];
      if (!(lam[i] > floor_)) bad = 1;
    }
    if (bad && status) atomicOr(status + b, 1);
    // a second orthonormalisation pass is needed only for an ill-conditioned
    // Gram matrix (one SVQB pass leaves an orthogonality error ~ eps kappa(S))
    if (again && tid == 0) {
      double lmin = lmax;
      for (int i = 0; i < nb; ++i) lmin = fmin(lmin, lam[i]);
      again[b] = !(lmin > 1e-4 * lmax);
    }
    for (int t = tid; t < nb * nb; t += nt) {
      const int r = t / nb, c = t % nb;
      const double l = lam[c] > floor_ ? lam[c] : floor_;
      const double s = dscale[r] / sqrt(l);
      Ob[(long long)r * nb + rank[c]] = make_double2(v[r][c].x * s, v[r][c].y * s);
    }
  }
}

// The Rayleigh-Ritz step's small matrices in one launch (nb <= kRRMax): the
// Hermitian part of S^H M S, its eigenvalues (ascending) and T = S Q.  Three
// matrices in LDS bound nb; larger blocks take small_gemm_kernel and heev_kernel.
// Bound by latency: a Jacobi round is a chain of two barriers, two reciprocal square
// roots and the update.  Measured with nb = 40 on the same solve: 233 us, against 528
// (Jacobi) + 3 x 27 us (products) in four launches; nb = 16: 87 against 163 + 3 x 5 us.
constexpr int kRRMax = 48;

__global__ void __launch_bounds__(1024)
rr_kernel(const double* M, const double* S, int nb, long long mat_stride, double* theta,
          double* T, const int* active) {
  __shared__ double2 a[kRRMax][kRRMax + 1];
  __shared__ double2 v[kRRMax][kRRMax + 1];
  __shared__ double2 s[kRRMax][kRRMax + 1];
  __shared__ Rot rot[kRRMax / 2];
  __shared__ double lam[kRRMax];
  __shared__ int rank[kRRMax];
  __shared__ double red[16];
  __shared__ int flag;

  const int b = blockIdx.x;
  if (active && !active[b]) return;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int n = nb + (nb & 1), nn = nb * nb;
  const double2* Mb = reinterpret_cast<const double2*>(M + 2 * (long long)b * mat_stride);
  const double2* Sb = reinterpret_cast<const double2*>(S + 2 * (long long)b * mat_stride);
  double2* Tb = reinterpret_cast<double2*>(T + 2 * (long long)b * mat_stride);
  for (int t = tid; t < nn; t += nt) {
    const int i = t / nb, j = t - i * nb;
    v[i][j] = Mb[t];
    s[i][j] = Sb[t];
  }
  __syncthreads();
  for (int t = tid; t < nn; t += nt) {   // a = M S
    const int i = t / nb, j = t - i * nb;
    double2 c = make_double2(0, 0);
    for (int k = 0; k < nb; ++k) {
      const double2 x = v[i][k], y = s[k][j];
      c.x = fma(x.x, y.x, fma(-x.y, y.y, c.x));
      c.y = fma(x.x, y.y, fma(x.y, y.x, c.y));
    }
    a[i][j] = c;
  }
  __syncthreads();
  for (int t = tid; t < nn; t += nt) {   // v = S^H a
    const int i = t / nb, j = t - i * nb;
    double2 c = make_double2(0, 0);
    for (int k = 0; k < nb; ++k) {
      const double2 x = s[k][i], y = a[k][j];
      c.x = fma(x.x, y.x, fma(x.y, y.y, c.x));
      c.y = fma(x.x, y.y, fma(-x.y, y.x, c.y));
    }
    v[i][j] = c;
  }
  __syncthreads();
  for (int t = tid; t < n * n; t += nt) {   // the Hermitian part (pad: zero)
    const int i = t / n, j = t - i * n;
    double2 c = make_double2(0, 0);
    if (i < nb && j < nb) {
      const double2 x = v[i][j], y = v[j][i];
      c = make_double2(0.5 * (x.x + y.x), i == j ? 0.0 : 0.5 * (x.y - y.y));
    }
    a[i][j] = c;
  }
  __syncthreads();
  const double frob = frobenius<kRRMax>(a, n, red);
  jacobi<kRRMax>(a, v, rot, n, false, frob, &flag);
  rank_eigenvalues<kRRMax>(a, n, nb, lam, rank);
  for (int i = tid; i < nb; i += nt) theta[(long long)b * nb + rank[i]] = lam[i];
  for (int t = tid; t < nn; t += nt) {   // T = S Q, columns in ascending order
    const int i = t / nb, j = t - i * nb;
    double2 c = make_double2(0, 0);
    for (int k = 0; k < nb; ++k) {
      const double2 x = s[i][k], y = v[k][j];
      c.x = fma(x.x, y.x, fma(-x.y, y.y, c.x));
      c.y = fma(x.x, y.y, fma(x.y, y.x, c.y));
    }
    Tb[(long long)i * nb + rank[j]] = c;
  }
}

// ---------------------------------------------------------------------------
// control: residual norms -> convergence; Ritz values -> next filter interval
// ---------------------------------------------------------------------------
// the work table of one member starting at (s32, s64, sall): its first entries and the sums
__device__ __forceinline__ void work_entry(const Control& c, int b, int batch, int nb, int* s32,
                                           int* s64, int* sall) {
  c.work[b] = *s32;
  c.work[batch + 1 + b] = *s64;
  c.work[2 * (batch + 1) + b] = *sall;
  const int nf = nb - c.lock[b];
  *s32 += c.act32[b] ? nf : 0;
  *s64 += c.act64[b] ? nf : 0;
  *sall += c.active[b] ? nb : 0;
}
__device__ __forceinline__ void work_end(const Control& c, int batch, int s32, int s64, int sall) {
  c.work[batch] = s32;
  c.work[batch + 1 + batch] = s64;
  c.work[2 * (batch + 1) + batch] = sall;
}

__device__ void control_member(const Control& c, int b, int nb, int nev, int degree, int kmax,
                               double tol, int mixed, int allow_switch, int allow_lock, int iter);

__global__ void control_kernel(Control c, int nb, int nev, int degree, int kmax, double tol,
                               int mixed, int allow_switch, int allow_lock, int iter) {
  if (threadIdx.x != 0) return;
  control_member(c, blockIdx.x, nb, nev, degree, kmax, tol, mixed, allow_switch, allow_lock, iter);
  if (gridDim.x == 1) {   // a single member: its work table needs no other's counts
    int s32 = 0, s64 = 0, sall = 0;
    work_entry(c, 0, 1, nb, &s32, &s64, &sall);
    work_end(c, 1, s32, s64, sall);
  }
}

__device__ void control_member(const Control& c, int b, int nb, int nev, int degree, int kmax,
                               double tol, int mixed, int allow_switch, int allow_lock, int iter) {
  int* fl = c.flags + 8 * b;
  const int was32 = c.act32[b];
  if (fl[0]) {   // done before this iteration: keep its results
    c.active[b] = 0;
    c.act32[b] = 0;
    c.act64[b] = 0;
    c.lock[b] = 0;
    c.sw[b] = 0;
    return;
  }
  const double* th = c.theta + (long long)b * nb;
  const double* r2 = c.r2 + (long long)b * nb;
  double* bd = c.bounds + 4 * b;
  int nconv = 0;
  double rmax = 0.0;
  for (int j = 0; j < nev; ++j) {
    const double r = sqrt(r2[j]);
    if (r <= tol) ++nconv;
    rmax = fmax(rmax, r);
  }
  const int it = fl[3] + 1;   // outer iterations so far (counted on the device)
  fl[3] = it;
  fl[4] = nconv;
  if (nconv == nev) fl[0] = 1;
  // mixed precision: leave the FP32 filter once it can no longer reduce the
  // residual.  FP32 rounding of the filtered block leaves a residual floor of
  // a few FP32 ulps of the spectral radius (measured: 2-4 eps32 |H|).  Any target:
  // stagnation within 30 eps32 |H| (less than a 30% decrease on two consecutive
  // iterations).  A target below the floor, which FP64 has to reach, does not wait for
  // it:
  //  - at the last iteration's rate q, n(r) = ceil(log(r / tol) / q) more iterations
  //    take a residual r to the target, whichever precision they run in; another FP32
  //    one would end at the floor or at q times the residual, and if no fewer FP64
  //    ones remain from there it is not worth its half of an FP64 one's time;
  //  - within 12 eps32 |H| a decrease of less than 70% is already the floor's doing, and
  //    the rate above no longer the filter's.
  // Against waiting for stagnation, 34 solves: 1.12-1.42 times as fast (mean 1.26; fin 128
  // x 40 x 40 134 -> 111 ms, double dot 256 x 48 x 48 1055 -> 927, eight of 96 x 32 x 32
  // 343 -> 306); the second rule alone 1.15, the first alone 1.24 but nothing where the
  // rate is poor (the last two of these).
  if (mixed && allow_switch && !fl[1] && !fl[0]) {
    const double prev = bd[3];
    const double near_floor = 30.0 * 5.96e-8 * bd[0];
    if (iter == 0 && rmax < near_floor && tol < 3.0 * 5.96e-8 * bd[0]) {
      // a restart that already starts near the floor, with a target below it,
      // gains nothing from FP32 filtering: FP64 from the first iteration
      fl[1] = 1;
      fl[5] = 1;
    } else {
      if (prev > 0.0 && rmax > 0.7 * prev && rmax < near_floor) fl[2] += 1; else fl[2] = 0;
      bool at_floor = false;
      if (prev > 0.0 && rmax < near_floor && tol < 3.0 * 5.96e-8 * bd[0]) {
        at_floor = rmax > 0.3 * prev && rmax < 12.0 * 5.96e-8 * bd[0];
        if (rmax < prev) {
          const double q = log(prev / rmax);
          const double next = fmax(rmax * (rmax / prev), 2.5 * 5.96e-8 * bd[0]);
          at_floor = at_floor || ceil(log(next / tol) / q) >= ceil(log(rmax / tol) / q);
        }
      }
      if (fl[2] >= 2 || at_floor) {
        fl[1] = 1;
        fl[5] = it + 1;
      }
    }
  }
  bd[3] = rmax;
  c.active[b] = fl[0] ? 0 : 1;
  c.act32[b] = (!fl[0] && mixed && !fl[1]) ? 1 : 0;
  c.act64[b] = (!fl[0] && !(mixed && !fl[1])) ? 1 : 0;
  c.sw[b] = (was32 && c.act64[b]) ? 1 : 0;
  // soft locking: the leading run of converged states, whole Kramers pairs,
  // is left out of the next filter (it stays in the block, so orthonormalisation
  // and Rayleigh-Ritz still see it, and it is released if its residual grows)
  int lead = 0;
  while (allow_lock && lead < nev && sqrt(r2[lead]) <= tol) ++lead;
  c.lock[b] = fl[0] ? 0 : (lead & ~1);
  fl[6] = c.lock[b];
  // next filter: damp [a_cut, b_up], scaled to 1 at a0 = lowest Ritz value
  const double bup = bd[0];
  const double a0 = th[0];
  double acut = th[nb - 1], e, cc, sigma1;
  cheb_interval(bup, a0, acut, &e, &cc, &sigma1);
  bd[1] = acut;
  bd[2] = a0;
  double* co = c.coef + (long long)b * kmax * 4;
  if (c.roots) {
    // product form: step k is (H - r_k) / (a0 - r_k), r_k the k-th root (Leja
    // order) mapped onto [a_cut, b_up]; degree = the next filter's m
    for (int k = 0; k < degree && k < kmax; ++k) {
      const double r = cc + e * c.roots[k];
      co[4 * k] = 1.0 / (a0 - r);
      co[4 * k + 1] = r;
      co[4 * k + 2] = 0.0;
    }
    return;
  }
  double sig = sigma1;
  co[0] = sigma1 / e;
  co[1] = cc;
  co[2] = 0.0;
  for (int k = 1; k < degree && k < kmax; ++k) {
    const double sn = 1.0 / (2.0 / sigma1 - sig);
    co[4 * k] = 2.0 * sn / e;
    co[4 * k + 1] = cc;
    co[4 * k + 2] = -sig * sn;
    sig = sn;
  }
}

// prefix sums of the vectors each member still has to process: the stencil
// launches map their live workgroups onto these so that converged members and
// locked vectors leave no XCD idle
__global__ void worktable_kernel(Control c, int batch, int nb) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  int s32 = 0, s64 = 0, sall = 0;
  for (int b = 0; b < batch; ++b) work_entry(c, b, batch, nb, &s32, &s64, &sall);
  work_end(c, batch, s32, s64, sall);
}

// eig[b][j] = theta[b][j], resid[b][j] = sqrt(r2[b][j]) for j < nev
__global__ void finish_kernel(const double* theta, const double* r2, int nb, int nev, int batch,
                              double* eig, double* resid) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= batch * nev) return;
  const int b = t / nev, j = t % nev;
  if (eig) eig[t] = theta[(long long)b * nb + j];
  if (resid) resid[t] = sqrt(r2[(long long)b * nb + j]);
}

__global__ void finite_kernel(const double* x, long long count, int* flag) {
  int bad = 0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (long long)gridDim.x * blockDim.x)
    bad |= !isfinite(x[i]);
  if (bad) atomicOr(flag, 1);
}

__global__ void fill_int_kernel(int* p, int count, int value) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < count) p[t] = value;
}

}  // namespace

hipError_t launch_finish(const double* theta, const double* r2, int nb, int nev, int batch,
                         double* eig, double* resid, hipStream_t s) {
  const int cnt = batch * nev;
  finish_kernel<<<(cnt + 255) / 256, 256, 0, s>>>(theta, r2, nb, nev, batch, eig, resid);
  return hipGetLastError();
}

hipError_t launch_check_finite(const double* x, long long count, int* flag, hipStream_t s) {
  long long g = (count + 255) / 256;
  if (g > 2048) g = 2048;
  if (g < 1) g = 1;
  finite_kernel<<<(unsigned)g, 256, 0, s>>>(x, count, flag);
  return hipGetLastError();
}

hipError_t launch_fill_int(int* p, int count, int value, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  fill_int_kernel<<<(count + 255) / 256, 256, 0, s>>>(p, count, value);
  return hipGetLastError();
}

namespace {

// small complex products of the block step, one workgroup per member, operands
// in LDS: C = op(A) B (op: A, or A^H), or with unit set C = I.  Row-major nb x nb.
constexpr int kGemmThreads = 256;

__global__ void __launch_bounds__(kGemmThreads)
small_gemm_kernel(const double* A, int adj, const double* B, double* C, int nb,
                  long long mat_stride, int herm, const int* active) {
  const int b = blockIdx.x;
  if (active && !active[b]) return;
  __shared__ double2 sa[kNBP * kNBP], sb[kNBP * kNBP];
  const double2* Ab = reinterpret_cast<const double2*>(A + 2 * (long long)b * mat_stride);
  const double2* Bb = reinterpret_cast<const double2*>(B + 2 * (long long)b * mat_stride);
  double2* Cb = reinterpret_cast<double2*>(C + 2 * (long long)b * mat_stride);
  const int nn = nb * nb;
  for (int t = threadIdx.x; t < nn; t += kGemmThreads) {
    sa[t] = Ab[t];
    sb[t] = Bb[t];
  }
  __syncthreads();
  // C[i][j] = sum_k op(A)[i][k] B[k][j]; op(A)[i][k] = A[i][k] or conj(A[k][i])
  auto entry = [&](int i, int j) {
    double re = 0.0, im = 0.0;
    for (int k = 0; k < nb; ++k) {
      const double2 a = adj ? make_double2(sa[k * nb + i].x, -sa[k * nb + i].y) : sa[i * nb + k];
      const double2 v = sb[k * nb + j];
      re = fma(a.x, v.x, fma(-a.y, v.y, re));
      im = fma(a.x, v.y, fma(a.y, v.x, im));
    }
    return make_double2(re, im);
  };
  for (int t = threadIdx.x; t < nn; t += kGemmThreads) {
    const int i = t / nb, j = t - (t / nb) * nb;
    double2 c = entry(i, j);
    if (herm) {   // the Hermitian part (the product is Hermitian up to rounding)
      const double2 d = entry(j, i);
      c = make_double2(0.5 * (c.x + d.x), 0.5 * (c.y - d.y));
      if (i == j) c.y = 0.0;
    }
    Cb[t] = c;
  }
}

__global__ void set_roots_kernel(double* dst, RootTable t, int m) {
  for (int k = threadIdx.x; k < m; k += blockDim.x) dst[k] = t.x[k];
}

__global__ void set_identity_kernel(double* C, int nb, long long mat_stride, const int* active) {
  const int b = blockIdx.x;
  if (active && !active[b]) return;
  double2* Cb = reinterpret_cast<double2*>(C + 2 * (long long)b * mat_stride);
  for (int t = threadIdx.x; t < nb * nb; t += blockDim.x)
    Cb[t] = make_double2(t / nb == t % nb ? 1.0 : 0.0, 0.0);
}

}  // namespace

hipError_t launch_small_gemm(const double* A, int adj, const double* B, double* C, int nb,
                             int batch, long long mat_stride, int herm, const int* active,
                             hipStream_t s) {
  if (nb > HKP_NB_MAX || nb < 1 || C == A || C == B) return hipErrorInvalidValue;
  small_gemm_kernel<<<batch, kGemmThreads, 0, s>>>(A, adj, B, C, nb, mat_stride, herm, active);
  return hipGetLastError();
}

hipError_t launch_set_roots(double* dst, const RootTable& t, int m, hipStream_t s) {
  if (m < 1 || m > kMaxDegree) return hipErrorInvalidValue;
  set_roots_kernel<<<1, 256, 0, s>>>(dst, t, m);
  return hipGetLastError();
}

hipError_t launch_set_identity(double* C, int nb, int batch, long long mat_stride,
                               const int* active, hipStream_t s) {
  set_identity_kernel<<<batch, 256, 0, s>>>(C, nb, mat_stride, active);
  return hipGetLastError();
}

hipError_t launch_heev(double* A, int nb, int batch, long long mat_stride, double* evals,
                       double* out, int mode, int* status, const int* active, hipStream_t s,
                       int* again) {
  if (nb > HKP_NB_MAX || nb < 1) return hipErrorInvalidValue;
  heev_kernel<<<batch, jacobi_threads(nb + (nb & 1)), 0, s>>>(A, nb, mat_stride, evals, out, mode,
                                                              status, active, again);
  return hipGetLastError();
}

bool rr_supported(int nb) { return nb >= 1 && nb <= kRRMax; }

hipError_t launch_rr(const double* M, const double* S, int nb, int batch, long long mat_stride,
                     double* theta, double* T, const int* active, hipStream_t s) {
  if (!rr_supported(nb) || T == M || T == S) return hipErrorInvalidValue;
  rr_kernel<<<batch, jacobi_threads(nb + (nb & 1)), 0, s>>>(M, S, nb, mat_stride, theta, T,
                                                            active);
  return hipGetLastError();
}

hipError_t launch_control(const Control& c, int batch, int nb, int nev, int degree, int kmax,
                          double tol, int mixed, int allow_switch, int allow_lock, int iter,
                          hipStream_t s) {
  control_kernel<<<batch, 64, 0, s>>>(c, nb, nev, degree, kmax, tol, mixed, allow_switch,
                                      allow_lock, iter);
  if (batch > 1) worktable_kernel<<<1, 64, 0, s>>>(c, batch, nb);
  return hipGetLastError();
}

hipError_t launch_worktable(const Control& c, int batch, int nb, hipStream_t s) {
  worktable_kernel<<<1, 64, 0, s>>>(c, batch, nb);
  return hipGetLastError();
}

}  // namespace hkp
