// Extraction of the eigenpairs inside the contour from the moments.
//
// With B0 = [S_{r+s}] and B1 = [S_{r+s+1}] (r, s = 0..K-1, each Kn x KL), the
// Keldysh expansion (eq. (resolvent)) gives B0 = V_K(X, M) W and
// B1 = V_K(X, M) M W with V_K the block matrix of eq. (invpair-split).  If
// B0 = V0 Sigma0 W0^H is its rank-m truncated SVD, V0^H B1 W0 Sigma0^{-1} is
// similar to M (the eigenvalues mu_i = (lambda_i - c)/rho inside); an
// eigenvector s gives V0 s = [x; mu x; ...], whose first block is x.  The pair
// (X, c + rho M) is a minimal invariant pair (Section 2).
//
// Device: Householder QR of B0 (panels of columns held in registers), the
// one-sided Jacobi SVD of the K*L x K*L factor R (up to kJacobiMax columns),
// Q applied to the small singular vectors in its compact WY form, V0^H B1, the
// eigenvectors, and the split-form residual T(lambda) x for the backward error
// of eq. (sressplit) (inf-norms).  Host: the m x m eigenproblem (sequential
// small dense work, as for the projected problems of the paper's solvers,
// Section 5) and the SVD of larger factors.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <numeric>

#include "dense.hpp"
#include "handle.hpp"

namespace nep {

struct ExtractWork {
  DevMem B0, B1, tau, V0, P, smat, X0, Rt, fz, Rp, Ur, sw, wy;
  size_t cap_rows = 0, cap_cols = 0;
};

std::shared_ptr<ExtractWork> make_extract_work() { return std::make_shared<ExtractWork>(); }

// ---------------------------------------------------------------------------
__global__ void k_hankel(const c128* __restrict__ S, int n, int L, int K, long long sstride, c128* __restrict__ B0,
                         c128* __restrict__ B1) {
  const long long M = (long long)K * n, KL = (long long)K * L;
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= M * KL) return;
  const long long col = e / M, row = e - col * M;
  const int r = (int)(row / n), i = (int)(row - (long long)r * n);
  const int s = (int)(col / L), c = (int)(col - (long long)s * L);
  const long long off = (long long)c * n + i;
  B0[e] = S[(long long)(r + s) * sstride + off];
  B1[e] = S[(long long)(r + s + 1) * sstride + off];
}

// R's leading KL x KL block (column-major, leading dimension M) into a
// contiguous KL x KL array, for one plain read-back
__global__ void k_pack_r(const c128* __restrict__ B, long long M, int KL, c128* __restrict__ R) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long long)KL * KL) return;
  const long long j = e / KL, i = e - j * KL;
  R[e] = B[j * M + i];
}

// block sum over 1024 threads
__device__ __forceinline__ c128 block_sum(c128 v, c128* red) {
  for (int o = 32; o >= 1; o >>= 1) {
    v.re += __shfl_xor(v.re, o, 64);
    v.im += __shfl_xor(v.im, o, 64);
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  c128 s = {0.0, 0.0};
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s = s + red[i];
  return s;
}

// Sum of N complex values over the block, each in v[i] (N a power of two, at
// most 16).  Within a wave by halving: each exchange sends the half of the
// values that the other lane keeps, N - 1 exchanges and then one value's, in
// place of 6 N (the exchanges go through the LDS pipe and bound a step
// otherwise).
template <int N>
struct BlockSums {
  c128 wave[16][N], total[N];
};
template <int N>
__device__ __forceinline__ void block_sums(c128 (&v)[N], BlockSums<N>& s) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  auto xchg = [](c128 a, int o) { return c128{__shfl_xor(a.re, o, 64), __shfl_xor(a.im, o, 64)}; };
  int o = 32;
#pragma unroll
  for (int h = N / 2; h >= 1; h >>= 1, o >>= 1) {
    const bool up = (lane & o) != 0;
#pragma unroll
    for (int i = 0; i < h; ++i) {
      const c128 send = csel(up, v[i], v[i + h]), keep = csel(up, v[i + h], v[i]);
      v[i] = keep + xchg(send, o);
    }
  }
#pragma unroll
  for (int q = 32 / N; q >= 1; q >>= 1) v[0] = v[0] + xchg(v[0], q);
  constexpr int LP = 64 / N;  // lanes that hold one value
  __syncthreads();
  if ((lane & (LP - 1)) == 0) s.wave[w][lane / LP] = v[0];
  __syncthreads();
  if (threadIdx.x < N) {
    c128 t = s.wave[0][threadIdx.x];
    for (int k = 1; k < (int)(blockDim.x >> 6); ++k) t = t + s.wave[k][threadIdx.x];
    s.total[threadIdx.x] = t;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = s.total[i];
}

// One step of the QR, a panel of W columns: the reflectors H_j = I - tau_j v_j
// v_j^H of the panel at column k (zlarfg convention: H^H x = beta e_1, v_0 = 1,
// beta real; v overwrites x below the diagonal) are applied to the columns
// right of it, and the next panel, whose columns belong to the first group, is
// factored by that group.  Columns are held in registers, RPT rows a thread,
// so a column is read and written once per panel.  (first: the panel at k is
// factored, nothing is applied.)  The chain of block sums bounds a step.
template <int NT, int RPT, int W>
__global__ __launch_bounds__(NT) void k_house_panel(c128* __restrict__ B, long long M, int k, int ncol,
                                                    c128* __restrict__ tau, int first) {
  __shared__ BlockSums<W> red;
  __shared__ BlockSums<1> red1;
  __shared__ c128 top[W];  // row j of the panel's columns
  const int tid = threadIdx.x;
  const int k1 = first ? k : min(k + W, ncol);  // first column of the next panel
  const bool lead = blockIdx.x == 0;
  const int c0 = lead ? k1 : k1 + W + (int)blockIdx.x - 1;
  const int nc = lead ? min(W, ncol - k1) : 1;
  if (c0 >= ncol) return;
  c128 b[W][RPT];
#pragma unroll
  for (int c = 0; c < W; ++c)
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const long long r = tid + (long long)NT * i;
      b[c][i] = (c < nc && r < M) ? B[(long long)(c0 + c) * M + r] : c128{0.0, 0.0};
    }
  if (!first) {
    for (int j = k; j < k1; ++j) {
      const c128* v = B + (long long)j * M;
      c128 vr[RPT], w[W];
#pragma unroll
      for (int c = 0; c < W; ++c) w[c] = c128{0.0, 0.0};
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const long long r = tid + (long long)NT * i;
        vr[i] = r == j ? c128{1.0, 0.0} : (r > j && r < M) ? v[r] : c128{0.0, 0.0};
        w[0] = cmac(w[0], conj(vr[i]), b[0][i]);
        if (lead)
#pragma unroll
          for (int c = 1; c < W; ++c) w[c] = cmac(w[c], conj(vr[i]), b[c][i]);
      }
      if (lead) {
        block_sums<W>(w, red);
      } else {
        c128 w1[1] = {w[0]};
        block_sums<1>(w1, red1);
        w[0] = w1[0];
      }
      const c128 tc = conj(tau[j]);
#pragma unroll
      for (int c = 0; c < W; ++c) {
        if (lead || c == 0) {
          const c128 f = tc * w[c];
#pragma unroll
          for (int i = 0; i < RPT; ++i) b[c][i] = fms(b[c][i], vr[i], f);
        }
      }
    }
  }
  if (lead) {
#pragma unroll
    for (int j = 0; j < W; ++j) {
      if (j < nc) {  // uniform
      const int row = c0 + j;
      // |x below the diagonal|^2 of column j, and its products with the later ones
      c128 w[W];
#pragma unroll
      for (int c = 0; c < W; ++c) w[c] = c128{0.0, 0.0};
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const long long r = tid + (long long)NT * i;
        const c128 xb = csel(r > row, b[j][i], c128{0.0, 0.0});
#pragma unroll
        for (int c = j; c < W; ++c) w[c] = cmac(w[c], conj(xb), b[c][i]);
        if (r == row) {
#pragma unroll
          for (int c = j; c < W; ++c) top[c] = b[c][i];
        }
      }
      block_sums<W>(w, red);  // (its barriers also publish top)
      const double sigma2 = w[j].re;
      const c128 alpha = top[j];
      c128 t = {0.0, 0.0}, scal = {0.0, 0.0};
      double beta = alpha.re;
      const bool zero = sigma2 == 0.0 && alpha.im == 0.0;
      if (!zero) {
        const double nrm = sqrt(norm2(alpha) + sigma2);
        beta = alpha.re >= 0.0 ? -nrm : nrm;
        t = c128{(beta - alpha.re) / beta, -alpha.im / beta};
        scal = cdiv(c128{1.0, 0.0}, c128{alpha.re - beta, alpha.im});
      }
      if (tid == 0) tau[row] = t;
      // v^H b_c = b_c[row] + conj(scal) (x below)^H b_c
      c128 f[W];
#pragma unroll
      for (int c = j + 1; c < W; ++c) f[c] = conj(t) * cmac(top[c], conj(scal), w[c]);
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const long long r = tid + (long long)NT * i;
        const c128 vi = r == row ? c128{1.0, 0.0} : csel(r > row, b[j][i] * scal, c128{0.0, 0.0});
#pragma unroll
        for (int c = j + 1; c < W; ++c) b[c][i] = fms(b[c][i], vi, f[c]);
        if (!zero && r >= row) b[j][i] = r == row ? c128{beta, 0.0} : vi;
      }
      __syncthreads();  // top and red are free
      }
    }
  }
#pragma unroll
  for (int c = 0; c < W; ++c)
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const long long r = tid + (long long)NT * i;
      if (c < nc && r < M) B[(long long)(c0 + c) * M + r] = b[c][i];
    }
}

// Householder vector of column k, by one group (blocks of more rows than the
// panels hold).
__device__ void house_vec(c128* __restrict__ B, long long M, int k, c128* __restrict__ tau, c128* red) {
  c128* x = B + (long long)k * M;
  double ss = 0.0;
  for (long long i = k + 1 + threadIdx.x; i < M; i += blockDim.x) ss += norm2(x[i]);
  const c128 tot = block_sum(c128{ss, 0.0}, red);
  const double sigma2 = tot.re;
  const c128 alpha = x[k];
  __syncthreads();
  if (sigma2 == 0.0 && alpha.im == 0.0) {
    if (threadIdx.x == 0) tau[k] = c128{0.0, 0.0};
    return;
  }
  const double nrm = sqrt(norm2(alpha) + sigma2);
  const double beta = alpha.re >= 0.0 ? -nrm : nrm;
  const c128 t = {(beta - alpha.re) / beta, -alpha.im / beta};
  const c128 scal = cdiv(c128{1.0, 0.0}, c128{alpha.re - beta, alpha.im});
  for (long long i = k + 1 + threadIdx.x; i < M; i += blockDim.x) x[i] = x[i] * scal;
  if (threadIdx.x == 0) {
    tau[k] = t;
    x[k] = c128{beta, 0.0};
  }
}

__global__ __launch_bounds__(1024) void k_house_vec(c128* __restrict__ B, long long M, int k, c128* __restrict__ tau) {
  __shared__ c128 red[16];
  house_vec(B, M, k, tau, red);
}

// b <- H^H b = b - conj(tau) v (v^H b) for columns k+1.. (one group each).
// The group of column k+1 then forms that column's Householder vector (the
// next step's), so a step is one launch: only this group writes column k+1.
__global__ __launch_bounds__(1024) void k_house_apply(c128* __restrict__ B, long long M, int k, int ncol,
                                                      c128* __restrict__ tau) {
  __shared__ c128 red[16];
  const int col = k + 1 + blockIdx.x;
  if (col >= ncol) return;
  const c128* v = B + (long long)k * M;
  c128* b = B + (long long)col * M;
  c128 acc = {0.0, 0.0};
  if (threadIdx.x == 0) acc = b[k];  // v_k = 1
  for (long long i = k + 1 + threadIdx.x; i < M; i += blockDim.x) acc = acc + conj(v[i]) * b[i];
  const c128 w = block_sum(acc, red);
  const c128 f = conj(tau[k]) * w;
  if (threadIdx.x == 0) b[k] = b[k] - f;
  for (long long i = k + 1 + threadIdx.x; i < M; i += blockDim.x) b[i] = b[i] - v[i] * f;
  if (blockIdx.x == 0) {
    __syncthreads();  // the group's updates of column k+1 are visible to all its threads
    house_vec(B, M, col, tau, red);
  }
}

template <int NT, int RPT, int W>
static hipError_t house_panels(c128* B, long long M, int ncol, c128* tau, hipStream_t st) {
  hipLaunchKernelGGL((k_house_panel<NT, RPT, W>), dim3(1), dim3(NT), 0, st, B, M, 0, ncol, tau, 1);
  for (int k = 0; k + W < ncol; k += W)
    hipLaunchKernelGGL((k_house_panel<NT, RPT, W>), dim3(1 + std::max(0, ncol - k - 2 * W)), dim3(NT), 0, st, B, M, k,
                       ncol, tau, 0);
  return hipGetLastError();
}

// QR of B (M x ncol): panels as wide as the registers allow for M rows (400
// rows, 16 columns: 150 us in 16 launches -> 55 us in two); one column per
// launch beyond 4096 rows, where panels of two columns took as long (6148
// rows, 64 columns: 0.75 ms either way).
static hipError_t house_qr(c128* B, long long M, int ncol, c128* tau, hipStream_t st) {
  if (M <= 512) return house_panels<512, 1, 8>(B, M, ncol, tau, st);
  if (M <= 1024) return house_panels<512, 2, 4>(B, M, ncol, tau, st);
  if (M <= 2048) return house_panels<512, 4, 4>(B, M, ncol, tau, st);
  if (M <= 4096) return house_panels<1024, 4, 4>(B, M, ncol, tau, st);
  hipLaunchKernelGGL(k_house_vec, dim3(1), dim3(1024), 0, st, B, M, 0, tau);
  for (int k = 0; k + 1 < ncol; ++k)
    hipLaunchKernelGGL(k_house_apply, dim3(ncol - k - 1), dim3(1024), 0, st, B, M, k, ncol, tau);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// One-sided (Hestenes) Jacobi SVD of the upper triangle R (k x k, k <=
// kJacobiMax, columns M apart in B), by one group in LDS: the column pairs of
// a round are disjoint (a round-robin tournament), kJacobiLanes lanes each,
// and a sweep is k - 1 rounds; it ends when a sweep rotates nothing (the same
// test as the host's, pair by pair).  The rotations act on the columns of R^H,
// which for these graded factors takes half the sweeps of R's own columns (10
// against 20 on a 64-column one).  R^H = W diag(s) U^H, s descending: W are the
// scaled columns and U the accumulated rotations.  Out: U (k x k) and, in one
// block for one copy to the host, s and W.  The host's sequential sweeps took
// 4.65 ms at k = 64 and 0.18 ms at k = 16; this kernel 1.16 ms and 0.09 ms,
// bound by the rounds' LDS traffic (256 KB each) and their chain of square
// roots.
// ---------------------------------------------------------------------------
constexpr int kJacobiMax = 64;

// 1/sqrt(x) to working precision: the hardware's estimate and two Newton steps
__device__ __forceinline__ double rsqrt2(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = y * (1.5 - 0.5 * x * y * y);
  return y * (1.5 - 0.5 * x * y * y);
}

constexpr int kJacobiLanes = 16;                             // lanes per pair
constexpr int kJacobiThreads = kJacobiLanes * kJacobiMax / 2;

__global__ __launch_bounds__(kJacobiThreads) void k_jacobi(const c128* __restrict__ Bm, long long M, int k,
                                                           c128* __restrict__ U, double* __restrict__ sout,
                                                           c128* __restrict__ Wout) {
  constexpr int RP = kJacobiMax / kJacobiLanes;  // rows per lane
  __shared__ c128 A[kJacobiMax][kJacobiMax + 1], W[kJacobiMax][kJacobiMax + 1];  // [column][row], zero past k
  __shared__ double sv[kJacobiMax], mx[kJacobiThreads / 64];
  __shared__ int rotated[2];
  const int tid = threadIdx.x, pair = tid / kJacobiLanes, l = tid % kJacobiLanes;
  // R scaled by a power of two to about 1, so that squares neither overflow nor vanish
  double big = 0.0;
  for (int e = tid; e < kJacobiMax * kJacobiMax; e += kJacobiThreads) {
    const int j = e / kJacobiMax, i = e % kJacobiMax;
    const c128 x = (j < k && i <= j) ? Bm[(long long)j * M + i] : c128{0.0, 0.0};
    A[i][j] = conj(x);  // column i of R^H
    W[j][i] = c128{i == j ? 1.0 : 0.0, 0.0};
    big = nanmax(big, fmax(fabs(x.re), fabs(x.im)));
  }
  for (int o = 32; o >= 1; o >>= 1) big = nanmax(big, __shfl_xor(big, o, 64));
  if ((tid & 63) == 0) mx[tid >> 6] = big;
  if (tid < 2) rotated[tid] = 0;
  __syncthreads();
  for (int w = 0; w < kJacobiThreads / 64; ++w) big = nanmax(big, mx[w]);
  const int ex = (big > 0.0 && isfinite(big)) ? ilogb(big) : 0;
  for (int e = tid; e < kJacobiMax * kJacobiMax; e += kJacobiThreads) {
    c128& x = A[e / kJacobiMax][e % kJacobiMax];
    x = c128{ldexp(x.re, -ex), ldexp(x.im, -ex)};
  }
  __syncthreads();
  const double eps = 1e-15;
  const int k2 = (k + 1) & ~1, rounds = k2 - 1;
  const int nr = (k + kJacobiLanes - 1) / kJacobiLanes;  // rows of this lane that exist in some column
  for (int sweep = 0; sweep < 60; ++sweep) {
    for (int r = 0; r < rounds; ++r) {
      int p = pair == 0 ? k2 - 1 : (r + pair) % rounds;
      int q = pair == 0 ? r : (r - pair + rounds) % rounds;
      if (p > q) {
        const int t = p;
        p = q;
        q = t;
      }
      if (2 * pair < k2 && q < k) {  // uniform over the pair's lanes
        c128 x[RP], y[RP];
        double al = 0.0, be = 0.0, gr = 0.0, gi = 0.0;
#pragma unroll
        for (int i = 0; i < RP; ++i)
          if (i < nr) {
            x[i] = A[p][l + kJacobiLanes * i];
            y[i] = A[q][l + kJacobiLanes * i];
            al += norm2(x[i]);
            be += norm2(y[i]);
            gr += x[i].re * y[i].re + x[i].im * y[i].im;
            gi += x[i].re * y[i].im - x[i].im * y[i].re;
          }
#pragma unroll
        for (int o = kJacobiLanes / 2; o >= 1; o >>= 1) {
          al += __shfl_xor(al, o, 64);
          be += __shfl_xor(be, o, 64);
          gr += __shfl_xor(gr, o, 64);
          gi += __shfl_xor(gi, o, 64);
        }
        const double g2 = gr * gr + gi * gi;
        if (!(g2 == 0.0 || g2 <= eps * eps * (al * be))) {
          if (l == 0) rotated[sweep & 1] = 1;
          const double ig = rsqrt2(g2);
          const c128 dc = {gr * ig, -gi * ig};  // conjugate phase of gamma
          // (an error of t leaves some of gamma to the next sweep; c and s, whose
          // squares must add up to 1, are to working precision)
          const double z = 0.5 * (be - al) * ig, az = fabs(z);
          const double h = 1.0 + z * z;
          double t = az < 1e8 ? 1.0 / (az + h * rsqrt2(h)) : 0.5 / az;
          t = z >= 0.0 ? t : -t;
          const double c = rsqrt2(1.0 + t * t), sn = c * t;
#pragma unroll
          for (int i = 0; i < RP; ++i)
            if (i < nr) {
              const int row = l + kJacobiLanes * i;
              const c128 v = y[i] * dc;
              A[p][row] = c128{c * x[i].re - sn * v.re, c * x[i].im - sn * v.im};
              A[q][row] = c128{sn * x[i].re + c * v.re, sn * x[i].im + c * v.im};
              const c128 u = W[p][row], wv = W[q][row] * dc;
              W[p][row] = c128{c * u.re - sn * wv.re, c * u.im - sn * wv.im};
              W[q][row] = c128{sn * u.re + c * wv.re, sn * u.im + c * wv.im};
            }
        }
      }
      __syncthreads();
    }
    const bool more = rotated[sweep & 1] != 0;
    if (tid == 0) rotated[(sweep + 1) & 1] = 0;
    __syncthreads();
    if (!more) break;  // uniform
  }
  for (int j = pair; j < k; j += kJacobiMax / 2) {
    double s2 = 0.0;
    for (int i = l; i < k; i += kJacobiLanes) s2 += norm2(A[j][i]);
#pragma unroll
    for (int o = kJacobiLanes / 2; o >= 1; o >>= 1) s2 += __shfl_xor(s2, o, 64);
    if (l == 0) sv[j] = sqrt(s2);
  }
  __syncthreads();
  for (int j = pair; j < k; j += kJacobiMax / 2) {
    const double s = sv[j];
    // descending, ties in column order; by their bits, so that a NaN (first) leaves a permutation too
    auto key = [](double x) { return (unsigned long long)__double_as_longlong(x) & ~(1ull << 63); };
    int pos = 0;
    for (int i = 0; i < k; ++i) pos += (key(sv[i]) > key(s) || (key(sv[i]) == key(s) && i < j)) ? 1 : 0;
    if (l == 0) sout[pos] = ldexp(s, ex);
    for (int i = l; i < k; i += kJacobiLanes) {
      Wout[(long long)pos * k + i] = s > 0.0 ? c128{A[j][i].re / s, A[j][i].im / s} : c128{0.0, 0.0};
      U[(long long)pos * k + i] = W[j][i];
    }
  }
}

// ---------------------------------------------------------------------------
// V0 = Q [U; 0] with Q = H_0 .. H_{r-1} = I - V T V^H, T^{-1} = diag(1/tau) +
// the strict upper triangle of V^H V: the Gram matrix, a back substitution per
// column, and one product, instead of r reflectors in turn (6148 rows, 64
// reflectors and 17 columns: 395 -> 85 us).
// ---------------------------------------------------------------------------
// G[a][b] = v_a^H v_b, a < b: one group per 4 x 4 block of columns
__global__ __launch_bounds__(256) void k_wy_gram(const c128* __restrict__ B, long long M, int r,
                                                 c128* __restrict__ G) {
  __shared__ BlockSums<16> red;
  int t = blockIdx.x, ta = 0, nt = (r + 3) / 4;
  while (t >= nt - ta) t -= nt - ta++;  // block row ta, block column ta + t
  const int a0 = 4 * ta, b0 = 4 * (ta + t);
  c128 acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = c128{0.0, 0.0};
  for (long long x = b0 + threadIdx.x; x < M; x += 256) {
    c128 va[4], vb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int a = a0 + i, b = b0 + i;
      va[i] = (a >= r || x < a) ? c128{0.0, 0.0} : x == a ? c128{1.0, 0.0} : B[(long long)a * M + x];
      vb[i] = (b >= r || x < b) ? c128{0.0, 0.0} : x == b ? c128{1.0, 0.0} : B[(long long)b * M + x];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[4 * i + j] = cmac(acc[4 * i + j], conj(va[i]), vb[j]);
  }
  block_sums<16>(acc, red);
  if (threadIdx.x < 16) {
    const int a = a0 + threadIdx.x / 4, b = b0 + (threadIdx.x & 3);
    c128 v = acc[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) v = csel((int)threadIdx.x == i, acc[i], v);
    if (a < b && b < r) G[(long long)b * r + a] = v;
  }
}

// X = T V_1^H U (r x m), V_1 the top r rows of V: one group per column, 256
// rows of the back substitution at a time, a row per thread (blocks of K*L <=
// 256 columns are one such block; probe pools reach 4096).
constexpr int kWyRows = 256;

__global__ __launch_bounds__(kWyRows) void k_wy_coef(const c128* __restrict__ B, long long M, int r,
                                                     const c128* __restrict__ tau, const c128* __restrict__ G,
                                                     const c128* __restrict__ U, c128* __restrict__ X) {
  __shared__ c128 xk;
  const int j = blockIdx.x;
  for (int b0 = (r - 1) / kWyRows * kWyRows; b0 >= 0; b0 -= kWyRows) {
    const int i = b0 + threadIdx.x, top = min(r, b0 + kWyRows);
    c128 c = {0.0, 0.0};
    if (i < top) {
      c = U[(long long)j * r + i];
      for (int l = i + 1; l < r; ++l) c = cmac(c, conj(B[(long long)i * M + l]), U[(long long)j * r + l]);
      for (int k = r - 1; k >= top; --k) c = fms(c, G[(long long)k * r + i], X[(long long)j * r + k]);
    }
    for (int k = top - 1; k >= b0; --k) {
      if (i == k) {
        xk = tau[k] * c;
        X[(long long)j * r + k] = xk;
      }
      __syncthreads();
      if (i < k) c = fms(c, G[(long long)k * r + i], xk);
      __syncthreads();  // (also makes the block's X visible to the next one)
    }
  }
}

// V0 = [U; 0] - V X: a thread per row, 8 columns per group, X staged kWyRows
// rows at a time.
__global__ __launch_bounds__(256) void k_wy_apply(const c128* __restrict__ B, long long M, int r, int m,
                                                  const c128* __restrict__ U, const c128* __restrict__ X,
                                                  c128* __restrict__ V0) {
  constexpr int CB = 8;
  __shared__ c128 Xs[kWyRows][CB];
  const int j0 = blockIdx.y * CB;
  const long long row = (long long)blockIdx.x * 256 + threadIdx.x;
  c128 acc[CB];
#pragma unroll
  for (int j = 0; j < CB; ++j)
    acc[j] = (row < r && j0 + j < m) ? U[(long long)(j0 + j) * r + row] : c128{0.0, 0.0};
  for (int k0 = 0; k0 < r; k0 += kWyRows) {
    const int kn = min(kWyRows, r - k0);
    if (k0 > 0) __syncthreads();  // the staged rows are read
    for (int e = threadIdx.x; e < kn * CB; e += 256) {
      const int k = e / CB, j = e & (CB - 1);
      Xs[k][j] = j0 + j < m ? X[(long long)(j0 + j) * r + k0 + k] : c128{0.0, 0.0};
    }
    __syncthreads();
    const int ke = row < M ? (int)min((long long)kn, row - k0 + 1) : 0;
#pragma unroll 4
    for (int k = 0; k < ke; ++k) {
      const c128 v = row == k0 + k ? c128{1.0, 0.0} : B[(long long)(k0 + k) * M + row];
#pragma unroll
      for (int j = 0; j < CB; ++j) acc[j] = fms(acc[j], v, Xs[k][j]);
    }
  }
  if (row >= M) return;
#pragma unroll
  for (int j = 0; j < CB; ++j)
    if (j0 + j < m) V0[(long long)(j0 + j) * M + row] = acc[j];
}

// P[i + j*m] = sum_r conj(V0[r, i]) B1[r, j]; one group per (i, j)
__global__ __launch_bounds__(256) void k_vhb(const c128* __restrict__ V0, const c128* __restrict__ B1, long long M,
                                             int m, c128* __restrict__ P) {
  __shared__ c128 red[16];
  const int i = blockIdx.x % m, j = blockIdx.x / m;
  const c128* a = V0 + (long long)i * M;
  const c128* b = B1 + (long long)j * M;
  c128 acc = {0.0, 0.0};
  for (long long r = threadIdx.x; r < M; r += blockDim.x) acc = acc + conj(a[r]) * b[r];
  const c128 s = block_sum(acc, red);
  if (threadIdx.x == 0) P[(long long)j * m + i] = s;
}

// X[:, q] = V0[0:n, :] s[:, q], normalized (2-norm 1, largest entry real > 0)
__global__ __launch_bounds__(256) void k_eigvec(const c128* __restrict__ V0, long long M, int n, int m,
                                                const c128* __restrict__ smat, c128* __restrict__ X) {
  __shared__ c128 red[16];
  __shared__ double rmax[4];
  __shared__ int ridx[4];
  const int q = blockIdx.x;
  c128* x = X + (long long)q * n;
  double ss = 0.0;
  double bm = -1.0;
  int bi = 0x7fffffff;
  for (int r = threadIdx.x; r < n; r += blockDim.x) {
    c128 acc = {0.0, 0.0};
    for (int j = 0; j < m; ++j) acc = acc + V0[(long long)j * M + r] * smat[(long long)q * m + j];
    x[r] = acc;
    const double a2 = norm2(acc);
    ss += a2;
    if (a2 > bm) { bm = a2; bi = r; }
  }
  const c128 tot = block_sum(c128{ss, 0.0}, red);
  for (int o = 32; o >= 1; o >>= 1) {
    const double ov = __shfl_xor(bm, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (ov > bm || (ov == bm && oi < bi)) { bm = ov; bi = oi; }
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) { rmax[w] = bm; ridx[w] = bi; }
  __syncthreads();
  bm = rmax[0];
  bi = ridx[0];
  for (int i = 1; i < 4; ++i)
    if (rmax[i] > bm || (rmax[i] == bm && ridx[i] < bi)) { bm = rmax[i]; bi = ridx[i]; }
  const double nrm = sqrt(tot.re);
  const c128 piv = x[bi];
  const double ap = sqrt(norm2(piv));
  // scale = conj(piv)/|piv| / nrm
  const c128 scale = (ap > 0.0 && nrm > 0.0) ? c128{piv.re / (ap * nrm), -piv.im / (ap * nrm)} : c128{0.0, 0.0};
  __syncthreads();
  for (int r = threadIdx.x; r < n; r += blockDim.x) x[r] = x[r] * scale;
}

// Rt[row, q] = sum_i coef[i*m + q] (A_i x_q)[row]  (split-form T(lambda_q) x_q)
// A and x tiles staged through LDS, the next tile's loads in flight while one
// is used; a diagonal or banded term runs over its rows' band only (kind[i]:
// bit 0 complex, the rest the half-width plus one, 0 for a dense term).  n =
// 1537 with two banded and two dense terms and 17 pairs: 391 -> 174 us; n =
// 200 with tridiagonal terms: 40 -> 9 us.
__global__ __launch_bounds__(512) void k_split_apply(int n, int ell, int m, const double* const* __restrict__ A,
                                                     const int* __restrict__ kind, const c128* __restrict__ coef,
                                                     const c128* __restrict__ X, c128* __restrict__ Rt) {
  // one group per 16 rows x 32 pairs, one output per thread: every A_i row
  // is read by one group only, and n/16 groups keep the CUs busy; each
  // output sums over k in ascending order
  constexpr int RB = 16, QB = 32, KC = 64;
  constexpr int AU = RB * KC / 512, XU = KC * QB / 512;
  __shared__ c128 As[RB][KC + 1];
  __shared__ c128 Xs[KC][QB + 1];
  const int row0 = blockIdx.x * RB, q0 = blockIdx.y * QB;
  const int tr = threadIdx.x >> 5, tq = threadIdx.x & 31;
  const int gq = q0 + tq;
  c128 out = {0.0, 0.0};
  for (int i = 0; i < ell; ++i) {
    const int cplx = kind[i] & 1, w = (kind[i] >> 1) - 1;
    const int kbeg = w >= 0 ? max(0, row0 - w) : 0, kend = w >= 0 ? min(n, row0 + RB + w) : n;
    c128 acc = {0.0, 0.0}, ra[AU], rx[XU];
    auto load = [&](int s0) {
#pragma unroll
      for (int u = 0; u < AU; ++u) {
        const int e = threadIdx.x + 512 * u, gr = row0 + e / KC, gs = s0 + (e & (KC - 1));
        c128 a = {0.0, 0.0};
        if (gr < n && gs < kend) {
          if (cplx) a = reinterpret_cast<const c128*>(A[i])[(long long)gr * n + gs];
          else a.re = A[i][(long long)gr * n + gs];
        }
        ra[u] = a;
      }
#pragma unroll
      for (int u = 0; u < XU; ++u) {
        const int e = threadIdx.x + 512 * u, xq = q0 + e / KC, gs = s0 + (e & (KC - 1));
        rx[u] = (gs < kend && xq < m) ? X[(long long)xq * n + gs] : c128{0.0, 0.0};
      }
    };
    load(kbeg);
    for (int s0 = kbeg; s0 < kend; s0 += KC) {
#pragma unroll
      for (int u = 0; u < AU; ++u) {
        const int e = threadIdx.x + 512 * u;
        As[e / KC][e & (KC - 1)] = ra[u];
      }
#pragma unroll
      for (int u = 0; u < XU; ++u) {
        const int e = threadIdx.x + 512 * u;
        Xs[e & (KC - 1)][e / KC] = rx[u];
      }
      __syncthreads();
      if (s0 + KC < kend) load(s0 + KC);
      const int ke = min(KC, kend - s0);
      if (ke == KC) {
#pragma unroll 8
        for (int k = 0; k < KC; ++k) acc = acc + As[tr][k] * Xs[k][tq];
      } else {
        for (int k = 0; k < ke; ++k) acc = acc + As[tr][k] * Xs[k][tq];
      }
      __syncthreads();
    }
    if (gq < m) out = out + coef[(long long)i * m + gq] * acc;
  }
  const int gr = row0 + tr;
  if (gr < n && gq < m) Rt[(long long)gq * n + gr] = out;
}

// per column: max |Rt|, max |X|
__global__ void k_colmax2(const c128* __restrict__ Rt, const c128* __restrict__ X, int n, double* __restrict__ out) {
  __shared__ double r1[256], r2[256];
  const int q = blockIdx.x;
  double a = 0.0, b = 0.0;
  for (int r = threadIdx.x; r < n; r += blockDim.x) {
    a = nanmax(a, sqrt(norm2(Rt[(long long)q * n + r])));
    b = nanmax(b, sqrt(norm2(X[(long long)q * n + r])));
  }
  r1[threadIdx.x] = a;
  r2[threadIdx.x] = b;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      r1[threadIdx.x] = nanmax(r1[threadIdx.x], r1[threadIdx.x + s]);
      r2[threadIdx.x] = nanmax(r2[threadIdx.x], r2[threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[2 * q] = r1[0];
    out[2 * q + 1] = r2[0];
  }
}

// ---------------------------------------------------------------------------
static nep_status grow(DevMem& m, size_t bytes) {
  if (m.bytes >= bytes) return NEP_OK;
  return m.alloc(bytes);
}

// eta for m pairs: X device (n x m column-major), lambda host.
hipError_t fn_points(const FnNode* nodes, const c128* coef, const int* roots, int ell, const c128* z, int m,
                     c128* out, int* bad, hipStream_t st);

// Device buffers of one backward-error evaluation of m pairs: what the host
// sends, then what it reads back, each in one block.
struct EtaBuffers {
  char* in;           // kMaxTerms term pointers, kMaxTerms term kinds, m points
  char* out;          // f_i(lambda_q) at [i*m + q], 2m column maxima, m flags (lambda_q on a pole or cut)
  c128* Rt;           // n x m residuals T(lambda_q) x_q
};
constexpr size_t kEtaTerms = (sizeof(void*) + sizeof(int)) * kMaxTerms;
static size_t eta_in_bytes(int m) { return kEtaTerms + sizeof(c128) * m; }
static size_t eta_out_bytes(int m, int ell) {
  return sizeof(c128) * (size_t)m * ell + sizeof(double) * 2 * m + sizeof(int) * m;
}
static size_t up256(size_t b) { return (b + 255) / 256 * 256; }
static size_t eta_small_bytes(int m, int ell) { return up256(eta_in_bytes(m)) + up256(eta_out_bytes(m, ell)); }
static EtaBuffers eta_carve(char* small, c128* Rt, int m) { return EtaBuffers{small, small + up256(eta_in_bytes(m)), Rt}; }

// eta of eq. (sressplit) with infinity norms for m pairs: lam host (m
// complex), X device (n x m column-major).  The device computes f_i(lambda_q),
// the split-form residuals T(lambda_q) x_q and the column maxima into b; the
// host reads them back and forms
// eta_q = max|T x| / (sum_i |f_i| ||A_i||_inf max|x|).
// host: room for the larger of b's two blocks.
static nep_status eta_run(Split& h, int m, const c128* lam, const c128* X, const EtaBuffers& b, char* host, double* eta,
                          hipStream_t st) {
  const int n = h.op.n, ell = h.op.ell;
  {
    const double** hA = reinterpret_cast<const double**>(host);
    int* kind = reinterpret_cast<int*>(host + sizeof(void*) * kMaxTerms);
    for (int i = 0; i < ell; ++i) {
      hA[i] = reinterpret_cast<const double*>(h.op.dA[i]);
      const int w = h.op.is_diag[i] ? 0 : h.op.band_w[i] > 0 ? h.op.band_w[i] : -1;  // -1: dense
      kind[i] = (h.op.is_cplx[i] ? 1 : 0) | ((w + 1) << 1);
    }
    std::memcpy(host + kEtaTerms, lam, sizeof(c128) * m);
  }
  NEP_HIP(hipMemcpyAsync(b.in, host, eta_in_bytes(m), hipMemcpyHostToDevice, st));
  const double* const* dA = reinterpret_cast<const double* const*>(b.in);
  const int* dkind = reinterpret_cast<const int*>(b.in + sizeof(void*) * kMaxTerms);
  const c128* z = reinterpret_cast<const c128*>(b.in + kEtaTerms);
  c128* fv = reinterpret_cast<c128*>(b.out);
  double* norms = reinterpret_cast<double*>(fv + (size_t)m * ell);
  int* bad = reinterpret_cast<int*>(norms + 2 * m);
  NEP_HIP(fn_points(h.op.dfn_nodes, h.op.dfn_coef, h.fn_roots.as<int>(), ell, z, m, fv, bad, st));
  dim3 grid(ceil_div(n, 16), ceil_div(m, 32));
  hipLaunchKernelGGL(k_split_apply, grid, dim3(512), 0, st, n, ell, m, dA, dkind, fv, X, b.Rt);
  NEP_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_colmax2, dim3(m), dim3(256), 0, st, b.Rt, X, n, norms);
  NEP_HIP(hipGetLastError());
  NEP_HIP(hipMemcpyAsync(host, b.out, eta_out_bytes(m, ell), hipMemcpyDeviceToHost, st));
  NEP_HIP(hipStreamSynchronize(st));
  const c128* fv_h = reinterpret_cast<const c128*>(host);
  const double* hn_h = reinterpret_cast<const double*>(fv_h + (size_t)m * ell);
  const int* bad_h = reinterpret_cast<const int*>(hn_h + 2 * m);
  for (int q = 0; q < m; ++q) {
    if (bad_h[q]) {
      eta[q] = NAN;
      continue;
    }
    double den = 0.0;
    for (int i = 0; i < ell; ++i) {
      const c128 f = fv_h[(size_t)i * m + q];
      den += std::sqrt(f.re * f.re + f.im * f.im) * h.op.normA[i];
    }
    den *= hn_h[2 * q + 1];
    eta[q] = den > 0.0 ? hn_h[2 * q] / den : NAN;
  }
  return NEP_OK;
}

static nep_status backward_errors(Split& h, int m, const std::vector<zc>& lam, const c128* X, std::vector<double>& eta,
                                  ExtractWork& w, hipStream_t st) {
  const int n = h.op.n, ell = h.op.ell;
  // the workspace grows and never shrinks: no device allocation or free once
  // it is large enough
  NEP_TRY(grow(w.fz, eta_small_bytes(m, ell)));
  NEP_TRY(grow(w.Rt, sizeof(c128) * (size_t)n * m));
  const EtaBuffers b = eta_carve(w.fz.as<char>(), w.Rt.as<c128>(), m);
  std::vector<char> host(eta_small_bytes(m, ell));
  eta.assign(m, 0.0);
  return eta_run(h, m, reinterpret_cast<const c128*>(lam.data()), X, b, host.data(), eta.data(), st);
}

// eta for m pairs (host points, device vectors) into host eta, with the given
// workspace or the handle's own.
nep_status backward_errors_dev(Split& h, int m, const c128* lam, const c128* X, double* eta, ExtractWork* w,
                               hipStream_t st) {
  if (!w) {
    if (!h.xw) h.xw = std::make_shared<ExtractWork>();
    w = h.xw.get();
  }
  std::vector<zc> lz(m);
  for (int q = 0; q < m; ++q) lz[q] = zc(lam[q].re, lam[q].im);
  std::vector<double> et;
  NEP_TRY(backward_errors(h, m, lz, X, et, *w, st));
  for (int q = 0; q < m; ++q) eta[q] = et[q];
  return NEP_OK;
}

nep_status rii_polish(Split& h, int m, zc* lam, c128* X, double* eta, const char* sel, double tol, int max_it,
                      int* iters, ExtractWork* w, hipStream_t st);

// ---------------------------------------------------------------------------
// Backward errors without allocation.  Callers that cannot allocate device
// memory (code under HIP graph capture, tight serving loops) use
// nep_backward_error_noalloc: its scratch is this file-scope device array, one
// copy per GPU, held until the process ends.  Host code must not use the
// array's name as a device address; each device's address comes from
// hipGetSymbolAddress, taken once per device with that device current.
constexpr int kNoAllocMaxPairs = 256;                       // m
constexpr size_t kNoAllocMaxResid = (size_t)1 << 18;        // n * m complex entries (4 MiB)
constexpr size_t kNoAllocSmall = 128 << 10;                 // points, f values, flags, maxima, term tables
constexpr size_t kNoAllocBytes = kNoAllocMaxResid * sizeof(c128) + kNoAllocSmall;
static __device__ __align__(256) char scratch[kNoAllocBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {nullptr};

static nep_status scratch_address(void** out) {
  int dev = 0;
  NEP_HIP(hipGetDevice(&dev));
  NEP_CHECK(dev >= 0 && dev < kMaxDevices, NEP_ERR_DEVICE, "device index %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      set_error("hipGetSymbolAddress of the scratch array failed: %s", hipGetErrorString(e));
      return NEP_ERR_DEVICE;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return NEP_OK;
}

static nep_status backward_errors_noalloc(Split& h, int m, const double* lambda, const c128* X, double* eta) {
  const int n = h.op.n;
  NEP_CHECK(m <= kNoAllocMaxPairs, NEP_ERR_ARG, "at most %d pairs per call without allocation (got %d)",
            kNoAllocMaxPairs, m);
  NEP_CHECK((size_t)n * m <= kNoAllocMaxResid, NEP_ERR_ARG,
            "n * m = %lld exceeds the %zu residual entries of the allocation-free scratch", (long long)n * m,
            kNoAllocMaxResid);
  static_assert(kEtaTerms + sizeof(c128) * kNoAllocMaxPairs + sizeof(c128) * kNoAllocMaxPairs * kMaxTerms +
                        sizeof(int) * kNoAllocMaxPairs + sizeof(double) * 2 * kNoAllocMaxPairs + 2 * 256 <=
                    kNoAllocSmall,
                "small scratch region too small");
  // the two host blocks take turns
  constexpr size_t kNoAllocHost = sizeof(c128) * kNoAllocMaxPairs * kMaxTerms + sizeof(double) * 2 * kNoAllocMaxPairs +
                                  sizeof(int) * kNoAllocMaxPairs;
  static_assert(kEtaTerms + sizeof(c128) * kNoAllocMaxPairs <= kNoAllocHost, "host block too small");
  void* base = nullptr;
  NEP_TRY(scratch_address(&base));
  char* p = static_cast<char*>(base);
  const EtaBuffers b = eta_carve(p + kNoAllocMaxResid * sizeof(c128), reinterpret_cast<c128*>(p), m);
  alignas(16) char host[kNoAllocHost];  // on the stack (bounded by the limits above)
  return eta_run(h, m, reinterpret_cast<const c128*>(lambda), X, b, host, eta, h.stream);
}

nep_status extract(Split& h, const nep_contour* g, const nep_ciss_opts* o, const void* S,
                   const nep_extract_opts* e, int* m_out, double* lambda, void* X, double* eta, int* inside,
                   double* sigma, ExtractWork* wk) {
  PlanOptions po;
  NEP_TRY(check_opts(o, po));
  return extract_strided(h, g, o, po.L, S, 0, e, m_out, lambda, X, eta, inside, sigma, wk);
}

nep_status extract_strided(Split& h, const nep_contour* g, const nep_ciss_opts* o, int L_eff, const void* S,
                           long long sstride, const nep_extract_opts* e, int* m_out, double* lambda, void* X,
                           double* eta, int* inside, double* sigma, ExtractWork* wk) {
  NEP_TRY(check_contour(g));
  PlanOptions po;
  NEP_TRY(check_opts(o, po));
  NEP_CHECK(e != nullptr && e->max_eigs >= 1, NEP_ERR_ARG, "extract options: max_eigs must be >= 1");
  NEP_CHECK(e->rank_tol >= 0.0 && e->eta_tol >= 0.0, NEP_ERR_ARG, "extract options: tolerances must be >= 0");
  NEP_CHECK(S != nullptr && X != nullptr && m_out && lambda && eta && inside, NEP_ERR_ARG, "null output array");
  const int n = h.op.n, L = L_eff, K = po.K;
  if (sstride <= 0) sstride = (long long)n * L;
  const long long M = (long long)K * n;
  const int KL = K * L;
  NEP_CHECK(KL <= M, NEP_ERR_ARG, "K*L exceeds K*n");
  hipStream_t st = o->stream ? (hipStream_t)o->stream : h.stream;
  if (!wk) {
    if (!h.xw) h.xw = std::make_shared<ExtractWork>();
    wk = h.xw.get();
  }
  ExtractWork& w = *wk;
  NEP_TRY(grow(w.B0, sizeof(c128) * M * KL));
  NEP_TRY(grow(w.B1, sizeof(c128) * M * KL));
  NEP_TRY(grow(w.tau, sizeof(c128) * KL));
  NEP_TRY(grow(w.Rp, sizeof(c128) * (size_t)KL * KL));
  c128* B0 = w.B0.as<c128>();
  c128* B1 = w.B1.as<c128>();
  c128* tau = w.tau.as<c128>();
  const long long tot = M * KL;
  hipLaunchKernelGGL(k_hankel, dim3((unsigned)ceil_div_ll(tot, 256)), dim3(256), 0, st, (const c128*)S, n, L, K,
                     sstride, B0, B1);
  NEP_HIP(hipGetLastError());
  NEP_HIP(house_qr(B0, M, KL, tau, st));
  // SVD of R (upper KL x KL): on the device up to kJacobiMax columns, its s
  // and W read back in one block; larger ones on the host
  NEP_TRY(grow(w.Ur, sizeof(c128) * (size_t)KL * KL));
  c128* Ur = w.Ur.as<c128>();
  std::vector<double> sv(KL);
  std::vector<zc> Wr((size_t)KL * KL);
  if (KL <= kJacobiMax) {
    const size_t woff = ((size_t)KL * sizeof(double) + 15) / 16 * 16, total = woff + sizeof(c128) * (size_t)KL * KL;
    NEP_TRY(grow(w.sw, total));
    hipLaunchKernelGGL(k_jacobi, dim3(1), dim3(kJacobiThreads), 0, st, B0, M, KL, Ur, w.sw.as<double>(),
                       reinterpret_cast<c128*>(w.sw.as<char>() + woff));
    NEP_HIP(hipGetLastError());
    std::vector<char> tmp(total);
    NEP_HIP(hipMemcpyAsync(tmp.data(), w.sw.p, total, hipMemcpyDeviceToHost, st));
    NEP_HIP(hipStreamSynchronize(st));
    std::memcpy(sv.data(), tmp.data(), sizeof(double) * KL);
    std::memcpy((void*)Wr.data(), tmp.data() + woff, sizeof(c128) * (size_t)KL * KL);
  } else {
    // (R packed on the device and read back in one plain copy: a pitched
    // device-to-host copy read back zeros in a process where a profiler had
    // loaded a second HSA runtime beside the HIP runtime's own)
    std::vector<zc> R((size_t)KL * KL), U;
    hipLaunchKernelGGL(k_pack_r, dim3((unsigned)ceil_div_ll((long long)KL * KL, 256)), dim3(256), 0, st, B0, M, KL,
                       w.Rp.as<c128>());
    NEP_HIP(hipGetLastError());
    NEP_HIP(hipMemcpyAsync(R.data(), w.Rp.p, sizeof(c128) * (size_t)KL * KL, hipMemcpyDeviceToHost, st));
    NEP_HIP(hipStreamSynchronize(st));
    for (int j = 0; j < KL; ++j)
      for (int i = j + 1; i < KL; ++i) R[(size_t)j * KL + i] = zc(0.0, 0.0);
    jacobi_svd(KL, R, sv, U, Wr);
    NEP_HIP(hipMemcpyAsync(Ur, U.data(), sizeof(c128) * (size_t)KL * KL, hipMemcpyHostToDevice, st));
    NEP_HIP(hipStreamSynchronize(st));  // U leaves scope
  }
  if (sigma)
    for (int i = 0; i < KL; ++i) sigma[i] = sv[i];
  const double tol = (e->rank_tol > 0.0 ? e->rank_tol : 1e-12) * sv[0];
  int m = 0;
  while (m < KL && sv[m] > tol) ++m;
  *m_out = m;
  NEP_CHECK(m > 0, NEP_ERR_RANK, "all moments vanish: no eigenvalue inside the contour is visible");
  NEP_CHECK(m < KL, NEP_ERR_RANK, "moment rank %d == K*L: more eigenvalues inside or near the contour pass the "
            "rank threshold than K*L=%d can resolve; increase L or K (or N)", m, KL);
  NEP_CHECK(m <= e->max_eigs, NEP_ERR_ARG, "rank %d exceeds max_eigs %d", m, e->max_eigs);
  // V0 = Q [Ur0; 0]
  NEP_TRY(grow(w.V0, sizeof(c128) * M * m));
  NEP_TRY(grow(w.wy, sizeof(c128) * (size_t)KL * m));
  c128* V0 = w.V0.as<c128>();
  {
    const int nt = ceil_div(KL, 4);
    c128* G = w.Rp.as<c128>();  // (the packed R has been read)
    hipLaunchKernelGGL(k_wy_gram, dim3(nt * (nt + 1) / 2), dim3(256), 0, st, B0, M, KL, G);
    hipLaunchKernelGGL(k_wy_coef, dim3(m), dim3(std::min(kWyRows, ceil_div(KL, 64) * 64)), 0, st, B0, M, KL, tau,
                       G, Ur, w.wy.as<c128>());
    NEP_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_wy_apply, dim3((unsigned)ceil_div_ll(M, 256), ceil_div(m, 8)), dim3(256), 0, st, B0, M, KL, m,
                       Ur, w.wy.as<c128>(), V0);
    NEP_HIP(hipGetLastError());
  }
  // Mt = V0^H B1 W0 Sigma0^{-1}
  NEP_TRY(grow(w.P, sizeof(c128) * (size_t)m * KL));
  hipLaunchKernelGGL(k_vhb, dim3(m * KL), dim3(256), 0, st, V0, B1, M, m, w.P.as<c128>());
  NEP_HIP(hipGetLastError());
  std::vector<zc> P((size_t)m * KL);
  NEP_HIP(hipMemcpyAsync(P.data(), w.P.p, sizeof(c128) * m * KL, hipMemcpyDeviceToHost, st));
  NEP_HIP(hipStreamSynchronize(st));
  std::vector<zc> Mt((size_t)m * m, zc(0.0, 0.0));
  for (int j = 0; j < m; ++j)
    for (int i = 0; i < m; ++i) {
      zc acc = 0.0;
      for (int k = 0; k < KL; ++k) acc += P[(size_t)k * m + i] * Wr[(size_t)j * KL + k];
      Mt[(size_t)j * m + i] = acc / sv[j];
    }
  std::vector<zc> mu, Sv;
  NEP_CHECK(eig_general(m, Mt, mu, Sv), NEP_ERR_RANK, "QR iteration on the projected matrix did not converge");
  // order by (Re lambda, Im lambda)
  const zc c0(g->c[0], g->c[1]);
  std::vector<zc> lam(m);
  for (int i = 0; i < m; ++i) lam[i] = c0 + g->rho * mu[i];
  std::vector<int> ord(m);
  std::iota(ord.begin(), ord.end(), 0);
  std::stable_sort(ord.begin(), ord.end(), [&](int a, int b) {
    if (lam[a].real() != lam[b].real()) return lam[a].real() < lam[b].real();
    return lam[a].imag() < lam[b].imag();
  });
  std::vector<zc> lam_s(m), Ss((size_t)m * m);
  for (int q = 0; q < m; ++q) {
    lam_s[q] = lam[ord[q]];
    for (int i = 0; i < m; ++i) Ss[(size_t)q * m + i] = Sv[(size_t)ord[q] * m + i];
  }
  NEP_TRY(grow(w.smat, sizeof(c128) * (size_t)m * m));
  NEP_HIP(hipMemcpyAsync(w.smat.p, Ss.data(), sizeof(c128) * m * m, hipMemcpyHostToDevice, st));
  hipLaunchKernelGGL(k_eigvec, dim3(m), dim3(256), 0, st, V0, M, n, m, w.smat.as<c128>(), (c128*)X);
  NEP_HIP(hipGetLastError());
  std::vector<double> et;
  NEP_TRY(backward_errors(h, m, lam_s, (const c128*)X, et, w, st));
  // The region filter (Section 3.2.4) keeps the eigenvalues inside the
  // contour; of those, a pair counts as converged when its backward error is
  // below the tolerance, the stopping test of the paper's solvers.  A pair
  // inside but above it (typically a spurious one from a numerical rank taken
  // at the moments' noise floor) is flagged apart.
  const double etol = e->eta_tol > 0.0 ? e->eta_tol : 1e-8;
  auto in_region = [&](zc l) {
    const zc mu_q = (l - c0) / g->rho;
    return g->kind == 0 ? (std::abs(mu_q) < 1.0)
                        : (mu_q.real() * mu_q.real() + (mu_q.imag() / g->v) * (mu_q.imag() / g->v) < 1.0);
  };
  if (e->polish_its > 0) {
    // pairs inside but above the tolerance (limited by the quadrature or by
    // the truncation of weakly filtered outside eigenvalues) are polished by
    // residual inverse iteration (Section 4.1) in FP64
    std::vector<char> sel(m, 0);
    int cnt = 0;
    for (int q = 0; q < m; ++q) {
      sel[q] = in_region(lam_s[q]) && !(et[q] <= etol) && std::isfinite(et[q]);
      cnt += sel[q];
    }
    if (cnt > 0) {
      NEP_TRY(rii_polish(h, m, lam_s.data(), (c128*)X, et.data(), sel.data(), 1e-14, e->polish_its, nullptr, &w, st));
      // keep the output sorted by (Re, Im): permute the eigenvectors if
      // polishing changed the order
      std::vector<int> ord2(m);
      std::iota(ord2.begin(), ord2.end(), 0);
      std::stable_sort(ord2.begin(), ord2.end(), [&](int a, int b) {
        if (lam_s[a].real() != lam_s[b].real()) return lam_s[a].real() < lam_s[b].real();
        return lam_s[a].imag() < lam_s[b].imag();
      });
      bool moved = false;
      for (int q = 0; q < m; ++q) moved |= ord2[q] != q;
      if (moved) {
        NEP_TRY(grow(w.X0, sizeof(c128) * (size_t)n * m));
        NEP_HIP(hipMemcpyAsync(w.X0.p, X, sizeof(c128) * (size_t)n * m, hipMemcpyDeviceToDevice, st));
        for (int q = 0; q < m; ++q)
          NEP_HIP(hipMemcpyAsync((c128*)X + (size_t)q * n, w.X0.as<c128>() + (size_t)ord2[q] * n, sizeof(c128) * n,
                                 hipMemcpyDeviceToDevice, st));
        NEP_HIP(hipStreamSynchronize(st));
        std::vector<zc> l2(m);
        std::vector<double> e2(m);
        for (int q = 0; q < m; ++q) {
          l2[q] = lam_s[ord2[q]];
          e2[q] = et[ord2[q]];
        }
        lam_s.swap(l2);
        et.swap(e2);
      }
    }
  }
  for (int q = 0; q < m; ++q) {
    lambda[2 * q] = lam_s[q].real();
    lambda[2 * q + 1] = lam_s[q].imag();
    eta[q] = et[q];
    inside[q] = !in_region(lam_s[q]) ? 0 : (et[q] <= etol ? 1 : 2);
  }
  // two converged pairs with one eigenvalue (a polished spurious pair can
  // land on an eigenvalue another pair already holds): the one with the
  // larger backward error is not counted
  for (int a = 0; a < m; ++a)
    for (int b = a + 1; b < m; ++b)
      if (inside[a] == 1 && inside[b] == 1 && std::abs(lam_s[a] - lam_s[b]) <= 1e-8 * std::abs(lam_s[a]))
        inside[et[a] <= et[b] ? b : a] = 2;
  return NEP_OK;
}

}  // namespace nep

using namespace nep;

extern "C" {

nep_status nep_extract(nep_split h, const nep_contour* g, const nep_ciss_opts* o, const void* S,
                       const nep_extract_opts* e, int* m, double* lambda, void* X, double* eta, int* inside,
                       double* sigma) {
  NEP_CHECK(h != nullptr, NEP_ERR_ARG, "null handle");
  return nep::extract(h->impl, g, o, S, e, m, lambda, X, eta, inside, sigma, nullptr);
}

nep_status nep_backward_error_noalloc(nep_split h, int m, const double* lambda, const void* X, double* eta) {
  NEP_CHECK(h != nullptr, NEP_ERR_ARG, "null handle");
  NEP_CHECK(m >= 1 && lambda && X && eta, NEP_ERR_ARG, "bad arguments");
  return backward_errors_noalloc(h->impl, m, lambda, (const c128*)X, eta);
}

nep_status nep_backward_error(nep_split h, int m, const double* lambda, const void* X, double* eta) {
  NEP_CHECK(h != nullptr, NEP_ERR_ARG, "null handle");
  NEP_CHECK(m >= 1 && lambda && X && eta, NEP_ERR_ARG, "bad arguments");
  if (!h->impl.xw) h->impl.xw = std::make_shared<ExtractWork>();
  std::vector<zc> lam(m);
  for (int q = 0; q < m; ++q) lam[q] = zc(lambda[2 * q], lambda[2 * q + 1]);
  std::vector<double> et;
  NEP_TRY(backward_errors(h->impl, m, lam, (const c128*)X, et, *h->impl.xw, h->impl.stream));
  for (int q = 0; q < m; ++q) eta[q] = et[q];
  return NEP_OK;
}

}  // extern "C"
