// Operators whose every term is diagonal or real banded with a half-width of
// at most kNarrowMax: T(z_j) is itself banded, and its factorization, solves
// and residual run on the band alone.
//
// The dense path spends (8/3) n^3 flops and n^2 entries of memory per node on
// such a matrix (the rational string's terms are tridiagonal); elimination
// with partial pivoting inside the band needs O(n W^2) and 3W + 2 entries per
// row.  What is left is a serial chain of n steps per node, so one lane runs
// one node (factorization) or one node and probe column (solves), the window
// of W + 1 rows in registers, and the lanes of a wave read and write
// consecutive entries: the factor is stored [row][entry][node], the right-hand
// sides [row][node][column].  A lane's next rows are loaded into a second
// register buffer while the current ones are eliminated.  Measured against the
// dense path: 256 strings of 64..1024 rows (32 nodes, 8 probes) 187 -> 5.7 ms
// per batch, one string of 200 rows with its extraction 1.44 -> 0.74 ms, of 65
// rows 0.93 -> 0.53 ms; there is no size at which the dense path is faster.
//
// Storage of a problem (element offset offF), NE = 3W + 2 entries per row:
//   0 .. 2W       first T(row, row - W .. row + W), then U(row, row .. row + 2W)
//   2W + 1        1 / U(row, row)
//   2W + 2 ..     the W multipliers of elimination step `row`
// and one byte per (row, node) at offP: which of the window's W + 1 rows was
// the pivot of that step.
#include <algorithm>

#include "engine.hpp"

namespace nep {

int band_class(int w) { return w <= 1 ? 1 : w <= 2 ? 2 : 4; }

template <int W>
constexpr int kBandEntries = 3 * W + 2;

int band_entries(int W) { return 3 * W + 2; }

template <typename P>
__device__ __forceinline__ cx<P> recip_p(cx<P> a) {
  if constexpr (sizeof(P) == 4) return recip_f32(a);
  else return recip(a);
}

// ---------------------------------------------------------------------------
// Assembly of the band: one thread per (row, node), node fastest; the FP64
// sums over the terms run in the order of the dense assembly and are rounded
// once.
// ---------------------------------------------------------------------------
template <typename P, int W>
__global__ __launch_bounds__(256) void k_band_assemble(const ProbDesc* __restrict__ pd,
                                                       const int* __restrict__ prefix, int cnt, int total,
                                                       NodeArrays na, cx<P>* __restrict__ F,
                                                       const int* __restrict__ skip) {
  const int v = xcd_remap(blockIdx.x, gridDim.x, total);
  if (v < 0) return;
  const int p = find_slot(prefix, cnt, v);
  const ProbDesc& D = pd[p];
  const int e = (v - prefix[p]) * 256 + threadIdx.x;
  const int n = D.n, N = D.N;
  if (e >= n * N) return;
  const int r = e / N, j = e - r * N, g = D.node0 + j;
  if (skip != nullptr && skip[g]) return;
  double sr[2 * W + 1], si[2 * W + 1];
#pragma unroll
  for (int d = 0; d <= 2 * W; ++d) sr[d] = si[d] = 0.0;
  for (int i = 0; i < D.ell; ++i) {
    const c128 f = na.fz[(long long)g * kMaxTerms + i];
    if (D.a_is_diag[i]) {
      const c128 a = D.Adiag[i][r];
      sr[W] += f.re * a.re - f.im * a.im;
      si[W] += f.re * a.im + f.im * a.re;
      continue;
    }
    const double* __restrict__ A = reinterpret_cast<const double*>(D.A[i]) + (long long)r * n;
#pragma unroll
    for (int d = 0; d <= 2 * W; ++d) {
      const int c = r + d - W;
      if (c >= 0 && c < n) {
        const double a = A[c];
        sr[d] += f.re * a;
        si[d] += f.im * a;
      }
    }
  }
  cx<P>* out = F + D.offF + (long long)r * kBandEntries<W> * N + j;
#pragma unroll
  for (int d = 0; d <= 2 * W; ++d) out[(long long)d * N] = cx<P>{P(sr[d]), P(si[d])};
}

// ---------------------------------------------------------------------------
// Factorization: one lane per node.  Bound by the latency of the chain (the
// pivot's modulus, its reciprocal, the multiplier, the next pivot column), not
// by memory: a tridiagonal step is about 60 instructions.
// ---------------------------------------------------------------------------
template <typename P, int W>
__global__ __launch_bounds__(64, 1) void k_band_lu(const ProbDesc* __restrict__ pd, const int* __restrict__ prefix,
                                                   int cnt, cx<P>* __restrict__ Fb, unsigned char* __restrict__ Pb,
                                                   int* __restrict__ info, double* __restrict__ pmin,
                                                   const int* __restrict__ skip) {
  const int v = blockIdx.x;
  const int p = find_slot(prefix, cnt, v);
  const ProbDesc& D = pd[p];
  const int n = D.n, N = D.N, j = (v - prefix[p]) * 64 + threadIdx.x;
  if (j >= N) return;
  const int g = D.node0 + j;
  if (skip != nullptr && skip[g]) return;
  constexpr int NE = kBandEntries<W>;
  constexpr int U = (W == 1 ? 16 : W == 2 ? 8 : 4) / (sizeof(P) == 8 ? 2 : 1);  // rows per register buffer
  cx<P>* __restrict__ F = Fb + D.offF + j;
  unsigned char* __restrict__ pv = Pb + D.offP + j;
  const long long rs = (long long)NE * N;  // row stride

  cx<P> a[W + 1][2 * W + 1];
  // rows 0..W: row i holds columns 0..2W (entry c - i + W of its band)
#pragma unroll
  for (int i = 0; i <= W; ++i)
#pragma unroll
    for (int c = 0; c <= 2 * W; ++c) {
      const int k = c - i + W;
      a[i][c] = (i < n && k >= 0 && k <= 2 * W) ? F[i * rs + (long long)(k <= 2 * W ? k : 0) * N] : cx<P>{P(0), P(0)};
    }
  struct Buf {
    cx<P> t[U][2 * W + 1];
  };
  Buf b0, b1;
  auto load = [&](Buf& b, int r0) {  // rows r0 .. r0 + U - 1 (clamped; masked when used)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const cx<P>* src = F + min(r0 + u, n - 1) * rs;
#pragma unroll
      for (int k = 0; k <= 2 * W; ++k) b.t[u][k] = src[(long long)k * N];
    }
  };
  int zp = n;
  double m2 = INFINITY;
  auto process = [&](const Buf& b, int r0) {  // steps r0 .. r0 + U - 1; b holds rows r0 + W + 1 ..
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int r = r0 + u;
      if (r < n) {  // uniform over the problem's lanes
        int q = 0;
        P best = abs1(a[0][0]);
#pragma unroll
        for (int i = 1; i <= W; ++i) {
          const P m = abs1(a[i][0]);
          if (m > best) {
            best = m;
            q = i;
          }
        }
#pragma unroll
        for (int c = 0; c <= 2 * W; ++c) {
          cx<P> top = a[0][c];
#pragma unroll
          for (int i = 1; i <= W; ++i) {
            const cx<P> x = a[i][c];
            a[i][c] = csel(q == i, a[0][c], x);
            top = csel(q == i, x, top);
          }
          a[0][c] = top;
        }
        const cx<P> piv = a[0][0];
        if (piv.re == P(0) && piv.im == P(0) && zp == n) zp = r;
        const double a2 = double(piv.re) * double(piv.re) + double(piv.im) * double(piv.im);
        m2 = (a2 < m2 || a2 != a2) ? a2 : m2;
        const cx<P> inv = recip_p(piv);
        cx<P>* dst = F + r * rs;
#pragma unroll
        for (int i = 1; i <= W; ++i) {
          const cx<P> l = a[i][0] * inv;
          dst[(long long)(2 * W + 1 + i) * N] = l;
#pragma unroll
          for (int c = 1; c <= 2 * W; ++c) a[i][c] = fms(a[i][c], l, a[0][c]);
        }
#pragma unroll
        for (int c = 0; c <= 2 * W; ++c) dst[(long long)c * N] = a[0][c];
        dst[(long long)(2 * W + 1) * N] = inv;
        pv[(long long)r * N] = (unsigned char)q;
        // shift; row r + W + 1 enters with columns r + 1 .. r + 1 + 2W
        const bool in = r + W + 1 < n;
#pragma unroll
        for (int i = 1; i <= W; ++i) {
#pragma unroll
          for (int c = 1; c <= 2 * W; ++c) a[i - 1][c - 1] = a[i][c];
          a[i - 1][2 * W] = cx<P>{P(0), P(0)};
        }
#pragma unroll
        for (int c = 0; c <= 2 * W; ++c) a[W][c] = csel(in, b.t[u][c], cx<P>{P(0), P(0)});
      }
    }
  };
  load(b0, W + 1);
  for (int r0 = 0; r0 < n; r0 += 2 * U) {
    load(b1, r0 + U + W + 1);
    process(b0, r0);
    load(b0, r0 + 2 * U + W + 1);
    process(b1, r0 + U);
  }
  info[g] = zp;
  if (pmin != nullptr) pmin[g] = sqrt(m2);
}

// ---------------------------------------------------------------------------
// Solve: one lane per (node, probe column).  kBandV: right-hand side V, Y = x;
// kBandR: right-hand side R, Y = x; kBandRefine: right-hand side R, Y += x.
// The forward sweep leaves its result where the backward sweep reads it.  With
// FP32 factors that is Wb, in FP32 as it was computed: the solve is bound by
// memory, and through R or Y it was widened to 16 bytes and back (256 strings of
// 64..1024 rows, 32 nodes, 8 probes: 542 -> 484 us a sweep).  With FP64
// factors it is Y, which then takes the solution, or, where Y's old value is
// needed, R (which the next residual recomputes).
// ---------------------------------------------------------------------------
template <typename P, int W>
__global__ __launch_bounds__(64, 1) void k_band_solve(const ProbDesc* __restrict__ pd, const int* __restrict__ prefix,
                                                      int cnt, const cx<P>* __restrict__ Fb,
                                                      const unsigned char* __restrict__ Pb, c128* __restrict__ Rb,
                                                      c128* __restrict__ Yb, cx<P>* __restrict__ Wb, int mode,
                                                      const int* __restrict__ conv, IrState ir) {
  const int v = blockIdx.x;
  const int p = find_slot(prefix, cnt, v);
  const ProbDesc& D = pd[p];
  const int n = D.n, N = D.N, L = D.L, NL = N * L, e = (v - prefix[p]) * 64 + threadIdx.x;
  if (e >= NL) return;
  const int j = e / L, c = e - j * L, g = D.node0 + j;
  if (conv != nullptr && conv[g]) return;
  constexpr int NE = kBandEntries<W>;
  constexpr int U = (W == 1 ? 16 : W == 2 ? 8 : 4) / (sizeof(P) == 8 ? 2 : 1);
  const cx<P>* __restrict__ F = Fb + D.offF + j;
  const unsigned char* __restrict__ pv = Pb + D.offP + j;
  const long long rs = (long long)NE * N;
  const bool refine = mode == kBandRefine;
  c128* Y = Yb + D.offY + e;
  cx<P>* W0;  // the forward sweep's result
  if constexpr (sizeof(P) == 4) W0 = Wb + D.offBW + e;
  else W0 = refine ? Rb + D.offY + e : Y;
  const c128* V = mode == kBandV ? D.V + (long long)c * n : Rb + D.offY + e;
  const long long vs = mode == kBandV ? 1 : NL;

  {  // forward: P L y = b
    cx<P> t[W + 1];
#pragma unroll
    for (int i = 0; i <= W; ++i) t[i] = i < n ? cvt<P>(V[i * vs]) : cx<P>{P(0), P(0)};
    struct Buf {
      cx<P> l[U][W];
      c128 b[U];
      int q[U];
    };
    Buf b0, b1;
    auto load = [&](Buf& b, int r0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = min(r0 + u, n - 1);
        b.q[u] = pv[(long long)r * N];
#pragma unroll
        for (int i = 0; i < W; ++i) b.l[u][i] = F[r * rs + (long long)(2 * W + 2 + i) * N];
        b.b[u] = V[min(r0 + u + W + 1, n - 1) * vs];
      }
    };
    auto process = [&](const Buf& b, int r0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = r0 + u;
        if (r < n) {
          cx<P> top = t[0];
#pragma unroll
          for (int i = 1; i <= W; ++i) {
            const cx<P> x = t[i];
            t[i] = csel(b.q[u] == i, t[0], x);
            top = csel(b.q[u] == i, x, top);
          }
          W0[(long long)r * NL] = top;
#pragma unroll
          for (int i = 1; i <= W; ++i) t[i - 1] = fms(t[i], b.l[u][i - 1], top);
          t[W] = csel(r + W + 1 < n, cvt<P>(b.b[u]), cx<P>{P(0), P(0)});
        }
      }
    };
    load(b0, 0);
    for (int r0 = 0; r0 < n; r0 += 2 * U) {
      load(b1, r0 + U);
      process(b0, r0);
      load(b0, r0 + 2 * U);
      process(b1, r0 + U);
    }
  }
  // backward: U x = y, rows n - 1 down to 0
  double y2 = 0.0;
  cx<P> x[2 * W];
#pragma unroll
  for (int i = 0; i < 2 * W; ++i) x[i] = cx<P>{P(0), P(0)};
  constexpr int UB = U > 1 ? U / 2 : 1;
  struct Buf {
    cx<P> u[UB][2 * W], inv[UB];
    cx<P> y[UB];
    c128 o[UB];
  };
  Buf b0, b1;
  auto load = [&](Buf& b, int r0) {  // rows r0, r0 - 1, ..
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int r = max(r0 - u, 0);
#pragma unroll
      for (int i = 0; i < 2 * W; ++i) b.u[u][i] = F[r * rs + (long long)(1 + i) * N];
      b.inv[u] = F[r * rs + (long long)(2 * W + 1) * N];
      b.y[u] = W0[(long long)r * NL];
      if (refine) b.o[u] = Y[(long long)r * NL];
    }
  };
  auto process = [&](const Buf& b, int r0) {
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int r = r0 - u;
      if (r >= 0) {
        cx<P> s = b.y[u];
        // the nearest unknown last: the others do not wait for it
#pragma unroll
        for (int i = 2 * W - 1; i >= 0; --i) s = fms(s, b.u[u][i], x[i]);
        s = s * b.inv[u];
#pragma unroll
        for (int i = 2 * W - 1; i >= 1; --i) x[i] = x[i - 1];
        x[0] = s;
        c128 nv = {double(s.re), double(s.im)};
        if (refine) nv = b.o[u] + nv;
        Y[(long long)r * NL] = nv;
        y2 = nanmax(y2, norm2(nv));
      }
    }
  };
  load(b0, n - 1);
  for (int r0 = n - 1; r0 >= 0; r0 -= 2 * UB) {
    load(b1, r0 - UB);
    process(b0, r0);
    load(b0, r0 - 2 * UB);
    process(b1, r0 - UB);
  }
  atomicMax(&ir.ynorm[(long long)g * kNormStride + c], (unsigned long long)__double_as_longlong(sqrt(y2)));
}

// ---------------------------------------------------------------------------
// Residual R = V - sum_i f_i(z_j) A_i Y_j over the band, FP64: a wave takes
// kBandRows rows of 64 consecutive (node, column) entries, so Y is read once
// (plus 2W rows of overlap) and R written once; bound by memory.  The matrix
// core kernel runs such a term's band in 64 x 64 tiles, most of whose products
// are by zeros (24 -> 7 ms per 256-problem batch when it took the place of
// dense products).
// ---------------------------------------------------------------------------
constexpr int kBandRows = 8;

template <int W>
__global__ __launch_bounds__(256) void k_band_resid(const ProbDesc* __restrict__ pd, const int* __restrict__ prefix,
                                                    int cnt, int total, NodeArrays na, const c128* __restrict__ Yb,
                                                    c128* __restrict__ Rb, IrState ir) {
  const int v = xcd_remap(blockIdx.x, gridDim.x, total);
  if (v < 0) return;
  const int p = find_slot(prefix, cnt, v);
  const ProbDesc& D = pd[p];
  const int n = D.n, L = D.L, NL = D.N * L;
  const int eb = (NL + 63) / 64;
  const int t = v - prefix[p], tr = t / eb;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e = (t - tr * eb) * 64 + lane;
  const int r0 = (tr * 4 + wave) * kBandRows;
  const int j = min(e, NL - 1) / L, c = min(e, NL - 1) - j * L, g = D.node0 + j;
  const bool live = e < NL && !ir.conv[g];
  __shared__ double red[4][64];
  double m2 = 0.0;
  if (live && r0 < n) {
    const c128* __restrict__ Y = Yb + D.offY + e;
    c128 y[kBandRows + 2 * W], acc[kBandRows];
#pragma unroll
    for (int k = 0; k < kBandRows + 2 * W; ++k) {
      const int r = r0 - W + k;
      y[k] = (r >= 0 && r < n) ? Y[(long long)r * NL] : c128{0.0, 0.0};
    }
#pragma unroll
    for (int k = 0; k < kBandRows; ++k)
      acc[k] = r0 + k < n ? D.V[(long long)c * n + r0 + k] : c128{0.0, 0.0};
    for (int i = 0; i < D.ell; ++i) {
      const c128 f = na.fz[(long long)g * kMaxTerms + i];
      if (D.a_is_diag[i]) {
        const c128* __restrict__ dg = D.Adiag[i];
#pragma unroll
        for (int k = 0; k < kBandRows; ++k)
          if (r0 + k < n) acc[k] = fms(acc[k], f * dg[r0 + k], y[k + W]);
        continue;
      }
      const double* __restrict__ A = reinterpret_cast<const double*>(D.A[i]);
#pragma unroll
      for (int k = 0; k < kBandRows; ++k) {
        if (r0 + k >= n) continue;
        c128 s = {0.0, 0.0};
#pragma unroll
        for (int d = 0; d <= 2 * W; ++d) {
          const int cc = r0 + k + d - W;
          const double a = (cc >= 0 && cc < n) ? A[(long long)(r0 + k) * n + cc] : 0.0;
          s.re = fma(a, y[k + d].re, s.re);
          s.im = fma(a, y[k + d].im, s.im);
        }
        acc[k] = fms(acc[k], f, s);
      }
    }
    c128* __restrict__ R = Rb + D.offY + e;
#pragma unroll
    for (int k = 0; k < kBandRows; ++k)
      if (r0 + k < n) {
        R[(long long)(r0 + k) * NL] = acc[k];
        m2 = nanmax(m2, norm2(acc[k]));
      }
  }
  red[wave][lane] = m2;
  __syncthreads();
  if (wave == 0 && live) {
#pragma unroll
    for (int w = 1; w < 4; ++w) m2 = nanmax(m2, red[w][lane]);
    atomicMax(&ir.rnorm[(long long)g * kNormStride + c], (unsigned long long)__double_as_longlong(sqrt(m2)));
  }
}

// log|det| and arg det per node from the factor: the pivots, and one sign
// change per step whose pivot was not the window's first row.
template <typename P, int W>
__global__ __launch_bounds__(64) void k_band_logdet(const ProbDesc* __restrict__ pd, const int* __restrict__ prefix,
                                                    int cnt, const cx<P>* __restrict__ Fb,
                                                    const unsigned char* __restrict__ Pb, int nnodes,
                                                    double* __restrict__ out) {
  const int v = blockIdx.x;
  const int p = find_slot(prefix, cnt, v);
  const ProbDesc& D = pd[p];
  const int n = D.n, N = D.N, j = v - prefix[p];  // one wave per node
  double la = 0.0, ar = 0.0;
  for (int r = threadIdx.x; r < n; r += 64) {
    const cx<P> u = Fb[D.offF + (long long)r * kBandEntries<W> * N + j];
    const double re = double(u.re), im = double(u.im);
    la += log(hypot(re, im));
    ar += atan2(im, re) + (Pb[D.offP + (long long)r * N + j] ? M_PI : 0.0);
  }
  for (int o = 32; o >= 1; o >>= 1) {
    la += __shfl_xor(la, o, 64);
    ar += __shfl_xor(ar, o, 64);
  }
  if (threadIdx.x == 0) {
    out[D.node0 + j] = la;
    out[nnodes + D.node0 + j] = remainder(ar, 2.0 * M_PI);
  }
}

// ---------------------------------------------------------------------------
// Host side: one launch per band class present in the plan.
// ---------------------------------------------------------------------------
void band_tables(BandTables& bt, std::vector<int>& buf, const std::vector<ProbDesc>& pd) {
  for (int k = 0; k < kBandClasses; ++k) {
    std::vector<int> ca, cl, cs, cr, cd;
    for (const ProbDesc& D : pd) {
      const bool in = D.band == (1 << k);
      const int NL = D.N * D.L;
      ca.push_back(in ? (int)ceil_div_ll((long long)D.n * D.N, 256) : 0);
      cl.push_back(in ? ceil_div(D.N, 64) : 0);
      cs.push_back(in ? ceil_div(NL, 64) : 0);
      cr.push_back(in ? ceil_div(D.n, 4 * kBandRows) * ceil_div(NL, 64) : 0);
      cd.push_back(in ? D.N : 0);
    }
    build_prefix(buf, bt.assemble[k], ca);
    build_prefix(buf, bt.lu[k], cl);
    build_prefix(buf, bt.solve[k], cs);
    build_prefix(buf, bt.resid[k], cr);
    build_prefix(buf, bt.node[k], cd);
  }
}

#define NEP_BAND_CLASSES(CALL) \
  do {                         \
    CALL(0, 1);                \
    CALL(1, 2);                \
    CALL(2, 4);                \
  } while (0)

template <typename P>
hipError_t band_factor(const BandTables& bt, const ProbDesc* pd, const int* prefix, const NodeArrays& na, cx<P>* F,
                       unsigned char* piv, int* info, double* pmin, const int* skip, hipStream_t st) {
#define NEP_BAND_LU(k, W)                                                                                       \
  if (bt.lu[k].total > 0) {                                                                                     \
    const Table &ta = bt.assemble[k], &tl = bt.lu[k];                                                           \
    hipLaunchKernelGGL((k_band_assemble<P, W>), dim3(xcd_grid(ta.total)), dim3(256), 0, st, pd, prefix + ta.off, \
                       ta.cnt, ta.total, na, F, skip);                                                          \
    hipLaunchKernelGGL((k_band_lu<P, W>), dim3(tl.total), dim3(64), 0, st, pd, prefix + tl.off, tl.cnt, F, piv, \
                       info, pmin, skip);                                                                       \
  }
  NEP_BAND_CLASSES(NEP_BAND_LU);
#undef NEP_BAND_LU
  return hipGetLastError();
}

template <typename P>
hipError_t band_solve(const BandTables& bt, const ProbDesc* pd, const int* prefix, const cx<P>* F,
                      const unsigned char* piv, c128* R, c128* Y, cx<P>* Wf, int mode, const int* conv, IrState ir,
                      hipStream_t st) {
#define NEP_BAND_SOLVE(k, W)                                                                                      \
  if (bt.solve[k].total > 0)                                                                                      \
  hipLaunchKernelGGL((k_band_solve<P, W>), dim3(bt.solve[k].total), dim3(64), 0, st, pd, prefix + bt.solve[k].off, \
                     bt.solve[k].cnt, F, piv, R, Y, Wf, mode, conv, ir)
  NEP_BAND_CLASSES(NEP_BAND_SOLVE);
#undef NEP_BAND_SOLVE
  return hipGetLastError();
}

hipError_t band_resid(const BandTables& bt, const ProbDesc* pd, const int* prefix, const NodeArrays& na,
                      const c128* Y, c128* R, IrState ir, hipStream_t st) {
#define NEP_BAND_RESID(k, W)                                                                              \
  if (bt.resid[k].total > 0)                                                                              \
  hipLaunchKernelGGL((k_band_resid<W>), dim3(xcd_grid(bt.resid[k].total)), dim3(256), 0, st, pd,           \
                     prefix + bt.resid[k].off, bt.resid[k].cnt, bt.resid[k].total, na, Y, R, ir)
  NEP_BAND_CLASSES(NEP_BAND_RESID);
#undef NEP_BAND_RESID
  return hipGetLastError();
}

template <typename P>
hipError_t band_logdet(const BandTables& bt, const ProbDesc* pd, const int* prefix, const cx<P>* F,
                       const unsigned char* piv, int nnodes, double* out, hipStream_t st) {
#define NEP_BAND_DET(k, W)                                                                                       \
  if (bt.node[k].total > 0)                                                                                      \
  hipLaunchKernelGGL((k_band_logdet<P, W>), dim3(bt.node[k].total), dim3(64), 0, st, pd, prefix + bt.node[k].off, \
                     bt.node[k].cnt, F, piv, nnodes, out)
  NEP_BAND_CLASSES(NEP_BAND_DET);
#undef NEP_BAND_DET
  return hipGetLastError();
}

#define NEP_BAND_INST(P)                                                                                             \
  template hipError_t band_factor<P>(const BandTables&, const ProbDesc*, const int*, const NodeArrays&, cx<P>*,      \
                                     unsigned char*, int*, double*, const int*, hipStream_t);                        \
  template hipError_t band_solve<P>(const BandTables&, const ProbDesc*, const int*, const cx<P>*,                    \
                                    const unsigned char*, c128*, c128*, cx<P>*, int, const int*, IrState, hipStream_t); \
  template hipError_t band_logdet<P>(const BandTables&, const ProbDesc*, const int*, const cx<P>*,                   \
                                     const unsigned char*, int, double*, hipStream_t);
NEP_BAND_INST(float)
NEP_BAND_INST(double)
#undef NEP_BAND_INST

}  // namespace nep
