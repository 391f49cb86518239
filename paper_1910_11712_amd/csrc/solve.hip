// Batched triangular solves with the factors of k_lu_*: Y_j = T(z_j)^{-1} B,
// with P T = L U (P through the row map), B the probe block V or a
// refinement residual R.
//
// The LU writes, as its panels complete, the inverses of the 64 x 64 diagonal
// blocks of L (unit lower) and U.  One launch per solve and size class: a
// group owns one node and a group of right-hand columns and runs forward then
// backward substitution over 64-row blocks, right-looking, with the right-hand
// sides of all rows in registers: k_trsm on the matrix cores (8 columns), or
// k_trsv on the vector units (4, 8 or 16), which is left for complex-FP64
// factors of more than 1024 rows and for the tuner.  The right-hand side is
// gathered through the row map; the result is stored to (or, for a correction,
// added to) Y in FP64, with the column maxima of |Y| for the refinement test.
#include "engine.hpp"

namespace nep {

// Threads per group: 512 for matrices of more than 512 rows, 256 below
// (two rows per thread up to 512 rows, one up to 256), so that small matrices
// of a ragged batch do not leave most of a large group idle.
constexpr int kTrsvThreads = 512, kTrsvThreadsSmall = 256;
constexpr int kTrsmCols = 8;  // right-hand columns per group of k_trsm

// ---------------------------------------------------------------------------
// Right-looking substitution with the accumulators in registers: thread t
// owns the logical rows t, t+512, ...  For each 64-row block (in order for
// L, reversed for U):
//   1. the owners of the block's rows publish t = acc (their pending sums)
//      and the group stages the stored inverse of the diagonal block;
//   2. x_q = Dinv_q t (all threads, 64 rows x LG columns);
//   3. every row not yet solved pulls its 64-wide segment of the factor and
//      subtracts segment * x_q from its accumulators.
// Step 3 issues many independent row loads, so the solve streams the factor
// instead of waiting on one dependent chain.
// 16 consecutive elements of a factor row; the segment starts at a multiple
// of 64 elements of a row whose stride is a multiple of 16, so it is 16-byte
// aligned.
__device__ __forceinline__ void load_seg16(const c64* __restrict__ s, c64 (&v)[16]) {
  const float4* q = reinterpret_cast<const float4*>(s);
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const float4 t = q[u];
    v[2 * u] = {t.x, t.y};
    v[2 * u + 1] = {t.z, t.w};
  }
}
__device__ __forceinline__ void load_seg16(const c128* __restrict__ s, c128 (&v)[16]) {
  const double2* q = reinterpret_cast<const double2*>(s);
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const double2 t = q[u];
    v[u] = {t.x, t.y};
  }
}

template <int Q, typename P>
__device__ __forceinline__ void load_seg(const cx<P>* __restrict__ s, cx<P> (&v)[Q]) {
  static_assert(Q % 16 == 0, "segments of 16 elements");
#pragma unroll
  for (int k = 0; k < Q; k += 16) {
    cx<P> t[16];
    load_seg16(s + k, t);
#pragma unroll
    for (int u = 0; u < 16; ++u) v[k + u] = t[u];
  }
}

// 256-thread groups with four rows per thread (the large class of big
// batches, two or more groups per CU) are held to three waves per SIMD: 168
// registers with a small spill, three groups per CU instead of two (the
// 256-problem batch 204.4 -> 203.1 ms)
template <typename P, int LG, int RPT, int NT>
__global__ __launch_bounds__(NT, (NT == 256 && RPT == 4) ? 3 : 1) void k_trsv(const MatDesc* __restrict__ md, int nmat, int groups,
                                                      const ProbDesc* __restrict__ pd, NodeArrays na,
                                                      const cx<P>* __restrict__ Tb, const int* __restrict__ rows,
                                                      const cx<P>* __restrict__ Dinv,
                                                      const long long* __restrict__ dinv_off,
                                                      const c128* __restrict__ R, c128* __restrict__ Y, int refine,
                                                      const int* __restrict__ conv, IrState ir) {
  constexpr int B = kSolveBlk;  // 64
  // register budget (32-bit words per thread) of the prefetched segment
  // columns (PF per row) and of the rows whose 16-column chunks load together
  // (GR): accumulators + prefetch + one chunk per grouped row stay within it
  constexpr int FW = 2 * (int)(sizeof(P) / 4);  // words per complex
  constexpr int kBudget = sizeof(P) == 8 ? 112 : 176;
  constexpr int PF = RPT * FW * (32 + 16 + LG) <= kBudget   ? 32
                     : RPT * FW * (16 + 16 + LG) <= kBudget ? 16
                                                            : 0;
  constexpr int GR = RPT * FW * (PF + 16 + LG) <= kBudget ? RPT : 1;
  // full blocks as a pipeline of 16-column chunks in two register buffers
  // (the prefetched first chunk is one of them): each chunk's loads are in
  // flight while the previous chunk is applied
  constexpr bool PIPE = PF == 16 && RPT * FW * (2 * 16 + LG) <= 160;
  // the column groups of one matrix run on one XCD and share its L2
  const int v = xcd_remap(blockIdx.x, gridDim.x, nmat * groups);
  if (v < 0) return;
  const int b = v / groups, grp = v - b * groups;
  const MatDesc d = md[b];
  const int g = d.node;
  if (conv != nullptr && conv[g]) return;
  const int p = na.prob[g], j = na.jnode[g];
  const ProbDesc& D = pd[p];
  const int n = d.n, ld = d.ld, L = D.L;
  const int c0 = grp * LG;
  const int nc = min(LG, L - c0);
  if (nc <= 0) return;
  const cx<P>* __restrict__ T = Tb + d.offT;
  const int* __restrict__ rat = rows + d.offRow;
  const cx<P>* __restrict__ Di = Dinv + dinv_off[b];
  const int nblk = (n + B - 1) / B;
  const int tid = threadIdx.x;

  __shared__ cx<P> Ds[B][B + 1];   // diagonal-block inverse
  __shared__ cx<P> Ts[B][LG];      // block right-hand side
  __shared__ cx<P> Xs[B][LG];      // block solution
  __shared__ double cmax[NT / 64][LG];

  // rows of this thread: slot i holds row i*T + tid (i even) or
  // (i+1)*T - 1 - tid (i odd), so every thread has rows from both ends and
  // the pending rows of a block are spread evenly over the waves
  auto row_of = [&](int i) { return (i & 1) ? (i + 1) * NT - 1 - tid : i * NT + tid; };
  // right-hand side P b gathered into the owners' accumulators
  cx<P> acc[RPT][LG];
  long long rowoff[RPT];
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int r = row_of(i);
    const int pr = r < n ? rat[r] : 0;
    rowoff[i] = (long long)pr * ld;
#pragma unroll
    for (int c = 0; c < LG; ++c) {
      c128 bv = {0.0, 0.0};
      if (r < n && c < nc)
        bv = refine ? R[D.offY + (long long)pr * D.N * L + (long long)j * L + c0 + c] : D.V[(long long)(c0 + c) * n + pr];
      acc[i][c] = cvt<P>(bv);
    }
  }
  double ymax[LG];
#pragma unroll
  for (int c = 0; c < LG; ++c) ymax[c] = 0.0;

  constexpr int DPT = B * B / NT;  // inverse elements per thread
  static_assert(DPT * NT == B * B, "inverse staging");
  cx<P> dreg[DPT];
#pragma unroll
  for (int u = 0; u < DPT; ++u) {  // block 0 of L
    const cx<P>* src = Di + tid + u * NT;
    dreg[u] = cx<P>{src->re, src->im};
  }
  for (int pass = 0; pass < 2; ++pass) {  // 0: L y = P b, 1: U x = y
    for (int qq = 0; qq < nblk; ++qq) {
      const int q = pass == 0 ? qq : nblk - 1 - qq;
      const int R0 = q * B, nr = min(B, n - R0);
      // 0. the factor segments of the pending rows do not depend on this
      // block's solution: the first PF columns are loaded now and arrive
      // while the block is solved
      cx<P> pre[RPT][PF > 0 ? PF : 1];
      if constexpr (PF > 0) {
        if (nr == B) {
#pragma unroll
          for (int i = 0; i < RPT; ++i) {
            const int r = row_of(i);
            if (r < n && (pass == 0 ? r >= R0 + B : r < R0)) load_seg<PF>(T + rowoff[i] + R0, pre[i]);
          }
        }
      }
      // 1. publish the block's pending sums; stage the inverse
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int r = row_of(i);
        if (r >= R0 && r < R0 + B) {
#pragma unroll
          for (int c = 0; c < LG; ++c) Ts[r - R0][c] = r < n ? acc[i][c] : cx<P>{P(0), P(0)};
        }
      }
      // the block's inverse arrived in registers during the previous block
      // (identity-padded past nr, so no masking is needed)
#pragma unroll
      for (int u = 0; u < DPT; ++u) {
        const int e = tid + u * NT;
        Ds[e / B][e % B] = cx<P>{dreg[u].re, dreg[u].im};
      }
      __syncthreads();
      // 2. x_q = Dinv_q t
      for (int e = tid; e < B * LG; e += NT) {
        const int i = e / LG, c = e - i * LG;
        cx<P> x = {P(0), P(0)};
#pragma unroll 16
        for (int k = 0; k < B; ++k) x = cmac(x, Ds[i][k], Ts[k][c]);
        Xs[i][c] = x;
      }
      __syncthreads();
      // prefetch the next block's inverse (forward order in pass 0, then
      // backward in pass 1)
      {
        const bool last = pass == 1 && qq + 1 == nblk;
        const int nq = pass == 0 ? (qq + 1 < nblk ? q + 1 : nblk - 1) : q - 1;
        const int npass = (pass == 0 && qq + 1 == nblk) ? 1 : pass;
        if (!last) {
          const cx<P>* __restrict__ nx = Di + ((long long)nq * 2 + npass) * B * B;
#pragma unroll
          for (int u = 0; u < DPT; ++u) {
            const cx<P>* src = nx + tid + u * NT;
            dreg[u] = cx<P>{src->re, src->im};
          }
        }
      }
      // 3. rows still pending subtract (factor segment) * x_q; the block's own
      // rows take their solution
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int r = row_of(i);
        if (r >= n) continue;
        if (r >= R0 && r < R0 + nr) {
#pragma unroll
          for (int c = 0; c < LG; ++c) acc[i][c] = Xs[r - R0][c];
          continue;
        }
        const bool pending = pass == 0 ? r >= R0 + nr : r < R0;
        if (!pending) continue;
        const cx<P>* __restrict__ seg = T + rowoff[i] + R0;
        if (nr == B && PIPE) continue;  // applied by the pipeline below
        if (nr == B) {  // full block: prefetched part first
#pragma unroll
          for (int u = 0; u < PF; ++u)
#pragma unroll
            for (int c = 0; c < LG; ++c) acc[i][c] = fms(acc[i][c], pre[i][u], Xs[u][c]);
        } else {  // ragged last block
          for (int k = 0; k < nr; ++k) {
            const cx<P> lv = seg[k];
#pragma unroll
            for (int c = 0; c < LG; ++c) acc[i][c] = fms(acc[i][c], lv, Xs[k][c]);
          }
        }
      }
      if constexpr (PIPE) {
        if (nr == B) {
          bool pend[RPT];
#pragma unroll
          for (int i = 0; i < RPT; ++i) {
            const int r = row_of(i);
            pend[i] = r < n && (pass == 0 ? r >= R0 + B : r < R0);
          }
          cx<P> nb[RPT][16];
          auto issue = [&](cx<P> (&buf)[RPT][PF > 0 ? PF : 1], int k0) {
#pragma unroll
            for (int i = 0; i < RPT; ++i)
              if (pend[i]) load_seg16(T + rowoff[i] + R0 + k0, reinterpret_cast<cx<P>(&)[16]>(buf[i]));
          };
          auto issue_nb = [&](int k0) {
#pragma unroll
            for (int i = 0; i < RPT; ++i)
              if (pend[i]) load_seg16(T + rowoff[i] + R0 + k0, nb[i]);
          };
          auto apply_pre = [&](int k0) {
#pragma unroll
            for (int i = 0; i < RPT; ++i)
              if (pend[i]) {
#pragma unroll
                for (int u = 0; u < 16; ++u)
#pragma unroll
                  for (int c = 0; c < LG; ++c) acc[i][c] = fms(acc[i][c], pre[i][u], Xs[k0 + u][c]);
              }
          };
          auto apply_nb = [&](int k0) {
#pragma unroll
            for (int i = 0; i < RPT; ++i)
              if (pend[i]) {
#pragma unroll
                for (int u = 0; u < 16; ++u)
#pragma unroll
                  for (int c = 0; c < LG; ++c) acc[i][c] = fms(acc[i][c], nb[i][u], Xs[k0 + u][c]);
              }
          };
          issue_nb(16);
          apply_pre(0);
          issue(pre, 32);
          apply_nb(16);
          issue_nb(48);
          apply_pre(32);
          apply_nb(48);
        }
      }
      // rest of the full-block segments, 16 columns at a time, every row's
      // loads issued together
      if (!PIPE && nr == B) {
#pragma unroll
        for (int i0 = 0; i0 < RPT; i0 += GR) {
          for (int k0 = PF; k0 < B; k0 += 16) {
            cx<P> lv[GR][16];
#pragma unroll
            for (int g = 0; g < GR; ++g) {
              const int r = row_of(i0 + g);
              if (r < n && (pass == 0 ? r >= R0 + B : r < R0)) load_seg16(T + rowoff[i0 + g] + R0 + k0, lv[g]);
            }
#pragma unroll
            for (int g = 0; g < GR; ++g) {
              const int r = row_of(i0 + g);
              const bool pending = r < n && (pass == 0 ? r >= R0 + B : r < R0);
              if (pending) {
#pragma unroll
                for (int u = 0; u < 16; ++u)
#pragma unroll
                  for (int c = 0; c < LG; ++c) acc[i0 + g][c] = fms(acc[i0 + g][c], lv[g][u], Xs[k0 + u][c]);
              }
            }
          }
        }
      }
      // (the next block's barrier after step 1 orders Xs reuse)
    }
    __syncthreads();
  }
  // acc now holds x for the owned rows: store to Y (FP64) and take maxima
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int r = row_of(i);
    if (r < n) {
      c128* y = Y + D.offY + (long long)r * D.N * L + (long long)j * L + c0;
#pragma unroll
      for (int c = 0; c < LG; ++c) {
        if (c < nc) {
          c128 nv = {double(acc[i][c].re), double(acc[i][c].im)};
          if (refine) nv = y[c] + nv;
          y[c] = nv;
          ymax[c] = nanmax(ymax[c], sqrt(norm2(nv)));
        }
      }
    }
  }
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int c = 0; c < LG; ++c) {
    double m = ymax[c];
    for (int o = 32; o >= 1; o >>= 1) m = nanmax(m, __shfl_xor(m, o, 64));
    if (lane == 0) cmax[wave][c] = m;
  }
  __syncthreads();
  if (tid < nc) {
    double m = 0.0;
    for (int w = 0; w < NT / 64; ++w) m = nanmax(m, cmax[w][tid]);
    atomicMax(&ir.ynorm[(long long)g * kNormStride + c0 + tid], (unsigned long long)__double_as_longlong(m));
  }
}

// ---------------------------------------------------------------------------

// Tile operations of k_trsm on the matrix cores.  A complex product runs as a
// real one: a row of the factor is 2K reals in memory order (re, im, re, im),
// and the right operand holds [xr xi; -xi xr] for every complex entry, so the
// A operand needs no rearrangement and an accumulator tile is 16 rows by 8
// complex columns (real column 2c + component).  A lane's 16-byte piece of its
// row (row l%16, piece l/16 of the 64 bytes) feeds consecutive products: the
// order of k is the same permutation on both sides.
template <typename P>
struct TriTile;
template <>
struct TriTile<float> {
  typedef float acc_t __attribute__((ext_vector_type(4)));
  typedef float4 seg_t;
  static constexpr int KL = 2;  // complex per piece
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
  static __device__ __forceinline__ acc_t mac(acc_t acc, seg_t a, seg_t b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, acc, 0, 0, 0);
  }
  // the first `left` complex of a piece
  static __device__ __forceinline__ seg_t head(seg_t a, int left) {
    return make_float4(left > 0 ? a.x : 0.f, left > 0 ? a.y : 0.f, left > 1 ? a.z : 0.f, left > 1 ? a.w : 0.f);
  }
  // the value of the lane beside (lane ^ 1)
  static __device__ __forceinline__ float other(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));
  }
};
template <>
struct TriTile<double> {
  typedef double acc_t __attribute__((ext_vector_type(4)));
  typedef double2 seg_t;
  static constexpr int KL = 1;
  static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
  static __device__ __forceinline__ acc_t mac(acc_t acc, seg_t a, seg_t b) {
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.y, acc, 0, 0, 0);
  }
  static __device__ __forceinline__ seg_t head(seg_t a, int left) {
    return make_double2(left > 0 ? a.x : 0.0, left > 0 ? a.y : 0.0);
  }
  static __device__ __forceinline__ double other(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), 0xB1, 0xF, 0xF, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), 0xB1, 0xF, 0xF, false));
  }
};

// Four loads of a row group (16 rows, 256 bytes of each; lane l of load m: row
// 4 (l/4 % 4) + m, piece l%4 of the 64 bytes l/16, so four lanes share a
// request) turned into operand pieces (piece m: row l%16, piece m of the 64
// bytes l/16): a 4 x 4 transposition within every four lanes.
template <typename S>
__device__ __forceinline__ void tri_turn(S (&v)[4]) {
  const bool o1 = threadIdx.x & 1, o2 = threadIdx.x & 2;
  union U {
    S s;
    int d[4];
  } u[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) u[m].s = v[m];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    int t[4];
#pragma unroll
    for (int m = 0; m < 4; m += 2) {
      const int x = u[m].d[c], y = u[m + 1].d[c];
      const int xo = __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);
      const int yo = __builtin_amdgcn_mov_dpp(y, 0xB1, 0xF, 0xF, true);
      t[m] = o1 ? yo : x;
      t[m + 1] = o1 ? y : xo;
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int xo = __builtin_amdgcn_mov_dpp(t[m], 0x4E, 0xF, 0xF, true);
      const int yo = __builtin_amdgcn_mov_dpp(t[m + 2], 0x4E, 0xF, 0xF, true);
      u[m].d[c] = o2 ? yo : t[m];
      u[m + 2].d[c] = o2 ? t[m + 2] : xo;
    }
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) v[m] = u[m].s;
}

// The solve on the matrix cores: one group per (matrix, 8 right-hand columns),
// right-looking over 64-row blocks like k_trsv, the accumulators of all rows
// in registers as 16-row tiles (tile t belongs to wave t mod NW).  Per block
// the owners of its four tiles publish their sums, multiply by the stored
// inverse of the diagonal block and publish the solution; then every wave
// subtracts (its pending tiles of the factor) x.  Tiles are streamed from
// global memory straight into the A operands, each 16-byte piece reloaded for
// the next tile (of the next block, past the last one) once it is used, so a
// tile per wave is in flight at all times, across the block's barriers too.
// 64 nodes of n = 1000, 16 columns, FP32: 0.29 ms (k_trsv: 0.41), the matrix
// cores busy for 0.115 of it, the block's own steps 0.05; with the factor
// resident in L2 0.24.  FP64, 32 nodes of n = 777: 0.34 ms (0.44).  The
// vector kernel read each row from one lane: 64 requests per load, where four
// lanes a row make 16.
template <typename P, int TPW, int NT>
__global__ __launch_bounds__(NT, 2) void k_trsm(const MatDesc* __restrict__ md, int nmat, int groups,
                                             const ProbDesc* __restrict__ pd, NodeArrays na,
                                             const cx<P>* __restrict__ Tb, const int* __restrict__ rows,
                                             const cx<P>* __restrict__ Dinv, const long long* __restrict__ dinv_off,
                                             const c128* __restrict__ R, c128* __restrict__ Y, int refine,
                                             const int* __restrict__ conv, IrState ir) {
  typedef TriTile<P> Op;
  typedef typename Op::acc_t acc_t;
  typedef typename Op::seg_t seg_t;
  constexpr int B = kSolveBlk, LG = kTrsmCols, NW = NT / 64, BT = B / 16;  // BT tiles per block
  // complex k per piece, per 64 bytes and per row group of four loads; groups
  constexpr int KL = Op::KL, KC = 4 * KL, KG = 4 * KC, NG = B / KG;
  // the column groups of one matrix run on one XCD and share its L2
  const int v = xcd_remap(blockIdx.x, gridDim.x, nmat * groups);
  if (v < 0) return;
  const int b = v / groups, grp = v - b * groups;
  const MatDesc d = md[b];
  const int g = d.node;
  if (conv != nullptr && conv[g]) return;
  const int p = na.prob[g], j = na.jnode[g];
  const ProbDesc& D = pd[p];
  const int n = d.n, ld = d.ld, L = D.L;
  const int c0 = grp * LG;
  const int nc = min(LG, L - c0);
  if (nc <= 0) return;
  const cx<P>* __restrict__ T = Tb + d.offT;
  const cx<P>* __restrict__ Di = Dinv + dinv_off[b];
  const int nblk = (n + B - 1) / B, ntile = (n + 15) / 16;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int jc = lane & 15, cc = jc >> 1, cf = jc & 1;  // this lane's real column: complex column, component
  const int lr = lane & 12, lk = KC * (lane >> 4) + KL * (lane & 3);  // its pieces when loading: first row, first k

  __shared__ __align__(16) int rat[NW * TPW * 16];  // physical rows (row 0 past n)
  __shared__ seg_t tb[NG * 4 * 64];                 // right operand: the block's right-hand sides
  __shared__ seg_t xb[NG * 4 * 64];                 // right operand: minus its solution
  __shared__ double cmax[NW][LG];

  for (int r = tid; r < NW * TPW * 16; r += NT) rat[r] = r < n ? rows[d.offRow + r] : 0;
  // the inverse of diagonal block q (pass 0: L's), as the wave's A operand
  // where it owns one of the block's tiles
  seg_t dreg[NG][4];
  auto load_inv = [&](int pass, int q) {
    const int i = w - BT * q % NW;
    if (q < 0 || q >= nblk || i < 0 || i >= BT) return;
    const cx<P>* src = Di + ((long long)q * 2 + pass) * B * B + (16 * i + lr) * B + lk;
#pragma unroll
    for (int h = 0; h < NG; ++h)
#pragma unroll
      for (int m = 0; m < 4; ++m) dreg[h][m] = *reinterpret_cast<const seg_t*>(src + m * B + KG * h);
  };
  constexpr int QS = NW / BT;  // a wave owns a tile of every QS-th block
  load_inv(0, w / BT);
  __syncthreads();
  // right-hand side P b in the owners' accumulators
  acc_t acc[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    int lo = lane;  // opaque (also below): what a tile needs is formed for that tile, or it spills
    asm volatile("" : "+v"(lo));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = (i * NW + w) * 16 + Op::row(lo, r);
      double bv = 0.0;
      if (row < n && cc < nc) {
        const int pr = rat[row];
        bv = refine ? reinterpret_cast<const double*>(R + D.offY + (long long)pr * D.N * L + (long long)j * L + c0)[jc]
                    : reinterpret_cast<const double*>(D.V + (long long)(c0 + cc) * n + pr)[cf];
      }
      acc[i][r] = P(bv);
    }
  }
  // four rows of a tile (rows 16 i + row(lane, r) of the block) into a right operand
  auto publish = [&](seg_t* dst, acc_t x, int i, P sign) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const P own = sign * x[r], oth = Op::other(own);
      const int k = 16 * i + Op::row(lane, r);
      P* o = reinterpret_cast<P*>(dst + (k / KG * 4 + k / KL % 4) * 64 + k / KC % 4 * 16 + jc) + 2 * (k % KL);
      o[0] = own;
      o[1] = cf ? oth : -oth;
    }
  };
  // a tile's four rows of this lane, at its first piece
  struct Ptr {
    const cx<P>* r[4];
  };
  auto seg = [&](int t, int R0, int lo) {
    const int4 pr = *reinterpret_cast<const int4*>(rat + 16 * t + (lo & 12));
    const cx<P>* s = T + R0 + lk;
    return Ptr{{s + (long long)pr.x * ld, s + (long long)pr.y * ld, s + (long long)pr.z * ld, s + (long long)pr.w * ld}};
  };
  // the wave's first pending tile of a block (ntile: none)
  auto first = [&](int pass, int q) {
    if (pass == 1) return w < BT * q ? w : ntile;
    const int lo = BT * (q + 1);
    return min(ntile, lo + ((w - lo) & (NW - 1)));
  };

  // row groups in flight: a tile (FP32) or half of one (FP64, twice the registers)
  constexpr int NB = 2;
  seg_t buf[NB][4];
  Ptr cur = {{T, T, T, T}};  // the tile whose first NB groups buf holds
  bool primed = false;   // it is the block's first pending tile
  for (int pass = 0; pass < 2; ++pass) {  // 0: L y = P b, 1: U x = y
    for (int qq = 0; qq < nblk; ++qq) {
      const int q = pass == 0 ? qq : nblk - 1 - qq;
      const int R0 = q * B, left = n - R0;
      const int tf = first(pass, q);
      if (!primed && tf < ntile && left >= B) {
        cur = seg(tf, R0, lane);
#pragma unroll
        for (int h = 0; h < NB; ++h)
#pragma unroll
          for (int m = 0; m < 4; ++m) buf[h][m] = *reinterpret_cast<const seg_t*>(cur.r[m] + KG * h);
      }
      primed = false;
      // the block's own tiles: this wave's, if it has one
      const int io = w - BT * q % NW;
      const bool own = io >= 0 && io < BT;
      if (own) {
        acc_t t = acc[0];
#pragma unroll
        for (int i = 1; i < TPW; ++i)
          if (i == q / QS) t = acc[i];
#pragma unroll
        for (int r = 0; r < 4; ++r) t[r] = R0 + 16 * io + Op::row(lane, r) < n ? t[r] : P(0);
        publish(tb, t, io, P(1));
#pragma unroll
        for (int h = 0; h < NG; ++h) tri_turn(dreg[h]);
      }
      __syncthreads();
      if (own) {  // x_q = Dinv_q t (the inverse is identity-padded past n)
        acc_t x0 = {P(0), P(0), P(0), P(0)}, x1 = x0, x2 = x0, x3 = x0;
#pragma unroll
        for (int h = 0; h < NG; ++h) {
          const seg_t* o = tb + 256 * h + lane;
          x0 = Op::mac(x0, dreg[h][0], o[0]);
          x1 = Op::mac(x1, dreg[h][1], o[64]);
          x2 = Op::mac(x2, dreg[h][2], o[128]);
          x3 = Op::mac(x3, dreg[h][3], o[192]);
        }
        x0 = (x0 + x1) + (x2 + x3);
#pragma unroll
        for (int i = 0; i < TPW; ++i)
          if (i == q / QS) acc[i] = x0;
        publish(xb, x0, io, P(-1));
        // the inverse of the wave's next block, a block's updates ahead
        if (pass == 1) load_inv(1, q - QS);
        else if (q + QS < nblk) load_inv(0, q + QS);
        else {  // its last block of the forward sweep is its first of the backward one
          load_inv(1, q);
        }
      }
      __syncthreads();
      if (tf >= ntile) continue;
      if (left >= B) {
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
          const int t = i * NW + w;
          if (pass == 0 ? t >= BT * (q + 1) && t < ntile : t < BT * q) {
            int tn = t + NW, Rn = R0;
            if (tn >= (pass == 0 ? ntile : BT * q)) {  // the next block's first (none: this one again)
              const int nq = pass == 0 ? q + 1 : q - 1;
              tn = first(pass, nq);
              primed = tn < ntile;
              if (primed) Rn = nq * B;
              else tn = t;
            }
            int lo = lane;
            asm volatile("" : "+v"(lo));
            const Ptr s = seg(tn, Rn, lo);
            // group h + 1 turns, and its registers load again, while group h multiplies
            // (the barriers keep that order: the loads else wait for the end of the tile)
            seg_t a[4];
            acc_t odd = {P(0), P(0), P(0), P(0)};  // a second chain of products
            auto ready = [&](int h) {
#pragma unroll
              for (int m = 0; m < 4; ++m) a[m] = buf[h % NB][m];
              tri_turn(a);
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int m = 0; m < 4; ++m)
                buf[h % NB][m] = *reinterpret_cast<const seg_t*>(h + NB < NG ? cur.r[m] + KG * (h + NB)
                                                                              : s.r[m] + KG * (h + NB - NG));
            };
            ready(0);
#pragma unroll
            for (int h = 0; h < NG; ++h) {
              seg_t am[4];
#pragma unroll
              for (int m = 0; m < 4; ++m) am[m] = a[m];
              __builtin_amdgcn_sched_barrier(0);
              if (h + 1 < NG) ready(h + 1);
#pragma unroll
              for (int m = 0; m < 4; m += 2) {
                acc[i] = Op::mac(acc[i], am[m], xb[256 * h + 64 * m + lo]);
                odd = Op::mac(odd, am[m + 1], xb[256 * h + 64 * (m + 1) + lo]);
              }
            }
            acc[i] += odd;
            cur = s;
          }
        }
      } else {
        // the ragged last block, once (backward): pieces past column n are read
        // from the row's last one and cleared
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
          const int t = i * NW + w;
          if (t < BT * q) {
            int lo = lane;
            asm volatile("" : "+v"(lo));
            const int k0 = KC * (lo >> 4) + KL * (lo & 3), kl = (left - 1) / KL * KL - k0;
            const Ptr s = seg(t, R0, lo);
#pragma unroll
            for (int h = 0; h < NG; ++h) {
              seg_t a[4];
#pragma unroll
              for (int m = 0; m < 4; ++m)
                a[m] = Op::head(*reinterpret_cast<const seg_t*>(s.r[m] + min(KG * h, kl)), left - k0 - KG * h);
              tri_turn(a);
#pragma unroll
              for (int m = 0; m < 4; ++m) acc[i] = Op::mac(acc[i], a[m], xb[256 * h + 64 * m + lo]);
            }
          }
        }
      }
    }
  }
  // acc now holds x for the owned rows: store to Y (FP64) and take maxima
  double ymax = 0.0;
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    int lo = lane;
    asm volatile("" : "+v"(lo));
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = (i * NW + w) * 16 + Op::row(lo, r);
      double nv = double(acc[i][r]);
      const bool in = row < n && cc < nc;
      if (in) {
        double* y = reinterpret_cast<double*>(Y + D.offY + (long long)row * D.N * L + (long long)j * L + c0) + jc;
        if (refine) nv = *y + nv;
        *y = nv;
      }
      const double oth = TriTile<double>::other(nv);
      if (in) ymax = nanmax(ymax, sqrt(nv * nv + oth * oth));
    }
  }
  ymax = nanmax(ymax, __shfl_xor(ymax, 16, 64));
  ymax = nanmax(ymax, __shfl_xor(ymax, 32, 64));
  if (lane < 16 && cf == 0) cmax[w][cc] = ymax;
  __syncthreads();
  if (tid < nc) {
    double m = 0.0;
    for (int u = 0; u < NW; ++u) m = nanmax(m, cmax[u][tid]);
    atomicMax(&ir.ynorm[(long long)g * kNormStride + c0 + tid], (unsigned long long)__double_as_longlong(m));
  }
}

template <typename P, int TPW, int NT>
static void launch_trsm_class(const SolvePlan& sp, int b0, int cnt, const ProbDesc* pd, const MatDesc* md,
                              const NodeArrays& na, const cx<P>* T, const int* rows, const cx<P>* Dinv,
                              const long long* dinv_off, const c128* R, c128* Y, int rf, const int* conv, IrState ir,
                              hipStream_t st) {
  if (cnt <= 0) return;
  const int groups = ceil_div(sp.L, kTrsmCols);
  hipLaunchKernelGGL((k_trsm<P, TPW, NT>), dim3(xcd_grid(cnt * groups)), dim3(NT), 0, st, md + b0, cnt, groups, pd, na,
                     T, rows, Dinv, dinv_off + b0, R, Y, rf, conv, ir);
}

template <typename P, int LG, int RPT, int NT>
static void launch_trsv_class(const SolvePlan& sp, int b0, int cnt, const ProbDesc* pd, const MatDesc* md,
                              const NodeArrays& na, const cx<P>* T, const int* rows, const cx<P>* Dinv,
                              const long long* dinv_off, const c128* R, c128* Y, int rf, const int* conv, IrState ir,
                              hipStream_t st) {
  if (cnt <= 0) return;
  hipLaunchKernelGGL((k_trsv<P, LG, RPT, NT>), dim3(xcd_grid(cnt * sp.groups)), dim3(NT), 0, st, md + b0, cnt,
                     sp.groups, pd, na, T, rows, Dinv, dinv_off + b0, R, Y, rf, conv, ir);
}

// One launch per size class of the (size-sorted) matrices: more than 512
// rows (512 threads, sp.rpt rows each), 257..512 rows and up to 256 rows
// (256 threads, two and one rows each).
template <typename P, int LG>
static void launch_trsv(const SolvePlan& sp, const ProbDesc* pd, const MatDesc* md, const NodeArrays& na,
                        const cx<P>* T, const int* rows, const cx<P>* Dinv, const long long* dinv_off, const c128* R,
                        c128* Y, int rf, const int* conv, IrState ir, hipStream_t st) {
  // the first nblk matrices took the blocked solve (complex FP32 only)
  const int b0 = sizeof(P) == 4 ? sp.nblk : 0;
  const int nb = sp.nbig - b0, nm = sp.nmid, ns = sp.nmat - sp.nbig - sp.nmid;
  // many large matrices (several rounds of groups): 256-thread groups with
  // twice the rows each, two per CU, so one group's barrier waits are
  // covered by the other's work
  // (complex FP32 with at most 8 columns per group: two such groups fit a CU's registers)
  constexpr bool kPaired = sizeof(P) == 4 && LG <= 8;
  if (kPaired && sp.rpt <= 2 && nb > 0 && sp.paired == 1) {
    if constexpr (kPaired)
      launch_trsv_class<P, LG, 4, kTrsvThreadsSmall>(sp, b0, nb, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv,
                                                     ir, st);
  } else switch (sp.rpt) {
    case 1:
    case 2: launch_trsv_class<P, LG, 2, kTrsvThreads>(sp, b0, nb, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir, st); break;
    case 4: launch_trsv_class<P, LG, 4, kTrsvThreads>(sp, b0, nb, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir, st); break;
    default: launch_trsv_class<P, LG, 8, kTrsvThreads>(sp, b0, nb, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir, st); break;
  }
  launch_trsv_class<P, LG, 2, kTrsvThreadsSmall>(sp, sp.nbig, nm, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir,
                                                 st);
  launch_trsv_class<P, LG, 1, kTrsvThreadsSmall>(sp, sp.nbig + nm, ns, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf,
                                                 conv, ir, st);
}

template <typename P>
static void launch_trsv_lg(const SolvePlan& sp, const ProbDesc* pd, const MatDesc* md, const NodeArrays& na,
                           const cx<P>* T, const int* rows, const cx<P>* Dinv, const long long* dinv_off, const c128* R,
                           c128* Y, int rf, const int* conv, IrState ir, hipStream_t st) {
  switch (sp.lg) {
    case 4: launch_trsv<P, 4>(sp, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir, st); break;
    case 8: launch_trsv<P, 8>(sp, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir, st); break;
    default: launch_trsv<P, 16>(sp, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir, st); break;
  }
}

// The size classes of k_trsm: 512 threads above 512 rows, four or eight waves
// below (an FP64 wave holds at most four tiles beside its operands there).
template <typename P>
static void launch_trsm(const SolvePlan& sp, const ProbDesc* pd, const MatDesc* md, const NodeArrays& na,
                        const cx<P>* T, const int* rows, const cx<P>* Dinv, const long long* dinv_off, const c128* R,
                        c128* Y, int rf, const int* conv, IrState ir, hipStream_t st) {
  const int b0 = sizeof(P) == 4 ? sp.nblk : sp.nhuge, nm = sp.nmid;
  const int nb = sp.nbig - b0, ns = sp.nmat - sp.nbig - sp.nmid;
#define NEP_TRSM(TPW, NT, FIRST, CNT) \
  launch_trsm_class<P, TPW, NT>(sp, FIRST, CNT, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir, st)
  if constexpr (sizeof(P) == 4) {
    if (sp.rpt <= 2) NEP_TRSM(8, kTrsvThreads, b0, nb);
    else if (sp.rpt <= 4) NEP_TRSM(16, kTrsvThreads, b0, nb);
    else NEP_TRSM(32, kTrsvThreads, b0, nb);
    NEP_TRSM(4, kTrsvThreads, sp.nbig, nm);
  } else {
    if (b0 > 0) {  // above 1024 rows a wave's FP64 tiles do not fit its registers
      SolvePlan h = sp;
      h.nmat = h.nbig = b0;
      h.nmid = 0;
      launch_trsv_lg<P>(h, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir, st);
    }
    NEP_TRSM(8, kTrsvThreads, b0, nb);
    NEP_TRSM(4, kTrsvThreads, sp.nbig, nm);
  }
  NEP_TRSM(4, kTrsvThreadsSmall, sp.nbig + nm, ns);
#undef NEP_TRSM
}

template <typename P>
hipError_t solve_run(const SolvePlan& sp, const ProbDesc* pd, const MatDesc* md, const NodeArrays& na,
                     const cx<P>* T, const int* rows, const cx<P>* Dinv, const long long* dinv_off,
                     const c128* R, c128* Y, bool refine, const int* conv, IrState ir, hipStream_t st) {
  if (sp.nmat == 0) return hipSuccess;
  const int rf = refine ? 1 : 0;
  if constexpr (sizeof(P) == 4) {
    if (sp.nblk > 0) {
      const hipError_t e = solve_blocked(sp, pd, md, na, T, rows, Dinv, dinv_off, R, Y, refine, conv, ir, st);
      if (e != hipSuccess) return e;
      if (sp.nblk == sp.nmat) return hipSuccess;
    }
  }
  if (sp.paired < 0)
    launch_trsm<P>(sp, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir, st);
  else
    launch_trsv_lg<P>(sp, pd, md, na, T, rows, Dinv, dinv_off, R, Y, rf, conv, ir, st);
  return hipGetLastError();
}

template hipError_t solve_run<float>(const SolvePlan&, const ProbDesc*, const MatDesc*, const NodeArrays&, const c64*,
                                     const int*, const c64*, const long long*, const c128*, c128*, bool,
                                     const int*, IrState, hipStream_t);
template hipError_t solve_run<double>(const SolvePlan&, const ProbDesc*, const MatDesc*, const NodeArrays&,
                                      const c128*, const int*, const c128*, const long long*, const c128*,
                                      c128*, bool, const int*, IrState, hipStream_t);

// Column-group size: enough groups to occupy the device when there are few
// matrices, bounded by L (the group is an unrolled register tile).
static int pick_lg(int nmat, int L) {
  // Each column group re-reads the node's factor (from the XCD's L2), so
  // prefer few groups per node; split only when there are too few nodes to
  // occupy the device.
  int lg = 16;
  while (lg > 4 && lg >= 2 * L) lg >>= 1;
  while (lg > 4 && (long long)nmat * ceil_div(L, lg) < 256) lg >>= 1;
  return lg;
}

void SolvePlan_build(SolvePlan& sp, std::vector<int>& /*buf*/, const std::vector<MatDesc>& sorted, int L, int prec,
                     std::vector<long long>& dinv_off, long long& dinv_elems) {
  sp.nmat = (int)sorted.size();
  const int nmax = sorted.empty() ? 0 : sorted[0].n;
  sp.rpt = nmax <= 512 ? 1 : nmax <= 1024 ? 2 : nmax <= 2048 ? 4 : 8;  // rows per thread of the 512-thread class
  sp.nbig = sp.nmid = sp.nhuge = 0;
  for (const auto& m : sorted) {
    if (m.n > 1024) ++sp.nhuge;
    if (m.n > 2 * kTrsvThreadsSmall) ++sp.nbig;
    else if (m.n > kTrsvThreadsSmall) ++sp.nmid;
  }
  // complex FP32 with an even number (at most 64) of right-hand sides: the
  // matrices of at least kSolveBlockedMinN rows take the blocked solve
  sp.nblk = 0;
  sp.L = L;
  if (prec != NEP_PREC_FP64 && L % 2 == 0 && L <= 64)
    while (sp.nblk < sp.nmat && sorted[sp.nblk].n >= kSolveBlockedMinN) ++sp.nblk;
  sp.npad = sp.nblk > 0 ? ceil_div(sorted[0].n, kSolveBlk) * kSolveBlk : 0;
  sp.nbk = 256;
  sp.W = nullptr;
  sp.lg = pick_lg(sp.nmat - sp.nblk, L);
  while (sp.lg > 4 && !solve_lg_fits(sp, sp.lg, L, prec)) sp.lg >>= 1;
  sp.groups = ceil_div(L, sp.lg);
  sp.paired = -1;
  dinv_off.clear();
  long long off = 0;
  for (const auto& m : sorted) {
    const int nb = ceil_div(m.n, kSolveBlk);
    dinv_off.push_back(off);
    off += (long long)nb * 2 * kSolveBlk * kSolveBlk;
  }
  dinv_elems = off;
}

bool solve_lg_fits(const SolvePlan& sp, int lg, int L, int prec) {
  if (lg != 4 && lg != 8 && lg != 16) return false;
  if (lg == 4) return true;  // the narrowest group always fits
  // accumulators live in registers: at most 32 complex FP32 (8 complex FP64)
  // values per thread
  const int cap = prec == NEP_PREC_FP64 ? 8 : 32;
  return lg < 2 * L && sp.rpt * lg <= cap;
}

void solve_set_lg(SolvePlan& sp, int lg, int L) {
  sp.lg = lg;
  sp.groups = ceil_div(L, lg);
}

hipError_t solve_configure() { return hipSuccess; }

}  // namespace nep
