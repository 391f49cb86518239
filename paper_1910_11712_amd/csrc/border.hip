// Operators whose terms are diagonal, real banded (half-width at most 32) or
// real low-rank (kept as G H^T since creation): complex-FP32 factors of T(z_j)
// as a bordered block-tridiagonal matrix, in place of a dense LU.
//
// T y = v is written over 32-row blocks with s_i = H_i^T y as further unknowns:
//
//     D y_I + E y_S + (f G)_I s = v_I      interior blocks, nch chunks
//     F y_I + T_SS y_S + (f G)_S s = v_S   nch - 1 separator blocks between them
//     H_I^T y_I + H_S^T y_S - s = 0        one row per column of the G's
//
// The chunks of D are block tridiagonal and independent: k_bd_lu eliminates
// each with partial pivoting inside a 64-row window, k_bd_solve applies its
// inverse to [E, f G] (kept as W) and later to every right-hand side, both on
// the FP32 matrix cores.  What remains is the border's Schur complement (size
// b = 32 (nch - 1) + r), factored by the batched dense LU.  At n = 4096 with
// half-width 32 and rank 128 that is 0.3 GFLOP per node in place of 183.
//
// Pivots are sought inside a chunk's window and inside the border only, so
// unlike the dense LU's the factors are not backward stable for every T: the
// FP64 refinement decides.  Its residual is that of T itself, and a node that
// it cannot bring to the tolerance (a chunk near singular where T is not)
// hands its problem over to dense factors (MomentsPlan::go_dense), for the
// passes and counts that follow too: the pivots here say nothing of det T then.
#include <algorithm>

#include "engine.hpp"

namespace nep {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int B = kBdBlk;       // 32
constexpr int B2 = B * B;

// first block of chunk c (c = nch: one past the last, plus one)
__host__ __device__ __forceinline__ int bd_start(const BdProb& q, int c) { return c * (q.nb + 1) / q.nch; }

// T(z)[gr][gc] without the low-rank terms, FP64 sums rounded once; identity past n
__device__ __forceinline__ c64 bd_elem(const ProbDesc& D, const c128* __restrict__ f, int w, int gr, int gc) {
  const int n = D.n;
  if (gr >= n || gc >= n) return c64{gr == gc ? 1.f : 0.f, 0.f};
  const int d = gr - gc;
  if (d > w || d < -w) return c64{0.f, 0.f};
  double sr = 0.0, si = 0.0;
  for (int i = 0; i < D.ell; ++i) {
    if (D.a_lr[i] > 0) continue;
    const c128 fi = f[i];
    if (D.a_is_diag[i]) {
      if (d == 0) {
        const c128 a = D.Adiag[i][gr];
        sr += fi.re * a.re - fi.im * a.im;
        si += fi.re * a.im + fi.im * a.re;
      }
    } else {
      const double a = reinterpret_cast<const double*>(D.A[i])[(long long)gr * n + gc];
      sr += fi.re * a;
      si += fi.im * a;
    }
  }
  return c64{float(sr), float(si)};
}

// the f_i of column h of the concatenated low-rank terms
__device__ __forceinline__ c128 bd_lowrank_f(const ProbDesc& D, const c128* __restrict__ f, int h) {
  for (int i = 0; i < D.ell; ++i) {
    if (D.a_lr[i] == 0) continue;
    if (h < D.a_lr[i]) return f[i];
    h -= D.a_lr[i];
  }
  return c128{0.0, 0.0};
}
// f times an entry of its G
__device__ __forceinline__ c64 bd_lowrank(c128 f, float g) { return c64{float(f.re * g), float(f.im * g)}; }

typedef float floatx4 __attribute__((ext_vector_type(4)));

// An 8 x 16 complex tile on v_mfma_f32_16x16x4f32 and the real 2x2 embedding:
// lane l feeds A row l%16 (complex row l%16/2, component l%2) and k-slot l/16
// (half l/32 of the complex k, component l/16%2), B column l%16; accumulator
// register r is complex row 2 (l/16) + r/2, component r%2, column l%16.
struct BdTile {
  int arow, acomp, crow, col, ku, kh;
  float asign;
  __device__ __forceinline__ BdTile(int rb, int cb) {
    const int l = threadIdx.x & 63, at = l & 1;
    ku = (l >> 4) & 1;
    kh = l >> 5;
    arow = rb + ((l & 15) >> 1);
    acomp = at ^ ku;
    crow = rb + 2 * (l >> 4);
    col = cb + (l & 15);
    asign = (at == 0 && ku == 1) ? -1.f : 1.f;
  }
  // acc += sign A B over K complex k: A row-major in LDS, b(k) this lane's
  // column of B's row k
  template <int K, int LDA, typename F>
  __device__ __forceinline__ floatx4 mul(const c64 (*A)[LDA], float sign, floatx4 acc, F&& b) const {
    const float* a = reinterpret_cast<const float*>(&A[arow][kh * (K / 2)]) + acomp;
    const float sg = sign * asign;
#pragma unroll
    for (int x = 0; x < K / 2; ++x)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(sg * a[2 * x], ku ? b(kh * (K / 2) + x).im : b(kh * (K / 2) + x).re,
                                                 acc, 0, 0, 0);
    return acc;
  }
};

// One complex k of a 16 x 32 complex product on the 2x2 real embedding: lane l
// feeds A row (l%32)/2, component l%2, with the sign of the embedding, and B
// column l%32, component l/32; accumulator register r holds complex row
// 4(r/4) + 2(l/32) + (r%4)/2, component r%2, column l%32.
struct BdLane {
  int arow, acomp, bcol, bcomp;
  float asign;
  __device__ __forceinline__ BdLane() {
    const int l = threadIdx.x & 63, at = l & 1, au = l >> 5;
    arow = (l & 31) >> 1;
    acomp = at ^ au;
    asign = (at == 0 && au == 1) ? -1.f : 1.f;
    bcol = l & 31;
    bcomp = au;
  }
  __device__ __forceinline__ int crow(int r) const { return 4 * (r >> 2) + 2 * bcomp + ((r & 3) >> 1); }
};
__device__ __forceinline__ float bd_comp(c64 x, int c) { return c ? x.im : x.re; }
__device__ __forceinline__ floatx16 bd_mfma(float a, float b, floatx16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ floatx16 bd_zero() {
  floatx16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

__device__ __forceinline__ float bd_readlane(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// ---------------------------------------------------------------------------
// Chunk factorization: one group of eight waves per (node, chunk), the 64 x 96
// window of the current block in LDS.  Per block: wave 0 factors the 64 x 32
// panel with one row per lane in registers (pivot rows stay in their lanes and
// are broadcast by readlane, no exchange), while the other waves assemble the
// rows that enter next; L11 and U11 are inverted (16 x 16 diagonal blocks, one
// column per lane, four waves; then their off-diagonal blocks as products);
// and all waves form U12 = L11^-1 A12 and A22 - L21 U12 on the matrix cores.
// Bound by the chain of panels (12 of 20 us per block); the chunks are what
// cuts it.  64 nodes of n = 4096: 0.63 ms (four waves, with 32-step inverses:
// 1.03).  Per block the store holds L11^-1, L21, U11^-1 and U12's two 32 x 32
// blocks.
// ---------------------------------------------------------------------------
constexpr int kBdLuThreads = 512;

__global__ __launch_bounds__(kBdLuThreads) void k_bd_lu(const BdProb* __restrict__ bp, const int* __restrict__ prefix,
                                                        int cnt, const ProbDesc* __restrict__ pd, NodeArrays na,
                                                        c64* __restrict__ blocks, unsigned char* __restrict__ perms,
                                                        c64* __restrict__ pivots, int* __restrict__ info) {
  const int v = blockIdx.x;
  const int s = find_slot(prefix, cnt, v);
  const BdProb& q = bp[s];
  const ProbDesc& D = pd[q.prob];
  const int j = (v - prefix[s]) / q.nch, c = (v - prefix[s]) - j * q.nch;
  const int g = D.node0 + j, w = q.w;
  const int st = bd_start(q, c), len = bd_start(q, c + 1) - 1 - st;
  const c128* __restrict__ f = na.fz + (long long)g * kMaxTerms;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (!D.active) return;  // (its problem is factored densely now; also below)
  if (c == 0 && tid == 0) info[g] = D.n;  // a zero pivot here is left to the refinement

  constexpr int H = B / 2;
  __shared__ c64 Wn[2 * B][3 * B + 1];  // window: rows of the current block, then of the next
  __shared__ c64 Nx[B][3 * B + 1];      // rows entering next
  __shared__ c64 LU[2 * B][B + 1];      // panel in pivot order
  __shared__ c64 Li[B][B + 1], Ui[B][B + 1];
  __shared__ c64 U12[B][2 * B + 1];     // (its first rows hold the inverses' products before)
  __shared__ int src[2 * B];

  c64* __restrict__ bout = blocks + q.offB + ((long long)j * q.nb + st) * 5 * B2;
  unsigned char* __restrict__ pout = perms + q.offPerm + ((long long)j * q.nb + st) * 2 * B;
  c64* __restrict__ vout = pivots + q.offPiv + ((long long)j * q.nb + st) * B;

  // rows of block kb (relative to the chunk), window columns 0..95 from block cb0 on
  auto row_elem = [&](int kb, int i, int cb0, int col) {
    const int cb = cb0 + col / B;
    if (kb >= len || cb >= len) return c64{0.f, 0.f};
    return bd_elem(D, f, w, (st + kb) * B + i, (st + cb) * B + (col & (B - 1)));
  };
  for (int e = tid; e < 2 * B * 3 * B; e += kBdLuThreads) {
    const int i = e / (3 * B), col = e - i * 3 * B;
    Wn[i][col] = row_elem(i / B, i & (B - 1), 0, col);
  }
  __syncthreads();
  const BdTile t0((wave & 3) * 8, (wave >> 2) * B), t1((wave & 3) * 8, (wave >> 2) * B + 16);
  const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < len; ++k) {
    const bool more = k + 1 < len;
    if (wave == 0) {
      c64 a[B];
#pragma unroll
      for (int x = 0; x < B; ++x) a[x] = c64{Wn[lane][x].re, Wn[lane][x].im};
      bool used = lane >= B && !more;
      int pos = -1;
      float dre = 0.f, dim = 0.f;  // lane x keeps pivot x
#pragma unroll
      for (int x = 0; x < B; ++x) {
        const unsigned key = used ? 0u : __float_as_uint(fabsf(a[x].re) + fabsf(a[x].im)) + 1u;
        const unsigned best = wave_max_u32(key);
        const int pl = __ffsll((unsigned long long)__ballot(key == best)) - 1;  // lowest row on ties
        const c64 piv = {bd_readlane(a[x].re, pl), bd_readlane(a[x].im, pl)};
        if (lane == x) {
          dre = piv.re;
          dim = piv.im;
        }
        const c64 inv = recip_f32(piv);
        if (lane == pl) {
          used = true;
          pos = x;
        }
        const c64 l = a[x] * inv;
        const c64 lm = csel(!used, l, c64{0.f, 0.f});
        a[x] = csel(!used, l, a[x]);
#pragma unroll
        for (int y = 0; y < B; ++y)
          if (y > x) a[y] = fms(a[y], lm, c64{bd_readlane(a[y].re, pl), bd_readlane(a[y].im, pl)});
      }
      // the rows left over keep their order
      const unsigned long long rest = __ballot(pos < 0);
      if (pos < 0) pos = B + __popcll(rest & ((1ull << lane) - 1ull));
      src[pos] = lane;
#pragma unroll
      for (int x = 0; x < B; ++x) {
        LU[pos][x].re = a[x].re;
        LU[pos][x].im = a[x].im;
      }
      pout[(long long)k * 2 * B + pos] = (unsigned char)lane;
      if (lane < B) vout[(long long)k * B + lane] = c64{dre, dim};
    } else if (more) {
      // the entering rows (block k + 2, columns from block k + 1 on), term by
      // term, every entry's load of a term in flight together
      constexpr int ET = kBdLuThreads - 64, EU = (B * 3 * B + ET - 1) / ET;
      double sr[EU], si[EU];
      int off[EU];  // entry's offset in a dense term, -1: outside the band or the chunk
#pragma unroll
      for (int u = 0; u < EU; ++u) {
        const int e = tid - 64 + ET * u, i = e / (3 * B), col = e - i * 3 * B;
        const int kb = k + 2, cb = k + 1 + col / B;
        const int gr = (st + kb) * B + i, gc = (st + cb) * B + (col & (B - 1)), d = gr - gc;
        const bool blk = e < B * 3 * B && kb < len && cb < len, in = blk && gr < D.n && gc < D.n;
        off[u] = in && d <= w && d >= -w ? gr * D.n + gc : -1;
        sr[u] = blk && !in && d == 0 ? 1.0 : 0.0;  // identity past n
        si[u] = 0.0;
      }
      for (int t = 0; t < D.ell; ++t) {
        if (D.a_lr[t] > 0) continue;
        const c128 ft = f[t];
        if (D.a_is_diag[t]) {
#pragma unroll
          for (int u = 0; u < EU; ++u) {
            const int e = tid - 64 + ET * u, i = e / (3 * B), col = e - i * 3 * B;
            if (col == B + i && off[u] >= 0) {
              const c128 a = D.Adiag[t][(st + k + 2) * B + i];
              sr[u] += ft.re * a.re - ft.im * a.im;
              si[u] += ft.re * a.im + ft.im * a.re;
            }
          }
          continue;
        }
        const double* __restrict__ A = reinterpret_cast<const double*>(D.A[t]);
        double av[EU];
#pragma unroll
        for (int u = 0; u < EU; ++u) av[u] = A[max(off[u], 0)];
#pragma unroll
        for (int u = 0; u < EU; ++u) {
          const double a = off[u] >= 0 ? av[u] : 0.0;
          sr[u] += ft.re * a;
          si[u] += ft.im * a;
        }
      }
#pragma unroll
      for (int u = 0; u < EU; ++u) {
        const int e = tid - 64 + ET * u, i = e / (3 * B), col = e - i * 3 * B;
        if (e < B * 3 * B) Nx[i][col] = c64{float(sr[u]), float(si[u])};
      }
    }
    __syncthreads();
    // 16 x 16 diagonal blocks: waves 0, 1 of L11^-1, 2, 3 of U11^-1, column
    // `lane`; each entry found updates the ones after it (independent sums)
    if (wave < 4 && lane < H) {
      const int o = (wave & 1) * H;
      c64 x[H];
#pragma unroll
      for (int i = 0; i < H; ++i) x[i] = c64{i == lane ? 1.f : 0.f, 0.f};
      if (wave < 2) {
#pragma unroll
        for (int i = 0; i < H; ++i) {
#pragma unroll
          for (int m = i + 1; m < H; ++m) x[m] = fms(x[m], LU[o + m][o + i], x[i]);
          Li[o + i][o + lane] = x[i];
        }
      } else {
#pragma unroll
        for (int i = H - 1; i >= 0; --i) {
          x[i] = x[i] * recip_f32(LU[o + i][o + i]);
#pragma unroll
          for (int m = 0; m < i; ++m) x[m] = fms(x[m], LU[o + m][o + i], x[i]);
          Ui[o + i][o + lane] = x[i];
        }
      }
    } else if (wave >= 4) {  // the blocks that stay zero
      for (int e = tid - 256; e < H * H; e += 256) {
        Li[e / H][H + e % H] = c64{0.f, 0.f};
        Ui[H + e / H][e % H] = c64{0.f, 0.f};
      }
    }
    __syncthreads();
    // L: -C^-1 (B A^-1) below the diagonal; U: -A^-1 (B C^-1) above it
    if (wave < 4) {
      const bool up = wave >= 2;
      const BdTile ti((wave & 1) * 8, 0);
      floatx4 acc;
      if (up)
        acc = ti.mul<H>(reinterpret_cast<const c64(*)[B + 1]>(&LU[0][H]), 1.f, zero,
                        [&](int x) { return Ui[H + x][H + ti.col]; });
      else
        acc = ti.mul<H>(reinterpret_cast<const c64(*)[B + 1]>(&LU[H][0]), 1.f, zero, [&](int x) { return Li[x][ti.col]; });
      U12[ti.crow][(up ? H : 0) + ti.col] = c64{acc[0], acc[1]};
      U12[ti.crow + 1][(up ? H : 0) + ti.col] = c64{acc[2], acc[3]};
    }
    __syncthreads();
    if (wave < 4) {
      const bool up = wave >= 2;
      const BdTile ti((wave & 1) * 8, 0);
      floatx4 acc;
      if (up) {
        acc = ti.mul<H>(reinterpret_cast<const c64(*)[B + 1]>(&Ui[0][0]), -1.f, zero,
                        [&](int x) { return U12[x][H + ti.col]; });
        Ui[ti.crow][H + ti.col] = c64{acc[0], acc[1]};
        Ui[ti.crow + 1][H + ti.col] = c64{acc[2], acc[3]};
      } else {
        acc = ti.mul<H>(reinterpret_cast<const c64(*)[B + 1]>(&Li[H][H]), -1.f, zero,
                        [&](int x) { return U12[x][ti.col]; });
        Li[H + ti.crow][ti.col] = c64{acc[0], acc[1]};
        Li[H + ti.crow + 1][ti.col] = c64{acc[2], acc[3]};
      }
    }
    __syncthreads();
    c64* __restrict__ bk = bout + (long long)k * 5 * B2;
    for (int e = tid; e < B2; e += kBdLuThreads) {
      const int i = e / B, m = e & (B - 1);
      bk[e] = Li[i][m];
      bk[B2 + e] = LU[B + i][m];
      bk[2 * B2 + e] = Ui[i][m];
    }
    if (!more) break;
    // U12 = L11^-1 A12 (the window's pivot rows, columns 32..95): two 8 x 16 tiles per wave
    floatx4 u0 = t0.mul<B>(Li, 1.f, zero, [&](int x) { return Wn[src[x]][B + t0.col]; });
    floatx4 u1 = t1.mul<B>(Li, 1.f, zero, [&](int x) { return Wn[src[x]][B + t1.col]; });
    // the rows left over, before any wave writes the window
    const c64 x00 = Wn[src[B + t0.crow]][B + t0.col], x01 = Wn[src[B + t0.crow + 1]][B + t0.col];
    const c64 x10 = Wn[src[B + t1.crow]][B + t1.col], x11 = Wn[src[B + t1.crow + 1]][B + t1.col];
    auto put = [&](const BdTile& t, floatx4 u) {
      U12[t.crow][t.col] = c64{u[0], u[1]};
      U12[t.crow + 1][t.col] = c64{u[2], u[3]};
      c64* bu = bk + (3 + (wave >> 2)) * B2 + t.crow * B + (t.col & (B - 1));
      bu[0] = c64{u[0], u[1]};
      bu[B] = c64{u[2], u[3]};
    };
    put(t0, u0);
    put(t1, u1);
    __syncthreads();
    // A22 - L21 U12
    const auto& L21 = *reinterpret_cast<const c64(*)[B][B + 1]>(&LU[B]);
    u0 = t0.mul<B>(L21, -1.f, floatx4{x00.re, x00.im, x01.re, x01.im}, [&](int x) { return U12[x][t0.col]; });
    u1 = t1.mul<B>(L21, -1.f, floatx4{x10.re, x10.im, x11.re, x11.im}, [&](int x) { return U12[x][t1.col]; });
    // the next window: the updated rows (columns shifted by a block), then the assembled ones
    Wn[t0.crow][t0.col] = c64{u0[0], u0[1]};
    Wn[t0.crow + 1][t0.col] = c64{u0[2], u0[3]};
    Wn[t1.crow][t1.col] = c64{u1[0], u1[1]};
    Wn[t1.crow + 1][t1.col] = c64{u1[2], u1[3]};
    for (int e = tid; e < B * 3 * B; e += kBdLuThreads) {
      const int i = e / (3 * B), col = e - i * 3 * B;
      Wn[B + i][col] = Nx[i][col];
      if (col >= 2 * B) Wn[i][col] = c64{0.f, 0.f};
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Chunk solve: X = D_c^-1 (32 columns), one group of eight waves per (node,
// chunk, column tile), each wave 8 rows x 16 columns of the block on
// v_mfma_f32_16x16x4f32.  rhs 0: the border's columns (tile 0: the separator
// before the chunk, 1: the one after, then f G), written to W; rhs 1: V, 2: R,
// written to X.  A block step is a chain of five 32 x 32 products between
// barriers, so a product is spread over all waves (512 cycles of matrix core
// each) and the matrices of a step go through LDS, loaded a step before.  64
// nodes of n = 4096, 32 columns: 0.20 ms, 6.5 us per block step (two waves,
// operands from global memory: 0.45); the six tiles of W 0.80 ms (1.68).
// ---------------------------------------------------------------------------
constexpr int kBdSolveThreads = 512;

__global__ __launch_bounds__(kBdSolveThreads) void k_bd_solve(const BdProb* __restrict__ bp,
                                                              const int* __restrict__ prefix, int cnt, int total,
                                                              const ProbDesc* __restrict__ pd, NodeArrays na,
                                                              const c64* __restrict__ blocks,
                                                              const unsigned char* __restrict__ perms, int rhs,
                                                              const c128* __restrict__ Rb, c64* __restrict__ out,
                                                              const int* __restrict__ conv) {
  const int v = xcd_remap(blockIdx.x, gridDim.x, total);
  if (v < 0) return;
  const int s = find_slot(prefix, cnt, v);
  const BdProb& q = bp[s];
  const ProbDesc& D = pd[q.prob];
  if (rhs == 0 && !D.active) return;
  const int tiles = rhs == 0 ? q.wc / B : q.Lp / B;
  int t = v - prefix[s];
  const int j = t / (q.nch * tiles);
  t -= j * q.nch * tiles;
  const int c = t / tiles, tile = t - c * tiles;
  const int g = D.node0 + j;
  if (conv != nullptr && conv[g]) return;
  if (rhs == 0 && ((tile == 0 && c == 0) || (tile == 1 && c == q.nch - 1))) return;  // no such separator
  const int st = bd_start(q, c), len = bd_start(q, c + 1) - 1 - st;
  const c128* __restrict__ f = na.fz + (long long)g * kMaxTerms;
  const int L = D.L, NL = D.N * L, n = D.n;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  __shared__ c64 T[2 * B][B + 1];  // right-hand side window
  __shared__ c64 X[3][B][B + 1];   // block solutions (backward: a ring of three)
  __shared__ c64 Ms[3][B][B + 1];  // the step's block matrices
  __shared__ __align__(16) unsigned char perm[kBdMaxBlocks * 2 * B];

  const c64* __restrict__ bin = blocks + q.offB + ((long long)j * q.nb + st) * 5 * B2;
  const unsigned char* __restrict__ pin = perms + q.offPerm + ((long long)j * q.nb + st) * 2 * B;
  const int os = rhs == 0 ? q.wc : q.Lp;
  c64* __restrict__ o = out + (rhs == 0 ? q.offW : q.offX) + ((long long)j * q.nb + st) * B * os + tile * B;

  // right-hand side entry (row i of block kb, column tid % 32)
  const int rc = tid & (B - 1), cc = tile * B + rc;
  const c128 fh = rhs == 0 && tile >= 2 ? bd_lowrank_f(D, f, cc - 2 * B) : c128{0.0, 0.0};
  auto rhs_elem = [&](int kb, int i) -> c64 {
    const int gr = (st + kb) * B + i;
    if (rhs == 0) {
      if (tile == 0) return kb == 0 ? bd_elem(D, f, q.w, gr, (st - 1) * B + rc) : c64{0.f, 0.f};
      if (tile == 1) return kb == len - 1 ? bd_elem(D, f, q.w, gr, (st + len) * B + rc) : c64{0.f, 0.f};
      return bd_lowrank(fh, D.G32[(long long)gr * q.rp + cc - 2 * B]);
    }
    if (gr >= n || cc >= L) return c64{0.f, 0.f};
    return to64(rhs == 1 ? D.V[(long long)cc * n + gr] : Rb[D.offY + (long long)gr * NL + (long long)j * L + cc]);
  };
  const BdTile tl((wave & 3) * 8, (wave >> 2) * 16);
  const int crow = tl.crow, col = tl.col;
  // a block matrix goes through registers (one 16-byte piece per thread, loaded
  // a step before it is needed) into LDS: read as the operand's lanes need it,
  // every entry would be fetched four times, 16 pieces per load instruction
  static_assert(B2 * sizeof(c64) == kBdSolveThreads * sizeof(float4), "a block matrix is one piece per thread");
  auto fetch = [&](int kb, int which) {
    const int k = max(0, min(kb, len - 1));
    return reinterpret_cast<const float4*>(bin + ((long long)k * 5 + which) * B2)[tid];
  };
  auto stage = [&](int slot, float4 m) {
    c64* d = &Ms[slot][tid / (B / 2)][2 * (tid & (B / 2 - 1))];
    d[0] = c64{m.x, m.y};
    d[1] = c64{m.z, m.w};
  };
  const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
  constexpr int PT = B2 / kBdSolveThreads;  // right-hand side entries per thread and block
  for (int e = tid; e < 2 * B2; e += kBdSolveThreads) {
    const int i = e / B;
    T[i][rc] = i / B < len ? rhs_elem(i / B, i & (B - 1)) : c64{0.f, 0.f};
  }
  for (int e = tid; e < len * B / 2; e += kBdSolveThreads)
    reinterpret_cast<unsigned*>(perm)[e] = reinterpret_cast<const unsigned*>(pin)[e];
  stage(0, fetch(0, 0));
  stage(1, fetch(0, 1));
  float4 pa = fetch(1, 0), pb = fetch(1, 1);
  c64 nxt[PT];
  auto load_rhs = [&](int kb) {
#pragma unroll
    for (int u = 0; u < PT; ++u)
      nxt[u] = kb < len ? rhs_elem(kb, tid / B + u * (kBdSolveThreads / B)) : c64{0.f, 0.f};
  };
  load_rhs(2);
  __syncthreads();
  for (int k = 0; k < len; ++k) {  // forward
    // x_k = L11^-1 t, its rows read through the pivot order
    const unsigned char* pk = perm + k * 2 * B;
    const uint4 pr = *reinterpret_cast<const uint4*>(pk + tl.kh * (B / 2));
    const unsigned pw[4] = {pr.x, pr.y, pr.z, pr.w};
    floatx4 acc = tl.mul<B>(Ms[0], 1.f, zero, [&](int x) {
      const int y = x & (B / 2 - 1);
      return T[(pw[y >> 2] >> (8 * (y & 3))) & 63u][col];
    });
    const c64 lo0 = T[pk[B + crow]][col], lo1 = T[pk[B + crow + 1]][col];
    X[0][crow][col] = c64{acc[0], acc[1]};
    X[0][crow + 1][col] = c64{acc[2], acc[3]};
    o[((long long)k * B + crow) * os + col] = c64{acc[0], acc[1]};
    o[((long long)k * B + crow + 1) * os + col] = c64{acc[2], acc[3]};
    __syncthreads();
    if (k + 1 < len) {
      stage(0, pa);  // every wave is done with L11^-1
      pa = fetch(k + 2, 0);
      acc = tl.mul<B>(Ms[1], -1.f, floatx4{lo0.re, lo0.im, lo1.re, lo1.im}, [&](int x) { return X[0][x][col]; });
      T[crow][col] = c64{acc[0], acc[1]};
      T[crow + 1][col] = c64{acc[2], acc[3]};
#pragma unroll
      for (int u = 0; u < PT; ++u) T[B + tid / B + u * (kBdSolveThreads / B)][rc] = nxt[u];
      load_rhs(k + 3);
      __syncthreads();
      stage(1, pb);  // read after the next step's barrier
      pb = fetch(k + 2, 1);
    }
  }
  // backward: x_k = U11^-1 (x_k - U12 [x_{k+1}; x_{k+2}]), ring slot k % 3
  auto& S0 = *reinterpret_cast<c64(*)[B][B + 1]>(&T[0]);
  stage(0, fetch(len - 1, 2));  // U11^-1; the U12 blocks of the last block are not used
  float4 pi = fetch(len - 2, 2);
  pa = fetch(len - 2, 3);
  pb = fetch(len - 2, 4);
  c64 xf0, xf1;
  auto load_x = [&](int kb) {  // written by this lane in the forward sweep
    const int k = max(kb, 0);
    xf0 = o[((long long)k * B + crow) * os + col];
    xf1 = o[((long long)k * B + crow + 1) * os + col];
  };
  load_x(len - 1);
  for (int k = len - 1; k >= 0; --k) {
    floatx4 acc = {xf0.re, xf0.im, xf1.re, xf1.im};
    load_x(k - 1);
    if (k + 2 < len) acc = tl.mul<B>(Ms[2], -1.f, acc, [&](int x) { return X[(k + 2) % 3][x][col]; });
    if (k + 1 < len) acc = tl.mul<B>(Ms[1], -1.f, acc, [&](int x) { return X[(k + 1) % 3][x][col]; });
    S0[crow][col] = c64{acc[0], acc[1]};
    S0[crow + 1][col] = c64{acc[2], acc[3]};
    __syncthreads();
    stage(1, pa);
    stage(2, pb);
    pa = fetch(k - 2, 3);
    pb = fetch(k - 2, 4);
    acc = tl.mul<B>(Ms[0], 1.f, zero, [&](int x) { return S0[x][col]; });
    X[k % 3][crow][col] = c64{acc[0], acc[1]};
    X[k % 3][crow + 1][col] = c64{acc[2], acc[3]};
    o[((long long)k * B + crow) * os + col] = c64{acc[0], acc[1]};
    o[((long long)k * B + crow + 1) * os + col] = c64{acc[2], acc[3]};
    __syncthreads();
    stage(0, pi);  // read after the next step's first barrier
    pi = fetch(k - 2, 2);
  }
}

// ---------------------------------------------------------------------------
// Partial products H_c^T Z_c of every chunk (Z = W or X): a group of four waves
// per (node, chunk, column tile, 128 rows of H^T), a real product over the
// chunk's rows on the matrix cores, Z's complex columns as pairs of real ones.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_bd_hprod(const BdProb* __restrict__ bp, const int* __restrict__ prefix,
                                                  int cnt, int total, const ProbDesc* __restrict__ pd, int rhs,
                                                  const c64* __restrict__ Zb, c64* __restrict__ part,
                                                  const int* __restrict__ conv) {
  const int v = xcd_remap(blockIdx.x, gridDim.x, total);
  if (v < 0) return;
  const int s = find_slot(prefix, cnt, v);
  const BdProb& q = bp[s];
  const ProbDesc& D = pd[q.prob];
  if (rhs == 0 && !D.active) return;
  const int os = rhs == 0 ? q.wc : q.Lp, tiles = os / B, hb = (q.rp + 127) / 128;
  int t = v - prefix[s];
  const int j = t / (q.nch * tiles * hb);
  t -= j * q.nch * tiles * hb;
  const int c = t / (tiles * hb);
  t -= c * tiles * hb;
  const int tile = t / hb, h0 = (t - tile * hb) * 128;
  if (conv != nullptr && conv[D.node0 + j]) return;
  if (rhs == 0 && ((tile == 0 && c == 0) || (tile == 1 && c == q.nch - 1))) return;
  const int st = bd_start(q, c), len = bd_start(q, c + 1) - 1 - st;
  __shared__ float Hs[B][128 + 4];
  __shared__ float Zs[B][2 * B + 4];
  const float* __restrict__ H = D.H32 + (long long)st * B * q.rp;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const c64* __restrict__ Z = Zb + (rhs == 0 ? q.offW : q.offX) + ((long long)j * q.nb + st) * B * os + tile * B;
  floatx16 acc[2] = {bd_zero(), bd_zero()};
  constexpr int HU = B * 128 / 256, ZU = B2 / 256;
  float hr[HU];
  c64 zr[ZU];
  auto load = [&](int k) {
#pragma unroll
    for (int u = 0; u < HU; ++u) {
      const int e = tid + 256 * u, h = h0 + (e & 127);
      hr[u] = h < q.rp ? H[(long long)(k * B + e / 128) * q.rp + h] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < ZU; ++u) {
      const int e = tid + 256 * u;
      zr[u] = Z[((long long)k * B + e / B) * os + (e & (B - 1))];
    }
  };
  load(0);
  for (int k = 0; k < len; ++k) {
#pragma unroll
    for (int u = 0; u < HU; ++u) {
      const int e = tid + 256 * u;
      Hs[e / 128][e & 127] = hr[u];
    }
#pragma unroll
    for (int u = 0; u < ZU; ++u) {
      const int e = tid + 256 * u;
      Zs[e / B][2 * (e & (B - 1))] = zr[u].re;
      Zs[e / B][2 * (e & (B - 1)) + 1] = zr[u].im;
    }
    __syncthreads();
    if (k + 1 < len) load(k + 1);
#pragma unroll
    for (int m = 0; m < B; m += 2) {
      const float a = Hs[m + (lane >> 5)][wave * 32 + (lane & 31)];
#pragma unroll
      for (int x = 0; x < 2; ++x) acc[x] = bd_mfma(a, Zs[m + (lane >> 5)][32 * x + (lane & 31)], acc[x]);
    }
    __syncthreads();
  }
  // register r: row 8(r/4) + 4(l/32) + r%4, real column l%32
  float* __restrict__ P = reinterpret_cast<float*>(part + q.offPart + ((long long)j * q.nch + c) * q.rp * q.pw);
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int h = h0 + wave * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      if (h < q.rp) P[2 * ((long long)h * q.pw + tile * B) + 32 * x + (lane & 31)] = acc[x][r];
    }
}

// ---------------------------------------------------------------------------
// Border matrix S = [T_SS, (f G)_S; H_S^T, -I] - [F; H_I^T] W.  Groups
// 0 .. nch - 2 of a node: the 32 rows of a separator (whose F blocks, toward
// the chunk before and after, are kept for the solves); the rest: 32 rows of
// the low-rank part each.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_bd_border(const BdProb* __restrict__ bp, const int* __restrict__ prefix,
                                                   int cnt, const ProbDesc* __restrict__ pd, NodeArrays na,
                                                   const c64* __restrict__ Wb, const c64* __restrict__ part,
                                                   c64* __restrict__ FB, c64* __restrict__ Sb) {
  const int v = blockIdx.x;
  const int s = find_slot(prefix, cnt, v);
  const BdProb& q = bp[s];
  const ProbDesc& D = pd[q.prob];
  const int ns = q.nch - 1, per = ns + q.rp / B;
  const int j = (v - prefix[s]) / per, grp = (v - prefix[s]) - j * per;
  if (!D.active) return;
  const int g = D.node0 + j, b = q.b, tid = threadIdx.x;
  const c128* __restrict__ f = na.fz + (long long)g * kMaxTerms;
  c64* __restrict__ S = Sb + q.offS + (long long)j * q.strideS;
  const int low0 = ns * B;
  if (grp < ns) {
    const int sb = bd_start(q, grp + 1) - 1;  // the separator's block
    __shared__ c64 F[2][B][B + 1];
    c64* __restrict__ fo = FB + q.offFB + ((long long)j * ns + grp) * 2 * B2;
    for (int e = tid; e < 2 * B2; e += 256) {
      const int side = e / B2, i = (e / B) & (B - 1), m = e & (B - 1);
      const c64 x = bd_elem(D, f, q.w, sb * B + i, (side == 0 ? sb - 1 : sb + 1) * B + m);
      F[side][i][m] = x;
      fo[e] = x;
    }
    __syncthreads();
    // last block of the chunk before, first of the chunk after
    const c64* __restrict__ W0 = Wb + q.offW + ((long long)j * q.nb + sb - 1) * B * q.wc;
    const c64* __restrict__ W1 = Wb + q.offW + ((long long)j * q.nb + sb + 1) * B * q.wc;
    for (int e = tid; e < B * b; e += 256) {
      const int i = e / b, col = e - i * b;
      c64 x = {0.f, 0.f};
      int c0 = -1, c1 = -1;  // the column in W of the chunk before / after
      if (col < low0) {
        const int sc = col / B, m = col & (B - 1);
        if (sc == grp) x = bd_elem(D, f, q.w, sb * B + i, sb * B + m);
        if (sc == grp) c0 = B + m;
        if (sc == grp - 1) c0 = m;
        if (sc == grp) c1 = m;
        if (sc == grp + 1) c1 = B + m;
      } else {
        x = bd_lowrank(bd_lowrank_f(D, f, col - low0), D.G32[(long long)(sb * B + i) * q.rp + col - low0]);
        c0 = c1 = 2 * B + col - low0;
      }
      if (c0 >= 0)
        for (int m = 0; m < B; ++m) x = fms(x, F[0][i][m], W0[(long long)m * q.wc + c0]);
      if (c1 >= 0)
        for (int m = 0; m < B; ++m) x = fms(x, F[1][i][m], W1[(long long)m * q.wc + c1]);
      S[(long long)(grp * B + i) * q.ldS + col] = x;
    }
    return;
  }
  const int h0 = (grp - ns) * B;
  const c64* __restrict__ P = part + q.offPart + (long long)j * q.nch * q.rp * q.pw;
  for (int e = tid; e < B * b; e += 256) {
    const int i = e / b, col = e - i * b, h = h0 + i;
    auto pe = [&](int c, int pc) { return P[((long long)c * q.rp + h) * q.pw + pc]; };
    c64 x = {0.f, 0.f};
    if (col < low0) {
      const int sc = col / B, m = col & (B - 1);
      x.re = D.H32[(long long)((bd_start(q, sc + 1) - 1) * B + m) * q.rp + h];
      x = x - pe(sc, B + m);   // the separator after chunk sc
      x = x - pe(sc + 1, m);   // and before chunk sc + 1
    } else {
      if (col - low0 == h) x.re = -1.f;
      for (int c = 0; c < q.nch; ++c) x = x - pe(c, 2 * B + col - low0);
    }
    S[(long long)(low0 + h) * q.ldS + col] = x;
  }
}

// Border right-hand side (FP32 values, as the border's solve reads it) and a
// cleared solution: v_S - F x_I for the separators, -H_I^T x_I for the rest.
__global__ __launch_bounds__(256) void k_bd_rhs(const BdProb* __restrict__ bp, const int* __restrict__ prefix, int cnt,
                                                const ProbDesc* __restrict__ pd, int rhs, const c128* __restrict__ Rb,
                                                const c64* __restrict__ Xb, const c64* __restrict__ part,
                                                const c64* __restrict__ FB, c128* __restrict__ RS,
                                                c128* __restrict__ YS, const int* __restrict__ conv) {
  const int v = blockIdx.x;
  const int s = find_slot(prefix, cnt, v);
  const BdProb& q = bp[s];
  const ProbDesc& D = pd[q.prob];
  const int L = D.L, NL = D.N * L, n = D.n, ns = q.nch - 1;
  const int per = (q.b * L + 255) / 256;
  const int j = (v - prefix[s]) / per, e = ((v - prefix[s]) - j * per) * 256 + threadIdx.x;
  if (e >= q.b * L) return;
  if (conv != nullptr && conv[D.node0 + j]) return;
  const int row = e / L, col = e - row * L;
  c64 x = {0.f, 0.f};
  if (row < ns * B) {
    const int sp = row / B, i = row & (B - 1), sb = bd_start(q, sp + 1) - 1, gr = sb * B + i;
    if (gr < n)
      x = to64(rhs == 1 ? D.V[(long long)col * n + gr] : Rb[D.offY + (long long)gr * NL + (long long)j * L + col]);
    const c64* __restrict__ F = FB + q.offFB + ((long long)j * ns + sp) * 2 * B2 + i * B;
    const c64* __restrict__ X = Xb + q.offX + ((long long)j * q.nb + sb) * B * q.Lp + col;
    for (int m = 0; m < B; ++m) x = fms(x, F[m], X[(long long)(m - B) * q.Lp]);
    for (int m = 0; m < B; ++m) x = fms(x, F[B2 + m], X[(long long)(m + B) * q.Lp]);
  } else {
    const c64* __restrict__ P = part + q.offPart + ((long long)j * q.nch * q.rp + row - ns * B) * q.pw + col;
    for (int c = 0; c < q.nch; ++c) x = x - P[(long long)c * q.rp * q.pw];
  }
  const long long o = q.offYS + (long long)row * NL + (long long)j * L + col;
  RS[o] = to128(x);
  YS[o] = c128{0.0, 0.0};
}

// ---------------------------------------------------------------------------
// y = x - W [y_S; s] on the interior blocks, y_S on the separators; Y = y or
// Y += y, with the column maxima.  One group of eight waves per (node, chunk
// with the separator after it, column tile): the border's solution is staged
// in LDS once, each wave takes 16-row strips of W in turn, the next 32
// columns of a strip in flight while one runs on the matrix cores.  Bound by
// reading W and by its products alike.
// ---------------------------------------------------------------------------
constexpr int kBdMaxTiles = 2 + kBdMaxRank / B;

__global__ __launch_bounds__(512) void k_bd_apply(const BdProb* __restrict__ bp, const int* __restrict__ prefix,
                                                  int cnt, int total, const ProbDesc* __restrict__ pd, int add,
                                                  const c64* __restrict__ Wb, const c64* __restrict__ Xb,
                                                  const c128* __restrict__ YS, c128* __restrict__ Yb,
                                                  const int* __restrict__ conv, IrState ir) {
  const int v = xcd_remap(blockIdx.x, gridDim.x, total);
  if (v < 0) return;
  const int s = find_slot(prefix, cnt, v);
  const BdProb& q = bp[s];
  const ProbDesc& D = pd[q.prob];
  const int tiles = q.Lp / B, L = D.L, NL = D.N * L, n = D.n, ns = q.nch - 1;
  int t = v - prefix[s];
  const int j = t / (q.nch * tiles);
  t -= j * q.nch * tiles;
  const int c = t / tiles, tile = t - c * tiles;
  const int g = D.node0 + j;
  if (conv != nullptr && conv[g]) return;
  const int st = bd_start(q, c), len = bd_start(q, c + 1) - 1 - st;
  const int tid = threadIdx.x, wave = tid >> 6;
  const BdLane bl;
  const int cc = tile * B + bl.bcol;
  const c128* __restrict__ ys = YS + q.offYS + (long long)j * L;
  // the border rows that W's column tiles multiply (0 and 1: the separators
  // before and after, where there are such)
  __shared__ c64 Sv[kBdMaxTiles][B][B + 1];
  __shared__ c64 Wt[8][16][B + 1];  // per wave: a strip's 32 columns of W
  const int nk = q.wc / B, nt = nk - (c == 0) - (c == ns);  // tiles that exist
  auto kt_of = [&](int i) {
    i += c == 0 ? 1 : 0;
    return c == ns && i >= 1 ? i + 1 : i;
  };
  for (int e = tid; e < nk * B2; e += 512) {
    const int kt = e / B2, i = (e / B) & (B - 1), m = e & (B - 1), col = tile * B + m;
    const int row = kt == 0 ? (c - 1) * B : kt == 1 ? c * B : ns * B + (kt - 2) * B;
    const bool none = (kt == 0 && c == 0) || (kt == 1 && c == ns) || col >= L;
    Sv[kt][i][m] = none ? c64{0.f, 0.f} : to64(ys[(long long)(row + i) * NL + col]);
  }
  __syncthreads();
  double m2 = 0.0;
  auto put = [&](int gr, c64 x) {
    if (gr < n && cc < L) {
      c128* __restrict__ Y = Yb + D.offY + (long long)gr * NL + (long long)j * L + cc;
      c128 y = to128(x);
      if (add) y = *Y + y;
      *Y = y;
      m2 = nanmax(m2, norm2(y));
    }
  };
  for (int strip = wave; strip < 2 * len; strip += 8) {
    const long long r0 = (long long)j * q.nb * B + st * B + strip * 16;
    const c64* __restrict__ X = Xb + q.offX + r0 * q.Lp + tile * B;
    // (16 bytes per lane and load, four lanes per row and 64-byte piece)
    const int lane = tid & 63, wrow = lane >> 2, wp = lane & 3;
    const float4* __restrict__ W = reinterpret_cast<const float4*>(Wb + q.offW + (r0 + wrow) * q.wc);
    floatx16 acc;
    float4 w4[4];
    auto load = [&](int i) {
#pragma unroll
      for (int x = 0; x < 4; ++x) w4[x] = W[kt_of(i) * (B / 2) + 4 * x + wp];
    };
    if (nt > 0) load(0);
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const c64 x = X[(long long)bl.crow(r) * q.Lp + bl.bcol];
      acc[r] = x.re;
      acc[r + 1] = x.im;
    }
#pragma unroll 1
    for (int i = 0; i < nt; ++i) {
      // (a wave's own LDS traffic is in order: no barrier)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        Wt[wave][wrow][8 * x + 2 * wp] = c64{w4[x].x, w4[x].y};
        Wt[wave][wrow][8 * x + 2 * wp + 1] = c64{w4[x].z, w4[x].w};
      }
      __builtin_amdgcn_wave_barrier();
      if (i + 1 < nt) load(i + 1);
      const c64(&S)[B][B + 1] = Sv[kt_of(i)];
#pragma unroll 8
      for (int x = 0; x < B; ++x)
        acc = bd_mfma(-bl.asign * bd_comp(Wt[wave][bl.arow][x], bl.acomp), bd_comp(S[x][bl.bcol], bl.bcomp), acc);
      __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int r = 0; r < 16; r += 2) put(st * B + strip * 16 + bl.crow(r), c64{acc[r], acc[r + 1]});
  }
  if (c < ns && wave < 2)  // the separator: 16 rows per wave
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const int i = 16 * wave + bl.crow(r);
      put((st + len) * B + i, Sv[1][i][bl.bcol]);
    }
  m2 = nanmax(m2, __shfl_xor(m2, 32, 64));
  if ((threadIdx.x & 63) < 32 && cc < L)
    atomicMax(&ir.ynorm[(long long)g * kNormStride + cc], (unsigned long long)__double_as_longlong(sqrt(m2)));
}

// Smallest pivot modulus, log|det T| and arg det T per node from the chunks'
// and the border's pivots: det of the bordered matrix is det T (times
// (-1)^rp, rp a multiple of 32: the border's -1 diagonal, padded columns
// included).
__global__ __launch_bounds__(64) void k_bd_pivots(const BdProb* __restrict__ bp, const int* __restrict__ prefix,
                                                  int cnt, const ProbDesc* __restrict__ pd,
                                                  const c64* __restrict__ pivots,
                                                  const unsigned char* __restrict__ perms,
                                                  const c64* __restrict__ Sb, const int* __restrict__ rowsS,
                                                  double* __restrict__ pmin, double* __restrict__ det, int nnodes) {
  const int v = blockIdx.x;
  const int s = find_slot(prefix, cnt, v);
  const BdProb& q = bp[s];
  const ProbDesc& D = pd[q.prob];
  const int j = v - prefix[s], g = D.node0 + j, lane = threadIdx.x;
  double m = INFINITY, la = 0.0, ar = 0.0;
  auto take = [&](c64 u) {
    const double re = u.re, im = u.im, a = sqrt(re * re + im * im);
    m = (a < m || a != a) ? a : m;
    if (det != nullptr) {
      la += log(hypot(re, im));
      ar += atan2(im, re);
    }
  };
  for (int c = 0; c < q.nch; ++c) {
    const int st = bd_start(q, c), len = bd_start(q, c + 1) - 1 - st;
    const c64* pv = pivots + q.offPiv + ((long long)j * q.nb + st) * B;
    for (int i = lane; i < len * B; i += 64) take(pv[i]);
    if (det != nullptr) {  // parity of every window's row order: its inversions, 64 entries per wave
      const unsigned char* pk = perms + q.offPerm + ((long long)j * q.nb + st) * 2 * B;
      for (int k = 0; k < len; ++k) {
        const int mine = pk[k * 2 * B + lane];
        int inv = 0;
        for (int o = 0; o < 2 * B; ++o) {
          const int other = pk[k * 2 * B + o];
          inv += (o < lane && other > mine) ? 1 : 0;
        }
        ar += (inv & 1) ? M_PI : 0.0;
      }
    }
  }
  const c64* S = Sb + q.offS + (long long)j * q.strideS;
  const int* rat = rowsS + q.offRowS + j * q.b;
  for (int i = lane; i < q.b; i += 64) {
    take(S[(long long)rat[i] * q.ldS + i]);
    if (det != nullptr) {
      int inv = 0;
      for (int o = 0; o < i; ++o) inv += rat[o] > rat[i] ? 1 : 0;
      ar += (inv & 1) ? M_PI : 0.0;
    }
  }
  for (int o = 32; o >= 1; o >>= 1) {
    const double x = __shfl_xor(m, o, 64);
    m = (x < m || x != x) ? x : m;
    la += __shfl_xor(la, o, 64);
    ar += __shfl_xor(ar, o, 64);
  }
  if (lane == 0) {
    pmin[g] = m;
    if (det != nullptr) {
      det[g] = la;
      det[nnodes + g] = remainder(ar, 2.0 * M_PI);
    }
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
void bd_tables(BdTables& bt, std::vector<int>& buf, const std::vector<BdProb>& bp, const std::vector<ProbDesc>& pd) {
  std::vector<int> lu, se, sv, he, hv, bo, rh, ap, nd;
  for (const BdProb& q : bp) {
    const int N = pd[q.prob].N, L = pd[q.prob].L, tw = q.wc / B, tl = q.Lp / B, hb = ceil_div(q.rp, 128);
    lu.push_back(N * q.nch);
    se.push_back(N * q.nch * tw);
    sv.push_back(N * q.nch * tl);
    he.push_back(N * q.nch * tw * hb);
    hv.push_back(N * q.nch * tl * hb);
    bo.push_back(N * (q.nch - 1 + q.rp / B));
    rh.push_back(N * ceil_div(q.b * L, 256));
    ap.push_back(N * q.nch * tl);
    nd.push_back(N);
  }
  build_prefix(buf, bt.lu, lu);
  build_prefix(buf, bt.solve_e, se);
  build_prefix(buf, bt.solve_v, sv);
  build_prefix(buf, bt.hprod_e, he);
  build_prefix(buf, bt.hprod_v, hv);
  build_prefix(buf, bt.border, bo);
  build_prefix(buf, bt.rhs, rh);
  build_prefix(buf, bt.apply, ap);
  build_prefix(buf, bt.node, nd);
}

hipError_t bd_factor(const BdTables& bt, const BdProb* bp, const ProbDesc* pd, const int* pre, const NodeArrays& na,
                     const BdBufs& m, int* info, hipStream_t st) {
  hipLaunchKernelGGL(k_bd_lu, dim3(bt.lu.total), dim3(kBdLuThreads), 0, st, bp, pre + bt.lu.off, bt.lu.cnt, pd, na, m.blocks,
                     m.perms, m.pivots, info);
  hipLaunchKernelGGL(k_bd_solve, dim3(xcd_grid(bt.solve_e.total)), dim3(kBdSolveThreads), 0, st, bp, pre + bt.solve_e.off,
                     bt.solve_e.cnt, bt.solve_e.total, pd, na, m.blocks, m.perms, 0, (const c128*)nullptr, m.W,
                     (const int*)nullptr);
  if (bt.hprod_e.total > 0)
    hipLaunchKernelGGL(k_bd_hprod, dim3(xcd_grid(bt.hprod_e.total)), dim3(256), 0, st, bp, pre + bt.hprod_e.off,
                       bt.hprod_e.cnt, bt.hprod_e.total, pd, 0, m.W, m.part, (const int*)nullptr);
  if (bt.border.total > 0)
    hipLaunchKernelGGL(k_bd_border, dim3(bt.border.total), dim3(256), 0, st, bp, pre + bt.border.off, bt.border.cnt, pd,
                       na, m.W, m.part, m.FB, m.S);
  return hipGetLastError();
}

hipError_t bd_solve_pre(const BdTables& bt, const BdProb* bp, const ProbDesc* pd, const int* pre, const NodeArrays& na,
                        const BdBufs& m, const c128* R, bool refine, const int* conv, hipStream_t st) {
  const int rhs = refine ? 2 : 1;
  hipLaunchKernelGGL(k_bd_solve, dim3(xcd_grid(bt.solve_v.total)), dim3(kBdSolveThreads), 0, st, bp, pre + bt.solve_v.off,
                     bt.solve_v.cnt, bt.solve_v.total, pd, na, m.blocks, m.perms, rhs, R, m.X, conv);
  if (bt.hprod_v.total > 0)
    hipLaunchKernelGGL(k_bd_hprod, dim3(xcd_grid(bt.hprod_v.total)), dim3(256), 0, st, bp, pre + bt.hprod_v.off,
                       bt.hprod_v.cnt, bt.hprod_v.total, pd, 1, m.X, m.part, conv);
  if (bt.rhs.total > 0)
    hipLaunchKernelGGL(k_bd_rhs, dim3(bt.rhs.total), dim3(256), 0, st, bp, pre + bt.rhs.off, bt.rhs.cnt, pd, rhs, R,
                       m.X, m.part, m.FB, m.RS, m.YS, conv);
  return hipGetLastError();
}

hipError_t bd_solve_post(const BdTables& bt, const BdProb* bp, const ProbDesc* pd, const int* pre, const BdBufs& m,
                         c128* Y, bool refine, const int* conv, IrState ir, hipStream_t st) {
  hipLaunchKernelGGL(k_bd_apply, dim3(xcd_grid(bt.apply.total)), dim3(512), 0, st, bp, pre + bt.apply.off,
                     bt.apply.cnt, bt.apply.total, pd, refine ? 1 : 0, m.W, m.X, m.YS, Y, conv, ir);
  return hipGetLastError();
}

hipError_t bd_pivots(const BdTables& bt, const BdProb* bp, const ProbDesc* pd, const int* pre, const BdBufs& m,
                     const int* rowsS, double* pmin, double* det, int nnodes, hipStream_t st) {
  hipLaunchKernelGGL(k_bd_pivots, dim3(bt.node.total), dim3(64), 0, st, bp, pre + bt.node.off, bt.node.cnt, pd,
                     m.pivots, m.perms, m.S, rowsS, pmin, det, nnodes);
  return hipGetLastError();
}

}  // namespace nep
