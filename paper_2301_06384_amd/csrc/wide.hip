// Small float64 kernels for block widths 65..512: the CholQR factors of the
// Lanczos blocks (Alg. 1, QR of X), the block orthogonality estimate of
// partial reorthogonalisation and the banded spline evaluation
// (eps I + H_m)^(-k) F_1, for matrices of up to 8 x 8 tiles of 64 x 64.
//
// A workgroup of 256 threads forms a tile: it stages the two operand tiles of
// each product from device memory (L2-resident at these sizes) into LDS and
// runs the 64-wide register-blocked product of tile64.h; the 64 x 64 diagonal
// Cholesky steps run the FP64-MFMA blocked factorisation of tile64.h on one
// tile.  Matrices are row-major with zero padding beyond s, so a partial last
// tile needs no special case.
#include "gk_internal.h"
#include "tile64.h"

namespace gk {

constexpr int WQ_MAX = 8;            // tiles per side (s <= 512)
constexpr int WCOL = 64 * WQ_MAX;

bool wide_ok(int ld) { return ld > WS && ld <= WCOL; }

// v[4a+b] = src[i * lds + c] (i = ty + 16a, c = tx + 16b) for i < nr, c < nc
__device__ __forceinline__ void fetch_rc(const double* __restrict__ src, int nr, int nc, int lds, double (&v)[16]) {
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = ty + 16 * a, c = tx + 16 * b;
      v[4 * a + b] = (i < nr && c < nc) ? src[i * lds + c] : 0.0;
    }
}

__device__ __forceinline__ void zero44(double (&t)[4][4]) {
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) t[a][b] = 0.0;
}

// This thread's 16 elements of tile (I, J) of an s x s matrix with leading
// dimension ld, in the lds_mm output layout: load (0 outside) and store.
__device__ __forceinline__ void tile_get(const double* __restrict__ M, int ld, int s, int I, int J, double (&t)[4][4]) {
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int r = 64 * I + acc_row(a), c = 64 * J + acc_col(b);
      t[a][b] = (r < s && c < s) ? M[(int64_t)r * ld + c] : 0.0;
    }
}
__device__ __forceinline__ void tile_put(double* __restrict__ M, int ld, int s, int I, int J, const double (&t)[4][4]) {
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int r = 64 * I + acc_row(a), c = 64 * J + acc_col(b);
      if (r < s && c < s) M[(int64_t)r * ld + c] = t[a][b];
    }
}

// tot += sign * sum_{K0 <= K < K1} op(X)_{IK} op(Y)_{KJ} on tiles of s x s
// matrices (op = transpose when tX / tY).  Both operand tiles go through LDS
// in the X^T B form of lds_mm: SA[l][r] = op(X)[r][l], SB[l][c] = op(Y)[l][c].
__device__ __forceinline__ void wterm(double (&tot)[4][4], double sign, const double* __restrict__ X, int ldx, bool tX,
                                      const double* __restrict__ Y, int ldy, bool tY, int s, int I, int J, int K0,
                                      int K1, double (*SA)[LP], double (*SB)[LP]) {
  for (int K = K0; K < K1; ++K) {
    const int kext = min(64, s - 64 * K);
    double va[16], vb[16];
    __syncthreads();   // earlier stores visible, earlier readers of SA / SB done
    if (!tX) fetch_rc(X + (int64_t)(64 * I) * ldx + 64 * K, s - 64 * I, s - 64 * K, ldx, va);
    else fetch_rc(X + (int64_t)(64 * K) * ldx + 64 * I, s - 64 * K, s - 64 * I, ldx, va);
    if (!tY) fetch_rc(Y + (int64_t)(64 * K) * ldy + 64 * J, s - 64 * K, s - 64 * J, ldy, vb);
    else fetch_rc(Y + (int64_t)(64 * J) * ldy + 64 * K, s - 64 * J, s - 64 * K, ldy, vb);
    if (!tX) put64T(SA, va); else put64(SA, va);
    if (!tY) put64(SB, vb); else put64T(SB, vb);
    __syncthreads();
    double acc[4][4];
    lds_mm<true, false>(SA, SB, kext, acc);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) tot[a][b] = fma(sign, acc[a][b], tot[a][b]);
  }
}

// Right-looking blocked Cholesky with inverse of an s x s symmetric matrix
// (tiles of 64): for each tile column k
//   A_kk = L_kk L_kk^T, Y_kk = L_kk^{-1}   (tile64 blocked factor, pivot rule MODE)
//   L_ik = A_ik Y_kk^T,  A_ij -= L_ik L_jk^T   (k < j <= i)
//   Z_ib += L_ik Y_kb   (b <= k < i),  Y_kb = -Y_kk Z_kb
// as a chain of launches, one per tile column, each tile of a step in its own
// workgroup.  A workgroup recomputes the panel tiles that it needs rather than
// wait for another's, and the one of (k+1, k+1) goes on to factor its tile, so
// the chain is a 64 x 64 Cholesky and three tile products a step.
// Bound by that chain.  In one workgroup the n^3 work ran at the rate of one of
// 256 compute units: s = 512: 2.4 ms, now 0.33; s = 128: 165 us, now 110.
// The launches are the faster form down to the narrowest widths here, also where
// the second pass is switched off (empty launches).  One workgroup | launches, ms
// of CholQR in a call of 19 steps, 20k nodes: s = 65 float64 3.40 | 2.42, mixed
// (17 second passes off) 2.24 | 1.78; s = 80 3.41 | 2.45, 2.45 | 1.78; s = 96 3.89 |
// 2.76, 2.71 | 1.85.  Factor and k = 2 substitutions of the spline, 20 blocks:
// s = 65 3.57 | 2.45, s = 96 4.07 | 2.71.
//
// Launch k reads the tiles of column k (L_kk, Y_kk and A_ik).  Storage: A and
// Y hold their diagonal tiles (L_kk, Y_kk) and, below them, the tiles still
// being updated (A_ij, Z_ib); what is final goes above the diagonal,
// transposed: R_kj = L_jk^T in A, (Y_kb)^T in Y.  No tile is written in the
// launch in which another workgroup reads it.
struct WideFac {
  const double* src;    // the matrix (ld), read by the first column's steps
  double *A, *Y;        // ld x ld
  int ld, s;
  const double* dprev;  // pivot rule 2
  double thr;
  double* dg;           // diagonal of L, negative where the pivot was clamped; null: not kept
  int* bad;
  const int* gate;      // non-null: nothing is done where *gate == 0
};

// T0: tile (b, b) of the matrix.  Factors it and stores L_bb, Y_bb, dg.
template <int MODE>
__device__ __forceinline__ void wide_diag(const WideFac& f, int b, double (*T0)[LP], double (*T1)[LP],
                                          double (*T2)[LP]) {
  __shared__ double g0[64], dp[64], dgl[64];
  __shared__ int clf[64];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int sb = min(64, f.s - 64 * b);
  if (MODE != 0 && tid < 64) {
    const int64_t q = 64 * b + tid;
    g0[tid] = (MODE == 1 && tid < sb) ? f.src[q * f.ld + q] : 0.0;
    dp[tid] = (MODE == 2 && tid < sb) ? f.dprev[q] : 0.0;
    clf[tid] = 0;
  }
  __syncthreads();
  blk_chol_inv_t<MODE>(T0, T1, T2, sb, MODE != 0 ? g0 : nullptr, MODE != 0 ? dp : nullptr, f.thr,
                       MODE != 0 ? dgl : nullptr, f.bad, MODE != 0 ? clf : nullptr);
  const int64_t o = (int64_t)(64 * b) * f.ld + 64 * b;
  for (int i = ty; i < sb; i += 16)
    for (int c = tx; c < sb; c += 16) {
      f.A[o + (int64_t)i * f.ld + c] = T0[i][c];
      f.Y[o + (int64_t)i * f.ld + c] = T1[i][c];
    }
  if (MODE != 0 && f.dg && tid < sb) f.dg[64 * b + tid] = clf[tid] ? -dgl[tid] : dgl[tid];
}

__device__ __forceinline__ bool wide_off(const WideFac& f) { return f.gate && *f.gate == 0; }
__device__ __forceinline__ void fetch_tile(const double* __restrict__ M, int ld, int s, int I, int J, double (&v)[16]) {
  fetch_rc(M + (int64_t)(64 * I) * ld + 64 * J, s - 64 * I, s - 64 * J, ld, v);
}
// the product held in acc as an operand: D[col][row]
__device__ __forceinline__ void put_accT(double (*D)[LP], const double (&acc)[4][4]) {
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) D[acc_col(b)][acc_row(a)] = acc[a][b];
}
__device__ __forceinline__ void put_acc(double (*D)[LP], const double (&acc)[4][4]) {
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) D[acc_row(a)][acc_col(b)] = acc[a][b];
}
// tile (I, J) of M = D (TR: its transpose)
template <bool TR>
__device__ __forceinline__ void store_tile(double* __restrict__ M, int ld, int nr, int nc, int I, int J,
                                           const double (*D)[LP]) {
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int i = ty + 16 * a, c = tx + 16 * b;
      if (64 * I + i < nr && 64 * J + c < nc) M[(int64_t)(64 * I + i) * ld + 64 * J + c] = TR ? D[c][i] : D[i][c];
    }
}

__host__ __device__ inline int wide_col_tasks(int nQ, int k) {
  const int r = nQ - 1 - k;
  return r < 1 ? 0 : r * (r + 1) / 2 + r * (k + 1);
}

template <int MODE>
__device__ __forceinline__ void wide_col_body(const WideFac& f, int k, int task) {
  __shared__ __align__(16) double T0[WS][LP];
  __shared__ __align__(16) double T1[WS][LP];
  __shared__ __align__(16) double T2[WS][LP];
  __shared__ __align__(16) double T3[WS][LP];
  const int nQ = (f.s + 63) >> 6, nr = nQ - 1 - k, na = nr * (nr + 1) / 2;
  if (task >= wide_col_tasks(nQ, k) || wide_off(f)) return;
  int i, j = 0, b = 0;
  const bool trail = task < na;
  if (trail) {
    int ii = 0, rem = task;
    while (rem > ii) { rem -= ii + 1; ++ii; }
    i = k + 1 + ii;
    j = k + 1 + rem;
  } else {
    i = k + 1 + (task - na) / (k + 1);
    b = (task - na) % (k + 1);
  }
  const double* M = k == 0 ? f.src : f.A;
  const int ld = f.ld, s = f.s;
  // column k is a full tile: a row tile follows it
  double vy[16], va[16], vb[16];
  fetch_tile(f.Y, ld, s, k, k, vy);
  fetch_tile(M, ld, s, i, k, va);
  if (trail) {
    if (j != i) fetch_tile(M, ld, s, j, k, vb);
  } else if (b < k) {
    fetch_tile(f.Y, ld, s, k, b, vb);   // Z_kb
  }
  double t[4][4];
  if (trail) tile_get(M, ld, s, i, j, t);
  else if (b < k) tile_get(f.Y, ld, s, i, b, t);
  else zero44(t);
  put64T(T3, vy);                        // T3[l][r] = Y_kk[r][l]
  put64T(T2, va);                        // T2[l][r] = A_ik[r][l]
  if (trail) {
    if (j != i) put64T(T0, vb);
  } else {
    put64(T1, b < k ? vb : vy);
  }
  __syncthreads();
  // L_ik, L_jk: columns with a clamped pivot stay decoupled
  auto panel = [&](double (*X)[LP], double (&acc)[4][4]) {
    lds_mm<true, false>(X, T3, 64, acc);
    if (MODE != 0) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (f.dg && signbit(f.dg[64 * k + acc_col(c)]))
#pragma unroll
          for (int a = 0; a < 4; ++a) acc[a][c] = 0.0;
    }
  };
  double li[4][4], lj[4][4];
  panel(T2, li);
  if (trail && j != i) panel(T0, lj);
  double yk[4][4];
  if (!trail && b < k) {
    lds_mm<true, false>(T3, T1, 64, yk);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int c = 0; c < 4; ++c) yk[a][c] = fma(-1.0, yk[a][c], 0.0);
  }
  __syncthreads();
  put_accT(T2, li);
  if (trail && j != i) put_accT(T0, lj);
  if (!trail && b < k) put_acc(T1, yk);
  __syncthreads();
  double p[4][4];
  lds_mm<true, false>(T2, trail ? (j != i ? T0 : T2) : T1, 64, p);
  const double sign = trail ? -1.0 : 1.0;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) t[a][c] = fma(sign, p[a][c], t[a][c]);
  if (trail) {
    if (j == k + 1) store_tile<false>(f.A, ld, s, s, k, i, T2);   // R_ki
    if (i != k + 1) {
      tile_put(f.A, ld, s, i, j, t);
    } else {
      __syncthreads();
      put_acc(T0, t);
      __syncthreads();
      wide_diag<MODE>(f, k + 1, T0, T1, T2);
    }
  } else {
    tile_put(f.Y, ld, s, i, b, t);
    if (b < k && i == k + 1) store_tile<true>(f.Y, ld, s, s, b, k, T1);   // (Y_kb)^T
  }
}

// the last row of the inverse: Y_kb = -Y_kk Z_kb, k = nQ - 1, b = task; with
// LOWER the off-diagonal tiles (i, b) of all rows also move to their place
// below the diagonal, and zeros above it
template <bool LOWER>
__device__ __forceinline__ void wide_last_body(const WideFac& f, int task) {
  __shared__ __align__(16) double T0[WS][LP];
  __shared__ __align__(16) double T1[WS][LP];
  const int nQ = (f.s + 63) >> 6;
  if (task >= (LOWER ? nQ * (nQ - 1) / 2 : nQ - 1) || wide_off(f)) return;
  int i = nQ - 1, b = task;
  if (LOWER) {
    int ii = 0;
    while (b > ii) { b -= ii + 1; ++ii; }
    i = ii + 1;
  }
  double v[16];
  if (i == nQ - 1) {
    const int sk = f.s - 64 * i;
    double vy[16], acc[4][4];
    fetch_tile(f.Y, f.ld, f.s, i, i, vy);
    fetch_tile(f.Y, f.ld, f.s, i, b, v);
    put64T(T0, vy);
    put64(T1, v);
    __syncthreads();
    lds_mm<true, false>(T0, T1, sk, acc);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[a][c] = fma(-1.0, acc[a][c], 0.0);
    __syncthreads();
    put_acc(T1, acc);
  } else {
    fetch_tile(f.Y, f.ld, f.s, b, i, v);
    put64T(T1, v);
  }
  __syncthreads();
  if (LOWER) {
    store_tile<false>(f.Y, f.ld, f.s, f.s, i, b, T1);
    double z[4][4];
    zero44(z);
    tile_put(f.Y, f.ld, f.s, b, i, z);
  } else {
    store_tile<true>(f.Y, f.ld, f.s, f.s, b, i, T1);
  }
}

// ---------------------------------------------------------------- CholQR
// Same factor as the 64-wide kernel (pass 1: clamped pivots, pass 2:
// combined-diagonal deflation, then Rc = R1inv R2inv and B = R2 R1), for
// 64 < ld <= 512, entry blockIdx.y of the batch.  Pass 2 does nothing where
// its gate is 0 (decided by the first pass and the projection).
struct CholqrWideBatch {
  CholqrArgs a[kCholqrBatch];
};
__device__ __forceinline__ WideFac cholqr_fac(const CholqrArgs& a) {
  return WideFac{a.G, a.wk, a.wk + (size_t)a.ld * a.ld, a.ld, a.s, a.diag_prev, a.thr, a.diag_out, nullptr,
                 a.pass == 2 ? a.gate : nullptr};
}
__global__ void __launch_bounds__(ST) cholqr_first_kernel(CholqrWideBatch b) {
  __shared__ __align__(16) double T0[WS][LP];
  __shared__ __align__(16) double T1[WS][LP];
  __shared__ __align__(16) double T2[WS][LP];
  const CholqrArgs& a = b.a[blockIdx.x];
  const WideFac f = cholqr_fac(a);
  if (wide_off(f)) {
    if (threadIdx.x == 0 && a.n_defl) a.n_defl[5] += 1;   // counted five entries after the deflations
    return;
  }
  double v[16];
  fetch_tile(a.G, a.ld, a.s, 0, 0, v);
  put64(T0, v);
  if (a.pass == 1) wide_diag<1>(f, 0, T0, T1, T2);
  else wide_diag<2>(f, 0, T0, T1, T2);
}
template <int PASS>
__global__ void __launch_bounds__(ST) cholqr_col_kernel(CholqrWideBatch b, int k) {
  wide_col_body<PASS>(cholqr_fac(b.a[blockIdx.y]), k, blockIdx.x);
}
__global__ void __launch_bounds__(ST) cholqr_last_kernel(CholqrWideBatch b) {
  wide_last_body<false>(cholqr_fac(b.a[blockIdx.y]), blockIdx.x);
}
// Pass 1 with a gate: one pass leaves X R^-1 orthonormal to about
// s u |D R^-1|_2^2 with D = diag(G)^(1/2) (Gram and Cholesky errors are
// relative to the column norms), and |D R^-1|_2^2 <= |Z|_1 |Z|_inf for
// Z = L^-1 D.  When that gives 1e-10 or better and no pivot was clamped, the
// first factor is final: Rc = R^-1, B = R and B^T are written with R and
// R^-1, and the gate tells the second pass (and the Gram launch before it) to
// do nothing.  Here the largest column sum, row sum and clamp flag of the
// indices 64 J .., to three doubles of the dead tile (1, 0) of A.
__device__ __forceinline__ double* wide_norms_at(const CholqrArgs& a, int J) { return a.wk + (int64_t)64 * a.ld + 3 * J; }
__global__ void __launch_bounds__(ST) cholqr_norms_kernel(CholqrWideBatch bt) {
  __shared__ double red[3][ST / 64];
  const CholqrArgs& a = bt.a[blockIdx.y];
  const int s = a.s, ld = a.ld, nQ = (s + 63) >> 6, J = blockIdx.x;
  if (!a.gate || J >= nQ) return;
  const double* Yw = a.wk + (size_t)ld * ld;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, end = min(s, 64 * J + 64);
  double cmax = 0.0, rmax = 0.0, cl = 0.0;
  for (int q = 64 * J + wv; q < end; q += ST / 64) {
    double u = 0.0, r = 0.0;
    // column q of Y: its diagonal tile, then row q above the diagonal tiles
    if (64 * J + lane < end) u = fabs(Yw[(int64_t)(64 * J + lane) * ld + q]);
    for (int c = 64 * J + 64 + lane; c < s; c += 64) u += fabs(Yw[(int64_t)q * ld + c]);
    // row q of Y: column q above the diagonal tile, then the tile's row
    for (int c = lane; c < 64 * J; c += 64) r += fabs(Yw[(int64_t)c * ld + q]) * sqrt(fmax(a.G[(int64_t)c * ld + c], 0.0));
    if (64 * J + lane < end) {
      const int64_t c = 64 * J + lane;
      r += fabs(Yw[(int64_t)q * ld + c]) * sqrt(fmax(a.G[c * ld + c], 0.0));
    }
    for (int o = 32; o > 0; o >>= 1) {
      u += __shfl_xor(u, o);
      r += __shfl_xor(r, o);
    }
    cmax = fmax(cmax, u * sqrt(fmax(a.G[(int64_t)q * ld + q], 0.0)));
    rmax = fmax(rmax, r);
    const double d = a.diag_out[q];
    if (signbit(d) || d == 0.0) cl = 1.0;
  }
  if (lane == 0) {
    red[0][wv] = cmax;
    red[1][wv] = rmax;
    red[2][wv] = cl;
  }
  __syncthreads();
  if (tid < 3) {
    double v = 0.0;
    for (int w = 0; w < ST / 64; ++w) v = fmax(v, red[tid][w]);
    wide_norms_at(a, J)[tid] = v;
  }
}
// results of the factorisation, tile (I, J), I <= J, and its mirror
__global__ void __launch_bounds__(ST) cholqr_out_kernel(CholqrWideBatch bt) {
  __shared__ __align__(16) double T0[WS][LP];
  __shared__ __align__(16) double T1[WS][LP];
  const CholqrArgs& a = bt.a[blockIdx.y];
  const WideFac f = cholqr_fac(a);
  const int s = a.s, ld = a.ld, nQ = (s + 63) >> 6, tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  int I = 0, J = blockIdx.x;
  if (J >= nQ * (nQ + 1) / 2 || wide_off(f)) return;
  {
    int jj = 0;
    while (J > jj) { J -= jj + 1; ++jj; }
    I = J;
    J = jj;
  }
  const double* A = f.A;
  const double* Y = f.Y;
  if (I == J && tid < 64) {
    const int q = 64 * I + tid;
    if (q < ld) a.diag_out[q] = q < s ? fabs(a.diag_out[q]) : 0.0;
  }
  // tile (P, Q), P <= Q, of R (from A) or R^-1 (from Y), D[row][col]
  auto upper = [&](const double* M, int P, int Q, double (*D)[LP]) {
    double v[16];
    fetch_tile(M, ld, s, P, Q, v);
    if (P == Q) put64T(D, v);
    else put64(D, v);
  };
  // tile and zero mirror of an upper triangular matrix
  auto out_upper = [&](double* M, int ldm, int nm, const double (*D)[LP]) {
    store_tile<false>(M, ldm, nm, nm, I, J, D);
    if (I != J) {
      double z[4][4];
      zero44(z);
      tile_put(M, ldm, nm, J, I, z);
    }
  };
  auto out_transposed = [&](double* M, const double (*D)[LP]) {
    store_tile<true>(M, ld, ld, ld, J, I, D);
    if (I != J) {
      double z[4][4];
      zero44(z);
      tile_put(M, ld, ld, I, J, z);
    }
  };
  if (a.pass == 1) {
    bool sk = false;
    if (a.gate) {
      double nm[3] = {0.0, 0.0, 0.0};
      for (int w = 0; w < nQ; ++w)
        for (int c = 0; c < 3; ++c) nm[c] = fmax(nm[c], wide_norms_at(a, w)[c]);
      sk = nm[2] == 0.0 && nm[0] * nm[1] * (double)s * 0x1p-53 <= 1e-10;
      if (blockIdx.x == 0 && tid == 0) *a.gate = sk ? 0 : 1;
    }
    if (!a.R) return;
    upper(A, I, J, T0);
    upper(Y, I, J, T1);
    __syncthreads();
    out_upper(a.R, ld, ld, T0);
    out_upper(a.Rinv, ld, ld, T1);
    if (sk) {
      out_upper(a.Bout, s, s, T0);
      out_upper(a.Rc, ld, ld, T1);
      if (a.BT) out_transposed(a.BT, T0);
    }
    return;
  }
  if (blockIdx.x == 0 && tid == 0 && a.n_defl) {
    int cnt = 0;
    for (int q = 0; q < s; ++q) cnt += (a.diag_out[q] == 0.0);   // -0 too
    a.n_defl[0] += cnt;
  }
  // B = R2 R1, Rc = R1^-1 R2^-1
  double bb[4][4], rc[4][4];
  zero44(bb);
  zero44(rc);
  for (int which = 0; which < 2; ++which)
    for (int K = I; K <= J; ++K) {
      double v[16];
      __syncthreads();
      if (which == 0) {
        // T0[l][r] = R2[r][l], T1[l][c] = R1[l][c]
        fetch_tile(A, ld, s, I, K, v);
        if (K == I) put64(T0, v);
        else put64T(T0, v);
        fetch_tile(a.R1, ld, s, K, J, v);
        put64(T1, v);
      } else {
        fetch_tile(a.R1inv, ld, s, I, K, v);
        put64T(T0, v);
        upper(Y, K, J, T1);
      }
      __syncthreads();
      double acc[4][4];
      lds_mm<true, false>(T0, T1, min(64, s - 64 * K), acc);
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y) {
          double& d = which == 0 ? bb[x][y] : rc[x][y];
          d = fma(1.0, acc[x][y], d);
        }
    }
  __syncthreads();
  // entries at and beyond s are zero
  put_acc(T0, bb);
  put_acc(T1, rc);
  __syncthreads();
  for (int r = ty; r < 64; r += 16)
    for (int c = tx; c < 64; c += 16)
      if (64 * I + r >= s || 64 * J + c >= s) T0[r][c] = T1[r][c] = 0.0;
  __syncthreads();
  out_upper(a.Bout, s, s, T0);
  out_upper(a.Rc, ld, ld, T1);
  if (a.BT) out_transposed(a.BT, T0);
}

size_t cholqr_wide_scratch_elems(int ld) { return (size_t)2 * ld * ld; }

void launch_cholqr_wide_batched(const CholqrArgs* a, int count, hipStream_t st) {
  for (int c0 = 0; c0 < count; c0 += kCholqrBatch) {
    const int nb = std::min(kCholqrBatch, count - c0);
    CholqrWideBatch pass[2]{};
    int ns[2] = {0, 0}, nq[2] = {0, 0};
    double bytes = 0, flops = 0;
    for (int i = 0; i < nb; ++i) {
      const CholqrArgs& x = a[c0 + i];
      GK_REQUIRE(x.s > 64 && x.s <= x.ld && wide_ok(x.ld) && (x.pass == 1 || x.pass == 2), GK_EUNSUPPORTED,
                 "wide CholQR: unsupported block shape");
      const int p = x.pass - 1;
      pass[p].a[ns[p]++] = x;
      nq[p] = std::max(nq[p], (x.s + 63) >> 6);
      bytes += 8.0 * 6 * x.ld * x.ld;
      flops += (double)x.s * x.s * x.s * (x.pass == 2 ? 3.0 : 1.0);
    }
    kt_begin(KC_CHOLQR, st);
    for (int p = 0; p < 2; ++p) {
      if (!ns[p]) continue;
      const CholqrWideBatch& b = pass[p];
      const int nQ = nq[p];
      hipLaunchKernelGGL(cholqr_first_kernel, dim3(ns[p]), dim3(ST), 0, st, b);
      for (int k = 0; k + 1 < nQ; ++k) {
        int tasks = 0;
        for (int q = 0; q < ns[p]; ++q) tasks = std::max(tasks, wide_col_tasks((b.a[q].s + 63) >> 6, k));
        const dim3 grid(tasks, ns[p]);
        if (p == 0) hipLaunchKernelGGL(cholqr_col_kernel<1>, grid, dim3(ST), 0, st, b, k);
        else hipLaunchKernelGGL(cholqr_col_kernel<2>, grid, dim3(ST), 0, st, b, k);
      }
      hipLaunchKernelGGL(cholqr_last_kernel, dim3(nQ - 1, ns[p]), dim3(ST), 0, st, b);
      bool gated = false;
      for (int q = 0; q < ns[p]; ++q) gated = gated || b.a[q].gate;
      if (p == 0 && gated) hipLaunchKernelGGL(cholqr_norms_kernel, dim3(nQ, ns[p]), dim3(ST), 0, st, b);
      hipLaunchKernelGGL(cholqr_out_kernel, dim3(nQ * (nQ + 1) / 2, ns[p]), dim3(ST), 0, st, b);
    }
    GK_HIP(hipGetLastError());
    kt_end(st, bytes, flops);
  }
}

// ------------------------------------------------- orthogonality estimate
// Block omega recurrence (the same estimate as the 64-wide kernel): first
// the right-hand side
//   W_{k,j+1} B_j + W_{k,j} H_j - H_k W_{k,j} + W_{k,j-1} B_{j-1}^T - B_{k-1} W_{k-1,j}
// plus the rounding model (+-nu in the direction of each entry), one
// workgroup per (j, tile); then W_{k+1,j} = Rc^T RHS and the tile maxima.
__global__ void __launch_bounds__(ST)
omega_rhs_wide_kernel(int k, int s, const double* __restrict__ Wk, const double* __restrict__ Wkm1,
                      const double* __restrict__ Hd, const double* __restrict__ Bd, double nu,
                      double* __restrict__ rhs) {
  __shared__ __align__(16) double SA[WS][LP];
  __shared__ __align__(16) double SB[WS][LP];
  const int j = blockIdx.x, I = blockIdx.y, J = blockIdx.z;
  const int nQ = (s + 63) >> 6;
  const int64_t ss = (int64_t)s * s;
  double t[4][4];
  zero44(t);
  wterm(t, 1.0, Wk + (j + 1) * ss, s, false, Bd + j * ss, s, false, s, I, J, 0, nQ, SA, SB);
  wterm(t, 1.0, Wk + j * ss, s, false, Hd + j * ss, s, false, s, I, J, 0, nQ, SA, SB);
  wterm(t, -1.0, Hd + (int64_t)k * ss, s, false, Wk + j * ss, s, false, s, I, J, 0, nQ, SA, SB);
  if (j >= 1) wterm(t, 1.0, Wk + (j - 1) * ss, s, false, Bd + (j - 1) * ss, s, true, s, I, J, 0, nQ, SA, SB);
  wterm(t, -1.0, Bd + (int64_t)(k - 1) * ss, s, false, Wkm1 + j * ss, s, false, s, I, J, 0, nQ, SA, SB);
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) t[a][b] += copysign(nu, t[a][b]);
  tile_put(rhs + j * ss, s, s, I, J, t);
}

__global__ void __launch_bounds__(ST)
omega_apply_wide_kernel(int s, int ld, const double* __restrict__ Rc, const double* __restrict__ rhs,
                        double* __restrict__ Wk1, double* __restrict__ est_part) {
  __shared__ __align__(16) double SA[WS][LP];
  __shared__ __align__(16) double SB[WS][LP];
  __shared__ double red[ST];
  const int j = blockIdx.x, I = blockIdx.y, J = blockIdx.z;
  const int nQ = (s + 63) >> 6;
  const int64_t ss = (int64_t)s * s;
  const int tid = threadIdx.x;
  double t[4][4];
  zero44(t);
  wterm(t, 1.0, Rc, ld, true, rhs + j * ss, s, false, s, I, J, 0, nQ, SA, SB);
  tile_put(Wk1 + j * ss, s, s, I, J, t);
  double mx = 0.0;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) mx = fmax(mx, fabs(t[a][b]));   // zero outside s
  red[tid] = mx;
  __syncthreads();
  for (int w = ST / 2; w > 0; w >>= 1) {
    if (tid < w) red[tid] = fmax(red[tid], red[tid + w]);
    __syncthreads();
  }
  if (tid == 0) est_part[((int64_t)j * nQ + I) * nQ + J] = red[0];
}

size_t omega_wide_scratch_elems(int m, int s) { return (size_t)m * s * s; }

void launch_omega_wide(int k, int s, int ld, const double* Wk, const double* Wkm1, double* Wk1, const double* Hd,
                       const double* Bd, const double* Rc, double nu, double* rhs, double* est_part, hipStream_t st) {
  const int nj = k - 1;
  const int nQ = (s + 63) >> 6;
  kt_begin(KC_OMEGA, st);
  hipLaunchKernelGGL(omega_rhs_wide_kernel, dim3(nj, nQ, nQ), dim3(ST), 0, st, k, s, Wk, Wkm1, Hd, Bd, nu, rhs);
  GK_HIP(hipGetLastError());
  hipLaunchKernelGGL(omega_apply_wide_kernel, dim3(nj, nQ, nQ), dim3(ST), 0, st, s, ld, Rc, rhs, Wk1, est_part);
  GK_HIP(hipGetLastError());
  kt_end(st, 8.0 * 12 * nj * (double)s * s, 12.0 * nj * (double)s * s * s);
}

// ------------------------------------------------------ banded spline
// (eps I + H_m)^(-k) F_1 by block Cholesky of the block tridiagonal
// eps I + H_m (same factorisation as the 64-wide kernels):
//   A_j = eps I + H_jj - Lsub_{j-1} Lsub_{j-1}^T = L_jj L_jj^T,
//   Linv_j = L_jj^{-1},  Lsub_j = B_j Linv_j^T,
// then k forward / backward block substitutions.  Work layout (s x s each):
// Linv_0..m-1, Lsub_0..m-1, one factor scratch.
// A chain of launches per block: A_j, one lower tile a workgroup, the one of
// (0, 0) going on to factor it; the launches of WideFac; Lsub_j, one tile a
// workgroup.  The substitutions are two launches per block and direction, one
// tile a workgroup.  s = 512, 30 blocks, factor and k = 1 substitutions: 14 ms
// (in one workgroup and one per column tile: 99 + 23).
__global__ void __launch_bounds__(ST)
banded_a_kernel(WideFac f, const double* __restrict__ Hj, double eps, const double* __restrict__ Lp) {
  __shared__ __align__(16) double T0[WS][LP];
  __shared__ __align__(16) double T1[WS][LP];
  __shared__ __align__(16) double T2[WS][LP];
  const int nQ = (f.s + 63) >> 6;
  int J = blockIdx.x, I = 0;
  while (J > I) { J -= I + 1; ++I; }
  double t[4][4];
  tile_get(Hj, f.s, f.s, I, J, t);
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  if (I == J) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (acc_row(a) == acc_col(b)) t[a][b] += eps;
  }
  if (Lp) wterm(t, -1.0, Lp, f.s, false, Lp, f.s, true, f.s, I, J, 0, nQ, T0, T1);
  if (I > 0) {
    tile_put(f.A, f.ld, f.s, I, J, t);
    return;
  }
  __syncthreads();
  put_acc(T0, t);
  __syncthreads();
  for (int r = ty; r < 64; r += 16)   // zero beyond s, as the tile would be read back
    for (int c = tx; c < 64; c += 16)
      if (r >= f.s || c >= f.s) T0[r][c] = 0.0;
  wide_diag<0>(f, 0, T0, T1, T2);
}
__global__ void __launch_bounds__(ST) banded_col_kernel(WideFac f, int k) { wide_col_body<0>(f, k, blockIdx.x); }
__global__ void __launch_bounds__(ST) banded_last_kernel(WideFac f) { wide_last_body<true>(f, blockIdx.x); }
// out (I, J) = sum_{K <= J} B_IK (Linv^T)_KJ
__global__ void __launch_bounds__(ST)
banded_sub_kernel(int s, const double* __restrict__ B, const double* __restrict__ Li, double* __restrict__ out) {
  __shared__ __align__(16) double T0[WS][LP];
  __shared__ __align__(16) double T1[WS][LP];
  const int I = blockIdx.x, J = blockIdx.y;
  double t[4][4];
  zero44(t);
  wterm(t, 1.0, B, s, false, Li, s, true, s, I, J, 0, J + 1, T0, T1);
  tile_put(out, s, s, I, J, t);
}
// One step of the substitution
//   forward:  Z_j = Linv_j (Y_j - Lsub_{j-1} Z_{j-1})
//   backward: Y_j = Linv_j^T (Z_j - Lsub_j^T Y_{j+1}),  tile (I, J) = (blockIdx.x, blockIdx.y):
// out = add + sign sum_K op(X)_IK Y_KJ over K0 <= K < K1 (lower: K <= I,
// upper: K >= I); tr: op = transpose
__global__ void __launch_bounds__(ST)
banded_step_kernel(int s, const double* __restrict__ add, double sign, const double* __restrict__ X, int tr, int tri,
                   const double* __restrict__ Y, double* __restrict__ out) {
  __shared__ __align__(16) double SA[WS][LP];
  __shared__ __align__(16) double SB[WS][LP];
  const int I = blockIdx.x, J = blockIdx.y, nQ = (s + 63) >> 6;
  double t[4][4];
  if (add) tile_get(add, s, s, I, J, t);
  else zero44(t);
  if (X) wterm(t, sign, X, s, tr != 0, Y, s, false, s, I, J, tri == 2 ? I : 0, tri == 1 ? I + 1 : nQ, SA, SB);
  tile_put(out, s, s, I, J, t);
}
__global__ void banded_f1_kernel(int64_t tot, int s, double* __restrict__ U) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q < tot) U[q] = (q < (int64_t)s * s && q / s == q % s) ? 1.0 : 0.0;
}

size_t banded_wide_work_elems(int m, int s) { return (size_t)(2 * m + 2) * s * s; }

void launch_banded_spline_wide(int m, int s, const double* Hd, const double* Bd, double eps, int k, double* work,
                               double* U, int* bad, hipStream_t st) {
  const size_t ss = (size_t)s * s;
  const int nQ = (s + 63) >> 6;
  double* Linv = work;
  double* Lsub = work + m * ss;
  double* Aw = work + 2 * m * ss;
  double* T = Aw + ss;
  GK_REQUIRE(nQ >= 2 && nQ <= WQ_MAX, GK_EUNSUPPORTED, "banded spline: unsupported block width");
  kt_begin(KC_BANDED_FACTOR, st);
  for (int j = 0; j < m; ++j) {
    const WideFac f{Aw, Aw, Linv + j * ss, s, s, nullptr, 0.0, nullptr, bad, nullptr};
    hipLaunchKernelGGL(banded_a_kernel, dim3(nQ * (nQ + 1) / 2), dim3(ST), 0, st, f, Hd + j * ss, eps,
                       j > 0 ? (const double*)(Lsub + (j - 1) * ss) : nullptr);
    for (int q = 0; q + 1 < nQ; ++q)
      hipLaunchKernelGGL(banded_col_kernel, dim3(wide_col_tasks(nQ, q)), dim3(ST), 0, st, f, q);
    hipLaunchKernelGGL(banded_last_kernel, dim3(nQ * (nQ - 1) / 2), dim3(ST), 0, st, f);
    if (j + 1 < m)
      hipLaunchKernelGGL(banded_sub_kernel, dim3(nQ, nQ), dim3(ST), 0, st, s, Bd + j * ss, (const double*)f.Y,
                         Lsub + j * ss);
  }
  GK_HIP(hipGetLastError());
  kt_end(st, 8.0 * 4 * m * (double)ss, (double)m * ss * s * (2.0 + 1.0 / 3.0 + 1.0));
  kt_begin(KC_BANDED_SOLVE, st);
  hipLaunchKernelGGL(banded_f1_kernel, dim3((unsigned)((m * ss + 255) / 256)), dim3(256), 0, st, (int64_t)(m * ss), s,
                     U);
  const dim3 grid(nQ, nQ);
  for (int rep = 0; rep < k; ++rep) {
    for (int j = 0; j < m; ++j) {
      double* Uj = U + j * ss;
      if (j > 0)
        hipLaunchKernelGGL(banded_step_kernel, grid, dim3(ST), 0, st, s, (const double*)Uj, -1.0,
                           (const double*)(Lsub + (j - 1) * ss), 0, 0, (const double*)(Uj - ss), T);
      else
        hipLaunchKernelGGL(banded_step_kernel, grid, dim3(ST), 0, st, s, (const double*)Uj, 0.0,
                           (const double*)nullptr, 0, 0, (const double*)nullptr, T);
      hipLaunchKernelGGL(banded_step_kernel, grid, dim3(ST), 0, st, s, (const double*)nullptr, 1.0,
                         (const double*)(Linv + j * ss), 0, 1, (const double*)T, Uj);
    }
    for (int j = m - 1; j >= 0; --j) {
      double* Uj = U + j * ss;
      if (j + 1 < m)
        hipLaunchKernelGGL(banded_step_kernel, grid, dim3(ST), 0, st, s, (const double*)Uj, -1.0,
                           (const double*)(Lsub + j * ss), 1, 0, (const double*)(Uj + ss), T);
      else
        hipLaunchKernelGGL(banded_step_kernel, grid, dim3(ST), 0, st, s, (const double*)Uj, 0.0,
                           (const double*)nullptr, 0, 0, (const double*)nullptr, T);
      hipLaunchKernelGGL(banded_step_kernel, grid, dim3(ST), 0, st, s, (const double*)nullptr, 1.0,
                         (const double*)(Linv + j * ss), 1, 2, (const double*)T, Uj);
    }
  }
  GK_HIP(hipGetLastError());
  kt_end(st, 8.0 * 4 * 2 * k * m * (double)ss, 4.0 * 2 * k * m * (double)ss * s);
}

// ------------------------------------------------ Chebyshev series step
// One term of the series of exp(-t lam) applied to F_1 through the block
// tridiagonal H_m (blocks H_jj, sub-diagonal B_j = H_{j+1,j}):
//   out_j = alpha (B_{j-1} Y_{j-1} + H_jj Y_j + B_j^T Y_{j+1}) + beta Y_j + gamma Yp_j,
//   acc_j += coef[kk] out_j,
// one workgroup per 64 x 64 output tile (j, I, J) on the tile path above.
__global__ void __launch_bounds__(ST)
btd_cheb_tile_kernel(int m, int s, const double* __restrict__ Hd, const double* __restrict__ Bd,
                     const double* __restrict__ Y, const double* __restrict__ Yp, double* __restrict__ out,
                     double alpha, double beta, double gamma, double* __restrict__ acc,
                     const double* __restrict__ coef, int kk) {
  __shared__ __align__(16) double SA[WS][LP];
  __shared__ __align__(16) double SB[WS][LP];
  const int j = blockIdx.x, I = blockIdx.y, J = blockIdx.z;
  const int nQ = (s + 63) >> 6;
  const int64_t ss = (int64_t)s * s;
  double t[4][4];
  zero44(t);
  wterm(t, 1.0, Hd + j * ss, s, false, Y + j * ss, s, false, s, I, J, 0, nQ, SA, SB);
  if (j > 0) wterm(t, 1.0, Bd + (j - 1) * ss, s, false, Y + (j - 1) * ss, s, false, s, I, J, 0, nQ, SA, SB);
  if (j + 1 < m) wterm(t, 1.0, Bd + j * ss, s, true, Y + (j + 1) * ss, s, false, s, I, J, 0, nQ, SA, SB);
  double yv[4][4], pv[4][4], av[4][4];
  tile_get(Y + j * ss, s, s, I, J, yv);
  if (Yp) tile_get(Yp + j * ss, s, s, I, J, pv);
  else zero44(pv);
  tile_get(acc + j * ss, s, s, I, J, av);
  const double ck = coef[kk];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const double v = alpha * t[a][b] + beta * yv[a][b] + gamma * pv[a][b];
      t[a][b] = v;
      av[a][b] += ck * v;
    }
  tile_put(out + j * ss, s, s, I, J, t);
  tile_put(acc + j * ss, s, s, I, J, av);
}

void launch_btd_cheb_tile(int m, int s, const double* Hd, const double* Bd, const double* Y, const double* Yp,
                          double* out, double alpha, double beta, double gamma, double* acc, const double* coef,
                          int kk, hipStream_t st) {
  GK_REQUIRE(s <= WCOL, GK_EINVAL, "Chebyshev step: block width above 512");
  const int nQ = (s + 63) >> 6;
  hipLaunchKernelGGL(btd_cheb_tile_kernel, dim3(m, nQ, nQ), dim3(ST), 0, st, m, s, Hd, Bd, Y, Yp, out, alpha, beta,
                     gamma, acc, coef, kk);
  GK_HIP(hipGetLastError());
}

}  // namespace gk
