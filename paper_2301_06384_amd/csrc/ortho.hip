// Tall-skinny block products: Gram matrices A^T B, block updates X -= A C,
// kernel-column assembly [Q_1..Q_m] U, and the column-wise (Frobenius /
// sequential) variants.
//
// These realise the DOT and AXPY work of Table 1: H_kk = Q_k^T X (Alg. 1),
// the projections that keep the basis orthonormal (Sec. 3.1), the QR of X,
// tr(Q_k^T X) and ||X||_F (Alg. 2), and the final [Q_1..Q_m] U (Alg. 1, 2).
// A "block list" is nb equally shaped n x ld row-major blocks, float or
// double, seen as one n x (nb*ld) matrix.  All accumulation is float64.
// Reductions over rows are split in fixed chunks whose partial results are
// summed in a fixed order by a second kernel: no atomics, so results are
// bitwise reproducible and independent of other work on the device.
#include <type_traits>

#include "gk_internal.h"

namespace gk {

template <bool F32>
__device__ __forceinline__ double ldA(const void* base, int64_t off) {
  if (F32) return (double)static_cast<const float*>(base)[off];
  return static_cast<const double*>(base)[off];
}

// ------------------------------------------------------------------ Gram
constexpr int G_TA = 64, G_TB = 64, G_RS = 16;

template <bool F32>
__global__ void __launch_bounds__(256)
gram_kernel(int64_t n, int ld, const void* __restrict__ Abase, int64_t astride, int nb,
            const double* __restrict__ B, double* __restrict__ part, int64_t rows_per_chunk,
            const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  __shared__ double sA[G_RS][G_TA + 1];
  __shared__ double sB[G_RS][G_TB + 1];
  const int pa = nb * ld;
  const int a0 = blockIdx.x * G_TA;
  const int b0 = blockIdx.y * G_TB;
  const int64_t r_begin = (int64_t)blockIdx.z * rows_per_chunk;
  const int64_t r_end = min(n, r_begin + rows_per_chunk);
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  double acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;
  for (int64_t r0 = r_begin; r0 < r_end; r0 += G_RS) {
    for (int q = threadIdx.x; q < G_RS * G_TA; q += 256) {
      const int rr = q / G_TA, cc = q % G_TA;
      const int64_t r = r0 + rr;
      const int a = a0 + cc, b = b0 + cc;
      double va = 0.0, vb = 0.0;
      if (r < r_end) {
        if (a < pa) {
          const int blk = a / ld, col = a - blk * ld;
          va = ldA<F32>(Abase, (int64_t)blk * astride + r * ld + col);
        }
        if (b < ld) vb = B[r * ld + b];
      }
      sA[rr][cc] = va;
      sB[rr][cc] = vb;
    }
    __syncthreads();
#pragma unroll 4
    for (int rr = 0; rr < G_RS; ++rr) {
      double av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = sA[rr][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) bv[j] = sB[rr][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fma(av[i], bv[j], acc[i][j]);
    }
    __syncthreads();
  }
  double* P = part + (int64_t)blockIdx.z * pa * ld;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int a = a0 + ty * 4 + i, b = b0 + tx * 4 + j;
      if (a < pa && b < ld) P[(int64_t)a * ld + b] = acc[i][j];
    }
}

// The same sums at ld = 8, where 64-wide tiles are mostly padding: workgroup
// (four blocks, chunk), wavefront w forms block 4 blockIdx.x + w, one element
// a lane.  Each element is one chain of fma over the chunk's rows, as above
// (the same bits); rounds of G8_R rows in LDS, the next one in registers.
// Bound by that chain and the first loads.  24^3 grid, two blocks: 38 us on the
// 64-wide tiles, now 7.
constexpr int G8_R = 64;
template <bool F32>
__global__ void __launch_bounds__(256)
gram8_kernel(int64_t n, const void* __restrict__ Abase, int64_t astride, int nb, const double* __restrict__ B,
             double* __restrict__ part, int64_t rows_per_chunk, const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  __shared__ double sA[4][G8_R * 8];
  __shared__ double sB[G8_R * 8];
  const int64_t rb = (int64_t)blockIdx.y * rows_per_chunk, re = min(n, rb + rows_per_chunk);
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int blk = 4 * blockIdx.x + w;
  const bool on = blk < nb;
  // a wavefront stages its own block, and each a quarter of B
  double va[8], vb[2];
  auto fetch = [&](int64_t r0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = l + 64 * q;
      va[q] = (on && r0 + (e >> 3) < re) ? ldA<F32>(Abase, (int64_t)blk * astride + r0 * 8 + e) : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int e = tid + 256 * q;
      vb[q] = r0 + (e >> 3) < re ? B[r0 * 8 + e] : 0.0;
    }
  };
  double acc = 0.0;
  if (rb < re) fetch(rb);
  for (int64_t r0 = rb; r0 < re; r0 += G8_R) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) sA[w][l + 64 * q] = va[q];
#pragma unroll
    for (int q = 0; q < 2; ++q) sB[tid + 256 * q] = vb[q];
    __syncthreads();
    if (r0 + G8_R < re) fetch(r0 + G8_R);
    if (on) {
#pragma unroll 16
      for (int r = 0; r < G8_R; ++r) acc = fma(sA[w][8 * r + (l >> 3)], sB[8 * r + (l & 7)], acc);
    }
  }
  if (on) part[((int64_t)blockIdx.y * nb + blk) * 64 + l] = acc;
}

// out[i] = sum_{c < nparts} part[c*len + i] in a fixed order: block b owns
// outputs [16b, 16b+16); its 16 thread groups sum interleaved parts (eight
// running sums per thread, so eight loads are in flight, combined pairwise),
// then the 16 group sums are added in group order.  sym_ld > 0: the parts
// hold only the sym_t x sym_t tiles on and above the diagonal of a symmetric
// sym_ld x sym_ld matrix (sym_ld and sym_t multiples of 16, so a block's
// outputs lie in one row of one tile); blocks below the diagonal return at
// once and those above it also write the mirrored entries.
__global__ void __launch_bounds__(256)
reduce_parts_kernel(int64_t len, int nparts, const double* __restrict__ part, double* __restrict__ out,
                    const int* __restrict__ flag, int sym_ld, int sym_t) {
  if (flag && *flag == 0) return;
  __shared__ double red[16][17];
  const int o = threadIdx.x & 15, g = threadIdx.x >> 4;
  // groups of 16 outputs, taken in turn by the workgroups of a capped grid
  // (a gated launch that has nothing to do then dispatches few workgroups)
  const int64_t ngrp = (len + 15) / 16;
  for (int64_t gb = blockIdx.x; gb < ngrp; gb += gridDim.x) {
    const int64_t i = gb * 16 + o;
    const int64_t src = i;
    int64_t mirror = -1;
    if (sym_ld > 0) {
      const int64_t r = (gb * 16) / sym_ld, c = i - r * sym_ld;
      const int64_t tr = r / sym_t, tc = (gb * 16 - r * sym_ld) / sym_t;
      if (tr > tc) continue;   // the whole group: lower tiles come from their mirror
      if (tr < tc) mirror = c * sym_ld + r;
    }
    double s = 0.0;
    if (i < len) {
      double a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = 0.0;
      int c = g;
      for (; c + 16 * 7 < nparts; c += 16 * 8)
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] += part[(int64_t)(c + 16 * u) * len + src];
      for (; c < nparts; c += 16) a[0] += part[(int64_t)c * len + src];
      s = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    }
    red[g][o] = s;
    __syncthreads();
    if (g == 0 && i < len) {
      double t = 0.0;
      for (int q = 0; q < 16; ++q) t += red[q][o];
      out[i] = t;
      if (mirror >= 0) out[mirror] = t;
    }
    __syncthreads();
  }
}

void launch_reduce_parts(int64_t len, int nparts, const double* part, double* out, const int* flag, hipStream_t st,
                        int sym_ld, int sym_t) {
  // entries read per part: the whole vector, or the tiles on and above the diagonal
  double rd = (double)len;
  if (sym_ld > 0) {
    const double nt = sym_ld / sym_t;
    rd = nt * (nt + 1) / 2 * sym_t * sym_t;
  }
  kt_begin(KC_REDUCE, st);
  const int64_t ngrp = (len + 15) / 16;
  hipLaunchKernelGGL(reduce_parts_kernel, dim3((unsigned)std::min<int64_t>(ngrp, 1024)), dim3(256), 0, st, len, nparts,
                     part, out, flag, sym_ld, sym_t);
  GK_HIP(hipGetLastError());
  kt_end(st, 8.0 * (rd * nparts + len), rd * nparts, flag);
}

// Blocks 64 and wider use the FP64 matrix-core kernels below (rows staged
// 32 at a time, 64-wide output tiles); narrower ones the vector kernel above.
static bool mfma_ok(int ld) { return ld >= 64 && ld % 16 == 0; }
constexpr int MG_T = 64, MG_RS = 32;

static void gram_geometry(int64_t n, int nb, int ld, int* nx, int* ny, int* nch, int64_t* rpc) {
  const int rs = mfma_ok(ld) ? MG_RS : G_RS;
  const int pa = nb * ld;
  *nx = (pa + G_TA - 1) / G_TA;
  *ny = (ld + G_TB - 1) / G_TB;
  int64_t want = (2048 + (*nx) * (*ny) - 1) / ((*nx) * (*ny));
  int64_t maxc = (n + 255) / 256;
  if (want > maxc) want = maxc;
  if (want < 1) want = 1;
  if (want > 1024) want = 1024;
  // a multiple of 8 chunks, so that every XCD gets the same number of them
  // (the MFMA Gram kernels run each chunk's tiles on one XCD); chunks past
  // the last row are empty and contribute zero partials
  want = (want + 7) / 8 * 8;
  int64_t r = (n + want - 1) / want;
  r = ((r + rs - 1) / rs) * rs;
  *rpc = r;
  *nch = (int)want;
}

// Workgroup order of the MFMA tile kernels (one-dimensional grids).
// Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.
// Gram with the float32 archive (tiles nx x ny per row chunk): the nx ny tiles of chunk c are
// consecutive workgroups of XCD c % 8, so the rows of a chunk are fetched
// into one L2 and read there by all its tiles, not once per tile.
__device__ __forceinline__ void gram_tile(int nx, int ny, int& ta, int& tb, int& tc) {
  const unsigned L = blockIdx.x, x = L & 7, j = L >> 3, T = (unsigned)(nx * ny);
  const unsigned t = j % T;
  tc = (int)((j / T) * 8 + x);
  ta = (int)(t % (unsigned)nx);
  tb = (int)(t / (unsigned)nx);
}
// Row-tile products (row tiles x ny column tiles): the ny column tiles of
// row tile rt are consecutive workgroups of XCD rt % 8, so the rows they all
// read come from one L2.  False past the last row tile.
__device__ __forceinline__ bool row_tile(int64_t nrt, int ny, int64_t& rt, int& tb) {
  const unsigned L = blockIdx.x, x = L & 7, j = L >> 3;
  tb = (int)(j % (unsigned)ny);
  rt = (int64_t)(j / (unsigned)ny) * 8 + x;
  return rt < nrt;
}
static inline unsigned row_tile_grid(int64_t nrt, int ny) { return (unsigned)(8 * ((nrt + 7) / 8) * ny); }

size_t gram_scratch_elems(int64_t n, int nb, int ld) {
  int nx, ny, nch;
  int64_t rpc;
  gram_geometry(n, nb, ld, &nx, &ny, &nch, &rpc);
  return (size_t)nch * nb * ld * ld;
}

// ------------------------------------------- FP64 matrix-core Gram / update
typedef double d4v __attribute__((ext_vector_type(4)));

// Eight consecutive elements (16-byte aligned) held as loaded: the float to
// double conversion happens only when they are stored to LDS, so a prefetch
// does not wait for its own loads.
template <bool F32>
struct Raw8 {
  float4 f[2];
  __device__ __forceinline__ void load(const void* __restrict__ base, int64_t off) {
    const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(base) + off);
    f[0] = p[0];
    f[1] = p[1];
  }
  __device__ __forceinline__ void zero() { f[0] = f[1] = make_float4(0.f, 0.f, 0.f, 0.f); }
  __device__ __forceinline__ double get(int q) const {
    const float4& t = f[q >> 2];
    const int e = q & 3;
    return (double)(e == 0 ? t.x : e == 1 ? t.y : e == 2 ? t.z : t.w);
  }
};
template <>
struct Raw8<false> {
  double2 d[4];
  __device__ __forceinline__ void load(const void* __restrict__ base, int64_t off) {
    const double2* p = reinterpret_cast<const double2*>(static_cast<const double*>(base) + off);
#pragma unroll
    for (int q = 0; q < 4; ++q) d[q] = p[q];
  }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int q = 0; q < 4; ++q) d[q] = make_double2(0.0, 0.0);
  }
  __device__ __forceinline__ double get(int q) const { return (q & 1) ? d[q >> 1].y : d[q >> 1].x; }
};

// Assembly P[perm(r), c] = sum_a A[r, a] U[a, c] (c < ncols) from a float64
// basis, one 64-row x 64-column tile per workgroup, 32 contraction indices
// per stage; A is staged transposed so both operands are read along their
// contiguous LDS rows.  Column-major output (leading dimension ldo) written
// through an LDS transpose.
constexpr int MT_R = 64, MT_C = 64, MT_K = 32;
// The transposed staging writes contraction index k of tile row r at column
// (r + tsw(k)) mod 64 of LDS row k.  One store instruction writes rows
// k = 8 g + q (g = 0..3 by lane, q fixed): unrotated, the four g fell on the
// same banks.  LDS serves 32-bit accesses 32 lanes at a time and 64-bit ones
// 16 lanes at a time over 32 four-byte banks, so floats are rotated by 8 g
// columns and doubles by 4 g, which spreads each group over all banks.  The
// product loop reads four consecutive k at once, which share one rotation.
template <typename T>
__device__ __forceinline__ int tsw(int k) { return (sizeof(T) == 8 ? 4 : 8) * ((k >> 3) & 3); }
// Coefficient staging: lane j of a row's 8 holds the elements q = 0..7 at
// columns cpos(j, q), pairs 16 columns apart, so each pair-wide load or
// store instruction of the 8 lanes covers one contiguous stretch of the row.
__device__ __forceinline__ int cpos(int j, int q) { return 2 * j + 16 * (q >> 1) + (q & 1); }
__global__ void __launch_bounds__(256)
assemble_mfma_kernel(int64_t n, int ld, const double* __restrict__ Abase, int64_t astride, int nb,
                     const double* __restrict__ C, int ldc, int ncols, double* __restrict__ out, int64_t ldo,
                     const int64_t* __restrict__ perm) {
  __shared__ __align__(16) double sAT[MT_K][MT_R + 2];
  __shared__ __align__(16) double sC[MT_K][MT_C + 2];
  __shared__ double sO[MT_C][MT_R + 1];
  const int pa = nb * ld;
  int64_t rt;
  int tb;
  if (!row_tile((n + MT_R - 1) / MT_R, (ncols + MT_C - 1) / MT_C, rt, tb)) return;
  const int64_t r0 = rt * MT_R;
  const int b0 = tb * MT_C;
  const int tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const int wr = 32 * (w >> 1), wc = 32 * (w & 1);
  const int ar = tid >> 2, ak = 8 * (tid & 3);     // A staging: row, 8 contraction indices
  const int cr = tid >> 3, cj = tid & 7;           // C staging: row, lane of the row (columns cpos)
  const int64_t arow = r0 + ar;
  double vcs[8];   // scalar coefficient loads (ldc need not be even)
  d4v acc[2][2];
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj) acc[ti][tj] = d4v{0.0, 0.0, 0.0, 0.0};
  Raw8<false> va;
  auto fetch = [&](int a0) {
    const int ga = a0 + ak;
    if (arow < n && ga < pa) {
      const int blk = ga / ld;
      va.load(Abase, (int64_t)blk * astride + arow * ld + (ga - blk * ld));
    } else {
      va.zero();
    }
    const int gc = a0 + cr;
    const int gcc = gc < pa ? gc : pa - 1;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int col = b0 + cpos(cj, q);
      vcs[q] = C[(int64_t)gcc * ldc + (col < ncols ? col : ncols - 1)];
    }
  };
  fetch(0);
  for (int a0 = 0; a0 < pa; a0 += MT_K) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) sAT[ak + q][(ar + tsw<double>(ak)) & 63] = va.get(q);
    const bool rin = a0 + cr < pa;
#pragma unroll
    for (int q = 0; q < 8; ++q) sC[cr][cpos(cj, q)] = (rin && b0 + cpos(cj, q) < ncols) ? vcs[q] : 0.0;
    __syncthreads();
    if (a0 + MT_K < pa) fetch(a0 + MT_K);
#pragma unroll
    for (int ks = 0; ks < MT_K / 4; ++ks) {
      double av[2], bv[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        av[t] = sAT[4 * ks + lk][(wr + 16 * t + li + tsw<double>(4 * ks)) & 63];
        bv[t] = sC[4 * ks + lk][wc + 16 * t + li];
      }
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
          acc[ti][tj] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[ti], bv[tj], acc[ti][tj], 0, 0, 0);
    }
  }
  // transpose through LDS: each column is then written as contiguous rows
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj)
#pragma unroll
      for (int q = 0; q < 4; ++q) sO[wc + 16 * tj + li][wr + 16 * ti + 4 * q + lk] = acc[ti][tj][q];
  __syncthreads();
  for (int q = tid; q < MT_C * MT_R; q += 256) {
    const int cc2 = q / MT_R, rr = q - cc2 * MT_R;
    const int64_t r = r0 + rr;
    const int b = b0 + cc2;
    if (r < n && b < ncols) out[(int64_t)b * ldo + (perm ? perm[r] : r)] = sO[cc2][rr];
  }
}

// ---------------------------- FP32 matrix-core products with the archive
// The float32 basis archive against a float64 block (reorthogonalisation
// coefficients C = Q^T X and the update X -= Q C), on v_mfma_f32_16x16x4f32:
// the coefficients only need the accuracy of the archive itself (unit
// roundoff 2^-24 relative to |Q||X|), so X and C are rounded to float in
// LDS, and the float accumulators are added into float64 every 32 terms.
// Same tiles as the FP64 kernels above; operand layout of the float MFMA:
// lane l = i + 16 k holds A[i][k] and B[k][i], accumulator register r holds
// D[4 k + r][i].  LDS pitch 80 floats (16 mod 32): the four 16-lane rows of
// an operand read fall in distinct bank halves.
typedef float f4v __attribute__((ext_vector_type(4)));
constexpr int FP = 80;

// 64 archive columns x 128 columns of X per workgroup of 8 wavefronts (wave w
// owns the 32 x 32 part (w % 2, w / 2)), X already rounded to float (X32).  The vector ALU does not run beside these matrix instructions: what
// the products alone do at 145 TFLOP/s fell to 126 with the float64 sums and
// to 96 with the staging through registers (300k x 256, 28 blocks).  So rounds
// of 32 rows go from memory straight to LDS (two buffers, one barrier a round,
// the next round in flight during the products) at addresses that advance in
// scalar registers.  Rows are contiguous in LDS; the 16-byte chunks of row r are
// permuted by chunk ^ 4 (r % 4), so that the four rows of an operand read fall
// in distinct banks.  Columns past the tile's matrices read the last ones; they
// only reach results that are not stored.  Rows past the range are zeroed.
// 300k x 256, 28 blocks: 11.5 ms staged through registers, 10.1 now with the
// rounding pass (109 TFLOP/s); 128 x 128 tiles 12.9 (three wavefronts a SIMD).
constexpr int MG_TB2 = 128;
__global__ void __launch_bounds__(512, 2)
gram_f32mma_kernel(int64_t n, int ld, const float* __restrict__ Abase, int64_t astride, int nb,
                   const float* __restrict__ X32, double* __restrict__ part, int64_t rows_per_chunk,
                   const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  constexpr int TA = MG_T;
  __shared__ __align__(16) float sA[2][MG_RS * TA];
  __shared__ __align__(16) float sB[2][MG_RS * MG_TB2];
  const int pa = nb * ld;
  int ta, tb, tc;
  gram_tile((pa + TA - 1) / TA, (ld + MG_TB2 - 1) / MG_TB2, ta, tb, tc);
  const int a0 = ta * TA, b0 = tb * MG_TB2;
  const int64_t rb = (int64_t)tc * rows_per_chunk;
  const int64_t re = min(n, rb + rows_per_chunk);
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, li = l & 15, lk = l >> 4;
  const int wa = 32 * (w & 1), wb = 32 * (w >> 1);
  // a load of a wavefront fills 256 consecutive floats of LDS: one a round of
  // A (row rA of its lanes, column oA), two of X
  constexpr int RA = 256 / TA, RB = 256 / MG_TB2;   // rows a load covers
  int rB[2];
  int64_t oB[2];
  const int rA = RA * w + l / (TA / 4);
  const int ga = min(a0 + 4 * ((l % (TA / 4)) ^ (4 * (rA & 3))), pa - 4), gblk = ga / ld;
  const int64_t oA = (int64_t)gblk * astride + (ga - gblk * ld);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    rB[q] = RB * (w + 8 * q) + l / (MG_TB2 / 4);
    oB[q] = min(b0 + 4 * ((l % (MG_TB2 / 4)) ^ (4 * (rB[q] & 3))), ld - 4);
  }
  auto put = [&](const float* a, float* lds) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)a,
                                     (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
  };
  // the barrier before a buffer is read: loads to LDS are counted with the
  // wavefront's memory loads, which a barrier alone does not wait for
  auto landed = [&]() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  // rows r0 .. of full rounds; of the last one when fewer are left, its rows
  // past the range read the last row
  auto load = [&](int64_t r0, int p) {
    if (r0 + MG_RS <= re) {
      const float* A0 = Abase + r0 * ld;
      const float* B0 = X32 + r0 * ld;
      put(A0 + (oA + rA * ld), &sA[p][256 * w]);
#pragma unroll
      for (int q = 0; q < 2; ++q) put(B0 + (oB[q] + rB[q] * ld), &sB[p][256 * (w + 8 * q)]);
    } else {
      put(Abase + oA + min(r0 + rA, re - 1) * ld, &sA[p][256 * w]);
#pragma unroll
      for (int q = 0; q < 2; ++q) put(X32 + oB[q] + min(r0 + rB[q], re - 1) * ld, &sB[p][256 * (w + 8 * q)]);
    }
  };
  int xa[2], xb[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) xa[t] = lk * TA + ((wa + 16 * t + li) ^ (16 * lk));
#pragma unroll
  for (int t = 0; t < 2; ++t) xb[t] = lk * MG_TB2 + ((wb + 16 * t + li) ^ (16 * lk));
  double a64[2][2][4];
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj)
#pragma unroll
      for (int q = 0; q < 4; ++q) a64[ti][tj][q] = 0.0;
  if (rb < re) load(rb, 0);
  landed();
  int p = 0;
  for (int64_t r0 = rb; r0 < re; r0 += MG_RS) {
    if (r0 + MG_RS < re) {
      load(r0 + MG_RS, p ^ 1);
    } else if (r0 + MG_RS > re) {
      const int have = (int)(re - r0);
      for (int q = tid; q < (MG_RS - have) * TA; q += 512) sA[p][have * TA + q] = 0.f;
      for (int q = tid; q < (MG_RS - have) * MG_TB2; q += 512) sB[p][have * MG_TB2 + q] = 0.f;
      __syncthreads();
    }
    f4v acc[2][2];
    const float* A = sA[p];
    const float* B = sB[p];
#pragma unroll
    for (int ks = 0; ks < MG_RS / 4; ++ks) {
      float av[2], bv[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        av[t] = A[xa[t] + 4 * ks * TA];
        bv[t] = B[xb[t] + 4 * ks * MG_TB2];
      }
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
          acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(
              av[ti], bv[tj], ks == 0 ? f4v{0.f, 0.f, 0.f, 0.f} : acc[ti][tj], 0, 0, 0);
    }
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int tj = 0; tj < 2; ++tj)
#pragma unroll
        for (int q = 0; q < 4; ++q) a64[ti][tj][q] += (double)acc[ti][tj][q];
    landed();
    p ^= 1;
  }
  double* P = part + (int64_t)tc * pa * ld;
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int a = a0 + wa + 16 * ti + 4 * lk + q, b = b0 + wb + 16 * tj + li;
        if (a < pa && b < ld) P[(int64_t)a * ld + b] = a64[ti][tj][q];
      }
}

__global__ void round_kernel(int64_t quads, const double* __restrict__ X, float* __restrict__ X32,
                             const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < quads; q += step) {
    const double2 a = reinterpret_cast<const double2*>(X)[2 * q], b = reinterpret_cast<const double2*>(X)[2 * q + 1];
    reinterpret_cast<float4*>(X32)[q] = make_float4((float)a.x, (float)a.y, (float)b.x, (float)b.y);
  }
}

// out[r, b] = beta in[r, b] + alpha sum_a Q[r, a] C[a, b] (row-major, ld
// columns), one 64-row x 64-column tile per workgroup, 32 contraction
// indices per stage (the archive rows staged transposed).
__global__ void __launch_bounds__(256)
tsgemm_f32mma_kernel(int64_t n, int ld, const float* __restrict__ Abase, int64_t astride, int nb,
                     const double* __restrict__ C, const double* __restrict__ in, double* __restrict__ out,
                     double alpha, double beta, const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  __shared__ __align__(16) float sAT[MT_K][FP];
  __shared__ __align__(16) float sC[MT_K][FP];
  const int pa = nb * ld;
  int64_t rt;
  int tb;
  if (!row_tile((n + MT_R - 1) / MT_R, (ld + MT_C - 1) / MT_C, rt, tb)) return;
  const int64_t r0 = rt * MT_R;
  const int b0 = tb * MT_C;
  const int tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const int wr = 32 * (w >> 1), wc = 32 * (w & 1);
  const int ar = tid >> 2, ak = 8 * (tid & 3);     // archive staging: row, 8 contraction indices
  const int cr = tid >> 3, cj = tid & 7;           // coefficient staging: row, lane of the row
  const int64_t arow = r0 + ar;
  f4v acc[2][2];
  double a64[2][2][4];
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj) {
      acc[ti][tj] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 4; ++q) a64[ti][tj][q] = 0.0;
    }
  Raw8<true> va;
  double2 vcp[4];
  auto fetch = [&](int a0) {
    const int ga = a0 + ak;
    if (arow < n && ga < pa) {
      const int blk = ga / ld;
      va.load(Abase, (int64_t)blk * astride + arow * ld + (ga - blk * ld));
    } else {
      va.zero();
    }
    const int gc = a0 + cr;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = b0 + 2 * cj + 16 * q;
      vcp[q] = (gc < pa && col < ld) ? *reinterpret_cast<const double2*>(C + (int64_t)gc * ld + col)
                                     : make_double2(0.0, 0.0);
    }
  };
  fetch(0);
  for (int a0 = 0; a0 < pa; a0 += MT_K) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) sAT[ak + q][(ar + tsw<float>(ak)) & 63] = (float)va.get(q);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float2*>(&sC[cr][2 * cj + 16 * q]) = make_float2((float)vcp[q].x, (float)vcp[q].y);
    __syncthreads();
    if (a0 + MT_K < pa) fetch(a0 + MT_K);
#pragma unroll
    for (int ks = 0; ks < MT_K / 4; ++ks) {
      float av[2], bv[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        av[t] = sAT[4 * ks + lk][(wr + 16 * t + li + tsw<float>(4 * ks)) & 63];
        bv[t] = sC[4 * ks + lk][wc + 16 * t + li];
      }
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
          acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[ti], bv[tj], acc[ti][tj], 0, 0, 0);
    }
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int tj = 0; tj < 2; ++tj) {
#pragma unroll
        for (int q = 0; q < 4; ++q) a64[ti][tj][q] += (double)acc[ti][tj][q];
        acc[ti][tj] = f4v{0.f, 0.f, 0.f, 0.f};
      }
  }
  // the 16 `in` values of this thread are loaded together (rows and columns
  // out of range read element 0 and are not stored)
  double inv[2][2][4];
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t r = r0 + wr + 16 * ti + 4 * lk + q;
        const int b = b0 + wc + 16 * tj + li;
        inv[ti][tj][q] = (beta != 0.0) ? in[(r < n && b < ld) ? r * ld + b : 0] : 0.0;
      }
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int64_t r = r0 + wr + 16 * ti + 4 * lk + q;
        const int b = b0 + wc + 16 * tj + li;
        if (r < n && b < ld) out[r * ld + b] = alpha * a64[ti][tj][q] + beta * inv[ti][tj][q];
      }
}

// Assembly P[perm(r), c] = sum_a Q[r, a] U[a, c] (c < ncols) from the
// float32 archive on FP32 matrix cores, U rounded to float (the accuracy of
// the archive itself, as for the 64-wide assembly of arch.hip); float
// accumulators added into float64 after every 32 contraction indices;
// column-major output (leading dimension ldo) written through an LDS
// transpose, each column as contiguous rows.
__global__ void __launch_bounds__(256)
assemble_f32mma_kernel(int64_t n, int ld, const float* __restrict__ Abase, int64_t astride, int nb,
                       const double* __restrict__ U, int ldu, int ncols, double* __restrict__ out, int64_t ldo,
                       const int64_t* __restrict__ perm) {
  __shared__ __align__(16) float sAT[MT_K][FP];
  __shared__ __align__(16) float sC[MT_K][FP];
  __shared__ double sO[MT_C][MT_R + 1];
  const int pa = nb * ld;
  int64_t rt;
  int tb;
  if (!row_tile((n + MT_R - 1) / MT_R, (ncols + MT_C - 1) / MT_C, rt, tb)) return;
  const int64_t r0 = rt * MT_R;
  const int b0 = tb * MT_C;
  const int tid = threadIdx.x;
  const int w = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
  const int wr = 32 * (w >> 1), wc = 32 * (w & 1);
  const int ar = tid >> 2, ak = 8 * (tid & 3);     // archive staging: row, 8 contraction indices
  const int cr = tid >> 3, cj = tid & 7;           // coefficient staging: row, lane of the row
  const int64_t arow = r0 + ar;
  f4v acc[2][2];
  double a64[2][2][4];
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj) {
      acc[ti][tj] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 4; ++q) a64[ti][tj][q] = 0.0;
    }
  Raw8<true> va;
  double vcs[8];   // scalar coefficient loads (ldu need not be even)
  auto fetch = [&](int a0) {
    const int ga = a0 + ak;
    if (arow < n && ga < pa) {
      const int blk = ga / ld;
      va.load(Abase, (int64_t)blk * astride + arow * ld + (ga - blk * ld));
    } else {
      va.zero();
    }
    const int gc = a0 + cr;
    const int gcc = gc < pa ? gc : pa - 1;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int col = b0 + cpos(cj, q);
      vcs[q] = U[(int64_t)gcc * ldu + (col < ncols ? col : ncols - 1)];
    }
  };
  fetch(0);
  for (int a0 = 0; a0 < pa; a0 += MT_K) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) sAT[ak + q][(ar + tsw<float>(ak)) & 63] = (float)va.get(q);
    {
      const bool rin = a0 + cr < pa;
#pragma unroll
      for (int q = 0; q < 8; ++q) sC[cr][cpos(cj, q)] = (rin && b0 + cpos(cj, q) < ncols) ? (float)vcs[q] : 0.f;
    }
    __syncthreads();
    if (a0 + MT_K < pa) fetch(a0 + MT_K);
#pragma unroll
    for (int ks = 0; ks < MT_K / 4; ++ks) {
      float av[2], bv[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        av[t] = sAT[4 * ks + lk][(wr + 16 * t + li + tsw<float>(4 * ks)) & 63];
        bv[t] = sC[4 * ks + lk][wc + 16 * t + li];
      }
#pragma unroll
      for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
          acc[ti][tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[ti], bv[tj], acc[ti][tj], 0, 0, 0);
    }
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
      for (int tj = 0; tj < 2; ++tj) {
#pragma unroll
        for (int q = 0; q < 4; ++q) a64[ti][tj][q] += (double)acc[ti][tj][q];
        acc[ti][tj] = f4v{0.f, 0.f, 0.f, 0.f};
      }
  }
  // D[4 k + r][i]: row wr + 16 ti + 4 lk + r, column wc + 16 tj + li
#pragma unroll
  for (int ti = 0; ti < 2; ++ti)
#pragma unroll
    for (int tj = 0; tj < 2; ++tj)
#pragma unroll
      for (int q = 0; q < 4; ++q) sO[wc + 16 * tj + li][wr + 16 * ti + 4 * lk + q] = a64[ti][tj][q];
  __syncthreads();
  for (int q = tid; q < MT_C * MT_R; q += 256) {
    const int cc2 = q / MT_R, rr = q - cc2 * MT_R;
    const int64_t r = r0 + rr;
    const int b = b0 + cc2;
    if (r < n && b < ncols) out[(int64_t)b * ldo + (perm ? perm[r] : r)] = sO[cc2][rr];
  }
}

void launch_gram(int64_t n, int ld, BlockList A, const double* B, double* C, double* part,
                 const int* flag, hipStream_t st, float* x32) {
  int nx, ny, nch;
  int64_t rpc;
  gram_geometry(n, A.nb, ld, &nx, &ny, &nch, &rpc);
  dim3 grid(nx, ny, nch);
  // the Gram of a block with itself: only the tiles on and above the diagonal
  // are formed
  const bool self_gram = A.nb == 1 && !A.f32 && A.base == (const void*)B;
  const bool sym = mfma_ok(ld) && self_gram;
  // the float32 archive (reorthogonalisation coefficients) on the FP32
  // matrix cores
  const bool f32mma = mfma_ok(ld) && A.f32;
  kt_begin(f32mma ? KC_ARCH_GRAM : KC_GRAM, st);
  if (f32mma) {   // the chunk count of the 64 x 64 geometry
    GK_REQUIRE(x32 && ld % 16 == 0 && A.nb >= 1 && n >= 1 && rpc % MG_RS == 0 && rpc * nch >= n, GK_EUNSUPPORTED,
               "float32 Gram: unsupported block shape");
    hipLaunchKernelGGL(round_kernel, dim3((unsigned)std::min<int64_t>((n * ld / 4 + 255) / 256, 4096)), dim3(256), 0, st,
                       n * ld / 4, B, x32, flag);
    const int ny2 = (ld + MG_TB2 - 1) / MG_TB2, pa = A.nb * ld;
    hipLaunchKernelGGL(gram_f32mma_kernel, dim3((unsigned)((pa + MG_T - 1) / MG_T * ny2 * nch)), dim3(512), 0, st, n, ld,
                       (const float*)A.base, A.stride, A.nb, (const float*)x32, part, rpc, flag);
  }
  else if (mfma_ok(ld))
    launch_gram64(n, ld, A, B, part, nch, rpc, sym, flag, st);
  else if (ld == 8 && A.f32)
    hipLaunchKernelGGL(gram8_kernel<true>, dim3((A.nb + 3) / 4, nch), dim3(256), 0, st, n, A.base, A.stride, A.nb, B,
                       part, rpc, flag);
  else if (ld == 8)
    hipLaunchKernelGGL(gram8_kernel<false>, dim3((A.nb + 3) / 4, nch), dim3(256), 0, st, n, A.base, A.stride, A.nb, B,
                       part, rpc, flag);
  else if (A.f32)
    hipLaunchKernelGGL(gram_kernel<true>, grid, dim3(256), 0, st, n, ld, A.base, A.stride, A.nb, B,
                       part, rpc, flag);
  else
    hipLaunchKernelGGL(gram_kernel<false>, grid, dim3(256), 0, st, n, ld, A.base, A.stride, A.nb, B,
                       part, rpc, flag);
  GK_HIP(hipGetLastError());
  // method's own work: the Gram of a block with itself reads it once and
  // forms one triangle
  kt_end(st, self_gram ? 8.0 * n * ld : (double)n * ld * ((A.f32 ? 4.0 : 8.0) * A.nb + 8.0),
         self_gram ? (double)n * ld * (ld + 1) : 2.0 * (double)n * ld * ld * A.nb, flag);
  launch_reduce_parts((int64_t)A.nb * ld * ld, nch, part, C, flag, st, sym ? ld : 0, 16);
}

// Does the projection X1 = X - Q C have to be repeated?  Not when it took
// away at most 1e-8 of every column of X1 (G: the Gram matrix of X1): what it
// leaves along the basis is (I - Q^T Q) C, below the rounding of X1 itself,
// which a second projection has as well.  So a step that passes this test is as
// orthogonal as one that projects twice, whatever its place in the call and the
// width of its block, and every float64 step takes it, with one local pass ahead.
// The columns then differ from those of two projections by roundings.  Where
// the method amplifies roundings (columns not converged yet), by as much as two
// projections change when the nodes are renumbered: geometric graphs, spline, of
// the columns' norm, largest over the sample sets, renumbered | once:
//   100k, s = 64: m = 40 (100 sets) 1.6e-10 | 2.1e-10, m = 80 7.3e-5 | 7.3e-5
//   100k, m = 60..200: s = 48 1.7e-7 | 1.6e-7, 16 1.3e-4 | 1e-4, 1 6.6e-7 | 5.4e-7
//   50k, s = 20: sbl m = 80 6.2e-8 | 7.7e-8, gbl m = 150 6.6e-6 | 3.2e-6
// with the same distance to phi(L) in all digits shown (2.8e-5 to 0.75).  Against
// the method in extended precision, twice, renumbered | once: the set of the first
// line that moved most 8.1e-10, 7.2e-10 | 1.4e-10; 20k, s = 64, m = 80 1.4e-8,
// 1.9e-8 | 1.6e-8; 20k, s = 16, m = 100 2.8e-5, 3.1e-5 | 2.9e-5.
// 100k, s = 64, m = 40: 70.6 ms a call twice, 40.1 so.  Workgroup (j, y): block j,
// columns 16 y ..; a column not known to be small (NaN too) sets the flag, which
// the caller has cleared.
__global__ void __launch_bounds__(256)
again_kernel(int nb, int ld, int s, const double* __restrict__ C, const double* __restrict__ G, int* __restrict__ flag) {
  __shared__ double red[256];
  const int t = threadIdx.x, c = blockIdx.y * 16 + (t & 15);
  const double* Cj = C + (int64_t)blockIdx.x * ld * ld;
  double v = 0.0;
  if (c < s)
    for (int r = t >> 4; r < s; r += 16) v = fma(Cj[(int64_t)r * ld + c], Cj[(int64_t)r * ld + c], v);
  red[t] = v;
  __syncthreads();
  if (t < 16 && c < s) {
    double sum = 0.0;
    for (int q = 0; q < 16; ++q) sum += red[16 * q + t];
    if (!(sum * nb <= 1e-16 * G[(int64_t)c * ld + c])) *flag = 1;
  }
}

void launch_again(int nb, int ld, int s, const double* C, const double* G, int* flag, hipStream_t st) {
  hipLaunchKernelGGL(again_kernel, dim3(nb, (s + 15) / 16), dim3(256), 0, st, nb, ld, s, C, G, flag);
  GK_HIP(hipGetLastError());
}

// ------------------------------------------------------- tall-skinny GEMM
constexpr int T_TR = 64, T_TB = 64, T_KS = 16;

// out[r,b] = beta*in[r,b] + alpha*sum_a A[r,a] C[a,b]   (b < ncols)
// row-major output (ld) or column-major output (ld_out rows, optional perm)
template <bool F32, bool COLMAJ>
__global__ void __launch_bounds__(256)
tsgemm_kernel(int64_t n, int ld, int ncols, const void* __restrict__ Abase, int64_t astride, int nb,
              const double* __restrict__ C, int ldc, const double* __restrict__ in,
              double* __restrict__ out, float* __restrict__ out32, double alpha, double beta,
              int64_t ldo, const int64_t* __restrict__ perm, const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  __shared__ double sA[T_TR][T_KS + 1];
  __shared__ double sC[T_KS][T_TB + 1];
  const int pa = nb * ld;
  const int64_t r0 = (int64_t)blockIdx.x * T_TR;
  const int b0 = blockIdx.y * T_TB;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  double acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.0;
  for (int a0 = 0; a0 < pa; a0 += T_KS) {
    for (int q = threadIdx.x; q < T_TR * T_KS; q += 256) {
      const int rr = q / T_KS, kk = q % T_KS;
      const int64_t r = r0 + rr;
      const int a = a0 + kk;
      double v = 0.0;
      if (r < n && a < pa) {
        const int blk = a / ld, col = a - blk * ld;
        v = ldA<F32>(Abase, (int64_t)blk * astride + r * ld + col);
      }
      sA[rr][kk] = v;
    }
    for (int q = threadIdx.x; q < T_KS * T_TB; q += 256) {
      const int kk = q / T_TB, cc = q % T_TB;
      const int a = a0 + kk, b = b0 + cc;
      sC[kk][cc] = (a < pa && b < ncols) ? C[(int64_t)a * ldc + b] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < T_KS; ++kk) {
      double av[4], cv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) av[i] = sA[ty * 4 + i][kk];
#pragma unroll
      for (int j = 0; j < 4; ++j) cv[j] = sC[kk][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fma(av[i], cv[j], acc[i][j]);
    }
    __syncthreads();
  }
  if (!COLMAJ) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t r = r0 + ty * 4 + i;
      if (r >= n) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int b = b0 + tx * 4 + j;
        if (b >= ld) continue;
        double v = alpha * acc[i][j];
        if (beta != 0.0) v += beta * in[r * ld + b];
        if (b >= ncols) v = (beta != 0.0) ? beta * in[r * ld + b] : 0.0;
        out[r * ld + b] = v;
        if (out32) out32[r * ld + b] = (float)v;
      }
    }
  } else {
    // stage through LDS so that each column is written as contiguous rows
    __shared__ double sO[T_TB][T_TR + 1];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) sO[tx * 4 + j][ty * 4 + i] = alpha * acc[i][j];
    __syncthreads();
    for (int q = threadIdx.x; q < T_TB * T_TR; q += 256) {
      const int cc = q / T_TR, rr = q % T_TR;
      const int64_t r = r0 + rr;
      const int b = b0 + cc;
      if (r < n && b < ncols) {
        const int64_t orow = perm ? perm[r] : r;
        out[(int64_t)b * ldo + orow] = sO[cc][rr];
      }
    }
  }
}

// The update at ld = 8 against one or two float64 blocks: an element of the
// result a lane, its column of the coefficients in registers, rows a grid stride
// apart.  The sums of tsgemm_kernel (contraction index ascending, the same
// bits), without its 64-wide tiles.  Bound by the blocks it moves.  24^3 grid,
// two blocks: 6.9 -> 4.0 us; 300k nodes, s = 1, m = 30: 13.4 -> 5.1 ms a call with
// gram8_kernel.
template <int NB>
__global__ void __launch_bounds__(256)
update8_kernel(int64_t n, const double* Abase, int64_t astride, const double* __restrict__ C, const double* in,
               double* out, float* __restrict__ out32, double alpha, double beta, const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  const int c = threadIdx.x & 7;
  double cc[NB][8];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int k = 0; k < 8; ++k) cc[j][k] = C[j * 64 + k * 8 + c];
  const int64_t step = (int64_t)gridDim.x * 32;
  for (int64_t r = (int64_t)blockIdx.x * 32 + (threadIdx.x >> 3); r < n; r += step) {
    double a[NB][8];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double2 v = *reinterpret_cast<const double2*>(Abase + (int64_t)j * astride + r * 8 + 2 * k);
        a[j][2 * k] = v.x;
        a[j][2 * k + 1] = v.y;
      }
    const double iv = beta != 0.0 ? in[r * 8 + c] : 0.0;
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int k = 0; k < 8; ++k) acc = fma(a[j][k], cc[j][k], acc);
    double v = alpha * acc;
    if (beta != 0.0) v += beta * iv;
    out[r * 8 + c] = v;
    if (out32) out32[r * 8 + c] = (float)v;
  }
}

void launch_tsgemm(int64_t n, int ld, BlockList A, const double* C, const double* in, double* out,
                   float* out32, double alpha, double beta, const int* flag, hipStream_t st, bool upper,
                   bool tri0) {
  const int up = (upper && A.nb == 1) ? 1 : 0;
  // X -= A C against the float32 archive at widths 64 k: BF16 matrix cores
  if (A.f32 && !up && !out32 && !tri0 && in == out && alpha == -1.0 && beta == 1.0 && update_bf3_ok(ld)) {
    launch_update_bf3(n, ld, A, C, out, flag, st);
    return;
  }
  dim3 grid((unsigned)((n + T_TR - 1) / T_TR), (ld + T_TB - 1) / T_TB);
  // the float32 archive (reorthogonalisation update) on the FP32 matrix
  // cores
  const bool f32mma = mfma_ok(ld) && A.f32;
  GK_REQUIRE(!f32mma || (!up && !out32 && !tri0), GK_EUNSUPPORTED, "unsupported update against the float32 archive");
  kt_begin(f32mma ? KC_ARCH_UPDATE : KC_TSGEMM, st);
  if (f32mma) {
    static_assert(MT_R == T_TR && MT_C == T_TB, "same tile grid");
    const dim3 g1(row_tile_grid((n + MT_R - 1) / MT_R, (ld + MT_C - 1) / MT_C));   // row_tile order
    hipLaunchKernelGGL(tsgemm_f32mma_kernel, g1, dim3(256), 0, st, n, ld, (const float*)A.base, A.stride, A.nb, C, in,
                       out, alpha, beta, flag);
  } else if (mfma_ok(ld)) {
    launch_update64(n, ld, A, C, in, out, out32, alpha, beta, flag, up ? 1 : (tri0 ? 2 : 0), st);
  } else if (ld == 8 && !A.f32 && A.nb <= 2) {
    const dim3 g8((unsigned)std::min<int64_t>((n + 31) / 32, 8192));
    if (A.nb == 1)
      hipLaunchKernelGGL(update8_kernel<1>, g8, dim3(256), 0, st, n, (const double*)A.base, A.stride, C, in, out, out32,
                         alpha, beta, flag);
    else
      hipLaunchKernelGGL(update8_kernel<2>, g8, dim3(256), 0, st, n, (const double*)A.base, A.stride, C, in, out, out32,
                         alpha, beta, flag);
  } else if (A.f32)
    hipLaunchKernelGGL((tsgemm_kernel<true, false>), grid, dim3(256), 0, st, n, ld, ld, A.base, A.stride,
                       A.nb, C, ld, in, out, out32, alpha, beta, (int64_t)ld, (const int64_t*)nullptr,
                       flag);
  else
    hipLaunchKernelGGL((tsgemm_kernel<false, false>), grid, dim3(256), 0, st, n, ld, ld, A.base,
                       A.stride, A.nb, C, ld, in, out, out32, alpha, beta, (int64_t)ld,
                       (const int64_t*)nullptr, flag);
  GK_HIP(hipGetLastError());
  // method's own flops: a triangular coefficient block (R^-1, or B_{k-1}^T
  // of the recurrence) costs n ld (ld + 1)
  const int ntri = (up || tri0) ? 1 : 0;
  kt_end(st, (double)n * ld * ((A.f32 ? 4.0 : 8.0) * A.nb + (beta != 0.0 ? 16.0 : 8.0) + (out32 ? 4.0 : 0.0)),
         2.0 * (double)n * ld * ld * (A.nb - ntri) + ntri * (double)n * ld * (ld + 1), flag);
}

// The assembly at ld = 8: a row a lane, its s <= 8 results in registers, the
// coefficients of 32 blocks at a time in LDS (read by all lanes at once).  The
// sums of tsgemm_kernel (contraction index ascending, the same bits).  Bound by
// the read of the blocks: 318k nodes, 30 float64 blocks 118 us (64-wide tiles 653).
constexpr int A8_NB = 32;
template <bool F32>
__global__ void __launch_bounds__(256)
assemble8_kernel(int64_t n, int s, const void* __restrict__ Abase, int64_t astride, int nb,
                 const double* __restrict__ U, int ldu, double* __restrict__ P, int64_t ldo,
                 const int64_t* __restrict__ perm) {
  __shared__ __align__(16) double sU[A8_NB * 64];
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x, rc = min(r, n - 1);
  double acc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) acc[c] = 0.0;
  for (int j0 = 0; j0 < nb; j0 += A8_NB) {
    const int nj = min(A8_NB, nb - j0);
    __syncthreads();
    for (int q = threadIdx.x; q < nj * 64; q += 256) {
      const int a = j0 * 8 + (q >> 3), c = q & 7;
      sU[q] = c < s ? U[(int64_t)a * ldu + c] : 0.0;
    }
    __syncthreads();
#pragma unroll 2
    for (int j = 0; j < nj; ++j) {
      const int64_t o = (int64_t)(j0 + j) * astride + rc * 8;
      double a[8];
      if (F32) {
        const float4* p = reinterpret_cast<const float4*>(static_cast<const float*>(Abase) + o);
        const float4 x = p[0], y = p[1];
        a[0] = x.x; a[1] = x.y; a[2] = x.z; a[3] = x.w;
        a[4] = y.x; a[5] = y.y; a[6] = y.z; a[7] = y.w;
      } else {
        const double2* p = reinterpret_cast<const double2*>(static_cast<const double*>(Abase) + o);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const double2 x = p[k];
          a[2 * k] = x.x;
          a[2 * k + 1] = x.y;
        }
      }
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[c] = fma(a[k], sU[j * 64 + k * 8 + c], acc[c]);
    }
  }
  if (r >= n) return;
  const int64_t orow = perm ? perm[r] : r;
#pragma unroll
  for (int c = 0; c < 8; ++c)
    if (c < s) P[(int64_t)c * ldo + orow] = acc[c];
}

void launch_assemble(int64_t n, int ld, int s, BlockList A, const double* U, int ldu, double* P,
                     const int64_t* perm, hipStream_t st) {
  dim3 grid((unsigned)((n + T_TR - 1) / T_TR), (s + T_TB - 1) / T_TB);
  kt_begin(KC_ASSEMBLE, st);
  if (mfma_ok(ld)) {
    const dim3 g1(row_tile_grid((n + MT_R - 1) / MT_R, (s + MT_C - 1) / MT_C));   // row_tile order
    if (A.f32)
      hipLaunchKernelGGL(assemble_f32mma_kernel, g1, dim3(256), 0, st, n, ld, (const float*)A.base, A.stride, A.nb,
                         U, ldu, s, P, n, perm);
    else
      hipLaunchKernelGGL(assemble_mfma_kernel, g1, dim3(256), 0, st, n, ld, (const double*)A.base, A.stride, A.nb, U,
                         ldu, s, P, n, perm);
  } else if (ld == 8 && s <= 8) {
    const dim3 g8((unsigned)((n + 255) / 256));
    if (A.f32)
      hipLaunchKernelGGL(assemble8_kernel<true>, g8, dim3(256), 0, st, n, s, A.base, A.stride, A.nb, U, ldu, P, n, perm);
    else
      hipLaunchKernelGGL(assemble8_kernel<false>, g8, dim3(256), 0, st, n, s, A.base, A.stride, A.nb, U, ldu, P, n, perm);
  } else if (A.f32)
    hipLaunchKernelGGL((tsgemm_kernel<true, true>), grid, dim3(256), 0, st, n, ld, s, A.base, A.stride,
                       A.nb, U, ldu, (const double*)nullptr, P, (float*)nullptr, 1.0, 0.0, n, perm,
                       (const int*)nullptr);
  else
    hipLaunchKernelGGL((tsgemm_kernel<false, true>), grid, dim3(256), 0, st, n, ld, s, A.base, A.stride,
                       A.nb, U, ldu, (const double*)nullptr, P, (float*)nullptr, 1.0, 0.0, n, perm,
                       (const int*)nullptr);
  GK_HIP(hipGetLastError());
  kt_end(st, (double)n * ((A.f32 ? 4.0 : 8.0) * ld * A.nb + 8.0 * s), 2.0 * (double)n * ld * s * A.nb);
}

// ------------------------------------------------------------- predictor
// out[perm[r]] = sum_k sum_c A_k[r, c] z[k ld + c] (the GEMV of the kernel
// machine predictor, HBM-bound): q lanes per row (a power of two with
// 16 q >= ld), lane j reading float4 / double4 groups j, j + q, .. of each
// block row (contiguous across the lanes of a row), float64 accumulation,
// butterfly reduction over the q lanes.
template <bool F32>
__global__ void __launch_bounds__(256)
predict_kernel(int64_t n, int ld, int q, const void* __restrict__ Abase, int64_t astride, int nb,
               const double* __restrict__ z, double* __restrict__ out, const int64_t* __restrict__ perm) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t r = t / q;
  const int j = (int)(t - r * q);
  double acc = 0.0;
  if (r < n) {
    for (int k = 0; k < nb; ++k) {
      const int64_t base = (int64_t)k * astride + r * ld;
      const double* zk = z + (int64_t)k * ld;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = 4 * (j + q * u);
        if (c < ld) {
          double a0, a1, a2, a3;
          if (F32) {
            const float4 v = *reinterpret_cast<const float4*>(static_cast<const float*>(Abase) + base + c);
            a0 = v.x; a1 = v.y; a2 = v.z; a3 = v.w;
          } else {
            const double2* p = reinterpret_cast<const double2*>(static_cast<const double*>(Abase) + base + c);
            const double2 v0 = p[0], v1 = p[1];
            a0 = v0.x; a1 = v0.y; a2 = v1.x; a3 = v1.y;
          }
          acc = fma(a0, zk[c], acc);
          acc = fma(a1, zk[c + 1], acc);
          acc = fma(a2, zk[c + 2], acc);
          acc = fma(a3, zk[c + 3], acc);
        }
      }
    }
  }
  for (int o = q >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if (r < n && j == 0) out[perm ? perm[r] : r] = acc;
}

void launch_predict(int64_t n, int ld, BlockList A, const double* z, double* out, const int64_t* perm,
                    hipStream_t st) {
  int q = 1;
  while (16 * q < ld) q <<= 1;
  GK_REQUIRE(q <= 64 && ld % 4 == 0, GK_EINVAL, "predictor: unsupported block width");
  const int64_t tot = n * q;
  kt_begin(KC_PREDICT, st);
  if (A.f32)
    hipLaunchKernelGGL(predict_kernel<true>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, ld, q, A.base,
                       A.stride, A.nb, z, out, perm);
  else
    hipLaunchKernelGGL(predict_kernel<false>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, ld, q,
                       A.base, A.stride, A.nb, z, out, perm);
  GK_HIP(hipGetLastError());
  kt_end(st, (double)n * ld * A.nb * (A.f32 ? 4.0 : 8.0) + 8.0 * n, 2.0 * (double)n * ld * A.nb);
}

// ------------------------------------------------- column-wise operations
// out[i, c] = sum_k D[k*ld + c] * A_k[i, c]
template <bool F32, bool COLMAJ>
__global__ void assemble_diag_kernel(int64_t n, int ld, int s, const void* __restrict__ Abase,
                                     int64_t astride, int nb, const double* __restrict__ D,
                                     double* __restrict__ P, const int64_t* __restrict__ perm) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = t / ld;
  const int c = (int)(t - i * ld);
  if (i >= n || c >= s) return;
  double acc = 0.0;
  for (int k = 0; k < nb; ++k) acc = fma(D[k * ld + c], ldA<F32>(Abase, (int64_t)k * astride + i * ld + c), acc);
  const int64_t orow = perm ? perm[i] : i;
  if (COLMAJ)
    P[(int64_t)c * n + orow] = acc;
  else
    P[orow * ld + c] = acc;
}

void launch_assemble_diag(int64_t n, int ld, int s, BlockList A, const double* D, double* P,
                          const int64_t* perm, bool colmajor, hipStream_t st) {
  const int64_t tot = n * ld;
  dim3 grid((unsigned)((tot + 255) / 256));
#define GK_AD(F, CM)                                                                              \
  hipLaunchKernelGGL((assemble_diag_kernel<F, CM>), grid, dim3(256), 0, st, n, ld, s, A.base, A.stride, \
                     A.nb, D, P, perm)
  if (A.f32) {
    if (colmajor) GK_AD(true, true); else GK_AD(true, false);
  } else {
    if (colmajor) GK_AD(false, true); else GK_AD(false, false);
  }
#undef GK_AD
  GK_HIP(hipGetLastError());
}

// Column dot products and their updates (gbl and sbl).  A thread owns one
// column of a chunk of rows and walks the rows in order (DR of them loaded
// ahead), so the bits of a dot product depend on the chunks alone, not on the
// kernel that forms it or on the blocks beside it.
constexpr int DR = 4;
// sum over the row groups of a workgroup, P[c] for its columns
__device__ __forceinline__ void dots_out(double v, double* red, int cols, int groups, bool on, double* P) {
  const int tid = threadIdx.x;
  red[tid] = v;
  __syncthreads();
  if (tid < cols && on) {
    double t = 0.0;
    for (int q = 0; q < groups; ++q) t += red[q * cols + tid];
    *P = t;
  }
  __syncthreads();
}

// part[chunk][k*ld + c] = sum_{i in chunk} A_k[i,c] * B[i,c] for JB blocks
// from blockIdx.y * JB.  Bound by the read of the blocks: B serves JB of them
// (200k x 256, two blocks: 215 us; one block a pass, a row at a time: 415).
template <bool F32, int JB>
__global__ void __launch_bounds__(256)
coldots_kernel(int64_t n, int ld, const void* __restrict__ Abase, int64_t astride, int nb,
               const double* __restrict__ B, double* __restrict__ part, int64_t rows_per_chunk,
               const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  __shared__ double red[256];
  const int cols = ld < 256 ? ld : 256;
  const int groups = 256 / cols;
  const int64_t r_begin = (int64_t)blockIdx.x * rows_per_chunk;
  const int64_t r_end = min(n, r_begin + rows_per_chunk);
  const int k0 = blockIdx.y * JB;
  const int cl = threadIdx.x % cols, gr = threadIdx.x / cols;
  double* P = part + (int64_t)blockIdx.x * nb * ld;
  for (int cb = 0; cb < ld; cb += cols) {
    const int c = cb + cl;
    const bool on = gr < groups && c < ld;
    double acc[JB];
#pragma unroll
    for (int q = 0; q < JB; ++q) acc[q] = 0.0;
    if (on)
      for (int64_t r = r_begin + gr; r < r_end; r += (int64_t)DR * groups) {
        double b[DR], a[JB][DR];
        // rows past the chunk and blocks past the list read the last one
#pragma unroll
        for (int u = 0; u < DR; ++u) {
          const int64_t o = min(r + (int64_t)u * groups, r_end - 1) * ld + c;
          b[u] = B[o];
#pragma unroll
          for (int q = 0; q < JB; ++q) a[q][u] = ldA<F32>(Abase, (int64_t)min(k0 + q, nb - 1) * astride + o);
        }
#pragma unroll
        for (int u = 0; u < DR; ++u)
          if (r + (int64_t)u * groups < r_end)
#pragma unroll
            for (int q = 0; q < JB; ++q) acc[q] = fma(a[q][u], b[u], acc[q]);
      }
#pragma unroll
    for (int q = 0; q < JB; ++q)
      dots_out(acc[q], red, cols, groups, c < ld && k0 + q < nb, P + (int64_t)(k0 + q) * ld + c);
  }
}

// X -= sum_k A_k diag(D_k) over NB float64 blocks, then of the result, in the
// same pass: its dots with the NB blocks (DOTS) and with itself, the last
// block of the partials.  Four block passes where the update, the dots and
// the norm on their own take nine.  Bound by them: 200k x 256, 1.6 GB, 315 us
// (5.2 TB/s; the separate kernels 900 us).
template <int NB, bool DOTS>
__global__ void __launch_bounds__(256)
axpy_dots_kernel(int64_t n, int ld, const double* __restrict__ Abase, int64_t astride, const double* __restrict__ D,
                 double* X, double* __restrict__ part, int64_t rows_per_chunk) {
  __shared__ double red[256];
  const int cols = ld < 256 ? ld : 256;
  const int groups = 256 / cols;
  const int64_t r_begin = (int64_t)blockIdx.x * rows_per_chunk;
  const int64_t r_end = min(n, r_begin + rows_per_chunk);
  const int cl = threadIdx.x % cols, gr = threadIdx.x / cols;
  constexpr int NP = DOTS ? NB + 1 : 1;
  double* P = part + (int64_t)blockIdx.x * NP * ld;
  for (int cb = 0; cb < ld; cb += cols) {
    const int c = cb + cl;
    const bool on = gr < groups && c < ld;
    double acc[NP], d[NB];
#pragma unroll
    for (int q = 0; q < NP; ++q) acc[q] = 0.0;
    if (on) {
#pragma unroll
      for (int q = 0; q < NB; ++q) d[q] = -D[q * ld + c];
      for (int64_t r = r_begin + gr; r < r_end; r += (int64_t)DR * groups) {
        double x[DR], a[NB][DR];
#pragma unroll
        for (int u = 0; u < DR; ++u) {
          const int64_t o = min(r + (int64_t)u * groups, r_end - 1) * ld + c;
          x[u] = X[o];
#pragma unroll
          for (int q = 0; q < NB; ++q) a[q][u] = Abase[(int64_t)q * astride + o];
        }
#pragma unroll
        for (int u = 0; u < DR; ++u) {
          const int64_t ru = r + (int64_t)u * groups;
          if (ru < r_end) {
            double v = x[u];
#pragma unroll
            for (int q = 0; q < NB; ++q) v = fma(d[q], a[q][u], v);
            X[ru * ld + c] = v;
            if (DOTS)
#pragma unroll
              for (int q = 0; q < NB; ++q) acc[q] = fma(a[q][u], v, acc[q]);
            acc[NP - 1] = fma(v, v, acc[NP - 1]);
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < NP; ++q) dots_out(acc[q], red, cols, groups, c < ld, P + q * ld + c);
  }
}

// The same over a list of blocks, and the dots of the result with itself.
// Bound by the read of the list; four rows of four blocks are in flight.
__global__ void __launch_bounds__(256)
axpy_list_norms_kernel(int64_t n, int ld, const double* __restrict__ Abase, int64_t astride, int nb,
                       const double* __restrict__ D, double* X, double* __restrict__ part, int64_t rows_per_chunk,
                       const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  __shared__ double red[256];
  const int cols = ld < 256 ? ld : 256;
  const int groups = 256 / cols;
  const int64_t r_begin = (int64_t)blockIdx.x * rows_per_chunk;
  const int64_t r_end = min(n, r_begin + rows_per_chunk);
  const int cl = threadIdx.x % cols, gr = threadIdx.x / cols;
  for (int cb = 0; cb < ld; cb += cols) {
    const int c = cb + cl;
    double acc = 0.0;
    if (gr < groups && c < ld)
      for (int64_t r = r_begin + gr; r < r_end; r += (int64_t)DR * groups) {
        double x[DR];
        int64_t o[DR];
#pragma unroll
        for (int u = 0; u < DR; ++u) {
          o[u] = min(r + (int64_t)u * groups, r_end - 1) * ld + c;   // past the chunk: its last row, not written
          x[u] = X[o[u]];
        }
#pragma unroll 4
        for (int k = 0; k < nb; ++k) {
          const double d = -D[k * ld + c];
#pragma unroll
          for (int u = 0; u < DR; ++u) x[u] = fma(d, Abase[(int64_t)k * astride + o[u]], x[u]);
        }
#pragma unroll
        for (int u = 0; u < DR; ++u)
          if (r + (int64_t)u * groups < r_end) {
            X[o[u]] = x[u];
            acc = fma(x[u], x[u], acc);
          }
      }
    dots_out(acc, red, cols, groups, c < ld, part + (int64_t)blockIdx.x * ld + c);
  }
}

// *flag = 1 when the projection with coefficients D that left columns of
// squared norms nrm took away more than 1e-8 of one (each: sbl) or of all
// together (gbl, D equal over the columns); cf. again_kernel
__global__ void __launch_bounds__(256)
again_diag_kernel(int nb, int ld, int s, int global, const double* __restrict__ D, const double* __restrict__ nrm,
                  int* __restrict__ flag) {
  __shared__ double red[256];
  const int t = threadIdx.x;
  if (global) {
    double v = 0.0;
    for (int c = t; c < s; c += 256) v += nrm[c];
    red[t] = v;
    __syncthreads();
    if (t == 0) {
      double w = 0.0, d = 0.0;
      for (int q = 0; q < 256; ++q) w += red[q];
      for (int k = 0; k < nb; ++k) d = fma(D[k * ld], D[k * ld], d);
      if (!(d <= 1e-16 * w)) *flag = 1;
    }
    return;
  }
  for (int c = t; c < s; c += 256) {
    double d = 0.0;
    for (int k = 0; k < nb; ++k) d = fma(D[k * ld + c], D[k * ld + c], d);
    if (!(d <= 1e-16 * nrm[c])) *flag = 1;
  }
}

static void coldots_geometry(int64_t n, int* nch, int64_t* rpc) {
  int64_t want = 512;
  int64_t maxc = (n + 63) / 64;
  if (want > maxc) want = maxc;
  if (want < 1) want = 1;
  int64_t r = (n + want - 1) / want;
  *rpc = r;
  *nch = (int)((n + r - 1) / r);
}

size_t coldots_scratch_elems(int64_t n, int nb, int ld) {
  int nch;
  int64_t rpc;
  coldots_geometry(n, &nch, &rpc);
  return (size_t)nch * nb * ld;
}

void launch_coldots(int64_t n, int ld, BlockList A, const double* B, double* out, double* part,
                    const int* flag, hipStream_t st) {
  int nch;
  int64_t rpc;
  coldots_geometry(n, &nch, &rpc);
  const int jb = A.nb <= 2 ? A.nb : 4;
  const dim3 grid(nch, (A.nb + jb - 1) / jb);
#define GK_CD(F_, J_)                                                                                               \
  hipLaunchKernelGGL((coldots_kernel<F_, J_>), grid, dim3(256), 0, st, n, ld, A.base, A.stride, A.nb, B, part, rpc, \
                     flag)
  if (jb == 1) {
    if (A.f32) GK_CD(true, 1);
    else GK_CD(false, 1);
  } else if (jb == 2) {
    if (A.f32) GK_CD(true, 2);
    else GK_CD(false, 2);
  } else {
    if (A.f32) GK_CD(true, 4);
    else GK_CD(false, 4);
  }
#undef GK_CD
  GK_HIP(hipGetLastError());
  launch_reduce_parts((int64_t)A.nb * ld, nch, part, out, flag, st);
}

// X -= A diag(D) for float64 blocks A, nrm = the squared column norms of X
void launch_axpy_norms(int64_t n, int ld, BlockList A, const double* D, double* X, double* nrm, double* part,
                       const int* flag, hipStream_t st) {
  GK_REQUIRE(!A.f32, GK_EUNSUPPORTED, "update with norms of float64 blocks");
  int nch;
  int64_t rpc;
  coldots_geometry(n, &nch, &rpc);
  hipLaunchKernelGGL(axpy_list_norms_kernel, dim3(nch), dim3(256), 0, st, n, ld, (const double*)A.base, A.stride, A.nb,
                     D, X, part, rpc, flag);
  GK_HIP(hipGetLastError());
  launch_reduce_parts(ld, nch, part, nrm, flag, st);
}

void launch_again_diag(int nb, int ld, int s, bool global, const double* D, const double* nrm, int* flag,
                       hipStream_t st) {
  hipLaunchKernelGGL(again_diag_kernel, dim3(1), dim3(256), 0, st, nb, ld, s, global ? 1 : 0, D, nrm, flag);
  GK_HIP(hipGetLastError());
}

// X -= A diag(D) for the one or two float64 blocks A, and out = the dots of
// the new X: A_0^T X, .. (dots), X^T X
void launch_axpy_dots(int64_t n, int ld, BlockList A, const double* D, double* X, bool dots, double* out, double* part,
                      hipStream_t st) {
  GK_REQUIRE(!A.f32 && (A.nb == 1 || A.nb == 2), GK_EUNSUPPORTED, "fused update of one or two float64 blocks");
  int nch;
  int64_t rpc;
  coldots_geometry(n, &nch, &rpc);
#define GK_AD(N_, D_)                                                                                               \
  hipLaunchKernelGGL((axpy_dots_kernel<N_, D_>), dim3(nch), dim3(256), 0, st, n, ld, (const double*)A.base, A.stride, \
                     D, X, part, rpc)
  if (A.nb == 1) {
    if (dots) GK_AD(1, true);
    else GK_AD(1, false);
  } else {
    if (dots) GK_AD(2, true);
    else GK_AD(2, false);
  }
#undef GK_AD
  GK_HIP(hipGetLastError());
  launch_reduce_parts((int64_t)(dots ? A.nb + 1 : 1) * ld, nch, part, out, nullptr, st);
}

template <bool F32>
__global__ void axpy_diag_kernel(int64_t n, int ld, const void* __restrict__ Abase, int64_t astride,
                                 int nb, const double* __restrict__ D, double* __restrict__ X,
                                 const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n * ld; t += step) {
    const int c = (int)(t % ld);
    double x = X[t];
    for (int k = 0; k < nb; ++k) x = fma(-D[k * ld + c], ldA<F32>(Abase, (int64_t)k * astride + t), x);
    X[t] = x;
  }
}

void launch_axpy_diag(int64_t n, int ld, BlockList A, const double* D, double* X, const int* flag,
                      hipStream_t st) {
  const int64_t tot = n * ld;
  // capped: a gated launch that has nothing to do then dispatches few
  // workgroups (200k x 256: 43 us for 200k of them)
  dim3 grid((unsigned)std::min<int64_t>((tot + 255) / 256, 8192));
  if (A.f32)
    hipLaunchKernelGGL(axpy_diag_kernel<true>, grid, dim3(256), 0, st, n, ld, A.base, A.stride, A.nb, D,
                       X, flag);
  else
    hipLaunchKernelGGL(axpy_diag_kernel<false>, grid, dim3(256), 0, st, n, ld, A.base, A.stride, A.nb, D,
                       X, flag);
  GK_HIP(hipGetLastError());
}

__global__ void colscale_kernel(int64_t n, int ld, const double* __restrict__ X,
                                const double* __restrict__ scale, double* __restrict__ Y,
                                float* __restrict__ Y32) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * ld) return;
  const double v = X[t] * scale[t % ld];
  Y[t] = v;
  if (Y32) Y32[t] = (float)v;
}

void launch_colscale(int64_t n, int ld, const double* X, const double* scale, double* Y, float* Y32,
                     hipStream_t st) {
  const int64_t tot = n * ld;
  hipLaunchKernelGGL(colscale_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, n, ld, X,
                     scale, Y, Y32);
  GK_HIP(hipGetLastError());
}

// out[r*s + c] = sum_k D[k*ld + c] * A_k[rows[r], c]   (D == null: single block, weight 1)
template <bool F32>
__global__ void gather_rows_kernel(int ld, int s, const void* __restrict__ Abase, int64_t astride,
                                   int nb, const double* __restrict__ D, const int64_t* __restrict__ rows,
                                   double* __restrict__ out) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= s * s) return;
  const int r = t / s, c = t % s;
  const int64_t i = rows[r];
  double acc = 0.0;
  for (int k = 0; k < nb; ++k) {
    const double w = D ? D[k * ld + c] : 1.0;
    acc = fma(w, ldA<F32>(Abase, (int64_t)k * astride + i * ld + c), acc);
  }
  out[t] = acc;
}

void launch_gather_diag(int64_t n, int ld, int s, BlockList A, const double* D, const int64_t* rows,
                        double* out, hipStream_t st) {
  (void)n;
  const int tot = s * s;
  if (A.f32)
    hipLaunchKernelGGL(gather_rows_kernel<true>, dim3((tot + 255) / 256), dim3(256), 0, st, ld, s, A.base,
                       A.stride, A.nb, D, rows, out);
  else
    hipLaunchKernelGGL(gather_rows_kernel<false>, dim3((tot + 255) / 256), dim3(256), 0, st, ld, s,
                       A.base, A.stride, A.nb, D, rows, out);
  GK_HIP(hipGetLastError());
}

// ------------------------------------------------------------ misc
__global__ void start_block_kernel(int64_t n, int ld, int s, const int64_t* __restrict__ samples,
                                   double value, double* __restrict__ V, float* __restrict__ V32) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= s) return;
  const int64_t w = samples[j];
  V[w * ld + j] = value;
  if (V32) V32[w * ld + j] = (float)value;
}

__global__ void zero_kernel(uint64_t* __restrict__ p, size_t words) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < words; i += stride) p[i] = 0;
}

void launch_zero(void* p, size_t bytes, hipStream_t st) {
  // buffers come from the arena and are multiples of 256 bytes
  const size_t words = (bytes + 7) / 8;
  size_t blocks = (words + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks == 0) return;
  hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (uint64_t*)p, words);
  GK_HIP(hipGetLastError());
}

void launch_start_block(int64_t n, int ld, int s, const int64_t* dev_samples, double value, double* V,
                        float* V32, hipStream_t st) {
  launch_zero(V, (size_t)n * ld * sizeof(double), st);
  if (V32) launch_zero(V32, (size_t)n * ld * sizeof(float), st);
  hipLaunchKernelGGL(start_block_kernel, dim3((s + 255) / 256), dim3(256), 0, st, n, ld, s, dev_samples,
                     value, V, V32);
  GK_HIP(hipGetLastError());
}

__global__ void fill_columns_kernel(int64_t n, int32_t* __restrict__ zcol) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) zcol[i] = -1;
}
__global__ void sample_columns_kernel(int s, const int64_t* __restrict__ samples, int32_t* __restrict__ zcol) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < s) zcol[samples[j]] = j;
}
// zcol[i] = the column of E_W with a one in row i, -1 for the other rows
void launch_sample_columns(int64_t n, int s, const int64_t* dev_samples, int32_t* zcol, hipStream_t st) {
  hipLaunchKernelGGL(fill_columns_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, zcol);
  hipLaunchKernelGGL(sample_columns_kernel, dim3((s + 255) / 256), dim3(256), 0, st, s, dev_samples, zcol);
  GK_HIP(hipGetLastError());
}

__global__ void f64_to_f32_kernel(const double* __restrict__ a, float* __restrict__ b, size_t cnt) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) b[i] = (float)a[i];
}

void launch_copy_f64_to_f32(const double* a, float* b, size_t count, hipStream_t st) {
  hipLaunchKernelGGL(f64_to_f32_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, a, b,
                     count);
  GK_HIP(hipGetLastError());
}

}  // namespace gk
