// Float64 tall-skinny products of blocks 64 columns and wider on the FP64
// matrix cores: the Gram matrices C = A^T B (H_kk = Q_k^T X of Alg. 1, the
// projection coefficients, X^T X for CholQR) and the updates out = beta in +
// alpha A C (the recurrence of Alg. 1, the projections, X R^-1).
//
// Widths are multiples of 16; tiles are counted in units of 16 columns.  All
// products run as 16 x 16 x 4 steps of mfma4.h.  FP64 matrix instructions
// occupy the vector ALU, so every other vector instruction of the inner loops
// costs matrix time: operands come from LDS in the layout the instruction
// takes (no lane moves), addresses advance by pointer increments, and only
// the last round of a row range is masked.
//
// Summation order: each element of C sums its rows in ascending order inside
// a row chunk, four at a time, and each element of A C its contraction
// indices in ascending order, whatever the tile shape (symmetric products
// form x y for y x), so results do not depend on the tiling.
#include <type_traits>

#include "gk_internal.h"
#include "mfma4.h"

namespace gk {

typedef double d2 __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------ Gram C = A^T B
// Workgroup: UA wavefronts over an A tile of UA units (units of all A blocks
// counted through, so a tile may span blocks) and a B tile of UB units, rows
// of one chunk.  Rounds of 16 rows are staged in LDS (double buffered, one
// barrier a round; the next round is in flight in registers during the
// products).  Wavefront w owns A unit w: per four rows it reads its unit in
// the four quad rotations and each B unit once (4 + UB LDS reads for 4 UB
// matrix instructions).
//
// The Gram of a block with itself runs as tile pairs ta <= tb only.  On a
// diagonal tile (GK_SELF, staged once) wavefront w forms the unit pairs (w, (w + d) % T), d = 0 .. T / 2: every
// unordered pair once, the same count for each wavefront but for d = T / 2 at
// even T; pairs with (w + d) % T < w are stored transposed.  The reduction
// mirrors the rest.
constexpr int GR = 16;   // rows per round

enum { GK_ALL = 0, GK_SELF = 1, GK_OFF = 2 };   // tile pairs of a launch
template <int UA, int UB, int KIND>
__global__ void __launch_bounds__(64 * UA, 2)
gram64_kernel(int64_t n, int ld, int u, const double* __restrict__ Abase, int64_t astride, int nua,
              const double* __restrict__ B, double* __restrict__ part, int64_t rpc, int nta, int ntb,
              const int* __restrict__ flag) {
  if (flag && *flag == 0) return;
  constexpr int NT = 64 * UA;
  constexpr int PA = 16 * UA + 2, PB = 16 * UB + 2;
  constexpr int QB = (GR * 8 * UB + NT - 1) / NT;   // 16-byte pieces of B per thread and round
  constexpr int DC = UB / 2;                        // largest d on a symmetric diagonal
  constexpr bool diag = KIND == GK_SELF;
  __shared__ __align__(16) double sA[2][GR * PA];
  __shared__ __align__(16) double sB[2][diag ? 2 : GR * PB];
  // the tile pairs of a chunk are consecutive workgroups of XCD chunk % 8
  const unsigned L = blockIdx.x, x = L & 7, jj = L >> 3;
  const unsigned npair = diag ? (unsigned)ntb : (KIND == GK_OFF ? (unsigned)(ntb * (ntb - 1) / 2) : (unsigned)(nta * ntb));
  const int tc = (int)((jj / npair) * 8 + x);
  int ta = (int)(jj % npair), tb;
  if (diag) {
    tb = ta;
  } else if (KIND == GK_OFF) {   // ta < tb, row by row
    int t = ta;
    ta = 0;
    while (t >= ntb - 1 - ta) { t -= ntb - 1 - ta; ++ta; }
    tb = ta + 1 + t;
  } else {
    tb = ta / nta;
    ta -= tb * nta;
  }
  const int64_t rb = (int64_t)tc * rpc;
  const int64_t re = min(n, rb + rpc);
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63, li = l & 15, lk = l >> 4;
  double* P = part + (int64_t)tc * ((int64_t)nua * 16) * ld;

  // A: the thread's 16-byte column of the tile, rows ra and ra + 8
  const int ra = tid / (8 * UA), ca = 2 * (tid % (8 * UA));
  const double* pa[2];
  {
    const int g = min(ta * UA + ca / 16, nua - 1);   // units past the last repeat it (not stored)
    pa[0] = Abase + (int64_t)(g / u) * astride + (g % u) * 16 + (ca & 15) + (rb + ra) * ld;
    pa[1] = pa[0] + 8 * ld;
  }
  // B: uniform base of the round and a 32-bit offset per piece
  int rbq[QB], lbq[QB];
  unsigned ob[QB];
  const char* bb = reinterpret_cast<const char*>(B + rb * ld);
#pragma unroll
  for (int q = 0; q < QB; ++q) {
    const int idx = min(tid + NT * q, GR * 8 * UB - 1);
    const int c = 2 * (idx % (8 * UB));
    rbq[q] = idx / (8 * UB);
    lbq[q] = rbq[q] * PB + c;
    ob[q] = 8u * (unsigned)(min(tb * UB + c / 16, u - 1) * 16 + (c & 15) + rbq[q] * ld);
  }
  d2 va0[2], vb0[QB], va1[2], vb1[QB];   // rounds of even and odd index in flight
  const int64_t step = (int64_t)GR * ld;
  // a whole round, and the last one of the range (rows past it are zero)
  auto fetch = [&](d2 (&va)[2], d2 (&vb)[QB]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      va[q] = *reinterpret_cast<const d2*>(pa[q]);
      pa[q] += step;
    }
    if (!diag) {
#pragma unroll
      for (int q = 0; q < QB; ++q) vb[q] = *reinterpret_cast<const d2*>(bb + ob[q]);
      bb += 8 * step;
    }
  };
  auto fetch_last = [&](int rows, d2 (&va)[2], d2 (&vb)[QB]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int back = max(0, ra + 8 * q - (rows - 1));   // rows past the range read its last one
      const d2 v = *reinterpret_cast<const d2*>(pa[q] - (int64_t)back * ld);
      va[q] = back ? d2{0.0, 0.0} : v;
    }
    if (!diag) {
#pragma unroll
      for (int q = 0; q < QB; ++q) {
        const int back = max(0, rbq[q] - (rows - 1));
        const d2 v = *reinterpret_cast<const d2*>(bb + (ob[q] - 8u * (unsigned)(back * ld)));
        vb[q] = back ? d2{0.0, 0.0} : v;
      }
    }
  };
  auto fetch_at = [&](int64_t r0, d2 (&va)[2], d2 (&vb)[QB]) {
    const int64_t left = re - r0;
    if (left >= GR) fetch(va, vb);
    else if (left > 0) fetch_last((int)left, va, vb);
  };
  auto put = [&](int p, const d2 (&va)[2], const d2 (&vb)[QB]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) *reinterpret_cast<d2*>(&sA[p][(ra + 8 * q) * PA + ca]) = va[q];
    if (!diag) {
#pragma unroll
      for (int q = 0; q < QB; ++q)
        if (QB * NT == GR * 8 * UB || tid + NT * q < GR * 8 * UB) *reinterpret_cast<d2*>(&sB[p][lbq[q]]) = vb[q];
    }
  };
  // LDS columns of the four rotations of this wavefront's A unit
  int cr[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) cr[r] = 16 * w + 4 * (((li >> 2) + r) & 3) + (li & 3);

  m4d acc[UB];
#pragma unroll
  for (int j = 0; j < UB; ++j) acc[j] = m4d{0.0, 0.0, 0.0, 0.0};
  if (rb < re) {
    fetch_at(rb, va0, vb0);
    fetch_at(rb + GR, va1, vb1);
    put(0, va0, vb0);
  }
  __syncthreads();
  // round r0 from buffer p: the round after the next goes into the registers
  // (va, vb) that held this one, the next one (vna, vnb) to LDS at the end
  auto round = [&](int64_t r0, auto buf, d2 (&va)[2], d2 (&vb)[QB], const d2 (&vna)[2], const d2 (&vnb)[QB]) {
    constexpr int p = decltype(buf)::value;
    fetch_at(r0 + 2 * GR, va, vb);
    const double* a = sA[p] + lk * PA;
    const double* b = (diag ? sA[p] : sB[p]) + lk * PB + li;
    // the operands of the next four rows are read before the products of the
    // current ones (LDS latency)
    constexpr int NU = diag ? DC + 1 : UB;
    double ar[2][4], br[2][NU];
    auto operands = [&](int ks, double (&ar)[4], double (&br)[NU]) {
#pragma unroll
      for (int r = 0; r < 4; ++r) ar[r] = a[4 * ks * PA + cr[r]];
#pragma unroll
      for (int d = 0; d < NU; ++d) {
        int j = d;
        if (diag) {
          j = w + d;
          if (j >= UB) j -= UB;
        }
        br[d] = b[4 * ks * PB + 16 * j];
      }
    };
    operands(0, ar[0], br[0]);
#pragma unroll
    for (int ks = 0; ks < GR / 4; ++ks) {
      if (ks + 1 < GR / 4) operands(ks + 1, ar[(ks + 1) & 1], br[(ks + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int d = 0; d < NU; ++d) mma4(ar[ks & 1], br[ks & 1][d], acc[d]);
    }
    if (r0 + GR < re) put(p ^ 1, vna, vnb);
    __syncthreads();
  };
  for (int64_t r0 = rb; r0 < re; r0 += 2 * GR) {
    round(r0, std::integral_constant<int, 0>{}, va0, vb0, va1, vb1);
    if (r0 + GR < re) round(r0 + GR, std::integral_constant<int, 1>{}, va1, vb1, va0, vb0);
  }
  const int ga = ta * UA + w;
  if (ga >= nua) return;
#pragma unroll
  for (int j = 0; j < UB; ++j) {
    if (diag && (j > DC || (UB % 2 == 0 && j == DC && w >= DC))) continue;
    int jb = j;
    if (diag) {
      jb = w + j;
      if (jb >= UB) jb -= UB;
    }
    const int gb = tb * UB + jb;
    if (gb >= u || (diag && ta * UA + w >= u)) continue;
    double v[4];
    unrot4(acc[j], v);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = 16 * ga + 4 * q + lk, c = 16 * gb + li;
      if (diag && jb < w) P[(int64_t)c * ld + i] = v[q];
      else P[(int64_t)i * ld + c] = v[q];
    }
  }
}

// The tile size of 4, 5, 6 units that pads a width of u units least (four on a tie).
static int small_units(int u) {
  int best = 4;
  for (int T = 5; T <= 6; ++T)
    if ((u + T - 1) / T * T < (u + best - 1) / best * best) best = T;
  return best;
}
// Units per tile of the Gram of a block with itself: one tile up to eight; beyond that
// small tiles, which with the chunk counts of the callers is 4 to 6
// workgroups a CU.
static int self_units(int u) { return u <= 8 ? u : small_units(u); }
// Units per B tile otherwise: as few tiles of at most eight as cover u, evenly.
static int even_units(int u) {
  const int nt = (u + 7) / 8;
  return (u + nt - 1) / nt;
}

// part[c] (nb ld x ld) = A^T B over the rows of chunk c of nch (rpc rows
// each; chunks past the last row write zeros); self: B = A (then only the
// 16 x 16 units on and above the diagonal are written).
void launch_gram64(int64_t n, int ld, BlockList A, const double* B, double* part, int nch, int64_t rpc, bool self,
                   const int* flag, hipStream_t st) {
  GK_REQUIRE(ld >= 64 && ld % 16 == 0 && !A.f32 && A.nb >= 1 && (!self || A.nb == 1) && nch % 8 == 0 && n >= 1 &&
                 rpc >= 1 && rpc * nch >= n,
             GK_EUNSUPPORTED, "float64 Gram: unsupported block shape");
  const int u = ld / 16, nua = A.nb * u;
  int T = self ? self_units(u) : even_units(u), nt = (u + T - 1) / T, nta = (nua + 7) / 8;
  // few rows: 4 x 4 unit tiles where the large ones would leave CUs without work
  const bool few = !self && (int64_t)nch * nta * nt < 512;
  if (few) {
    T = 4;
    nt = (u + 3) / 4;
    nta = (nua + 3) / 4;
  }
#define GK_G(UA_, UB_, K_, PAIRS_)                                                                                  \
  hipLaunchKernelGGL((gram64_kernel<UA_, UB_, K_>), dim3((unsigned)nch * (unsigned)(PAIRS_)), dim3(64 * UA_), 0, st, \
                     n, ld, u, (const double*)A.base, A.stride, nua, B, part, rpc, nta, nt, flag)
#define GK_T(T_)                                   \
  case T_:                                         \
    if (few) GK_G(4, 4, GK_ALL, nta * nt);         \
    else if (!self) GK_G(8, T_, GK_ALL, nta * nt); \
    else GK_G(T_, T_, GK_SELF, nt)
  // a block with itself in several tiles (of 4 to 6 units): the pairs off the diagonal
#define GK_TO(T_)                                                    \
    GK_T(T_);                                                        \
    if (self && nt > 1) GK_G(T_, T_, GK_OFF, nt * (nt - 1) / 2);     \
    break
  switch (T) {
    GK_TO(4);
    GK_TO(5);
    GK_TO(6);
    GK_T(7);
    break;
    GK_T(8);
    break;
    default: throw Error{GK_EUNSUPPORTED, "float64 Gram: unsupported block width"};
  }
#undef GK_TO
#undef GK_T
#undef GK_G
  GK_HIP(hipGetLastError());
}

// ------------------------------------------- out = beta in + alpha A C
// Workgroup: 4 wavefronts over 64 rows and a column tile of T units;
// wavefront w owns 16 rows and all T units.  Chunks of 16 contraction indices
// of A and C go through LDS (double buffered, one barrier a chunk; a chunk
// never crosses a block): per four indices a wavefront reads its rows of A in
// the four quad rotations and each unit of C once (4 + T LDS reads for 4 T
// matrix instructions).  LDS pitch of A odd: the 16 rows of a column read
// fall on different banks.  A is loaded two chunks ahead.  Tiles of 4 to 6
// units leave three to four workgroups a CU, whose first loads and epilogues
// run beside the others' products; one tile of 8 units over the whole width
// of 128 (A read once, two workgroups a CU) took 575 us where tiles of 4 take
// 405 us (500k rows, one block).
//
// tri 1: C (one block) is upper triangular, tri 2: the first coefficient
// block is lower triangular (B_{k-1}^T of the recurrence); zeros are stored
// on the other side, and units without a non-zero in a chunk are left out.
constexpr int UK = 16;        // contraction indices per chunk
constexpr int UPA = UK + 1;

constexpr int NW = 4;          // wavefronts
template <int T>
__global__ void __launch_bounds__(64 * NW, 2)
update64_kernel(int64_t n, int ld, const double* __restrict__ Abase, int64_t astride, int nb,
                const double* __restrict__ C, const double* in, double* out, float* __restrict__ out32, double alpha,
                double beta, int nct, const int* __restrict__ flag, int tri) {
  if (flag && *flag == 0) return;
  constexpr int NT = 64 * NW, UROWS = 16 * NW, PC = 16 * T + 2;
  constexpr int NC = UK * 8 * T;               // 16-byte pieces of a chunk of C
  constexpr int QC = (NC + NT - 1) / NT;
  __shared__ __align__(16) double sA[2][UROWS * UPA];
  __shared__ __align__(16) double sC[2][UK * PC];
  // the column tiles of row tile rt are consecutive workgroups of XCD rt % 8
  const unsigned L = blockIdx.x, x = L & 7, jj = L >> 3;
  const int tb = (int)(jj % (unsigned)nct);
  const int64_t rt = (int64_t)(jj / (unsigned)nct) * 8 + x;
  if (rt * UROWS >= n) return;
  const int b0 = 16 * T * tb;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l = tid & 63, li = l & 15, lk = l >> 4;
  const int cpb = ld / UK;                         // chunks per block
  // chunks with a non-zero coefficient: all, or up to the tile's last column
  // (upper), or from the tile's first column on in the first block (lower)
  const int cend = tri == 1 ? min(cpb, tb * T + T) : nb * cpb;
  const int cbeg = tri == 2 ? tb * T : 0;

  // A: rows ar and ar + 8 NW of the tile, 16-byte column ac (rows past n read
  // row n - 1, not stored); C: row and column of each piece.  Uniform bases
  // that advance with the chunk, 32-bit offsets that do not.
  const int ar = tid >> 3, ac = 2 * (tid & 7);
  const int64_t r0 = rt * UROWS;
  const int blk0 = cbeg / cpb;
  const char* ba = reinterpret_cast<const char*>(Abase + (int64_t)blk0 * astride + (cbeg - blk0 * cpb) * UK + r0 * ld);
  const char* bc = reinterpret_cast<const char*>(C + (int64_t)cbeg * UK * ld);
  unsigned oa[2], oc[QC];
  int lc[QC];
#pragma unroll
  for (int q = 0; q < 2; ++q) oa[q] = 8u * (unsigned)((int)min((int64_t)(ar + 8 * NW * q), n - 1 - r0) * ld + ac);
#pragma unroll
  for (int q = 0; q < QC; ++q) {
    const int idx = min(tid + NT * q, NC - 1);
    const int row = idx / (8 * T), col = 2 * (idx % (8 * T));
    lc[q] = row * PC + col;
    oc[q] = 8u * (unsigned)(row * ld + min(b0 + col, ld - 2));
  }
  d2 va0[2], va1[2], vc[QC];   // A of even and odd chunks in flight
  int kc = cbeg % cpb;   // chunk within its block
  const int64_t cstep = (int64_t)UK * ld * 8, bstep = (astride - ld) * 8;
  auto fetch_c = [&]() {
#pragma unroll
    for (int q = 0; q < QC; ++q) vc[q] = *reinterpret_cast<const d2*>(bc + oc[q]);
    bc += cstep;
  };
  auto fetch_a = [&](d2 (&va)[2]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) va[q] = *reinterpret_cast<const d2*>(ba + oa[q]);
    ba += 8 * UK;
    if (++kc == cpb) {   // the next block's first chunk
      kc = 0;
      ba += bstep;
    }
  };
  auto put = [&](int p, const d2 (&va)[2]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      sA[p][(ar + 8 * NW * q) * UPA + ac] = va[q].x;
      sA[p][(ar + 8 * NW * q) * UPA + ac + 1] = va[q].y;
    }
#pragma unroll
    for (int q = 0; q < QC; ++q)
      if (QC * NT == NC || tid + NT * q < NC) *reinterpret_cast<d2*>(&sC[p][lc[q]]) = vc[q];
  };
  // LDS offsets of the four rotations of this wavefront's rows
  int rr[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) rr[r] = (16 * w + 4 * (((li >> 2) + r) & 3) + (li & 3)) * UPA + lk;

  m4d acc[T];
#pragma unroll
  for (int t = 0; t < T; ++t) acc[t] = m4d{0.0, 0.0, 0.0, 0.0};
  fetch_c();
  fetch_a(va0);
  if (cbeg + 1 < cend) fetch_a(va1);
  put(0, va0);
  __syncthreads();
  // chunk c from buffer p: A of the chunk after the next goes into the
  // registers that held this one's, the next chunk to LDS at the end
  auto chunk = [&](int c, auto buf, d2 (&va)[2], const d2 (&vn)[2]) {
    constexpr int p = decltype(buf)::value;
    if (c + 1 < cend) fetch_c();
    if (c + 2 < cend) fetch_a(va);
    const double* a = sA[p];
    const double* s = sC[p] + lk * PC + li;
    // units t0 .. t1 - 1 have non-zero coefficients in this chunk
    const int t0 = tri == 1 ? max(0, c - tb * T) : 0;
    const int t1 = tri == 2 && c < cpb ? min(T, c + 1 - tb * T) : T;
    if (t0 == 0 && t1 == T) {
      // the operands of the next four indices are read before the products
      // of the current ones (LDS latency)
      double av[2][4], bv[2][T];
      auto operands = [&](int ks, double (&av)[4], double (&bv)[T]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) av[r] = a[rr[r] + 4 * ks];
#pragma unroll
        for (int t = 0; t < T; ++t) bv[t] = s[4 * ks * PC + 16 * t];
      };
      operands(0, av[0], bv[0]);
#pragma unroll
      for (int ks = 0; ks < UK / 4; ++ks) {
        if (ks + 1 < UK / 4) operands(ks + 1, av[(ks + 1) & 1], bv[(ks + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < T; ++t) mma4(av[ks & 1], bv[ks & 1][t], acc[t]);
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < UK / 4; ++ks) {
        double av[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) av[r] = a[rr[r] + 4 * ks];
#pragma unroll
        for (int t = 0; t < T; ++t)
          if (t >= t0 && t < t1) mma4(av, s[4 * ks * PC + 16 * t], acc[t]);
      }
    }
    if (c + 1 < cend) put(p ^ 1, vn);
    __syncthreads();
  };
  for (int c = cbeg; c < cend; c += 2) {
    chunk(c, std::integral_constant<int, 0>{}, va0, va1);
    if (c + 1 < cend) chunk(c + 1, std::integral_constant<int, 1>{}, va1, va0);
  }
#pragma unroll
  for (int t = 0; t < T; ++t) {
    if (b0 + 16 * t >= ld) continue;
    double v[4], iv[4];
    unrot4(acc[t], v);
    const int c = b0 + 16 * t + li;
    const int64_t rw = r0 + 16 * w + lk;
#pragma unroll
    for (int q = 0; q < 4; ++q) iv[q] = beta != 0.0 ? in[min(rw + 4 * q, n - 1) * ld + c] : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t r = rw + 4 * q;
      if (r < n) {
        const double o = alpha * v[q] + beta * iv[q];
        out[r * ld + c] = o;
        if (out32) out32[r * ld + c] = (float)o;
      }
    }
  }
}

void launch_update64(int64_t n, int ld, BlockList A, const double* C, const double* in, double* out, float* out32,
                     double alpha, double beta, const int* flag, int tri, hipStream_t st) {
  GK_REQUIRE(ld >= 64 && ld % 16 == 0 && !A.f32 && A.nb >= 1 && n >= 1 && (tri != 1 || A.nb == 1), GK_EUNSUPPORTED,
             "float64 update: unsupported block shape");
  const int u = ld / 16, T = small_units(u), nct = (u + T - 1) / T;
  const int64_t nrt = (n + 16 * NW - 1) / (16 * NW), g = 8 * ((nrt + 7) / 8) * nct;
  GK_REQUIRE(g < (int64_t(1) << 23), GK_EUNSUPPORTED, "float64 update: too many rows for one launch");
#define GK_T(T_)                                                                                                  \
  case T_:                                                                                                        \
    hipLaunchKernelGGL((update64_kernel<T_>), dim3((unsigned)g), dim3(64 * NW), 0, st, n, ld,                  \
                       (const double*)A.base, A.stride, A.nb, C, in, out, out32, alpha, beta, nct, flag, tri);     \
    break
  switch (T) {
    GK_T(4);
    GK_T(5);
    GK_T(6);
    default: throw Error{GK_EUNSUPPORTED, "float64 update: unsupported block width"};
  }
#undef GK_T
  GK_HIP(hipGetLastError());
}

}  // namespace gk
