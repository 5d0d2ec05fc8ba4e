// FP64 dense linear algebra for the modal covariance and the estimator.
//
//   zeta = (1/(6N)) sum_i b_i b_i^T                         (eq. linearterm)
//   zeta = L L^T, y = L^-1 alpha, z_s = L^-1 beta_s          (eq. Cholrot)
//   E_s = y.z_s / y.y,  sigma^2 = 6 / y.y                    (eqs. modalest, modalvariance)
//
// The products run on the FP64 matrix cores (v_mfma_f64_16x16x4_f64: lane l holds
// A[l % 16][l / 16] and B[l / 16][l % 16], accumulator register r is
// D[4 r + l / 16][l % 16], checked on the device).  The sample covariance and the Cholesky's trailing update
// are one lower-triangle tile kernel (128 x 64 tiles, four waves of 64 x 32, 16 k per
// LDS stage).  The Cholesky is right-looking with 64-wide panels: the diagonal block is
// factored in LDS by one workgroup, which also inverts it (W = L_kk^-1, kept in the
// block's unused upper triangle); the panel is then the product A_panel W^T on the matrix
// cores instead of a row-by-row substitution.  A non-positive (or NaN) pivot is recorded
// in flag[0] as 1 + its index; later steps then carry NaN and the host reports ENOTPD.
#include "common.h"

namespace modal {
namespace {

constexpr int NB = 64;

// Factor the diagonal block A[k0:k0+kb, k0:k0+kb] in place (lower triangle) and invert it,
// blocked by 16 so that the dependent chain is 4 x 16 short steps instead of 64 long ones.
// The block is in LDS; for each 16-column sub-block:
//   1. wave 0 factors its 16 x 16 diagonal block D (lane r holds row r in registers; the
//      pivot and the column of each step are broadcast by readlane).  Sixteen more lanes
//      hold the rows of the identity and take the same column operations, which leaves
//      D^-T in them: the inverse costs no step of its own;
//   2. the 16 x 16 blocks below it become A_I D^-T, one wave each on the matrix cores;
//   3. the trailing blocks of the lower triangle are updated, dealt to the waves.
// Then W = L^-1 from the four inverted diagonal blocks, by block distance:
//   W_IJ = -D_I^-1 (sum_{J <= K < I} L_IK W_KJ).
// L goes back to the lower triangle and W's strictly lower part, transposed, to the
// block's upper triangle (A[k0 + c][k0 + q] = W[q][c]).  Rows and columns past kb are an
// identity block.  A non-positive pivot is recorded in flag and turns into NaN.
// Bound by the chain of 64 pivots, which the look-ahead cannot hide: with LDS shuffles, a
// square root and a division per entry in the chain and scalar block products it took 57 us; 22.6
// now (33 with the inverses formed by substitution).
constexpr int SB = 16;       // sub-block
constexpr int DS = NB + 2;   // LDS row stride: 16 rows x 2 columns of doubles fill the 64 banks
typedef double d4 __attribute__((ext_vector_type(4)));

__device__ inline double lane_value(double v, int i) {   // lane i's v, i uniform
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, i), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), i);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// acc += X Y^T of two 16 x 16 blocks in LDS rows x0.., y0.., columns xc.., yc.. (YT: acc += X Y,
// Y's rows y0.. being the inner index)
template <bool YT>
__device__ inline d4 block_product(d4 acc, const double (*X)[DS], int x0, int xc, const double (*Y)[DS], int y0, int yc,
                                   int lane) {
  const int l16 = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int ks = 0; ks < SB / 4; ++ks) {
    const int k = 4 * ks + kq;
    const double b = YT ? Y[y0 + k][yc + l16] : Y[y0 + l16][yc + k];
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[x0 + l16][xc + k], b, acc, 0, 0, 0);
  }
  return acc;   // register r of lane l: row 4 r + l / 16, column l % 16
}

// copy: the block below, A[k0 + NB ..][k0 ..], is left transposed in the upper triangle for
// k_panel_update, whose workgroups all need it while one of them overwrites it.
__global__ __launch_bounds__(256) void k_potrf_diag(int n, double* __restrict__ A, int k0, int kb, int* flag,
                                                    bool copy) {
  __shared__ double a[NB][DS];
  __shared__ double Wf[NB][DS];   // W = L^-1 (diagonal blocks first, then the rest)
  __shared__ double T[NB][DS];    // block products of the inverse
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int l16 = lane & 15, kq = lane >> 4;
  double av[NB * NB / 256], bv[NB * NB / 256];
  if (copy) {   // uniform
#pragma unroll
    for (int u = 0; u < NB * NB / 256; ++u) {
      const int e = t + 256 * u, r = e / NB, c = e - r * NB;
      bv[u] = A[(size_t)min(k0 + NB + r, n - 1) * n + k0 + c];
    }
#pragma unroll
    for (int u = 0; u < NB * NB / 256; ++u) {
      const int e = t + 256 * u, r = e / NB, c = e - r * NB;
      if (k0 + NB + r < n) A[(size_t)(k0 + c) * n + k0 + NB + r] = bv[u];
    }
  }
#pragma unroll
  for (int u = 0; u < NB * NB / 256; ++u) {
    const int e = t + 256 * u, r = e / NB, c = e - r * NB;
    av[u] = A[(size_t)(k0 + min(r, kb - 1)) * n + k0 + min(c, kb - 1)];
  }
#pragma unroll
  for (int u = 0; u < NB * NB / 256; ++u) {
    const int e = t + 256 * u, r = e / NB, c = e - r * NB;
    a[r][c] = (r < kb && c < kb && c <= r) ? av[u] : (c == r ? 1.0 : 0.0);
    Wf[r][c] = 0.0;
  }
  __syncthreads();
  for (int kk = 0; kk < NB / SB; ++kk) {
    const int c0 = SB * kk;
    if (wv == 0) {   // 1. factor and invert the 16 x 16 diagonal block (every 16 lanes own its rows)
      const int r = l16;
      const bool id = lane & 16;   // lanes 16..31 (and 48..63) carry the rows of the identity along
      double d[SB];
#pragma unroll
      for (int c = 0; c < SB; ++c) d[c] = id ? (c == r ? 1.0 : 0.0) : a[c0 + r][c0 + c];
#pragma unroll
      for (int j = 0; j < SB; ++j) {
        const double p = lane_value(d[j], j);
        const bool ok = p > 0.0;
        if (lane == 0 && !ok && c0 + j < kb) atomicCAS(flag, 0, k0 + c0 + j + 1);
        // divided, not multiplied by 1 / sqrt(p): correctly rounded, and an infinite pivot (a mode
        // without weight) leaves a column of zeros
        const double sd = ok ? sqrt(p) : __builtin_nan("");   // uniform
        d[j] = !id && r == j ? sd : d[j] / sd;
#pragma unroll
        for (int c = j + 1; c < SB; ++c) d[c] -= d[j] * lane_value(d[j], c);   // entries past the diagonal are never read
      }
      // lane 16 + r holds row r of I D^-T, which is column r of D^-1.  Lane r's entries past the
      // diagonal are no part of L and never read.
      if (lane < 2 * SB) {
        double* q = id ? &Wf[c0][c0 + r] : &a[c0 + r][c0];
        const int step = id ? DS : 1;
#pragma unroll
        for (int c = 0; c < SB; ++c) q[c * step] = d[c];
      }
    }
    __syncthreads();
    // 2. blocks below: A_I <- A_I D^-T (each read and written by one wave)
    if (const int I = kk + 1 + wv; I < NB / SB) {
      const d4 x = block_product<false>(d4{0.0, 0.0, 0.0, 0.0}, a, SB * I, c0, Wf, c0, c0, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) a[SB * I + 4 * r + kq][c0 + l16] = x[r];
    }
    __syncthreads();
    // 3. trailing blocks (I, J), kk < J <= I
    const int nt = NB / SB - 1 - kk;
    for (int e = wv; e < nt * (nt + 1) / 2; e += 4) {
      const int i = e < 1 ? 0 : e < 3 ? 1 : 2, I = kk + 1 + i, J = kk + 1 + e - i * (i + 1) / 2;
      const d4 x = block_product<false>(d4{0.0, 0.0, 0.0, 0.0}, a, SB * I, c0, a, SB * J, c0, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) a[SB * I + 4 * r + kq][SB * J + l16] -= x[r];
    }
    __syncthreads();
  }
  // the off-diagonal blocks of W, by block distance: wave b forms (I, J) = (b + dist, b)
  for (int dist = 1; dist < NB / SB; ++dist) {
    const int J = wv, I = wv + dist;
    if (I < NB / SB) {   // T_IJ = sum_{J <= K < I} L_IK W_KJ
      d4 x = d4{0.0, 0.0, 0.0, 0.0};
      for (int K = J; K < I; ++K) x = block_product<true>(x, a, SB * I, SB * K, Wf, SB * K, SB * J, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) T[SB * I + 4 * r + kq][SB * J + l16] = x[r];
    }
    __syncthreads();
    if (I < NB / SB) {   // W_IJ = -D_I^-1 T_IJ
      const d4 x = block_product<true>(d4{0.0, 0.0, 0.0, 0.0}, Wf, SB * I, SB * I, T, SB * I, SB * J, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) Wf[SB * I + 4 * r + kq][SB * J + l16] = -x[r];
    }
    __syncthreads();
  }
  for (int e = t; e < NB * NB; e += 256) {
    const int r = e / NB, c = e - r * NB;
    if (r < kb && c < kb) A[(size_t)(k0 + r) * n + k0 + c] = c <= r ? a[r][c] : Wf[c][r];
  }
}

// Forward substitution on the diagonal block for every right-hand side row.
__global__ __launch_bounds__(64) void k_trsv_diag(int n, const double* __restrict__ A, int k0, int kb,
                                                  double* __restrict__ B) {
  __shared__ double L[NB][NB + 1];
  __shared__ double y[NB];
  for (int e = threadIdx.x; e < NB * NB; e += 64) {
    const int i = e / NB, j = e - i * NB;
    L[i][j] = (i < kb && j < kb) ? A[(size_t)(k0 + i) * n + k0 + j] : 0.0;
  }
  double* b = B + (size_t)blockIdx.x * n + k0;
  if (threadIdx.x < kb) y[threadIdx.x] = b[threadIdx.x];
  __syncthreads();
  for (int c = 0; c < kb; ++c) {
    if (threadIdx.x == 0) y[c] = y[c] / L[c][c];
    __syncthreads();
    const int i = threadIdx.x;
    if (i > c && i < kb) y[i] -= L[i][c] * y[c];
    __syncthreads();
  }
  if (threadIdx.x < kb) b[threadIdx.x] = y[threadIdx.x];
}

// B[r][i] -= sum_c A[i][k0+c] B[r][k0+c] for i >= k0 + kb, all rows r < nrhs (chunks of 64).
__global__ __launch_bounds__(256) void k_trsv_update(int n, const double* __restrict__ A, int k0, int kb, int nrhs,
                                                     double* __restrict__ B) {
  __shared__ double y[64][NB];
  const int r0 = blockIdx.y * 64;
  const int nr = min(64, nrhs - r0);
  for (int e = threadIdx.x; e < 64 * NB; e += 256) {
    const int r = e / NB, c = e - r * NB;
    y[r][c] = (r < nr && c < kb) ? B[(size_t)(r0 + r) * n + k0 + c] : 0.0;
  }
  __syncthreads();
  const int i = k0 + kb + blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  double l[NB];
  const double* row = A + (size_t)i * n + k0;
#pragma unroll
  for (int c = 0; c < NB; ++c) l[c] = c < kb ? row[c] : 0.0;
  for (int r = 0; r < nr; ++r) {
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < NB; ++c) acc += l[c] * y[r][c];
    B[(size_t)(r0 + r) * n + i] -= acc;
  }
}

// One step of the blocked forward substitution with the inverted diagonal blocks that
// k_potrf_diag leaves in the upper triangles: for the right-hand sides r (rows of B
// [nrhs][n]), y_r = W b_r[k0:k0+kb] (W = L_kk^-1), written to Y by workgroup 0; the other
// workgroups each form the same y (a 64 x 64 product, cheaper than a second launch) and
// update their 256 rows below: B[r][i] -= sum_c L[i][k0 + c] y_r[c].  B's block rows are
// only read, so no workgroup writes what another still reads.
constexpr int TRS_R = 16;   // right-hand sides per workgroup
__global__ __launch_bounds__(256) void k_trsv_inv_step(int n, const double* __restrict__ A, int k0, int kb, int nrhs,
                                                       double* __restrict__ B, double* __restrict__ Y) {
  __shared__ double W[NB][NB + 1];
  __shared__ double b[TRS_R][NB];
  __shared__ double y[TRS_R][NB];
  const int tid = threadIdx.x;
  const int r0 = blockIdx.y * TRS_R, nr = min(TRS_R, nrhs - r0);
#pragma unroll
  for (int u = 0; u < NB * NB / 256; ++u) {
    const int e = tid + 256 * u, i = e / NB, k = e - i * NB;   // W[i][k], k <= i
    const int ic = min(i, kb - 1), kc = min(k, kb - 1);   // clamped into the block
    const double v = A[(size_t)(k0 + min(kc, ic)) * n + k0 + max(kc, ic)];   // L_ii on the diagonal
    W[i][k] = (i < kb && k < kb) ? (k == i ? 1.0 / v : (k < i ? v : 0.0)) : 0.0;
  }
  for (int e = tid; e < TRS_R * NB; e += 256) {
    const int r = e / NB, c = e - r * NB;
    b[r][c] = (r < nr && c < kb) ? B[(size_t)(r0 + r) * n + k0 + c] : 0.0;
  }
  __syncthreads();
  for (int e = tid; e < TRS_R * NB; e += 256) {
    const int r = e / NB, i = e - r * NB;
    double v = 0.0;
    for (int k = 0; k <= i; ++k) v += W[i][k] * b[r][k];
    y[r][i] = v;
  }
  __syncthreads();
  if (blockIdx.x == 0) {
    for (int e = tid; e < TRS_R * NB; e += 256) {
      const int r = e / NB, c = e - r * NB;
      if (r < nr && c < kb) Y[(size_t)(r0 + r) * n + k0 + c] = y[r][c];
    }
    return;
  }
  const int i = k0 + kb + (blockIdx.x - 1) * 256 + tid;
  if (i >= n) return;
  const double* row = A + (size_t)i * n + k0;
  double l[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) l[c] = row[c];   // kb == NB whenever rows remain below
  for (int r = 0; r < nr; ++r) {
    double acc = 0.0;
#pragma unroll
    for (int c = 0; c < NB; ++c) acc += l[c] * y[r][c];
    B[(size_t)(r0 + r) * n + i] -= acc;
  }
}

// out[0] = y.y, out[1+s] = y.z_s with y = rows[0], z_s = rows[1+s].
__global__ __launch_bounds__(256) void k_dots(int n, const double* __restrict__ rows, double* __restrict__ out) {
  const double* y = rows;
  const double* z = rows + (size_t)blockIdx.x * n;
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) acc += y[i] * z[i];
  __shared__ double red[256];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = red[0];
}

typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));   // rows of odd length: 8-byte aligned
constexpr int TK = 16;     // k per LDS stage of the matrix-core update kernel
constexpr int TRL = 128;   // rows per tile
constexpr int TC = 64;     // columns per tile, and rows of the small tile

// Lower-triangle tile update on the matrix cores, tile (bi, bj) of TR x 64, j0 <= i0 + TR - 1 (TR 128, or 64):
//   C[i][j] = alpha sum_k P(i, k) P(j, k)                 (COLS: P(i, k) = X[k][i], rows of X
//                                                          [K][n] are the samples), or
//   C[i][j] -= sum_k P(i, k) P(j, k)                      (P(i, k) = X[(r0 + i) ld + k], a panel).
// The panel's sums start from zero and meet the old values once: started from the old values, each
// of their 128 steps rounds at the old value's size, and the backward error of the factor at
// 1140 modes was 3.7e-15 instead of 1.0e-15.
// Rows and columns start at r0 for C.  MIRROR: the upper triangle gets the same values (a
// symmetric result), transposed through LDS.  Four waves of TR / 2 x 32; a wave wholly above the
// diagonal only stages.  COLS numbers the lower triangle's tiles alone (row bi has TR / 64 (bi + 1)), so
// that the workgroups which leave at once are not dealt unevenly over the chip.  LDS: k-major rows of COLS 16 doubles past a multiple of 64 words, so
// that two k of 16 rows fill the banks; row-major of 18 doubles for a panel, the same.
// Bound by the matrix cores and by the staging's L2 reads (10.7 flop per byte; 64 x 64 tiles
// had 8).  6000 x 4960 samples: 4.93 ms with 64 x 64 tiles and two-way bank conflicts, 3.35 ms
// (44 TFLOP/s of the triangle's flops) now, 3.64 with the triangle cut out of a square grid.
template <bool COLS, bool MIRROR, int TR>
__global__ __launch_bounds__(256, 3) void k_tile_update(int n, int K, int r0, const double* __restrict__ X, int ld,
                                                        double alpha, double* __restrict__ C) {
  constexpr int NR = TR / TC, MA = TR / 32;   // column tiles per tile row of the diagonal; a wave's 16-row tiles
  int bi = blockIdx.y, bj = blockIdx.x;
  if (COLS) {
    const int t = 2 / NR * blockIdx.x;   // rows before bi hold NR bi (bi + 1) / 2 tiles
    bi = (int)((sqrtf(1.0f + 4.0f * t) - 1.0f) * 0.5f);
    while (bi * (bi + 1) > t) --bi;
    while ((bi + 1) * (bi + 2) <= t) ++bi;
    bj = (t - bi * (bi + 1)) / (2 / NR);
  }
  const int i0 = r0 + bi * TR, j0 = r0 + bj * TC;
  if (j0 > i0 + TR - 1 || i0 >= n || j0 >= n) return;   // whole workgroup, before any barrier
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  const int wr = wv >> 1, wc = wv & 1, l16 = lane & 15, kq = lane >> 4;
  const int iw = i0 + TR / 2 * wr, jw = j0 + 32 * wc;             // the wave's first row and column
  const bool live = jw <= iw + TR / 2 - 1 && iw < n && jw < n;    // uniform
  constexpr int SI = COLS ? TR + 16 : TK + 2, SJ = COLS ? TC + 16 : TK + 2;   // row strides
  constexpr int NI = COLS ? TK : TR, NJ = COLS ? TK : TC;                     // LDS rows
  constexpr int TS = 17;                                                      // mirror staging row
  constexpr size_t kBytes = sizeof(double) * (NI * SI + NJ * SJ), kMir = MIRROR ? sizeof(double) * 4 * 32 * TS : 0;
  __shared__ __attribute__((aligned(16))) unsigned char raw[kBytes > kMir ? kBytes : kMir];
  double(*Pi)[SI] = reinterpret_cast<double(*)[SI]>(raw);
  double(*Pj)[SJ] = reinterpret_cast<double(*)[SJ]>(raw + sizeof(double) * NI * SI);
  d4 acc[MA][2];
#pragma unroll
  for (int ta = 0; ta < MA; ++ta)
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) acc[ta][tb] = d4{0.0, 0.0, 0.0, 0.0};
  // The next stage's operands are loaded, two doubles at a time, while this stage multiplies.
  // COLS: 16 k x 64 pairs of rows and 16 k x 32 of columns; panel: rows of 8 pairs of k.
  constexpr int LI = TR * TK / 512, LJ = TC * TK / 512;
  d2 pi[LI], pj[LJ];
  const bool inside = i0 + TR <= n && j0 + TC <= n;   // every row and column of the tile exists
  auto at = [&](int idx, int base, int k) {   // pair idx of a stage: (k, column pair) or (row, k pair)
    d2 v;
    if (COLS) {
      const double* row = X + (size_t)min(k, K - 1) * ld;
      v.x = row[min(base + idx, n - 1)];
      v.y = row[min(base + idx + 1, n - 1)];
      if (k >= K) v = d2{0.0, 0.0};
    } else {
      const double* row = X + (size_t)min(base + idx, n - 1) * ld;
      v.x = k < K ? row[min(k, K - 1)] : 0.0;
      v.y = k + 1 < K ? row[min(k + 1, K - 1)] : 0.0;
    }
    return v;
  };
  auto load = [&](int k0) {
    if (inside && k0 + TK <= K) {   // uniform
#pragma unroll
      for (int u = 0; u < LI; ++u) {
        const int e = tid + 256 * u;
        pi[u] = COLS ? *reinterpret_cast<const d2*>(X + (size_t)(k0 + e / (TR / 2)) * ld + i0 + 2 * (e % (TR / 2)))
                     : *reinterpret_cast<const d2*>(X + (size_t)(i0 + e / (TK / 2)) * ld + k0 + 2 * (e % (TK / 2)));
      }
#pragma unroll
      for (int u = 0; u < LJ; ++u) {
        const int e = tid + 256 * u;
        pj[u] = COLS ? *reinterpret_cast<const d2*>(X + (size_t)(k0 + e / (TC / 2)) * ld + j0 + 2 * (e % (TC / 2)))
                     : *reinterpret_cast<const d2*>(X + (size_t)(j0 + e / (TK / 2)) * ld + k0 + 2 * (e % (TK / 2)));
      }
    } else {
#pragma unroll
      for (int u = 0; u < LI; ++u) {
        const int e = tid + 256 * u;
        pi[u] = COLS ? at(2 * (e % (TR / 2)), i0, k0 + e / (TR / 2)) : at(e / (TK / 2), i0, k0 + 2 * (e % (TK / 2)));
      }
#pragma unroll
      for (int u = 0; u < LJ; ++u) {
        const int e = tid + 256 * u;
        pj[u] = COLS ? at(2 * (e % (TC / 2)), j0, k0 + e / (TC / 2)) : at(e / (TK / 2), j0, k0 + 2 * (e % (TK / 2)));
      }
    }
  };
  load(0);
  for (int k0 = 0; k0 < K; k0 += TK) {
#pragma unroll
    for (int u = 0; u < LI; ++u) {
      const int e = tid + 256 * u;
      constexpr int W = COLS ? TR / 2 : TK / 2;
      *reinterpret_cast<d2*>(&Pi[e / W][2 * (e % W)]) = pi[u];
    }
#pragma unroll
    for (int u = 0; u < LJ; ++u) {
      const int e = tid + 256 * u;
      constexpr int W = COLS ? TC / 2 : TK / 2;
      *reinterpret_cast<d2*>(&Pj[e / W][2 * (e % W)]) = pj[u];
    }
    __syncthreads();
    if (k0 + TK < K) load(k0 + TK);
    if (live) {
#pragma unroll
      for (int ks = 0; ks < TK / 4; ++ks) {
        const int kk = 4 * ks + kq;
        double a[MA], b[2];
#pragma unroll
        for (int t = 0; t < MA; ++t) {
          const int r = TR / 2 * wr + 16 * t + l16;
          a[t] = COLS ? Pi[kk][r] : Pi[r][kk];
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int c = 32 * wc + 16 * t + l16;
          b[t] = COLS ? Pj[kk][c] : Pj[c][kk];
        }
#pragma unroll
        for (int ta = 0; ta < MA; ++ta)
#pragma unroll
          for (int tb = 0; tb < 2; ++tb) acc[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ta], b[tb], acc[ta][tb], 0, 0, 0);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int ta = 0; ta < MA; ++ta) {
    d4 cold[2];   // the old values of a row tile, all loaded before the first is used
    if (!COLS)
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          cold[tb][r] = C[(size_t)min(iw + 16 * ta + 4 * r + kq, n - 1) * n + min(jw + 16 * tb + l16, n - 1)];
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = iw + 16 * ta + 4 * r + kq, j = jw + 16 * tb + l16;
        if (COLS) acc[ta][tb][r] *= alpha;
        if (live && i < n && j <= i) C[(size_t)i * n + j] = COLS ? acc[ta][tb][r] : cold[tb][r] - acc[ta][tb][r];
      }
  }
  if constexpr (MIRROR) {   // 16 rows x 32 columns at a time: row j of the upper triangle, 16 consecutive i
    double(*tr)[TS] = reinterpret_cast<double(*)[TS]>(raw) + 32 * wv;
#pragma unroll
    for (int ta = 0; ta < MA; ++ta) {
#pragma unroll
      for (int tb = 0; tb < 2; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) tr[16 * tb + l16][4 * r + kq] = acc[ta][tb][r];
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = jw + 4 * u + kq, i = iw + 16 * ta + l16;
        if (live && i < n && j < i) C[(size_t)j * n + i] = tr[4 * u + kq][l16];
      }
      __syncthreads();
    }
  }
}

// Panel: rows i >= k0 + kb, A[i, k0:k0+kb] <- A[i, k0:k0+kb] W^T with W = L_kk^-1, whose
// strictly lower part k_potrf_diag left transposed in the block's upper triangle and
// whose diagonal is 1 / L_jj.  64 rows per workgroup, four waves of 32 x 32.
__global__ __launch_bounds__(256) void k_panel_mfma(int n, double* __restrict__ A, int k0, int kb) {
  __shared__ double Ar[NB][NB + 1];   // the workgroup's panel rows
  __shared__ double Wt[NB][NB + 1];   // Wt[k][c] = W[c][k]
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  const int l16 = lane & 15, kq = lane >> 4;
  const int rbase = k0 + kb + blockIdx.x * NB;
  // loads unconditional (clamped indices, values selected after); kb == NB for a panel
#pragma unroll
  for (int u = 0; u < NB * NB / 256; ++u) {
    const int e = tid + 256 * u;
    const int r = e / NB, c = e - r * NB;
    const double av = A[(size_t)min(rbase + r, n - 1) * n + k0 + c];
    // Wt[k][c] = W[c][k]: W[c][k] for k < c sits at A[k0 + k][k0 + c]; W[c][c] = 1 / L_cc
    const int k = r;
    const double wv_ = A[(size_t)(k0 + min(k, c)) * n + k0 + c];
    Ar[r][c] = rbase + r < n ? av : 0.0;
    Wt[k][c] = k == c ? 1.0 / wv_ : (k < c ? wv_ : 0.0);
  }
  __syncthreads();
  const int wr = wv >> 1, wc = wv & 1;
  d4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int ks = 0; ks < NB / 4; ++ks) {
    const int kk = 4 * ks + kq;
    double a[2], b[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      a[t] = Ar[32 * wr + 16 * t + l16][kk];
      b[t] = Wt[kk][32 * wc + 16 * t + l16];
    }
#pragma unroll
    for (int ta = 0; ta < 2; ++ta)
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) acc[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ta], b[tb], acc[ta][tb], 0, 0, 0);
  }
  // every read of the rows is done (the stores below overwrite them)
#pragma unroll
  for (int ta = 0; ta < 2; ++ta)
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = rbase + 32 * wr + 16 * ta + 4 * r + kq, c = 32 * wc + 16 * tb + l16;
        if (i < n && c < kb) A[(size_t)i * n + k0 + c] = acc[ta][tb][r];
      }
}

// The panel of block column k0 (as k_panel_mfma) and its update of the next block column,
//   P = A[rows, k0 ..] W^T,   A[rows, k2 ..] -= P P_0^T,   k2 = k0 + NB,
// in one launch: every workgroup forms P_0, the panel of the rows k2 .., for itself from the copy
// that k_potrf_diag left (a product of 64^3 against a launch and the wait for the panel).
// Bound by latency, on the chain of the factorization.  The estimator at 4960 modes: 8.95 ms with the
// panel and the update as two launches, 8.76 in one.
__global__ __launch_bounds__(256) void k_panel_update(int n, double* __restrict__ A, int k0) {
  __shared__ double X[NB][DS], Y[NB][DS], Wt[NB][DS];   // the workgroup's rows (then P), rows k2 .. (then P_0), W^T
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  const int l16 = lane & 15, kq = lane >> 4, wr = wv >> 1, wc = wv & 1;
  const int k2 = k0 + NB, rbase = k2 + blockIdx.x * NB;
  double xv[NB * NB / 256], yv[NB * NB / 256], wv_[NB * NB / 256];
#pragma unroll
  for (int u = 0; u < NB * NB / 256; ++u) {
    const int e = tid + 256 * u, r = e / NB, c = e - r * NB;
    xv[u] = A[(size_t)min(rbase + r, n - 1) * n + k0 + c];
    yv[u] = A[(size_t)(k0 + r) * n + min(k2 + c, n - 1)];
    wv_[u] = A[(size_t)(k0 + min(r, c)) * n + k0 + c];
  }
  d4 cv[2][2];
#pragma unroll
  for (int ta = 0; ta < 2; ++ta)
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = min(rbase + 32 * wr + 16 * ta + 4 * r + kq, n - 1), j = min(k2 + 32 * wc + 16 * tb + l16, n - 1);
        cv[ta][tb][r] = A[(size_t)i * n + j];
      }
#pragma unroll
  for (int u = 0; u < NB * NB / 256; ++u) {
    const int e = tid + 256 * u, r = e / NB, c = e - r * NB;
    X[r][c] = rbase + r < n ? xv[u] : 0.0;
    Y[c][r] = k2 + c < n ? yv[u] : 0.0;
    Wt[r][c] = r == c ? 1.0 / wv_[u] : (r < c ? wv_[u] : 0.0);
  }
  __syncthreads();
  d4 p[2][2], q[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) p[a][b] = q[a][b] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int ks = 0; ks < NB / 4; ++ks) {
    const int kk = 4 * ks + kq;
    double a[2], c[2], b[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      a[t] = X[32 * wr + 16 * t + l16][kk];
      c[t] = Y[32 * wr + 16 * t + l16][kk];
      b[t] = Wt[kk][32 * wc + 16 * t + l16];
    }
#pragma unroll
    for (int ta = 0; ta < 2; ++ta)
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        p[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ta], b[tb], p[ta][tb], 0, 0, 0);
        q[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[ta], b[tb], q[ta][tb], 0, 0, 0);
      }
  }
  __syncthreads();   // every read of the rows is done
#pragma unroll
  for (int ta = 0; ta < 2; ++ta)
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ri = 32 * wr + 16 * ta + 4 * r + kq, c = 32 * wc + 16 * tb + l16;
        X[ri][c] = p[ta][tb][r];
        Y[ri][c] = q[ta][tb][r];
        if (rbase + ri < n) A[(size_t)(rbase + ri) * n + k0 + c] = p[ta][tb][r];
      }
  __syncthreads();
  d4 u[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) u[a][b] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int ks = 0; ks < NB / 4; ++ks) {
    const int kk = 4 * ks + kq;
    double a[2], b[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      a[t] = X[32 * wr + 16 * t + l16][kk];
      b[t] = Y[32 * wc + 16 * t + l16][kk];
    }
#pragma unroll
    for (int ta = 0; ta < 2; ++ta)
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) u[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ta], b[tb], u[ta][tb], 0, 0, 0);
  }
#pragma unroll
  for (int ta = 0; ta < 2; ++ta)
#pragma unroll
    for (int tb = 0; tb < 2; ++tb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = rbase + 32 * wr + 16 * ta + 4 * r + kq, j = k2 + 32 * wc + 16 * tb + l16;
        if (i < n && j <= i) A[(size_t)i * n + j] = cv[ta][tb][r] - u[ta][tb][r];
      }
}

__global__ void k_copy_lower(int n, const double* __restrict__ src, double* __restrict__ dst) {
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (size_t)n * n) return;
  const size_t i = e / n, j = e - i * n;
  dst[e] = j <= i ? src[e] : 0.0;
}

}  // namespace

// C[i][k] = B[i][k] - (1/N) sum_j B[j][k] (rows of B [N][n]); one thread per column
__global__ __launch_bounds__(256) void k_center_rows(int n, int N, const double* __restrict__ B,
                                                     double* __restrict__ C) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  double m = 0.0;
  for (int i = 0; i < N; ++i) m += B[(size_t)i * n + k];
  m /= N;
  for (int i = 0; i < N; ++i) C[(size_t)i * n + k] = B[(size_t)i * n + k] - m;
}

hipError_t launch_center_rows(int n, int N, const double* B, double* C, hipStream_t st) {
  hipLaunchKernelGGL(k_center_rows, dim3((n + 255) / 256), dim3(256), 0, st, n, N, B, C);
  return hipGetLastError();
}

hipError_t launch_syrk(int n, int N, const double* B, double scale, double* Z, hipStream_t st) {
  // Tiles of 64 x 64 while those of 128 x 64 are fewer than the CUs: each workgroup runs through all
  // the samples by itself there, and the smaller tile's stage is the shorter one (1000 samples: 120
  // modes 110 and 74 us, 816 modes 123 and 99, 1540 modes (182 tiles) 119 and 110; 2600 modes (462
  // tiles) 171 and 178, 11,480 modes with 200 samples 533 and 548).  The sums are the same bit for bit.
  const int nb = (n + TRL - 1) / TRL, nc = (n + TC - 1) / TC;
  if (nb * (nb + 1) <= 256)
    hipLaunchKernelGGL((k_tile_update<true, true, TC>), dim3(nc * (nc + 1) / 2), dim3(256), 0, st, n, N, 0, B, n, scale, Z);
  else
    hipLaunchKernelGGL((k_tile_update<true, true, TRL>), dim3(nb * (nb + 1)), dim3(256), 0, st, n, N, 0, B, n, scale, Z);
  return hipGetLastError();
}

hipError_t launch_copy_lower(int n, const double* src, double* dst, hipStream_t st) {
  const size_t tot = (size_t)n * n;
  hipLaunchKernelGGL(k_copy_lower, dim3((tot + 255) / 256), dim3(256), 0, st, n, src, dst);
  return hipGetLastError();
}

hipError_t launch_cholesky_lookahead(int n, double* A, int* flag, hipStream_t st, hipStream_t side, hipEvent_t ev_a,
                                     hipEvent_t ev_p, int nrhs, double* B, double* Y) {
  constexpr int T = TC;
  // A[i][j] -= sum_c A[i][k0 + c] A[j][k0 + c], i >= j >= r0, tile columns [bj0, ...) of the
  // (n - r0)-square trailing grid; nbx tile columns
  auto update = [&](int k0, int kb, int r0, int nbx, hipStream_t s) {
    hipLaunchKernelGGL((k_tile_update<false, false, TRL>), dim3(nbx, (n - r0 + TRL - 1) / TRL), dim3(256), 0, s, n, kb, r0, A + k0,
                       n, -1.0, A);
  };
  // Factor the block column [k, k + 2 NB) (its two NB-wide halves), all updates from the
  // columns left of k applied: diagonal block and panel of the first half, its update of the
  // second half's columns, then the second half's diagonal block and panel.
  auto factor2 = [&](int k, hipStream_t s) {
    const int kb = n - k < NB ? n - k : NB;
    const int k2 = k + NB;
    hipLaunchKernelGGL(k_potrf_diag, dim3(1), dim3(256), 0, s, n, A, k, kb, flag, k2 < n);
    if (k2 < n) {
      hipLaunchKernelGGL(k_panel_update, dim3((n - k2 + NB - 1) / NB), dim3(256), 0, s, n, A, k);
      const int kb2 = n - k2 < NB ? n - k2 : NB;
      hipLaunchKernelGGL(k_potrf_diag, dim3(1), dim3(256), 0, s, n, A, k2, kb2, flag, false);
      if (n - k2 - kb2 > 0)
        hipLaunchKernelGGL(k_panel_mfma, dim3((n - k2 - kb2 + NB - 1) / NB), dim3(256), 0, s, n, A, k2, kb2);
    }
  };
  // The solve steps of a factored block column (Y_k = W_kk B_k, and the rows below updated
  // with its panel): they need only that block column, so they overlap the next one's
  // factorization instead of following the whole.  About 45 us per block column: on the main stream
  // after the event that releases side they stay off the chain of the factorization; behind the
  // factorization on side they delayed it (the estimator at 4960 modes 8.76 ms, 8.34 now; at 11,480
  // 21.2 and 21.1).
  auto solve2 = [&](int k, hipStream_t s) {
    for (int kk = k; kk < k + 2 * NB && kk < n; kk += NB) {
      const int kb = n - kk < NB ? n - kk : NB, rem = n - kk - kb;
      hipLaunchKernelGGL(k_trsv_inv_step, dim3(1 + (rem + 255) / 256, (nrhs + TRS_R - 1) / TRS_R), dim3(256), 0, s, n,
                         A, kk, kb, nrhs, B, Y);
    }
  };
  // The trailing updates take both halves of a factored block column at once (K = 2 NB), so
  // each trailing tile is read and written once per 2 NB columns instead of per NB.
  factor2(0, st);
  int solved = 0;   // block column whose solve steps run next
  for (int k0 = 0; k0 + 2 * NB < n; k0 += 2 * NB) {
    const int k1 = k0 + 2 * NB;   // the next block column (both halves of [k0, k1) are NB wide)
    const int w1 = n - k1 < 2 * NB ? n - k1 : 2 * NB;
    const int nb1 = (w1 + T - 1) / T;   // its tile columns
    // the next block column's tiles first, then the rest of the trailing matrix
    update(k0, 2 * NB, k1, nb1, st);
    hipError_t e = hipEventRecord(ev_a, st);
    if (e != hipSuccess) return e;
    if (nrhs > 0) solve2(solved, st);
    if (n - k1 > 2 * NB) update(k0, 2 * NB, k1 + 2 * NB, (n - k1 - 2 * NB + T - 1) / T, st);
    if ((e = hipStreamWaitEvent(side, ev_a, 0)) != hipSuccess) return e;
    factor2(k1, side);
    if ((e = hipEventRecord(ev_p, side)) != hipSuccess) return e;
    if ((e = hipStreamWaitEvent(st, ev_p, 0)) != hipSuccess) return e;
    solved = k1;
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (nrhs > 0) solve2(solved, st);
  return hipGetLastError();
}

hipError_t launch_trsm_rows(int n, const double* L, int nrhs, double* B, hipStream_t st) {
  for (int k0 = 0; k0 < n; k0 += NB) {
    const int kb = n - k0 < NB ? n - k0 : NB;
    hipLaunchKernelGGL(k_trsv_diag, dim3(nrhs), dim3(64), 0, st, n, L, k0, kb, B);
    const int rem = n - k0 - kb;
    if (rem > 0)
      hipLaunchKernelGGL(k_trsv_update, dim3((rem + 255) / 256, (nrhs + 63) / 64), dim3(256), 0, st, n, L, k0, kb,
                         nrhs, B);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_estimator(int n, const double* rows, const double* /*unused*/, int S, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_dots, dim3(S + 1), dim3(256), 0, st, n, rows, out);
  return hipGetLastError();
}

}  // namespace modal
