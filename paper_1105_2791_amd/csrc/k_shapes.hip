// Theory mode coefficients of separable bispectra, eq. (abispect), and the ideal
// (full-sky, isotropic) covariance of the separable modes, eq. (cbispect) with a
// diagonal covariance, which is also their Gram matrix: its Cholesky factor
// orthonormalises the basis (Sec. II).
//
// Both are triple sums over (l1, l2, l3) weighted by
//   h^2_{l1 l2 l3} = (2l1+1)(2l2+1)(2l3+1)/(8 pi) int_{-1}^{1} P_l1 P_l2 P_l3 dmu,
// since the squared 3j symbol (l1 l2 l3; 0 0 0)^2 is half the Legendre triple
// integral.  The sums then factor into one-dimensional Legendre series on a
// Gauss-Legendre rule in mu with ceil((3 lmax + 1) / 2) nodes, exact because the
// integrand has degree at most 3 lmax:
//   F_{f,a}(mu_k) = sum_l (2l+1) U_f(l) B_a(l) P_l(mu_k)
//   alpha_(pqr) = 1/(48 pi) sum_k w_k sum_t sum_{sigma in S3} F_{t,sigma1,p} F_{t,sigma2,q} F_{t,sigma3,r}
//       U = (X_t, Y_t, Z_t) for b = sum_t X_t Y_t Z_t, B_a = q_a / sqrt(C)
//   zeta0_(abc),(def) = 1/(48 pi) sum_k w_k sum_{sigma in S3} Q_{a,sigma d} Q_{b,sigma e} Q_{c,sigma f}
//       Q_ab = F_{b,a} with U_b = c q_b, B_a = q_a (c_l = <|a~_lm|^2> of the whitened sky)
// FP64 throughout.  Q_ab = Q_ba, so zeta0 needs the symmetric sums
//   T_ijk = sum_k' w Q_i Q_j Q_k (mu_k'),  i <= j <= k over the P (P + 1) / 2 pairs,
// each once: the covariance is a contraction on the matrix cores over the nodes, and each of
// its n_max^2 / 2 entries the sum of six of the T (k_node_triples, k_ideal_gather).
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace modal {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
constexpr int NT = 64;      // tile side of the matrix-core kernels (pairs or nodes)
constexpr int NK = 16;      // inner steps (l or nodes) per LDS stage
constexpr int NS = NT + 16; // LDS row stride: two rows of 16 doubles fill the 64 banks
__host__ __device__ inline int pad_to(int n, int m) { return (n + m - 1) / m * m; }

// Legendre series on the FP64 matrix cores (v_mfma_f64_16x16x4_f64, the layout of
// k_linalg.hip): the product of P_l(mu_k) (rows: 64 nodes) and (2l+1) U_f(l) B_a(l) (columns:
// 64 combinations (f, a)) over l, 16 l per stage.  Every wave runs Bonnet's recurrence of the
// workgroup's 64 nodes (one per lane) and stores a quarter of the stage's l, so that no wave
// waits for another's.  The recurrence steps the difference D_l = P_l - P_{l-1} at |mu|,
//   D_{l+1} = l/(l+1) D_l - (2l+1)/(l+1) (1 - |mu|) P_l,
// with P_l(-mu) = (-1)^l P_l(mu): 1 - |mu| is exact where P_l varies fastest, and P_l comes out
// to 4e-16 (rms over the 1501 nodes at l = 1000) where Bonnet's form leaves 1.8e-14.
//   PAIRS: combinations a <= f, F[k][pair(a, f)], nodes padded to a multiple of NK with zeros
//   and pairs to a multiple of NT;  otherwise F[f][k][a].
// Bound by latency.  One thread per node and 16 modes with a division in every step of the
// recurrence took 187 us for the 465 pairs at l_max 500, P 30; 62 us now.
__device__ inline double lane_value(double v, int i) {   // lane i's v, i uniform
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, i), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), i);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <bool PAIRS>
__global__ __launch_bounds__(256) void k_legendre_series(int L, int nmu, int P, int nrow,
                                                         const int* __restrict__ pair_a, const int* __restrict__ pair_b,
                                                         const double* __restrict__ U, const double* __restrict__ B,
                                                         const double* __restrict__ mu, double* __restrict__ F) {
  __shared__ double W[NK][NS], Pl[NK][NS];
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const int wr = wv >> 1, wc = wv & 1;
  const int k0 = blockIdx.x * NT, c0 = blockIdx.y * NT;
  const double xm = mu[min(k0 + lane, nmu - 1)], y = 1.0 - fabs(xm);
  // staged coefficients: this thread's l within a stage and its combinations cs + 16 u
  const int ll = tid & (NK - 1), cs = tid / NK;
  const double *Ur[4], *Br[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int r = min(c0 + cs + 16 * u, nrow - 1);   // columns past the last repeat it, never stored
    Ur[u] = U + (size_t)(PAIRS ? pair_b[r] : r / P) * L;
    Br[u] = B + (size_t)(PAIRS ? pair_a[r] : r % P) * L;
  }
  double pu[4], pb[4];
  auto load = [&](int l0) {
    const int l = min(l0 + ll, L - 1);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      pu[u] = Ur[u][l];
      pb[u] = Br[u][l];
    }
  };
  d4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
  double dl = 0.0, pl = 1.0;   // D_l, P_l at |mu| (D_0 is not used: its factor is 0)
  const bool flip = xm < 0.0;
  load(0);
  for (int l0 = 0; l0 < L; l0 += NK) {
    // lane i holds the step's coefficients for l = l0 + i
    const double lc = l0 + ll, c1 = lc / (lc + 1.0), c2 = (2.0 * lc + 1.0) / (lc + 1.0);
#pragma unroll
    for (int u = 0; u < 4; ++u) W[ll][cs + 16 * u] = l0 + ll < L ? (2.0 * lc + 1.0) * pu[u] * pb[u] : 0.0;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      if (i / 4 == wv) Pl[i][lane] = (i & 1) && flip ? -pl : pl;   // l0 is even
      dl = lane_value(c1, i) * dl - lane_value(c2, i) * y * pl;
      pl += dl;
    }
    __syncthreads();
    if (l0 + NK < L) load(l0 + NK);
#pragma unroll
    for (int ks = 0; ks < NK / 4; ++ks) {
      const int kk = 4 * ks + kq;
      double a[2], b[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        a[t] = Pl[kk][32 * wr + 16 * t + l16];
        b[t] = W[kk][32 * wc + 16 * t + l16];
      }
#pragma unroll
      for (int ta = 0; ta < 2; ++ta)
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) acc[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ta], b[tb], acc[ta][tb], 0, 0, 0);
    }
    __syncthreads();
  }
  const int ncol = PAIRS ? pad_to(nrow, NT) : nrow, nnode = PAIRS ? pad_to(nmu, NK) : nmu;
#pragma unroll
  for (int tb = 0; tb < 2; ++tb) {
    const int c = c0 + 32 * wc + 16 * tb + l16;
    if (c >= ncol) continue;
#pragma unroll
    for (int ta = 0; ta < 2; ++ta)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = k0 + 32 * wr + 16 * ta + 4 * r + kq;
        if (k < nnode)
          F[PAIRS ? (size_t)k * ncol + c : ((size_t)(c / P) * nmu + k) * P + c % P] = k < nmu ? acc[ta][tb][r] : 0.0;
      }
  }
}

// alpha[n] = 1/(48 pi) sum_k w_k sum_t sum_sigma F[3t + sigma1][k][p] F[3t + sigma2][k][q] F[3t + sigma3][k][r]
// A workgroup takes AMC modes, its threads AMP phases of the nodes k; the phases are added
// in a fixed order through LDS.
constexpr int AMC = 32;
constexpr int AMP = 256 / AMC;

__global__ __launch_bounds__(256) void k_alpha_modes(int nmax, int P, int T, int nmu, const int* __restrict__ tri,
                                                     const double* __restrict__ F, const double* __restrict__ wmu,
                                                     double* __restrict__ alpha) {
  __shared__ double red[AMP][AMC];
  const int ml = threadIdx.x % AMC, ph = threadIdx.x / AMC;
  const int n = blockIdx.x * AMC + ml;
  double acc = 0.0;
  if (n < nmax) {
    const int p = tri[6 * n], q = tri[6 * n + 1], r = tri[6 * n + 2];
    for (int k = ph; k < nmu; k += AMP) {
      double sm = 0.0;
      for (int t = 0; t < T; ++t) {
        const double* X = F + ((size_t)(3 * t) * nmu + k) * P;
        const double* Y = X + (size_t)nmu * P;
        const double* Z = Y + (size_t)nmu * P;
        const double xp = X[p], xq = X[q], xr = X[r], yp = Y[p], yq = Y[q], yr = Y[r], zp = Z[p], zq = Z[q], zr = Z[r];
        sm += xp * (yq * zr + zq * yr) + yp * (xq * zr + zq * xr) + zp * (xq * yr + yq * xr);
      }
      acc = fma(wmu[k], sm, acc);
    }
  }
  red[ph][ml] = acc;
  __syncthreads();
  if (ph == 0 && n < nmax) {
    double s = 0.0;
    for (int i = 0; i < AMP; ++i) s += red[i][ml];
    alpha[n] = s * (1.0 / (48.0 * 3.14159265358979323846));
  }
}

// T_ijk, i <= j <= k, is stored at (triples with a smaller i) + (with this i, a smaller j) + k - j.
__host__ __device__ inline size_t tet(size_t n) { return n * (n + 1) * (n + 2) / 6; }
__host__ __device__ inline size_t tri2(size_t n) { return n * (n + 1) / 2; }
// pairs of i that the row tile rt needs (i <= j)
__host__ __device__ inline int node_pairs(int N, int rt) { return ((N < NT * (rt + 1) ? N : NT * (rt + 1)) + 1) / 2; }

// T_ijk on the FP64 matrix cores (v_mfma_f64_16x16x4_f64, the layout of k_linalg.hip): for two
// i at a time, the 64 x 64 tile (j, k) of Q_j (w Q_i) Q_k over the nodes.  A workgroup's four
// waves are two i x two halves of the columns; the tiles of Q_j and Q_k are staged once for
// both i, which halves the L2 reads per multiply (the tile pair's nodes, 0.8 MB at l_max 500,
// come from L2 for every i), and w Q_i multiplies the row operand as it is read.  Bound by
// the matrix cores: of the cells formed 28 % lie outside i <= j <= k for 465 pairs, 16 % for 820.  At
// l_max 500, P 30: 756 us, 46 TF with the cells outside (a plain FP64 library product reaches
// 72 on this card); the six-term permanents formed per entry and node on the vector ALUs took
// 14.3 ms.  At l_max 1000, P 40: 5.6 ms (143 ms).
__global__ __launch_bounds__(256, 3) void k_node_triples(int N, int nmu, const double* __restrict__ Q,
                                                      const double* __restrict__ wmu, double* __restrict__ T) {
  const int nt = (N + NT - 1) / NT;
  int rt = nt - 1, b = blockIdx.x;   // tile pairs rt <= ct, the long rows of i first
  while (b >= (nt - rt) * node_pairs(N, rt)) b -= (nt - rt) * node_pairs(N, rt), --rt;
  const int ct = rt + b / node_pairs(N, rt), i0 = 2 * (b % node_pairs(N, rt));
  __shared__ __attribute__((aligned(16))) double Qj[NK][NS], Qk[NK][NS], wi[2][NK];
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const int wr = wv >> 1, wc = wv & 1;
  const int j0 = NT * rt, k0 = NT * ct;
  d4 acc[4][2];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
  // two nodes' rows of 64 pairs per wave and load; Q's padding (zero nodes, repeated pairs)
  // keeps every load inside without a clamp
  constexpr int NL = NK * NT / 512;
  const int np = pad_to(N, NT), kk0 = tid >> 5, c2 = 2 * (tid & 31);
  const double *gj = Q + (size_t)kk0 * np + j0 + c2, *gk = Q + (size_t)kk0 * np + k0 + c2;
  const int wk = tid & (NK - 1);
  const double* gi = Q + (size_t)wk * np + i0 + ((tid >> 4) & 1);
  d2 pj[NL], pk[NL];
  double pw = 0.0;
  auto load = [&](int x0) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      pj[u] = *reinterpret_cast<const d2*>(gj + (size_t)(x0 + 8 * u) * np);
      pk[u] = *reinterpret_cast<const d2*>(gk + (size_t)(x0 + 8 * u) * np);
    }
    if (tid < 2 * NK) pw = wmu[min(x0 + wk, nmu - 1)] * gi[(size_t)x0 * np];
  };
  // the wave's first row tile that holds a j >= i (uniform); none if its columns lie below the
  // rows' or past the last pair
  const int i = i0 + wr, kend = min(N, k0 + 32 * wc + 32);
  const int first = i >= N || k0 + 32 * wc >= N || kend <= max(i, j0) ? 4 : i <= j0 ? 0 : (i - j0) / 16;
  auto step = [&](auto fa) {
    constexpr int FA = decltype(fa)::value;
#pragma unroll
    for (int ks = 0; ks < NK / 4; ++ks) {
      const int kk = 4 * ks + kq;
      const double wq = wi[wr][kk];
      double a[4], b[2];
#pragma unroll
      for (int t = FA; t < 4; ++t) a[t] = wq * Qj[kk][16 * t + l16];
#pragma unroll
      for (int t = 0; t < 2; ++t) b[t] = Qk[kk][32 * wc + 16 * t + l16];
#pragma unroll
      for (int ta = FA; ta < 4; ++ta)
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) acc[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ta], b[tb], acc[ta][tb], 0, 0, 0);
    }
  };
  load(0);
  for (int x0 = 0; x0 < nmu; x0 += NK) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      *reinterpret_cast<d2*>(&Qj[kk0 + 8 * u][c2]) = pj[u];
      *reinterpret_cast<d2*>(&Qk[kk0 + 8 * u][c2]) = pk[u];
    }
    if (tid < 2 * NK) wi[tid / NK][wk] = pw;
    __syncthreads();
    if (x0 + NK < nmu) load(x0 + NK);
    if (first == 0) step(std::integral_constant<int, 0>{});
    else if (first == 1) step(std::integral_constant<int, 1>{});
    else if (first == 2) step(std::integral_constant<int, 2>{});
    else if (first == 3) step(std::integral_constant<int, 3>{});
    __syncthreads();
  }
  if (i >= N) return;
  const size_t ib = tet(N) - tet(N - i) + tri2(N - i);
#pragma unroll
  for (int ta = 0; ta < 4; ++ta)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = j0 + 16 * ta + 4 * r + kq;
      if (j < i || j >= N) continue;
      double* row = T + (ib - tri2(N - j)) - j;
#pragma unroll
      for (int tb = 0; tb < 2; ++tb) {
        const int k = k0 + 32 * wc + 16 * tb + l16;
        if (k >= j && k < N) row[k] = acc[ta][tb][r];
      }
    }
}

// zeta0_nm = scale times the permanent's six triples of pairs, 64 x 64 entries per workgroup of
// the lower triangle, mirrored through LDS.  Bound by the reads of T: six 8-byte gathers
// per entry, of which the columns of a run of equal (d, e) read neighbouring places: 0.27 ms
// for 4960^2 entries, 1.5 ms for 11,480^2.
constexpr int GT = 64;
__global__ __launch_bounds__(256) void k_ideal_gather(int nmax, int P, int N, const int* __restrict__ tri,
                                                      const int* __restrict__ pair_of, const double* __restrict__ T,
                                                      double* __restrict__ Z) {
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bj > bi) return;
  extern __shared__ unsigned char graw[];
  double(*out)[GT + 1] = reinterpret_cast<double(*)[GT + 1]>(graw);
  uint32_t* ib = reinterpret_cast<uint32_t*>(graw + sizeof(double) * GT * (GT + 1));   // T's offsets by i
  uint32_t* jb = ib + N;                                                                // and by j
  uint16_t* pof = reinterpret_cast<uint16_t*>(jb + N);
  for (int e = threadIdx.x; e < N; e += 256) {
    ib[e] = (uint32_t)(tet(N) - tet(N - e) + tri2(N - e));
    jb[e] = (uint32_t)(tri2(N - e) + e);
  }
  for (int e = threadIdx.x; e < P * P; e += 256) pof[e] = (uint16_t)pair_of[e];
  __syncthreads();
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  auto at = [&](int x, int y, int z) {
    const int lo = min(x, y), hi = max(x, y);
    const int i = min(lo, z), k = max(hi, z), j = max(lo, min(hi, z));
    return T[(size_t)(uint32_t)(ib[i] - jb[j] + (uint32_t)k)];
  };
  const double scale = 1.0 / (48.0 * 3.14159265358979323846);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int* tr = tri + 6 * min(bi * GT + ty + 16 * u, nmax - 1);
    const uint16_t *pa = pof + tr[0] * P, *pb = pof + tr[1] * P, *pc = pof + tr[2] * P;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int* tc = tri + 6 * min(bj * GT + tx + 16 * v, nmax - 1);
      const int d = tc[0], e = tc[1], f = tc[2];
      const int ad = pa[d], ae = pa[e], af = pa[f], bd = pb[d], be = pb[e], bf = pb[f], cd = pc[d], ce = pc[e], cf = pc[f];
      const double s = ((at(ad, be, cf) + at(ae, bd, cf)) + (at(ad, bf, ce) + at(af, bd, ce))) +
                       (at(ae, bf, cd) + at(af, be, cd));
      out[ty + 16 * u][tx + 16 * v] = scale * s;
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < GT * GT; e += 256) {
    const int r = e / GT, q = e - r * GT;
    const int n = bi * GT + r, m = bj * GT + q;
    if (n < nmax && m < nmax) Z[(size_t)n * nmax + m] = bi == bj && q > r ? out[q][r] : out[r][q];
    if (bi != bj) {   // the mirrored tile, rows of the block bj
      const int n2 = bj * GT + r, m2 = bi * GT + q;
      if (n2 < nmax && m2 < nmax) Z[(size_t)n2 * nmax + m2] = out[q][r];
    }
  }
}

}  // namespace

int shapes_nmu(int lmax) { return (3 * lmax + 2) / 2; }

hipError_t launch_legendre_series(int L, int nmu, int P, int nf, const double* U, const double* B, const double* mu,
                                  double* F, hipStream_t st) {
  hipLaunchKernelGGL(k_legendre_series<false>, dim3((nmu + NT - 1) / NT, (nf * P + NT - 1) / NT), dim3(256), 0, st, L,
                     nmu, P, nf * P, (const int*)nullptr, (const int*)nullptr, U, B, mu, F);
  return hipGetLastError();
}

hipError_t launch_pair_series(int L, int nmu, int P, const int* pair_a, const int* pair_b, const double* U,
                              const double* B, const double* mu, double* Q, hipStream_t st) {
  const int N = P * (P + 1) / 2;
  hipLaunchKernelGGL(k_legendre_series<true>, dim3((nmu + NT - 1) / NT, (N + NT - 1) / NT), dim3(256), 0, st, L, nmu, P,
                     N, pair_a, pair_b, U, B, mu, Q);
  return hipGetLastError();
}

hipError_t launch_alpha_modes(int nmax, int P, int T, int nmu, const int* tri, const double* F, const double* wmu,
                              double* alpha, hipStream_t st) {
  hipLaunchKernelGGL(k_alpha_modes, dim3((nmax + AMC - 1) / AMC), dim3(256), 0, st, nmax, P, T, nmu, tri, F, wmu, alpha);
  return hipGetLastError();
}

size_t ideal_triples_bytes(int npairs) { return tet(npairs) * 8; }
size_t ideal_series_bytes(int npairs, int nmu) { return (size_t)pad_to(npairs, NT) * pad_to(nmu, NK) * 8; }

hipError_t launch_ideal_cov(int nmax, int P, int nmu, const int* tri, const int* pair_of, const double* Q,
                            const double* wmu, double* T, double* Z, hipStream_t st) {
  const int N = P * (P + 1) / 2, nt = (N + NT - 1) / NT;
  int blocks = 0;
  for (int rt = 0; rt < nt; ++rt) blocks += (nt - rt) * node_pairs(N, rt);
  hipLaunchKernelGGL(k_node_triples, dim3(blocks), dim3(256), 0, st, N, nmu, Q, wmu, T);
  const int ng = (nmax + GT - 1) / GT;
  const size_t lds = sizeof(double) * GT * (GT + 1) + 8 * (size_t)N + 2 * (size_t)P * P;   // < 64 KB at P 64
  hipLaunchKernelGGL(k_ideal_gather, dim3(ng, ng), dim3(256), lds, st, nmax, P, N, tri, pair_of, T, Z);
  return hipGetLastError();
}

}  // namespace modal
