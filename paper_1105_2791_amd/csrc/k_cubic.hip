// Cubic pixel reduction as a pair x mode contraction over pixels (FP64 contexts), and the
// reductions of the partial sums.
//
//   E_{(ab),t} = sum_x w(x) M_a(x) M_b(x) M_t(x)
//   out_prs = scale E_{(pr),s} + scale2 (L_{(pr),s} + L_{(ps),r} + L_{(rs),p})
//
// The three pairings of beta_prs are equal, so the contraction forms the cells (a <= b,
// t >= b) only and the reduction reads the one cell of a triple; with L the linear-term sums
// of k_lin_harm.hip and scale2 = -1 the second term subtracts lin_prs (eq. bbispect with the
// three pairings of the "3 C a" linear term of eq. bispectrumest).
//
// The FP32 and split contexts contract on the matrix cores in k_cubic_split.hip and use
// the reduction k_reduce_single below.
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace modal {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kChunk = 65536;  // pixels per split-K chunk that the workspace's own region holds
constexpr int kMinChunk = 64;  // pixels per chunk at least
constexpr int kTile = 32;      // pixels staged in LDS per step
// Row stride of the staged maps: 4 words modulo the 64 banks per row, so that the 16 rows x
// 2 pixels that half a wave reads together (8 bytes each) fall into different banks.
constexpr int kStride = kTile + 2;

constexpr int kRows = 32;      // pair rows per wave (two MFMA row tiles)

// FP64 contraction on the matrix cores (v_mfma_f64_16x16x4_f64: lane l holds A[l % 16][l / 16]
// and B[l / 16][l % 16], accumulator register r is D[4 r + l / 16][l % 16]): rows = pairs,
// columns = modes, inner index = pixels.  The pairs are taken by their larger mode, row
// r = b (b + 1) / 2 + a, so that the 32 rows of a wave have neighbouring b and the 16-mode
// column tiles that lie wholly below b are skipped: about half of the pair x mode cells is
// formed.  A workgroup is 128 rows (32 per wave, so that each mode value read from LDS feeds
// two MFMAs) x all modes of one pixel chunk and sky.  C1 is the number of column tiles.
// Bound by latency at small grids and by the matrix cores and the LDS at large ones.  The
// chunks are short (64 pixels on small grids) because the chunks are all that fills the GPU
// there: one 48 x 96 sky of 8 modes ran as one workgroup, 1.30 ms, when chunks were 65536
// pixels and the vector ALUs formed every cell; 6.9 us now.  Seven skies of 309 x 640 pixels
// and 50 modes: 12.1 ms with 16 rows per wave and a branch per column
// tile, 3.4 ms now (the vector-ALU kernel: 50 ms).
template <int C1>
__global__ __launch_bounds__(256) void k_cubic_f64(int P, int npairs, int npix, int nchunk, int chunk_px,
                                                   const int* __restrict__ pair_of, const double* __restrict__ maps,
                                                   const double* __restrict__ w, double* __restrict__ part) {
  __shared__ double Mt[16 * C1][kStride];
  __shared__ double wt[kTile];
  const int chunk = blockIdx.x, s = blockIdx.z;
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const int row0 = blockIdx.y * (4 * kRows) + wv * kRows;
  auto mode_b = [](int r) {   // largest b with b (b + 1) / 2 <= r
    int b = (int)((sqrtf(8.f * (float)r + 1.f) - 1.f) * 0.5f);
    while ((b + 1) * (b + 2) / 2 <= r) ++b;
    while (b * (b + 1) / 2 > r) --b;
    return b;
  };
  int ma[2], mb[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {   // rows past the last pair repeat it, never stored
    const int row = min(row0 + 16 * u + l16, npairs - 1);
    mb[u] = mode_b(row);
    ma[u] = row - mb[u] * (mb[u] + 1) / 2;
  }
  // column tiles [c0, C1), uniform per wave; a wave wholly past the last pair forms none
  const int c0 = row0 < npairs ? __builtin_amdgcn_readfirstlane(mode_b(row0) >> 4) : C1;
  const double* Ms = maps + (size_t)s * P * npix;
  const int x0c = chunk * chunk_px, x1c = min(npix, x0c + chunk_px);
  d4 acc[2][C1];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int c = 0; c < C1; ++c) acc[u][c] = d4{0.0, 0.0, 0.0, 0.0};
  // modes past P are staged as zeros: their columns are formed with the last tile, never stored
  constexpr int NL = 16 * C1 * kTile / 256;
  double pre[NL], prew;
  auto load = [&](int x0) {
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int e = tid + 256 * u, p = e / kTile, x = x0 + e % kTile;
      const double v = Ms[(size_t)min(p, P - 1) * npix + min(x, npix - 1)];
      pre[u] = (p < P && x < x1c) ? v : 0.0;
    }
    const int x = x0 + (tid & (kTile - 1));
    const double v = w[min(x, npix - 1)];
    prew = x < x1c ? v : 0.0;
  };
  // the products of one staged step over the column tiles [CA, C1)
  auto step = [&](auto ca) {
    constexpr int CA = decltype(ca)::value;
    if constexpr (CA < C1)
#pragma unroll
    for (int ks = 0; ks < kTile / 4; ++ks) {
      const int xx = 4 * ks + kq;
      const double wx = wt[xx];
      double a[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) a[u] = Mt[ma[u]][xx] * Mt[mb[u]][xx] * wx;
#pragma unroll
      for (int c = CA; c < C1; ++c) {
        const double b = Mt[16 * c + l16][xx];
#pragma unroll
        for (int u = 0; u < 2; ++u) acc[u][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b, acc[u][c], 0, 0, 0);
      }
    }
  };
  load(x0c);
  for (int x0 = x0c; x0 < x1c; x0 += kTile) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int e = tid + 256 * u;
      Mt[e / kTile][e % kTile] = pre[u];
    }
    if (tid < kTile) wt[tid] = prew;
    __syncthreads();
    if (x0 + kTile < x1c) load(x0 + kTile);
    if (c0 == 0) step(std::integral_constant<int, 0>{});
    else if (C1 > 1 && c0 == 1) step(std::integral_constant<int, C1 < 1 ? C1 : 1>{});
    else if (C1 > 2 && c0 == 2) step(std::integral_constant<int, C1 < 2 ? C1 : 2>{});
    else if (C1 > 3 && c0 == 3) step(std::integral_constant<int, C1 < 3 ? C1 : 3>{});
  }
  double* dst = part + ((size_t)s * nchunk + chunk) * npairs * P;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rr = row0 + 16 * u + 4 * r + kq;
      if (rr >= npairs) continue;
      const int b = mode_b(rr), a = rr - b * (b + 1) / 2;
      double* d = dst + (size_t)pair_of[a * P + b] * P;
#pragma unroll
      for (int c = 0; c < C1; ++c) {
        const int t = 16 * c + l16;
        if (t >= b && t < P) d[t] = acc[u][c][r];   // t >= b lies in the tiles from c0 on
      }
    }
}

// out_n = three pairings of E2
__global__ void k_symm(int nmax, int npairs, int P, int S, const int* __restrict__ tri, const double* __restrict__ E2,
                       double* __restrict__ out) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  const int s = blockIdx.y;
  if (n >= nmax) return;
  const int* tr = tri + 6 * n;  // p, r, s, pair(pr), pair(ps), pair(rs)
  const size_t o = (size_t)s * npairs * P;
  out[(size_t)s * nmax + n] = E2[o + (size_t)tr[3] * P + tr[2]] + E2[o + (size_t)tr[4] * P + tr[1]] +
                              E2[o + (size_t)tr[5] * P + tr[0]];
}

// out_n = scale * sum_c part[s][c][cell_n] + scale2 * (three pairings of E2): beta_prs is
// the one cell (pair, mode) of the contraction that holds it (any of the three pairings of
// the triple; the table of cells comes with the contraction's plan).  A workgroup takes RDN
// triples n = order[i], the triples sorted by cell, so that RDN threads read runs of
// neighbouring cells of each chunk's partial sums, and its RDP phases take every RDP-th chunk,
// added in a fixed order through LDS.  Bound by the latency of the partial sums' loads: with
// one thread per triple over all chunks, eight skies of 4960 triples in 576 chunks took 131 us, 30 us now.
constexpr int RDN = 32;
constexpr int RDP = 256 / RDN;

__global__ __launch_bounds__(256) void k_reduce_single(int nmax, int npairs, int P, int nchunk,
                                                       const int* __restrict__ tri, const int* __restrict__ cell,
                                                       const int* __restrict__ order, const double* __restrict__ part,
                                                       double scale, double scale2, const double* __restrict__ E2,
                                                       double* __restrict__ out) {
  __shared__ double red[RDP][RDN];
  const int il = threadIdx.x % RDN, ph = threadIdx.x / RDN;
  const int i = blockIdx.x * RDN + il;
  const int s = blockIdx.y;
  const int n = order[min(i, nmax - 1)];
  const size_t per = (size_t)npairs * P;
  const double* src = part + (size_t)s * nchunk * per + (size_t)cell[n];
  double v = 0.0;
#pragma unroll 8
  for (int c = ph; c < nchunk; c += RDP) v += src[(size_t)c * per];
  red[ph][il] = v;
  __syncthreads();
  if (ph != 0 || i >= nmax) return;
  v = 0.0;
#pragma unroll
  for (int k = 0; k < RDP; ++k) v += red[k][il];
  v *= scale;
  if (E2) {
    const int* tr = tri + 6 * n;
    const size_t o = (size_t)s * per;
    v += scale2 * (E2[o + (size_t)tr[3] * P + tr[2]] + E2[o + (size_t)tr[4] * P + tr[1]] +
                   E2[o + (size_t)tr[5] * P + tr[0]]);
  }
  out[(size_t)s * nmax + n] = v;
}

}  // namespace

hipError_t launch_reduce_single(const modal_ctx* c, const double* part, int S, int nchunk, double scale,
                                const double* E2, double scale2, double* out, hipStream_t st) {
  if (!c->t.cell || !c->t.cell_order) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_reduce_single, dim3((c->nmax + RDN - 1) / RDN, S), dim3(256), 0, st, c->nmax, c->npairs, c->P,
                     nchunk, c->t.tri, c->t.cell, c->t.cell_order, part, scale, scale2, E2, out);
  return hipGetLastError();
}

int cubic_nchunk_ws(const modal_ctx* c) { return (c->npix + kChunk - 1) / kChunk; }

// Chunks of the FP64 contraction: enough for four workgroups per CU per sky (128 pairs each),
// of at least kMinChunk pixels, as many as the ring coefficients' region holds.  It does not
// depend on the number of skies, so a sky's sums do not depend on its batch.
int cubic_nchunk(const modal_ctx* c) {
  const int want = std::min((c->npix + kMinChunk - 1) / kMinChunk, std::max(64, 1024 / ((c->npairs + 4 * kRows - 1) / (4 * kRows))));
  const size_t room = f_bytes_per_sky(c) / ((size_t)c->npairs * c->P * 8);
  return std::max(cubic_nchunk_ws(c), (int)std::min<size_t>(want, room));
}

hipError_t launch_cubic_f64(const modal_ctx* c, const void* maps, int S, double* part, hipStream_t st) {
  // FP64 contexts only: the others contract in k_cubic_split.hip
  if (!is_f64(c)) return hipErrorInvalidValue;
  const int nchunk = cubic_nchunk(c);
  const int per = (c->npix + nchunk - 1) / nchunk, chunk_px = (per + kTile - 1) / kTile * kTile;
  dim3 grid(nchunk, (c->npairs + 4 * kRows - 1) / (4 * kRows), S);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, c->P, c->npairs, c->npix, nchunk, chunk_px, c->t.pair_of,
                       (const double*)maps, c->t.w64, part);
  };
  static_assert(kMaxP == 64, "column tiles");
  if (c->P <= 16) launch(k_cubic_f64<1>);
  else if (c->P <= 32) launch(k_cubic_f64<2>);
  else if (c->P <= 48) launch(k_cubic_f64<3>);
  else launch(k_cubic_f64<4>);
  return hipGetLastError();
}

hipError_t launch_symm(const modal_ctx* c, int S, const double* E2, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_symm, dim3((c->nmax + 255) / 256, S), dim3(256), 0, st, c->nmax, c->npairs, c->P, S, c->t.tri, E2,
                     out);
  return hipGetLastError();
}

}  // namespace modal
