// Modal trispectrum (Sec. IV): for separable modes q_p q_r q_s q_u, p <= r <= s <= u,
//   tau_prsu = sum_x w [M_p M_r M_s M_u - (6 pairs) V_ab M_c M_d + (3 pairings) V_ab V_cd].
// Rearranged exactly as a symmetric rank-npix update over the pairs:
//   K_(ab),(cd) = sum_x w A_ab A_cd - 6 sum_x w V_ab V_cd,   A_ab = M_a M_b - 3 V_ab,
//   tau_prsu = (K_(pr),(su) + K_(ps),(ru) + K_(pu),(rs)) / 3,
// since the three pairings of A A expand to 3 MMMM - 3 (6 pairs) V M M + 9 (3 pairings) V V.
// Without a linear-term state V = 0.  The V V term is sky-independent and formed once
// per call as one more sky of the same launch, with A = V.
//
// The update is a pairs x pairs SYRK with K = pixels.  Operands sqrt(w) A are formed on
// the fly (w >= 0 splits evenly over both sides), never stored in HBM:
//   * float maps (bf16x3 / f16x3 contexts): split-bf16 MFMA 32x32x16 with three
//     products, 128 x 128 output tiles, two skies per workgroup, operands of the next 32
//     pixels formed into LDS between the products of these (each thread 4 pixels of 4
//     operand rows of both skies), maps and pair means read from pixel-block-major copies
//     (k_quad_vtile), FP32 chains of CH steps joined in FP32, FP32 partial sums per pixel
//     chunk reduced in FP64.  Bound by the operands' vector work (about 240 instructions per
//     wave and step against 24 products) and the two barriers of a step; one workgroup per CU (150
//     KB of LDS).  4 skies, 465 pairs, 1.18 M pixels, with pair means: 13.7 ms for the skies and 5.5
//     for the means with a sky per half, operands and products in turn (three barriers, one operand
//     buffer) and means exchanged through LDS; 9.1 ms for both in one launch with the two
//     overlapped, 7.5 now with the longest workgroups first and a row's next means loaded in place;
//   * double maps (f64 contexts): FP64 on the vector ALUs, 64 x 64 tiles, 4 x 4 per thread.
#include "common.h"

#include <algorithm>

namespace modal {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int TT = 128;      // output tile of the MFMA kernel (rows = cols)
constexpr int PXS = 32;      // pixels per staged step (two MFMA K = 16 steps)
constexpr int MPS = PXS + 4; // map row stride in LDS (floats; rows stay 16-byte aligned)
constexpr int CH = 16;       // staged steps per MFMA accumulation chain (96 MFMAs per tile)
constexpr int GPR = PXS / 4; // 4-pixel groups per row
constexpr int NTQ = 512;     // threads
constexpr int RPT = 2 * TT * GPR / NTQ;   // operand rows per thread (4)
constexpr int SKW = 2;       // skies per workgroup: the pair means are loaded once for both

struct TriLds {
  // operand words, two steps in turn; rows 0..127 of tile ti, then tile tj's.  A row is four
  // 16-byte quads, quad q at place q ^ ((row >> 2) & 3): 16 rows' reads of a quad fill the banks.
  uint16_t oh[2][SKW][2 * TT][PXS];
  uint16_t ol[2][SKW][2 * TT][PXS];
  float ms[SKW][kMaxP][MPS];
  float sw[PXS];           // sqrt(w)
};

__device__ inline uint32_t bf16_pair(float a, float b) {
  typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
  bf16x2 h;
  h[0] = (__bf16)a;
  h[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, h);
}

// hi = RNE bf16(v), lo = RNE bf16(v - hi) of two values, packed
__device__ inline void split2(float v0, float v1, uint32_t& hi, uint32_t& lo) {
  asm("" : "+v"(v0), "+v"(v1));
  hi = bf16_pair(v0, v1);
  lo = bf16_pair(v0 - __builtin_bit_cast(float, hi << 16), v1 - __builtin_bit_cast(float, hi & 0xffff0000u));
}

// One chunk of one tile pair (ti, tj), ti <= tj, for NSK skies s0, s0 + 1 (index S: the pair means
// themselves, A = V, formed as 0 * 0 + 1 * V): part[s][c][tp][TT][TT], the FP32 sums of the chunk.
//   * thread t forms the operands of the 4 pixels 4 (t % 8) .. + 3 of the rows t / 8 + 64 j,
//     j < 4 (j < 2 in tile ti), for both skies: it loads the pair means it needs straight to
//     registers, a step ahead, and reads the maps from LDS (staged a step ahead too);
//   * NSK 2: waves 0..3 multiply for sky s0 and waves 4..7 for s0 + 1, 64 x 64 each; NSK 1: all
//     eight for s0, 64 x 32 each;
//   * the operands of step k + 1 are formed between the products of step k (operand words in
//     two buffers): a group is one row and sky's words (its maps read a group ahead) and its
//     share of the products; a row's next pair means are loaded when its last sky has used them.
// DIAG: ti == tj, tile tj's operands are tile ti's and half the rows are formed.
// Rows past R compute on row R - 1's data (their outputs are not read); pixels past npix are
// zero in the block-major copies.
template <int NSK, bool DIAG, bool STATE>
__device__ __forceinline__ void quad_chunk(TriLds& L, int P, int R, int npix, int S, int s0, int2 tt, int x0, int x1,
                                           const int* __restrict__ pair_a, const int* __restrict__ pair_b,
                                           const float* __restrict__ maps, const float* __restrict__ V,
                                           const float* __restrict__ w, float* __restrict__ dst, size_t dst_sky) {
  constexpr int NB = NSK;                     // 32-column tiles per wave
  constexpr int NR = DIAG ? RPT / 2 : RPT;    // rows formed per thread
  constexpr int NG = NR * NSK, NP = 12 * NB;  // groups and products per step
  const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int h = wv >> 2, wi = (wv >> 1) & 1, wj = wv & 1;
  const int g = tid & (GPR - 1), rsub = tid / GPR;
  const int nblk = (npix + PXS - 1) / PXS, xb = x0 / PXS, n = (x1 - x0 + PXS - 1) / PXS;
  // operand rows: offsets of the two modes' maps in LDS (bytes, 16 bits each) and of V's row
  uint32_t mo[NR], vo[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    const int row = min((j < RPT / 2 ? tt.x : tt.y) * TT + rsub + 64 * (j & 1), R - 1);
    mo[j] = (uint32_t)(pair_a[row] * MPS + 4 * g) * 4 | (uint32_t)(pair_b[row] * MPS + 4 * g) * 4 << 16;
    vo[j] = (uint32_t)(row * PXS + 4 * g);
  }
  // map groups this thread stages: at most SKW kMaxP GPR / NTQ = 2
  constexpr int NML = (NSK * kMaxP * GPR + NTQ - 1) / NTQ;
  const float* mp[NML];
  f4* md[NML];
  bool mok[NML];
  const int nmg = NSK * P * GPR;
#pragma unroll
  for (int q = 0; q < NML; ++q) {
    const int e = min(tid + NTQ * q, nmg - 1), k = e / (P * GPR), r = (e - k * P * GPR) / GPR, gg = e % GPR;
    mok[q] = s0 + k < S;
    mp[q] = maps + ((size_t)min(s0 + k, S - 1) * nblk + xb) * P * PXS + r * PXS + 4 * gg;
    md[q] = reinterpret_cast<f4*>(&L.ms[k][r][4 * gg]);
  }
  float cv[NSK];   // A = M_a M_b + cv V
#pragma unroll
  for (int k = 0; k < NSK; ++k) cv[k] = s0 + k < S ? -3.f : 1.f;

  f4 pm[NML], pv[NR];
  float pw;
  auto load_maps = [&](int k) {   // steps past the chunk repeat its last
    const size_t o = (size_t)min(k, n - 1) * P * PXS;
#pragma unroll
    for (int q = 0; q < NML; ++q) pm[q] = *reinterpret_cast<const f4*>(mp[q] + o);
    pw = w[min(x0 + min(k, n - 1) * PXS + (tid & (PXS - 1)), npix - 1)];
  };
  auto load_mean = [&](int j, int k) {
    if (STATE) pv[j] = *reinterpret_cast<const f4*>(V + (size_t)(xb + min(k, n - 1)) * R * PXS + vo[j]);
  };
  auto stage_maps = [&]() {
#pragma unroll
    for (int q = 0; q < NML; ++q) {
      const f4 z = {0.f, 0.f, 0.f, 0.f};
      *md[q] = mok[q] ? pm[q] : z;
    }
    if (tid < PXS) L.sw[tid] = sqrtf(pw);
  };
  // operand words of row j, sky k into buffer b; the maps read beforehand
  const int wo = rsub * PXS + (((g >> 1) ^ ((rsub >> 2) & 3)) << 3) + 4 * (g & 1);
  auto form = [&](int j, int k, int b, const f4 ma, const f4 mb, const f4 sq) {
    const float c = cv[k];
    f4 v;
    if (STATE) {
      v.x = fmaf(ma.x, mb.x, c * pv[j].x) * sq.x;
      v.y = fmaf(ma.y, mb.y, c * pv[j].y) * sq.y;
      v.z = fmaf(ma.z, mb.z, c * pv[j].z) * sq.z;
      v.w = fmaf(ma.w, mb.w, c * pv[j].w) * sq.w;
    } else {
      v.x = ma.x * mb.x * sq.x;
      v.y = ma.y * mb.y * sq.y;
      v.z = ma.z * mb.z * sq.z;
      v.w = ma.w * mb.w * sq.w;
    }
    uint32_t h0, l0, h1, l1;
    split2(v.x, v.y, h0, l0);
    split2(v.z, v.w, h1, l1);
    *reinterpret_cast<uint2*>(&L.oh[b][k][64 * j][0] + wo) = make_uint2(h0, h1);
    *reinterpret_cast<uint2*>(&L.ol[b][k][64 * j][0] + wo) = make_uint2(l0, l1);
  };
  auto map_at = [&](int k, uint32_t o) {
    return *reinterpret_cast<const f4*>(reinterpret_cast<const unsigned char*>(&L.ms[k][0][0]) + o);
  };

  f32x16 acc[2][NB], cha[2][NB];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = cha[a][b][r] = 0.f;

  // step 0's operands
  load_maps(0);
#pragma unroll
  for (int j = 0; j < NR; ++j) load_mean(j, 0);
  stage_maps();
  load_maps(1);
  __syncthreads();
  {
    const f4 sq = *reinterpret_cast<const f4*>(&L.sw[4 * g]);
#pragma unroll
    for (int j = 0; j < NR; ++j) {
#pragma unroll
      for (int k = 0; k < NSK; ++k) form(j, k, 0, map_at(k, mo[j] & 0xffff), map_at(k, mo[j] >> 16), sq);
      load_mean(j, 1);
    }
  }
  __syncthreads();
  stage_maps();
  __syncthreads();

  // this wave's operand fragments: rows fr + 32 u of tile ti and fc + 32 u of tile tj
  const int sk = NSK == 2 ? h : 0;
  const int l32 = lane & 31, z = (l32 >> 2) & 3, kh = lane >> 5;
  const int fr = 64 * wi + l32, fc = (DIAG ? 0 : TT) + 64 * wj + (NSK == 2 ? 0 : 32 * h) + l32;
  int link = 0;
  for (int k = 0; k < n; ++k) {
    const int b = k & 1;
    load_maps(k + 2);
    const f4 sq = *reinterpret_cast<const f4*>(&L.sw[4 * g]);
    f4 ma = map_at(0, mo[0] & 0xffff), mb = map_at(0, mo[0] >> 16);
    bf16x8 ah[2], al[2], bh[NB], bl[NB];
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
      const int j = gi / NSK, k2 = gi % NSK;   // the group's row and sky
      if (gi % (NG / 2) == 0) {
        const int q = ((2 * (gi / (NG / 2)) + kh) ^ z) << 3;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          ah[u] = *reinterpret_cast<const bf16x8*>(&L.oh[b][sk][fr + 32 * u][q]);
          al[u] = *reinterpret_cast<const bf16x8*>(&L.ol[b][sk][fr + 32 * u][q]);
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
          bh[u] = *reinterpret_cast<const bf16x8*>(&L.oh[b][sk][fc + 32 * u][q]);
          bl[u] = *reinterpret_cast<const bf16x8*>(&L.ol[b][sk][fc + 32 * u][q]);
        }
      }
      f4 na = ma, nb = mb;
      if (gi + 1 < NG) {
        const int jn = (gi + 1) / NSK, kn = (gi + 1) % NSK;
        na = map_at(kn, mo[jn] & 0xffff);
        nb = map_at(kn, mo[jn] >> 16);
      }
#pragma unroll
      for (int i = 0; i < NP / NG; ++i) {   // 2 NB each of lo hi, hi lo, hi hi, in this order per output
        const int e = NP / NG * (gi % (NG / 2)) + i, t = e / (2 * NB), a = e / NB % 2, c = e % NB;
        cha[a][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(t == 0 ? al[a] : ah[a], t == 1 ? bl[c] : bh[c], cha[a][c], 0, 0, 0);
      }
      form(j, k2, b ^ 1, ma, mb, sq);
      if (k2 == NSK - 1) load_mean(j, k + 2);
      ma = na;
      mb = nb;
      __builtin_amdgcn_sched_barrier(0);
    }
    if (++link == CH || k + 1 == n) {   // uniform
      link = 0;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < NB; ++c) {
          acc[a][c] += cha[a][c];
#pragma unroll
          for (int r = 0; r < 16; ++r) cha[a][c][r] = 0.f;
        }
    }
    __syncthreads();   // every wave has read this step's words and the next step's maps
    stage_maps();
    __syncthreads();
  }
  // acc[a][c][r] = D[64 wi + 32 a + 8 (r / 4) + 4 (lane / 32) + r % 4][column fc + 32 c]
  dst += sk * dst_sky;
  const int cb = 64 * wj + (NSK == 2 ? 0 : 32 * h) + l32;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        dst[(64 * wi + 32 * a + 8 * (r >> 2) + 4 * kh + (r & 3)) * TT + cb + 32 * c] = acc[a][c][r];
}

// Units (sky pair, chunk), each with its ntp tile pairs (tpairs: off the diagonal first).  With eight
// units or more, unit u runs on XCD u % 8, with 8 or 16 chunks then all sky pairs of a chunk, so that
// the pair means come from that XCD's L2.  The means' own product is sky S of S + 1: it fills
// the last pair instead of a launch of its own.  On each XCD the longest workgroups come first:
// two skies before one, tiles off the diagonal before those on it (half the rows to form).
template <bool STATE>
__global__ __launch_bounds__(NTQ) __attribute__((amdgpu_waves_per_eu(2))) void k_quad_syrk(
    int P, int R, int npix, int S, int nchunk, int chunk_px, int ntile, const int2* __restrict__ tpairs,
    const int* __restrict__ pair_a, const int* __restrict__ pair_b, const float* __restrict__ maps,
    const float* __restrict__ V, const float* __restrict__ w, float* __restrict__ part) {
  extern __shared__ __attribute__((aligned(16))) unsigned char traw[];
  TriLds& L = *reinterpret_cast<TriLds*>(traw);
  const int ntp = ntile * (ntile + 1) / 2, noff = ntp - ntile;
  const int nsky = S + (STATE ? 1 : 0), nf = nsky / SKW * nchunk, nu = (nsky + SKW - 1) / SKW * nchunk;
  const int nx = nu >= 8 ? 8 : 1, x = blockIdx.x % nx;
  const int uf = (nf - x + nx - 1) / nx, uh = (nu - x + nx - 1) / nx - uf;   // this XCD's units of two skies, of one
  int i = blockIdx.x / nx, v = 0, q = -1;
  auto take = [&](int v0, int units, int q0, int pairs) {
    if (q >= 0) return;
    if (i < units * pairs) {
      v = v0 + i / pairs;
      q = q0 + i % pairs;
    } else {
      i -= units * pairs;
    }
  };
  take(0, uf, 0, noff);
  take(0, uf, noff, ntile);
  take(uf, uh, 0, noff);
  take(uf, uh, noff, ntile);
  if (q < 0) return;   // whole workgroup
  const int u = x + nx * v, s0 = SKW * (u / nchunk), chunk = u % nchunk;
  const int2 tt = tpairs[q];
  const int tp = tt.x * ntile - tt.x * (tt.x - 1) / 2 + tt.y - tt.x;
  const int x0 = chunk * chunk_px, x1 = min(npix, x0 + chunk_px);
  const size_t sky = (size_t)nchunk * ntp * TT * TT;
  float* dst = part + s0 * sky + ((size_t)chunk * ntp + tp) * TT * TT;
#define RUN(NSK, DIAG) quad_chunk<NSK, DIAG, STATE>(L, P, R, npix, S, s0, tt, x0, x1, pair_a, pair_b, maps, V, w, dst, sky)
  if (s0 + 1 < nsky) {
    if (tt.x != tt.y) RUN(2, false);
    else RUN(2, true);
  } else {
    if (tt.x != tt.y) RUN(1, false);
    else RUN(1, true);
  }
#undef RUN
}

// Pixel-block-major copy of the pair means: Vt[b][pair][i] = V[pair][32 b + i] (zero past
// npix).  The update reads, per 32-pixel step, 256 rows of one block: contiguous here,
// 256 separate 128-byte pieces of the pair-major planes otherwise.  A workgroup copies
// 32 rows x 8 blocks; each row is read as 1 KB runs, each block written as 4 KB runs.
__global__ __launch_bounds__(256) void k_quad_vtile(int R, int npix, int nblk, int vec, const float* __restrict__ V,
                                                    float* __restrict__ Vt) {
  const int row = blockIdx.y * 32 + (threadIdx.x >> 3), g = threadIdx.x & 7;
  if (row >= R) return;
  V += (size_t)blockIdx.z * R * npix;   // batch z: R rows of npix -> nblk blocks of R x 32
  Vt += (size_t)blockIdx.z * nblk * R * PXS;
  const float* src = V + (size_t)row * npix;
#pragma unroll
  for (int b8 = 0; b8 < 8; ++b8) {
    const int blk = blockIdx.x * 8 + b8;
    if (blk >= nblk) break;
    const int x = blk * PXS + 4 * g;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (vec && x < npix) {
      v = *reinterpret_cast<const float4*>(src + x);   // npix % 4 == 0: the group is inside
    } else if (!vec) {
      v.x = x < npix ? src[x] : 0.f;
      v.y = x + 1 < npix ? src[x + 1] : 0.f;
      v.z = x + 2 < npix ? src[x + 2] : 0.f;
      v.w = x + 3 < npix ? src[x + 3] : 0.f;
    }
    *reinterpret_cast<float4*>(Vt + ((size_t)blk * R + row) * PXS + 4 * g) = v;
  }
}

// K[s][i][j] (i, j < R, FP64, both triangles) = sum over chunks of the tile partials; sky S is KVV.
__global__ __launch_bounds__(256) void k_quad_reduce(int R, int nchunk, int ntp, int ntile, int S,
                                                     const float* __restrict__ part, double* __restrict__ K,
                                                     double* __restrict__ KVV) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int s = blockIdx.y;
  if (e >= (size_t)R * R) return;
  const int i = (int)(e / R), j = (int)(e - (size_t)i * R);
  int ti = i / TT, tj = j / TT, ii = i - ti * TT, jj = j - tj * TT;
  if (ti > tj) {   // the lower tiles are the transposes of the upper ones
    const int t = ti; ti = tj; tj = t;
    const int u = ii; ii = jj; jj = u;
  }
  const int tp = ti * ntile - ti * (ti - 1) / 2 + (tj - ti);
  double acc = 0.0;
  for (int c = 0; c < nchunk; ++c) acc += (double)part[(((size_t)s * nchunk + c) * ntp + tp) * TT * TT + ii * TT + jj];
  (s < S ? K + (size_t)s * R * R : KVV)[e] = acc;
}

// FP64 path: K[s][i][j] for a 64 x 64 tile (bi, bj), bj <= bi, mirrored; whole pixel range.
__global__ __launch_bounds__(256) void k_quad_syrk64(int P, int R, int npix, const int* __restrict__ pair_a,
                                                     const int* __restrict__ pair_b, const double* __restrict__ maps,
                                                     const double* __restrict__ V, const double* __restrict__ w,
                                                     int vmode, double* __restrict__ K) {
  constexpr int KC = 16;
  __shared__ double Ai[KC][65], Aj[KC][65];
  const int bi = blockIdx.y, bj = blockIdx.x, s = blockIdx.z;
  if (bj > bi) return;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const double* Msky = maps + (size_t)s * P * npix;
  double acc[4][4] = {};
  for (int x0 = 0; x0 < npix; x0 += KC) {
    __syncthreads();
    for (int e = threadIdx.x; e < 2 * KC * 64; e += 256) {
      const int side = e / (KC * 64), rem = e - side * KC * 64, r = rem / KC, k = rem - r * KC;
      const int row = (side ? bj : bi) * 64 + r, x = x0 + k;
      double v = 0.0;
      if (row < R && x < npix) {
        const double vv = V ? V[(size_t)row * npix + x] : 0.0;
        v = vmode ? vv : Msky[(size_t)pair_a[row] * npix + x] * Msky[(size_t)pair_b[row] * npix + x] - 3.0 * vv;
        v *= sqrt(w[x]);
      }
      (side ? Aj : Ai)[k][r] = v;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      double a[4], b[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        a[u] = Ai[k][ty * 4 + u];
        b[u] = Aj[k][tx * 4 + u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[u][v] = fma(a[u], b[v], acc[u][v]);
    }
  }
  double* Ks = K + (size_t)s * R * R;
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = bi * 64 + ty * 4 + u, j = bj * 64 + tx * 4 + v;
      if (i < R && j < R && (bi != bj || j <= i)) {
        Ks[(size_t)i * R + j] = acc[u][v];
        Ks[(size_t)j * R + i] = acc[u][v];
      }
    }
}

// tau[s][n] = (1/3) sum over the three pairings of (K[s] - 6 KVV)
__global__ __launch_bounds__(256) void k_quad_gather(int R, int nquad, int S, const int* __restrict__ quad,
                                                     const double* __restrict__ K, const double* __restrict__ KVV,
                                                     double* __restrict__ tau) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= S * nquad) return;
  const int s = e / nquad, n = e - s * nquad;
  const int* qd = quad + 6 * n;
  const double* Ks = K + (size_t)s * R * R;
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const size_t o = (size_t)qd[2 * j] * R + qd[2 * j + 1];
    acc += Ks[o] - (KVV ? 6.0 * KVV[o] : 0.0);
  }
  tau[e] = acc * (1.0 / 3.0);
}

}  // namespace

int quad_chunks(int npix) { return std::max(1, std::min(16, npix / 4096)); }
int quad_ntile(int R) { return (R + TT - 1) / TT; }
size_t quad_lds() { return sizeof(TriLds); }

hipError_t quad_set_lds() {
  hipError_t e =
      hipFuncSetAttribute((const void*)k_quad_syrk<true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(TriLds));
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)k_quad_syrk<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)sizeof(TriLds));
}

// K [S][R][R] FP64 for the S skies' maps and, with pair means V, KVV [R][R] for V itself.  For
// the float contexts the maps and V are pixel-block-major copies (launch_quad_vtile), for
// FP64 the maps and the pair-major planes of the state.
hipError_t launch_quad_syrk(const modal_ctx* c, const void* maps, const void* V, int S, const int2* tpairs, float* part,
                            double* K, double* KVV, hipStream_t st) {
  const int R = c->npairs;
  if (c->prec == MODAL_F64) {
    const int nb = (R + 63) / 64;
    auto run = [&](int skies, int vmode, double* out) {
      hipLaunchKernelGGL(k_quad_syrk64, dim3(nb, nb, skies), dim3(256), 0, st, c->P, R, c->npix, c->t.pair_a, c->t.pair_b,
                         (const double*)maps, (const double*)V, c->t.w64, vmode, out);
    };
    run(S, 0, K);
    if (V) run(1, 1, KVV);
    return hipGetLastError();
  }
  const int ntile = quad_ntile(R), ntp = ntile * (ntile + 1) / 2;
  const int nchunk = quad_chunks(c->npix);
  const int chunk_px = ((c->npix + nchunk - 1) / nchunk + PXS - 1) / PXS * PXS;
  hipError_t e = quad_set_lds();
  if (e != hipSuccess) return e;
  const int nsky = S + (V ? 1 : 0), nu = (nsky + SKW - 1) / SKW * nchunk;
  const dim3 grid((nu >= 8 ? (nu + 7) / 8 * 8 : nu) * ntp);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(NTQ), sizeof(TriLds), st, c->P, R, c->npix, S, nchunk, chunk_px, ntile, tpairs,
                       c->t.pair_a, c->t.pair_b, (const float*)maps, (const float*)V, c->t.w32, part);
  };
  if (V) run(k_quad_syrk<true>);
  else run(k_quad_syrk<false>);
  const size_t tot = (size_t)R * R;
  hipLaunchKernelGGL(k_quad_reduce, dim3((tot + 255) / 256, nsky), dim3(256), 0, st, R, nchunk, ntp, ntile, S, part, K, KVV);
  return hipGetLastError();
}

hipError_t launch_quad_gather(const modal_ctx* c, int nquad, int S, const int* quad, const double* K, const double* KVV,
                              double* tau, hipStream_t st) {
  hipLaunchKernelGGL(k_quad_gather, dim3((S * nquad + 255) / 256), dim3(256), 0, st, c->npairs, nquad, S, quad, K, KVV,
                     tau);
  return hipGetLastError();
}

size_t quad_vtile_bytes(const modal_ctx* c) {
  if (c->prec == MODAL_F64) return 0;
  return (size_t)((c->npix + PXS - 1) / PXS) * c->npairs * PXS * 4;
}

hipError_t launch_quad_vtile(const modal_ctx* c, const void* V, int rows, int batch, float* Vt, hipStream_t st) {
  const int nblk = (c->npix + PXS - 1) / PXS;
  hipLaunchKernelGGL(k_quad_vtile, dim3((nblk + 7) / 8, (rows + 31) / 32, batch), dim3(256), 0, st, rows, c->npix,
                     nblk, c->npix % 4 == 0 ? 1 : 0, (const float*)V, Vt);
  return hipGetLastError();
}

size_t quad_mtile_bytes(const modal_ctx* c, int S) {
  if (c->prec == MODAL_F64) return 0;
  return (size_t)S * ((c->npix + PXS - 1) / PXS) * c->P * PXS * 4;
}

size_t quad_part_bytes(const modal_ctx* c, int S) {   // S skies and the pair means
  if (c->prec == MODAL_F64) return 0;
  const int ntile = quad_ntile(c->npairs), ntp = ntile * (ntile + 1) / 2;
  return (size_t)(S + 1) * quad_chunks(c->npix) * ntp * TT * TT * 4;
}

}  // namespace modal
