// Legendre synthesis of the FP32 contexts on the matrix cores, recurrence computed on the fly.
//
// For each m: F_c(theta_j) = sum_l Lambda[j][l] Coef[l][c],
//   Lambda[j][l] = lambda_lm(theta_j)  (north rings j, FP64 three-term recurrence),
//   Coef[l][c]   = qw_p(l) Re/Im a_{s,lm}  (column c = (s, p, re/im)),
// a GEMM with M = rings, N = columns, K = l, split by the parity of l - m so that
// F_north = E + O and F_south = E - O (lambda_lm(-x) = (-1)^{l+m} lambda_lm(x)).
//
// Workgroup = 4 waves = 256 north rings (64 per wave, one lane per ring in the
// recurrence) x 64 columns, one m.  Per chunk of 64 consecutive l (32 of each
// parity): every lane advances its ring's recurrence (FP64) and writes lambda to the
// wave's LDS tile; the workgroup writes the coefficient tile; then each wave runs
// the 2 parities x 4 ring tiles x 4 column tiles of v_mfma_f32_16x16x4_f32, a chain of
// eight per chunk that starts from zero and joins the running sum with a vector add.
// Output goes through LDS so that F (f_index layout) is written in runs of rings.
//
// Bound by the matrix cores (256 MFMAs of 32 cycles per wave and chunk) and by what keeps them
// waiting.  What took the time before, at l_max 500, 768 rings, 480 columns (2.75 ms; 17.7 ms at
// l_max 1000, 1536 rings, 640 columns), and what is done about it:
//   * tiles of 32 l per ring, in which the 16 lanes of an MFMA row read one LDS bank: tiles in
//     operand order, free of conflicts, and hardly a register spilled (1.06 ms; of the kernels
//     below the one with a table and three ring tiles keeps 20 bytes per lane in memory);
//   * half-empty workgroups (384 north rings are one and a half of 256): rings spread evenly
//     over workgroups and waves (0.87 ms);
//   * the recurrence, repeated by each block of 64 columns: from three blocks on lambda comes
//     from a table in operand order, built into the maps' memory, which is free until the ring
//     transform (0.71 + 0.07 ms), with loads that no branch separates from their waits;
//   * 64-bit addresses of the mode coefficients: 32-bit offsets (0.69 + 0.07 ms; 4.4 + 0.42 ms
//     at l_max 1000).
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace modal {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int LCH = 64;    // l per chunk
constexpr int LH = 32;     // l per parity per chunk
constexpr int RW = 64;     // rings per wave at most (NRT tiles of 16)
constexpr int NCOL = 64;   // columns per workgroup
constexpr int NWAVE = 4;
constexpr int CPT = NCOL * LH / (64 * NWAVE);   // columns a thread stages per chunk
static_assert(RW == 64 && NCOL == 64, "one tile row per 64 LDS banks");

constexpr int COEF_F = 2 * LH * NCOL;   // floats of the coefficient tile
constexpr int LAM_F = 2 * LH * RW;      // floats of a wave's lambda tile
constexpr int SS = NCOL + 1;            // output staging row
constexpr size_t kLds = sizeof(float) * (COEF_F + NWAVE * LAM_F);
static_assert(RW * SS <= LAM_F + COEF_F / NWAVE, "the output staging reuses the tiles");

__device__ inline double lane_value(double v, int i) {   // lane i's v, i uniform
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, i), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), i);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

__device__ inline int wave_min(int v) {
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return __builtin_amdgcn_readfirstlane(v);
}

// Tile positions (floats) of the value (parity, index i of the chunk's l, ring or column): in
// the order of the MFMA operands, 64 lanes (16 rings or columns x 4 groups of 8 l) of one k
// after the other, so that an operand read is 64 consecutive words at a constant offset.
// lambda is written with the 64 rings over the lanes: the four ring tiles go to different
// banks by the XOR with the l group.
__device__ inline int lam_at(int par, int rt, int k, int kg, int row) {
  return ((par * 4 + rt) * 8 + k) * 64 + (((kg ^ rt) << 4) | row);
}
__device__ inline int coef_at(int par, int ct, int k, int kg, int row) {
  return ((par * 4 + ct) * 8 + k) * 64 + ((kg << 4) | row);
}

// Output of a wave: N = E + O, then S = E - O, through its [RW][NCOL + 1] float slab of the idle
// tiles, so that F is written in runs of rings.  All waves of the workgroup call it.
template <int NRT>
__device__ inline void store_rings(const f32x4 (&acc)[2][NRT][4], float* stg, int lane, int jring, bool ring_ok, int c0,
                                   int ncols, int m, int lmax, int ntheta, float2* __restrict__ F) {
  const int row = lane & 15, kg = lane >> 4;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const float sg = half ? -1.f : 1.f;
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
      for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          stg[(16 * rt + 4 * kg + r) * SS + 16 * ct + row] = acc[0][rt][ct][r] + sg * acc[1][rt][ct][r];
    __syncthreads();
    if (ring_ok) {
      const int jw = half ? ntheta - 1 - jring : jring;
      if (!(half && jw == jring)) {
        const size_t step = f_index(1, 0, 0, lmax, f_ring_blocks(ntheta));   // from one sequence to the next
        float2* dst = F + f_index(c0 >> 1, jw, m, lmax, f_ring_blocks(ntheta));
        const int nc = min(NCOL, ncols - c0);
#pragma unroll 4
        for (int c = 0; c < nc; c += 2, dst += step) *dst = make_float2(stg[lane * SS + c], stg[lane * SS + c + 1]);
      }
    }
    __syncthreads();
  }
}

// The largest byte offset of a coefficient from its block's first sky fits in 32 bits: a block's
// 32 sequences (s, p) reach at most 1 + 30 / P skies past the one it starts in.
constexpr bool offsets_fit(int lmax, int P, int S) {
  const uint64_t nalm = (uint64_t)(lmax + 1) * (lmax + 2) / 2;
  const uint64_t past = S - 1 < 1 + 30 / P ? S - 1 : 1 + 30 / P;
  return 8 * (past * nalm + lmax) + 4 <= UINT32_MAX;
}
static_assert(offsets_fit(5883, 1, 1000) && !offsets_fit(5884, 1, 32) && offsets_fit(5884, 1, 31), "32 skies of P 1");
static_assert(offsets_fit(8190, 2, 1000) && !offsets_fit(8191, 2, 1000) && offsets_fit(8191, 2, 16), "17 skies of P 2");

// A thread's part of the coefficient tile: index ci of both parities, columns cc + 8 u (eight
// columns x four l groups x two k over a wave: two lanes per bank, 64-byte runs of l).  The
// offsets are byte offsets from uniform bases (the block's first sky, the mode functions), in 32
// bits (Off) where they fit, so that a load costs one add; 64-bit addresses formed per load were
// most of the kernel's vector instructions.  Columns past the last repeat it and are not stored.
template <typename Off>
struct CoefLoader {
  int ci, ck, cc, kg;
  Off ao[CPT];
  uint32_t qo[CPT];
  const char *ab, *qb;
  float a[CPT][2], q[CPT][2];
  __device__ inline void init(int wv, int lane, int c0, int ncols, int P, int nalm, int lmax, const float* alm,
                              const float* qw, size_t off, int m) {
    kg = lane >> 4;
    ck = 2 * wv + ((lane >> 3) & 1);
    ci = 8 * kg + ck;
    cc = lane & 7;
    const int s0 = (c0 >> 1) / P;
    ab = reinterpret_cast<const char*>(alm + 2 * ((size_t)s0 * nalm + off - m));
    qb = reinterpret_cast<const char*>(qw);
#pragma unroll
    for (int u = 0; u < CPT; ++u) {   // column parity (re, im) is cc's: 8 u is even
      const int sq = min(c0 + cc + 8 * u, ncols - 1) >> 1, s = sq / P;
      ao[u] = (Off)(s - s0) * (Off)nalm * 8u + 4u * (cc & 1);
      qo[u] = (uint32_t)(sq - s * P) * (uint32_t)(lmax + 1) * 4u;
    }
  }
  __device__ inline void load(int l0, int lmax) {
    const uint32_t lc0 = min(l0 + 2 * ci, lmax), lc1 = min(l0 + 2 * ci + 1, lmax);
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      a[u][0] = *reinterpret_cast<const float*>(ab + (ao[u] + 8u * lc0));
      a[u][1] = *reinterpret_cast<const float*>(ab + (ao[u] + 8u * lc1));
      q[u][0] = *reinterpret_cast<const float*>(qb + (qo[u] + 4u * lc0));
      q[u][1] = *reinterpret_cast<const float*>(qb + (qo[u] + 4u * lc1));
    }
  }
  __device__ inline void store(int l0, int lmax, float* coef) const {
    const bool in0 = l0 + 2 * ci <= lmax, in1 = l0 + 2 * ci + 1 <= lmax;
    float* dst = coef + coef_at(0, 0, ck, kg, cc);
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      dst[coef_at(0, u >> 1, 0, 0, 8 * (u & 1))] = in0 ? q[u][0] * a[u][0] : 0.f;
      dst[coef_at(1, u >> 1, 0, 0, 8 * (u & 1))] = in1 ? q[u][1] * a[u][1] : 0.f;
    }
  }
};

// NRT: ring tiles of 16 per wave.  The host spreads the rings evenly over the workgroups and
// waves: 384 north rings are two workgroups of four waves of 48 rings, not one and a half of 64.
template <int NRT, typename Off>
__global__ __launch_bounds__(256, 2) void k_legendre_f32(int lmax, int ntheta, int nrp, int P, int ncols, int nalm,
                                                         const double* __restrict__ x, const double* __restrict__ rec,
                                                         const double* __restrict__ seed,
                                                         const int* __restrict__ lstart, const float* __restrict__ qw,
                                                         const float* __restrict__ alm, float2* __restrict__ F) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int m = blockIdx.z;
  const int c0 = blockIdx.x * NCOL;
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  const int row = lane & 15, kg = lane >> 4;
  const int jring = (blockIdx.y * NWAVE + wv) * (16 * NRT) + lane;
  const bool ring_ok = lane < 16 * NRT && jring < nrp;
  const size_t off = (size_t)m * (2 * lmax + 3 - m) / 2;
  float* coef = lds;
  float* lam = lds + COEF_F + wv * LAM_F;

  double l1 = 0.0, l2 = 0.0, s0 = 0.0, s1 = 0.0, xx = 0.0;   // lambda_{l-1}, lambda_{l-2}, the seeds at ls, ls + 1
  int ls = lmax + 1;
  if (ring_ok) {
    xx = x[jring];
    ls = lstart[(size_t)m * nrp + jring];
    s0 = seed[2 * ((size_t)m * nrp + jring)];
    s1 = seed[2 * ((size_t)m * nrp + jring) + 1];
  }
  // the wave's first significant l, and the first l from which every ring's recurrence runs
  const int wlmin = wave_min(ls), wrun = -wave_min(-(ring_ok ? ls : -2)) + 2;
  if (lane == 0) lds[wv] = __builtin_bit_cast(float, wlmin);
  __syncthreads();
  int lmin = lmax + 1;
#pragma unroll
  for (int w = 0; w < NWAVE; ++w) lmin = min(lmin, __builtin_bit_cast(int, lds[w]));
  lmin = __builtin_amdgcn_readfirstlane(lmin);
  __syncthreads();

  f32x4 acc[2][NRT][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < NRT; ++b)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[a][b][c] = f32x4{0.f, 0.f, 0.f, 0.f};

  CoefLoader<Off> cl;
  cl.init(wv, lane, c0, ncols, P, nalm, lmax, alm, qw, off, m);

  // chunks start at l = m + 64 k so that parity(l - m) = parity(l - l0)
  const int kfirst = (lmin > m) ? (lmin - m) / LCH : 0;
  for (int l0 = m + kfirst * LCH; l0 <= lmax; l0 += LCH) {
    // ---- loads: recurrence coefficients (kRecPad entries follow the last), a_lm and q
    const double2 rc = reinterpret_cast<const double2*>(rec)[off + (l0 - m) + lane];
    cl.load(l0, lmax);
    // ---- lambda tile of this wave's rings (FP64 recurrence; past lmax the coefficients are 0)
    const bool live = l0 + LCH > wlmin && wlmin <= lmax;   // uniform: a ring of this wave has started
    if (live && l0 >= wrun) {
#pragma unroll
      for (int t = 0; t < LCH; ++t) {
        const double v = lane_value(rc.x, t) * xx * l1 - lane_value(rc.y, t) * l2;
        l2 = l1;
        l1 = v;
        lam[lam_at(t & 1, lane >> 4, (t >> 1) & 7, t >> 4, row)] = (float)v;
      }
    } else if (live) {
#pragma unroll 8
      for (int t = 0; t < LCH; ++t) {
        const int l = l0 + t;
        const double w = lane_value(rc.x, t) * xx * l1 - lane_value(rc.y, t) * l2;
        const double v = l < ls ? 0.0 : l == ls ? s0 : l == ls + 1 ? s1 : w;
        l2 = l1;
        l1 = v;
        lam[lam_at(t & 1, lane >> 4, (t >> 1) & 7, t >> 4, row)] = (float)v;
      }
    }
    // ---- coefficient tile
    __builtin_amdgcn_sched_barrier(0);
    cl.store(l0, lmax, coef);
    __syncthreads();
    // ---- MFMA (uniform per wave: skipped when all its rings are still below l_start)
    if (live) {
#pragma unroll
      for (int par = 0; par < 2; ++par) {
        float bv[4][8];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
          for (int k = 0; k < 8; ++k) bv[ct][k] = coef[coef_at(par, ct, k, kg, row)];
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) {
          float av[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) av[k] = lam[lam_at(par, rt, k, kg, row)];
          f32x4 t[4];
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) t[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) t[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[k], bv[ct][k], t[ct], 0, 0, 0);
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) acc[par][rt][ct] += t[ct];
          __builtin_amdgcn_sched_barrier(0);   // one tile row's operands at a time (registers)
        }
      }
    }
    __syncthreads();
  }

  store_rings<NRT>(acc, lds + (size_t)wv * RW * SS, lane, jring, ring_ok, c0, ncols, m, lmax, ntheta, F);
}

// ---------------------------------------------------------------------------
// the same with lambda from a table in operand order
// ---------------------------------------------------------------------------
// A record holds 16 rings x 64 l of one m, [lane = 16 (l group) + ring][16 l]: the lane's 16
// consecutive l are its A operands of both parities, so a wave reads a record as 4 KB with
// four 16-byte loads per lane and needs neither the recurrence nor the LDS for it.
constexpr int TREC = 16 * LCH;   // floats per record

__host__ __device__ inline int m_chunks(int lmax, int m) { return (lmax - m) / LCH + 1; }
// chunks of all m' < m: sum of floor(n / 64) + 1 over n = lmax - m', in closed form
__host__ __device__ inline size_t chunks_before(int lmax, int m) {
  auto upto = [](long long n) {   // sum over i in [0, n) of floor(i / 64) + 1
    const long long q = n / LCH, r = n % LCH;
    return n + LCH * q * (q - 1) / 2 + q * r;
  };
  return (size_t)(upto(lmax + 1) - upto(lmax + 1 - m));
}

// One wave per 64 rings and m: the recurrence into LDS 64 l at a time, the records out of it.
// A record wholly below its rings' first significant l is neither written nor read.
constexpr int TS = LCH + 4;      // LDS row of a ring (16-byte aligned)
__global__ __launch_bounds__(64) void k_lambda_records(int lmax, int nrp, const double* __restrict__ x,
                                                       const double* __restrict__ rec, const double* __restrict__ seed,
                                                       const int* __restrict__ lstart, float* __restrict__ tab) {
  __shared__ __attribute__((aligned(16))) float buf[64][TS];
  const int m = blockIdx.y, lane = threadIdx.x, row = lane & 15, kg = lane >> 4;
  const int jring = blockIdx.x * 64 + lane;
  const size_t off = (size_t)m * (2 * lmax + 3 - m) / 2;
  double l1 = 0.0, l2 = 0.0, s0 = 0.0, s1 = 0.0, xx = 0.0;
  int ls = lmax + 1;
  if (jring < nrp) {
    xx = x[jring];
    ls = lstart[(size_t)m * nrp + jring];
    s0 = seed[2 * ((size_t)m * nrp + jring)];
    s1 = seed[2 * ((size_t)m * nrp + jring) + 1];
  }
  int tmin = ls;   // first significant l of this lane's 16-ring tile
  for (int o = 8; o > 0; o >>= 1) tmin = min(tmin, __shfl_xor(tmin, o));
  const int wlmin = wave_min(ls), wrun = -wave_min(-(jring < nrp ? ls : -2)) + 2;
  const int ntile = (nrp + 15) / 16;
  float* out = tab + (chunks_before(lmax, m) * ntile) * TREC;
  const int kfirst = wlmin > m ? (wlmin - m) / LCH : 0;
  for (int l0 = m + kfirst * LCH, ch = kfirst; l0 <= lmax; l0 += LCH, ++ch) {
    const double2 rc = reinterpret_cast<const double2*>(rec)[off + (l0 - m) + lane];
    if (l0 >= wrun) {
#pragma unroll 16
      for (int t = 0; t < LCH; ++t) {
        const double v = lane_value(rc.x, t) * xx * l1 - lane_value(rc.y, t) * l2;
        l2 = l1;
        l1 = v;
        buf[lane][t] = (float)v;
      }
    } else {
#pragma unroll 8
      for (int t = 0; t < LCH; ++t) {
        const int l = l0 + t;
        const double w = lane_value(rc.x, t) * xx * l1 - lane_value(rc.y, t) * l2;
        const double v = l < ls ? 0.0 : l == ls ? s0 : l == ls + 1 ? s1 : w;
        l2 = l1;
        l1 = v;
        buf[lane][t] = (float)v;
      }
    }
    __syncthreads();
#pragma unroll
    for (int rt = 0; rt < 4; ++rt) {
      const int tile = blockIdx.x * 4 + rt;
      if (tile < ntile && l0 + LCH > __builtin_amdgcn_readlane(tmin, 16 * rt)) {
        float4* dst = reinterpret_cast<float4*>(out + ((size_t)ch * ntile + tile) * TREC) + 4 * lane;
#pragma unroll
        for (int q = 0; q < 4; ++q) dst[q] = *reinterpret_cast<const float4*>(&buf[16 * rt + row][16 * kg + 4 * q]);
      }
    }
    __syncthreads();
  }
}

// Workgroup as k_legendre_f32; per chunk only the coefficient tile goes through LDS (two
// buffers, one barrier per chunk).  The ring tiles run one after the other, the next one's
// record in flight, and a tile whose rings have not started is skipped.
template <int NRT>
__global__ __launch_bounds__(256, 2) void k_legendre_f32_tab(int lmax, int ntheta, int nrp, int P, int ncols, int nalm,
                                                             int nblk, int ncb,
                                                             const int* __restrict__ lstart,
                                                             const float* __restrict__ qw,
                                                             const float* __restrict__ alm,
                                                             const float* __restrict__ tab, float2* __restrict__ F) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  // unit = (m, workgroup of rings), its column blocks back to back on one XCD (workgroups are
  // dealt to the 8 XCDs round-robin), so that its records come from HBM once and from L2 after
  const int idx = blockIdx.x >> 3, unit = (idx / ncb) * 8 + (blockIdx.x & 7);
  if (unit >= nblk * (lmax + 1)) return;   // whole workgroup, before any barrier
  const int m = unit / nblk, rblk = unit % nblk;
  const int c0 = (idx % ncb) * NCOL;
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  const int row = lane & 15, kg = lane >> 4;
  const int tile0 = (rblk * NWAVE + wv) * NRT, ntile = (nrp + 15) / 16;
  const int jring = tile0 * 16 + lane;
  const bool ring_ok = lane < 16 * NRT && jring < nrp;
  const size_t off = (size_t)m * (2 * lmax + 3 - m) / 2;
  int tmin = ring_ok ? lstart[(size_t)m * nrp + jring] : lmax + 1;
  for (int o = 8; o > 0; o >>= 1) tmin = min(tmin, __shfl_xor(tmin, o));
  int tm[NRT];   // first significant l of each of the wave's tiles (uniform)
  int lmin = lmax + 1;
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) {
    tm[rt] = __builtin_amdgcn_readlane(tmin, 16 * rt);
    lmin = min(lmin, tm[rt]);
  }
  if (lane == 0) lds[wv] = __builtin_bit_cast(float, lmin);
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NWAVE; ++w) lmin = min(lmin, __builtin_bit_cast(int, lds[w]));
  lmin = __builtin_amdgcn_readfirstlane(lmin);
  __syncthreads();

  f32x4 acc[2][NRT][4];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < NRT; ++b)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[a][b][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  CoefLoader<uint32_t> cl;
  cl.init(wv, lane, c0, ncols, P, nalm, lmax, alm, qw, off, m);
  const int kfirst = (lmin > m) ? (lmin - m) / LCH : 0, nch = m_chunks(lmax, m);
  const f32x4* rec = reinterpret_cast<const f32x4*>(tab + chunks_before(lmax, m) * ntile * TREC) + 4 * lane;
  // Every load is unconditional (indices clamped; records that no ring of the tile has reached
  // hold nothing and their tile is skipped), so that a wait counts exactly the loads it needs:
  // behind branches each tile waited for the loads just issued for the next.
  auto load_rec = [&](f32x4 (&r)[4], int ch, int rt) {
    const f32x4* src = rec + ((size_t)min(ch, nch - 1) * ntile + min(tile0 + rt, ntile - 1)) * (TREC / 4);
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = src[q];
  };
  constexpr int NB = NRT == 3 ? 3 : 2;   // record buffers: tile rt reads lr[rt % NB], NRT of them end where they began
  f32x4 lr[NB][4];
  if (kfirst < nch) {
    cl.load(m + kfirst * LCH, lmax);
    load_rec(lr[0], kfirst, 0);
    cl.store(m + kfirst * LCH, lmax, lds);
  }
  for (int ch = kfirst; ch < nch; ++ch) {
    const int l0 = m + ch * LCH;
    const float* coef = lds + ((ch - kfirst) & 1) * COEF_F;
    __syncthreads();   // this chunk's tile is written, the other's reads are done
    cl.load(l0 + LCH, lmax);
    auto tile = [&](auto rt_, f32x4 (&cur)[4], f32x4 (&next)[4]) {
      constexpr int rt = decltype(rt_)::value;
      load_rec(next, rt + 1 < NRT ? ch : ch + 1, rt + 1 < NRT ? rt + 1 : 0);
      if (l0 + LCH > tm[rt]) {
#pragma unroll
        for (int par = 0; par < 2; ++par) {
          f32x4 t[4];
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) t[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
              t[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(cur[(2 * k + par) / 4][(2 * k + par) % 4],
                                                           coef[coef_at(par, ct, k, kg, row)], t[ct], 0, 0, 0);
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) acc[par][rt][ct] += t[ct];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    if (NRT > 1 || ((ch - kfirst) & 1) == 0) {
      tile(std::integral_constant<int, 0>{}, lr[0], lr[1]);
      if constexpr (NRT > 1) tile(std::integral_constant<int, 1>{}, lr[1], lr[2 % NB]);
      if constexpr (NRT > 2) tile(std::integral_constant<int, 2>{}, lr[2 % NB], lr[3 % NB]);
      if constexpr (NRT > 3) tile(std::integral_constant<int, 3>{}, lr[1], lr[0]);
    } else {   // one tile per wave: the two buffers swap per chunk
      tile(std::integral_constant<int, 0>{}, lr[1], lr[0]);
    }
    cl.store(l0 + LCH, lmax, lds + ((ch + 1 - kfirst) & 1) * COEF_F);
  }
  __syncthreads();
  store_rings<NRT>(acc, lds + (size_t)wv * RW * SS, lane, jring, ring_ok, c0, ncols, m, lmax, ntheta, F);
}

}  // namespace

size_t legendre_mfma_lds() { return kLds; }

hipError_t legendre_mfma_set_lds(size_t bytes) {
  const void* f[] = {(const void*)k_legendre_f32<1, uint32_t>, (const void*)k_legendre_f32<2, uint32_t>,
                     (const void*)k_legendre_f32<3, uint32_t>, (const void*)k_legendre_f32<4, uint32_t>,
                     (const void*)k_legendre_f32<1, uint64_t>, (const void*)k_legendre_f32<2, uint64_t>,
                     (const void*)k_legendre_f32<3, uint64_t>, (const void*)k_legendre_f32<4, uint64_t>,
                     (const void*)k_legendre_f32_tab<1>, (const void*)k_legendre_f32_tab<2>,
                     (const void*)k_legendre_f32_tab<3>, (const void*)k_legendre_f32_tab<4>};
  for (const void* k : f) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

size_t legendre_mfma_tab_bytes(const modal_ctx* c) {
  return sizeof(float) * TREC * chunks_before(c->lmax, c->lmax + 1) * ((c->nrp + 15) / 16);
}

// scratch: device memory that the call may overwrite (the maps that are formed next).  Lambda
// comes from a table there when at least three column blocks share it (below that, building it
// costs what running the recurrence in each block does: 72 us against 24 us a block at l_max
// 500, 768 rings) and it fits, 16-byte aligned, beside a_lm that may lie in the same memory (a
// caller's maps may replace the a_lm they are formed from).  Skies too large for 32-bit offsets (32 of them in
// a block from l_max 5884 on) take the recurrence with 64-bit ones.
hipError_t launch_legendre_mfma(const modal_ctx* c, const void* alm, int S, void* F, void* scratch,
                                size_t scratch_bytes, hipStream_t st) {
  if (c->prec != MODAL_F32) return hipErrorInvalidValue;
  const int ncols = 2 * S * c->P;
  const int blocks = (c->nrp + NWAVE * RW - 1) / (NWAVE * RW);          // workgroups of at most 256 rings
  const int nrt = (c->nrp + blocks * NWAVE * 16 - 1) / (blocks * NWAVE * 16);   // 16-ring tiles per wave, <= 4
  const dim3 grid((ncols + NCOL - 1) / NCOL, blocks, c->lmax + 1);
  const bool fit = offsets_fit(c->lmax, c->P, S);
  const uintptr_t t0 = reinterpret_cast<uintptr_t>(scratch), a0 = reinterpret_cast<uintptr_t>(alm);
  const size_t tab = legendre_mfma_tab_bytes(c), na = (size_t)S * c->nalm * sizeof(float2);
  const bool apart = a0 + na <= t0 || t0 + tab <= a0;
  const bool table = fit && apart && grid.x >= 3 && scratch && scratch_bytes >= tab && t0 % 16 == 0;
  if (table) {
    hipLaunchKernelGGL(k_lambda_records, dim3((c->nrp + 63) / 64, c->lmax + 1), dim3(64), 0, st, c->lmax, c->nrp, c->t.x,
                       c->t.rec, c->t.seed, c->t.lstart, (float*)scratch);
    const int units = blocks * (c->lmax + 1);
    const size_t lds = sizeof(float) * std::max<size_t>(2 * COEF_F, NWAVE * RW * SS);
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(8 * ((units + 7) / 8) * grid.x), dim3(256), lds, st, c->lmax, c->ntheta, c->nrp,
                         c->P, ncols, c->nalm, blocks, (int)grid.x, c->t.lstart,
                         c->t.qw32, (const float*)alm, (const float*)scratch, (float2*)F);
    };
    if (nrt == 1) launch(k_legendre_f32_tab<1>);
    else if (nrt == 2) launch(k_legendre_f32_tab<2>);
    else if (nrt == 3) launch(k_legendre_f32_tab<3>);
    else launch(k_legendre_f32_tab<4>);
    return hipGetLastError();
  }
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), kLds, st, c->lmax, c->ntheta, c->nrp, c->P, ncols, c->nalm, c->t.x,
                       c->t.rec, c->t.seed, c->t.lstart, c->t.qw32, (const float*)alm, (float2*)F);
  };
  auto tiles = [&](auto o) {
    using Off = decltype(o);
    if (nrt == 1) launch(k_legendre_f32<1, Off>);
    else if (nrt == 2) launch(k_legendre_f32<2, Off>);
    else if (nrt == 3) launch(k_legendre_f32<3, Off>);
    else launch(k_legendre_f32<4, Off>);
  };
  if (fit) tiles(uint32_t{});
  else tiles(uint64_t{});
  return hipGetLastError();
}

}  // namespace modal
