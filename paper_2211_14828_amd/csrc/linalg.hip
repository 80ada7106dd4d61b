// Float64 dense linear algebra on small matrices (the Krylov basis, the
// projected matrix Z and its eigenvectors).  Every routine here works on
// matrices of at most a few thousand rows/columns and runs entirely on the
// device.
#include <hip/hip_cooperative_groups.h>
#include <cstdlib>

#include "rbki_kernels.h"

namespace cg = cooperative_groups;

namespace rbki {

namespace {

// ------------------------------------------------------------------ DGEMM
// Small float64 products on the float64 matrix cores (16x16x4), several
// independent ones (the modes of a decomposition) in one launch.  They are
// bound by latency, not by arithmetic: a product of the Krylov chain has a few
// dozen output tiles and an inner dimension of a few hundred, and the chain
// runs them one after the other.  So a workgroup owns one tile of 16 columns by
// 16 or 64 rows, its eight waves take the stages of the inner dimension in
// turn, with operands straight from memory (they stay in the caches from one
// product to the next), and the eight partial tiles are added through LDS in a
// fixed order: no second launch, and a wave has one or two stages to wait for.
// Inner dimensions of 1024 and more (TR-SVD, modes of thousands of rows) are
// also split over workgroups, their partials summed in order by a second kernel.
// Tiles of 64 rows are taken from 1024 tiles of 16 x 16 on, where the bytes
// read matter: the columns' operand is then read once per 64 rows.
//
// 400^3, S = 30, q = 3, bf16 form, three modes together: 41 launches of the
// chain against 78 products, 57 reductions and 45 others for the modes one by
// one on the vector units; the decomposition went from 2.98 to 1.75 ms.
constexpr int GW = 8;                        // waves of a workgroup
typedef double f64x2u_t __attribute__((ext_vector_type(2), aligned(8)));

// KS consecutive values p[t * stride] (p at index k0), t < KS, zero from K on.
template <int KS>
__device__ inline void gemm_run(const double* p, int64_t stride, int k0, int K, double (&out)[KS]) {
  if (stride == 1 && k0 + KS <= K) {
#pragma unroll
    for (int t = 0; t < KS; t += 2) {
      const f64x2u_t v = *(const f64x2u_t*)(p + t);
      out[t] = v.x;
      out[t + 1] = v.y;
    }
  } else {
#pragma unroll
    for (int t = 0; t < KS; ++t) out[t] = k0 + t < K ? p[t * stride] : 0.0;
  }
}

// One tile of 16 RB rows by 16 columns over the inner range [kb, ke).  Lane
// l holds values k0 + KS (l / 16) + t of row (column) l % 16 of a stage of
// 4 KS values; rows and columns past the end repeat the last one.
template <int RB, int KS>
__device__ inline void gemm_tile(const GemmJob& g, int r0, int c0, int kb, int ke, double* sums, double* part) {
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int ST = 4 * KS;
  const double* pa[RB];
#pragma unroll
  for (int u = 0; u < RB; ++u) {
    const int i = r0 + 16 * u + li;
    pa[u] = g.A + (int64_t)(i < g.m ? i : g.m - 1) * g.sai;
  }
  const int j = c0 + li;
  const double* pb = g.B + (int64_t)(j < g.n ? j : g.n - 1) * g.sbj;
  f64x4_t acc[RB];
#pragma unroll
  for (int u = 0; u < RB; ++u) acc[u] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  double a0[RB][KS], b0[KS], a1[RB][KS], b1[KS];
  auto load = [&](double (&a)[RB][KS], double (&b)[KS], int k) {
    k += KS * lg;
#pragma unroll
    for (int u = 0; u < RB; ++u) gemm_run<KS>(pa[u] + (int64_t)k * g.sak, g.sak, k, ke, a[u]);
    gemm_run<KS>(pb + (int64_t)k * g.sbk, g.sbk, k, ke, b);
  };
  auto mul = [&](const double (&a)[RB][KS], const double (&b)[KS]) {
#pragma unroll
    for (int t = 0; t < KS; ++t)
#pragma unroll
      for (int u = 0; u < RB; ++u) acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][t], b[t], acc[u], 0, 0, 0);
  };
  int k = kb + wave * ST;
  if (k < ke) load(a0, b0, k);
  while (k < ke) {
    const int k1 = k + GW * ST, k2 = k1 + GW * ST;
    if (k1 < ke) load(a1, b1, k1);
    mul(a0, b0);
    if (k2 < ke) load(a0, b0, k2);
    if (k1 < ke) mul(a1, b1);
    k = k2;
  }
#pragma unroll
  for (int u = 0; u < RB; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) sums[wave * (RB * 256) + (16 * u + 4 * v + lg) * 16 + li] = acc[u][v];
  __syncthreads();
  for (int e = threadIdx.x; e < RB * 256; e += 64 * GW) {
    double v = sums[e];
#pragma unroll
    for (int w = 1; w < GW; ++w) v += sums[w * (RB * 256) + e];
    const int64_t r = r0 + e / 16, c = c0 + e % 16;
    if (r >= g.m || c >= g.n) continue;
    if (part) {
      part[r * g.n + c] = v;
    } else {
      double* p = g.C + r * g.ldc + c;
      v = g.beta == 0.0 ? g.alpha * v : g.alpha * v + g.beta * *p;
      *p = v;
      if (g.C2) g.C2[r * g.ldc2 + c] = v;
    }
  }
}

__global__ void __launch_bounds__(64 * GW) gemm_kernel(GemmArgs a) {
  extern __shared__ double gemm_lds[];
  const GemmJob& g = a.job[blockIdx.y];
  const int tiles = g.trows * g.tcols;
  const int id = blockIdx.x;
  if (id >= tiles * g.splits) {
    // the squared norms of A's rows, one wave a row
    const int row = (id - tiles * g.splits) * GW + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (!g.norms || row >= g.m) return;
    double s = 0.0;
    for (int c = lane; c < g.k; c += 64) {
      const double v = g.A[(int64_t)row * g.sai + (int64_t)c * g.sak];
      s = fma(v, v, s);
    }
    s = warp_sum(s);
    if (lane == 0) g.norms[row] = s;
    return;
  }
  const int split = id / tiles, t = id % tiles;
  const int kb = split * g.kchunk, ke = kb + g.kchunk < g.k ? kb + g.kchunk : g.k;
  double* part = g.splits > 1 ? g.part + (int64_t)split * g.m * g.n : nullptr;
  if (g.rows == 64) gemm_tile<4, 4>(g, (t / g.tcols) * 64, (t % g.tcols) * 16, kb, ke, gemm_lds, part);
  else gemm_tile<1, 8>(g, (t / g.tcols) * 16, (t % g.tcols) * 16, kb, ke, gemm_lds, part);
}

// C = alpha * sum of the partials + beta * C, summed in a fixed order.
__global__ void gemm_reduce_kernel(GemmArgs a) {
  const GemmJob& g = a.job[blockIdx.y];
  if (g.splits <= 1) return;
  const int64_t mn = (int64_t)g.m * g.n;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < mn; e += (int64_t)gridDim.x * blockDim.x) {
    double v = 0.0;
#pragma unroll 4
    for (int z = 0; z < g.splits; ++z) v += g.part[z * mn + e];
    const int64_t r = e / g.n, c = e - r * g.n;
    double* p = g.C + r * g.ldc + c;
    v = g.beta == 0.0 ? g.alpha * v : g.alpha * v + g.beta * *p;
    *p = v;
    if (g.C2) g.C2[r * g.ldc2 + c] = v;
  }
}

// ------------------------------------------------------------ Cholesky QR
// CholeskyQR step for s <= 96 in one launch: Yout = L^{-1} Y where G = L L^T, with
// column dropping.  A pivot d_k (the Schur-complement diagonal) is dropped, with its
// column of the factor set to zero and a zero row of Yout, when
// d_k <= tau_rel * G_kk (the vector lies within the span of the earlier kept ones to
// working accuracy), when d_k <= tau_abs^2 * max_k ref2[k] (it is at round-off level
// relative to the block before projection; without ref2, to vectors of length 1) or when the direction budget is spent.
// flags[k] = 1 for kept vectors.
//
// A workgroup of four waves takes 64 columns of Y and factors G itself, so no
// workgroup waits for another.  G is zero-padded to 16 NB in LDS (a padded pivot is
// dropped and changes nothing) and factored in panels of 16 columns by wave 0: a
// lane holds a row of the panel in registers, and column k is read from the lanes
// that hold it (v_readlane).  Sixteen more lanes start as the identity's rows: the
// column operations that turn the diagonal block into D turn those into D^{-T}, at
// no cost.  The waves then apply the panel to the trailing blocks and, once all are
// factored, solve L y = Y by blocks, y_b = D_b^{-1} (Y_b - sum_a L_ba y_a), sixteen
// columns a wave, on the float64 matrix cores: an item of a product is the next
// product's operand as it stands.  The pivot is d * rsqrt(d) and its reciprocal the
// Newton-refined rsqrt itself.
//
// The time is latency: launch, the read of G and Y, and 16 NB dependent columns of
// about 0.2 us.  Against one wave that substituted in every column from LDS
// broadcasts: s = 15 6.1 us (7.6), s = 30 9.9 (17.1), s = 60 25 (42); and for s = 90
// against the unblocked factor and inverse of one workgroup and a product, 45 us (200
// and 12), with other modes beside them.
constexpr int CHOL_MAX = 96;

__device__ inline double lane_f64(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// G = Y Y^T formed by the workgroup itself, the lower blocks into Ls: for few columns
// (chol_forms_g) the product is less than the launch of one.  Wave w takes the column
// blocks of 16 congruent to w modulo 4; lane group g of a block columns 4 g + u (the
// same for both operands), so a lane reads 32 consecutive bytes.  The waves' sums are
// added in order.  Measured, a step's two launches / the one: s = 15, n = 64 to 200 9.6 /
// 8.3 us; s = 30, n = 190 to 300 14.2 / 15.0, level with the gap between launches, and n
// = 400 15.8 / 18.2.  So up to 768 columns times blocks; it also takes 6 of the 58
// launches of a served request (3910 -> 4150 solves/s with 16 slots, host-bound).
typedef double d2u_t __attribute__((ext_vector_type(2), aligned(8)));
constexpr int CHOL_FORM_NB = 4;
inline bool chol_forms_g(int64_t s, int64_t n) {
  const int64_t nb = ceil_div(s, 16);
  return nb <= CHOL_FORM_NB && n <= 512 && nb * (nb + 1) / 2 * n <= 768;
}

template <int NB, int LD>
__device__ inline void form_gram(double (*Ls)[LD], const double* Y, int s, int64_t n, int wave, int lane) {
  constexpr int AHEAD = NB <= 2 ? 4 : 2;
  const int li = lane & 15, lg = lane >> 4;
  f64x4_t acc[NB * (NB + 1) / 2];
#pragma unroll
  for (int t = 0; t < NB * (NB + 1) / 2; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[t][v] = 0.0;
  for (int64_t k0 = 16 * wave; k0 < n; k0 += 64 * AHEAD) {
    double f[AHEAD][NB][4];
#pragma unroll
    for (int h = 0; h < AHEAD; ++h)
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        // (the last columns from where they end, those before moved out)
        const int row = 16 * t + li;
        const int64_t k = k0 + 64 * h + 4 * lg, from = k + 4 <= n ? k : n >= 4 ? n - 4 : 0;
        const double* p = Y + (int64_t)(row < s ? row : s - 1) * n + from;
        double v[4];
        if (n >= 4) {
          const d2u_t v0 = *(const d2u_t*)p, v1 = *(const d2u_t*)(p + 2);
          v[0] = v0.x; v[1] = v0.y; v[2] = v1.x; v[3] = v1.y;
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) v[u] = p[u < n ? u : n - 1];
        }
        const int skip = (int)(k - from < 4 ? k - from : 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) f[h][t][u] = row < s && u >= skip && from + u < n ? v[u] : 0.0;
      }
#pragma unroll
    for (int h = 0; h < AHEAD; ++h)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int ti = 0; ti < NB; ++ti)
#pragma unroll
          for (int tj = 0; tj <= ti; ++tj)
            acc[ti * (ti + 1) / 2 + tj] =
                __builtin_amdgcn_mfma_f64_16x16x4f64(f[h][ti][u], f[h][tj][u], acc[ti * (ti + 1) / 2 + tj], 0, 0, 0);
  }
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int ti = 0; ti < NB; ++ti)
#pragma unroll
        for (int tj = 0; tj <= ti; ++tj)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            double& d = Ls[16 * ti + 4 * v + lg][16 * tj + li];
            const double x = acc[ti * (ti + 1) / 2 + tj][v];
            d = w == 0 ? x : d + x;
          }
    }
    __syncthreads();
  }
}

template <int NB>
__global__ void __launch_bounds__(256) chol_solve_kernel(CholArgs a) {
  constexpr int SM = 16 * NB, LD = SM + 4;       // rows 4 banks (of 8 bytes) apart: no conflicts in a fragment
  constexpr bool TWO = SM > 48;                  // rows of a panel beyond the first 48
  const CholJob& job = a.job[blockIdx.y];
  const int s = (int)job.s;
  const int64_t n = job.n;
  if ((int64_t)blockIdx.x * 64 >= n) return;
  __shared__ double Ls[SM][LD];
  __shared__ double Di[NB][16][20];              // inverses of the diagonal blocks
  __shared__ double diag[SM];
  __shared__ int keep[SM];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  // this wave's columns of Y: item v of lane (li, lg) of block b is row 16 b + 4 v + lg
  const int64_t c = (int64_t)blockIdx.x * 64 + wave * 16 + li;
  const int64_t cc = c < n ? c : n - 1;
  f64x4_t y[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int k = 16 * b + 4 * v + lg;
      y[b][v] = job.Y[(int64_t)(k < s ? k : s - 1) * n + cc];
    }
  bool formed = false;
  if constexpr (NB <= CHOL_FORM_NB) {
    if (job.form_g) {
      form_gram<NB, LD>(Ls, job.Y, s, n, wave, lane);
      formed = true;
    }
  }
  if (!formed) {
    const double* G = job.G;
    double gv[NB * NB];
#pragma unroll
    for (int q = 0; q < NB * NB; ++q) {
      const int e = tid + 256 * q, i = e / SM, j = e - i * SM;
      gv[q] = G[(i < s ? i : s - 1) * s + (j < s ? j : s - 1)];
    }
#pragma unroll
    for (int q = 0; q < NB * NB; ++q) {
      const int e = tid + 256 * q, i = e / SM, j = e - i * SM;
      Ls[i][j] = (i < s && j < s) ? gv[q] : 0.0;
    }
  }
  __syncthreads();
  for (int k = tid; k < SM; k += 256) diag[k] = Ls[k][k];
  double mx = job.ref2 ? 0.0 : 1.0;
  if (job.ref2)
    for (int k = lane; k < s; k += 64) mx = fmax(mx, formed ? (job.norms ? Ls[k][k] : job.ref2[k]) : job.ref2[k]);
  const double abs_floor = job.tau_abs * job.tau_abs * warp_max(mx);
  const double tau_rel = a.tau_rel;
  const DimBudget bud = job.bud;
  const int64_t allowed = bud.allowed();
  int64_t nkept = 0;
  __syncthreads();
#pragma unroll 1
  for (int b = 0; b < NB; ++b) {
    const int c0 = 16 * b;
    if (wave == 0) {
      // lanes 0..47: rows c0 + lane; 48..63: the identity's; then rows c0 + 48 + lane
      const int row0 = c0 + lane, row1 = c0 + 48 + lane;
      const bool in0 = lane < 48 && row0 < SM, in1 = TWO && row1 < SM;
      double r0[16], r1[TWO ? 16 : 1];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        r0[j] = in0 ? Ls[row0][c0 + j] : (lane == 48 + j ? 1.0 : 0.0);
        if constexpr (TWO) r1[j] = in1 ? Ls[row1][c0 + j] : 0.0;
      }
      // the least pivot that is kept (none: infinity)
      const double d0 = lane < 16 ? diag[c0 + lane] : 0.0;
      const double least = d0 > 0.0 && abs_floor == abs_floor ? fmax(tau_rel * d0, abs_floor) : __builtin_inf();
      unsigned kept = 0;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const double v = r0[k];                   // G(i, k) minus the earlier columns' terms
        const double d = lane_f64(v, k);
        const bool kp = d > lane_f64(least, k) && nkept < allowed;
        nkept += kp;
        kept |= (unsigned)kp << k;
        const double rs = rsq_nr(d);
        const double inv = kp ? rs : 0.0;
        const double l0 = v * inv;                // (above the diagonal: not used)
        r0[k] = l0;
        if constexpr (TWO) r1[k] *= inv;
#pragma unroll
        for (int j = k + 1; j < 16; ++j) {
          const double lj = lane_f64(l0, j);
          r0[j] -= l0 * lj;
          if constexpr (TWO) r1[j] -= r1[k] * lj;
        }
      }
      if (lane < 16) keep[c0 + lane] = (kept >> lane) & 1;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        if (in0) Ls[row0][c0 + j] = r0[j];
        if (TWO && in1) Ls[row1][c0 + j] = r1[j];
        if (lane >= 48) Di[b][j][lane - 48] = r0[j];
      }
    }
    __syncthreads();
    // trailing blocks (ti, tj <= ti): A -= L_ti L_tj^T
    const int m = NB - 1 - b;
    for (int t = wave; t < m * (m + 1) / 2; t += 4) {
      int ti = 0, tj = t;
      while (tj > ti) tj -= ++ti;
      const int i0 = c0 + 16 + 16 * ti, j0 = c0 + 16 + 16 * tj;
      f64x4_t acc;
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[v] = Ls[i0 + 4 * v + lg][j0 + li];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-Ls[i0 + li][c0 + 4 * k + lg], Ls[j0 + li][c0 + 4 * k + lg], acc, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) Ls[i0 + 4 * v + lg][j0 + li] = acc[v];
    }
    __syncthreads();
  }
  if (blockIdx.x == 0) {
    for (int k = tid; k < s; k += 256) job.flags[k] = keep[k];
    // every workgroup reads the count of earlier blocks; one writes the total
    if (tid == 0) bud.record(nkept);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    f64x4_t t = y[b];
#pragma unroll
    for (int p = 0; p < b; ++p)
#pragma unroll
      for (int k = 0; k < 4; ++k)
        t = __builtin_amdgcn_mfma_f64_16x16x4f64(-Ls[16 * b + li][16 * p + 4 * k + lg], y[p][k], t, 0, 0, 0);
    f64x4_t z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 4; ++k) z = __builtin_amdgcn_mfma_f64_16x16x4f64(Di[b][li][4 * k + lg], t[k], z, 0, 0, 0);
    y[b] = z;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int k = 16 * b + 4 * v + lg;
      if (k < s && c < n) job.Yout[(int64_t)k * n + c] = z[v];
    }
  }
}

// Left-looking Cholesky of the s x s Gram matrix G with column dropping, one
// workgroup, for s beyond the LDS variant (same drop rule).
__global__ void __launch_bounds__(1024) chol_drop_kernel(const double* G, int64_t s, double* L, int* flags,
                                                         const double* ref2, double tau_rel, double tau_abs,
                                                         DimBudget bud) {
  __shared__ double red[16];
  __shared__ double sh_ref;
  __shared__ int sh_keep;
  __shared__ double sh_piv;
  const int tid = threadIdx.x;
  double mx = ref2 ? 0.0 : 1.0;
  if (ref2)
    for (int64_t i = tid; i < s; i += blockDim.x) mx = fmax(mx, ref2[i]);
  mx = warp_max(mx);
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  if (tid == 0) {
    double v = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) v = fmax(v, red[w]);
    sh_ref = v;
  }
  for (int64_t i = tid; i < s * s; i += blockDim.x) L[i] = 0.0;
  __syncthreads();
  const double abs_floor = tau_abs * tau_abs * sh_ref;
  const int64_t allowed = bud.allowed();
  int64_t nkept = 0;                               // meaningful in thread 0
  for (int64_t kc = 0; kc < s; ++kc) {
    if (tid == 0) {
      double d = G[kc * s + kc];
      for (int64_t j = 0; j < kc; ++j) d -= L[kc * s + j] * L[kc * s + j];
      const double gkk = G[kc * s + kc];
      const int keep = (gkk > 0.0) && (d > tau_rel * gkk) && (d > abs_floor) && nkept < allowed;
      nkept += keep;
      sh_keep = keep;
      sh_piv = keep ? sqrt(d) : 0.0;
      flags[kc] = keep;
      if (keep) L[kc * s + kc] = sh_piv;
    }
    __syncthreads();
    if (sh_keep) {
      const double piv = sh_piv;
      for (int64_t i = kc + 1 + tid; i < s; i += blockDim.x) {
        double v = G[i * s + kc];
        for (int64_t j = 0; j < kc; ++j) v -= L[i * s + j] * L[kc * s + j];
        L[i * s + kc] = v / piv;
      }
    }
    __syncthreads();
  }
  if (tid == 0) bud.record(nkept);
}

// Y (s x n rows) <- L^{-1} Y row-wise (forward substitution along the s
// vectors), one thread per column; dropped vectors become zero.
__global__ void trsm_rows_kernel(double* Y, int64_t s, int64_t n, const double* L, const int* flags) {
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n; c += (int64_t)gridDim.x * blockDim.x) {
    for (int64_t kc = 0; kc < s; ++kc) {
      if (!flags[kc]) {
        Y[kc * n + c] = 0.0;
        continue;
      }
      double v = Y[kc * n + c];
      for (int64_t j = 0; j < kc; ++j)
        if (flags[j]) v -= L[kc * s + j] * Y[j * n + c];
      Y[kc * n + c] = v / L[kc * s + kc];
    }
  }
}

__global__ void row_norms2_kernel(const double* Y, int64_t s, int64_t n, double* out) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (row >= s) return;
  double acc = 0.0;
  for (int64_t c = lane; c < n; c += 64) {
    const double v = Y[row * n + c];
    acc = fma(v, v, acc);
  }
  acc = warp_sum(acc);
  if (lane == 0) out[row] = acc;
}

// ------------------------------------------------------------ Jacobi
// Block one-sided (Hestenes) Jacobi on the columns of symmetric PSD matrices,
// several matrices per launch.  The columns of each matrix are split into
// nblk blocks of nb columns (zero-padded).  Rounds follow the circle method
// over blocks: in each round a workgroup takes one pair of blocks and stages
// their 2 nb columns P in LDS.  It forms the small Gram matrix G = P^T P once,
// diagonalises it by cyclic two-sided Jacobi sweeps on G itself while
// accumulating the rotation V (the rotation angles come from three entries of
// G instead of three length-n dot products), and applies P <- P V once.  The
// nblk - 1 rounds of a sweep are separated by grid barriers.  A matrix is done
// when a whole sweep met no pair of its columns with |cos| above tol.  At
// convergence A = Z V has orthogonal columns a_j = lambda_j v_j: eigenvalues
// are the column norms and eigenvectors the normalised columns.
constexpr int JAC_MAXB = 8;    // matrices per launch
constexpr int JAC_APPLY_MAX = 5;   // 16 x 16 output blocks per wave in the apply phase

struct JacobiArgs {
  double* A[JAC_MAXB];         // npad x n column-major working copies
  int64_t n[JAC_MAXB];
  int nblk[JAC_MAXB];
  int* info[JAC_MAXB];         // info[0]: 0 or sweeps at the limit, info[1]: sweeps used
  int nmat, nb, npos, max_nblk;
  int64_t ld;
  int max_sweeps, inner_sweeps;
  double tol;
  unsigned long long* offmax;  // [3][JAC_MAXB] per-sweep max |cos| bit patterns
  unsigned long long* prof;    // nullable: phase clocks of workgroup 0 (diagnostics)
};

// Circle ordering: position pos (0 <= pos < nblk) holds this element in round
// `round` (0 <= round < nblk - 1); position 0 is fixed, the others rotate.
__device__ inline int circle_block(int pos, int round, int nblk) {
  if (pos == 0) return 0;
  int v = pos - 1 + round;              // < 2 (nblk - 1)
  if (v >= nblk - 1) v -= nblk - 1;
  return 1 + v;
}


// Rotation (c, s) zeroing the (p, q) entry of a 2x2 Gram block
// [al ga; ga be]: new_p = c p - s q, new_q = s p + c q.  Returns false when
// |ga| <= tol sqrt(al be) (the pair is already orthogonal to tolerance).
// The rotation is the standard one: zeta = (be - al) / (2 ga),
// t = sign(zeta) / (|zeta| + sqrt(1 + zeta^2)), c = 1 / sqrt(1 + t^2), s = c t.
__device__ inline bool jacobi_rotation(double al, double be, double ga, double tol, double& c, double& s,
                                       double& cosang) {
  c = 1.0;
  s = 0.0;
  al = fmax(al, 0.0);
  be = fmax(be, 0.0);
  if (!(al > 1e-300 && be > 1e-300)) { cosang = 0.0; return false; }
  cosang = fabs(ga) * rsq_nr(al) * rsq_nr(be);
  if (cosang <= tol) return false;
  const double zeta = (be - al) * rcp_nr(2.0 * ga);
  const double z2 = fma(zeta, zeta, 1.0);
  const double root = z2 < 1e300 ? z2 * rsq_nr(z2) : fabs(zeta);   // sqrt(1 + zeta^2)
  const double tm = rcp_nr(fabs(zeta) + root);
  const double t = zeta >= 0.0 ? tm : -tm;
  c = rsq_nr(fma(t, t, 1.0));
  s = c * t;
  return true;
}

// COOP: one workgroup per (matrix, pair position), rounds separated by grid
// barriers (cooperative launch).  !COOP: one workgroup per matrix walks every
// position of a round itself; an ordinary launch, so that solves on other
// streams can run beside it.  The pairs of a round touch disjoint columns and
// every pair does the same arithmetic in either form, so the two give
// bit-identical results.
template <bool COOP>
__global__ void __launch_bounds__(1024) jacobi_kernel(JacobiArgs J) {
  extern __shared__ double sm[];
  __shared__ double sh_off[16];
  __shared__ int sh_done[JAC_MAXB];
  __shared__ double rot_c[16], rot_s[16];
  __shared__ int rot_p[16], rot_q[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m = COOP ? blockIdx.x / J.npos : blockIdx.x;
  const int pos0 = COOP ? blockIdx.x % J.npos : 0;
  const int nb = J.nb, two = 2 * nb;
  const int nbk = (two + 15) / 16;                 // 16-wide MFMA blocks across the pair
  const int64_t n = J.n[m];
  const int64_t ld = J.ld;                         // odd stride >= n: conflict-free column reads
  double* P = sm;                                  // columns-major [two][ld]
  double* G = P + (int64_t)two * ld;               // [two][two + 1]
  double* V = G + two * (two + 1);
  double* S = V + two * (two + 1);                 // Gram partials [16][256]
  const int gs = two + 1;
  if (tid < JAC_MAXB) sh_done[tid] = 0;
  __syncthreads();
  int sweep;
  for (sweep = 0; sweep < J.max_sweeps; ++sweep) {
    if (COOP && blockIdx.x == 0 && tid < J.nmat) J.offmax[((sweep + 1) % 3) * JAC_MAXB + tid] = 0ull;
    double local_off = 0.0;
    const int npos_m = J.nblk[m] / 2;
    const bool mine = !sh_done[m] && pos0 < npos_m;
    const int pos_end = COOP ? pos0 + 1 : npos_m;
    for (int round = 0; round < (COOP ? J.max_nblk : J.nblk[m]) - 1; ++round) {
      for (int pos = pos0; pos < pos_end; ++pos) {
      unsigned long long t0 = wall_clock64();
      if (mine && round < J.nblk[m] - 1) {
        const int bp = circle_block(pos, round, J.nblk[m]);
        const int bq = circle_block(J.nblk[m] - 1 - pos, round, J.nblk[m]);
        double* A = J.A[m];
        for (int c = wave; c < two; c += 16) {
          const int gc = c < nb ? bp * nb + c : bq * nb + (c - nb);
          const double* src = A + (int64_t)gc * n;
          for (int64_t r = lane; r < n; r += 64) P[c * ld + r] = src[r];
        }
        __syncthreads();
        unsigned long long t1 = wall_clock64();
        // G = P^T P on fp64 MFMA 16x16x4: wave w takes output block (w % nbk^2)
        // and K slice (w / nbk^2); slices are summed through LDS.
        {
          const int nblk2 = nbk * nbk;
          const int nslice = 16 / nblk2;
          const int blk = wave % nblk2, sl = wave / nblk2;
          const int bi = blk / nbk, bj = blk % nbk;
          const int i = bi * 16 + (lane & 15), j = bj * 16 + (lane & 15);
          const int64_t ksteps = (n + 3) / 4;
          const int64_t k0 = ksteps * sl / nslice, k1 = ksteps * (sl + 1) / nslice;
          f64x4_t d = {0.0, 0.0, 0.0, 0.0};
          for (int64_t kt = k0; kt < k1; ++kt) {
            const int64_t r = kt * 4 + (lane >> 4);
            const double a = (i < two && r < n) ? P[i * ld + r] : 0.0;
            const double b = (j < two && r < n) ? P[j * ld + r] : 0.0;
            d = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d, 0, 0, 0);
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) S[(sl * nblk2 + blk) * 256 + (4 * v + (lane >> 4)) * 16 + (lane & 15)] = d[v];
          __syncthreads();
          for (int e = tid; e < two * two; e += blockDim.x) {
            const int ii = e / two, jj = e % two;
            const int b2 = (ii >> 4) * nbk + (jj >> 4);
            double acc = 0.0;
            for (int q = 0; q < nslice; ++q) acc += S[(q * nblk2 + b2) * 256 + (ii & 15) * 16 + (jj & 15)];
            G[ii * gs + jj] = acc;
            V[ii * gs + jj] = ii == jj ? 1.0 : 0.0;
          }
          __syncthreads();
        }
        unsigned long long t2 = wall_clock64();
        // inner cyclic sweep on G (two-sided), accumulating V.  In each step
        // lanes k < nb of wave 0 form the rotation of pair k once and publish
        // it in LDS; then, in one phase, thread t < nb^2 applies both
        // rotations of its 2 x 2 block of G (rows of pair t / nb, columns of
        // pair t % nb: G' = J^T G J restricted to that block), and the next
        // 2 nb^2 threads apply the column rotations to V.  The pairs partition
        // the indices, so every entry has exactly one writer.
        {
          for (int isw = 0; isw < J.inner_sweeps; ++isw) {
            double inner_off = 0.0;
            for (int ir = 0; ir < two - 1; ++ir) {
              if (tid < nb) {
                const int p = circle_block(tid, ir, two);
                const int q = circle_block(two - 1 - tid, ir, two);
                double c, s, ca;
                jacobi_rotation(G[p * gs + p], G[q * gs + q], G[p * gs + q], J.tol, c, s, ca);
                inner_off = fmax(inner_off, ca);
                rot_c[tid] = c;
                rot_s[tid] = s;
                rot_p[tid] = p;
                rot_q[tid] = q;
              }
              __syncthreads();
              if (tid < nb * nb) {
                const int k1 = tid / nb, k2 = tid - k1 * nb;
                const double c1 = rot_c[k1], s1 = rot_s[k1], c2 = rot_c[k2], s2 = rot_s[k2];
                if (s1 != 0.0 || s2 != 0.0) {
                  const int a0 = rot_p[k1], a1 = rot_q[k1], b0 = rot_p[k2], b1 = rot_q[k2];
                  const double g00 = G[a0 * gs + b0], g01 = G[a0 * gs + b1];
                  const double g10 = G[a1 * gs + b0], g11 = G[a1 * gs + b1];
                  // rows: p' = c1 p - s1 q, q' = s1 p + c1 q
                  const double h00 = c1 * g00 - s1 * g10, h01 = c1 * g01 - s1 * g11;
                  const double h10 = s1 * g00 + c1 * g10, h11 = s1 * g01 + c1 * g11;
                  // columns: p' = c2 p - s2 q, q' = s2 p + c2 q
                  G[a0 * gs + b0] = c2 * h00 - s2 * h01;
                  G[a0 * gs + b1] = s2 * h00 + c2 * h01;
                  G[a1 * gs + b0] = c2 * h10 - s2 * h11;
                  G[a1 * gs + b1] = s2 * h10 + c2 * h11;
                }
              } else if (tid < nb * nb + two * nb) {
                const int e = tid - nb * nb;
                const int i = e / nb, k = e - i * nb;
                const double c = rot_c[k], sn = rot_s[k];
                if (sn != 0.0) {
                  const int p = rot_p[k], q = rot_q[k];
                  const double vp = V[i * gs + p], vq = V[i * gs + q];
                  V[i * gs + p] = c * vp - sn * vq;
                  V[i * gs + q] = sn * vp + c * vq;
                }
              }
              __syncthreads();
            }
            if (wave == 0) {
              const double w = warp_max(inner_off);
              if (lane == 0) sh_off[0] = w;
            }
            __syncthreads();
            const double mx = sh_off[0];
            __syncthreads();
            if (isw == 0) local_off = fmax(local_off, mx);
            if (mx <= J.tol) break;
          }
        }
        unsigned long long t3 = wall_clock64();
        // A(:, pair) <- P V on fp64 MFMA: 16 x 16 output blocks over
        // (row block, column block), K = two.  The blocks are held in
        // registers until every wave has finished reading P, written back
        // into P, and then copied out column by column (coalesced).
        {
          const int64_t rblocks = (n + 15) / 16;
          const int64_t nblocks = rblocks * nbk;   // <= 16 * JAC_APPLY_MAX (host check)
          f64x4_t d[JAC_APPLY_MAX];
#pragma unroll
          for (int it = 0; it < JAC_APPLY_MAX; ++it) {
            d[it] = f64x4_t{0.0, 0.0, 0.0, 0.0};
            const int64_t ob = wave + 16 * it;
            if (ob < nblocks) {
              const int64_t rb = ob / nbk;
              const int cb = (int)(ob % nbk);
              const int64_t r = rb * 16 + (lane & 15);
              const int j = cb * 16 + (lane & 15);
              for (int kt = 0; kt < (two + 3) / 4; ++kt) {
                const int k = kt * 4 + (lane >> 4);
                const double a = (r < n && k < two) ? P[k * ld + r] : 0.0;
                const double b = (j < two && k < two) ? V[k * gs + j] : 0.0;
                d[it] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d[it], 0, 0, 0);
              }
            }
          }
          __syncthreads();
#pragma unroll
          for (int it = 0; it < JAC_APPLY_MAX; ++it) {
            const int64_t ob = wave + 16 * it;
            if (ob < nblocks) {
              const int64_t rb = ob / nbk;
              const int cb = (int)(ob % nbk);
              const int jo = cb * 16 + (lane & 15);
              if (jo < two) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                  const int64_t ro = rb * 16 + 4 * v + (lane >> 4);
                  if (ro < n) P[jo * ld + ro] = d[it][v];
                }
              }
            }
          }
          __syncthreads();
          for (int c = wave; c < two; c += 16) {
            const int gc = c < nb ? bp * nb + c : bq * nb + (c - nb);
            double* dst = A + (int64_t)gc * n;
            for (int64_t r = lane; r < n; r += 64) dst[r] = P[c * ld + r];
          }
        }
        __threadfence();
        if (J.prof && blockIdx.x == 0 && tid == 0) {
          unsigned long long t4 = wall_clock64();
          J.prof[0] += t1 - t0;
          J.prof[1] += t2 - t1;
          J.prof[2] += t3 - t2;
          J.prof[3] += t4 - t3;
          J.prof[5] += 1;
        }
        if (!COOP) __syncthreads();               // P, G and V are reused by the next position
      }
      }
      if constexpr (COOP) {
        unsigned long long tg = wall_clock64();
        cg::this_grid().sync();
        if (J.prof && blockIdx.x == 0 && tid == 0) J.prof[4] += wall_clock64() - tg;
      }
    }
    if constexpr (!COOP) {
      // local_off is uniform across the workgroup: the sweep's largest |cos|
      // over every pair of this matrix
      if (!sh_done[m] && local_off <= J.tol && tid == 0) {
        J.info[m][0] = 0;
        J.info[m][1] = sweep + 1;
      }
      __syncthreads();
      if (local_off <= J.tol) {
        if (tid == 0) sh_done[m] = 1;
        break;
      }
      continue;
    }
    // publish this workgroup's largest |cos| of the sweep (first inner sweep of
    // each round: the state before any rotation of that round)
    if (tid == 0 && mine)
      atomicMax(&J.offmax[(sweep % 3) * JAC_MAXB + m], (unsigned long long)__double_as_longlong(local_off));
    __threadfence();
    cg::this_grid().sync();
    if (tid < J.nmat && !sh_done[tid]) {
      const double v = __longlong_as_double(
          (long long)__atomic_load_n(&J.offmax[(sweep % 3) * JAC_MAXB + tid], __ATOMIC_RELAXED));
      if (v <= J.tol) {
        sh_done[tid] = 1;
        if (blockIdx.x == 0) {
          J.info[tid][0] = 0;
          J.info[tid][1] = sweep + 1;
        }
      }
    }
    __syncthreads();
    bool all = true;
    for (int k = 0; k < J.nmat; ++k) all = all && sh_done[k];
    if (all) break;
  }
  if (COOP && blockIdx.x == 0 && tid < J.nmat && !sh_done[tid]) {
    J.info[tid][0] = sweep;
    J.info[tid][1] = sweep;
  }
  if (!COOP && tid == 0 && !sh_done[m]) {
    J.info[m][0] = sweep;
    J.info[m][1] = sweep;
  }
}

// Column norms of the converged A, then a rank sort (descending, ties by
// index) and normalised columns as rows of Vt.  One workgroup per matrix.
struct FinishArgs {
  const double* A[JAC_MAXB];
  int64_t n[JAC_MAXB];
  double* lam[JAC_MAXB];
  double* Vt[JAC_MAXB];
  double* norms[JAC_MAXB];
};

__global__ void jacobi_finish_kernel(FinishArgs F) {
  const int m = blockIdx.x;
  const double* A = F.A[m];
  const int64_t n = F.n[m];
  double* lam = F.lam[m];
  double* Vt = F.Vt[m];
  double* norms = F.norms[m];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwaves = blockDim.x >> 6;
  for (int64_t j = wave; j < n; j += nwaves) {
    double acc = 0.0;
    for (int64_t r = lane; r < n; r += 64) acc = fma(A[j * n + r], A[j * n + r], acc);
    acc = warp_sum(acc);
    if (lane == 0) norms[j] = sqrt(acc);
  }
  __syncthreads();
  for (int64_t j = tid; j < n; j += blockDim.x) {
    const double v = norms[j];
    int64_t rank = 0;
    for (int64_t i = 0; i < n; ++i) {
      const double w = norms[i];
      rank += (w > v) || (w == v && i < j);
    }
    lam[rank] = v;
    norms[n + j] = (double)rank;
  }
  __syncthreads();
  for (int64_t e = tid; e < n * n; e += blockDim.x) {
    const int64_t j = e / n, r = e - j * n;
    const int64_t dst = (int64_t)norms[n + j];
    const double nv = norms[j];
    Vt[dst * n + r] = nv > 0.0 ? A[j * n + r] / nv : 0.0;
  }
}

__global__ void pad_copy_kernel(const double* Z, int64_t n, int64_t npad, double* A) {
  // A column-major n x npad: column j = row j of Z (Z symmetric), zero beyond n
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < npad * n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = e / n, r = e - j * n;
    A[e] = j < n ? Z[j * n + r] : 0.0;
  }
}

__global__ void copy_rows_kernel(double* dst, int64_t ldd, const double* src, int64_t lds, int64_t rows,
                                 int64_t cols) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < rows * cols;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = e / cols, c = e - r * cols;
    dst[r * ldd + c] = src[r * lds + c];
  }
}

template <class T>
__global__ void store_factor_kernel(const double* Ut, int64_t R, int64_t I, T* out) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < R * I;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e / R, r = e - i * R;
    out[e] = (T)Ut[r * I + i];
  }
}

// Sign rule for singular/eigen vectors: flip each row of V (rows x n) so that
// its largest-magnitude entry (lowest index on ties) is positive.  One wave per row.
__global__ void canonical_sign_rows_kernel(double* V, int64_t rows, int64_t n) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (row >= rows) return;
  double* v = V + row * n;
  double best = -1.0;
  int64_t bi = n;
  for (int64_t c = lane; c < n; c += 64) {
    const double a = fabs(v[c]);
    if (a > best) { best = a; bi = c; }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const double ob = __shfl_xor(best, o, 64);
    const int64_t oi = __shfl_xor(bi, o, 64);
    if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
  }
  if (best <= 0.0 || bi >= n) return;
  const double sgn = v[bi] < 0.0 ? -1.0 : 1.0;
  if (sgn < 0.0)
    for (int64_t c = lane; c < n; c += 64) v[c] = -v[c];
}

template <class T> __device__ inline T factor_value(double v);
template <> __device__ inline float factor_value<float>(double v) { return (float)v; }
template <> __device__ inline bf16_t factor_value<bf16_t>(double v) { return f32_to_bf16((float)v); }

__device__ inline void put_factor(void* p, int elem, int64_t at, double v) {
  if (elem == E_F64) ((double*)p)[at] = v;
  else if (elem == E_F32) ((float*)p)[at] = factor_value<float>(v);
  else ((bf16_t*)p)[at] = factor_value<bf16_t>(v);
}

// The factors of all modes once their rows are formed: the sign rule above, and
// every copy that the calls after it read (the operand of the mode product, its
// transpose for the reconstruction, the caller's factor), in one launch.  Apart
// they were nine to twelve launches of 4 us, a tenth of a small decomposition.
struct FactorArgs {
  FinishJob job[8];
};
__global__ void __launch_bounds__(256) finish_factors_kernel(FactorArgs args) {
  const FinishJob& f = args.job[blockIdx.y];
  const int64_t row = blockIdx.x, n = f.I;
  if (row >= f.R) return;
  const int tid = threadIdx.x;
  double* v = f.Ut + row * n;
  double best = -1.0;
  int64_t bi = n;
  auto take = [&](double ob, int64_t oi) {
    if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
  };
  for (int64_t c = tid; c < n; c += 256) {
    const double a = fabs(v[c]);
    if (a > best) { best = a; bi = c; }
  }
  for (int o = 32; o > 0; o >>= 1) take(__shfl_xor(best, o, 64), __shfl_xor(bi, o, 64));
  __shared__ double sb[4];
  __shared__ int64_t si[4];
  if ((tid & 63) == 0) {
    sb[tid >> 6] = best;
    si[tid >> 6] = bi;
  }
  __syncthreads();
  for (int w = 0; w < 4; ++w) take(sb[w], si[w]);
  const bool flip = best > 0.0 && bi < n && v[bi < n ? bi : 0] < 0.0;
  __syncthreads();                 // every thread has read the entry before one turns it
  for (int64_t c = tid; c < n; c += 256) {
    const double x = flip ? -v[c] : v[c];
    if (flip) v[c] = x;
    if (f.copy) f.copy[row * n + c] = x;
    if (f.rows) put_factor(f.rows, f.rows_elem, row * n + c, x);
    if (f.cols) put_factor(f.cols, f.cols_elem, c * f.R + row, x);
    if (f.out) put_factor(f.out, f.out_elem, c * f.R + row, x);
  }
}

__global__ void fill_zero_kernel(unsigned* p, size_t words) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < words; e += (size_t)gridDim.x * blockDim.x)
    p[e] = 0u;
}

inline unsigned grid_for(int64_t work, int64_t per = 256, int64_t cap = 8192) {
  int64_t g = ceil_div(work, per);
  if (g < 1) g = 1;
  return (unsigned)(g > cap ? cap : g);
}

}  // namespace

// per host thread: the scratch of the call being enqueued by that thread
static thread_local double* g_dgemm_scratch = nullptr;
static thread_local size_t g_dgemm_scratch_bytes = 0;

void dgemm_set_scratch(double* p, size_t bytes) {
  g_dgemm_scratch = p;
  g_dgemm_scratch_bytes = bytes;
}

GemmJob gemm_job(int opA, int opB, int64_t m, int64_t n, int64_t k, double alpha, const double* A, int64_t lda,
                 const double* B, int64_t ldb, double beta, double* C, int64_t ldc) {
  GemmJob g = {};
  g.A = A;
  g.B = B;
  g.C = C;
  g.m = (int)m;
  g.n = (int)n;
  g.k = (int)k;
  g.sai = opA ? 1 : lda;
  g.sak = opA ? lda : 1;
  g.sbk = opB ? 1 : ldb;
  g.sbj = opB ? ldb : 1;
  g.ldc = ldc;
  g.alpha = alpha;
  g.beta = beta;
  return g;
}

// Every choice depends on the job alone, so a product has the same bits in
// any company.  (The scratch is divided by the most jobs of a launch.)
hipError_t dgemm_batched(const GemmJob* jobs, int njobs, hipStream_t s) {
  if (njobs < 1 || njobs > kGemmJobs) return hipErrorInvalidValue;
  GemmArgs a = {};
  unsigned gx = 0;
  int64_t red = 0;
  int rows = 16;
  const size_t share = g_dgemm_scratch ? g_dgemm_scratch_bytes / kGemmJobs / 8 : 0;   // doubles per job
  for (int i = 0; i < njobs; ++i) {
    GemmJob& g = a.job[i];
    g = jobs[i];
    if (g.m <= 0 || g.n <= 0) {
      g.m = g.n = 0;
      continue;
    }
    const int64_t cols = ceil_div(g.n, 16);
    g.rows = g.m > 16 && ceil_div(g.m, 16) * cols >= 1024 ? 64 : 16;
    rows = std::max(rows, g.rows);
    g.trows = (int)ceil_div(g.m, g.rows);
    g.tcols = (int)cols;
    const int64_t tiles = (int64_t)g.trows * g.tcols;
    int64_t splits = std::min<int64_t>(ceil_div(256, tiles), std::max(1, g.k / 512));
    splits = std::min<int64_t>(splits, (int64_t)(share / ((size_t)g.m * g.n)));
    g.kchunk = splits > 1 ? (int)(ceil_div(ceil_div(g.k, splits), 32) * 32) : std::max(g.k, 1);
    g.splits = splits > 1 ? (int)ceil_div(g.k, g.kchunk) : 1;
    if (g.splits > 1) {
      g.part = g_dgemm_scratch + (size_t)i * share;
      red = std::max(red, (int64_t)g.m * g.n);
    }
    const int64_t blocks = tiles * g.splits + (g.norms ? ceil_div(g.m, GW) : 0);
    if (blocks * 64 * GW > 0xffffffff) return hipErrorInvalidValue;   // the threads of a launch
    gx = std::max(gx, (unsigned)blocks);
  }
  if (gx == 0) return hipSuccess;
  hipLaunchKernelGGL(gemm_kernel, dim3(gx, njobs), dim3(64 * GW), (size_t)GW * rows * 16 * 8, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || red == 0) return e;
  hipLaunchKernelGGL(gemm_reduce_kernel, dim3((unsigned)std::min<int64_t>(ceil_div(red, 256), 4096), njobs), dim3(256),
                     0, s, a);
  return hipGetLastError();
}

hipError_t dgemm(int opA, int opB, int64_t m, int64_t n, int64_t k, double alpha, const double* A, int64_t lda,
                 const double* B, int64_t ldb, double beta, double* C, int64_t ldc, hipStream_t s) {
  const GemmJob g = gemm_job(opA, opB, m, n, k, alpha, A, lda, B, ldb, beta, C, ldc);
  return dgemm_batched(&g, 1, s);
}

hipError_t row_norms2(const double* Y, int64_t s, int64_t n, double* out, hipStream_t st) {
  if (s <= 0) return hipSuccess;
  hipLaunchKernelGGL(row_norms2_kernel, dim3((unsigned)ceil_div(s, 4)), dim3(256), 0, st, Y, s, n, out);
  return hipGetLastError();
}

hipError_t chol_orth_batched(const CholJob* jobs, int njobs, double tau_rel, hipStream_t st) {
  if (njobs < 1 || njobs > kGemmJobs) return hipErrorInvalidValue;
  GemmJob gj[kGemmJobs];
  // (sketches of more than 64 columns in a launch of their own)
  CholArgs fit[2] = {};
  int nfit[2] = {}, ng = 0;
  int64_t smax = 0, nmax[2] = {};
  for (int i = 0; i < njobs; ++i) {
    CholJob j = jobs[i];
    j.form_g = chol_forms_g(j.s, j.n);
    if (!j.form_g) {
      gj[ng] = gemm_job(0, 1, j.s, j.s, j.n, 1.0, j.Y, j.n, j.Y, j.n, 0.0, j.G, j.s);
      gj[ng++].norms = j.norms;
    }
    if (j.s <= CHOL_MAX) {
      const int w = j.s > 64;
      fit[w].tau_rel = tau_rel;
      fit[w].job[nfit[w]++] = j;
      if (!w) smax = std::max(smax, j.s);
      nmax[w] = std::max(nmax[w], j.n);
    }
  }
  hipError_t e = hipSuccess;
  if (ng && (e = dgemm_batched(gj, ng, st)) != hipSuccess) return e;
  if (nfit[0]) {
    const dim3 grid((unsigned)ceil_div(nmax[0], 64), nfit[0]), block(256);
    if (smax <= 16) hipLaunchKernelGGL(chol_solve_kernel<1>, grid, block, 0, st, fit[0]);
    else if (smax <= 32) hipLaunchKernelGGL(chol_solve_kernel<2>, grid, block, 0, st, fit[0]);
    else if (smax <= 48) hipLaunchKernelGGL(chol_solve_kernel<3>, grid, block, 0, st, fit[0]);
    else hipLaunchKernelGGL(chol_solve_kernel<4>, grid, block, 0, st, fit[0]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (nfit[1]) {
    hipLaunchKernelGGL(chol_solve_kernel<6>, dim3((unsigned)ceil_div(nmax[1], 64), nfit[1]), dim3(256), 0, st, fit[1]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  for (int i = 0; i < njobs; ++i) {
    const CholJob& j = jobs[i];
    if (j.s <= CHOL_MAX) continue;
    hipLaunchKernelGGL(chol_drop_kernel, dim3(1), dim3(1024), 0, st, j.G, j.s, j.Lm, j.flags, j.ref2, tau_rel,
                       j.tau_abs, j.bud);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(trsm_rows_kernel, dim3(grid_for(j.n)), dim3(256), 0, st, j.Y, j.s, j.n, j.Lm, j.flags);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = copy_rows_f64(j.Yout, j.n, j.Y, j.n, j.s, j.n, st)) != hipSuccess) return e;
  }
  return hipSuccess;
}

// Block width: the staged pair (2 nb columns of length n), G, V and the
// Gram partials (16 x 256 doubles) must fit in 160 KB of LDS.
static size_t jacobi_lds_bytes(int64_t n, int nb) {
  const int two = 2 * nb;
  const int64_t ld = (n & 1) ? n : n + 1;
  return (size_t)(two * ld + 2 * two * (two + 1) + 16 * 256) * 8;
}

static void jacobi_geometry(int64_t n, int& nb, int& nblk) {
  nb = 16;
  while (nb > 2 && jacobi_lds_bytes(n, nb) > 160 * 1024 - 1024) nb /= 2;
  if (n <= 2 * nb) nb = (int)std::max<int64_t>(1, (n + 1) / 2);
  nblk = (int)ceil_div(n, nb);
  if (nblk < 2) nblk = 2;
  if (nblk & 1) ++nblk;
}

size_t jacobi_work_bytes(int64_t n) {
  // npad <= n + 2 * nb <= n + 32, so this bound grows with n and covers every
  // smaller matrix that reuses the same scratch
  return (size_t)((n + 32) * n * 8 + 2 * n * 8 + 256);  // A, norms/ranks, offmax
}

hipError_t jacobi_eig_batched(int nmat, const double* const* Z, const int64_t* ns, double* const* lam,
                              double* const* Vt, void* const* work, int* const* info, int max_sweeps, hipStream_t st,
                              bool per_matrix) {
  if (nmat <= 0) return hipSuccess;
  if (nmat > JAC_MAXB) return hipErrorInvalidValue;
  int64_t nmax = 0;
  for (int k = 0; k < nmat; ++k) nmax = std::max(nmax, ns[k]);
  int nb, nblk_dummy;
  jacobi_geometry(nmax, nb, nblk_dummy);
  if (ceil_div(nmax, 16) * ceil_div(2 * nb, 16) > 16 * JAC_APPLY_MAX) return hipErrorInvalidValue;
  JacobiArgs ja = {};
  FinishArgs fa = {};
  ja.nmat = nmat;
  ja.nb = nb;
  ja.max_sweeps = max_sweeps;
  ja.inner_sweeps = 1;
  if (const char* e = getenv("RBKI_JACOBI_INNER")) ja.inner_sweeps = std::max(1, atoi(e));
  ja.tol = 1e-12;
  ja.max_nblk = 2;
  hipError_t e;
  for (int k = 0; k < nmat; ++k) {
    const int64_t n = ns[k];
    int nbk = (int)ceil_div(n, nb);
    if (nbk < 2) nbk = 2;
    if (nbk & 1) ++nbk;
    const int64_t npad = (int64_t)nb * nbk;
    char* w = (char*)work[k];
    ja.A[k] = (double*)w;
    ja.n[k] = n;
    ja.nblk[k] = nbk;
    ja.info[k] = info[k];
    ja.max_nblk = std::max(ja.max_nblk, nbk);
    fa.A[k] = ja.A[k];
    fa.n[k] = n;
    fa.lam[k] = lam[k];
    fa.Vt[k] = Vt[k];
    fa.norms[k] = (double*)(w + npad * n * 8);
    hipLaunchKernelGGL(pad_copy_kernel, dim3(grid_for(npad * n)), dim3(256), 0, st, Z[k], n, npad, ja.A[k]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // the convergence slots live after matrix 0's scratch
  {
    int nb0 = (int)ceil_div(ns[0], nb);
    if (nb0 < 2) nb0 = 2;
    if (nb0 & 1) ++nb0;
    (void)nb0;
  }
  ja.offmax = (unsigned long long*)((char*)work[0] + jacobi_work_bytes(ns[0]) - 256);
  ja.prof = getenv("RBKI_JACOBI_PROF") ? ja.offmax + 3 * JAC_MAXB : nullptr;   // 6 slots after offmax
  hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(64), 0, st, (unsigned*)ja.offmax, (size_t)(3 * JAC_MAXB * 2 + 12));
  if ((e = hipGetLastError()) != hipSuccess) return e;
  ja.npos = ja.max_nblk / 2;
  ja.ld = (nmax & 1) ? nmax : nmax + 1;
  const size_t shmem = jacobi_lds_bytes(nmax, nb);
  if (per_matrix) {
    e = hipFuncSetAttribute((const void*)jacobi_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)shmem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(jacobi_kernel<false>, dim3(nmat), dim3(1024), shmem, st, ja);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  } else {
    e = hipFuncSetAttribute((const void*)jacobi_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)shmem);
    if (e != hipSuccess) return e;
    void* args[] = {&ja};
    e = hipLaunchCooperativeKernel((const void*)jacobi_kernel<true>, dim3(ja.npos * nmat), dim3(1024), args, shmem,
                                   st);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(jacobi_finish_kernel, dim3(nmat), dim3(1024), 0, st, fa);
  return hipGetLastError();
}

hipError_t jacobi_eig(const double* Z, int64_t n, double* lam, double* Vt, void* work, int* info, int max_sweeps,
                      hipStream_t st) {
  const double* Zs[1] = {Z};
  int64_t ns[1] = {n};
  double* ls[1] = {lam};
  double* vs[1] = {Vt};
  void* ws[1] = {work};
  int* is[1] = {info};
  return jacobi_eig_batched(1, Zs, ns, ls, vs, ws, is, max_sweeps, st);
}

hipError_t copy_rows_f64(double* dst, int64_t ldd, const double* src, int64_t lds, int64_t rows, int64_t cols,
                         hipStream_t st) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(copy_rows_kernel, dim3(grid_for(rows * cols)), dim3(256), 0, st, dst, ldd, src, lds, rows, cols);
  return hipGetLastError();
}

hipError_t store_factor(const double* Ut, int64_t R, int64_t I, void* out, int out_elem, hipStream_t st) {
  if (out_elem == E_F64)
    hipLaunchKernelGGL(store_factor_kernel<double>, dim3(grid_for(R * I)), dim3(256), 0, st, Ut, R, I, (double*)out);
  else
    hipLaunchKernelGGL(store_factor_kernel<float>, dim3(grid_for(R * I)), dim3(256), 0, st, Ut, R, I, (float*)out);
  return hipGetLastError();
}

hipError_t canonical_sign_rows(double* V, int64_t rows, int64_t n, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(canonical_sign_rows_kernel, dim3((unsigned)ceil_div(rows, 4)), dim3(256), 0, st, V, rows, n);
  return hipGetLastError();
}

hipError_t finish_factors(const FinishJob* jobs, int njobs, hipStream_t st) {
  if (njobs < 1) return hipSuccess;
  if (njobs > 8) return hipErrorInvalidValue;
  FactorArgs args = {};
  int64_t rows = 1;
  for (int i = 0; i < njobs; ++i) {
    args.job[i] = jobs[i];
    rows = std::max(rows, jobs[i].R);
  }
  hipLaunchKernelGGL(finish_factors_kernel, dim3((unsigned)rows, njobs), dim3(256), 0, st, args);
  return hipGetLastError();
}

hipError_t fill_zero(void* p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for((int64_t)(bytes / 4))), dim3(256), 0, st, (unsigned*)p, bytes / 4);
  return hipGetLastError();
}

}  // namespace rbki
