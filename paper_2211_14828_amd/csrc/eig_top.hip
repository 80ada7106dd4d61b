// The R leading eigenpairs of small symmetric positive semidefinite float64
// matrices: the small eigenproblem of Alg. 2, steps 4-5, where only the R
// eigenvectors of Z = Q^T X_(n) X_(n)^T Q that become factor columns are
// needed.  The method is the textbook dense one for a few eigenpairs:
//
//  1. Householder reduction Z = H T H^T to a symmetric tridiagonal T.  The
//     matrix stays in the registers of G workgroups (G = 1 up to n = 165),
//     its columns dealt round-robin to their waves.  The rank-2 update of
//     step k is fused with the matrix-vector product of step k+1; with G > 1
//     the workgroups exchange their partial products and the next reflector's
//     row through a small global buffer once per step.
//  2. The R largest eigenvalues of T by multisection on Sturm counts (the
//     number of negative pivots of the LDL^T factorisation of T - x I equals
//     the number of eigenvalues below x), one wave per eigenvalue testing
//     128 points a round, in a kernel of its own.
//  3. Their eigenvectors of T by inverse iteration: a pivoted LU of
//     T - lambda I per eigenvalue, one thread each, three solves.  Eigenvalues
//     closer than 1e-3 ||T|| form a cluster whose vectors are
//     re-orthogonalised (modified Gram-Schmidt) after every solve.
//  4. Back-transformation by the Householder reflectors, one wave per vector.
//
// Results are deterministic: every sum is taken in a fixed order.
#include <cfloat>
#include <cstdlib>

#include "rbki_kernels.h"

namespace rbki {
namespace {

constexpr int EIG_MAXB = 8;
constexpr int EIG_NS_MAX = 8;                // n <= 64 * EIG_NS_MAX
constexpr int SOLVE_THREADS = 512;          // eigenvalue / eigenvector workgroup (R <= 512)
constexpr int SOLVE_WAVES = SOLVE_THREADS / 64;
constexpr int EIG_ITERS = 3;                 // inverse-iteration solves
constexpr int RED_THREADS = 512;             // reduction workgroup
constexpr int RED_WAVES = RED_THREADS / 64;
constexpr unsigned SPIN_LIMIT = 1u << 20;    // polls of one value before giving up (default)
constexpr double EPS = 0x1p-53;              // unit roundoff of float64

struct EigArgs {
  const double* Z[EIG_MAXB];
  int n[EIG_MAXB], R[EIG_MAXB];
  double* A[EIG_MAXB];       // n x n working copy; row k holds reflector k after the reduction
  double* d[EIG_MAXB];       // diagonal of T (n)
  double* e[EIG_MAXB];       // off-diagonal of T (n, last entry 0)
  double* tau[EIG_MAXB];     // reflector scalars (n)
  double* X[EIG_MAXB];       // eigenvectors of T, [r][i] (R x n)
  double* Y[EIG_MAXB];       // forward-substitution results, [r][i]
  double* ainv[EIG_MAXB];    // LU of T - lambda I per eigenvalue, [i][R]: 1 / U(i,i)
  double* bu[EIG_MAXB];      //   U(i, i+1)
  double* du[EIG_MAXB];      //   U(i, i+2)
  double* cm[EIG_MAXB];      //   multiplier of L at step i
  unsigned char* piv[EIG_MAXB];  // row interchange at step i
  double* lam[EIG_MAXB];
  double* Vt[EIG_MAXB];
  int* info[EIG_MAXB];
  int G[EIG_MAXB];           // workgroups sharing the reduction
  unsigned long long* P[EIG_MAXB];   // exchange ring, [RING][G + 1][64 NS] (zero at launch)
  unsigned spin_limit;       // polls before giving up; 0: give up at the first exchange
};

// Lane permutation of a float64 by DPP (both 32-bit halves moved alike).
template <int CTRL>
__device__ inline double dpp_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ inline double lane_f64(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}
// Sum over the 64 lanes, the same in every lane: exchanges within 16-lane
// rows by DPP (lane xor 1, xor 2, half-row mirror, row mirror), then the four
// row sums read from lanes 0, 16, 32, 48; a fixed order throughout.
__device__ inline double wave_sum(double v) {
  v += dpp_f64<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += dpp_f64<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0x141>(v);   // row_half_mirror
  v += dpp_f64<0x140>(v);   // row_mirror
  return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}

template <class T> __device__ inline T warp_min(T v) {
  for (int o = 32; o > 0; o >>= 1) { T w = __shfl_xor(v, o, 64); v = v < w ? v : w; }
  return v;
}

// Number of eigenvalues of T (diagonal dl, squared off-diagonal e2l) below
// x0 and x1, evaluated together.  A pivot smaller than pivmin in magnitude is
// replaced by -pivmin, which keeps the recurrence finite.
// 1/x from the hardware estimate and one Newton-Raphson step (relative
// error about 2^-50, which perturbs the counts as a change of e^2 in the last
// bits would)
__device__ inline double rcp_nr1(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(r, fma(-x, r, 1.0), r);
}

__device__ inline void sturm2(const double* dl, const double* e2l, int n, double pivmin, double x0, double x1,
                              int& c0, int& c1) {
  double q0 = dl[0] - x0, q1 = dl[0] - x1;
  if (fabs(q0) < pivmin) q0 = -pivmin;
  if (fabs(q1) < pivmin) q1 = -pivmin;
  c0 = q0 < 0.0;
  c1 = q1 < 0.0;
  for (int i = 1; i < n; ++i) {
    const double di = dl[i], ee = e2l[i - 1];
    q0 = (di - x0) - ee * rcp_nr1(q0);
    q1 = (di - x1) - ee * rcp_nr1(q1);
    if (fabs(q0) < pivmin) q0 = -pivmin;
    if (fabs(q1) < pivmin) q1 = -pivmin;
    c0 += q0 < 0.0;
    c1 += q1 < 0.0;
  }
}

__device__ inline double start_entry(int i, int r) {
  // fixed pseudo-random start vector entry in (-1, 1) (an integer hash)
  uint32_t h = (uint32_t)i * 0x9E3779B1u ^ ((uint32_t)r + 1u) * 0x85EBCA77u;
  h ^= h >> 16;
  h *= 0x7FEB352Du;
  h ^= h >> 15;
  h *= 0x846CA68Bu;
  h ^= h >> 16;
  return ((double)h + 0.5) * 0x1p-31 - 1.0;
}

__device__ inline double away_from_zero(double u, double tol) {
  return fabs(u) < tol ? (u < 0.0 ? -tol : tol) : u;
}

// Step 1.  The whole symmetric matrix (both triangles) stays in the registers
// of G workgroups of eight waves.  Lane l holds rows l, l + 64, ...; column j
// belongs to the wave (workgroup j % 64 % 8G / 8, wave % 8), so a wave's columns
// are the lanes wid, wid + 8G, ... of every 64, cyclic, and the waves stay level
// as the matrix shrinks.  A product y = A v is NS multiplications per column,
// with v's entry read from the lane that holds it (v_readlane) and no sum across
// lanes: the eight waves' parts of y are added from LDS.  The rank-2 update of
// step k - 1 is made on the way.
//
// G > 1 (n > 165, where one compute unit's registers end): the workgroups
// exchange their sums of y, and the owner of column k + 1 that column, once a
// step, with words that are their own flags: a cell of the exchange ring is zero
// until its value arrives as bits ^ EXCH_KEY, which is zero for no value that is
// sent (a NaN is sent as the canonical one).  So a step waits for one store and
// one load at the point where the XCDs meet, with no counter and no L2
// write-back in between.  The ring holds four steps; a workgroup clears its cells
// of step k - 2 once it has all words of step k, which no one can have sent
// without having read those of step k - 2, and the clearing is complete before
// it sends its words of step k + 1, so a cell is zero when its turn comes again.
// Polls are bounded: on time-out red_failed is raised, the call reports failure
// and no later poll waits.
//
// The rest of a step is latency: in wave 0 p, w and the next reflector (two sums
// over 64 lanes, a reciprocal square root and a reciprocal).  Against the upper
// triangle packed in LDS with a counter barrier a step: n = 39 36 us (69), n =
// 120 0.17 ms (0.37), n = 165 0.36 (0.70), n = 300 on four workgroups 1.05 ms
// (1.9), of whose 3.6 us a step the exchange takes 1.6.
constexpr int RING = 4;
constexpr unsigned long long EXCH_KEY = 0x7FF8A5C35A3CA5C3ull;
__shared__ int red_failed;

__device__ inline void exch_send(unsigned long long* p, double v) {
  const unsigned long long w = v == v ? (unsigned long long)__double_as_longlong(v) : 0x7FF8000000000000ull;
  __hip_atomic_store(p, w ^ EXCH_KEY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The workgroups that hold a matrix: registers for 8 NS^2 / G values of 8 bytes
// a thread beside the vectors.
__host__ __device__ inline int red_groups(int64_t n) {
  const int ns = (int)((n + 63) / 64);
  return n <= 165 ? 1 : ns <= 4 ? 2 : ns <= 6 ? 4 : 8;
}

// Element idx (the same in every lane) of a vector spread as x[t] = v[64 t + lane].
template <int NS>
__device__ inline double element(const double (&x)[NS], int idx) {
  // (every slot's lane is read and one kept: a chosen slot would be indexed in
  // memory)
  double v = lane_f64(x[0], idx & 63);
#pragma unroll
  for (int t = 1; t < NS; ++t) {
    const double vt = lane_f64(x[t], idx & 63);
    v = t == (idx >> 6) ? vt : v;
  }
  return v;
}

template <int NS, int G>
__device__ inline void reduce_matrix(const EigArgs& g, int m, int gi, double* sm) {
  constexpr int NM = 64 * NS, U = 8 / G, NC = NS * U;   // columns of a wave: U of every 64
  double* Vs = sm;                 // [NM] the reflector
  double* Ws = Vs + NM;            // [NM] its rank-2 partner
  double* part = Ws + NM;          // [8][NM] the waves' parts of the product
  double* ysum = part + RED_WAVES * NM;     // the product
  double* rowbuf = ysum + NM;      // column k + 1
  double* dsh = rowbuf + NM;       // diagonal, off-diagonal and tau of T, written out at the end
  double* esh = dsh + NM;
  double* tsh = esh + NM;
  double* last = tsh + NM;         // the last entry

  const int n = g.n[m];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  const int wid = gi * RED_WAVES + wave;
  const double* Z = g.Z[m];
  double* H = g.A[m];              // reflector k is written to row k (columns k+2..)

  double A[NS][NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int j = 64 * (c / U) + wid + 8 * G * (c % U);
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int i = 64 * t + lane;
      A[t][c] = (i < n && j < n) ? (i >= j ? Z[(int64_t)j * n + i] : Z[(int64_t)i * n + j]) : 0.0;
    }
  }
  for (int j = tid; j < NM; j += RED_THREADS) {
    Vs[j] = 0.0;
    Ws[j] = 0.0;
    rowbuf[j] = j < n ? Z[j] : 0.0;
  }
  if (tid == 0) red_failed = 0;
  __syncthreads();

  // Reflector k (wave 0, identical in every workgroup) from x = row k from the
  // diagonal on: v = x - beta e_{k+1} scaled so that v_{k+1} = 1,
  // tau = (beta - alpha) / beta, beta = -sign(alpha) ||x||.
  double tau = 0.0;                // wave 0: of the current reflector
  auto reflector = [&](int k, const double (&x)[NS]) {
    const double dk = element(x, k), alpha = element(x, k + 1);
    double s2 = 0.0;
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const double xt = 64 * t + lane >= k + 2 ? x[t] : 0.0;
      s2 = fma(xt, xt, s2);
    }
    s2 = wave_sum(s2);
    double beta = alpha, scal = 0.0;
    tau = 0.0;
    if (s2 > 0.0) {
      const double q = fma(alpha, alpha, s2), rs = rsq_nr(q), r = q * rs;
      beta = alpha >= 0.0 ? -r : r;
      tau = fma(fabs(alpha), rs, 1.0);
      scal = rcp_nr(alpha - beta);
    }
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int j = 64 * t + lane;
      Vs[j] = j == k + 1 ? 1.0 : (j >= k + 2 ? x[t] * scal : 0.0);
    }
    if (lane == 0) {
      dsh[k] = dk;
      esh[k] = beta;
      tsh[k] = tau;
    }
  };

  if (wave == 0 && n >= 3) {
    double x[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) x[t] = rowbuf[64 * t + lane];
    reflector(0, x);
  }
  __syncthreads();
  double v[NS], vp[NS];            // the reflectors of this and the previous step
#pragma unroll
  for (int t = 0; t < NS; ++t) v[t] = 0.0;
  for (int k = 0; k + 2 < n; ++k) {
    // columns j > k: the previous step's update A -= v w^T + w v^T, then this
    // wave's part of y = A v
    auto cell = [&](int q, int j) { return g.P[m] + ((int64_t)(k % RING) * (G + 1) + q) * NM + j; };
    {
      double wp[NS], y[NS];
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        vp[t] = v[t];
        v[t] = Vs[64 * t + lane];
        wp[t] = Ws[64 * t + lane];
        y[t] = 0.0;
      }
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (64 * s + 63 <= k || 64 * s >= n) continue;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int c = s * U + u, l = wid + 8 * G * u;
          if (64 * s + l <= k || 64 * s + l >= n) continue;
          const double vj = lane_f64(v[s], l), vpj = lane_f64(vp[s], l), wpj = lane_f64(wp[s], l);
#pragma unroll
          for (int t = 0; t < NS; ++t) {
            A[t][c] = fma(-vp[t], wpj, fma(-wp[t], vpj, A[t][c]));
            y[t] = fma(A[t][c], vj, y[t]);
          }
        }
      }
#pragma unroll
      for (int t = 0; t < NS; ++t) part[wave * NM + 64 * t + lane] = y[t];
      // column k + 1, from the wave that holds it
      if (((k + 1) & 63) % (8 * G) == wid) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          if (s != (k + 1) >> 6) continue;
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (u != ((k + 1) & 63) / (8 * G)) continue;
#pragma unroll
            for (int t = 0; t < NS; ++t) {
              rowbuf[64 * t + lane] = A[t][s * U + u];
              if (G > 1) exch_send(cell(G, 64 * t + lane), A[t][s * U + u]);
            }
          }
        }
      }
      // the reflector goes out (to be applied to the eigenvectors of T)
      if (gi == k % G && wave == RED_WAVES - 1) {
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          const int j = 64 * t + lane;
          if (j >= k + 2 && j < n) H[(int64_t)k * n + j] = v[t];
        }
      }
    }
    __syncthreads();

    auto parts = [&](int j) {
      double p[RED_WAVES];
#pragma unroll
      for (int w = 0; w < RED_WAVES; ++w) p[w] = part[w * NM + j];
      return ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    };
    double y[NS];                  // wave 0: the product
    if constexpr (G == 1) {
      if (wave == 0) {
#pragma unroll
        for (int t = 0; t < NS; ++t) y[t] = parts(64 * t + lane);
      }
    } else {
      // wave t adds the parts of rows 64 t.., sends the sum and adds those of
      // all workgroups in order
      if (wave < NS) {
        const int j = 64 * wave + lane;
        const int owner = ((k + 1) & 63) % (8 * G) / 8;
        const double own = parts(j);
        exch_send(cell(gi, j), own);
        unsigned long long w[G + 1];
        unsigned spins = 0;
        if (g.spin_limit == 0) red_failed = 1;
        for (;;) {
          bool all = true;
#pragma unroll
          for (int q = 0; q <= G; ++q) {
            w[q] = __hip_atomic_load(cell(q, j), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
#pragma unroll
          for (int q = 0; q <= G; ++q) all = all && (w[q] != 0);
          if (__all(all)) break;
          if (++spins > g.spin_limit) red_failed = 1;
          if (__hip_atomic_load(&red_failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
        }
        double sum = 0.0;
#pragma unroll
        for (int q = 0; q < G; ++q) sum += __longlong_as_double((long long)(w[q] ^ EXCH_KEY));
        ysum[j] = sum;
        if (owner != gi) rowbuf[j] = __longlong_as_double((long long)(w[G] ^ EXCH_KEY));
        // everyone has read the cells of two steps ago
        if (k >= 2) {
          unsigned long long* old = g.P[m] + (int64_t)((k - 2) % RING) * (G + 1) * NM + j;
          __hip_atomic_store(old + (int64_t)gi * NM, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (((k - 1) & 63) % (8 * G) / 8 == gi)
            __hip_atomic_store(old + (int64_t)G * NM, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __builtin_amdgcn_s_waitcnt(0);
        }
      }
      __syncthreads();
      if (wave == 0) {
#pragma unroll
        for (int t = 0; t < NS; ++t) y[t] = ysum[64 * t + lane];
      }
    }

    if (wave == 0) {
      // p = tau y, K = tau p^T v / 2, w = p - K v (zero up to k); then the next
      // reflector from row k+1, which this step's update changes by
      // w + w_{k+1} v (v_{k+1} = 1)
      double x[NS], w[NS], pv = 0.0;
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        x[t] = rowbuf[64 * t + lane];
        w[t] = 64 * t + lane > k ? tau * y[t] : 0.0;
        pv = fma(w[t], v[t], pv);
      }
      const double K = 0.5 * tau * wave_sum(pv);
#pragma unroll
      for (int t = 0; t < NS; ++t) {
        w[t] = fma(-K, v[t], w[t]);
        Ws[64 * t + lane] = w[t];
      }
      if (k + 3 < n) {
        const double wk = element(w, k + 1);
#pragma unroll
        for (int t = 0; t < NS; ++t) x[t] = 64 * t + lane > k ? x[t] - fma(wk, v[t], w[t]) : 0.0;
        reflector(k + 1, x);
      }
    }
    __syncthreads();
  }

  // the last 2 x 2 block: row n-2 (rowbuf) and entry (n-1, n-1) (its owner)
  // after the last update; then T goes out
  const bool owner = ((n - 1) & 63) % (8 * G) / 8 == gi;
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (64 * (c / U) + wid + 8 * G * (c % U) == n - 1 && lane == ((n - 1) & 63)) {
#pragma unroll
      for (int t = 0; t < NS; ++t)
        if (t == (n - 1) >> 6) last[0] = A[t][c];
    }
  __syncthreads();
  if (tid == 0) {
    if (n <= 2) {
      dsh[0] = Z[0];
      esh[0] = n == 2 ? Z[1] : 0.0;
      if (n == 2) dsh[1] = Z[3];
    } else {
      const int p = n - 2, q = n - 1;
      dsh[p] = fma(-Vs[p], Ws[p], fma(-Ws[p], Vs[p], rowbuf[p]));
      esh[p] = fma(-Vs[p], Ws[q], fma(-Ws[p], Vs[q], rowbuf[q]));
      if (owner) g.d[m][q] = fma(-Vs[q], Ws[q], fma(-Ws[q], Vs[q], last[0]));
    }
    if (red_failed && g.info[m]) g.info[m][0] = 1;
  }
  __syncthreads();
  if (gi == 0) {
    for (int i = tid; i < n; i += RED_THREADS) {
      if (i < n - 1 || n <= 2) g.d[m][i] = dsh[i];
      g.e[m][i] = i < n - 1 ? esh[i] : 0.0;
      g.tau[m][i] = i + 2 < n ? tsh[i] : 0.0;
    }
  }
}

// Each matrix takes the form of its own size, whatever else is in the launch.
// LARGE: matrices above 192 among them.
template <bool LARGE>
__global__ void __launch_bounds__(RED_THREADS) eig_reduce_kernel(EigArgs g) {
  extern __shared__ __attribute__((aligned(16))) double sm[];
  const int m = blockIdx.y, gi = blockIdx.x, n = g.n[m];
  if (gi >= g.G[m]) return;
  if (n <= 64) reduce_matrix<1, 1>(g, m, gi, sm);
  else if (n <= 128) reduce_matrix<2, 1>(g, m, gi, sm);
  else if (n <= 165) reduce_matrix<3, 1>(g, m, gi, sm);
  else if (n <= 192) reduce_matrix<3, 2>(g, m, gi, sm);
  if constexpr (LARGE) {
    if (n <= 192) return;
    if (n <= 256) reduce_matrix<4, 2>(g, m, gi, sm);
    else if (n <= 320) reduce_matrix<5, 4>(g, m, gi, sm);
    else if (n <= 384) reduce_matrix<6, 4>(g, m, gi, sm);
    else if (n <= 448) reduce_matrix<7, 8>(g, m, gi, sm);
    else reduce_matrix<8, 8>(g, m, gi, sm);
  }
}

// Bounds of the spectrum of T (wave 0 of a workgroup, from d and e in
// global memory): out[0] = ||T|| (max row sum), out[1] = the pivot floor of
// the Sturm counts, out[2], out[3] = Gershgorin lower and upper bounds;
// e2l[i] = e_i^2.
template <int NS>
__device__ inline void spectrum_bounds(const double* d, const double* e, int n, int lane, double* e2l,
                                       double* out) {
  double rmax = 0.0, e2max = 0.0, lo = DBL_MAX, hi = -DBL_MAX;
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    const int i = 64 * t + lane;
    if (i < n) {
      const double ei = e[i], off = fabs(ei) + (i > 0 ? fabs(e[i - 1]) : 0.0);
      rmax = fmax(rmax, fabs(d[i]) + off);
      e2max = fmax(e2max, ei * ei);
      lo = fmin(lo, d[i] - off);
      hi = fmax(hi, d[i] + off);
      e2l[i] = ei * ei;
    }
  }
  rmax = warp_max(rmax);
  e2max = warp_max(e2max);
  lo = warp_min(lo);
  hi = warp_max(hi);
  if (lane == 0) {
    out[0] = rmax;
    out[1] = DBL_MIN * fmax(1.0, e2max);
    out[2] = lo;
    out[3] = hi;
  }
}

// Step 2: the R largest eigenvalues of T by multisection on Sturm counts
// (the number of negative pivots of the LDL^T factorisation of T - x I is
// the number of eigenvalues below x).  A workgroup of BIS_WAVES waves takes
// one eigenvalue and tests 128 points per wave a round (P = 128 BIS_WAVES),
// so the interval shrinks P + 1-fold per round: 6 rounds to float64 accuracy
// with four waves, against 8 with one (each round is a sequential Sturm
// count, the cost).  The waves add their counts in LDS; every wave then holds
// the same interval, so all take the same exits.  Grid (R, matrices).
constexpr int BIS_WAVES = 4;

template <int NS>
__global__ void __launch_bounds__(64 * BIS_WAVES) eig_bisect_kernel(EigArgs g) {
  constexpr int NM = 64 * NS;
  __shared__ double dl[NM], e2l[NM], bnd[4];
  __shared__ int cnt[2][BIS_WAVES];
  const int m = blockIdx.y;
  const int n = g.n[m], R = g.R[m];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = (int)blockIdx.x;
  if (r >= R) return;                              // the same for the whole workgroup
  for (int i = tid; i < n; i += blockDim.x) dl[i] = g.d[m][i];
  if (wave == 0) spectrum_bounds<NS>(g.d[m], g.e[m], n, lane, e2l, bnd);
  __syncthreads();
  const double tnorm = bnd[0], pivmin = bnd[1];
  const double margin = 2.0 * n * EPS * tnorm + 2.0 * pivmin;
  const double atol = EPS * tnorm;
  constexpr int P = 128 * BIS_WAVES;               // points a round
  const int kk = n - 1 - r;                        // ascending index of the eigenvalue
  double lo = bnd[2] - margin, hi = bnd[3] + margin;
  // lo and hi are the same in every thread, so the loop is uniform
  for (int it = 0; it < 96; ++it) {
    if (hi - lo <= fmax(atol, 2.0 * EPS * fmax(fabs(lo), fabs(hi)))) break;
    const double wd = hi - lo;
    const int q = 128 * wave + lane;               // this lane's points q and q + 64
    const double x0 = lo + wd * ((double)(q + 1) / (double)(P + 1));
    const double x1 = lo + wd * ((double)(q + 65) / (double)(P + 1));
    int c0, c1;
    sturm2(dl, e2l, n, pivmin, x0, x1, c0, c1);
    const int nw = __popcll(__ballot(c0 <= kk)) + __popcll(__ballot(c1 <= kk));
    if (lane == 0) cnt[it & 1][wave] = nw;
    __syncthreads();
    int nb = 0;
#pragma unroll
    for (int w = 0; w < BIS_WAVES; ++w) nb += cnt[it & 1][w];
    const double nlo = nb > 0 ? lo + wd * ((double)nb / (double)(P + 1)) : lo;
    const double nhi = nb < P ? lo + wd * ((double)(nb + 1) / (double)(P + 1)) : hi;
    const bool progress = nhi - nlo < wd;          // false once float64 cannot split further
    lo = nlo;
    hi = nhi;
    if (!progress) break;
  }
  if (tid == 0) g.lam[m][r] = 0.5 * (lo + hi);
}

// Step 3 for one matrix per workgroup, from d and e of T and the eigenvalues.
template <int NS>
__global__ void __launch_bounds__(SOLVE_THREADS) eig_solve_kernel(EigArgs g) {
  constexpr int NM = 64 * NS;
  extern __shared__ __attribute__((aligned(16))) double sm[];
  double* dl = sm;
  double* el = dl + NM;
  double* e2l = el + NM;
  double* laml = e2l + NM;
  double* shl = laml + NM;
  double* red = shl + NM;          // 64 scalars
  int* cl = (int*)(red + 64);      // cluster starts (NM + 1)

  const int m = blockIdx.x;
  const int n = g.n[m], R = g.R[m];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < n; i += SOLVE_THREADS) {
    dl[i] = g.d[m][i];
    el[i] = g.e[m][i];
  }
  __syncthreads();

  // the spectrum's bounds, and the eigenvalues from eig_bisect_kernel
  if (wave == 0) spectrum_bounds<NS>(g.d[m], g.e[m], n, lane, e2l, red + 32);
  for (int r = tid; r < R; r += SOLVE_THREADS) laml[r] = g.lam[m][r];
  __syncthreads();
  const double tnorm = red[32];

  // ---- 3. eigenvectors of T by inverse iteration
  if (tid == 0) {
    // clusters of close eigenvalues; equal shifts within a cluster are
    // separated by a few ulps so that the factorisations differ
    const double ortol = 1e-3 * tnorm;
    int ncl = 0;
    for (int r = 0; r < R; ++r) {
      double s = laml[r];
      if (r == 0 || laml[r - 1] - laml[r] > ortol) {
        cl[ncl++] = r;
      } else {
        const double pt = 10.0 * EPS * fmax(fabs(s), EPS * tnorm);
        if (shl[r - 1] - s < pt) s = shl[r - 1] - pt;
      }
      shl[r] = s;
    }
    cl[ncl] = R;
    red[36] = (double)ncl;
  }
  __syncthreads();
  const int ncl = (int)red[36];
  const double ptol = tnorm > 0.0 ? EPS * tnorm : DBL_MIN;
  double* __restrict__ X = g.X[m];
  double* __restrict__ Y = g.Y[m];
  double* __restrict__ ainv = g.ainv[m];
  double* __restrict__ bu = g.bu[m];
  double* __restrict__ du = g.du[m];
  double* __restrict__ cm = g.cm[m];
  unsigned char* __restrict__ piv = g.piv[m];
  if (tid < R) {
    // pivoted LU of T - s I (U with two superdiagonals), and the start vector
    const int r = tid;
    const double s = shl[r];
    double* xr = X + r * n;
    double acur = dl[0] - s, bcur = n > 1 ? el[0] : 0.0;
    // branch-free: the pivot choice only selects operands
    for (int k = 0; k + 1 < n; ++k) {
      const double ck = el[k], an = dl[k + 1] - s, bn = k + 2 < n ? el[k + 1] : 0.0;
      const int o = k * R + r;
      const bool swap = fabs(acur) < fabs(ck);
      const double piv_v = swap ? ck : acur;          // U(k, k)
      const double other = swap ? acur : ck;          // entry eliminated below it
      const double mult = piv_v != 0.0 ? other * rcp_nr(piv_v) : 0.0;
      ainv[o] = rcp_nr(away_from_zero(piv_v, ptol));
      bu[o] = swap ? an : bcur;
      du[o] = swap ? bn : 0.0;
      cm[o] = mult;
      piv[o] = swap ? 1 : 0;
      const double na = swap ? fma(-mult, an, bcur) : fma(-mult, bcur, an);
      bcur = swap ? -mult * bn : bn;
      acur = na;
      xr[k] = start_entry(k, r);
    }
    const int o = (n - 1) * R + r;
    ainv[o] = rcp_nr(away_from_zero(acur, ptol));
    bu[o] = 0.0;
    du[o] = 0.0;
    xr[n - 1] = start_entry(n - 1, r);
  }
  for (int it = 0; it < EIG_ITERS; ++it) {
    if (tid < R) {
      // entries of x are at most 1 (start vector, then unit vectors); y =
      // ptol x keeps the solve finite: x <- U^-1 L^-1 P y
      const int r = tid;
      double* xr = X + r * n;
      double* yr = Y + r * n;
      // blocks of steps: all inputs of a block are loaded before any of its
      // results is stored, so that the loads overlap; each block waits about
      // one memory latency, so the blocks are as long as the registers allow
      // (32 steps forward, 24 backward)
      constexpr int B = 32;
      double yk = xr[0] * ptol;
      for (int k0 = 0; k0 + 1 < n; k0 += B) {
        double xv[B], mv[B];
        bool sv[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
          const int k = k0 + u < n - 1 ? k0 + u : n - 2;
          xv[u] = xr[k + 1];
          mv[u] = cm[k * R + r];
          sv[u] = piv[k * R + r] != 0;
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
          if (k0 + u + 1 < n) {
            // rows k and k+1 exchanged when piv: (top, bottom) = (y_{k+1}, y_k)
            const double yn = xv[u] * ptol;
            const double top = sv[u] ? yn : yk, bot = sv[u] ? yk : yn;
            yr[k0 + u] = top;
            yk = fma(-mv[u], top, bot);
          }
        }
      }
      yr[n - 1] = yk;
      double x1 = 0.0, x2 = 0.0;
      constexpr int BB = 24;
      for (int k0 = n - 1; k0 >= 0; k0 -= BB) {
        double yv[BB], dv[BB], bv[BB], av[BB];
#pragma unroll
        for (int u = 0; u < BB; ++u) {
          const int k = k0 - u >= 0 ? k0 - u : 0;
          yv[u] = yr[k];
          dv[u] = du[k * R + r];
          bv[u] = bu[k * R + r];
          av[u] = ainv[k * R + r];
        }
#pragma unroll
        for (int u = 0; u < BB; ++u) {
          if (k0 - u >= 0) {
            const double xk = fma(-dv[u], x2, fma(-bv[u], x1, yv[u])) * av[u];
            xr[k0 - u] = xk;
            x2 = x1;
            x1 = xk;
          }
        }
      }
    }
    __syncthreads();
    // modified Gram-Schmidt inside each cluster, then unit 2-norm
    for (int c = wave; c < ncl; c += SOLVE_WAVES) {
      const int s0 = cl[c], s1 = cl[c + 1];
      for (int j = s0; j < s1; ++j) {
        double xj[NS];
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          const int i = 64 * t + lane;
          const double v = X[j * n + (i < n ? i : n - 1)];
          xj[t] = i < n ? v : 0.0;
        }
        for (int p = s0; p < j; ++p) {
          double xp[NS], dot = 0.0;
#pragma unroll
          for (int t = 0; t < NS; ++t) {
            const int i = 64 * t + lane;
            const double v = X[p * n + (i < n ? i : n - 1)];
            xp[t] = i < n ? v : 0.0;
            dot = fma(xp[t], xj[t], dot);
          }
          dot = wave_sum(dot);
#pragma unroll
          for (int t = 0; t < NS; ++t) xj[t] = fma(-dot, xp[t], xj[t]);
        }
        double nn = 0.0;
#pragma unroll
        for (int t = 0; t < NS; ++t) nn = fma(xj[t], xj[t], nn);
        nn = wave_sum(nn);
        const double inv = nn > 0.0 ? 1.0 / sqrt(nn) : 0.0;
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          const int i = 64 * t + lane;
          if (i < n) X[j * n + i] = xj[t] * inv;
        }
      }
    }
    __syncthreads();
  }
}

// Step 4: x <- H_0 H_1 ... H_{n-3} x for eigenvector r of matrix m (one wave),
// written as row r of Vt.
template <int NS>
__global__ void __launch_bounds__(64) eig_back_kernel(EigArgs g) {
  const int r = blockIdx.x, m = blockIdx.y, lane = threadIdx.x;
  const int n = g.n[m], R = g.R[m];
  if (r >= R) return;
  __shared__ double taus[64 * NS];
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    const int i = 64 * t + lane;
    taus[i] = i < n ? g.tau[m][i] : 0.0;
  }
  __syncthreads();
  const double* A = g.A[m];
  const double* X = g.X[m];
  double x[NS];
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    const int i = 64 * t + lane;
    x[t] = i < n ? X[r * n + i] : 0.0;
  }
  // row k of A from a clamped address, and tau_k; the reflector (1 at k+1,
  // zero before) is formed from the row at use, so that the loads stay in
  // flight.  A zero tau gives a zero update, so no branch waits on it.
  auto load_v = [&](int k, double (&v)[NS], double& tk) {
    const int kc = k >= 0 ? k : 0;
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int j = 64 * t + lane;
      v[t] = A[kc * n + (j < n ? j : n - 1)];
    }
    tk = taus[kc];
  };
  auto apply = [&](int k, const double (&a)[NS], double tk) {
    if (k < 0) return;                             // uniform: past the last reflector
    double v[NS], dot = 0.0;
#pragma unroll
    for (int t = 0; t < NS; ++t) {
      const int j = 64 * t + lane;
      v[t] = j == k + 1 ? 1.0 : (j >= k + 2 && j < n ? a[t] : 0.0);
      dot = fma(v[t], x[t], dot);
    }
    const double f = tk * wave_sum(dot);
#pragma unroll
    for (int t = 0; t < NS; ++t) x[t] = fma(-f, v[t], x[t]);
  };
  // reflectors n-3 down to 0, BD in flight: each waits on its row about a
  // memory latency after the request, so the ring holds enough rows to
  // cover it (one wave per workgroup, registers to spare)
  constexpr int BD = 16;
  double vr[BD][NS], tr[BD];
  int k = n - 3;
#pragma unroll
  for (int u = 0; u < BD; ++u) load_v(k - u, vr[u], tr[u]);
  for (; k >= 0; k -= BD) {
#pragma unroll
    for (int u = 0; u < BD; ++u) {
      apply(k - u, vr[u], tr[u]);
      load_v(k - u - BD, vr[u], tr[u]);
    }
  }
  double* out = g.Vt[m] + (size_t)r * n;
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    const int j = 64 * t + lane;
    if (j < n) out[j] = x[t];
  }
}

size_t solve_lds_bytes(int ns) {
  const int nm = 64 * ns;
  return (size_t)(5 * nm + 64) * 8 + (size_t)(nm + 1) * 4;
}
size_t reduce_lds_bytes(int ns) { return (size_t)((7 + RED_WAVES) * 64 * ns + 8) * 8; }
size_t ring_bytes(int64_t n) {
  const int G = red_groups(n);
  return G > 1 ? (size_t)RING * (G + 1) * (size_t)(ceil_div(n, 64) * 64) * 8 : 0;
}

struct Layout {
  size_t A, d, e, tau, X, Y, ainv, bu, du, cm, piv, P, total;
};
inline size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }
Layout layout(int64_t n, int64_t R) {
  Layout L;
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o = al256(o + bytes); return at; };
  L.A = take((size_t)n * n * 8);
  L.d = take((size_t)n * 8);
  L.e = take((size_t)n * 8);
  L.tau = take((size_t)n * 8);
  L.X = take((size_t)n * R * 8);
  L.Y = take((size_t)n * R * 8);
  L.ainv = take((size_t)n * R * 8);
  L.bu = take((size_t)n * R * 8);
  L.du = take((size_t)n * R * 8);
  L.cm = take((size_t)n * R * 8);
  L.piv = take((size_t)n * R);
  L.P = take(ring_bytes(n));
  L.total = o;
  return L;
}

template <int NS>
hipError_t launch_ns(EigArgs& a, int nmat, int gmax, int rmax, bool coop, hipStream_t st) {
  hipError_t e;
  const size_t rshm = reduce_lds_bytes(NS);
  constexpr bool LARGE = NS > 3;
  const void* reduce = (const void*)eig_reduce_kernel<LARGE>;
  if ((e = hipFuncSetAttribute(reduce, hipFuncAttributeMaxDynamicSharedMemorySize, (int)reduce_lds_bytes(LARGE ? 8 : 3))) !=
      hipSuccess)
    return e;
  if (gmax > 1) {
    // the workgroups of a matrix wait for each other: a cooperative launch
    // guarantees that they are all resident.  An ordinary launch (coop false,
    // for a solve that runs beside other work) relies on the few workgroups
    // becoming resident as the device frees room; the bounded polls report a
    // failure rather than waiting for ever.
    for (int k = 0; k < nmat; ++k)
      if (a.G[k] > 1 && (e = fill_zero(a.P[k], ring_bytes(a.n[k]), st)) != hipSuccess) return e;
    if (coop) {
      void* args[] = {&a};
      e = hipLaunchCooperativeKernel(reduce, dim3(gmax, nmat), dim3(RED_THREADS), args, rshm, st);
      if (e != hipSuccess) return e;
    } else {
      hipLaunchKernelGGL(eig_reduce_kernel<LARGE>, dim3(gmax, nmat), dim3(RED_THREADS), rshm, st, a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  } else {
    hipLaunchKernelGGL(eig_reduce_kernel<LARGE>, dim3(1, nmat), dim3(RED_THREADS), rshm, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const size_t sshm = solve_lds_bytes(NS);
  if ((e = hipFuncSetAttribute((const void*)eig_solve_kernel<NS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)sshm)) != hipSuccess)
    return e;
  hipLaunchKernelGGL(eig_bisect_kernel<NS>, dim3((unsigned)rmax, nmat), dim3(64 * BIS_WAVES), 0, st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(eig_solve_kernel<NS>, dim3(nmat), dim3(SOLVE_THREADS), sshm, st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(eig_back_kernel<NS>, dim3(rmax, nmat), dim3(64), 0, st, a);
  return hipGetLastError();
}

}  // namespace

bool eig_top_ok(int64_t n, int64_t R) {
  return n >= 1 && n <= 64 * EIG_NS_MAX && R >= 1 && R <= n;
}

size_t eig_top_work_bytes(int64_t n, int64_t R) { return layout(n, R).total; }

hipError_t eig_top_batched(int nmat, const double* const* Z, const int64_t* ns, const int64_t* Rs,
                           double* const* lam, double* const* Vt, void* const* work, int* const* info,
                           hipStream_t st, bool coop) {
  if (nmat <= 0) return hipSuccess;
  if (nmat > EIG_MAXB) return hipErrorInvalidValue;
  EigArgs a = {};
  // RBKI_EIG_SPIN_LIMIT: polls of a value of a multi-workgroup reduction before
  // it gives up and reports failure (0: at once), to test the error path
  a.spin_limit = SPIN_LIMIT;
  if (const char* lim = getenv("RBKI_EIG_SPIN_LIMIT")) a.spin_limit = (unsigned)strtoul(lim, nullptr, 10);
  int64_t nmax = 0, rmax = 0;
  int gmax = 1;
  for (int k = 0; k < nmat; ++k) {
    if (!eig_top_ok(ns[k], Rs[k])) return hipErrorInvalidValue;
    const Layout L = layout(ns[k], Rs[k]);
    char* w = (char*)work[k];
    a.Z[k] = Z[k];
    a.n[k] = (int)ns[k];
    a.R[k] = (int)Rs[k];
    a.A[k] = (double*)(w + L.A);
    a.d[k] = (double*)(w + L.d);
    a.e[k] = (double*)(w + L.e);
    a.tau[k] = (double*)(w + L.tau);
    a.X[k] = (double*)(w + L.X);
    a.Y[k] = (double*)(w + L.Y);
    a.ainv[k] = (double*)(w + L.ainv);
    a.bu[k] = (double*)(w + L.bu);
    a.du[k] = (double*)(w + L.du);
    a.cm[k] = (double*)(w + L.cm);
    a.piv[k] = (unsigned char*)(w + L.piv);
    a.lam[k] = lam[k];
    a.Vt[k] = Vt[k];
    a.info[k] = info ? info[k] : nullptr;
    a.G[k] = red_groups(ns[k]);
    a.P[k] = (unsigned long long*)(w + L.P);
    gmax = std::max(gmax, a.G[k]);
    nmax = std::max(nmax, ns[k]);
    rmax = std::max(rmax, Rs[k]);
  }
  switch ((int)ceil_div(nmax, 64)) {
    case 1: return launch_ns<1>(a, nmat, gmax, (int)rmax, coop, st);
    case 2: return launch_ns<2>(a, nmat, gmax, (int)rmax, coop, st);
    case 3: return launch_ns<3>(a, nmat, gmax, (int)rmax, coop, st);
    case 4: return launch_ns<4>(a, nmat, gmax, (int)rmax, coop, st);
    case 5: return launch_ns<5>(a, nmat, gmax, (int)rmax, coop, st);
    case 6: return launch_ns<6>(a, nmat, gmax, (int)rmax, coop, st);
    case 7: return launch_ns<7>(a, nmat, gmax, (int)rmax, coop, st);
    default: return launch_ns<8>(a, nmat, gmax, (int)rmax, coop, st);
  }
}

}  // namespace rbki
