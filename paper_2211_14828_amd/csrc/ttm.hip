// Mode-n products (Alg. 2, step 6: G <- G x_n U^(n)T, and the reconstruction
// G x_n U^(n)) and the fused reconstruction-error reduction, on MFMA.
//
// Both are products out[row, col] = sum_k Aop[row, k] * Bop[col, k] in which
// each operand is strided: either k is its contiguous index ("k-contiguous")
// or the row is ("row-contiguous", transposed while staged into LDS).  A
// mode-n product with U on the view [A, I, B] is, for every a, the product
// Y[a] (R x B) = U^T (R x I) X[a] (I x B); for the last mode (B = 1) it is
// Y (A x R) = X (A x I) U (I x R).  The error pass computes the mode-0
// reconstruction Xhat_(0) = U^(1) H tile by tile and folds (x - xhat)^2 and
// x^2 into float64 partial sums without writing Xhat.
#include "rbki_kernels.h"
#include "rbki_mma.h"

namespace rbki {

namespace {

struct Operand {
  const void* base;
  int64_t row_stride, k_stride;   // one of them is 1
  int64_t batch_stride;
  int64_t rows;                   // valid rows
};

struct ProdArgs {
  Operand a, b;
  int64_t K;                      // contraction length
  int64_t row_tiles, col_tiles;
  // store epilogue
  void* out;
  int64_t out_rs, out_cs, out_bs;
  int64_t out_in, out_inp;        // out_inp > 0: output columns are padded (groups of out_inp, out_in valid)
  // residual epilogue: X (row-major rows x J) of element x_elem
  const void* X;
  int x_elem;
  int64_t xJ;
  double* partial;                // [grid] x 2
  int vec_a, vec_b;
};

// Stage 4 chunks (16 bytes each) of one operand tile in registers.
// VEC (row starts 16-byte aligned, and the sizes make every chunk wholly in
// or wholly out of range): each lane loads unconditionally from a clamped,
// valid address and keeps a validity bit per chunk; the mask is applied when
// the chunks are written to LDS, so no load sits under divergent control flow.
template <int E, bool VEC>
__device__ inline void load_op(uint4* chunk, unsigned& valid, const Operand& op, int64_t batch, int64_t row0,
                               int64_t k0, int64_t K) {
  typedef typename Mma<E>::T T;
  constexpr int EPC = 16 / (int)sizeof(T);
  constexpr int BK = Mma<E>::BK;
  const T* base = (const T*)op.base + batch * op.batch_stride;
  const int tid = threadIdx.x;
  valid = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = tid + 256 * j;
    if (op.k_stride == 1) {
      const int row = c / (BK / EPC);
      const int kk = (c % (BK / EPC)) * EPC;
      const int64_t r = row0 + row, k = k0 + kk;
      if (VEC) {
        const int64_t rc = r < op.rows ? r : op.rows - 1;
        const int64_t kc = k < K ? k : 0;
        chunk[j] = *(const uint4*)(base + rc * op.row_stride + kc);
        valid |= (r < op.rows && k < K) ? 1u << j : 0u;
      } else {
        union { uint4 v; T e[EPC]; } u;
        u.v = make_uint4(0, 0, 0, 0);
        if (r < op.rows) {
          const T* p = base + r * op.row_stride + k;
#pragma unroll
          for (int e = 0; e < EPC; ++e)
            if (k + e < K) u.e[e] = p[e];
        }
        chunk[j] = u.v;
        valid |= 1u << j;
      }
    } else {
      const int per_k = TILE / EPC;
      const int kk = c / per_k;
      const int row = (c % per_k) * EPC;
      const int64_t r = row0 + row, k = k0 + kk;
      if (VEC) {
        const int64_t rc = r < op.rows ? r : op.rows - EPC;
        const int64_t kc = k < K ? k : 0;
        chunk[j] = *(const uint4*)(base + kc * op.k_stride + rc);
        valid |= (r < op.rows && k < K) ? 1u << j : 0u;
      } else {
        union { uint4 v; T e[EPC]; } u;
        u.v = make_uint4(0, 0, 0, 0);
        if (k < K) {
          const T* p = base + k * op.k_stride + r;
#pragma unroll
          for (int e = 0; e < EPC; ++e)
            if (r + e < op.rows) u.e[e] = p[e];
        }
        chunk[j] = u.v;
        valid |= 1u << j;
      }
    }
  }
}

template <int E>
__device__ inline void store_op(const uint4* chunk, unsigned valid, const Operand& op, char* lds) {
  typedef typename Mma<E>::T T;
  constexpr int EPC = 16 / (int)sizeof(T);
  constexpr int BK = Mma<E>::BK;
  const int tid = threadIdx.x;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = tid + 256 * j;
    const uint4 v = ((valid >> j) & 1u) ? chunk[j] : make_uint4(0, 0, 0, 0);
    if (op.k_stride == 1) {
      const int row = c / (BK / EPC);
      const int kk = (c % (BK / EPC)) * EPC;
      *(uint4*)(lds + row * LDS_ROW + kk * (int)sizeof(T)) = v;
    } else {
      const int per_k = TILE / EPC;
      const int kk = c / per_k;
      const int row = (c % per_k) * EPC;
      union { uint4 v; T e[EPC]; } u;
      u.v = v;
#pragma unroll
      for (int e = 0; e < EPC; ++e) *(T*)(lds + (row + e) * LDS_ROW + kk * (int)sizeof(T)) = u.e[e];
    }
  }
}

template <class T> __device__ inline double load_x(const void* X, int64_t i);
template <> __device__ inline double load_x<double>(const void* X, int64_t i) { return ((const double*)X)[i]; }
template <> __device__ inline double load_x<float>(const void* X, int64_t i) { return (double)((const float*)X)[i]; }
template <> __device__ inline double load_x<bf16_t>(const void* X, int64_t i) {
  return (double)bf16_to_f32(((const bf16_t*)X)[i]);
}

// EPI = 0: store; EPI = 1: residual with X of type XT
template <int E, int EPI, class XT, bool VEC>
__global__ void __launch_bounds__(256, E == E_F64 ? 1 : 2) prod_kernel(ProdArgs p) {
  typedef Mma<E> M;
  typedef typename M::Out Out;
  constexpr int BK = M::BK;
  __shared__ __attribute__((aligned(16))) char lds[2][2][TILE * LDS_ROW];
  __shared__ double red[2][4];

  const int64_t tile = blockIdx.x;
  const int64_t batch = blockIdx.y;
  const int64_t rt = tile % p.row_tiles, ct = tile / p.row_tiles;
  const int64_t r0 = rt * TILE, c0 = ct * TILE;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = (wave >> 1) * 64, wc = (wave & 1) * 64;

  typename M::Frag f;
  M::zero(f);
  uint4 ca[4], cb[4];
  unsigned va, vb;
  const int64_t nk = ceil_div(p.K, BK);
  load_op<E, VEC>(ca, va, p.a, batch, r0, 0, p.K);
  load_op<E, VEC>(cb, vb, p.b, batch, c0, 0, p.K);
  store_op<E>(ca, va, p.a, lds[0][0]);
  store_op<E>(cb, vb, p.b, lds[0][1]);
  __syncthreads();
  for (int64_t kt = 0; kt < nk; ++kt) {
    const int buf = (int)(kt & 1);
    const bool more = kt + 1 < nk;
    if (more) {
      load_op<E, VEC>(ca, va, p.a, batch, r0, (kt + 1) * BK, p.K);
      load_op<E, VEC>(cb, vb, p.b, batch, c0, (kt + 1) * BK, p.K);
    }
    M::step(f, lds[buf][0], lds[buf][1], lane, wr, wc);
    if (more) {
      store_op<E>(ca, va, p.a, lds[buf ^ 1][0]);
      store_op<E>(cb, vb, p.b, lds[buf ^ 1][1]);
    }
    __syncthreads();
  }

  if (EPI == 0) {
    Out* out = (Out*)p.out + batch * p.out_bs;
#pragma unroll
    for (int j = 0; j < M::NACC; ++j) {
      int row, col;
      M::coord(j, lane, row, col);
      const int64_t r = r0 + wr + row;
      int64_t c = c0 + wc + col;
      if (r < p.a.rows && c < p.b.rows) {
        if (p.out_inp > 0) {                       // padded column -> true column
          const int64_t hi = c / p.out_inp, lo = c - hi * p.out_inp;
          if (lo >= p.out_in) continue;
          c = hi * p.out_in + lo;
        }
        out[r * p.out_rs + c * p.out_cs] = M::get(f, j);
      }
    }
  } else {
    double res = 0.0, nrm = 0.0;
#pragma unroll
    for (int j = 0; j < M::NACC; ++j) {
      int row, col;
      M::coord(j, lane, row, col);
      const int64_t r = r0 + wr + row, c = c0 + wc + col;
      if (r < p.a.rows && c < p.b.rows) {
        const double x = load_x<XT>(p.X, r * p.xJ + c);
        const double d = x - (double)M::get(f, j);
        res = fma(d, d, res);
        nrm = fma(x, x, nrm);
      }
    }
    res = warp_sum(res);
    nrm = warp_sum(nrm);
    if (lane == 0) {
      red[0][wave] = res;
      red[1][wave] = nrm;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const int64_t g = blockIdx.y * (int64_t)gridDim.x + blockIdx.x;
      p.partial[2 * g] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
      p.partial[2 * g + 1] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    }
  }
}

// Fixed-order sum of the per-workgroup partials.
__global__ void sum_pairs_kernel(const double* partial, int64_t n, double* out) {
  __shared__ double sr[16], sn[16];
  double r = 0.0, q = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
    r += partial[2 * i];
    q += partial[2 * i + 1];
  }
  r = warp_sum(r);
  q = warp_sum(q);
  if ((threadIdx.x & 63) == 0) {
    sr[threadIdx.x >> 6] = r;
    sn[threadIdx.x >> 6] = q;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
      a += sr[w];
      b += sn[w];
    }
    out[0] = a;
    out[1] = b;
  }
}

// ------------------------------------------------------------------------
// Streaming reconstruction-error pass of the precision forms, R <= 64, in split
// bfloat16: each workgroup owns 64 columns j0.. of X_(0),
// their H block split into bfloat16 hi + lo parts in LDS; wave w walks the
// 16-row tiles w, w + 4, ... and forms Xhat (16 x 64) of a tile as four
// 16 x 16 blocks on 16x16x32 bfloat16 MFMA, K = 64 in two steps, three
// products (Ul Hh + Uh Hl + Uh Hh).  Column c of block n is X column
// j0 + 4 c + n (H is staged in that order), so a lane's four values of a row
// are four consecutive X values, one 16-byte load.  The bound is the bytes in
// flight: with small tiles each wave has X three tiles ahead and U one tile
// ahead, two workgroups per compute unit (1.05 ms alone at 1000^3, against
// 1.16 ms with 32-row tiles one tile ahead; three workgroups per compute unit
// spill registers and took 1.55 ms).  The loads are unconditional (a tile past the
// wave's last is clamped to it) so that the wait before each product counts
// only the loads issued after its operands'.
constexpr int RS_COLS = 64;
constexpr int RS_LDS_ROW = 72;       // bf16 per LDS row: 64 k + 16 bytes of padding
constexpr int RS_TR = 16;            // rows per tile
struct ResSplitArgs {
  const bf16_t* Uh;     // I x 64 (columns >= R zero), hi parts
  const bf16_t* Ul;     // lo parts
  const float* H;       // R x J row-major
  const void* X;        // I x J row-major
  int64_t I, J;
  int R;
  double* partial;      // [gridDim.x] x 2
};

// four consecutive values of X as floats (VEC: one 16-byte or 8-byte load)
template <class XT, bool VEC>
__device__ inline float4 load_x4(const XT* p);
template <> __device__ inline float4 load_x4<float, true>(const float* p) { return *(const float4*)p; }
template <> __device__ inline float4 load_x4<float, false>(const float* p) { return make_float4(p[0], p[1], p[2], p[3]); }
template <> __device__ inline float4 load_x4<bf16_t, true>(const bf16_t* p) {
  const uint2 v = *(const uint2*)p;
  return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16),
                     __uint_as_float(v.y & 0xFFFF0000u));
}
template <> __device__ inline float4 load_x4<bf16_t, false>(const bf16_t* p) {
  return make_float4(bf16_to_f32(p[0]), bf16_to_f32(p[1]), bf16_to_f32(p[2]), bf16_to_f32(p[3]));
}

template <class XT, bool VEC>
__global__ void __launch_bounds__(256, 2) residual_split_kernel(ResSplitArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t hh[RS_COLS * RS_LDS_ROW];
  __shared__ __attribute__((aligned(16))) bf16_t hl[RS_COLS * RS_LDS_ROW];
  __shared__ double red[2][4];
  // the wave index is uniform across the wave: readfirstlane lets the
  // compiler keep row pointers and loop counters in scalar registers
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, g = lane >> 4;
  const int64_t j0 = (int64_t)blockIdx.x * RS_COLS;

  // H block -> LDS as [p][k], row p = 16 n + c holding column j0 + 4 c + n:
  // a thread takes 4 consecutive columns at one k
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = tid + 256 * q;
    const int kk = c >> 4, jj = (c & 15) * 4;
    const bool ok = kk < a.R && j0 + jj < a.J;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (ok) v = *(const float4*)(a.H + (int64_t)kk * a.J + j0 + jj);
    const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int p = 16 * e + (jj >> 2);
      const bf16_t hi = f32_to_bf16(vv[e]);
      hh[p * RS_LDS_ROW + kk] = hi;
      hl[p * RS_LDS_ROW + kk] = f32_to_bf16(vv[e] - bf16_to_f32(hi));
    }
  }
  __syncthreads();

  const XT* X = (const XT*)a.X;
  const int64_t NT = ceil_div(a.I, RS_TR);
  const int ns = NT > wave ? (int)((NT - wave + 3) / 4) : 0;      // this wave's tiles wave + 4 s
  if (ns > 0) {
    const bool whole_cols = j0 + RS_COLS <= a.J;
    // this lane's first column, clamped into the matrix (columns past J are masked)
    const int64_t jl = std::min<int64_t>(j0 + 4 * c16, a.J - 4 > 0 ? a.J - 4 : 0);
    auto tile_of = [&](int s) { return (int64_t)wave + 4 * (int64_t)std::min(s, ns - 1); };
    // X: rows 16 t + 4 g + v (clamped), columns jl .. jl + 3
    auto load_x = [&](int s, float4 (&xv)[4]) {
      const int64_t i0 = tile_of(s) * RS_TR + 4 * g;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t i = i0 + v < a.I ? i0 + v : a.I - 1;
        xv[v] = load_x4<XT, VEC>(X + i * a.J + jl);
      }
    };
    // U fragments: row 16 t + c16, k = 32 ks + 8 g .. + 7, hi then lo
    auto load_u = [&](int s, bf16x8_t (&u)[4]) {
      int64_t iu = tile_of(s) * RS_TR + c16;
      iu = iu < a.I ? iu : a.I - 1;
      const bf16_t* ph = a.Uh + iu * 64 + 8 * g;
      const bf16_t* pl = a.Ul + iu * 64 + 8 * g;
      u[0] = *(const bf16x8_t*)ph;
      u[1] = *(const bf16x8_t*)(ph + 32);
      u[2] = *(const bf16x8_t*)pl;
      u[3] = *(const bf16x8_t*)(pl + 32);
    };
    double res = 0.0, nrm = 0.0;
    auto tile = [&](int s, const bf16x8_t (&u)[4], const float4 (&xv)[4]) {
      f32x4_t acc[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) acc[n] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          const int row = (16 * n + c16) * RS_LDS_ROW + 32 * ks + 8 * g;
          const bf16x8_t bh = *(const bf16x8_t*)(hh + row);
          const bf16x8_t bl = *(const bf16x8_t*)(hl + row);
          acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u[2 + ks], bh, acc[n], 0, 0, 0);
          acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u[ks], bl, acc[n], 0, 0, 0);
          acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(u[ks], bh, acc[n], 0, 0, 0);
        }
      // item v of acc[n]: row 16 t + 4 g + v, column j0 + 4 c16 + n
      const int64_t i0 = ((int64_t)wave + 4 * (int64_t)s) * RS_TR + 4 * g;
      if (whole_cols && i0 - 4 * g + RS_TR <= a.I) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float xs[4] = {xv[v].x, xv[v].y, xv[v].z, xv[v].w};
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const double x = (double)xs[n];
            const double d = x - (double)acc[n][v];
            res = fma(d, d, res);
            nrm = fma(x, x, nrm);
          }
        }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float xs[4] = {xv[v].x, xv[v].y, xv[v].z, xv[v].w};
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            // the loaded column is jl + n; it is the tile's column only when unclamped
            const bool ok = i0 + v < a.I && j0 + 4 * c16 + n < a.J && jl == j0 + 4 * c16;
            const double x = ok ? (double)xs[n] : 0.0;
            const double d = ok ? x - (double)acc[n][v] : 0.0;
            res = fma(d, d, res);
            nrm = fma(x, x, nrm);
          }
        }
      }
    };
    // X three tiles ahead, U one tile ahead; the register sets rotate with s
    float4 x0[4], x1[4], x2[4], x3[4];
    bf16x8_t ua[4], ub[4];
    load_x(0, x0);
    load_u(0, ua);
    load_x(1, x1);
    load_x(2, x2);
    auto step = [&](int s, const bf16x8_t (&ucur)[4], bf16x8_t (&unext)[4], const float4 (&xcur)[4],
                    float4 (&xfar)[4]) {
      load_u(s + 1, unext);
      load_x(s + 3, xfar);
      if (s < ns) tile(s, ucur, xcur);
    };
    for (int s = 0; s < ns; s += 4) {
      step(s, ua, ub, x0, x3);
      step(s + 1, ub, ua, x1, x0);
      step(s + 2, ua, ub, x2, x1);
      step(s + 3, ub, ua, x3, x2);
    }
    res = warp_sum(res);
    nrm = warp_sum(nrm);
    if (lane == 0) {
      red[0][wave] = res;
      red[1][wave] = nrm;
    }
  } else if (lane == 0) {
    red[0][wave] = 0.0;
    red[1][wave] = 0.0;
  }
  __syncthreads();
  if (tid == 0) {
    a.partial[2 * blockIdx.x] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    a.partial[2 * blockIdx.x + 1] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
  }
}

// ------------------------------------------------------------------------
// Streaming mode products, float32 and float64: one operand is the tensor (or
// an intermediate), read once, the other a factor of at most a few hundred
// kilobytes.  The product is bound by the bytes of the tensor for factors of up
// to about 48 columns and by the matrix cores beyond, so a wave works alone,
// without LDS or barriers: it reads 16-byte pieces of the tensor straight into
// the operand layout of the 16x16x4 MFMA, two stages ahead, and the factor from
// L1 / L2.  With V = 16 / sizeof(T) values to a piece:
//
//  middle modes (LAST false): Y[a] (R x B) = Ut (R x K) X[a] (K x B).  The 16
//    lanes of a group take V consecutive columns each, so that the V column
//    blocks of a wave are the V values of its pieces; lane group g of a stage
//    of 4 V inner values reads rows k0 + V g + t, t < V.
//  last mode (LAST true): Y (A x R) = X (A x K) Ut^T.  A wave takes V blocks of
//    16 rows; lane group g reads values k0 + V g + t of its row.
//
// The factor's lane (row r, group g) holds Ut[r][k0 + V g + t], one piece, in
// both.  A wave forms 16 NR rows of the output (NR chosen so that R splits
// evenly over the waves that share a piece of the tensor).  Column pieces past
// the end of a slab (rows past the end) repeat the last ones and store the same
// values again; no load needs more than the element's alignment.
//
// Against tiles of 128 x 128 through LDS: 200^3 float64, R = 10, the core's and
// the reconstruction's six products 63 us (284); 64^5 float32, R = 16, the first
// product 0.96 ms (3.6; 4.5 TB/s) and the last expansion, 1.07 GB written, 0.28
// ms (1.3); 1000^3 float32, R = 50, the first product 2.0 ms beside a Gram pass
// (16 ms), the last expansion, 200 MB written, 0.10 ms (0.13).
struct StreamArgs {
  const void* X;
  const void* Ut;        // R x K row-major
  void* Y;
  int64_t A, B;          // LAST: B unused
  int K, R;
  int chunks;            // output row groups of 16 NR
  int64_t groups;        // column pieces of V (LAST: blocks of 16 V rows)
  int64_t nbg;           // column pieces per slab
  int64_t wg0;           // first workgroup of this launch
};

template <int E> struct Vec;
template <> struct Vec<E_F32> {
  typedef float T;
  static constexpr int V = 4;
  typedef float vec __attribute__((ext_vector_type(4), aligned(4)));
  typedef f32x4_t Acc;
  __device__ static inline Acc mma(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static inline int row(int g, int v) { return 4 * g + v; }      // of result value v, lane group g
};
template <> struct Vec<E_F64> {
  typedef double T;
  static constexpr int V = 2;
  typedef double vec __attribute__((ext_vector_type(2), aligned(8)));
  typedef f64x4_t Acc;
  __device__ static inline Acc mma(double a, double b, Acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static inline int row(int g, int v) { return 4 * v + g; }
};

// KS > 1: the KS waves of a workgroup split the inner dimension of one block
// of 16 rows (LAST only) and add their tiles through LDS, in float64; a wave's
// own sums move to float64 every 6 stages (inner dimensions of thousands).
template <int E, int NR, bool LAST, int KS>
__global__ void __launch_bounds__(64 * (KS > 1 ? KS : 4)) stream_kernel(StreamArgs p) {
  typedef Vec<E> W;
  typedef typename W::T T;
  typedef typename W::vec vec;
  constexpr int V = W::V, ST = 4 * V;
  constexpr int NX = KS > 1 ? 1 : V;                 // tensor pieces of a stage
  const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t unit = KS > 1 ? (int64_t)blockIdx.x : (p.wg0 + blockIdx.x) * 4 + wave;
  const int64_t blk = unit / p.chunks;
  const int r0 = (int)(unit - blk * p.chunks) * 16 * NR;
  const T* X = (const T*)p.X;
  const T* px[NX];                                   // piece n at inner value 0 (LAST) / this lane's columns
  int64_t col = 0;                                   // first column of this lane in its slab's output
  T* py[LAST ? NX : 1];
  if constexpr (LAST) {
    if (blk >= p.groups) return;
#pragma unroll
    for (int n = 0; n < NX; ++n) {
      const int64_t a = (blk * NX + n) * 16 + li, ac = a < p.A ? a : p.A - 1;
      px[n] = X + ac * p.K;
      py[n] = (T*)p.Y + ac * p.R;
    }
  } else {
    if (blk * 16 >= p.groups) return;
    const int64_t q = blk * 16 + li, qc = q < p.groups ? q : p.groups - 1;
    const int64_t a = qc / p.nbg;
    const int64_t b = (qc - a * p.nbg) * V;
    col = b < p.B - V ? b : p.B - V;
    px[0] = X + a * p.K * p.B + col;
    py[0] = (T*)p.Y + a * p.R * p.B + col;
  }
  const T* pu[NR];
#pragma unroll
  for (int u = 0; u < NR; ++u) {
    const int r = r0 + 16 * u + li;
    pu[u] = (const T*)p.Ut + (int64_t)(r < p.R ? r : p.R - 1) * p.K;
  }
  typename W::Acc acc[NR][NX];
#pragma unroll
  for (int u = 0; u < NR; ++u)
#pragma unroll
    for (int n = 0; n < NX; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[u][n][v] = 0;

  struct Stage {
    vec x[LAST ? NX : V];
    vec u[NR];
  };
  auto load = [&](Stage& s, int k0) {
    const int k = k0 + V * g;
#pragma unroll
    for (int i = 0; i < (LAST ? NX : V); ++i)
      s.x[i] = LAST ? *(const vec*)(px[LAST ? i : 0] + k) : *(const vec*)(px[0] + (int64_t)(k + i) * p.B);
#pragma unroll
    for (int u = 0; u < NR; ++u) s.u[u] = *(const vec*)(pu[u] + k);
  };
  // the last, partial stage: values from K on are zeros of both operands
  auto load_tail = [&](Stage& s, int k0) {
    const int k = k0 + V * g;
#pragma unroll
    for (int i = 0; i < (LAST ? NX : V); ++i)
#pragma unroll
      for (int t = 0; t < V; ++t) {
        if (LAST) s.x[i][t] = k + t < p.K ? px[LAST ? i : 0][k + t] : (T)0;
        else s.x[i][t] = k + i < p.K ? px[0][(int64_t)(k + i) * p.B + t] : (T)0;
      }
#pragma unroll
    for (int u = 0; u < NR; ++u)
#pragma unroll
      for (int t = 0; t < V; ++t) s.u[u][t] = k + t < p.K ? pu[u][k + t] : (T)0;
  };
  auto mul = [&](const Stage& s) {
#pragma unroll
    for (int t = 0; t < V; ++t)
#pragma unroll
      for (int u = 0; u < NR; ++u)
#pragma unroll
        for (int n = 0; n < NX; ++n) acc[u][n] = W::mma(s.u[u][t], LAST ? s.x[LAST ? n : 0][t] : s.x[t][n], acc[u][n]);
  };
  // whole stages, this wave's share (KS > 1: every KS-th)
  const int ns = p.K / ST, first = KS > 1 ? wave : 0;
  constexpr int step = KS > 1 ? KS : 1;
  Stage s0, s1, s2;
  auto at = [&](int s) { return (s < ns ? s : ns - 1) * ST; };
  double big[KS > 1 ? NR : 1][4] = {};
  auto flush = [&]() {
#pragma unroll
    for (int u = 0; u < (KS > 1 ? NR : 0); ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        big[u][v] += (double)acc[u][0][v];
        acc[u][0][v] = 0;
      }
  };
  if (first < ns) {
    load(s0, first * ST);
    load(s1, at(first + step));
    for (int s = first; s < ns; s += 3 * step) {
      load(s2, at(s + 2 * step));
      mul(s0);
      if (s + step >= ns) break;
      load(s0, at(s + 3 * step));
      mul(s1);
      if (s + 2 * step >= ns) break;
      load(s1, at(s + 4 * step));
      mul(s2);
      if (KS > 1 && (s - first) / step % 6 == 3) flush();
    }
  }
  if (ns * ST < p.K && (KS == 1 || wave == ns % KS)) {
    load_tail(s0, ns * ST);
    mul(s0);
  }

  if constexpr (KS > 1) {
    __shared__ double sums[KS][NR * 256];
    flush();
#pragma unroll
    for (int u = 0; u < NR; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) sums[wave][(16 * u + W::row(g, v)) * 16 + li] = big[u][v];
    __syncthreads();
    for (int e = threadIdx.x; e < NR * 256; e += 64 * KS) {
      // consecutive threads take consecutive output columns of a row
      const int i = e / (16 * NR), rr = e % (16 * NR);
      double v = sums[0][rr * 16 + i];
#pragma unroll
      for (int w = 1; w < KS; ++w) v += sums[w][rr * 16 + i];
      const int64_t a = blk * 16 + i;
      if (a < p.A && r0 + rr < p.R) ((T*)p.Y)[a * p.R + r0 + rr] = (T)v;
    }
  } else {
#pragma unroll
    for (int u = 0; u < NR; ++u) {
      if constexpr (LAST && E == E_F32) {
        // a lane's four result values are consecutive columns
        const int r = r0 + 16 * u + 4 * g;
#pragma unroll
        for (int n = 0; n < NX; ++n) {
          if (r + 4 <= p.R) {
            *(vec*)(py[LAST ? n : 0] + r) = vec{acc[u][n][0], acc[u][n][1], acc[u][n][2], acc[u][n][3]};
          } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (r + v < p.R) py[LAST ? n : 0][r + v] = acc[u][n][v];
          }
        }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = r0 + 16 * u + W::row(g, v);
          if (r >= p.R) continue;
          if constexpr (LAST) {
#pragma unroll
            for (int n = 0; n < NX; ++n) py[n][r] = acc[u][n][v];
          } else {
            vec o;
#pragma unroll
            for (int n = 0; n < V; ++n) o[n] = acc[u][n][v];
            *(vec*)(py[0] + (int64_t)r * p.B) = o;
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------------------
// Reconstruction error in the operand types' own precision: sum (x - xhat)^2
// and sum x^2 over X_(0) (I x J), Xhat = U H with R <= 128, on the same MFMA.
// A wave owns 16 column pieces of V values; H's R x 16 V block stays in its
// registers and the wave walks its share of the 16-row tiles: U's tile from L1 /
// L2 (one value a lane and inner step, from Ut as it is), X's tile as 16-byte
// pieces in the layout of the result, two tiles ahead.  No LDS and no barrier
// until the sums.  x - xhat and both sums are float64; each of a lane's V
// columns has its own sums, and those that a shifted last piece repeats are left
// out at the end.
// Against 128-row tiles: 1000^3 float32, R = 50, 1.40 ms (1.82; the float32
// matrix cores need 0.75 of it, the float64 sums most of the rest); 64^5, R = 16,
// 1.08 ms (2.95; 4.0 TB/s); 200^3 float64, R = 10, 16 us (81).
struct ResidualArgs {
  const void* X;        // I x J
  const void* Ut;       // R x I
  const void* H;        // R x J
  int64_t I, J;
  int R;
  int64_t blocks;       // column blocks of 16 V
  int rchunks;          // row ranges
  double* partial;      // [gridDim.x] x 2
};

template <class XT, int V> struct XPiece;
template <> struct XPiece<float, 4> { typedef float vec __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct XPiece<double, 2> { typedef double vec __attribute__((ext_vector_type(2), aligned(8))); };
template <> struct XPiece<bf16_t, 4> { typedef unsigned short vec __attribute__((ext_vector_type(4), aligned(2))); };
template <class XT> __device__ inline double x_value(XT v) {
  if constexpr (sizeof(XT) == 2) return (double)bf16_to_f32(v);
  else return (double)v;
}

template <class XT, int E, int NK>
__global__ void __launch_bounds__(256, NK > 4 ? 1 : 2) residual_stream_kernel(ResidualArgs p) {
  typedef Vec<E> W;
  typedef typename W::T T;
  constexpr int V = W::V;
  typedef typename W::vec vec;
  typedef typename XPiece<XT, V>::vec xvec;
  __shared__ double red[2][4];
  const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t ntile = ceil_div(p.I, 16);
  double res = 0.0, nrm = 0.0;
  for (int64_t unit = (int64_t)blockIdx.x * 4 + wave; unit < p.blocks * p.rchunks; unit += (int64_t)gridDim.x * 4) {
    const int64_t blk = unit / p.rchunks, rc = unit - blk * p.rchunks;
    const int64_t t0 = rc * ntile / p.rchunks, t1 = (rc + 1) * ntile / p.rchunks;
    const int64_t want = (blk * 16 + li) * V;                    // this lane's columns
    const int64_t c = want < p.J - V ? want : p.J - V;
    // H: inner step k, lane group g: row 4 k + g
    T h[NK * 4][V];
#pragma unroll
    for (int k = 0; k < NK * 4; ++k) {
      const int r = 4 * k + g;
      const vec v = *(const vec*)((const T*)p.H + (int64_t)(r < p.R ? r : p.R - 1) * p.J + c);
#pragma unroll
      for (int n = 0; n < V; ++n) h[k][n] = r < p.R ? v[n] : (T)0;
    }
    double rs[V] = {}, ns[V] = {};
    struct Tile { xvec x[4]; };
    auto load = [&](Tile& t, int64_t it) {
      it = it < t1 ? it : t1 - 1;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        int64_t i = it * 16 + W::row(g, v);
        i = i < p.I ? i : p.I - 1;
        t.x[v] = *(const xvec*)((const XT*)p.X + i * p.J + c);
      }
    };
    auto tile = [&](const Tile& t, int64_t it) {
      const int64_t i = it * 16 + li;
      const T* pu = (const T*)p.Ut + (i < p.I ? i : p.I - 1);
      typename W::Acc acc[V];
#pragma unroll
      for (int n = 0; n < V; ++n)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[n][v] = 0;
      T u[NK * 4];
#pragma unroll
      for (int k = 0; k < NK * 4; ++k) {
        const int r = 4 * k + g;
        u[k] = pu[(int64_t)(r < p.R ? r : p.R - 1) * p.I];
      }
#pragma unroll
      for (int k = 0; k < NK * 4; ++k) {
        if (NK > 2 && k > NK * 4 - 4 && 4 * k >= p.R) break;    // steps past R
#pragma unroll
        for (int n = 0; n < V; ++n) acc[n] = W::mma(u[k], h[k][n], acc[n]);
      }
      auto add = [&](int n, double x, double xh) {
        const double d = x - xh;
        rs[n] = fma(d, d, rs[n]);
        ns[n] = fma(x, x, ns[n]);
      };
      if (it * 16 + 16 <= p.I) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int n = 0; n < V; ++n) add(n, x_value<XT>(t.x[v][n]), (double)acc[n][v]);
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (it * 16 + W::row(g, v) < p.I)
#pragma unroll
            for (int n = 0; n < V; ++n) add(n, x_value<XT>(t.x[v][n]), (double)acc[n][v]);
      }
    };
    Tile a, b2, c2;
    load(a, t0);
    load(b2, t0 + 1);
    for (int64_t it = t0; it < t1; it += 3) {
      load(c2, it + 2);
      tile(a, it);
      if (it + 1 >= t1) break;
      load(a, it + 3);
      tile(b2, it + 1);
      if (it + 2 >= t1) break;
      load(b2, it + 4);
      tile(c2, it + 2);
    }
#pragma unroll
    for (int n = 0; n < V; ++n) {
      // a shifted piece counts only the columns from its place on
      if (want < p.J && c + n >= want) {
        res += rs[n];
        nrm += ns[n];
      }
    }
  }
  res = warp_sum(res);
  nrm = warp_sum(nrm);
  if (lane == 0) {
    red[0][wave] = res;
    red[1][wave] = nrm;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    p.partial[2 * blockIdx.x] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    p.partial[2 * blockIdx.x + 1] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
  }
}

// U (given as Ut, R x I float32) -> Up (I x 64, zero-padded columns) in split
// bfloat16: hi = rounded value, lo = rounded remainder, the lo block after the
// hi block
__global__ void pad_u_kernel(const float* Ut, int64_t R, int64_t I, bf16_t* Up) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < I * 64;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = e >> 6, k = e & 63;
    const float v = k < R ? Ut[k * I + i] : 0.f;
    const bf16_t hi = f32_to_bf16(v);
    Up[e] = hi;
    Up[I * 64 + e] = f32_to_bf16(v - bf16_to_f32(hi));
  }
}

template <class S, class D> __device__ inline D conv(S v);
template <> __device__ inline float conv<double, float>(double v) { return (float)v; }
template <> __device__ inline double conv<float, double>(float v) { return (double)v; }
template <> __device__ inline float conv<float, float>(float v) { return v; }
template <> __device__ inline double conv<double, double>(double v) { return v; }
template <> __device__ inline bf16_t conv<float, bf16_t>(float v) { return f32_to_bf16(v); }
template <> __device__ inline bf16_t conv<double, bf16_t>(double v) { return f32_to_bf16((float)v); }
template <> __device__ inline float conv<bf16_t, float>(bf16_t v) { return bf16_to_f32(v); }
template <> __device__ inline double conv<bf16_t, double>(bf16_t v) { return (double)bf16_to_f32(v); }
template <> __device__ inline bf16_t conv<bf16_t, bf16_t>(bf16_t v) { return v; }

template <class S, class D>
__global__ void convert_kernel(const S* src, D* dst, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = conv<S, D>(src[i]);
}

// ------------------------------------------------------------------------
// First mode product of the precision forms from the mode's K-blocked copy
// (the Gram operand, [K tile][ipad rows][64 bytes], bfloat16 or block-scaled
// e4m3): Y[a, r, b] = sum_i U[i, r] X[a, i, b], R <= 64.  A workgroup owns 64
// padded columns (one e4m3 K tile or two bfloat16 ones) and all R rows of Y.
// The contraction over the ipad rows runs in chunks of 256: each chunk is
// decoded to bfloat16 and transposed into LDS as [column][row] (a thread
// decodes 8 rows x 8 columns and writes 8 16-byte column pieces).  Wave w
// takes positions 64 w .. 64 w + 63 of every chunk for the whole 64 x 64
// block (2 x 2 32x32x16 bfloat16 MFMA tiles, one row tile when R <= 32); the
// four partial blocks are added through LDS at the end of the block.  A
// workgroup takes a run of consecutive blocks and walks their chunks as one
// stream, so the loads run ahead across block ends and the next block's first
// chunks arrive while a block's partials are added.  The loads are ordered for the in-order retirement of
// vector loads: the chunk two steps ahead is in flight while a chunk is
// multiplied, and a wave's U pieces for the next step are loaded one step
// ahead into registers, so no MFMA waits on a load issued after an X load.
// U (bfloat16, zero past R and I) is stored in the order the waves read it:
// for chunk ch, wave w, k step s and row tile t, the 64 lanes' 8-value pieces
// are 1 KB contiguous, so a U load reads whole cache lines.
struct FirstArgs {
  const unsigned char* X;    // blocked copy
  const unsigned char* sc;   // e4m3 scales (the Gram operand's layout), or null
  const bf16_t* U;           // fragment order, 64 x ipad values
  float* Y;                  // [A][R][B]
  int64_t ipad, Bp, B, IN, INp;
  int64_t nblk;              // 64-column blocks
  int bpw;                   // consecutive blocks per workgroup
  int R;
};

constexpr int F_CH = 256;                    // rows per chunk
constexpr int F_ROW = F_CH * 2 + 16;         // LDS bytes per column row (padded)
constexpr int F_PART = 65;                   // floats per row of a partial block in LDS
constexpr int FIRST_RUN = 4;                 // 64-column blocks per workgroup
static_assert(4 * 64 * F_PART * 4 <= 2 * 64 * F_ROW, "the partial blocks reuse the chunk buffers");

// two floats -> packed bfloat16 (a in the low half), rounded to nearest even
__device__ inline uint32_t pack_bf16x2(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f2v;
  typedef __attribute__((ext_vector_type(2))) __bf16 b2v;
  const b2v h = __builtin_convertvector((f2v){a, b}, b2v);
  return __builtin_bit_cast(uint32_t, h);
}

// one thread's share of a chunk: 8 rows x 16 bytes (bfloat16) or 8 bytes
// (e4m3, in .x .y) and, for e4m3, the 8 rows' scale bytes
struct FirstRaw {
  uint4 v[8];
  uint2 scl;
};

template <int E, bool TWO>
__global__ void __launch_bounds__(256, 2) ttm_first_kernel(FirstArgs a) {
  __shared__ __attribute__((aligned(16))) char lds[2][64 * F_ROW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // staging: thread (rl, cg) takes rows rl + 32 e (e = 0..7) of the chunk and
  // columns 8 cg .. 8 cg + 7.  Row rl + 32 e goes to chunk position 8 rl + e
  // (the contraction order inside a chunk is free; U is stored in the same
  // order), so a thread writes 8 consecutive positions of every column, and
  // its 8 e4m3 scales are 8 consecutive bytes of the scale layout.  rl runs
  // fastest over the lanes: the 8 lanes of a group write 8 consecutive 16-byte
  // pieces of one column row (distinct LDS banks), and a wave still loads 8
  // whole 64-byte rows.
  const int rl = (wave << 3) | (lane & 7), cg = lane >> 3;
  const int half = lane >> 5, lr = lane & 31;
  const int kw = wave * 64 + half * 8;             // this lane's first position in a chunk
  const int nch = (int)(a.ipad / F_CH);
  // this workgroup's stream: step s is chunk s % nch of block first + s / nch
  const int64_t first = (int64_t)blockIdx.x * a.bpw;
  const int nmine = (int)std::min<int64_t>(a.bpw, a.nblk - first);
  const int S = nmine * nch;
  if (S <= 0) return;
  auto block_of = [&](int s) { return first + s / nch; };

  auto load_x = [&](int s, FirstRaw& x) {
    const int64_t blk = block_of(s);
    const int ch = s % nch;
    const int64_t row0 = (int64_t)ch * F_CH;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t i = row0 + rl + 32 * e;
      if (E == E_FP8) {
        const uint2 v = *(const uint2*)(a.X + (blk * a.ipad + i) * 64 + cg * 8);
        x.v[e] = make_uint4(v.x, v.y, 0u, 0u);
      } else {
        const int64_t kt = blk * 2 + (cg >> 2);
        x.v[e] = *(const uint4*)(a.X + (kt * a.ipad + i) * 64 + (cg & 3) * 16);
      }
    }
    if (E == E_FP8) {
      // scale byte e of row rl + 32 e: [K tile][256-row tile][half][row % 32][row / 32]
      const int64_t tile = (blk * a.ipad + row0) >> 8;
      x.scl = *(const uint2*)(a.sc + (tile * 2 + (cg >> 2)) * 256 + rl * 8);
    }
  };
  // U pieces of a chunk: [k step][row tile] (rows lr and 32 + lr, positions
  // kw + 16 s .. + 7)
  auto load_u = [&](int ch, bf16x8_t (&u)[4][2]) {
    const bf16_t* p = a.U + ((int64_t)ch * 4 + wave) * 4096 + lane * 8;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u[s][0] = *(const bf16x8_t*)(p + s * 1024);
      if (TWO) u[s][1] = *(const bf16x8_t*)(p + s * 1024 + 512);
    }
  };
  // decode and write the transposed pieces: column 8 cg + c, positions 8 rl .. 8 rl + 7
  // (dword j of a piece: positions 2 j and 2 j + 1, the even one in the low half)
  auto store = [&](char* buf, const FirstRaw& x) {
    uint32_t o[8][4];                              // [column][position pair]
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e0 = 2 * j, e1 = 2 * j + 1;
      if (E == E_FP8) {
        // the scaled conversion gives code * 2^(byte - 127) exactly (a zero
        // byte is 2^-127); the products are e4m3 values times powers of two,
        // exact in bf16 except below bf16's subnormal range (runs of scale
        // byte 0, which hold zeros), so the packing rounds nothing else
        const uint32_t sw = j < 2 ? x.scl.x : x.scl.y;
        const float s0 = __uint_as_float(((sw >> (16 * (j & 1))) & 0xFFu) << 23);
        const float s1 = __uint_as_float(((sw >> (16 * (j & 1) + 8)) & 0xFFu) << 23);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const f32x2_t f0 = (p & 1) ? __builtin_amdgcn_cvt_scalef32_pk_f32_fp8((int)(p < 2 ? x.v[e0].x : x.v[e0].y), s0, true)
                                     : __builtin_amdgcn_cvt_scalef32_pk_f32_fp8((int)(p < 2 ? x.v[e0].x : x.v[e0].y), s0, false);
          const f32x2_t f1 = (p & 1) ? __builtin_amdgcn_cvt_scalef32_pk_f32_fp8((int)(p < 2 ? x.v[e1].x : x.v[e1].y), s1, true)
                                     : __builtin_amdgcn_cvt_scalef32_pk_f32_fp8((int)(p < 2 ? x.v[e1].x : x.v[e1].y), s1, false);
          o[2 * p][j] = pack_bf16x2(f0.x, f1.x);
          o[2 * p + 1][j] = pack_bf16x2(f0.y, f1.y);
        }
      } else {
        const uint32_t wa[4] = {x.v[e0].x, x.v[e0].y, x.v[e0].z, x.v[e0].w};
        const uint32_t wb[4] = {x.v[e1].x, x.v[e1].y, x.v[e1].z, x.v[e1].w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          o[2 * q][j] = (wa[q] & 0xFFFFu) | (wb[q] << 16);
          o[2 * q + 1][j] = (wa[q] >> 16) | (wb[q] & 0xFFFF0000u);
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c)
      *(uint4*)(buf + (cg * 8 + c) * F_ROW + rl * 16) = make_uint4(o[c][0], o[c][1], o[c][2], o[c][3]);
  };

  f32x16_t acc[2][2];                              // [row tile][column tile]
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][c][v] = 0.f;
  auto mma = [&](const char* buf, const bf16x8_t (&u)[4][2]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int k = kw + 16 * s;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const bf16x8_t bv = *(const bf16x8_t*)(buf + (c * 32 + lr) * F_ROW + k * 2);
        acc[0][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u[s][0], bv, acc[0][c], 0, 0, 0);
        if (TWO) acc[1][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u[s][1], bv, acc[1][c], 0, 0, 0);
      }
    }
  };
  // the sum of the four waves' partial blocks of block blk -> Y (the chunk
  // buffers are free when it starts; it ends with the block's partials read)
  auto finish = [&](int64_t blk) {
    // partial blocks [wave][row][column]; value v of lane l: row
    // 8 (v / 4) + 4 (l / 32) + v % 4 of the tile, column l % 32
    float* part = (float*)&lds[0][0];
#pragma unroll
    for (int t = 0; t < (TWO ? 2 : 1); ++t)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int r = t * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
          part[(wave * 64 + r) * F_PART + c * 32 + lr] = acc[t][c][v];
          acc[t][c][v] = 0.f;
        }
    __syncthreads();
    const int col = tid & 63;
    const int64_t g0 = blk * 64;                   // first padded column (over all a)
    const int64_t av_ = g0 / a.Bp, bp0 = g0 - av_ * a.Bp;
    const int64_t bp = bp0 + col;
    const int64_t hi = bp / a.INp, lo = bp - hi * a.INp;
    if (lo < a.IN) {
      float* out = a.Y + av_ * a.R * a.B + hi * a.IN + lo;
#pragma unroll
      for (int j = 0; j < (TWO ? 16 : 8); ++j) {
        const int r = (tid >> 6) + 4 * j;
        if (r < a.R) {
          float sum = 0.f;
#pragma unroll
          for (int w = 0; w < 4; ++w) sum += part[(w * 64 + r) * F_PART + col];
          out[(int64_t)r * a.B] = sum;
        }
      }
    }
    __syncthreads();
  };
  // stream step s: issue U of step s + 1 then X of step s + 2, multiply step
  // s's chunk, then write step s + 1's chunk (loaded one step earlier) to the
  // other LDS buffer; at a block's last chunk its partials are added first.
  // The loads are unconditional (a step past the end is clamped to the last
  // one, an L2 hit) so that the wait before each MFMA counts only the loads
  // issued after its operand's.
  auto step = [&](int s, const bf16x8_t (&ucur)[4][2], bf16x8_t (&unext)[4][2], const FirstRaw& have,
                  FirstRaw& next) {
    const int ch = s % nch;
    const bool last = ch + 1 == nch;
    load_u(last ? 0 : ch + 1, unext);
    load_x(min(s + 2, S - 1), next);
    mma(lds[s & 1], ucur);
    if (last) {
      __syncthreads();
      finish(block_of(s));
    }
    if (s + 1 < S) store(lds[(s + 1) & 1], have);
    __syncthreads();
  };

  FirstRaw x0, x1;
  bf16x8_t u0[4][2], u1[4][2];
  load_u(0, u0);
  load_x(0, x0);
  load_x(min(1, S - 1), x1);
  store(lds[0], x0);
  __syncthreads();
  int s = 0;
  for (; s + 1 < S; s += 2) {
    step(s, u0, u1, x1, x0);
    step(s + 1, u1, u0, x0, x1);
  }
  if (s < S) step(s, u0, u1, x1, x0);             // odd length: the last step
}

// U (given as Ut, R x I float64) -> bfloat16 in ttm_first_kernel's read
// order: element 8 (64 (2 (4 (4 ch + w) + s) + t) + l) + e is row
// 32 t + l % 32 at chunk position 64 w + 16 s + 8 (l / 32) + e, and position
// 8 q + e' of a 256-row chunk holds row q + 32 e' of U; zero past R and I
__global__ void u_first_kernel(const double* Ut, int64_t R, int64_t I, int64_t ipad, bf16_t* U) {
  for (int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; idx < 64 * ipad;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int e = (int)(idx & 7), l = (int)((idx >> 3) & 63), t = (int)((idx >> 9) & 1);
    const int s = (int)((idx >> 10) & 3), w = (int)((idx >> 12) & 3);
    const int64_t ch = idx >> 14;
    const int64_t r = 32 * t + (l & 31);
    const int pc = 64 * w + 16 * s + 8 * (l >> 5) + e;     // position in the chunk
    const int64_t i = ch * F_CH + (pc >> 3) + 32 * (pc & 7);
    U[idx] = (r < R && i < I) ? f32_to_bf16((float)Ut[r * I + i]) : (bf16_t)0;
  }
}

template <int E, int EPI, class XT>
hipError_t launch_prod(const ProdArgs& p, int64_t batches, hipStream_t s) {
  // the batch index runs on grid.y (at most 65535 per launch)
  typedef typename Mma<E>::T T;
  typedef typename Mma<E>::Out Out;
  for (int64_t b0 = 0; b0 < batches; b0 += 65535) {
    const int64_t nb = std::min<int64_t>(65535, batches - b0);
    ProdArgs q = p;
    q.a.base = (const T*)p.a.base + b0 * p.a.batch_stride;
    q.b.base = (const T*)p.b.base + b0 * p.b.batch_stride;
    if (EPI == 0) q.out = (Out*)p.out + b0 * p.out_bs;
    dim3 grid((unsigned)(p.row_tiles * p.col_tiles), (unsigned)nb);
    if (p.vec_a && p.vec_b) hipLaunchKernelGGL((prod_kernel<E, EPI, XT, true>), grid, dim3(256), 0, s, q);
    else hipLaunchKernelGGL((prod_kernel<E, EPI, XT, false>), grid, dim3(256), 0, s, q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

size_t ttm_work_bytes(int, int64_t, int64_t, int64_t, int64_t) { return 0; }

// (a launch has fewer than 2^32 threads: products of more columns take several)
constexpr int64_t STREAM_GRID = 1 << 22;
template <int E, int NR, bool LAST>
static hipError_t launch_stream_waves(StreamArgs& p, int64_t wgs, hipStream_t s) {
  for (p.wg0 = 0; p.wg0 < wgs; p.wg0 += STREAM_GRID) {
    hipLaunchKernelGGL((stream_kernel<E, NR, LAST, 1>), dim3((unsigned)std::min(STREAM_GRID, wgs - p.wg0)), dim3(256), 0,
                       s, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int E, int NR>
static hipError_t launch_stream_nr(StreamArgs& p, bool last, hipStream_t s) {
  constexpr int V = Vec<E>::V;
  if (!last) return launch_stream_waves<E, NR, false>(p, ceil_div(ceil_div(p.groups, 16) * p.chunks, 4), s);
  const int64_t wide = ceil_div(p.A, 16 * V) * p.chunks;
  if (wide < 1024 && p.K >= 8 * 4 * V) {
    // too few waves to fill the chip: eight waves share a block's inner range
    const int64_t wgs = ceil_div(p.A, 16) * p.chunks;
    p.groups = ceil_div(p.A, 16);
    hipLaunchKernelGGL((stream_kernel<E, NR, true, 8>), dim3((unsigned)wgs), dim3(512), 0, s, p);
    return hipGetLastError();
  }
  p.groups = ceil_div(p.A, 16 * V);
  return launch_stream_waves<E, NR, true>(p, ceil_div(wide, 4), s);
}

template <int E>
static hipError_t launch_stream(const void* X, int64_t A, int64_t I, int64_t B, const void* Ut, int64_t R, void* Y,
                                hipStream_t s) {
  StreamArgs p = {};
  p.X = X;
  p.Ut = Ut;
  p.Y = Y;
  p.A = A;
  p.B = B;
  p.K = (int)I;
  p.R = (int)R;
  p.chunks = (int)ceil_div(R, 64);
  p.nbg = ceil_div(B, (int64_t)Vec<E>::V);
  p.groups = A * p.nbg;
  switch ((int)ceil_div(ceil_div(R, p.chunks), 16)) {
    case 1: return launch_stream_nr<E, 1>(p, B == 1, s);
    case 2: return launch_stream_nr<E, 2>(p, B == 1, s);
    case 3: return launch_stream_nr<E, 3>(p, B == 1, s);
    default: return launch_stream_nr<E, 4>(p, B == 1, s);
  }
}

hipError_t launch_ttm(int elem, const void* X, int64_t A, int64_t I, int64_t B, const void* Ut, int64_t R,
                      void* Y, void*, size_t, hipStream_t s) {
  // float32 and float64 stream; slabs shorter than a 16-byte piece (a trailing
  // dimension of 2 or 3 below the mode) and bfloat16 take the tiles
  if (elem == E_F32 && (B == 1 || B >= Vec<E_F32>::V)) return launch_stream<E_F32>(X, A, I, B, Ut, R, Y, s);
  if (elem == E_F64) return launch_stream<E_F64>(X, A, I, B, Ut, R, Y, s);
  const int es = elem_size(elem);
  ProdArgs p = {};
  p.K = I;
  int64_t batches;
  if (B > 1) {
    // Y[a] (R x B) = Ut (R x I) . X[a] (I x B): rows r, cols b
    p.a = {Ut, I, 1, 0, R};
    p.b = {X, 1, B, I * B, B};
    p.out = Y;
    p.out_rs = B;
    p.out_cs = 1;
    p.out_bs = R * B;
    p.row_tiles = ceil_div(R, TILE);
    p.col_tiles = ceil_div(B, TILE);
    p.vec_a = (I * es) % 16 == 0 && aligned16(Ut);
    p.vec_b = (B * es) % 16 == 0 && aligned16(X);
    batches = A;
  } else {
    // Y (A x R) = X (A x I) . U (I x R): rows a, cols r
    p.a = {X, I, 1, 0, A};
    p.b = {Ut, I, 1, 0, R};
    p.out = Y;
    p.out_rs = R;
    p.out_cs = 1;
    p.out_bs = 0;
    p.row_tiles = ceil_div(A, TILE);
    p.col_tiles = ceil_div(R, TILE);
    p.vec_a = (I * es) % 16 == 0 && aligned16(X);
    p.vec_b = (I * es) % 16 == 0 && aligned16(Ut);
    batches = 1;
  }
  switch (elem) {
    case E_F32: return launch_prod<E_F32, 0, float>(p, batches, s);
    case E_BF16: return launch_prod<E_BF16, 0, float>(p, batches, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_ttm_padded(const void* Xpad, int64_t A, int64_t I, int64_t B, int64_t IN, bool last,
                             const void* Ut, int64_t R, void* Y, hipStream_t s) {
  const int64_t INp = pad64(IN);
  ProdArgs p = {};
  p.K = I;
  int64_t batches;
  if (!last) {
    // Y[a] (R x B) = Ut (R x I) . Xpad[a] (I x Bp): rows r, padded columns mapped back
    const int64_t Bp = (B / IN) * INp;
    p.a = {Ut, I, 1, 0, R};
    p.b = {Xpad, 1, Bp, I * Bp, Bp};
    p.out = Y;
    p.out_rs = B;
    p.out_cs = 1;
    p.out_bs = R * B;
    p.out_in = IN;
    p.out_inp = INp;
    p.row_tiles = ceil_div(R, TILE);
    p.col_tiles = ceil_div(Bp, TILE);
    p.vec_a = (I * 2) % 16 == 0 && aligned16(Ut);
    p.vec_b = aligned16(Xpad);
    batches = A;
  } else {
    // last mode: Y (A x R) = Xpad (A x I, row pitch I_Npad) . U (I x R)
    p.a = {Xpad, INp, 1, 0, A};
    p.b = {Ut, I, 1, 0, R};
    p.out = Y;
    p.out_rs = R;
    p.out_cs = 1;
    p.out_bs = 0;
    p.row_tiles = ceil_div(A, TILE);
    p.col_tiles = ceil_div(R, TILE);
    p.vec_a = (I * 2) % 16 == 0 && aligned16(Xpad);
    p.vec_b = (I * 2) % 16 == 0 && aligned16(Ut);
    batches = 1;
  }
  return launch_prod<E_BF16, 0, float>(p, batches, s);
}

hipError_t launch_ttm_first_blocked(int elem, const void* xb, const void* scales, int64_t A, int64_t I,
                                    int64_t B, int64_t IN, const double* Ut, int64_t R, void* U16, void* Y,
                                    hipStream_t s) {
  if (R < 1 || R > 64 || (elem != E_FP8 && elem != E_BF16)) return hipErrorInvalidValue;
  const int64_t INp = pad64(IN), ipad = block_rows(I);
  const int64_t Bp = (B / IN) * INp;
  hipLaunchKernelGGL(u_first_kernel, dim3((unsigned)std::min<int64_t>(ceil_div(64 * ipad, 256), 2048)), dim3(256), 0,
                     s, Ut, R, I, ipad, (bf16_t*)U16);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  FirstArgs fa;
  fa.X = (const unsigned char*)xb;
  fa.sc = (const unsigned char*)scales;
  fa.U = (const bf16_t*)U16;
  fa.Y = (float*)Y;
  fa.ipad = ipad;
  fa.Bp = Bp;
  fa.B = B;
  fa.IN = IN;
  fa.INp = INp;
  fa.R = (int)R;
  const int64_t blocks = A * Bp / 64;
  fa.nblk = blocks;
  if (blocks < 1) return hipSuccess;
  // runs of FIRST_RUN blocks: long enough to amortise a workgroup's start
  // (its first loads and LDS fill), short enough that the dispatcher balances
  // the grid against kernels running beside it
  fa.bpw = FIRST_RUN;
  const int64_t wgs = ceil_div(blocks, (int64_t)FIRST_RUN);
  if (wgs * 256 > 0xffffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)wgs), block(256);
  if (elem == E_FP8) {
    if (R > 32) hipLaunchKernelGGL((ttm_first_kernel<E_FP8, true>), grid, block, 0, s, fa);
    else hipLaunchKernelGGL((ttm_first_kernel<E_FP8, false>), grid, block, 0, s, fa);
  } else {
    if (R > 32) hipLaunchKernelGGL((ttm_first_kernel<E_BF16, true>), grid, block, 0, s, fa);
    else hipLaunchKernelGGL((ttm_first_kernel<E_BF16, false>), grid, block, 0, s, fa);
  }
  return hipGetLastError();
}

size_t residual_work_bytes(int64_t I, int64_t J) {
  const int64_t tiles = std::max<int64_t>(ceil_div(I, TILE) * ceil_div(J, TILE), ceil_div(J, RS_COLS));
  return (size_t)tiles * 16 + 256 + (size_t)I * 64 * 4 + 64;
}

template <class XT, int E>
static hipError_t launch_residual_stream(const ResidualArgs& p, dim3 grid, hipStream_t s) {
  const int nk = (int)ceil_div(p.R, 16);
#define RS(NK)                                                                                          \
  if (nk <= NK) {                                                                                       \
    hipLaunchKernelGGL((residual_stream_kernel<XT, E, NK>), grid, dim3(256), 0, s, p);                  \
    return hipGetLastError();                                                                           \
  }
  RS(1) RS(2) RS(3) RS(4) RS(6) RS(8)
#undef RS
  return hipErrorInvalidValue;
}

hipError_t launch_residual(int x_elem, const void* X, int op_elem, const void* Ut, const void* H, int64_t I,
                           int64_t J, int64_t R, double* out, void* work, size_t, hipStream_t s, bool bf16_products) {
  const int64_t tiles = std::max<int64_t>(ceil_div(I, TILE) * ceil_div(J, TILE), ceil_div(J, RS_COLS));
  double* partial = (double*)work;
  if (bf16_products && op_elem == E_F32 && R <= 64 && (x_elem == E_F32 || x_elem == E_BF16) && J % 4 == 0 &&
      aligned16(H) && ceil_div(J, RS_COLS) * 256 <= 0xffffffff) {
    // the precision forms' streaming pass
    void* Up = (char*)work + ((tiles * 16 + 255) / 256) * 256;
    const dim3 pgrid((unsigned)std::min<int64_t>(ceil_div(I * 64, 256), 4096));
    hipLaunchKernelGGL(pad_u_kernel, pgrid, dim3(256), 0, s, (const float*)Ut, R, I, (bf16_t*)Up);
    ResSplitArgs rs;
    rs.Uh = (const bf16_t*)Up;
    rs.Ul = (const bf16_t*)Up + I * 64;
    rs.H = (const float*)H;
    rs.X = X;
    rs.I = I;
    rs.J = J;
    rs.R = (int)R;
    rs.partial = partial;
    const dim3 grid((unsigned)ceil_div(J, RS_COLS));
    // VEC: every row starts on a 4-value boundary, so a lane's 4 values are one load
    const bool vec = J % 4 == 0 && aligned16(X);
    if (x_elem == E_F32) {
      if (vec) hipLaunchKernelGGL((residual_split_kernel<float, true>), grid, dim3(256), 0, s, rs);
      else hipLaunchKernelGGL((residual_split_kernel<float, false>), grid, dim3(256), 0, s, rs);
    } else {
      if (vec) hipLaunchKernelGGL((residual_split_kernel<bf16_t, true>), grid, dim3(256), 0, s, rs);
      else hipLaunchKernelGGL((residual_split_kernel<bf16_t, false>), grid, dim3(256), 0, s, rs);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sum_pairs_kernel, dim3(1), dim3(1024), 0, s, (const double*)partial, (int64_t)grid.x, out);
    return hipGetLastError();
  }
  // Factors of up to 128 columns (H's block in registers) on rows of at least
  // one 16-byte piece, X in the product's type (or bfloat16 with float32
  // products); the tiles otherwise.
  const int V = op_elem == E_F64 ? Vec<E_F64>::V : Vec<E_F32>::V;
  const bool pair = (op_elem == E_F64 && x_elem == E_F64) || (op_elem == E_F32 && x_elem != E_F64);
  if (pair && R <= 128 && J >= V) {
    ResidualArgs p = {};
    p.X = X;
    p.Ut = Ut;
    p.H = H;
    p.I = I;
    p.J = J;
    p.R = (int)R;
    p.blocks = ceil_div(J, (int64_t)16 * V);
    // row ranges so that some 4096 waves have work, of four tiles at least; up
    // to 2048 workgroups then take the (column block, range) pairs in turn
    p.rchunks = (int)std::min<int64_t>(ceil_div(4096, p.blocks), std::max<int64_t>(1, ceil_div(I, 16) / 4));
    p.partial = partial;
    const dim3 grid((unsigned)std::min<int64_t>({ceil_div(p.blocks * p.rchunks, 4), 2048, tiles}));
    hipError_t e;
    if (op_elem == E_F64) e = launch_residual_stream<double, E_F64>(p, grid, s);
    else if (x_elem == E_F32) e = launch_residual_stream<float, E_F32>(p, grid, s);
    else e = launch_residual_stream<bf16_t, E_F32>(p, grid, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sum_pairs_kernel, dim3(1), dim3(1024), 0, s, (const double*)partial, (int64_t)grid.x, out);
    return hipGetLastError();
  }
  const int es = elem_size(op_elem);
  ProdArgs p = {};
  p.K = R;
  // Xhat[i, j] = sum_r U[i, r] H[r, j]: rows i from Ut (R x I, row-contiguous),
  // cols j from H (R x J, row-contiguous)
  p.a = {Ut, 1, I, 0, I};
  p.b = {H, 1, J, 0, J};
  p.row_tiles = ceil_div(I, TILE);
  p.col_tiles = ceil_div(J, TILE);
  p.vec_a = (I * es) % 16 == 0 && aligned16(Ut);
  p.vec_b = (J * es) % 16 == 0 && aligned16(H);
  p.X = X;
  p.x_elem = x_elem;
  p.xJ = J;
  p.partial = partial;
  hipError_t e;
  if (op_elem == E_F64) {
    if (x_elem != E_F64) return hipErrorInvalidValue;
    e = launch_prod<E_F64, 1, double>(p, 1, s);
  } else if (op_elem == E_F32) {
    if (x_elem == E_F32) e = launch_prod<E_F32, 1, float>(p, 1, s);
    else if (x_elem == E_BF16) e = launch_prod<E_F32, 1, bf16_t>(p, 1, s);
    else e = launch_prod<E_F32, 1, double>(p, 1, s);
  } else if (op_elem == E_BF16) {
    if (x_elem == E_F32) e = launch_prod<E_BF16, 1, float>(p, 1, s);
    else if (x_elem == E_BF16) e = launch_prod<E_BF16, 1, bf16_t>(p, 1, s);
    else e = launch_prod<E_BF16, 1, double>(p, 1, s);
  } else {
    return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  const int64_t n = p.row_tiles * p.col_tiles;
  hipLaunchKernelGGL(sum_pairs_kernel, dim3(1), dim3(1024), 0, s, (const double*)partial, n, out);
  return hipGetLastError();
}

hipError_t convert_tensor(int src_elem, const void* src, int dst_elem, void* dst, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  unsigned grid = (unsigned)std::min<int64_t>(ceil_div(n, 256), 65536);
#define CV(SE, ST, DE, DT)                                                                                    \
  if (src_elem == SE && dst_elem == DE) {                                                                     \
    hipLaunchKernelGGL((convert_kernel<ST, DT>), dim3(grid), dim3(256), 0, s, (const ST*)src, (DT*)dst, n); \
    return hipGetLastError();                                                                                 \
  }
  CV(E_F64, double, E_F32, float)
  CV(E_F32, float, E_F64, double)
  CV(E_F32, float, E_F32, float)
  CV(E_F64, double, E_F64, double)
  CV(E_F32, float, E_BF16, bf16_t)
  CV(E_F64, double, E_BF16, bf16_t)
  CV(E_BF16, bf16_t, E_F32, float)
  CV(E_BF16, bf16_t, E_F64, double)
  CV(E_BF16, bf16_t, E_BF16, bf16_t)
#undef CV
  return hipErrorInvalidValue;
}

}  // namespace rbki
