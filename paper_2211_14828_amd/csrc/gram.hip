// Sketch and Gram products of one mode, in a single pass over the tensor
// (float64, float32 and bfloat16 operands; the mixed forms' large modes have a
// pipelined kernel of their own, gram_pipe.hip).
//
// For the mode-n view [A, I, B] of the row-major tensor (Table 1:
// X_(n)[i, a*B + b] = X[a, i, b], never materialised) this computes
//   C = X_(n) X_(n)^T            (I x I, lower triangle)           (Remark 1)
//   W = X_(n) Omega^(n)          (I x S, as Omega^T X_(n)^T)       (Alg. 1, step 2)
// The output is cut into 32 x 32 blocks, and only the wanted ones are formed
// and stored: the lower triangle of C and S rows of W^T.  A workgroup of four
// waves owns one tile and a slice of the contraction (split-K); each wave forms
// up to 2 x 2 blocks.  Tiles:
//   C     128 rows x 128 columns, lower triangle (a diagonal tile stages its
//         rows once; its upper-right wave has nothing to do);
//   W     64 sketch rows x 256 columns;
//   thin  I <= 64 and S <= 64: the mode's 64 rows and the sketch's 64 rows
//         staged together, each wave 32 of them by the mode's 64 columns, so X
//         is read once (the modes of a 64^5 tensor are bound by that read).
// The slices are summed in a fixed order in float64 by a second kernel, so
// results are deterministic.
//
// Float32 operands are split exactly into three bfloat16 parts while they are
// staged, x = h + m + l with h = bf16(x), m = bf16(x - h), l = x - h - m (24
// significand bits in three parts of 8, exact where the last of them is a bfloat16
// value, subnormal or not: |x| from 2^-110 up to the largest bfloat16 value),
// and every product is formed from the six part products above 2^-24,
// hh + hm + mh + mm + hl + lh, on 32x32x16 bfloat16 MFMA with float32
// accumulation.  The terms left out (ml, lm, ll) are below 2^-25 of a product
// and of either sign.  hh and the five smaller products have an accumulator
// each, so a sum is rounded once per 16 K values against 16 times with the
// 32x32x2 float32 MFMA: for 32 rows of Gaussian values over 16384 columns the
// diagonal's error against float64 is 6.2e-7 (1.9e-6 with the float32 MFMA,
// 3.1e-6 with one accumulator for all six), over 256 columns 8.4e-8 (1.9e-7).
// The float32 MFMA has a sixteenth of the bfloat16 rate; six products leave
// 2.7 times its rate.
//
// K tiles are 128 bytes of a row.  For B of at least a tile, a tile is
// (a, b0 .. b0 + KT), rows contiguous in b, read as 16-byte pieces (which need
// no alignment beyond the element's).  For smaller B (the last mode, and the
// mode before a thin last one) a tile is KT / B whole values of a; the lanes
// then run over the mode's rows and each thread gathers its K values, so the
// staged layout needs no transposition.  A slab's last tile overlaps the one
// before it, with the values they share zeroed, so no load is masked.
//
// The bfloat16 tiles keep one order of their sums, whatever the launch: slices by the
// count of 128-row tiles (slices), K tiles of 64 values from the slab's start with
// zeros past its end, and in the MFMA of step t the values 8 t .. and 32 + 8 t ...
// One factor of a decomposition is rounded to bfloat16 again in the first mode
// product, and an entry that another order moves by 1e-7 across a rounding edge moves
// the core by a few 1e-5 (7e-5 at 100 x 128 x 144).
//
// Workgroups are dispatched round-robin over the 8 XCDs.  Those of one XCD take
// consecutive (split, tile) pairs, so the tiles of a split, which share a slab
// of X, run on one XCD (or two) and the slab is fetched from HBM once into its
// L2, for any number of splits.
// Measured per mode, against 128 x 128 tiles on the MFMA of the operand's own
// type: float32 64^5, S = 22, 1.55 ms (2.75), and 2.05 with the sketch made in place
// (below; 2.1 apart, 0.55 of it the sketch's own kernel, and the read of the sketch:
// the vector unit is busy for four fifths of it, two thirds of that on the sketch);
// float64 200^3, S = 15, 0.11 ms (0.22).
//
// Large float32 modes take the wide form below (gram_wide_kernel), modes of at most
// eight rows a form of their own (gram_tiny_kernel).
#include "rbki_kernels.h"
#include "rbki_philox.h"

namespace rbki {

namespace {

constexpr int BLK = 32;                  // output blocks
constexpr int GROUP = 64;                // staged rows come in groups of 64
constexpr int GROUPS_TILE = 5;           // the most groups of a tile (W: 1 + 4)
constexpr int GROUPS_THIN = 2;

template <int E> struct Op;
template <> struct Op<E_F64> {
  typedef double T;
  typedef double Out;
  typedef f64x4_t Acc;
  // NACC: accumulators of one row of two blocks (float32: also those of the
  // part products below hh)
  static constexpr int KT = 16, EPC = 2, NACC = 8, GROUP_BYTES = GROUP * 128;
};
template <> struct Op<E_F32> {
  typedef float T;
  typedef float Out;
  typedef f32x16_t Acc;
  static constexpr int KT = 32, EPC = 4, NACC = 4, GROUP_BYTES = GROUP * 192;   // three bfloat16 planes
};
template <> struct Op<E_BF16> {
  typedef bf16_t T;
  typedef float Out;
  typedef f32x16_t Acc;
  static constexpr int KT = 64, EPC = 8, NACC = 2, GROUP_BYTES = GROUP * 128;
};

typedef __attribute__((ext_vector_type(2))) float f32pair_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16pair_t;
typedef uint32_t u32x4u_t __attribute__((ext_vector_type(4), aligned(2)));

// The bfloat16 parts of two floats, packed (low half first).
__device__ inline uint32_t pack_bf16(float x0, float x1) {
  const f32pair_t v = {x0, x1};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16pair_t));
}
__device__ inline void split3(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = pack_bf16(x0, x1);
  const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xFFFF0000u);
  m = pack_bf16(r0, r1);
  l = pack_bf16(r0 - __uint_as_float(m << 16), r1 - __uint_as_float(m & 0xFFFF0000u));
}

// Where the K values of a tile lie: element offsets from a row's start, and
// the values [lo, hi) of the tile that count (the others are zeroed).
struct KTile {
  int64_t x, o;      // in X (a I B + b0) and in a row of Omega^T (a B + b0)
  int lo, hi;
};

// One thread's share of a staged group: 32 bytes of K values, as words.
struct Piece {
  uint32_t u[8];
};

// Rows by 16-byte pieces: piece j of a thread is row (tid / 8) + 32 j, K
// values (tid % 8) EPC ...  p[j] points at the first of them for K offset 0.
template <int E>
__device__ inline void load_rows(Piece& r, const typename Op<E>::T* const (&p)[2], int64_t off) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const u32x4u_t v = *(const u32x4u_t*)(p[j] + off);
    r.u[4 * j] = v.x; r.u[4 * j + 1] = v.y; r.u[4 * j + 2] = v.z; r.u[4 * j + 3] = v.w;
  }
}

// The same for a tile that ends with its slab after n < KT values (bfloat16): the
// values past it are zeros.
__device__ inline void load_rows_end(Piece& r, const bf16_t* const (&p)[2], int64_t off, int n) {
  const int k0 = (threadIdx.x & 7) * 8;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t lo = 0, hi = 0;
      if (k0 + 2 * i < n) lo = p[j][off + 2 * i];
      if (k0 + 2 * i + 1 < n) hi = p[j][off + 2 * i + 1];
      r.u[4 * j + i] = lo | hi << 16;
    }
}

// Rows across the lanes: thread (row tid % 64, wave w) takes K values
// w KT / 4 ... of its row at byte offset rb; koff: the values' offsets (the
// same for the whole wave), those from nk on do not exist.
template <int E>
__device__ inline void load_gather(Piece& r, const typename Op<E>::T* X, uint32_t rb, const int64_t* koff, int64_t off,
                                   int nk) {
  typedef typename Op<E>::T T;
  constexpr int KW = Op<E>::KT / 4;
  const int k0 = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * KW;
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    T v = 0;
    if (k0 + k < nk) v = *(const T*)((const char*)(X + (off + koff[k])) + rb);
    if constexpr (E == E_F64) {
      const uint64_t w = __builtin_bit_cast(uint64_t, v);
      r.u[2 * k] = (uint32_t)w;
      r.u[2 * k + 1] = (uint32_t)(w >> 32);
    } else if constexpr (E == E_F32) {
      r.u[k] = __float_as_uint(v);
    } else {
      r.u[k / 2] = k & 1 ? r.u[k / 2] | (uint32_t)v << 16 : (uint32_t)v;
    }
  }
}

// Zero the values of a piece outside [lo, hi); k(e): the K value of element e.
template <int E, class K>
__device__ inline void clip(Piece& r, int lo, int hi, K k) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if constexpr (E == E_BF16) {
      const int k0 = k(2 * i), k1 = k(2 * i + 1);
      r.u[i] &= (k0 >= lo && k0 < hi ? 0x0000FFFFu : 0u) | (k1 >= lo && k1 < hi ? 0xFFFF0000u : 0u);
    } else {
      const int ki = k(E == E_F64 ? i / 2 : i);
      if (ki < lo || ki >= hi) r.u[i] = 0;
    }
  }
}

// LDS: a row holds its K values in 16-byte chunks, the chunk index XOR-swizzled
// with the row so that the 32 (or 16) rows of one operand read and the 64 banks
// meet without conflicts.  Float32: three planes of 64-byte rows.
// (A multiple of 16 rows more moves the place by whole rows.)
template <int E> constexpr int LDS_ROW_BYTES = E == E_F32 ? 64 : 128;
template <int E>
__device__ inline int lds_at(int row, int q) {
  if constexpr (E == E_F32) return row * 64 + ((q ^ (row >> 2)) & 3) * 16;
  else return row * 128 + ((q ^ (row >> 1)) & 7) * 16;
}

template <int E, bool GATHER>
__device__ inline void store_piece(Piece r, char* lds, int plane, int grow, const KTile& t) {
  typedef Op<E> O;
  const int tid = threadIdx.x;
  if (t.lo > 0 || t.hi < O::KT)
    clip<E>(r, t.lo, t.hi, [&](int e) {
      return GATHER ? (tid >> 6) * (O::KT / 4) + e : (tid & 7) * O::EPC + e % O::EPC;
    });
  if constexpr (E == E_F32) {
    uint32_t h[4], m[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      split3(__uint_as_float(r.u[2 * i]), __uint_as_float(r.u[2 * i + 1]), h[i], m[i], l[i]);
    if constexpr (GATHER) {
      char* d = lds + lds_at<E>(grow + (tid & 63), tid >> 6);
      *(uint4*)d = make_uint4(h[0], h[1], h[2], h[3]);
      *(uint4*)(d + plane) = make_uint4(m[0], m[1], m[2], m[3]);
      *(uint4*)(d + 2 * plane) = make_uint4(l[0], l[1], l[2], l[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        char* d = lds + lds_at<E>(grow + (tid >> 3) + 32 * j, (tid & 7) >> 1) + (tid & 1) * 8;
        *(uint2*)d = make_uint2(h[2 * j], h[2 * j + 1]);
        *(uint2*)(d + plane) = make_uint2(m[2 * j], m[2 * j + 1]);
        *(uint2*)(d + 2 * plane) = make_uint2(l[2 * j], l[2 * j + 1]);
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int row = GATHER ? (tid & 63) : (tid >> 3) + 32 * j;
      const int q = GATHER ? 2 * (tid >> 6) + j : (tid & 7);
      *(uint4*)(lds + lds_at<E>(grow + row, q)) = make_uint4(r.u[4 * j], r.u[4 * j + 1], r.u[4 * j + 2], r.u[4 * j + 3]);
    }
  }
}

// Sketch values made in place (the thin float32 form, whose one tile reads each of
// them once; the other forms' tiles would make them several times over, and the
// float64 pair takes more registers than the thin form has): the tile's S rows of KT values, as the stream's pairs, thread by thread
// from thread index tid on.  When a row starts at an odd index of the stream (J or
// the tile's offset o odd) its pairs straddle the words of a row, and there is one
// more of them.  (A loop: pairs side by side would take the products' registers.)
__device__ inline void store_sketch(const GramArgs& g, char* lds, int plane, int64_t o, int tid) {
  constexpr int E = E_F32, KT = Op<E>::KT;
  const bool odd = (g.J | o) & 1;
  const int per = KT / 2 + (odd ? 1 : 0), np = g.S * per;
#pragma unroll 1
  for (int p = tid; p < np; p += 256) {
    const int row = odd ? p / (KT / 2 + 1) : p / (KT / 2);
    const int64_t L = row * g.J + o;
    const int64_t m = (L >> 1) + (p - row * per);
    const int k = 2 * (p - row * per) - (int)(L & 1);     // K value of the pair's first
    float z0, z1;
    gauss_pair_f32((uint64_t)m, (uint32_t)g.om_mode, 0u, g.seed, z0, z1);
    uint32_t part[3];
    split3(z0, z1, part[0], part[1], part[2]);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      char* d = lds + q * plane;
      if (!odd) {
        *(uint32_t*)(d + lds_at<E>(GROUP + row, k >> 3) + (k & 7) * 2) = part[q];
      } else {
        if (k >= 0 && k < KT) *(uint16_t*)(d + lds_at<E>(GROUP + row, k >> 3) + (k & 7) * 2) = (uint16_t)part[q];
        if (k + 1 < KT)
          *(uint16_t*)(d + lds_at<E>(GROUP + row, (k + 1) >> 3) + ((k + 1) & 7) * 2) = (uint16_t)(part[q] >> 16);
      }
    }
  }
}

// One K tile of a wave's MB x 2 blocks: rows ra + .., columns rb + .. of the
// staged rows; bit 2 m + n of mask: 32 x 32 block (m, n) is wanted.
template <int E, int MB>
__device__ inline void tile_step(typename Op<E>::Acc (&c)[Op<E>::NACC * MB], const char* lds, int plane, int lane, int ra,
                                 int rb, int mask) {
  constexpr int RB = LDS_ROW_BYTES<E>;
  const char* la = lds + ra * RB;
  const char* lb = lds + rb * RB;
  if constexpr (E == E_F64) {
    const int g = lane >> 4, r = lane & 15;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      // lane group g takes K values 4 g + 2 t, 4 g + 2 t + 1
      const int at = lds_at<E>(r, 2 * g + t);
      double2 a[2 * MB], b[4];
#pragma unroll
      for (int m = 0; m < 2 * MB; ++m) a[m] = *(const double2*)(la + at + 16 * m * RB);
#pragma unroll
      for (int n = 0; n < 4; ++n) b[n] = *(const double2*)(lb + at + 16 * n * RB);
#pragma unroll
      for (int m = 0; m < 2 * MB; ++m)
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          if ((mask >> (2 * (m >> 1) + (n >> 1))) & 1) {
            c[4 * m + n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m].x, b[n].x, c[4 * m + n], 0, 0, 0);
            c[4 * m + n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m].y, b[n].y, c[4 * m + n], 0, 0, 0);
          }
        }
    }
  } else {
    constexpr int NP = E == E_F32 ? 3 : 1, NT = E == E_F32 ? 2 : 4;
    const int half = lane >> 5, r = lane & 31;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int at = lds_at<E>(r, E == E_BF16 ? t + 4 * half : 2 * t + half);
      bf16x8_t a[MB][NP], b[2][NP];
#pragma unroll
      for (int p = 0; p < NP; ++p) {
#pragma unroll
        for (int m = 0; m < MB; ++m) a[m][p] = *(const bf16x8_t*)(la + at + p * plane + 32 * m * RB);
#pragma unroll
        for (int n = 0; n < 2; ++n) b[n][p] = *(const bf16x8_t*)(lb + at + p * plane + 32 * n * RB);
      }
#pragma unroll
      for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
          if ((mask >> (2 * m + n)) & 1) {
            f32x16_t& big = c[2 * m + n];
            if constexpr (E == E_F32) {
              f32x16_t& low = c[2 * MB + 2 * m + n];
              low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m][2], b[n][0], low, 0, 0, 0);
              low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m][0], b[n][2], low, 0, 0, 0);
              low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m][1], b[n][1], low, 0, 0, 0);
              low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m][1], b[n][0], low, 0, 0, 0);
              low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m][0], b[n][1], low, 0, 0, 0);
            }
            big = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m][0], b[n][0], big, 0, 0, 0);
          }
    }
  }
}

// (ti, tj <= ti) of lower-triangle position t = ti (ti + 1) / 2 + tj.
__device__ inline void tri_at(int t, int& ti, int& tj) {
  int i = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  while (i * (i + 1) / 2 > t) --i;
  ti = i;
  tj = t - i * (i + 1) / 2;
}

template <int E, bool GATHER, int NG>
__global__ void __launch_bounds__(256, NG == GROUPS_THIN ? 4 : 2) gram_tile_kernel(GramArgs g) {
  typedef Op<E> O;
  typedef typename O::T T;
  typedef typename O::Out Out;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int plane = NG * GROUP * 64;           // float32: bytes of one part's rows
  constexpr int MB = NG == GROUPS_THIN ? 1 : 2;    // block rows of a wave
  constexpr int NACC = O::NACC * MB;
  constexpr bool GEN = NG == GROUPS_THIN && E == E_F32;   // the sketch is made here
  const T* X = (const T*)g.X;
  const T* Om = (const T*)g.omegaT;

  // workgroup -> (split, tile): the workgroups of one XCD (ids equal modulo 8)
  // take consecutive (split, tile) pairs
  const int per = (g.ntiles * g.splits) >> 3, spare = (g.ntiles * g.splits) & 7, xcd = blockIdx.x & 7;
  const int id = xcd * per + (xcd < spare ? xcd : spare) + (int)(blockIdx.x >> 3);
  const int split = id / g.ntiles, tile = id % g.ntiles;

  // the tile's groups: first row and rows that exist (<= 0: not staged), and
  // whether they are sketch rows
  int grow[NG], gn[NG];
  bool gom[NG];
  // this wave's role: staged rows of its operands, first row and column of its
  // output (row in the sketch for a W block), wanted blocks
  const int lane = threadIdx.x & 63;
  const int wave = (int)__builtin_amdgcn_readfirstlane((threadIdx.x >> 6) + split) & 3;
  int ra, rb, row0, col0, nrow, mask = 0;
  bool is_w, diag = false;
  const int I = (int)g.I, S = g.S;
  if constexpr (NG == GROUPS_THIN) {
    grow[0] = 0; gn[0] = I; gom[0] = false;
    grow[1] = 0; gn[1] = GEN ? 0 : S; gom[1] = true;
    is_w = wave >= 2;
    ra = 32 * wave;
    rb = 0;
    row0 = 32 * (wave & 1);
    col0 = 0;
    diag = !is_w;
    nrow = is_w ? S : I;
  } else {
    is_w = tile >= g.ntri;
    if (!is_w) {
      int ti, tj;
      tri_at(tile, ti, tj);
      diag = ti == tj;
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        grow[i] = (i < 2 ? ti : tj) * 128 + (i & 1) * 64;
        gn[i] = i < 2 ? I - grow[i] : (i < 4 && !diag) ? 64 : 0;
        gom[i] = false;
      }
      ra = (wave >> 1) * 64;
      rb = (diag ? 0 : 128) + (wave & 1) * 64;
      row0 = ti * 128 + (wave >> 1) * 64;
      col0 = tj * 128 + (wave & 1) * 64;
      nrow = I;
    } else {
      const int w = tile - g.ntri, sg = w / g.nw, cg = w % g.nw;
#pragma unroll
      for (int i = 0; i < NG; ++i) {
        grow[i] = i == 0 ? sg * 64 : cg * 256 + (i - 1) * 64;
        gn[i] = (i == 0 ? S : I) - grow[i];
        gom[i] = i == 0;
      }
      ra = 0;
      rb = 64 + 64 * wave;
      row0 = sg * 64;
      col0 = cg * 256 + 64 * wave;
      nrow = S;
    }
  }
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int r = row0 + 32 * m, c = col0 + 32 * n;
      if (r < nrow && c < I && (is_w || r >= c)) mask |= 1 << (2 * m + n);
    }

  // row pointers at K offset 0 (rows past the end repeat the last one: their
  // products are not wanted)
  const T* p[NG][2];
  uint32_t rbyte[NG];
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    const int last = gn[i] < GROUP ? gn[i] - 1 : GROUP - 1;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = (int)(threadIdx.x >> 3) + 32 * j;
      p[i][j] = (gom[i] ? Om : X) + (grow[i] + (r < last ? r : last)) * (gom[i] ? g.J : g.B) + (threadIdx.x & 7) * O::EPC;
    }
    const int r = (int)(threadIdx.x & 63);
    rbyte[i] = (uint32_t)(grow[i] + (r < last ? r : last)) * (uint32_t)g.B * (uint32_t)sizeof(T);
  }
  // GATHER: K value k of a tile is (a0 + k / B, k % B); nk of them
  int64_t koff[GATHER ? O::KT / 4 : 1];
  const int nk = GATHER ? (int)(g.nbt * g.B) : O::KT;
  if constexpr (GATHER) {
    const int k0 = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (O::KT / 4);
#pragma unroll
    for (int k = 0; k < O::KT / 4; ++k) koff[k] = (int64_t)((k0 + k) / (int)g.B) * g.I * g.B + (k0 + k) % (int)g.B;
  }

  const int64_t kt0 = (int64_t)split * g.nkt / g.splits;
  const int64_t kt1 = (int64_t)(split + 1) * g.nkt / g.splits;
  Piece st[NG];
  auto load = [&](const KTile& t) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      if (gn[i] <= 0) continue;
      if constexpr (E == E_BF16 && !GATHER) {
        if (t.hi < O::KT) {
          load_rows_end(st[i], p[i], gom[i] ? t.o : t.x, t.hi);
          continue;
        }
      }
      if (GATHER && !gom[i]) load_gather<E>(st[i], X, rbyte[i], koff, t.x, nk);
      else load_rows<E>(st[i], p[i], gom[i] ? t.o : t.x);
    }
  };
  // K tile kt: slab a from b0 on (GATHER: g.nbt values of a from a on).  The
  // last tile of a slab (of the mode) is moved back to end with it, its values
  // that the tile before holds zeroed; in bfloat16 it stays, with zeros past the end.  GATHER: the up to B - 1 sketch values
  // past nk are read (at the very end of Omega^T from the workspace behind it)
  // and zeroed.
  int64_t a, b0 = 0;
  if (GATHER) {
    a = kt0 * g.nbt;
  } else {
    a = kt0 / g.nbt;
    b0 = (kt0 - a * g.nbt) * O::KT;
  }
  auto tile_now = [&]() {
    KTile k;
    const int64_t at = GATHER ? a : b0, end = GATHER ? g.A - g.nbt : g.B - O::KT;
    const int64_t from = at < end || (E == E_BF16 && !GATHER) ? at : end;
    k.lo = (int)(at - from) * (GATHER ? (int)g.B : 1);
    k.hi = E == E_BF16 && !GATHER && at > end ? (int)(g.B - at) : nk;
    k.x = GATHER ? from * g.I * g.B : a * g.I * g.B + from;
    k.o = GATHER ? from * g.B : a * g.B + from;
    return k;
  };
  auto advance = [&]() {
    if (GATHER) {
      a += g.nbt;
    } else {
      b0 += O::KT;
      if (b0 >= g.B) {
        b0 = 0;
        ++a;
      }
    }
  };

  typename O::Acc acc[NACC];
#pragma unroll
  for (int i = 0; i < NACC; ++i)
#pragma unroll
    for (int v = 0; v < (E == E_F64 ? 4 : 16); ++v) acc[i][v] = 0;

  // (the pairs start at another wave from split to split: there may be fewer than
  // threads, and the waves of a SIMD would all have them)
  const int stid = (int)(threadIdx.x + 64 * (split >> 3)) & 255;
  KTile now = {};
  if (kt0 < kt1) {
    now = tile_now();
    load(now);
  }
  for (int64_t kt = kt0; kt < kt1; ++kt) {
#pragma unroll
    for (int i = 0; i < NG; ++i) {
      if (gn[i] <= 0) continue;
      if (GATHER && !gom[i]) store_piece<E, true>(st[i], lds, plane, i * GROUP, now);
      else store_piece<E, false>(st[i], lds, plane, i * GROUP, now);
    }
    if constexpr (GEN) store_sketch(g, lds, plane, now.o, stid);
    __syncthreads();
    if (kt + 1 < kt1) {
      advance();
      now = tile_now();
      load(now);
    }
    if (mask) tile_step<E, MB>(acc, lds, plane, lane, ra, rb, mask);
    __syncthreads();
  }

  // the wanted blocks, [block][32][32]: C's lower triangle of blocks, then W^T
  const int nb = (I + BLK - 1) / BLK;
  Out* part = (Out*)g.partial + (int64_t)split * g.blocks * (BLK * BLK);
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      if (!((mask >> (2 * m + n)) & 1)) continue;
      const int bi = row0 / BLK + m, bj = col0 / BLK + n;
      Out* out = part + (int64_t)(is_w ? nb * (nb + 1) / 2 + bi * nb + bj : bi * (bi + 1) / 2 + bj) * (BLK * BLK);
      if constexpr (E == E_F64) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            out[((i >> 1) * 16 + 4 * v + (lane >> 4)) * BLK + (i & 1) * 16 + (lane & 15)] =
                acc[4 * (2 * m + (i >> 1)) + 2 * n + (i & 1)][v];
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          out[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * BLK + (lane & 31)] =
              E == E_F32 ? acc[2 * m + n][v] + acc[(2 * MB + 2 * m + n) % NACC][v] : acc[2 * m + n][v];
      }
    }
}

// The wide form of float32: tiles of 256 x 256 of C, eight waves of 2 x 4 blocks,
// K tiles of 16 values.  A diagonal tile has work for six waves and its rows for
// four staging waves, so it forms the first 64 sketch rows by its 256 columns
// too; sketch rows from 64 on have tiles of 128 rows x 384 columns.  Wave w loads,
// splits and stores the 64 rows of staged group w.  A block's six part products of
// a K tile are accumulated from zero and then added to its sum, so one accumulator
// serves, a sum is rounded once per 16 K values, and the part products are rounded
// at their own magnitude.
//
// A 128 x 128 tile stages 256 rows for 16 blocks and its two barriers a K tile keep
// loads, splitting and products apart; here it is 512 rows for 64 blocks, with one
// barrier, three LDS buffers and the two waves of a SIMD in opposite phases.
// Measured per mode: 1000^3, S = 60, 7.3 ms (12.9 with the 128-row tiles, 20.2 on
// the float32 MFMA): 1.07 PFLOP/s of bfloat16 products, where an 8192^3 bfloat16
// matrix product of the vendor's library reaches 1.19; the clock falls to 1.7 GHz
// under it (power), so fewer cycles on the vector unit change nothing there.
// 400^3, S = 30, 0.31 ms (0.41, 1.12).
constexpr int WIDE_K = 16, WIDE_GROUPS = 8, WIDE_WROWS = 128, WIDE_WCOLS = 384;
// LDS: [buffer][part][half of the K tile][row][16 bytes]; the pad puts the two
// halves of a row on different banks (a wave writes both at once)
constexpr int WIDE_HALF = WIDE_GROUPS * GROUP * 16 + 128;
constexpr int WIDE_PLANE = 2 * WIDE_HALF, WIDE_BUF = 3 * WIDE_PLANE;

template <bool GATHER>
__global__ void __launch_bounds__(512, 2) gram_wide_kernel(GramArgs g) {
  __shared__ __attribute__((aligned(16))) char lds[3 * WIDE_BUF];
  const int per = (g.ntiles * g.splits) >> 3, spare = (g.ntiles * g.splits) & 7, xcd = blockIdx.x & 7;
  const int id = xcd * per + (xcd < spare ? xcd : spare) + (int)(blockIdx.x >> 3);
  const int split = id / g.ntiles, tile = id % g.ntiles;
  int lane = threadIdx.x & 63;
  const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int I = (int)g.I, S = g.S;

  // this wave's staged group (first row, rows that exist, sketch or mode) and
  // blocks (staged rows of the operands, first row and column of the output;
  // live: whether any is wanted).  Waves w and w + 4 share a SIMD: of a diagonal
  // tile (64-row, 128-column) (0, 0) and (1, 0); (2, 0) and the sketch's first 128
  // columns; (3, 0) and its other 128; (2, 1) and (3, 1).
  int grow, gn, ra, rb, row0, col0;
  bool gom = false, is_w = tile >= g.ntri, live;
  if (!is_w) {
    int ti, tj;
    tri_at(tile, ti, tj);
    const bool diag = ti == tj;
    const int r = (0x31012320 >> (4 * wave)) & 3, c = (0xE8 >> wave) & 1;
    gom = diag && wave == 4;
    grow = gom ? 0 : (wave < 4 ? ti : tj) * 256 + (wave & 3) * 64;
    gn = gom ? S : wave < 4 || !diag ? I - grow : 0;
    ra = r * 64;
    rb = (diag ? 0 : 256) + c * 128;
    row0 = ti * 256 + r * 64;
    col0 = tj * 256 + c * 128;
    live = row0 < I;
    if (diag && (wave == 5 || wave == 6)) {
      is_w = true;
      ra = 256;
      rb = (wave - 5) * 128;
      row0 = 0;
      col0 = tj * 256 + rb;
      live = S > 0 && col0 < I;
    }
  } else {
    const int w = tile - g.ntri, sg = w / g.nw, cg = w % g.nw;
    gom = wave < 2;
    grow = gom ? GROUP + sg * WIDE_WROWS + wave * 64 : cg * WIDE_WCOLS + (wave - 2) * 64;
    gn = (gom ? S : I) - grow;
    ra = (wave & 1) * 64;
    rb = 128 + (wave >> 1) * 128;
    row0 = GROUP + sg * WIDE_WROWS + ra;
    col0 = cg * WIDE_WCOLS + (wave >> 1) * 128;
    live = wave < 6 && row0 < S && col0 < I;
  }

  // staging: 16-byte pieces of rows lane / 4 + 16 j, or (GATHER, mode rows) 16
  // values of row lane.  Rows past the end repeat the last one: their products
  // are not wanted.  (A row, of more than 128 in a tensor that fits the card, is
  // below 4 GB.)
  const int last = gn < GROUP ? gn - 1 : GROUP - 1;
  const uint32_t stride = (uint32_t)((gom ? g.J : g.B) * 4);
  const char* base = (const char*)(gom ? g.omegaT : g.X) + (int64_t)grow * stride;
  const int nk = GATHER ? (int)(g.nbt * g.B) : WIDE_K;
  const bool gat = GATHER && !gom;
  const int64_t kt0 = (int64_t)split * g.nkt / g.splits, kt1 = (int64_t)(split + 1) * g.nkt / g.splits;

  uint32_t st[16];
  int lo = 0;                      // values of st from which on they count
  int64_t a, b0 = 0;
  if (GATHER) {
    a = kt0 * g.nbt;
  } else {
    a = kt0 / g.nbt;
    b0 = (kt0 - a * g.nbt) * WIDE_K;
  }
  // load the K tile (a, b0) and step to the next
  auto load = [&]() {
    const int64_t at = GATHER ? a : b0, end = GATHER ? g.A - g.nbt : g.B - WIDE_K;
    const int64_t from = at < end ? at : end;
    lo = (int)(at - from) * (GATHER ? (int)g.B : 1);
    const int64_t xoff = (GATHER ? from * g.I * g.B : a * g.I * g.B + from) * 4;
    const int64_t ooff = (GATHER ? from * g.B : a * g.B + from) * 4;
    asm volatile("" : "+v"(lane));   // addresses are formed anew each time: registers are short
    if (gn > 0) {
      if (gat) {
        const char* p = base + xoff;
        const uint32_t rbyte = (uint32_t)(lane < last ? lane : last) * stride;
        int b = 0;
#pragma unroll
        for (int k = 0; k < WIDE_K; ++k) {
          st[k] = k < nk ? *(const uint32_t*)(p + rbyte) : 0u;
          // (the next K value: the next b, or the next a)
          const bool wrap = ++b == (int)g.B;
          p += wrap ? (g.I * g.B - g.B + 1) * 4 : 4;
          b = wrap ? 0 : b;
        }
      } else {
        const char* p = base + (gom ? ooff : xoff) + (lane & 3) * 16;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int r = (lane >> 2) + 16 * j;
          const u32x4u_t v = *(const u32x4u_t*)(p + (uint64_t)(uint32_t)(r < last ? r : last) * stride);
          st[4 * j] = v.x; st[4 * j + 1] = v.y; st[4 * j + 2] = v.z; st[4 * j + 3] = v.w;
        }
      }
    }
    if (GATHER) {
      a += g.nbt;
    } else {
      b0 += WIDE_K;
      if (b0 >= g.B) {
        b0 = 0;
        ++a;
      }
    }
  };
  auto store = [&](char* buf) {
    if (gn <= 0) return;
    if (lo > 0 || nk < WIDE_K) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int k = gat ? i : (lane & 3) * 4 + (i & 3);
        if (k < lo || k >= nk) st[i] = 0;
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      uint32_t h[4], m[4], l[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        split3(__uint_as_float(st[8 * j + 2 * i]), __uint_as_float(st[8 * j + 2 * i + 1]), h[i], m[i], l[i]);
      if (gat) {
        char* d = buf + j * WIDE_HALF + (wave * GROUP + lane) * 16;
        *(uint4*)d = make_uint4(h[0], h[1], h[2], h[3]);
        *(uint4*)(d + WIDE_PLANE) = make_uint4(m[0], m[1], m[2], m[3]);
        *(uint4*)(d + 2 * WIDE_PLANE) = make_uint4(l[0], l[1], l[2], l[3]);
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          char* d = buf + ((lane >> 1) & 1) * WIDE_HALF + (wave * GROUP + (lane >> 2) + 16 * (2 * j + i)) * 16 + (lane & 1) * 8;
          *(uint2*)d = make_uint2(h[2 * i], h[2 * i + 1]);
          *(uint2*)(d + WIDE_PLANE) = make_uint2(m[2 * i], m[2 * i + 1]);
          *(uint2*)(d + 2 * WIDE_PLANE) = make_uint2(l[2 * i], l[2 * i + 1]);
        }
      }
    }
  };

  f32x16_t acc[2][4];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[m][n][v] = 0;
  // operands: x of the wave's rows, y of 32 columns at a time (the next 32 read
  // while these are used)
  bf16x8_t x[2][3], y[2][3];
  const int frag = (lane >> 5) * WIDE_HALF + (lane & 31) * 16;
  const int fa = frag + ra * 16, fb = frag + rb * 16;
  auto read_x = [&](const char* buf) {
#pragma unroll
    for (int q = 2; q >= 0; --q)
#pragma unroll
      for (int m = 0; m < 2; ++m) x[m][q] = *(const bf16x8_t*)(buf + fa + m * 512 + q * WIDE_PLANE);
  };
  auto read_y = [&](const char* buf, int n) {
#pragma unroll
    for (int q = 0; q < 3; ++q) y[n & 1][q] = *(const bf16x8_t*)(buf + fb + n * 512 + q * WIDE_PLANE);
  };
  auto products = [&](const char* buf, const char* ahead) {
    f32x16_t t[2];
    // the sum of the block before, a quarter between two products, so that it
    // runs beside them (the order as written: the compiler would gather them)
    auto add = [&](int blk, int quarter) {
      if (blk < 0) return;
#pragma unroll
      for (int v = 4 * quarter; v < 4 * quarter + 4; ++v) acc[blk & 1][blk >> 1][v] += t[blk & 1][v];
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int blk = 0; blk < 8; ++blk) {
      const int n = blk >> 1, m = blk & 1;
      if (m == 0 && n < 3) read_y(buf, n + 1);
      const bf16x8_t(&c)[3] = y[n & 1];
#pragma unroll
      for (int v = 0; v < 16; ++v) t[m][v] = 0;
      t[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[m][2], c[0], t[m], 0, 0, 0);
      t[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[m][0], c[2], t[m], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      add(blk - 1, 0);
      t[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[m][1], c[1], t[m], 0, 0, 0);
      add(blk - 1, 1);
      t[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[m][1], c[0], t[m], 0, 0, 0);
      add(blk - 1, 2);
      t[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[m][0], c[1], t[m], 0, 0, 0);
      add(blk - 1, 3);
      t[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[m][0], c[0], t[m], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    read_x(ahead);
    read_y(ahead, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) add(7, q);
  };

  // K tile kt is formed from one buffer while kt + 2 is put into another and
  // kt + 3 is on its way; kt + 1 is complete, so its first operands are read
  // before the barrier.  Of the two waves of a SIMD one splits and stores before
  // its products and one after them, so that the matrix core and the vector unit
  // work at the same time.
  const int64_t nt = kt1 - kt0;
  if (nt > 0) {
    load();
    store(lds);
    if (nt > 1) {
      load();
      store(lds + WIDE_BUF);
    }
    if (nt > 2) load();
  }
  __syncthreads();
  read_x(lds);
  read_y(lds, 0);
  int cur = 0;
  for (int64_t kt = 0; kt < nt; ++kt) {
    const int ahead = cur == 2 * WIDE_BUF ? 0 : cur + WIDE_BUF;
    const int next = ahead == 2 * WIDE_BUF ? 0 : ahead + WIDE_BUF;
    auto stage = [&]() {
      if (kt + 2 < nt) store(lds + next);
      if (kt + 3 < nt) load();
    };
    if (wave < 4) stage();
    if (live) products(lds + cur, lds + ahead);
    if (wave >= 4) stage();
    __syncthreads();
    cur = ahead;
  }

  if (!live) return;
  const int nb = (I + BLK - 1) / BLK;
  float* part = (float*)g.partial + (int64_t)split * g.blocks * (BLK * BLK);
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const int r = row0 + 32 * m, c = col0 + 32 * n;
      if (r >= (is_w ? S : I) || c >= I || (!is_w && r < c)) continue;
      const int bi = r / BLK, bj = c / BLK;
      float* out = part + (int64_t)(is_w ? nb * (nb + 1) / 2 + bi * nb + bj : bi * (bi + 1) / 2 + bj) * (BLK * BLK);
#pragma unroll
      for (int v = 0; v < 16; ++v) out[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * BLK + (lane & 31)] = acc[m][n][v];
    }
}

// The flat form of float64, for modes of 65 to 256 rows: a workgroup of eight waves
// stages every row of the mode and of the sketch (at most five groups of 64) and forms
// a share of all the wanted blocks, up to four a wave, dealt out evenly, so that the
// SIMDs stay level (in 128-row tiles a wave has 0 to 4 blocks) and each row is staged
// once or twice instead of three times.  Two LDS buffers, one barrier a K tile.
// Measured: 200^3, S = 15, 71 us (110 in 128-row tiles), 40 TFLOP/s of wanted blocks,
// where an 8192^3 product of the vendor's library reaches 71: the rest is the first
// loads, 37 MB of partial sums and the shares' unevenness (18 and 17 blocks).  Whole pass with
// the reduction, us (128-row tiles): 72^3 17 (18), 128^3 25 (32), 160^3 41 (62), 256^3
// 133 (172); S = 60: 128^3 33 (35), 256^3 158 (179).
constexpr int FLAT_GROUPS = 5, FLAT_BLOCKS = 4;
constexpr int FLAT_BUF = FLAT_GROUPS * Op<E_F64>::GROUP_BYTES;

template <bool GATHER>
__global__ void __launch_bounds__(512, 2) gram_flat_kernel(GramArgs g) {
  constexpr int E = E_F64, KT = Op<E>::KT;
  __shared__ __attribute__((aligned(16))) char lds[2 * FLAT_BUF];
  const int per = (g.ntiles * g.splits) >> 3, spare = (g.ntiles * g.splits) & 7, xcd = blockIdx.x & 7;
  const int id = xcd * per + (xcd < spare ? xcd : spare) + (int)(blockIdx.x >> 3);
  const int split = id / g.ntiles, share = id % g.ntiles;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  const int I = (int)g.I, S = g.S;
  const int xg = (I + GROUP - 1) / GROUP, ng = xg + (S > 0 ? 1 : 0);   // groups: the mode's, the sketch

  // this wave's blocks: share + ntiles (wave + 8 i) of the wanted ones; their staged
  // rows, and which of their 16 x 16 quarters have a wanted entry (bit 2 m + n)
  const int nb = (I + BLK - 1) / BLK, ntri = nb * (nb + 1) / 2;
  int blk[FLAT_BLOCKS], ra[FLAT_BLOCKS], rb[FLAT_BLOCKS], mask[FLAT_BLOCKS];
#pragma unroll
  for (int i = 0; i < FLAT_BLOCKS; ++i) {
    blk[i] = share + g.ntiles * (wave + 8 * i);
    int bi = 0, bj = 0;
    const bool w = blk[i] >= ntri;
    if (w) {
      bi = (blk[i] - ntri) / nb;
      bj = (blk[i] - ntri) % nb;
    } else {
      tri_at(blk[i], bi, bj);
    }
    ra[i] = (w ? xg * GROUP : 0) + 32 * bi;
    rb[i] = 32 * bj;
    mask[i] = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (blk[i] < g.blocks && 32 * bi + 16 * (q >> 1) < (w ? S : I) && 32 * bj + 16 * (q & 1) < I &&
          (w || bi > bj || (q >> 1) >= (q & 1)))
        mask[i] |= 1 << q;
  }

  // staging: 16-byte piece tid % 8 of row tid / 8 of every group, or (GATHER, mode
  // rows) K values 2 wave, 2 wave + 1 of row lane; rows past the end repeat the last
  const int nk = GATHER ? (int)(g.nbt * g.B) : KT;
  const double* p[FLAT_GROUPS];
  uint32_t rbyte[FLAT_GROUPS];
  double2 st[FLAT_GROUPS];
#pragma unroll
  for (int i = 0; i < FLAT_GROUPS; ++i) {
    const bool om = i == xg;
    const int first = om ? 0 : i * GROUP, last = (om ? S : I) - 1;
    const int r = first + (tid >> 3), rg = first + lane;
    p[i] = (const double*)(om ? g.omegaT : g.X) + (r < last ? r : last) * (om ? g.J : g.B) + (tid & 7) * 2;
    rbyte[i] = (uint32_t)(rg < last ? rg : last) * (uint32_t)g.B * 8u;
  }
  int64_t koff[2] = {0, 0};
  if (GATHER) {
#pragma unroll
    for (int k = 0; k < 2; ++k) koff[k] = (int64_t)((2 * wave + k) / (int)g.B) * g.I * g.B + (2 * wave + k) % (int)g.B;
  }
  const int64_t kt0 = (int64_t)split * g.nkt / g.splits, kt1 = (int64_t)(split + 1) * g.nkt / g.splits;
  int64_t a, b0 = 0;
  if (GATHER) {
    a = kt0 * g.nbt;
  } else {
    a = kt0 / g.nbt;
    b0 = (kt0 - a * g.nbt) * KT;
  }
  int lo = 0;                      // K values of the loaded tile from which on they count
  auto load = [&]() {
    const int64_t at = GATHER ? a : b0, end = GATHER ? g.A - g.nbt : g.B - KT;
    const int64_t from = at < end ? at : end;
    lo = (int)(at - from) * (GATHER ? (int)g.B : 1);
    const int64_t x = GATHER ? from * g.I * g.B : a * g.I * g.B + from, o = GATHER ? from * g.B : a * g.B + from;
#pragma unroll
    for (int i = 0; i < FLAT_GROUPS; ++i) {
      if (i >= ng) continue;
      if (GATHER && i < xg) {
        const double* X = (const double*)g.X + x;
        st[i].x = 2 * wave < nk ? *(const double*)((const char*)(X + koff[0]) + rbyte[i]) : 0.0;
        st[i].y = 2 * wave + 1 < nk ? *(const double*)((const char*)(X + koff[1]) + rbyte[i]) : 0.0;
      } else {
        const u32x4u_t v = *(const u32x4u_t*)(p[i] + (i == xg ? o : x));
        st[i] = __builtin_bit_cast(double2, v);
      }
    }
    if (GATHER) {
      a += g.nbt;
    } else {
      b0 += KT;
      if (b0 >= g.B) {
        b0 = 0;
        ++a;
      }
    }
  };
  auto store = [&](char* buf) {
#pragma unroll
    for (int i = 0; i < FLAT_GROUPS; ++i) {
      if (i >= ng) continue;
      const bool gat = GATHER && i < xg;
      const int row = i * GROUP + (gat ? lane : tid >> 3), q = gat ? wave : tid & 7;
      double2 v = st[i];
      if (lo > 0 || nk < KT) {
        if (2 * q < lo || 2 * q >= nk) v.x = 0.0;
        if (2 * q + 1 < lo || 2 * q + 1 >= nk) v.y = 0.0;
      }
      *(double2*)(buf + lds_at<E>(row, q)) = v;
    }
  };

  f64x4_t acc[FLAT_BLOCKS][4];
#pragma unroll
  for (int i = 0; i < FLAT_BLOCKS; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][q][v] = 0.0;
  const int lg = lane >> 4, li = lane & 15;
  if (kt0 < kt1) {
    load();
    store(lds);
    if (kt0 + 1 < kt1) load();
  }
  __syncthreads();
  for (int64_t kt = kt0; kt < kt1; ++kt) {
    const char* cur = lds + ((kt - kt0) & 1) * FLAT_BUF;
    if (kt + 1 < kt1) store(lds + ((kt - kt0 + 1) & 1) * FLAT_BUF);
    if (kt + 2 < kt1) load();
#pragma unroll
    for (int i = 0; i < FLAT_BLOCKS; ++i) {
      if (!mask[i]) continue;
      double2 x[2][2], y[2][2];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          x[t][m] = *(const double2*)(cur + ra[i] * 128 + lds_at<E>(li, 2 * lg + t) + 16 * m * 128);
          y[t][m] = *(const double2*)(cur + rb[i] * 128 + lds_at<E>(li, 2 * lg + t) + 16 * m * 128);
        }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if ((mask[i] >> q) & 1) {
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            acc[i][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[t][q >> 1].x, y[t][q & 1].x, acc[i][q], 0, 0, 0);
            acc[i][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[t][q >> 1].y, y[t][q & 1].y, acc[i][q], 0, 0, 0);
          }
        }
    }
    __syncthreads();
  }

  double* part = (double*)g.partial + (int64_t)split * g.blocks * (BLK * BLK);
#pragma unroll
  for (int i = 0; i < FLAT_BLOCKS; ++i) {
    if (!mask[i]) continue;
    double* out = part + (int64_t)blk[i] * (BLK * BLK);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) out[(16 * (q >> 1) + 4 * v + lg) * BLK + 16 * (q & 1) + li] = acc[i][q][v];
  }
}

// Modes of a few rows (I and S at most 8: the channels of images and video): bound
// by the read of X and the sketch, which the tiles above, of 64 rows each, spend on
// staging rows that do not exist.  A thread takes V consecutive K values of every
// row straight from memory and keeps all the products in registers; the threads of
// a workgroup add theirs in float64, in which the partial sums stay.  V: 16 bytes (slabs of at least V values), or 1.
// Measured: 3 rows and 3 sketch columns of 25.3 M float32 values, 0.14 ms, 4.3 TB/s
// (1.36 ms).
constexpr int TINY = 8;

template <int E, int N, int V>
__global__ void __launch_bounds__(256) gram_tiny_kernel(GramArgs g) {
  typedef Op<E> O;
  typedef typename O::T T;
  typedef typename O::Out Out;
  typedef T tv __attribute__((ext_vector_type(V), aligned(sizeof(T))));
  constexpr int NC = N * (N + 1) / 2;
  const T* X = (const T*)g.X;
  const T* Om = (const T*)g.omegaT;
  const int I = (int)g.I, S = g.S;
  auto value = [](T v) -> Out {
    if constexpr (E == E_BF16) return __uint_as_float((uint32_t)v << 16);
    else return v;
  };
  Out c[NC], w[N * N];
#pragma unroll
  for (int i = 0; i < NC; ++i) c[i] = 0;
#pragma unroll
  for (int i = 0; i < N * N; ++i) w[i] = 0;

  // chunks of V values, nbt to a slab; consecutive threads take consecutive ones
  const int64_t step = (int64_t)g.splits * 256;
  const int64_t da = step / g.nbt, db = step % g.nbt;
  int64_t kt = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int64_t a = kt / g.nbt, q = kt % g.nbt;
  for (; kt < g.nkt; kt += step) {
    // a slab's last chunk is moved back to end with it, the values that the chunk
    // before holds zeroed
    const int64_t from = q * V < g.B - V ? q * V : g.B - V;
    const int lo = (int)(q * V - from);
    const T* x = X + a * g.I * g.B + from;
    const T* o = Om + a * g.B + from;
    tv xv[N], ov[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      xv[i] = i < I ? *(const tv*)(x + i * g.B) : tv{};
      ov[i] = i < S ? *(const tv*)(o + i * g.J) : tv{};
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
      Out xs[N];
#pragma unroll
      for (int i = 0; i < N; ++i) xs[i] = v < lo ? (Out)0 : value(xv[i][v]);
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) c[i * (i + 1) / 2 + j] += xs[i] * xs[j];
#pragma unroll
      for (int r = 0; r < N; ++r) {
        const Out os = v < lo ? (Out)0 : value(ov[r][v]);
#pragma unroll
        for (int i = 0; i < N; ++i) w[r * N + i] += os * xs[i];
      }
    }
    a += da;
    q += db;
    if (q >= g.nbt) {
      q -= g.nbt;
      ++a;
    }
  }

  __shared__ double sums[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double* part = (double*)g.partial + (int64_t)blockIdx.x * g.blocks * (BLK * BLK);
  auto put = [&](Out v, int at) {
    double d = (double)v;
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) d += __shfl_xor(d, m, 64);
    __syncthreads();
    if (lane == 0) sums[wave] = d;
    __syncthreads();
    if (threadIdx.x == 0) part[at] = (sums[0] + sums[1]) + (sums[2] + sums[3]);
  };
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j <= i; ++j)
      if (i < I) put(c[i * (i + 1) / 2 + j], i * BLK + j);
#pragma unroll
  for (int r = 0; r < N; ++r)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (r < S && i < I) put(w[r * N + i], BLK * BLK + r * BLK + i);
}

// Sum the split-K partials in a fixed order: C (I x I, both triangles) and
// W^T (S x I), float64.  64 consecutive values of a block per workgroup, the
// splits dealt to 16 groups of lanes whose sums are added in order, so that a
// few thousand outputs (a thin mode with hundreds of splits) still fill the
// chip.  A launch has fewer than 2^32 threads, which modes of 23000 rows and more
// would pass with a workgroup for every 64 values: at most RED_GRID workgroups, which
// then take several.
constexpr int RED_GROUPS = 16;
constexpr int64_t RED_GRID = 1 << 20;
template <class Out>
__global__ void __launch_bounds__(64 * RED_GROUPS) gram_reduce_kernel(GramArgs g, double* C, double* Wt) {
  __shared__ double sums[RED_GROUPS][64];
  const int l = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int64_t stride = (int64_t)g.blocks * (BLK * BLK);
  const int nb = (int)ceil_div(g.I, BLK), ntri = nb * (nb + 1) / 2;
  for (int64_t e0 = (int64_t)blockIdx.x * 64; e0 < stride; e0 += (int64_t)gridDim.x * 64) {
    const int64_t e = e0 + l;
    const Out* P = (const Out*)g.partial + e;
    double acc = 0.0;
#pragma unroll 4
    for (int sp = grp; sp < g.splits; sp += RED_GROUPS) acc += (double)P[sp * stride];
    sums[grp][l] = acc;
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int i = 1; i < RED_GROUPS; ++i) acc += sums[i][l];
      const int blk = (int)(e / (BLK * BLK)), at = (int)(e % (BLK * BLK));
      int bi, bj;
      if (blk < ntri) tri_at(blk, bi, bj);
      else {
        bi = (blk - ntri) / nb;
        bj = (blk - ntri) % nb;
      }
      const int64_t i = bi * BLK + at / BLK, j = bj * BLK + at % BLK;
      if (blk >= ntri) {
        if (i < g.S && j < g.I) Wt[i * g.I + j] = acc;
      } else if (i < g.I && j <= i) {
        C[i * g.I + j] = acc;
        C[j * g.I + i] = acc;
      }
    }
    __syncthreads();               // sums is written again
  }
}

// Omega^T (S x J) in the element type of the product.
template <int E>
__global__ void omega_kernel(uint64_t seed, uint32_t mode, int64_t total, void* out) {
  const int64_t npairs = (total + 1) / 2;
  for (int64_t m = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; m < npairs;
       m += (int64_t)gridDim.x * blockDim.x) {
    const int64_t L = 2 * m;
    if (E == E_F64) {
      double z0, z1;
      gauss_pair_f64((uint64_t)m, mode, 0u, seed, z0, z1);
      double* o = (double*)out;
      o[L] = z0;
      if (L + 1 < total) o[L + 1] = z1;
    } else {
      float z0, z1;
      if (E == E_F32) gauss_pair_f32((uint64_t)m, mode, 0u, seed, z0, z1);
      else gauss_pair_bf16((uint64_t)m, mode, 0u, seed, z0, z1);
      if (E == E_F32) {
        float* o = (float*)out;
        o[L] = z0;
        if (L + 1 < total) o[L + 1] = z1;
      } else if (E == E_BF16) {
        bf16_t* o = (bf16_t*)out;
        o[L] = f32_to_bf16(z0);
        if (L + 1 < total) o[L + 1] = f32_to_bf16(z1);
      } else {
        fp8_t* o = (fp8_t*)out;
        o[L] = f32_to_e4m3(z0);
        if (L + 1 < total) o[L + 1] = f32_to_e4m3(z1);
      }
    }
  }
}

__global__ void philox_kernel(const uint32_t* ctr, int64_t count, uint64_t seed, uint32_t* out) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x) {
    PhiloxOut o = philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3],
                                (uint32_t)seed, (uint32_t)(seed >> 32));
    out[4 * i] = o.w0;
    out[4 * i + 1] = o.w1;
    out[4 * i + 2] = o.w2;
    out[4 * i + 3] = o.w3;
  }
}

}  // namespace

// ------------------------------------------------------------------ planning

int elem_size(int elem) { return elem == E_F64 ? 8 : elem == E_F32 ? 4 : elem == E_BF16 ? 2 : 1; }

static int gram_kt(int elem) { return elem == E_F64 ? Op<E_F64>::KT : elem == E_F32 ? Op<E_F32>::KT : Op<E_BF16>::KT; }

// Two slices per compute unit of 128 x 128 tiles of the rows and the sketch, each of
// at least 8 K tiles: the slices of the bfloat16 form (64^3, three modes: 382 us a call
// against 356 with slices by cost as below, whose sums have another order), and what
// bounds the others' partials.
static int64_t slices(int elem, int64_t A, int64_t I, int64_t B, int S, int cu_count, int64_t& tiles) {
  const int64_t nt = ceil_div(I, 128);
  const bool thin = elem == E_F32 && I <= 64 && S >= 1 && S <= 64;
  tiles = thin ? 1 : nt * (nt + 1) / 2 + nt * ceil_div(S, 128);
  const int kt = gram_kt(elem);
  const int64_t nkt = B > 1 ? A * ceil_div(B, kt) : ceil_div(A, kt);
  int64_t splits = std::min(std::max<int64_t>(ceil_div(2 * (int64_t)cu_count, tiles), 1), std::max<int64_t>(nkt / 8, 1));
  if (splits >= 8) splits = (splits + 7) / 8 * 8;
  return std::min(splits, std::max<int64_t>(nkt, 1));
}

// The most bytes that the partials may take.
static size_t partial_limit(int elem, int64_t A, int64_t I, int64_t B, int S, int cu_count) {
  int64_t tiles;
  const int64_t splits = slices(elem, A, I, B, S, cu_count, tiles);
  const size_t more = elem == E_F32 && A * I * B >= ((int64_t)1 << 26) ? (size_t)16 << 20 : 0;
  return (size_t)(splits * tiles) * 128 * 128 * (elem == E_F64 ? 8 : 4) + more;
}

GramArgs gram_plan(int elem, int64_t A, int64_t I, int64_t B, int S, int cu_count, int S_scratch, bool any_order) {
  GramArgs g = {};
  g.A = A;
  g.I = I;
  g.B = B;
  g.J = A * B;
  g.S = S;
  g.thin = I <= GROUP && S <= GROUP;
  auto tiles = [&](bool wide) {
    g.wide = wide;
    g.nt = (int)ceil_div(I, wide ? 256 : 128);
    g.ntri = g.nt * (g.nt + 1) / 2;
    g.nw = (int)ceil_div(I, wide ? WIDE_WCOLS : 256);
    const int wrows = wide ? (int)ceil_div(std::max(S - GROUP, 0), WIDE_WROWS) : (int)ceil_div(S, GROUP);
    g.ntiles = g.ntri + wrows * g.nw;
  };
  tiles(true);
  const double wide = g.ntri + 0.6 * (g.ntiles - g.ntri);
  tiles(false);
  if (g.thin) {
    g.ntri = g.ntiles = 1;
    g.gen = elem == E_F32 && S > 0;
  } else if (elem == E_F32 && (B < WIDE_K ? 2.4 * wide + 0.8 : 3.1 * wide + 1.2) < g.ntiles) {
    // The wide form where its tiles take less time than the others' count of
    // their own.  A wide tile takes the time of 2.9 to 3.4 of 128 rows (2.4 where
    // the rows run across the lanes, whose K values the narrow form stages by
    // single words), one of the sketch alone 0.6 of that; over 1.2 (0.8) for the
    // longer pipeline.  Measured (us, wide / 128 rows, S = 15, I^3): 192 36 / 33,
    // 256 67 / 58, 384 252 / 228, 448 424 / 531, 512 580 / 658; last mode 224
    // 52 / 66, 384 268 / 301, 512 643 / 939; 1000^3, S = 60, 7.3 ms / 12.9.
    tiles(true);
  }
  const int nb = (int)ceil_div(I, BLK);
  g.blocks = nb * (nb + 1) / 2 + (int)ceil_div(S, BLK) * nb;
  if (I <= TINY && S <= TINY && (elem != E_BF16 || any_order)) {
    // at least 4 chunks to a thread, at most 4 workgroups to a compute unit
    g.tiny = 1;
    g.gen = 0;
    const int64_t v = B >= 16 / elem_size(elem) ? 16 / elem_size(elem) : 1;
    g.nbt = ceil_div(B, v);
    g.nkt = A * g.nbt;
    const size_t limit = partial_limit(elem, A, I, B, S_scratch < 0 ? S : S_scratch, cu_count);
    const int64_t fit = (int64_t)(limit / ((size_t)g.blocks * BLK * BLK * 8));
    g.splits = (int)std::max<int64_t>(std::min({ceil_div(g.nkt, 4 * 256), 4 * (int64_t)cu_count, fit}), 1);
    return g;
  }
  // (five staged groups; faster than the tiles over that whole range, see there)
  if (elem == E_F64 && !g.thin && I <= 256 && S <= GROUP) {
    g.flat = 1;
    g.ntiles = (int)ceil_div(g.blocks, 8 * FLAT_BLOCKS);
  }
  const int kt = g.wide ? WIDE_K : gram_kt(elem);
  g.gather = B < kt;
  g.nbt = g.gather ? std::min(kt / B, A) : ceil_div(B, kt);
  g.nkt = g.gather ? ceil_div(A, g.nbt) : A * g.nbt;
  if (elem == E_BF16) {
    int64_t tiles128;
    g.splits = (int)slices(elem, A, I, B, S, cu_count, tiles128);
    return g;
  }
  // Splits: a compute unit's share of the workgroups, two at a time (one alone
  // leaves the matrix cores idle between its loads and its products: taken as
  // 1.6 of the time of each of two), times a workgroup's K tiles plus about 6
  // of prologue and epilogue, plus the partials' traffic in K tiles (about
  // 7.5 MB pass in the 1.5 us of one).  The thin form, bound by its loads, is
  // four workgroups to a compute unit.
  const double per = (double)g.blocks * BLK * BLK * (elem == E_F64 ? 16 : 8);
  const size_t limit = partial_limit(elem, A, I, B, S_scratch < 0 ? S : S_scratch, cu_count);
  double best = -1.0;
  g.splits = 1;
  for (int64_t s = 1; s <= std::min<int64_t>(g.nkt, 8 * (int64_t)cu_count); ++s) {
    if (s > 1 && (size_t)s * g.blocks * BLK * BLK * (elem == E_F64 ? 8 : 4) > limit) break;
    const int64_t n = ceil_div(g.ntiles * s, cu_count);
    const double share = g.wide || g.flat ? 1.2 * (double)n : g.thin ? 4.0 * (double)ceil_div(n, 4) : (double)n + (n & 1 ? 0.6 : 0.0);
    const double cost = share * ((double)ceil_div(g.nkt, s) + 6.0) + per * s / 7.5e6;
    if (best < 0 || cost < best) {
      best = cost;
      g.splits = (int)s;
    }
  }
  return g;
}

size_t gram_partial_bytes(const GramArgs& g, int elem) {
  return (size_t)g.splits * g.blocks * BLK * BLK * (elem == E_F64 || g.tiny ? 8 : 4);
}

template <int E, bool GATHER, int NG>
static hipError_t launch_tiles(const GramArgs& g, hipStream_t s) {
  hipLaunchKernelGGL((gram_tile_kernel<E, GATHER, NG>), dim3((unsigned)(g.ntiles * g.splits)), dim3(256),
                     NG * Op<E>::GROUP_BYTES, s, g);
  return hipGetLastError();
}

template <bool GATHER>
static hipError_t launch_wide(const GramArgs& g, hipStream_t s) {
  hipLaunchKernelGGL(gram_wide_kernel<GATHER>, dim3((unsigned)(g.ntiles * g.splits)), dim3(512), 0, s, g);
  return hipGetLastError();
}

template <int E>
static hipError_t launch_tiny(const GramArgs& g, hipStream_t s) {
  constexpr int V = 16 / (int)sizeof(typename Op<E>::T);
  const bool small = g.I <= 4 && g.S <= 4, vec = g.B >= V;
  const dim3 grid(g.splits), block(256);
  if (small && vec) hipLaunchKernelGGL((gram_tiny_kernel<E, 4, V>), grid, block, 0, s, g);
  else if (small) hipLaunchKernelGGL((gram_tiny_kernel<E, 4, 1>), grid, block, 0, s, g);
  else if (vec) hipLaunchKernelGGL((gram_tiny_kernel<E, TINY, V>), grid, block, 0, s, g);
  else hipLaunchKernelGGL((gram_tiny_kernel<E, TINY, 1>), grid, block, 0, s, g);
  return hipGetLastError();
}

template <int E>
static hipError_t launch_gram(const GramArgs& g, hipStream_t s) {
  if (g.tiny) return launch_tiny<E>(g, s);
  if constexpr (E == E_F64)
    if (g.flat) {
      if (g.gather) hipLaunchKernelGGL(gram_flat_kernel<true>, dim3((unsigned)(g.ntiles * g.splits)), dim3(512), 0, s, g);
      else hipLaunchKernelGGL(gram_flat_kernel<false>, dim3((unsigned)(g.ntiles * g.splits)), dim3(512), 0, s, g);
      return hipGetLastError();
    }
  if (g.wide) return g.gather ? launch_wide<true>(g, s) : launch_wide<false>(g, s);
  if (g.thin) return g.gather ? launch_tiles<E, true, GROUPS_THIN>(g, s) : launch_tiles<E, false, GROUPS_THIN>(g, s);
  return g.gather ? launch_tiles<E, true, GROUPS_TILE>(g, s) : launch_tiles<E, false, GROUPS_TILE>(g, s);
}

hipError_t launch_gram_main(int elem, const GramArgs& g, hipStream_t s) {
  switch (elem) {
    case E_F64: return launch_gram<E_F64>(g, s);
    case E_F32: return launch_gram<E_F32>(g, s);
    case E_BF16: return launch_gram<E_BF16>(g, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gram_reduce(int elem, const GramArgs& g, double* C, double* Wt, hipStream_t s) {
  const dim3 grid((unsigned)std::min<int64_t>((int64_t)g.blocks * (BLK * BLK / 64), RED_GRID));
  if (elem == E_F64 || g.tiny) hipLaunchKernelGGL(gram_reduce_kernel<double>, grid, dim3(64 * RED_GROUPS), 0, s, g, C, Wt);
  else hipLaunchKernelGGL(gram_reduce_kernel<float>, grid, dim3(64 * RED_GROUPS), 0, s, g, C, Wt);
  return hipGetLastError();
}

hipError_t launch_omega(int elem, uint64_t seed, int mode, int64_t total, void* out, hipStream_t s) {
  const int64_t npairs = (total + 1) / 2;
  unsigned grid = (unsigned)std::min<int64_t>(ceil_div(npairs, 256), 16384);
  if (grid == 0) return hipSuccess;
  switch (elem) {
    case E_F64: hipLaunchKernelGGL(omega_kernel<E_F64>, dim3(grid), dim3(256), 0, s, seed, (uint32_t)mode, total, out); break;
    case E_F32: hipLaunchKernelGGL(omega_kernel<E_F32>, dim3(grid), dim3(256), 0, s, seed, (uint32_t)mode, total, out); break;
    case E_BF16: hipLaunchKernelGGL(omega_kernel<E_BF16>, dim3(grid), dim3(256), 0, s, seed, (uint32_t)mode, total, out); break;
    default: hipLaunchKernelGGL(omega_kernel<E_FP8>, dim3(grid), dim3(256), 0, s, seed, (uint32_t)mode, total, out); break;
  }
  return hipGetLastError();
}

hipError_t launch_philox(const uint32_t* ctr, int64_t count, uint64_t seed, uint32_t* out, hipStream_t s) {
  unsigned grid = (unsigned)std::min<int64_t>(ceil_div(count, 256), 4096);
  if (grid == 0) return hipSuccess;
  hipLaunchKernelGGL(philox_kernel, dim3(grid), dim3(256), 0, s, ctr, count, seed, out);
  return hipGetLastError();
}

}  // namespace rbki
