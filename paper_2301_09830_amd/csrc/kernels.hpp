// HIP kernels of liboptcc for gfx950 (CDNA4): shared helpers and the small
// kernels common to both rank paths (Q padding, Gram-partial sums, Q
// reduction, stand-alone reconstruction and error update).
//
// Streaming kernels read the error-fed input A = M + err_prev straight from
// HBM (M as bf16 or fp32, err_prev fp32).  Sums run in a fixed order, so
// every result is deterministic and the fused and unfused entry points agree
// bitwise.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "plan.hpp"

namespace occ {

typedef const __attribute__((address_space(4))) float* cfloat_p;
typedef const __attribute__((address_space(4))) double* cdouble_p;

__device__ __forceinline__ cfloat_p as_const(const float* p) { return (cfloat_p)(uintptr_t)p; }
__device__ __forceinline__ cdouble_p as_const(const double* p) { return (cdouble_p)(uintptr_t)p; }

enum { DT_F32 = 0, DT_BF16 = 1 };
enum : uint32_t { FLAG_NONFINITE = 1u, FLAG_RANK_DEFICIENT = 2u, FLAG_BAD_ROWS = 4u };

// Index of this thread's wave in its block, as a wave-uniform (SGPR) value so
// that addresses derived from it qualify for scalar loads.
__device__ __forceinline__ int wave_id() {
  return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// bf16 bit pattern of an fp32 value, rounded to nearest even (NaN stays NaN).
__device__ __forceinline__ uint16_t bf16_rne(float v) {
  return __builtin_bit_cast(uint16_t, (__bf16)v);
}

__device__ __forceinline__ uint32_t bf16_pack2(float lo, float hi) {
  return (uint32_t)bf16_rne(lo) | ((uint32_t)bf16_rne(hi) << 16);
}

// Element (row, col) of M as fp32 (exact widening for bf16).
template <int DT>
__device__ __forceinline__ float m_elem(const Desc& d, int64_t off) {
  if (DT == DT_F32) return ((const float*)d.M)[off];
  const uint16_t h = ((const uint16_t*)d.M)[off];
  return __uint_as_float((uint32_t)h << 16);
}

// Row of M, err and M_hat that holds row `row` (< d.m) of the compressed
// matrix: the same row, or with RM (row-sparse step) the row the validated
// row list names.
template <bool RM>
__device__ __forceinline__ int64_t prow(const Desc& d, int row) {
  if constexpr (RM) return (int64_t)d.rmap[row];
  else return (int64_t)row;
}

// Vector accesses at element alignment.  The hardware takes 16-byte global
// loads and stores at any address that is a multiple of the element size, so
// rows that start at any element use the same instructions as aligned ones
// (measured on a 1 GiB stream: loads at 4-byte alignment 5.1 TB/s, as aligned;
// at 2-byte alignment 4.9 TB/s).  `AL` only states that the address is known
// to be naturally aligned.
typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef float f2u_t __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t u4h_t __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u2h_t __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t u1h_t __attribute__((aligned(2)));

template <bool AL>
__device__ __forceinline__ float4 ld_f4(const float* p) {
  if constexpr (AL) {
    return *(const float4*)p;
  } else {
    const f4u_t v = *(const f4u_t*)p;
    return make_float4(v[0], v[1], v[2], v[3]);
  }
}

// eight / four bf16 elements
template <bool AL>
__device__ __forceinline__ uint4 ld_h8(const uint16_t* p) {
  if constexpr (AL) {
    return *(const uint4*)p;
  } else {
    const u4h_t v = *(const u4h_t*)p;
    return make_uint4(v[0], v[1], v[2], v[3]);
  }
}

template <bool AL>
__device__ __forceinline__ uint2 ld_h4(const uint16_t* p) {
  if constexpr (AL) {
    return *(const uint2*)p;
  } else {
    const u2h_t v = *(const u2h_t*)p;
    return make_uint2(v[0], v[1]);
  }
}

// One value, stored nontemporally or plainly.
template <bool NT, class T>
__device__ __forceinline__ void st_as(T v, T* p) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// Four consecutive elements of an output row.  NT (every output row on
// 64-byte boundaries): nontemporal, since the dirty lines of these streaming
// outputs would otherwise be written back during the next pass.  Other rows:
// plain stores at element alignment, whose partly written lines meet in the
// L2 (16-byte stores along rows 16 bytes off the 64-byte grid: 6.3 TB/s
// plain, 3.1 TB/s nontemporal; on the grid 6.9 and 5.6-5.8).
template <bool NT>
__device__ __forceinline__ void store_f4(float* o, float a, float b, float c, float e) {
  typedef float nt4 __attribute__((ext_vector_type(4)));
  if constexpr (NT) __builtin_nontemporal_store(nt4{a, b, c, e}, (nt4*)o);
  else *(f4u_t*)o = f4u_t{a, b, c, e};
}

// Block -> matrix lookup for batched launches: the last matrix whose first
// block of this kernel kind is <= b.
__device__ __forceinline__ int find_matrix(const Desc* __restrict__ table, int count, int kind,
                                           int b) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (table[mid].blk[kind] <= b) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Dispatch helpers: run BODY(d, local_block) on the matrix owning block B
// of kind KIND (this block, for OCC_DISPATCH).
#define OCC_DISPATCH_AT(KIND, BODY, B)                                  \
  if (count == 1) {                                                     \
    BODY(single, (B));                                                  \
  } else {                                                              \
    const int j_ = find_matrix(table, count, KIND, (B));                \
    const Desc& d_ = table[j_];                                         \
    BODY(d_, (B) - d_.blk[KIND]);                                       \
  }

#define OCC_DISPATCH(KIND, BODY) OCC_DISPATCH_AT(KIND, BODY, (int)blockIdx.x)

#define OCC_KARGS const Desc* __restrict__ table, int count, Desc single

// Tile index of a block of a kernel whose neighbouring tiles share an operand
// slice (the Q columns of a left-product split, the P_hat rows of a
// right-product split or reconstruction row block).  Workgroups are dealt to
// the 8 XCDs round-robin (workgroup b to XCD b % 8), each XCD with its own L2;
// renumbering so that XCD x takes the contiguous tile range
// [x G8 / 8, (x + 1) G8 / 8) (G8 = the grid rounded down to a multiple of 8;
// the last G - G8 blocks keep their index) keeps the tiles that run on one
// XCD on few slices.  A bijection of [0, G): results do not change.
__device__ __forceinline__ int xcd_tile() {
  const int g8 = (int)gridDim.x & ~7, b = (int)blockIdx.x;
  return b < g8 ? (b & 7) * (g8 >> 3) + (b >> 3) : b;
}

#define OCC_DISPATCH_X(KIND, BODY)                                      \
  if (count == 1) {                                                     \
    BODY(single, xcd_tile());                                           \
  } else {                                                              \
    const int v_ = xcd_tile();                                          \
    const int j_ = find_matrix(table, count, KIND, v_);                 \
    const Desc& d_ = table[j_];                                         \
    BODY(d_, v_ - d_.blk[KIND]);                                        \
  }

// gsum[k][l] = sum_b gpart[b][k][l] for k <= l (fixed order), zero below the
// diagonal (the Gram partials hold the upper triangle only).  MODE 1: second
// CholeskyQR pass, skipped unless the first pass asked for it.  A block takes
// GS_ENT entries; GS_SL threads per entry sum interleaved slices of the
// partials with their loads issued in batches of 8, and the slices are added in
// slice order.
constexpr int GS_SL = 8;
constexpr int GS_ENT = kBlock / GS_SL;

template <int RP, int MODE>
__device__ __forceinline__ void gsum_body(const Desc& d, int b) {
  if (MODE == 1 && !d.info[0]) return;
  __shared__ double part[GS_SL][GS_ENT];
  const int sl = threadIdx.x / GS_ENT, el = threadIdx.x % GS_ENT;
  const int idx = b * GS_ENT + el;
  const int k = idx / RP, l = idx % RP;
  const bool upper = idx < RP * RP && k <= l;
  double s = 0.0;
  if (upper) {
    for (int g0 = sl; g0 < d.ng; g0 += 8 * GS_SL) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int g = g0 + GS_SL * u;
        v[u] = (g < d.ng) ? d.gpart[(int64_t)g * RP * RP + idx] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (g0 + GS_SL * u < d.ng) s = (g0 + GS_SL * u == sl) ? v[u] : s + v[u];
    }
  }
  part[sl][el] = s;
  __syncthreads();
  if (sl == 0 && idx < RP * RP) {
    double tot = 0.0;
    if (upper) {
      tot = part[0][el];
      for (int x = 1; x < GS_SL && x < d.ng; ++x) tot += part[x][el];
    }
    d.gsum[idx] = tot;
  }
}

template <int RP, int MODE>
__global__ __launch_bounds__(kBlock) void k_gsum(OCC_KARGS) {
#define B_(d, b) gsum_body<RP, MODE>(d, b)
  OCC_DISPATCH(K_GSUM, B_)
#undef B_
}

// ---------------------------------------------------------------------------
// Pivot rules shared by the Cholesky kernels: a pivot <= kPivotTol * max diag(G)
// marks its column dependent; a second CholeskyQR pass runs when the
// surviving diagonal of the Cholesky factor spans more than kSecondPassCond.
// ---------------------------------------------------------------------------
constexpr double kPivotTol = 1e-12;
constexpr double kSecondPassCond = 1e3;

// ---------------------------------------------------------------------------
// Large-rank path: Q padding (k_qpadl) and the Q reduction (k_qredl) over
// column tiles.  Both write qpad (n_pad x RP) and, when M is bf16, Q as
// two bf16 parts hi = bf16(v), lo = bf16(v - hi) (v - hi - lo is below
// 2^-16 |v|) in qbf, transposed so that the left product stages 32 columns
// of a rank row with 16-byte copies: rank k goes to row (k % NU) * 32 + k / NU,
// NU = RP / 32, the order in which that kernel's lanes read them.  The
// transpose goes through LDS, so each qbf row is written in 16-byte chunks.
// k_qpadl covers all n_pad columns (zeros past n) in 32-column tiles;
// k_qredl sums the row-split partials (fixed order, 16 loads in flight per
// element) for the n real columns, in tiles of d.qr_cols columns (8 or 32),
// and also writes the caller's Q.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint16_t bf16_bits(__bf16 h) { return __builtin_bit_cast(uint16_t, h); }

constexpr int QT_COLS = 32;                 // columns per block, at most

template <int RP>
struct QTSmem {
  uint16_t t[2][RP * QT_COLS];
};

template <int RP, bool REDUCE>
__device__ __forceinline__ void qtile_body(const Desc& d, int b, QTSmem<RP>& sm) {
  constexpr int NU = RP / 32;
  const int QT_P = REDUCE ? d.qr_cols : QT_COLS;   // columns of this tile = LDS pitch (bf16)
  const int QT_CH = QT_P / 8;                      // 16-byte chunks of a transposed rank row
  const int c0 = b * QT_P;
  const int c_end = REDUCE ? d.n : d.n_pad;
  for (int e = threadIdx.x; e < QT_P * RP; e += kBlock) {
    const int c = c0 + e / RP, k = e % RP;
    if (c >= c_end) continue;
    const int64_t idx = (int64_t)c * RP + k;
    float v;
    if (REDUCE) {
      // fixed order; loads issued in batches of 16
      v = 0.f;
      for (int s0 = 0; s0 < d.sq; s0 += 16) {
        float p[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) p[u] = (s0 + u < d.sq) ? d.qpart[(int64_t)(s0 + u) * d.n * RP + idx] : 0.f;
#pragma unroll
        for (int u = 0; u < 16; ++u)
          if (s0 + u < d.sq) v = (s0 + u == 0) ? p[u] : v + p[u];
      }
      if (k < d.r) d.Q[(int64_t)c * d.r + k] = v;
    } else {
      v = (c < d.n && k < d.r) ? d.Q[(int64_t)c * d.r + k] : 0.f;
    }
    d.qpad[idx] = v;
    if (d.qbf) {
      const int prow = (k % NU) * 32 + k / NU;
      const __bf16 hi = (__bf16)v;
      sm.t[0][prow * QT_P + (c - c0)] = bf16_bits(hi);
      sm.t[1][prow * QT_P + (c - c0)] = bf16_bits((__bf16)(v - (float)hi));
    }
  }
  if (!d.qbf) return;
  __syncthreads();
  // 2 x RP rows of QT_COLS columns, QT_CH 16-byte chunks each
  for (int f = threadIdx.x; f < 2 * RP * QT_CH; f += kBlock) {
    const int h = f / (RP * QT_CH), prow = (f / QT_CH) % RP, part = f % QT_CH;
    const int c = c0 + 8 * part;
    if (c >= c_end) continue;
    if (c + 8 <= c_end) {
      *(uint4*)(d.qbf + ((int64_t)h * RP + prow) * d.n_pad + c) = *(const uint4*)(&sm.t[h][prow * QT_P + 8 * part]);
    } else {
      for (int j = 0; j < 8 && c + j < c_end; ++j)
        d.qbf[((int64_t)h * RP + prow) * d.n_pad + c + j] = sm.t[h][prow * QT_P + 8 * part + j];
    }
  }
}

template <int RP>
__global__ __launch_bounds__(kBlock) void k_qpadl(OCC_KARGS) {
  __shared__ __attribute__((aligned(16))) QTSmem<RP> sm;
#define B_(d, b) qtile_body<RP, false>(d, b, sm)
  OCC_DISPATCH(K_QPAD, B_)
#undef B_
}

template <int RP>
__global__ __launch_bounds__(kBlock) void k_qredl(OCC_KARGS) {
  __shared__ __attribute__((aligned(16))) QTSmem<RP> sm;
#define B_(d, b) qtile_body<RP, true>(d, b, sm)
  OCC_DISPATCH(K_QRED, B_)
#undef B_
}

// ---------------------------------------------------------------------------
// Stand-alone error update: err_new = (M + err_prev) - M_hat, elementwise,
// same operation order as the fused pass.  Bound by memory (s_M + 12 bytes
// an element); one element per thread and a 64-bit division per element ran
// at 3.4 TB/s.  A thread takes U chunks of four columns, all of their loads
// in flight at once; chunk q of the matrix is row q / cpr, columns
// 4 (q % cpr) .. + 3 (cpr chunks a row).  The last chunk of a row may be short:
// it is loaded from as many columns to the left as it lacks, in vectors like
// the others, and stored element by element.
// 8192 x 4096 bf16: 139 -> 70 us.
// ---------------------------------------------------------------------------
// Chunks per thread: four, and one up to 2^19 chunks, where fewer threads leave
// compute units without a block (in place, four / two / one chunks, and one
// element per thread: 1303 x 161 fp32 3.8 / 3.1 / 2.7 / 2.6 us, 1000 x 1001 bf16
// 4.6 / 3.8 / 3.7 / 4.9, 4096 x 1024 fp32 11.0 / 11.4 / 11.5 / 14.5, 8192 x 4096
// fp32 82 / 93 / 91 / 114).
constexpr int64_t EU_SMALL = (int64_t)1 << 19;

template <int DT, bool NT, int U>
__global__ __launch_bounds__(kBlock) void k_err_update(Desc d, uint32_t cpr) {
  const int64_t total = (int64_t)d.m * cpr;
  const int64_t step = (int64_t)gridDim.x * (kBlock * U);
  for (int64_t q0 = (int64_t)blockIdx.x * (kBlock * U) + threadIdx.x; q0 < total; q0 += step) {
    float4 m4[U], e4[U], h4[U];
    int row[U], col[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = q0 + kBlock * u;
      row[u] = d.m;
      if (q >= total) continue;
      // 32-bit division where it is enough
      row[u] = total <= 0xffffffffll ? (int)((uint32_t)q / cpr) : (int)(q / cpr);
      col[u] = 4 * (int)(q - (int64_t)row[u] * cpr);
      const int c = min(col[u], d.n - 4);
      const int64_t mo = (int64_t)row[u] * d.ldm + c;
      if (d.n < 4) {
        // rows narrower than a chunk: their elements in the last places
        float m[4], e[4], h[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          m[j] = c + j >= 0 ? m_elem<DT>(d, mo + j) : 0.f;
          e[j] = d.err_in && c + j >= 0 ? d.err_in[(int64_t)row[u] * d.lde_in + c + j] : -0.f;
          h[j] = c + j >= 0 ? d.Mhat[(int64_t)row[u] * d.ldh + c + j] : 0.f;
        }
        m4[u] = make_float4(m[0], m[1], m[2], m[3]);
        e4[u] = make_float4(e[0], e[1], e[2], e[3]);
        h4[u] = make_float4(h[0], h[1], h[2], h[3]);
        continue;
      }
      if constexpr (DT == DT_F32) {
        m4[u] = ld_f4<false>((const float*)d.M + mo);
      } else {
        const uint2 w = ld_h4<false>((const uint16_t*)d.M + mo);
        m4[u] = make_float4(bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y));
      }
      e4[u] = d.err_in ? ld_f4<false>(d.err_in + (int64_t)row[u] * d.lde_in + c)
                       : make_float4(-0.f, -0.f, -0.f, -0.f);
      h4[u] = ld_f4<false>(d.Mhat + (int64_t)row[u] * d.ldh + c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (row[u] >= d.m) continue;
      float* o = d.err_out + (int64_t)row[u] * d.lde_out + col[u];
      const int left = d.n - col[u];   // columns of the row from here
      const float v[4] = {(m4[u].x + e4[u].x) - h4[u].x, (m4[u].y + e4[u].y) - h4[u].y,
                          (m4[u].z + e4[u].z) - h4[u].z, (m4[u].w + e4[u].w) - h4[u].w};
      if (left >= 4) {
        store_f4<NT>(o, v[0], v[1], v[2], v[3]);
      } else {
        // v[4 - left] is the first of the chunk's own columns
        o[0] = left == 3 ? v[1] : (left == 2 ? v[2] : v[3]);
        if (left > 1) o[1] = left == 3 ? v[2] : v[3];
        if (left > 2) o[2] = v[3];
      }
    }
  }
}

// Copy descriptor chunks passed by value into the workspace table (12
// descriptors, 3.3 KB of kernel arguments per launch).
constexpr int kTableChunk = 12;
struct TableChunk {
  Desc d[kTableChunk];
};

__global__ void k_write_table(Desc* dst, TableChunk src, int n) {
  const int words = (int)(sizeof(Desc) / 4) * n;
  const uint32_t* s = (const uint32_t*)&src;
  uint32_t* o = (uint32_t*)dst;
  for (int w = threadIdx.x; w < words; w += blockDim.x) o[w] = s[w];
}

__global__ void k_zero_words(uint32_t* p, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0u;
}

// Row list of the row-sparse step: rows[0 .. n) copied to dst, each index
// clamped into [0, m_rows) so that no kernel can address outside M, err or
// M_hat; an index out of range, or not larger than the one before it (the
// list must be strictly increasing), raises FLAG_BAD_ROWS.  The streaming
// kernels read the row map from the copy only.
__global__ __launch_bounds__(kBlock) void k_rows_check(const int32_t* rows, int64_t n,
                                                       int32_t m_rows, int32_t* dst,
                                                       uint32_t* flags) {
  bool bad = false;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kBlock) {
    const int32_t v = rows[i];
    bad = bad || v < 0 || v >= m_rows || (i > 0 && v <= rows[i - 1]);
    dst[i] = v < 0 ? 0 : (v >= m_rows ? m_rows - 1 : v);
  }
  if (bad) atomicOr(flags, FLAG_BAD_ROWS);
}

// Row-sparse step with an empty row list: A is zero, so P_hat = 0 and
// Q = A^T P_hat = 0 (the dense step on an all-zero matrix gives the same and
// flags the rank deficiency).
__global__ __launch_bounds__(kBlock) void k_rows_empty(float* Q, int64_t n, uint32_t* flags) {
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kBlock)
    Q[i] = 0.f;
  if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(flags, FLAG_RANK_DEFICIENT);
}

}  // namespace occ
