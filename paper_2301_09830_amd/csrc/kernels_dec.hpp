// Stand-alone decompression at padded rank 32, 64 or 128: M_hat = P Q^T from
// the caller's factors (the receiving side of compressed backpropagation).
//
// The only traffic that counts is the output, so the pass should run at the
// rate of a write stream.  The reconstruction kernels of the fused step keep
// Q columns in registers and share each 32-row P tile through LDS with a
// barrier per tile; without A to read they wait for the next P tile, and in
// bf16 they stored 2 bytes a lane into 64-byte pieces of rows (16384 x 8192,
// rank 128, bf16 out: 203 us for 268 MB).  Here a block stages 128 columns of
// Q (64 for small outputs) in LDS once, and each wave then walks 32-row tiles
// by itself, with no barrier: its P rows are loaded whole, two tiles ahead, and
// turned into the B operands through the wave's own LDS tile (loading them in
// operand order fetched every line four times), the 32-column tiles take their
// A operands from the Q tile, and the results pass through the wave's LDS tile
// to be stored as 256-byte pieces of rows (128 in bf16 from 64 columns), 16
// bytes a lane.  The products run
// transposed (M_hat^T = Q P^T), so that a lane holds four consecutive columns
// of a row and writes them to LDS at once.  The common tile has no bounds
// tests: one at every load made each load wait for the one before.
// 16384 x 8192, rank 128, bf16 out: 203 -> 112-119 us; 8192 x 4096, rank 64, fp32
// out: 57 -> 31 us (4.4 TB/s).  At rank 128 neither the products nor the
// stores bound the pass alone (a third of the products takes 14 % less time,
// none of the stores 19 % less): two waves per SIMD overlap them only partly.
//
// The products and their order are those of the fused step (k_mlx when SPLIT,
// k_ml otherwise), so M_hat is bitwise the one that step writes.
#pragma once

#include "kernels_large.hpp"

namespace occ {

constexpr int DC_COLS = 128;               // columns per block
constexpr int DC_COLS_SMALL = 64;          // the same where the blocks would fill at most half the chip
// waves per block: at rank 128 a tile of DC_COLS columns of Q leaves room for
// one block per compute unit, which then holds eight waves
__host__ __device__ constexpr int dc_waves(int rp, int cols) { return rp >= 128 && cols == DC_COLS ? 8 : 4; }
// blocks that a compute unit is planned for (one where LDS holds no more; at
// the smaller ranks LDS would hold three, but two fill the store stream)
__host__ __device__ constexpr int dc_blocks_per_cu(int rp, int cols) { return rp >= 128 && cols == DC_COLS ? 1 : 2; }

template <int RP, bool SPLIT, bool OUTBF, int COLS>
struct DCShape {
  static constexpr int NW = dc_waves(RP, COLS);
  static constexpr int PT = SPLIT ? RP + 8 : RP + 4;      // LDS pitch of a Q column (bf16 / float)
  static constexpr int Q_BYTES = SPLIT ? 2 * COLS * PT * 2 : COLS * PT * 4;
  static constexpr int EC = OUTBF ? COLS : 64;             // columns of the wave's output tile
  static constexpr int EP = EC + (OUTBF ? 8 : 4);         // its pitch in elements
  static constexpr int O_BYTES = 32 * EP * (OUTBF ? 2 : 4);
  // P's operands pass through the same tile: one bf16 part of it, or 64 ranks in fp32
  static constexpr int P_BYTES = SPLIT ? 32 * PT * 2 : 32 * ((RP < 64 ? RP : 64) + 4) * 4;
  static constexpr int E_BYTES = O_BYTES > P_BYTES ? O_BYTES : P_BYTES;
  static constexpr int BYTES = Q_BYTES + NW * E_BYTES;
};

// Factor rows are read in float4s of consecutive ranks straight from the
// caller's array.  Unless r is the padded rank, the last ones of a row run on
// into the next rows, so the values from rank r on are dropped when used.  At
// the end of the array (INSIDE false; `last` its last element) a float4 may not
// leave it.  A bounds test at every float4 made each load wait for the one
// before, and so did reading those rows element by element behind tests, which
// every small output waited for.  In 64-column blocks (small outputs) such a
// float4 is taken from the last four elements and shifted: 512 x 512 rank 108,
// fp32 products 13.0 -> 9.9 us, split products 10.1 -> 6.9 us.  In 128-column
// blocks its elements are loaded one by one without tests, the last one in the
// place of those past it: the shifts' registers there cost every tile (8192 x
// 4096 rank 64, fp32 products 47.4 against 46.9 us, rank 128 82.6 against 79.1).
template <bool INSIDE, int COLS>
__device__ __forceinline__ f4v dc_load4(const float* row, int k, const float* last) {
  const float* const p = row + k;
  if constexpr (INSIDE) {
    return *(const f4u_t*)p;
  } else if constexpr (COLS == DC_COLS) {
    f4v v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = *(p + e < last ? p + e : last);
    return v;
  } else {
    const float* const q = last - 3;   // (a factor above rank 16 holds hundreds of elements)
    f4v v = *(const f4u_t*)(p < q ? p : q);
    const int sh = p < q ? 0 : (int)min(p - q, (int64_t)4);
    v = sh & 1 ? f4v{v[1], v[2], v[3], 0.f} : v;
    v = sh & 2 ? f4v{v[2], v[3], 0.f, 0.f} : v;
    return sh & 4 ? f4v{0.f, 0.f, 0.f, 0.f} : v;
  }
}

// Whether float4s up to padded rank rp of rows up to `last` (of `rows`) stay
// inside the array.
__device__ __forceinline__ bool dc_inside(int64_t last, int64_t rows, int r, int rp) {
  return last < rows && last * r + rp <= rows * r;
}

// 16 bytes of an output row (4 fp32 or 8 bf16 elements).
template <bool OUTBF, bool NT>
__device__ __forceinline__ void dc_store16(const Desc& d, int64_t off, const uint4& v) {
  if constexpr (NT) {
    typedef uint32_t nu4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(nu4{v.x, v.y, v.z, v.w}, (nu4*)((uint8_t*)d.Mhat + off * (OUTBF ? 2 : 4)));
  } else if constexpr (OUTBF) {
    *(u4h_t*)((uint16_t*)d.Mhat + off) = u4h_t{v.x, v.y, v.z, v.w};
  } else {
    *(f4u_t*)(d.Mhat + off) = f4u_t{__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z),
                                    __uint_as_float(v.w)};
  }
}

// (waves per SIMD: those that LDS leaves room for; at rank 128 in 64-column
// blocks the compiler is otherwise ten registers over two, and 4096 x 1024 takes
// 10.7 us instead of 8.3)
template <int RP, bool SPLIT, bool OUTBF, bool NT, int COLS>
__global__ __launch_bounds__(dc_waves(RP, COLS) * kWave, RP >= 128 ? 2 : 3) void k_dec(Desc d) {
  using S = DCShape<RP, SPLIT, OUTBF, COLS>;
  constexpr int NW = S::NW, NTH = NW * kWave, PT = S::PT, EP = S::EP;
  constexpr int NF = RP / 8;               // float4s of a P row per lane
  __shared__ __attribute__((aligned(16))) uint8_t smem[S::BYTES];
  const int wave = wave_id(), lane = threadIdx.x & 63;
  const int li = lane & 31, g = lane >> 5;
  const int col_tiles = (d.n + COLS - 1) / COLS;
  const int ct = (int)blockIdx.x % col_tiles, rb = (int)blockIdx.x / col_tiles;
  const int c0 = ct * COLS;
  const int r_lo = rb * d.mr, r_hi = min(d.m, r_lo + d.mr);

  // P rows of one tile as loaded, whole rows side by side: float4 x of a lane
  // is float4 64 x + lane of the tile.
  f4v raw[NF];
  auto p_load_as = [&](auto in, int row0) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < NF; ++x) {
      const int f = 64 * x + lane, row = min(row0 + f / (RP / 4), d.m - 1);
      raw[x] = dc_load4<decltype(in)::value, COLS>(d.P + (int64_t)row * d.r, 4 * (f % (RP / 4)),
                                                   d.P + (int64_t)d.m * d.r - 1);
    }
  };
  auto p_load = [&](int row0) __attribute__((always_inline)) {
    if (dc_inside(row0 + 31, d.m, d.r, RP)) p_load_as(std::true_type{}, row0);
    else p_load_as(std::false_type{}, row0);
  };
  int row0 = r_lo + 32 * wave;
  if (row0 < r_hi) p_load(row0);

  // Q columns c0 .. c0 + 127 into LDS (zero past n and r).  SPLIT: bf16 hi and
  // lo rows, [part][column][rank]; fp32: [column][g][kp], rank 2 kp + g, so
  // that a lane reads four MFMAs' operands at once.
  uint16_t* qh = (uint16_t*)smem;
  uint16_t* ql = qh + COLS * PT;
  float* qf = (float*)smem;
  {
    constexpr int QL = COLS * RP / 4 / NTH;   // float4s per thread
    static_assert(QL * NTH * 4 == COLS * RP, "Q tile must split evenly");
    f4v q4[QL];
    auto q_load = [&](auto in) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < QL; ++x) {
        const int f = threadIdx.x + NTH * x, c = f / (RP / 4), k = 4 * (f % (RP / 4));
        q4[x] = dc_load4<decltype(in)::value, COLS>(d.Q + (int64_t)min(c0 + c, d.n - 1) * d.r, k,
                                                    d.Q + (int64_t)d.n * d.r - 1);
      }
    };
    if (dc_inside(c0 + COLS - 1, d.n, d.r, RP)) q_load(std::true_type{});
    else q_load(std::false_type{});
#pragma unroll
    for (int x = 0; x < QL; ++x) {
      const int f = threadIdx.x + NTH * x, c = f / (RP / 4), k = 4 * (f % (RP / 4));
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = c0 + c < d.n && k + e < d.r ? q4[x][e] : 0.f;
      if constexpr (SPLIT) {
        uint16_t hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const __bf16 h = (__bf16)v[e];
          hi[e] = bf16_bits(h);
          lo[e] = bf16_bits((__bf16)(v[e] - (float)h));
        }
        *(uint2*)(qh + c * PT + k) = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
        *(uint2*)(ql + c * PT + k) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
      } else {
        float* q = qf + c * PT + k / 2;
        *(float2*)q = make_float2(v[0], v[2]);
        *(float2*)(q + RP / 2) = make_float2(v[1], v[3]);
      }
    }
  }
  __syncthreads();

  // B operands of a tile from its raw rows, through the wave's LDS tile.
  // SPLIT: lane (g, li) supplies ranks 16 s + 8 g .. + 7 of row li to K-step
  // s; the hi parts pass first, then the lo parts.  fp32: ranks 2 kp + g to
  // MFMA kp; 64 ranks pass at a time.
  uint8_t* const ep = smem + S::Q_BYTES + wave * S::E_BYTES;
  bf16x8 ph[SPLIT ? RP / 16 : 1], pl[SPLIT ? RP / 16 : 1];
  float pf[SPLIT ? 1 : RP / 2];
  auto p_operands = [&]() __attribute__((always_inline)) {
    if (d.r != RP) {
      // ranks past r
#pragma unroll
      for (int x = 0; x < NF; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          raw[x][e] = 4 * ((64 * x + lane) % (RP / 4)) + e < d.r ? raw[x][e] : 0.f;
    }
    if constexpr (SPLIT) {
      static_assert(32 * PT * 2 <= S::E_BYTES, "a part of the tile must fit");
      uint16_t* t = (uint16_t*)ep;
#pragma unroll
      for (int part = 0; part < 2; ++part) {
#pragma unroll
        for (int x = 0; x < NF; ++x) {
          const int f = 64 * x + lane;
          uint16_t o[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = raw[x][e];
            const __bf16 h = (__bf16)v;
            o[e] = part == 0 ? bf16_bits(h) : bf16_bits((__bf16)(v - (float)h));
          }
          *(uint2*)(t + (f / (RP / 4)) * PT + 4 * (f % (RP / 4))) =
              make_uint2(o[0] | ((uint32_t)o[1] << 16), o[2] | ((uint32_t)o[3] << 16));
        }
        // written and read by this wave only; LDS keeps a wave's operations
        // in order, and the waits also order them for the compiler
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int s = 0; s < RP / 16; ++s)
          (part == 0 ? ph : pl)[s] = *(const bf16x8*)(t + li * PT + 16 * s + 8 * g);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
    } else {
      constexpr int HR = RP < 64 ? RP : 64, HP = HR + 4;   // ranks at a time, pitch
      static_assert(32 * HP * 4 <= S::E_BYTES, "the ranks that pass at a time must fit");
      float* t = (float*)ep;
#pragma unroll
      for (int h = 0; h < RP / HR; ++h) {
#pragma unroll
        for (int x = 0; x < NF; ++x) {
          const int f = 64 * x + lane, k = 4 * (f % (RP / 4)) - HR * h;
          if (k >= 0 && k < HR) *(f4v*)(t + (f / (RP / 4)) * HP + k) = raw[x];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int x = 0; x < HR / 4; ++x) {
          const f4v v = *(const f4v*)(t + li * HP + 4 * x);
          pf[HR / 2 * h + 2 * x] = g ? v[1] : v[0];
          pf[HR / 2 * h + 2 * x + 1] = g ? v[3] : v[2];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
    }
  };
  if (row0 < r_hi) p_operands();
  if (row0 + 32 * NW < r_hi) p_load(row0 + 32 * NW);

  for (; row0 < r_hi; row0 += 32 * NW) {
#pragma unroll
    for (int c2 = 0; c2 < COLS / 64; ++c2) {       // two 32-column tiles at a time
      f16v acc[2] = {f16v{}, f16v{}};
      if constexpr (SPLIT) {
#pragma unroll
        for (int s = 0; s < RP / 16; ++s) {
          bf16x8 qhv[2], qlv[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int o = (64 * c2 + 32 * u + li) * PT + 16 * s + 8 * g;
            qhv[u] = *(const bf16x8*)(qh + o);
            qlv[u] = *(const bf16x8*)(ql + o);
          }
          // the two tiles' products alternate: each accumulates in the order
          // hi hi, lo hi, hi lo, and no product waits for the one before it
#pragma unroll
          for (int u = 0; u < 2; ++u) acc[u] = mfma32bf(qhv[u], ph[s], acc[u]);
#pragma unroll
          for (int u = 0; u < 2; ++u) acc[u] = mfma32bf(qlv[u], ph[s], acc[u]);
#pragma unroll
          for (int u = 0; u < 2; ++u) acc[u] = mfma32bf(qhv[u], pl[s], acc[u]);
        }
      } else {
#pragma unroll
        for (int k4 = 0; k4 < RP / 8; ++k4) {
          f4v b[2];
#pragma unroll
          for (int u = 0; u < 2; ++u)
            b[u] = *(const f4v*)(qf + (64 * c2 + 32 * u + li) * PT + g * (RP / 2) + 4 * k4);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[u] = mfma32(b[u][e], pf[4 * k4 + e], acc[u]);
        }
      }
      // acc[u][4 q + w] = M_hat[row0 + li][c0 + 64 c2 + 32 u + 8 q + 4 g + w]
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int o = li * EP + 32 * u + 8 * q + 4 * g;
          if constexpr (OUTBF)
            *(uint2*)((uint16_t*)ep + o + 64 * c2) =
                make_uint2(bf16_pack2(acc[u][4 * q], acc[u][4 * q + 1]),
                           bf16_pack2(acc[u][4 * q + 2], acc[u][4 * q + 3]));
          else
            *(float4*)((float*)ep + o) = make_float4(acc[u][4 * q], acc[u][4 * q + 1],
                                                     acc[u][4 * q + 2], acc[u][4 * q + 3]);
        }
      if (OUTBF && c2 < COLS / 64 - 1) continue;
      // The tile is written and read by this wave only; LDS keeps a wave's
      // operations in order, and the waits also order them for the compiler.
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      constexpr int W = OUTBF ? 8 : 4;     // elements of a lane's 16 bytes
      constexpr int LPR = S::EC / W;       // lanes per row, rows per instruction
      constexpr int RPI = kWave / LPR, NX = 32 / RPI;
      const int cl = W * (lane % LPR), rl = lane / LPR;
      const int col = c0 + cl + (OUTBF ? 0 : 64 * c2);
      uint4 ov[NX];
#pragma unroll
      for (int x = 0; x < NX; ++x)
        ov[x] = *(const uint4*)(ep + ((RPI * x + rl) * EP + cl) * (OUTBF ? 2 : 4));
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (c2 == COLS / 64 - 1) {
        // the next tile's operands, and the loads of the one after it
        if (row0 + 32 * NW < r_hi) p_operands();
        if (row0 + 64 * NW < r_hi) p_load(row0 + 64 * NW);
      }
      if (row0 + 32 <= r_hi && c0 + COLS <= d.n) {
        // the common tile, without tests
#pragma unroll
        for (int x = 0; x < NX; ++x)
          dc_store16<OUTBF, NT>(d, (int64_t)(row0 + RPI * x + rl) * d.ldh + col, ov[x]);
      } else {
#pragma unroll
        for (int x = 0; x < NX; ++x) {
          const int row = row0 + RPI * x + rl;
          const int64_t off = (int64_t)row * d.ldh + col;
          if (row < r_hi && col + W <= d.n) {
            dc_store16<OUTBF, NT>(d, off, ov[x]);
          } else if (row < r_hi) {
            const uint32_t w[4] = {ov[x].x, ov[x].y, ov[x].z, ov[x].w};
#pragma unroll
            for (int j = 0; j < W; ++j)
              if (col + j < d.n) {
                if constexpr (OUTBF) ((uint16_t*)d.Mhat)[off + j] = (uint16_t)(w[j / 2] >> (16 * (j % 2)));
                else d.Mhat[off + j] = __uint_as_float(w[j]);
              }
          }
        }
      }
    }
  }
}

}  // namespace occ
