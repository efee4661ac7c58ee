// Stand-alone decompression at padded rank 32, 64 or 128: M_hat = P Q^T from
// the caller's factors (the receiving side of compressed backpropagation).
//
// The only traffic that counts is the output, so the pass should run at the
// rate of a write stream.  The reconstruction kernels of the fused step keep
// Q columns in registers and share each 32-row P tile through LDS with a
// barrier per tile; without A to read they wait for the next P tile, and in
// bf16 they stored 2 bytes a lane into 64-byte pieces of rows (16384 x 8192,
// rank 128, bf16 out: 203 us for 268 MB).  Here a block stages 128 columns of
// Q in LDS once, and each wave then walks 32-row tiles by itself, with no
// barrier: its P rows come straight into the A operands (the next tile's
// loads in flight during the products), the four 32-column tiles take their
// B operands from LDS, and the results pass through a wave's own LDS tile to
// be stored as 256-byte pieces of rows, 16 bytes a lane.  16384 x 8192, rank
// 128, bf16 out: 203 -> 119 us; 8192 x 4096, rank 64, fp32 out: 57 -> 34 us.
//
// The products and their order are those of the fused step (k_mlx when SPLIT,
// k_ml otherwise), so M_hat is bitwise the one that step writes.
#pragma once

#include "kernels_large.hpp"

namespace occ {

constexpr int DC_COLS = 128;               // columns per block
// waves per block: at rank 128 the Q tile leaves room for one block per
// compute unit, which then holds eight waves
__host__ __device__ constexpr int dc_waves(int rp) { return rp >= 128 ? 8 : 4; }
// blocks that one compute unit holds (LDS)
__host__ __device__ constexpr int dc_blocks_per_cu(int rp) { return rp >= 128 ? 1 : 2; }

template <int RP, bool SPLIT, bool OUTBF>
struct DCShape {
  static constexpr int NW = dc_waves(RP);
  static constexpr int PT = SPLIT ? RP + 8 : RP + 4;      // LDS pitch of a Q column (bf16 / float)
  static constexpr int Q_BYTES = SPLIT ? 2 * DC_COLS * PT * 2 : DC_COLS * PT * 4;
  static constexpr int EC = OUTBF ? 128 : 64;             // columns of the wave's output tile
  static constexpr int EP = EC + (OUTBF ? 8 : 4);         // its pitch in elements
  static constexpr int E_BYTES = 32 * EP * (OUTBF ? 2 : 4);
  static constexpr int BYTES = Q_BYTES + NW * E_BYTES;
};

// Four consecutive ranks k .. k+3 of a caller's factor row (zero past r).
__device__ __forceinline__ f4v dc_load4(const float* row, int k, int r) {
  f4v v = f4v{0.f, 0.f, 0.f, 0.f};
  if (k + 4 <= r) {
    v = *(const f4u_t*)(row + k);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < r) v[e] = row[k + e];
  }
  return v;
}

template <int RP, bool SPLIT, bool OUTBF, bool NT>
__global__ __launch_bounds__(dc_waves(RP) * kWave) void k_dec(Desc d) {
  using S = DCShape<RP, SPLIT, OUTBF>;
  constexpr int NW = S::NW, NTH = NW * kWave, PT = S::PT, EP = S::EP;
  constexpr int NF = RP / 8;               // float4s of a P row per lane
  __shared__ __attribute__((aligned(16))) uint8_t smem[S::BYTES];
  const int wave = wave_id(), lane = threadIdx.x & 63;
  const int li = lane & 31, g = lane >> 5;
  const int col_tiles = (d.n + DC_COLS - 1) / DC_COLS;
  const int ct = (int)blockIdx.x % col_tiles, rb = (int)blockIdx.x / col_tiles;
  const int c0 = ct * DC_COLS;
  const int r_lo = rb * d.mr, r_hi = min(d.m, r_lo + d.mr);

  // P rows of one tile, as loaded.  SPLIT: lane (g, li) supplies ranks
  // 16 s + 8 g .. + 7 of row li to K-step s, two float4s each.  fp32: ranks
  // 2 kp + g to MFMA kp; both halves load the row's float4s 4 j .. 4 j + 3
  // (two MFMAs each) and keep their own two values.
  f4v raw[SPLIT ? NF : 2 * NF];
  auto p_load = [&](int row0) {
    const float* row = d.P + (int64_t)min(row0 + li, d.m - 1) * d.r;
    if constexpr (SPLIT) {
#pragma unroll
      for (int x = 0; x < NF; ++x) raw[x] = dc_load4(row, 16 * (x / 2) + 8 * g + 4 * (x % 2), d.r);
    } else {
#pragma unroll
      for (int x = 0; x < 2 * NF; ++x) raw[x] = dc_load4(row, 4 * x, d.r);
    }
  };
  int row0 = r_lo + 32 * wave;
  if (row0 < r_hi) p_load(row0);

  // Q columns c0 .. c0 + 127 into LDS (zero past n and r).  SPLIT: bf16 hi and
  // lo rows, [part][column][rank]; fp32: [column][g][kp], rank 2 kp + g, so
  // that a lane reads four MFMAs' operands at once.
  uint16_t* qh = (uint16_t*)smem;
  uint16_t* ql = qh + DC_COLS * PT;
  float* qf = (float*)smem;
  for (int f = threadIdx.x; f < DC_COLS * RP / 4; f += NTH) {
    const int c = f / (RP / 4), k = 4 * (f % (RP / 4));
    f4v v = f4v{0.f, 0.f, 0.f, 0.f};
    if (c0 + c < d.n) v = dc_load4(d.Q + (int64_t)(c0 + c) * d.r, k, d.r);
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
  __syncthreads();

  uint8_t* const ep = smem + S::Q_BYTES + wave * S::E_BYTES;
  for (; row0 < r_hi; row0 += 32 * NW) {
    // operands of this tile, then the next tile's loads
    bf16x8 ah[SPLIT ? RP / 16 : 1], al[SPLIT ? RP / 16 : 1];
    float pa[SPLIT ? 1 : RP / 2];
    if constexpr (SPLIT) {
#pragma unroll
      for (int s = 0; s < RP / 16; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float v = raw[2 * s + e / 4][e % 4];
          const __bf16 h = (__bf16)v;
          ah[s][e] = h;
          al[s][e] = (__bf16)(v - (float)h);
        }
    } else {
#pragma unroll
      for (int x = 0; x < 2 * NF; ++x) {
        pa[2 * x] = g ? raw[x][1] : raw[x][0];
        pa[2 * x + 1] = g ? raw[x][3] : raw[x][2];
      }
    }
    if (row0 + 32 * NW < r_hi) p_load(row0 + 32 * NW);

#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2) {       // two 32-column tiles at a time
      f16v acc[2] = {f16v{}, f16v{}};
      if constexpr (SPLIT) {
#pragma unroll
        for (int s = 0; s < RP / 16; ++s) {
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int o = (64 * c2 + 32 * u + li) * PT + 16 * s + 8 * g;
            const bf16x8 bh = *(const bf16x8*)(qh + o);
            const bf16x8 bl = *(const bf16x8*)(ql + o);
            acc[u] = mfma32bf(ah[s], bh, acc[u]);
            acc[u] = mfma32bf(ah[s], bl, acc[u]);
            acc[u] = mfma32bf(al[s], bh, acc[u]);
          }
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
            for (int u = 0; u < 2; ++u) acc[u] = mfma32(pa[4 * k4 + e], b[u][e], acc[u]);
        }
      }
      // acc[u][v] = M_hat[row0 + mf32_row(v, g)][c0 + 64 c2 + 32 u + li]
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int o = mf32_row(v, g) * EP + 32 * u + li;
          if constexpr (OUTBF) ((uint16_t*)ep)[o + 64 * c2] = bf16_rne(acc[u][v]);
          else ((float*)ep)[o] = acc[u][v];
        }
      if (OUTBF && c2 == 0) continue;
      // The tile is written and read by this wave only; LDS keeps a wave's
      // operations in order, and the waits also order them for the compiler.
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      constexpr int W = OUTBF ? 8 : 4;     // elements of a lane's 16 bytes
      const int cl = W * (lane & 15);
      const int col = c0 + cl + (OUTBF ? 0 : 64 * c2);
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const int rr = 4 * x + (lane >> 4), row = row0 + rr;
        const uint4 v = *(const uint4*)(ep + (rr * EP + cl) * (OUTBF ? 2 : 4));
        if (row >= r_hi || col >= d.n) continue;
        const int64_t off = (int64_t)row * d.ldh + col;
        if (col + W <= d.n) {
          if constexpr (NT) {
            typedef uint32_t nu4 __attribute__((ext_vector_type(4)));
            __builtin_nontemporal_store(nu4{v.x, v.y, v.z, v.w},
                                        (nu4*)((uint8_t*)d.Mhat + off * (OUTBF ? 2 : 4)));
          } else if constexpr (OUTBF) {
            *(u4h_t*)((uint16_t*)d.Mhat + off) = u4h_t{v.x, v.y, v.z, v.w};
          } else {
            *(f4u_t*)(d.Mhat + off) = f4u_t{__uint_as_float(v.x), __uint_as_float(v.y),
                                            __uint_as_float(v.z), __uint_as_float(v.w)};
          }
        } else {
          const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int j = 0; j < W; ++j)
            if (col + j < d.n) {
              if constexpr (OUTBF) ((uint16_t*)d.Mhat)[off + j] = (uint16_t)(w[j / 2] >> (16 * (j % 2)));
              else d.Mhat[off + j] = __uint_as_float(w[j]);
            }
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
  }
}

}  // namespace occ
