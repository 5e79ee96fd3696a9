// Stage kernels of a wide layer on few input maps (the first layer, one image at a time).  Part of the stage kernels'
// translation unit.
#pragma once
#include "cnn355_stage.h"

namespace cnn355 {

typedef float v4acc __attribute__((ext_vector_type(4)));
constexpr int FIRST_MAPS = 32;   // output maps of one work item
// floats between the filter rows of two output maps in LDS: whole groups of four taps, 4 beyond a multiple of 32 (16 rows by
// 4 taps of a matrix operand then lie in different banks)
constexpr int first_pitch(int taps) { return (taps + 27) / 32 * 32 + 4; }

// FP of a layer whose whole contraction (input maps x taps) is short, on the matrix cores, with its activation and pooling.
// Work item = (32 output maps, band of conv rows): the rows of the input maps under the band and the filters of the maps
// lie in LDS; a wavefront computes 16 maps by 16 pixels at a time (v_mfma_f32_16x16x4_f32, four taps an instruction), the
// sums pass through LDS to 32 lanes a map for tanh, pooling and the arg-max (index of the first maximum).
// 300C6S1 on 2 x 96 x 96, in a kernel trace: 10.1 us, 34.0 with a lane per pixel (two LDS reads a multiply-add, 900 items of one map); bound by the
// latency of its three steps (operands, product, epilogue), not by the 0.6 us of arithmetic.
__device__ void conv_fwd_mx_item(const LayerDev& L, const Stage& st, int item, const gfloat* in, float* lds) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  constexpr int WAVES = WG / 64;
  const int jt = item / st.n_tiles, band = item - jt * st.n_tiles;
  const int j0 = jt * FIRST_MAPS;
  const int K = L.K, KK = K * K, Kd = L.Mi * KK, Mo = L.Mo, Wi = L.Wi, Wo = L.Wo, stride = L.S + 1, Kp = L.Kp;
  const int y0 = band * st.tile_rows, rows = min(st.tile_rows, L.Ho - y0), P = rows * Wo;
  const int in_rows = (rows - 1) * stride + K, map_sz = in_rows * Wi, Kd4 = (Kd + 3) & ~3, Kd1 = Kd & ~3;
  const int WP = first_pitch(Kd), PP = P | 1;

  float* lds_w = lds;                          // [32][WP] filters, zero from Kd on
  int* koff = (int*)(lds_w + FIRST_MAPS * WP); // [Kd4] place of a tap in the staged input
  float* lds_in = (float*)(koff + Kd4);        // [Mi][map_sz]
  float* lds_pre = lds_in + L.Mi * map_sz;     // [32][PP] the sums the units received
  float* lds_out = lds_pre + FIRST_MAPS * PP;  // [32][PP] after the activation

  const int r = tid >> 5, xl = tid & 31, j = j0 + r;   // 32 lanes of a map, outside the product
  const float b = L.bias[min(j, Mo - 1)];
  {
    const gfloat* w = L.w + (size_t)min(j, Mo - 1) * Kd;
    for (int x = xl; x < Kd4; x += 32) lds_w[r * WP + x] = x < Kd ? w[x] : 0.f;
    for (int i = 0; i < L.Mi; ++i) {
      const gfloat* src = in + (size_t)i * L.Hi * Wi + (size_t)y0 * stride * Wi;
#pragma unroll 4
      for (int x = tid; x < map_sz; x += WG) lds_in[i * map_sz + x] = src[x];
    }
    for (int x = tid; x < Kd4; x += WG) {
      const int i = x / KK, t = x - i * KK, ky = t / K;
      koff[x] = x < Kd ? i * map_sz + ky * Wi + (t - ky * K) : 0;
    }
  }
  __syncthreads();
  const int lr = lane & 15, lk = lane >> 4, CT = (P + 15) >> 4;
  for (int task = wave; task < 2 * CT; task += WAVES) {
    const int half = task & 1, p = (task >> 1) * 16 + lr;
    const int y = p / Wo, x = p - y * Wo;
    const float* xb = lds_in + (p < P ? (y * Wi + x) * stride : 0);
    const float* wa = lds_w + (half * 16 + lr) * WP + lk;
    v4acc acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 6
    for (int k = 0; k < Kd1; k += 4) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[k], xb[koff[k + lk]], acc, 0, 0, 0);
    if (Kd1 < Kd4) {   // the last taps, filled up with zeros on both sides (an infinite pixel times a weight of zero is no zero)
      const float x = xb[koff[Kd1 + lk]];
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[Kd1], Kd1 + lk < Kd ? x : 0.f, acc, 0, 0, 0);
    }
    if (p < P) {
#pragma unroll
      for (int v = 0; v < 4; ++v) lds_pre[(half * 16 + lk * 4 + v) * PP + p] = acc[v];
    }
  }
  __syncthreads();
  float* pre = lds_pre + r * PP;
  float* out = lds_out + r * PP;
  if (j < Mo) {
    const size_t o = ((size_t)j * L.Ho + y0) * Wo;
    for (int p = xl; p < P; p += 32) {
      const float sum = pre[p] + b, a = act_f(sum);
      pre[p] = sum;
      out[p] = a;
      L.act[o + p] = a;
      if (Kp == 1) L.dact[o + p] = dact_pre_f(sum);
    }
  }
  __syncthreads();
  if (j < Mo && Kp > 1) {
    const int Wp = L.Wp;
    for (int py = 0; py < rows / Kp; ++py)
      for (int px = xl; px < Wp; px += 32) {
        const float* win = out + py * Kp * Wo + px * Kp;
        float best = win[0];
        int wy = 0, wx = 0;
        for (int dy = 0; dy < Kp; ++dy)
          for (int dx = 0; dx < Kp; ++dx) {
            const float v = win[dy * Wo + dx];
            if (v > best) { best = v; wy = dy; wx = dx; }
          }
        const size_t o = ((size_t)j * L.Hp + (y0 / Kp + py)) * Wp + px;
        L.out[o] = best;
        L.dact[o] = dact_pre_f(pre[(py * Kp + wy) * Wo + px * Kp + wx]);
        L.arg[o] = (uint8_t)(wy * Kp + wx);
        L.argyx[o] = ((y0 + py * Kp + wy) << 16) | (px * Kp + wx);
      }
  }
  __syncthreads();
}

// AW of such a layer (Sec. 3.4) over the pooling winners.  Work item = st.chunk output maps: the whole input lies in LDS; the
// wavefronts share a map's winners, a lane is a weight.  A group of 64 weights takes a winner at a time (place and delta are
// scalars), the r weights left over 64 / r winners.  The rows of the input have a pitch of K beyond a multiple of 32 floats and
// the maps one of K * K, so that the K * K taps of a winner lie in as many banks.
// 300C6S1 on 2 x 96 x 96 with 529 winners, in a kernel trace: 12.9 us, 21.6 with a workgroup per map (two rounds of them, three LDS
// reads a term); 300C3 on 3 x 32 x 32 7.8, 11.6.  Issue of the readlanes and reads bounds the large one.
__host__ __device__ constexpr int first_row_pitch(int Wi, int K) { return Wi + ((K - Wi) % 32 + 32) % 32; }
__host__ __device__ constexpr int first_map_pitch(int Hi, int Wi, int K) {
  return Hi * first_row_pitch(Wi, K) + ((K * K - Hi * first_row_pitch(Wi, K)) % 32 + 32) % 32;
}
// up to 64 winners (deltas and places in the lanes of d and off): a read and a multiply-add per winner and group of 64 weights
template <int G>
__device__ __forceinline__ void first_groups(const float* in, float d, int off, int nq, const int (&at)[3], float (&acc)[3][2]) {
  constexpr int B = G == 1 ? 8 : 4;   // winners whose reads are in flight together (past the end: the last one with a delta of zero)
  for (int q = 0; q < nq; q += B) {
    float v[B][G];
#pragma unroll
    for (int c = 0; c < B; ++c)
#pragma unroll
      for (int g = 0; g < G; ++g) v[c][g] = in[__builtin_amdgcn_readlane(off, q + c) + at[g]];
#pragma unroll
    for (int c = 0; c < B; ++c) {
      const float dk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(d), q + c));
#pragma unroll
      for (int g = 0; g < G; ++g) acc[g][c & 1] = fmaf(dk, v[c][g], acc[g][c & 1]);
    }
  }
}
// the R rows of all maps into LDS: U rows of a wavefront in flight, H loads each
template <int U, int H>
__device__ __forceinline__ void first_rows(float* lds_in, const gfloat* in, int R, int Hi, int Wi, int RP, int MP) {
  constexpr int WAVES = WG / 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  int i = 0;
  for (int y0 = wave; y0 < R; y0 += U * WAVES)
    for (int x0 = 0; x0 < Wi; x0 += 64 * H) {
      float v[U][H];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int h = 0; h < H; ++h) v[u][h] = in[min(y0 + u * WAVES, R - 1) * Wi + min(x0 + h * 64 + lane, Wi - 1)];
      while (y0 >= (i + 1) * Hi) ++i;   // (a division is dearer than the copy of a row)
      int iu = i;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int y = y0 + u * WAVES;
        while (y >= (iu + 1) * Hi) ++iu;
        float* dst = lds_in + iu * MP + (y - iu * Hi) * RP + x0 + lane;
#pragma unroll
        for (int h = 0; h < H; ++h)
          if (y < R && x0 + h * 64 + lane < Wi) dst[h * 64] = v[u][h];
      }
    }
}
__device__ void conv_wgrad_first_item(const LayerDev& L, const Stage& st, int item, const gfloat* in, const Ctx& ctx, float* lds) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  constexpr int WAVES = WG / 64, GMAX = 3;
  const int K = L.K, KK = K * K, Kd = L.Mi * KK, Wi = L.Wi, HW = L.Hp * L.Wp, stride = L.S + 1;
  const int RP = first_row_pitch(Wi, K), MP = first_map_pitch(L.Hi, Wi, K);
  const int JG = st.chunk, j0 = item * JG, nj = min(JG, L.Mo - j0), SH = WAVES / JG;
  const int jl = wave / SH, share = wave - jl * SH;
  const bool on = jl < nj;
  const int G = Kd >> 6, r = Kd & 63, S = r ? 64 / r : 0;

  float* lds_in = lds;                       // [Mi] maps, MP apart, of rows RP apart
  float* lds_d = lds_in + L.Mi * MP;         // [JG][HW] deltas
  int* lds_off = (int*)(lds_d + JG * HW);    // [JG][HW] places of the winners' fields
  const int NW = nj * Kd;                    // weights of the item, side by side in memory (full table)
  gfloat* w_at = L.w + (size_t)j0 * Kd;
  float w_old = tid < NW ? w_at[tid] : 0.f;
  {
    for (int x = tid; x < nj * HW; x += WG) {
      const int yx = L.argyx[(size_t)j0 * HW + x];
      lds_d[x] = L.delta[(size_t)j0 * HW + x];
      lds_off[x] = ((yx >> 16) * RP + (yx & 0xffff)) * stride;
    }
    const int R = L.Mi * L.Hi;   // (loads past the last row cost as much as the others)
    if (Wi > 64) first_rows<12, 2>(lds_in, in, R, L.Hi, Wi, RP, MP);
    else if (R > 6 * WAVES) first_rows<12, 1>(lds_in, in, R, L.Hi, Wi, RP, MP);
    else if (R > 2 * WAVES) first_rows<6, 1>(lds_in, in, R, L.Hi, Wi, RP, MP);
    else first_rows<2, 1>(lds_in, in, R, L.Hi, Wi, RP, MP);
  }
  // places of this lane's weights in a field: the full groups, then the rest
  const float by_KK = 1.f / KK, by_K = 1.f / K;
  auto place = [&](int w) {   // (quotients of numbers below 256: half a step off the whole numbers, exact)
    const int i = (int)((w + 0.5f) * by_KK), t = w - i * KK, ky = (int)((t + 0.5f) * by_K);
    return i * MP + ky * RP + t - ky * K;
  };
  int at[GMAX], at_r = 0;
#pragma unroll
  for (int g = 0; g < GMAX; ++g) at[g] = g < G ? place(g * 64 + lane) : 0;
  const int sub = r ? lane / r : 0;
  if (r) at_r = place(G * 64 + (sub < S ? lane - sub * r : 0));
  __syncthreads();
  float acc[GMAX][2], acc_r[2] = {0.f, 0.f}, dsum = 0.f;
#pragma unroll
  for (int g = 0; g < GMAX; ++g) acc[g][0] = acc[g][1] = 0.f;
  if (on) {
    const int per = (HW + SH - 1) / SH, q_lo = min(share * per, HW), q_hi = min(q_lo + per, HW);
    const float* dl = lds_d + jl * HW;
    const int* of = lds_off + jl * HW;
    for (int q0 = q_lo; q0 < q_hi; q0 += 64) {
      const int nq = min(64, q_hi - q0);
      const float d = lane < nq ? dl[q0 + lane] : 0.f;   // (past the end: a delta of zero at the field of the last winner, which is read anyway)
      const int off = of[q0 + min(lane, nq - 1)];
      dsum += d;
      switch (G) {   // (a loop for every number of groups: a branch a group would wait for every read by itself)
        case 1: first_groups<1>(lds_in, d, off, nq, at, acc); break;
        case 2: first_groups<2>(lds_in, d, off, nq, at, acc); break;
        case 3: first_groups<3>(lds_in, d, off, nq, at, acc); break;
        default: break;
      }
    }
    if (r && sub < S) {
      const float* x = lds_in + at_r;
      int q = q_lo + sub;
#pragma unroll 2
      for (; q + S < q_hi; q += 2 * S) {
        acc_r[0] = fmaf(dl[q], x[of[q]], acc_r[0]);
        acc_r[1] = fmaf(dl[q + S], x[of[q + S]], acc_r[1]);
      }
      if (q < q_hi) acc_r[0] = fmaf(dl[q], x[of[q]], acc_r[0]);
    }
    if (r) {   // the winners side by side in the lanes added in their order
      const float v = acc_r[0] + acc_r[1];
      acc_r[0] = 0.f;
      for (int u = 0; u < S; ++u) acc_r[0] += __shfl(v, u * r + (lane < r ? lane : 0), 64);
    }
    dsum = wave_sum(dsum);
  }
  __syncthreads();   // (the input is done with)
  // [wavefront][group][lane], then the wavefronts' sums of deltas
  float* red = lds;
  const int RG = G + (r ? 1 : 0);
  if (on) {
#pragma unroll
    for (int g = 0; g < GMAX; ++g)
      if (g < G) red[(wave * RG + g) * 64 + lane] = acc[g][0] + acc[g][1];
    if (r) red[(wave * RG + G) * 64 + lane] = acc_r[0];
    if (lane == 0) red[WAVES * RG * 64 + wave] = dsum;
  }
  __syncthreads();
  gfloat* g_out = ctx.grad_out;
  for (int x = tid; x < NW; x += WG) {
    const int jj = x / Kd, w = x - jj * Kd;
    float s = 0.f;
#pragma unroll 8
    for (int k = 0; k < SH; ++k) s += red[((jj * SH + k) * RG + (w >> 6)) * 64 + (w & 63)];
    if (g_out) g_out[L.w_canon + (size_t)j0 * Kd + x] = s;
    else w_at[x] = (x < WG ? w_old : w_at[x]) - ctx.lr * s;
  }
  if (tid < nj) {
    float s = 0.f;
    for (int k = 0; k < SH; ++k) s += red[WAVES * RG * 64 + tid * SH + k];
    if (g_out) g_out[L.b_canon + j0 + tid] = s;
    else L.bias[j0 + tid] -= ctx.lr * s;
  }
  __syncthreads();
}

}  // namespace cnn355
