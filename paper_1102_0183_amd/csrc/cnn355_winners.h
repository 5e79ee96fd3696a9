// Stage kernels of wide convolutional layers that visit the pooling winners only (full connection table, one image
// at a time): what the stage kernels' translation unit holds of them, and what it shares with cnn355_winners.hip.
//
// Behind a Kp x Kp max-pooling layer one output neuron in Kp^2 carries a delta (Sec. 2.3), so the sums of Sec. 3.3 and
// 3.4 have 1 / Kp^2 of the terms of the dense product.  Which neuron won is the same for every input map: a lane
// is an input map, and what differs from lane to lane is only data.  Places and deltas of the winners are scalars of
// the wavefront.
#pragma once
#include "cnn355_stage.h"

namespace cnn355 {

constexpr int WIN_LANES = 64;            // input maps of one work item, a lane each
constexpr int WIN_PITCH = WIN_LANES + 1; // floats between pixels of the staged maps: 64 maps side by side, odd

typedef float v4a4 __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at any float
typedef float v4f __attribute__((ext_vector_type(4)));

// The K x K filters of 64 input maps and one output map, side by side in memory, in the registers of a wavefront: as
// they lie (`raw`: consecutive lanes take consecutive words, 16 bytes at a time where K * K is a multiple of four), or a
// filter a lane.  From one to the other through FILTERS_LDS floats of LDS of the wavefront's own.  (Loading a filter a
// lane from global memory visits 64 places an instruction.)
constexpr int filters_pitch(int KK) { return KK % 4 == 0 ? KK + 4 : KK; }   // floats between two filters in LDS
constexpr int filters_lds(int KK) { return 64 * filters_pitch(KK); }
template <int KK>
__device__ __forceinline__ void load_raw(float (&raw)[KK], const gfloat* base, int n) {
  const int lane = threadIdx.x & 63;
  if constexpr (KK % 4 == 0) {
#pragma unroll
    for (int s = 0; s < KK / 4; ++s) {
      const v4a4 q = *(const CNN_GLOBAL v4a4*)(base + min(s * 256 + lane * 4, n * KK - 4));
      raw[4 * s] = q.x; raw[4 * s + 1] = q.y; raw[4 * s + 2] = q.z; raw[4 * s + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int s = 0; s < KK; ++s) raw[s] = base[min(s * 64 + lane, n * KK - 1)];
  }
}
template <int KK>
__device__ __forceinline__ void store_raw(gfloat* base, const float (&raw)[KK], int n) {
  const int lane = threadIdx.x & 63;
  if constexpr (KK % 4 == 0) {
#pragma unroll
    for (int s = 0; s < KK / 4; ++s) {
      v4a4 q;
      q.x = raw[4 * s]; q.y = raw[4 * s + 1]; q.z = raw[4 * s + 2]; q.w = raw[4 * s + 3];
      if (s * 256 + lane * 4 < n * KK) *(CNN_GLOBAL v4a4*)(base + s * 256 + lane * 4) = q;
    }
  } else {
#pragma unroll
    for (int s = 0; s < KK; ++s)
      if (s * 64 + lane < n * KK) base[s * 64 + lane] = raw[s];
  }
}
// (LDS serves a wavefront in order; the fences keep the compiler's order)
template <int KK>
__device__ __forceinline__ void raw_to_filter(float (&w)[KK], const float (&raw)[KK], float* buf) {
  const int lane = threadIdx.x & 63;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  if constexpr (KK == 4) {
#pragma unroll
    for (int t = 0; t < 4; ++t) w[t] = raw[t];
  } else if constexpr (KK % 4 == 0) {
#pragma unroll
    for (int s = 0; s < KK / 4; ++s) {
      const int f = s * 256 + lane * 4, at = f / KK;
      *(v4f*)(buf + f + 4 * at) = v4f{raw[4 * s], raw[4 * s + 1], raw[4 * s + 2], raw[4 * s + 3]};
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int s = 0; s < KK / 4; ++s) {
      const v4f q = *(const v4f*)(buf + lane * (KK + 4) + 4 * s);
      w[4 * s] = q.x; w[4 * s + 1] = q.y; w[4 * s + 2] = q.z; w[4 * s + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int s = 0; s < KK; ++s) buf[s * 64 + lane] = raw[s];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int t = 0; t < KK; ++t) w[t] = buf[lane * KK + t];
  }
}
template <int KK>
__device__ __forceinline__ void filter_to_raw(float (&raw)[KK], const float (&w)[KK], float* buf) {
  const int lane = threadIdx.x & 63;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  if constexpr (KK == 4) {
#pragma unroll
    for (int t = 0; t < 4; ++t) raw[t] = w[t];
  } else if constexpr (KK % 4 == 0) {
#pragma unroll
    for (int s = 0; s < KK / 4; ++s)
      *(v4f*)(buf + lane * (KK + 4) + 4 * s) = v4f{w[4 * s], w[4 * s + 1], w[4 * s + 2], w[4 * s + 3]};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int s = 0; s < KK / 4; ++s) {
      const int f = s * 256 + lane * 4, at = f / KK;
      const v4f q = *(const v4f*)(buf + f + 4 * at);
      raw[4 * s] = q.x; raw[4 * s + 1] = q.y; raw[4 * s + 2] = q.z; raw[4 * s + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int t = 0; t < KK; ++t) buf[lane * KK + t] = w[t];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
    for (int s = 0; s < KK; ++s) raw[s] = buf[s * 64 + lane];
  }
}
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// AW of a wide layer (Sec. 3.4) over the pooling winners.  Work item = (64 input maps, st.chunk <= 16 output maps).  The input
// maps lie in LDS pixel by pixel, 64 maps side by side; a wavefront takes one output map j (or some of its winners, where
// that gives more of the wavefronts work: one alone waits 16 clocks for a read), a lane one filter w_{j,i}: for every winner the K x K input pixels of its field, one LDS read (64 maps of a pixel) and one multiply-add
// each, summed in C chains (500C4 on 300 maps, in a kernel trace: 16.7 us in one launch with the sums of the pull and as long without
// them, 46.5 as a dense matrix product; the LDS reads of 14 output maps an item are 5 us of it, the rest staging, the adjustment and their waits).  The gradients then change places in LDS so that the adjustment reads and writes whole lines.
template <int K>
__device__ void conv_wgrad_win(const LayerDev& L, const Stage& st, int item, const gfloat* in, const Ctx& ctx, float* lds) {
  constexpr int KK = K * K, C = KK <= 9 ? 4 : 2;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  constexpr int WAVES = WG / 64;
  static_assert(WAVES * filters_lds(KK) <= LDS_FLOATS && WAVES * (KK + 1) * 64 <= LDS_FLOATS, "the gradients of a work item change places in LDS");
  const int NC = st.n_tiles, g = item / NC, c = item - g * NC;
  const int Mi = L.Mi, Wi = L.Wi, HiWi = L.Hi * Wi, HW = L.Hp * L.Wp, stride = L.S + 1;
  const int i0 = c * WIN_LANES, n = min(WIN_LANES, Mi - i0);
  int wl2 = 0;   // log2 of the wavefronts that share an output map
  while ((st.chunk << (wl2 + 1)) <= WAVES && (2 * C << wl2) <= HW) ++wl2;
  const int part = wave & ((1 << wl2) - 1), jl = wave >> wl2, j = g * st.chunk + jl;
  const bool on = jl < st.chunk && j < L.Mo;
  const int share = ((HW + (C << wl2) - 1) >> wl2) / C * C;   // winners of one of them: whole rounds of the chains
  const int q_lo = min(part * share, HW), q_hi = min(q_lo + share, HW);
  // what this wavefront's output map needs, in flight before the staging waits
  const int jc = on ? j : 0;
  gfloat* const w_at = L.w + ((size_t)jc * Mi + i0) * KK;
  float w[KK];
  if (on && part == 0) load_raw<KK>(w, w_at, n);
  float dq = L.delta[(size_t)jc * HW + min(q_lo + lane, HW - 1)];
  int yx = L.argyx[(size_t)jc * HW + min(q_lo + lane, HW - 1)];
  {
    constexpr int U = 5, M = WIN_LANES / WAVES;   // pixels a lane and maps a wavefront of one batch of loads
    const gfloat* src = in + (size_t)i0 * HiWi;
    for (int p0 = 0; p0 < HiWi; p0 += 64 * U) {
      float v[M][U];
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int u = 0; u < U; ++u)
          v[m][u] = src[min(wave + m * WAVES, n - 1) * HiWi + min(p0 + u * 64 + lane, HiWi - 1)];
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (p0 + u * 64 + lane < HiWi) lds[(p0 + u * 64 + lane) * WIN_PITCH + wave + m * WAVES] = v[m][u];
    }
  }
  __syncthreads();
  float acc[C][KK];
#pragma unroll
  for (int k = 0; k < C; ++k)
#pragma unroll
    for (int t = 0; t < KK; ++t) acc[k][t] = 0.f;
  float dsum = 0.f;
  for (int q0 = q_lo; q0 < (on ? q_hi : 0); q0 += 64) {
    const int nq = min(64, q_hi - q0);
    float d = dq;
    const int off = ((yx >> 16) * Wi + (yx & 0xffff)) * stride * WIN_PITCH;
    if (lane >= nq) d = 0.f;   // (past the end: a delta of zero at the field of a later winner of the map, or its last one)
    const size_t o = (size_t)j * HW + min(q0 + 64 + lane, HW - 1);   // the next block of winners
    dq = L.delta[o];
    yx = L.argyx[o];
    dsum += d;
    for (int q = 0; q < nq; q += C) {
#pragma unroll
      for (int k = 0; k < C; ++k) {
        const float dk = lane_value(d, q + k);
        const float* x = lds + __builtin_amdgcn_readlane(off, q + k) + lane;
#pragma unroll
        for (int ky = 0; ky < K; ++ky)
#pragma unroll
          for (int kx = 0; kx < K; ++kx)
            acc[k][ky * K + kx] = fmaf(dk, x[(ky * Wi + kx) * WIN_PITCH], acc[k][ky * K + kx]);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < KK; ++t) {
    float s = acc[0][t] + acc[1][t];
    if constexpr (C == 4) s += acc[2][t] + acc[3][t];
    acc[0][t] = s;
  }
  __syncthreads();   // (the input maps are done with)
  if (wl2 > 0) {     // the shares of an output map added in their order
    float* mine = lds + wave * (KK + 1) * 64 + lane;
    if (part > 0) {
#pragma unroll
      for (int t = 0; t < KK; ++t) mine[t * 64] = acc[0][t];
      mine[KK * 64] = dsum;
    }
    __syncthreads();
    if (part == 0)
      for (int p = 1; p < (1 << wl2); ++p) {
#pragma unroll
        for (int t = 0; t < KK; ++t) acc[0][t] += mine[(p * (KK + 1) + t) * 64];
        dsum += mine[(p * (KK + 1) + KK) * 64];
      }
    __syncthreads();
  }
  gfloat* g_out = ctx.grad_out;
  if (on && part == 0) {
    filter_to_raw<KK>(acc[1], acc[0], lds + wave * filters_lds(KK));
    if (g_out) {
      store_raw<KK>(g_out + L.w_canon + ((size_t)j * Mi + i0) * KK, acc[1], n);
    } else {
#pragma unroll
      for (int t = 0; t < KK; ++t) w[t] -= ctx.lr * acc[1][t];
      store_raw<KK>(w_at, w, n);
    }
    if (c == 0) {
      dsum = wave_sum(dsum);
      if (lane == 0) {
        if (g_out) g_out[L.b_canon + j] = dsum;
        else L.bias[j] -= ctx.lr * dsum;
      }
    }
  }
  __syncthreads();
}
__device__ __forceinline__ void conv_wgrad_win_item(const LayerDev& L, const Stage& st, int item, const gfloat* in, const Ctx& ctx,
                                                    float* lds) {
  switch (L.K) {
    case 2: conv_wgrad_win<2>(L, st, item, in, ctx, lds); break;
    case 3: conv_wgrad_win<3>(L, st, item, in, ctx, lds); break;
    case 4: conv_wgrad_win<4>(L, st, item, in, ctx, lds); break;
    case 5: conv_wgrad_win<5>(L, st, item, in, ctx, lds); break;
    default: break;   // (the planner gives this stage no other kernel size)
  }
}

// the pull over the winners (cnn355_winners.hip)
constexpr int WIN_BWD_WAVES = 8;
constexpr int WIN_BWD_REGS = 112;        // sums a lane keeps at most
// windows of one wavefront: as many as the registers hold, 8 at most
constexpr int win_group(int K, int KP) {
  int n = 1;
  while (n < 8 && (KP + K - 1) * (KP * (n + 1) + K - 1) <= WIN_BWD_REGS) ++n;
  return n;
}
// The slices and the overlapping regions of the pull over the winners added in a fixed order, times the derivative of the activation
// function at the output of the layer below.  Work item = (64 input maps, st.chunk <= 64 input pixels): a lane is an
// input map while it adds, a pixel when it stores.
__device__ void conv_bwd_wepi_item(const LayerDev& L, const LayerDev& Lp, const Stage& st, int item, float* lds) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  constexpr int WAVES = WG / 64;
  const int K = L.K, KP = L.Kp, NW = st.tile_rows, KS = st.rows_per_wg, PB = st.chunk;
  const int RH = KP + K - 1, RW = KP * NW + K - 1, R = RH * RW, Wp = L.Wp, GX = (Wp + NW - 1) / NW, NG = L.Hp * GX;
  const int Mi = L.Mi, Wi = L.Wi, P = L.Hi * Wi;
  const int c = item / st.n_tiles, p0 = (item - c * st.n_tiles) * PB, np = min(PB, P - p0);
  const int i0 = c * 64, n = min(64, Mi - i0);
  if (PB <= WAVES) {   // a pixel a wavefront: its regions one by one, in the fewest instructions (300C3 on 10 x 10: with the
                       // adjustment 9.9 us, 13.5 in the form below, whose code takes longer to come than the loads it saves)
    if (wave < np) {
      const int y = (p0 + wave) / Wi, x = (p0 + wave) - y * Wi;
      const int wy_lo = max(0, (y - RH + KP) / KP), wy_hi = min(L.Hp - 1, y / KP);   // (y - RH + 1 rounded up; y - RH + KP >= 0 or the maximum takes 0)
      const int gx_lo = max(0, (x - RW + KP * NW) / (KP * NW)), gx_hi = min(GX - 1, x / (KP * NW));
      float s = 0.f;
      for (int wy = wy_lo; wy <= wy_hi; ++wy)
        for (int gx = gx_lo; gx <= gx_hi; ++gx) {
          const int col = x - gx * KP * NW;
          if (col >= min(NW, Wp - gx * NW) * KP + K - 1) continue;
          const gfloat* src = L.mm_part + ((size_t)(wy * GX + gx) * R + (y - wy * KP) * RW + col) * Mi + i0 + min(lane, n - 1);
#pragma unroll 8
          for (int k = 0; k < KS; ++k) s += src[(size_t)k * NG * R * Mi];
        }
      lds[wave * 65 + lane] = s;
    }
  } else {
    // The terms of a pixel (its regions row by row, the slices of each) lie NG * R rows of Mi floats and less apart: a lane works out
    // the row of a term.  Those of all the wavefront's pixels are in flight together: one pixel after the other, each region by
    // itself, the loads of 23 x 23 pixels waited some five times (with the adjustment beside them 19.5 us, 16.9 so).
    constexpr int PU = 64 / WAVES, TU = 16, TB = 4;   // pixels of a wavefront, terms of one of them in flight, terms under one branch
    const float by_KS = 1.f / KS;                     // (quotients of whole numbers below 2^16, taken half a step off: exact)
    float s[PU];
    int first[PU], terms[PU], across[PU], t_max = 0;
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int q = wave + u * WAVES, p = p0 + min(q, np - 1), y = p / Wi, x = p - y * Wi;
      const int wy_lo = max(0, (y - RH + KP) / KP), wy_hi = min(L.Hp - 1, y / KP);  
      const int gx_lo = max(0, (x - RW + KP * NW) / (KP * NW));
      int gx_hi = min(GX - 1, x / (KP * NW));
      if (gx_hi == GX - 1 && x - gx_hi * KP * NW >= (Wp - gx_hi * NW) * KP + K - 1) --gx_hi;   // (the last group may be short)
      s[u] = 0.f;
      across[u] = max(0, gx_hi - gx_lo + 1);   // (two at most: a group is at least K - 1 pixels wide)
      terms[u] = q < np ? across[u] * max(0, wy_hi - wy_lo + 1) * KS : 0;
      first[u] = (wy_lo * GX + gx_lo) * R + (y - wy_lo * KP) * RW + x - gx_lo * KP * NW;
      t_max = max(t_max, terms[u]);
    }
    const gfloat* src = L.mm_part + i0 + min(lane, n - 1);
    for (int b = 0; b < t_max; b += 64) {
      int row[PU];
      const int reg = (int)((b + lane + 0.5f) * by_KS), k = b + lane - reg * KS;
#pragma unroll
      for (int u = 0; u < PU; ++u) {
        const int wy = across[u] == 2 ? reg >> 1 : reg, gx = across[u] == 2 ? reg & 1 : 0;
        row[u] = first[u] + wy * (GX * R - KP * RW) + gx * (R - KP * NW) + k * NG * R;
      }
      for (int t0 = 0; t0 < 64 && b + t0 < t_max; t0 += TU) {
        float v[PU][TU];
#pragma unroll
        for (int u = 0; u < PU; ++u)
#pragma unroll
          for (int t = 0; t < TU; t += TB)
            if (b + t0 + t < terms[u]) {
#pragma unroll
              for (int c = t; c < t + TB; ++c)
                v[u][c] = src[(size_t)__builtin_amdgcn_readlane(row[u], min(t0 + c, terms[u] - 1 - b)) * Mi];
            }
#pragma unroll
        for (int u = 0; u < PU; ++u)
#pragma unroll
          for (int t = 0; t < TU; t += TB)
            if (b + t0 + t < terms[u]) {
#pragma unroll
              for (int c = t; c < t + TB; ++c) s[u] += b + t0 + c < terms[u] ? v[u][c] : 0.f;
            }
      }
    }
#pragma unroll
    for (int u = 0; u < PU; ++u)
      if (wave + u * WAVES < np) lds[(wave + u * WAVES) * 65 + lane] = s[u];
  }
  __syncthreads();
  for (int m = wave; m < n; m += WAVES)
    if (lane < np) {
      const size_t o = (size_t)(i0 + m) * P + p0 + lane;
      Lp.delta[o] = lds[lane * 65 + m] * Lp.dact[o];
    }
  __syncthreads();
}

}  // namespace cnn355
