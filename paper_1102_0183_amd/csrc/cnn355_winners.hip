// gfx950: the delta pull through a wide convolutional layer over the pooling winners, a lane per input map.
//
// This file is compiled with the structurizer told to leave uniform branches alone (build.py): every wavefront branches as one on the
// place of a winner, and only as plain jumps do the sums stay in the registers they are in (else each branch ends in
// copies of them: twice the vector instructions, the pull through 500C4 21.6 us instead of 16.1).
#include "cnn355_winners.h"

namespace cnn355 {

// ------------------------------------------------------------------------------------------
// BP through a wide layer (Sec. 3.3; skipping factor 0) over the pooling winners.  A wavefront owns up to NW pooling
// windows side by side, for 64 input maps (a lane each) and some of the output maps.  The winners of those windows reach
// RH x RW input pixels, whose sums a lane keeps in registers: which of them a winner's K x K terms go to is a branch of
// the wavefront (KP * KP places in the window, each with its registers fixed), so a term is one multiply-add with
// the delta in a scalar register, and LDS is not touched until the end.  Work item = (64 input maps, a group of
// windows, slice of the output maps); its wavefronts share the slice, add up in LDS in a fixed order and leave one
// region of partial sums; ST_CONV_BWD_WEPI adds the slices and the regions that overlap.
// Pull through 500C4 on 300 maps of 23 x 23 behind 4 x 4 pooling (1/16 of 0.96 G multiply-adds), in a kernel trace: 16.1 us, 45.9 as a
// matrix product; bound by the issue of the multiply-adds and the branches around them (7.6 us of it) and by the
// latency of a short kernel.  Groups of windows of one slice run on one XCD, whose L2 then holds their filters: 19.2 us else.
// ------------------------------------------------------------------------------------------
// acc += d * w at the K x K pixels of winner `a` (counted row by row from LO) of window `win`
template <int K, int KP, int RW, int LO, int HI, int R>
__device__ __forceinline__ void win_add(float (&acc)[R], const float (&w)[K * K], float d, int a, int win0) {
  if constexpr (HI - LO == 1) {
    constexpr int dy = LO / KP, dx = LO - dy * KP;
    // (a mark of its own at both ends of every branch: the optimiser would else merge the branches into one with
    // an index into the sums, and the sums then lie in scratch memory)
    asm volatile("; winner %0" ::"i"(LO));
#pragma unroll
    for (int ky = 0; ky < K; ++ky)
#pragma unroll
      for (int kx = 0; kx < K; ++kx) {
        float& s = acc[(dy + ky) * RW + win0 + dx + kx];
        s = fmaf(d, w[ky * K + kx], s);
      }
    asm volatile("; winner %0 added" ::"i"(LO));
  } else {
    constexpr int MID = (LO + HI) / 2;
    if (a < MID) win_add<K, KP, RW, LO, MID>(acc, w, d, a, win0);
    else win_add<K, KP, RW, MID, HI>(acc, w, d, a, win0);
  }
}

template <int K, int KP>
__global__ void __launch_bounds__(WIN_BWD_WAVES * 64) k_conv_bwd_win(const ProgramDev* __restrict__ P, int s, StatusDev* status, RunArgs a) {
  constexpr int KK = K * K, NW = win_group(K, KP), RH = KP + K - 1, RW = KP * NW + K - 1, R = RH * RW;
  constexpr int PF = KK > 16 ? 2 : 3, JB = 64 / NW / PF * PF;   // filters in flight; output maps whose winners a register holds
  constexpr int SLOTS = WIN_BWD_WAVES / 2;
  constexpr int LDS = SLOTS * R * 64 > WIN_BWD_WAVES * filters_lds(KK) ? SLOTS * R * 64 : WIN_BWD_WAVES * filters_lds(KK);
  __shared__ __align__(16) float red[LDS];
  const Ctx ctx = make_ctx(*P, a, 0, status);
  const Stage& st = P->stages[s];
  if (st.train_only && !ctx.train) return;
  const LayerDev& L = P->layers[st.layer];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int Mi = L.Mi, Mo = L.Mo, Wp = L.Wp, HW = L.Hp * Wp;
  const int GX = (Wp + NW - 1) / NW, NG = L.Hp * GX, KS = st.rows_per_wg;
  // the groups of windows of a slice read the same filters: from one L2
  const int item = xcd_item(blockIdx.x, gridDim.x);
  const int c = item / (NG * KS), rest = item - c * NG * KS, ks = rest / NG, g = rest - ks * NG;
  const int wy = g / GX, gx = g - wy * GX, n_win = min(NW, Wp - gx * NW);
  const int i0 = c * 64, n = min(64, Mi - i0);
  const int per = (Mo + KS - 1) / KS;
  const int j0 = ks * per + wave, j_hi = min(Mo, (ks + 1) * per);
  const int nj = j0 < j_hi ? (j_hi - j0 + WIN_BWD_WAVES - 1) / WIN_BWD_WAVES : 0;   // output maps j0, j0 + 8, ...

  float acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.f;
  if (nj > 0) {
    const gfloat* wbase = L.w + (size_t)i0 * KK;
    float* const turn = red + wave * filters_lds(KK);
    float w[PF][KK];
#pragma unroll
    for (int u = 0; u < PF; ++u) load_raw<KK>(w[u], wbase + (size_t)(j0 + min(u, nj - 1) * WIN_BWD_WAVES) * Mi * KK, n);
    for (int jb = 0; jb < nj; jb += JB) {
      float d;
      int at;
      {  // lane jj * NW + window: the delta and the place of the winner of output map jb + jj
        const int jj = lane / NW, win = lane - jj * NW;
        const size_t o = (size_t)(j0 + min(jb + jj, nj - 1) * WIN_BWD_WAVES) * HW + wy * Wp + gx * NW + min(win, n_win - 1);
        d = L.delta[o];
        at = L.arg[o];
      }
      for (int u0 = 0; u0 < JB && jb + u0 < nj; u0 += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
          if (jb + u0 + u < nj) {
            float f[KK];
            raw_to_filter<KK>(f, w[u], turn);
            load_raw<KK>(w[u], wbase + (size_t)(j0 + min(jb + u0 + u + PF, nj - 1) * WIN_BWD_WAVES) * Mi * KK, n);
#pragma unroll
            for (int win = 0; win < NW; ++win)
              if (win < n_win)
                win_add<K, KP, RW, 0, KP * KP>(acc, f, lane_value(d, (u0 + u) * NW + win),
                                               __builtin_amdgcn_readlane(at, (u0 + u) * NW + win), win * KP);
          }
        }
      }
    }
  }
  // the wavefronts' sums: the upper half hands its own to the lower half, then every thread adds what is left
  __syncthreads();   // (the filters are done with)
  float* mine = red + (wave & (SLOTS - 1)) * (R * 64) + lane;
  if (wave >= SLOTS) {
#pragma unroll
    for (int r = 0; r < R; ++r) mine[r * 64] = acc[r];
  }
  __syncthreads();
  if (wave < SLOTS) {
#pragma unroll
    for (int r = 0; r < R; ++r) mine[r * 64] += acc[r];
  }
  __syncthreads();
  const int cols = n_win * KP + K - 1;
  gfloat* out = L.mm_part + (size_t)(ks * NG + g) * R * Mi + i0 + lane;
  for (int r = wave; r < R; r += WIN_BWD_WAVES) {
    if (r % RW >= cols) continue;
    const float* q = red + r * 64 + lane;
    const float v = (q[0] + q[R * 64]) + (q[2 * R * 64] + q[3 * R * 64]);
    if (lane < n) out[(size_t)r * Mi] = v;
  }
}

template <int K>
static const void* of_window(int KP) {
  switch (KP) {
    case 2: return (const void*)k_conv_bwd_win<K, 2>;
    case 3: return (const void*)k_conv_bwd_win<K, 3>;
    case 4: return (const void*)k_conv_bwd_win<K, 4>;
    default: return nullptr;
  }
}
// the kernel for a kernel size and a pooling window (null: none compiled), the threads of its workgroup
const void* conv_bwd_win_kernel(int K, int KP, int* threads) {
  *threads = WIN_BWD_WAVES * 64;
  switch (K) {
    case 3: return of_window<3>(KP);
    case 4: return of_window<4>(KP);
    case 5: return of_window<5>(KP);
    default: return nullptr;
  }
}
int conv_bwd_win_group(int K, int KP) { return win_group(K, KP); }

}  // namespace cnn355
