// Batched forward propagation (Sec. 3.2 for many images at once): validation and test passes
// change no weight (Sec. 4), so their images are independent and every layer becomes one dense
// matrix product over the whole batch,
//     sums[j][n] = sum_k  Wt[k][j] * X[k][n],     n = (image b, output pixel p),  k = (input map i, ky, kx),
// which is what the matrix cores are for.  X is never formed: its element is
// in[b][i][(y (S+1) + ky)][(x (S+1) + kx)], read from the images staged in LDS at offset
// koff(k) + pbase(n).  A fully connected layer is the same product with 1 x 1 maps and K = 1.
// fp32 operands and fp32 accumulation (v_mfma_f32_32x32x2_f32): the results stay within the
// tolerance of the one-image path.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#define CNN_GLOBAL __attribute__((address_space(1)))
#include "cnn355_dev.h"

namespace cnn355 {

typedef const CNN_GLOBAL float* cgf;
typedef CNN_GLOBAL float* gf;
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

namespace {

constexpr int BT = 256;        // threads of a GEMM workgroup: four wavefronts, 32 columns each
constexpr int BCOLS = 128;     // columns (image, pixel) of a workgroup

// scaled tanh 1.7159 tanh(0.6666 a) (Sec. 4) as A (1 - 2 / (e^{2 B a} + 1)) on the hardware
// exponential and reciprocal: absolute error about 3e-7; below |B a| = 0.3 the odd series of tanh up to x^9
// (5e-8 of the result there), so that small activations keep their digits
__device__ __forceinline__ float b_act(float a) {
  const float z = __builtin_amdgcn_exp2f((2.0f * 0.6666f * 1.44269504088896340736f) * a);
  const float big = 1.7159f - (2.0f * 1.7159f) * __builtin_amdgcn_rcpf(z + 1.0f);
  const float x = 0.6666f * a, x2 = x * x;
  float p = fmaf(x2, 62.0f / 2835.0f, -17.0f / 315.0f);
  p = fmaf(x2, p, 2.0f / 15.0f);
  p = fmaf(x2, p, -1.0f / 3.0f);
  const float small = 1.7159f * fmaf(x, x2 * p, x);
  return fabsf(x) < 0.3f ? small : big;
}

constexpr int PRE_IN = 16;     // floats per thread a prefetched chunk may hold: staged images ...
constexpr int PRE_W = 48;      // ... and rows of Wt

__host__ __device__ __forceinline__ int batch_slot(int IC, int HiWi) { return HiWi == 1 ? IC | 1 : IC * HiWi; }

// Workgroup (x, y): columns [128 x, 128 x + 128) and map tiles [MT y, MT y + MT) of TR maps each.  TR = 32:
// v_mfma_f32_32x32x2_f32, a wavefront's 32 columns are one tile wide, a lane takes the even or the odd k.  TR = 16:
// v_mfma_f32_16x16x4_f32, the 32 columns are two tiles of 16, a lane takes one k in four; it is chosen where 16-row
// tiles pad fewer maps (40 maps: 48 rows instead of 64).
// Every wavefront owns 32 columns and all MT map tiles, so one operand fetched from the staged
// images feeds MT matrix instructions.  The k range is walked in chunks of IC input maps: the
// chunk's maps of every image the columns touch, and the chunk's rows of Wt, are staged in LDS.
// With g.prefetch the next chunk is fetched into registers while the matrix cores work on the
// present one (global latency hidden behind arithmetic); the host sets it only when a chunk
// fits the register budget (PRE_IN, PRE_W floats per thread).
template <int MT, int TR>
__global__ void __launch_bounds__(BT) k_batch_gemm(BatchGemm g) {
  extern __shared__ float lds[];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  constexpr int KS = TR == 32 ? 2 : 4;             // k values one instruction takes, one per group of 64 / KS lanes
  constexpr int CT = 32 / TR;                      // column tiles of a wavefront
  constexpr int AV = TR == 32 ? 16 : 4;            // accumulator floats per lane and tile
  const int lrow = lane & (TR - 1), lk = lane / TR;
  const int HiWi = g.Hi * g.Wi, KK = g.K * g.Kx;
  // floats of a staged image; odd for one-pixel maps (fully connected layers), whose IC is a power of two: the 32 columns
  // of an operand, an image each, would all lie in one bank (360 -> 150 units of 4096 images 30.5 -> 25 us)
  const int slot_sz = batch_slot(g.IC, HiWi);
  const int KC = g.IC * KK;                        // k per full chunk
  constexpr int WROW = MT * TR;
  float* lds_in = lds;                              // [n_img_max][IC][Hi*Wi]
  float* lds_w = lds + ((g.n_img_max * slot_sz + 3) & ~3);  // [KC + 1][MT * 32]; the row behind the last is zero
  // byte offset of k inside a staged image, the k of every residue mod KS apart so that a lane (which takes the
  // k of its own residue) finds the four it needs next to each other: [KS][KH], KH a multiple of 4
  const int KH = (((KC + KS - 1) / KS) + 3) & ~3;
  int* koff = (int*)(lds_w + (KC + 1) * WROW);

  // (columns are counted in 32 bits: the host keeps batch * P below 2^31)
  const int N = (int)g.N;
  const int n0 = blockIdx.x * BCOLS;
  const int mt0 = blockIdx.y * MT;                 // first tile (of TR maps) of the workgroup
  const int b_lo = n0 / g.P;
  const int n_last = min(n0 + BCOLS, N) - 1;
  const int n_img = n_last / g.P - b_lo + 1;

  for (int x = tid; x < KS * KH; x += BT) {
    const int par = x / KH, h = x - par * KH;
    const int k = min(KS * h + par, KC - 1);
    const int c = k / KK, t = k - c * KK;
    const int ky = t / g.Kx, kx = t - ky * g.Kx;
    koff[x] = (c * HiWi + ky * g.Wi + kx) * 4;
  }
  // the lane's column in each of the wavefront's column tiles
  bool col_ok[CT];
  int cb[CT], cp[CT], pbase[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int n = n0 + wave * 32 + ct * TR + lrow;
    col_ok[ct] = n < N;
    cb[ct] = 0; cp[ct] = 0; pbase[ct] = 0;
    if (col_ok[ct]) {
      cb[ct] = n / g.P;
      cp[ct] = n - cb[ct] * g.P;
      const int y = cp[ct] / g.Wo, x = cp[ct] - y * g.Wo;
      pbase[ct] = (cb[ct] - b_lo) * slot_sz + y * (g.Kp * g.stride) * g.Wi + x * (g.Kpx * g.stride_x);
    }
  }
  typedef float accv __attribute__((ext_vector_type(AV)));
  accv acc[MT][CT], best[MT][CT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int v = 0; v < AV; ++v) { acc[m][ct][v] = 0.f; best[m][ct][v] = -INFINITY; }

  // Element e of a chunk's staged images is float x of image slot s, e = s * cnt + x, where
  // cnt = n_ic * Hi * Wi is the run of contiguous floats the chunk takes from one image; a thread
  // walks e = tid, tid + BT, ... and keeps (s, x) by carrying instead of dividing.  Element e of
  // the chunk's weights is Wt[ic0 * KK + e / WROW][mt0 * 32 + e % WROW], WROW a power of two.
  struct Walk {
    int s, x, cnt, sh;   // sh >= 0: cnt == 1 << sh
    __device__ __forceinline__ Walk(int tid, int cnt_) : cnt(cnt_) {
      sh = (cnt_ & (cnt_ - 1)) == 0 ? __ffs(cnt_) - 1 : -1;
      s = sh >= 0 ? tid >> sh : tid / cnt_;
      x = tid - s * cnt_;
    }
    __device__ __forceinline__ void step() {
      x += BT;
      if (sh >= 0) { s += x >> sh; x &= cnt - 1; }
      else while (x >= cnt) { x -= cnt; ++s; }
    }
  };
  // addresses as a uniform base plus a 32-bit offset per lane (the host keeps every array the
  // kernel indexes this way below 2^31 floats)
  const cgf in0 = g.in + (long long)b_lo * g.in_stride;
  const unsigned in_stride32 = (unsigned)g.in_stride;
  auto in_ptr = [&](int ic0, const Walk& w, bool ok) -> cgf {
    return in0 + ic0 * HiWi + (ok ? (unsigned)w.s * in_stride32 + (unsigned)w.x : 0u);
  };
  // four weights at a time: rows of Wt and of the staged copy start on 128-byte boundaries
  auto w_val = [&](int ic0, int kc, int e4) -> v4f {
    const int kr = e4 / (WROW / 4), c = (e4 - kr * (WROW / 4)) * 4;
    if (kr >= kc) return v4f{0.f, 0.f, 0.f, 0.f};
    return *(const CNN_GLOBAL v4f*)(g.wt + ((long long)ic0 * KK * g.MoPad + mt0 * TR) + (unsigned)(kr * g.MoPad + c));
  };
  // straight to LDS, eight loads in flight per thread (first chunk, and every chunk without prefetch)
  auto stage_now = [&](int ic0) {
    const int n_ic = min(g.IC, g.Mi - ic0);
    const int cnt = n_ic * HiWi, tot = n_img * cnt;
    Walk w(tid, cnt);
    for (int e0 = 0; e0 < tot; e0 += 8 * BT) {
      float v[8];
      int d[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool ok = e0 + u * BT + tid < tot;
        v[u] = *in_ptr(ic0, w, ok);
        d[u] = ok ? w.s * slot_sz + w.x : -1;
        w.step();
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (d[u] >= 0) lds_in[d[u]] = v[u];
    }
    const int kc = n_ic * KK, wtot = (kc + 1) * (WROW / 4);
    for (int e0 = 0; e0 < wtot; e0 += 4 * BT) {
      v4f v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = w_val(ic0, kc, min(e0 + u * BT + tid, wtot - 1));
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (e0 + u * BT + tid < wtot) ((v4f*)lds_w)[e0 + u * BT + tid] = v[u];
    }
  };
  float ri[PRE_IN];
  v4f rw[PRE_W / 4];
  auto fetch = [&](int ic0) {
    const int n_ic = min(g.IC, g.Mi - ic0);
    const int cnt = n_ic * HiWi, tot = n_img * cnt;
    Walk w(tid, cnt);
#pragma unroll
    for (int u = 0; u < PRE_IN; ++u) {
      ri[u] = *in_ptr(ic0, w, u * BT + tid < tot);
      w.step();
    }
    const int kc = n_ic * KK, wtot = (kc + 1) * (WROW / 4);
#pragma unroll
    for (int u = 0; u < PRE_W / 4; ++u)
      rw[u] = (u * BT < wtot) ? w_val(ic0, kc, min(u * BT + tid, wtot - 1)) : v4f{0.f, 0.f, 0.f, 0.f};
  };
  auto put = [&](int ic0) {
    const int n_ic = min(g.IC, g.Mi - ic0);
    const int cnt = n_ic * HiWi, tot = n_img * cnt;
    Walk w(tid, cnt);
#pragma unroll
    for (int u = 0; u < PRE_IN; ++u) {
      if (u * BT + tid < tot) lds_in[w.s * slot_sz + w.x] = ri[u];
      w.step();
    }
    const int wtot = (n_ic * KK + 1) * (WROW / 4);
#pragma unroll
    for (int u = 0; u < PRE_W / 4; ++u)
      if (u * BT + tid < wtot) ((v4f*)lds_w)[u * BT + tid] = rw[u];
  };

  // slice blockIdx.z of the k range: chunks [z * cps, (z + 1) * cps)
  const int ic_first = blockIdx.z * g.chunks_per_slice * g.IC;
  const int ic_end = min(g.Mi, ic_first + g.chunks_per_slice * g.IC);
  for (int ic0 = ic_first; ic0 < ic_end; ic0 += g.IC) {
    const int n_ic = min(g.IC, g.Mi - ic0);
    const int kc = n_ic * KK;
    if (ic0 == ic_first || !g.prefetch) stage_now(ic0);
    else put(ic0);
    __syncthreads();
    if (g.prefetch && ic0 + g.IC < ic_end) fetch(ic0 + g.IC);
    // Members of the pooling window, one after the other (one member, the pixel itself, without
    // pooling; with it the host has made the k range a single chunk, so a member's sums are
    // complete when its loop ends).
    for (int d = 0; d < g.Kp * g.Kpx; ++d) {
      const int dy = d / g.Kpx, dx = d - dy * g.Kpx;
      const int pd = dy * g.stride * g.Wi + dx * g.stride_x;
      // KS k per instruction (lanes 0 .. 64/KS - 1 the first, and so on); the operands of four instructions per
      // tile are fetched together.  Whole groups of 4 KS k first, without any clamping; then the tail, where k
      // beyond the chunk meets the zero row of Wt.
      const char* in_b[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) in_b[ct] = (const char*)lds_in + (pbase[ct] + pd) * 4;
#define CNN355_MAC(a, bv)                                                                                            \
  _Pragma("unroll") for (int u = 0; u < 4; ++u)                                                                      \
  _Pragma("unroll") for (int m = 0; m < MT; ++m)                                                                     \
  _Pragma("unroll") for (int ct = 0; ct < CT; ++ct) {                                                                \
    if constexpr (TR == 32) acc[m][ct] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][m], bv[u][ct], acc[m][ct], 0, 0, 0); \
    else acc[m][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][m], bv[u][ct], acc[m][ct], 0, 0, 0);                  \
  }
      constexpr int KG = 4 * KS;
      const int kcg = kc - kc % KG;
      for (int kk = 0; kk < kcg; kk += KG) {
        const int4 ko = *(const int4*)(koff + lk * KH + kk / KS);
        const float* wr = lds_w + (kk + lk) * WROW + lrow;
        float a[4][MT], bv[4][CT];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int m = 0; m < MT; ++m) a[u][m] = wr[KS * u * WROW + m * TR];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          bv[0][ct] = *(const float*)(in_b[ct] + ko.x);
          bv[1][ct] = *(const float*)(in_b[ct] + ko.y);
          bv[2][ct] = *(const float*)(in_b[ct] + ko.z);
          bv[3][ct] = *(const float*)(in_b[ct] + ko.w);
        }
        CNN355_MAC(a, bv)
      }
      if (kcg < kc) {
        float a[4][MT], bv[4][CT];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = kcg + KS * u + lk;
          const int kr = min(k, kc);               // row kc is the zero row
          const int ko = koff[lk * KH + min(k / KS, KH - 1)];
#pragma unroll
          for (int m = 0; m < MT; ++m) a[u][m] = lds_w[kr * WROW + m * TR + lrow];
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {   // (k beyond the chunk: nothing was staged there, and no number times zero is none)
            const float t = *(const float*)(in_b[ct] + ko);
            bv[u][ct] = k < kc ? t : 0.f;
          }
        }
        CNN355_MAC(a, bv)
      }
#undef CNN355_MAC
      if (g.Kp * g.Kpx > 1) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int v = 0; v < AV; ++v) {
              best[m][ct][v] = fmaxf(best[m][ct][v], acc[m][ct][v]);
              acc[m][ct][v] = 0.f;
            }
      }
    }
    __syncthreads();
  }
  // element v of a lane, 32-row tiles: row (v / 4) * 8 + (lane / 32) * 4 + v % 4 of the tile, column lane % 32;
  // 16-row tiles: row (lane / 16) * 4 + v, column lane % 16
  gf dst = g.out + (long long)blockIdx.z * g.slice_stride;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    if (!col_ok[ct]) continue;
    const unsigned o0 = (unsigned)cb[ct] * (unsigned)g.out_stride + (unsigned)cp[ct];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int v = 0; v < AV; ++v) {
        const int j = (mt0 + m) * TR + (TR == 32 ? (v >> 2) * 8 + lk * 4 + (v & 3) : lk * 4 + v);
        if (j < g.Mo) {
          float sv = (g.Kp * g.Kpx > 1) ? best[m][ct][v] : acc[m][ct][v];
          if (g.fuse) sv += g.bias[j];
          if (g.fuse == 1) sv = b_act(sv);
          dst[o0 + (unsigned)j * (unsigned)g.P] = sv;
        }
      }
  }
}

// ---- a convolutional layer of a whole batch -------------------------------------------------------------------
// The same product with everything between the arithmetic taken out of its way:
//  * The next chunk (input maps, rows of Wt) goes straight to the other half of LDS (global_load_lds: no registers, no
//    instructions to store it) while the matrix cores work on the present one; one barrier a chunk.
//  * A workgroup is persistent: it takes column blocks blockIdx.x, + gridDim.x, ..., and fetches the next block's first
//    chunk during the last of this one.  Where the k range is one chunk the weights are staged once and stay.
//  * Up to 160 maps a workgroup (MT tiles of TR): one operand of the staged images feeds MT matrix instructions.
//  * Pooling: the columns are (image, window, member of the window), so a window's sums lie side by side in one
//    accumulator register of adjacent lanes.  2 x 2 windows are four lanes, reduced by DPP, each lane going on with one
//    row in four (bias, tanh and store at full lanes); others pass through LDS tile by tile.  The full-resolution sums
//    never reach memory, however long the k range.
// Bound by the matrix pipes in layers with a long k range: busy 73 % of the time in 300C2, 78 in 300C4, 66 in 40C5 (at the
// 2.1 GHz the chip keeps there); staging is hidden in them (without it the products take as long), the rest is blocks that
// do not divide evenly.  First layers (k of 16 or 27) by the epilogue's vector instructions: 300C3 38 % and 42 % of the
// vector issue, 20C4 27 and 61.  Per 512 images of 300 maps, under the tracer: 300C3 on 3 maps 206 -> 183 us, 300C2 on 300
// maps with its pooling 1286 + 45 -> 772 us (94 TFLOP/s), 300C4 405 -> 235 us; 4096 digits: 20C4 83 -> 76 us, 40C5 243 + 24
// -> 183 us (73 TFLOP/s).  Tried and not kept: the next group's operands in a second set of registers (300C2 794 -> 852
// us), all of a group's LDS reads before its first product (833), three or four workgroups a compute unit (795, 791).
// Layout of dynamic LDS: [1 or 2][KC][MT * TR] weights, [2][n_img_max][slot] images, koff, biases, [TR][EP] sums of one tile.
constexpr int EP = 132;

__device__ __forceinline__ int fast_div(int n, FastDiv d) { return (int)(__umulhi(2u * (unsigned)n, d.m) >> d.s); }

// Lane l's 4 or 16 bytes at base + off go to lds_byte + 4 l or 16 l; the wavefront has them after s_waitcnt vmcnt(0).
// (Not the builtin: the compiler then waits for the load before every LDS read that it cannot tell apart from its
// destination.)
// lds_byte and base are the same for the whole wavefront; the wait in front is what an address fresh from a vector
// instruction needs.
__device__ __forceinline__ const CNN_GLOBAL char* uniform(const CNN_GLOBAL char* p) {
  const unsigned long long v = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return (const CNN_GLOBAL char*)(((unsigned long long)hi << 32) | lo);
}
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // (m0 is a reserved register: nothing else would say that it is written)
__device__ __forceinline__ void lds_dma4(unsigned lds_byte, const CNN_GLOBAL char* base, unsigned off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dword %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(lds_byte)),
               "v"(off), "s"(uniform(base)) : "memory", "m0");
}
__device__ __forceinline__ void lds_dma16(unsigned lds_byte, const CNN_GLOBAL char* base, unsigned off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(__builtin_amdgcn_readfirstlane(lds_byte)),
               "v"(off), "s"(uniform(base)) : "memory", "m0");
}
#pragma clang diagnostic pop

template <int MT, int TR>
__global__ void __launch_bounds__(BT, MT * TR > 96 ? 2 : 3) k_batch_conv(BatchConv g) {
  extern __shared__ __align__(16) float lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int KS = TR == 32 ? 2 : 4;             // k values one instruction takes, one per group of 64 / KS lanes
  constexpr int CT = 32 / TR;                      // column tiles of a wavefront
  constexpr int AV = TR == 32 ? 16 : 4;            // accumulator floats per lane and tile
  constexpr int WROW = MT * TR;
  const int lrow = lane & (TR - 1), lk = lane / TR;
  const int HiWi = g.Hi * g.Wi, KK = g.K * g.Kx, KC = g.IC * KK;
  const int w_size = (KC * WROW + 255) & ~255, in_size = g.n_img_max * g.slot;
  float* lds_w = lds;
  float* lds_in = lds_w + (g.resident ? 1 : 2) * w_size;
  const int KH = (((KC + KS - 1) / KS) + 3) & ~3;
  int* koff = (int*)(lds_in + 2 * in_size);        // [KS][KH] byte offset of k inside a staged image
  float* lds_b = (float*)(koff + KS * KH);         // [MT * TR] biases
  float* ep = lds_b + WROW;
  const unsigned w_byte = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)lds_w;
  const unsigned in_byte = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float*)lds_in;
  for (int x = tid; x < KS * KH; x += BT) {
    const int par = x / KH, h = x - par * KH;
    const int k = min(KS * h + par, KC - 1);
    const int c = k / KK, t = k - c * KK;
    const int ky = t / g.Kx, kx = t - ky * g.Kx;
    koff[x] = (c * HiWi + ky * g.Wi + kx) * 4;
  }
  const int j0 = blockIdx.y * WROW;
  for (int x = tid; x < WROW; x += BT) lds_b[x] = g.fuse && j0 + x < g.Mo ? g.bias[j0 + x] : 0.f;
  const int ic_first = blockIdx.z * g.run;
  const int ic_end = min(g.Mi, ic_first + g.run);
  const int M = g.Kp * g.Kpx;
  // a column block's first and last image
  auto first_image = [&](int cb) { return fast_div(cb * g.wins, g.by_win_img); };
  auto last_image = [&](int cb) { return fast_div(min((cb + 1) * g.wins, g.n_win) - 1, g.by_win_img); };
  // A wavefront takes every fourth run of 64 lanes, of a float each, or of four where every image and chunk starts on 16
  // bytes (g.vec); lanes behind the last element of a map or group fetch nothing.
  auto fetch = [&](int b0, int b1, int ic0, int buf, bool with_w) {
    const int n_ic = min(g.IC, ic_end - ic0), cnt = n_ic * HiWi;
    const int run = g.vec ? 256 : 64;
    const CNN_GLOBAL char* base = (const CNN_GLOBAL char*)(g.in + (long long)b0 * g.in_stride + ic0 * HiWi + wave * run);
    unsigned dst = in_byte + (unsigned)(buf * in_size + wave * run) * 4u;
    const unsigned whole = (unsigned)lane * 4u;
    for (int s = b0; s <= b1; ++s, base += g.in_stride * 4, dst += (unsigned)g.slot * 4u) {
      const CNN_GLOBAL char* p = base;
      unsigned d = dst;
      int left = cnt - wave * run;
      if (g.vec) {
        for (; left >= 256; left -= 4 * BT, p += BT * 16, d += BT * 16u) lds_dma16(d, p, whole * 4u);
        if (left > 0) {
          if (lane * 4 + 4 <= left) lds_dma16(d, p, whole * 4u);
          const unsigned q = (unsigned)(left & ~3) * 4u;
          if (lane < (left & 3)) lds_dma4(d + q, p, q + whole);
        }
      } else {
        for (; left >= 64; left -= BT, p += BT * 4, d += BT * 4u) lds_dma4(d, p, whole);
        if (lane < left) lds_dma4(d, p, whole);
      }
    }
    if (!with_w) return;
    const CNN_GLOBAL char* wb = (const CNN_GLOBAL char*)(g.wt + ((long long)blockIdx.y * g.k_total + ic0 * KK) * WROW + wave * 256);
    const int n_w = n_ic * KK * WROW;   // a multiple of 16
    unsigned wdst = w_byte + (unsigned)((g.resident ? 0 : buf) * w_size + wave * 256) * 4u;
    int x = wave * 256;
    for (; x + 256 <= n_w; x += 4 * BT, wb += 16 * BT, wdst += 16u * BT) lds_dma16(wdst, wb, whole * 4u);
    if (lane * 4 < n_w - x) lds_dma16(wdst, wb, whole * 4u);
  };

  typedef float accv __attribute__((ext_vector_type(AV)));
  int buf = 0;
  int b0 = first_image(blockIdx.x), b1 = last_image(blockIdx.x);
  fetch(b0, b1, ic_first, 0, true);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  for (int cb = blockIdx.x; cb < g.n_cb; cb += gridDim.x) {
    // the lane's column in each of the wavefront's column tiles
    int pbase[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const int c = wave * 32 + ct * TR + lrow;
      const int wl = c / M, d = c - wl * M, w = cb * g.wins + wl;
      pbase[ct] = 0;
      if (wl < g.wins && w < g.n_win) {
        const int b = fast_div(w, g.by_win_img), wi = w - b * g.win_img;
        const int wy = fast_div(wi, g.by_wp), wx = wi - wy * g.Wp, dy = d / g.Kpx, dx = d - dy * g.Kpx;
        pbase[ct] = ((b - b0) * g.slot + (wy * g.Kp + dy) * g.stride * g.Wi + (wx * g.Kpx + dx) * g.stride_x) * 4;
      }
    }
    accv acc[MT][CT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int v = 0; v < AV; ++v) acc[m][ct][v] = 0.f;
    const int cb_b0 = b0;
    for (int ic0 = ic_first; ic0 < ic_end; ic0 += g.IC, buf ^= 1) {
      // the chunk has arrived (every wavefront has waited for its own loads), and nobody reads the other half any more
      __syncthreads();
      if (ic0 + g.IC < ic_end) {
        fetch(b0, b1, ic0 + g.IC, buf ^ 1, true);
      } else if (cb + (int)gridDim.x < g.n_cb) {
        b0 = first_image(cb + gridDim.x);
        b1 = last_image(cb + gridDim.x);
        fetch(b0, b1, ic_first, buf ^ 1, !g.resident);
      }
      const int kc = min(g.IC, ic_end - ic0) * KK;
      const char* in_b[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) in_b[ct] = (const char*)(lds_in + buf * in_size) + pbase[ct];
      const float* w_b = lds_w + (g.resident ? 0 : buf) * w_size;
#define CNN355_MAC(a, bv)                                                                                            \
  _Pragma("unroll") for (int u = 0; u < 4; ++u)                                                                      \
  _Pragma("unroll") for (int m = 0; m < MT; ++m)                                                                     \
  _Pragma("unroll") for (int ct = 0; ct < CT; ++ct) {                                                                \
    if constexpr (TR == 32) acc[m][ct] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][m], bv[u][ct], acc[m][ct], 0, 0, 0); \
    else acc[m][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][m], bv[u][ct], acc[m][ct], 0, 0, 0);                  \
  }
      constexpr int KG = 4 * KS;
      const int kcg = kc - kc % KG;
      for (int kk = 0; kk < kcg; kk += KG) {
        const int4 ko = *(const int4*)(koff + lk * KH + kk / KS);
        const float* wr = w_b + (kk + lk) * WROW + lrow;
        float a[4][MT], bv[4][CT];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int m = 0; m < MT; ++m) a[u][m] = wr[KS * u * WROW + m * TR];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          bv[0][ct] = *(const float*)(in_b[ct] + ko.x);
          bv[1][ct] = *(const float*)(in_b[ct] + ko.y);
          bv[2][ct] = *(const float*)(in_b[ct] + ko.z);
          bv[3][ct] = *(const float*)(in_b[ct] + ko.w);
        }
        CNN355_MAC(a, bv)
      }
      if (kcg < kc) {   // the rest of the chunk: k beyond it counts as zero on both sides
        float a[4][MT], bv[4][CT];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = kcg + KS * u + lk, kr = min(k, kc - 1);
          const int ko = koff[lk * KH + min(k / KS, KH - 1)];
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            const float t = w_b[kr * WROW + m * TR + lrow];
            a[u][m] = k < kc ? t : 0.f;
          }
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            const float t = *(const float*)(in_b[ct] + (k < kc ? ko : 0));
            bv[u][ct] = k < kc ? t : 0.f;
          }
        }
        CNN355_MAC(a, bv)
      }
#undef CNN355_MAC
      // here and not behind the barrier: the wait would take in the stores of the results (and those read no memory
      // themselves, biases are in LDS: a load's wait takes in the stores before it too)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    // element v of a lane, 32-row tiles: row (v / 4) * 8 + (lane / 32) * 4 + v % 4 of the tile, column lane % 32;
    // 16-row tiles: row (lane / 16) * 4 + v, column lane % 16
    gf dst = g.out + (long long)blockIdx.z * g.slice_stride;
    auto finish = [&](float sv, int j) {
      if (g.fuse) sv += lds_b[j - j0];
      return g.fuse == 1 ? b_act(sv) : sv;
    };
    if (M == 1 || M == 4) {
      const int q = M == 4 ? lane & 3 : 0;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int c = wave * 32 + ct * TR + lrow;
        const int w = cb * g.wins + (M == 4 ? c >> 2 : c);
        const bool ok = w < g.n_win;
        const int b = ok ? fast_div(w, g.by_win_img) : cb_b0, wi = ok ? w - b * g.win_img : 0;
        const unsigned o0 = (unsigned)b * (unsigned)g.out_stride + (unsigned)wi;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          if (M == 4) {
#pragma unroll
            for (int v4 = 0; v4 < AV; v4 += 4) {
              if (j0 + m * TR + v4 * 2 >= g.Mo) break;   // (TR = 16: v4 is 0)
              float r[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                float x = acc[m][ct][v4 + u];
                x = fmaxf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xf, 0xf, true)));   // lanes 1 0 3 2
                r[u] = fmaxf(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4E, 0xf, 0xf, true)));  // 2 3 0 1
              }
              const float mine = fmaxf(q < 2 ? (q == 0 ? r[0] : r[1]) : (q == 2 ? r[2] : r[3]), -INFINITY);  // (no number at all: -inf)
              const int j = j0 + m * TR + (TR == 32 ? (v4 >> 2) * 8 : 0) + lk * 4 + q;
              if (ok && j < g.Mo) dst[o0 + (unsigned)j * (unsigned)g.win_img] = finish(mine, j);
            }
          } else {
#pragma unroll
            for (int v = 0; v < AV; ++v) {
              const int j = j0 + m * TR + (TR == 32 ? (v >> 2) * 8 + lk * 4 + (v & 3) : lk * 4 + v);
              if (ok && j < g.Mo) dst[o0 + (unsigned)j * (unsigned)g.win_img] = finish(acc[m][ct][v], j);
            }
          }
        }
      }
    } else {
      // a thread's window stays its own for all rows it takes
      const int rows = BT / g.wins, jr = tid / g.wins, wl = tid - jr * g.wins;
      const int w = cb * g.wins + wl;
      const bool ok = jr < rows && w < g.n_win;
      const int b = ok ? fast_div(w, g.by_win_img) : cb_b0, wi = ok ? w - b * g.win_img : 0;
      const unsigned o0 = (unsigned)b * (unsigned)g.out_stride + (unsigned)wi;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        __syncthreads();   // the previous tile has been read
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int v = 0; v < AV; ++v)
            ep[(TR == 32 ? (v >> 2) * 8 + lk * 4 + (v & 3) : lk * 4 + v) * EP + wave * 32 + ct * TR + lrow] = acc[m][ct][v];
        __syncthreads();
        if (ok)
          for (int r = jr; r < TR; r += rows) {
            const int j = j0 + m * TR + r;
            if (j >= g.Mo) break;
            const float* win = ep + r * EP + wl * M;
            float best = -INFINITY;
            for (int d = 0; d < M; ++d) best = fmaxf(best, win[d]);
            dst[o0 + (unsigned)j * (unsigned)g.win_img] = finish(best, j);
          }
      }
    }
  }
}

// the planes of partial sums of one output, added in their order, up to eight loads in flight
__device__ __forceinline__ float add_planes(cgf p, int n, long long stride) {
  if (n == 1) return 0.f + p[0];
  float v = 0.f;
  for (int s0 = 0; s0 < n; s0 += 8) {
    float t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (s0 + u < n) t[u] = p[(long long)(s0 + u) * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (s0 + u < n) v += t[u];
  }
  return v;
}

// bias + scaled tanh + max-pooling (Sec. 2.2, 2.3) of the raw sums of a whole batch; the sums may
// come as several planes (slices of the k range), added here in a fixed order.  The activation
// function is increasing, so the maximum is taken first: one tanh per window.  act 0: none (the
// output layer's sums go on to the output units).
__global__ void __launch_bounds__(256) k_batch_pool(BatchPool q) {
  const long long x = (long long)blockIdx.x * 256 + threadIdx.x;
  if (x >= q.total) return;
  const int HpWp = q.Hp * q.Wp;
  const long long bj = x / HpWp;
  const int w = (int)(x - bj * HpWp);
  const int j = (int)(bj % q.Mo);
  const int py = w / q.Wp, px = w - py * q.Wp;
  cgf src = q.sums + bj * ((long long)q.Ho * q.Wo) + (py * q.Kp) * q.Wo + px * q.Kpx;
  float best = -INFINITY;
  for (int dy = 0; dy < q.Kp; ++dy)
    for (int dx = 0; dx < q.Kpx; ++dx) {
      const float v = add_planes(src + dy * q.Wo + dx, q.n_slices, q.slice_stride);
      best = fmaxf(best, v);
    }
  best += q.bias[j];
  q.out[x] = q.act ? b_act(best) : best;
}

// Output units of a whole batch: soft-max of the output layer's sums (as n_slices planes without the bias, or one with
// it: bias null), or the scaled tanh for the variant with tanh output neurons.  One thread per image.
__global__ void __launch_bounds__(256) k_batch_outputs(cgf sums, int n_slices, long long slice_stride, cgf bias, gf probs,
                                                       long long n_images, int n_classes, int out_units) {
  const long long b = (long long)blockIdx.x * 256 + threadIdx.x;
  if (b >= n_images) return;
  cgf a = sums + b * n_classes;
  gf o = probs + b * n_classes;
  cgf v = a;
  if (bias || out_units == 1) {
    for (int k = 0; k < n_classes; ++k) {
      const float x = bias ? fmaxf(add_planes(a + k, n_slices, slice_stride), -INFINITY) + bias[k] : a[k];
      o[k] = out_units == 1 ? b_act(x) : x;
    }
    if (out_units == 1) return;
    v = o;
  }
  // (sums that are there already are read where they are: through the outputs, 1000 classes took 1.25 times as long)
  float mx = v[0];
  for (int k = 1; k < n_classes; ++k) mx = fmaxf(mx, v[k]);
  float z = 0.f;
  for (int k = 0; k < n_classes; ++k) z += expf(v[k] - mx);
  for (int k = 0; k < n_classes; ++k) o[k] = expf(v[k] - mx) / z;
}

// Wt[group of `row` maps][k][map] of every layer (blockIdx.y) from the canonical weights: k = (input map, ky, kx), j =
// output map; absent connections and the padding maps are zero.  Tiles of 64 k x 32 maps, turned round in LDS: rows of
// the canonical weights are read, rows of Wt written.  Two launches a layer (clear, scatter) before: 10000 digits 38 us
// of launches -> 5.
constexpr int PK = 64, PJ = 32;
__global__ void __launch_bounds__(256) k_batch_pack(BatchPackAll all) {
  __shared__ float t[PJ][PK + 1];
  const BatchPack q = all.l[blockIdx.y];
  const int KK = q.K * q.Kx, tk = (q.k_total + PK - 1) / PK;
  const int rows = (q.Mo + q.row - 1) / q.row * q.row, tiles = tk * ((rows + PJ - 1) / PJ);
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int j0 = tile / tk * PJ, k0 = tile % tk * PK;
    const int k = k0 + (threadIdx.x & (PK - 1));
    const int i = k / KK;
    for (int r = threadIdx.x / PK; r < PJ; r += 256 / PK) {
      const int j = j0 + r;
      float v = 0.f;
      if (j < q.Mo && k < q.k_total) {
        if (q.full_table) {
          v = q.w[(long long)j * q.k_total + k];
        } else {   // the slot of input map i among the row's connections, which ascend
          int lo = q.csr_ptr[j], hi = q.csr_ptr[j + 1];
          const int end = hi;
          while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (q.csr_idx[mid] < i) lo = mid + 1; else hi = mid;
          }
          if (lo < end && q.csr_idx[lo] == i) v = q.w[(long long)lo * KK + (k - i * KK)];
        }
      }
      t[r][k - k0] = v;
    }
    __syncthreads();
    const int j = j0 + (threadIdx.x & (PJ - 1));
    if (j < rows) {
      const gf dst = q.wt + (long long)(j / q.row) * q.k_total * q.row + j % q.row;
      for (int c = threadIdx.x / PJ; c < PK && k0 + c < q.k_total; c += 256 / PJ) dst[(long long)(k0 + c) * q.row] = t[j - j0][c];
    }
    __syncthreads();
  }
}

}  // namespace
size_t batch_conv_lds_bytes(const BatchConv& g);
// workgroups of k_batch_conv a compute unit holds at once, estimated: accumulators and 64 more registers, LDS.  By the
// compiler's registers two to five tiles of 32 maps fit one workgroup less (4, 3, 2, 2), seven of 16 too, one of 32 and two
// of 16 one more; where LDS does not bind, the surplus workgroups of a launch start as the first ones end.  With the
// compiler's counts here and in the time models fitted with these, 10000 digits took 756 us instead of 746, 777 images of
// the widest net 1887 instead of 1877, 300 of them 772 instead of 733.
int batch_conv_fit(int MT, int TR, size_t lds_bytes) {
  const int regs = (MT * (TR == 32 ? 16 : 8) + 64 + 7) & ~7;
  return std::max(1, std::min({512 / regs, (int)(160 * 1024 / lds_bytes), 8}));
}
// workgroups along the column blocks: about as many as the chip holds at once, over all groups of maps and slices
int batch_conv_grid_x(const BatchConv& g) {
  const int groups = (g.Mo + g.MT * g.TR - 1) / (g.MT * g.TR) * g.n_slices;
  return (int)std::min<long long>(g.n_cb, std::max(1, 256 * batch_conv_fit(g.MT, g.TR, batch_conv_lds_bytes(g)) / groups));
}
namespace {

template <int MT, int TR>
hipError_t launch_conv_mt(hipStream_t stream, const BatchConv& g, size_t lds_bytes) {
  hipError_t e = hipFuncSetAttribute((const void*)k_batch_conv<MT, TR>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  if (e != hipSuccess) return e;
  const int groups = (g.Mo + MT * TR - 1) / (MT * TR);
  hipLaunchKernelGGL((k_batch_conv<MT, TR>), dim3((unsigned)batch_conv_grid_x(g), (unsigned)groups, (unsigned)g.n_slices), dim3(BT),
                     lds_bytes, stream, g);
  return hipGetLastError();
}

template <int MT, int TR>
hipError_t launch_gemm_mt(hipStream_t stream, const BatchGemm& g, size_t lds_bytes) {
  hipError_t e = hipFuncSetAttribute((const void*)k_batch_gemm<MT, TR>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  if (e != hipSuccess) return e;
  const unsigned gx = (unsigned)((g.N + BCOLS - 1) / BCOLS);
  const unsigned gy = (unsigned)((g.MoPad / TR + MT - 1) / MT);
  hipLaunchKernelGGL((k_batch_gemm<MT, TR>), dim3(gx, gy, (unsigned)g.KS), dim3(BT), lds_bytes, stream, g);
  return hipGetLastError();
}

}  // namespace

size_t batch_gemm_lds_bytes(const BatchGemm& g) {
  const int KC = g.IC * g.K * g.Kx;
  const size_t KS = g.TR == 32 ? 2 : 4;
  const size_t KH = ((((size_t)KC + KS - 1) / KS) + 3) & ~(size_t)3;
  return ((((size_t)g.n_img_max * batch_slot(g.IC, g.Hi * g.Wi) + 3) & ~(size_t)3) + (size_t)(KC + 1) * g.MT * g.TR + KS * KH) * sizeof(float);
}

size_t batch_conv_lds_bytes(const BatchConv& g) {
  const size_t KC = (size_t)g.IC * g.K * g.Kx, KS = g.TR == 32 ? 2 : 4, M = (size_t)g.Kp * g.Kpx;
  const size_t KH = (((KC + KS - 1) / KS) + 3) & ~(size_t)3;
  const size_t w_size = (KC * g.MT * g.TR + 255) & ~(size_t)255;
  return ((g.resident ? 1 : 2) * w_size + 2 * (size_t)g.n_img_max * g.slot + KS * KH + g.MT * g.TR +
          (M == 1 || M == 4 ? 0 : (size_t)g.TR * EP)) * sizeof(float);
}

hipError_t launch_batch_conv(hipStream_t stream, const BatchConv& g) {
  if (g.n_win <= 0) return hipSuccess;
  const size_t lds_bytes = batch_conv_lds_bytes(g);
  if (g.TR == 32) {
    switch (g.MT) {
      case 1: return launch_conv_mt<1, 32>(stream, g, lds_bytes);
      case 2: return launch_conv_mt<2, 32>(stream, g, lds_bytes);
      case 3: return launch_conv_mt<3, 32>(stream, g, lds_bytes);
      case 4: return launch_conv_mt<4, 32>(stream, g, lds_bytes);
      case 5: return launch_conv_mt<5, 32>(stream, g, lds_bytes);
      default: return hipErrorInvalidValue;
    }
  }
  if (g.TR != 16) return hipErrorInvalidValue;
  switch (g.MT) {
    case 1: return launch_conv_mt<1, 16>(stream, g, lds_bytes);
    case 2: return launch_conv_mt<2, 16>(stream, g, lds_bytes);
    case 3: return launch_conv_mt<3, 16>(stream, g, lds_bytes);
    case 4: return launch_conv_mt<4, 16>(stream, g, lds_bytes);
    case 5: return launch_conv_mt<5, 16>(stream, g, lds_bytes);
    case 6: return launch_conv_mt<6, 16>(stream, g, lds_bytes);
    case 7: return launch_conv_mt<7, 16>(stream, g, lds_bytes);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_batch_gemm(hipStream_t stream, const BatchGemm& g) {
  if (g.N <= 0) return hipSuccess;
  const size_t lds_bytes = batch_gemm_lds_bytes(g);
  if (g.TR == 32) {
    switch (g.MT) {
      case 1: return launch_gemm_mt<1, 32>(stream, g, lds_bytes);
      case 2: return launch_gemm_mt<2, 32>(stream, g, lds_bytes);
      case 4: return launch_gemm_mt<4, 32>(stream, g, lds_bytes);
      default: return hipErrorInvalidValue;
    }
  }
  if (g.TR != 16) return hipErrorInvalidValue;
  switch (g.MT) {
    case 2: return launch_gemm_mt<2, 16>(stream, g, lds_bytes);
    case 3: return launch_gemm_mt<3, 16>(stream, g, lds_bytes);
    case 4: return launch_gemm_mt<4, 16>(stream, g, lds_bytes);
    case 5: return launch_gemm_mt<5, 16>(stream, g, lds_bytes);
    case 6: return launch_gemm_mt<6, 16>(stream, g, lds_bytes);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_batch_pool(hipStream_t stream, const BatchPool& q) {
  if (q.total <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_pool, dim3((unsigned)((q.total + 255) / 256)), dim3(256), 0, stream, q);
  return hipGetLastError();
}

hipError_t launch_batch_outputs(hipStream_t stream, const float* sums, int n_slices, long long slice_stride, const float* bias,
                                float* probs, long long n_images, int n_classes, int out_units) {
  if (n_images <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_batch_outputs, dim3((unsigned)((n_images + 255) / 256)), dim3(256), 0, stream, (cgf)sums, n_slices,
                     slice_stride, (cgf)bias, (gf)probs, n_images, n_classes, out_units);
  return hipGetLastError();
}

hipError_t launch_batch_pack(hipStream_t stream, const BatchPackAll& all) {
  long long most = 1;
  for (int l = 0; l < all.n; ++l) {
    const BatchPack& q = all.l[l];
    const long long rows = (q.Mo + q.row - 1) / q.row * (long long)q.row;
    most = std::max(most, (q.k_total + PK - 1) / PK * ((rows + PJ - 1) / PJ));
  }
  hipLaunchKernelGGL(k_batch_pack, dim3((unsigned)std::min(most, 4096ll), (unsigned)all.n), dim3(256), 0, stream, all);
  return hipGetLastError();
}

}  // namespace cnn355
