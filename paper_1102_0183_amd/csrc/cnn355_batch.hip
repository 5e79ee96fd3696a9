// Batched forward propagation (Sec. 3.2 for many images at once): validation and test passes
// change no weight (Sec. 4), so their images are independent and every layer becomes one dense
// matrix product over the whole batch,
//     sums[j][n] = sum_k  Wt[k][j] * X[k][n],     n = (image b, output pixel p),  k = (input map i, ky, kx),
// which is what the matrix cores are for.  X is never formed: its element is
// in[b][i][(y (S+1) + ky)][(x (S+1) + kx)], read from the images staged in LDS at offset
// koff(k) + pbase(n).  A fully connected layer is the same product with 1 x 1 maps and K = 1.
// fp32 operands and fp32 accumulation (v_mfma_f32_32x32x2_f32), or operands as two halves each
// (k_batch_split, k_batch_first): the results stay within the tolerance of the one-image path.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <cstdint>

#define CNN_GLOBAL __attribute__((address_space(1)))
#include "cnn355_dev.h"

namespace cnn355 {

typedef const CNN_GLOBAL float* cgf;
typedef CNN_GLOBAL float* gf;
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

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

// Activation v as split halves (BatchSplit).  off: byte offset of the high half in `out`, the low one lies a plane behind it.
__device__ __forceinline__ void put_split(CNN_GLOBAL char* out, unsigned plane, unsigned off, float v) {
  const float x = v * (float)(1 << SPLIT_SHIFT);
  const _Float16 h = (_Float16)x;
  *(CNN_GLOBAL _Float16*)(out + off) = h;
  *(CNN_GLOBAL _Float16*)(out + plane + off) = (_Float16)(x - (float)h);
}
// the same of four maps side by side
__device__ __forceinline__ void put_split4(CNN_GLOBAL char* out, unsigned plane, unsigned off, const float (&v)[4]) {
  v4h h, l;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const float x = v[u] * (float)(1 << SPLIT_SHIFT);
    h[u] = (_Float16)x;
    l[u] = (_Float16)(x - (float)h[u]);
  }
  *(CNN_GLOBAL v4h*)(out + off) = h;
  *(CNN_GLOBAL v4h*)(out + plane + off) = l;
}

// Activation v as it is, in the place of its halves (SplitMarks)
__device__ __forceinline__ void put_whole(CNN_GLOBAL char* out, unsigned plane, unsigned off, float v) {
  const unsigned b = __float_as_uint(v);
  *(CNN_GLOBAL _Float16*)(out + off) = __builtin_bit_cast(_Float16, (unsigned short)(b >> 16));
  *(CNN_GLOBAL _Float16*)(out + plane + off) = __builtin_bit_cast(_Float16, (unsigned short)b);
}
__device__ __forceinline__ void put_whole4(CNN_GLOBAL char* out, unsigned plane, unsigned off, const float (&v)[4]) {
  v4h h, l;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const unsigned b = __float_as_uint(v[u]);
    h[u] = __builtin_bit_cast(_Float16, (unsigned short)(b >> 16));
    l[u] = __builtin_bit_cast(_Float16, (unsigned short)b);
  }
  *(CNN_GLOBAL v4h*)(out + off) = h;
  *(CNN_GLOBAL v4h*)(out + plane + off) = l;
}
// the activation that is stored in these halves, times 2^14
__device__ __forceinline__ float whole_of(_Float16 high, _Float16 low) {
  const unsigned b = (unsigned)__builtin_bit_cast(unsigned short, high) << 16 | __builtin_bit_cast(unsigned short, low);
  return __uint_as_float(b) * (float)(1 << SPLIT_SHIFT);
}

// (21600 wavefronts that all store the word took 750 us)
__device__ __forceinline__ void mark_any(const SplitMarks& m) {
  if (__hip_atomic_load(m.any, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) __hip_atomic_store(m.any, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 2 x 2 windows whose members are the four lanes of a quad: the window's largest sum of row u (of four) goes to lane q = u.
// (The maximum of what the compiler cannot tell is no signalling NaN costs it three instructions, the statement's one; the
// operands come from an instruction that it sees, so it is the one that waits for the matrix cores.)
__device__ __forceinline__ float pool_quad(float a0, float a1, float a2, float a3, int q) {
  const float x0 = __builtin_canonicalizef(a0), x1 = __builtin_canonicalizef(a1), x2 = __builtin_canonicalizef(a2), x3 = __builtin_canonicalizef(a3);
  float r0, r1, r2, r3;
  asm("s_nop 1\n\t"
      "v_max_f32_dpp %0, %4, %4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %5, %5 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %2, %6, %6 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %3, %7, %7 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %2, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %3, %3, %3 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
      : "=&v"(r0), "=&v"(r1), "=&v"(r2), "=&v"(r3)
      : "v"(x0), "v"(x1), "v"(x2), "v"(x3));
  return fmaxf(q < 2 ? (q == 0 ? r0 : r1) : (q == 2 ? r2 : r3), -INFINITY);   // (no number at all: -inf)
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
// N runs of 64 lanes' 16 bytes, one behind the other at either end (an instruction's offset counts for both addresses).
// lds_byte and base come from scalar instructions.
template <int N>
__device__ __forceinline__ void lds_dma16_runs(unsigned lds_byte, const CNN_GLOBAL char* base, unsigned off) {
  if constexpr (N == 1)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_byte), "v"(off), "s"(base) : "memory", "m0");
  else if constexpr (N == 2)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024" ::"s"(lds_byte),
                 "v"(off), "s"(base) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024\n\t"
                 "global_load_lds_dwordx4 %1, %2 offset:2048\n\tglobal_load_lds_dwordx4 %1, %2 offset:3072" ::"s"(lds_byte),
                 "v"(off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop
__device__ __forceinline__ void lds_dma16_n(unsigned lds_byte, const CNN_GLOBAL char* base, unsigned off, int n) {
  for (; n >= 4; n -= 4, lds_byte += 4096, off += 4096) lds_dma16_runs<4>(lds_byte, base, off);
  if (n >= 2) { lds_dma16_runs<2>(lds_byte, base, off); n -= 2; lds_byte += 2048; off += 2048; }
  if (n > 0) lds_dma16_runs<1>(lds_byte, base, off);
}

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

// ---- the first convolutional layer in front of one in products of halves ---------------------------------------
// A wavefront takes 32 windows and walks their members one after the other, keeping the largest sums of T tiles of 32 maps in
// registers: no sums pass between lanes, and a lane has four maps of its window side by side for a store.  A lane gathers its
// k's pixels straight from memory (the caches serve the overlapping fields), the next member's while it works on this one, and
// splits them into halves as put_split does; the weights are split into LDS at the start.  Nothing is staged and no wavefront
// waits for another -- unless the windows are few: then four wavefronts share the members of 32 windows (g.share).
// Why halves: 32-bit products leave the vector units idle (a wavefront's vector instructions wait for another one's products:
// 103 us of products and 122 of vector work on the same SIMD took 220 together, with products of halves 62 and 122 took 148),
// and these layers have as much of the one as of the other.  300C3 on 3 maps, 512 images: k_batch_conv 177 us, this kernel with
// 32-bit products 146, with halves 90 (105 in a trace of whole passes); 20C4 of 4096 digits 77, 51, 45.
// Pixels that do not split (4 and larger, infinite, or all of a lane's below 2^-14 and not zero) and weights that do not (not
// finite, or all of a row's below 2^-81) take 32-bit products, member by member, for the 32 windows of a wavefront (images of 0..255:
// 4096 digits 148 -> 162 us a call, 512 images of 300 maps a layer 431 -> 485; k_batch_conv's nets 292 and 1151).
constexpr int first_waves(int T, int H) {   // wavefronts a SIMD, by the registers of pixels, offsets, halves and sums
  const int regs = (H <= 4 ? 24 : 16) * H + 16 * T + 72;
  return regs <= 124 ? 4 : regs <= 164 ? 3 : 2;
}
template <int T, int H>
__global__ void __launch_bounds__(BT, first_waves(T, H)) k_batch_first(BatchFirst g) {
  extern __shared__ __align__(16) char lds_s[];
  constexpr int N = 8 * H, ROWS = T * 32;
  const int tid = threadIdx.x, lane = tid & 63, lrow = lane & 31, lk = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j0 = max(0, (int)blockIdx.y * ROWS - g.shift), end = min(g.Mo, ((int)blockIdx.y + 1) * ROWS - g.shift);   // maps
  char* lds_h = lds_s;                                   // [T][H][high, low][k / 8 mod 2][32 maps][8] halves
  float* lds_f = (float*)(lds_h + T * H * 2048);         // [k_total][ROWS] weights
  float* lds_b = lds_f + g.k_total * ROWS;               // [ROWS] biases
  int* lds_e = (int*)(lds_b + ROWS);                     // [ROWS] -(e + SPLIT_SHIFT), halves are w 2^e
  int* koff = lds_e + ROWS;                              // [16 H] byte offset of k from a member's first pixel
  float* ex = (float*)(koff + 16 * H);                   // [4][T * 16][64] where wavefronts share
  float* all_most = ex + 4 * T * 1024;                   // [4][32] of the same
  const int KK = g.K * g.Kx, HiWi = g.Hi * g.Wi;
  for (int x = tid; x < 16 * H; x += BT) {
    const int k = min(x, g.k_total - 1), c = k / KK, t = k - c * KK, ky = t / g.Kx;
    koff[x] = (c * HiWi + ky * g.Wi + t - ky * g.Kx) * 4;
  }
  for (int x = tid; x < ROWS; x += BT) lds_b[x] = j0 + x < g.Mo ? g.bias[j0 + x] : 0.f;
  for (int x0 = tid; x0 < g.k_total * ROWS; x0 += 8 * BT) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int x = x0 + u * BT, k = x / ROWS, j = j0 + x % ROWS;
      v[u] = k < g.k_total && j < g.row ? g.wt[(long long)k * g.row + j] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (x0 + u * BT < g.k_total * ROWS) lds_f[x0 + u * BT] = v[u];
  }
  __syncthreads();
  bool odd = false;
  for (int r = tid; r < ROWS; r += BT) {
    float most = 0.f;
    for (int k = 0; k < g.k_total; ++k) {
      const float v = fabsf(lds_f[k * ROWS + r]);
      odd |= !(v < INFINITY);
      most = fmaxf(most, v);
    }
    int e = 0;
    if (most > 0.f && most < INFINITY) { frexpf(most, &e); e = 15 - e; }
    odd |= e > 96;
    lds_e[r] = -(e + SPLIT_SHIFT);
  }
  odd = __syncthreads_or(odd);
  if (odd)
    for (int r = tid; r < ROWS; r += BT) lds_e[r] = 0;
  else
    for (int x = tid; x < T * H * 64; x += BT) {         // (tile, h, k / 8 mod 2, map)
      const int r = x & 31, l = (x >> 5) & 1, h = (x >> 6) % H, m = x / (64 * H), e = -lds_e[m * 32 + r] - SPLIT_SHIFT;
      v8h hi, lo;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = h * 16 + l * 8 + i;
        const float v = k < g.k_total ? ldexpf(lds_f[k * ROWS + m * 32 + r], e) : 0.f;
        hi[i] = (_Float16)v;
        lo[i] = (_Float16)(v - (float)hi[i]);
      }
      *(v8h*)(lds_h + ((m * H + h) * 4 + l) * 512 + r * 16) = hi;
      *(v8h*)(lds_h + ((m * H + h) * 4 + 2 + l) * 512 + r * 16) = lo;
    }
  __syncthreads();
  // a lane's k = 16 h + 8 lk + i; the offsets of long sums are read again for every member
  constexpr bool KEEP = H <= 4;
  int ko[KEEP ? N : 1];
#pragma unroll
  for (int s = 0; s < N; ++s)
    if constexpr (KEEP) ko[s] = koff[(s >> 3) * 16 + lk * 8 + (s & 7)];
  const int M = g.Kp * g.Kpx, n_tiles = (g.n_win + 31) >> 5, share = g.share;
  // the largest number of none: of several members -inf, of one member what its sum is (the largest of two is the number of them)
  const float none = M == 1 ? __builtin_nanf("") : -INFINITY;
  const unsigned plane = (unsigned)g.split_out * 16u;
  float px[N];
  const CNN_GLOBAL char* src = nullptr;            // the first image of the wavefront's next windows
  int at = 0;                                      // the lane's first pixel, bytes from there
  auto aim = [&](int t) {
    const int b0 = fast_div(t * 32, g.by_win_img), w = min(t * 32 + lrow, g.n_win - 1);
    const int b = fast_div(w, g.by_win_img), wi = w - b * g.win_img, wy = fast_div(wi, g.by_wp), wx = wi - wy * g.Wp;
    src = (const CNN_GLOBAL char*)(g.in + (long long)b0 * g.in_stride);
    at = ((b - b0) * (int)g.in_stride + wy * g.Kp * g.stride * g.Wi + wx * g.Kpx * g.stride_x) * 4;
  };
  auto fetch = [&](int d) {   // member d's pixels
    const int dy = fast_div(d, g.by_kpx), dx = d - dy * g.Kpx;
    const CNN_GLOBAL char* p = src + (unsigned)((dy * g.stride * g.Wi + dx * g.stride_x) * 4);
    int a = at;
    asm volatile("" : "+v"(a));   // (or the sums of it and every ko are kept too)
#pragma unroll
    for (int s = 0; s < N; ++s) px[s] = *(const CNN_GLOBAL float*)(p + (unsigned)(a + (KEEP ? ko[KEEP ? s : 0] : koff[(s >> 3) * 16 + lk * 8 + (s & 7)])));
  };
  const int step = gridDim.x * (share ? 1 : 4), d_first = share ? wave : 0, d_step = share ? 4 : 1;
  int t = share ? (int)blockIdx.x : (int)blockIdx.x * 4 + wave;
  if (t >= n_tiles) return;                        // (sharing wavefronts leave together)
  aim(t);
  fetch(d_first);
  for (; t < n_tiles; t += step) {
    v16f best[T];
#pragma unroll
    for (int m = 0; m < T; ++m)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float x = none;
        asm volatile("" : "+v"(x));   // (or sixteen of them are kept in registers)
        best[m][v] = x;
      }
    for (int d = d_first; d < M; d += d_step) {
      v8h xh[H], xl[H];
      float most = 0.f;
#pragma unroll
      for (int s = 0; s < N; ++s) {
        const float x = px[s] * (float)(1 << SPLIT_SHIFT);
        most = fmaxf(most, fabsf(px[s]));
        xh[s >> 3][s & 7] = (_Float16)x;
        xl[s >> 3][s & 7] = (_Float16)(x - (float)xh[s >> 3][s & 7]);
      }
      const bool splits = !odd && !__any(most >= 3.99f || (most < 0x1p-14f && most > 0.f));
      if (!splits) {   // (k beyond the last one count as zero on both sides)
#pragma unroll
        for (int m = 0; m < T; ++m) {
          v16f acc;
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
          for (int s = 0; s < N; ++s) {
            const int k = (s >> 3) * 16 + lk * 8 + (s & 7);
            const float w = lds_f[min(k, g.k_total - 1) * ROWS + m * 32 + lrow];
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(k < g.k_total ? w : 0.f, k < g.k_total ? px[s] : 0.f, acc, 0, 0, 0);
          }
#pragma unroll
          for (int v = 0; v < 16; ++v) best[m][v] = fmaxf(best[m][v], ldexpf(acc[v], -lds_e[m * 32 + (v >> 2) * 8 + lk * 4 + (v & 3)]));
        }
      }
      const bool last = d + d_step >= M;
      if (last && t + step < n_tiles) aim(t + step);
      fetch(last ? d_first : d + d_step);          // (behind the last windows: once more)
      __builtin_amdgcn_sched_barrier(0);           // (the loads are not put off until their registers are free)
      if (!splits) continue;
#pragma unroll
      for (int m = 0; m < T; ++m) {
        if (m && j0 + m * 32 >= end) break;
        const char* w = lds_h + m * H * 2048 + lane * 16;
        v16f acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        // the small products first: they are rounded to what they are, not to the whole sum
        v8h wh[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
          wh[h] = *(const v8h*)(w + h * 2048);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wh[h], xl[h], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(*(const v8h*)(w + h * 2048 + 1024), xh[h], acc, 0, 0, 0);
        }
#pragma unroll
        for (int h = 0; h < H; ++h) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(wh[h], xh[h], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float sum = __builtin_canonicalizef(acc[v]);
          asm("v_max_f32 %0, %0, %1" : "+v"(best[m][v]) : "v"(sum));   // (as in pool_quad)
        }
      }
    }
    if (share) {
      __syncthreads();   // the last windows' have been read
#pragma unroll
      for (int m = 0; m < T; ++m)
#pragma unroll
        for (int v = 0; v < 16; ++v) ex[(wave * T + m) * 1024 + v * 64 + lane] = best[m][v];
      __syncthreads();
    }
    // element v of a lane: map (v / 4) * 8 + lk * 4 + v % 4 of the tile
    const int w = t * 32 + lrow;
    int lk4 = lk * 4;
    asm volatile("" : "+v"(lk4));
    // the outputs of four maps of a lane
    auto outputs = [&](int m, int v4, int row, float sum, float (&sv)[4]) {
      const bool part = j0 + m * 32 + v4 * 2 + 8 > end;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float x = u ? best[m][v4 + u] : sum;
        if (share)
          for (int o = 0; o < 4; ++o) x = fmaxf(x, ex[(o * T + m) * 1024 + (v4 + u) * 64 + lane]);
        sv[u] = b_act(ldexpf(x, lds_e[row + u]) + lds_b[row + u]);
        if (part && j0 + row + u >= end) sv[u] = 0.f;   // (maps that fill the last group of eight up)
      }
    };
    auto out_of = [&](int first) { return (CNN_GLOBAL char*)g.out + (size_t)((unsigned)(j0 + first) >> 3) * 2 * plane; };
    float most = 0.f;
#pragma unroll
    for (int m = 0; m < T; ++m)
#pragma unroll
      for (int v4 = 0; v4 < 16; v4 += 4) {
        const int first = m * 32 + v4 * 2;
        if (j0 + first >= end) break;
        if (share && (m * 4 + v4 / 4) % 4 != wave) continue;
        float sv[4];
        outputs(m, v4, first + lk4, best[m][v4], sv);
#pragma unroll
        for (int u = 0; u < 4; ++u) most = fmaxf(most, fabsf(sv[u]));
        if (w < g.n_win) put_split4(out_of(first), plane, (unsigned)w * 16u + (unsigned)lk4 * 2u, sv);
      }
    if (share) {   // (the wavefronts have the window's maps between them)
      most = fmaxf(most, __shfl_xor(most, 32));
      if (lane < 32) all_most[wave * 32 + lane] = most;
      __syncthreads();
      for (int o = 0; o < 4; ++o) most = fmaxf(most, all_most[o * 32 + lrow]);
    }
    unsigned long long small = __ballot(!(most >= SPLIT_TINY));
    small &= small >> 32;
    bool tiny = false;
    if (__builtin_expect(small != 0, 0)) {
      most = fmaxf(most, __shfl_xor(most, 32));
      tiny = w < g.n_win && most < SPLIT_TINY;
      if (!__any(tiny && most > 0.f)) tiny = false;   // (zeros are halves, and floats)
      else {                                          // once more: these are stored as they are
        if (lane == 0) mark_any(g.out_marks);
#pragma unroll
        for (int m = 0; m < T; ++m)
#pragma unroll
          for (int v4 = 0; v4 < 16; v4 += 4) {
            const int first = m * 32 + v4 * 2;
            if (j0 + first >= end) break;
            if (share && (m * 4 + v4 / 4) % 4 != wave) continue;
            float sum = best[m][v4], sv[4];
            asm volatile("" : "+v"(lk4), "+v"(sum));   // (or what is worked out above is kept in registers for here)
            outputs(m, v4, first + lk4, sum, sv);
            if (tiny) put_whole4(out_of(first), plane, (unsigned)w * 16u + (unsigned)lk4 * 2u, sv);
          }
      }
    }
    if (w < g.n_win && lane < 32) g.out_marks.at[(size_t)blockIdx.y * (unsigned)g.split_out + (unsigned)w] = tiny;
  }
}

// ---- a convolutional layer behind another one, in products of halves --------------------------------------------
// The product of k_batch_conv on v_mfma_f32_{32x32x16,16x16x32}_f16, which take sixteen times the terms a clock: both
// operands are split into two halves (23 bits together), a = ah + al, and ah xh + ah xl + al xh summed in 32 bits; al xl is
// below 2^-22 of the term.  An instruction adds its terms in groups of eight to the running sum, each group's sum rounded; so a
// running sum ends after whole slabs of at most SPLIT_RUN groups together and is added to the total, which keeps the error against
// 64 bits below that of the 32-bit products.  The layer below has split its activations already (put_split), in groups of eight
// maps, so that a lane's eight k are one 16-byte read from LDS: k = (group of eight maps, ky, kx, map of the group).
// What a workgroup writes of a window is stored as floats where all of it is tiny (SplitMarks): the largest output is kept along
// with the stores, and the stores are done again where it is.  40C5 of 4096 digits 76.8 -> 80.2 us with it, the first layer's 20C4
// 43.6 -> 45.9, 300C2 of 512 images 225 -> 227 (one trace).
// Error against 64 bits (2-norm, of a layer's outputs from the images on, 32-bit products / halves): 300C4 behind 300C2 behind
// 300C3 10.8e-7 / 3.4e-7, 300C2 5.8 / 2.2, 40C5 behind 20C4 4.8 / 2.4, 128C3 behind 50C5 2.3 / 2.0; of 300C4 alone 5.7 / 3.3, and
// 8.8 without runs.
// Staging as in k_batch_conv: the next slab of weights (a run of the k range, packed in the order it is read) and the next
// chunk of input maps go to the other halves of their buffers by 16-byte loads to LDS while the present ones are multiplied,
// one barrier a slab, nothing between two column blocks.
// Matrix pipes 40 % busy in 300C2: a step's other instructions fit beside the products of two wavefronts a SIMD, what lies outside
// the steps does not: a wait for all loads and a barrier a slab, and, a block, scalars that the compiler keeps in lanes of vector
// registers.  Larger tiles, one wavefront a SIMD, were slower (300C2: 128 x 256 columns 694 us of the pass, 64 x 256 543).  Against
// k_batch_conv, in traces of whole passes: 300C2 of 512 images 772 -> 227 us (318 TFLOP/s of the layer's own sums), 300C4 235 -> 89,
// 40C5 of 4096 digits 183 -> 80, 128C3 of 33 stereo pairs 42 (with its k_batch_pool) -> 16.
// FC: a fully connected layer behind such a layer.  A column is an image, and a lane of a staging load fetches an image's eight
// maps at one pixel (16 bytes a line of memory; neighbouring pixels follow in the same chunk and meet it in the caches); the k
// range in slices where the images are few.  Against k_batch_gemm and its k_batch_pool: 150N of 4096 digits 30 us -> 13.6, 300N of
// 512 images 27 -> 12.9, 100N of 33 stereo pairs 21.5 -> 8.0.
// wavefronts a SIMD, by the registers of sums, totals and two sets of columns
constexpr int split_waves(int RT, int CT, int TR) {
  const int regs = 2 * RT * CT * (TR == 32 ? 16 : 4) + 16 * CT + 48;
  return regs <= 120 ? 4 : regs <= 136 ? 3 : 2;
}
template <int RT, int CT, int TR, bool FC>
__global__ void __launch_bounds__(BT, split_waves(RT, CT, TR)) k_batch_split(BatchSplit g) {
  extern __shared__ __align__(16) char lds_s[];
  constexpr int S = TR == 32 ? 2 : 4;              // groups of eight k an instruction takes, one per 64 / S lanes
  constexpr int AV = TR == 32 ? 16 : 4;            // accumulator floats per lane and tile
  constexpr int ROWS = RT * TR, COLS = 4 * CT * TR, EPS = COLS + 4;
  int tid = threadIdx.x, lane = tid & 63;
  int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int lrow = lane & (TR - 1), lk = lane / TR;
  const int plane = g.run_px * 16;                 // bytes of a staged plane: eight maps' high or low halves
  const int x_bytes = g.IC * 2 * plane, slab_bytes = g.slab * ROWS * 32;
  char* lds_x = lds_s;
  char* lds_w = lds_x + 2 * x_bytes;
  int* koff = (int*)(lds_w + 2 * slab_bytes);      // byte offset of a (group, tap) pair from a column's first pixel
  int* lds_e = koff + g.n_kg;                      // [ROWS] exponents
  float* lds_b = (float*)(lds_e + ROWS);           // [ROWS] biases
  float* ep = lds_b + ROWS;                        // [TR][EPS] where windows are pooled through LDS
  unsigned* w_most = (unsigned*)(ep + TR * EPS);   // [wins] the largest output of each, of the same
  const unsigned x_at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds_x;
  const unsigned w_at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds_w;
  // (asked for side by side, as vector loads: one after the other they are three trips to memory before anything is staged)
  static_assert(ROWS <= BT, "a row a thread");
  const int j0 = blockIdx.y * ROWS, row = min(tid, ROWS - 1);
  int none = 0;
  asm volatile("" : "+v"(none));
  const int any_marks = g.in_marks.any[none], e_row = g.exps[j0 + row];
  const float b_row = g.bias[min(j0 + row, g.Mo - 1)];
  const int KK = FC ? 1 : g.K * g.Kx;
  for (int x = tid; x < g.n_kg; x += BT) {         // (pairs that fill an instruction up have no weights: a pixel that is read anyway)
    const int k = min(x, g.IC * KK - 1), c = k / KK, t = k - c * KK, ky = t / g.Kx;
    koff[x] = c * 2 * plane + (ky * g.Wi + t - ky * g.Kx) * 16;
  }
  bool slow = false;
  if (tid < ROWS) {
    slow = e_row >= SPLIT_SLOW / 2;
    lds_e[tid] = slow ? e_row - SPLIT_SLOW : e_row;
    lds_b[tid] = j0 + tid < g.Mo ? b_row : 0.f;
  }
  slow = __builtin_amdgcn_readfirstlane(__syncthreads_or(slow));
  const int n_chunks = g.n_cg / g.IC, ch_first = FC ? blockIdx.z * g.cps : 0, ch_end = FC ? min(n_chunks, ch_first + g.cps) : n_chunks;
  const int slabs = (g.n_kg + g.slab - 1) / g.slab, M = FC ? 1 : g.Kp * g.Kpx;
  const int longest = min(SPLIT_RUN, n_chunks * g.n_kg / 2);
  const CNN_GLOBAL char* wt = g.wt + (long long)blockIdx.y * n_chunks * g.n_kg * ROWS * 32;
  // Pixels of the batch that block cb reads: from the first of its first window to the last of its last.  Staged in loads of 64
  // pixels of a plane, whose last ones may reach past the block's (into memory of the call's: its end is 64 pixels off), and of
  // 64 units of weights; a wavefront takes a run of them.
  int x_first = 0, x_n = 0;
  auto aim = [&](int cb) {
    if constexpr (FC) {
      x_first = cb * COLS * g.pix;
      return;
    }
    const int w0 = cb * g.wins, w1 = min(w0 + g.wins, g.n_win) - 1;
    const int b0 = fast_div(w0, g.by_win_img), b1 = fast_div(w1, g.by_win_img);
    const int i0 = w0 - b0 * g.win_img, i1 = w1 - b1 * g.win_img, y0 = fast_div(i0, g.by_wp), y1 = fast_div(i1, g.by_wp);
    x_first = b0 * g.pix + y0 * g.Kp * g.stride * g.Wi + (i0 - y0 * g.Wp) * g.Kpx * g.stride_x;
    x_n = b1 * g.pix + ((y1 * g.Kp + g.Kp - 1) * g.stride + g.K - 1) * g.Wi + ((i1 - y1 * g.Wp) * g.Kpx + g.Kpx - 1) * g.stride_x + g.Kx - x_first;
  };
  unsigned image[FC ? COLS / 64 : 1];              // FC: the lane's images of a block, bytes from the first one
  auto fetch_x = [&](int chunk, int buf) {
    if constexpr (FC) {
      for (int p = wave; p < g.IC * 2; p += 4) {
        const int vg = chunk * g.IC + (p >> 1), cg = fast_div(vg, g.by_pix);
        const CNN_GLOBAL char* src = g.in + (long long)(cg * 2 + (p & 1)) * g.in_plane + (long long)(x_first + vg - cg * g.pix) * 16;
#pragma unroll
        for (int q = 0; q < COLS / 64; ++q) lds_dma16_runs<1>(x_at + (unsigned)(buf * x_bytes + p * plane + q * 1024), src, image[q]);
      }
      return;
    }
    const CNN_GLOBAL char* src = g.in + (long long)chunk * g.IC * 2 * g.in_plane + (long long)x_first * 16;
    const int per = (x_n + 63) >> 6, half = (per + 1) >> 1;
    const bool halves = g.IC == 1;   // two planes: two wavefronts each
    const int q = halves ? (wave & 1) * half : 0, n = halves ? min(half, per - q) : per;
    for (int p = halves ? wave >> 1 : wave; p < g.IC * 2; p += 4)
      lds_dma16_n(x_at + (unsigned)(buf * x_bytes + p * plane + q * 1024), src + p * g.in_plane, (unsigned)(q * 64 + lane) * 16u, n);
  };
  auto fetch_w = [&](int at, int n, int buf) {     // n pairs from pair `at` of the group's stream
    const int loads = n * ROWS / 32, share = (loads + 3) >> 2, q = wave * share;
    lds_dma16_n(w_at + (unsigned)(buf * slab_bytes + q * 1024), wt, (unsigned)(at * ROWS * 32 + (q * 64 + lane) * 16), min(share, loads - q));
  };

  typedef float accv __attribute__((ext_vector_type(AV)));
  auto aim_lanes = [&](int cb) {                   // (behind the last image: that one)
#pragma unroll
    for (int q = 0; q < COLS / 64; ++q) image[q] = (unsigned)(min(q * 64 + lane, g.n_win - 1 - cb * COLS) * g.pix * 16);
  };
  auto start = [&](int cb, int xb, int wb) {       // the first chunk and slab of a block
    if constexpr (FC) aim_lanes(cb);
    aim(cb);
    fetch_x(ch_first, xb);
    fetch_w(ch_first * g.n_kg, min(g.slab, g.n_kg), wb);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  auto all_halves = [&](int cb) {                  // of what a block reads
    aim(cb);
    const int n_px = FC ? min(COLS, g.n_win - cb * COLS) * g.pix : x_n;
    bool found = false;
    for (int m = 0; m < g.in_groups; ++m) {
      const CNN_GLOBAL unsigned char* marks = g.in_marks.at + (g.in_plane >> 4) * m + x_first;
      for (int x = tid; x < n_px; x += BT) found |= marks[x] != 0;
    }
    return __builtin_amdgcn_readfirstlane(__syncthreads_or(found)) == 0;
  };
  bool marked = false;
  auto run = [&](auto careful) {
    constexpr bool CAREFUL = decltype(careful)::value;
    // (what the lanes need is worked out once more: kept from the products of halves it cost those registers)
    if constexpr (CAREFUL) asm volatile("" : "+v"(tid), "+v"(lane), "+v"(lrow), "+v"(lk), "+s"(wave));
    int xb = 0, wb = 0;
    if constexpr (!CAREFUL) start(blockIdx.x, 0, 0);
    for (int cb = blockIdx.x; cb < g.n_cb; cb += gridDim.x) {
      if constexpr (CAREFUL) {
        if (!slow && all_halves(cb)) continue;
        __syncthreads();   // what is staged has been read
        start(cb, xb, wb);
      }
      const bool more = !CAREFUL && cb + (int)gridDim.x < g.n_cb;
      const int first = x_first;
      // the first pixel of the batch that column c reads (columns that are not there: the block's first)
      auto column = [&](int c) {
        const int wl = c / M, d = c - wl * M, w = cb * g.wins + wl;
        if (wl >= g.wins || w >= g.n_win) return first;
        const int b = fast_div(w, g.by_win_img);
        const int wi = w - b * g.win_img, wy = fast_div(wi, g.by_wp), wx = wi - wy * g.Wp, dy = d / g.Kpx, dx = d - dy * g.Kpx;
        return b * g.pix + (wy * g.Kp + dy) * g.stride * g.Wi + (wx * g.Kpx + dx) * g.stride_x;
      };
      int pbase[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int c = (wave * CT + ct) * TR + lrow;
        pbase[ct] = (FC ? c : column(c) - first) * 16;
      }
      accv acc[RT][CT], tot[RT][CT];
#pragma unroll
      for (int m = 0; m < RT; ++m)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int v = 0; v < AV; ++v) acc[m][ct][v] = tot[m][ct][v] = 0.f;
      int pairs = 0;
      for (int ch = ch_first; ch < ch_end; ++ch, xb ^= 1) {
        for (int sl = 0; sl < slabs; ++sl, wb ^= 1) {
          // slab and chunk have arrived (every wavefront has waited for its own loads), the other halves are read no more
          __syncthreads();
          const int at = ch * g.n_kg + sl * g.slab, here = min(g.slab, g.n_kg - sl * g.slab);
          const bool last = ch + 1 == ch_end;
          if (sl + 1 < slabs) fetch_w(at + here, min(g.slab, g.n_kg - (sl + 1) * g.slab), wb ^ 1);
          else if (!last || more) fetch_w(last ? ch_first * g.n_kg : at + here, min(g.slab, g.n_kg), wb ^ 1);
          if (sl == 0) {
            if (!last) fetch_x(ch + 1, xb ^ 1);
            else if (more) {
              if constexpr (FC) aim_lanes(cb + gridDim.x);
              aim(cb + gridDim.x);
              fetch_x(ch_first, xb ^ 1);
            }
          }
          // A step is one instruction's k.  The operands of the next tile of maps, and at the first tile the columns of the next
          // step, are on their way from LDS while the present tile is multiplied.
          const char* x_b = lds_x + xb * x_bytes;
          const char* w_b = lds_w + wb * slab_bytes + (lk * 2 * ROWS + lrow) * 16;
          const int* ko = koff + sl * g.slab + lk;
          const int steps = here / S;
          if constexpr (CAREFUL) {   // (infinity times either half of zero, or of signs that differ, is no number: halves are put together first)
#pragma clang loop unroll(disable)
            for (int st = 0; st < steps; ++st) {
              const int k = ko[st * S], c = k / (2 * plane), vg = ch * g.IC + c, eight = FC ? fast_div(vg, g.by_pix) : vg;
              float x[CT][8];
#pragma unroll
              for (int ct = 0; ct < CT; ++ct) {
                const char* p = x_b + (pbase[ct] + k);
                const v8h ph = *(const v8h*)p, pl = *(const v8h*)(p + plane);
                bool whole = false;
                if (marked) {
                  const int px = FC ? min(cb * COLS + (pbase[ct] >> 4), g.n_win - 1) * g.pix + vg - eight * g.pix
                                    : first + ((pbase[ct] + k - c * 2 * plane) >> 4);
                  whole = g.in_marks.at[(g.in_plane >> 4) * fast_div(eight + g.in_shift, g.by_eights) + px] != 0;
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) x[ct][i] = whole ? whole_of(ph[i], pl[i]) : (float)ph[i] + (float)pl[i];
              }
#pragma unroll
              for (int m = 0; m < RT; ++m) {
                const char* w = w_b + (st * S * 2 * ROWS + m * TR) * 16;
                const v8h qh = *(const v8h*)w, ql = *(const v8h*)(w + ROWS * 16);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                  const float wi = (float)qh[i] + (float)ql[i];
#pragma unroll
                  for (int ct = 0; ct < CT; ++ct) {
                    if constexpr (TR == 32) acc[m][ct] = __builtin_amdgcn_mfma_f32_32x32x2f32(wi, x[ct][i], acc[m][ct], 0, 0, 0);
                    else acc[m][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(wi, x[ct][i], acc[m][ct], 0, 0, 0);
                  }
                }
                __builtin_amdgcn_sched_barrier(0);   // (fewer registers)
              }
            }
          } else {
            v8h xh[2][CT], xl[2][CT], wh[2], wl[2];
            auto load_x = [&](int set, int k) {
#pragma unroll
              for (int ct = 0; ct < CT; ++ct) {
                const char* p = x_b + (pbase[ct] + k);
                xh[set][ct] = *(const v8h*)p;
                xl[set][ct] = *(const v8h*)(p + plane);
              }
            };
            auto load_w = [&](int set, const char* w, int m) {
              wh[set] = *(const v8h*)(w + m * TR * 16);
              wl[set] = *(const v8h*)(w + (ROWS + m * TR) * 16);
            };
            load_x(0, ko[0]);
            load_w(0, w_b, 0);
            int k_next = ko[steps > 1 ? S : 0];
#define CNN355_MAC(a, x)                                                                                             \
  _Pragma("unroll") for (int ct = 0; ct < CT; ++ct) {                                                                \
    if constexpr (TR == 32) acc[m][ct] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, x[ct], acc[m][ct], 0, 0, 0);      \
    else acc[m][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, x[ct], acc[m][ct], 0, 0, 0);                         \
  }
#define CNN355_STEP(P, st)                                                                                           \
  {                                                                                                                  \
    const char* w_next = w_b + (st + 1 < steps ? S * 2 * ROWS * 16 : 0);                                             \
    _Pragma("unroll") for (int m = 0; m < RT; ++m) {                                                                 \
      constexpr int odd = (P)*RT & 1;                                                                                \
      const int set = (odd + m) & 1;                                                                                 \
      if (m + 1 < RT) load_w(set ^ 1, w_b, m + 1);                                                                   \
      else load_w(set ^ 1, w_next, 0);                                                                               \
      if (m == 0) {                                                                                                  \
        load_x((P) ^ 1, k_next);                                                                                     \
        k_next = ko[min(st + 2, steps - 1) * S];                                                                     \
      }                                                                                                              \
      CNN355_MAC(wh[set], xh[P])                                                                                     \
      CNN355_MAC(wh[set], xl[P])                                                                                     \
      CNN355_MAC(wl[set], xh[P])                                                                                     \
      __builtin_amdgcn_sched_barrier(0);                                                                             \
    }                                                                                                                \
    w_b = w_next;                                                                                                    \
  }
            for (int st = 0; st < steps; st += 2) {
              CNN355_STEP(0, st)
              if (st + 1 >= steps) break;
              CNN355_STEP(1, st + 1)
            }
          }
#undef CNN355_STEP
#undef CNN355_MAC
          pairs += here;
          if (pairs + g.slab > longest || (last && sl + 1 == slabs)) {
            pairs = 0;
#pragma unroll
            for (int m = 0; m < RT; ++m)
#pragma unroll
              for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                for (int v = 0; v < AV; ++v) { tot[m][ct][v] += acc[m][ct][v]; acc[m][ct][v] = 0.f; }
          }
          // here and not behind the barrier: the wait would take in the stores of the results
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
      }
      // element v of a lane, 32-row tiles: row (v / 4) * 8 + (lane / 32) * 4 + v % 4 of the tile, column lane % 32;
      // 16-row tiles: row (lane / 16) * 4 + v, column lane % 16
      // (worked out here: what depends on a row only would otherwise be kept in registers over all of the arithmetic)
      int lk4 = lk * 4;
      asm volatile("" : "+v"(lk4));
      auto row_of = [&](int m, int v) { return m * TR + (TR == 32 ? (v >> 2) * 8 + lk4 + (v & 3) : lk4 + v); };
      // the output of row r from a window's best sum times 2^-e
      auto finish = [&](int r, float sv, int e) {
        sv = ldexpf(sv, e);
        if constexpr (FC)
          if (g.drop) sv = fmaxf(sv, -INFINITY);
        return b_act(sv + lds_b[r]);
      };
      const gf out_z = FC ? g.out + (long long)blockIdx.z * g.slice_stride : g.out;
      const unsigned plane_out = (unsigned)g.split_out * 16u;
      CNN_GLOBAL unsigned char* marks = g.out_marks.at + (size_t)blockIdx.y * (unsigned)g.split_out;
      auto store = [&](int w, int r, float out, bool whole) {
        const int j = j0 + r;
        if (g.split_out) {   // (the last map brings the zeros that fill its group up)
          const unsigned off = (unsigned)(j >> 3) * 2u * plane_out + (unsigned)w * 16u + (unsigned)(j & 7) * 2u;
          if (whole) put_whole((CNN_GLOBAL char*)g.out, plane_out, off, out);
          else put_split((CNN_GLOBAL char*)g.out, plane_out, off, out);
          if (j == g.Mo - 1)
            for (int u = 1; u < 8 - (j & 7); ++u) put_split((CNN_GLOBAL char*)g.out, plane_out, off + 2u * u, 0.f);
          return;
        }
        const int b = fast_div(w, g.by_win_img);
        (out_z + (long long)b * g.out_stride)[j * g.win_img + w - b * g.win_img] = out;
      };
      if (M == 1 || M == 4) {
        const int q = M == 4 ? lane & 3 : 0;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const int c = (wave * CT + ct) * TR + lrow;
          const int w = cb * g.wins + (M == 4 ? c >> 2 : c);
          const bool ok = w < g.n_win && (M == 4 ? c >> 2 : c) < g.wins;
          // the sums of four rows of a lane, eight (TR = 32) or sixteen of the tile, as outputs (M == 4: the one of row + q)
          auto outputs = [&](int m, int v4, int row, float sum, float (&sv)[4]) {
            if (M == 4) {
              sv[0] = pool_quad(sum, tot[m][ct][v4 + 1], tot[m][ct][v4 + 2], tot[m][ct][v4 + 3], q);
              sv[0] = finish(row + q, sv[0], lds_e[row + q]);
            } else {
#pragma unroll
              for (int u = 0; u < 4; ++u) sv[u] = finish(row + u, u ? tot[m][ct][v4 + u] : sum, lds_e[row + u]);
            }
          };
          if (!g.split_out) {
            const int b = ok ? fast_div(w, g.by_win_img) : 0, wi = ok ? w - b * g.win_img : 0;
            const unsigned o0 = (unsigned)b * (unsigned)g.out_stride + (unsigned)wi;
            if constexpr (FC)
              if (g.raw) {   // (not a branch of every output: the code jumped to and fro, a trip to memory each time)
#pragma unroll
                for (int m = 0; m < RT; ++m)
#pragma unroll
                  for (int v = 0; v < AV; ++v) {
                    const int row = row_of(m, v);
                    if (ok && j0 + row < g.Mo) out_z[o0 + (unsigned)(j0 + row)] = ldexpf(tot[m][ct][v], lds_e[row]);
                  }
                continue;
              }
#pragma unroll
            for (int m = 0; m < RT; ++m) {
#pragma unroll
              for (int v4 = 0; v4 < AV; v4 += 4) {
                __builtin_amdgcn_sched_barrier(0);   // (fewer registers: the next rows' work stays behind this one's)
                const int first = m * TR + v4 * 2, row = first + lk4;   // (TR = 16: v4 is 0)
                if (j0 + first >= g.Mo) break;
                float sv[4];
                outputs(m, v4, row, tot[m][ct][v4], sv);
                if (M == 4) {
                  if (ok && j0 + row + q < g.Mo) out_z[o0 + (unsigned)(j0 + row + q) * (unsigned)g.win_img] = sv[0];
                } else {
#pragma unroll
                  for (int u = 0; u < 4; ++u)
                    if (ok && j0 + row + u < g.Mo) out_z[o0 + (unsigned)(j0 + row + u) * (unsigned)g.win_img] = sv[u];
                }
              }
            }
            continue;
          }
          // groups of eight maps: maps behind the last one are zero
          auto eights = [&](int m, int v4, float (&sv)[4]) {
            const int row = m * TR + v4 * 2 + lk4;
            const bool part = j0 + m * TR + v4 * 2 + (TR == 32 ? 8 : 16) > g.Mo;
            if (M == 4) {
              if (part && j0 + row + q >= g.Mo) sv[0] = 0.f;
              return !part || j0 + row + q < ((g.Mo + 7) & ~7);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (part && j0 + row + u >= g.Mo) sv[u] = 0.f;
            return !part || j0 + row < ((g.Mo + 7) & ~7);
          };
          auto off_of = [&]() { return (TR == 32 ? 0u : (unsigned)(lk4 >> 3) * 2u * plane_out) + (unsigned)w * 16u + (unsigned)(lk4 & 4) * 2u; };
          auto out_of = [&](int first) { return (CNN_GLOBAL char*)g.out + (size_t)((unsigned)(j0 + first) >> 3) * 2 * plane_out; };
          float most = 0.f;
#pragma unroll
          for (int m = 0; m < RT; ++m) {
#pragma unroll
            for (int v4 = 0; v4 < AV; v4 += 4) {
              __builtin_amdgcn_sched_barrier(0);
              const int first = m * TR + v4 * 2;
              if (j0 + first >= g.Mo) break;
              float sv[4];
              outputs(m, v4, first + lk4, tot[m][ct][v4], sv);
              const bool there = eights(m, v4, sv);
              if (M == 4) {
                most = fmaxf(most, fabsf(sv[0]));
                if (ok && there) put_split(out_of(first), plane_out, off_of() + (unsigned)q * 2u, sv[0]);
              } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) most = fmaxf(most, fabsf(sv[u]));
                if (ok && there) put_split4(out_of(first), plane_out, off_of(), sv);
              }
            }
          }
          unsigned long long small = __ballot(ok && !(most >= SPLIT_TINY));   // the lanes of a window
          if (M == 4) { small &= small >> 1; small &= small >> 2; small &= 0x1111111111111111ull; }
          for (int d = 32; d >= TR; d >>= 1) small &= small >> d;
          bool tiny = false;
          if (__builtin_expect(small != 0, 0)) {
            if (M == 4) { most = fmaxf(most, __shfl_xor(most, 1)); most = fmaxf(most, __shfl_xor(most, 2)); }
            for (int d = 32; d >= TR; d >>= 1) most = fmaxf(most, __shfl_xor(most, d));
            tiny = ok && most < SPLIT_TINY;
            if (!__any(tiny && most > 0.f)) tiny = false;   // (zeros are halves, and floats)
            else {                                          // once more: these are stored as they are
              if (lane == 0) mark_any(g.out_marks);
#pragma unroll
              for (int m = 0; m < RT; ++m)
#pragma unroll
                for (int v4 = 0; v4 < AV; v4 += 4) {
                  const int first = m * TR + v4 * 2;
                  if (j0 + first >= g.Mo) break;
                  float sum = tot[m][ct][v4], sv[4];
                  asm volatile("" : "+v"(lk4), "+v"(sum));   // (or what is worked out above is kept in registers for here)
                  outputs(m, v4, first + lk4, sum, sv);
                  const bool there = eights(m, v4, sv);
                  if (!tiny || !there) continue;
                  if (M == 4) put_whole(out_of(first), plane_out, off_of() + (unsigned)q * 2u, sv[0]);
                  else put_whole4(out_of(first), plane_out, off_of(), sv);
                }
            }
          }
          if (ok && lane < TR && q == 0) marks[w] = tiny;
        }
      } else {
        // a thread's window stays its own for all rows it takes
        const int rows = BT / g.wins, jr = tid / g.wins, wl = tid - jr * g.wins;
        const int w = cb * g.wins + wl;
        const bool ok = jr < rows && w < g.n_win;
        auto tiles = [&](auto whole, bool mine) {
          float most = 0.f;
#pragma unroll
          for (int m = 0; m < RT; ++m) {
            __syncthreads();   // the previous tile has been read
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
#pragma unroll
              for (int v = 0; v < AV; ++v) ep[(row_of(0, v)) * EPS + (wave * CT + ct) * TR + lrow] = tot[m][ct][v];
            __syncthreads();
            if (mine)
              for (int r = jr; r < TR; r += rows) {
                if (j0 + m * TR + r >= g.Mo) break;
                const float* win = ep + r * EPS + wl * M;
                float best = -INFINITY;
                for (int d = 0; d < M; ++d) best = fmaxf(best, win[d]);
                const float out = finish(m * TR + r, best, lds_e[m * TR + r]);
                most = fmaxf(most, fabsf(out));
                store(w, m * TR + r, out, whole);
              }
          }
          return most;
        };
        if (tid < g.wins) w_most[tid] = 0;
        const float most = tiles(std::false_type{}, ok);
        if (!g.split_out) continue;
        if (ok) atomicMax(&w_most[wl], __float_as_uint(most));
        __syncthreads();
        bool any = false;
        for (int x = lane; x < g.wins; x += 64) {   // (every wavefront looks at all of them)
          const float v = __uint_as_float(w_most[x]);
          any |= v > 0.f && v < SPLIT_TINY;
        }
        any = __any(any);
        if (wave == 0)
          for (int x = lane; x < g.wins && cb * g.wins + x < g.n_win; x += 64) marks[cb * g.wins + x] = any && __uint_as_float(w_most[x]) < SPLIT_TINY;
        if (__builtin_expect(any, 0)) {             // once more: these are stored as they are
          if (tid == 0) mark_any(g.out_marks);
          tiles(std::true_type{}, ok && __uint_as_float(w_most[min(wl, g.wins - 1)]) < SPLIT_TINY);
        }
      }
    }
  };
  // Products in 32 bits for a group with an infinite weight, and, behind those of halves, for blocks that read values that are no
  // halves: they are done again.  (Whether there are such values is asked for at the start and looked at here: a wait for it in
  // front of the halves cost every launch 0.5 us, 281 images of 20C4 11C5 182 us a call and 179.5.)  Code of its own: as a branch of
  // the step loop it cost the products of halves 2 % (30 registers), as one of a block 3 to 6 %.  4096 digits: 148 us a call in
  // halves; with an infinity in every 97th weight 402 (35600 with the sums of such rows by a thread an output), with all weights 1e-7
  // of that 519; 512 images of 300 maps a layer 431, 1467 (214000) and 1850.  k_batch_conv and k_batch_gemm took 292 and 1151.
  if (!slow) run(std::false_type{});
  marked = __builtin_amdgcn_readfirstlane(any_marks) != 0;
  if (slow || marked) run(std::true_type{});
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

// The last hidden layer's units (planes of sums added up, bias, scaled tanh, where they come as sums), the output layer and its
// units: a wavefront an image, 64 U hidden neurons' places, the output layer's weights in LDS.  One launch for k_batch_pool,
// k_batch_gemm, k_batch_pool and k_batch_outputs: 4096 digits 27.5 us -> 8.6, 512 images of 300 neurons 28 -> 9.7, 33 of 100 19 ->
// 6.2.  Bound by the latency of its loads, which are under way together: the weights, and four planes of the wavefront's first
// image (one after the other: 12.8, 20 and 8.5 us).
template <int U>
__global__ void __launch_bounds__(256) k_batch_tail(BatchTail g) {
  extern __shared__ float lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_w = g.n_out * g.n_hidden;
  float* lds_b = lds + n_w;
  float h[U], bias_h[U];
  auto load = [&](long long b) {
    const cgf p = g.in + b * g.n_hidden;
    unsigned at[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { at[u] = (unsigned)min(u * 64 + lane, g.n_hidden - 1); h[u] = 0.f; }
    constexpr int Q = U > 8 ? 2 : 4;
    int s = 0;
    for (; s + Q <= g.n_slices; s += Q) {
      float t[Q][U];
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int u = 0; u < U; ++u) t[q][u] = (p + (s + q) * g.slice_stride)[at[u]];
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int u = 0; u < U; ++u) h[u] += t[q][u];
    }
    for (; s < g.n_slices; ++s)
#pragma unroll
      for (int u = 0; u < U; ++u) h[u] += (p + s * g.slice_stride)[at[u]];
  };
  long long b = (long long)blockIdx.x * 4 + wave;
#pragma unroll
  for (int u = 0; u < U; ++u) bias_h[u] = g.bias_h ? g.bias_h[min(u * 64 + lane, g.n_hidden - 1)] : 0.f;
  if (b < g.n) load(b);
  int x = threadIdx.x;
  for (; x + 1792 < n_w; x += 2048) {
    float t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = g.w[x + u * 256];
#pragma unroll
    for (int u = 0; u < 8; ++u) lds[x + u * 256] = t[u];
  }
  float t[7];
#pragma unroll
  for (int u = 0; u < 7; ++u) t[u] = g.w[min(x + u * 256, n_w - 1)];
#pragma unroll
  for (int u = 0; u < 7; ++u)
    if (x + u * 256 < n_w) lds[x + u * 256] = t[u];
  if (threadIdx.x < g.n_out) lds_b[threadIdx.x] = g.bias[threadIdx.x];
  __syncthreads();
  int top = 32;                                    // lanes that hold outputs, halved
  while (top > 1 && top >= g.n_out) top >>= 1;
  for (; b < g.n; b += (long long)gridDim.x * 4) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (g.bias_h) h[u] = b_act(fmaxf(h[u], -INFINITY) + bias_h[u]);
      if (u * 64 + lane >= g.n_hidden) h[u] = 0.f;
    }
    float mine = -INFINITY;
    for (int k0 = 0; k0 < g.n_out; k0 += 8) {      // eight outputs' sums, halved over the lanes until lane 8 c + i has a part of sum c
      float s[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const float* w = lds + min(k0 + c, g.n_out - 1) * g.n_hidden;
        s[c] = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float v = w[min(u * 64 + lane, g.n_hidden - 1)];
          s[c] = fmaf(h[u], u * 64 + lane < g.n_hidden ? v : 0.f, s[c]);
        }
      }
#pragma unroll
      for (int d = 4; d; d >>= 1) {
        const bool up = lane & (d * 8);
#pragma unroll
        for (int c = 0; c < d; ++c) {
          const float keep = up ? s[c + d] : s[c], give = up ? s[c] : s[c + d];
          s[c] = keep + __shfl_xor(give, d * 8);
        }
      }
#pragma unroll
      for (int d = 4; d; d >>= 1) s[0] += __shfl_xor(s[0], d);
      const float v = __shfl(s[0], (lane & 7) * 8);
      if (lane >> 3 == k0 >> 3 && lane < g.n_out) mine = (g.drop ? fmaxf(v, -INFINITY) : v) + lds_b[lane];
    }
    float out = 0.f;
    if (g.out_units == 1) out = b_act(mine);
    else {
      float most = mine;
      for (int d = top; d; d >>= 1) most = fmaxf(most, __shfl_xor(most, d));
      const float e = lane < g.n_out ? expf(mine - most) : 0.f;
      float z = e;
      for (int d = top; d; d >>= 1) z += __shfl_xor(z, d);
      out = e / z;
    }
    if (lane < g.n_out) g.out[b * g.n_out + lane] = out;
    if (b + (long long)gridDim.x * 4 < g.n) load(b + (long long)gridDim.x * 4);
  }
}

// Wt[group of `row` maps][k][map] of every layer (blockIdx.y) from the canonical weights: k = (input map, ky, kx), j =
// output map; absent connections and the padding maps are zero.  Tiles of 64 k x 32 maps, turned round in LDS: rows of
// the canonical weights are read, rows of Wt written.  Two launches a layer (clear, scatter) before: 10000 digits 38 us
// of launches -> 5.
constexpr int PK = 64, PJ = 32;
// The slot of input map i in map j's row of a sparse table (the connections ascend), -1 where there is none
__device__ __forceinline__ int table_slot(const BatchPack& q, int j, int i) {
  int lo = q.csr_ptr[j], hi = q.csr_ptr[j + 1];
  const int end = hi;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (q.csr_idx[mid] < i) lo = mid + 1; else hi = mid;
  }
  return lo < end && q.csr_idx[lo] == i ? lo : -1;
}

// Weights of k_batch_split: a wavefront finds the largest finite weight of a row, whose power of two brings the row below
// 2^15; then the workgroup writes a piece of four rows in groups of eight k, high and low halves.  The pieces of a row find its
// largest weight each for itself: with a workgroup to four whole rows 300 maps of 4800 weights took 45 us, so 10.
typedef float v4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ void pack_split(const BatchPack& q, int* e4) {
  const int KK = q.K * q.Kx, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rows = (q.Mo + q.row - 1) / q.row * q.row, total = q.n_chunks * q.n_kg;
  const int pieces = (total + q.piece - 1) / q.piece;
  if (blockIdx.x == 0 && threadIdx.x == 0) *q.any = 0;
  for (int job = blockIdx.x; job < rows / 4 * pieces; job += gridDim.x) {
    const int tile = job / pieces, piece = job - tile * pieces;
    const int jw = tile * 4 + wave;
    float most = 0.f;
    bool inf = false;
    auto look = [&](float x) {
      x = fabsf(x);
      inf |= x == INFINITY;
      most = fmaxf(most, x < INFINITY ? x : 0.f);
    };
    if (jw < q.Mo) {
      const long long first = q.full_table ? (long long)jw * q.k_total : (long long)q.csr_ptr[jw] * KK;
      const int n = q.full_table ? q.k_total : (q.csr_ptr[jw + 1] - q.csr_ptr[jw]) * KK;
      const cgf w = q.w + first;
      int x0 = 0;
      for (; x0 + 256 <= n; x0 += 8 * 256) {
        v4f v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (x0 + u * 256 + 256 <= n) v[u] = *(const CNN_GLOBAL v4u*)(w + x0 + u * 256 + lane * 4);
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (x0 + u * 256 + 256 <= n)
            for (int i = 0; i < 4; ++i) look(v[u][i]);
      }
      for (int x = (n & ~255) + lane; x < n; x += 64) look(w[x]);
    }
    for (int d = 32; d; d >>= 1) most = fmaxf(most, __shfl_xor(most, d));
    int e = 0;
    if (most > 0.f) { frexpf(most, &e); e = 15 - e; }   // (most = f 2^x, f below 1: below 2^15 then)
    const int word = -(e + SPLIT_SHIFT) + (__any(inf) ? SPLIT_SLOW : 0);
    __syncthreads();
    if (lane == 0) { e4[wave] = e; q.exps[jw] = word; }
    __syncthreads();
    CNN_GLOBAL char* dst = (CNN_GLOBAL char*)q.wt + ((long long)(tile * 4 / q.row) * total * 2 * q.row + tile * 4 % q.row) * 16;
    const int end = min(total, (piece + 1) * q.piece) * 4;
    for (int u = piece * q.piece * 4 + threadIdx.x; u < end; u += 256) {
      const int r = u & 3, x = u >> 2, ch = x / q.n_kg, kg = x - ch * q.n_kg, at = ch * q.per_chunk + kg, c = at / KK, t = at - c * KK, j = tile * 4 + r;
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int map = c * 8 + i;
        v[i] = 0.f;
        if (j < q.Mo && kg < q.per_chunk && map < q.Mi) {
          if (q.full_table) v[i] = q.w[(long long)j * q.k_total + map * KK + t];
          else {
            const int slot = table_slot(q, j, map);
            if (slot >= 0) v[i] = q.w[(long long)slot * KK + t];
          }
        }
      }
      v8h h, l;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float s = ldexpf(v[i], e4[r]);
        h[i] = (_Float16)s;
        l[i] = fabsf(s) < INFINITY ? (_Float16)(s - (float)h[i]) : (_Float16)0.f;
      }
      CNN_GLOBAL char* p = dst + ((long long)x * 2 * q.row + r) * 16;
      *(CNN_GLOBAL v8h*)p = h;
      *(CNN_GLOBAL v8h*)(p + q.row * 16) = l;
    }
  }
}

__global__ void __launch_bounds__(256) k_batch_pack(BatchPackAll all) {
  __shared__ float t[PJ][PK + 1];
  const BatchPack q = all.l[blockIdx.y];
  if (q.exps) { pack_split(q, (int*)t); return; }
  const int KK = q.K * q.Kx, tk = (q.k_total + PK - 1) / PK;
  const int rows = (q.Mo + q.row - 1) / q.row * q.row, tiles = tk * ((rows + PJ - 1) / PJ);
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int j0 = tile / tk * PJ, k0 = tile % tk * PK;
    const int k = k0 + (threadIdx.x & (PK - 1));
    const int i = k / KK;
    if (q.full_table) {   // (a tile's loads under way together: a pass over 148000 x 600 weights 458 us, 498 with a loop of loads)
      float v[PJ * PK / 256];
      const int r0 = threadIdx.x / PK;
#pragma unroll
      for (int u = 0; u < PJ * PK / 256; ++u) {
        const int j = j0 + r0 + u * (256 / PK);
        v[u] = q.w[(long long)min(j, q.Mo - 1) * q.k_total + min(k, q.k_total - 1)];
      }
#pragma unroll
      for (int u = 0; u < PJ * PK / 256; ++u) {
        const int r = r0 + u * (256 / PK);
        t[r][k - k0] = j0 + r < q.Mo && k < q.k_total ? v[u] : 0.f;
      }
    } else {
      for (int r = threadIdx.x / PK; r < PJ; r += 256 / PK) {
        const int j = j0 + r, slot = j < q.Mo && k < q.k_total ? table_slot(q, j, i) : -1;
        t[r][k - k0] = slot >= 0 ? q.w[(long long)slot * KK + (k - i * KK)] : 0.f;
      }
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

// steps of 16 k that k_batch_first is compiled for, 0: more than that
int batch_first_steps(int k_total) {
  for (int H : {1, 2, 4, 5, 7})
    if (k_total <= 16 * H) return H;
  return 0;
}
size_t batch_first_lds_bytes(const BatchFirst& g) {
  const size_t rows = (size_t)g.T * 32;
  return (size_t)g.T * g.H * 2048 + (rows * g.k_total + rows * 2 + (size_t)16 * g.H + (g.share ? (size_t)4 * g.T * 1024 + 128 : 0)) * 4;
}
// workgroups a compute unit holds at once: registers, LDS
int batch_first_fit(const BatchFirst& g) {
  return std::max(1, std::min(first_waves(g.T, g.H), (int)(160 * 1024 / batch_first_lds_bytes(g))));
}

namespace {
template <int T, int H>
hipError_t launch_first(hipStream_t stream, const BatchFirst& g) {
  const size_t lds_bytes = batch_first_lds_bytes(g);
  hipError_t e = hipFuncSetAttribute((const void*)k_batch_first<T, H>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  if (e != hipSuccess) return e;
  const int groups = (g.Mo + T * 32 - 1) / (T * 32), wgs = (g.n_win + (g.share ? 31 : 127)) / (g.share ? 32 : 128);
  hipLaunchKernelGGL((k_batch_first<T, H>), dim3((unsigned)std::min(wgs, std::max(1, 256 * batch_first_fit(g) / groups)), (unsigned)groups),
                     dim3(BT), lds_bytes, stream, g);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_batch_first(hipStream_t stream, const BatchFirst& g) {
  if (g.n_win <= 0) return hipSuccess;
#define CNN355_CASE(T_, H_) \
  if (g.T == T_ && g.H == H_) return launch_first<T_, H_>(stream, g);
  CNN355_CASE(1, 1) CNN355_CASE(2, 1) CNN355_CASE(5, 1) CNN355_CASE(1, 2) CNN355_CASE(2, 2) CNN355_CASE(5, 2)
  CNN355_CASE(1, 4) CNN355_CASE(2, 4) CNN355_CASE(1, 5) CNN355_CASE(2, 5) CNN355_CASE(1, 7)
#undef CNN355_CASE
  return hipErrorInvalidValue;
}

size_t batch_split_lds_bytes(const BatchSplit& g) {
  const int M = g.Kp * g.Kpx, rows = g.RT * g.TR, cols = 4 * g.CT * g.TR;
  return 2 * (size_t)g.IC * 2 * g.run_px * 16 + 2 * (size_t)g.slab * rows * 32 + (size_t)g.n_kg * 4 + (size_t)rows * 8 +
         (M == 1 || M == 4 ? 0 : ((size_t)g.TR * (cols + 4) + g.wins) * 4);
}
// workgroups a compute unit holds at once: registers, LDS
int batch_split_fit(const BatchSplit& g) {
  return std::max(1, std::min(split_waves(g.RT, g.CT, g.TR), (int)(160 * 1024 / batch_split_lds_bytes(g))));
}

namespace {
template <int RT, int CT, int TR, bool FC>
hipError_t launch_split(hipStream_t stream, const BatchSplit& g) {
  const size_t lds_bytes = batch_split_lds_bytes(g);
  hipError_t e = hipFuncSetAttribute((const void*)k_batch_split<RT, CT, TR, FC>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  if (e != hipSuccess) return e;
  const int groups = (g.Mo + RT * TR - 1) / (RT * TR), slices = (g.n_cg / g.IC + g.cps - 1) / g.cps;
  const int gx = std::min(g.n_cb, std::max(1, 256 * batch_split_fit(g) / (groups * slices)));
  hipLaunchKernelGGL((k_batch_split<RT, CT, TR, FC>), dim3((unsigned)gx, (unsigned)groups, (unsigned)slices), dim3(BT), lds_bytes, stream, g);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_batch_split(hipStream_t stream, const BatchSplit& g) {
  if (g.n_win <= 0) return hipSuccess;
#define CNN355_CASE(RT_, CT_, TR_) \
  if (g.RT == RT_ && g.CT == CT_ && g.TR == TR_) return g.fc ? launch_split<RT_, CT_, TR_, true>(stream, g) : launch_split<RT_, CT_, TR_, false>(stream, g);
  CNN355_CASE(1, 1, 32) CNN355_CASE(1, 2, 32) CNN355_CASE(2, 1, 32) CNN355_CASE(2, 2, 32)
  CNN355_CASE(1, 2, 16) CNN355_CASE(1, 4, 16) CNN355_CASE(3, 2, 16) CNN355_CASE(3, 4, 16) CNN355_CASE(5, 2, 16) CNN355_CASE(7, 2, 16)
#undef CNN355_CASE
  return hipErrorInvalidValue;
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

hipError_t launch_batch_tail(hipStream_t stream, const BatchTail& g) {
  if (g.n <= 0) return hipSuccess;
  const size_t lds_bytes = ((size_t)g.n_out * g.n_hidden + g.n_out) * sizeof(float);
  const dim3 grid((unsigned)std::min<long long>((g.n + 3) / 4, 1024));
#define CNN355_CASE(U_) \
  if (g.n_hidden <= 64 * U_) { hipLaunchKernelGGL(k_batch_tail<U_>, grid, dim3(256), lds_bytes, stream, g); return hipGetLastError(); }
  CNN355_CASE(1) CNN355_CASE(2) CNN355_CASE(3) CNN355_CASE(5) CNN355_CASE(8) CNN355_CASE(16)
#undef CNN355_CASE
  return hipErrorInvalidValue;
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
    if (q.exps) { most = std::max(most, rows / 4 * ((q.n_chunks * q.n_kg + q.piece - 1) / q.piece)); continue; }
    most = std::max(most, (q.k_total + PK - 1) / PK * ((rows + PJ - 1) / PJ));
  }
  hipLaunchKernelGGL(k_batch_pack, dim3((unsigned)std::min(most, 4096ll), (unsigned)all.n), dim3(256), 0, stream, all);
  return hipGetLastError();
}

}  // namespace cnn355
