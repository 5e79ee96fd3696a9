// On-line deformation of training images (Sec. 4.1: affine maps -- translation, rotation, scaling,
// horizontal shearing -- combined with elastic deformations after Simard et al. 2003; Sec. 4.2, 4.3:
// random translations), one workgroup per image.  It depends on no weight, so it runs fully parallel
// over a batch of presentations ahead of the on-line training chain, on the same stream.
//
// Every random number is a function of (seed, presentation number, draw number) alone: mix64, the output
// function of SplitMix64 (Steele, Lea, Flood 2014), applied to key + GOLDEN * (draw + 1), where the key
// of a presentation is mix64(seed + GOLDEN * (presentation + 1)).  A draw's two 32-bit halves give two
// numbers of 24 bits each, so the same values exist exactly in float and in double.
#include <hip/hip_runtime.h>

#include <algorithm>

// device pointers of the job descriptor are global-address-space pointers in this translation unit
#define CNN_GLOBAL __attribute__((address_space(1)))
#include "cnn355_dev.h"

namespace cnn355 {

namespace {

constexpr int DT = 256;  // threads per workgroup
constexpr unsigned long long GOLDEN = 0x9E3779B97F4A7C15ull;

__device__ __forceinline__ unsigned long long mix64(unsigned long long z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// 32 random bits -> [-1, 1) in steps of 2^-23
// (the bits opaque: half of a 64-bit number, they would be converted as 64 bits)
__device__ __forceinline__ float sym(unsigned int bits) {
  asm("" : "+v"(bits));
  return (float)(bits >> 8) * (2.0f / 16777216.0f) - 1.0f;
}

constexpr int SW = 4;    // outputs of one lane along the line being smoothed

// One pass of the separable Gaussian over both fields: the lane's SW outputs out[k], k = at .. at + SW - 1,
// of the line starting at `ax` / `ay` (elements `step` apart, `len` of them; outside counts as zero).  The loop
// runs over the source elements that reach any of the outputs; the tap that links source j to output k is
// tp[j - k]: as j advances the SW taps in use slide by one, so an iteration reads one tap and one element of
// each field for 2 * SW multiply-adds.  tp points at the centre tap; R + SW zeros lie on either side of the taps.
__device__ __forceinline__ void blur_strip(const float* ax, const float* ay, int at, int len, int step, const float* tp,
                                           int R, float (&ox)[SW], float (&oy)[SW]) {
  const int jlo = max(0, at - R), jhi = min(len - 1, at + SW - 1 + R);
  float t[SW];
#pragma unroll
  for (int o = 0; o < SW; ++o) {
    ox[o] = 0.f;
    oy[o] = 0.f;
    t[o] = tp[jlo - 1 - (at + o)];  // the taps of the element before the first
  }
  for (int j = jlo; j <= jhi; ++j) {
#pragma unroll
    for (int o = SW - 1; o > 0; --o) t[o] = t[o - 1];  // tp[j - (at + o)] = what output o - 1 used one element ago
    t[0] = tp[j - at];
    const float vx = ax[j * step], vy = ay[j * step];
#pragma unroll
    for (int o = 0; o < SW; ++o) {
      ox[o] = fmaf(t[o], vx, ox[o]);
      oy[o] = fmaf(t[o], vy, oy[o]);
    }
  }
}

// The affine part of presentation k: displacement = (A - I) (u, v) + (tx, ty), A = Rot . Shear . Scale.
// (In double: the products reach tens of pixels on large maps, where a float keeps 1e-5 of a pixel at best.)
struct Affine {
  double a00, a01, a10, a11, tx, ty;
};
__device__ __forceinline__ unsigned long long presentation_key(const DeformJob& J, long long k) {
  return mix64(J.seed + GOLDEN * (J.first_index + (unsigned long long)k + 1ull));
}
__device__ __forceinline__ Affine draw_affine(const DeformJob& J, unsigned long long key) {
  const unsigned long long d0 = mix64(key + GOLDEN * 1ull), d1 = mix64(key + GOLDEN * 2ull), d2 = mix64(key + GOLDEN * 3ull);
  const double theta = sym((unsigned int)(d1 >> 32)) * J.max_rot, sh = sym((unsigned int)d1) * J.max_shear;
  const double sx = 1.0 + sym((unsigned int)(d2 >> 32)) * J.max_scale, sy = 1.0 + sym((unsigned int)d2) * J.max_scale;
  double sn, cs;
  sincospi(theta, &sn, &cs);
  Affine A;
  A.tx = sym((unsigned int)(d0 >> 32)) * J.max_tx;
  A.ty = sym((unsigned int)d0) * J.max_ty;
  A.a00 = cs * sx - 1.0;
  A.a01 = (cs * sh - sn) * sy;
  A.a10 = sn * sx;
  A.a11 = (sn * sh + cs) * sy - 1.0;
  return A;
}

// The affine parts of a workgroup's next AFF images (blockIdx.x + gridDim.x i), one a lane: a sine and cosine in double
// cost more than a wavefront's share of a small image's pixels, and 64 lanes would work out the same ones.
constexpr int AFF = 16;
__device__ __forceinline__ const Affine& affine_of(const DeformJob& J, Affine* ring, long long k, int i) {
  if ((i & (AFF - 1)) == 0) {
    __syncthreads();  // the previous ones have been read
    const long long q = k + (long long)threadIdx.x * gridDim.x;
    if (threadIdx.x < AFF && q < J.n) ring[threadIdx.x] = draw_affine(J, presentation_key(J, q));
    __syncthreads();
  }
  return ring[i & (AFF - 1)];
}

// Where presentation k reads and writes; an index that names no source image gives an image of `fill`.
struct Image {
  const CNN_GLOBAL char* src;
  CNN_GLOBAL char* dst;
  long long k;
  bool known;
};
__device__ __forceinline__ Image image_of(const DeformJob& J, long long k) {
  const long long sz = (long long)J.C * (J.H * J.W);
  long long s = J.src_index ? (long long)__builtin_amdgcn_readfirstlane(J.src_index[k]) : k;
  const bool known = s >= 0 && s < J.n_src;
  if (!known) s = 0;
  return Image{(const CNN_GLOBAL char*)(J.src + s * sz), (CNN_GLOBAL char*)(J.dst + k * sz), k, known};
}

// N pixels (x[i], y[i]) of a lane, displaced by ax[i] + ex[i] and ay[i] + ey[i] (the affine map's share and the elastic
// part); pixels with !ok[i] are worked out and not written.  All loads of a map are in flight together, then the stores
// (a load behind a store waits for the store too).  A neighbour outside takes `fill`; what it reads is the nearest pixel
// inside, in a cache line that other lanes want too (a pixel at a time: 10000 turned 3x32x32 images 63 us, 67 with the
// image's first pixel), or, several pixels at a time, the image's first, which takes fewer instructions (60000 of 1x29x29
// translated 134 us, 145; in matrix form 331, 335).  Positions are floored in double, as they are worked out.  RARE: the
// caller wants the displacements, or they are unbounded.
template <int N, bool ELASTIC, bool RARE>
__device__ __forceinline__ void sample_pixels(const DeformJob& J, const Image& im, const int (&x)[N], const int (&y)[N],
                                              const bool (&ok)[N], const double (&ax)[N], const double (&ay)[N],
                                              const float (&ex)[N], const float (&ey)[N]) {
  const int H = J.H, W = J.W;
  float fx[N], fy[N];
  int x0[N], y0[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double dx = ax[i], dy = ay[i];
    if (ELASTIC) { dx += (double)ex[i]; dy += (double)ey[i]; }
    if (RARE && J.disp && ok[i]) {
      J.disp[(im.k * 2) * (H * W) + y[i] * W + x[i]] = (float)dx;
      J.disp[(im.k * 2 + 1) * (H * W) + y[i] * W + x[i]] = (float)dy;
    }
    if (RARE) {   // far outside in any direction reads the fill value only; the clamp keeps the integers small
      dx = fmin(fmax(dx, -(double)(W + 2)), (double)(W + 2));
      dy = fmin(fmax(dy, -(double)(H + 2)), (double)(H + 2));
    }
    const double fdx = floor(dx), fdy = floor(dy);
    fx[i] = (float)(dx - fdx);
    fy[i] = (float)(dy - fdy);
    x0[i] = x[i] + (int)fdx;
    y0[i] = y[i] + (int)fdy;
  }
  bool in00[N], in01[N], in10[N], in11[N];
  unsigned int o00[N], o01[N], o10[N], o11[N], od[N];  // bytes
  float w00[N], w01[N], w10[N], w11[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const bool in_x0 = (unsigned int)x0[i] < (unsigned int)W, in_x1 = (unsigned int)(x0[i] + 1) < (unsigned int)W;
    const bool in_y0 = (unsigned int)y0[i] < (unsigned int)H, in_y1 = (unsigned int)(y0[i] + 1) < (unsigned int)H;
    in00[i] = in_y0 && in_x0; in01[i] = in_y0 && in_x1; in10[i] = in_y1 && in_x0; in11[i] = in_y1 && in_x1;
    if (N == 1) {
      const int xa = min(max(x0[i], 0), W - 1), xb = min(max(x0[i] + 1, 0), W - 1);
      const int ya = __mul24(min(max(y0[i], 0), H - 1), W), yb = __mul24(min(max(y0[i] + 1, 0), H - 1), W);
      o00[i] = (unsigned int)(ya + xa) * 4u; o01[i] = (unsigned int)(ya + xb) * 4u;
      o10[i] = (unsigned int)(yb + xa) * 4u; o11[i] = (unsigned int)(yb + xb) * 4u;
    } else {
      const unsigned int at = (unsigned int)(__mul24(y0[i], W) + x0[i]) * 4u, row = (unsigned int)W * 4u;
      o00[i] = in00[i] ? at : 0u; o01[i] = in01[i] ? at + 4u : 0u;
      o10[i] = in10[i] ? at + row : 0u; o11[i] = in11[i] ? at + row + 4u : 0u;
    }
    od[i] = (unsigned int)(__mul24(y[i], W) + x[i]) * 4u;
    w00[i] = (1.f - fy[i]) * (1.f - fx[i]); w01[i] = (1.f - fy[i]) * fx[i]; w10[i] = fy[i] * (1.f - fx[i]); w11[i] = fy[i] * fx[i];
  }
  const unsigned int map_bytes = (unsigned int)(H * W) * 4u;
  const CNN_GLOBAL char* m = im.src;
  CNN_GLOBAL char* o = im.dst;
  for (int c = 0; c < J.C; ++c, m += map_bytes, o += map_bytes) {
    float v00[N], v01[N], v10[N], v11[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      // (opaque here, so that the address stays a uniform base and a 32-bit offset and no 64-bit sum per lane)
      asm("" : "+v"(o00[i]), "+v"(o01[i]), "+v"(o10[i]), "+v"(o11[i]), "+v"(od[i]));
      v00[i] = *(const CNN_GLOBAL float*)(m + o00[i]);
      v01[i] = *(const CNN_GLOBAL float*)(m + o01[i]);
      v10[i] = *(const CNN_GLOBAL float*)(m + o10[i]);
      v11[i] = *(const CNN_GLOBAL float*)(m + o11[i]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float a = in00[i] ? v00[i] : J.fill, b = in01[i] ? v01[i] : J.fill;
      const float d = in10[i] ? v10[i] : J.fill, e = in11[i] ? v11[i] : J.fill;
      v00[i] = im.known ? fmaf(w00[i], a, fmaf(w01[i], b, fmaf(w10[i], d, w11[i] * e))) : J.fill;
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (ok[i]) *(CNN_GLOBAL float*)(o + od[i]) = v00[i];
  }
}

// A lane PXL pixels at a time, all their loads in flight.  The smoothing (ELASTIC) as sums over a line, a strip of outputs
// a lane.
template <int PXL, bool ELASTIC, bool RARE>
__global__ void __launch_bounds__(DT) k_deform(const DeformJob J) {
  extern __shared__ float lds[];
  __shared__ Affine ring[AFF];
  const int H = J.H, W = J.W, HW = H * W, R = J.R;
  const int Wp = W | 1;       // odd row pitch: lanes on consecutive rows fall on different LDS banks
  float* rx = lds;            // [H][Wp] random fields, then the smoothed ones
  float* ry = lds + H * Wp;
  float* hx = lds + 2 * H * Wp;   // after the pass along rows
  float* hy = lds + 3 * H * Wp;
  float* taps = lds + 4 * H * Wp; // [R + SW zeros][2R + 1 taps][R + SW zeros]
  const float* tp = taps + 2 * R + SW;  // the centre tap
  const int tid = threadIdx.x;
  if constexpr (ELASTIC) {
    for (int i = tid; i < 4 * R + 2 * SW + 1; i += DT) {
      const int q = i - (R + SW);
      taps[i] = q >= 0 && q <= 2 * R ? J.taps[q] : 0.f;
    }
  }
  const double cx = 0.5 * (double)(W - 1), cy = 0.5 * (double)(H - 1);
  const int step_y = DT / W, step_x = DT - step_y * W, first_y = tid / W, first_x = tid - first_y * W;
  int i = 0;
  for (long long k = blockIdx.x; k < J.n; k += gridDim.x, ++i) {
    const unsigned long long key = presentation_key(J, k);
    const Affine A = affine_of(J, ring, k, i);
    // ---- the elastic part: two random fields, smoothed along rows, then along columns
    if constexpr (ELASTIC) {
      __syncthreads();  // the previous image's fields have been read
      unsigned long long ctr = key + GOLDEN * (unsigned long long)(tid + 4);
      for (int p = tid; p < HW; p += DT, ctr += GOLDEN * (unsigned long long)DT) {
        const unsigned long long d = mix64(ctr);
        const int y = p / W, x = p - y * W;
        rx[y * Wp + x] = sym((unsigned int)(d >> 32));
        ry[y * Wp + x] = sym((unsigned int)d);
      }
      __syncthreads();
      const int nsx = (W + SW - 1) / SW, nsy = (H + SW - 1) / SW;
      for (int it = tid; it < H * nsx; it += DT) {  // along rows; consecutive lanes take consecutive rows
        const int s = it / H, y = it - s * H, x0 = s * SW;
        float ox[SW], oy[SW];
        blur_strip(rx + y * Wp, ry + y * Wp, x0, W, 1, tp, R, ox, oy);
#pragma unroll
        for (int o = 0; o < SW; ++o)
          if (x0 + o < W) {
            hx[y * Wp + x0 + o] = ox[o];
            hy[y * Wp + x0 + o] = oy[o];
          }
      }
      __syncthreads();
      for (int it = tid; it < W * nsy; it += DT) {  // along columns; consecutive lanes take consecutive columns
        const int s = it / W, x = it - s * W, y0 = s * SW;
        float ox[SW], oy[SW];
        blur_strip(hx + x, hy + x, y0, H, Wp, tp, R, ox, oy);
#pragma unroll
        for (int o = 0; o < SW; ++o)
          if (y0 + o < H) {
            rx[(y0 + o) * Wp + x] = ox[o];
            ry[(y0 + o) * Wp + x] = oy[o];
          }
      }
      __syncthreads();
    }
    // ---- sample the source
    const Image im = image_of(J, k);
    int x = first_x, y = first_y;
    for (int p = tid; p < HW; p += PXL * DT) {
      int px[PXL], py[PXL];
      bool ok[PXL];
      double ax[PXL], ay[PXL];
      float ex[PXL], ey[PXL];
#pragma unroll
      for (int q = 0; q < PXL; ++q) {
        px[q] = x;
        py[q] = y;
        ok[q] = p + q * DT < HW;
        const double u = (double)x - cx, v = (double)y - cy;
        ax[q] = fma(A.a00, u, fma(A.a01, v, A.tx));
        ay[q] = fma(A.a10, u, fma(A.a11, v, A.ty));
        const int at = ok[q] ? y * Wp + x : 0;
        ex[q] = ELASTIC ? J.alpha * rx[at] : 0.f;
        ey[q] = ELASTIC ? J.alpha * ry[at] : 0.f;
        x += step_x;
        y += step_y;
        if (x >= W) { x -= W; ++y; }
      }
      sample_pixels<PXL, ELASTIC, RARE>(J, im, px, py, ok, ax, ay, ex, ey);
    }
  }
}

typedef float v4f __attribute__((ext_vector_type(4)));

// The same deformation with the Gaussian on the matrix cores: smoothing along a row is a product with the banded
// matrix G[j][x] = tap[j - x], smoothing along a column one with its transpose, both in tiles of 16 x 16
// (v_mfma_f32_16x16x4_f32: fp32 in, fp32 sums).  A wavefront takes a strip of 16 columns and walks down it:
//   rows:    Hx[yt][xt]  = sum over d of  Rand[yt][xt + d] . G_d
//   columns: V[yt - d]  += G_d' . Hx[yt]                          |d| <= D (further tiles are all zero or outside)
// Lane l = 16 g + c holds element k = 4 g + v of an operand's contraction at step v = 0 .. 3.  With that order a tile of
// Hx leaves the first product in the very registers the second one reads it from, and G_d is the same four registers in
// both (a tap depends on j - x alone), loaded once per workgroup.  Only the random fields pass through LDS: every one of
// the 2 D + 1 strips that read a tile would have to draw it again.  V[-D .. D] of the walk are 2 D + 1 tiles of sums.
// The fields lie in LDS with zeros around them up to whole tiles, at a row pitch of 4 x odd floats (a lane's four
// elements are one 128-bit read, 16 rows fall on different banks).
// Bound by vector-ALU issue (1930 instructions a 29 x 29 image: 37 a draw, 64 a sampled pixel), matrix pipes a quarter
// busy.  Before, sums by fmaf over a line, in a chain of passes: 60000 of 1x29x29 541 -> 331 us (1.2 TB/s; 358 under the
// profiler), 1000 of 2x96x96 380 -> 134 us.
// Pixels of a lane in flight together.  The bound of four wavefronts a SIMD leaves 128 registers; 16 of D = 2 and 43 of
// D = 3 lie in scratch memory as it is (8, 36 and 71 of D = 1, 2, 3 where the displacements are asked for), with four
// pixels more.
constexpr int PX = 2;
template <int D, bool RARE>
__global__ void __launch_bounds__(512, 4) k_deform_mx(const DeformJob J) {
  extern __shared__ float lds[];
  __shared__ Affine ring[AFF];
  const int H = J.H, W = J.W, HW = H * W, R = J.R;
  const int nxt = (W + 15) >> 4, nyt = (H + 15) >> 4;
  const int pitch = 16 * nxt + 4, plane = 16 * nyt * pitch;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63;
  const int c = lane & 15, g4 = (lane >> 4) * 4;
  v4f G[2 * D + 1];
#pragma unroll
  for (int d = 0; d <= 2 * D; ++d)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int off = 16 * (d - D) + g4 + v - c;
      const float t = J.taps[min(max(off + R, 0), 2 * DEFORM_MAX_R)];
      G[d][v] = off >= -R && off <= R ? t : 0.f;
    }
  for (int q = tid; q < 2 * plane; q += nt) lds[q] = 0.f;
  const double cx = 0.5 * (double)(W - 1), cy = 0.5 * (double)(H - 1);
  const int step_y = nt / W, step_x = nt - step_y * W;
  const int first_y = tid / W, first_x = tid - first_y * W;
  int n_done = 0;
  for (long long k = blockIdx.x; k < J.n; k += gridDim.x, ++n_done) {
    const unsigned long long key = presentation_key(J, k);
    const Affine& A = affine_of(J, ring, k, n_done);
    __syncthreads();  // the previous image's fields have been read
    {
      unsigned long long ctr = key + GOLDEN * (unsigned long long)(tid + 4);
      int x = first_x, at = first_y * pitch + first_x;
      for (int p = tid; p < HW; p += nt, ctr += GOLDEN * (unsigned long long)nt) {
        const unsigned long long d = mix64(ctr);
        lds[at] = sym((unsigned int)(d >> 32));
        lds[at + plane] = sym((unsigned int)d);
        x += step_x;
        at += step_y * pitch + step_x;
        if (x >= W) { x -= W; at += pitch - W; }
      }
    }
    const Image im = image_of(J, k);
    __syncthreads();
    for (int xt = __builtin_amdgcn_readfirstlane(tid >> 6); xt < nxt; xt += nt >> 6) {
      const int x = 16 * xt + c;
      const double u = (double)x - cx;
      const double ax = fma(A.a00, u, A.tx), ay = fma(A.a10, u, A.ty);
      v4f vx[2 * D + 1], vy[2 * D + 1];  // the tile of rows yt + D - i, i = 0 .. 2 D
#pragma unroll
      for (int i = 0; i <= 2 * D; ++i) { vx[i] = v4f{0.f, 0.f, 0.f, 0.f}; vy[i] = vx[i]; }
      for (int yt = 0; yt < nyt + D; ++yt) {
        if (yt < nyt) {
          v4f hx = v4f{0.f, 0.f, 0.f, 0.f}, hy = hx;
          const float* f = lds + (16 * yt + c) * pitch + 16 * xt + g4;
#pragma unroll
          for (int d = 0; d <= 2 * D; ++d) {
            if (xt + d - D < 0 || xt + d - D >= nxt) continue;
            const v4f fx = *(const v4f*)(f + 16 * (d - D)), fy = *(const v4f*)(f + plane + 16 * (d - D));
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              hx = __builtin_amdgcn_mfma_f32_16x16x4f32(fx[v], G[d][v], hx, 0, 0, 0);
              hy = __builtin_amdgcn_mfma_f32_16x16x4f32(fy[v], G[d][v], hy, 0, 0, 0);
            }
          }
#pragma unroll
          for (int i = 0; i <= 2 * D; ++i) {
            const int yo = yt + D - i;
            if (yo < 0 || yo >= nyt) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              vx[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(G[i][v], hx[v], vx[i], 0, 0, 0);
              vy[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(G[i][v], hy[v], vy[i], 0, 0, 0);
            }
          }
        }
        if (yt >= D) {   // tile yt - D has all its sums
          const double v0 = (double)(16 * (yt - D) + g4) - cy;
          const double bx = A.a01, by = A.a11, ax0 = fma(bx, v0, ax), ay0 = fma(by, v0, ay);
#pragma unroll
          for (int v = 0; v < 4; v += PX) {
            int px[PX], py[PX];
            bool ok[PX];
            double dx[PX], dy[PX];
            float ex[PX], ey[PX];
#pragma unroll
            for (int q = 0; q < PX; ++q) {
              px[q] = x;
              py[q] = 16 * (yt - D) + g4 + v + q;
              ok[q] = x < W && py[q] < H;
              dx[q] = fma(bx, (double)(v + q), ax0);
              dy[q] = fma(by, (double)(v + q), ay0);
              ex[q] = J.alpha * vx[2 * D][v + q];
              ey[q] = J.alpha * vy[2 * D][v + q];
            }
            sample_pixels<PX, true, RARE>(J, im, px, py, ok, dx, dy, ex, ey);
          }
        }
#pragma unroll
        for (int i = 2 * D; i > 0; --i) { vx[i] = vx[i - 1]; vy[i] = vy[i - 1]; }
        vx[0] = v4f{0.f, 0.f, 0.f, 0.f};
        vy[0] = vx[0];
      }
    }
  }
}

}  // namespace

static size_t line_lds_bytes(const DeformJob& J) { return ((size_t)4 * J.H * (J.W | 1) + 4 * J.R + 2 * SW + 1) * sizeof(float); }
static size_t mx_lds_bytes(const DeformJob& J) {
  return (size_t)2 * 16 * ((J.H + 15) / 16) * (16 * ((J.W + 15) / 16) + 4) * sizeof(float);
}

// Whether the matrix form smooths such images (J.R >= 0): the shape of the images and the width of the Gaussian decide, not
// how many there are, so that a stream gives the same bits however it is cut into calls.  Time models of the two forms in
// microseconds, fitted to 2900 random calls (1 to 16 maps of 1x1 to 200x47, sigma 0.3 to 16, 1 to 60000 images; 12 and 15 %
// off): draws, multiply-adds along lines or products of tiles, sampled pixels with the loads of their maps, in steps of a
// workgroup's lanes; first their share of a compute unit's issue slots, then their latency, once for every time the images
// fill the chip.  Matrix form where it costs many images at most 5 % and few at most 15 % more than sums over a line (which
// have become 8 % faster themselves).  Of the calls above 9 us 1 % are slower by it than with every map in line form
// before; with maps of more than 24 pixels and half full tiles, and of one tile, in matrix form 12 % were, by up to 50 %
// (narrow Gaussians on maps of two or three tiles, many maps an image).  Both sides, us, matrix form / line form: sigma 6,
// 60000 of 1x29x29 331 / 447, 1000 of 2x96x96 131 / 340, 10000 of 3x32x32 94 / 103, 877 of 16x29x29 59 / 54, 30000 of 16x16
// 39 / 100, 17x17 139 / 118, 24x24 150 / 168, 10000 of 24x64 156 / 132; sigma 0.8, 9773 of 36x36 136 / 84; sigma 1.3, 14 of
// 4x27x30 12.0 / 9.6.
bool deform_mx_is_faster(const DeformJob& J) {
  auto up = [](long long x, long long d) { return (x + d - 1) / d; };
  const size_t lds = mx_lds_bytes(J);
  if (lds > 150 * 1024) return false;   // (thin maps)
  const int H = J.H, W = J.W, R = J.R;
  const double C = J.C;
  const double rounds = (double)up((long long)H * W, DT);
  const double taps = (double)up(H * up(W, SW), DT) * (std::min(W, 2 * R + SW) + 4) + (double)up(W * up(H, SW), DT) * (std::min(H, 2 * R + SW) + 4);
  const int line_fit = std::max(1, std::min(6, (int)(160 * 1024 / line_lds_bytes(J))));
  const int nxt = (W + 15) / 16, nyt = (H + 15) / 16, D = std::min((R + 15) / 16, std::max(nxt, nyt) - 1), waves = std::min(nxt, 8);
  const double draws = (double)up((long long)H * W, 64 * waves), strips = (double)up(nxt, waves);
  const double steps = strips * (nyt + D) * (2 * D + 1), rows = strips * nyt;
  const int mx_fit = std::max(1, std::min(16 / waves, (int)(160 * 1024 / (lds + sizeof(Affine) * AFF))));
  auto within = [&](int n, double share) {
    const double line = 5.25 + n / 256.0 * (0.176 * rounds + 0.0036 * taps + 0.0161 * rounds * C) +
                        (double)up(n, 256 * line_fit) * (0.285 * rounds + 0.0509 * taps + 0.168 * rounds * C);
    const double mx = 5.19 + n / 256.0 * (waves / 4.0) * (0.173 * draws + 0.062 * steps + 0.166 * rows * C) +
                      (double)up(n, 256 * mx_fit) * (0.267 * draws + 0.104 * steps + 0.705 * rows + 0.412 * rows * C);
    return mx < share * line;
  };
  return within(1, 1.15) && within(256, 1.15) && within(1024, 1.15) && within(60000, 1.05);
}

template <int PXL, bool ELASTIC, bool RARE>
static hipError_t launch_deform_px(hipStream_t stream, const DeformJob& J, unsigned int grid) {
  const size_t lds = ELASTIC ? line_lds_bytes(J) : 0;
  hipError_t e = hipFuncSetAttribute((const void*)k_deform<PXL, ELASTIC, RARE>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_deform<PXL, ELASTIC, RARE>), dim3(grid), dim3(DT), lds, stream, J);
  return hipGetLastError();
}

template <int D, bool RARE>
static hipError_t launch_deform_mx(hipStream_t stream, const DeformJob& J, unsigned int grid) {
  const int nxt = (J.W + 15) / 16;
  const size_t lds = mx_lds_bytes(J);
  hipError_t e = hipFuncSetAttribute((const void*)k_deform_mx<D, RARE>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_deform_mx<D, RARE>), dim3(grid), dim3(64u * (nxt < 8 ? nxt : 8)), lds, stream, J);
  return hipGetLastError();
}

template <bool RARE>
static hipError_t launch_deform_any(hipStream_t stream, const DeformJob& J, unsigned int grid) {
  if (J.R < 0) {
    // Two pixels a lane keep more loads in flight: 60000 translated 1x29x29 images 133 us, one 159.  Turned images of
    // several maps lose by it (1559 of 8x48x48 85 us with one, 91 with two; 1000 of 2x96x96 70, 68), small maps leave the
    // second pixels idle.
    return J.C == 1 && J.H * J.W > 2 * DT ? launch_deform_px<2, false, RARE>(stream, J, grid) : launch_deform_px<1, false, RARE>(stream, J, grid);
  }
  if (!deform_mx_is_faster(J)) return launch_deform_px<1, true, RARE>(stream, J, grid);
  const int tx = (J.W + 15) / 16, ty = (J.H + 15) / 16, tiles = tx > ty ? tx : ty;
  const int d = (J.R + 15) / 16;   // neighbouring tiles a tap reaches, as far as there are any
  switch (d < tiles ? d : tiles - 1) {
    case 0: return launch_deform_mx<0, RARE>(stream, J, grid);
    case 1: return launch_deform_mx<1, RARE>(stream, J, grid);
    case 2: return launch_deform_mx<2, RARE>(stream, J, grid);
    case 3: return launch_deform_mx<3, RARE>(stream, J, grid);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_deform(hipStream_t stream, const DeformJob& J) {
  if (J.n <= 0) return hipSuccess;
  const unsigned int grid = (unsigned int)(J.n < 8192 ? J.n : 8192);
  return J.disp || !J.bounded ? launch_deform_any<true>(stream, J, grid) : launch_deform_any<false>(stream, J, grid);
}

}  // namespace cnn355
