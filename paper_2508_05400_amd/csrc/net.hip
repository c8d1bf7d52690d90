// FP32 HIP kernels of the learned-start network and their C-ABI entry points.
//
// The network maps a coarse sample of the operator's velocity field
// (2 x h x w) to one start vector on the same grid; it is a stack of 3x3
// dilated convolutions with zero padding, ReLU between layers.  Training
// minimises the fraction of the prediction outside the wanted invariant
// subspace, 1 - ||V^T u||^2 / ||u||^2, with Adam.  The predicted vector is
// resampled bilinearly to the full grid and handed to rks_solve as u0.
// Tensors are dense row-major: activations B x C x H x W, weights
// O x C x 3 x 3, targets B x P x K (P = H W).
#include <hip/hip_runtime.h>

#include "rks.h"

namespace {

// A 3x3 dilated convolution with zero padding, in both directions.
//   forward (BWD = false): in = x, out(o) = bias[o] + sum over c, taps of w[o, c, tap] x(c, p + offset(tap)), ReLU
//   data gradient (BWD):   in = g, out(c) = sum over o, taps of w[o, c, tap] g(o, p - offset(tap)),
//                          g = dy, masked by y > 0 when RELU (act = y)
// One output is one chain of fused multiply-adds (input channels in order,
// taps in order), whatever OT and CU.
// A tap outside the image adds nothing: its input is taken as 0, which leaves
// the sum as it is unless a weight is infinite or NaN; a sum that ends
// infinite or NaN is formed again with those taps left out (conv_masked).
template <bool BWD, bool RELU>
__device__ __attribute__((noinline)) float conv_masked(const float* __restrict__ xb, const float* __restrict__ ab,
                                                       const float* __restrict__ w, float acc, int o, int CI, int CO,
                                                       int HW, int H, int W, int i, int j, int dil) {
  for (int c = 0; c < CI; ++c)
    for (int t = 0; t < 9; ++t) {
      const int di = BWD ? 1 - t / 3 : t / 3 - 1, dj = BWD ? 1 - t % 3 : t % 3 - 1;
      const int ii = i + dil * di, jj = j + dil * dj;
      if (ii < 0 || ii >= H || jj < 0 || jj >= W) continue;
      const int64_t e = (int64_t)c * HW + ii * W + jj;
      float v = xb[e];
      if (BWD && RELU && !(ab[e] > 0.f)) v = 0.f;
      acc = __builtin_fmaf(BWD ? w[((int64_t)c * CO + o) * 9 + t] : w[((int64_t)o * CI + c) * 9 + t], v, acc);
    }
  return acc;
}

// Reads at byte offsets from a pointer that all lanes share, 0 for an offset
// past the end.  With 32-bit offsets (IT = uint32_t, for tensors under 1 GiB;
// n its elements) they are buffer loads, for which the hardware does that:
// nothing has to be done to the value (and hence waited for) after the load.
// A row and a column outside the image add kOutRow and kOutCol to the offset,
// which keep any sum of an offset and one or both past the end.
template <typename IT>
struct Plane {  // tensors of any size
  static constexpr IT kOutRow = (IT)1 << (8 * sizeof(IT) - 1), kOutCol = kOutRow >> 1;
  const float* p;
  __device__ __forceinline__ Plane(const float* q, int64_t) : p(q) {}
  __device__ __forceinline__ float get(IT off) const {
    return off >= kOutCol ? 0.f : *(const float*)((const char*)p + off);
  }
};
template <>
struct Plane<uint32_t> {
  static constexpr uint32_t kOutRow = 0x80000000u, kOutCol = 0x40000000u;
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ Plane(const float* q, int64_t n)
      : r(__builtin_amdgcn_make_buffer_rsrc((void*)q, 0, (int)(4 * n), 0x00027000)) {}
  __device__ __forceinline__ float get(uint32_t off) const {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
  }
};

// A lane owns one pixel and OT output channels, so an input value is loaded
// once per tap for OT products, and the weights, which all lanes share, come
// through scalar loads; the nine taps of CU input channels are loaded before
// their first product (0 from offsets out of range for taps outside the
// image), contiguous across a wave.
template <int OT, int CU, bool BWD, bool RELU, typename IT>
__global__ __launch_bounds__(256) void k_conv(const float* __restrict__ in, const float* __restrict__ act,
                                              const float* __restrict__ w, const float* __restrict__ bias,
                                              float* __restrict__ out, int B, int CI, int CO, int H, int W, int dil) {
  const int HW = H * W;
  const int64_t total = (int64_t)B * HW;
  const int q0 = (int)(blockIdx.z * gridDim.y + blockIdx.y) * OT;  // first output channel
  if (q0 >= CO) return;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int b = sizeof(IT) == 4 ? (int)((uint32_t)idx / (uint32_t)HW) : (int)(idx / HW);
    const int pix = (int)(idx - (int64_t)b * HW);
    const int i = pix / W, j = pix - i * W;
    IT off[9];
    {
      IT ro[3], co[3];
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const int ii = i + dil * (BWD ? 1 - t : t - 1), jj = j + dil * (BWD ? 1 - t : t - 1);
        ro[t] = ii >= 0 && ii < H ? ((IT)b * CI * HW + (IT)ii * W) * 4 : Plane<IT>::kOutRow;
        co[t] = jj >= 0 && jj < W ? (IT)jj * 4 : Plane<IT>::kOutCol;
      }
#pragma unroll
      for (int t = 0; t < 9; ++t) off[t] = ro[t / 3] + co[t % 3];
    }
    float acc[OT];
#pragma unroll
    for (int q = 0; q < OT; ++q) acc[q] = BWD ? 0.f : bias[q0 + q < CO ? q0 + q : CO - 1];
    for (int c0 = 0; c0 < CI; c0 += CU) {
      float v[CU][9];
#pragma unroll
      for (int u = 0; u < CU; ++u) {
        const int64_t ch = (int64_t)(c0 + u < CI ? c0 + u : CI - 1) * HW;
        const Plane<IT> pi(in + ch, total * CI - ch);
#pragma unroll
        for (int t = 0; t < 9; ++t) v[u][t] = pi.get(off[t]);
        if constexpr (RELU && BWD) {
          const Plane<IT> pa(act + ch, total * CI - ch);
          float av[9];
#pragma unroll
          for (int t = 0; t < 9; ++t) av[t] = pa.get(off[t]);
#pragma unroll
          for (int t = 0; t < 9; ++t) v[u][t] = av[t] > 0.f ? v[u][t] : 0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < CU; ++u) {
        const int c = c0 + u;
        if (c < CI) {
#pragma unroll
          for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int q = 0; q < OT; ++q) {
              const int o = q0 + q < CO ? q0 + q : CO - 1;
              const float wt = BWD ? w[((int64_t)c * CO + o) * 9 + t] : w[((int64_t)o * CI + c) * 9 + t];
              acc[q] = __builtin_fmaf(wt, v[u][t], acc[q]);
            }
        }
      }
    }
    float* ob = out + (int64_t)b * CO * HW + pix;
#pragma unroll
    for (int q = 0; q < OT; ++q)
      if (q0 + q < CO) {
        float s = acc[q];
        if (!__builtin_isfinite(s))
          s = conv_masked<BWD, RELU>(in + (int64_t)b * CI * HW, RELU && BWD ? act + (int64_t)b * CI * HW : nullptr, w,
                                     BWD ? 0.f : bias[q0 + q], q0 + q, CI, CO, HW, H, W, i, j, dil);
        ob[(int64_t)(q0 + q) * HW] = (!BWD && RELU && s < 0.f) ? 0.f : s;
      }
  }
}

// One chain of k_conv_bwd_filter with g = 0 and outside taps left out one by
// one: for sums that came out infinite or NaN.
template <bool RELU>
__device__ __attribute__((noinline)) float filter_masked(const float* __restrict__ x, const float* __restrict__ dy,
                                                         const float* __restrict__ y, int B, int C, int O, int H,
                                                         int W, int dil, int c, int o, int t, int chain) {
  const int HW = H * W;
  float acc = 0.f;
  for (int64_t q = chain; q < (int64_t)B * HW; q += 256) {
    const int64_t b = q / HW;
    const int pix = (int)(q - b * HW);
    const int64_t e = (b * O + o) * HW + pix;
    float g = dy[e];
    if (RELU && !(y[e] > 0.f)) g = 0.f;
    if (g == 0.f) continue;
    const int ii = pix / W + dil * (t / 3 - 1), jj = pix % W + dil * (t % 3 - 1);
    if (ii >= 0 && ii < H && jj >= 0 && jj < W)
      acc = __builtin_fmaf(g, x[(b * C + c) * HW + ii * W + jj], acc);
  }
  return acc;
}

// dw[o, c, tap] = sum_{b, pixel} g[b, o, pixel] x[b, c, pixel + offset(tap)];
// db[o] = sum g[b, o, :] (g = dy, masked by y > 0 when RELU).  Every sum is
// 256 chains of fused multiply-adds (chain t takes the pixels t, t + 256, ...
// of the whole batch in order, leaving out g = 0 and taps outside the image),
// added by a fixed tree, so it does not depend on how the work is split.
// A workgroup owns one output channel, one input channel and NT taps (9, or
// the 3 of one row of the filter); its thread t runs chain t of all of them,
// with the loads of U pixels issued before the first product.  Taps outside
// the image have an offset out of range, which reads x = 0.  g = 0 and x = 0
// leave a finite sum as it is; a chain that ends infinite or NaN is run again
// with them left out.
template <int NT, int U, bool RELU, typename IT, bool TINY>
__global__ __launch_bounds__(256) void k_conv_bwd_filter(const float* __restrict__ x, const float* __restrict__ dy,
                                                         const float* __restrict__ y, float* __restrict__ dw,
                                                         float* __restrict__ db, int B, int C, int O, int H, int W,
                                                         int dil) {
  constexpr int NR3 = NT / 3;
  const int HW = H * W;
  const int tg = blockIdx.x % (9 / NT), oc = blockIdx.x / (9 / NT);
  const int c = oc % C, o = oc / C, t0 = tg * NT;
  const int64_t npix = (int64_t)B * HW;
  float acc[NT], ab = 0.f;
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = 0.f;
  // the chain's pixel: column j, row offset rw = W i, and the byte offsets
  // xo, go of its sample in x and dy; one step is 256 pixels
  const int sj = 256 % W, srw = 256 / W * W;
  const int drow = (dil < H ? dil : H) * W, dcol = dil < W ? dil : W;
  const int p0 = (int)threadIdx.x % HW;
  int j = p0 % W, rw = p0 - j;
  const IT xs = (IT)C * HW * 4, gs = (IT)O * HW * 4;
  IT xo = (IT)((int)threadIdx.x / HW) * xs, go = (IT)((int)threadIdx.x / HW) * gs;
  const float* xc = x + (int64_t)c * HW;
  const Plane<IT> px(xc, npix * C - (int64_t)c * HW);
  const int64_t ch = (int64_t)o * HW;
  auto load = [&](int64_t q, float(&g)[U], float(&yv)[U], float(&v)[U][NT]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = (IT)q + 256 * u < (IT)npix;
      const IT gb = in ? go + (IT)(rw + j) * 4 : Plane<IT>::kOutRow;
      g[u] = Plane<IT>(dy + ch, npix * O - ch).get(gb);
      yv[u] = RELU ? Plane<IT>(y + ch, npix * O - ch).get(gb) : 1.f;
      // the pixel's own row is in the image; the ones drow away are if they do not leave [0, HW)
      const IT xb = in ? xo : Plane<IT>::kOutRow;
      const IT co[3] = {j >= dcol ? (IT)(j - dcol) * 4 : Plane<IT>::kOutCol, (IT)j * 4,
                        j + dcol < W ? (IT)(j + dcol) * 4 : Plane<IT>::kOutCol};
#pragma unroll
      for (int r = 0; r < NR3; ++r) {
        const int e = t0 / 3 + r - 1;
        const int rr = rw + drow * e;
        IT ro = xb + (IT)rr * 4;
        if (e < 0) ro = rr >= 0 ? ro : Plane<IT>::kOutRow;
        if (e > 0) ro = rr < HW ? ro : Plane<IT>::kOutRow;
#pragma unroll
        for (int t = 0; t < 3; ++t) v[u][3 * r + t] = px.get(ro + co[t]);
      }
      j += sj;
      rw += srw;
      const int cj = j >= W ? W : 0;
      j -= cj;
      rw += cj;
      if (TINY) {
        while (rw >= HW) {
          rw -= HW;
          xo += xs;
          go += gs;
        }
      } else {
        const bool cr = rw >= HW;
        rw -= cr ? HW : 0;
        xo += cr ? xs : 0;
        go += cr ? gs : 0;
      }
    }
  };
  auto add = [&](const float(&dv)[U], const float(&yv)[U], const float(&v)[U][NT]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float g = yv[u] > 0.f ? dv[u] : 0.f;
      ab += g;
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = __builtin_fmaf(g, v[u][t], acc[t]);
    }
  };
  // two sets of registers: the next U pixels load while the current ones are added
  float g0[U], y0[U], v0[U][NT], g1[U], y1[U], v1[U][NT];
  load(threadIdx.x, g0, y0, v0);
  for (int64_t q = threadIdx.x; q < npix; q += 512 * U) {
    load(q + 256 * U, g1, y1, v1);
    __builtin_amdgcn_sched_barrier(0);
    add(g0, y0, v0);
    load(q + 512 * U, g0, y0, v0);
    __builtin_amdgcn_sched_barrier(0);
    add(g1, y1, v1);
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (!__builtin_isfinite(acc[t]))
      acc[t] = filter_masked<RELU>(x, dy, y, B, C, O, H, W, dil, c, o, t0 + t, threadIdx.x);
  // the tree over the chains: 128, 64, then 32 .. 1 apart
  constexpr int NR = NT + 1;
  __shared__ float red[NR][256];
#pragma unroll
  for (int t = 0; t < NT; ++t) red[t][threadIdx.x] = acc[t];
  red[NT][threadIdx.x] = ab;
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int t = wv; t < NR; t += 4) {
    float s = (red[t][lane] + red[t][lane + 128]) + (red[t][lane + 64] + red[t][lane + 192]);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) s += __shfl_down(s, d);
    if (lane == 0) {
      if (t < NT) dw[((int64_t)o * C + c) * 9 + t0 + t] = s;
      else if (c == 0 && tg == 0) db[o] = s;
    }
  }
}

// Per sample b: loss[b] = 1 - ||V_b^T u_b||^2/||u_b||^2 and
// du_b = -2 (V_b V_b^T u_b - rho u_b) / ||u_b||^2 / B.  One block per sample:
// each inner product is 256 chains (chain t takes p = t, t + 256, ...) and a
// fixed tree; four groups of 256 threads share the columns, and the loads of
// four p go out together (the samples are few, so the kernel is bound by
// latency: 23 us, 35 us with one group and one p at a time, for 32 samples of
// 4096 x 17).
__global__ __launch_bounds__(1024) void k_subspace_loss(const float* __restrict__ u, const float* __restrict__ V,
                                                        float* __restrict__ loss, float* __restrict__ du, int B,
                                                        int P, int K) {
  constexpr int KM = 32, KG = KM / 4, U = 4;
  const int b = blockIdx.x;
  const float* ub = u + (int64_t)b * P;
  const float* Vb = V + (int64_t)b * P * K;
  __shared__ float red[KM + 1][256];
  __shared__ float pk[KM + 1];
  const int t = threadIdx.x & 255, kg = threadIdx.x >> 8;  // columns kg, kg + 4, ...
  float acc[KG], uu0 = 0.f;
#pragma unroll
  for (int k = 0; k < KG; ++k) acc[k] = 0.f;
  for (int p = t; p < P; p += 256 * U) {
    float up[U], v[U][KG];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int pc = p + 256 * q < P ? p + 256 * q : p;
      up[q] = ub[pc];
#pragma unroll
      for (int k = 0; k < KG; ++k) v[q][k] = kg + 4 * k < K ? Vb[(int64_t)pc * K + kg + 4 * k] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < U; ++q)
      if (p + 256 * q < P) {
#pragma unroll
        for (int k = 0; k < KG; ++k) acc[k] = __builtin_fmaf(v[q][k], up[q], acc[k]);
        uu0 = __builtin_fmaf(up[q], up[q], uu0);
      }
  }
#pragma unroll
  for (int k = 0; k < KG; ++k) red[kg + 4 * k][t] = acc[k];
  if (kg == 0) red[KM][t] = uu0;
  __syncthreads();
  // the tree over the chains: 128, 64, then 32 .. 1 apart
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int k = wv; k <= KM; k += 16) {
    float s = (red[k][lane] + red[k][lane + 128]) + (red[k][lane + 64] + red[k][lane + 192]);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) s += __shfl_down(s, d);
    if (lane == 0) pk[k] = s;
  }
  __syncthreads();
  const float uu = pk[KM];
  float pp = 0.f;
  for (int k = 0; k < K; ++k) pp += pk[k] * pk[k];
  const float rho = pp / uu;
  if (threadIdx.x == 0) loss[b] = 1.f - rho;
  const float scale = -2.f / (uu * (float)B);
  for (int p = threadIdx.x; p < P; p += blockDim.x) {
    float vp = 0.f;
#pragma unroll 8
    for (int k = 0; k < K; ++k) vp += Vb[(int64_t)p * K + k] * pk[k];
    du[(int64_t)b * P + p] = scale * (vp - rho * ub[p]);
  }
}

__global__ __launch_bounds__(256) void k_adam(float* __restrict__ w, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, int64_t n, float lr,
                                              float b1, float b2, float eps, float c1, float c2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

// Bilinear resampling with half-pixel centres, clamped to the grid.
__global__ __launch_bounds__(256) void k_upsample(const float* __restrict__ u, int h, int w, double* __restrict__ out,
                                                  int H, int W) {
  const int64_t total = (int64_t)H * W;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int I = (int)(idx / W), J = (int)(idx % W);
    double y = ((double)I + 0.5) * h / H - 0.5;
    double x = ((double)J + 0.5) * w / W - 0.5;
    y = fmin(fmax(y, 0.0), (double)(h - 1));
    x = fmin(fmax(x, 0.0), (double)(w - 1));
    const int y0 = (int)floor(y), x0 = (int)floor(x);
    const int y1 = y0 + 1 < h ? y0 + 1 : h - 1, x1 = x0 + 1 < w ? x0 + 1 : w - 1;
    const double fy = y - y0, fx = x - x0;
    out[idx] = (1.0 - fy) * ((1.0 - fx) * u[y0 * w + x0] + fx * u[y0 * w + x1]) +
               fy * ((1.0 - fx) * u[y1 * w + x0] + fx * u[y1 * w + x1]);
  }
}

int grid_of(int64_t total) {
  int64_t g = (total + 255) / 256;
  if (g > 65535) g = 65535;
  return (int)(g < 1 ? 1 : g);
}

template <int OT, int CU, bool BWD>
void conv_launch_t(const float* in, const float* act, const float* w, const float* bias, float* out, int B, int CI,
                   int CO, int H, int W, int dil, int relu, int block, hipStream_t st) {
  const int64_t total = (int64_t)B * H * W;
  int64_t g = (total + block - 1) / block;
  if (g > 65535) g = 65535;
  const int gy = (CO + OT - 1) / OT;
  const dim3 grid((unsigned)g, gy < 32768 ? gy : 32768, (gy + 32767) / 32768);
  const bool small = total * (CI > CO ? CI : CO) < ((int64_t)1 << 28);  // 32-bit byte offsets reach every element
#define RKS_CONV_K(R, IT) k_conv<OT, CU, BWD, R, IT><<<grid, block, 0, st>>>(in, act, w, bias, out, B, CI, CO, H, W, dil)
  if (relu) {
    if (small) RKS_CONV_K(true, uint32_t);
    else RKS_CONV_K(true, uint64_t);
  } else {
    if (small) RKS_CONV_K(false, uint32_t);
    else RKS_CONV_K(false, uint64_t);
  }
#undef RKS_CONV_K
}

// Output channels per lane: the most of 8, 4, 2, 1 that the layer has and that
// still give three quarters of the 1,024 SIMDs a wave (more channels per lane
// load less, fewer run on more SIMDs).  Measured, microseconds, forward / data
// gradient of a 16-to-16 layer: 32 samples of 64 x 64 with 8 channels 16 / 23,
// with 1 channel 54 / 107; one sample with 8 channels 9 / 13, with 1 channel
// 4.4 / 7.3; 7 samples of 41 x 53 with 4 channels 6.5 / 7.0, 1: 9.4 / 16.
// (One output per thread, every input and weight loaded for each product and
// the taps skipped one by one: 87 / 161 and 16 / 28 for 32 samples and one.)
// Bound by the vector pipes: 604 MFLOP in 16 us, 38 TFLOP/s of about 79
// without packed arithmetic.
template <bool BWD>
void conv_launch(const float* in, const float* act, const float* w, const float* bias, float* out, int B, int CI,
                 int CO, int H, int W, int dil, int relu, hipStream_t st) {
  const int64_t waves = ((int64_t)B * H * W + 63) / 64;
  auto fits = [&](int ot) { return CO >= ot && waves * ((CO + ot - 1) / ot) >= 768; };
#define RKS_CONV(OT, CU, BLK) conv_launch_t<OT, CU, BWD>(in, act, w, bias, out, B, CI, CO, H, W, dil, relu, BLK, st)
  if (fits(8)) RKS_CONV(8, 2, 256);
  else if (fits(4)) RKS_CONV(4, 1, 256);
  else if (fits(2)) RKS_CONV(2, 2, 64);
  else RKS_CONV(1, 4, 64);
#undef RKS_CONV
}

template <int NT, int U>
void filter_launch_t(const float* x, const float* dy, const float* y, float* dw, float* db, int B, int C, int O, int H,
                     int W, int dil, int relu, hipStream_t st) {
  const unsigned grid = (unsigned)(O * C * (9 / NT));
  const bool small = (int64_t)B * H * W * (C > O ? C : O) < ((int64_t)1 << 28);
#define RKS_FILT_K(R, IT, T) k_conv_bwd_filter<NT, U, R, IT, T><<<grid, 256, 0, st>>>(x, dy, y, dw, db, B, C, O, H, W, dil)
  if (!small) {
    if (relu) RKS_FILT_K(true, uint64_t, true);
    else RKS_FILT_K(false, uint64_t, true);
  } else if (H * W < 256) {
    if (relu) RKS_FILT_K(true, uint32_t, true);
    else RKS_FILT_K(false, uint32_t, true);
  } else {
    if (relu) RKS_FILT_K(true, uint32_t, false);
    else RKS_FILT_K(false, uint32_t, false);
  }
#undef RKS_FILT_K
}

// One pair of channels per workgroup with all nine taps (1,024 waves for a
// 16-to-16 layer, one per SIMD), or one row of the filter where there are too
// few pairs for that.  Measured, microseconds, 32 samples of 64 x 64: 16 to 16
// channels 84 with nine taps, 120 with three; 2 to 16 and 16 to 1 channels 84
// and 76 with nine, 64 and 52 with three.  Two and four output channels per
// workgroup load less but leave SIMDs idle (105 and 150).  With the taps
// skipped one by one and each pixel's loads waited for: 820.  Bound by the
// instructions of the 512 serial steps of each chain (about 11 loads and 45
// vector instructions a step, one wave per SIMD).
void filter_launch(const float* x, const float* dy, const float* y, float* dw, float* db, int B, int C, int O, int H,
                   int W, int dil, int relu, hipStream_t st) {
  if ((int64_t)C * O >= 128)
    filter_launch_t<9, 4>(x, dy, y, dw, db, B, C, O, H, W, dil, relu, st);
  else
    filter_launch_t<3, 4>(x, dy, y, dw, db, B, C, O, H, W, dil, relu, st);
}

// A dilation that leaves the image in any case: every one from max(H, W) on is the same, and stays in range here.
int dil_in_range(int dil, int H, int W) { return dil < H || dil < W ? dil : (H > W ? H : W); }

int ok_or_hip() { return hipGetLastError() == hipSuccess ? RKS_OK : RKS_EHIP; }

}  // namespace

extern "C" {

int rks_net_conv3x3_forward(const float* x, const float* w, const float* b, float* y, int32_t B, int32_t Cin,
                            int32_t Cout, int32_t H, int32_t W, int32_t dil, int32_t relu, void* stream) {
  if (!x || !w || !b || !y || B < 1 || Cin < 1 || Cout < 1 || H < 1 || W < 1 || dil < 1) return RKS_EINVAL;
  dil = dil_in_range(dil, H, W);
  conv_launch<false>(x, nullptr, w, b, y, B, Cin, Cout, H, W, dil, relu, (hipStream_t)stream);
  return ok_or_hip();
}

int rks_net_conv3x3_backward(const float* x, const float* w, const float* y, const float* dy, float* dx, float* dw,
                             float* db, int32_t B, int32_t Cin, int32_t Cout, int32_t H, int32_t W, int32_t dil,
                             int32_t relu, void* stream) {
  if (!x || !w || !dy || !dw || !db || (relu && !y) || B < 1 || Cin < 1 || Cout < 1 || H < 1 || W < 1 || dil < 1)
    return RKS_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  dil = dil_in_range(dil, H, W);
  filter_launch(x, dy, y, dw, db, B, Cin, Cout, H, W, dil, relu, st);
  if (dx) conv_launch<true>(dy, y, w, nullptr, dx, B, Cout, Cin, H, W, dil, relu, st);
  return ok_or_hip();
}

int rks_net_subspace_loss(const float* u, const float* V, float* loss, float* du, int32_t B, int32_t P, int32_t K,
                          void* stream) {
  if (!u || !V || !loss || !du || B < 1 || P < 1 || K < 1 || K > 32) return RKS_EINVAL;
  k_subspace_loss<<<B, 1024, 0, (hipStream_t)stream>>>(u, V, loss, du, B, P, K);
  return ok_or_hip();
}

int rks_net_adam(float* w, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2, float eps,
                 int32_t t, void* stream) {
  if (!w || !g || !m || !v || n < 0 || t < 1) return RKS_EINVAL;
  const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
  k_adam<<<grid_of(n), 256, 0, (hipStream_t)stream>>>(w, g, m, v, n, lr, b1, b2, eps, c1, c2);
  return ok_or_hip();
}

int rks_net_upsample(const float* u, int32_t h, int32_t w, double* out, int32_t H, int32_t W, void* stream) {
  if (!u || !out || h < 1 || w < 1 || H < 1 || W < 1) return RKS_EINVAL;
  k_upsample<<<grid_of((int64_t)H * W), 256, 0, (hipStream_t)stream>>>(u, h, w, out, H, W);
  return ok_or_hip();
}

}  // extern "C"
