// Temporal transforms of a field in memory with one lane per pixel: a lane
// holds the W samples of its pixel in registers, takes components out of
// them (PCA, SSA), transforms them in time and reduces them to the images
// (Sec. III-B.1).  The field is read once, with every load of a lane in flight
// together, and nothing goes through LDS.
//
// PCA and SSA keep the components c1..c2 of a window, X_f = X V_S V_S^H.  V is
// unitary, so the sum over the kept components is what is left of X when the
// others are taken out one after the other,
//   y = sum_t x_t V[t][c],  x_t -= conj(V[t][c]) y,
// which costs two passes over W registers per component left out: with the few
// that are left out in practice (the static one, the default) far less than
// forming the kept ones.  The subtraction is done on the samples, not on the
// energies, so what is left keeps single precision relative to |x| like the
// sum of the kept components does.
#include <hip/hip_runtime.h>

#include "gmem.h"
#include "hv_internal.h"
#include "reg_fft.h"

using namespace hvk;

namespace {

__device__ inline float2 load_c(const float2* p) { return *p; }
__device__ inline float2 load_c(const hv_h2* p) {
  hv_h2 h = *p;
  return make_float2((float)h.x, (float)h.y);
}

struct FieldArgs {
  const float2* vec;    // [nwin][component][W] (null: no components taken out)
  int c1, c2;           // kept components
  uint64_t mask;        // DFT bins of the band
  const float* wk;      // [2][W]: f_k, f_k^2
  const int* index;     // [W]: place of bin k in the band
  int npair;
  float amp;            // scale of every amplitude
  float* out[3];
  float2* spec;         // [nwin][npair][npix] or null
};

// sum_t x_t v_t in four partial sums
template <int W>
__device__ inline float2 dot(const float2* x, const float2* __restrict__ v) {
  float2 y[4] = {};
#pragma unroll
  for (int t = 0; t < W; ++t) {
    const float2 w = v[t];
    y[t & 3].x += x[t].x * w.x - x[t].y * w.y;
    y[t & 3].y += x[t].x * w.y + x[t].y * w.x;
  }
  return c2::add(c2::add(y[0], y[1]), c2::add(y[2], y[3]));
}

// Takes the components outside c1..c2 out of x.
template <int W>
__device__ inline void take_out(float2* x, const FieldArgs& g, long jj) {
  const int n = W - (g.c2 - g.c1 + 1);
  for (int i = 0; i < n; ++i) {
    const int c = i < g.c1 ? i : g.c2 + 1 + (i - g.c1);
    const float2* __restrict__ v = g.vec + (jj * W + c) * W;
    const float2 y = dot<W>(x, v);
#pragma unroll
    for (int t = 0; t < W; ++t) {
      const float2 w = v[t];
      x[t].x -= w.x * y.x + w.y * y.y;
      x[t].y -= w.x * y.y - w.y * y.x;
    }
  }
}

enum Mode { DFT, ENERGY_LEFT, ENERGY_OF };

constexpr int NTF = 256;

// DFT: moments and band bins of the window (after take_out when vec is given);
// ENERGY_LEFT: energy of the kept components as what is left without the
// others; ENERGY_OF: the sum over the kept components themselves.
template <int W, typename TIN, Mode MODE>
__global__ __launch_bounds__(NTF, (W >= 64 ? 3 : W >= 32 ? 4 : 6)) void k_field(const TIN* __restrict__ u, long npix,
                                                                               int stride, FieldArgs g) {
  const long jj = blockIdx.y;
  const long p0 = (long)blockIdx.x * NTF;
  const TIN* src = u + jj * stride * npix + p0;
  const uint32_t off = threadIdx.x * (uint32_t)sizeof(TIN);
  TIN raw[W];
  constexpr int N1 = W <= 16 ? 1 : W / 8;  // the order in which the transform consumes them
#pragma unroll
  for (int n1 = 0; n1 < N1; ++n1)
#pragma unroll
    for (int n2 = 0; n2 < W / N1; ++n2) raw[n1 + N1 * n2] = ld_off(src + (n1 + N1 * n2) * npix, off);
  float2 x[W];
#pragma unroll
  for (int t = 0; t < W; ++t) x[t] = load_c(&raw[t]);
  const long o = jj * npix + p0 + threadIdx.x;
  const float a2 = g.amp * g.amp;
  if constexpr (MODE == DFT) {
    if (g.vec) take_out<W>(x, g, jj);
    reg_fft<W>(x);
    if (g.spec) {
      float2* dst = g.spec + jj * g.npair * npix + p0 + threadIdx.x;
#pragma unroll
      for (int k = 0; k < W; ++k)
        if (g.mask >> k & 1) dst[g.index[k] * npix] = c2::scale(x[k], g.amp);
    }
    if (!g.out[0] && !g.out[1] && !g.out[2]) return;
    // four partial sums, bin 0, the largest, last: one chain of 30 bins loses twice as
    // much to rounding
    float e[3][4] = {};
#pragma unroll
    for (int k = W - 1; k >= 0; --k) {
      if (g.mask >> k & 1) {
        const float pw = x[k].x * x[k].x + x[k].y * x[k].y;
        e[0][k & 3] += pw;
        e[1][k & 3] += g.wk[k] * pw;
        e[2][k & 3] += g.wk[W + k] * pw;
      }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (g.out[i]) g.out[i][o] = ((e[i][0] + e[i][1]) + (e[i][2] + e[i][3])) * a2;
  } else if constexpr (MODE == ENERGY_LEFT) {
    take_out<W>(x, g, jj);
    float e[4] = {};
#pragma unroll
    for (int t = 0; t < W; ++t) e[t & 3] += x[t].x * x[t].x + x[t].y * x[t].y;
    g.out[0][o] = ((e[0] + e[1]) + (e[2] + e[3])) * a2;
  } else {
    float e = 0.f, e1 = 0.f;  // of every other component
    for (int c = g.c1; c <= g.c2; ++c) {
      const float2 y = dot<W>(x, g.vec + (jj * W + c) * W);
      const float t = e1;
      e1 = e + (y.x * y.x + y.y * y.y);
      e = t;
    }
    g.out[0][o] = (e + e1) * a2;
  }
}

template <int W, Mode MODE>
void go_field(const void* u, bool half_in, long npix, int stride, int nwin, const FieldArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)(npix / NTF), nwin);
  if (half_in)
    hipLaunchKernelGGL((k_field<W, hv_h2, MODE>), grid, dim3(NTF), 0, st, (const hv_h2*)u, npix, stride, a);
  else
    hipLaunchKernelGGL((k_field<W, float2, MODE>), grid, dim3(NTF), 0, st, (const float2*)u, npix, stride, a);
}

hv_status launched(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hvi::fail(HV_ERR_DEVICE, "%s launch failed: %s", what, hipGetErrorString(e));
  return HV_OK;
}

// Components that the lane-per-pixel kernel takes out (a range with few left
// out) or sums (a range of few), and past which the coefficient GEMM over the
// kept components is the faster one.  A component costs a lane one (sum) or two
// (take out) passes over W registers, which hide behind the reads of the field
// up to a number, larger for the wider FP32 field.  Measured on 512 frames of
// 512^2, this kernel / GEMM, us, W = 16, 32, 64 (ranges of PCA, then SSA):
//   FP32 8 out 197/305, 271/444, 361/852; 12 out 198/308, 392/437, 526/849
//        12 of -, 214/275, 244/372; 24 of -, -, 431/530
//        SSA 6 out 246/316, 249/290, 334/535; 8 out 298/317, 297/289, 417/534
//   fp16 4 out 162/181, 155/182, 205/296; 6 out 229/181, 221/181, 298/293
//        6 of 124/180, 121/147, 133/177; 8 of 155/182, 153/150, 165/177
//        SSA 2 out 129/186, 140/155, 177/228; 4 out 180/185, 187/153, 262/227
bool few_out(bool half, int window, int c1, int c2) { return window - (c2 - c1 + 1) <= (half ? 4 : 8); }
bool few_of(bool half, int c1, int c2) { return c2 - c1 + 1 <= (half ? 6 : 12); }

}  // namespace

namespace hvi {

bool field_dft_fits(bool half_in, int window, int c1, int c2) {
  return window - (c2 - c1 + 1) <= (half_in ? 2 : 6);
}

bool field_energy_fits(bool half_in, int window, int c1, int c2) {
  return few_of(half_in, c1, c2) || few_out(half_in, window, c1, c2);
}

hv_status launch_field_dft(const void* u, bool half_in, long npix, int stride, int nwin, const FieldBand& b,
                           const float2* vec, int c1, int c2, float amp, float* out0, float* out1, float* out2,
                           float2* spec, hipStream_t st) {
  if (nwin <= 0) return HV_OK;
  if (npix % NTF) return fail(HV_ERR_SHAPE, "pixel count %ld not a multiple of %d", npix, NTF);
  const FieldArgs a{vec, c1, c2, b.mask, b.wk, b.index, b.npair, amp, {out0, out1, out2}, spec};
  switch (b.window) {
    case 8: go_field<8, DFT>(u, half_in, npix, stride, nwin, a, st); break;
    case 16: go_field<16, DFT>(u, half_in, npix, stride, nwin, a, st); break;
    case 32: go_field<32, DFT>(u, half_in, npix, stride, nwin, a, st); break;
    case 64: go_field<64, DFT>(u, half_in, npix, stride, nwin, a, st); break;
    default: return fail(HV_ERR_SHAPE, "window %d not supported", b.window);
  }
  return launched("field_dft");
}

hv_status launch_field_energy(const void* u, bool half_in, long npix, int stride, int nwin, int window,
                              const float2* vec, int c1, int c2, float amp, float* m0, hipStream_t st) {
  if (nwin <= 0) return HV_OK;
  if (npix % NTF) return fail(HV_ERR_SHAPE, "pixel count %ld not a multiple of %d", npix, NTF);
  const FieldArgs a{vec, c1, c2, 0, nullptr, nullptr, 0, amp, {m0, nullptr, nullptr}, nullptr};
  const bool left = few_out(half_in, window, c1, c2) &&
                    (!few_of(half_in, c1, c2) || 2 * (window - (c2 - c1 + 1)) < c2 - c1 + 1);  // the fewer passes
#define HV_ENERGY(WV)                                                              \
  left ? go_field<WV, ENERGY_LEFT>(u, half_in, npix, stride, nwin, a, st)          \
       : go_field<WV, ENERGY_OF>(u, half_in, npix, stride, nwin, a, st);           \
  break;
  switch (window) {
    case 16: HV_ENERGY(16)
    case 32: HV_ENERGY(32)
    case 64: HV_ENERGY(64)
    default: return fail(HV_ERR_SHAPE, "window %d not supported", window);
  }
#undef HV_ENERGY
  return launched("field_energy");
}

}  // namespace hvi
