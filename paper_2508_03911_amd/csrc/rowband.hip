// Temporal transform fused with the last step of the angular spectrum.
//
// The column pass leaves z[t][y][kx]: every frame propagated, but for the
// inverse row transform.  That transform acts along x and the temporal one
// along t, so a workgroup takes one row y of a window (a few of a narrow
// frame), transforms the W samples of every kx in time, in the registers of one
// lane per kx, keeps the band's bins in LDS, inverse-transforms those rows and
// sums their weighted powers.  The window's rows are read once, nothing else is
// read or written, and only the nb rows of the band are transformed along x,
// not W.  (The order of the two linear steps is the one freedom used; every
// frame goes through all passes of the propagation before.)
//
// Bound: the reads (128 frames of 256^2 FP32, W = 32, 14 bins: 70 MB in 17.8 us
// with the launch).  Before, the W rows were inverse-transformed in LDS and
// reduced by a DFT GEMM there (24.3 us; fp16 20.8 -> 15.1), where they fitted
// (W nx <= 8192), else the field was written to memory and read back.  Passes,
// us, before and after: 16,384 frames of 64^2 515 -> 353, 1,024 of 256^2 395 -> 347
// (fp16 318 -> 269), 512 of 512^2 at W = 32 1298 -> 870, 1,280 of 320^2 1844 -> 1139.
#include <hip/hip_runtime.h>

#include "gmem.h"
#include "hv_internal.h"
#include "reg_fft.h"

using namespace hvk;

namespace {

typedef float f2v __attribute__((ext_vector_type(2)));
template <typename TIN> struct RawOf { using T = f2v; };
template <> struct RawOf<hv_h2> { using T = hv_h2; };

struct BandArgs {
  uint64_t mask;       // DFT bins of the band
  const int* index;    // [W]: place of bin k in the band
  int nb;
  float amp;           // scale of every amplitude
  float* out[3];
  float2* spec;        // [nwin][nb][ny * NX] or null
};

// Threads, rows per workgroup, and sequences that the waves transform at a
// time: whole sequences per wave, as many as fill its lanes in every pass of a
// power of two; 800 and 1280 take their columns in two rounds, 1024 too.
template <int NX>
constexpr int band_rows() {
  return NX < 256 ? 256 / NX : 1;
}
template <int NX, int ROWS_ = band_rows<NX>()>
struct BandShape {
  static constexpr int ROWS = ROWS_;
  static constexpr int NT = NX == 800 ? 448 : NX == 1280 ? 640 : NX == 1024 ? 512 : NX * ROWS;
  static constexpr int RW = NX <= 128 ? 8 : NX == 256 ? 4 : NX == 320 ? 3 : NX == 384 || NX == 512 || NX == 800 ? 2 : 1;
  static constexpr int GROUP = RW * (NT / 64);
  static constexpr int ROUNDS = (NX * ROWS + NT - 1) / NT;
  static constexpr int lds_rows(int nb) { return (nb * ROWS + GROUP - 1) / GROUP * GROUP; }
  static constexpr size_t lds_bytes(int nb) {
    return ((size_t)lds_rows(nb) * lds_stride(NX) + tw_size(NX)) * sizeof(float2);
  }
};

template <int NX, int W, typename TIN, int ROWS>
__global__ __launch_bounds__((BandShape<NX, ROWS>::NT), (W >= 64 || NX == 800 || NX == 1280 ? 2 : 4)) void k_row_band(const TIN* __restrict__ z, int ny,
                                                                                    int stride, int nwin,
                                                                                    const float* __restrict__ f1,
                                                                                    const float* __restrict__ f2,
                                                                                    BandArgs g) {
  using Sh = BandShape<NX, ROWS>;
  constexpr int NT = Sh::NT, GROUP = Sh::GROUP, S = lds_stride(NX);
  static_assert(wave_tile<GROUP, NT>(), "whole sequences per wave");
  extern __shared__ float2 lds[];
  float2* tw = lds;
  float2* buf = lds + tw_size(NX);
  const int tid = threadIdx.x;
  // Workgroups go to the 8 XCDs round-robin by linear index.  Where windows
  // overlap, the windows of one row group follow each other on one XCD, whose
  // L2 then holds the frames that they share.
  const int groups = ny / ROWS;
  int y, win;
  if (stride < W && groups % 8 == 0) {
    const int q = blockIdx.x >> 3;
    win = q % nwin;
    y = (q / nwin * 8 + (blockIdx.x & 7)) * ROWS;
  } else {
    win = blockIdx.x / groups;
    y = blockIdx.x % groups * ROWS;
  }
  y = __builtin_amdgcn_readfirstlane(y);  // keeps the rows' addresses in scalar registers
  win = __builtin_amdgcn_readfirstlane(win);
  const long npix = (long)ny * NX;
  const TIN* src = z + (long)win * stride * npix + (long)y * NX;
#pragma unroll 1
  for (int r = 0; r < Sh::ROUNDS; ++r) {
    const int e = tid + r * NT;  // element of the ROWS * NX run of each frame
    if ((ROWS * NX) % NT == 0 || e < ROWS * NX) {
      uint32_t off = (uint32_t)e * (uint32_t)sizeof(TIN);
      asm("" : "+v"(off));  // kept apart from the scalar base of each frame's row
      using Raw = typename RawOf<TIN>::T;
      Raw raw[W];
      constexpr int N1 = W <= 16 ? 1 : W / 8;  // the order in which the transform consumes them
#pragma unroll
      for (int n1 = 0; n1 < N1; ++n1)
#pragma unroll
        for (int n2 = 0; n2 < W / N1; ++n2) {
          typedef const __attribute__((address_space(1))) char* gptr;
          gptr row = (gptr)(src + (n1 + N1 * n2) * npix);
          asm("" : "+s"(row));  // a scalar base per frame, not a chain of vector ones
          raw[n1 + N1 * n2] = *(const __attribute__((address_space(1))) Raw*)(row + off);
        }
      if (r == 0) fill_twiddles<NX>(tw, tid, NT);
      float2 x[W];
#pragma unroll
      for (int t = 0; t < W; ++t) x[t] = make_float2((float)raw[t].x, (float)raw[t].y);
      reg_fft<W>(x);
      // the transform is done before the first branch of the stores: sunk into
      // their blocks it keeps both halves of every butterfly alive
#pragma unroll
      for (int k = 0; k < W; ++k) asm("" : "+v"(x[k].x), "+v"(x[k].y));
      float2* dst = buf + (e / NX) * S + place<NX>(e % NX);
#pragma unroll
      for (int k = 0; k < W; ++k)
        if (g.mask >> k & 1) dst[g.index[k] * (ROWS * S)] = x[k];
    }
  }
  __syncthreads();
  // sequence b * ROWS + row; a wave whose sequences are all past the band skips
  const int nseq = g.nb * ROWS;
  for (int s0 = 0; s0 < nseq; s0 += GROUP)
    if (s0 + (tid >> 6) * Sh::RW < nseq) fft_tile<NX, GROUP, NT, +1>(buf + s0 * S, tw, tid);
  __syncthreads();
  const long o = (long)win * npix + (long)y * NX;
  const float a2 = g.amp * g.amp;
  const bool images = g.out[0] || g.out[1] || g.out[2];
#pragma unroll 1
  for (int r = 0; r < Sh::ROUNDS; ++r) {
    const int e = tid + r * NT;
    if ((ROWS * NX) % NT != 0 && e >= ROWS * NX) continue;
    const float2* col = buf + (e / NX) * S + place<NX>(e % NX);
    if (g.spec) {
      float2* dst = g.spec + (long)win * g.nb * npix + (long)y * NX + e;
      for (int b = 0; b < g.nb; ++b) dst[b * npix] = c2::scale(col[b * (ROWS * S)], g.amp);
    }
    if (!images) continue;
    // four partial sums, bin 0, the largest, last: one chain of 30 bins loses twice as
    // much to rounding
    float m[3][4] = {};
    auto add = [&](int i, float2 v, float w1, float w2) {
      const float pw = v.x * v.x + v.y * v.y;
      m[0][i] += pw;
      m[1][i] += w1 * pw;
      m[2][i] += w2 * pw;
    };
    int b = g.nb;
#pragma unroll 1
    while (b & 3) {
      --b;
      add(0, col[b * (ROWS * S)], f1[b], f2[b]);
    }
#pragma unroll 1  // unrolled further, the weights come in pieces that are waited for one by one
    while (b > 0) {
      b -= 4;
      const float2* c = col + b * (ROWS * S);
#pragma unroll
      for (int i = 0; i < 4; ++i) add(i, c[i * (ROWS * S)], f1[b + i], f2[b + i]);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (g.out[i]) g.out[i][o + e] = ((m[i][0] + m[i][1]) + (m[i][2] + m[i][3])) * a2;
  }
}

template <int NX, int W, typename TIN, int ROWS = band_rows<NX>()>
void go(const void* z, int ny, int stride, int nwin, const float* f1, const float* f2, const BandArgs& a,
        hipStream_t st) {
  using Sh = BandShape<NX, ROWS>;
  // few windows of a narrow frame: a row per workgroup (64^2, one window: 9.3 -> 8.0 us)
  if constexpr (ROWS > 1)
    if (ny / ROWS * nwin < 512) return go<NX, W, TIN, 1>(z, ny, stride, nwin, f1, f2, a, st);
  hipLaunchKernelGGL((k_row_band<NX, W, TIN, ROWS>), dim3(ny / Sh::ROWS * nwin), dim3(Sh::NT), Sh::lds_bytes(a.nb), st,
                     (const TIN*)z, ny, stride, nwin, f1, f2, a);
}

template <int NX>
hv_status go_nx(const void* z, bool half_in, int ny, int stride, int nwin, const hvi::FieldBand& b, const BandArgs& a,
                hipStream_t st) {
  const int w = b.window;
  switch (w) {
    case 8: half_in ? go<NX, 8, hv_h2>(z, ny, stride, nwin, b.f1, b.f2, a, st) : go<NX, 8, float2>(z, ny, stride, nwin, b.f1, b.f2, a, st); break;
    case 16: half_in ? go<NX, 16, hv_h2>(z, ny, stride, nwin, b.f1, b.f2, a, st) : go<NX, 16, float2>(z, ny, stride, nwin, b.f1, b.f2, a, st); break;
    case 32: half_in ? go<NX, 32, hv_h2>(z, ny, stride, nwin, b.f1, b.f2, a, st) : go<NX, 32, float2>(z, ny, stride, nwin, b.f1, b.f2, a, st); break;
    case 64: half_in ? go<NX, 64, hv_h2>(z, ny, stride, nwin, b.f1, b.f2, a, st) : go<NX, 64, float2>(z, ny, stride, nwin, b.f1, b.f2, a, st); break;
    default: return hvi::fail(HV_ERR_SHAPE, "window %d not supported", w);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hvi::fail(HV_ERR_DEVICE, "row_band launch failed: %s", hipGetErrorString(e));
  return HV_OK;
}

size_t lds_of(int nx, int nb) {
  switch (nx) {
    case 64: return BandShape<64>::lds_bytes(nb);
    case 128: return BandShape<128>::lds_bytes(nb);
    case 256: return BandShape<256>::lds_bytes(nb);
    case 320: return BandShape<320>::lds_bytes(nb);
    case 384: return BandShape<384>::lds_bytes(nb);
    case 512: return BandShape<512>::lds_bytes(nb);
    case 800: return BandShape<800>::lds_bytes(nb);
    case 1024: return BandShape<1024>::lds_bytes(nb);
    case 1280: return BandShape<1280>::lds_bytes(nb);
  }
  return ~(size_t)0;
}

}  // namespace

namespace hvi {

bool no_field_workspace(int nx, int window) { return skewed(nx) && (long)nx * window <= 8192; }

// This kernel transforms the nb rows of the band of every window along x, the
// field path (K3, then field.hip) the s = min(stride, W) new rows, but that one
// writes the field and reads it back.  Where the band's rows fit the 160 KB of
// LDS of a CU, the line lies, by measurement (2^27 pixels of frames, this path /
// field path, us):
//   FP32, powers of two  nb = s     923/1075 (64^2, W 64), 1023/1192 (256^2, W 64), 1004/1275 (512^2, W 32)
//                        nb = 2 s   1329/1197, 1533/1546, 1498/1743: taken up to nb = 1.5 s
//   mixed radix, whose row transforms cost twice as much:
//                        15 of 32: 1139/1435 (320^2); 32 of 32: 1421/1449; 2 of 8: 1794/1891 (800^2); s = 4: 2258/1878
// fp16 storage keeps the field path, faster or not (753/796 at 512^2, W 32, but
// 1166/1073 with overlap): its images carry the rounding of the stored field, and
// stay what they were.
// Shapes without a field workspace always come here (their bands fit).
bool row_band_fits(int nx, int window, int stride, int nb, bool half) {
  if (no_field_workspace(nx, window)) return true;
  if (half || lds_of(nx, nb) > (size_t)160 << 10) return false;
  const int s = stride < window ? stride : window;
  return skewed(nx) ? 2 * nb <= 3 * s : nb < s && s >= 8;
}

hv_status launch_row_band(const void* z, bool half_in, int ny, int nx, int stride, int nwin, const FieldBand& b,
                          float amp, float* out0, float* out1, float* out2, float2* spec, hipStream_t st) {
  if (nwin <= 0) return HV_OK;
  const BandArgs a{b.mask, b.index, b.npair, amp, {out0, out1, out2}, spec};
  switch (nx) {
    case 64: return go_nx<64>(z, half_in, ny, stride, nwin, b, a, st);
    case 128: return go_nx<128>(z, half_in, ny, stride, nwin, b, a, st);
    case 256: return go_nx<256>(z, half_in, ny, stride, nwin, b, a, st);
    case 320: return go_nx<320>(z, half_in, ny, stride, nwin, b, a, st);
    case 384: return go_nx<384>(z, half_in, ny, stride, nwin, b, a, st);
    case 512: return go_nx<512>(z, half_in, ny, stride, nwin, b, a, st);
    case 800: return go_nx<800>(z, half_in, ny, stride, nwin, b, a, st);
    case 1024: return go_nx<1024>(z, half_in, ny, stride, nwin, b, a, st);
    case 1280: return go_nx<1280>(z, half_in, ny, stride, nwin, b, a, st);
  }
  return fail(HV_ERR_SHAPE, "nx=%d not supported", nx);
}

}  // namespace hvi
