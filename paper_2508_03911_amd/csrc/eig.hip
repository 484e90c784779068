// FP64 eigensolver of the PCA and SSA paths (Sec. III-B.1: the covariance of
// a window, its eigendecomposition): cyclic Jacobi for a Hermitian W x W
// matrix, one workgroup per window.
#include <hip/hip_runtime.h>

#include "hv_internal.h"

namespace {

struct dc {
  double x, y;
};

// The round-robin (circle) ordering.  Position pos holds one player (index);
// pair k is (T_k, B_k) = the players at positions k and W - 1 - k.  After a
// step, position 0 keeps its player and every other position takes that of the
// next one (position W - 1 that of position 1): T_k moves to T_{k-1}, B_k to
// B_{k+1}, T_1 to B_0 and B_{H-1} to T_{H-1}.  After W - 1 steps all are back.
struct Side {
  int k;   // pair
  int b;   // 0: T, 1: B
};
template <int H>
__device__ inline Side moved(Side s) {
  if (s.b) return s.k == H - 1 ? Side{H - 1, 0} : Side{s.k + 1, 1};
  return s.k == 0 ? Side{0, 0} : s.k == 1 ? Side{0, 1} : Side{s.k - 1, 0};
}

// The H (H - 1) / 2 blocks (i, j), i < j, in the order of the lanes that own
// them: first, for k = 0..H-1, the block that holds the pair k of the next
// step: (0, 1), (k - 1, k + 1), (H - 2, H - 1); then the others row by row.
// Row i >= 1 of the others holds j = i + 1, i + 3, i + 4, ..., row 0 j = 3, 4, ...
template <int H>
__device__ inline int row_start(int i) {  // blocks of the rows before i that do not lead
  return i * (H - 1) - i * (i - 1) / 2 - min(i, H - 2) - (i > 0) - (i > H - 2);
}
template <int H>
__device__ inline int block_of(int i, int j) {
  if (j - i == 2) return i + 1;
  if (j - i == 1 && i == 0) return 0;
  if (j - i == 1 && i == H - 2) return H - 1;
  return H + row_start<H>(i) + (i == 0 ? j - 3 : j == i + 1 ? 0 : j - i - 2);
}

__device__ inline double flip(double v, unsigned sign) {  // sign: 0 or 0x80000000
  return __hiloint2double(__double2hiint(v) ^ (int)sign, __double2loint(v));
}

// Barrier that orders LDS only: the rotation log's global stores stay in
// flight across it.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int W>
struct JacobiShape {
  static constexpr int H = W / 2;               // pairs of a step
  static constexpr int NBLK = H * (H - 1) / 2;  // 2 x 2 blocks above the diagonal
  static constexpr int NA = (NBLK + 63) / 64 * 64;
};

// The rotations of all steps, for the eigenvector kernel: pair k of step s of
// window j at ((j * max_steps + s) * H + k), steps[j] = the steps taken,
// rank[j][c] = the place of column c in descending order.
struct JacobiLog {
  double* c;
  dc* s;
  int* steps;
  int* rank;
  int max_sweeps;
};

// One rotation step zeroes A_pq of every pair (p, q) = (T_k, B_k) at once:
// J = [[c, s], [-conj s, c]] on columns (p, q) with a = A_pp, d = A_qq,
// b = A_pq, D = d - a, r = sqrt(D^2 + 4 |b|^2): cos^2 = (1 + |D| / r) / 2,
// s = sgn(D) b / (r c), and the diagonal becomes a - t|b|, d + t|b| with
// t|b| = sgn(D) |b|^2 / (r c^2): two reciprocal square roots in a chain.
//
// What bounds it: the chain of W - 1 dependent steps per sweep, about eight
// sweeps, on one CU per window.  A step therefore has one barrier and no
// address arithmetic:
//   * the matrix is held above the diagonal only, as the H (H - 1) / 2
//     independent 2 x 2 blocks of rows (T_i, B_i) by columns (T_j, B_j), one
//     per lane, stored by position: a lane reads its four entries at fixed
//     places of one LDS buffer and writes them where the next step looks for
//     them in the other, places that are the same in every step;
//   * the pairs of the next step come out of the leading blocks, so lanes
//     0..H-1 of wave 0, which hold the diagonal in registers, go on at once
//     to the next step's (c, s);
//   * the rotations are logged, and the eigenvectors are formed from the log
//     by a kernel that spreads their rows over the chip.
// Before, each step had two barriers, the parameters were computed between
// them (with a division and four roots in a chain), the full matrix and V
// went through LDS, and one lane sorted the eigenvalues: 1310 us per launch at
// W = 64 and 292 us at W = 32, against 386 and 167 us now, and 78 and 39 us for
// the eigenvectors.
template <int W>
__global__ __launch_bounds__((JacobiShape<W>::NA)) void k_jacobi(const double* __restrict__ cov,
                                                                 double* __restrict__ evals,
                                                                 double* __restrict__ offdiag, JacobiLog log) {
  using Sh = JacobiShape<W>;
  constexpr int H = Sh::H, NA = Sh::NA;
  __shared__ dc A[2][4][NA];  // entries TT, TB, BT, BB of every block
  __shared__ double pc[2][H];
  __shared__ dc ps[2][H];
  __shared__ double red[2][NA / 64];
  __shared__ double ev[W];
  const int tid = threadIdx.x, lane = tid & 63;
  const long jj = blockIdx.x;
  const dc* src = reinterpret_cast<const dc*>(cov) + jj * W * W;
  const bool act = tid < Sh::NBLK;  // owns a block
  const bool lead = tid < H;        // owns a leading block and the pair `tid`
  int bi = 0, bj = 1;
  if (lead) {
    bi = tid == 0 ? 0 : tid == H - 1 ? H - 2 : tid - 1;
    bj = tid == 0 ? 1 : tid == H - 1 ? H - 1 : tid + 1;
  } else if (act) {
    while (bi < H - 2 && row_start<H>(bi + 1) <= tid - H) ++bi;
    const int r = tid - H - row_start<H>(bi);
    bj = bi == 0 ? r + 3 : r == 0 ? bi + 1 : bi + 2 + r;
  }
  // where the block's four entries go: place e * NA + block, conjugated or
  // not; a leading block's entry that becomes a pair is kept in a register and
  // written to a place that no lane reads (of blocks NBLK .. NA - 1)
  constexpr int FREE = NA - Sh::NBLK;
  static_assert(4 * FREE >= H, "a free place for every pair");
  int to[4];
  unsigned sign[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const Side x = moved<H>({bi, e >> 1}), y = moved<H>({bj, e & 1});
    sign[e] = 0;
    if (x.k == y.k) {
      to[e] = (tid / FREE & 3) * NA + Sh::NBLK + tid % FREE;
      sign[e] = x.b ? 0x80000000u : 0u;
    } else if (x.k < y.k) {
      to[e] = (2 * x.b + y.b) * NA + block_of<H>(x.k, y.k);
    } else {
      to[e] = (2 * y.b + x.b) * NA + block_of<H>(y.k, x.k);
      sign[e] = 0x80000000u;
    }
  }
  // the rotated pair's zero entry
  int to_zero = 0;
  double da = 0.0, dd = 0.0, na = 0.0, nd = 0.0;
  dc b = {0.0, 0.0};
  if (lead) {
    const Side x = moved<H>({tid, 0}), y = moved<H>({tid, 1});
    to_zero = x.k < y.k ? (2 * x.b + y.b) * NA + block_of<H>(x.k, y.k) : (2 * y.b + x.b) * NA + block_of<H>(y.k, x.k);
    da = src[tid * W + tid].x;
    dd = src[(W - 1 - tid) * W + W - 1 - tid].x;
    b = src[tid * W + W - 1 - tid];
  }
  double off = lead ? b.x * b.x + b.y * b.y : 0.0;
  if (act) {
    const int p[2] = {bi, W - 1 - bi}, q[2] = {bj, W - 1 - bj};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int x = p[e >> 1], y = q[e & 1];
      dc v = x < y ? src[x * W + y] : src[y * W + x];  // above the diagonal
      if (x > y) v.y = -v.y;
      A[0][e][tid] = v;
      off += v.x * v.x + v.y * v.y;
    }
  }
  // rotation of pair `tid` from its diagonal (da, dd) and b; new diagonal in na, nd
  auto rotation = [&](int buf) {
    const double b2 = b.x * b.x + b.y * b.y;
    const double D = dd - da, r2 = D * D + 4.0 * b2;
    // |b| negligible: no rotation
    const bool none = b2 == 0.0 || b2 < 1e-300 * (da * da + dd * dd) || r2 < 1e-290;
    const double inv = rsqrt(none ? 1.0 : r2);
    const double c2 = 0.5 + 0.5 * fabs(D) * inv;
    const double ic = rsqrt(none ? 1.0 : c2);
    const double g = none ? 0.0 : D >= 0 ? inv * ic : -inv * ic;
    const double c = none ? 1.0 : c2 * ic;
    const double t = g * ic * b2;
    pc[buf][tid] = c;
    ps[buf][tid] = {g * b.x, g * b.y};
    na = da - t;
    nd = dd + t;
  };
  if (lead) rotation(0);
  long at = jj * log.max_sweeps * (W - 1) * H + tid;  // this lane's entry of the log
  int buf = 0, sweep = 0;
  for (;; ++sweep) {
    // convergence: off-diagonal energy relative to the total; at exit the
    // ratio sqrt(off / total) is reported, so a window that reached the
    // sweep limit unconverged is visible to the caller
    double s = 2.0 * off, t = lead ? da * da + dd * dd : 0.0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      s += __shfl_xor(s, o);
      t += __shfl_xor(t, o);
    }
    if (lane == 0) {
      red[0][tid >> 6] = s;
      red[1][tid >> 6] = t;
    }
    lds_barrier();  // also: the matrix and the parameters of the first step are in place
    double off_all = 0.0, diag_all = 0.0;
#pragma unroll
    for (int i = 0; i < NA / 64; ++i) {
      off_all += red[0][i];
      diag_all += red[1][i];
    }
    const double tot_all = off_all + diag_all;
    if (!(off_all > 1e-30 * tot_all) || sweep >= log.max_sweeps) {
      if (offdiag && tid == 0) offdiag[jj] = tot_all > 0 ? sqrt(off_all / tot_all) : 0.0;
      break;
    }
    for (int step = 0; step < W - 1; ++step) {
      if (act) {
        const double ci = pc[buf][bi], cj = pc[buf][bj];
        const dc si = ps[buf][bi], sj = ps[buf][bj];
        dc v[4] = {A[buf][0][tid], A[buf][1][tid], A[buf][2][tid], A[buf][3][tid]};
        if (lead) {
          log.c[at] = pc[buf][tid];
          log.s[at] = ps[buf][tid];
          at += H;
        }
        // columns: x_T' = c x_T - conj(s) x_B, x_B' = s x_T + c x_B
        auto cols = [&](dc& t, dc& q) {
          const dc a = t, e = q;
          t = {cj * a.x - (sj.x * e.x + sj.y * e.y), cj * a.y - (sj.x * e.y - sj.y * e.x)};
          q = {sj.x * a.x - sj.y * a.y + cj * e.x, sj.x * a.y + sj.y * a.x + cj * e.y};
        };
        // rows: T_y' = c T_y - s B_y, B_y' = conj(s) T_y + c B_y
        auto rows = [&](dc& t, dc& q) {
          const dc a = t, e = q;
          t = {ci * a.x - (si.x * e.x - si.y * e.y), ci * a.y - (si.x * e.y + si.y * e.x)};
          q = {si.x * a.x + si.y * a.y + ci * e.x, si.x * a.y - si.y * a.x + ci * e.y};
        };
        cols(v[0], v[1]);
        cols(v[2], v[3]);
        rows(v[0], v[2]);
        rows(v[1], v[3]);
        if (step == W - 2) {
          off = 0.0;
#pragma unroll
          for (int e = 0; e < 4; ++e) off += v[e].x * v[e].x + v[e].y * v[e].y;
        }
        dc* dst = &A[buf ^ 1][0][0];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e].y = flip(v[e].y, sign[e]);
          dst[to[e]] = v[e];
        }
        b = tid == 0 ? v[0] : tid == H - 1 ? v[3] : v[2];  // leading blocks: the next pair
        if (lead) dst[to_zero] = {0.0, 0.0};
      }
      if (tid < 64) {
        // the diagonal moves with its players: T one lane down, B one up
        const double a0 = na, tl = __shfl_down(na, 1), br = __shfl_up(nd, 1);
        da = tid == 0 ? a0 : tid == H - 1 ? nd : tl;
        dd = tid == 0 ? tl : br;
        if (lead) rotation(buf ^ 1);
      }
      buf ^= 1;
      lds_barrier();
    }
  }
  if (lead) {
    ev[tid] = da;
    ev[W - 1 - tid] = dd;
  }
  if (tid == 0) log.steps[jj] = sweep * (W - 1);
  __syncthreads();
  // descending order, ties keep the lower index: each value's rank, by a key
  // that orders NaN too, so that the ranks are always a permutation
  if (tid < W) {
    auto key = [&](int i) {
      const long long k = __double_as_longlong(ev[i] + 0.0);
      return k < 0 ? k ^ 0x7fffffffffffffffLL : k;
    };
    const long long mine = key(tid);
    int r = 0;
    for (int i = 0; i < W; ++i) {
      const long long k = key(i);
      r += k > mine || (k == mine && i < tid);
    }
    log.rank[jj * W + tid] = r;
    evals[jj * W + r] = ev[tid];
  }
}

// Value of the lane one above (wave_shl) or below (wave_shr) in the wave.
constexpr int WAVE_SHL1 = 0x130, WAVE_SHR1 = 0x138;

// Eigenvectors V = J_1 J_2 ... from the rotation log: a lane holds columns T_k
// and B_k of one row of V, H lanes a row, and the columns move between lanes
// as their players do, by DPP shifts; the ends turn round by bit selects (a
// branch there costs more than the rotation).  Waves are independent: the
// only chain is a row's own rotations, with the next steps' parameters loaded
// ahead.
template <int W>
__global__ __launch_bounds__(128) void k_jacobi_vectors(JacobiLog log, double* __restrict__ evecs,
                                                        float2* __restrict__ vec32) {
  constexpr int H = W / 2, AHEAD = W >= 32 ? 16 : 8;  // steps in flight: the log comes from another XCD
  const long jj = blockIdx.y;
  const int q = blockIdx.x * 128 + threadIdx.x;
  const int row = q / H, k = q % H;  // W * H is a multiple of 128: every lane has a row
  const unsigned m0 = k == 0 ? ~0u : 0u, mh = k == H - 1 ? ~0u : 0u;
  const int steps = log.steps[jj];
  const double* pc = log.c + jj * log.max_sweeps * (W - 1) * H + k;
  const dc* ps = log.s + jj * log.max_sweeps * (W - 1) * H + k;
  dc t = {row == k ? 1.0 : 0.0, 0.0}, b = {row == W - 1 - k ? 1.0 : 0.0, 0.0};
  auto pick = [](unsigned m, unsigned x, unsigned y) { return (m & x) | (~m & y); };
  auto move = [&](double& tv, double& bv) {
    unsigned o[2][2];
    const unsigned ti[2] = {(unsigned)__double2loint(tv), (unsigned)__double2hiint(tv)};
    const unsigned bi[2] = {(unsigned)__double2loint(bv), (unsigned)__double2hiint(bv)};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned tl = __builtin_amdgcn_update_dpp(0, (int)ti[i], WAVE_SHL1, 0xf, 0xf, false);
      const unsigned br = __builtin_amdgcn_update_dpp(0, (int)bi[i], WAVE_SHR1, 0xf, 0xf, false);
      o[0][i] = pick(m0, ti[i], pick(mh, bi[i], tl));
      o[1][i] = pick(m0, tl, br);
    }
    tv = __hiloint2double((int)o[0][1], (int)o[0][0]);
    bv = __hiloint2double((int)o[1][1], (int)o[1][0]);
  };
  double c[AHEAD];
  dc s[AHEAD];
  if (steps > 0) {
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) {  // max_steps >= W - 1 > AHEAD: in bounds, and past `steps` unused
      c[a] = pc[a * H];
      s[a] = ps[a * H];
    }
    for (int n = 0; n < steps; n += AHEAD) {
#pragma unroll
      for (int a = 0; a < AHEAD; ++a) {
        if (n + a >= steps) break;
        const double cc = c[a];
        const dc ss = s[a];
        const long at = (long)min(n + a + AHEAD, steps - 1) * H;
        c[a] = pc[at];
        s[a] = ps[at];
        const dc p = t, v = b;
        t = {cc * p.x - (ss.x * v.x + ss.y * v.y), cc * p.y - (ss.x * v.y - ss.y * v.x)};
        b = {ss.x * p.x - ss.y * p.y + cc * v.x, ss.x * p.y + ss.y * p.x + cc * v.y};
        move(t.x, b.x);
        move(t.y, b.y);
      }
    }
  }
  const int* rank = log.rank + jj * W;
  if (evecs) {
    dc* dst = reinterpret_cast<dc*>(evecs) + (jj * W + row) * W;
    dst[rank[k]] = t;
    dst[rank[W - 1 - k]] = b;
  }
  if (vec32) {
    float2* v = vec32 + jj * W * W + row;
    v[rank[k] * W] = make_float2((float)t.x, (float)t.y);
    v[rank[W - 1 - k] * W] = make_float2((float)b.x, (float)b.y);
  }
}

template <int W>
void go_jacobi(const double* cov, int nwin, double* evals, double* evecs, double* offdiag, const JacobiLog& log,
               float2* vec32, hipStream_t st) {
  hipLaunchKernelGGL(k_jacobi<W>, dim3(nwin), dim3(JacobiShape<W>::NA), 0, st, cov, evals, offdiag, log);
  hipLaunchKernelGGL(k_jacobi_vectors<W>, dim3(W * W / 2 / 128, nwin), dim3(128), 0, st, log, evecs, vec32);
}

}  // namespace

namespace hvi {

static size_t log_entries(int nwin, int window, int max_sweeps) {
  return (size_t)nwin * max_sweeps * (window - 1) * (window / 2);
}

size_t jacobi_log_bytes(int nwin, int window, int max_sweeps) {
  return log_entries(nwin, window, max_sweeps) * 24 + (size_t)nwin * (window + 1) * 4;
}

hv_status launch_jacobi(const double* cov, int nwin, int window, double* evals, double* evecs, double* offdiag,
                        int max_sweeps, void* log_ws, int log_windows, float2* vec32, hipStream_t st) {
  if (nwin <= 0) return HV_OK;
  if (log_windows < 1) return fail(HV_ERR_ARG, "the rotation log holds no window");
  const size_t n = log_entries(log_windows, window, max_sweeps);
  JacobiLog log;
  log.s = (dc*)log_ws;
  log.c = (double*)(log.s + n);
  log.steps = (int*)(log.c + n);
  log.rank = log.steps + log_windows;
  log.max_sweeps = max_sweeps;
  const size_t w = (size_t)window;
  for (int j = 0; j < nwin; j += log_windows) {
    const int g = nwin - j < log_windows ? nwin - j : log_windows;
    const double* c = cov + j * w * w * 2;
    double *ev = evals + j * w, *vec = evecs ? evecs + j * w * w * 2 : nullptr, *off = offdiag ? offdiag + j : nullptr;
    float2* v32 = vec32 ? vec32 + j * w * w : nullptr;
    switch (window) {
      case 16: go_jacobi<16>(c, g, ev, vec, off, log, v32, st); break;
      case 32: go_jacobi<32>(c, g, ev, vec, off, log, v32, st); break;
      case 64: go_jacobi<64>(c, g, ev, vec, off, log, v32, st); break;
      default: return fail(HV_ERR_SHAPE, "PCA window %d not supported", window);
    }
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HV_ERR_DEVICE, "jacobi launch failed: %s", hipGetErrorString(e));
  return HV_OK;
}

}  // namespace hvi
