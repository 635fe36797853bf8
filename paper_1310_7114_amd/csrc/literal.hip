// The paper's own accelerated ITC: Algorithm 1 with the update eq. (6).
// P = X * G_xi comes from the convolution kernels (the A plane of the maps
// with sigma = xi). Every sweep then needs, per lattice codevector w_k,
//   a_k = sum_N P F,  b_k = sum_N P F x,  e_k = sum_N Q F,  d_k = sum_N Q F x
// over its window N (|x - w_k| <= R on the lattice, F the sampled G_omega),
// with Q = W * G_omega the codebook's impulse image convolved with the mask,
// and the lattice entropies V(X;W) = sum P Q = sum_k a_k and
// V(W) = sum Q^2 = sum_k e_k (each Q value is a sum of the masks of the
// codevectors whose window holds the pixel). Q is never formed:
//   e_k = sum_j K_u(j, k) K_v(j, k),  d_k = sum_j (K1_u K_v, K_u K1_v)(j, k),
//   K_u(j, k) = sum_u g(u - w_ju) g(u - w_ku),  K1_u = sum_u u g g
// over the lattice rows both windows cover (the lattice is a rectangle, so
// the 2-D overlap factorises). Away from the border K_u depends only on
// |w_ju - w_ku| (a table) and K1_u = (w_ju + w_ku)/2 K_u by symmetry.
// Then c = V(X;W)/V(W), w_k^new = (b_k - c d_k + c e_k w_k)/a_k, rounded to
// the nearest lattice point (halves upward) and clamped into the lattice.
//
// One sweep is one launch, t = 0 .. iters + 1: a workgroup per codevector first
// completes sweep t - 1, identically in every workgroup (the entropies from the
// terms of all codevectors in a fixed order, c, the rounded update), then forms
// its own codevector's sums at W^t (FP64 accumulation) for the next launch;
// terms and positions are double buffered by the parity of t. One more workgroup
// forms D of sweep t - 1 when a trace is asked for. A state word lets the launches
// after the final codebook return at once, so the host can enqueue every sweep up
// front.
//
// A launch is a chain of latencies: everything the previous one left is loaded
// at once, and 18 window values per lane are in flight (a wave reads four rows of
// a panel, 256 contiguous bytes). 512^2, M = 100, omega = 13.2 (81 x 81
// windows): 5.6 us per sweep launch in a queue (3.4 of them the launch itself; 7.0
// under the profiler), against 13.4 in two launches (9.5 for the sums, 3.9 for the
// update of one workgroup).
#include "itc_device.h"

namespace itc {

namespace {

constexpr int LIT_NT = 512;
constexpr int LIT_WAVES = LIT_NT / 64;
constexpr int LIT_MAXR = 256;  // largest window radius of G_omega the host accepts
constexpr int LIT_MAXM = ITC_MAX_CODEVECTORS_DEV;
constexpr int LIT_PER = LIT_MAXM / LIT_NT;  // codevectors per thread in the update
constexpr int LIT_VX_NT = 256;
constexpr int LIT_PB = 6, LIT_SB = 3;  // 96 columns and 96 rows at once: a window of R <= 40
typedef double term2 __attribute__((ext_vector_type(2), aligned(8)));  // the terms are 8-byte aligned

__device__ __forceinline__ double gtap(const double* g, int t) { return g[t < 0 ? -t : t]; }

// Tables of G_omega, in FP64, one after the other: g [R + 1]; k1 [2 R + 1], the
// overlap of two whole windows at distance d; ed [2 R + 1], exp(-d^2 / 4 omega^2);
// and for overlaps that the border cuts the prefix sums S and Q [4 R + 3] each of
// exp(-x^2 / 4 omega^2) and x exp(..) over every second x from -2 R, at x + 2 R + 2:
// g(u - a) g(u - b) = ed(|a - b|) exp(-x^2 / 4 omega^2) with x = 2 u - a - b, so the
// sum over u = l .. h is ed (S(x_h) - S(x_l - 2)) whatever the border (a loop over the
// window took 2.9 of the 9.9 us of a sweep).
__host__ __device__ constexpr int lit_k1(int R) { return R + 1; }
__host__ __device__ constexpr int lit_ed(int R) { return 3 * R + 2; }
__host__ __device__ constexpr int lit_s(int R) { return 5 * R + 3; }
__host__ __device__ constexpr int lit_q(int R) { return 9 * R + 6; }

// 1-D overlap of the windows of two lattice coordinates a, b on [0, n).
__device__ __forceinline__ void overlap1d(int a, int b, int n, int R, const double* tab, double& K, double& K1) {
  const int d = a > b ? a - b : b - a;
  const int lo = (a > b ? a : b) - R, hi = (a < b ? a : b) + R;
  const double mid = 0.5 * (double)(a + b);
  if (lo >= 0 && hi <= n - 1) {
    K = tab[lit_k1(R) + d];
    K1 = mid * K;
  } else {
    const int l = lo < 0 ? 0 : lo, h = hi > n - 1 ? n - 1 : hi;
    const int xh = 2 * h - (a + b) + 2 * R + 2, xl = 2 * l - (a + b) + 2 * R;  // entries of x_h and x_l - 2
    const double ed = tab[lit_ed(R) + d];
    K = ed * (tab[lit_s(R) + xh] - tab[lit_s(R) + xl]);
    K1 = fma(mid, K, ed * 0.5 * (tab[lit_q(R) + xh] - tab[lit_q(R) + xl]));
  }
}

// Block b < nvx: V(X) = sum P^2 over rows 16 b .. 16 b + 15 in a fixed order (a
// thread takes one pixel of the 16 x 16 tile of every panel; columns past the
// width count 0). Block nvx: the taps, their overlaps and the state.
__global__ void __launch_bounds__(LIT_VX_NT) literal_setup_kernel(LiteralArgs la) {
  __shared__ double red[LIT_VX_NT / 64];
  __shared__ double g[LIT_MAXR + 1];
  __shared__ double sums[2][4 * LIT_MAXR + 3];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x == la.nvx) {
    const int R = la.R;
    const double k2 = -0.5 / (la.omega * la.omega);
    for (int t = tid; t <= R; t += LIT_VX_NT) {
      g[t] = exp(k2 * (double)(t * t));
      la.taps[t] = g[t];
    }
    for (int i = tid; i < 4 * R + 3; i += LIT_VX_NT) {
      const double x = (double)(i - 2 * R - 2), e = i < 2 ? 0.0 : exp(0.5 * k2 * x * x);
      sums[0][i] = e;
      sums[1][i] = e * x;
    }
    __syncthreads();
    for (int d = tid; d <= 2 * R; d += LIT_VX_NT) {
      double s = 0.0;
      for (int q = d - R; q <= R; ++q) s += gtap(g, q) * gtap(g, q - d);
      la.tabs[lit_k1(R) + d - lit_k1(R)] = s;
      la.tabs[lit_ed(R) + d - lit_k1(R)] = exp(0.5 * k2 * (double)(d * d));
    }
    __syncthreads();
    if (tid >= 64 && tid < 68) {  // four sequential sums: S and Q at even and at odd entries
      double* f = sums[(tid >> 1) & 1];
      double s = 0.0;
#pragma unroll 4
      for (int i = 2 + (tid & 1); i < 4 * R + 3; i += 2) {
        s += f[i];
        f[i] = s;
      }
    }
    __syncthreads();
    for (int i = tid; i < 4 * R + 3; i += LIT_VX_NT) {
      la.tabs[lit_s(R) + i - lit_k1(R)] = sums[0][i];
      la.tabs[lit_q(R) + i - lit_k1(R)] = sums[1][i];
    }
    if (tid == 0) {
      la.state[0] = -1;  // sweep count of the final codebook: not known yet
      la.state[1] = 0;   // launch that ended the fit: none
    }
    return;
  }
  const int u = (int)blockIdx.x * 16 + (tid >> 4), c = tid & 15;
  const int np = n_panels(la.W);
  const float* P = la.P + (int64_t)min(u, la.H - 1) * MAP_PANEL + c;
  const int64_t step = (int64_t)la.H * MAP_PANEL;
  double s = 0.0;
  constexpr int B = 8;
  for (int p0 = 0; p0 < np; p0 += B) {
    float v[B];
#pragma unroll
    for (int i = 0; i < B; ++i) v[i] = P[(int64_t)min(p0 + i, np - 1) * step];
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const double x = u < la.H && (p0 + i) * MAP_PANEL + c < la.W ? (double)v[i] : 0.0;
      s = fma(x, x, s);
    }
  }
  s = block_reduce_fixed(s, red);
  if (tid == 0) la.vx_part[blockIdx.x] = s;
}

// The workgroup totals of two FP64 values per thread, in a fixed order.
__device__ __forceinline__ void block_sum2(double& x, double& y, double2* red) {
  wave_sum2(x, y);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = make_double2(x, y);
  __syncthreads();
  x = y = 0.0;
#pragma unroll
  for (int w = 0; w < LIT_WAVES; ++w) {
    x += red[w].x;
    y += red[w].y;
  }
}

__global__ void __launch_bounds__(LIT_NT) literal_sweep_kernel(LiteralArgs la, const int32_t* __restrict__ w_init,
                                                               int32_t* __restrict__ w_out, int t) {
  __shared__ double2 red[3 * LIT_WAVES];
  __shared__ float redf[LIT_WAVES];
  __shared__ double tab[lit_q(LIT_MAXR) + 4 * LIT_MAXR + 3];
  __shared__ int2 wpos[LIT_MAXM];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = la.M, R = la.R, k = blockIdx.x;
  for (int i = tid; i < lit_q(R) + 4 * R + 3; i += LIT_NT) tab[i] = i <= R ? la.taps[i] : la.tabs[i - lit_k1(R)];
  int2 w[LIT_PER];
  if (t == 0) {
    if (k == M) return;  // no sweep before this one
#pragma unroll
    for (int i = 0; i < LIT_PER; ++i) {
      const int j = i * LIT_NT + tid;
      w[i] = make_int2(0, 0);
      if (j < M) w[i] = make_int2(min(max(w_init[2 * j], 0), la.H - 1), min(max(w_init[2 * j + 1], 0), la.W - 1));
    }
  } else {
    // ---- complete sweep t - 1 ----
    const int final_t = la.state[0], ended = la.state[1];
    const int2* pprev = la.pos + (size_t)((t - 1) & 1) * M;
    const term2* tp = reinterpret_cast<const term2*>(la.terms[(t - 1) & 1]);
    term2 q0[LIT_PER], q1[LIT_PER], q2[LIT_PER];  // (a, b_u), (b_v, e), (d_u, d_v)
#pragma unroll
    for (int i = 0; i < LIT_PER; ++i) {
      const int j = min(i * LIT_NT + tid, M - 1);
      w[i] = pprev[j];
      q0[i] = tp[3 * j];
      q1[i] = tp[3 * j + 1];
      q2[i] = tp[3 * j + 2];
    }
    double vx = 0.0, none = 0.0;
    if (k == M)
      for (int i = tid; i < la.nvx; i += LIT_NT) vx += la.vx_part[i];
    if (ended != 0 && ended < t) return;  // an earlier launch ended the fit (this one may be setting it: t)
    double v_xw = 0.0, v_w = 0.0;
#pragma unroll
    for (int i = 0; i < LIT_PER; ++i) {
      if (i * LIT_NT + tid < M) {
        v_xw += q0[i].x;
        v_w += q1[i].y;
      }
    }
    block_sum2(v_xw, v_w, red);
    if (k == M) {  // the trace's workgroup
      block_sum2(vx, none, red + LIT_WAVES);
      if (tid == 0) la.d_trace[t - 1] = log(v_w) + log(vx) - 2.0 * log(v_xw);
      return;
    }
    if (t == la.iters + 1 || t == final_t + 1) {  // W^{t-1} is the final codebook
      if (k == 0) {
#pragma unroll
        for (int i = 0; i < LIT_PER; ++i) {
          const int j = i * LIT_NT + tid;
          if (j < M) {
            w_out[2 * j] = w[i].x;
            w_out[2 * j + 1] = w[i].y;
          }
        }
        if (tid == 0) {
          if (la.iters_done) *la.iters_done = t - 1;
          la.state[1] = t;
        }
      }
      return;
    }
    const double c = v_xw / v_w;
    float step = 0.0f;
#pragma unroll
    for (int i = 0; i < LIT_PER; ++i) {
      const double a = q0[i].x;
      if (i * LIT_NT + tid < M && a > 0.0) {
        const int ou = w[i].x, ov = w[i].y;
        const double nu = (q0[i].y - c * q2[i].x + c * q1[i].y * (double)ou) / a;
        const double nv = (q1[i].x - c * q2[i].y + c * q1[i].y * (double)ov) / a;
        double ru = floor(nu + 0.5), rv = floor(nv + 0.5);
        ru = ru < 0.0 ? 0.0 : (ru > (double)(la.H - 1) ? (double)(la.H - 1) : ru);
        rv = rv < 0.0 ? 0.0 : (rv > (double)(la.W - 1) ? (double)(la.W - 1) : rv);
        const int iu = (int)ru, iv = (int)rv;
        step = fmaxf(step, sqrtf((float)((iu - ou) * (iu - ou) + (iv - ov) * (iv - ov))));
        w[i] = make_int2(iu, iv);
      }
    }
    if (la.theta >= 0.0 && k == 0) {  // uniform
      step = wave_max_nonneg(step);
      if (lane == 0) redf[wave] = step;
      __syncthreads();
      if (tid == 0) {
        float smax = 0.0f;
        for (int q = 0; q < LIT_WAVES; ++q) smax = fmaxf(smax, redf[q]);
        // this launch may set it (to t), which matters only from launch t + 1 on
        if ((double)smax <= la.theta) la.state[0] = t;  // W^t is final
      }
    }
  }
#pragma unroll
  for (int i = 0; i < LIT_PER; ++i) {
    const int j = i * LIT_NT + tid;
    if (j < M) {
      wpos[j] = w[i];
      if (j == k) la.pos[(size_t)(t & 1) * M + j] = w[i];
    }
  }
  __syncthreads();

  // ---- the four window sums of codevector k at W^t ----
  const double* g = tab;
  const int wu = wpos[k].x, wv = wpos[k].y;
  const int u0 = max(wu - R, 0), u1 = min(wu + R, la.H - 1);
  const int v0 = max(wv - R, 0), v1 = min(wv + R, la.W - 1);
  // data: a, b over the window, in tiles of four rows of one panel (256 contiguous bytes, a value per lane);
  // the waves take every eighth tile row, LIT_PB panels and LIT_SB tile rows at a time with all their loads in
  // flight. Per tile row P is summed over the panels with g(v) and v g(v), then weighed by the row. Values
  // outside the window are loaded clamped and count 0 (map columns past the width hold anything).
  const int pa = v0 / MAP_PANEL, pz = v1 / MAP_PANEL;
  const int lr = lane >> 4, lc = lane & 15;
  double a = 0.0, bu = 0.0, bv = 0.0;
  for (int p0 = pa; p0 <= pz; p0 += LIT_PB) {
    double gv[LIT_PB], gvv[LIT_PB];
    bool okv[LIT_PB];
#pragma unroll
    for (int i = 0; i < LIT_PB; ++i) {
      const int v = (p0 + i) * MAP_PANEL + lc;
      okv[i] = v >= v0 && v <= v1;
      gv[i] = okv[i] ? gtap(g, v - wv) : 0.0;
      gvv[i] = gv[i] * (double)v;
    }
    for (int s0 = u0 + 4 * wave; s0 <= u1; s0 += 4 * LIT_WAVES * LIT_SB) {  // uniform
      float pv[LIT_SB][LIT_PB];
#pragma unroll
      for (int j = 0; j < LIT_SB; ++j) {
        const int u = min(s0 + 4 * LIT_WAVES * j + lr, u1);
#pragma unroll
        for (int i = 0; i < LIT_PB; ++i)
          pv[j][i] = la.P[((int64_t)min(p0 + i, pz) * la.H + u) * MAP_PANEL + lc];
      }
#pragma unroll
      for (int j = 0; j < LIT_SB; ++j) {
        const int u = s0 + 4 * LIT_WAVES * j + lr;
        const double gu = u <= u1 ? gtap(g, u <= u1 ? u - wu : 0) : 0.0;
        double r = 0.0, rv = 0.0;
#pragma unroll
        for (int i = 0; i < LIT_PB; ++i) {
          const double x = okv[i] ? (double)pv[j][i] : 0.0;
          r = fma(x, gv[i], r);
          rv = fma(x, gvv[i], rv);
        }
        r *= gu;
        a += r;
        bu = fma((double)u, r, bu);
        bv = fma(gu, rv, bv);
      }
    }
  }
  // codebook: e, d over the other codevectors' overlapping windows (threads along j)
  double e = 0.0, du = 0.0, dv = 0.0;
  for (int j = tid; j < M; j += LIT_NT) {
    const int2 wj = wpos[j];
    if (abs(wj.x - wu) > 2 * R || abs(wj.y - wv) > 2 * R) continue;
    double Ku, K1u, Kv, K1v;
    overlap1d(wj.x, wu, la.H, R, tab, Ku, K1u);
    overlap1d(wj.y, wv, la.W, R, tab, Kv, K1v);
    e = fma(Ku, Kv, e);
    du = fma(K1u, Kv, du);
    dv = fma(Ku, K1v, dv);
  }
  wave_sum2(a, bu);
  wave_sum2(bv, e);
  wave_sum2(du, dv);
  if (lane == 0) {  // red was last read before the barrier above
    red[3 * wave] = make_double2(a, bu);
    red[3 * wave + 1] = make_double2(bv, e);
    red[3 * wave + 2] = make_double2(du, dv);
  }
  __syncthreads();
  if (tid < 3) {
    double2 s = make_double2(0.0, 0.0);
#pragma unroll
    for (int ww = 0; ww < LIT_WAVES; ++ww) {
      s.x += red[3 * ww + tid].x;
      s.y += red[3 * ww + tid].y;
    }
    reinterpret_cast<term2*>(la.terms[t & 1])[3 * k + tid] = term2{s.x, s.y};
  }
}

}  // namespace

hipError_t launch_literal(const LiteralArgs& la, const int32_t* w_init, int32_t* w_out, hipStream_t s) {
  if (la.R < 1 || la.R > LIT_MAXR) return hipErrorInvalidValue;
  if (la.M < 1 || la.M > LIT_MAXM) return hipErrorInvalidValue;
  hipLaunchKernelGGL(literal_setup_kernel, dim3(la.nvx + 1), dim3(LIT_VX_NT), 0, s, la);
  const dim3 grid(la.M + (la.d_trace ? 1 : 0));
  for (int t = 0; t <= la.iters + 1; ++t) {
    hipLaunchKernelGGL(literal_sweep_kernel, grid, dim3(LIT_NT), 0, s, la, w_init, w_out, t);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace itc

// ---------------------------------------------------------------------------
// Algorithm 1 without a caller work buffer: the work memory is a file-scope
// device array, one per GPU, held until the process ends. Its address on the
// current device is taken with hipGetSymbolAddress at the first call on that
// device (the array's name in host code is not a device address).
// ---------------------------------------------------------------------------
#include <mutex>

namespace itc {
namespace {

constexpr size_t LITERAL_SCRATCH_BYTES = (size_t)ITC_LITERAL_SCRATCH_MIB << 20;
static __device__ __align__(256) unsigned char scratch[LITERAL_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES] = {};

}  // namespace
}  // namespace itc

extern "C" itc_status itc_lattice_literal_fit_noalloc(const itc_lattice_desc* d, const void* weights, double omega,
                                                      int32_t radius_omega, int32_t M, const int32_t* w_init,
                                                      int32_t iters, double theta, int32_t* w_out, double* d_trace,
                                                      int32_t* iters_done, void* stream) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= itc::MAX_DEVICES)
    return itc::report_error(ITC_E_DEVICE, "no current HIP device");
  void* work = nullptr;
  {
    std::lock_guard<std::mutex> lock(itc::g_scratch_mu);
    if (!itc::g_scratch_ptr[dev]) {
      void* p = nullptr;
      const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(itc::scratch));
      if (e != hipSuccess || !p) return itc::report_error(ITC_E_DEVICE, "hipGetSymbolAddress of the scratch array failed");
      itc::g_scratch_ptr[dev] = p;
    }
    work = itc::g_scratch_ptr[dev];
  }
  return itc::literal_fit_with_work(d, weights, omega, radius_omega, M, w_init, iters, theta, w_out, d_trace,
                                    iters_done, work, itc::LITERAL_SCRATCH_BYTES, stream);
}
