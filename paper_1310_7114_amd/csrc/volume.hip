// Lattice ITC on 3-D lattices (volumes): the maps of Section 3.1 with a
// third separable pass and the update eq. (4) in three dimensions (the paper
// develops the method on 2-D lattices and notes it carries over to higher
// dimensions). Coordinates x = (s, u, v): slice, row, column.
//
// Maps: A = h * g(s) g(u) g(v) and the moments M_a = sum_y h(y) (x_a - y_a)
// g(x - y) for a = s, u, v, each a chain of 1-D correlations:
//   v pass:  P0 = h *_v g,   P1 = h *_v tg
//   u pass:  Q00 = P0 *_u g, Q01 = P0 *_u tg, Q10 = P1 *_u g
//   s pass:  A = Q00 *_s g,  M_s = Q00 *_s tg, M_u = Q01 *_s g, M_v = Q10 *_s g
// (tg[t] = t g[t], t = x_a - y_a). Two kernels:
//   * in-plane: a workgroup stages a 64-column x 32-row tile of one slice
//     with its R halo in LDS, runs the v pass in place (each row becomes its
//     P0 | P1) and the u pass out to the three FP32 Q volumes in the caller's
//     work buffer;
//   * depth: each thread walks 8 consecutive outputs along s for one (u, v),
//     reading every Q value of its window once, writes A, M_s, M_u, M_v and
//     adds h A into a per-workgroup FP64 partial of S_X.
// The column passes are register-blocked: input k of the window feeds the 8
// outputs through a zero-padded tap table, so every input is loaded once and
// no tap index leaves the table. Taps are kernel arguments (scalar loads).
// S_X is summed in two fixed-order levels (workgroups, then their partials).
//
// Fit: one workgroup, from one wave for up to 16 codevectors to 1,024 threads;
// P lanes share a codevector (FP64 positions); per sweep trilinear reads of the
// four maps at w_k (eight corners, off-lattice corners 0; the corner values are
// kept while w_k stays in its cell), the M x M Gaussian terms over an FP32 copy of the codebook in
// LDS (scaled by sqrt(log2 e / 2 sigma^2) and centred on the volume, so each
// pair is one exp2), FP64 reductions of S_XW and S_W in a fixed order, and the
// Jacobi update.
#include <climits>
#include <cmath>
#include <type_traits>

#include "itc_device.h"

namespace itc {

namespace {

constexpr int VOL_NT = 256;
constexpr int VOL_TR = 32;   // rows of an in-plane tile (4 waves x VOL_RUN)
constexpr int VOL_RUN = 8;   // outputs per thread of a column pass
constexpr int VOL_STEP = 4;  // window inputs of a depth-pass step
constexpr int VOL_UR = 4;    // rows of a depth-pass workgroup (one per wave)
constexpr int VOL_MAXR = 32;
constexpr int VOL_TAPS = 2 * VOL_MAXR + 1 + 2 * (VOL_RUN - 1);

// Taps with VOL_RUN - 1 zeros on each side: f[t + R + VOL_RUN - 1] = f(t) for
// |t| <= R, zero elsewhere in the table.
struct VolTaps {
  float g[VOL_TAPS];
  float tg[VOL_TAPS];
};

template <typename WT>
__device__ __forceinline__ double weight_at(const WT* x, const VolumeGeom& vg, int s, int u, int v) {
  return vg.scale * (double)x[(int64_t)s * vg.slice_pitch + (int64_t)u * vg.row_pitch + v];
}

// In-plane passes of one tile: Q00, Q01, Q10 for rows [u0, u0 + 32) and
// columns [v0, v0 + 64) of slice s (blockIdx = (column tile, row tile, s)).
// SROWS >= (32 + 2R) / 4 rows of the staged tile per wave (12, 16 or 24).
// 96 x 192 x 256 voxels, R = 6: 25 us (staging 8, v pass 6, u pass 6, stores 4); with an
// LDS read for every tap and row the v pass took 9 (R = 24: all maps 168 us, now 138).
template <typename WT, int SROWS>
__global__ void __launch_bounds__(VOL_NT) vol_plane_kernel(const WT* __restrict__ x, VolumeGeom vg, VolTaps tp,
                                                           float* __restrict__ q00, float* __restrict__ q01,
                                                           float* __restrict__ q10) {
  // [4 SROWS][RP]: weights of rows u0 - R.., columns v0 - R.. (64 + 2 R <= RP of them), then P0 | P1
  extern __shared__ __align__(16) float X[];
  constexpr int RP = 128, NS = SROWS / 4;
  static_assert(64 + 2 * VOL_MAXR <= RP && SROWS % 4 == 0, "a staged row; four rows a step of the v pass");
  const int R = vg.R, XW = 64 + 2 * R;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int v0 = blockIdx.x * 64, u0 = blockIdx.y * VOL_TR, s = blockIdx.z;
  // staging: wave wv takes rows 16 m + 4 wv .. + 3 (SROWS of them, at most 2
  // columns per lane) and issues all their loads before the first is used;
  // positions off the lattice load a clamped position and store 0
  const WT* xs = x + (int64_t)s * vg.slice_pitch;
  auto staged_row = [&](int q) { return 16 * (q >> 2) + 4 * wv + (q & 3); };
  WT raw[SROWS][2];
#pragma unroll
  for (int q = 0; q < SROWS; ++q) {
    const int u = min(max(u0 - R + staged_row(q), 0), vg.H - 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int v = min(max(v0 - R + lane + 64 * h, 0), vg.W - 1);
      raw[q][h] = xs[(int64_t)u * vg.row_pitch + v];
    }
  }
#pragma unroll
  for (int q = 0; q < SROWS; ++q) {
    const int j = staged_row(q), u = u0 - R + j;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = lane + 64 * h, v = v0 - R + c;
      const bool on = u >= 0 && u < vg.H && v >= 0 && v < vg.W;
      if (c < XW) X[j * RP + c] = on ? (float)(vg.scale * (double)raw[q][h]) : 0.f;
    }
  }
  wave_lds_order();
  // v pass, taps outermost (each tap is fetched once per wave): lane (r, c) makes columns 4c .. 4c + 3 of the
  // wave's rows 16 m + 4 wv + r from a window of registers that takes four more columns, one LDS read, every
  // four taps. No other wave touches the rows, so P0 | P1 overwrite them in place.
  {
    typedef float f4 __attribute__((ext_vector_type(4)));
    float* xr = X + (4 * wv + (lane >> 4)) * RP + 4 * (lane & 15);
    f4 w[NS], a0[NS], a1[NS];
#pragma unroll
    for (int m = 0; m < NS; ++m) {
      w[m] = *reinterpret_cast<const f4*>(xr + 16 * m * RP);
      a0[m] = a1[m] = f4{0.f, 0.f, 0.f, 0.f};
    }
    // taps R - u - e for e < n: output i takes window column i + e
    auto taps = [&](int u, auto N) __attribute__((always_inline)) {
      constexpr int n = decltype(N)::value;
      float g[n], tg[n];
#pragma unroll
      for (int e = 0; e < n; ++e) {
        g[e] = tp.g[2 * R - u - e + VOL_RUN - 1];
        tg[e] = tp.tg[2 * R - u - e + VOL_RUN - 1];
      }
#pragma unroll
      for (int m = 0; m < NS; ++m) {
        f4 nx = w[m];
        if constexpr (n > 1) nx = *reinterpret_cast<const f4*>(xr + 16 * m * RP + u + 4);
#pragma unroll
        for (int e = 0; e < n; ++e)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float h = i + e < 4 ? w[m][(i + e) & 3] : nx[(i + e) & 3];
            a0[m][i] = fmaf(g[e], h, a0[m][i]);
            a1[m][i] = fmaf(tg[e], h, a1[m][i]);
          }
        w[m] = nx;
      }
    };
    int u = 0;
    for (; u + 3 <= 2 * R; u += 4) taps(u, std::integral_constant<int, 4>{});
    if (u == 2 * R)  // uniform: 2 R + 1 taps leave one or three
      taps(u, std::integral_constant<int, 1>{});
    else
      taps(u, std::integral_constant<int, 3>{});
    wave_lds_order();
#pragma unroll
    for (int m = 0; m < NS; ++m) {
      *reinterpret_cast<f4*>(xr + 16 * m * RP) = a0[m];
      *reinterpret_cast<f4*>(xr + 16 * m * RP + 64) = a1[m];
    }
  }
  __syncthreads();
  // u pass: wave wv makes tile rows r0 .. r0 + 7; input k of the window is
  // P row r0 + k (image row u0 - R + r0 + k) and reaches output o with
  // t = o + R - k, |t| <= R. For R >= 3 the window splits into a ramp-up
  // (k < 7: outputs 0..k), a middle (all outputs) and a ramp-down (k = 2R + d:
  // outputs d..7), so no zero tap is multiplied.
  const int r0 = wv * VOL_RUN;
  float c00[VOL_RUN], c01[VOL_RUN], c10[VOL_RUN];
#pragma unroll
  for (int o = 0; o < VOL_RUN; ++o) c00[o] = c01[o] = c10[o] = 0.f;
  auto feed = [&](int k, int olo, int ohi) __attribute__((always_inline)) {
    const float p0 = X[(r0 + k) * RP + lane], p1 = X[(r0 + k) * RP + 64 + lane];
    const int b = 2 * R - k + VOL_RUN - 1;
#pragma unroll
    for (int o = olo; o <= ohi; ++o) {
      const float g = tp.g[b + o], tg = tp.tg[b + o];
      c00[o] = fmaf(g, p0, c00[o]);
      c01[o] = fmaf(tg, p0, c01[o]);
      c10[o] = fmaf(g, p1, c10[o]);
    }
  };
  if (R >= 3) {
#pragma unroll
    for (int k = 0; k < VOL_RUN - 1; ++k) feed(k, 0, k);
#pragma unroll 2
    for (int k = VOL_RUN - 1; k <= 2 * R; ++k) feed(k, 0, VOL_RUN - 1);
#pragma unroll
    for (int d = 1; d < VOL_RUN; ++d) feed(2 * R + d, d, VOL_RUN - 1);
  } else {
    for (int k = 0; k < 2 * R + VOL_RUN; ++k) feed(k, 0, VOL_RUN - 1);
  }
  const int v = v0 + lane;
  if (v >= vg.W) return;
#pragma unroll
  for (int o = 0; o < VOL_RUN; ++o) {
    const int u = u0 + r0 + o;
    if (u < vg.H) {
      const int64_t i = ((int64_t)s * vg.H + u) * vg.W + v;
      q00[i] = c00[o];
      q01[i] = c01[o];
      q10[i] = c10[o];
    }
  }
}

// Depth pass and S_X partials: blockIdx = (column tile, 4-row group, 8-slice
// group); thread (wave wv, lane) owns (u, v) and slices s0 .. s0 + 7. Bound by
// the caches: 1 + R / 4 reads of the three Q volumes, from L2 and the memory-side
// cache, and one write of the maps.
// 96 x 192 x 256 voxels, R = 6: 25 us (217 MB); 31 us with a step's loads
// behind a branch each and nothing in flight during the arithmetic.
template <typename WT>
__global__ void __launch_bounds__(VOL_NT) vol_depth_kernel(const WT* __restrict__ x, VolumeGeom vg, VolTaps tp,
                                                           const float* __restrict__ q00,
                                                           const float* __restrict__ q01,
                                                           const float* __restrict__ q10, float* __restrict__ maps,
                                                           double* __restrict__ blk) {
  __shared__ double red[VOL_NT / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int v = blockIdx.x * 64 + lane, u = blockIdx.y * VOL_UR + wv, s0 = blockIdx.z * VOL_RUN;
  const bool in = u < vg.H && v < vg.W;
  const int R = vg.R;
  const int64_t plane = (int64_t)vg.H * vg.W, n = plane * vg.D, col = (int64_t)u * vg.W + v;
  float a[VOL_RUN], ms[VOL_RUN], mu[VOL_RUN], mv[VOL_RUN];
#pragma unroll
  for (int o = 0; o < VOL_RUN; ++o) a[o] = ms[o] = mu[o] = mv[o] = 0.f;
  // Input k is slice s0 - R + k; only slices inside the lattice contribute. VOL_STEP inputs a step; the loads
  // of the next step are in flight behind a step's arithmetic (past the window and outside the lattice they
  // read 0 at an offset past the volume).
  const int k0 = R - s0 > 0 ? R - s0 : 0;
  const int k1 = min(2 * R + VOL_RUN, vg.D - s0 + R);
  const uint32_t pb = (uint32_t)(plane * 4), nb = (uint32_t)(n * 4);
  const rsrc_t r00 = make_rsrc(q00, nb), r01 = make_rsrc(q01, nb), r10 = make_rsrc(q10, nb);
  const uint32_t cb = in ? (uint32_t)col * 4u : BUF_OOB;
  float f[2][VOL_STEP][3];
  auto fetch = [&](float (&x3)[VOL_STEP][3], int k) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < VOL_STEP; ++q) {
      const uint32_t off = k + q < k1 ? cb + (uint32_t)(s0 - R + k + q) * pb : BUF_OOB;
      x3[q][0] = buf_load<float>(r00, off, 0);
      x3[q][1] = buf_load<float>(r01, off, 0);
      x3[q][2] = buf_load<float>(r10, off, 0);
    }
  };
  auto feed = [&](const float (&x3)[VOL_STEP][3], int k) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < VOL_STEP; ++q) {
      if (k + q >= k1) break;  // uniform
      const int b = 2 * R - (k + q) + VOL_RUN - 1;
#pragma unroll
      for (int o = 0; o < VOL_RUN; ++o) {
        const float g = tp.g[b + o], tg = tp.tg[b + o];
        a[o] = fmaf(g, x3[q][0], a[o]);
        ms[o] = fmaf(tg, x3[q][0], ms[o]);
        mu[o] = fmaf(g, x3[q][1], mu[o]);
        mv[o] = fmaf(g, x3[q][2], mv[o]);
      }
    }
  };
  fetch(f[0], k0);
  for (int k = k0; k < k1; k += 2 * VOL_STEP) {
    fetch(f[1], k + VOL_STEP);
    feed(f[0], k);
    fetch(f[0], k + 2 * VOL_STEP);
    feed(f[1], k + VOL_STEP);
  }
  double sx = 0.0;
#pragma unroll
  for (int o = 0; o < VOL_RUN; ++o) {
    const int s = s0 + o;
    if (in && s < vg.D) {
      const int64_t i = (int64_t)s * plane + col;
      maps[i] = a[o];
      maps[n + i] = ms[o];
      maps[2 * n + i] = mu[o];
      maps[3 * n + i] = mv[o];
      sx = fma(weight_at(x, vg, s, u, v), (double)a[o], sx);
    }
  }
  sx = block_reduce_fixed(sx, red);
  if (threadIdx.x == 0) blk[((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = sx;
}

__global__ void __launch_bounds__(VOL_NT) vol_sx_total_kernel(const double* __restrict__ blk, int nb, double* s_x) {
  __shared__ double red[VOL_NT / 64];
  const double s = block_sum_fixed(blk, (int64_t)nb, red);
  if (threadIdx.x == 0) *s_x = s;
}

// The workgroup totals of two FP64 values per thread (each wave by a fixed
// DPP tree, then the waves in order); every thread gets both. Aligned groups of
// SAME lanes hold one value, which counts once.
template <int SAME, int NW>
__device__ __forceinline__ void block_reduce2(double& x, double& y, double2 (*red)) {
  wave_sum2<SAME>(x, y);
  if constexpr (NW == 1) return;
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = make_double2(x, y);
  __syncthreads();
  x = y = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    x += red[w].x;
    y += red[w].y;
  }
}

// The eight corners of a lattice cell for the four maps, kept in registers
// while a codevector stays in the cell.
struct Cell {
  int s0, u0, v0;
  float a[8], ms[8], mu[8], mv[8];
};

__device__ __forceinline__ void cell_load(Cell& c, rsrc_t rs, uint32_t plane_bytes, const VolumeGeom& vg, int s0,
                                          int u0, int v0) {
  c.s0 = s0;
  c.u0 = u0;
  c.v0 = v0;
  // off-lattice corners take an offset with bit 31 set, past the buffer: the load returns 0 (arithmetic, not a
  // select, which the compiler turns into a branch for each corner)
  auto off_axis = [](int x, int n) { return (uint32_t)!((unsigned)x < (unsigned)n) << 31; };
  const uint32_t bs[2] = {off_axis(s0, vg.D), off_axis(s0 + 1, vg.D)}, bu[2] = {off_axis(u0, vg.H), off_axis(u0 + 1, vg.H)},
                 bv[2] = {off_axis(v0, vg.W), off_axis(v0 + 1, vg.W)};
  const uint32_t base = (((uint32_t)s0 * (uint32_t)vg.H + (uint32_t)u0) * (uint32_t)vg.W + (uint32_t)v0) * 4u;
  const uint32_t row = (uint32_t)vg.W * 4u, slice = (uint32_t)vg.H * row;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int ds = q >> 2, du = (q >> 1) & 1, dv = q & 1;
    uint32_t off = base + (ds ? slice : 0u) + (du ? row : 0u) + (dv ? 4u : 0u);
    // an offset on the lattice stays below 2^31: the bit of one off it cannot carry away
    off = (off & 0x7fffffffu) | bs[ds] | bu[du] | bv[dv];
    c.a[q] = buf_load<float>(rs, off, 0);
    c.ms[q] = buf_load<float>(rs, off, plane_bytes);
    c.mu[q] = buf_load<float>(rs, off, 2 * plane_bytes);
    c.mv[q] = buf_load<float>(rs, off, 3 * plane_bytes);
  }
}

// Trilinear read at fractional offsets fr: A and g = sum_c b_c ((c - w) A(c) - M(c)).
__device__ __forceinline__ void cell_read(const Cell& c, const float fr[3], float& A, float g[3]) {
  A = 0.f;
  g[0] = g[1] = g[2] = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int ds = q >> 2, du = (q >> 1) & 1, dv = q & 1;
    const float bs = ds ? fr[0] : 1.f - fr[0], bu = du ? fr[1] : 1.f - fr[1], bv = dv ? fr[2] : 1.f - fr[2];
    const float b = bs * bu * bv;
    A = fmaf(b, c.a[q], A);
    g[0] = fmaf(b, fmaf((float)ds - fr[0], c.a[q], -c.ms[q]), g[0]);
    g[1] = fmaf(b, fmaf((float)du - fr[1], c.a[q], -c.mu[q]), g[1]);
    g[2] = fmaf(b, fmaf((float)dv - fr[2], c.a[q], -c.mv[q]), g[2]);
  }
}

// Codebook entries in LDS for M codevectors and P lanes: padded with points at
// 1e30, whose Gaussian is exactly 0, to whole blocks of four per lane.
__host__ __device__ inline int vol_padded(int M, int P) { return (M + 4 * P - 1) / (4 * P) * (4 * P); }

// P lanes per codevector, NT threads, M P <= NT. A sweep is a chain of latencies: the lane's pair terms go four at a
// time, 1 / A_k is formed before the sums are known, and two barriers a sweep (none
// for one wave) separate the reads of the codebook and the sums from the next
// writes. us per sweep: M = 16 0.98 (1.21 with three barriers, one pair term at a
// time and 256 threads at most), M = 64 1.73 (2.24), M = 100 2.56 (4.33), M = 256
// 7.0 (12.2), M = 1000 70 (149).
template <int P, int NT>
__global__ void __launch_bounds__(NT) vol_fit_kernel(const float* __restrict__ maps, VolumeGeom vg,
                                                     const double* __restrict__ s_x_in, int M,
                                                     const float* __restrict__ w_init, int iters, double theta,
                                                     float* w_out, double* d_trace, int32_t* iters_done) {
  constexpr int NW = NT / 64;
  extern __shared__ float4 cb[];  // [vol_padded(M, P)] scaled centred codebook
  __shared__ double2 red[NW];
  __shared__ float redf[NW];
  const int tid = threadIdx.x, part = tid % P, k = tid / P;
  const bool own = k < M;
  const int64_t n = (int64_t)vg.D * vg.H * vg.W;
  const uint32_t plane_bytes = (uint32_t)(n * 4);
  const rsrc_t rs = make_rsrc(maps, 4 * plane_bytes);
  const double s_x = *s_x_in;
  const double sc = sqrt(1.4426950408889634 / (2.0 * vg.sigma * vg.sigma)), isc = 1.0 / sc;
  const double cs0 = 0.5 * vg.D, cu0 = 0.5 * vg.H, cv0 = 0.5 * vg.W;
  const int Mp = vol_padded(M, P);
  double ws = 0.0, wu = 0.0, wv = 0.0;
  Cell cell;
  cell.s0 = INT_MIN;
  auto scaled = [&]() {
    return make_float4((float)(sc * (ws - cs0)), (float)(sc * (wu - cu0)), (float)(sc * (wv - cv0)), 0.f);
  };
  for (int j = M + tid; j < Mp; j += NT) cb[j] = make_float4(1e30f, 1e30f, 1e30f, 0.f);
  if (own) {
    ws = w_init[3 * k];
    wu = w_init[3 * k + 1];
    wv = w_init[3 * k + 2];
    if (part == 0) cb[k] = scaled();
  }
  __syncthreads();
  bool stop = false;
  int t = 0;
  for (;; ++t) {
    const bool last = t == iters || stop;
    float A = 0.f, g[3] = {}, E[3] = {};
    double inv = 0.0, sxw = 0.0, sw = 0.0;
    if (own) {
      const double fs = floor(ws), fu = floor(wu), fv = floor(wv);
      const int s0 = (int)fs, u0 = (int)fu, v0 = (int)fv;
      if (s0 != cell.s0 || u0 != cell.u0 || v0 != cell.v0) cell_load(cell, rs, plane_bytes, vg, s0, u0, v0);
      const float4 hk = cb[k];
      float C[2] = {}, E0[2] = {}, E1[2] = {}, E2[2] = {};
      for (int j = part; j < Mp; j += 4 * P) {
        float4 h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) h[i] = cb[j + i * P];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float d0 = h[i].x - hk.x, d1 = h[i].y - hk.y, d2 = h[i].z - hk.z;
          const float e = __builtin_amdgcn_exp2f(-fmaf(d0, d0, fmaf(d1, d1, d2 * d2)));
          C[i & 1] += e;
          E0[i & 1] = fmaf(e, d0, E0[i & 1]);
          E1[i & 1] = fmaf(e, d1, E1[i & 1]);
          E2[i & 1] = fmaf(e, d2, E2[i & 1]);
        }
      }
      const float Ck = group_sum<P>(C[0] + C[1]);
      E[0] = group_sum<P>(E0[0] + E0[1]);
      E[1] = group_sum<P>(E1[0] + E1[1]);
      E[2] = group_sum<P>(E2[0] + E2[1]);
      const float fr[3] = {(float)(ws - fs), (float)(wu - fu), (float)(wv - fv)};
      cell_read(cell, fr, A, g);
      sxw = (double)A;
      sw = (double)Ck;
      inv = 1.0 / (double)A;
    }
    block_reduce2<P, NW>(sxw, sw, red);
    const double S_XW = sxw, S_W = sw;
    // D = log(S_W S_X / S_XW^2): the argument now, the logarithms after the
    // last sweep by all threads at once
    if (tid == 0 && d_trace) d_trace[t] = S_W * s_x / (S_XW * S_XW);
    if (last) break;
    const double c = S_XW / S_W * isc;  // E = E' / sc
    float step = 0.f;
    if (own && A != 0.f) {
      const double d0 = ((double)g[0] - c * (double)E[0]) * inv;
      const double d1 = ((double)g[1] - c * (double)E[1]) * inv;
      const double d2 = ((double)g[2] - c * (double)E[2]) * inv;
      ws += d0;
      wu += d1;
      wv += d2;
      if (theta >= 0.0) step = (float)sqrt(d0 * d0 + d1 * d1 + d2 * d2);
      // every thread has read the codebook before the barrier of the sums
      if (part == 0) cb[k] = scaled();
    }
    if (theta >= 0.0) {
      step = wave_max_nonneg(step);
      if ((tid & 63) == 0) redf[tid >> 6] = step;
    }
    __syncthreads();  // the new codebook is visible; the sums are read before they are written again
    if (theta >= 0.0) {
      float smax = 0.f;
      for (int q = 0; q < NW; ++q) smax = fmaxf(smax, redf[q]);
      stop = (double)smax <= theta;
    }
  }
  if (own && part == 0) {
    w_out[3 * k] = (float)ws;
    w_out[3 * k + 1] = (float)wu;
    w_out[3 * k + 2] = (float)wv;
  }
  if (tid == 0 && iters_done) *iters_done = t;
  if (d_trace) {
    __threadfence_block();
    __syncthreads();
    for (int i = tid; i <= t; i += NT) d_trace[i] = log(d_trace[i]);
  }
}

VolTaps make_taps(const VolumeGeom& vg) {
  VolTaps tp;
  for (int i = 0; i < VOL_TAPS; ++i) tp.g[i] = tp.tg[i] = 0.f;
  for (int t = -vg.R; t <= vg.R; ++t) {
    const double g = std::exp(-(double)(t * t) / (2.0 * vg.sigma * vg.sigma));
    tp.g[t + vg.R + VOL_RUN - 1] = (float)g;
    tp.tg[t + vg.R + VOL_RUN - 1] = (float)((double)t * g);
  }
  return tp;
}

dim3 depth_grid(const VolumeGeom& vg) {
  return dim3((vg.W + 63) / 64, (vg.H + VOL_UR - 1) / VOL_UR, (vg.D + VOL_RUN - 1) / VOL_RUN);
}

template <typename WT>
hipError_t launch_volume_maps_t(const VolumeGeom& vg, const void* x, float* work, float* maps, double* sx_blk,
                                double* s_x, hipStream_t s) {
  const int64_t n = (int64_t)vg.D * vg.H * vg.W;
  float *Q00 = work, *Q01 = work + n, *Q10 = work + 2 * n;
  const VolTaps tp = make_taps(vg);
  // the staged tile has 32 + 2R <= 4 SROWS rows of 128 floats (64 + 2R of them staged): at most 48 KiB
  constexpr size_t rp = 128 * sizeof(float);
  const dim3 pg((vg.W + 63) / 64, (vg.H + VOL_TR - 1) / VOL_TR, vg.D);
  if (vg.R <= 8)
    hipLaunchKernelGGL((vol_plane_kernel<WT, 12>), pg, dim3(VOL_NT), 48 * rp, s, (const WT*)x, vg, tp, Q00, Q01, Q10);
  else if (vg.R <= 16)
    hipLaunchKernelGGL((vol_plane_kernel<WT, 16>), pg, dim3(VOL_NT), 64 * rp, s, (const WT*)x, vg, tp, Q00, Q01, Q10);
  else
    hipLaunchKernelGGL((vol_plane_kernel<WT, 24>), pg, dim3(VOL_NT), 96 * rp, s, (const WT*)x, vg, tp, Q00, Q01, Q10);
  const dim3 dg = depth_grid(vg);
  hipLaunchKernelGGL(vol_depth_kernel<WT>, dg, dim3(VOL_NT), 0, s, (const WT*)x, vg, tp, (const float*)Q00,
                     (const float*)Q01, (const float*)Q10, maps, sx_blk);
  hipLaunchKernelGGL(vol_sx_total_kernel, dim3(1), dim3(VOL_NT), 0, s, (const double*)sx_blk,
                     (int)(dg.x * dg.y * dg.z), s_x);
  return hipGetLastError();
}

template <int P, int NT>
void launch_fit_t(const VolumeGeom& vg, const float* maps, const double* s_x, int M, const float* w_init, int iters,
                  double theta, float* w_out, double* d_trace, int32_t* iters_done, hipStream_t s) {
  hipLaunchKernelGGL((vol_fit_kernel<P, NT>), dim3(1), dim3(NT), (size_t)vol_padded(M, P) * sizeof(float4), s,
                     maps, vg, s_x, M, w_init, iters, theta, w_out, d_trace, iters_done);
}

}  // namespace

int volume_sx_blocks(const VolumeGeom& vg) {
  const dim3 dg = depth_grid(vg);
  return (int)(dg.x * dg.y * dg.z);
}

hipError_t launch_volume_maps(const VolumeGeom& vg, int wdtype, const void* x, float* work, float* maps,
                              double* sx_blk, double* s_x, hipStream_t s) {
  if (vg.R < 1 || vg.R > VOL_MAXR) return hipErrorInvalidValue;
  switch (wdtype) {
    case 0: return launch_volume_maps_t<uint8_t>(vg, x, work, maps, sx_blk, s_x, s);
    case 1: return launch_volume_maps_t<float>(vg, x, work, maps, sx_blk, s_x, s);
    default: return launch_volume_maps_t<double>(vg, x, work, maps, sx_blk, s_x, s);
  }
}

hipError_t launch_volume_fit(const VolumeGeom& vg, const float* maps, const double* s_x, int M, const float* w_init,
                             int iters, double theta, float* w_out, double* d_trace, int32_t* iters_done,
                             hipStream_t s) {
  if (M > ITC_MAX_CODEVECTORS_DEV) return hipErrorInvalidValue;
  const auto go = [&](auto p, auto nt) {
    launch_fit_t<decltype(p)::value, decltype(nt)::value>(vg, maps, s_x, M, w_init, iters, theta, w_out, d_trace,
                                                          iters_done, s);
  };
  using std::integral_constant;
  // up to four pair terms a lane in one wave, without a barrier (M = 32 on one wave 1.39 us a sweep, on four
  // 1.26); then waves so that a lane has at most 4, 16, 32, 64 terms, up to the 1,024 threads of a workgroup
  // (twice the waves: M = 64 1.78 against 1.73, M = 100 3.31 against 2.56)
  if (M <= 4)
    go(integral_constant<int, 16>{}, integral_constant<int, 64>{});
  else if (M <= 8)
    go(integral_constant<int, 8>{}, integral_constant<int, 64>{});
  else if (M <= 16)
    go(integral_constant<int, 4>{}, integral_constant<int, 64>{});
  else if (M <= 32)
    go(integral_constant<int, 8>{}, integral_constant<int, 256>{});
  else if (M <= 64)
    go(integral_constant<int, 4>{}, integral_constant<int, 256>{});
  else if (M <= 128)
    go(integral_constant<int, 4>{}, integral_constant<int, 512>{});
  else if (M <= 256)
    go(integral_constant<int, 4>{}, integral_constant<int, 1024>{});
  else if (M <= 512)
    go(integral_constant<int, 2>{}, integral_constant<int, 1024>{});
  else
    go(integral_constant<int, 1>{}, integral_constant<int, 1024>{});
  return hipGetLastError();
}

}  // namespace itc
