// Maps for large kernel widths by recursive filtering (Section 3.1: for large
// widths the finite masks give way to recursive filters; the paper cites
// Deriche and van Vliet). The filter is Young and van Vliet's third-order
// recursive Gaussian: along a line, a causal pass
//   w[n] = B x[n] + a1 w[n-1] + a2 w[n-2] + a3 w[n-3]
// then an anticausal pass y[n] = B w[n] + a1 y[n+1] + a2 y[n+2] + a3 y[n+3],
// with B, a1..a3 from sigma (host side) and unit DC gain; the output is
// scaled by sqrt(2 pi) sigma to the mass of the sampled unnormalised Gaussian.
// Its cost per pixel does not depend on sigma. Every line is the lattice line
// grown by one zero pixel at each end plus m = ceil(6 sigma) zeros after it,
// so the causal response has decayed before the anticausal pass starts.
// A is filtered along v, then along u, on the lattice grown by a one-pixel
// ring; M = -sigma^2 grad A by central differences (exact for a Gaussian
// kernel: sum_y h(y) (x - y) g(x - y) = -sigma^2 d/dx sum_y h(y) g(x - y)).
//
// The recursions run in FP64, segment-parallel along the lines, in two forms.
// Lines of up to 64 x 39 samples along v and as many as the column workgroups
// hold along u (RR_SEG, RC_SEG below) stay in registers, a segment a lane: two
// kernels (second half of this file). Longer lines run down the columns of FP64
// buffers (lanes along columns, coalesced rows): the image is transposed into
// E1 (rows = v), filtered, transposed into E2 (rows = u), filtered, and the maps
// and S_X partials are read off E2.
#include "itc_device.h"

namespace itc {

namespace {

constexpr int RT = 32;  // transpose tile

// E1[r][c] = h(u = c - 1, v = r - 1) on the grown lattice, zero elsewhere.
template <typename WT>
__global__ void __launch_bounds__(RT * 8) rec_load_kernel(const WT* __restrict__ x, int64_t pitch, double scale,
                                                          int H, int W, double* __restrict__ E1, int64_t p1,
                                                          int rows1) {
  __shared__ double tile[RT][RT + 1];
  const int r0 = blockIdx.y * RT, c0 = blockIdx.x * RT;  // E1 tile: rows r0.., cols c0..
  const int tx = threadIdx.x & (RT - 1), ty = threadIdx.x / RT;
  // read along v (E1 rows) for fixed u (E1 column): contiguous in x
  for (int k = ty; k < RT; k += 8) {
    const int u = c0 + k - 1, v = r0 + tx - 1;
    double val = 0.0;
    if (u >= 0 && u < H && v >= 0 && v < W) val = scale * (double)x[(int64_t)u * pitch + v];
    tile[k][tx] = val;  // tile[u][v]
  }
  __syncthreads();
  for (int k = ty; k < RT; k += 8) {
    const int r = r0 + k, c = c0 + tx;
    if (r < rows1 && c < H + 2) E1[(int64_t)r * p1 + c] = tile[tx][k];
  }
}

// E2[r][c] = E1[c][r] for r < H + 2 (rows = u, cols = v), zero in the margin rows.
__global__ void __launch_bounds__(RT * 8) rec_transpose_kernel(const double* __restrict__ E1, int64_t p1, int H,
                                                               int W, double* __restrict__ E2, int64_t p2,
                                                               int rows2) {
  __shared__ double tile[RT][RT + 1];
  const int r0 = blockIdx.y * RT, c0 = blockIdx.x * RT;  // E2 tile
  const int tx = threadIdx.x & (RT - 1), ty = threadIdx.x / RT;
  for (int k = ty; k < RT; k += 8) {
    const int v = c0 + k, u = r0 + tx;  // E1 row v, column u
    tile[k][tx] = (v < W + 2 && u < H + 2) ? E1[(int64_t)v * p1 + u] : 0.0;
  }
  __syncthreads();
  for (int k = ty; k < RT; k += 8) {
    const int r = r0 + k, c = c0 + tx;
    if (r < rows2 && c < W + 2) E2[(int64_t)r * p2 + c] = tile[tx][k];
  }
}

// The recursions run down columns of E (rows x cols, one lane per column),
// split into segments of REC_SEG rows so that every segment of every column
// has a lane. With the state z = (w[n-1], w[n-2], w[n-3]) the recursion is
// linear, z' = A z + B x e1 with the companion matrix A of (a1, a2, a3), so
// the state after a segment is A^REC_SEG z_start plus the state the segment
// reaches from zero. Per direction: every segment's zero-state end, a scan
// over the segments of each column for the true start states, and a rerun of
// every segment from its start state that writes the values.
constexpr int RB = 8;

// Recursion over rows [lo, hi) of one column, ascending (dir > 0) or
// descending, from and into (z1, z2, z3); with OUT the values times `gain`
// replace the inputs.
template <bool OUT>
__device__ __forceinline__ void rec_run(double* col, int64_t p, int lo, int hi, int dir, const RecCoeffs& rc,
                                        double gain, double& z1, double& z2, double& z3) {
  const int n = hi - lo;
  for (int k0 = 0; k0 < n; k0 += RB) {
    double v[RB];
#pragma unroll
    for (int k = 0; k < RB; ++k) {
      const int r = dir > 0 ? lo + k0 + k : hi - 1 - k0 - k;
      v[k] = k0 + k < n ? col[(int64_t)r * p] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < RB; ++k) {
      if (k0 + k < n) {  // uniform: every lane runs the same segment
        const double w = fma(rc.a1, z1, fma(rc.a2, z2, fma(rc.a3, z3, rc.B * v[k])));
        z3 = z2;
        z2 = z1;
        z1 = w;
        v[k] = w * gain;
      }
    }
    if (OUT) {
#pragma unroll
      for (int k = 0; k < RB; ++k) {
        const int r = dir > 0 ? lo + k0 + k : hi - 1 - k0 - k;
        if (k0 + k < n) col[(int64_t)r * p] = v[k];
      }
    }
  }
}

// Z layout: [segment][3][cols].
__device__ __forceinline__ double* zat(double* Z, int sg, int q, int cols, int c) {
  return Z + ((int64_t)sg * 3 + q) * cols + c;
}

// Zero-state end of every segment along dir (blockIdx.y = segment).
__global__ void __launch_bounds__(64) rec_seg_end_kernel(double* __restrict__ E, int64_t p, int rows, int cols,
                                                         RecCoeffs rc, int dir, double* __restrict__ Z) {
  const int c = blockIdx.x * 64 + threadIdx.x, sg = blockIdx.y;
  if (c >= cols) return;
  const int lo = sg * REC_SEG, hi = min(lo + REC_SEG, rows);
  double z1 = 0.0, z2 = 0.0, z3 = 0.0;
  rec_run<false>(E + c, p, lo, hi, dir, rc, 1.0, z1, z2, z3);
  *zat(Z, sg, 0, cols, c) = z1;
  *zat(Z, sg, 1, cols, c) = z2;
  *zat(Z, sg, 2, cols, c) = z3;
}

// Start states from the zero-state ends, in place: segments in the order of
// dir, z_start(first) = 0, z_start(next) = A^REC_SEG z_start + z_end0. Only
// the segment last in that order can be shorter, and its end is not carried.
__global__ void __launch_bounds__(64) rec_seg_scan_kernel(double* __restrict__ Z, int nseg, int cols, RecCoeffs rc,
                                                          int dir) {
  const int c = blockIdx.x * 64 + threadIdx.x;
  if (c >= cols) return;
  const double* P = rc.P;
  double z1 = 0.0, z2 = 0.0, z3 = 0.0;
  constexpr int SB = 8;  // segments whose ends are loaded together
  for (int i0 = 0; i0 < nseg; i0 += SB) {
    double f[SB][3];
#pragma unroll
    for (int q = 0; q < SB; ++q) {
      const int i = i0 + q;
      const int sg = dir > 0 ? i : nseg - 1 - i;
      f[q][0] = f[q][1] = f[q][2] = 0.0;
      if (i < nseg) {
        f[q][0] = *zat(Z, sg, 0, cols, c);
        f[q][1] = *zat(Z, sg, 1, cols, c);
        f[q][2] = *zat(Z, sg, 2, cols, c);
      }
    }
#pragma unroll
    for (int q = 0; q < SB; ++q) {
      const int i = i0 + q;
      if (i >= nseg) break;
      const int sg = dir > 0 ? i : nseg - 1 - i;
      *zat(Z, sg, 0, cols, c) = z1;
      *zat(Z, sg, 1, cols, c) = z2;
      *zat(Z, sg, 2, cols, c) = z3;
      const double n1 = fma(P[0], z1, fma(P[1], z2, fma(P[2], z3, f[q][0])));
      const double n2 = fma(P[3], z1, fma(P[4], z2, fma(P[5], z3, f[q][1])));
      const double n3 = fma(P[6], z1, fma(P[7], z2, fma(P[8], z3, f[q][2])));
      z1 = n1;
      z2 = n2;
      z3 = n3;
    }
  }
}

// Rerun of every segment from its start state. Causal (dir > 0): writes w,
// then leaves in Z the zero-state end of the anticausal pass over the same
// rows (this lane's own values, just written). Anticausal: writes y * gain.
__global__ void __launch_bounds__(64) rec_seg_apply_kernel(double* __restrict__ E, int64_t p, int rows, int cols,
                                                           RecCoeffs rc, int dir, double* __restrict__ Z) {
  const int c = blockIdx.x * 64 + threadIdx.x, sg = blockIdx.y;
  if (c >= cols) return;
  const int lo = sg * REC_SEG, hi = min(lo + REC_SEG, rows);
  double z1 = *zat(Z, sg, 0, cols, c), z2 = *zat(Z, sg, 1, cols, c), z3 = *zat(Z, sg, 2, cols, c);
  if (dir > 0) {
    rec_run<true>(E + c, p, lo, hi, 1, rc, 1.0, z1, z2, z3);
    z1 = z2 = z3 = 0.0;
    rec_run<false>(E + c, p, lo, hi, -1, rc, 1.0, z1, z2, z3);
    *zat(Z, sg, 0, cols, c) = z1;
    *zat(Z, sg, 1, cols, c) = z2;
    *zat(Z, sg, 2, cols, c) = z3;
  } else {
    rec_run<true>(E + c, p, lo, hi, -1, rc, rc.gain, z1, z2, z3);
  }
}

// Causal then anticausal pass down every column of E, in place.
void rec_filter(double* E, int64_t p, int rows, int cols, const RecCoeffs& rc, double* Z, hipStream_t s) {
  const dim3 g((cols + 63) / 64, (rows + REC_SEG - 1) / REC_SEG), b(64);
  const int nseg = (int)g.y;
  hipLaunchKernelGGL(rec_seg_end_kernel, g, b, 0, s, E, p, rows, cols, rc, 1, Z);
  hipLaunchKernelGGL(rec_seg_scan_kernel, dim3(g.x), b, 0, s, Z, nseg, cols, rc, 1);
  hipLaunchKernelGGL(rec_seg_apply_kernel, g, b, 0, s, E, p, rows, cols, rc, 1, Z);
  hipLaunchKernelGGL(rec_seg_scan_kernel, dim3(g.x), b, 0, s, Z, nseg, cols, rc, -1);
  hipLaunchKernelGGL(rec_seg_apply_kernel, g, b, 0, s, E, p, rows, cols, rc, -1, Z);
}

// Maps (FP32 planes, panel layout) and the FP64 S_X partials from the
// filtered E2: a block of 64 threads takes one panel (16 columns) of one
// S_X row group, lane (c, r) = (lane mod 16, lane / 16) columns c and rows
// r, r + 4, ... of it. Panels past the width (the last strip's) only clear
// their partial slot; columns past the width inside the last panel are 0.
template <typename WT>
__global__ void __launch_bounds__(64) rec_maps_kernel(const double* __restrict__ E2, int64_t p2, const WT* x,
                                                      int64_t pitch, double scale, double sigma, ImageDesc im,
                                                      char* maps) {
  const int panel = blockIdx.x, grp = blockIdx.y;
  const int lane = threadIdx.x, c = lane & 15, r = lane >> 4;
  const int v = panel * MAP_PANEL + c;
  float* A = reinterpret_cast<float*>(maps);
  float* Mu = A + im.plane;
  float* Mv = Mu + im.plane;
  const double k = -0.5 * sigma * sigma;
  double sx = 0.0;
  if (panel < im.npanels) {
    for (int i = 0; i < SX_ROWS / 4; ++i) {
      const int u = grp * SX_ROWS + r + 4 * i;
      if (u >= im.H) break;
      float a = 0.f, mu = 0.f, mv = 0.f;
      if (v < im.W) {
        const double* e = E2 + (int64_t)(u + 1) * p2 + (v + 1);
        const double ac = e[0];
        a = (float)ac;
        mu = (float)(k * (e[p2] - e[-p2]));
        mv = (float)(k * (e[1] - e[-1]));
        sx = fma(scale * (double)x[(int64_t)u * pitch + v], (double)a, sx);
      }
      const int64_t o = map_index(im.H, u, v);
      A[o] = a;
      Mu[o] = mu;
      Mv[o] = mv;
    }
  }
  sx = wave_sum(sx);
  if (lane == 0) {
    double* part = reinterpret_cast<double*>(maps + im.part_off);
    part[((int64_t)(panel / 4) * im.nsxg + grp) * SX_SLOTS + panel % 4] = sx;
  }
}

// ---------------------------------------------------------------------------
// Lines held in registers: two launches instead of fifteen over FP64 buffers.
//
// A line is cut into segments of SEG entries, one thread per segment, and the
// thread keeps its segment in registers through both directions: a run for the
// zero-state end, a scan of the ends over the segments of the line, a rerun
// from the true start, and the same backwards. The scale, B and the gain of
// both axes are one factor on the input, so a step is three FMAs.
//   * rows (along v): a wave takes one image row, lane = segment; the row goes
//     through LDS on its way in and out, so that global accesses are contiguous
//     and a lane finds its own entries (SEG is odd: 64 lanes meet all banks);
//     the scan is six steps of lane shifts with the powers P^1 .. P^32 of
//     P = A^SEG. Writes E1: for each run of columns of the second pass, the
//     rows of its columns and one more on each side, contiguous.
//   * columns (along u): a workgroup takes half a map panel, 8 columns, and one
//     more column on each side for M_v (10 x 48 threads: column, segment); it
//     reads E1 once, scans in LDS (groups of six segments, then the eight groups),
//     and writes A, M_u, M_v and S_X straight from the registers: M_u from the
//     thread's own neighbours (the ends of the next segments through LDS), M_v
//     from the lanes beside it. Half panels rather than whole ones (18 x 56
//     threads, 47 us): a 2048-wide image then gives 256 workgroups instead of
//     128, and a thread may use twice the registers, so nothing spills. Whole
//     panels are kept for images of one S_X row group (at most 64 rows), where a
//     panel has one S_X slot.
// 2048 x 2048 8-bit, sigma = 16: 48 us a call, one queued after another (rows 16,
// columns 31, S_X 4 under the profiler) against 177; 64 x 100: 27 against 77. Bound by E1's way through the caches (42 MB out and in)
// and the maps' 50 MB, then by the chains of dependent FMAs.
// ---------------------------------------------------------------------------
// The column pass for COLS columns: threads, segments in groups.
template <int COLS>
struct RecCols {
  static constexpr int C = COLS + 2, NT = COLS == 8 ? 512 : 1024, GROUPS = 8, PER = COLS == 8 ? 6 : 7,
                       SEGS = GROUPS * PER, WAVES = NT / 64;
  static_assert(C * SEGS <= NT, "one thread per column and segment");
};
constexpr int RR_LANES = 64, RR_ROWS = 4;

// a1..a3 and powers of P = A^SEG (row-major): rows P^1, P^2, .., P^32; columns P, P^(segments of a group).
struct RecLine {
  double a1, a2, a3;
  double P[6][9];
};

__device__ __forceinline__ void mat_add(const double* P, const double (&x)[3], double (&y)[3]) {
  y[0] = fma(P[0], x[0], fma(P[1], x[1], fma(P[2], x[2], y[0])));
  y[1] = fma(P[3], x[0], fma(P[4], x[1], fma(P[5], x[2], y[1])));
  y[2] = fma(P[6], x[0], fma(P[7], x[1], fma(P[8], x[2], y[2])));
}

__device__ __forceinline__ double rec_step(const RecLine& rl, double x, double (&z)[3]) {
  const double w = fma(rl.a1, z[0], fma(rl.a2, z[1], fma(rl.a3, z[2], x)));
  z[2] = z[1];
  z[1] = z[0];
  z[0] = w;
  return w;
}

// Segment runs over x[0 .. SEG), ascending or descending, from the state z;
// with OUT the values replace the inputs.
template <int SEG, bool UP, bool OUT>
__device__ __forceinline__ void seg_run(const RecLine& rl, double (&x)[SEG], double (&z)[3]) {
#pragma unroll
  for (int q = 0; q < SEG; ++q) {
    const int j = UP ? q : SEG - 1 - q;
    const double w = rec_step(rl, x[j], z);
    if constexpr (OUT) x[j] = w;
  }
}

// Zeroes the entries of a segment from line position `len` on (the causal
// response ends there; the anticausal pass starts from zero).
template <int SEG>
__device__ __forceinline__ void cut_line(double (&x)[SEG], int n0, int len) {
  if (n0 + SEG > len) {
#pragma unroll
    for (int j = 0; j < SEG; ++j) x[j] = n0 + j < len ? x[j] : 0.0;
  }
}

// Start states of a wave's segments (lane = segment) from their zero-state
// ends z; UP: segments in lane order, else from lane 63 down.
template <bool UP>
__device__ __forceinline__ void lane_scan(const RecLine& rl, double (&z)[3], int lane) {
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const int d = 1 << k;
    double y[3];
    const bool on = UP ? lane >= d : lane + d < 64;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const double o = UP ? __shfl_up(z[q], d, 64) : __shfl_down(z[q], d, 64);
      y[q] = on ? o : 0.0;
    }
    mat_add(rl.P[k], y, z);
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const double o = UP ? __shfl_up(z[q], 1, 64) : __shfl_down(z[q], 1, 64);
    z[q] = (UP ? lane >= 1 : lane < 63) ? o : 0.0;
  }
}

template <typename WT, int COLS, int SEG>
__global__ void __launch_bounds__(64 * RR_ROWS) rec_rows_kernel(const WT* __restrict__ x, int64_t pitch, double factor,
                                                                int H, int W, int len, RecLine rl,
                                                                double* __restrict__ E1) {
  extern __shared__ __align__(16) double rline[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int u = blockIdx.x * RR_ROWS + wave;
  if (u >= H) return;  // no barrier below: a wave uses its own line of LDS only
  double* buf = rline + wave * (RR_LANES * SEG);
  const rsrc_t xr = make_rsrc(x + (int64_t)u * pitch, (uint32_t)W * (uint32_t)sizeof(WT));
  WT raw[SEG];
#pragma unroll
  for (int q = 0; q < SEG; ++q) {  // position i = v + 1; outside the row reads 0
    const int v = 64 * q + lane - 1;
    raw[q] = buf_load<WT>(xr, v < 0 || v >= W ? BUF_OOB : (uint32_t)v * (uint32_t)sizeof(WT), 0);
  }
#pragma unroll
  for (int q = 0; q < SEG; ++q) buf[64 * q + lane] = factor * (double)raw[q];
  wave_lds_order();
  double s[SEG], z[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < SEG; ++j) s[j] = buf[lane * SEG + j];
  seg_run<SEG, true, false>(rl, s, z);
  lane_scan<true>(rl, z, lane);
  seg_run<SEG, true, true>(rl, s, z);
  cut_line<SEG>(s, lane * SEG, len);
  z[0] = z[1] = z[2] = 0.0;
  seg_run<SEG, false, false>(rl, s, z);
  lane_scan<false>(rl, z, lane);
  seg_run<SEG, false, true>(rl, s, z);
  wave_lds_order();
#pragma unroll
  for (int j = 0; j < SEG; ++j) buf[lane * SEG + j] = s[j];
  wave_lds_order();
  // E1[run][u][C]: columns COLS run - 1 .. COLS run + COLS of the image
  constexpr int C = RecCols<COLS>::C;
  const int n = (W + COLS - 1) / COLS * C;
  for (int i = lane; i < n; i += 64) {
    const int run = i / C, c = i - run * C;
    E1[((int64_t)run * H + u) * C + c] = buf[min(run * COLS + c, RR_LANES * SEG - 1)];  // past W + 1: not read
  }
}

// LDS of the column pass.
template <int COLS, int SEG>
struct RecColsSmem {
  using G = RecCols<COLS>;
  double st[G::SEGS][3][G::C];   // segment ends, then starts
  double grp[G::GROUPS][3][G::C];
  double first[G::SEGS + 1][G::C], last[G::SEGS + 1][G::C];  // end values of the segments, for M_u
  double edge[G::WAVES + 2][2][SEG];  // values of each wave's first and last lane, for M_v
  double red[G::WAVES];
};

template <int C>
__device__ __forceinline__ void get3(double (&z)[3], const double (*e)[C], int c) {
  z[0] = e[0][c], z[1] = e[1][c], z[2] = e[2][c];
}
template <int C>
__device__ __forceinline__ void put3(double (*e)[C], int c, const double (&z)[3]) {
  e[0][c] = z[0], e[1][c] = z[1], e[2][c] = z[2];
}

// Start states of every segment from the zero-state ends in sm.st, in place;
// UP: segments in increasing order. The segments of a group, one thread each,
// then the groups, then the segments again from their group's start. One entry
// is loaded ahead of its use (more would take the segments' registers).
template <bool UP, typename SM>
__device__ __forceinline__ void seg_scan(SM& sm, const RecLine& rl, int tid) {
  using G = typename SM::G;
  constexpr int PER = G::PER;
  __syncthreads();
  const int c = tid % G::C, g = tid / G::C;
  auto seg_of = [&](int i) { return UP ? g * PER + i : G::SEGS - 1 - (g * PER + i); };
  if (g < G::GROUPS) {
    double z[3] = {0.0, 0.0, 0.0}, f[3];
    get3(f, sm.st[seg_of(0)], c);
#pragma unroll 1
    for (int i = 0; i < PER; ++i) {
      double n[3] = {f[0], f[1], f[2]};
      get3(f, sm.st[seg_of(min(i + 1, PER - 1))], c);
      mat_add(rl.P[0], z, n);
      z[0] = n[0], z[1] = n[1], z[2] = n[2];
    }
    put3(sm.grp[g], c, z);
  }
  __syncthreads();
  if (tid < G::C) {
    double z[3] = {0.0, 0.0, 0.0}, f[3];
    get3(f, sm.grp[0], tid);
#pragma unroll 1
    for (int i = 0; i < G::GROUPS; ++i) {
      double n[3] = {f[0], f[1], f[2]};
      get3(f, sm.grp[min(i + 1, G::GROUPS - 1)], tid);
      put3(sm.grp[i], tid, z);
      mat_add(rl.P[1], z, n);
      z[0] = n[0], z[1] = n[1], z[2] = n[2];
    }
  }
  __syncthreads();
  if (g < G::GROUPS) {
    double z[3], f[3];
    get3(z, sm.grp[g], c);
    get3(f, sm.st[seg_of(0)], c);
#pragma unroll 1
    for (int i = 0; i < PER; ++i) {
      double n[3] = {f[0], f[1], f[2]};
      get3(f, sm.st[seg_of(min(i + 1, PER - 1))], c);
      put3(sm.st[seg_of(i)], c, z);
      mat_add(rl.P[0], z, n);
      z[0] = n[0], z[1] = n[1], z[2] = n[2];
    }
  }
  __syncthreads();
}

// The value of the lane before (or after) this one; lane 0 (63) gets its `edge`.
template <bool BEFORE>
__device__ __forceinline__ double lane_beside(double x, double edge) {
  constexpr int CTRL = BEFORE ? 0x138 : 0x130;  // wave_shr:1, wave_shl:1
  const int2 v = __builtin_bit_cast(int2, x), e = __builtin_bit_cast(int2, edge);
  int2 o;  // a lane without a source keeps the old value
  o.x = __builtin_amdgcn_update_dpp(e.x, v.x, CTRL, 0xf, 0xf, false);
  o.y = __builtin_amdgcn_update_dpp(e.y, v.y, CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, o);
}

// A workgroup takes run `which` of a panel; the runs of one panel, whose stores
// share its lines, are 8 workgroups apart, on one XCD. Panels past the width
// (the last strip's) only clear their S_X slots.
template <typename WT, int COLS, int SEG>
__global__ void __launch_bounds__(RecCols<COLS>::NT) rec_cols_kernel(const double* __restrict__ E1,
                                                                     const WT* __restrict__ x, int64_t pitch,
                                                                     double scale, double sigma, int len, RecLine rl,
                                                                     ImageDesc im, char* maps) {
  using G = RecCols<COLS>;
  constexpr int PARTS = MAP_PANEL / COLS;  // workgroups of a panel
  extern __shared__ __align__(16) char rsm[];
  auto& sm = *reinterpret_cast<RecColsSmem<COLS, SEG>*>(rsm);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bx = blockIdx.x / CONV_XCDS, panel = bx / PARTS * CONV_XCDS + blockIdx.x % CONV_XCDS, which = bx % PARTS;
  const int H = im.H, W = im.W, run = panel * PARTS + which;
  if (panel >= im.nstrips * SX_SLOTS) return;  // uniform
  double* part = reinterpret_cast<double*>(maps + im.part_off) + (int64_t)(panel / 4) * im.nsxg * SX_SLOTS + panel % 4;
  // S_X of the whole line goes to the slot of row group `which` (there are at least PARTS)
  for (int g = PARTS + tid; g < im.nsxg; g += G::NT)
    if (which == 0) part[(int64_t)g * SX_SLOTS] = 0.0;
  if (COLS * run >= W) {  // uniform: past the width
    if (tid == 0) part[(int64_t)which * SX_SLOTS] = 0.0;
    if (panel >= im.npanels) return;
  }
  const int c = tid % G::C, sg = tid / G::C;
  const bool on = sg < G::SEGS;
  const int vg = COLS * run + c;  // v + 1
  const int n0 = sg * SEG;                    // line position of the segment; u = n - 1
  constexpr uint32_t rowb = G::C * 8u;
  const rsrc_t er = make_rsrc(E1 + (int64_t)run * H * G::C, COLS * run < W ? (uint32_t)H * rowb : 0u);
  double s[SEG];
  {
    // rows after the image are past the buffer, and so is the row before it (entry 0 has an offset of its own,
    // which wraps; the others are at constant distances from entry 1)
    uint32_t e0 = on ? (uint32_t)(n0 - 1) * rowb + (uint32_t)c * 8u : BUF_OOB;
    uint32_t e1 = on ? (uint32_t)n0 * rowb + (uint32_t)c * 8u : BUF_OOB;
    asm("" : "+v"(e0));
    asm("" : "+v"(e1));
#pragma unroll
    for (int j = 0; j < SEG; ++j) s[j] = buf_load<double>(er, j == 0 ? e0 : e1 + (uint32_t)(j - 1) * rowb, 0);
  }
  double z[3] = {0.0, 0.0, 0.0};
  seg_run<SEG, true, false>(rl, s, z);
  if (on) put3(sm.st[sg], c, z);
  seg_scan<true>(sm, rl, tid);
  if (on) get3(z, sm.st[sg], c);
  seg_run<SEG, true, true>(rl, s, z);
  cut_line<SEG>(s, n0, len);
  z[0] = z[1] = z[2] = 0.0;
  seg_run<SEG, false, false>(rl, s, z);
  if (on) put3(sm.st[sg], c, z);  // own slot, read above
  seg_scan<false>(sm, rl, tid);
  if (on) get3(z, sm.st[sg], c);
  seg_run<SEG, false, true>(rl, s, z);
  if (on) {
    sm.first[sg][c] = s[0];
    sm.last[sg + 1][c] = s[SEG - 1];
  }
  if (tid < G::C) sm.first[G::SEGS][tid] = sm.last[0][tid] = 0.0;
  if (lane == 0 || lane == 63) {
    double* e = sm.edge[wave + 1][lane == 63];
#pragma unroll
    for (int j = 0; j < SEG; ++j) e[j] = s[j];
  }
  __syncthreads();
  // ---- maps and S_X ----
  const double k = -0.5 * sigma * sigma;
  const bool mine = on && c >= 1 && c <= COLS;
  const int v = vg - 1, pc = COLS * which + c - 1;  // image column, column of the panel
  // One descriptor per plane that ends with the panel's rows: rows past the image are dropped. Lanes without
  // a pixel column take offsets past it (columns past the width are cleared below). Entry 0 has an offset of
  // its own (row -1 wraps past the end); the others are at constant distances from entry 1.
  const uint32_t panelb = (uint32_t)H * (uint32_t)(MAP_PANEL * 4);
  char* pbase = maps + (int64_t)panel * panelb;
  const int64_t planeb = im.plane * 4;
  const rsrc_t ra = make_rsrc(pbase, panelb), ru = make_rsrc(pbase + planeb, panelb), rv = make_rsrc(pbase + 2 * planeb, panelb);
  const bool px = mine && v < W;
  uint32_t o0 = px ? (uint32_t)(n0 - 1) * (uint32_t)(MAP_PANEL * 4) + (uint32_t)pc * 4u : BUF_OOB;
  uint32_t o1 = px ? (uint32_t)n0 * (uint32_t)(MAP_PANEL * 4) + (uint32_t)pc * 4u : BUF_OOB;
  asm("" : "+v"(o0));
  asm("" : "+v"(o1));
  const rsrc_t xr = make_rsrc(x, (uint32_t)((uint64_t)H * (uint64_t)pitch * sizeof(WT)));
  const uint32_t xrow = (uint32_t)pitch * (uint32_t)sizeof(WT);
  // The weights of the line's rows, below 2^31 like xrow. Rows past the image stay at BUF_OOB: with a wide pitch
  // their offsets would wrap back into the buffer.
  auto weight_off = [&](int u) {
    return px && (unsigned)u < (unsigned)H ? (uint32_t)u * xrow + (uint32_t)v * (uint32_t)sizeof(WT) : BUF_OOB;
  };
  const uint32_t x0 = weight_off(n0 - 1);
  uint32_t xo = weight_off(n0);
  const double* eb = sm.edge[lane == 0 ? wave : wave + 2][lane == 0];  // lane 0: the wave before's last lane
  const double before = on ? sm.last[sg][c] : 0.0, after = on ? sm.first[sg + 1][c] : 0.0;
  double sx = 0.0;
  constexpr int XB = 8;  // image entries loaded together
  for_each_index(
      [&](auto bb) {
        constexpr int j0 = decltype(bb)::value * XB, nb = SEG - j0 < XB ? SEG - j0 : XB;
        WT h[nb];
#pragma unroll
        for (int q = 0; q < nb; ++q) {
          h[q] = buf_load<WT>(xr, j0 + q == 0 ? x0 : xo, 0);
          if (j0 + q > 0) xo = min(xo + xrow, BUF_OOB);
        }
#pragma unroll
        for (int q = 0; q < nb; ++q) {
          const int j = j0 + q;
          const double edge = eb[j];
          const double l = lane_beside<true>(s[j], edge), r = lane_beside<false>(s[j], edge);
          const double up = j > 0 ? s[j > 0 ? j - 1 : 0] : before, dn = j + 1 < SEG ? s[j + 1 < SEG ? j + 1 : j] : after;
          const float a = (float)s[j];
          const uint32_t off = j == 0 ? o0 : o1 + (uint32_t)(j - 1) * (MAP_PANEL * 4);
          buf_store(a, ra, off, 0);
          buf_store((float)(k * (dn - up)), ru, off, 0);
          buf_store((float)(k * (r - l)), rv, off, 0);
          sx = fma((double)h[q], (double)a, sx);
        }
        __builtin_amdgcn_sched_barrier(0);
      },
      std::make_integer_sequence<int, (SEG + XB - 1) / XB>{});
  sx = block_reduce_fixed(sx, sm.red);
  if (tid == 0 && COLS * run < W) part[(int64_t)which * SX_SLOTS] = scale * sx;
  const int past = COLS * (run + 1) - W;  // columns past the width among the COLS
  if (past > 0) {
    const int np = min(past, COLS);
    for (int i = tid; i < H * np; i += G::NT) {
      const uint32_t off = (uint32_t)(i / np) * (uint32_t)(MAP_PANEL * 4) + (uint32_t)(COLS * which + COLS - 1 - i % np) * 4u;
      buf_store(0.f, ra, off, 0);
      buf_store(0.f, ru, off, 0);
      buf_store(0.f, rv, off, 0);
    }
  }
}

constexpr int REC_NSEG = 6;
constexpr int RR_SEG[REC_NSEG] = {7, 13, 19, 25, 35, 39}, RC_SEG[REC_NSEG] = {8, 16, 25, 34, 45, 52};
constexpr int RC_SEG_LOW = 8;  // whole panels: images of at most 64 rows

// First compiled segment length that holds a line of len entries cut in n segments (REC_NSEG: none).
inline int seg_index(const int (&segs)[REC_NSEG], int n, int len) {
  int i = 0;
  while (i < REC_NSEG && segs[i] * n < len) ++i;
  return i;
}

// A 3 x 3 matrix in extended precision: the companion matrix of (a1, a2, a3) has
// its poles crowded at 1 for large sigma, and rounding the products that form its
// powers to FP64 would cost 1e-9 relative in the maps at sigma = 40 (4e-11 so).
struct Mat3 {
  long double m[9];
  Mat3 operator*(const Mat3& o) const {
    Mat3 r;
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j)
        r.m[3 * i + j] = m[3 * i] * o.m[j] + m[3 * i + 1] * o.m[3 + j] + m[3 * i + 2] * o.m[6 + j];
    return r;
  }
  Mat3 power(int n) const {  // n >= 1
    Mat3 a = *this;
    for (; !(n & 1); n >>= 1) a = a * a;
    Mat3 r = a;
    while (n >>= 1) {
      a = a * a;
      if (n & 1) r = a * r;
    }
    return r;
  }
  void get(double* p) const {
    for (int i = 0; i < 9; ++i) p[i] = (double)m[i];
  }
};

Mat3 companion(const RecCoeffs& rc) { return Mat3{{rc.a1, rc.a2, rc.a3, 1, 0, 0, 0, 1, 0}}; }

template <typename WT, int COLS, int SEG>
hipError_t launch_rec_rows(const ImageDesc& im, const WT* x, double factor, int len, const RecCoeffs& rc, double* E1,
                           hipStream_t s) {
  RecLine rl{rc.a1, rc.a2, rc.a3, {}};
  Mat3 P = companion(rc).power(SEG);
  for (int k = 0; k < 6; ++k, P = P * P) P.get(rl.P[k]);
  hipLaunchKernelGGL((rec_rows_kernel<WT, COLS, SEG>), dim3((im.H + RR_ROWS - 1) / RR_ROWS), dim3(64 * RR_ROWS),
                     (size_t)RR_ROWS * RR_LANES * SEG * sizeof(double), s, x, im.pitch, factor, im.H, im.W, len, rl, E1);
  return hipGetLastError();
}

template <typename WT, int COLS, int SEG>
hipError_t launch_rec_cols(const ImageDesc& im, const WT* x, double scale, double sigma, int len, const RecCoeffs& rc,
                           const double* E1, void* maps, hipStream_t s) {
  using G = RecCols<COLS>;
  RecLine rl{rc.a1, rc.a2, rc.a3, {}};
  const Mat3 P = companion(rc).power(SEG);
  P.get(rl.P[0]);
  P.power(G::PER).get(rl.P[1]);
  const int panels = (im.nstrips * SX_SLOTS + CONV_XCDS - 1) / CONV_XCDS * CONV_XCDS;
  hipLaunchKernelGGL((rec_cols_kernel<WT, COLS, SEG>), dim3((unsigned)(panels * (MAP_PANEL / COLS))), dim3(G::NT), sizeof(RecColsSmem<COLS, SEG>), s, E1, x, im.pitch, scale, sigma, len, rl, im,
                     (char*)maps);
  return hipGetLastError();
}

// f(integral_constant<int, I>) for the index i < REC_NSEG.
template <typename F, int... I>
hipError_t with_index(int i, F&& f, std::integer_sequence<int, I...>) {
  hipError_t e = hipErrorInvalidValue;
  ((i == I ? (void)(e = f(std::integral_constant<int, I>{})) : (void)0), ...);
  return e;
}

template <typename WT>
hipError_t launch_recursive_t(const ImageDesc& im, const void* x, double scale, double sigma, const RecCoeffs& rc,
                              double* E1, double* E2, double* Z, void* maps, hipStream_t s) {
  const int H = im.H, W = im.W;
  const int rows1 = W + 2 + rc.m, cols1 = H + 2;
  const int rows2 = H + 2 + rc.m, cols2 = W + 2;
  const int ir = seg_index(RR_SEG, RR_LANES, rows1), ic = seg_index(RC_SEG, RecCols<8>::SEGS, rows2);
  const bool low = im.nsxg < 2;
  const int cols = low ? 16 : 8;
  const size_t e1 = (size_t)((W + cols - 1) / cols) * (size_t)H * (size_t)(cols + 2) * sizeof(double);
  // both lines fit the registers, and E1 the buffers of the other form (it does unless W is 1 or 2); E1, the
  // image and a panel stay below 2 GiB
  if (ir < REC_NSEG && (low ? rows2 <= RC_SEG_LOW * RecCols<16>::SEGS : ic < REC_NSEG) &&
      e1 <= (size_t)((const char*)Z - (const char*)E1)) {
    const double axis = rc.B * rc.B * rc.gain, factor = scale * axis * axis;
    const WT* xw = (const WT*)x;
    const auto idx = std::make_integer_sequence<int, REC_NSEG>{};
    const hipError_t e = with_index(
        ir,
        [&](auto i) {
          constexpr int SEG = RR_SEG[decltype(i)::value];
          return low ? launch_rec_rows<WT, 16, SEG>(im, xw, factor, rows1, rc, E1, s)
                     : launch_rec_rows<WT, 8, SEG>(im, xw, factor, rows1, rc, E1, s);
        },
        idx);
    if (e != hipSuccess) return e;
    if (low) return launch_rec_cols<WT, 16, RC_SEG_LOW>(im, xw, scale, sigma, rows2, rc, E1, maps, s);
    return with_index(
        ic,
        [&](auto i) {
          return launch_rec_cols<WT, 8, RC_SEG[decltype(i)::value]>(im, xw, scale, sigma, rows2, rc, E1, maps, s);
        },
        idx);
  }
  const int64_t p1 = cols1, p2 = cols2;
  hipLaunchKernelGGL(rec_load_kernel<WT>, dim3((cols1 + RT - 1) / RT, (rows1 + RT - 1) / RT), dim3(RT * 8), 0, s,
                     (const WT*)x, im.pitch, scale, H, W, E1, p1, rows1);
  rec_filter(E1, p1, rows1, cols1, rc, Z, s);
  hipLaunchKernelGGL(rec_transpose_kernel, dim3((cols2 + RT - 1) / RT, (rows2 + RT - 1) / RT), dim3(RT * 8), 0, s,
                     (const double*)E1, p1, H, W, E2, p2, rows2);
  rec_filter(E2, p2, rows2, cols2, rc, Z, s);
  static_assert(SX_SLOTS * MAP_PANEL == CONV_TW, "four panels per strip");
  hipLaunchKernelGGL(rec_maps_kernel<WT>, dim3((unsigned)(im.nstrips * SX_SLOTS), (unsigned)im.nsxg), dim3(64), 0,
                     s, (const double*)E2, p2, (const WT*)x, im.pitch, scale, sigma, im, (char*)maps);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_recursive(const ImageDesc& im, const void* x, double scale, double sigma, const RecCoeffs& rc,
                            double* E1, double* E2, double* Z, void* maps, hipStream_t s) {
  switch (im.wdtype) {
    case 0: return launch_recursive_t<uint8_t>(im, x, scale, sigma, rc, E1, E2, Z, maps, s);
    case 1: return launch_recursive_t<float>(im, x, scale, sigma, rc, E1, E2, Z, maps, s);
    default: return launch_recursive_t<double>(im, x, scale, sigma, rc, E1, E2, Z, maps, s);
  }
}

}  // namespace itc
