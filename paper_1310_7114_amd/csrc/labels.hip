// Pixel-to-codevector labelling: every pixel of weight > 0 gets the index of
// the nearest codevector (Euclidean; the smaller index on ties), every other
// pixel -1 (the shape segments that a codebook induces, Section 4). The
// squared distance is (u - w_u)^2 + (v - w_v)^2 in FP64 with two rounded
// products and a rounded sum (no fused multiply-add), so the decisions are
// reproducible bit for bit by any IEEE evaluation in the same order.
//
// A wave labels tiles of 16 x 32 pixels, eight per lane (two rows of four
// adjacent ones; one per lane where codevectors are dense, label_dense below), on
// its own: no barrier and no list. Per tile it scans only the
// codevectors that can be nearest to one of its pixels: with L_k and U_k a lower
// and an upper bound of the squared distance from w_k to the box of the tile's
// pixel centres, every pixel's nearest distance is at most U* = min_k U_k, so a
// codevector with L_k > U* (1 + 1e-5) is farther than the nearest one from every
// pixel of the tile, by more than any rounding of the FP64 distances (a few
// 2^-53 relative). The bounds are formed 64 codevectors at a time, one per lane,
// from FP64 differences to the box's centre rounded outwards to FP32; the others
// are taken in increasing index from the wave's ballot, their coordinates read
// out of their lane into scalar registers, and scanned with the same arithmetic
// and the same strict comparison as a scan over all codevectors, so the labels,
// ties included, are those of the full scan. Tiles without a pixel of weight > 0
// skip all of it.
//
// Bound by memory (5 B/px) and, on the foreground tiles, by seven vector
// instructions per pixel and candidate; the bounds cost about 60 instructions
// per 64 codevectors and 512 pixels. The labels go out in non-temporal stores: 0.46 ms
// against 0.50 for 1,400 silhouettes, whose dirty lines the next call evicted (one
// image 6.9 us, 9.3). 1,400 silhouettes (355 Mpx): 0.46 ms, 3.9 TB/s,
// against 1.06 ms with 8 x 32 tiles of a whole workgroup, a list in LDS and three
// barriers a tile; one image: 7 us against 22.
#include "itc_device.h"

namespace itc {

namespace {

constexpr int LB_NT = 256;
constexpr int LB_WAVES = LB_NT / 64;
// A tile of a wave: 8 x 8 lanes with Q rows and V adjacent columns each; WR of a workgroup's waves one below the
// other, the others beside them.
template <int Q, int V, int WR>
struct LabelTile {
  static constexpr int ROWS = 8 * Q, COLS = 8 * V, GROUP_ROWS = ROWS * WR, STEP = COLS * (LB_WAVES / WR);
};
constexpr float LB_MARGIN = 1.0f + 1e-5f;
constexpr float LB_ROUND = 3e-7f;  // more than the relative rounding of a difference to FP32

typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));

// Codebook of one image into LDS as FP64 (u, v).
template <typename T>
__device__ __forceinline__ void stage_codebook(const T* w, int M, double2* sw) {
  for (int k = threadIdx.x; k < M; k += LB_NT) sw[k] = make_double2((double)w[2 * k], (double)w[2 * k + 1]);
}

// V adjacent stored weights.
template <typename WT, int V>
struct Adjacent {
  WT w[V];
};
// 8-bit rows whose length and start are multiples of four: one load.
__device__ __forceinline__ Adjacent<uint8_t, 4> unpack(uint32_t x) {
  return Adjacent<uint8_t, 4>{{(uint8_t)x, (uint8_t)(x >> 8), (uint8_t)(x >> 16), (uint8_t)(x >> 24)}};
}

// A workgroup's rows from r0 of one image. `quads`: 8-bit rows are 4-byte aligned (base and pitch).
template <int Q, int V, int WR, typename WT>
__device__ __forceinline__ void label_rows_t(const char* x, double scale, int64_t pitch, int H, int W, int r0,
                                             bool quads, const double2* sw, int M, int32_t* lab) {
  using Tile = LabelTile<Q, V, WR>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  r0 += Tile::ROWS * (wave % WR);
  if (r0 >= H) return;  // no barrier below
  const int lr = lane >> 3, lc = V * (lane & 7);
  const int rows = min(Tile::ROWS, H - r0);
  const rsrc_t xr = make_rsrc(x + (int64_t)r0 * pitch * (int64_t)sizeof(WT),
                              (uint32_t)((uint64_t)rows * (uint64_t)pitch * sizeof(WT)));
  auto fetch = [&](int c0, int q) {
    const int r = lr + 8 * q, v = c0 + lc;
    const uint32_t off = ((uint32_t)r * (uint32_t)pitch + (uint32_t)v) * (uint32_t)sizeof(WT);
    if constexpr (sizeof(WT) == 1 && V == 4) {
      if (quads) return unpack(buf_load<uint32_t>(xr, r < rows && v < W ? off : BUF_OOB, 0));  // v + 3 < pitch
    }
    Adjacent<WT, V> g;
#pragma unroll
    for (int i = 0; i < V; ++i)
      g.w[i] = buf_load<WT>(xr, r < rows && v + i < W ? off + (uint32_t)(i * sizeof(WT)) : BUF_OOB, 0);
    return g;
  };
  int c0 = Tile::COLS * (wave / WR);
  if (c0 >= W) return;
  // a NaN codevector 0 starts the full scan's comparisons with a NaN and so
  // wins every pixel there; other NaNs never win
  const bool nan0 = isnan(sw[0].x) || isnan(sw[0].y);
  Adjacent<WT, V> nx[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) nx[q] = fetch(c0, q);
  for (; c0 < W; c0 += Tile::STEP) {
    Adjacent<WT, V> cur[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) cur[q] = nx[q];
    if (c0 + Tile::STEP < W) {  // the next tile's weights, in flight while this one is labelled
#pragma unroll
      for (int q = 0; q < Q; ++q) nx[q] = fetch(c0 + Tile::STEP, q);
    }
    uint32_t fg = 0u;  // bit V q + i: pixel i of row q has a positive weight
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int i = 0; i < V; ++i)
        fg |= ((double)cur[q].w[i] * scale > 0.0 && c0 + lc + i < W ? 1u : 0u) << (V * q + i);
    // a scan that finds no distance below infinity ends at codevector 0
    double best[Q][V];
    int32_t best_k[Q][V];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int i = 0; i < V; ++i) {
        best[q][i] = __builtin_huge_val();
        best_k[q][i] = 0;
      }
    if (!nan0 && __any(fg != 0u)) {
      // box of the tile's pixel centres: centre and half extents (exact)
      const double hu = 0.5 * (double)(rows - 1), hv = 0.5 * (double)(min(c0 + Tile::COLS, W) - 1 - c0);
      const double mu = (double)r0 + hu, mv = (double)c0 + hv;
      const float fu = (float)hu, fv = (float)hv;
      // |w - centre| along each axis, in FP32
      auto dist = [&](int k, float& du, float& dv) {
        const double2 w = sw[k];
        du = (float)fabs(w.x - mu);
        dv = (float)fabs(w.y - mv);
        return w;
      };
      float ustar = __builtin_huge_valf();
      for (int k0 = 0; k0 < M; k0 += 64) {
        const int k = min(k0 + lane, M - 1);
        float du, dv;
        dist(k, du, dv);
        du = __builtin_fmaf(du, LB_ROUND, du) + fu;
        dv = __builtin_fmaf(dv, LB_ROUND, dv) + fv;
        ustar = fminf(ustar, __builtin_fmaf(du, du, dv * dv));  // a NaN codevector bounds nothing
      }
      ustar = -wave_max(-ustar);
      const float thr = ustar * LB_MARGIN;
      for (int k0 = 0; k0 < M; k0 += 64) {
        const int k = min(k0 + lane, M - 1);
        float du, dv;
        const double2 w = dist(k, du, dv);
        du = fmaxf(__builtin_fmaf(-du, LB_ROUND, du) - fu, 0.f);  // a NaN or infinite difference becomes 0
        dv = fmaxf(__builtin_fmaf(-dv, LB_ROUND, dv) - fv, 0.f);
        const bool keep = k0 + lane < M && !(isnan(w.x) || isnan(w.y)) && !(__builtin_fmaf(du, du, dv * dv) > thr);
        uint64_t m = __ballot(keep);
        while (m) {  // uniform
          const int l = __builtin_ctzll(m);
          m &= m - 1;
          const double wu = lane_value(w.x, l), wv = lane_value(w.y, l);
          const int kk = k0 + l;
          double sv[V];
#pragma unroll
          for (int i = 0; i < V; ++i) {
            const double d = (double)(c0 + lc + i) - wv;
            sv[i] = __dmul_rn(d, d);
          }
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const double d = (double)(r0 + lr + 8 * q) - wu, su = __dmul_rn(d, d);
#pragma unroll
            for (int i = 0; i < V; ++i) {
              const double t = __dadd_rn(su, sv[i]);
              const bool less = t < best[q][i];
              best[q][i] = less ? t : best[q][i];
              best_k[q][i] = less ? kk : best_k[q][i];
            }
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int i = 0; i < V; ++i) best_k[q][i] = fg >> (V * q + i) & 1u ? best_k[q][i] : -1;
    const int v = c0 + lc;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (lr + 8 * q >= rows) continue;
      int32_t* p = lab + (int64_t)(r0 + lr + 8 * q) * pitch + v;
      if constexpr (V == 4) {
        if (v + 3 < W) {
          __builtin_nontemporal_store(i32x4{best_k[q][0], best_k[q][1], best_k[q][2], best_k[q][3]},
                                      reinterpret_cast<i32x4*>(p));
          continue;
        }
      }
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (v + i < W) p[i] = best_k[q][i];
    }
  }
}

template <int Q, int V, int WR>
__device__ __forceinline__ void label_rows(const char* x, int wdtype, double scale, int64_t pitch, int H, int W, int r0,
                                           const double2* sw, int M, int32_t* lab) {
  if (wdtype == 0)
    label_rows_t<Q, V, WR, uint8_t>(x, scale, pitch, H, W, r0, ((uintptr_t)x % 4 == 0) && pitch % 4 == 0, sw, M, lab);
  else if (wdtype == 1)
    label_rows_t<Q, V, WR, float>(x, scale, pitch, H, W, r0, false, sw, M, lab);
  else
    label_rows_t<Q, V, WR, double>(x, scale, pitch, H, W, r0, false, sw, M, lab);
}

template <int Q, int V, typename T>
__global__ void __launch_bounds__(LB_NT) label_kernel(const char* x, int wdtype, double scale, int64_t pitch, int H,
                                                      int W, const T* w, int M, int32_t* lab) {
  extern __shared__ double2 sw[];
  stage_codebook(w, M, sw);
  __syncthreads();
  label_rows<Q, V, 1>(x, wdtype, scale, pitch, H, W, (int)blockIdx.x * LabelTile<Q, V, 1>::GROUP_ROWS, sw, M, lab);
}

// Where codevectors are dense, of the narrow images whose rows leave waves of a workgroup without a tile: tiles of
// 8 x 8, one pixel a lane, two rows of them. A tile's time is then its candidates' (a codevector for every 256
// pixels is two for each large tile, and its neighbours'), in proportion to the pixels a lane holds. us of large
// and small tiles: one 16 x 16 image, M = 1,000, 153 and 59 (two rows of tiles, of 8 x 32 pixels and a workgroup
// each, before either: 74); 1,500 of 40 x 40, M = 200, 231 and 132 (127); 1,500 of 100 x 100, M = 100, 205 and 129
// (195). Sparser, 1,500 of 40 x 40, M = 8, 20 and 24; wider, one 256 x 256 image, M = 200, 12 and 22.
inline __host__ __device__ bool label_dense(int H, int W, int M) {
  return M >= 24 && W <= 128 && (int64_t)H * W <= (int64_t)256 * M;
}

// Workgroups 2 b and 2 b + 1: the upper and the lower half of the 32-row band b.
__global__ void __launch_bounds__(LB_NT) label_batched_kernel(const ImageDesc* __restrict__ images,
                                                              const ChamferTask* __restrict__ bands, const char* x,
                                                              const float* w, int32_t* lab) {
  static_assert(LabelTile<2, 4, 1>::GROUP_ROWS == 16 && LabelTile<1, 1, 2>::GROUP_ROWS == 16, "half a band");
  extern __shared__ double2 sw[];
  const ChamferTask t = bands[blockIdx.x >> 1];
  const ImageDesc& im = images[t.img];
  const int r0 = t.pos + 16 * (int)(blockIdx.x & 1);
  if (r0 >= im.H) return;  // uniform
  stage_codebook(w + 2 * im.w_off, im.M, sw);
  __syncthreads();
  const int64_t esz = im.wdtype == 0 ? 1 : (im.wdtype == 1 ? 4 : 8);
  const char* xi = x + im.weight_off;
  int32_t* li = lab + im.weight_off / esz;
  if (label_dense(im.H, im.W, im.M))
    label_rows<1, 1, 2>(xi, im.wdtype, im.scale, im.pitch, im.H, im.W, r0, sw, im.M, li);
  else
    label_rows<2, 4, 1>(xi, im.wdtype, im.scale, im.pitch, im.H, im.W, r0, sw, im.M, li);
}

}  // namespace

int label_rows_per_band() { return 32; }

template <int Q, int V>
static void launch_label_t(bool f64, const ImageDesc& im, const void* x, const void* w, int M, int32_t* lab, hipStream_t s) {
  constexpr int ROWS = LabelTile<Q, V, 1>::GROUP_ROWS;
  const dim3 grid((im.H + ROWS - 1) / ROWS);
  const size_t smem = (size_t)M * sizeof(double2);
  if (f64)
    hipLaunchKernelGGL((label_kernel<Q, V, double>), grid, dim3(LB_NT), smem, s, (const char*)x, im.wdtype, im.scale,
                       im.pitch, im.H, im.W, (const double*)w, M, lab);
  else
    hipLaunchKernelGGL((label_kernel<Q, V, float>), grid, dim3(LB_NT), smem, s, (const char*)x, im.wdtype, im.scale,
                       im.pitch, im.H, im.W, (const float*)w, M, lab);
}

hipError_t launch_label(bool f64, const ImageDesc& im, const void* x, const void* w, int M, int32_t* lab,
                        hipStream_t s) {
  if (label_dense(im.H, im.W, M))
    launch_label_t<1, 1>(f64, im, x, w, M, lab, s);
  else
    launch_label_t<2, 4>(f64, im, x, w, M, lab, s);
  return hipGetLastError();
}

hipError_t launch_label_batched(const ImageDesc* d_images, const ChamferTask* d_bands, int nbands, int m_max,
                                const void* x, const void* w, int32_t* lab, hipStream_t s) {
  hipLaunchKernelGGL(label_batched_kernel, dim3(2 * nbands), dim3(LB_NT), (size_t)m_max * sizeof(double2), s, d_images,
                     d_bands, (const char*)x, (const float*)w, lab);
  return hipGetLastError();
}

}  // namespace itc
