// FP32 convolution maps (A, M_u, M_v and the FP64 partials of S_X, as in
// conv.hip) on the FP32 matrix cores, for what the split-FP16 kernel does not
// take: FP32 and FP64 weights, and 8-bit rows that are not 4-byte aligned.
//
// Each 1-D pass is a banded Toeplitz product: sixteen outputs along an axis are
// a 16 x K window of inputs times the K x 16 matrix T[k][n] = f(n + RA - k), RA the
// radius rounded up to 4, K = 16 + 2 RA, f zero past the true radius, evaluated
// with v_mfma_f32_16x16x4_f32: FP32 operands, products and sums, as in a direct
// FP32 sum (largest error against 64 bits over R = 1..24: 5.0e-7 of the largest
// map value, 5.3e-7 as vector FMAs). The matrix unit runs at twice the rate of
// unpacked vector FMAs, so the band's zeros (K = 40 terms instead of 25 at R = 12)
// still leave it ahead, and the vector unit only stages and addresses. At R <= 3 they
// do not (K = 24 terms for 5 or 7): the same segments with both passes as vector FMAs
// over the taps of the radius, four adjacent columns a lane. us at R = 2, matrix and
// vector form: 16 images of 1024 x 1023 bytes 46 and 43, 24 images 66
// and 57, 32 images 700 x 333 33 and 25, one 2048 x 2047 image 19.4 and 16.4; at R = 3
// 48 images 700 x 333 bytes 42 and 36, FP64 weights 2 to 4 % more in the vector form.
//
// Work decomposition: a workgroup of four waves owns a strip of 64 columns and a
// segment of rows (starting at a multiple of SX_ROWS) and streams down it in
// chunks of 16 rows. Per chunk:
//   1. staging: the chunk's 16 input rows with their column halo, fetched a chunk
//      earlier (16 bytes per lane and load where no group of four straddles the
//      width), scaled, into one of two LDS buffers; one barrier;
//   2. row pass: wave w makes columns 16w..16w+15 of R0 and R1 and writes them to
//      its ring, column-major (vector form: row-major); no other wave reads them;
//   3. column pass, 2 RA rows behind: ring columns are the A operand, so a lane
//      holds four adjacent columns of one output row: one 16-byte store per map,
//      a 16 x 16 tile of a panel is one contiguous KiB. h A goes into an FP64
//      partial of S_X per SX_ROWS-row group; h is loaded again (from L2).
// The k index of a product is permuted so that a lane's operands of four steps
// (two in the last group of eight) are consecutive in LDS: one 16-byte read.
// Pitches of 4 x odd words spread 16 lanes' reads over all banks.
//
// A zero tap times a non-finite value is not zero. Every output of a 16 x 16 tile
// sees every value of its window, so such a value (a weight that is not finite, an
// overflow) leaves none of the tile's A or M_v finite; a wave that finds one makes its
// columns of the S_X row groups concerned again from the window sums (rows_by_windows),
// so that the value reaches exactly the pixels within R of it. The test rides on the S_X
// sum: as eight multiply-adds per row pass and a vote of the workgroup it took
// 60 us of 280 (R = 4, below). One such weight, with and without: 64 images of 1024^2
// 0.29 and 0.28 ms at R = 12, 0.67 and 0.48 at R = 32; one image 0.06 and 0.013, 0.23
// and 0.026 (a sum over the whole window for each pixel of the segment: 10.3 at R = 32).
//
// Bound by memory (4 B read and 12 B written per pixel) up to R of about 8, then
// by the matrix unit. 64 x 1024^2 FP32 weights: R = 4 209 us (5.1 TB/s; 290 us
// with vector FMAs), R = 12 275 us (362), R = 24 380 us (600); one 1024^2
// image: 10.4 us (12.4), 12.4 us (16.4), 21 us (33). One to three chunks of
// loads in flight are the same; stores past the caches take 211 us at R = 4, as
// ordinary stores 242 (where all maps, up to 200 MB, fit the memory-side cache and are
// written again and again, ordinary stores of 4-byte words took 37 us for those 16
// images of 1024 x 1023 bytes).
#include <type_traits>
#include <utility>

#include "itc_device.h"

namespace itc {

namespace {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));

constexpr int CF_NT = 256, CF_CH = 16;
static_assert(SX_SLOTS == CF_NT / 64 && CONV_TW == 4 * MAP_PANEL, "one S_X slot and one panel per wave");
constexpr int CF_STREAM = 2;  // map stores are non-temporal

// A kernel: 2 and 3 are the vector form of that radius, the others the matrix form of that aligned radius.
constexpr int cf_kernel_of(int rclass) { return rclass < 4 ? rclass : (rclass + 3) / 4 * 4; }

template <int V>
struct CfGeom {
  static constexpr int RV = V < 4 ? V : 0, RA = V < 4 ? 4 : V;  // radius of the vector form (0: matrix), aligned radius
  static_assert(RA % 4 == 0 && RA >= 4 && RA <= 32, "aligned radius");
  static constexpr int K = 16 + 2 * RA, KS = K / 4;          // window, MFMA steps
  static constexpr int NG = K / 16, REM = K % 16;            // groups of 16, and 8 or none
  static constexpr int J0 = (2 * RA + CF_CH - 1) / CF_CH;  // chunks before the first column pass
  static constexpr int NB = J0 + 1;                          // ring blocks of 16 rows
  static constexpr int RINGP = NB * CF_CH + 4;               // ring column pitch
  static constexpr int SW = 48 + K;                          // staged columns (image columns v0 - RA + c)
  static constexpr int SWP = SW + 4;
  // a chunk, and a slot per spare item of the threads' equal shares of groups of four
  static constexpr int STAGE = CF_CH * SWP + 4 * ((4 * SW + CF_NT - 1) / CF_NT * CF_NT - 4 * SW);
  static constexpr int RING = CONV_TW * RINGP;
  static constexpr int VP = 20;                              // vector form: a wave's ring is [2][16 NB][VP], row-major
  static constexpr int MINE = RV ? 2 * NB * CF_CH * VP : 16 * RINGP;  // floats from one wave's part to the next
  static constexpr int PLANE = RV ? NB * CF_CH * VP : RING;           // from R0 to R1
  static_assert(!RV || MINE >= 2 * 16 * RINGP, "rows_by_windows fits a wave's part");
  // workgroups per compute unit that the registers are held to; LDS allows three to RA = 24 and two above, and one or
  // two more to RA = 16
  static constexpr int WGS = RV ? 4 : RA <= 24 ? 3 : 2;
  static constexpr size_t SMEM = (2 * (size_t)STAGE + (RV ? 4 * (size_t)MINE : 2 * (size_t)RING)) * sizeof(float);
  static_assert(RINGP / 4 % 2 == 1 && SWP / 4 % 2 == 1, "bank-spread pitches");
  static_assert(REM == 0 || REM == 8, "K is a multiple of eight");
};

__device__ __forceinline__ f4_t mfma(float a, float b, f4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Tap f(t) for the k of step st held by lane group q, f symmetric or odd.
template <int V>
__device__ __forceinline__ constexpr int k_of(int st, int q) {
  using G = CfGeom<V>;
  return st < 4 * G::NG ? 16 * (st / 4) + 4 * q + st % 4 : 16 * G::NG + 2 * q + (st - 4 * G::NG);
}

// A wave's 16 columns of the S_X row groups of [s0, seg_end) that see a value that is not finite (this wave's partials,
// written before, are not finite) from the window sums themselves: vector FMAs over the taps of the true radius only,
// through this wave's part of the ring like the passes of cf_segment. t = 0 has no tg term. Lane (n, q) makes
// rows 4q .. 4q + 3 of column n.
template <int V, typename WT>
__device__ __forceinline__ void rows_by_windows(const ImageDesc& im, int strip, int s0, int seg_end, const char* wbase,
                                                char* mbase, float* mine) {
  using G = CfGeom<V>;
  constexpr int RA = G::RA, PLANE = G::RV ? 16 * G::RINGP : G::RING;  // column-major in either form
  const int H = im.H, W = im.W, R = im.R;
  constexpr uint32_t esz = sizeof(WT);
  const uint32_t rowbytes = (uint32_t)im.pitch * esz;
  const rsrc_t wres = make_rsrc(wbase + im.weight_off, (uint32_t)H * rowbytes);
  float* maps = reinterpret_cast<float*>(mbase + im.map_off);
  const float scale = (float)im.scale;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, q = lane >> 4;
  const int v = strip * CONV_TW + 16 * wave + n;
  const double gl = exp(-0.5 / (im.sigma * im.sigma) * (double)(lane * lane));
  const float gT = (float)gl, tgT = (float)((double)lane * gl);  // the taps |t| = lane
  double* part = reinterpret_cast<double*>(mbase + im.map_off + im.part_off) + (int64_t)strip * im.nsxg * SX_SLOTS + wave;
  float* col = mine + n * G::RINGP;
  // the rows from the first such group to the last
  int r0 = seg_end, r1 = s0;
  for (int o = s0; o < seg_end; o += SX_ROWS) {
    const double tot = lane == 0 ? part[(int64_t)(o / SX_ROWS) * SX_SLOTS] : 0.0;  // as this lane wrote it
    if (__any(!(fabs(tot) < INFINITY))) {
      r0 = min(r0, o);
      r1 = min(o + SX_ROWS, seg_end);
    }
  }
  const int nout = (r1 - r0 + CF_CH - 1) / CF_CH;
  double sxd = 0.0;
  wave_lds_order();
#pragma unroll 1
  for (int j = 0; j < G::J0 + nout; ++j) {
    uint32_t off[4];
    f4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int y = r0 - RA + CF_CH * j + 4 * q + i;
      off[i] = y >= 0 && y < H ? (uint32_t)y * rowbytes : BUF_OOB;
    }
    constexpr int NT = 4;  // taps whose loads are in flight together; past R they read 0
#pragma unroll 1
    for (int t0 = -R; t0 <= R; t0 += NT) {  // uniform
      float h[NT][4];
#pragma unroll
      for (int e = 0; e < NT; ++e) {
        const int c = v - t0 - e;
        const bool in = t0 + e <= R && c >= 0 && c < W;
#pragma unroll
        for (int i = 0; i < 4; ++i) h[e][i] = (float)buf_load<WT>(wres, in ? off[i] + (uint32_t)c * esz : BUF_OOB, 0) * scale;
      }
#pragma unroll
      for (int e = 0; e < NT; ++e) {
        const int t = t0 + e, at = t < 0 ? -t : t;
        const float g = lane_value(gT, at), tg = t < 0 ? -lane_value(tgT, at) : lane_value(tgT, at);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s0[i] = fmaf(g, h[e][i], s0[i]);
          if (t) s1[i] = fmaf(tg, h[e][i], s1[i]);
        }
      }
    }
    float* rp = col + (j % G::NB) * CF_CH + 4 * q;
    *reinterpret_cast<f4_t*>(rp) = s0;
    *reinterpret_cast<f4_t*>(rp + PLANE) = s1;
    wave_lds_order();
    const int jo = j - G::J0;
    if (jo < 0) continue;
    float a[4] = {}, mu[4] = {}, mv[4] = {};
    int slot = (jo % G::NB) * CF_CH + 4 * q + RA - R;  // ring row of row 4q's t = R
    float y0[4] = {}, y1[4] = {};  // the rows of the four outputs at one t
    auto next = [&]() {
      const float* y = col + (slot < G::NB * CF_CH ? slot : slot - G::NB * CF_CH);
      ++slot;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        y0[i] = y0[i + 1];
        y1[i] = y1[i + 1];
      }
      y0[3] = y[0];
      y1[3] = y[PLANE];
    };
    next();
    next();
    next();
#pragma unroll 1
    for (int t = R; t >= -R; --t) {  // uniform
      next();
      const int at = t < 0 ? -t : t;
      const float g = lane_value(gT, at), tg = t < 0 ? -lane_value(tgT, at) : lane_value(tgT, at);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = fmaf(g, y0[i], a[i]);
        mv[i] = fmaf(g, y1[i], mv[i]);
        if (t) mu[i] = fmaf(tg, y0[i], mu[i]);
      }
    }
    const int o0 = r0 + CF_CH * jo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = o0 + 4 * q + i;
      if (o >= r1 || v >= im.npanels * MAP_PANEL) continue;
      const int64_t m = map_index(H, o, v);
      maps[m] = a[i];
      maps[im.plane + m] = mu[i];
      maps[2 * im.plane + m] = mv[i];
      if (v < W) sxd += (double)((float)buf_load<WT>(wres, (uint32_t)o * rowbytes + (uint32_t)v * esz, 0) * a[i]);
    }
    if ((jo + 1) % (SX_ROWS / CF_CH) == 0 || jo == nout - 1) {  // uniform
      const double tot = wave_sum(sxd);
      if (lane == 0) part[(int64_t)(o0 / SX_ROWS) * SX_SLOTS] = tot * im.scale;
      sxd = 0.0;
    }
  }
}

// VEC: FP32 weights, and no group of four columns of this strip straddles the width.
template <int V, typename WT, bool VEC>
__device__ __forceinline__ void cf_segment(const ImageDesc& im, int strip, int s0, int S,
                                           const char* __restrict__ wbase, char* __restrict__ mbase,
                                           float* __restrict__ smem) {
  using G = CfGeom<V>;
  constexpr int RA = G::RA;
  float* stage = smem;                   // [2][STAGE]
  float* ring = smem + 2 * G::STAGE;     // R0, R1: [2][64][RINGP], a column's rows together (vector form: see MINE)

  // lane-derived values are recomputed per segment: an opaque thread index
  // keeps the compiler from hoisting them out of the persistent tile loop
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, q = lane >> 4;
  const int H = im.H, W = im.W;
  const int v0 = strip * CONV_TW;
  const int seg_end = min(s0 + S, H);
  const int n_out = (seg_end - s0 + CF_CH - 1) / CF_CH;
  const int nchunks = G::J0 + n_out;
  const int origin = s0 - RA;  // image row of row 0 of chunk 0
  const int need_end = min(H, seg_end + RA);

  constexpr uint32_t esz = sizeof(WT);
  const uint32_t rowbytes = (uint32_t)im.pitch * esz;
  const rsrc_t wres = make_rsrc(wbase + im.weight_off, (uint32_t)H * rowbytes);
  const float scale = (float)im.scale;

  // ---- staging: thread item i of a chunk is columns v0 - RA + C d .. + C - 1 of row r ----
  // Columns left of the image or past the width, rows outside the image and items past the chunk load at an
  // offset past the end of the buffer, which reads 0 without a memory request. Single columns are dealt to
  // adjacent lanes (C = 1): 64 x 1024 x 1023 bytes at R = 2 took 216 us as four loads of a group of four.
  // FP64 weights stay as stored until they are staged, so that no conversion waits for a load.
  using One = std::conditional_t<sizeof(WT) == 8, WT, float>;
  using Unit = std::conditional_t<VEC, f4_t, One>;
  constexpr int C = VEC ? 4 : 1, PER = G::SW / C;             // columns per item, items per row
  constexpr int NI = (CF_CH * PER + CF_NT - 1) / CF_NT;       // items per thread and chunk
  static_assert(C * (NI * CF_NT - CF_CH * PER) <= G::STAGE - CF_CH * G::SWP, "a slot per spare item");
  int irow[NI], ioff[NI];
  uint32_t ibyte[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int idx = tid + CF_NT * i;
    const int r = idx / PER, d = idx - r * PER;
    const int x = v0 - RA + C * d;
    const bool item = idx < CF_CH * PER;
    irow[i] = item && x >= 0 && x < W ? r : -(1 << 30);  // never inside the image
    ibyte[i] = (uint32_t)x * esz;
    ioff[i] = item ? r * G::SWP + C * d : CF_CH * G::SWP + C * (idx - CF_CH * PER);
  }
  // stored weights of this lane's outputs: row o0 + n, columns c0 .. c0 + 3
  const int oc = v0 + 16 * wave + 4 * q;
  Unit pre[NI];
  std::conditional_t<VEC, f4_t, One[4]> hpre;
  auto fetch = [&](int j) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int y = origin + j * CF_CH + irow[i];
      const uint32_t off = y >= 0 && y < need_end ? (uint32_t)y * rowbytes + ibyte[i] : BUF_OOB;
      if constexpr (VEC)
        pre[i] = __builtin_bit_cast(f4_t, __builtin_amdgcn_raw_buffer_load_b128(wres, off, 0, 0));
      else
        pre[i] = (One)buf_load<WT>(wres, off, 0);
    }
    const int o = s0 + (j - G::J0) * CF_CH + n;
    const uint32_t off = o >= s0 && o < seg_end && oc < W ? (uint32_t)o * rowbytes + (uint32_t)oc * esz : BUF_OOB;
    if constexpr (VEC) {
      hpre = __builtin_bit_cast(f4_t, __builtin_amdgcn_raw_buffer_load_b128(wres, off, 0, 0));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        hpre[e] = (One)buf_load<WT>(wres, oc + e < W && off < BUF_OOB ? off + (uint32_t)e * esz : BUF_OOB, 0);
    }
  };

  // ---- outputs: wave w writes panel 4 strip + w, a 16 x 16 tile per chunk ----
  const int panel = 4 * strip + wave;
  const bool pan_ok = panel < im.npanels;  // the strip's last panels may lie past the width
  const uint32_t planeb = (uint32_t)(im.plane * (int64_t)sizeof(float));
  const char* mimg = mbase + im.map_off;
  const rsrc_t resA = make_rsrc(mimg, planeb), resU = make_rsrc(mimg + planeb, planeb),
               resV = make_rsrc(mimg + 2 * (size_t)planeb, planeb);
  const uint32_t pan_base = (uint32_t)panel * (uint32_t)H * 64u + 16u * (uint32_t)q;
  double* part = reinterpret_cast<double*>(mbase + im.map_off + im.part_off) +
                 ((int64_t)strip * im.nsxg) * SX_SLOTS + wave;
  float* mine = ring + wave * G::MINE;
  float* ring_col = mine + n * G::RINGP;
  double sxd = 0.0;   // this lane's share of the current S_X row group
  bool odd = false;   // a map value of this wave is not finite

  // the three stores of a column pass, dropped: keeps the sequence of pending memory operations the same
  // in the prologue and the warm-up chunks, so that the compiler's waits for a chunk's loads leave the
  // stores after them pending
  auto pad_stores = [&]() {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int d = 0; d < 3; ++d) __builtin_amdgcn_raw_buffer_store_b32(0u, resA, BUF_OOB + 16u * d, 0, 0);
    asm volatile("" ::: "memory");
  };

  fetch(0);
  pad_stores();

  // ---- taps: step st of lane (n, q) holds f(t), t = n + RA - k; vector form: f(0 .. RV), uniform ----
  constexpr int NT = G::RV ? G::RV + 1 : G::KS;
  float g[NT], tg[NT];
  {
    const double k2 = -0.5 / (im.sigma * im.sigma);
    const double gl = lane <= im.R ? exp(k2 * (double)(lane * lane)) : 0.0;
    const float gT = (float)gl, tgT = (float)((double)lane * gl);
#pragma unroll
    for (int st = 0; st < NT; ++st) {
      if constexpr (G::RV) {
        g[st] = lane_value(gT, st);
        tg[st] = lane_value(tgT, st);
      } else {
        const int t = n + RA - k_of<V>(st, q), at = t < 0 ? -t : t;  // |t| <= 15 + RA < 64
        const float a = __shfl(gT, at), b = __shfl(tgT, at);
        g[st] = a;
        tg[st] = t < 0 ? -b : b;
      }
    }
  }

  auto chunk = [&](int j, auto B) {
    float* xs = stage + decltype(B)::value * G::STAGE;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if constexpr (VEC)
        *reinterpret_cast<f4_t*>(xs + ioff[i]) = pre[i] * scale;
      else
        xs[ioff[i]] = (float)pre[i] * scale;
    }
    f4_t h;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = (float)hpre[e];
    __syncthreads();
    fetch(j + 1);  // past the last chunk: rows outside the segment, zeros

    // ---------------- row pass: chunk j -> ring block j mod NB ----------------
    if constexpr (G::RV) {  // lane (n, q): columns 4q .. 4q + 3 of row n
      const float* xr = xs + n * G::SWP + 16 * wave + 4 * q;
      float x[4 + 2 * RA];
#pragma unroll
      for (int e = 0; e < 1 + RA / 2; ++e) *reinterpret_cast<f4_t*>(x + 4 * e) = *reinterpret_cast<const f4_t*>(xr + 4 * e);
      f4_t r0, r1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        r0[i] = g[0] * x[i + RA];
        r1[i] = 0.f;
#pragma unroll
        for (int t = 1; t <= G::RV; ++t) {
          r0[i] = fmaf(g[t], x[i + RA - t], fmaf(g[t], x[i + RA + t], r0[i]));
          r1[i] = fmaf(tg[t], x[i + RA - t], fmaf(-tg[t], x[i + RA + t], r1[i]));
        }
      }
      float* rp = mine + (CF_CH * (j % G::NB) + n) * G::VP + 4 * q;
      *reinterpret_cast<f4_t*>(rp) = r0;
      *reinterpret_cast<f4_t*>(rp + G::PLANE) = r1;
    } else {
      const float* xr = xs + n * G::SWP + 16 * wave;
      f4_t r0 = {0.f, 0.f, 0.f, 0.f}, r1 = r0;
#pragma unroll
      for (int s = 0; s < G::NG; ++s) {
        const f4_t a = *reinterpret_cast<const f4_t*>(xr + 16 * s + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          r0 = mfma(a[e], g[4 * s + e], r0);
          r1 = mfma(a[e], tg[4 * s + e], r1);
        }
      }
      if constexpr (G::REM) {
        const f2_t a = *reinterpret_cast<const f2_t*>(xr + 16 * G::NG + 2 * q);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          r0 = mfma(a[e], g[4 * G::NG + e], r0);
          r1 = mfma(a[e], tg[4 * G::NG + e], r1);
        }
      }
      float* rp = ring_col + (j % G::NB) * CF_CH + 4 * q;
      *reinterpret_cast<f4_t*>(rp) = r0;
      *reinterpret_cast<f4_t*>(rp + G::PLANE) = r1;
    }
    // the column pass reads ring rows this wave has just written: keep the
    // compiler from moving LDS accesses across (the hardware keeps their order)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    const int jo = j - G::J0;
    if (jo < 0) {  // uniform: warm-up
      pad_stores();
      return;
    }

    // ---------------- column pass: output rows o0..o0+15 ----------------
    const int o0 = s0 + jo * CF_CH;
    f4_t am = {0.f, 0.f, 0.f, 0.f}, um = am, vm = am;
    if constexpr (G::RV) {
      // row o0 + n + t is ring row 16 jo + RA + n + t of the 16 NB
#pragma unroll
      for (int t = -G::RV; t <= G::RV; ++t) {
        const float* rp = mine + ((CF_CH * jo + RA + n + t) & (CF_CH * G::NB - 1)) * G::VP + 4 * q;
        const f4_t y0 = *reinterpret_cast<const f4_t*>(rp), y1 = *reinterpret_cast<const f4_t*>(rp + G::PLANE);
        const float gt = g[t < 0 ? -t : t], tgt = t < 0 ? tg[-t] : -tg[t];  // f(x_out - x_in)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          am[i] = fmaf(gt, y0[i], am[i]);
          if (t) um[i] = fmaf(tgt, y0[i], um[i]);
          vm[i] = fmaf(gt, y1[i], vm[i]);
        }
      }
    } else {
#pragma unroll
      for (int s = 0; s < G::NG; ++s) {
        const float* rp = ring_col + (jo + s) % G::NB * CF_CH + 4 * q;
        const f4_t y0 = *reinterpret_cast<const f4_t*>(rp), y1 = *reinterpret_cast<const f4_t*>(rp + G::PLANE);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          am = mfma(y0[e], g[4 * s + e], am);
          um = mfma(y0[e], tg[4 * s + e], um);
          vm = mfma(y1[e], g[4 * s + e], vm);
        }
      }
      if constexpr (G::REM) {
        const float* rp = ring_col + (jo + G::NG) % G::NB * CF_CH + 2 * q;
        const f2_t y0 = *reinterpret_cast<const f2_t*>(rp), y1 = *reinterpret_cast<const f2_t*>(rp + G::PLANE);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          am = mfma(y0[e], g[4 * G::NG + e], am);
          um = mfma(y0[e], tg[4 * G::NG + e], um);
          vm = mfma(y1[e], g[4 * G::NG + e], vm);
        }
      }
    }
    // lane (n, q) holds row o0 + n, columns 16 wave + 4q + i
    const int row = o0 + n;
    const bool ok = row < seg_end;
    const uint32_t off = ok && pan_ok ? pan_base + (uint32_t)row * 64u : BUF_OOB;
    float sx = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) sx = fmaf(h[i], am[i], sx);  // h is 0 past the width and the segment
    sx = fmaf(0.f, (vm[0] + vm[1]) + (vm[2] + vm[3]), sx);   // not a number if a map value is none or infinite
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4_t, am), resA, off, 0, CF_STREAM);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4_t, um), resU, off, 0, CF_STREAM);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4_t, vm), resV, off, 0, CF_STREAM);
    sxd += ok ? (double)sx : 0.0;
    // the last chunk of an S_X row group (or of the segment): one FP64 partial per wave
    if ((jo + 1) % (SX_ROWS / CF_CH) == 0 || jo == n_out - 1) {  // uniform
      const double tot = wave_sum(sxd);
      if (lane == 0) part[(int64_t)(o0 / SX_ROWS) * SX_SLOTS] = tot * im.scale;
      odd |= !(fabs(tot) < INFINITY);
      sxd = 0.0;
    }
  };

  int j = 0;
  for (; j + 2 <= nchunks; j += 2) {
    chunk(j, std::integral_constant<int, 0>{});
    chunk(j + 1, std::integral_constant<int, 1>{});
  }
  if (j < nchunks) chunk(j, std::integral_constant<int, 0>{});
  if (__builtin_amdgcn_readfirstlane(odd)) rows_by_windows<V, WT>(im, strip, s0, seg_end, wbase, mbase, mine);
}

// One segment for the image's stored weight type (one uniform branch per segment).
template <int V>
__device__ __forceinline__ void cf_segment_any(const ImageDesc& im, int strip, int s0, int S, const char* wbase,
                                               char* mbase, float* smem) {
  if (im.wdtype == 1) {
    if (im.W % 4 == 0 || strip * CONV_TW + CONV_TW + CfGeom<V>::RA <= im.W)
      cf_segment<V, float, true>(im, strip, s0, S, wbase, mbase, smem);
    else
      cf_segment<V, float, false>(im, strip, s0, S, wbase, mbase, smem);
  } else if (im.wdtype == 0) {
    cf_segment<V, uint8_t, false>(im, strip, s0, S, wbase, mbase, smem);
  } else {
    cf_segment<V, double, false>(im, strip, s0, S, wbase, mbase, smem);
  }
}

template <int V>
__global__ void __launch_bounds__(CF_NT, CfGeom<V>::WGS) conv_f32_image_kernel(ImageDesc im, int S, const char* wbase, char* mbase) {
  __shared__ __align__(16) float smem[CfGeom<V>::SMEM / sizeof(float)];
  const int strip = blockIdx.x % im.nstrips;
  const int seg = blockIdx.x / im.nstrips;
  cf_segment_any<V>(im, strip, seg * S, S, wbase, mbase, smem);
}

// Persistent launch over the tiles of one radius class: workgroup b walks the
// sublist of its XCD, b mod CONV_XCDS.
template <int V>
__global__ void __launch_bounds__(CF_NT, CfGeom<V>::WGS) conv_f32_tiles_kernel(const ImageDesc* __restrict__ images,
                                                               const ConvTile* __restrict__ tiles, XcdSplit xs,
                                                               const char* wbase, char* mbase) {
  __shared__ __align__(16) float smem[CfGeom<V>::SMEM / sizeof(float)];
  const int x = blockIdx.x % CONV_XCDS, nx = gridDim.x / CONV_XCDS;
  const int end = xs.beg[x + 1];
  for (int i = xs.beg[x] + (int)blockIdx.x / CONV_XCDS; i < end; i += nx) {
    const ConvTile t = tiles[i];
    const ImageDesc im = images[t.img];
    cf_segment_any<V>(im, t.strip, t.s0, t.S, wbase, mbase, smem);
    __syncthreads();  // the next tile restages the shared memory
  }
}

}  // namespace

#define ITC_FOR_CF(X) X(2) X(3) X(4) X(8) X(12) X(16) X(20) X(24) X(28) X(32)

hipError_t launch_conv_f32_image(const ImageDesc& im, const void* w, void* m, hipStream_t s) {
  const int S = conv_segment_rows(im);
  const dim3 grid(im.nstrips * ((im.H + S - 1) / S));
#define ITC_CASE(V)                                                                                 \
  case V:                                                                                           \
    hipLaunchKernelGGL((conv_f32_image_kernel<V>), grid, dim3(CF_NT), 0, s, im, S, (const char*)w, \
                       (char*)m);                                                                   \
    return hipGetLastError();
  switch (cf_kernel_of(im.rclass)) { ITC_FOR_CF(ITC_CASE) default: return hipErrorInvalidValue; }
#undef ITC_CASE
}

hipError_t launch_conv_f32_tiles(int rclass, const ImageDesc* d_images, const ConvTile* d_tiles, const XcdSplit& xs,
                                 const void* w, void* m, int grid, hipStream_t s) {
  if (grid % CONV_XCDS != 0) return hipErrorInvalidValue;
#define ITC_CASE(V)                                                                                    \
  case V:                                                                                              \
    hipLaunchKernelGGL((conv_f32_tiles_kernel<V>), dim3(grid), dim3(CF_NT), 0, s, d_images, d_tiles,  \
                       xs, (const char*)w, (char*)m);                                                  \
    return hipGetLastError();
  switch (cf_kernel_of(rclass)) { ITC_FOR_CF(ITC_CASE) default: return hipErrorInvalidValue; }
#undef ITC_CASE
}

int conv_f32_blocks_per_cu(int rclass) {
  int nb = 0;
  hipError_t e = hipErrorInvalidValue;
#define ITC_CASE(V)                                                                             \
  case V:                                                                                       \
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, conv_f32_tiles_kernel<V>, CF_NT, 0); \
    break;
  switch (cf_kernel_of(rclass)) { ITC_FOR_CF(ITC_CASE) default: break; }
#undef ITC_CASE
  return e == hipSuccess ? nb : 0;
}

}  // namespace itc
