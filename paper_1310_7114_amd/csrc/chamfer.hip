// Chamfer distance transform T(X) of a binary lattice image (Section 5: the
// foreground pixels are weighted by a distance transform so that interior
// pixels count more, P = T(X) * G_xi; the paper names Borgefors' chamfer
// transforms). T(p) is the least cost of a path from p to the background on
// the 8-connected lattice, orthogonal steps costing a and diagonal steps b;
// everything outside the H x W lattice is background. Borgefors computes it
// with two sequential raster passes. Here the same values come from two
// data-parallel passes over the whole image, or, where every cost fits 16 bits
// and the image has at most 1,024 rows and 2,048 columns, from bands of rows
// (second half of this file). The two passes rest on:
//
// * For 1 <= a <= b <= 2a the least path cost to a pixel q is
//     phi(|du|, |dv|) = a max(|du|, |dv|) + (b - a) min(|du|, |dv|)
//   (diagonal steps for the shorter extent, orthogonal for the rest), so
//   T(i, j) = min over background q of phi(|i - q_u|, |j - q_v|).
// * phi is non-decreasing in |du| for a fixed |dv|, so the best background
//   pixel of column l is the one nearest to row i in that column:
//     T(i, j) = min over l of phi(|j - l|, g(i, l)),
//   g(i, l) = rows from (i, l) to the nearest background pixel of column l
//   (rows -1 and H and columns -1 and W are background).
//
// Pass 1 (columns): a workgroup of four waves takes a strip of 64 columns,
// one lane per column. Columns of up to 1,024 rows are packed into a bit mask
// in LDS (the waves share the rows), then for every word the first background
// row at or after it and the last at or before it are found, and the four
// waves walk their quarters of the rows writing g. So the image is read once
// and g written once, as 16-bit integers at the start of each row of the
// output (the FP32 row has room for two). Pass 2 (rows): a workgroup stages
// one row of g in LDS and every thread searches outward from its column on
// both sides at once, stopping once a |j - l| reaches the best cost found
// (phi >= a |j - l|). The row of g is in LDS before any T of the row is
// written over it; T values are exact integers, stored as FP32 so that T can
// feed the convolution as a weight image. When every cost fits 16 bits the
// two sides of the search share packed 16-bit registers (one multiply-add per
// term for both), three steps per trip with their LDS reads issued together
// (2.92 -> 2.51 ms for the batch of 1,400 silhouettes; one step per trip 2.78,
// two 2.57, four 3.09: the steps past the stop grow with the trip).
#include <type_traits>

#include "itc_device.h"

namespace itc {

namespace {

constexpr int CH_ROWS_NT = 256;
constexpr int CH_ROWS_PER_TASK = 8;
constexpr int CH_COLS_NT = 256;  // four waves share one strip of 64 columns
constexpr int CH_COLS_WAVES = CH_COLS_NT / 64;
constexpr int CH_WORDS = 32;     // columns of up to 32 CH_WORDS rows take the bit-mask pass
constexpr int CH_GUARD = 4;      // zero columns on each side of the row of g in LDS
#ifndef ITC_CH_STEP
#define ITC_CH_STEP 3
#endif
constexpr int CH_STEP = ITC_CH_STEP;  // search steps per trip of the packed row search
static_assert(CH_STEP >= 1 && CH_STEP <= CH_GUARD, "the steps past the stop stay within the guards");

// Every cost of the row search fits 16 bits: a g + c r and c g + a r with
// g <= H and r <= W + CH_GUARD (the guard columns), and the least found so
// far below a (W + 1).
__device__ __forceinline__ bool chamfer_packed(int H, int W, int a, int b) {
  return (int64_t)(a + b) * (int64_t)(H + W + 2 * CH_GUARD) < 65536;
}

// g of row i (16-bit, at the start of row i of the output)
__device__ __forceinline__ uint16_t* g_row(float* t, int64_t pitch, int i) {
  return reinterpret_cast<uint16_t*>(t + (int64_t)i * pitch);
}

// Pass 1, two walks down and up the column (columns taller than the bit-mask
// pass takes), by the first wave: lane = column.
__device__ __forceinline__ void chamfer_cols_walk(const uint8_t* __restrict__ x, int64_t pitch,
                                                  float* __restrict__ t, int H, int W, int v0) {
  const int j = v0 + (int)(threadIdx.x & 63);
  if (threadIdx.x >= 64 || j >= W) return;
  const uint8_t* xc = x + j;
  int run = 0;  // rows to the nearest background pixel above (row -1 is background)
#pragma unroll 8
  for (int i = 0; i < H; ++i) {
    run = xc[(int64_t)i * pitch] ? run + 1 : 0;
    g_row(t, pitch, i)[j] = (uint16_t)run;
  }
  run = 0;  // and below (row H is background)
#pragma unroll 8
  for (int i = H - 1; i >= 0; --i) {
    run = xc[(int64_t)i * pitch] ? run + 1 : 0;
    uint16_t* gp = g_row(t, pitch, i) + j;
    const int up = *gp;
    *gp = (uint16_t)(up < run ? up : run);
  }
}

// Pass 1 with the bit mask: bit k of word w is row 32 w + k (rows >= H and
// columns >= W are background). LDS: sbits, snext (first background row at or
// after word w, H if none), slast (last background row at or before the end
// of word w, -1 if none), each [CH_WORDS][64].
__device__ __forceinline__ void chamfer_cols_bits(const uint8_t* __restrict__ x, int64_t pitch,
                                                  float* __restrict__ t, int H, int W, int v0,
                                                  uint32_t* __restrict__ sbits, int32_t* __restrict__ snext,
                                                  int32_t* __restrict__ slast) {
  const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
  const int j = v0 + lane;
  const bool col = j < W;
  // byte offsets below 2^31 (the image is smaller than 2 GiB)
  const rsrc_t xr = make_rsrc(x, (uint32_t)((int64_t)H * pitch));
  const int nw = (H + 31) / 32;
  // a word's 32 loads are issued together: rows past the image and columns
  // past the width load at an offset with bit 31 set (beyond the buffer),
  // which reads 0, so no branch makes the compiler wait for each load
  const uint32_t cbad = (uint32_t)!col << 31;
  for (int w = wave; w < nw; w += CH_COLS_WAVES) {
    uint32_t v[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const int i = 32 * w + k;
      const uint32_t rbad = (uint32_t)(i >= H) << 31;  // uniform
      v[k] = buf_load<uint8_t>(xr, ((uint32_t)i * (uint32_t)pitch + (uint32_t)j) | rbad | cbad, 0);
    }
    uint32_t m = 0u;
#pragma unroll
    for (int k = 0; k < 32; ++k) m |= (v[k] != 0u ? 1u : 0u) << k;
    sbits[w * 64 + lane] = m;
  }
  __syncthreads();
  if (wave == 0) {
    int nxt = H;  // row H is background
    for (int w = nw - 1; w >= 0; --w) {
      const uint32_t inv = ~sbits[w * 64 + lane];
      if (inv) nxt = 32 * w + __builtin_ctz(inv);
      snext[w * 64 + lane] = nxt;
    }
  } else if (wave == 1) {
    int lst = -1;  // row -1 is background
    for (int w = 0; w < nw; ++w) {
      const uint32_t inv = ~sbits[w * 64 + lane];
      if (inv) lst = 32 * w + 31 - __builtin_clz(inv);
      slast[w * 64 + lane] = lst;
    }
  }
  __syncthreads();
  const int w0 = nw * wave / CH_COLS_WAVES, w1 = nw * (wave + 1) / CH_COLS_WAVES;
  if (col) {
    int last = w0 > 0 ? slast[(w0 - 1) * 64 + lane] : -1;
    for (int w = w0; w < w1; ++w) {
      const uint32_t m = sbits[w * 64 + lane];
      const int after = w + 1 < nw ? snext[(w + 1) * 64 + lane] : H;
      const int kn = min(32, H - 32 * w);
      for (int k = 0; k < kn; ++k) {
        const int i = 32 * w + k;
        const uint32_t inv = ~m >> k;  // background rows at or after i within the word
        const int down = inv ? i + __builtin_ctz(inv) : after;
        const int g = min(i - last, down - i);  // 0 on a background row (down == i)
        last = (m >> k) & 1u ? last : i;
        g_row(t, pitch, i)[j] = (uint16_t)g;
      }
    }
  }
  __syncthreads();  // LDS is reused by the next strip
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));

// Least cost over a row of g (LDS, CH_GUARD zeros on each side) from column j,
// both sides in the halves of packed 16-bit registers.
__device__ __forceinline__ int row_search(const uint16_t* __restrict__ gs, int j, int W, int a, int c) {
  const u16x2 A2 = {(uint16_t)a, (uint16_t)a}, C2 = {(uint16_t)c, (uint16_t)c};
  const int b0 = a * min(min(j + 1, W - j), (int)gs[j]);
  u16x2 best = {(uint16_t)b0, (uint16_t)b0};  // least cost found left and right of j
  u16x2 ar = A2, cr = C2;                      // a r and c r at the next r
  int lim = b0;
  // CH_STEP steps per trip, their reads issued together; the steps past
  // the stop cost at least a r >= lim and change nothing, and their reads
  // stay within the guards (r < min(j + 1, W - j) + CH_STEP)
  for (int r = 1; a * r < lim; r += CH_STEP) {
    u16x2 g2[CH_STEP];
#pragma unroll
    for (int q = 0; q < CH_STEP; ++q) g2[q] = u16x2{gs[j - r - q], gs[j + r + q]};
#pragma unroll
    for (int q = 0; q < CH_STEP; ++q) {
      // phi(r, g) = max(a g + c r, c g + a r) on both sides
      best = __builtin_elementwise_min(best, __builtin_elementwise_max(A2 * g2[q] + cr, C2 * g2[q] + ar));
      ar += A2;
      cr += C2;
    }
    lim = min((int)best.x, (int)best.y);
  }
  return min((int)best.x, (int)best.y);
}

// Pass 2 for rows r0 .. r0 + n - 1, in place; gs: one row of g (LDS). With
// packed set ((a + b)(H + W) < 2^16, so every cost below fits 16 bits) the
// two sides of the search run in the two halves of packed 16-bit registers:
// one multiply-add per term for both sides.
__device__ __forceinline__ void chamfer_rows(float* __restrict__ t, int64_t pitch, int W, int r0, int n, int a,
                                             int b, bool packed, uint16_t* __restrict__ gs) {
  const int c = b - a;
  for (int i = r0; i < r0 + n; ++i) {
    float* tr = t + (int64_t)i * pitch;
    const uint16_t* gr = g_row(t, pitch, i);
    // gs[-CH_GUARD .. -1] and gs[W .. W + CH_GUARD - 1] hold 0: columns
    // outside the image are background
    for (int j = threadIdx.x - CH_GUARD; j < W + CH_GUARD; j += blockDim.x)
      gs[j] = j >= 0 && j < W ? gr[j] : (uint16_t)0;
    __syncthreads();
    if (packed) {  // uniform
      for (int j = threadIdx.x; j < W; j += blockDim.x) tr[j] = (float)row_search(gs, j, W, a, c);
      __syncthreads();
      continue;
    }
    for (int j = threadIdx.x; j < W; j += blockDim.x) {
      // columns -1 and W are background, and this column: best <= a (j + 1), a (W - j),
      // so the search below stays inside 0 .. W - 1
      int best = a * min(min(j + 1, W - j), (int)gs[j]);
      for (int r = 1; a * r < best; ++r) {
        // phi(d, g) = a max(d, g) + (b - a) min(d, g) = max(a g + c d, a d + c g)
        const int ar = a * r, cr = c * r;
        const int gl = gs[j - r], gh = gs[j + r];
        best = min(best, max(a * gl + cr, c * gl + ar));
        best = min(best, max(a * gh + cr, c * gh + ar));
      }
      tr[j] = (float)best;
    }
    __syncthreads();
  }
}

__device__ __forceinline__ void cols_task(const uint8_t* x, int64_t pitch, float* t, int H, int W, int v0,
                                          uint32_t* sbits, int32_t* snext, int32_t* slast) {
  if (H <= 32 * CH_WORDS)
    chamfer_cols_bits(x, pitch, t, H, W, v0, sbits, snext, slast);
  else
    chamfer_cols_walk(x, pitch, t, H, W, v0);
}

__global__ void __launch_bounds__(CH_COLS_NT) chamfer_cols_kernel(const uint8_t* x, int64_t pitch, float* t, int H,
                                                                  int W) {
  __shared__ uint32_t sbits[CH_WORDS * 64];
  __shared__ int32_t snext[CH_WORDS * 64];
  __shared__ int32_t slast[CH_WORDS * 64];
  cols_task(x, pitch, t, H, W, blockIdx.x * 64, sbits, snext, slast);
}

__global__ void __launch_bounds__(CH_ROWS_NT) chamfer_rows_kernel(float* t, int64_t pitch, int H, int W, int a,
                                                                  int b) {
  extern __shared__ uint16_t gsh[];
  const int r0 = blockIdx.x * CH_ROWS_PER_TASK;
  uint16_t* gs = gsh + CH_GUARD;
  chamfer_rows(t, pitch, W, r0, min(CH_ROWS_PER_TASK, H - r0), a, b, chamfer_packed(H, W, a, b), gs);
}

__global__ void __launch_bounds__(CH_COLS_NT) chamfer_cols_batched_kernel(const ImageDesc* __restrict__ images,
                                                                          const ChamferTask* __restrict__ tasks,
                                                                          int ntasks, const uint8_t* x, float* t) {
  __shared__ uint32_t sbits[CH_WORDS * 64];
  __shared__ int32_t snext[CH_WORDS * 64];
  __shared__ int32_t slast[CH_WORDS * 64];
  for (int k = blockIdx.x; k < ntasks; k += gridDim.x) {
    const ChamferTask c = tasks[k];
    const ImageDesc im = images[c.img];
    cols_task(x + im.weight_off, im.pitch, t + im.weight_off, im.H, im.W, c.pos * 64, sbits, snext, slast);
  }
}

__global__ void __launch_bounds__(CH_ROWS_NT) chamfer_rows_batched_kernel(const ImageDesc* __restrict__ images,
                                                                          const ChamferTask* __restrict__ tasks,
                                                                          int ntasks, float* t, int a, int b) {
  extern __shared__ uint16_t gsh[];
  uint16_t* gs = gsh + CH_GUARD;
  for (int k = blockIdx.x; k < ntasks; k += gridDim.x) {
    const ChamferTask c = tasks[k];
    const ImageDesc im = images[c.img];
    chamfer_rows(t + im.weight_off, im.pitch, im.W, c.pos, min(CH_ROWS_PER_TASK, im.H - c.pos), a, b,
                 chamfer_packed(im.H, im.W, a, b), gs);
  }
}

// ---------------------------------------------------------------------------
// Band form (costs in 16 bits, at most 32 CH_WORDS rows and CHB_MAX_W columns).
//
// With E = a min(g, h), g and h the distances to the nearest background pixel
// of the same column and of the same row,
//   T(p) = min over the four diagonal directions f, m >= 0 of b m + E(p + m f):
// a least path to the background is its min(|du|, |dv|) diagonal steps followed
// by straight ones, and every candidate is a path. So T is two min-plus scans of
// slope b along the diagonals, at a fixed cost per pixel, where the row search
// costs T / a steps. The image is cut into bands of 32 rows that need nothing of
// each other: of the rows outside, a band sees g (every straight vertical path)
// and the exact T of the seam rows 32, 64, .. (every path that crosses a seam on
// a diagonal step: T(p) = b m + T(p + m f) there). Three kernels:
//   * edges: bit masks of whole columns give, at every seam row, the distances
//     up and down the column to the background, and stay in the output's row
//     below each seam, one word per column, for the bands;
//   * seams: T of the seam rows by the row search of the other form (1 / 32 of
//     its work), kept as T | up in the seam's row of the output and T | down in
//     the row above it, which the bands of those rows own;
//   * bands: one workgroup per band reads its rows' bit words (a single band or a
//     single row: the image), E goes to LDS as 16-bit integers, and one thread per diagonal scans its 33 entries
//     both ways in registers, first along one diagonal in place, then along the
//     other out to T. (The second scan starts from the first one's result: a
//     path with steps along both diagonals is a path too.) Outside the lattice E
//     is 0. The row stride of E is an odd number of words, so that 32 lanes on
//     32 rows meet 32 banks.
// Strips of 64 columns without foreground in a band skip the bit words and the
// scans, and are filled with zeros only where a neighbour's scan reads them.
// Traffic: the image and T once and 3/32 words per pixel of edges, 5.4 B/px.
// Measured on 1,400 silhouettes (355 Mpx, 23 % of the strips with foreground):
// 0.58 ms (edges 0.12, seams 0.07, bands 0.39) against 2.42 ms of the column and
// row passes (0.34 + 2.10). T goes out in non-temporal 16-byte stores: ordinary
// ones cost the bands 0.09 ms and the next call's edges, whose reads evict
// them, 0.04; written along the second scan's diagonals they cost 0.02.
// ---------------------------------------------------------------------------
constexpr int CHB_ROWS = 32;
constexpr int CHB_NT = 512;
constexpr int CHB_WAVES = CHB_NT / 64;
constexpr int CHB_MAX_W = 2048;

// Row stride of E in 16-bit entries for images up to PW columns: 32 guard
// columns on each side (a diagonal leaves the band's columns by at most 32).
constexpr int chb_stride(int PW) { return PW + 2 * CHB_ROWS + 2; }
constexpr size_t chb_smem(int PW) {
  const size_t e = ((size_t)(CHB_ROWS + 1) * chb_stride(PW) * sizeof(uint16_t) + 7) / 8 * 8;
  return e + (size_t)CHB_ROWS * (PW / 32 + 1) * sizeof(uint32_t) + (size_t)CHB_ROWS * sizeof(uint64_t) +
         sizeof(uint32_t);
}

// Every image of a launch takes the band form.
inline bool chb_fits(int h_max, int w_max, int a, int b) {
  return h_max <= 32 * CH_WORDS && w_max <= CHB_MAX_W &&
         (int64_t)(a + b) * (int64_t)(h_max + w_max + 2 * CH_GUARD) < 65536;
}

__device__ __forceinline__ uint32_t* t_word(float* t, int64_t pitch, int i) {
  return reinterpret_cast<uint32_t*>(t + (int64_t)i * pitch);
}

// Bytes of the n <= 32 rows from row i0 of one column (columns past the image
// read 0, rows past the n are those of the last row: the callers mask them). The
// row is in the scalar offset, so a load takes no vector instruction of its own.
__device__ __forceinline__ void load_rows(rsrc_t xr, int64_t pitch, int i0, int n, int j, bool col, uint32_t (&v)[32]) {
  const uint32_t off = (uint32_t)j | (uint32_t)!col << 31;
#pragma unroll
  for (int k = 0; k < 32; ++k) v[k] = buf_load<uint8_t>(xr, off, (uint32_t)(i0 + min(k, n - 1)) * (uint32_t)pitch);
}

// Lane `l` of the per-lane value v takes the wave-uniform x (the compiler's own
// intrinsic, so that it sees the wait states between the writer of x and the move).
extern "C" __device__ int itc_writelane(int x, int l, int v) __asm("llvm.amdgcn.writelane.i32");

__device__ __forceinline__ uint32_t rows_mask(int n) { return n >= 32 ? ~0u : (1u << n) - 1u; }

// Edges of one strip of 64 columns: at each seam row 32 w, up | down << 16, and
// in the row after it the bit word of the column's rows 32 w .. 32 w + 31.
__device__ __forceinline__ void chamfer_edges(const uint8_t* __restrict__ x, int64_t pitch, float* __restrict__ t,
                                              int H, int W, int v0, uint32_t* __restrict__ sbits,
                                              uint16_t* __restrict__ sup, uint16_t* __restrict__ sdown) {
  const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
  const int j = v0 + lane;
  const bool col = j < W;
  const rsrc_t xr = make_rsrc(x, (uint32_t)((int64_t)H * pitch));
  const int nw = (H + 31) / 32;
  const bool quads = (((uintptr_t)x | (uintptr_t)pitch) & 3u) == 0;  // rows start 4-byte aligned (uniform)
  for (int w = wave; w < nw; w += CH_COLS_WAVES) {
    const int n = min(32, H - 32 * w);
    if (quads) {
      // lane (q, c): four columns 4c .. 4c + 3 of rows 8q .. 8q + 7, whose bits are a byte of each column's word
      const int q = lane >> 4, c = 4 * (lane & 15);
      const uint32_t off = (uint32_t)(32 * w + 8 * q) * (uint32_t)pitch + (uint32_t)(v0 + c);
      uint32_t v[8], acc = 0u;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        v[k] = buf_load<uint32_t>(xr, 8 * q + k < n && v0 + c < W ? off + (uint32_t)k * (uint32_t)pitch : BUF_OOB, 0);
#pragma unroll
      for (int k = 0; k < 8; ++k)
        acc = acc >> 1 | ((((v[k] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v[k]) & 0x80808080u);
      uint8_t* sb = reinterpret_cast<uint8_t*>(sbits + w * 64 + c) + q;
#pragma unroll
      for (int e = 0; e < 4; ++e) sb[4 * e] = (uint8_t)(acc >> (8 * e));
      continue;
    }
    uint32_t v[32];
    load_rows(xr, pitch, 32 * w, n, j, col, v);
    uint32_t m = 0u;
#pragma unroll
    for (int k = 0; k < 32; ++k) m |= (v[k] != 0u ? 1u : 0u) << k;
    sbits[w * 64 + lane] = m & rows_mask(n);
  }
  __syncthreads();
  if (wave == 0) {
    int nxt = H;  // row H is background
    for (int w = nw - 1; w >= 1; --w) {
      const uint32_t inv = ~sbits[w * 64 + lane];
      if (inv) nxt = 32 * w + __builtin_ctz(inv);
      sdown[w * 64 + lane] = (uint16_t)(nxt - 32 * w);
    }
  } else if (wave == 1) {
    int lst = -1;  // row -1 is background
    for (int w = 0; w < nw; ++w) {
      const uint32_t inv = ~sbits[w * 64 + lane];
      sup[w * 64 + lane] = (uint16_t)(inv & 1u ? 0 : 32 * w - lst);
      if (inv) lst = 32 * w + 31 - __builtin_clz(inv);
    }
  }
  __syncthreads();
  if (col) {
    for (int w = wave; w < nw; w += CH_COLS_WAVES) {
      if (w > 0) t_word(t, pitch, 32 * w)[j] = (uint32_t)sup[w * 64 + lane] | (uint32_t)sdown[w * 64 + lane] << 16;
      if (32 * w + 1 < H) t_word(t, pitch, 32 * w + 1)[j] = sbits[w * 64 + lane];
    }
  }
  __syncthreads();  // LDS is reused by the next strip
}

// Seam row i (a multiple of 32, below H).
__device__ __forceinline__ void chamfer_seam(float* __restrict__ t, int64_t pitch, int W, int i, int a, int b,
                                             uint16_t* __restrict__ gs) {
  uint32_t* row = t_word(t, pitch, i);
  uint32_t* above = t_word(t, pitch, i - 1);
  for (int j = (int)threadIdx.x - CH_GUARD; j < W + CH_GUARD; j += blockDim.x) {
    const uint32_t e = j >= 0 && j < W ? row[j] : 0u;
    gs[j] = (uint16_t)min(e & 0xffffu, e >> 16);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < W; j += blockDim.x) {
    const uint32_t e = row[j];  // this thread alone rewrites it
    const uint32_t T = (uint32_t)row_search(gs, j, W, a, b - a);
    if (e != 0u) row[j] = T | e << 16;  // T | up (a background pixel's word is 0 already)
    above[j] = T | (e & 0xffff0000u);  // T | down
  }
}

// The 33 entries e[i st] of one diagonal scanned both ways with slope b: f[i].x
// downwards at i, f[i].y upwards at 32 - i, both in one packed register (half i
// and half 32 - i are loaded into the halves of one register; past the middle
// they swap).
__device__ __forceinline__ void scan_both(const uint16_t* __restrict__ e, int st, u16x2 B2, u16x2 (&f)[CHB_ROWS + 1]) {
  u16x2 p[CHB_ROWS / 2 + 1];
#pragma unroll
  for (int i = 0; i <= CHB_ROWS / 2; ++i) p[i] = u16x2{e[i * st], e[(CHB_ROWS - i) * st]};
  f[0] = p[0];
#pragma unroll
  for (int i = 1; i <= CHB_ROWS; ++i)
    f[i] = __builtin_elementwise_min(i <= CHB_ROWS / 2 ? p[i] : p[CHB_ROWS - i].yx, f[i - 1] + B2);
}

// One band: rows r0 .. min(r0 + 32, H) - 1 of one image of at most PW columns.
template <int PW>
__device__ __forceinline__ void chamfer_band(const uint8_t* __restrict__ x, int64_t pitch, float* __restrict__ t,
                                             int H, int W, int r0, int a, int b, char* smem) {
  constexpr int P = chb_stride(PW), NWD = PW / 32, FS = NWD + 1;
  static_assert((P / 2) % 2 == 1 && P % 2 == 0, "an odd number of words per row of E");
  constexpr size_t E_BYTES = ((size_t)(CHB_ROWS + 1) * P * sizeof(uint16_t) + 7) / 8 * 8;
  uint16_t* E = reinterpret_cast<uint16_t*>(smem);                            // [33][P]
  uint64_t* S = reinterpret_cast<uint64_t*>(smem + E_BYTES);                  // [32]: words of the row with background
  uint32_t* F = reinterpret_cast<uint32_t*>(smem + E_BYTES + CHB_ROWS * sizeof(uint64_t));  // [32][FS]
  uint32_t* fg = F + CHB_ROWS * FS;
  const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ns = (W + 63) / 64;
  const bool first = r0 == 0, last = r0 + CHB_ROWS >= H;
  const int n = min(CHB_ROWS, H - r0);
  const bool words = H > CHB_ROWS && n > 1;  // the edges pass left the columns' bit words in row r0 + 1
  const rsrc_t xr = make_rsrc(x, (uint32_t)((int64_t)H * pitch));
  // guard columns of E: outside the lattice, background
  for (int q = tid; q < (CHB_ROWS + 1) * 2 * CHB_ROWS; q += CHB_NT) {
    const int i = q >> 6, c = q & 63;
    E[i * P + (c < 32 ? c : 64 * ns + c)] = 0;
  }
  if (tid < CHB_ROWS) S[tid] = 0;
  if (tid == 0) *fg = 0u;
  __syncthreads();
  // ---- rows of the band: bit words, and a g into E (lane = column) ----
  for (int st = wave; st < ns; st += CHB_WAVES) {
    const int j = 64 * st + lane;
    const bool col = j < W;
    uint32_t m = 0u, lo = 0u, hi = 0u;
    if (words) {
      if (col) m = t_word(t, pitch, r0 + 1)[j];
    } else {
      uint32_t v[32];
      load_rows(xr, pitch, r0, n, j, col, v);
#pragma unroll
      for (int k = 0; k < 32; ++k) m |= (v[k] != 0u ? 1u : 0u) << k;
      m &= rows_mask(n);
    }
    uint32_t top = 0u, bot = 0u;  // T | up of the first row, T | down of the seam below
    if (col && !first) top = t_word(t, pitch, r0)[j];
    if (col && !last) bot = t_word(t, pitch, r0 + CHB_ROWS - 1)[j];
    const bool some_fg = __any(m != 0u);  // uniform
    if (some_fg) {
      for_each_index(
          [&](auto kk) {
            constexpr int k = decltype(kk)::value;
            const uint64_t row = __ballot((m & (1u << k)) != 0u);
            lo = (uint32_t)itc_writelane((int)(uint32_t)row, k, (int)lo);  // lane k keeps row k's words
            hi = (uint32_t)itc_writelane((int)(uint32_t)(row >> 32), k, (int)hi);
          },
          std::make_integer_sequence<int, 32>{});
      if (lane == 0) atomicOr(fg, 1u << st);
    }
    if (lane < CHB_ROWS) {
      F[lane * FS + 2 * st] = lo;
      F[lane * FS + 2 * st + 1] = hi;
      const uint64_t some = (uint64_t)((~lo != 0u ? 1u : 0u) | (~hi != 0u ? 2u : 0u)) << (2 * st);
      if (some) atomicOr((unsigned long long*)&S[lane], (unsigned long long)some);
    }
    uint16_t* e = E + CHB_ROWS + j;
    e[CHB_ROWS * P] = (uint16_t)(bot & 0xffffu);  // 0 below the lattice
    if (!some_fg) continue;  // its zeros follow below, where a scan reads them
    // distances in units of a: up from the first row's, down from the seam below
    uint32_t dn[CHB_ROWS], run = (uint32_t)a * (bot >> 16);
#pragma unroll
    for (int k = CHB_ROWS - 1; k >= 0; --k) {
      run = (run + (uint32_t)a) & (uint32_t)((int32_t)(m << (31 - k)) >> 31);
      dn[k] = run;
    }
    // the first row of the lattice follows row -1; a seam row's own up distance is known, and its T
    run = first ? (m & 1u ? (uint32_t)a : 0u) : (uint32_t)a * (top >> 16);
    e[0] = (uint16_t)(first ? min(run, dn[0]) : top & 0xffffu);
#pragma unroll
    for (int k = 1; k < CHB_ROWS; ++k) {
      run = (run + (uint32_t)a) & (uint32_t)((int32_t)(m << (31 - k)) >> 31);
      e[k * P] = (uint16_t)min(run, dn[k]);
    }
  }
  __syncthreads();
  const uint32_t strips = *fg;  // strips with a foreground pixel
  // ---- E = min(E, a h): lane = (row, word of 32 columns), pairs of columns ----
  for (int st = wave; st < ns; st += CHB_WAVES) {
    const int r = lane & 31, w = 2 * st + (lane >> 5);
    if (!(strips >> st & 1u)) {
      if ((((uint64_t)strips << 1 | strips >> 1) >> st & 1u) == 0) continue;  // nor has a neighbour foreground
#pragma unroll
      for (int k = 0; k < CHB_ROWS; k += 2)
        *reinterpret_cast<u16x2*>(E + (k + (lane >> 5)) * P + CHB_ROWS + 64 * st + 2 * r) = u16x2{0, 0};
      continue;
    }
    const uint32_t m = F[r * FS + w];
    const uint64_t sr = S[r];
    const uint64_t before = sr & ((1ull << w) - 1ull);
    const uint64_t after = w >= 63 ? 0ull : sr >> (w + 1);
    uint32_t run = (uint32_t)a * (uint32_t)(32 * w), rn = (uint32_t)a * (uint32_t)(64 * ns - 32 * (w + 1));
    if (before) {
      const int q = 63 - __builtin_clzll(before);
      run = (uint32_t)a * (uint32_t)(32 * (w - 1 - q) + __builtin_clz(~F[r * FS + q]));
    }
    if (after) {
      const int q = w + 1 + __builtin_ctzll(after);
      rn = (uint32_t)a * (uint32_t)(32 * (q - w - 1) + __builtin_ctz(~F[r * FS + q]));
    }
    uint32_t lf[32];
#pragma unroll
    for (int c = 0; c < 32; ++c) {
      run = (run + (uint32_t)a) & (uint32_t)((int32_t)(m << (31 - c)) >> 31);
      lf[c] = run;
    }
    u16x2* e = reinterpret_cast<u16x2*>(E + r * P + CHB_ROWS + 32 * w);
#pragma unroll
    for (int c = 30; c >= 0; c -= 2) {
      rn = (rn + (uint32_t)a) & (uint32_t)((int32_t)(m << (30 - c)) >> 31);
      const uint32_t h1 = min(lf[c + 1], rn);
      rn = (rn + (uint32_t)a) & (uint32_t)((int32_t)(m << (31 - c)) >> 31);
      const uint32_t h0 = min(lf[c], rn);
      e[c / 2] = __builtin_elementwise_min(e[c / 2], u16x2{(uint16_t)h0, (uint16_t)h1});
    }
  }
  __syncthreads();
  // ---- scans along the diagonals j - i = d, then along j + i = s, in place ----
  // A task of 64 diagonals reads columns d0 - 32 .. d0 + 63 (strips d0 / 64 - 1 and d0 / 64); without
  // foreground there, all it reads is 0.
  const u16x2 B2 = {(uint16_t)b, (uint16_t)b};
  auto scan = [&](uint16_t* row0, int st) __attribute__((always_inline)) {
    for (int d0 = 64 * wave; d0 < W + CHB_ROWS; d0 += CHB_NT) {
      if ((((uint64_t)strips << 1) >> (d0 >> 6) & 3u) == 0) continue;
      const int d = d0 + lane;
      if (d < W + CHB_ROWS) {
        uint16_t* e = row0 + d;
        u16x2 f[CHB_ROWS + 1];
        scan_both(e, st, B2, f);
#pragma unroll
        for (int i = 0; i <= CHB_ROWS / 2; ++i) {
          const u16x2 r = __builtin_elementwise_min(f[i], f[CHB_ROWS - i].yx);
          e[i * st] = r.x;
          e[(CHB_ROWS - i) * st] = r.y;
        }
      }
    }
    __syncthreads();
  };
  scan(E, P + 1);             // entry (i, d + i) of the guarded rows
  scan(E + CHB_ROWS, P - 1);  // entry (i, s - i)
  // ---- out: four columns a lane, a quarter of the wave's rows in flight ----
  for (int c0 = 0; c0 < W; c0 += 256) {
    const int j = c0 + 4 * lane;
    const bool some = strips >> ((j >> 6) & 31) & 1u;
    for (int i = wave; i < n; i += CHB_WAVES) {
      if (j >= W) continue;
      const u16x2* e = reinterpret_cast<const u16x2*>(E + i * P + CHB_ROWS + j);
      u16x2 x = {0, 0}, y = {0, 0};
      if (some) {
        x = e[0];
        y = e[1];
      }
      float* o = t + (int64_t)(r0 + i) * pitch + j;
      const f32x4 T = {(float)x.x, (float)x.y, (float)y.x, (float)y.y};
      if (j + 3 < W) {
        __builtin_nontemporal_store(T, reinterpret_cast<f32x4*>(o));
      } else {
#pragma unroll
        for (int k = 0; k < 3; ++k)
          if (j + k < W) __builtin_nontemporal_store(T[k], o + k);
      }
    }
  }
}

__global__ void __launch_bounds__(CH_COLS_NT) chamfer_edges_kernel(const uint8_t* x, int64_t pitch, float* t, int H,
                                                                   int W) {
  __shared__ uint32_t sbits[CH_WORDS * 64];
  __shared__ uint16_t sup[CH_WORDS * 64], sdown[CH_WORDS * 64];
  chamfer_edges(x, pitch, t, H, W, blockIdx.x * 64, sbits, sup, sdown);
}

__global__ void __launch_bounds__(CH_ROWS_NT) chamfer_seams_kernel(float* t, int64_t pitch, int W, int a, int b) {
  extern __shared__ uint16_t gsh[];
  chamfer_seam(t, pitch, W, ((int)blockIdx.x + 1) * CHB_ROWS, a, b, gsh + CH_GUARD);
}

template <int PW>
__global__ void __launch_bounds__(CHB_NT) chamfer_bands_kernel(const uint8_t* x, int64_t pitch, float* t, int H, int W,
                                                               int a, int b) {
  extern __shared__ __align__(16) char bsm[];
  chamfer_band<PW>(x, pitch, t, H, W, (int)blockIdx.x * CHB_ROWS, a, b, bsm);
}

__global__ void __launch_bounds__(CH_COLS_NT) chamfer_edges_batched_kernel(const ImageDesc* __restrict__ images,
                                                                           const ChamferTask* __restrict__ tasks,
                                                                           int ntasks, const uint8_t* x, float* t) {
  __shared__ uint32_t sbits[CH_WORDS * 64];
  __shared__ uint16_t sup[CH_WORDS * 64], sdown[CH_WORDS * 64];
  for (int k = blockIdx.x; k < (ntasks + 63) / 64 * 64; k += gridDim.x) {
    // workgroups b, b + 8, .. share an XCD: it takes runs of eight strips, whose rows share cache lines
    // (0.155 ms of edges for 0.165 one strip apart)
    const int kt = (k & ~63) + 8 * (k & 7) + (k >> 3 & 7);
    if (kt >= ntasks) continue;
    const ChamferTask c = tasks[kt];
    const ImageDesc& im = images[c.img];
    if (im.H <= CHB_ROWS) continue;  // one band, no seam (uniform)
    chamfer_edges(x + im.weight_off, im.pitch, t + im.weight_off, im.H, im.W, c.pos * 64, sbits, sup, sdown);
  }
}

__global__ void __launch_bounds__(CH_ROWS_NT) chamfer_seams_batched_kernel(const ImageDesc* __restrict__ images,
                                                                           const ChamferTask* __restrict__ bands,
                                                                           float* t, int a, int b) {
  extern __shared__ uint16_t gsh[];
  const ChamferTask c = bands[blockIdx.x];
  if (c.pos == 0) return;  // the first band has no seam above it
  const ImageDesc& im = images[c.img];
  chamfer_seam(t + im.weight_off, im.pitch, im.W, c.pos, a, b, gsh + CH_GUARD);
}

template <int PW>
__global__ void __launch_bounds__(CHB_NT) chamfer_bands_batched_kernel(const ImageDesc* __restrict__ images,
                                                                       const ChamferTask* __restrict__ bands,
                                                                       const uint8_t* x, float* t, int a, int b) {
  extern __shared__ __align__(16) char bsm[];
  const ChamferTask c = bands[blockIdx.x];
  const ImageDesc& im = images[c.img];
  chamfer_band<PW>(x + im.weight_off, im.pitch, t + im.weight_off, im.H, im.W, c.pos, a, b, bsm);
}

// f(integral_constant<int, PW>) for the narrowest compiled width that holds w.
template <typename F>
void with_band_width(int w, F&& f) {
  if (w <= 512)
    f(std::integral_constant<int, 512>{});
  else if (w <= 1024)
    f(std::integral_constant<int, 1024>{});
  else
    f(std::integral_constant<int, CHB_MAX_W>{});
}

}  // namespace

int chamfer_rows_per_task() { return CH_ROWS_PER_TASK; }
int chamfer_rows_per_band() { return CHB_ROWS; }

hipError_t launch_chamfer(const ImageDesc& im, const void* x, float* t, int a, int b, hipStream_t s) {
  const size_t grow = (size_t)(im.W + 2 * CH_GUARD) * sizeof(uint16_t);
  const int strips = (im.W + 63) / 64, nb = (im.H + CHB_ROWS - 1) / CHB_ROWS;
  if (chb_fits(im.H, im.W, a, b)) {
    if (nb > 1) {
      hipLaunchKernelGGL(chamfer_edges_kernel, dim3(strips), dim3(CH_COLS_NT), 0, s, (const uint8_t*)x, im.pitch, t,
                         im.H, im.W);
      hipLaunchKernelGGL(chamfer_seams_kernel, dim3(nb - 1), dim3(CH_ROWS_NT), grow, s, t, im.pitch, im.W, a, b);
    }
    with_band_width(im.W, [&](auto pw) {
      constexpr int PW = decltype(pw)::value;
      hipLaunchKernelGGL(chamfer_bands_kernel<PW>, dim3(nb), dim3(CHB_NT), chb_smem(PW), s, (const uint8_t*)x,
                         im.pitch, t, im.H, im.W, a, b);
    });
    return hipGetLastError();
  }
  hipLaunchKernelGGL(chamfer_cols_kernel, dim3(strips), dim3(CH_COLS_NT), 0, s, (const uint8_t*)x,
                     im.pitch, t, im.H, im.W);
  hipLaunchKernelGGL(chamfer_rows_kernel, dim3((im.H + CH_ROWS_PER_TASK - 1) / CH_ROWS_PER_TASK),
                     dim3(CH_ROWS_NT), grow, s, t, im.pitch, im.H, im.W, a, b);
  return hipGetLastError();
}

hipError_t launch_chamfer_batched(const ImageDesc* d_images, const ChamferTask* d_cols, int ncols,
                                  const ChamferTask* d_rows, int nrows, const ChamferTask* d_bands, int nbands,
                                  int h_max, int w_max, const void* x, float* t, int a, int b, int grid_cols,
                                  int grid_rows, hipStream_t s) {
  if (chb_fits(h_max, w_max, a, b)) {
    if (h_max > CHB_ROWS) {
      hipLaunchKernelGGL(chamfer_edges_batched_kernel, dim3(grid_cols), dim3(CH_COLS_NT), 0, s, d_images, d_cols,
                         ncols, (const uint8_t*)x, t);
      hipLaunchKernelGGL(chamfer_seams_batched_kernel, dim3(nbands), dim3(CH_ROWS_NT),
                         (size_t)(w_max + 2 * CH_GUARD) * sizeof(uint16_t), s, d_images, d_bands, t, a, b);
    }
    with_band_width(w_max, [&](auto pw) {
      constexpr int PW = decltype(pw)::value;
      hipLaunchKernelGGL(chamfer_bands_batched_kernel<PW>, dim3(nbands), dim3(CHB_NT), chb_smem(PW), s, d_images,
                         d_bands, (const uint8_t*)x, t, a, b);
    });
    return hipGetLastError();
  }
  hipLaunchKernelGGL(chamfer_cols_batched_kernel, dim3(grid_cols), dim3(CH_COLS_NT), 0, s, d_images, d_cols, ncols,
                     (const uint8_t*)x, t);
  hipLaunchKernelGGL(chamfer_rows_batched_kernel, dim3(grid_rows), dim3(CH_ROWS_NT),
                     (size_t)(w_max + 2 * CH_GUARD) * sizeof(uint16_t), s, d_images, d_rows, nrows, t, a, b);
  return hipGetLastError();
}

}  // namespace itc
