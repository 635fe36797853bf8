// ITC fixed-point iteration on precomputed lattice maps (eq. (4) with the data
// sums read from the convolution maps, Section 3.1; loop of Algorithm 1).
//
// One 256-thread workgroup fits one image. Thread t owns codevectors
// k = t, t + 256, ...: it reads the maps bilinearly at w_k, keeps w_k in FP64
// registers and applies its update. The sum over j of the codebook Gaussian
// terms (M^2 pairs per sweep) is spread evenly over the 64 lanes of the four
// waves: the codebook is cut, by the binary digits of M, into chunks of
// 64 / P codevectors (P = 1 for every full 64, then P = 2, 4, .., 64 for the
// remaining powers of two), so that each chunk fills one wave with P lanes
// per codevector; the step sequence of all chunks (a step: one pair per lane)
// is divided into four contiguous equal parts, one per wave. A wave writes
// the P-lane sums (a fixed cross-lane DPP tree) of each chunk it visits to a
// per-(codevector, wave) slot in LDS, and the owner adds the four slots in
// wave order. S_XW = sum_k A_k and S_W = sum_k C_k are reduced in FP64 in a
// fixed order, so results are bitwise reproducible and identical between the
// single-image and the batched launch. Every wave reduces its own A_k and its
// own pair terms before the barrier that ends the pair phase, so one barrier
// serves the slots and both sums and a second one the new codebook.
//
// A codebook of at most FIT_SMALL codevectors is one wave's work (fit_small):
// P = 2 .. 16 lanes share a codevector and keep it, no barrier at all. A sweep is
// a chain of latencies there: 0.70 us at M = 16 and 0.99 at M = 32 (with a trace;
// FP32), against 1.85 and 1.95 on four waves with three barriers. 33 .. 64
// codevectors would take 64 pair steps a lane, 1.4 us, against 1.6 with all else.
//
// The D trace needs three FP64 logarithms a sweep (0.4 us on the chain); 64
// sweeps' sums wait in the lanes of a wave, which then takes the logarithms of
// all of them at once.
//
// Precision: codevector positions are FP64 whatever the map type (with FP32
// coordinates the rounding of w, 2.4e-4 px near u = 2048, accumulated over
// the sweeps, would dominate the error). LDS holds a copy in the map type,
// relative to the image centre and scaled by s = sqrt(log2(e) / (2 sigma^2)),
// so that a pair's Gaussian is exp2(-|w_j' - w_k'|^2) and its repulsion sum
// is E = E'/s. Pair differences are one subtraction in the map type: in FP32
// the rounding of the centred, scaled copies (at most half an ulp of
// s max(H, W) / 2) perturbs a near pair's Gaussian by a few 1e-5 relative, far
// below the data term's effect; FP64 keeps FP64 differences. The LDS codebook
// is padded with points at 1e30, whose Gaussian is exactly 0.
#include <type_traits>

#include "itc_device.h"

namespace itc {

constexpr int FIT_NT = 256;
constexpr int FIT_WAVES = FIT_NT / 64;
constexpr double FIT_FAR = 1e30;
// A byte offset past the end of any maps buffer (< 2 GiB with every plane
// added): buffer loads there return 0 without touching memory.
constexpr uint32_t FIT_OOB = 0x80000000u;

using P2 = V2<double>;

// Per-image status bits (the batched fit's status output).
constexpr int32_t FIT_STATUS_SUMS = 1;  // S_XW or S_W not finite: the fit stopped at the last finite codebook
constexpr int32_t FIT_STATUS_W = 2;     // a codevector step was not finite
constexpr int32_t FIT_STATUS_D = 4;     // D not finite

__device__ __forceinline__ float exp2_neg(float x) { return __builtin_amdgcn_exp2f(-x); }
__device__ __forceinline__ float recip(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }
__device__ __forceinline__ double exp2_neg(double x) { return exp2(-x); }

// Owner passes: thread t owns k = t + 256 ps for ps < ceil(M / 256).
__host__ __device__ inline int fit_passes(int M) { return (M + FIT_NT - 1) / FIT_NT; }
// LDS codebook entries: the pair loop of a chunk with P lanes per codevector
// reads 4 P ceil(M / 4P) entries, at most 256 ceil(M / 256), and one block
// of 4 P <= 256 past them (read ahead, unused).
__host__ __device__ inline int fit_codebook_len(int M) { return (M + 255) / 256 * 256 + 256; }

// Steps of a chunk with P = 2^lg lanes per codevector, in units of four.
__device__ __forceinline__ int chunk_units(int M, int lg) { return (M + (4 << lg) - 1) / (4 << lg); }

// Sums of the Gaussian terms of one codevector (scaled position hu, hv) over
// this lane's column of the LDS codebook (entries col[0], col[P], ...), in
// blocks of four entries, nun blocks. Two register sets alternate: the reads
// of the next block are issued before the arithmetic of the current one, so
// the LDS latency is hidden behind it (the scheduling barriers keep the
// compiler from sinking the reads). The read after the last block falls in
// the padding of the codebook. Even and odd entries of a block accumulate
// separately: two independent chains.
template <typename T, int P>
__device__ __forceinline__ void pair_blocks(const V2<T>* __restrict__ col, int nun, T hu, T hv, T& C, T& Cu,
                                            T& Cv) {
  T C0 = 0, Cu0 = 0, Cv0 = 0, C1 = 0, Cu1 = 0, Cv1 = 0;
  auto acc = [&](const V2<T>(&x)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const T du = x[i].u - hu, dv = x[i].v - hv;
      const T e = exp2_neg(fma_t(du, du, dv * dv));
      if (i & 1) {
        C1 += e;
        Cu1 = fma_t(e, du, Cu1);
        Cv1 = fma_t(e, dv, Cv1);
      } else {
        C0 += e;
        Cu0 = fma_t(e, du, Cu0);
        Cv0 = fma_t(e, dv, Cv0);
      }
    }
  };
  V2<T> a[4], b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = col[i * P];
  int u = 0;
  for (; u + 2 <= nun; u += 2) {
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = col[(u + 1) * 4 * P + i * P];
    __builtin_amdgcn_sched_barrier(0);
    acc(a);
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = col[(u + 2) * 4 * P + i * P];
    __builtin_amdgcn_sched_barrier(0);
    acc(b);
  }
  if (u < nun) acc(a);
  C = C0 + C1;
  Cu = Cu0 + Cu1;
  Cv = Cv0 + Cv1;
}

// Sums over j = p, p + P, .. (steps [u0, u1) in units of four) of the
// Gaussian terms of codevector k: this lane's share of C, and E over the P
// lanes of each codevector.
template <typename T, int P>
__device__ __forceinline__ void pair_chunk(const V2<T>* __restrict__ Wh, int k, int p, int u0, int u1, T& C, T& Cu,
                                           T& Cv) {
  const V2<T> hk = Wh[k];
  pair_blocks<T, P>(Wh + p + u0 * 4 * P, u1 - u0, hk.u, hk.v, C, Cu, Cv);
  Cu = group_sum<P>(Cu);
  Cv = group_sum<P>(Cv);
}

// The codebook's chunks: every full 64 codevectors with P = 1, then the
// remainder r = M mod 64 as at most two chunks: the largest power of two in r
// (P = 64 / that), then the rest, with the most lanes per codevector that fit
// a wave (some lanes idle). Chunk c starting at codevector k0: returns log2 P
// and its size.
__device__ __forceinline__ int chunk_lg(int M, int k0, int& size) {
  const int rem = M - k0;
  if (rem >= 64) {
    size = 64;
    return 0;
  }
  const int hb = 31 - __builtin_clz((unsigned)rem);  // floor(log2 rem)
  const bool first = (M & 63) == rem;                 // the first remainder chunk
  if (first && (rem & (rem - 1))) {
    size = 1 << hb;
    return 6 - hb;
  }
  size = rem;
  return 6 - ((rem & (rem - 1)) ? hb + 1 : hb);
}

// Steps of all chunks, in units of four.
__device__ __forceinline__ int pair_units(int M) {
  int units = 0;
  for (int k0 = 0, size = 0; k0 < M; k0 += size) units += chunk_units(M, chunk_lg(M, k0, size));
  return units;
}

// A wave's share [ua, ub) of the chunk steps, as the chunks it visits: lane i
// keeps visit i (at most 18: 16 full chunks and the remainder's two). They are laid
// out once per image: finding the chunks in every sweep's scalar code took 0.33 of
// 2.44 us a sweep at M = 100, 0.37 of 4.98 at M = 200, 27 of 668 us of 1,400 silhouettes.
// Reading a visit's first entries ahead of the one before it costs more registers
// than it saves (2.34 us, 4.98).
struct Visits {
  int n = 0;
  uint32_t where = 0;  // first codevector | size << 16 | log2 P << 24
  uint32_t steps = 0;  // first unit | units << 16
};

__device__ __forceinline__ Visits pair_visits(int M, int ua, int ub, int lane) {
  Visits v;
  int cu0 = 0, k0 = 0;
  while (k0 < M && cu0 < ub) {  // uniform
    int size = 0;
    const int lg = chunk_lg(M, k0, size);
    const int nu = chunk_units(M, lg);
    const int s0 = ua > cu0 ? ua : cu0, s1 = ub < cu0 + nu ? ub : cu0 + nu;
    if (s0 < s1) {
      if (lane == v.n) {
        v.where = (uint32_t)k0 | (uint32_t)size << 16 | (uint32_t)lg << 24;
        v.steps = (uint32_t)(s0 - cu0) | (uint32_t)(s1 - s0) << 16;
      }
      ++v.n;
    }
    cu0 += nu;
    k0 += size;
  }
  return v;
}

// The pair phase of one sweep: the wave's visits, each visited codevector's E
// to part[wave * M + k] (consecutive lanes meet consecutive words). Returns this
// lane's sum of its C terms.
template <typename T>
__device__ __forceinline__ double pair_phase(const V2<T>* __restrict__ Wh, V2<T>* __restrict__ part, int M,
                                             const Visits& vis, int wave, int lane) {
  double csum = 0.0;
#pragma unroll 1
  for (int i = 0; i < vis.n; ++i) {  // uniform
    const uint32_t where = __builtin_amdgcn_readlane(vis.where, i), steps = __builtin_amdgcn_readlane(vis.steps, i);
    const int k0 = (int)(where & 0xffffu), size = (int)(where >> 16 & 0xffu), lg = (int)(where >> 24);
    const int u0 = (int)(steps & 0xffffu), u1 = u0 + (int)(steps >> 16);
    const int k = k0 + (lane >> lg), p = lane & ((1 << lg) - 1);
    T C = 0, Cu = 0, Cv = 0;
    switch (lg) {
      case 0: pair_chunk<T, 1>(Wh, k, p, u0, u1, C, Cu, Cv); break;
      case 1: pair_chunk<T, 2>(Wh, k, p, u0, u1, C, Cu, Cv); break;
      case 2: pair_chunk<T, 4>(Wh, k, p, u0, u1, C, Cu, Cv); break;
      case 3: pair_chunk<T, 8>(Wh, k, p, u0, u1, C, Cu, Cv); break;
      case 4: pair_chunk<T, 16>(Wh, k, p, u0, u1, C, Cu, Cv); break;
      case 5: pair_chunk<T, 32>(Wh, k, p, u0, u1, C, Cu, Cv); break;
      default: pair_chunk<T, 64>(Wh, k, p, u0, u1, C, Cu, Cv); break;
    }
    if (k < k0 + size) csum += (double)C;  // lanes past the chunk read padding and are idle
    if (p == 0 && k < k0 + size) part[wave * M + k] = V2<T>{Cu, Cv};
  }
  return csum;
}

struct FitImageArgs {
  const char* mbase;
  const void* w_init;
  void* w_out;
  double s_x;        // S_X of the image (used only for D)
  double* d_trace;   // [iters+1] or null
  double* d_out;     // one double or null
  int32_t* iters_done;
  int32_t* status;   // FIT_STATUS_* bits of this image, or null
  double theta;
  bool write_w;
  void* grad_w;          // gradient mode: dL/dw [M][2] at w_init (no update)
  const double* grad_d;  // dL/dD (one double), gradient mode only
};

// The lattice cell that a codevector was last read in (key -2: none yet), with
// the corner values of A, M_u and M_v: they stay in registers until the
// codevector enters another cell (near convergence it rarely does), so the maps
// are read again only then.
template <typename T>
struct Cell {
  int key = -2;
  T a[4] = {}, mu[4] = {}, mv[4] = {};
};

struct CellMaps {
  rsrc_t res;
  uint32_t planeb;
  int H, W;
};

// The cell of (u, v) (ok: a codevector is there): its fractions, and its corner
// values if it is another one than before. Off-lattice corners load at an offset
// past the end of the maps, which reads 0. The loads are issued here and
// consumed by cell_read.
template <typename T>
__device__ __forceinline__ void cell_fetch(Cell<T>& c, const CellMaps& m, double u, double v, bool ok, T& fu, T& fv) {
  const bool inside = ok && u > -1.0 && u < (double)m.H && v > -1.0 && v < (double)m.W;
  const double fu0 = inside ? floor(u) : 0.0, fv0 = inside ? floor(v) : 0.0;
  const int i0 = (int)fu0, j0 = (int)fv0;
  fu = (T)(u - fu0);
  fv = (T)(v - fv0);
  const int key = inside ? (i0 + 1) * (m.W + 2) + (j0 + 1) : -1;
  if (key != c.key) {
    c.key = key;
    const bool r0 = inside && i0 >= 0, r1 = inside && i0 + 1 < m.H;
    const bool c0 = j0 >= 0, c1 = j0 + 1 < m.W;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int di = q >> 1, dj = q & 1;
      const bool in = (di ? r1 : r0) && (dj ? c1 : c0);
      const uint32_t off = in ? (uint32_t)map_index(m.H, i0 + di, j0 + dj) * (uint32_t)sizeof(T) : FIT_OOB;
      c.a[q] = buf_load<T>(m.res, off, 0);
      c.mu[q] = buf_load<T>(m.res, off, m.planeb);
      c.mv[q] = buf_load<T>(m.res, off, 2 * m.planeb);
    }
  }
}

// Bilinear combination: A = sum_c b_c A(c), g = sum_c b_c ((c - w_k) A(c) - M(c)).
template <typename T>
__device__ __forceinline__ void cell_read(const Cell<T>& c, T fu, T fv, T& A, T& gu, T& gv) {
  A = gu = gv = (T)0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int di = q >> 1, dj = q & 1;
    const T b = (di ? fu : (T)1 - fu) * (dj ? fv : (T)1 - fv);
    A = fma_t(b, c.a[q], A);
    gu = fma_t(b, fma_t((T)di - fu, c.a[q], -c.mu[q]), gu);
    gv = fma_t(b, fma_t((T)dj - fv, c.a[q], -c.mv[q]), gv);
  }
}

// Slope of the bilinear interpolant of A: d/du and d/dv of sum_c b_c A(c),
// corners c = (di, dj) in (0,0),(0,1),(1,0),(1,1).
template <typename T>
__device__ __forceinline__ void cell_slope(const Cell<T>& c, T fu, T fv, T& du, T& dv) {
  du = ((T)1 - fv) * (c.a[2] - c.a[0]) + fv * (c.a[3] - c.a[1]);
  dv = ((T)1 - fu) * (c.a[1] - c.a[0]) + fu * (c.a[3] - c.a[2]);
}

// c / s (E = E' / s), in the map type.
template <typename T>
__device__ __forceinline__ T repulsion(double S_XW, double S_W, double s) {
  if constexpr (sizeof(T) == 4)
    return (T)S_XW * recip((T)S_W * (T)s);
  else
    return (T)(S_XW / S_W / s);
}

// D of eq. (1) from the sums.
__device__ __forceinline__ double divergence_of(double S_XW, double S_W, double s_x) {
  return log(S_W) + log(s_x) - 2.0 * log(S_XW);
}

// The D trace of one wave: lane t mod 64 keeps the sums of sweep t, and 64
// sweeps (or what is left at the end) take their logarithms together.
struct TraceRing {
  double sxw = 1.0, sw = 1.0;
  __device__ __forceinline__ void put(int t, double S_XW, double S_W, double s_x, double* d_trace, int lane) {
    if (lane == (t & 63)) {
      sxw = S_XW;
      sw = S_W;
    }
    if ((t & 63) == 63) flush(t, s_x, d_trace, lane);
  }
  // the sweeps t & ~63 .. t
  __device__ __forceinline__ void flush(int t, double s_x, double* d_trace, int lane) {
    if (lane <= (t & 63)) d_trace[(t & ~63) + lane] = divergence_of(sxw, sw, s_x);
  }
};

// Codebooks of at most FIT_SMALL codevectors, one wave: lanes k P .. k P + P - 1
// hold codevector k (the same values in each) and take the pair terms of j = p,
// p + P, .. (p their place among the P), M <= 64 / P. Wh: 64 entries in LDS, padded
// with FIT_FAR. lane: the caller's opaque one.
constexpr int FIT_SMALL = 32;

template <typename T, int P, bool TRACE>
__device__ void fit_small(const ImageDesc& im, const FitImageArgs& a, V2<T>* __restrict__ Wh, int lane) {
  constexpr int NJ = 64 / P / P > 1 ? 64 / P / P : 1;  // pair terms of a lane
  const int M = im.M, k = lane / P, p = lane % P;
  const bool own = k < M, lead = own && p == 0;
  const double s = sqrt(1.4426950408889634 / (2.0 * im.sigma * im.sigma));
  const double cu = 0.5 * im.H, cv = 0.5 * im.W;
  auto lds_pos = [&](double u, double v) { return V2<T>{(T)(s * (u - cu)), (T)(s * (v - cv))}; };
  const V2<T>* w_in = reinterpret_cast<const V2<T>*>(a.w_init) + im.w_off;
  double wu = 0.0, wv = 0.0;
  if (own) {
    const V2<T> w = w_in[k];
    wu = (double)w.u;
    wv = (double)w.v;
  }
  V2<T> h = own ? lds_pos(wu, wv) : V2<T>{(T)FIT_FAR, (T)FIT_FAR};
  // entries past 64 / P are padding for the lanes of the last block
  Wh[lane] = V2<T>{(T)FIT_FAR, (T)FIT_FAR};
  __builtin_amdgcn_wave_barrier();
  if (lead) Wh[k] = h;
  __builtin_amdgcn_wave_barrier();

  CellMaps cm;
  cm.planeb = (uint32_t)(im.plane * (int64_t)sizeof(T));
  cm.res = make_rsrc(a.mbase + im.map_off, 3u * cm.planeb);
  cm.H = im.H;
  cm.W = im.W;
  const bool need_d = a.d_trace != nullptr || a.d_out != nullptr || a.status != nullptr;
  Cell<T> cell;
  TraceRing ring;
  bool stop = false;
  int32_t flags = 0;
  int t = 0;
  for (;; ++t) {
    const bool last = (t == im.iters) || stop;
    if (last && !need_d && !a.grad_w) break;
    V2<T> x[NJ];  // issued first: the cell's arithmetic hides the LDS latency
#pragma unroll
    for (int i = 0; i < NJ; ++i) x[i] = Wh[p + P * i];
    T fu, fv;
    cell_fetch(cell, cm, wu, wv, own, fu, fv);
    // ---- codebook terms ----
    T C[2] = {}, Eu[2] = {}, Ev[2] = {};
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
      if (i > 0 && P * i >= M) break;  // uniform: padding only
      const T du = x[i].u - h.u, dv = x[i].v - h.v;
      const T e = exp2_neg(fma_t(du, du, dv * dv));
      C[i & 1] += e;
      Eu[i & 1] = fma_t(e, du, Eu[i & 1]);
      Ev[i & 1] = fma_t(e, dv, Ev[i & 1]);
    }
    const T Ck = group_sum<P>(C[0] + C[1]), Euk = group_sum<P>(Eu[0] + Eu[1]), Evk = group_sum<P>(Ev[0] + Ev[1]);
    // ---- data terms, sums ----
    T A, gu, gv;
    cell_read(cell, fu, fv, A, gu, gv);
    double S_XW = own ? (double)A : 0.0, S_W = own ? (double)Ck : 0.0;
    wave_sum2<P>(S_XW, S_W);
    // non-finite sums (non-finite weights or maps) end the fit at this codebook
    const bool sums_ok = isfinite(S_XW) && isfinite(S_W);  // uniform
    const bool final_eval = last || !sums_ok;
    if (!sums_ok) flags |= FIT_STATUS_SUMS;
    if (final_eval && (a.d_out || a.status)) {
      const double D = divergence_of(S_XW, S_W, a.s_x);
      if (!isfinite(D)) flags |= FIT_STATUS_D;
      if (lane == 0 && a.d_out) *a.d_out = D;
    }
    if constexpr (TRACE) {
      if (a.d_trace) {
        ring.put(t, S_XW, S_W, a.s_x, a.d_trace, lane);
        if (final_eval && (t & 63) != 63) ring.flush(t, a.s_x, a.d_trace, lane);
      }
    }
    if (a.grad_w) {  // adjoint of D at this codebook (eq. (1) differentiated through the reads)
      const double gd = *a.grad_d;
      const T ca = (T)(-2.0 * gd / S_XW);
      const T cb = (T)(2.0 * gd / (im.sigma * im.sigma * S_W) / s);  // E = E'/s
      V2<T>* gw = reinterpret_cast<V2<T>*>(a.grad_w) + im.w_off;
      T dAu, dAv;
      cell_slope(cell, fu, fv, dAu, dAv);
      if (lead) gw[k] = V2<T>{fma_t(ca, dAu, cb * Euk), fma_t(ca, dAv, cb * Evk)};
      break;
    }
    if (final_eval) break;
    // ---- Jacobi update ----
    const T cs = repulsion<T>(S_XW, S_W, s);
    float step = 0.0f;
    if (own && A != (T)0) {
      const T inv = recip(A);
      const T du = (gu - cs * Euk) * inv;
      const T dv = (gv - cs * Evk) * inv;
      if (!isfinite(du) || !isfinite(dv)) flags |= FIT_STATUS_W;
      wu += (double)du;
      wv += (double)dv;
      if (a.theta >= 0.0) step = (float)sqrt((double)du * du + (double)dv * dv);
      h = lds_pos(wu, wv);
    }
    __builtin_amdgcn_wave_barrier();
    if (lead) Wh[k] = h;
    __builtin_amdgcn_wave_barrier();
    if (a.theta >= 0.0) stop = (double)wave_max_nonneg(step) <= a.theta;
  }
  if (a.write_w && lead) {
    V2<T>* w_o = reinterpret_cast<V2<T>*>(a.w_out) + im.w_off;
    w_o[k] = V2<T>{(T)wu, (T)wv};
  }
  if (lane == 0 && a.iters_done) *a.iters_done = t;
  if (a.status) {
    const bool any_w = __any((flags & FIT_STATUS_W) != 0);
    if (lane == 0) *a.status = (flags & ~FIT_STATUS_W) | (any_w ? FIT_STATUS_W : 0);
  }
}

template <typename T, int MAXPASS, bool TRACE>
__device__ void fit_image(const ImageDesc& im, const FitImageArgs& a, char* smem) {
  const int M = im.M;
  const int WL = fit_codebook_len(M);
  // lane-derived values are recomputed per image: an opaque thread index
  // keeps the compiler from hoisting them out of the persistent image loop,
  // where they would stay live in registers across it
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: the pair phase's loops are scalar
  const int npass = fit_passes(M);
  using Q2 = V2<T>;
  Q2* Wh = reinterpret_cast<Q2*>(smem);  // centred scaled positions [WL]
  if (M <= FIT_SMALL) {  // uniform
    if (wave == 0) {
      if (M > 16)
        fit_small<T, 2, TRACE>(im, a, Wh, lane);
      else if (M > 8)
        fit_small<T, 4, TRACE>(im, a, Wh, lane);
      else if (M > 4)
        fit_small<T, 8, TRACE>(im, a, Wh, lane);
      else
        fit_small<T, 16, TRACE>(im, a, Wh, lane);
    }
    __syncthreads();  // shared memory is reused by the next image
    return;
  }
  Q2* part = Wh + WL;                                                // [4 waves][M]
  double* red = reinterpret_cast<double*>(part + FIT_WAVES * M);     // [4 waves][2]
  double* red2 = red + 8;                                            // [4 waves]

  const double s = sqrt(1.4426950408889634 / (2.0 * im.sigma * im.sigma));
  const double cu = 0.5 * im.H, cv = 0.5 * im.W;  // reference point of the LDS copy
  auto lds_pos = [&](double u, double v) { return Q2{(T)(s * (u - cu)), (T)(s * (v - cv))}; };
  const V2<T>* w_in = reinterpret_cast<const V2<T>*>(a.w_init) + im.w_off;

  // owned codevectors (FP64, in registers)
  double wu[MAXPASS], wv[MAXPASS];
#pragma unroll
  for (int ps = 0; ps < MAXPASS; ++ps) {
    const int k = ps * FIT_NT + tid;
    wu[ps] = wv[ps] = 0.0;
    if (ps < npass && k < M) {
      const V2<T> w = w_in[k];
      wu[ps] = (double)w.u;
      wv[ps] = (double)w.v;
    }
  }
  for (int k = tid; k < WL; k += FIT_NT) {
    Q2 h{(T)FIT_FAR, (T)FIT_FAR};
    if (k < M) {
      const V2<T> w = w_in[k];
      h = lds_pos((double)w.u, (double)w.v);
    }
    Wh[k] = h;
  }
  // slots no wave writes (a codevector's chunk may span fewer than four waves) stay 0
  for (int i = tid; i < M * FIT_WAVES; i += FIT_NT) part[i] = Q2{(T)0, (T)0};
  __syncthreads();

  CellMaps cm;
  cm.planeb = (uint32_t)(im.plane * (int64_t)sizeof(T));
  cm.res = make_rsrc(a.mbase + im.map_off, 3u * cm.planeb);
  cm.H = im.H;
  cm.W = im.W;
  const bool need_d = a.d_trace != nullptr || a.d_out != nullptr || a.status != nullptr;
  const int units = pair_units(M), ua = units * wave / FIT_WAVES, ub = units * (wave + 1) / FIT_WAVES;
  const Visits vis = pair_visits(M, ua, ub, lane);
  Cell<T> cell[MAXPASS];
  TraceRing ring;

  bool stop = false;
  int32_t flags = 0;   // status bits (uniform except FIT_STATUS_W, combined at the end)
  int t = 0;
  for (;; ++t) {
    const bool last = (t == im.iters) || stop;
    if (last && !need_d && !a.grad_w) break;

    // ---- data terms: bilinear read of A, M_u, M_v at w_k (the loads are issued
    // before the pair phase and consumed after it, which hides their latency) ----
    T fu[MAXPASS], fv[MAXPASS];
#pragma unroll
    for (int ps = 0; ps < MAXPASS; ++ps) {
      fu[ps] = fv[ps] = (T)0;
      if (ps < npass) cell_fetch(cell[ps], cm, wu[ps], wv[ps], ps * FIT_NT + tid < M, fu[ps], fv[ps]);
    }

    // ---- codebook terms of every codevector (scaled coordinates) ----
    double sw = pair_phase<T>(Wh, part, M, vis, wave, lane);

    // ---- A_k and g_k of the owned codevectors; this wave's shares of S_XW and S_W in FP64 ----
    T Ak[MAXPASS], gu[MAXPASS], gv[MAXPASS];
    double sxw = 0.0;
#pragma unroll
    for (int ps = 0; ps < MAXPASS; ++ps) {
      Ak[ps] = gu[ps] = gv[ps] = (T)0;
      if (ps < npass && ps * FIT_NT + tid < M) {
        cell_read(cell[ps], fu[ps], fv[ps], Ak[ps], gu[ps], gv[ps]);
        sxw += (double)Ak[ps];
      }
    }
    wave_sum2(sxw, sw);
    if (lane == 0) {
      red[2 * wave] = sxw;
      red[2 * wave + 1] = sw;
    }
    __syncthreads();
    double S_XW = 0.0, S_W = 0.0;
#pragma unroll
    for (int w = 0; w < FIT_WAVES; ++w) {
      S_XW += red[2 * w];
      S_W += red[2 * w + 1];
    }
    // non-finite sums (non-finite weights or maps) end the fit at this codebook
    const bool sums_ok = isfinite(S_XW) && isfinite(S_W);  // uniform
    const bool final_eval = last || !sums_ok;
    if (!sums_ok) flags |= FIT_STATUS_SUMS;
    if (tid == 0 && final_eval && (a.d_out || a.status)) {
      const double D = divergence_of(S_XW, S_W, a.s_x);
      if (!isfinite(D)) flags |= FIT_STATUS_D;
      if (a.d_out) *a.d_out = D;
    }
    if constexpr (TRACE) {
      if (a.d_trace && wave == 0) {
        ring.put(t, S_XW, S_W, a.s_x, a.d_trace, lane);
        if (final_eval && (t & 63) != 63) ring.flush(t, a.s_x, a.d_trace, lane);
      }
    }
    // E_k: the four waves' sums, in wave order
    auto slots = [&](int k, T& Eu, T& Ev) {
      Q2 e[FIT_WAVES];
#pragma unroll
      for (int w = 0; w < FIT_WAVES; ++w) e[w] = part[w * M + k];
      Eu = e[0].u;
      Ev = e[0].v;
#pragma unroll
      for (int w = 1; w < FIT_WAVES; ++w) {
        Eu += e[w].u;
        Ev += e[w].v;
      }
    };
    if (a.grad_w) {  // adjoint of D at this codebook (eq. (1) differentiated through the reads)
      const double gd = *a.grad_d;
      const T ca = (T)(-2.0 * gd / S_XW);
      const T cb = (T)(2.0 * gd / (im.sigma * im.sigma * S_W) / s);  // E = E'/s
      V2<T>* gw = reinterpret_cast<V2<T>*>(a.grad_w) + im.w_off;
#pragma unroll
      for (int ps = 0; ps < MAXPASS; ++ps) {
        const int k = ps * FIT_NT + tid;
        if (ps < npass && k < M) {
          T dAu, dAv, Eu, Ev;
          cell_slope(cell[ps], fu[ps], fv[ps], dAu, dAv);
          slots(k, Eu, Ev);
          gw[k] = V2<T>{fma_t(ca, dAu, cb * Eu), fma_t(ca, dAv, cb * Ev)};
        }
      }
      break;
    }
    if (final_eval) break;

    // ---- Jacobi update of every owned codevector ----
    const T cs = repulsion<T>(S_XW, S_W, s);
    float step = 0.0f;
#pragma unroll
    for (int ps = 0; ps < MAXPASS; ++ps) {
      const int k = ps * FIT_NT + tid;
      if (ps < npass && k < M && Ak[ps] != (T)0) {
        T Eu, Ev;
        slots(k, Eu, Ev);
        const T inv = recip(Ak[ps]);
        const T du = (gu[ps] - cs * Eu) * inv;
        const T dv = (gv[ps] - cs * Ev) * inv;
        if (!isfinite(du) || !isfinite(dv)) flags |= FIT_STATUS_W;
        wu[ps] += (double)du;
        wv[ps] += (double)dv;
        if (a.theta >= 0.0) step = fmaxf(step, (float)sqrt((double)du * du + (double)dv * dv));
        Wh[k] = lds_pos(wu[ps], wv[ps]);
      }
    }
    if (a.theta >= 0.0) {  // the largest step is needed only for the theta test
      step = wave_max_nonneg(step);
      if (lane == 0) red2[wave] = (double)step;
    }
    __syncthreads();  // the new codebook; red and the slots are read
    if (a.theta >= 0.0) {
      double smax = 0.0;
#pragma unroll
      for (int w = 0; w < FIT_WAVES; ++w) smax = fmax(smax, red2[w]);
      stop = smax <= a.theta;
    }
  }

  if (a.write_w) {
    V2<T>* w_o = reinterpret_cast<V2<T>*>(a.w_out) + im.w_off;
#pragma unroll
    for (int ps = 0; ps < MAXPASS; ++ps) {
      const int k = ps * FIT_NT + tid;
      if (ps < npass && k < M) w_o[k] = V2<T>{(T)wu[ps], (T)wv[ps]};
    }
  }
  if (tid == 0 && a.iters_done) *a.iters_done = t;
  if (a.status) {
    const int32_t any_w = __syncthreads_or((flags & FIT_STATUS_W) != 0);
    if (tid == 0) *a.status = (flags & ~FIT_STATUS_W) | (any_w ? FIT_STATUS_W : 0);
  }
  __syncthreads();  // shared memory is reused by the next image
}

template <typename T, int MAXPASS>
__global__ void __launch_bounds__(FIT_NT) fit_image_kernel(ImageDesc im, FitArgs fa) {
  extern __shared__ __align__(16) char smem[];
  FitImageArgs a;
  a.mbase = (const char*)fa.maps;
  a.w_init = fa.w_init;
  a.w_out = fa.w_out;
  a.s_x = fa.s_x_in ? *fa.s_x_in : 1.0;
  a.d_trace = fa.d_trace;
  a.d_out = fa.d_out;
  a.iters_done = fa.iters_done;
  a.status = nullptr;
  a.theta = fa.theta;
  a.write_w = fa.write_w != 0;
  a.grad_w = fa.grad_w;
  a.grad_d = fa.grad_d;
  fit_image<T, MAXPASS, true>(im, a, smem);
}

// Waves per SIMD the batched FP32 single-pass fit is compiled for: five (96
// registers, 19 of them spilled) of the four its registers would allow. ms at
// four, five and six waves: 1,400 silhouettes 0.68, 0.70, 0.68; 4,000 images with
// 4 to 255 codevectors 1.66, 1.53, 1.51; 3,000 with 40 0.34, 0.30, 0.32; 8 with 256
// 0.39, 0.40, 0.39. (54 were spilled, some in the sweep loops, while the one-wave
// form took its lane from threadIdx: 1,400 images with up to 32 codevectors 0.113 ms,
// now 0.101.)
template <typename T, int MAXPASS>
constexpr int fit_batched_min_waves() {
  return std::is_same<T, float>::value && MAXPASS == 1 ? 5 : 1;
}

// Workgroup g fits the images sched[G + 1 + sched[g]] .. sched[G + 1 + sched[g + 1] - 1]
// (G workgroups: the first G + 1 entries are the offsets of each workgroup's list).
template <typename T, int MAXPASS>
__global__ void __launch_bounds__(FIT_NT, (fit_batched_min_waves<T, MAXPASS>())) fit_batched_kernel(const ImageDesc* __restrict__ images,
                                                             const int32_t* __restrict__ sched, FitArgs fa) {
  extern __shared__ __align__(16) char smem[];
  double* red = reinterpret_cast<double*>(smem);
  const int32_t* list = sched + gridDim.x + 1;
  const int end = sched[blockIdx.x + 1];
  for (int ii = sched[blockIdx.x]; ii < end; ++ii) {
    const int i = list[ii];
    const ImageDesc im = images[i];
    // S_X: the fixed-order sum of the FP64 partials written with the maps
    const double* sxp = reinterpret_cast<const double*>((const char*)fa.maps + im.map_off + im.part_off);
    const double s_x =
        fa.s_x_in ? fa.s_x_in[i] : block_sum_fixed(sxp, (int64_t)im.nstrips * im.nsxg * SX_SLOTS, red);
    if (threadIdx.x == 0 && fa.s_x_out) fa.s_x_out[i] = s_x;
    FitImageArgs a;
    a.mbase = (const char*)fa.maps;
    a.w_init = fa.w_init;
    a.w_out = fa.w_out;
    a.s_x = s_x;
    a.d_trace = nullptr;
    a.d_out = fa.d_out ? fa.d_out + i : nullptr;
    a.iters_done = fa.iters_done ? fa.iters_done + i : nullptr;
    a.status = fa.status ? fa.status + i : nullptr;
    a.theta = fa.theta;
    a.write_w = fa.write_w != 0;
    a.grad_w = fa.grad_w;
    a.grad_d = fa.grad_d ? fa.grad_d + i : nullptr;
    fit_image<T, MAXPASS, false>(im, a, smem);
  }
}

// Shared memory of the fit for codebooks up to m_max: the padded scaled
// codebook, the per-wave pair sums and the reduction scratch.
static size_t fit_smem(int m_max) {
  return ((size_t)fit_codebook_len(m_max) + (size_t)m_max * FIT_WAVES) * sizeof(P2) + 12 * sizeof(double) + 64;
}

int fit_passes_of(int M) { return fit_passes(M); }

static int maxpass_bound(int np) { return np <= 1 ? 1 : (np <= 2 ? 2 : 4); }
static int maxpass_for(int m_max) { return maxpass_bound(fit_passes(m_max)); }

template <typename T, int MP>
static int fit_occupancy(int m_max) {
  int nb = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fit_batched_kernel<T, MP>, FIT_NT, fit_smem(m_max));
  return e == hipSuccess ? nb : 0;
}

int fit_blocks_per_cu(bool f64, int m_max, int max_passes) {
  switch (maxpass_bound(max_passes)) {
    case 1: return f64 ? fit_occupancy<double, 1>(m_max) : fit_occupancy<float, 1>(m_max);
    case 2: return f64 ? fit_occupancy<double, 2>(m_max) : fit_occupancy<float, 2>(m_max);
    default: return f64 ? fit_occupancy<double, 4>(m_max) : fit_occupancy<float, 4>(m_max);
  }
}

template <typename T, int MP>
static void launch_fit_t(const ImageDesc* d_images, const int32_t* d_sched, const FitArgs& a, int grid,
                         hipStream_t s, const ImageDesc* h_image) {
  if (h_image)
    hipLaunchKernelGGL((fit_image_kernel<T, MP>), dim3(1), dim3(FIT_NT), fit_smem(h_image->M), s, *h_image, a);
  else
    hipLaunchKernelGGL((fit_batched_kernel<T, MP>), dim3(grid), dim3(FIT_NT), fit_smem(a.m_max), s, d_images,
                       d_sched, a);
}

hipError_t launch_fit(bool f64, const ImageDesc* d_images, const int32_t* d_sched, const FitArgs& a,
                      int grid, hipStream_t s, const ImageDesc* h_image) {
  // passes are bounded by the largest codebook of the launch (in the
  // gradient-only mode as well, which runs the same per-image code)
  switch (h_image ? maxpass_for(h_image->M) : (a.max_passes > 0 ? maxpass_bound(a.max_passes) : 4)) {
    case 1:
      f64 ? launch_fit_t<double, 1>(d_images, d_sched, a, grid, s, h_image)
          : launch_fit_t<float, 1>(d_images, d_sched, a, grid, s, h_image);
      break;
    case 2:
      f64 ? launch_fit_t<double, 2>(d_images, d_sched, a, grid, s, h_image)
          : launch_fit_t<float, 2>(d_images, d_sched, a, grid, s, h_image);
      break;
    default:
      f64 ? launch_fit_t<double, 4>(d_images, d_sched, a, grid, s, h_image)
          : launch_fit_t<float, 4>(d_images, d_sched, a, grid, s, h_image);
      break;
  }
  return hipGetLastError();
}

}  // namespace itc
