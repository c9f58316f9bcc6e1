// General-length kernels: the transverse passes and the fused line stages for
// every length whose factors group into two or three radices up to 23, with
// run-time sizes, for one instance or a whole batch in one launch per stage.
//
//   k_gtr_x1    DFT over the first detector axis, real input, half spectrum
//   k_gtr_x2    DFT over the second detector axis (either direction, in place)
//   k_gtr_c2r   inverse DFT over the first axis from the half spectrum
//   k_gline2    a2 + a3 + inverse depth DFT (R, A^T)
//   k_gline1    depth DFT + spreading + transposed a2 (R^T, A)
//
// Every FFT is a GFft (pat_internal.h): each stage loads one butterfly's
// points into registers, transforms them with a fully unrolled R-point DFT
// whose roots are compile-time constants, and writes them back; the first
// stage of a pass reads from memory and the last one writes to memory, so a
// two-stage length crosses LDS once.  The last stage has no twiddles, and the
// plan puts the large primes there.
#include "general.h"
#include "linepair.h"

namespace pat {

// ---------------------------------------------------------------------------
// Transverse passes: tiles of tb columns (a power of two; the contiguous t or
// z axis) by the full transform length; lanes run along the columns.

// Twiddled first stage: the rows come from load(row), and go to buf.
template <typename T, typename Load>
__device__ __forceinline__ void gtr_first(CFft& g, cx<T>* buf, const cx<T>* tw, int ltb, Load load) {
  const int tb = 1 << ltb, total = g.sub0 << ltb;
  with_tw_radix(g.r0, [&](auto tag) {
    constexpr int R = decltype(tag)::v;
#pragma unroll 1
    for (int id = threadIdx.x; id < total; id += (int)blockDim.x) {
      const int col = id & (tb - 1), j = id >> ltb;
      cx<T> v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = load(j + r * g.sub0, col);
      // point d2 rl + e of sub-transform r: row r bs + d2 rlp + e
      cx<T>* p = buf + ((j + fdiv(j, g.m_rl) * (g.rlp - g.rl)) << ltb) + col;
      const int st = g.bs << ltb;
      dft_emit<T, R>(v, [&](int d, cx<T> x) { p[d * st] = d ? cmul(x, tw[j * d]) : x; });
    }
  });
  __syncthreads();
}

// Twiddled middle stage, in place (three-stage lengths).
template <typename T>
__device__ __forceinline__ void gtr_mid(CFft& g, cx<T>* buf, const cx<T>* tw, int ltb) {
  if (g.r1 == 1) return;
  const int tb = 1 << ltb, total = (g.r0 * g.rl) << ltb;
  with_tw_radix(g.r1, [&](auto tag) {
    constexpr int R = decltype(tag)::v;
#pragma unroll 1
    for (int id = threadIdx.x; id < total; id += (int)blockDim.x) {
      const int col = id & (tb - 1), bf = id >> ltb;
      const int blk = fdiv(bf, g.m_rl), j = bf - blk * g.rl;
      cx<T>* p = buf + ((blk * g.bs + j) << ltb) + col;
      const int st = g.rlp << ltb;
      cx<T> v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = p[r * st];
      dft_emit<T, R>(v, [&](int d, cx<T> x) { p[d * st] = d ? cmul(x, tw[j * d * g.r0]) : x; });
    }
  });
  __syncthreads();
}

// Last stage: store(k, col, X_k) receives every output.
template <typename T, typename Store>
__device__ __forceinline__ void gtr_last(CFft& g, const cx<T>* buf, int ltb, Store store) {
  const int tb = 1 << ltb, total = g.nbl << ltb;
  with_last_radix(g.rl, [&](auto tag) {
    constexpr int R = decltype(tag)::v;
#pragma unroll 1
    for (int id = threadIdx.x; id < total; id += (int)blockDim.x) {
      const int col = id & (tb - 1), bf = id >> ltb;
      const int d1 = fdiv(bf, g.m_r1), d2 = bf - d1 * g.r1;
      const cx<T>* p = buf + ((d1 * g.bs + d2 * g.rlp) << ltb) + col;
      cx<T> v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = p[r << ltb];
      const int k0 = d1 + g.r0 * d2;
      dft_emit<T, R>(v, [&](int r, cx<T> x) { store(k0 + r * g.nbl, col, x); });
    }
  });
}

__host__ __device__ __forceinline__ int capped(int v, int cap) { return cap && cap < v ? cap : v; }

template <typename T>
constexpr int gtr_waves() { return sizeof(T) == 4 ? 4 : 2; }

// Loop over the items of a persistent grid: item, its instance I and its index
// li within the instance; `fresh` when the instance differs from the last.
#define PAT_G_ITEMS(a)                                                             \
  int cur_ = -1;                                                                   \
  for (int it_ = blockIdx.x; it_ < (a).total; it_ += gridDim.x) {                  \
    const int item = xcd_item(it_, (a).total);                                     \
    const int inst = __builtin_amdgcn_readfirstlane(find_inst(a, item));           \
    const bool fresh = inst != cur_;                                               \
    cur_ = inst;                                                                   \
    CInst& I = *(CInst*)(a).inst[inst];                                              \
    const int li = item - (a).off[inst];

template <typename T>
__device__ __forceinline__ void g_roots(cx<T>* dst, CInst& I, CFft& g) {
  const cx<T>* src = static_cast<const cx<T>*>(I.tw) + g.tw;
  for (int e = threadIdx.x; e < g.L; e += (int)blockDim.x) dst[e] = src[e];
}

// Cut-off weights of one column x2 of the data-side passes: the slice
// W[b1][b(x2)][b3] in LDS, and the weights of the samples t and t + 1 of row x
// (see cut_slice, cut_pair).
template <typename T>
__device__ __forceinline__ void g_cut_slice(CInst& I, T* ws, int x2) {
  const int E = I.cut_e, e1 = E + 1, b2 = I.n2 > 1 ? cut_band(x2, I.n2, E) : E;
  const T* W = static_cast<const T*>(I.cutw);
  for (int e = threadIdx.x; e < e1 * e1; e += (int)blockDim.x) {
    const int b1 = e / e1, b3 = e - b1 * e1;
    ws[e] = W[(b1 * e1 + b2) * e1 + b3];
  }
}
template <typename T>
__device__ __forceinline__ cx<T> g_cut(CInst& I, const T* ws, int x, int t, int len, cx<T> v) {
  const T* w = ws + cut_band(x, I.n1, I.cut_e) * (I.cut_e + 1);
  return mk(v.x * w[cut_band(t, len, I.cut_e)], v.y * w[cut_band(t + 1, len, I.cut_e)]);
}

template <typename T, bool CUT>
__global__ __launch_bounds__(kBlock, gtr_waves<T>()) void k_gtr_x1(StageArgs a) {
  PAT_G_ITEMS(a)
  CFft& g = I.g1;
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = tw + g.L;
  const int len = a.len_nz ? I.nz : I.nt;  // even
  const int tb = capped(I.gtb1, a.tb_cap), ltb = __builtin_ctz((unsigned)tb);
  const int ntile = (len + 2 * tb - 1) / (2 * tb);
  const int x2 = li / ntile;
  const bool cut = CUT && I.cut_e;
  T* cws = reinterpret_cast<T*>(buf + g.rows * tb);
  __syncthreads();
  if (fresh) g_roots(tw, I, g);
  if (cut) g_cut_slice(I, cws, x2);
  if (fresh || cut) __syncthreads();
  const int t0 = (li - x2 * ntile) * 2 * tb;
  const size_t base = (size_t)x2 * len + t0;
  const cx<T>* in = reinterpret_cast<const cx<T>*>(static_cast<const T*>(a.in[inst]) + base);
  cx<T>* out = static_cast<cx<T>*>(a.out[inst]) + base;
  const uint32_t row = (uint32_t)(I.n2 * len) * (uint32_t)sizeof(T);  // bytes of a real row
  const int w = (len - t0) >> 1;  // columns of this tile
  // complex column b holds the samples t0 + 2b (real part) and t0 + 2b + 1
  gtr_first<T>(g, buf, tw, ltb, [&](int x, int b) {
    const cx<T> v = b < w ? ld_cx<T, true>(at_off(in, (uint32_t)x * row + (uint32_t)b * (uint32_t)sizeof(cx<T>)))
                          : mk(T(0), T(0));
    return cut ? g_cut(I, cws, x, min(t0 + 2 * b, len - 2), len, v) : v;
  });
  gtr_mid<T>(g, buf, tw, ltb);
  // in place: output r of a butterfly goes to the row its input r came from
  with_last_radix(g.rl, [&](auto tag) {
    constexpr int R = decltype(tag)::v;
#pragma unroll 1
    for (int id = threadIdx.x; id < (g.nbl << ltb); id += (int)blockDim.x) {
      const int col = id & (tb - 1), bf = id >> ltb;
      const int d1 = fdiv(bf, g.m_r1), d2 = bf - d1 * g.r1;
      cx<T>* p = buf + ((d1 * g.bs + d2 * g.rlp) << ltb) + col;
      cx<T> v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = p[r << ltb];
      dft_emit<T, R>(v, [&](int r, cx<T> x) { p[r << ltb] = x; });
    }
  });
  __syncthreads();
  // The transforms of the two samples: bin k of the columns' transform Z and
  // the conjugate of bin L - k give pa and pb.  A thread walks the outputs
  // k = n + d nbl of one butterfly n and the outputs of its mirror butterfly
  // (their LDS rows differ by one per step).
  const int nb = g.nbl << ltb, half = g.L / 2;
  const int nq = nb < (int)blockDim.x ? (int)blockDim.x / nb : 1;  // threads per butterfly
  for (int id = threadIdx.x; id < nb * nq; id += (int)blockDim.x) {
    const int b = id & (tb - 1), q = fdiv(id >> ltb, g.m_nbl), n = (id >> ltb) - q * g.nbl;
    if (b >= w) continue;
    const int nm = n ? g.nbl - n : 0;
    const int e2 = fdiv(n, g.m_r0), f2 = fdiv(nm, g.m_r0);
    const cx<T>* own = buf + (((n - e2 * g.r0) * g.bs + e2 * g.rlp) << ltb) + b;
    const cx<T>* mir = buf + (((nm - f2 * g.r0) * g.bs + f2 * g.rlp) << ltb) + b;
    const uint32_t ob = (uint32_t)b * (uint32_t)(2 * sizeof(cx<T>));
    for (int d = q; n + d * g.nbl <= half; d += nq) {
      const int k = n + d * g.nbl;
      const int dm = n ? g.rl - 1 - d : d ? g.rl - d : 0;
      const cx<T> z = own[d << ltb], zn = cconj(mir[dm << ltb]);
      const T h = T(0.5);
      const cx<T> pa = cscl(cadd(z, zn), h);
      const cx<T> df = csub(z, zn);
      const cx<T> pb = mk(h * df.y, -h * df.x);
      st_pair(at_off(out, (uint32_t)k * (2 * row) + ob), pa, pb);
    }
  }
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock, gtr_waves<T>()) void k_gtr_x2(StageArgs a) {
  PAT_G_ITEMS(a)
  CFft& g = I.g2;
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = tw + g.L;
  __syncthreads();
  if (fresh) {
    g_roots(tw, I, g);
    __syncthreads();
  }
  const int len = a.len_nz ? I.nz : I.nt;
  const int tb = capped(I.gtb2, a.tb_cap), ltb = __builtin_ctz((unsigned)tb);
  const int ntile = (len + tb - 1) / tb;
  const int k1 = li / ntile;
  const int t0 = (li - k1 * ntile) * tb;
  cx<T>* io = static_cast<cx<T>*>(a.out[inst]) + (size_t)k1 * I.n2 * len + t0;
  const uint32_t row = (uint32_t)len * (uint32_t)sizeof(cx<T>);
  const int w = len - t0;
  const T sg = a.mode != 0 ? T(-1) : T(1);  // the inverse as conj(FFT(conj(.)))
  gtr_first<T>(g, buf, tw, ltb, [&](int x, int b) {
    const cx<T> v = b < w ? *at_off(io, (uint32_t)x * row + (uint32_t)b * (uint32_t)sizeof(cx<T>)) : mk(T(0), T(0));
    return mk(v.x, sg * v.y);
  });
  gtr_mid<T>(g, buf, tw, ltb);
  gtr_last<T>(g, buf, ltb, [&](int k, int b, cx<T> v) {
    if (b < w) *at_off(io, (uint32_t)k * row + (uint32_t)b * (uint32_t)sizeof(cx<T>)) = mk(v.x, sg * v.y);
  });
  }
}

template <typename T, bool CUT>
__global__ __launch_bounds__(kBlock, gtr_waves<T>()) void k_gtr_c2r(StageArgs a) {
  PAT_G_ITEMS(a)
  CFft& g = I.g1;
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = tw + g.L;
  const int len = a.len_nz ? I.nz : I.nt;
  const int tb = capped(I.gtb1, a.tb_cap), ltb = __builtin_ctz((unsigned)tb);
  const int ntile = (len + 2 * tb - 1) / (2 * tb);
  const int x2 = li / ntile;
  const bool cut = CUT && I.cut_e;
  T* cws = reinterpret_cast<T*>(buf + g.rows * tb);
  __syncthreads();
  if (fresh) g_roots(tw, I, g);
  if (cut) g_cut_slice(I, cws, x2);
  if (fresh || cut) __syncthreads();
  const int t0 = (li - x2 * ntile) * 2 * tb;
  const size_t base = (size_t)x2 * len + t0;
  const cx<T>* in = static_cast<const cx<T>*>(a.in[inst]) + base;
  cx<T>* out = reinterpret_cast<cx<T>*>(static_cast<T*>(a.out[inst]) + base);
  const uint32_t row = (uint32_t)(I.n2 * len) * (uint32_t)sizeof(T);
  const int w = (len - t0) >> 1, half = g.L / 2;
  gtr_first<T>(g, buf, tw, ltb, [&](int k, int b) {
    // Z = X_a + i X_b of two neighbouring samples, stored conjugated; bins
    // above n1/2 are the conjugates of their mirror bins, and the imaginary
    // parts of the bins 0 and n1/2 are dropped (the real part of the inverse)
    const int src = k <= half ? k : g.L - k;
    cx<T> xa = mk(T(0), T(0)), xb = mk(T(0), T(0));
    if (b < w) ld_pair(at_off(in, (uint32_t)src * (2 * row) + (uint32_t)b * (uint32_t)(2 * sizeof(cx<T>))), &xa, &xb);
    const T sg = k == 0 || k == half ? T(0) : k > half ? T(-1) : T(1);
    // (multiplied only where a sign is wanted: 0 times an infinite part would
    // not be 0)
    const T ya = sg == T(0) ? T(0) : sg * xa.y, yb = sg == T(0) ? T(0) : sg * xb.y;
    return mk(xa.x - yb, -(ya + xb.x));
  });
  gtr_mid<T>(g, buf, tw, ltb);
  gtr_last<T>(g, buf, ltb, [&](int x, int b, cx<T> v) {
    cx<T> y = mk(v.x, -v.y);
    if (cut) y = g_cut(I, cws, x, min(t0 + 2 * b, len - 2), len, y);
    if (b < w) st_cx<T, true>(at_off(out, (uint32_t)x * row + (uint32_t)b * (uint32_t)sizeof(cx<T>)), y);
  });
  }
}

// ---------------------------------------------------------------------------
// Line stages, on line pairs (linepair.h).  2D plans have no mirror lines: a
// "pair" is one line there, its second half zero.

// The roots of the middle stage for tw_powers in LDS: butterfly j takes the powers d of
// root 8 j, d = 1, 4, 2, 3, 8, 12 in row 0 .. 5 as far as r1 asks for them (tw8_rows).
__device__ __forceinline__ constexpr int tw8_row(int d) { return d == 1 ? 0 : d == 4 ? 1 : d < 4 ? d : d / 4 + 2; }
template <typename T>
__device__ __forceinline__ void grid_roots(CFft& g, cx<T>* tw8, const cx<T>* tm) {
  for (int e = threadIdx.x; e < kTw8 * tw8_rows(g.r1, (int)sizeof(cx<T>)); e += (int)blockDim.x) {
    const int row = e / kTw8, j = e % kTw8;
    const int d = row == 0 ? 1 : row == 1 ? 4 : row < 4 ? row : 4 * (row - 2);
    if (j < g.rl) tw8[e] = tm[8 * j * d];
  }
}

// (tw8: see grid_roots)
template <typename T>
__device__ __forceinline__ void grid_mid(CFft& g, px<T>* buf, const cx<T>* tw8, int np) {
  const int NT = blockDim.x;
  auto run = [&](auto tag) {
    constexpr int R = decltype(tag)::v;
#pragma unroll 1
    for (int id = threadIdx.x; id < np * 8 * g.rl; id += NT) {
      const int p = fdiv(id, g.m_nb1), q = id - p * (8 * g.rl);
      const int blk = fdiv(q, g.m_rl), j = q - blk * g.rl;
      px<T>* s = buf + p * g.rows + blk * g.bs + j;
      if constexpr (R * sizeof(T) <= 32) {
        px<T> v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = s[r * g.rlp];
        dft_px<T, R>(v);
        twiddle_px<T, R>(v, [&](int d) { return tw8[kTw8 * tw8_row(d) + j]; });
#pragma unroll
        for (int r = 0; r < R; ++r) s[r * g.rlp] = v[r];
      } else {
        // (both halves at once would not fit in registers)
#pragma unroll 1
        for (int h = 0; h < 2; ++h) {
          cx<T>* c = h ? &s->b : &s->a;
          cx<T> v[R];
#pragma unroll
          for (int r = 0; r < R; ++r) v[r] = c[2 * r * g.rlp];
          dft_reg<T, R>(v);
          twiddle_reg<T, R>(v, [&](int d) { return tw8[kTw8 * tw8_row(d) + j]; });
#pragma unroll
          for (int r = 0; r < R; ++r) c[2 * r * g.rlp] = v[r];
        }
      }
    }
  };
  switch (g.r1) {
    case 2: run(RadixTag<2>{}); break;
    case 4: run(RadixTag<4>{}); break;
    case 8: run(RadixTag<8>{}); break;
    case 16: run(RadixTag<16>{}); break;
    default: return;
  }
  __syncthreads();
}

// Last grid stage over the natural digits n = d1 + 8 d2 of the butterflies, so
// that the lanes' outputs k = n + d nbl are neighbours.
template <typename F>
__device__ __forceinline__ void with_grid_radix(int r, F f) {
  switch (r) {
    PAT_CASE(8) PAT_CASE(10) PAT_CASE(12) PAT_CASE(14) PAT_CASE(16)
    default: break;
  }
}
// In place to natural order (line p at p * rows): at most one butterfly per
// thread (np nbl <= NT), whose outputs wait in registers until every thread
// has read its inputs.
template <typename T>
__device__ __forceinline__ void grid_last_natural(CFft& g, px<T>* buf, int np) {
  with_grid_radix(g.rl, [&](auto tag) {
    constexpr int R = decltype(tag)::v;
    const int id = threadIdx.x, lnb = __builtin_ctz((unsigned)g.nbl);
    const int p = id >> lnb, n = id & (g.nbl - 1);
    px<T> v[R];
    if (p < np) {
      const px<T>* s = buf + p * g.rows + (n & 7) * g.bs + (n >> 3) * g.rlp;
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = s[r];
      dft_px<T, R>(v);
    }
    __syncthreads();
    if (p < np) {
      px<T>* d = buf + p * g.rows + n;
#pragma unroll
      for (int r = 0; r < R; ++r) d[r * g.nbl] = v[r];
    }
  });
}
// put(p, k, half, X_k) receives the outputs, one half after the other
template <typename T, typename Put>
__device__ __forceinline__ void grid_last_put(CFft& g, const px<T>* buf, int np, Put put) {
  with_grid_radix(g.rl, [&](auto tag) {
    constexpr int R = decltype(tag)::v;
    const int lnb = __builtin_ctz((unsigned)g.nbl);
#pragma unroll 1
    for (int id = threadIdx.x; id < (np << lnb); id += blockDim.x) {
      const int p = id >> lnb, n = id & (g.nbl - 1);
      const px<T>* s = buf + p * g.rows + (n & 7) * g.bs + (n >> 3) * g.rlp;
      bfly_px<T, R>([&](int r, int h) { return h ? s[r].b : s[r].a; }, [&](int, cx<T> v) { return v; },
                    [&](int r, int h, cx<T> v) { put(p, n + r * g.nbl, h, v); });
    }
  });
}

// Depth FFT (any radices) over np pairs, point i of pair p in row(i) at
// p * rows.  One butterfly of one line per thread, the two lines of a pair in
// neighbouring lanes: a depth line has few butterflies of a large radix (8 of
// radix 23 at nz = 184), so the lines, not the pairs, fill the lanes.
template <typename T, typename Get>
__device__ __forceinline__ void depth_first(CFft& g, px<T>* z, const cx<T>* tw, int np, Get get) {
  const int NT = blockDim.x;
  with_tw_radix(g.r0, [&](auto tag) {
    constexpr int R = decltype(tag)::v;
#pragma unroll 1
    for (int id = threadIdx.x; id < 2 * np * g.sub0; id += NT) {
      const int h = id & 1, p = fdiv(id >> 1, g.m_sub0), j = (id >> 1) - p * g.sub0;
      cx<T>* s = reinterpret_cast<cx<T>*>(z + p * g.rows + j + fdiv(j, g.m_rl) * (g.rlp - g.rl)) + h;
      cx<T> v[R];
      get(p, h, j, s, v, tag);
      dft_emit<T, R>(v, [&](int d, cx<T> x) { s[2 * d * g.bs] = d ? cmul(x, tw[j * d]) : x; });
    }
  });
  __syncthreads();
}
template <typename T>
__device__ __forceinline__ void depth_mid(CFft& g, px<T>* z, const cx<T>* tw, int np) {
  if (g.r1 == 1) return;
  const int NT = blockDim.x;
  with_tw_radix(g.r1, [&](auto tag) {
    constexpr int R = decltype(tag)::v;
#pragma unroll 1
    for (int id = threadIdx.x; id < 2 * np * g.r0 * g.rl; id += NT) {
      const int h = id & 1, p = fdiv(id >> 1, g.m_nb1), q = (id >> 1) - p * (g.r0 * g.rl);
      const int blk = fdiv(q, g.m_rl), j = q - blk * g.rl;
      cx<T>* s = reinterpret_cast<cx<T>*>(z + p * g.rows + blk * g.bs + j) + h;
      cx<T> v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = s[2 * r * g.rlp];
      dft_emit<T, R>(v, [&](int d, cx<T> x) { s[2 * d * g.rlp] = d ? cmul(x, tw[j * d * g.r0]) : x; });
    }
  });
  __syncthreads();
}
// sink(p, half, n, d, X_k) receives output k = n + d nbl; neighbouring lanes
// hold neighbouring n
template <typename T, typename Sink>
__device__ __forceinline__ void depth_last(CFft& g, const px<T>* z, int np, Sink sink) {
  const int NT = blockDim.x;
  with_last_radix(g.rl, [&](auto tag) {
    constexpr int R = decltype(tag)::v;
#pragma unroll 1
    for (int id = threadIdx.x; id < 2 * np * g.nbl; id += NT) {
      const int h = id & 1, p = fdiv(id >> 1, g.m_nbl), n = (id >> 1) - p * g.nbl;
      const int d2 = fdiv(n, g.m_r0), d1 = n - d2 * g.r0;
      const cx<T>* s = reinterpret_cast<const cx<T>*>(z + p * g.rows + d1 * g.bs + d2 * g.rlp) + h;
      cx<T> v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = s[2 * r];
      auto put = sink(p, h, n);
      dft_emit<T, R>(v, [&](int d, cx<T> x) { put(d, x); });
    }
  });
}

// Sums of one window over both lines of a pair: +nup at up, -nup at un.
template <typename T, bool REV>
__device__ __forceinline__ void gpair_sums(const px<T>* up, const px<T>* un, const PairWin<T, kGTaps>& pw, px<T>* sp,
                                           px<T>* sn) {
#pragma unroll
  for (int t = 0; t < kGTaps; ++t) {
    const px<T> g = up[t], h = un[t];
    const T w = pw.w[t], b = REV ? pw.w[kGTaps - 1 - t] : bitsel(pw.on, pw.w[t], pw.w[kGTaps - 1 - t]);
    sp->a.x += w * g.a.x;
    sp->a.y += w * g.a.y;
    sp->b.x += w * g.b.x;
    sp->b.y += w * g.b.y;
    sn->a.x += b * h.a.x;
    sn->a.y += b * h.a.y;
    sn->b.x += b * h.b.x;
    sn->b.y += b * h.b.y;
  }
}
template <typename T>
__device__ __forceinline__ void gpair_values(const px<T>* U, int m, const PairWin<T, kGTaps>& pw, px<T>* vp,
                                             px<T>* vn) {
  const cx<T> z = mk(T(0), T(0));
  px<T> sp{z, z}, sn{z, z};
  if (pw.jp <= m - kGTaps && pw.jn <= m - kGTaps) {
    if (__any(pw.on)) gpair_sums<T, false>(U + pw.jp, U + pw.jn, pw, &sp, &sn);
    else gpair_sums<T, true>(U + pw.jp, U + pw.jn, pw, &sp, &sn);
  } else {
    // a window runs past the end of the line: wrap its taps
#pragma unroll
    for (int t = 0; t < kGTaps; ++t) {
      int jp = pw.jp + t, jn = pw.jn + t;
      jp -= jp >= m ? m : 0;
      jn -= jn >= m ? m : 0;
      const px<T> g = U[jp], h = U[jn];
      const T w = pw.w[t], b = bitsel(pw.on, pw.w[t], pw.w[kGTaps - 1 - t]);
      sp.a.x += w * g.a.x;
      sp.a.y += w * g.a.y;
      sp.b.x += w * g.b.x;
      sp.b.y += w * g.b.y;
      sn.a.x += b * h.a.x;
      sn.a.y += b * h.a.y;
      sn.b.x += b * h.b.x;
      sn.b.y += b * h.b.y;
    }
  }
  const cx<T> cp = cconj(pw.ph);
  vp->a = cmul(sp.a, pw.ph);
  vp->b = cmul(sp.b, pw.ph);
  vn->a = cmul(sn.a, cp);
  vn->b = cmul(sn.b, cp);
}

// pair_window on the internal grid of m points (c_g of them per time bin)
template <typename T>
__device__ __forceinline__ void gpair_window(double nup, double c_g, double ck, const StageArgs& a, int m,
                                             double inv_m, PairWin<T, kGTaps>& pw) {
  pw.ph = phase_mpi<T>(nup);
  int j0;
  const double d = tap_origin(c_g * nup, ck, &j0);
  tap_weights_pairs<T, kGTaps>(a, (T)(2.0 * d + 1.0), pw.w);
  pw.on = d == -1.0;
  pw.jp = wrap_tap<false>(j0, m, inv_m);
  pw.jn = wrap_tap<false>(pw.on ? -(j0 + kGTaps - 2) : -(j0 + kGTaps - 1), m, inv_m);
}

template <typename T>
constexpr int gline_waves() { return sizeof(T) == 4 ? 3 : 2; }

// R and A^T: per item np line pairs.  The first grid stage takes its nonzero
// inputs (the centred samples: with m >= 2 nt only the inputs 0, 1, 6, 7 of
// a radix-8 butterfly) from registers that were loaded during the previous
// item; the last stage brings the grid to natural order in place; the node
// values go to a region of their own, whose depth FFT writes its outputs to
// memory.
template <typename T>
__global__ __launch_bounds__(kBlock, gline_waves<T>()) void k_gline2(StageArgs a) {
  const int NT = blockDim.x, tid = threadIdx.x;
  px<T>* buf = reinterpret_cast<px<T>*>(pat_smem);
  const cx<T> zero = mk(T(0), T(0));
  px<T> pre[4];
  // sample of input i of first-stage butterfly j: position j + {0, 1, 6, 7} S
  // holds sample (position + nt/2) mod m
  auto sample = [&](CInst& I, int j, int i) {
    const int S = I.gm.sub0;
    return i < 2 ? j + i * S + I.nt / 2 : j + (4 + i) * S - I.gm.L + I.nt / 2;
  };
  auto fetch = [&](int item) {
    const int inst = __builtin_amdgcn_readfirstlane(find_inst(a, item));
    CInst& I = *(CInst*)a.inst[inst];
    const int p = fdiv(tid, I.gm.m_sub0), j = tid - p * I.gm.sub0, np = capped(I.np, a.np_cap);
    const int P = (item - a.off[inst]) * np + p;
    const bool ok = p < np && P < I.npair;
    const PairLines q = pair_lines(I, ok ? P : 0);
    const cx<T>* in = static_cast<const cx<T>*>(a.in[inst]);
    const uint32_t oa = (uint32_t)q.la * (uint32_t)I.nt, ob = (uint32_t)(q.lb < 0 ? 0 : q.lb) * (uint32_t)I.nt;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int n = sample(I, j, i);
      const bool in_range = ok && n >= 0 && n < I.nt;
      pre[i].a = in_range ? *at_off(in, (oa + (uint32_t)n) * (uint32_t)sizeof(cx<T>)) : zero;
      pre[i].b = in_range && q.lb >= 0 ? *at_off(in, (ob + (uint32_t)n) * (uint32_t)sizeof(cx<T>)) : zero;
    }
  };
  int cur = -1;
  T snr[4] = {T(0), T(0), T(0), T(0)};
  cx<T> w1 = zero, w4 = zero;  // first-stage roots (FP64: w1)
  int item = blockIdx.x;
  if (item < a.total) fetch(item);
  for (; item < a.total; item += gridDim.x) {
    const int inst = __builtin_amdgcn_readfirstlane(find_inst(a, item));
    CInst& I = *(CInst*)a.inst[inst];
    CFft &g = I.gm, &gz = I.gz;
    const int m = g.L, nz = I.nz, half = nz / 2, np = capped(I.np, a.np_cap);
    px<T>* dz = buf + np * g.rows;
    cx<T>* twz = reinterpret_cast<cx<T>*>(dz + np * gz.rows);
    cx<T>* tw8 = twz + nz;
    const int p0 = fdiv(tid, g.m_sub0), j0 = tid - p0 * g.sub0;
    if (inst != cur) {
      __syncthreads();
      const cx<T>* tz = static_cast<const cx<T>*>(I.tw) + gz.tw;
      const cx<T>* tm = static_cast<const cx<T>*>(I.tw) + g.tw;
      for (int e = tid; e < nz; e += NT) twz[e] = tz[e];
      grid_roots(g, tw8, tm);
      const T* sn = static_cast<const T*>(I.sn_g);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int n = sample(I, j0, i);
        snr[i] = n >= 0 && n < I.nt ? sn[n] : T(0);
      }
      w1 = tm[j0];
      if constexpr (sizeof(T) == 4) w4 = tm[4 * j0];
      cur = inst;
      __syncthreads();
    }
    const int P0 = (item - a.off[inst]) * np;
    const int npi = min(np, I.npair - P0);
    if (p0 < np) {
      px<T> v[8];
      const px<T> pz{zero, zero};
      auto in = [&](int i) { return px<T>{cscl(pre[i].a, snr[i]), cscl(pre[i].b, snr[i])}; };
      v[0] = in(0);
      v[1] = in(1);
      v[2] = v[3] = v[4] = v[5] = pz;
      v[6] = in(2);
      v[7] = in(3);
      dft_px<T, 8>(v);
      twiddle_px<T, 8>(v, [&](int d) { return d == 1 ? w1 : w4; });
      px<T>* s = buf + p0 * g.rows + j0 + fdiv(j0, g.m_rl) * (g.rlp - g.rl);
#pragma unroll
      for (int r = 0; r < 8; ++r) s[r * g.bs] = v[r];
    }
    __syncthreads();
    grid_mid<T>(g, buf, tw8, np);
    grid_last_natural<T>(g, buf, np);
    if (item + (int)gridDim.x < a.total) fetch(item + gridDim.x);
    __syncthreads();
    {
      const double inv_m = 1.0 / (double)m, wsc = I.wcoef * I.scale;
      const int per = a.mode == 0 ? half : half + 1;
      const uint32_t mper = a.mode == 0 ? I.m_half : I.m_half1;
#pragma unroll 1
      for (int e = tid; e < npi * per; e += NT) {
        const int p = fdiv(e, mper), la = e - p * per + (a.mode == 0 ? 1 : 0);
        const PairLines q = pair_lines(I, P0 + p);
        const double bl = I.b * (double)la * (double)la;
        const px<T>* U = buf + p * g.rows;
        double nup = sqrt_nt(q.ka + bl);
        // (the weight, halved on the Nyquist lane, rides on the node phase)
        const double wla = a.mode == 0 ? wsc * (double)la * (la < half ? 1.0 : 0.5) : 0.5 * I.scale;
        PairWin<T, kGTaps> pw;
        gpair_window<T>(nup, I.c_g, I.ck, a, m, inv_m, pw);
        pw.ph = cscl(pw.ph, T(a.mode == 0 ? wla * rcp_nt(nup) : wla));
        px<T> vp, vn;
        gpair_values<T>(U, m, pw, &vp, &vn);
        if (!q.shared) {
          nup = sqrt_nt(q.kb + bl);
          gpair_window<T>(nup, I.c_g, I.ck, a, m, inv_m, pw);
          pw.ph = cscl(pw.ph, T(a.mode == 0 ? wla * rcp_nt(nup) : wla));
          px<T> wp, wn;
          gpair_values<T>(U, m, pw, &wp, &wn);
          vp.b = wp.b;
          vn.b = wn.b;
        }
        // conjugated into the depth FFT's rows (point l in row l + pad)
        px<T>* D = dz + p * gz.rows;
        auto zrow = [&](int l) {
          const int d1 = fdiv(l, gz.m_sub0), rest = l - d1 * gz.sub0;
          return d1 * gz.bs + rest + fdiv(rest, gz.m_rl) * (gz.rlp - gz.rl);
        };
        const px<T> sum{cconj(cadd(vp.a, vn.a)), cconj(cadd(vp.b, vn.b))};
        if (a.mode != 0) {
          D[zrow(la)] = sum;
          if (la > 0 && la < half) D[zrow(nz - la)] = sum;
        } else if (la < half) {
          D[zrow(la)] = px<T>{cconj(vp.a), cconj(vp.b)};
          D[zrow(nz - la)] = px<T>{cconj(vn.a), cconj(vn.b)};
        } else {
          D[zrow(half)] = sum;
          D[0] = px<T>{zero, zero};  // l = 0 has weight 0
        }
      }
    }
    __syncthreads();
    depth_first<T>(gz, dz, twz, npi, [&](int, int, int, const cx<T>* s, cx<T>* v, auto tag) {
#pragma unroll
      for (int r = 0; r < decltype(tag)::v; ++r) v[r] = s[2 * r * gz.bs];
    });
    depth_mid<T>(gz, dz, twz, npi);
    cx<T>* out = static_cast<cx<T>*>(a.out[inst]);
    depth_last<T>(gz, dz, npi, [&](int p, int h, int n) {
      const int line = pair_line(I, P0 + p, h);
      const uint32_t o = ((uint32_t)line * (uint32_t)nz + (uint32_t)n) * (uint32_t)sizeof(cx<T>);
      const uint32_t st = (uint32_t)gz.nbl * (uint32_t)sizeof(cx<T>);
      return [=](int d, cx<T> v) {
        if (line >= 0) *at_off(out, o + (uint32_t)d * st) = cconj(v);
      };
    });
  }
}

// Spreading of an item's npi pairs (depth spectra D in natural order, pair stride
// ds) into their grid lines G (m pair cells, zeroed; pair stride gs).  With more
// waves than pairs, a pair's batches of 64 node pairs go to several waves: they
// form their batches' windows side by side and add them to the grid in turn.
template <typename T>
__device__ __forceinline__ void gspread_item(CInst& I, const StageArgs& a, int P0, int npi, px<T>* G, int gs,
                                             const px<T>* D, int ds) {
  const int L = (int)(threadIdx.x & 63);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), nw = (int)blockDim.x >> 6;
  const int m = I.gm.L, half = I.nz / 2, mode = a.mode;
  const int q0 = mode == 0 ? 1 : 0, nq = half - q0 + 1;
  const double inv_m = 1.0 / (double)m;
  // waves per pair (uniform over the workgroup: barriers depend on it)
  const int wpp = nw >= 2 * npi && nq > 64 ? nw / npi : 1;
  const int i = wave % wpp;
#pragma unroll 1
  for (int p = wave / wpp; p < npi || (wpp > 1 && p < nw); p += nw) {
    const bool mine = p < npi;
    const PairLines q = pair_lines(I, P0 + (mine ? p : 0));
    const px<T>* Dp = D + (mine ? p : 0) * ds;
    const int passes = wpp > 1 || !q.shared ? 2 : 1;
#pragma unroll 1
    for (int t = 0; t < passes; ++t)
#pragma unroll 1
      for (int base0 = 0; base0 < nq; base0 += 64 * wpp) {
        const int base = base0 + 64 * i, nact = min(64, nq - base);
        const bool act = L < nact;
        const int la = act ? q0 + base + L : q0;
        const double nup = sqrt_nt((t ? q.kb : q.ka) + I.b * (double)la * (double)la);
        px<T> qp, qm;
        double cf;
        node_values<T>(I, mode, la, nup, [&](int l) { return Dp[l]; }, &qp, &qm, &cf);
        SpreadBatch<T> b =
            spread_setup<T, 0>(a, I.c_g, I.ck, m, inv_m, nup, cscl(phase_mpi<T>(nup), (T)cf), act, nact, t == 0,
                               q.shared || t == 1, qp, qm);
        const bool some = mine && nact > 0 && (t == 0 || !q.shared);
        // the pair's waves in turn: wave i adds its batch between its i-th and
        // (i+1)-th barrier of wpp
        for (int o = 0; o < i; ++o) __syncthreads();
        if (some) spread_apply<T>(b, m, plane_stride(m), G + p * gs);
        if (wpp > 1) {
          for (int o = i; o < wpp; ++o) __syncthreads();
        }
      }
  }
}

// R^T and A: per item np line pairs.  Their depth DFTs read the spectra from
// memory and leave them in natural order in LDS; wavefronts spread the pairs into
// their grid lines, one each or, where a pair's nodes make two batches, several per
// pair that add theirs in turn (gspread_item); the grid DFTs of all pairs run
// together and the last stage writes the picked, deconvolved samples X_n = s_n
// conj(G_k), k = (n - nt/2) mod m, to memory.
template <typename T>
__global__ __launch_bounds__(kBlock, gline_waves<T>()) void k_gline1(StageArgs a) {
  const int NT = blockDim.x, tid = threadIdx.x;
  px<T>* buf = reinterpret_cast<px<T>*>(pat_smem);
  const cx<T> zero = mk(T(0), T(0));
  PAT_G_ITEMS(a)
  CFft &g = I.gm, &gz = I.gz;
  const int m = g.L, nz = I.nz, nt = I.nt, np = capped(I.np, a.np_cap);
  px<T>* dz = buf + np * g.rows;
  cx<T>* twz = reinterpret_cast<cx<T>*>(dz + np * gz.rows);
  cx<T>* tw8 = twz + nz;
  __syncthreads();
  if (fresh) {
    const cx<T>* tz = static_cast<const cx<T>*>(I.tw) + gz.tw;
    const cx<T>* tm = static_cast<const cx<T>*>(I.tw) + g.tw;
    for (int e = tid; e < nz; e += NT) twz[e] = tz[e];
    grid_roots(g, tw8, tm);
    __syncthreads();
  }
  const int P0 = li * np, npi = min(np, I.npair - P0);
  const cx<T>* in = static_cast<const cx<T>*>(a.in[inst]);
  cx<T>* out = static_cast<cx<T>*>(a.out[inst]);
  // (the depth scratch lies in the grid region, the plan has seen to its size; each
  // pair's natural-order spectra go to dz)
  px<T>* zs = buf;
  depth_first<T>(gz, zs, twz, npi, [&](int p, int h, int j, const cx<T>*, cx<T>* v, auto tag) {
    const int line = pair_line(I, P0 + p, h);
    const uint32_t o = ((uint32_t)line * (uint32_t)nz + (uint32_t)j) * (uint32_t)sizeof(cx<T>);
    const uint32_t st = (uint32_t)gz.sub0 * (uint32_t)sizeof(cx<T>);
#pragma unroll
    for (int r = 0; r < decltype(tag)::v; ++r) {
      v[r] = mk(T(0), T(0));
      if (line >= 0) v[r] = *at_off(in, o + (uint32_t)r * st);
    }
  });
  depth_mid<T>(gz, zs, twz, npi);
  depth_last<T>(gz, zs, npi, [&](int p, int h, int n) {
    cx<T>* D = reinterpret_cast<cx<T>*>(dz + p * gz.rows + n) + h;
    const int st = 2 * gz.nbl;
    return [=](int d, cx<T> v) { D[d * st] = v; };
  });
  __syncthreads();
  for (int e = tid; e < npi * g.rows; e += NT) buf[e] = px<T>{zero, zero};
  __syncthreads();
  gspread_item<T>(I, a, P0, npi, buf, g.rows, dz, gz.rows);
  __syncthreads();
  {
    // first grid stage: from natural order into the padded rows
    const int p0 = fdiv(tid, g.m_sub0), j0 = tid - p0 * g.sub0;
    const bool act = p0 < npi;
    px<T> v[8];
    if (act) {
#pragma unroll
      for (int r = 0; r < 8; ++r) v[r] = buf[p0 * g.rows + plane_cell(j0 + r * g.sub0, plane_stride(m))];
      dft_px<T, 8>(v);
      const cx<T>* tm = static_cast<const cx<T>*>(I.tw) + g.tw;
      twiddle_px<T, 8>(v, [&](int d) { return tm[j0 * d]; });
    }
    __syncthreads();
    if (act) {
      px<T>* s = buf + p0 * g.rows + j0 + fdiv(j0, g.m_rl) * (g.rlp - g.rl);
#pragma unroll
      for (int r = 0; r < 8; ++r) s[r * g.bs] = v[r];
    }
  }
  __syncthreads();
  grid_mid<T>(g, buf, tw8, npi);
  const T* sn = static_cast<const T*>(I.sn_g);
  grid_last_put<T>(g, buf, npi, [&](int p, int k, int h, cx<T> v) {
    int n = k + nt / 2;
    n -= n >= m ? m : 0;
    const int line = pair_line(I, P0 + p, h);
    if (n < nt && line >= 0)
      *at_off(out, ((uint32_t)line * (uint32_t)nt + (uint32_t)n) * (uint32_t)sizeof(cx<T>)) = cscl(cconj(v), sn[n]);
  });
  }
}

// ---------------------------------------------------------------------------
// Launches

namespace {

template <typename Items>
void count_items(StageArgs& a, Items items) {
  a.off[0] = 0;
  for (int i = 0; i < a.n; ++i) a.off[i + 1] = a.off[i] + items(i);
  a.total = a.off[a.n];
  a.counter = nullptr;
}

int cdiv(int x, int y) { return (x + y - 1) / y; }

template <typename T>
size_t cut_bytes(const Inst& I, bool data) {
  return data && I.cut_e ? (size_t)(I.cut_e + 1) * (I.cut_e + 1) * sizeof(T) : 0;
}

// whether this is the data-side pass of an instance with a cut-off
bool any_cut(const StageArgs& a, const Inst* h) {
  bool c = false;
  for (int i = 0; i < a.n && !a.len_nz; ++i) c = c || h[i].cut_e;
  return c;
}

template <typename F>
size_t max_bytes(int n, F f) {
  size_t mx = 0;
  for (int i = 0; i < n; ++i) mx = f(i) > mx ? f(i) : mx;
  return mx;
}

// A single instance too small to give every CU an item takes narrower tiles
// (down to two columns) and fewer pairs per item: its time is the latency of
// one item.  `items(w)` counts the items at width w.
template <typename Items>
int spread_out(int n, int w, int least, Items items) {
  if (n != 1) return 0;
  const int full = w;
  while (w > least && items(w) < num_cu()) w = (w + 1) / 2;
  return w < full ? w : 0;
}

// Threads of a transverse pass: one per butterfly of its larger outer stage,
// at most kBlock.
int gtr_threads(int n, const GFft& g, int tb) {
  if (n != 1) return kBlock;
  const int most = (g.sub0 > g.nbl ? g.sub0 : g.nbl) * tb;
  return most >= kBlock ? kBlock : (most + 63) / 64 * 64;
}

}  // namespace

template <typename T>
hipError_t General<T>::x1(StageArgs& a, const Inst* h, hipStream_t st, StageTimer* tm) {
  auto tiles = [&](int i, int tb) { return h[i].n2 * cdiv(a.len_nz ? h[i].nz : h[i].nt, 2 * tb); };
  a.tb_cap = spread_out(a.n, h[0].gtb1, 2, [&](int tb) { return tiles(0, tb); });
  auto tb = [&](int i) { return capped(h[i].gtb1, a.tb_cap); };
  count_items(a, [&](int i) { return tiles(i, tb(i)); });
  const size_t shm =
      max_bytes(a.n, [&](int i) { return lds_gtile(h[i].g1, tb(i), sizeof(cx<T>)) + cut_bytes<T>(h[i], !a.len_nz); });
  const int nt = gtr_threads(a.n, h[0].g1, tb(0));
  if (any_cut(a, h)) return launch_persistent(k_gtr_x1<T, true>, "dft_x1", a, shm, st, tm, nt);
  return launch_persistent(k_gtr_x1<T, false>, "dft_x1", a, shm, st, tm, nt);
}

template <typename T>
hipError_t General<T>::x2(StageArgs& a, const Inst* h, hipStream_t st, StageTimer* tm) {
  auto tiles = [&](int i, int tb) { return h[i].n2 > 1 ? h[i].h1 * cdiv(a.len_nz ? h[i].nz : h[i].nt, tb) : 0; };
  a.tb_cap = spread_out(a.n, h[0].gtb2, 2, [&](int tb) { return tiles(0, tb); });
  auto tb = [&](int i) { return capped(h[i].gtb2, a.tb_cap); };
  count_items(a, [&](int i) { return tiles(i, tb(i)); });
  const size_t shm = max_bytes(a.n, [&](int i) { return h[i].n2 > 1 ? lds_gtile(h[i].g2, tb(i), sizeof(cx<T>)) : 0; });
  return launch_persistent(k_gtr_x2<T>, a.mode ? "idft_x2" : "dft_x2", a, shm, st, tm, gtr_threads(a.n, h[0].g2, tb(0)));
}

template <typename T>
hipError_t General<T>::c2r(StageArgs& a, const Inst* h, hipStream_t st, StageTimer* tm) {
  auto tiles = [&](int i, int tb) { return h[i].n2 * cdiv(a.len_nz ? h[i].nz : h[i].nt, 2 * tb); };
  a.tb_cap = spread_out(a.n, h[0].gtb1, 2, [&](int tb) { return tiles(0, tb); });
  auto tb = [&](int i) { return capped(h[i].gtb1, a.tb_cap); };
  count_items(a, [&](int i) { return tiles(i, tb(i)); });
  const size_t shm =
      max_bytes(a.n, [&](int i) { return lds_gtile(h[i].g1, tb(i), sizeof(cx<T>)) + cut_bytes<T>(h[i], !a.len_nz); });
  const int nt = gtr_threads(a.n, h[0].g1, tb(0));
  if (any_cut(a, h)) return launch_persistent(k_gtr_c2r<T, true>, "idft_x1_c2r", a, shm, st, tm, nt);
  return launch_persistent(k_gtr_c2r<T, false>, "idft_x1_c2r", a, shm, st, tm, nt);
}

// Pairs per item (a cap for one instance), LDS and threads (at least one first-stage
// butterfly each) of a line kernel.
struct GlineShape {
  int np_cap, threads;
  size_t shm;
};
static GlineShape gline_shape(int n, const Inst* h, size_t cs, bool spread) {
  GlineShape g;
  g.np_cap = spread_out(n, h[0].np, 1, [&](int np) { return cdiv(h[0].npair, np); });
  auto np = [&](int i) { return capped(h[i].np, g.np_cap); };
  int t = 64;
  for (int i = 0; i < n; ++i) {
    // (spreading: two waves per pair where its nodes make two batches)
    const int s = spread && h[i].nz > 128 ? 128 * np(i) : 0, f = np(i) * h[i].gm.sub0;
    t = s > t && s <= kBlock ? s : t;
    t = f > t ? f : t;
  }
  g.threads = (t + 63) / 64 * 64;
  g.shm = max_bytes(n, [&](int i) { return lds_gline(h[i], np(i), cs); });
  return g;
}
static void gline_items(StageArgs& a, const Inst* h, const GlineShape& g) {
  a.np_cap = g.np_cap;
  count_items(a, [&](int i) { return cdiv(h[i].npair, capped(h[i].np, g.np_cap)); });
}

template <typename T>
hipError_t General<T>::line2(StageArgs& a, const Inst* h, hipStream_t st, StageTimer* tm) {
  const GlineShape g = gline_shape(a.n, h, sizeof(cx<T>), false);
  gline_items(a, h, g);
  return launch_persistent(k_gline2<T>, "nufft_fused", a, g.shm, st, tm, g.threads);
}

template <typename T>
hipError_t General<T>::line1(StageArgs& a, const Inst* h, hipStream_t st, StageTimer* tm) {
  const GlineShape g = gline_shape(a.n, h, sizeof(cx<T>), true);
  gline_items(a, h, g);
  return launch_persistent(k_gline1<T>, "nufft_adjoint_fused", a, g.shm, st, tm, g.threads);
}

template <typename T>
double General<T>::line1_rounds(const Inst& h) {
  const GlineShape g = gline_shape(1, &h, sizeof(cx<T>), true);
  hipError_t e = hipSuccess;
  const int res = resident_blocks(reinterpret_cast<const void*>(k_gline1<T>), g.shm, g.threads, &e);
  return e == hipSuccess ? (double)cdiv(h.npair, capped(h.np, g.np_cap)) / (res * num_cu()) : 0.0;
}

template struct General<float>;
template struct General<double>;

}  // namespace pat
