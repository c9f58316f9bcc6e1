// Transverse passes of one instance for lengths of 128, 256 and 512 points, with
// the transform and the tile fixed at compile time.
//
// Each pass is a software pipeline: a persistent grid strides over tiles of TB
// complex columns; a thread holds the first-stage inputs of its butterflies of
// the next tile in registers, loaded while the current tile is finished.  The
// first stage transforms them in registers and writes LDS, the last stage reads
// LDS and writes memory, so a tile crosses LDS once (twice at 512 points) and
// the store needs no position table.  Bound by memory: in place passes over
// data that sit in the 256 MB Infinity Cache reach 7.2 TB/s as a plain copy.
// (Three or four in-place LDS stages between a load into LDS and a permuted
// copy out, which this replaces, moved a tile through LDS five to six times.)
#include "general.h"
#include "regfft.h"

namespace pat {

// Radices, tile width and threads of a length of 2^LL points.  Rows in LDS as
// in GFft: the last digit padded to RLP (odd).
template <typename T, int LL>
struct TrPlan {
  static constexpr bool F = sizeof(T) == 4;
  static constexpr int L = 1 << LL;
  // (FP64 at 256 points in three stages: two of radix 16 take 190 registers)
  static constexpr int R0 = F && LL == 8 ? 16 : 8, R1 = LL == 9 ? 8 : !F && LL == 8 ? 4 : 1, RL = LL == 9 || (!F && LL == 8) ? 8 : 16;
  // 128-byte rows (FP64 at 512 points: 64, or the tile would leave one
  // workgroup per CU)
  static constexpr int TB = F ? 16 : LL == 9 ? 4 : LL == 8 ? 8 : 16;
  static constexpr int NT = F && LL == 9 ? 512 : 256;
  static constexpr int RLP = RL | 1, BS = (R1 * RLP) | 1, SUB0 = R1 * RL, NBL = R0 * R1, ROWS = R0 * BS;
  static constexpr int U = SUB0 * TB / NT;  // first-stage butterflies per thread
  static constexpr int STEP = NT / TB;      // butterflies between two of them
  static_assert(U * NT == SUB0 * TB, "whole butterflies per thread");
  static constexpr int lds = (ROWS * TB + L) * 2 * (int)sizeof(T);
  static constexpr int waves = F ? 4 : LL == 8 ? 3 : 2;
  // row of point j + r SUB0 of the first stage, less r BS
  static __device__ __forceinline__ int row0(int j) { return j + j / RL * (RLP - RL); }
};

// base advanced by n >= 0 rows (uniform: the row offsets of a butterfly then stay in
// scalar registers beside one offset per lane)
template <typename V>
__device__ __forceinline__ V* rows_on(V* base, int n, uint32_t row) {
  using C = std::conditional_t<std::is_const_v<V>, const char, char>;
  return reinterpret_cast<V*>(reinterpret_cast<C*>(base) + (size_t)((uint32_t)n * row));
}

// First stage from the registers v of butterfly j (column col) into buf.
template <typename T, int LL>
__device__ __forceinline__ void ftr_first(cx<T>* buf, const cx<T>* tw, int j, int col, cx<T>* v) {
  using P = TrPlan<T, LL>;
  dft_reg<T, P::R0>(v);
  cx<T>* p = buf + P::row0(j) * P::TB + col;
  p[0] = v[0];
#pragma unroll
  for (int d = 1; d < P::R0; ++d) p[d * P::BS * P::TB] = cmul(v[d], tw[j * d]);
}
// Middle stage (512 points), in place, between two barriers.
template <typename T, int LL>
__device__ __forceinline__ void ftr_mid(cx<T>* buf, const cx<T>* tw) {
  using P = TrPlan<T, LL>;
  if constexpr (P::R1 > 1) {
#pragma unroll 1
    for (int id = threadIdx.x; id < P::R0 * P::RL * P::TB; id += P::NT) {
      const int col = id & (P::TB - 1), bf = id / P::TB, blk = bf / P::RL, j = bf % P::RL;
      cx<T>* p = buf + (blk * P::BS + j) * P::TB + col;
      cx<T> v[P::R1];
#pragma unroll
      for (int r = 0; r < P::R1; ++r) v[r] = p[r * P::RLP * P::TB];
      dft_reg<T, P::R1>(v);
      p[0] = v[0];
#pragma unroll
      for (int d = 1; d < P::R1; ++d) p[d * P::RLP * P::TB] = cmul(v[d], tw[j * d * P::R0]);
    }
    __syncthreads();
  }
}
// LDS row of the first output of the last-stage butterfly of digits n = d1 +
// R0 d2 (its outputs are k = n + d NBL, in consecutive rows)
template <typename T, int LL>
__device__ __forceinline__ int ftr_row(int n) {
  using P = TrPlan<T, LL>;
  return P::R1 > 1 ? (n % P::R0) * P::BS + (n / P::R0) * P::RLP : n * P::BS;
}
// Last stage over all butterflies: run(n, col, v) gets the butterfly's outputs.
template <typename T, int LL, typename Run>
__device__ __forceinline__ void ftr_last(cx<T>* buf, Run run) {
  using P = TrPlan<T, LL>;
#pragma unroll 1
  for (int id = threadIdx.x; id < P::NBL * P::TB; id += P::NT) {
    const int col = id & (P::TB - 1), n = id / P::TB;
    cx<T>* p = buf + ftr_row<T, LL>(n) * P::TB + col;
    cx<T> v[P::RL];
#pragma unroll
    for (int r = 0; r < P::RL; ++r) v[r] = p[r * P::TB];
    dft_reg<T, P::RL>(v);
    run(n, col, p, v);
  }
}

template <typename T, int LL>
__device__ __forceinline__ void ftr_roots(cx<T>* tw, const void* table, int at) {
  const cx<T>* src = static_cast<const cx<T>*>(table) + at;
  for (int e = threadIdx.x; e < TrPlan<T, LL>::L; e += TrPlan<T, LL>::NT) tw[e] = src[e];
}

// DFT over the second detector axis, in place, either direction.
template <typename T, int LL>
__global__ __launch_bounds__((TrPlan<T, LL>::NT), (TrPlan<T, LL>::waves)) void k_ftr_x2(StageArgs a) {
  using P = TrPlan<T, LL>;
  CInst& I = *(CInst*)a.inst[0];
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = tw + P::L;
  ftr_roots<T, LL>(tw, I.tw, I.g2.tw);
  const int len = a.len_nz ? I.nz : I.nt;
  const int ntile = (len + P::TB - 1) / P::TB;
  const uint32_t row = (uint32_t)len * (uint32_t)sizeof(cx<T>);
  const int col = (int)threadIdx.x & (P::TB - 1), j0 = (int)threadIdx.x / P::TB;
  const T sg = a.mode != 0 ? T(-1) : T(1);  // the inverse as conj(FFT(conj(.)))
  const uint32_t off = (uint32_t)j0 * row + (uint32_t)col * (uint32_t)sizeof(cx<T>);
  cx<T> pre[P::U][P::R0];
  auto tile = [&](int slot, int* w) {
    const int item = xcd_item(slot, a.total);
    const int k1 = item / ntile, t0 = (item - k1 * ntile) * P::TB;
    *w = len - t0;
    return static_cast<cx<T>*>(a.out[0]) + (size_t)k1 * P::L * len + t0;
  };
  auto fetch = [&](int slot) {
    int w;
    const cx<T>* io = tile(slot, &w);
#pragma unroll
    for (int u = 0; u < P::U; ++u)
#pragma unroll
      for (int r = 0; r < P::R0; ++r)
        pre[u][r] = col < w ? *at_off(rows_on(io, u * P::STEP + r * P::SUB0, row), off) : mk(T(0), T(0));
  };
  int slot = blockIdx.x;
  if (slot < a.total) fetch(slot);
  __syncthreads();
  for (; slot < a.total; slot += gridDim.x) {
#pragma unroll
    for (int u = 0; u < P::U; ++u) {
#pragma unroll
      for (int r = 0; r < P::R0; ++r) pre[u][r].y *= sg;
      ftr_first<T, LL>(buf, tw, j0 + u * P::STEP, col, pre[u]);
    }
    __syncthreads();
    if (slot + (int)gridDim.x < a.total) fetch(slot + gridDim.x);
    ftr_mid<T, LL>(buf, tw);
    int w;
    cx<T>* io = tile(slot, &w);
    ftr_last<T, LL>(buf, [&](int n, int b, cx<T>*, cx<T>* v) {
      if (b >= w) return;
      const uint32_t o = (uint32_t)n * row + (uint32_t)b * (uint32_t)sizeof(cx<T>);
#pragma unroll
      for (int d = 0; d < P::RL; ++d) *at_off(rows_on(io, d * P::NBL, row), o) = mk(v[d].x, sg * v[d].y);
    });
    __syncthreads();
  }
}

// DFT over the first detector axis, real input, bins 0 .. L/2: complex column b
// holds the samples t0 + 2b and t0 + 2b + 1.  With a cut-off on this (data-
// side) pass the samples are weighted as they enter the first stage; the
// column's slice of the weight table sits in LDS, two slices in turn.
template <typename T, int LL>
__global__ __launch_bounds__((TrPlan<T, LL>::NT), (TrPlan<T, LL>::waves)) void k_ftr_x1(StageArgs a) {
  using P = TrPlan<T, LL>;
  CInst& I = *(CInst*)a.inst[0];
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = tw + P::L;
  T* cws = reinterpret_cast<T*>(buf + P::ROWS * P::TB);
  ftr_roots<T, LL>(tw, I.tw, I.g1.tw);
  const int len = a.len_nz ? I.nz : I.nt;
  const int ntile = (len + 2 * P::TB - 1) / (2 * P::TB);
  const uint32_t row = (uint32_t)(I.n2 * len) * (uint32_t)sizeof(T);  // bytes of a real row
  const int col = (int)threadIdx.x & (P::TB - 1), j0 = (int)threadIdx.x / P::TB;
  const uint32_t off = (uint32_t)j0 * row + (uint32_t)col * (uint32_t)sizeof(cx<T>);
  const bool cut = !a.len_nz && I.cut_e;
  const int E = I.cut_e, ew = (E + 1) * (E + 1);
  auto slice = [&](int item, int s) {
    const int x2 = item / ntile, b2 = I.n2 > 1 ? cut_band(x2, I.n2, E) : E;
    const T* W = static_cast<const T*>(I.cutw);
    for (int e = threadIdx.x; e < ew; e += P::NT) {
      const int b1 = e / (E + 1), b3 = e - b1 * (E + 1);
      cws[s * ew + e] = W[(b1 * (E + 1) + b2) * (E + 1) + b3];
    }
  };
  cx<T> pre[P::U][P::R0];
  auto fetch = [&](int slot) {
    const int item = xcd_item(slot, a.total);
    const int x2 = item / ntile, t0 = (item - x2 * ntile) * 2 * P::TB;
    const cx<T>* in = reinterpret_cast<const cx<T>*>(static_cast<const T*>(a.in[0]) + (size_t)x2 * len + t0);
    const int w = (len - t0) >> 1;
#pragma unroll
    for (int u = 0; u < P::U; ++u)
#pragma unroll
      for (int r = 0; r < P::R0; ++r)
        pre[u][r] = col < w ? ld_cx<T, true>(at_off(rows_on(in, u * P::STEP + r * P::SUB0, row), off))
                            : mk(T(0), T(0));
  };
  int slot = blockIdx.x;
  if (slot < a.total) {
    fetch(slot);
    if (cut) slice(xcd_item(slot, a.total), 0);
  }
  __syncthreads();
  for (int it = 0; slot < a.total; slot += gridDim.x, ++it) {
    const int item = xcd_item(slot, a.total);
    const int x2 = item / ntile, t0 = (item - x2 * ntile) * 2 * P::TB;
    const int w = (len - t0) >> 1;
    if (cut && col < w) {
      const T* ws = cws + (it & 1) * ew;
      const int b2 = I.n2 > 1 ? cut_band(x2, I.n2, E) : E, t = t0 + 2 * col;
#pragma unroll
      for (int u = 0; u < P::U; ++u)
#pragma unroll
        for (int r = 0; r < P::R0; ++r) {
          const int b1 = cut_band(j0 + u * P::STEP + r * P::SUB0, P::L, E);
          if (b1 == E && b2 == E && t >= E && t + 1 <= len - E) continue;
          pre[u][r].x *= ws[b1 * (E + 1) + cut_band(t, len, E)];
          pre[u][r].y *= ws[b1 * (E + 1) + cut_band(t + 1, len, E)];
        }
    }
#pragma unroll
    for (int u = 0; u < P::U; ++u) ftr_first<T, LL>(buf, tw, j0 + u * P::STEP, col, pre[u]);
    __syncthreads();
    if (slot + (int)gridDim.x < a.total) {
      fetch(slot + gridDim.x);
      if (cut) slice(xcd_item(slot + gridDim.x, a.total), (it + 1) & 1);
    }
    ftr_mid<T, LL>(buf, tw);
    ftr_last<T, LL>(buf, [&](int, int, cx<T>* p, cx<T>* v) {
#pragma unroll
      for (int d = 0; d < P::RL; ++d) p[d * P::TB] = v[d];
    });
    __syncthreads();
    // bin k of Z and the conjugate of bin L - k (in the mirror butterfly's
    // rows) give the two samples' bins pa and pb
    cx<T>* out = static_cast<cx<T>*>(a.out[0]) + (size_t)x2 * len + t0;
    constexpr int NQ = P::NT / (P::NBL * P::TB) > 0 ? P::NT / (P::NBL * P::TB) : 1;  // threads per butterfly
#pragma unroll 1
    for (int id = threadIdx.x; id < P::NBL * P::TB * NQ; id += P::NT) {
      const int b = id & (P::TB - 1), n = id / P::TB % P::NBL, q = id / P::TB / P::NBL;
      if (b >= w) continue;
      const int nm = (P::NBL - n) % P::NBL;
      const cx<T>* own = buf + ftr_row<T, LL>(n) * P::TB + b;
      const cx<T>* mir = buf + ftr_row<T, LL>(nm) * P::TB + b;
      const uint32_t ob = (uint32_t)(n + q * P::NBL) * (2 * row) + (uint32_t)b * (uint32_t)(2 * sizeof(cx<T>));
#pragma unroll
      for (int i = 0; i < P::RL / 2 / NQ; ++i) {
        const int d = q + i * NQ, dm = n ? P::RL - 1 - d : (P::RL - d) % P::RL;
        const cx<T> z = own[d * P::TB], zn = cconj(mir[dm * P::TB]);
        const T h = T(0.5);
        const cx<T> pa = cscl(cadd(z, zn), h);
        const cx<T> df = csub(z, zn);
        st_pair(at_off(rows_on(out, i * NQ * P::NBL, 2 * row), ob), pa, mk(h * df.y, -h * df.x));
      }
      // bin L/2 (its own mirror): output RL/2 of butterfly 0
      if (n == 0 && q == 0) {
        const cx<T> z = own[P::RL / 2 * P::TB];
        st_pair(at_off(rows_on(out, P::RL / 2 * P::NBL, 2 * row), ob), mk(z.x, T(0)), mk(z.y, T(0)));
      }
    }
    __syncthreads();
  }
}

// Inverse DFT over the first axis from bins 0 .. L/2, real part; two
// neighbouring samples as one complex column (see k_tr_c2r_k1).  A
// prefetched tile (FP64) waits as loaded; it is combined when the first stage
// takes it.
template <typename T, int LL>
__global__ __launch_bounds__((TrPlan<T, LL>::NT), (TrPlan<T, LL>::waves)) void k_ftr_c2r(StageArgs a) {
  using P = TrPlan<T, LL>;
  CInst& I = *(CInst*)a.inst[0];
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = tw + P::L;
  T* cws = reinterpret_cast<T*>(buf + P::ROWS * P::TB);
  ftr_roots<T, LL>(tw, I.tw, I.g1.tw);
  const int len = a.len_nz ? I.nz : I.nt;
  const int ntile = (len + 2 * P::TB - 1) / (2 * P::TB);
  const uint32_t row = (uint32_t)(I.n2 * len) * (uint32_t)sizeof(T);
  const int col = (int)threadIdx.x & (P::TB - 1), j0 = (int)threadIdx.x / P::TB;
  const bool cut = !a.len_nz && I.cut_e;
  const int E = I.cut_e, ew = (E + 1) * (E + 1);
  // A butterfly's rows k = j + r SUB0 below L/2 are read as they are, the ones
  // from L/2 on from their mirror rows L - k: upwards resp. downwards from a
  // row that is the same for all lanes.
  const uint32_t offu = (uint32_t)j0 * (2 * row) + (uint32_t)col * (uint32_t)(2 * sizeof(cx<T>));
  const uint32_t offd = (uint32_t)(P::STEP - j0) * (2 * row) + (uint32_t)col * (uint32_t)(2 * sizeof(cx<T>));
  // (FP32: the loaded pairs beside the last stage's points would spill, and
  // four workgroups per CU cover the loads)
  constexpr bool PRE = !P::F && P::U * P::R0 <= 8;
  cx<T> pa[P::U][P::R0], pb[P::U][P::R0];
  auto fetch1 = [&](int slot, int u) {
    const int item = xcd_item(slot, a.total);
    const int x2 = item / ntile, t0 = (item - x2 * ntile) * 2 * P::TB;
    const cx<T>* in = static_cast<const cx<T>*>(a.in[0]) + (size_t)x2 * len + t0;
    const int w = (len - t0) >> 1;
#pragma unroll
    for (int r = 0; r < P::R0; ++r) {
      pa[u][r] = pb[u][r] = mk(T(0), T(0));
      if (col < w) {
        const cx<T>* p = r < P::R0 / 2
                             ? at_off(rows_on(in, u * P::STEP + r * P::SUB0, 2 * row), offu)
                             : at_off(rows_on(in, (P::R0 - r) * P::SUB0 - (u + 1) * P::STEP, 2 * row), offd);
        ld_pair(p, &pa[u][r], &pb[u][r]);
      }
    }
  };
  auto fetch = [&](int slot) {
    if constexpr (PRE) {
#pragma unroll
      for (int u = 0; u < P::U; ++u) fetch1(slot, u);
    }
  };
  int slot = blockIdx.x;
  if (slot < a.total) fetch(slot);
  __syncthreads();
  for (; slot < a.total; slot += gridDim.x) {
    const int item = xcd_item(slot, a.total);
    const int x2 = item / ntile, t0 = (item - x2 * ntile) * 2 * P::TB;
    const int w = (len - t0) >> 1;
#pragma unroll
    for (int u = 0; u < P::U; ++u) {
      if constexpr (!PRE) fetch1(slot, u);
      cx<T> v[P::R0];
#pragma unroll
      for (int r = 0; r < P::R0; ++r) {
        // Z = X_a + i X_b, conjugated; mirror bins conjugated first, the
        // imaginary parts of the bins 0 and L/2 dropped
        const bool real = (r == 0 || r == P::R0 / 2) && u == 0 && j0 == 0;
        const T ya = real ? T(0) : r >= P::R0 / 2 ? -pa[u][r].y : pa[u][r].y;
        const T yb = real ? T(0) : r >= P::R0 / 2 ? -pb[u][r].y : pb[u][r].y;
        v[r] = mk(pa[u][r].x - yb, -(ya + pb[u][r].x));
      }
      ftr_first<T, LL>(buf, tw, j0 + u * P::STEP, col, v);
    }
    if (cut) {
      const int b2 = I.n2 > 1 ? cut_band(x2, I.n2, E) : E;
      const T* W = static_cast<const T*>(I.cutw);
      for (int e = threadIdx.x; e < ew; e += P::NT) {
        const int b1 = e / (E + 1), b3 = e - b1 * (E + 1);
        cws[e] = W[(b1 * (E + 1) + b2) * (E + 1) + b3];
      }
    }
    __syncthreads();
    if (slot + (int)gridDim.x < a.total) fetch(slot + gridDim.x);
    ftr_mid<T, LL>(buf, tw);
    cx<T>* out = reinterpret_cast<cx<T>*>(static_cast<T*>(a.out[0]) + (size_t)x2 * len + t0);
    ftr_last<T, LL>(buf, [&](int n, int b, cx<T>*, cx<T>* v) {
      if (b >= w) return;
      const uint32_t o = (uint32_t)n * row + (uint32_t)b * (uint32_t)sizeof(cx<T>);
#pragma unroll
      for (int d = 0; d < P::RL; ++d) {
        T x = v[d].x, y = -v[d].y;
        if (cut) {
          const int t = t0 + 2 * b, b1 = cut_band(n + d * P::NBL, P::L, E);
          x *= cws[b1 * (E + 1) + cut_band(t, len, E)];
          y *= cws[b1 * (E + 1) + cut_band(t + 1, len, E)];
        }
        st_cx<T, true>(at_off(rows_on(out, d * P::NBL, row), o), mk(x, y));
      }
    });
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Launches: false when the length or the array is not theirs.

namespace {

template <typename T>
size_t cut_bytes(const Inst& I, bool data) {
  const size_t e1 = (size_t)I.cut_e + 1;
  return data && I.cut_e ? 2 * e1 * e1 * sizeof(T) : 0;
}

}  // namespace

template <typename T>
bool Fixed<T>::takes(int L, int rows, int len) {
  return (L == 128 || L == 256 || L == 512) && (int64_t)rows * len >= 32ll * num_cu();
}

#define PAT_FIXED(KERN, L, ITEMS, NAME, EXTRA)                                                                        \
  auto go = [&](auto ll) {                                                                                            \
    using P = TrPlan<T, decltype(ll)::v>;                                                                             \
    const int len = a.len_nz ? h.nz : h.nt;                                                                           \
    a.total = (ITEMS);                                                                                                \
    return launch_persistent(KERN<T, decltype(ll)::v>, NAME, a, P::lds + (EXTRA), st, tm, P::NT);                     \
  };                                                                                                                  \
  if ((L) == 128) return go(RadixTag<7>{});                                                                           \
  if ((L) == 256) return go(RadixTag<8>{});                                                                           \
  return go(RadixTag<9>{});

template <typename T>
hipError_t Fixed<T>::x1(StageArgs& a, const Inst& h, hipStream_t st, StageTimer* tm) {
  PAT_FIXED(k_ftr_x1, h.n1, h.n2 * ((len + 2 * P::TB - 1) / (2 * P::TB)), "dft_x1", cut_bytes<T>(h, !a.len_nz))
}
template <typename T>
hipError_t Fixed<T>::x2(StageArgs& a, const Inst& h, hipStream_t st, StageTimer* tm) {
  PAT_FIXED(k_ftr_x2, h.n2, h.h1 * ((len + P::TB - 1) / P::TB), a.mode ? "idft_x2" : "dft_x2", 0)
}
template <typename T>
hipError_t Fixed<T>::c2r(StageArgs& a, const Inst& h, hipStream_t st, StageTimer* tm) {
  PAT_FIXED(k_ftr_c2r, h.n1, h.n2 * ((len + 2 * P::TB - 1) / (2 * P::TB)), "idft_x1_c2r",
            cut_bytes<T>(h, !a.len_nz))
}

template struct Fixed<float>;
template struct Fixed<double>;

}  // namespace pat
