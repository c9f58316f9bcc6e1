// CDNA4 (gfx950) kernels of the NUFFT-based planar photoacoustic
// reconstruction.  Every kernel runs 256-thread workgroups over a list of work
// items (instance, tile or group of lines); items come either one per
// workgroup or from a device work counter drained by a persistent grid (the
// batched form).
//
// Stages (a1 .. a5 are the steps of R as pat.h lists them under
// pat_reconstruct; see pat.h for the operators they compose):
//   k_tr_x1_r2c   DFT over the first detector axis, real input, half spectrum
//   k_tr_x2       DFT over the second detector axis (either direction)
//   k_tr_c2r_k1   inverse DFT over the first axis from the half spectrum, real part
//   k_tr_*_pipe   the three above as software pipelines (one FP32 instance)
//   k_line_fft    DFT along contiguous lines (depth axis)
//   k_line_a2     deconvolve by 1/Psi, centre, zero-pad to c*nt, FFT (eq. nufft-c)
//                 (k_line_a2_pipe: its software pipeline, c = 2, sizes fixed
//                 at compile time)
//   k_line_a2t    its transpose: inverse FFT, pick, multiply by 1/Psi
//                 (k_line_a2t_pipe: likewise)
//   k_line_interp type-2 interpolation with 2cK Kaiser-Bessel taps (eq. nufft-a)
//                 and the Jacobian weight (eq. fft-0) (k_line_interp_stream:
//                 persistent, the next line group streamed into registers)
//   k_line_spread its transpose (type-1), gathered per grid cell over the
//                 monotone node list of the line: no atomics, deterministic
//                 (k_line_spread_w: one line per wavefront, segmented sums
//                 across lanes, FP32)
//   k_line_nufft2 a2 + a3 + inverse depth DFT fused per line group in LDS
//                 (k_line_nufft2_pipe: its software pipeline for c = 2;
//                 k_line_nufft2_pipe_c: the same for sizes fixed at compile
//                 time; k_line_nufft2_mirror: R on 3D plans with nz = m/4,
//                 the lines of an item in mirror pairs sharing node windows,
//                 for the bf16 grid only the stages after it)
//   k_line_nufft1 depth DFT + spreading + transposed a2 fused per line in LDS
//                 (k_line_nufft1_c: sizes fixed at compile time;
//                 k_line_nufft1_w: one line per wavefront, FP32)
// The fused kernels never store the oversampled grid; the staged ones do
// (bf16 grid option where k_line_nufft2_mirror does not apply, long grid lines,
// and the stand-alone a3 / spreading entry points).
//
// Beside these: transverse.hip (transverse passes of 128, 256 and 512 points),
// general.hip (transverse passes and line stages of other lengths) and
// linepair.hip (type-1 line stages of 3D plans by mirror line pairs); Runner
// chooses.
//
// Uniform FFTs here are in-place decimation-in-frequency mixed-radix transforms in
// LDS; bin k ends at position perm[k] (a table built by the host plan).  Two
// instantiations exist: radices 2/4/8 with shift arithmetic (all lengths
// powers of two), and the general one (odd primes up to 23).
#include "device.h"

#include <cmath>
#include <map>
#include <mutex>
#include <tuple>

#include "general.h"

namespace pat {

// ---------------------------------------------------------------------------
// Transverse passes.  Tiles of consecutive samples (t or z, the contiguous
// axis) by the full transform length; lanes run along the samples, so global
// accesses are contiguous runs.  The real passes pack two neighbouring real
// samples into one complex column (real and imaginary part) and separate the
// two transforms afterwards, so a tile of tb complex columns covers 2 tb
// samples.  Global accesses move two columns (16 bytes in float) per lane
// where the alignment allows it.

template <typename T, int RS>
__global__ __launch_bounds__(kBlock) void k_tr_x1_r2c(StageArgs a) {
  [[maybe_unused]] constexpr bool P2 = RS == 0;
  PAT_FOR_EACH_ITEM(a)
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = tw + I.n1;
  if (new_inst_) load_twiddles(tw, I, I.f1);
  const int len = a.len_nz ? I.nz : I.nt;  // even
  const int tb = I.tb;
  const int ntile = (len + 2 * tb - 1) / (2 * tb);
  const int x2 = li / ntile;
  const int t0 = (li - x2 * ntile) * 2 * tb;
  const T* in = static_cast<const T*>(a.in[inst_]);
  cx<T>* out = static_cast<cx<T>*>(a.out[inst_]);
  const int L = I.n1;
  const size_t rstride = (size_t)I.n2 * len;
  const T* in0 = in + (size_t)x2 * len + t0;
  const bool cut = !a.len_nz && I.cut_e;  // data-side pass with a cut-off
  // the column's cut-off weights, read from LDS while the tile is stored
  T* cws = reinterpret_cast<T*>(buf + L * tb);
  const int cb2 = cut && I.n2 > 1 ? cut_band(x2, I.n2, I.cut_e) : I.cut_e;
  if (cut) {
    cut_slice(I, cws, x2);
    __syncthreads();
  }
  if (len % 4 == 0 && tb % 2 == 0) {
    // column pairs: samples t0 + 4c .. t0 + 4c + 3 (len is a multiple of 4)
    const int hb = tb / 2;
    copy_batched<4>(
        L * hb,
        [&](int e) {
          int x, c;
          divmod<true>(e, hb, &x, &c);
          cx<T> u[2] = {mk(T(0), T(0)), mk(T(0), T(0))};
          if (t0 + 4 * c < len)
            ld_pair<T, true>(reinterpret_cast<const cx<T>*>(in0 + x * rstride + 4 * c), &u[0], &u[1]);
          return cx<cx<T>>{u[0], u[1]};
        },
        [&](int e, cx<cx<T>> v) {
          if (cut) {
            int x, c;
            divmod<true>(e, hb, &x, &c);
            if (t0 + 4 * c < len) {
              cut_pair(I, cws, cb2, x, t0 + 4 * c, len, &v.x);
              cut_pair(I, cws, cb2, x, t0 + 4 * c + 2, len, &v.y);
            }
          }
          buf[2 * e] = v.x;
          buf[2 * e + 1] = v.y;
        });
  } else {
    copy_batched<8>(
        L * tb,
        [&](int e) {
          int x, b;
          divmod<true>(e, tb, &x, &b);
          // samples t0 + 2b (real part) and t0 + 2b + 1 (imaginary part); len is even
          return t0 + 2 * b < len ? *reinterpret_cast<const cx<T>*>(in0 + x * rstride + 2 * b) : mk(T(0), T(0));
        },
        [&](int e, cx<T> v) {
          if (cut) {
            int x, b;
            divmod<true>(e, tb, &x, &b);
            if (t0 + 2 * b < len) cut_pair(I, cws, cb2, x, t0 + 2 * b, len, &v);
          }
          buf[e] = v;
        });
  }
  __syncthreads();
  fft_lds<T, RS, false>(buf, I.f1, tw, tb, 1, tb);
  const int32_t* perm = I.perm + I.f1.perm;
  cx<T>* out0 = out + (size_t)x2 * len + t0;
  for (int e = threadIdx.x; e < I.h1 * tb; e += kBlock) {
    int k, b;
    divmod<true>(e, tb, &k, &b);
    if (t0 + 2 * b >= len) continue;
    const int kn = k == 0 ? 0 : L - k;
    const cx<T> z = buf[perm[k] * tb + b];
    const cx<T> zn = cconj(buf[perm[kn] * tb + b]);
    const T h = T(0.5);
    // transforms of the real and imaginary parts
    const cx<T> pa = cscl(cadd(z, zn), h);
    const cx<T> d = csub(z, zn);
    const cx<T> pb = mk(h * d.y, -h * d.x);
    st_pair(out0 + (size_t)k * rstride + 2 * b, pa, pb);
  }
  PAT_END_ITEM
}

template <typename T, int RS>
__global__ __launch_bounds__(kBlock) void k_tr_x2(StageArgs a) {
  [[maybe_unused]] constexpr bool P2 = RS == 0;
  PAT_FOR_EACH_ITEM(a)
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = tw + I.n2;
  if (new_inst_) load_twiddles(tw, I, I.f2);
  const int len = a.len_nz ? I.nz : I.nt;
  const int tb = I.tb;
  const int ntile = (len + tb - 1) / tb;
  const int k1 = li / ntile;
  const int t0 = (li - k1 * ntile) * tb;
  cx<T>* io = static_cast<cx<T>*>(a.out[inst_]) + (size_t)k1 * I.n2 * len + t0;
  const int L = I.n2;
  const bool inv = a.mode != 0;
  // column pairs b, b + 1 when tb is even (b even; len is even, so both or
  // neither exist), single columns otherwise
  const int hb = tb / 2;
  if (tb % 2 == 0) {
    copy_batched<4>(
        L * hb,
        [&](int e) {
          int x, c;
          divmod<true>(e, hb, &x, &c);
          cx<T> u[2] = {mk(T(0), T(0)), mk(T(0), T(0))};
          if (t0 + 2 * c < len) ld_pair(io + (size_t)x * len + 2 * c, &u[0], &u[1]);
          return cx<cx<T>>{inv ? cconj(u[0]) : u[0], inv ? cconj(u[1]) : u[1]};
        },
        [&](int e, cx<cx<T>> v) {
          buf[2 * e] = v.x;
          buf[2 * e + 1] = v.y;
        });
  } else {
    copy_batched<8>(
        L * tb,
        [&](int e) {
          int x, b;
          divmod<true>(e, tb, &x, &b);
          const cx<T> v = t0 + b < len ? io[(size_t)x * len + b] : mk(T(0), T(0));
          return inv ? cconj(v) : v;
        },
        [&](int e, cx<T> v) { buf[e] = v; });
  }
  __syncthreads();
  fft_lds<T, RS, false>(buf, I.f2, tw, tb, 1, tb);
  const int32_t* perm = I.perm + I.f2.perm;
  if (tb % 2 == 0) {
    for (int e = threadIdx.x; e < L * hb; e += kBlock) {
      int k, c;
      divmod<true>(e, hb, &k, &c);
      if (t0 + 2 * c < len) {
        const cx<T>* s = buf + perm[k] * tb + 2 * c;
        st_pair(io + (size_t)k * len + 2 * c, inv ? cconj(s[0]) : s[0], inv ? cconj(s[1]) : s[1]);
      }
    }
  } else {
    for (int e = threadIdx.x; e < L * tb; e += kBlock) {
      int k, b;
      divmod<true>(e, tb, &k, &b);
      if (t0 + b < len) {
        const cx<T> v = buf[perm[k] * tb + b];
        io[(size_t)k * len + b] = inv ? cconj(v) : v;
      }
    }
  }
  PAT_END_ITEM
}

// k_tr_x1_r2c as a software pipeline (see k_tr_x2_pipe), for one instance,
// len a multiple of 4, tb even and n1 * tb / 2 <= kPipeU * kBlock
// four-sample loads per tile.  With a cut-off on this (data-side) pass, two
// LDS slices of the weight table alternate: the slice of the next tile's
// column is written while the current tile is transformed, and read when
// the next tile is stored into LDS.  LL > 0 fixes the transform length at
// 2^LL (and its FFT stages) at compile time, in all three pipelines.
template <typename T, int RS, int LL = 0>
__global__ __launch_bounds__(kBlock, RS == 0 ? (sizeof(T) == 4 ? 4 : 2) : 1) void k_tr_x1_pipe(StageArgs a);

// k_tr_x2 as a software pipeline for one instance whose tile is at most
// kPipeU column pairs per thread (n2 * tb / 2 <= kPipeU * kBlock, tb even): a
// persistent grid strides over the tiles, and each workgroup issues the
// loads of its next tile into registers right after storing the current one
// into LDS, so they are in flight while the current tile is transformed and
// written back.  The output positions sit in LDS beside the twiddles (a
// table read from memory in the store loop would wait for those loads).
constexpr int kPipeU = 8;
// tile width of the plans (FP32: 16 columns, 8 once a tile of 2^9-point
// columns would pass 64 KB of LDS; FP64: 8, then 4), fixed with the length in
// the instances that take it at compile time
template <typename T>
constexpr int pipe_tb(int ll) { return sizeof(T) == 4 ? (ll >= 9 ? 8 : 16) : (ll >= 9 ? 4 : 8); }
// registers per thread for a prefetched tile of 2^LL points by tb columns
// (LL > 0), or for the largest tile a run-time length may have
template <int LL>
constexpr int pipe_units(int per_col) {
  return LL > 0 ? ((1 << LL) * per_col + kBlock - 1) / kBlock : 0;
}
template <typename T, int RS, int LL = 0>
__global__ __launch_bounds__(kBlock) void k_tr_x2_pipe(StageArgs a) {
  const Inst& I = *a.inst[0];
  const int L = LL > 0 ? 1 << LL : I.n2;
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  int32_t* pos = reinterpret_cast<int32_t*>(tw + L);
  cx<T>* buf = reinterpret_cast<cx<T>*>(pos + ((L + 3) & ~3));
  load_twiddles(tw, I, I.f2);
  const int32_t* perm = I.perm + I.f2.perm;
  for (int e = threadIdx.x; e < L; e += kBlock) pos[e] = perm[e];
  const int len = a.len_nz ? I.nz : I.nt;
  const int tb = LL > 0 ? pipe_tb<T>(LL) : I.tb, hb = tb / 2;
  const int ntile = (len + tb - 1) / tb;
  const bool inv = a.mode != 0;
  cx<T>* base = static_cast<cx<T>*>(a.out[0]);
  constexpr int PU = LL > 0 ? pipe_units<LL>(pipe_tb<T>(LL) / 2) : kPipeU;  // column pairs per thread
  cx<T> pre[2 * PU];
  auto fetch = [&](int item) {
    const int k1 = item / ntile;
    const int t0 = (item - k1 * ntile) * tb;
    const cx<T>* io = base + (size_t)k1 * L * len + t0;
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int e = (int)threadIdx.x + u * kBlock;
      pre[2 * u] = pre[2 * u + 1] = mk(T(0), T(0));
      if (e < L * hb) {
        int x, c;
        divmod<true>(e, hb, &x, &c);
        if (t0 + 2 * c < len) ld_pair(io + (size_t)x * len + 2 * c, &pre[2 * u], &pre[2 * u + 1]);
      }
    }
  };
  int item = blockIdx.x;
  if (item < a.total) fetch(item);
  for (; item < a.total; item += gridDim.x) {
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int e = (int)threadIdx.x + u * kBlock;
      if (e < L * hb) {
        buf[2 * e] = inv ? cconj(pre[2 * u]) : pre[2 * u];
        buf[2 * e + 1] = inv ? cconj(pre[2 * u + 1]) : pre[2 * u + 1];
      }
    }
    __syncthreads();
    const int k1 = item / ntile;
    const int t0 = (item - k1 * ntile) * tb;
    cx<T>* io = base + (size_t)k1 * L * len + t0;
    if (item + (int)gridDim.x < a.total) fetch(item + gridDim.x);
    if constexpr (LL > 0) p2_fft<T, (LL > 0 ? LL : 1), false>(buf, tw, tb, 1, tb);
    else fft_lds<T, RS, false>(buf, I.f2, tw, tb, 1, tb);
    for (int e = threadIdx.x; e < L * hb; e += kBlock) {
      int kk, c;
      divmod<true>(e, hb, &kk, &c);
      if (t0 + 2 * c < len) {
        const cx<T>* s = buf + pos[kk] * tb + 2 * c;
        st_pair(io + (size_t)kk * len + 2 * c, inv ? cconj(s[0]) : s[0], inv ? cconj(s[1]) : s[1]);
      }
    }
    __syncthreads();
  }
}

template <typename T, int RS, int LL>
__global__ __launch_bounds__(kBlock, RS == 0 ? (sizeof(T) == 4 ? 4 : 2) : 1) void k_tr_x1_pipe(StageArgs a) {
  [[maybe_unused]] constexpr bool P2 = RS == 0;
  const Inst& I = *a.inst[0];
  const int L = LL > 0 ? 1 << LL : I.n1;
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  int32_t* pos = reinterpret_cast<int32_t*>(tw + L);
  cx<T>* buf = reinterpret_cast<cx<T>*>(pos + ((L + 3) & ~3));
  const bool cut = !a.len_nz && I.cut_e;  // data-side pass with a cut-off
  const int ew = (I.cut_e + 1) * (I.cut_e + 1);
  T* cws0 = reinterpret_cast<T*>(buf + L * I.tb);  // two column slices of the weights
  load_twiddles(tw, I, I.f1);
  const int32_t* perm = I.perm + I.f1.perm;
  for (int e = threadIdx.x; e < L; e += kBlock) pos[e] = perm[e];
  const int len = a.len_nz ? I.nz : I.nt;
  const int tb = LL > 0 ? pipe_tb<T>(LL) : I.tb, hb = tb / 2;
  const int ntile = (len + 2 * tb - 1) / (2 * tb);
  const size_t rstride = (size_t)I.n2 * len;
  const T* in = static_cast<const T*>(a.in[0]);
  cx<T>* out = static_cast<cx<T>*>(a.out[0]);
  constexpr int PU = LL > 0 ? pipe_units<LL>(pipe_tb<T>(LL) / 2) : kPipeU;  // column pairs per thread
  cx<T> pre[2 * PU];
  auto fetch = [&](int item) {
    const int x2 = item / ntile;
    const int t0 = (item - x2 * ntile) * 2 * tb;
    const T* in0 = in + (size_t)x2 * len + t0;
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int e = (int)threadIdx.x + u * kBlock;
      pre[2 * u] = pre[2 * u + 1] = mk(T(0), T(0));
      if (e < L * hb) {
        int x, c;
        divmod<true>(e, hb, &x, &c);
        if (t0 + 4 * c < len)
          ld_pair<T, true>(reinterpret_cast<const cx<T>*>(in0 + x * rstride + 4 * c), &pre[2 * u], &pre[2 * u + 1]);
      }
    }
  };
  int item = blockIdx.x;
  if (item < a.total) {
    fetch(item);
    if (cut) {
      cut_slice(I, cws0, item / ntile);
      __syncthreads();
    }
  }
  for (int it = 0; item < a.total; item += gridDim.x, ++it) {
    const int x2 = item / ntile;
    const int t0 = (item - x2 * ntile) * 2 * tb;
    const T* cws = cws0 + (it & 1) * ew;
    const int cb2 = cut && I.n2 > 1 ? cut_band(x2, I.n2, I.cut_e) : I.cut_e;
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      const int e = (int)threadIdx.x + u * kBlock;
      if (e < L * hb) {
        cx<T> v0 = pre[2 * u], v1 = pre[2 * u + 1];
        if (cut) {
          int x, c;
          divmod<true>(e, hb, &x, &c);
          if (t0 + 4 * c < len) {
            cut_pair(I, cws, cb2, x, t0 + 4 * c, len, &v0);
            cut_pair(I, cws, cb2, x, t0 + 4 * c + 2, len, &v1);
          }
        }
        buf[2 * e] = v0;
        buf[2 * e + 1] = v1;
      }
    }
    __syncthreads();
    if (item + (int)gridDim.x < a.total) {
      // The next column's weights are loaded before the next tile and
      // written to the other slice after it (last read before the barrier
      // above): their LDS writes then wait for these loads only, not for
      // the tile's.
      const int nx2 = (item + (int)gridDim.x) / ntile;
      T sv[2];
      if (cut) {
        const int e1 = I.cut_e + 1;
        const int b2 = I.n2 > 1 ? cut_band(nx2, I.n2, I.cut_e) : I.cut_e;
        const T* W = static_cast<const T*>(I.cutw);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int e = (int)threadIdx.x + h * kBlock;
          if (e < ew) {
            const int b1 = e / e1, b3 = e - b1 * e1;
            sv[h] = W[(b1 * e1 + b2) * e1 + b3];
          }
        }
      }
      fetch(item + gridDim.x);
      if (cut) {
        T* dst = cws0 + ((it + 1) & 1) * ew;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int e = (int)threadIdx.x + h * kBlock;
          if (e < ew) dst[e] = sv[h];
        }
      }
    }
    if constexpr (LL > 0) p2_fft<T, (LL > 0 ? LL : 1), false>(buf, tw, tb, 1, tb);
    else fft_lds<T, RS, false>(buf, I.f1, tw, tb, 1, tb);
    cx<T>* out0 = out + (size_t)x2 * len + t0;
    for (int e = threadIdx.x; e < I.h1 * tb; e += kBlock) {
      int kk, b;
      divmod<true>(e, tb, &kk, &b);
      if (t0 + 2 * b >= len) continue;
      const int kn = kk == 0 ? 0 : L - kk;
      const cx<T> z = buf[pos[kk] * tb + b];
      const cx<T> zn = cconj(buf[pos[kn] * tb + b]);
      const T h = T(0.5);
      const cx<T> pa = cscl(cadd(z, zn), h);
      const cx<T> d = csub(z, zn);
      const cx<T> pb = mk(h * d.y, -h * d.x);
      st_pair(out0 + (size_t)kk * rstride + 2 * b, pa, pb);
    }
    __syncthreads();
  }
}

// Inverse DFT over the first axis from bins 0..n1/2 (the others are the
// complex conjugates of their mirror bins), real part.  Two neighbouring
// samples are transformed together: Z = X_a + i X_b inverts to x_a + i x_b.
// The imaginary parts of the bins 0 and n1/2 are dropped, which is what
// taking the real part of the full inverse DFT does.
template <typename T, int RS>
__global__ __launch_bounds__(kBlock) void k_tr_c2r_k1(StageArgs a) {
  [[maybe_unused]] constexpr bool P2 = RS == 0;
  PAT_FOR_EACH_ITEM(a)
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = tw + I.n1;
  if (new_inst_) load_twiddles(tw, I, I.f1);
  const int len = a.len_nz ? I.nz : I.nt;
  const int tb = I.tb;
  const int ntile = (len + 2 * tb - 1) / (2 * tb);
  const int x2 = li / ntile;
  const int t0 = (li - x2 * ntile) * 2 * tb;
  const cx<T>* in = static_cast<const cx<T>*>(a.in[inst_]);
  T* out = static_cast<T*>(a.out[inst_]);
  const int L = I.n1;
  const int half = L / 2;
  const size_t rstride = (size_t)I.n2 * len;
  const cx<T>* in0 = in + (size_t)x2 * len + t0;
  const bool cut = !a.len_nz && I.cut_e;  // data-side pass with a cut-off
  T* cws = reinterpret_cast<T*>(buf + L * tb);  // the column's cut-off weights
  if (cut) cut_slice(I, cws, x2);
  copy_batched<4>(
      L * tb,
      [&](int e) {
        int k, b;
        divmod<true>(e, tb, &k, &b);
        const int src = k <= half ? k : L - k;
        cx<T> xa = mk(T(0), T(0)), xb = mk(T(0), T(0));
        if (t0 + 2 * b < len) ld_pair(in0 + (size_t)src * rstride + 2 * b, &xa, &xb);
        if (k == 0 || k == half) {
          xa.y = T(0);
          xb.y = T(0);
        } else if (k > half) {
          xa = cconj(xa);
          xb = cconj(xb);
        }
        // Z = xa + i xb, stored conjugated (inverse DFT as conj(FFT(conj(.))))
        return mk(xa.x - xb.y, -(xa.y + xb.x));
      },
      [&](int e, cx<T> v) { buf[e] = v; });
  __syncthreads();
  fft_lds<T, RS, false>(buf, I.f1, tw, tb, 1, tb);
  const int32_t* perm = I.perm + I.f1.perm;
  T* out0 = out + (size_t)x2 * len + t0;
  const int cb2 = cut && I.n2 > 1 ? cut_band(x2, I.n2, I.cut_e) : I.cut_e;
  if (len % 4 == 0 && tb % 2 == 0) {
    // four samples per lane (len is a multiple of 4)
    const int hb = tb / 2;
    for (int e = threadIdx.x; e < L * hb; e += kBlock) {
      int x, c;
      divmod<true>(e, hb, &x, &c);
      if (t0 + 4 * c < len) {
        const cx<T>* y = buf + perm[x] * tb + 2 * c;  // conj of x_a + i x_b
        cx<T> v0 = mk(y[0].x, -y[0].y), v1 = mk(y[1].x, -y[1].y);
        if (cut) {
          cut_pair(I, cws, cb2, x, t0 + 4 * c, len, &v0);
          cut_pair(I, cws, cb2, x, t0 + 4 * c + 2, len, &v1);
        }
        st_pair<T, true>(reinterpret_cast<cx<T>*>(out0 + (size_t)x * rstride + 4 * c), v0, v1);
      }
    }
  } else {
    for (int e = threadIdx.x; e < L * tb; e += kBlock) {
      int x, b;
      divmod<true>(e, tb, &x, &b);
      if (t0 + 2 * b < len) {
        const cx<T> y = buf[perm[x] * tb + b];  // conj of x_a + i x_b
        cx<T> v = mk(y.x, -y.y);
        if (cut) cut_pair(I, cws, cb2, x, t0 + 2 * b, len, &v);
        *reinterpret_cast<cx<T>*>(out0 + (size_t)x * rstride + 2 * b) = v;
      }
    }
  }
  PAT_END_ITEM
}

// k_tr_c2r_k1 as a software pipeline (see k_tr_x2_pipe), for one instance
// without a cut-off on this pass, len a multiple of 4, tb even and
// n1 * tb <= 2 kPipeU * kBlock bins per tile.
template <typename T, int RS, int LL = 0>
__global__ __launch_bounds__(kBlock, RS == 0 ? (sizeof(T) == 4 ? 4 : 2) : 1) void k_tr_c2r_pipe(StageArgs a) {
  const Inst& I = *a.inst[0];
  const int L = LL > 0 ? 1 << LL : I.n1, half = L / 2;
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  int32_t* pos = reinterpret_cast<int32_t*>(tw + L);
  cx<T>* buf = reinterpret_cast<cx<T>*>(pos + ((L + 3) & ~3));
  load_twiddles(tw, I, I.f1);
  const int32_t* perm = I.perm + I.f1.perm;
  for (int e = threadIdx.x; e < L; e += kBlock) pos[e] = perm[e];
  const int len = a.len_nz ? I.nz : I.nt;
  const int tb = LL > 0 ? pipe_tb<T>(LL) : I.tb, hb = tb / 2;
  const int ntile = (len + 2 * tb - 1) / (2 * tb);
  const size_t rstride = (size_t)I.n2 * len;
  const cx<T>* in = static_cast<const cx<T>*>(a.in[0]);
  T* out = static_cast<T*>(a.out[0]);
  constexpr int U = LL > 0 ? pipe_units<LL>(pipe_tb<T>(LL)) : 2 * kPipeU;  // bins per thread
  cx<T> pre[U];
  auto fetch = [&](int item) {
    const int x2 = item / ntile;
    const int t0 = (item - x2 * ntile) * 2 * tb;
    const cx<T>* in0 = in + (size_t)x2 * len + t0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = (int)threadIdx.x + u * kBlock;
      pre[u] = mk(T(0), T(0));
      if (e < L * tb) {
        int kk, b;
        divmod<true>(e, tb, &kk, &b);
        const int src = kk <= half ? kk : L - kk;
        cx<T> xa = mk(T(0), T(0)), xb = mk(T(0), T(0));
        if (t0 + 2 * b < len) ld_pair(in0 + (size_t)src * rstride + 2 * b, &xa, &xb);
        if (kk == 0 || kk == half) {
          xa.y = T(0);
          xb.y = T(0);
        } else if (kk > half) {
          xa = cconj(xa);
          xb = cconj(xb);
        }
        // Z = xa + i xb, stored conjugated (inverse DFT as conj(FFT(conj(.))))
        pre[u] = mk(xa.x - xb.y, -(xa.y + xb.x));
      }
    }
  };
  int item = blockIdx.x;
  if (item < a.total) fetch(item);
  for (; item < a.total; item += gridDim.x) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = (int)threadIdx.x + u * kBlock;
      if (e < L * tb) buf[e] = pre[u];
    }
    __syncthreads();
    const int x2 = item / ntile;
    const int t0 = (item - x2 * ntile) * 2 * tb;
    if (item + (int)gridDim.x < a.total) fetch(item + gridDim.x);
    if constexpr (LL > 0) p2_fft<T, (LL > 0 ? LL : 1), false>(buf, tw, tb, 1, tb);
    else fft_lds<T, RS, false>(buf, I.f1, tw, tb, 1, tb);
    T* out0 = out + (size_t)x2 * len + t0;
    for (int e = threadIdx.x; e < L * hb; e += kBlock) {
      int x, c;
      divmod<true>(e, hb, &x, &c);
      if (t0 + 4 * c < len) {
        const cx<T>* y = buf + pos[x] * tb + 2 * c;  // conj of x_a + i x_b
        st_pair<T, true>(reinterpret_cast<cx<T>*>(out0 + (size_t)x * rstride + 4 * c), mk(y[0].x, -y[0].y),
                         mk(y[1].x, -y[1].y));
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Line stages: a group of consecutive frequency lines (k1, k2) per work item.

// DFT of length nz along each line, in place.
template <typename T, int RS>
__global__ __launch_bounds__(kBlock) void k_line_fft(StageArgs a) {
  constexpr bool P2 = RS == 0;
  PAT_FOR_EACH_ITEM(a)
  cx<T>* tw = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = tw + I.nz;
  if (new_inst_) load_twiddles(tw, I, I.fz);
  const int L = I.nz;
  const int line0 = li * I.lpw_z;
  const int nl = min(I.lpw_z, I.lines - line0);
  cx<T>* io = static_cast<cx<T>*>(a.out[inst_]) + (size_t)line0 * L;
  const bool inv = a.mode != 0;
  copy_batched<4>(
      nl * L,
      [&](int e) {
        const cx<T> v = io[e];
        return inv ? cconj(v) : v;
      },
      [&](int e, cx<T> v) { buf[e] = v; });
  __syncthreads();
  fft_lds<T, RS, true>(buf, I.fz, tw, nl, L, 1);
  const int32_t* perm = I.perm + I.fz.perm;
  for (int e = threadIdx.x; e < nl * L; e += kBlock) {
    int b, j;
    divmod<P2>(e, L, &b, &j);
    const cx<T> v = buf[b * L + perm[j]];
    io[e] = inv ? cconj(v) : v;
  }
  PAT_END_ITEM
}

// a2 loading: u_n = G_n s_n placed at (n - nt/2) mod m, zeros elsewhere.  The
// centring turns the per-tap factor exp(i pi j / c) of eq. (nufft-a) into a
// shift, leaving only exp(-i pi nu) per node.
template <typename T, bool P2>
__device__ __forceinline__ void load_deconv_pad(const Inst& I, const cx<T>* g, int nl, cx<T>* buf) {
  const int m = I.m, nt = I.nt;
  const T* sn = static_cast<const T*>(I.sn);
  copy_batched<4>(
      nl * m,
      [&](int e) {
        int b, j;
        divmod<P2>(e, m, &b, &j);
        // centred: grid position j holds sample (j + nt/2) mod m; otherwise j
        int n = I.centred ? j + nt / 2 : j;
        if (n >= m) n -= m;
        return n < nt ? cscl(g[(size_t)b * nt + n], sn[n]) : mk(T(0), T(0));
      },
      [&](int e, cx<T> v) { buf[e] = v; });
}

template <typename T, typename G, int RS>
__global__ __launch_bounds__(kBlock) void k_line_a2(StageArgs a) {
  constexpr bool P2 = RS == 0;
  PAT_FOR_EACH_ITEM(a)
  // the twiddle table in LDS before the lines, or read from memory: for
  // long lines, and for power-of-two lengths (their workgroups, one item
  // each, copy the table slower than the FFT reads it from cache; the LDS
  // region stays reserved, which holds the kernel to fewer workgroups per
  // CU: freeing it made the kernel 1.5x slower)
  cx<T>* lds = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = I.twg_m ? lds : lds + I.m;
  const bool twg = P2 || I.twg_m;
  const cx<T>* tw = twg ? static_cast<const cx<T>*>(I.tw) + I.fm.tw : lds;
  if (new_inst_ && !twg) load_twiddles(lds, I, I.fm);
  const int m = I.m, nt = I.nt;
  const int line0 = li * I.lpw_m;
  const int nl = min(I.lpw_m, I.lines - line0);
  load_deconv_pad<T, P2>(I, static_cast<const cx<T>*>(a.in[inst_]) + (size_t)line0 * nt, nl, buf);
  __syncthreads();
  fft_lds<T, RS, true>(buf, I.fm, tw, nl, m, 1);
  const int32_t* perm = I.perm + I.fm.perm;
  G* grid = static_cast<G*>(a.out[inst_]);
  for (int e = threadIdx.x; e < nl * m; e += kBlock) {
    int b, j;
    divmod<P2>(e, m, &b, &j);
    // (power-of-two lengths: the DIF position from the index, no table)
    const int pos = P2 ? dif_position_p2(I.fm, j) : perm[j];
    GridIO<T, G>::st(grid, (size_t)line0 * m + e, buf[b * m + pos]);
  }
  PAT_END_ITEM
}

// Stage a2 alone (the staged and bf16-grid paths) as a software pipeline for
// one FP32 instance with the centred c = 2 grid and m = 2^LM points, the
// first half of k_line_nufft2_pipe_c: a persistent grid strides over line
// groups of 2048/m lines; each workgroup's first FFT stage takes the four
// nonzero samples per butterfly from registers loaded during the previous
// group, the radix plan is compile-time, the last stage writes natural
// order into an LDS buffer, and the grid lines leave it in coalesced stores.
template <typename G, int LM>
__global__ __launch_bounds__(kBlock, 4) void k_line_a2_pipe(StageArgs a) {
  using T = float;
  const Inst& I = *a.inst[0];
  constexpr int m = 1 << LM, nt = m / 2, lpw = 2048 / m;
  using PM = P2Plan<LM, p2_l16_m(LM)>;
  static_assert(PM::rad(0) == 8 && PM::nst >= 2, "pipelined first stage");
  constexpr int PADL = 4;
  auto pad = [](int i) { return i + (i >> PADL); };
  constexpr int sub = m >> 3, lsub = LM - 3;
  const int j = (int)threadIdx.x & (sub - 1), bb = (int)threadIdx.x >> lsub;
  const cx<T>* twm = static_cast<const cx<T>*>(I.tw) + I.fm.tw;
  cx<T>* gn = reinterpret_cast<cx<T>*>(pat_smem);  // grid lines, natural order
  cx<T>* gp = gn + lpw * m;                          // FFT scratch, padded
  const T* sn = static_cast<const T*>(I.sn);
  const int q = nt >> 2;
  // inputs r = 0, 1, 6, 7 of the butterfly: samples j + nt/2, j + 3nt/4, j, j + nt/4
  const int ns[4] = {j + 2 * q, j + 3 * q, j, j + q};
  T snr[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) snr[i] = sn[ns[i]];
  const cx<T> w1 = twm[j];
  const cx<T>* in = static_cast<const cx<T>*>(a.in[0]);
  G* grid = static_cast<G*>(a.out[0]);
  cx<T> pre[4];
  auto fetch = [&](int item) {
    const int line = item * lpw + bb;
    const bool ok = line < I.lines;
    const cx<T>* gin = in + (size_t)line * nt;
#pragma unroll
    for (int i = 0; i < 4; ++i) pre[i] = ok ? gin[ns[i]] : mk(T(0), T(0));
  };
  constexpr int step = m / PM::rad(PM::nst - 1);
  int item = blockIdx.x;
  if (item < a.total) fetch(item);
  for (; item < a.total; item += gridDim.x) {
    const int line0 = item * lpw;
    const int nl = min(lpw, I.lines - line0);
    {
      cx<T> v[8];
      v[0] = cscl(pre[0], snr[0]);
      v[1] = cscl(pre[1], snr[1]);
      v[2] = v[3] = v[4] = v[5] = mk(T(0), T(0));
      v[6] = cscl(pre[2], snr[2]);
      v[7] = cscl(pre[3], snr[3]);
      dft_pow2<T, 8>(v);
      twiddle_pow2<T, 8>(v, w1);
#pragma unroll
      for (int r = 0; r < 8; ++r) gp[pad(bb * m + j + r * sub)] = v[r];
    }
    __syncthreads();
    p2_stages<T, LM, 1, p2_l16_m(LM), PADL>(gp, twm, lpw);
    if (item + (int)gridDim.x < a.total) fetch(item + gridDim.x);
    fft_last_stage_p2<T, PM::rad(PM::nst - 1), true, PADL>(gp, m, lpw, m, 1, [&](int b, int blk, const auto& v) {
      constexpr int R = sizeof(v) / sizeof(v[0]);
      cx<T>* g = gn + b * m;
      const int k0 = PM::natural(blk * R);
#pragma unroll
      for (int r = 0; r < R; ++r) g[k0 + r * step] = v[r];
    });
    __syncthreads();
    for (int e = threadIdx.x; e < nl * m; e += kBlock) GridIO<T, G>::st(grid, (size_t)line0 * m + e, gn[e]);
    __syncthreads();
  }
}

// transpose of a2 on LDS grids (natural order, conjugated on entry by the
// caller): X_n = s_n (inverse DFT of the grid line)[(n - nt/2) mod m]
template <typename T, int RS>
__device__ __forceinline__ void ifft_pick_deconv(const Inst& I, cx<T>* buf, int nl, cx<T>* x, const cx<T>* twm) {
  constexpr bool P2 = RS == 0;
  const int m = I.m, nt = I.nt;
  const T* sn = static_cast<const T*>(I.sn);
  fft_lds<T, RS, true>(buf, I.fm, twm, nl, m, 1);
  const int32_t* perm = I.perm + I.fm.perm;
  for (int e = threadIdx.x; e < nl * nt; e += kBlock) {
    int b, n;
    divmod<P2>(e, nt, &b, &n);
    int k = n - nt / 2;
    if (k < 0) k += m;
    // (power-of-two lengths: the DIF position from the index, no table)
    const int pos = P2 ? dif_position_p2(I.fm, k) : perm[k];
    x[e] = cscl(cconj(buf[b * m + pos]), sn[n]);
  }
}

template <typename T, typename G, int RS>
__global__ __launch_bounds__(kBlock) void k_line_a2t(StageArgs a) {
  constexpr bool P2 = RS == 0;
  PAT_FOR_EACH_ITEM(a)
  // the twiddle table in LDS before the lines, or read from memory (long
  // lines, power-of-two lengths: see k_line_a2)
  cx<T>* lds = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* buf = I.twg_m ? lds : lds + I.m;
  const bool twg = P2 || I.twg_m;
  const cx<T>* tw = twg ? static_cast<const cx<T>*>(I.tw) + I.fm.tw : lds;
  if (new_inst_ && !twg) load_twiddles(lds, I, I.fm);
  const int m = I.m, nt = I.nt;
  const int line0 = li * I.lpw_m;
  const int nl = min(I.lpw_m, I.lines - line0);
  const G* grid = static_cast<const G*>(a.in[inst_]);
  copy_batched<4>(
      nl * m, [&](int e) { return cconj(GridIO<T, G>::ld(grid, (size_t)line0 * m + e)); },
      [&](int e, cx<T> v) { buf[e] = v; });
  __syncthreads();
  ifft_pick_deconv<T, RS>(I, buf, nl, static_cast<cx<T>*>(a.out[inst_]) + (size_t)line0 * nt, tw);
  PAT_END_ITEM
}

// The transpose of a2 alone (the staged paths of R^T and A) as a software
// pipeline for one FP32 instance with the centred c = 2 grid and m = 2^LM
// points: a persistent grid strides over line groups of 2048/m lines; each
// workgroup stores its group's grid lines (conjugated) into a padded LDS
// scratch, issues the loads of the next group into registers, runs the
// compile-time FFT, and its last stage writes the picked, deconvolved time
// samples X_n = s_n conj(G_k), k = (n - nt/2) mod m, straight to memory.
template <typename G, int LM>
__global__ __launch_bounds__(kBlock, 4) void k_line_a2t_pipe(StageArgs a) {
  using T = float;
  const Inst& I = *a.inst[0];
  constexpr int m = 1 << LM, nt = m / 2, lpw = 2048 / m, per = 2048 / kBlock;
  using PM = P2Plan<LM, p2_l16_m(LM)>;
  static_assert(PM::nst >= 2, "two or more stages");
  constexpr int PADL = 4;
  auto pad = [](int i) { return i + (i >> PADL); };
  cx<T>* gp = reinterpret_cast<cx<T>*>(pat_smem);
  const cx<T>* twm = static_cast<const cx<T>*>(I.tw) + I.fm.tw;
  const T* sn = static_cast<const T*>(I.sn);
  const G* grid = static_cast<const G*>(a.in[0]);
  cx<T>* xout = static_cast<cx<T>*>(a.out[0]);
  const size_t npts = (size_t)I.lines * m;
  cx<T> pre[per];
  auto fetch = [&](int item) {
    const size_t base = (size_t)item * lpw * m;
#pragma unroll
    for (int u = 0; u < per; ++u) {
      const size_t e = base + threadIdx.x + u * kBlock;
      pre[u] = e < npts ? GridIO<T, G>::ld(grid, e) : mk(T(0), T(0));
    }
  };
  constexpr int step = m / PM::rad(PM::nst - 1);
  int item = blockIdx.x;
  if (item < a.total) fetch(item);
  for (; item < a.total; item += gridDim.x) {
    const int line0 = item * lpw;
    const int nl = min(lpw, I.lines - line0);
#pragma unroll
    for (int u = 0; u < per; ++u) gp[pad((int)threadIdx.x + u * kBlock)] = cconj(pre[u]);
    __syncthreads();
    if (item + (int)gridDim.x < a.total) fetch(item + gridDim.x);
    p2_stages<T, LM, 0, p2_l16_m(LM), PADL>(gp, twm, lpw);
    fft_last_stage_p2<T, PM::rad(PM::nst - 1), true, PADL>(gp, m, lpw, m, 1, [&](int b, int blk, const auto& v) {
      constexpr int R = sizeof(v) / sizeof(v[0]);
      if (b >= nl) return;
      const int k0 = PM::natural(blk * R);
      cx<T>* x = xout + (size_t)(line0 + b) * nt;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int n = (k0 + r * step + nt / 2) & (m - 1);
        if (n < nt) x[n] = cscl(cconj(v[r]), sn[n]);
      }
    });
    __syncthreads();
  }
}

// Four consecutive grid cells to memory (p 16-byte aligned for the vector
// forms; bf16 falls back to single cells otherwise).
template <typename T, typename G>
__device__ __forceinline__ void grid_store4(G* p, const cx<T>* v) {
  if constexpr (sizeof(G) == 8 && sizeof(T) == 4) {
    float4* q = reinterpret_cast<float4*>(p);
    q[0] = make_float4(v[0].x, v[0].y, v[1].x, v[1].y);
    q[1] = make_float4(v[2].x, v[2].y, v[3].x, v[3].y);
  } else if constexpr (sizeof(G) == 16) {
    double2* q = reinterpret_cast<double2*>(p);
#pragma unroll
    for (int c = 0; c < 4; ++c) q[c] = make_double2(v[c].x, v[c].y);
  } else {
    if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {
      uint4 u;
      u.x = (uint32_t)f2bf(v[0].x) | ((uint32_t)f2bf(v[0].y) << 16);
      u.y = (uint32_t)f2bf(v[1].x) | ((uint32_t)f2bf(v[1].y) << 16);
      u.z = (uint32_t)f2bf(v[2].x) | ((uint32_t)f2bf(v[2].y) << 16);
      u.w = (uint32_t)f2bf(v[3].x) | ((uint32_t)f2bf(v[3].y) << 16);
      *reinterpret_cast<uint4*>(p) = u;
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) GridIO<T, G>::st(p, c, v[c]);
    }
  }
}

// 16-byte chunks of a stored grid line: EPC elements per chunk, unpacked to
// compute precision and stored to LDS (dst is 16-byte aligned).
template <typename T, typename G>
struct GridChunk;
template <>
struct GridChunk<float, cx<float>> {
  static constexpr int EPC = 2;
  static __device__ __forceinline__ void put(uint4 v, cx<float>* dst) { *reinterpret_cast<uint4*>(dst) = v; }
};
template <>
struct GridChunk<double, cx<double>> {
  static constexpr int EPC = 1;
  static __device__ __forceinline__ void put(uint4 v, cx<double>* dst) { *reinterpret_cast<uint4*>(dst) = v; }
};
template <>
struct GridChunk<float, bf2> {
  static constexpr int EPC = 4;
  static __device__ __forceinline__ void put(uint4 v, cx<float>* dst) {
    float4 lo, hi;
    lo.x = __uint_as_float(v.x << 16);
    lo.y = __uint_as_float(v.x & 0xffff0000u);
    lo.z = __uint_as_float(v.y << 16);
    lo.w = __uint_as_float(v.y & 0xffff0000u);
    hi.x = __uint_as_float(v.z << 16);
    hi.y = __uint_as_float(v.z & 0xffff0000u);
    hi.z = __uint_as_float(v.w << 16);
    hi.w = __uint_as_float(v.w & 0xffff0000u);
    reinterpret_cast<float4*>(dst)[0] = lo;
    reinterpret_cast<float4*>(dst)[1] = hi;
  }
};

// a3 alone on the stored grid of one instance, streamed.  A persistent
// workgroup walks line groups (lpw_i lines) with stride gridDim.x; the next
// group's grid is loaded into registers (16-byte loads) before the current
// group is interpolated, so each workgroup keeps its memory requests in
// flight while it computes.  One LDS buffer of lpw_i lines (with a halo of
// TAPS - 1 and a stride rounded to 16 bytes), refilled after a barrier that
// follows the interpolation: half the LDS of a double buffer, so one more
// workgroup fits a compute unit, which is worth the extra barrier.
template <typename T, typename G, int TAPS, bool P2, int NPRE>
__global__ __launch_bounds__(kBlock) void k_line_interp_stream(StageArgs a) {
  using C = GridChunk<T, G>;
  constexpr int EPC = C::EPC;
  constexpr int H = TAPS - 1;
  constexpr int Q = 16 / (int)sizeof(cx<T>) > 0 ? 16 / (int)sizeof(cx<T>) : 1;
  const Inst& I = *a.inst[0];
  const int m = I.m, nz = I.nz, lpw = I.lpw_i, lines = I.lines;
  const int ls = (m + H + Q - 1) / Q * Q;
  const int ngroups = a.total;
  const G* grid = static_cast<const G*>(a.in[0]);
  cx<T>* out = static_cast<cx<T>*>(a.out[0]);
  cx<T>* bufs = reinterpret_cast<cx<T>*>(pat_smem);
  __shared__ double s_ak[2][16];
  uint4 pre[NPRE];
  auto fetch = [&](int g) {
    const int line0 = g * lpw;
    const int nch = min(lpw, lines - line0) * m / EPC;
    const uint4* src = reinterpret_cast<const uint4*>(grid + (size_t)line0 * m);
#pragma unroll
    for (int u = 0; u < NPRE; ++u) {
      const int c = (int)threadIdx.x + u * kBlock;
      if (c < nch) pre[u] = src[c];
    }
  };
  int g = blockIdx.x;
  if (g >= ngroups) return;
  fetch(g);
  for (int k = 0; g < ngroups; g += gridDim.x, ++k) {
    cx<T>* buf = bufs;
    const int line0 = g * lpw;
    const int nl = min(lpw, lines - line0);
    const int nch = nl * m / EPC;
#pragma unroll
    for (int u = 0; u < NPRE; ++u) {
      const int c = (int)threadIdx.x + u * kBlock;
      if (c < nch) {
        int b, j;
        divmod<P2>(c * EPC, m, &b, &j);
        cx<T>* dst = buf + b * ls + j;
        C::put(pre[u], dst);
        if (j < H) {
#pragma unroll
          for (int e = 0; e < EPC; ++e)
            if (j + e < H) dst[m + e] = dst[e];
        }
      }
    }
    if ((int)threadIdx.x < nl) s_ak[k & 1][threadIdx.x] = line_ak(I, line0 + (int)threadIdx.x);
    if (g + (int)gridDim.x < ngroups) fetch(g + (int)gridDim.x);
    __syncthreads();
    cx<T>* o = out + (size_t)line0 * nz;
    const double* akk = s_ak[k & 1];
    interp_lines<T, TAPS, true, P2>(I, a, buf, ls, [&](int b) { return akk[b]; }, nl, a.mode,
                                    [&](int e, cx<T> v) { o[e] = v; });
    __syncthreads();  // every read of the buffer is done before it is refilled
  }
}

// a3 alone: grid lines from memory, weighted node values to memory.
template <typename T, typename G, int TAPS, bool P2>
__global__ __launch_bounds__(kBlock) void k_line_interp(StageArgs a) {
  cx<T>* buf = reinterpret_cast<cx<T>*>(pat_smem);
  __shared__ double s_ak[16];
  PAT_FOR_EACH_ITEM(a)
  const int m = I.m, nz = I.nz;
  const int line0 = li * I.lpw_i;
  const int nl = min(I.lpw_i, I.lines - line0);
  const bool pairs = TAPS > 0 && a.pair_ok;
  const int H = pairs ? TAPS - 1 : 0;
  const int ls = m + H;
  const G* grid = static_cast<const G*>(a.in[inst_]);
  copy_batched<4>(
      nl * m, [&](int e) { return GridIO<T, G>::ld(grid, (size_t)line0 * m + e); },
      [&](int e, cx<T> v) {
        const int b = e / m;
        const int j = e - b * m;
        buf[b * ls + j] = v;
        if (j < H) buf[b * ls + m + j] = v;
      });
  if (threadIdx.x < nl) s_ak[threadIdx.x] = line_ak(I, line0 + threadIdx.x);
  __syncthreads();
  cx<T>* out = static_cast<cx<T>*>(a.out[inst_]) + (size_t)line0 * nz;
  if (pairs) {
    interp_lines<T, (TAPS > 0 ? TAPS : 2), true, P2>(I, a, buf, ls, [&](int b) { return s_ak[b]; }, nl, a.mode,
                                                     [&](int e, cx<T> v) { out[e] = v; });
  } else {
    interp_lines<T, 0, false, P2>(I, a, buf, ls, [&](int b) { return s_ak[b]; }, nl, a.mode,
                                  [&](int e, cx<T> v) { out[e] = v; });
  }
  PAT_END_ITEM
}

// spreading alone: depth spectra from memory, grid lines to memory.
template <typename T, typename G, int TAPS>
__global__ __launch_bounds__(kBlock) void k_line_spread(StageArgs a) {
  PAT_FOR_EACH_ITEM(a)
  const SpreadLds<T> L = SpreadLds<T>::carve(pat_smem, I.nz, I.taps);
  const cx<T>* F = static_cast<const cx<T>*>(a.in[inst_]) + (size_t)li * I.nz;
  G* grid = static_cast<G*>(a.out[inst_]);
  const size_t row = (size_t)li * I.m;
  auto fget = [&](int l) { return F[l]; };
  auto put = [&](int j, cx<T> v) { GridIO<T, G>::st(grid, row + j, v); };
  auto put4 = [&](int j, const cx<T>* v) { grid_store4<T, G>(grid + row + j, v); };
  if (TAPS > 0 && a.pair_ok) {
    spread_line<T, (TAPS > 0 ? TAPS : 2), true>(I, a, li, a.mode, L, fget, put, put4);
  } else {
    spread_line<T, 0, false>(I, a, li, a.mode, L, fget, put, put4);
  }
  PAT_END_ITEM
}

// Fused a2 + a3 + inverse depth DFT (operators R and A^T): per group of nl
// lines, the detector spectrum is deconvolved, padded and transformed in
// LDS, brought to natural order, interpolated at the line's nodes, and the
// node values are inverse-transformed over depth before the only store.
template <typename T, int RS, int TAPS>
__global__ __launch_bounds__(kBlock) void k_line_nufft2(StageArgs a) {
  constexpr bool P2 = RS == 0;
  PAT_FOR_EACH_ITEM(a)
  const int m = I.m, nt = I.nt, nz = I.nz;
  const int lpw = I.lpw_f;
  const int line0 = li * lpw;
  const int nl = min(lpw, I.lines - line0);
  const bool pairs = TAPS > 0 && a.pair_ok;
  // (no halo: the rare windows that run past the end of a line wrap their
  // taps, which keeps two lines' buffers within 32 KB of LDS)
  const int ls = m;
  auto ak = [&](int b) { return line_ak(I, line0 + b); };
  const int sp = m > nz ? m : nz;
  // (twiddles stay in global memory here: an LDS copy costs this kernel a
  // resident workgroup per CU and the strided reads conflict on banks)
  const cx<T>* twm = static_cast<const cx<T>*>(I.tw) + I.fm.tw;
  const cx<T>* twz = static_cast<const cx<T>*>(I.tw) + I.fz.tw;
  cx<T>* gp = reinterpret_cast<cx<T>*>(pat_smem);  // FFT output (permuted order), later the depth line
  cx<T>* gn = gp + lpw * sp;                         // grid in natural order, with halo
  const cx<T>* gin = static_cast<const cx<T>*>(a.in[inst_]) + (size_t)line0 * nt;
  if constexpr (P2) {
    // the first FFT stage reads the deconvolved, centred samples from memory
    // (grid position j holds sample (j + nt/2) mod m, zero from nt on); the
    // last writes the grid in natural order (with its halo)
    const T* sn = static_cast<const T*>(I.sn);
    auto src = [&](int b, int j) {
      int n = j + nt / 2;
      if (n >= m) n -= m;
      return n < nt ? cscl(gin[(size_t)b * nt + n], sn[n]) : mk(T(0), T(0));
    };
    const int step = m / I.fm.rad[I.fm.nst - 1];  // weight of the last digit in k
    fft_lds_p2_src_sink<T, true>(gp, I.fm, twm, nl, m, 1, src, [&](int b, int blk, const auto& v) {
      constexpr int R = sizeof(v) / sizeof(v[0]);
      cx<T>* g = gn + b * ls;
      const int k0 = dif_natural_p2(I.fm, blk * R);
#pragma unroll
      for (int r = 0; r < R; ++r) g[k0 + r * step] = v[r];
    });
  } else {
    load_deconv_pad<T, P2>(I, gin, nl, gp);
    __syncthreads();
    fft_lds<T, RS, true>(gp, I.fm, twm, nl, m, 1);
    const int32_t* permm = I.perm + I.fm.perm;
    for (int e = threadIdx.x; e < nl * m; e += kBlock) {
      int b, j;
      divmod<P2>(e, m, &b, &j);
      gn[b * ls + j] = gp[b * m + permm[j]];
    }
    __syncthreads();
  }
  cx<T>* fz = gp;  // the permuted grid is no longer needed
  if (pairs) {
    interp_lines<T, (TAPS > 0 ? TAPS : 2), true, P2, false>(I, a, gn, ls, ak, nl, a.mode,
                                                            [&](int e, cx<T> v) { fz[e] = cconj(v); });
  } else {
    interp_lines<T, 0, false, P2>(I, a, gn, ls, ak, nl, a.mode, [&](int e, cx<T> v) { fz[e] = cconj(v); });
  }
  __syncthreads();
  cx<T>* out = static_cast<cx<T>*>(a.out[inst_]) + (size_t)line0 * nz;
  if constexpr (P2) {
    // the last stage stores each output at its natural position: for a given
    // r, a wave's butterflies cover one contiguous run of the line
    const int stepz = nz / I.fz.rad[I.fz.nst - 1];
    fft_lds_p2_sink<T, true>(fz, I.fz, twz, nl, nz, 1, [&](int b, int blk, const auto& v) {
      constexpr int R = sizeof(v) / sizeof(v[0]);
      cx<T>* o = out + b * nz;
      const int k0 = dif_natural_p2(I.fz, blk * R);
#pragma unroll
      for (int r = 0; r < R; ++r) o[k0 + r * stepz] = cconj(v[r]);
    });
  } else {
    fft_lds<T, RS, true>(fz, I.fz, twz, nl, nz, 1);
    const int32_t* permz = I.perm + I.fz.perm;
    for (int e = threadIdx.x; e < nl * nz; e += kBlock) {
      int b, j;
      divmod<P2>(e, nz, &b, &j);
      out[e] = cconj(fz[b * nz + permz[j]]);
    }
  }
  PAT_END_ITEM
}

// k_line_nufft2 as a software pipeline for one FP32 instance with c = 2
// (m = 2 nt), power-of-two lengths, a first radix of 8 and exactly one
// first-stage butterfly per thread ((m / 8) lpw_f = kBlock).  With c = 2 and
// the centred padding, butterfly j of a line takes the samples j, j + nt/4,
// j + nt/2 and j + 3nt/4 (the other four inputs are zeros).  A persistent grid
// strides over the line groups; each workgroup loads its next group's
// samples into registers before the last stage of the oversampled FFT, so
// they are in flight through that stage and the interpolation, which load
// nothing else from memory.  The deconvolution factors and the first-stage
// twiddle of a thread are the same for every group and are read once.
template <typename T, int TAPS>
__global__ __launch_bounds__(kBlock, 5) void k_line_nufft2_pipe(StageArgs a) {
  const Inst& I = *a.inst[0];
  const int m = I.m, nt = I.nt, nz = I.nz, lpw = I.lpw_f;
  const int sub = m >> 3, lsub = __builtin_ctz((unsigned)sub);
  const int j = (int)threadIdx.x & (sub - 1), bb = (int)threadIdx.x >> lsub;
  const cx<T>* twm = static_cast<const cx<T>*>(I.tw) + I.fm.tw;
  const cx<T>* twz = static_cast<const cx<T>*>(I.tw) + I.fz.tw;
  cx<T>* gp = reinterpret_cast<cx<T>*>(pat_smem);  // FFT scratch, later the depth lines
  cx<T>* gn = gp + lpw * m;                          // grid lines in natural order
  const T* sn = static_cast<const T*>(I.sn);
  const int q = nt >> 2;
  // inputs r = 0, 1, 6, 7 of the butterfly: samples j + nt/2, j + 3nt/4, j, j + nt/4
  const int ns[4] = {j + 2 * q, j + 3 * q, j, j + q};
  T snr[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) snr[i] = sn[ns[i]];
  const cx<T> w1 = twm[j];
  const cx<T>* in = static_cast<const cx<T>*>(a.in[0]);
  cx<T>* outb = static_cast<cx<T>*>(a.out[0]);
  cx<T> pre[4];
  auto fetch = [&](int item) {
    const int line0 = item * lpw;
    const bool ok = line0 + bb < I.lines;
    const cx<T>* gin = in + (size_t)(line0 + bb) * nt;
#pragma unroll
    for (int i = 0; i < 4; ++i) pre[i] = ok ? gin[ns[i]] : mk(T(0), T(0));
  };
  const int step = m / I.fm.rad[I.fm.nst - 1];
  const int stepz = nz / I.fz.rad[I.fz.nst - 1];
  int item = blockIdx.x;
  if (item < a.total) fetch(item);
  for (; item < a.total; item += gridDim.x) {
    const int line0 = item * lpw;
    const int nl = min(lpw, I.lines - line0);
    {
      cx<T> v[8];
      v[0] = cscl(pre[0], snr[0]);
      v[1] = cscl(pre[1], snr[1]);
      v[2] = v[3] = v[4] = v[5] = mk(T(0), T(0));
      v[6] = cscl(pre[2], snr[2]);
      v[7] = cscl(pre[3], snr[3]);
      dft_pow2<T, 8>(v);
      twiddle_pow2<T, 8>(v, w1);
      cx<T>* p = gp + bb * m + j;
#pragma unroll
      for (int r = 0; r < 8; ++r) p[r * sub] = v[r];
    }
    __syncthreads();
    int Li = sub;
    for (int s = 1; s + 1 < I.fm.nst; ++s) {
      const int R = I.fm.rad[s];
      if (R == 8) fft_stage<T, 8, true, true>(gp, Li, m, twm, lpw, m, 1);
      else if (R == 4) fft_stage<T, 4, true, true>(gp, Li, m, twm, lpw, m, 1);
      else fft_stage<T, 2, true, true>(gp, Li, m, twm, lpw, m, 1);
      __syncthreads();
      Li /= R;
    }
    if (item + (int)gridDim.x < a.total) fetch(item + gridDim.x);
    auto sink = [&](int b, int blk, const auto& v) {
      constexpr int R = sizeof(v) / sizeof(v[0]);
      cx<T>* g = gn + b * m;
      const int k0 = dif_natural_p2(I.fm, blk * R);
#pragma unroll
      for (int r = 0; r < R; ++r) g[k0 + r * step] = v[r];
    };
    {
      const int R = I.fm.rad[I.fm.nst - 1];
      if (R == 8) fft_last_stage_p2<T, 8, true>(gp, m, lpw, m, 1, sink);
      else if (R == 4) fft_last_stage_p2<T, 4, true>(gp, m, lpw, m, 1, sink);
      else fft_last_stage_p2<T, 2, true>(gp, m, lpw, m, 1, sink);
    }
    __syncthreads();
    cx<T>* fz = gp;
    interp_lines<T, TAPS, true, true, false>(I, a, gn, m, [&](int b) { return line_ak(I, line0 + b); }, nl, a.mode,
                                             [&](int e, cx<T> v) { fz[e] = cconj(v); });
    __syncthreads();
    cx<T>* out = outb + (size_t)line0 * nz;
    fft_lds_p2_sink<T, true>(fz, I.fz, twz, nl, nz, 1, [&](int b, int blk, const auto& v) {
      constexpr int R = sizeof(v) / sizeof(v[0]);
      cx<T>* o = out + b * nz;
      const int k0 = dif_natural_p2(I.fz, blk * R);
#pragma unroll
      for (int r = 0; r < R; ++r) o[k0 + r * stepz] = cconj(v[r]);
    });
  }
}

// k_line_nufft2_pipe for m = 2^LM and nz = 2^LZ known at compile time (the
// line group then holds 2^(11 - LM) lines): the same work, with the FFT
// stages, their loops and the output positions fixed by P2Plan.  Bounded at
// four waves per SIMD (128 registers): a five-wave cap (96) made several
// instances spill, while those that need no more than 96 still run five.
// In FP64 (twice the registers and LDS) at two.
template <typename T, int TAPS, int LM, int LZ>
__global__ __launch_bounds__(kBlock, sizeof(T) == 4 ? 4 : 2) void k_line_nufft2_pipe_c(StageArgs a) {
  const Inst& I = *a.inst[0];
  constexpr int m = 1 << LM, nt = m / 2, nz = 1 << LZ, lpw = 2048 / m;
  using PM = P2Plan<LM, p2_l16_m(LM)>;
  using PZ = P2Plan<LZ, p2_l16_z(LZ)>;
  static_assert(PM::rad(0) == 8 && PM::nst >= 2 && LZ <= LM, "pipelined first stage");
  const int sub = m >> 3, lsub = __builtin_ctz((unsigned)sub);
  const int j = (int)threadIdx.x & (sub - 1), bb = (int)threadIdx.x >> lsub;
  const cx<T>* twm = static_cast<const cx<T>*>(I.tw) + I.fm.tw;
  const cx<T>* twz = static_cast<const cx<T>*>(I.tw) + I.fz.tw;
  // grid lines in natural order at the start of LDS (the tap reads then take
  // their offsets as immediates), then the FFT scratch (later the depth
  // lines), padded by one point every 16: its strided stages spread over the
  // LDS banks
  constexpr int PADL = 4;
  auto pad = [](int i) { return i + (i >> PADL); };
  cx<T>* gn = reinterpret_cast<cx<T>*>(pat_smem);
  cx<T>* gp = gn + lpw * m;
  const T* sn = static_cast<const T*>(I.sn);
  const int q = nt >> 2;
  // inputs r = 0, 1, 6, 7 of the butterfly: samples j + nt/2, j + 3nt/4, j, j + nt/4
  const int ns[4] = {j + 2 * q, j + 3 * q, j, j + q};
  T snr[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) snr[i] = sn[ns[i]];
  const cx<T> w1 = twm[j];
  const cx<T>* in = static_cast<const cx<T>*>(a.in[0]);
  cx<T>* outb = static_cast<cx<T>*>(a.out[0]);
  cx<T> pre[4];
  auto fetch = [&](int item) {
    const int line0 = item * lpw;
    const bool ok = line0 + bb < I.lines;
    const cx<T>* gin = in + (size_t)(line0 + bb) * nt;
#pragma unroll
    for (int i = 0; i < 4; ++i) pre[i] = ok ? gin[ns[i]] : mk(T(0), T(0));
  };
  constexpr int step = m / PM::rad(PM::nst - 1);
  constexpr int stepz = nz / PZ::rad(PZ::nst - 1);
  int item = blockIdx.x;
  if (item < a.total) fetch(item);
  for (; item < a.total; item += gridDim.x) {
    const int line0 = item * lpw;
    const int nl = min(lpw, I.lines - line0);
    {
      cx<T> v[8];
      v[0] = cscl(pre[0], snr[0]);
      v[1] = cscl(pre[1], snr[1]);
      v[2] = v[3] = v[4] = v[5] = mk(T(0), T(0));
      v[6] = cscl(pre[2], snr[2]);
      v[7] = cscl(pre[3], snr[3]);
      dft_pow2<T, 8>(v);
      twiddle_pow2<T, 8>(v, w1);
#pragma unroll
      for (int r = 0; r < 8; ++r) gp[pad(bb * m + j + r * sub)] = v[r];
    }
    __syncthreads();
    p2_stages<T, LM, 1, p2_l16_m(LM), PADL>(gp, twm, lpw);
    if (item + (int)gridDim.x < a.total) fetch(item + gridDim.x);
    auto sink = [&](int b, int blk, const auto& v) {
      constexpr int R = sizeof(v) / sizeof(v[0]);
      cx<T>* g = gn + b * m;
      const int k0 = PM::natural(blk * R);
#pragma unroll
      for (int r = 0; r < R; ++r) g[k0 + r * step] = v[r];
    };
    fft_last_stage_p2<T, PM::rad(PM::nst - 1), true, PADL>(gp, m, lpw, m, 1, sink);
    __syncthreads();
    cx<T>* fz = gp;
    interp_lines<T, TAPS, true, true, false>(I, a, gn, m, [&](int b) { return line_ak<true>(I, line0 + b); }, nl, a.mode,
                                             [&](int e, cx<T> v) { fz[pad(e)] = cconj(v); });
    __syncthreads();
    cx<T>* out = outb + (size_t)line0 * nz;
    p2_stages<T, LZ, 0, p2_l16_z(LZ), PADL>(fz, twz, lpw);
    fft_last_stage_p2<T, PZ::rad(PZ::nst - 1), true, PADL>(fz, nz, lpw, nz, 1, [&](int b, int blk, const auto& v) {
      constexpr int R = sizeof(v) / sizeof(v[0]);
      if (b >= nl) return;
      cx<T>* o = out + b * nz;
      const int k0 = PZ::natural(blk * R);
#pragma unroll
      for (int r = 0; r < R; ++r) o[k0 + r * stepz] = cconj(v[r]);
    });
    __syncthreads();
  }
}

// Entries k < L / r of the twiddle table that the twiddled stages (all but
// the last) of a compile-time plan read, r the smallest of their radices.
template <typename Pl, int L>
constexpr int twiddle_extent() {
  int r = 16;
  for (int s = 0; s + 1 < Pl::nst; ++s) r = Pl::rad(s) < r ? Pl::rad(s) : r;
  return L / r;
}
// Waves per SIMD of k_line_nufft2_mirror: four in FP32, two in FP64 (its
// registers).
template <typename T>
constexpr int mirror_waves() { return sizeof(T) == 4 ? 4 : 2; }
// LDS of k_line_nufft2_mirror with NT threads: its 16 NT padded points, the
// twiddles of both FFTs' twiddled stages and, where the workgroups of
// mirror_waves per SIMD still fit in 160 KB, the deconvolution factors s_n.
template <typename T, int LM, int NT>
struct MirrorLds {
  static constexpr int m = 1 << LM, nt = m / 2, nz = m / 4, P = 16 * NT, cs = 2 * (int)sizeof(T);
  static constexpr int TWM = twiddle_extent<P2Plan<LM, p2_l16_m(LM)>, m>();
  static constexpr int TWZ = twiddle_extent<P2Plan<LM - 2, p2_l16_z(LM - 2)>, nz>();
  static constexpr int kPts = P + (P >> 4);
  static constexpr int kTw = (TWM + TWZ) * cs, kSn = nt * (int)sizeof(T);
  static constexpr int kGroups = 4 * mirror_waves<T>() * 64 / NT;  // workgroups per CU
  static constexpr bool SN = (kPts * cs + kTw + kSn) * kGroups <= 160 * 1024;
  static constexpr int bytes = kPts * cs + kTw + (SN ? kSn : 0);
  static constexpr bool fits = bytes * kGroups <= 160 * 1024;
};
static_assert(MirrorLds<float, 10, 256>::TWM == 128 && MirrorLds<float, 10, 256>::TWZ == 64 &&
                  MirrorLds<float, 10, 256>::SN && !MirrorLds<float, 11, 256>::SN &&
                  MirrorLds<float, 11, 256>::fits && MirrorLds<float, 10, 128>::fits &&
                  MirrorLds<double, 10, 128>::fits && MirrorLds<double, 11, 256>::fits,
              "the resident waves per SIMD fit in LDS");

// k_line_nufft2_pipe_c for R on 3D plans whose depth lines are a quarter of
// the grid lines (nz = m/4, m = 2^LM), with NT threads: a work item holds
// NL = 16 NT/m lines, taken in mirror pairs (mirror_line), in 16 NT padded
// points of LDS (four waves per SIMD in FP32, two in FP64).  Each thread runs
// two first-stage butterflies, and in the interpolation one node pair of one
// mirror pair: its window, phase and weight serve both lines (the two lines
// of a pair with r = 0 form their own).  The last grid-FFT stage works in
// place: every thread reads its butterflies' 16 points, and after a barrier
// writes them in natural order over the scratch; the interpolation outputs
// wait in registers for a barrier and then overwrite the grid as the depth
// lines.
//
// BF: the stages after the grid alone.  The grid lines come from memory, in bf16
// as k_line_a2_pipe stores them, in place of the grid FFT.  (Rounding the FFT's
// result in LDS instead took 92 us for all of it, but the compiler contracts
// the two copies of the FFT differently: bf16 roundings then flip now and then,
// up to 1.5e-5 of the output's norm, where FP32 rounding leaves 2e-7.)
template <typename T, int TAPS, int LM, int LZ, int NT, bool BF = false>
__global__ __launch_bounds__(NT, mirror_waves<T>()) void k_line_nufft2_mirror(StageArgs a) {
  const Inst& I = *a.inst[0];
  constexpr int m = 1 << LM, nt = m / 2, nz = 1 << LZ, NL = 16 * NT / m, half = nz / 2;
  using PM = P2Plan<LM, p2_l16_m(LM)>;
  using PZ = P2Plan<LZ, p2_l16_z(LZ)>;
  static_assert(LZ == LM - 2 && NL >= 2 && (NL / 2) * half == NT, "one node pair of one mirror pair per thread");
  static_assert(PM::rad(0) == 8 && PM::nst >= 2, "pipelined first stage");
  constexpr int PADL = 4;
  constexpr int LS = m + (m >> PADL);  // line stride in LDS
  auto pad = [](int i) { return i + (i >> PADL); };
  constexpr int sub = m >> 3, lsub = LM - 3;
  constexpr int LPP = NT / sub;  // lines of one pass of first-stage butterflies (NL / 2)
  const int j = (int)threadIdx.x & (sub - 1), bb = (int)threadIdx.x >> lsub;
  using ML = MirrorLds<T, LM, NT>;
  cx<T>* buf = reinterpret_cast<cx<T>*>(pat_smem);
  // the item-invariant tables, copied once into LDS after the points (read
  // at every item, they would otherwise wait on the L2 there)
  cx<T>* twm = buf + ML::kPts;
  cx<T>* twz = twm + ML::TWM;
  T* snl = reinterpret_cast<T*>(twz + ML::TWZ);
  {
    const cx<T>* gm = static_cast<const cx<T>*>(I.tw) + I.fm.tw;
    const cx<T>* gz = static_cast<const cx<T>*>(I.tw) + I.fz.tw;
    for (int i = threadIdx.x; i < ML::TWM; i += NT) twm[i] = gm[i];
    for (int i = threadIdx.x; i < ML::TWZ; i += NT) twz[i] = gz[i];
    if constexpr (ML::SN) {
      const T* gs = static_cast<const T*>(I.sn);
      for (int i = threadIdx.x; i < nt; i += NT) snl[i] = gs[i];
    }
    __syncthreads();
  }
  auto sn_at = [&](int n) {
    if constexpr (ML::SN) return snl[n];
    return static_cast<const T*>(I.sn)[n];
  };
  const int q = nt >> 2;
  // inputs r = 0, 1, 6, 7 of a butterfly: samples j + nt/2, j + 3nt/4, j, j + nt/4
  // (formed where used: nothing per thread is held across the item loop that
  // can be recomputed)
  auto ns = [&](int i) { return j + (i == 0 ? 2 * q : i == 1 ? 3 * q : i == 2 ? 0 : q); };
  const cx<T>* in = static_cast<const cx<T>*>(a.in[0]);
  cx<T>* outb = static_cast<cx<T>*>(a.out[0]);
  const int lines = I.lines;
  cx<T> pre[2][4];
  // (where a wavefront's butterflies lie in one line, its line index is
  // wave-uniform and taken into scalar registers, so that the line
  // arithmetic and the row address run on the scalar unit)
  constexpr bool WU = sub >= 64;
  auto uni = [](int v) { return WU ? __builtin_amdgcn_readfirstlane(v) : v; };
  uint4 raw[4];  // (BF: four grid values each, points 4 (thread + u NT) ..)
  auto fetch = [&](int item) {
    if constexpr (BF) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = 4 * ((int)threadIdx.x + u * NT), slot = item * NL + (e >> LM);
        bool sh;
        const int row = slot < lines ? mirror_line<true>(I, slot, &sh) : 0;
        raw[u] = *reinterpret_cast<const uint4*>(static_cast<const bf2*>(a.in[0]) + ((size_t)row << LM) + (e & (m - 1)));
      }
      return;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int slot = uni(item * NL + bb + u * LPP);
      const bool ok = slot < lines;
      bool sh;
      const cx<T>* gin = in + (size_t)uni(ok ? mirror_line<true>(I, slot, &sh) : 0) * nt;
#pragma unroll
      for (int i = 0; i < 4; ++i) pre[u][i] = ok ? gin[ns(i)] : mk(T(0), T(0));
    }
  };
  constexpr int RL = PM::rad(PM::nst - 1), LRL = RL == 16 ? 4 : RL == 8 ? 3 : RL == 4 ? 2 : 1;
  constexpr int NB = 16 / RL;  // last-stage butterflies per thread
  constexpr int step = m / RL;
  constexpr int stepz = nz / PZ::rad(PZ::nst - 1);
  const double wsc = I.wcoef * I.scale;
  int item = blockIdx.x;
  if (item < a.total) fetch(item);
  for (; item < a.total; item += gridDim.x) {
    const int line0 = item * NL;
    const int nl = min(NL, lines - line0);
    if constexpr (BF) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = 4 * ((int)threadIdx.x + u * NT);
        cx<T>* g = buf + (e >> LM) * LS + (e & (m - 1));
        const uint32_t w[4] = {raw[u].x, raw[u].y, raw[u].z, raw[u].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) g[i] = mk(bf2f((uint16_t)w[i]), bf2f((uint16_t)(w[i] >> 16)));
      }
      if (item + (int)gridDim.x < a.total) fetch(item + gridDim.x);
    } else {
    // (the deconvolution factors and the first twiddle are read per item, not
    // held across it: the registers go to the later phases)
    T snr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) snr[i] = sn_at(ns(i));
    const cx<T> w1 = twm[j];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      cx<T> v[8];
      v[0] = cscl(pre[u][0], snr[0]);
      v[1] = cscl(pre[u][1], snr[1]);
      v[2] = v[3] = v[4] = v[5] = mk(T(0), T(0));
      v[6] = cscl(pre[u][2], snr[2]);
      v[7] = cscl(pre[u][3], snr[3]);
      dft_pow2<T, 8>(v);
      twiddle_pow2<T, 8>(v, w1);
      const int b = bb + u * LPP;
#pragma unroll
      for (int r = 0; r < 8; ++r) buf[pad(b * m + j + r * sub)] = v[r];
    }
    __syncthreads();
    p2_stages<T, LM, 1, p2_l16_m(LM), PADL, NT>(buf, twm, NL);
    if (item + (int)gridDim.x < a.total) fetch(item + gridDim.x);
    {
      // last grid stage, in place: read, barrier, write in natural order
      // (line b at buf + b LS, unpadded within its line)
      cx<T> lv[NB][RL];
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int id = (int)threadIdx.x + u * NT;
        const int b = id >> (LM - LRL), blk = id & ((m >> LRL) - 1);
        const cx<T>* p = buf + pad(b * m + blk * RL);
#pragma unroll
        for (int r = 0; r < RL; ++r) lv[u][r] = p[r];
        dft_pow2<T, RL>(lv[u]);
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int id = (int)threadIdx.x + u * NT;
        const int b = id >> (LM - LRL), blk = id & ((m >> LRL) - 1);
        cx<T>* g = buf + b * LS;
        const int k0 = PM::natural(blk * RL);
#pragma unroll
        for (int r = 0; r < RL; ++r) g[k0 + r * step] = lv[u][r];
      }
    }
    }
    __syncthreads();
    {
      // interpolation (R: |l| = 1 .. nz/2, node pairs +-nu+): node pair p of
      // mirror pair h
      // (h is wave-uniform from half = 64 on)
      constexpr bool HU = half >= 64;
      auto hu = [](int v) { return HU ? __builtin_amdgcn_readfirstlane(v) : v; };
      const int h = hu((int)threadIdx.x >> (LZ - 1)), la = ((int)threadIdx.x & (half - 1)) + 1;
      const bool act = 2 * h < nl;
      cx<T> o[4] = {mk(T(0), T(0)), mk(T(0), T(0)), mk(T(0), T(0)), mk(T(0), T(0))};
      if (act) {
        bool sh, sh1;
        const int L0 = hu(mirror_line<true>(I, line0 + 2 * h, &sh));
        const int L1 = hu(mirror_line<true>(I, line0 + 2 * h + 1, &sh1));
        const double bl = I.b * (double)la * (double)la;
        double nup = sqrt_nt(line_ak<true>(I, L0) + bl);
        // (the weight, halved on the Nyquist lane, rides on the node phase)
        const double wla = wsc * (double)la * (la < half ? 1.0 : 0.5);
        PairWin<T, TAPS> pw;
        pair_window<T, TAPS, true>(nup, I, a, m, 0.0, pw);
        pw.ph = cscl(pw.ph, T(wla * rcp_nt(nup)));
        cx<T> vp, vn;
        pair_values<T, TAPS, false>(buf + 2 * h * LS, m, pw, &vp, &vn);
        if (la < half) {
          o[0] = vp;
          o[1] = vn;
        } else {
          o[0] = cadd(vp, vn);
        }
        if (!sh) {
          nup = sqrt_nt(line_ak<true>(I, L1) + bl);
          pair_window<T, TAPS, true>(nup, I, a, m, 0.0, pw);
          pw.ph = cscl(pw.ph, T(wla * rcp_nt(nup)));
        }
        pair_values<T, TAPS, false>(buf + (2 * h + 1) * LS, m, pw, &vp, &vn);
        if (la < half) {
          o[2] = vp;
          o[3] = vn;
        } else {
          o[2] = cadd(vp, vn);
        }
      }
      __syncthreads();
      // the depth lines over the grid: line b at b nz (padded); the Nyquist
      // lane also writes l = 0 (weight 0)
      const int e0 = 2 * h * nz, e1 = e0 + nz;
      const int lp = la < half ? la : half, ln = la < half ? nz - la : 0;
      buf[pad(e0 + lp)] = cconj(o[0]);
      buf[pad(e0 + ln)] = cconj(o[1]);
      buf[pad(e1 + lp)] = cconj(o[2]);
      buf[pad(e1 + ln)] = cconj(o[3]);
    }
    __syncthreads();
    p2_stages<T, LZ, 0, p2_l16_z(LZ), PADL, NT>(buf, twz, NL);
    fft_last_stage_p2<T, PZ::rad(PZ::nst - 1), true, PADL, NT>(buf, nz, NL, nz, 1, [&](int b, int blk, const auto& v) {
      constexpr int R = sizeof(v) / sizeof(v[0]);
      if (b >= nl) return;
      bool sh;
      cx<T>* o = outb + (size_t)mirror_line<true>(I, line0 + b, &sh) * nz;
      const int k0 = PZ::natural(blk * R);
#pragma unroll
      for (int r = 0; r < R; ++r) o[k0 + r * stepz] = cconj(v[r]);
    });
    __syncthreads();
  }
}

// Fused depth DFT + spreading + transposed a2 (operators R^T and A).  A work
// item holds lpw_a lines: their depth DFTs run together (power-of-two
// builds: the first stage reads the spectra from memory and the last writes
// them in natural order), then each line is spread onto the grid and
// transformed back, and only its time line is stored.
template <typename T, int RS, int TAPS>
__global__ __launch_bounds__(kBlock) void k_line_nufft1(StageArgs a) {
  constexpr bool P2 = RS == 0;
  PAT_FOR_EACH_ITEM(a)
  const int m = I.m, nz = I.nz, nt = I.nt;
  const int lpw = I.lpw_a;
  const int line0 = li * lpw;
  const int nl = min(lpw, I.lines - line0);
  const cx<T>* twm = static_cast<const cx<T>*>(I.tw) + I.fm.tw;  // (global, as in k_line_nufft2)
  const cx<T>* twz = static_cast<const cx<T>*>(I.tw) + I.fz.tw;
  const int sg = m > lpw * nz ? m : lpw * nz;
  cx<T>* grid = reinterpret_cast<cx<T>*>(pat_smem);  // depth-FFT scratch, then one grid line
  cx<T>* qn = grid + sg;                              // lpw depth spectra, natural order
  const SpreadLds<T, 2> L = SpreadLds<T, 2>::carve(qn + lpw * nz, nz, I.taps);
  const cx<T>* in = static_cast<const cx<T>*>(a.in[inst_]) + (size_t)line0 * nz;
  if constexpr (P2) {
    const int stepz = nz / I.fz.rad[I.fz.nst - 1];  // weight of the last digit in k
    fft_lds_p2_src_sink<T, true>(
        grid, I.fz, twz, nl, nz, 1, [&](int b, int pos) { return in[(size_t)b * nz + pos]; },
        [&](int b, int blk, const auto& v) {
          constexpr int R = sizeof(v) / sizeof(v[0]);
          cx<T>* d = qn + b * nz;
          const int k0 = dif_natural_p2(I.fz, blk * R);
#pragma unroll
          for (int r = 0; r < R; ++r) d[k0 + r * stepz] = v[r];
        });
  } else {
    copy_batched<2>(nl * nz, [&](int e) { return in[e]; }, [&](int e, cx<T> v) { grid[e] = v; });
    __syncthreads();
    fft_lds<T, RS, true>(grid, I.fz, twz, nl, nz, 1);
    const int32_t* permz = I.perm + I.fz.perm;
    for (int e = threadIdx.x; e < nl * nz; e += kBlock) {
      int b, l;
      divmod<P2>(e, nz, &b, &l);
      qn[e] = grid[b * nz + permz[l]];
    }
    __syncthreads();
  }
  auto put = [&](int j, cx<T> v) { grid[j] = cconj(v); };
  auto put4 = [&](int j, const cx<T>* v) {
#pragma unroll
    for (int c = 0; c < 2; ++c) grid[j + c] = cconj(v[c]);
  };
  for (int b = 0; b < nl; ++b) {
    // (spread_line's first barrier also ends every read of the previous
    // line's grid)
    const cx<T>* qb = qn + b * nz;
    auto fget = [&](int l) { return qb[l]; };
    if (TAPS > 0 && a.pair_ok) {
      spread_line<T, (TAPS > 0 ? TAPS : 2), true>(I, a, line0 + b, a.mode, L, fget, put, put4);
    } else {
      spread_line<T, 0, false>(I, a, line0 + b, a.mode, L, fget, put, put4);
    }
    __syncthreads();
    ifft_pick_deconv<T, RS>(I, grid, 1, static_cast<cx<T>*>(a.out[inst_]) + (size_t)(line0 + b) * nt, twm);
  }
  PAT_END_ITEM
}

// k_line_nufft1 for m = 2^LM and nz = 2^LZ known at compile time (FP32,
// one instance): the same work, with both FFTs' stages fixed by P2Plan; the
// last stage of the grid FFT writes the picked, deconvolved samples straight
// to memory.  Five waves per SIMD (the register cap of 96 costs a 20-byte
// spill): the spreading is bound by instruction issue and gains more from
// the fifth wave than the spill takes.
template <typename T, int TAPS, int LM, int LZ>
__global__ __launch_bounds__(kBlock, 5) void k_line_nufft1_c(StageArgs a) {
  constexpr int m = 1 << LM, nz = 1 << LZ;
  using PM = P2Plan<LM>;  // (no radix-16 last stage: it spills at this kernel's register
  using PZ = P2Plan<LZ>;  // cap in the grid FFT and gained nothing in the depth FFT)
  static_assert(PM::nst >= 2 && PZ::nst >= 2, "two or more stages");
  PAT_FOR_EACH_ITEM(a)
  const int nt = I.nt;
  const int lpw = I.lpw_a;
  const int line0 = li * lpw;
  const int nl = min(lpw, I.lines - line0);
  const cx<T>* twm = static_cast<const cx<T>*>(I.tw) + I.fm.tw;
  const cx<T>* twz = static_cast<const cx<T>*>(I.tw) + I.fz.tw;
  const int sg = m > lpw * nz ? m : lpw * nz;
  cx<T>* grid = reinterpret_cast<cx<T>*>(pat_smem);  // depth-FFT scratch, then one grid line
  cx<T>* qn = grid + sg;                              // lpw depth spectra, natural order
  const SpreadLds<T, 2> L = SpreadLds<T, 2>::carve(qn + lpw * nz, nz, I.taps);
  const cx<T>* in = static_cast<const cx<T>*>(a.in[inst_]) + (size_t)line0 * nz;
  constexpr int stepz = nz / PZ::rad(PZ::nst - 1);
  fft_first_stage_p2<T, PZ::rad(0), true>(grid, nz, twz, nl, nz, 1,
                                          [&](int b, int pos) { return in[(size_t)b * nz + pos]; });
  __syncthreads();
  p2_stages<T, LZ, 1>(grid, twz, nl);
  fft_last_stage_p2<T, PZ::rad(PZ::nst - 1), true>(grid, nz, nl, nz, 1, [&](int b, int blk, const auto& v) {
    constexpr int R = sizeof(v) / sizeof(v[0]);
    cx<T>* d = qn + b * nz;
    const int k0 = PZ::natural(blk * R);
#pragma unroll
    for (int r = 0; r < R; ++r) d[k0 + r * stepz] = v[r];
  });
  __syncthreads();
  auto put = [&](int j, cx<T> v) { grid[j] = cconj(v); };
  auto put4 = [&](int j, const cx<T>* v) {
#pragma unroll
    for (int c = 0; c < 2; ++c) grid[j + c] = cconj(v[c]);
  };
  const T* sn = static_cast<const T*>(I.sn);
  constexpr int step = m / PM::rad(PM::nst - 1);
  for (int b = 0; b < nl; ++b) {
    const cx<T>* qb = qn + b * nz;
    auto fget = [&](int l) { return qb[l]; };
    if (TAPS > 0 && a.pair_ok) {
      spread_line<T, (TAPS > 0 ? TAPS : 2), true>(I, a, line0 + b, a.mode, L, fget, put, put4);
    } else {
      spread_line<T, 0, false>(I, a, line0 + b, a.mode, L, fget, put, put4);
    }
    __syncthreads();
    // X_n = s_n conj(G_k) for the natural index k = (n - nt/2) mod m
    cx<T>* x = static_cast<cx<T>*>(a.out[inst_]) + (size_t)(line0 + b) * nt;
    p2_stages<T, LM, 0>(grid, twm, 1);
    fft_last_stage_p2<T, PM::rad(PM::nst - 1), true>(grid, m, 1, m, 1, [&](int, int blk, const auto& v) {
      constexpr int R = sizeof(v) / sizeof(v[0]);
      const int k0 = PM::natural(blk * R);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int n = (k0 + r * step + nt / 2) & (m - 1);
        if (n < nt) x[n] = cscl(cconj(v[r]), sn[n]);
      }
    });
  }
  PAT_END_ITEM
}

// The fused type-1 kernel with wavefront spreading (FP32 at four waves per
// SIMD, FP64 at two; m = 2^LM and nz = 2^LZ at compile time): a work item
// holds one line per wavefront.  The depth DFTs of its lines run together,
// then each wavefront spreads its line into its own grid line in LDS (no
// block barrier inside), and the grid DFTs of all lines run together; the
// last stage writes the picked, deconvolved samples to memory.  LDS: the
// lines' grids (also the depth-FFT scratch) and their depth spectra in
// natural order.
template <typename T, int TAPS, int LM, int LZ>
__global__ __launch_bounds__(kBlock, sizeof(T) == 4 ? 4 : 2) void k_line_nufft1_w(StageArgs a) {
  constexpr int m = 1 << LM, nz = 1 << LZ, NL = kBlock / 64;
  using PM = P2Plan<LM, p2_l16_m(LM)>;  // (radix-16 last stages, as in the type-2 kernel)
  using PZ = P2Plan<LZ, p2_l16_z(LZ)>;
  static_assert(PM::nst >= 2 && PZ::nst >= 2 && LZ <= LM, "two or more stages");
  cx<T>* grid = reinterpret_cast<cx<T>*>(pat_smem);  // NL grid lines (first the depth-FFT scratch)
  cx<T>* qn = grid + NL * m;                         // NL depth spectra, natural order
  PAT_FOR_EACH_ITEM(a)
  const int nt = I.nt;
  const int line0 = li * NL;
  const int nl = min(NL, I.lines - line0);
  const cx<T>* twm = static_cast<const cx<T>*>(I.tw) + I.fm.tw;
  const cx<T>* twz = static_cast<const cx<T>*>(I.tw) + I.fz.tw;
  const cx<T>* in = static_cast<const cx<T>*>(a.in[inst_]) + (size_t)line0 * nz;
  constexpr int stepz = nz / PZ::rad(PZ::nst - 1);
  fft_first_stage_p2<T, PZ::rad(0), true>(grid, nz, twz, nl, nz, 1,
                                          [&](int b, int pos) { return in[(size_t)b * nz + pos]; });
  __syncthreads();
  p2_stages<T, LZ, 1, p2_l16_z(LZ)>(grid, twz, nl);
  fft_last_stage_p2<T, PZ::rad(PZ::nst - 1), true>(grid, nz, nl, nz, 1, [&](int b, int blk, const auto& v) {
    constexpr int R = sizeof(v) / sizeof(v[0]);
    cx<T>* d = qn + b * nz;
    const int k0 = PZ::natural(blk * R);
#pragma unroll
    for (int r = 0; r < R; ++r) d[k0 + r * stepz] = v[r];
  });
  __syncthreads();
  const int wv = (int)(threadIdx.x >> 6);
  if (wv < nl) {
    const cx<T>* qb = qn + wv * nz;
    spread_line_wave<T, TAPS, true>(I, a, line0 + wv, a.mode, m, nz, grid + wv * m, [&](int l) { return qb[l]; });
  }
  __syncthreads();
  // X_n = s_n conj(G_k) for the natural index k = (n - nt/2) mod m
  const T* sn = static_cast<const T*>(I.sn);
  constexpr int step = m / PM::rad(PM::nst - 1);
  cx<T>* xout = static_cast<cx<T>*>(a.out[inst_]) + (size_t)line0 * nt;
  p2_stages<T, LM, 0, p2_l16_m(LM)>(grid, twm, nl);
  fft_last_stage_p2<T, PM::rad(PM::nst - 1), true>(grid, m, nl, m, 1, [&](int b, int blk, const auto& v) {
    constexpr int R = sizeof(v) / sizeof(v[0]);
    const int k0 = PM::natural(blk * R);
    cx<T>* x = xout + (size_t)b * nt;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int n = (k0 + r * step + nt / 2) & (m - 1);
      if (n < nt) x[n] = cscl(cconj(v[r]), sn[n]);
    }
  });
  PAT_END_ITEM
}

// Spreading alone with wavefront spreading (FP32 compute; grid stored as
// float or bf16 pairs): one line per wavefront, built in LDS and written out
// by the same wavefront with 16-byte stores.
template <typename G, int TAPS, bool P2>
__global__ __launch_bounds__(kBlock) void k_line_spread_w(StageArgs a) {
  constexpr int NL = kBlock / 64;
  PAT_FOR_EACH_ITEM(a)
  const int m = I.m, nz = I.nz;
  const int line0 = li * NL;
  const int wv = (int)(threadIdx.x >> 6), L = (int)(threadIdx.x & 63);
  if (line0 + wv < I.lines) {
    const int line = line0 + wv;
    cx<float>* Gl = reinterpret_cast<cx<float>*>(pat_smem) + wv * m;
    const cx<float>* F = static_cast<const cx<float>*>(a.in[inst_]) + (size_t)line * nz;
    spread_line_wave<float, TAPS, P2>(I, a, line, a.mode, m, nz, Gl, [&](int l) { return F[l]; });
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    G* row = static_cast<G*>(a.out[inst_]) + (size_t)line * m;
    for (int j = 4 * L; j < m; j += 4 * 64) {
      cx<float> v4[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) v4[c] = cconj(Gl[j + c]);
      grid_store4<float, G>(row + j, v4);
    }
  }
  PAT_END_ITEM
}

__global__ void k_zero_u32(uint32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Host launchers

int num_cu() {
  static const int n = [] {
    int v = 0, dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
      v = 256;
    return v;
  }();
  return n;
}

// Workgroups of `block` threads that one CU holds at once for this kernel and
// LDS size; 0 and *err on a HIP error.  The first query of a device raises the
// kernel's dynamic LDS limit where it needs more than 64 KB; both answers are
// kept (neither call is free on a path that launches in microseconds).
int resident_blocks(const void* kernel, size_t shmem, int block, hipError_t* err) {
  static std::mutex mu;
  static std::map<std::tuple<const void*, size_t, int, int>, int> cache;
  int dev = 0;
  *err = hipGetDevice(&dev);
  if (*err != hipSuccess) return 0;
  std::lock_guard<std::mutex> lock(mu);
  auto it = cache.find({kernel, shmem, block, dev});
  if (it != cache.end()) return it->second;
  if (shmem > 65536) {
    // (the limit only ever rises: another size of the same kernel may be larger)
    static std::map<std::pair<const void*, int>, size_t> limit;
    size_t& lim = limit[{kernel, dev}];
    if (shmem > lim) {
      *err = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
      if (*err != hipSuccess) return 0;
      lim = shmem;
    }
  }
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, shmem) != hipSuccess || per_cu < 1)
    per_cu = 1;
  cache[{kernel, shmem, block, dev}] = per_cu;
  return per_cu;
}

// launches left before an injected failure (0: none); see set_launch_fault
static thread_local int t_fault_countdown = 0;

// True when this launch is the one the PAT_FAULT hook fails.
bool launch_faulted() { return t_fault_countdown > 0 && --t_fault_countdown == 0; }

namespace {

enum Items { IT_X1, IT_X2, IT_C2R, IT_LM, IT_LZ, IT_LI, IT_LF, IT_LA, IT_LINE, IT_LWAVE };

int cdiv(int a, int b) { return (a + b - 1) / b; }

int items_of(const Inst& I, Items kind, bool nz) {
  const int len = nz ? I.nz : I.nt;
  switch (kind) {
    case IT_X1: return I.n2 * cdiv(len, 2 * I.tb);
    case IT_X2: return I.n2 > 1 ? I.h1 * cdiv(len, I.tb) : 0;
    case IT_C2R: return I.n2 * cdiv(len, 2 * I.tb);
    case IT_LM: return cdiv(I.lines, I.lpw_m);
    case IT_LZ: return cdiv(I.lines, I.lpw_z);
    case IT_LI: return cdiv(I.lines, I.lpw_i);
    case IT_LF: return cdiv(I.lines, I.lpw_f);
    case IT_LA: return cdiv(I.lines, I.lpw_a);
    case IT_LINE: return I.lines;
    case IT_LWAVE: return cdiv(I.lines, kBlock / 64);  // one line per wavefront
  }
  return 0;
}

template <typename T, typename G, int RS, int TAPS>
struct Runner {
  static constexpr bool P2 = RS == 0;
  int n;
  const Inst* h;
  const Inst* const* d;
  const void* const* hp;  // host tap-polynomial tables
  uint32_t* counters;
  int next_counter;
  hipStream_t st;
  StageTimer* tm;

  static constexpr size_t cs = sizeof(cx<T>);

  StageArgs base(Items kind, bool nz, int mode, const void* const* in, void* const* out) {
    StageArgs a;
    a.n = n;
    a.len_nz = nz ? 1 : 0;
    a.np_cap = a.tb_cap = 0;
    a.mode = mode;
    a.off[0] = 0;
    for (int i = 0; i < n; ++i) {
      a.inst[i] = d[i];
      a.in[i] = in[i];
      a.out[i] = out[i];
      a.off[i + 1] = a.off[i] + items_of(h[i], kind, nz);
    }
    a.total = a.off[n];
    a.counter = counters ? counters + (next_counter++ % kNumCounters) : nullptr;
    fill_pairs(a);
    return a;
  }

  // Mirrored tap-pair coefficients into the arguments when every instance
  // uses the same fitted table with TAPS (even) taps.
  void fill_pairs(StageArgs& a) const {
    a.pair_ok = 0;
    constexpr int D = Deg<T>::v, D1 = D + 1, NE = D / 2 + 1, NO = (D + 1) / 2, PW = NE + NO;
    if (TAPS <= 0 || TAPS % 2 != 0 || (size_t)(TAPS / 2) * PW * sizeof(T) > sizeof(a.pc) || !hp) return;
    for (int i = 0; i < n; ++i) {
      if (!h[i].poly || h[i].taps != TAPS || !hp[i]) return;
      if (std::memcmp(hp[i], hp[0], (size_t)TAPS * D1 * sizeof(T)) != 0) return;
    }
    const T* mono = static_cast<const T*>(hp[0]);
    T pc[(TAPS > 0 ? TAPS / 2 : 1) * PW];
    for (int p = 0; p < TAPS / 2; ++p) {
      for (int e = 0; e < NE; ++e) pc[p * PW + e] = mono[p * D1 + 2 * e];
      for (int o = 0; o < NO; ++o) pc[p * PW + NE + o] = mono[p * D1 + 2 * o + 1];
    }
    std::memcpy(a.pc, pc, sizeof(pc));
    a.pair_ok = 1;
  }

  // Whether every instance's transverse passes can run the general-length
  // kernels, and every instance's fused line stage.
  bool gtr_ok() const {
    for (int i = 0; i < n; ++i)
      if (!h[i].gtr) return false;
    return true;
  }
  bool gln_ok() const {
    for (int i = 0; i < n; ++i)
      if (!h[i].gln) return false;
    return true;
  }
  // The passes before the grid keep their arithmetic with the bf16 grid: a
  // change of their FP32 rounding (1e-7) moves grid values across bf16 rounding
  // boundaries and the output by up to 4e-5 of itself.
  static constexpr bool kBeforeGrid = std::is_same_v<G, bf2>;

  // Transverse passes of one instance of powers of two below the Fixed kernels'
  // threshold that run this file's kernels and not the general-length ones: a
  // launch of a few workgroups takes the latency of one, and there run-time sizes
  // cost more than narrower tiles give back.  `pts`: columns of the pass; `pipe`:
  // the compile-time pipeline applies to it.  Kernel times, these against the
  // general-length kernels':
  //   FP32, 128 points, x1 and c2r: 4.2 to 5.4 against 4.9 to 6.6 us up to 4096
  //     columns, 7.9 against 6.4 at 8192 (x2, and 256 and 512 points: slower at
  //     every size)
  //   FP64, 128, 256 and 512 points: 3.9 to 8.8 against 5.8 to 12.2 us up to the
  //     Fixed kernels' threshold (x2 at 512: even; c2r with a cut-off, which the
  //     pipeline does not take, gains at 128 only)
  //   FP64, 64 points and less: 3.9 to 6.4 against 4.0 to 7.1 us up to 4096 columns
  //     (x2: 1024), slower from there on
  enum Pass { PASS_X1, PASS_X2, PASS_C2R };
  bool short_pass(Pass ps, int L, int64_t pts, bool pipe) const {
    if (RS != 0 || n != 1 || counters) return false;
    if (sizeof(T) == 4) return L == 128 && ps != PASS_X2 && pipe && pts <= 16 * num_cu();
    if (L >= 128) return (pipe || (L == 128 && ps == PASS_C2R)) && L <= 512 && !(ps == PASS_X2 && L == 512);
    return pts <= (ps == PASS_X2 ? 4 : 16) * num_cu();
  }
  // whether the plan's tile is the one of the compile-time pipeline of L points
  bool pipe_length(int L) const {
    const int ll = L == 128 ? 7 : L == 256 ? 8 : L == 512 ? 9 : 0;
    return RS == 0 && ll && h[0].tb == pipe_tb<T>(ll);
  }

  template <typename F>
  size_t max_over(F f) const {
    size_t mx = 0;
    for (int i = 0; i < n; ++i) {
      const size_t v = f(h[i]);
      if (v > mx) mx = v;
    }
    return mx;
  }

  // The pipelined transverse kernels run for one instance where neither the Fixed
  // nor the general-length kernels do: before a bf16 grid, in small launches
  // (short_pass), for lengths without a general plan (578) and for arrays of 4 GiB
  // and more.  Lengths of 128, 256 and 512 points with the plan's tile width take
  // the compile-time instances (FP64 only these: its run-time-size pipelines,
  // sized for the largest tile, would spill), other FP32 lengths the run-time-size
  // ones.
  hipError_t x1(const void* const* in, void* const* out, bool nz) {
    StageArgs a = base(IT_X1, nz, 0, in, out);
    const int len = nz ? h[0].nz : h[0].nt;
    const bool pipe = n == 1 && !a.counter && len % 4 == 0 && h[0].tb % 2 == 0 && h[0].n1 * (h[0].tb / 2) <= kPipeU * kBlock;
    if (!kBeforeGrid && n == 1 && h[0].gtr && Fixed<T>::takes(h[0].n1, h[0].n2, len)) return Fixed<T>::x1(a, h[0], st, tm);
    if (!kBeforeGrid && gtr_ok() && !short_pass(PASS_X1, h[0].n1, (int64_t)h[0].n2 * len, pipe && pipe_length(h[0].n1)))
      return General<T>::x1(a, h, st, tm);
    {
      if (pipe) {
        const size_t ew = (size_t)(h[0].cut_e + 1) * (h[0].cut_e + 1);
        const size_t shm = (size_t)h[0].n1 * (h[0].tb + 1) * cs + (size_t)((h[0].n1 + 3) & ~3) * sizeof(int32_t) +
                           (!nz && h[0].cut_e ? 2 * ew * sizeof(T) : 0);
        auto go = [&](auto kern) { return launch_persistent(kern, "dft_x1", a, shm, st, tm); };
        if constexpr (RS == 0) {
          const int L = h[0].n1, tb = h[0].tb;
          if (L == 128 && tb == pipe_tb<T>(7)) return go(k_tr_x1_pipe<T, RS, 7>);
          if (L == 256 && tb == pipe_tb<T>(8)) return go(k_tr_x1_pipe<T, RS, 8>);
          if (L == 512 && tb == pipe_tb<T>(9)) return go(k_tr_x1_pipe<T, RS, 9>);
        }
        if constexpr (sizeof(T) == 4) return go(k_tr_x1_pipe<T, RS>);
      }
    }
    return launch(k_tr_x1_r2c<T, RS>, "dft_x1", a, max_over([](const Inst& I) { return lds_tile_x1(I, cs); }), st,
                  tm);
  }
  hipError_t x2(void* const* io, bool nz, int inv) {
    StageArgs a = base(IT_X2, nz, inv, io, io);
    const char* name = inv ? "idft_x2" : "dft_x2";
    const bool before_grid = kBeforeGrid && !inv;
    if (!before_grid && n == 1 && h[0].gtr && h[0].n2 > 1 && Fixed<T>::takes(h[0].n2, 2 * h[0].h1, nz ? h[0].nz : h[0].nt))
      return Fixed<T>::x2(a, h[0], st, tm);
    const bool pipe = n == 1 && !a.counter && h[0].tb % 2 == 0 && h[0].n2 * (h[0].tb / 2) <= kPipeU * kBlock;
    if (!before_grid && gtr_ok() &&
        !short_pass(PASS_X2, h[0].n2, (int64_t)h[0].h1 * (nz ? h[0].nz : h[0].nt), pipe && pipe_length(h[0].n2)))
      return General<T>::x2(a, h, st, tm);
    {
      if (pipe) {
        const size_t shm = lds_tile_x2(h[0], cs) + (size_t)((h[0].n2 + 3) & ~3) * sizeof(int32_t);
        auto go = [&](auto kern) { return launch_persistent(kern, name, a, shm, st, tm); };
        if constexpr (RS == 0) {
          const int L = h[0].n2, tb = h[0].tb;
          if (L == 128 && tb == pipe_tb<T>(7)) return go(k_tr_x2_pipe<T, RS, 7>);
          if (L == 256 && tb == pipe_tb<T>(8)) return go(k_tr_x2_pipe<T, RS, 8>);
          if (L == 512 && tb == pipe_tb<T>(9)) return go(k_tr_x2_pipe<T, RS, 9>);
        }
        if constexpr (sizeof(T) == 4) return go(k_tr_x2_pipe<T, RS>);
      }
    }
    return launch(k_tr_x2<T, RS>, name, a, max_over([](const Inst& I) { return lds_tile_x2(I, cs); }), st, tm);
  }
  hipError_t c2r(const void* const* in, void* const* out, bool nz) {
    StageArgs a = base(IT_C2R, nz, 0, in, out);
    const int len = nz ? h[0].nz : h[0].nt;
    if (n == 1 && h[0].gtr && Fixed<T>::takes(h[0].n1, h[0].n2, len)) return Fixed<T>::c2r(a, h[0], st, tm);
    const bool pipe = n == 1 && !a.counter && !(!nz && h[0].cut_e) && len % 4 == 0 && h[0].tb % 2 == 0 &&
                      h[0].n1 * h[0].tb <= 2 * kPipeU * kBlock;
    if (gtr_ok() && !short_pass(PASS_C2R, h[0].n1, (int64_t)h[0].n2 * len, pipe && pipe_length(h[0].n1)))
      return General<T>::c2r(a, h, st, tm);
    {
      if (pipe) {
        const size_t shm = (size_t)h[0].n1 * (h[0].tb + 1) * cs + (size_t)((h[0].n1 + 3) & ~3) * sizeof(int32_t);
        auto go = [&](auto kern) { return launch_persistent(kern, "idft_x1_c2r", a, shm, st, tm); };
        if constexpr (RS == 0) {
          const int L = h[0].n1, tb = h[0].tb;
          if (L == 128 && tb == pipe_tb<T>(7)) return go(k_tr_c2r_pipe<T, RS, 7>);
          // (FP32 arrays of 256 points and this tile end below 4 GiB: the general kernels' range)
          if constexpr (sizeof(T) == 8) {
            if (L == 256 && tb == pipe_tb<T>(8)) return go(k_tr_c2r_pipe<T, RS, 8>);
          }
          if (L == 512 && tb == pipe_tb<T>(9)) return go(k_tr_c2r_pipe<T, RS, 9>);
        }
        if constexpr (sizeof(T) == 4) return go(k_tr_c2r_pipe<T, RS>);
      }
    }
    return launch(k_tr_c2r_k1<T, RS>, "idft_x1_c2r", a, max_over([](const Inst& I) { return lds_tile_x1(I, cs); }),
                  st, tm);
  }
  hipError_t zfft(void* const* io, int inv) {
    StageArgs a = base(IT_LZ, true, inv, io, io);
    return launch(k_line_fft<T, RS>, inv ? "idft_z" : "dft_z", a,
                  max_over([](const Inst& I) { return lds_line_z(I, cs); }), st, tm);
  }
  hipError_t a2(const void* const* in, void* const* out) {
    StageArgs a = base(IT_LM, false, 0, in, out);
    if constexpr (sizeof(T) == 4 && P2) {
      // one instance, centred c = 2 grid, m = 2^8 .. 2^11: the pipelined kernel
      const Inst& I = h[0];
      const int lm = __builtin_ctz((unsigned)I.m);
      if (n == 1 && !a.counter && I.centred && I.m == 2 * I.nt && lm >= 8 && lm <= 11 && I.fm.rad[0] == 8 &&
          I.lpw_m == 2048 / I.m) {
        const size_t shm = (size_t)(2048 + 2048 + 2048 / 16) * cs;
        auto go = [&](auto kern) { return launch_persistent(kern, "deconv_pad_fft", a, shm, st, tm); };
        if (lm == 8) return go(k_line_a2_pipe<G, 8>);
        if (lm == 9) return go(k_line_a2_pipe<G, 9>);
        if (lm == 10) return go(k_line_a2_pipe<G, 10>);
        return go(k_line_a2_pipe<G, 11>);
      }
    }
    return launch(k_line_a2<T, G, RS>, "deconv_pad_fft", a, max_over([](const Inst& I) { return lds_line_m(I, cs); }),
                  st, tm);
  }
  hipError_t a2t(const void* const* in, void* const* out) {
    StageArgs a = base(IT_LM, false, 0, in, out);
    if constexpr (sizeof(T) == 4 && P2) {
      // one instance, centred c = 2 grid, m = 2^8 .. 2^11: the pipelined kernel
      const Inst& I = h[0];
      const int lm = __builtin_ctz((unsigned)I.m);
      if (n == 1 && !a.counter && I.centred && I.m == 2 * I.nt && lm >= 8 && lm <= 11 && I.lpw_m == 2048 / I.m) {
        const size_t shm = (size_t)(2048 + 2048 / 16) * cs;
        auto go = [&](auto kern) { return launch_persistent(kern, "ifft_pick_deconv", a, shm, st, tm); };
        if (lm == 8) return go(k_line_a2t_pipe<G, 8>);
        if (lm == 9) return go(k_line_a2t_pipe<G, 9>);
        if (lm == 10) return go(k_line_a2t_pipe<G, 10>);
        return go(k_line_a2t_pipe<G, 11>);
      }
    }
    return launch(k_line_a2t<T, G, RS>, "ifft_pick_deconv", a,
                  max_over([](const Inst& I) { return lds_line_m(I, cs); }), st, tm);
  }
  hipError_t interp(const void* const* in, void* const* out, int mode) {
    StageArgs a = base(IT_LI, true, mode, in, out);
    if constexpr (TAPS > 0) {
      // one instance with the paired taps: the streamed kernel, with enough
      // 16-byte registers per thread for a line group
      constexpr int EPC = GridChunk<T, G>::EPC;
      const Inst& I = h[0];
      const int per = (I.lpw_i * I.m / EPC + kBlock - 1) / kBlock;
      if (n == 1 && a.pair_ok && I.m % EPC == 0 && per <= 8 && !counters) {
        const size_t shm = lds_interp_stream(I, cs);
        if (per <= 1) return launch_persistent(k_line_interp_stream<T, G, TAPS, P2, 1>, "interp", a, shm, st, tm);
        if (per <= 2) return launch_persistent(k_line_interp_stream<T, G, TAPS, P2, 2>, "interp", a, shm, st, tm);
        if (per <= 4) return launch_persistent(k_line_interp_stream<T, G, TAPS, P2, 4>, "interp", a, shm, st, tm);
        return launch_persistent(k_line_interp_stream<T, G, TAPS, P2, 8>, "interp", a, shm, st, tm);
      }
    }
    return launch(k_line_interp<T, G, TAPS, P2>, "interp", a,
                  max_over([](const Inst& I) { return lds_interp(I, cs); }), st, tm);
  }
  hipError_t spread(const void* const* in, void* const* out, int mode) {
    if constexpr (sizeof(T) == 8 && TAPS == 12) {
      // one 3D instance with pairs enough: its lines in mirror pairs (256^3: 319 us
      // against 377, 128^3: 48 against 83; see spreads)
      if (n == 1 && PairLine<T>::spreads(h[0])) {
        StageArgs a = base(IT_LINE, true, mode, in, out);
        if (a.pair_ok) return PairLine<T>::spread(a, h[0], st, tm);
        next_counter--;  // (the counter taken by base() above is not used)
      }
    }
    if constexpr (sizeof(T) == 4 && TAPS > 0 && TAPS % 2 == 0) {
      // FP32 with the paired taps: one line per wavefront (its grid line in
      // LDS, up to 2048 points)
      StageArgs a = base(IT_LWAVE, true, mode, in, out);
      const size_t shm = max_over([](const Inst& I) { return lds_spread_wave(I); });
      bool ok = a.pair_ok && shm <= 65536;
      for (int i = 0; i < n; ++i) ok = ok && h[i].m % 4 == 0;
      if (ok) return launch(k_line_spread_w<G, TAPS, P2>, "spread", a, shm, st, tm);
      next_counter--;  // (the counter taken by base() above is not used)
    }
    StageArgs a = base(IT_LINE, true, mode, in, out);
    return launch(k_line_spread<T, G, TAPS>, "spread", a,
                  max_over([](const Inst& I) { return lds_spread(I, cs); }), st, tm);
  }
  // R on 3D plans with nz = m/4, m = 2^8 .. 2^11: line groups in mirror pairs
  bool mirrors(const StageArgs& a, int mode) const {
    const Inst& I = h[0];
    return n == 1 && !a.counter && a.pair_ok && mode == 0 && I.m == 2 * I.nt && 4 * I.nz == I.m && I.n2 >= 4 &&
           I.fm.nst >= 2 && I.fm.rad[0] == 8 && I.m >= 256 && I.m <= 2048;
  }
  hipError_t mirror(StageArgs& a) {
    if constexpr (P2 && TAPS > 0) {
      constexpr bool BF = sizeof(G) < sizeof(cx<T>);
      const Inst& I = h[0];
      // two waves per workgroup up to m = 1024 (one mirror pair there), four at
      // m = 2048
      const int nt_ = I.m <= 1024 ? 128 : 256;
      a.total = cdiv(I.lines, 16 * nt_ / I.m);
      a.off[1] = a.total;
      auto go = [&](auto kern, int shm) { return launch_persistent(kern, BF ? "interp_idft_z" : "nufft_fused", a, shm, st, tm, nt_); };
      if (I.m == 256) return go(k_line_nufft2_mirror<T, TAPS, 8, 6, 128, BF>, MirrorLds<T, 8, 128>::bytes);
      if (I.m == 512) return go(k_line_nufft2_mirror<T, TAPS, 9, 7, 128, BF>, MirrorLds<T, 9, 128>::bytes);
      if (I.m == 1024) return go(k_line_nufft2_mirror<T, TAPS, 10, 8, 128, BF>, MirrorLds<T, 10, 128>::bytes);
      return go(k_line_nufft2_mirror<T, TAPS, 11, 9, 256, BF>, MirrorLds<T, 11, 256>::bytes);
    }
    return hipErrorInvalidValue;
  }
  // R's interpolation and depth FFT from a stored bf16 grid in one kernel, where
  // the mirror kernel applies (256^3: 58 us against 55 + 43, 128^3: 16 against 27,
  // 512^3: 393 against 339 + 383).
  bool bf_mirror(const void* const* in, void* const* out, int mode, hipError_t* e) {
    if constexpr (P2 && TAPS > 0 && sizeof(G) < sizeof(cx<T>)) {
      StageArgs a = base(IT_LF, true, mode, in, out);
      if (mirrors(a, mode)) {
        *e = mirror(a);
        return true;
      }
      next_counter--;  // (the counter taken by base() above is not used)
    }
    return false;
  }
  // Type-2 line stages of one instance of powers of two that k_gline2 could take and
  // that run k_line_nufft2(_pipe): the lengths without a compile-time kernel, as long
  // as the lines do not fill the chip.  A k_gline2 workgroup carries more pairs and
  // pays for run-time radices; in 2D half of its pair points are empty.  Kernel
  // times, these against k_gline2's:
  //   FP32, 3D: m = 32, 8256 lines 8.3 against 11.8 us, 33024 lines 16.3 against 12.4;
  //     m = 128, 8256 lines 12.6 against 13.2, 16512 lines 18.1 against 15.7; m = 512,
  //     nz = 64, 2080 lines 12.5 against 12.8, 4128 lines 16.6 against 13.6; m = 2048,
  //     nz = 256, 640 lines 14.3 against 15.1, 1032 lines 18.9 against 14.9
  //   FP32, 2D: 33 to 2049 lines 7.3 to 10.9 against 8.9 to 11.7; m = 1024, nz = 128,
  //     1025 lines 12.9 against 11.8; m = 2048, 2049 lines 29 against 34
  //   (m = 128 with nz = 64 only: 11.9 against 10.8)
  //   FP64, 3D: m = 64, 4352 lines 14.2 against 15.6, 8256 lines 20.2 against 17.0;
  //     m = 512, nz = 64, 1040 lines 15.9 against 17.3, 2080 lines 25.2 against 19.4;
  //     m = 2048, nz = 256, 1280 lines 43.5 against 48.9, 2080 lines 67
  //   FP64, 2D: m up to 64, 11 to 13 against 13 to 15; m = 128 even, from 1500 lines on
  //     14.9 against 16.2; m = 2048, 257 lines 17.6 against 27.8
  // FP64 lines whose general grid is not the plan's (m below 64) stay on it: R^T and A
  // are transposes of R and A^T to 1e-12 only where both take the same window.
  bool short_type2() const {
    const Inst& I = h[0];
    if (RS != 0 || n != 1 || counters || (I.m == 128 && I.nz == 64)) return false;
    if (sizeof(T) == 8 && I.gln && I.gm.L != I.m) return false;
    const int64_t pts = (int64_t)I.lines * I.m, cu = num_cu();
    if (sizeof(T) == 4) {
      if (I.n2 == 1) return I.m >= 2048 || pts <= 3600 * cu;
      return pts <= (I.m <= 64 ? 3072 : 4608) * cu;
    }
    if (I.n2 == 1) return I.m <= 64 || I.m >= 2048 || (I.m <= 256 && I.lines >= 6 * cu);
    if (I.m >= 2048) return pts <= 12288 * cu;
    return I.lines <= 20 * cu && pts <= 2200 * cu;
  }
  hipError_t nufft2(const void* const* in, void* const* out, int mode) {
    StageArgs a = base(IT_LF, true, mode, in, out);
    if constexpr (P2 && TAPS > 0) {
      if (mirrors(a, mode)) return mirror(a);
    }
    if constexpr (P2 && TAPS > 0) {
      // FP32, and FP64 at two waves per SIMD (its launch bound)
      const Inst& I = h[0];
      if (n == 1 && !a.counter && a.pair_ok && I.m == 2 * I.nt && I.m >= I.nz && I.fm.nst >= 2 &&
          I.fm.rad[0] == 8 && (I.m / 8) * I.lpw_f == kBlock) {
        // compile-time sizes for m = 2^8 .. 2^11 and nz = m/4 or m/2 (with
        // the padded scratch)
        const size_t shm = lds_fused2(I, cs) + (size_t)I.lpw_f * (I.m / 16) * cs;
        const int lm = __builtin_ctz((unsigned)I.m), dz = lm - __builtin_ctz((unsigned)I.nz);
        auto go = [&](auto kern) { return launch_persistent(kern, "nufft_fused", a, shm, st, tm); };
        if (dz == 2) {
          if (lm == 8) return go(k_line_nufft2_pipe_c<T, TAPS, 8, 6>);
          if (lm == 9) return go(k_line_nufft2_pipe_c<T, TAPS, 9, 7>);
          if (lm == 10) return go(k_line_nufft2_pipe_c<T, TAPS, 10, 8>);
          if (lm == 11) return go(k_line_nufft2_pipe_c<T, TAPS, 11, 9>);
        } else if (dz == 1) {
          if (lm == 8) return go(k_line_nufft2_pipe_c<T, TAPS, 8, 7>);
          if (lm == 9) return go(k_line_nufft2_pipe_c<T, TAPS, 9, 8>);
          if (lm == 10) return go(k_line_nufft2_pipe_c<T, TAPS, 10, 9>);
          if (lm == 11) return go(k_line_nufft2_pipe_c<T, TAPS, 11, 10>);
        }
        if constexpr (sizeof(T) == 4) {
          if (!gln_ok() || short_type2()) return go(k_line_nufft2_pipe<T, TAPS>);
        }
      }
    }
    if (gln_ok() && a.pair_ok && !short_type2()) return General<T>::line2(a, h, st, tm);
    return launch(k_line_nufft2<T, RS, TAPS>, "nufft_fused", a,
                  max_over([](const Inst& I) { return lds_fused2(I, cs); }), st, tm);
  }
  // Type-1 line stages of one instance that k_gline1 could take and that run
  // k_line_nufft1, one line per workgroup.  Alone on a CU its line takes 14 to 25 us in
  // FP32 and 16 to 30 in FP64, k_gline1's pair 16 to 45 and 21 to 58 (run-time radices,
  // the pair's batches in turn; in 2D half a pair is empty), but its gather is walked
  // once more for every time window that the nodes reach over, and more lines than
  // workgroups fit at once cost another such time.  So: its rounds over the resident
  // workgroups (`mine`) against k_gline1's (`theirs`) times the ratio r of the two times
  // of a round, and the nodes' reach in time windows against a limit.  The line and
  // both sides, k_line_nufft1's first:
  //   FP32, 3D, nt = 80: 984 lines 17 against 21 us, 1464 lines 29 against 26; nt = 300:
  //     504 lines 18 against 26, 1056 lines 30 against 26; nt = nz = 300: 20 against 34 at
  //     1008 lines; nt = 1000: 504 lines 28 against 36, 732 lines 49 against 40
  //   FP64, 3D, nt = 80: 732 lines 38 against 39; nt = 300: 252 lines 20 against 36, 528
  //     lines 35 against 35; nt = 1024 as powers of two: 144 lines 25 against 50, 2112
  //     lines 185 against 212, 2304 lines 181 against 171
  //   2D, nt = 300, n1 = 240 (reach 0.94) 17.9 against 19.1 in FP32, n1 = 300 (1.1) 24
  //     against 20; FP64 21.7 against 27.6 and, n1 = 600 (2.1), 36.7 against 33.7; nt = 1024,
  //     n1 = 512 in FP64: 48 against 65
  //   reach, 3D: nt = 20, FP32, n1 = 80 (5.7) 17.6 against 18.6, n1 = 120 (8.5) 21.8 against 18.6
  //   radices above 8 (nz = 184): 25 to 26 against 24 to 27 in FP32, 2D 31 against 20
  //   powers of two with several depth lines per workgroup (lpw_a): two against one 17 to
  //     20 against 18 to 20 (FP64 22 to 25 against 25 to 28), four and eight 25 to 70
  //     against 16 to 25
  bool short_type1() const {
    if constexpr (TAPS > 0) {
      const Inst& I = h[0];
      const bool flat = I.n2 == 1, wide = sizeof(T) == 8, two = I.lpw_a == 2;
      if (n != 1 || counters || (flat ? RS == 23 || I.lpw_a > 1 : I.lpw_a > 2)) return false;
      if (wide && I.gln && I.gm.L != I.m) return false;  // (see short_type2)
      hipError_t e = hipSuccess;
      const int res = resident_blocks(reinterpret_cast<const void*>(k_line_nufft1<T, RS, TAPS>), lds_fused1(I, cs), kBlock, &e);
      if (e != hipSuccess) return false;
      const double mine = std::ceil((double)cdiv(I.lines, I.lpw_a) / (res * num_cu()));
      double theirs = General<T>::line1_rounds(I);
      const bool full = theirs > 1.0;
      theirs = full ? std::fmin(theirs + 0.5, std::ceil(theirs)) : 1.0;
      const double n1h = 0.5 * I.n1, n2h = 0.5 * I.n2, nzh = 0.5 * I.nz;
      const double reach = std::sqrt(I.a1 * n1h * n1h + I.a2 * n2h * n2h + I.b * nzh * nzh) / I.nt;
      const bool deep = 2 * I.nz >= I.m;
      double r, most;
      if (flat) {
        r = 1.56;
        most = wide ? (full ? 5.0 : 2.0) : I.m <= 1024 || deep ? 1.1 : 0.8;
      } else {
        if (RS == 23) r = wide ? 1.15 : I.nz > 128 ? 0.95 : 1.3;
        else if (!wide) r = (deep ? 1.65 : 1.5) * (full ? 0.7 : 1.0);
        else if (two) r = 1.2;
        else if (RS == 0 && I.m == 2048 && 4 * I.nz == I.m) r = 1.95;
        else r = deep ? (full ? 1.9 : 2.0) : 1.6;
        r *= 1.0 + (full ? 1.3 : 0.4) / I.n2;
        most = !two ? 7.0 : !wide && I.lines >= 4 * num_cu() ? 1.6 : 0.7;
      }
      return (mine > 1.0 ? mine - 0.1 : 1.0) <= r * theirs && reach <= most;
    }
    return false;
  }
  hipError_t nufft1(const void* const* in, void* const* out, int mode) {
    if constexpr (P2 && TAPS > 0 && TAPS % 2 == 0) {
      // one line per wavefront, compile-time sizes for m = 2^8 .. 2^10 and
      // nz = m/4 or m/2
      const Inst& I = h[0];
      const int lm = __builtin_ctz((unsigned)I.m), dz = lm - __builtin_ctz((unsigned)I.nz);
      StageArgs a = base(IT_LWAVE, true, mode, in, out);
      // one 3D instance: its lines in mirror pairs (128^3: 31 us against 40)
      if (n == 1 && a.pair_ok && PairLine<T>::takes(I)) return PairLine<T>::line1(a, I, st, tm);
      if (n == 1 && a.pair_ok && (dz == 1 || dz == 2) && lm >= 8 && lm <= 10) {
        const size_t shm = lds_fused1_wave(I, cs);
        auto go = [&](auto kern) { return launch(kern, "nufft_adjoint_fused", a, shm, st, tm); };
        if (dz == 2) {
          if (lm == 8) return go(k_line_nufft1_w<T, TAPS, 8, 6>);
          if (lm == 9) return go(k_line_nufft1_w<T, TAPS, 9, 7>);
          return go(k_line_nufft1_w<T, TAPS, 10, 8>);
        }
        if (lm == 8) return go(k_line_nufft1_w<T, TAPS, 8, 7>);
        if (lm == 9) return go(k_line_nufft1_w<T, TAPS, 9, 8>);
        return go(k_line_nufft1_w<T, TAPS, 10, 9>);
      }
      next_counter--;
    }
    StageArgs a = base(IT_LA, true, mode, in, out);
    if constexpr (sizeof(T) == 4 && P2 && TAPS > 0) {
      // compile-time sizes for m = 2^8 .. 2^11 and nz = m/4 or m/2
      const Inst& I = h[0];
      const int lm = __builtin_ctz((unsigned)I.m), dz = lm - __builtin_ctz((unsigned)I.nz);
      const size_t shm = lds_fused1(I, cs);
      auto go = [&](auto kern) { return launch(kern, "nufft_adjoint_fused", a, shm, st, tm); };
      if (n == 1 && dz == 2) {
        if (lm == 8) return go(k_line_nufft1_c<T, TAPS, 8, 6>);
        if (lm == 9) return go(k_line_nufft1_c<T, TAPS, 9, 7>);
        if (lm == 10) return go(k_line_nufft1_c<T, TAPS, 10, 8>);
        if (lm == 11) return go(k_line_nufft1_c<T, TAPS, 11, 9>);
      } else if (n == 1 && dz == 1) {
        if (lm == 8) return go(k_line_nufft1_c<T, TAPS, 8, 7>);
        if (lm == 9) return go(k_line_nufft1_c<T, TAPS, 9, 8>);
        if (lm == 10) return go(k_line_nufft1_c<T, TAPS, 10, 9>);
        if (lm == 11) return go(k_line_nufft1_c<T, TAPS, 11, 10>);
      }
    }
    if (gln_ok() && a.pair_ok && !short_type1()) return General<T>::line1(a, h, st, tm);
    return launch(k_line_nufft1<T, RS, TAPS>, "nufft_adjoint_fused", a,
                  max_over([](const Inst& I) { return lds_fused1(I, cs); }), st, tm);
  }
};

#define PAT_TRY(x)                   \
  do {                               \
    hipError_t e_ = (x);             \
    if (e_ != hipSuccess) return e_; \
  } while (0)

template <typename T, typename G, int RS, int TAPS>
hipError_t run_op_t(Op op, int stage, int n, const Inst* h, const Inst* const* d, const void* const* hp,
                    const void* const* in, void* const* out, void* const* ws, uint32_t* counters, int counter0,
                    hipStream_t st, StageTimer* tm) {
  // stage s (1 .. 5) of the operator; the persistent launches of a stage
  // take work counters from counter0 on (stage 3 may launch three kernels)
  static const int kCounterAt[6] = {0, 0, 1, 2, 5, 6};
  Runner<T, G, RS, TAPS> r{n, h, d, hp, counters, counter0 + kCounterAt[stage], st, tm};
  void* bg[kMaxBatch];
  void* bu[kMaxBatch];
  void* bf[kMaxBatch];
  bool fused = true;
  for (int i = 0; i < n; ++i) {
    char* w = static_cast<char*>(ws[i]);
    bg[i] = w + h[i].off_g;
    bu[i] = w + h[i].off_u;
    bf[i] = w + h[i].off_f;
    fused = fused && h[i].fused;
  }
  const bool fwd = op == OP_R || op == OP_AT;  // type-2 line stage (else type-1)
  void* const* a = fwd ? bg : bf;               // the transverse spectrum of the input
  void* const* b = fwd ? bf : bg;               // the transverse spectrum of the output
  const int mode = (op == OP_R || op == OP_RT) ? 0 : 1;
  switch (stage) {
    case 1: return r.x1(in, a, !fwd);
    case 2: return r.x2(a, !fwd, 0);
    case 3:
      if (fwd) {
        if (fused) return r.nufft2(bg, bf, mode);
        PAT_TRY(r.a2(bg, bu));
        if (hipError_t e = hipSuccess; r.bf_mirror(bu, bf, mode, &e)) return e;
        PAT_TRY(r.interp(bu, bf, mode));
        return r.zfft(bf, 1);
      }
      if (fused) return r.nufft1(bf, bg, mode);
      PAT_TRY(r.zfft(bf, 0));
      PAT_TRY(r.spread(bf, bu, mode));
      return r.a2t(bu, bg);
    case 4: return r.x2(b, fwd, 1);
    case 5: return r.c2r(b, out, fwd);
  }
  return hipSuccess;
}

bool all_pow2(int n, const Inst* h) {
  for (int i = 0; i < n; ++i)
    if (!h[i].pow2) return false;
  return true;
}

// Largest radix over every FFT of the instances.
int max_radix(int n, const Inst* h) {
  int mx = 2;
  for (int i = 0; i < n; ++i) {
    for (const FftDesc* f : {&h[i].f1, &h[i].f2, &h[i].fm, &h[i].fz})
      for (int s = 0; s < f->nst; ++s) mx = f->rad[s] > mx ? f->rad[s] : mx;
  }
  return mx;
}

bool all_taps(int n, const Inst* h, int taps) {
  for (int i = 0; i < n; ++i)
    if (h[i].taps != taps) return false;
  return true;
}

// Stage `stage` of an operator over n instances with one kernel build (the
// radix set of their largest prime).
template <typename T, typename G>
hipError_t dispatch_one_build(Op op, int stage, int n, const Inst* h, const Inst* const* d, const void* const* hp,
                              const void* const* in, void* const* out, void* const* ws, uint32_t* counters,
                              int counter0, hipStream_t st, StageTimer* tm) {
  const bool t12 = all_taps(n, h, 12);
  if (all_pow2(n, h)) {
    if (t12) return run_op_t<T, G, 0, 12>(op, stage, n, h, d, hp, in, out, ws, counters, counter0, st, tm);
    return run_op_t<T, G, 0, 0>(op, stage, n, h, d, hp, in, out, ws, counters, counter0, st, tm);
  }
  if (max_radix(n, h) <= 8) {
    if (t12) return run_op_t<T, G, 7, 12>(op, stage, n, h, d, hp, in, out, ws, counters, counter0, st, tm);
    return run_op_t<T, G, 7, 0>(op, stage, n, h, d, hp, in, out, ws, counters, counter0, st, tm);
  }
  if (t12) return run_op_t<T, G, 23, 12>(op, stage, n, h, d, hp, in, out, ws, counters, counter0, st, tm);
  return run_op_t<T, G, 23, 0>(op, stage, n, h, d, hp, in, out, ws, counters, counter0, st, tm);
}

// The class of an instance in a batch: 0 powers of two, 1 every other length
// that the general-length kernels take in all stages, and, for the rest, the
// kernel build that their FFT lengths need: 2 radices up to 8, 3 larger primes.
constexpr int kClasses = 4;
int radix_class(const Inst& I) {
  if (I.pow2) return 0;
  if (I.gtr && I.gln && I.fused) return 1;
  return max_radix(1, &I) <= 8 ? 2 : 3;
}

// An operator over n instances.  Several instances are grouped by radix
// class, so that every instance runs the kernel build its own lengths need
// (one build over all would give every instance the registers of the largest
// prime's butterflies); each stage then runs one persistent launch per class
// present, all classes' stage s before any class's stage s + 1, so that only
// the last stage writes the outputs.  A class of one instance takes the
// single-instance kernels.  The work counters are cleared once, up front.
template <typename T, typename G>
hipError_t dispatch(Op op, int n, const Inst* h, const Inst* const* d, const void* const* hp, const void* const* in,
                    void* const* out, void* const* ws, uint32_t* counters, hipStream_t st, StageTimer* tm,
                    const ForkStreams* fork) {
  if (counters) {
    if (launch_faulted()) return hipErrorLaunchFailure;
    if (tm) tm->begin("zero_counters", st);
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, st, counters, kNumCounters);
    PAT_TRY(hipGetLastError());
    if (tm) tm->end(st);
  }
  if (n == 1) {
    for (int stage = 1; stage <= 5; ++stage) {
      const hipError_t e = dispatch_one_build<T, G>(op, stage, 1, h, d, hp, in, out, ws, counters, 0, st, tm);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  struct Group {
    int k = 0;
    Inst h[kMaxBatch];
    const Inst* d[kMaxBatch];
    const void* hp[kMaxBatch];
    const void* in[kMaxBatch];
    void* out[kMaxBatch];
    void* ws[kMaxBatch];
  };
  static thread_local Group g[kClasses];
  for (int c = 0; c < kClasses; ++c) g[c].k = 0;
  for (int i = 0; i < n; ++i) {
    Group& G_ = g[radix_class(h[i])];
    const int k = G_.k++;
    G_.h[k] = h[i];
    G_.d[k] = d[i];
    G_.hp[k] = hp[i];
    G_.in[k] = in[i];
    G_.out[k] = out[i];
    G_.ws[k] = ws[i];
  }
  // With the plan's fork streams (and no timer), each class after the first
  // runs on a stream of its own, forked from st after the counters are
  // cleared and joined back into st at the end, so that one class's launch
  // tails overlap another's work.  The host enqueues in the same order.
  int ncls = 0;
  for (int c = 0; c < kClasses; ++c) ncls += g[c].k > 0 ? 1 : 0;
  const bool forked = fork && !tm && ncls > 1;
  hipStream_t cs[kClasses] = {st, st, st, st};
  if (forked) {
    PAT_TRY(hipEventRecord(fork->ev[0], st));
    int j = 0;
    bool first = true;
    for (int c = 0; c < kClasses; ++c) {
      if (g[c].k == 0) continue;
      if (first) {
        first = false;
        continue;
      }
      cs[c] = fork->s[j++];
      PAT_TRY(hipStreamWaitEvent(cs[c], fork->ev[0], 0));
    }
  }
  hipError_t e = hipSuccess;
  for (int stage = 1; stage <= 5 && e == hipSuccess; ++stage) {
    for (int c = 0; c < kClasses && e == hipSuccess; ++c) {
      if (g[c].k == 0) continue;
      e = dispatch_one_build<T, G>(op, stage, g[c].k, g[c].h, g[c].d, g[c].hp, g[c].in, g[c].out, g[c].ws,
                                   g[c].k == 1 ? nullptr : counters, 8 * c, cs[c], tm);
    }
  }
  if (forked) {
    // (joined also after a failed launch: st then orders after everything
    // that was enqueued)
    int j = 1;
    for (int c = 0; c < kClasses; ++c) {
      if (cs[c] == st) continue;
      const hipError_t r = hipEventRecord(fork->ev[j], cs[c]);
      const hipError_t w = r == hipSuccess ? hipStreamWaitEvent(st, fork->ev[j], 0) : r;
      if (e == hipSuccess) e = w;
      ++j;
    }
  }
  return e;
}

template <typename T, typename G>
hipError_t interp_only(const Inst& h, const Inst* dinst, const void* hpoly, const void* grid, void* out,
                       hipStream_t st, StageTimer* tm) {
  const Inst* d[1] = {dinst};
  const void* hp[1] = {hpoly};
  const void* in[1] = {grid};
  void* o[1] = {out};
  if (h.taps == 12) {
    if (h.pow2) {
      Runner<T, G, 0, 12> r{1, &h, d, hp, nullptr, 0, st, tm};
      return r.interp(in, o, 0);
    }
    Runner<T, G, 23, 12> r{1, &h, d, hp, nullptr, 0, st, tm};
    return r.interp(in, o, 0);
  }
  Runner<T, G, 23, 0> r{1, &h, d, hp, nullptr, 0, st, tm};
  return r.interp(in, o, 0);
}

template <typename T, typename G>
hipError_t spread_only(const Inst& h, const Inst* dinst, const void* hpoly, const void* vals, void* grid,
                       hipStream_t st, StageTimer* tm) {
  const Inst* d[1] = {dinst};
  const void* hp[1] = {hpoly};
  const void* in[1] = {vals};
  void* o[1] = {grid};
  if (h.taps == 12) {
    if (h.pow2) {
      Runner<T, G, 0, 12> r{1, &h, d, hp, nullptr, 0, st, tm};
      return r.spread(in, o, 0);
    }
    Runner<T, G, 23, 12> r{1, &h, d, hp, nullptr, 0, st, tm};
    return r.spread(in, o, 0);
  }
  Runner<T, G, 23, 0> r{1, &h, d, hp, nullptr, 0, st, tm};
  return r.spread(in, o, 0);
}

}  // namespace

hipError_t run_op(int prec, Op op, int n, const Inst* hinst, const Inst* const* dinst, const void* const* hpoly,
                  const void* const* in, void* const* out, void* const* ws, uint32_t* counters, hipStream_t stream,
                  StageTimer* timer, const ForkStreams* fork) {
  switch (prec) {
    case PREC_F64:
      return dispatch<double, cx<double>>(op, n, hinst, dinst, hpoly, in, out, ws, counters, stream, timer, fork);
    case PREC_F32:
      return dispatch<float, cx<float>>(op, n, hinst, dinst, hpoly, in, out, ws, counters, stream, timer, fork);
    case PREC_BF16:
      return dispatch<float, bf2>(op, n, hinst, dinst, hpoly, in, out, ws, counters, stream, timer, fork);
  }
  return hipErrorInvalidValue;
}

hipError_t run_interp(int prec, const Inst& hinst, const Inst* dinst, const void* hpoly, const void* grid, void* out,
                      hipStream_t stream, StageTimer* timer) {
  switch (prec) {
    case PREC_F64: return interp_only<double, cx<double>>(hinst, dinst, hpoly, grid, out, stream, timer);
    case PREC_F32: return interp_only<float, cx<float>>(hinst, dinst, hpoly, grid, out, stream, timer);
    case PREC_BF16: return interp_only<float, bf2>(hinst, dinst, hpoly, grid, out, stream, timer);
  }
  return hipErrorInvalidValue;
}

// Workspace of the allocation-free entry point: one array per device, held
// until the process ends.  Host code never passes `scratch` itself (on the
// host it is only a stand-in for the symbol): kernels get the device address
// that hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

void set_launch_fault(int k) { t_fault_countdown = k > 0 ? k : 0; }

hipError_t scratch_buffer(void** ptr) {
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

hipError_t run_spread(int prec, const Inst& hinst, const Inst* dinst, const void* hpoly, const void* vals, void* grid,
                      hipStream_t stream, StageTimer* timer) {
  switch (prec) {
    case PREC_F64: return spread_only<double, cx<double>>(hinst, dinst, hpoly, vals, grid, stream, timer);
    case PREC_F32: return spread_only<float, cx<float>>(hinst, dinst, hpoly, vals, grid, stream, timer);
    case PREC_BF16: return spread_only<float, bf2>(hinst, dinst, hpoly, vals, grid, stream, timer);
  }
  return hipErrorInvalidValue;
}

}  // namespace pat
