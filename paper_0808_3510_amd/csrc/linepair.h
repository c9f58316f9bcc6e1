// Line pairs: two lines side by side at every point of LDS (one 16-byte access
// in float), so that they share index arithmetic and twiddles, and, for the
// mirror lines (k1, +-k2) of a 3D plan, node windows, phases and weights.
#pragma once

#include "regfft.h"

namespace pat {

template <typename T>
struct alignas(16) px {
  cx<T> a, b;
};

// lines and |K_x|^2 terms of pair P
struct PairLines {
  int la, lb;     // line indices (lb = -1: none)
  bool shared;    // the second line has the first one's nodes (or is absent)
  double ka, kb;  // nu+^2 = k. + b l^2
};
__device__ __forceinline__ PairLines pair_lines(CInst& I, int P) {
  PairLines q;
  if (I.n2 == 1) {
    q.la = P;
    q.lb = -1;
    q.shared = true;
    q.ka = q.kb = I.a1 * (double)P * (double)P;
    return q;
  }
  const int h2 = I.n2 >> 1;
  const int k1 = fdiv(P, I.m_h2), r = P - k1 * h2;
  q.la = k1 * I.n2 + r;
  q.lb = k1 * I.n2 + (r ? I.n2 - r : h2);
  q.shared = r != 0;
  const double k1t = I.a1 * (double)k1 * (double)k1;
  q.ka = k1t + I.a2 * (double)r * (double)r;
  q.kb = r ? q.ka : k1t + I.a2 * (double)h2 * (double)h2;
  return q;
}

// line index of one half of pair P (-1: none)
__device__ __forceinline__ int pair_line(CInst& I, int P, int half) {
  if (I.n2 == 1) return half ? -1 : P;
  const int h2 = I.n2 >> 1;
  const int k1 = fdiv(P, I.m_h2), r = P - k1 * h2;
  return k1 * I.n2 + (half ? (r ? I.n2 - r : h2) : r);
}

// DFT of both halves of R pair points
template <typename T, int R>
__device__ __forceinline__ void dft_px(px<T>* v) {
  cx<T> u[R];
#pragma unroll
  for (int r = 0; r < R; ++r) u[r] = v[r].a;
  dft_reg<T, R>(u);
#pragma unroll
  for (int r = 0; r < R; ++r) v[r].a = u[r];
#pragma unroll
  for (int r = 0; r < R; ++r) u[r] = v[r].b;
  dft_reg<T, R>(u);
#pragma unroll
  for (int r = 0; r < R; ++r) v[r].b = u[r];
}
template <typename T>
__device__ __forceinline__ px<T> pmul(px<T> v, cx<T> w) {
  v.a = cmul(v.a, w);
  v.b = cmul(v.b, w);
  return v;
}

// v[d] *= w^d, d = 1 .. R-1 (R a power of two up to 16).  FP32: root(d) reads w^d from
// the table for d = 1 and 4, at R = 16 for 1 .. 4, 8 and 12, and the other powers are
// products of those, one (R = 16) to three deep.  Powers of w alone, each square
// doubling the error of the one before, took the error of a 1792-point transform from
// 8e-8 to 2.7e-7.  FP64 takes the powers of w: their error, below 1e-15, is nothing
// beside the window's 1e-11.
constexpr bool tw_read(int R, int d) { return R == 16 ? d <= 4 || d % 4 == 0 : d == 1 || d == 4; }
template <typename T, int R, typename Root>
__device__ __forceinline__ void tw_powers(cx<T>* w, Root root) {
#pragma unroll
  for (int d = 1; d < R; ++d) {
    if constexpr (sizeof(T) == 4)
      w[d] = tw_read(R, d) ? root(d) : d < 4 ? cmul(w[d - 1], w[1]) : cmul(w[d & ~3], w[d & 3]);
    else
      w[d] = d == 1 ? root(1) : (d & (d - 1)) == 0 ? cmul(w[d / 2], w[d / 2]) : cmul(w[d & (d - 1)], w[d & -d]);
  }
}
template <typename T, int R, typename Root>
__device__ __forceinline__ void twiddle_reg(cx<T>* v, Root root) {
  cx<T> w[R > 1 ? R : 2];
  tw_powers<T, R>(w, root);
#pragma unroll
  for (int d = 1; d < R; ++d) v[d] = cmul(v[d], w[d]);
}
template <typename T, int R, typename Root>
__device__ __forceinline__ void twiddle_px(px<T>* v, Root root) {
  cx<T> w[R > 1 ? R : 2];
  tw_powers<T, R>(w, root);
#pragma unroll
  for (int d = 1; d < R; ++d) v[d] = pmul(v[d], w[d]);
}

// One butterfly of R pair points, one half after the other (both at once would
// not fit in registers for the larger radices): get(r, half) reads the inputs,
// tw(d, X) applies the twiddle of output d, put(r, half, X) receives them.
template <typename T, int R, typename Get, typename Tw, typename Put>
__device__ __forceinline__ void bfly_px(Get get, Tw tw, Put put) {
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    cx<T> v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = get(r, h);
    dft_emit<T, R>(v, [&](int d, cx<T> x) { put(d, h, d ? tw(d, x) : x); });
  }
}

constexpr int kGTaps = 12;  // taps of the default window (2cK at c = 2, K = 3)

// Cell j of a grid line in LDS (ps = plane_stride(m)).
__device__ __forceinline__ int plane_cell(int j, int ps) { return (j & 3) * ps + (j >> 2); }

// ---------------------------------------------------------------------------
// Spreading of a line pair by one wavefront (the scheme of spread_line_wave,
// device.h): one node pair +-nu+ of both lines per lane, one tap per round.

template <typename T>
__device__ __forceinline__ void add_px(px<T>* c, px<T> v) {
  px<T> o = *c;
  o.a = cadd(o.a, v.a);
  o.b = cadd(o.b, v.b);
  *c = o;
}
template <typename T>
__device__ __forceinline__ px<T> scl_px(px<T> v, T w) {
  return px<T>{cscl(v.a, w), cscl(v.b, w)};
}
__device__ __forceinline__ int lane_get(int v, int k) { return __builtin_amdgcn_readlane(v, k); }
__device__ __forceinline__ float lane_get(float v, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}
__device__ __forceinline__ double lane_get(double v, int k) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, k);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), k);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Segments of a pass (see WaveSeg) from its first taps; a pass without equal
// first taps, the common case away from a line's smallest |nu|, has none.
// *gap: the distance to the lane before's first tap (large on lane 0 and past
// the active lanes).
__device__ __forceinline__ WaveSeg pair_segments(int j0, bool act, int* gap) {
  const int L = (int)(threadIdx.x & 63);
  const int key = act ? j0 : 0x40000000 + L;
  const int prev = __builtin_amdgcn_update_dpp(0, key, 0x138, 0xf, 0xf, true);  // wave_shr:1
  *gap = L == 0 || !act ? 64 : key - prev;
  if (__ballot(L == 0 || prev != key) == ~0ull) return WaveSeg{0u, 0u, true};
  return wave_segments(key);
}

// The segmented inclusive sums of a round: both halves of both passes' values,
// a step as x += on * (x of the source lane) with on = 0 or 1.  In float one
// instruction per value (a DPP multiply-add; written out, since the compiler
// keeps the move apart; the s_nop covers the DPP read of a value that the
// instruction before may have written).  Values that are not finite do not come
// here: times 0 they would reach other segments.
#define PAT_SEG_FMAC(K, CTRL) "v_fmac_f32_dpp %" #K ", %" #K ", %8 " CTRL "\n\t"
#define PAT_SEG_STEP(BIT, CTRL)                                                                                      \
  if (s.use & BIT) {                                                                                                 \
    const float on = (s.on & BIT) ? 1.0f : 0.0f;                                                                     \
    asm("s_nop 1\n\t" PAT_SEG_FMAC(0, CTRL) PAT_SEG_FMAC(1, CTRL) PAT_SEG_FMAC(2, CTRL) PAT_SEG_FMAC(3, CTRL)        \
            PAT_SEG_FMAC(4, CTRL) PAT_SEG_FMAC(5, CTRL) PAT_SEG_FMAC(6, CTRL) PAT_SEG_FMAC(7, CTRL)                  \
        : "+v"(p.a.x), "+v"(p.a.y), "+v"(p.b.x), "+v"(p.b.y), "+v"(m.a.x), "+v"(m.a.y), "+v"(m.b.x), "+v"(m.b.y)     \
        : "v"(on));                                                                                                  \
  }
__device__ __forceinline__ void seg_sum_px(const WaveSeg& s, px<float>& p, px<float>& m) {
  PAT_SEG_STEP(1u, "row_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0")
  PAT_SEG_STEP(2u, "row_shr:2 row_mask:0xf bank_mask:0xf bound_ctrl:0")
  PAT_SEG_STEP(4u, "row_shr:4 row_mask:0xf bank_mask:0xf bound_ctrl:0")
  PAT_SEG_STEP(8u, "row_shr:8 row_mask:0xf bank_mask:0xf bound_ctrl:0")
  PAT_SEG_STEP(16u, "row_bcast:15 row_mask:0xa bank_mask:0xf bound_ctrl:0")
  PAT_SEG_STEP(32u, "row_bcast:31 row_mask:0xc bank_mask:0xf bound_ctrl:0")
}
#undef PAT_SEG_STEP
#undef PAT_SEG_FMAC
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_0(double x) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROWS, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROWS, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <unsigned BIT, int CTRL, int ROWS>
__device__ __forceinline__ void seg_step_px(const WaveSeg& s, px<double>& p, px<double>& m) {
  if (s.use & BIT) {
    const double on = (s.on & BIT) ? 1.0 : 0.0;
    auto add = [&](double& x) { x = fma(dpp_0<CTRL, ROWS>(x), on, x); };
    add(p.a.x);
    add(p.a.y);
    add(p.b.x);
    add(p.b.y);
    add(m.a.x);
    add(m.a.y);
    add(m.b.x);
    add(m.b.y);
  }
}
__device__ __forceinline__ void seg_sum_px(const WaveSeg& s, px<double>& p, px<double>& m) {
  seg_step_px<1u, 0x111, 0xf>(s, p, m);
  seg_step_px<2u, 0x112, 0xf>(s, p, m);
  seg_step_px<4u, 0x114, 0xf>(s, p, m);
  seg_step_px<8u, 0x118, 0xf>(s, p, m);
  seg_step_px<16u, 0x142, 0xa>(s, p, m);
  seg_step_px<32u, 0x143, 0xc>(s, p, m);
}

// The 12 rounds of a batch, both passes in one loop: tap t of +nu+ and the tap of
// -nu+ with the same weight (-nu+ takes w reversed).
// BLOCK: no window wraps, the passes' cells are disjoint and the writers' first
//   taps at least two cells apart, so that two rounds go as one block (their
//   reads, then their writes): a round is an LDS round trip, and few waves fit
//   beside 16 KB of grid each.
// FLAT: no window wraps, the passes' cells are disjoint; segmented sums where
//   first taps coincide.
// else: cells wrapped; the passes one after the other, as they may meet.
// A node on a grid point (on) has its last tap on the window's edge, and -nu+
// includes the opposite edge: that tap is left out here.
// Four rounds are written out and run three times, the weights moved round by
// four: the instruction cache (64 KB for two CUs) holds the whole kernel then.
template <typename T, bool BLOCK, bool FLAT>
__device__ __forceinline__ void gspread_rounds(px<T>* G, int ps, int m, int rp, int rm, bool wr, bool on, px<T> vp,
                                               px<T> vm, T* w, const WaveSeg& sg) {
  static_assert(kGTaps == 12, "three turns of four taps");
  // (offsets, not pointers: pointers carried round the loop lose their LDS
  // address space, and a flat access takes several times as long)
  int op[4], om[4];
  if constexpr (FLAT) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      op[s] = plane_cell(rp + s, ps);
      om[s] = plane_cell(rm + s, ps) + 2;
    }
  }
#pragma unroll 1
  for (int t0 = 0; t0 < kGTaps; t0 += 4) {
    const T w3 = t0 == kGTaps - 4 && on ? T(0) : w[3];
    if constexpr (BLOCK) {
#pragma unroll
      for (int t = 0; t < 4; t += 2) {
        if (wr) {
          px<T> c[4], x[4];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            c[u] = G[op[t + u]];
            c[2 + u] = G[om[3 - t - u]];
            x[u] = scl_px(vp, w[t + u]);
            x[2 + u] = scl_px(vm, t + u == 3 ? w3 : w[t + u]);
          }
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            G[op[t + u]] = px<T>{cadd(c[u].a, x[u].a), cadd(c[u].b, x[u].b)};
            G[om[3 - t - u]] = px<T>{cadd(c[2 + u].a, x[2 + u].a), cadd(c[2 + u].b, x[2 + u].b)};
          }
        }
        // the next block's reads come after this block's writes
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      }
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        px<T> xp = scl_px(vp, w[t]), xm = scl_px(vm, t == 3 ? w3 : w[t]);
        if (sg.use) seg_sum_px(sg, xp, xm);
        if constexpr (FLAT) {
          if (wr) {
            const px<T> c = G[op[t]], d = G[om[3 - t]];
            G[op[t]] = px<T>{cadd(c.a, xp.a), cadd(c.b, xp.b)};
            G[om[3 - t]] = px<T>{cadd(d.a, xm.a), cadd(d.b, xm.b)};
          }
        } else {
          int cp = rp + t0 + t, cm = rm + kGTaps - 1 - t0 - t;
          cp -= cp >= m ? m : 0;
          cm -= cm >= m ? m : 0;
          if (wr) add_px(G + plane_cell(cp, ps), xp);
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
          if (wr) add_px(G + plane_cell(cm, ps), xm);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const T wt = w[t];
      w[t] = w[t + 4];
      w[t + 4] = w[t + 8];
      w[t + 8] = wt;
    }
    if constexpr (FLAT) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        ++op[s];
        --om[s];
      }
    }
  }
}

// first tap j mod m: m = M (a power of two) or run time
template <int M>
__device__ __forceinline__ int wrap_m(int j, int m, double inv_m) {
  if constexpr (M > 0) return j & (M - 1);
  return wrap_tap<false>(j, m, inv_m);
}

// One batch: lane L < nact holds the node pair +-nup, with the values conj(qp) pc
// and conj(qm) conj(pc) (pc: the node phase times the weight), for the halves of
// the pair that ha and hb select.  spread_setup forms windows, cells and segments
// (independent of the grid: the waves of a pair do it side by side, and it takes
// most of the time), spread_apply adds the batch to the grid lines G.
template <typename T>
struct SpreadBatch {
  px<T> vp, vm;
  T w[kGTaps];
  int j0, rp, rm, nact;
  bool act, on;
};
template <typename T, int M>
__device__ __forceinline__ SpreadBatch<T> spread_setup(const StageArgs& a, double c, double ck, int m, double inv_m,
                                                       double nup, cx<T> pc, bool act, int nact, bool ha, bool hb,
                                                       px<T> qp, px<T> qm) {
  SpreadBatch<T> s;
  const cx<T> zero = mk(T(0), T(0)), pcc = cconj(pc);
  s.vp = px<T>{cmul(cconj(qp.a), pc), cmul(cconj(qp.b), pc)};
  s.vm = px<T>{cmul(cconj(qm.a), pcc), cmul(cconj(qm.b), pcc)};
  if (!(act && ha)) s.vp.a = s.vm.a = zero;
  if (!(act && hb)) s.vp.b = s.vm.b = zero;
  const double d = tap_origin(c * nup, ck, &s.j0);
  s.act = act;
  s.nact = nact;
  tap_weights_pairs<T, kGTaps>(a, (T)(2.0 * d + 1.0), s.w);
  s.on = d == -1.0;
  s.rp = wrap_m<M>(s.j0, m, inv_m);
  s.rm = wrap_m<M>(-(s.j0 + kGTaps - 1), m, inv_m);
  return s;
}
template <typename T>
__device__ __forceinline__ void spread_apply(SpreadBatch<T>& s, int m, int ps, px<T>* G) {
  const int L = (int)(threadIdx.x & 63);
  const int nact = s.nact;
  auto mag = [](const px<T>& v) { return fabs(v.a.x) + fabs(v.a.y) + fabs(v.b.x) + fabs(v.b.y); };
  const T big = mag(s.vp) + mag(s.vm);
  const int jf = lane_get(s.j0, 0), jl = lane_get(s.j0, nact - 1);
  // one by one, one tap per lane (+nu+ on lanes 0 .., -nu+ on lanes 32 ..): a few
  // nodes, values that are not finite (the sums of others stay clear of them;
  // lanes past nact count too: they read a valid node and carry zeros), windows
  // that may meet at any distance of lanes, nodes that coincide on a grid point
  // (l^2 lost beside K^2: their edge taps, added after the rounds, share a cell)
  const bool anyon = __any(s.act && s.on);
  bool twins = false;
  if (anyon) {
    const int key = s.act && s.on ? s.j0 : 0x40000000 + L;
    twins = __any(__builtin_amdgcn_update_dpp(0, key, 0x138, 0xf, 0xf, true) == key && L > 0);
  }
  if (nact <= 2 || twins || __any(!(big - big == T(0))) || jl - jf >= m) {
#pragma unroll 1
    for (int k = 0; k < nact; ++k) {
      const bool onk = lane_get((int)s.on, k) != 0, minus = L >= 32;
      const int t = L & 31;
      T w = T(0);
#pragma unroll
      for (int i = 0; i < kGTaps; ++i) {
        const T wi = lane_get(s.w[i], k);
        w = t == i ? wi : w;
      }
      auto get = [&](T p, T q) {
        const T vp = lane_get(p, k), vq = lane_get(q, k);
        return minus ? vq : vp;
      };
      const px<T> v{mk(get(s.vp.a.x, s.vm.a.x), get(s.vp.a.y, s.vm.a.y)),
                    mk(get(s.vp.b.x, s.vm.b.x), get(s.vp.b.y, s.vm.b.y))};
      const int rp = lane_get(s.rp, k) + t, rm = lane_get(s.rm, k) + (onk ? t + 1 : kGTaps - 1 - t);
      int c = minus ? rm : rp;
      c -= c >= m ? m : 0;
      if (t < kGTaps && !minus) add_px(G + plane_cell(c, ps), scl_px(v, w));
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      if (t < kGTaps && minus) add_px(G + plane_cell(c, ps), scl_px(v, w));
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    return;
  }
  int gap;
  const WaveSeg sg = pair_segments(s.j0, s.act, &gap);
  const bool wr = s.act && sg.tail;
  if (!passes_disjoint<kGTaps>(jf, jl, m) || __any(wr && (s.rp > m - kGTaps || s.rm > m - kGTaps)))
    gspread_rounds<T, false, false>(G, ps, m, s.rp, s.rm, wr, s.on, s.vp, s.vm, s.w, sg);
  else if (sg.use || __any(gap < 2))
    gspread_rounds<T, false, true>(G, ps, m, s.rp, s.rm, wr, s.on, s.vp, s.vm, s.w, sg);
  else
    gspread_rounds<T, true, true>(G, ps, m, s.rp, s.rm, wr, s.on, s.vp, s.vm, s.w, sg);
  // the edge taps left out: 12 cells above where w reversed would have them (no
  // two of the wave's nodes on grid points share a first tap here, and they span
  // less than m)
  if (anyon) {
    int c = s.rm + kGTaps;
    c -= c >= m ? m : 0;
    if (s.act && s.on) add_px(G + plane_cell(c, ps), scl_px(s.vm, s.w[kGTaps - 1]));
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  }
}

// Values of the node pair |l| = la of depth spectra D (natural order): R^T (mode
// 0) takes Qhat_l and Qhat_-l (the Nyquist plane for both nodes at l = nz/2), A
// their sum for both; *cf is the weight that goes with them.
template <typename T, typename Get>
__device__ __forceinline__ void node_values(CInst& I, int mode, int la, double nup, Get D, px<T>* qp, px<T>* qm,
                                            double* cf) {
  const int half = I.nz / 2;
  *qp = D(la);
  if (mode == 0) {
    *qm = la == half ? *qp : D(I.nz - la);
    *cf = I.wcoef * I.scale * (double)la * rcp_nt(nup) * (la == half ? 0.5 : 1.0);
  } else {
    if (la != 0 && la != half) {
      const px<T> o = D(I.nz - la);
      qp->a = cadd(qp->a, o.a);
      qp->b = cadd(qp->b, o.b);
    }
    *qm = *qp;
    *cf = 0.5 * I.scale;
  }
}

}  // namespace pat
