// Type-1 line stages of 3D plans with m = 512 or 1024 grid points and nz = m/4:
// one line pair per workgroup, of one wave per batch of 64 node pairs.
//
// The two lines of a mirror pair (k1, +-k2) share their nodes: window polynomials,
// phase, FP64 position and segments are formed once for both, by the waves of the
// pair side by side, and every LDS access serves both lines.  The batches are then
// added to the grid in turn.  Of 161 us for 256^3 the FFTs and the memory traffic
// take 59, the set-up of the nodes 17, and the rounds the rest: read-add-write
// trips through LDS one after the other, at four waves per SIMD.  One line per wave
// (k_line_nufft1_w): 174 us, and 40 against 31 for 128^3.  Where the chip is not filled
// the shorter chains of k_line_nufft1_w win (64^3: 14 against 18.6 us; see takes).  In
// FP64 (32 bytes a pair point, two waves per SIMD): 367 us against 412 for 256^3,
// 57 against 79 for 128^3.  (No instance for m = 2048 or nz = m/2: R^T and A at 512^3 run
// k_line_nufft1_c, nt = nz k_line_nufft1_w.)
#include "general.h"
#include "linepair.h"

namespace pat {

// Digits of the grid FFT (m = 8 G1 GL) and the depth FFT (nz = Z0 Z1 ZL), rows as
// in GFft.
template <int LM>
struct PairPlan {
  static constexpr int m = 1 << LM, nz = m / 4, nt = m / 2, half = nz / 2;
  static constexpr int G1 = 8, GL = LM == 10 ? 16 : 8;
  static constexpr int GLP = GL | 1, GB = (G1 * GLP) | 1, GS = G1 * GL, GN = 8 * G1, rows = 8 * GB;
  static constexpr int Z0 = LM == 10 ? 8 : 4, Z1 = 8, ZL = 4;
  static constexpr int ZLP = ZL | 1, ZB = (Z1 * ZLP) | 1, ZS = Z1 * ZL, ZN = Z0 * Z1, zrows = Z0 * ZB;
  static_assert(8 * G1 * GL == m && Z0 * Z1 * ZL == nz && zrows + nz <= rows, "digits");
  // batches of 64 node pairs, one per wave
  static constexpr int NB = (half + 63) / 64, NT = 64 * NB;
  static constexpr int PS = plane_stride(m);
  static_assert(4 * PS <= rows, "planes");
  static constexpr int points = rows;
};

template <typename T, int LM>
__global__ __launch_bounds__((PairPlan<LM>::NT), (sizeof(T) == 4 ? 4 : 2)) void k_pair_nufft1(StageArgs a) {
  using P = PairPlan<LM>;
  CInst& I = *(CInst*)a.inst[0];
  constexpr int m = P::m, nz = P::nz, nt = P::nt, half = P::half, NT = P::NT;
  px<T>* buf = reinterpret_cast<px<T>*>(pat_smem);
  const cx<T>* twm = static_cast<const cx<T>*>(I.tw) + I.gm.tw;
  const cx<T>* twz = static_cast<const cx<T>*>(I.tw) + I.gz.tw;
  const int tid = (int)threadIdx.x;
  const PairLines q = pair_lines(I, (int)blockIdx.x);
  const int h = tid & 1;  // line of the pair, where lanes alternate
  // depth FFTs of both lines (neighbouring lanes), into natural order behind
  // their scratch
  {
    const cx<T>* in = static_cast<const cx<T>*>(a.in[0]) + (size_t)(h ? q.lb : q.la) * nz;
    cx<T>* z = reinterpret_cast<cx<T>*>(buf) + h;
#pragma unroll
    for (int id = tid >> 1; id < P::ZS; id += NT / 2) {
      cx<T> v[P::Z0];
#pragma unroll
      for (int r = 0; r < P::Z0; ++r) v[r] = in[id + r * P::ZS];
      dft_reg<T, P::Z0>(v);
      twiddle_reg<T, P::Z0>(v, [&](int d) { return twz[id * d]; });
      cx<T>* s = z + 2 * (id + id / P::ZL * (P::ZLP - P::ZL));
#pragma unroll
      for (int r = 0; r < P::Z0; ++r) s[2 * r * P::ZB] = v[r];
    }
    __syncthreads();
#pragma unroll
    for (int id = tid >> 1; id < P::Z0 * P::ZL; id += NT / 2) {
      const int blk = id / P::ZL, j = id % P::ZL;
      cx<T>* s = z + 2 * (blk * P::ZB + j);
      cx<T> v[P::Z1];
#pragma unroll
      for (int r = 0; r < P::Z1; ++r) v[r] = s[2 * r * P::ZLP];
      dft_reg<T, P::Z1>(v);
      twiddle_reg<T, P::Z1>(v, [&](int d) { return twz[j * P::Z0 * d]; });
#pragma unroll
      for (int r = 0; r < P::Z1; ++r) s[2 * r * P::ZLP] = v[r];
    }
    __syncthreads();
#pragma unroll
    for (int id = tid >> 1; id < P::ZN; id += NT / 2) {
      const int d1 = id % P::Z0, d2 = id / P::Z0;
      const cx<T>* s = z + 2 * (d1 * P::ZB + d2 * P::ZLP);
      cx<T> v[P::ZL];
#pragma unroll
      for (int r = 0; r < P::ZL; ++r) v[r] = s[2 * r];
      dft_reg<T, P::ZL>(v);
      cx<T>* d = z + 2 * (P::zrows + id);
#pragma unroll
      for (int r = 0; r < P::ZL; ++r) d[2 * r * P::ZN] = v[r];
    }
    __syncthreads();
  }
  // each wave takes its batch's node values into registers, then the whole
  // region becomes the grid
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const px<T>* D = buf + P::zrows;
  px<T> q0 = D[0];
  q0 = px<T>{mk(lane_get(q0.a.x, 0), lane_get(q0.a.y, 0)), mk(lane_get(q0.b.x, 0), lane_get(q0.b.y, 0))};
  constexpr int nact = half < 64 ? half : 64;
  const bool act = (tid & 63) < nact;
  const int la = min(64 * wave + (tid & 63) + 1, half);
  px<T> qp, qm;
  double cf;
  node_values<T>(I, 1, la, 0.0, [&](int l) { return D[l]; }, &qp, &qm, &cf);  // (A: cf holds for every node)
  if (a.mode == 0) {
    qp = D[la];
    qm = la == half ? qp : D[nz - la];
  }
  __syncthreads();
  const px<T> zero{mk(T(0), T(0)), mk(T(0), T(0))};
  for (int e = tid; e < 4 * P::PS; e += NT) buf[e] = zero;
  // (A's node l = 0 is a pass of its own, of the last wave)
  const int passes = (q.shared ? 1 : 2) * (a.mode == 0 ? 1 : 2);
#pragma unroll 1
  for (int s = 0; s < passes; ++s) {
    const bool l0 = a.mode != 0 && (s & 1), second = (a.mode == 0 ? s : s >> 1) != 0;
    const bool some = !l0 || wave == P::NB - 1;
    const int l = l0 ? 0 : la;
    const double nup = sqrt_nt((second ? q.kb : q.ka) + I.b * (double)l * (double)l);
    const double w = a.mode == 0 ? I.wcoef * I.scale * (double)la * rcp_nt(nup) * (la == half ? 0.5 : 1.0) : cf;
    SpreadBatch<T> b = spread_setup<T, m>(a, 2.0, I.ck, m, 0.0, nup, cscl(phase_mpi<T>(nup), (T)w),
                                          l0 ? (tid & 63) == 0 : act, l0 ? 1 : nact, !second, q.shared || second,
                                          l0 ? q0 : qp, l0 ? q0 : qm);
    // the waves add their batches in turn
    __syncthreads();
    for (int o = 0; o < wave; ++o) __syncthreads();
    if (some) spread_apply<T>(b, m, P::PS, buf);
    for (int o = wave + 1; o < P::NB; ++o) __syncthreads();
  }
  __syncthreads();
  // grid FFTs: the first stage takes the line from natural order into the
  // padded rows through registers
  {
    constexpr int U = P::GS >= NT ? P::GS / NT : 1;
    px<T> v[U][8];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = tid + NT * u;
      if (j < P::GS) {
#pragma unroll
        for (int r = 0; r < 8; ++r) v[u][r] = buf[plane_cell(j, P::PS) + r * (P::GS / 4)];
        dft_px<T, 8>(v[u]);
        twiddle_px<T, 8>(v[u], [&](int d) { return twm[j * d]; });
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = tid + NT * u;
      if (j < P::GS) {
        px<T>* s = buf + j + j / P::GL * (P::GLP - P::GL);
#pragma unroll
        for (int r = 0; r < 8; ++r) s[r * P::GB] = v[u][r];
      }
    }
    __syncthreads();
  }
#pragma unroll 1
  for (int id = tid; id < 8 * P::GL; id += NT) {
    const int blk = id / P::GL, j = id % P::GL;
    px<T>* s = buf + blk * P::GB + j;
    px<T> v[P::G1];
#pragma unroll
    for (int r = 0; r < P::G1; ++r) v[r] = s[r * P::GLP];
    dft_px<T, P::G1>(v);
    twiddle_px<T, P::G1>(v, [&](int d) { return twm[8 * j * d]; });
#pragma unroll
    for (int r = 0; r < P::G1; ++r) s[r * P::GLP] = v[r];
  }
  __syncthreads();
  // last stage, one line per lane: X_n = s_n conj(G_k), k = (n - nt/2) mod m: the
  // outputs k = n + d GN of the first and the last quarter of d, the others are
  // not formed
  const T* sn = static_cast<const T*>(I.sn_g);
  cx<T>* x = static_cast<cx<T>*>(a.out[0]) + (size_t)(h ? q.lb : q.la) * nt;
#pragma unroll 1
  for (int id = tid >> 1; id < P::GN; id += NT / 2) {
    const cx<T>* s = reinterpret_cast<const cx<T>*>(buf + id % 8 * P::GB + id / 8 * P::GLP) + h;
    cx<T> v[P::GL];
#pragma unroll
    for (int r = 0; r < P::GL; ++r) v[r] = s[2 * r];
    dft_reg<T, P::GL>(v);
#pragma unroll
    for (int d = 0; d < P::GL / 4; ++d) {
      const int np = id + d * P::GN + nt / 2, nm = id + (d + 3 * P::GL / 4) * P::GN - m + nt / 2;
      x[np] = cscl(cconj(v[d]), sn[np]);
      x[nm] = cscl(cconj(v[d + 3 * P::GL / 4]), sn[nm]);
    }
  }
}

// Stand-alone spreading of 3D plans (any m that is a multiple of 4, one instance):
// one line pair per workgroup as above, the grid lines written out conjugated.  In
// FP64 319 us for 256^3, where the gather (k_line_spread) takes 377 and the writes
// alone about 90; in FP32 it equals k_line_spread_w there (135 us) and loses below,
// so only the FP64 one is built.
template <typename T>
__global__ __launch_bounds__(kBlock, (sizeof(T) == 4 ? 4 : 2)) void k_pair_spread(StageArgs a) {
  CInst& I = *(CInst*)a.inst[0];
  px<T>* buf = reinterpret_cast<px<T>*>(pat_smem);
  const int NT = blockDim.x, tid = (int)threadIdx.x, L = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = NT >> 6;
  const int m = I.m, ps = plane_stride(m), nz = I.nz, half = nz / 2;
  const double inv_m = 1.0 / (double)m;
  const PairLines q = pair_lines(I, (int)blockIdx.x);
  const cx<T>* fa = static_cast<const cx<T>*>(a.in[0]) + (size_t)q.la * nz;
  const cx<T>* fb = static_cast<const cx<T>*>(a.in[0]) + (size_t)q.lb * nz;
  const px<T> zero{mk(T(0), T(0)), mk(T(0), T(0))};
  for (int e = tid; e < 4 * ps; e += NT) buf[e] = zero;
  // turns of nw batches; A's node l = 0 is a turn of its own, of the last wave
  const int turns = (half + 64 * nw - 1) / (64 * nw) + (a.mode == 0 ? 0 : 1), all = q.shared ? turns : 2 * turns;
#pragma unroll 1
  for (int s = 0; s < all; ++s) {
    const bool second = s >= turns;
    const int u = second ? s - turns : s;
    const bool l0 = a.mode != 0 && u == turns - 1;
    const int base = l0 ? 0 : 64 * (u * nw + wave) + 1;
    const int nact = l0 ? (wave == nw - 1 ? 1 : 0) : min(64, half + 1 - base);
    const bool act = L < nact;
    const int la = l0 ? 0 : act ? base + L : 1;
    const double nup = sqrt_nt((second ? q.kb : q.ka) + I.b * (double)la * (double)la);
    px<T> qp, qm;
    double cf;
    node_values<T>(I, a.mode, la, nup, [&](int l) { return px<T>{fa[l], fb[l]}; }, &qp, &qm, &cf);
    const cx<T> ph = I.centred ? phase_mpi<T>(nup) : mk(T(1), T(0));
    SpreadBatch<T> b = spread_setup<T, 0>(a, I.c, I.ck, m, inv_m, nup, cscl(ph, (T)cf), act, nact, !second,
                                          q.shared || second, qp, qm);
    __syncthreads();
    for (int o = 0; o < wave; ++o) __syncthreads();
    if (nact > 0) spread_apply<T>(b, m, ps, buf);
    for (int o = wave + 1; o < nw; ++o) __syncthreads();
  }
  __syncthreads();
  cx<T>* ga = static_cast<cx<T>*>(a.out[0]) + (size_t)q.la * m;
  cx<T>* gb = static_cast<cx<T>*>(a.out[0]) + (size_t)q.lb * m;
  for (int j = 2 * tid; j < m; j += 2 * NT) {
    const px<T> v = buf[plane_cell(j, ps)], w = buf[plane_cell(j + 1, ps)];
    *reinterpret_cast<px<T>*>(ga + j) = px<T>{cconj(v.a), cconj(w.a)};
    *reinterpret_cast<px<T>*>(gb + j) = px<T>{cconj(v.b), cconj(w.b)};
  }
}

// FP64 only, from 8 pairs per CU on (32^3: 17 us against 12 of k_line_spread, 96^3: 31
// against 50), where a pair's wave or waves find enough others beside them.  Times
// against k_line_spread's, first the pairs':
//   one batch per line (nz up to 128): m = 400 to 1600 23 to 49 against 39 to 51 us at 2112
//     pairs; m = 1800 58 against 53 (nz = 64), 64 against 53 (nz = 128); nz = 16 at any m
//     (m = 2520: 59 against 83)
//   several (nz up to 500), whose turns wait for each other: m = 600, nz = 150: 53 against
//     42 at 2112 pairs, 88 against 87 at 4160; m = 736: 93 against 108 at 5236, 137 against
//     181 at 8556; m = 1024, nz = 256: 97 against 84 at 4160, 319 against 377 at 16512; m =
//     1600: 242 against 249 at 10100; m = 2000: 328 against 244 at 8320
//   nz from 500 on, where k_line_spread's node lists leave two workgroups per CU: 129 against
//     141 at m = 2000, 155 against 190 at m = 2400
template <typename T>
bool PairLine<T>::spreads(const Inst& h) {
  const int cu = num_cu();
  if (sizeof(T) != 8 || h.n2 == 1 || h.npair < 8 * cu || h.m % 4 != 0 || h.m < 2 * kGTaps) return false;
  if ((size_t)h.npair * (h.n2 / 2) >= (size_t(1) << 32) || 4 * (size_t)plane_stride(h.m) * sizeof(px<T>) > 80 * 1024) return false;
  if (h.nz <= 32 || h.nz >= 500) return true;
  if (h.nz <= 128) return h.m <= 1600;
  return h.npair >= 32 * cu ? h.m <= 1600 : h.npair >= 16 * cu && h.m <= 800;
}

template <typename T>
hipError_t PairLine<T>::spread(StageArgs& a, const Inst& h, hipStream_t st, StageTimer* tm) {
  a.total = h.npair;
  a.counter = nullptr;
  const int nw = (h.nz / 2 + 63) / 64;
  if constexpr (sizeof(T) == 4) return hipErrorInvalidValue;
  else
    return launch(k_pair_spread<T>, "spread", a, 4 * plane_stride(h.m) * sizeof(px<T>), st, tm, 64 * (nw < 4 ? nw : 4));
}

// From 4.5 pairs per CU on in FP32; in FP64, where a pair's latency is longer, from 2.1
// (m = 512) and 8.2 (m = 1024) on, and with 128 lines k2 or more at any number (the pair
// r = 0, which takes two passes, is then one in 64).  k_line_nufft1_w below, its time
// first: FP32, m = 512: 20 to 2300 lines 13 to 17 against 13 to 19 us, 4200 lines 28
// against 22; m = 1024: 1040 lines 21 against 23, 2300 lines 26 against 26, 4224 lines 40
// against 36.  FP64, m = 512: 516 lines 21 against 25, 2064 lines 36 against 30; m = 1024:
// 1032 lines 32 against 37, 4128 lines 73 against 84; with n2 = 128, 640 lines 19 against 17.
template <typename T>
bool PairLine<T>::takes(const Inst& h) {
  if (!h.gln || h.n2 == 1 || h.m != 2 * h.nt || 4 * h.nz != h.m || (h.m != 512 && h.m != 1024)) return false;
  const int cu = num_cu();
  if (sizeof(T) == 4) return 2 * h.npair > 9 * cu;
  return h.n2 >= 128 || 10 * h.npair > (h.m == 512 ? 21 : 82) * cu;
}

template <typename T>
hipError_t PairLine<T>::line1(StageArgs& a, const Inst& h, hipStream_t st, StageTimer* tm) {
  a.total = h.npair;
  a.counter = nullptr;
  auto go = [&](auto kern, int points, int threads) {
    return launch(kern, "nufft_adjoint_fused", a, points * sizeof(px<T>), st, tm, threads);
  };
  if (h.m == 512) return go(k_pair_nufft1<T, 9>, PairPlan<9>::points, PairPlan<9>::NT);
  return go(k_pair_nufft1<T, 10>, PairPlan<10>::points, PairPlan<10>::NT);
}

template struct PairLine<float>;
template struct PairLine<double>;

}  // namespace pat
