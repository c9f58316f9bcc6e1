// Internal data shared by the host plan (plan.cpp), the kernels
// (kernels.hip) and the C ABI layer (capi.cpp).  Plain structs only: the
// descriptor is built on the host in FP64 and copied verbatim to the device.
#pragma once

#include <cstddef>
#include <cstdint>

namespace pat {

constexpr int kMaxStages = 16;   // radix stages of one FFT
constexpr int kMaxBatch = 32;    // instances in one batched call
constexpr int kMaxTaps = 64;     // 2cK
constexpr double kMaxCutoff = 8.0;  // cut-off radius in sampling steps
constexpr int kBlock = 256;      // threads per workgroup of every kernel
constexpr int kNumCounters = 32; // persistent work counters per batched call (8 per radix class)
// Bytes of the static per-device scratch array behind the allocation-free
// entry point (pat_reconstruct_noalloc); a plan whose workspace needs more is
// refused there.
constexpr size_t kScratchBytes = size_t(64) << 20;
constexpr int kMaxDevices = 64;   // devices the scratch addresses are cached for
constexpr size_t kLdsMax = 160 * 1024;  // LDS of one CDNA4 compute unit
constexpr double kPi = 3.14159265358979323846264338327950288;
// Degree of the per-tap polynomial that replaces the kernel evaluation
// (float and double paths).
constexpr int kPolyDegF = 8;
constexpr int kPolyDegD = 15;
// 32-bit words of the mirrored tap-pair coefficients passed in kernel arguments
constexpr int kPolyWords = 192;

// One FFT length: in-place decimation-in-frequency mixed-radix factorisation.
// After the transform the natural-order bin k sits at LDS position perm[k].
struct FftDesc {
  int32_t L;
  int32_t nst;
  int32_t rad[kMaxStages];
  int32_t tw;    // element offset of the L roots exp(-2 pi i k / L) in the twiddle table
  int32_t perm;  // element offset of the bin -> position map in the index table
};

// Division by a constant d >= 2 as a 32-bit multiply-high: n / d for
// n d < 2^32 is the high word of n (floor(2^32 / d) + 1); 0 stands for d = 1.
inline uint32_t div_magic(int d) { return d <= 1 ? 0u : (uint32_t)((1ull << 32) / (uint64_t)d) + 1u; }

// One FFT length of the general-length kernels (general.hip): an in-place
// decimation-in-frequency transform of L = r0 r1 rl points in two or three
// stages (r1 = 1: two), every radix up to 23 transformed in registers.  In
// LDS the points are kept in rows: point d1 (r1 rl) + d2 rl + e sits in row
// d1 bs + d2 rlp + e, with rlp >= rl and bs >= r1 rlp odd, so that lanes that
// walk the last stage's butterflies or the first stage's digits meet
// different banks.
struct GFft {
  int32_t L, r0, r1, rl;
  int32_t rlp, bs;  // row strides of the digits d2 and d1
  int32_t sub0;     // r1 rl: first-stage butterflies
  int32_t nbl;      // r0 r1: last-stage butterflies
  int32_t rows;     // r0 bs: rows of one transform
  int32_t tw;       // element offset of the L roots in the twiddle table
  uint32_t m_sub0, m_rl, m_r1, m_r0, m_nbl, m_nb1;  // div_magic of sub0, rl, r1, r0, nbl, r0 rl
};

// Everything a kernel needs about one reconstruction instance.
struct Inst {
  int32_t n1, n2, nt, nz, m;  // detectors, time samples, depth samples, c*nt
  int32_t h1;                 // n1/2 + 1 (half spectrum over the first axis)
  int32_t lines;              // h1 * n2 frequency lines
  int32_t taps;               // 2cK
  int32_t tb;                 // batch width of the transverse tiles
  int32_t poly;               // 1: per-tap polynomial table valid, 0: direct kernel evaluation
  int32_t lpw_m, lpw_z, lpw_i;  // lines per work item: length-m FFT stages, depth FFT, interp/spread
  int32_t pow2;               // every FFT length is a power of two
  int32_t lpw_f;              // lines per work item of the fused line kernels
  int32_t lpw_a;              // lines per work item of the fused adjoint kernel
  int32_t kind;               // pat_interp: how the nonuniform sums are evaluated
  int32_t centred;            // grid from centred samples (KB, sinc) or not (linear, nearest)
  int32_t fused;              // 1: line stages fused in LDS (grid never stored), 0: staged
  int32_t cut_e;              // cut-off band width E = ceil(2 eps) in samples; 0: no cut-off
  int32_t twg_m;              // 1: the staged grid-line kernels read the c*nt-point twiddles from
                              // memory (table and line together exceed LDS), 0: from LDS
  double c, K, alpha;
  double ck;                  // c*K
  // node and weight:  nu+^2 = a1 k1^2 + a2 k2^2 + b l^2 ;  W = wcoef |l| / nu+
  double a1, a2, b, wcoef;
  // 1 / (pi c n1 n2 nz): the 1/(2 pi c) of the NUFFT identity with the factor
  // 2 e^{alpha K} folded into the deconvolution table, and the inverse-DFT
  // normalisation.
  double scale;
  FftDesc f1, f2, fm, fz;
  // General-length kernels: gtr = 1 when they can take the transverse passes,
  // gln = 1 the fused line stages.  The line kernels run the Kaiser-Bessel sums on
  // a grid of gm.L = 8 r1 rl >= m points of their own choice (c_g = gm.L / nt)
  // with the plan's window in grid units; np lines or mirror pairs per item.
  int32_t gtr, gln;
  int32_t gtb1, gtb2;        // tile widths (complex columns) of the x1 and x2 passes
  int32_t np, npair;         // pairs per work item, pairs of the instance
  uint32_t m_half, m_half1;  // div_magic of nz/2, nz/2 + 1
  uint32_t m_h2;             // div_magic of n2/2 (pairs per k1)
  GFft g1, g2, gm, gz;
  double c_g;
  // device addresses inside this instance's table buffer (set at upload)
  const void* tw;        // cplx<T>[]
  const int32_t* perm;   // int32[]
  const void* sn;        // T[nt]: e^{alpha K} / I0(K sqrt(alpha^2 - theta_n^2))
  const void* sn_g;      // T[nt]: the same factors for the grid of gm.L points
  const void* poly_c;    // T[taps][deg+1]: tap t as a polynomial in x = 2 (delta - cK) + 1
  // T[(E+1)^3]: cut-off weight by the samples' distances d_i = min(s, n - s)
  // to the data box faces per axis (x1, x2, t), each clamped to E; entry
  // ((d1 (E+1) + d2) (E+1) + d3).  2D plans use d2 = E.
  const void* cutw;
  // workspace byte offsets
  int64_t off_g, off_u, off_f;
};

// LDS bytes each kernel needs for one instance (cs: bytes per complex
// element, rs: per real).  The kernels carve their LDS exactly as described
// here; the host plan uses the same functions for its capacity checks and the
// launchers for the dynamic LDS request.
// (FFT kernels start with the twiddle table of each length they transform)
// (x1 passes: plus one column's (E+1)^2 cut-off weights when a cut-off is set)
inline size_t lds_tile_x1(const Inst& I, size_t cs) {
  const size_t e1 = (size_t)I.cut_e + 1;
  return (size_t)I.n1 * (I.tb + 1) * cs + (I.cut_e ? e1 * e1 * (cs / 2) : 0);
}
inline size_t lds_tile_x2(const Inst& I, size_t cs) { return (size_t)I.n2 * (I.tb + 1) * cs; }
inline size_t lds_line_z(const Inst& I, size_t cs) { return (size_t)I.nz * (I.lpw_z + 1) * cs; }
inline size_t lds_line_m(const Inst& I, size_t cs) { return (size_t)I.m * (I.lpw_m + (I.twg_m ? 0 : 1)) * cs; }
// interp: lpw_i grid lines of m entries plus a halo of taps - 1
inline size_t lds_interp(const Inst& I, size_t cs) { return (size_t)I.lpw_i * ((size_t)I.m + I.taps) * cs; }
// streamed interp: one buffer of lpw_i lines, line stride m + taps - 1
// rounded up to 16 bytes
inline size_t lds_interp_stream(const Inst& I, size_t cs) {
  const size_t q = cs >= 16 ? 1 : 16 / cs;
  const size_t ls = ((size_t)I.m + I.taps - 1 + q - 1) / q * q;
  return (size_t)I.lpw_i * ls * cs;
}
// spreading lists: per-node value, zero-padded tap-weight row (taps + 6
// entries, made odd), first tap; nz + 2 nodes at most
inline size_t lds_spread_lists(int nz, int taps, size_t cs, int kcells = 4) {
  const size_t row = (size_t)((taps + 2 * (kcells - 1)) | 1);
  return ((size_t)nz + 2) * (cs + row * (cs / 2) + sizeof(int32_t));
}
// stand-alone spreading gathers 4 cells per thread, the fused adjoint 2
inline size_t lds_spread(const Inst& I, size_t cs) { return lds_spread_lists(I.nz, I.taps, cs); }
inline size_t lds_spread_fused(const Inst& I, size_t cs) { return lds_spread_lists(I.nz, I.taps, cs, 2); }
// fused type-2 line kernel: lpw_f lines of max(m, nz) (FFT scratch, then the
// depth line) and lpw_f grid lines of m (natural order, no halo: at 1024
// points two lines take exactly 32 KB, five workgroups per compute unit)
inline size_t lds_fused2(const Inst& I, size_t cs) {
  const size_t sp = (size_t)(I.m > I.nz ? I.m : I.nz);
  return (size_t)I.lpw_f * (sp + (size_t)I.m) * cs;
}
// FP32 spreading by wavefronts: one grid line of m complex floats per
// wavefront of the workgroup (stand-alone), plus the depth spectra in the
// fused type-1 kernel
inline size_t lds_spread_wave(const Inst& I) { return (size_t)(kBlock / 64) * I.m * 8; }
inline size_t lds_fused1_wave(const Inst& I, size_t cs) {
  return (size_t)(kBlock / 64) * ((size_t)I.m + I.nz) * cs;
}
// fused type-1 line kernel: a region of max(m, lpw_a nz) (the depth FFTs,
// then one grid line), lpw_a depth spectra in natural order, the lists
inline size_t lds_fused1(const Inst& I, size_t cs) {
  const size_t za = (size_t)I.lpw_a * I.nz;
  return ((size_t)I.m > za ? (size_t)I.m : za) * cs + za * cs + lds_spread_fused(I, cs);
}

// general-length line kernels: np pairs of grid lines and of depth lines
// (two complex values per point), the depth roots, the roots of the middle grid
// stage
// Grid lines of the paired line kernels lie in LDS as four planes by cell mod 4,
// cell j at (j & 3) ps + (j >> 2).  The nodes of neighbouring lanes lie up to
// m / nz cells apart, 4 at nt = 2 nz: in natural order the lanes of an LDS cycle
// would meet in a quarter of its 16-byte banks.  With ps = 4 or 12 mod 16 cells 1,
// 2 and 4 apart all spread over the 16.
constexpr int plane_stride(int m) { return ((m / 4 + 3) & ~7) + 4; }
constexpr int kTw8 = 16;  // row length, the largest rl
constexpr int tw8_rows(int r1, int cs) { return r1 == 1 ? 0 : cs == 16 || r1 <= 4 ? 1 : r1 == 8 ? 2 : 6; }
inline size_t lds_gline(const Inst& I, int np, size_t cs) {
  return ((size_t)np * (I.gm.rows + I.gz.rows) * 2 + I.nz + kTw8 * tw8_rows(I.gm.r1, (int)cs)) * cs;
}
// general-length transverse passes: a tile and the roots
inline size_t lds_gtile(const GFft& g, int tb, size_t cs) { return ((size_t)g.rows * tb + g.L) * cs; }

}  // namespace pat
