// Host entry points of the general-length kernels (general.hip): the stages of
// an operator over instances of any length the plans accept, in one launch
// per stage.  `a` holds the instances and arrays; the item counts, the
// tables' LDS and the launch shape are set here.
#pragma once

#include "device.h"

namespace pat {

template <typename T>
struct General {
  static hipError_t x1(StageArgs& a, const Inst* h, hipStream_t st, StageTimer* tm);
  static hipError_t x2(StageArgs& a, const Inst* h, hipStream_t st, StageTimer* tm);
  static hipError_t c2r(StageArgs& a, const Inst* h, hipStream_t st, StageTimer* tm);
  static hipError_t line2(StageArgs& a, const Inst* h, hipStream_t st, StageTimer* tm);
  static hipError_t line1(StageArgs& a, const Inst* h, hipStream_t st, StageTimer* tm);
  // line1's items of one instance over the workgroups that are resident at once (0 on
  // a HIP error)
  static double line1_rounds(const Inst& h);
};

// The transverse passes of one instance at 128, 256 and 512 points, sizes
// fixed at compile time (transverse.hip).
template <typename T>
struct Fixed {
  // Length L on `rows` lines of len samples, where its tiles of 32 samples give
  // every CU one (below that the general-length kernels' narrower tiles take
  // less time).
  static bool takes(int L, int rows, int len);
  static hipError_t x1(StageArgs& a, const Inst& h, hipStream_t st, StageTimer* tm);
  static hipError_t x2(StageArgs& a, const Inst& h, hipStream_t st, StageTimer* tm);
  static hipError_t c2r(StageArgs& a, const Inst& h, hipStream_t st, StageTimer* tm);
};

// The fused type-1 line stage of a 3D instance with m = 512 or 1024 grid
// points and nz = m/4, one line pair per workgroup (linepair.hip).
template <typename T>
struct PairLine {
  static bool takes(const Inst& h);
  static hipError_t line1(StageArgs& a, const Inst& h, hipStream_t st, StageTimer* tm);
  // stand-alone spreading of one 3D instance, the grid in the compute type
  static bool spreads(const Inst& h);
  static hipError_t spread(StageArgs& a, const Inst& h, hipStream_t st, StageTimer* tm);
};

}  // namespace pat
