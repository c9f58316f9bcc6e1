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
};

}  // namespace pat
