// Register DFTs and access helpers of the general-length and fixed-length
// kernels (general.hip, transverse.hip).
#pragma once

#include "device.h"

namespace pat {

// Descriptors are read through the constant address space: their fields then
// come by scalar loads, once, whatever the kernel stores in between (through a
// plain pointer they were vector loads, repeated after every barrier).
using CInst = const __attribute__((address_space(4))) Inst;
using CFft = const __attribute__((address_space(4))) GFft;

__device__ __forceinline__ int fdiv(int n, uint32_t m) { return m ? (int)__umulhi((unsigned)n, m) : n; }

// ---------------------------------------------------------------------------
// R-point DFTs in registers, natural order in and out.

template <typename T, int R>
__device__ __forceinline__ void dft_reg(cx<T>* v);

// odd prime, by the symmetric form of bfly_prime with every root a constant
template <typename T, int R>
__device__ __forceinline__ void dft_prime(cx<T>* v) {
  constexpr int H = (R - 1) / 2;
  cx<T> av[H], bv[H];
  const cx<T> x0 = v[0];
  cx<T> s = x0;
#pragma unroll
  for (int r = 1; r <= H; ++r) {
    av[r - 1] = cadd(v[r], v[R - r]);
    bv[r - 1] = csub(v[r], v[R - r]);
    s = cadd(s, av[r - 1]);
  }
  v[0] = s;
#pragma unroll
  for (int d = 1; d <= H; ++d) {
    cx<T> A = x0, B = mk(T(0), T(0));
#pragma unroll
    for (int r = 1; r <= H; ++r) {
      const T c = T(Roots<R>::t.c[(r * d) % R]), sn = T(Roots<R>::t.s[(r * d) % R]);
      A.x += av[r - 1].x * c;
      A.y += av[r - 1].y * c;
      B.x += bv[r - 1].x * sn;
      B.y += bv[r - 1].y * sn;
    }
    v[d] = mk(A.x + B.y, A.y - B.x);
    v[R - d] = mk(A.x - B.y, A.y + B.x);
  }
}

// R = A B with coprime factors (prime-factor map): input n = B n1 + A n2,
// output k with k = k1 mod A, k = k2 mod B; no twiddles
constexpr int crt(int A, int B, int k1, int k2) {
  for (int k = 0; k < A * B; ++k)
    if (k % A == k1 && k % B == k2) return k;
  return 0;
}
template <typename T, int A, int B>
__device__ __forceinline__ void dft_pfa(cx<T>* v) {
  cx<T> t[A][B];
#pragma unroll
  for (int i = 0; i < A; ++i) {
#pragma unroll
    for (int j = 0; j < B; ++j) t[i][j] = v[(B * i + A * j) % (A * B)];
    dft_reg<T, B>(t[i]);
  }
#pragma unroll
  for (int j = 0; j < B; ++j) {
    cx<T> u[A];
#pragma unroll
    for (int i = 0; i < A; ++i) u[i] = t[i][j];
    dft_reg<T, A>(u);
#pragma unroll
    for (int i = 0; i < A; ++i) v[crt(A, B, i, j)] = u[i];
  }
}

// 9 = 3 x 3 with the roots of 9 between the two steps
template <typename T>
__device__ __forceinline__ void dft_9(cx<T>* v) {
  cx<T> t[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int j = 0; j < 3; ++j) t[i][j] = v[3 * j + i];
    dft_reg<T, 3>(t[i]);
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    cx<T> u[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const T c = T(Roots<9>::t.c[i * j]), s = T(Roots<9>::t.s[i * j]);
      u[i] = mk(t[i][j].x * c + t[i][j].y * s, t[i][j].y * c - t[i][j].x * s);
    }
    dft_reg<T, 3>(u);
#pragma unroll
    for (int i = 0; i < 3; ++i) v[3 * i + j] = u[i];
  }
}

template <typename T, int R>
__device__ __forceinline__ void dft_reg(cx<T>* v) {
  if constexpr (R == 1) {
  } else if constexpr (R == 2 || R == 4 || R == 8 || R == 16) dft_pow2<T, R>(v);
  else if constexpr (R == 9) dft_9<T>(v);
  else if constexpr (R == 6) dft_pfa<T, 2, 3>(v);
  else if constexpr (R == 10) dft_pfa<T, 2, 5>(v);
  else if constexpr (R == 12) dft_pfa<T, 4, 3>(v);
  else if constexpr (R == 14) dft_pfa<T, 2, 7>(v);
  else if constexpr (R == 15) dft_pfa<T, 3, 5>(v);
  else if constexpr (R == 18) dft_pfa<T, 2, 9>(v);
  else if constexpr (R == 20) dft_pfa<T, 4, 5>(v);
  else if constexpr (R == 21) dft_pfa<T, 3, 7>(v);
  else if constexpr (R == 22) dft_pfa<T, 2, 11>(v);
  else dft_prime<T, R>(v);
}

// The R outputs of a butterfly handed to emit(k, X_k): the larger primes one
// output pair at a time (their R outputs beside the R combined inputs would
// not fit in registers), the others after the whole transform.
template <typename T, int R, typename Emit>
__device__ __forceinline__ void dft_emit(cx<T>* v, Emit emit) {
  if constexpr (R == 13 || R == 17 || R == 19 || R == 23) {
    constexpr int H = (R - 1) / 2;
    cx<T> s = v[0];
#pragma unroll
    for (int r = 1; r <= H; ++r) {
      const cx<T> p = cadd(v[r], v[R - r]);
      v[R - r] = csub(v[r], v[R - r]);
      v[r] = p;
      s = cadd(s, p);
    }
    emit(0, s);
#pragma unroll
    for (int d = 1; d <= H; ++d) {
      cx<T> A = v[0], B = mk(T(0), T(0));
#pragma unroll
      for (int r = 1; r <= H; ++r) {
        const T c = T(Roots<R>::t.c[(r * d) % R]), sn = T(Roots<R>::t.s[(r * d) % R]);
        A.x += v[r].x * c;
        A.y += v[r].y * c;
        B.x += v[R - r].x * sn;
        B.y += v[R - r].y * sn;
      }
      emit(d, mk(A.x + B.y, A.y - B.x));
      emit(R - d, mk(A.x - B.y, A.y + B.x));
    }
  } else {
    dft_reg<T, R>(v);
#pragma unroll
    for (int d = 0; d < R; ++d) emit(d, v[d]);
  }
}

// f.operator()<R>() for the run-time radix r of a twiddled stage (the set
// plan_general takes r0 and r1 from) and of a last stage
template <int R>
struct RadixTag {
  static constexpr int v = R;
};
#define PAT_CASE(R) \
  case R: f(RadixTag<R>{}); break;
template <typename F>
__device__ __forceinline__ void with_tw_radix(int r, F f) {
  switch (r) {
    PAT_CASE(1) PAT_CASE(2) PAT_CASE(3) PAT_CASE(4) PAT_CASE(5) PAT_CASE(6) PAT_CASE(7) PAT_CASE(8) PAT_CASE(9)
    PAT_CASE(10) PAT_CASE(11) PAT_CASE(12) PAT_CASE(13) PAT_CASE(16)
    default: break;
  }
}
template <typename F>
__device__ __forceinline__ void with_last_radix(int r, F f) {
  switch (r) {
    PAT_CASE(2) PAT_CASE(3) PAT_CASE(4) PAT_CASE(5) PAT_CASE(6) PAT_CASE(7) PAT_CASE(8) PAT_CASE(9) PAT_CASE(10)
    PAT_CASE(11) PAT_CASE(12) PAT_CASE(13) PAT_CASE(14) PAT_CASE(15) PAT_CASE(16) PAT_CASE(17) PAT_CASE(18)
    PAT_CASE(19) PAT_CASE(20) PAT_CASE(21) PAT_CASE(22) PAT_CASE(23)
    default: break;
  }
}

// element at a 32-bit byte offset from a workgroup-uniform base
template <typename V>
__device__ __forceinline__ V* at_off(V* base, uint32_t bytes) {
  using C = std::conditional_t<std::is_const_v<V>, const char, char>;
  return reinterpret_cast<V*>(reinterpret_cast<C*>(base) + bytes);
}

template <typename T, bool NT>
__device__ __forceinline__ cx<T> ld_cx(const cx<T>* p) {
  if constexpr (NT && sizeof(T) == 4) {
    typedef float v2f __attribute__((ext_vector_type(2)));
    const v2f v = __builtin_nontemporal_load(reinterpret_cast<const v2f*>(p));
    return mk(v.x, v.y);
  } else {
    return *p;
  }
}
template <typename T, bool NT>
__device__ __forceinline__ void st_cx(cx<T>* p, cx<T> v) {
  if constexpr (NT && sizeof(T) == 4) {
    typedef float v2f __attribute__((ext_vector_type(2)));
    const v2f u = {v.x, v.y};
    __builtin_nontemporal_store(u, reinterpret_cast<v2f*>(p));
  } else {
    *p = v;
  }
}

// Item of slot i: workgroups go to the eight XCDs in turn, so slot i runs on
// XCD i mod 8; each XCD gets one contiguous run of items, whose neighbours (tiles
// that share cache lines where a row is no multiple of a line) then meet in
// its L2.
__device__ __forceinline__ int xcd_item(int i, int total) {
  const int q = total >> 3, r = total & 7, x = i & 7;
  return x * q + min(x, r) + (i >> 3);
}

}  // namespace pat
