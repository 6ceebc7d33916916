// Shared pieces of the pair-block kernels (pntile.hip: proton-neutron part; flytile.hip:
// single-species two-body part): the matrix-core instruction per precision and its output layout,
// the sign flip, the work-item order and the buffer accesses.
#pragma once
#include "internal.h"

namespace trbl {
namespace tiles {

// Per precision: the matrix-core accumulator, the instruction, and the row of its output a lane
// register holds (measured on gfx950: FP64 D[l / 16 + 4 v][l % 16], FP32 D[4 (l / 16) + v][l % 16]).
template <class T>
struct Mfma;
template <>
struct Mfma<double> {
  typedef double acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc run(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int kq, int v) { return kq + 4 * v; }
};
template <>
struct Mfma<float> {
  typedef float acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc run(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int kq, int v) { return 4 * kq + v; }
};

constexpr int PN_TPB = 256;       // most core pairs of one work item
constexpr int PN_MAXPAIR = 64;    // widest pair block (one ballot)

// work item -> position: consecutive items (one proton core) go to one XCD
__device__ __forceinline__ int pn_xcd_item(int bid, int n) {
  const int per = (n + 7) / 8;
  return (bid % 8) * per + bid / 8;
}

__device__ __forceinline__ double flip_if(double x, unsigned s) {
  return __hiloint2double(__double2hiint(x) ^ (int)(s << 31), __double2loint(x));
}
__device__ __forceinline__ float flip_if(float x, unsigned s) { return __int_as_float(__float_as_int(x) ^ (int)(s << 31)); }

// CT adjacent columns of one lane: CT column tiles interleave their columns (lane c of a 16-lane
// group holds columns CT c .. CT c + CT - 1), so a lane's share of a row is one load or store.
// In memory a lane's columns start at any column (`stored`): the last lane of a ragged row overlaps its neighbour.
template <class T, int CT>
struct Cols {
  typedef T type __attribute__((ext_vector_type(CT)));
  typedef T stored __attribute__((ext_vector_type(CT), aligned(sizeof(T))));
};
template <class T>
struct Cols<T, 1> {
  typedef T type;
  typedef T stored;
};

// A byte offset beyond every V and slot offset: buffer loads return 0 there, stores write nothing.
constexpr unsigned NO_ROW = 0xFFFF0000u;

// Buffer accesses. Slot rows of 64 bytes or more are streamed past the caches (NT): they are read back by
// a later kernel; narrower rows are left for the L2 to merge into whole lines.
#if defined(__HIP_DEVICE_COMPILE__)  // buffer descriptors exist only in the device pass
template <int BYTES>
struct Buf;
template <>
struct Buf<4> {
  typedef unsigned raw;
  static __device__ __forceinline__ raw load(__amdgpu_buffer_rsrc_t r, unsigned o) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0);
  }
  template <bool NT>
  static __device__ __forceinline__ void store(raw v, __amdgpu_buffer_rsrc_t r, unsigned o) {
    __builtin_amdgcn_raw_buffer_store_b32(v, r, o, 0, NT ? 2 : 0);
  }
};
template <>
struct Buf<8> {
  typedef unsigned raw __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ raw load(__amdgpu_buffer_rsrc_t r, unsigned o) {
    return __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0);
  }
  template <bool NT>
  static __device__ __forceinline__ void store(raw v, __amdgpu_buffer_rsrc_t r, unsigned o) {
    __builtin_amdgcn_raw_buffer_store_b64(v, r, o, 0, NT ? 2 : 0);
  }
};
template <>
struct Buf<16> {
  typedef unsigned raw __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ raw load(__amdgpu_buffer_rsrc_t r, unsigned o) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0);
  }
  template <bool NT>
  static __device__ __forceinline__ void store(raw v, __amdgpu_buffer_rsrc_t r, unsigned o) {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, o, 0, NT ? 2 : 0);
  }
};
#endif

inline int64_t binom(int n, int k) {
  if (k < 0 || k > n) return 0;
  long double r = 1.0L;
  for (int i = 0; i < k; i++) r = r * (n - i) / (i + 1);
  return (int64_t)(r + 0.5L);
}

}  // namespace tiles
}  // namespace trbl
