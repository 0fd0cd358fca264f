// Pieces shared by the GEMM consumers: axis maps (the separable form row_offset(m) +
// col_offset(k) of a 2-D operand's index map), their device evaluators, MFMA wrappers.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "vt_device.h"
#include "vt_numeric.h"

namespace vt {
namespace gemm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void* lptr_t;

template <int ND>
struct AxisMap {
  FastDiv radix[ND];        // outer -> inner
  int64_t stride[ND];       // elements
  const int32_t* table;     // digit `tdig` is looked up in this table first (index_select), or NULL
  int32_t nd, tdig;
};

// Offset contributed by index v along an axis.  Unused digits are padded on the host with
// radix 1 / stride 0 (in the outer slots), so the walk is branch-free.
template <int ND>
__device__ __forceinline__ int64_t axis_off(const AxisMap<ND>& a, uint32_t v) {
  int64_t off = 0;
#pragma unroll
  for (int d = ND - 1; d >= 0; --d) {
    uint32_t r;
    if (d > 0) {
      uint32_t q = fdiv(v, a.radix[d]);
      r = v - q * a.radix[d].d;
      v = q;
    } else {
      r = v;
    }
    off += (int64_t)r * a.stride[d];
  }
  return off;
}

// The same with an index table on digit a.tdig (index_select): only the row axis of A can
// carry one, and it is evaluated once per thread before the K loop.
template <int ND>
__device__ __forceinline__ int64_t axis_off_table(const AxisMap<ND>& a, uint32_t v) {
  int64_t off = 0;
  uint32_t rt = 0;
  int64_t st = 0;
#pragma unroll
  for (int d = ND - 1; d >= 0; --d) {
    uint32_t r;
    if (d > 0) {
      uint32_t q = fdiv(v, a.radix[d]);
      r = v - q * a.radix[d].d;
      v = q;
    } else {
      r = v;
    }
    const bool is_t = d == a.tdig;
    rt = is_t ? r : rt;
    st = is_t ? a.stride[d] : st;
    off += is_t ? 0 : (int64_t)r * a.stride[d];
  }
  return off + (int64_t)a.table[rt] * st;
}

__device__ __forceinline__ uint32_t word(const uint4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

// x / k: the product with the reciprocal and what it left over (a division is ten instructions).
__device__ __forceinline__ float over_k(float x, float k, float inv_k) {
  const float d = x * inv_k;
  return fmaf(fmaf(-d, k, x), inv_k, d);
}
// The same for a sum of squares: one past fp32's range stays infinite (nothing is left over; inf - inf is not a number),
// so that its reciprocal root is zero, as with a division.
__device__ __forceinline__ float squares_over_k(float q, float k, float inv_k) {
  return q < __builtin_inff() ? over_k(q, k, inv_k) : q;
}

// 16 bytes per lane straight from global memory into LDS: lane l's, from base + off, land at LDS byte dst + 16 l.  (M0 holds
// the destination; it is saved and put back.)  Written as assembly so that the request stays unknown to the compiler, which
// would otherwise order every later LDS access of the kernel behind it; the waits for these requests are written by hand.
__device__ __forceinline__ void request(uint32_t off, const char* base, uint32_t dst) {
  uint32_t m0_saved;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_nop 0\n\ts_mov_b32 m0, %0"
               : "=&s"(m0_saved) : "v"(off), "s"(base), "s"(dst) : "memory");
}

// The same from a lane's own address.
__device__ __forceinline__ void request_far(const char* from, uint32_t dst) {
  uint32_t m0_saved;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_nop 0\n\ts_mov_b32 m0, %0"
               : "=&s"(m0_saved) : "v"(from), "s"(dst) : "memory");
}

// two results that lie side by side
template <typename T>
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  if constexpr (std::is_same<T, bf16_t>::value) {
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2));
  } else {
    Vec<T, 2> v;
    v.v[0] = from_float<T>(a), v.v[1] = from_float<T>(b);
    return __builtin_bit_cast(uint32_t, v);
  }
}

// the matrix cores: 32 x 32 blocks, 16 of K; 16 x 16 blocks, 32 of K
template <typename T>
struct Mma;
template <>
struct Mma<bf16_t> {
  typedef bf16x8 vec;
  static __device__ __forceinline__ f32x16 run(vec a, vec b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mma<f16_t> {
  typedef f16x8 vec;
  static __device__ __forceinline__ f32x16 run(vec a, vec b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
};

template <typename T>
struct Mma16;
template <>
struct Mma16<bf16_t> {
  typedef bf16x8 vec;
  static __device__ __forceinline__ f32x4 run(vec a, vec b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};
template <>
struct Mma16<f16_t> {
  typedef f16x8 vec;
  static __device__ __forceinline__ f32x4 run(vec a, vec b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};

// ---------------------------------------------------------------- host: descriptor -> axis maps
// Concatenates the digit groups of dims [d0, d1) of a single-piece, single-stage descriptor.
template <int ND>
int make_axis(const vt_desc& d, const Piece& p, int d0, int d1, AxisMap<ND>* out, const char* what, bool allow_table = false) {
  memset(out, 0, sizeof(*out));
  out->tdig = -1;
  // neighbours that form one dense digit are merged
  Digit m[ND + 1];
  int n = 0;
  for (int i = d0; i < d1; ++i)
    for (const Digit& g : p.v.groups[i]) {
      if (n > 0 && m[n - 1].table < 0 && g.table < 0 && m[n - 1].stride == g.stride * g.radix) {
        m[n - 1].radix *= g.radix;
        m[n - 1].stride = g.stride;
      } else if (n <= ND) {
        m[n++] = g;
      }
    }
  if (n > ND) return fail(VT_ERR_UNSUPPORTED, std::string(what) + ": too many index digits for the GEMM loader");
  out->nd = n;
  for (int i = 0; i < ND; ++i) {        // padding: digits that are always 0
    out->radix[i] = make_fastdiv(1);
    out->stride[i] = 0;
  }
  // real digits occupy the innermost slots so that slot 0 (which takes what is left of the
  // index without a division) is either the outermost real digit or padding over a zero
  const int shift = ND - n;
  for (int i0 = 0; i0 < n; ++i0) {
    const int i = i0 + shift;
    const Digit& mi = m[i0];
    if (mi.radix >= (1ll << 31)) return fail(VT_ERR_UNSUPPORTED, std::string(what) + ": extent too large");
    out->radix[i] = make_fastdiv((uint32_t)mi.radix);
    out->stride[i] = mi.stride;
    if (mi.table >= 0) {
      if (!allow_table) return fail(VT_ERR_UNSUPPORTED, std::string(what) + ": index_select is only supported on the rows of A");
      if (out->table) return fail(VT_ERR_UNSUPPORTED, std::string(what) + ": two index tables on one axis");
      const Table& t = d.tables[mi.table];
      if (!t.dev) return fail(VT_ERR_INVALID_ARG, std::string(what) + ": index table without a device pointer");
      out->table = t.dev + mi.table_off;
      out->tdig = i;
    }
  }
  return VT_OK;
}

// Rows of N 16-bit results in pieces of 64 columns: streaming stores, unless rows are not whole 64-byte units and C is larger
// than what the L2 caches (8 x 4 MB) keep of it: every unit at a piece's end is then written twice, half filled.  LayerNorm + linear,
// plain : streaming over 79 such shapes, 0.97 up to 20 MB (0.93 to 1.10), 0.92 from there to 32 MB, 0.70 above (us: 10076 x 256 ->
// 1304 17.9 / 20.7, 31074 x 128 -> 2480 41.1 / 83.6, 86546 x 128 -> 3496 131 / 300); over 51 of whole units 1.06 up to 60 MB.
inline bool streaming_rows(int64_t M, int64_t N) { return N % 32 == 0 || M * N * 2 < (20ll << 20); }

// Elements of its source that a piece with one stage can reach, counted from the piece's base: the farthest one that its
// digits name (a source's rows may lie apart; the entries of a table over a Concat count from the first of its
// inputs), with a table the whole of a dense source at least.
inline int64_t reach(const vt_desc& d, const Piece& p) {
  int64_t last = 0, all = 0;
  for (const auto& group : p.v.groups)
    for (const Digit& g : group) {
      last += (g.table >= 0 ? g.table_max : g.radix - 1) * g.stride;
      if (g.table >= 0) all = 1;
    }
  const vt_source& s = d.sources[p.src];
  for (int i = 0; i < s.ndim; ++i) all *= s.shape[i];
  return std::max(last + 1, all);
}
constexpr int64_t kReach32 = 1ll << 31;   // of 16-bit elements: their byte offsets take 32 bits

template <int ND>
bool strides_multiple_of(const AxisMap<ND>& a, int64_t q, int skip_inner) {
  for (int i = 0; i < ND - skip_inner; ++i)
    if (a.stride[i] % q) return false;
  return true;
}

}  // namespace gemm
}  // namespace vt
