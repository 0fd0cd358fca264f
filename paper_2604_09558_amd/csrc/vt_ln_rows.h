// Arguments of the LayerNorm + linear kernels of 128 to 512 features (vt_ln_gemm_ring.hip, vt_ln_gemm_panel.hip), and the
// normalisation of a wave's rows that lie in LDS.  (The ring kernel has the same statements in its own body: called from there, this
// made 1 % of its time, in s_nop between products.)
#pragma once

#include "vt_gemm_common.h"

namespace vt {
namespace gemm {

struct LnParams {
  const char* a;
  const char* b;
  char* c;
  AxisMap<5> a_row;
  int64_t ldb;                    // elements between rows of W
  int32_t M, N, K;
  float eps;
  int32_t tiles_per_group;        // k_ln_gemm_ring: column tiles of one workgroup, dealt to its waves in turn
};

// Sum over LP2 = 16 or 32 consecutive lanes, every lane gets the total.
template <int LP2>
__device__ __forceinline__ float ln_row_sum(float v) {
  v = group_sum<16>(v);
  if (LP2 >= 32) v += __shfl_xor(v, 16, 64);
  return v;
}

// Normalises the rows of a wave: NP passes of 64 / LP2 rows, LP2 lanes to a row, a lane with two chunks of 8 elements, chunk
// lane % LP2 + h LP2 (zeros where a row has ended).  read(pass, h) gives a chunk, write(pass, h, words) takes it rounded to T.
template <typename T, int LP2, int NP, typename Read, typename Write>
__device__ __forceinline__ void ln_rows(int K, float eps, int lane, Read read, Write write) {
  constexpr int CH = 2;
  const int c0 = lane % LP2;
  const float k = (float)K, inv_k = 1.0f / k;
  constexpr int Q = NP < 4 ? NP : 4;               // passes that share a root and a division
#pragma unroll
  for (int p0 = 0; p0 < NP; p0 += Q) {
    float x[Q][CH][8], q[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      if (p0 + i >= NP) continue;
      float s = 0.f;
#pragma unroll
      for (int h = 0; h < CH; ++h) {
        const Vec<T, 8> v = __builtin_bit_cast(Vec<T, 8>, read(p0 + i, h));
#pragma unroll
        for (int j = 0; j < 8; ++j) x[i][h][j] = to_float(v.v[j]);
        s += ((x[i][h][0] + x[i][h][1]) + (x[i][h][2] + x[i][h][3])) + ((x[i][h][4] + x[i][h][5]) + (x[i][h][6] + x[i][h][7]));
      }
      const float mean = over_k(ln_row_sum<LP2>(s), k, inv_k);
      float d2 = 0.f;
#pragma unroll
      for (int h = 0; h < CH; ++h) {
        const bool in = (c0 + h * LP2) * 8 < K;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          x[i][h][j] = in ? x[i][h][j] - mean : 0.f;
          d2 += x[i][h][j] * x[i][h][j];
        }
      }
      q[i] = ln_row_sum<LP2>(d2);
    }
    // One root and one division (some 40 instructions) for the rows of up to four passes: lane 4 n + i of a row takes
    // pass i's, and the four receive the results.  As in the generic kernel, a subnormal variance (eps = 0) has a
    // finite root, which v_rsq_f32 does not give.
    float qs = q[0];
#pragma unroll
    for (int i = 1; i < Q; ++i)
      if (p0 + i < NP) qs = (lane & 3) == i ? q[i] : qs;
    const float rstd = 1.0f / sqrtf(squares_over_k(qs, k, inv_k) + eps);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      if (p0 + i >= NP) continue;
      const float rs = i == 0 ? dpp_move<0x00>(rstd) : i == 1 ? dpp_move<0x55>(rstd) : i == 2 ? dpp_move<0xAA>(rstd) : dpp_move<0xFF>(rstd);
#pragma unroll
      for (int h = 0; h < CH; ++h) {
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = pack2<T>(x[i][h][2 * j] * rs, x[i][h][2 * j + 1] * rs);
        if ((c0 + h * LP2) * 8 < K) write(p0 + i, h, make_uint4(w[0], w[1], w[2], w[3]));
      }
    }
  }
}

}  // namespace gemm
}  // namespace vt
