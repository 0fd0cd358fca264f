// LayerNorm fused into the load stage of a GEMM whose weight does not fit the registers of one
// workgroup: C = LN(A) . W, A virtual [.., K] with contiguous rows, K <= 1024, W a row-major [K, N]
// matrix, any N (K and N multiples of 8).  (vt_ln_gemm.hip and vt_ln_gemm_slice.hip keep W in registers for up to
// 128 features; vt_ln_gemm_panel.hip and vt_ln_gemm_ring.hip take most calls of 128 to 512 features in multiples of 64.)
// Bound by HBM at small K (a token's K values are read once and its N outputs written once), by the matrix pipes and
// the reads of W from L2 as K and N grow.
//
// A workgroup takes 64 or 128 rows: they are fetched through the map (16 bytes per lane, LP2 lanes per row,
// one lane evaluates a row's offset for the wave), normalised in registers (fp32, two passes), rounded
// to the operand type and parked in LDS, rows 16 bytes further apart than they are long, so that the
// 16 rows of a fragment read start in different banks (0.9 of the kernel's 2.1 million LDS
// cycles are conflicts all the same, 2 us of a unit's time).  One barrier later every wave works alone: it
// owns a tile of 64 columns and walks K in steps of 32 with W straight from L2 - a lane loads 8
// consecutive k of its 4 columns (128-byte row segments per 16 lanes), transposes the 8x4 block in
// registers (v_perm_b32) and multiplies it with all rows, C^T += W^T . LN(A)^T on
// v_mfma_f32_16x16x32.  Nothing of W is shared between the waves of a workgroup, so staging it in LDS
// would only add traffic and barriers; the rows are what is reused.  Three register sets keep the
// next two K steps in flight while one is multiplied.  A lane ends up with 4 consecutive columns of a
// row; a wave turns 16 rows at a time round in LDS and leaves with whole 128-byte row segments.
// (64 rows x 128 columns per wave spilled; four or six register sets measured no faster than three.)
// 25088 x 264 -> 768, bf16 (51.8 MB, 10.2 GFLOP): 25.6 us; 25088 x 256 -> 768 27 us with inputs cold in every cache (24
// through the rings, which take it), 2295 us on the generic kernel, which evaluates the map for every element of A and W.  What is
// left is latency: rows, statistics and W follow each other inside a workgroup, and only two or three waves per SIMD overlap
// (of the 27 us the matrix pipes of a working unit are busy 5, the vector instructions 7; counters:
// profiles/small_tiles_streamed_ln_split_rowsum.txt).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "vt_gemm_common.h"

using namespace vt;
using namespace vt::gemm;

namespace {

constexpr int WBN = 64;           // columns per wave
constexpr int kMaxWaves = 8;
constexpr int kSets = 3;          // K steps of W in flight or being multiplied

struct WideParams {
  const char* a;
  const char* b;
  char* c;
  AxisMap<5> a_row;
  int64_t ldb;                    // elements between rows of W
  int32_t M, N, K;
  float eps;
  int32_t tiles_per_group;        // column tiles of one workgroup, dealt to its waves in turn
};

// Sum over LP2 = 8, 16, 32 or 64 consecutive lanes, every lane gets the total.
template <int LP2>
__device__ __forceinline__ float row_sum(float v) {
  v = group_sum<LP2 < 16 ? LP2 : 16>(v);
  if (LP2 >= 32) v += __shfl_xor(v, 16, 64);
  if (LP2 >= 64) v += __shfl_xor(v, 32, 64);
  return v;
}

// MB blocks of 16 rows per workgroup; LP2 lanes hold a row, CH chunks of 8 elements each: K <= 8 * LP2 * CH
template <typename T, bool C_F32, int MB, int LP2, int CH>
__global__ void __launch_bounds__(kMaxWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_ln_gemm_wide(const WideParams P) {
  typedef Mma16<T> M_;
  typedef typename M_::vec opvec;
  constexpr int WBM = MB * 16, RPL = WBM / 64;   // rows; rows whose offset a lane evaluates
  constexpr int kPitch = LP2 * CH + 1;           // 16-byte units between rows (at most)
  __shared__ uint4 tile[WBM * kPitch];
  __shared__ uint4 turn[C_F32 ? 1 : kMaxWaves][C_F32 ? 1 : 16 * 8];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n_waves = blockDim.x >> 6;
  const int l16 = lane & 15, lg = lane >> 4;
  const int M = P.M, N = P.N, K = P.K;
  const int steps = (K + 31) >> 5, pitch = steps * 4 + 1;
  const int row0 = blockIdx.x * WBM;
  // this wave's column tiles: tile0, tile0 + n_waves, ... below tile_end (none: it only normalises)
  const int tile0 = blockIdx.y * P.tiles_per_group + wave;
  const int tile_end = min((int)(blockIdx.y + 1) * P.tiles_per_group, (N + WBN - 1) / WBN);

  // ---- W: a cursor over (tile, K step) runs two steps ahead of the multiplication; the first two are
  // requested before anything else.
  // (one wave-uniform base per load plus ONE per-lane offset: the host checks that 24 rows of W < 4 GiB)
  const size_t row_bytes = (size_t)P.ldb * 2;
  const uint32_t w_lane = (uint32_t)(lg * 8 * row_bytes);
  uint32_t w_off = w_lane + (uint32_t)min(tile0 * WBN + l16 * 4, N - 4) * 2;
  int ld_tile = tile0, ld_step = 0;
  uint2 wr[kSets][8];
  auto load_w = [&](auto set) {
    constexpr int S = decltype(set)::value;
    if (ld_tile >= tile_end) return;
    const char* base = P.b + (size_t)(ld_step * 32) * row_bytes;
    if (ld_step * 32 + 32 <= K) {
#pragma unroll
      for (int j = 0; j < 8; ++j) wr[S][j] = *reinterpret_cast<const uint2*>(base + j * row_bytes + w_off);
    } else {
      // K is a multiple of 8: a lane's 8 rows are all there or all past the end
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        wr[S][j] = make_uint2(0, 0);
        if (ld_step * 32 + lg * 8 < K) wr[S][j] = *reinterpret_cast<const uint2*>(base + j * row_bytes + w_off);
      }
    }
    if (++ld_step == steps) {
      ld_step = 0;
      ld_tile += n_waves;
      w_off = w_lane + (uint32_t)min(ld_tile * WBN + l16 * 4, N - 4) * 2;
    }
  };
  typedef std::integral_constant<int, 0> S0;
  typedef std::integral_constant<int, 1> S1;
  typedef std::integral_constant<int, 2> S2;
  load_w(S0{});
  load_w(S1{});

  // ---- stage 1 through the map: lane l evaluates rows l and, with 128 rows, 64 + l; 64 / LP2 rows per pass
  {
    int ro_lo[RPL], ro_hi[RPL];
#pragma unroll
    for (int i = 0; i < RPL; ++i) {
      const uint32_t m = (uint32_t)min(row0 + lane + 64 * i, M - 1);
      const int64_t ro = (P.a_row.tdig >= 0 ? axis_off_table(P.a_row, m) : axis_off(P.a_row, m)) * 2;
      ro_lo[i] = (int)(uint32_t)(uint64_t)ro, ro_hi[i] = (int)(ro >> 32);
    }
    constexpr int RPP = 64 / LP2, NP = WBM / RPP;
    constexpr int U = 2;           // passes whose rows are in flight together
    const int c0 = lane % LP2, r0 = lane / LP2;
    const float k = (float)K, inv_k = 1.0f / k;
    for (int p0 = wave; p0 < NP; p0 += n_waves * U) {
      uint4 raw[U][CH];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = min(p0 + u * n_waves, NP - 1) * RPP + r0;
        const int half = RPL == 1 ? 0 : __builtin_amdgcn_readfirstlane(r >> 6);   // a pass does not straddle row 64
        const uint64_t off = (uint32_t)__shfl(ro_lo[half ? RPL - 1 : 0], r & 63, 64) |
                             ((uint64_t)(uint32_t)__shfl(ro_hi[half ? RPL - 1 : 0], r & 63, 64) << 32);
        const char* rp = P.a + (int64_t)off;
#pragma unroll
        for (int h = 0; h < CH; ++h) {
          raw[u][h] = make_uint4(0, 0, 0, 0);
          if ((c0 + h * LP2) * 8 < K) raw[u][h] = *reinterpret_cast<const uint4*>(rp + (c0 + h * LP2) * 16);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float x[CH][8];
        float s = 0.f;
#pragma unroll
        for (int h = 0; h < CH; ++h) {
          const Vec<T, 8> v = __builtin_bit_cast(Vec<T, 8>, raw[u][h]);
#pragma unroll
          for (int j = 0; j < 8; ++j) x[h][j] = to_float(v.v[j]);
          s += ((x[h][0] + x[h][1]) + (x[h][2] + x[h][3])) + ((x[h][4] + x[h][5]) + (x[h][6] + x[h][7]));
        }
        const float mean = over_k(row_sum<LP2>(s), k, inv_k);
        float q = 0.f;
#pragma unroll
        for (int h = 0; h < CH; ++h) {
          const bool in = (c0 + h * LP2) * 8 < K;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            x[h][j] = in ? x[h][j] - mean : 0.f;
            q += x[h][j] * x[h][j];
          }
        }
        // as in the generic kernel: a subnormal variance (eps = 0) has a finite root, which v_rsq_f32 does not give
        const float rstd = 1.0f / sqrtf(squares_over_k(row_sum<LP2>(q), k, inv_k) + P.eps);
        const int p = p0 + u * n_waves;
        if (p < NP) {
#pragma unroll
          for (int h = 0; h < CH; ++h) {
            Vec<T, 8> o;
#pragma unroll
            for (int j = 0; j < 8; ++j) o.v[j] = from_float<T>(x[h][j] * rstd);
            // chunks past K are zeros (up to the last K step's end)
            if (c0 + h * LP2 < steps * 4) tile[(p * RPP + r0) * pitch + c0 + h * LP2] = __builtin_bit_cast(uint4, o);
          }
        }
      }
    }
  }
  __syncthreads();

  // ---- K steps: nothing shared is written from here on
  f32x4 acc[4][MB];
  int tile_n = tile0, step = 0;
  auto multiply = [&](auto set) {
    constexpr int S = decltype(set)::value;
    opvec af[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) af[mb] = __builtin_bit_cast(opvec, tile[(mb * 16 + l16) * pitch + step * 4 + lg]);
    if (step == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[e][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
      uint32_t w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        w[u] = e < 2 ? __builtin_amdgcn_perm(wr[S][2 * u + 1].x, wr[S][2 * u].x, sel) : __builtin_amdgcn_perm(wr[S][2 * u + 1].y, wr[S][2 * u].y, sel);
      const opvec wop = __builtin_bit_cast(opvec, make_uint4(w[0], w[1], w[2], w[3]));
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[e][mb] = M_::run(wop, af[mb], acc[e][mb]);
    }
    ++step;
  };
  // stage 3: lane holds row mb*16 + l16, columns (lg*4 + r)*4 + e
  auto store_tile = [&]() {
    const int col0 = tile_n * WBN;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      if (C_F32) {
        const int row = row0 + mb * 16 + l16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int col = col0 + (lg * 4 + r) * 4;
          if (row < M && col < N)
            *reinterpret_cast<float4*>(reinterpret_cast<float*>(P.c) + (size_t)row * N + col) =
                make_float4(acc[0][mb][r], acc[1][mb][r], acc[2][mb][r], acc[3][mb][r]);
        }
      } else {
        // 16 rows of 8 chunks of 16 bytes; chunk c of row r at r * 8 + (c ^ (r >> 1 & 7)): two rows
        // lie in the 256 bytes that 16 lanes move at once
        uint4* mine = turn[C_F32 ? 0 : wave];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          Vec<T, 8> o;
#pragma unroll
          for (int e = 0; e < 8; ++e) o.v[e] = from_float<T>(acc[e & 3][mb][2 * h + (e >> 2)]);
          mine[l16 * 8 + ((lg * 2 + h) ^ (l16 >> 1))] = __builtin_bit_cast(uint4, o);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int rr = q * 8 + (lane >> 3), ch = lane & 7;   // 8 lanes per row
          const uint4 v = mine[rr * 8 + (ch ^ (rr >> 1))];
          const int row = row0 + mb * 16 + rr, col = col0 + ch * 8;
          if (row < M && col < N) *reinterpret_cast<uint4*>(P.c + ((size_t)row * N + col) * 2) = v;
        }
      }
    }
    tile_n += n_waves;
    step = 0;
  };
  while (tile_n < tile_end) {
    load_w(S2{});
    multiply(S0{});
    if (step == steps) store_tile();
    if (tile_n >= tile_end) break;
    load_w(S0{});
    multiply(S1{});
    if (step == steps) store_tile();
    if (tile_n >= tile_end) break;
    load_w(S1{});
    multiply(S2{});
    if (step == steps) store_tile();
  }
}

// 128 rows per workgroup halve the reads of W and the rounds, once there are workgroups for most of
// the chip's 256 units (measured, us, 64 / 128 rows: 25088 x 264 -> 768: 43.7 / 25.6, 25088 x 328 -> 1312: 83 / 41,
// 100352 x 72 -> 288: 28.2 / 26.5, but 18432 x 200 -> 200: 10.8 / 11.6 and 1568 x 328 -> 1312: 12.1 / 18.7).
// Waves: four, two workgroups sharing a compute unit, or eight where there is at most one workgroup
// per unit (100352 x 72 -> 288: 26.4 / 30.8 with four / eight, 25088 x 264 -> 768: 36.4 / 25.6).
// Column groups only to reach the units that the rows leave idle: each group normalises its rows
// again (25088 x 264 -> 768 in one / two / four groups: 25.6 / 35.8 / 61; 1568 x 328 -> 1312: 23.5 / 17.2 / 12.8).
template <typename T, bool C_F32>
int launch_wide(const WideParams& P, hipStream_t st) {
  const int tiles = (P.N + WBN - 1) / WBN;
  const bool tall = !C_F32 && P.K <= 512 && P.M >= 192 * 128;
  const int rows = tall ? 128 : 64, blocks = (P.M + rows - 1) / rows;
  const int waves = blocks > (tall ? 512 : 256) ? 4 : 8;
  const int groups = std::max(1, std::min(256 / blocks, (tiles + 1) / 2));
  WideParams Q = P;
  Q.tiles_per_group = (tiles + groups - 1) / groups;
  const dim3 grid((unsigned)blocks, (unsigned)((tiles + Q.tiles_per_group - 1) / Q.tiles_per_group)), block(waves * 64);
#define VT_WIDE(MB, LP2, CH) hipLaunchKernelGGL((k_ln_gemm_wide<T, C_F32, MB, LP2, CH>), grid, block, 0, st, Q)
  if (!C_F32 && tall) {
    if (P.K <= 128) VT_WIDE(C_F32 ? 4 : 8, 8, 2);
    else if (P.K <= 256) VT_WIDE(C_F32 ? 4 : 8, 16, 2);
    else VT_WIDE(C_F32 ? 4 : 8, 32, 2);
  } else {
    if (P.K <= 128) VT_WIDE(4, 8, 2);
    else if (P.K <= 256) VT_WIDE(4, 16, 2);
    else if (P.K <= 512) VT_WIDE(4, 32, 2);
    else VT_WIDE(4, 64, 2);
  }
#undef VT_WIDE
  return check_launch("vt_gemm(layernorm)");
}

}  // namespace

namespace vt {

// One group of vt_gemm with prologue = VT_GEMM_LAYERNORM on the kernel above, or
// VT_ERR_UNSUPPORTED (shapes, maps or alignments it does not take, and every error that the
// generic kernel reports: the caller goes on to that one).
int ln_gemm_wide_launch(const vt_desc& A, const vt_desc& B, void* C, int c_dtype, float eps, hipStream_t st) {
  const char* no = "vt_gemm(layernorm): outside the fused kernels";
  const int n = (int)A.shape.size();
  if (n < 2 || B.shape.size() != 2 || B.shape[0] != A.shape[n - 1]) return fail(VT_ERR_UNSUPPORTED, no);
  const int64_t K = A.shape[n - 1], N = B.shape[1];
  int64_t M = 1;
  for (int i = 0; i < n - 1; ++i) M *= A.shape[i];
  if (M < 1 || K < 8 || K % 8 || K > 1024 || N < 8 || N % 8) return fail(VT_ERR_UNSUPPORTED, no);
  // (the limits of the generic kernel, which took these calls before there was this one)
  if (M > 65535ll * 64 || N > 65535ll * 64 || M * K >= (1ll << 31) || K * N >= (1ll << 31)) return fail(VT_ERR_UNSUPPORTED, no);
  if (A.pieces.size() != 1 || !A.pieces[0].v.lower.empty() || B.pieces.size() != 1 || !B.pieces[0].v.lower.empty())
    return fail(VT_ERR_UNSUPPORTED, no);
  WideParams P;
  memset(&P, 0, sizeof(P));
  const Piece& pa = A.pieces[0];
  const Piece& pb = B.pieces[0];
  AxisMap<3> a_col, b_row, b_col;
  if (make_axis(A, pa, 0, n - 1, &P.a_row, "A rows", true) != VT_OK || make_axis(A, pa, n - 1, n, &a_col, "A columns") != VT_OK ||
      make_axis(B, pb, 0, 1, &b_row, "B rows") != VT_OK || make_axis(B, pb, 1, 2, &b_col, "B columns") != VT_OK)
    return fail(VT_ERR_UNSUPPORTED, no);
  const vt_source& sa = A.sources[pa.src];
  const vt_source& sb = B.sources[pb.src];
  if (!sa.ptr || !sb.ptr) return fail(VT_ERR_UNSUPPORTED, no);
  P.a = static_cast<const char*>(sa.ptr) + pa.v.base * 2;
  P.b = static_cast<const char*>(sb.ptr) + pb.v.base * 2;
  P.c = static_cast<char*>(C);
  P.ldb = b_row.stride[2];
  const bool rows_ok = a_col.nd == 1 && a_col.stride[2] == 1 && (uintptr_t)P.a % 16 == 0 && strides_multiple_of(P.a_row, 8, 0);
  const bool w_ok = b_row.nd == 1 && b_col.nd == 1 && b_col.stride[2] == 1 && P.ldb % 8 == 0 && P.ldb >= 0 && (uintptr_t)P.b % 16 == 0 &&
                    P.ldb * 48 + N * 2 < (1ll << 32);
  if (!rows_ok || !w_ok || (uintptr_t)P.c % 16) return fail(VT_ERR_UNSUPPORTED, no);
  P.M = (int32_t)M;
  P.N = (int32_t)N;
  P.K = (int32_t)K;
  P.eps = eps;
  const bool c32 = c_dtype == VT_F32;
  if (A.dtype == VT_BF16) return c32 ? launch_wide<bf16_t, true>(P, st) : launch_wide<bf16_t, false>(P, st);
  return c32 ? launch_wide<f16_t, true>(P, st) : launch_wide<f16_t, false>(P, st);
}

}  // namespace vt
