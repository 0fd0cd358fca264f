// LayerNorm fused into the load stage of a GEMM, many rows, weight held in registers a slice of columns at a time:
// C = LN(A) . W, A virtual [.., K] with contiguous rows, K = 64, 96 or 128, W a row-major [K, N] matrix.
// (vt_ln_gemm.hip holds all of W, for K = 64 / 128 and N <= 384; vt_ln_gemm_wide.hip streams W past every block of rows.)
// Bound by HBM and, close behind, by the vector instructions of LayerNorm: ten per element in the first version,
// 12 of 29 us (100352 x 96 -> 288).  Now five and a half: packed conversions, one root and division for several rows.
//
// A persistent workgroup of 8 waves owns up to 512 columns and walks over blocks of 64 rows; a wave owns one or two
// tiles of 64 columns and 32 of the rows.  Its share of W stays in registers as operands of v_mfma_f32_16x16x32 (a
// lane loads 8 consecutive k of its 4 columns and transposes the 8x4 block with v_perm_b32).  Rows go through three
// LDS tiles in place: arriving (global_load_lds_dwordx4, requested two blocks ahead, already swizzled: the lane that
// lands at position p of row r asks for chunk p ^ key(r)), normalised by the lanes that requested them (fp32, two
// passes, rounded to the operand type), multiplied.  One barrier per block.  Outputs leave as streaming stores of
// 128-byte row segments.
// Measured (bf16, us, streamed weight -> this; in the caches / in HBM): 100352 x 96 -> 288 27.0 / 31.9 -> 22.0 / 22.0,
// 100352 x 96 -> 96 18.8 / 22.2 -> 13.9 / 14.0, 100352 x 128 -> 512 37.8 / 40.8 -> 30.3 / 28.9, 50176 x 96 -> 288 16.9 /
// 18.9 -> 12.8 / 13.4.  (K = 256 was measured too, slices of 256 columns: 25 us against 22 for 25088 x 256 -> 768; loading
// 128 KB of W costs 4 us and every slice normalises all rows again.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "vt_gemm_common.h"

using namespace vt;
using namespace vt::gemm;

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int SBM = 64;           // rows per block
constexpr int kThreads = 512;
constexpr int kSliceCols = 512;

struct SliceParams {
  const char* a;
  const char* b;
  char* c;
  AxisMap<5> a_row;
  int64_t ldb;                    // elements between rows of W
  int32_t M, N;
  float eps;
  int32_t n_slices, slice_cols;   // slice_cols: a multiple of 64
  int32_t groups, n_blocks;       // workgroups per slice; blocks of SBM rows: group g takes blocks g, g + groups, ..
  int32_t stream;                 // 16-bit results leave as streaming stores
};

// Sum over LPR = 8, 16 or 32 consecutive lanes, every lane gets the total.
template <int LPR>
__device__ __forceinline__ float row_sum(float v) {
  return group_sum<LPR>(v);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <typename T, bool C_F32, int KS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_ln_gemm_slice(const SliceParams P) {
  typedef Mma16<T> M_;
  typedef typename M_::vec opvec;
  constexpr int K = KS * 32, kChunks = KS * 4;       // 16-byte chunks per row
  constexpr int LPR = kChunks <= 8 ? 8 : 16;         // lanes (and LDS units) per row
  constexpr int RPP = kThreads / LPR, PASSES = SBM / RPP, RW = 64 / LPR;
  constexpr int kTileUnits = SBM * LPR;
  constexpr int MB = 2, CT = 2;                      // blocks of 16 rows; tiles of 64 columns
  static_assert(RW * PASSES == 8, "a wave stages 8 rows per block");
  __shared__ __attribute__((aligned(1024))) uint4 tiles[3 * kTileUnits];
  __shared__ uint4 turn[C_F32 ? 1 : 8][C_F32 ? 1 : 16 * 8];

  // workgroups of one group of rows, a slice each, are on one compute die: their rows meet in its L2
  const int j = blockIdx.x >> 3;
  const int slice = j % P.n_slices, group = j / P.n_slices * 8 + (blockIdx.x & 7);
  const int n_it = (P.n_blocks - group + P.groups - 1) / P.groups;
  if (group >= P.groups || n_it <= 0) return;

  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  const int wc = wave & 3, wr = wave >> 2;
  const int M = P.M, N = P.N;
  // this wave's tiles of 64 columns: wc and wc + 4 of the slice (none: it stages and normalises only)
  const int slice0 = slice * P.slice_cols, slice_end = min(slice0 + P.slice_cols, N);
  const int col0 = slice0 + wc * 64;
  const int n_ct = slice_end <= col0 ? 0 : slice_end <= col0 + 256 ? 1 : 2;

  // ---- stage 1 through the map: a wave stages 8 rows of every block; their offsets are evaluated for 8 blocks at
  // a time (lane: block lane / 8 of the batch, row lane % 8) and handed to the lanes that load them
  auto key = [](int r) { return LPR == 8 ? r >> 1 & 7 : r & 15; };
  const int a_c = t % LPR, a_r0 = t / LPR;
  const int ev_row = wave * RW + (lane & 7) % RW + RPP * ((lane & 7) / RW);
  uint32_t ro32 = 0;                                  // byte offset of this lane's row (the host checks that A spans < 4 GiB)
  auto eval_rows = [&](int it0) {
    const int blk = min(it0 + (lane >> 3), n_it - 1) * P.groups + group;    // past the last block: it again, not used
    const uint32_t m = (uint32_t)min(blk * SBM + ev_row, M - 1);
    ro32 = (uint32_t)((P.a_row.tdig >= 0 ? axis_off_table(P.a_row, m) : axis_off(P.a_row, m)) * 2);
  };
  auto load_rows = [&](int jb, int slot) {            // block jb of the evaluated batch -> tile `slot`
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      const uint32_t o = (uint32_t)__shfl((int)ro32, jb * 8 + i * RW + lane / LPR, 64);
      const int c = a_c ^ key(a_r0 + RPP * i);
      const uint32_t dst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lptr_t)&tiles[slot * kTileUnits + (wave * RW + RPP * i) * LPR]);
      if (kChunks == LPR || c < kChunks)              // (some lane of a wave always has a chunk: the requests of a step can be counted)
        request(o + c * 16, P.a, dst);
    }
  };
  eval_rows(0);
  load_rows(0, 0);
  load_rows(1, 1);

  // ---- this wave's share of W: operand e of a k32 step holds columns col0 + l16 * 4 + e
  opvec wf[CT][KS][4];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    if (ct >= n_ct) continue;
    const size_t row_bytes = (size_t)P.ldb * 2;
    const uint32_t w_off = (uint32_t)(lg * 8 * row_bytes) + (uint32_t)min(col0 + ct * 256 + l16 * 4, N - 4) * 2;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint2 w[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] = *reinterpret_cast<const uint2*>(P.b + (size_t)(ks * 32 + i) * row_bytes + w_off);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
        uint32_t o[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          o[u] = e < 2 ? __builtin_amdgcn_perm(w[2 * u + 1].x, w[2 * u].x, sel) : __builtin_amdgcn_perm(w[2 * u + 1].y, w[2 * u].y, sel);
        wf[ct][ks][e] = __builtin_bit_cast(opvec, make_uint4(o[0], o[1], o[2], o[3]));
      }
    }
  }

  // ---- LayerNorm in place of the rows that landed in tile `slot`: a lane reads back the 16 bytes of its own request
  constexpr float k = (float)K, inv_k = 1.0f / k;
  auto norm_tile = [&](int slot) {
    uint4* mine = &tiles[slot * kTileUnits + wave * RW * LPR + lane];
    float x[PASSES][8], q[PASSES];
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      const bool in = kChunks == LPR || (a_c ^ key(a_r0 + RPP * i)) < kChunks;
      const Vec<T, 8> v = __builtin_bit_cast(Vec<T, 8>, mine[i * RPP * LPR]);
#pragma unroll
      for (int e = 0; e < 8; ++e) x[i][e] = to_float(v.v[e]);
      const float s = ((x[i][0] + x[i][1]) + (x[i][2] + x[i][3])) + ((x[i][4] + x[i][5]) + (x[i][6] + x[i][7]));
      const float mean = over_k(row_sum<LPR>(in ? s : 0.f), k, inv_k);
      float d2 = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        x[i][e] -= mean;
        d2 += x[i][e] * x[i][e];
      }
      q[i] = row_sum<LPR>(in ? d2 : 0.f);
    }
    // One root and one division for the rows of all passes (some 40 instructions): lane 4 n + i of a row takes pass i's,
    // and every lane of the four receives the results.  As in the generic kernel, a subnormal variance (eps = 0) has a
    // finite root, which v_rsq_f32 does not give.
    float qs = q[0];
#pragma unroll
    for (int i = 1; i < PASSES; ++i) qs = (lane & (PASSES - 1)) == i ? q[i] : qs;
    const float rstd = 1.0f / sqrtf(squares_over_k(qs, k, inv_k) + P.eps);
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      const bool in = kChunks == LPR || (a_c ^ key(a_r0 + RPP * i)) < kChunks;
      const float r = PASSES == 1 ? rstd : i == 0 ? dpp_move<0x00>(rstd) : i == 1 ? dpp_move<0x55>(rstd) : i == 2 ? dpp_move<0xAA>(rstd) : dpp_move<0xFF>(rstd);
      uint32_t o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = pack2<T>(x[i][2 * e] * r, x[i][2 * e + 1] * r);
      if (in) mine[i * RPP * LPR] = make_uint4(o[0], o[1], o[2], o[3]);
    }
  };

  // fragment addresses: chunk 4 ks + lg of row r lies at position (4 ks + lg) ^ key(r)
  const int f_row = wr * 32 + l16;
  int f_unit[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) f_unit[ks] = f_row * LPR + ((ks * 4 + lg) ^ key(f_row));

  constexpr int kStores = C_F32 ? MB * 4 : MB * 2;
  auto product = [&](int it, int slot, auto tile_of_wave) {
    constexpr int ct = decltype(tile_of_wave)::value;
    const int col_ct = col0 + ct * 256;
    const uint4* tile = tiles + slot * kTileUnits;
    f32x4 acc[4][MB];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[e][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      opvec af[MB];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) af[mb] = __builtin_bit_cast(opvec, tile[f_unit[ks] + mb * 16 * LPR]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[e][mb] = M_::run(wf[ct][ks][e], af[mb], acc[e][mb]);
    }
    // ---- stage 3: a lane holds row mb*16 + l16, columns (lg*4 + r)*4 + e.  The buffer descriptor ends with the block's
    // last row and columns past N get an offset outside of it: no store is conditional, the waits count on it.
    const int row0 = (it * P.groups + group) * SBM;
    const int rows = min(SBM, M - row0);
    constexpr int ES = C_F32 ? 4 : 2;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(P.c + (size_t)row0 * (size_t)N * ES, 0, rows * N * ES, 0x00020000);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int r0 = wr * 32 + mb * 16;
      if constexpr (C_F32) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int col = col_ct + (lg * 4 + r) * 4;
          const uint32_t off = col < N ? (uint32_t)((r0 + l16) * N + col) * 4u : 0x80000000u;
          const u32x4 v = __builtin_bit_cast(u32x4, make_float4(acc[0][mb][r], acc[1][mb][r], acc[2][mb][r], acc[3][mb][r]));
          __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, (int)off, 0, 0);
        }
      } else {
        // 16 rows of 8 chunks of 16 bytes; chunk c of row r at r * 8 + (c ^ (r >> 1 & 7))
        uint4* mine = turn[C_F32 ? 0 : wave];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          Vec<T, 8> o;
#pragma unroll
          for (int e = 0; e < 8; ++e) o.v[e] = from_float<T>(acc[e & 3][mb][2 * h + (e >> 2)]);
          mine[l16 * 8 + ((lg * 2 + h) ^ (l16 >> 1))] = __builtin_bit_cast(uint4, o);
        }
        u32x4 v[2];
        uint32_t off[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int rr = q * 8 + (lane >> 3), ch = lane & 7;   // 8 lanes per row of 64 columns
          v[q] = __builtin_bit_cast(u32x4, mine[rr * 8 + (ch ^ (rr >> 1))]);
          const int col = col_ct + ch * 8;
          off[q] = col < N ? (uint32_t)((r0 + rr) * N + col) * 2u : 0x80000000u;
        }
        if (P.stream) {                                // whole lines, not read again here
          __builtin_amdgcn_raw_buffer_store_b128(v[0], rsrc, (int)off[0], 0, 2);
          __builtin_amdgcn_raw_buffer_store_b128(v[1], rsrc, (int)off[1], 0, 2);
        } else {
          __builtin_amdgcn_raw_buffer_store_b128(v[0], rsrc, (int)off[0], 0, 0);
          __builtin_amdgcn_raw_buffer_store_b128(v[1], rsrc, (int)off[1], 0, 0);
        }
      }
    }
  };

  wait_vmcnt<0>();
  norm_tile(0);
  int slot = 0;
  for (int it = 0; it < n_it; ++it) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // tile `slot` is normalised, that of block it - 1 is free
    {
      const int jb = (it + 2) & 7;
      if (jb == 0) eval_rows(it + 2);
      load_rows(jb, slot == 0 ? 2 : slot - 1);
    }
    const int next = slot == 2 ? 0 : slot + 1;
    // The rows requested one step ago: behind them are this step's requests and the stores of one step or two.  The waves of a SIMD
    // (wave and wave + 4) take product and LayerNorm in opposite order.
    if (wave & 4) {
      if (n_ct == 2) wait_vmcnt<2 * kStores + PASSES>();
      else if (n_ct == 1) wait_vmcnt<kStores + PASSES>();
      else wait_vmcnt<PASSES>();
      norm_tile(next);
    }
    if (n_ct > 0) product(it, slot, std::integral_constant<int, 0>{});
    if (n_ct > 1) product(it, slot, std::integral_constant<int, 1>{});
    if (!(wave & 4)) {
      if (n_ct == 2) wait_vmcnt<4 * kStores + PASSES>();
      else if (n_ct == 1) wait_vmcnt<2 * kStores + PASSES>();
      else wait_vmcnt<PASSES>();
      norm_tile(next);
    }
    slot = next;
  }
  wait_vmcnt<0>();                                    // requests past the last block still target this workgroup's LDS
}

template <typename T, bool C_F32>
int launch_slice(const SliceParams& P, int ks, hipStream_t st) {
  const dim3 grid((unsigned)(P.groups * P.n_slices));   // (groups are a multiple of 8)
#define VT_SLICE(KS)                                                                              \
  if (ks == KS) {                                                                                 \
    hipLaunchKernelGGL((k_ln_gemm_slice<T, C_F32, KS>), grid, dim3(kThreads), 0, st, P);          \
    return check_launch("vt_gemm(layernorm)");                                                    \
  }
  VT_SLICE(2) VT_SLICE(3) VT_SLICE(4)
#undef VT_SLICE
  return fail(VT_ERR_UNSUPPORTED, "vt_gemm(layernorm): outside the fused kernels");
}

}  // namespace

namespace vt {

// One group of vt_gemm with prologue = VT_GEMM_LAYERNORM on the kernel above, or VT_ERR_UNSUPPORTED (shapes, maps or
// alignments it does not take, fewer rows than it is the better kernel for, and every error that the generic kernel
// reports).
int ln_gemm_slice_launch(const vt_desc& A, const vt_desc& B, void* C, int c_dtype, float eps, hipStream_t st) {
  const char* no = "vt_gemm(layernorm): outside the fused kernels";
  const int n = (int)A.shape.size();
  if (n < 2 || B.shape.size() != 2 || B.shape[0] != A.shape[n - 1]) return fail(VT_ERR_UNSUPPORTED, no);
  const int64_t K = A.shape[n - 1], N = B.shape[1];
  int64_t M = 1;
  for (int i = 0; i < n - 1; ++i) M *= A.shape[i];
  if (M < 1 || K % 32 || K < 64 || K > 128 || N < 8 || N % 8) return fail(VT_ERR_UNSUPPORTED, no);
  const int ks = (int)(K / 32);
  // (the limits of the generic kernel, which took these calls before there was this one)
  if (M > 65535ll * 64 || N > 65535ll * 64 || M * K >= (1ll << 31) || K * N >= (1ll << 31)) return fail(VT_ERR_UNSUPPORTED, no);
  if (A.pieces.size() != 1 || !A.pieces[0].v.lower.empty() || B.pieces.size() != 1 || !B.pieces[0].v.lower.empty())
    return fail(VT_ERR_UNSUPPORTED, no);
  SliceParams P;
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
  if (reach(A, pa) > kReach32) return fail(VT_ERR_UNSUPPORTED, no);   // a row's byte offset is 32 bits
  P.M = (int32_t)M;
  P.N = (int32_t)N;
  P.eps = eps;
  P.stream = streaming_rows(M, N);
  P.n_blocks = (int32_t)((M + SBM - 1) / SBM);
  const int64_t tiles = (N + 63) / 64;
  P.n_slices = (int32_t)((N + kSliceCols - 1) / kSliceCols);
  if (P.n_slices > 32) return fail(VT_ERR_UNSUPPORTED, no);
  P.slice_cols = (int32_t)((tiles + P.n_slices - 1) / P.n_slices * 64);
  // Two blocks per compute unit (256 of them) at least: below, loading W and filling the pipeline cost what they save (us
  // in the caches, streamed weight / here: 25088 x 96 -> 288 9.9 / 9.4, x 128 -> 512 11.8 / 12.1, x 128 -> 1024 17.5 / 18.5,
  // 12544 x 96 -> 288 7.0 / 7.5; 37632 x 96 -> 288 17.0 / 11.2).
  if (P.n_blocks < 512) return fail(VT_ERR_UNSUPPORTED, no);
  P.groups = 32 / P.n_slices * 8;
  const bool c32 = c_dtype == VT_F32;
  if (A.dtype == VT_BF16) return c32 ? launch_slice<bf16_t, true>(P, ks, st) : launch_slice<bf16_t, false>(P, ks, st);
  return c32 ? launch_slice<f16_t, true>(P, ks, st) : launch_slice<f16_t, false>(P, ks, st);
}

}  // namespace vt
