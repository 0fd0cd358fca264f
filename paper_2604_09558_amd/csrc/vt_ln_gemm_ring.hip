// LayerNorm fused into the load stage of a GEMM, rows of 128 to 512 features (a multiple of 64):
// C = LN(A) . W, A virtual [.., K] with contiguous rows, W a row-major [K, N] matrix.  (vt_ln_gemm.hip and
// vt_ln_gemm_slice.hip hold W in registers for up to 128 features, vt_ln_gemm_wide.hip streams it through registers.)
// Bound by a chain of phases inside a workgroup: rows arrive, are normalised, the product, the stores; the matrix pipes are
// busy for a third of it, HBM is at half of the copy rate.
//
// A workgroup of 8 waves takes 64, 96, 128 or 160 rows: fetched through the map (16 bytes per lane), normalised in
// registers (fp32, two passes, one root and division for four rows), rounded to the operand type and parked in LDS,
// where they stay.  After the one barrier every wave works alone: it owns tiles of 64 columns, and its share of W
// comes straight from global memory into a ring of its own in LDS (global_load_lds_dwordx4, four or six stages of 16
// rows of W: 64 to 96 KB under way per compute unit, without registers; the kernel that streams through registers has two
// steps under way and turns every 8x4 block with v_perm_b32).  Waits count the requests by hand; nobody else
// reads a ring, so there are no barriers.  C^T += W^T . LN(A)^T on v_mfma_f32_32x32x16 (W's fragments by transposing
// reads): a lane ends up with 4 consecutive columns of a row, a wave turns 32 rows at a time round in the two stages
// of its ring that are free and leaves with whole 128-byte row segments (streaming stores: 18.5 us, plain ones 19.8 for
// 25088 x 256 -> 768; without turning, 32-byte pieces after v_permlane32_swap: 21.5).
// Measured (us, through registers -> here; floor by bytes or operations): 25088 x 256 -> 768 21 -> 18 (10), 21952 x 512 -> 512 46
// -> 20 (10), 33600 x 192 -> 768 34 -> 22 (12.5).  Workgroups of 4 waves, two to a compute unit: 20.9 for the first (1 %
// better on average over all shapes with them than without, not kept).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "vt_ln_rows.h"

using namespace vt;
using namespace vt::gemm;

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8;
constexpr int kLds = 160 * 1024;
constexpr int TBN = 64;           // columns of a wave's tile
constexpr int KST = 16;           // rows of W per stage of a ring
constexpr int kStage = KST * TBN * 2;

// at most N vector memory operations outstanding, no LDS operation
template <int N>
__device__ __forceinline__ void wait_ops() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

// Sum over LP2 = 16 or 32 consecutive lanes, every lane gets the total.
template <int LP2>
__device__ __forceinline__ float row_sum(float v) {
  v = group_sum<16>(v);
  if (LP2 >= 32) v += __shfl_xor(v, 16, 64);
  return v;
}

// MB blocks of 32 rows per workgroup; LP2 lanes hold a row, two chunks of 8 elements each: K <= 16 * LP2; rings of STAGES.
// STREAM: 16-bit results leave as streaming stores (asked for in the kernel, both kinds' code costs 0.15 us a launch).
template <typename T, bool C_F32, bool STREAM, int MB, int LP2, int STAGES>
__global__ void __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_ln_gemm_ring(const LnParams P) {
  typedef Mma<T> M_;
  typedef typename M_::vec opvec;
  static_assert(STAGES % 2 == 0 && STAGES >= 4, "the last two stages of a tile lie side by side");
  constexpr int BM = MB * 32, WR = BM / kWaves;      // rows of the workgroup, and those that a wave normalises
  constexpr int RPP = 64 / LP2, NP = WR / RPP;       // rows per pass, passes
  constexpr int CH = 2;
  __shared__ __attribute__((aligned(1024))) uint4 lds[kLds / 16];   // the rows, then a ring per wave
  char* const lds_b = reinterpret_cast<char*>(lds);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l32 = lane & 31, lh = lane >> 5;
  const int M = P.M, N = P.N, K = P.K;
  const int pitch = K * 2;                           // bytes of a row
  const int steps = K / KST;                         // even
  const int row0 = blockIdx.x * BM;
  const int tile0 = blockIdx.y * P.tiles_per_group + wave;
  const int tile_end = min((int)(blockIdx.y + 1) * P.tiles_per_group, (N + TBN - 1) / TBN);

  // ---- W: a cursor over (tile, stage) runs STAGES ahead of the multiplication.  Chunk c of k-row k lies at
  // c ^ ((k >> 1 & 1) << 2) (the four k-rows x 64 bytes that 32 lanes of a transposing read touch lie in different
  // banks): the lane that lands at position p asks for chunk p ^ key.  Past the last stage it is asked for again (it
  // hits the caches and is not read).
  const int ring = __builtin_amdgcn_readfirstlane(BM * pitch + wave * (STAGES * kStage));     // byte in lds
  const uint32_t ring_dst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lptr_t)&lds[0] + ring);
  const int64_t row_bytes = P.ldb * 2;
  const int w_k = lane >> 3, w_chunk = (lane & 7) ^ ((w_k >> 1 & 1) << 2);
  const uint32_t w_lane = (uint32_t)(w_k * row_bytes);
  uint32_t w_off = w_lane + (uint32_t)min(tile0 * TBN + w_chunk * 8, N - 8) * 2;
  int ld_tile = tile0, ld_step = 0;
  auto request_stage = [&](int slot) {
    const char* base = P.b + (int64_t)(ld_step * KST) * row_bytes;
    request(w_off, base, ring_dst + slot * kStage);
    request(w_off, base + 8 * row_bytes, ring_dst + slot * kStage + 1024);
    if (ld_step + 1 < steps) {
      ++ld_step;
    } else if (ld_tile + kWaves < tile_end) {
      ld_step = 0;
      ld_tile += kWaves;
      w_off = w_lane + (uint32_t)min(ld_tile * TBN + w_chunk * 8, N - 8) * 2;
    }
  };
  const bool works = tile0 < tile_end;               // (else this wave only normalises)

  // ---- rows.  Chunk c (16 bytes) of row r lies at c ^ key(r), so that 16 rows of a fragment read fall into
  // different banks: rows of a multiple of 256 bytes start in the same one, others in every second one.
  const int key_mask = K % 128 ? 7 : 15, key_shift = K % 128 ? 1 : 0;
  auto key = [&](int r) { return r >> key_shift & key_mask; };
  {
    const uint32_t m = (uint32_t)min(row0 + wave * WR + min(lane, WR - 1), M - 1);
    const int64_t ro = (P.a_row.tdig >= 0 ? axis_off_table(P.a_row, m) : axis_off(P.a_row, m)) * 2;
    const int ro_lo = (int)(uint32_t)(uint64_t)ro, ro_hi = (int)(ro >> 32);
    const int c0 = lane % LP2, r0 = lane / LP2;
    uint4 raw[NP][CH];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const int r = p * RPP + r0;
      const uint64_t off = (uint32_t)__shfl(ro_lo, r, 64) | ((uint64_t)(uint32_t)__shfl(ro_hi, r, 64) << 32);
      const char* rp = P.a + (int64_t)off;
#pragma unroll
      for (int h = 0; h < CH; ++h) {
        raw[p][h] = make_uint4(0, 0, 0, 0);
        if ((c0 + h * LP2) * 8 < K) raw[p][h] = *reinterpret_cast<const uint4*>(rp + (c0 + h * LP2) * 16);
      }
    }
    // the first stages of W are asked for behind the rows, and arrive while these are normalised
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (works) {
#pragma unroll
      for (int s = 0; s < STAGES; ++s) request_stage(s);
    }
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
          const Vec<T, 8> v = __builtin_bit_cast(Vec<T, 8>, raw[p0 + i][h]);
#pragma unroll
          for (int j = 0; j < 8; ++j) x[i][h][j] = to_float(v.v[j]);
          s += ((x[i][h][0] + x[i][h][1]) + (x[i][h][2] + x[i][h][3])) + ((x[i][h][4] + x[i][h][5]) + (x[i][h][6] + x[i][h][7]));
        }
        const float mean = over_k(row_sum<LP2>(s), k, inv_k);
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
        q[i] = row_sum<LP2>(d2);
      }
      // One root and one division (some 40 instructions) for the rows of up to four passes: lane 4 n + i of a row takes
      // pass i's, and the four receive the results.  As in the generic kernel, a subnormal variance (eps = 0) has a
      // finite root, which v_rsq_f32 does not give.
      float qs = q[0];
#pragma unroll
      for (int i = 1; i < Q; ++i)
        if (p0 + i < NP) qs = (lane & 3) == i ? q[i] : qs;
      const float rstd = 1.0f / sqrtf(squares_over_k(qs, k, inv_k) + P.eps);
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        if (p0 + i >= NP) continue;
        const float rs = i == 0 ? dpp_move<0x00>(rstd) : i == 1 ? dpp_move<0x55>(rstd) : i == 2 ? dpp_move<0xAA>(rstd) : dpp_move<0xFF>(rstd);
        const int r = wave * WR + (p0 + i) * RPP + r0;
#pragma unroll
        for (int h = 0; h < CH; ++h) {
          uint32_t w[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) w[j] = pack2<T>(x[i][h][2 * j] * rs, x[i][h][2 * j + 1] * rs);
          const int c = c0 + h * LP2;
          if (c * 8 < K) *reinterpret_cast<uint4*>(lds_b + r * pitch + (c ^ key(r)) * 16) = make_uint4(w[0], w[1], w[2], w[3]);
        }
      }
    }
  }
  __syncthreads();
  if (!works) return;                                // (nothing of this wave is under way)

  // ---- the product: every wave by itself from here on
  struct Frags {
    opvec a[MB], w[2];
  };
  const char* a_row_of[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) a_row_of[mb] = lds_b + (mb * 32 + l32) * pitch;
  const int a_chunk = (lh ^ key(l32)) * 16;          // chunk 2 step + lh: XOR with 32 step
  const int lq = lane >> 4, ll = lane & 15;
  int w_frag[2][2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = 8 * (lq >> 1) + (ll >> 2) + 4 * h, chunk = nb * 4 + 2 * (lq & 1) + ((ll & 3) >> 1);
      w_frag[nb][h] = ring + k * (TBN * 2) + ((chunk ^ ((k >> 1 & 1) << 2)) * 16) + (ll & 1) * 8;
    }
  auto read = [&](Frags& f, int step, int slot) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      struct { s16x4 lo, hi; } v;
      v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(lds_b + w_frag[nb][0] + slot * kStage));
      v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(lds_b + w_frag[nb][1] + slot * kStage));
      f.w[nb] = __builtin_bit_cast(opvec, v);
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) f.a[mb] = __builtin_bit_cast(opvec, *reinterpret_cast<const uint4*>(a_row_of[mb] + (a_chunk ^ (step * 32))));
  };
  f32x16 acc[2][MB];
  auto clear = [&]() {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[nb][mb][e] = 0.f;
  };
  auto multiply = [&](const Frags& f) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = M_::run(f.w[nb], f.a[mb], acc[nb][mb]);
  };
  // stage 3: a lane holds row mb * 32 + l32, columns nb * 32 + 8 j + 4 lh + i.  The buffer descriptor ends with the
  // block's last row and columns past N get an offset outside of it: no store is conditional, the waits count on it.
  constexpr int ES = C_F32 ? 4 : 2, kStores = C_F32 ? MB * 8 : MB * 4;
  const int rows = min(BM, M - row0);
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(P.c + (size_t)row0 * (size_t)N * ES, 0, rows * N * ES, 0x00020000);
  auto store_tile = [&](int tile, char* turn) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      if constexpr (C_F32) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int col = tile * TBN + nb * 32 + 8 * j + 4 * lh;
            const uint32_t off = col < N ? (uint32_t)((mb * 32 + l32) * N + col) * 4u : 0x80000000u;
            const u32x4 v = __builtin_bit_cast(u32x4, make_float4(acc[nb][mb][4 * j], acc[nb][mb][4 * j + 1], acc[nb][mb][4 * j + 2], acc[nb][mb][4 * j + 3]));
            __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, (int)off, 0, 0);
          }
      } else {
        // 32 rows of 8 chunks of 16 bytes turned round in the ring's two free stages; chunk c of row r at c ^ (r >> 1 & 7)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            *reinterpret_cast<uint2*>(turn + l32 * 128 + (((nb * 4 + j) ^ (l32 >> 1 & 7)) * 16) + lh * 8) =
                make_uint2(pack2<T>(acc[nb][mb][4 * j], acc[nb][mb][4 * j + 1]), pack2<T>(acc[nb][mb][4 * j + 2], acc[nb][mb][4 * j + 3]));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int rr = q * 8 + (lane >> 3), ch = lane & 7;   // 8 lanes per row of 64 columns
          const u32x4 v = __builtin_bit_cast(u32x4, *reinterpret_cast<const uint4*>(turn + rr * 128 + ((ch ^ (rr >> 1 & 7)) * 16)));
          const int col = tile * TBN + ch * 8;
          const uint32_t off = col < N ? (uint32_t)((mb * 32 + rr) * N + col) * 2u : 0x80000000u;
          __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, (int)off, 0, STREAM ? 2 : 0);   // (streaming: whole lines, not read again here)
        }
      }
    }
  };

  // Operations behind the requests of the next stage when its step waits for it: those of STAGES - 2 stages; at a tile's
  // last step one stage fewer (its last two stages are asked for after the stores); in the first steps of a
  // later tile the stores of the tile before as well.
  constexpr int kBehind = (STAGES - 2) * 2;
  Frags f[2];
  wait_ops<(STAGES - 1) * 2>();
  read(f[0], 0, 0);
  int slot = 0;                                      // the stage whose fragments are in registers
  for (int tile = tile0; tile < tile_end; tile += kWaves) {
    clear();
    auto one = [&](int step, auto parity) {
      constexpr int B = decltype(parity)::value;
      const int next = slot == STAGES - 1 ? 0 : slot + 1;
      if (B == 1 && step == steps - 1) wait_ops<kBehind - 2>();
      else if (tile != tile0 && step <= STAGES - 4) wait_ops<kBehind + kStores>();
      else wait_ops<kBehind>();
      if (step < steps - 2) request_stage(slot);
      read(f[1 - B], step == steps - 1 ? 0 : step + 1, next);
      multiply(f[B]);
      slot = next;
    };
    for (int step = 0; step < steps; step += 2) {
      one(step, std::integral_constant<int, 0>{});
      one(step + 1, std::integral_constant<int, 1>{});
    }
    // `slot` is the next tile's first stage; the two before it are free
    const int free0 = slot == 0 ? STAGES - 2 : slot - 2;
    store_tile(tile, lds_b + ring + free0 * kStage);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    request_stage(free0);
    request_stage(free0 + 1);
  }
  wait_ops<0>();                                     // requests past the last stage still target this workgroup's LDS
}

// LDS of blocks of 32 mb rows and of the shortest rings
bool rows_fit(int mb, int K) { return mb * 32 * K * 2 + kWaves * 4 * kStage <= kLds && (mb < 5 || K <= 256); }

template <typename T, bool C_F32, bool STREAM>
int launch_ring(LnParams P, int mb, int groups, hipStream_t st) {
  const int tiles = (P.N + TBN - 1) / TBN;
  P.tiles_per_group = (tiles + groups - 1) / groups;
  const dim3 grid((unsigned)((P.M + mb * 32 - 1) / (mb * 32)), (unsigned)((tiles + P.tiles_per_group - 1) / P.tiles_per_group));
#define VT_RING(MB, LP2, S)                                                                             \
  if (mb == MB && (P.K <= 256) == (LP2 == 16) && MB * 32 * P.K * 2 + kWaves * S * kStage <= kLds) {     \
    hipLaunchKernelGGL((k_ln_gemm_ring<T, C_F32, STREAM, MB, LP2, S>), grid, dim3(kWaves * 64), 0, st, P);      \
    return check_launch("vt_gemm(layernorm)");                                                          \
  }
  VT_RING(2, 16, 6) VT_RING(3, 16, 6) VT_RING(4, 16, 6) VT_RING(5, 16, 4)   // (160 rows: longer rings spill)
  VT_RING(2, 32, 6) VT_RING(3, 32, 4) VT_RING(4, 32, 4)
#undef VT_RING
  return fail(VT_ERR_UNSUPPORTED, "vt_gemm(layernorm): outside the fused kernels");
}

// Rows per workgroup and groups of columns (each normalises its rows again), or false where the kernel that streams W
// through registers is the better one.  The model, fitted over 238 shapes (K 128 to 512, N 200 to 4 K, M 324 to 96100)
// and every choice there: rounds of 256 workgroups of 2.5 us each, LayerNorm 0.36 us per 32 rows x 64 features, and per four
// tiles of 64 columns (one wave of each SIMD) what W's arrival, the product and the stores take.  Some of them (bf16, us):
//   M x K -> N           other kernel   64 rows   96   128   160
//   25088 x 256 -> 768       21            22     28    18    20
//   21904 x 512 -> 512       45            30     20     -     -
//   33600 x 192 -> 768       34            31     27    32    22
//   12544 x 192 -> 768       12.8          10.3   11.7  13.1  14.9
//    7744 x 256 -> 768       10.5     8.9 in two groups
// The other kernel stays for fewer than 1024 rows (324 x 512 -> 2048: 11.1 against 12.1, 588 x 384 -> 384: 9.7 against 9.9); for more than 384
// features where its blocks of 128 rows, which do not fit here, need fewer rounds than blocks of 96 (24964 x 512 -> 512: 26 against
// 29); and where its blocks of 64 rows make one round with less than a tile for each of its eight waves, if there are up to
// 256 columns (4096 x 192 -> 200, f16: 6.0 against 6.6), rows are not whole 64-byte units, whose pieces are stored
// slower here, or the choice here would be taller blocks that several groups normalise again (5058 x 192 -> 768: 28 % longer here).
// At 750 shapes drawn apart (M from 1000, two thirds of them below 18000, operands in turn) the choice takes 1.3 % longer
// than the best one on average, 25 % at most, 27 of them more than 10 %.  (Without the last two: 2.9 %, 90 of them.)
bool choose_ring(int64_t M, int64_t N, int64_t K, int* mb_out, int* groups_out) {
  if (M < 1024) return false;
  auto rounds = [](int64_t wgs) { return (wgs + 255) / 256; };
  if (K > 384 && M >= 192 * 128 && M <= 512 * 128 && rounds((M + 95) / 96) > rounds((M + 127) / 128)) return false;
  const int64_t tiles = (N + TBN - 1) / TBN, k = K / 64;
  int64_t best = 0;
  for (int mb = 2; mb <= 5; ++mb) {
    if (!rows_fit(mb, (int)K)) continue;
    const int64_t blocks = (M + mb * 32 - 1) / (mb * 32);
    for (int g = 1; g <= 8 && (g == 1 || (blocks * g <= 256 && g <= (tiles + 1) / 2)); g *= 2) {
      const int64_t per_group = (tiles + g - 1) / g, quads = (per_group + 3) / 4;
      const int64_t cost = rounds(blocks * ((tiles + per_group - 1) / per_group)) * (2540 + mb * k * 363 + quads * (mb * k * 61 + k * 287 + mb * 128));
      if (best == 0 || cost < best) {
        best = cost;
        *mb_out = mb, *groups_out = g;
      }
    }
  }
  if (best != 0 && M <= 256 * 64) {
    const int64_t groups = std::max<int64_t>(1, std::min(256 / ((M + 63) / 64), (tiles + 1) / 2));   // the other kernel's
    if ((tiles + groups - 1) / groups < 8 && (N <= 256 || N % 32 || (*mb_out >= 3 && *groups_out > 1))) return false;
  }
  return best != 0;
}

}  // namespace

namespace vt {

int ln_gemm_panel_launch(const gemm::LnParams& L, int dtype, bool c_f32, hipStream_t st);   // vt_ln_gemm_panel.hip

// One group of vt_gemm with prologue = VT_GEMM_LAYERNORM on the kernel above, or VT_ERR_UNSUPPORTED (shapes, maps or
// alignments it does not take, and every error that the generic kernel reports).
int ln_gemm_ring_launch(const vt_desc& A, const vt_desc& B, void* C, int c_dtype, float eps, hipStream_t st) {
  const char* no = "vt_gemm(layernorm): outside the fused kernels";
  const int n = (int)A.shape.size();
  if (n < 2 || B.shape.size() != 2 || B.shape[0] != A.shape[n - 1]) return fail(VT_ERR_UNSUPPORTED, no);
  const int64_t K = A.shape[n - 1], N = B.shape[1];
  int64_t M = 1;
  for (int i = 0; i < n - 1; ++i) M *= A.shape[i];
  if (M < 1 || K % 64 || K < 128 || K > 512 || N < 8 || N % 8) return fail(VT_ERR_UNSUPPORTED, no);
  // (the limits of the generic kernel, which took these calls before there was this one; a block of C stays below 2 GiB)
  if (M > 65535ll * 64 || N > 65535ll * 32 || M * K >= (1ll << 31) || K * N >= (1ll << 31)) return fail(VT_ERR_UNSUPPORTED, no);
  if (A.pieces.size() != 1 || !A.pieces[0].v.lower.empty() || B.pieces.size() != 1 || !B.pieces[0].v.lower.empty())
    return fail(VT_ERR_UNSUPPORTED, no);
  LnParams P;
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
  // a lane's share of W's address is 32 bits
  const bool w_ok = b_row.nd == 1 && b_col.nd == 1 && b_col.stride[2] == 1 && P.ldb % 8 == 0 && P.ldb >= 0 && (uintptr_t)P.b % 16 == 0 &&
                    P.ldb * 16 + N * 2 < (1ll << 32);
  if (!rows_ok || !w_ok || (uintptr_t)P.c % 16) return fail(VT_ERR_UNSUPPORTED, no);
  P.M = (int32_t)M;
  P.N = (int32_t)N;
  P.K = (int32_t)K;
  P.eps = eps;
  const int rc = ln_gemm_panel_launch(P, A.dtype, c_dtype == VT_F32, st);      // few rows
  if (rc != VT_ERR_UNSUPPORTED) return rc;
  int mb = 0, groups = 1;
  if (!choose_ring(M, N, K, &mb, &groups)) return fail(VT_ERR_UNSUPPORTED, no);
  const bool c32 = c_dtype == VT_F32, stream = streaming_rows(M, N);
  if (A.dtype == VT_BF16)
    return c32 ? launch_ring<bf16_t, true, false>(P, mb, groups, st) : stream ? launch_ring<bf16_t, false, true>(P, mb, groups, st) : launch_ring<bf16_t, false, false>(P, mb, groups, st);
  return c32 ? launch_ring<f16_t, true, false>(P, mb, groups, st) : stream ? launch_ring<f16_t, false, true>(P, mb, groups, st) : launch_ring<f16_t, false, false>(P, mb, groups, st);
}

}  // namespace vt
