// Tiled GEMM for products that the 256 x 256 tiles of vt_gemm.hip would spread over too few compute
// units: the same product, operand maps, order of accumulation (identical bits) and tile walk, with
// smaller tiles and a deeper pipeline.  A short prompt or a decode batch's experts are bound by
// pulling the operands into the compute units, not by the matrix cores: the requests alone, with the
// operands in the caches, go at some 100 GB/s a unit and 22 TB/s in all (in HBM, at two thirds of that), so what
// counts is how many units share the work and how few bytes each has to read (BM + BN per K step and tile).
//
// One workgroup of 4 waves computes a BM x BN tile of C in 32 x 32 matrix-core blocks
// (v_mfma_f32_32x32x16; tiles of 32 rows: 16 x 16 blocks).  K steps of 64 run through a ring of STAGES stages in LDS, each of
// one step or, for 32 rows, two; operands go from
// global memory straight into it (global_load_lds_dwordx4: no registers, no store instructions),
// STAGES stages ahead, one barrier per stage; a stage's fragments are read into registers during the
// one before.  The lanes of a request land in the order of their numbers, so the swizzle that keeps
// the fragment reads free of bank conflicts (4.3 million conflict cycles per launch without it, 4600
// with it, 333 x 4096 x 4096) is applied to what a lane asks for.  Waits count the requests by hand: a wave issues the
// same number in every stage and nothing else that goes through the vector memory counter.
// Measured (f16/bf16, K = 4096, operands in HBM / in the caches, us): 333 x 4096 32.5 / 22.2 (256 x 256 tiles 88 / 83),
// 400 x 6144 37.3 / 31.6 (90 / 84), 1024 x 4096 43.3 / 36.5 (89 / 80); the requests of the first without anything
// else 27.4 / 18.1.  A step of 64 x 128 takes 265 ns there, of which the requests need 231.  Rings twice as
// deep, and waves divided over K instead of over the tile (half the LDS reads), measured no faster.
// Few tiles (a short prompt) leave most of the chip idle, and a step of 64 x 64 then takes 0.2 us on a chain of barrier,
// fragment reads and four dependent products of 60 cycles.  Tiles of 32 rows bring four times the units to work, blocks of 16 halve
// the chain, two steps per stage the barriers.  Measured (us, 64 x 64 / 32 x 64 / 32 x 32; in the caches): 34 x 2048 -> 1000 10.5 / 8.6 / 7.2,
// 62 x 1024 -> 2048 7.4 / 6.3 / 5.4, 100 x 4096 -> 1000 16.9 / 13.9 / 11.8, 212 x 4096 -> 2048 (mapped) 19.6 / 16.1 / 18.3, 168 x 1024 ->
// 4096 7.8 / 7.9 / 9.1.  (In 32 x 32 blocks, one or two waves multiplying: 8.2 for the first; K divided among the waves and their four
// sums added: 6.3, in bits that depend on how many tiles the launch has.  One step per stage 7.8, four 7.7, longer rings 7.4 to 8.3.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "vt_gemm_common.h"
#include "vt_gemm_params.h"

using namespace vt;
using namespace vt::gemm;

namespace {

constexpr int BK = 64;
constexpr int kMaxSteps = 256;        // K <= 16384

// The swizzle: chunk c (16 bytes) of a 128-byte row r lies at position c ^ row_key(r): the 16 rows of a
// fragment read fall into different banks.  Chunk c of B's k-row k lies at c ^ k_key(k): so do the
// four k-rows x 64 bytes that 32 lanes of a transposing read touch (blocks of 16: twice four, eight apart, x 32 bytes).
__device__ __forceinline__ int row_key(int r) { return r >> 1 & 7; }
template <int BN, int BLK>
__device__ __forceinline__ int k_key(int k) {
  if (BLK == 16) return (BN == 32 ? 0 : (k >> 1 & 1) << 2) | (k >> 3 & 1) << 1;
  return BN == 64 ? (k >> 1 & 1) << 2 : (k & 3) << 2;
}

// Matrix-core blocks of 32 x 32 (16 of K at a time) or, in tiles too small for four waves of those, 16 x 16 (32 of K).  Both add
// the products of a chain in the same order: the same bits (test_every_tile_gives_the_same_bits).
template <typename T, int BLK>
struct BlockMma {
  typedef typename Mma<T>::vec vec;
  typedef f32x16 acc;
  static constexpr int K = 16, kRows = 4;            // a lane holds rows 8 j + 4 lh + i of its column, j < kRows
  static __device__ __forceinline__ acc run(vec a, vec b, acc c) { return Mma<T>::run(a, b, c); }
};
template <typename T>
struct BlockMma<T, 16> {
  typedef typename Mma16<T>::vec vec;
  typedef f32x4 acc;
  static constexpr int K = 32, kRows = 1;            // rows 4 lq + i
  static __device__ __forceinline__ acc run(vec a, vec b, acc c) { return Mma16<T>::run(a, b, c); }
};

template <typename T, bool C_F32, bool MAPPED, bool B_KMAJOR, int NG, int BM, int BN, int WM, int STAGES, int R, int BLK>
__global__ void __launch_bounds__(256)
k_gemm_tile(const GemmParamsT<NG> P, const typename std::conditional<MAPPED, OutMap, NoMap>::type O) {
  typedef BlockMma<T, BLK> M_;
  typedef typename M_::vec opvec;
  constexpr int kABytes = BM * BK * 2, kStep = (BM + BN) * BK * 2, kStage = R * kStep;
  constexpr int AI = BM / 32, BI = BN / 32;          // requests per wave and K step (1 KB each)
  constexpr int WN = 4 / WM;                         // the waves' grid
  constexpr int MB = BM / (BLK * WM), NB = BN / (BLK * WN);   // blocks per wave
  static_assert(!MAPPED || 4 * BM * 8 <= STAGES * kStage, "the row offsets of the output fit the ring");
  __shared__ __attribute__((aligned(1024))) char lds[STAGES * kStage];
  // byte offsets of every K step along A's columns and B's rows (a step of 64 stays inside the
  // innermost K digit of both), evaluated once: nothing in the K loop reads kernel arguments
  __shared__ uint4 steps[kMaxSteps];

  int gi, tm, tn;
  if (!pick_tile(P, blockIdx.x, &gi, &tm, &tn)) return;
  const GemmGroup& G = P.g[gi];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int lb = lane % BLK, lh = lane / BLK;        // a lane's row (A) or column (B) of a block, and its 8 of the block's K
  const int Mg = G.M, N = P.N, nk = P.K / BK;

  // ---- stage 1 through the map.  A: 8 lanes per row of 64 k, 8 rows per request; B: BN / 8 lanes per
  // k-row; B_KMAJOR: like A, rows are the columns n.  (32-bit offsets: checked on the host.)
  const char* const a_base = G.a;
  const char* const b_base = G.b;
  const int r8 = lane >> 3, p8 = lane & 7;
  uint32_t a_off[AI], b_off[BI];
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int r = (wave * AI + i) * 8 + r8;
    const uint32_t m = (uint32_t)min(tm * BM + r, Mg - 1);
    const int64_t ro = G.a_row.tdig >= 0 ? axis_off_table(G.a_row, m) : axis_off(G.a_row, m);
    a_off[i] = (uint32_t)(ro * 2) + (uint32_t)((p8 ^ row_key(r)) * 16);
  }
  constexpr int LB = BN / 8, RB = 64 / LB;           // lanes per k-row of B, k-rows per request
  const int64_t b_kstride = G.b_row.stride[2] * 2;
  if (B_KMAJOR) {
#pragma unroll
    for (int i = 0; i < BI; ++i) {
      const int r = (wave * BI + i) * 8 + r8;
      b_off[i] = (uint32_t)(axis_off(G.b_col, (uint32_t)min(tn * BN + r, N - 1)) * 2) + (uint32_t)((p8 ^ row_key(r)) * 16);
    }
  } else {
    // a lane's k-row in request i: (wave * BI + i) * RB + kr, of which the first part is whole periods of the key
    static_assert(BI * RB % (BLK == 16 ? 16 : 4) == 0, "the key's period");
    const int kr = lane / LB;
#pragma unroll
    for (int i = 0; i < BI; ++i) {
      const uint32_t n = (uint32_t)min(tn * BN + ((lane % LB) ^ k_key<BN, BLK>(i * RB + kr)) * 8, N - 8);
      b_off[i] = (uint32_t)(axis_off(G.b_col, n) * 2) + (uint32_t)(kr * b_kstride);
    }
  }
  if ((int)threadIdx.x < nk) {
    const uint32_t k = threadIdx.x * BK;
    const uint64_t bo = (uint64_t)(axis_off(G.b_row, k) * 2);
    steps[threadIdx.x] = make_uint4((uint32_t)(axis_off(G.a_col, k) * 2), (uint32_t)bo, (uint32_t)(bo >> 32), 0);
  }
  __syncthreads();
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)&lds[0];
  // a stage holds R K steps: where their operands start
  struct Starts {
    const char *a[R], *b[R];
  };
  struct Offsets {
    uint4 o[R];
  };
  auto offsets_of = [&](int stage) {
    Offsets f;
#pragma unroll
    for (int r = 0; r < R; ++r) f.o[r] = steps[min(stage * R + r, nk - 1)];
    return f;
  };
  auto starts_of = [&](const Offsets& f) {
    Starts s;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t lo = __builtin_amdgcn_readfirstlane(f.o[r].y), hi = __builtin_amdgcn_readfirstlane(f.o[r].z);
      s.a[r] = a_base + (uint32_t)__builtin_amdgcn_readfirstlane(f.o[r].x);
      s.b[r] = b_base + (int64_t)(((uint64_t)hi << 32) | lo);
    }
    return s;
  };
  // request q (of each step the AI of A, then the BI of B) of the stage that starts at `s`, into ring position `slot`
  auto request_one = [&](int q, const Starts& s, int slot) {
    const int r = q / (AI + BI), i = q % (AI + BI), j = i - AI;
    const uint32_t dst = lds0 + slot * kStage + r * kStep;
    if (i < AI) request(a_off[i], s.a[r], dst + (wave * AI + i) * 1024);
    else request(b_off[j], B_KMAJOR ? s.b[r] : s.b[r] + (wave * BI + j) * RB * b_kstride, dst + kABytes + (wave * BI + j) * 1024);
  };

  // ---- fragment addresses in a stage (bytes), for its first MFMA
  uint32_t a_frag[MB], b_frag[NB][2];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int r = (wm * MB + mb) * BLK + lb;
    a_frag[mb] = r * 128 + ((lh ^ row_key(r)) * 16);    // chunk K / 8 ks + lh: XOR with 2 K ks
  }
  const int lq = lane >> 4, ll = lane & 15;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    if (B_KMAJOR) {
      const int r = (wn * NB + nb) * BLK + lb;
      b_frag[nb][0] = kABytes + r * 128 + ((lh ^ row_key(r)) * 16);
      b_frag[nb][1] = 0;
    } else {
      // lane ll of a 16-lane group points at k-row (ll >> 2) (and 4 further) of the group's 8, columns 4 (ll & 3) .. + 3;
      // it receives the 4 consecutive k of column ll
      const int k8 = BLK == 16 ? lq : lq >> 1;
      const int chunk = (wn * NB + nb) * (BLK / 8) + (BLK == 16 ? 0 : 2 * (lq & 1)) + ((ll & 3) >> 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = 8 * k8 + (ll >> 2) + 4 * h;
        b_frag[nb][h] = kABytes + k * (BN * 2) + ((chunk ^ k_key<BN, BLK>(k)) * 16) + (ll & 1) * 8;
      }
    }
  }

  typename M_::acc acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4 * M_::kRows; ++e) acc[i][j][e] = 0.f;

  // all fragments of one stage: read from LDS during the stage before, so that neither the barrier
  // nor the latency of the reads stands between two stages' products
  constexpr int KS = BK / M_::K;
  struct Frags {
    opvec a[R * KS][MB], b[R * KS][NB];
  };
  constexpr int kReads = R * KS * (MB + NB), kMma = R * KS * MB * NB, kRequests = R * (AI + BI);
  auto read_one = [&](const char* stage, Frags& f, int i) {
    const int km = i / (MB + NB), ks = km % KS, x = i % (MB + NB), nb = x - MB;
    const char* const st = stage + km / KS * kStep;
    if (x < MB) {
      f.a[km][x] = __builtin_bit_cast(opvec, *reinterpret_cast<const uint4*>(st + (a_frag[x] ^ (ks * 2 * M_::K))));
    } else if (B_KMAJOR) {
      f.b[km][nb] = __builtin_bit_cast(opvec, *reinterpret_cast<const uint4*>(st + (b_frag[nb][0] ^ (ks * 2 * M_::K))));
    } else {
      typedef short s16x4 __attribute__((ext_vector_type(4)));
      typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
      struct { s16x4 lo, hi; } v;
      v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(st + b_frag[nb][0] + ks * M_::K * (BN * 2)));
      v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(st + b_frag[nb][1] + ks * M_::K * (BN * 2)));
      f.b[km][nb] = __builtin_bit_cast(opvec, v);
    }
  };
  auto multiply_one = [&](const Frags& f, int i) {
    const int ks = i / (MB * NB), mb = i / NB % MB, nb = i % NB;
    acc[mb][nb] = M_::run(f.a[ks][mb], f.b[ks][nb], acc[mb][nb]);
  };
  // What was loaded above (index tables) has to be out of the vector memory counter's way.  Requests past
  // the last step repeat it (they hit the caches and land in stages that are not read again), so that
  // every step issues the same number and the loop has no branches.
  __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0)
#pragma unroll
  for (int s = 0; s < STAGES; ++s) {
    const Starts first = starts_of(offsets_of(s));
#pragma unroll
    for (int q = 0; q < kRequests; ++q) request_one(q, first, s);
  }
  constexpr int kFirst = (STAGES - 1) * kRequests;    // requests behind those of the first step,
  constexpr int kBehind = (STAGES - 2) * kRequests;   // and in the loop behind those of the next one
  static_assert(kFirst < 64, "vmcnt has 6 bits");
  Frags f0, f1;
  __builtin_amdgcn_s_waitcnt((kFirst & 15) | ((kFirst >> 4) << 14) | 0x0F70);
  asm volatile("s_barrier" ::: "memory");
#pragma unroll
  for (int i = 0; i < kReads; ++i) read_one(lds, f0, i);
  Offsets ahead = offsets_of(STAGES);
  int slot = 0;                                       // the stage that step `it` came from: in registers, free to be filled
  auto k_step = [&](int it, const Frags& cur, Frags& nxt) {
    // this wave has its fragments of step `it`, and its requests of step it + 1 have landed; behind
    // the barrier that holds for every wave
    __builtin_amdgcn_s_waitcnt((kBehind & 15) | ((kBehind >> 4) << 14) | 0x0070);   // vmcnt(kBehind) lgkmcnt(0)
    asm volatile("s_barrier" ::: "memory");
    const Starts next = starts_of(ahead);
    const int free_slot = slot;
    slot = slot == STAGES - 1 ? 0 : slot + 1;
    ahead = offsets_of(it + STAGES + 1);
    const char* const st = lds + slot * kStage;
    // A product, then its share of the requests and of the next step's reads.  A request holds its wave up
    // while the unit's address path works off those before it (16 cycles each, of all four waves), and
    // there is one wave per SIMD: all of a step's requests in a row left the matrix pipe idle for as long
    // as they took.  They are dealt out over seven eighths of the products, the reads over six, so that the
    // last ones have landed when the step ends.  (us, all in a row in front -> dealt out, operands in the caches:
    // 128 x 128 tiles, 333 x 4096 x 4096: 35.8 -> 28.7; 256 x 128: 59.8 -> 45.5; 64 x 128: 27.0 -> 23.5.)
    constexpr int kReqSpan = kMma * 7 / 8, kReadSpan = kMma * 6 / 8;
#pragma unroll
    for (int i = 0; i < kMma; ++i) {
      multiply_one(cur, i);
      if (i < kReqSpan) {
#pragma unroll
        for (int q = i * kRequests / kReqSpan; q < (i + 1) * kRequests / kReqSpan; ++q) request_one(q, next, free_slot);
      }
      if (i < kReadSpan) {
#pragma unroll
        for (int q = i * kReads / kReadSpan; q < (i + 1) * kReads / kReadSpan; ++q) read_one(st, nxt, q);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // full stages, then the last one, which may hold fewer steps than R = 2: the first of them
  const int n_full = nk / R;
  int it = 0;
  for (; it + 1 < n_full; it += 2) {
    k_step(it, f0, f1);
    k_step(it + 1, f1, f0);
  }
  if (nk % R) {
    if (it < n_full) {
      k_step(it, f0, f1);
      f0 = f1;
    }
#pragma unroll
    for (int i = 0; i < kMma / R; ++i) multiply_one(f0, i);
  } else if (it < n_full) {
#pragma unroll
    for (int i = 0; i < kMma; ++i) multiply_one(f0, i);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);                 // requests still target this workgroup's LDS

  // ---- stage 3 (as in vt_gemm.hip): a lane holds column lb of a block and rows 8 j + 4 lh + i
  if constexpr (MAPPED) {
    __syncthreads();
    int64_t* rowoff = reinterpret_cast<int64_t*>(lds);               // [pieces][BM]
    for (int pc = 0; pc < O.n; ++pc)
      for (int r = threadIdx.x; r < BM; r += 256) rowoff[pc * BM + r] = axis_off(O.p[pc].row, (uint32_t)min(tm * BM + r, Mg - 1));
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int col = tn * BN + (wn * NB + nb) * BLK + lb;
      if (col >= N) continue;
      int pc = 0;
#pragma unroll
      for (int i = 1; i < 4; ++i)
        if (i < O.n && col >= O.p[i].col_lo) pc = i;
      T* base = reinterpret_cast<T*>(O.p[pc].base) + axis_off(O.p[pc].col, (uint32_t)(col - O.p[pc].col_lo));
      const int64_t* ro = rowoff + pc * BM;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const int r0 = (wm * MB + mb) * BLK + lh * 4;
#pragma unroll
        for (int j = 0; j < M_::kRows; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (tm * BM + r0 + 8 * j + i < Mg) base[ro[r0 + 8 * j + i]] = from_float<T>(acc[mb][nb][4 * j + i]);
      }
    }
    return;
  }
  typedef typename std::conditional<C_F32, float, T>::type CT;
  CT* cbase = reinterpret_cast<CT*>(G.c);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int col = tn * BN + (wn * NB + nb) * BLK + lb;
      const int row0 = tm * BM + (wm * MB + mb) * BLK + lh * 4;
      CT* cp = cbase + (size_t)row0 * N + col;
      if (col < N) {
#pragma unroll
        for (int j = 0; j < M_::kRows; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (row0 + 8 * j + i < Mg) cp[(size_t)(8 * j + i) * N] = from_float<CT>(acc[mb][nb][4 * j + i]);
      }
    }
}

template <typename T, bool C_F32, bool MAPPED, bool B_KMAJOR, int NG = 1>
int launch_tile(GemmParams P8, const typename std::conditional<MAPPED, OutMap, NoMap>::type& O, int bm, int bn, hipStream_t st) {
  if constexpr (NG == 1 && !MAPPED)
    if (P8.n_groups > 1) return launch_tile<T, C_F32, MAPPED, B_KMAJOR, kMaxGroups>(P8, O, bm, bn, st);
  set_tiles(&P8, bm, bn);
  GemmParamsT<NG> P;
  static_cast<GemmSizes&>(P) = P8;
  for (int i = 0; i < NG; ++i) P.g[i] = P8.g[i];
  const dim3 grid(P.chunk * 8);
#define VT_TILE(BM_, BN_, WM_, S_, R_, BLK_)                                                                        \
  if (bm == BM_ && bn == BN_) {                                                                                     \
    hipLaunchKernelGGL((k_gemm_tile<T, C_F32, MAPPED, B_KMAJOR, NG, BM_, BN_, WM_, S_, R_, BLK_>), grid, dim3(256), 0, st, P, O); \
    return check_launch(MAPPED ? "vt_gemm_store" : "vt_gemm");                                                      \
  }
  VT_TILE(128, 256, 2, 3, 1, 32)
  VT_TILE(128, 128, 2, 4, 1, 32)
  VT_TILE(96, 128, 1, 5, 1, 32)
  VT_TILE(64, 512, 1, 2, 1, 32)
  VT_TILE(64, 256, 1, 3, 1, 32)
  VT_TILE(64, 128, 2, 3, 1, 32)
  VT_TILE(64, 64, 2, 4, 1, 32)
  VT_TILE(32, 64, 2, 3, 2, 16)
  VT_TILE(32, 32, 2, 3, 2, 16)
#undef VT_TILE
  return fail(VT_ERR_UNSUPPORTED, "vt_gemm: no such tile");
}

// The tile with the shortest estimated time: a launch, a start for every round of tiles over the compute units; then per K
// step of 64 a share for every round and one for every tile of an average unit (a last round that is nearly empty costs less
// than a full one, and the board's power limit slows full ones), or the draw of the weights where that takes longer (5.4 us of
// it beside the start); and C.  Weights are counted at 4 TB/s, which every tile exceeds; rows of [K,N] whose
// distance is a multiple of 4096 bytes are drawn slower, the slower the narrower the tile: its part of every row lies in the same channels of
// HBM (8 x 13 rows, K = 4096 -> 14336: 155 us on 64 x 512, 181 on 64 x 128; K = 5120 -> 11008: 175 and 159).
// The constants (ns; thousandths for weights and C) are fitted over every tile forced at 1505 shapes: 1 to 16384 rows, 1 to 8 groups,
// K 64 to 16384, N 48 to 28672, weights as [K,N] and [N,K], through the output map and not.  At 605 others, drawn apart, the tile taken is
// 0.8 % slower than the best one on average, 28 % at most, 2 % of them by more than 10 %.  (Fitted over 163 shapes from K = 512 on, without the
// term for C: 5 % there, 56 % at most, 15 to 20 % throughout K <= 256.)  Some of them, us:
//   rows x columns of C           256x256 / 128x256 / 128x128 / 96x128 / 64x512 / 64x256 / 64x128 / 64x64
//   333 x 4096, K = 4096               83 /  46 /  29 /  26 /  65 /  31 /  22 /  24
//   400 x 6144, K = 4096               84 /  47 /  31 /  30 /  68 /  33 /  36 /  41
//   8 x 50 x 14336, K = 4096 (groups) 240 / 175 / 198 / 194 / 159 / 169 / 193 / 212
//   8 x 200 x 8192, K = 2048           76 /  88 / 105 / 126 / 120 / 111 / 113 / 134
//   4 x 254 x 8192, K = 4096          107 / 129 / 129 / 118 / 190 / 137 / 132 / 156
//   1783 x 1552, K = 512, [N,K]        24 /  14 /  10 / 9.5 /  15 /  10 / 9.5 /  11
//   3105 x 11368, K = 128              36 /  46 /  52 /  61 /  46 /  52 /  42 /  60
// 0 x 0: the 256 x 256 kernel.  Returns the estimate in ns.
struct TileWork {
  int64_t N, K, weights;
  int n_groups;
  bool c_f32, same_channels;     // rows of [K,N] a multiple of 4096 bytes apart
};
template <typename Rows>         // group -> rows
int64_t choose_tile(const TileWork& P, Rows M, int* bm, int* bn) {
  static const int n_cu = [] {
    int dev = 0, n = 256;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) n = 256;
    return n > 0 ? n : 256;
  }();
  static const struct {
    int bm, bn, launch, round, step_round, step_tile, weights, out;
  } kTiles[] = {{256, 256, 7597, 5831, 1070, 679, 745, 289}, {128, 256, 2905, 5843, 613, 349, 717, 335},
                {128, 128, 1487, 5297, 333, 305, 733, 0}, {96, 128, 2206, 4989, 290, 195, 857, 0},
                {64, 512, 2976, 5368, 728, 546, 728, 574}, {64, 256, 1918, 4869, 372, 233, 733, 2},
                {64, 128, 3099, 1541, 270, 64, 748, 0}, {64, 64, 3285, 1105, 242, 15, 744, 0},
                {32, 64, 4032, 555, 191, 21, 871, 845}, {32, 32, 3499, 26, 120, 11, 944, 3073}};
  int64_t rows = 0;
  for (int i = 0; i < P.n_groups; ++i) rows += M(i);
  const int64_t steps = P.K / BK, weights_ns = P.weights * P.N * P.K * 2 / 4000, out_ns = rows * P.N * (P.c_f32 ? 4 : 2) / 4000;
  int64_t best = 0;
  for (const auto& t : kTiles) {
    int64_t tiles = 0;
    for (int i = 0; i < P.n_groups; ++i) tiles += ((int64_t)M(i) + t.bm - 1) / t.bm * ((P.N + t.bn - 1) / t.bn);
    const int64_t rounds = (tiles + n_cu - 1) / n_cu;
    const int64_t k_loop = steps * (rounds * t.step_round + tiles * t.step_tile / n_cu);
    const int64_t draw = weights_ns * (P.same_channels ? t.weights : 450) / 1000 - 5410;
    const int64_t cost = t.launch + rounds * t.round + std::max(k_loop, draw) + out_ns * t.out / 1000;
    if (best == 0 || cost < best) {
      best = cost;
      *bm = t.bm, *bn = t.bn;
    }
  }
  if (*bm == 256 && *bn == 256) *bm = *bn = 0;
  return best;
}

// bytes that an axis can span (the columns of B carry no index table: make_axis refuses it)
template <int ND>
int64_t axis_span(const AxisMap<ND>& a) {
  int64_t span = 0;
  for (int i = 0; i < ND; ++i) span += (int64_t)(a.radix[i].d - 1) * a.stride[i] * 2;
  return span;
}

}  // namespace

namespace vt {

// The estimate for one product of M rows with a [K,N] weight whose rows are `ldb` elements apart; 0: outside these tiles.
int64_t gemm_tile_estimate_ns(int64_t M, int64_t N, int64_t K, int64_t ldb) {
  if (K % BK || K < BK || K > kMaxSteps * BK || N < 8) return 0;
  int bm, bn;
  return choose_tile(TileWork{N, K, 1, 1, false, ldb * 2 % 4096 == 0}, [&](int) { return M; }, &bm, &bn);
}

// The product of P (operands planned, tiles not yet cut) on smaller tiles, or VT_ERR_UNSUPPORTED when
// the 256 x 256 kernel is the better one or the only one, or when the estimate is not below below_ns (if that is not 0).
int gemm_tile_launch(const GemmParams& P, const OutMap* O, int dtype, hipStream_t st, int64_t below_ns) {
  const char* no = "vt_gemm: outside the small-tile kernel";
  if (P.K % BK || P.K < BK || P.K > kMaxSteps * BK || P.N < 8) return fail(VT_ERR_UNSUPPORTED, no);
  for (int i = 0; i < P.n_groups; ++i) {
    const GemmGroup& g = P.g[i];
    if (!g.k64 || g.b_kmajor != P.g[0].b_kmajor) return fail(VT_ERR_UNSUPPORTED, no);
    // a lane's share of B's address is 32 bits
    const int64_t span = axis_span(g.b_col) + (g.b_kmajor ? 128 : 16 * g.b_row.stride[2] * 2 + 16);
    if (span >= (1ll << 32)) return fail(VT_ERR_UNSUPPORTED, no);
  }
  int bm = 0, bn = 0;
  TileWork w = {P.N, P.K, 0, P.n_groups, P.c_f32 != 0, !P.g[0].b_kmajor && P.g[0].b_row.stride[2] * 2 % 4096 == 0};
  for (int i = 0; i < P.n_groups; ++i) w.weights += i == 0 || P.g[i].b != P.g[i - 1].b;   // groups that are pieces of one A share their B
  const int64_t estimate_ns = choose_tile(w, [&](int i) { return P.g[i].M; }, &bm, &bn);
  if (below_ns && estimate_ns >= below_ns) return fail(VT_ERR_UNSUPPORTED, no);
  if (!bm) return fail(VT_ERR_UNSUPPORTED, no);
  const NoMap none;
  const bool km = P.g[0].b_kmajor != 0;
#define VT_TILE_T(TT)                                                                            \
  do {                                                                                           \
    if (O) return launch_tile<TT, false, true, false>(P, *O, bm, bn, st);                        \
    if (P.c_f32) return km ? launch_tile<TT, true, false, true>(P, none, bm, bn, st) : launch_tile<TT, true, false, false>(P, none, bm, bn, st); \
    return km ? launch_tile<TT, false, false, true>(P, none, bm, bn, st) : launch_tile<TT, false, false, false>(P, none, bm, bn, st);            \
  } while (0)
  if (dtype == VT_BF16) VT_TILE_T(bf16_t);
  else VT_TILE_T(f16_t);
#undef VT_TILE_T
}

}  // namespace vt
