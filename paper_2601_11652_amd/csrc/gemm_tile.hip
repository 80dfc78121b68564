// Dense projections of the verification step on LDS-staged output tiles.
//
// Both operands are fragment-packed (32 x 16 blocks in the lane order of gfx950's
// v_mfma_f32_32x32x16_bf16, 1 KiB contiguous per block), so one global_load_lds_dwordx4
// moves one fragment into LDS in exactly the order the waves read it back (each lane's
// 16 bytes at lane * 16: conflict-free ds_read_b128), without a trip through registers.
// Two kernels: gemm_tile_kernel up to 64 rows, where the weight stream is everything, and
// gemm_wave_kernel (one wave per SIMD, hand-scheduled) from 65 rows on.
//
// gemm_tile_kernel: a workgroup of WGM x WGN waves computes a (32 WGM MTW) x (32 WGN NTW)
// output tile, each wave a tile of MTW x NTW fragments; its A and W slices stream through a
// ring of ST LDS stages of KS K-steps, ST - 1 of them in flight while one is consumed.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace wisp {

// calls f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>) in order
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// the same for data read once (the weight stream): marked non-temporal, so the caches do
// not keep it at the expense of the activation slices that the other tiles re-read (measured
// on weight-heavy tiles: the weight stream runs about a third faster)
__device__ __forceinline__ void lds_dma16_stream(const void *src, const void *dst) {
  const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)dst);
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off nt" : : "v"(src), "s"(m0) : "memory", "m0");
}

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt in bits
// 3:0 and 15:14, expcnt 6:4 and lgkmcnt 11:8 left at their maxima)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

template <int WGM, int WGN, int MTW, int NTW, int KS, int ST, bool SW>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_tile_kernel(const uint16_t *__restrict__ A,
                                                        const uint16_t *__restrict__ W,
                                                        float *__restrict__ C, int M, int N, int K,
                                                        int ldc, int tiles_m, int tiles, int per_xcd,
                                                        int kc_split, SwigluOut sw) {
  constexpr int NW = WGM * WGN;               // waves
  constexpr int AF = WGM * MTW, BF = WGN * NTW;   // A / W fragments of the tile per K step
  constexpr int SF = (AF + BF) * KS;          // fragments per stage
  static_assert(SF % NW == 0, "every wave issues the same number of loads");
  constexpr int LPW = SF / NW;                // loads per wave per stage
  static_assert((ST - 2) * LPW < 64, "outstanding loads fit the counter");
  // one LDS object per stage: with distinct objects the compiler can tell that a stage's
  // in-flight loads do not alias the stage being read, and inserts no wait for them
  __shared__ __attribute__((aligned(1024))) uint4 lds0[SF][64];
  __shared__ __attribute__((aligned(1024))) uint4 lds1[SF][64];
  __shared__ __attribute__((aligned(1024))) uint4 lds2[SF][64];
  __shared__ __attribute__((aligned(1024))) uint4 lds3[SF][64];
  static_assert(ST >= 2 && ST <= 4, "stage ring of 2 to 4 buffers");
  auto stage = [&](auto b) -> uint4 (*)[64] {
    constexpr int B = decltype(b)::value;
    if constexpr (B == 0) return lds0;
    else if constexpr (B == 1) return lds1;
    else if constexpr (B == 2) return lds2;
    else return lds3;
  };

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int KF = K >> 4, MF = (M + 31) >> 5, NF = N >> 5;
  const int KC_all = KF / KS;                 // K chunks (K is a multiple of 16 KS)
  // Workgroups are dealt to the 8 XCDs in turn (id mod 8).  Each XCD takes a contiguous run
  // of per_xcd tiles, column-tile major, so the workgroups resident on one XCD share the
  // A row slices and W column slices of few tiles, which its L2 then serves; the mapping
  // only moves traffic between cache levels, results do not depend on it.
  // Work items are (K range, tile) pairs, K range major: an XCD's run mostly shares one K
  // range, i.e. one slice of A, in its L2.  K range z sums chunks [z kc_split, ...) into
  // its own fp32 partial C[z]; the consumer adds the partials in fixed order.
  const int v = (int)(blockIdx.x % 8u) * per_xcd + (int)(blockIdx.x / 8u);
  const int splits = (KC_all + kc_split - 1) / kc_split;
  if (v >= tiles * splits) return;
  const int z = v / tiles, t = v % tiles;
  const int tm = t % tiles_m, tn = t / tiles_m;
  const int kc0 = z * kc_split;
  const int KC = min(KC_all, kc0 + kc_split) - kc0;
  C += (int64_t)z * M * ldc;
  const int rb0 = tm * AF, nb0 = tn * BF;

  // this wave's loads of chunk c into stage buffer b: fragment f of the stage is A block
  // (f / KS, f % KS) for f < AF KS, else W block; fragments past the matrix edge re-read
  // the last block (their products land in rows / columns that are never stored)
  auto issue = [&](int c, auto b) {
    uint4 (*buf)[64] = stage(b);
#pragma unroll
    for (int t = 0; t < LPW; ++t) {
      const int f = wave * LPW + t;
      if (f < AF * KS) {
        const int rb = min(rb0 + f / KS, MF - 1), kb = (kc0 + c) * KS + f % KS;
        lds_dma16(A + ((int64_t)rb * KF + kb) * 512 + lane * 8, &buf[f][0]);
      } else {
        const int g = f - AF * KS;
        const int nb = min(nb0 + g / KS, NF - 1), kb = (kc0 + c) * KS + g % KS;
        lds_dma16_stream(W + ((int64_t)nb * KF + kb) * 512 + lane * 8, &buf[f][0]);
      }
    }
  };

  floatx16 acc[MTW][NTW];
#pragma unroll
  for (int i = 0; i < MTW; ++i)
#pragma unroll
    for (int j = 0; j < NTW; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // this wave's operands of the chunk in stage buffer b, read from LDS into registers
  auto read_ops = [&](auto b, uint4 (&a)[KS][MTW], uint4 (&w)[KS][NTW]) {
    uint4 (*buf)[64] = stage(b);
#pragma unroll
    for (int k = 0; k < KS; ++k) {
#pragma unroll
      for (int i = 0; i < MTW; ++i) a[k][i] = buf[(wm * MTW + i) * KS + k][lane];
#pragma unroll
      for (int j = 0; j < NTW; ++j) w[k][j] = buf[AF * KS + (wn * NTW + j) * KS + k][lane];
    }
  };
  auto products = [&](const uint4 (&a)[KS][MTW], const uint4 (&w)[KS][NTW]) {
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int j = 0; j < NTW; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a[k][i]), as_bf16x8(w[k][j]), acc[i][j],
                                                             0, 0, 0);
  };

  static_for<ST - 1>([&](auto sb) {
    if (sb.value < KC) issue(sb.value, sb);
  });
  // one step of the ring: chunk c sits in stage buffer B; the load of chunk c + ST - 1 goes
  // to buffer (B + ST - 1) % ST, freed by chunk c - 1.  With `guarded` false the caller
  // knows c + ST - 1 < KC (steady state), so the step has no conditions: with them the
  // compiler keeps the accumulators of the two paths in different registers and copies
  auto step = [&](int c, auto bc, auto guarded) {
    constexpr int B = decltype(bc)::value;
    constexpr bool G = decltype(guarded)::value;
    // chunk c's loads (this wave's) have landed once at most the later in-flight chunks'
    // remain; at the tail fewer chunks are in flight, so wait for all
    if (!G || c + ST - 2 < KC)
      wait_vmcnt<(ST - 2) * LPW>();
    else
      wait_vmcnt<0>();
    // every wave's loads of chunk c are in LDS, and every wave is done reading chunk c - 1
    // (its reads completed before its last products): a bare barrier, no memory fence
    __builtin_amdgcn_s_barrier();
    if (!G || c + ST - 1 < KC) issue(c + ST - 1, std::integral_constant<int, (B + ST - 1) % ST>{});
    // all of the stage's operands are read up front, so the reads of step k + 1 overlap the
    // products of step k
    uint4 a[KS][MTW], w[KS][NTW];
    read_ops(bc, a, w);
    products(a, w);
  };
  int c = 0;
  for (; c + 2 * ST - 2 < KC; c += ST) static_for<ST>([&](auto bc) { step(c + bc.value, bc, std::false_type{}); });
  for (; c < KC; c += ST)
    static_for<ST>([&](auto bc) {
      if (c + bc.value < KC) step(c + bc.value, bc, std::true_type{});
    });

  wait_vmcnt<0>();
  if constexpr (SW) {
    // gate/up projection with its weights packed by wisp_pack_gate_up: column fragment 2b
    // holds gate columns 32b .. 32b + 31 and fragment 2b + 1 the up columns of the same b,
    // so silu(gate) * up of column j = 32b + (lane % 32) pairs fragments 2b and 2b + 1 at
    // the same lane and accumulator element.  The tile's first fragment is even (BF is).
    static_assert(BF % 2 == 0, "gate/up fragment pairs stay inside one tile");
    auto emit = [&](int i, int nb_gate, const floatx16 &g, const floatx16 &u) {
      if (nb_gate >= NF) return;
      const int rbase = (rb0 + wm * MTW + i) * 32 + 4 * (lane >> 5);
      const int j = (nb_gate >> 1) * 32 + (lane & 31);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = rbase + 8 * (e >> 2) + (e & 3);
        if (row < M) sw.out[packed_off(row, j, sw.F)] = f2bf(silu_mul(g[e], u[e]));
      }
    };
    if constexpr (NTW % 2 == 0) {   // both fragments of a pair in this wave's registers
#pragma unroll
      for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int q = 0; q < NTW; q += 2) emit(i, nb0 + wn * NTW + q, acc[i][q], acc[i][q + 1]);
    } else {
      // one fragment per wave: wave wn + 1 (odd) holds the up half of wave wn's gate
      // fragment; it hands its accumulators over through LDS, one row fragment at a time
      static_assert(NTW == 1 && WGN % 2 == 0, "gate/up pairs across neighbouring waves");
      static_assert(WGM * (WGN / 2) * 16 * 64 * 4 <= SF * 1024, "the exchange fits one stage buffer");
      float *x = reinterpret_cast<float *>(&lds0[0][0]) + ((wm * (WGN / 2) + (wn >> 1)) * 16) * 64 + lane;
#pragma unroll
      for (int i = 0; i < MTW; ++i) {
        __syncthreads();   // every wave is done with the stage buffers / the previous round
        if (wn & 1) {
#pragma unroll
          for (int e = 0; e < 16; ++e) x[e * 64] = acc[i][0][e];
        }
        __syncthreads();
        if (!(wn & 1)) {
          floatx16 u;
#pragma unroll
          for (int e = 0; e < 16; ++e) u[e] = x[e * 64];
          emit(i, nb0 + wn, acc[i][0], u);
        }
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < MTW; ++i) {
    const int rbase = (rb0 + wm * MTW + i) * 32 + 4 * (lane >> 5);
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
      const int nb = nb0 + wn * NTW + j;
      if (nb >= NF) continue;
      const int col = nb * 32 + (lane & 31);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = rbase + 8 * (e >> 2) + (e & 3);
        if (row < M) C[(int64_t)row * ldc + col] = acc[i][j][e];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// One wave per SIMD: 4 waves (WM x WN) of a (32 WM MT) x (32 WN NT) output tile, for 65 rows
// and more.
//
// What bounds these shapes, and why the tile is cut this way (measured on the 8B and 70B
// projections at 171-4108 rows):
//  - Under full matrix load the clock is set by power (1.6-1.9 GHz with random data), so
//    energy counts as much as issue slots.  v_mfma_f32_16x16x32 runs at 15 % more clock than
//    v_mfma_f32_32x32x16 on the same data (1.85 against 1.61 GHz, 256 x 256 tiles, K 4096),
//    and one wave per SIMD with up to 256 accumulators reads an operand byte from LDS for
//    twice as many products as two waves with half-size tiles.
//  - With a single wave there is no second one to hide a stall, so the loop is scheduled by
//    hand: every product is followed by at most one LDS read or one LDS-direct load, the
//    operands of chunk c + 1 are read during the products of chunk c into a second register
//    set, and the wait and barrier of a chunk sit between its products.  A chunk of the 256
//    x 256 tile (64 products, 1024 cycles of matrix work per SIMD) takes 1190 cycles with
//    its loads and 1086 without them; 1278 with the same work in bursts between barriers.
//  - The loads (32 KiB per chunk and CU) come from L2 as long as the workgroups of one XCD
//    cover a compact block of tiles; see the tile order below.
// Operands swap places in the product (weights first), so lane l holds row l % 16 and four
// consecutive columns 4 (l / 16) .. + 3 of each 16 x 16 block: results leave as 16-byte
// stores and SwiGLU pairs stay inside the lane.
//
// The operand of a 16-row block and 32 K columns is four 256-byte runs of two packed
// fragments: lane l reads row l % 16, columns 8 (l / 16) .. + 7 (conflict-free).
// ---------------------------------------------------------------------------------------
constexpr int kWaveStages = 4;   // LDS stages of one 32-column K chunk each

// LDS-direct load as above, the global address as a scalar base plus a per-lane offset:
// no vector arithmetic between the products
template <bool STREAM>
__device__ __forceinline__ void lds_dma16_at(const void *base, uint32_t lane_off, uint32_t m0) {
  if constexpr (STREAM)
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 nt" : : "v"(lane_off), "s"(base), "s"(m0) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(lane_off), "s"(base), "s"(m0) : "memory", "m0");
}

// at most VM vector-memory operations outstanding, every LDS operation done
template <int VM>
__device__ __forceinline__ void wait_vm_lds() {
  static_assert(VM >= 0 && VM < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (7 << 4));
}

// Where the barrier and the memory operations sit among a chunk's P products: the barrier
// before product `bar`, then the R operand reads every `rs` products, the loads every `ds`
// products from `d0` on.
struct WaveSched {
  int bar, rs, d0, ds;
};
constexpr WaveSched wave_sched(int P, int R, int LPW) {
  const int bar = P >= 64 ? 16 : P >= 48 ? 8 : P >= 24 ? 4 : 2;
  const int rs = (P - 1 - bar) / R >= 2 ? 2 : 1;
  const int d0 = 3 < P ? 3 : 0;
  const int ds = (P - 1 - d0) / LPW > 0 ? (P - 1 - d0) / LPW : 1;
  return WaveSched{bar, rs, d0, ds};
}

// STREAM: weight loads marked non-temporal, for launches of one row tile (each weight is
// then read by one workgroup only; with several row tiles it costs 10-15 % because the
// other tiles' reads miss).  SW: SwiGLU (gate/up).
template <int WM, int WN, int MT, int NT, bool STREAM, bool SW>
__global__ __launch_bounds__(256, 1) void gemm_wave_kernel(const uint16_t *__restrict__ A,
                                                           const uint16_t *__restrict__ W, float *__restrict__ C,
                                                           int M, int N, int K, int ldc, int tiles_m, int tiles,
                                                           int per_xcd, int kc_split, SwigluOut sw) {
  static_assert(WM * WN == 4, "one wave per SIMD");
  constexpr int ST = kWaveStages;
  constexpr int AF = WM * MT, BF = WN * NT;     // A / W row blocks (32 rows) of the tile
  constexpr int SF = (AF + BF) * 2;             // fragments per stage
  constexpr int LPW = SF / 4;                   // fragments each wave loads per stage
  static_assert(SF % 4 == 0, "every wave issues the same number of loads");
  constexpr int MA = 2 * MT, NB = 2 * NT;       // 16-row blocks of the wave's tile
  constexpr int P = MA * NB, R = MA + NB;       // products and operand reads per chunk
  constexpr WaveSched S = wave_sched(P, R, LPW);
  constexpr int LB = S.bar > S.d0 ? (S.bar - S.d0 + S.ds - 1) / S.ds : 0;   // loads before the barrier
  constexpr int L0 = LPW - LB;                                              // and after it
  static_assert(LB < LPW && S.bar + S.rs * (R - 1) < P && S.d0 + S.ds * (LPW - 1) < P, "everything has a slot");
  static_assert((ST - 1) * LPW < 64, "outstanding loads fit the counter");
  __shared__ __attribute__((aligned(1024))) uint4 lds[ST * SF * 64];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int KF = K >> 4, MF = (M + 31) >> 5, NF = N >> 5;
  const int KC_all = KF / 2;                    // 32-column chunks
  // Work items are (K range, tile) pairs, K range major, dealt XCD-contiguously as in
  // gemm_tile_kernel, row tile fastest.  From 16 row tiles on they run through groups of 4 row
  // tiles: the 32 workgroups resident on one XCD then cover a block of about 4 x 8 tiles and
  // re-read each other's A and W slices in its L2 (calls of 4 layers at the 8B widths: 8210 rows
  // 15.4 -> 14.9 ms, 4108 rows 8.03 -> 7.98).  With fewer row tiles a ragged last group costs
  // more than that brings (1279 rows 3.69 -> 3.59 ms without groups, 1512 rows 2.84 -> 2.80;
  // 2060 rows the same).
  const int v = (int)(blockIdx.x % 8u) * per_xcd + (int)(blockIdx.x / 8u);
  const int splits = (KC_all + kc_split - 1) / kc_split;
  if (v >= tiles * splits) return;
  const int z = v / tiles, t = v % tiles;
  const int gm = tiles_m >= 16 ? 4 : tiles_m;
  const int tiles_n = tiles / tiles_m;
  const int g0 = t / (gm * tiles_n) * gm, gr = min(gm, tiles_m - g0), tg = t - g0 * tiles_n;
  const int tm = g0 + tg % gr, tn = tg / gr;
  const int kc0 = z * kc_split;
  const int KC = min(KC_all, kc0 + kc_split) - kc0;
  C += (int64_t)z * M * ldc;
  const int rb0 = tm * AF, nb0 = tn * BF;

  // this wave's fragments of a stage: fragment f is row block f / 2 (A's, then W's) at K step
  // f % 2; row blocks past the matrix edge re-read the last one (their products are never
  // stored)
  const uint32_t lane_off = lane * 16;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)lds;
  constexpr uint32_t SB = SF * 1024;
  const char *src[LPW];
#pragma unroll
  for (int r = 0; r < LPW; ++r) {
    const int f = wave * LPW + r, b = f >> 1;
    const uint16_t *base = b < AF ? A + (int64_t)min(rb0 + b, MF - 1) * KF * 512
                                  : W + (int64_t)min(nb0 + b - AF, NF - 1) * KF * 512;
    src[r] = reinterpret_cast<const char *>(base + ((int64_t)kc0 * 2 + (f & 1)) * 512);
  }
  // load r of the wave's next chunk into the stage at LDS byte `stage`
  auto issue = [&](int r, uint32_t stage) {
    const int f = wave * LPW + r;
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(stage + f * 1024);
    if constexpr (STREAM) {
      if (f < AF * 2) lds_dma16_at<false>(src[r], lane_off, m0);
      else lds_dma16_at<true>(src[r], lane_off, m0);
    } else {
      lds_dma16_at<false>(src[r], lane_off, m0);
    }
    src[r] += 2048;
  };

  floatx4 acc[MA][NB];
#pragma unroll
  for (int i = 0; i < MA; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  const uint32_t lo = (lane >> 4) * 32 + (lane & 15);
  uint4 a[2][MA], w[2][NB];
  // operand read q of a chunk in order of first use: W blocks, then A blocks
  auto read = [&](auto bufc, auto qc, uint32_t s) {
    constexpr int B = decltype(bufc)::value, q = decltype(qc)::value;
    if constexpr (q < NB)
      w[B][q] = lds[s * (SF * 64) + AF * 128 + (wn * NT + (q >> 1)) * 128 + (q & 1) * 16 + lo];
    else
      a[B][q - NB] = lds[s * (SF * 64) + (wm * MT + ((q - NB) >> 1)) * 128 + ((q - NB) & 1) * 16 + lo];
  };

  // chunks 0 .. ST - 2 and the first L0 loads of chunk ST - 1, as chunk -1 would have issued;
  // a K range of fewer than ST chunks is filled up with zeros
  const bool full = KC >= ST;
#pragma unroll
  for (int s = 0; s < ST; ++s) {
    if (s < KC) {
#pragma unroll
      for (int r = 0; r < (s == ST - 1 ? L0 : LPW); ++r) issue(r, lds0 + s * SB);
    } else {
#pragma unroll
      for (int r = 0; r < LPW; ++r) lds[(s * SF + wave * LPW + r) * 64 + lane] = make_uint4(0, 0, 0, 0);
    }
  }
  if (full) wait_vm_lds<(ST - 2) * LPW + L0>();
  else wait_vm_lds<0>();
  __builtin_amdgcn_s_barrier();
  static_for<R>([&](auto q) { read(std::integral_constant<int, 0>{}, q, 0); });
  __builtin_amdgcn_sched_barrier(0);

  // One chunk from stage st with its operands in register set B.  kSteady: chunk c + ST
  // exists; kDrain: chunk c + ST - 1 is the last; kTail: nothing left to load; kLast: the last
  // chunk.  Before the barrier the rest of chunk c + ST - 1 is loaded into the stage freed
  // by chunk c - 1; at the barrier every wave's part of chunk c + 1 has landed and every
  // wave holds chunk c in registers, so the first loads of chunk c + ST may overwrite stage st.
  constexpr int kSteady = 0, kDrain = 1, kTail = 2, kLast = 3;
  uint32_t st = 0;
  auto chunk = [&](auto modec, auto bufc) {
    constexpr int MODE = decltype(modec)::value, B = decltype(bufc)::value;
    const uint32_t nst = st + 1 == ST ? 0 : st + 1, pst = st == 0 ? ST - 1 : st - 1;
    static_for<P>([&](auto nc) {
      constexpr int n = decltype(nc)::value;
      if constexpr (n == S.bar && MODE != kLast) {
        wait_vm_lds<MODE == kTail ? 0 : (ST - 2) * LPW>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      constexpr int i = n / NB, j = n % NB;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w[B][j]), as_bf16x8(a[B][i]), acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (MODE != kLast && n >= S.bar && (n - S.bar) % S.rs == 0 && (n - S.bar) / S.rs < R)
        read(std::integral_constant<int, B ^ 1>{}, std::integral_constant<int, (n - S.bar) / S.rs>{}, nst);
      if constexpr (n >= S.d0 && (n - S.d0) % S.ds == 0 && (n - S.d0) / S.ds < LPW) {
        constexpr int d = (n - S.d0) / S.ds;
        if constexpr (d < LB) {
          if constexpr (MODE == kSteady) issue(L0 + d, lds0 + pst * SB);
          if constexpr (MODE == kDrain) {
            if (full) issue(L0 + d, lds0 + pst * SB);
          }
        } else {
          if constexpr (MODE == kSteady) issue(d - LB, lds0 + st * SB);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    st = nst;
  };
  constexpr std::integral_constant<int, 0> b0;
  constexpr std::integral_constant<int, 1> b1;
  constexpr std::integral_constant<int, kSteady> steady;
  constexpr std::integral_constant<int, kDrain> drain;
  constexpr std::integral_constant<int, kTail> tail;
  constexpr std::integral_constant<int, kLast> last;
  int c = 0;
  if ((KC & 1) && KC > ST) {   // an odd count starts with one chunk on its own (KC >= ST + 1)
    chunk(steady, b0);
#pragma unroll
    for (int i = 0; i < MA; ++i) a[0][i] = a[1][i];
#pragma unroll
    for (int j = 0; j < NB; ++j) w[0][j] = w[1][j];
    c = 1;
  }
  for (; c + ST < KC; c += 2) {   // the register sets alternate: two chunks per turn
    chunk(steady, b0);
    chunk(steady, b1);
  }
  chunk(drain, b0);   // the last ST = 4 chunks
  chunk(tail, b1);
  chunk(tail, b0);
  chunk(last, b1);

  const int row_w = (rb0 + wm * MT) * 32 + (lane & 15);   // + 16 i
  if constexpr (SW) {
    // 16-column blocks 4q, 4q + 1 of the wave hold gate columns, 4q + 2, 4q + 3 the up columns
    // of the same model columns (weights packed by wisp_pack_gate_up)
    static_assert(NT % 2 == 0, "gate/up pairs stay inside one wave");
#pragma unroll
    for (int i = 0; i < MA; ++i) {
      const int row = row_w + 16 * i;
      if (row >= M) continue;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        if (j & 2) continue;
        const int nb = nb0 + wn * NT + (j >> 1);          // gate fragment
        if (nb >= NF) continue;
        const floatx4 g = acc[i][j], u = acc[i][j + 2];
        const int col = (nb >> 1) * 32 + (j & 1) * 16 + 4 * (lane >> 4);
        uint2 o;
        o.x = pack2bf(silu_mul(g[0], u[0]), silu_mul(g[1], u[1]));
        o.y = pack2bf(silu_mul(g[2], u[2]), silu_mul(g[3], u[3]));
        *reinterpret_cast<uint2 *>(sw.out + packed_off(row, col, sw.F)) = o;
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < MA; ++i) {
    const int row = row_w + 16 * i;
    if (row >= M) continue;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int nb = nb0 + wn * NT + (j >> 1);
      if (nb >= NF) continue;
      *reinterpret_cast<floatx4 *>(C + (int64_t)row * ldc + nb * 32 + (j & 1) * 16 + 4 * (lane >> 4)) = acc[i][j];
    }
  }
}

template <int WM, int WN, int MT, int NT, bool STREAM>
static void launch_wave_as(const uint16_t *A, const uint16_t *W, float *C, int M, int N, int K, int ldc, hipStream_t s,
                           int kc_split, SwigluOut sw) {
  const int tiles_m = ((M + 31) / 32 + WM * MT - 1) / (WM * MT);
  const int tiles_n = (N / 32 + WN * NT - 1) / (WN * NT);
  const int splits = (K / 32 + kc_split - 1) / kc_split;
  const int tiles = tiles_m * tiles_n, per_xcd = (tiles * splits + 7) / 8;
  auto go = [&](auto kernel) {
    launch(kernel, 8 * per_xcd, 256, 0, s, A, W, C, M, N, K, ldc, tiles_m, tiles, per_xcd, kc_split, sw);
  };
  if (sw.out) go(gemm_wave_kernel<WM, WN, MT, NT, STREAM, true>);
  else go(gemm_wave_kernel<WM, WN, MT, NT, STREAM, false>);
}

template <int WM, int WN, int MT, int NT>
static void launch_wave(const uint16_t *A, const uint16_t *W, float *C, int M, int N, int K, int ldc, hipStream_t s,
                        int kc_split, SwigluOut sw) {
  if (M <= 32 * WM * MT)
    launch_wave_as<WM, WN, MT, NT, true>(A, W, C, M, N, K, ldc, s, kc_split, sw);
  else
    launch_wave_as<WM, WN, MT, NT, false>(A, W, C, M, N, K, ldc, s, kc_split, sw);
}

template <int WGM, int WGN, int MTW, int NTW, int KS, int ST>
static void launch_tile(const uint16_t *A, const uint16_t *W, float *C, int M, int N, int K, int ldc,
                        hipStream_t s, int kc_split, SwigluOut sw) {
  const int tiles_m = ((M + 31) / 32 + WGM * MTW - 1) / (WGM * MTW);
  const int tiles_n = (N / 32 + WGN * NTW - 1) / (WGN * NTW);
  const int KC = K / (16 * KS);
  const int splits = (KC + kc_split - 1) / kc_split;
  const int tiles = tiles_m * tiles_n, per_xcd = (tiles * splits + 7) / 8;
  if (sw.out)
    launch(gemm_tile_kernel<WGM, WGN, MTW, NTW, KS, ST, true>, 8 * per_xcd, 64 * WGM * WGN, 0, s, A, W, C, M,
           N, K, ldc, tiles_m, tiles, per_xcd, kc_split, sw);
  else
    launch(gemm_tile_kernel<WGM, WGN, MTW, NTW, KS, ST, false>, 8 * per_xcd, 64 * WGM * WGN, 0, s, A, W, C, M,
           N, K, ldc, tiles_m, tiles, per_xcd, kc_split, sw);
}

// Tile shapes.  65 rows and more: the one-wave-per-SIMD kernel.  At 33-64 rows 64 x 128 tiles
// of 8 waves with single-fragment wave tiles; at most 32 rows a 32 x 256 tile of 4 waves with
// a deep K split.  At these row counts the activation slice and the fp32 partials are small
// next to the weights, so the loads are almost all weights.
TileShape tile_shape(int variant) {
  switch (variant) {
    case 1: return {192, 128, 2, 512};
    case 4: return {192, 256, 2, 128};
    case 7: return {128, 128, 2, 512};
    case 8: return {128, 256, 2, 512};
    case 13: return {256, 128, 2, 256};
    case 17: return {256, 256, 2, 128};
    case 5: return {32, 256, 4, 512};
    case 6: return {64, 128, 4, 512};
  }
  return {0, 0, 0, 0};
}

void gemm_bf16_tile(const uint16_t *A, const uint16_t *W, float *C, int M, int N, int K, int ldc, int variant,
                    int kc_split, hipStream_t s, SwigluOut sw) {
  switch (variant) {
    case 1: launch_wave<2, 2, 3, 2>(A, W, C, M, N, K, ldc, s, kc_split, sw); break;
    case 4: launch_wave<2, 2, 3, 4>(A, W, C, M, N, K, ldc, s, kc_split, sw); break;
    case 7: launch_wave<2, 2, 2, 2>(A, W, C, M, N, K, ldc, s, kc_split, sw); break;
    case 8: launch_wave<2, 2, 2, 4>(A, W, C, M, N, K, ldc, s, kc_split, sw); break;
    case 13: launch_wave<2, 2, 4, 2>(A, W, C, M, N, K, ldc, s, kc_split, sw); break;
    case 17: launch_wave<2, 2, 4, 4>(A, W, C, M, N, K, ldc, s, kc_split, sw); break;
    case 5: launch_tile<1, 4, 1, 2, 4, 4>(A, W, C, M, N, K, ldc, s, kc_split, sw); break;   // 4 waves
    case 6: launch_tile<2, 4, 1, 1, 4, 4>(A, W, C, M, N, K, ldc, s, kc_split, sw); break;
  }
}

}  // namespace wisp
