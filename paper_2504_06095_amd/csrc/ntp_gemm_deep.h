// Deep-pipelined form of the GEMM kernel for problems with few output tiles: one workgroup per (output tile, K chunk), the
// whole LDS as a ring of STAGES K tiles (both operands of one K tile each), all but one of them in flight.
//
// What bounds these problems is the time from a DMA instruction to its data (1-2 us from HBM): the persistent kernels keep
// one to two K tiles in flight, so that a small problem pays that time once per K tile (512 x 586 x 1024: 16 K tiles, 21 us).
// Here a workgroup asks for STAGES - 1 K tiles before it waits for the first.  Smaller tiles also give the launch more
// workgroups, and the K axis is cut (k_splits) where there are still fewer of them than compute units.  A K tile takes 0.46-0.56 us
// (bound by LDS reads, 96 KB a K tile, and the barrier); with four wavefronts of 64 x 64 it is a third less LDS traffic and 20-50 %
// slower, because nothing overlaps a wavefront's reads.  512 x 586 x 1024: 16 -> 12 us; 1200 x 1712 x 3272: 46 -> 34 us.
//
// Per K tile: wait for this wavefront's share of it, one barrier (now it is complete, and every wavefront has read its
// fragments of the previous one), start the DMA of the K tile STAGES - 1 ahead into the previous one's slot, read all
// fragments, multiply.  Past the last K tile the schedule asks for the last one again (clamped index, slots nobody reads), so that the
// instruction counts that the waits rely on stay static.  LDS reads are inline assembly (see ntp_gemm_pp.h).
//
// (The two wavefronts of a SIMD alternating, one reading a whole K tile while the other one multiplies, from 20 K tiles on: over 170 random projections of 2 to
// 40 GFLOP 1.003 of the time with cold operands, shared launches 1.005 (0.98 to 1.04), and 0.996 with cached ones.  DMA instructions among the matrix instructions, in
// step: 0.92-1.06 of the time, no gain on the mean.  What is left, 0.45-0.5 us a K tile with all compute units at it, is the 32 KB that each of them asks its L2 for: 64 GB/s a unit.)
//
// K tail (K % 64): K-contiguous operands are read in chunks of 8, and chunks at k >= K are sent past the end of the buffer view, where
// loads read zeros; lines of a K-strided operand at k >= K lie past its end by themselves.  A chunk that K cuts must
// hold zeros from K on (the host sees to that: gemm_launch).
#ifndef NTP_GEMM_DEEP_H_
#define NTP_GEMM_DEEP_H_

#include "ntp_gemm_pp.h"

namespace ntp_gemm {

// Nothing that uses v moves ahead of this.
__device__ __forceinline__ void pin(bf16x8& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v)::"memory");
#endif
}

// One (output tile, K chunk): workgroup `block` of problem g, with the ring in `ring`.
template <bool AKC, bool BKC, int EPI, int BM_, int BN_, int WGM, int WGN, int STAGES>
__device__ __forceinline__ void deep_tile(const GemmArgs& g, const int block, uint16_t* const ring) {
  constexpr int NW = WGM * WGN;
  constexpr int TM = BM_ / WGM, TN = BN_ / WGN;  // wavefront tile
  constexpr int MI = TM / 16, NI = TN / 16;      // 16 x 16 accumulator blocks
  static_assert(TM % 16 == 0 && TN % 16 == 0, "wavefront tile: 16 x 16 blocks");
  constexpr int NAI = BM_ * DK * 2 / 1024 / NW, NBI = BN_ * DK * 2 / 1024 / NW;  // DMA instructions per K tile and wavefront
  static_assert((BM_ * DK * 2 / 1024) % NW == 0 && (BN_ * DK * 2 / 1024) % NW == 0, "operands split evenly over the wavefronts");
  constexpr int WAIT = (STAGES - 2) * (NAI + NBI);
  static_assert(STAGES >= 2 && WAIT <= 63, "the in-order counter holds 63 instructions");
  constexpr int SA = BM_ * DK, SB = BN_ * DK, STAGE = SA + SB;  // elements
  static_assert(STAGES * STAGE * 2 <= 160 * 1024, "LDS of a compute unit");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;

  const int nblk = g.tiles_m * g.tiles_n, per_split = (nblk + 7) & ~7;  // (keeps workgroup & 7 == tile & 7: the XCD)
  const int split = block / per_split, vblk = block - split * per_split;
  if (vblk >= nblk) return;  // padding workgroup (the whole workgroup leaves, before any barrier)
  const TilePos tp = place_tile(vblk, g.tiles_m, g.tiles_n);
  const int row0 = tp.tile_m * BM_, col0 = tp.tile_n * BN_;
  const int64_t k_first = int64_t(split) * g.k_chunk;
  const int K = min(g.k_chunk, g.K - int(k_first));
  const int nk = (K + DK - 1) / DK;

  const uint32_t a_shift = deep_view_shift(AKC, k_first, g.lda), b_shift = deep_view_shift(BKC, k_first, g.ldb);
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(g.A) + a_shift / 2, 0, int(g.a_extent - a_shift), 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(g.B) + b_shift / 2, 0, int(g.b_extent - b_shift), 0x00020000);
  const uint32_t astep_b = uint32_t(AKC ? DK : DK * g.lda) * 2, bstep_b = uint32_t(BKC ? DK : DK * g.ldb) * 2;
  FragAddr<AKC, BM_, MI> fra;
  FragAddr<BKC, BN_, NI> frb;
  fra.init(wm * TM, lane);
  frb.init(wn * TN, lane);

  // DMA offsets; in the K tail the chunks at k >= K go past every buffer view
  uint32_t offa[NAI], offb[NBI];
  bool cuta[NAI], cutb[NBI];
#pragma unroll
  for (int i = 0; i < NAI; ++i) {
    int line, chunk;
    slot_src<AKC, BM_>((wave * NAI + i) * 64 + lane, line, chunk);
    offa[i] = dma_offset<AKC>(g.lda, row0, g.M, line, chunk);
    cuta[i] = deep_cut<AKC>(nk, chunk, K);
  }
#pragma unroll
  for (int i = 0; i < NBI; ++i) {
    int line, chunk;
    slot_src<BKC, BN_>((wave * NBI + i) * 64 + lane, line, chunk);
    offb[i] = dma_offset<BKC>(g.ldb, col0, g.N, line, chunk);
    cutb[i] = deep_cut<BKC>(nk, chunk, K);
  }
  auto dma = [&](int t, int slot) {
    const int kt = min(t, nk - 1);
    const bool last = kt == nk - 1;
    uint16_t* const sa = ring + slot * STAGE + wave * NAI * 512;
    uint16_t* const sb = ring + slot * STAGE + SA + wave * NBI * 512;
#pragma unroll
    for (int i = 0; i < NAI; ++i) dma_issue(ra, sa + i * 512, last && cuta[i] ? kNowhere : offa[i], uint32_t(kt) * astep_b);
#pragma unroll
    for (int i = 0; i < NBI; ++i) dma_issue(rb, sb + i * 512, last && cutb[i] ? kNowhere : offb[i], uint32_t(kt) * bstep_b);
  };

  u16x4 aux[MI][NI];  // asked for before the first K tile: the epilogue finds them there
  if constexpr (EPI == ntp::EPI_DGELU) {
#pragma unroll
    for (int i = 0; i < MI; ++i) load_aux_row(g, row0 + wm * TM + i * 16 + (lane & 15), col0 + wn * TN + (lane >> 4) * 4, aux[i]);
    __builtin_amdgcn_sched_barrier(0);
  }
  f32x4 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const uint32_t ring0 = lds_addr(ring);
  if constexpr (BM_ > 64) {
    constexpr int RDS = MI * (AKC ? 1 : 2) + NI * (BKC ? 1 : 2);  // LDS reads of a K-step
    bf16x8 fa[2][MI], fb[2][NI];
    auto read_frags = [&](auto kss, uint32_t sa, uint32_t sb) {
      constexpr int ks = decltype(kss)::value;
      static_for(std::make_integer_sequence<int, MI>{}, [&](auto i) { fa[ks][decltype(i)::value] = frag_read_asm<AKC, BM_, MI, decltype(i)::value, ks>(fra, sa); });
      static_for(std::make_integer_sequence<int, NI>{}, [&](auto j) { fb[ks][decltype(j)::value] = frag_read_asm<BKC, BN_, NI, decltype(j)::value, ks>(frb, sb); });
    };
    auto multiply = [&](int ks) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
    };
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) dma(s, s);
    int slot = 0, free_slot = STAGES - 1;
    for (int t = 0; t < nk; ++t) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(WAIT));
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      const uint32_t sa = ring0 + uint32_t(slot) * (STAGE * 2), sb = sa + SA * 2;
      read_frags(Int<0>{}, sa, sb);
      __builtin_amdgcn_sched_barrier(0);
      dma(t + STAGES - 1, free_slot);
      __builtin_amdgcn_sched_barrier(0);
      read_frags(Int<1>{}, sa, sb);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(lgkm_imm(RDS <= 15 ? RDS : 15));
      __builtin_amdgcn_sched_barrier(0);
      multiply(0);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(lgkm_imm(0));
      __builtin_amdgcn_sched_barrier(0);
      multiply(1);
      __builtin_amdgcn_sched_barrier(0);
      free_slot = slot;
      slot = slot + 1 == STAGES ? 0 : slot + 1;
    }
  } else {
    // 64 x 64: four wavefronts with 8 matrix instructions each have too little to do to hide a K tile's LDS reads, so the fragments of
    // the next K tile are read under the products of the one in hand (weight gradients over K = 2048: 16.0 -> 14.0 us; on the larger
    // tiles, whose two wavefronts per SIMD hide each other's reads, it costs 0.5 us a launch)
    bf16x8 fa[2][2][MI], fb[2][2][NI];
    auto read_frags = [&](auto setc, uint32_t sa, uint32_t sb) {
      constexpr int set = decltype(setc)::value;
      static_for(std::make_integer_sequence<int, 2 * MI>{}, [&](auto ic) {
        constexpr int i = decltype(ic)::value % MI, ks = decltype(ic)::value / MI;
        fa[set][ks][i] = frag_read_asm<AKC, BM_, MI, i, ks>(fra, sa);
      });
      static_for(std::make_integer_sequence<int, 2 * NI>{}, [&](auto jc) {
        constexpr int j = decltype(jc)::value % NI, ks = decltype(jc)::value / NI;
        fb[set][ks][j] = frag_read_asm<BKC, BN_, NI, j, ks>(frb, sb);
      });
    };
    auto frags_arrived = [&](auto setc) {
      constexpr int set = decltype(setc)::value;
      __builtin_amdgcn_s_waitcnt(lgkm_imm(0));
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
        for (int i = 0; i < MI; ++i) pin(fa[set][ks][i]);
#pragma unroll
        for (int j = 0; j < NI; ++j) pin(fb[set][ks][j]);
      }
    };
#pragma unroll
    for (int s = 0; s < STAGES; ++s) dma(s, s);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(WAIT + NAI + NBI));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_frags(Int<0>{}, ring0, ring0 + SA * 2);
    frags_arrived(Int<0>{});
    int slot = 0;  // of the K tile in hand
    auto step = [&](auto setc, int t) {
      constexpr int set = decltype(setc)::value;
      const int next = slot + 1 == STAGES ? 0 : slot + 1;
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(WAIT));  // this wavefront's share of the next K tile has landed ...
      __builtin_amdgcn_s_barrier();                 // ... and everyone's; everyone has read the one in hand
      __builtin_amdgcn_sched_barrier(0);
      const uint32_t sa = ring0 + uint32_t(next) * (STAGE * 2);
      read_frags(Int<1 - set>{}, sa, sa + SA * 2);
      __builtin_amdgcn_sched_barrier(0);
      dma(t + STAGES, slot);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][ks][j], fa[set][ks][i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      frags_arrived(Int<1 - set>{});
      __builtin_amdgcn_sched_barrier(0);
      slot = next;
    };
    for (int t = 0; t < nk; t += 2) {
      step(Int<0>{}, t);
      if (t + 1 < nk) step(Int<1>{}, t + 1);
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // the clamped DMA instructions write LDS that this workgroup still owns

  if constexpr (EPI == ntp::EPI_F32_ACCUM) {
    if (g.k_splits == 1 && g.n_segs == 1) return accumulate_blocks<MI, NI>(g, row0 + wm * TM + (lane & 15), col0 + wn * TN + (lane >> 4) * 4, acc);
  }
  constexpr bool PAIRED = EPI == ntp::EPI_BF16 || EPI == ntp::EPI_GELU || EPI == ntp::EPI_DGELU;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int m = row0 + wm * TM + i * 16 + (lane & 15);
    if (g.k_splits > 1) {  // fp32 partial sums
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int n0 = col0 + wn * TN + j * 16 + (lane >> 4) * 4;
        if (m < g.M && n0 < g.n_store)
          *reinterpret_cast<f32x4*>(static_cast<float*>(g.C) + int64_t(split) * g.split_stride + int64_t(m) * g.ldc + n0) = acc[i][j];
      }
    } else if constexpr (PAIRED) {
      static_assert(NI % 2 == 0, "blocks are stored in pairs");
#pragma unroll
      for (int j = 0; j < NI; j += 2) store8_pair<EPI>(g, m, col0 + wn * TN + j * 16, lane >> 4, acc[i][j], acc[i][j + 1], aux[i][j], aux[i][j + 1]);
    } else {
#pragma unroll
      for (int j = 0; j < NI; ++j) store4<EPI>(g, m, col0 + wn * TN + j * 16 + (lane >> 4) * 4, acc[i][j]);
    }
  }
}

// The 64 x 64 form (48 KB; two workgroups on a compute unit at a time, see choose_deep) for launches that leave most of the device idle with 128 x 128: a K tile takes
// 0.225 us instead of 0.47 (16 DMA instructions, of which a compute unit takes one in 18 cycles, instead of 32), and there are four times as
// many workgroups, so that the K axis needs no cut and no second launch.  512 x 584 over K = 1024 13.5 -> 9.6 us, 512 x 1024 over 584
// 10.5 -> 8.0, 384 x 512 over 4096 in four chunks 18.9 -> 13.2.  Five K tiles in LDS are 0.3 us slower, seven 30 % where
// a compute unit has more than one workgroup to take.
template <bool AKC, bool BKC, int EPI, int BM_, int BN_, int WGM, int WGN, int STAGES>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_deep_kernel(const GemmArgs g) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[STAGES * (BM_ + BN_) * DK];
  deep_tile<AKC, BKC, EPI, BM_, BN_, WGM, WGN, STAGES>(g, int(blockIdx.x), ring);
}

// Up to three problems that do not depend on each other in one launch (the 128 x 128 tile with five K tiles in LDS or the 64 x 64 one, no cut K axis):
// a layer's small gradient GEMMs take 10-12 us each, of which launch, first loads and the last tiles' stores are the larger
// part, and leave most of the device idle.  512 x 1024 x 586: dB, dA and dX 34 -> 14 us.
constexpr int kMaxGroup = 3;
struct GroupArgs {
  GemmArgs g[kMaxGroup];
  int32_t kind[kMaxGroup];   // GroupKind
  int32_t first[kMaxGroup];  // first workgroup (a multiple of 8), ascending
  int32_t n;
};
enum GroupKind : int32_t { kGroupNt = 0, kGroupNn, kGroupTn, kGroupTnAccum };  // layout and epilogue: bf16, bf16, fp32, fp32 accumulate

template <int B, int WG, int STAGES>
__global__ __launch_bounds__(128 * WG) void gemm_deep_group_kernel(const GroupArgs a) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[STAGES * 2 * B * DK];
  int p = 0;
  for (int i = 1; i < a.n; ++i)
    if (int(blockIdx.x) >= a.first[i]) p = i;
  const GemmArgs& g = a.g[p];
  const int block = int(blockIdx.x) - a.first[p];
  switch (a.kind[p]) {
    case kGroupNt: deep_tile<true, true, ntp::EPI_BF16, B, B, 2, WG, STAGES>(g, block, ring); break;
    case kGroupNn: deep_tile<true, false, ntp::EPI_BF16, B, B, 2, WG, STAGES>(g, block, ring); break;
    case kGroupTn: deep_tile<false, false, ntp::EPI_F32, B, B, 2, WG, STAGES>(g, block, ring); break;
    default: deep_tile<false, false, ntp::EPI_F32_ACCUM, B, B, 2, WG, STAGES>(g, block, ring); break;
  }
}

}  // namespace ntp_gemm

#endif  // NTP_GEMM_DEEP_H_
