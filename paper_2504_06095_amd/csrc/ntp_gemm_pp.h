// Ping-pong form of the ring GEMM kernel (8 wavefronts).  Same tiles, slot layouts, DMA addressing
// and epilogues as gemm_ring_kernel (ntp_gemm_ring.h); what differs is who does what when in the K loop.
//
// The two wavefronts of a SIMD (w and w + 4: wavefronts are dealt to the four SIMDs in turn) alternate between
// two kinds of slot, with a workgroup barrier after every slot:
//   memory slot   read all fragments of one K-step (32 k) of the current K tile from LDS into registers and
//                 wait for them; where both operands are K-contiguous, DMA instructions of the long operand (below) behind the reads of the second one;
//   compute slot  MI x NI matrix instructions on those fragments, this wavefront's other DMA instructions evenly among them.
// Wavefronts 0-3 ("early") run M0 C0 M1 C1 per K tile, wavefronts 4-7 ("late") the same one slot behind, so
// in every slot one wavefront of each SIMD computes while the other one's LDS latency hides behind it.
//
// What bounds the loop is the longer of the two kinds of slot, then the board's power.  A compute slot is 448 cycles on a 256 x 224 tile.  With all DMA
// instructions in the memory slots these took 390 (M0) and 600-680 cycles (M1, which also held a prefetch to L2), 510 and 750-780 where both
// operands are K-strided; without them they take 210-250 (340-400), and a compute slot with four DMA instructions in it about 500: the vector memory
// path takes about 18 cycles per 1 KiB instruction and compute unit, and 16 of them in 448 cycles do not queue up.  M1 with the long operand's takes 310-410.  The prefetch (a
// 4-byte load per 128-byte line four K tiles ahead, by turns) cost a slot more than it brought to most products and is gone.  Whole GEMMs: use_pingpong in ntp_gemm.hip.  A K chunk,
// which ran on the ring kernel before: 8192 x 752 over K = 16384 in two chunks 207 -> 188 us, 4096 x 640 over 8192 in three 67.3 -> 60.4 (operands from HBM).
//
// Where the long operand's instructions go: with both operands K-contiguous the memory slots have room for them, and a compute slot is not held up by the vector memory
// path.  Twenty-five such products with cold operands take 0.990 of the time with them in M1 against the compute slots, cached 0.993 (2048 x 7040 over 12288 279.9 -> 272.9 us,
// 3024 x 3976 over 4488 109.4 -> 105.3, the other way 16384 x 1024 over 4096 102 -> 104.6); both operands' there 1.005 and 1.000, the short one's alone 1.011 and 1.005.  With one
// operand K-strided M1 and the compute slots are even, with both M1 takes 1.003 and 1.006.
// What the prefetch is missed for: rows that do not start on cache lines, in launches of one round of tiles with cold operands, up to 1.08 of the time that they took with it (2048 x
// 8264 over 1544 73.1 -> 78.7 us; cached 70.2 -> 62.8); rows of whole lines take 0.93 to 1.00, launches of more rounds 0.89 to 0.98.  Put back, one load a wavefront in M0 that is
// waited for a K tile later, it took 1.05 of the time cold and 1.10 cached over thirty shapes, and spilled registers on the widest tiles.
//
// LDS is a ring of five operand slots that runs on from one output tile of a persistent workgroup into the next.  Of the two operands one ("long", the
// one of more rows) is asked for two K tiles ahead, the other ("short") one to two.  While K tile t is multiplied the slots hold
//   long t, short t, long t+1, short t+1, long t+2;
// the last reader of tile t is the late group's M1, the fourth slot of the tile, after which its two slots take short t+2 and long t+3.
// Every wavefront moves an eighth of both operands:
//   early group: short t+1 in C0 of tile t (second slot), long t+2 in C1 (fourth), or M1 (third) where both operands are K-contiguous;
//   late group:  long t+2 in C0 of tile t (third slot), or M1 (fourth), short t+2 in C1 (first slot of tile t+1);
//   before the barrier that ends the fourth slot both wait for everything up to short t+1 (the instructions of long t+2 may stay in flight).
// After that barrier tile t+1 is complete in LDS.  What a K tile asks for past the output tile's last one are the first K tiles of the workgroup's next
// output tile, so that a tile switch is the epilogue alone; where there is none the loads lie past their view (zeros, no memory traffic), so that instruction
// counts stay static.
//
// K tail (K % 64): as in the deep-pipelined kernel, a K tile of its own through the ring.  Chunks at k >= K lie past the view in the last K tile and read as
// zeros (a chunk that K cuts holds zeros from K on: the host sees to that).
//
// LDS reads in the loop are inline assembly: the compiler then neither sees nor guards them (it would put a
// wait for every DMA in flight in front of each), and the waits above are the only ones.
#ifndef NTP_GEMM_PP_H_
#define NTP_GEMM_PP_H_

#include "ntp_gemm_ring.h"

namespace ntp_gemm {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// 32-bit LDS address of an object in shared memory
__device__ __forceinline__ uint32_t lds_addr(const void* p) { return uint32_t(reinterpret_cast<uintptr_t>(p)); }

// Fragment I (16 rows) of K-step KS of an operand slot, by inline-assembly LDS reads (see FragAddr for the layout).
// The caller waits for lgkmcnt before using the result.
template <bool KC, int R, int NF, int I, int KS>
__device__ __forceinline__ bf16x8 frag_read_asm(const FragAddr<KC, R, NF>& f, uint32_t slot_addr) {
#if !defined(__HIP_DEVICE_COMPILE__)
  // (the host pass only needs the signature: its compiler does not know the GPU's register constraints)
  return bf16x8{};
#else
  if constexpr (KC) {
    u32x4_t v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(slot_addr + f.o[KS] * 2u), "n"(I * 16 * DK * 2) : "memory");
    return __builtin_bit_cast(bf16x8, v);
  } else {
    u32x2_t lo, hi;
    const uint32_t a = slot_addr + f.o[I] * 2u;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(a), "n"(KS * 32 * R * 2) : "memory");
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(a), "n"(KS * 32 * R * 2 + 4 * R * 2) : "memory");
    const u32x4_t v = {lo[0], lo[1], hi[0], hi[1]};
    return __builtin_bit_cast(bf16x8, v);
  }
#endif
}

// one DMA instruction: 64 lanes x 16 bytes from the buffer view (lane offset voff + scalar offset soff) to 1 KiB of LDS at dst
__device__ __forceinline__ void dma_issue(__amdgpu_buffer_rsrc_t rsrc, uint16_t* dst, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)dst, 16, voff, soff, 0, 0);
}

// the same with the 32-bit LDS address of the destination
__device__ __forceinline__ void dma_issue_at(__amdgpu_buffer_rsrc_t rsrc, uint32_t dst, uint32_t voff, uint32_t soff) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)dst, 16, voff, soff, 0, 0);
#endif
}

template <int... Is, typename F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, Is...>, F&& f) {
  (f(Int<Is>{}), ...);
}

// SPLIT: the non-persistent form, one workgroup per unit of work.  The K axis is cut into g.k_splits
// chunks of g.k_chunk (a multiple of the K tile; the last chunk takes what is left).  The grid holds
// k_splits groups of round_up(tiles, 8) workgroups; group s computes every output tile over chunk s.
// With several chunks the fp32 partial sums go to slice s of a workspace (g.C + s * g.split_stride
// floats, rows of g.ldc); with one chunk the tile gets its normal epilogue.
template <bool AKC, bool BKC, int EPI, int BM_, int BN_, int WGM, int WGN, bool SPLIT = false>
__global__ __launch_bounds__(512) void gemm_pp_kernel(const GemmArgs g) {
  static_assert(!SPLIT || EPI == ntp::EPI_F32 || EPI == ntp::EPI_F32_ACCUM, "partial sums are stored as fp32");
  static_assert(WGM * WGN == 8, "wavefront w is paired with wavefront w + 4");
  constexpr int TM = BM_ / WGM, TN = BN_ / WGN;  // wavefront tile
  constexpr int MI = TM / 16, NI = TN / 16;      // 16 x 16 accumulator blocks
  static_assert(TM % 16 == 0 && TN % 16 == 0, "wavefront tile: 16 x 16 blocks");
  constexpr int RA = slot_rows(AKC, BM_), RB = slot_rows(BKC, BN_);
  static_assert(BM_ <= 256 && BN_ <= 256, "tile sides up to 256");
  constexpr int SLOT = (RA > RB ? RA : RB) * DK;
  constexpr bool LB = RB > RA;  // the long operand is B
  constexpr bool LKC = LB ? BKC : AKC, SKC = LB ? AKC : BKC;
  constexpr int RL = LB ? RB : RA, RS = LB ? RA : RB;
  // DMA instructions per K tile and wavefront for the long and the short operand
  constexpr int NL = RL * DK * 2 / 1024 / 8, NS = RS * DK * 2 / 1024 / 8;
  constexpr bool LMEM = AKC && BKC;  // the long operand's instructions in the second memory slot
  static_assert((RL * DK * 2 / 1024) % 8 == 0 && (RS * DK * 2 / 1024) % 8 == 0, "operands split evenly over the wavefronts");
  __shared__ __attribute__((aligned(1024))) uint16_t ring[5 * SLOT];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const bool late = wave >= 4;  // uniform within a wavefront

  // persistent workgroups, XCD-aware tile walk: as in gemm_ring_kernel, each XCD begun a round later than the one before
  const int nblk = g.tiles_m * g.tiles_n;
  auto place = [&](int v) {
    TilePos t = place_tile(rotate_walk(v, nblk), g.tiles_m, g.tiles_n);
    t.tile_m *= BM_;
    t.tile_n *= BN_;
    return t;  // first row and column
  };
  int vblk = blockIdx.x;
  int split = 0;
  if constexpr (SPLIT) {
    const int per_split = (nblk + 7) & ~7;  // keeps (workgroup index & 7) == (tile index & 7)
    split = blockIdx.x / per_split;
    vblk = blockIdx.x - split * per_split;
    if (vblk >= nblk) return;  // padding workgroup (the whole workgroup leaves, before any barrier)
  }
  // this workgroup's share of the K axis
  const int64_t k_first = SPLIT ? int64_t(split) * g.k_chunk : 0;
  const int K = SPLIT ? min(g.k_chunk, g.K - int(k_first)) : g.K;
  const int nk = (K + DK - 1) / DK;  // (three at least in the persistent form: use_pingpong in ntp_gemm.hip)
  TilePos pos = place(vblk);

  f32x4 acc[MI][NI];
  // range-checked buffer views of the operands (see gemm_ring_kernel)
  const uint32_t a_shift = deep_view_shift(AKC, k_first, g.lda), b_shift = deep_view_shift(BKC, k_first, g.ldb);
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(g.A) + a_shift / 2, 0, int(g.a_extent - a_shift), 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(g.B) + b_shift / 2, 0, int(g.b_extent - b_shift), 0x00020000);
  const __amdgpu_buffer_rsrc_t rl = LB ? rb : ra, rs = LB ? ra : rb;
  const int64_t ldl = LB ? g.ldb : g.lda, lds = LB ? g.lda : g.ldb;
  const int liml = LB ? g.N : g.M, lims = LB ? g.M : g.N;
  const uint32_t stepl = uint32_t(LKC ? DK : DK * ldl) * 2, steps = uint32_t(SKC ? DK : DK * lds) * 2;  // bytes per K tile
  FragAddr<AKC, RA, MI> fra;
  FragAddr<BKC, RB, NI> frb;
  fra.init(wm * TM, lane);
  frb.init(wn * TN, lane);

  // this wavefront's DMA offsets in the output tile at p
  uint32_t offl[NL], offs[NS];
  auto set_long = [&](const TilePos& p) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      int line, chunk;
      slot_src<LKC, RL>((wave * NL + i) * 64 + lane, line, chunk);
      offl[i] = dma_offset<LKC>(ldl, LB ? p.tile_n : p.tile_m, liml, line, chunk);
    }
  };
  auto set_short = [&](const TilePos& p) {
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      int line, chunk;
      slot_src<SKC, RS>((wave * NS + i) * 64 + lane, line, chunk);
      offs[i] = dma_offset<SKC>(lds, LB ? p.tile_m : p.tile_n, lims, line, chunk);
    }
  };
  // ... in its last K tile (of a ragged K), and where there is nothing more to ask for
  const bool cut = nk * DK > K;
  auto cut_long = [&](bool all) {
    if (!all && !cut) return;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      int line, chunk;
      slot_src<LKC, RL>((wave * NL + i) * 64 + lane, line, chunk);
      offl[i] = all ? kPastAll : pp_cut_offset<LKC>(offl[i], stepl, nk, line, chunk, K);
    }
  };
  auto cut_short = [&](bool all) {
    if (!all && !cut) return;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      int line, chunk;
      slot_src<SKC, RS>((wave * NS + i) * 64 + lane, line, chunk);
      offs[i] = all ? kPastAll : pp_cut_offset<SKC>(offs[i], steps, nk, line, chunk, K);
    }
  };
  // DMA instruction i of the K tile at scalar offset `at` into the slot at LDS address sl
  auto dma_long = [&](int i, uint32_t at, uint32_t sl) { dma_issue_at(rl, sl + uint32_t(wave * NL + i) * 1024u, offl[i], at); };
  auto dma_short = [&](int i, uint32_t at, uint32_t sl) { dma_issue_at(rs, sl + uint32_t(wave * NS + i) * 1024u, offs[i], at); };

  bf16x8 fa[MI], fb[NI];
  auto read_frags = [&](auto kss, uint32_t sa_addr, uint32_t sb_addr) {
    constexpr int ks = decltype(kss)::value;
    static_for(std::make_integer_sequence<int, MI>{}, [&](auto i) { fa[decltype(i)::value] = frag_read_asm<AKC, RA, MI, decltype(i)::value, ks>(fra, sa_addr); });
    static_for(std::make_integer_sequence<int, NI>{}, [&](auto j) { fb[decltype(j)::value] = frag_read_asm<BKC, RB, NI, decltype(j)::value, ks>(frb, sb_addr); });
  };
  // the matrix instructions of a K-step with `ND` DMA instructions evenly among them
  auto compute_slot = [&](auto nd, auto&& dma) {
    constexpr int ND = decltype(nd)::value, NM = MI * NI;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    static_for(std::make_integer_sequence<int, ND + 1>{}, [&](auto dc) {
      constexpr int d = decltype(dc)::value;
      // operands swapped so that each lane ends up with 4 consecutive columns of one row
#pragma unroll
      for (int n = d * NM / (ND + 1); n < (d + 1) * NM / (ND + 1); ++n)
        acc[n / NI][n % NI] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[n % NI], fa[n / NI], acc[n / NI][n % NI], 0, 0, 0);
      if constexpr (d < ND) {
        __builtin_amdgcn_sched_barrier(0);
        dma(d);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // LDS addresses of the slots: long t, short t, long t+1, short t+1, long t+2
  const uint32_t ring0 = lds_addr(ring);
  uint32_t s0 = ring0, s1 = s0 + SLOT * 2, s2 = s1 + SLOT * 2, s3 = s2 + SLOT * 2, s4 = s3 + SLOT * 2;
  bool more = false;
  TilePos npos = pos;
  auto pp_tile = [&](auto latec, int t) {
    constexpr bool LATE = decltype(latec)::value;
    const uint32_t atl = pp_scalar_offset(t + 2, nk, cut, more, stepl), ats = pp_scalar_offset(t + (LATE ? 2 : 1), nk, cut, more, steps);
    if (t + 3 >= nk) {
      // (before the reads: nothing but the wait stands between a read and the use of its registers)  What this K tile asks for is the output tile's last K tile, or past it
      if (t + 3 == nk) cut_long(false);
      if (t + 2 == nk) more ? set_long(npos) : cut_long(true);
      if (t + (LATE ? 3 : 2) == nk) cut_short(false);
      if (t + (LATE ? 2 : 1) == nk) more ? set_short(npos) : cut_short(true);
    }
    // M0
    __builtin_amdgcn_sched_barrier(0);
    read_frags(Int<0>{}, LB ? s1 : s0, LB ? s0 : s1);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(lgkm0_imm());
    __builtin_amdgcn_s_barrier();
    // C0
    if constexpr (!LATE) compute_slot(Int<NS>{}, [&](int i) { dma_short(i, ats, s3); });
    else if constexpr (LMEM) compute_slot(Int<0>{}, [](int) {});
    else compute_slot(Int<NL>{}, [&](int i) { dma_long(i, atl, s4); });
    __builtin_amdgcn_s_barrier();
    // M1
    __builtin_amdgcn_sched_barrier(0);
    read_frags(Int<1>{}, LB ? s1 : s0, LB ? s0 : s1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (LMEM) {
#pragma unroll
      for (int i = 0; i < NL; ++i) dma_long(i, atl, s4);
      __builtin_amdgcn_sched_barrier(0);
    }
    // late group: the tile's fourth slot
    if constexpr (LATE) __builtin_amdgcn_s_waitcnt(vmcnt_lgkm0_imm(NL));
    else __builtin_amdgcn_s_waitcnt(lgkm0_imm());
    __builtin_amdgcn_s_barrier();
    // C1
    if constexpr (LATE) compute_slot(Int<NS>{}, [&](int i) { dma_short(i, ats, s0); });
    else if constexpr (LMEM) compute_slot(Int<0>{}, [](int) {});
    else compute_slot(Int<NL>{}, [&](int i) { dma_long(i, atl, s4); });
    // early group: its C1 is the tile's fourth slot
    if constexpr (!LATE) __builtin_amdgcn_s_waitcnt(vmcnt_imm(NL));
    __builtin_amdgcn_s_barrier();
    const uint32_t u0 = s0, u1 = s1;
    s0 = s2;
    s1 = s3;
    s2 = s4;
    s3 = u0;
    s4 = u1;
  };

  // the first output tile's first DMA instructions: K tile 0 whole, long of K tile 1, and the late group's share of short of K tile 1
  set_long(pos);
  set_short(pos);
  if (SPLIT && nk == 1) {
    cut_long(false);
    cut_short(false);
  }
#pragma unroll
  for (int i = 0; i < NL; ++i) dma_long(i, 0, s0);
#pragma unroll
  for (int i = 0; i < NS; ++i) dma_short(i, 0, s1);
  if (SPLIT && nk <= 2) {
    cut_long(nk == 1);
    if (late || nk == 1) cut_short(nk == 1);
  }
#pragma unroll
  for (int i = 0; i < NL; ++i) dma_long(i, pp_scalar_offset(1, nk, cut, false, stepl), s2);
  if (late) {
#pragma unroll
    for (int i = 0; i < NS; ++i) dma_short(i, pp_scalar_offset(1, nk, cut, false, steps), s3);
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  __builtin_amdgcn_s_barrier();

  constexpr bool PAIRED = !SPLIT && (EPI == ntp::EPI_BF16 || EPI == ntp::EPI_GELU || EPI == ntp::EPI_DGELU);
  constexpr int NODD = NI & 1;
  while (true) {
    const int vnext = vblk + int(gridDim.x);
    more = !SPLIT && vnext < nblk;
    if (more) npos = place(vnext);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // Every wavefront passes 4 nk + 1 barriers in the loop: the late group one before its first slot, the
    // early group one after its last (nk is the same for the whole workgroup).
    if (late) {
      __builtin_amdgcn_s_barrier();
      for (int t = 0; t < nk; ++t) pp_tile(std::true_type{}, t);
    } else {
      for (int t = 0; t < nk; ++t) pp_tile(std::false_type{}, t);
      __builtin_amdgcn_s_barrier();
    }
    const int erow0 = pos.tile_m, ecol0 = pos.tile_n;
    vblk = vnext;
    pos = npos;
    __builtin_amdgcn_sched_barrier(0);  // the epilogue's memory instructions stay behind the loop's
    if constexpr (EPI == ntp::EPI_F32_ACCUM && NI <= 4) {  // (wider block rows would spill)
      if (g.n_segs == 1 && (!SPLIT || g.k_splits == 1)) {
        accumulate_blocks<MI, NI>(g, erow0 + wm * TM + (lane & 15), ecol0 + wn * TN + (lane >> 4) * 4, acc);
        if (!more) break;
        continue;
      }
    }
    u16x4 aux[2][NI];
    if constexpr (EPI == ntp::EPI_DGELU) load_aux_row(g, erow0 + wm * TM + (lane & 15), ecol0 + wn * TN + (lane >> 4) * 4, aux[0]);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int m = erow0 + wm * TM + i * 16 + (lane & 15);
      if constexpr (EPI == ntp::EPI_DGELU) {
        if (i + 1 < MI) load_aux_row(g, m + 16, ecol0 + wn * TN + (lane >> 4) * 4, aux[(i + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (PAIRED) {
#pragma unroll
        for (int j = 0; j + 1 < NI; j += 2) store8_pair<EPI>(g, m, ecol0 + wn * TN + j * 16, lane >> 4, acc[i][j], acc[i][j + 1], aux[i & 1][j], aux[i & 1][j + 1]);
      }
#pragma unroll
      for (int j = PAIRED ? NI - NODD : 0; j < NI; ++j) {
        const int n0 = ecol0 + wn * TN + j * 16 + (lane >> 4) * 4;
        if (SPLIT && g.k_splits > 1) {
          if (m < g.M && n0 < g.n_store)
            *reinterpret_cast<f32x4*>(static_cast<float*>(g.C) + int64_t(split) * g.split_stride + int64_t(m) * g.ldc + n0) = acc[i][j];
        } else {
          store4<EPI>(g, m, n0, acc[i][j], aux[i & 1][j]);
        }
      }
    }
    if (!more) break;
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // the last DMA instructions write LDS that this workgroup still owns
}

}  // namespace ntp_gemm

#endif  // NTP_GEMM_PP_H_
