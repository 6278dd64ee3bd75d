// Backward kernels of the attention core with 32 owned rows per wavefront (head dimension 128).
//
// With 16 owned rows every fragment read from LDS feeds one matrix instruction, and the LDS (256 bytes per cycle and compute
// unit) is busy longer than the matrix pipe.  32 rows halve the reads, but dK and dV of 32 keys, their key and value
// fragments and two sets of scores are 350 registers: one wavefront per SIMD, so that nothing else overlaps one
// wavefront's softmax with another's products.  The overlap is written out instead: a walk goes in halves of 32 rows, and
// while the vector unit works on the scores of one half the matrix pipe computes those of the next, in slots of one
// matrix instruction with the LDS reads (16 slots ahead of their use), the DMA (up to three tile pairs ahead, a ring of four) and
// the vector instructions dealt out over them.  One barrier per 64 rows.
//
// What bounds them: the issue port of the one wavefront (a loop of nothing but such slots: 8 cycles a matrix instruction, 4.6 a
// vector one, 8.6 an exponential, about 5 an LDS read: 2400 cycles per 128 keys x 64 query rows of dK/dV, where the matrix pipe
// needs 2048; measured in the kernel 3100), and in long launches the clock, which the power limit holds near 2.05 GHz.
// 32x32x16 instructions need 12 % fewer cycles but the clock falls to 1.75 GHz: 1450 against 1360 us.
// 14 heads x 8192 tokens, unmasked, forward excluded: 1583 -> 1275 us (760 -> 943 TFLOP/s of the five products).
#pragma once

// (included by ntp_attn_core.hip, inside its unnamed namespace)

constexpr int kWideRing = 4;                      // tile pairs in the LDS ring
constexpr uint32_t kWideBuf = 2 * kDmaTile * 2;   // bytes of one: two 64-row tiles
// Behind the ring of the dK/dV walk: zeros where the immediate offsets of the transposed reads (multiples of 4 KB below kWideBuf) lead from
// the ring's end, 16 bytes each, and behind the first four of them the row values of the four buffers.
constexpr uint32_t kWideStep = 4096;
constexpr uint32_t kWideLds = kWideRing * kWideBuf + kWideBuf - kWideStep + 16;  // bytes
static_assert(16 + 4 * kBKV * 4 <= kWideStep && kWideRing * kWideStep <= kWideBuf && kWideLds <= 160 * 1024, "LDS of the dK/dV walk");

// f is called with 0 .. N - 1 as compile-time constants
template <int N, typename F, int... I>
__device__ __forceinline__ void unrolled_(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  unrolled_<N>(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

// At most N later LDS reads are in flight, so the reads into f have arrived; `with` names more registers of which that is
// known (see lds_reads_done).
template <int N, typename V>
__device__ __forceinline__ void arrived(V& a, V& b, V& c, V& d) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(N) : "memory");
#endif
}
template <typename V>
__device__ __forceinline__ void with(V& a, V& b, V& c, V& d) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d)::"memory");
#endif
}
template <typename V>
__device__ __forceinline__ void with(V& a, V& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(a), "+v"(b)::"memory");
#endif
}
template <int N>
__device__ __forceinline__ void wait_dma() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}

__device__ __forceinline__ void lds_stored() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#endif
}

// One matrix instruction with the registers where these kernels want them (the compiler, left to itself, moves
// accumulators between the two halves of the register file in the loop): scores in vector registers, owned operands and
// gradient sums in accumulation registers.  The compiler does not know an instruction in assembly as a matrix
// instruction, so the distances that the hardware leaves to the program are kept here (and checked in the compiler's output by
// tests/test_host_attn_schedule.py).  A vector instruction reads a result 16 matrix instructions after its last one at the earliest, but for the
// first half of a walk, before which scores_settle waits.  Packed weights, which two wait states must follow, are ready (operand_ready) a
// whole slot, at least a matrix instruction and an LDS read, before the one that reads them.  What an accumulator starts from
// (mfma_from) comes from LDS or from before the loop and is not overwritten for 16 matrix instructions more.
__device__ __forceinline__ void mfma_zero(f32x4& d, const attn_u32x4& x, const attn_u32x4& own) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(x), "a"(own));
#endif
}
__device__ __forceinline__ void mfma_from(f32x4& d, const attn_u32x4& x, const attn_u32x4& own, const f32x4& c) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(x), "a"(own), "v"(c));
#endif
}
__device__ __forceinline__ void mfma_score(f32x4& d, const attn_u32x4& x, const attn_u32x4& own) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(x), "a"(own));
#endif
}
__device__ __forceinline__ void mfma_grad(f32x4& d, const attn_u32x2& lo, const attn_u32x2& hi, const attn_u32x4& w) {
#if defined(__HIP_DEVICE_COMPILE__)
  const attn_u32x4 both = {lo[0], lo[1], hi[0], hi[1]};
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(both), "v"(w));
#endif
}
// two fp32 values as a pair of bf16
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  bf16x2_t v;
  v[0] = static_cast<__bf16>(lo);
  v[1] = static_cast<__bf16>(hi);
  return __builtin_bit_cast(uint32_t, v);
}
// What the vector unit makes for a matrix instruction is computed by here.
template <typename V>
__device__ __forceinline__ void operand_ready(V& w) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(w));
#endif
}
// Scores may be read by vector instructions after this.
__device__ __forceinline__ void scores_settle(f32x4 (&s)[2][2], f32x4 (&p)[2][2]) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 15" : "+v"(s[0][0]), "+v"(s[0][1]), "+v"(s[1][0]), "+v"(s[1][1]), "+v"(p[0][0]), "+v"(p[0][1]), "+v"(p[1][0]), "+v"(p[1][1]));
#endif
}
// The owned operands are in place before the first matrix instruction reads them
__device__ __forceinline__ void owned_ready(attn_u32x4 (&own)[2][4]) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int b = 0; b < 2; ++b) asm volatile("s_nop 1" : "+a"(own[b][0]), "+a"(own[b][1]), "+a"(own[b][2]), "+a"(own[b][3]));
#endif
}
// the last matrix instructions' results may be read after this
__device__ __forceinline__ void acc_settle(f32x4 (&acc)[8][2]) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int d = 0; d < 8; ++d) asm volatile("s_nop 15" : "+a"(acc[d][0]), "+a"(acc[d][1]));
#endif
}
__device__ __forceinline__ void zero_acc(f32x4 (&acc)[8][2]) {
#pragma unroll
  for (int d = 0; d < 8; ++d)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[d][b] = f32x4{0.f, 0.f, 0.f, 0.f};
}
// eight bf16 values with their signs flipped
__device__ __forceinline__ attn_u32x4 negated(const attn_u32x4& v) { return v ^ 0x80008000u; }

// Read addresses of a wavefront in buffer 0 of the ring: ak[s], the rows' (lane % 16) columns 32 s + 8 (lane / 16) ..; at[b],
// transposed, the rows 4 (lane / 16) .. + 3 of column 16 b + lane % 16.  Other rows (multiples of 16) are immediates.
__device__ __forceinline__ void transposed_addresses(uint32_t base, int lane, uint32_t (&at)[8]) {
  const int lq = lane & 15, lh = lane >> 4, rv = lh * 4 + (lq >> 2);
#pragma unroll
  for (int b = 0; b < 8; ++b) at[b] = base + uint32_t(rv) * 256u + uint32_t(lq & 1) * 8u + ((uint32_t(b * 2 + ((lq & 3) >> 1)) ^ row_swz(rv)) * 16u);
}
__device__ __forceinline__ void wide_addresses(const uint16_t* ring, int lane, uint32_t (&ak)[4], uint32_t (&at)[8]) {
  const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>(ring));
  const int lq = lane & 15, lh = lane >> 4;
#pragma unroll
  for (int s = 0; s < 4; ++s) ak[s] = base + uint32_t(lq) * 256u + ((uint32_t(s * 4 + lh) ^ row_swz(lq)) * 16u);
  transposed_addresses(base, lane, at);
}
// Bytes from the start of a tile in memory to what this lane's part of DMA instruction j of a wavefront brings: LDS chunk
// (4 wave + j) 64 + lane of the tile.
__device__ __forceinline__ void wide_dma_offsets(int64_t ld, int wave, int lane, uint32_t (&voff)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int p = (wave * 4 + j) * 64 + lane;
    const int row = p >> 4, slot = p & 15;
    voff[j] = uint32_t((int64_t(row) * ld + int64_t(uint32_t(slot) ^ row_swz(row)) * 8) * 2);
  }
}

// Stores a wavefront's 32 x 128 sums as bf16 rows: through 8 KB of LDS of its own, so that an instruction stores four whole rows (straight
// from the registers it would store 32 bytes of 16 rows: 64 KB of a workgroup took 10 400 cycles, 5 us).
__device__ __forceinline__ void store_wide_rows(const f32x4 (&acc)[8][2], float factor, uint16_t* lds, uint16_t* dst, int64_t ld, int rows, int lane) {
  const int lq = lane & 15, lh = lane >> 4;
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      u16x4 o;
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = ntp_gemm::f32_to_bf16(acc[b][rb][r] * factor);
      *reinterpret_cast<u16x4*>(lds + (rb * 16 + lq) * 128 + ((b * 2 + (lh >> 1)) ^ lq) * 8 + (lh & 1) * 4) = o;
    }
  lds_stored();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = i * 4 + lh;
    const attn_u32x4 v = *reinterpret_cast<const attn_u32x4*>(lds + row * 128 + (lq ^ (row & 15)) * 8);
    if (row < rows) *reinterpret_cast<attn_u32x4*>(dst + row * ld + lq * 8) = v;
  }
}

// Workgroup number `place` of a section of a launch -> (sequence, head) sh, 128-row tile and part.  Without the mask a section is
// all of a kernel's tiles.  Under it the walks run from 2 to all 64-row tiles, so that a kernel's workgroups go out in two
// sections, the longer half of the walks first (SHORT false) and then the shorter half, its longest first; within a
// section the walks of a head become shorter, and an XCD gets a contiguous eighth of the heads' pairs of a long and a short
// walk in both (see xcd_major).  False: no workgroup (the sections are rounded up to 8, and the middle tile of an odd
// number has no short partner).  long_first: tile 0 has the longest walk (dK/dV), otherwise the last one.
__device__ __forceinline__ bool wide_place(const CoreBwdArgs& a, uint32_t place, bool is_short, bool tile0_longest, uint32_t n_sh, int& sh, int& tile, int& part) {
  const uint32_t tiles2 = uint32_t(a.tiles + 1) / 2, per_sh = a.causal ? (tiles2 + 1) / 2 : tiles2;
  const uint32_t total = n_sh * per_sh * uint32_t(a.n_parts), x = place & 7, q = total >> 3, r = total & 7;
  const uint32_t first = x * q + (x < r ? x : r), count = q + (x < r ? 1 : 0);
  uint32_t n = place >> 3;
  if (n >= count) return false;
  n = first + (is_short ? count - 1 - n : n);
  part = int(n % uint32_t(a.n_parts));
  n /= uint32_t(a.n_parts);
  const uint32_t u = n % per_sh, other = tiles2 - 1 - u;
  sh = int(n / per_sh);
  if (is_short && other == u) return false;
  tile = int(!a.causal || tile0_longest != is_short ? u : other);
  return true;
}

__device__ __forceinline__ void bwd_dkv_wide_body(const CoreBwdArgs& a, uint32_t place, bool is_short, uint16_t* ring) {
  constexpr int D = 128;
  int sh, kt, part;
  if (!wide_place(a, place, is_short, true, uint32_t(a.n_seq) * uint32_t(a.kv_cnt), sh, kt, part)) return;
  const int seq = sh % a.n_seq, g = sh / a.n_seq;  // g: local KV head
  const int S = a.seq_len;
  const int64_t tok0 = int64_t(seq) * S, Mtot = int64_t(a.n_seq) * S;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 15, lh = lane >> 4;
  uint32_t voffq[4], voffg[4];
  wide_dma_offsets(a.ld, wave, lane, voffq);
  wide_dma_offsets(a.lddc, wave, lane, voffg);
  uint32_t ak[4], at[8];
  wide_addresses(ring, lane, ak, at);
  uint16_t* const tail = ring + kWideRing * kWideBuf / 2;
  const uint32_t zeros = uint32_t(reinterpret_cast<uintptr_t>(tail));
  uint32_t al = zeros + 16u + uint32_t(lh) * 16u;
  if (threadIdx.x < 8) *reinterpret_cast<attn_u32x4*>(tail + threadIdx.x * (kWideStep / 2)) = attn_u32x4{0, 0, 0, 0};
  // the local query heads that read this KV head are consecutive
  const int64_t group_first = int64_t(a.kv_off + g) * a.group - a.q_off;
  const int head_first = int(max(group_first, int64_t(0)));
  const int heads_here = max(int(min(group_first + a.group, int64_t(a.q_cnt))) - head_first, 0);

  int buf = 0;
  const int k0 = kt * 128 + wave * 32;  // first key of this wavefront

  f32x4 dk[8][2], dv[8][2];
  zero_acc(dk);
  zero_acc(dv);
  // query tiles this workgroup needs: all, or from the tile that holds its first key on; the walk is the list of
  // (query head, query tile) units, head-major, and part p of n_parts takes an even, contiguous share of it
  const int q_first = a.causal ? kt * 2 : 0;
  const int q_tiles = (S + kBKV - 1) / kBKV;
  const int nt = max(q_tiles - q_first, 0);
  const int units = heads_here * nt;
  const int u_lo = a.n_parts > 1 ? int(int64_t(part) * units / a.n_parts) : 0;
  const int u_hi = a.n_parts > 1 ? int(int64_t(part + 1) * units / a.n_parts) : units;

  if (u_lo < u_hi) {
    int t = q_first + u_lo % nt;                                         // query tile in hand
    int f_head = head_first + u_lo / nt, f_t = t, f_left = u_hi - u_lo;  // the next unit to fetch
    // 9 DMA instructions a wavefront and unit: two tiles and a row of log-sum-exp (even wavefronts) or delta values (odd ones).  Past
    // the last unit the last one is fetched again, so that the number in flight is the same everywhere.
    TileSrc<D> srcQ, srcG;  // rows past the sequence end lie outside the views: zeros
    __amdgpu_buffer_rsrc_t rsL;
    auto fetch_head = [&]() {
      srcQ.init(a.QKV + int64_t(f_head) * D + tok0 * a.ld, a.ld, S);
      srcG.init(a.dC + int64_t(f_head) * D + tok0 * a.lddc, a.lddc, S);
      const float* rows = ((wave & 1) ? a.Delta : a.LSE) + int64_t(f_head) * Mtot + tok0;
      rsL = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(rows), 0, S * 4, 0x00020000);
    };
    auto fetch_part = [&](int to, int i) {
      if (i == 8) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsL, (ntp_gemm::lds_void*)(tail + to * (kWideStep / 2) + 8 + wave * (kBKV * 2)), 4, uint32_t(lane) * 4u, uint32_t(f_t) * (kBKV * 4), 0, 0);
        return;
      }
      uint16_t* dst = ring + to * (kWideBuf / 2) + (i & 1) * kDmaTile + (wave * 4 + (i >> 1)) * 512;
      if (i & 1) dma_16(srcG.rs, dst, voffg[i >> 1], uint32_t(f_t) * srcG.step);
      else dma_16(srcQ.rs, dst, voffq[i >> 1], uint32_t(f_t) * srcQ.step);
    };
    auto fetch_next = [&]() {
      if (f_left > 1) {
        --f_left;
        if (++f_t == q_tiles) {
          f_t = q_first;
          ++f_head;
          fetch_head();
        }
      }
    };
    // bytes from the buffer in hand to the next one, of the tiles and of the row values (an eighth of it)
    auto to_next = [&]() { return buf == kWideRing - 1 ? -int32_t((kWideRing - 1) * kWideBuf) : int32_t(kWideBuf); };
    static_assert(kWideBuf == 8 * kWideStep, "row values");

    // the first unit first, then the owned rows, then two more units
    fetch_head();
#pragma unroll
    for (int i = 0; i < 9; ++i) fetch_part(buf, i);
    fetch_next();
    __builtin_amdgcn_sched_barrier(0);
    // key and value fragments (operand B: j = key), the values with their signs flipped: see mfma_from below
    attn_u32x4 kf[2][4], vf[2][4];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const uint16_t* kp = a.QKV + (tok0 + min(k0 + kb * 16 + lq, S - 1)) * a.ld + int64_t(a.q_cnt + g) * D + lh * 8;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        kf[kb][s] = *reinterpret_cast<const attn_u32x4*>(kp + s * 32);
        vf[kb][s] = *reinterpret_cast<const attn_u32x4*>(kp + int64_t(a.kv_cnt) * D + s * 32);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 1; n < 3; ++n) {
#pragma unroll
      for (int i = 0; i < 9; ++i) fetch_part((buf + n) & 3, i);
      fetch_next();
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) vf[i / 4][i % 4] = negated(vf[i / 4][i % 4]);
    wait_dma<18>();
    lds_stored();
    __builtin_amdgcn_s_barrier();
    owned_ready(kf);
    owned_ready(vf);

    // fragments of the scores of the next half: f[2 s + b], column step s of query block b; f[8 + 2 s + b], output gradient
    attn_u32x4 f[16];
    attn_u32x2 tg[16], tq[16];  // transposed fragments of this half: [2 column block + row block]
    f32x4 nl[2], lr[2], dl[2];  // -log2(e) LSE of this half's rows, LSE and delta of the next half's
    f32x4 s_a[2][2], p_a[2][2], s_b[2][2], p_b[2][2];  // scores and delta - dP of the half in hand and of the next one: [query block][key block]
    unrolled<8>([&](auto j) { f[j] = lds_frag_b128<(j & 1) * 4096>(ak[j / 2]); });
    unrolled<8>([&](auto j) { f[8 + j] = lds_frag_b128<16384 + (j & 1) * 4096>(ak[j / 2]); });
    unrolled<2>([&](auto j) {
      lr[j] = __builtin_bit_cast(f32x4, lds_frag_b128<j * 64>(al));
      dl[j] = __builtin_bit_cast(f32x4, lds_frag_b128<256 + j * 64>(al));
    });
    arrived<0>(lr[0], lr[1], dl[0], dl[1]);
    nl[0] = lr[0] * -1.4426950408889634f;
    nl[1] = lr[1] * -1.4426950408889634f;
    unrolled<4>([&](auto j) { with(f[4 * j], f[4 * j + 1], f[4 * j + 2], f[4 * j + 3]); });
    unrolled<32>([&](auto ic) {
      constexpr int i = decltype(ic)::value, s = (i % 16) / 4, qb = (i / 2) % 2, kb = i % 2;
      if constexpr (i < 4) mfma_zero(s_a[qb][kb], f[i / 2], kf[kb][s]);
      else if constexpr (i < 16) mfma_score(s_a[qb][kb], f[i / 2], kf[kb][s]);
      else if constexpr (i < 20) mfma_from(p_a[qb][kb], f[i / 2], vf[kb][s], dl[qb]);
      else mfma_score(p_a[qb][kb], f[i / 2], vf[kb][s]);
    });
    scores_settle(s_a, p_a);
    // what the steady state has in flight at the start of a half
    unrolled<4>([&](auto j) { f[j] = lds_frag_b128<8192 + (j & 1) * 4096>(ak[j / 2]); });
    unrolled<2>([&](auto j) { dl[j] = __builtin_bit_cast(f32x4, lds_frag_b128<256 + 128 + j * 64>(al)); });
    unrolled<4>([&](auto j) { f[4 + j] = lds_frag_b128<8192 + (j & 1) * 4096>(ak[2 + j / 2]); });

    // the units of which some score is masked: past the sequence end or (causal) before the wavefront's last key
    const int open_lo[2] = {a.causal ? (k0 + 31 + 63) >> 6 : 0, a.causal ? (k0 + 31 - 32 + 63) >> 6 : 0};
    const int open_n[2] = {max(((S - 32) >> 6) + 1 - open_lo[0], 0), max(((S - 64) >> 6) + 1 - open_lo[1], 0)};
    int32_t step = 0;
    auto half = [&](auto hc, f32x4 (&sc)[2][2], f32x4 (&dp)[2][2], f32x4 (&sn)[2][2], f32x4 (&dn)[2][2]) {
      constexpr int H = decltype(hc)::value;
      constexpr int CO = H * 8192, NO = (1 - H) * 8192;  // this half's rows, and the next half's in its buffer
      const int qbase = t * kBKV + H * 32;
      __builtin_amdgcn_sched_barrier(0);
      if (__builtin_expect(uint32_t(t - open_lo[H]) >= uint32_t(open_n[H]), 0)) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int qrow = qbase + qb * 16 + lh * 4 + r, key = k0 + kb * 16 + lq;
              const bool masked = qrow >= S || (a.causal && key > qrow);
              sc[qb][kb][r] = masked ? -INFINITY : sc[qb][kb][r];
              dp[qb][kb][r] = masked ? 0.f : dp[qb][kb][r];
            }
        // (a row whose log-sum-exp is a NaN or an infinity has weights of zero all the same where it is masked)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int r = 0; r < 4; ++r) nl[qb][r] = fminf(nl[qb][r], FLT_MAX);
      }
      __builtin_amdgcn_sched_barrier(0);
      attn_u32x4 pf[2], dsf[2];
      // 64 slots of one matrix instruction each (0-31: the scores and dP of the next half; 32-47: dV^T += dC^T P, 48-63:
      // dK^T -= Q^T dS of this one), at most one or two LDS reads in each, 16 slots ahead of their use, and the DMA and the
      // vector arithmetic spread over them, so that none of them holds up the matrix pipe
      unrolled<64>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (i == 0) arrived<5>(f[0], f[1], f[2], f[3]);
        if constexpr (i == 8) {
          arrived<4>(f[4], f[5], f[6], f[7]);
          with(dl[0], dl[1]);
        }
        if constexpr (i == 16) arrived<4>(f[8], f[9], f[10], f[11]);
        if constexpr (i == 24) {
          arrived<8>(f[12], f[13], f[14], f[15]);
          with(dl[0], dl[1]);  // (not overwritten before the matrix instructions that start from them are through)
        }
        if constexpr (i == 32 || i == 40) {
          constexpr int j = i - 32;
          arrived<8>(tg[j], tg[j + 1], tg[j + 2], tg[j + 3]);
          with(tg[j + 4], tg[j + 5], tg[j + 6], tg[j + 7]);
        }
        if constexpr (i == 48) {
          arrived<10>(tq[0], tq[1], tq[2], tq[3]);
          with(tq[4], tq[5], tq[6], tq[7]);
          if constexpr (H == 0) {
            wait_dma<9>();                 // this wavefront's share of the next unit has landed ...
            __builtin_amdgcn_s_barrier();  // ... and everyone's; the unit before this one has been read by everyone
          }
        }
        if constexpr (i == 56) {
          arrived<6>(tq[8], tq[9], tq[10], tq[11]);
          with(tq[12], tq[13], tq[14], tq[15]);
          with(lr[0], lr[1]);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the matrix instruction
        if constexpr (i < 32) {
          constexpr int s = (i % 16) / 4, qb = (i / 2) % 2, kb = i % 2;
          if constexpr (i < 4) mfma_zero(sn[qb][kb], f[i / 2], kf[kb][s]);
          else if constexpr (i < 16) mfma_score(sn[qb][kb], f[i / 2], kf[kb][s]);
          else if constexpr (i < 20) mfma_from(dn[qb][kb], f[i / 2], vf[kb][s], dl[qb]);  // starts as delta, the values' signs are flipped: delta - dP
          else mfma_score(dn[qb][kb], f[i / 2], vf[kb][s]);
        } else if constexpr (i < 48) {
          constexpr int b = (i - 32) / 4 * 2 + i % 2, kb = (i / 2) % 2;  // (the first key block's weights in slots 32 and 33: the second's are packed in slot 32)
          mfma_grad(dv[b][kb], tg[2 * b], tg[2 * b + 1], pf[kb]);
        } else {
          constexpr int b = (i - 48) / 2;
          mfma_grad(dk[b][i % 2], tq[2 * b], tq[2 * b + 1], dsf[i % 2]);
        }
        // LDS reads
        if constexpr (i < 16 && i % 2 == 0) f[8 + i / 2] = lds_frag_b128<16384 + NO + ((i / 2) & 1) * 4096>(ak[i / 4]);
        if constexpr (i >= 16 && i < 32) tg[i - 16] = lds_tr_b64<16384 + CO + (i & 1) * 4096>(at[(i - 16) / 2]);
        if constexpr (i >= 32 && i < 48) tq[i - 32] = lds_tr_b64<CO + (i & 1) * 4096>(at[(i - 32) / 2]);
        if constexpr (i == 46 || i == 47) lr[i - 46] = __builtin_bit_cast(f32x4, lds_frag_b128<(1 - H) * 128 + (i - 46) * 64>(al));
        if constexpr (i >= 48 && i % 2 == 0) f[(i - 48) / 2] = lds_frag_b128<CO + (((i - 48) / 2) & 1) * 4096>(ak[(i - 48) / 4]);  // of the half after the next
        if constexpr (i == 53 || i == 55) dl[(i - 53) / 2] = __builtin_bit_cast(f32x4, lds_frag_b128<256 + H * 128 + (i - 53) * 32>(al));
        // on to the next buffer
        if constexpr (H == 0 && i == 47) al += uint32_t(step / 8);
        if constexpr (H == 0 && i >= 47 && i < 60 && i % 4 == 3) ak[(i - 47) / 4] += uint32_t(step);
        if constexpr (H == 1 && i >= 48 && i < 56) at[i - 48] += uint32_t(step);
        // DMA
        // (one instruction every ten slots or so: the memory path of a compute unit takes one in 18 cycles)
        if constexpr (H == 0 && (i == 51 || i == 59)) fetch_part((buf + 3) & 3, (i - 51) / 8);
        if constexpr (H == 1 && i % 10 == 3 && i < 60) fetch_part((buf + 3) & 3, 2 + i / 10);
        if constexpr (H == 1 && i == 61) fetch_part((buf + 3) & 3, 8);
        if constexpr (H == 1 && i == 61) fetch_next();
        // vector arithmetic: element e of a key block is query block e / 4, row e % 4
        if constexpr (i < 32) {
          constexpr int kb = i / 16, qb = (i / 8) % 2, r = (i / 2) % 4;
          if constexpr (i % 2 == 0) sc[qb][kb][r] = fmaf(sc[qb][kb][r], a.scale_log2, nl[qb][r]);
          else sc[qb][kb][r] = fast_exp2(sc[qb][kb][r]);
        }
        if constexpr (i >= 4 && i <= 32 && i % 4 == 0) {
          constexpr int j = i / 4 - 1, kb = j / 4, qb = (j / 2) % 2, r = (j % 2) * 2;
          pf[kb][j % 4] = pack2(sc[qb][kb][r], sc[qb][kb][r + 1]);
        }
        if constexpr (i >= 32 && i < 40) dp[(i - 32) / 4][0][i % 4] *= sc[(i - 32) / 4][0][i % 4];
        if constexpr (i >= 38 && i < 46) dp[(i - 38) / 4][1][(i - 38) % 4] *= sc[(i - 38) / 4][1][(i - 38) % 4];
        if constexpr (i >= 34 && i <= 40 && i % 2 == 0) {
          constexpr int j = (i - 34) / 2;
          dsf[0][j] = pack2(dp[j / 2][0][(j % 2) * 2], dp[j / 2][0][(j % 2) * 2 + 1]);
        }
        if constexpr (i >= 40 && i <= 46 && i % 2 == 0) {
          constexpr int j = (i - 40) / 2;
          dsf[1][j] = pack2(dp[j / 2][1][(j % 2) * 2], dp[j / 2][1][(j % 2) * 2 + 1]);
        }
        if constexpr (i >= 56) nl[(i - 56) / 4][i % 4] = lr[(i - 56) / 4][i % 4] * -1.4426950408889634f;
        if constexpr (i == 18) operand_ready(pf[0]);
        if constexpr (i == 32) operand_ready(pf[1]);
        if constexpr (i == 42) operand_ready(dsf[0]);
        if constexpr (i == 47) operand_ready(dsf[1]);
        __builtin_amdgcn_sched_barrier(0);
      });
    };

    for (int w = u_lo; w < u_hi; ++w) {
      step = to_next();
      // Every query row of the tile comes before this wavefront's keys (the first unit of a head, the upper two wavefronts): all weights are
      // zero, and the transposed fragments are read from zeros, so that they do not meet infinities and NaNs of rows that do not see these keys.
      const bool unseen = a.causal && t * kBKV + kBKV - 1 < k0;
      if (__builtin_expect(unseen, 0)) {
#pragma unroll
        for (int b = 0; b < 8; ++b) at[b] = zeros;
      }
      half(std::integral_constant<int, 0>{}, s_a, p_a, s_b, p_b);
      half(std::integral_constant<int, 1>{}, s_b, p_b, s_a, p_a);
      if (__builtin_expect(unseen, 0)) {
        transposed_addresses(zeros - kWideRing * kWideBuf + uint32_t((buf + 1) & 3) * kWideBuf, lane, at);
      }
      if (++t == q_tiles) t = q_first;
      buf = (buf + 1) & 3;
    }
    // nothing may land in a register or in LDS any more
    arrived<0>(f[0], f[1], f[2], f[3]);
    with(f[4], f[5], f[6], f[7]);
    with(lr[0], lr[1], dl[0], dl[1]);
    wait_dma<0>();
  }
  acc_settle(dk);
  acc_settle(dv);

  // the 64-row tile that holds this wavefront's keys, and this lane's first row of it
  const int tile = kt * 2 + (wave >> 1), row = (wave & 1) * 32 + lq;
  if (a.n_parts > 1) {
    // fp32 sums of this part, dK without its factor: per key a row of [dK | dV]
    if (tile < a.tiles) {
      float* pp = a.part_sums + (((int64_t(sh) * a.tiles + tile) * a.n_parts + part) * 64 + row) * (2 * D) + lh * 4;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          *reinterpret_cast<f32x4*>(pp + kb * 16 * (2 * D) + b * 16) = -dk[b][kb];
          *reinterpret_cast<f32x4*>(pp + kb * 16 * (2 * D) + D + b * 16) = dv[b][kb];
        }
    }
    return;
  }
  __builtin_amdgcn_s_barrier();  // the ring has been read, and its last DMA has landed, everywhere
  uint16_t* const lds = ring + wave * (2 * 32 * D);
  uint16_t* const kp = a.dQKV + (tok0 + k0) * a.ldd + int64_t(a.q_cnt + g) * D;
  store_wide_rows(dk, -a.scale, lds, kp, a.ldd, S - k0, lane);
  store_wide_rows(dv, 1.0f, lds + 32 * D, kp + int64_t(a.kv_cnt) * D, a.ldd, S - k0, lane);
}

__device__ __forceinline__ void bwd_dq_wide_body(const CoreBwdArgs& a, uint32_t place, bool is_short, uint16_t* ring) {
  constexpr int D = 128;
  int sh, qt, piece;
  if (!wide_place(a, place, is_short, false, uint32_t(a.n_seq) * uint32_t(a.q_cnt), sh, qt, piece)) return;
  const int seq = sh % a.n_seq, head = sh / a.n_seq;
  const int g = (a.q_off + head) / a.group - a.kv_off;
  const int S = a.seq_len;
  const int64_t tok0 = int64_t(seq) * S, Mtot = int64_t(a.n_seq) * S;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 15, lh = lane >> 4;
  TileSrc<D> srcK, srcV;
  srcK.init(a.QKV + int64_t(a.q_cnt + g) * D + tok0 * a.ld, a.ld, S);
  srcV.init(a.QKV + int64_t(a.q_cnt + a.kv_cnt + g) * D + tok0 * a.ld, a.ld, S);
  uint32_t voff[4];
  wide_dma_offsets(a.ld, wave, lane, voff);
  uint32_t ak[4], at[8];
  wide_addresses(ring, lane, ak, at);

  int buf = 0;
  const int q0 = qt * 128 + wave * 32;  // first query row of this wavefront

  f32x4 acc[8][2];
  zero_acc(acc);
  const int kv_end = a.causal ? min(S, qt * 128 + 128) : S;
  const int n_tiles = (kv_end + kBKV - 1) / kBKV;
  const int t_lo = a.n_parts > 1 ? int(int64_t(piece) * n_tiles / a.n_parts) : 0;
  const int t_hi = a.n_parts > 1 ? int(int64_t(piece + 1) * n_tiles / a.n_parts) : n_tiles;

  // 8 DMA instructions a wavefront and tile pair; past the last tile the last one is fetched again
  auto fetch_part = [&](int to, int t, int i) {
    uint16_t* dst = ring + to * (kWideBuf / 2) + (i & 1) * kDmaTile + (wave * 4 + (i >> 1)) * 512;
    dma_16((i & 1) ? srcV.rs : srcK.rs, dst, voff[i >> 1], uint32_t(t) * srcK.step);
  };
  // the first tile first, then the owned rows, then two more tiles
  if (t_lo < t_hi) {
#pragma unroll
    for (int i = 0; i < 8; ++i) fetch_part(buf, t_lo, i);
  }
  __builtin_amdgcn_sched_barrier(0);
  // query and output-gradient fragments (operand B: j = query row), the latter with their signs flipped: see mfma_from below
  attn_u32x4 qf[2][4], gf[2][4], of[2][4];
  float nlse[2];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const int64_t tok = tok0 + min(q0 + qb * 16 + lq, S - 1);
    const uint16_t* qp = a.QKV + tok * a.ld + int64_t(head) * D + lh * 8;
    const uint16_t* gp = a.dC + tok * a.lddc + int64_t(head) * D + lh * 8;
    const uint16_t* op = a.C + tok * a.ldc + int64_t(head) * D + lh * 8;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      qf[qb][s] = *reinterpret_cast<const attn_u32x4*>(qp + s * 32);
      gf[qb][s] = *reinterpret_cast<const attn_u32x4*>(gp + s * 32);
      of[qb][s] = *reinterpret_cast<const attn_u32x4*>(op + s * 32);
    }
    nlse[qb] = a.LSE[int64_t(head) * Mtot + tok];
  }
  __builtin_amdgcn_sched_barrier(0);
  if (t_lo < t_hi) {
#pragma unroll
    for (int n = 1; n < 3; ++n)
#pragma unroll
      for (int i = 0; i < 8; ++i) fetch_part((buf + n) & 3, min(t_lo + n, t_hi - 1), i);
  }
  __builtin_amdgcn_sched_barrier(0);
  f32x4 dl[2];  // delta of the lane's rows
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    float sum = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bf16x8 gb = __builtin_bit_cast(bf16x8, gf[qb][s]), ob = __builtin_bit_cast(bf16x8, of[qb][s]);
#pragma unroll
      for (int e = 0; e < 8; ++e) sum += float(gb[e]) * float(ob[e]);
      gf[qb][s] = negated(gf[qb][s]);
    }
    const float delta = xor_sum(sum);
    dl[qb] = f32x4{delta, delta, delta, delta};
    nlse[qb] *= -1.4426950408889634f;
    const int qrow = q0 + qb * 16 + lq;
    if (lh == 0 && piece == 0 && !a.delta_stored && qrow < S) a.Delta[int64_t(head) * Mtot + tok0 + qrow] = delta;
  }
  if (t_lo < t_hi) {
    wait_dma<16>();
    __builtin_amdgcn_s_barrier();
    owned_ready(qf);
    owned_ready(gf);

    attn_u32x4 f[16];   // fragments of the scores of the next half: f[2 s + b], column step s of key block b; f[8 + 2 s + b], values
    attn_u32x2 tk[16];  // transposed key fragments of this half: [2 column block + row block]
    f32x4 s_a[2][2], p_a[2][2], s_b[2][2], p_b[2][2];  // scores and delta - dP of the half in hand and of the next one: [key block][query block]
    operand_ready(dl[0]);
    operand_ready(dl[1]);
    unrolled<8>([&](auto j) { f[j] = lds_frag_b128<(j & 1) * 4096>(ak[j / 2]); });
    unrolled<8>([&](auto j) { f[8 + j] = lds_frag_b128<16384 + (j & 1) * 4096>(ak[j / 2]); });
    arrived<0>(f[0], f[1], f[2], f[3]);
    unrolled<3>([&](auto j) { with(f[4 + 4 * j], f[5 + 4 * j], f[6 + 4 * j], f[7 + 4 * j]); });
    unrolled<32>([&](auto ic) {
      constexpr int i = decltype(ic)::value, s = (i % 16) / 4, kb = (i / 2) % 2, qb = i % 2;
      if constexpr (i < 4) mfma_zero(s_a[kb][qb], f[i / 2], qf[qb][s]);
      else if constexpr (i < 16) mfma_score(s_a[kb][qb], f[i / 2], qf[qb][s]);
      else if constexpr (i < 20) mfma_from(p_a[kb][qb], f[i / 2], gf[qb][s], dl[qb]);
      else mfma_score(p_a[kb][qb], f[i / 2], gf[qb][s]);
    });
    scores_settle(s_a, p_a);
    // what the steady state has in flight at the start of a half
    unrolled<8>([&](auto j) { f[j] = lds_frag_b128<8192 + (j & 1) * 4096>(ak[j / 2]); });

    // the tiles of which no score is masked are the first open_n: before the sequence end and (causal) the wavefront's first row
    const int open_end = a.causal ? min(S, q0 + 1) : S;
    const int open_n[2] = {(open_end + 32) >> 6, open_end >> 6};
    int32_t step = 0;
    auto half = [&](auto hc, int t, f32x4 (&sc)[2][2], f32x4 (&dp)[2][2], f32x4 (&sn)[2][2], f32x4 (&dn)[2][2]) {
      constexpr int H = decltype(hc)::value;
      constexpr int CO = H * 8192, NO = (1 - H) * 8192;  // this half's rows, and the next half's in its buffer
      const int kv0 = t * kBKV + H * 32;
      __builtin_amdgcn_sched_barrier(0);
      if (__builtin_expect(t >= open_n[H], 0)) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int key = kv0 + kb * 16 + lh * 4 + r, qrow = q0 + qb * 16 + lq;
              sc[kb][qb][r] = key >= S || (a.causal && key > qrow) ? -INFINITY : sc[kb][qb][r];
            }
      }
      __builtin_amdgcn_sched_barrier(0);
      attn_u32x4 dsf[2];
      // 48 slots of one matrix instruction each (0-31: the scores and dP of the next half; 32-47: dQ^T -= K^T dS^T of this one)
      unrolled<48>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (i == 0) arrived<4>(f[0], f[1], f[2], f[3]);
        if constexpr (i == 8) arrived<4>(f[4], f[5], f[6], f[7]);
        if constexpr (i == 16) arrived<4>(f[8], f[9], f[10], f[11]);
        if constexpr (i == 24) arrived<8>(f[12], f[13], f[14], f[15]);
        if constexpr (i == 32) {
          arrived<8>(tk[0], tk[1], tk[2], tk[3]);
          with(tk[4], tk[5], tk[6], tk[7]);
          if constexpr (H == 0) {
            wait_dma<8>();                 // this wavefront's share of the next tile has landed ...
            __builtin_amdgcn_s_barrier();  // ... and everyone's; the tile before this one has been read by everyone
          }
        }
        if constexpr (i == 40) {
          arrived<4>(tk[8], tk[9], tk[10], tk[11]);
          with(tk[12], tk[13], tk[14], tk[15]);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the matrix instruction
        if constexpr (i < 32) {
          constexpr int s = (i % 16) / 4, kb = (i / 2) % 2, qb = i % 2;
          if constexpr (i < 4) mfma_zero(sn[kb][qb], f[i / 2], qf[qb][s]);
          else if constexpr (i < 16) mfma_score(sn[kb][qb], f[i / 2], qf[qb][s]);
          else if constexpr (i < 20) mfma_from(dn[kb][qb], f[i / 2], gf[qb][s], dl[qb]);  // starts as delta, dC's signs are flipped: delta - dP
          else mfma_score(dn[kb][qb], f[i / 2], gf[qb][s]);
        } else {
          constexpr int b = (i - 32) / 2;
          mfma_grad(acc[b][i % 2], tk[2 * b], tk[2 * b + 1], dsf[i % 2]);
        }
        // LDS reads
        if constexpr (i < 16 && i % 2 == 0) f[8 + i / 2] = lds_frag_b128<16384 + NO + ((i / 2) & 1) * 4096>(ak[i / 4]);
        if constexpr (i >= 16 && i < 32) tk[i - 16] = lds_tr_b64<CO + (i & 1) * 4096>(at[(i - 16) / 2]);
        if constexpr (i >= 32 && i % 2 == 0) f[(i - 32) / 2] = lds_frag_b128<CO + (((i - 32) / 2) & 1) * 4096>(ak[(i - 32) / 4]);  // of the half after the next
        // on to the next buffer
        if constexpr (H == 0 && i >= 31 && i < 44 && i % 4 == 3) ak[(i - 31) / 4] += uint32_t(step);
        if constexpr (H == 1 && i >= 32 && i < 40) at[i - 32] += uint32_t(step);
        // DMA
        // (one instruction every eight slots: the memory path of a compute unit takes one in 18 cycles)
        if constexpr (H == 0 && (i == 35 || i == 43)) fetch_part((buf + 3) & 3, min(t + 3, t_hi - 1), (i - 35) / 8);
        if constexpr (H == 1 && i % 8 == 3) fetch_part((buf + 3) & 3, min(t + 3, t_hi - 1), 2 + i / 8);
        // vector arithmetic: element e of a lane's 16 (query block e / 8, key block (e / 4) % 2, row e % 4) from slot 7 e / 4 on
        unrolled<16>([&](auto ec) {
          constexpr int e = decltype(ec)::value, at_slot = 7 * e / 4, qb = e / 8, kb = (e / 4) % 2, r = e % 4;
          if constexpr (i == at_slot) sc[kb][qb][r] = fmaf(sc[kb][qb][r], a.scale_log2, nlse[qb]);
          if constexpr (i == at_slot + 1) sc[kb][qb][r] = fast_exp2(sc[kb][qb][r]);
          if constexpr (i == at_slot + 2) dp[kb][qb][r] *= sc[kb][qb][r];
          if constexpr (i == at_slot + 3 && e % 2 == 1) dsf[qb][(e % 8) / 2] = pack2(dp[kb][qb][r - 1], dp[kb][qb][r]);
        });
        if constexpr (i == 17) operand_ready(dsf[0]);
        if constexpr (i == 31) operand_ready(dsf[1]);
        __builtin_amdgcn_sched_barrier(0);
      });
    };

    // under the mask the lower two wavefronts' rows see nothing of the last tile: no products there (see bwd_dkv_wide_body), only the others' barrier
    const int t_own = a.causal ? min(t_hi, ((q0 + 31) >> 6) + 1) : t_hi;
    for (int t = t_lo; t < t_own; ++t) {
      step = buf == kWideRing - 1 ? -int32_t((kWideRing - 1) * kWideBuf) : int32_t(kWideBuf);
      half(std::integral_constant<int, 0>{}, t, s_a, p_a, s_b, p_b);
      half(std::integral_constant<int, 1>{}, t, s_b, p_b, s_a, p_a);
      buf = (buf + 1) & 3;
    }
    // nothing may land in a register or in LDS any more
    arrived<0>(f[0], f[1], f[2], f[3]);
    with(f[4], f[5], f[6], f[7]);
    wait_dma<0>();
    for (int t = max(t_lo, t_own); t < t_hi; ++t) __builtin_amdgcn_s_barrier();
  }
  acc_settle(acc);

  // the 64-row tile that holds this wavefront's rows, and this lane's first row of it
  const int tile = qt * 2 + (wave >> 1), row = (wave & 1) * 32 + lq;
  if (a.n_parts > 1) {
    // unscaled fp32 sums of this part
    if (tile < a.tiles) {
      float* pp = a.part_sums + (((int64_t(sh) * a.tiles + (a.causal ? a.tiles - 1 - tile : tile)) * a.n_parts + piece) * 64 + row) * D + lh * 4;
#pragma unroll
      for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int b = 0; b < 8; ++b) *reinterpret_cast<f32x4*>(pp + qb * 16 * D + b * 16) = -acc[b][qb];
    }
    return;
  }
  __builtin_amdgcn_s_barrier();  // the ring has been read, and its last DMA has landed, everywhere
  store_wide_rows(acc, -a.scale, ring + wave * (32 * D), a.dQKV + (tok0 + q0) * a.ldd + int64_t(head) * D, a.ldd, S - q0, lane);
}

// One kind of workgroups, `n_long` of them in the first section.
__global__ __attribute__((amdgpu_flat_work_group_size(kThreads, kThreads), amdgpu_waves_per_eu(1, 1))) void
attn_core_bwd_dkv_wide_kernel(const CoreBwdArgs a, const uint32_t n_long) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kWideLds / 2];
  const bool is_short = blockIdx.x >= n_long;
  bwd_dkv_wide_body(a, is_short ? blockIdx.x - n_long : blockIdx.x, is_short, ring);
}

__global__ __attribute__((amdgpu_flat_work_group_size(kThreads, kThreads), amdgpu_waves_per_eu(1, 1))) void
attn_core_bwd_dq_wide_kernel(const CoreBwdArgs a, const uint32_t n_long) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kWideRing * kWideBuf / 2];
  const bool is_short = blockIdx.x >= n_long;
  bwd_dq_wide_body(a, is_short ? blockIdx.x - n_long : blockIdx.x, is_short, ring);
}

// Both in one launch, in sections by their longest walks: the long dK/dV walks (four products a tile pair), the long dQ walks (three)
// and the short dK/dV walks, these two in either order, and the short dQ walks.
__global__ __attribute__((amdgpu_flat_work_group_size(kThreads, kThreads), amdgpu_waves_per_eu(1, 1))) void
attn_core_bwd_both_wide_kernel(const CoreBwdArgs adq, const CoreBwdArgs adkv, const uint32_t n_dq, const uint32_t n_dkv, const uint32_t kv_first) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kWideLds / 2];
  uint32_t b = blockIdx.x;
  bool dkv = b < n_dkv, is_short = false;
  if (!dkv) {
    b -= n_dkv;
    const uint32_t second = adkv.causal && kv_first ? n_dkv : n_dq;  // (without the mask there are no short walks)
    dkv = adkv.causal && kv_first && b < second;
    is_short = dkv;
    if (b >= second) {
      b -= second;
      const uint32_t third = kv_first ? n_dq : n_dkv;
      dkv = !kv_first && b < third;
      is_short = dkv;
      if (b >= third) {
        b -= third;
        is_short = true;
      }
    }
  }
  if (dkv) bwd_dkv_wide_body(adkv, b, is_short, ring);
  else bwd_dq_wide_body(adq, b, is_short, ring);
}
