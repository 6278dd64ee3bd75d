// Attention core at head dimension 64 by DMA (included by ntp_attn_core.hip), 128 rows per workgroup, 32 per wavefront: backward (dQ and dK/dV workgroups of one launch) and forward.
//
// Backward: what bound the register-copy bodies (bwd_dq_body, bwd_dkv_body, 16 rows per wavefront) was the LDS: a (64 x 64) tile pair of either kind reads 96 and 128 KB of fragments, one
// matrix instruction each, and writes 16 KB of copies, 2000 of the 2160 cycles that both took together.  With two blocks every fragment feeds two
// matrix instructions; the tiles come by DMA into two buffers (rows of 128 bytes with permuted chunks, see ntp_attn_small.h), one barrier a tile, no staging
// registers.  Products, masks and rounding are those of the other bodies, and so are the tiles that a row meets.  14 heads, 8192 tokens causal 541 -> 450 us, 2048
// unmasked 94 -> 69, 28 heads x 4096 causal 298 -> 239; with 16 rows per wavefront the same DMA form is not faster than the register copies (0.97-1.08 of the time: two
// workgroups on a unit instead of three).  What bounds it now is issue: 1200 cycles of vector work and 900 of matrix work a pair of either kind on two wavefronts per SIMD.
constexpr int kTile64 = kBKV * 64;  // elements of a tile
constexpr int kBlocks64 = 2;        // 16-row blocks of a wavefront

// LDS read addresses of a lane (the first tile; the others and the 16-row block are immediates)
struct Addr64 {
  SmallAddr<64> ad;
  __device__ __forceinline__ void init(const uint16_t* lds, int lq, int lh) {
    ad.init(lq, lh);
    const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>(lds));
#pragma unroll
    for (int i = 0; i < 2; ++i) ad.row[i] += base;
#pragma unroll
    for (int i = 0; i < 4; ++i) ad.col[i] += base;
  }
  // row fragments of tile T, f[rb * 2 + ks]; transposed ones, of 16-column blocks 2 H and 2 H + 1: f[(db % 2) * 4 + s2 * 2 + half]
  template <int T>
  __device__ __forceinline__ void rows(attn_u32x4 (&f)[8]) const {
    small_for(std::make_integer_sequence<int, 8>{}, [&](auto i) {
      constexpr int rb = decltype(i)::value / 2, ks = decltype(i)::value % 2;
      f[decltype(i)::value] = lds_frag_b128<T * kTile64 * 2 + rb * 16 * 128>(ad.row[ks]);
    });
  }
  template <int T, int H>
  __device__ __forceinline__ void cols(attn_u32x2 (&f)[8]) const {
    small_for(std::make_integer_sequence<int, 8>{}, [&](auto i) {
      constexpr int db = H * 2 + decltype(i)::value / 4, q = decltype(i)::value % 4;
      f[decltype(i)::value] = lds_tr_b64<T * kTile64 * 2 + q * 16 * 128>(ad.col[db]);
    });
  }
};

struct Dma64 {  // this wavefront's two DMA instructions of a tile
  uint32_t voff[2];
  __device__ __forceinline__ void init(int64_t ld, int wave, int lane) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int p = (wave * 2 + j) * 64 + lane, row = p >> 3, slot = p & 7;
      voff[j] = uint32_t((int64_t(row) * ld + int64_t(uint32_t(slot) ^ SmallTile<64>::swz(row)) * 8) * 2);
    }
  }
  __device__ __forceinline__ void tile(__amdgpu_buffer_rsrc_t rs, uint16_t* dst, int wave, uint32_t soff) const {
#pragma unroll
    for (int j = 0; j < 2; ++j) dma_16(rs, dst + (wave * 2 + j) * 512, voff[j], soff);
  }
};

// blocks 2 H and 2 H + 1 of acc^T += tile^T f (slots in the order the scores sit in the registers)
template <int H>
__device__ __forceinline__ void products64(const attn_u32x2 (&t)[8], const bf16x8 (&f)[kBlocks64][2], f32x4 (&acc)[kBlocks64][4]) {
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int b = 0; b < kBlocks64; ++b)
        acc[b][H * 2 + d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(small_col_frag(t[d * 4 + s2 * 2], t[d * 4 + s2 * 2 + 1]), f[b][s2], acc[b][H * 2 + d], 0, 0, 0);
}

// dQ: 128 query rows of one (sequence, head).  lds: four tiles, key buffers 0 and 1, value buffers 0 and 1.
template <bool PAIRED>
__device__ __forceinline__ void bwd_dq64_body(const CoreBwdArgs& a, const uint32_t first, const uint32_t count, uint16_t* const lds) {
  constexpr int D = 64, KS = 2, DB = 4, B = kBlocks64, kRows = 64 * B;
  const uint32_t bid = xcd_major(first, count);
  const int per_seq = PAIRED ? a.pairs : a.tiles;
  const int u = int(bid) % per_seq, sh = int(bid) / per_seq;
  const int seq = sh % a.n_seq, head = sh / a.n_seq;
  const int g = (a.q_off + head) / a.group - a.kv_off;
  const int S = a.seq_len;
  const int64_t tok0 = int64_t(seq) * S, Mtot = int64_t(a.n_seq) * S;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 15, lh = lane >> 4;
  const uint16_t* const Qp = a.QKV + int64_t(head) * D;
  TileSrc<D> srcK, srcV;
  srcK.init(a.QKV + int64_t(a.q_cnt + g) * D + tok0 * a.ld, a.ld, S);
  srcV.init(a.QKV + int64_t(a.q_cnt + a.kv_cnt + g) * D + tok0 * a.ld, a.ld, S);
  Dma64 dma;
  dma.init(a.ld, wave, lane);
  Addr64 ad;
  ad.init(lds, lq, lh);
  auto ask = [&](int t, int buf) {  // rows past the sequence end arrive as zeros (masked below)
    dma.tile(srcK.rs, lds + buf * kTile64, wave, uint32_t(t) * srcK.step);
    dma.tile(srcV.rs, lds + (2 + buf) * kTile64, wave, uint32_t(t) * srcV.step);
  };

  for (int seg = 0; seg < (PAIRED ? 2 : 1); ++seg) {
    const int qt = PAIRED ? (seg == 0 ? a.tiles - 1 - u : u) : (a.causal ? a.tiles - 1 - u : u);
    if (seg == 1) {
      if (qt == a.tiles - 1 - u) break;  // odd tile count: the middle tile has no partner
      __syncthreads();                   // the first pass's last tile has been read by everyone
    }
    const int q0 = qt * kRows + wave * (16 * B);
    const int n_tiles = ((a.causal ? min(S, qt * kRows + kRows) : S) + kBKV - 1) / kBKV;
    ask(0, 0);
    bf16x8 qf[B][KS], gf[B][KS];
    float lse2[B], delta[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int qr = min(q0 + b * 16 + lq, S - 1);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        qf[b][ks] = *reinterpret_cast<const bf16x8*>(Qp + (tok0 + qr) * a.ld + ks * 32 + lh * 8);
        gf[b][ks] = *reinterpret_cast<const bf16x8*>(a.dC + (tok0 + qr) * a.lddc + int64_t(head) * D + ks * 32 + lh * 8);
      }
      delta[b] = a.Delta[int64_t(head) * Mtot + tok0 + qr];
      lse2[b] = a.LSE[int64_t(head) * Mtot + tok0 + qr] * 1.4426950408889634f;
    }
    f32x4 acc[B][DB];
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[b][db] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto step = [&](auto bufc, int t) {
      constexpr int BUF = decltype(bufc)::value;
      dma_done();       // this wavefront's share of tile t has landed ...
      __syncthreads();  // ... and everyone's; everyone has read the tile before
      if (t + 1 < n_tiles) ask(t + 1, BUF ^ 1);
      const int kv0 = t * kBKV;
      if (a.causal && kv0 > q0 + 16 * B - 1) return;  // nothing of this tile is visible to the wavefront's rows
      attn_u32x4 kf[8], vf[8];
      ad.rows<BUF>(kf);
      ad.rows<2 + BUF>(vf);
      lds_reads_left<8>(kf);
      f32x4 st[4][B], dpt[4][B];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int b = 0; b < B; ++b) {
          st[kb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) st[kb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[kb * KS + ks]), qf[b][ks], st[kb][b], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
      lds_reads_done(vf);
      attn_u32x2 t0[8], t1[8];
      ad.cols<BUF, 0>(t0);
      ad.cols<BUF, 1>(t1);
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int b = 0; b < B; ++b) {
          dpt[kb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) dpt[kb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[kb * KS + ks]), gf[b][ks], dpt[kb][b], 0, 0, 0);
        }
      const bool edge = kv0 + kBKV > S || (a.causal && kv0 + kBKV - 1 > q0);
      bf16x8 dsf[B][2];
#pragma unroll
      for (int b = 0; b < B; ++b) {
        float ds[4][4];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int r = 0; r < 4; ++r) ds[kb][r] = fast_exp2(fmaf(st[kb][b][r], a.scale_log2, -lse2[b]));
        if (edge) {
          const int qrow = q0 + b * 16 + lq, last = (a.causal ? min(qrow, S - 1) : S - 1) - kv0 - lh * 4;
#pragma unroll
          for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (kb * 16 + r > last) ds[kb][r] = 0.f;
        }
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int r = 0; r < 4; ++r) ds[kb][r] *= dpt[kb][b][r] - delta[b];
        small_pack(ds, dsf[b]);
      }
      __builtin_amdgcn_sched_barrier(0);
      lds_reads_done(t0);
      lds_reads_tied(t1);
      products64<0>(t0, dsf, acc);
      products64<1>(t1, dsf, acc);
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = 0; t < n_tiles; t += 2) {
      step(std::integral_constant<int, 0>{}, t);
      if (t + 1 < n_tiles) step(std::integral_constant<int, 1>{}, t + 1);
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int qrow = q0 + b * 16 + lq;
      if (qrow >= S) continue;
      uint16_t* const op = a.dQKV + (tok0 + qrow) * a.ldd + int64_t(head) * D + lh * 4;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        u16x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = ntp_gemm::f32_to_bf16(acc[b][db][r] * a.scale);
        *reinterpret_cast<u16x4*>(op + db * 16) = o;
      }
    }
  }  // the workgroup's passes
}

// dK and dV: 128 keys of one (sequence, KV head); the walk over the query tiles of every query head that reads it is one stream through the two buffers.
// lds: four tiles, query buffers 0 and 1, output-gradient buffers 0 and 1; sLD: [buffer][log-sum-exp, delta][row].
template <bool PAIRED>
__device__ __forceinline__ void bwd_dkv64_body(const CoreBwdArgs& a, const uint32_t first, const uint32_t count, uint16_t* const lds, float* const sLD) {
  constexpr int D = 64, KS = 2, DB = 4, B = kBlocks64;
  const uint32_t bid = xcd_major(first, count);
  const int per_seq = PAIRED ? a.pairs : a.tiles;
  const int u = int(bid) % per_seq, sh = int(bid) / per_seq;
  const int seq = sh % a.n_seq, g = sh / a.n_seq;  // g: local KV head
  const int S = a.seq_len;
  const int64_t tok0 = int64_t(seq) * S, Mtot = int64_t(a.n_seq) * S;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 15, lh = lane >> 4;
  const uint16_t* const Kp = a.QKV + int64_t(a.q_cnt + g) * D;
  const uint16_t* const Vp = a.QKV + int64_t(a.q_cnt + a.kv_cnt + g) * D;
  Dma64 dmaq, dmag;
  dmaq.init(a.ld, wave, lane);
  dmag.init(a.lddc, wave, lane);
  Addr64 ad;
  ad.init(lds, lq, lh);
  const uint32_t row_values = uint32_t(reinterpret_cast<uintptr_t>(sLD)) + uint32_t(lh) * 16u;
  const int h_lo = max(0, (a.kv_off + g) * a.group - a.q_off), h_hi = min(a.q_cnt, (a.kv_off + g + 1) * a.group - a.q_off);
  const int q_tiles = (S + kBKV - 1) / kBKV;

  for (int seg = 0; seg < (PAIRED ? 2 : 1); ++seg) {
    // this pass's key tile: with pairing an early one (whose keys most query tiles see), then its partner from the end
    const int kt = PAIRED && seg == 1 ? a.tiles - 1 - u : u;
    if (seg == 1) {
      if (kt == u) break;  // odd tile count: the middle tile has no partner
      __syncthreads();     // the first pass's last tile has been read by everyone
    }
    const int k0 = kt * (64 * B) + wave * (16 * B);  // first key of this wavefront
    const int q_first = a.causal ? kt * B : 0, nt = q_tiles - q_first;
    const int units = max(h_hi - h_lo, 0) * nt;
    float rl = 0.f, rd = 0.f;  // of the tile asked for last, row threadIdx.x
    int ask_head = h_lo, ask_t = q_first;
    auto ask = [&](int buf) {  // the walk's next unit; rows past the sequence end arrive as zeros (masked below)
      TileSrc<D> srcQ, srcG;
      srcQ.init(a.QKV + int64_t(ask_head) * D + tok0 * a.ld, a.ld, S);
      srcG.init(a.dC + int64_t(ask_head) * D + tok0 * a.lddc, a.lddc, S);
      dmaq.tile(srcQ.rs, lds + buf * kTile64, wave, uint32_t(ask_t) * srcQ.step);
      dmag.tile(srcG.rs, lds + (2 + buf) * kTile64, wave, uint32_t(ask_t) * srcG.step);
      if (threadIdx.x < kBKV) {
        const int64_t row = int64_t(ask_head) * Mtot + tok0 + min(ask_t * kBKV + int(threadIdx.x), S - 1);
        rl = a.LSE[row] * 1.4426950408889634f;
        rd = a.Delta[row];
      }
      if (++ask_t == q_tiles) {
        ask_t = q_first;
        ++ask_head;
      }
    };
    if (units > 0) ask(0);
    // key and value fragments (operand B: j = key)
    bf16x8 kf[B][KS], vf[B][KS];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int64_t row = (tok0 + min(k0 + b * 16 + lq, S - 1)) * a.ld + lh * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        kf[b][ks] = *reinterpret_cast<const bf16x8*>(Kp + row + ks * 32);
        vf[b][ks] = *reinterpret_cast<const bf16x8*>(Vp + row + ks * 32);
      }
    }
    f32x4 dk[B][DB], dv[B][DB];
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        dk[b][db] = f32x4{0.f, 0.f, 0.f, 0.f};
        dv[b][db] = f32x4{0.f, 0.f, 0.f, 0.f};
      }

    int t = q_first;  // of the unit in hand
    auto step = [&](auto bufc, bool more) {
      constexpr int BUF = decltype(bufc)::value;
      const int qbase = t * kBKV;
      t = t + 1 == q_tiles ? q_first : t + 1;
      dma_done();  // this wavefront's share of the unit has landed ...
      if (threadIdx.x < kBKV) {
        sLD[BUF * 128 + threadIdx.x] = rl;
        sLD[BUF * 128 + 64 + threadIdx.x] = rd;
      }
      __syncthreads();  // ... and everyone's; everyone has read the unit before
      if (more) ask(BUF ^ 1);
      if (a.causal && qbase + kBKV - 1 < k0) return;  // every query row of the tile comes before this wavefront's keys
      attn_u32x4 qa[8], ga[8];
      ad.rows<BUF>(qa);
      ad.rows<2 + BUF>(ga);
      lds_reads_left<8>(qa);
      // S and dP blocks: [query qb*16 + (lane/16)*4 + r][key b*16 + lane%16]
      f32x4 sc[4][B], dp[4][B];
#pragma unroll
      for (int qb = 0; qb < 4; ++qb)
#pragma unroll
        for (int b = 0; b < B; ++b) {
          sc[qb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) sc[qb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, qa[qb * KS + ks]), kf[b][ks], sc[qb][b], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
      lds_reads_done(ga);
      attn_u32x4 ld[8];  // log-sum-exp of row block qb, then delta
      small_for(std::make_integer_sequence<int, 8>{}, [&](auto i) {
        constexpr int n = decltype(i)::value;
        ld[n] = lds_frag_b128<(BUF * 128 + (n / 4) * 64 + (n % 4) * 16) * 4>(row_values);
      });
#pragma unroll
      for (int qb = 0; qb < 4; ++qb)
#pragma unroll
        for (int b = 0; b < B; ++b) {
          dp[qb][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) dp[qb][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ga[qb * KS + ks]), vf[b][ks], dp[qb][b], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
      lds_reads_done(ld);
      attn_u32x2 g0[8], g1[8];
      ad.cols<2 + BUF, 0>(g0);
      ad.cols<2 + BUF, 1>(g1);
      const bool edge = qbase + kBKV > S || k0 + 16 * B > S || (a.causal && qbase < k0 + 16 * B - 1);
      bf16x8 pf[B][2], dsf[B][2];
#pragma unroll
      for (int b = 0; b < B; ++b) {
        float p[4][4], ds[4][4];
#pragma unroll
        for (int qb = 0; qb < 4; ++qb) {
          const f32x4 l4 = __builtin_bit_cast(f32x4, ld[qb]), d4 = __builtin_bit_cast(f32x4, ld[4 + qb]);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            p[qb][r] = fast_exp2(fmaf(sc[qb][b][r], a.scale_log2, -l4[r]));
            ds[qb][r] = dp[qb][b][r] - d4[r];
          }
        }
        if (edge) {
          const int key = k0 + b * 16 + lq;
#pragma unroll
          for (int qb = 0; qb < 4; ++qb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int qrow = qbase + qb * 16 + lh * 4 + r;
              if (qrow >= S || key >= S || (a.causal && key > qrow)) p[qb][r] = 0.f;
            }
        }
#pragma unroll
        for (int qb = 0; qb < 4; ++qb)
#pragma unroll
          for (int r = 0; r < 4; ++r) ds[qb][r] *= p[qb][r];
        small_pack(p, pf[b]);
        small_pack(ds, dsf[b]);
      }
      __builtin_amdgcn_sched_barrier(0);
      // dV^T += dC^T P, dK^T += Q^T dS
      lds_reads_done(g0);
      lds_reads_tied(g1);
      attn_u32x2 t0[8], t1[8];
      ad.cols<BUF, 0>(t0);
      ad.cols<BUF, 1>(t1);
      products64<0>(g0, pf, dv);
      products64<1>(g1, pf, dv);
      __builtin_amdgcn_sched_barrier(0);
      lds_reads_done(t0);
      lds_reads_tied(t1);
      products64<0>(t0, dsf, dk);
      products64<1>(t1, dsf, dk);
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int i = 0; i < units; i += 2) {
      step(std::integral_constant<int, 0>{}, i + 1 < units);
      if (i + 1 < units) step(std::integral_constant<int, 1>{}, i + 2 < units);
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int key = k0 + b * 16 + lq;
      if (key >= S) continue;
      uint16_t* const kp = a.dQKV + (tok0 + key) * a.ldd + int64_t(a.q_cnt + g) * D + lh * 4;
      uint16_t* const vp = a.dQKV + (tok0 + key) * a.ldd + int64_t(a.q_cnt + a.kv_cnt + g) * D + lh * 4;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        u16x4 ok, ov;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          ok[r] = ntp_gemm::f32_to_bf16(dk[b][db][r] * a.scale);
          ov[r] = ntp_gemm::f32_to_bf16(dv[b][db][r]);
        }
        *reinterpret_cast<u16x4*>(kp + db * 16) = ok;
        *reinterpret_cast<u16x4*>(vp + db * 16) = ov;
      }
    }
  }  // the workgroup's passes
}

template <bool PAIRED>
__global__ __launch_bounds__(kThreads, 2) void attn_core_bwd_both64_dma_kernel(const CoreBwdArgs adq, const CoreBwdArgs adkv, const BothOrder o) {
  __shared__ __attribute__((aligned(1024))) uint16_t tiles[4 * kTile64];
  __shared__ __attribute__((aligned(16))) float row_values[2 * 2 * kBKV];
  uint32_t b = blockIdx.x;
  if (both_place(o, b)) bwd_dkv64_body<PAIRED>(adkv, b, o.n_dkv, tiles, row_values);
  else bwd_dq64_body<PAIRED>(adq, b, gridDim.x - o.n_dkv, tiles);
}

// Forward: 128 query rows of one (sequence, head), or under the mask a pair of such tiles.  The register-copy kernel with 32 rows per wavefront waited at two barriers a
// tile and spent vector instructions on its copies.  40 random launches: 0.79-0.92 of its time (2 x 6583 tokens, 14 heads causal 279 -> 223 us; 4 x 2655 unmasked 165 -> 150).
// What bounds it is the softmax's vector work, 1000 of the 1400 cycles a tile takes on a unit with two workgroups or three.
template <bool PAIRED>
__global__ __attribute__((amdgpu_flat_work_group_size(kThreads, kThreads), amdgpu_waves_per_eu(2, 2))) void attn_core_fwd64_dma_kernel(const CoreArgs a) {
  constexpr int D = 64, KS = 2, DB = 4, B = kBlocks64, kRows = 64 * B;
  __shared__ __attribute__((aligned(1024))) uint16_t lds[4 * kTile64];  // key buffers 0 and 1, value buffers 0 and 1
  const uint32_t bid = xcd_major(blockIdx.x, gridDim.x);
  const int per_seq = PAIRED ? a.pairs : a.q_tiles;
  const int u = int(bid) % per_seq, sh = int(bid) / per_seq;
  const int seq = sh % a.n_seq, head = sh / a.n_seq;
  const int g = (a.q_off + head) / a.group - a.kv_off;
  const int S = a.seq_len;
  const int64_t tok0 = int64_t(seq) * S;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 15, lh = lane >> 4;
  const uint16_t* const Qp = a.QKV + int64_t(head) * D;
  TileSrc<D> srcK, srcV;
  srcK.init(a.QKV + int64_t(a.q_cnt + g) * D + tok0 * a.ld, a.ld, S);
  srcV.init(a.QKV + int64_t(a.q_cnt + a.kv_cnt + g) * D + tok0 * a.ld, a.ld, S);
  Dma64 dma;
  dma.init(a.ld, wave, lane);
  Addr64 ad;
  ad.init(lds, lq, lh);
  auto ask = [&](int t, int buf) {  // rows past the sequence end arrive as zeros (masked below)
    dma.tile(srcK.rs, lds + buf * kTile64, wave, uint32_t(t) * srcK.step);
    dma.tile(srcV.rs, lds + (2 + buf) * kTile64, wave, uint32_t(t) * srcV.step);
  };

  for (int seg = 0; seg < (PAIRED ? 2 : 1); ++seg) {
    const int qt = PAIRED ? (seg == 0 ? a.q_tiles - 1 - u : u) : (a.causal ? a.q_tiles - 1 - u : u);
    if (seg == 1) {
      if (qt == a.q_tiles - 1 - u) break;  // odd tile count: the middle tile has no partner
      __syncthreads();                     // the first pass's last tile has been read by everyone
    }
    const int q0 = qt * kRows + wave * (16 * B);
    const int n_tiles = ((a.causal ? min(S, qt * kRows + kRows) : S) + kBKV - 1) / kBKV;
    ask(0, 0);
    bf16x8 qf[B][KS];
    f32x4 acc[B][DB];
    float m_run[B], l_run[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int qr = min(q0 + b * 16 + lq, S - 1);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) qf[b][ks] = *reinterpret_cast<const bf16x8*>(Qp + (tok0 + qr) * a.ld + ks * 32 + lh * 8);
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[b][db] = f32x4{0.f, 0.f, 0.f, 0.f};
      m_run[b] = -INFINITY;
      l_run[b] = 0.f;
    }

    auto step = [&](auto bufc, int t) {
      constexpr int BUF = decltype(bufc)::value;
      dma_done();       // this wavefront's share of tile t has landed ...
      __syncthreads();  // ... and everyone's; everyone has read the tile before
      if (t + 1 < n_tiles) ask(t + 1, BUF ^ 1);
      const int kv0 = t * kBKV;
      if (a.causal && kv0 > q0 + 16 * B - 1) return;  // every key of the tile lies after this wavefront's last query row
      attn_u32x4 kf[8];
      ad.rows<BUF>(kf);
      lds_reads_done(kf);
      attn_u32x2 v0[8], v1[8];
      ad.cols<2 + BUF, 0>(v0);
      ad.cols<2 + BUF, 1>(v1);
      // scores, transposed: [key kb*16 + (lane/16)*4 + r][query b*16 + lane%16]
      f32x4 st[B][4];
#pragma unroll
      for (int b = 0; b < B; ++b)
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
          st[b][kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) st[b][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[kb * KS + ks]), qf[b][ks], st[b][kb], 0, 0, 0);
        }
      const bool edge = kv0 + kBKV > S || (a.causal && kv0 + kBKV - 1 > q0);
      bf16x8 pf[B][2];
#pragma unroll
      for (int b = 0; b < B; ++b) {
        if (edge) {
          const int qrow = q0 + b * 16 + lq, last = (a.causal ? min(qrow, S - 1) : S - 1) - kv0 - lh * 4;
#pragma unroll
          for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (kb * 16 + r > last) st[b][kb][r] = -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int r = 0; r < 4; ++r) mx = fmaxf(mx, st[b][kb][r]);
        mx = xor_max(mx) * a.scale_log2;
        const float m_new = fmaxf(m_run[b], mx);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = fast_exp2(m_run[b] - m_use);
        float ls = 0.f, p[4][4];
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            p[kb][r] = fast_exp2(fmaf(st[b][kb][r], a.scale_log2, -m_use));
            ls += p[kb][r];
          }
        l_run[b] = l_run[b] * alpha + ls;
        m_run[b] = m_new;
        if (__any(alpha != 1.0f)) {
#pragma unroll
          for (int db = 0; db < DB; ++db) acc[b][db] *= alpha;
        }
        small_pack(p, pf[b]);
      }
      __builtin_amdgcn_sched_barrier(0);
      lds_reads_done(v0);
      lds_reads_tied(v1);
      products64<0>(v0, pf, acc);
      products64<1>(v1, pf, acc);
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = 0; t < n_tiles; t += 2) {
      step(std::integral_constant<int, 0>{}, t);
      if (t + 1 < n_tiles) step(std::integral_constant<int, 1>{}, t + 1);
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int qrow = q0 + b * 16 + lq;
      const float l = xor_sum(l_run[b]);
      const float inv = 1.0f / l;
      if (qrow >= S) continue;
      uint16_t* const cp = a.C + (tok0 + qrow) * a.ldc + int64_t(head) * D + lh * 4;
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        u16x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = ntp_gemm::f32_to_bf16(acc[b][db][r] * inv);
        *reinterpret_cast<u16x4*>(cp + db * 16) = o;
      }
      if (lh == 0 && a.LSE) a.LSE[int64_t(head) * (int64_t(a.n_seq) * S) + tok0 + qrow] = (m_run[b] + log2f(l)) * 0.6931471805599453f;
    }
  }  // the workgroup's passes
}
