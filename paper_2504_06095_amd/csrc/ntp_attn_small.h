// Attention core kernels for launches that are short of workgroups (included by ntp_attn_core.hip).
//
// The other kernels give a workgroup 64 rows and a walk over all tiles of the other side, one tile after the other; a small launch then has
// a few dozen workgroups whose time is the latency of their walks (12 sequences and heads x 512 causal tokens: 48 workgroups of nine steps of
// about 1 us).  Here a workgroup owns 16 rows, and its four wavefronts share out the walk: wavefront w takes tiles w, w + 4, ... in a part of
// the LDS of its own, so that nothing but the end needs a barrier; the four partial results are put together through LDS (in the order of
// the wavefronts).  Four times the workgroups, walks a quarter as long; what it costs is that a tile is read for 16 rows instead of 64, which is
// why larger launches keep the other kernels (small_pays).  Products and masks are those of the other kernels; but each wavefront has a running maximum of its own, so that
// probabilities are rounded to bf16 against another one, and partial sums are added in another order (results differ from theirs by 0.002, both are 0.0036 from 64 bits).  Head
// dimension 64, three heads, causal, forward and backward: 512 tokens 10.4 -> 5.0 and 18.8 -> 8.3 us, 1432 tokens 15.3 -> 8.6 and 35.5 -> 16.1; head dimension 128, 883
// tokens 18.7 -> 9.9 and 31.3 -> 20.3.  What bounds it then is the way into and out of a workgroup (about 3 us), and at 128 the DMA of four tiles a step (1.1 us).
//
// Tiles come by DMA as there.  Rows of D = 64 are 128 bytes: chunk c of row r sits at slot c ^ (((r >> 1) & 3) << 1), so that the 16 lanes that a
// 128-bit read serves at a time (see attn_core_fwd_dma_kernel) and the 8 rows x 32 bytes of a transposing read lie on distinct banks, as with row_swz at 128.

template <int D>
struct SmallTile {
  static constexpr int KS = D / 32, DB = D / 16, CPR = D / 8;  // K-steps of a row product, 16-column blocks, 16-byte chunks of a row
  static constexpr int BYTES = kBKV * D * 2, ROW = D * 2;      // of a tile, of a row
  static constexpr int NI = BYTES / 1024;                      // DMA instructions of a tile
  static __device__ __forceinline__ uint32_t swz(int r) { return D == 128 ? row_swz(r) : uint32_t(((r >> 1) & 3) << 1); }
  // lane offsets of the DMA instructions in a matrix of row length ld
  static __device__ __forceinline__ void dma_offsets(int64_t ld, int lane, uint32_t (&voff)[NI]) {
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int p = j * 64 + lane, row = p / CPR, slot = p % CPR;
      voff[j] = uint32_t((int64_t(row) * ld + int64_t(uint32_t(slot) ^ swz(row)) * 8) * 2);
    }
  }
  static __device__ __forceinline__ void dma(__amdgpu_buffer_rsrc_t rs, unsigned char* tile, const uint32_t (&voff)[NI], uint32_t soff) {
#pragma unroll
    for (int j = 0; j < NI; ++j) dma_16(rs, reinterpret_cast<uint16_t*>(tile + j * 1024), voff[j], soff);
  }
};

template <int... Is, typename F>
__device__ __forceinline__ void small_for(std::integer_sequence<int, Is...>, F&& f) {
  (f(std::integral_constant<int, Is>{}), ...);
}

// Workgroup b of a kind: its 16-row tile u and its (sequence, head) sh of `heads`.  Head by head, a head's tiles together on one XCD; or by length, the longest
// tiles of all heads first (small_by_length).  (One division and no branch; called once, before the backward kernel's two bodies part, of which the dQ body is the first in
// the code: with the same lines in either body, or the other order, launches of grouped heads took 1.04-1.09 of the time.)
__device__ __forceinline__ void small_place(uint32_t b, int tiles, int heads, bool by_length, int& u, int& sh) {
  const uint32_t major = xcd_major(b, uint32_t(tiles) * uint32_t(heads));
  const uint32_t bid = by_length ? b : major, n = uint32_t(by_length ? heads : tiles), quotient = bid / n, rest = bid - quotient * n;
  u = int(by_length ? quotient : rest);
  sh = int(by_length ? rest : quotient);
}

// This lane's read addresses in a tile at LDS address 0: rows (operand A, 16 rows a block) and transposed (operand A, 16 columns a block)
template <int D>
struct SmallAddr {
  using T = SmallTile<D>;
  uint32_t row[T::KS], col[T::DB];
  __device__ __forceinline__ void init(int lq, int lh) {
#pragma unroll
    for (int ks = 0; ks < T::KS; ++ks) row[ks] = uint32_t(lq) * T::ROW + ((uint32_t(ks * 4 + lh) ^ T::swz(lq)) * 16u);
    const int rv = lh * 4 + (lq >> 2);
#pragma unroll
    for (int db = 0; db < T::DB; ++db)
      col[db] = uint32_t(rv) * T::ROW + uint32_t(lq & 1) * 8u + ((uint32_t(db * 2 + ((lq & 3) >> 1)) ^ T::swz(rv)) * 16u);
  }
};

// (A group of reads is waited for before anything else happens: the compiler takes their registers as written at once, and short of registers
// it might move one that is still in flight.)
// All row fragments of a tile, f[rb * KS + ks]: rows rb * 16 + lane % 16, columns ks * 32 + lane / 16 * 8 on.
template <int D, int N>
__device__ __forceinline__ void small_rows(const SmallAddr<D>& ad, uint32_t tile, attn_u32x4 (&f)[N]) {
  using T = SmallTile<D>;
  static_assert(N == 4 * T::KS, "");
  small_for(std::make_integer_sequence<int, N>{}, [&](auto i) {
    constexpr int rb = decltype(i)::value / T::KS, ks = decltype(i)::value % T::KS;
    f[decltype(i)::value] = lds_frag_b128<rb * 16 * T::ROW>(tile + ad.row[ks]);
  });
}
// All transposed fragments, f[(db * 2 + s2) * 2 + half]: columns db * 16 + lane % 16, rows s2 * 32 + half * 16 + lane / 16 * 4 on.
template <int D, int N>
__device__ __forceinline__ void small_cols(const SmallAddr<D>& ad, uint32_t tile, attn_u32x2 (&f)[N]) {
  using T = SmallTile<D>;
  static_assert(N == 4 * T::DB, "");
  small_for(std::make_integer_sequence<int, N>{}, [&](auto i) {
    constexpr int db = decltype(i)::value / 4, q = decltype(i)::value % 4;
    f[decltype(i)::value] = lds_tr_b64<q * 16 * T::ROW>(tile + ad.col[db]);
  });
}
// The reads have arrived (see lds_reads_done).
template <int N, typename V>
__device__ __forceinline__ void small_reads_done(V (&f)[N]) {
  static_assert(N % 8 == 0, "");
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int i = 0; i < N; i += 8)
    asm volatile("" : "+v"(f[i]), "+v"(f[i + 1]), "+v"(f[i + 2]), "+v"(f[i + 3]), "+v"(f[i + 4]), "+v"(f[i + 5]), "+v"(f[i + 6]), "+v"(f[i + 7]) : : "memory");
#endif
}
__device__ __forceinline__ bf16x8 small_col_frag(attn_u32x2 lo, attn_u32x2 hi) {
  const attn_u32x4 both = {lo[0], lo[1], hi[0], hi[1]};
  return __builtin_bit_cast(bf16x8, both);
}
// 16 values of a lane as operand B of the second products: [32-row step]
__device__ __forceinline__ void small_pack(const float (&p)[4][4], bf16x8 (&f)[2]) {
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2) {
    bf16x8 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      v[r] = static_cast<__bf16>(p[2 * s2][r]);
      v[4 + r] = static_cast<__bf16>(p[2 * s2 + 1][r]);
    }
    f[s2] = v;
  }
}

// Forward: workgroup = 16 query rows of one (sequence, head).
// (a.pairs: nonzero where the tiles are dealt out by length)
template <int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(D == 128 ? 1 : 2, D == 128 ? 1 : 2))) void attn_core_fwd_small_kernel(const CoreArgs a) {
  using T = SmallTile<D>;
  constexpr int KS = T::KS, DB = T::DB;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[4 * 2 * T::BYTES];
  int u, sh;
  small_place(blockIdx.x, a.q_tiles, a.n_seq * a.q_cnt, a.pairs != 0, u, sh);
  const int qt = a.causal ? a.q_tiles - 1 - u : u;  // the longest walks first
  const int seq = sh % a.n_seq, head = sh / a.n_seq;
  const int g = (a.q_off + head) / a.group - a.kv_off;
  const int S = a.seq_len;
  const int64_t tok0 = int64_t(seq) * S;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 15, lh = lane >> 4;
  const int q0 = qt * 16, qrow = q0 + lq;
  unsigned char* const sK = lds + wave * (2 * T::BYTES);
  unsigned char* const sV = sK + T::BYTES;
  const uint32_t lK = uint32_t(reinterpret_cast<uintptr_t>(sK)), lV = lK + T::BYTES;
  TileSrc<D> srcK, srcV;
  srcK.init(a.QKV + int64_t(a.q_cnt + g) * D + tok0 * a.ld, a.ld, S);
  srcV.init(a.QKV + int64_t(a.q_cnt + a.kv_cnt + g) * D + tok0 * a.ld, a.ld, S);
  uint32_t voff[T::NI];
  T::dma_offsets(a.ld, lane, voff);
  SmallAddr<D> ad;
  ad.init(lq, lh);

  const int kv_end = a.causal ? min(S, q0 + 16) : S;
  const int n_tiles = (kv_end + kBKV - 1) / kBKV;
  bf16x8 qf[KS];
  {
    const uint16_t* const qp = a.QKV + int64_t(head) * D + (tok0 + min(qrow, S - 1)) * a.ld + lh * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 32);
  }
  auto ask = [&](int t) {
    T::dma(srcK.rs, sK, voff, uint32_t(t) * srcK.step);
    T::dma(srcV.rs, sV, voff, uint32_t(t) * srcV.step);
  };
  if (wave < n_tiles) ask(wave);
  f32x4 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  for (int t = wave; t < n_tiles; t += 4) {
    dma_done();
    attn_u32x4 kf[4 * KS];
    attn_u32x2 vf[4 * DB];
    small_rows<D>(ad, lK, kf);
    small_reads_done(kf);
    small_cols<D>(ad, lV, vf);
    small_reads_done(vf);
    if (t + 4 < n_tiles) ask(t + 4);  // (everything of this tile is in registers)
    f32x4 st[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      st[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) st[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[kb * KS + ks]), qf[ks], st[kb], 0, 0, 0);
    }
    const int kv0 = t * kBKV;
    if (kv0 + kBKV > S || (a.causal && kv0 + kBKV - 1 > q0)) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = kv0 + kb * 16 + lh * 4 + r;
          if (key >= S || (a.causal && key > qrow)) st[kb][r] = -INFINITY;
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = fmaxf(mx, st[kb][r]);
    mx = xor_max(mx) * a.scale_log2;
    const float m_new = fmaxf(m_run, mx);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = fast_exp2(m_run - m_use);
    float ls = 0.f, p[4][4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[kb][r] = fast_exp2(fmaf(st[kb][r], a.scale_log2, -m_use));
        ls += p[kb][r];
      }
    l_run = l_run * alpha + ls;
    m_run = m_new;
    if (__any(alpha != 1.0f)) {
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[db] *= alpha;
    }
    bf16x8 pf[2];
    small_pack(p, pf);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
        acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(small_col_frag(vf[(db * 2 + s2) * 2], vf[(db * 2 + s2) * 2 + 1]), pf[s2], acc[db], 0, 0, 0);
  }

  // The four wavefronts' rows: outputs, maximum and sum, to this wavefront's part of the LDS (its tiles have been read).
  constexpr int LDO = D + 4;
  float* const mine = reinterpret_cast<float*>(sK);
  {
    const float l = xor_sum(l_run);
#pragma unroll
    for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(mine + lq * LDO + db * 16 + lh * 4) = acc[db];
    if (lh == 0) {
      mine[lq * LDO + D] = m_run;
      mine[lq * LDO + D + 1] = l;
    }
  }
  __syncthreads();
  constexpr int W = D / 16;  // columns of a lane: wavefront w, lane / 16 = h: (4 w + h) W on
  const float* const all = reinterpret_cast<const float*>(lds) + lq * LDO;
  constexpr int PART = 2 * T::BYTES / 4;  // floats from one wavefront's part to the next
  float m = -INFINITY;
#pragma unroll
  for (int w = 0; w < 4; ++w) m = fmaxf(m, all[w * PART + D]);
  const float m_use = m == -INFINITY ? 0.f : m;
  float l = 0.f, o[W];
#pragma unroll
  for (int c = 0; c < W; ++c) o[c] = 0.f;
  const int c0 = (wave * 4 + lh) * W;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float f = fast_exp2(all[w * PART + D] - m_use);
    l += f * all[w * PART + D + 1];
#pragma unroll
    for (int c = 0; c < W; c += 4) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(all + w * PART + c0 + c);
#pragma unroll
      for (int r = 0; r < 4; ++r) o[c + r] += f * v[r];
    }
  }
  if (qrow >= S) return;
  const float inv = 1.0f / l;
  uint16_t* const cp = a.C + (tok0 + qrow) * a.ldc + int64_t(head) * D + c0;
#pragma unroll
  for (int c = 0; c < W; c += 4) {
    u16x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = ntp_gemm::f32_to_bf16(o[c + r] * inv);
    *reinterpret_cast<u16x4*>(cp + c) = v;
  }
  if (wave == 0 && lh == 0 && a.LSE) a.LSE[int64_t(head) * (int64_t(a.n_seq) * S) + tok0 + qrow] = (m + log2f(l)) * 0.6931471805599453f;
}

// Sums of the four wavefronts' rows (NB blocks of 16 columns), f times, as bf16 to rows of ld from dst on; columns as in the forward kernel.
template <int D, int NB, typename Out>
__device__ __forceinline__ void small_sum(unsigned char* lds, int wave, int lq, int lh, const f32x4 (&acc)[NB], Out&& out) {
  constexpr int W = NB, LDO = NB * 16 + 4, PART = 2 * SmallTile<D>::BYTES / 4;
  float* const mine = reinterpret_cast<float*>(lds) + wave * PART + lq * LDO;
#pragma unroll
  for (int b = 0; b < NB; ++b) *reinterpret_cast<f32x4*>(mine + b * 16 + lh * 4) = acc[b];
  __syncthreads();
  const int c0 = (wave * 4 + lh) * W;
  const float* const all = reinterpret_cast<const float*>(lds) + lq * LDO + c0;
#pragma unroll
  for (int c = 0; c < W; c += 4) {
    f32x4 s = *reinterpret_cast<const f32x4*>(all + c);
#pragma unroll
    for (int w = 1; w < 4; ++w) s = s + *reinterpret_cast<const f32x4*>(all + w * PART + c);
    out(c0 + c, s);
  }
}

// dQ: 16 query rows of one (sequence, head); u: their tile, the longest walk first.
template <int D, bool STORE_DELTA>
__device__ __forceinline__ void bwd_dq_small_body(const CoreBwdArgs& a, const int u, const int sh, unsigned char* const lds) {
  using T = SmallTile<D>;
  constexpr int KS = T::KS, DB = T::DB;
  const int qt = a.causal ? a.tiles - 1 - u : u;
  const int seq = sh % a.n_seq, head = sh / a.n_seq;
  const int g = (a.q_off + head) / a.group - a.kv_off;
  const int S = a.seq_len;
  const int64_t tok0 = int64_t(seq) * S, Mtot = int64_t(a.n_seq) * S;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 15, lh = lane >> 4;
  const int q0 = qt * 16, qrow = q0 + lq;
  unsigned char* const sK = lds + wave * (2 * T::BYTES);
  unsigned char* const sV = sK + T::BYTES;
  const uint32_t lK = uint32_t(reinterpret_cast<uintptr_t>(sK)), lV = lK + T::BYTES;
  TileSrc<D> srcK, srcV;
  srcK.init(a.QKV + int64_t(a.q_cnt + g) * D + tok0 * a.ld, a.ld, S);
  srcV.init(a.QKV + int64_t(a.q_cnt + a.kv_cnt + g) * D + tok0 * a.ld, a.ld, S);
  uint32_t voff[T::NI];
  T::dma_offsets(a.ld, lane, voff);
  SmallAddr<D> ad;
  ad.init(lq, lh);
  const int kv_end = a.causal ? min(S, q0 + 16) : S;
  const int n_tiles = (kv_end + kBKV - 1) / kBKV;
  bf16x8 qf[KS], gf[KS];
  float lse2, delta;
  {
    const int qr = min(qrow, S - 1);
    float part = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qf[ks] = *reinterpret_cast<const bf16x8*>(a.QKV + int64_t(head) * D + (tok0 + qr) * a.ld + ks * 32 + lh * 8);
      gf[ks] = *reinterpret_cast<const bf16x8*>(a.dC + (tok0 + qr) * a.lddc + int64_t(head) * D + ks * 32 + lh * 8);
      const bf16x8 of = *reinterpret_cast<const bf16x8*>(a.C + (tok0 + qr) * a.ldc + int64_t(head) * D + ks * 32 + lh * 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) part += float(gf[ks][e]) * float(of[e]);
    }
    delta = xor_sum(part);
    lse2 = a.LSE[int64_t(head) * Mtot + tok0 + qr] * 1.4426950408889634f;
    if (STORE_DELTA && wave == 0 && lh == 0 && qrow < S) a.Delta[int64_t(head) * Mtot + tok0 + qrow] = delta;
  }
  auto ask = [&](int t) {
    T::dma(srcK.rs, sK, voff, uint32_t(t) * srcK.step);
    T::dma(srcV.rs, sV, voff, uint32_t(t) * srcV.step);
  };
  if (wave < n_tiles) ask(wave);
  f32x4 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int t = wave; t < n_tiles; t += 4) {
    dma_done();
    attn_u32x4 kf[4 * KS], vf[4 * KS];
    attn_u32x2 kt[4 * DB];
    small_rows<D>(ad, lK, kf);
    small_reads_done(kf);
    small_rows<D>(ad, lV, vf);
    small_reads_done(vf);
    small_cols<D>(ad, lK, kt);
    small_reads_done(kt);
    if (t + 4 < n_tiles) ask(t + 4);
    f32x4 st[4], dpt[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      st[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
      dpt[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        st[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[kb * KS + ks]), qf[ks], st[kb], 0, 0, 0);
        dpt[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[kb * KS + ks]), gf[ks], dpt[kb], 0, 0, 0);
      }
    }
    const int kv0 = t * kBKV;
    float ds[4][4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) ds[kb][r] = fast_exp2(fmaf(st[kb][r], a.scale_log2, -lse2));
    if (kv0 + kBKV > S || (a.causal && kv0 + kBKV - 1 > q0)) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = kv0 + kb * 16 + lh * 4 + r;
          if (key >= S || (a.causal && key > qrow)) ds[kb][r] = 0.f;
        }
    }
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) ds[kb][r] *= dpt[kb][r] - delta;
    bf16x8 dsf[2];
    small_pack(ds, dsf);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
        acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(small_col_frag(kt[(db * 2 + s2) * 2], kt[(db * 2 + s2) * 2 + 1]), dsf[s2], acc[db], 0, 0, 0);
  }
  small_sum<D>(lds, wave, lq, lh, acc, [&](int c, f32x4 s) {
    if (qrow >= S) return;
    u16x4 o;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = ntp_gemm::f32_to_bf16(s[r] * a.scale);
    *reinterpret_cast<u16x4*>(a.dQKV + (tok0 + qrow) * a.ldd + int64_t(head) * D + c) = o;
  });
}

// dK and dV: the 16 keys of tile kt (early ones have the longest walks) of one (sequence, KV head); the walk goes over the query tiles of every query head that reads it.
// (FORM_DELTA: the rows' delta values are formed from their rows of C, which are read with the tile; else a launch before this one has stored them.)
template <int D, bool FORM_DELTA>
__device__ __forceinline__ void bwd_dkv_small_body(const CoreBwdArgs& a, const int kt, const int sh, unsigned char* const lds, float (*const sLD)[2][kBKV]) {
  using T = SmallTile<D>;
  constexpr int KS = T::KS, DB = T::DB;
  const int seq = sh % a.n_seq, g = sh / a.n_seq;  // g: local KV head
  const int S = a.seq_len;
  const int64_t tok0 = int64_t(seq) * S, Mtot = int64_t(a.n_seq) * S;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 15, lh = lane >> 4;
  const int k0 = kt * 16, key = k0 + lq;
  unsigned char* const sQ = lds + wave * (2 * T::BYTES);
  unsigned char* const sG = sQ + T::BYTES;
  const uint32_t lQ = uint32_t(reinterpret_cast<uintptr_t>(sQ)), lG = lQ + T::BYTES;
  uint32_t voffq[T::NI], voffg[T::NI];
  T::dma_offsets(a.ld, lane, voffq);
  T::dma_offsets(a.lddc, lane, voffg);
  SmallAddr<D> ad;
  ad.init(lq, lh);
  // the walk: query heads [h_lo, h_hi) read this KV head, query tiles [t_lo, t_hi) of each see a key of these
  const int h_lo = max(0, (a.kv_off + g) * a.group - a.q_off), h_hi = min(a.q_cnt, (a.kv_off + g + 1) * a.group - a.q_off);
  const int t_lo = a.causal ? k0 / kBKV : 0, nt = (S + kBKV - 1) / kBKV - t_lo;
  const int units = max(h_hi - h_lo, 0) * nt;
  bf16x8 kf[KS], vf[KS];
  {
    const int64_t row = (tok0 + min(key, S - 1)) * a.ld + lh * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      kf[ks] = *reinterpret_cast<const bf16x8*>(a.QKV + int64_t(a.q_cnt + g) * D + row + ks * 32);
      vf[ks] = *reinterpret_cast<const bf16x8*>(a.QKV + int64_t(a.q_cnt + a.kv_cnt + g) * D + row + ks * 32);
    }
  }
  float rl = 0.f, rd = 0.f;  // of the tile's row `lane`
  bf16x8 cf[4 * KS];         // FORM_DELTA: the tile's rows of C, laid out as the fragments of dC
  auto ask = [&](int unit) {
    const int head = h_lo + unit / nt, t = t_lo + unit % nt;
    TileSrc<D> srcQ, srcG;
    srcQ.init(a.QKV + int64_t(head) * D + tok0 * a.ld, a.ld, S);
    srcG.init(a.dC + int64_t(head) * D + tok0 * a.lddc, a.lddc, S);
    const int64_t row = int64_t(head) * Mtot + tok0 + min(t * kBKV + lane, S - 1);
    rl = a.LSE[row] * 1.4426950408889634f;
    if constexpr (FORM_DELTA) {
#pragma unroll
      for (int qb = 0; qb < 4; ++qb) {
        const uint16_t* const cp = a.C + (tok0 + min(t * kBKV + qb * 16 + lq, S - 1)) * a.ldc + int64_t(head) * D + lh * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) cf[qb * KS + ks] = *reinterpret_cast<const bf16x8*>(cp + ks * 32);
      }
    } else {
      rd = a.Delta[row];
    }
    T::dma(srcQ.rs, sQ, voffq, uint32_t(t) * srcQ.step);
    T::dma(srcG.rs, sG, voffg, uint32_t(t) * srcG.step);
  };
  if (wave < units) ask(wave);
  f32x4 acc[2 * DB];  // dK, then dV
#pragma unroll
  for (int i = 0; i < 2 * DB; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int unit = wave; unit < units; unit += 4) {
    const int qbase = (t_lo + unit % nt) * kBKV;
    dma_done();
    sLD[wave][0][lane] = rl;
    if constexpr (!FORM_DELTA) sLD[wave][1][lane] = rd;
    attn_u32x4 qf[4 * KS], gf[4 * KS];
    small_rows<D>(ad, lQ, qf);
    small_reads_done(qf);
    small_rows<D>(ad, lG, gf);
    small_reads_done(gf);
    if constexpr (FORM_DELTA) {
      // sum_d dC C is the diagonal of a product of 16-row blocks, row r of which is in the lanes with lane % 16 = r and lane / 16 = r / 4
#pragma unroll
      for (int qb = 0; qb < 4; ++qb) {
        f32x4 dd = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) dd = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, gf[qb * KS + ks]), cf[qb * KS + ks], dd, 0, 0, 0);
        const float lo = lq & 1 ? dd[1] : dd[0], hi = lq & 1 ? dd[3] : dd[2];
        if ((lq >> 2) == lh) sLD[wave][1][qb * 16 + lq] = lq & 2 ? hi : lo;
      }
    }
    f32x4 l4[4], d4[4];
#pragma unroll
    for (int qb = 0; qb < 4; ++qb) {
      l4[qb] = *reinterpret_cast<const f32x4*>(&sLD[wave][0][qb * 16 + lh * 4]);
      d4[qb] = *reinterpret_cast<const f32x4*>(&sLD[wave][1][qb * 16 + lh * 4]);
    }
    // S and dP blocks: [query qb*16 + (lane/16)*4 + r][key lane%16]
    f32x4 sc[4], dp[4];
#pragma unroll
    for (int qb = 0; qb < 4; ++qb) {
      sc[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
      dp[qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        sc[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, qf[qb * KS + ks]), kf[ks], sc[qb], 0, 0, 0);
        dp[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, gf[qb * KS + ks]), vf[ks], dp[qb], 0, 0, 0);
      }
    }
    const bool edge = qbase + kBKV > S || k0 + 16 > S || (a.causal && qbase < k0 + 15);
    float p[4][4], ds[4][4];
#pragma unroll
    for (int qb = 0; qb < 4; ++qb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[qb][r] = fast_exp2(fmaf(sc[qb][r], a.scale_log2, -l4[qb][r]));
        ds[qb][r] = dp[qb][r] - d4[qb][r];
      }
    if (edge) {
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
    bf16x8 pf[2], dsf[2];
    small_pack(p, pf);
    small_pack(ds, dsf);
    attn_u32x2 qt[4 * DB], gt[4 * DB];
    small_cols<D>(ad, lG, gt);
    small_reads_done(gt);
    small_cols<D>(ad, lQ, qt);
    small_reads_done(qt);
    if (unit + 4 < units) ask(unit + 4);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        acc[DB + db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(small_col_frag(gt[(db * 2 + s2) * 2], gt[(db * 2 + s2) * 2 + 1]), pf[s2], acc[DB + db], 0, 0, 0);
        acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(small_col_frag(qt[(db * 2 + s2) * 2], qt[(db * 2 + s2) * 2 + 1]), dsf[s2], acc[db], 0, 0, 0);
      }
  }
  small_sum<D>(lds, wave, lq, lh, acc, [&](int c, f32x4 s) {
    if (key >= S) return;
    const bool is_v = c >= D;
    u16x4 o;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = ntp_gemm::f32_to_bf16(s[r] * (is_v ? 1.0f : a.scale));
    *reinterpret_cast<u16x4*>(a.dQKV + (tok0 + key) * a.ldd + int64_t(a.q_cnt + (is_v ? a.kv_cnt : 0) + g) * D + (is_v ? c - D : c)) = o;
  });
}

// Both in one launch: dK/dV workgroups first (their walks are the longer ones).  a.pairs: 1 the queries', 2 the keys' tiles are dealt out by length.  DELTA: they form the rows' delta values for themselves and the dQ workgroups store
// them, instead of a launch before this one (small_forms_delta).
template <int D, bool DELTA>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(D == 128 ? 1 : 2, D == 128 ? 1 : 2))) void attn_core_bwd_small_kernel(const CoreBwdArgs a, const uint32_t n_dkv) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[4 * 2 * SmallTile<D>::BYTES];
  __shared__ __attribute__((aligned(16))) float sLD[4][2][kBKV];
  const bool dkv = blockIdx.x < n_dkv;
  int u, sh;
  small_place(dkv ? blockIdx.x : blockIdx.x - n_dkv, a.tiles, a.n_seq * (dkv ? a.kv_cnt : a.q_cnt), (a.pairs & (dkv ? 2 : 1)) != 0, u, sh);
  if (!dkv) bwd_dq_small_body<D, DELTA>(a, u, sh, lds);
  else bwd_dkv_small_body<D, DELTA>(a, u, sh, lds, sLD);
}
