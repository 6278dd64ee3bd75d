// bf16 MFMA GEMM family for the NTP shard layers (Sec. 3.1, Eq. 2-3 and 4, 6, and
// their chain-rule gradients): C[M x N] = op(A) op(B) with fp32 accumulation and a
// fused epilogue (bf16 store, GeLU, GeLU', fp32 store / accumulate).
//
// Any M, N, K is accepted: ragged shard widths show up as N (column-parallel
// forward), as K (row-parallel forward, dX) and as M (weight gradients).  Rows and
// columns past the edge are never stored; the K tail is zero-filled in LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdint>
#include <cstring>
#include <type_traits>

#include "ntp_gemm_kernels.h"
#include "ntp_gemm_launch.h"
#include "ntp_internal.h"

namespace {

using namespace ntp_gemm;

template <typename F>
int dispatch_epilogue(int epi, F&& f) {
  switch (epi) {
    case ntp::EPI_BF16: return f(std::integral_constant<int, ntp::EPI_BF16>{});
    case ntp::EPI_GELU: return f(std::integral_constant<int, ntp::EPI_GELU>{});
    case ntp::EPI_DGELU: return f(std::integral_constant<int, ntp::EPI_DGELU>{});
    case ntp::EPI_F32: return f(std::integral_constant<int, ntp::EPI_F32>{});
    case ntp::EPI_F32_ACCUM: return f(std::integral_constant<int, ntp::EPI_F32_ACCUM>{});
    default: return NTP_ERR_INVALID_ARG;
  }
}

template <bool AKC, bool BKC>
int launch_generic(GemmArgs g, int epi, hipStream_t s) {
  g.tiles_m = (g.M + BM - 1) / BM;
  g.tiles_n = (g.n_store + BN - 1) / BN;
  if (int64_t(g.tiles_m) * g.tiles_n > 0x7fffffff) return NTP_ERR_UNSUPPORTED;
  const dim3 grid(uint32_t(g.tiles_m) * uint32_t(g.tiles_n)), block(256);
  return dispatch_epilogue(epi, [&](auto e) {
    hipLaunchKernelGGL((gemm_generic_kernel<AKC, BKC, decltype(e)::value>), grid, block, 0, s, g);
    return hipGetLastError() == hipSuccess ? NTP_OK : NTP_ERR_LAUNCH;
  });
}

// Relative throughput of one workgroup per tile shape at full occupancy, per operand layout: smaller wavefront tiles read more LDS fragments
// per MFMA, smaller workgroup tiles move more bytes per flop.  Fitted to 2500 random GEMMs (all layouts, 8 to 450 GFLOP, operands streaming from
// HBM), every tile shape timed on each, with the ping-pong kernel on the 8-wavefront tiles: the tile that the table picks takes 1.012 (A, B K-contiguous), 1.003
// and 1.009 of the best tile's time on the mean (with the table made for the ring schedule 1.014, 1.021 and 1.016).
// The 4-wavefront 128 x 128 variant reaches its rate with two workgroups on a compute unit; alone on one
// (at most 256 tiles) it runs at kLoneSmallTileRate, where the 8-wavefront variant of the same tile is faster; with both operands K-strided it always is.
//                                             256x256 256x224 224x256 256x192 192x256 256x128 128x256 128x128 128x128w8
constexpr double kTileRate[3][kNumTileShapes] = {{1.050, 1.008, 0.945, 0.924, 0.975, 0.714, 0.764, 0.60, 0.53},   // A, B K-contiguous
                                                 {1.100, 0.977, 1.055, 1.023, 1.029, 0.705, 0.816, 0.60, 0.53},   // B K-strided
                                                 {1.080, 1.007, 1.107, 0.985, 1.000, 0.806, 0.883, 0.50, 0.53}};  // both K-strided
constexpr double kLoneSmallTileRate = 0.43;
// The rates that decide what a GEMM is before it gets its tile: whether its K axis is cut and into how many chunks, and whether the deep-pipelined kernel takes it.
// They and the constants of choose_split were measured with the ring schedule and stay: the chunks fix the order of a product's fp32 sums, what
// ntp_workspace_bytes reports and which shapes the call with static scratch takes.  The rates above in their place, with a reduce refitted to them, gave 36 of
// 20000 random products other chunks (4096 x 640 over K = 8192: five instead of three, 60.0 us instead of 63.6 with 52 MB of workspace instead of 31) and cut
// products that run whole on 128 x 256 tiles without weighing that kernel.
constexpr double kPlanRate[3][kNumTileShapes] = {{1.000, 0.957, 0.969, 0.917, 0.923, 0.761, 0.754, 0.65, 0.53},
                                                 {1.000, 0.929, 0.986, 0.908, 0.944, 0.770, 0.749, 0.65, 0.53},
                                                 {1.100, 0.984, 1.000, 0.956, 0.962, 0.797, 0.779, 0.65, 0.53}};

// Pick the tile shape with the least estimated time: the busiest compute unit's number of
// workgroups (they are dealt evenly; co-resident ones share its throughput) times tile area over rate.
int choose_tile(const double (&rates)[3][kNumTileShapes], int64_t M, int64_t N, int layout, int cus) {
  int best = 0;
  double best_t = 1e300;
  for (int i = 0; i < kNumTileShapes; ++i) {
    const TileShape& ts = kTileShapes[i];
    const int64_t tiles = ((M + ts.bm - 1) / ts.bm) * ((N + ts.bn - 1) / ts.bn);
    const int64_t cu_load = (tiles + cus - 1) / cus;
    const double rate = ts.waves == 4 && tiles <= cus ? kLoneSmallTileRate : rates[layout][i];
    const double t = double(cu_load) * ts.bm * ts.bn / rate;
    if (t < best_t) {
      best_t = t;
      best = i;
    }
  }
  return best;
}

void variant_name(int v, char* out, size_t n) {
  if (v < 0) snprintf(out, n, "generic128");
  else if (kTileShapes[v].bm == 128 && kTileShapes[v].bn == 128 && kTileShapes[v].waves == 8) snprintf(out, n, "128x128w8");
  else snprintf(out, n, "%dx%d", kTileShapes[v].bm, kTileShapes[v].bn);
}

// Variant used for a shape: -1 = generic kernel, else an index into kTileShapes.  The handle's
// NTP_OPT_GEMM_TILE overrides the choice (1: generic, 2 + i: tile shape i).
int choose_variant(const ntp_handle* h, const GemmArgs& g, bool ring_ok, int layout) {
  if (const int64_t f = h->opt[NTP_OPT_GEMM_TILE]) {
    if (!ring_ok || f == 1) return -1;
    if (f - 2 < kNumTileShapes) return int(f - 2);
  }
  // the generic 128x128x32 kernel only below two output tiles or two K tiles: from there on the ring kernel
  // measured faster (512 x 586 x 1024: 15 us against 31 us per GEMM)
  if (int64_t(g.M) * g.N < 128 * 128 * 2 || g.K < 128) return -1;
  if (!ring_ok) return -1;
  return choose_tile(kPlanRate, g.M, g.n_store, layout, h->compute_units);
}

// (layout, epilogue) pairs the shard layers use have ring instantiations; anything else runs on
// the generic kernel
bool ring_combo(bool a_kc, bool b_kc, int epi) {
  if (a_kc && b_kc) return epi == ntp::EPI_BF16 || epi == ntp::EPI_GELU || epi == ntp::EPI_DGELU;
  if (a_kc && !b_kc) return epi == ntp::EPI_BF16;
  if (!a_kc && !b_kc) return epi == ntp::EPI_F32 || epi == ntp::EPI_F32_ACCUM;
  return false;
}

// ---- split-K ---------------------------------------------------------------------
// A column-parallel shard at a high TP degree is a skinny GEMM: few output tiles, long K.  With
// fewer tiles than compute units the K axis is cut as well: `splits` workgroups per tile store fp32
// partial sums to a caller-provided workspace, and a second kernel adds the slices in ascending
// order and applies the epilogue.
struct SplitChoice {
  int tile, splits, k_chunk;
  int deep;  // DeepForm
};

constexpr double kTileCycles = 2650.0;      // one 256 x 256 x 64 K tile on one compute unit at rate 1
constexpr int kTileOverhead = 4;            // prologue and epilogue of an output tile, in K tiles
constexpr double kReduceBytesPerCycle = 2000.0, kReduceFixedCycles = 6000.0;
constexpr int kMaxSplits = 8, kMinSplitTiles = 8;

// Workgroups of the busiest XCD's share of a launch with `splits` K chunks a tile: a tile and its chunks are on one XCD, so that 85 tiles in three
// chunks are 33 workgroups on five of the XCDs and 30 on the others, whose 32 compute units take them in two rounds (2066 x 536 over K =
// 3992: 43 us; in two chunks 31).
int64_t xcd_load(int64_t tiles, int64_t splits) { return (tiles + 7) / 8 * splits; }

double tile_time(int64_t M, int64_t N, int64_t ktiles, int layout, int i, int splits, int cus) {
  const TileShape& ts = kTileShapes[i];
  const int64_t tiles = ((M + ts.bm - 1) / ts.bm) * ((N + ts.bn - 1) / ts.bn);
  const int64_t units = std::max(cus / 8, 1), cu_load = splits == 1 ? (tiles + cus - 1) / cus : (xcd_load(tiles, splits) + units - 1) / units;
  const double rate = ts.waves == 4 && tiles <= cus ? kLoneSmallTileRate : kPlanRate[layout][i];
  const int64_t kt = (ktiles + splits - 1) / splits + kTileOverhead;
  return double(cu_load) * double(kt) * kTileCycles * (ts.bm * ts.bn / 65536.0) / rate;
}

// Least estimated time over (tile shape, splits); splits == 1 means: leave the GEMM as it is.
// ws_bytes: room for the partial sums (0: never split).
SplitChoice choose_split(const ntp_handle* h, int64_t ws_bytes, int64_t M, int64_t N, int64_t K, int layout, int plain_tile,
                         int64_t ldw) {
  SplitChoice best{plain_tile, 1, 0, kNotDeep};
  const int64_t ktiles = (K + 63) / 64;
  const int cus = h->compute_units;
  const int forced = int(h->opt[NTP_OPT_GEMM_SPLIT]);  // 1: never split; n > 1: n chunks if they fit
  const int64_t forced_tile = h->opt[NTP_OPT_GEMM_TILE];
  if (ws_bytes <= 0 || forced == 1) return best;
  // splitting has to beat the plain launch by a margin: the estimate is coarse
  double best_t = plain_tile >= 0 ? 0.85 * tile_time(M, N, ktiles, layout, plain_tile, 1, cus) : 1e300;
  if (forced > 1) best_t = 1e300;
  for (int i = 0; i < kNumTileShapes; ++i) {
    if (!kSplitTile[i]) continue;
    if (forced_tile >= 2 && forced_tile - 2 != i) continue;
    for (int sp = 2; sp <= kMaxSplits; ++sp) {
      if (forced > 1 && sp != forced) continue;
      const int64_t chunk_tiles = (ktiles + sp - 1) / sp;
      if (forced <= 1 && chunk_tiles < kMinSplitTiles) break;
      if ((sp - 1) * chunk_tiles * 64 >= K) continue;  // the last chunk would be empty
      if (int64_t(sp) * M * ldw * 4 > ws_bytes) break;
      const double reduce = kReduceFixedCycles + double(M) * double(N) * (4.0 * sp + 4.0) / kReduceBytesPerCycle;
      const double t = tile_time(M, N, ktiles, layout, i, sp, cus) + reduce;
      if (t < best_t) {
        best_t = t;
        best = SplitChoice{i, sp, int(chunk_tiles * 64), kNotDeep};
      }
    }
  }
  return best;
}

// Adds the partial-sum slices of a split-K launch and applies the GEMM's own epilogue.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const GemmArgs g, const float* __restrict__ ws, int64_t slice,
                                                            int64_t ldw, int splits) {
  const int quads = g.n_store >> 2;  // n_store is a multiple of 4
  const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int64_t m = idx / quads;
  if (m >= g.M) return;
  const int n0 = int(idx - m * quads) * 4;
  const float* p = ws + m * ldw + n0;
  f32x4 acc = *reinterpret_cast<const f32x4*>(p);
  for (int s = 1; s < splits; ++s) acc = acc + *reinterpret_cast<const f32x4*>(p + s * slice);
  store4<EPI>(g, int(m), n0, acc);
}

constexpr int kDeepTile = 8, kDeepWideTile = 6;  // indices of the deep-pipelined kernel's tile shapes
constexpr int kMaxDeepSplits = 16;
constexpr double kSmallTileUs = 0.225;  // a K tile of the 64 x 64 form
// K tiles of a piece in that form.  No measurement sets this line: K axes of 2048 and more stay cut on 128 x 128 tiles, as they were before this form
// came and as callers that set a workspace for it (and the tests of cut products) have it, also where one piece is faster: 2048 x 584 over
// K = 2048 16.2 us in one piece, 20.3 in three.
constexpr int kMaxSmallChunk = 31;
// K tiles of a shared launch's longest problem from which it may take that form (with 16 both take 14 us: 512 x 1024 x 586).
constexpr double kGroupSmallFrom = 24;
constexpr double kSmallPerUnit = 2.0;  // workgroups of that form per compute unit at a time

// Whether the deep-pipelined kernel takes over from `old`, and in how many K chunks.  Measured over 45 random shapes of up to one
// 128 x 128 tile per compute unit, all layouts: against the persistent kernels on 128 x 128 tiles it is never slower (2 % at
// five K tiles, 20-45 % at 10-60, up to 5.5 times where few tiles meet a long K axis that was not cut: 752 x 160 over K = 9544
// 125 -> 22 us); against larger tiles with a cut K axis it is 15-45 % faster up to half as many tiles as compute units (224 x
// 4344 over K = 6136: 50 -> 33 us) and slower above (280 x 7944 over K = 9152, 189 tiles: 75 -> 83 us).
// Chunks: every one has a compute unit to itself.  A K tile takes 0.47 us (LDS reads: 96 KB a K tile and workgroup), the reduce launch 3.5 us
// and its traffic at 4.4 TB/s; a chunk has at least four K tiles.
//
// Above one tile per compute unit, for a K axis that is not cut (32 random shapes):
//  - weight gradients up to nine K tiles, any number of tiles: the time is the output's, and two workgroups on a compute unit keep storing
//    while the next tile loads: 4456 x 7936 over K = 152 50 -> 43 us, 8072 x 3704 over 568 67 -> 60 us, 15520 x 11640 over 152
//    267 -> 216 us and accumulating 502 -> 406 us (-14 to +1 %; at ten K tiles and more the larger tiles win);
//  - 128 x 256 tiles that all fit on the device at once, from 20 K tiles on: 10160 x 432 over K = 1496 34 -> 27 us, 368 x 16040 over
//    1584 34 -> 31 us, 1376 x 4672 over 3440 56 -> 54 us;
//  - up to two 128 x 128 tiles per compute unit and 25 K tiles (weight gradients: 32): 1984 x 2664 over K = 328 16 -> 13.5 us, 584 x 7304
//    over 1400 28 -> 25 us, 2192 x 2304 over 1888 38 -> 35 us; at 54 K tiles 10 % slower.
SplitChoice choose_deep(const ntp_handle* h, int64_t ws_bytes, int layout, int64_t M, int64_t N, int64_t K, int64_t ldw, const SplitChoice& old, bool small_ok) {
  const TileShape& ts = kTileShapes[old.tile];
  const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128), wide = ((M + 127) / 128) * ((N + 255) / 256), ktiles = (K + 63) / 64;
  const int cus = h->compute_units;
  if (tiles > cus) {
    const SplitChoice deep2{kDeepTile, 1, int(ktiles * 64), kDeep2};
    if (old.splits > 1) return old;
    if (layout == 2 && ktiles <= 9) return deep2;
    if (wide <= cus && ktiles >= 20) return SplitChoice{kDeepWideTile, 1, int(ktiles * 64), kDeepWide};
    return tiles <= 2 * cus && ktiles <= (layout == 2 ? 32 : 25) ? deep2 : old;
  }
  if (old.splits > 1 ? tiles * 2 > cus : ts.bm != 128 || ts.bn != 128) return old;
  SplitChoice best{kDeepTile, 1, int(ktiles * 64), kDeep5};
  double best_t = 0.47 * double(ktiles);
  for (int sp = 2; sp <= kMaxDeepSplits && xcd_load(tiles, sp) * 8 <= cus; ++sp) {
    const int64_t chunk_tiles = (ktiles + sp - 1) / sp;
    if (chunk_tiles < 4 || int64_t(sp) * M * ldw * 4 > ws_bytes) break;
    if ((sp - 1) * chunk_tiles * 64 >= K) continue;  // the last chunk would be empty
    const double t = 0.47 * double(chunk_tiles) + 3.5 + double(M) * double(ldw) * (4.0 * sp + 4.0) / 4.4e6;
    if (t < best_t) {
      best_t = t;
      best = SplitChoice{kDeepTile, sp, int(chunk_tiles * 64), kDeep5};
    }
  }
  // Where the caller has set a workspace, the same with 64 x 64 tiles, which need a cut less often: up to two on a compute unit at a time,
  // which share its rate (both sides in ntp_gemm_deep.h; without a workspace, and below six K tiles, whose launches are mostly fixed
  // costs, the tiles stay 128 x 128; so do weight gradients, which share a launch where they are small).  Not more than two: 576 x 3776 over K = 1024
  // (2.07 per unit) takes 13.5 us, 10.7 with 128 x 128 tiles, over 1984 22.4 and 16.4, where 2048 x 1024 (2.0) takes 9.7 and 10.5, 13.3 and
  // 16.4.  Nor, uncut, more than 1.3 where both operands are K-contiguous and their rows do not start on cache lines (twice the lines a
  // tile): 640 x 2304 over K = 1264 (1.41) 13.4 and 12.0, 2048 x 1024 over 1264 13.6 and 12.8; 1664 x 640 over 1904 (1.02) 15.2 and 21.1.
  if (!small_ok || layout == 2 || ws_bytes <= 0 || ktiles < 6) return best;
  const double small = double((M + 63) / 64) * double((N + 63) / 64) / double(cus);
  for (int sp = 1; sp <= kMaxSplits; ++sp) {
    const int64_t chunk_tiles = (ktiles + sp - 1) / sp;
    if (sp > 1 && (chunk_tiles < 4 || int64_t(sp) * M * ldw * 4 > ws_bytes)) break;
    if ((sp - 1) * chunk_tiles * 64 >= K || chunk_tiles > kMaxSmallChunk) continue;  // (the last chunk would be empty)
    if (small * sp > (sp == 1 && layout == 0 && K % 64 ? 1.3 : kSmallPerUnit)) break;
    const double t = kSmallTileUs * double(chunk_tiles) * std::max(1.0, small * sp) + (sp > 1 ? 3.5 + double(M) * double(ldw) * (4.0 * sp + 4.0) / 4.4e6 : 0.0);
    if (t < best_t) {
      best_t = t;
      best = SplitChoice{kDeepTile, sp, int(chunk_tiles * 64), kDeepSmall};
    }
  }
  return best;
}

// Kernel variant (-1 generic, else a tile shape) and K chunks for a GEMM (g: M, N, K, n_store).
SplitChoice plan_gemm(const ntp_handle* h, int64_t ws_bytes, const GemmArgs& g, int layout, bool ring_ok, bool split_ok,
                      int64_t ldw, bool deep_ok, bool small_ok = true) {
  SplitChoice sc{choose_variant(h, g, ring_ok, layout), 1, 0, kNotDeep};
  if (split_ok && int64_t(g.M) * g.N >= 128 * 128 * 8) sc = choose_split(h, ws_bytes, g.M, g.n_store, g.K, layout, sc.tile, ldw);
  // (options that ask for a ring tile, a cut, a schedule, a cap on the persistent grid or a K tail through registers mean the ring kernels)
  const bool ring_asked = h->opt[NTP_OPT_GEMM_TILE] || h->opt[NTP_OPT_GEMM_SPLIT] || h->opt[NTP_OPT_GEMM_SCHEDULE] || h->opt[NTP_OPT_GEMM_WORKGROUPS] ||
                          (h->opt[NTP_OPT_GEMM_NO_RING_TAIL] && layout == 1 && g.K % 64 != 0);
  if (deep_ok && sc.tile >= 0 && !ring_asked)
    sc = choose_deep(h, split_ok ? ws_bytes : 0, layout, g.M, g.n_store, g.K, ldw, sc, small_ok);
  // What stays whole on the persistent kernels takes the best tile by their own rates; the order of its sums is the same on every tile.
  if (sc.tile >= 0 && sc.splits == 1 && !sc.deep && !h->opt[NTP_OPT_GEMM_TILE]) sc.tile = choose_tile(kTileRate, g.M, g.n_store, layout, h->compute_units);
  return sc;
}

// Which kernel a persistent launch on an 8-wavefront tile gets: the ping-pong one (tile shapes 0-6, three K tiles or more), whose wavefronts read
// fragments while the others of their SIMDs compute, unless NTP_OPT_GEMM_SCHEDULE = 1 asks for the ring kernel.  Ping-pong against ring over 34 shapes of 17 to 730
// GFLOP, each on its own best tile, with operands from HBM: column-parallel 0.96 of the time on the mean (0.82 to 1.03, above 1 where one round of tiles has rows that do not start on cache
// lines), row-parallel 0.93 (0.81 to 0.99), weight gradients with the column-parallel product before them 0.97 (0.93 to 1.03); with cached operands 0.91, 0.91 and 0.95, nowhere slower.
bool use_pingpong(const ntp_handle* h, int variant, int64_t K) {
  return variant >= 0 && variant <= 6 && K > 128 && h->opt[NTP_OPT_GEMM_SCHEDULE] != 1;
}

// Compute units that a persistent launch uses.
int32_t resident_units(const ntp_handle* h) {
  const int64_t cap = h->opt[NTP_OPT_GEMM_WORKGROUPS];
  return int32_t(cap ? std::min<int64_t>(cap, h->compute_units) : h->compute_units);
}

// Whether a weight gradient on 256 x 256 tiles runs the ping-pong kernel with one workgroup per output tile (which takes one and two K tiles too) instead of the
// persistent one; the ring kernel does not have that tile.  A workgroup's next tile under its stores pays where there is one and a tile is short: with more tiles than
// compute units and K up to 4096 the persistent form takes 0.961 of the time on the mean of sixteen shapes (0.89 to 1.00), accumulating 0.992 (0.97 to 1.03): 5376 x 12288
// over 2048 259 -> 250 us, 8440 x 8072 over 720 150 -> 134.  With fewer tiles, or longer, it takes 1.001 on twenty-eight (0.95 to 1.03), accumulating 1.006 (0.98 to 1.07).
bool one_tile_each(const ntp_handle* h, int layout, int variant, const GemmArgs& g) {
  if (layout != 2 || variant != 0) return false;
  const int64_t tiles = ((g.M + 255ll) / 256) * ((g.n_store + 255ll) / 256);
  return !use_pingpong(h, variant, g.K) || tiles <= g.resident || g.K > 4096;
}

// Whether a product runs on the ping-pong kernel: every cut one on an 8-wavefront tile, whole ones as above.  pp_ok: Prepared::pp_ok.
bool on_pingpong(const ntp_handle* h, int layout, const SplitChoice& sc, const GemmArgs& g, bool pp_ok) {
  if (sc.deep || sc.tile < 0 || sc.tile > 6) return false;
  return sc.splits > 1 || one_tile_each(h, layout, sc.tile, g) || (pp_ok && use_pingpong(h, sc.tile, g.K));
}

// A K tail that a persistent launch of it takes (whole_chunks: see prepare).
bool pingpong_takes(const ntp_handle* h, int layout, int64_t K, bool whole_chunks) {
  return K % 64 == 0 || (whole_chunks && !(layout == 1 && h->opt[NTP_OPT_GEMM_NO_RING_TAIL]));
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

namespace ntp {

int64_t gemm_workspace_wish(const ntp_handle* h, int layout, int64_t M, int64_t N, int64_t n_store, int64_t K, bool deep) {
  if (M < 1 || N < 1 || K < 1 || M > 0x7fffff00 || N > 0x7fffff00 || K > 0x7fffff00) return 0;
  GemmArgs g{};
  g.M = int32_t(M);
  g.N = int32_t(N);
  g.K = int32_t(K);
  g.n_store = int32_t(n_store);
  const int64_t ldw = (n_store + 15) / 16 * 16;
  // (what 128 x 128 tiles would be cut into counts where 64 x 64 tiles take their place uncut: those are for handles with a workspace)
  const SplitChoice sc = plan_gemm(h, INT64_MAX / 2, g, layout, true, true, ldw, deep), wide = plan_gemm(h, INT64_MAX / 2, g, layout, true, true, ldw, deep, false);
  const int splits = std::max(sc.splits, wide.splits);
  return splits > 1 ? int64_t(splits) * M * ldw * 4 : 0;
}

namespace {

// A checked GEMM: kernel arguments and the launcher's choice.
struct Prepared {
  GemmArgs g;
  SplitChoice sc;
  int layout;
  bool ring_ok;
  bool pp_ok;    // pingpong_takes
  bool empty;    // no output element: nothing else is filled in
  bool nothing;  // no output that has a destination
  void* ws_ptr;
  int64_t ldw;
};

int prepare(ntp_handle* h, const GemmDesc& d, Prepared* out) {
  out->empty = out->nothing = true;
  if (!h || d.M < 0 || d.N < 0 || d.K < 0) return NTP_ERR_INVALID_ARG;
  if (d.M == 0 || d.N == 0) return NTP_OK;
  if (h->device < 0) return NTP_ERR_NO_DEVICE;
  if (d.M > 0x7fffff00 || d.N > 0x7fffff00 || d.K > 0x7fffff00) return NTP_ERR_UNSUPPORTED;
  const bool to_segs = d.n_segs > 0;
  if ((!d.C && !to_segs) || (d.K > 0 && (!d.A || !d.B))) return NTP_ERR_INVALID_ARG;
  const bool f32_out = d.epilogue == EPI_F32 || d.epilogue == EPI_F32_ACCUM;
  if (d.epilogue == EPI_GELU && !d.C2) return NTP_ERR_INVALID_ARG;
  if (d.epilogue == EPI_DGELU && !d.AUX) return NTP_ERR_INVALID_ARG;

  // extents along the contiguous axis of each operand, and alignment of every 16-byte access
  const int64_t a_cols = d.a_kc ? d.K : d.M, b_cols = d.b_kc ? d.K : d.N;
  if (d.K > 0) {
    if (d.lda < a_cols || d.ldb < b_cols) return NTP_ERR_INVALID_ARG;
    if (!aligned16(d.A) || !aligned16(d.B) || d.lda % 8 || d.ldb % 8) return NTP_ERR_ALIGNMENT;
  }
  int64_t n_store = d.N;
  if (f32_out) {
    if (d.N % 4) return NTP_ERR_ALIGNMENT;
    if (!to_segs && (!aligned16(d.C) || d.ldc % 4)) return NTP_ERR_ALIGNMENT;
  } else {
    if (to_segs) return NTP_ERR_INVALID_ARG;
    if (d.zero_pad_n) n_store = d.pad_n_64 ? (d.N + 63) / 64 * 64 : (d.N + 7) / 8 * 8;
    if (n_store % 4) return NTP_ERR_ALIGNMENT;
    if (!aligned16(d.C) || d.ldc % 8) return NTP_ERR_ALIGNMENT;
    if (d.epilogue == EPI_GELU && (!aligned16(d.C2) || d.ldc2 % 8 || d.ldc2 < n_store)) return NTP_ERR_ALIGNMENT;
    if (d.epilogue == EPI_DGELU && (!aligned16(d.AUX) || d.ldaux % 8 || d.ldaux < n_store)) return NTP_ERR_ALIGNMENT;
  }
  if (!to_segs && d.ldc < n_store) return NTP_ERR_INVALID_ARG;

  GemmArgs g{};
  g.all_rows = 1;
  if (to_segs) {
    // destinations of the output rows: inside [0, M), aligned, wide enough, not overlapping in memory
    // (a row that no segment lists is not stored)
    if (!d.segs || d.n_segs < 0) return NTP_ERR_INVALID_ARG;
    if (d.n_segs > kMaxRowSegs) return NTP_ERR_UNSUPPORTED;
    for (int32_t i = 0; i < d.n_segs; ++i) {
      const ntp_row_segment_t& r = d.segs[i];
      if (r.row_begin < 0 || r.rows < 0 || r.row_begin + r.rows > d.M) return NTP_ERR_INVALID_ARG;
      if (r.rows == 0) continue;
      if (!r.dst || r.ld < d.N) return NTP_ERR_INVALID_ARG;
      if (!aligned16(r.dst) || r.ld % 4) return NTP_ERR_ALIGNMENT;
      const uintptr_t lo = reinterpret_cast<uintptr_t>(r.dst), hi = lo + uintptr_t(((r.rows - 1) * r.ld + d.N) * 4);
      for (int32_t j = 0; j < g.n_segs; ++j) {
        const uintptr_t lo2 = reinterpret_cast<uintptr_t>(g.seg[j].ptr);
        const uintptr_t hi2 = lo2 + uintptr_t(((int64_t(g.seg[j].end - g.seg[j].begin) - 1) * g.seg[j].ld + d.N) * 4);
        if (lo < hi2 && lo2 < hi) return NTP_ERR_INVALID_ARG;
      }
      g.seg[g.n_segs].begin = int32_t(r.row_begin);
      g.seg[g.n_segs].end = int32_t(r.row_begin + r.rows);
      g.seg[g.n_segs].ptr = r.dst;
      g.seg[g.n_segs].ld = r.ld;
      ++g.n_segs;
    }
    int64_t covered = 0;  // rows [0, covered) have a destination
    for (bool grown = true; grown;) {
      grown = false;
      for (int32_t i = 0; i < g.n_segs; ++i)
        if (g.seg[i].begin <= covered && g.seg[i].end > covered) {
          covered = g.seg[i].end;
          grown = true;
        }
    }
    g.all_rows = covered >= d.M;
  }
  g.A = static_cast<const uint16_t*>(d.A);
  g.B = static_cast<const uint16_t*>(d.B);
  g.C = d.C;
  g.C2 = d.C2;
  g.AUX = static_cast<const uint16_t*>(d.AUX);
  g.lda = d.lda;
  g.ldb = d.ldb;
  g.ldc = d.ldc;
  g.ldc2 = d.ldc2;
  g.ldaux = d.ldaux;
  g.M = int32_t(d.M);
  g.N = int32_t(d.N);
  g.K = int32_t(d.K);
  g.n_store = int32_t(n_store);
  g.gelu_mode = d.gelu_mode;
  // the ring kernel addresses each operand with 32-bit byte offsets from its base
  const int64_t a_rows = d.a_kc ? d.M : d.K, b_rows = d.b_kc ? d.N : d.K;
  const bool ring_ok = ring_combo(d.a_kc, d.b_kc, d.epilogue) && a_rows * d.lda * 2 < (int64_t(1) << 32) &&
                       b_rows * d.ldb * 2 < (int64_t(1) << 32);
  const int layout = d.a_kc ? (d.b_kc ? 0 : 1) : 2;
  // K tail through the ring (row-parallel layout; K is the ragged shard width): B's lines past K lie past its
  // extent and read as zeros, A's columns past K are zeros by the caller's word.  NTP_OPT_GEMM_NO_RING_TAIL
  // switches it off (tests, tuning).
  if (layout == 1 && ring_ok && d.a_k_pad_64 && d.K % 64 != 0 && d.K >= 128 && d.lda >= (d.K + 63) / 64 * 64 &&
      !h->opt[NTP_OPT_GEMM_NO_RING_TAIL])
    g.ring_tail = 1;
  // what the DMA loads are range-checked against (< 4 GiB when ring_ok)
  g.a_extent = uint32_t(std::min<int64_t>(0xFFFFFFFFll, operand_extent_bytes(d.a_kc, d.M, d.K, d.lda, g.ring_tail != 0)));
  g.b_extent = uint32_t(std::min<int64_t>(0xFFFFFFFFll, operand_extent_bytes(d.b_kc, d.N, d.K, d.ldb, false)));
  g.resident = resident_units(h);
  // split-K: any (layout, epilogue) whose operands the ring kernel can address, except B K-contiguous
  // with A K-strided (no ring kernel)
  const bool split_ok = a_rows * d.lda * 2 < (int64_t(1) << 32) && b_rows * d.ldb * 2 < (int64_t(1) << 32) && (d.a_kc || !d.b_kc);
  const int64_t ldw = (n_store + 15) / 16 * 16;
  void* const ws_ptr = d.ws_override ? d.ws_override : h->workspace;
  const int64_t ws_bytes = d.ws_override ? d.ws_override_bytes : (h->workspace ? h->workspace_bytes : 0);
  // deep-pipelined and ping-pong kernels: a K tail of whole chunks; the former's 32-bit byte offsets with room for one that lies past every operand
  const bool whole_chunks = !d.a_kc || d.K % 8 == 0 || (d.a_k_pad_8 && !d.b_kc);
  const bool deep_ok = ring_ok && whole_chunks && a_rows * d.lda * 2 < (int64_t(1) << 31) && b_rows * d.ldb * 2 < (int64_t(1) << 31);
  const bool pp_ok = pingpong_takes(h, layout, d.K, whole_chunks);
  const SplitChoice sc = plan_gemm(h, ws_ptr ? ws_bytes : 0, g, layout, ring_ok, split_ok && whole_chunks, ldw, deep_ok);
  *out = Prepared{g, sc, layout, ring_ok, pp_ok, false, to_segs && g.n_segs == 0, ws_ptr, ldw};
  return NTP_OK;
}

// The arguments of a deep-pipelined launch without a cut K axis.
GemmArgs deep_args(const Prepared& p, const GemmDesc& d) {
  GemmArgs g = p.g;
  g.a_extent = uint32_t(deep_extent_bytes(d.a_kc, d.M, d.K, d.lda));
  g.k_splits = 1;
  g.k_chunk = int32_t((d.K + 63) / 64 * 64);
  return g;
}

// Enqueues a checked GEMM by its choice.
int launch_prepared(ntp_handle* h, const GemmDesc& d, const Prepared& p, void* stream) {
  if (p.nothing) return NTP_OK;
  int st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  static const char* const kEpiName[] = {"bf16", "gelu", "dgelu", "f32", "f32acc"};
  const GemmArgs& g = p.g;
  const SplitChoice sc = p.sc;
  const int layout = p.layout;
  const bool ring_ok = p.ring_ok;
  const int64_t n_store = g.n_store, ldw = p.ldw;
  void* const ws_ptr = p.ws_ptr;
  const int variant = sc.tile;
  if (ntp::timing_on(h)) {
    char name[48], vn[16], sn[8] = "";
    if (sc.deep == kDeepSmall) snprintf(vn, sizeof(vn), "64x64");
    else variant_name(variant, vn, sizeof(vn));
    if (sc.splits > 1) snprintf(sn, sizeof(sn), "k%d", sc.splits);
    const bool pp = sc.splits == 1 && on_pingpong(h, layout, sc, g, p.pp_ok);
    snprintf(name, sizeof(name), "gemm_%c%c_%s_%s%s%s%s", d.a_kc ? 'n' : 't', d.b_kc ? 't' : 'n', kEpiName[d.epilogue], vn,
             sc.deep == kDeep2 ? "d2" : sc.deep ? "d" : "", sn, pp ? "pp" : "");
    ntp::timing_begin(h, stream, name, 2.0 * double(d.M) * double(d.N) * double(d.K), 0.0);
  }
  if (sc.deep && sc.splits == 1) {
    st = launch_deep(deep_args(p, d), d.a_kc, d.b_kc, d.epilogue, sc.deep, s);
  } else if (one_tile_each(h, layout, variant, g) && sc.splits == 1 && ring_ok) {
    GemmArgs gp = g;
    gp.k_splits = 1;
    gp.k_chunk = int32_t((d.K + 63) / 64 * 64);
    st = launch_split_tn(gp, d.epilogue, variant, s);
  } else if (sc.splits > 1) {
    GemmArgs gp = g;  // the partial-sum launch: fp32 to the workspace, no row segments
    gp.ring_tail = 0;
    gp.a_extent = uint32_t(deep_extent_bytes(d.a_kc, d.M, d.K, d.lda));
    gp.C = ws_ptr;
    gp.ldc = ldw;
    gp.n_segs = 0;
    gp.k_splits = sc.splits;
    gp.k_chunk = sc.k_chunk;
    gp.split_stride = int64_t(d.M) * ldw;
    if (sc.deep) st = launch_deep(gp, d.a_kc, d.b_kc, EPI_F32, sc.deep, s);
    else if (d.a_kc && d.b_kc) st = launch_split_nt(gp, variant, s);
    else if (d.a_kc) st = launch_split_nn(gp, variant, s);
    else st = launch_split_tn(gp, EPI_F32, variant, s);
    if (st == NTP_OK) {
      const int64_t threads = int64_t(d.M) * (n_store / 4);
      const dim3 grid(uint32_t((threads + 255) / 256)), block(256);
      const float* ws = static_cast<const float*>(ws_ptr);
      st = dispatch_epilogue(d.epilogue, [&](auto e) {
        hipLaunchKernelGGL((splitk_reduce_kernel<decltype(e)::value>), grid, block, 0, s, g, ws, gp.split_stride, ldw, sc.splits);
        return hipGetLastError() == hipSuccess ? NTP_OK : NTP_ERR_LAUNCH;
      });
    }
  } else if (p.pp_ok && use_pingpong(h, variant, d.K)) {
    GemmArgs gp = g;
    gp.a_extent = uint32_t(std::min<int64_t>(0xFFFFFFFFll, deep_extent_bytes(d.a_kc, d.M, d.K, d.lda)));
    if (d.a_kc && d.b_kc) st = launch_pp_nt(gp, d.epilogue, variant, s);
    else if (d.a_kc) st = launch_pp_nn(gp, d.epilogue, variant, s);
    else st = launch_pp_tn(gp, d.epilogue, variant, s);
  } else if (variant >= 0) {
    if (d.a_kc && d.b_kc) st = launch_ring_nt(g, d.epilogue, variant, s);
    else if (d.a_kc) st = launch_ring_nn(g, d.epilogue, variant, s);
    else st = launch_ring_tn(g, d.epilogue, variant, s);
  } else if (d.a_kc && d.b_kc) st = launch_generic<true, true>(g, d.epilogue, s);
  else if (d.a_kc && !d.b_kc) st = launch_generic<true, false>(g, d.epilogue, s);
  else if (!d.a_kc && !d.b_kc) st = launch_generic<false, false>(g, d.epilogue, s);
  else st = launch_generic<false, true>(g, d.epilogue, s);
  ntp::timing_end(h, stream);
  return st;
}

}  // namespace

int gemm_launch(ntp_handle* h, const GemmDesc& d, void* stream) {
  Prepared p;
  const int st = prepare(h, d, &p);
  return st != NTP_OK ? st : launch_prepared(h, d, p, stream);
}

namespace {

struct Span {
  uintptr_t lo, hi;
};

// Whether what `a` writes touches anything that `b` reads or writes.
bool writes_into(const GemmDesc& a, const GemmDesc& b) {
  auto span = [](const void* p, int64_t rows, int64_t ld, int64_t cols, int64_t esz) {
    const uintptr_t lo = reinterpret_cast<uintptr_t>(p);
    return Span{lo, p && rows > 0 ? lo + uintptr_t(((rows - 1) * ld + cols) * esz) : lo};
  };
  auto outputs = [&](const GemmDesc& d, auto&& f) {
    const bool f32 = d.epilogue == EPI_F32 || d.epilogue == EPI_F32_ACCUM;
    if (d.n_segs > 0) {
      for (int32_t i = 0; i < d.n_segs; ++i) f(span(d.segs[i].dst, d.segs[i].rows, d.segs[i].ld, d.N, 4));
    } else {
      f(span(d.C, d.M, d.ldc, d.ldc, f32 ? 4 : 2));
    }
  };
  bool hit = false;
  outputs(a, [&](Span x) {
    auto test = [&](Span y) { hit = hit || (x.lo < y.hi && y.lo < x.hi); };
    test(span(b.A, b.a_kc ? b.M : b.K, b.lda, b.lda, 2));
    test(span(b.B, b.b_kc ? b.N : b.K, b.ldb, b.ldb, 2));
    outputs(b, test);
  });
  return hit;
}

}  // namespace

// GEMMs that do not need each other's results.  One launch, without cutting a K axis, where all of them would run on the deep-pipelined
// kernel anyway and the estimate says so; else one after the other by their own choices.  Estimate: a launch costs 6 us beside its K tiles
// (launch, first loads, stores); the group's K tiles take as long as its longest problem, or as all its tiles dealt out over the device.
// The numbers must not depend on where the outputs go, so the decision looks at shapes and workspace only: products without a destination
// here count like the others, and where one product writes what another reads or writes (a caller may pass such buffers), the products run
// one after the other in the form that they have in the shared launch.
int gemm_launch_group(ntp_handle* h, const GemmDesc* d, int n, void* stream) {
  constexpr int kMax = 3;
  if (n > kMax) return NTP_ERR_INVALID_ARG;
  Prepared p[kMax];
  int status[kMax] = {NTP_OK, NTP_OK, NTP_OK};
  bool group = n >= 2, apart_only = false;
  double apart = 0.0, longest = 0.0, longest_small = 0.0, work = 0.0, tiles_small = 0.0, work_small = 0.0, flops = 0.0;
  for (int i = 0; i < n; ++i) {
    status[i] = prepare(h, d[i], &p[i]);
    group = group && status[i] == NTP_OK && !p[i].empty && (p[i].sc.deep == kDeep5 || p[i].sc.deep == kDeepSmall) &&
            (p[i].layout == 2 ? d[i].epilogue == EPI_F32 || d[i].epilogue == EPI_F32_ACCUM : d[i].epilogue == EPI_BF16);
    if (!group) continue;
    const GemmArgs& g = p[i].g;
    const double tiles = double((g.M + 127) / 128) * double((g.n_store + 127) / 128), kt = double((g.K + 63) / 64), sp = p[i].sc.splits;
    const double small = double((g.M + 63) / 64) * double((g.n_store + 63) / 64);
    apart += 6.0 + (p[i].sc.deep == kDeep5 ? 0.47 : kSmallTileUs * std::max(1.0, small * sp / h->compute_units)) * std::ceil(kt / sp) + (sp > 1 ? 3.5 + double(g.M) * double(p[i].ldw) * (4.0 * sp + 4.0) / 4.4e6 : 0.0);
    longest = std::max(longest, kt);
    work += tiles * kt;
    tiles_small += small;
    longest_small = std::max(longest_small, kt + (tiles_small > kSmallPerUnit * h->compute_units ? work_small / h->compute_units : 0.0));
    work_small += small * kt * (p[i].layout == 0 && g.K % 64 ? 1.5 : 1.0);
  }
  // 64 x 64 tiles on the terms of choose_deep, where a problem has a long K axis: its K tiles, 0.47 us each with 128 x 128, are then most of
  // the launch's time (2048 x 192 over K = 1024 with 192 x 1024 over 2048 21.5 -> 14.7 us, 2048 x 1024 over 576 with 576 x 1024 over 2048 20.4 -> 14).
  // A problem that finds the device full (two workgroups a unit) starts behind those before it, and K-contiguous operands whose rows do not start
  // on cache lines cost half as much again: without these two terms 4856 x 768 over K = 952 with 768 x 952 over 4856 took 50 us instead of 37,
  // 4667 x 512 over 1640 with 512 x 1640 over 4667 52 instead of 38, 3792 x 768 over 568 with 768 x 568 over 3792 34 instead of 28.  (Over 246
  // groups: 0.78 of the time without this form on the mean, three more than 2 % slower: 3460 x 776 over K = 512 with 512 x 776 over 3460 by 22 %,
  // 4685 x 456 over 1024 with 1024 x 456 over 4685 and 592 x 384 over 5080 with 384 x 5080 over 592 by 5-7 %.)
  const double shared = 0.47 * std::max(longest, 1.15 * work / h->compute_units), shared_small = kSmallTileUs * std::max(longest_small, 1.15 * work_small / h->compute_units);
  const bool by_small = h && h->workspace && longest >= kGroupSmallFrom && shared_small < shared;
  group = group && 6.0 + (by_small ? shared_small : shared) < apart;
  if (group) {
    for (int i = 0; i < n; ++i) {
      p[i].sc.splits = 1;
      p[i].sc.deep = by_small ? kDeepSmall : kDeep5;
      for (int j = 0; j < i; ++j) apart_only = apart_only || writes_into(d[i], d[j]) || writes_into(d[j], d[i]);
    }
  }
  if (!group || apart_only) {
    for (int i = 0; i < n; ++i) {
      const int st = status[i] != NTP_OK ? status[i] : launch_prepared(h, d[i], p[i], stream);
      if (st != NTP_OK) return st;
    }
    return NTP_OK;
  }
  GemmArgs g[kMax];
  int layout[kMax], epi[kMax], m = 0;
  for (int i = 0; i < n; ++i) {
    if (p[i].nothing) continue;
    g[m] = deep_args(p[i], d[i]);
    layout[m] = p[i].layout;
    epi[m++] = d[i].epilogue;
    flops += 2.0 * double(d[i].M) * double(d[i].N) * double(d[i].K);
  }
  if (m == 0) return NTP_OK;
  if (ntp::timing_on(h)) ntp::timing_begin(h, stream, by_small ? "gemm_group_64x64d" : "gemm_group_128x128w8d", flops, 0.0);
  const int st = launch_deep_group(g, layout, epi, m, by_small ? kDeepSmall : kDeep5, static_cast<hipStream_t>(stream));
  ntp::timing_end(h, stream);
  return st;
}

}  // namespace ntp

extern "C" int ntp_gemm_choice(const ntp_handle_t* h, int32_t layout, int64_t M, int64_t N, int64_t K, ntp_gemm_choice_t* out) {
  if (!h || !out || layout < 0 || layout > 2 || M < 1 || N < 1 || K < 0 || M > 0x7fffff00 || N > 0x7fffff00 || K > 0x7fffff00)
    return NTP_ERR_INVALID_ARG;
  GemmArgs g{};
  g.M = int32_t(M);
  g.N = int32_t(N);
  g.K = int32_t(K);
  g.n_store = int32_t((N + 7) / 8 * 8);
  g.resident = resident_units(h);
  const SplitChoice sc = plan_gemm(h, h->workspace ? h->workspace_bytes : 0, g, layout, true, true, (g.n_store + 15) / 16 * 16, true);
  *out = ntp_gemm_choice_t{};
  out->k_splits = sc.splits;
  if (sc.tile < 0) {
    out->tile_m = out->tile_n = 128;
    out->wavefronts = 4;
    out->ring = 0;
  } else {
    const TileShape ts = sc.deep == kDeepSmall ? TileShape{64, 64, 4} : kTileShapes[sc.tile];
    out->tile_m = ts.bm;
    out->tile_n = ts.bn;
    out->wavefronts = ts.waves;
    out->ring = 1;
  }
  out->persistent = sc.tile >= 0 && !sc.deep && sc.splits == 1 && !one_tile_each(h, layout, sc.tile, g) ? 1 : 0;
  out->pingpong = on_pingpong(h, layout, sc, g, pingpong_takes(h, layout, K, true)) ? 1 : 0;
  return NTP_OK;
}
