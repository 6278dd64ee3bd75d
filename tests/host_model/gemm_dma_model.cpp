// Host model of the GEMM kernels' operand DMA addressing (no GPU).
//
// It includes the kernels' own index arithmetic (csrc/ntp_gemm_addr.h) and enumerates, for every tile
// variant, operand layout and a list of ragged shapes, every (offset, K tile) pair that the
// ring kernel's schedule can issue, and checks each 16-byte load against the operand as the caller's contract
// defines it:
//   - a load lies wholly inside the operand, or
//   - (K tail through the ring, B operand only) wholly outside the range-checked extent, where the hardware
//     returns zeros, and then only for K lines >= K.
// The deep-pipelined kernel's loads (ntp_gemm_deep.h) are enumerated the same way for its two tile sizes, 1 to 16 K chunks and
// allocations that end with the operand: each lies wholly inside the operand and inside its view and starts at k < K, or wholly outside the
// view, and then starts at k >= K.
// The ping-pong kernel's (ntp_gemm_pp.h) are enumerated for its seven tile shapes, whole with and without a next output tile and in 1 to 8 K chunks (chunks of one
// and two K tiles and ragged last ones among them), operands of 2 to 4 GiB included: each K tile's loads as above, what is asked for past the last K tile lies wholly
// outside the view or is a K tile of the next output tile, and no scalar offset lies past the view.
//
// It also evaluates the schedule of a K loop padded to a multiple of five K tiles WITHOUT the clamp on the
// tile index (a variant that was tried and faulted) and reports how far past the operand it reads.
//
// Prints "OK <cases> <loads>" and exits 0, or prints the first violation and exits 1.
// With the argument "padded" it prints "OVERRUN <bytes>" for the unclamped padded loop instead.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <utility>
#include <vector>

#include "ntp_gemm_addr.h"

using namespace ntp_gemm;

struct Tile {
  int bm, bn, nw;
};
static const Tile kTiles[] = {{256, 256, 8}, {256, 224, 8}, {224, 256, 8}, {256, 192, 8}, {192, 256, 8},
                              {256, 128, 8}, {128, 256, 8}, {128, 128, 4}, {128, 128, 8}};

// What the caller's contract says an operand's memory holds, in bytes from its first element, derived from
// the element ranges rather than from the library's formula: the largest byte offset + 1 of any element that
// may legitimately be read.  K-contiguous [rows x K] with ld: elements (r, k), k < k_reach.  K-strided
// [K x rows] with ld: elements (k, c), c < rows rounded up to 8 (rows of such operands are padded to 8).
static int64_t contract_bytes(bool kc, int64_t rows, int64_t K, int64_t ld, int64_t k_reach) {
  int64_t last = -1;
  if (kc) {
    if (rows > 0 && k_reach > 0) last = (rows - 1) * ld + (k_reach - 1);
  } else {
    const int64_t c = (rows + 7) / 8 * 8;
    if (K > 0 && c > 0) last = (K - 1) * ld + (c - 1);
  }
  return (last + 1) * 2;
}

template <bool KC, int R>
static void offsets(int64_t ld, int row0, int lim, std::vector<uint32_t>* out, std::vector<int>* lines) {
  out->clear();
  lines->clear();
  for (int pos = 0; pos < R * 8; ++pos) {  // every chunk position of a slot: all wavefronts, instructions, lanes
    int line, chunk;
    slot_src<KC, R>(pos, line, chunk);
    out->push_back(dma_offset<KC>(ld, row0, lim, line, chunk));
    lines->push_back(line);
  }
}

static void offsets_dyn(bool kc, int R, int64_t ld, int row0, int lim, std::vector<uint32_t>* out, std::vector<int>* lines) {
  if (kc) {
    switch (R) {
      case 64: return offsets<true, 64>(ld, row0, lim, out, lines);
      case 128: return offsets<true, 128>(ld, row0, lim, out, lines);
      case 192: return offsets<true, 192>(ld, row0, lim, out, lines);
      case 256: return offsets<true, 256>(ld, row0, lim, out, lines);
    }
  } else {
    switch (R) {
      case 128: return offsets<false, 128>(ld, row0, lim, out, lines);
      case 256: return offsets<false, 256>(ld, row0, lim, out, lines);
    }
  }
  fprintf(stderr, "no slot of %d rows\n", R);
  exit(2);
}

struct Shape {
  int M, N, K;
  int pad_a, pad_b;  // extra elements on the leading dimensions (multiples of 8)
};

static int64_t g_loads = 0, g_cases = 0;
static int64_t g_overrun = 0;

// One operand of one output tile.  ring_tail: the K tail goes through the ring; zero_tail_ok: loads at K lines >= K may be out of range.
static bool check_operand(const char* what, bool kc, int b, int64_t ld, int row0, int lim, int K, bool ring_tail, bool zero_tail_ok, int64_t extent,
                          int64_t contract, bool padded_loop) {
  std::vector<uint32_t> off;
  std::vector<int> lines;
  offsets_dyn(kc, slot_rows(kc, b), ld, row0, lim, &off, &lines);
  const int64_t kstep = (kc ? int64_t(DK) : int64_t(DK) * ld) * 2;  // bytes per K tile
  const int nk = ring_k_tiles(K, ring_tail);
  if (nk == 0) return true;
  // K tiles the schedule issues: 0 .. nk-1 (it clamps t+1 and t+2 to nk-1).  The padded loop ran on to the
  // next multiple of five tiles, plus the two tiles of look-ahead, unclamped.
  const int last_kt = padded_loop ? (nk + 4) / 5 * 5 + 1 : nk - 1;
  for (int kt = 0; kt <= last_kt; ++kt) {
    for (size_t i = 0; i < off.size(); ++i) {
      const int64_t o = int64_t(off[i]) + int64_t(kt) * kstep;  // from the operand's first element
      ++g_loads;
      if (padded_loop) {
        if (o + 16 > contract && o + 16 - contract > g_overrun) g_overrun = o + 16 - contract;
        continue;
      }
      if (o > 0xFFFFFFFFll) {
        printf("FAIL %s: 32-bit offset overflow\n", what);
        return false;
      }
      if (o + 16 <= contract && o + 16 <= extent) continue;  // inside the operand and inside the checked range
      // Otherwise the hardware must zero the whole load (it checks each lane's 16 bytes against the extent),
      // and that is only legitimate for K lines at or past K of the tail tile.
      const int64_t kline = int64_t(kt) * DK + (kc ? 0 : lines[i]);
      if (zero_tail_ok && o >= extent && !kc && kline >= K) continue;
      printf("FAIL %s: kc=%d tile side %d ld=%lld row0=%d lim=%d K=%d kt=%d off=%u -> byte %lld, contract %lld, extent %lld\n", what, int(kc), b,
             (long long)ld, row0, lim, K, kt, off[i], (long long)o, (long long)contract, (long long)extent);
      return false;
    }
  }
  return true;
}

static bool run_gemm(bool akc, bool bkc, const Tile& t, const Shape& s, bool a_pad64, bool padded_loop) {
  const int64_t a_cols = akc ? s.K : s.M, b_cols = bkc ? s.K : s.N;
  int64_t lda = (a_cols + 7) / 8 * 8 + s.pad_a, ldb = (b_cols + 7) / 8 * 8 + s.pad_b;
  const bool layout_nn = akc && !bkc;
  // the launcher's rule for sending the K tail through the ring (row-parallel layout)
  bool ring_tail = layout_nn && a_pad64 && s.K % 64 != 0 && s.K >= 128;
  if (ring_tail) lda = (s.K + 63) / 64 * 64 + s.pad_a;
  const int64_t a_ext = operand_extent_bytes(akc, s.M, s.K, lda, ring_tail);
  const int64_t b_ext = operand_extent_bytes(bkc, s.N, s.K, ldb, false);
  const int64_t a_con = contract_bytes(akc, s.M, s.K, lda, ring_tail ? (s.K + 63) / 64 * 64 : s.K);
  const int64_t b_con = contract_bytes(bkc, s.N, s.K, ldb, s.K);
  if (a_ext > a_con || b_ext > b_con) {
    printf("FAIL extent beyond the contract: a %lld > %lld or b %lld > %lld\n", (long long)a_ext, (long long)a_con,
           (long long)b_ext, (long long)b_con);
    return false;
  }
  const int tiles_m = (s.M + t.bm - 1) / t.bm, tiles_n = (s.N + t.bn - 1) / t.bn;
  // An operand's addresses depend on its own tile index only (A on tile_m, B on tile_n), and only the last
  // tile of a side clamps differently from the others: first, middle and last tile of each side cover all cases.
  for (int side = 0; side < 2; ++side) {
    const int n_tiles = side == 0 ? tiles_m : tiles_n;
    int picks[3] = {0, n_tiles / 2, n_tiles - 1};
    for (int pi = 0; pi < 3; ++pi) {
      if (pi > 0 && picks[pi] == picks[pi - 1]) continue;
      ++g_cases;
      if (side == 0 ? !check_operand("A", akc, t.bm, lda, picks[pi] * t.bm, s.M, s.K, ring_tail, false, a_ext, a_con, padded_loop)
                    : !check_operand("B", bkc, t.bn, ldb, picks[pi] * t.bn, s.N, s.K, ring_tail, ring_tail, b_ext, b_con, padded_loop))
        return false;
    }
  }
  for (int v = 0; v < tiles_m * tiles_n; ++v) {
    const TilePos p = place_tile(v, tiles_m, tiles_n);
    if (p.tile_m < 0 || p.tile_m >= tiles_m || p.tile_n < 0 || p.tile_n >= tiles_n) {
      printf("FAIL tile walk: block %d -> (%d, %d) of %d x %d\n", v, p.tile_m, p.tile_n, tiles_m, tiles_n);
      return false;
    }
  }
  // the tile walk must visit every tile exactly once
  std::vector<int> seen(size_t(tiles_m) * tiles_n, 0);
  for (int v = 0; v < tiles_m * tiles_n; ++v) {
    const TilePos p = place_tile(v, tiles_m, tiles_n);
    ++seen[size_t(p.tile_m) * tiles_n + p.tile_n];
  }
  for (int x : seen)
    if (x != 1) {
      printf("FAIL tile walk: a tile is visited %d times (%d x %d tiles)\n", x, tiles_m, tiles_n);
      return false;
    }
  return true;
}

// One operand of one output tile of the deep-pipelined kernel over one K chunk [first, first + Kc).
template <bool KC, int R>
static bool check_deep(const char* what, int64_t ld, int row0, int lim, int K_total, int64_t first, int Kc, int64_t extent, int64_t contract) {
  const int nk = (Kc + DK - 1) / DK;
  const int64_t shift = deep_view_shift(KC, first, ld), view = extent - shift, kstep = int64_t(KC ? DK : DK * ld) * 2;
  if (shift != (KC ? first : first * ld) * 2 || view <= 0 || extent >= (int64_t(1) << 31)) {
    printf("FAIL deep %s: view\n", what);
    return false;
  }
  for (int pos = 0; pos < R * 8; ++pos) {  // every chunk position of a slot: all wavefronts, instructions, lanes
    int line, chunk;
    slot_src<KC, R>(pos, line, chunk);
    const uint32_t off = dma_offset<KC>(ld, row0, lim, line, chunk);
    const bool cut = deep_cut<KC>(nk, chunk, Kc);
    for (int kt = 0; kt < nk; ++kt) {  // (the schedule clamps what it asks for past the end to the last K tile)
      const int64_t voff = kt == nk - 1 && cut ? kNowhere : off, soff = int64_t(kt) * kstep, o = voff + soff;
      const int64_t k = first + int64_t(kt) * DK + (KC ? chunk * 8 : line);  // where the 16 bytes start on the K axis
      ++g_loads;
      bool ok = soff <= 0xFFFFFFFFll && o <= 0xFFFFFFFFll;  // 32-bit sums
      if (o + 16 <= view) ok = ok && shift + o + 16 <= contract && k < K_total;
      else ok = ok && o >= view && k >= K_total;  // the range check returns zeros
      if (ok) continue;
      printf("FAIL deep %s: kc=%d R=%d ld=%lld row0=%d lim=%d K=%d first=%lld Kc=%d kt=%d k=%lld -> byte %lld of a view of %lld, contract %lld\n", what, int(KC), R,
             (long long)ld, row0, lim, K_total, (long long)first, Kc, kt, (long long)k, (long long)o, (long long)view, (long long)contract);
      return false;
    }
  }
  return true;
}

static bool run_deep(bool akc, bool bkc, int bm, int bn, const Shape& s, int splits) {
  const bool nn = akc && !bkc;
  if (akc && s.K % 8 && !nn) return true;  // not this kernel's: only a row-parallel GEMM's A has its pad columns zeroed
  const int a_cols = akc ? s.K : s.M, b_cols = bkc ? s.K : s.N;
  const int64_t lda = (a_cols + 7) / 8 * 8 + s.pad_a, ldb = (b_cols + 7) / 8 * 8 + s.pad_b;
  const int64_t a_ext = deep_extent_bytes(akc, s.M, s.K, lda), b_ext = operand_extent_bytes(bkc, s.N, s.K, ldb, false);
  const int64_t a_con = contract_bytes(akc, s.M, s.K, lda, nn ? (s.K + 7) / 8 * 8 : s.K), b_con = contract_bytes(bkc, s.N, s.K, ldb, s.K);
  if (a_ext > a_con || b_ext > b_con) {
    printf("FAIL deep: extent beyond the contract\n");
    return false;
  }
  const int chunk = ((s.K + 63) / 64 + splits - 1) / splits * 64;
  if (int64_t(splits - 1) * chunk >= s.K) return true;  // the launcher never makes an empty chunk
  for (int sp = 0; sp < splits; ++sp) {
    const int64_t first = int64_t(sp) * chunk;
    const int Kc = imin(chunk, s.K - int(first));
    for (int side = 0; side < 2; ++side) {
      const int b = side ? bn : bm, lim = side ? s.N : s.M, tiles = (lim + b - 1) / b;
      const bool kc = side ? bkc : akc;
      for (int tile : {0, tiles / 2, tiles - 1}) {
        ++g_cases;
        const int64_t ld = side ? ldb : lda, ext = side ? b_ext : a_ext, con = side ? b_con : a_con;
        const char* const what = side ? "B" : "A";
        const bool ok = b == 64 ? (kc ? check_deep<true, 64>(what, ld, tile * b, lim, s.K, first, Kc, ext, con)
                                      : check_deep<false, 64>(what, ld, tile * b, lim, s.K, first, Kc, ext, con))
                        : b == 128 ? (kc ? check_deep<true, 128>(what, ld, tile * b, lim, s.K, first, Kc, ext, con)
                                       : check_deep<false, 128>(what, ld, tile * b, lim, s.K, first, Kc, ext, con))
                                 : (kc ? check_deep<true, 256>(what, ld, tile * b, lim, s.K, first, Kc, ext, con)
                                       : check_deep<false, 256>(what, ld, tile * b, lim, s.K, first, Kc, ext, con));
        if (!ok) return false;
      }
    }
  }
  return true;
}

// One operand of one output tile of the ping-pong kernel over one K chunk [first, first + Kc).  next_row0: first row of the workgroup's next output tile, or -1.
template <bool KC, int R>
static bool check_pp(const char* what, int64_t ld, int row0, int next_row0, int lim, int K_total, int64_t first, int Kc, int64_t extent, int64_t contract) {
  const int nk = (Kc + DK - 1) / DK;
  const int64_t shift = deep_view_shift(KC, first, ld), view = extent - shift;
  const uint32_t step = uint32_t(KC ? DK : DK * ld) * 2;
  const bool cut = nk * DK > Kc, more = next_row0 >= 0;
  if (shift != (KC ? first : first * ld) * 2 || view <= 0 || extent > 0xFFFFFFF0ll || int64_t(step) != int64_t(KC ? DK : DK * ld) * 2) {
    printf("FAIL ping-pong %s: view\n", what);
    return false;
  }
  for (int pos = 0; pos < R * 8; ++pos) {  // every chunk position of a slot: all wavefronts, instructions, lanes
    int line, chunk;
    slot_src<KC, R>(pos, line, chunk);
    uint32_t voff = dma_offset<KC>(ld, row0, lim, line, chunk);
    for (int j = 0; j < std::max(nk, 2) + 2; ++j) {  // the first two K tiles before the loop, and two past the last
      if (j == nk - 1 && cut) voff = pp_cut_offset<KC>(voff, step, nk, line, chunk, Kc);
      if (j >= nk) voff = more ? dma_offset<KC>(ld, next_row0, lim, line, chunk) : kPastAll;
      const int64_t soff = pp_scalar_offset(j, nk, cut, more, step), o = voff + soff;
      const bool nothing = j >= nk && !more;
      const int64_t k = first + int64_t(j < nk ? j : j - nk) * DK + (KC ? chunk * 8 : line);  // where the 16 bytes start on the K axis
      ++g_loads;
      bool ok = soff < view && o <= 0xFFFFFFFFll;  // the range check subtracts the one from the other; 32-bit sums
      if (o + 16 <= view) ok = ok && !nothing && shift + o + 16 <= contract && k < K_total;
      else ok = ok && o >= view && (nothing || k >= K_total);  // the range check returns zeros
      if (!nothing && k < K_total) {  // and they are the bytes that the slot is to hold
        const int64_t row = imin((j < nk ? row0 : next_row0) + (KC ? line : chunk * 8), KC ? lim - 1 : (lim - 1) / 8 * 8);
        ok = ok && shift + o == (KC ? row * ld + k : k * ld + row) * 2;
      }
      if (ok) continue;
      printf("FAIL ping-pong %s: kc=%d R=%d ld=%lld row0=%d next=%d lim=%d K=%d first=%lld Kc=%d j=%d k=%lld -> %u + %lld of a view of %lld, contract %lld\n", what, int(KC), R,
             (long long)ld, row0, next_row0, lim, K_total, (long long)first, Kc, j, (long long)k, voff, (long long)soff, (long long)view, (long long)contract);
      return false;
    }
  }
  return true;
}

static bool check_pp_dyn(bool kc, int R, const char* what, int64_t ld, int row0, int next, int lim, int K, int64_t first, int Kc, int64_t extent, int64_t contract) {
  if (kc) return R == 128   ? check_pp<true, 128>(what, ld, row0, next, lim, K, first, Kc, extent, contract)
                 : R == 192 ? check_pp<true, 192>(what, ld, row0, next, lim, K, first, Kc, extent, contract)
                            : check_pp<true, 256>(what, ld, row0, next, lim, K, first, Kc, extent, contract);
  return R == 128 ? check_pp<false, 128>(what, ld, row0, next, lim, K, first, Kc, extent, contract)
                  : check_pp<false, 256>(what, ld, row0, next, lim, K, first, Kc, extent, contract);
}

static bool run_pp(bool akc, bool bkc, const Tile& t, const Shape& s, int splits) {
  const bool nn = akc && !bkc;
  if (akc && s.K % 8 && !nn) return true;  // not this kernel's: only a row-parallel GEMM's A has its pad columns zeroed
  const int a_cols = akc ? s.K : s.M, b_cols = bkc ? s.K : s.N;
  const int64_t lda = (a_cols + 7) / 8 * 8 + int64_t(s.pad_a), ldb = (b_cols + 7) / 8 * 8 + int64_t(s.pad_b);
  if (int64_t(akc ? s.M : s.K) * lda * 2 >= int64_t(1) << 32 || int64_t(bkc ? s.N : s.K) * ldb * 2 >= int64_t(1) << 32) return true;  // the generic kernel's
  const int64_t a_ext = deep_extent_bytes(akc, s.M, s.K, lda), b_ext = operand_extent_bytes(bkc, s.N, s.K, ldb, false);
  const int64_t a_con = contract_bytes(akc, s.M, s.K, lda, nn ? (s.K + 7) / 8 * 8 : s.K), b_con = contract_bytes(bkc, s.N, s.K, ldb, s.K);
  if (a_ext > a_con || b_ext > b_con) {
    printf("FAIL ping-pong: extent beyond the contract\n");
    return false;
  }
  const int chunk = ((s.K + 63) / 64 + splits - 1) / splits * 64;
  if (int64_t(splits - 1) * chunk >= s.K) return true;  // the launcher never makes an empty chunk
  for (int sp = 0; sp < splits; ++sp) {
    const int64_t first = int64_t(sp) * chunk;
    const int Kc = imin(chunk, s.K - int(first));
    for (int side = 0; side < 2; ++side) {
      const int b = side ? t.bn : t.bm, lim = side ? s.N : s.M, tiles = (lim + b - 1) / b;
      const bool kc = side ? bkc : akc;
      const int picks[3] = {0, tiles / 2, tiles - 1};
      for (int pi = 0; pi < 3; ++pi)
        for (int next : {-1, 0, tiles - 1}) {
          if (pi > 0 && picks[pi] == picks[pi - 1]) continue;
          if (next >= 0 && (splits > 1 || s.K <= 128)) continue;  // only the persistent form has a next output tile, and it has three K tiles
          ++g_cases;
          if (!check_pp_dyn(kc, slot_rows(kc, b), side ? "B" : "A", side ? ldb : lda, picks[pi] * b, next < 0 ? -1 : next * b, lim, s.K, first, Kc, side ? b_ext : a_ext, side ? b_con : a_con))
            return false;
        }
    }
  }
  return true;
}

int main(int argc, char** argv) {
  const bool padded = argc > 1 && !strcmp(argv[1], "padded");
  const Shape shapes[] = {
      {777, 1001, 1096, 0, 0},  {1, 8, 128, 0, 0},        {3, 17, 200, 8, 16},     {65, 64, 64, 0, 0},     {520, 1500, 1032, 0, 0},
      {2048, 7022, 12288, 0, 0}, {2048, 12288, 7022, 0, 40}, {7022, 12288, 2048, 0, 0}, {8192, 750, 16384, 0, 0}, {8192, 16384, 750, 18 * 8, 0},
      {750, 16384, 8192, 0, 0},  {4096, 640, 8192, 0, 0},  {4096, 8192, 384, 0, 0},  {896, 8192, 4096, 0, 0}, {1100, 1171, 1096, 0, 0},
      {257, 255, 321, 0, 0},     {256, 256, 5376, 0, 0},   {300, 513, 5376 + 41, 0, 0},
  };
  const bool layouts[3][2] = {{true, true}, {true, false}, {false, false}};
  for (const auto& lay : layouts)
    for (const Tile& t : kTiles)
      for (const Shape& s : shapes)
        for (int pad64 = 0; pad64 < 2; ++pad64) {
          if (pad64 && !(lay[0] && !lay[1])) continue;
          if (!run_gemm(lay[0], lay[1], t, s, pad64 != 0, padded)) return 1;
        }
  const Shape deep_shapes[] = {{512, 586, 1024, 0, 0}, {257, 129, 264, 0, 0}, {1, 1, 8, 0, 0}, {130, 383, 1288, 8, 16}, {300, 131, 4096, 0, 0}, {520, 1032, 1500, 0, 0},
                               {777, 1096, 1001, 0, 40}, {1001, 1096, 777, 0, 0}, {752, 160, 9544, 0, 0}, {129, 513, 2051, 64, 8}, {128, 256, 63, 0, 0}, {64, 8, 65, 0, 0}};
  if (!padded)
    for (const auto& lay : layouts)
      for (const auto& t : {std::pair<int, int>{64, 64}, {128, 128}, {128, 256}})
        for (const Shape& s : deep_shapes)
          for (int splits = 1; splits <= 16; ++splits)
            if (!run_deep(lay[0], lay[1], t.first, t.second, s, splits)) return 1;
  // ping-pong: chunks of one and two K tiles, last chunks of one K tile and of less; then operands of 2 to 4 GiB, in whole and ragged K tiles, and 4 GiB short of 16 bytes
  const Shape pp_shapes[] = {{700, 704, 488, 0, 0}, {700, 704, 987, 0, 0}, {257, 449, 40, 0, 0},    {300, 513, 64, 0, 0},   {129, 225, 104, 0, 8},  {520, 1500, 3624, 0, 0}, {777, 1001, 1096, 0, 0},
                             {488, 704, 705, 0, 0}, {65, 190, 131, 0, 0},  {1300, 1400, 321, 8, 0}, {1, 8, 456, 0, 0},      {750, 2048, 1032, 0, 16}, {2400, 130, 1001, 500000, 0},
                             {2400, 130, 1024, 500000, 0}, {130, 600, 1000, 3000000, 2000000}, {1000, 520, 1320, 1000000, 1600000}, {1001, 513, 2047, 0, 1047056 - 8}, {8191, 64, 2056, 262144 - 2056, 0}};
  if (!padded)
    for (const auto& lay : layouts)
      for (int i = 0; i < 7; ++i)
        for (const Shape& s : pp_shapes)
          for (int splits = 1; splits <= 8; ++splits)
            if (!run_pp(lay[0], lay[1], kTiles[i], s, splits)) return 1;
  if (padded) printf("OVERRUN %lld\n", (long long)g_overrun);
  else printf("OK %lld %lld\n", (long long)g_cases, (long long)g_loads);
  return 0;
}
