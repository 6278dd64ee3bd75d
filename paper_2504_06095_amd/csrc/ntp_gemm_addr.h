// Index arithmetic of the GEMM kernels' operand DMA, kept apart from the kernels so that a host
// program can include it too and enumerate every address that they can form (the kernels' loads are
// range-checked by the hardware against the operand's extent; the host model checks the same
// arithmetic against the same extent without a GPU).
#ifndef NTP_GEMM_ADDR_H_
#define NTP_GEMM_ADDR_H_

#include <stdint.h>

#if defined(__HIPCC__)
#define NTP_HD __host__ __device__ __forceinline__
#else
#define NTP_HD inline
#endif

namespace ntp_gemm {

constexpr int DK = 64;  // K extent of a tile

NTP_HD int imin(int a, int b) { return a < b ? a : b; }

// chunk permutation of a K-strided slot line of `rows` rows (a line of 64 rows is half of the 256 bytes that the LDS banks span, so
// that two lines side by side take the place of the lowest bit)
NTP_HD constexpr int kline_swz(int k, int rows) {
  return rows == 64 ? (((k >> 1) & 1) | (((k >> 3) & 1) << 1)) << 1 : ((k & 3) | (((k >> 3) & 1) << 2)) << 1;
}

// Rows a tile side of `b` occupies in an LDS slot: whole DMA instructions of 64 rows (K-contiguous), or a
// power-of-two number of 8-element chunks per K line (K-strided).
constexpr int slot_rows(bool kc, int b) { return kc ? (b + 63) / 64 * 64 : (b <= 128 ? 128 : 256); }

// chunk position `pos` of a slot -> (line, chunk) it holds.  K-contiguous [R rows][64 k]: chunk p of row r
// holds k-chunk p ^ ((r >> 1) & 7).  K-strided [64 k][R rows]: chunk p of line k holds row-chunk p ^ kline_swz(k, R).
template <bool KC, int R>
NTP_HD void slot_src(int pos, int& line, int& chunk) {
  if constexpr (KC) {
    line = pos >> 3;
    chunk = (pos & 7) ^ ((line >> 1) & 7);
  } else {
    constexpr int CPL = R / 8;
    line = pos / CPL;
    chunk = (pos % CPL) ^ kline_swz(line, R);
  }
}

// Byte offset, from the operand's base at K tile 0, of the 16-byte chunk that slot position (line, chunk)
// takes from a tile whose first row (of the non-K dimension) is row0; lim = extent of that dimension.
// Rows past the edge repeat the last one; a K-strided chunk past the edge repeats the last whole chunk.
template <bool KC>
NTP_HD uint32_t dma_offset(int64_t ld, int row0, int lim, int line, int chunk) {
  if constexpr (KC) {
    const int row = imin(row0 + line, lim - 1);
    return uint32_t((int64_t(row) * ld + chunk * 8) * 2);
  } else {
    const int col = imin(row0 + chunk * 8, ((lim - 1) >> 3) << 3);
    return uint32_t((int64_t(line) * ld + col) * 2);
  }
}

// Bytes of an operand that the kernel may touch, counted from its first element: the hardware range check
// of the DMA loads is set to this, so that an offset beyond it reads zeros instead of memory.
//   K-contiguous [rows x K], ld: rows - 1 whole rows and k_reach elements of the last one, k_reach = K, or K
//     rounded up to 64 when the caller vouches for zero-filled pad columns (K tail through the ring);
//   K-strided [K x rows], ld: K - 1 whole lines and the last one up to the end of its last 8-element chunk.
NTP_HD int64_t operand_extent_bytes(bool kc, int64_t rows, int64_t K, int64_t ld, bool k_pad_64) {
  if (rows <= 0 || K <= 0) return 0;
  if (kc) return ((rows - 1) * ld + (k_pad_64 ? (K + 63) / 64 * 64 : K)) * 2;
  return ((K - 1) * ld + (rows + 7) / 8 * 8) * 2;
}

// ---- the deep-pipelined kernel (ntp_gemm_deep.h): the whole K range of a chunk, tail included, goes through the ring ----
// A K chunk that starts at k_first has buffer views that start this many bytes into the operand and end where the operand ends.
NTP_HD uint32_t deep_view_shift(bool kc, int64_t k_first, int64_t ld) { return uint32_t((kc ? k_first : k_first * ld) * 2); }
// Bytes of the operand that the loads may touch: a K-contiguous A is read in whole chunks of 8 (the caller vouches for zeros from K on).
NTP_HD int64_t deep_extent_bytes(bool kc, int64_t rows, int64_t K, int64_t ld) {
  return operand_extent_bytes(kc, rows, kc ? (K + 7) / 8 * 8 : K, ld, false);
}
// Offset past every view of that kernel (its operands are below 2 GiB): where the loads of a K-contiguous operand's chunks at k >= K of the last K tile go.
constexpr uint32_t kNowhere = 0x80000000u;
// Whether chunk `chunk` of the last of nk K tiles of a K range of K elements starts at or past K.
template <bool KC>
NTP_HD bool deep_cut(int nk, int chunk, int K) {
  return KC && (nk - 1) * DK + chunk * 8 >= K;
}

// ---- the ping-pong kernel (ntp_gemm_pp.h): views, extents and K tails as above, operands up to 4 GiB, and a ring that runs on past an output tile ----
// Offset at or past the end of every view: an operand is below 4 GiB and a whole number of 16-byte chunks (a multiple of 8 elements a row).  It goes with a scalar
// offset of 0: no sum of the two overflows, and no scalar offset lies past the view that it is checked against.
constexpr uint32_t kPastAll = 0xFFFFFFF0u;
// K tile j of an output tile with nk of them: the scalar offset of its loads.  The last one of a ragged K (cut) has it in its vector offsets; past it come the
// first K tiles of the next output tile (more), or nothing.
NTP_HD uint32_t pp_scalar_offset(int j, int nk, bool cut, bool more, uint32_t step) {
  if (j < nk) return cut && j == nk - 1 ? 0u : uint32_t(j) * step;
  return more ? uint32_t(j - nk) * step : 0u;
}
// Vector offset of the chunk at slot position (line, chunk) in the last K tile of a ragged K, from its offset in K tile 0: past the view where it starts at or past K.
template <bool KC>
NTP_HD uint32_t pp_cut_offset(uint32_t off, uint32_t step, int nk, int line, int chunk, int K) {
  return (nk - 1) * DK + (KC ? chunk * 8 : line) >= K ? kPastAll : off + uint32_t(nk - 1) * step;
}

// Virtual block v of nblk = tiles_m * tiles_n -> output tile.  Workgroups are dealt round-robin to the 8
// XCDs (each with its own L2), so virtual block v belongs to XCD v & 7; every XCD walks a contiguous range
// of tiles in groups of 8 tile rows, so that its workgroups share operands.
struct TilePos {
  int tile_m, tile_n;
};
NTP_HD TilePos place_tile(int v, int tiles_m, int tiles_n) {
  const int nblk = tiles_m * tiles_n;
  const int xq = nblk >> 3, xr = nblk & 7, xcd = v & 7;
  const int L = xcd * xq + imin(xcd, xr) + (v >> 3);
  constexpr int GM = 8;
  const int width = GM * tiles_n;
  const int first_m = (L / width) * GM;
  const int gsz = imin(tiles_m - first_m, GM);
  TilePos p;
  p.tile_m = first_m + (L % width) % gsz;
  p.tile_n = (L % width) / gsz;
  return p;
}

// Order in which the XCDs walk over their tiles where they have more than a round of their 32 compute units: XCD x begins x rounds into its range and
// comes to the range's start last.  Begun at their starts, the XCDs are at the same few columns, or half a row apart, all the time, and where rows are a power
// of two long their loads and stores then meet in the same memory channels (8192 x 16384 over K = 750, 256 x 256 tiles, rows of 32 KiB: 236 -> 196 us; 8192 x
// 8192 over 1024 130 -> 121; rows of 24 KiB 271 -> 273, within the runs' spread; by an eighth of a round or by two rounds 233 and 207).
NTP_HD int rotate_walk(int v, int nblk) {
  const int xcd = v & 7, n_x = (nblk >> 3) + (xcd < (nblk & 7) ? 1 : 0);
  return n_x > 32 ? ((v >> 3) + 32 * xcd) % n_x * 8 + xcd : v;
}

// K tiles that go through the ring for a contraction of K elements: the whole ones, plus the tail tile when
// it may go through the ring too.
NTP_HD int ring_k_tiles(int K, bool ring_tail) { return K / DK + ((ring_tail && K % DK) ? 1 : 0); }

}  // namespace ntp_gemm

#endif  // NTP_GEMM_ADDR_H_
