// Gradient reshard: repack a partitioned tensor between two TP layouts.
// (Sec. 3.1 "Shard-mapping algorithm"; Appendix: pre-sync hook and post-sync reshard.)
//
// The host turns the two shard plans into sub-shards (segments); each segment is a
// 2-D copy: `rows` rows of `row_bytes` bytes with independent source / destination
// strides.  One kernel launch copies up to kMaxSegs segments.  A workgroup takes about
// 64 KiB of a segment (a block of rows, or 8 KiB pieces of long rows) and deals all
// its 16-byte chunks to the threads as one flat list, so short rows (small sub-shards)
// and long rows use the lanes equally well.  The 16-byte accesses need only 4-byte
// alignment, so the two layouts may be misaligned against each other (odd shard
// widths); loads are non-temporal, stores too when the destination rows are 16-byte
// aligned.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <utility>
#include <vector>

#include "ntp_internal.h"

namespace {

constexpr int kMaxSegs = 56;          // per launch; the argument block stays below 4 KiB
constexpr int kThreads = 256;         // 4 wavefronts
constexpr int kWaves = kThreads / 64;
constexpr int64_t kColChunk = 8192;   // bytes of a row handled by one workgroup
constexpr int64_t kBlockBytes = 65536;  // target bytes per workgroup

struct CopySeg {
  const char* src;
  char* dst;
  int64_t src_stride, dst_stride;  // bytes between rows
  int64_t row_bytes, rows;
  uint32_t first_block;     // first workgroup of this segment
  uint32_t col_chunks;      // pieces a row is cut into
  uint32_t rows_per_block;
  uint32_t pad_;
};

struct CopyBatch {
  CopySeg seg[kMaxSegs];
  int32_t nseg;
  int32_t elem_size;
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));

// An address that was read from LDS, as a pointer to device memory (without the address space the compiler would use flat loads).
template <typename T>
__device__ __forceinline__ const T __attribute__((address_space(1))) * global_ptr(uint64_t p) {
  return reinterpret_cast<const T __attribute__((address_space(1)))*>(p);
}

constexpr int kUnroll = 4;  // independent 16-byte transfers per lane in flight

// Exact n / d by a multiply-high with m = ceil(2^32 / d), valid for d >= 2 and n * d <= 2^32
// (d = 1 would need m = 2^32: fast_div passes n through).
__device__ __forceinline__ uint32_t div_magic(uint32_t d) { return uint32_t(((uint64_t(1) << 32) + d - 1) / d); }
__device__ __forceinline__ uint32_t fast_div(uint32_t n, uint32_t d, uint32_t magic) {
  return d == 1 ? n : __umulhi(n, magic);
}

// A workgroup copies `nrows` row pieces of `n` bytes each (row i at s + i * ss -> d + i * ds).
// The pieces are cut into 16-byte chunks counted from the piece start and ALL chunks of all rows
// are dealt to the threads as one flat list (item -> row, chunk by a multiply-high), so that short
// pieces (a few elements per row: the small sub-shards) keep every lane busy just like long ones.
// The 16-byte accesses need only 4-byte alignment, so source and destination may be misaligned
// against each other (odd shard widths).  What is left of each piece (n % 16 bytes) is copied
// element by element from a second flat list.
template <int ESZ, bool NT_STORE>
__device__ __forceinline__ void block_copy(const char* __restrict__ s, int64_t ss, char* __restrict__ d, int64_t ds,
                                           uint32_t nrows, uint32_t n, uint32_t tid) {
  const uint32_t cpr = n >> 4;  // whole chunks per row piece
  if (cpr > 0) {
    const uint32_t magic = div_magic(cpr), nitems = nrows * cpr;
    for (uint32_t base = tid; base < nitems; base += kThreads * kUnroll) {
      u32x4 v[kUnroll];
      uint32_t row[kUnroll], off[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const uint32_t item = base + u * kThreads;
        row[u] = fast_div(item, cpr, magic);
        off[u] = (item - row[u] * cpr) << 4;
        if (item < nitems)
          v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_a4*>(s + int64_t(row[u]) * ss + off[u]));
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        if (base + u * kThreads < nitems) {
          char* p = d + int64_t(row[u]) * ds + off[u];
          if constexpr (NT_STORE)
            __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4*>(p));
          else
            *reinterpret_cast<u32x4_a4*>(p) = v[u];
        }
      }
    }
  }
  const uint32_t te = (n & 15) / ESZ;  // leftover elements per row piece
  if (te > 0) {
    const uint32_t magic = div_magic(te), nitems = nrows * te, t0 = cpr << 4;
    for (uint32_t item = tid; item < nitems; item += kThreads) {
      const uint32_t row = fast_div(item, te, magic);
      const uint32_t o = t0 + (item - row * te) * ESZ;
      if constexpr (ESZ == 4)
        *reinterpret_cast<uint32_t*>(d + int64_t(row) * ds + o) = *reinterpret_cast<const uint32_t*>(s + int64_t(row) * ss + o);
      else
        *reinterpret_cast<uint16_t*>(d + int64_t(row) * ds + o) = *reinterpret_cast<const uint16_t*>(s + int64_t(row) * ss + o);
    }
  }
}

// 2-byte elements whose addresses are only 2-byte aligned: element-wise copy
__device__ __forceinline__ void block_copy_halfwords(const char* __restrict__ s, int64_t ss, char* __restrict__ d, int64_t ds,
                                                     uint32_t nrows, uint32_t n, uint32_t tid) {
  const uint32_t epr = n >> 1, magic = div_magic(epr), nitems = nrows * epr;
  for (uint32_t item = tid; item < nitems; item += kThreads) {
    const uint32_t row = fast_div(item, epr, magic);
    const uint32_t o = (item - row * epr) << 1;
    *reinterpret_cast<uint16_t*>(d + int64_t(row) * ds + o) = *reinterpret_cast<const uint16_t*>(s + int64_t(row) * ss + o);
  }
}

__global__ __launch_bounds__(kThreads) void reshard_copy_kernel(const CopyBatch batch) {
  // find this workgroup's segment (segments are few; the table sits in the kernel arguments)
  const uint32_t b = blockIdx.x;
  int si = 0;
  for (int i = 1; i < batch.nseg; ++i)
    if (batch.seg[i].first_block <= b) si = i;
  const CopySeg& sg = batch.seg[si];
  const uint32_t lb = b - sg.first_block;
  const uint32_t rg = lb / sg.col_chunks;
  const uint32_t cc = lb - rg * sg.col_chunks;
  const int64_t c0 = int64_t(cc) * kColChunk;
  const uint32_t nbytes = uint32_t(std::min<int64_t>(kColChunk, sg.row_bytes - c0));
  const int64_t r0 = int64_t(rg) * sg.rows_per_block;
  const uint32_t nrows = uint32_t(std::min<int64_t>(sg.rows - r0, sg.rows_per_block));
  const char* s = sg.src + r0 * sg.src_stride + c0;
  char* d = sg.dst + r0 * sg.dst_stride + c0;
  const uintptr_t sa = reinterpret_cast<uintptr_t>(sg.src), da = reinterpret_cast<uintptr_t>(sg.dst);
  // 16-byte accesses need 4-byte aligned rows on both sides (always true for 4-byte elements)
  const bool wide = batch.elem_size == 4 || (((sa | da | uintptr_t(sg.src_stride) | uintptr_t(sg.dst_stride)) & 3) == 0);
  const bool dst16 = ((da | uintptr_t(sg.dst_stride)) & 15) == 0;
  const uint32_t tid = threadIdx.x;
  if (batch.elem_size == 4) {
    if (dst16)
      block_copy<4, true>(s, sg.src_stride, d, sg.dst_stride, nrows, nbytes, tid);
    else
      block_copy<4, false>(s, sg.src_stride, d, sg.dst_stride, nrows, nbytes, tid);
  } else if (wide) {
    block_copy<2, false>(s, sg.src_stride, d, sg.dst_stride, nrows, nbytes, tid);
  } else {
    block_copy_halfwords(s, sg.src_stride, d, sg.dst_stride, nrows, nbytes, tid);
  }
}


// ---- column-partitioned tensors: destination-major gather ------------------
// A job is a block of destination columns of one destination shard together with the pieces
// (sub-shards) that fill it, each from another source shard.  A workgroup takes a block of
// destination rows and copies all pieces of those rows, so destination rows are written whole and
// in order.  Within a piece the 16-byte chunks are aligned on the DESTINATION address (aligned
// non-temporal stores; the loads tolerate any 4-byte alignment); what lies before the first and
// after the last aligned chunk of a row piece is copied word by word.
constexpr int kMaxPieces = 8;
constexpr int kMaxJobs = 14;  // the argument block stays below 4 KiB

struct Piece {
  const char* src;      // byte that goes to column `begin` of destination row 0 of the job
  int64_t src_stride;   // bytes between source rows
  uint32_t begin, end;  // byte range within the job's destination row
};
struct GatherJob {
  char* dst;            // first byte of the job's column block in destination row 0
  int64_t dst_stride;
  uint32_t rows, npieces;
  Piece piece[kMaxPieces];
};
struct GatherBatch {
  GatherJob job[kMaxJobs];  // all with the same number of rows
  int32_t njobs;
  uint32_t rows_per_block;
};

// One piece of `nrows` destination rows, n bytes per row.  HBM is written in 64-byte units, and a
// unit written in two parts costs two transactions, so in every row the copy is cut at the 64-byte
// boundaries of the DESTINATION address: `head` bytes (a multiple of 4 below 64) come before the
// first boundary.  Pass 1 moves the whole units of all rows as one flat list of 16-byte chunks (four
// neighbouring lanes fill one unit with one aligned non-temporal store instruction; the loads take
// any 4-byte alignment); pass 2 moves what is left at the two ends of each row word by word, again as
// one flat list.  Offsets inside the block fit in 32 bits (the host sees to that).
__device__ __forceinline__ void piece_copy_aligned(const char* __restrict__ s, uint32_t ss, char* __restrict__ d, uint32_t ds,
                                                   uint32_t nrows, uint32_t n, uint32_t tid) {
  const uint32_t dlow = uint32_t(reinterpret_cast<uintptr_t>(d)) & 63u;
  const uint32_t cpr = (n >> 6) << 2;  // chunks of the most whole units a row can hold
  if (cpr > 0) {
    const uint32_t magic = div_magic(cpr), nitems = nrows * cpr;
    for (uint32_t base = tid; base < nitems; base += kThreads * kUnroll) {
      u32x4 v[kUnroll];
      uint32_t doff[kUnroll];
      bool ok[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const uint32_t item = base + u * kThreads;
        const uint32_t row = nrows == 1 ? 0u : fast_div(item, cpr, magic);
        const uint32_t k = item - row * cpr;
        const uint32_t drow = row * ds;
        const uint32_t head = (0u - (dlow + drow)) & 63u;
        const uint32_t st = head + (k << 4);
        ok[u] = item < nitems && head + ((k | 3u) << 4) + 16u <= n;  // the whole unit of this chunk fits
        doff[u] = drow + st;
        if (ok[u]) v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_a4*>(s + (row * ss + st)));
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u)
        if (ok[u]) __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4*>(d + doff[u]));
    }
  }
  // the ends, one word per item: item = 32 row + 16 (0: before the first boundary, 1: after the last whole unit) + word
  for (uint32_t item = tid; item < 32 * nrows; item += kThreads) {
    const uint32_t row = item >> 5, drow = row * ds, w = item & 15u;
    const uint32_t head = min(n, (0u - (dlow + drow)) & 63u);
    const uint32_t st = (item & 16u) ? head + ((n - head) & ~63u) : 0u;
    const uint32_t en = (item & 16u) ? n : head;
    if (st + 4u * w < en)
      *reinterpret_cast<uint32_t*>(d + (drow + st + 4u * w)) = *reinterpret_cast<const uint32_t*>(s + (row * ss + st + 4u * w));
  }
}

// Workgroup b takes row block b / njobs of job b % njobs: the workgroups that run at the same time
// cover the same rows of neighbouring destination shards, so the two destination shards that split
// a source row read it close together in time (its lines are fetched from HBM once).
__global__ __launch_bounds__(kThreads) void reshard_gather_kernel(const GatherBatch batch) {
  const uint32_t rbi = blockIdx.x / uint32_t(batch.njobs), ji = blockIdx.x - rbi * uint32_t(batch.njobs);
  const GatherJob& job = batch.job[ji];
  const int64_t r0 = int64_t(rbi) * batch.rows_per_block;
  const uint32_t nrows = uint32_t(std::min<int64_t>(int64_t(job.rows) - r0, batch.rows_per_block));
  for (uint32_t p = 0; p < job.npieces; ++p) {
    const Piece& pc = job.piece[p];
    piece_copy_aligned(pc.src + r0 * pc.src_stride, uint32_t(pc.src_stride), job.dst + r0 * job.dst_stride + pc.begin,
                       uint32_t(job.dst_stride), nrows, pc.end - pc.begin, threadIdx.x);
  }
}

// Dense destination shards: the destination is treated as ONE flat byte range, cut into blocks at
// 64-byte boundaries, and every 16-byte chunk of it is stored whole and aligned no matter where rows
// and pieces begin (odd shard widths).  A chunk that lies inside one piece of one row is read with
// one (unaligned) 16-byte load; a chunk that straddles a row end or a piece boundary is assembled
// from four single words.  Needs: destination 64-byte aligned and dense, (kFlatBlock + W) * W <= 2^32
// for the row width W in bytes (exact multiply-high division), source offsets inside a block < 2^32.
constexpr uint32_t kFlatBlockMax = 65536;

__global__ __launch_bounds__(kThreads) void reshard_flat_kernel(const GatherBatch batch) {
  // consecutive workgroups take consecutive blocks of one job (measured faster than dealing the jobs round)
  const uint32_t nblk = gridDim.x / uint32_t(batch.njobs);
  const uint32_t ji = blockIdx.x / nblk, bi = blockIdx.x - ji * nblk;
  const GatherJob& job = batch.job[ji];
  const uint32_t np = job.npieces;
  const uint32_t W = job.piece[np - 1].end;
  const int64_t T = int64_t(job.rows) * W;
  const uint32_t kFlatBlock = batch.rows_per_block;  // bytes per block here
  const int64_t b0 = int64_t(bi) * kFlatBlock;
  if (b0 >= T) return;
  const uint32_t nb = uint32_t(std::min<int64_t>(kFlatBlock, T - b0));
  const int64_t row0 = b0 / W;
  const uint32_t c0 = uint32_t(b0 - row0 * W);
  const uint32_t magic = div_magic(W);
  char* __restrict__ d = job.dst + b0;
  const uint32_t nchunks = (nb + 15) >> 4;
  for (uint32_t base = threadIdx.x; base < nchunks; base += kThreads * kUnroll) {
    u32x4 v[kUnroll];
    uint32_t len[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint32_t k = base + u * kThreads;
      len[u] = k < nchunks ? min(16u, nb - (k << 4)) : 0u;
      const uint32_t x = c0 + (k << 4);
      const uint32_t rr = fast_div(x, W, magic);
      const uint32_t col = x - rr * W;
      bool got = len[u] == 0;
      if (len[u] == 16 && col + 16u <= W) {
        for (uint32_t p = 0; p < np; ++p) {
          const Piece& pc = job.piece[p];
          if (col >= pc.begin && col + 16u <= pc.end) {
            const char* sb = pc.src + row0 * pc.src_stride;
            v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_a4*>(sb + (rr * uint32_t(pc.src_stride) + (col - pc.begin))));
            got = true;
          }
        }
      }
      if (!got) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          if (uint32_t(w) * 4 >= len[u]) continue;
          const uint32_t rw = fast_div(x + 4u * w, W, magic), cw = x + 4u * w - rw * W;  // rows may be shorter than a chunk
          for (uint32_t p = 0; p < np; ++p) {
            const Piece& pc = job.piece[p];
            if (cw >= pc.begin && cw < pc.end) {
              const char* sb = pc.src + row0 * pc.src_stride;
              v[u][w] = *reinterpret_cast<const uint32_t*>(sb + (rw * uint32_t(pc.src_stride) + (cw - pc.begin)));
            }
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      char* dp = d + ((base + u * kThreads) << 4);
      if (len[u] == 16) {
        __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4*>(dp));
      } else {
#pragma unroll
        for (int w = 0; w < 3; ++w)
          if (uint32_t(w) * 4 < len[u]) reinterpret_cast<uint32_t*>(dp)[w] = v[u][w];
      }
    }
  }
}

// The same for 2-byte elements: loads of any 2-byte alignment, and a chunk that straddles a row end or a piece boundary is
// put together half-word by half-word in a second pass (halves have to be waited for before they are packed), whose loads
// go out before the first pass's are waited for.  The pieces are looked up in LDS.  Bound by HBM: 12288 x 49152 from 8 to 7
// ranks 612 to 421 us (5.7 TB/s) against the row-by-row copy, whose 16-byte stores are not aligned.  (4-byte elements stay
// with the kernel above: the same second pass costs them 4 % at odd widths.)
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6))) void reshard_flat2_kernel(const GatherBatch batch) {
  struct PieceLds {
    uint64_t adj;  // what goes to column c of the block's row r is at adj + r * stride + c
    uint32_t stride, end;
  };
  __shared__ PieceLds piece[kMaxPieces];
  // consecutive workgroups take consecutive blocks of one job (measured faster than dealing the jobs round)
  const uint32_t nblk = gridDim.x / uint32_t(batch.njobs);
  const uint32_t ji = blockIdx.x / nblk, bi = blockIdx.x - ji * nblk;
  const GatherJob& job = batch.job[ji];
  const uint32_t np = job.npieces;
  const uint32_t W = job.piece[np - 1].end;
  const int64_t T = int64_t(job.rows) * W;
  const uint32_t blk = batch.rows_per_block;  // bytes per block here
  const int64_t b0 = int64_t(bi) * blk;
  if (b0 >= T) return;  // the whole workgroup, before the barrier
  const uint32_t nb = uint32_t(std::min<int64_t>(blk, T - b0));
  const int64_t row0 = b0 / W;
  const uint32_t c0 = uint32_t(b0 - row0 * W);
  if (threadIdx.x < np) {
    const Piece& pc = job.piece[threadIdx.x];
    piece[threadIdx.x] = PieceLds{uint64_t(reinterpret_cast<uintptr_t>(pc.src)) + uint64_t(row0 * pc.src_stride) - pc.begin, uint32_t(pc.src_stride), pc.end};
  }
  __syncthreads();
  const bool wide = W > blk + 16u;  // at most one row end in a block
  const uint32_t magic = div_magic(W);
  char* __restrict__ d = job.dst + b0;
  const uint32_t nchunks = (nb + 15) >> 4;
  auto locate = [&](uint32_t x, uint32_t& row, uint32_t& col) {
    row = wide ? uint32_t(x >= W) : fast_div(x, W, magic);
    col = x - row * W;
  };
  auto piece_of = [&](uint32_t col) {
    uint32_t pi = 0;
    for (uint32_t p = 1; p < np; ++p) pi += col >= job.piece[p].begin;
    return piece[pi];
  };
  for (uint32_t base = threadIdx.x; base < nchunks; base += kThreads * kUnroll) {
    u32x4 v[kUnroll];
    bool run[kUnroll];
    uint32_t split = 0;  // bit u: chunk u goes half-word by half-word
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint32_t k = base + u * kThreads;
      uint32_t row, col;
      locate(c0 + (k < nchunks ? k << 4 : 0u), row, col);
      const PieceLds pc = piece_of(col);
      run[u] = (k << 4) + 16u <= nb && col + 16u <= pc.end;
      split |= k < nchunks && !run[u] ? 1u << u : 0u;
      if (run[u]) v[u] = __builtin_nontemporal_load(global_ptr<u32x4_a2>(pc.adj + (row * pc.stride + col)));
    }
#pragma unroll 1
    while (split) {
      const uint32_t k = base + uint32_t(__ffs(split) - 1) * kThreads;
      split &= split - 1;
      const uint32_t len = min(16u, nb - (k << 4));
      uint16_t val[8];
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        if (uint32_t(w) * 2 >= len) continue;
        uint32_t row, col;  // rows may be shorter than a chunk
        locate(c0 + (k << 4) + uint32_t(w) * 2, row, col);
        const PieceLds pc = piece_of(col);
        val[w] = *global_ptr<uint16_t>(pc.adj + (row * pc.stride + col));
      }
      char* dp = d + (k << 4);
      if (len == 16) {
        u32x4 out;
#pragma unroll
        for (int w = 0; w < 4; ++w) out[w] = uint32_t(val[2 * w]) | uint32_t(val[2 * w + 1]) << 16;
        __builtin_nontemporal_store(out, reinterpret_cast<u32x4*>(dp));
      } else {
#pragma unroll
        for (int w = 0; w < 8; ++w)
          if (uint32_t(w) * 2 < len) reinterpret_cast<uint16_t*>(dp)[w] = val[w];
      }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (run[u]) __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4*>(d + ((base + u * kThreads) << 4)));
  }
}

// Whether a job's destination is a dense aligned shard that its flat kernel can divide into rows exactly.
bool flat_ok(const GatherJob& j, int64_t block, int64_t esz) {
  const int64_t W = j.piece[j.npieces - 1].end;
  int64_t smax = 0;
  for (uint32_t p = 0; p < j.npieces; ++p) smax = std::max(smax, j.piece[p].src_stride);
  return j.dst_stride == W && (reinterpret_cast<uintptr_t>(j.dst) & 63) == 0 &&
         ((esz == 2 && W > block + 16) || (block + W + 16) * W <= (int64_t(1) << 32)) && smax * (block / W + 2) < (int64_t(1) << 32);
}

// ---- dense ranges (row-partitioned tensors whose shards are dense): plain streaming copy --------
constexpr int kMaxRanges = 100;  // 100 x 32 B + header < 4 KiB of kernel arguments
constexpr int64_t kDenseBlock = 16384;  // bytes per workgroup
struct DenseRange {
  const char* src;
  char* dst;
  int64_t bytes;         // multiple of 16; both pointers 16-byte aligned
  uint32_t first_block;
  uint32_t pad_;
};
struct DenseBatch {
  DenseRange r[kMaxRanges];
  int32_t n;
};

__global__ __launch_bounds__(kThreads) void reshard_dense_kernel(const DenseBatch batch) {
  const uint32_t b = blockIdx.x;
  // last range whose first block is <= b (one load per lane and a ballot: 1-2 % slower at 7 of 15 shapes, 16384 x 16384 in heads from 71 to 72
  // ranks 481 -> 487 us, 28672 x 8192 from 9 to 8 329 -> 337; faster at 49152 x 12288 between 7 and 8 only, 861 -> 848)
  int lo = 0, hi = batch.n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (batch.r[mid].first_block <= b) lo = mid;
    else hi = mid - 1;
  }
  const DenseRange& rg = batch.r[lo];
  const int64_t off = int64_t(b - rg.first_block) * kDenseBlock;
  const uint32_t n16 = uint32_t(std::min<int64_t>(kDenseBlock, rg.bytes - off) >> 4);
  const u32x4* s = reinterpret_cast<const u32x4*>(rg.src + off);
  u32x4* d = reinterpret_cast<u32x4*>(rg.dst + off);
  for (uint32_t base = threadIdx.x; base < n16; base += kThreads * kUnroll) {
    u32x4 v[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (base + u * kThreads < n16) v[u] = __builtin_nontemporal_load(s + base + u * kThreads);
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (base + u * kThreads < n16) __builtin_nontemporal_store(v[u], d + base + u * kThreads);
  }
}

// ---- layouts given unit by unit (Sec. 3.1, Alg. 1): gather through a unit table -------------------
// The destination shards are dense and are written as one flat byte range each, cut into blocks, every
// 16-byte chunk stored whole and aligned.  The plan keeps in device memory, for every unit of every
// destination shard (one shard after the other), where it comes from: rank << 24 | unit in that rank's shard.
// The table is 4 bytes a unit and stays in the L2s; nothing about it has to fit in LDS, so every layout of a plan
// goes through it, whether a destination shard is two long runs or every unit comes from another rank.
// (The run table, reshard_runs_kernel, keeps a 32-byte record per run in LDS: without the unit table, layouts with more than about
// 1300 runs a shard, or with rows above 57 KB, were copied sub-shard by sub-shard, 8 units a job: 93.8 ms for the gradients of a
// hidden-12800 layer between TP 7 and TP 5, which this table moves in 2.10 ms.)
constexpr int kMaxRanks = 96;       // source ranks, and destination shards per launch: the argument block stays below 4 KiB
constexpr uint32_t kUnitBits = 24;  // of a table entry; the rank has the other 8

// Column-partitioned tensors are copied in bands of rows of about this many bytes, every destination shard's part of a band
// before the next band: where the units of one source row go to several destination shards in turn, its lines are still in the
// device's last-level cache when the next shard needs them (54 to 45 ranks and back 1397 to 960 us).  Elsewhere whole shards one after the other are 3-5 % faster
// (few write streams): ntp_reshard_plan::interleaved.
constexpr int64_t kBandBytes = int64_t(64) << 20;

struct UnitSrc {
  const char* base;  // first byte of the source shard
  uint64_t stride;   // bytes between its rows
};
struct TableDst {
  char* dst;
  uint32_t first_unit, n_units;    // this shard's slice of the table
  uint32_t first_block, per_band;  // its blocks in a band
};
struct TableBatch {
  UnitSrc src[kMaxRanks];
  TableDst dst[kMaxRanks];
  const uint32_t* table;
  uint32_t rows;        // columns partitioned: rows of the tensor
  uint32_t row_bytes;   // rows partitioned: bytes of a row
  uint32_t unit;        // columns partitioned: bytes of a unit; rows partitioned: rows of a unit
  uint32_t block_bytes;
  uint32_t band_blocks;
  int32_t ndst, nsrc;
};

// The destination shard of block `b` of a band (the last one whose first block is <= b): one load per lane instead of a
// chain of scalar loads.
__device__ __forceinline__ int table_dst(const TableBatch& batch, uint32_t b) {
  const int lane = threadIdx.x & 63;
  int n = 0;
#pragma unroll
  for (int i = 0; i < kMaxRanks; i += 64) n += __popcll(__ballot(i + lane < batch.ndst && batch.dst[min(i + lane, kMaxRanks - 1)].first_block <= b));
  return n - 1;
}

// Column-partitioned, 4-byte elements; ONE: units of one element.  A chunk whose four words follow each other in one source
// row is moved by one 16-byte load (any 4-byte alignment), the others (units of several ranks side by side, row ends) by four
// word loads in a second pass, before the first pass's loads are waited for.  Bound by HBM where the runs are long (49152
// columns of fp32 between 32 and 30 ranks: 5.4 TB/s, 892 us; the run table in LDS took 900), by the word loads where they are
// single units (54 to 45 ranks and back: 3.1 TB/s).  Six wavefronts per SIMD: at eight the second pass spills or has to wait
// for the stores (920 us).
template <bool ONE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6))) void reshard_table_cols_kernel(const TableBatch batch) {
  __shared__ UnitSrc src[kMaxRanks];
  for (int i = threadIdx.x; i < batch.nsrc; i += kThreads) src[i] = batch.src[i];
  const uint32_t band = blockIdx.x / batch.band_blocks, bb = blockIdx.x - band * batch.band_blocks;
  const TableDst& dd = batch.dst[table_dst(batch, bb)];
  const uint32_t ub = ONE ? 4u : batch.unit, blk = batch.block_bytes;
  const uint32_t W = dd.n_units * ub;
  const int64_t T = int64_t(batch.rows) * W;
  const int64_t b0 = (int64_t(band) * dd.per_band + (bb - dd.first_block)) * blk;
  if (b0 >= T) return;  // the whole workgroup, before the barrier
  const uint32_t nb = uint32_t(std::min<int64_t>(blk, T - b0));
  const uint32_t row0 = uint32_t(b0 / W), c0 = uint32_t(b0 - int64_t(row0) * W);
  char* __restrict__ d = dd.dst + b0;
  const uint32_t* __restrict__ tab = batch.table + dd.first_unit;
  const bool wide = W > blk + 16u;  // at most one row end in a block; else the multiply-high is exact (see table_path_ok)
  const uint32_t magic_w = div_magic(W), magic_u = div_magic(ub);
  const uint32_t nchunks = (nb + 15) >> 4;
  auto row_of = [&](uint32_t x) { return wide ? uint32_t(x >= W) : __umulhi(x, magic_w); };
  auto unit_of = [&](uint32_t c) { return ONE ? c >> 2 : __umulhi(c, magic_u); };
  auto locate = [&](uint32_t k, uint32_t& row, uint32_t& col) {
    const uint32_t x = c0 + (k < nchunks ? k << 4 : 0u);
    row = row_of(x);
    col = x - row * W;
  };
  auto entries = [&](uint32_t col) {
    u32x4 e;
    if constexpr (ONE) {
      e = *reinterpret_cast<const u32x4_a4*>(tab + (col >> 2));  // the table ends in three spare entries
    } else {
#pragma unroll
      for (int w = 0; w < 4; ++w) e[w] = tab[min(unit_of(col + 4u * w), dd.n_units - 1u)];
    }
    return e;
  };
  auto at = [&](uint32_t row, uint32_t e, uint32_t off) {
    const UnitSrc sr = src[e >> kUnitBits];
    return uint64_t(reinterpret_cast<uintptr_t>(sr.base)) + (uint64_t(row) * uint32_t(sr.stride) + ((e & ((1u << kUnitBits) - 1u)) * ub + off));
  };
  for (uint32_t first = 0; first < nchunks; first += kThreads * kUnroll) {
    const uint32_t base = first + threadIdx.x;
    u32x4 v[kUnroll], e[kUnroll];
    uint32_t row[kUnroll], col[kUnroll];
    uint32_t words = 0;  // bit u: chunk u goes word by word
    bool run[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint32_t k = base + u * kThreads;
      locate(k, row[u], col[u]);
      e[u] = entries(col[u]);
    }
    if (first == 0) __syncthreads();  // `src` is whole; the first entries are on their way
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint32_t k = base + u * kThreads, u0 = unit_of(col[u]);
      bool one = (k << 4) + 16u <= nb && col[u] + 16u <= W;
#pragma unroll
      for (int w = 1; w < 4; ++w) one = one && e[u][w] - e[u][0] == unit_of(col[u] + 4u * w) - u0;
      run[u] = one;
      words |= k < nchunks && !one ? 1u << u : 0u;
      if (one)
        v[u] = __builtin_nontemporal_load(global_ptr<u32x4_a4>(at(row0 + row[u], e[u][0], col[u] - u0 * ub)));
    }
    // looked up again rather than held in registers (the entries are in the first-level cache); every lane takes its next one,
    // so that a wavefront with a few of them in different places makes few rounds
#pragma unroll 1
    while (words) {
      const uint32_t k = base + uint32_t(__ffs(words) - 1) * kThreads;
      words &= words - 1;
      uint32_t r0, cc;
      locate(k, r0, cc);
      const u32x4 en4 = entries(cc);
      const uint32_t len = min(16u, nb - (k << 4));
      u32x4 val;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        uint32_t r = r0, c = cc + 4u * w, en = en4[w];
        if (c >= W) {  // rows may be shorter than a chunk
          const uint32_t x = r * W + c;
          r = row_of(x);
          c = x - r * W;
          en = tab[unit_of(c)];
        }
        if (4u * w < len) val[w] = *global_ptr<uint32_t>(at(row0 + r, en, c - unit_of(c) * ub));
      }
      char* dp = d + (k << 4);
      if (len == 16) {
        __builtin_nontemporal_store(val, reinterpret_cast<u32x4*>(dp));
      } else {
#pragma unroll
        for (int w = 0; w < 3; ++w)
          if (uint32_t(w) * 4 < len) reinterpret_cast<uint32_t*>(dp)[w] = val[w];
      }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint32_t k = base + u * kThreads;
      if (run[u]) __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4*>(d + (k << 4)));
    }
  }
}

// ---- the same through a run table, for rows of a few KB ------------------------------------------------------------------
// A destination shard is a sequence of runs (units that follow each other in one source shard too); the plan keeps, in device
// memory, the runs of every destination shard and for every destination unit the number of its run.  A workgroup copies both
// tables into LDS (runs joined with this call's source pointers) and then takes one block of the shard, or walks over several
// when the shard is very large.  Chunks that straddle a run boundary or a row end are put on a queue that each wavefront keeps in
// LDS and are put together word by word when the loads of the others are done, with most lanes in use.
// Where the line to the unit table lies (run_table_wanted): 170 layouts, fp32, both kernels in turn.  Rows up to 4.4 KB, tensors from 256 MB
// on, layouts that are not copied in bands: this kernel takes 0.85 to 1.04 of the other's time, 0.95 on
// average over 46 (13824 x 55296 from 67 to 60 ranks 1252 against 1440 us, 16384 x 53248 from 71 to 72 1399 against 1455).  Above 5 KB its
// tables cost more per block than the unit table's lookups (14080 x 56320 from 33 to 25 ranks 1871 against 1357 us), in smaller tensors too
// (4096 x 14336 from 48 to 47 191 against 178), and where lines go to several shards in turn the bands give more (up to 1.5 times).
constexpr int kRunDsts = 16;               // destination shards per launch: few write streams at a time measured fastest
constexpr uint32_t kQueueCap = 512;        // queued chunks per wavefront
constexpr uint32_t kRunBlocksPerCu = 256;  // workgroups per compute unit and launch before they start to walk over several blocks
constexpr int64_t kRunRowMax = 4480;       // bytes of a destination row: at most 1120 units and runs, 55 KB of LDS
constexpr int64_t kRunTensorMin = int64_t(256) << 20;

struct RunDev {      // one run of a destination shard (plan, device memory)
  uint32_t begin, end;  // byte range in a destination row
  uint32_t src_off;     // byte offset in a source row of what goes to `begin`
  uint32_t rank;        // source rank
};
struct RunLds {      // the same, joined with the source pointers of this call
  uint32_t begin, end, stride, pad_;
  uint64_t adj;      // source base + src_off - begin: column c of row r is at adj + r * stride + c
  uint64_t pad2_;
};
struct RunDst {
  char* dst;
  uint32_t idx_first, n_units;   // this shard's slice of the unit -> run numbers
  uint32_t runs_first, n_runs;   // this shard's slice of the runs
};
struct RunBatch {
  UnitSrc src[kMaxRanks];
  RunDst dst[kRunDsts];
  const RunDev* runs;
  const uint16_t* run_of_unit;
  uint32_t rows, unit_bytes, ndst, block_bytes;
};

__host__ __device__ inline uint32_t run_tables_bytes(uint32_t n_runs, uint32_t n_units) {
  return n_runs * uint32_t(sizeof(RunLds)) + ((n_units * 2u + 15u) & ~15u);
}
__host__ __device__ inline uint32_t run_lds_bytes(uint32_t n_runs, uint32_t n_units) {
  return run_tables_bytes(n_runs, n_units) + kWaves * kQueueCap * uint32_t(sizeof(uint2));
}

__global__ __launch_bounds__(kThreads) void reshard_runs_kernel(const RunBatch batch) {
  extern __shared__ __align__(16) unsigned char run_lds[];
  // consecutive workgroups take consecutive blocks of one destination shard
  const uint32_t nslots = gridDim.x / batch.ndst;
  const uint32_t di = blockIdx.x / nslots, slot = blockIdx.x - di * nslots;
  const RunDst& dd = batch.dst[di];
  const uint32_t ub = batch.unit_bytes, blk = batch.block_bytes;
  const uint32_t W = dd.n_units * ub;
  const int64_t T = int64_t(batch.rows) * W;
  int64_t b0 = int64_t(slot) * blk;
  if (b0 >= T) return;  // the whole workgroup leaves: nothing left for it in this shard
  RunLds* const runs = reinterpret_cast<RunLds*>(run_lds);
  uint16_t* const run_of = reinterpret_cast<uint16_t*>(run_lds + dd.n_runs * sizeof(RunLds));
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  uint2* const queue = reinterpret_cast<uint2*>(run_lds + run_tables_bytes(dd.n_runs, dd.n_units)) + wave * kQueueCap;
  for (uint32_t r = threadIdx.x; r < dd.n_runs; r += kThreads) {
    const RunDev rd = batch.runs[dd.runs_first + r];
    const UnitSrc sr = batch.src[rd.rank];
    RunLds o;
    o.begin = rd.begin;
    o.end = rd.end;
    o.stride = uint32_t(sr.stride);
    o.pad_ = 0;
    o.adj = uint64_t(reinterpret_cast<uintptr_t>(sr.base)) + rd.src_off - rd.begin;
    o.pad2_ = 0;
    runs[r] = o;
  }
  for (uint32_t j = threadIdx.x; j < dd.n_units; j += kThreads) run_of[j] = batch.run_of_unit[dd.idx_first + j];
  __syncthreads();  // the only workgroup-wide wait: from here on the wavefronts run on their own

  // W and the unit size are at least 4: the multiply-high division needs no special case
  const uint32_t magic_w = div_magic(W), magic_u = div_magic(ub);
  const char* const dummy = reinterpret_cast<const char*>(batch.runs);  // 16 readable bytes for lanes with nothing to load
  // queued chunks of this wavefront, word by word
  uint32_t nq = 0;  // chunks on this wavefront's queue (the same value in all lanes)
  auto flush = [&]() {
    // what other lanes have queued becomes visible
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t i = lane; i < nq; i += 64) {
      const uint2 e = queue[i];  // {row, byte column} of the chunk's first word
      const int64_t at = int64_t(e.x) * W + e.y;
      const uint32_t len = uint32_t(std::min<int64_t>(16, T - at));
      u32x4 v;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const bool have = uint32_t(w) * 4 < len;
        const uint32_t xw = e.y + (have ? 4u * w : 0u);
        const uint32_t rw = __umulhi(xw, magic_w), cw = xw - rw * W;  // rows may be shorter than a chunk
        const RunLds rn = runs[run_of[__umulhi(cw, magic_u)]];
        v[w] = *reinterpret_cast<const uint32_t*>(rn.adj + (uint64_t(e.x + rw) * rn.stride + cw));
      }
      char* dp = dd.dst + at;
      if (len == 16) {
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dp));
      } else {
#pragma unroll
        for (int w = 0; w < 3; ++w)
          if (uint32_t(w) * 4 < len) reinterpret_cast<uint32_t*>(dp)[w] = v[w];
      }
    }
    // the entries have been read before the queue is filled again
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    nq = 0;
  };

  // this workgroup's blocks: slot, slot + nslots, ...; (row0, c0) = position of the block's first byte
  const int64_t step = int64_t(nslots) * blk;
  const uint32_t step_rows = uint32_t(step / W), step_cols = uint32_t(step - int64_t(step_rows) * W);
  uint32_t row0 = uint32_t(b0 / W);
  uint32_t c0 = uint32_t(b0 - int64_t(row0) * W);
  for (; b0 < T; b0 += step) {
    const uint32_t nb = uint32_t(std::min<int64_t>(blk, T - b0));
    char* __restrict__ d = dd.dst + b0;
    const uint32_t nchunks = (nb + 15) >> 4;
    // the loop bounds are the same for all lanes of a wavefront: every lane takes part in flush()
    for (uint32_t wbase = wave << 6; wbase < nchunks; wbase += kThreads * kUnroll) {
      const uint32_t base = wbase + lane;
      u32x4 v[kUnroll];
      bool ok[kUnroll], slow[kUnroll];
      uint32_t rowq[kUnroll], colq[kUnroll];
      // look every chunk up and start its load; lanes with no chunk, or with a chunk for the slow way,
      // go through the same steps on chunk 0 and load the dummy bytes (no branches, four loads in flight)
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const uint32_t k = base + u * kThreads;
        const bool valid = k < nchunks;
        const uint32_t kb = valid ? k << 4 : 0u;
        const uint32_t x = c0 + kb;
        const uint32_t rr = __umulhi(x, magic_w), col = x - rr * W;
        const RunLds rn = runs[run_of[__umulhi(col, magic_u)]];
        ok[u] = valid && kb + 16u <= nb && col + 16u <= rn.end;
        slow[u] = valid && !ok[u];
        rowq[u] = row0 + rr;
        colq[u] = col;
        const char* p = reinterpret_cast<const char*>(rn.adj + (uint64_t(row0 + rr) * rn.stride + col));
        v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_a4*>(ok[u] ? p : dummy));
      }
      // the chunks that need the slow way go on the queue, in lane order
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const uint64_t m = __ballot(slow[u]);
        if (slow[u]) queue[nq + __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u))] = make_uint2(rowq[u], colq[u]);
        nq += uint32_t(__popcll(m));
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u)
        if (ok[u]) __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4*>(d + ((base + u * kThreads) << 4)));
      // one pass of the loop queues at most 64 * kUnroll chunks per wavefront
      if (nq > kQueueCap - 64 * kUnroll) flush();
    }
    row0 += step_rows;
    c0 += step_cols;
    if (c0 >= W) {
      c0 -= W;
      ++row0;
    }
  }
  flush();
}

// Row-partitioned, rows a multiple of 16 bytes on 16-byte aligned addresses: every chunk lies in one unit.  A source shard
// that is not on this GPU leaves its units' rows untouched.  Bound by HBM: 6.1 TB/s.  One launch for a whole tensor, where the dense
// kernel takes one per 100 runs (a run is one row where several ranks are unloaded onto one): 4608 rows between TP 7 and TP 5,
// with the other two tensors of that layer, 98 to 50 us; 49152 rows between TP 32 and TP 30 890 to 794 us.
__global__ __launch_bounds__(kThreads) void reshard_table_rows_kernel(const TableBatch batch) {
  __shared__ UnitSrc src[kMaxRanks];
  for (int i = threadIdx.x; i < batch.nsrc; i += kThreads) src[i] = batch.src[i];
  const TableDst& dd = batch.dst[table_dst(batch, blockIdx.x)];
  __syncthreads();
  const uint32_t R = batch.row_bytes, unit = batch.unit, blk = batch.block_bytes;
  const int64_t T = int64_t(dd.n_units) * unit * R;
  const int64_t b0 = int64_t(blockIdx.x - dd.first_block) * blk;
  const uint32_t n16 = uint32_t(std::min<int64_t>(blk, T - b0) >> 4);
  const uint32_t row0 = uint32_t(b0 / R), c0 = uint32_t(b0 - int64_t(row0) * R);
  const uint32_t unit0 = row0 / unit, r0 = row0 - unit0 * unit;
  u32x4* __restrict__ d = reinterpret_cast<u32x4*>(dd.dst + b0);
  const uint32_t* __restrict__ tab = batch.table + dd.first_unit + unit0;
  const bool wide = R > blk;  // at most one row end in a block
  const uint32_t magic_r = div_magic(R), magic_u = div_magic(unit);
  for (uint32_t base = threadIdx.x; base < n16; base += kThreads * kUnroll) {
    u32x4 v[kUnroll];
    uint64_t p[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint32_t k = base + u * kThreads, x = c0 + (k < n16 ? k << 4 : 0u);
      const uint32_t rr = wide ? uint32_t(x >= R) : __umulhi(x, magic_r), r = r0 + rr;
      const uint32_t du = fast_div(r, unit, magic_u);
      const uint32_t e = tab[du];
      const UnitSrc sr = src[e >> kUnitBits];
      const uint32_t srow = (e & ((1u << kUnitBits) - 1u)) * unit + (r - du * unit);
      p[u] = sr.base && k < n16 ? uint64_t(reinterpret_cast<uintptr_t>(sr.base)) + (uint64_t(srow) * sr.stride + (x - rr * R)) : 0;
      if (p[u]) v[u] = __builtin_nontemporal_load(global_ptr<u32x4>(p[u]));
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (p[u]) __builtin_nontemporal_store(v[u], d + base + u * kThreads);
  }
}

struct Extent {
  uintptr_t lo, hi;
};

int64_t gather_block_bytes(const ntp_handle* h) {
  if (const int64_t e = h->opt[NTP_OPT_RESHARD_BLOCK]) return std::max<int64_t>(1024, e);
  return kBlockBytes;
}

// Plain dense copy of 16-byte words: the yardstick that profiler byte counters are scaled by.
__global__ __launch_bounds__(256) void calibration_copy_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst,
                                                               int64_t words) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < words; i += stride) dst[i] = src[i];
}

}  // namespace

extern "C" int ntp_calibration_copy(ntp_handle_t* h, void* dst, const void* src, int64_t bytes, void* stream) {
  if (!h || !dst || !src || bytes < 0) return NTP_ERR_INVALID_ARG;
  if (h->device < 0) return NTP_ERR_NO_DEVICE;
  if (bytes % 16 || reinterpret_cast<uintptr_t>(dst) % 16 || reinterpret_cast<uintptr_t>(src) % 16) return NTP_ERR_ALIGNMENT;
  if (bytes == 0) return NTP_OK;
  const int64_t words = bytes / 16;
  const uint32_t blocks = uint32_t(std::min<int64_t>((words + 255) / 256, int64_t(h->compute_units) * 32));
  if (ntp::timing_on(h)) ntp::timing_begin(h, stream, "calibration_copy", 0.0, 2.0 * double(bytes));
  hipLaunchKernelGGL(calibration_copy_kernel, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<const u32x4*>(src), static_cast<u32x4*>(dst), words);
  const bool ok = hipGetLastError() == hipSuccess;
  ntp::timing_end(h, stream);
  return ok ? NTP_OK : NTP_ERR_LAUNCH;
}

// ---- sum of replicated units over their holders --------------------------------------------------
namespace {

constexpr int kMaxHolders = 96;  // ranks that may hold one unit (kernel argument space)

// One replicated unit: a [rows x cols] fp32 block in each of n holders' shards.
struct ReplicaGroup {
  float* ptr[kMaxHolders];
  int64_t ld[kMaxHolders];
  int32_t n, rows, cols, vec4;  // vec4: every pointer is 16-byte aligned, cols % 4 == 0, every ld % 4 == 0
};

// Every element: the holders' values added in ascending rank order (a fixed order, so the result is
// deterministic), then written back to all of them.  One thread owns an element (or four) in every holder, so
// the update in place is safe.
__global__ __launch_bounds__(256) void replica_sum_kernel(const ReplicaGroup g) {
  const int64_t per_row = g.vec4 ? g.cols / 4 : g.cols;
  const int64_t total = int64_t(g.rows) * per_row, stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += stride) {
    const int64_t r = i / per_row, c = i - r * per_row;
    if (g.vec4) {
      typedef float f4 __attribute__((ext_vector_type(4)));
      f4 sum = *reinterpret_cast<const f4*>(g.ptr[0] + r * g.ld[0] + c * 4);
      for (int k = 1; k < g.n; ++k) sum = sum + *reinterpret_cast<const f4*>(g.ptr[k] + r * g.ld[k] + c * 4);
      for (int k = 0; k < g.n; ++k) *reinterpret_cast<f4*>(g.ptr[k] + r * g.ld[k] + c * 4) = sum;
    } else {
      float sum = g.ptr[0][r * g.ld[0] + c];
      for (int k = 1; k < g.n; ++k) sum += g.ptr[k][r * g.ld[k] + c];
      for (int k = 0; k < g.n; ++k) g.ptr[k][r * g.ld[k] + c] = sum;
    }
  }
}

}  // namespace

extern "C" int ntp_replica_sum(ntp_handle_t* h, const ntp_tensor_spec_t* spec, int32_t tp, void* const* shards,
                               const int64_t* ld, void* stream) {
  if (!h || !shards || !ld) return NTP_ERR_INVALID_ARG;
  int64_t n_units = 0;
  int st = ntp::check_spec(spec, tp, tp, &n_units);
  if (st != NTP_OK) return st;
  if (spec->elem_size != 4) return NTP_ERR_INVALID_ARG;  // the sum is fp32 arithmetic
  if (spec->kind == NTP_KIND_PLAIN) return NTP_OK;       // every unit has one holder
  // shape and alignment of the shards, and: no two shards may overlap
  std::vector<int64_t> units(tp), none;
  for (int32_t r = 0; r < tp; ++r)
    if ((st = ntp::shard_units(spec, n_units, tp, r, &units[r])) != NTP_OK) return st;
  std::vector<void*> no_dst;
  {
    std::vector<Extent> ext(tp, Extent{0, 0});
    const bool by_rows = spec->partition_dim == 0;
    for (int32_t r = 0; r < tp; ++r) {
      if (!shards[r] || units[r] == 0) continue;
      const int64_t srows = by_rows ? units[r] * spec->unit : spec->rows, scols = by_rows ? spec->cols : units[r] * spec->unit;
      if (srows == 0 || scols == 0) continue;
      if (ld[r] < scols) return NTP_ERR_INVALID_ARG;
      const uintptr_t p = reinterpret_cast<uintptr_t>(shards[r]);
      if (p % 4) return NTP_ERR_ALIGNMENT;
      ext[r] = Extent{p, p + uintptr_t(((srows - 1) * ld[r] + scols) * 4)};
    }
    for (int32_t a = 0; a < tp; ++a)
      for (int32_t b = a + 1; b < tp; ++b)
        if (ext[a].hi > ext[a].lo && ext[b].hi > ext[b].lo && ext[a].lo < ext[b].hi && ext[b].lo < ext[a].hi) return NTP_ERR_INVALID_ARG;
  }
  if (h->device < 0) return NTP_ERR_NO_DEVICE;
  // holders of every logical unit, ascending rank order
  std::vector<std::vector<std::pair<int32_t, int64_t>>> holders(static_cast<size_t>(n_units));
  std::vector<ntp::Run> runs;
  for (int32_t r = 0; r < tp; ++r) {
    if ((st = ntp::rank_runs(spec, n_units, tp, r, &runs)) != NTP_OK) return st;
    for (const ntp::Run& run : runs)
      for (int64_t i = 0; i < run.count; ++i) holders[size_t(run.first + i)].push_back({r, run.local + i});
  }
  hipStream_t hs = static_cast<hipStream_t>(stream);
  const bool by_rows = spec->partition_dim == 0;
  for (int64_t u = 0; u < n_units; ++u) {
    const auto& hd = holders[size_t(u)];
    if (hd.size() < 2) continue;
    if (hd.size() > size_t(kMaxHolders)) return NTP_ERR_UNSUPPORTED;
    ReplicaGroup g{};
    g.rows = int32_t(by_rows ? spec->unit : spec->rows);
    g.cols = int32_t(by_rows ? spec->cols : spec->unit);
    if ((by_rows ? spec->cols : spec->rows) > 0x7fffffffll) return NTP_ERR_UNSUPPORTED;
    g.vec4 = g.cols % 4 == 0;
    for (const auto& [r, local] : hd) {
      if (!shards[r]) continue;  // a holder that is not on this GPU takes no part
      float* base = static_cast<float*>(shards[r]);
      g.ptr[g.n] = by_rows ? base + local * spec->unit * ld[r] : base + local * spec->unit;
      g.ld[g.n] = ld[r];
      if ((reinterpret_cast<uintptr_t>(g.ptr[g.n]) & 15) || ld[r] % 4) g.vec4 = 0;
      ++g.n;
    }
    if (g.n < 2 || g.rows == 0 || g.cols == 0) continue;
    const int64_t work = int64_t(g.rows) * (g.vec4 ? g.cols / 4 : g.cols);
    const uint32_t blocks = uint32_t(std::max<int64_t>(1, std::min<int64_t>((work + 255) / 256, int64_t(h->compute_units) * 16)));
    if (ntp::timing_on(h)) ntp::timing_begin(h, stream, "replica_sum", 0.0, 2.0 * 4.0 * double(g.n) * double(g.rows) * double(g.cols));
    hipLaunchKernelGGL(replica_sum_kernel, dim3(blocks), dim3(256), 0, hs, g);
    const bool ok = hipGetLastError() == hipSuccess;
    ntp::timing_end(h, stream);
    if (!ok) return NTP_ERR_LAUNCH;
  }
  return NTP_OK;
}

extern "C" int ntp_reshard_grad(ntp_handle_t* h, const ntp_tensor_spec_t* spec, int32_t src_tp, int32_t dst_tp,
                                const void* const* src_shards, const int64_t* src_ld,
                                void* const* dst_shards, const int64_t* dst_ld, void* stream) {
  if (!h || !src_shards || !dst_shards || !src_ld || !dst_ld) return NTP_ERR_INVALID_ARG;
  std::vector<ntp_segment_t> segs;
  int st = ntp::build_segments(spec, src_tp, dst_tp, &segs);
  if (st != NTP_OK) return st;
  int64_t n_units = 0;
  ntp::check_spec(spec, src_tp, dst_tp, &n_units);
  std::vector<int64_t> su(src_tp), du(dst_tp);
  for (int32_t r = 0; r < src_tp; ++r)
    if ((st = ntp::shard_units(spec, n_units, src_tp, r, &su[r])) != NTP_OK) return st;
  for (int32_t r = 0; r < dst_tp; ++r)
    if ((st = ntp::shard_units(spec, n_units, dst_tp, r, &du[r])) != NTP_OK) return st;
  return ntp::reshard_launch(h, spec, segs, su, du, src_shards, src_ld, dst_shards, dst_ld, stream);
}

int ntp::check_shards(const ntp_tensor_spec_t* spec, const std::vector<int64_t>& src_units,
                      const std::vector<int64_t>& dst_units, const void* const* src_shards, const int64_t* src_ld,
                      void* const* dst_shards, const int64_t* dst_ld) {
  if (!src_shards || !dst_shards || !src_ld || !dst_ld) return NTP_ERR_INVALID_ARG;
  const int64_t esz = spec->elem_size;
  const bool by_rows = spec->partition_dim == 0;
  auto extents = [&](const std::vector<int64_t>& nunits, const void* const* ptrs, const int64_t* ld,
                     std::vector<Extent>* out) -> int {
    const int32_t tp = int32_t(nunits.size());
    out->assign(tp, Extent{0, 0});
    for (int32_t r = 0; r < tp; ++r) {
      const int64_t units = nunits[r];
      if (!ptrs[r] || units == 0) continue;
      const int64_t srows = by_rows ? units * spec->unit : spec->rows;
      const int64_t scols = by_rows ? spec->cols : units * spec->unit;
      if (srows == 0 || scols == 0) continue;
      if (ld[r] < scols) return NTP_ERR_INVALID_ARG;
      const uintptr_t p = reinterpret_cast<uintptr_t>(ptrs[r]);
      if (p % esz != 0) return NTP_ERR_ALIGNMENT;
      (*out)[r] = Extent{p, p + uintptr_t(((srows - 1) * ld[r] + scols) * esz)};
    }
    return NTP_OK;
  };
  std::vector<Extent> se, de;
  int st;
  if ((st = extents(src_units, src_shards, src_ld, &se)) != NTP_OK) return st;
  if ((st = extents(dst_units, reinterpret_cast<const void* const*>(dst_shards), dst_ld, &de)) != NTP_OK) return st;
  for (const Extent& a : se)
    for (const Extent& b : de)
      if (a.hi > a.lo && b.hi > b.lo && a.lo < b.hi && b.lo < a.hi) return NTP_ERR_INVALID_ARG;
  return NTP_OK;
}

int ntp::reshard_launch(ntp_handle* h, const ntp_tensor_spec_t* spec, const std::vector<ntp_segment_t>& segs,
                        const std::vector<int64_t>& src_units, const std::vector<int64_t>& dst_units,
                        const void* const* src_shards, const int64_t* src_ld, void* const* dst_shards,
                        const int64_t* dst_ld, void* stream) {
  const int st = check_shards(spec, src_units, dst_units, src_shards, src_ld, dst_shards, dst_ld);
  if (st != NTP_OK) return st;
  if (h->device < 0) return NTP_ERR_NO_DEVICE;
  const int64_t esz = spec->elem_size;
  const bool by_rows = spec->partition_dim == 0;

  hipStream_t hs = static_cast<hipStream_t>(stream);

  std::vector<CopySeg> copies;
  std::vector<DenseRange> ranges;
  if (!by_rows) {
    // destination-major gather: consecutive sub-shards of one destination shard form a job
    std::vector<GatherJob> jobs;
    int32_t cur_dst = -1;
    int64_t cur_end = 0;  // destination column (bytes) where the current job ends
    int64_t job_col0 = 0;
    for (const ntp_segment_t& g : segs) {
      const char* sp = static_cast<const char*>(src_shards[g.src_rank]);
      char* dp = static_cast<char*>(dst_shards[g.dst_rank]);
      const int64_t c0 = g.dst_unit * spec->unit * esz, c1 = c0 + g.units * spec->unit * esz;
      if (!sp || !dp || c1 == c0 || spec->rows == 0) continue;  // not on this GPU, or empty
      if (spec->rows > 0xffffffffll || c1 - c0 > 0x7fffffffll) {
        if (esz == 4) return NTP_ERR_UNSUPPORTED;
        const int64_t sld = src_ld[g.src_rank] * esz, dld = dst_ld[g.dst_rank] * esz;
        copies.push_back(CopySeg{sp + g.src_unit * spec->unit * esz, dp + c0, sld, dld, c1 - c0, spec->rows, 0, 0, 0, 0});
        continue;
      }
      const bool fresh = jobs.empty() || g.dst_rank != cur_dst || c0 != cur_end || jobs.back().npieces == kMaxPieces ||
                         c1 - job_col0 > 0x7fffffffll;
      if (fresh) {
        GatherJob j{};
        j.dst = dp + c0;
        j.dst_stride = dst_ld[g.dst_rank] * esz;
        j.rows = uint32_t(spec->rows);
        jobs.push_back(j);
        cur_dst = g.dst_rank;
        job_col0 = c0;
      }
      GatherJob& j = jobs.back();
      Piece& pc = j.piece[j.npieces++];
      pc.src = sp + g.src_unit * spec->unit * esz;
      pc.src_stride = src_ld[g.src_rank] * esz;
      pc.begin = uint32_t(c0 - job_col0);
      pc.end = uint32_t(c1 - job_col0);
      cur_end = c1;
    }
    // jobs whose destination is a dense, 64-byte aligned shard go to the flat kernel
    const int64_t kFlatBlock = h->opt[NTP_OPT_RESHARD_FLAT_BLOCK]
                                   ? std::min<int64_t>(kFlatBlockMax, std::max<int64_t>(1024, h->opt[NTP_OPT_RESHARD_FLAT_BLOCK] & ~63ll))
                                   : 16384;
    std::vector<GatherJob> flat, rowwise;
    for (const GatherJob& j : jobs) (flat_ok(j, kFlatBlock, esz) && !h->opt[NTP_OPT_RESHARD_NO_FLAT] ? flat : rowwise).push_back(j);
    for (size_t base = 0; base < flat.size(); base += kMaxJobs) {
      GatherBatch batch{};
      batch.njobs = int32_t(std::min<size_t>(kMaxJobs, flat.size() - base));
      int64_t nblk = 0;
      double bytes = 0.0;
      for (int i = 0; i < batch.njobs; ++i) {
        const GatherJob& j = flat[base + i];
        const int64_t total = int64_t(j.rows) * j.piece[j.npieces - 1].end;
        nblk = std::max(nblk, (total + kFlatBlock - 1) / kFlatBlock);
        bytes += 2.0 * double(total);
        batch.job[i] = j;
      }
      batch.rows_per_block = uint32_t(kFlatBlock);
      const uint64_t blocks = uint64_t(nblk) * uint64_t(batch.njobs);
      if (blocks > 0x7fffffffull) return NTP_ERR_UNSUPPORTED;
      if (blocks == 0) continue;
      if (ntp::timing_on(h)) ntp::timing_begin(h, stream, "reshard_flat", 0.0, bytes);
      hipLaunchKernelGGL(esz == 4 ? reshard_flat_kernel : reshard_flat2_kernel, dim3(uint32_t(blocks)), dim3(kThreads), 0, hs, batch);
      const bool ok = hipGetLastError() == hipSuccess;
      ntp::timing_end(h, stream);
      if (!ok) return NTP_ERR_LAUNCH;
    }
    jobs.swap(rowwise);
    if (esz != 4) {  // the row-wise kernel moves words: what is left of 2-byte elements is copied piece by piece
      for (const GatherJob& j : jobs)
        for (uint32_t p = 0; p < j.npieces; ++p) {
          const Piece& pc = j.piece[p];
          copies.push_back(CopySeg{pc.src, j.dst + pc.begin, pc.src_stride, j.dst_stride, int64_t(pc.end - pc.begin), int64_t(j.rows), 0, 0, 0, 0});
        }
      jobs.clear();
    }
    for (size_t base = 0; base < jobs.size(); base += kMaxJobs) {
      GatherBatch batch{};
      batch.njobs = int32_t(std::min<size_t>(kMaxJobs, jobs.size() - base));
      // rows per workgroup: about kBlockBytes of the widest job, and row offsets inside a block that
      // fit in 32 bits
      int64_t rpb = spec->rows;
      double bytes = 0.0;
      for (int i = 0; i < batch.njobs; ++i) {
        const GatherJob& j = jobs[base + i];
        const int64_t row_bytes = j.piece[j.npieces - 1].end;
        int64_t stride = j.dst_stride;
        for (uint32_t p = 0; p < j.npieces; ++p) stride = std::max(stride, j.piece[p].src_stride);
        rpb = std::min(rpb, std::max<int64_t>(1, gather_block_bytes(h) / row_bytes));
        rpb = std::min(rpb, std::max<int64_t>(1, (int64_t(1) << 31) / std::max<int64_t>(stride, 1)));
        bytes += 2.0 * double(j.rows) * double(row_bytes);
        batch.job[i] = j;
      }
      if (rpb > 1 && jobs[base].dst_stride > (int64_t(1) << 31)) return NTP_ERR_UNSUPPORTED;
      batch.rows_per_block = uint32_t(rpb);
      const uint64_t blocks = uint64_t((spec->rows + rpb - 1) / rpb) * uint64_t(batch.njobs);
      if (blocks > 0x7fffffffull) return NTP_ERR_UNSUPPORTED;
      if (blocks == 0) continue;
      if (ntp::timing_on(h)) ntp::timing_begin(h, stream, "reshard_gather", 0.0, bytes);
      hipLaunchKernelGGL(reshard_gather_kernel, dim3(uint32_t(blocks)), dim3(kThreads), 0, hs, batch);
      const bool ok = hipGetLastError() == hipSuccess;
      ntp::timing_end(h, stream);
      if (!ok) return NTP_ERR_LAUNCH;
    }
  }

  // row-partitioned: segments -> dense ranges and 2-D copies
  for (const ntp_segment_t& g : segs) {
    if (!by_rows) break;
    const char* sp = static_cast<const char*>(src_shards[g.src_rank]);
    char* dp = static_cast<char*>(dst_shards[g.dst_rank]);
    if (!sp || !dp) continue;  // not on this GPU
    const int64_t sld = src_ld[g.src_rank] * esz, dld = dst_ld[g.dst_rank] * esz;
    CopySeg c{};
    c.src = sp + g.src_unit * spec->unit * sld;
    c.dst = dp + g.dst_unit * spec->unit * dld;
    c.rows = g.units * spec->unit;
    c.row_bytes = spec->cols * esz;
    c.src_stride = sld;
    c.dst_stride = dld;
    if (c.rows == 0 || c.row_bytes == 0) continue;
    if (c.src_stride == c.row_bytes && c.dst_stride == c.row_bytes) {
      // dense on both sides: one long run.  The 16-byte aligned middle goes to the streaming kernel,
      // what is left (misaligned pointers, a few bytes at the end) to the general one.
      const int64_t total = c.rows * c.row_bytes;
      const bool al = ((reinterpret_cast<uintptr_t>(c.src) | reinterpret_cast<uintptr_t>(c.dst)) & 15) == 0;
      const int64_t body = al ? total & ~int64_t(15) : 0;
      if (body > 0) ranges.push_back(DenseRange{c.src, c.dst, body, 0, 0});
      if (total > body) {
        CopySeg d = c;
        d.src += body;
        d.dst += body;
        d.rows = 1;
        d.row_bytes = d.src_stride = d.dst_stride = total - body;
        if (d.row_bytes > (int64_t(1) << 20)) {  // long misaligned run: recut into 4 KiB rows
          const int64_t full = d.row_bytes / 4096;
          CopySeg e = d;
          e.rows = full;
          e.row_bytes = e.src_stride = e.dst_stride = 4096;
          copies.push_back(e);
          d.src += full * 4096;
          d.dst += full * 4096;
          d.row_bytes = d.src_stride = d.dst_stride = d.row_bytes - full * 4096;
        }
        if (d.row_bytes > 0) copies.push_back(d);
      }
    } else {
      copies.push_back(c);
    }
  }

  for (size_t base = 0; base < ranges.size(); base += kMaxRanges) {
    DenseBatch batch{};
    batch.n = int32_t(std::min<size_t>(kMaxRanges, ranges.size() - base));
    uint64_t blocks = 0;
    double bytes = 0.0;
    for (int i = 0; i < batch.n; ++i) {
      DenseRange r = ranges[base + i];
      r.first_block = uint32_t(blocks);
      blocks += uint64_t((r.bytes + kDenseBlock - 1) / kDenseBlock);
      if (blocks > 0x7fffffffull) return NTP_ERR_UNSUPPORTED;
      bytes += 2.0 * double(r.bytes);
      batch.r[i] = r;
    }
    if (ntp::timing_on(h)) ntp::timing_begin(h, stream, "reshard_dense", 0.0, bytes);
    hipLaunchKernelGGL(reshard_dense_kernel, dim3(uint32_t(blocks)), dim3(kThreads), 0, hs, batch);
    const bool ok = hipGetLastError() == hipSuccess;
    ntp::timing_end(h, stream);
    if (!ok) return NTP_ERR_LAUNCH;
  }
  for (size_t base = 0; base < copies.size(); base += kMaxSegs) {
    CopyBatch batch{};
    batch.nseg = int32_t(std::min<size_t>(kMaxSegs, copies.size() - base));
    batch.elem_size = int32_t(esz);
    uint64_t blocks = 0;
    for (int i = 0; i < batch.nseg; ++i) {
      CopySeg c = copies[base + i];
      c.col_chunks = uint32_t((c.row_bytes + kColChunk - 1) / kColChunk);
      const int64_t per_row = std::min<int64_t>(c.row_bytes, kColChunk);
      // about kBlockBytes per workgroup; rows * elements-per-row stays far below 2^32 (exact multiply-high division)
      int64_t rpb = std::max<int64_t>(1, std::min<int64_t>(kBlockBytes / per_row, 16384));
      c.rows_per_block = uint32_t(std::min<int64_t>(rpb, std::max<int64_t>(c.rows, 1)));
      const uint64_t row_groups = uint64_t((c.rows + c.rows_per_block - 1) / c.rows_per_block);
      c.first_block = uint32_t(blocks);
      blocks += row_groups * c.col_chunks;
      if (blocks > 0x7fffffffull) return NTP_ERR_UNSUPPORTED;
      batch.seg[i] = c;
    }
    if (blocks == 0) continue;
    if (ntp::timing_on(h)) {
      double bytes = 0.0;
      for (int i = 0; i < batch.nseg; ++i) bytes += 2.0 * double(batch.seg[i].rows) * double(batch.seg[i].row_bytes);
      ntp::timing_begin(h, stream, "reshard_copy", 0.0, bytes);
    }
    hipLaunchKernelGGL(reshard_copy_kernel, dim3(uint32_t(blocks)), dim3(kThreads), 0, hs, batch);
    const bool ok = hipGetLastError() == hipSuccess;
    ntp::timing_end(h, stream);
    if (!ok) return NTP_ERR_LAUNCH;
  }
  return NTP_OK;
}

// ---- reshard plan between two unit -> rank maps (Sec. 3.1, Alg. 1; Appendix: precomputed splits) -----
struct ntp_reshard_plan {
  ntp_tensor_spec_t spec;
  int32_t src_tp, dst_tp;
  std::vector<ntp_segment_t> segs;           // destination order
  std::vector<int64_t> src_units, dst_units;  // units per rank
  std::vector<int64_t> splits;                // [src_tp x dst_tp] units from rank r to rank s
  std::vector<ntp_unit_source_t> table;       // per destination unit, destination shards one after the other
  std::vector<int64_t> dst_first;             // first table entry of each destination shard
  std::vector<uint32_t> unit_src;             // `table` as the table kernels read it (empty: they cannot take this plan)
  bool large = false;                         // column-partitioned, kRunTensorMin bytes and more
  bool interleaved = false;                   // column-partitioned, neighbouring source units often go to different shards
  // instead of `unit_src` where the run-table kernel takes the plan (run_table_wanted)
  std::vector<RunDev> runs;                   // runs of all destination shards, one shard after the other
  std::vector<int64_t> runs_first;            // first run of each destination shard
  std::vector<uint16_t> run_of_unit;          // per destination unit (indexed like `table`): run number in its shard
  void* dev_table = nullptr;                  // `unit_src`, or `runs` then `run_of_unit`, on device `dev`, made by ntp_reshard_plan_prepare
  int dev = -1;                               // device the plan was prepared on (-1: not prepared)
};

namespace {

// Whether a column-partitioned plan of 4-byte elements goes through the run table (see reshard_runs_kernel).
bool run_table_wanted(const ntp_reshard_plan* p) {
  const ntp_tensor_spec_t& sp = p->spec;
  const int64_t widest = *std::max_element(p->dst_units.begin(), p->dst_units.end()) * sp.unit * 4;
  return p->large && !p->interleaved && widest <= kRunRowMax;
}

void build_run_table(ntp_reshard_plan* p) {
  const uint32_t ub = uint32_t(p->spec.unit) * 4u;
  p->runs_first.assign(size_t(p->dst_tp) + 1, 0);
  p->run_of_unit.resize(p->table.size());
  int32_t cur = 0;
  for (const ntp_segment_t& g : p->segs) {
    while (cur < g.dst_rank) p->runs_first[size_t(++cur)] = int64_t(p->runs.size());
    const uint16_t number = uint16_t(int64_t(p->runs.size()) - p->runs_first[size_t(cur)]);
    p->runs.push_back(RunDev{uint32_t(g.dst_unit) * ub, uint32_t(g.dst_unit + g.units) * ub, uint32_t(g.src_unit) * ub, uint32_t(g.src_rank)});
    std::fill_n(p->run_of_unit.begin() + p->dst_first[size_t(g.dst_rank)] + g.dst_unit, g.units, number);
  }
  while (cur < p->dst_tp) p->runs_first[size_t(++cur)] = int64_t(p->runs.size());
}

}  // namespace

extern "C" int ntp_reshard_plan_create(const ntp_tensor_spec_t* spec, int64_t map_len, int32_t src_tp,
                                       const int32_t* src_rank_of_unit, int32_t dst_tp,
                                       const int32_t* dst_rank_of_unit, ntp_reshard_plan_t** plan) {
  if (!plan) return NTP_ERR_INVALID_ARG;
  *plan = nullptr;
  int64_t n_units = 0;
  int st = ntp::check_spec(spec, 1, 1, &n_units);
  if (st != NTP_OK) return st;
  if (spec->kind != NTP_KIND_PLAIN || n_units > 0x7fffffffll || map_len != n_units) return NTP_ERR_INVALID_ARG;
  ntp_reshard_plan* p = new ntp_reshard_plan;
  p->spec = *spec;
  p->src_tp = src_tp;
  p->dst_tp = dst_tp;
  st = ntp::build_segments_mapped(n_units, src_tp, src_rank_of_unit, dst_tp, dst_rank_of_unit, &p->segs, &p->src_units,
                                  &p->dst_units);
  if (st != NTP_OK) {
    delete p;
    return st;
  }
  p->splits.assign(size_t(src_tp) * size_t(dst_tp), 0);
  p->dst_first.assign(size_t(dst_tp) + 1, 0);
  for (int32_t s = 0; s < dst_tp; ++s) p->dst_first[s + 1] = p->dst_first[s] + p->dst_units[s];
  p->table.resize(size_t(n_units));
  for (const ntp_segment_t& g : p->segs) {
    p->splits[size_t(g.src_rank) * dst_tp + g.dst_rank] += g.units;
    for (int64_t i = 0; i < g.units; ++i)
      p->table[size_t(p->dst_first[g.dst_rank] + g.dst_unit + i)] = ntp_unit_source_t{g.src_rank, int32_t(g.src_unit + i)};
  }
  if (spec->partition_dim == 1 && n_units > 0) {
    // how many times a 128-byte line of a source row changes its destination shard.  More than once: bands; in tensors below 256 MiB from
    // once in four on (3200 x 12800 from 40 to 33 ranks 156 us whole, 144 in bands; 16384 x 65536 from 71 to 55 1950 and 2053, 15104 x
    // 60416 from 64 to 52 1653 and 1776)
    std::vector<int32_t> dst_of(size_t(n_units), 0);
    std::vector<int64_t> first(size_t(src_tp) + 1, 0);
    for (int32_t r = 0; r < src_tp; ++r) first[size_t(r) + 1] = first[size_t(r)] + p->src_units[size_t(r)];
    for (const ntp_segment_t& g : p->segs)
      std::fill_n(dst_of.begin() + first[size_t(g.src_rank)] + g.src_unit, g.units, g.dst_rank);
    int64_t turns = 0;
    for (int64_t u = 1; u < n_units; ++u) turns += dst_of[size_t(u)] != dst_of[size_t(u) - 1];
    const int64_t row_bytes = n_units * spec->unit * spec->elem_size;
    p->large = spec->rows >= (kRunTensorMin + row_bytes - 1) / row_bytes;
    p->interleaved = turns * 128 * (p->large ? 1 : 4) > row_bytes;
  }
  if (n_units > 0 && n_units <= (int64_t(1) << kUnitBits) && src_tp <= kMaxRanks && (spec->partition_dim == 0 || spec->elem_size == 4)) {
    if (spec->partition_dim == 1 && run_table_wanted(p)) {
      build_run_table(p);
      *plan = p;
      return NTP_OK;
    }
    p->unit_src.assign(size_t(n_units) + 3, 0);  // a chunk's four entries are read with one load
    for (int64_t u = 0; u < n_units; ++u)
      p->unit_src[size_t(u)] = uint32_t(p->table[size_t(u)].src_rank) << kUnitBits | uint32_t(p->table[size_t(u)].src_unit);
  }
  *plan = p;
  return NTP_OK;
}

extern "C" int ntp_reshard_plan_destroy(ntp_reshard_plan_t* plan) {
  if (!plan) return NTP_OK;
  if (plan->dev_table) {
    int cur = -1;
    (void)hipGetDevice(&cur);
    if (cur != plan->dev) (void)hipSetDevice(plan->dev);
    (void)hipFree(plan->dev_table);
    if (cur != plan->dev && cur >= 0) (void)hipSetDevice(cur);
  }
  delete plan;
  return NTP_OK;
}

extern "C" int ntp_reshard_plan_segments(const ntp_reshard_plan_t* plan, ntp_segment_t* out, int64_t max_segments,
                                         int64_t* count) {
  if (!plan || !count || max_segments < 0 || (max_segments > 0 && !out)) return NTP_ERR_INVALID_ARG;
  *count = int64_t(plan->segs.size());
  for (int64_t i = 0; i < std::min<int64_t>(max_segments, *count); ++i) out[i] = plan->segs[size_t(i)];
  return NTP_OK;
}

extern "C" int ntp_reshard_plan_splits(const ntp_reshard_plan_t* plan, int64_t* units) {
  if (!plan || !units) return NTP_ERR_INVALID_ARG;
  std::copy(plan->splits.begin(), plan->splits.end(), units);
  return NTP_OK;
}

extern "C" int ntp_reshard_plan_table(const ntp_reshard_plan_t* plan, ntp_unit_source_t* out, int64_t max_units,
                                      int64_t* count) {
  if (!plan || !count || max_units < 0 || (max_units > 0 && !out)) return NTP_ERR_INVALID_ARG;
  *count = int64_t(plan->table.size());
  for (int64_t i = 0; i < std::min<int64_t>(max_units, *count); ++i) out[i] = plan->table[size_t(i)];
  return NTP_OK;
}

namespace {

// Whether the table kernels can take this call with blocks of `block` bytes: dense aligned destinations, and divisions that
// are exact (n / d by multiply-high needs n * d <= 2^32).
bool table_path_ok(const ntp_handle* h, const ntp_reshard_plan* p, const void* const* src_shards, const int64_t* src_ld,
                   void* const* dst_shards, const int64_t* dst_ld, int64_t block) {
  const ntp_tensor_spec_t& sp = p->spec;
  if (!p->dev_table || h->opt[NTP_OPT_RESHARD_NO_TABLE]) return false;
  constexpr int64_t kMax = int64_t(1) << 32;
  const int64_t esz = sp.elem_size;
  const bool by_rows = sp.partition_dim == 0;
  if (sp.rows == 0 || sp.cols == 0 || sp.rows > 0x7fffffffll || sp.cols * esz > 0x7fffffffll) return false;
  if (by_rows) {
    const int64_t R = sp.cols * esz;
    if (R % 16 || (R <= block && (block + R) * R > kMax) || (int64_t(sp.unit) + block / 16 + 2) * sp.unit > kMax) return false;
  }
  for (int32_t r = 0; r < p->src_tp; ++r) {
    if (p->src_units[r] == 0) continue;
    if (src_ld[r] * esz >= kMax) return false;
    if (by_rows ? (reinterpret_cast<uintptr_t>(src_shards[r]) | uintptr_t(src_ld[r] * esz)) & 15 : !src_shards[r]) return false;
  }
  bool any = false;
  for (int32_t s = 0; s < p->dst_tp; ++s) {
    if (p->dst_units[s] == 0 || !dst_shards[s]) continue;
    const int64_t W = by_rows ? sp.cols * esz : p->dst_units[s] * sp.unit * esz;
    if (dst_ld[s] * esz != W || reinterpret_cast<uintptr_t>(dst_shards[s]) & (by_rows ? 15 : 63)) return false;
    if (!by_rows && ((W <= block + 16 && (block + W + 16) * W > kMax) || (W + 16) * sp.unit * esz > kMax)) return false;
    any = true;
  }
  return any;
}

// The plan's table goes to the current device (allocates and waits for the copy).
int upload_table(ntp_reshard_plan_t* plan) {
  const size_t runs_bytes = plan->runs.size() * sizeof(RunDev), idx_bytes = plan->run_of_unit.size() * sizeof(uint16_t);
  const size_t units_bytes = plan->unit_src.size() * sizeof(uint32_t);
  if (hipMalloc(&plan->dev_table, runs_bytes + idx_bytes + units_bytes) != hipSuccess) {
    plan->dev_table = nullptr;
    return NTP_ERR_LAUNCH;
  }
  char* const at = static_cast<char*>(plan->dev_table);
  auto put = [](char* to, const void* from, size_t n) { return n == 0 || hipMemcpy(to, from, n, hipMemcpyHostToDevice) == hipSuccess; };
  if (!put(at, plan->runs.data(), runs_bytes) || !put(at + runs_bytes, plan->run_of_unit.data(), idx_bytes) ||
      !put(at, plan->unit_src.data(), units_bytes)) {  // (a plan has one of the two tables)
    (void)hipFree(plan->dev_table);
    plan->dev_table = nullptr;
    return NTP_ERR_LAUNCH;
  }
  return NTP_OK;
}

// The launches of a checked call whose plan has a run table.
int run_by_runs(ntp_handle* h, const ntp_reshard_plan* plan, const void* const* src_shards, const int64_t* src_ld, void* const* dst_shards,
                int64_t block, void* stream) {
  const ntp_tensor_spec_t& sp = plan->spec;
  RunBatch batch{};
  batch.runs = static_cast<const RunDev*>(plan->dev_table);
  batch.run_of_unit = reinterpret_cast<const uint16_t*>(static_cast<const char*>(plan->dev_table) + plan->runs.size() * sizeof(RunDev));
  batch.rows = uint32_t(sp.rows);
  batch.unit_bytes = uint32_t(sp.unit) * 4u;
  batch.block_bytes = uint32_t(block);
  for (int32_t r = 0; r < plan->src_tp; ++r)
    batch.src[r] = UnitSrc{static_cast<const char*>(src_shards[r]), uint64_t(src_ld[r]) * 4u};
  for (int32_t s = 0; s < plan->dst_tp;) {
    batch.ndst = 0;
    int64_t nblk = 0;
    uint32_t lds = 0;
    double bytes = 0.0;
    for (; s < plan->dst_tp && batch.ndst < uint32_t(kRunDsts); ++s) {
      if (plan->dst_units[s] == 0 || !dst_shards[s]) continue;
      const int64_t total = sp.rows * plan->dst_units[s] * sp.unit * 4;
      const uint32_t n_runs = uint32_t(plan->runs_first[s + 1] - plan->runs_first[s]);
      batch.dst[batch.ndst++] = RunDst{static_cast<char*>(dst_shards[s]), uint32_t(plan->dst_first[s]), uint32_t(plan->dst_units[s]),
                                       uint32_t(plan->runs_first[s]), n_runs};
      nblk = std::max(nblk, (total + block - 1) / block);
      lds = std::max(lds, run_lds_bytes(n_runs, uint32_t(plan->dst_units[s])));
      bytes += 2.0 * double(total);
    }
    if (batch.ndst == 0) break;
    // workgroups per destination shard: one per block, or fewer that walk over several blocks each when
    // the shards are very large (the tables are copied into LDS once per workgroup)
    const int64_t slots = std::max<int64_t>(1, std::min<int64_t>(nblk, (int64_t(h->compute_units) * int64_t(kRunBlocksPerCu) + batch.ndst - 1) / batch.ndst));
    if (ntp::timing_on(h)) ntp::timing_begin(h, stream, "reshard_runs", 0.0, bytes);
    hipLaunchKernelGGL(reshard_runs_kernel, dim3(uint32_t(slots) * batch.ndst), dim3(kThreads), lds, static_cast<hipStream_t>(stream), batch);
    const bool ok = hipGetLastError() == hipSuccess;
    ntp::timing_end(h, stream);
    if (!ok) return NTP_ERR_LAUNCH;
  }
  return NTP_OK;
}

}  // namespace

extern "C" int ntp_reshard_plan_prepare(ntp_reshard_plan_t* plan) {
  if (!plan) return NTP_ERR_INVALID_ARG;
  int cur = -1;
  if (hipGetDevice(&cur) != hipSuccess || cur < 0) {
    (void)hipGetLastError();
    return NTP_ERR_NO_DEVICE;
  }
  if (plan->dev >= 0) return cur == plan->dev ? NTP_OK : NTP_ERR_INVALID_ARG;  // a plan lives on one device
  if (!plan->unit_src.empty() || !plan->runs.empty()) {
    const int st = upload_table(plan);
    if (st != NTP_OK) return st;
  }
  plan->dev = cur;
  return NTP_OK;
}

extern "C" int ntp_reshard_plan_run(ntp_handle_t* h, ntp_reshard_plan_t* plan, const void* const* src_shards,
                                    const int64_t* src_ld, void* const* dst_shards, const int64_t* dst_ld, void* stream) {
  if (!h || !plan) return NTP_ERR_INVALID_ARG;
  int st = ntp::check_shards(&plan->spec, plan->src_units, plan->dst_units, src_shards, src_ld, dst_shards, dst_ld);
  if (st != NTP_OK) return st;
  if (h->device < 0) return NTP_ERR_NO_DEVICE;
  if (plan->dev != h->device) return NTP_ERR_NOT_PREPARED;
  int64_t block = 16384;
  if (const int64_t e = h->opt[NTP_OPT_RESHARD_TABLE_BLOCK]) block = std::min<int64_t>(1 << 20, std::max<int64_t>(1024, e & ~63ll));
  if (!table_path_ok(h, plan, src_shards, src_ld, dst_shards, dst_ld, block))
    return ntp::reshard_launch(h, &plan->spec, plan->segs, plan->src_units, plan->dst_units, src_shards, src_ld, dst_shards,
                               dst_ld, stream);
  if (!plan->runs.empty()) return run_by_runs(h, plan, src_shards, src_ld, dst_shards, block, stream);

  const ntp_tensor_spec_t& sp = plan->spec;
  const bool by_rows = sp.partition_dim == 0;
  TableBatch batch{};
  batch.table = static_cast<const uint32_t*>(plan->dev_table);
  batch.rows = uint32_t(sp.rows);
  batch.row_bytes = uint32_t(sp.cols * sp.elem_size);
  batch.unit = uint32_t(by_rows ? sp.unit : sp.unit * sp.elem_size);
  batch.block_bytes = uint32_t(block);
  batch.nsrc = plan->src_tp;
  for (int32_t r = 0; r < plan->src_tp; ++r)
    batch.src[r] = UnitSrc{static_cast<const char*>(src_shards[r]), uint64_t(src_ld[r]) * uint64_t(sp.elem_size)};
  const int64_t per_unit = int64_t(sp.unit) * (by_rows ? sp.cols : sp.rows) * sp.elem_size;  // bytes
  // columns that are not copied in bands: few write streams at a time (16384 x 53248 from 31 to 32 ranks 880 us in one launch, 854 in two)
  const int32_t per_launch = by_rows || plan->interleaved ? kMaxRanks : kRunDsts;
  for (int32_t s = 0; s < plan->dst_tp;) {
    batch.ndst = 0;
    int64_t total = 0;
    for (; s < plan->dst_tp && batch.ndst < per_launch; ++s) {
      if (plan->dst_units[s] == 0 || !dst_shards[s]) continue;
      batch.dst[batch.ndst++] = TableDst{static_cast<char*>(dst_shards[s]), uint32_t(plan->dst_first[s]), uint32_t(plan->dst_units[s]), 0, 0};
      total += plan->dst_units[s] * per_unit;
    }
    if (batch.ndst == 0) break;
    const int64_t bands = plan->interleaved ? std::max<int64_t>(1, total / kBandBytes) : 1;
    uint64_t blocks = 0;
    for (int32_t i = 0; i < batch.ndst; ++i) {
      TableDst& d = batch.dst[i];
      const int64_t n = (int64_t(d.n_units) * per_unit + block - 1) / block, q = (n + bands - 1) / bands;
      if (uint64_t(q) * uint64_t(bands) > 0x7fffffffull) return NTP_ERR_UNSUPPORTED;
      d.first_block = uint32_t(blocks);
      d.per_band = uint32_t(q);
      blocks += uint64_t(q);
    }
    batch.band_blocks = uint32_t(blocks);
    blocks *= uint64_t(bands);
    if (blocks > 0x7fffffffull) return NTP_ERR_UNSUPPORTED;
    const double bytes = 2.0 * double(total);
    if (ntp::timing_on(h)) ntp::timing_begin(h, stream, "reshard_table", 0.0, bytes);
    const auto kernel = by_rows ? reshard_table_rows_kernel : batch.unit == 4 ? reshard_table_cols_kernel<true> : reshard_table_cols_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3(uint32_t(blocks)), dim3(kThreads), 0, static_cast<hipStream_t>(stream), batch);
    const bool ok = hipGetLastError() == hipSuccess;
    ntp::timing_end(h, stream);
    if (!ok) return NTP_ERR_LAUNCH;
  }
  return NTP_OK;
}
