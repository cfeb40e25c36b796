// Dense fp16 -> MACKO conversion on the GPU (format of Section 4.1, tail
// padding of Section 4.5).  Passes: count the stored entries of every row,
// prefix-sum the counts into row_ptr, write values and packed codes.  The output is
// bit-identical to the host encoder's.
//
// One wavefront works on one row; per step a lane looks at 8 consecutive
// columns (one load, issued ahead).  The position of the
// previous stored entry is carried across lanes and steps, so each lane can price its own non-zeros: a non-zero at
// distance g from the previously stored column costs (g-1) / 2^b_delta padding
// entries plus itself.  Per-row counts go to arrays that the scan kernels total (no atomics).
//
// Roofline: HBM (2 x the dense matrix read, the second time mostly from the last-level cache, and the encoding
// written once); what the passes are short of in practice is vector issue, hence the packed zero test, the table of
// what a mask of 8 columns stores, and padding entries that cost no instruction (see encode_fill_kernel).
#include "macko_device.h"
#include "macko_internal.h"

#include <chrono>
#include <mutex>
#include <new>

namespace macko {
namespace {

struct EncodeStats {
  unsigned long long nnz;
  unsigned long long pad_nnz;
  unsigned int empty_rows;
  unsigned int max_row_entries;
};
// The host's view of an encoding, in pinned memory: the counting pass's totals, and the number of the last encoding that is over.
struct EncodeReport {
  EncodeStats stats;
  uint32_t done;
};

// 8 consecutive columns of one row as loaded: fp16 values, or bytes (8-bit values).
template <bool IN8>
struct Chunk {
  static constexpr int kWords = IN8 ? 2 : 4;
  uint32_t u[kWords];
};

// Loads only; columns at or beyond `cols` read as +0.  The caller looks at the
// result two loop iterations later, so the load is in flight behind the work on
// earlier chunks.  Rows may start at any element: the wide load is an unaligned one where they do (one instruction as well).
// Rows and columns are counted without a sign: the steps loaded ahead reach 2048 columns behind the last one, whose number
// may be all but 2^31, and a wavefront's next row may lie as far behind the last row.
template <bool IN8>
__device__ __forceinline__ Chunk<IN8> load_chunk(const void* __restrict__ row_v, uint32_t col0, uint32_t cols) {
  Chunk<IN8> c;
#pragma unroll
  for (int k = 0; k < Chunk<IN8>::kWords; ++k) c.u[k] = 0u;
  if (IN8) {
    const uint8_t* row = static_cast<const uint8_t*>(row_v);
    if (col0 + 8 <= cols) {
      __builtin_memcpy(c.u, row + col0, 8);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (col0 + k < cols) c.u[(k >> 2) % Chunk<IN8>::kWords] |= (uint32_t)row[col0 + k] << (8 * (k & 3));
    }
  } else {
    const uint16_t* row = static_cast<const uint16_t*>(row_v);
    if (col0 + 8 <= cols) {
      __builtin_memcpy(c.u, row + col0, 16);
    } else {
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (col0 + k < cols) c.u[(k >> 1) % Chunk<IN8>::kWords] |= (uint32_t)row[col0 + k] << (16 * (k & 1));
    }
  }
  return c;
}

// The same for rows of 8 columns or more, one load without a branch around it: at the last 8 columns where the chunk reaches
// behind them, put right by end_chunk.  Behind a load that not every lane executes the compiler waits for all loads under
// way, so that nothing was in flight: the counting pass is bound by the reads of the matrix and takes, us, with load_chunk
// and with this: 11008 x 4096 18.6 / 15.9, 4096 x 11008 17.9 / 15.5, 8-bit values 11.5 / 10.1.
template <bool IN8>
__device__ __forceinline__ Chunk<IN8> load_whole_chunk(const void* __restrict__ row, uint32_t col0, uint32_t cols) {
  Chunk<IN8> c;
  __builtin_memcpy(c.u, static_cast<const unsigned char*>(row) + (size_t)min(col0, cols - 8u) * (IN8 ? 1 : 2), sizeof(c.u));
  return c;
}
// columns at or beyond `cols` become +0; `base`: the step's first column
template <bool IN8>
__device__ __forceinline__ void end_chunk(Chunk<IN8>& c, uint32_t base, uint32_t col0, uint32_t cols) {
  if (base + 512u <= cols) return;                     // (all lanes alike)
  const uint32_t here = col0 < cols ? min(cols - col0, 8u) : 0u;
  const uint32_t shift = (IN8 ? 8u : 16u) * (8u - here);         // the load began this many bits too early
  uint64_t lo, hi = 0;
  __builtin_memcpy(&lo, c.u, 8);
  if (IN8) {
    lo = here ? lo >> shift : 0;
  } else {
    __builtin_memcpy(&hi, c.u + Chunk<IN8>::kWords - 2, 8);
    lo = shift >= 64u ? (here ? hi >> (shift - 64u) : 0) : (shift ? lo >> shift | hi << (64u - shift) : lo);
    hi = shift >= 64u ? 0 : hi >> shift;
    __builtin_memcpy(c.u + Chunk<IN8>::kWords - 2, &hi, 8);
  }
  __builtin_memcpy(c.u, &lo, 8);
}

// The same through a buffer that ends with the row: what lies behind its end reads as zero, and nothing stands between the loads.  Ends are
// checked per 4 bytes, so rows begin and end on words.  For the fill kernel (the counting pass is no faster, 16.3 / 16.7).
template <bool IN8>
struct RowBuffer {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ RowBuffer(const void* row, uint32_t cols)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(row), 0, (int)((IN8 ? 1u : 2u) * cols), 0x00020000)) {}
  __device__ __forceinline__ Chunk<IN8> load(uint32_t col0) const {
    Chunk<IN8> c;
    if constexpr (IN8) {
      const auto q = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)col0, 0, 0);
      c.u[0] = (uint32_t)q[0];
      c.u[1] = (uint32_t)q[1];
    } else {
      const auto q = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(2u * col0), 0, 0);
#pragma unroll
      for (int k = 0; k < 4; ++k) c.u[k] = (uint32_t)q[k];
    }
    return c;
  }
};
constexpr int64_t kMaxBufferCols = int64_t{1} << 29;   // the loads ahead of a row's end stay below 2^32 bytes

// Bit k set iff column k is neither +0 nor -0.  Packed: adding 0x7FFF (0x7F) to the bits other than the sign carries
// into the sign position exactly when one of them is set, and never further.
template <bool IN8>
__device__ __forceinline__ unsigned nonzero_mask(const Chunk<IN8>& c) {
  if (IN8) {
    const uint32_t a = ((c.u[0] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) & 0x80808080u;
    const uint32_t b = ((c.u[1] & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) & 0x80808080u;
    uint32_t x = (a >> 7) | (b >> 3);                   // bits 0, 8, 16, 24 and 4, 12, 20, 28
    x |= x >> 7;
    return (x | (x >> 14)) & 0xFFu;
  }
  uint32_t x = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {                         // columns 2j and 2j + 1 at bits 2j and 16 + 2j
    const uint32_t t = ((c.u[j % Chunk<IN8>::kWords] & 0x7FFF7FFFu) + 0x7FFF7FFFu) & 0x80008000u;
    x |= t >> (15 - 2 * j);
  }
  return (x | (x >> 15)) & 0xFFu;
}

// What 8 columns store from their first non-zero on, for every mask of non-zeros.  Gaps inside the 8 columns need padding
// entries with 1- and 2-bit codes only; with wider ones only the first non-zero can have padding in front of it.
struct MaskInfo {
  uint64_t codes;          // 2^b_delta - 1 - code of entry e at bits e * b_delta (0 for the first, and for padding)
  uint32_t pos;            // entry number of column k at bits 4k (non-zeros only)
  uint32_t count;          // entries
};
template <int BD>
__device__ __forceinline__ MaskInfo mask_info(unsigned mask) {
  constexpr int kFull = (1 << BD) - 1;
  MaskInfo m{0, 0u, 0u};
  int e = 0, prev = -1;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    if (!((mask >> k) & 1u)) continue;
    if (prev >= 0) {
      const int g1 = k - prev - 1;                      // columns skipped
      e += 1 + (g1 >> BD);
      m.codes |= (uint64_t)(kFull - (g1 & kFull)) << (BD * e);
    }
    m.pos |= (uint32_t)e << (4 * k);
    m.count = (uint32_t)e + 1u;
    prev = k;
  }
  return m;
}

// Columns skipped in front of the chunk's first non-zero (0 without one).  `carry` is the position (column + 1, 0 = none) of
// the last stored entry of the steps already consumed; it is advanced over this step.
__device__ __forceinline__ int lead_of_chunk(unsigned mask, uint32_t col0, int lane, uint32_t* carry) {
  const uint32_t lastpos = mask ? col0 + 32u - (uint32_t)__clz((int)mask) : 0u;
  uint32_t incl = lastpos;
  // where every lane has a non-zero the lane before holds the previous one: no scan
  if (!__all(mask != 0u)) incl = wave_incl_scan_max_u32(lastpos);
  uint32_t prevpos = (uint32_t)__shfl_up((int)incl, 1);
  if (lane == 0) prevpos = 0;
  prevpos = max(prevpos, *carry);
  *carry = max(*carry, (uint32_t)__builtin_amdgcn_readlane((int)incl, 63));
  return mask ? (int)(col0 + (uint32_t)(__ffs((int)mask) - 1) - prevpos) : 0;
}

// steps of 512 columns loaded ahead
constexpr int kEncodeAhead = 2;

// WIDE: loads without a branch, for rows of 8 columns or more
template <bool IN8, bool WIDE, int BD>
__global__ void __launch_bounds__(256)
encode_count_kernel(const void* __restrict__ dense, uint32_t rows, uint32_t cols, int64_t ld,
                    uint32_t* __restrict__ row_entries, uint32_t* __restrict__ row_nnz) {
  __shared__ uint32_t counts[256];                      // entries from the first non-zero on, by mask (narrow codes)
  if (BD < 3) {
    counts[threadIdx.x] = mask_info<BD>(threadIdx.x).count;
    __syncthreads();
  }
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int nwaves = blockDim.x >> 6;
  for (uint32_t row = blockIdx.x * nwaves + wave; row < rows; row += gridDim.x * nwaves) {
    const void* src = static_cast<const unsigned char*>(dense) + (int64_t)row * ld * (IN8 ? 1 : 2);
    uint32_t carry = 0;
    unsigned entries = 0, nnz = 0;
    auto load = [&](uint32_t col0) { return WIDE ? load_whole_chunk<IN8>(src, col0, cols) : load_chunk<IN8>(src, col0, cols); };
    Chunk<IN8> ring[kEncodeAhead];
#pragma unroll
    for (int j = 0; j < kEncodeAhead; ++j) ring[j] = load(512u * j + 8u * lane);
    for (uint32_t base = 0; base < cols; base += 512u * kEncodeAhead) {
#pragma unroll
      for (int j = 0; j < kEncodeAhead; ++j) {
        const uint32_t col0 = base + 512u * j + 8u * lane;     // steps behind the last column count nothing
        if (WIDE) end_chunk<IN8>(ring[j], base + 512u * j, col0, cols);
        const unsigned mask = nonzero_mask<IN8>(ring[j]);
        ring[j] = load(col0 + 512u * kEncodeAhead);
        const int lead = lead_of_chunk(mask, col0, lane, &carry);
        const unsigned n = (unsigned)__popc(mask);
        nnz += n;
        entries += (BD < 3 ? counts[mask] : n) + (unsigned)(lead >> BD);
      }
    }
    entries = wave_incl_scan_u32(entries);
    nnz = wave_incl_scan_u32(nnz);
    if (lane == 63) {
      row_entries[row] = entries;
      row_nnz[row] = nnz;
    }
  }
}

// Row pointers from the per-row counts in small launches: every block of
// 1024 rows totals its counts, one workgroup turns the block totals into block
// offsets (and totals the statistics of the storage report, which it writes to pinned host memory: no copy to wait
// for), every block then prefix-sums its own rows.  Up to kFusedBlocks blocks the one workgroup does the first of
// these as well, a wavefront per block (11008 rows: 4.8 + 4.9 us and a launch -> one launch).  The entry total is kept as a 64-bit number so that
// the host can detect overflow of the 32-bit row pointers before anything is
// written through them.
struct BlockSums {
  unsigned long long entries;
  unsigned long long nnz;
  unsigned int empty;
  unsigned int longest;
};

__device__ __forceinline__ unsigned long long wave_incl_scan_u64(unsigned long long v, int lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned long long up = __shfl_up(v, off);
    if (lane >= off) v += up;
  }
  return v;
}

__global__ void __launch_bounds__(1024)
encode_block_sums_kernel(const uint32_t* __restrict__ row_entries, const uint32_t* __restrict__ row_nnz, uint32_t rows,
                         BlockSums* __restrict__ sums) {
  __shared__ BlockSums part[16];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t r = blockIdx.x * 1024u + t;
  const uint32_t e = r < rows ? row_entries[r] : 0u;
  unsigned long long se = e, sn = r < rows ? row_nnz[r] : 0u;
  unsigned int empty = (r < rows && e == 0) ? 1u : 0u, longest = e;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    se += __shfl_xor(se, off);
    sn += __shfl_xor(sn, off);
    empty += __shfl_xor(empty, off);
    longest = max(longest, __shfl_xor(longest, off));
  }
  if (lane == 0) part[wave] = BlockSums{se, sn, empty, longest};
  __syncthreads();
  if (t == 0) {
    BlockSums b = part[0];
    for (int i = 1; i < 16; ++i) {
      b.entries += part[i].entries;
      b.nnz += part[i].nnz;
      b.empty += part[i].empty;
      b.longest = max(b.longest, part[i].longest);
    }
    sums[blockIdx.x] = b;
  }
}

constexpr int kFusedBlocks = 64;

// one workgroup: block_off[b] = entries of the blocks in front of b; totals to *report.  FUSED: from the rows' counts,
// at most kFusedBlocks blocks; else from the block totals.
template <bool FUSED>
__global__ void __launch_bounds__(1024)
encode_block_offsets_kernel(const BlockSums* __restrict__ sums, const uint32_t* __restrict__ row_entries,
                            const uint32_t* __restrict__ row_nnz, int rows, int nblocks,
                            unsigned long long* __restrict__ block_off, EncodeReport* __restrict__ report) {
  __shared__ BlockSums fused[FUSED ? kFusedBlocks : 1];
  if (FUSED) {
    const int lane = threadIdx.x & 63;
    for (int b = threadIdx.x >> 6; b < nblocks; b += 16) {
      uint32_t e[16], z[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = 1024 * b + 64 * i + lane;
        e[i] = r < rows ? row_entries[r] : 0u;
        z[i] = r < rows ? row_nnz[r] : 0u;
      }
      unsigned long long se = 0, sn = 0;
      unsigned int empty = 0, longest = 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        se += e[i];
        sn += z[i];
        empty += (1024 * b + 64 * i + lane < rows && e[i] == 0) ? 1u : 0u;
        longest = max(longest, e[i]);
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        se += __shfl_xor(se, off);
        sn += __shfl_xor(sn, off);
        empty += __shfl_xor(empty, off);
        longest = max(longest, __shfl_xor(longest, off));
      }
      if (lane == 0) fused[b] = BlockSums{se, sn, empty, longest};
    }
    __syncthreads();
    sums = fused;
  }
  __shared__ unsigned long long wave_tot[16];
  __shared__ unsigned long long carry_s;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  unsigned long long nnz = 0;
  unsigned int empty = 0, longest = 0;
  if (t == 0) carry_s = 0;
  __syncthreads();
  for (int base = 0; base < nblocks; base += 1024) {
    const int b = base + t;
    const BlockSums v = b < nblocks ? sums[b] : BlockSums{0, 0, 0, 0};
    nnz += v.nnz;
    empty += v.empty;
    longest = max(longest, v.longest);
    const unsigned long long incl = wave_incl_scan_u64(v.entries, lane);
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    unsigned long long before = carry_s;
    for (int i = 0; i < wave; ++i) before += wave_tot[i];
    if (b < nblocks) block_off[b] = before + incl - v.entries;
    __syncthreads();
    if (t == 1023) carry_s = before + incl;
    __syncthreads();
  }
  // totals of the statistics over the workgroup
  __shared__ unsigned long long s_nnz[16];
  __shared__ unsigned int s_empty[16], s_long[16];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    nnz += __shfl_xor(nnz, off);
    empty += __shfl_xor(empty, off);
    longest = max(longest, __shfl_xor(longest, off));
  }
  if (lane == 0) {
    s_nnz[wave] = nnz;
    s_empty[wave] = empty;
    s_long[wave] = longest;
  }
  __syncthreads();
  if (t == 0) {
    unsigned long long nn = 0;
    unsigned int em = 0, mx = 0;
    for (int i = 0; i < 16; ++i) {
      nn += s_nnz[i];
      em += s_empty[i];
      mx = max(mx, s_long[i]);
    }
    report->stats = EncodeStats{nn, carry_s, em, mx};
  }
}

// Everything before it on the stream is over when the host reads `number`.
__global__ void __launch_bounds__(64) encode_done_kernel(EncodeReport* report, uint32_t number) {
  if (threadIdx.x == 0) __hip_atomic_store(&report->done, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ void __launch_bounds__(1024)
encode_row_ptr_kernel(const uint32_t* __restrict__ row_entries, uint32_t rows, const unsigned long long* __restrict__ block_off,
                      uint32_t* __restrict__ row_ptr, uint32_t total, int b_delta, uint32_t* __restrict__ deltas) {
  __shared__ unsigned long long wave_tot[16];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const uint32_t r = blockIdx.x * 1024u + t;
  const unsigned long long e = r < rows ? row_entries[r] : 0u;
  const unsigned long long incl = wave_incl_scan_u64(e, lane);
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  unsigned long long before = block_off[blockIdx.x];
  for (int i = 0; i < wave; ++i) before += wave_tot[i];
  // a 32-bit word of codes that two rows share is put together with atomic ORs by the fill kernel: it has to be zero
  auto clear_shared_word = [&](uint64_t entry) {
    if ((entry * (unsigned)b_delta) & 31u) deltas[(entry * (unsigned)b_delta) >> 5] = 0u;
  };
  if (r < rows) {
    const uint32_t p = (uint32_t)(before + incl - e);
    row_ptr[r] = p;
    clear_shared_word(p);
  }
  if (r == rows - 1) {
    row_ptr[rows] = total;
    clear_shared_word(total);
  }
}

// Second pass: values and packed codes.  A wavefront collects its row's entries in LDS, a window of kFillWindow entries
// at a time (numbered from a multiple of 32 entries at or before the row's start, so that 16-byte pieces of values and
// 32-bit words of codes are aligned in LDS as in memory), and writes full windows out in full-width stores.
//  - Codes are ORed into the window as 2^b_delta - 1 - code and inverted on the way out: a padding entry is then all
//    zeros, value and code, and costs nothing but its place.
//  - What a lane stores follows from the mask of its 8 columns, looked up in a table (MaskInfo); only the code of its
//    first non-zero depends on the columns before.
//  - An entry in front of the window or behind it lands in a margin that is never read (a lane's entries, without the padding
//    in front of them, span at most 8); a step that reaches behind the window is put into it once more when
//    the window has moved on.
//  - The words of codes that two rows share are ORed into memory (cleared beforehand by encode_row_ptr_kernel).
// The previous version wrote a code byte per entry to scratch, packed by another kernel, and visited a lane's columns with two
// predicated stores each: 11008 x 4096 at 50 % took 55.8 us + 6.0 us to pack, 36864 x 12288 411 us.
constexpr int kFillWindow = 1024;
constexpr int kFillWaves = 4;
constexpr int kFillMargin = 8;                          // entries

// BUFFER: loads through RowBuffer
template <bool IN8, bool BUFFER, int BD>
__global__ void __launch_bounds__(64 * kFillWaves)
encode_fill_kernel(const void* __restrict__ dense, uint32_t rows, uint32_t cols, int64_t ld,
                   const uint32_t* __restrict__ row_ptr, void* __restrict__ values_v,
                   uint32_t* __restrict__ deltas, uint32_t pad_nnz, uint32_t alloc_nnz) {
  constexpr uint32_t kFull = (1u << BD) - 1u;
  constexpr int kValueBytes = IN8 ? 1 : 2;
  constexpr int kPiece = 16 / kValueBytes;              // entries per 16-byte piece of values
  constexpr int kWordEntries = 32 / BD;                 // entries per word of codes
  constexpr int kWords = kFillWindow / kWordEntries;    // of a window; one margin of 4 words on either side
  __shared__ __align__(16) unsigned char stage_v[kFillWaves][(kFillWindow + 2 * kPiece) * kValueBytes];   // margins of a piece
  __shared__ uint32_t stage_c[kFillWaves][kWords + 8];
  __shared__ uint32_t table_pos[256];
  __shared__ uint32_t table_codes[256];
  __shared__ uint32_t table_high[BD == 8 ? 256 : (BD < 3 ? 256 : 1)];     // codes 4 ... 7 of 8-bit codes; counts of narrow ones
  static_assert(kPiece >= kFillMargin && 4 * 32 >= BD * kFillMargin, "margins");
  uint16_t* values16 = static_cast<uint16_t*>(values_v);
  uint8_t* values8 = static_cast<uint8_t*>(values_v);
  // the zero tail of both arrays (fewer than 128 entries): the first workgroup writes it
  if (blockIdx.x == 0) {
    for (uint32_t k = pad_nnz + threadIdx.x; k < alloc_nnz; k += blockDim.x) {
      if (IN8) values8[k] = 0;
      else values16[k] = 0;
    }
    const uint64_t first = ((uint64_t)pad_nnz * BD + 31) >> 5, last = ((uint64_t)alloc_nnz * BD) >> 5;
    for (uint64_t k = first + threadIdx.x; k < last; k += blockDim.x) deltas[k] = 0u;
  }
  {
    const MaskInfo m = mask_info<BD>(threadIdx.x);      // 256 threads, 256 masks
    table_pos[threadIdx.x] = m.pos;
    table_codes[threadIdx.x] = (uint32_t)m.codes;
    if (BD == 8) table_high[threadIdx.x] = (uint32_t)(m.codes >> 32);
    if (BD < 3) table_high[threadIdx.x] = m.count;
  }
  const int lane = threadIdx.x & 63;
  // A buffer has to be the wavefront's, or every load through it stands in a loop over the lanes' descriptors (11008 x 4096 with 8-bit values
  // 27.7 / 26.1 us without it).  The version with branches is slower with a uniform row (36864 x 12288 350 / 413, 11008 x 4096 34.8 / 37.0).
  const int wave = BUFFER ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : (int)(threadIdx.x >> 6);
  unsigned char* sv = stage_v[wave] + 16;               // entry 0 of the window
  uint32_t* sc = stage_c[wave] + 4;
  for (int i = lane; i < (kFillWindow + 2 * kPiece) * kValueBytes / 16; i += 64)
    reinterpret_cast<uint4*>(stage_v[wave])[i] = make_uint4(0, 0, 0, 0);
  for (int i = lane; i < kWords + 8; i += 64) stage_c[wave][i] = 0u;
  __syncthreads();

  for (uint32_t row = blockIdx.x * kFillWaves + wave; row < rows; row += gridDim.x * kFillWaves) {
    const uint32_t begin = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_ptr[row]);
    const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_ptr[row + 1]);
    const void* src = static_cast<const unsigned char*>(dense) + (int64_t)row * ld * kValueBytes;
    uint32_t carry = 0;
    uint32_t cursor = begin;                            // first entry of this step
    uint32_t window = begin & ~31u;                     // first entry of the window
    // entries [max(begin, window), min(end, window + kFillWindow)) to memory, the window zero again
    auto flush = [&]() {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");     // a wavefront's LDS operations complete in order
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const uint32_t lo = begin > window ? begin - window : 0u;             // in entries of the window
      const uint32_t hi = min(end - window, (uint32_t)kFillWindow);
#pragma unroll
      for (int j = 0; j < kFillWindow / kPiece / 64; ++j) {
        const uint32_t p = (uint32_t)(lane + 64 * j), first = kPiece * p, last = first + kPiece;
        if (last > lo && first < hi) {
          uint4* q = reinterpret_cast<uint4*>(sv) + p;
          const uint4 v = *q;
          const size_t at = (size_t)window + first;
          if (first >= lo && last <= hi) {
            *reinterpret_cast<uint4*>(static_cast<unsigned char*>(values_v) + at * kValueBytes) = v;
          } else {                                      // the row's first or last entries
            for (uint32_t k = max(first, lo); k < min(last, hi); ++k) {
              if (IN8) values8[window + k] = sv[k];
              else values16[window + k] = reinterpret_cast<const uint16_t*>(sv)[k];
            }
          }
          *q = make_uint4(0, 0, 0, 0);
        }
      }
#pragma unroll
      for (int j = 0; j < (kWords + 63) / 64; ++j) {
        const uint32_t p = (uint32_t)(lane + 64 * j), first = kWordEntries * p, last = first + kWordEntries;
        if ((kWords % 64 == 0 || p < (uint32_t)kWords) && last > lo && first < hi) {
          const uint32_t c = ~sc[p];
          sc[p] = 0u;
          uint32_t* out = deltas + (((uint64_t)window * BD) >> 5) + p;
          if (first >= lo && last <= hi) {
            *out = c;
          } else {
            const uint32_t from = first < lo ? BD * (lo - first) : 0u, to = last > hi ? BD * (hi - first) : 32u;
            atomicOr(out, c & (0xFFFFFFFFu << from) & (0xFFFFFFFFu >> (32u - to)));
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    const RowBuffer<IN8> buffer(src, cols);
    auto load = [&](uint32_t col0) { return BUFFER ? buffer.load(col0) : load_chunk<IN8>(src, col0, cols); };
    Chunk<IN8> ring[kEncodeAhead];
#pragma unroll
    for (int j = 0; j < kEncodeAhead; ++j) ring[j] = load(512u * j + 8u * lane);
    for (uint32_t base = 0; base < cols; base += 512u * kEncodeAhead) {
#pragma unroll
      for (int j = 0; j < kEncodeAhead; ++j) {
        const uint32_t col0 = base + 512u * j + 8u * lane;     // steps behind the last column store nothing
        const Chunk<IN8> c = ring[j];
        ring[j] = load(col0 + 512u * kEncodeAhead);
        const unsigned mask = nonzero_mask<IN8>(c);
        const uint32_t pos = table_pos[mask];
        const uint32_t low = table_codes[mask];
        const int lead = lead_of_chunk(mask, col0, lane, &carry);
        const uint32_t count = BD < 3 ? table_high[mask] : (uint32_t)__popc(mask);
        const uint32_t pads = (uint32_t)lead >> BD;     // padding entries in front, greedy
        const uint32_t incl = wave_incl_scan_u32(pads + count);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        const uint32_t first = cursor + incl - count;   // the lane's first non-zero
        // its code, and the others', from bit 0 on
        uint64_t codes = low | (mask ? kFull - ((uint32_t)lead & kFull) : 0u);
        if (BD == 8) codes |= (uint64_t)table_high[mask] << 32;
        for (;;) {
          const int rel = (int)(first - window);
          if (mask != 0u && (uint32_t)(rel + kFillMargin) < (uint32_t)(kFillWindow + kFillMargin)) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              if ((mask >> k) & 1u) {
                const int at = rel + (int)((pos >> (4 * k)) & 15u);
                if (IN8) sv[at] = (uint8_t)(c.u[(k >> 2) % Chunk<IN8>::kWords] >> (8 * (k & 3)));
                else reinterpret_cast<uint16_t*>(sv)[at] = (uint16_t)(c.u[(k >> 1) % Chunk<IN8>::kWords] >> (16 * (k & 1)));
              }
            }
            const uint32_t bit = (uint32_t)(BD * rel + 128);         // the margin in front is 4 words
            uint32_t* w = sc - 4 + (bit >> 5);
            const uint64_t shifted = codes << (bit & 31u);
            atomicOr(w, (uint32_t)shifted);
            atomicOr(w + 1, (uint32_t)(shifted >> 32));
            if (BD == 8) atomicOr(w + 2, (uint32_t)((codes >> 1) >> (63u - (bit & 31u))));
          }
          if (cursor + total - window <= (uint32_t)kFillWindow) break;
          flush();
          window += kFillWindow;
        }
        cursor += total;
      }
    }
    if (end > window && end > begin) flush();
  }
}

// Freed unless the call succeeds.
struct DeviceBuf {
  void* p = nullptr;
  ~DeviceBuf() {
    if (p) (void)hipFree(p);
  }
  void* release() {
    void* q = p;
    p = nullptr;
    return q;
  }
};

// Scratch memory of the encoder (per-row counts and block sums: about 8 bytes per row), kept per
// device and reused from call to call.  One encoder call at a time uses it.
struct Workspace {
  void* p = nullptr;
  size_t cap = 0;
  EncodeReport* report = nullptr;   // host, pinned: the kernels report through it
  uint32_t encodings = 0;
};
std::mutex g_ws_mutex;
Workspace g_ws[64];
constexpr size_t kKeepScratchBytes = size_t{64} << 20;

hipError_t workspace_reserve(Workspace& ws, size_t bytes) {
  if (bytes <= ws.cap) return hipSuccess;
  if (ws.p) (void)hipFree(ws.p);
  ws.p = nullptr;
  ws.cap = 0;
  const size_t want = bytes + bytes / 4;             // some slack so that similar sizes do not reallocate
  const hipError_t e = device_malloc(&ws.p, want);
  if (e == hipSuccess) ws.cap = want;
  return e;
}

template <bool WIDE>
auto count_kernel(bool in8, int b_delta) {
  return in8 ? encode_count_kernel<true, WIDE, 4> : b_delta == 4 ? encode_count_kernel<false, WIDE, 4>
         : b_delta == 2 ? encode_count_kernel<false, WIDE, 2> : b_delta == 8 ? encode_count_kernel<false, WIDE, 8>
                                                                             : encode_count_kernel<false, WIDE, 1>;
}

// Waits until the stream has come to the end of encoding `number`.  Looked at by the host itself it is seen 5.9 us after a launch,
// hipStreamSynchronize returns after 11.4.  The look ends after 2 ms, then the runtime waits (and says what is wrong, if the
// number never comes).  Only the last wait of an encoding is of this kind: the runtime does not learn from it that the launches are over, and
// where more than about 8 of them pile up a program's next synchronization takes it 16 us longer and the launches after it 1 to 2 us each
// (512 x 512, us: 4 kernels of the caller, encoding, 1 kernel, synchronization, product and synchronization: both waits by the runtime 21 + 43
// + 7 + 12 + 18, both by the host 25 + 34 + 7 + 28 + 20, the first by the runtime and the last by the host 21 + 39 + 7 + 12 + 18; the encoding of 4096 x
// 4096 158 / 122 / 128, most of that from the kept blocks).
hipError_t wait_for_encoding(const EncodeReport* report, uint32_t number, hipStream_t stream) {
  const auto begin = std::chrono::steady_clock::now();
  do {
    for (int i = 0; i < 64; ++i) {
      if (__atomic_load_n(&report->done, __ATOMIC_ACQUIRE) == number) return hipSuccess;
      __builtin_ia32_pause();
    }
  } while (std::chrono::steady_clock::now() - begin < std::chrono::milliseconds(2));
  return hipStreamSynchronize(stream);
}

template <bool BUFFER>
auto fill_kernel(bool in8, int b_delta) {
  return in8 ? encode_fill_kernel<true, BUFFER, 4> : b_delta == 4 ? encode_fill_kernel<false, BUFFER, 4>
         : b_delta == 2 ? encode_fill_kernel<false, BUFFER, 2> : b_delta == 8 ? encode_fill_kernel<false, BUFFER, 8>
                                                                              : encode_fill_kernel<false, BUFFER, 1>;
}

constexpr size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace

// The handle's three arrays live in ONE allocation (*block, of encoded_layout, to be given back with block_release).
int encode_on_device(const void* dense, int64_t rows, int64_t cols, int64_t ld, int b_delta, int b_val,
                     hipStream_t stream, void** block,
                     void** values, uint8_t** deltas, uint32_t** row_ptr, int64_t* nnz,
                     int64_t* pad_nnz, int64_t* alloc_nnz, int64_t* empty_rows,
                     int64_t* max_row_entries) {
  const int cus = device_cu_count();
  const bool in8 = b_val == 8;
  int dev = 0;
  MACKO_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return MACKO_E_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_ws_mutex);
  Workspace& ws = g_ws[dev];
  if (!ws.report) {
    void* h = nullptr;
    if (hipHostMalloc(&h, sizeof(EncodeReport), hipHostMallocCoherent) != hipSuccess) {
      (void)hipGetLastError();
      return MACKO_E_OUT_OF_MEMORY;
    }
    ws.report = new (h) EncodeReport{};
  }
  // scratch layout of the counting pass
  const int64_t nblocks = (rows + 1023) / 1024;
  const size_t o_counts = 0;
  const size_t o_nnz = align_up(o_counts + 4 * (size_t)rows, 256);
  const size_t o_sums = align_up(o_nnz + 4 * (size_t)rows, 256);
  const size_t o_boff = align_up(o_sums + sizeof(BlockSums) * (size_t)std::max<int64_t>(nblocks, 1), 256);
  const size_t scratch_bytes = o_boff + 8 * (size_t)std::max<int64_t>(nblocks, 1);
  if (workspace_reserve(ws, scratch_bytes) != hipSuccess) {
    (void)hipGetLastError();
    return MACKO_E_OUT_OF_MEMORY;
  }
  auto at = [&](size_t off) { return static_cast<unsigned char*>(ws.p) + off; };
  uint32_t* counts = reinterpret_cast<uint32_t*>(at(o_counts));
  uint32_t* nnzs = reinterpret_cast<uint32_t*>(at(o_nnz));
  BlockSums* sums = reinterpret_cast<BlockSums*>(at(o_sums));
  unsigned long long* boff = reinterpret_cast<unsigned long long*>(at(o_boff));

  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((rows + 3) / 4, (int64_t)cus * 16));
  if (rows > 0) {
    // Lanes behind the row's last column load too, which costs where 16-byte loads lie across 4 bytes: such rows of fp16 only
    // from 3 steps on, where the loads under way pay for it (whole call, us, with a branch / without: 120000 x 9 149 / 162, x 201 208 /
    // 220, 60000 x 1025 197 / 205; but 15000 x 1537 112.4 / 111.8, x 3001 123.1 / 120.2, and on 4 bytes 120000 x 100 220 / 215).
    const bool on_words = in8 || ((reinterpret_cast<uintptr_t>(dense) & 3) == 0 && ld % 2 == 0);
    auto kcount = cols >= (on_words ? 8 : 1536) ? count_kernel<true>(in8, b_delta) : count_kernel<false>(in8, b_delta);
    hipLaunchKernelGGL(kcount, dim3(grid), dim3(256), 0, stream, dense, (uint32_t)rows, (uint32_t)cols, ld, counts, nnzs);
    if (nblocks > kFusedBlocks)
      hipLaunchKernelGGL(encode_block_sums_kernel, dim3((unsigned)nblocks), dim3(1024), 0, stream, counts, nnzs,
                         (uint32_t)rows, sums);
  }
  hipLaunchKernelGGL(nblocks > kFusedBlocks ? encode_block_offsets_kernel<false> : encode_block_offsets_kernel<true>,
                     dim3(1), dim3(1024), 0, stream, static_cast<const BlockSums*>(sums),
                     static_cast<const uint32_t*>(counts), static_cast<const uint32_t*>(nnzs), (int)rows, (int)nblocks,
                     boff, ws.report);
  MACKO_HIP_TRY(hipGetLastError());
  MACKO_HIP_TRY(hipStreamSynchronize(stream));
  const EncodeStats st = ws.report->stats;
  if (st.pad_nnz >= (1ull << 32)) return MACKO_E_OVERFLOW;
  const int64_t pad = (int64_t)st.pad_nnz;
  const int64_t granule = alloc_granule(b_delta);
  const int64_t alloc = (pad + granule - 1) / granule * granule;
  if (alloc >= (int64_t{1} << 32)) return MACKO_E_OVERFLOW;

  // the output block
  const EncodedLayout layout = encoded_layout(rows, alloc, b_delta, b_val);
  DeviceBuf out;
  if (block_acquire(&out.p, layout.total) != hipSuccess) {
    (void)hipGetLastError();
    return MACKO_E_OUT_OF_MEMORY;
  }
  unsigned char* ob = static_cast<unsigned char*>(out.p);
  void* vals = ob;
  uint32_t* dels = reinterpret_cast<uint32_t*>(ob + layout.deltas);
  uint32_t* rp = reinterpret_cast<uint32_t*>(ob + layout.row_ptr);
  if (rows > 0)
    hipLaunchKernelGGL(encode_row_ptr_kernel, dim3((unsigned)nblocks), dim3(1024), 0, stream, counts, (uint32_t)rows,
                       boff, rp, (uint32_t)pad, b_delta, dels);
  else
    MACKO_HIP_TRY(hipMemsetAsync(rp, 0, 4, stream));
  if (rows > 0 && alloc > 0) {
    // A wavefront's loads are under way with RowBuffer; with load_chunk only other wavefronts cover them, and those reach the rate of a large
    // fp16 matrix better.  us, load_chunk / RowBuffer: up to as many rows as the chip holds wavefronts, 280 x 504 5.8 / 5.0, 2000 x 2000 9.9 / 8.1,
    // 4096 x 11008 33.8 / 32.3; 8-bit values of any size, 11008 x 4096 29.3 / 26.1, 36864 x 12288 277 / 249; few columns, 120000 x 128 89 / 77,
    // 1000000 x 64 660 / 549; else by the cells, 11008 x 1024 16.7 / 14.4, 20000 x 2048 35.1 / 36.5, 11008 x 4096 34.8 / 35.3, 36864 x 4096 at 90 % 86 / 116;
    // more of them where 16 bytes of a row lie across two lines, 11008 x 4100 40.7 / 38.0, 36864 x 4100 153 / 166, and with 8-bit codes, which
    // take load_chunk more registers, 11008 x 4096 at 90 % 31.3 / 27.7, 24576 x 4096 56.6 / 54.6, 60000 x 4096 147 / 186.
    const int per_word = in8 ? 4 : 2;
    const uintptr_t row_starts = reinterpret_cast<uintptr_t>(dense) | (uintptr_t)(ld * (in8 ? 1 : 2));
    const bool whole_words = (row_starts & 3) == 0 && cols % per_word == 0;
    const int64_t cells = b_delta == 8 ? 100000000 : (row_starts & 15) != 0 ? 64000000 : 20000000;
    const bool buffer = whole_words && cols <= kMaxBufferCols && (in8 || rows <= (int64_t)cus * 28 || cols <= 256 || rows * cols <= cells);
    auto kfill = buffer ? fill_kernel<true>(in8, b_delta) : fill_kernel<false>(in8, b_delta);
    hipLaunchKernelGGL(kfill, dim3(grid), dim3(64 * kFillWaves), 0, stream, dense, (uint32_t)rows, (uint32_t)cols, ld,
                       static_cast<const uint32_t*>(rp), vals, dels, (uint32_t)pad, (uint32_t)alloc);
  }
  hipLaunchKernelGGL(encode_done_kernel, dim3(1), dim3(64), 0, stream, ws.report, ++ws.encodings);
  MACKO_HIP_TRY(hipGetLastError());
  MACKO_HIP_TRY(wait_for_encoding(ws.report, ws.encodings, stream));
  // a large scratch buffer is not kept (from 6.7 M rows on: 8 bytes per row and a quarter more)
  if (ws.cap > kKeepScratchBytes) {
    (void)hipFree(ws.p);
    ws.p = nullptr;
    ws.cap = 0;
  }
  *block = out.release();
  *values = vals;
  *deltas = reinterpret_cast<uint8_t*>(dels);
  *row_ptr = rp;
  *nnz = (int64_t)st.nnz;
  *pad_nnz = pad;
  *alloc_nnz = alloc;
  *empty_rows = st.empty_rows;
  *max_row_entries = st.max_row_entries;
  return MACKO_OK;
}

}  // namespace macko
