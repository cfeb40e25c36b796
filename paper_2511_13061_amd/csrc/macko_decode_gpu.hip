// Expanding the format on the device: the column index of every stored entry
// (Section 4.4: a column is the running sum of the row's deltas; the sums are
// formed as in Algorithm 1, per lane and then across the wavefront) and, from
// those, the dense matrix back (the format is lossless, Section 5.2).
//
// Both use the in-register decode and the cross-lane prefix sum of the product
// kernels, so the column indices they write are the ones the product gathers x
// with; the tests compare them entry by entry with the CPU oracle.
//
// One wavefront per row and 512 entries per step, as in the product.  Expanding
// a matrix is a conversion, not a per-token operation.  Roofline: HBM; the dense
// expansion reads 2.5 n bytes and writes 2 R C bytes once (rows are assembled in
// LDS, whole or a window at a time; a few rows longer than LDS are cleared and scattered into).
#include "macko_decode.h"
#include "macko_device.h"
#include "macko_internal.h"

namespace macko {
namespace {

constexpr int kExpandBlock = 256;

// DENSE: the stored values to their places in a cleared fp16 matrix; else every entry's column to cols_out.
template <int BD, bool DENSE>
__global__ void __launch_bounds__(kExpandBlock)
expand_kernel(const void* __restrict__ values, const uint32_t* __restrict__ deltas, const uint32_t* __restrict__ row_ptr,
              const int rows, const int cols, int32_t* __restrict__ cols_out, uint16_t* __restrict__ dense, const int64_t ld) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kExpandBlock / 64) + (threadIdx.x >> 6)));
  const int nwaves = (int)gridDim.x * (kExpandBlock / 64);
  for (uint32_t row = wave; row < (uint32_t)rows; row += nwaves) {          // wavefront-uniform
    const uint32_t start = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_ptr[row]);
    const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_ptr[row + 1]);
    if (end <= start) continue;
    const uint32_t a0 = start & ~7u;                         // the lanes' chunks are aligned to 8 entries
    const int nsteps = (int)((end - a0 + 511u) >> 9);
    int base2 = 0;                                           // doubled position before this step
    for (int step = 0; step < nsteps; ++step) {
      const uint32_t e0 = a0 + 512u * (uint32_t)step + 8u * (uint32_t)lane;
      const uint32_t chunk = min(e0, end - 1u) >> 3;         // lanes past the row end re-read its last chunk
      LaneCodes<BD> w;
      LaneValues<16> v;
      w.load(deltas, chunk);
      if (DENSE) v.load(values, chunk);
      w.keep_if(e0 < end);
      w.decode();
      const LanePositions<BD> pos{w};
      const uint32_t tot = w.total();
      const uint32_t incl = wave_incl_scan_u32(tot);
      if (step == 0) {
        const int before = (int)(start - a0);                // entries of the previous row in lane 0's chunk
        if (before > 0) base2 = -(int)w.through(before - 1);
      }
      const int lanebase = base2 + (int)(incl - tot);
#define MACKO_ENTRY(k)                                                                  \
  {                                                                                     \
    const uint32_t e = e0 + k;                                                          \
    const int col = (lanebase + pos.template offset<k>()) >> 1;                           \
    if (e >= start && e < end) {                                                        \
      if (!DENSE) cols_out[e] = col;                                                    \
      else if (col < cols) dense[(int64_t)row * ld + col] = (uint16_t)v.template bits<k>(); \
    }                                                                                   \
  }
      MACKO_ENTRY(0) MACKO_ENTRY(1) MACKO_ENTRY(2) MACKO_ENTRY(3)
      MACKO_ENTRY(4) MACKO_ENTRY(5) MACKO_ENTRY(6) MACKO_ENTRY(7)
#undef MACKO_ENTRY
      base2 += (int)__builtin_amdgcn_readlane((int)incl, 63);
    }
  }
}

// dense[r][0 .. cols) = +0 for every row (cells between cols and ld are left alone)
template <bool VEC>
__global__ void __launch_bounds__(256) zero_rows_kernel(uint16_t* __restrict__ dense, const int rows, const int cols,
                                                         const int64_t ld) {
  const int per_row = VEC ? cols / 8 : cols;                 // stores per row
  const int64_t total = (int64_t)rows * per_row;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t r = i / per_row;
    const int c = (int)(i - r * per_row);
    if (VEC) reinterpret_cast<uint4*>(dense + r * ld)[c] = make_uint4(0, 0, 0, 0);
    else dense[r * ld + c] = 0;
  }
}

// What the product kernels take on trust about an encoding, checked row by row:
// row_ptr starts at 0, never decreases and ends at pad_nnz, and no entry decodes
// to a column at or beyond cols.  The smallest offending row number is left in
// *first_bad (which the caller sets to `rows` beforehand).  A row whose pointers
// are out of order or out of range is reported without being decoded, so the
// check itself reads nothing outside [0, pad_nnz).
template <int BD>
__global__ void __launch_bounds__(kExpandBlock)
check_kernel(const uint32_t* __restrict__ deltas, const uint32_t* __restrict__ row_ptr, const int rows,
             const int cols, const uint32_t pad_nnz, unsigned int* __restrict__ first_bad) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kExpandBlock / 64) + (threadIdx.x >> 6)));
  const int nwaves = (int)gridDim.x * (kExpandBlock / 64);
  for (uint32_t row = wave; row < (uint32_t)rows; row += nwaves) {          // wavefront-uniform
    const uint32_t start = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_ptr[row]);
    const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_ptr[row + 1]);
    bool bad = end < start || end > pad_nnz || (row == 0u && start != 0u) || (row == (uint32_t)rows - 1u && end != pad_nnz);
    if (!bad && end > start) {
      const uint32_t a0 = start & ~7u;
      const int nsteps = (int)((end - a0 + 511u) >> 9);
      int base2 = 0;
      bool lane_bad = false;
      for (int step = 0; step < nsteps; ++step) {
        const uint32_t e0 = a0 + 512u * (uint32_t)step + 8u * (uint32_t)lane;
        const uint32_t chunk = min(e0, end - 1u) >> 3;
        LaneCodes<BD> w;
        w.load(deltas, chunk);
        w.keep_if(e0 < end);
        w.decode();
        const LanePositions<BD> pos{w};
        const uint32_t tot = w.total();
        const uint32_t incl = wave_incl_scan_u32(tot);
        if (step == 0) {
          const int before = (int)(start - a0);
          if (before > 0) base2 = -(int)w.through(before - 1);
        }
        const int lanebase = base2 + (int)(incl - tot);
#define MACKO_ENTRY(k)                                                                    \
  {                                                                                       \
    const uint32_t e = e0 + k;                                                            \
    if (e >= start && e < end && ((lanebase + pos.template offset<k>()) >> 1) >= cols) lane_bad = true; \
  }
        MACKO_ENTRY(0) MACKO_ENTRY(1) MACKO_ENTRY(2) MACKO_ENTRY(3)
        MACKO_ENTRY(4) MACKO_ENTRY(5) MACKO_ENTRY(6) MACKO_ENTRY(7)
#undef MACKO_ENTRY
        base2 += (int)__builtin_amdgcn_readlane((int)incl, 63);
        // a row that runs past the last column keeps running: stop before the positions overflow
        if (__any(lane_bad)) break;
      }
      bad = __any(lane_bad);
    }
    if (bad && lane == 0) atomicMin(first_bad, row);
  }
}

// The dense matrix back, one pass: a wavefront builds its row in LDS (zeros, then the stored
// values at their columns) and writes it out with full-width stores, so every byte of the dense
// matrix is written exactly once and nothing of it is read.  Every wavefront of the workgroup has
// a row buffer of cols values rounded up to 16 bytes.  VB: bits per value (16: fp16, 8: E4M3
// bytes).  VEC: 16-byte stores (dense and ld aligned to 16 bytes, a row a multiple of 16 bytes).
template <int BD, int VB, bool VEC>
__global__ void __launch_bounds__(512)
decode_rows_kernel(const void* __restrict__ values, const uint32_t* __restrict__ deltas,
                   const uint32_t* __restrict__ row_ptr, const int rows, const int cols,
                   void* __restrict__ dense, const int64_t ld) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr int EB = VB / 8;                                  // bytes per value
  const int lane = threadIdx.x & 63;
  const int wave_in_wg = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int waves_per_wg = (int)blockDim.x >> 6;
  const int wave = (int)blockIdx.x * waves_per_wg + wave_in_wg;
  const int nwaves = (int)gridDim.x * waves_per_wg;
  const int chunks = (cols * EB + 15) >> 4;                   // 16-byte chunks of the row buffer
  unsigned char* rowbuf = lds + (size_t)wave_in_wg * chunks * 16;
  uint4* rowbuf4 = reinterpret_cast<uint4*>(rowbuf);
  for (uint32_t row = wave; row < (uint32_t)rows; row += nwaves) {          // wavefront-uniform
    const uint32_t start = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_ptr[row]);
    const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_ptr[row + 1]);
    for (int c = lane; c < chunks; c += 64) rowbuf4[c] = make_uint4(0, 0, 0, 0);
    if (end > start) {
      const uint32_t a0 = start & ~7u;
      const int nsteps = (int)((end - a0 + 511u) >> 9);
      int base2 = 0;
      LaneCodes<BD> wn;                                      // the next step's loads, one step ahead
      LaneValues<VB> vn;
      {
        const uint32_t chunk = min(a0 + 8u * (uint32_t)lane, end - 1u) >> 3;
        wn.load(deltas, chunk);
        vn.load(values, chunk);
      }
      for (int step = 0; step < nsteps; ++step) {
        const uint32_t e0 = a0 + 512u * (uint32_t)step + 8u * (uint32_t)lane;
        LaneCodes<BD> w = wn;
        const LaneValues<VB> v = vn;
        {                                                    // lanes past the row end re-read its last chunk
          const uint32_t chunk = min(e0 + 512u, end - 1u) >> 3;
          wn.load(deltas, chunk);
          vn.load(values, chunk);
        }
        w.keep_if(e0 < end);
        w.decode();
        const LanePositions<BD> pos{w};
        const uint32_t tot = w.total();
        const uint32_t incl = wave_incl_scan_u32(tot);
        if (step == 0) {
          const int before = (int)(start - a0);
          if (before > 0) base2 = -(int)w.through(before - 1);
        }
        const int lanebase = base2 + (int)(incl - tot);
#define MACKO_ENTRY(k)                                                                  \
  {                                                                                     \
    const uint32_t e = e0 + k;                                                          \
    const int col = (lanebase + pos.template offset<k>()) >> 1;                           \
    if (e >= start && e < end && col < cols) {                                          \
      if (VB == 16) reinterpret_cast<uint16_t*>(rowbuf)[col] = (uint16_t)v.template bits<k>(); \
      else rowbuf[col] = (unsigned char)v.template bits<k>();                           \
    }                                                                                   \
  }
        MACKO_ENTRY(0) MACKO_ENTRY(1) MACKO_ENTRY(2) MACKO_ENTRY(3)
        MACKO_ENTRY(4) MACKO_ENTRY(5) MACKO_ENTRY(6) MACKO_ENTRY(7)
#undef MACKO_ENTRY
        base2 += (int)__builtin_amdgcn_readlane((int)incl, 63);
      }
    }
    // the row buffer is private to the wavefront, whose LDS operations complete in order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    unsigned char* out = static_cast<unsigned char*>(dense) + (int64_t)row * ld * EB;
    if (VEC) {
      typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
      for (int c = lane; c < chunks; c += 64) {
        const uint4 t = rowbuf4[c];
        u32x4 q = {t.x, t.y, t.z, t.w};
        __builtin_nontemporal_store(q, reinterpret_cast<u32x4*>(out) + c);
      }
    } else if (VB == 16) {
      for (int c = lane; c < cols; c += 64)
        reinterpret_cast<uint16_t*>(out)[c] = reinterpret_cast<const uint16_t*>(rowbuf)[c];
    } else {
      for (int c = lane; c < cols; c += 64) out[c] = rowbuf[c];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();                         // the buffer is cleared again only after it was read
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// The same for rows that leave too few row buffers in LDS (see long_rows_way), or that do not lie on 16 bytes: the wavefront assembles its row
// a window at a time.  The window is aligned to 16 bytes as the row lies in memory: full-width
// stores whatever the alignment of dense and ld, value by value only at the row's two ends.  A step (512 stored entries)
// that reaches behind the window is put into it in parts, out of registers; what a lane's entries leave outside
// the window lands in a margin in front of it or behind it.
//
// Bound by HBM and by the wavefronts in flight (16 per compute unit; seven row buffers of 22 KB left 7): 4096 x 11008 at
// 50 % 38.5 -> 34.5 us (4.3 TB/s), 1000 x 4093: 7.1 -> 6.1.  Short aligned rows stay with the kernel above (11008 x 4096 at 90 %:
// 20.9 there, 21.5-24 here; 9000 x 300: 4.6 and 5.3: they run each part of the code once or twice, and here is more of it).
// Windows of 2, 4 and 8 KB, and 1 or 2 steps loaded ahead are within 3 % of each other on long rows.
constexpr int kWindowBytes = 8192;
constexpr int kWindowWaves = 4;
constexpr int window_margin(int b_delta, int b_val) { return b_delta == 8 ? 16 : 8 * (1 << b_delta) * (b_val / 8); }

template <int BD, int VB>
__global__ void __launch_bounds__(64 * kWindowWaves)
decode_windows_kernel(const void* __restrict__ values, const uint32_t* __restrict__ deltas,
                      const uint32_t* __restrict__ row_ptr, const int rows, const int cols,
                      unsigned char* __restrict__ dense, const int64_t ld) {
  constexpr int EB = VB / 8;                                  // bytes per value
  // a lane's 8 entries span at most 8 * 2^BD columns; with 8-bit codes they are checked one by one instead
  constexpr int kMargin = window_margin(BD, VB);
  static_assert(kMargin % 16 == 0, "the window starts on a 16-byte boundary");
  constexpr int RING = 2;
  __shared__ __align__(16) unsigned char lds[kWindowWaves * (kMargin + kWindowBytes) + kMargin];   // margin, window, ..., margin
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & 63;
  const int wave_in_wg = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wave = (int)blockIdx.x * kWindowWaves + wave_in_wg;
  const int nwaves = (int)gridDim.x * kWindowWaves;
  unsigned char* win = lds + wave_in_wg * (kWindowBytes + kMargin) + kMargin;
  u32x4* win4 = reinterpret_cast<u32x4*>(win);
  for (int c = lane; c < kWindowBytes / 16; c += 64) win4[c] = u32x4{0, 0, 0, 0};
  for (uint32_t row = wave; row < (uint32_t)rows; row += nwaves) {          // wavefront-uniform
    const uint32_t start = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_ptr[row]);
    const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane((int)row_ptr[row + 1]);
    unsigned char* out = static_cast<unsigned char*>(dense) + (int64_t)row * ld * EB;
    const int skew = (int)(reinterpret_cast<uintptr_t>(out) & 15);          // bytes of the first 16 that are not the row's
    out -= skew;
    const int64_t row_end = skew + (int64_t)cols * EB;       // in bytes from the aligned start
    int64_t at = 0;                                          // first byte of the window
    int put_end = 0;                                         // no entry was put at this byte or behind it
    auto flush = [&]() {
      // the window is private to the wavefront, whose LDS operations complete in order
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int from = at == 0 ? skew : 0, to = (int)min(row_end - at, (int64_t)kWindowBytes);       // the row's bytes
      unsigned char* to_mem = out + at;
      if ((from | to) & 15) {                                // values of the row in a 16-byte piece that is not all its own
        constexpr int kPiece = 16 / EB;
        const int p = lane < kPiece ? (from & ~15) + EB * lane : (to & ~15) + EB * (lane - kPiece);
        if (lane < 2 * kPiece && p >= from && p < to) {
          if (VB == 16) *reinterpret_cast<uint16_t*>(to_mem + p) = *reinterpret_cast<const uint16_t*>(win + p);
          else to_mem[p] = win[p];
        }
      }
      // Behind a right row's end the window holds zeros.  An entry at or beyond the last column (a wrong encoding) goes no
      // further than this row.
      const int clear_to = max(to, min(put_end - (int)at, kWindowBytes));
      for (int lo = 16 * lane; lo < clear_to; lo += 1024) {
        const u32x4 t = win4[lo >> 4];
        win4[lo >> 4] = u32x4{0, 0, 0, 0};
        if (lo >= from && lo + 16 <= to) __builtin_nontemporal_store(t, reinterpret_cast<u32x4*>(to_mem + lo));
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      at += kWindowBytes;
    };
    if (end > start) {
      const uint32_t a0 = start & ~7u;
      const int nsteps = (int)((end - a0 + 511u) >> 9);
      LaneCodes<BD> wq[RING];
      LaneValues<VB> vq[RING];
      auto issue = [&](int j, int step) {                    // lanes past the row end re-read its last chunk
        const uint32_t chunk = min(a0 + 512u * (uint32_t)step + 8u * (uint32_t)lane, end - 1u) >> 3;
        wq[j].load(deltas, chunk);
        vq[j].load(values, chunk);
      };
#pragma unroll
      for (int j = 0; j < RING; ++j) issue(j, min(j, nsteps - 1));
      int base2 = 0;                                         // doubled position behind the steps so far
      for (int step0 = 0; step0 < nsteps; step0 += RING) {
#pragma unroll
        for (int j = 0; j < RING; ++j) {
          const int step = step0 + j;
          if (step >= nsteps) break;
          const uint32_t e0 = a0 + 512u * (uint32_t)step + 8u * (uint32_t)lane;
          LaneCodes<BD> w = wq[j];
          LaneValues<VB> v = vq[j];
          issue(j, min(step + RING, nsteps - 1));
          if (step == nsteps - 1) {                          // what lies behind the row's end is put as zeros
            const uint32_t nv = e0 < end ? end - e0 : 0u;
            w.keep_if(nv != 0);
            v.keep_first(nv);
          }
          w.decode();
          const LanePositions<BD> pos{w};
          const uint32_t tot = w.total();
          const uint32_t incl = wave_incl_scan_u32(tot);
          if (step == 0) {                                   // entries of the previous row land in front of column 0
            const int before = (int)(start - a0);
            if (before > 0) base2 = -(int)w.through(before - 1);
          }
          const int lanebase = base2 + (int)(incl - tot);
          base2 += (int)__builtin_amdgcn_readlane((int)incl, 63);
          for (;;) {
            const int rel = skew + (lanebase >> (VB == 8 ? 1 : 0)) - (int)at;    // the lane's first column in the window
            if (BD != 8) {
              // Lanes entirely outside write to the margin.  What is put behind the row's end is zero, and what the
              // previous row's entries put in front of a row that does not start on 16 bytes is not written out.
              unsigned char* p = win + ((uint32_t)(rel + kMargin) < (uint32_t)(kWindowBytes + kMargin) ? rel : -kMargin);
#define MACKO_PUT(K)                                                                                          \
  if (VB == 16) *reinterpret_cast<uint16_t*>(p + pos.template offset<K>()) = (uint16_t)v.template bits<K>();      \
  else p[pos.template offset<K>() >> 1] = (unsigned char)v.template bits<K>();
              MACKO_PUT(0) MACKO_PUT(1) MACKO_PUT(2) MACKO_PUT(3) MACKO_PUT(4) MACKO_PUT(5) MACKO_PUT(6) MACKO_PUT(7)
#undef MACKO_PUT
            } else {
#define MACKO_PUT(K)                                                                                          \
  {                                                                                                           \
    const int q = rel + pos.template offset<K>();                                                                \
    if (e0 + K >= start && e0 + K < end && q >= 0 && q < kWindowBytes)                                         \
      *reinterpret_cast<uint16_t*>(win + q) = (uint16_t)v.template bits<K>();                                  \
  }
              MACKO_PUT(0) MACKO_PUT(1) MACKO_PUT(2) MACKO_PUT(3) MACKO_PUT(4) MACKO_PUT(5) MACKO_PUT(6) MACKO_PUT(7)
#undef MACKO_PUT
            }
            if (at + kWindowBytes >= row_end || skew + (base2 >> (VB == 8 ? 1 : 0)) <= at + kWindowBytes) break;
            flush();
          }
        }
      }
      // the lanes behind the row's last entry went on by 8 columns each; that entry's own lane by the codes behind it as well
      const int idle = 63 - (int)((end - 1u - (a0 + 512u * (uint32_t)(nsteps - 1))) >> 3);
      put_end = skew + ((base2 - 16 * idle) >> (VB == 8 ? 1 : 0));
    }
    while (at < row_end) flush();
  }
}

template <int BD, int VB>
int launch_decode_windows_bd(const SpmvProblem& p, void* dense, int64_t ld, hipStream_t stream) {
  const int64_t waves_wanted = std::min<int64_t>(p.rows, (int64_t)device_cu_count() * 32);
  const dim3 grid((unsigned)((waves_wanted + kWindowWaves - 1) / kWindowWaves));
  hipLaunchKernelGGL((decode_windows_kernel<BD, VB>), grid, dim3(64 * kWindowWaves), 0, stream,
                     static_cast<const void*>(p.values), reinterpret_cast<const uint32_t*>(p.deltas), p.row_ptr,
                     (int)p.rows, (int)p.cols, static_cast<unsigned char*>(dense), ld);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? MACKO_OK : hip_fail(e);
}

template <int BD, int VB>
int launch_decode_rows_bd(const SpmvProblem& p, void* dense, int64_t ld, bool vec, int waves_per_wg, int64_t lds_bytes,
                          hipStream_t stream) {
  const int block = 64 * waves_per_wg;
  const int64_t waves_wanted = std::min<int64_t>(p.rows, (int64_t)device_cu_count() * 32);
  const dim3 grid((unsigned)((waves_wanted + waves_per_wg - 1) / waves_per_wg));
  const uint32_t* deltas = reinterpret_cast<const uint32_t*>(p.deltas);
  auto kfn = vec ? decode_rows_kernel<BD, VB, true> : decode_rows_kernel<BD, VB, false>;
  if (lds_bytes > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds_bytes);
    if (e != hipSuccess) return hip_fail(e);
  }
  hipLaunchKernelGGL(kfn, grid, dim3(block), (size_t)lds_bytes, stream, static_cast<const void*>(p.values), deltas,
                     p.row_ptr, (int)p.rows, (int)p.cols, dense, ld);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? MACKO_OK : hip_fail(e);
}

template <bool DENSE>
int launch_expand(const SpmvProblem& p, int32_t* cols_out, uint16_t* dense, int64_t ld, hipStream_t stream) {
  const int64_t waves_wanted = std::min<int64_t>(p.rows, (int64_t)device_cu_count() * 64);
  const dim3 grid((unsigned)((waves_wanted + kExpandBlock / 64 - 1) / (kExpandBlock / 64))), block(kExpandBlock);
  auto kfn = p.b_delta == 1 ? expand_kernel<1, DENSE> : p.b_delta == 2 ? expand_kernel<2, DENSE>
             : p.b_delta == 4 ? expand_kernel<4, DENSE> : p.b_delta == 8 ? expand_kernel<8, DENSE> : nullptr;
  if (!kfn) return MACKO_E_UNSUPPORTED;
  hipLaunchKernelGGL(kfn, grid, block, 0, stream, static_cast<const void*>(p.values),
                     reinterpret_cast<const uint32_t*>(p.deltas), p.row_ptr, (int)p.rows, (int)p.cols, cols_out, dense, ld);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? MACKO_OK : hip_fail(e);
}

// Clears the matrix, then scatters the stored values (two kernels in stream order).
int launch_clear_and_scatter(const SpmvProblem& p, uint16_t* dense, int64_t ld, bool vec, hipStream_t stream) {
  const int64_t stores = p.rows * (vec ? p.cols / 8 : p.cols);
  const int64_t wgs = std::min<int64_t>((stores + 255) / 256, (int64_t)device_cu_count() * 32);
  hipLaunchKernelGGL(vec ? zero_rows_kernel<true> : zero_rows_kernel<false>, dim3((unsigned)wgs), dim3(256), 0, stream, dense,
                     (int)p.rows, (int)p.cols, ld);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e);
  return p.pad_nnz == 0 ? MACKO_OK : launch_expand<true>(p, nullptr, dense, ld, stream);
}

// How a matrix whose rows leave fewer than 8 row buffers per compute unit is decoded.  The windows have 16 wavefronts in
// flight per compute unit whatever the row's length, but visit every window of the row one after the other, and with 8-bit codes check
// each entry against it.  All times are in windows over the other way, rows on 16 bytes, 16-bit values (8-bit values are
// within 10 % either way and take the windows).
enum class LongRows { kWindows, kBuffers, kScatter };
LongRows long_rows_way(const SpmvProblem& p, int64_t per_cu, bool vec) {
  if (p.b_val != 16) return LongRows::kWindows;
  const int64_t room = (int64_t)device_cu_count() * per_cu;
  const double density = (double)p.pad_nnz / (double)p.rows / (double)p.cols;
  if (per_cu > 0) {
    // row buffers, all rows at once (4096 x 11008 at 50 %: 0.83; otherwise 0.53 ... 0.98)
    if (!vec || p.rows > room) return LongRows::kWindows;
    if (p.b_delta == 8) return LongRows::kBuffers;                           // 1.02 ... 1.42, 16 x 40000: 1.37
    if (p.b_delta < 4) return 2 * p.rows >= room ? LongRows::kBuffers : LongRows::kWindows;   // 1500 x 11008: 1.21; 256 x 11008: 0.88
    if (density < 0.08 && per_cu <= 5) return LongRows::kBuffers;            // hardly more than padding: 1.00 ... 1.17
    return per_cu <= 4 && 4 * p.rows >= 3 * room ? LongRows::kBuffers : LongRows::kWindows;   // 512 x 40000 at 93 %: 1.20; 256: 1.00
  }
  // rows longer than LDS: a few sparse ones are sooner cleared by the whole chip and scattered into
  const double most = p.b_delta == 8 ? (p.rows <= 2 ? 0.25 : p.rows <= 64 ? 0.11 : p.rows <= 128 ? 0.06 : p.rows <= 256 ? 0.025 : 0.0)
                                     : (p.rows <= 2 ? 0.13 : p.rows <= 16 ? 0.07 : 0.0);
  return density < most ? LongRows::kScatter : LongRows::kWindows;           // 4 x 100000, 98 %, 8-bit codes: 2.54; 256 x 100000: 1.05
}

}  // namespace

int launch_check(const SpmvProblem& p, unsigned int* first_bad, hipStream_t stream) {
  const int64_t waves_wanted = std::min<int64_t>(p.rows, (int64_t)device_cu_count() * 64);
  const dim3 grid((unsigned)((waves_wanted + kExpandBlock / 64 - 1) / (kExpandBlock / 64))), block(kExpandBlock);
  const uint32_t* deltas = reinterpret_cast<const uint32_t*>(p.deltas);
  switch (p.b_delta) {
    case 1:
      hipLaunchKernelGGL(check_kernel<1>, grid, block, 0, stream, deltas, p.row_ptr, (int)p.rows, (int)p.cols,
                         (uint32_t)p.pad_nnz, first_bad);
      break;
    case 2:
      hipLaunchKernelGGL(check_kernel<2>, grid, block, 0, stream, deltas, p.row_ptr, (int)p.rows, (int)p.cols,
                         (uint32_t)p.pad_nnz, first_bad);
      break;
    case 4:
      hipLaunchKernelGGL(check_kernel<4>, grid, block, 0, stream, deltas, p.row_ptr, (int)p.rows, (int)p.cols,
                         (uint32_t)p.pad_nnz, first_bad);
      break;
    case 8:
      hipLaunchKernelGGL(check_kernel<8>, grid, block, 0, stream, deltas, p.row_ptr, (int)p.rows, (int)p.cols,
                         (uint32_t)p.pad_nnz, first_bad);
      break;
    default:
      return MACKO_E_UNSUPPORTED;
  }
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? MACKO_OK : hip_fail(e);
}

int launch_columns(const SpmvProblem& p, int32_t* cols_out, hipStream_t stream) {
  if (p.rows == 0 || p.pad_nnz == 0) return MACKO_OK;
  return launch_expand<false>(p, cols_out, nullptr, 0, stream);
}

int launch_decode(const SpmvProblem& p, void* dense_any, int64_t ld, hipStream_t stream) {
  if (p.rows == 0 || p.cols == 0) return MACKO_OK;
  const int eb = p.b_val / 8;                                // bytes per value
  const bool vec = (p.cols * eb) % 16 == 0 && (ld * eb) % 16 == 0 && (reinterpret_cast<uintptr_t>(dense_any) & 15) == 0;
  const int64_t row_bytes = 16 * ((p.cols * eb + 15) / 16);
  constexpr int64_t kLdsLimit = 160 * 1024;
  // 8-bit rows of more than 163840 columns: no kernel below has that limit any more, but the interface states it
  if (p.b_val == 8 && row_bytes > kLdsLimit) return MACKO_E_UNSUPPORTED;
  if (p.b_val == 8 && p.b_delta != 4) return MACKO_E_UNSUPPORTED;           // 8-bit values come with 4-bit codes
  // Row buffers per compute unit: at least 8 (4096 x 11008 has 7: 38.5 us, in windows 34.5; 9000 columns have 8: 9.8 us for 2000
  // rows, in windows 10.3), and rows on 16 bytes unless they are short (1000 x 4093: 7.1 and 6.1; 9000 x 300: 4.6 and 5.3).
  const int64_t per_cu = kLdsLimit / row_bytes;
  LongRows way = LongRows::kBuffers;
  if (per_cu < 8) way = long_rows_way(p, per_cu, vec);
  else if (!vec && row_bytes >= 2048) way = LongRows::kWindows;
  if (way == LongRows::kScatter) return launch_clear_and_scatter(p, static_cast<uint16_t*>(dense_any), ld, vec, stream);
  if (way == LongRows::kWindows) {
    if (p.b_val == 8) return launch_decode_windows_bd<4, 8>(p, dense_any, ld, stream);
    switch (p.b_delta) {
      case 1: return launch_decode_windows_bd<1, 16>(p, dense_any, ld, stream);
      case 2: return launch_decode_windows_bd<2, 16>(p, dense_any, ld, stream);
      case 4: return launch_decode_windows_bd<4, 16>(p, dense_any, ld, stream);
      case 8: return launch_decode_windows_bd<8, 16>(p, dense_any, ld, stream);
      default: return MACKO_E_UNSUPPORTED;
    }
  }
  // one pass through a row buffer in LDS per wavefront, in workgroups of 4 wavefronts or one workgroup per compute unit
  const int waves_per_wg = per_cu >= 8 ? 4 : (int)per_cu;
  const int64_t lds_bytes = row_bytes * waves_per_wg;
  if (p.b_val == 8) return launch_decode_rows_bd<4, 8>(p, dense_any, ld, vec, waves_per_wg, lds_bytes, stream);
  switch (p.b_delta) {
    case 1: return launch_decode_rows_bd<1, 16>(p, dense_any, ld, vec, waves_per_wg, lds_bytes, stream);
    case 2: return launch_decode_rows_bd<2, 16>(p, dense_any, ld, vec, waves_per_wg, lds_bytes, stream);
    case 4: return launch_decode_rows_bd<4, 16>(p, dense_any, ld, vec, waves_per_wg, lds_bytes, stream);
    case 8: return launch_decode_rows_bd<8, 16>(p, dense_any, ld, vec, waves_per_wg, lds_bytes, stream);
    default: return MACKO_E_UNSUPPORTED;
  }
}

}  // namespace macko
