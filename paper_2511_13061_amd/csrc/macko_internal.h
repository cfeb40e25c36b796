// Internal declarations shared by the translation units of libmacko.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "macko.h"

namespace macko {

constexpr int kDeltaBits = 4;           // default b_delta
// entries per 16 bytes of packed codes: both arrays are padded to a multiple of this
constexpr int64_t alloc_granule(int b_delta) { return 128 / b_delta; }

struct Tuning {
  int64_t spmv_kernel = 0;
  int64_t spmv_lanes = 0;
  int64_t spmv_block = 0;
  int64_t spmv_rows_per_wg = 0;
  int64_t spmv_ring = 0;
  int64_t spmv_resident = 0;      // 0 auto, 1 never, 2 always one resident round of workgroups
  int64_t spmv_wgs_per_cu = 0;    // resident round: workgroups per compute unit (0 = planner's choice)
  int64_t spmv_steps_per_wave = 0; // many-workgroup regime: steps of work per wavefront (0 = default)
  int64_t spmv_step_align = 0;     // entries a row's first step is aligned to (8 ... 512, power of two; 0 = by row length)
  int64_t spmv_resident_steps = 0; // largest work (steps per compute unit) launched as one resident round (0 = default)
  int64_t spmm_kernel = 0;         // batches that both ways serve: 0 the faster one, 1 vector units, 2 matrix cores
  int64_t chain_wait_us = 0;       // longest wait of a chain's workgroups for each other (0 = default, -1 = none)
  int64_t chain_no_wait = 0;       // 1: such a wait gives up at once when the phase before is unfinished
  int64_t gemv_block = 0;
  int64_t gemv_rows_per_wg = 0;
  int64_t gemv_ring = 0;
  int64_t gemv_resident = 0;
  int64_t gemv_wgs_per_cu = 0;
};
Tuning& tuning();

// record a failing HIP call for macko_last_hip_error()
int hip_fail(hipError_t e);
#define MACKO_HIP_TRY(expr)                                   \
  do {                                                        \
    hipError_t e__ = (expr);                                  \
    if (e__ != hipSuccess) return ::macko::hip_fail(e__);     \
  } while (0)

int device_cu_count();

// ---- LDS of the product kernels -----------------------------------------------
// The activation vector x sits in LDS between two zero-filled guard regions:
//   [0, front) zeros | x[0 .. C) | zeros up to the end of the allocation.
// Entries that a lane loads but that belong to a neighbouring row decode to
// positions just before column 0 or after the row's last column; the guards
// make those reads return +0 so that they contribute nothing.
// Front guard: a row's first chunk holds at most 7 entries of the previous row,
// each at most 2^b_delta columns wide (224 bytes before x[0] for 4-bit codes,
// 3584 for 8-bit ones).  Back guard: in a row's last step the lanes past the row
// end advance by one column per entry, plus at most 7 real deltas in the lane
// that straddles the end (at most 504 + 7 * 2^b_delta columns); the dense kernel
// reads at most 62 16-byte chunks past the end.
constexpr int kFrontPad = 256;   // bytes, codes of up to 4 bits (and the dense kernel)
constexpr int kBackPad = 1280;   // bytes

constexpr int front_pad_for(int b_delta) { return b_delta <= 4 ? kFrontPad : 3584; }
constexpr int back_pad_for(int b_delta) { return b_delta <= 4 ? kBackPad : 4608; }

constexpr int64_t lds_bytes_for(int64_t cols, int b_delta = 4) {
  return front_pad_for(b_delta) + 16 * ((cols + 7) / 8) + back_pad_for(b_delta);
}

constexpr int kMaxStepAlign = 512;      // what the "spmv_step_align" knob may ask for
// The sparse product may begin a row up to kMaxStepAlign entries early (see macko_spmv.hip): its cleared lanes in front of a
// row advance 16 bytes each below x[0], and the front guard grows by that.
constexpr int kAlignFrontPad = 2 * kMaxStepAlign;
constexpr int spmv_front_pad(int b_delta) { return front_pad_for(b_delta) + kAlignFrontPad; }
constexpr int64_t spmv_lds_bytes(int64_t cols, int b_delta) { return lds_bytes_for(cols, b_delta) + kAlignFrontPad; }
constexpr int64_t kMaxLdsBytes = 160 * 1024 - 64;   // 160 KB per CU minus the static row counter
constexpr int64_t kWideLdsBytes = 36 * 1024;        // an x copy of at least this makes a matrix "wide" for the launch planner

// launchers implemented in the .hip files; all return a macko_status
constexpr int kMaxGroup = 8;            // MACKO_MAX_GROUP
constexpr int kMaxWide = 32;            // products in one launch of macko_spmv_many

struct SpmvProblem {
  const uint16_t* values;
  const uint8_t* deltas;
  const uint32_t* row_ptr;
  int64_t rows, cols, pad_nnz;
  const void* x;
  void* y;
  int b_delta = kDeltaBits;
  int b_val = 16;           // bits per value: 16 (fp16) or 8 (E4M3)
};
struct GemvProblem {
  const void* W;
  int64_t rows, cols, ld;
  const void* x;
  void* y;
};
// n independent products, as few kernel launches as the shapes allow (1 <= n <= kMaxGroup; kMaxWide for the sparse product).
// in_call: products of the caller's call, which may take several launches (n <= in_call).  The kernel is chosen by it and not by n, so that
// a product takes the same one in whichever launch of the call it lands.
int launch_spmv_group(int n, const SpmvProblem* problems, int64_t in_call, hipStream_t stream);
// Stored entries per row on average from which a product takes the wave-per-row kernel.  A row takes a wavefront one step of up to 512
// entries, however short it is; the sub-wave kernel takes its rows 4 at a time, but one launch to a product, whose start is longer.
// Measured on 5600 calls, both kernels on the same matrices in graphs of 20 to 40 calls: 100 to 45000 rows, 100 to 60000 columns, 4 to 300 entries a
// row, all code widths.  One product: by rows per compute unit, within 0.14 % of the better kernel in the mean, 1.14 at worst (us, sub-wave /
// wave-per-row: 1000 x 40 2.9 / 2.9, 2046 x 109 3.7 / 3.1, 5318 x 119 4.1 / 5.0, 7174 x 113 4.0 / 5.6, 7460 x 172 4.7 / 5.9, 30064 x 245 9.0 / 10.5).
// 8-bit codes with few rows: the larger zero guards cost the wave-per-row kernel what its start saves (693 x 82 3.3 / 3.6).
// in_call > 1, several products of a call: the wave-per-row kernel takes them in one launch, which counts for more the more they are (4 of
// 504 x 43 12.5 / 3.4, 2 of 13186 x 58 7.4 / 10.7, 4 of 14499 x 6 16.6 / 23.4, 8 of 17902 x 208 54 / 33, 8 of 17747 x 44 38 / 33): within
// 0.2 to 0.4 % in the mean, 1.37 at worst.
constexpr int64_t kWaveRowMinEntries = 192;            // where nothing more is known of the call
inline int64_t wave_row_min_entries(const SpmvProblem& p, int64_t in_call) {
  constexpr int64_t kLargest = 248;
  if (p.pad_nnz >= kLargest * p.rows) return kLargest;   // no need to ask which device it is (0.08 us of a small call's 3.4)
  const int64_t per_cu = p.rows / device_cu_count();
  if (in_call <= 1) {
    if (per_cu < 4) return p.b_delta == 8 ? 104 : 1;
    return per_cu < 16 ? 104 : per_cu < 48 ? 200 : kLargest;
  }
  if (per_cu < (p.b_delta == 8 ? 20 : 24) + 6 * std::min<int64_t>(in_call, 8)) return 1;
  return per_cu < (in_call == 2 ? 72 : 80) ? 104 : in_call == 2 ? 208 : 136;
}
// Whether the product goes to the wave-per-row kernel (8-bit values: it has to).
inline bool spmv_takes_wave_row(const SpmvProblem& p, int64_t min_entries = kWaveRowMinEntries) {
  if (p.rows == 0 || p.pad_nnz == 0 || spmv_lds_bytes(p.cols, p.b_delta) > kMaxLdsBytes) return false;
  if (p.b_val == 8) return p.b_delta == 4;
  const int64_t knob = tuning().spmv_kernel;
  return knob != 0 ? knob == 2 : p.pad_nnz / p.rows >= min_entries || min_entries <= 1;
}
// 0: the product may need a launch of its own, or a kernel that a knob asks for; products whose numbers differ in bit 0 at
// most fit one launch of the wave-per-row kernel.  Bit 0: a wide x.
inline int spmv_launch_class(const SpmvProblem& p, int64_t min_entries = kWaveRowMinEntries) {
  const Tuning& t = tuning();
  if (!spmv_takes_wave_row(p, min_entries) || t.spmv_kernel != 0 || (t.spmv_ring != 0 && t.spmv_ring != 2)) return 0;
  return 2 * (p.b_val * 16 + p.b_delta) + (spmv_lds_bytes(p.cols, p.b_delta) - kAlignFrontPad >= kWideLdsBytes ? 1 : 0);
}
int launch_gemv_group(int n, const GemvProblem* problems, hipStream_t stream);
// phases of products in one launch, phase p + 1 after phase p: sizes[p] products in phase p, listed in
// phase order; `scratch` is chain_scratch_bytes() of zeroed device memory that the launch leaves zeroed
int launch_spmv_chain(int n_phases, const int* sizes, const SpmvProblem* problems, uint32_t* scratch,
                      uint32_t wait_ticks, hipStream_t stream);
constexpr int64_t chain_scratch_bytes() { return 8192; }
// device address, on the current device, of the library's own chain scratch (a static device array)
int chain_static_scratch(uint32_t** out);
constexpr int chain_error_word() { return 25 * 64; }
// batch products with one matrix: Y[b] = W X[b], vectors ldx / ldy elements apart (p.x, p.y unused)
int launch_spmm(const SpmvProblem& p, const void* X, int64_t ldx, void* Y, int64_t ldy, int batch,
                hipStream_t stream);
// the same on the matrix cores: which calls it can serve (any batch up to 64), and the launch
bool spmm_tile_serves(const SpmvProblem& p, int64_t ldx);
// Whether vectors share passes over the matrix on the vector units, in pieces of 8, 4 and 2, instead of going as single products in groups:
// rows of at least kLongRow stored entries.  Shorter ones with codes of up to 4 bits go to the matrix cores from a few vectors on; with 8-bit
// codes, which those do not serve, they share passes as well where the vectors are copied 8 columns at a time and there are rows enough to pay for a
// workgroup's copy of 2, 4 or 8 of them.  Both ways timed on 2563 calls of 200 to 30000 rows, 64 to 45000 columns, 2 to 16 vectors: 0.3 % from the faster
// one in the mean, 1.21 at worst; the line is a number of columns per row of a compute unit, and lower where four copies do not fit LDS (us, single products / pieces: 9232 x 1152 with 71 entries, 2 vectors 8.0 / 5.3, 17 54 / 22; 4096 x 4096 with 287, 5 9.1 / 7.2;
// 2048 x 16384 with 208, 3, 5 and 16 5.4 / 7.7, 7.7 / 11.9 and 15.8 / 34.2; 4096 x 16384, 3 and 8 8.0 / 8.7 and 13.1 / 18.4).
constexpr int64_t kLongRow = 384;
inline bool spmm_shares_passes(const SpmvProblem& p, int batch) {
  if (p.pad_nnz / p.rows >= kLongRow) return true;
  if (p.b_delta != 8 || p.cols % 8 != 0) return false;
  const int64_t cus = device_cu_count(), most = batch <= 2 ? 1500 : batch <= 4 && p.cols <= 16368 ? 1200 : 650;
  return p.rows >= 4 * cus && p.cols * cus <= most * p.rows;
}
int64_t spmm_tile_windows(const SpmvProblem& p);       // windows that a workgroup goes through, of up to 16 vectors
bool spmm_tile_pairs_groups(const SpmvProblem& p, int batch);      // two groups of columns share an operand there
// Units of `per_unit` entries that a wavefront takes of a row there, from the 8 entries its start lies in; one, all cleared, for a row
// without entries, and for row pointers that decrease (no encoding's: the difference would be a row of 2^32 entries).
constexpr uint32_t panel_row_units(uint32_t start, uint32_t end, uint32_t per_unit) {
  return end > start ? (end - (start & ~7u) + per_unit - 1u) / per_unit : 1u;
}
// ---- rows of the vector kernels ------------------------------------------------
struct RowCursor {
  int i;               // row index within the wavefront's rows (== nb when exhausted)
  uint32_t start, end; // its entry range
  uint32_t a0;         // start rounded down to the alignment: where the row's first step begins
  int nsteps, step;
};
// Move the cursor to the first non-empty row at or after cur.i of nb, whose pointers lo(i) and hi(i) give.
// amask + 1 is the alignment of the row's first step in entries: 8 is the reverse-offset
// alignment of the paper (a lane's 16-byte chunk never straddles the row start); larger powers
// of two up to 512 make every step of the row begin on a multiple of that many entries.
// TAILS: a last step of one chunk (behind at least one other step) is left out, see row_tail.
// Behind the last row the range is empty, at entry 0, whatever the last pointers are: the buffer opened on it (buffer_entries) holds nothing.
// Left as they are, pointers that decrease there (no encoding's) made one of 2^32 entries.
template <bool TAILS, class Lo, class Hi>
__attribute__((always_inline)) constexpr void seek_row(RowCursor& cur, int nb, const Lo& lo, const Hi& hi, uint32_t amask) {
  cur.start = cur.end = 0;
  while (cur.i < nb) {
    cur.start = lo(cur.i);
    cur.end = hi(cur.i);
    if (cur.end > cur.start) break;
    ++cur.i;
    cur.start = cur.end = 0;
  }
  cur.a0 = cur.start & ~amask;
  const uint32_t len = cur.end - cur.a0;
  cur.nsteps = (int)((len + 511u - (TAILS && len > 512u ? 8u : 0u)) >> 9);
  cur.step = 0;
}
// What the buffers hold that these kernels read a row through, from chunk c0 (8 entries, the row's first or an earlier one) to entry `end`:
// entries, and their bytes (ends are checked per 4 bytes, and codes are read by chunks).
constexpr uint32_t buffer_entries(uint32_t c0, uint32_t end) { return end - (c0 << 3); }
constexpr uint32_t buffer_value_bytes(uint32_t entries, int b_val) { return (entries * (uint32_t)(b_val / 8) + 3u) & ~3u; }
constexpr uint32_t buffer_code_bytes(uint32_t entries, int b_delta) { return ((entries + 7u) >> 3) * (uint32_t)b_delta; }
// The tails of 8-bit rows are read through the arrays as a whole: a lane that has one reads the last chunk of its own row, wherever that is;
// the others, at the last chunk below 2^32 bytes, are behind the end (the launchers take fewer than 2^32 - 4096 entries).
struct TailBuffer {
  uint32_t c0, end;
};
constexpr TailBuffer tail_buffer() { return {0u, 0xFFFFFFE0u}; }
int launch_spmm_tile(const SpmvProblem& p, const uint16_t* X, int64_t ldx, uint16_t* Y, int64_t ldy, int batch,
                     hipStream_t stream);
// bytes of the encoder's block: values, codes and row pointers, each from a multiple of 256 bytes on
struct EncodedLayout {
  size_t deltas, row_ptr, total;
};
constexpr EncodedLayout encoded_layout(int64_t rows, int64_t alloc_nnz, int b_delta, int b_val) {
  const size_t deltas = ((size_t)alloc_nnz * (b_val / 8) + 255) / 256 * 256;
  const size_t row_ptr = deltas + ((size_t)alloc_nnz * b_delta / 8 + 255) / 256 * 256;
  return {deltas, row_ptr, row_ptr + 4 * (size_t)(rows + 1)};
}
// device-side expansion: column index of every stored entry; the dense matrix back
int launch_columns(const SpmvProblem& p, int32_t* cols_out, hipStream_t stream);
// structural check of bound device arrays; *first_bad (device) must hold `rows` beforehand
int launch_check(const SpmvProblem& p, unsigned int* first_bad, hipStream_t stream);
int launch_decode(const SpmvProblem& p, void* dense, int64_t ld, hipStream_t stream);
// Device memory of the encoder's handles.  A block that macko_destroy releases is kept for the next handle of its size, a few
// per device: block_bytes rounds a size up (by 1.6 % at most) so that matrices of one shape share one although their entry counts differ a little.
constexpr size_t kStoredBlockMin = size_t{2} << 20;    // smaller ones cost hipMalloc and hipFree 0.4 us
constexpr size_t kStoredBytes = size_t{256} << 20;     // kept per device, at most
constexpr size_t block_bytes(size_t bytes) {
  if (bytes < kStoredBlockMin) return bytes ? bytes : 16;
  size_t granule = kStoredBlockMin / 64;
  while (granule * 128 <= bytes) granule *= 2;
  return (bytes + granule - 1) / granule * granule;
}
constexpr bool block_is_kept(size_t bytes) { return block_bytes(bytes) >= kStoredBlockMin && block_bytes(bytes) <= kStoredBytes; }
// hipMalloc on the current device for all that the library allocates: when it fails, what is kept there is given back and it tries again.
hipError_t device_malloc(void** p, size_t bytes);
// A block of block_bytes(bytes) on the current device.  It is kept only with an idle_probe, a small allocation on its device, which goes with it.
hipError_t block_acquire(void** block, size_t bytes);
void block_release(void* block, size_t bytes, int device, void* idle_probe);
void block_trim(int device);                           // frees what is kept
// GPU encoder: counting pass + fill pass.  The three arrays are parts of one *block (block_acquire).
int encode_on_device(const void* dense, int64_t rows, int64_t cols, int64_t ld, int b_delta, int b_val,
                     hipStream_t stream, void** block,
                     void** values, uint8_t** deltas, uint32_t** row_ptr, int64_t* nnz,
                     int64_t* pad_nnz, int64_t* alloc_nnz, int64_t* empty_rows,
                     int64_t* max_row_entries);

void fill_report(macko_report_t* rep, int64_t rows, int64_t cols, int64_t nnz, int64_t pad_nnz,
                 int64_t alloc_nnz, int64_t empty_rows, int64_t max_row_entries, int b_delta, int b_val = 16);

}  // namespace macko

struct macko_matrix {
  int64_t rows = 0, cols = 0;
  int64_t pad_nnz = 0, alloc_nnz = 0;
  int b_delta = macko::kDeltaBits;
  int b_val = 16;            // 16: fp16 values; 8: OCP E4M3 values (h_values8 holds the host copy)
  macko_report_t report{};
  // host copy (empty for device-encoded and wrapped handles)
  bool has_host = false;
  std::vector<uint16_t> h_values;
  std::vector<uint8_t> h_values8;
  std::vector<uint8_t> h_deltas;
  std::vector<uint32_t> h_row_ptr;
  // device binding
  const uint16_t* d_values = nullptr;
  const uint8_t* d_deltas = nullptr;
  const uint32_t* d_row_ptr = nullptr;
  bool bound = false;
  bool owns_device = false;
  void* d_block = nullptr;   // owns_device: the one allocation that holds the three arrays,
  int d_block_device = -1;   // its device, and a small allocation that block_release waits with
  void* d_idle_probe = nullptr;
};
