// Small-batch product Y = W X^T for the MACKO format on gfx950: the same
// wavefront-per-row streaming kernel as the matrix-vector product (Section 4.4
// of the paper), with the decode done once per stored entry and reused for
// BT = 2, 4 or 8 activation vectors, for every code width and for 16- and 8-bit values.  The paper leaves matrix-matrix products
// with small batch dimensions as future work (Section 7); this is the natural
// extension: the streamed bytes per entry stay 2.5, the arithmetic per byte
// grows with the batch.
//
// LDS holds the activations interleaved by column: the BT values of column c
// are adjacent (2*BT bytes), so one gather address per entry fetches all of
// them with a single ds_read_b32 / b64 / b128.  Guards of zeros in front of and
// behind the columns play the same role as in the matrix-vector kernel.
#include "macko_decode.h"
#include "macko_device.h"
#include "macko_internal.h"
#include "macko_plan.h"

#include <algorithm>
#include <climits>
#include <cmath>

namespace macko {
namespace {

template <int BT> struct XVec;
template <> struct XVec<2> { using type = uint32_t; };
template <> struct XVec<4> { using type = uint2; };
template <> struct XVec<8> { using type = uint4; };

template <int BT>
__device__ __forceinline__ void unpack_x(const typename XVec<BT>::type& v, float* out);
template <>
__device__ __forceinline__ void unpack_x<2>(const uint32_t& v, float* out) {
  out[0] = f16_bits_to_f32((uint16_t)(v & 0xFFFFu));
  out[1] = f16_bits_to_f32((uint16_t)(v >> 16));
}
template <>
__device__ __forceinline__ void unpack_x<4>(const uint2& v, float* out) {
  unpack_x<2>(v.x, out);
  unpack_x<2>(v.y, out + 2);
}
template <>
__device__ __forceinline__ void unpack_x<8>(const uint4& v, float* out) {
  unpack_x<2>(v.x, out);
  unpack_x<2>(v.y, out + 2);
  unpack_x<2>(v.z, out + 4);
  unpack_x<2>(v.w, out + 6);
}

// Copy X (batch vectors of `cols` fp16, vector b at X + b*ldx) into LDS, interleaved
// by column, between zero guards of front_pad*BT and back_pad*BT bytes.  Vectors
// b >= batch are filled with zeros.  In two parts, so that the kernel can send its
// first streaming loads between them: begin() only issues the global loads of the
// thread's first 8 columns into registers; finish() writes them to LDS, copies the
// rest, clears the guards and ends with a barrier.  Both are called by every thread.
template <int BT>
struct XStageBatch {
  uint32_t u[BT][4];      // vector b, the thread's first 8 columns, two per word

  // 16-byte loads, all issued together (a vector past the batch re-reads vector 0 and is cleared)
  static __device__ __forceinline__ void load_fast(uint32_t (&u)[BT][4], const uint16_t* __restrict__ X, int64_t ldx,
                                                   int batch, int t) {
#pragma unroll
    for (int b = 0; b < BT; ++b) {
      const uint4 q = *reinterpret_cast<const uint4*>(X + (int64_t)(b < batch ? b : 0) * ldx + 8 * t);
      u[b][0] = q.x; u[b][1] = q.y; u[b][2] = q.z; u[b][3] = q.w;
    }
#pragma unroll
    for (int b = 0; b < BT; ++b)
      if (b >= batch) u[b][0] = u[b][1] = u[b][2] = u[b][3] = 0u;
  }
  static __device__ __forceinline__ void load_slow(uint32_t (&u)[BT][4], const uint16_t* __restrict__ X, int64_t ldx,
                                                   int batch, int cols, int t) {
#pragma unroll
    for (int b = 0; b < BT; ++b) {
      const uint16_t* src = X + (int64_t)b * ldx + 8 * t;
#pragma unroll
      for (int k = 0; k < 8; k += 2) {
        const uint32_t lo = (b < batch && 8 * t + k < cols) ? src[k] : 0u;
        const uint32_t hi = (b < batch && 8 * t + k + 1 < cols) ? src[k + 1] : 0u;
        u[b][k >> 1] = lo | (hi << 16);
      }
    }
  }
  // column 8t+k of vectors b, b+1 -> one word; the BT values of a column are adjacent in LDS
  static __device__ __forceinline__ void store(const uint32_t (&u)[BT][4], uint16_t* xs, int t) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      uint32_t out[BT / 2];
#pragma unroll
      for (int b = 0; b < BT; b += 2) {
        const uint32_t lo = u[b][k >> 1], hi = u[b + 1][k >> 1];
        out[b >> 1] = (k & 1) ? __builtin_amdgcn_perm(hi, lo, 0x07060302u) : __builtin_amdgcn_perm(hi, lo, 0x05040100u);
      }
      unsigned char* dst = reinterpret_cast<unsigned char*>(xs + (size_t)(8 * t + k) * BT);
      if (BT == 8) *reinterpret_cast<uint4*>(dst) = make_uint4(out[0], out[1], out[2 % (BT / 2)], out[3 % (BT / 2)]);
      else if (BT == 4) *reinterpret_cast<uint2*>(dst) = make_uint2(out[0], out[1 % (BT / 2)]);
      else *reinterpret_cast<uint32_t*>(dst) = out[0];
    }
  }

  __device__ __forceinline__ void begin(const uint16_t* __restrict__ X, int64_t ldx, int batch, int cols) {
    const int t = threadIdx.x;
    const bool vec_ok = (reinterpret_cast<uintptr_t>(X) & 15) == 0 && (ldx & 7) == 0;
    if (vec_ok && 8 * t + 8 <= cols) load_fast(u, X, ldx, batch, t);
  }

  __device__ __forceinline__ void finish(unsigned char* lds, const uint16_t* __restrict__ X, int64_t ldx, int batch,
                                         int cols, int front_pad, int back_pad) {
    const int tid = threadIdx.x, nt = blockDim.x;
    const int chunks = (cols + 7) >> 3;
    const bool vec_ok = (reinterpret_cast<uintptr_t>(X) & 15) == 0 && (ldx & 7) == 0;
    uint4* lds16 = reinterpret_cast<uint4*>(lds);
    const uint4 zero = make_uint4(0, 0, 0, 0);
    const int front16 = front_pad * BT / 16, back16 = back_pad * BT / 16, body16 = chunks * BT;   // 16-byte units
    for (int i = tid; i < front16 + back16; i += nt) lds16[i < front16 ? i : i + body16] = zero;
    uint16_t* xs = reinterpret_cast<uint16_t*>(lds + front_pad * BT);
    if (tid < chunks) {
      if (!(vec_ok && 8 * tid + 8 <= cols)) load_slow(u, X, ldx, batch, cols, tid);   // else begin() loaded it
      store(u, xs, tid);
    }
    for (int t = tid + nt; t < chunks; t += nt) {
      uint32_t v[BT][4];
      if (vec_ok && 8 * t + 8 <= cols) load_fast(v, X, ldx, batch, t);
      else load_slow(v, X, ldx, batch, cols, t);
      store(v, xs, t);
    }
    __syncthreads();
  }
};

// VB: bits per stored value (16: fp16; 8: E4M3, 4-bit codes only).
template <int BT, int BD, int VB>
__global__ void __launch_bounds__(1024)
spmm_wave_row_kernel(const void* __restrict__ values, const uint32_t* __restrict__ deltas,
                     const uint32_t* __restrict__ row_ptr, const uint16_t* __restrict__ X, int64_t ldx,
                     uint16_t* __restrict__ Y, int64_t ldy, int batch, int rows, int cols, int q, int r_extra,
                     int inv_nwaves) {
  constexpr int RING = 2;
  using XV = typename XVec<BT>::type;
  extern __shared__ __align__(16) unsigned char lds[];
  // rows dealt out evenly: q per workgroup, one more for the first r_extra; the same over the wavefronts
  const int wg = (int)blockIdx.x;
  const int row_begin = wg * q + min(wg, r_extra);
  const int wg_rows = q + (wg < r_extra ? 1 : 0);
  const int nwaves = blockDim.x >> 6;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const unsigned char* xbase = lds + front_pad_for(BD) * BT;   // LDS address of column 0
  const uint32_t lane8 = 8u * lane;
  const int per_wave = (wg_rows * inv_nwaves) >> 16;     // wg_rows / nwaves (exact for wg_rows <= 1024)
  const int extra = wg_rows - per_wave * nwaves;
  const int blk = row_begin + wave * per_wave + min(wave, extra);
  const int nb = per_wave + (wave < extra ? 1 : 0);      // at most 64: the host sees to that

  RowCursor ld, cp;
  LaneCodes<BD> wq[RING];
  LaneValues<VB> vq[RING];
  const int r = min(blk + lane, rows - 1);             // unconditional loads, clamped to the last row
  const uint32_t rp_lo = row_ptr[r];
  const uint32_t rp_hi = row_ptr[r + 1];
  // start-up order as in the matrix-vector kernel: row pointers and activations are requested
  // together, the first streaming loads follow, and only then are the activations written to LDS
  XStageBatch<BT> xst;
  xst.begin(X, ldx, batch, cols);

  // every row is a buffer of its own, as in the matrix-vector kernel (us, clamped addresses and
  // masks / this: 4096 x 4096 at 50 %, 2 / 4 / 8 vectors, 7.47 / 8.13 / 11.8 -> 6.79 / 7.37 / 10.3, 11008 x 4096 12.7 / 15.1 / 22.6 -> 12.5 / 14.1 /
  // 20.7; over 144 calls on rows of 1 to 5 steps 0.95).  The position in a row is kept as its step alone: with a register each for values and
  // codes the kernel of two vectors needs 82 scalar ones, beyond 80 a SIMD holds 7 wavefronts instead of 8 (it has 800, and the trap handler takes
  // 16 of a wavefront's), and where a resident round has workgroups of 13 wavefronts and more half of it waits (us, 82 / 80: 6373 x 4096 with 570 8-bit values, 2 vectors, 6.6 / 5.6, 7477 x 4096 7.1 / 6.2).
  EntryBuffers<BD, VB> row;
  auto open_row = [&]() {
    if (ld.i >= nb) ld.nsteps = INT_MAX;               // no row follows
    row.open(values, deltas, ld.start >> 3, ld.end);
  };
  auto issue = [&](int j) {
    wq[j].load(row.codes, BD * (lane + 64 * ld.step));
    vq[j].load(row.values, VB * (lane + 64 * ld.step));
    if (++ld.step == ld.nsteps) {
      ++ld.i;
      seek_nonempty(ld, nb, rp_lo, rp_hi);
      open_row();
    }
  };
  ld.i = 0;
  seek_nonempty(ld, nb, rp_lo, rp_hi);
  cp = ld;
  open_row();
#pragma unroll
  for (int j = 0; j < RING; ++j) issue(j);
  xst.finish(lds, X, ldx, batch, cols, front_pad_for(BD), back_pad_for(BD));    // ends with a barrier

  float yv[BT], acc[BT];
#pragma unroll
  for (int b = 0; b < BT; ++b) yv[b] = acc[b] = 0.0f;
  int base2 = 0;
  int shared_step = -1;                                // the row's step whose last word of values holds some of the next row's, if any
  auto find_shared_step = [&]() { shared_step = (cp.end & (32 / VB - 1)) != 0u ? cp.nsteps - 1 : -1; };
  find_shared_step();
  while (cp.i < nb) {
#pragma unroll
    for (int j = 0; j < RING; ++j) {
      const bool live = cp.i < nb;                     // false for the padding items after the last row: they are left out
      if (live) {
        LaneCodes<BD> w = wq[j];
        LaneValues<VB> v = vq[j];
        if (cp.step == shared_step) {
          const uint32_t e0 = cp.a0 + 512u * cp.step + lane8;
          v.keep_first_of_words(e0 < cp.end ? cp.end - e0 : 0u);
        }
        w.decode();
        const uint32_t tot = w.total();
        const uint32_t incl = wave_incl_scan_u32(tot);
        if (cp.step == 0) {
          base2 = 0;
          const int before = (int)(cp.start - cp.a0);
          if (before > 0) {
            base2 = -(int)w.through(before - 1);
            // lane 0 also holds the previous row's last entries: they read the zero guard, and their values
            // are cleared so that an infinity or a NaN among them cannot become a NaN of this row
            v.clear_first((uint32_t)before, lane == 0);
          }
        }
        const int lanebase = base2 + (int)(incl - tot);
        // entry K: one gather address fetches the BT activations of its column
#define MACKO_ENTRY(K)                                                                       \
        {                                                                                      \
          const int q = lanebase + w.template offset<K>();     /* byte offset for one vector */ \
          const XV xraw = *reinterpret_cast<const XV*>(xbase + q * BT);                          \
          float xf[BT];                                                                        \
          unpack_x<BT>(xraw, xf);                                                              \
          const float wk = v.template get<K>();                                                \
          _Pragma("unroll") for (int b = 0; b < BT; ++b) acc[b] = fmaf(wk, xf[b], acc[b]);     \
        }
        MACKO_ENTRY(0) MACKO_ENTRY(1) MACKO_ENTRY(2) MACKO_ENTRY(3)
        MACKO_ENTRY(4) MACKO_ENTRY(5) MACKO_ENTRY(6) MACKO_ENTRY(7)
#undef MACKO_ENTRY
        base2 += (int)__builtin_amdgcn_readlane((int)incl, 63);
      }
      issue(j);
      if (live && ++cp.step == cp.nsteps) {
        wave_sum_to_last_lane_n<BT>(acc);                // the BT sums side by side
#pragma unroll
        for (int b = 0; b < BT; ++b) {
          const int tbits = __builtin_amdgcn_readlane(__builtin_bit_cast(int, acc[b]), 63);
          yv[b] = lane == cp.i ? __builtin_bit_cast(float, tbits) : yv[b];
          acc[b] = 0.0f;
        }
        ++cp.i;
        seek_nonempty(cp, nb, rp_lo, rp_hi);
        find_shared_step();
      }
    }
  }
  if (lane < nb) {
#pragma unroll
    for (int b = 0; b < BT; ++b)
      if (b < batch) Y[(int64_t)b * ldy + blk + lane] = f32_to_f16_bits(yv[b]);
  }
}

__global__ void __launch_bounds__(256) zero_Y_kernel(uint16_t* __restrict__ Y, int64_t ldy, int batch, int rows) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < rows)
    for (int b = 0; b < batch; ++b) Y[(int64_t)b * ldy + i] = 0;
}

template <int BT, int BD, int VB = 16>
int launch_bt_bd(const SpmvProblem& p, const uint16_t* X, int64_t ldx, uint16_t* Y, int64_t ldy, int batch,
                 hipStream_t stream) {
  const int cus = device_cu_count();
  const int64_t lds = (int64_t)BT * lds_bytes_for(p.cols, BD);
  const int64_t avg = p.pad_nnz / p.rows;
  PlanInput in{p.rows, std::max<int64_t>(1, (avg + 511) / 512), lds};
  // The interleaved copy of X is BT times the size of x, so a workgroup is expensive to start:
  // one resident round (a single 16-wavefront workgroup per compute unit once the copy passes
  // 36 KB) unless the matrix is large, as for the matrix-vector kernel.
  Plan plan;
  bool planned = false;
  if (in.rows * in.steps_per_row <= (int64_t)cus * 800 || lds >= 36 * 1024)
    planned = plan_resident(plan, 1, &in, cus, 0, lds >= 36 * 1024 ? 1 : 0, true);
  if (!planned) {
    const int block = lds > 48 * 1024 ? 1024 : 512;
    const int64_t want = (16 + in.steps_per_row - 1) / in.steps_per_row;
    const int64_t cap = std::max<int64_t>(1, p.rows / ((int64_t)cus * 16));
    const int64_t rpw = std::min(want, cap) * (block / 64);
    plan_by_rows_per_wg(plan, 1, &in, block, &rpw);
  }
  const int block = plan.block;
  const int64_t grid = plan.total_wgs;
  if (grid >= (int64_t{1} << 31)) return MACKO_E_UNSUPPORTED;
  auto kfn = spmm_wave_row_kernel<BT, BD, VB>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_fail(e);
  }
  hipLaunchKernelGGL(kfn, dim3((unsigned)grid), dim3(block), (size_t)lds, stream,
                     static_cast<const void*>(p.values), reinterpret_cast<const uint32_t*>(p.deltas),
                     p.row_ptr, X, ldx, Y, ldy, batch, (int)p.rows, (int)p.cols, plan.m[0].q, plan.m[0].r,
                     65536 / (block / 64) + 1);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? MACKO_OK : hip_fail(e);
}

template <int BT>
int launch_bt(const SpmvProblem& p, const uint16_t* X, int64_t ldx, uint16_t* Y, int64_t ldy, int batch,
              hipStream_t stream) {
  if (p.b_val == 8) return p.b_delta == 4 ? launch_bt_bd<BT, 4, 8>(p, X, ldx, Y, ldy, batch, stream) : MACKO_E_UNSUPPORTED;
  switch (p.b_delta) {
    case 1: return launch_bt_bd<BT, 1>(p, X, ldx, Y, ldy, batch, stream);
    case 2: return launch_bt_bd<BT, 2>(p, X, ldx, Y, ldy, batch, stream);
    case 4: return launch_bt_bd<BT, 4>(p, X, ldx, Y, ldy, batch, stream);
    case 8: return launch_bt_bd<BT, 8>(p, X, ldx, Y, ldy, batch, stream);
    default: return MACKO_E_UNSUPPORTED;
  }
}

constexpr int64_t kBatchLdsLimit = 160 * 1024 - 64;
// Vectors that the next pass over the matrix takes, of `left`: a piece of 8, 4 or 2 whose interleaved copies fit LDS, or one;
// with short rows up to kMaxGroup single products (pass = 0).
struct Piece {
  int pass, take;
};
Piece next_piece(bool long_rows, int64_t one, int left) {
  if (long_rows && left >= 5 && 8 * one <= kBatchLdsLimit) return {8, std::min(left, 8)};
  if (long_rows && left >= 3 && 4 * one <= kBatchLdsLimit) return {4, std::min(left, 4)};
  if (long_rows && left >= 2 && 2 * one <= kBatchLdsLimit) return {2, 2};
  if (long_rows) return {1, 1};
  return {0, std::min(left, kMaxGroup)};
}

// Whether pieces and single products can serve the call.  8-bit values have no kernel for an x beyond LDS (more than 80608
// columns), and how long it would take does not matter then: the matrix cores take every such batch of two vectors or more.
bool vectors_serve(const SpmvProblem& p) { return p.b_val != 8 || spmv_takes_wave_row(p); }

// Whether the matrix cores are the faster way for a call that both can take: from estimates of both times (us).
//
// Up to 16 vectors take the matrix cores one launch whose time is a sum of its parts (the phases of a window do not overlap, see
// macko_spmm_tile.hip).  The vector kernel takes a launch per piece: its start, the steps of 512 entries that the busiest wavefront
// takes one after the other (16 wavefronts to a compute unit) and that a compute unit takes in all, and the copy of the vectors,
// element by element where their length is no multiple of 8.  The factors were fitted to 16 000 calls timed both ways, before rows were read as
// buffers; over 18 000 others timed since (2 to 16 vectors, 16 to 40000 rows, 64 to 40000 columns, 30 to 99 % pruned, rows of 8 entries on, all code widths up
// to 4 bits, both value widths) the matrix cores' times are 5 % below the estimate and off by 5 % from there, the vectors' 7 % below and off by
// 8 %.  The way chosen is 0.22 % slower than the better one in the mean, for rows below and above kLongRow alike; factors fitted again to half of them chose no
// better on the other half (0.24 %).  What is left is at most 1.43 times as slow: 4 vectors on 32000 rows and more of 10 to 30 entries, and two on as many of
// 150 (34434 x 188 26.0 / 18.2, 32167 x 1920 13.6 / 18.7); with long rows 1.26, where the copy of odd vectors costs more than estimated (2654 x 3548 8.2 / 6.5).
// Without the busiest wavefront 3 or 4 vectors on 2049 to 4096 dense rows were up to 1.3 times as slow (3832 x 10352 at 53 %, 8-bit values, 3
// vectors, 15.5 -> 12.0; 2733 x 11072 at 33 %, 4: 17.8 -> 14.0).  A group of single products has to be priced as the launch it takes: as a launch
// to each product, as it was for rows of fewer than 192 entries before the wave-per-row kernel took them, the choice was 8.2 % slower with short rows (us,
// matrix cores / vectors: 504 x 448 with 43 entries, 4 vectors, 4.8 / 3.4; 195 x 3240 with 186, 3, 5.2 / 3.2).
// Up to 28 rows per compute unit in all, a resident round, such a launch takes the time of its wavefronts' rows one after the other: over 693 calls on
// 200 to 6000 short rows the choice is 0.9 % slower than the better one, 1.07 times at worst, 1.55 % and 1.13 with one slope for all (us, matrix
// cores / vectors: 600 x 100 with 60 entries, 8 vectors, 4.5 / 5.1, 900 x 400, 6, 4.5 / 5.0; 500 x 400, 8, 4.5 / 4.2).
// The matrix cores' estimate has to be 3 % below the vectors'; with short rows, where both take about 5 us, 3 % above it is enough.
double tile_estimate(const SpmvProblem& p, int batch) {
  const double cols = (double)p.cols / 4096.0, tiles = std::ceil((double)p.rows / (16.0 * device_cu_count()));
  const double steps = tiles * std::ceil((double)p.pad_nnz / (double)p.rows / 512.0), more = batch > 8 ? 1.0 : 0.0;
  const double mbytes = (double)p.pad_nnz * (p.b_val + p.b_delta) / 8e6, windows = (double)spmm_tile_windows(p);
  if (spmm_tile_pairs_groups(p, batch)) return 3.08 + 1.31 * windows + (0.78 + 0.09 * more) * tiles * cols + 0.47 * steps + 0.049 * mbytes;
  return 2.54 + 2.14 * windows + (0.37 + 0.18 * more) * tiles * cols + 0.44 * steps + 0.058 * mbytes;
}

double vector_estimate(const SpmvProblem& p, int batch) {
  const double cus = device_cu_count(), rows = (double)p.rows, cols = (double)p.cols / 4096.0, ragged = p.cols % 8 != 0 ? 1.0 : 0.0;
  const double entries = (double)p.pad_nnz, steps = std::ceil(entries / rows / 512.0), all = rows * steps / cus;
  const double busiest = std::ceil(rows / (16.0 * cus)) * steps;        // steps of one wavefront
  const double few = rows < 4.0 * cus ? steps : 0.0;                   // no resident round: nothing covers a step's latency
  const double mbytes = entries * (p.b_val + p.b_delta) / 8e6;
  const bool long_rows = spmm_shares_passes(p, batch);
  const bool one_launch = spmv_takes_wave_row(p, wave_row_min_entries(p, batch));      // of a group of single products, as launch_spmv_group decides
  const int64_t one = lds_bytes_for(p.cols, p.b_delta);
  double us = 0.0;
  for (int left = batch; left > 0;) {
    const Piece q = next_piece(long_rows, one, left);
    if (q.pass == 8)
      us += 3.36 + 0.348 * busiest + 0.027 * all + 2.16 * cols + ragged * (1.67 + 4.61 * cols) + 0.443 * few + 0.096 * rows / cus;
    else if (q.pass == 4)
      us += 2.94 + 0.331 * busiest + 0.020 * all + 0.59 * cols + ragged * (0.93 + 2.70 * cols) + 0.212 * few + 0.057 * rows / cus;
    else if (q.pass == 2)
      us += 2.87 + 0.358 * busiest + 0.018 * all + 0.21 * cols + ragged * (0.60 + 1.50 * cols) + 0.113 * few + 0.044 * rows / cus;
    else if (q.pass == 1)
      us += 2.07 + 0.317 * busiest + 0.023 * all + 0.14 * cols + ragged * (0.94 + 0.25 * cols) + 0.135 * few + 0.039 * rows / cus;
    else if (one_launch)
      us += std::max(3.47 + 0.056 * q.take * all, 2.95 + 0.105 * std::min(28.0, q.take * all)) + q.take * 0.033 * mbytes + (0.86 * ragged + 0.68 * std::min(1.0, rows / (4.0 * cus))) * cols;
    else
      us += q.take * (2.89 + 1.025 * entries / 1e6 + 0.46 * cols) + 3.45 * ragged * cols;
    left -= q.take;
  }
  return us;
}

bool tile_is_faster(const SpmvProblem& p, int batch) {
  if (batch > 16) return true;                         // at least three pieces (11008 x 4096, 64 vectors: 183 / 32)
  // x beyond LDS: every vector is gathered from memory by itself, at two vectors already the slower way in all of 111 calls (us,
  // vectors / matrix cores: 25 x 487832, 2 vectors, 686 / 361; 226 x 178280 at 99 %, 6, 754 / 112; 301 x 118384 at 93 %, 5, 587 / 76)
  if (spmv_lds_bytes(p.cols, p.b_delta) > kMaxLdsBytes) return true;
  return (p.pad_nnz / p.rows >= kLongRow ? 1.03 : 0.97) * tile_estimate(p, batch) < vector_estimate(p, batch);
}

}  // namespace

// Y[b][r] = sum over row r of W * X[b][column], b < batch.  The batch is cut into
// pieces of 8, 4, 2 or 1 vectors, each the largest that fits LDS; single vectors
// (and matrices with short rows) go through the matrix-vector path; larger batches go to the
// matrix cores in one piece (macko_spmm_tile.hip) where that is faster.
int launch_spmm(const SpmvProblem& p, const void* X, int64_t ldx, void* Y, int64_t ldy, int batch,
                hipStream_t stream) {
  if (p.pad_nnz > (int64_t{1} << 32) - 4096) return MACKO_E_UNSUPPORTED;   // 32-bit entry indices in the kernel
  const uint16_t* Xp = static_cast<const uint16_t*>(X);
  uint16_t* Yp = static_cast<uint16_t*>(Y);
  if (p.rows == 0 || batch == 0) return MACKO_OK;
  if (p.pad_nnz == 0) {
    hipLaunchKernelGGL(zero_Y_kernel, dim3((unsigned)((p.rows + 255) / 256)), dim3(256), 0, stream, Yp, ldy,
                       batch, (int)p.rows);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? MACKO_OK : hip_fail(e);
  }
  const int64_t one = lds_bytes_for(p.cols, p.b_delta);
  const bool long_rows = spmm_shares_passes(p, batch);
  const int64_t knob = tuning().spmm_kernel;
  if (batch > 1 && spmm_tile_serves(p, ldx) && (!vectors_serve(p) || (knob != 0 ? knob == 2 : tile_is_faster(p, batch))))
    return launch_spmm_tile(p, Xp, ldx, Yp, ldy, batch, stream);
  int done = 0;
  while (done < batch) {
    const Piece piece = next_piece(long_rows, one, batch - done);
    const int take = piece.take;
    const uint16_t* Xb = Xp + (int64_t)done * ldx;
    uint16_t* Yb = Yp + (int64_t)done * ldy;
    int st;
    if (piece.pass == 8) {
      st = launch_bt<8>(p, Xb, ldx, Yb, ldy, take, stream);
    } else if (piece.pass == 4) {
      st = launch_bt<4>(p, Xb, ldx, Yb, ldy, take, stream);
    } else if (piece.pass == 2) {
      st = launch_bt<2>(p, Xb, ldx, Yb, ldy, take, stream);
    } else {
      SpmvProblem q[kMaxGroup];
      for (int i = 0; i < take; ++i) {
        q[i] = p;
        q[i].x = Xb + (int64_t)i * ldx;
        q[i].y = Yb + (int64_t)i * ldy;
      }
      st = launch_spmv_group(take, q, batch, stream);
    }
    if (st != MACKO_OK) return st;
    done += take;
  }
  return MACKO_OK;
}

}  // namespace macko
