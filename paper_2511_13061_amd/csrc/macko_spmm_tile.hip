// Batch product Y = W X^T for the MACKO format on the matrix cores of gfx950.
//
// The vector kernel of macko_spmm.hip multiplies every stored entry with every vector (one
// v_fma_mix_f32 per entry and vector) and is bound by vector arithmetic from 8 vectors on.  This one
// expands the rows instead: the wavefronts of a workgroup decode 16 rows, one row each, and put the
// values at their columns into a dense fp16 tile in LDS, a window of columns at a time; the tile is
// the A operand of v_mfma_f32_16x16x32_f16 (fp16 products, fp32 accumulation), the vectors are the B
// operand.  The cost per stored entry no longer depends on the batch.
//
// What bounds it: vector issue.  Of 19 us for 4096 x 11008 at 50 % with 8 vectors, the decode takes
// about 6 (65 vector instructions per step of 512 entries), memory latency 4 (one 16-wavefront
// workgroup per compute unit), scattering into LDS 2, and the window products 4, half of that the
// transposes of the B operand (times found by leaving one part out).  Counters: 4.96 M vector instructions, 8 us of issue,
// there, and 11.7 M, 19 of 43 us, for 11008 x 4096 with 64 vectors; the rest is waited for.  A second workgroup per compute
// unit could cover that; LDS has room for two (with windows of 2048 columns), registers do not (75 to 125, where 64 would do).
// The vectors are read again for every tile, and after its last window twice: what follows that window is requested before
// its reduction and once more behind it, and the last tile requests a window that nobody uses.  With 64 vectors of 4096
// elements that is 10 loads of 256 KB per workgroup where 6 are used, 0.7 GB through the caches for a problem of 58 MB (0.78 M
// vector loads counted per call).  Measured against the vector kernel
// at 50 % (us, batch 8 / 16 / 64): 4096 x 11008: 29.6 / 59 / 239 -> 20.5 / 21.2 / 38.7, 11008 x 4096:
// 23.6 / 46 / 183 -> 22.7 / 23.2 / 43.6, 4096 x 4096: 12.1 / 24 / 96 -> 11.5 / 11.7 / 19.0.
//
// Tried: 8 rows per workgroup and two workgroups per compute unit (28-40 us where 16 rows take 21: half
// of the matrix instruction is idle and every B element is fetched twice); 3 and 4 steps loaded ahead
// instead of 2 (slower); the B operand loaded straight into the operand's lane order (16
// vectors on 16 neighbouring lanes: every lane is a memory request of its own, 64 vectors took 63 us).
#include "macko_decode.h"
#include "macko_device.h"
#include "macko_internal.h"

namespace macko {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTileRows = 16;                          // rows of a tile = wavefronts of a workgroup
// Bytes in front of every row of the tile (and behind the last) that are written but never read: entries
// in front of the window or behind it land there.  A lane's 8 entries span at most 8 * 2 * 16 bytes.
constexpr int kTilePad = 256;
constexpr int tile_window(int groups) { return 128 * kTileRows * groups; }          // columns
// 16 bytes more per row: the 16 rows that a matrix instruction reads at one column fall on different banks
constexpr int tile_stride(int groups) { return 2 * tile_window(groups) + kTilePad + 16; }
constexpr int tile_lds(int groups) { return kTileRows * tile_stride(groups) + kTilePad; }
static_assert(64 * kTileRows == 1024 && 4 * (kTileRows - 1) * 1024 <= tile_lds(1), "the partial sums of 64 vectors fit the tile's memory");

struct TileArgs {
  const void* values;
  const uint32_t* deltas;
  const uint32_t* row_ptr;
  const uint16_t* X;
  uint16_t* Y;
  int64_t ldx, ldy;
  int rows, cols, batch, q, r;                         // rows per workgroup: q, one more for the first r
};

// dst = src as real register moves.  The source registers are free afterwards, so that the next load can go
// into the same ones; left to itself the compiler renames instead, and then has to copy, that is to wait for,
// the load that is under way where the loop closes.
template <class T>
__device__ __forceinline__ void move_regs(T& dst, const T& src) {
  constexpr int n = sizeof(T) / 4;
  uint32_t a[n], b[n];
  __builtin_memcpy(a, &src, sizeof(T));
#pragma unroll
  for (int i = 0; i < n; ++i) asm volatile("v_mov_b32 %0, %1" : "=v"(b[i]) : "v"(a[i]));
  __builtin_memcpy(&dst, b, sizeof(T));
}

// The compiler takes these as changed here: what is computed from them afterwards cannot have been computed earlier.
__device__ __forceinline__ void keep_opaque(uint32_t& w, LaneValues<16>& v) {
  asm volatile("" : "+v"(w), "+v"(v.v.x), "+v"(v.v.y), "+v"(v.v.z), "+v"(v.v.w));
}
__device__ __forceinline__ void keep_opaque(uint32_t& w, LaneValues<8>& v) { asm volatile("" : "+v"(w), "+v"(v.v.x), "+v"(v.v.y)); }

template <int CTRL>
__device__ __forceinline__ uint32_t quad_dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}
// 4 x 4 transpose of 16-byte blocks within every four lanes: register r of lane 4 i + q goes to register q of lane 4 i + r
__device__ __forceinline__ void quad_transpose(u32x4 (&b)[4], bool odd, bool high) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t a0 = b[0][i], a1 = b[1][i], a2 = b[2][i], a3 = b[3][i];
    // (the moves on their own: inside a conditional operator they would run with the other lanes switched off)
    const uint32_t s0 = quad_dpp<0xB1>(a0), s1 = quad_dpp<0xB1>(a1), s2 = quad_dpp<0xB1>(a2), s3 = quad_dpp<0xB1>(a3);
    const uint32_t c0 = odd ? s1 : a0, c1 = odd ? a1 : s0, c2 = odd ? s3 : a2, c3 = odd ? a3 : s2;
    const uint32_t d0 = quad_dpp<0x4E>(c0), d1 = quad_dpp<0x4E>(c1), d2 = quad_dpp<0x4E>(c2), d3 = quad_dpp<0x4E>(c3);
    b[0][i] = high ? d2 : c0;
    b[2][i] = high ? c2 : d0;
    b[1][i] = high ? d3 : c1;
    b[3][i] = high ? c3 : d1;
  }
}

// The results of one row for the vectors of `vectors` (bit b: vector b), entry by entry.  The product with the expanded
// row multiplies zeros with every element of x; where that gives something else than leaving them out, i.e. where
// x holds an infinity or a NaN, the result of the product is not finite and this takes its place.  Rare and slow.
// An entry at or beyond the last column (a wrong encoding) counts for nothing, as in the product.
template <int BD, int VB>
__device__ __forceinline__ void tile_row_by_entries(const TileArgs& a, int row, uint32_t start, uint32_t end, uint64_t vectors) {
  const int lane = threadIdx.x & 63;
  while (vectors) {
    const int vec = __builtin_ctzll(vectors);
    vectors &= vectors - 1;
    const uint16_t* x = a.X + (int64_t)vec * a.ldx;
    float acc = 0.0f;
    int base2 = 0;
    for (uint32_t e0 = start & ~7u; e0 < end; e0 += 512u) {
      const uint32_t e = e0 + 8u * lane;
      const uint32_t chunk = min(e, end - 1u) >> 3;
      LaneCodes<BD> w;
      LaneValues<VB> v;
      w.load(a.deltas, chunk);
      v.load(a.values, chunk);
      w.keep_if(e < end);
      w.decode();
      const uint32_t tot = w.total();
      const uint32_t incl = wave_incl_scan_u32(tot);
      if (e0 < start) base2 = -(int)w.through((int)(start - e0) - 1);
      const int lanebase = base2 + (int)(incl - tot);
#define MACKO_ENTRY(K)                                                              \
  {                                                                                 \
    const int col = (lanebase + w.template offset<K>()) >> 1;                       \
    if (e + K >= start && e + K < end && (uint32_t)col < (uint32_t)a.cols)          \
      acc = fmaf(v.template get<K>(), f16_bits_to_f32(x[col]), acc);                \
  }
      MACKO_ENTRY(0) MACKO_ENTRY(1) MACKO_ENTRY(2) MACKO_ENTRY(3) MACKO_ENTRY(4) MACKO_ENTRY(5) MACKO_ENTRY(6) MACKO_ENTRY(7)
#undef MACKO_ENTRY
      base2 += (int)__builtin_amdgcn_readlane((int)incl, 63);
    }
    acc = wave_sum_to_last_lane(acc);
    if (lane == 63) a.Y[(int64_t)vec * a.ldy + row] = f32_to_f16_bits(acc);
  }
}

// NT: tiles of 16 vectors.  G: groups of 128 columns per wavefront and window.  S: steps loaded ahead.
//
// A workgroup works on one tile of 16 rows after the other; a wavefront's rows (one per tile) form one stream
// of steps, so that the loads run on across windows and tiles.  Decoding and the products of the windows
// alternate; a step that reaches behind the window is put into the tile in parts, one window after the other, out
// of registers.  Every wavefront takes part in every window's product (128 G columns each) whatever its row
// holds, so all of them execute the same number of barriers.
template <int NT, int BD, int VB, int G, int S>
__global__ void __launch_bounds__(64 * kTileRows)
spmm_tile_kernel(const TileArgs a) {
  static_assert(BD <= 4, "a lane's 8 entries have to fit the pad");
  constexpr int kWindow = tile_window(G);
  constexpr int kStride = tile_stride(G);
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ uint32_t odd_results[64 * kTileRows][2];  // per row of the workgroup, a bit per vector: not finite
  __shared__ uint32_t any_odd;
  float4v* red = reinterpret_cast<float4v*>(lds);      // [NT][kTileRows - 1][64]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wg = (int)blockIdx.x;
  const int row0 = wg * a.q + min(wg, a.r);
  const int wg_rows = a.q + (wg < a.r ? 1 : 0);
  const int tiles = (wg_rows + kTileRows - 1) / kTileRows;      // at most 64: the host sees to that
  const int nb = wave < wg_rows ? (wg_rows - wave + kTileRows - 1) / kTileRows : 0;   // this wavefront's rows
  const int cols = a.cols;
  const uint32_t lane8 = 8u * lane;

  uint32_t rp_lo, rp_hi;                               // lane i: the pointers of the wavefront's row i
  {
    const int r = min(row0 + wave + kTileRows * lane, a.rows - 1);
    rp_lo = a.row_ptr[r];
    rp_hi = a.row_ptr[r + 1];
  }

  // A operand: lane holds row lane % 16, 8 columns; matrix instruction r of a group of 128 columns takes columns
  // 32 (lane / 16) + 8 r ... + 7 (the order of the columns within the sum is free, as long as B has the same).
  const int n = lane & 15;
  unsigned char* arow = lds + kTilePad + n * kStride + 2 * (128 * G * wave + 32 * (lane >> 4));
  // B operand: lane has to hold vector lane % 16 of the same columns.  Neighbouring lanes would then read from 16
  // different vectors, which costs a memory request per lane; instead four neighbouring lanes read 64 consecutive
  // bytes of one vector, load r from vector 4 (lane / 4 % 4) + r, and exchange 16-byte blocks afterwards.
  const bool odd_lane = lane & 1, high_lane = lane & 2;
  // The vectors are one buffer (base rounded down to 4 bytes): what lies behind its end, vectors past the batch among
  // it, reads as zero; what lies between two vectors is cleared where it is used.  The end is checked per 4 bytes, so
  // the buffer ends in front of the last element of an odd number of columns, which would be half of such a piece: the
  // last vector's is loaded by itself and put in its place where the vectors end.  (The other vectors' are inside: the
  // element behind them is the next vector's, or lies between the two; a single column is not served.)
  const uint32_t xmis = (uint32_t)(reinterpret_cast<uintptr_t>(a.X) & 2);
  const uint32_t xbytes = (uint32_t)(((int64_t)(a.batch - 1) * a.ldx + (cols & ~1)) * 2) + xmis;
  uint32_t last_x = 0u;
  if (cols & 1) last_x = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.X[(int64_t)(a.batch - 1) * a.ldx + cols - 1]);
  const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(reinterpret_cast<const unsigned char*>(a.X) - xmis), 0, (int)xbytes, 0x00020000);
  const uint32_t ldx2 = 2u * (uint32_t)a.ldx;
  const int bcol = 128 * G * wave + 8 * (4 * (lane >> 4) + (lane & 3));     // the lane's first column within the window
  const uint32_t xoff = xmis + 4u * ((lane >> 2) & 3) * ldx2 + 2u * bcol;
  u32x4 b[G][NT][4];
  int k0 = 0, tile = 0;                                // first column of the window, tile
  const int cols2 = 2 * ((cols + 127) & ~127);         // doubled end of the groups that are multiplied
  uint32_t put_bytes = (uint32_t)min(2 * kWindow, cols2) + kTilePad;       // lanes that start in the window, and in these groups
  auto load_b = [&]() {
    uint32_t xo = xoff;
    if (NT > 2) asm volatile("" : "+v"(xo));           // no offsets computed in front of the loop and kept in registers
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const auto q = __builtin_amdgcn_raw_buffer_load_b128(
              xrsrc, (int)(xo + 2u * (uint32_t)(k0 + 128 * g) + (uint32_t)(16 * t + r) * ldx2), 0, 0);
          b[g][t][r] = u32x4{(uint32_t)q[0], (uint32_t)q[1], (uint32_t)q[2], (uint32_t)q[3]};
        }
  };

  // the load side of the stream of steps; a row without entries takes one step with everything cleared
  LaneCodes<BD> wq[S];
  LaneValues<VB> vq[S];
  int ld_i = 0;
  uint32_t ld_e0 = 0, ld_end = 0, chunk = 0;
  auto open_load_row = [&](int i) {
    ld_e0 = (uint32_t)__builtin_amdgcn_readlane((int)rp_lo, i) & ~7u;
    ld_end = (uint32_t)__builtin_amdgcn_readlane((int)rp_hi, i);
  };
  auto issue = [&](int j) {
    if (ld_i < nb) {                                   // else the previous chunk once more
      chunk = min(ld_e0 + lane8, max(ld_end, 1u) - 1u) >> 3;     // lanes past the row end re-read its last chunk
      ld_e0 += 512u;
      if (ld_e0 >= ld_end && ++ld_i < nb) open_load_row(ld_i);
    }
    wq[j].load(a.deltas, chunk);
    vq[j].load(a.values, chunk);
  };

  // the tile starts out as zeros; the product of a window leaves what it has read zero again
  for (int i = threadIdx.x; i < tile_lds(G) / 16; i += 64 * kTileRows) reinterpret_cast<u32x4*>(lds)[i] = u32x4{0, 0, 0, 0};
  odd_results[threadIdx.x][0] = odd_results[threadIdx.x][1] = 0u;
  if (threadIdx.x == 0) any_odd = 0u;
  load_b();
  if (nb > 0) open_load_row(0);
#pragma unroll
  for (int j = 0; j < S; ++j) issue(j);

  float4v acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = float4v{0.f, 0.f, 0.f, 0.f};
  __syncthreads();

  // the product of the window at k0 and, behind the last window, the results of the tile
  auto finish_window = [&]() {
    __syncthreads();                                   // every row's entries of the window are in the tile
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int kg = k0 + 128 * (G * wave + g);        // first column of the group
      if (kg < cols) {
        // (marked as rare: 1.5 % at 64 vectors, by keeping its code out of the loop's)
        if (__builtin_expect(kg + 128 > cols, 0)) {    // the vectors end in it
          const int left = cols - (k0 + 128 * g + bcol);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t mask = left > 2 * i + 1 ? 0xFFFFFFFFu : (left > 2 * i ? 0xFFFFu : 0u);
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
              for (int r = 0; r < 4; ++r) b[g][t][r][i] &= mask;
          }
          if (__builtin_expect(cols & 1, 0)) {         // the last element of the last vector (left is odd here)
            const int last = a.batch - 1 - 4 * ((lane >> 2) & 3);        // load r of tile t is vector `last` if 16 t + r is
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const uint32_t e = left == 2 * i + 1 ? last_x : 0u;
#pragma unroll
              for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) b[g][t][r][i] |= last == 16 * t + r ? e : 0u;
            }
          }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          quad_transpose(b[g][t], odd_lane, high_lane);
          if (NT > 2) __builtin_amdgcn_sched_barrier(0);         // keeps the temporaries of one t at a time: no spills
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          half8* ap = reinterpret_cast<half8*>(arow + 256 * g + 16 * r);
          const half8 av = *ap;
          *ap = half8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
          for (int t = 0; t < NT; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, __builtin_bit_cast(half8, b[g][t][r]), acc[t], 0, 0, 0);
          if (NT > 2) __builtin_amdgcn_sched_barrier(0);
        }
      } else if (kg < cols + 128) {
        // Groups behind the last column are not multiplied.  What a wrong encoding's row puts into the first of them (into
        // the others nothing is put) would be part of the next tile's row: a right one's leaves zeros.
#pragma unroll
        for (int r = 0; r < 4; ++r) *reinterpret_cast<half8*>(arow + 256 * g + 16 * r) = half8{0, 0, 0, 0, 0, 0, 0, 0};
      }
    }
    k0 += kWindow;
    const bool done = k0 >= cols;
    if (done) k0 = 0;
    put_bytes = (uint32_t)min(2 * kWindow, cols2 - 2 * k0) + kTilePad;
    __builtin_amdgcn_sched_barrier(0);
    load_b();                                          // under way while the next window is decoded
    __syncthreads();                                   // the tile is zero again
    if (done) {
      // wavefront t adds up vectors 16 t ... 16 t + 15; the others hand their sums over in the tile's memory
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (wave != t) red[(t * (kTileRows - 1) + (wave < t ? wave : wave - 1)) * 64 + lane] = acc[t];
      __syncthreads();
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (wave == t) {
          float4v sum = acc[t];
#pragma unroll 5
          for (int g = 0; g < kTileRows - 1; ++g) {
            float4v* p = red + (t * (kTileRows - 1) + g) * 64 + lane;
            sum += *p;
            *p = float4v{0.f, 0.f, 0.f, 0.f};
          }
          int l = lane;
          if (NT > 2) asm volatile("" : "+v"(l));      // nor pointers into Y
          const int n = l & 15;
          const int m0 = 4 * (l >> 4), left = wg_rows - kTileRows * tile - m0;     // lane holds rows m0 ... m0 + 3
          if (16 * t + n < a.batch) {
            uint16_t* y = a.Y + (int64_t)(16 * t + n) * a.ldy + (row0 + kTileRows * tile + m0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (i < left) {
                if (__builtin_fabsf(sum[i]) <= 3.4028234e38f) {
                  y[i] = f32_to_f16_bits(sum[i]);
                } else {                               // an infinity or a NaN in the row or in the vector
                  atomicOr(&odd_results[kTileRows * tile + m0 + i][t >> 1], 1u << (16 * (t & 1) + n));
                  any_odd = 1u;
                }
              }
          }
        }
        acc[t] = float4v{0.f, 0.f, 0.f, 0.f};
      }
      __builtin_amdgcn_sched_barrier(0);
      load_b();
      __syncthreads();
      ++tile;
    }
  };

  unsigned char* rowbuf = lds + kTilePad + wave * kStride;
  LaneCodes<BD> wh[S];                                 // steps 1 ... S - 1 of the group taken out of the load registers last
  LaneValues<VB> vh[S];
  int next = 0;                                        // the step of the group that comes next
  int base2 = 0;                                       // doubled position behind the row's steps decoded so far
  int i = 0;
  uint32_t e0 = 0, start = 0, end = 0;
  auto open_row = [&]() {
    start = (uint32_t)__builtin_amdgcn_readlane((int)rp_lo, i);
    end = (uint32_t)__builtin_amdgcn_readlane((int)rp_hi, i);
    e0 = start & ~7u;
  };
  if (nb > 0) open_row();
  for (;;) {
    const bool live = i < nb;
    const int target = live ? i : tiles;
    // S steps are loaded at a time: out of the load registers with all of them, then the next S are requested
    LaneCodes<BD> w;
    LaneValues<VB> v;
    if (next == 0) {
      move_regs(w.w, wq[0].w);
      move_regs(v, vq[0]);
#pragma unroll
      for (int j = 1; j < S; ++j) {
        move_regs(wh[j].w, wq[j].w);
        move_regs(vh[j], vq[j]);
      }
#pragma unroll
      for (int j = 0; j < S; ++j) issue(j);
    }
#pragma unroll
    for (int j = 1; j < S; ++j)
      if (next == j) {
        w.w = wh[j].w;
        v = vh[j];
      }
    if (++next == S) next = 0;
    if (e0 + 512u > end) {                             // the row's last step: clear what lies behind its end
      const uint32_t nv = e0 + lane8 < end ? end - (e0 + lane8) : 0u;
      w.keep_if(nv != 0);
      v.keep_first(nv);
    }
    w.decode();
    const uint32_t tot = w.total();
    const uint32_t incl = wave_incl_scan_u32(tot);
    if (e0 <= start) {                                 // the row's first step
      base2 = 0;
      const int before = (int)(start - e0);            // entries of the previous row: they land in front of column 0
      if (before > 0) base2 = -(int)w.through(before - 1);
    }
    const int lanebase = base2 + (int)(incl - tot);
    base2 += (int)__builtin_amdgcn_readlane((int)incl, 63);
    for (;;) {
      if (tile == target) {
        if (!live) goto out;
        // with many vectors every register counts: nothing about the entries is computed in front of this loop and kept
        if (NT > 1) keep_opaque(w.w, v);
        // lanes without an entry in the window write to the pad; so do a lane's entries in front of the window or
        // behind it.  What is behind the row's end is zero, and so is the tile there.
        int rel = lanebase - 2 * k0;
        rel = (uint32_t)(rel + kTilePad) < put_bytes ? rel : -kTilePad;
        unsigned char* p = rowbuf + rel;
#define MACKO_PUT(K) *reinterpret_cast<uint16_t*>(p + w.template offset<K>()) = (uint16_t)v.template half<K>();
        MACKO_PUT(0) MACKO_PUT(1) MACKO_PUT(2) MACKO_PUT(3) MACKO_PUT(4) MACKO_PUT(5) MACKO_PUT(6) MACKO_PUT(7)
#undef MACKO_PUT
        if (k0 + kWindow >= cols || base2 <= 2 * (k0 + kWindow)) break;
      }
      finish_window();
    }
    e0 += 512u;
    if (e0 >= end && ++i < nb) open_row();
  }
out:
  if (any_odd) {                                       // set, if at all, in front of the last barrier
    for (i = 0; i < nb; ++i) {
      const int r = kTileRows * i + wave;
      const uint64_t vectors = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)odd_results[r][0]) |
                               ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)odd_results[r][1]) << 32);
      if (vectors)
        tile_row_by_entries<BD, VB>(a, row0 + r, (uint32_t)__builtin_amdgcn_readlane((int)rp_lo, i),
                                    (uint32_t)__builtin_amdgcn_readlane((int)rp_hi, i), vectors);
    }
  }
}

template <int NT, int BD, int VB, int G, int S>
int launch_tile_as(TileArgs a, hipStream_t stream) {
  constexpr int lds = tile_lds(G);
  auto kfn = spmm_tile_kernel<NT, BD, VB, G, S>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return hip_fail(e);
  // One workgroup per compute unit with an equal share of the rows: registers allow no second one, and the fewer
  // workgroups, the fewer times the vectors are read.  A wavefront keeps the pointers of at most 64 rows.
  int64_t grid = std::min<int64_t>(((int64_t)a.rows + kTileRows - 1) / kTileRows, (int64_t)device_cu_count());
  grid = std::max<int64_t>(grid, ((int64_t)a.rows + 64 * kTileRows - 1) / (64 * kTileRows));
  a.q = (int)(a.rows / grid);
  a.r = (int)(a.rows % grid);
  hipLaunchKernelGGL(kfn, dim3((unsigned)grid), dim3(64 * kTileRows), (size_t)lds, stream, a);
  e = hipGetLastError();
  return e == hipSuccess ? MACKO_OK : hip_fail(e);
}

// Windows of 4096 columns where the registers allow it (up to 16 vectors) and the row is longer than 2048: fewer
// products of windows to wait for (4096 x 4096, 8 vectors: 11.3 -> 10.6 us; 14336 x 1024 would lose, 14.0 -> 15.9,
// its tile being cleared and read twice as wide as needed).  One step ahead instead of two from 33 vectors on: two
// would spill registers in the loop (44 -> 60 us).
template <int BD, int VB>
int launch_tile_bd(const TileArgs& a, hipStream_t stream) {
  const int nt = (a.batch + 15) / 16;
  if (nt == 1) return a.cols > tile_window(1) ? launch_tile_as<1, BD, VB, 2, 2>(a, stream) : launch_tile_as<1, BD, VB, 1, 2>(a, stream);
  if (nt == 2) return launch_tile_as<2, BD, VB, 1, 2>(a, stream);
  if (nt == 3) return launch_tile_as<3, BD, VB, 1, 1>(a, stream);
  return launch_tile_as<4, BD, VB, 1, 1>(a, stream);
}

}  // namespace

bool spmm_tile_serves(const SpmvProblem& p, int64_t ldx) {
  if (p.b_delta > 4 || p.pad_nnz == 0 || p.rows == 0) return false;   // the pad of the tile holds 4-bit deltas
  if (p.cols < 2) return false;                        // see the end of the vectors' buffer in the kernel
  return ldx < (int64_t{1} << 24);                     // vectors are addressed with 32-bit byte offsets
}

int launch_spmm_tile(const SpmvProblem& p, const uint16_t* X, int64_t ldx, uint16_t* Y, int64_t ldy, int batch,
                     hipStream_t stream) {
  const TileArgs a{p.values, reinterpret_cast<const uint32_t*>(p.deltas), p.row_ptr, X, Y, ldx, ldy,
                   (int)p.rows, (int)p.cols, batch, 0, 0};
  if (p.b_val == 8) return p.b_delta == 4 ? launch_tile_bd<4, 8>(a, stream) : MACKO_E_UNSUPPORTED;
  switch (p.b_delta) {
    case 1: return launch_tile_bd<1, 16>(a, stream);
    case 2: return launch_tile_bd<2, 16>(a, stream);
    case 4: return launch_tile_bd<4, 16>(a, stream);
    default: return MACKO_E_UNSUPPORTED;
  }
}

}  // namespace macko
