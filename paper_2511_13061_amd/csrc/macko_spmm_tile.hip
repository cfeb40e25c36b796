// Batch product Y = W X^T for the MACKO format on the matrix cores of gfx950.
//
// The vector kernel of macko_spmm.hip multiplies every stored entry with every vector (one
// v_fma_mix_f32 per entry and vector) and is bound by vector arithmetic from 8 vectors on.  This one
// expands the rows instead: the wavefronts of a workgroup decode 16 rows, one row each, and put the
// values at their columns into a dense fp16 tile in LDS, a window of columns at a time; the tile is
// the A operand of v_mfma_f32_16x16x32_f16 (fp16 products, fp32 accumulation), the vectors are the B
// operand.  The cost per stored entry no longer depends on the batch.
//
// A workgroup takes a panel of 16 P rows (P = 1, 2 or 3 tiles of 16) through the windows; each of its 16 wavefronts decodes P
// rows.  The window's vectors are loaded and turned into the B operand once for all tiles of the panel, which is what counts
// with many vectors: X passes a compute unit's L1 at 64 bytes a clock, 3.4 us for 64 vectors of 4096 elements, and used to be
// read for every 16 rows.  LDS holds about 65 000 cells in all, so a panel of more rows has narrower windows.
//
// What bounds it: no unit by itself.  11008 x 4096 at 50 % with 64 vectors, 30 us: vector issue 12 (decode 45 instructions
// per step of 512 entries, 11 per window that a step reaches into, 64 per four 16-byte loads of B), LDS 9, HBM 8.5, matrix
// cores 2.6, loads of B 3.4; but the phases of a window (decode, product, clearing) alternate behind barriers, and one
// 16-wavefront workgroup per compute unit covers little of one with another.  Leaving out the puts into the tile takes 4 us off, B and its
// transposes 8, the matrix instructions 3; a window costs about 2 us whatever is in it, so few, large windows are best.
// Measured before (16 rows at a time, X read for each, transposes behind the barrier) and now, us, batch 8 / 16 / 32 / 64 at 50 %:
// 4096 x 11008: 20.0 / 21.1 / 26.0 / 39.0 -> 17.3 / 19.7 / 24.7 / 33.0; 11008 x 4096: 23.4 / 23.1 / 29.3 / 43.2 -> 18.7 /
// 21.9 / 27.6 / 30.4; 4096 x 4096: 12.3 / 11.4 / 13.4 / 19.1 -> 7.9 / 9.1 / 11.9 / 15.9; 11008 x 4096 at 90 %, 64: 35.4 -> 19.9.
// Over 7441 calls of 256 to 14336 rows and columns, 30 to 97 % pruned, 2 to 64 vectors, 0.73 of the time (geometric mean).  Slower than
// before are dense rows of many columns on few compute units, where the clearing of a window and the wait for its vectors show: 17 to 32
// vectors on 2049 to 3700 rows (3635 x 13192 at 47 %, 31: 27.4 -> 29.5; 2720 x 11160 at 33 %, 26: 25.0 -> 25.9), 9 to 16 on up to 4096 rows of more than
// 18000 columns (2409 x 20936 at 47 %, 16: 30.6 -> 32.2; 102 x 139864 at 89 %, 10: 93.6 -> 102; clearing inside the product gives the last
// back what it lost, and takes as much from all others), and 9 to 16 on three tiles a workgroup of 4097 to 6144 columns (11976 x 5544 at 40 %, 16:
// 33.0 -> 35.5; panels of one tile 34.0, but at 80 % 25.0 instead of 23.8).
//
// Tried: two workgroups of 8 wavefronts per compute unit, each with half of the rows (5 to 30 % slower: X is read twice, and
// more windows); 512-column windows in two buffers for panels of 48 rows (34 -> 41 us); a ring of 2 to 4 steps of loads refilled one by one
// (no gain over units of S steps); 3 and 4 steps per unit (within 3 % either way); the prefix sums of a unit's steps interleaved
// (no gain); B loaded straight into the operand's lane order (16 vectors on 16 neighbouring lanes: every lane is a
// memory request of its own).
#include "macko_decode.h"
#include "macko_device.h"
#include "macko_internal.h"

namespace macko {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 16;                             // wavefronts of a workgroup, and rows of a tile
// Bytes in front of every row of the tile (and behind the last) that are written but never read: entries
// in front of the window or behind it land there.  A lane's 8 entries span at most 8 * 2 * 16 bytes.
constexpr int kTilePad = 256;
constexpr int kHalfVectors = 8;                        // up to here two groups of columns share one operand (HALF in the kernel)
// 16 bytes more per row: the 16 rows that a matrix instruction reads at one column fall on different banks
constexpr int panel_stride(int window) { return 2 * window + kTilePad + 16; }
constexpr int panel_slices(int vs) { return kWaves / vs; }       // wavefronts along the columns of a window

struct TileArgs {
  const void* values;
  const uint32_t* deltas;
  const uint32_t* row_ptr;
  const uint16_t* X;
  uint16_t* Y;
  int64_t ldx, ldy;
  int rows, cols, batch, q, r;                         // fours of rows per workgroup: q, one more for the first r
  int window;                                          // columns of a window, a multiple of 128
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
// the value of the lane 8 further on within the 16 (8 further back for the upper 8)
__device__ __forceinline__ float half_row_swap(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x128, 0xf, 0xf, true));
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

// NT: tiles of 16 vectors; a launch of more vectors has several rows of workgroups.  P: tiles of 16 rows in a panel.  W: columns
// of the largest window (a.window: of this launch's).  VS: parts into which the vector tiles are dealt to the wavefronts.
// HALF: up to 8 vectors, see below.  DBL: two buffers.  S: steps of 512 entries that are loaded, taken and decoded together (a unit).
// AHEAD: the vectors are requested behind the product of the window before.
//
// Window by window, a wavefront
//  - clears its own rows of the tile and puts what it holds of them (the last unit taken may reach into several windows: its
//    codes, values and position stay in registers until the row's next unit takes their place);
//  - takes further units of its P rows until every row has passed the window's end.  All rows' units are taken out of the load
//    registers before the next ones are requested (the compiler waits for every load under way where it cannot count
//    them, so a take behind a request would wait for that request);
//  - requests the window's vectors a few at a time between the rows' decodes (all at once they hold up the wavefront:
//    16 clocks of L1 each, 128 of them), and turns them into operand order in front of the barrier, where the early wavefronts wait.
//    One tile of vectors and of rows requests them in front of the decode: there are only four or eight, and behind it the second
//    unit of a window waits for them (2409 x 20936 at 47 %, 16 vectors: 37.1 -> 34.2 us, 2636 x 13808 at 41 %, 15: 26.3 -> 24.9,
//    4096 x 11008 at 50 %, 8: 17.7 -> 17.2).
//    AHEAD (panels of one tile): behind the product of the window before, so that barrier and decode cover them.  The take of the window's
//    first unit may not wait for them, so the compiler has to be able to count: the requests stand in a straight line behind all others
//    on every way there (what a window lacks is requested behind the buffer's end), and the first unit is taken in front of
//    the loop.  It costs shorter rows more than it gives.  us, without / with: 17 to 32 vectors, from 7 steps a row on, 3635 x 13192
//    at 47 % 32.1 / 29.5, 2720 x 11160 at 33 % 27.5 / 25.9, 4096 x 10508 at 35 %, 8-bit values, 26.5 / 23.9, 4096 x 7386 at 51 % 17.4 / 17.1, but 2300 x 3000
//    at 70 % 7.3 / 7.6; 9 to 16 vectors, from 14 on, 2409 x 20936 at 47 % 33.8 / 32.2, 4096 x 12696 at 31 % 26.6 / 25.8, but 2657 x 13835 at 59 %, 8-bit
//    values, 24.4 / 25.3, 2100 x 6000 at 50 % 10.7 / 11.9; up to 8 vectors and 33 and more not tried with it, or no better (4096 x 11008 at 80 %, 8: 12.3 / 12.7);
//  - behind the barrier multiplies its columns' part: the window's groups of 128 columns are dealt to kSlices wavefronts
//    for each of the VS parts of the vectors (part vpart), every one for all tiles of rows.
// With two buffers the next window goes into the other one at once; with one a second barrier keeps it apart.  The pad behind a row is
// the one in front of the next: two wavefronts may write it, nobody reads it.
// Every wavefront executes the same number of barriers whatever its rows hold.
template <int NT, int P, int W, int VS, bool DBL, int S, bool HALF, bool AHEAD, int BD, int VB>
__global__ void __launch_bounds__(64 * kWaves)
spmm_panel_kernel(const TileArgs all) {
  TileArgs a = all;                                    // this workgroup's vectors
  constexpr int kVectors = HALF ? kHalfVectors : 16 * NT;
  a.X += (int64_t)blockIdx.y * kVectors * a.ldx;
  a.Y += (int64_t)blockIdx.y * kVectors * a.ldy;
  a.batch = min(a.batch - (int)blockIdx.y * kVectors, kVectors);
  static_assert(BD <= 4, "a lane's 8 entries have to fit the pad");
  constexpr int kSlices = panel_slices(VS), G = W / 128 / kSlices;          // groups of columns of a wavefront
  static_assert(kSlices * G * 128 == W && kSlices * VS == kWaves && NT % VS == 0, "every wavefront has its part of a window");
  static_assert(!HALF || (NT == 1 && G % 2 == 0), "pairs of groups of one vector tile");
  static_assert(!AHEAD || P == 1, "one unit is taken at a time");
  constexpr int BG = HALF ? G / 2 : G, kPair = HALF ? 2 : 1;                // operands of a wavefront, groups of each
  constexpr int NTW = NT / VS;                                              // vector tiles of a wavefront
  constexpr int kStride = panel_stride(W), kBuffer = 16 * P * kStride;
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ uint32_t odd_results[64 * kWaves][2];     // per row of the workgroup, a bit per vector: not finite
  __shared__ uint32_t any_odd;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wg = (int)blockIdx.x;
  const int row0 = 4 * (wg * a.q + min(wg, a.r));
  const int wg_rows = min(4 * (a.q + (wg < a.r ? 1 : 0)), a.rows - row0);
  const int panels = (wg_rows + 16 * P - 1) / (16 * P);
  const int nb = wave < wg_rows ? (wg_rows - wave + 15) / 16 : 0;     // this wavefront's rows (at most 64: the host sees to that)
  const int cols = a.cols, wr = a.window;
  const uint32_t lane8 = 8u * lane;

  uint32_t rp_lo, rp_hi;                               // lane i: the pointers of the wavefront's row i
  {
    const int r = min(row0 + wave + 16 * lane, a.rows - 1);
    rp_lo = a.row_ptr[r];
    rp_hi = a.row_ptr[r + 1];
  }

  const int slice = wave % kSlices, vpart = wave / kSlices % VS;
  const int n = lane & 15;
  const uint32_t aoff = kTilePad + n * kStride + 2 * (128 * G * slice + 32 * (lane >> 4));
  const bool odd_lane = lane & 1, high_lane = lane & 2;
  // The vectors are one buffer (base rounded down to 4 bytes): what lies behind its end, vectors past the batch among
  // it, reads as zero; what lies between two vectors is cleared where it is used.  The end is checked per 4 bytes, so
  // the buffer ends in front of the last element of an odd number of columns: the last vector's is loaded by itself and put in its
  // place where the vectors end.  (The other vectors' are inside; a single column is not served.)
  const uint32_t xmis = (uint32_t)(reinterpret_cast<uintptr_t>(a.X) & 2);
  const uint32_t xbytes = (uint32_t)(((int64_t)(a.batch - 1) * a.ldx + (cols & ~1)) * 2) + xmis;
  uint32_t last_x = 0u;
  if (cols & 1) last_x = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.X[(int64_t)(a.batch - 1) * a.ldx + cols - 1]);
  const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<unsigned char*>(reinterpret_cast<const unsigned char*>(a.X) - xmis), 0, (int)xbytes, 0x00020000);
  const uint32_t ldx2 = 2u * (uint32_t)a.ldx;
  // HALF, up to 8 vectors: the lanes of vectors 8 ... 15 take vectors 0 ... 7 of the next group instead, so that one operand serves two
  // groups.  The products of the first count in lanes 0 ... 7 of each 16, those of the second in lanes 8 ... 15 of another sum.
  // Half the loads and transposes: 4096 x 11008 at 50 %, 8 vectors, 19.2 -> 17.4 us, 4096 x 4096 8.7 -> 7.9, 300 x 13000 at 80 % 16.0 -> 13.8.
  const int bcol = 128 * G * slice + (HALF ? 128 * ((lane >> 3) & 1) : 0) + 8 * (4 * (lane >> 4) + (lane & 3));        // the lane's first column within the window
  const uint32_t xoff = xmis + (uint32_t)(16 * vpart + 4 * ((lane >> 2) & (HALF ? 1 : 3))) * ldx2 + 2u * bcol;
  u32x4 b[BG][NTW][4];
  int k0 = 0;                                          // first column of the window
  // loads `from` ... `to` - 1 of the window's 4 BG NTW
  auto load_b = [&](int from, int to) {
#pragma unroll
    for (int g = 0; g < BG; ++g)
      if ((AHEAD || 128 * (G * slice + kPair * g) < min(wr, cols - k0)) && to > 4 * NTW * g && from < 4 * NTW * (g + 1)) {
        uint32_t xo = xoff + 2u * (uint32_t)(k0 + 128 * kPair * g);
        if (AHEAD && 128 * (G * slice + kPair * g) >= min(wr, cols - k0)) xo = 0x80000000u;      // behind the buffer's end: zeros, and nothing is read
        asm volatile("" : "+v"(xo));
#pragma unroll
        for (int i = 0; i < 4 * NTW; ++i)
          if (4 * NTW * g + i >= from && 4 * NTW * g + i < to) {
            const auto q = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, (int)(xo + (uint32_t)(16 * VS * (i >> 2) + (i & 3)) * ldx2), 0, 0);
            b[g][i >> 2][i & 3] = u32x4{(uint32_t)q[0], (uint32_t)q[1], (uint32_t)q[2], (uint32_t)q[3]};
          }
      }
  };

  LaneCodes<BD> rw[P][S], hw[P][S];
  LaneValues<VB> rv[P][S], hv[P][S];
  int hbase[P][S];                                     // lane's doubled position
  int hend[P][S];                                      // doubled position behind the step
  uint32_t e0[P], start[P], end[P];
  int base2[P];
  int left[P];                                         // units of S steps not taken yet
  int j0 = 0;                                          // the wavefront's row of slot 0
  auto issue = [&](int p, uint32_t from, uint32_t to) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const uint32_t chunk = min(from + 512u * s + lane8, max(to, 1u) - 1u) >> 3;
      rw[p][s].load(a.deltas, chunk);
      rv[p][s].load(a.values, chunk);
    }
  };
  auto open_row = [&](int p) {
    const int j = min(j0 + p, 63);
    start[p] = (uint32_t)__builtin_amdgcn_readlane((int)rp_lo, j);
    end[p] = (uint32_t)__builtin_amdgcn_readlane((int)rp_hi, j);
    e0[p] = start[p] & ~7u;
    left[p] = j0 + p < nb ? (int)panel_row_units(start[p], end[p], 512u * S) : 0;
    base2[p] = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) hend[p][s] = -1;
  };
  if (NT == 1 && !AHEAD) load_b(0, 4 * BG * NTW);      // under way while the row pointers are waited for
#pragma unroll
  for (int p = 0; p < P; ++p) {
    open_row(p);
    if (left[p] > 0) issue(p, e0[p], end[p]);
  }
  if (NT > 1 || AHEAD) load_b(0, 4 * BG * NTW);        // many of them would hold up the first units
  odd_results[threadIdx.x][0] = odd_results[threadIdx.x][1] = 0u;
  if (threadIdx.x == 0) any_odd = 0u;

  float4v acc[P][NTW], acc_pair[P];                    // acc_pair: HALF, the second groups' sums
#pragma unroll
  for (int i = 0; i < P; ++i) {
    acc_pair[i] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NTW; ++t) acc[i][t] = float4v{0.f, 0.f, 0.f, 0.f};
  }

  const int cols2 = 2 * ((cols + 127) & ~127);
  const bool y_aligned = (reinterpret_cast<uintptr_t>(a.Y) & 7) == 0 && a.ldy % 4 == 0;
  uint32_t buf = 0;                                    // byte offset of the window's buffer
  int panel = 0;
  bool b_due = false;
  for (;;) {
    // ---- the window's part of this wavefront's rows into the tile
    const uint32_t put_bytes = (uint32_t)min(2 * wr, cols2 - 2 * k0) + kTilePad;
    const bool last_window = k0 + wr >= cols;
    const int limit = last_window ? 0x7FFFFFFF : 2 * (k0 + wr);       // everything that is left goes to the last window
    unsigned char* rowbuf = lds + buf + kTilePad + wave * kStride;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int i = 0; i < W / 512; ++i)
        *reinterpret_cast<u32x4*>(rowbuf + 16 * p * kStride + 1024 * i + 16 * lane) = u32x4{0, 0, 0, 0};
    asm volatile("" ::: "memory");
    auto put = [&](int p, int s) {
      const int rel = hbase[p][s] - 2 * k0;
      if ((uint32_t)(rel + kTilePad) < put_bytes) {
        unsigned char* q = rowbuf + 16 * p * kStride + rel;
#define MACKO_PUT(K) *reinterpret_cast<uint16_t*>(q + hw[p][s].template offset<K>()) = (uint16_t)hv[p][s].template half<K>();
        MACKO_PUT(0) MACKO_PUT(1) MACKO_PUT(2) MACKO_PUT(3) MACKO_PUT(4) MACKO_PUT(5) MACKO_PUT(6) MACKO_PUT(7)
#undef MACKO_PUT
      }
    };
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (hend[p][s] > 2 * k0) {
          if (P > 2 || NTW * S > 6) {                  // every register counts: the codes are kept, not the positions
            keep_opaque(hw[p][s].w, hv[p][s]);
            hw[p][s].decode();
          }
          put(p, s);
        }
    if (NT * P == 1 && b_due) {
      load_b(0, 4 * BG * NTW);
      b_due = false;
    }
    // out of the load registers with the next unit of every row that has not passed the window's end (bit p: of row p), all of them first
    auto take = [&]() -> uint32_t {
      uint32_t need = 0;
#pragma unroll
      for (int p = 0; p < P; ++p) need |= (uint32_t)(left[p] > 0 && base2[p] < limit) << p;
#pragma unroll
      for (int p = 0; p < P; ++p)
        if (need & (1u << p)) {
#pragma unroll
          for (int s = 0; s < S; ++s) {
            move_regs(hw[p][s].w, rw[p][s].w);
            move_regs(hv[p][s], rv[p][s]);
          }
          e0[p] += 512u * S;
          --left[p];
        }
      return need;
    };
    uint32_t first = AHEAD ? take() : 0u;
    for (;;) {
      const uint32_t need = AHEAD && first ? first : take();
      first = 0u;
      if (!need && !b_due) break;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int p = 0; p < P; ++p) {
        if (need & (1u << p)) {
          const bool more = left[p] > 0;
          const int j = j0 + p + P;
          if (more || j < nb) {
            const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)rp_lo, j & 63) & ~7u;
            const uint32_t to = (uint32_t)__builtin_amdgcn_readlane((int)rp_hi, j & 63);
            issue(p, more ? e0[p] : from, more ? end[p] : to);
          }
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const uint32_t e = e0[p] - 512u * (uint32_t)(S - s);
            if (s > 0 && e >= end[p]) {
              hend[p][s] = -1;
            } else {
              LaneCodes<BD>& w = hw[p][s];
              if (e + 512u > end[p]) {                 // the row's last step: clear what lies behind its end
                const uint32_t nv = e + lane8 < end[p] ? end[p] - (e + lane8) : 0u;
                w.keep_if(nv != 0);
                hv[p][s].keep_first(nv);
              }
              w.decode();
              const uint32_t tot = w.total();
              const uint32_t incl = wave_incl_scan_u32(tot);
              if (s == 0 && e <= start[p]) {           // the row's first step
                const int before = (int)(start[p] - e);      // entries of the previous row: they land in front of column 0
                if (before > 0) base2[p] = -(int)w.through(before - 1);
              }
              hbase[p][s] = base2[p] + (int)(incl - tot);
              base2[p] += (int)__builtin_amdgcn_readlane((int)incl, 63);
              hend[p][s] = base2[p];
              put(p, s);
            }
          }
        }
        if (b_due) load_b(4 * BG * NTW * p / P, 4 * BG * NTW * (p + 1) / P);
      }
      b_due = false;
    }
    // the vectors into the operand's layout
    const int groups = min(wr, cols - k0);             // columns of the window that are multiplied
#pragma unroll
    for (int g = 0; g < BG; ++g)
      if (128 * (G * slice + kPair * g) < groups) {
        if (__builtin_expect(k0 + 128 * (G * slice + kPair * g) + 128 * kPair > cols, 0)) {      // the vectors end in it
          int l = lane;
          if (NTW > 1) asm volatile("" : "+v"(l));
          const int left = cols - (k0 + 128 * (G * slice + kPair * g + (HALF ? (l >> 3) & 1 : 0)) + 8 * (4 * (l >> 4) + (l & 3)));
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t mask = left > 2 * i + 1 ? 0xFFFFFFFFu : (left > 2 * i ? 0xFFFFu : 0u);
#pragma unroll
            for (int t = 0; t < NTW; ++t)
#pragma unroll
              for (int r = 0; r < 4; ++r) b[g][t][r][i] &= mask;
          }
          if (__builtin_expect(cols & 1, 0)) {         // the last element of the last vector (left is odd here)
            const int last = a.batch - 1 - 16 * vpart - 4 * ((l >> 2) & (HALF ? 1 : 3));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const uint32_t e = left == 2 * i + 1 ? last_x : 0u;
#pragma unroll
              for (int t = 0; t < NTW; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) b[g][t][r][i] |= last == 16 * VS * t + r ? e : 0u;
            }
          }
        }
#pragma unroll
        for (int t = 0; t < NTW; ++t) {
          quad_transpose(b[g][t], odd_lane, high_lane);
          if (NTW > 1) __builtin_amdgcn_sched_barrier(0);        // keeps the temporaries of one t at a time: no spills
        }
      }
    __syncthreads();                                   // every row's entries of the window are in the tile
    // ---- the product of the window
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (128 * (G * slice + g) < groups) {
        const unsigned char* ap = lds + buf + aoff + 256 * g;
#pragma unroll
        for (int i = 0; i < P; ++i) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const half8 av = *reinterpret_cast<const half8*>(ap + 16 * i * kStride + 16 * r);
#pragma unroll
            for (int t = 0; t < NTW; ++t) {
              float4v& sum = HALF && g % 2 == 1 ? acc_pair[i] : acc[i][t];
              sum = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, __builtin_bit_cast(half8, b[g / kPair][t][r]), sum, 0, 0, 0);
            }
          }
        }
      }
    b_due = !AHEAD;
    if (!last_window) {
      k0 += wr;
      if (AHEAD) {
        __builtin_amdgcn_sched_barrier(0);
        load_b(0, 4 * BG * NTW);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (DBL) buf = kBuffer - buf;
      else __syncthreads();                            // the tile has been read
      continue;
    }
    // ---- the results of the panel: the slices' sums are handed over in the tile's memory (the other buffer's, if there are two)
    k0 = 0;
    float4v* red = reinterpret_cast<float4v*>(lds + kTilePad + (DBL ? kBuffer - buf : 0));      // [P * NT][kSlices][64]
    if (HALF) {
#pragma unroll
      for (int i = 0; i < P; ++i) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][0][e] += half_row_swap(acc_pair[i][e]);
        acc_pair[i] = float4v{0.f, 0.f, 0.f, 0.f};
      }
    }
    if (!DBL) __syncthreads();
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
      for (int t = 0; t < NTW; ++t) {
        red[((i * NT + VS * t + vpart) * kSlices + slice) * 64 + lane] = acc[i][t];
        acc[i][t] = float4v{0.f, 0.f, 0.f, 0.f};
      }
    __syncthreads();
    for (int u = wave; u < P * NT; u += kWaves) {
      const float4v* p = red + u * kSlices * 64 + lane;
      float4v sum = *p;
      int l = lane;
      if (NTW > 1) asm volatile("" : "+v"(l));       // no pointers into Y kept in registers
      const int n = l & 15;
#pragma unroll
      for (int g = 1; g < kSlices; ++g) sum += p[64 * g];
      const int rt = u / NT, vt = u - NT * rt;
      const int m0 = 16 * (P * panel + rt) + 4 * (l >> 4), left = wg_rows - m0;     // lane holds rows m0 ... m0 + 3
      if (16 * vt + n < a.batch) {
        uint16_t* y = a.Y + (int64_t)(16 * vt + n) * a.ldy + (row0 + m0);
        bool fine = true;                              // no infinity and no NaN in the rows or in the vector
#pragma unroll
        for (int i = 0; i < 4; ++i) fine = fine && __builtin_fabsf(sum[i]) <= 3.4028234e38f;
        if (fine && left >= 4 && y_aligned) {
          *reinterpret_cast<uint2*>(y) = make_uint2(f32_to_f16_bits(sum[0]) | (uint32_t)f32_to_f16_bits(sum[1]) << 16,
                                                    f32_to_f16_bits(sum[2]) | (uint32_t)f32_to_f16_bits(sum[3]) << 16);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (i < left) {
              if (__builtin_fabsf(sum[i]) <= 3.4028234e38f) {
                y[i] = f32_to_f16_bits(sum[i]);
              } else {
                atomicOr(&odd_results[m0 + i][vt >> 1], 1u << (16 * (vt & 1) + n));
                any_odd = 1u;
              }
            }
        }
      }
    }
    if (++panel == panels) break;
    j0 += P;
#pragma unroll
    for (int p = 0; p < P; ++p) open_row(p);
    if (AHEAD) load_b(0, 4 * BG * NTW);
    if (!DBL) __syncthreads();                         // the sums have been read
  }
  __syncthreads();
  if (any_odd) {
    for (int i = 0; i < nb; ++i) {
      const int r = 16 * i + wave;
      const uint64_t vectors = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)odd_results[r][0]) |
                               ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)odd_results[r][1]) << 32);
      if (vectors)
        tile_row_by_entries<BD, VB>(a, row0 + r, (uint32_t)__builtin_amdgcn_readlane((int)rp_lo, i),
                                    (uint32_t)__builtin_amdgcn_readlane((int)rp_hi, i), vectors);
    }
  }
}

template <int NT, int P, int W, int VS, bool DBL, int S, bool HALF, bool AHEAD, int BD, int VB>
int launch_panel_as(TileArgs a, hipStream_t stream) {
  constexpr int vectors = HALF ? kHalfVectors : 16 * NT;
  constexpr int buffer = 16 * P * panel_stride(W), lds = (DBL ? 2 : 1) * buffer + kTilePad;
  static_assert(P * NT * panel_slices(VS) * 1024 + kTilePad <= buffer, "the partial sums fit one buffer");
  static_assert(lds + 64 * kWaves * 8 + 16 <= 160 * 1024, "LDS of a compute unit");
  auto kfn = spmm_panel_kernel<NT, P, W, VS, DBL, S, HALF, AHEAD, BD, VB>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return hip_fail(e);
  // One workgroup per compute unit with an equal share of the rows: LDS holds no second one, and the fewer workgroups,
  // the fewer times the vectors are read.  A wavefront keeps the pointers of at most 64 rows.
  int64_t grid = std::min<int64_t>(((int64_t)a.rows + 15) / 16, (int64_t)device_cu_count());
  grid = std::max<int64_t>(grid, ((int64_t)a.rows + 64 * 16 - 1) / (64 * 16));
  const int64_t fours = ((int64_t)a.rows + 3) / 4;     // four results of a vector lie in one lane: stored together 11008 x 4096, 64 vectors: 33.1 -> 32.1 us
  a.q = (int)(fours / grid);
  a.r = (int)(fours % grid);
  // as few windows as LDS allows, all about equally wide (11008 columns: 6 of 1920 instead of 5 of 2048 and one of 768)
  const int64_t windows = ((int64_t)a.cols + W - 1) / W;
  a.window = (int)((((int64_t)a.cols + windows - 1) / windows + 127) / 128 * 128);
  hipLaunchKernelGGL(kfn, dim3((unsigned)grid, (unsigned)((a.batch + vectors - 1) / vectors)), dim3(64 * kWaves), (size_t)lds, stream, a);
  e = hipGetLastError();
  return e == hipSuccess ? MACKO_OK : hip_fail(e);
}

// Tiles of 16 rows per workgroup, and whether up to 16 vectors take panels of two of them: whole rows of up to 4096 columns in one
// window, or two tiles in windows of half that width where that makes no more windows (us, one / two: 8192 x 4096 at 80 % 12.1 /
// 11.3, 14336 x 700 13.6 / 9.5; but 11008 x 4096 at 90 % 15.2 / 15.8)
int64_t tiles_per_wg(int64_t rows) {
  const int64_t cus = device_cu_count();
  return (rows + 16 * cus - 1) / (16 * cus);
}
bool two_tiles(int64_t tiles, int64_t cols) {
  return tiles > 1 && (tiles + 1) / 2 * ((cols + 2047) / 2048) <= tiles * ((cols + 4095) / 4096);
}

// Whether the vectors go in groups of at most 8, each with a workgroup of its own for every 16 rows: where one group is all there is,
// and where the compute units hold all groups at once.
bool eights_fit(int64_t rows, int64_t cols, int batch) {
  if (batch <= kHalfVectors) return !two_tiles(tiles_per_wg(rows), cols);
  return (rows + 15) / 16 * ((batch + kHalfVectors - 1) / kHalfVectors) <= device_cu_count();
}

// The shape of a launch.  A workgroup's work is its panels times their windows, about 2 us each, and the reads of X once per panel.
// Figures: us at the sizes given, from 260 matrices timed with every shape.
// row_entries: stored entries of a row on average.
template <int BD, int VB>
int launch_tile_bd(const TileArgs& a, int64_t row_entries, hipStream_t stream) {
  const int64_t cus = device_cu_count();
  const int64_t tiles = tiles_per_wg(a.rows);
  const bool dense = 4 * row_entries >= a.cols;        // more than one step of a row in 2048 columns
  int nt = (a.batch + 15) / 16;
  // Few rows leave compute units idle: they take the same rows with other vectors, in groups of 8 if there are enough of them, else
  // of 16 (256 x 4096, 64 vectors: 14.9 -> 8.7 in groups of 16, 7.9 in
  // groups of 8; 106 x 13022 at 52 %, 16: 22.2 -> 18.9; but 300 x 700, 64: 5.7 and 6.1).
  const bool half = eights_fit(a.rows, a.cols, a.batch);
  if (!half && a.rows <= 8 * cus) {
    const int groups = (int)std::min<int64_t>(nt, cus / ((a.rows + 15) / 16));
    nt = (nt + groups - 1) / groups;
  }
#define MACKO_PANEL(...) return launch_panel_as<__VA_ARGS__, BD, VB>(a, stream)
  if (half || nt == 1) {
    if (!half && two_tiles(tiles, a.cols)) MACKO_PANEL(1, 2, 2048, 1, false, 1, false, false);
    // few long rows: nothing but each wavefront's own loads hides their latency (300 x 13000 at 80 %, 16 vectors: 13.6 with two steps a
    // unit, 13.2).  In groups of 16 three are no better (1500 x 9000, 32: 15.5 / 15.5; 700 x 30000, 48: 42.2 / 43.0).
    if (half && a.rows <= 8 * cus && a.cols > 8192) MACKO_PANEL(1, 1, 4096, 1, false, 3, true, false);
    if (half) MACKO_PANEL(1, 1, 4096, 1, false, 2, true, false);
    if (row_entries >= 14 * 512) MACKO_PANEL(1, 1, 4096, 1, false, 2, false, true);          // see AHEAD
    MACKO_PANEL(1, 1, 4096, 1, false, 2, false, false);
  }
  // From here on X counts as well: the shape whose panels have the fewest empty places, 3 tiles if equal
  const bool three = (tiles + 2) / 3 * 3 <= (tiles + 1) / 2 * 2;
  if (nt == 2) {
    if (tiles == 1 && row_entries >= 7 * 512) MACKO_PANEL(2, 1, 2048, 1, true, 2, false, true);
    if (tiles == 1) MACKO_PANEL(2, 1, 2048, 1, true, 2, false, false);
    if (three) MACKO_PANEL(2, 3, 1024, 2, false, 1, false, false);                   // 10000 x 1800: 15.3 with panels of 2, 13.5
    MACKO_PANEL(2, 2, 2048, 1, false, 1, false, false);                              // 5000 x 4096: 18.5 with panels of 1, 15.4
  }
  if (tiles == 1) {
    if (nt == 3) MACKO_PANEL(3, 1, 2048, 1, true, 2, false, false);                  // 4096 x 4096: 15.2; with a fourth, empty tile 17.1
    if (a.cols <= 3072) MACKO_PANEL(4, 1, 1024, 2, true, 2, false, false);           // 4096 x 2600: 13.1 / 14.2 with 2048, 4096 x 4096 at 90 %: 13.5 / 12.6
    // dense rows: two steps loaded at a time (us, one / two: 2100 x 13256, 64 vectors, at 30 % 50.9 / 44.1, at
    // 50 % 44.5 / 38.8, at 70 % 35.9 / 34.9; 4096 x 11008 at 50 % 35.9 / 33.2, but at 80 % 28.2 / 28.4, at 90 % 25.7 / 26.7)
    if (dense) MACKO_PANEL(4, 1, 2048, 1, true, 2, false, false);
    MACKO_PANEL(4, 1, 2048, 1, true, 1, false, false);
  }
  if (three) MACKO_PANEL(4, 3, 1024, 2, false, 1, false, false);                     // 11008 x 4096: 40.9 with panels of 2, 33.1
  MACKO_PANEL(4, 2, 1024, 2, true, 1, false, false);                                 // 8192 x 4096 at 80 %: 22.8 with panels of 1, 19.0
#undef MACKO_PANEL
}

}  // namespace

bool spmm_tile_serves(const SpmvProblem& p, int64_t ldx) {
  if (p.b_delta > 4 || p.pad_nnz == 0 || p.rows == 0) return false;   // the pad of the tile holds 4-bit deltas
  if (p.cols < 2) return false;                        // see the end of the vectors' buffer in the kernel
  return ldx < (int64_t{1} << 24);                     // vectors are addressed with 32-bit byte offsets
}

int64_t spmm_tile_windows(const SpmvProblem& p) {
  const int64_t tiles = tiles_per_wg(p.rows);
  return two_tiles(tiles, p.cols) ? (tiles + 1) / 2 * ((p.cols + 2047) / 2048) : tiles * ((p.cols + 4095) / 4096);
}

bool spmm_tile_pairs_groups(const SpmvProblem& p, int batch) { return eights_fit(p.rows, p.cols, batch); }

int launch_spmm_tile(const SpmvProblem& p, const uint16_t* X, int64_t ldx, uint16_t* Y, int64_t ldy, int batch,
                     hipStream_t stream) {
  const TileArgs a{p.values, reinterpret_cast<const uint32_t*>(p.deltas), p.row_ptr, X, Y, ldx, ldy,
                   (int)p.rows, (int)p.cols, batch, 0, 0, 0};
  if (p.b_val == 8) return p.b_delta == 4 ? launch_tile_bd<4, 8>(a, p.pad_nnz / p.rows, stream) : MACKO_E_UNSUPPORTED;
  switch (p.b_delta) {
    case 1: return launch_tile_bd<1, 16>(a, p.pad_nnz / p.rows, stream);
    case 2: return launch_tile_bd<2, 16>(a, p.pad_nnz / p.rows, stream);
    case 4: return launch_tile_bd<4, 16>(a, p.pad_nnz / p.rows, stream);
    default: return MACKO_E_UNSUPPORTED;
  }
}

}  // namespace macko
