// The memory of the GPU encoder's handles, without a GPU: the library's host translation unit linked with a stand-in for the HIP
// runtime that counts what is allocated and which allocation a device has waited on (hipFree waits until the device is idle), and with an encoder
// that only takes its block.  Built and run by tests/test_library_host.py; prints "ok" on success.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <vector>

#include "macko_internal.h"

static int failures = 0;
#define EXPECT(cond, ...)                                                                              \
  do {                                                                                                 \
    if (!(cond)) {                                                                                     \
      std::printf("FAIL line %d %s: ", __LINE__, #cond);                                               \
      std::printf(__VA_ARGS__);                                                                        \
      std::printf("\n");                                                                               \
      ++failures;                                                                                      \
    }                                                                                                  \
  } while (0)

// ---- the runtime ----------------------------------------------------------------
struct Allocation {
  size_t bytes;
  int device;
};
static std::map<void*, Allocation> live;
static std::set<void*> busy;                            // blocks that work still under way on their device uses
static int device = 0, mallocs = 0;
static size_t used[2] = {}, capacity = size_t{64} << 30;
static bool small_ones_fail = false;
static uintptr_t next_address = 1 << 20;

extern "C" {
hipError_t hipMalloc(void** p, size_t bytes) {
  ++mallocs;
  if (used[device] + bytes > capacity || (small_ones_fail && bytes <= 16)) return hipErrorOutOfMemory;
  *p = reinterpret_cast<void*>(next_address);
  next_address += (bytes + 4095) / 4096 * 4096;
  used[device] += bytes;
  live[*p] = {bytes, device};
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  const auto at = live.find(p);
  EXPECT(at != live.end(), "freed twice, or never allocated: %p", p);
  if (at == live.end()) return hipErrorInvalidValue;
  for (auto b = busy.begin(); b != busy.end();) b = live.count(*b) && live[*b].device == at->second.device ? busy.erase(b) : std::next(b);
  used[at->second.device] -= at->second.bytes;
  live.erase(at);
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { return *d = device, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned int) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t*, unsigned) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
}

// ---- the launchers ---------------------------------------------------------------
namespace macko {
int launch_spmv_group(int, const SpmvProblem*, int64_t, hipStream_t) { std::abort(); }
int launch_gemv_group(int, const GemvProblem*, hipStream_t) { std::abort(); }
int launch_spmv_chain(int, const int*, const SpmvProblem*, uint32_t*, uint32_t, hipStream_t) { std::abort(); }
int chain_static_scratch(uint32_t**) { std::abort(); }
int launch_spmm(const SpmvProblem&, const void*, int64_t, void*, int64_t, int, hipStream_t) { std::abort(); }
int launch_columns(const SpmvProblem&, int32_t*, hipStream_t) { std::abort(); }
int launch_check(const SpmvProblem&, unsigned int*, hipStream_t) { return MACKO_OK; }
int launch_decode(const SpmvProblem&, void*, int64_t, hipStream_t) { std::abort(); }
// every cell is kept
int encode_on_device(const void*, int64_t rows, int64_t cols, int64_t, int b_delta, int b_val, hipStream_t, void** block, void** values,
                     uint8_t** deltas, uint32_t** row_ptr, int64_t* nnz, int64_t* pad_nnz, int64_t* alloc_nnz, int64_t* empty_rows,
                     int64_t* max_row_entries) {
  const int64_t granule = alloc_granule(b_delta), alloc = (rows * cols + granule - 1) / granule * granule;
  const EncodedLayout layout = encoded_layout(rows, alloc, b_delta, b_val);
  if (block_acquire(block, layout.total) != hipSuccess) return MACKO_E_OUT_OF_MEMORY;
  EXPECT(live.count(*block) && live[*block].device == device && live[*block].bytes >= layout.total, "a block of %zu bytes", layout.total);
  EXPECT(!busy.count(*block), "the block is still in use");
  *values = *block;
  *deltas = static_cast<uint8_t*>(*block) + layout.deltas;
  *row_ptr = reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(*block) + layout.row_ptr);
  *nnz = *pad_nnz = rows * cols;
  *alloc_nnz = alloc;
  *empty_rows = 0;
  *max_row_entries = cols;
  return MACKO_OK;
}
}  // namespace macko

static macko_handle_t encoded(int64_t rows, int64_t cols, int want = MACKO_OK) {
  static int something;
  macko_handle_t h = nullptr;
  const int st = macko_encode_device(&something, rows, cols, cols, nullptr, &h, nullptr);
  EXPECT(st == want, "%lld x %lld: %d", (long long)rows, (long long)cols, st);
  return h;
}
static size_t large_ones() {
  size_t n = 0;
  for (const auto& a : live) n += a.second.bytes > 16;
  return n;
}

int main() {
  const size_t MiB = size_t{1} << 20;
  // A block goes to the next handle of its size class, and only after a wait for the device
  macko_handle_t h = encoded(2048, 4096);
  void* first = h->d_block;
  busy.insert(first);                                   // some stream still reads it
  macko_destroy(h);
  EXPECT(live.count(first) && busy.empty(), "kept, and idle");
  const int before = mallocs;
  h = encoded(2049, 4096);                              // 0.05 % larger: the same class
  EXPECT(h->d_block == first && mallocs == before + 1, "reused; the only allocation is the one for the next wait");
  macko_handle_t other = encoded(2048, 4096);
  EXPECT(other->d_block != first, "handles that live share nothing");
  macko_destroy(other);
  macko_destroy(h);
  h = encoded(1024, 4096);
  EXPECT(h->d_block != first, "another size");
  macko_destroy(h);
  macko_trim();
  EXPECT(live.empty() && used[0] == 0, "%zu allocations left", live.size());

  // Small blocks are not kept, and take nothing for a wait
  h = encoded(100, 100);
  EXPECT(live.size() == 1, "%zu allocations", live.size());
  macko_destroy(h);
  EXPECT(live.empty(), "a small block is freed");

  // Bounds: 8 blocks and 256 MiB a device; a block larger than that is not kept
  std::vector<macko_handle_t> many;
  for (int i = 0; i < 20; ++i) many.push_back(encoded(1024, 4096));
  for (int i = 0; i < 19; ++i) macko_destroy(many[i]);
  EXPECT(large_ones() == 9, "%zu blocks: 8 kept and one in use", large_ones());
  macko_trim();
  EXPECT(large_ones() == 1, "the one in use");
  macko_destroy(many[19]);
  many.clear();
  for (int i = 0; i < 5; ++i) many.push_back(encoded(8192, 4096));
  for (macko_handle_t m : many) macko_destroy(m);
  EXPECT(used[0] <= 256 * MiB && large_ones() == 3, "%zu MiB in %zu blocks", used[0] / MiB, large_ones());
  h = encoded(32768, 4096);
  const size_t with = used[0];
  macko_destroy(h);
  EXPECT(used[0] + 300 * MiB < with, "320 MiB are not kept");
  macko_trim();
  EXPECT(live.empty(), "%zu allocations left", live.size());

  // Devices: a block stays on its own, whichever is current when its handle is destroyed
  h = encoded(2048, 4096);
  first = h->d_block;
  device = 1;
  macko_destroy(h);
  other = encoded(2048, 4096);
  EXPECT(other->d_block != first, "device 0's block");
  macko_destroy(other);
  macko_trim();
  EXPECT(used[1] == 0 && large_ones() == 1, "device 1 is trimmed, device 0 is not");
  device = 0;
  h = encoded(2048, 4096);
  EXPECT(h->d_block == first, "found on its device");
  macko_destroy(h);
  macko_trim();

  // Memory runs out: whatever the library allocates takes back what is kept
  h = encoded(2048, 4096);
  other = encoded(3000, 4096);
  macko_destroy(other);
  capacity = used[0];                                   // nothing left but the kept block
  EXPECT(macko_check_device(h, nullptr, nullptr) == MACKO_OK, "the check's 4 bytes");
  EXPECT(large_ones() == 1, "the kept block went for them");
  capacity = size_t{64} << 30;
  other = encoded(3000, 4096);
  macko_destroy(other);
  capacity = used[0] + MiB;
  other = encoded(2900, 4096);
  EXPECT(other && large_ones() == 2, "the kept block went for a new one");
  macko_handle_t none = encoded(2900, 4096, MACKO_E_OUT_OF_MEMORY);
  EXPECT(!none, "nothing left");
  macko_destroy(other);
  macko_destroy(h);
  capacity = size_t{64} << 30;
  macko_trim();
  EXPECT(live.empty(), "%zu allocations left", live.size());

  // no allocation for the wait: the block is freed with its handle
  small_ones_fail = true;
  h = encoded(2048, 4096);
  macko_destroy(h);
  EXPECT(live.empty(), "%zu allocations left", live.size());

  if (failures) return std::printf("%d failures\n", failures), 1;
  std::puts("ok");
}
