"""The library's host side against the oracle (CPU only, no GPU calls).

The host encoder of libmacko is a separate implementation (two parallel passes
and a closed-form padding count); it must agree with the oracle byte for byte.
"""
import ctypes
import os
import re
import subprocess
import sys

import numpy as np
import pytest

import oracle
import workloads as wl

M = pytest.importorskip("paper_2511_13061_amd")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def same_encoding(m, enc):
    v, d, r = m.host_buffers()
    assert v.dtype == np.uint16 and d.dtype == np.uint8 and r.dtype == np.uint32
    assert np.array_equal(v, enc.values)
    assert np.array_equal(d, enc.deltas)
    assert np.array_equal(r, enc.row_ptr)


def same_report(rep, enc, W, b_delta=4):
    assert (rep.rows, rep.cols) == W.shape
    assert rep.nnz == enc.nnz and rep.pad_nnz == enc.pad_nnz and rep.alloc_nnz == enc.alloc_nnz
    assert rep.padding_entries == enc.padding_entries
    assert rep.values_bytes == enc.values_bytes and rep.deltas_bytes == enc.deltas_bytes
    assert rep.rowptr_bytes == enc.rowptr_bytes and rep.total_bytes == enc.total_bytes
    assert rep.dense_bytes == enc.dense_bytes
    ent = np.diff(enc.row_ptr.astype(np.int64))
    assert rep.empty_rows == int((ent == 0).sum())
    assert rep.max_row_entries == (int(ent.max()) if ent.size else 0)
    assert rep.b_val == 16 and rep.b_delta == b_delta
    if W.size:
        d = enc.nnz / W.size
        cf = oracle.closed_forms
        assert rep.density == pytest.approx(d, abs=1e-15)
        assert rep.effd == pytest.approx(enc.effd, rel=1e-14)
        assert rep.effd_best == pytest.approx(cf.effd_macko_best(d, b_delta=b_delta), rel=1e-13)
        assert rep.effd_worst == pytest.approx(cf.effd_macko_worst(d, b_delta=b_delta), rel=1e-13)
        assert rep.effd_expected == pytest.approx(cf.effd_macko_expected(d, b_delta=b_delta), rel=1e-12)


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "macko.h")).read()
    declared = set(re.findall(r"MACKO_API\s+[\w\s\*]+?\b(macko_\w+)\s*\(", header))
    assert declared == set(M.binding.EXPORTED_SYMBOLS)
    lib = ctypes.CDLL(M.library_path())
    for name in declared:
        assert hasattr(lib, name), name


def test_header_is_plain_c_and_cpp(tmp_path):
    """The boundary is a C ABI: include/macko.h must compile as C99 and as C++11, pedantic, without warnings."""
    c = tmp_path / "use.c"
    c.write_text('#include "macko.h"\nint main(void) { macko_report_t r; macko_handle_t h = 0; (void)r; (void)h; return 0; }\n')
    inc = os.path.join(ROOT, "include")
    subprocess.check_call(["gcc", "-std=c99", "-pedantic", "-Wall", "-Werror", "-fsyntax-only", "-I", inc, str(c)])
    cpp = tmp_path / "use.cpp"
    cpp.write_text(c.read_text())
    subprocess.check_call(["g++", "-std=c++11", "-pedantic", "-Wall", "-Werror", "-fsyntax-only", "-I", inc, str(cpp)])


CASES = [
    ("c1", lambda: wl.config1().W),
    ("bern_sparse", lambda: wl.bernoulli(97, 1531, 0.03, 1.0, 5, 1)),
    ("bern_half", lambda: wl.bernoulli(130, 777, 0.5, 0.02, 5, 2)),
    ("dense", lambda: wl.bernoulli(33, 257, 1.0, 0.02, 5, 3)),
    ("c4", lambda: wl.config4(rows=96, cols=1200).W),
    ("c4b", lambda: wl.config4b(rows=40, cols=992).W),
    ("one_col", lambda: wl.bernoulli(50, 1, 0.5, 1.0, 5, 4)),
    ("wide_empty", lambda: np.zeros((9, 4000), dtype=np.uint16)),
]


@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_host_encoder_is_bit_exact_against_the_oracle(name, make):
    W = make()
    enc = oracle.encode(W)
    rep_holder = M.encode(W)
    same_encoding(rep_holder, enc)
    same_report(rep_holder.report, enc, W)
    assert np.array_equal(rep_holder.decode(), oracle.decode(enc))
    rep_holder.destroy()


@pytest.mark.parametrize("b_delta", [1, 2, 8])
@pytest.mark.parametrize("name,make", CASES, ids=[c[0] for c in CASES])
def test_host_encoder_other_code_widths_bit_exact_against_the_oracle(name, make, b_delta):
    """macko_encode_ex: 1-, 2- and 8-bit codes (Section 4.1 allows exactly 1, 2, 4, 8)."""
    W = make()
    enc = oracle.encode(W, b_delta)
    m = M.encode(W, b_delta)
    same_encoding(m, enc)
    same_report(m.report, enc, W, b_delta)
    assert np.array_equal(m.decode(), oracle.decode(enc))
    vb, db, rb = m.device_bytes()
    assert (vb, db, rb) == (enc.values_bytes, enc.deltas_bytes, enc.rowptr_bytes)
    m.destroy()


def test_worked_example_of_section_4_1_through_the_library():
    """The paper's row (values 1..4 at 1-based columns 2, 5, 12, 13) with 2-bit codes stores
    values [1, 2, 0, 3, 4] with deltas [2, 3, 4, 3, 1]."""
    one = np.float16([1, 2, 3, 4]).view(np.uint16)
    W = np.zeros((1, 16), dtype=np.uint16)
    W[0, [1, 4, 11, 12]] = one
    m = M.encode(W, 2)
    v, d, r = m.host_buffers()
    assert r.tolist() == [0, 5]
    assert v[:5].tolist() == [one[0], one[1], 0, one[2], one[3]]
    codes = [(int(d[k // 4]) >> (2 * (k % 4))) & 3 for k in range(5)]
    assert [c + 1 for c in codes] == [2, 3, 4, 3, 1]
    assert m.report.padding_entries == 1 and m.report.alloc_nnz == 64


def test_code_width_argument_is_validated():
    lib = M.load_library()
    W = np.ones((2, 2), dtype=np.uint16)
    h = ctypes.c_void_p(5)
    for bad in (0, 3, 5, 16, -4):
        assert lib.macko_encode_ex(W.ctypes.data, 2, 2, 2, bad, ctypes.byref(h), None) == -1
        assert h.value is None
        assert lib.macko_wrap_device_ex(2, 2, 4, bad, 256, 256, 256, ctypes.byref(h)) == -1
    m = M.encode(W, 2)
    assert lib.macko_spmm(m._h, 2, 16, 2, 16, 2, None) == -5    # not bound: refused before any device work


def test_special_bit_patterns_and_strided_input():
    W = np.zeros((6, 100), dtype=np.uint16)
    W[0, 3] = 0x8000      # -0 dropped
    W[0, 99] = 0x0001     # subnormal kept, long gap
    W[1, 0] = 0x7C00
    W[2, 50] = 0xFE00
    W[5, 17] = 0x8001
    big = np.zeros((6, 128), dtype=np.uint16)
    big[:, :100] = W
    m = M.encode(big[:, :100])          # ld = 128 > cols
    same_encoding(m, oracle.encode(W))
    canon = W.copy(); canon[0, 3] = 0
    assert np.array_equal(m.decode(), canon)


def test_empty_shapes_and_error_codes():
    lib = M.load_library()
    for shape in [(0, 5), (5, 0), (0, 0)]:
        m = M.encode(np.zeros(shape, dtype=np.uint16))
        assert m.report.pad_nnz == 0 and m.report.alloc_nnz == 0
        v, d, r = m.host_buffers()
        assert r.tolist() == [0] * (shape[0] + 1) and v.size == 0 and d.size == 0
    h = ctypes.c_void_p(123)
    W = np.ones((2, 2), dtype=np.uint16)
    assert lib.macko_encode(W.ctypes.data, 2, 2, 1, ctypes.byref(h), None) == -1   # ld < cols
    assert h.value is None
    assert lib.macko_encode(None, 2, 2, 2, ctypes.byref(h), None) == -1
    assert lib.macko_encode(W.ctypes.data, -1, 2, 2, ctypes.byref(h), None) == -1
    assert lib.macko_encode(W.ctypes.data, 2, 2, 2, None, None) == -1
    m = M.encode(W)
    # not bound: device operations are refused without touching the GPU
    assert lib.macko_spmv(m._h, 16, 16, None) == -5
    assert lib.macko_fetch_device(m._h, 16, 16, 16) == -5
    assert M.status_string(-5) == "handle has no device buffers"
    assert M.status_string(0) == "ok"
    with pytest.raises(M.MackoError):
        M.set_tuning("no_such_knob", 1)
    with pytest.raises(M.MackoError):
        M.set_tuning("spmv_block", 100)
    with pytest.raises(M.MackoError):
        M.set_tuning("spmm_kernel", 3)
    M.set_tuning("spmm_kernel", 2)
    assert M.get_tuning("spmm_kernel") == 2
    M.set_tuning("spmm_kernel", 0)
    M.set_tuning("spmv_block", 256)
    assert M.get_tuning("spmv_block") == 256
    M.set_tuning("spmv_block", 0)
    for bad in (4, 100, 1024):                            # a power of two from 8 to 512
        with pytest.raises(M.MackoError):
            M.set_tuning("spmv_step_align", bad)
    M.set_tuning("spmv_step_align", 128)
    assert M.get_tuning("spmv_step_align") == 128
    M.set_tuning("spmv_step_align", 0)
    lib.macko_destroy(None)


def test_padding_bound_reported_for_llama_like_rows():
    W = wl.half_row_matrix(64, 4096, 77)
    m = M.encode(W)
    r = m.report
    assert r.nnz == 64 * 2048 and r.density == 0.5
    assert r.effd_best <= r.effd <= r.effd_worst
    assert r.padding_entries <= 64 * 4096 * 0.5 / 16


def test_kernels_use_no_scratch_memory(tmp_path):
    """No kernel may spill registers or keep a run-time-indexed array in scratch memory: a scratch
    store per step costs more HBM bandwidth than the format saves (this happened to the 8-bit decode)."""
    import shutil
    import subprocess
    from paper_2511_13061_amd import build as B
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-fPIC",)]
    for src in (s for s in B.SOURCES if s.endswith(".hip")):
        out = tmp_path / (src + ".s")
        subprocess.check_call([hipcc, *flags, "-I", os.path.join(ROOT, "include"), "-I", B.CSRC, "-x", "hip",
                               "--cuda-device-only", "-S", "-o", str(out), os.path.join(B.CSRC, src)],
                              stderr=subprocess.DEVNULL)
        text = out.read_text()
        assert ".amdhsa_kernel" in text, src
        assert not re.search(r"^\s*scratch_(load|store)", text, re.M), f"{src}: scratch memory access"
        assert not re.search(r"\.private_segment_fixed_size:\s*[1-9]", text), f"{src}: private segment in use"
        # (scalar registers parked in lanes of a vector register are not memory: only vector spills count)
        assert not re.search(r"\.vgpr_spill_count:\s*[1-9]", text), f"{src}: vector register spills"


def test_launch_planner_covers_every_row_exactly_once(tmp_path):
    """Host logic of the launch planner: tests/planner_check.cpp replays, for 3000 random groups of
    matrices and both launch regimes, the row assignment the kernels derive from a plan."""
    import shutil
    import subprocess
    from paper_2511_13061_amd import build as B
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    exe = tmp_path / "planner_check"
    subprocess.check_call([hipcc, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", B.CSRC,
                           os.path.join(ROOT, "tests", "planner_check.cpp"), "-o", str(exe)],
                          stderr=subprocess.DEVNULL)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout + out.stderr


def test_native_calls_leave_a_forked_child_to_the_general_way():
    """A child of a process that has used the GPU may not: PyTorch's Python calls say so, its C++ calls do not.  So the binding's native
    functions return None there.  (This parent has not used it; decode_device is the one that needs no device tensor to get that far.)"""
    script = """
import os
from paper_2511_13061_amd import binding as B
B.load_library()
assert B._native is not None
pid = os.fork()
if pid == 0:
    try:
        ok = B._native.decode_device(None, 4, 4, 16) is None
    except BaseException:
        ok = False
    os._exit(0 if ok else 1)
raise SystemExit(os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]))
"""
    assert subprocess.run([sys.executable, "-c", script], cwd=ROOT, timeout=120).returncode == 0


@pytest.mark.parametrize("state", ["missing", "broken"])
def test_a_native_part_that_cannot_be_loaded_is_reported(tmp_path, state):
    """Not built, or built against another PyTorch: the calls go through ctypes, and a warning says so and how to change that."""
    import shutil
    from paper_2511_13061_amd import build as B
    pkg = tmp_path / "paper_2511_13061_amd"
    shutil.copytree(os.path.join(ROOT, "paper_2511_13061_amd"), pkg, ignore=shutil.ignore_patterns("_native*", "csrc", "__pycache__"))
    if state == "broken":
        (pkg / os.path.basename(B.BINDING)).write_bytes(b"not a library")
    script = """
import warnings
with warnings.catch_warnings(record=True) as said:
    warnings.simplefilter("always")
    import paper_2511_13061_amd as M
    M.load_library()
assert M.binding._native is None
said = [str(w.message) for w in said if w.category is RuntimeWarning]
assert len(said) == 1 and "native part" in said[0] and "paper_2511_13061_amd.build" in said[0], said
"""
    run = subprocess.run([sys.executable, "-c", script], cwd=tmp_path, timeout=120, capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-2000:]


def test_the_build_sees_a_stale_native_part(monkeypatch, tmp_path):
    """Older than its source, or than the installed PyTorch, or missing: build_library() makes it again."""
    from paper_2511_13061_amd import build as B
    copy = tmp_path / "_native.so"
    copy.write_bytes(b"")
    monkeypatch.setattr(B, "BINDING", str(copy))
    assert not B.binding_is_stale()
    os.utime(copy, (1, 1))
    for there in (copy, tmp_path / "none.so"):
        monkeypatch.setattr(B, "BINDING", str(there))
        assert B.binding_is_stale()
        made = []
        monkeypatch.setattr(B, "build_binding", lambda verbose=False: made.append(1))
        monkeypatch.setattr(B, "is_stale", lambda: False)
        B.build_library(force=False)
        assert made


def test_decode_device_without_a_device_in_use_goes_the_general_way(monkeypatch):
    """Before PyTorch has initialised the device (or in a forked child) the tensor is PyTorch's to make, with its own errors."""
    import torch
    m = M.encode(np.full((4, 64), 0x3C00, dtype=np.uint16))

    class Native:
        def decode_device(self, *args):
            raise AssertionError("native call")

    monkeypatch.setattr(M.binding, "_native", Native())
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)
    with pytest.raises(RuntimeError):                      # no GPU, or the handle has no device buffers
        m.decode_device()


def test_units_of_a_row_in_the_batch_kernel(tmp_path):
    """Every unit that holds an entry of the row is taken, and none behind it; a row without entries and one whose pointers
    decrease (trusted input, but no reason to walk 2^32 entries) take one."""
    import shutil
    import subprocess
    from paper_2511_13061_amd import build as B
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("needs g++ and the HIP headers")
    src, exe = tmp_path / "units.cpp", tmp_path / "units"
    src.write_text(r"""
#include <cstdio>
#include "macko_internal.h"
int main() {
  for (uint32_t per : {512u, 1024u, 1536u})
    for (uint64_t start : {0ull, 1ull, 7ull, 8ull, 513ull, 4294960000ull})
      for (uint64_t len = 0; len <= 3200; ++len) {
        if (start + len > 4294963200ull) continue;           // what the launchers take
        uint32_t want = 0;                                    // units from the row's first 8 entries that begin in front of its end
        for (uint64_t e = start & ~7ull; e < start + len; e += per) ++want;
        if (len == 0) want = 1;
        if (macko::panel_row_units((uint32_t)start, (uint32_t)(start + len), per) != want) return std::printf("%llu + %llu by %u\n", (unsigned long long)start, (unsigned long long)len, per), 1;
      }
  for (uint32_t per : {512u, 1024u, 1536u})
    if (macko::panel_row_units(10, 9, per) != 1 || macko::panel_row_units(4000, 8, per) != 1 || macko::panel_row_units(4294963200u, 0, per) != 1) return std::puts("decreasing"), 1;
  std::puts("ok");
}
""")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-w", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           "-I", B.CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout


def test_memory_of_the_encoders_handles(tmp_path):
    """Kept blocks, their bounds, devices, the wait before one is used again and what happens when memory runs out
    (tests/block_store_check.cpp)."""
    import shutil
    import subprocess
    from paper_2511_13061_amd import build as B
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("needs g++ and the HIP headers")
    exe = tmp_path / "block_store_check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-w", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", B.CSRC,
                           os.path.join(ROOT, "tests", "block_store_check.cpp"), os.path.join(B.CSRC, "macko_host.cpp"), "-o", str(exe), "-lpthread"])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout


def test_no_buffer_load_stands_in_a_loop_over_descriptors(tmp_path):
    """A buffer descriptor that the compiler takes as different from lane to lane puts each load through it in a loop of its own (its block
    ends in a branch back to itself while lanes are left).  The encoder's kernels hold none."""
    import re
    import subprocess
    from paper_2511_13061_amd import build as B
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    out = tmp_path / "encode.txt"
    subprocess.check_call([hipcc, *B.HIPCC_FLAGS, "-w", "-I", os.path.join(ROOT, "include"), "-I", B.CSRC, "-x", "hip", "--offload-device-only", "-S",
                           os.path.join(B.CSRC, "macko_encode_gpu.hip"), "-o", str(out)], stderr=subprocess.DEVNULL)
    loads = 0
    for label, block in re.findall(r"^(\.LBB\w+):(.*?)(?=^\.LBB|^\.Lfunc_end)", out.read_text(), re.S | re.M):
        loads += len(re.findall(r"\bbuffer_load_dword", block))
        assert not (re.search(r"\bbuffer_load_dword", block) and re.search(r"s_cbranch_execnz " + re.escape(label) + r"\b", block)), label
    assert loads >= 10


def test_a_simd_holds_8_wavefronts_of_the_resident_kernels(tmp_path):
    """A resident round of the product kernels, and of the batch kernel of two vectors, counts on 8 wavefronts to a SIMD: at most 64 vector
    registers and at most 80 scalar ones (800 to a SIMD, 16 more to a wavefront for the trap handler)."""
    import subprocess
    from paper_2511_13061_amd import build as B
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    seen = 0
    for src, kernels in (("macko_spmv.hip", r"spmv_(wave_row|chain)\w*"), ("macko_spmm.hip", r"spmm_wave_row_kernelILi2E\w*")):
        out = tmp_path / (src + ".txt")
        subprocess.check_call([hipcc, *B.HIPCC_FLAGS, "-w", "-I", os.path.join(ROOT, "include"), "-I", B.CSRC, "-x", "hip", "--offload-device-only", "-S",
                               os.path.join(B.CSRC, src), "-o", str(out)], stderr=subprocess.DEVNULL)
        for name, sgprs, vgprs in re.findall(r"\.name:\s+(_Z\S+)\n(?:(?!\.name:).)*?\.sgpr_count:\s+(\d+)(?:(?!\.name:).)*?\.vgpr_count:\s+(\d+)",
                                             out.read_text(), re.S):
            if re.search(kernels, name):
                assert int(sgprs) <= 80 and int(vgprs) <= 64, (name, sgprs, vgprs)
                seen += 1
    assert seen >= 20


def test_row_buffers_stay_inside_the_arrays(tmp_path):
    """The product kernels read a row through buffers whose ends come from its pointers.  Replayed here for a wavefront's rows, empty ones among
    them and (trusted input, but no reason to read outside the arrays) pointers that decrease: what a lane requests, in a step, behind
    the last row or for a row's tail, is behind the buffer's end or inside the arrays."""
    import shutil
    import subprocess
    from paper_2511_13061_amd import build as B
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("needs g++ and the HIP headers")
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(r"""
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <random>
#include <vector>
#include "macko_internal.h"
using namespace macko;
static int64_t pad_nnz;
static const char* what;
// one lane's load of `size` bytes at `at` of a buffer of `records` bytes that begins `base` bytes into an array of `bytes`
static void load(uint64_t base, uint32_t at, uint32_t records, int size, uint64_t bytes) {
  for (int k = 0; k < size; k += 4) {
    const uint64_t end = (uint64_t)at + k + std::min(size, 4);
    if (end > records) continue;                              // reads as zero
    if (base + end > bytes) std::printf("%s: %llu + %u of %llu\n", what, (unsigned long long)base, at, (unsigned long long)bytes), std::exit(1);
  }
}
struct Row { uint32_t start, end; };
template <bool TAILS>
static void wavefront(const std::vector<Row>& rows, uint32_t amask, int b_delta, int b_val, int ahead) {
  const int64_t alloc = (pad_nnz + alloc_granule(b_delta) - 1) / alloc_granule(b_delta) * alloc_granule(b_delta);
  const uint64_t vbytes = (uint64_t)alloc * (b_val / 8), cbytes = (uint64_t)alloc * b_delta / 8;
  auto lo = [&](int i) { return rows[i].start; };
  auto hi = [&](int i) { return rows[i].end; };
  const int nb = (int)rows.size();
  RowCursor cur{};
  seek_row<TAILS>(cur, nb, lo, hi, amask);
  for (int behind = 0; behind < ahead;) {                     // every step, and as many items behind the last row as a wavefront requests
    if (TAILS && cur.i >= nb) break;
    const uint32_t c0 = cur.start >> 3, n = buffer_entries(c0, cur.end), skipped = c0 - (cur.a0 >> 3);
    const uint32_t step = cur.i < nb ? (uint32_t)cur.step : (uint32_t)behind++;
    for (uint32_t lane = 0; lane < 64; ++lane) {
      load((uint64_t)b_val * c0, (uint32_t)b_val * (64 * step + lane - skipped), buffer_value_bytes(n, b_val), b_val, vbytes);
      load((uint64_t)b_delta * c0, (uint32_t)b_delta * (64 * step + lane - skipped), buffer_code_bytes(n, b_delta), b_delta, cbytes);
    }
    if (cur.i < nb && ++cur.step == cur.nsteps) {
      ++cur.i;
      seek_row<TAILS>(cur, nb, lo, hi, amask);
    }
  }
  if (!TAILS) return;
  const uint32_t n = buffer_entries(tail_buffer().c0, tail_buffer().end);
  for (const Row& r : rows) {                                 // behind the last row: every lane its row's last chunk, or nothing
    const uint32_t chunk = (r.end - 1u) >> 3;
    const bool has = r.end > r.start;
    load(0, has ? b_val * chunk : 0u - b_val, buffer_value_bytes(n, b_val), b_val, vbytes);
    load(0, has ? b_delta * chunk : 0u - b_delta, buffer_code_bytes(n, b_delta), b_delta, cbytes);
  }
}
int main() {
  std::mt19937_64 rng(7);
  for (int trial = 0; trial < 4000; ++trial) {
    std::vector<uint32_t> rp(2 + rng() % 64);
    const bool far = trial % 3 == 0;                          // entries from 2^32 - 20000 on, as far as the launchers go
    const uint32_t first = far ? 4294947300u : 0u;
    pad_nnz = far ? 4294963200ll : 16000 - (int64_t)(rng() % 40);
    const uint32_t room = (uint32_t)(pad_nnz - first);
    for (uint32_t& p : rp) p = first + (uint32_t)(rng() % (room + 1));
    if (trial % 2) std::sort(rp.begin(), rp.end());
    for (size_t i = 1; i < rp.size(); ++i)
      if (rng() % 3 == 0) rp[i] = rp[i - 1];
    if (rng() % 2) rp.back() = first + room;
    if (rng() % 4 == 0) rp.back() = first + (uint32_t)(rng() % 200);
    std::vector<Row> rows;
    for (size_t i = 0; i + 1 < rp.size(); ++i) rows.push_back({rp[i], rp[i + 1]});
    for (uint32_t amask : {7u, 31u, 255u, 511u})
      for (int b_delta : {1, 2, 4, 8})
        for (int b_val : {16, 8}) {
          what = b_val == 8 ? "8-bit values" : "16-bit values";
          if (b_val == 8 && b_delta != 4) continue;
          wavefront<false>(rows, amask, b_delta, b_val, 4);
          if (b_val == 8) wavefront<true>(rows, amask, b_delta, b_val, 4);
        }
  }
  std::puts("ok");
}
""")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-w", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           "-I", B.CSRC, str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout


def test_host_code_under_address_and_undefined_behaviour_sanitizers(tmp_path):
    """The library's host translation unit (encoders for every code and value width, decoders, storage
    report, argument checks) linked with stand-ins for the GPU launchers and run under ASan + UBSan on
    random, ragged, strided, empty and overflowing inputs (tests/host_sanitizer_check.cpp)."""
    import shutil
    import subprocess
    from paper_2511_13061_amd import build as B
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/lib/libamdhip64.so"):
        pytest.skip("needs g++ and the HIP runtime library to link against")
    exe = tmp_path / "host_sanitizer_check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=undefined", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), "-I", B.CSRC,
                           os.path.join(ROOT, "tests", "host_sanitizer_check.cpp"),
                           os.path.join(ROOT, "tests", "host_sanitizer_stubs.cpp"),
                           os.path.join(B.CSRC, "macko_host.cpp"), "-o", str(exe),
                           "-L/opt/rocm/lib", "-lamdhip64", "-lpthread", "-Wl,-rpath,/opt/rocm/lib"],
                          stderr=subprocess.DEVNULL)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0",
               UBSAN_OPTIONS="print_stacktrace=1")
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=600, env=env)
    assert out.returncode == 0 and out.stdout.strip().endswith("ok"), out.stdout[-2000:] + out.stderr[-4000:]


# ------------------------------------------------------------------ 8-bit values (host side)

@pytest.mark.parametrize("shape,density", [((64, 512), 0.5), ((33, 1031), 0.07), ((5, 40), 1.0), ((300, 2000), 0.3)])
def test_host_encoder_for_8_bit_values_is_bit_exact_against_the_oracle(shape, density):
    rng = np.random.default_rng(shape[0])
    W = rng.integers(0, 256, size=shape, dtype=np.uint8)
    W[rng.random(shape) >= density] = 0
    W[0, :] = 0
    W[1, 0] = 0x80                                         # -0 is a zero
    W[2, shape[1] - 1] = 0xFF                              # a NaN pattern is a value like any other
    enc = oracle.encode8(W, 4)
    m = M.encode_fp8(W)
    v, d, r = m.host_buffers()
    assert v.dtype == np.uint8
    assert np.array_equal(v, enc.values) and np.array_equal(d, enc.deltas) and np.array_equal(r, enc.row_ptr)
    rep = m.get_report()
    assert (rep.b_val, rep.b_delta, rep.nnz, rep.pad_nnz, rep.alloc_nnz) == (8, 4, enc.nnz, enc.pad_nnz, enc.alloc_nnz)
    assert (rep.values_bytes, rep.deltas_bytes, rep.total_bytes, rep.dense_bytes) == \
        (enc.values_bytes, enc.deltas_bytes, enc.total_bytes, enc.dense_bytes)
    assert rep.effd == pytest.approx(enc.effd, rel=1e-12)
    dd = enc.nnz / (shape[0] * shape[1])
    assert rep.effd_best == pytest.approx(oracle.closed_forms.effd_macko_best(dd, 8, 4), rel=1e-12)
    assert rep.effd_worst == pytest.approx(oracle.closed_forms.effd_macko_worst(dd, 8, 4), rel=1e-12)
    assert rep.effd_expected == pytest.approx(oracle.closed_forms.effd_macko_expected(dd, 8, 4), rel=1e-12)
    assert np.array_equal(m.decode(), oracle.decode8(enc))
    assert m.device_bytes() == (enc.alloc_nnz, enc.alloc_nnz // 2, 4 * (shape[0] + 1))
    # strided input
    wide = np.zeros((shape[0], shape[1] + 7), dtype=np.uint8)
    wide[:, :shape[1]] = W
    v2, d2, r2 = M.encode_fp8(wide[:, :shape[1]]).host_buffers()
    assert np.array_equal(v2, enc.values) and np.array_equal(d2, enc.deltas) and np.array_equal(r2, enc.row_ptr)


def test_8_bit_handles_refuse_what_they_do_not_support():
    lib = M.load_library()
    W = np.full((4, 64), 0x38, dtype=np.uint8)
    m8 = M.encode_fp8(W)
    m16 = M.encode(np.full((4, 64), 0x3C00, dtype=np.uint16))
    buf16 = np.zeros((4, 64), dtype=np.uint16)
    buf8 = np.zeros((4, 64), dtype=np.uint8)
    assert lib.macko_decode(m8._h, buf16.ctypes.data, 64) == -3            # MACKO_E_UNSUPPORTED
    assert lib.macko_decode_fp8(m16._h, buf8.ctypes.data, 64) == -3
    p = ctypes.c_void_p()
    assert lib.macko_host_values_fp8(m16._h, ctypes.byref(p)) == -3
    assert lib.macko_host_buffers(m8._h, ctypes.byref(p), None, None) == -3
    assert lib.macko_encode_fp8(None, 4, 64, 64, ctypes.byref(p), None) == -1
    assert lib.macko_encode_fp8(W.ctypes.data, 4, 64, 63, ctypes.byref(p), None) == -1
    empty = M.encode_fp8(np.zeros((0, 16), dtype=np.uint8))
    assert empty.get_report().pad_nnz == 0


def test_storage_by_code_width_equals_the_oracles_encodings():
    """Bytes per code width counted without encoding (Section 4.2 / Appendix C) against the oracle's
    encodings at each width, and the choice: 1 bit for dense rows, 2 bits around 40 %, 4 bits at
    70 %, 8 bits at 97 % sparsity (the ranges of Appendix C)."""
    cases = {
        "dense": (wl.bernoulli(40, 1031, 1.0, 0.02, 91, 1), 1),
        "sparsity40": (wl.bernoulli(64, 3000, 0.6, 0.02, 91, 2), 2),
        "sparsity70": (wl.bernoulli(64, 3000, 0.3, 0.02, 91, 3), 4),
        "sparsity97": (wl.bernoulli(300, 9000, 0.03, 1.0, 91, 4), 8),
        "worked_example": (None, None),
    }
    for name, (W, want_best) in cases.items():
        if W is None:
            W = np.zeros((3, 12), dtype=np.uint16)
            W[0, [0, 4, 11]] = 0x3C00
            W[2, 7] = 0x4000
        table, best = M.storage_by_code_width(W)
        for b in (1, 2, 4, 8):
            assert table[b] == oracle.encode(W, b).total_bytes, (name, b)
        assert table[best] == min(table.values())
        if want_best is not None:
            assert best == want_best, (name, table)
    # empty matrix: only the row pointers (and a tie, which goes to 4 bits)
    table, best = M.storage_by_code_width(np.zeros((5, 0), dtype=np.uint16))
    assert set(table.values()) == {4 * 6} and best == 4
    lib = M.load_library()
    out = (ctypes.c_int64 * 4)()
    assert lib.macko_storage_by_code_width(None, 2, 2, 2, out, None) == -1
    assert lib.macko_storage_by_code_width(W.ctypes.data, 3, 12, 4, out, None) == -1       # ld < cols
