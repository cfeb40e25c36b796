"""GPU parity: the HIP path (through the C ABI) against the CPU oracle.

Encodings must match the oracle byte for byte.  Every y_i must satisfy
|y_gpu - y_fp64| <= 1e-2 * sum_j |w_ij x_j| + 1e-3, with y_fp64 the dense
product by definition (Appendix A of the paper) computed by the oracle.
"""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
M = pytest.importorskip("paper_2511_13061_amd")

REL_TOL = 1e-2
ABS_TOL = 1e-3


@pytest.fixture(scope="module", autouse=True)
def _need_gpu_and_library():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    M.load_library()          # raises if libmacko.so is missing: no fallback
    yield
    for knob in ("spmv_kernel", "spmv_lanes", "spmv_block", "spmv_rows_per_wg", "spmv_ring", "spmv_resident",
                 "spmv_wgs_per_cu", "spmv_resident_steps", "spmv_steps_per_wave", "spmv_step_align", "gemv_block", "gemv_rows_per_wg", "gemv_ring", "gemv_resident",
                 "gemv_wgs_per_cu", "spmm_kernel"):
        M.set_tuning(knob, 0)


def to_dev(a_u16):
    return torch.from_numpy(np.ascontiguousarray(a_u16).view(np.float16)).cuda()


def check_y(y_dev, W, x, what=""):
    y64, s64 = oracle.dense_matvec(W, x)
    y = y_dev.float().cpu().numpy().astype(np.float64)
    assert y.shape == y64.shape
    assert np.isfinite(y).all(), what
    err = np.abs(y - y64)
    bound = REL_TOL * s64 + ABS_TOL
    worst = int(np.argmax(err - bound))
    assert (err <= bound).all(), (
        f"{what}: row {worst}: |{y[worst]} - {y64[worst]}| = {err[worst]} > {bound[worst]}")
    # the tolerance is loose; fp32 accumulation should in fact sit well inside it
    return float(np.max(err / bound))


def spmv_case(W, x, b_delta=4, **knobs):
    for k, v in knobs.items():
        M.set_tuning(k, v)
    try:
        m = M.encode(W, b_delta).to_device()
        y = m.spmv(to_dev(x))
        torch.cuda.synchronize()
    finally:
        for k in knobs:
            M.set_tuning(k, 0)
    return y


def assert_same_encoding(arrays, enc):
    v, d, r = arrays
    assert np.array_equal(r, enc.row_ptr)
    assert np.array_equal(v, enc.values)
    assert np.array_equal(d, enc.deltas)


# ------------------------------------------------------------------ small and ragged

SMALL = {
    "c1_512": lambda: (wl.config1().W, wl.config1().x),
    "ragged_777": lambda: (wl.bernoulli(301, 777, 0.5, 0.02, 9, 1), wl.x_vector(777, 9, 1)),
    "long_rows_5000": lambda: (wl.bernoulli(70, 5000, 0.6, 0.02, 9, 2), wl.x_vector(5000, 9, 2)),
    "very_sparse": lambda: (wl.bernoulli(200, 3000, 0.02, 1.0, 9, 3), wl.x_vector(3000, 9, 3)),
    "dense": lambda: (wl.bernoulli(100, 1031, 1.0, 0.02, 9, 4), wl.x_vector(1031, 9, 4)),
    "c4_small": lambda: (wl.config4(rows=256, cols=2048).W, wl.config4(rows=256, cols=2048).x),
    "c4b_small": lambda: (wl.config4b(rows=128, cols=2048).W, wl.config4b(rows=128, cols=2048).x),
    "one_row": lambda: (wl.bernoulli(1, 9000, 0.5, 0.02, 9, 5), wl.x_vector(9000, 9, 5)),
    "one_col": lambda: (wl.bernoulli(300, 1, 0.5, 1.0, 9, 6), wl.x_vector(1, 9, 6)),
}

VARIANTS = {
    "auto": {},
    "sub16": {"spmv_kernel": 1, "spmv_lanes": 16},
    "sub32": {"spmv_kernel": 1, "spmv_lanes": 32},
    "sub64": {"spmv_kernel": 1, "spmv_lanes": 64},
    "wave_row": {"spmv_kernel": 2},
    "wave_row_b256_r5": {"spmv_kernel": 2, "spmv_block": 256, "spmv_rows_per_wg": 5},
    "wave_row_b1024_r700": {"spmv_kernel": 2, "spmv_block": 1024, "spmv_rows_per_wg": 700},
    "wave_row_b64_r200": {"spmv_kernel": 2, "spmv_block": 64, "spmv_rows_per_wg": 200},
    "wave_row_b256_r37": {"spmv_kernel": 2, "spmv_block": 256, "spmv_rows_per_wg": 37},
    "wave_row_b128_r63": {"spmv_kernel": 2, "spmv_block": 128, "spmv_rows_per_wg": 63},
    # every step of a row on a multiple of 64 / 256 / 512 stored entries (lanes before the row cleared)
    "wave_row_align64": {"spmv_kernel": 2, "spmv_step_align": 64},
    "wave_row_align256_b256_r37": {"spmv_kernel": 2, "spmv_step_align": 256, "spmv_block": 256, "spmv_rows_per_wg": 37},
    "wave_row_align512": {"spmv_kernel": 2, "spmv_step_align": 512},
}


@pytest.mark.parametrize("variant", list(VARIANTS))
@pytest.mark.parametrize("case", list(SMALL))
def test_spmv_small_cases_all_kernels(case, variant):
    W, x = SMALL[case]()
    y = spmv_case(W, x, **VARIANTS[variant])
    check_y(y, W, x, f"{case}/{variant}")


@pytest.mark.parametrize("bits", [16, 8])
@pytest.mark.parametrize("cols", [2, 6, 258, 514, 1022, 1030, 2050, 2148, 3022, 4098])
def test_spmv_x_of_an_even_length_ends_where_it_ends(cols, bits):
    """x is loaded in pairs of elements up to its end, whatever remains of a chunk of 8: NaN in front of x and behind it stays out of y.
    The rows hold from nothing to all columns, so that their first steps begin on every multiple that a row length is given."""
    rng = np.random.default_rng(cols)
    rows = 300
    W = (rng.standard_normal((rows, cols)) * (rng.random((rows, cols)) < np.linspace(0, 1, rows)[:, None])).astype(np.float16)
    W[5, -1] = 1.0
    W[7, -2:] = 2.0
    x = rng.standard_normal(cols).astype(np.float16)
    big = torch.full((cols + 16,), float("nan"), dtype=torch.float16, device="cuda")
    big[8:8 + cols] = torch.from_numpy(x).cuda()
    for keep in (1.0, 0.4, 0.1):
        Wk = W * (rng.random((rows, cols)) < keep)
        if bits == 8:
            W8 = wl.fp8_values_of(Wk.astype(np.float16).view(np.uint16))
            check_y8(M.encode_fp8(W8).to_device().spmv(big[8:8 + cols]), W8, x.view(np.uint16), f"{cols} {keep}")
        else:
            Wk = Wk.astype(np.float16).view(np.uint16)
            check_y(M.encode(Wk).to_device().spmv(big[8:8 + cols]), Wk, x.view(np.uint16), f"{cols} {keep}")


@pytest.mark.parametrize("n", [1, 2, 5, 11])
@pytest.mark.parametrize("b_delta,rows,entries", [(4, 300, 1), (4, 1023, 30), (2, 1500, 111), (4, 1500, 113), (8, 8300, 100), (8, 8300, 143), (1, 8300, 144),
                                                  (4, 12400, 239), (4, 12400, 241), (8, 16500, 20)])
def test_short_rows_on_either_side_of_the_choice_of_kernel(b_delta, rows, entries, n):
    """Short rows go to one launch of wavefronts per row or to sub-wave launches, by rows per compute unit, their mean length and whether
    the call holds several products.  Rows from empty to three times the mean."""
    gen = torch.Generator(device="cuda").manual_seed(rows + n)
    cols = 3 * entries + 7 if b_delta < 8 else 40 * entries
    for many in (False, True) if n > 1 else (False,):
        mats, xs, want = [], [], []
        for _ in range(n):
            share = torch.rand((rows, 1), generator=gen, device="cuda") * 2 * entries / cols
            share[::7] = 0
            W = torch.randn((rows, cols), generator=gen, device="cuda").half()
            W *= torch.rand((rows, cols), generator=gen, device="cuda") < share
            W[3, :] = 1.0
            x = torch.randn(cols, generator=gen, device="cuda").half()
            mats.append(M.encode_device(W, b_delta=b_delta))
            xs.append(x)
            want.append((W.double() @ x.double(), W.double().abs() @ x.double().abs()))
            del W
        ys = [torch.full((rows,), float("nan"), dtype=torch.float16, device="cuda") for _ in range(n)]
        if many:
            M.SpmvMany(mats, xs, ys).launch()
        elif n <= 8:
            M.SpmvGroup(mats, xs, ys).launch()
        else:
            continue
        for y, (y64, s64) in zip(ys, want):
            assert bool(((y.double() - y64).abs() <= 1e-3 * s64 + 1e-3).all())
        if n == 1:
            assert torch.equal(mats[0].spmv(xs[0]), ys[0])


@pytest.mark.parametrize("kind", ["all alike", "two kinds", "batch"])
@pytest.mark.parametrize("rows,entries", [(2000, 60), (300, 30), (9000, 90), (20000, 150)])
def test_short_rows_give_equal_bits_in_every_launch_of_a_call(rows, entries, kind):
    """One matrix and one vector, 33 times in a call: a launch of 32 and one of 1, or (with a second kind of matrix among them) launches of 8
    and one of 1 on side streams; nine equal vectors of a batch: products in groups of 8 and 1.  All results are the same bit for bit."""
    gen = torch.Generator(device="cuda").manual_seed(rows)
    cols = 8 * entries
    W = torch.randn((rows, cols), generator=gen, device="cuda").half() * (torch.rand((rows, cols), generator=gen, device="cuda") < 0.125)
    x = torch.randn(cols, generator=gen, device="cuda").half()
    m = M.encode_device(W)
    want, scale = W.double() @ x.double(), W.double().abs() @ x.double().abs()
    if kind == "batch":
        M.set_tuning("spmm_kernel", 1)
        try:
            ys = list(m.spmm(x.expand(9, cols).contiguous()))
        finally:
            M.set_tuning("spmm_kernel", 0)
    else:
        other = M.encode_device(W, b_delta=8)
        mats = [other if kind == "two kinds" and i % 5 == 4 else m for i in range(33)]
        ys = [torch.full((rows,), float("nan"), dtype=torch.float16, device="cuda") for _ in mats]
        M.SpmvMany(mats, [x] * 33, ys).launch()
        ys = [y for y, o in zip(ys, mats) if o is m]
    for i, y in enumerate(ys):
        assert torch.equal(y, ys[0]), i
    assert bool(((ys[0].double() - want).abs() <= 1e-3 * scale + 1e-3).all())


@pytest.mark.parametrize("batch", [2, 3, 5, 8, 13, 64])
@pytest.mark.parametrize("rows,cols", [(2047, 512), (2048, 512), (2300, 520), (2300, 523), (3000, 8)])
def test_spmm_short_rows_with_8_bit_codes(rows, cols, batch):
    """Either side of the line from which short rows with 8-bit codes share passes over the matrix; results in a wider buffer."""
    gen = torch.Generator(device="cuda").manual_seed(rows + batch)
    W = torch.randn((rows, cols), generator=gen, device="cuda").half() * (torch.rand((rows, cols), generator=gen, device="cuda") < 0.08)
    W[5] = 0
    X = torch.randn((batch, cols), generator=gen, device="cuda").half()
    Y = torch.full((batch, rows + 3), 7.0, dtype=torch.float16, device="cuda")
    M.encode_device(W, b_delta=8).spmm(X, Y[:, :rows])
    want, scale = X.double() @ W.double().t().contiguous(), X.double().abs() @ W.double().abs().t().contiguous()
    assert bool(((Y[:, :rows].double() - want).abs() <= 1e-3 * scale + 1e-3).all())
    assert bool((Y[:, rows:] == 7.0).all())


def test_spmv_empty_rows_mixed_with_full_rows_and_row_boundaries_inside_chunks():
    rng = np.random.default_rng(5)
    C = 4096
    W = wl.bernoulli(400, C, 0.5, 0.02, 11, 1)
    W[rng.choice(400, 120, replace=False)] = 0           # empty rows, some adjacent
    W[10:30] = 0
    W[395:] = 0                                          # trailing empty rows
    # rows with 1..9 entries so that several rows share one 8-entry chunk
    for r in range(40, 60):
        W[r] = 0
        cols = rng.choice(C, size=(r - 39) % 10 + 1, replace=False)
        W[r, cols] = wl.normal_f16(cols.size, 1.0, 11, r, nonzero=True)
    x = wl.x_vector(C, 11, 1)
    for variant in ("auto", "wave_row", "sub16", "wave_row_b64_r200", "wave_row_b256_r37", "wave_row_b128_r63",
                    "wave_row_align64", "wave_row_align256_b256_r37", "wave_row_align512"):
        y = spmv_case(W, x, **VARIANTS[variant])
        check_y(y, W, x, variant)
        assert (y[10:30] == 0).all() and (y[395:] == 0).all()


@pytest.mark.parametrize("b_delta", [1, 4, 8])
def test_aligned_steps_with_rows_starting_at_chosen_offsets(b_delta):
    """Rows whose first k columns are non-zero (no padding), so that every row starts at a known
    entry: multiples of the step alignment, one entry after, eight after, one before; rows of one
    entry, empty rows and rows of exactly one and two steps between them.  Each alignment of the
    wave-per-row kernel, and the choice it makes by itself."""
    C = 4096
    lengths = [512, 256, 1, 7, 8, 9, 247, 248, 1, 255, 256, 257, 0, 0, 3, 1024, 511, 513, 2048, 64, 63, 65,
               4096, 1, 4095, 0, 1536, 8, 504, 16, 1000, 3000, 2, 510, 4096, 4096, 5, 251]
    W = np.zeros((len(lengths), C), dtype=np.uint16)
    for r, n in enumerate(lengths):
        if n:
            W[r, :n] = wl.normal_f16(n, 1.0, 77, r, nonzero=True)
    x = wl.x_vector(C, 77, 1)
    enc = oracle.encode(W, b_delta)
    assert enc.pad_nnz == sum(lengths) and list(np.diff(enc.row_ptr.astype(np.int64))) == lengths
    for knobs in ({}, {"spmv_kernel": 2}, {"spmv_kernel": 2, "spmv_step_align": 64},
                  {"spmv_kernel": 2, "spmv_step_align": 256, "spmv_block": 128, "spmv_rows_per_wg": 5},
                  {"spmv_kernel": 2, "spmv_step_align": 512, "spmv_block": 64, "spmv_rows_per_wg": 38},
                  {"spmv_kernel": 2, "spmv_step_align": 512, "spmv_ring": 4},
                  {"spmv_kernel": 2, "spmv_step_align": 16, "spmv_ring": 3}):
        y = spmv_case(W, x, b_delta, **knobs)
        check_y(y, W, x, f"b{b_delta}/{knobs}")
        assert y[12] == 0 and y[13] == 0 and y[25] == 0


def test_random_matrices_with_random_launch_knobs():
    """Forty seeded draws of shape, density, code width and launch knobs (kernel, block, rows per
    workgroup, resident round, ring depth, step alignment): the planner has to turn every
    combination into a launch that computes each row exactly once."""
    rng = np.random.default_rng(20251113)
    for case in range(40):
        rows = int(rng.integers(1, 400))
        cols = int(rng.choice([1, 7, 64, 500, 1031, 2048, 4096, 6000, 9000]))
        dens = float(rng.choice([0.02, 0.1, 0.3, 0.5, 0.8, 1.0]))
        b_delta = int(rng.choice([1, 2, 4, 8]))
        W = wl.bernoulli(rows, cols, dens, 0.05, 700 + case, 1)
        if rows > 5:
            W[rng.choice(rows, rows // 5, replace=False)] = 0     # empty rows
        x = wl.x_vector(cols, 700 + case, 2)
        block = int(rng.choice([0, 64, 128, 192, 256, 512, 704, 1024]))
        knobs = {"spmv_kernel": int(rng.choice([0, 2, 2, 2])), "spmv_block": block,
                 "spmv_step_align": int(rng.choice([0, 8, 16, 32, 64, 128, 256, 512])),
                 "spmv_ring": int(rng.choice([0, 2, 3, 4])), "spmv_resident": int(rng.choice([0, 1, 2]))}
        if rng.random() < 0.5:
            knobs["spmv_rows_per_wg"] = int(rng.integers(1, 64 * max(block, 64) // 64 + 1))
        else:
            knobs["spmv_wgs_per_cu"] = int(rng.choice([0, 1, 2, 3, 4]))
            knobs["spmv_steps_per_wave"] = int(rng.choice([0, 1, 3, 8, 40]))
        y = spmv_case(W, x, b_delta, **knobs)
        check_y(y, W, x, f"case {case}: {rows}x{cols} d={dens} b={b_delta} {knobs}")


RESIDENT_VARIANTS = {
    "auto": {},
    "never": {"spmv_resident": 1},
    "k1": {"spmv_resident": 2, "spmv_wgs_per_cu": 1},
    "k2_ring4": {"spmv_resident": 2, "spmv_wgs_per_cu": 2, "spmv_ring": 4},
    "k3_b320": {"spmv_resident": 2, "spmv_wgs_per_cu": 3, "spmv_block": 320},
    "k4": {"spmv_resident": 2, "spmv_wgs_per_cu": 4},
    "k1_b1024": {"spmv_resident": 2, "spmv_wgs_per_cu": 1, "spmv_block": 1024},
    "k2_b704": {"spmv_resident": 2, "spmv_wgs_per_cu": 2, "spmv_block": 704},
    "many_wgs_r40_b256": {"spmv_resident": 1, "spmv_rows_per_wg": 40, "spmv_block": 256},
    "many_wgs_r63_b64": {"spmv_resident": 1, "spmv_rows_per_wg": 63, "spmv_block": 64},
    "many_wgs_steps3": {"spmv_resident_steps": 1, "spmv_steps_per_wave": 3},
    "many_wgs_steps40": {"spmv_resident_steps": 1, "spmv_steps_per_wave": 40, "spmv_block": 192},
}


@pytest.mark.parametrize("variant", list(RESIDENT_VARIANTS))
def test_spmv_resident_round_launch_shapes(variant):
    """One resident round of workgroups (a multiple of the compute-unit count) with row counts
    that do not divide evenly: every row must still be computed exactly once, single and grouped."""
    W = wl.bernoulli(2311, 1536, 0.5, 0.02, 41, 1)
    W[100:140] = 0                                        # a run of empty rows inside one workgroup's share
    x = wl.x_vector(1536, 41, 1)
    y = spmv_case(W, x, spmv_kernel=2, **RESIDENT_VARIANTS[variant])
    check_y(y, W, x, variant)
    # grouped: three matrices of different heights and widths share the round
    specs = [(1500, 2048, 0.5), (1031, 1024, 0.6), (777, 4096, 0.4)]
    Ws = [wl.bernoulli(r, c, d, 0.02, 42, i) for i, (r, c, d) in enumerate(specs)]
    xs = [wl.x_vector(c, 42, i) for i, (_, c, _) in enumerate(specs)]
    for k, v in dict(spmv_kernel=2, **RESIDENT_VARIANTS[variant]).items():
        M.set_tuning(k, v)
    try:
        ms = [M.encode(Wi).to_device() for Wi in Ws]
        ys = M.spmv_group(ms, [to_dev(xi) for xi in xs])
        torch.cuda.synchronize()
    finally:
        for k in dict(spmv_kernel=2, **RESIDENT_VARIANTS[variant]):
            M.set_tuning(k, 0)
    for i, (Wi, xi, yi) in enumerate(zip(Ws, xs, ys)):
        check_y(yi, Wi, xi, f"{variant} group member {i}")


def test_spmv_under_graph_capture_and_on_two_streams():
    """The products only enqueue kernels, so they can be captured into a HIP graph and replayed,
    and one handle can be used from two streams at once."""
    W = wl.half_row_matrix(1024, 4096, 77)
    x1, x2 = wl.x_vector(4096, 43, 1), wl.x_vector(4096, 43, 2)
    m = M.encode(W).to_device()
    xd = to_dev(x1)
    y = torch.empty(1024, dtype=torch.float16, device="cuda")
    eager1 = m.spmv(to_dev(x1)).clone()
    eager2 = m.spmv(to_dev(x2)).clone()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        m.spmv(xd, y, stream=side)                       # warm-up on the capture stream
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            m.spmv(xd, y, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    for rep, (xv, want) in enumerate([(x1, eager1), (x2, eager2), (x1, eager1), (x2, eager2)]):
        xd.copy_(to_dev(xv))
        y.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want), f"replay {rep}"
    # two streams, same handle, different vectors
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    xa, xb = to_dev(x1), to_dev(x2)
    ya = torch.empty(1024, dtype=torch.float16, device="cuda")
    yb = torch.empty(1024, dtype=torch.float16, device="cuda")
    torch.cuda.synchronize()
    for _ in range(20):
        m.spmv(xa, ya, stream=s1)
        m.spmv(xb, yb, stream=s2)
    torch.cuda.synchronize()
    assert torch.equal(ya, eager1) and torch.equal(yb, eager2)


def test_spmv_all_zero_matrix_and_zero_sized():
    x = wl.x_vector(640, 3, 3)
    y = spmv_case(np.zeros((77, 640), dtype=np.uint16), x, spmv_kernel=2)
    assert (y == 0).all()
    y = spmv_case(np.zeros((77, 640), dtype=np.uint16), x)
    assert (y == 0).all()
    m = M.encode(np.zeros((0, 640), dtype=np.uint16)).to_device()
    m.spmv(to_dev(x), torch.empty(0, dtype=torch.float16, device="cuda"))
    torch.cuda.synchronize()


def test_subnormal_weights_are_not_flushed():
    # every weight is an fp16 subnormal; x = 2048 makes the exact row sums O(1)
    rng = np.random.default_rng(1)
    R, C = 64, 2048
    W = np.zeros((R, C), dtype=np.uint16)
    mask = rng.random((R, C)) < 0.5
    W[mask] = rng.integers(1, 0x400, size=int(mask.sum()), dtype=np.uint16)   # positive subnormals
    x = np.full(C, np.float16(2048.0)).view(np.uint16)
    for variant in ("wave_row", "sub64"):
        y = spmv_case(W, x, **VARIANTS[variant])
        check_y(y, W, x, variant)
        y64, _ = oracle.dense_matvec(W, x)
        assert y64.min() > 10.0                                   # flushing would give exactly 0
        assert np.allclose(y.float().cpu().numpy(), y64, rtol=2e-3)


def test_unaligned_x_and_y_pointers():
    W = wl.bernoulli(150, 1000, 0.5, 0.02, 4, 4)
    x = wl.x_vector(1000, 4, 4)
    xbuf = torch.zeros(1001, dtype=torch.float16, device="cuda")
    xbuf[1:] = to_dev(x)
    ybuf = torch.zeros(151, dtype=torch.float16, device="cuda")
    m = M.encode(W).to_device()
    for kernel in (1, 2):
        M.set_tuning("spmv_kernel", kernel)
        m.spmv(xbuf[1:], ybuf[1:])
        torch.cuda.synchronize()
        check_y(ybuf[1:], W, x, f"kernel {kernel}")
    M.set_tuning("spmv_kernel", 0)


def test_x_larger_than_64k_lds_and_x_larger_than_lds():
    # 40000 columns need ~82 KB of LDS (above the 64 KB default limit)
    W = wl.bernoulli(40, 40000, 0.3, 0.02, 6, 1)
    x = wl.x_vector(40000, 6, 1)
    check_y(spmv_case(W, x, spmv_kernel=2), W, x, "80KB LDS wave_row")
    check_y(spmv_case(W, x, spmv_kernel=1, spmv_lanes=64), W, x, "80KB LDS sub64")
    # 100000 columns do not fit in LDS at all: x is gathered from global memory
    W = wl.bernoulli(24, 100000, 0.2, 0.02, 6, 2)
    x = wl.x_vector(100000, 6, 2)
    check_y(spmv_case(W, x), W, x, "global x")


def test_wrap_device_reuses_an_existing_encoding():
    W = wl.bernoulli(300, 2048, 0.5, 0.02, 8, 8)
    x = wl.x_vector(2048, 8, 8)
    m = M.encode(W).to_device()
    v, d, r = [b.clone() for b in m.device_buffers()]
    w = M.wrap_device(300, 2048, m.report.pad_nnz, v, d, r)
    y = w.spmv(to_dev(x))
    torch.cuda.synchronize()
    check_y(y, W, x, "wrapped")
    assert torch.equal(y, m.spmv(to_dev(x)))


# ------------------------------------------------------------------ other code widths

WIDTH_CASES = {
    "half_1200x3000": lambda: (wl.bernoulli(1200, 3000, 0.5, 0.02, 51, 1), wl.x_vector(3000, 51, 1)),
    "dense_300x1031": lambda: (wl.bernoulli(300, 1031, 1.0, 0.02, 51, 2), wl.x_vector(1031, 51, 2)),
    "sparse97_600x9000": lambda: (wl.bernoulli(600, 9000, 0.03, 1.0, 51, 3), wl.x_vector(9000, 51, 3)),
    "ragged_301x777": lambda: (wl.bernoulli(301, 777, 0.7, 0.02, 51, 4), wl.x_vector(777, 51, 4)),
    "c4_512x4096": lambda: (wl.config4(rows=512, cols=4096).W, wl.config4(rows=512, cols=4096).x),
    "one_row_20000": lambda: (wl.bernoulli(1, 20000, 0.3, 0.02, 51, 5), wl.x_vector(20000, 51, 5)),
}


@pytest.mark.parametrize("variant", ["auto", "sub32", "wave_row", "wave_row_b64_r200", "wave_row_b256_r37",
                                     "wave_row_align64", "wave_row_align256_b256_r37", "wave_row_align512"])
@pytest.mark.parametrize("b_delta", [1, 2, 8])
@pytest.mark.parametrize("case", list(WIDTH_CASES))
def test_spmv_other_code_widths(case, b_delta, variant):
    """1-, 2- and 8-bit codes: same product, same tolerance, on both kernels."""
    W, x = WIDTH_CASES[case]()
    y = spmv_case(W, x, b_delta, **VARIANTS[variant])
    check_y(y, W, x, f"{case}/b{b_delta}/{variant}")


@pytest.mark.parametrize("b_delta", [1, 2, 8])
def test_other_code_widths_gpu_encoder_wrap_and_groups(b_delta):
    W = wl.bernoulli(700, 2500, 0.35, 0.02, 52, b_delta)
    W[13] = 0
    x = wl.x_vector(2500, 52, 1)
    enc = oracle.encode(W, b_delta)
    g = M.encode_device(to_dev(W), b_delta=b_delta)
    assert_same_encoding(g.fetch_device(), enc)
    rep = g.get_report()
    assert (rep.nnz, rep.pad_nnz, rep.alloc_nnz, rep.b_delta) == (enc.nnz, enc.pad_nnz, enc.alloc_nnz, b_delta)
    check_y(g.spmv(to_dev(x)), W, x, f"device-encoded b{b_delta}")
    # adopt the same device arrays through the wrap call
    bufs = [torch.from_numpy(a.copy()).cuda() for a in g.fetch_device()]
    w = M.wrap_device(700, 2500, enc.pad_nnz, *bufs, b_delta=b_delta)
    assert torch.equal(w.spmv(to_dev(x)), g.spmv(to_dev(x)))
    # a group that mixes code widths: one launch per width, same results
    others = [M.encode(W, b).to_device() for b in (4, 2, 8)]
    ys = M.spmv_group([g] + others, [to_dev(x)] * 4)
    torch.cuda.synchronize()
    for i, yi in enumerate(ys):
        check_y(yi, W, x, f"mixed group member {i}")
    # the small-batch product decodes the same widths (1-bit codes: one vector at a time)
    X = torch.stack([to_dev(wl.x_vector(2500, 52, 10 + b)) for b in range(7)])
    Y = g.spmm(X)
    torch.cuda.synchronize()
    for b in range(7):
        check_y(Y[b], W, wl.x_vector(2500, 52, 10 + b), f"spmm b{b_delta} column {b}")


def test_code_widths_full_size_llama_shape():
    """4096 x 11008 at 50 % (2-bit codes) and at 97 % (8-bit codes), in the launch shape bench.py times."""
    for b_delta, density, stream in ((2, 0.5, 61), (8, 0.03, 62), (2, 0.75, 63)):
        W = wl.bernoulli(4096, 11008, density, 0.02, 53, stream)
        x = wl.x_vector(11008, 53, stream)
        m = M.encode(W, b_delta).to_device()
        check_y(m.spmv(to_dev(x)), W, x, f"b{b_delta} d{density}")


# ------------------------------------------------------------------ grouped launches

def test_spmv_group_mixed_shapes_one_call():
    specs = [(300, 2048, 0.5), (64, 4096, 0.5), (500, 1000, 0.3), (40, 8000, 0.9),   # wave-per-row kernel
             (200, 300, 0.5),                                                         # short rows, few of them: the same kernel
             (77, 640, 0.0),                                                          # nothing stored
             (10, 100000, 0.2),                                                       # x larger than LDS
             (129, 5000, 1.0)]
    Ws = [wl.bernoulli(r, c, d, 0.02, 31, i) if d > 0 else np.zeros((r, c), dtype=np.uint16)
          for i, (r, c, d) in enumerate(specs)]
    xs = [wl.x_vector(c, 31, i) for i, (_, c, _) in enumerate(specs)]
    ms = [M.encode(W).to_device() for W in Ws]
    xd = [to_dev(x) for x in xs]
    ys = M.spmv_group(ms, xd)
    torch.cuda.synchronize()
    for i, (W, x, y) in enumerate(zip(Ws, xs, ys)):
        check_y(y, W, x, f"group member {i} {specs[i]}")
    # the single-product call gives bit-identical results (same kernel, same order of operations)
    for m, x, y in zip(ms, xd, ys):
        assert torch.equal(m.spmv(x), y)
    # q/k/v style: three matrices, one shared x
    q = [M.encode(wl.half_row_matrix(256, 4096, 60 + i)).to_device() for i in range(3)]
    xq = to_dev(wl.x_vector(4096, 31, 99))
    yq = M.spmv_group(q, [xq, xq, xq])
    torch.cuda.synchronize()
    for i in range(3):
        check_y(yq[i], wl.half_row_matrix(256, 4096, 60 + i), wl.x_vector(4096, 31, 99), f"qkv {i}")


def test_spmv_group_of_short_and_long_rows():
    """Short rows in so many that they go to sub-wave launches of their own, next to rows of the wave-per-row launch."""
    specs = [(20000, 300, 0.05), (300, 2048, 0.5), (24000, 96, 0.2), (500, 1000, 0.3)]
    Ws = [wl.bernoulli(r, c, d, 0.02, 33, i) for i, (r, c, d) in enumerate(specs)]
    xs = [wl.x_vector(c, 33, i) for i, (_, c, _) in enumerate(specs)]
    ms = [M.encode(W).to_device() for W in Ws]
    xd = [to_dev(x) for x in xs]
    ys = M.spmv_group(ms, xd)
    torch.cuda.synchronize()
    for i, (W, x, y) in enumerate(zip(Ws, xs, ys)):
        check_y(y, W, x, f"group member {i} {specs[i]}")
    for i, kernel in ((0, 1), (1, 2), (2, 1), (3, 2)):          # the kernels that the comment above says: sub-wave, wave-per-row
        M.set_tuning("spmv_kernel", kernel)
        try:
            assert torch.equal(ms[i].spmv(xd[i]), ys[i]), specs[i]
        finally:
            M.set_tuning("spmv_kernel", 0)


def test_group_argument_errors():
    lib = M.load_library()
    m = M.encode(wl.config1().W).to_device()
    x = to_dev(wl.config1().x)
    y = torch.empty(512, dtype=torch.float16, device="cuda")
    import ctypes
    VP = ctypes.c_void_p * 9
    hs = VP(*[m._h.value] * 9); xs = VP(*[x.data_ptr()] * 9); ys = VP(*[y.data_ptr()] * 9)
    assert lib.macko_spmv_group(0, hs, xs, ys, None) == -1
    assert lib.macko_spmv_group(9, hs, xs, ys, None) == -1
    unbound = M.encode(wl.config1().W)
    hs2 = VP(*([m._h.value] * 8 + [unbound._h.value]))
    hs2[1] = unbound._h.value
    assert lib.macko_spmv_group(2, hs2, xs, ys, None) == -5
    torch.cuda.synchronize()


def test_dense_gemv_group():
    shapes = [(300, 1024), (64, 4096), (33, 777), (128, 8200)]
    Ws = [wl.bernoulli(r, c, 1.0, 0.02, 41, i) for i, (r, c) in enumerate(shapes)]
    xs = [wl.x_vector(c, 41, i) for i, (_, c) in enumerate(shapes)]
    ys = M.dense_gemv_group([to_dev(W) for W in Ws], [to_dev(x) for x in xs])
    torch.cuda.synchronize()
    for W, x, y, shp in zip(Ws, xs, ys, shapes):
        check_y(y, W, x, f"gemv group {shp}")


# ------------------------------------------------------------------ small-batch products

def check_Y(Y_dev, W, X, what):
    for b in range(X.shape[0]):
        check_y(Y_dev[b], W, X[b], f"{what} vector {b}")


@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5, 7, 8, 11, 16])
def test_spmm_batches(batch):
    W = wl.bernoulli(333, 2000, 0.5, 0.02, 51, 1)
    W[5] = 0
    W[100:110] = 0
    X = np.stack([wl.x_vector(2000, 51, 10 + b) for b in range(batch)])
    m = M.encode(W).to_device()
    Y = m.spmm(to_dev(X))
    torch.cuda.synchronize()
    assert Y.shape == (batch, 333)
    check_Y(Y, W, X, f"batch {batch}")
    assert (Y[:, 5] == 0).all() and (Y[:, 100:110] == 0).all()
    # each vector agrees with the matrix-vector kernel to within both tolerances
    y0 = m.spmv(to_dev(X[0]))
    assert torch.allclose(Y[0].float(), y0.float(), atol=2e-3, rtol=2e-2)


def test_spmm_shapes_strides_and_fallbacks():
    cases = [
        (wl.bernoulli(70, 5000, 0.6, 0.02, 52, 1), 8),        # long rows
        (wl.bernoulli(40, 12000, 0.3, 0.02, 52, 2), 8),       # 8 vectors do not fit LDS: pieces of 4
        (wl.bernoulli(24, 30000, 0.2, 0.02, 52, 3), 6),       # pieces of 2
        (wl.bernoulli(10, 100000, 0.2, 0.02, 52, 4), 3),      # x larger than LDS: vector by vector
        (wl.bernoulli(200, 300, 0.5, 0.02, 52, 5), 4),        # short rows: vector by vector
        (wl.config4(rows=128, cols=2048).W, 8),
        (np.zeros((50, 640), dtype=np.uint16), 5),
        (wl.bernoulli(129, 1001, 1.0, 0.02, 52, 6), 8),       # dense, odd column count
    ]
    for i, (W, batch) in enumerate(cases):
        C = W.shape[1]
        X = np.stack([wl.x_vector(C, 52, 100 * i + b) for b in range(batch)])
        m = M.encode(W).to_device()
        # strided, unaligned X and Y
        Xbuf = torch.zeros((batch, C + 9), dtype=torch.float16, device="cuda")
        Xbuf[:, 1:C + 1] = to_dev(X)
        Ybuf = torch.full((batch, W.shape[0] + 5), 7.0, dtype=torch.float16, device="cuda")
        m.spmm(Xbuf[:, 1:C + 1], Ybuf[:, 3:3 + W.shape[0]])
        torch.cuda.synchronize()
        check_Y(Ybuf[:, 3:3 + W.shape[0]], W, X, f"case {i}")
        assert (Ybuf[:, :3] == 7).all() and (Ybuf[:, 3 + W.shape[0]:] == 7).all()


@pytest.mark.parametrize("batch", [2, 4, 8, 13])
@pytest.mark.parametrize("kind", ["b1", "b2", "b4", "b8", "fp8"])
def test_spmm_batch_kernel_every_code_width_and_8_bit_values(kind, batch):
    """Rows long enough for vectors to share a pass over the matrix, whichever batch kernel the library takes: one decode per
    stored entry, `batch` products.  Row lengths straddle steps, rows start inside chunks, some rows are empty."""
    b_delta = {"b1": 1, "b2": 2, "b4": 4, "b8": 8, "fp8": 4}[kind]
    density = {"b1": 0.9, "b2": 0.6, "b4": 0.5, "b8": 0.25, "fp8": 0.5}[kind]
    rows, cols = 150, 4100
    W = wl.bernoulli(rows, cols, density, 0.02, 54, b_delta)
    W[7] = 0
    W[40:43] = 0
    X = np.stack([wl.x_vector(cols, 54, 10 * batch + b) for b in range(batch)])
    if kind == "fp8":
        W8 = wl.fp8_values_of(W)
        m = M.encode_fp8(W8).to_device()
        assert m.report.pad_nnz // rows >= 384
        Y = m.spmm(to_dev(X))
        torch.cuda.synchronize()
        for b in range(batch):
            check_y8(Y[b], W8, X[b], f"fp8 batch {batch} vector {b}")
        y0 = m.spmv(to_dev(X[0]))
    else:
        m = M.encode(W, b_delta).to_device()
        assert m.report.pad_nnz // rows >= 384
        Y = m.spmm(to_dev(X))
        torch.cuda.synchronize()
        check_Y(Y, W, X, f"{kind} batch {batch}")
        y0 = m.spmv(to_dev(X[0]))
    torch.cuda.synchronize()
    assert (Y[:, 7] == 0).all() and (Y[:, 40:43] == 0).all()
    assert torch.allclose(Y[0].float(), y0.float(), atol=2e-3, rtol=2e-2)


def test_spmm_llama_shape_full_size():
    case = next(iter(wl.config2()))
    X = np.stack([wl.x_vector(case.cols, 53, b) for b in range(8)])
    m = M.encode(case.W).to_device()
    Y = m.spmm(to_dev(X))
    torch.cuda.synchronize()
    check_Y(Y, case.W, X, case.name)


@pytest.fixture(params=[1, 2], ids=["vector_units", "matrix_cores"])
def spmm_kernel(request):
    """Batches that both kernels serve go to the named one, whatever the library's estimates of their times say."""
    M.set_tuning("spmm_kernel", request.param)
    yield request.param
    M.set_tuning("spmm_kernel", 0)


@pytest.mark.parametrize("batch", [2, 3, 4, 5, 6, 7, 8, 13, 16])
def test_spmm_batches_on_either_kernel(spmm_kernel, batch):
    test_spmm_batches(batch)


def test_spmm_shapes_strides_and_fallbacks_on_either_kernel(spmm_kernel):
    test_spmm_shapes_strides_and_fallbacks()


@pytest.mark.parametrize("batch", [2, 4, 5, 6, 7, 8, 13])
@pytest.mark.parametrize("kind", ["b1", "b2", "b4", "b8", "fp8"])
def test_spmm_every_code_width_and_8_bit_values_on_either_kernel(spmm_kernel, kind, batch):
    test_spmm_batch_kernel_every_code_width_and_8_bit_values(kind, batch)


def test_spmm_llama_shape_full_size_on_either_kernel(spmm_kernel):
    test_spmm_llama_shape_full_size()


@pytest.mark.parametrize("kind", ["b1", "b2", "b4", "fp8"])
@pytest.mark.parametrize("rows,cols,batch", [(129, 1001, 8), (70, 5000, 7), (300, 2003, 6), (40, 12000, 8), (24, 30001, 5), (1030, 1100, 3), (50, 700, 2)])
def test_spmm_unaligned_vectors_on_either_kernel(spmm_kernel, kind, rows, cols, batch):
    """Pieces of 8, 4 and 2 vectors, filled and partly filled, and the same calls on the matrix cores: inputs (strided vectors on
    2 bytes, NaN around them, empty rows) and bound of test_spmm_tile_edges."""
    test_spmm_tile_edges(kind, rows, cols, batch)


# ------------------------------------------------------------------ GPU encoder

ENC_CASES = {
    "c1": lambda: wl.config1().W,
    "ragged": lambda: wl.bernoulli(301, 777, 0.5, 0.02, 9, 1),
    "very_sparse": lambda: wl.bernoulli(200, 3000, 0.02, 1.0, 9, 3),
    "dense": lambda: wl.bernoulli(100, 1031, 1.0, 0.02, 9, 4),
    "c4": lambda: wl.config4(rows=256, cols=2048).W,
    "c4b": lambda: wl.config4b(rows=128, cols=2048).W,
    "one_col": lambda: wl.bernoulli(300, 1, 0.5, 1.0, 9, 6),
    "empty": lambda: np.zeros((50, 600), dtype=np.uint16),
    "llama_slice": lambda: wl.half_row_matrix(512, 4096, 42),
}


@pytest.mark.parametrize("case", list(ENC_CASES))
def test_gpu_encoder_is_bit_exact(case):
    W = ENC_CASES[case]()
    enc = oracle.encode(W)
    g = M.encode_device(to_dev(W))
    assert_same_encoding(g.fetch_device(), enc)
    rep = g.report
    assert (rep.nnz, rep.pad_nnz, rep.alloc_nnz) == (enc.nnz, enc.pad_nnz, enc.alloc_nnz)
    ent = np.diff(enc.row_ptr.astype(np.int64))
    assert rep.empty_rows == int((ent == 0).sum()) and rep.max_row_entries == int(ent.max(initial=0))
    assert rep.total_bytes == enc.total_bytes
    # and the device-encoded handle multiplies correctly
    x = wl.x_vector(W.shape[1], 1, 1)
    y = g.spmv(to_dev(x))
    torch.cuda.synchronize()
    check_y(y, W, x, case)


def test_gpu_encoder_special_values_and_strided_unaligned_input():
    W = wl.bernoulli(64, 1001, 0.3, 0.02, 2, 2)
    W[0, 3] = 0x8000
    W[0, 5] = 0x0001
    W[1, 0] = 0x7C00
    W[2, 50] = 0xFE00
    W[5, 17] = 0x8001
    enc = oracle.encode(W)
    big = torch.zeros((64, 1003), dtype=torch.float16, device="cuda")     # ld = 1003: no 16-byte rows
    big[:, 1:1002] = to_dev(W)
    g = M.encode_device(big[:, 1:1002])
    assert_same_encoding(g.fetch_device(), enc)
    # the host encoder bound to the device gives the same bytes
    h = M.encode(W).to_device()
    assert_same_encoding(h.fetch_device(), enc)


# ------------------------------------------------------------------ dense GEMV baseline

@pytest.mark.parametrize("shape", [(512, 512), (300, 1000), (77, 4096), (64, 8200), (10, 40000), (33, 777), (5, 3)])
def test_dense_gemv(shape):
    R, C = shape
    W = wl.bernoulli(R, C, 1.0, 0.02, 12, R)
    x = wl.x_vector(C, 12, R)
    y = M.dense_gemv(to_dev(W), to_dev(x))
    torch.cuda.synchronize()
    check_y(y, W, x, f"gemv {shape}")
    for knobs in ({"gemv_block": 256, "gemv_rows_per_wg": 3}, {"gemv_block": 1024, "gemv_rows_per_wg": 1000}):
        for k, v in knobs.items():
            M.set_tuning(k, v)
        y = M.dense_gemv(to_dev(W), to_dev(x))
        torch.cuda.synchronize()
        check_y(y, W, x, f"gemv {shape} {knobs}")
        for k in knobs:
            M.set_tuning(k, 0)


def test_dense_gemv_with_leading_dimension_and_on_sparse_input():
    W = wl.half_row_matrix(200, 1024, 5)
    x = wl.x_vector(1024, 5, 5)
    big = torch.zeros((200, 1040), dtype=torch.float16, device="cuda")
    big[:, :1024] = to_dev(W)
    y = M.dense_gemv(big[:, :1024], to_dev(x))
    torch.cuda.synchronize()
    check_y(y, W, x, "ld=1040")
    # sparse and dense paths agree on the same matrix to within both tolerances
    ys = spmv_case(W, x)
    assert torch.allclose(ys.float(), y.float(), atol=2e-3, rtol=2e-2)


# ------------------------------------------------------------------ full-size configurations

def grouped_like_the_bench(handles, xs, singles):
    """The launches bench.py times: {q,k,v}, {o}, {gate,up}, {down}, and all seven at once.  Every product
    must come out exactly as from its own launch (the arithmetic per row does not depend on the launch shape)."""
    sq, gu, dn = handles
    xq, xg, xd = xs
    yq, yg, yd = singles
    for group, xv, want in (([sq] * 3, [xq] * 3, [yq] * 3), ([sq], [xq], [yq]), ([gu] * 2, [xg] * 2, [yg] * 2),
                            ([dn], [xd], [yd]),
                            ([sq] * 4 + [gu] * 2 + [dn], [xq] * 4 + [xg] * 2 + [xd], [yq] * 4 + [yg] * 2 + [yd])):
        got = M.spmv_group(group, xv)
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            assert torch.equal(g, w)


def test_config2_llama2_7b_shapes_full_size():
    handles, xs, singles = [], [], []
    for case in wl.config2():
        enc = oracle.encode(case.W)
        m = M.encode(case.W)
        assert_same_encoding(m.host_buffers(), enc)
        m.to_device()
        y = m.spmv(to_dev(case.x))
        torch.cuda.synchronize()
        check_y(y, case.W, case.x, case.name)
        handles.append(m); xs.append(to_dev(case.x)); singles.append(y)
        yd = M.dense_gemv(to_dev(case.W), to_dev(case.x))
        torch.cuda.synchronize()
        check_y(yd, case.W, case.x, case.name + " dense")
        g = M.encode_device(to_dev(case.W))
        assert_same_encoding(g.fetch_device(), enc)
    grouped_like_the_bench(handles, xs, singles)


@pytest.mark.parametrize("sparsity", wl.SWEEP_SPARSITIES)
def test_config3_sweep_matrix_full_size(sparsity):
    """Every level of the sparsity sweep at its full size: both encoders byte for byte against the
    oracle's encoding, y against the dense product by definition."""
    case = wl.config3(sparsity)
    enc = oracle.encode(case.W)
    m = M.encode(case.W)
    assert_same_encoding(m.host_buffers(), enc)
    m.to_device()
    y = m.spmv(to_dev(case.x))
    torch.cuda.synchronize()
    check_y(y, case.W, case.x, case.name)
    rep = m.report
    assert rep.effd_best <= rep.effd + 1e-9
    assert rep.pad_nnz == enc.pad_nnz and rep.padding_entries == enc.pad_nnz - enc.nnz
    assert_same_encoding(m.fetch_device(), enc)
    g = M.encode_device(to_dev(case.W))
    assert_same_encoding(g.fetch_device(), enc)
    yg = g.spmv(to_dev(case.x))
    torch.cuda.synchronize()
    assert torch.equal(yg, y)


def test_config4_adversarial_full_size():
    for case in (wl.config4(), wl.config4b()):
        enc = oracle.encode(case.W)
        m = M.encode(case.W)
        assert_same_encoding(m.host_buffers(), enc)
        m.to_device()
        y = m.spmv(to_dev(case.x))
        torch.cuda.synchronize()
        check_y(y, case.W, case.x, case.name)
        g = M.encode_device(to_dev(case.W))
        assert_same_encoding(g.fetch_device(), enc)


def test_config5_llama2_13b_layer_shapes_full_size():
    handles, xs, singles = [], [], []
    for case in wl.config5_layer():
        m = M.encode(case.W).to_device()
        y = m.spmv(to_dev(case.x))
        torch.cuda.synchronize()
        check_y(y, case.W, case.x, case.name)
        handles.append(m); xs.append(to_dev(case.x)); singles.append(y)
    grouped_like_the_bench(handles, xs, singles)


def test_config5_whole_stack_as_the_bench_issues_it():
    """The 224 products of the 32-layer 13B-shaped stack, built the way bench.py builds them (one layer's
    three matrices, the device buffers replicated to 224 distinct addresses: the first copy from the host
    encoder, the others from the GPU encoder), once through macko_spmv_many and once as the 128 grouped
    launches {q,k,v}, {o}, {gate,up}, {down} per layer.  Every one of the 448 results is compared with the
    oracle's dense product of its matrix."""
    plan = [("qkvo", 4), ("gate_up", 2), ("down", 1)]
    handles, xs, want = {}, {}, {}
    for case, (tag, mult) in zip(wl.config5_layer(), plan):
        enc = oracle.encode(case.W)
        first = M.encode(case.W).to_device()
        Wd = to_dev(case.W)
        hs = [first] + [M.encode_device(Wd) for _ in range(32 * mult - 1)]
        del Wd
        assert_same_encoding(hs[-1].fetch_device(), enc)
        handles[tag], xs[tag] = hs, to_dev(case.x)
        y64, s64 = oracle.dense_matvec(case.W, case.x)
        want[tag] = (y64, REL_TOL * s64 + ABS_TOL)

    def check(tag, y, what):
        y64, bound = want[tag]
        got = y.float().cpu().numpy().astype(np.float64)
        assert np.isfinite(got).all(), what
        assert (np.abs(got - y64) <= bound).all(), what

    seq = [(tag, layer * mult + k) for layer in range(32) for tag, mult in plan for k in range(mult)]
    assert len(seq) == 224
    # one library call
    ys = [torch.full((handles[t][0].rows,), float("nan"), dtype=torch.float16, device="cuda") for t, _ in seq]
    many = M.SpmvMany([handles[t][c] for t, c in seq], [xs[t] for t, _ in seq], ys)
    many.launch()
    torch.cuda.synchronize()
    for i, (t, c) in enumerate(seq):
        check(t, ys[i], f"spmv_many product {i} ({t} copy {c})")
    first_of = {t: next(ys[i] for i, (tt, _) in enumerate(seq) if tt == t) for t, _ in plan}
    for i, (t, _) in enumerate(seq):                      # same bytes, same kernel arithmetic: same bits
        assert torch.equal(ys[i], first_of[t])
    # 128 grouped launches on one stream
    n_launches = 0
    for layer in range(32):
        for tag, ks in (("qkvo", [0, 1, 2]), ("qkvo", [3]), ("gate_up", [0, 1]), ("down", [0])):
            mult = dict(plan)[tag]
            hs = [handles[tag][layer * mult + k] for k in ks]
            out = [torch.full((hs[0].rows,), float("nan"), dtype=torch.float16, device="cuda") for _ in ks]
            M.SpmvGroup(hs, [xs[tag]] * len(ks), out).launch()
            n_launches += 1
            torch.cuda.synchronize()
            for k, yk in zip(ks, out):
                check(tag, yk, f"grouped launch layer {layer} {tag}[{k}]")
    assert n_launches == 128


# Appendix D: the 31 matrix shapes of the paper's runtime sweep, each at its full size.
_APPD_SMALLEST = sorted(wl.APPENDIX_D_SHAPES, key=lambda rc: rc[0] * rc[1])[:5]
_APPD_CASES = [(r, c, 50) for r, c in wl.APPENDIX_D_SHAPES] + [(r, c, 90) for r, c in _APPD_SMALLEST]


@pytest.mark.parametrize("rows,cols,sparsity", _APPD_CASES, ids=[f"{r}x{c}_s{s}" for r, c, s in _APPD_CASES])
def test_appendix_d_shapes_full_size(rows, cols, sparsity):
    case = wl.appendix_d_case(rows, cols, sparsity)
    m = M.encode(case.W).to_device()
    y = m.spmv(to_dev(case.x))
    torch.cuda.synchronize()
    check_y(y, case.W, case.x, case.name)
    yd = M.dense_gemv(to_dev(case.W), to_dev(case.x))
    torch.cuda.synchronize()
    check_y(yd, case.W, case.x, case.name + " dense")


# ------------------------------------------------------------------ expanding the format on the device

EXPAND_CASES = dict(WIDTH_CASES)
EXPAND_CASES["empty_rows_257x1500"] = lambda: (_with_empty_rows(wl.bernoulli(257, 1500, 0.4, 0.02, 61, 1)),
                                                wl.x_vector(1500, 61, 1))
EXPAND_CASES["first_nonzero_late_64x5000"] = lambda: (_late_start(wl.bernoulli(64, 5000, 0.6, 0.02, 61, 2)),
                                                       wl.x_vector(5000, 61, 2))
# row buffers of the one-pass decoder: two wavefronts per workgroup, one, and rows too long for LDS
EXPAND_CASES["wide_6x30000"] = lambda: (wl.bernoulli(6, 30000, 0.5, 0.02, 61, 3), wl.x_vector(30000, 61, 3))
EXPAND_CASES["wide_5x45000"] = lambda: (wl.bernoulli(5, 45000, 0.4, 0.02, 61, 4), wl.x_vector(45000, 61, 4))
EXPAND_CASES["exactly_lds_2x81920"] = lambda: (wl.bernoulli(2, 81920, 0.2, 0.02, 61, 6), wl.x_vector(81920, 61, 6))
EXPAND_CASES["just_over_lds_2x81928"] = lambda: (wl.bernoulli(2, 81928, 0.2, 0.02, 61, 7), wl.x_vector(81928, 61, 7))
EXPAND_CASES["too_wide_for_lds_3x90000"] = lambda: (wl.bernoulli(3, 90000, 0.3, 0.02, 61, 5),
                                                     wl.x_vector(90000, 61, 5))


def _with_empty_rows(W):
    W[0] = 0
    W[100:131] = 0
    W[-1] = 0
    return W


def _late_start(W):
    W[:, :3000] = 0            # every row starts with padding entries only
    W[5, :] = 0
    W[5, 4999] = 0x3C00        # a row whose only non-zero is in the last column
    return W


@pytest.mark.parametrize("b_delta", [1, 2, 4, 8])
@pytest.mark.parametrize("case", list(EXPAND_CASES))
def test_columns_on_the_device_equal_the_oracles(case, b_delta):
    """Index reconstruction (Section 4.4, Alg. 1) in isolation: the column index of every stored
    entry, formed with the decode and the wavefront prefix sum the product uses, bit for bit."""
    W, _ = EXPAND_CASES[case]()
    enc = oracle.encode(W, b_delta)
    _, want = oracle.unpack(enc)
    m = M.encode(W, b_delta).to_device()
    got = m.columns_device()
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    assert got.shape[0] == max(enc.alloc_nnz, 1)
    assert np.array_equal(got[: enc.pad_nnz], want)
    assert (got[enc.pad_nnz:] == -1).all()                 # the tail is not touched


@pytest.mark.parametrize("b_delta", [1, 2, 4, 8])
@pytest.mark.parametrize("case", list(EXPAND_CASES))
def test_decode_on_the_device_round_trips_exactly(case, b_delta):
    W, _ = EXPAND_CASES[case]()
    want = oracle.decode(oracle.encode(W, b_delta))
    m = M.encode_device(to_dev(W), b_delta=b_delta)       # device encoder -> device decoder
    back = m.decode_device()
    torch.cuda.synchronize()
    assert np.array_equal(back.cpu().numpy().view(np.uint16), want)
    # into a wider, unaligned buffer: cells beyond cols keep their contents
    rows, cols = W.shape
    buf = torch.full((rows, cols + 5), 7.0, dtype=torch.float16, device="cuda")
    view = buf[:, 1: 1 + cols]
    rc = M.load_library().macko_decode_device(m._h, view.data_ptr(), buf.stride(0), 0)
    assert rc == 0
    torch.cuda.synchronize()
    host = buf.cpu().numpy().view(np.uint16)
    assert np.array_equal(host[:, 1: 1 + cols], want)
    assert (host[:, 0] == 0x4700).all() and (host[:, 1 + cols:] == 0x4700).all()


def test_expand_special_values_errors_and_full_size():
    W = wl.bernoulli(130, 900, 0.5, 0.02, 62, 1)
    W[3, 10:20] = [0x7C00, 0xFC00, 0x7E00, 0x0001, 0x8001, 0x8000, 0x0000, 0x7BFF, 0xFBFF, 0x03FF]
    m = M.encode(W).to_device()
    back = m.decode_device()
    torch.cuda.synchronize()
    assert np.array_equal(back.cpu().numpy().view(np.uint16), oracle.decode(oracle.encode(W)))
    lib = M.load_library()
    unbound = M.encode(W)
    rc = lib.macko_decode_device(unbound._h, back.data_ptr(), 900, 0)
    assert rc < 0 and "no device buffers" in M.status_string(rc)
    assert lib.macko_decode_device(m._h, back.data_ptr(), 899, 0) < 0          # ld < cols
    assert lib.macko_decode_device(m._h, 0, 900, 0) < 0
    assert lib.macko_columns_device(m._h, 0, 0) < 0
    assert lib.macko_columns_device(unbound._h, back.data_ptr(), 0) < 0
    # all-zero and zero-sized matrices
    z = M.encode(np.zeros((5, 64), dtype=np.uint16)).to_device()
    out = torch.full((5, 64), 3.0, dtype=torch.float16, device="cuda")
    z.decode_device(out)
    torch.cuda.synchronize()
    assert (out == 0).all()
    assert (z.columns_device().cpu().numpy() == -1).all()
    # one decoder-layer shape at full size, both ways
    case = list(wl.config2())[1]
    enc = oracle.encode(case.W)
    g = M.encode_device(to_dev(case.W))
    cols = g.columns_device()
    dense = g.decode_device()
    torch.cuda.synchronize()
    assert np.array_equal(cols.cpu().numpy()[: enc.pad_nnz], oracle.unpack(enc)[1])
    assert np.array_equal(dense.cpu().numpy().view(np.uint16), oracle.decode(enc))


# ------------------------------------------------------------------ checking adopted device arrays

@pytest.mark.parametrize("b_delta", [1, 2, 4, 8])
def test_check_device_accepts_valid_encodings_and_names_the_first_bad_row(b_delta):
    """Mistakes are planted in host copies of a valid encoding (made by the oracle), the copies are
    adopted with macko_wrap_device, and macko_check_device must name the first row that is wrong.
    No planted mistake makes a kernel read outside the arrays: bad pointers are reported undecoded."""
    rows, cols = 300, 2100
    W = wl.bernoulli(rows, cols, 0.4, 0.02, 71, b_delta)
    W[17] = 0
    W[299, cols - 1] = 0x3C00                                  # the last row reaches the last column
    enc = oracle.encode(W, b_delta)

    def wrapped(values, deltas, row_ptr, pad_nnz=None, ncols=cols):
        v = torch.from_numpy(values.copy()).cuda()
        d = torch.from_numpy(deltas.copy()).cuda()
        r = torch.from_numpy(row_ptr.astype(np.int64).astype(np.uint32).view(np.int32).copy()).cuda()
        return M.wrap_device(rows, ncols, enc.pad_nnz if pad_nnz is None else pad_nnz, v, d, r, b_delta)

    assert wrapped(enc.values, enc.deltas, enc.row_ptr).check_device() is None
    assert M.encode(W, b_delta).to_device().check_device() is None
    assert M.encode_device(to_dev(W), b_delta=b_delta).check_device() is None

    # one column too few: exactly the rows that reach the last column are wrong (row 299 does; find the first)
    _, colidx = oracle.unpack(enc)
    reach = [r for r in range(rows) if enc.row_ptr[r + 1] > enc.row_ptr[r] and colidx[enc.row_ptr[r + 1] - 1] == cols - 1]
    assert wrapped(enc.values, enc.deltas, enc.row_ptr, ncols=cols - 1).check_device() == reach[0]

    rp = enc.row_ptr.astype(np.int64)
    bad = rp.copy(); bad[0] = 8
    assert wrapped(enc.values, enc.deltas, bad).check_device() == 0                 # does not start at 0
    assert rp[119] > 0
    bad = rp.copy(); bad[120] = rp[119] - 1
    assert wrapped(enc.values, enc.deltas, bad).check_device() == 119              # decreasing
    bad = rp.copy(); bad[200] = enc.pad_nnz + 4096
    assert wrapped(enc.values, enc.deltas, bad).check_device() == 199              # beyond the arrays
    bad = rp.copy(); bad[rows] = enc.pad_nnz - 1
    assert wrapped(enc.values, enc.deltas, bad, pad_nnz=enc.pad_nnz).check_device() == rows - 1   # does not end at pad_nnz
    # a row boundary moved forward by a few entries: the row above it now decodes entries of the next row
    # and, being long enough, runs past the last column
    bad = rp.copy(); bad[51] = rp[53]
    got = wrapped(enc.values, enc.deltas, bad).check_device()
    assert got in (50, 51, 52)
    # all-zero and empty
    z = M.encode(np.zeros((4, 16), dtype=np.uint16), b_delta).to_device()
    assert z.check_device() is None
    lib = M.load_library()
    assert lib.macko_check_device(M.encode(W, b_delta)._h, 0, None) < 0             # not bound


# ------------------------------------------------------------------ 8-bit values

def check_y8(y_dev, W8, x, what=""):
    y64, s64 = oracle.dense_matvec8(W8, x)
    y = y_dev.float().cpu().numpy().astype(np.float64)
    err = np.abs(y - y64)
    tol = 1e-2 * s64 + 1e-3
    assert (err <= tol).all(), f"{what}: worst excess {float((err - tol).max()):.3e} at row {int((err - tol).argmax())}"


def test_fp8_every_bit_pattern_is_converted_like_the_oracle():
    """One row per E4M3 pattern (NaNs aside), a single entry each, x = 1: y must be the value itself,
    exactly (every E4M3 number is an fp16 number), including subnormals and both signs."""
    codes = np.array([c for c in range(256) if (c & 0x7F) not in (0, 0x7F)], dtype=np.uint8)
    W = np.zeros((len(codes), 512), dtype=np.uint8)
    W[np.arange(len(codes)), (np.arange(len(codes)) * 37) % 512] = codes
    W = np.repeat(W, 3, axis=0)                         # several rows per wavefront
    x = np.full(512, 0x3C00, dtype=np.uint16)
    m = M.encode_fp8(W).to_device()
    y = m.spmv(to_dev(x))
    torch.cuda.synchronize()
    want = oracle.fp8_to_double(np.repeat(codes, 3))
    assert np.array_equal(y.float().cpu().numpy().astype(np.float64), want)


FP8_CASES = {
    "half_1200x3000": lambda: wl.fp8_case(1200, 3000, 50),
    "dense_300x1031": lambda: wl.fp8_case(300, 1031, 0),
    "sparse90_600x9000": lambda: wl.fp8_case(600, 9000, 90),
    "ragged_301x777": lambda: wl.fp8_case(301, 777, 30),
    "one_row_20000": lambda: wl.fp8_case(1, 20000, 70),
    "short_rows_2000x96": lambda: wl.fp8_case(2000, 96, 50),
}


@pytest.mark.parametrize("variant", ["auto", "resident", "many_wgs_b256", "many_wgs_r37_b128", "align64",
                                     "align512_b256"])
@pytest.mark.parametrize("case", list(FP8_CASES))
def test_spmv_with_8_bit_values(case, variant):
    knobs = {"auto": {}, "resident": {"spmv_resident": 2}, "many_wgs_b256": {"spmv_resident": 1, "spmv_block": 256},
             "many_wgs_r37_b128": {"spmv_resident": 1, "spmv_rows_per_wg": 37, "spmv_block": 128},
             "align64": {"spmv_step_align": 64}, "align512_b256": {"spmv_step_align": 512, "spmv_block": 256}}[variant]
    c = FP8_CASES[case]()
    W = c.W.copy()
    if W.shape[0] > 40:
        W[10:30] = 0                                    # a run of empty rows
    enc = oracle.encode8(W, 4)
    for k, v in knobs.items():
        M.set_tuning(k, v)
    try:
        m = M.encode_fp8(W).to_device()
        v, d, r = m.fetch_device()
        assert np.array_equal(v, enc.values) and np.array_equal(d, enc.deltas) and np.array_equal(r, enc.row_ptr)
        y = m.spmv(to_dev(c.x))
        torch.cuda.synchronize()
    finally:
        for k in knobs:
            M.set_tuning(k, 0)
    check_y8(y, W, c.x, f"{case}/{variant}")
    if W.shape[0] > 40:
        assert (y[10:30] == 0).all()
    g = M.encode_device_fp8(torch.from_numpy(W).cuda())        # the GPU encoder: same bytes, same report
    gv, gd, gr = g.fetch_device()
    assert np.array_equal(gv, enc.values) and np.array_equal(gd, enc.deltas) and np.array_equal(gr, enc.row_ptr)
    rep = g.get_report()
    assert (rep.b_val, rep.nnz, rep.pad_nnz, rep.alloc_nnz, rep.total_bytes) == \
        (8, enc.nnz, enc.pad_nnz, enc.alloc_nnz, enc.total_bytes)
    for k, v in knobs.items():                          # same launch shape, hence the same summation order
        M.set_tuning(k, v)
    try:
        yg = g.spmv(to_dev(c.x))
    finally:
        for k in knobs:
            M.set_tuning(k, 0)
    assert torch.equal(yg, y)
    assert m.check_device() is None
    assert np.array_equal(m.columns_device().cpu().numpy()[: enc.pad_nnz], oracle.unpack(enc)[1])


def test_fp8_groups_unsupported_calls_and_full_size():
    lib = M.load_library()
    a, b = wl.fp8_case(700, 2048, 50), wl.fp8_case(900, 1024, 60)
    c16 = wl.appendix_d_case(500, 2048, 50)
    ma, mb, mc = M.encode_fp8(a.W).to_device(), M.encode_fp8(b.W).to_device(), M.encode(c16.W).to_device()
    ys = M.spmv_group([ma, mc, mb], [to_dev(a.x), to_dev(c16.x), to_dev(b.x)])      # mixed value widths, one call
    torch.cuda.synchronize()
    check_y8(ys[0], a.W, a.x, "group/a")
    check_y(ys[1], c16.W, c16.x, "group/16-bit")
    check_y8(ys[2], b.W, b.x, "group/b")
    # adopt a copy of the device arrays (a checkpoint loaded elsewhere)
    v, d, r = [t.clone() for t in ma.device_buffers()]
    w = M.wrap_device_fp8(700, 2048, ma.report.pad_nnz, v, d, r)
    assert w.get_report().b_val == 8 and w.check_device() is None
    yw = w.spmv(to_dev(a.x))
    torch.cuda.synchronize()
    assert torch.equal(yw, ys[0])
    # a batch of vectors, on whichever kernel
    xs = [wl.x_vector(2048, 88, i) for i in range(11)]
    X = torch.stack([to_dev(v) for v in xs])
    Y = ma.spmm(X)
    torch.cuda.synchronize()
    assert Y.shape == (11, 700)
    for i in (0, 7, 8, 10):
        check_y8(Y[i], a.W, xs[i], f"spmm/vector {i}")
    # the dense matrix back on the device, as bytes: aligned, and into a wider unaligned buffer
    for m, c in ((ma, a), (mb, b)):
        want = oracle.decode8(oracle.encode8(c.W, 4))
        back = m.decode_device()
        torch.cuda.synchronize()
        assert back.dtype == torch.uint8 and np.array_equal(back.cpu().numpy(), want)
        rows, cols = c.W.shape
        buf = torch.full((rows, cols + 5), 0x77, dtype=torch.uint8, device="cuda")
        assert lib.macko_decode_device(m._h, buf[:, 3:].data_ptr(), buf.stride(0), 0) == 0
        torch.cuda.synchronize()
        host = buf.cpu().numpy()
        assert np.array_equal(host[:, 3: 3 + cols], want)
        assert (host[:, :3] == 0x77).all() and (host[:, 3 + cols:] == 0x77).all()
    # the layer shapes at full size
    for (r, c) in ((4096, 4096), (11008, 4096), (4096, 11008)):
        case = wl.fp8_case(r, c, 50)
        m = M.encode_fp8(case.W).to_device()
        y = m.spmv(to_dev(case.x))
        torch.cuda.synchronize()
        check_y8(y, case.W, case.x, case.name)


def test_fp8_gpu_encoder_special_patterns_and_strided_unaligned_input():
    rng = np.random.default_rng(81)
    W = rng.integers(0, 256, size=(123, 1001), dtype=np.uint8)
    W[rng.random(W.shape) < 0.6] = 0
    W[3, 10:16] = [0x80, 0x7F, 0xFF, 0x01, 0x81, 0x00]      # -0 is a zero; NaN patterns and subnormals are values
    W[7] = 0
    enc = oracle.encode8(W, 4)
    big = torch.zeros((123, 1001 + 11), dtype=torch.uint8, device="cuda")
    big[:, 3: 3 + 1001] = torch.from_numpy(W).cuda()
    view = big[:, 3: 3 + 1001]                               # unaligned start, odd leading dimension
    lib = M.load_library()
    import ctypes
    h = ctypes.c_void_p()
    assert lib.macko_encode_device_fp8(view.data_ptr(), 123, 1001, big.stride(0), 0, ctypes.byref(h), None) == 0
    g = M.binding.MackoMatrix(h.value, None)
    gv, gd, gr = g.fetch_device()
    assert np.array_equal(gv, enc.values) and np.array_equal(gd, enc.deltas) and np.array_equal(gr, enc.row_ptr)
    # a layer shape at full size, against the host encoder's bytes
    case = wl.fp8_case(11008, 4096, 50)
    hv, hd, hr = M.encode_fp8(case.W).host_buffers()
    gv, gd, gr = M.encode_device_fp8(torch.from_numpy(case.W).cuda()).fetch_device()
    assert np.array_equal(gv, hv) and np.array_equal(gd, hd) and np.array_equal(gr, hr)
    assert np.array_equal(hv, oracle.encode8(case.W, 4).values)


# ------------------------------------------------------------------ maximum sizes

def test_more_than_2_pow_31_stored_entries():
    """46400 x 46400, fully dense: 2.15e9 stored entries, past the sign bit of a 32-bit index and half
    way to the format's limit of 2^32.  The encoding of a dense matrix is known in closed form (every
    code 0, row r starts at r * C, values = the matrix), so the GPU encoder is checked without the
    oracle's encoder; the product is checked against the oracle's dense product of the 464 distinct rows."""
    R = C = 46400
    blk = wl.bernoulli(464, C, 1.0, 0.02, 99, 1)            # 464 distinct rows, repeated 100 times
    assert ((blk & 0x7FFF) != 0).all()
    x = wl.x_vector(C, 99, 1)
    Wd = torch.from_numpy(blk.view(np.float16)).cuda().repeat(100, 1)
    m = M.encode_device(Wd)
    rep = m.get_report()
    assert rep.pad_nnz == R * C > 2 ** 31 and rep.nnz == R * C and rep.alloc_nnz == R * C
    vals, dels, rp = m.fetch_device()
    assert np.array_equal(rp.astype(np.int64), np.arange(R + 1, dtype=np.int64) * C)
    assert not dels.any()
    for row in (0, 463, 464, 23199, R - 1):
        assert np.array_equal(vals[row * C:(row + 1) * C], blk[row % 464]), row
    del vals, dels
    assert m.check_device() is None
    xd = to_dev(x)
    y = m.spmv(xd)
    torch.cuda.synchronize()
    y64, s64 = oracle.dense_matvec(blk, x)
    err = np.abs(y.float().cpu().numpy().astype(np.float64).reshape(100, 464) - y64[None, :])
    assert (err <= 1e-2 * s64[None, :] + 1e-3).all(), float(err.max())
    cols = m.columns_device()
    torch.cuda.synchronize()
    for row in (0, 1, 30000, R - 1):                          # entries beyond index 2^31 included
        assert torch.equal(cols[row * C:(row + 1) * C].cpu(), torch.arange(C, dtype=torch.int32)), row
    yd = M.dense_gemv(Wd, xd)
    torch.cuda.synchronize()
    err = np.abs(yd.float().cpu().numpy().astype(np.float64).reshape(100, 464) - y64[None, :])
    assert (err <= 1e-2 * s64[None, :] + 1e-3).all(), float(err.max())


# ------------------------------------------------------------------ many independent products in one call

def test_spmv_many_independent_products_eager_ordered_and_under_graph_capture():
    """macko_spmv_many deals grouped launches to the library's side streams.  Every product must equal
    the single-product call; work enqueued on the caller's stream before the call must be seen (the x
    vectors are written by a kernel on that stream right before) and work enqueued after it must see
    the results; captured into a graph, every replay must give the eager results again."""
    shapes = [(600, 2048, 0.5), (333, 1024, 0.6), (1200, 4096, 0.4), (64, 512, 0.5), (2000, 1536, 0.7)]
    mats, Ws = [], []
    for i in range(21):                                         # 21 products: three launches over three streams
        r, c, d = shapes[i % len(shapes)]
        W = wl.bernoulli(r, c, d, 0.02, 91, i)
        Ws.append(W)
        mats.append(M.encode(W, [4, 2, 4, 8, 4][i % 5]).to_device() if i % 7 else M.encode_fp8(wl.fp8_values_of(W)).to_device())
    xs_host = [wl.x_vector(W.shape[1], 91, i) for i, W in enumerate(Ws)]
    src = [to_dev(x) for x in xs_host]
    xs = [torch.zeros_like(s) for s in src]
    ys = [torch.empty(W.shape[0], dtype=torch.float16, device="cuda") for W in Ws]
    want = []
    for m, s in zip(mats, src):
        want.append(m.spmv(s).clone())
    torch.cuda.synchronize()
    many = M.SpmvMany(mats, xs, ys)
    main = torch.cuda.Stream()
    sums = [torch.zeros(1, dtype=torch.float32, device="cuda") for _ in ys]

    def enqueue():
        for x, s in zip(xs, src):                               # producers on the caller's stream ...
            x.copy_(s)
        many.launch(stream=torch.cuda.current_stream())
        for y, acc in zip(ys, sums):                            # ... and consumers after the call
            acc.copy_(y.float().abs().sum().reshape(1))

    with torch.cuda.stream(main):
        for rep in range(3):
            for x in xs:
                x.zero_()
            for y in ys:
                y.fill_(7.0)
            enqueue()
            main.synchronize()
            for i, (y, w, acc) in enumerate(zip(ys, want, sums)):
                assert torch.equal(y, w), f"eager rep {rep} product {i}"
                assert float(acc) == float(w.float().abs().sum()), f"consumer saw stale y, product {i}"
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=main):
            many.launch(stream=torch.cuda.current_stream())
        for rep in range(3):
            for y in ys:
                y.fill_(7.0)
            main.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for i, (y, w) in enumerate(zip(ys, want)):
                assert torch.equal(y, w), f"replay {rep} product {i}"
    # argument checks happen before anything is enqueued
    lib = M.load_library()
    assert lib.macko_spmv_many(-1, None, None, None, 0) < 0
    assert lib.macko_spmv_many(0, None, None, None, 0) == 0
    unbound = M.encode(Ws[0])
    bad = M.SpmvMany(mats[:9] + [unbound], xs[:9] + [xs[0]], ys[:9] + [ys[0]])
    assert bad.launch_raw(0) < 0


# ------------------------------------------------------------------ a chain of dependent products in one launch

def _chain_handles(shapes, seed, b_delta=4):
    return [M.encode(wl.half_row_matrix(r, c, 3000 + 10 * seed + i), b_delta).to_device()
            for i, (r, c) in enumerate(shapes)]


CHAINS = {
    # x of every product is the y of the one before: any stale or early read shows
    "tiny_4_phases": [(512, 512), (512, 512), (1024, 512), (512, 1024)],
    "ragged_3_phases": [(300, 777), (777, 300), (301, 777)],
    "layer_shapes": [(4096, 4096), (4096, 4096), (11008, 4096), (4096, 11008)],
    "eight_phases": [(640, 640)] * 8,
}


@pytest.mark.parametrize("b_delta", [4, 2])
@pytest.mark.parametrize("name", list(CHAINS))
def test_chain_of_dependent_products_equals_separate_launches(name, b_delta):
    """macko_spmv_chain: phase p + 1 reads what phase p wrote.  Per row the arithmetic is that of the
    wave-per-row kernel, so the results must equal those of separate launches in stream order bit
    for bit, and the first and last product are also checked against the oracle."""
    shapes = CHAINS[name]
    seed = sorted(CHAINS).index(name) + (10 if b_delta == 2 else 0)
    hs = _chain_handles(shapes, seed, b_delta)
    x0h = wl.x_vector(shapes[0][1], 7, seed)
    x0 = to_dev(x0h)
    M.set_tuning("spmv_kernel", 2)
    try:
        ref, x = [], x0
        for h in hs:
            x = h.spmv(x)
            ref.append(x)
        torch.cuda.synchronize()
    finally:
        M.set_tuning("spmv_kernel", 0)
    check_y(ref[0], wl.half_row_matrix(*shapes[0], 3000 + 10 * seed), x0h, name)
    ws = M.chain_workspace()
    ys = [torch.empty(h.rows, dtype=torch.float16, device="cuda") for h in hs]
    chain = M.SpmvChain([[(hs[i], x0 if i == 0 else ys[i - 1], ys[i])] for i in range(len(hs))], ws)
    for rep in range(10):
        for y in ys:
            y.fill_(float("nan"))
        chain.launch()
        torch.cuda.synchronize()
        assert chain.status() == (0, -1)
        for i, (y, r) in enumerate(zip(ys, ref)):
            assert torch.equal(y, r), f"{name} repetition {rep} phase {i}: {(y != r).sum().item()} rows differ"
    assert int(ws.to(torch.int32).abs().sum().item()) == 0          # the workspace is left zeroed
    last = len(hs) - 1
    check_y(ys[last], wl.half_row_matrix(*shapes[last], 3000 + 10 * seed + last),
            ref[last - 1].cpu().numpy().view(np.uint16), name + " last phase")


def test_chain_layer_step_as_the_bench_issues_it():
    """{q,k,v} -> {o} -> {gate,up} -> {down} of a Llama2-7B-shaped layer, several products per phase,
    against the four grouped launches of the same products, and against the oracle."""
    cases = list(wl.config2())
    h = {c.name.split("_")[1]: M.encode(c.W).to_device() for c in cases}
    x = {c.name.split("_")[1]: to_dev(c.x) for c in cases}
    hq, hg, hd = h["qkvo"], h["gate"], h["down"]
    xq, xg, xd = x["qkvo"], x["gate"], x["down"]

    def outs(m, n):
        return [torch.full((m.rows,), float("nan"), dtype=torch.float16, device="cuda") for _ in range(n)]
    yq, yo, yg, yd = outs(hq, 3), outs(hq, 1), outs(hg, 2), outs(hd, 1)
    phases = [[(hq, xq, y) for y in yq], [(hq, xq, yo[0])], [(hg, xg, y) for y in yg], [(hd, xd, yd[0])]]
    ws = M.chain_workspace()
    M.SpmvChain(phases, ws).launch()
    torch.cuda.synchronize()
    assert M.chain_status(ws) == (0, -1)
    for ph in phases:
        got = [y for _, _, y in ph]
        want = M.spmv_group([m for m, _, _ in ph], [xx for _, xx, _ in ph])
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            assert torch.equal(g, w)
    for c, y in zip(cases, (yq[0], yg[1], yd[0])):
        check_y(y, c.W, c.x, "chain " + c.name)
    check_y(yo[0], cases[0].W, cases[0].x, "chain o")


def test_chain_gives_up_when_told_not_to_wait_and_recovers():
    """The bounded wait, forced from the host: with "chain_no_wait" a workgroup that finds the phase
    before unfinished gives up at once.  The launch still ends normally, the status call reports the
    phase, and the next chain on the same workspace runs as if nothing had happened."""
    hs = _chain_handles([(4096, 4096), (4096, 4096), (4096, 4096)], 5)
    x0 = to_dev(wl.x_vector(4096, 7, 5))
    ys = [torch.empty(4096, dtype=torch.float16, device="cuda") for _ in hs]
    ws = M.chain_workspace()
    chain = M.SpmvChain([[(hs[i], x0 if i == 0 else ys[i - 1], ys[i])] for i in range(3)], ws)
    chain.launch()
    torch.cuda.synchronize()
    assert chain.status() == (0, -1)
    good = [y.clone() for y in ys]
    M.set_tuning("chain_no_wait", 1)
    try:
        chain.launch()
        torch.cuda.synchronize()                      # returns: every workgroup has left
        st, phase = chain.status()
    finally:
        M.set_tuning("chain_no_wait", 0)
    assert st == M.MACKO_E_WAIT_EXPIRED and phase in (1, 2)
    assert torch.equal(ys[0], good[0])                # phase 0 waits for nothing and is complete
    assert chain.status() == (0, -1)                  # the record was cleared by the call that read it
    for y in ys:
        y.fill_(float("nan"))
    chain.launch()
    torch.cuda.synchronize()
    assert chain.status() == (0, -1)
    for y, g in zip(ys, good):
        assert torch.equal(y, g)
    assert int(ws.to(torch.int32).abs().sum().item()) == 0


def test_chain_argument_checks():
    lib = M.load_library()
    hs = _chain_handles([(512, 512)], 6)
    x = to_dev(wl.x_vector(512, 7, 6))
    y = torch.empty(512, dtype=torch.float16, device="cuda")
    ws = M.chain_workspace()
    # one phase of one product is an ordinary product
    M.SpmvChain([[(hs[0], x, y)]], ws).launch()
    torch.cuda.synchronize()
    assert torch.equal(y, spmv_case(wl.half_row_matrix(512, 512, 3060), wl.x_vector(512, 7, 6), spmv_kernel=2))
    # nine phases, seventeen products
    assert M.SpmvChain([[(hs[0], x, y)]] * 9, ws).launch_raw(0) == -3
    assert M.SpmvChain([[(hs[0], x, y)] * 3] * 6, ws).launch_raw(0) == -3
    assert M.SpmvChain([[(hs[0], x, y)] * 9], ws).launch_raw(0) == -1            # more than MACKO_MAX_GROUP in a phase
    # workspace: too small, misaligned, missing
    small = torch.zeros(4096, dtype=torch.uint8, device="cuda")
    assert M.SpmvChain([[(hs[0], x, y)]], small).launch_raw(0) == -1
    big = torch.zeros(M.CHAIN_WORKSPACE_BYTES + 256, dtype=torch.uint8, device="cuda")
    assert M.SpmvChain([[(hs[0], x, y)]], big[8:]).launch_raw(0) == -1
    # 8-bit values and unbound handles are refused
    h8 = M.encode_fp8(wl.fp8_case(512, 512).W).to_device()
    assert M.SpmvChain([[(h8, x, y)]], ws).launch_raw(0) == -3
    assert M.SpmvChain([[(M.encode(wl.half_row_matrix(64, 64, 1)), x, y)]], ws).launch_raw(0) == -5
    empty = M.encode(np.zeros((64, 512), dtype=np.uint16)).to_device()
    assert M.SpmvChain([[(empty, x, torch.empty(64, dtype=torch.float16, device="cuda"))]], ws).launch_raw(0) == -3
    torch.cuda.synchronize()


# ------------------------------------------------------------------ a row depends on its own entries only

def _rows_ending_in_nonfinite(rows, cols, density, seed, fp8=False):
    """Every even row's last non-zero is an infinity or a NaN (a NaN only, for 8-bit values); odd rows are
    ordinary.  Most even rows end inside an 8-entry chunk that also holds the start of the next row."""
    W = wl.bernoulli(rows, cols, density, 0.02, 77, seed)
    if fp8:
        W = wl.fp8_values_of(W)
    for r in range(0, rows, 2):
        nz = np.flatnonzero(W[r])
        if nz.size:
            W[r, nz[-1]] = (0x7F if fp8 else (0x7C00, 0xFC00, 0x7E00)[(r // 2) % 3])
    return W


def _check_rows_independent(y_dev, W, x, what, dense=oracle.dense_matvec):
    y64, s64 = dense(W, x)
    y = y_dev.float().cpu().numpy().astype(np.float64)
    odd = np.arange(1, W.shape[0], 2)
    assert np.isfinite(y64[odd]).all()
    assert np.isfinite(y[odd]).all(), f"{what}: rows {odd[~np.isfinite(y[odd])][:8]} picked up a neighbour's inf/NaN"
    assert (np.abs(y[odd] - y64[odd]) <= REL_TOL * s64[odd] + ABS_TOL).all(), what
    even = np.arange(0, W.shape[0], 2)
    assert not np.isfinite(y[even]).any(), what
    assert np.array_equal(np.isnan(y[even]), np.isnan(y64[even])), what
    inf = even[np.isinf(y64[even])]
    assert np.array_equal(np.sign(y[inf]), np.sign(y64[inf])), what


@pytest.mark.parametrize("b_delta", [1, 2, 4, 8])
def test_inf_or_nan_at_the_end_of_a_row_stays_in_that_row(b_delta):
    """Section 4.4 makes y_i a function of row i alone.  The wave-per-row kernels load whole 8-entry chunks,
    so the lane that holds a row's start also holds the previous row's last entries; those must not reach
    this row's sum, not even as 0 * inf."""
    rows, cols = 130, 2048
    density = {1: 0.9, 2: 0.6, 4: 0.5, 8: 0.2}[b_delta]
    W = _rows_ending_in_nonfinite(rows, cols, density, b_delta)
    x = wl.x_vector(cols, 77, b_delta)
    x[x == 0] = 0x3C00
    for knobs in ({"spmv_kernel": 2}, {"spmv_kernel": 2, "spmv_step_align": 256},
                  {"spmv_kernel": 2, "spmv_step_align": 64, "spmv_block": 128, "spmv_rows_per_wg": 7},
                  {"spmv_kernel": 1, "spmv_lanes": 16}):
        y = spmv_case(W, x, b_delta=b_delta, **knobs)
        _check_rows_independent(y, W, x, f"b_delta {b_delta} {knobs}")
    # the small-batch kernel shares the pattern
    m = M.encode(W, b_delta).to_device()
    X = torch.stack([to_dev(x), to_dev(x)])
    Y = m.spmm(X)
    torch.cuda.synchronize()
    for b in range(2):
        _check_rows_independent(Y[b], W, x, f"spmm b_delta {b_delta} vector {b}")
    # and the chain (2- and 4-bit codes)
    if b_delta in (2, 4):
        y = torch.empty(rows, dtype=torch.float16, device="cuda")
        M.SpmvChain([[(m, to_dev(x), y)]]).launch()
        torch.cuda.synchronize()
        _check_rows_independent(y, W, x, f"chain b_delta {b_delta}")


def test_nan_at_the_end_of_a_row_stays_in_that_row_with_8_bit_values():
    rows, cols = 130, 2048
    W8 = _rows_ending_in_nonfinite(rows, cols, 0.5, 9, fp8=True)
    x = wl.x_vector(cols, 77, 9)
    x[x == 0] = 0x3C00
    for knobs in ({}, {"spmv_step_align": 256}):
        for k, v in knobs.items():
            M.set_tuning(k, v)
        try:
            y = M.encode_fp8(W8).to_device().spmv(to_dev(x))
            torch.cuda.synchronize()
        finally:
            for k in knobs:
                M.set_tuning(k, 0)
        _check_rows_independent(y, W8, x, f"8-bit values {knobs}", dense=oracle.dense_matvec8)


def test_chain_under_graph_capture_replays_like_eager():
    """macko_spmv_chain_static allocates nothing and records no memset, so it can be captured; every replay,
    with eager work and synchronisations between the replays, must reproduce the eager results, also when the
    chain's inputs changed in between (the graph holds pointers, not values)."""
    shapes = [(2048, 1536), (1536, 2048), (1024, 1536), (512, 1024)]
    hs = _chain_handles(shapes, 8)
    xa, xb = to_dev(wl.x_vector(1536, 7, 80)), to_dev(wl.x_vector(1536, 7, 81))
    x0 = torch.empty_like(xa)
    ys = [torch.empty(h.rows, dtype=torch.float16, device="cuda") for h in hs]
    chain = M.SpmvChain([[(hs[i], x0 if i == 0 else ys[i - 1], ys[i])] for i in range(4)])     # static scratch

    def eager(x):
        x0.copy_(x)
        chain.launch(stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert M.chain_status(None) == (0, -1)
        return [y.clone() for y in ys]

    main = torch.cuda.Stream()
    with torch.cuda.stream(main):
        want_a, want_b = eager(xa), eager(xb)        # also the first calls on this device: look-ups happen here
        assert not torch.equal(want_a[3], want_b[3])
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=main):
            chain.launch(stream=torch.cuda.current_stream())
        for rep, (x, want) in enumerate([(xa, want_a), (xb, want_b), (xb, want_b), (xa, want_a)]):
            x0.copy_(x)
            for y in ys:
                y.fill_(float("nan"))
            main.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for i, (y, w) in enumerate(zip(ys, want)):
                assert torch.equal(y, w), f"replay {rep} phase {i}"
            # eager work between replays: an ordinary product and another eager chain
            assert torch.equal(eager(x)[3], want[3])
        assert M.chain_status(None) == (0, -1)


# ------------------------------------------------------------------ batches on the matrix cores

def _batch_reference(W64, X64):
    """Y and the sums of magnitudes in 64 bits, [batch, rows]."""
    return X64 @ W64.T, np.abs(X64) @ np.abs(W64).T


@pytest.mark.parametrize("kind", ["b1", "b2", "b4", "fp8"])
@pytest.mark.parametrize("rows,cols,batch", [
    (1, 8, 9), (15, 63, 16), (16, 64, 17), (17, 65, 32), (33, 127, 33), (40, 129, 48), (31, 1000, 49), (48, 2047, 64),
    (20, 2048, 9), (19, 2049, 16), (18, 4095, 10), (16, 4096, 15), (35, 4097, 12), (23, 4097, 64), (9, 8193, 20), (7, 12000, 7),
    (4099, 77, 5), (4100, 300, 11), (4200, 130, 50),
    # several tiles a workgroup and several windows a tile; more than 64 rows a wavefront in 256 workgroups
    (4200, 4500, 12), (8500, 2300, 40), (9001, 2049, 64), (262160, 16, 9), (262160, 16, 17)])
def test_spmm_tile_edges(kind, rows, cols, batch):
    """Tiles of 16 rows, windows of 2048 or 4096 columns, groups of 128 columns, 16 vectors per instruction: the sizes
    around them, with empty rows, rows that start inside a chunk, values below 2^-14, strided and 2-byte aligned
    vectors whose surroundings hold NaN."""
    b_delta = {"b1": 1, "b2": 2, "b4": 4, "fp8": 4}[kind]
    rng = np.random.default_rng(rows * 131 + cols * 7 + batch)
    density = rng.choice([0.03, 0.3, 0.5, 0.9])
    W = (rng.standard_normal((rows, cols)) * 0.02 * (rng.random((rows, cols)) < density)).astype(np.float16)
    W[rng.random((rows, cols)) < 0.01] = np.float16(3e-6)                 # a subnormal number
    if rows > 4:
        W[3] = 0
        W[-1] = 0
    X = rng.standard_normal((batch, cols)).astype(np.float16)
    if kind == "fp8":
        W8 = wl.fp8_values_of(W.view(np.uint16))
        W64 = oracle.fp8_to_double(np.arange(256, dtype=np.uint8))[W8]
        m = M.encode_fp8(W8).to_device()
    else:
        W64 = W.astype(np.float64)
        m = M.encode(W, b_delta).to_device()
    Xbuf = torch.full((batch, cols + 3), float("nan"), dtype=torch.float16, device="cuda")
    Xbuf[:, 1:cols + 1] = torch.from_numpy(X).cuda()
    Ybuf = torch.full((batch, rows + 3), 7.0, dtype=torch.float16, device="cuda")
    m.spmm(Xbuf[:, 1:cols + 1], Ybuf[:, 1:rows + 1])
    torch.cuda.synchronize()
    Y = Ybuf[:, 1:rows + 1].cpu().numpy().astype(np.float64)
    ref, mag = _batch_reference(W64, X.astype(np.float64))
    # one rounding to fp16 (relative 2^-11, or half of the smallest fp16 number) of a 32-bit sum of `cols` terms
    bound = np.abs(ref) * 2.0 ** -11 + 2.0 ** -25 + mag * cols * 2.0 ** -24
    worst = np.max(np.abs(Y - ref) / bound)
    assert worst <= 1.01, (kind, rows, cols, batch, worst)
    assert (Ybuf[:, 0] == 7).all() and (Ybuf[:, rows + 1:] == 7).all()


@pytest.mark.parametrize("kind", ["b1", "b4", "fp8"])
@pytest.mark.parametrize("rows,cols,batch", [
    # panels of one tile: windows of 4096, 2048 and 1024 columns, one or two vector tiles a wavefront, three and four of them
    (2100, 3073, 60), (2500, 700, 60), (2500, 2049, 40), (2300, 2500, 30),
    # of two tiles, in two windows of one buffer and in two buffers; of three; several panels a workgroup
    (4300, 2050, 9), (4300, 2100, 20), (4300, 1030, 64), (8300, 1100, 31), (8300, 1200, 40), (20600, 130, 20), (20600, 130, 33),
    # one step of a row loaded at a time (3 % of the columns kept, by the seed), and two (90, 30 and 90 %)
    (2049, 3080, 64), (2051, 4100, 49), (2064, 4111, 50), (2050, 6200, 61),
    # vectors dealt to several workgroups: two groups of two tiles, the last one partly filled; groups of 8, as many as there are
    # compute units for and one too many
    (1500, 1100, 40), (1500, 129, 33), (2048, 300, 16), (2049, 300, 16), (40, 4500, 61),
    # groups of 16 on rows of more than two windows, groups of 8 on them, and more rows than that for up to 16 vectors
    (1500, 8200, 20), (1100, 9001, 32), (300, 8205, 12), (2100, 4100, 11),
    # rows of 7 steps and more with 17 to 32 vectors, of 14 and more with up to 16 (50, 30 and 50 % kept, by the seed)
    (2050, 9200, 17), (2064, 12417, 32), (2052, 19500, 16),
    # up to 8 vectors: pairs of groups of 128 columns, the second of a pair there, partly there and missing
    (40, 127, 3), (40, 128, 8), (41, 129, 8), (40, 256, 5), (40, 257, 7), (70, 383, 8), (33, 4097, 8), (2100, 2049, 7)])
def test_spmm_panel_shapes(kind, rows, cols, batch):
    """Every shape of the matrix-core kernel, with inputs and bound of test_spmm_tile_edges, whatever the estimates say about the call."""
    M.set_tuning("spmm_kernel", 2)
    try:
        test_spmm_tile_edges(kind, rows, cols, batch)
    finally:
        M.set_tuning("spmm_kernel", 0)


@pytest.mark.parametrize("kind", ["b1", "b4", "fp8"])
def test_spmm_tile_leaves_out_what_is_not_stored(kind):
    """An infinity or a NaN of a vector reaches the rows that store an entry at its column and no others; one of the
    matrix stays in its row.  Reference: the stored entries (padding included) one by one in 64 bits."""
    _leaves_out_what_is_not_stored(kind, 50, 2300, 34)


@pytest.mark.parametrize("kind", ["b1", "b4", "fp8"])
@pytest.mark.parametrize("rows,cols,batch", [
    # one row tile: one, two, three and four vector tiles, windows of 4096, 2048 and 1024 columns, one buffer and two; two and three row tiles
    (2100, 2300, 12), (2100, 2301, 20), (2100, 2300, 34), (2100, 301, 64), (2100, 3101, 64), (4300, 301, 12), (4300, 302, 20), (4300, 303, 64),
    (8300, 141, 20), (8300, 142, 64)])
def test_spmm_tile_leaves_out_what_is_not_stored_in_every_shape(kind, rows, cols, batch):
    """The same in the shapes that more rows take."""
    M.set_tuning("spmm_kernel", 2)
    try:
        _leaves_out_what_is_not_stored(kind, rows, cols, batch)
    finally:
        M.set_tuning("spmm_kernel", 0)


@pytest.mark.parametrize("rows,cols,batch", [(2100, 7301, 20), (2100, 14500, 12)])
def test_spmm_tile_leaves_out_what_is_not_stored_in_long_rows(rows, cols, batch):
    """The same where the vectors of a window are requested a window ahead (rows of 7 and of 14 steps and more)."""
    _leaves_out_what_is_not_stored("b4", rows, cols, batch)


def _leaves_out_what_is_not_stored(kind, rows, cols, batch):
    rng = np.random.default_rng(5)
    W = (rng.standard_normal((rows, cols)) * (rng.random((rows, cols)) < 0.5)).astype(np.float16)
    X = rng.standard_normal((batch, cols)).astype(np.float16)
    X[2, 100] = np.inf
    X[batch // 2, cols - 1] = np.nan
    X[batch - 1, 0] = -np.inf
    if kind == "fp8":
        m = M.encode_fp8(wl.fp8_values_of(W.view(np.uint16))).to_device()
        values, _, row_ptr = m.host_buffers()
        values = oracle.fp8_to_double(np.arange(256, dtype=np.uint8))[values]
    else:
        W[20, cols - 1] = np.inf
        m = M.encode(W, {"b1": 1, "b4": 4}[kind]).to_device()
        values, _, row_ptr = m.host_buffers()
        values = values.view(np.float16).astype(np.float64)
    Y = m.spmm(torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
    n = int(row_ptr[-1])
    columns = m.columns_device().cpu().numpy()[:n]
    with np.errstate(invalid="ignore"):
        ref = np.add.reduceat(values[:n] * X.astype(np.float64)[:, columns], row_ptr[:-1].astype(np.int64), axis=1)
    fine = np.isfinite(ref)
    assert not fine[2].all() and fine[2].any() and not fine[batch // 2].all() and fine[batch // 2].any() and fine[0, :20].all()
    assert np.array_equal(Y[~fine], ref[~fine], equal_nan=True)
    assert np.allclose(Y[fine], ref[fine], atol=2e-3, rtol=2e-3)


@pytest.mark.parametrize("kind", ["b2", "b4", "fp8"])
@pytest.mark.parametrize("cols,batch", [(2100, 20), (4300, 10), (900, 50)])
def test_spmm_tile_not_finite_in_later_tiles(kind, cols, batch):
    """Three tiles a workgroup (9000 rows): results that hold an infinity or a NaN are found and computed apart in each of
    them, their neighbours are what they are without it.  Reference as above, for rows of all three tiles."""
    rng = np.random.default_rng(cols + batch)
    rows = 9000
    W = (rng.standard_normal((rows, cols)) * (rng.random((rows, cols)) < 0.05)).astype(np.float16)
    X = rng.standard_normal((batch, cols)).astype(np.float16)
    X[1, 7] = np.inf
    X[batch - 1, cols - 1] = np.nan
    W[3::9, 7] = 0.5                                                       # in every tile some rows store these columns
    W[5::9, -1] = -0.25
    if kind == "fp8":
        m = M.encode_fp8(wl.fp8_values_of(W.view(np.uint16))).to_device()
        values, _, row_ptr = m.host_buffers()
        values = oracle.fp8_to_double(np.arange(256, dtype=np.uint8))[values]
    else:
        W[8999, 3] = -np.inf
        m = M.encode(W, int(kind[1])).to_device()
        values, _, row_ptr = m.host_buffers()
        values = values.view(np.float16).astype(np.float64)
    Y = m.spmm(torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
    columns = m.columns_device().cpu().numpy()
    X64 = X.astype(np.float64)
    hit = np.zeros((2, 3), dtype=bool)
    for r in list(range(0, 36)) + list(range(4500, 4572)) + list(range(8964, 9000)):      # 35 or 36 rows a workgroup
        a, b = int(row_ptr[r]), int(row_ptr[r + 1])
        with np.errstate(invalid="ignore"):
            ref = X64[:, columns[a:b]] @ values[a:b]
        fine = np.isfinite(ref)
        assert np.array_equal(Y[~fine, r], ref[~fine], equal_nan=True), r
        assert np.allclose(Y[fine, r], ref[fine], atol=2e-3, rtol=2e-3), r
        if r < 36:
            hit[0, r // 16] |= not fine[1]
            hit[1, r // 16] |= not fine[batch - 1]
    assert hit[:, :2].all()                                                # in the first workgroup's first two tiles at least


# ------------------------------------------------------------------ GPU encoder: windows, shared words, unaligned rows

@pytest.mark.parametrize("kind", ["b1", "b2", "b4", "b8", "fp8"])
@pytest.mark.parametrize("rows,cols,density,shift", [
    (70001, 3, 0.5, 0), (1000, 3, 0.5, 0), (257, 8, 1.0, 1), (300, 9, 0.1, 3), (64, 511, 0.9, 0), (65, 513, 0.5, 1), (40, 1024, 1.0, 0),
    (33, 1031, 0.97, 5), (30, 2055, 0.02, 7), (9, 40000, 0.0005, 0), (5, 70000, 0.0, 2), (12, 5000, 0.6, 0)])
def test_gpu_encoder_window_edges(kind, rows, cols, density, shift):
    """Rows of a few entries (many rows in one word of codes), rows that end at and around a full window of 1024 entries,
    gaps of more padding than a window holds, rows that begin at any element."""
    rng = np.random.default_rng(rows + 17 * cols)
    W = ((rng.standard_normal((rows, cols)) + 3) * (rng.random((rows, cols)) < density)).astype(np.float16)
    W[::3, 0] = 1.5
    W[1::3, -1] = -2.0
    W[rng.random((rows, cols)) < 0.01] = np.float16(-0.0)
    big = torch.full((rows, cols + shift + 1), 9.0, dtype=torch.float16, device="cuda")
    if kind == "fp8":
        W8 = wl.fp8_values_of(W.view(np.uint16))
        enc = oracle.encode8(W8)
        big = torch.full((rows, cols + shift + 1), 9, dtype=torch.uint8, device="cuda")
        big[:, shift:shift + cols] = torch.from_numpy(W8).cuda()
        g = M.encode_device_fp8(big[:, shift:shift + cols])
    else:
        b_delta = int(kind[1])
        enc = oracle.encode(W.view(np.uint16), b_delta)
        big[:, shift:shift + cols] = torch.from_numpy(W).cuda()
        g = M.encode_device(big[:, shift:shift + cols], b_delta=b_delta)
    assert_same_encoding(g.fetch_device(), enc)
    assert (g.report.nnz, g.report.pad_nnz, g.report.alloc_nnz) == (enc.nnz, enc.pad_nnz, enc.alloc_nnz)


@pytest.mark.parametrize("kind", ["b1", "b4", "fp8"])
@pytest.mark.parametrize("first", [1, 497, 1017, 1525])
def test_gpu_encoder_row_ends(kind, first):
    """Every remainder of the columns around one chunk of 8, one step of 512, two and three: the counting pass loads the last 8 columns of
    such rows out of place (of rows that do not lie on 4 bytes from three steps on).  The columns behind a row hold non-zeros."""
    rng = np.random.default_rng(first)
    for cols in range(first, first + 24):
        W = (rng.standard_normal((5, cols)) * (rng.random((5, cols)) < 0.4)).astype(np.float16)
        W[1] = 0
        W[2, -1] = 1.0
        big = torch.full((5, cols + 9), 9.0, dtype=torch.float16, device="cuda")
        if kind == "fp8":
            W8 = wl.fp8_values_of(W.view(np.uint16))
            enc = oracle.encode8(W8)
            big = torch.full((5, cols + 9), 9, dtype=torch.uint8, device="cuda")
            big[:, :cols] = torch.from_numpy(W8).cuda()
            g = M.encode_device_fp8(big[:, :cols])
        else:
            enc = oracle.encode(W.view(np.uint16), int(kind[1]))
            big[:, :cols] = torch.from_numpy(W).cuda()
            g = M.encode_device(big[:, :cols], b_delta=int(kind[1]))
        assert_same_encoding(g.fetch_device(), enc)
        assert (g.report.nnz, g.report.pad_nnz, g.report.alloc_nnz) == (enc.nnz, enc.pad_nnz, enc.alloc_nnz)


@pytest.mark.parametrize("rows,cols", [(3, 40), (700, 1501), (4096, 4096), (70000, 24)])
def test_gpu_encoding_is_over_when_the_call_returns(rows, cols):
    """The call watches a number that the stream writes behind the last kernel.  Other streams and the host read the arrays at once, and the
    dense matrix is overwritten on another stream at once."""
    gen = torch.Generator(device="cuda").manual_seed(rows)
    writer, reader = torch.cuda.Stream(), torch.cuda.Stream()
    for turn in range(6):
        W = torch.randn((rows, cols), generator=gen, device="cuda").half() * (torch.rand((rows, cols), generator=gen, device="cuda") < 0.5)
        keep = W.clone()
        torch.cuda.synchronize()
        g = M.encode_device(W, stream=writer)
        with torch.cuda.stream(reader):
            W.fill_(float("nan"))
            dense = g.decode_device()
        host = g.fetch_device()
        torch.cuda.synchronize()
        assert torch.equal(dense, keep + 0)
        if turn == 0:
            enc = oracle.encode(keep.cpu().numpy().view(np.uint16))
            assert_same_encoding(host, enc)
            assert (g.report.nnz, g.report.pad_nnz, g.report.alloc_nnz) == (enc.nnz, enc.pad_nnz, enc.alloc_nnz)


def test_gpu_encoder_blocks_are_reused_once_the_device_is_idle():
    """The memory of a destroyed handle goes to the next one of its size (equal patterns, so that it surely does).  Whatever stream still reads it
    when the handle is destroyed has read it before the next encoding writes there: the side stream is busy for some milliseconds
    before it comes to its reads."""
    gen = torch.Generator(device="cuda").manual_seed(5)
    side = torch.cuda.Stream()
    first = torch.randn((4096, 3072), generator=gen, device="cuda").half() * (torch.rand((4096, 3072), generator=gen, device="cuda") < 0.5)
    second = first.flip(0).contiguous()
    busy = torch.randn((8192, 8192), generator=gen, device="cuda")
    with torch.cuda.stream(side):
        for _ in range(2):                                     # what PyTorch and its libraries allocate for this is there before free memory is read
            busy = torch.tanh(busy @ busy)
        warm = [torch.empty_like(first) for _ in range(3)]
    warm.append(torch.empty_like(first))
    del warm
    M.encode_device(second).decode_device()
    for _ in range(4):
        torch.cuda.synchronize()
        m = M.encode_device(first)
        with torch.cuda.stream(side):
            for _ in range(4):
                busy = torch.tanh(busy @ busy)
            dense = [m.decode_device() for _ in range(3)]
        free = torch.cuda.mem_get_info()[0]
        waiting = not side.query()
        m.destroy()
        assert waiting and side.query()
        m = M.encode_device(second)
        assert abs(torch.cuda.mem_get_info()[0] - free) < 4 << 20          # the 30 MiB were neither freed nor allocated again
        again = m.decode_device()
        m.destroy()
        torch.cuda.synchronize()
        assert all(torch.equal(d, first + 0) for d in dense) and torch.equal(again, second + 0)


def test_kept_blocks_are_bounded_and_given_back():
    """At most 8 blocks and 256 MiB are kept; trim() frees them; handles that live share nothing."""
    W = torch.ones((2048, 4096), dtype=torch.float16, device="cuda")              # 20 MiB encoded
    torch.cuda.synchronize()
    M.trim()
    before = torch.cuda.mem_get_info()[0]
    handles = [M.encode_device(W) for _ in range(20)]
    alive = torch.cuda.mem_get_info()[0]
    assert before - alive >= 20 * (20 << 20)
    for m in handles[:19]:
        m.destroy()
    assert torch.equal(handles[19].decode_device(), W)
    assert before - torch.cuda.mem_get_info()[0] <= (256 + 40) << 20
    M.trim()
    assert before - torch.cuda.mem_get_info()[0] <= 40 << 20
    assert torch.equal(handles[19].decode_device(), W)


@pytest.mark.parametrize("kind", ["b1", "b2", "b4", "b8", "fp8"])
@pytest.mark.parametrize("first", [4, 504, 1016, 2040])
def test_gpu_encoder_rows_on_words(kind, first):
    """Rows that begin and end on 4 bytes go through a buffer that ends with the row: every such remainder around one chunk of 8, one
    step of 512, two and four.  The columns behind a row hold non-zeros."""
    rng = np.random.default_rng(first + 1)
    word = 4 if kind == "fp8" else 2
    for cols in range(first, first + 24, word):
        W = (rng.standard_normal((5, cols)) * (rng.random((5, cols)) < 0.4)).astype(np.float16)
        W[1] = 0
        W[2, -1] = 1.0
        if kind == "fp8":
            W8 = wl.fp8_values_of(W.view(np.uint16))
            enc = oracle.encode8(W8)
            big = torch.full((5, cols + 2 * word), 9, dtype=torch.uint8, device="cuda")
            big[:, :cols] = torch.from_numpy(W8).cuda()
            g = M.encode_device_fp8(big[:, :cols])
        else:
            enc = oracle.encode(W.view(np.uint16), int(kind[1]))
            big = torch.full((5, cols + 2 * word), 9.0, dtype=torch.float16, device="cuda")
            big[:, :cols] = torch.from_numpy(W).cuda()
            g = M.encode_device(big[:, :cols], b_delta=int(kind[1]))
        assert_same_encoding(g.fetch_device(), enc)
        assert (g.report.nnz, g.report.pad_nnz, g.report.alloc_nnz) == (enc.nnz, enc.pad_nnz, enc.alloc_nnz)


@pytest.mark.parametrize("kind", ["b1", "b2", "b4", "b8", "fp8"])
@pytest.mark.parametrize("rows,cols,density,shift", [
    (70, 1, 0.5, 0), (50, 7, 0.9, 1), (33, 2047, 0.5, 3), (20, 2048, 0.5, 0), (20, 2049, 0.4, 5), (12, 4096, 0.9, 8),
    (11, 4103, 0.03, 2), (7, 40001, 0.0003, 7), (3, 100000, 0.3, 0), (40, 300, 0.0, 4),
    (14, 4095, 0.5, 3), (14, 4097, 0.4, 0), (9, 8191, 0.5, 1), (9, 8192, 0.5, 0), (9, 8193, 0.5, 5)])
def test_decode_device_windows(kind, rows, cols, density, shift):
    """Rows around a window of 8192 bytes (4096 values of 16 bits, 8192 of 8), rows that begin at any element, steps that reach over several windows; the
    cells around the matrix keep what they hold."""
    rng = np.random.default_rng(rows + 13 * cols)
    W = ((rng.standard_normal((rows, cols)) + 3) * (rng.random((rows, cols)) < density)).astype(np.float16)
    W[::2, -1] = -2.0
    W[1::4] = 0
    W[W == 0] = 0                                                          # no -0
    if kind == "fp8":
        W = wl.fp8_values_of(W.view(np.uint16))
        W[W == 0x80] = 0                                                   # -0 comes back as +0
        m = M.encode_fp8(W).to_device()
        buf = torch.full((rows, cols + shift + 3), 9, dtype=torch.uint8, device="cuda")
    else:
        m = M.encode(W, int(kind[1])).to_device()
        buf = torch.full((rows, cols + shift + 3), 9.0, dtype=torch.float16, device="cuda")
    m.decode_device(buf[:, shift:shift + cols])
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert np.array_equal(got[:, shift:shift + cols].view(W.dtype), W)
    assert (got[:, :shift] == 9).all() and (got[:, shift + cols:] == 9).all()


@pytest.mark.parametrize("kind", ["b1", "b2", "b4", "b8", "fp8"])
@pytest.mark.parametrize("n", [9, 17, 32, 33, 65])
def test_spmv_many_wide_launches(kind, n):
    """More than 8 products of one code width: up to 32 in one launch, over ragged shapes (column counts that the lean
    staging of x does not take among them) and a matrix without rows; the arithmetic per row is that of a single launch."""
    rng = np.random.default_rng(n)
    mats, xs = [], []
    for i in range(n):
        rows, cols = (0, 700) if i == 4 else (int(rng.integers(1, 90)), int(rng.integers(700, 3000)))
        cols = cols // 8 * 8 if kind == "b4" else cols
        W = (rng.standard_normal((rows, cols)) * (rng.random((rows, cols)) < 0.6)).astype(np.float16)
        if kind == "fp8":
            mats.append(M.encode_fp8(wl.fp8_values_of(W.view(np.uint16)) if rows else W.astype(np.uint8)).to_device())
        else:
            mats.append(M.encode(W, int(kind[1])).to_device())
        xs.append(torch.from_numpy(rng.standard_normal(cols).astype(np.float16)).cuda())
    ys = [torch.full((m.rows,), 7.0, dtype=torch.float16, device="cuda") for m in mats]
    M.SpmvMany(mats, xs, ys).launch()
    want = [m.spmv(x) for m, x in zip(mats, xs)]
    torch.cuda.synchronize()
    for i in range(n):
        assert torch.equal(ys[i], want[i]), (kind, n, i)


@pytest.mark.parametrize("rows,cols", [(12287, 1500), (12288, 1500), (12289, 1500), (12288, 900), (12288, 2600), (24576, 700)])
def test_spmv_wavefronts_per_compute_unit_do_not_change_the_result(rows, cols):
    """Shapes on both sides of the rule that takes 24 instead of 16 wavefronts per compute unit (rows of up to 4 steps of
    512 entries, at least 128 steps or 64 rows per compute unit): a row is one wavefront's, whichever split is taken."""
    x = wl.x_vector(cols, 5, 1)
    W = wl.bernoulli(rows, cols, 0.1, 0.02, 5, rows)
    y = spmv_case(W, x)
    check_y(y, W, x, f"{rows}x{cols}")
    for block in (512, 768):
        assert torch.equal(y, spmv_case(W, x, spmv_resident=2, spmv_block=block)), (rows, cols, block)


@pytest.mark.parametrize("kind", ["b1", "b2", "b4", "fp8"])
@pytest.mark.parametrize("rows,cols,batch,skip", [(70, 1, 9, 0), (40, 3, 9, 0), (33, 127, 64, 0), (50, 129, 33, 2), (20, 2047, 12, 0),
                                                  (20, 2049, 17, 0), (37, 4097, 16, 0), (37, 4099, 50, 6), (16, 511, 7, 0),
                                                  # more rows: two to four vector tiles a wavefront or shared out to two, panels of
                                                  # one, two and three row tiles
                                                  (2100, 4099, 12, 0), (2100, 2051, 20, 0), (2100, 257, 40, 1), (2100, 129, 64, 0), (2100, 3073, 50, 0),
                                                  (4300, 131, 16, 0), (4300, 131, 17, 2), (4300, 133, 64, 0), (8300, 65, 20, 0), (8300, 67, 33, 0)])
def test_spmm_odd_columns_wherever_the_vectors_end(kind, rows, cols, batch, skip):
    """The vectors of an odd number of columns end in the middle of 4 bytes.  Whether they end at a page (4096 bytes), one
    element in front of or behind it, and whatever lies behind them, the result is the same bit for bit."""
    rng = np.random.default_rng(rows + cols)
    W = (rng.standard_normal((rows, cols)) * (rng.random((rows, cols)) < 0.6)).astype(np.float16)
    W[:, -1] = rng.standard_normal(rows).astype(np.float16)                # every row stores the last column
    if kind == "fp8":
        W8 = wl.fp8_values_of(W.view(np.uint16))
        W64 = oracle.fp8_to_double(np.arange(256, dtype=np.uint8))[W8]
        m = M.encode_fp8(W8).to_device()
    else:
        W64 = W.astype(np.float64)
        m = M.encode(W, int(kind[1])).to_device()
    X = rng.standard_normal((batch, cols)).astype(np.float16)
    ldx = cols + skip
    length = (batch - 1) * ldx + cols
    got = []
    for end in (0, 1, 2, -1, 1000):                                        # elements behind a page
        buf = torch.full((length + 6144,), float("nan"), dtype=torch.float16, device="cuda")
        at = ((length + 2047) // 2048 * 2048 + 2048 - length + end) - (buf.data_ptr() % 4096) // 2
        assert 0 <= at and (buf.data_ptr() + 2 * (at + length - end)) % 4096 == 0
        Xd = buf[at:at + length].as_strided((batch, cols), (ldx, 1))
        Xd.copy_(torch.from_numpy(X))
        got.append(m.spmm(Xd))
    torch.cuda.synchronize()
    ref, mag = _batch_reference(W64, X.astype(np.float64))
    bound = np.abs(ref) * 2.0 ** -11 + 2.0 ** -25 + mag * cols * 2.0 ** -24        # as in test_spmm_tile_edges
    assert np.max(np.abs(got[0].cpu().numpy().astype(np.float64) - ref) / bound) <= 1.01
    for y in got[1:]:
        assert torch.equal(y, got[0])


def _wrap_with_fewer_columns(W, cols, b_delta):
    """W on the device, encoded, and its arrays adopted again as a matrix of `cols` columns: the entries behind them
    are an encoding's that macko_check_device rejects."""
    m = M.encode_device(W, b_delta=b_delta)
    bufs = [torch.from_numpy(a.copy()).cuda() for a in m.fetch_device()]
    return M.wrap_device(W.shape[0], cols, m.report.pad_nnz, *bufs, b_delta=b_delta)


@pytest.mark.parametrize("b_delta", [1, 4])
@pytest.mark.parametrize("cols,beyond,batch", [(2112, 500, 20), (4200, 300, 9), (300, 900, 40)])
def test_spmm_tile_entries_beyond_the_last_column_stay_in_their_row(b_delta, cols, beyond, batch):
    """Rows that run past the last column (columns between the last one and the end of the tile's window) count there for
    nothing, also where a vector holds an infinity, and spoil no row of the next tile (4200 rows: two tiles a workgroup)."""
    rows = 4200
    g = torch.Generator(device="cuda").manual_seed(cols + batch)
    W = torch.empty((rows, cols + beyond), dtype=torch.float16, device="cuda").normal_(0.0, 0.02, generator=g)
    W.mul_(torch.rand(W.shape, generator=g, device="cuda") < 0.5)
    W[1::3, cols:] = 0
    w = _wrap_with_fewer_columns(W, cols, b_delta)
    X = torch.empty((batch, cols), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    X[2, 5] = float("inf")
    Y = w.spmm(X)
    torch.cuda.synchronize()
    Wc, Y = W[:, :cols].double().cpu().numpy(), Y.cpu().numpy().astype(np.float64)
    X = X.double().cpu().numpy()
    stored = Wc[:, 5] != 0
    # rows that store nothing at column 5 are as if it held 0 (padding entries of value 0 may lie there with 1-bit codes)
    ref = np.where(np.isfinite(X), X, 0.0) @ Wc.T
    fine = np.ones(Y.shape, dtype=bool)
    fine[2] = ~stored if b_delta == 4 else np.isfinite(Y[2])
    assert np.allclose(Y[fine], ref[fine], atol=2e-3, rtol=2e-3)
    assert not np.isfinite(Y[2][stored]).any()


@pytest.mark.parametrize("b_delta", [1, 4, 8])
@pytest.mark.parametrize("rows,cols,beyond", [(9000, 10300, 1500), (9000, 5001, 700), (300, 777, 90)])
def test_decode_device_entries_beyond_the_last_column_are_left_out(rows, cols, beyond, b_delta):
    """Rows that run past the last column lose what lies there and spoil no other row (9000 rows: a wavefront assembles
    several rows in the same window)."""
    g = torch.Generator(device="cuda").manual_seed(cols)
    W = torch.empty((rows, cols + beyond), dtype=torch.float16, device="cuda").normal_(0.0, 0.02, generator=g)
    W.mul_(torch.rand(W.shape, generator=g, device="cuda") < 0.06)
    W += 0.0                                                               # no -0
    W[1::3, cols:] = 0
    w = _wrap_with_fewer_columns(W, cols, b_delta)
    assert torch.equal(w.decode_device(), W[:, :cols])


def test_gpu_encoder_row_of_all_but_2_31_columns():
    """The widest row there is (2^31 - 1 columns, 4 GB): the loads ahead of its end stay in front of it.  Expected arrays by
    the format's rule: a gap of g columns takes (g - 1) / 256 padding entries of code 255 and a code of (g - 1) % 256."""
    cols = 2 ** 31 - 1
    W = torch.zeros((1, cols), dtype=torch.float16, device="cuda")
    at = [5, 6, 2 ** 30 + 3, cols - 1500, cols - 1]
    values, codes, prev = [], [], -1
    for i, c in enumerate(at):
        W[0, c] = i + 1.0
        pads, code = divmod(c - prev - 1, 256)
        values += [np.zeros(pads, np.float16), np.array([i + 1.0], np.float16)]
        codes += [np.full(pads, 255, np.uint8), np.array([code], np.uint8)]
        prev = c
    values, codes = np.concatenate(values), np.concatenate(codes)
    m = M.encode_device(W, b_delta=8)
    v, d, r = m.fetch_device()
    n = len(values)
    assert list(r) == [0, n] and m.report.nnz == len(at) and m.report.pad_nnz == n
    assert np.array_equal(v[:n].view(np.float16), values) and np.array_equal(d[:n], codes)
    assert not v[n:].any() and not d[n:].any()


@pytest.mark.parametrize("rows,cols,density,b_delta", [
    # row buffers where all rows are on the chip at once, and one round more
    (20, 11008, 0.02, 8), (1100, 10408, 0.5, 2), (1800, 10408, 0.5, 2), (300, 20000, 0.001, 4), (400, 28672, 0.07, 4), (260, 40000, 0.4, 1),
    # rows longer than LDS, cleared and scattered into, and the same in windows
    (1, 100000, 0.02, 4), (2, 81928, 0.1, 4), (16, 90000, 0.001, 4), (17, 90000, 0.001, 4), (60, 81928, 0.02, 8), (100, 81928, 0.02, 8),
    (200, 82000, 0.002, 8), (1, 100000, 0.0, 2), (2, 81928, 0.5, 1)])
@pytest.mark.parametrize("shift,pad", [(0, 8), (3, 5)])
def test_decode_device_long_rows_either_way(rows, cols, density, b_delta, shift, pad):
    """Both sides of the rule that decodes rows of more than 20 KB in windows, in row buffers or by a scatter, with rows on 16 bytes
    and not: the dense matrix back bit for bit, the cells around it untouched."""
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    W = torch.empty((rows, cols), dtype=torch.float16, device="cuda").normal_(0.0, 0.02, generator=g)
    W.mul_(torch.rand(W.shape, generator=g, device="cuda") < density)
    W[::2, -1] = 3.0
    W[1::5] = 0
    W += 0.0                                                               # no -0
    m = M.encode_device(W, b_delta=b_delta)
    buf = torch.full((rows, cols + pad), 9.0, dtype=torch.float16, device="cuda")
    m.decode_device(buf[:, shift:shift + cols])
    assert torch.equal(buf[:, shift:shift + cols], W)
    assert (buf[:, :shift] == 9).all() and (buf[:, shift + cols:] == 9).all()


@pytest.mark.parametrize("rows,cols,sparsity,batch", [
    # rows shorter than a step: one or two launches of the product with one vector, or the matrix cores
    (4200, 4096, 0.98, 5), (4200, 5000, 0.98, 6), (5000, 4096, 0.98, 6), (16, 5000, 0.98, 9), (513, 5000, 0.98, 9), (256, 4096, 0.97, 16),
    (256, 4500, 0.97, 12), (4200, 4100, 0.98, 5),
    # 9 to 12 vectors on sparse rows, in one round of tiles and more
    (4097, 6000, 0.97, 9), (4096, 6000, 0.97, 9), (4097, 6000, 0.97, 12), (4097, 6000, 0.97, 13), (4097, 6004, 0.97, 9),
    # 5 to 8 vectors where 8, 4 or 2 of them fit LDS: few rows, one round of tiles, more
    (300, 11008, 0.95, 8), (300, 11008, 0.8, 5), (1100, 11008, 0.9, 7), (1100, 11008, 0.3, 5), (4200, 9480, 0.9, 6), (4200, 9480, 0.3, 6),
    (300, 20008, 0.9, 5), (4200, 20008, 0.97, 6), (4200, 20008, 0.5, 8)])
@pytest.mark.parametrize("kind", ["b2", "b4", "fp8"])
def test_spmm_on_both_sides_of_the_rule_that_picks_its_kernel(kind, rows, cols, sparsity, batch):
    g = torch.Generator(device="cuda").manual_seed(rows + cols + batch)
    W = torch.empty((rows, cols), dtype=torch.float16, device="cuda").normal_(0.0, 0.02, generator=g)
    W.mul_(torch.rand(W.shape, generator=g, device="cuda") >= sparsity)
    if kind == "fp8":
        W8 = (W.float() * 32.0).to(torch.float8_e4m3fn)
        m, W64 = M.encode_device_fp8(W8.view(torch.uint8)), W8.float().double()
    else:
        m, W64 = M.encode_device(W, b_delta=int(kind[1])), W.double()
    X = torch.empty((batch, cols), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    Y = m.spmm(X).double()
    ref, mag = X.double() @ W64.T.contiguous(), X.double().abs() @ W64.abs().T.contiguous()
    bound = ref.abs() * 2.0 ** -11 + 2.0 ** -25 + mag * cols * 2.0 ** -24          # as in test_spmm_tile_edges
    assert float(((Y - ref).abs() / bound).max()) <= 1.01


def test_native_calls_do_what_the_general_ones_do(monkeypatch):
    """The binding's native functions against the same calls through ctypes: results, tensors handed in, errors; what they do not
    serve (another stream, tensors of a subclass, layouts the library refuses) goes the general way with them as without."""
    from paper_2511_13061_amd import binding as B
    native = B._native
    assert native is not None
    W = (torch.randn((70, 130), device="cuda") * (torch.rand((70, 130), device="cuda") < 0.5)).half()
    m, m8 = M.encode_device(W), M.encode_device_fp8(W.to(torch.float8_e4m3fn).view(torch.uint8))
    unbound, gone = M.encode(W.cpu().numpy()), M.encode_device(W)
    gone.destroy()
    x, X, wide = torch.randn(130, device="cuda").half(), torch.randn((5, 130), device="cuda").half(), torch.randn((5, 140), device="cuda").half()
    side = torch.cuda.Stream()

    class Sub(torch.Tensor):
        pass

    def on_side(f):
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            r = f()
        side.synchronize()
        return r

    y, Y = torch.empty(70, dtype=torch.float16, device="cuda"), torch.empty((5, 75), dtype=torch.float16, device="cuda")
    calls = [lambda: m.spmv(x), lambda: m.spmv(x, y), lambda: m8.spmv(x), lambda: m.spmv(x, stream=side), lambda: on_side(lambda: m.spmv(x)),
             lambda: m.spmv(x.as_subclass(Sub)), lambda: m.spmv(torch.nn.Parameter(x)), lambda: unbound.spmv(x), lambda: gone.spmv(x),
             lambda: gone.spmv(x, y), lambda: m.spmv(x.view(torch.uint8)[1:]), lambda: m.spmm(X), lambda: m.spmm(X[:1]), lambda: m.spmm(X[:0]),
             lambda: m.spmm(wide[:, 2:132]), lambda: m.spmm(X, Y[:, 1:71]), lambda: m.spmm(X, Y[:, :60][:, ::1]), lambda: m.spmm(X[:, ::2]),
             lambda: m.spmm(x), lambda: m.spmm(X.repeat(14, 1)), lambda: m.spmm(X[:, :99]), lambda: m8.spmm(X), lambda: unbound.spmm(X),
             lambda: m.decode_device(), lambda: m8.decode_device(), lambda: unbound.decode_device(), lambda: gone.decode_device(),
             lambda: on_side(lambda: m.decode_device())]

    def outcome(call):
        y.fill_(-3)
        Y.fill_(-3)
        try:
            r = call()
        except Exception as e:
            return type(e), str(e)
        torch.cuda.synchronize()
        return r.dtype, r.device, r.shape, r.stride(), r.requires_grad, r.view(torch.uint8 if r.dtype == torch.uint8 else torch.int16).tolist(), y.tolist(), Y.tolist()

    for i, call in enumerate(calls):
        with_native = outcome(call)
        with monkeypatch.context() as patch:
            patch.setattr(B, "_native", None)
            assert with_native == outcome(call), i


def test_native_calls_are_captured_into_a_graph():
    """spmv, spmm and decode_device without a stream argument go to PyTorch's current stream: captured on a side stream and replayed with
    other inputs they give the eager results.  A launch on any other stream would fail the capture or miss from the replays."""
    g = torch.Generator(device="cuda").manual_seed(3)
    W = torch.empty((300, 520), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    W.mul_(torch.rand(W.shape, generator=g, device="cuda") < 0.5)
    W += 0.0                                                               # no -0
    m = M.encode_device(W)
    x, X = torch.empty(520, dtype=torch.float16, device="cuda"), torch.empty((20, 520), dtype=torch.float16, device="cuda")
    y, Y = torch.empty(300, dtype=torch.float16, device="cuda"), torch.empty((20, 300), dtype=torch.float16, device="cuda")
    inputs = [(torch.randn(520, device="cuda", generator=g).half(), torch.randn((20, 520), device="cuda", generator=g).half()) for _ in range(3)]
    want = [(m.spmv(a), m.spmm(b)) for a, b in inputs]
    assert not torch.equal(want[0][0], want[1][0])
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        m.spmv(x, y)
        made = m.spmv(x)
        m.spmm(X, Y)
        dense = m.decode_device()
    for i in (0, 1, 2, 0):
        x.copy_(inputs[i][0])
        X.copy_(inputs[i][1])
        for t in (y, made, Y, dense):
            t.fill_(-3)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want[i][0]) and torch.equal(made, want[i][0]) and torch.equal(Y, want[i][1]) and torch.equal(dense, W), i
        assert torch.equal(m.spmv(x), want[i][0])                          # eager work between the replays


@pytest.mark.parametrize("align", [0, 8, 64, 256])
@pytest.mark.parametrize("rows,cols", [(1, 4096), (61, 4096), (1030, 4096), (33, 8192)])
def test_rows_in_step_with_8_bit_values_end_in_any_chunk(rows, cols, align):
    """Rows of about a multiple of 2048 entries with 8-bit values: those that end in one chunk of a step have it taken by one
    lane behind the last row.  Lengths of 9 less to 9 more than half of the columns, so that rows start and end anywhere in a chunk,
    one row empty, one NaN at a row's end, one launch of one matrix and one of two.  Reference and bound as for the batch products."""
    _rows_in_step(rows, cols, align, 0)


@pytest.mark.parametrize("shift", [-6, 1, 2, 3, 6])
@pytest.mark.parametrize("rows,cols", [(61, 4096), (700, 8192)])
def test_rows_in_step_on_both_sides_of_the_rule_for_their_ends(rows, cols, shift):
    """The same around the rule that gives such ends to one lane: whole steps and one entry on average, and more."""
    _rows_in_step(rows, cols, 0, shift)


def _rows_in_step(rows, cols, align, shift):
    rng = np.random.default_rng(rows + cols)
    W8 = np.zeros((rows, cols), dtype=np.uint8)
    for r in range(rows):
        n = cols // 2 + (r * 5) % 19 - 9 + shift
        W8[r, np.sort(rng.choice(cols, n, replace=False))] = rng.integers(1, 0x7F, n).astype(np.uint8) | (rng.integers(0, 2, n) << 7).astype(np.uint8)
    W64 = oracle.fp8_to_double(np.arange(256, dtype=np.uint8))[W8]
    if rows > 1000:
        W8[500], W64[500] = 0, 0.0
    if rows > 30:
        W8[20, np.flatnonzero(W8[20])[-1]] = 0x7F                          # NaN
    m = M.encode_fp8(W8).to_device()
    x = rng.standard_normal((2, cols)).astype(np.float16)
    xd = [torch.from_numpy(v).cuda() for v in x]
    M.set_tuning("spmv_step_align", align)
    try:
        ys = [m.spmv(xd[0]).cpu().numpy()] + [y.cpu().numpy() for y in M.spmv_group([m, m], xd)]
    finally:
        M.set_tuning("spmv_step_align", 0)
    assert np.array_equal(ys[0], ys[1], equal_nan=True)
    for y, v in zip(ys[1:], x.astype(np.float64)):
        ref, mag = W64 @ v, np.abs(W64) @ np.abs(v)
        fine = np.ones(rows, dtype=bool)
        if rows > 30:
            assert np.isnan(y[20])
            fine[20] = False
        bound = np.abs(ref) * 2.0 ** -11 + 2.0 ** -25 + mag * cols * 2.0 ** -24
        assert (np.abs(y.astype(np.float64) - ref)[fine] <= 1.01 * bound[fine]).all()


@pytest.mark.parametrize("rows,cols,batch,offset,ldy", [(4099, 300, 5, 4, 4108), (4099, 300, 20, 4, 4108), (70, 2100, 64, 0, 76), (70, 2100, 9, 2, 76),
                                                        (9, 130, 16, 8, 17)])
def test_spmm_results_stored_four_at_a_time(rows, cols, batch, offset, ldy):
    """Results on 8 bytes and off them, last rows of a panel that are no four, an infinity among four results; nothing beside
    the results is written.  Reference and bound as in test_spmm_tile_edges."""
    rng = np.random.default_rng(rows + batch)
    W = (rng.standard_normal((rows, cols)) * (rng.random((rows, cols)) < 0.4)).astype(np.float16)
    W[rows - 2, 3] = np.inf
    X = rng.standard_normal((batch, cols)).astype(np.float16)
    Y = torch.full((batch, ldy), 7.0, dtype=torch.float16, device="cuda")
    M.encode(W).to_device().spmm(torch.from_numpy(X).cuda(), Y[:, offset:offset + rows])
    torch.cuda.synchronize()
    Y = Y.cpu().numpy().astype(np.float64)
    assert (Y[:, :offset] == 7).all() and (Y[:, offset + rows:] == 7).all()
    Y = Y[:, offset:offset + rows]
    assert np.array_equal(Y[:, rows - 2], np.sign(X[:, 3].astype(np.float64)) * np.inf)
    W[rows - 2, 3] = 0
    Y[:, rows - 2] = (X.astype(np.float64) @ W[rows - 2].astype(np.float64))
    ref, mag = _batch_reference(W.astype(np.float64), X.astype(np.float64))
    assert (np.abs(Y - ref) <= 1.01 * (np.abs(ref) * 2.0 ** -11 + 2.0 ** -25 + mag * cols * 2.0 ** -24)).all()


@pytest.mark.parametrize("kind", ["b1", "b4", "fp8"])
@pytest.mark.parametrize("rows,cols,sparsity,batch", [
    # 2 to 8 vectors: short rows, few rows and many, pieces of 8, 4 and 2, odd columns
    (344, 352, 0.62, 8), (2960, 656, 0.82, 4), (1256, 352, 0.53, 3), (4100, 2, 0.1, 2), (70, 2001, 0.9, 2), (1024, 4096, 0.5, 8),
    (4096, 4096, 0.5, 4), (718, 8797, 0.5, 8), (500, 9000, 0.6, 3), (60, 30000, 0.7, 2),
    # long rows of few: three steps loaded at a time
    (300, 13000, 0.8, 16), (40, 8200, 0.5, 9)])
def test_spmm_either_way_for_few_vectors(kind, rows, cols, sparsity, batch):
    """Both ways that the estimates of tile_is_faster choose from, with inputs and bound of the test above."""
    test_spmm_on_both_sides_of_the_rule_that_picks_its_kernel(kind, rows, cols, sparsity, batch)


@pytest.mark.parametrize("rows,cols,sparsity,batch,vals", [
    # x beyond LDS: vector by vector 2 to 9 times as slow
    (226, 178280, 0.99, 6, 16), (52, 88736, 0.95, 5, 16), (40, 300001, 0.999, 2, 16),
    # pieces of 3 and 4 vectors, one dense row to a wavefront: the matrix cores 1.3 times as slow; x of one vector fits LDS: 1.5 times
    (3832, 10352, 0.526, 3, 8), (2733, 11072, 0.333, 4, 8), (3077, 5728, 0.317, 3, 8), (376, 53088, 0.956, 2, 16),
    # short rows, a group of single products in one launch: the matrix cores 1.3 to 1.6 times as slow
    (504, 448, 0.904, 4, 16), (195, 3240, 0.957, 3, 16), (47, 2608, 0.945, 2, 16), (1000, 300, 0.5, 2, 16),
    # and calls that the matrix cores win by as much
    (1392, 1012, 0.87, 8, 16), (718, 8797, 0.5, 8, 16), (8872, 280, 0.49, 2, 16),
    # a group whose wavefronts take two rows, one after the other
    (600, 100, 0.4, 8, 16), (900, 100, 0.4, 7, 16)])
def test_spmm_takes_the_faster_kernel(rows, cols, sparsity, batch, vals):
    """Where the two batch kernels differ by 1.25 times and more the library's choice is within 1.15 times of the better one (a graph of 20
    calls, so that the host's pace does not count; least of 5 replays), and the results are right."""
    g = torch.Generator(device="cuda").manual_seed(rows)
    W = torch.empty((rows, cols), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    W.mul_(torch.rand(W.shape, generator=g, device="cuda") >= sparsity)
    W8 = W.to(torch.float8_e4m3fn)
    m = M.encode_device_fp8(W8.view(torch.uint8)) if vals == 8 else M.encode_device(W)
    X = torch.empty((batch, cols), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)

    out = torch.empty((batch, rows), dtype=torch.float16, device="cuda")

    def time_of(kernel):
        M.set_tuning("spmm_kernel", kernel)
        m.spmm(X, out)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                m.spmm(X, out)
        M.set_tuning("spmm_kernel", 0)
        best = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            b.synchronize()
            best.append(a.elapsed_time(b))
        return min(best[1:])

    auto, vectors, cores = time_of(0), time_of(1), time_of(2)
    assert auto <= 1.15 * min(vectors, cores), (auto, vectors, cores)
    Y, X64, W64 = m.spmm(X).double(), X.double(), (W8.float() if vals == 8 else W).double()
    bound = (X64 @ W64.T).abs() * 2.0 ** -11 + 2.0 ** -25 + (X64.abs() @ W64.abs().T) * cols * 2.0 ** -24      # as in test_spmm_tile_edges
    assert float(((Y - X64 @ W64.T).abs() / bound).max()) <= 1.01


@pytest.mark.parametrize("batch", [2, 4, 5, 9, 16])
@pytest.mark.parametrize("rows,cols,sparsity", [(300, 82000, 0.95), (1000, 82000, 0.995), (17, 82001, 0.99), (60, 81000, 0.5)])
def test_spmm_of_8_bit_values_with_x_beyond_lds(rows, cols, sparsity, batch):
    """8-bit values and an x beyond LDS have no vector kernel: from two vectors on the matrix cores serve the call whatever the
    estimates say, one vector is refused as macko_spmv refuses it."""
    g = torch.Generator(device="cuda").manual_seed(rows + batch)
    W = torch.empty((rows, cols), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    W.mul_(torch.rand(W.shape, generator=g, device="cuda") >= sparsity)
    W8 = W.to(torch.float8_e4m3fn)
    m = M.encode_device_fp8(W8.view(torch.uint8))
    X = torch.empty((batch, cols), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    with pytest.raises(M.MackoError) as refused:
        m.spmm(X[:1])
    assert refused.value.status == -3
    Y = m.spmm(X).double()
    W64 = W8.float().double()
    ref, mag = X.double() @ W64.T.contiguous(), X.double().abs() @ W64.abs().T.contiguous()
    bound = ref.abs() * 2.0 ** -11 + 2.0 ** -25 + mag * cols * 2.0 ** -24          # as in test_spmm_tile_edges
    assert float(((Y - ref).abs() / bound).max()) <= 1.01


@pytest.mark.parametrize("kind", ["b2", "b4", "fp8"])
@pytest.mark.parametrize("rows,cols,sparsity,batch", [
    # 17 to 32 vectors: a row of just under and just over 7 steps, odd columns; 9 to 16: of 14 steps, several rows a wavefront
    (2101, 7169, 0.501, 20), (2101, 7177, 0.495, 20), (2049, 9001, 0.4, 17), (4096, 12417, 0.5, 32), (4000, 8192, 0.3, 31),
    (2101, 14337, 0.501, 12), (2101, 14345, 0.495, 12), (2049, 16385, 0.4, 9), (2500, 19500, 0.5, 16), (8300, 8001, 0.05, 12)])
def test_spmm_vectors_requested_a_window_ahead(kind, rows, cols, sparsity, batch):
    """Both sides of the rules for long rows, with inputs and bound of test_spmm_on_both_sides_of_the_rule_that_picks_its_kernel."""
    M.set_tuning("spmm_kernel", 2)
    try:
        test_spmm_on_both_sides_of_the_rule_that_picks_its_kernel(kind, rows, cols, sparsity, batch)
    finally:
        M.set_tuning("spmm_kernel", 0)


@pytest.mark.parametrize("kind", ["b4", "fp8"])
@pytest.mark.parametrize("rows_of_the_wide,n_wide", [(300, 1), (700, 8), (2100, 1)])
def test_spmv_many_with_a_wide_x_among_others(kind, rows_of_the_wide, n_wide):
    """Matrices whose x takes more than 36 KB of LDS share the launch of the others or go apart, by their rows; the results are
    those of single products, whatever the order and with a matrix without rows between them."""
    rng = np.random.default_rng(rows_of_the_wide + n_wide)
    shapes = [(int(rng.integers(1, 90)), int(rng.integers(700, 3000))) for _ in range(23)] + [(rows_of_the_wide, 20000 + 8 * i) for i in range(n_wide)]
    shapes = [shapes[i] for i in rng.permutation(len(shapes))]
    shapes.insert(5, (0, 700))
    mats, xs = [], []
    for rows, cols in shapes:
        W = (rng.standard_normal((rows, cols)) * (rng.random((rows, cols)) < 0.5)).astype(np.float16)
        mats.append((M.encode_fp8(wl.fp8_values_of(W.view(np.uint16)) if rows else W.astype(np.uint8)) if kind == "fp8" else M.encode(W)).to_device())
        xs.append(torch.from_numpy(rng.standard_normal(cols).astype(np.float16)).cuda())
    ys = [torch.full((m.rows,), 7.0, dtype=torch.float16, device="cuda") for m in mats]
    M.SpmvMany(mats, xs, ys).launch()
    want = [m.spmv(x) for m, x in zip(mats, xs)]
    torch.cuda.synchronize()
    for i in range(len(mats)):
        assert torch.equal(ys[i], want[i]), (kind, i, shapes[i])
