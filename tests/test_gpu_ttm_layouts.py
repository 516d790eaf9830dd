"""FP64 mode products over every layout of the operands that the direct-load
kernel takes, itself or through an aligned copy of the factor, against numpy
in FP64.

Tolerance: a sum of J products in another order differs by at most about
J u |M||Y| (1e-12 of it here), plus one rounding of a float32 output; FP32
products (J + 2) 2^-23 |M||Y|.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def tk():
    import paper_1901_06043_amd as tk
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    tk.lib()
    return tk


def check(tk, dims, n, K, layout, ydt, zdt, offset=0, fp32=False):
    rng = np.random.default_rng(sum(dims) + K)
    shape = list(reversed(dims))
    Y = rng.standard_normal(shape).astype(ydt)
    M = rng.standard_normal((K, dims[n]))
    t = {np.float32: torch.float32, np.float64: torch.float64}
    buf = torch.empty(Y.size + offset, dtype=t[ydt], device="cuda")
    buf[offset:] = torch.from_numpy(Y.reshape(-1))
    if layout == "rows":
        m = torch.from_numpy(M).cuda()
    elif layout == "columns":
        m = torch.from_numpy(np.ascontiguousarray(M.T)).cuda().t()
    else:  # every other column of a wider matrix
        wide = torch.zeros((K, 2 * dims[n]), dtype=torch.float64, device="cuda")
        wide[:, ::2] = torch.from_numpy(M)
        m = wide[:, ::2]
    z = tk.ttm(buf[offset:].view(shape), n, m, dims=dims, out_dtype=t[zdt], fp32_products=fp32).cpu().numpy()
    ax = len(dims) - 1 - n
    ref = np.moveaxis(np.tensordot(M, Y.astype(np.float64), axes=([1], [ax])), 0, ax)
    mag = np.moveaxis(np.tensordot(np.abs(M), np.abs(Y).astype(np.float64), axes=([1], [ax])), 0, ax)
    assert z.dtype == zdt
    tol = 1e-12 * mag + (2.0 ** -23 * np.abs(ref) if zdt == np.float32 else 0.0)
    if fp32:
        tol = tol + (dims[n] + 2) * 2.0 ** -23 * mag
    assert np.all(np.abs(z - ref) <= tol), (dims, n, K, layout)


# L = 1 and L > 1; strides that are 0, 1, 2, 3 modulo 4 (16-byte, 4-byte
# loads); one chunk, a ragged last chunk of at most and of more than 8 indices;
# one, several and ragged row tiles; few and ragged columns
SHAPES = [
    ([16, 131], 0, 65), ([17, 130], 0, 129), ([18, 300], 0, 200), ([19, 129], 0, 65), ([40, 9, 15], 0, 90),
    ([4, 33, 40], 1, 66), ([5, 24, 30], 1, 65), ([6, 41, 30], 1, 130), ([131, 47], 1, 301), ([128, 64, 2], 1, 65),
    ([63, 313, 3], 1, 235), ([3, 7, 16], 2, 70),
]


@pytest.mark.parametrize("dims,n,K", SHAPES)
@pytest.mark.parametrize("layout", ["rows", "columns", "strided"])
def test_ttm_layouts(tk, dims, n, K, layout):
    for ydt in (np.float64, np.float32):
        for zdt in (np.float64, np.float32):
            check(tk, dims, n, K, layout, ydt, zdt)
    # one element past an aligned address: 4-byte loads
    check(tk, dims, n, K, layout, np.float32, np.float64, offset=1)
    check(tk, dims, n, K, layout, np.float64, np.float64, offset=1)


def test_ttm_capture_odd_factor(tk):
    """A captured product whose factor is not in 16-byte units allocates nothing and replays."""
    rng = np.random.default_rng(0)
    y = torch.from_numpy(rng.standard_normal((30, 41, 12))).cuda()
    m = torch.from_numpy(rng.standard_normal((70, 41))).cuda()
    want = tk.ttm(y, 1, m)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        z = tk.ttm(y, 1, m)
    for s in (1.0, 2.0):
        y.mul_(s)
        g.replay()
        torch.cuda.synchronize()
        torch.testing.assert_close(z, s * want, rtol=1e-12, atol=1e-12)


# odd mode sizes and ranks: factors that are copied, a zero slice appended to
# an odd mode 0, ranges that begin at an odd row
@pytest.mark.parametrize("dims,ranks", [([131, 90, 77], [65, 67, 66]), ([200, 75, 101], [17, 66, 65])])
def test_odd_factors_whole_path(tk, orc, dims, ranks):
    rng = np.random.default_rng(5)
    X = rng.standard_normal(int(np.prod(dims)))
    x = torch.from_numpy(X.reshape(list(reversed(dims)))).cuda()
    for order in ([2, 0, 1], [0, 1, 2]):
        t = tk.sthosvd_ranks(x, ranks, mode_order=order)
        ref = orc.sthosvd(X, dims, 0.0, order, ranks=ranks)
        assert t.ranks == list(ref.ranks)
        full, _ = orc.reconstruct(ref, [0, 0, 0], dims)
        got = t.reconstruct().cpu().numpy().reshape(-1)
        assert np.abs(got - full).max() <= 1e-9 * np.abs(full).max()
        b, e = [1, 3, 5], dims
        part, _ = orc.reconstruct(ref, b, e)
        for dt, tol in ((torch.float64, 1e-9), (torch.float32, 1e-6)):
            got = t.reconstruct(b, e, out_dtype=dt).cpu().numpy().reshape(-1)
            assert np.abs(got - part).max() <= tol * np.abs(part).max()
        t.free()


# small products on slabs of pairs of columns: one and two blocks of reduction
# rows (whole, ragged, one row), one to four blocks of output rows, fewer
# columns than a wave's tile, a column count that ends inside one, several
# tiles per wave; odd slabs and unaligned bases take the other kernel
@pytest.mark.parametrize("dims,n,K", [
    ([2, 1, 3], 1, 1), ([2, 16, 5], 1, 16), ([6, 17, 40], 1, 17), ([34, 12, 3], 1, 50), ([64, 32], 1, 64),
    ([30, 5, 11, 7], 2, 33), ([1000, 31, 3], 1, 48), ([3, 12, 20], 1, 50), ([700, 4, 400], 1, 10),
])
def test_ttm_small_slabs(tk, dims, n, K):
    for ydt in (np.float64, np.float32):
        for zdt in (np.float64, np.float32):
            for fp32 in (False, True):
                check(tk, dims, n, K, "columns", ydt, zdt, fp32=fp32)
            check(tk, dims, n, K, "rows", ydt, zdt, offset=1)


def test_ttm_small_slabs_infinity(tk):
    """A row past J is not multiplied in: an infinity stays in its own column."""
    y = torch.zeros((3, 5, 8), dtype=torch.float64, device="cuda")
    y[1, 4, 3] = float("inf")
    z = tk.ttm(y, 1, torch.ones((7, 5), dtype=torch.float64, device="cuda"))
    want = torch.zeros((3, 7, 8), dtype=torch.float64)
    want[1, :, 3] = float("inf")
    assert torch.equal(z.cpu(), want)


def test_ttm_without_scratch(tk):
    """A factor that would be laid out again is read as it is where no memory is given."""
    import ctypes
    alloc, free = (f[1] for f in tk._Allocator._fields_[:2])
    none = tk._Allocator(alloc(lambda nbytes, ctx, stream: None), free(lambda p, ctx, stream: None), None)
    assert tk.lib().tucker_set_allocator(ctypes.byref(none)) == 0
    try:
        check(tk, [33, 50, 7], 1, 71, "columns", np.float64, np.float64, offset=1)
        check(tk, [33, 51, 7], 0, 71, "rows", np.float32, np.float64)
    finally:
        assert tk.lib().tucker_set_allocator(None) == 0


# past 1e9 flops the factor is laid out first where it is not in 16-byte units:
# slabs and unit stride, every layout, and no memory for the copy
@pytest.mark.parametrize("dims,n,K", [([66, 201, 700], 1, 71), ([201, 46200], 0, 71), ([65, 201, 711], 1, 71)])
def test_ttm_factor_laid_out(tk, dims, n, K):
    import ctypes
    check(tk, dims, n, K, "columns", np.float64, np.float32)
    check(tk, dims, n, K, "rows", np.float32, np.float64)
    check(tk, dims, n, K, "strided", np.float64, np.float64)
    alloc, free = (f[1] for f in tk._Allocator._fields_[:2])
    none = tk._Allocator(alloc(lambda nbytes, ctx, stream: None), free(lambda p, ctx, stream: None), None)
    assert tk.lib().tucker_set_allocator(ctypes.byref(none)) == 0
    try:
        check(tk, dims, n, K, "columns", np.float64, np.float64)
    finally:
        assert tk.lib().tucker_set_allocator(None) == 0


# around the number of tiles (128), of rows (two chunks) and of columns (1000)
# at which float tensors and laid-out factors go to the direct-load kernel
@pytest.mark.parametrize("dims,n,K", [
    ([128, 32, 128], 1, 65), ([128, 33, 128], 1, 65), ([128, 33, 129], 1, 65), ([63, 34, 128], 1, 200),
    ([63, 34, 131], 1, 200), ([251, 999], 0, 2049), ([251, 1000], 0, 2049), ([251, 7937], 0, 257),
])
def test_ttm_few_tiles(tk, dims, n, K):
    for zdt in (np.float64, np.float32):
        check(tk, dims, n, K, "rows", np.float32, zdt)
    check(tk, dims, n, K, "columns", np.float32, np.float64)
    check(tk, dims, n, K, "columns", np.float64, np.float64)


def raw_ttm(tk, y, M, z, stream):
    """Mode 0 of y (cols x J) into z without an allocation on the way."""
    st = tk.lib().tucker_ttm(y.data_ptr(), tk.F64, tk._i64([y.shape[1], y.shape[0]]), 2, 0, M.data_ptr(), M.shape[0],
                             M.stride(0), M.stride(1), z.data_ptr(), tk.F64, 0, int(stream.cuda_stream))
    assert st == 0


def laid_out_operands():
    g = torch.Generator(device="cuda").manual_seed(4)
    y = torch.randn(40000, 201, dtype=torch.float64, device="cuda", generator=g)
    M = torch.randn(71, 201, dtype=torch.float64, device="cuda", generator=g)
    z = torch.zeros(40000, 71, dtype=torch.float64, device="cuda")
    return y, M, z, y @ M.t(), 1e-12 * (y.abs() @ M.abs().t())


def test_ttm_beside_a_capture(tk):
    """A product that wants scratch, on a stream that has none, while another
    stream is being captured: it runs, and the capture stays valid."""
    y, M, z, ref, tol = laid_out_operands()
    x = torch.ones(1000, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = x * 2.0
        raw_ttm(tk, y, M, z, side)
        out = out + 1.0
    side.synchronize()
    assert bool(((z - ref).abs() <= tol).all())
    for v in (1.0, 5.0):
        x.fill_(v)
        g.replay()
        torch.cuda.synchronize()
        assert bool((out == 2.0 * v + 1.0).all())


def test_ttm_on_a_full_device_waits_for_nothing(tk):
    """Scratch that is not at hand is done without: no idle block is given back
    and other streams are not waited for."""
    y, M, z, ref, tol = laid_out_operands()
    busy = torch.randn(8192, 8192, device="cuda")
    busy @ busy
    tk.gram(y, 0)  # leaves idle blocks in the pool
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    out = torch.empty_like(busy)
    filler = torch.empty(torch.cuda.mem_get_info()[0] - (1 << 29), dtype=torch.uint8, device="cuda")
    try:
        with torch.cuda.stream(sa):
            for _ in range(20):
                torch.mm(busy, busy, out=out)
        raw_ttm(tk, y, M, z, sb)
        assert not sa.query()
        sb.synchronize()
        assert bool(((z - ref).abs() <= tol).all())
    finally:
        torch.cuda.synchronize()
        del filler
        torch.cuda.empty_cache()


# what ttm_slab_kernel takes: an even slab of at least 64 columns, enough words
# read and written (slab_words); one and two reduction blocks, whole, ragged and
# of one row; one to four row blocks, whole and ragged; rows of Z in whole
# 64-byte pieces and not; tiles that straddle slabs and a last one that the
# columns do not fill
SLABS = [
    (64, 20500, 1, 1), (64, 4097, 16, 16), (66, 3973, 5, 17), (96, 2731, 12, 50), (98, 2675, 16, 33),
    (1024, 257, 4, 64), (100, 3000, 7, 2), (202, 1299, 12, 51),
    (64, 8193, 17, 16), (66, 7945, 31, 32), (96, 5462, 32, 33), (1000, 525, 20, 50), (200, 2622, 32, 63),
    (66, 7945, 17, 64), (80, 8300, 24, 5), (64, 8193, 32, 64),
    (64, 4097, 8, 32), (64, 4097, 11, 48), (128, 2049, 17, 32),
]


def slab_words(J):
    return max(5 << 19, J * J << 15)  # for FP32 products to floats, the most of all


def slab_check(tk, L, R, J, K, ydt, zdt, fp32, layout, zoff=0):
    g = torch.Generator(device="cuda").manual_seed(L + J + K)
    y = torch.randn(R, J, L, dtype=torch.float64, device="cuda", generator=g).to(ydt)
    M = torch.randn(K, J, dtype=torch.float64, device="cuda", generator=g)
    m = M if layout == "rows" else M.t().contiguous().t()
    buf = torch.full((R * K * L + 2 * zoff,), 7.0, dtype=zdt, device="cuda")
    z = buf[zoff:zoff + R * K * L].view(R, K, L)
    code = {torch.float32: tk.F32, torch.float64: tk.F64}
    st = tk.lib().tucker_ttm(y.data_ptr(), code[ydt], tk._i64([L, J, R]), 3, 1, m.data_ptr(), K, m.stride(0),
                             m.stride(1), z.data_ptr(), code[zdt], int(fp32), tk._stream())
    assert st == 0
    cols = y.double().permute(1, 0, 2).reshape(J, R * L).contiguous()
    ref, mag = M @ cols, M.abs() @ cols.abs()
    tol = 1e-12 * mag
    if zdt == torch.float32:
        tol = tol + 2.0 ** -23 * ref.abs()
    if fp32:
        tol = tol + (J + 2) * 2.0 ** -23 * mag
    d = (z.double().permute(1, 0, 2).reshape(K, R * L) - ref).abs()
    assert bool((d <= tol).all()), (L, R, J, K, ydt, zdt, fp32, layout)
    assert bool((buf[:zoff] == 7.0).all()) and bool((buf[zoff + R * K * L:] == 7.0).all())


@pytest.mark.parametrize("L,R,J,K", SLABS)
def test_ttm_slab_kernel(tk, L, R, J, K):
    assert L * R * (J + K) >= slab_words(J) and J <= 8 * K
    f32, f64 = torch.float32, torch.float64
    for ydt, zdt, fp32 in ((f64, f64, False), (f64, f32, False), (f32, f64, False), (f32, f32, False),
                           (f32, f32, True), (f64, f64, True)):
        slab_check(tk, L, R, J, K, ydt, zdt, fp32, "columns")
    slab_check(tk, L, R, J, K, f32, f64, False, "rows")
    # Z past a 64-byte boundary
    slab_check(tk, L, R, J, K, f64, f64, False, "columns", zoff=2)
    slab_check(tk, L, R, J, K, f32, f32, True, "columns", zoff=2)


@pytest.mark.parametrize("L,R,J", [(64, 4097, 5), (66, 4500, 13), (96, 5462, 21), (66, 12200, 30)])
@pytest.mark.parametrize("fp32", [False, True])
def test_ttm_slab_infinity(tk, L, R, J, fp32):
    """Rows past J, which hold a repeated row, are not multiplied in: an
    infinity in the last row stays in its own column."""
    assert L * R * (J + 7) >= slab_words(J)
    dt = torch.float32 if fp32 else torch.float64
    y = torch.zeros((R, J, L), dtype=dt, device="cuda")
    y[1, J - 1, 3] = float("inf")
    y[R - 1, J - 1, L - 1] = float("-inf")
    z = tk.ttm(y, 1, torch.ones((7, J), dtype=torch.float64, device="cuda"), fp32_products=fp32)
    want = torch.zeros((R, 7, L), dtype=dt, device="cuda")
    want[1, :, 3] = float("inf")
    want[R - 1, :, L - 1] = float("-inf")
    assert torch.equal(z, want)


def test_ttm_captured_with_a_factor_to_lay_out(tk):
    """A captured product that would lay its factor out takes no scratch, and
    replays on new data."""
    y, M, z, ref, tol = laid_out_operands()
    side = torch.cuda.Stream()
    raw_ttm(tk, y, M, z, side)  # leaves an idle block that fits in the pool of this stream
    torch.cuda.synchronize()
    assert bool(((z - ref).abs() <= tol).all())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        raw_ttm(tk, y, M, z, side)
    for s in (1.0, -2.0, 3.0):
        z.zero_()
        y.mul_(s)
        ref, tol = ref * s, tol * abs(s)
        g.replay()
        junk = torch.randn(1 << 20, device="cuda").sum()
        torch.cuda.synchronize()
        assert bool(((z - ref).abs() <= tol).all())
        del junk


# products past 1e9 flops whose factor is in odd rows: of an odd mode while the
# eigensolver's workspace, which takes the copy, is used again by the modes after
# it; of an odd mode at full rank, applied last; and of row ranges that begin at
# an odd row or have an odd stride, in reconstructions
@pytest.mark.parametrize("dims,ranks,order", [
    ([131, 240, 241], [67, 40, 41], [0, 1, 2]),
    ([240, 131, 241], [40, 67, 41], [1, 2, 0]),
    ([201, 150, 160], [201, 112, 111], [0, 1, 2]),
    ([150, 201, 160], [113, 201, 112], [1, 0, 2]),
])
def test_laid_out_factors_whole_path(tk, orc, dims, ranks, order):
    rng = np.random.default_rng(sum(dims))
    X = rng.standard_normal(int(np.prod(dims)))
    x = torch.from_numpy(X.reshape(list(reversed(dims)))).cuda()
    t = tk.sthosvd_ranks(x, ranks, mode_order=order)
    ref = orc.sthosvd(X, dims, 0.0, order, ranks=ranks)
    assert t.ranks == list(ref.ranks)
    np.testing.assert_allclose(t.discarded, ref.discarded, rtol=1e-9, atol=1e-12 * float(np.dot(X, X)))
    full, _ = orc.reconstruct(ref, [0, 0, 0], dims)
    got = t.reconstruct().cpu().numpy().reshape(-1)
    assert np.abs(got - full).max() <= 1e-9 * np.abs(full).max()
    b, e = [1, 1, 1], dims
    part, _ = orc.reconstruct(ref, b, e)
    for o in (None, [2, 1, 0], [1, 2, 0]):
        got = t.reconstruct(b, e, order=o).cpu().numpy().reshape(-1)
        assert np.abs(got - part).max() <= 1e-9 * np.abs(part).max()
    t.free()
