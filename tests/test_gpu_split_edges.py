"""GPU kernels at the edges of the splits that their launches choose: workgroup
counts, remainders, aligned and unaligned loads, against the FP64 CPU oracle.

Tolerances: sums of n values in FP64 in another order differ by at most about
n u sum|x|, taken as 1e-12 (statistics) and 1e-11 sqrt(S_aa S_bb) (Grams), as in
the parity tests.
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


def to_dev(x, dims, dtype):
    return torch.from_numpy(np.ascontiguousarray(x).reshape(list(reversed(dims)))).to("cuda", dtype)


# columns of the mode: one group of 16, a group and a column, one workgroup's
# four groups and their neighbours, around 256 workgroups of four groups, and
# past 8192 groups, where the waves take several groups each
@pytest.mark.parametrize("J", [1, 16, 17, 33, 61, 64])
@pytest.mark.parametrize("cols", [1, 16, 17, 63, 64, 65, 16383, 16385, 131073])
def test_small_mode_gram_splits(tk, orc, J, cols):
    rng = np.random.default_rng(J * 1000 + cols)
    for dims, n in (([J, cols], 0), ([cols, J], 1), ([3, J, -(-cols // 3)], 1)):
        X = rng.standard_normal(int(np.prod(dims)))
        S, nrm = tk.gram(to_dev(X, dims, torch.float64), n, dims=dims, with_norm=True)
        ref = orc.gram(X, dims, n)
        d = np.sqrt(np.outer(np.diag(ref), np.diag(ref)))
        assert np.all(np.abs(S.cpu().numpy() - ref) <= 1e-11 * d), (dims, n)
        assert abs(float(nrm[0]) - np.dot(X, X)) <= 1e-12 * np.dot(X, X)


# row mapping with 16-byte and scalar loads, ragged batches of 16; period
# mapping with 1 .. 512 periods per group, incomplete groups and batches
@pytest.mark.parametrize("dims,n", [
    ([64, 5, 3], 1), ([66, 5, 3], 1), ([65, 3, 31], 1), ([4096, 2, 9], 1), ([128, 40], 1), ([1500, 3], 0),
    ([2, 4100], 0), ([2, 4097], 0), ([7, 1000], 0), ([1, 8, 999], 1), ([3, 5, 70], 1), ([31, 33, 10], 1),
    ([513, 77], 0), ([1024, 17], 0), ([2, 1], 0),
])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("offset", [0, 1])
def test_slice_stats_edges(tk, orc, dims, n, dtype, offset):
    rng = np.random.default_rng(sum(dims) + n)
    size = int(np.prod(dims))
    X = (rng.standard_normal(size) * 2.0 + 1.0e3).astype(dtype)
    tdt = torch.float64 if dtype == np.float64 else torch.float32
    buf = torch.empty(size + offset, dtype=tdt, device="cuda")
    buf[offset:] = torch.from_numpy(X)
    st = tk.slice_stats(buf[offset:], n, dims=dims).cpu().numpy()
    ref = orc.slice_stats(X.astype(np.float64), dims, n)
    cnt = size // dims[n]
    np.testing.assert_array_equal(st[2:4], ref[2:4])
    assert np.all(np.abs(st[0] - ref[0]) <= 1e-12 * ref[4] / cnt)
    assert np.all(np.abs(st[1] - ref[1]) <= 1e-12 * ref[5] / np.sqrt(cnt))
    np.testing.assert_allclose(st[4:], ref[4:], rtol=1e-12)


@pytest.mark.parametrize("dims,n", [([4, 3, 700], 1), ([640, 3, 5], 1)])
def test_slice_stats_special_values(tk, dims, n):
    """A constant slice has no deviation; one infinity or NaN stays in its slice."""
    size = int(np.prod(dims))
    rng = np.random.default_rng(3)
    X = rng.standard_normal(size).reshape(list(reversed(dims)))
    v = np.moveaxis(X, len(dims) - 1 - n, 0)
    v[0] = 0.1
    v[1].flat[7] = np.inf
    st = tk.slice_stats(to_dev(X.reshape(-1), dims, torch.float64), n, dims=dims).cpu().numpy()
    assert st[1][0] <= 1e-15 and st[2][0] == st[3][0] == 0.1
    assert st[0][1] == np.inf and np.isnan(st[1][1]) and st[3][1] == np.inf and st[5][1] == np.inf
    np.testing.assert_allclose(st[1][2], v[2].std(), rtol=1e-12)
    v[1].flat[7] = np.nan
    st = tk.slice_stats(to_dev(X.reshape(-1), dims, torch.float64), n, dims=dims).cpu().numpy()
    assert np.isnan(st[0][1]) and np.isnan(st[1][1]) and np.isfinite(st[3][1])


# tile pairs with direct loads: one to four row tiles, the last whole, ragged or
# of one row; unit stride and row segments, 16-byte and 4-byte loads, chunks cut
# by the end of a slab or of the tensor, fewer columns than a chunk
@pytest.mark.parametrize("J", [129, 161, 249, 256, 257, 313, 400])
@pytest.mark.parametrize("L,rest", [(1, 7), (1, 333), (64, 3), (65, 4), (66, 1), (90, 5), (128, 2)])
def test_tile_pair_gram_edges(tk, orc, J, L, rest):
    rng = np.random.default_rng(J * 100 + L)
    dims, n = ([J, rest], 0) if L == 1 else ([L, J, rest], 1)
    X = rng.standard_normal(int(np.prod(dims))).astype(np.float32).astype(np.float64)
    ref = orc.gram(X, dims, n)
    d = np.sqrt(np.outer(np.diag(ref), np.diag(ref)))
    for dt, prec, tol in ((torch.float64, "fp64", 1e-11), (torch.float32, "fp64", 1e-11),
                          (torch.float32, "fp32", 2.4e-6), (torch.float32, "bf16x6", 1.2e-5)):
        if prec == "fp64" and J <= 240:
            continue  # the whole triangle per workgroup
        for offset in (0, 1):
            buf = torch.empty(X.size + offset, dtype=dt, device="cuda")
            buf[offset:] = torch.from_numpy(X)
            S, nrm = tk.gram(buf[offset:], n, prec=prec, dims=dims, with_norm=True)
            assert np.all(np.abs(S.cpu().numpy() - ref) <= tol * d), (dims, prec, offset)
            assert abs(float(nrm[0]) - np.dot(X, X)) <= 1e-12 * np.dot(X, X)


def _tri_case(kind, J):
    """Symmetric matrices that are hard for counting eigenvalues by minors."""
    rng = np.random.default_rng(J)
    S = np.zeros((J, J))
    if kind == "integer":  # diagonal, exactly hit, many equal
        S = np.diag(rng.integers(0, 4, J).astype(float))
    elif kind == "blocks":  # decoupled, the same pair of eigenvalues in each
        for i in range(0, J - 1, 2):
            S[i:i + 2, i:i + 2] = [[2.0, 1.0], [1.0, 2.0]]
    elif kind == "toeplitz":  # tridiagonal already, minors that vanish exactly
        S = 2.0 * np.eye(J) + np.eye(J, k=1) + np.eye(J, k=-1)
    elif kind in ("graded", "tiny", "huge"):
        Q = np.linalg.qr(rng.standard_normal((J, J)))[0]
        S = (Q * 10.0 ** np.linspace(0, -18, J)) @ Q.T
        S = 0.5 * (S + S.T) * {"graded": 1.0, "tiny": 1e-90, "huge": 1e90}[kind]
    return S


# rows in groups of 8 and their neighbours, one and several rounds of 64 tails
@pytest.mark.parametrize("J", [1, 2, 7, 8, 9, 63, 64, 65, 128, 129, 200])
@pytest.mark.parametrize("kind", ["zero", "integer", "blocks", "toeplitz", "graded", "tiny", "huge"])
def test_eigenvalue_counts_and_truncation(tk, orc, J, kind):
    S = _tri_case(kind, J)
    ref = np.linalg.eigvalsh(S)[::-1]
    nS = np.abs(ref).max()
    tail = np.concatenate([np.cumsum(np.clip(ref, 0, None)[::-1])[::-1], [0.0]])
    for R0 in sorted({1, 2, J // 2 + 1, J}):
        if R0 > J:
            continue
        thr = 0.5 * (tail[R0] + tail[R0 - 1])
        lam, U, R, disc = tk.eig_truncate(torch.from_numpy(S).cuda(), thr)
        lam = lam.cpu().numpy()
        assert np.abs(lam - ref).max() <= 1e-12 * nS
        assert R >= 1 and tail[R] <= thr + 1e-12 * J * nS and (R == 1 or tail[R - 1] >= thr - 1e-12 * J * nS)
        assert abs(disc - tail[R]) <= 1e-12 * J * nS


@pytest.mark.parametrize("J", [1, 8, 63, 65, 128])
def test_eigenvalue_counts_in_a_batch(tk, J):
    """Diagonal unfoldings: eigenvalues that the counts hit exactly, and none but zero."""
    d = (np.arange(J) % 4).astype(np.float32)
    xs = [to_dev(np.diag(d).reshape(-1), [J, J], torch.float32), to_dev(np.zeros(J * J), [J, J], torch.float32),
          to_dev(np.eye(J).reshape(-1), [J, J], torch.float32)]
    b = tk.Batch(xs, 1e-4, prec="fp64", dims=[[J, J]] * 3)
    b.run()
    nz = max(1, int(np.count_nonzero(d)))
    assert b.ranks() == [[nz, nz], [1, 1], [J, J]]


# one row short of, at and past the 160-row phase, and either side of the others
@pytest.mark.parametrize("J", [4, 31, 95, 127, 159, 160, 161, 191, 194, 225])
def test_tridiagonalisation_phase_edges(tk, J):
    """Eigenpairs of a full matrix with 17 zero rows and columns (tau = 0) for J > 31;
    residual within 1e-11 ||S||, orthogonality within 1e-11 (u over the gap of 1e-3 ||S||
    from which inverse iteration is left to itself)."""
    rng = np.random.default_rng(J)
    A = rng.standard_normal((J, J + 3))
    if J > 31:
        A[J // 2:J // 2 + 17] = 0.0
    S = A @ A.T
    lam, U, R, _ = tk.eig_truncate(torch.from_numpy(S).cuda(), 1e-13 * np.trace(S))
    lam, U = lam.cpu().numpy(), U.cpu().numpy()
    ref = np.linalg.eigvalsh(S)[::-1]
    assert np.abs(lam - ref).max() <= 1e-12 * ref[0]
    assert R == (J if J <= 31 else J - 17)
    assert np.abs(U.T @ U - np.eye(R)).max() <= 1e-11
    assert np.linalg.norm(S @ U - U * lam[:R], 2) <= 1e-11 * ref[0]


# double rows that are not 16-byte aligned, on both sides of the lines between
# the tile-pair kernels (two, three and four tiles)
@pytest.mark.parametrize("L,J", [(67, 250), (129, 250), (65, 384), (67, 384), (129, 384), (65, 300), (65, 512)])
def test_double_row_segments(tk, orc, L, J):
    dims = [L, J, 9]
    X = np.random.default_rng(L + J).standard_normal(int(np.prod(dims)))
    S, nrm = tk.gram(to_dev(X, dims, torch.float64), 1, dims=dims, with_norm=True)
    ref = orc.gram(X, dims, 1)
    d = np.sqrt(np.outer(np.diag(ref), np.diag(ref)))
    assert np.all(np.abs(S.cpu().numpy() - ref) <= 1e-11 * d)
    assert abs(float(nrm[0]) - np.dot(X, X)) <= 1e-12 * np.dot(X, X)


# slices in one piece, whose statistics the first kernel writes: many, and short
# ones; one wave and four per slice; both orders of merging a period's values
@pytest.mark.parametrize("dims,n", [
    ([66, 2500, 3], 1), ([5, 3000, 1], 1), ([1, 4100, 2], 1), ([64, 2048, 17], 1), ([65, 33, 15], 1), ([1025, 3], 1),
    ([7, 140, 3], 1), ([8, 128, 3], 1), ([63, 3, 3], 1), ([1, 1024, 2], 1),
])
def test_slice_stats_whole_slices(tk, orc, dims, n):
    rng = np.random.default_rng(sum(dims))
    X = rng.standard_normal(int(np.prod(dims))) * 2.0 + 1.0e3
    st = tk.slice_stats(to_dev(X, dims, torch.float64), n, dims=dims).cpu().numpy()
    ref = orc.slice_stats(X, dims, n)
    cnt = X.size // dims[n]
    np.testing.assert_array_equal(st[2:4], ref[2:4])
    assert np.all(np.abs(st[0] - ref[0]) <= 1e-12 * ref[4] / cnt)
    assert np.all(np.abs(st[1] - ref[1]) <= 1e-12 * ref[5] / np.sqrt(cnt))
    np.testing.assert_allclose(st[4:], ref[4:], rtol=1e-12)


# enough elements for four groups per thread and iteration: whole groups, groups
# that straddle slices, a last iteration and a last group that are not full
@pytest.mark.parametrize("dims", [[64, 33, 15903], [193, 33, 5311], [201, 7, 23999]])
@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
def test_slice_transform_large(tk, dims, dt):
    L, J, R = dims
    g = torch.Generator(device="cuda").manual_seed(L)
    x = torch.randn(R, J, L, device="cuda", dtype=dt, generator=g)
    sh = torch.randn(J, device="cuda", dtype=torch.float64, generator=g)
    sc = torch.rand(J, device="cuda", dtype=torch.float64, generator=g) + 0.5
    y = tk.slice_transform(x, 1, sh, sc, dims=dims)
    want = ((x.double() - sh[:, None]) / sc[:, None]).to(dt)
    assert torch.equal(y, want)
    back = tk.slice_transform(y, 1, sh, sc, dims=dims, inverse=True)
    assert bool(((back - x).abs() <= (2.0 ** -21 if dt == torch.float32 else 1e-14) * (x.abs() + 4.0)).all())


# what the direct-load tile pairs take beside 16-byte loads of FP64 and of unit
# stride: at least 1024 items, each of 16 chunks of 32 columns (16 of doubles), and
# a gain past the lines; unaligned columns, row segments and bases, slabs that end
# inside a chunk, last tiles of a few and of most rows
@pytest.mark.parametrize("J,L,rest,prec,dt", [
    (401, 1, 53000, "fp64", torch.float32), (401, 1, 26500, "fp64", torch.float64),
    (400, 1, 53000, "fp64", torch.float32), (400, 67, 570, "fp64", torch.float32),
    (400, 67, 335, "fp64", torch.float64), (500, 129, 340, "fp64", torch.float32),
    (401, 1, 53000, "fp32", torch.float32), (200, 447, 395, "fp32", torch.float32),
    (672, 256, 99, "fp32", torch.float32), (335, 96, 935, "fp32", torch.float32),
    (401, 1, 53000, "bf16x6", torch.float32), (200, 447, 395, "bf16x6", torch.float32),
    (200, 416, 425, "bf16x6", torch.float32),
])
def test_tile_pair_gram_many_items(tk, J, L, rest, prec, dt):
    dims, n = ([J, rest], 0) if L == 1 else ([L, J, rest], 1)
    tol = {"fp64": 1e-11, "fp32": 2.4e-6, "bf16x6": 1.2e-5}[prec]
    g = torch.Generator(device="cuda").manual_seed(J + L)
    buf = torch.randn(J * L * rest + 1, device="cuda", dtype=dt, generator=g)
    for offset in (0, 1):
        y = buf[offset:offset + J * L * rest]
        S, nrm = tk.gram(y, n, prec=prec, dims=dims, with_norm=True)
        A = y.view(rest, J, L).double().permute(1, 0, 2).reshape(J, rest * L).contiguous()
        ref = A @ A.t()
        d = torch.sqrt(torch.outer(ref.diagonal(), ref.diagonal()))
        assert bool(((S - ref).abs() <= tol * d).all()), offset
        n2 = float((A * A).sum())
        assert abs(float(nrm[0]) - n2) <= 1e-12 * n2
