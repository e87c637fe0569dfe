"""Split products of the grouped GEMMs (fp32 operands as scaled sums of two fp16 terms) where
they can go wrong: short and odd contractions, rows and columns of very different magnitude,
growth past the scale of the first values, values below all that the scale holds, zeros, infinities
and NaN; against float64.

Per entry, |error| <= (K + 8) 2^-24 sum |a b|.  The split leaves out up to 2^-23 of each operand and 2^-22
of each product, 8 of the 2^-24 together, and at the low end up to 8 more; the sum has at most K / 8
roundings (two accumulators, 16 products an instruction)."""
import numpy as np
import pytest

from helpers import banner

pytestmark = pytest.mark.gpu

# tiles of 64 rows (few tiles) and of 128 (more than 256 workgroups)
SIZES = {"few": [130, 0, 7], "many": [33_000, 0, 61]}


@pytest.fixture(scope="module")
def ctx():
    from paper_2604_15821_amd import janus
    from paper_2604_15821_amd.synth import WORKLOADS
    c = janus.Context(WORKLOADS["tiny"].model)
    yield c
    c.close()


def _values(kind, rng, shape, k_axis):
    x = rng.standard_normal(shape)
    K = shape[k_axis]
    k = np.arange(K).reshape([-1 if a == k_axis % x.ndim else 1 for a in range(x.ndim)])
    if kind == "magnitudes":       # per row (column), 2^-40 .. 2^39
        s = list(shape)
        s[k_axis] = 1
        x = np.ldexp(x, rng.integers(-40, 40, s))
    elif kind == "growth":         # later values 2^16 times the first ones
        x = np.where(k >= 32, np.ldexp(x, 16), x)
    elif kind == "fits":           # later values up to 2^14 (row products 2^6) times the largest of the first 32
        m = np.abs(np.where(k < 32, x, 0.0)).max(axis=k_axis, keepdims=True)
        x = np.where(k >= 32, np.clip(x, -1.0, 1.0) * np.ldexp(m, 14 if k_axis == 0 else 6), x)
    elif kind == "decay":          # later values 2^-16 of the first ones
        x = np.where(k >= 32, np.ldexp(x, -16), x)
    elif kind == "late":           # zeros in the first 32
        x = np.where(k >= 32, x, 0.0)
    elif kind == "zeros":
        x = np.zeros(shape)
    return x.astype(np.float32)


def _run(ctx, A, B, off, trans_b):
    import torch
    K, N = A.shape[1], B.shape[1 if trans_b else 2]
    out = torch.full((A.shape[0], N), 7.0, device="cuda:0")
    ctx.grouped_gemm(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), torch.from_numpy(off).cuda(), K, N,
                     trans_b, out=out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


# kinds that change values after the first 32 need more than 32 of them; "growth" overflows the scale, so the
# pairs with it take the fp32 pass, "decay" with anything else the split
_WHOLE = [("normal", "normal"), ("magnitudes", "magnitudes"), ("zeros", "normal")]
_AFTER_32 = [("growth", "decay"), ("decay", "growth"), ("decay", "normal"), ("normal", "decay"), ("decay", "fits"),
             ("fits", "normal"), ("late", "normal"), ("normal", "late")]
_ROWS = [(K, N, size, a, b) for K, N in [(16, 64), (32, 64), (48, 192), (64, 128), (224, 320)]
         for size in (["few", "many"] if K in (32, 64) else ["few"])
         for a, b in _WHOLE + (_AFTER_32 if K > 32 else [])]


@pytest.mark.parametrize("trans_b", [0, 1])
@pytest.mark.parametrize("K,N,size,kind_a,kind_b", _ROWS)
def test_rows(ctx, K, N, trans_b, kind_a, kind_b, size):
    banner("split rows", K, N, trans_b, kind_a, kind_b, size)
    rng = np.random.default_rng(K + N + trans_b)
    sizes = SIZES[size]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    A = _values(kind_a, rng, (int(off[-1]), K), 1)
    B = _values(kind_b, rng, (len(sizes), N, K) if trans_b else (len(sizes), K, N), 2 if trans_b else 1)
    got = _run(ctx, A, B, off, trans_b)
    for g in range(len(sizes)):
        a = A[off[g]:off[g + 1]].astype(np.float64)
        b = (B[g].T if trans_b else B[g]).astype(np.float64)
        bound = (K + 8) * 2.0 ** -24 * (np.abs(a) @ np.abs(b)) + 1e-45
        assert (np.abs(got[off[g]:off[g + 1]] - a @ b) <= bound).all(), g


@pytest.mark.parametrize("rows", [5, 16, 33, 700])
@pytest.mark.parametrize("kind_a,kind_b", [("normal", "normal"), ("magnitudes", "normal"), ("growth", "decay"),
                                           ("decay", "normal"), ("normal", "decay"), ("decay", "fits"),
                                           ("fits", "normal"), ("late", "normal"), ("normal", "zeros")])
def test_wgrad(ctx, rows, kind_a, kind_b):
    import torch
    banner("split wgrad", rows, kind_a, kind_b)
    rng = np.random.default_rng(rows)
    off = np.array([0, rows, rows, rows + 3], np.int32)
    A = _values(kind_a, rng, (rows + 3, 192), 0)
    B = _values(kind_b, rng, (rows + 3, 64), 0)
    got = ctx.grouped_wgrad(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), torch.from_numpy(off).cuda())
    got = got.cpu().numpy()
    for g in range(3):
        a, b = (x[off[g]:off[g + 1]].astype(np.float64) for x in (A, B))
        bound = (rows + 8) * 2.0 ** -24 * (np.abs(a).T @ np.abs(b)) + 1e-45
        assert (np.abs(got[g] - a.T @ b) <= bound).all(), g


def _mask(big, zero, e, where, line):
    """Contraction index 5 times 2^e in `big` (first axis the contraction) and zero in `zero`: what is left of
    the result comes from values 2^e below the one that sets the scale.  "entry": one line of each only."""
    at = line if where == "entry" else slice(None)
    big[5, 18 if where == "entry" else slice(None)] *= np.float32(2.0 ** e)
    zero[5, at] = 0.0


# from below the range that the split holds in full to beyond all that it holds
_MASKS = [8, 12, 14, 16, 20, 24, 30, 38, 100]


@pytest.mark.parametrize("size", ["few", "many"])
@pytest.mark.parametrize("trans_b", [0, 1])
@pytest.mark.parametrize("where", ["a", "b", "entry"])
@pytest.mark.parametrize("e", _MASKS)
def test_rows_whose_largest_value_meets_zero(ctx, e, where, trans_b, size):
    banner("split masked rows", e, where, trans_b, size)
    rng = np.random.default_rng(e)
    K, N = 64, 192
    off = np.concatenate([[0], np.cumsum(SIZES[size])]).astype(np.int32)
    A = rng.standard_normal((int(off[-1]), K)).astype(np.float32)
    A[3::7] = 0.0   # rows of zeros beside them
    B = rng.standard_normal((3, K, N)).astype(np.float32)
    for g in range(3):
        a = A[off[g]:off[g + 1]].T
        if where == "b":
            _mask(B[g], a, e, where, 0)
        elif a.shape[1] > 18 or where == "a":
            _mask(a, B[g], e, where, 130)
    got = _run(ctx, A, np.ascontiguousarray(B.transpose(0, 2, 1)) if trans_b else B, off, trans_b)
    for g in range(3):
        a, b = A[off[g]:off[g + 1]].astype(np.float64), B[g].astype(np.float64)
        bound = (K + 8) * 2.0 ** -24 * (np.abs(a) @ np.abs(b)) + 1e-45
        assert (np.abs(got[off[g]:off[g + 1]] - a @ b) <= bound).all(), g


@pytest.mark.parametrize("rows", [20, 700])
@pytest.mark.parametrize("where", ["a", "b", "entry"])
@pytest.mark.parametrize("e", _MASKS)
def test_wgrad_whose_largest_row_meets_zero(ctx, e, where, rows):
    import torch
    banner("split masked wgrad", e, where, rows)
    rng = np.random.default_rng(e + rows)
    off = np.array([0, rows, rows, rows + 40], np.int32)
    A = rng.standard_normal((rows + 40, 192)).astype(np.float32)
    B = rng.standard_normal((rows + 40, 64)).astype(np.float32)
    A[:, 3::7] = 0.0
    for g in (0, 2):
        a, b = A[off[g]:off[g + 1]], B[off[g]:off[g + 1]]
        _mask(*((b, a) if where == "b" else (a, b)), e, where, 40)
    got = ctx.grouped_wgrad(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), torch.from_numpy(off).cuda())
    got = got.cpu().numpy()
    for g in range(3):
        a, b = (x[off[g]:off[g + 1]].astype(np.float64) for x in (A, B))
        bound = (a.shape[0] + 8) * 2.0 ** -24 * (np.abs(a).T @ np.abs(b)) + 1e-45
        assert (np.abs(got[g] - a.T @ b) <= bound).all(), g


def _check_nonfinite(got, a, b):
    """a [m, K], b [K, n] in float64, K at most 96 + 8: as float32, infinities and NaN where a b has them."""
    with np.errstate(all="ignore"):
        ref = a @ b
        ref32 = ref.astype(np.float32)
        bound = (a.shape[1] + 8) * 2.0 ** -24 * (np.abs(a) @ np.abs(b))
    fin = np.isfinite(ref32)
    assert (np.isnan(got) == np.isnan(ref32)).all()
    assert (got[np.isinf(ref32)] == ref32[np.isinf(ref32)]).all()
    assert (np.abs(got[fin] - ref[fin]) <= bound[fin]).all()


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 3.4e38])
def test_infinities_and_nan_of_the_transposed_product_and_the_weight_gradient(ctx, bad):
    import torch
    banner("split non-finite, NT and weight gradient", bad)
    rng = np.random.default_rng(2)
    off = np.array([0, 200], np.int32)
    A = rng.standard_normal((200, 96)).astype(np.float32)
    B = rng.standard_normal((1, 128, 96)).astype(np.float32) * np.float32(0.01)
    A[17, 50] = bad
    B[0, 70, 3] = bad
    _check_nonfinite(_run(ctx, A, B, off, 1), A.astype(np.float64), B[0].T.astype(np.float64))
    X = rng.standard_normal((200, 192)).astype(np.float32) * np.float32(0.01)
    X[150, 130] = bad
    got = ctx.grouped_wgrad(torch.from_numpy(A).cuda(), torch.from_numpy(X).cuda(), torch.from_numpy(off).cuda())
    _check_nonfinite(got.cpu().numpy()[0], A.T.astype(np.float64), X.astype(np.float64))


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("rows", [200, 33_000])
def test_infinities_and_nan_stay_in_their_rows_and_columns(ctx, bad, rows):
    banner("split non-finite", bad, rows)
    rng = np.random.default_rng(1)
    off = np.array([0, rows], np.int32)
    A = rng.standard_normal((rows, 96)).astype(np.float32)
    B = rng.standard_normal((1, 96, 128)).astype(np.float32) * np.float32(0.01)
    A[17, 50] = bad
    B[0, 3, 70] = bad
    got = _run(ctx, A, B, off, 0)
    with np.errstate(all="ignore"):
        ref = A.astype(np.float64) @ B[0].astype(np.float64)
        ref32 = ref.astype(np.float32)
    fin = np.isfinite(ref32)
    assert (np.isnan(got) == np.isnan(ref32)).all()
    assert (got[np.isinf(ref32)] == ref32[np.isinf(ref32)]).all()
    bound = 104 * 2.0 ** -24 * (np.abs(A[:, :]).astype(np.float64) @ np.abs(B[0]).astype(np.float64))
    assert (np.abs(got[fin] - ref[fin]) <= bound[fin]).all()


def _ranges(rng, rows, K):
    """Rows over K with a random spread of magnitudes, signs and zeros."""
    kind = rng.integers(4)
    lo, hi = -45.0 * rng.random(), 12.0 * rng.random()
    e = np.floor(lo + (hi - lo) * rng.random((rows, K)))
    if kind == 1:
        e *= rng.random((1, K)) < 0.5
    elif kind == 2:
        e.sort(axis=1)
    elif kind == 3:
        e = np.where(rng.random((rows, K)) < 0.02, e + 20.0, lo // 1.0)
    x = np.ldexp((1.0 + rng.random((rows, K))) * rng.choice([-1.0, 1.0], (rows, K)), e.astype(int))
    if rng.random() < 0.6:
        x *= rng.random((rows, K)) < rng.random()
    if rng.random() < 0.3:
        x *= rng.random((rows, 1)) < 0.8
    return x


def _meet_zeros(rng, A, B):
    """Some of the contraction 2^e times as large in A and zero in B."""
    if rng.random() < 0.5:
        at = rng.random(A.shape[1]) < 0.3
        A[:, at] *= 2.0 ** rng.integers(40)
        B[:, at] = 0.0
    return A.astype(np.float32), B.astype(np.float32)


@pytest.mark.parametrize("seed", range(40))
def test_random_ranges(ctx, seed):
    import torch
    banner("split random ranges", seed)
    rng = np.random.default_rng(seed)
    K, M, N = int(rng.choice([32, 64, 96, 128, 256, 512])), int(rng.integers(1, 300)), 64 * int(rng.integers(1, 4))
    A, B = _meet_zeros(rng, _ranges(rng, M, K), _ranges(rng, N, K))
    a, b = A.astype(np.float64), B.astype(np.float64)
    bound = 2.0 ** -24 * (np.abs(a) @ np.abs(b).T)
    off = np.array([0, M], np.int32)
    for trans_b in (0, 1):
        got = _run(ctx, A, B[None] if trans_b else np.ascontiguousarray(B.T)[None], off, trans_b)
        assert (np.abs(got - a @ b.T) <= (K + 8) * bound + 1e-45).all(), trans_b
    rows, P = int(rng.integers(1, 1500)), 64 * int(rng.integers(1, 4))
    A, B = _meet_zeros(rng, _ranges(rng, P, rows), _ranges(rng, N, rows))
    got = ctx.grouped_wgrad(torch.from_numpy(np.ascontiguousarray(A.T)).cuda(),
                            torch.from_numpy(np.ascontiguousarray(B.T)).cuda(),
                            torch.tensor([0, rows], dtype=torch.int32, device="cuda:0")).cpu().numpy()[0]
    a, b = A.astype(np.float64), B.astype(np.float64)
    assert (np.abs(got - a @ b.T) <= (rows + 8) * 2.0 ** -24 * (np.abs(a) @ np.abs(b).T) + 1e-45).all()
