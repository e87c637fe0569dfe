"""Split products of the grouped GEMMs (fp32 operands as scaled sums of two fp16 terms) where
they can go wrong: short and odd contractions, rows and columns of very different magnitude,
growth past the scale of the first values, zeros, infinities and NaN; against float64.

Per entry, |error| <= (K + 8) 2^-24 sum |a b|: the K roundings of an fp32 sum, and the terms
the split leaves out (below 2^-23 of each product)."""
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
    if kind == "magnitudes":       # per row, 2^-100 .. 2^100
        s = list(shape)
        s[k_axis] = 1
        x = np.ldexp(x, rng.integers(-40, 40, s))
    elif kind == "growth":         # later values 2^16 times the first ones
        x = np.where(k >= 32, np.ldexp(x, 16), x)
    elif kind == "fits":           # later values up to just under 2^15 times the largest of the first 32
        m = np.abs(np.where(k < 32, x, 0.0)).max(axis=k_axis, keepdims=True)
        x = np.where(k >= 32, np.clip(x, -1.0, 1.0) * np.ldexp(m, 14), x)
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


@pytest.mark.parametrize("K,N", [(16, 64), (32, 64), (48, 192), (64, 128), (224, 320)])
@pytest.mark.parametrize("trans_b", [0, 1])
@pytest.mark.parametrize("kind_a,kind_b", [("normal", "normal"), ("magnitudes", "magnitudes"), ("growth", "decay"),
                                           ("decay", "growth"), ("fits", "normal"), ("late", "normal"), ("normal", "late"),
                                           ("zeros", "normal")])
@pytest.mark.parametrize("size", ["few", "many"])
def test_rows(ctx, K, N, trans_b, kind_a, kind_b, size):
    banner("split rows", K, N, trans_b, kind_a, kind_b, size)
    if size == "many" and K not in (32, 64):
        pytest.skip("covered by the other widths")
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
