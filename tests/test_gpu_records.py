"""The caller-record tensor product at the edges of its record walk and row
tiles: record counts around a chunk of 64 and the look-ahead, output rows
without records (first, last, in between), row and channel remainders, both
kinds of y, both precisions, against a float64 sum record by record.

Bars: rel-L2 1e-6 in float32 and 1e-14 in float64.  An output row sums at most
137 records, and a shared y's cotangent those of its channels too, in runs of
64 (137 records over 4 output rows, 320 channels: chains of 137, 64 and 5); at
random the roundings of such chains, each 6e-8 of a partial sum at most, add to
under 16 of them.
"""
import numpy as np
import pytest

from gpu_util import rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def e3():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2609_35099_amd import e3mi
    e3mi.lib()
    return e3mi


def _check(e3, nnz, dims, rows, C, ypc, f64):
    rng = np.random.default_rng(nnz * 7 + rows)
    dx_, dy_, dz_ = dims
    # output rows 0, dz - 1 and every fourth one get no record
    outs = [o for o in range(dz_) if o % 4 != 0 and o != dz_ - 1] or [0]
    i0 = rng.choice(outs, nnz).astype(np.int32)
    i1, i2 = rng.integers(0, dx_, nnz).astype(np.int32), rng.integers(0, dy_, nnz).astype(np.int32)
    val = rng.standard_normal(nnz)
    dt = np.float64 if f64 else np.float32
    x = rng.standard_normal((rows, dx_, C)).astype(dt)
    y = rng.standard_normal((rows, dy_, C) if ypc else (rows, dy_)).astype(dt)
    dz = rng.standard_normal((rows, dz_, C)).astype(dt)
    print("[case]", nnz, dims, rows, C, ypc, f64, flush=True)
    tp = e3.RecordTP(dx_, dy_, dz_, i0, i1, i2, val, y_per_channel=ypc)
    z = tp.forward(to_dev(x), to_dev(y))
    gx, gy = tp.backward(to_dev(x), to_dev(y), to_dev(dz))
    x, y, dz = x.astype(np.float64), y.astype(np.float64), dz.astype(np.float64)
    yc = y if ypc else np.repeat(y[..., None], C, 2)
    rz, rx, ry = np.zeros((rows, dz_, C)), np.zeros_like(x), np.zeros_like(yc)
    v = val if f64 else val.astype(np.float32).astype(np.float64)
    for a, b, c, w in zip(i0, i1, i2, v):
        rz[:, a] += w * x[:, b] * yc[:, c]
        rx[:, b] += w * dz[:, a] * yc[:, c]
        ry[:, c] += w * dz[:, a] * x[:, b]
    ry = ry if ypc else ry.sum(2)
    tol = 1e-14 if f64 else 1e-6
    for got, ref in ((z, rz), (gx, rx), (gy, ry)):
        assert rel_l2(to_np(got), ref) < tol
    empty = [o for o in range(dz_) if o not in set(i0.tolist())]
    assert not to_np(z)[:, empty].any()


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("ypc", [False, True])
@pytest.mark.parametrize("nnz,dims,rows,C", [
    (0, (2, 3, 4), 5, 7), (1, (1, 1, 1), 1, 1), (3, (4, 2, 5), 2, 63), (63, (5, 4, 7), 3, 64),
    (64, (5, 4, 7), 4, 65), (65, (9, 9, 9), 5, 100), (67, (9, 9, 9), 9, 12), (137, (9, 4, 16), 13, 130),
    (260, (40, 3, 30), 6, 20), (90, (60, 50, 8), 3, 10),
    (137, (9, 16, 20), 5, 64), (90, (30, 7, 8), 3, 128), (70, (3, 4, 5), 7, 192), (65, (70, 9, 9), 2, 320),
])
def test_record_walk_edges(e3, nnz, dims, rows, C, ypc, f64):
    _check(e3, nnz, dims, rows, C, ypc, f64)


# enough pairs for the widest tiles: 4, 2 and 1 pairs per lane, four and eight
# records ahead, a shared y per row of the tile (1 to 66 rows) and per 64 pairs
@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("ypc", [False, True])
@pytest.mark.parametrize("nnz,dims,rows,C", [
    (21, (4, 4, 4), 2_100, 128), (21, (4, 3, 4), 2_701, 100), (70, (16, 5, 16), 4_200, 64), (70, (16, 16, 3), 2_701, 100),
    (135, (9, 9, 9), 13_300, 20), (33, (3, 4, 5), 262_201, 1), (66, (30, 7, 8), 1_400, 192), (40, (25, 4, 9), 2_001, 132),
])
def test_wide_tiles(e3, nnz, dims, rows, C, ypc, f64):
    assert rows * C >= 4 * 64 * 1024
    _check(e3, nnz, dims, rows, C, ypc, f64)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("ypc,C", [(True, 100), (False, 100), (False, 64)])
def test_infinities_and_nans(e3, ypc, C, f64):
    """Infinities and NaNs where the sum record by record has them, in the first
    operand rows too, which output rows without records and the table's padding
    name; every other element as without them."""
    rng = np.random.default_rng(C)
    nnz, dx_, dy_, dz_, rows = 67, 5, 4, 9, 50
    i0 = rng.choice([1, 2, 3, 5, 6, 7], nnz).astype(np.int32)
    i1, i2 = rng.integers(0, dx_, nnz).astype(np.int32), rng.integers(0, dy_, nnz).astype(np.int32)
    val, dt = rng.standard_normal(nnz), np.float64 if f64 else np.float32
    x = rng.standard_normal((rows, dx_, C)).astype(dt)
    y = rng.standard_normal((rows, dy_, C) if ypc else (rows, dy_)).astype(dt)
    tp = e3.RecordTP(dx_, dy_, dz_, i0, i1, i2, val, y_per_channel=ypc)
    print("[case] infinities", ypc, C, f64, flush=True)
    clean = to_np(tp.forward(to_dev(x), to_dev(y)))
    x[3, 0, 7], x[20, 2, 99 % C], x[20, 0, 1] = np.inf, np.nan, -np.inf
    y[(31, 0, 5) if ypc else (31, 0)] = np.inf
    z = to_np(tp.forward(to_dev(x), to_dev(y)))
    ref, yc = np.zeros((rows, dz_, C)), y if ypc else np.repeat(y[..., None], C, 2)
    with np.errstate(all="ignore"):
        for a, b, c, w in zip(i0, i1, i2, val):
            ref[:, a] += w * x[:, b].astype(np.float64) * yc[:, c]
    assert np.array_equal(np.isnan(z), np.isnan(ref)) and np.isnan(ref).any()
    inf = np.isinf(ref)
    assert np.array_equal(np.isinf(z), inf) and np.array_equal(np.sign(z[inf]), np.sign(ref[inf])) and inf.any()
    ok = np.isfinite(ref)
    assert np.array_equal(z[ok], clean[ok])


def test_wide_shared_operands_f64(e3):
    """float64 operands of 200 rows with a shared y: more than 64 KiB staged per wave."""
    rng = np.random.default_rng(5)
    nnz, dx_, dy_, dz_, rows, C = 300, 100, 100, 8, 7, 70
    i0, i1, i2 = (rng.integers(0, d, nnz).astype(np.int32) for d in (dz_, dx_, dy_))
    val, x, y = rng.standard_normal(nnz), rng.standard_normal((rows, dx_, C)), rng.standard_normal((rows, dy_))
    print("[case] wide shared operands", flush=True)
    z = e3.RecordTP(dx_, dy_, dz_, i0, i1, i2, val, y_per_channel=False).forward(to_dev(x), to_dev(y))
    ref = np.zeros((rows, dz_, C))
    for a, b, c, w in zip(i0, i1, i2, val):
        ref[:, a] += w * x[:, b] * y[:, c, None]
    assert rel_l2(to_np(z), ref) < 1e-14


def test_more_tiles_than_a_grid_row(e3):
    """43 million rows in two pieces of 64 channels (dy of 40 rows): 5.5e9 threads,
    which a launch wraps without an error if they lie along x."""
    import torch
    rows, C = 43_000_000, 100
    g = torch.Generator(device="cuda").manual_seed(1)
    k = np.arange(40, dtype=np.int32)
    tp = e3.RecordTP(1, 40, 1, 0 * k, 0 * k, k, np.ones(40), y_per_channel=False)
    x, dz = (torch.randn(rows, 1, C, generator=g, device="cuda") for _ in range(2))
    y = torch.randn(rows, 40, generator=g, device="cuda")
    print("[case] many tiles", rows * C, flush=True)
    z = tp.forward(x, y)
    dx, dy = tp.backward(x, y, dz)
    for a in range(0, rows, 4_000_000):
        xs, ys, ds = (t[a:a + 4_000_000].double() for t in (x[:, 0], y, dz[:, 0]))
        s = ys.sum(1, keepdim=True)
        for got, ref in ((z[a:a + 4_000_000, 0], xs * s), (dx[a:a + 4_000_000, 0], ds * s),
                         (dy[a:a + 4_000_000], (xs * ds).sum(1, keepdim=True).expand(-1, 40))):
            assert float((got.double() - ref).norm() / ref.norm()) < 1e-6


@pytest.mark.parametrize("C", [64, 100, 128, 256, 320])
def test_shared_y_channel_sum(e3, C):
    """One record: dy sums C products of one sign.  Runs of at most 64 channels,
    then the runs: no further from float64 than that order in numpy (1.1: the
    order within a run differs)."""
    rng = np.random.default_rng(C)
    rows = 20_000
    tp = e3.RecordTP(1, 1, 1, *(np.zeros(1, np.int32) for _ in range(3)), np.ones(1), y_per_channel=False)
    x, dz = (rng.uniform(0.5, 1.5, (rows, 1, C)).astype(np.float32) for _ in range(2))
    y = np.ones((rows, 1), np.float32)
    print("[case] channel sum", C, flush=True)
    _, gy = tp.backward(to_dev(x), to_dev(y), to_dev(dz))
    prod = x[:, 0] * dz[:, 0]
    runs = [np.cumsum(prod[:, a:a + 64], 1, dtype=np.float32)[:, -1:] for a in range(0, C, 64)]
    want = np.cumsum(np.concatenate(runs, 1), 1, dtype=np.float32)[:, -1]
    ref = (x[:, 0].astype(np.float64) * dz[:, 0]).sum(1)
    assert rel_l2(to_np(gy)[:, 0], ref) < 1.1 * rel_l2(want, ref)
