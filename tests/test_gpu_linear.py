"""The linear mixing's tiles and operand splitting at their edges, against
float64: row remainders of the 128-row tile, channel counts on either side of
the 64- and 128-wide tiles, odd counts of 16-wide reduction halves, several
blocks per type, W off 16-byte alignment; operands over the whole float32
range; infinities and NaNs where float32 has them.

Bar: relative L2 1e-6 per output.  A forward or dx sum has at most 336 terms in
11 steps, each a few roundings of 6e-8 of the running sum; a dW element sums
up to 9,000 rows as 64 partials of up to five steps.  At random they add to
about 3e-7.  The products themselves are exact but for l l, 2^-34.
"""
import numpy as np
import pytest

from gpu_util import rel_l2, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def e3():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2609_35099_amd import e3mi
    e3mi.lib()
    return e3mi


def _blocks(irreps):
    out, row = [], 0
    for tok in irreps.split("+"):
        l = int(tok[:-1])
        out.append((tok, row, 2 * l + 1))
        row += 2 * l + 1
    return out, row


def _reference(ins, outs, ci, co, x, W, d):
    """out, dx, dW in float64."""
    (bi, di), (bo, do) = _blocks(ins), _blocks(outs)
    out, dx, dW, o = np.zeros((len(x), do, co)), np.zeros((len(x), di, ci)), [], 0
    for to, ro, n in bo:
        for ti, ri, _ in bi:
            if ti == to:
                w = W[o:o + ci * co].reshape(ci, co)
                xi, dd = x[:, ri:ri + n], d[:, ro:ro + n]
                out[:, ro:ro + n] += xi @ w
                dx[:, ri:ri + n] += dd @ w.T
                dW.append((xi.reshape(-1, ci).T @ dd.reshape(-1, co)).reshape(-1))
                o += ci * co
    return out, dx, np.concatenate(dW) if dW else np.zeros(0)


def _run(e3, ins, outs, ci, co, x, W, d, shift=0):
    import torch
    L = e3.Linear("+".join(f"{ci}x{t}" for t in ins.split("+")), "+".join(f"{co}x{t}" for t in outs.split("+")))
    buf = torch.empty(len(W) + 4, device="cuda")
    Wd = buf[shift:shift + len(W)]
    Wd.copy_(torch.from_numpy(W))
    xd, dd = torch.from_numpy(x).cuda(), torch.from_numpy(d).cuda()
    print("[case]", ins, outs, ci, co, len(x), shift, flush=True)
    return [to_np(t) for t in (L.forward(xd, Wd), *L.backward(xd, Wd, dd))]


def _inputs(ins, outs, ci, co, n, seed=1):
    rng = np.random.default_rng(seed)
    (bi, di), (bo, do) = _blocks(ins), _blocks(outs)
    nw = sum(ti[0] == to[0] for ti in bi for to in bo) * ci * co
    return [rng.standard_normal(s).astype(np.float32) for s in ((n, di, ci), (nw,), (n, do, co))]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("ins,outs,ci,co,n", [
    ("0e", "0e", 16, 16, 1), ("0e+1o", "1o+0e", 16, 48, 43), ("1o+1o+0e", "1o+0e", 48, 64, 128),
    ("0e", "0e", 64, 80, 129), ("0e+1o+2e+0e", "0e+2e+1o+1o", 80, 128, 77), ("3o+1o", "1o+3o", 128, 144, 300),
    ("1o+1o+1o", "1o", 112, 192, 127), ("0e+1e", "0e+1o", 256, 16, 1000), ("2e+70e", "70e+2e", 16, 32, 11),
    ("0e+0e", "0e+0e", 96, 96, 9000),
])
def test_linear_tiles(e3, ins, outs, ci, co, n, shift):
    x, W, d = _inputs(ins, outs, ci, co, n)
    got = _run(e3, ins, outs, ci, co, x, W, d, shift)
    for g, r in zip(got, _reference(ins, outs, ci, co, *(a.astype(np.float64) for a in (x, W, d)))):
        assert rel_l2(g, r) < 1e-6


@pytest.mark.parametrize("sx,sw", [(1e-37, 1.0), (1.0, 1e-37), (1e-30, 1e20), (1e-19, 1e-19), (1e26, 1e-3),
                                   (1e33, 1e-20), (1e-12, 1e33), (1e36, 1.0)])
def test_linear_magnitudes(e3, sx, sw):
    """Operands from the subnormals to the largest floats (the last ones take the float32 instruction)."""
    ins = outs = "0e+1o"
    x, W, d = _inputs(ins, outs, 128, 64, 150)
    x, W = (np.clip(x, -3, 3) * np.float32(sx)).astype(np.float32), (np.clip(W, -3, 3) * np.float32(sw)).astype(np.float32)
    got = _run(e3, ins, outs, 128, 64, x, W, d)
    for g, r in zip(got, _reference(ins, outs, 128, 64, *(a.astype(np.float64) for a in (x, W, d)))):
        assert np.isfinite(r).all() and np.abs(r).max() < 3e38
        top = np.abs(r).max()
        assert rel_l2(g.astype(np.float64) / top, r / top) < 1e-6


def test_linear_infinities_and_nans(e3):
    ins = outs = "0e+1o"
    x, W, d = _inputs(ins, outs, 64, 128, 400)
    x[5, 0, 7], x[9, 2, 3], x[300, 0, 1], x[300, 0, 2] = np.inf, np.nan, np.inf, -np.inf
    x[11, 1, 0], d[20, 3, 5] = 3.4e38, -np.inf
    W = (W / 8).astype(np.float32)
    W[9] = 0.0
    got = _run(e3, ins, outs, 64, 128, x, W, d)
    with np.errstate(all="ignore"):
        ref = _reference(ins, outs, 64, 128, *(a.astype(np.float64) for a in (x, W, d)))
    for g, r in zip(got, ref):
        r = np.where(np.abs(r) > np.finfo(np.float32).max, np.sign(r) * np.inf, r)
        assert (np.isnan(g) == np.isnan(r)).all()
        inf = np.isinf(r)
        assert (np.isinf(g) == inf).all() and (np.sign(g[inf]) == np.sign(r[inf])).all()
        ok = np.isfinite(r) & (np.abs(r) < 1e30)
        assert rel_l2(g[ok], r[ok]) < 1e-6


def test_linear_single_products(e3):
    """One non-zero term per sum: the float32 product, rounded once (2^-24, and
    the rounding of the lower terms' sum, below 2^-30)."""
    ci, co, n = 128, 64, 500
    x, W, d = _inputs("0e+0e", "0e", ci, co, n)
    x[:, :, 1:], x[:, 1], d[:, :, 1:] = 0, 0, 0
    out, dx, dW = _run(e3, "0e+0e", "0e", ci, co, x, W, d)
    w = W.reshape(2, ci, co).astype(np.float64)
    _, _, dW1 = _run(e3, "0e+0e", "0e", ci, co, *(a[:1] if a.ndim > 1 else a for a in _inputs("0e+0e", "0e", ci, co, 1)))
    x1, _, d1 = (a.astype(np.float64) for a in _inputs("0e+0e", "0e", ci, co, 1))
    for got, ref in ((out[:, 0], np.outer(x[:, 0, 0], w[0, 0])), (dx[:, 0], np.outer(d[:, 0, 0], w[0, :, 0])),
                     (dW1.reshape(2, ci, co), x1[0, :, :, None] * d1[0, 0])):
        err = np.abs(got - ref) / np.abs(ref)
        assert err.max() < 2.0**-24 * (1 + 2.0**-6)


@pytest.mark.parametrize("blocks,C,n,bars", [
    (8, 512, 100, (1.0e-6, 1.0e-6, 1e-6)), (1, 64, 200_000, (1e-6, 1e-6, 9e-7)),
])
def test_linear_long_sums(e3, blocks, C, n, bars):
    """4,096 terms (forward, dx) and 200,000 (dW): below what the float32
    instruction leaves (1.15e-6 and 1.03e-6; here 4.5e-7 and 3.0e-7)."""
    irreps = "+".join(["0e"] * blocks)
    x, W, d = _inputs(irreps, irreps, C, C, n)
    got = _run(e3, irreps, irreps, C, C, x, W, d)
    ref = _reference(irreps, irreps, C, C, *(a.astype(np.float64) for a in (x, W, d)))
    for g, r, bar in zip(got, ref, bars):
        assert rel_l2(g, r) < bar


def test_linear_dw_row_offsets(e3):
    """Node rows of 164 MB: a chunk's 16 scalar rows lie up to 2.4 GB apart."""
    import torch
    n, ci, co = 16, 4096, 16
    g = torch.Generator(device="cuda").manual_seed(2)
    L = e3.Linear("+".join([f"{ci}x0e"] + [f"{ci}x999e"] * 5), f"{co}x0e")
    assert 15 * L.D_in * ci * 4 > 2**31
    x = torch.zeros(n, L.D_in, ci, device="cuda")
    x[:, 0] = torch.randn(n, ci, generator=g, device="cuda")
    W, d = (torch.randn(s, generator=g, device="cuda") for s in ((ci * co,), (n, 1, co)))
    print("[case] dW row offsets", L.D_in * ci * 4, flush=True)
    _, dW = L.backward(x, W, d)
    ref = x[:, 0].double().T.contiguous() @ d[:, 0].double()
    assert rel_l2(to_np(dW), to_np(ref).reshape(-1)) < 1e-6


def test_linear_dw_long_chunks(e3):
    """Chunks of 2,488,750 rows of a block of 1,991 per node: row number times
    block height passes 2^32, where a quotient by multiplication needs its
    correction (at 2,174,171 for the first time)."""
    import torch
    n, C, R = 80_000, 16, 1991
    g = torch.Generator(device="cuda").manual_seed(3)
    L = e3.Linear(f"{C}x0e+{C}x995e", f"{C}x995e+{C}x0e")
    x, d = (torch.randn(n, R + 1, C, generator=g, device="cuda") for _ in range(2))
    W = torch.randn(L.n_weights, generator=g, device="cuda")
    print("[case] dW long chunks", n * R // 64, flush=True)
    _, dW = L.backward(x, W, d)
    ref = torch.zeros(2, C, C, dtype=torch.float64, device="cuda")
    for a in range(0, n, 4000):
        xs, ds = x[a:a + 4000].double(), d[a:a + 4000].double()
        ref[0] += xs[:, 1:].reshape(-1, C).T.contiguous() @ ds[:, :R].reshape(-1, C)
        ref[1] += xs[:, 0].T.contiguous() @ ds[:, R]
    # 78,000 sums of 32 rows per chunk, each addition rounding the partial by up
    # to 6e-8: sqrt(78,000) of them at random leave up to 1.7e-5 of a result,
    # whose size is that of its random sum; a step of wrong rows gives 1e-2
    got = to_np(dW).reshape(2, C, C)
    assert rel_l2(got[0], to_np(ref[0])) < 2e-5 and rel_l2(got[1], to_np(ref[1])) < 1e-6


def test_linear_dw_more_tiles_than_a_grid_row(e3):
    """57 x 57 pairs of 528 channels, 81 tiles of 64 in each of 64 chunks: 4.3e9
    threads, which a launch wraps without an error if they lie along x (the
    partials take 232 GB)."""
    import gc
    import torch
    gc.collect()
    torch.cuda.empty_cache()
    B, C, n = 57, 528, 3
    irreps = "+".join([f"{C}x0e"] * B)
    L = e3.Linear(irreps, irreps)
    assert B * B * 64 * 81 * 256 > 2**32
    g = torch.Generator(device="cuda").manual_seed(4)
    x, d = (torch.randn(n, B, C, generator=g, device="cuda") for _ in range(2))
    W = torch.zeros(L.n_weights, device="cuda")
    print("[case] dW tiles", L.n_weights, flush=True)
    _, dW = L.backward(x, W, d)
    del W
    dW = dW.reshape(B, B * C, C)
    xt = x.double().reshape(n, B * C).T.contiguous()
    for o in range(B):
        ref = xt @ d[:, o].double()
        assert float((dW[o].double() - ref).norm() / ref.norm()) < 1e-6
    del dW, ref, xt
    torch.cuda.empty_cache()


def test_linear_elements_depend_on_their_own_operands(e3):
    """Infinities, NaNs and operands that the terms cannot hold change no bit of
    any other row (forward, dx) or channel pair (dW)."""
    ins = outs = "0e+1o"
    ci, co, n = 64, 128, 400
    x, W, d = _inputs(ins, outs, ci, co, n)
    clean = _run(e3, ins, outs, ci, co, x, W, d)
    xr, xc, dr, dc = [5, 9, 130], [7, 40], [20, 300], [3, 100]
    x[5, :, 7], x[9, 2, 7], x[130, 0, 40], d[20, :, 3], d[300, 1, 100] = np.inf, np.nan, 1e30, -np.inf, 3.4e38
    out, dx, dW = _run(e3, ins, outs, ci, co, x, W, d)
    for got, ref, rows in ((out, clean[0], xr), (dx, clean[1], dr)):
        keep = np.setdiff1d(np.arange(n), rows)
        assert (got[keep] == ref[keep]).all()
        assert not np.isfinite(got[rows[0]]).any()
    k, j = np.setdiff1d(np.arange(ci), xc), np.setdiff1d(np.arange(co), dc)
    got, ref = (a.reshape(2, ci, co)[:, k][:, :, j] for a in (dW, clean[2]))
    assert (got == ref).all()
