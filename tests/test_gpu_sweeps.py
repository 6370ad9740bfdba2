"""GPU parity of the convolution's kernels at the edges of their size rules:
the sender segment sum on short and long slots, in float32 and float64,
against the fp64 oracle on a graph with uneven degrees (a hub sender and a
hub receiver, nodes without edges, degrees around the steps of the sweeps).

Bars: relative L2 <= 1e-5 per float32 output and <= 1e-12 per float64 output
(one rounding per term of sums of at most a few thousand terms).
"""
import numpy as np
import pytest

from oracle import conv as oconv
from oracle import irreps as oirreps

from gpu_util import TOL, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

TOL64 = 1e-12


@pytest.fixture(scope="module")
def e3():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2609_35099_amd import e3mi
    e3mi.lib()
    return e3mi


def _graph(rng, pad):
    """Receiver degrees 0, 1, 2, ..., 20 and 67, sender 0 a hub of every third edge."""
    deg = list(range(21)) + [67]
    rcv = np.repeat(np.arange(len(deg)), deg)
    n = len(deg) + 3
    snd = rng.integers(1, len(deg), rcv.shape[0])
    snd[::3] = 0
    order = rng.permutation(rcv.shape[0])
    snd, rcv = snd[order], rcv[order]
    if pad >= 0:   # every 11th edge is padding, on either side
        snd[::22], rcv[11::22] = pad, pad
    vec = rng.standard_normal((rcv.shape[0], 3))
    return snd.astype(np.int32), rcv.astype(np.int32), vec, n


def _check_conv(e3, irreps, lsh, lout, f64, pad=-1, natural=False, composed=False):
    rng = np.random.default_rng(11)
    dt = np.float64 if f64 else np.float32
    lay = oirreps.layout(irreps, lsh, lout, "natural" if natural else "all")
    plan = e3.Plan(irreps, lsh, lout, natural=natural, composed=composed)
    snd, rcv, vec, n = _graph(rng, pad)
    E, C = rcv.shape[0], lay.channels
    x, s, dm = (rng.standard_normal(sh).astype(dt) for sh in
                ((n, lay.d_in, C), (E, lay.n_paths, C), (n, lay.d_out, C)))
    vec = vec.astype(dt)
    G = e3.Graph(to_dev(snd), to_dev(rcv), n, pad_node=pad)
    print("[case]", irreps, lsh, lout, "f64" if f64 else "f32", plan.kernels, pad, flush=True)
    dev = [to_dev(a) for a in (x, vec, s)]
    fwd, bwd = (e3.conv_fwd_f64, e3.conv_bwd_f64) if f64 else (e3.conv_fwd, e3.conv_bwd)
    m = fwd(plan, G, *dev)
    dx, dvec, ds = bwd(plan, G, *dev, to_dev(dm))
    ref_m = oconv.conv_fwd(lay, x, vec, s, snd, rcv, n, pad_node=pad).numpy()
    ref = oconv.conv_bwd(lay, x, vec, s, dm, snd, rcv, n, pad_node=pad)
    errs = {"m": rel_l2(to_np(m), ref_m), "dx": rel_l2(to_np(dx), ref["dx"].numpy()),
            "ds": rel_l2(to_np(ds), ref["ds"].numpy()), "dvec": rel_l2(to_np(dvec), ref["dvec"].numpy())}
    for k, v in errs.items():
        assert v < (TOL64 if f64 else TOL), (k, v)
    again = (fwd(plan, G, *dev), *bwd(plan, G, *dev, to_dev(dm)))
    for a, b in zip((m, dx, dvec, ds), again):
        assert a.equal(b)


# slots of 1, 12, 20, 128, 144, 256 and 272 16-byte units (float64: twice as many)
@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("irreps,lsh,lout", [
    ("4x0e", 1, 1), ("12x0e+12x1o", 2, 2), ("20x0e+20x1o", 2, 2), ("128x0e+128x1o", 2, 2),
    ("64x0e+64x1o+64x2e", 2, 2), ("64x0e+64x1o+64x2e+64x3o", 3, 3), ("68x0e+68x1o+68x2e+68x3o", 3, 3),
])
def test_segment_sum_widths(e3, irreps, lsh, lout, f64):
    _check_conv(e3, irreps, lsh, lout, f64)
