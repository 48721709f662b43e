"""fp32 contexts whose layers run on fp16 pairs (B d_l d_{l-1} >= 2.2e9, at
least 128 wide on both sides, at least 512 rows): parity with the fp64 oracle at the edges of the
tiles, K groups and row chunks, the scaling of badly scaled inputs, and
infinities and NaN.

Bounds: a pair holds 22 significant bits or more of every value within 2^-16
of its tensor's largest, so a product of two is off by less than 3 x 2^-22; the
sums add at most the rounding of an fp32 accumulator per 32 terms.  Through a
net of at most 4 layers with well-scaled values that stays below 4e-6, 25
times under the fp32 bar of the other parity tests.
"""

import numpy as np
import pytest

from oracle import hf_oracle as O
from paper_1606_00511_amd import workloads as WL
from tests.parity_util import check, rel, relu_margins

pytestmark = pytest.mark.gpu

TOL = 4e-6


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def net(dims, act, B):
    from paper_1606_00511_amd.hf import HFNet
    return HFNet(dims, act, B)


def ran_on_pairs(h, call):
    h.prof_enable(True)
    h.prof_reset()
    out = call()
    names = set(h.prof_stats())
    h.prof_enable(False)
    assert any(n.startswith("hf_sgemm") for n in names), sorted(names)
    return out


# widths and rows around the K group of 32, the chunk of 64, the tiles of 128
# and 256, the third plane (contractions up to 1,024), the smallest batch on
# pairs, and layers on fp32 kernels beside layers on pairs
CASES = [
    ((129, 1601, 130), "tanh", 10753),
    ((1056, 1030, 333), "sigmoid", 2049),
    ((1024, 1025, 1300), "tanh", 2100),
    ((784, 1500, 1501, 12), "relu", 2000),
    ((2200, 2100, 2050), "sigmoid", 512),
    # the weight gradient's last split holds one K block, fewer than the
    # stages of a grid with one workgroup per CU
    ((256, 512, 10), "tanh", 16870),
]


@pytest.mark.parametrize("dims,act,B", CASES, ids=lambda v: str(v))
def test_pairs_parity(dims, act, B):
    p = WL.make_small(dims, act, B, seed=811 + B)
    h = net(dims, act, B)
    W, X, y, v = dev(p["theta"]), dev(p["X"]), dev(p["y"]), dev(p["v"])
    m = relu_margins(dims, act, p["theta"], p["X"])
    kink = lambda f: (lambda k: f(k)) if act == "relu" else None
    f, g = ran_on_pairs(h, lambda: h.hf_loss_grad(W, X, y))
    f_o, g_o = O.loss_grad(dims, act, p["theta"], p["X"], p["y"])
    assert abs(float(host(f)[0]) - f_o) <= 1e-6 * abs(f_o)
    check(host(g), g_o, act, tol=TOL, margins=m, bracket=kink(
        lambda k: O.loss_grad(dims, act, p["theta"], p["X"], p["y"], kink=k)[1]))
    for mode in ("hessian", "gauss_newton"):
        out = h.hf_hvp(W, X, y, v, mode)
        ref = O.curvature(dims, act, p["theta"], p["X"], p["y"], p["v"], mode)
        check(host(out), ref, act, tol=TOL, margins=m, bracket=kink(
            lambda k: O.curvature(dims, act, p["theta"], p["X"], p["y"], p["v"], mode,
                                  kink=k)))
    h.hf_check()
    h.close()


def test_feature_scales_and_zero_operands():
    """Features 12 orders of magnitude apart (weights compensating), a zero
    feature and a zero direction: every layer-1 column keeps the precision of
    its own scale.  The exact Hessian product is the difference of larger
    terms here, so the bound is the error of the fp32 kernels on the same
    input (as the mean over batches of 300 rows, which they serve), with half
    as much again for a column of few elements, plus that of a pair."""
    dims, act, B = (1500, 1501, 1000), "tanh", 1500
    p = WL.make_small(dims, act, B, seed=31)
    s = np.float32(2.0) ** np.linspace(-20, 20, dims[0]).round().astype(np.float32)
    X = (p["X"] * s).astype(np.float32)
    X[:, 7] = 0.0
    theta, v = p["theta"].copy(), p["v"].copy()
    n1 = dims[0] * dims[1]
    theta[:n1] = (theta[:n1].reshape(dims[1], dims[0]) / s).reshape(-1)
    v[:n1] = (v[:n1].reshape(dims[1], dims[0]) / s).reshape(-1)
    h = net(dims, act, B)
    W, Xd, y, vd = dev(theta), dev(X), dev(p["y"]), dev(v)

    def both(f):
        parts = [host(f(Xd[i:i + 300].contiguous(), y[i:i + 300].contiguous()))
                 .astype(np.float64) for i in range(0, B, 300)]
        return host(ran_on_pairs(h, lambda: f(Xd, y))), sum(parts) / len(parts)

    _, g_o = O.loss_grad(dims, act, theta, X, p["y"])
    ref = O.curvature(dims, act, theta, X, p["y"], v, "hessian")
    for (got, f32), want in (
            (both(lambda a, b: h.hf_loss_grad(W, a, b)[1]), g_o),
            (both(lambda a, b: h.hf_hvp(W, a, b, vd, "hessian")), ref)):
        a, b, c = (t[:n1].reshape(dims[1], dims[0]) for t in (got, want, f32))
        for k in range(dims[0]):
            if k == 7:
                assert not a[:, k].any()
            else:
                assert rel(a[:, k], b[:, k]) <= 1.5 * rel(c[:, k], b[:, k]) + 2.0 ** -22, k
        assert rel(got[n1:], want[n1:]) <= 1.5 * rel(f32[n1:], want[n1:]) + 2.0 ** -22
    zero = h.hf_hvp(W, Xd, y, dev(np.zeros_like(v)), "gauss_newton")
    assert not host(zero).any()
    h.close()


@pytest.mark.parametrize("where", ["X inf", "X nan", "W inf", "v nan", "W huge"])
def test_nonfinite_as_on_fp32(where):
    """A tensor that cannot be split: the GEMMs that read it take their fp32
    operands, so that infinities and NaN come out where the fp32 kernels put
    them.  Those serve batches of 300 rows, whose mean is the whole batch's
    product."""
    import torch
    dims, act, B = (1500, 1000, 1500), "sigmoid", 1500
    p = WL.make_small(dims, act, B, seed=5)
    X, theta, v = p["X"].copy(), p["theta"].copy(), p["v"].copy()
    n1 = dims[0] * dims[1]
    if where == "X inf":
        X[3, 5] = np.inf            # saturates row 3's hidden units
    elif where == "X nan":
        X[3, 5] = np.nan
    elif where == "W inf":
        theta[2 * dims[0] + 1] = np.inf
    elif where == "W huge":
        theta[:n1] *= np.float32(1e36)   # finite, sums overflow
    else:
        v[n1 + dims[1] + 4] = np.nan
    h = net(dims, act, B)
    W, Xd, y, vd = dev(theta), dev(X), dev(p["y"]), dev(v)
    for mode in ("hessian", "gauss_newton"):
        got = host(ran_on_pairs(h, lambda: h.hf_hvp(W, Xd, y, vd, mode)))
        parts = [host(h.hf_hvp(W, Xd[i:i + 300].contiguous(), y[i:i + 300].contiguous(),
                               vd, mode)).astype(np.float64) for i in range(0, B, 300)]
        want = sum(parts) / len(parts)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        ok = np.isfinite(want)
        assert np.array_equal(got[~ok & ~np.isnan(want)], want[~ok & ~np.isnan(want)])
        if ok.any():
            assert rel(got[ok], want[ok]) <= 1e-4
    h.close()
