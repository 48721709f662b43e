"""fp32 contexts with large layers: parity with the fp64 oracle at the edges of
the tiles and K blocks, infinities and NaN, and operands that are held,
multiplied and summed as fp32 numbers whatever their scale.

Scaling a feature or a ReLU unit by a power of two, and the weights that read
it by the inverse, changes only exponents: every fp32 product, sum and
rounding scales with them, so the results are the unscaled ones times powers
of two, bit for bit.  A saturated tanh unit is exactly +-1 and its derivative
exactly 0, so the size of what saturates it cannot be seen in any result.
"""

import numpy as np
import pytest

from oracle import hf_oracle as O
from paper_1606_00511_amd import workloads as WL
from tests.parity_util import check, rel, relu_margins

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def net(dims, act, B, **kw):
    from paper_1606_00511_amd.hf import HFNet
    return HFNet(dims, act, B, **kw)


def results(h, theta, X, y, v):
    """Gradient and both products."""
    W, X, y, v = dev(theta), dev(X), dev(y), dev(v)
    return [host(h.hf_loss_grad(W, X, y)[1]), host(h.hf_hvp(W, X, y, v, "hessian")),
            host(h.hf_hvp(W, X, y, v, "gauss_newton"))]


def blocks(dims, t):
    """[(W_l, b_l), ...] as views of a copy of the parameter-layout vector."""
    t, out, at = t.copy(), [], 0
    for i, o in zip(dims[:-1], dims[1:]):
        out.append((t[at:at + i * o].reshape(o, i), t[at + i * o:at + i * o + o]))
        at += i * o + o
    return t, out


@pytest.mark.parametrize("dims,act,B", [((784, 500, 500, 500, 10), "tanh", 10000),
                                        ((440, 2048, 100), "sigmoid", 4096)],
                         ids=["digit", "speech"])
def test_gemms_are_fp32(dims, act, B):
    """Every GEMM of an fp32 context is one of the fp32 kernels."""
    p = WL.make_small(dims, act, B, seed=17)
    h = net(dims, act, B)
    W, X, y, v = dev(p["theta"]), dev(p["X"]), dev(p["y"]), dev(p["v"])
    h.prof_enable(True)
    h.prof_reset()
    _, g = h.hf_loss_grad(W, X, y)
    h.hf_hvp(W, X, y, v, "hessian")
    h.hf_cg(W, X, y, g, 1e-2, 2, mode="gauss_newton")
    names = set(h.prof_stats())
    h.prof_enable(False)
    h.close()
    assert any(n.startswith("hf_gemm") for n in names)
    assert not [n for n in names if "gemm" in n and not n.startswith("hf_gemm")]


# widths and rows around the tiles of 64 and 128, the K blocks and the splits
# of a weight gradient
CASES = [
    ((129, 1601, 130), "tanh", 10753),
    ((1056, 1030, 333), "sigmoid", 2049),
    ((1024, 1025, 1300), "tanh", 2100),
    ((784, 1500, 1501, 12), "relu", 2000),
    ((2200, 2100, 2050), "sigmoid", 512),
    ((256, 512, 10), "tanh", 16870),
]


@pytest.mark.parametrize("dims,act,B", CASES, ids=lambda v: str(v))
def test_parity(dims, act, B):
    p = WL.make_small(dims, act, B, seed=811 + B)
    h = net(dims, act, B)
    W, X, y, v = dev(p["theta"]), dev(p["X"]), dev(p["y"]), dev(p["v"])
    m = relu_margins(dims, act, p["theta"], p["X"])
    kink = lambda f: (lambda k: f(k)) if act == "relu" else None
    f, g = h.hf_loss_grad(W, X, y)
    f_o, g_o = O.loss_grad(dims, act, p["theta"], p["X"], p["y"])
    assert abs(float(host(f)[0]) - f_o) <= 1e-6 * abs(f_o)
    check(host(g), g_o, act, margins=m, bracket=kink(
        lambda k: O.loss_grad(dims, act, p["theta"], p["X"], p["y"], kink=k)[1]))
    for mode in ("hessian", "gauss_newton"):
        out = h.hf_hvp(W, X, y, v, mode)
        ref = O.curvature(dims, act, p["theta"], p["X"], p["y"], p["v"], mode)
        check(host(out), ref, act, margins=m, bracket=kink(
            lambda k: O.curvature(dims, act, p["theta"], p["X"], p["y"], p["v"], mode,
                                  kink=k)))
    h.hf_check()
    h.close()


@pytest.mark.parametrize("where", ["X inf", "X nan", "W inf", "v nan", "W huge"])
def test_nonfinite(where):
    """Infinities and NaN come out where the mean over batches of 300 rows has
    them, and nowhere else."""
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
        got = host(h.hf_hvp(W, Xd, y, vd, mode))
        parts = [host(h.hf_hvp(W, Xd[i:i + 300].contiguous(), y[i:i + 300].contiguous(),
                               vd, mode)).astype(np.float64) for i in range(0, B, 300)]
        want = sum(parts) / len(parts)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        ok = np.isfinite(want)
        assert np.array_equal(got[~ok & ~np.isnan(want)], want[~ok & ~np.isnan(want)])
        if ok.any():
            assert rel(got[ok], want[ok]) <= 1e-4
    h.close()


@pytest.mark.parametrize("k", [8, 24, 40])
def test_rescaled_features_and_units(k):
    """Half the features and half of each layer's ReLU units scaled by 2^-k,
    the weights (and direction) that read them by 2^k."""
    dims, act, B = (1100, 1500, 1000, 300), "relu", 1500
    p = WL.make_small(dims, act, B, seed=31)
    down = [np.where(np.arange(d) % 2 == 0, np.float32(2.0) ** -k, np.float32(1.0))
            .astype(np.float32) for d in dims]
    down[-1] = np.ones(dims[-1], np.float32)
    h = net(dims, act, B)
    plain = results(h, p["theta"], p["X"], p["y"], p["v"])

    def scaled(t, inverse):
        t, bl = blocks(dims, t)
        for l, (Wl, b) in enumerate(bl):
            s_in, s_out = down[l], down[l + 1]
            if inverse:                      # a gradient or product
                s_in, s_out = 1 / s_in, 1 / s_out
            Wl[:] = Wl * s_out[:, None] / s_in[None, :]
            b[:] = b * s_out
        return t

    got = results(h, scaled(p["theta"], False), p["X"] * down[0], p["y"],
                  scaled(p["v"], False))
    for a, b in zip(got, plain):
        assert np.array_equal(a, scaled(b, True))
    zero = h.hf_hvp(dev(p["theta"]), dev(p["X"]), dev(p["y"]), dev(np.zeros_like(p["v"])),
                    "gauss_newton")
    assert not host(zero).any()
    h.close()


def test_outlier_in_the_input():
    """One element of X large enough to saturate its row's tanh units: the
    oracle's results within the fp32 bar, and no trace of its size."""
    dims, act, B = (440, 2048, 100), "tanh", 2600
    p = WL.make_small(dims, act, B, seed=41)
    h = net(dims, act, B)
    out = []
    for size in (2.0 ** 40, 2.0 ** 60, 1e30):
        X = p["X"].copy()
        X[1234, 56] = size
        out.append(results(h, p["theta"], X, p["y"], p["v"]))
    h.close()
    for a, b in zip(out[0], out[1]):
        assert np.array_equal(a, b)
    for a, b in zip(out[0], out[2]):
        assert np.array_equal(a, b)
    X = p["X"].copy()
    X[1234, 56] = 2.0 ** 40
    check(out[0][0], O.loss_grad(dims, act, p["theta"], X, p["y"])[1], act)
    for mode, a in (("hessian", out[0][1]), ("gauss_newton", out[0][2])):
        check(a, O.curvature(dims, act, p["theta"], X, p["y"], p["v"], mode), act)


def test_one_large_weight():
    """A weight that saturates its tanh unit in every row leaves the other
    units' results within the fp32 bar."""
    dims, act, B = (1100, 1500, 300), "tanh", 1500
    p = WL.make_small(dims, act, B, seed=43)
    theta = p["theta"].copy()
    theta[7 * dims[0] + 3] = 2.0 ** 40
    p["X"][:, 3] = 0.5
    h = net(dims, act, B)
    g, hv, gv = results(h, theta, p["X"], p["y"], p["v"])
    h.close()
    check(g, O.loss_grad(dims, act, theta, p["X"], p["y"])[1], act)
    for mode, a in (("hessian", hv), ("gauss_newton", gv)):
        check(a, O.curvature(dims, act, theta, p["X"], p["y"], p["v"], mode), act)


@pytest.mark.parametrize("dims,ws,most", [((300, 1024, 1024, 1000), 12800, 40000),
                                          ((1600, 1600, 1600, 100), 4096, 40000)],
                         ids=["rows", "weights"])
def test_workspace_size_leaves_the_results(dims, ws, most):
    """The same call in a workspace for its own rows and in a larger one."""
    act = "tanh"
    p = WL.make_small(dims, act, ws, seed=47)
    out = []
    for rows in (ws, most):
        h = net(dims, act, most, ws_batch=rows)
        out.append(results(h, p["theta"], p["X"], p["y"], p["v"]))
        h.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
