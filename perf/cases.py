"""The work that a user of this library has it do, as cases that can be timed.

The listed cases are the entry points of ``HFNet`` on the nets that the
library's workloads name (digit-image nets of 784 inputs, speech-frame nets of
440 inputs and 1,973 classes), from one worker's smallest call to the full
speech minibatch, in both GEMM precisions.  ``draw`` varies nets, batches,
activations, entry points and precisions over the same ranges.

A case: ``op`` (the entry point), ``d0``/``hidden``/``depth``/``classes`` (the
net), ``act``, ``prec``, ``batch`` rows and, for the solvers, ``iters`` and
``damping``; ``iterate`` takes its gradient on ``batch`` rows and its curvature
on the first ``curv_batch`` of them.
"""

import torch

from paper_1606_00511_amd import hf

OPS = ("loss", "grad", "fisher", "hv", "gv", "cg", "pcg", "bicgstab", "iterate")


def _case(name, op, net, act, batch, prec="fp32", iters=0, damping=1e-2,
          curv_batch=0):
    d0, hidden, depth, classes = net
    c = dict(op=op, d0=d0, hidden=hidden, depth=depth, classes=classes, act=act,
             prec=prec, batch=batch, iters=iters, damping=damping,
             curv_batch=curv_batch)
    if name:
        c["name"] = name
    return c


SMALL = (784, 100, 1, 10)
DIGIT = (784, 500, 3, 10)
SPEECH = (440, 2048, 4, 1973)
RAGGED = (351, 1021, 2, 203)


def listed():
    return [
        # the smallest calls, bound by launches: gradient, exact product and
        # solve of the one-hidden-layer digit net on a minibatch of 1,000
        _case("small_grad_b1000", "grad", SMALL, "sigmoid", 1000),
        _case("small_hv_b1000", "hv", SMALL, "sigmoid", 1000),
        _case("small_cg_b1000", "cg", SMALL, "sigmoid", 1000, iters=10),
        # the Newton-CG inner loop of the deeper digit net
        _case("digit_tanh_cg_b10000", "cg", DIGIT, "tanh", 10000, iters=10),
        # one whole outer iteration: gradient on 60,000 rows, solve on a
        # subsample of 6,000, line search
        _case("digit_relu_iterate_b60000", "iterate", DIGIT, "relu", 60000,
              iters=10, curv_batch=6000),
        # sizes that are multiples of nothing
        _case("ragged_gv_b3001", "gv", RAGGED, "tanh", 3001),
        # one worker's share of a data-parallel step on the speech net:
        # gradient on 4,096 rows, solve on 1,024
        _case("speech_grad_b4096", "grad", SPEECH, "sigmoid", 4096),
        _case("speech_cg_b1024", "cg", SPEECH, "sigmoid", 1024, iters=10),
        # the full speech minibatch: an exact product on its own, and the
        # inner loop
        _case("speech_hv_b16384", "hv", SPEECH, "sigmoid", 16384),
        _case("speech_cg_b16384", "cg", SPEECH, "sigmoid", 16384, iters=5),
        # the same work with bf16 GEMM operands
        _case("speech_hv_bf16_b4096", "hv", SPEECH, "sigmoid", 4096, prec="bf16"),
        _case("speech_cg_bf16_b16384", "cg", SPEECH, "sigmoid", 16384,
              prec="bf16", iters=5),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(("small", "digit", "speech", "speech"))
        act = rng.choice(("sigmoid", "tanh", "relu"))
        prec = "fp32"
        if kind == "small":
            net = (_log(rng, 256, 1024), _log(rng, 32, 128), rng.choice((1, 1, 2)),
                   rng.randint(5, 40))
            batch = _log(rng, 250, 4000)
        elif kind == "digit":
            net = (_log(rng, 400, 1024), _log(rng, 200, 800), rng.randint(2, 3),
                   rng.randint(10, 64))
            batch = _log(rng, 1000, 20000)
        else:
            net = (_log(rng, 300, 500), _log(rng, 1000, 2048), rng.randint(2, 4),
                   _log(rng, 500, 2000))
            batch = _log(rng, 512, 16384)
            prec = rng.choice(("fp32", "fp32", "bf16"))
        op = rng.choice(("loss", "grad", "grad", "fisher", "hv", "hv", "gv", "gv",
                         "cg", "cg", "pcg", "bicgstab"))
        iters, damping = 0, 1e-2
        if op in ("cg", "pcg"):
            iters = rng.randint(3, 10 if prec == "fp32" else 5)
        elif op == "bicgstab":
            iters, damping = rng.randint(1, 3), 1e-1
        c = _case(None, op, net, act, batch, prec, iters, damping)
        if work(c)["flops"] <= most:
            return c


def _dims(case):
    return (case["d0"],) + (case["hidden"],) * case["depth"] + (case["classes"],)


# ------------------------------------------------------------------- inputs

def _inputs(case, seed):
    """theta, X, y and v on the GPU, of the shapes and distributions of the
    digit-image (uniform pixels, uniform labels) or speech-frame (normal
    features, Zipf labels) workloads."""
    dims, B = _dims(case), case["batch"]
    speech = case["classes"] >= 500
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kw = dict(device="cuda", dtype=torch.float32, generator=gen)
    draw_x = torch.randn if speech else torch.rand
    X = draw_x(B, dims[0], **kw)
    C = dims[-1]
    w = torch.ones(C, device="cuda")
    if speech:
        w = torch.arange(1, C + 1, device="cuda").float() ** -1.1
    y = torch.multinomial(w, B, replacement=True, generator=gen).to(torch.int32)
    parts = []
    for i, o in zip(dims[:-1], dims[1:]):
        parts += [torch.randn(o * i, **kw) / i ** 0.5, torch.randn(o, **kw) * 0.1]
    W = torch.cat(parts)
    v = torch.randn(W.numel(), **kw)
    return W, X, y, v


def _solver_inputs(case, W, X, y):
    """The gradient that a solve starts from and, for a preconditioned one,
    M^-1, in 64 bits and rounded once."""
    ref = _Ref(case, W, X, y)
    g = ref.grad().float()
    minv = None
    if case["op"] == "pcg":
        minv = (ref.fisher() + case["damping"]).pow(-0.75).float()
    return g, minv


def prepare(case, seed):
    W, X, y, v = _inputs(case, seed)
    net = hf.HFNet(_dims(case), case["act"], case["batch"], prec=case["prec"])
    st = dict(case=case, net=net, W=W, X=X, y=y, v=v,
              out=torch.empty_like(W), out2=torch.empty_like(W),
              loss=torch.empty(1, device="cuda"))
    if case["op"] in ("cg", "pcg", "bicgstab"):
        st["g"], st["minv"] = _solver_inputs(case, W, X, y)
    if case["op"] == "iterate":
        st["Xc"], st["yc"] = X[:case["curv_batch"]], y[:case["curv_batch"]]
    return st


def run(st):
    c, net = st["case"], st["net"]
    W, X, y = st["W"], st["X"], st["y"]
    op = c["op"]
    if op == "loss":
        return {"loss": net.hf_loss(W, X, y, loss=st["loss"])}
    if op == "grad":
        loss, grad = net.hf_loss_grad(W, X, y, loss=st["loss"], grad=st["out"])
        return {"loss": loss, "grad": grad}
    if op == "fisher":
        return {"fisher": net.hf_fisher_diag(W, X, y, out=st["out"])}
    if op == "hv":
        return {"hv": net.hf_hvp(W, X, y, st["v"], "hessian", out=st["out"])}
    if op == "gv":
        return {"gv": net.hf_hvp(W, X, None, st["v"], "gauss_newton", out=st["out"])}
    if op == "iterate":
        W1, delta = st["out"], st["out2"]
        W1.copy_(W)
        delta.zero_()
        info, _ = net.hf_iterate(W1, X, y, st["Xc"], st["yc"], delta, solver="cg",
                                 curvature="gauss_newton", damping=c["damping"],
                                 max_iters=c["iters"])
        return {"W": W1, "delta": delta, "f0": info["f0"], "f1": info["f1"]}
    kw = dict(mode="gauss_newton", step=st["out"], neg_dir=st["out2"])
    if op == "cg":
        step, _, info = net.hf_cg(W, X, y, st["g"], c["damping"], c["iters"], **kw)
    elif op == "pcg":
        step, _, info = net.hf_pcg(W, X, y, st["g"], st["minv"], c["damping"],
                                   c["iters"], **kw)
    else:
        step, _, info = net.hf_bicgstab(W, X, y, st["g"], c["damping"], c["iters"],
                                        **kw)
    return {"step": step, "rr_final": info["rr_final"], "iters": info["iters"]}


# --------------------------------------------------------------------- work

def work(case):
    """One product per matrix and direction of each pass: a forward pass
    (B P multiply-adds for P weights), a backward pass to the first hidden
    layer, a weight gradient, and the two products per layer that the
    R-operator adds."""
    dims, B, it = _dims(case), case["batch"], case["iters"]
    P = sum(i * o for i, o in zip(dims[:-1], dims[1:]))
    P1 = dims[0] * dims[1]
    n = P + sum(dims[1:])
    op = case["op"]
    fwd, bwd, wg = P, P - P1, P
    rfwd = P + (P - P1)
    gnp = rfwd + bwd + wg                       # a Gauss-Newton product
    mac = {"loss": fwd, "grad": fwd + bwd + wg, "fisher": fwd + bwd + wg,
           "hv": fwd + bwd + rfwd + 2 * bwd + wg + (P - P1), "gv": fwd + gnp,
           "cg": fwd + it * gnp, "pcg": fwd + it * gnp,
           "bicgstab": fwd + 2 * it * gnp}
    vecs = {"loss": 1, "grad": 2, "fisher": 2, "hv": 3, "gv": 3, "cg": 4,
            "pcg": 5, "bicgstab": 4, "iterate": 4}
    inputs = 4 * B * dims[0] + (0 if op == "gv" else 4 * B)
    if op == "iterate":
        macs = B * mac["grad"] + case["curv_batch"] * (fwd + it * gnp) + B * fwd
    else:
        macs = B * mac[op]
    return {"bytes": inputs + 4 * vecs[op] * n, "flops": 2 * macs}


# ---------------------------------------------------------------- tolerance

def tolerance(case):
    """Four times what the path was seen off 64 bits, or from itself with its
    sums in another order, over the listed and drawn cases."""
    op, relu = case["op"], case["act"] == "relu"
    if case["prec"] == "bf16":
        return {"rel": 0.03, "max": 0.9}
    if op == "iterate":
        return {"rel": 5e-3, "max": 0.2}
    if op in ("cg", "pcg", "bicgstab"):
        return {"rel": 2e-3 if relu else 3e-4, "max": 0.2 if relu else 1e-2}
    # a ReLU unit whose input rounds to the other side of 0 changes its whole
    # column of one row
    return {"rel": 2e-4 if relu else 4e-5, "max": 0.1 if relu else 2e-3}


# -------------------------------------------------------------------- exact

class _Ref:
    """The same quantities in float64, from the equations."""

    def __init__(self, case, W, X, y):
        self.dims, self.act = _dims(case), case["act"]
        self.layers = self._split(W.double())
        self.X, self.y = X.double(), y.long()
        self.B = X.shape[0]
        self.A, self.Z = [self.X], []
        for k, (Wl, bl) in enumerate(self.layers):
            z = self.A[-1] @ Wl.t() + bl
            self.Z.append(z)
            if k + 1 < len(self.layers):
                self.A.append(self._phi(z))
        self.P = torch.softmax(self.Z[-1], dim=1)

    def _split(self, t):
        out, at = [], 0
        for i, o in zip(self.dims[:-1], self.dims[1:]):
            out.append((t[at:at + i * o].view(o, i), t[at + i * o:at + i * o + o]))
            at += i * o + o
        return out

    def _phi(self, z):
        return {"sigmoid": torch.sigmoid, "tanh": torch.tanh, "relu": torch.relu}[self.act](z)

    def _d1(self, a):
        if self.act == "sigmoid":
            return a * (1 - a)
        if self.act == "tanh":
            return 1 - a * a
        return (a > 0).double()

    def _d2(self, a):
        if self.act == "sigmoid":
            return a * (1 - a) * (1 - 2 * a)
        if self.act == "tanh":
            return -2 * a * (1 - a * a)
        return torch.zeros_like(a)

    def loss(self):
        z = self.Z[-1]
        return (torch.logsumexp(z, 1) - z.gather(1, self.y[:, None])[:, 0]).mean()

    def _delta(self):
        d = self.P.clone()
        d[torch.arange(self.B, device=d.device), self.y] -= 1
        return d

    @staticmethod
    def _join(parts):
        return torch.cat([t.reshape(-1) for pair in reversed(parts) for t in pair])

    def grad(self):
        d, parts = self._delta() / self.B, []
        for k in reversed(range(len(self.layers))):
            parts.append((d.t() @ self.A[k], d.sum(0)))
            if k:
                d = (d @ self.layers[k][0]) * self._d1(self.A[k])
        return self._join(parts)

    def fisher(self):
        d, parts = self._delta(), []
        for k in reversed(range(len(self.layers))):
            d2 = d * d
            parts.append((d2.t() @ (self.A[k] ** 2) / self.B, d2.sum(0) / self.B))
            if k:
                d = (d @ self.layers[k][0]) * self._d1(self.A[k])
        return self._join(parts)

    def product(self, v, hessian):
        V = self._split(v.double())
        RA, RZ = [None], []
        for k, ((Wl, _), (Vl, cl)) in enumerate(zip(self.layers, V)):
            rz = self.A[k] @ Vl.t() + cl
            if RA[k] is not None:
                rz += RA[k] @ Wl.t()
            RZ.append(rz)
            if k + 1 < len(self.layers):
                RA.append(self._d1(self.A[k + 1]) * rz)
        rz = RZ[-1]
        rd = self.P * (rz - (self.P * rz).sum(1, keepdim=True)) / self.B
        d = self._delta() / self.B if hessian else None
        parts = []
        for k in reversed(range(len(self.layers))):
            gw = rd.t() @ self.A[k]
            if hessian and RA[k] is not None:
                gw += d.t() @ RA[k]
            parts.append((gw, rd.sum(0)))
            if k:
                Wl, a = self.layers[k][0], self.A[k]
                back = rd @ Wl
                if hessian:
                    e = d @ Wl
                    rd = (back + d @ V[k][0]) * self._d1(a) + e * self._d2(a) * RZ[k - 1]
                    d = e * self._d1(a)
                else:
                    rd = back * self._d1(a)
        return self._join(parts)

    def cg(self, g, lam, iters, minv=None):
        m = 1.0 if minv is None else minv.double()
        g = g.double()
        x, r = torch.zeros_like(g), g.clone()
        z = m * r
        p, rz = -z, r @ z
        for _ in range(iters):
            q = self.product(p, False) + lam * p
            a = rz / (p @ q)
            x, r = x + a * p, r + a * q
            z = m * r
            new = r @ z
            p, rz = -z + (new / rz) * p, new
        return x, float(r @ r)

    def bicgstab(self, g, lam, iters):
        r = -g.double()
        r0, p, x = r.clone(), r.clone(), torch.zeros_like(r)
        for _ in range(iters):
            q = self.product(p, False) + lam * p
            a = (r @ r0) / (q @ r0)
            s = r - a * q
            t = self.product(s, False) + lam * s
            w = (t @ s) / (t @ t)
            x = x + a * p + w * s
            new = s - w * t
            p = new + (new @ r0) / (r @ r0) * (a / w) * (p - w * q)
            r = new
        return x, float(r @ r)


def exact(case, seed):
    W, X, y, v = _inputs(case, seed)
    op, lam, it = case["op"], float(torch.tensor(case["damping"])), case["iters"]
    ref = _Ref(case, W, X, y)
    if op == "loss":
        return {"loss": ref.loss().reshape(1)}
    if op == "grad":
        return {"loss": ref.loss().reshape(1), "grad": ref.grad()}
    if op == "fisher":
        return {"fisher": ref.fisher()}
    if op in ("hv", "gv"):
        return {op: ref.product(v, op == "hv")}
    if op == "iterate":
        Bc = case["curv_batch"]
        f0, g = float(ref.loss()), ref.grad()
        d, _ = _Ref(case, W, X[:Bc], y[:Bc]).cg(g, lam, it)
        gd, alpha = float(g @ d), 1.0
        for _ in range(21):
            W1 = W.double() + alpha * d
            f1 = float(_Ref(case, W1, X, y).loss())
            if f1 <= f0 + 1e-4 * alpha * gd:
                return {"W": W1, "delta": d, "f0": f0, "f1": f1}
            alpha *= 0.5
        return {"W": W.double(), "delta": torch.zeros_like(d), "f0": f0, "f1": f0}
    g, minv = _solver_inputs(case, W, X, y)
    if op == "bicgstab":
        x, rr = ref.bicgstab(g, lam, it)
    else:
        x, rr = ref.cg(g, lam, it, minv)
    return {"step": x, "rr_final": rr, "iters": it}
