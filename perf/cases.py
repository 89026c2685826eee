"""Performance cases of the polyspectrum estimator: what a program has it compute.

A case names a geometry (grid, order, shells), a precision and the calls it makes
through the package's public entry points: the differentiable ``polyspectrum``, the
``Plan`` calls shells / contract / backward, or the allocation-free
``polyspec_forward_static``.  Sizes are those of the repository's workloads and tests,
with ragged ones (shell counts that fill no 16-shell block) beside them.

    listed()            the cases themselves
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs and plan on the GPU
    run(state)          one pass; returns its outputs
    work(case)          bytes and flops that one pass cannot do without
    exact(case, seed)   the outputs of run in float64, by plain torch
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

import paper_1904_11055_amd as ps

PRECISION = {"fp32": ps.FP32, "bf16": ps.SPLIT_BF16, "fp16": ps.SPLIT_FP16}


def _case(name, N, order, shells, width=1.0, batch=1, precision="fp32", backward="", call="plan", field="lognormal",
          half=False, box=0.0, stream=False, multipole=-1):
    """backward: the adjoint's precision, or "" for a forward pass only.  multipole: ell, or -1."""
    return {"name": name, "N": N, "order": order, "shells": shells, "width": width, "batch": batch,
            "precision": precision, "backward": backward, "call": call, "field": field, "half": half, "box": box,
            "stream": stream, "multipole": multipole}


def listed():
    return [
        # power spectrum of a small box in a serving loop: launches and latency
        _case("power_64_static", 64, 2, 31, precision="fp32", call="static", field="gaussian"),
        # the differentiable call with its defaults on the small test grid: a fit's inner loop
        _case("bispec_64_autograd", 64, 3, 16, precision="fp32", backward="fp32", call="autograd", field="gaussian"),
        # redshift-space quadrupole of a survey-like box; 46 fields fill no whole shell block
        _case("multipole_128", 128, 3, 23, width=1.5, precision="fp16", multipole=2),
        # a batch of fields with its gradient, as field-level inference runs it
        _case("bispec_grad_128x8", 128, 3, 24, batch=8, precision="fp16", backward="bf16", field="gaussian"),
        # bispectrum of one box in plain float32
        _case("bispec_256_fp32", 256, 3, 40, width=2.0, precision="fp32"),
        # a program that holds the half spectrum and wants physical units; ragged shells, BF16 split
        _case("bispec_256_half", 256, 3, 53, width=1.5, precision="bf16", backward="bf16", half=True, box=1000.0),
        # trispectrum with its gradient, up to 32 shells
        _case("trispec_256", 256, 4, 24, width=2.0, precision="fp16", backward="bf16"),
        # trispectrum with its gradient, more than 32 shells
        _case("trispec_256_40", 256, 4, 40, precision="fp16", backward="bf16"),
        # order 5
        _case("quadspec_256", 256, 5, 16, precision="fp16"),
        # order 6
        _case("pentaspec_256", 256, 6, 8, precision="fp16"),
        # the benchmark's step: forward in the FP16 split, gradient in the BF16 split
        _case("bispec_512", 512, 3, 64, precision="fp16", backward="bf16"),
        # the largest grid, streamed in slabs, forward and gradient
        _case("bispec_1024_streamed", 1024, 3, 64, precision="fp16", backward="bf16", stream=True),
    ]


def draw(rng):
    """One more case of the listed ranges; no costlier than the 512^3 and 1024^3 ones."""
    while True:
        order = rng.choice([2, 3, 3, 3, 3, 4, 4, 5, 6])
        N = rng.choice({2: [32, 64, 128, 256, 512], 3: [32, 64, 128, 256, 256, 512], 4: [32, 64, 128, 256],
                        5: [64, 128, 256], 6: [64, 128, 256]}[order])
        width = rng.choice([1.0, 1.0, 1.0, 1.5, 2.0, 0.5] if order <= 4 else [1.0])
        top = int(N / (order * width) - 0.5)
        cap = {2: 100, 3: 64, 4: 40, 5: 16, 6: 8}[order]
        if order == 4:
            cap = min(cap, int(52 / width))     # polygon counts stay below their limit
        top = min(top, cap)
        if top < 3:
            continue
        shells = min(top, max(3, int(round(math.exp(rng.uniform(math.log(4), math.log(top + 0.5)))))))
        batch = rng.choice([1, 1, 2, 3, 5, 8]) if N <= 128 else 1
        precision = rng.choice(["fp32", "bf16", "fp16", "fp16"])
        multipole = -1
        backward = ""
        half = stream = False
        call = "plan"
        if order in (3, 4):
            kind = rng.choice(["forward", "grad", "grad", "autograd"] + (["multipole", "stream"] if order == 3 else []))
            if kind == "multipole":
                multipole = rng.choice([0, 2, 4])
                shells = min(shells, 32)
            elif kind == "stream":
                stream = N >= 128
                backward = "fp32" if precision == "fp32" else "bf16"
            elif kind != "forward":
                backward = precision if kind == "autograd" else ("fp32" if precision == "fp32"
                                                                 else rng.choice(["bf16", precision]))
                call = "autograd" if kind == "autograd" else "plan"
            half = kind in ("forward", "grad") and rng.random() < 0.25
        elif order == 2 and N == 64 and batch == 1:
            call = "static"
            shells = min(shells, 31)
        case = _case(None, N, order, shells, width=width, batch=batch, precision=precision, backward=backward, call=call,
                     field=rng.choice(["gaussian", "lognormal"]), half=half,
                     box=rng.choice([0.0, 0.0, 1000.0]), stream=stream, multipole=multipole)
        del case["name"]
        if work(case)["flops"] <= 5e13:
            return case


# --- inputs ------------------------------------------------------------------
def _spectrum_grid(N, device):
    k = torch.fft.fftfreq(N, d=1.0 / N, device=device)
    k2 = torch.arange(N // 2 + 1, device=device, dtype=torch.float32)
    return k[:, None, None] ** 2 + k[None, :, None] ** 2 + k2[None, None, :] ** 2


def _field(case, seed, device):
    """float32 [batch, N, N, N]: unit-variance Gaussian with P = k^-2, or its lognormal sibling."""
    N = case["N"]
    gen = torch.Generator(device=device).manual_seed(1000003 * (seed % 1000003) + N)
    kk = _spectrum_grid(N, device)
    kk[0, 0, 0] = 1.0
    if case["field"] == "gaussian":
        amp = kk ** -0.5
    else:
        amp = kk ** -0.375 * torch.exp(-0.5 * kk / (N / 4.0) ** 2)
    del kk
    amp[0, 0, 0] = 0.0
    out = torch.empty((case["batch"], N, N, N), dtype=torch.float32, device=device)
    for b in range(case["batch"]):
        w = torch.fft.rfftn(torch.randn((N, N, N), generator=gen, device=device))
        w *= amp
        g = torch.fft.irfftn(w, s=(N, N, N))
        del w
        g /= g.flatten()[:: max(1, N // 64)].std()
        if case["field"] == "lognormal":
            g.sub_(0.5).exp_().sub_(1.0)
        out[b] = g
        del g
    return out


def _input(case, seed, device):
    x = _field(case, seed, device)
    return torch.fft.rfftn(x, dim=(1, 2, 3)).contiguous() if case["half"] else x


def _loss_weights(tuples, device):
    """Weights of the squares in the loss: the inverse of a red spectrum's expected scatter."""
    t = np.asarray(tuples, dtype=np.float64)
    w = np.prod(t ** 1.5, axis=1)
    return torch.as_tensor(2.0 * w / w.mean(), dtype=torch.float64, device=device)


def prepare(case, seed):
    device = torch.device("cuda", torch.cuda.current_device())
    flags = (ps.INPUT_HALF_SPECTRUM if case["half"] else 0) | (ps.STREAM_SLABS if case["stream"] else 0)
    plan = ps.Plan(case["N"], case["order"], case["shells"], case["width"], batch=case["batch"],
                   precision=PRECISION[case["precision"]], box_length=case["box"], flags=flags, device=device,
                   multipole=case["multipole"] if case["multipole"] >= 0 else None)
    state = {"case": case, "plan": plan, "x": _input(case, seed, device)}
    if case["backward"]:
        state["weights"] = _loss_weights(plan.tuples, device)
    if case["call"] == "static":
        state["out"] = torch.empty((case["batch"], plan.n_closing), dtype=torch.float64, device=device)
    return state


def run(state):
    case, plan, x = state["case"], state["plan"], state["x"]
    if case["call"] == "static":
        ps.polyspec_forward_static(plan.handle, x.data_ptr(), state["out"].data_ptr())
        return state["out"]
    if case["call"] == "autograd":
        leaf = x.detach().requires_grad_(True)
        B = ps.polyspectrum(leaf, plan)
        (grad,) = torch.autograd.grad(B, leaf, grad_outputs=state["weights"] * B.detach())
        return B.detach(), grad
    plan.shells(x)
    B = plan.contract()
    if not case["backward"]:
        return B
    if case["backward"] != case["precision"]:      # the adjoint's own arithmetic
        plan.precision = PRECISION[case["backward"]]
    grad = plan.backward(state["weights"] * B)
    if case["backward"] != case["precision"]:
        plan.precision = PRECISION[case["precision"]]
    return B, grad


# --- work --------------------------------------------------------------------
def _sorted_tuples(order, nb):
    """Sorted tuples of shells 1..nb whose largest side the others can reach, lexicographic."""
    rows = np.array(list(itertools.combinations_with_replacement(range(1, nb + 1), order)), dtype=np.int64)
    return rows[2 * rows[:, -1] < 2 * rows[:, :-1].sum(1) + order]


def work(case):
    N, nb, n, batch = case["N"], case["shells"], case["order"], case["batch"]
    G = float(N) ** 3
    tuples = len(_sorted_tuples(n, nb)) * (3 if case["multipole"] >= 0 else 1)
    fields = nb * (2 if case["multipole"] >= 0 else 1)
    values = 8.0 * N * N * (N // 2 + 1) if case["half"] else 4.0 * G
    # an input transform, one real transform's last pass per shell field, a product and a
    # sum per tuple and point; the gradient: two products per tuple and point, and the
    # same transforms the other way
    fft = (7.5 + 2.5 * fields) * G * math.log2(N)
    flops = fft + 2.0 * tuples * G
    nbytes = values + 8.0 * tuples
    if case["backward"]:
        flops += fft + 4.0 * tuples * G
        nbytes += values + 8.0 * tuples
    return {"bytes": nbytes * batch, "flops": flops * batch}


# --- float64 -----------------------------------------------------------------
def _legendre(ell, mu):
    p0, p1 = torch.ones_like(mu), mu
    if ell == 0:
        return p0
    for m in range(1, ell):
        p0, p1 = p1, ((2 * m + 1) * mu * p1 - m * p0) / (m + 1)
    return p1


class _Exact:
    """The estimator and its gradient by full-grid float64 transforms and matrix products."""

    def __init__(self, case, device):
        self.N, self.n, self.nb, self.device = case["N"], case["order"], case["shells"], device
        N = self.N
        k = torch.fft.fftfreq(N, d=1.0 / N, device=device, dtype=torch.float64).round().to(torch.int32)
        c = torch.arange(N // 2 + 1, device=device, dtype=torch.int32)
        q2 = k[:, None, None] ** 2 + k[None, :, None] ** 2 + c[None, None, :] ** 2
        # |q|^2 < ((s + 1/2) D)^2, decided on integers (D is a binary fraction)
        edges = [math.ceil(((2 * s - 1) * case["width"]) ** 2 / 4) for s in range(1, self.nb + 2)]
        self.shell = torch.bucketize(q2, torch.tensor(edges, dtype=torch.int32, device=device), right=True).to(torch.int16)
        self.shell[q2 >= edges[-1]] = 0
        self.weight = None
        if case["multipole"] >= 0:
            mu = c.to(torch.float64)[None, None, :] / q2.to(torch.float64).clamp_min(1).sqrt()
            self.weight = _legendre(case["multipole"], mu)
        del q2
        self.rows = [list(itertools.combinations_with_replacement(range(self.nb), m)) for m in range(4)]
        # tuple = left part (left shells) + right part
        self.left = {2: 1, 3: 2, 4: 2, 5: 2, 6: 3}[self.n]

    def fields(self, hat):
        """[n_shells, N^3] inverse transforms of hat restricted to each shell."""
        N = self.N
        out = torch.empty((self.nb, N ** 3), dtype=torch.float64, device=self.device)
        for s in range(self.nb):
            m = torch.where(self.shell == s + 1, hat, torch.zeros((), dtype=torch.complex128, device=self.device))
            out[s] = torch.fft.irfftn(m, s=(N, N, N), norm="forward").flatten()
        return out

    def products(self, d, m):
        rows = torch.tensor(self.rows[m], device=self.device)
        out = d[rows[:, 0]]
        for j in range(1, m):
            out *= d[rows[:, j]]
        return out

    def chunk(self):
        big = max(len(self.rows[self.left]), len(self.rows[self.n - self.left]))
        return max(4096, min(1 << 18, (1 << 28) // big))

    def sums(self, d, right=None):
        """Matrix of sum_x left product times right product (right: other fields for the last side)."""
        total = 0.0
        step = self.chunk()
        for x0 in range(0, d.shape[1], step):
            a = self.products(d[:, x0:x0 + step], self.left)
            b = right[:, x0:x0 + step] if right is not None else self.products(d[:, x0:x0 + step], self.n - self.left)
            total = total + a @ b.T
        return total

    def locate(self, tuples):
        """Left and right row of each tuple (0-based shells)."""
        m, r = self.left, self.n - self.left
        li = {t: i for i, t in enumerate(self.rows[m])}
        ri = {t: i for i, t in enumerate(self.rows[r])}
        a = torch.tensor([li[tuple(t[:m])] for t in tuples], device=self.device)
        b = torch.tensor([ri[tuple(t[m:])] for t in tuples], device=self.device)
        return a, b

    def counts(self):
        """Closing tuples (0-based shells) and their polygon counts."""
        tuples = (_sorted_tuples(self.n, self.nb) - 1).tolist()
        ones = torch.ones((), dtype=torch.complex128, device=self.device)
        S = self.sums(self.fields(ones))
        a, b = self.locate(tuples)
        q = (S[a, b] / float(self.N) ** 3).round()
        keep = (q > 0).cpu().numpy()
        return [t for t, k in zip(tuples, keep) if k], q[q > 0]

    def adjoint(self, d, a, b, g):
        """dL/d(fields) of L = sum_t g_t S_t (orders 3 and 4), in place of the fields."""
        rows = torch.tensor(self.rows[2], device=self.device)
        W = torch.zeros((len(self.rows[2]), len(self.rows[self.n - 2])), dtype=torch.float64, device=self.device)
        W[a, b] = g
        step = self.chunk()
        for x0 in range(0, d.shape[1], step):
            c = d[:, x0:x0 + step].clone()
            P = self.products(c, 2)
            out = torch.zeros_like(c)
            if self.n == 3:
                dP = W @ c
                out += W.T @ P
            else:
                dP = (W + W.T) @ P
            out.index_add_(0, rows[:, 0], c[rows[:, 1]] * dP)
            out.index_add_(0, rows[:, 1], c[rows[:, 0]] * dP)
            d[:, x0:x0 + step] = out
        return d


def exact(case, seed):
    if case["N"] > 512:
        return None
    device = torch.device("cuda", torch.cuda.current_device())
    N, n = case["N"], case["order"]
    x = _input(case, seed, device)
    e = _Exact(case, device)
    tuples, counts = e.counts()
    factor = 1.0
    if case["box"] > 0:
        factor = (case["box"] ** 3) ** (n - 1) / float(N) ** (3 * n)
    rows = tuples
    if case["multipole"] >= 0:                      # (u, v; w): each distinct weighted side
        table = {}
        for t, q in zip(tuples, counts.tolist()):
            for w in range(3):
                rest = tuple(t[:w] + t[w + 1:])
                table[rest + (t[w],)] = q
        rows = sorted(table)
        counts = torch.tensor([table[t] for t in rows], dtype=torch.float64, device=device)
        factor *= 2 * case["multipole"] + 1
    norm = factor / (float(N) ** 3 * counts)
    a, b = e.locate(rows)
    weights = _loss_weights(np.array(rows) + 1, device)
    Bs, grads = [], []
    for i in range(case["batch"]):
        hat = x[i].to(torch.complex128) if case["half"] else torch.fft.rfftn(x[i].to(torch.float64))
        if case["half"]:                            # the DC column of a real field's transform is Hermitian
            hat = hat.contiguous()
        d = e.fields(hat)
        right = e.fields(hat * e.weight) if e.weight is not None else None
        S = e.sums(d, right)
        B = S[a, b] * norm
        Bs.append(B)
        if not case["backward"]:
            del d, right
            continue
        d = e.adjoint(d, a, b, weights * B * norm)
        g = torch.zeros((N, N, N // 2 + 1), dtype=torch.complex128, device=device)
        for s in range(e.nb):
            h = torch.fft.rfftn(d[s].view(N, N, N))
            g = torch.where(e.shell == s + 1, h, g)
        del d
        if case["half"]:
            g[:, :, 1:N // 2] *= 2.0
            grads.append(g)
        else:
            grads.append(torch.fft.irfftn(g, s=(N, N, N), norm="forward"))
    B = torch.stack(Bs)
    return (B, torch.stack(grads)) if case["backward"] else B
