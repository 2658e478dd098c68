"""Performance cases: the work that a user of this framework has it do.

Each case is one pass through a public entry point of the binding: the
product of two tensor trains (full and randomized swap SVD, d = 8 grid
fields, binary sites, mixed dimensions), the variational baseline, a batch of
uneven products, the gradient of <W, A*B>, and a training step through the
truncated product.

A product's cores are fixed only up to rotations on its bonds, so a pass that
ends in a train also evaluates it on its grid (a few matrix products): the
values there, and the train's bonds, are what a caller reads.
"""
import math

import numpy as np
import torch

import paper_2410_19747_amd as T

F64 = torch.float64


def listed():
    return [
        # The smallest call: ten binary sites at bond 8 (the smoke test's random trains).
        dict(name="random-n10-chi8", kind="multiply", data="random", phys="2," * 9 + "2", chi_a=8, chi_b=8,
             chi=8, tol=1e-14, svd="jacobi"),
        # Mixed physical dimensions and odd bonds: a parameter grid rather than a field.
        dict(name="mixed-n7-chi21", kind="multiply", data="random", phys="3,5,2,7,4,6,3", chi_a=23, chi_b=19,
             chi=21, tol=1e-12, svd="jacobi"),
        # A 64^3 field in the paper's own binary encoding (18 sites of d = 2, 153 swaps).
        dict(name="binary-n18-chi32", kind="multiply", data="field", grid=64, binary=True, chi_a=32, chi_b=32,
             chi=32, tol=1e-14, svd="jacobi"),
        # Products of two velocity components on a 256^3 grid: the benchmark workload at its two bonds.
        dict(name="grid256-chi64", kind="multiply", data="field", grid=256, binary=False, chi_a=64, chi_b=64,
             chi=64, tol=1e-14, svd="jacobi"),
        dict(name="grid256-chi128", kind="multiply", data="field", grid=256, binary=False, chi_a=128, chi_b=128,
             chi=128, tol=1e-14, svd="jacobi"),
        # The upper end of the bond dimension that a pass of under two seconds reaches.
        dict(name="grid128-chi256", kind="multiply", data="field", grid=128, binary=False, chi_a=256, chi_b=256,
             chi=256, tol=1e-14, svd="jacobi"),
        # The reduced-accuracy option on the benchmark workload.
        dict(name="grid256-chi128-rsvd", kind="multiply", data="field", grid=256, binary=False, chi_a=128, chi_b=128,
             chi=128, tol=1e-14, svd="randomized"),
        # The variational baseline on the same field.
        dict(name="fit-grid256-chi64", kind="fit", data="field", grid=256, binary=False, chi_a=64, chi_b=64,
             chi=64, tol=1e-12),
        # The advection term's nine products at uneven bonds, in one call.
        dict(name="batch9-grid64", kind="batch", data="field", grid=64, binary=False,
             chis="64,16,8,32,4,16,8,32,4", tol=1e-14, streams=4),
        # Gradient of <W, A*B>: the adjoint benchmark's size, and a ragged one with FP32 operands.
        dict(name="grad-n10-chi128", kind="grad", phys="8," * 9 + "8", chi_a=128, chi_b=128, chi_w=32, prec="f64"),
        dict(name="grad-n9-chi97-f32", kind="grad", phys="8,5,8,7,8,6,8,3,8", chi_a=97, chi_b=61, chi_w=13,
             prec="f32"),
        # A training step: loss and both gradients through the truncated product.
        dict(name="loss-n6-chi24", kind="loss", phys="4,4,4,4,4,4", chi_a=24, chi_b=24, chi_w=8, chi=24, tol=1e-12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["field", "field", "field", "binary", "random", "random", "rsvd", "fit", "batch", "grad",
                       "grad", "loss"])
    tol = rng.choice([1e-14, 1e-14, 1e-12, 1e-10])
    if kind in ("field", "rsvd"):
        chi = _log_int(rng, 12, 112)
        return dict(kind="multiply", data="field", grid=rng.choice([32, 64, 128, 256]), binary=False, chi_a=chi,
                    chi_b=max(4, int(chi * rng.uniform(0.5, 1.0))), chi=max(4, int(chi * rng.uniform(0.7, 1.1))),
                    tol=tol, svd="randomized" if kind == "rsvd" else "jacobi")
    if kind == "binary":
        chi = _log_int(rng, 6, 40)
        return dict(kind="multiply", data="field", grid=rng.choice([16, 32, 64]), binary=True, chi_a=chi, chi_b=chi,
                    chi=max(4, int(chi * rng.uniform(0.7, 1.1))), tol=tol, svd="jacobi")
    if kind == "random":
        n = rng.randint(4, 10)
        phys = [rng.randint(2, 8 if n < 7 else 4) for _ in range(n)]
        chi = _log_int(rng, 4, 40)
        return dict(kind="multiply", data="random", phys=",".join(map(str, phys)), chi_a=chi,
                    chi_b=max(2, int(chi * rng.uniform(0.5, 1.2))), chi=chi, tol=tol, svd="jacobi")
    if kind == "fit":
        chi = _log_int(rng, 6, 56)
        return dict(kind="fit", data="field", grid=rng.choice([32, 64, 128]), binary=False, chi_a=chi, chi_b=chi,
                    chi=max(4, int(chi * rng.uniform(0.7, 1.1))), tol=1e-12)
    if kind == "batch":
        return dict(kind="batch", data="field", grid=rng.choice([16, 32, 64]), binary=False,
                    chis=",".join(str(_log_int(rng, 3, 48)) for _ in range(rng.randint(3, 9))), tol=1e-14,
                    streams=rng.randint(1, 4))
    if kind == "grad":
        n = rng.randint(4, 10)
        chi = _log_int(rng, 8, 120)
        return dict(kind="grad", phys=",".join(str(rng.randint(2, 8)) for _ in range(n)), chi_a=chi,
                    chi_b=max(4, int(chi * rng.uniform(0.5, 1.0))), chi_w=_log_int(rng, 2, 32),
                    prec=rng.choice(["f64", "f64", "f32"]))
    n = rng.randint(4, 7)
    chi = _log_int(rng, 4, 24)
    return dict(kind="loss", phys=",".join(str(rng.randint(2, 4)) for _ in range(n)), chi_a=chi, chi_b=chi,
                chi_w=_log_int(rng, 2, 8), chi=chi, tol=1e-12)


# ---------------------------------------------------------------- inputs
def _phys(case):
    if "phys" in case:
        return [int(p) for p in case["phys"].split(",")]
    bits = case["grid"].bit_length() - 1
    return [2] * (3 * bits) if case["binary"] else [8] * bits


def _bonds(phys, chi):
    n = len(phys)
    b = [1] * (n + 1)
    for i in range(1, n):
        b[i] = min(math.prod(phys[:i]), math.prod(phys[i:]), chi)
    return b


def _packed(cores):
    offs, pos = [], 0
    for c in cores:
        offs.append(pos)
        pos += c.numel()
    data = torch.cat([c.reshape(-1) for c in cores]).contiguous()
    return T.PackedTT(data, [c.shape[1] for c in cores], [1] + [c.shape[2] for c in cores], offs)


def _random_train(phys, chi, gen):
    """Gaussian cores whose bonds carry a slowly falling power-law weight."""
    b = _bonds(phys, chi)
    cores = []
    for i, d in enumerate(phys):
        c = torch.randn((b[i], d, b[i + 1]), generator=gen, dtype=F64, device="cuda") / math.sqrt(b[i] * d)
        if i + 1 < len(phys):
            c = c * torch.arange(1, b[i + 1] + 1, dtype=F64, device="cuda") ** -0.5 * math.sqrt(b[i + 1]) / 2
        cores.append(c)
    return _packed(cores)


def _field(n, gen):
    """One component of a random-phase turbulence field (|u_k| ~ k^(-11/6)
    with a sigmoid cut-off at n / 8, unit RMS) in the interleaved-bit order of
    the quantics encoding, flattened."""
    phase = torch.angle(torch.fft.rfftn(torch.randn((n, n, n), generator=gen, dtype=F64, device="cuda")))
    k1 = torch.fft.fftfreq(n, 1.0 / n, dtype=F64, device="cuda")
    kr = torch.fft.rfftfreq(n, 1.0 / n, dtype=F64, device="cuda")
    k = torch.sqrt(k1[:, None, None] ** 2 + k1[None, :, None] ** 2 + kr[None, None, :] ** 2)
    amp = torch.where((k > 0) & (k <= n / 2), k.clamp_min(1.0) ** (-11.0 / 6.0), 0.0)
    amp = amp / (1.0 + torch.exp((k - n / 8) * (16.0 / n)))
    u = torch.fft.irfftn(torch.polar(amp, phase), s=(n, n, n))
    u = u / u.square().mean().sqrt()
    # bits of x, y, z interleaved, most significant first: one site at a time
    bits = n.bit_length() - 1
    u = u[None]
    for _ in range(bits):
        m = u.shape[1] // 2
        u = u.reshape(-1, 2, m, 2, m, 2, m).permute(0, 1, 3, 5, 2, 4, 6).reshape(-1, m, m, m)
    return u.reshape(-1)


def _compress(field, phys, chi):
    """Left-to-right TT-SVD through the Gram matrix of each unfolding's smaller side."""
    cores, rest, rl = [], field, 1
    for d in phys[:-1]:
        mat = rest.reshape(rl * d, -1)
        m, n = mat.shape
        r = min(m, n, chi)
        if m <= n:
            u = torch.linalg.eigh(mat @ mat.T)[1][:, -r:].flip(1).contiguous()
            rest = u.T @ mat
        else:
            v = torch.linalg.eigh(mat.T @ mat)[1][:, -r:].flip(1).contiguous()
            u = mat @ v
            s = torch.linalg.norm(u, dim=0)
            u = u / torch.where(s > 0, s, 1.0)
            rest = s[:, None] * v.T
        cores.append(u.reshape(rl, d, r))
        rl = r
    cores.append(rest.reshape(rl, phys[-1], 1))
    return _packed(cores)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    phys = _phys(case)
    if case["kind"] == "batch":
        f = [_field(case["grid"], gen) for _ in range(3)]
        chis = [int(c) for c in case["chis"].split(",")]
        return [(_compress(f[p % 3], phys, c), _compress(f[p // 3], phys, c)) for p, c in enumerate(chis)], chis
    if case.get("data") == "field":
        return [_compress(_field(case["grid"], gen), phys, c) for c in (case["chi_a"], case["chi_b"])]
    chis = (case["chi_a"], case["chi_b"]) + ((case["chi_w"],) if "chi_w" in case else ())
    return [_random_train(phys, c, gen) for c in chis]


def prepare(case, seed):
    st = dict(case=case, inputs=_inputs(case, seed), ws=T.Workspace())
    if case["kind"] == "batch":
        st["ws"] = [T.Workspace() for _ in st["inputs"][0]]
    if case["kind"] == "loss":
        A, B, W = st["inputs"]
        for t in (A, B):
            t.data.requires_grad_(True)
    return st


# ---------------------------------------------------------------- the pass
def _values(cores):
    """The train on its whole grid (the products of its two halves)."""
    half = len(cores) // 2
    left = cores[0].reshape(-1, cores[0].shape[2])
    for c in cores[1:half]:
        left = (left @ c.reshape(c.shape[0], -1)).reshape(-1, c.shape[2])
    right = cores[-1].reshape(cores[-1].shape[0], -1)
    for c in cores[half:-1][::-1]:
        right = (c.reshape(-1, c.shape[2]) @ right).reshape(c.shape[0], -1)
    return (left @ right).reshape(-1)


def _read(train):
    return {"values": _values(train.cores()), "bonds": torch.tensor(train.bonds)}


def run(state):
    c, ws = state["case"], state["ws"]
    if c["kind"] == "multiply":
        A, B = state["inputs"]
        C, _ = T.multiply(A, B, c["chi"], c["tol"], workspace=ws, svd_mode=c["svd"])
        return _read(C)
    if c["kind"] == "fit":
        A, B = state["inputs"]
        C, _ = T.conventional(A, B, c["chi"], c["tol"], workspace=ws)
        return _read(C)
    if c["kind"] == "batch":
        pairs, chis = state["inputs"]
        return [_read(C) for C, _ in T.multiply_batch(pairs, chis, c["tol"], streams=c["streams"], workspaces=ws)]
    A, B, W = state["inputs"]
    if c["kind"] == "grad":
        value, dA, dB = T.inner_grad(W, A, B, contract_precision=c["prec"], workspace=ws)
        return {"value": value, "dA": dA.data, "dB": dB.data}
    loss = T.ttm_inner_loss(W, A, B, c["chi"], c["tol"])
    dA, dB = torch.autograd.grad(loss, (A.data, B.data))
    return {"value": loss.detach(), "dA": dA, "dB": dB}


# ---------------------------------------------------------------- its work
def _size(phys, chi):
    b = _bonds(phys, chi)
    return sum(b[i] * d * b[i + 1] for i, d in enumerate(phys))


def _product_work(phys, ca, cb, chi, grid=True):
    """Bytes and flops of one product: both trains read, the product's train
    (and its grid values) written; every merge and contraction of the swap
    schedule, and per swap the two products that project onto the kept rank."""
    n = len(phys)
    ba, bb = _bonds(phys, ca), _bonds(phys, cb)
    flops = 0.0
    for j in range(n - 2, -1, -1):
        for p in range(n - 1, j, -1):
            dl = ba[p] if p == j + 1 else min(chi, math.prod(phys[j + 1:p]) * ba[j + 1], math.prod(phys[p:]) * phys[j])
            dm = min(chi, math.prod(phys[p:])) if p < n - 1 else bb[j + 1]
            dr = 1 if p == n - 1 else min(chi, math.prod(phys[p + 1:]))
            m, k = dl * phys[j], phys[p] * dr
            flops += 2.0 * m * k * dm + 4.0 * m * k * min(chi, m, k)
        flops += 2.0 * phys[j] * ba[j] * ba[j + 1] * min(chi, bb[j])
    out = math.prod(phys) if grid else 0
    if grid:
        h = n // 2
        flops += 2.0 * out * min(chi, math.prod(phys[:h]), math.prod(phys[h:]))
    return 8.0 * (_size(phys, ca) + _size(phys, cb) + _size(phys, chi) + out), flops


def _grad_work(phys, ca, cb, cw):
    a, b, w = (_bonds(phys, c) for c in (ca, cb, cw))
    flops = 0.0
    for i, d in enumerate(phys):  # right sweep, then T1, T2, both gradients, the next left environment
        one = 2.0 * d * (w[i] * w[i + 1] * a[i] * b[i] + w[i + 1] * a[i] * a[i + 1] * b[i]
                         + w[i + 1] * a[i + 1] * b[i] * b[i + 1])
        two = 2.0 * d * (w[i + 1] * a[i + 1] * b[i] * b[i + 1] + w[i + 1] * a[i] * a[i + 1] * b[i])
        flops += 2 * one + two
    return 8.0 * (2 * _size(phys, ca) + 2 * _size(phys, cb) + _size(phys, cw)), flops


def work(case):
    phys = _phys(case)
    if case["kind"] == "multiply":
        b, f = _product_work(phys, case["chi_a"], case["chi_b"], case["chi"])
    elif case["kind"] == "batch":
        each = [_product_work(phys, c, c, c) for c in (int(x) for x in case["chis"].split(","))]
        b, f = (sum(v) for v in zip(*each))
    elif case["kind"] == "grad":
        b, f = _grad_work(phys, case["chi_a"], case["chi_b"], case["chi_w"])
    elif case["kind"] == "loss":
        b, f = _product_work(phys, case["chi_a"], case["chi_b"], case["chi"], grid=False)
        # the backward pass undoes the forward pass's products, two for each
        f = 3 * f + _grad_work(phys, case["chi"], 1, case["chi_w"])[1]
        b += 8.0 * (_size(phys, case["chi_a"]) + _size(phys, case["chi_b"]) + _size(phys, case["chi_w"]))
    else:  # one sweep in each direction: the environments and the projected core at every site
        b, f = _product_work(phys, case["chi_a"], case["chi_b"], case["chi"])
        a, bb, c = (_bonds(phys, case[k]) for k in ("chi_a", "chi_b", "chi"))
        f = 2.0 * math.prod(phys) * case["chi"]
        for i, d in enumerate(phys):
            f += 2 * 2.0 * d * (c[i] * a[i] * bb[i] * bb[i + 1] + c[i] * a[i] * bb[i + 1] * a[i + 1]
                                + c[i] * a[i + 1] * bb[i + 1] * c[i + 1])
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- in 64 bits, by LAPACK
def _host(train):
    return [c.detach().cpu().numpy() for c in train.cores()]


def _cut(s, tol, cap):
    """The smallest rank whose discarded weight is below tol of the total, at most cap."""
    tail = np.append(np.cumsum((s ** 2)[::-1])[::-1], 0.0)
    return min(next(k for k in range(1, len(s) + 1) if tail[k] < tol * tail[0] or tail[k] == 0), cap)


def _right(core, nxt):
    q, r = np.linalg.qr(core.reshape(-1, core.shape[2]))
    return q.reshape(core.shape[0], core.shape[1], -1), np.tensordot(r, nxt, axes=(1, 0))


def _plain_product(A, B, chi, tol):
    """The truncated product, step by step: the second train reversed, each
    of its carriages swapped leftwards to its partner and joined with it, and
    one truncating sweep at the end."""
    n = len(A)
    A, B = list(A), list(B)
    for t in (A, B):
        for i in range(n - 1):
            t[i], t[i + 1] = _right(t[i], t[i + 1])
    B = [b.transpose(2, 1, 0) for b in B]

    def join(a, b):
        return np.stack([a[:, s] @ b[:, s] for s in range(a.shape[1])], axis=1)

    P = [None] * n
    P[-1] = join(A[-1], B[-1])
    for j in range(n - 2, -1, -1):
        for p in range(j + 1, n - 1):
            P[p], P[p + 1] = _right(P[p], P[p + 1])
        x = B[j]
        for p in range(n - 1, j, -1):
            m = np.tensordot(P[p], x, axes=(2, 0)).transpose(0, 2, 1, 3)  # [left, moved, fixed, right]
            u, s, vt = np.linalg.svd(m.reshape(m.shape[0] * m.shape[1], -1), full_matrices=False)
            r = _cut(s, tol, chi)
            x = (u[:, :r] * s[:r]).reshape(m.shape[0], m.shape[1], r)
            P[p] = vt[:r].reshape(r, m.shape[2], m.shape[3])
        P[j] = join(A[j], x)
    for i in range(n - 1):
        u, s, vt = np.linalg.svd(P[i].reshape(-1, P[i].shape[2]), full_matrices=False)
        r = _cut(s, tol, chi)
        P[i], P[i + 1] = (u[:, :r].reshape(P[i].shape[0], -1, r),
                          np.tensordot(s[:r, None] * vt[:r], P[i + 1], axes=(1, 0)))
    return P


def _plain_inner(W, A, B):
    """<W, A*B>, site by site (torch, differentiable)."""
    e = torch.ones((1, 1, 1), dtype=F64, device=W[0].device)
    for w, a, b in zip(W, A, B):
        t = torch.einsum("wab,wsx->absx", e, w)
        e = sum(torch.einsum("abx,ay,bz->xyz", t[:, :, s], a[:, s], b[:, s]) for s in range(a.shape[1]))
    return e.reshape(())


def _torch_values(P):
    return _values([torch.from_numpy(np.ascontiguousarray(c)) for c in P])


def exact(case, seed):
    if case["kind"] == "fit":
        return None  # an iteration stopped by its sweep limit has no value of its own
    if case["kind"] == "batch":
        pairs, chis = _inputs(case, seed)
        return [{"values": _torch_values(_plain_product(_host(a), _host(b), c, case["tol"])), "bonds": None}
                for (a, b), c in zip(pairs, chis)]
    if case["kind"] == "multiply":
        if max(_phys(case)) * case["chi"] > 1100:
            return None  # LAPACK's SVDs alone take longer than 20 seconds
        A, B = _inputs(case, seed)
        return {"values": _torch_values(_plain_product(_host(A), _host(B), case["chi"], case["tol"])), "bonds": None}
    A, B, W = _inputs(case, seed)
    if case["kind"] == "grad":
        for t in (A, B):
            t.data.requires_grad_(True)
        value = _plain_inner(W.cores(), A.cores(), B.cores())
        dA, dB = torch.autograd.grad(value, (A.data, B.data))
        return {"value": float(value), "dA": dA, "dB": dB}
    C = _plain_product(_host(A), _host(B), case["chi"], case["tol"])
    ones = [np.ones((1, c.shape[1], 1)) for c in C]
    value = _plain_inner(*([torch.from_numpy(np.ascontiguousarray(c)) for c in t] for t in (_host(W), C, ones)))
    return {"value": value, "dA": None, "dB": None}
