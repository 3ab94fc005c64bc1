"""The work that the framework's performance is measured on: owner optimizer steps as a training
program makes them, through the public calls of ``paper_2607_05895_amd``.

A case is a dict of plain values. ``shapes`` lists the stored matrices as ``COUNTxROWSxCOLS`` joined by
``+``; ``tails`` lists the non-matrix tensors as ``COUNTxNUMEL``. The kinds are

* ``optimizer``  ``OwnerMuon.step()``, matrices and tails, as a training loop calls it
* ``muon``       ``muon_step_t``: the Muon step on a list of matrices (bf16 or fp32 Newton-Schulz)
* ``reduce``     ``muon_step_reduce_t``: the Muon step whose gradient arrives as the span's parts
* ``ns``         ``newton_schulz_t``: the orthogonalisation of one matrix
* ``adamw``      ``adamw_step_t`` on tail tensors and embeddings
* ``shampoo``    ``shampoo_step_t``, with the preconditioners recomputed (``refresh``) or stored
* ``soap``       ``soap_step_t``, with the bases refreshed (``refresh``) or stored

The optimizer state is that of a run well under way: momentum, moments, statistics, preconditioners and
bases that belong to the gradients' distribution. For Shampoo and SOAP the gradients are
G = E_L diag(sqrt(l)) N diag(sqrt(r)) E_R^T with N normal and the spectra l, r falling as 1 / (1 + i), so
that the statistics L ~ E[G G^T] have the same falling spectrum.
"""
from __future__ import annotations

import math

import torch

from paper_2607_05895_amd import native
from paper_2607_05895_amd.optim import OwnerMuon

NS = (3.4445, -4.7750, 2.0315)

# two decoder layers of width 768 with a 3072-wide MLP; one decoder layer of width 4096 with grouped
# key/value heads and a 14336-wide MLP
GPT2_LAYERS = "8x768x768+2x3072x768+2x768x3072"
LLAMA_LAYER = "2x4096x4096+2x1024x4096+2x14336x4096+1x4096x14336"


def listed():
    return [
        # the smallest owner share: one fp32 matrix; launches and latency are all there is
        dict(name="muon_one_fp32_256x512", kind="muon", shapes="1x256x512", dtype="f32", ns="f32", steps=5),
        # a single orthogonalisation of an odd, wide matrix (a program with its own momentum)
        dict(name="ns_bf16_1000x2777", kind="ns", shapes="1x1000x2777", dtype="bf16", ns="bf16", steps=5),
        # a small model's training loop: the torch optimizer on two GPT-2-small layers with their norms
        dict(name="optimizer_gpt2_layers", kind="optimizer", shapes=GPT2_LAYERS, tails="4x768", dtype="bf16",
             ns="bf16", steps=5),
        # the main path at its full size: one of eight ranks' share of a Llama-3-8B model, 28 matrices
        dict(name="muon_llama8b_share", kind="muon", shapes="+".join([LLAMA_LAYER] * 4), dtype="bf16", ns="bf16",
             steps=5),
        # an uneven plan: matrices of many sizes, some odd, tall and wide, under the two-step setting
        dict(name="muon_uneven_share", kind="muon", shapes="1x512x1920+1x1408x640+1x2333x1001+1x1152x4480+1x3712x3072"
             "+1x2560x2560+1x777x3011+1x4736x1280+1x640x640+1x1792x3328+1x300x300+1x2048x3584", dtype="bf16",
             ns="bf16", steps=2),
        # fp32 training: the Newton-Schulz products in fp32 too
        dict(name="muon_fp32_gpt2_layer", kind="muon", shapes="4x768x768+1x3072x768+1x768x3072+1x1024x4096",
             dtype="f32", ns="f32", steps=5),
        # the owner sums the eight ranks' gradients of one Llama-3-8B layer inside its step
        dict(name="reduce8_llama_layer", kind="reduce", shapes=LLAMA_LAYER, parts=8, dtype="bf16", ns="bf16",
             steps=5),
        # the tail owner: a 128256 x 4096 embedding and the norm vectors of eight layers
        dict(name="adamw_embedding_and_norms", kind="adamw", tails="1x525336576+16x4096", dtype="bf16"),
        # Shampoo on two GPT-2-small layers: a step that recomputes the inverse roots, and one that does not
        dict(name="shampoo_refresh_gpt2_layers", kind="shampoo", shapes=GPT2_LAYERS, dtype="bf16", refresh=True),
        dict(name="shampoo_stored_gpt2_layers", kind="shampoo", shapes=GPT2_LAYERS, dtype="bf16", refresh=False),
        # SOAP: a basis refresh on one such layer; a plain step on one Llama-3-8B layer, whose 14336-long
        # sides have no basis
        dict(name="soap_refresh_gpt2_layer", kind="soap", shapes="4x768x768+1x3072x768+1x768x3072", dtype="bf16",
             refresh=True),
        dict(name="soap_stored_llama_layer", kind="soap", shapes=LLAMA_LAYER, dtype="bf16", refresh=False),
    ]


def _size(rng, lo, hi):
    """A size spread over the logarithm of lo .. hi: as it comes, or rounded to 16, 64 or 128."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    q = rng.choice((1, 1, 16, 64, 128))
    return max(lo, min(hi, (v + q - 1) // q * q))


def draw(rng):
    """Another case of the listed ones' ranges: every kind, any sizes, one matrix or several."""
    # kind, options, smallest and largest side, most matrices, most work (in the listed case's measure)
    kind, opt, lo, hi, most, cap = rng.choice((
        ("optimizer", dict(ns="bf16"), 64, 4096, 16, 1.5e13),
        ("muon", dict(ns="bf16"), 64, 8192, 12, 3e13),
        ("muon", dict(ns="bf16"), 64, 8192, 12, 3e13),
        ("muon", dict(ns="f32"), 32, 2048, 6, 5e11),
        ("reduce", dict(ns="bf16"), 128, 4096, 6, 1.5e13),
        ("ns", dict(ns="bf16"), 32, 8192, 1, 1.5e13),
        ("ns", dict(ns="f32"), 32, 2048, 1, 5e11),
        ("adamw", {}, 64, 1 << 28, 20, 4e9),
        ("shampoo", dict(refresh=True), 32, 3072, 6, 1.2e12),
        ("shampoo", dict(refresh=False), 32, 4096, 8, 1.2e12),
        ("soap", dict(refresh=True), 32, 2560, 6, 6e11),
        ("soap", dict(refresh=False), 32, 6000, 8, 4e12)))
    while True:
        case = dict(kind=kind, dtype="f32" if opt.get("ns") == "f32" else rng.choice(("bf16", "bf16", "f32")), **opt)
        if kind == "adamw":
            case["tails"] = "+".join("1x%d" % _size(rng, lo, hi) for _ in range(rng.randint(1, most)))
        else:
            dims = [(_size(rng, lo, hi), _size(rng, lo, hi)) for _ in range(rng.randint(1, most))]
            case["shapes"] = "+".join("1x%dx%d" % d for d in dims)
        if "ns" in opt:
            case["steps"] = rng.choice((2, 5, 5))
        if kind == "optimizer":
            case["tails"] = "%dx%d" % (rng.randint(1, 8), _size(rng, 64, 8192))
        if kind == "reduce":
            case["parts"] = rng.choice((2, 3, 4, 8))
        w = work(case)
        if (w["bytes"] if kind == "adamw" else w["flops"]) <= cap and w["bytes"] <= 8e9:
            return case


# ------------------------------------------------------------------------------- inputs

def _list(text):
    """The tuples of a ``COUNTxA[xB]`` list."""
    out = []
    for item in (text or "").split("+"):
        if item:
            n, *dims = (int(v) for v in item.split("x"))
            out += [tuple(dims)] * n
    return out


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


class _Draw:
    """Normal and uniform values on the GPU, from one seeded stream."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)
        self.dct = {}

    def normal(self, shape, std=1.0, dtype=torch.float32, mean=0.0):
        t = torch.empty(shape, device="cuda", dtype=torch.float32).normal_(mean, std, generator=self.gen)
        return t if dtype == torch.float32 else t.to(dtype)

    def uniform(self, shape, lo, hi):
        return torch.empty(shape, device="cuda", dtype=torch.float32).uniform_(lo, hi, generator=self.gen)

    def basis(self, d):
        """An orthogonal d x d matrix: a cosine transform, two random reflections and random signs."""
        if d not in self.dct:
            i = torch.arange(d, device="cuda", dtype=torch.int64)
            ph = ((2 * i + 1)[:, None] * i[None, :]) % (4 * d)   # the cosine's argument in quarter turns / d
            c = torch.cos(ph.to(torch.float64) * (math.pi / (2 * d))) * math.sqrt(2.0 / d)
            c[:, 0] *= math.sqrt(0.5)
            self.dct[d] = c
        q = self.dct[d]
        for _ in range(2):
            u = self.normal((d, 1)).to(torch.float64)
            u /= u.norm()
            q = q - 2.0 * u @ (u.t() @ q)
        sign = torch.where(self.uniform((d,), -1.0, 1.0) < 0, -1.0, 1.0).to(torch.float64)
        return q * sign[None, :]


def _muon_tensors(case, seed):
    """Per matrix: parameter, gradient (or its parts), momentum."""
    r, dt = _Draw(seed), _dtype(case)
    out = []
    for m, n in _list(case["shapes"]):
        p = r.normal((m, n), 0.02, dt)
        if case["kind"] == "reduce":
            g = [r.normal((m, n), 1e-3, dt) for _ in range(case["parts"])]
        else:
            g = r.normal((m, n), 1e-3, dt)
        out.append((p, g, r.normal((m, n), 1e-3)))
    return out


def _tail_tensors(case, seed):
    r, dt = _Draw(seed + 1000003), _dtype(case)
    out = []
    for (n,) in _list(case.get("tails")):
        big = n >= 1 << 20   # an embedding; the others are norm weights
        out.append((r.normal((n,), 0.02, dt, 0.0 if big else 1.0), r.normal((n,), 1e-3, dt),
                    r.normal((n,), 3e-4), r.normal((n,), 1e-3).square_().add_(1e-8)))
    return out


_TAIL_STEP = 100   # steps taken before the pass
_MAXD = 4096       # longest side that SOAP gives a basis


def _kron_tensors(case, seed):
    """Shampoo and SOAP: per matrix a dict of parameter, gradient, statistics, preconditioners or bases."""
    r, dt, soap = _Draw(seed), _dtype(case), case["kind"] == "soap"
    out = []
    for m, n in _list(case["shapes"]):
        side = []
        for d in (m, n):
            if soap and d > _MAXD:   # no basis: flat spectrum
                side.append((None, torch.ones(d, device="cuda", dtype=torch.float64)))
            else:
                lam = 1.0 / (1.0 + torch.arange(d, device="cuda", dtype=torch.float64))
                side.append((r.basis(d), lam * r.uniform((d,), 0.8, 1.2).to(torch.float64)))
        (el, ll), (er, lr) = side
        scale = 1e-3 / math.sqrt(float(ll.mean()) * float(lr.mean()))

        def colored(std):
            x = r.normal((m, n), std * scale) * (ll.sqrt()[:, None] * lr.sqrt()[None, :]).float()
            x = el.float() @ x if el is not None else x
            return x @ er.float().t() if er is not None else x

        t = dict(param=r.normal((m, n), 0.02, dt), grad=colored(1.0).to(dt))
        for name, e, lam, other in (("L", el, ll, lr), ("R", er, lr, ll)):
            if e is None:
                continue
            w = lam * (scale * scale * float(other.sum()))
            s = (e * w[None, :]) @ e.t()
            t[name] = ((s + s.t()) * 0.5).float()
            if soap:
                t["Q" + name] = e.float()
            else:
                ridge = 1e-12 + 1e-6 * float(w.norm())
                pr = (e * (w + ridge).pow(-0.25)[None, :]) @ e.t()
                t["P" + name] = ((pr + pr.t()) * 0.5).float()
        if soap:
            t["exp_avg"] = colored(0.16)
            t["exp_avg_sq"] = (ll[:, None] * lr[None, :]).float() * (scale * scale) * r.uniform((m, n), 0.5, 1.5)
        out.append(t)
    return out


_SHAMPOO = dict(lr=1e-3, weight_decay=0.01, beta=0.95, weight=0.05, eps=1e-12, eps_rel=1e-6, root_iters=20)
_SOAP = dict(lr=3e-3, weight_decay=0.01, beta1=0.95, beta2=0.95, eps=1e-8, shampoo_beta=0.95, shampoo_weight=0.05,
             step=100)
_ADAMW = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)
_MUON = dict(lr=0.02, weight_decay=0.01, momentum=0.95, lr_adjust="original")


def prepare(case, seed):
    kind = case["kind"]
    if kind == "optimizer":
        mats, tails = _muon_tensors(case, seed), _tail_tensors(case, seed)
        params = []
        for p, g, *_ in mats + tails:
            params.append(torch.nn.Parameter(p))
            params[-1].grad = g
        opt = OwnerMuon(params, ns_steps=case["steps"], ns_dtype=case["ns"], adamw_lr=_ADAMW["lr"], **_MUON)
        for q, t in zip(params, mats + tails):
            if len(t) == 3:
                opt.state[q]["momentum_buffer"] = t[2]
            else:
                opt.state[q].update(exp_avg=t[2], exp_avg_sq=t[3], step=_TAIL_STEP)
        return dict(case=case, opt=opt, out=[[t.data if i == 0 else t for i, t in enumerate((q,) + t[2:])]
                                             for q, t in zip(params, mats + tails)])
    if kind in ("muon", "reduce"):
        mats = _muon_tensors(case, seed)
        hp = native.muon_hparams(ns_steps=case["steps"], ns_dtype=case["ns"], **_MUON)
        grads = [g[0] if kind == "reduce" else g for _, g, _ in mats]
        ents = [native.muon_entry_t(p, g, mo) for (p, _, mo), g in zip(mats, grads)]
        return dict(case=case, ents=ents, hp=hp, ws=native.muon_workspace_t(ents, hp), keep=mats,
                    parts=[g for _, g, _ in mats], out=[[p, mo] for p, _, mo in mats])
    if kind == "ns":
        r, ((m, n),) = _Draw(seed), _list(case["shapes"])
        x = r.normal((m, n), 1e-3, _dtype(case))
        nsd = native.BF16 if case["ns"] == "bf16" else native.F32
        ws = torch.empty(native.mfsdp_ns_workspace_size(m, n, nsd), dtype=torch.uint8, device="cuda")
        return dict(case=case, x=x, ws=ws, res=torch.empty((m, n), dtype=torch.float32, device="cuda"))
    if kind == "adamw":
        ts = _tail_tensors(case, seed)
        return dict(case=case, ents=[native.adamw_entry_t(*t) for t in ts], keep=ts,
                    out=[[t[0], t[2], t[3]] for t in ts])
    ts = _kron_tensors(case, seed)
    if kind == "shampoo":
        ents = [native.shampoo_entry_t(t["param"], t["grad"], t["L"], t["R"], t["PL"], t["PR"]) for t in ts]
        hp = native.shampoo_hparams(refresh=case["refresh"], **_SHAMPOO)
        ws = native.shampoo_workspace_t(ents, hp)
        names = ("param", "L", "R", "PL", "PR") if case["refresh"] else ("param", "L", "R")
    else:
        ents = [native.soap_entry_t(t["param"], t["grad"], t["exp_avg"], t["exp_avg_sq"], t.get("L"), t.get("R"),
                                    t.get("QL"), t.get("QR")) for t in ts]
        hp = native.soap_hparams(refresh=case["refresh"], **_SOAP)
        ws = native.soap_workspace_t(ents, hp)
        names = ("param", "exp_avg", "exp_avg_sq", "L", "R") + (("QL", "QR") if case["refresh"] else ())
    return dict(case=case, ents=ents, hp=hp, ws=ws, keep=ts, out=[[t[k] for k in names if k in t] for t in ts])


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "optimizer":
        state["opt"].step()
    elif kind == "muon":
        native.muon_step_t(state["ents"], state["hp"], state["ws"])
    elif kind == "reduce":
        native.muon_step_reduce_t(state["ents"], state["parts"], 1.0 / case["parts"], state["hp"], state["ws"])
    elif kind == "ns":
        a, b, c = NS
        native.newton_schulz_t(state["x"], state["res"], a=a, b=b, c=c, steps=case["steps"], ns_dtype=case["ns"],
                               workspace=state["ws"])
        return state["res"]
    elif kind == "adamw":
        native.adamw_step_t(state["ents"], step=_TAIL_STEP + 1, **_ADAMW)
    elif kind == "shampoo":
        native.shampoo_step_t(state["ents"], state["hp"], state["ws"])
    else:
        native.soap_step_t(state["ents"], state["hp"], state["ws"])
    return state["out"]


# ------------------------------------------------------------------------------- needs and answers

def work(case):
    """Each input read and each output written once; symmetric products counted once."""
    kind, eb = case["kind"], 2 if case["dtype"] == "bf16" else 4
    by = fl = 0.0
    for m, n in _list(case.get("shapes")):
        k, s, l = m * n, min(m, n), max(m, n)
        if kind in ("optimizer", "muon", "reduce", "ns"):
            by += k * (2 * eb + case.get("parts", 1) * eb + 8) if kind != "ns" else k * (eb + 4)
            fl += case["steps"] * (3.0 * s * s * l + float(s) ** 3)
        elif kind == "shampoo":
            by += k * 3 * eb + (8 + 4) * (m * m + n * n)
            fl += 3.0 * (float(m) * m * n + float(n) * n * m)
            if case["refresh"]:   # an eigendecomposition's order of work per side
                fl += 10.0 * (float(m) ** 3 + float(n) ** 3)
        else:
            by += k * (3 * eb + 16)
            for d, o in ((m, n), (n, m)):
                if d <= _MAXD:
                    by += d * d * (16 if case["refresh"] else 12)
                    fl += 7.0 * d * d * o   # statistic (once), both projections, the projection back
                    if case["refresh"]:     # power step, Householder QR and its factor
                        fl += (2.0 + 8.0 / 3.0) * float(d) ** 3
    for (n,) in _list(case.get("tails")):
        by += n * (3 * eb + 16)
        fl += 12.0 * n
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """Relative errors that another correct implementation at the same precision shows: about four times
    what the library shows against 64 bits (or against another order of its sums)."""
    kind, f32 = case["kind"], case["dtype"] == "f32"
    if kind == "ns":
        return {"rel": 2e-2, "max": 0.2} if case["ns"] == "bf16" else {"rel": 2e-4, "max": 5e-3}
    if kind in ("optimizer", "muon", "reduce"):
        if case["ns"] == "f32":
            return {"rel": 1e-6, "max": 1e-4}
        return {"rel": 2e-3, "max": 0.1} if f32 else {"rel": 3e-3, "max": 0.1}
    if kind == "adamw":
        return {"rel": 1e-6, "max": 1e-4} if f32 else {"rel": 1e-4, "max": 1e-2}
    if kind == "shampoo":
        return {"rel": 3e-4, "max": 5e-2}
    return {"rel": 1e-3, "max": 0.2}


def _ns64(x, case):
    tall = x.shape[0] > x.shape[1]
    x = x.t() if tall else x
    x = x / max(float(x.norm()), 1e-7)
    a, b, c = NS
    for _ in range(case["steps"]):
        g = x @ x.t()
        x = a * x + (b * g + c * (g @ g)) @ x
    return x.t() if tall else x


def _muon64(p, g, mo, case):
    p, g, mo = p.double(), g.double(), mo.double()
    be, lr, wd = _MUON["momentum"], _MUON["lr"], _MUON["weight_decay"]
    mo = mo + (1 - be) * (g - mo)
    o = _ns64(g + be * (mo - g), case)
    m, n = p.shape
    return [p * (1 - lr * wd) - lr * math.sqrt(max(1.0, m / n)) * o, mo]


def _adamw64(p, g, m, v):
    p, g, m, v = p.double(), g.double(), m.double(), v.double()
    t, b1, b2 = _TAIL_STEP + 1, _ADAMW["beta1"], _ADAMW["beta2"]
    m = b1 * m + (1 - b1) * g
    v = b2 * v + (1 - b2) * g * g
    p = p * (1 - _ADAMW["lr"] * _ADAMW["weight_decay"])
    p = p - _ADAMW["lr"] / (1 - b1 ** t) * m / (v.sqrt() / math.sqrt(1 - b2 ** t) + _ADAMW["eps"])
    return [p, m, v]


def _root64(s):
    """(S + rho I)^(-1/4) by the coupled Newton iteration in 64 bits."""
    d = s.shape[0]
    eye = torch.eye(d, device=s.device, dtype=torch.float64)
    s = s + (_SHAMPOO["eps"] + _SHAMPOO["eps_rel"] * float(s.norm())) * eye
    z = 2.5 / float(s.norm())
    m, x = z * s, z ** 0.25 * eye
    for _ in range(40):
        if float((m - eye).abs().max()) < 1e-12:
            break
        t = (5.0 * eye - m) / 4.0
        x = x @ t
        t = t @ t
        m = t @ t @ m
        m, x = (m + m.t()) * 0.5, (x + x.t()) * 0.5
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "ns":
        ((m, n),) = _list(case["shapes"])
        return _ns64(_Draw(seed).normal((m, n), 1e-3, _dtype(case)).double(), case)
    if kind == "adamw":
        return [_adamw64(*t) for t in _tail_tensors(case, seed)]
    if kind in ("optimizer", "muon", "reduce"):
        out = []
        for p, g, mo in _muon_tensors(case, seed):
            if kind == "reduce":
                g = sum(x.double() for x in g) / case["parts"]
            out.append(_muon64(p, g, mo, case))
        return out + ([_adamw64(*t) for t in _tail_tensors(case, seed)] if kind == "optimizer" else [])
    out = []
    for t in _kron_tensors(case, seed):
        p, g = t["param"].double(), t["grad"].double()
        stat = {}
        if "L" in t:
            stat["L"] = 0.95 * t["L"].double() + 0.05 * (g @ g.t())
        if "R" in t:
            stat["R"] = 0.95 * t["R"].double() + 0.05 * (g.t() @ g)
        if kind == "shampoo":
            h = _SHAMPOO
            pl, pr = (_root64(stat[k]) if case["refresh"] else t["P" + k].double() for k in "LR")
            p = p * (1 - h["lr"] * h["weight_decay"]) - h["lr"] * (pl @ g @ pr)
            out.append([p, stat["L"], stat["R"]] + ([pl, pr] if case["refresh"] else []))
            continue
        h = _SOAP
        ql, qr = (t[k].double() if k in t else None for k in ("QL", "QR"))

        def into(x):
            x = ql.t() @ x if ql is not None else x
            return x @ qr if qr is not None else x

        gp = into(g)
        mo = h["beta1"] * t["exp_avg"].double() + (1 - h["beta1"]) * g
        v = h["beta2"] * t["exp_avg_sq"].double() + (1 - h["beta2"]) * gp * gp
        step = (into(mo) / (1 - h["beta1"] ** h["step"])) / (v.sqrt() / math.sqrt(1 - h["beta2"] ** h["step"]) + h["eps"])
        step = ql @ step if ql is not None else step
        step = step @ qr.t() if qr is not None else step
        p = p * (1 - h["lr"] * h["weight_decay"]) - h["lr"] * step
        qs = [torch.linalg.qr(stat[k] @ t["Q" + k].double())[0] for k in "LR" if k in stat] if case["refresh"] else []
        out.append([p, mo, v] + [stat[k] for k in "LR" if k in stat] + qs)
    return out
