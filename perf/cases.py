"""The timed workloads of the library: what a training program asks of it, from one call over a few
small pages to a whole billion-parameter step.

Every case goes through the public binding (`paper_2303_02868_amd`), on the default stream, with
library-owned pools as a program creates them.  The kinds:

  step     apm_page_adamw_step / apm_page_adamw_step_noalloc: gradients born in pages
  fused    apm_page_adamw_step_fused: gradients read from, bf16 parameters written to tensors
  delayed  apm_step_delayed (+ apm_delayed_accumulate for further micro-batches)
  pack     apm_pack_tensors (tensors -> pages)
  unpack   apm_unpack (pages -> tensors)
  stream   apm_streamer_step: fp32 state in pinned host memory

Models are GPT-style tensor lists (two embeddings, per layer two norms and four matrices with
biases, ffn = 4 * width), mixture-of-experts lists (per layer a dense attention part, a router and
`experts` two-matrix experts) or one flat tensor of `params` elements.
"""
import math

import numpy as np
import torch

import paper_2303_02868_amd as apm

DEV = "cuda:0"
STEP0 = 1000     # the training step the synchronous kinds resume at: moments are warm
LR, B1, B2, EPS, WD = 1e-4, 0.9, 0.999, 1e-8, 0.01


# ---- the cases --------------------------------------------------------------------------------

def listed():
    return [
        # the smallest job: eight quarter-size pages of one tensor, no clipping; latency and launches
        {"name": "step_8_pages", "kind": "step", "params": 8 * 262144, "page": 262144, "clip": 0.0,
         "order": "run", "entry": "step"},
        # a small ragged model trained with clipping and norm monitoring: a few dozen tiny pages
        {"name": "fused_small_ragged", "kind": "fused", "layers": 4, "width": 264, "vocab": 5003, "ctx": 512,
         "page": 65536, "clip": 1.0, "skip": False, "subset": False},
        # the 124 M shape, plain AdamW: ordinary single-GPU training
        {"name": "fused_124m", "kind": "fused", "layers": 12, "width": 768, "vocab": 50257, "ctx": 1024,
         "page": 1 << 20, "clip": 0.0, "skip": False, "subset": False},
        # the 1.3 B shape with per-page clipping: the headline step, the largest call here
        {"name": "fused_1p3b_clip", "kind": "fused", "layers": 24, "width": 2048, "vocab": 50257, "ctx": 2048,
         "page": 1 << 20, "clip": 1.0, "skip": False, "subset": False},
        # gradients born in pages, updated in the order the backward pass finishes them (last page
        # first), odd width, clipping
        {"name": "step_backward_order", "kind": "step", "layers": 8, "width": 1001, "vocab": 30011, "ctx": 777,
         "page": 1 << 20, "clip": 1.0, "order": "reversed", "entry": "step"},
        # mixture of experts, an eighth of the experts active, the library finds the untouched pages
        {"name": "moe_skip", "kind": "fused", "layers": 2, "width": 1024, "experts": 64, "active": 8,
         "page": 1 << 20, "clip": 0.0, "skip": True, "subset": False},
        # the same model when the program knows its routing and lists the touched pages itself
        {"name": "moe_listed_pages", "kind": "fused", "layers": 2, "width": 1024, "experts": 64, "active": 8,
         "page": 1 << 20, "clip": 0.0, "skip": False, "subset": True},
        # one-step-stale update of a 24-layer model: hand over a gradient, apply the previous one
        {"name": "delayed_24_layers", "kind": "delayed", "layers": 24, "width": 1024, "vocab": 50257, "ctx": 1024,
         "page": 1 << 20, "clip": 1.0, "micro": 1},
        # the same with four micro-batches accumulated into the buffered gradient
        {"name": "delayed_accumulate", "kind": "delayed", "layers": 12, "width": 768, "vocab": 50257, "ctx": 1024,
         "page": 1 << 20, "clip": 0.0, "micro": 4},
        # bf16 gradients of an odd-width model, views of one flat buffer (any alignment), into pages
        {"name": "pack_bf16_flat_views", "kind": "pack", "layers": 10, "width": 923, "vocab": 20011, "ctx": 1024,
         "page": 1 << 20, "dtype": "bf16", "flat": True},
        # fp32 masters of the 124 M shape out of their pages, as for a checkpoint
        {"name": "unpack_f32_124m", "kind": "unpack", "layers": 12, "width": 768, "vocab": 50257, "ctx": 1024,
         "page": 1 << 20, "dtype": "f32", "flat": False},
        # fp32 state in pinned host memory, the staged pipeline (the direct mode is among draw()'s)
        {"name": "stream_staged_124m", "kind": "stream", "layers": 12, "width": 768, "vocab": 50257, "ctx": 1024,
         "page": 1 << 20, "clip": 1.0, "mode": "staged"},
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _gpt(rng, lo, hi):
    n = _log_between(rng, lo, hi)
    layers = rng.randint(1, 24)
    width = max(24, min(4096, int(math.sqrt(n / (12 * layers)))))
    if rng.random() < 0.5:
        width -= width % 8
    return {"layers": layers, "width": width, "vocab": _log_between(rng, 500, 50257), "ctx": rng.randint(64, 2048)}


def draw(rng):
    """One more case of the ranges above (host-resident models are the smaller ones: a pass over
    PCIe costs a hundred times a pass over HBM)."""
    kind = rng.choice(["step", "fused", "fused", "moe", "delayed", "pack", "unpack", "stream"])
    page = rng.choice([65536, 262144, 1 << 20, 1 << 20])
    clip = rng.choice([0.0, 1.0, 0.05])
    if kind == "moe":
        skip = rng.random() < 0.5
        width = rng.choice([256, 320, 500, 512, 768, 1000, 1024])
        return {"kind": "fused", "layers": rng.randint(1, 2), "width": width, "experts": rng.randint(8, 64),
                "active": rng.randint(1, 8), "page": page, "clip": clip, "skip": skip, "subset": not skip}
    if kind == "step":
        c = _gpt(rng, 1 << 19, 5 * 10 ** 8)
        return dict(c, kind=kind, page=page, clip=clip, order=rng.choice(["run", "reversed"]),
                    entry="step") if rng.random() < 0.6 else dict(c, kind=kind, page=page, clip=clip, order="run",
                                                                  entry="noalloc")
    if kind == "fused":
        return dict(_gpt(rng, 1 << 19, 8 * 10 ** 8), kind=kind, page=page, clip=clip, skip=False, subset=False)
    if kind == "delayed":
        return dict(_gpt(rng, 1 << 19, 4 * 10 ** 8), kind=kind, page=page, clip=clip, micro=rng.choice([1, 1, 2, 4]))
    if kind == "stream":
        return dict(_gpt(rng, 1 << 21, 10 ** 8), kind=kind, page=1 << 20, clip=clip,
                    mode=rng.choice(["direct", "staged"]))
    return dict(_gpt(rng, 1 << 19, 5 * 10 ** 8), kind=kind, page=page, dtype=rng.choice(["bf16", "f32"]),
                flat=rng.random() < 0.5)


# ---- models, their layout in pages, their seeded values ----------------------------------------

def _numels(case):
    """(numel of every tensor, expert number or -1 of every tensor, layer of every tensor)"""
    if "params" in case:
        return [case["params"]], [-1], [0]
    d, out, expert, layer = case["width"], [], [], []

    def add(n, l, e=-1):
        out.append(n)
        layer.append(l)
        expert.append(e)

    if "experts" in case:
        for l in range(case["layers"]):
            for n in (d, d, 3 * d * d, 3 * d, d * d, d, d, d, d * case["experts"]):
                add(n, l)
            for e in range(case["experts"]):
                add(4 * d * d, l, e)
                add(4 * d * d, l, e)
        return out, expert, layer
    add(case["vocab"] * d, -1)
    add(case["ctx"] * d, -1)
    for l in range(case["layers"]):
        for n in (d, d, 3 * d * d, 3 * d, d * d, d, d, d, 4 * d * d, 4 * d, 4 * d * d, d):
            add(n, l)
    add(d, -1)
    add(d, -1)
    return out, expert, layer


def _plan(numels, E):
    """The documented packing rule: [(tensor, tensor_off, page, page_off, n)], pages."""
    segs, n_pages, open_at = [], 0, None     # open_at: (page, first free element) that admits a second tenant
    for t, n in enumerate(numels):
        if n == 0:
            continue
        if n < E:
            segs.append((t, 0, n_pages, 0, n))
            n_pages += 1
            continue
        done = 0
        if open_at is not None:
            page, off = open_at
            done = min(n, E - off)
            segs.append((t, 0, page, off, done))
            open_at = None
        while done < n:
            k = min(E, n - done)
            segs.append((t, done, n_pages, 0, k))
            free = (k + 7) // 8 * 8
            open_at = (n_pages, free) if free < E else None
            n_pages += 1
            done += k
    return segs, n_pages


class _Model:
    def __init__(self, case, seed):
        self.case, self.E = case, case["page"]
        self.numels, self.expert, self.layer = _numels(case)
        self.segs, self.n_pages = _plan(self.numels, self.E)
        align = 1 if case.get("flat") else 256  # allocations of their own start on 512 bytes
        self.off, at = [], 0
        for n in self.numels:
            self.off.append(at)
            at += -(-n // align) * align
        self.total = at
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(seed)
        self.active = [True] * len(self.numels)
        if "experts" in case:
            r = np.random.RandomState(seed % (1 << 32))
            on = [set(r.permutation(case["experts"])[:min(case["active"], case["experts"])].tolist())
                  for _ in range(case["layers"])]
            self.active = [e < 0 or e in on[l] for e, l in zip(self.expert, self.layer)]

    def params(self):
        return torch.randn(self.total, generator=self.gen, device=DEV).mul_(0.02)

    def momentum(self):
        return torch.randn(self.total, generator=self.gen, device=DEV).mul_(3e-4)

    def variance(self):
        return torch.rand(self.total, generator=self.gen, device=DEV).mul_(1e-6).add_(5e-7)

    def grad(self):
        g = torch.randn(self.total, generator=self.gen, device=DEV).mul_(1e-3).bfloat16()
        for o, n, on in zip(self.off, self.numels, self.active):
            if not on:
                g[o:o + n] = 0
        return g

    def tensors(self, flat):
        size, base = flat.element_size(), flat.data_ptr()
        kind = apm.APM_BF16 if flat.dtype == torch.bfloat16 else apm.APM_F32
        return apm.make_tensors(self.numels, kind, [base + o * size for o in self.off])

    def to_pages(self, flat, dtype=None):
        out = torch.zeros(self.n_pages, self.E, dtype=dtype or flat.dtype, device=DEV)
        for t, t_off, page, off, n in self.segs:
            out[page, off:off + n] = flat[self.off[t] + t_off:self.off[t] + t_off + n]
        return out

    def to_flat(self, pages):
        out = torch.zeros(self.total, dtype=pages.dtype, device=DEV)
        for t, t_off, page, off, n in self.segs:
            out[self.off[t] + t_off:self.off[t] + t_off + n] = pages[page, off:off + n]
        return out

    def touched_pages(self):
        return sorted({page for t, _, page, _, _ in self.segs if self.active[t]})


class _Region:
    """A library-owned class region as an array torch can wrap (it keeps the pool alive)."""

    def __init__(self, pool, state, n_pages):
        size, self.pool = (4 if state <= apm.APM_V32 else 2), pool
        self.__cuda_array_interface__ = {
            "shape": (n_pages, pool.desc.page_elems), "typestr": "<f4" if size == 4 else "<i2",
            "data": (apm.apm_pool_state_ptr(pool, state), False), "version": 3}

    @staticmethod
    def view(pool, state, n_pages):
        t = torch.as_tensor(_Region(pool, state, n_pages), device=DEV)
        return t if state <= apm.APM_V32 else t.view(torch.bfloat16)


# ---- what a program has in hand ----------------------------------------------------------------

def _hyper(case):
    return apm.make_hyper(LR, B1, B2, EPS, WD, case.get("clip", 0.0),
                          apm.APM_SKIP_UNTOUCHED if case.get("skip") else apm.APM_SKIP_NONE)


def _fill(pool, model, states):
    """Masters and moments into their pages, as a program does when it resumes."""
    for st in states:
        flat = (model.params, model.momentum, model.variance)[st]()
        apm.apm_pack_tensors(pool, st, model.tensors(flat), len(model.numels))
        torch.cuda.synchronize()
        del flat


def prepare(case, seed):
    m = _Model(case, seed)
    n_t, kind = len(m.numels), case["kind"]
    s = {"case": case, "m": m, "n_t": n_t, "t": STEP0, "hyper": _hyper(case)}
    if kind in ("pack", "unpack"):
        bf16 = case["dtype"] == "bf16"
        st = (apm.APM_G16 if kind == "pack" else apm.APM_P16) if bf16 else apm.APM_P32
        pool = apm.apm_pool_create(apm.APM_DEV_GPU, m.E, m.n_pages, state_mask=1 << st)
        flat = m.grad() if bf16 else m.params()
        s.update(pool=pool, state=st, flat=flat, list=m.tensors(flat), pages=_Region.view(pool, st, m.n_pages))
        if kind == "unpack":
            apm.apm_pack_tensors(pool, st, s["list"], n_t)
            s["flat"] = torch.zeros_like(flat)
            s["list"] = m.tensors(s["flat"])
        else:
            apm.apm_pool_set_layout(pool, s["list"], n_t)
        torch.cuda.synchronize()
        return s

    s["norm"] = torch.zeros(m.n_pages, device=DEV) if case.get("clip", 0.0) > 0 else None
    if kind == "stream":
        host = {st: torch.empty(m.n_pages, m.E, pin_memory=True) for st in (0, 1, 2)}
        for st in host:
            host[st].copy_(m.to_pages((m.params, m.momentum, m.variance)[st]()))
        hp = apm.apm_pool_create(apm.APM_DEV_HOST, m.E, m.n_pages, state_mask=apm.FP32_STATES,
                                 flags=apm.APM_POOL_NO_ZERO, base=host)
        dp = apm.apm_pool_create(apm.APM_DEV_GPU, m.E, m.n_pages, state_mask=apm.B16_STATES)
        g = m.grad()
        apm.apm_pack_tensors(dp, apm.APM_G16, m.tensors(g), n_t)
        torch.cuda.synchronize()
        st = apm.apm_streamer_create(hp, dp, min(16, m.n_pages), 3)
        apm.apm_streamer_set_mode(st, apm.APM_STREAM_STAGED if case["mode"] == "staged" else apm.APM_STREAM_DIRECT, 0, 0)
        s.update(streamer=st, host=host, p16=_Region.view(dp, apm.APM_P16, m.n_pages))
        return s

    mask = apm.ALL_STATES if kind == "step" else apm.ALL_STATES & ~(1 << apm.APM_G16)
    mask = apm.FP32_STATES if kind == "fused" else mask
    pool = apm.apm_pool_create(apm.APM_DEV_GPU, m.E, m.n_pages, state_mask=mask)
    _fill(pool, m, (0, 1, 2))
    s["pool"] = pool
    s["out"] = {n: _Region.view(pool, st, m.n_pages) for n, st in (("p", 0), ("m", 1), ("v", 2))}
    if kind != "fused":
        s["out"]["p16"] = _Region.view(pool, apm.APM_P16, m.n_pages)
    if s["norm"] is not None:
        s["out"]["norm"] = s["norm"]
    if kind == "step":
        g = m.grad()
        apm.apm_pack_tensors(pool, apm.APM_G16, m.tensors(g), n_t)
        s["pages"] = list(range(m.n_pages))[::-1] if case["order"] == "reversed" else None
    elif kind == "fused":
        s["g"], s["q"] = m.grad(), torch.zeros(m.total, dtype=torch.bfloat16, device=DEV)
        s["g_list"], s["q_list"] = m.tensors(s["g"]), m.tensors(s["q"])
        s["pages"] = m.touched_pages() if case["subset"] else None
        s["n_pages"] = len(s["pages"]) if case["subset"] else m.n_pages
        s["skipped"] = torch.zeros(m.n_pages, dtype=torch.uint8, device=DEV) if case["skip"] else None
        s["out"]["p16"] = s["q"]
        if case["skip"]:
            s["out"]["skipped"] = s["skipped"]
    else:
        apm.apm_delayed_set_outputs(pool, s["norm"], None)
        s["g"] = [m.to_pages(m.grad()) for _ in range(case["micro"])]
        _hand_over(s)
    torch.cuda.synchronize()
    return s


def _hand_over(s):
    """One iteration's gradient: the first micro-batch is handed over (the previous iteration's
    gradient is applied), the others are added to it."""
    n = s["m"].n_pages
    apm.apm_step_delayed(s["pool"], None, n, s["g"][0], s["hyper"])
    for g in s["g"][1:]:
        apm.apm_delayed_accumulate(s["pool"], None, n, g)


def run(s):
    case, kind, m = s["case"], s["case"]["kind"], s["m"]
    s["t"] += 1
    if kind == "pack":
        apm.apm_pack_tensors(s["pool"], s["state"], s["list"], s["n_t"])
        return s["pages"]
    if kind == "unpack":
        apm.apm_unpack(s["pool"], s["state"], s["list"], s["n_t"])
        return s["flat"]
    if kind == "stream":
        apm.apm_streamer_step(s["streamer"], s["t"], s["hyper"], s["norm"], None)
        out = {"p": s["host"][0], "m": s["host"][1], "v": s["host"][2], "p16": s["p16"]}
        if s["norm"] is not None:
            out["norm"] = s["norm"]
        return out
    if kind == "delayed":
        _hand_over(s)
    elif kind == "fused":
        apm.apm_page_adamw_step_fused(s["pool"], s["pages"], s["n_pages"], s["t"], s["hyper"], s["g_list"], s["q_list"],
                                      s["n_t"], s["norm"], s["skipped"])
    elif case["entry"] == "noalloc":
        apm.apm_page_adamw_step_noalloc(s["pool"], m.n_pages, s["t"], s["hyper"], s["norm"], None)
    else:
        apm.apm_page_adamw_step(s["pool"], s["pages"], m.n_pages, s["t"], s["hyper"], s["norm"], None)
    return s["out"]


# ---- what a pass cannot do without --------------------------------------------------------------

def work(case):
    numels, expert, _ = _numels(case)
    n, kind = sum(numels), case["kind"]
    if kind in ("pack", "unpack"):
        return {"bytes": 2 * n * (2 if case["dtype"] == "bf16" else 4), "flops": 0}
    if "experts" in case:   # every gradient is looked at if the library has to find the untouched pages
        on = sum(k for k, e in zip(numels, expert) if e < 0) + \
            sum(k for k, e in zip(numels, expert) if e >= 0) * min(case["active"], case["experts"]) // case["experts"]
        return {"bytes": 28 * on + (2 * (n - on) if case["skip"] else 0), "flops": 16 * on}
    if kind == "delayed":   # the update, the hand-over's copy, and per further micro-batch a sum
        return {"bytes": (28 + 4 + 6 * (case["micro"] - 1)) * n, "flops": (16 + case["micro"] - 1) * n}
    return {"bytes": 28 * n, "flops": (18 if case["clip"] > 0 else 16) * n}


def tolerance(case):
    """Copies are exact.  The update is fp32 with one rounding per operation; its sum of squares is
    fp64.  Between two correct orders of the arithmetic p, m, v differ by a few units in the last
    place (2^-24); a master that lies that close to the middle of two bf16 values may round the other
    way, one value in some ten thousand, by one bf16 unit (2^-8 of the value)."""
    if case["kind"] in ("pack", "unpack"):
        return "exact"
    return {"rel": 4e-5, "max": 8e-3}


# ---- the same in 64 bits -------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind in ("pack", "unpack"):
        return None
    m = _Model(case, seed)
    mean = {}
    for name, make in (("p", m.params), ("m", m.momentum), ("v", m.variance)):
        mean[name] = m.to_pages(make(), torch.float64)
    if kind == "delayed":   # micro-batches are added in bf16, one rounding each
        grads = [m.grad() for _ in range(case["micro"])]
        g16 = grads[0]
        for x in grads[1:]:
            g16 = (g16.float() + x.float()).bfloat16()
    else:
        g16 = m.grad()
    g = m.to_pages(g16, torch.float64)
    t = 1 if kind == "delayed" else STEP0 + 1
    norm, out = g.square().sum(1).sqrt(), {}
    live = torch.ones(m.n_pages, dtype=torch.bool, device=DEV)
    if case.get("skip"):
        live = (g != 0).any(1)
    elif case.get("subset"):
        live[:] = False
        live[m.touched_pages()] = True
    if case.get("clip", 0.0) > 0:
        g *= (case["clip"] / (norm + 1e-6)).clamp(max=1.0)[:, None]
    p, mo, v = mean["p"], mean["m"], mean["v"]
    p16 = torch.zeros_like(p)
    for k in live.nonzero().flatten().split(64):
        k0, k1 = int(k[0]), int(k[-1]) + 1
        k = slice(k0, k1) if k1 - k0 == len(k) else k
        gk = g[k]
        mk = B1 * mo[k] + (1 - B1) * gk
        vk = B2 * v[k] + (1 - B2) * gk * gk
        pk = p[k]
        pk = pk - LR * WD * pk - LR * (mk / (1 - B1 ** t)) / ((vk / (1 - B2 ** t)).sqrt() + EPS)
        mo[k], v[k], p[k], p16[k] = mk, vk, pk, pk
    out.update(p=p, m=mo, v=v, p16=m.to_flat(p16) if kind == "fused" else p16)
    if case.get("clip", 0.0) > 0:
        listed_pages = list(range(m.n_pages))
        if case.get("order") == "reversed":
            norm = norm.flip(0)
        elif case.get("subset"):
            listed_pages = m.touched_pages()
            norm = torch.cat([norm[listed_pages], torch.zeros(m.n_pages - len(listed_pages), device=DEV, dtype=torch.float64)])
        out["norm"] = norm
    if kind == "stream":
        for name in ("p", "m", "v"):
            out[name] = out[name].cpu()
    if case.get("skip"):
        out["skipped"] = None
    return out
