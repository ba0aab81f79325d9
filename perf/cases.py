"""The layer's work as a training program has it done, as a list of cases that can be timed and compared.

Every case is one call sequence through the public entry points (the functions of the package that carry the C ABI's
names) on inputs that are resident on the GPU:

    forward   the layer's forward alone: validation, scoring
    step      forward + backward of one (micro-)batch
    update    forward + auxiliary router losses + backward + AdamW on the trainable experts and the router
    sync      the node packs what it trained, then the copies of all nodes are merged, matrix by matrix
    warmup    the expert-merging warm-up: similarity, peers, mix of the three matrices

Shapes are the repository's own layer workloads (spes_workloads.CONFIGS), their reduced versions and token counts
around them.  Values: activations N(0,1), weights N(0,0.02), a router bias that skews the expert load where the workload
has one, tokens whose router margin is below 1e-3 drawn again (as spes_workloads does), so that the identity of the
selected experts does not hinge on rounding.
"""
import math

import numpy as np
import torch

import paper_2602_11543_amd as S

MARGIN = 1e-3
MAX_REDRAWS = 64


def _layer(name, kind, T, d, M, f, k, trainable, dtype="bf16", renorm=False, bias="none", upcycled=False, accumulate=False):
    return dict(name=name, kind=kind, T=T, d=d, M=M, f=f, k=k, trainable=trainable, dtype=dtype, renorm=renorm, bias=bias,
                upcycled=upcycled, accumulate=accumulate)


def listed():
    return [
        # the full-precision workload: a small layer in fp32 storage, bound by the latency of its kernels
        _layer("step_cfg1_f32", "step", 512, 256, 8, 512, 2, 4, dtype="f32", renorm=True),
        # a short, ragged batch with many small experts and a skewed load: odd token count, f not a multiple of a tile
        _layer("step_cfg3_small", "step", 1531, 512, 64, 352, 8, 8, bias="gumbel"),
        # scoring of one short sequence through the 7B-shaped layer: every expert's weights are read for a few rows each
        _layer("forward_7b_short", "forward", 200, 2048, 32, 2048, 4, 0),
        # one whole update of the 1B-shaped layer on a micro-batch of 2 x 2048 tokens
        _layer("update_paper_1b", "update", 4096, 768, 16, 2048, 2, 4),
        # the 2B-shaped layer, one trainable expert per node, a last batch that is not full
        _layer("step_paper_2b_ragged", "step", 3777, 1536, 16, 1280, 2, 1),
        # the 7B-shaped layer inside gradient accumulation
        _layer("micro_paper_7b", "step", 4096, 2048, 32, 2048, 4, 8, accumulate=True),
        # validation pass of the upcycled 9B-shaped layer: few wide experts, near-identical, renormalised gates
        _layer("forward_paper_9b", "forward", 4096, 2048, 8, 6144, 2, 0, renorm=True, upcycled=True),
        # the three large training workloads
        _layer("step_cfg2", "step", 16384, 2048, 64, 1024, 8, 16, bias="normal"),
        _layer("step_cfg3", "step", 32768, 4096, 64, 1408, 8, 8, bias="gumbel"),
        _layer("step_cfg4", "step", 16384, 3584, 32, 4864, 2, 8, renorm=True, upcycled=True),
        # synchronisation of 16 nodes that trained 16 of 64 experts each, and the warm-up merge of the same store
        dict(name="sync_cfg5", kind="sync", nodes=16, per_node=16, M=64, d=2048, f=1024, dtype="bf16"),
        dict(name="warmup_cfg5", kind="warmup", M=64, d=2048, f=1024, K=4, dtype="bf16"),
    ]


def _log(rng, lo, hi, step=1):
    return max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step)


def draw(rng):
    """Another case of the same ranges: 64 to 32768 tokens, 4 to 64 experts, widths of 128 to 6144 (any multiple of 8)."""
    kind = rng.choice(["step"] * 9 + ["forward"] * 4 + ["update"] * 3 + ["sync"] * 2 + ["warmup"] * 2)
    if kind in ("sync", "warmup"):
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        M = rng.choice([8, 16, 32, 64, rng.randint(5, 64)])
        while True:
            d, f = _log(rng, 256, 4096, 8), _log(rng, 256, 6144, 8)
            if M * d * f <= 64 * 2048 * 1024 * (1.0 if dtype == "bf16" else 0.5):
                break
        if kind == "warmup":
            return dict(kind=kind, M=M, d=d, f=f, K=rng.randint(1, min(8, M - 1)), dtype=dtype)
        nodes = rng.choice([2, 4, 8, 16, rng.randint(2, 16)])
        return dict(kind=kind, nodes=nodes, per_node=rng.randint(1, max(1, M // 4)), M=M, d=d, f=f, dtype=dtype)
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    while True:
        M = rng.choice([8, 16, 32, 64, 8, 16, 32, 64, rng.randint(4, 64)])
        k = min(M, rng.choice([1, 2, 2, 4, 8, 8, rng.randint(1, 8)]))
        if dtype == "f32":
            T, d, f = _log(rng, 64, 2048), _log(rng, 128, 768, 8), _log(rng, 128, 1024, 8)
        else:
            T, d, f = _log(rng, 64, 32768), _log(rng, 256, 4096, 8), _log(rng, 256, 6144, 8)
        # no dearer than the largest listed case, in operations and in memory
        if T * k * d * f <= 0.8 * 32768 * 8 * 4096 * 1408 and M * d * f <= 32 * 3584 * 4864:
            break
    upcycled = dtype == "bf16" and rng.random() < 0.2
    return dict(kind=kind, T=T, d=d, M=M, f=f, k=k, trainable=0 if kind == "forward" else rng.randint(1, max(1, M // 2)), dtype=dtype,
                renorm=upcycled or rng.random() < 0.3, bias="none" if upcycled else rng.choice(["none", "normal", "gumbel"]),
                upcycled=upcycled, accumulate=rng.random() < 0.3)


# ---------------------------------------------------------------------------- inputs


def _st(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _normal(g, shape, sigma, dtype):
    t = torch.randn(shape, device="cuda", generator=g)
    return (t.mul_(sigma) if sigma != 1.0 else t).to(dtype)


def _experts(g, case, rows, cols):
    dt = _st(case)
    if not case["upcycled"]:
        return _normal(g, (case["M"], rows, cols), 0.02, dt)
    dense = torch.randn((rows, cols), device="cuda", generator=g) * 0.02
    return torch.stack([(dense + 1e-4 * torch.randn((rows, cols), device="cuda", generator=g)).to(dt) for _ in range(case["M"])])


def _tokens(g, case, w_router, bias):
    """[T, d] tokens; one whose k+1 best scores are not MARGIN apart is drawn again."""
    k, wr = case["k"], w_router.float()
    x = _normal(g, (case["T"], case["d"]), 1.0, _st(case))
    for _ in range(MAX_REDRAWS):
        s = x.float() @ wr.t()
        if bias is not None:
            s += bias
        top = s.topk(min(k + 1, case["M"]), dim=1).values
        if top.shape[1] < 2:
            return x
        bad = torch.nonzero((top[:, :-1] - top[:, 1:]).amin(1) < MARGIN).flatten()
        if bad.numel() == 0:
            return x
        x[bad] = _normal(g, (bad.numel(), case["d"]), 1.0, _st(case))
    raise RuntimeError("tokens below the router margin are left")


def _prepare_layer(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    T, d, M, f, k, dt = case["T"], case["d"], case["M"], case["f"], case["k"], _st(case)
    w_router = _normal(g, (M, d), 1e-3 if case["upcycled"] else 0.02, dt)
    bias = None
    if case["bias"] == "normal":
        bias = torch.randn(M, device="cuda", generator=g) * 0.5
    elif case["bias"] == "gumbel":
        bias = -torch.log(-torch.log(torch.rand(M, device="cuda", generator=g).clamp_(1e-6, 1 - 1e-6)))
    st = dict(case=case, shape=S.moe_shape(T, d, M, f, k, S.SPES_F32 if case["dtype"] == "f32" else S.SPES_BF16, int(case["renorm"])),
              w_router=w_router, bias=bias, x=_tokens(g, case, w_router, bias),
              w_gate=_experts(g, case, f, d), w_up=_experts(g, case, f, d), w_down=_experts(g, case, d, f),
              y=torch.empty(T, d, dtype=dt, device="cuda"), idx=torch.empty(T, k, dtype=torch.int32, device="cuda"),
              gate=torch.empty(T, k, device="cuda"), count=torch.empty(M, dtype=torch.int32, device="cuda"))
    st["ctx"] = torch.empty(S.spes_moe_ctx_bytes(st["shape"]), dtype=torch.uint8, device="cuda")
    if case["kind"] == "forward":
        return st
    n = case["trainable"]
    mask = np.zeros(M, dtype=np.uint8)
    mask[np.random.default_rng(seed).permutation(M)[:n]] = 1
    st.update(mask=mask, dy=_normal(g, (T, d), 1.0, dt), dx=torch.empty(T, d, dtype=dt, device="cuda"),
              d_w_router=torch.zeros(M, d, device="cuda"), d_w_gate=torch.zeros(n, f, d, device="cuda"),
              d_w_up=torch.zeros(n, f, d, device="cuda"), d_w_down=torch.zeros(n, d, f, device="cuda"))
    if case["kind"] == "update":
        own = np.nonzero(mask)[0].tolist()
        st["losses"] = torch.zeros(2, device="cuda")
        st["step"] = 0
        st["opt"] = []
        for w, m, gr in ((st["w_gate"], mask, st["d_w_gate"]), (st["w_up"], mask, st["d_w_up"]), (st["w_down"], mask, st["d_w_down"]),
                         (w_router.view(1, M, d), np.ones(1, dtype=np.uint8), st["d_w_router"])):
            master = w[own].float() if w.shape[0] == M else w.float()
            st["opt"].append((w, m, master, torch.zeros_like(master), torch.zeros_like(master), gr))
    return st


def _prepare_sync(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    M, E, n, dt = case["M"], case["d"] * case["f"], case["per_node"], _st(case)
    slot = np.full((case["nodes"], M), -1, dtype=np.int32)
    for i in range(case["nodes"]):
        slot[i, np.sort(rng.permutation(M)[:n])] = np.arange(n, dtype=np.int32)
    st = dict(case=case, slot=slot, weight=(0.5 + rng.random(case["nodes"])).astype(np.float32), mask=(slot[0] >= 0).astype(np.uint8),
              count=torch.empty(M, dtype=torch.int32, device="cuda"), mats=[])
    for _ in range(3):       # gate, up and down projections; node 0 is this one and packs its experts from its own store
        base = torch.randn((M, E), device="cuda", generator=g) * 0.02
        stores = []
        for i in range(case["nodes"]):
            own = torch.from_numpy(np.nonzero(slot[i] >= 0)[0]).cuda()
            stores.append((base[own] + 1e-3 * torch.randn((n, E), device="cuda", generator=g)).to(dt))
        store = base.to(dt)
        store[torch.from_numpy(np.nonzero(slot[0] >= 0)[0]).cuda()] = stores[0]
        st["mats"].append((base.to(dt), store, [torch.empty_like(stores[0])] + stores[1:]))
    return st


def _prepare_warmup(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    M, E, K, dt = case["M"], case["d"] * case["f"], case["K"], _st(case)
    # experts that share a part of their weights in different measure, as they do after some training: the similarities
    # of an expert's peers are then apart by more than rounding
    share = (0.1 + 0.8 * torch.randperm(M, device="cuda", generator=g) / M).view(M, 1)
    src = []
    for _ in range(3):
        w = torch.randn((M, E), device="cuda", generator=g)
        w *= 0.02 * torch.sqrt(1 - share * share)
        src.append(w.add_(0.02 * share * torch.randn((1, E), device="cuda", generator=g)).to(dt))
    return dict(case=case, src=src, dst=[torch.empty_like(t) for t in src], sim=torch.empty(M, M, device="cuda"),
                nbr=torch.empty(M, K, dtype=torch.int32, device="cuda"),
                scratch=torch.empty(S.spes_warmup_scratch_bytes(M, E), dtype=torch.uint8, device="cuda"))


def prepare(case, seed):
    if case["kind"] == "sync":
        return _prepare_sync(case, seed)
    if case["kind"] == "warmup":
        return _prepare_warmup(case, seed)
    return _prepare_layer(case, seed)


# ---------------------------------------------------------------------------- one pass


def run(st):
    c = st["case"]
    dt = S.SPES_F32 if c["dtype"] == "f32" else S.SPES_BF16
    if c["kind"] == "sync":
        E = c["d"] * c["f"]
        for base, store, stores in st["mats"]:
            S.spes_expert_pack(c["M"], E, dt, store, st["mask"], stores[0], 0)
            S.spes_expert_merge(c["M"], E, dt, stores, st["slot"], st["weight"], base, st["count"])
        return dict(packed=[m[2][0] for m in st["mats"]], merged=[m[0] for m in st["mats"]], count=st["count"])
    if c["kind"] == "warmup":
        E = c["d"] * c["f"]
        S.spes_expert_warmup_merge(c["M"], dt, c["K"], 0.1, st["src"][0], E, st["src"], st["dst"], [E] * 3, st["sim"], st["nbr"], st["scratch"])
        return dict(dst=st["dst"], sim=st["sim"], nbr=st["nbr"])
    S.spes_moe_fwd(st["shape"], st["x"], st["w_router"], st["bias"], st["w_gate"], st["w_up"], st["w_down"], st["y"], st["idx"],
                   st["gate"], st["count"], st["ctx"])
    out = dict(y=st["y"], idx=st["idx"], gate=st["gate"], count=st["count"])
    if c["kind"] == "forward":
        return out
    if c["kind"] == "update":
        S.spes_moe_router_aux(st["shape"], st["ctx"], 0.01, 0.001, 1.0, st["losses"])
        out["losses"] = st["losses"]
    S.spes_moe_bwd(st["shape"], st["dy"], st["x"], st["w_router"], st["w_gate"], st["w_up"], st["w_down"], st["ctx"], st["mask"],
                   st["dx"], st["d_w_router"], st["d_w_gate"], st["d_w_up"], st["d_w_down"],
                   1 if c["accumulate"] and c["kind"] == "step" else 0)
    out.update({n: st[n] for n in ("dx", "d_w_router", "d_w_gate", "d_w_up", "d_w_down")})
    if c["kind"] == "update":
        st["step"] += 1
        # the learning rate of the first updates of a linear warm-up: the weights stay those of the case however often it runs
        for i, (w, mask, master, m, v, gr) in enumerate(st["opt"]):
            S.spes_masked_adamw(len(mask), gr.numel() // int(mask.sum()), dt, w, mask, master, m, v, gr, lr=1e-7, beta1=0.9, beta2=0.95,
                                eps=1e-8, weight_decay=0.1, step=st["step"])
            out.update({f"w{i}": w, f"master{i}": master, f"m{i}": m, f"v{i}": v})
    return out


# ---------------------------------------------------------------------------- what a pass cannot do without


def work(case):
    c, s = case, 4 if case["dtype"] == "f32" else 2
    if c["kind"] == "sync":
        E, M, n, nodes = c["d"] * c["f"], c["M"], c["per_node"], c["nodes"]
        written = M * (1 - (1 - n / M) ** nodes)          # experts that somebody trained
        return dict(bytes=3.0 * E * s * (2 * n + nodes * n + written), flops=3.0 * 3 * E * nodes * n)
    if c["kind"] == "warmup":
        E, M = c["d"] * c["f"], c["M"]
        return dict(bytes=3.0 * 2 * M * E * s, flops=1.0 * M * M * E + 3.0 * M * E * (2 * c["K"] + 1))
    T, d, M, f, k = c["T"], c["d"], c["M"], c["f"], c["k"]
    R, live = T * k, min(c["M"], c["T"] * c["k"])
    by = 3.0 * live * d * f * s + M * d * s + 2 * T * d * s + 2 * R * 4
    fl = 6.0 * R * d * f + 2.0 * T * d * M
    if c["kind"] != "forward":
        n = c["trainable"]
        grads = 3.0 * n * d * f + M * d
        by += 2 * T * d * s + grads * 4 * (2 if c["accumulate"] and c["kind"] == "step" else 1)
        fl += 6.0 * R * d * f * (1 + n / M) + 4.0 * T * d * M
        if c["kind"] == "update":
            by += grads * (28 + s)
            fl += 15.0 * grads
    return dict(bytes=by, flops=fl)


def tolerance(case):
    """About four times what each path differs by from the same computation in 64 bits (norm of the difference / largest)."""
    f32 = case["dtype"] == "f32"
    if case["kind"] == "sync":
        # an average rounded once: 1e-5 in bf16, made of single elements that fall to the neighbouring value (7.8e-3 of it)
        return {"rel": 3e-7, "max": 2e-6} if f32 else {"rel": 4e-5, "max": 8e-3}
    if case["kind"] == "warmup":
        # similarities 1.2e-7 / 3.6e-7; the mix is rounded once, as above (9e-7 in bf16)
        return {"rel": 5e-7, "max": 2e-6} if f32 else {"rel": 1e-5, "max": 8e-3}
    # fp32: 5e-7 / 7e-6, bf16: 3.4e-3 (dx) / 5.3e-2 (weight gradients of experts with a handful of rows); second moments are
    # squares of gradients and differ by up to twice as much, which both bounds hold
    return {"rel": 3e-6, "max": 3e-5} if f32 else {"rel": 1.3e-2, "max": 0.2}
