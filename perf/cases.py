"""Workloads of this package as a user's program runs them, for timing and comparison.

Four kinds of call cover the framework's paths:

* ``step``: one draft step of ``DraftStep`` (candidates, selector, tree and mask from the
  proposer's logits), what a serving loop calls once per drafting round;
* ``head``: the LM head fused with the candidate sets, for a proposer that hands over
  hidden states instead of logits;
* ``verify``: one layer's tree attention, then the acceptance walk and the commit of the
  accepted rows (the decode direction's consumer of the tree);
* ``loss``: one training step's objective on proposer and target logits with the
  gradients (candidates first, as the objective needs them).

Sizes are those of ``synth``'s workloads, of ``bench.py`` and of the tests, or generic
ones of the same ranges.  Inputs follow ``synth``'s distributions, drawn on the GPU.
"""
import math

import torch

import paper_2609_39972_amd as ubt


def listed():
    return [
        # The smallest configuration: one chat request, short block, fp32 throughout.
        dict(name="step-b1-f32", kind="step", B=1, gamma=7, V=32000, K=4, r=32, W=3, budget=16, dtype="f32",
             feat="f32", logits="normal3"),
        # The paper's own operating point: one sequence per round, 64 candidates.
        dict(name="step-b1-k64", kind="step", B=1, gamma=15, V=151936, K=64, r=256, W=12, budget=64, dtype="bf16",
             feat="bf16", logits="zipf"),
        # Sizes that are no powers of two: odd vocabulary (rows not 16-byte aligned), K = 10.
        dict(name="step-b6-ragged", kind="step", B=6, gamma=11, V=50257, K=10, r=96, W=10, budget=48, dtype="bf16",
             feat="bf16", logits="zipf"),
        # The headline batch of a serving node.
        dict(name="step-b32-k8", kind="step", B=32, gamma=15, V=151936, K=8, r=128, W=12, budget=64, dtype="bf16",
             feat="bf16", logits="zipf"),
        # The same batch at high sampling entropy: more candidates, a larger tree.
        dict(name="step-b32-k16-entropy", kind="step", B=32, gamma=15, V=151936, K=16, r=128, W=24, budget=128,
             dtype="bf16", feat="bf16", logits="normal0.7"),
        # The paper's tree configuration on the headline batch.
        dict(name="step-b32-k64", kind="step", B=32, gamma=15, V=151936, K=64, r=256, W=12, budget=64, dtype="bf16",
             feat="bf16", logits="zipf"),
        # A full node's batch with long blocks: the largest step.
        dict(name="step-b256-k16", kind="step", B=256, gamma=31, V=151936, K=16, r=256, W=24, budget=128,
             dtype="bf16", feat="bf16", logits="zipf"),
        # One drafting block through the head (batch-1 decode).
        dict(name="head-m15", kind="head", M=15, d=2560, V=151936, K=64),
        # The drafting blocks of the headline batch through a larger head.
        dict(name="head-m480", kind="head", M=480, d=4096, V=151936, K=8),
        # Verification of one long-context request.
        dict(name="verify-b1-long", kind="verify", B=1, N=65, H=32, Hkv=8, D=128, P=16384),
        # Verification of the headline batch, contexts of many lengths.
        dict(name="verify-b32", kind="verify", B=32, N=65, H=32, Hkv=8, D=128, P=4096),
        # One training step on the headline batch.
        dict(name="loss-b32", kind="loss", B=32, gamma=15, V=151936, K=8, r=128, T=1.0, beta=0.1, dtype="bf16",
             feat="bf16"),
    ]


def _log(rng, lo, hi):
    """An integer spread evenly over the logarithm of lo..hi."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _vocab(rng):
    v = _log(rng, 32000, 151936)
    return v if rng.random() < 0.3 else v // 64 * 64  # most vocabularies are padded


def draw(rng):
    kind = rng.choice(["step", "step", "step", "head", "verify", "loss"])
    if kind == "step":
        K = rng.choice([4, 8, 8, 10, 16, 16, 24, 32, 64, 64])
        V, gamma = _vocab(rng), rng.randint(5, 31)
        f32 = rng.random() < 0.2
        B = _log(rng, 1, max(1, min(256, 256 * 31 * 151936 // (gamma * V * (2 if f32 else 1)))))
        return dict(kind="step", B=B, gamma=gamma, V=V, K=K, r=rng.choice([32, 64, 96, 128, 256]),
                    W=rng.randint(3, 24), budget=rng.randint(16, 128), dtype="f32" if f32 else "bf16",
                    feat="f32" if f32 and rng.random() < 0.5 else "bf16",
                    logits=rng.choice(["zipf", "zipf", "normal3", "normal0.7"]))
    if kind == "head":
        return dict(kind="head", M=_log(rng, 5, 480), d=rng.choice([1024, 1536, 2048, 2560, 2880, 4096]),
                    V=_vocab(rng), K=rng.choice([4, 8, 10, 16, 64]))
    if kind == "verify":
        H, Hkv = rng.choice([(32, 8), (32, 8), (16, 8), (40, 8), (16, 2), (8, 8)])
        D = rng.choice([64, 128, 128])
        P = _log(rng, 256, 32768)
        B = _log(rng, 1, max(1, min(64, 32 * 4096 * 8 * 128 // (P * Hkv * D))))
        return dict(kind="verify", B=B, N=rng.randint(17, 129), H=H, Hkv=Hkv, D=D, P=P)
    V, gamma = _vocab(rng), rng.randint(5, 31)
    f32 = rng.random() < 0.2
    return dict(kind="loss", B=_log(rng, 1, max(1, 64 * 15 * 151936 // (gamma * V * (2 if f32 else 1)))), gamma=gamma,
                V=V, K=rng.choice([4, 8, 16, 64]), r=rng.choice([32, 64, 128, 256]), T=rng.choice([0.7, 1.0]),
                beta=rng.choice([0.1, 0.5]), dtype="f32" if f32 else "bf16", feat="f32" if f32 else "bf16")


# ---- inputs -------------------------------------------------------------------------------

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _logit_rows(g, rows, V, how):
    """fp32 logit rows: i.i.d. normal, or Zipf (s = 1.1) over uniformly drawn ranks with noise
    of variance 0.5."""
    n = torch.randn(rows, V, generator=g, device="cuda")
    if how != "zipf":
        return n * float(how[6:])
    rank = torch.rand(rows, V, generator=g, device="cuda").mul_(V).floor_().add_(1.0)
    k = torch.arange(1, V + 1, dtype=torch.float64)
    return n.mul_(math.sqrt(0.5)).sub_(rank.log_().mul_(1.1)).sub_(float((k ** -1.1).sum().log()))


def _logits(g, B, gamma, V, how, dtype):
    out = torch.empty(B, gamma, V, dtype=_DT[dtype], device="cuda")
    for b in range(B):
        out[b] = _logit_rows(g, gamma, V, how)
    return out


def _selector(g, c):
    V, r, dt = c["V"], c["r"], _DT[c["feat"]]
    sd = r ** -0.5
    return dict(phi=(torch.randn(V, r, generator=g, device="cuda") * sd).to(dt),
                psi=(torch.randn(V, r, generator=g, device="cuda") * sd).to(dt),
                gate=torch.randn(c["B"], c["gamma"], r, generator=g, device="cuda").to(dt),
                anchor=torch.randint(0, V, (c["B"],), generator=g, device="cuda", dtype=torch.int32))


def _trees(seed, B, N, gamma=15):
    """Random draft trees: parents [B, N], the boolean ancestors-and-self matrix [B, N, N]."""
    g = torch.Generator()
    g.manual_seed(seed)
    parent = torch.full((B, N), -1, dtype=torch.int64)
    depth = torch.zeros(B, N, dtype=torch.int64)
    anc = torch.zeros(B, N, N, dtype=torch.bool)
    anc[:, 0, 0] = True
    u = torch.rand(B, N, 8, generator=g, dtype=torch.float64)
    rows = torch.arange(B)
    for n in range(1, N):
        p = torch.zeros(B, dtype=torch.int64)
        for t in range(8):  # the first of a few proposals that is not too deep, else the root
            q = (u[:, n, t].sqrt() * n).long()
            p = torch.where((p == 0) & (depth[rows, q] < gamma), q, p)
        parent[:, n] = p
        depth[:, n] = depth[rows, p] + 1
        anc[:, n] = anc[rows, p]
        anc[:, n, n] = True
    return parent, anc


def _pack(anc):
    B, N, _ = anc.shape
    words = (N + 31) // 32
    bits = torch.zeros(B, N, words * 32, dtype=torch.int64)
    bits[:, :, :N] = anc
    w = (bits.view(B, N, words, 32) << torch.arange(32)).sum(-1)
    return torch.where(w >= 1 << 31, w - (1 << 32), w).to(torch.int32)


def _prefix(c):
    """Context lengths of the batch: spread evenly between half of P and P."""
    B, P = c["B"], c["P"]
    return [P if B == 1 else P // 2 + (P - P // 2) * b // (B - 1) for b in range(B)]


def prepare(case, seed):
    c, g = case, _gen(seed)
    kind = c["kind"]
    if kind == "step":
        logits = _logits(g, c["B"], c["gamma"], c["V"], c["logits"], c["dtype"])
        s = _selector(g, c)
        ones = [1.0] * c["gamma"]
        step = ubt.DraftStep(c["B"], c["gamma"], c["V"], c["K"], c["W"], c["budget"], s["phi"], s["psi"], s["gate"],
                             s["anchor"], ones, ones, one_call=True, logit_dtype=_DT[c["dtype"]])
        return dict(kind=kind, logits=logits, step=step)
    if kind == "head":
        M, d, V, K = c["M"], c["d"], c["V"], c["K"]
        h = torch.randn(M, d, generator=g, device="cuda").to(torch.bfloat16)
        w = torch.empty(V, d, dtype=torch.bfloat16, device="cuda")
        for v in range(0, V, 32768):
            n = min(32768, V - v)
            w[v:v + n] = torch.randn(n, d, generator=g, device="cuda") * (3.0 * d ** -0.5)
        return dict(kind=kind, h=h, w=w, K=K, workspace=ubt.lm_head_workspace(M, d, V, K))
    if kind == "verify":
        B, N, H, Hkv, D = (c[k] for k in ("B", "N", "H", "Hkv", "D"))
        rows = c["P"] + N

        def normal(*shape):
            x = torch.empty(*shape, dtype=torch.bfloat16, device="cuda")
            for b in range(shape[0]):
                x[b] = torch.randn(*shape[1:], generator=g, device="cuda")
            return x

        parent, anc = _trees(seed, B, N)
        token = torch.stack([torch.randperm(151936, generator=g, device="cuda")[:N] for _ in range(B)]).cpu()
        target = torch.randint(0, 151936, (B, N), generator=g, device="cuda").cpu()
        follow = torch.rand(B, N, generator=g, device="cuda").cpu() < 0.8
        for n in range(N - 1, 0, -1):  # the sample at a node is often its first child's token
            for b in range(B):
                if follow[b, n]:
                    target[b, parent[b, n]] = token[b, n]
        i32 = dict(dtype=torch.int32, device="cuda")
        return dict(kind=kind, q=normal(B, N, H, D), kc=normal(B, rows, Hkv, D), vc=normal(B, rows, Hkv, D),
                    kt=normal(B, N, Hkv, D), vt=normal(B, N, Hkv, D), mask=_pack(anc).cuda(),
                    n_nodes=torch.full((B,), N, **i32), prefix=torch.tensor(_prefix(c), **i32),
                    token=token.to(**i32), parent=parent.to(**i32), target=target.to(**i32))
    logits = _logits(g, c["B"], c["gamma"], c["V"], "zipf", c["dtype"])
    target = torch.empty_like(logits)
    y = torch.empty(c["B"], c["gamma"], dtype=torch.int32, device="cuda")
    weight = torch.arange(1, 65, dtype=torch.float32, device="cuda") ** -1.1
    for b in range(c["B"]):  # the target agrees with the proposer only roughly
        target[b] = logits[b].float() + torch.randn(c["gamma"], c["V"], generator=g, device="cuda")
        pick = torch.multinomial(weight, c["gamma"], replacement=True, generator=g)
        y[b] = logits[b].float().topk(64, dim=1).indices.gather(1, pick[:, None])[:, 0]
    y[torch.rand(y.shape, generator=g, device="cuda") < 0.05] = -1  # padding
    return dict(kind=kind, c=c, logits=logits, target=target, y=y, ones=[1.0] * c["gamma"], **_selector(g, c))


def run(s):
    kind = s["kind"]
    if kind == "step":
        return s["step"].run(s["logits"])
    if kind == "head":
        return ubt.lm_head_topk(s["h"], s["w"], s["K"], workspace=s["workspace"])
    if kind == "verify":
        out, lse = ubt.tree_attention(s["q"], s["kc"], s["vc"], s["prefix"], s["kt"], s["vt"], s["mask"],
                                      s["n_nodes"])
        acc = ubt.verify_accept(s["token"], s["parent"], s["n_nodes"], s["target"])
        length = s["prefix"].clone()  # every layer commits from the same lengths
        ubt.commit_kv(s["kt"], s["vt"], acc["accept_nodes"], acc["accept_len"], length, s["kc"], s["vc"])
        return dict(out=out, lse=lse, **acc, prefix_len=length, k_cache=s["kc"], v_cache=s["vc"])
    c = s["c"]
    cand = ubt.topk(s["logits"], c["K"])
    got = ubt.tree_kl_loss(s["logits"], cand, s["target"], s["y"], s["anchor"], s["phi"], s["psi"], s["gate"],
                           s["ones"], s["ones"], c["T"], c["beta"])
    return {**cand, **got}


# ---- what a pass cannot do without --------------------------------------------------------


def _es(name):
    return 2 if name == "bf16" else 4


def work(case):
    c = case
    if c["kind"] == "head":
        return dict(bytes=2 * (c["V"] * c["d"] + c["M"] * c["d"]) + c["M"] * (12 * c["K"] + 4),
                    flops=2 * c["M"] * c["V"] * c["d"])
    if c["kind"] == "verify":
        B, N, H, Hkv, D = (c[k] for k in ("B", "N", "H", "Hkv", "D"))
        ctx = sum(_prefix(c))
        words = (N + 31) // 32
        return dict(bytes=4 * Hkv * D * (ctx + B * N) + 4 * B * N * H * D + 4 * B * N * (H + words + 3),
                    flops=4 * D * H * N * (ctx + B * 8))
    rows, K = c["B"] * c["gamma"], c["K"]
    cand = rows * (12 * K + 4)
    if c["kind"] == "step":
        pairs = c["B"] * (K + (c["gamma"] - 1) * K * K)
        gathers = (c["B"] * (1 + (c["gamma"] - 1) * K) + rows * K + rows) * c["r"] * _es(c["feat"])
        N = c["budget"] + 1
        tree = c["B"] * (4 + N * (20 + 4 * ((N + 31) // 32)))
        return dict(bytes=rows * c["V"] * _es(c["dtype"]) + cand + gathers + 4 * rows * K * K + tree,
                    flops=2 * pairs * c["r"] + 3 * rows * c["V"])
    return dict(bytes=rows * c["V"] * (_es(c["dtype"]) + 4) + cand + rows * (16 + 4 * K + _es(c["dtype"]) * K)
                + rows * (K + 2) * c["r"] * _es(c["feat"]),
                flops=6 * rows * c["V"])


def tolerance(case):
    # Sums of fp32 in another order; whole values may differ where two scores tie to rounding.
    if case["kind"] == "step":
        return dict(rel=1e-5, max=1e-4, differ=0.005)
    if case["kind"] == "head":
        return dict(rel=1e-5, max=1e-4, differ=0.005)
    if case["kind"] == "verify":  # probabilities and outputs are rounded to bf16
        return dict(rel=1e-2, max=5e-2)
    return dict(rel=1e-5, max=1e-4)


# ---- the same in 64 bits ------------------------------------------------------------------


def _candidates(u, K):
    """ids and values of the K largest per row, by (value desc, id asc), and the LSE."""
    bits = u.float().add(0.0).view(torch.int32).long()
    key = torch.where(bits >= 0, bits, -(bits & 0x7FFFFFFF) - 1)
    ids = torch.arange(u.shape[1] - 1, -1, -1, device=u.device)
    pick = (key * (1 << 32) + ids).topk(K, dim=1).indices
    x = u.double()
    return pick, x.gather(1, pick), x.logsumexp(1)


def _grow(logq, W, budget):
    """Scores [B, budget + 1] of the selected nodes in pruning order (the root first)."""
    B, gamma, K, _ = logq.shape
    score = torch.zeros(B, 1, dtype=torch.float64, device=logq.device)
    cand = torch.zeros(B, 1, dtype=torch.int64, device=logq.device)
    every = []
    for i in range(gamma):
        ext = score[:, :, None] + logq[:, i].gather(1, cand[:, :, None].expand(-1, -1, K))
        top, at = ext.flatten(1).sort(dim=1, descending=True, stable=True)
        score, cand = top[:, :W], at[:, :W] % K
        every.append(score)
    best = torch.cat(every, 1).sort(dim=1, descending=True, stable=True).values[:, :budget]
    out = torch.full((B, budget + 1), -math.inf, dtype=torch.float64, device=logq.device)
    out[:, 0] = 0.0
    out[:, 1:1 + best.shape[1]] = best
    return out


def exact(case, seed):
    c, s = case, prepare(case, seed)
    if c["kind"] == "step":
        B, gamma, K = c["B"], c["gamma"], c["K"]
        step = s["step"]
        got = dict(cand_ids=None, cand_logit=[], cand_logprob=[], lse=[], logq=[])
        psi, phi = step.psi, step.phi
        for b in range(B):
            ids, u, lse = _candidates(s["logits"][b], K)
            slabs = []
            for i in range(gamma):
                prev = step.anchor[b:b + 1].long() if i == 0 else ids[i - 1]
                z = u[i][None] + (step.gate[b, i].double() * phi[prev].double()) @ psi[ids[i]].double().T
                q = z.log_softmax(1)
                slabs.append(q if i else torch.cat([q, torch.zeros(K - 1, K, dtype=q.dtype, device=q.device)]))
            for k, v in (("cand_logit", u), ("cand_logprob", u - lse[:, None]), ("lse", lse),
                         ("logq", torch.stack(slabs))):
                got[k].append(v)
        got = {k: torch.stack(v) if v is not None else None for k, v in got.items()}
        return dict(got, score=_grow(got["logq"], c["W"], c["budget"]))
    if c["kind"] == "head":
        h, K = s["h"].double(), c["K"]
        u = torch.cat([h @ s["w"][v:v + 16384].double().T for v in range(0, c["V"], 16384)], 1)
        top, lse = u.topk(K, dim=1).values, u.logsumexp(1)
        return dict(cand_logit=top, cand_logprob=top - lse[:, None], lse=lse)
    if c["kind"] == "verify":
        B, N, H, Hkv, D = (c[k] for k in ("B", "N", "H", "Hkv", "D"))
        g, anc = H // Hkv, _trees(seed, B, N)[1].cuda()
        out = torch.empty(B, N, H, D, dtype=torch.float64, device="cuda")
        lse = torch.empty(B, N, H, dtype=torch.float64, device="cuda")
        for b, P in enumerate(_prefix(c)):
            see = torch.cat([torch.ones(N, P, dtype=torch.bool, device="cuda"), anc[b]], 1)
            for kv in range(Hkv):
                k = torch.cat([s["kc"][b, :P, kv], s["kt"][b, :, kv]]).double()
                v = torch.cat([s["vc"][b, :P, kv], s["vt"][b, :, kv]]).double()
                for h in range(kv * g, kv * g + g):
                    z = (s["q"][b, :, h].double() @ k.T * D ** -0.5).masked_fill(~see, -math.inf)
                    lse[b, :, h] = z.logsumexp(1)
                    out[b, :, h] = z.softmax(1) @ v
        return dict(out=out, lse=lse)
    B, gamma, V, K = (c[k] for k in ("B", "gamma", "V", "K"))
    got = {k: [] for k in ("cand_logit", "cand_logprob", "lse", "loss", "kl", "ce", "grad_s", "grad_logits")}
    rows = torch.arange(gamma, device="cuda")
    for b in range(B):
        ids, u, lse = _candidates(s["logits"][b], K)
        y = s["y"][b].long()
        ok = y >= 0
        prev = torch.cat([s["anchor"][b:b + 1].long(), y[:-1]])
        a = s["gate"][b].double() * s["phi"][prev.clamp(min=0)].double() * (prev >= 0).double()[:, None]
        z = u + (s["psi"][ids].double() * a[:, None, :]).sum(2)
        q, p = z.log_softmax(1), (s["target"][b].double().gather(1, ids) / c["T"]).log_softmax(1)
        x = s["logits"][b].double()
        kl = (p.exp() * (p - q)).sum(1) * ok
        ce = (lse - x[rows, y.clamp(min=0)]) * ok
        gs = (q.exp() - p.exp()) * ok[:, None]
        grad = c["beta"] * (x - lse[:, None]).exp_()
        grad[rows, y.clamp(min=0)] -= c["beta"]
        grad = grad.scatter_add_(1, ids, gs) * ok[:, None]
        for k, v in (("cand_logit", u), ("cand_logprob", u - lse[:, None]), ("lse", lse), ("kl", kl), ("ce", ce),
                     ("loss", kl + c["beta"] * ce), ("grad_s", gs), ("grad_logits", grad)):
            got[k].append(v)
    return {k: torch.stack(v) for k, v in got.items()}
