"""The work that programs have this library do, as cases that can be timed and compared.

Users of the library are RL trainers (likelihoods of compute schedules, episodes, rewards) and servers (prompt
passes, decode steps, periodic cache refresh) of action-conditioned Llama decoders. A case names one public call and
its sizes: `prepare` makes what such a program holds before the call, `run` is the call, `exact` the same results in
plain 64-bit torch for the calls of one layer, where they are defined to better than the method's own decisions.
"""
import math

import torch

from paper_2605_10875_amd import sol, synth

SHAPES = {"tiny": synth.TINY, "1b": synth.LLAMA_1B, "8b": synth.LLAMA_8B}
TABLES = {
    "c1": synth.TABLE_C1, "c2": synth.TABLE_C2,
    # 8-bit codes at the linear inputs: with 4- and 6-bit codes there a layer's result is off by 13 % when its norm's sum
    # is taken in another order, so that nothing could be compared (the calls' work does not depend on the bits)
    "c8": synth.action_table((0.125, 0.25, 0.5, 1.0), (0.0, 0.25, 0.5, 0.75), (8, 16)),
    # attention keep-rates and MLP pruning alone, for whole models: with quantisers one unit in the last place of a
    # weight moves a whole model's results by 4 % (NLL) to 50 % (hidden states)
    "keep": synth.action_table((0.0625, 0.125, 0.25, 0.5, 1.0), (0.0, 0.25, 0.5, 0.75), (16,)),
}
# key-selection rules: exact top-k with quantised linear inputs (the library's default), the paper's configuration
RULES = {"topk": {}, "pages": sol.PAPER_PRESET}
REWARD = dict(alpha=(1.0, 0.5, 0.25), tau=0.02, gamma=0.99)


def listed():
    return [
        # the reward reduction that follows a likelihood pass: a few small launches on whole batches of NLLs
        dict(name="reward", op="reward", B=2, G=8, T=2048),
        # the smallest likelihood pass (one tiny fp32 layer, 4 schedules of 128 tokens): latency and launches
        dict(name="loglik_tiny_fp32", op="schedule", shape="tiny", layers=1, vocab=1000, dtype="fp32", rule="topk",
             table="c1", B=1, G=4, T=128),
        # a layer in fp32, as it is run to check a bf16 deployment: two prompts of odd length
        dict(name="layer_1b_fp32", op="layer", shape="1b", dtype="fp32", rule="topk", table="keep", n_seq=2, T=509, past=0),
        # one user's prompt of odd length through a layer
        dict(name="layer_1b_prompt", op="layer", shape="1b", dtype="bf16", rule="topk", table="c8", n_seq=1, T=333, past=0),
        # a full batch of long sequences through a layer of the larger model
        dict(name="layer_8b_batch", op="layer", shape="8b", dtype="bf16", rule="topk", table="c8", n_seq=8, T=4096, past=0),
        # a few prompts of odd length under the paper's configuration (pages, sink and window keys, MLP-input pruning)
        dict(name="layer_8b_pages", op="layer", shape="8b", dtype="bf16", rule="pages", table="c2", n_seq=3, T=1777, past=0),
        # the trainer's teacher-forced likelihood pass of the whole model
        dict(name="loglik_1b", op="schedule", shape="1b", layers=16, vocab=128256, dtype="bf16", rule="topk", table="keep",
             B=2, G=8, T=2048),
        # an episode: dense prefix once per input, 32 schedules of 16 steps on it, whole model
        dict(name="episode_1b", op="episode", shape="1b", layers=16, vocab=128256, dtype="bf16", rule="topk", table="keep",
             B=8, K=32, P=1024, T=16),
        # cache refresh of a serving batch: the last 16 tokens of 64 sequences, densely, one layer of the pass
        dict(name="refresh_1b", op="refresh", shape="1b", layers=1, rule="topk", B=64, L=4096, T=16),
        # one user's decode step, whole model, replayed as a HIP graph
        dict(name="decode_1b_single", op="decode", shape="1b", layers=16, vocab=128256, rule="topk", table="keep", B=1,
             L=4096, graph=True),
        # a serving batch's decode step, whole model, replayed as a HIP graph
        dict(name="decode_1b_batch", op="decode", shape="1b", layers=16, vocab=128256, rule="topk", table="keep", B=64,
             L=8192, graph=True),
        # one layer's decode step of the larger model under the page rule with kept page metadata, called directly
        dict(name="decode_8b_pages", op="decode", shape="8b", layers=1, vocab=0, rule="pages", table="c2", B=32, L=8192,
             graph=False),
    ]


def _size(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(("layer", "layer", "layer", "decode", "decode", "schedule", "episode", "refresh", "reward"))
    rule = rng.choice(("topk", "pages"))
    if op == "reward":
        return dict(op=op, B=_size(rng, 1, 16), G=_size(rng, 2, 32), T=_size(rng, 16, 2048))
    if op == "layer":
        shape = rng.choice(("1b", "8b"))
        if rng.random() < 0.2:
            return dict(op=op, shape="1b", dtype="fp32", rule="topk", table="keep", n_seq=_size(rng, 1, 4), T=_size(rng, 65, 700), past=0)
        T = _size(rng, 65, 3000)
        return dict(op=op, shape=shape, dtype="bf16", rule=rule, table="c8" if rule == "topk" else "c2", n_seq=_size(rng, 1, max(1, 12000 // T)), T=T,
                    past=rng.choice((0, 0, _size(rng, 1, 1000))))
    if op == "decode":
        shape, layers = rng.choice((("1b", 16), ("8b", 1))) if rule == "topk" else (rng.choice(("1b", "8b")), 1)
        return dict(op=op, shape=shape, layers=layers, vocab=128256 if layers > 1 else 0, rule=rule,
                    table="keep" if layers > 1 else "c8" if rule == "topk" else "c2", B=_size(rng, 1, 64), L=_size(rng, 200, 8192), graph=rng.random() < 0.5)
    layers = 16 if rule == "topk" else 2     # (flips of whole pages move the results of a whole model by 4 %)
    if op == "schedule":
        if rng.random() < 0.3:
            return dict(op=op, shape="tiny", layers=1, vocab=1000, dtype="fp32", rule="topk", table="c1", B=_size(rng, 1, 4),
                        G=_size(rng, 2, 8), T=_size(rng, 64, 300))
        return dict(op=op, shape="1b", layers=layers, vocab=128256, dtype="bf16", rule=rule, table="keep", B=rng.randint(1, 2),
                    G=rng.randint(2, 8), T=_size(rng, 100, 1500))
    if op == "episode":
        return dict(op=op, shape="1b", layers=layers, vocab=128256, dtype="bf16", rule=rule, table="keep", B=rng.randint(1, 8),
                    K=_size(rng, 4, 32), P=64 * _size(rng, 2, 20), T=rng.randint(16, 40))
    return dict(op=op, shape="1b", layers=1, rule=rule, B=_size(rng, 5, 64), L=_size(rng, 256, 4096), T=rng.randint(16, 64))


# ---- inputs -------------------------------------------------------------------------------------------------------
def _weights(shape, layers, vocab, dt, rnd):
    def one():
        d, nq, nkv, ff = shape.d_model, shape.n_q_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim, shape.d_ff
        dims = {"wq": (nq, d), "wk": (nkv, d), "wv": (nkv, d), "wo": (d, nq), "w_gate": (ff, d), "w_up": (ff, d), "w_down": (d, ff)}
        w = {k: rnd(*sz).mul_(0.02).to(dt) for k, sz in dims.items()}
        for k in ("w_in_norm", "w_post_norm"):
            w[k] = rnd(d).mul_(0.1).add_(1.0).to(dt)
        return w

    head = None
    if vocab:
        head = {"embed": rnd(vocab, shape.d_model).mul_(0.02).to(dt), "w_final_norm": rnd(shape.d_model).mul_(0.1).add_(1.0).to(dt),
                "lm_head": rnd(vocab, shape.d_model).mul_(0.02).to(dt)}
    return [one() for _ in range(layers)], head


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)
    fp32 = case.get("dtype") == "fp32"
    dt, code = (torch.float32, sol.F32) if fp32 else (torch.bfloat16, sol.BF16)

    def rnd(*sz):
        return torch.randn(sz, generator=gen, device="cuda", dtype=torch.float32 if math.prod(sz) < 1 << 28 else dt)

    def ints(hi, *sz):
        return torch.randint(0, hi, sz, generator=gen, device="cuda", dtype=torch.int32)

    op = case["op"]
    if op == "reward":
        shape, table = SHAPES["1b"], TABLES["c2"]
        ctx = sol.Sol(shape, table, max_positions=16)
        sh = (case["B"], case["G"], case["T"])
        return dict(case=case, ctx=ctx, nll=rnd(*sh).abs_().mul_(3.0), ids=ints(len(table), *sh),
                    targets=torch.rand((case["B"], 3), generator=gen, device="cuda"),
                    eff=(torch.rand((case["B"], case["T"]), generator=gen, device="cuda") < 0.9).to(torch.int32))
    shape = SHAPES[case["shape"]]
    table = TABLES[case.get("table", "c2")]
    s = dict(case=case)
    n_layers = case.get("layers", 1)
    vocab = case.get("vocab", 0)
    s["layers"], s["head"] = _weights(shape, n_layers, vocab, dt, rnd)
    shape = synth.with_layers(shape, n_layers, vocab)

    def context(positions):
        return sol.Sol(shape, table, dtype=code, max_positions=positions, **RULES[case["rule"]])

    def caches(n, L, fill=True):
        sz = (n, shape.n_kv_heads, L, shape.head_dim)
        return rnd(*sz).to(dt) if fill else torch.zeros(sz, dtype=dt, device="cuda")

    if op == "layer":
        n, T, past = case["n_seq"], case["T"], case["past"]
        s["ctx"] = context(past + T)
        s["x"], s["ids"] = rnd(n, T, shape.d_model).to(dt), ints(len(table), n, T)
        s["kc"], s["vc"] = caches(n, past + T, past > 0), caches(n, past + T, past > 0)
        s["pos0"] = torch.full((n,), past, dtype=torch.int32, device="cuda") if past else None
        s["out"] = torch.empty_like(s["x"])
        s["ws"] = s["ctx"].workspace(sol.OP_LAYER_FORWARD, n, T, past + T)
    elif op == "schedule":
        B, G, T = case["B"], case["G"], case["T"]
        s["ctx"] = context(T)
        s["tokens"], s["targets"] = ints(vocab, B, T), ints(vocab, B, T)
        fresh, hold = ints(len(table), B * G, T), torch.rand((B * G, T), generator=gen, device="cuda") < 0.8
        at = torch.where(hold, 0, torch.arange(T, device="cuda")).cummax(1).values          # bursty schedules: an action is
        s["ids"] = fresh.gather(1, at).view(B, G, T).contiguous()                           # held with probability 0.8
        s["ws"] = s["ctx"].workspace(sol.OP_SCHEDULE_LOGLIK, B * G, T, T)
    elif op == "episode":
        B, K, P, T = case["B"], case["K"], case["P"], case["T"]
        s["ctx"] = context(P + T)
        s["prefix"], s["tokens"], s["targets"] = ints(vocab, B, P), ints(vocab, B, T), ints(vocab, B, T)
        s["ids"] = ints(len(table), B, K, T)
        s["ws"] = torch.empty(int(sol.lib().sol_episode_workspace_bytes(s["ctx"].cfg, B, K, P, T)), dtype=torch.uint8, device="cuda")
    elif op == "refresh":
        B, L, T = case["B"], case["L"], case["T"]
        s["ctx"] = context(L)
        s["x"] = rnd(B, T, shape.d_model).to(dt)
        s["kc"], s["vc"] = [caches(B, L) for _ in range(n_layers)], [caches(B, L) for _ in range(n_layers)]
        s["pos0"] = torch.full((B,), L - T, dtype=torch.int32, device="cuda")
        s["ws"] = s["ctx"].workspace(sol.OP_KV_REFRESH, B, T, L)
    elif op == "decode":
        B, L = case["B"], case["L"]
        s["ctx"] = context(L + 8)
        s["ids"] = ints(len(table), B)
        s["len"] = ints(L // 4 + 1, B).neg_().add_(L)                                       # ragged: 3/4 L .. L tokens in the cache
        s["kc"], s["vc"] = [caches(B, L + 8) for _ in range(n_layers)], [caches(B, L + 8) for _ in range(n_layers)]
        s["meta"] = [s["ctx"].page_meta_build(k, s["len"]) for k in s["kc"]] if case["rule"] == "pages" else None
        if vocab:
            s["tokens"], s["targets"], s["x"] = ints(vocab, B), ints(vocab, B), None
        else:
            s["tokens"], s["targets"], s["x"] = None, None, rnd(B, shape.d_model).to(dt)
        s["ws"] = s["ctx"].workspace(sol.OP_DECODE_STEP, B, 1, L + 8)
        if case["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                _decode(s)
            torch.cuda.current_stream().wait_stream(side)
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                s["outs"] = _decode(s)
    return s


# ---- the calls ----------------------------------------------------------------------------------------------------
def _decode(s):
    x, nll = s["ctx"].decode_step(s["layers"], s["head"], s["ids"], s["len"], s["kc"], s["vc"], token_ids=s["tokens"], x_in=s["x"],
                                  targets=s["targets"], want_hidden=s["head"] is None, workspace=s["ws"], page_meta=s["meta"])
    return {"x": x, "nll": nll, "k": s["kc"], "v": s["vc"], "meta": s["meta"]}


def run(s):
    c, ctx = s["case"], s["ctx"]
    op = c["op"]
    if op == "reward":
        return ctx.reward_advantages(s["nll"], s["ids"], s["targets"], eff=s["eff"], **REWARD)
    if op == "layer":
        x = ctx.layer_forward(s["layers"][0], s["x"], s["ids"], s["kc"], s["vc"], pos0=s["pos0"], x_out=s["out"], workspace=s["ws"])
        return {"x": x, "k": s["kc"], "v": s["vc"]}
    if op == "schedule":
        return ctx.schedule_loglik(s["layers"], s["head"], s["tokens"], s["targets"], s["ids"], workspace=s["ws"])
    if op == "episode":
        return ctx.episode_loglik(s["layers"], s["head"], s["prefix"], s["tokens"], s["targets"], s["ids"], workspace=s["ws"])
    if op == "refresh":
        x = ctx.kv_refresh(s["layers"], None, s["pos0"], s["kc"], s["vc"], x_in=s["x"], workspace=s["ws"])
        return {"x": x, "k": s["kc"], "v": s["vc"]}
    if c["graph"]:
        s["graph"].replay()
        return s["outs"]
    return _decode(s)


# ---- what a pass cannot do without --------------------------------------------------------------------------------
def _kept(case, table, n):
    """Mean number of keys of n that a query head keeps."""
    page = RULES[case["rule"]].get("page_size", 1)
    tot = 0
    for a in TABLES[table]:
        b = -(-a[0] * n // a[1])
        tot += n if b >= n else min(n, -(-b // page) * page)
    return tot / len(TABLES[table])


def _union(kept, n, heads, page=1):
    """Keys that at least one of `heads` heads keeps, the heads being independent."""
    return n * (1.0 - (1.0 - min(1.0, kept / n)) ** heads)


def work(case):
    op = case["op"]
    if op == "reward":
        n = case["B"] * case["G"] * case["T"]
        return {"bytes": 4 * (5 * n + case["B"] * case["T"]), "flops": 12 * n}
    shape, es = SHAPES[case["shape"]], 4 if case.get("dtype") == "fp32" else 2
    d, ff, dh, Hq, Hkv = shape.d_model, shape.d_ff, shape.head_dim, shape.n_q_heads, shape.n_kv_heads
    nq, nkv = Hq * dh, Hkv * dh
    per_layer = d * (nq + 2 * nkv) + nq * d + 3 * d * ff
    nl, vocab, table = case.get("layers", 1), case.get("vocab", 0), case.get("table", "c2")

    def attention(rows, T, past):
        """flops of one layer: causal scores of every key (selection needs them), values of the kept ones."""
        f = 0.0
        for n in range(past + 1, past + T + 1, max(1, T // 64)):
            f += 2 * dh * Hq * (n + _kept(case, table, n))
        return rows * T * f / len(range(past + 1, past + T + 1, max(1, T // 64)))

    if op == "layer":
        n, T, past = case["n_seq"], case["T"], case["past"]
        M = n * T
        return {"bytes": es * (per_layer + 2 * M * d + 2 * n * (past + 2 * T) * nkv), "flops": 2 * M * per_layer + attention(n, T, past)}
    if op == "schedule":
        M = case["B"] * case["G"] * case["T"]
        return {"bytes": es * (nl * per_layer + vocab * d + 2 * nl * M * nkv) + 8 * M,
                "flops": nl * (2 * M * per_layer + attention(case["B"] * case["G"], case["T"], 0)) + 2 * M * d * vocab}
    if op == "episode":
        B, K, P, T = case["B"], case["K"], case["P"], case["T"]
        Mp, M = B * P, B * K * T
        dense = 2 * dh * Hq * B * P * (P + 1)                       # scores and values of every causal key of the prefix
        return {"bytes": es * (nl * per_layer + vocab * d + 2 * nl * (Mp + M) * nkv) + 8 * M,
                "flops": nl * (2 * (Mp + M) * per_layer + dense + attention(B * K, T, P)) + 2 * M * d * vocab}
    if op == "refresh":
        B, L, T = case["B"], case["L"], case["T"]
        return {"bytes": nl * es * (per_layer + 2 * B * T * d + 2 * B * (L + T) * nkv), "flops": nl * (2 * B * T * per_layer + 4 * dh * Hq * B * T * L)}
    B, L = case["B"], case["L"] - case["L"] // 8                    # mean cache length
    page = RULES[case["rule"]].get("page_size", 1)
    union = _union(_kept(case, table, L), L, Hq // Hkv)
    keys = B * nkv * (2 * (L / page) + 2 * union) if page > 1 else B * nkv * (L + union)
    return {"bytes": es * (nl * (per_layer + keys + 2 * B * nkv) + B * d + vocab * d),
            "flops": B * (nl * (2 * per_layer + 2 * dh * Hq * L) + 2 * d * vocab)}


def tolerance(case):
    """About four times what another order of the sums was seen to change: the attention by the kernels of other cache
    lengths, the linear maps by those of other batch sizes, or the distance from `exact`."""
    op = case["op"]
    if op == "reward":
        return {"rel": 1e-5, "max": 1e-4}                           # 1.5e-6 from exact: 32-bit sums over 2048 steps
    if case.get("dtype") == "fp32":
        return {"rel": 1e-3, "max": 0.3}                            # 2.6e-4: a kept key or channel flips in a few rows
    if op == "refresh":
        return {"rel": 7e-3, "max": 0.1}                            # 1.7e-3: bf16 results
    if case["rule"] == "topk" and case.get("layers", 1) == 1:
        return {"rel": 0.025, "max": 0.4}                           # 6e-3, single values 0.1: some codes and kept keys flip
    # page rule: 1.3e-2, single values 0.63 of the root mean square (whole pages flip, 4-bit codes of the MLP's output);
    # whole models: 1.3e-2 of the NLL after a change in the last place of some weights
    return {"rel": 0.03, "max": 0.95}


# ---- 64-bit results of one layer ----------------------------------------------------------------------------------
def _norm(x, w, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * w


def _quant(z, bits):
    q = (2.0 ** (bits.double() - 1) - 1).unsqueeze(-1)
    scale = z.abs().amax(-1, keepdim=True) / q
    scale = torch.where(scale > 0, scale, torch.ones_like(scale))
    y = torch.minimum(torch.maximum((z / scale).round(), -q), q) * scale
    return torch.where((bits >= 16).unsqueeze(-1), z, y)


def _prune(a, m):
    kth = a.abs().sort(-1, descending=True).values.gather(-1, (m.long() - 1).unsqueeze(-1))
    return torch.where(a.abs() >= kth, a, torch.zeros_like(a))


def _by_rows(f, x, *rows):
    """f over chunks of rows of x (and of the vectors that go with the rows): bounds the memory of sorts."""
    step = max(1, (1 << 26) // x.shape[-1])
    return torch.cat([f(x[i:i + step], *(r[i:i + step] for r in rows)) for i in range(0, x.shape[0], step)])


def _attend(q, k, v, budgets, past, rule):
    """q [T][g][dh] of one KV head's g query heads at positions past.., k and v [past + T][dh]."""
    T, g, dh = q.shape
    n_all = k.shape[0]
    page, sink, window = rule.get("page_size", 1), rule.get("n_sink", 0), rule.get("n_window", 0)
    out = torch.empty_like(q)
    if page > 1:
        pages = -(-n_all // page)
        hi, lo = (torch.full((pages * page, dh), fill, dtype=k.dtype, device=k.device) for fill in (-math.inf, math.inf))
        hi[:n_all], lo[:n_all] = k, k
        hi, lo = hi.view(pages, page, dh).cummax(1).values, lo.view(pages, page, dh).cummin(1).values
        full_hi, full_lo = hi[:, -1].clone(), lo[:, -1].clone()
        run_hi, run_lo = hi.reshape(-1, dh), lo.reshape(-1, dh)     # extremes of a key's page up to that key
    step = max(1, (1 << 25) // (g * n_all))
    for t0 in range(0, T, step):
        qq = q[t0:t0 + step]
        pos = past + t0 + torch.arange(qq.shape[0], device=q.device)
        causal = torch.arange(n_all, device=q.device)[None, :] <= pos[:, None]
        s = (qq.reshape(-1, dh) @ k.t()).view(qq.shape[0], g, n_all) / math.sqrt(dh)
        s = s.masked_fill(~causal[:, None], -math.inf)
        b, n = budgets[t0:t0 + step].long(), pos + 1
        if page > 1:
            qp, qn = qq.clamp(min=0), qq.clamp(max=0)
            bound = (qp.reshape(-1, dh) @ full_hi.t() + qn.reshape(-1, dh) @ full_lo.t()).view(qq.shape[0], g, pages)
            own = (qp * run_hi[pos][:, None]).sum(-1) + (qn * run_lo[pos][:, None]).sum(-1)
            mine = pos // page
            bound.scatter_(2, mine[:, None, None].expand(-1, g, 1), own[:, :, None])
            bound = bound.masked_fill(torch.arange(pages, device=q.device)[None, None] > mine[:, None, None], -math.inf)
            want = torch.minimum(-(-b // page), mine + 1)
            kth = bound.sort(-1, descending=True).values.gather(2, (want - 1)[:, None, None].expand(-1, g, 1))
            keep = (bound >= kth).repeat_interleave(page, 2)[:, :, :n_all]
            at = torch.arange(n_all, device=q.device)[None, :]
            keep = keep | ((at < sink) | (at > (pos - window)[:, None]))[:, None]
        else:
            kth = s.sort(-1, descending=True).values.gather(2, (b - 1)[:, None, None].expand(-1, g, 1))
            keep = s >= kth
        keep = (keep | (b >= n)[:, None, None]) & causal[:, None]
        p = torch.softmax(s.masked_fill(~keep, -math.inf), -1)
        out[t0:t0 + step] = (p.reshape(-1, n_all) @ v).view(qq.shape[0], g, dh)
    return out


def _layer64(shape, w, x, table, ids, kc, vc, pos0, rule, dt=torch.bfloat16):
    """One layer in 64 bits: x [n][T][d], action ids [n][T], caches [n][Hkv][L][dh] (rows written), start positions.
    The tensors that operators hand on are of type `dt` by the library's definition of a run in that type; without
    these roundings the codes and kept sets, and with them the results, would be others."""
    store = lambda z: z.to(dt).double()  # noqa: E731
    n, T, d = x.shape
    Hq, Hkv, dh = shape.n_q_heads, shape.n_kv_heads, shape.head_dim
    w = {k: t.double() for k, t in w.items()}
    sites, prune_in = rule.get("quant_sites", sol.QS_ALL_LINEAR_INPUTS), rule.get("prune_site", 0) == 1
    tab = torch.tensor(table, device=x.device)[ids.long().reshape(-1)]
    bits = tab[:, 4]
    site = lambda z, bit: _quant(z, bits) if sites & bit else z  # noqa: E731
    x0 = x.reshape(-1, d).double()
    h = store(site(_norm(x0, w["w_in_norm"], shape.rms_eps), sol.QS_QKV_IN))
    pos = (pos0.long()[:, None] + torch.arange(T, device=x.device)[None]).reshape(-1)
    inv = torch.tensor([float(shape.rope_theta) ** (-2.0 * c / dh) for c in range(dh // 2)], dtype=torch.float64, device=x.device)
    cos, sin = (f(pos[:, None].double() * inv)[:, None] for f in (torch.cos, torch.sin))

    def rotate(t):
        a, b = t[..., : dh // 2], t[..., dh // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    q = store(rotate((h @ w["wq"].t()).view(-1, Hq, dh)))
    k, v = store(rotate((h @ w["wk"].t()).view(-1, Hkv, dh))), store((h @ w["wv"].t()).view(-1, Hkv, dh))
    o = torch.empty_like(q)
    g = Hq // Hkv
    for s in range(n):
        p0 = int(pos0[s])
        rows = slice(s * T, (s + 1) * T)
        kc[s, :, p0:p0 + T], vc[s, :, p0:p0 + T] = k[rows].transpose(0, 1), v[rows].transpose(0, 1)
        num, den, nk = tab[rows, 0], tab[rows, 1], pos[rows] + 1
        budgets = torch.minimum(-(-num * nk // den), nk)
        for j in range(Hkv):
            o[rows, j * g:(j + 1) * g] = _attend(q[rows, j * g:(j + 1) * g], kc[s, j, :p0 + T], vc[s, j, :p0 + T], budgets, p0, rule)
    x2 = x0 + store(site(o.reshape(-1, Hq * dh), sol.QS_O_IN)) @ w["wo"].t()
    h2 = _norm(x2, w["w_post_norm"], shape.rms_eps)
    m = lambda width: -(-tab[:, 2] * width // tab[:, 3])  # noqa: E731
    if prune_in:
        h2 = _by_rows(_prune, h2, m(d))
    h2 = store(site(h2, sol.QS_GATEUP_IN))
    a = store(torch.nn.functional.silu(h2 @ w["w_gate"].t()) * (h2 @ w["w_up"].t()))
    if not prune_in:
        a = _by_rows(_prune, a, m(shape.d_ff))
    y = site(store(site(a, sol.QS_DOWN_IN)) @ w["w_down"].t(), sol.QS_MLP_OUT)
    return (x2 + y).view(n, T, d)


def _reward64(s):
    nll, ids, eff = s["nll"].double(), s["ids"].long(), s["eff"].double()
    tab = torch.tensor(TABLES["c2"], dtype=torch.float64, device=nll.device)[ids]
    rates = torch.stack([tab[..., 0] / tab[..., 1], tab[..., 2] / tab[..., 3], tab[..., 4].clamp(max=16) / 16], -1)
    live = eff.sum(-1)[:, None, None]
    goal = s["targets"].double()[:, None]
    avg = torch.where(live > 0, (rates * eff[:, None, :, None]).sum(2) / live.clamp(min=1), goal.expand(-1, nll.shape[1], -1))
    over = ((avg - goal).abs() - REWARD["tau"]).clamp(min=0).square()
    penalty = (over * torch.tensor(REWARD["alpha"], dtype=torch.float64, device=nll.device)).sum(-1)
    ret, acc = torch.empty_like(nll), torch.zeros_like(nll[..., 0])
    for t in range(nll.shape[2] - 1, -1, -1):
        acc = -nll[..., t] + REWARD["gamma"] * acc
        ret[..., t] = acc
    signal = ret - penalty[..., None]
    adv = signal - signal.mean(1, keepdim=True)
    adv = (adv - adv.mean()) / (adv.std(correction=0) + 1e-8)
    return {"avg": avg, "penalty": penalty, "returns": ret, "signal": signal, "adv": adv}


def exact(case, seed):
    op = case["op"]
    if op in ("schedule", "episode") and case["shape"] != "tiny" or op == "decode" and case["layers"] > 1:
        return None     # a whole model's hard decisions (kept keys, kept channels, codes) amplify rounding without bound
    s = prepare(dict(case, graph=False) if op == "decode" else case, seed)
    if op == "reward":
        return _reward64(s)
    shape, rule, table = SHAPES[case["shape"]], RULES[case["rule"]], TABLES[case.get("table", "c2")]
    if op == "layer":
        kc, vc = s["kc"].double(), s["vc"].double()
        pos0 = s["pos0"] if s["pos0"] is not None else torch.zeros(case["n_seq"], dtype=torch.int32, device="cuda")
        return {"x": _layer64(shape, s["layers"][0], s["x"], table, s["ids"], kc, vc, pos0, rule, s["x"].dtype), "k": kc, "v": vc}
    if op == "schedule":
        B, G, T = case["B"], case["G"], case["T"]
        x = s["head"]["embed"].double()[s["tokens"].long()][:, None].expand(B, G, T, -1).reshape(B * G, T, -1)
        kc = torch.zeros((B * G, shape.n_kv_heads, T, shape.head_dim), dtype=torch.float64, device="cuda")
        x = _layer64(shape, s["layers"][0], x, table, s["ids"].view(B * G, T), kc, kc.clone(), torch.zeros(B * G, dtype=torch.int32, device="cuda"), rule,
                     torch.float32)
        logits = _norm(x, s["head"]["w_final_norm"].double(), shape.rms_eps) @ s["head"]["lm_head"].double().t()
        want = s["targets"].long()[:, None].expand(B, G, T).reshape(B * G, T, 1)
        return (torch.logsumexp(logits, -1) - logits.gather(-1, want)[..., 0]).view(B, G, T)
    kc, vc = [t.double() for t in s["kc"]], [t.double() for t in s["vc"]]
    if op == "refresh":                                             # dense: every key, every channel, no quantiser
        x = _layer64(shape, s["layers"][0], s["x"], [synth.DENSE_ACTION], torch.zeros(s["x"].shape[:2], device="cuda"), kc[0], vc[0],
                     s["pos0"], {"quant_sites": 0})
        return {"x": x, "k": kc, "v": vc}
    x = _layer64(shape, s["layers"][0], s["x"][:, None], table, s["ids"][:, None], kc[0], vc[0], s["len"], rule)
    return {"x": x[:, 0], "nll": None, "k": kc, "v": vc, "meta": None}
