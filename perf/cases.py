"""The workloads this framework is timed on, through its public entry points.

A case is a dict of plain values; `kind` says which calls one pass makes:

  step          GtoPath.step: both trees, rewards, advantage, surrogate forward and gradient rows
  reward        one tree per root: expand, select, reward and walk (scoring without a training step)
  rows          the draft row statistics alone
  tree          expansion, top-g selection and reward scan from statistics that are already there
  surrogate     surrogate forward (reference rows' log-sum-exp recomputed) and gradient rows on long accepted paths
  token         token-level loss, forward and backward, on teacher-forced positions
  fused_step    GtoFusedPath.step: the same step from hidden states and LM heads
  fused_reward  expand, select, reward and walk from hidden states and LM heads
  fused_bwd     fused surrogate forward and the gradient carried on to the hidden states
  fused_token   fused token-level loss, forward and backward

Logits stand in for a trained drafter's: Gaussian noise with 32 planted peaks of Zipf(1.1) profile per row, the first
of them well above the others, the target sharing the drafter's peaks on 80 % of the rows; hidden states and heads are Gaussian, the target head
correlated with the draft head.  `exact` recomputes the outputs in 64 bits with plain torch.
"""
import math

import torch

import paper_2509_22134_amd as G
from paper_2509_22134_amd.pipeline import GtoFusedPath, GtoPath

DEV = "cuda:0"
ETA, EPS, DELTA, SCALE = 1.0, 0.2, 1e-6, 0.5
DT = {"bf16": torch.bfloat16, "f32": torch.float32}
ES = {"bf16": 2, "f32": 4}


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # a unit-test sized training step (fp32): nothing but launches and their latency
        dict(name="tiny_step", kind="step", R=4, V=1000, k=4, d=3, g=10, m=4, dtype="f32", prune=False),
        # rescoring a handful of prompts between other work: few rows, wide vocabulary
        dict(name="few_roots_reward", kind="reward", R=4, V=151936, k=8, d=7, g=64, dtype="bf16", prune=False),
        # Vicuna-sized vocabulary, the reward of a whole batch (the ablation / data-selection pass)
        dict(name="vicuna_reward", kind="reward", R=512, V=32000, k=10, d=6, g=60, dtype="bf16", prune=True),
        # the headline training step: every draft row of both models, the needed target rows, gradient rows
        dict(name="llama31_step", kind="step", R=1024, V=128256, k=10, d=6, g=60, m=8, dtype="bf16", prune=True),
        # fp32 logits over a vocabulary that is no multiple of anything (a drafter with added tokens)
        dict(name="ragged_f32_rows", kind="rows", R=128, V=32003, k=10, d=6, dtype="f32"),
        # trees re-scored from kept statistics (another budget g or reward mode): the per-root kernels only
        dict(name="tree_from_stats", kind="tree", R=1024, V=4096, k=10, d=6, g=60, dtype="bf16"),
        # a well-trained drafter: four accepted tokens per root, so the backward writes a thousand rows
        dict(name="long_path_surrogate", kind="surrogate", R=256, V=128256, k=10, d=6, g=60, m=8, dtype="bf16", p=0.85),
        # token-level loss next to the surrogate, one supervised position per root
        dict(name="token_loss", kind="token", R=1024, V=128256, dtype="bf16"),
        # the largest: 70B-shaped heads, logits never stored, both trees and the gradient rows
        dict(name="fused_step", kind="fused_step", R=1024, V=128256, k=8, d=8, g=80, m=8, hidden=8192, corr=0.95, prune=True),
        # a handful of prompts through the same heads
        dict(name="fused_few_roots", kind="fused_reward", R=8, V=128256, k=8, d=8, g=80, hidden=8192, corr=0.95, prune=True),
        # gradient with respect to the drafter's hidden states on long accepted paths
        dict(name="fused_backward", kind="fused_bwd", R=256, V=128256, k=8, d=8, g=80, m=8, hidden=8192, p=0.8),
        # token-level loss from hidden states
        dict(name="fused_token_loss", kind="fused_token", R=1024, V=128256, hidden=8192),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the same kinds, sizes log-uniform over the ranges, odd vocabularies among them."""
    kind = rng.choice(["step", "reward", "rows", "tree", "surrogate", "token", "fused_step", "fused_reward", "fused_bwd",
                       "fused_token"])
    k, d = rng.choice([4, 6, 8, 10]), rng.choice([3, 5, 6, 7, 8])
    g = rng.choice([50, 60, 64, 80])
    m = rng.choice([4, 8])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    V = _log(rng, 1000, 152000)
    if rng.random() < 0.5:
        V -= V % 256
    prune = rng.random() < 0.5
    rows_most = 6 << 30                          # elements of one logits tensor at most
    if kind.startswith("fused"):
        hidden = 64 * _log(rng, 8, 128)
        V = max(1024, V - V % 32)
        if kind == "fused_step":
            R = m * _log(rng, 1, 512 // m)
            return dict(kind=kind, R=R, V=V, k=min(k, 10), d=d, g=g, m=m, hidden=hidden, corr=0.95, prune=prune)
        if kind == "fused_reward":
            return dict(kind=kind, R=_log(rng, 1, 128), V=V, k=k, d=d, g=g, hidden=hidden, corr=0.95, prune=prune)
        if kind == "fused_bwd":
            return dict(kind=kind, R=m * _log(rng, 1, 512 // m), V=V, k=k, d=d, g=g, m=m, hidden=hidden, p=0.8)
        return dict(kind=kind, R=_log(rng, 16, 1024), V=V, hidden=hidden)
    if kind == "tree":
        return dict(kind=kind, R=_log(rng, 1, 4096), V=4096, k=k, d=d, g=g, dtype=dtype)
    if kind == "token":
        return dict(kind=kind, R=_log(rng, 8, 4096), V=V, dtype=dtype)
    most = max(m, min(1024, rows_most // (d * k * V * (ES[dtype] // 2))))
    R = m * _log(rng, 1, max(1, most // m))
    if kind == "step":
        return dict(kind=kind, R=R, V=V, k=k, d=d, g=g, m=m, dtype=dtype, prune=prune)
    if kind == "surrogate":
        return dict(kind=kind, R=R, V=V, k=k, d=d, g=g, m=m, dtype=dtype, p=rng.choice([0.6, 0.85]))
    if kind == "reward":
        return dict(kind=kind, R=R, V=V, k=k, d=d, g=g, dtype=dtype, prune=prune)
    return dict(kind=kind, R=R, V=V, k=k, d=d, dtype=dtype)


# ------------------------------------------------------------------------------------------------ inputs
def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + what * 7919 + 17) & 0x7FFFFFFFFFFFFFFF)
    return g


def _stride(V, dtype):
    n = 16 // ES[dtype]
    return (V + n - 1) // n * n


PEAKS = 32


def _peak_heights():
    h = 14.0 - 1.1 * torch.log(torch.arange(1, PEAKS + 1, device=DEV, dtype=torch.float32))
    h[0] += 4.0
    return h


def _positions(rows, V, gen):
    return torch.randint(0, V, (rows, PEAKS), generator=gen, device=DEV)


def _fill(out, V, pos, gen, add=None, sigma=2.0):
    """out [rows, stride]: noise (+ `add`, the reference model's own logits) with the peaks at pos."""
    rows, h = out.shape[0], _peak_heights()
    step = max(1, (1 << 28) // out.shape[1])
    for r0 in range(0, rows, step):
        r1 = min(rows, r0 + step)
        x = torch.randn((r1 - r0, out.shape[1]), generator=gen, device=DEV, dtype=torch.float32).mul_(sigma)
        if add is not None:
            x += add[r0:r1]
        else:
            x.scatter_add_(1, pos[r0:r1], h.expand(r1 - r0, PEAKS))
        out[r0:r1] = x
        del x


def _logits(c, seed, tags):
    """D_cur, T_cur (and D_ref, T_ref): [R, d, k, stride]; D_ref is a perturbed D_cur, the target rows share the
    draft rows' peaks with probability 0.8."""
    rows, V, st = c["R"] * c["d"] * c["k"], c["V"], _stride(c["V"], c["dtype"])
    shape = (c["R"], c["d"], c["k"], st)
    pos = _positions(rows, V, _gen(seed, 1))
    out = {}
    D = torch.empty((rows, st), dtype=DT[c["dtype"]], device=DEV)
    _fill(D, V, pos, _gen(seed, 2))
    out["D_cur"] = D.view(shape)
    if "ref" in tags:
        Dr = torch.empty_like(D)
        _fill(Dr, V, None, _gen(seed, 3), add=D, sigma=0.125)
        out["D_ref"] = Dr.view(shape)
    for i, tag in enumerate(tags):
        coin = torch.rand((rows, 1), generator=_gen(seed, 10 + i), device=DEV) < 0.8
        pt = torch.where(coin, pos, _positions(rows, V, _gen(seed, 20 + i)))
        T = torch.empty_like(D)
        _fill(T, V, pt, _gen(seed, 30 + i))
        out["T_" + tag] = T.view(shape)
    return out


def _heads(c, seed, both=True):
    W = {}
    V, H = c["V"], c["hidden"]
    Wd = torch.empty((V, H), dtype=torch.bfloat16, device=DEV)
    Wt = torch.empty_like(Wd) if both else None
    ga, gb = _gen(seed, 41), _gen(seed, 42)
    corr = c.get("corr", 0.95)
    step = max(1, (1 << 28) // H)
    for v0 in range(0, V, step):
        v1 = min(V, v0 + step)
        a = torch.randn((v1 - v0, H), generator=ga, device=DEV).mul_(0.02)
        Wd[v0:v1] = a
        if both:
            b = torch.randn((v1 - v0, H), generator=gb, device=DEV).mul_(0.02 * math.sqrt(1 - corr * corr))
            Wt[v0:v1] = b.add_(a, alpha=corr)
    W["W_draft"] = Wd
    if both:
        W["W_target"] = Wt
    return W


def _hiddens(c, seed, ref):
    shape = (c["R"], c.get("d", 1), c.get("k", 1), c["hidden"])
    h = torch.randn(shape, generator=_gen(seed, 51), device=DEV)
    out = {"H_cur": h.to(torch.bfloat16)}
    if ref:
        out["H_ref"] = h.add_(torch.randn(shape, generator=_gen(seed, 52), device=DEV), alpha=0.07).to(torch.bfloat16)
    return out


def _paths(c, seed):
    """Accepted paths as a drafter whose tokens are accepted with probability p leaves them: path_len, path_slot,
    and (by construction) the node of step t at position t of the kept list."""
    R, d, k = c["R"], c["d"], c["k"]
    g = _gen(seed, 61)
    ok = (torch.rand((R, d), generator=g, device=DEV) < c["p"]).int().cumprod(1)
    slot = torch.randint(0, k, (R, d), generator=g, device=DEV, dtype=torch.int32)
    slot[:, 0] = 0
    on = ok > 0
    step = torch.arange(d, device=DEV, dtype=torch.int32).expand(R, d)
    minus = torch.full_like(slot, -1)
    return ok.sum(1).int(), torch.where(on, slot, minus), torch.where(on, step, minus)


def _lse(rows64):
    return torch.logsumexp(rows64, dim=-1)


def _path_state(c, seed, cfg):
    tree, rew = G.alloc_tree(cfg, DEV), G.alloc_reward(cfg, DEV)
    rew["path_len"], rew["path_slot"], rew["path_node"] = _paths(c, seed)
    tree["n_sel"].fill_(min(c["g"], cfg.C))
    return tree, rew


def _cfg(c, **kw):
    base = dict(R=c["R"], d=c.get("d", 1), k=c.get("k", 1), g=c.get("g", 1), V=c["V"],
                dtype=DT[c.get("dtype", "bf16")], group_size=c.get("m", 1), eta=ETA, eps=EPS, delta=DELTA, grad_scale=SCALE,
                flags=G.GTO_FLAG_TARGET_PRUNE if c.get("prune") else 0)
    if "dtype" in c:
        base["row_stride"] = _stride(c["V"], c["dtype"])
    base.update(kw)
    return G.make_config(**base)


def _tree_tables(c, seed):
    """Row statistics as a draft and a target pass leave them, and the target logits behind them (narrow
    vocabulary: the per-root kernels only look single entries up)."""
    R, d, k, V = c["R"], c["d"], c["k"], c["V"]
    g = _gen(seed, 71)
    lp = torch.log_softmax(torch.randn((R, d, k, 64), generator=g, device=DEV) * 2.5, -1)
    lp = lp.topk(k, dim=-1).values.contiguous()
    tok = torch.rand((R, d, k, V), generator=g, device=DEV).topk(k, dim=-1).indices.int().contiguous()
    T = torch.randn((R, d, k, V), generator=g, device=DEV)
    best = torch.where(torch.rand((R, d, k, 1), generator=g, device=DEV) < 0.7, tok[..., :1].long(),
                       torch.randint(0, V, (R, d, k, 1), generator=g, device=DEV))
    T.scatter_(-1, best, 9.0)
    T = T.to(DT[c["dtype"]])
    t_lse = torch.empty((R, d, k), device=DEV)
    for r0 in range(0, R, 64):
        t_lse[r0:r0 + 64] = _lse(T[r0:r0 + 64].double())
    return lp, tok, T, t_lse, best[..., 0].int().contiguous()


# ------------------------------------------------------------------------------------------------ prepare / run
def prepare(c, seed):
    kind = c["kind"]
    s = {"c": c}
    if kind == "step":
        s.update(_logits(c, seed, ("cur", "ref")))
        s["path"] = p = GtoPath(R=c["R"], d=c["d"], k=c["k"], g=c["g"], V=c["V"], dtype=DT[c["dtype"]], group_size=c["m"],
                                device=DEV, row_stride=_stride(c["V"], c["dtype"]), eta=ETA, eps=EPS, delta=DELTA,
                                grad_scale=SCALE, flags=G.GTO_FLAG_TARGET_PRUNE if c["prune"] else 0)
        p.grad_rows.zero_()                      # rows that carry no gradient stay as they are
    elif kind == "reward":
        s.update(_logits(c, seed, ("cur",)))
        s["path"] = GtoPath(R=c["R"], d=c["d"], k=c["k"], g=c["g"], V=c["V"], dtype=DT[c["dtype"]], group_size=1,
                            device=DEV, row_stride=_stride(c["V"], c["dtype"]), eta=ETA, eps=EPS, delta=DELTA,
                            flags=G.GTO_FLAG_TARGET_PRUNE if c["prune"] else 0, full_path=False)
    elif kind == "rows":
        cfg = s["cfg"] = _cfg(c, g=1)
        s["D"] = _logits(c, seed, ())["D_cur"]
        s["dstats"] = G.alloc_draft_stats(cfg, DEV)
    elif kind == "tree":
        cfg = s["cfg"] = _cfg(c)
        lp, tok, T, t_lse, best = _tree_tables(c, seed)
        s["T"] = T
        s["dstats"], s["tstats"] = G.alloc_draft_stats(cfg, DEV), G.alloc_target_stats(cfg, DEV)
        s["dstats"]["top_logp"], s["dstats"]["top_tok"] = lp, tok
        s["tstats"]["t_lse"], s["tstats"]["t_argmax"] = t_lse, best
        s["pool"], s["tree"], s["rew"] = G.alloc_pool(cfg, DEV), G.alloc_tree(cfg, DEV), G.alloc_reward(cfg, DEV)
    elif kind == "surrogate":
        cfg = s["cfg"] = _cfg(c)
        R, d, k, g, V = c["R"], c["d"], c["k"], c["g"], c["V"]
        rows, st = R * d * k, _stride(V, c["dtype"])
        pos = _positions(rows, V, _gen(seed, 1))
        D = torch.empty((rows, st), dtype=DT[c["dtype"]], device=DEV)
        _fill(D, V, pos, _gen(seed, 2))
        Dr = torch.empty_like(D)
        _fill(Dr, V, None, _gen(seed, 3), add=D, sigma=0.125)
        s["D"], s["Dr"] = D.view(R, d, k, st), Dr.view(R, d, k, st)
        s["tree"], s["rew"] = _path_state(c, seed, cfg)
        s["tree"]["sel_tok"][:, :d] = _path_tokens(s["rew"]["path_slot"], pos.view(R, d, k, PEAKS))
        s["dstats"] = G.alloc_draft_stats(cfg, DEV)
        s["dstats"]["row_lse"].copy_(_path_lse(s["D"], s["rew"]["path_slot"], V))
        s["adv"] = torch.randn((R,), generator=_gen(seed, 62), device=DEV)
        s["ppo"] = G.alloc_ppo(cfg, DEV)
        s["ws"] = torch.empty((G.gto_workspace_bytes(cfg),), dtype=torch.uint8, device=DEV)
        s["grad_rows"] = torch.zeros((R, d, V), device=DEV)
        s["grad_slot"] = torch.empty((R, d), dtype=torch.int32, device=DEV)
    elif kind == "token":
        cfg = s["cfg"] = _cfg(c)
        t = _logits(dict(c, d=1, k=1), seed, ("cur",))
        s["D"], s["T"] = t["D_cur"], t["T_cur"]
        s["dstats"], s["tstats"] = G.alloc_draft_stats(cfg, DEV), G.alloc_target_stats(cfg, DEV)
        for x, o in ((s["D"], s["dstats"]["row_lse"]), (s["T"], s["tstats"]["t_lse"])):
            for r0 in range(0, c["R"], 256):
                o[r0:r0 + 256] = _lse(x[r0:r0 + 256, ..., :c["V"]].double())
        _token_buffers(s, c, seed)
    elif kind == "fused_step":
        s.update(_heads(c, seed))
        s.update(_hiddens(c, seed, True))
        s["path"] = p = GtoFusedPath(R=c["R"], d=c["d"], k=c["k"], g=c["g"], V=c["V"], hidden=c["hidden"], group_size=c["m"],
                                     device=DEV, eta=ETA, eps=EPS, delta=DELTA, grad_scale=SCALE,
                                     flags=G.GTO_FLAG_TARGET_PRUNE if c["prune"] else 0)
        p.grad_rows.zero_()
    elif kind == "fused_reward":
        cfg = s["cfg"] = _cfg(c)
        s.update(_heads(c, seed))
        s.update(_hiddens(c, seed, False))
        s["ws"] = torch.empty((G.gto_fused_workspace_bytes(cfg, c["hidden"]),), dtype=torch.uint8, device=DEV)
        s["dstats"], s["tstats"] = G.alloc_draft_stats(cfg, DEV), G.alloc_target_stats(cfg, DEV)
        s["pool"], s["tree"], s["rew"] = G.alloc_pool(cfg, DEV), G.alloc_tree(cfg, DEV), G.alloc_reward(cfg, DEV)
    elif kind == "fused_bwd":
        cfg = s["cfg"] = _cfg(c)
        R, d, H = c["R"], c["d"], c["hidden"]
        s.update(_heads(c, seed, both=False))
        s.update(_hiddens(c, seed, True))
        s["W_hv"] = s["W_draft"].t().contiguous()
        s["tree"], s["rew"] = _path_state(c, seed, cfg)
        s["dstats"], s["rstats"] = G.alloc_draft_stats(cfg, DEV), G.alloc_draft_stats(cfg, DEV)
        rt, idx = _path_rows(s["rew"]["path_slot"], c["k"])
        Wf = s["W_draft"].float()
        for name, st in (("H_cur", s["dstats"]), ("H_ref", s["rstats"])):
            h = s[name].view(-1, H)[idx].float()
            for i0 in range(0, len(idx), 512):
                L = h[i0:i0 + 512] @ Wf.t()
                st["row_lse"].view(-1)[idx[i0:i0 + 512]] = _lse(L.double()).float()
                if name == "H_cur":
                    i = rt[i0:i0 + 512]
                    s["tree"]["sel_tok"][i // d, i % d] = L.argmax(-1).int()
        del Wf
        s["adv"] = torch.randn((R,), generator=_gen(seed, 62), device=DEV)
        s["ppo"] = G.alloc_ppo(cfg, DEV)
        s["ws"] = torch.empty((G.gto_fused_workspace_bytes(cfg, H),), dtype=torch.uint8, device=DEV)
        s["dws"] = torch.empty((G.gto_fused_dh_workspace_bytes(cfg, H),), dtype=torch.uint8, device=DEV)
        s["dh_rows"] = torch.zeros((R, d, H), device=DEV)
        s["dh_slot"] = torch.empty((R, d), dtype=torch.int32, device=DEV)
    elif kind == "fused_token":
        cfg = s["cfg"] = _cfg(c)
        s.update(_heads(c, seed))
        s.update(_hiddens(c, seed, False))
        s["dstats"], s["tstats"] = G.alloc_draft_stats(cfg, DEV), G.alloc_target_stats(cfg, DEV)
        h = s["H_cur"].view(c["R"], -1).float()
        for wn, o in (("W_draft", s["dstats"]["row_lse"]), ("W_target", s["tstats"]["t_lse"])):
            Wf = s[wn].float()
            for r0 in range(0, c["R"], 512):
                o.view(-1)[r0:r0 + 512] = _lse((h[r0:r0 + 512] @ Wf.t()).double()).float()
            del Wf
        s["ws"] = torch.empty((G.gto_fused_token_loss_workspace_bytes(cfg, c["hidden"]),), dtype=torch.uint8, device=DEV)
        _token_buffers(s, c, seed)
    else:
        raise ValueError(kind)
    return s


def _token_buffers(s, c, seed):
    R = c["R"]
    s["weight"] = (torch.rand((R,), generator=_gen(seed, 63), device=DEV) < 0.9).float()
    s["weight"][0] = 1.0
    s["loss_rows"], s["loss"], s["inv"] = (torch.zeros((n,), device=DEV) for n in (R, 1, 1))
    s["grad"] = torch.empty((R, c["V"]), device=DEV)


def _path_rows(path_slot, k):
    """(root, step) pairs on the accepted paths and their slot index in [R, d, k]."""
    rt = (path_slot.view(-1) >= 0).nonzero().view(-1)
    return rt, rt * k + path_slot.view(-1)[rt].long()


def _path_tokens(path_slot, pos):
    """The accepted token of step t: the first planted peak of the row it was drawn from."""
    first = pos[..., 0]
    return first.gather(2, path_slot.clamp(min=0).long().unsqueeze(-1))[..., 0].int()


def _path_lse(D, path_slot, V):
    R, d, k, st = D.shape
    out = torch.zeros((R * d * k,), device=DEV)
    _, idx = _path_rows(path_slot, k)
    flat = D.view(-1, st)
    for i0 in range(0, len(idx), 512):
        i = idx[i0:i0 + 512]
        out[i] = _lse(flat[i, :V].double()).float()
    return out.view(R, d, k)


TREE_OUT = ("sel_tok", "sel_parent", "sel_score", "n_sel")
REWARD_OUT = ("reward", "reward_aux", "path_len", "path_slot")
PPO_OUT = ("logM", "logM0", "ratio", "term", "active", "coef", "loss_group", "loss")


def _tree_outputs(b):
    out = {n: b["dstats"][n] for n in ("row_max", "row_lse", "top_tok", "top_logp")}
    out.update({n: b["tree"][n] for n in TREE_OUT})
    out.update({n: b["rew" if "rew" in b else "reward"][n] for n in REWARD_OUT})
    return out


def run(s):
    kind = s["c"]["kind"]
    if kind in ("step", "fused_step"):
        p = s["path"]
        if kind == "step":
            p.step(s["D_cur"], s["T_cur"], s["D_ref"], s["T_ref"])
        else:
            p.step(s["H_cur"], s["H_ref"], s["W_draft"], s["W_target"])
        return dict(cur=_tree_outputs(p.buf["cur"]), ref=_tree_outputs(p.buf["ref"]), adv=p.adv,
                    ppo={n: p.ppo[n] for n in PPO_OUT}, grad_rows=p.grad_rows, grad_slot=p.grad_slot)
    if kind == "reward":
        s["path"].step(s["D_cur"], s["T_cur"])
        return _tree_outputs(s["path"].buf["cur"])
    cfg = s["cfg"]
    if kind == "rows":
        return G.gto_draft_row_stats(cfg, s["D"], s["dstats"])
    if kind == "tree":
        G.gto_expand_from_stats(cfg, s["dstats"], s["pool"])
        G.gto_select_topg(cfg, s["pool"], s["tree"])
        G.gto_reward_from_stats(cfg, s["tree"], s["T"], s["tstats"], s["rew"])
        return dict(pool=s["pool"], tree=s["tree"], reward=s["rew"])
    if kind == "surrogate":
        G.gto_ppo_surrogate_fwd(cfg, s["tree"], s["rew"], s["D"], s["dstats"], s["Dr"], None, s["adv"], s["ppo"],
                                workspace=s["ws"])
        G.gto_ppo_surrogate_bwd(cfg, s["tree"], s["rew"], s["ppo"], s["D"], s["dstats"], s["grad_rows"], s["grad_slot"])
        return dict(ppo={n: s["ppo"][n] for n in PPO_OUT}, grad_rows=s["grad_rows"], grad_slot=s["grad_slot"])
    if kind == "token":
        G.gto_token_loss_fwd(cfg, s["D"], s["T"], s["dstats"], s["tstats"], s["weight"], s["loss_rows"], s["loss"], s["inv"])
        G.gto_token_loss_bwd(cfg, s["D"], s["T"], s["dstats"], s["tstats"], s["weight"], s["inv"], SCALE, s["grad"])
        return dict(loss_rows=s["loss_rows"], loss=s["loss"], inv_count=s["inv"], grad=s["grad"])
    if kind == "fused_reward":
        G.gto_expand_tree_fused(cfg, s["H_cur"], s["W_draft"], s["dstats"], s["pool"], s["ws"])
        G.gto_select_topg(cfg, s["pool"], s["tree"])
        G.gto_tree_reward_fused(cfg, s["tree"], s["H_cur"], s["W_target"], s["tstats"], s["rew"], s["ws"])
        return _tree_outputs(s)
    if kind == "fused_bwd":
        G.gto_ppo_surrogate_fwd_fused(cfg, s["tree"], s["rew"], s["H_cur"], s["H_ref"], s["W_draft"], s["dstats"],
                                      s["rstats"], s["adv"], s["ppo"], s["ws"])
        G.gto_ppo_surrogate_bwd_fused_dh(cfg, s["tree"], s["rew"], s["ppo"], s["H_cur"], s["W_draft"], s["W_hv"],
                                         s["dstats"], s["dh_rows"], s["dh_slot"], s["dws"])
        return dict(ppo={n: s["ppo"][n] for n in PPO_OUT}, dh_rows=s["dh_rows"], dh_slot=s["dh_slot"])
    G.gto_token_loss_fwd_fused(cfg, s["H_cur"], s["W_draft"], s["W_target"], s["dstats"], s["tstats"], s["weight"],
                               s["loss_rows"], s["loss"], s["inv"], s["ws"])
    G.gto_token_loss_bwd_fused(cfg, s["dstats"], s["tstats"], s["weight"], s["inv"], SCALE, s["grad"], s["ws"])
    return dict(loss_rows=s["loss_rows"], loss=s["loss"], inv_count=s["inv"], grad=s["grad"])


# ------------------------------------------------------------------------------------------------ work / tolerance
def _rho(c):
    return 1 + (c["d"] - 1) * c["k"]


def _small(c):
    """Bytes of the per-root tables (candidate pool, statistics, kept tree) of one tree per root."""
    C = c["k"] + (c["d"] - 1) * c["k"] ** 2
    return c["R"] * (C * (8 + 6 * 4) + c["g"] * 10 * 4 * 2)


def _steps(c):
    """Expected accepted length."""
    return sum(c["p"] ** i for i in range(1, c["d"] + 1))


def work(c):
    kind, R, V = c["kind"], c["R"], c["V"]
    es = ES[c.get("dtype", "bf16")]
    # a kept tree of g nodes refers to about half of the expanded slots' target rows
    target = 0.5 if c.get("prune") else 1.0
    if kind == "step":
        n = 2 * R * _rho(c) * (1 + target)
        grads = 1.5 * R                             # accepted length of these logits
        return {"bytes": n * V * es + grads * V * (es + 4) + 2 * _small(c), "flops": 5 * n * V}
    if kind == "reward":
        n = R * _rho(c) * (1 + target)
        return {"bytes": n * V * es + _small(c), "flops": 5 * n * V}
    if kind == "rows":
        n = R * _rho(c)
        return {"bytes": n * (V * es + 8 + 8 * c["k"]), "flops": 5 * n * V}
    if kind == "tree":
        return {"bytes": _small(c), "flops": R * c["d"] * c["k"] ** 2 * 20}
    if kind == "surrogate":
        n = R * _steps(c)
        return {"bytes": n * V * (2 * es + 4), "flops": 8 * n * V}
    if kind == "token":
        return {"bytes": R * V * (2 * es + 4), "flops": 12 * R * V}
    H = c["hidden"]
    if kind == "fused_step":
        n = 2 * R * _rho(c) * (1 + 0.25) + 1.7 * R
        return {"bytes": 2 * 2 * V * H + 2 * R * _rho(c) * H * 2 + 1.7 * R * V * 4, "flops": 2 * n * V * H}
    if kind == "fused_reward":
        n = R * _rho(c) * (1 + (0.25 if c.get("prune") else 1.0))
        return {"bytes": 2 * 2 * V * H + R * _rho(c) * H * 2, "flops": 2 * n * V * H}
    if kind == "fused_bwd":
        n = R * _steps(c)
        return {"bytes": 2 * 2 * V * H + n * H * (2 + 4), "flops": 2 * 2 * n * V * H}
    return {"bytes": 2 * 2 * V * H + R * V * 4 + R * H * 2, "flops": 2 * 2 * R * V * H}


def tolerance(c):
    """Statistics are fp32 sums and logarithms rounded once; ids are exact but for near ties of fp32 scores (and, with
    fp32-accumulated logits, of the logits themselves).  Standardising within a group divides the rewards' rounding by
    the group's spread, so whole steps carry the largest bounds (measured against another summation order and against
    64 bits, times four)."""
    kind = c["kind"]
    if kind in ("step", "reward"):
        return {"rel": 1e-3 if kind == "step" else 1e-5, "max": 0.1, "differ": 2e-3}
    if kind == "rows":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    if kind == "tree":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    if kind in ("surrogate", "token"):
        return {"rel": 1e-5, "max": 1e-3}
    if kind in ("fused_step", "fused_reward"):
        return {"rel": 1.5e-2 if kind == "fused_step" else 1e-3, "max": 0.5, "differ": 8e-3}
    return {"rel": 5e-5, "max": 5e-3}


# ------------------------------------------------------------------------------------------------ 64-bit results
def _top(x, V, k):
    """k best (values in 64 bits, ids): value descending, id ascending."""
    if x.dtype == torch.float64:
        v, i = x.topk(k, dim=-1)
        return v, i
    b = x.float().contiguous().view(torch.int32).long()
    b = torch.where(b < 0, -(b & 0x7FFFFFFF), b)          # monotone in the value
    key = b * (1 << 20) + ((1 << 20) - 1 - torch.arange(V, device=DEV))
    i = (1 << 20) - 1 - (key.topk(k, dim=-1).values & ((1 << 20) - 1))
    return x.gather(-1, i).double(), i


def _root_blocks(R, per_root):
    step = max(1, (1 << 28) // per_root)
    return [(r, min(R, r + step)) for r in range(0, R, step)]


def _tree_block(c, lp, lp64, tok, target, tl, best):
    """Tree, reward and walk of a block of roots from its row statistics.  Ranking is on the documented fp32 scores;
    target(root, level, slot, token): target logits in 64 bits."""
    d, k, g = c["d"], c["k"], c["g"]
    B, C = lp.shape[0], k + (d - 1) * k * k
    n = min(g, C)
    sc, sc64, par = [lp[:, 0, 0]], [lp64[:, 0, 0]], [torch.full((B, k), -1, device=DEV, dtype=torch.long)]
    slots = [None, torch.arange(k, device=DEV).expand(B, k)]
    s32, s64 = sc[0], sc64[0]
    for l in range(1, d):
        a = (s32.unsqueeze(-1) + lp[:, l]).reshape(B, k * k)
        b = (s64.unsqueeze(-1) + lp64[:, l]).reshape(B, k * k)
        sc.append(a)
        sc64.append(b)
        par.append(slots[l].unsqueeze(-1).expand(B, k, k).reshape(B, k * k))
        o = a.sort(dim=-1, descending=True, stable=True).indices[:, :k]
        s32, s64 = a.gather(1, o), b.gather(1, o)
        slots.append(o + k + (l - 1) * k * k)
    sc, sc64, par = torch.cat(sc, 1), torch.cat(sc64, 1), torch.cat(par, 1)
    ctok = torch.cat([tok[:, 0, 0]] + [tok[:, l].reshape(B, k * k) for l in range(1, d)], 1)
    cdep = torch.cat([torch.ones(k, device=DEV, dtype=torch.long)] +
                     [torch.full((k * k,), l + 1, device=DEV, dtype=torch.long) for l in range(1, d)])
    cslot = torch.cat([torch.zeros(k, device=DEV, dtype=torch.long)] +
                      [torch.arange(k * k, device=DEV) // k for _ in range(1, d)])
    order = sc.sort(dim=-1, descending=True, stable=True).indices
    rank = torch.empty_like(order).scatter_(1, order, torch.arange(C, device=DEV).expand(B, C))
    sel = order[:, :n]
    sp = par.gather(1, sel)
    sp = torch.where(sp >= 0, rank.gather(1, sp.clamp(min=0)), sp)
    dep, psl, stok = cdep[sel], cslot[sel], ctok.gather(1, sel)
    bi = torch.arange(B, device=DEV).unsqueeze(1).expand(B, n)
    logt = target(bi, dep - 1, psl, stok) - tl[bi, dep - 1, psl]
    lq, cum = torch.zeros_like(logt), torch.zeros_like(logt)
    for l in range(1, d + 1):
        p = sp.clamp(min=0)
        q = logt + torch.where(sp >= 0, lq.gather(1, p), 0.0)
        cm = q.exp() + torch.where(sp >= 0, cum.gather(1, p), 0.0)
        lq, cum = torch.where(dep == l, q, lq), torch.where(dep == l, cm, cum)
    leaf = torch.ones((B, n + 1), device=DEV, dtype=torch.bool)
    leaf.scatter_(1, torch.where(sp >= 0, sp, n), False)
    leaf = leaf[:, :n]
    L = torch.where(leaf, cum, float("-inf"))
    aux = torch.stack([torch.logsumexp(ETA * L, 1) / ETA, L.max(1).values,
                       torch.where(leaf, cum, 0.0).sum(1) / leaf.sum(1), lq.exp().sum(1)], 1)
    # the greedy verification walk
    own = torch.full((B, C), -1, device=DEV, dtype=torch.long)
    for l in range(1, d):
        own.scatter_(1, slots[l], torch.arange(k, device=DEV).expand(B, k))
    sown = own.gather(1, sel)
    cur = torch.full((B,), -1, device=DEV, dtype=torch.long)
    slot, plen, alive = torch.zeros_like(cur), torch.zeros_like(cur), torch.ones_like(cur, dtype=torch.bool)
    pnode, pslot = torch.full((B, d), -1, device=DEV), torch.full((B, d), -1, device=DEV)
    ar = torch.arange(B, device=DEV)
    for t in range(d):
        want = best[ar, t, slot.clamp(min=0)]
        hit = (sp == cur.unsqueeze(1)) & (dep == t + 1) & (stok == want.unsqueeze(1)) & alive.unsqueeze(1)
        found, at = hit.any(1), hit.int().argmax(1)
        pnode[:, t], pslot[:, t] = torch.where(found, at, -1), torch.where(found, slot, -1)
        plen = torch.where(found, t + 1, plen)
        cur = torch.where(found, at, cur)
        slot = torch.where(found, sown[ar, at], slot)
        alive = found & (slot >= 0)
    pad = lambda x: torch.nn.functional.pad(x, (0, g - n))  # noqa: E731
    return dict(sel_score=pad(sc64.gather(1, sel)), reward=aux[:, 0], reward_aux=aux, node_q=pad(lq.exp()),
                node_cum=pad(cum), cand_score=sc64, stok=stok, plen=plen, pnode=pnode, pslot=pslot)


def _exact_tree(c, rows_d, rows_t):
    """Statistics, tree, reward and walk of every root; rows_d / rows_t(r0, r1) give [n, d, k, V] logits."""
    R, d, k, V = c["R"], c["d"], c["k"], c["V"]
    outs = []
    for r0, r1 in _root_blocks(R, d * k * V):
        x = rows_d(r0, r1)
        val, tok = _top(x, V, k)
        lse = _lse(x.double())
        lp64 = val - lse.unsqueeze(-1)
        del x
        y = rows_t(r0, r1)
        o = _tree_block(c, lp64.float().clamp(max=0), lp64, tok, lambda b, l, j, t: y[b, l, j, t].double(),
                        _lse(y.double()), _top(y, V, 1)[1][..., 0])
        outs.append(dict(o, row_max=val[..., 0], row_lse=lse, top_logp=lp64))
        del y
    out = {n: torch.cat([o[n] for o in outs], 0) for n in outs[0]}
    for n in ("row_max", "row_lse", "top_logp"):      # slots (0, 1..) do not exist
        out[n][:, 0, 1:] = 0
    return out


def _exact_tree_outputs(o):
    out = {n: o[n] for n in ("row_max", "row_lse", "top_logp", "sel_score", "reward", "reward_aux")}
    for n in ("top_tok", "sel_tok", "sel_parent", "n_sel", "path_len", "path_slot"):
        out[n] = None
    return out


def _exact_ppo(c, adv, plen, lp_cur, lp_ref):
    """lp_*: [R, d] log-probability of the accepted token of each step (zero beyond the path)."""
    m, K = c["m"], c["R"] // c["m"]
    lm, lm0 = lp_cur.sum(1), lp_ref.sum(1)
    den = plen.clamp(min=1).double()
    s = ((lm - lm0) / den).exp()
    lo, hi = 1.0 - float(torch.tensor(EPS)), 1.0 + float(torch.tensor(EPS))
    term = torch.minimum(s * adv, s.clamp(lo, hi) * adv)
    act = (plen > 0) & torch.where(adv >= 0, s <= hi, s >= lo)
    coef = SCALE * (-adv / (m * K)) * act * s / den
    lg = -term.view(K, m).mean(1)
    return dict(logM=lm, logM0=lm0, ratio=s, term=term, active=None, coef=coef, loss_group=lg, loss=lg.mean().view(1))


def _grad_rows(c, coef, ptok, pslot, rows_of):
    """[R, d, V]: coef * (onehot - softmax) of the path rows; rows_of(slot indices) gives their logits in 64 bits."""
    R, d, k, V = c["R"], c["d"], c["k"], c["V"]
    out = torch.zeros((R * d, V), device=DEV, dtype=torch.float64)
    live = torch.where((coef != 0).unsqueeze(1), pslot, -1)
    rt, idx = _path_rows(live, k)
    for i0 in range(0, len(rt), 512):
        i, r = idx[i0:i0 + 512], rt[i0:i0 + 512]
        x = rows_of(i)
        p = torch.softmax(x, -1)
        tk = ptok.view(-1)[r].long().unsqueeze(1)
        rest = p.scatter(1, tk, 0.0).sum(1, keepdim=True)
        out[r] = coef[r // d].unsqueeze(1) * (-p).scatter(1, tk, rest)
    return out.view(R, d, V)


def _token_logp(path_slot, ptok, k, rows_of):
    rt, idx = _path_rows(path_slot, k)
    out = torch.zeros(path_slot.shape, device=DEV, dtype=torch.float64)
    for i0 in range(0, len(rt), 512):
        x = rows_of(idx[i0:i0 + 512])
        t = ptok.view(-1)[rt[i0:i0 + 512]].long().unsqueeze(1)
        out.view(-1)[rt[i0:i0 + 512]] = (x.gather(1, t)[:, 0] - _lse(x))
    return out


def _exact_step(c, cur, ref, cur_rows, ref_rows):
    R, d, k = c["R"], c["d"], c["k"]
    x = (cur["reward"] - ref["reward"]).view(-1, c["m"])
    adv = ((x - x.mean(1, keepdim=True)) / (x.std(1, unbiased=False, keepdim=True) + DELTA)).view(-1)
    ptok = torch.where(cur["pnode"] >= 0, cur["stok"].gather(1, cur["pnode"].clamp(min=0)), 0)
    lp = [_token_logp(cur["pslot"], ptok, k, f) for f in (cur_rows, ref_rows)]
    ppo = _exact_ppo(c, adv, cur["plen"], *lp)
    return dict(cur=_exact_tree_outputs(cur), ref=_exact_tree_outputs(ref), adv=adv, ppo=ppo,
                grad_rows=_grad_rows(c, ppo["coef"], ptok, cur["pslot"], cur_rows), grad_slot=None)


def _exact_token(rows_d, rows_t, weight, R, V):
    inv = 1.0 / weight.double().sum()
    loss = torch.empty((R,), device=DEV, dtype=torch.float64)
    grad = torch.empty((R, V), device=DEV, dtype=torch.float64)
    for r0 in range(0, R, 256):
        a, b = torch.log_softmax(rows_d(r0, r0 + 256), -1), torch.log_softmax(rows_t(r0, r0 + 256), -1)
        w = weight[r0:r0 + 256].double()
        loss[r0:r0 + 256] = -w * (b.exp() * a).sum(1)
        grad[r0:r0 + 256] = SCALE * inv * w.unsqueeze(1) * (a.exp() - b.exp())
    return dict(loss_rows=loss, loss=(loss.sum() * inv).view(1), inv_count=inv.view(1), grad=grad)


def exact(c, seed):
    kind, R, V = c["kind"], c["R"], c["V"]
    if kind in ("step", "reward"):
        t = _logits(c, seed, ("cur", "ref") if kind == "step" else ("cur",))
        block = lambda x: (lambda r0, r1: x[r0:r1, ..., :V])  # noqa: E731
        cur = _exact_tree(c, block(t["D_cur"]), block(t["T_cur"]))
        if kind == "reward":
            return _exact_tree_outputs(cur)
        ref = _exact_tree(c, block(t["D_ref"]), block(t["T_ref"]))
        some = lambda x: (lambda i: x.view(-1, x.shape[-1])[i, :V].double())  # noqa: E731
        return _exact_step(c, cur, ref, some(t["D_cur"]), some(t["D_ref"]))
    if kind == "rows":
        D = _logits(c, seed, ())["D_cur"]
        lse = torch.zeros((R, c["d"], c["k"]), device=DEV, dtype=torch.float64)
        top = torch.zeros((R, c["d"], c["k"], c["k"]), device=DEV, dtype=torch.float64)
        for r0, r1 in _root_blocks(R, c["d"] * c["k"] * V):
            x = D[r0:r1, ..., :V].double()
            lse[r0:r1], top[r0:r1] = _lse(x), x.topk(c["k"], dim=-1).values
        lp = top - lse.unsqueeze(-1)
        for x in (lse, lp, top):
            x[:, 0, 1:] = 0
        return dict(row_max=top[..., 0].contiguous(), row_lse=lse, top_logp=lp, top_tok=None)
    if kind == "tree":
        return _exact_from_tables(c, seed)
    if kind == "surrogate":
        s = prepare(c, seed)
        pslot, ptok = s["rew"]["path_slot"].long(), s["tree"]["sel_tok"][:, :c["d"]].long()
        f = [(lambda i, x=x: x.view(-1, x.shape[-1])[i, :V].double()) for x in (s["D"], s["Dr"])]
        lp = [_token_logp(pslot, ptok, c["k"], g) for g in f]
        ppo = _exact_ppo(c, s["adv"].double(), s["rew"]["path_len"].long(), *lp)
        return dict(ppo=ppo, grad_rows=_grad_rows(c, ppo["coef"], ptok, pslot, f[0]), grad_slot=None)
    if kind == "token":
        t = _logits(dict(c, d=1, k=1), seed, ("cur",))
        w = (torch.rand((R,), generator=_gen(seed, 63), device=DEV) < 0.9).float()
        w[0] = 1.0
        return _exact_token(*[(lambda r0, r1, x=t[n]: x[r0:r1, 0, 0, :V].double()) for n in ("D_cur", "T_cur")], w, R, V)
    H = c["hidden"]
    if kind in ("fused_step", "fused_reward"):
        if R * _rho(c) * float(V) * H * (2 if kind == "fused_step" else 1) > 5e13:
            return None                           # minutes of 64-bit products
        W = {n: x.double() for n, x in _heads(c, seed).items()}
        h = _hiddens(c, seed, kind == "fused_step")

        def block(hn, wn):
            return lambda r0, r1: (h[hn][r0:r1].double().view(-1, H) @ W[wn].t()).view(r1 - r0, c["d"], c["k"], V)

        cur = _exact_tree(c, block("H_cur", "W_draft"), block("H_cur", "W_target"))
        if kind == "fused_reward":
            return _exact_tree_outputs(cur)
        ref = _exact_tree(c, block("H_ref", "W_draft"), block("H_ref", "W_target"))
        some = lambda hn: (lambda i: h[hn].view(-1, H)[i].double() @ W["W_draft"].t())  # noqa: E731
        return _exact_step(c, cur, ref, some("H_cur"), some("H_ref"))
    if kind == "fused_bwd":
        s = prepare(c, seed)
        pslot, ptok = s["rew"]["path_slot"].long(), s["tree"]["sel_tok"][:, :c["d"]].long()
        W = s["W_draft"].double()
        f = [(lambda i, x=s[n]: x.view(-1, H)[i].double() @ W.t()) for n in ("H_cur", "H_ref")]
        lp = [_token_logp(pslot, ptok, c["k"], g) for g in f]
        ppo = _exact_ppo(c, s["adv"].double(), s["rew"]["path_len"].long(), *lp)
        gr = _grad_rows(c, ppo["coef"], ptok, pslot, f[0])
        return dict(ppo=ppo, dh_rows=(gr.view(-1, V) @ W).view(R, c["d"], H), dh_slot=None)
    W = {n: x.double() for n, x in _heads(c, seed).items()}
    h = _hiddens(c, seed, False)["H_cur"].double().view(R, H)
    w = (torch.rand((R,), generator=_gen(seed, 63), device=DEV) < 0.9).float()
    w[0] = 1.0
    return _exact_token(*[(lambda r0, r1, n=n: h[r0:r1] @ W[n].t()) for n in ("W_draft", "W_target")], w, R, V)


def _exact_from_tables(c, seed):
    """The `tree` kind: the same tree, from statistics instead of logits."""
    lp, tok, T, t_lse, best = _tree_tables(c, seed)
    o = _tree_block(c, lp, lp.double(), tok.long(), lambda b, l, j, t: T[b, l, j, t].double(), t_lse.double(), best.long())
    none = {n: None for n in ("cand_tok", "cand_parent", "cand_depth", "cand_pslot", "cand_slot", "slot_cand")}
    tree = {n: None for n in ("sel_cand", "sel_tok", "sel_parent", "sel_depth", "sel_pslot", "sel_slot", "sel_leaf", "n_sel",
                              "slot_need")}
    rew = {n: None for n in ("n_leaves", "path_len", "path_node", "path_slot")}
    return dict(pool=dict(none, cand_score=o["cand_score"]), tree=dict(tree, sel_score=o["sel_score"]),
                reward=dict(rew, node_q=o["node_q"], node_cum=o["node_cum"], reward=o["reward"], reward_aux=o["reward_aux"]))
