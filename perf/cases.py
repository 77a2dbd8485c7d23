"""Timed cases of the tree-verification path (prepare, verify, commit, fused step).

A case is one call sequence that a speculative decoder makes on one Gated
DeltaNet layer: the tree metadata from parent pointers, the read-only
verification of every node, the commit of the accepted path, or the fused
step that commits the previous tree and verifies the current one.  The shapes
are those of the repository's workloads (16 key heads, 32 or 48 value heads,
head dim 128, trees of 16..512 slots) plus smaller heads, fp32 inputs and
padded trees, which the entry points take as well.

Inputs are drawn on the device from the seed with the distributions of
``workloads.py``: unit-norm q and k, v ~ N(0, 1), beta = sigmoid(N(0, 1)),
alpha = exp(-softplus(N(0, 1))), S0 ~ 0.1 N(0, 1), conv weights ~ 0.5 N(0, 1).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_06763_amd import gdn_tree as G
from paper_2607_06763_amd import workloads as W

# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------
_HEADS = dict(Hk=16, Hv=32, dk=128, dv=128)
_WIDE = dict(Hk=16, Hv=48, dk=128, dv=128)


def listed():
    return [
        # the smallest call: one 7-node binary tree of a toy layer, fp32; launch latency
        dict(name="step-tiny-f32", op="step", B=1, T=7, Hk=2, Hv=2, dk=16, dv=16, dtype="f32", tree="heap", pad=0.0),
        # one user, a 16-token draft chain: what a chain drafter submits per decode step
        dict(name="step-b1-chain16", op="step", B=1, T=16, dtype="bf16", tree="chain", pad=0.0, **_HEADS),
        # one user, a best-first draft tree of budget 64
        dict(name="step-b1-topk64", op="step", B=1, T=64, dtype="bf16", tree="topk", pad=0.0, **_HEADS),
        # eight users, budget 64; verify and commit as separate calls, as in a
        # decoder that picks the accepted node between them
        dict(name="verify+commit-b8-t64", op="verify+commit", B=8, T=64, dtype="bf16", tree="random", pad=0.0, **_HEADS),
        # the benchmark workload: 32 users, budget 128, depth 16
        dict(name="step-b32-t128", op="step", B=32, T=128, dtype="bf16", tree="large", pad=0.0, **_WIDE),
        # its two halves on their own: re-verification, and the commit of a step
        dict(name="verify-b32-t128", op="verify", B=32, T=128, dtype="bf16", tree="large", pad=0.0, **_WIDE),
        dict(name="commit-b32-t128", op="commit", B=32, T=128, dtype="bf16", tree="large", pad=0.0, **_WIDE),
        # fp32 inputs, half-size heads, odd tree size, trees of unequal size padded to it
        dict(name="verify-b12-t99-f32", op="verify", B=12, T=99, Hk=8, Hv=16, dk=64, dv=64, dtype="f32", tree="random",
             pad=0.3),
        # a deep draft: single paths of 128 nodes
        dict(name="step-b4-chain128", op="step", B=4, T=128, dtype="bf16", tree="chain", pad=0.0, **_WIDE),
        # trees above the 128-slot on-chip size, of unequal size
        dict(name="verify-b16-t250", op="verify", B=16, T=250, dtype="bf16", tree="large", pad=0.2, **_HEADS),
        # the largest call: the benchmark recipe at the largest tree size
        dict(name="step-b32-t512", op="step", B=32, T=512, dtype="bf16", tree="large", pad=0.0, **_WIDE),
        # the chunked form of the verification, on the deep trees it is meant for
        dict(name="chunked-b8-chain256", op="chunked", B=8, T=256, dtype="bf16", tree="chain", pad=0.0, **_WIDE),
    ]


def draw(rng):
    """Another case of the same ranges: operation, batch 1..32, 5..512 slots
    (odd sizes among them), head counts and dims, dtype, tree shape, padding."""
    op = rng.choice(["step", "step", "verify", "verify+commit", "commit", "chunked"])
    T = max(5, min(512, int(round(math.exp(rng.uniform(math.log(5), math.log(513)))))))
    B = max(1, min(32, int(round(math.exp(rng.uniform(0.0, math.log(32.9)))))))
    Hk = rng.choice([2, 4, 8, 16, 16])
    Hv = Hk * rng.choice([1, 2, 2, 3])
    dk = rng.choice([16, 32, 64, 128, 128, 128])
    dv = rng.choice([dk, dk, 64, 128])
    tree = rng.choice(["topk", "random", "large", "large", "chain"])
    if tree == "topk" and T < 40:
        tree = "random"
    if tree == "chain":
        T = min(T, 256)
        B = min(B, 8)
    if op == "chunked":
        B = min(B, 8)
    pad = 0.0 if tree == "chain" else rng.choice([0.0, 0.0, 0.3])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    if dtype == "f32" or op == "verify+commit":  # never above the largest listed case
        B = min(B, 16)
    return dict(op=op, B=B, T=T, Hk=Hk, Hv=Hv, dk=dk, dv=dv, dtype=dtype, tree=tree, pad=pad)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _capped_tree(rng, n, max_parent_depth, spine, max_children):
    """workloads.random_depth_capped_tree with an incremental candidate list."""
    par, dep, nch, cand = [-1], [0], [0], [0]
    pick = rng.random(n)
    for i in range(1, n):
        if i <= spine:
            p = i - 1
            at = cand.index(p) if p in cand[-4:] else -1
        else:
            at = int(pick[i] * len(cand))
            p = cand[at]
        par.append(p)
        dep.append(dep[p] + 1)
        nch.append(0)
        nch[p] += 1
        if nch[p] >= max_children and at >= 0:
            cand[at] = cand[-1]
            cand.pop()
        if dep[i] <= max_parent_depth:
            cand.append(i)
    return np.array(par, np.int32)


def _trees(case, seed):
    """parent int32 [B][T]: valid trees of the case's shape; with pad > 0 each
    sequence holds (1 - pad) T .. T real nodes at random slots."""
    rng = np.random.default_rng([7, int(seed)])
    B, T, shape = case["B"], case["T"], case["tree"]
    out = np.full((B, T), W.PAD, np.int32)
    for b in range(B):
        n = T - int(rng.integers(0, int(case["pad"] * T) + 1))
        if shape == "heap":
            par = W.heap_tree(n)
        elif shape == "chain":
            par = W.chain_tree(n)
        elif shape == "topk":
            par = W.topk_best_first_tree(rng, n, 4, 8) if n >= 33 else _capped_tree(rng, n, 7, 0, 1 << 30)
        elif shape == "random":
            par = _capped_tree(rng, n, 7, 0, 1 << 30)
        else:
            par = _capped_tree(rng, n, 15, min(16, n - 1), 8)
        if case["pad"] > 0:
            slots = np.sort(rng.permutation(T)[:n])
            out[b, slots] = np.where(par < 0, -1, slots[np.maximum(par, 0)])
        else:
            out[b, :] = par
    return out


def _accepted(case, parent, seed):
    rng = np.random.default_rng([11, int(seed)])
    return np.array([rng.choice(np.nonzero(parent[b] != W.PAD)[0]) for b in range(case["B"])], np.int32)


def _raw(case, gen, dev):
    """Raw q, k, v, alpha, beta of one tree, in the input dtype."""
    B, T, Hk, Hv, dk, dv = (case[n] for n in ("B", "T", "Hk", "Hv", "dk", "dv"))
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=torch.float32)

    q, k = normal(B, T, Hk, dk), normal(B, T, Hk, dk)
    q, k = q / q.norm(dim=-1, keepdim=True), k / k.norm(dim=-1, keepdim=True)
    v = normal(B, T, Hv, dv)
    alpha = torch.exp(-torch.nn.functional.softplus(normal(B, T, Hv)))
    beta = torch.sigmoid(normal(B, T, Hv))
    return [x.to(dt).contiguous() for x in (q, k, v, alpha, beta)]


def prepare(case, seed):
    dev = "cuda"
    gen = torch.Generator(device=dev)
    gen.manual_seed(1000003 * int(seed) + 17)
    d = G.make_dims(case["B"], case["T"], case["Hk"], case["Hv"], case["dk"], case["dv"], case["dtype"])
    parent = _trees(case, seed)
    s = dict(op=case["op"], d=d, parent_np=parent)
    i32 = dict(dtype=torch.int32, device=dev)
    s["parent"] = torch.from_numpy(parent).to(dev)
    s["meta"] = torch.zeros(G.meta_bytes(d.B, d.T), dtype=torch.uint8, device=dev)
    s["tree_status"] = torch.zeros(d.B, **i32)
    s["raw"] = _raw(case, gen, dev)
    s["S"] = 0.1 * torch.randn((d.B, d.Hv, d.dv, d.dk), generator=gen, device=dev)
    s["conv_w"] = 0.5 * torch.randn((d.C, 4), generator=gen, device=dev)
    s["conv_state"] = torch.randn((d.B, 3, d.C), generator=gen, device=dev)
    s["out"] = torch.empty((d.B, d.T, d.Hv, d.dv), device=dev)
    s["commit_status"] = torch.zeros(d.B, **i32)
    s["accepted_np"] = _accepted(case, parent, seed)
    s["accepted"] = torch.from_numpy(s["accepted_np"]).to(dev)
    if s["op"] == "step":  # the previous decode step's tree, its metadata and inputs
        s["pparent_np"] = _trees(case, seed + 500009)
        s["accepted_np"] = _accepted(case, s["pparent_np"], seed)
        s["accepted"] = torch.from_numpy(s["accepted_np"]).to(dev)
        s["pmeta"] = torch.zeros_like(s["meta"])
        G.prepare(d, torch.from_numpy(s["pparent_np"]).to(dev), s["pmeta"])
        s["praw"] = _raw(case, gen, dev)
        s["conv_out"] = torch.empty_like(s["conv_state"])
    if s["op"] in ("commit", "verify", "chunked"):  # one of the layers that share the metadata
        G.prepare(d, s["parent"], s["meta"], s["tree_status"])
    return s


def run(s):
    """One decode step's share of a layer: its calls in order, every output."""
    d, op = s["d"], s["op"]
    if op in ("step", "verify+commit"):
        G.prepare(d, s["parent"], s["meta"], s["tree_status"])
    if op == "step":
        G.step(d, s["pmeta"], s["accepted"], *s["praw"], s["commit_status"], s["meta"], *s["raw"], s["conv_w"],
               s["conv_state"], s["conv_out"], s["S"], s["out"])
        return [s["out"], s["S"], s["conv_out"], s["commit_status"], s["tree_status"], s["meta"]]
    if op in ("verify", "chunked", "verify+commit"):
        G.verify(d, s["meta"], *s["raw"], s["conv_w"], s["conv_state"], s["S"], s["out"], chunked=op == "chunked")
        if op != "verify+commit":
            return [s["out"]]
    G.commit(d, s["meta"], s["accepted"], *s["raw"], s["conv_w"], s["conv_state"], s["S"], s["commit_status"])
    if op == "commit":
        return [s["S"], s["conv_state"], s["commit_status"]]
    return [s["out"], s["S"], s["conv_state"], s["commit_status"], s["tree_status"], s["meta"]]


# --------------------------------------------------------------------------
# what a pass cannot do without, and how exact it is
# --------------------------------------------------------------------------
def _depths(parent):
    """depth [B][T] (-1 for padding)."""
    dep = np.full(parent.shape, -1, np.int64)
    for b in range(parent.shape[0]):
        todo = [i for i in range(parent.shape[1]) if parent[b, i] == W.ROOT]
        kids = {}
        for i, p in enumerate(parent[b]):
            if p >= 0:
                kids.setdefault(int(p), []).append(i)
        lvl = 0
        while todo:
            dep[b, todo] = lvl
            todo = [c for i in todo for c in kids.get(i, ())]
            lvl += 1
    return dep


def work(case):
    """Bytes: every input read once and every output written once (a padding
    slot's output row is written, its inputs are not read; a commit reads the
    inputs of the accepted path).  Flops: the width-4 convs, one S0 readout per
    node and head, three vector operations per (node, path node), and two
    multiply-adds per state element and committed path node."""
    B, T, Hk, Hv, dk, dv, op = (case[n] for n in ("B", "T", "Hk", "Hv", "dk", "dv", "op"))
    esz = 2 if case["dtype"] == "bf16" else 4
    C = 2 * Hk * dk + Hv * dv
    row = (C + 2 * Hv) * esz  # raw inputs of one node
    state, conv = 4 * B * Hv * dv * dk, 4 * B * 3 * C
    dep = _depths(_trees(case, 0))
    nodes = int((dep >= 0).sum())
    steps = int((dep + 1).sum())
    path = nodes and int(round(steps * B / nodes))  # committed path nodes, all sequences (mean depth)
    W_ = (T + 63) // 64
    nbytes = flops = 0.0
    if op in ("step", "verify+commit"):  # prepare: parents in, metadata out
        nbytes += 4 * B * T + B * T * (8 * W_ + 24)
    if op != "commit":
        nbytes += nodes * row + 16 * C + 16 * B * T + 4 * B * T * Hv * dv + state + conv
        flops += nodes * (8.0 * C + 2.0 * Hv * dk * dv) + steps * Hv * 2.0 * (2 * dk + dv)
    if op in ("step", "commit", "verify+commit"):
        nbytes += path * row + 2 * state + 2 * conv + 16 * C + 8 * B * T
        flops += path * (8.0 * C + 4.0 * Hv * dk * dv)
    if op == "step":  # state, conv state and conv weights are read once
        nbytes -= state + conv + 16 * C
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the largest difference from 64 bits over the listed and
    some drawn cases.  Commit: fp32 sums (1.3e-7 measured, elementwise 4e-6).
    Chunked: operands of about 16 significant bits (2.7e-5).  Verify and step:
    the readout rounds both operands to 11 significant bits (1.5e-4 up to 128
    slots); above 128 slots the features are held in fp16 too (3.6e-4)."""
    if case["op"] == "commit":
        return {"rel": 1e-6, "max": 2e-5}
    if case["op"] == "chunked":
        return {"rel": 1.2e-4, "max": 4e-3}
    return {"rel": 6e-4, "max": 2e-2} if case["T"] <= 128 else {"rel": 1.5e-3, "max": 5e-2}


def _features(x, parent, conv_w, conv_state, slots):
    """Post-conv features of one sequence in float64: x raw [T][C] float64,
    rows of the real slots only."""
    T = x.shape[0]
    rows = torch.cat([x, conv_state], 0)  # conv-state slot s is row T + s
    tap = np.zeros((len(slots), 4), np.int64)
    for j, i in enumerate(slots):
        t, above = int(i), 0
        for w in (3, 2, 1, 0):
            if t >= 0:
                tap[j, w] = t
                t = int(parent[t])
            else:
                above += 1
                tap[j, w] = T + 3 - above
    y = torch.zeros((len(slots), x.shape[1]), dtype=torch.float64, device=x.device)
    for w in range(4):
        y += conv_w[:, w] * rows[torch.from_numpy(tap[:, w]).to(x.device)]
    return y * torch.sigmoid(y)


def _unit(x):
    return x / torch.sqrt((x * x).sum(-1, keepdim=True) + 1e-6)


def _split(y, case):
    Hk, Hv, dk, dv = (case[n] for n in ("Hk", "Hv", "dk", "dv"))
    n, g = y.shape[0], Hv // Hk
    q = _unit(y[:, :Hk * dk].reshape(n, Hk, dk)).repeat_interleave(g, 1).transpose(0, 1)
    k = _unit(y[:, Hk * dk:2 * Hk * dk].reshape(n, Hk, dk)).repeat_interleave(g, 1).transpose(0, 1)
    v = y[:, 2 * Hk * dk:].reshape(n, Hv, dv).transpose(0, 1)
    return q.contiguous(), k.contiguous(), v.contiguous()


def _raw64(raw, b):
    q, k, v, a, be = (x[b].double() for x in raw)
    T = q.shape[0]
    return torch.cat([q.reshape(T, -1), k.reshape(T, -1), v.reshape(T, -1)], 1), a, be


def _commit64(case, raw, parent, acc, conv_w, conv_state, S):
    """State and conv state of every sequence after the path root..accepted."""
    S, cs = S.double().clone(), conv_state.double().clone()
    for b in range(case["B"]):
        path, t = [], int(acc[b])
        while t >= 0:
            path.append(t)
            t = int(parent[b, t])
        path.reverse()
        x, a, be = _raw64(raw, b)
        _, k, v = _split(_features(x, parent[b], conv_w, cs[b], path), case)
        Sb = S[b]
        for j, t in enumerate(path):
            al, bt = a[t][:, None], be[t][:, None]
            u = (Sb * k[:, j][:, None, :]).sum(-1)  # S k
            Sb = al[..., None] * Sb + (bt * (v[:, j] - al * u))[..., None] * k[:, j][:, None, :]
        S[b] = Sb
        cs[b] = torch.cat([cs[b], x[torch.tensor(path, device=x.device)]], 0)[-3:]
    return S, cs


def _verify64(case, raw, parent, conv_w, conv_state, S):
    """Outputs of every node: the interaction system (I + X) U = beta (V - a K
    S^T) solved level by level, O = scale (a Q S^T + Y U)."""
    B, T, Hv, dk, dv = (case[n] for n in ("B", "T", "Hv", "dk", "dv"))
    dep_all = _depths(parent)
    out = torch.zeros((B, T, Hv, dv), dtype=torch.float64, device=conv_w.device)
    for b in range(B):
        dep = dep_all[b]
        slots = np.argsort(np.where(dep < 0, 1 << 30, dep), kind="stable")[:int((dep >= 0).sum())]
        n = len(slots)
        pos = np.full(T, -1)
        pos[slots] = np.arange(n)
        anc = np.zeros((n, n), bool)
        for j, i in enumerate(slots):
            if parent[b, i] >= 0:
                p = pos[parent[b, i]]
                anc[j] = anc[p]
                anc[j, p] = True
        x, a, be = _raw64(raw, b)
        idx = torch.from_numpy(slots).to(x.device)
        q, k, v = _split(_features(x, parent[b], conv_w, conv_state[b].double(), slots), case)
        A = torch.from_numpy(anc).to(x.device)
        E = torch.eye(n, dtype=torch.bool, device=x.device)
        la = torch.log(a[idx]).T  # [Hv][n]
        g = la @ (A | E).double().T
        Sb = S[b].double().transpose(1, 2)  # [Hv][dk][dv]
        ratio = torch.exp(torch.where(A | E, g[:, :, None] - g[:, None, :], torch.full_like(g[:, :, None], -1e30)))
        kt = k.transpose(1, 2).contiguous()
        bet = be[idx].T[..., None]
        X = torch.bmm(k, kt) * ratio * A * bet
        rhs = bet * (v - torch.exp(g)[..., None] * torch.bmm(k, Sb))
        U = torch.zeros_like(rhs)
        lvl = dep[slots]
        for L in range(int(lvl.max()) + 1):
            lo, hi = int(np.searchsorted(lvl, L)), int(np.searchsorted(lvl, L + 1))
            U[:, lo:hi] = rhs[:, lo:hi] - torch.bmm(X[:, lo:hi, :lo], U[:, :lo]) if lo else rhs[:, lo:hi]
        Y = torch.bmm(q, kt) * ratio * (A | E)
        o = (torch.exp(g)[..., None] * torch.bmm(q, Sb) + torch.bmm(Y, U)) / math.sqrt(dk)
        out[b, idx] = o.transpose(0, 1)
    return out


def exact(case, seed):
    s = prepare(case, seed)
    cw, cs, S = s["conv_w"].double(), s["conv_state"], s["S"]
    if s["op"] == "step":
        S, cs = _commit64(case, s["praw"], s["pparent_np"], s["accepted_np"], cw, cs, S)
        return [_verify64(case, s["raw"], s["parent_np"], cw, cs, S), S, cs, None, None, None]
    if s["op"] in ("verify", "chunked"):
        return [_verify64(case, s["raw"], s["parent_np"], cw, cs, S)]
    S2, cs2 = _commit64(case, s["raw"], s["parent_np"], s["accepted_np"], cw, cs, S)
    if s["op"] == "commit":
        return [S2, cs2, None]
    return [_verify64(case, s["raw"], s["parent_np"], cw, cs, S), S2, cs2, None, None, None]
