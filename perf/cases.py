"""The calls whose speed this library is judged by, and what they must return.

A case is one pass of one sequence-parallel rank through the library's public
entry points, with the shapes of the library's own workloads (7 heads over two
ranks, 28 query / 4 KV heads, a 131072-token ring, a packed batch of 65536
tokens, a 152064-entry vocabulary) or generic ones.  `listed()` names twelve;
`draw()` gives further ones of the same kinds over the same ranges:

  attn      one attention call over a rank's full sequence: the forward, the
            backward, or both; one sequence or a packed batch; GQA or MHA;
            head dimension 64 or 128; causal or full; dummy slots or none
  ring      one ring rank's pass over its KV chunks (contiguous or zigzag
            split), forward with the log-sum-exp merge in the epilogue,
            backward with the float32 dQ accumulator, or both
  step      one Ulysses rank's whole attention layer: pack, forward, unpack,
            pack, backward, unpack
  exchange  the copies around the all-to-alls of one Ulysses layer
  loss      token log-probabilities, SFT / DPO loss, gradient of the logits
  merge     the standalone log-sum-exp merge of two partial results

Activations are N(0, 1) in bf16 drawn on the GPU, logits N(0, 4).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2505_22296_amd as sp

DEV = "cuda"


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest call in use: one short sequence, 7 heads over two ranks
        # (this rank holds a dummy slot); launches and latency count
        dict(name="step_1k_d64", kind="step", L=1024, hs=7, hkv=7, sp=2, rank=1, D=64),
        # a short prompt on a Ulysses rank of a 28-query-head / 4-KV-head
        # model, forward only (reference model of DPO, evaluation)
        dict(name="fwd_4k", kind="attn", dir="fwd", T=4096, hq=4, hkv=1, dummies=0, D=128, causal=True,
             median=0, layout=0),
        # and its backward
        dict(name="bwd_4k", kind="attn", dir="bwd", T=4096, hq=4, hkv=1, dummies=0, D=128, causal=True,
             median=0, layout=0),
        # the same rank at the long context the library is built for
        dict(name="fwd_32k", kind="attn", dir="fwd", T=32768, hq=4, hkv=1, dummies=0, D=128, causal=True,
             median=0, layout=0),
        dict(name="bwd_32k", kind="attn", dir="bwd", T=32768, hq=4, hkv=1, dummies=0, D=128, causal=True,
             median=0, layout=0),
        # a neat-packed batch (segment lengths lognormal around 4096)
        dict(name="packed_64k", kind="attn", dir="both", T=65536, hq=4, hkv=1, dummies=0, D=128,
             causal=True, median=4096, layout=0),
        # a smaller packed batch of short, odd segments at head dimension 64
        dict(name="packed_odd_d64", kind="attn", dir="both", T=12289, hq=7, hkv=7, dummies=1, D=64,
             causal=True, median=700, layout=3),
        # one rank of a 131072-token ring in eight chunks: an earlier chunk
        # (every key visible) and its own (causal), merged
        dict(name="ring_fwd", kind="ring", dir="fwd", split="contiguous", C=16384, ring=8, rank=1, hq=28,
             hkv=4, D=128),
        dict(name="ring_bwd", kind="ring", dir="bwd", split="contiguous", C=16384, ring=8, rank=1, hq=28,
             hkv=4, D=128),
        # a zigzag rank (two pieces of one sequence a step), odd chunks
        dict(name="zigzag_odd", kind="ring", dir="both", split="zigzag", C=1367, ring=4, rank=1, hq=14,
             hkv=2, D=128),
        # all copies around the all-to-alls of a 28 / 4 head layer over eight ranks
        dict(name="exchange_7b", kind="exchange", T=4096, hs=28, hkv=4, sp=8, D=128),
        # the loss of one rank's tokens against a 152064-entry vocabulary
        dict(name="loss_4k", kind="loss", T=4096, V=152064, seqs=2, loss="dpo"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "ring", "ring", "step", "exchange", "loss", "merge"])
    if kind == "attn":
        D = rng.choice([64, 128, 128])
        causal = rng.random() < 0.85
        packed = rng.random() < 0.5
        T = _log(rng, 1000, 65536 if packed else 32768 if causal else 16384)
        hkv = rng.choice([1, 1, 2, 4])
        hq = hkv * rng.choice([1, 4, 7])
        if T > 12000:  # a rank of a long sequence holds few heads
            hkv, hq = 1, rng.choice([1, 3, 4])
        dummies = rng.choice([0, 0, 1])
        return dict(kind=kind, dir=rng.choice(["fwd", "bwd", "both"]), T=T, hq=hq, hkv=hkv, dummies=dummies, D=D,
                    causal=causal, median=_log(rng, 300, 4096) if packed else 0, layout=rng.randrange(1000))
    if kind == "ring":
        zz = rng.random() < 0.5
        ring = rng.choice([2, 4])
        hkv = rng.choice([1, 2, 4])
        return dict(kind=kind, dir=rng.choice(["fwd", "bwd", "both"]), split="zigzag" if zz else "contiguous",
                    C=_log(rng, 500, 2048 if zz else 8192), ring=ring, rank=rng.randrange(ring) if zz else 1,
                    hq=hkv * rng.choice([1, 4, 7]), hkv=hkv, D=rng.choice([64, 128, 128]))
    if kind == "step":
        hs, hkv, n = rng.choice([(7, 7, 2), (28, 4, 8), (40, 8, 16), (14, 2, 4)])
        return dict(kind=kind, L=n * _log(rng, 64, 8192 // n * 2), hs=hs, hkv=hkv, sp=n, rank=rng.randrange(n // 2 + 1),
                    D=rng.choice([64, 128]))
    if kind == "exchange":
        hs, hkv, n = rng.choice([(7, 7, 2), (28, 4, 8), (40, 8, 16), (14, 2, 4)])
        return dict(kind=kind, T=_log(rng, 256, 8192), hs=hs, hkv=hkv, sp=n, D=rng.choice([64, 128]))
    if kind == "loss":
        V = 8 * _log(rng, 4000, 19008)
        return dict(kind=kind, T=_log(rng, 100, 4000), V=V, seqs=2 * rng.randrange(1, 9), loss=rng.choice(["sft", "dpo"]))
    return dict(kind="merge", T=_log(rng, 500, 16384), H=rng.choice([4, 7, 28]), D=rng.choice([64, 128]),
                part=rng.choice(["bf16", "f32"]))


# ------------------------------------------------------------- descriptions
def _padded(hs, n):
    return hs if hs % n == 0 else hs + n - hs % n


def _q_map(hs, n):
    """Slot j*H_loc + h carries global head j*H_loc + h, or -1 (a dummy)."""
    m = np.arange(_padded(hs, n), dtype=np.int32)
    m[m >= hs] = -1
    return m


def _kv_ranges(hs, hkv, n):
    hloc, g = _padded(hs, n) // n, hs // hkv
    if hs == hkv:
        return [(min(j * hloc, hs), min((j + 1) * hloc, hs)) for j in range(n)], hloc
    real = [[h for h in range(j * hloc, (j + 1) * hloc) if h < hs] for j in range(n)]
    r = [(x[0] // g, x[-1] // g + 1) if x else (0, 0) for x in real]
    return r, max(b - a for a, b in r)


def _kv_map(hs, hkv, n):
    """Rank j receives the KV heads its real query heads read, then -1s."""
    r, width = _kv_ranges(hs, hkv, n)
    m = np.full(n * width, -1, dtype=np.int32)
    for j, (a, b) in enumerate(r):
        m[j * width:j * width + b - a] = np.arange(a, b)
    return m


def _ramp(cu, base=0):
    return np.concatenate([base + np.arange(b - a) for a, b in zip(cu[:-1], cu[1:])]).astype(np.int32)


def _lengths(case):
    """Segment lengths of an attn case: one sequence, or lognormal lengths
    around the median (from the case's own layout number) until T."""
    T, median = case["T"], case["median"]
    if not median:
        return [T]
    rng, out, left = np.random.default_rng(case["layout"]), [], T
    while left > 0:
        n = min(left, int(np.clip(np.rint(rng.lognormal(math.log(median), 1.0)), median // 8, 4 * median)))
        out.append(n)
        left -= n
    return out


def _problem(case):
    """The attention of one case, as the heads and tokens that its rank sees:
    H slots, `real` of them computed (real slot y reads local KV head kv[y]),
    and per call (one, or one a ring step) the key positions."""
    if case["kind"] == "attn":
        cu = np.concatenate([[0], np.cumsum(_lengths(case))]).astype(np.int32)
        real, H = case["hq"], case["hq"] + case["dummies"]
        g = real // case["hkv"]
        # the last of two ranks when there is a dummy slot (the first holds H
        # real heads on KV heads of its own)
        heads = dict(H_loc=H, head_offset=0, num_real_heads=real, num_padded_heads=H, gqa_group=g,
                     Hkv_loc=case["hkv"], kv_head_offset=0)
        kv = [y // g for y in range(real)]
        if case["dummies"]:
            hs = H + real
            heads.update(head_offset=H, num_real_heads=hs, num_padded_heads=2 * H)
            if g == 1:
                heads.update(gqa_group=1, Hkv_loc=H, kv_head_offset=H)
                kv = list(range(real))
            else:
                gg = hs  # one KV head for all: what is left of a larger group
                heads.update(gqa_group=gg, Hkv_loc=1, kv_head_offset=0)
                kv = [0] * real
        return dict(T=case["T"], D=case["D"], H=H, real=real, Hkv=heads["Hkv_loc"], kv=kv, heads=heads, cu=cu,
                    pos_q=_ramp(cu), pos_k=[_ramp(cu)], causal=case["causal"], single=False)
    if case["kind"] == "step":
        n, hs, hkv, j = case["sp"], case["hs"], case["hkv"], case["rank"]
        H = _padded(hs, n) // n
        r, width = _kv_ranges(hs, hkv, n)
        off = r[j][0] if hs != hkv else j * H
        real = max(0, min(H, hs - j * H))
        g = hs // hkv
        cu = np.array([0, case["L"]], dtype=np.int32)
        heads = dict(H_loc=H, head_offset=j * H, num_real_heads=hs, num_padded_heads=_padded(hs, n), gqa_group=g,
                     Hkv_loc=width, kv_head_offset=off)
        return dict(T=case["L"], D=case["D"], H=H, real=real, Hkv=width, kv=[(j * H + y) // g - off for y in range(real)],
                    heads=heads, cu=cu, pos_q=_ramp(cu), pos_k=[_ramp(cu)], causal=True, single=False)
    C, n, r = case["C"], case["ring"], case["rank"]
    heads = dict(H_loc=case["hq"], head_offset=0, num_real_heads=case["hq"], num_padded_heads=case["hq"],
                 gqa_group=case["hq"] // case["hkv"], Hkv_loc=case["hkv"], kv_head_offset=0)
    one = np.arange(C, dtype=np.int32)
    zz = case["split"] == "zigzag"

    def pos(rank):
        return np.concatenate([rank * C + one, (2 * n - 1 - rank) * C + one]) if zz else rank * C + one
    cu = np.array([0, C, 2 * C] if zz else [0, C], dtype=np.int32)
    steps = [pos((r - s) % n) for s in range(n)] if zz else [pos(c) for c in range(r + 1)]
    g = case["hq"] // case["hkv"]
    return dict(T=int(cu[-1]), D=case["D"], H=case["hq"], real=case["hq"], Hkv=case["hkv"],
                kv=[y // g for y in range(case["hq"])], heads=heads, cu=cu, pos_q=pos(r), pos_k=steps, causal=True,
                single=zz)


def _pairs(p):
    """(query, key) pairs that one head computes, over all calls."""
    if p["single"] or len(p["pos_k"]) > 1:
        return int(sum(np.searchsorted(k, p["pos_q"], side="right").astype(np.int64).sum() for k in p["pos_k"]))
    n = np.diff(p["cu"]).astype(np.int64)
    return int((n * (n + 1) // 2 if p["causal"] else n * n).sum())


def _desc(p, step, **flags):
    return sp.Desc(T_q=p["T"], T_k=p["T"], head_dim=p["D"], cu_seqlens_q=p["cu"], cu_seqlens_k=p["cu"],
                   position_ids_q=p["pos_q"], position_ids_k=p["pos_k"][step], causal=p["causal"],
                   softmax_scale=1.0 / math.sqrt(p["D"]), single_sequence=p["single"], **p["heads"], **flags)


# ------------------------------------------------------------------- inputs
def _randn(gen, *shape, scale=1.0):
    x = torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32)
    return (x * scale if scale != 1.0 else x).to(torch.bfloat16)


def _inputs(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    x = {}
    if case["kind"] in ("attn", "ring", "step"):
        p = _problem(case)
        T, D, H, Hkv, n = p["T"], p["D"], p["H"], p["Hkv"], len(p["pos_k"])
        x.update(q=_randn(gen, T, H, D), do=_randn(gen, T, H, D))
        x.update(k=[_randn(gen, T, Hkv, D) for _ in range(n)], v=[_randn(gen, T, Hkv, D) for _ in range(n)])
        x["q"][:, p["real"]:] = 0  # dummy slots arrive as zeros from the pack
        x["do"][:, p["real"]:] = 0
    if case["kind"] in ("step", "exchange"):
        n, hs, hkv, D = case["sp"], case["hs"], case["hkv"], case["D"]
        T = case["L"] // n if case["kind"] == "step" else case["T"]
        x.update({a: _randn(gen, T, hs, D) for a in ("q_pre", "do_pre")})
        x.update({a: _randn(gen, T, hkv, D) for a in ("k_pre", "v_pre")})
        width = len(_kv_map(hs, hkv, n)) // n
        x.update({a: _randn(gen, n, T, width, D) for a in ("dk_recv", "dv_recv")})
        if case["kind"] == "exchange":
            x.update({a: _randn(gen, n, T, _padded(hs, n) // n, D) for a in ("o_recv", "dq_recv")})
    if case["kind"] == "loss":
        T, V, S = case["T"], case["V"], case["seqs"]
        x["logits"] = torch.empty((T, V), dtype=torch.bfloat16, device=DEV)
        for t in range(0, T, 512):
            x["logits"][t:t + 512] = _randn(gen, min(512, T - t), V, scale=2.0)
        x["labels"] = torch.randint(0, V, (T,), generator=gen, device=DEV, dtype=torch.int32)
        cu = np.linspace(0, T, S + 1).astype(np.int32)
        for a, b in zip(cu[:-1], cu[1:]):  # a quarter of each is prompt, not scored
            x["labels"][int(a):int(a) + int(b - a) // 4] = -100
        x["cu"] = cu
        # the reference model scores its sequences much like the policy does
        lp = torch.cat([torch.log_softmax(x["logits"][t:t + 512].float(), 1).gather(
            1, x["labels"][t:t + 512].long().clamp(0)[:, None])[:, 0] for t in range(0, T, 512)])
        lp = torch.where(x["labels"] >= 0, lp, torch.zeros_like(lp))
        sums = torch.stack([lp[int(a):int(b)].sum() for a, b in zip(cu[:-1], cu[1:])])
        x["refs"] = (sums + 4.0 * torch.randn(S, generator=gen, device=DEV))[None].contiguous()
    if case["kind"] == "merge":
        T, H, D = case["T"], case["H"], case["D"]
        x["o_acc"] = torch.randn((T, H, D), generator=gen, device=DEV)
        x["lse_acc"] = torch.randn((H, T), generator=gen, device=DEV) + 8.0
        part = torch.randn((T, H, D), generator=gen, device=DEV)
        x["o_part"] = part.to(torch.bfloat16) if case["part"] == "bf16" else part
        x["lse_part"] = torch.randn((H, T), generator=gen, device=DEV) + 8.0
    return x


def _ws(desc, op):
    return sp.sp_attn_workspace_size(desc, op)


def prepare(case, seed):
    """Inputs, descriptors, workspaces and output buffers, kept from step to
    step by a training loop; a backward case also has its forward's results."""
    s = dict(case=case, **_inputs(case, seed))
    kind = case["kind"]
    new = lambda *shape, dtype=torch.bfloat16: torch.empty(shape, dtype=dtype, device=DEV)  # noqa: E731
    if kind in ("attn", "ring", "step"):
        p = _problem(case)
        n = len(p["pos_k"])
        ring = kind == "ring"
        s["desc"] = [_desc(p, c) for c in range(n)]
        s["desc_b"] = [_desc(p, c, rowstats_ready=ring and c > 0, dq_acc_init=ring and c == 0) for c in range(n)]
        op = sp.SP_OP_RING_STEP if ring else sp.SP_OP_FWD
        need = max(max(_ws(d, op) for d in s["desc"]), max(_ws(d, sp.SP_OP_BWD) for d in s["desc_b"]))
        s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
        T, D, H = p["T"], p["D"], p["H"]
        s.update(o=new(T, H, D), lse=new(H, T, dtype=torch.float32), dq=new(T, H, D),
                 dk=[new(T, p["Hkv"], D) for _ in range(n)], dv=[new(T, p["Hkv"], D) for _ in range(n)])
        if ring:
            s.update(o_acc=new(T, H, D, dtype=torch.float32), dq_acc=new(T, H, D, dtype=torch.float32))
        if case.get("dir") == "bwd":
            _forward(s)
    if kind in ("step", "exchange"):
        n, hs, hkv, D = case["sp"], case["hs"], case["hkv"], case["D"]
        T = s["q_pre"].shape[0]
        s["q_map"], s["kv_map"] = _q_map(hs, n), _q_map(hs, n) if hs == hkv else _kv_map(hs, hkv, n)
        H, Hk = len(s["q_map"]) // n, len(s["kv_map"]) // n
        s.update(q_send=new(n, T, H, D), do_send=new(n, T, H, D), k_send=new(n, T, Hk, D), v_send=new(n, T, Hk, D),
                 o_pre=new(T, hs, D), dq_pre=new(T, hs, D), dk_pre=new(T, hkv, D), dv_pre=new(T, hkv, D))
    if kind == "loss":
        T, S = case["T"], case["seqs"]
        s.update(logp=new(T, dtype=torch.float32), lse=new(T, dtype=torch.float32), sums=new(1, S, dtype=torch.float32),
                 value=new(1, dtype=torch.float32), grad=new(1, S, dtype=torch.float32),
                 dlogits=new(T, case["V"]))
    if kind == "merge":
        s.update(acc=torch.empty_like(s["o_acc"]), acc_lse=torch.empty_like(s["lse_acc"]),
                 o_out=torch.empty_like(s["o_acc"], dtype=torch.bfloat16))
    return s


# ---------------------------------------------------------------- the calls
def _forward(s):
    n = len(s["desc"])
    if s["case"]["kind"] != "ring":
        sp.sp_attn_fwd(s["desc"][0], s["q"], s["k"][0], s["v"][0], s["o"], s["lse"], workspace=s["ws"])
        return [s["o"], s["lse"]]
    for c in range(n):
        sp.sp_ring_step(s["desc"][c], s["q"], s["k"][c], s["v"][c], s["o_acc"], s["lse"], init=c == 0,
                        o_out=s["o"] if c == n - 1 else None, workspace=s["ws"])
    return [s["o"], s["lse"]]


def _backward(s):
    n = len(s["desc_b"])
    ring = s["case"]["kind"] == "ring"
    for c in range(n):
        sp.sp_attn_bwd(s["desc_b"][c], s["q"], s["k"][c], s["v"][c], s["o"], s["lse"], s["do"],
                       dq=s["dq"] if c == n - 1 else None, dq_acc=s["dq_acc"] if ring else None, dk=s["dk"][c],
                       dv=s["dv"][c], workspace=s["ws"])
    return [s["dq"], *s["dk"], *s["dv"]]


def _unpack_kv(s, recv, dst):
    if s["case"]["hs"] == s["case"]["hkv"]:
        return sp.sp_ulysses_unpack(recv, s["kv_map"], s["case"]["hkv"], dst=dst)
    return sp.sp_ulysses_unpack_add(recv, s["kv_map"], s["case"]["hkv"], dst=dst)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("attn", "ring"):
        return (_forward(s) if case["dir"] != "bwd" else []) + (_backward(s) if case["dir"] != "fwd" else [])
    if kind in ("step", "exchange"):
        n, hs = case["sp"], case["hs"]
        H, Hk = len(s["q_map"]) // n, len(s["kv_map"]) // n
        sp.sp_ulysses_pack(s["q_pre"], n, H, s["q_map"], dst=s["q_send"])
        sp.sp_ulysses_pack(s["k_pre"], n, Hk, s["kv_map"], dst=s["k_send"])
        sp.sp_ulysses_pack(s["v_pre"], n, Hk, s["kv_map"], dst=s["v_send"])
        out = []
        o, dq = s.get("o_recv"), s.get("dq_recv")
        if kind == "step":  # the full sequence is in q, k, v as received
            out += _forward(s)
            o, dq = s["o"].view(s["q_send"].shape), s["dq"].view(s["q_send"].shape)
        sp.sp_ulysses_unpack(o, s["q_map"], hs, dst=s["o_pre"])
        sp.sp_ulysses_pack(s["do_pre"], n, H, s["q_map"], dst=s["do_send"])
        if kind == "step":
            out += _backward(s)
        sp.sp_ulysses_unpack(dq, s["q_map"], hs, dst=s["dq_pre"])
        _unpack_kv(s, s["dk_recv"], s["dk_pre"])
        _unpack_kv(s, s["dv_recv"], s["dv_pre"])
        return out + [s[a] for a in ("q_send", "k_send", "v_send", "do_send", "o_pre", "dq_pre", "dk_pre", "dv_pre")]
    if kind == "loss":
        sp.sp_token_logprob(s["logits"], s["labels"], s["cu"], logp=s["logp"], lse=s["lse"], seq_sum=s["sums"][0])
        dpo = case["loss"] == "dpo"
        sp.sp_loss_reduce(s["sums"], sp.SP_LOSS_DPO if dpo else sp.SP_LOSS_SFT, _coef(case),
                          ref_partial_sums=s["refs"] if dpo else None, loss=s["value"], grad=s["grad"])
        sp.sp_token_logprob_bwd(s["logits"], s["labels"], s["lse"], s["cu"], s["grad"][0], dlogits=s["dlogits"])
        return [s["logp"], s["lse"], s["sums"], s["value"], s["grad"], s["dlogits"]]
    s["acc"].copy_(s["o_acc"])  # the merge works in place: on a copy of the partial it folds into
    s["acc_lse"].copy_(s["lse_acc"])
    sp.sp_lse_merge(s["acc"], s["acc_lse"], s["o_part"], s["lse_part"], o_out=s["o_out"])
    return [s["acc"], s["acc_lse"], s["o_out"]]


def _coef(case):
    return 0.1 if case["loss"] == "dpo" else 1.0 / case["T"]


# ------------------------------------------------------ what a pass must do
def work(case):
    b = f = 0
    kind = case["kind"]
    if kind in ("attn", "ring", "step"):
        p = _problem(case)
        rows, keys = p["T"] * p["D"], p["T"] * p["D"] * p["Hkv"] * len(p["pos_k"])
        d = case.get("dir", "both")
        f = (4 if d == "fwd" else 10 if d == "bwd" else 14) * p["D"] * p["real"] * _pairs(p)
        b = 2 * rows * p["real"] + 2 * 2 * keys + 4 * p["T"] * p["real"]  # q, k, v, lse
        b += 2 * rows * p["H"]                                           # o
        if d != "fwd":
            b += 2 * rows * (p["real"] + p["H"]) + 2 * 2 * keys          # do, dq, dk, dv
    if kind in ("step", "exchange"):
        n, hs, hkv = case["sp"], case["hs"], case["hkv"]
        row = 2 * case["D"] * (case["L"] // n if kind == "step" else case["T"])
        qm, km = _q_map(hs, n), _q_map(hs, n) if hs == hkv else _kv_map(hs, hkv, n)
        named = int((km >= 0).sum())
        b += row * 2 * (hs + len(qm)) + row * 2 * (named + len(km)) + row * 2 * 2 * hs + row * 2 * (named + hkv)
    if kind == "loss":
        b = 2 * 3 * case["T"] * case["V"]
    if kind == "merge":
        n = case["T"] * case["H"] * case["D"]
        # the copies read and write the partial once, the merge again
        b = n * (8 + 8 + (2 if case["part"] == "bf16" else 4) + 2) + 4 * 5 * case["T"] * case["H"]
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    """About four times the library's measured distance from the 64-bit
    results: bf16 operands of the second product, bf16 outputs (2e-3 to 2.7e-3
    per tensor).  Copies are exact but for the summed K/V gradients' one
    rounding, which is bit for bit defined."""
    kind = case["kind"]
    if kind == "exchange":
        return "exact"
    if kind == "loss":
        return {"rel": 8e-3, "max": 0.1}
    if kind == "merge":
        return {"rel": 8e-3, "max": 0.05}
    return {"rel": 1e-2, "max": 0.1}


# ----------------------------------------------------------- 64-bit results
def _exact_attention(x, p, want_b):
    """O, LSE and, with want_b, dQ and the dK, dV of every step, in float64:
    whole masked softmax rows of each head over the keys of all steps."""
    T, D, H = p["T"], p["D"], p["H"]
    k, v = torch.cat(x["k"]).double(), torch.cat(x["v"]).double()
    pq = torch.from_numpy(np.asarray(p["pos_q"], np.int64)).to(DEV)
    pk = torch.from_numpy(np.concatenate(p["pos_k"]).astype(np.int64)).to(DEV)
    n = len(p["pos_k"])
    segs = [(0, T, 0, n * T)] if p["single"] or n > 1 else [(int(a), int(b), int(a), int(b))
                                                            for a, b in zip(p["cu"][:-1], p["cu"][1:])]
    o = torch.zeros((T, H, D), dtype=torch.float64, device=DEV)
    lse = torch.full((H, T), -math.inf, dtype=torch.float64, device=DEV)
    dq, dk, dv = torch.zeros_like(o), torch.zeros_like(k), torch.zeros_like(v)
    scale = 1.0 / math.sqrt(D)
    for y in range(p["real"]):
        g = p["kv"][y]
        for qa, qb, ka, kb in segs:
            K, V = k[ka:kb, g].contiguous(), v[ka:kb, g].contiguous()
            Kt, Vt = K.t().contiguous(), V.t().contiguous()
            step = max(256, (1 << 27) // max(1, kb - ka))
            for a in range(qa, qb, step):
                b = min(qb, a + step)
                kn = kb if not p["causal"] or n > 1 or p["single"] else min(kb, b)
                m = kn - ka
                q = x["q"][a:b, y].double()
                s = q @ Kt[:, :m].contiguous() * scale
                if p["causal"]:
                    s.masked_fill_(pk[None, ka:kn] > pq[a:b, None], -math.inf)
                L = torch.logsumexp(s, 1)
                s = s.sub_(L[:, None]).exp_()
                O = s @ V[:m]
                o[a:b, y], lse[y, a:b] = O, L
                if not want_b:
                    continue
                do = x["do"][a:b, y].double()
                dv[ka:kn, g] += s.t().contiguous() @ do
                dp = do @ Vt[:, :m].contiguous()
                dp.sub_((do * O).sum(1)[:, None]).mul_(s).mul_(scale)
                dq[a:b, y] = dp @ K[:m]
                dk[ka:kn, g] += dp.t().contiguous() @ q
    return o, lse, dq, [t.contiguous() for t in dk.split(T)], [t.contiguous() for t in dv.split(T)]


def _exact_pack(src, m, n):
    T, _, D = src.shape
    out = torch.zeros((n, T, len(m) // n, D), dtype=torch.float64, device=DEV)
    for i, g in enumerate(m):
        if g >= 0:
            out[i // (len(m) // n), :, i % (len(m) // n)] = src[:, int(g)].double()
    return out


def _exact_unpack(src, m, heads):
    n, T, H, D = src.shape
    out = torch.zeros((T, heads, D), dtype=torch.float64, device=DEV)
    for i, g in enumerate(m):
        if g >= 0:
            out[:, int(g)] += src[i // H, :, i % H].double()
    return out


def exact(case, seed):
    x = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("attn", "ring"):
        d = case["dir"]
        o, lse, dq, dk, dv = _exact_attention(x, _problem(case), d != "fwd")
        return ([o, lse] if d != "bwd" else []) + ([dq, *dk, *dv] if d != "fwd" else [])
    if kind in ("step", "exchange"):
        n, hs, hkv = case["sp"], case["hs"], case["hkv"]
        qm, km = _q_map(hs, n), _q_map(hs, n) if hs == hkv else _kv_map(hs, hkv, n)
        out, o, dq = [], x.get("o_recv"), x.get("dq_recv")
        if kind == "step":
            o, lse, dq, dk, dv = _exact_attention(x, _problem(case), True)
            out = [o, lse, dq, *dk, *dv]
            shape = (n, case["L"] // n, len(qm) // n, case["D"])
            o, dq = o.view(shape), dq.view(shape)
        out += [_exact_pack(x[a], m, n) for a, m in (("q_pre", qm), ("k_pre", km), ("v_pre", km), ("do_pre", qm))]
        out += [_exact_unpack(o, qm, hs), _exact_unpack(dq, qm, hs)]
        return out + [_exact_unpack(x[a], km, hkv) for a in ("dk_recv", "dv_recv")]
    if kind == "loss":
        T, V, S, cu = case["T"], case["V"], case["seqs"], x["cu"]
        lab = x["labels"].long()
        scored = (lab >= 0) & (lab < V)
        at = lab.clamp(0, V - 1)
        lse = torch.empty(T, dtype=torch.float64, device=DEV)
        logp = torch.empty_like(lse)
        for t in range(0, T, 512):
            z = x["logits"][t:t + 512].double()
            lse[t:t + 512] = torch.logsumexp(z, 1)
            logp[t:t + 512] = z.gather(1, at[t:t + 512, None])[:, 0]
        logp = torch.where(scored, logp - lse, torch.zeros_like(lse))
        sums = torch.stack([logp[int(a):int(b)].sum() for a, b in zip(cu[:-1], cu[1:])])
        c = _coef(case)
        if case["loss"] == "sft":
            value, grad = -c * sums.sum(), torch.full_like(sums, -c)
        else:
            d = sums - x["refs"][0].double()
            z = c * (d[0::2] - d[1::2])
            value = torch.nn.functional.softplus(-z).mean()
            w = -c * torch.sigmoid(-z) / (S // 2)
            grad = torch.stack([w, -w], 1).reshape(-1)
        g = torch.repeat_interleave(grad, torch.from_numpy(np.diff(cu).astype(np.int64)).to(DEV)) * scored
        dz = torch.empty((T, V), dtype=torch.float64, device=DEV)
        for t in range(0, T, 512):
            b = min(T, t + 512)
            blk = (x["logits"][t:b].double() - lse[t:b, None]).exp_().neg_()
            blk[torch.arange(b - t, device=DEV), at[t:b]] += 1.0
            dz[t:b] = blk * g[t:b, None]
        return [logp, lse, sums[None], value[None], grad[None], dz]
    a, b = x["lse_acc"].double(), x["lse_part"].double()
    L = torch.logaddexp(a, b)
    wa, wb = ((t - L).exp().t()[:, :, None] for t in (a, b))
    o = wa * x["o_acc"].double() + wb * x["o_part"].double()
    return [o, L, o]
