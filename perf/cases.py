"""The workloads whose speed this library is measured by.

Each case is one call sequence that a program makes through the public
binding: the decode stacks of a serving loop, the attention of a prefill and
of a decode step, FFN forwards, whole FFN training steps, and the complete
gated FFN at the widths of the kernel study.  ``listed()`` holds one case per
use; ``draw()`` gives further cases over the same ranges.  ``exact()``
recomputes a case's outputs with plain torch in 64 bits.
"""

from __future__ import annotations

import math

import torch
import torch.nn.functional as F

import paper_2609_32814_amd as starq

DEV = "cuda"
BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64


# ---- cases -------------------------------------------------------------------


def listed():
    return [
        # One sequence being generated: a step through the FFNs of a 12-layer
        # model of width 768, its positions typed cyclically with q = 2.
        dict(name="decode_one_row", kind="decode", gated=False, law="star", q=2, D=768, F=3072, layers=12, M=1),
        # A batch of 48 sequences through the pretraining pilot's bias-free
        # SwiGLU stack (tensor-square law, q = 4).
        dict(name="decode_gated_48_rows", kind="decode", gated=True, law="tensor2", q=4, D=768, F=1536, layers=12,
             M=48),
        # A few sequences through FFNs of a wide model, where the projections
        # have more column tiles than the chip has CUs.
        dict(name="decode_wide_8_rows", kind="decode", gated=False, law="star", q=4, D=2560, F=9728, layers=4, M=8),
        # Attention of a decode step for 64 sequences at random depths of a
        # 2048-position cache, 12 heads of 64.
        dict(name="attention_decode_64", kind="attn_decode", law="star", q=4, B=64, S=2048, H=12, Hkv=12, D=64),
        # Attention of a training forward or a prefill at the pilot's context
        # length, log-sum-exp included.
        dict(name="attention_forward_16x1536", kind="attn", law="star", q=4, B=16, S=1536, H=12, Hkv=12, D=64,
             lse=True),
        # Grouped-query attention with 128-wide heads over an odd prompt
        # length (prefill).
        dict(name="attention_prefill_grouped_2777", kind="attn", law="star", q=4, B=2, S=2777, H=32, Hkv=8, D=128,
             lse=False),
        # FFN forward (prefill or evaluation) of the 768-wide model over 8
        # sequences of 1024 positions.
        dict(name="ffn_forward_8192", kind="ffn", train=False, law="star", q=2, dtype="bf16", act="gelu", D=768,
             F=3072, M=8192, ragged=False, bias=True),
        # Training step of the same FFN: forward, then every gradient.
        dict(name="ffn_train_16384", kind="ffn", train=True, law="star", q=2, dtype="bf16", act="gelu", D=768,
             F=3072, M=16384, ragged=False, bias=True),
        # Training step of the pilot's SwiGLU FFN (tensor-square law, q = 4).
        dict(name="swiglu_train_16384", kind="swiglu", law="tensor2", q=4, dtype="bf16", D=768, F=1536, M=16384),
        # Complete SwiGLU forward with the merged gate/up bank at a kernel
        # study width (4096 -> 12288), q = 32, over a 2048-token prompt ...
        dict(name="merged_ffn_2048_tokens", kind="merged", law="star", q=32, D=4096, F=12288, M=2048),
        # ... and over one new token.
        dict(name="merged_ffn_one_token", kind="merged", law="star", q=32, D=4096, F=12288, M=1),
        # Training step in fp32 with unequal group widths, an odd row count
        # and the tanh form of GELU.
        dict(name="ffn_train_fp32_ragged_1111", kind="ffn", train=True, law="star", q=3, dtype="f32",
             act="gelu_tanh", D=768, F=2304, M=1111, ragged=True, bias=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(v, m):
    return max(m, int(v) // m * m)


def draw(rng):
    """One more case; redrawn until it costs no more than the largest listed ones."""
    top = [work(c) for c in listed()]
    max_flops, max_bytes = max(w["flops"] for w in top), max(w["bytes"] for w in top)
    while True:
        case = _draw(rng)
        w = work(case)
        # 32-bit products run at a sixteenth of the 16-bit rate
        scale = 16 if case.get("dtype") == "f32" else 1
        if w["flops"] * scale <= max_flops and w["bytes"] <= max_bytes:
            return case


def _draw(rng):
    kind = rng.choice(["decode", "decode", "attn_decode", "attn", "ffn", "ffn", "ffn", "swiglu", "merged"])
    if kind == "decode":
        gated = rng.random() < 0.4
        law = rng.choice(["star", "dense", "tensor2"])
        q = 4 if law == "tensor2" else rng.choice([2, 3, 4, 8])
        D = _mult(_log_int(rng, 256, 768 if gated else 4096), 8 * q)
        Fw = _mult(D * rng.choice([2, 3, 4]), 8 * q)
        layers = rng.randint(2, 12) if D <= 1024 else rng.randint(1, 4)
        return dict(kind=kind, gated=gated, law=law, q=q, D=D, F=Fw, layers=layers,
                    M=_log_int(rng, 1, 40 if gated else 64))
    if kind in ("attn_decode", "attn"):
        law = rng.choice(["star", "star", "dense", "tensor2"])
        q = 4 if law == "tensor2" else rng.choice([2, 4, 8])
        D = rng.choice([64, 128])
        Hkv = rng.choice([2, 4, 8, 12])
        H = Hkv * rng.choice([1, 1, 2, 4])
        if kind == "attn_decode":
            return dict(kind=kind, law=law, q=q, B=_log_int(rng, 1, 64), S=_log_int(rng, 200, 8192), H=H, Hkv=Hkv,
                        D=D)
        return dict(kind=kind, law=law, q=q, B=_log_int(rng, 1, 16), S=_log_int(rng, 60, 4096), H=H, Hkv=Hkv, D=D,
                    lse=rng.random() < 0.5)
    if kind == "ffn":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        law = rng.choice(["star", "star", "dense", "tensor2", "graph"])
        q = 4 if law == "tensor2" else rng.choice([2, 3, 4, 8, 16])
        D = _mult(_log_int(rng, 256, 4096 if dtype == "bf16" else 1024), 16 * q)
        return dict(kind=kind, train=rng.random() < 0.5, law=law, q=q, dtype=dtype,
                    act=rng.choice(["gelu", "gelu", "gelu_tanh", "none"]), D=D, F=_mult(D * rng.choice([2, 3, 4]), 16 * q),
                    M=_log_int(rng, 64, 16384 if dtype == "bf16" else 4096), ragged=rng.random() < 0.4,
                    bias=rng.random() < 0.7)
    if kind == "swiglu":
        law = rng.choice(["star", "tensor2", "dense"])
        q = 4 if law == "tensor2" else rng.choice([2, 4, 8])
        D = _mult(_log_int(rng, 256, 2048), 16 * q)
        return dict(kind=kind, law=law, q=q, dtype="bf16", D=D, F=_mult(D * rng.choice([1.5, 2, 2.67]), 16 * q),
                    M=_log_int(rng, 64, 16384))
    q = rng.choice([8, 16, 32, 64])
    D = _mult(_log_int(rng, 1024, 7168), 8 * q)
    return dict(kind="merged", law="star", q=q, D=D, F=_mult(D * rng.choice([0.375, 2, 3, 3.8]), 8 * q),
                M=rng.choice([1, _log_int(rng, 2, 64), _log_int(rng, 64, 4096)]))


# ---- layouts and types ---------------------------------------------------------


def _widths(total, q, ragged):
    """q group widths, multiples of 8: equal, or spread about the mean."""
    if not ragged:
        return [total // q] * q
    unit, w = total // 8, []
    for g in range(q):
        mean = unit // q
        w.append(max(1, mean + ((g * 7 + 3) % 5 - 2) * max(1, mean // 8)))
    w[-1] = max(1, w[-1] + unit - sum(w))
    w[0] += unit - sum(w)
    return [8 * v for v in w]


def _edges(q):
    return [[int(i != j and (i + 2 * j) % 3 != 0) for j in range(q)] for i in range(q)]


def _algebras(case):
    q, law, ragged = case["q"], case["law"], case.get("ragged", False)
    d, f = _widths(case["D"], q, ragged), _widths(case["F"], q, ragged)
    edges = _edges(q) if law == "graph" else None
    return starq.Algebra(q, d, f, law, edges), starq.Algebra(q, f, d, law, edges)


def _support(law, q, i, j):
    """Input groups that output group j of a type-i row reads."""
    if law == "dense":
        return list(range(q))
    if law == "tensor2":
        return [k for k in range(q) if ((k ^ i) & (k ^ j)) == 0]
    if law == "graph" and i != j and not _edges(q)[i][j]:
        return []
    return sorted({i, j})


def _features(law, q, i, j):
    """Feature groups that the score of a type-i query and a type-j key keeps."""
    return _support(law if law != "graph" else "star", q, i, j)


def _types(positions, case):
    """Cyclic types; the tensor-square law's pilot types run in intervals."""
    q = case["q"]
    if case["law"] == "tensor2":
        return ((positions % 768) * q // 768).to(torch.int32)
    return (positions % q).to(torch.int32)


class _Draws:
    def __init__(self, seed):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(int(seed))

    def normal(self, shape, std, dtype):
        return (torch.randn(shape, generator=self.gen, device=DEV, dtype=F32) * std).to(dtype)

    def ints(self, lo, hi, n):
        return torch.randint(lo, hi, (n,), generator=self.gen, device=DEV)


# ---- what a program has in hand ------------------------------------------------


def _inputs(case, seed):
    """The tensors of a case, made from the seed alone."""
    r = _Draws(seed)
    kind, t = case["kind"], {}
    if kind == "decode":
        D, Fw, L, M = case["D"], case["F"], case["layers"], case["M"]
        t["types"] = _types(r.ints(0, 2048, M), case)
        t["X"] = r.normal((M, D), 1.0, BF16)
        std = 0.02
        t["W_up"] = [r.normal((D, Fw), std, BF16) for _ in range(L)]
        t["W_down"] = [r.normal((Fw, D), std, BF16) for _ in range(L)]
        if case["gated"]:
            t["W_gate"] = [r.normal((D, Fw), std, BF16) for _ in range(L)]
        else:
            t["b_up"] = [r.normal((Fw,), std, F32) for _ in range(L)]
            t["b_down"] = [r.normal((D,), std, F32) for _ in range(L)]
    elif kind in ("attn", "attn_decode"):
        B, S, H, Hkv, D = case["B"], case["S"], case["H"], case["Hkv"], case["D"]
        t["types"] = _types(torch.arange(S, device=DEV), case)
        t["Q"] = r.normal((B, S, H, D) if kind == "attn" else (B, H, D), 1.0, BF16)
        t["K"] = r.normal((B, S, Hkv, D), 1.0, BF16)
        t["V"] = r.normal((B, S, Hkv, D), 1.0, BF16)
        if kind == "attn_decode":
            t["lens"] = r.ints(1, S + 1, B).to(torch.int32)
    else:
        D, Fw, M = case["D"], case["F"], case["M"]
        dt = F32 if case.get("dtype") == "f32" else BF16
        start = int(r.ints(0, 4096, 1).item())
        t["types"] = _types((torch.arange(M, device=DEV) + start) % 4096, case)
        t["X"] = r.normal((M, D), 1.0, dt)
        t["W_up"] = r.normal((D, Fw), 1.0 / math.sqrt(D), dt)
        t["W_down"] = r.normal((Fw, D), 1.0 / math.sqrt(Fw), dt)
        if kind in ("swiglu", "merged"):
            t["W_gate"] = r.normal((D, Fw), 1.0 / math.sqrt(D), dt)
        if kind == "ffn" and case["bias"]:
            t["b_up"], t["b_down"] = r.normal((Fw,), 0.02, F32), r.normal((D,), 0.02, F32)
        if kind == "swiglu" or (kind == "ffn" and case["train"]):
            t["dY"] = r.normal((M, D), 1.0, dt)
    return t


def prepare(case, seed):
    st = _inputs(case, seed)
    st["case"] = case
    kind = case["kind"]
    if kind == "decode":
        st["up"], st["down"] = _algebras(case)
        nbytes = starq.star_workspace_bytes("decode", st["up"], st["down"], case["M"])
        st["ws"] = torch.empty(max(nbytes, 16), dtype=torch.uint8, device=DEV)
    elif kind in ("attn", "attn_decode"):
        st["shape"] = starq.AttnShape(case["B"], case["S"], case["H"], case["Hkv"], case["D"], case["q"], case["law"])
        if kind == "attn":  # the position types are the model's, not the batch's
            st["plan"] = starq.star_type_plan(case["q"], st["types"])
        else:
            nbytes = starq.star_attn_decode_workspace_bytes(st["shape"])
            st["ws"] = torch.empty(max(nbytes, 16), dtype=torch.uint8, device=DEV)
    else:
        st["up"], st["down"] = _algebras(case)
        if kind == "merged":
            st["W_gu"] = starq.pack_gate_up(st.pop("W_gate"), st.pop("W_up"))
            st["up_gu"] = st["up"].merged_gate_up()
    return st


# ---- one pass ------------------------------------------------------------------


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "decode":
        if case["gated"]:
            return starq.star_decode_gated(st["up"], st["down"], st["types"], st["X"], st["W_gate"], None, st["W_up"],
                                           None, st["W_down"], None, True, ws=st["ws"], check=False)
        return starq.star_decode(st["up"], st["down"], st["types"], st["X"], st["W_up"], st["b_up"], st["W_down"],
                                 st["b_down"], "gelu", True, ws=st["ws"], check=False)
    if kind == "attn":
        return starq.star_attn_fwd(st["shape"], st["plan"], st["Q"], st["K"], st["V"], want_lse=case["lse"])
    if kind == "attn_decode":
        return starq.star_attn_decode(st["shape"], st["types"], st["lens"], st["Q"], st["K"], st["V"], ws=st["ws"])
    if kind == "merged":
        plan = starq.star_type_plan(case["q"], st["types"])
        H = starq.star_swiglu_up_fwd_planned(st["up_gu"], plan, st["X"], st["W_gu"])
        return H, starq.star_proj_fwd_planned(st["down"], plan, H, st["W_down"])
    if kind == "swiglu":
        plan = starq.star_type_plan(case["q"], st["types"])
        Zg, Zu, H, Y = starq.star_swiglu_ffn_fwd(st["up"], st["down"], st["types"], st["X"], st["W_gate"], None,
                                                 st["W_up"], None, st["W_down"], None, plan=plan)
        g = starq.star_swiglu_ffn_bwd(st["up"], st["down"], st["types"], st["X"], Zg, Zu, H, st["W_gate"], st["W_up"],
                                      st["W_down"], st["dY"], plan=plan)
        return dict(Y=Y, H=H, **g)
    Z, H, Y = starq.star_ffn_fwd(st["up"], st["down"], st["types"], st["X"], st["W_up"], st.get("b_up"), st["W_down"],
                                 st.get("b_down"), case["act"], save_z=case["train"])
    if not case["train"]:
        return H, Y
    g = starq.star_ffn_bwd(st["up"], st["down"], st["types"], st["X"], Z, H, st["W_up"], st["W_down"], st["dY"],
                           case["act"])
    return dict(Y=Y, Z=Z, H=H, **g)


# ---- what a pass cannot do without -----------------------------------------------


def _macs_per_row(case, s, r):
    """Multiply-accumulates of one row, the mean over the types."""
    q, law = case["q"], case["law"]
    return sum(s[k] * r[j] for i in range(q) for j in range(q) for k in _support(law, q, i, j)) / q


def _bank_bytes(case, s, r, elem):
    """Bytes of the weight blocks that some row reaches, the types uniform."""
    q, law, M = case["q"], case["law"], case["M"]
    total = 0.0
    for k in range(q):
        for j in range(q):
            share = sum(k in _support(law, q, i, j) for i in range(q)) / q
            total += s[k] * r[j] * elem * (1.0 - (1.0 - share) ** M)
    return total


def work(case):
    kind = case["kind"]
    if kind in ("attn", "attn_decode"):
        B, S, H, Hkv, D, q = (case[k] for k in ("B", "S", "H", "Hkv", "D", "q"))
        keep = sum(len(_features(case["law"], q, i, j)) for i in range(q) for j in range(q)) / (q * q) * (D // q)
        if kind == "attn":
            pairs = B * H * S * (S + 1) / 2
            io = 2 * B * S * D * (2 * H + 2 * Hkv) + 4 * S + (4 * B * H * S if case["lse"] else 0)
            return dict(bytes=int(io), flops=int(pairs * 2 * (keep + D)))
        keys = B * (S + 1) / 2
        return dict(bytes=int(keys * Hkv * (keep + D) * 2 + 4 * B * H * D + 4 * S),
                    flops=int(keys * H * 2 * (keep + D)))
    q, M, D, Fw = case["q"], case["M"], case["D"], case["F"]
    d, f = _widths(D, q, case.get("ragged", False)), _widths(Fw, q, case.get("ragged", False))
    up, down = _macs_per_row(case, d, f), _macs_per_row(case, f, d)
    if kind == "decode":
        maps = 2 if case["gated"] else 1
        L = case["layers"]
        wb = maps * _bank_bytes(case, d, f, 2) + _bank_bytes(case, f, d, 2)
        return dict(bytes=int(L * (wb + (0 if case["gated"] else 4 * (D + Fw))) + 4 * M * D + 4 * M),
                    flops=int(2 * M * L * (maps * up + down)))
    e = 4 if case.get("dtype") == "f32" else 2
    bank = _bank_bytes(case, d, f, e), _bank_bytes(case, f, d, e)
    if kind == "merged":
        return dict(bytes=int(2 * bank[0] + bank[1] + e * M * (2 * D + Fw) + 4 * M), flops=int(2 * M * (2 * up + down)))
    if kind == "swiglu":
        # forward: X, the three banks -> Zg, Zu, H, Y; backward: dY -> dX, dZg, dZu and three fp32 gradients
        fwd = e * M * (2 * D + 3 * Fw) + 2 * bank[0] + bank[1]
        return dict(bytes=int(fwd + e * M * (D + 2 * Fw) + 4 * M * D + 12 * D * Fw + 4 * (2 * Fw + D) + 4 * M),
                    flops=int(6 * M * (2 * up + down)))
    bias = 4 * (D + Fw) if case["bias"] else 0
    fwd = e * M * (2 * D + Fw) + bank[0] + bank[1] + bias + 4 * M
    if not case["train"]:
        return dict(bytes=int(fwd), flops=int(2 * M * (up + down)))
    return dict(bytes=int(fwd + e * M * (2 * D + 2 * Fw) + 8 * D * Fw + 4 * (D + Fw)), flops=int(6 * M * (up + down)))


# ---- how far another correct implementation may be --------------------------------


def tolerance(case):
    """About four times the distance to the 64-bit result."""
    if case.get("dtype") == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.1}


# ---- the same in 64 bits -----------------------------------------------------------


def _proj64(case, s, r, types, X, W):
    q, law = case["q"], case["law"]
    S = [sum(s[:g]) for g in range(q + 1)]
    R = [sum(r[:g]) for g in range(q + 1)]
    rows = [torch.nonzero(types == i).flatten() for i in range(q)]
    parts = []
    for i in range(q):
        if rows[i].numel() == 0:
            continue
        Xi = X[rows[i]]
        cols = []
        for j in range(q):
            acc = X.new_zeros((Xi.shape[0], r[j]))
            for k in _support(law, q, i, j):
                acc = acc + Xi[:, S[k]:S[k + 1]].contiguous() @ W[S[k]:S[k + 1], R[j]:R[j + 1]].contiguous()
            cols.append(acc)
        parts.append(torch.cat(cols, 1))
    order = torch.cat([v for v in rows if v.numel()])
    return torch.cat(parts)[torch.argsort(order)]


def _act64(act, z):
    if act == "none":
        return z
    return F.gelu(z, approximate="tanh" if act == "gelu_tanh" else "none")


def _attn64(case, t):
    """(O, lse) of causal attention, one sequence and one key/value head at a time."""
    B, S, H, Hkv, D, q = (case[k] for k in ("B", "S", "H", "Hkv", "D", "q"))
    m, rep = D // q, H // Hkv
    types = t["types"].long()
    keep = torch.zeros((q, q, q), dtype=F64, device=DEV)
    for i in range(q):
        for j in range(q):
            for a in _features(case["law"], q, i, j):
                keep[a, i, j] = 1.0
    norm = 1.0 / torch.sqrt(keep.sum(0) * m)
    decode = case["kind"] == "attn_decode"
    O = torch.empty((B, H, D) if decode else (B, S, H, D), dtype=F64, device=DEV)
    lse = torch.empty((B, H, S), dtype=F64, device=DEV)
    causal = torch.ones((S, S), dtype=torch.bool, device=DEV).tril_() if not decode else None
    for b in range(B):
        n = int(t["lens"][b].item()) if decode else S
        tk = types[:n]
        tq = types[n - 1:n] if decode else tk
        scale = norm[tq][:, tk]
        masks = [keep[a][tq][:, tk] for a in range(q)]
        for g in range(Hkv):
            K, V = t["K"][b, :n, g].to(F64), t["V"][b, :n, g].to(F64)
            for h in range(g * rep, (g + 1) * rep):
                Q = (t["Q"][b, h][None] if decode else t["Q"][b, :, h]).to(F64)
                s = torch.zeros((Q.shape[0], n), dtype=F64, device=DEV)
                for a in range(q):
                    kt = K[:, a * m:(a + 1) * m].t().contiguous()
                    s += (Q[:, a * m:(a + 1) * m].contiguous() @ kt) * masks[a]
                s *= scale
                if not decode:
                    s.masked_fill_(~causal, float("-inf"))
                p = torch.softmax(s, -1) @ V
                if decode:
                    O[b, h] = p[0]
                else:
                    O[b, :, h] = p
                    lse[b, h] = torch.logsumexp(s, -1)
    return O, lse


def exact(case, seed):
    t = _inputs(case, seed)
    kind, types = case["kind"], t["types"]
    if kind in ("attn", "attn_decode"):
        O, lse = _attn64(case, t)
        return (O, lse) if case.get("lse") else O
    q, ragged = case["q"], case.get("ragged", False)
    d, f = _widths(case["D"], q, ragged), _widths(case["F"], q, ragged)
    if kind == "decode":
        h = t["X"].to(F64)
        for n in range(case["layers"]):
            up = _proj64(case, d, f, types, h, t["W_up"][n].to(F64))
            if case["gated"]:
                up = F.silu(_proj64(case, d, f, types, h, t["W_gate"][n].to(F64))) * up
                h = h + _proj64(case, f, d, types, up, t["W_down"][n].to(F64))
            else:
                up = F.gelu(up + t["b_up"][n].to(F64))
                h = h + _proj64(case, f, d, types, up, t["W_down"][n].to(F64)) + t["b_down"][n].to(F64)
        return h
    leaf = {k: t[k].to(F64).requires_grad_() for k in ("X", "W_gate", "W_up", "W_down", "b_up", "b_down") if k in t}
    if kind in ("swiglu", "merged"):
        Zg = _proj64(case, d, f, types, leaf["X"], leaf["W_gate"])
        Zu = _proj64(case, d, f, types, leaf["X"], leaf["W_up"])
        H = F.silu(Zg) * Zu
        Y = _proj64(case, f, d, types, H, leaf["W_down"])
        if kind == "merged":
            return H.detach(), Y.detach()
        names = dict(dX=leaf["X"], dZ_gate=Zg, dZ_up=Zu, dW_gate=leaf["W_gate"], dW_up=leaf["W_up"],
                     dW_down=leaf["W_down"])
        grads = dict(zip(names, torch.autograd.grad(Y, list(names.values()), t["dY"].to(F64))))
        return dict(Y=Y.detach(), H=H.detach(), dX=grads["dX"], dZ_gate=grads["dZ_gate"], dZ_up=grads["dZ_up"],
                    dW_gate=grads["dW_gate"], db_gate=grads["dZ_gate"].sum(0), dW_up=grads["dW_up"],
                    db_up=grads["dZ_up"].sum(0), dW_down=grads["dW_down"], db_down=t["dY"].to(F64).sum(0))
    Z = _proj64(case, d, f, types, leaf["X"], leaf["W_up"])
    if "b_up" in leaf:
        Z = Z + leaf["b_up"]
    H = _act64(case["act"], Z)
    Y = _proj64(case, f, d, types, H, leaf["W_down"])
    if "b_down" in leaf:
        Y = Y + leaf["b_down"]
    if not case["train"]:
        return H.detach(), Y.detach()
    wrt = [leaf["X"], Z, leaf["W_up"], leaf["W_down"]]
    dX, dZ, dWu, dWd = torch.autograd.grad(Y, wrt, t["dY"].to(F64))
    return dict(Y=Y.detach(), Z=Z.detach(), H=H.detach(), dX=dX, dZ=dZ, dW_up=dWu, db_up=dZ.sum(0), dW_down=dWd,
                db_down=t["dY"].to(F64).sum(0))
