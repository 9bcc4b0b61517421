"""Performance cases of the two training steps, through their public bindings.

Every case is one pass that a program using this package makes: an optimizer
step of a GPT-2 model, a micro-batch of an accumulated step, one block's
forward or backward, the logits of a prompt, a held-out loss, the scatter of
the embedding gradient, an adapter step of a Qwen3-shaped model. Sizes are
those of the package's own workloads (paper_2609_28568_amd/synth.py), its
tests' small and ragged models, and generic ones between them.

All inputs are drawn here with torch from the case's seed, so that exact() can
draw the same ones and compute the pass in 64 bits without the package.
"""
import math

import numpy as np
import torch

DEV = "cuda"
RP = 64   # padded adapter rank of the Qwen3-shaped layout

OPT = dict(lr_max=6e-4, lr_min=6e-5, warmup_steps=700, total_steps=18865, beta1=0.9, beta2=0.95, adam_eps=1e-8,
           weight_decay=0.1, grad_clip=1.0, ln_eps=1e-5)
QOPT = dict(lr=2e-4, beta1=0.9, beta2=0.95, adam_eps=1e-8, weight_decay=0.1, grad_clip=1.0, rms_eps=1e-6,
            rope_theta=1e6)
LORA_ALPHA = 32.0
TARGETS = {"qkv": ("q", "k", "v"), "o": ("o",), "gate_up": ("gate", "up"), "down": ("down",)}


def _gpt2(name, what, L, H, C, V, B, T, accum=1):
    c = dict(model="gpt2", what=what, L=L, H=H, C=C, F=4 * C, V=V, Vp=-(-V // 64) * 64, B=B, T=T, accum=accum)
    return dict(c, name=name) if name else c


def _qwen(name, what, L, H, Hkv, C, F, V, B, T, rank, groups):
    c = dict(model="qwen3", what=what, L=L, H=H, Hkv=Hkv, C=C, F=F, V=V, B=B, T=T, rank=rank, groups=groups)
    return dict(c, name=name) if name else c


GPT2_V, QWEN_V = 50257, 151936


def listed():
    return [
        # the smallest training step: two narrow layers on 64 tokens, as a test
        # or a toy run makes it; launches and latency count
        _gpt2("gpt2_tiny_step", "step", 2, 4, 64, 512, 2, 32),
        # the paper's model on one GPU's micro-batch: forward, backward, clip
        # and AdamW
        _gpt2("gpt2_124m_step", "step", 12, 12, 768, GPT2_V, 16, 1024),
        # an optimizer step accumulated over two small micro-batches of short
        # sequences
        _gpt2("gpt2_124m_accum2_step", "step", 12, 12, 768, GPT2_V, 4, 256, 2),
        # next-token logits of one prompt of odd length
        _gpt2("gpt2_124m_prompt_logits", "logits", 12, 12, 768, GPT2_V, 1, 203),
        # the held-out loss between training steps
        _gpt2("gpt2_124m_evaluate", "evaluate", 12, 12, 768, GPT2_V, 16, 1024),
        # one block in isolation, forward
        _gpt2("gpt2_block_forward", "block_fwd", 1, 12, 768, GPT2_V, 16, 1024),
        # ... and backward (after its forward, which prepare has made)
        _gpt2("gpt2_block_backward", "block_bwd", 1, 12, 768, GPT2_V, 16, 1024),
        # forward and backward of one block on a few sequences of odd length
        _gpt2("gpt2_block_ragged", "block", 1, 12, 768, GPT2_V, 3, 333),
        # scatter of the embedding gradient of a full micro-batch
        _gpt2("gpt2_embedding_backward", "embed_bwd", 1, 12, 768, GPT2_V, 16, 1024),
        # adapter fine-tuning of the 0.6B-parameter shape: four sequences of
        # 2048 tokens, adapters on the attention projections
        _qwen("qwen3_06b_step", "step", 28, 16, 8, 1024, 3072, QWEN_V, 4, 2048, 16, "qkv,o"),
        # held-out loss of the same model on two short question/answer pairs
        _qwen("qwen3_06b_loss", "loss", 28, 16, 8, 1024, 3072, QWEN_V, 2, 352, 16, "qkv,o"),
        # a small model with every projection adapted at an odd rank, ragged
        # sequences
        _qwen("qwen3_small_step", "step", 4, 4, 2, 256, 512, 1024, 2, 96, 20, "qkv,o,gate_up,down"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.65:
        H, C = rng.choice([(4, 64), (4, 128), (6, 384), (4, 512), (12, 768), (12, 768)])
        V = rng.choice([500, 512, 5003, GPT2_V]) if C < 768 else GPT2_V
        what = rng.choice(["step", "step", "logits", "evaluate", "block_fwd", "block_bwd", "block", "embed_bwd"])
        L = 1 if what.startswith("block") or what == "embed_bwd" else rng.randint(1, 12)
        T = _log_int(rng, 16, 1024)
        B = max(1, min(_log_int(rng, 1, 16), 16384 // T))
        return _gpt2(None, what, L, H, C, V, B, T, rng.choice([1, 1, 2]) if what == "step" else 1)
    H, Hkv, C, F, V = rng.choice([(4, 2, 256, 512, 1024), (8, 2, 512, 1536, 8192), (16, 8, 1024, 3072, QWEN_V)])
    L = rng.randint(1, 12)
    T = 16 * _log_int(rng, 2, 128)
    B = rng.choice([1, 2, 4])
    while (B * T) % 64 or B * T > 8192:
        if B * T > 8192:
            B, T = 1, T // 64 * 64
        else:
            B *= 2
    rank = rng.choice([1, 8, 16, 16, 20, 32])
    # the rank-1 gradient of the q adapter is a difference of nearly equal
    # terms, so the smallest rank adapts the output projections only
    groups = "o,down" if rank == 1 else rng.choice(["qkv,o", "qkv,o", "qkv,o,gate_up,down", "gate_up,down"])
    return _qwen(None, rng.choice(["step", "step", "loss"]), L, H, Hkv, C, F, V, B, T, rank, groups)


# ---------------------------------------------------------------- inputs

def _gen(seed, k):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + k)
    return g


def _zipf_ids(seed, k, n, vocab):
    """n token ids, Zipf(1.1) over the vocabulary as natural text has them."""
    w = np.arange(1, vocab + 1, dtype=np.float64) ** -1.1
    cdf = torch.from_numpy(np.cumsum(w) / w.sum()).to(DEV)
    u = torch.rand(n, generator=_gen(seed, k), device=DEV, dtype=torch.float64)
    return torch.searchsorted(cdf, u).clamp_(max=vocab - 1).to(torch.int32)


def _tokens(c, seed, micro=0):
    ids = _zipf_ids(seed, 100 + micro, c["B"] * (c["T"] + 1), c["V"]).view(c["B"], c["T"] + 1)
    return ids[:, :-1].contiguous(), ids[:, 1:].contiguous()


GPT2_KINDS = ("wte", "wpe", "ln1w", "ln1b", "qkvw", "qkvb", "attprojw", "attprojb", "ln2w", "ln2b", "fcw", "fcb",
              "fcprojw", "fcprojb", "lnfw", "lnfb")
GPT2_DECAY = ("wte", "wpe", "qkvw", "attprojw", "fcw", "fcprojw")


def _gpt2_shapes(c):
    L, C, F = c["L"], c["C"], c["F"]
    return dict(wte=(c["Vp"], C), wpe=(c["T"], C), ln1w=(L, C), ln1b=(L, C), qkvw=(L, 3 * C, C), qkvb=(L, 3 * C),
                attprojw=(L, C, C), attprojb=(L, C), ln2w=(L, C), ln2b=(L, C), fcw=(L, F, C), fcb=(L, F),
                fcprojw=(L, C, F), fcprojb=(L, C), lnfw=(C,), lnfb=(C,))


def _gpt2_weights(c, seed):
    """Flat fp32 weights (kinds in GPT2_KINDS' order) of a model in training:
    matrices N(0, 0.02), the residual projections scaled down with depth,
    gains around 1, shifts and biases around 0."""
    g, parts = _gen(seed, 1), []
    for k in GPT2_KINDS:
        shape = _gpt2_shapes(c)[k]
        t = torch.randn(shape, generator=g, device=DEV)
        if k in ("attprojw", "fcprojw"):
            t *= 0.02 / math.sqrt(2.0 * c["L"])
        elif k in GPT2_DECAY:
            t *= 0.02
        else:
            t *= 0.05
            if k in ("ln1w", "ln2w", "lnfw"):
                t += 1.0
        if k == "wte":
            t[c["V"]:] = 0.0   # padding rows of the token table
        parts.append(t.reshape(-1))
    return torch.cat(parts)


def _gpt2_blocks(c, flat):
    """The flat vector's parameters by kind (views)."""
    out, o = {}, 0
    for k, s in _gpt2_shapes(c).items():
        n = math.prod(s)
        out[k] = flat[o:o + n].view(s)
        o += n
    return out


def _block_range(c):
    """Elements of the flat vector that hold the blocks' parameters."""
    n = {k: math.prod(s) for k, s in _gpt2_shapes(c).items()}
    lo = n["wte"] + n["wpe"]
    return lo, sum(n.values()) - n["lnfw"] - n["lnfb"]


def _bf16_normal(c, seed, k, std):
    t = torch.randn((c["B"] * c["T"], c["C"]), generator=_gen(seed, k), device=DEV)
    return (t * std).to(torch.bfloat16)


def _qwen_geom(c):
    C, F, qd, kvd = c["C"], c["F"], c["H"] * 128, c["Hkv"] * 128
    return {"qkv": (C, (qd, kvd, kvd)), "o": (qd, (C,)), "gate_up": (C, (F, F)), "down": (F, (C,))}


def _qwen_base(c, seed):
    """Frozen bf16 tensors by name, in the layout of the package."""
    L, C, F, V = c["L"], c["C"], c["F"], c["V"]
    qd, kvd = c["H"] * 128, c["Hkv"] * 128
    shapes = dict(embed=(V, C), in_norm=(L, C), qkv=(L, qd + 2 * kvd, C), q_norm=(L, 128), k_norm=(L, 128),
                  o=(L, C, qd), post_norm=(L, C), gate_up=(L, 2 * F, C), down=(L, C, F), final_norm=(C,))
    g, out = _gen(seed, 2), {}
    for k, s in shapes.items():
        t = torch.randn(s, generator=g, device=DEV)
        out[k] = (1.0 + 0.05 * t if k.endswith("norm") else 0.02 * t).to(torch.bfloat16)
    return out


def _qwen_lora(c, seed):
    """fp32 adapters by name, rank padded with zeros: A [L, n*64, in], B [L, out, 64]."""
    g, out, r, L = _gen(seed, 3), {}, c["rank"], c["L"]
    for name, (i, outs) in _qwen_geom(c).items():
        if name not in c["groups"].split(","):
            continue
        A = torch.zeros((L, len(outs) * RP, i), device=DEV)
        B = torch.zeros((L, sum(outs), RP), device=DEV)
        for j in range(len(outs)):
            A[:, j * RP:j * RP + r] = 0.02 * torch.randn((L, r, i), generator=g, device=DEV)
        B[:, :, :r] = 0.02 * torch.randn((L, sum(outs), r), generator=g, device=DEV)
        out[name + "_A"], out[name + "_B"] = A, B
    return out


# ---------------------------------------------------------------- state and pass

def prepare(case, seed):
    return _prepare_gpt2(case, seed) if case["model"] == "gpt2" else _prepare_qwen(case, seed)


def _prepare_gpt2(c, seed):
    from paper_2609_28568_amd import binding
    cfg = binding.make_config(dict(n_layer=c["L"], n_head=c["H"], d_model=c["C"], d_ff=c["F"], vocab=c["V"],
                                   vocab_padded=c["Vp"], max_seq_len=c["T"], B=c["B"], T=c["T"],
                                   grad_accum=c["accum"]), OPT)
    m = binding.GPT2(cfg, device=DEV)
    m.flat("params").copy_(_gpt2_weights(c, seed))
    binding._check(m.L.gpt2_sync_weights(m.handle), m.handle)
    s = dict(case=c, m=m, step=0)
    what = c["what"]
    if what.startswith("block"):
        s["x"], s["dy"] = _bf16_normal(c, seed, 11, 1.0), _bf16_normal(c, seed, 12, 1e-3)
        s["out"], s["dx"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
        lo, hi = _block_range(c)
        s["grads"] = m.flat("grads")[lo:hi]
        if what == "block_bwd":
            m.block_forward(0, s["x"], s["out"])
    elif what == "embed_bwd":
        s["ids"], s["dy"] = _tokens(c, seed)[0], _bf16_normal(c, seed, 12, 1e-3)
        n = (c["Vp"] + c["T"]) * c["C"]
        s["grads"] = m.flat("grads")[:n]
    else:
        s["batches"] = [_tokens(c, seed, k) for k in range(c["accum"])]
        s["losses"] = torch.zeros(c["B"] * c["T"], device=DEV)
        s["norm"] = torch.zeros(1, device=DEV)
    return s


def _prepare_qwen(c, seed):
    from paper_2609_28568_amd import qwen3_binding as qb
    targets = tuple(t for g in c["groups"].split(",") for t in TARGETS[g])
    cfg = qb.make_config(dict(n_layer=c["L"], d_model=c["C"], n_head=c["H"], n_kv_head=c["Hkv"], head_dim=128,
                              d_ff=c["F"], vocab=c["V"], max_seq_len=c["T"], B=c["B"], T=c["T"],
                              lora_rank=c["rank"], lora_alpha=LORA_ALPHA, lora_targets=targets, loss_from=0.5), QOPT)
    m = qb.Qwen3(cfg, device=DEV)
    for name, t in _qwen_base(c, seed).items():
        m._view("base_bf16", torch.bfloat16, m.base_table, name).copy_(t)
    for name, t in _qwen_lora(c, seed).items():
        m._view("lora_f32", torch.float32, m.lora_table, name).copy_(t)
    qb._check(qb.lib().qwen3_sync_weights(m.h), m.h)
    return dict(case=c, m=m, step=0, batches=[_tokens(c, seed)], losses=torch.zeros(c["B"] * c["T"], device=DEV),
                norm=torch.zeros(1, device=DEV))


def run(s):
    c, m = s["case"], s["m"]
    what = c["what"]
    if what == "block_fwd":
        m.block_forward(0, s["x"], s["out"])
        return {"out": s["out"]}
    if what == "block_bwd":
        m.block_backward(0, s["dy"], s["dx"])
        return {"dx": s["dx"], "grads": s["grads"]}
    if what == "block":
        m.block_forward(0, s["x"], s["out"])
        m.block_backward(0, s["dy"], s["dx"])
        return {"out": s["out"], "dx": s["dx"], "grads": s["grads"]}
    if what == "embed_bwd":
        m.embedding_backward(s["ids"], s["dy"])
        return {"grads": s["grads"]}
    ids, tgt = s["batches"][0]
    if what == "logits":
        m.forward(ids)
        return {"logits": m.activation("logits")}
    if what == "evaluate":
        return {"loss": m.evaluate(ids, tgt, s["losses"]), "losses": s["losses"]}
    if what == "loss":
        m.forward(ids, tgt)
        return {"loss": m.loss(s["losses"]), "losses": s["losses"]}
    # an optimizer step
    if c["model"] == "gpt2":
        for k, (ids, tgt) in enumerate(s["batches"]):
            m.forward(ids, tgt)
            m.backward(accumulate=k > 0)
        m.adamw_step(s["step"], s["norm"])
        out = {"losses": m.activation("losses"), "grads": m.flat("grads"), "params": m.flat("params")}
    else:
        m.forward(ids, tgt)
        m.backward()
        m.adamw_step(s["step"], s["norm"])
        out = {"grads": m.flat("lora_grads"), "params": m.flat("lora_f32")}
    s["step"] += 1
    return dict(out, norm=s["norm"])


# ---------------------------------------------------------------- work

def work(case):
    """FLOPs of the matrix products and causal attention (a backward pass
    twice a forward one, the frozen base of the adapter step input gradients
    only) and the bytes of weights, gradients and moments, inputs and outputs
    that a pass reads and writes."""
    c = case
    B, T, L, H, C, F, V = (c[k] for k in ("B", "T", "L", "H", "C", "F", "V"))
    BT = B * T
    what = c["what"]
    if c["model"] == "gpt2":
        block_w = 4 * C * C + 2 * C * F
        block = 2.0 * BT * block_w + 4.0 * B * C * (T * (T + 1) / 2)
        head = 2.0 * BT * C * V
        act = 2.0 * BT * C
        block_p = block_w + 9 * C + F
        P = c["Vp"] * C + T * C + L * block_p + 2 * C
        if what == "block_fwd":
            return {"flops": block, "bytes": 2.0 * block_p + 2 * act}
        if what == "block_bwd":
            return {"flops": 2 * block, "bytes": 6.0 * block_p + 2 * act}
        if what == "block":
            return {"flops": 3 * block, "bytes": 6.0 * block_p + 4 * act}
        if what == "embed_bwd":
            return {"flops": float(BT * C), "bytes": act + 4.0 * BT + 4.0 * (c["Vp"] + T) * C}
        if what == "logits":
            return {"flops": L * block + head, "bytes": 2.0 * P + 2.0 * BT * c["Vp"]}
        if what == "evaluate":
            return {"flops": L * block + head, "bytes": 2.0 * P + 8.0 * BT}
        # gradients written (and read and written again per further
        # micro-batch), then read with p, m, v; p, m, v and the bf16 copy written
        n = c["accum"]
        return {"flops": 3 * n * (L * block + head), "bytes": (2.0 * n + 4 + 8 * (n - 1) + 30) * P + 12.0 * n * BT}
    qd, kvd = H * 128, c["Hkv"] * 128
    base_w = C * (qd + 2 * kvd) + qd * C + 3 * C * F
    rows = B * (T - T // 2)
    attn = 4.0 * B * qd * (T * (T + 1) / 2)
    lora = sum(len(o) * i * c["rank"] + sum(o) * c["rank"] for g, (i, o) in _qwen_geom(c).items()
               if g in c["groups"].split(","))
    fwd = L * (2.0 * BT * (base_w + lora) + attn) + 2.0 * rows * C * V
    nbytes = 2.0 * (V * C + L * base_w)
    if what == "loss":
        return {"flops": fwd, "bytes": nbytes + 2.0 * L * lora + 12.0 * BT}
    bwd = L * (2.0 * BT * (base_w + 2 * lora) + 2 * attn) + 2.0 * rows * C * V
    return {"flops": fwd + bwd, "bytes": nbytes + 36.0 * L * lora + 12.0 * BT}


# ---------------------------------------------------------------- tolerance

def tolerance(case):
    """About four times the error against exact() that the bf16 path shows
    (gradients of a whole model 3.5e-3 to 8.5e-3, logits 7.7e-3, one block
    3.5e-3, losses up to 7.6e-4)."""
    what = case["what"]
    if what == "embed_bwd":
        return {"rel": 1e-6, "max": 1e-4}   # fp32 sums in any order
    if what in ("evaluate", "loss"):
        return {"rel": 3e-3}
    if what == "logits":
        return {"rel": 3e-2}
    if what.startswith("block"):
        return {"rel": 1.5e-2}
    return {"rel": 1.5e-2 if case["model"] == "gpt2" else 3e-2}


# ---------------------------------------------------------------- 64-bit results

def exact(case, seed):
    with torch.enable_grad():
        return _exact_gpt2(case, seed) if case["model"] == "gpt2" else _exact_qwen(case, seed)


def _ln(x, w, b):
    return torch.nn.functional.layer_norm(x, x.shape[-1:], w, b, OPT["ln_eps"])


def _causal(q, k, v):
    """[n, heads, T, d] attention in the inputs' precision."""
    T = q.shape[-2]
    s = torch.matmul(q, k.transpose(-1, -2).contiguous()) / math.sqrt(q.shape[-1])
    s = s.masked_fill(torch.ones(T, T, dtype=torch.bool, device=s.device).triu(1), float("-inf"))
    return torch.matmul(torch.softmax(s, -1), v)


def _gpt2_block(c, p, l, x):
    """x [n, T, C] through block l."""
    n, T, C = x.shape
    h = _ln(x, p["ln1w"][l], p["ln1b"][l])
    qkv = h @ p["qkvw"][l].t() + p["qkvb"][l]
    q, k, v = (t.reshape(n, T, c["H"], C // c["H"]).transpose(1, 2) for t in qkv.split(C, -1))
    a = _causal(q, k, v).transpose(1, 2).reshape(n, T, C)
    x = x + a @ p["attprojw"][l].t() + p["attprojb"][l]
    h = _ln(x, p["ln2w"][l], p["ln2b"][l])
    f = torch.nn.functional.gelu(h @ p["fcw"][l].t() + p["fcb"][l], approximate="tanh")
    return x + f @ p["fcprojw"][l].t() + p["fcprojb"][l]


def _adamw(flat, g, decay, o, lr):
    """First step of AdamW from zero moments, after the global-norm clip."""
    norm = g.square().sum().sqrt()
    g = g * torch.clamp(o["grad_clip"] / norm, max=1.0)
    upd = g / (g.abs() + o["adam_eps"]) + o["weight_decay"] * decay * flat
    return flat - lr * upd, norm.view(1)


def _exact_gpt2(c, seed):
    what, B, T, C, V = c["what"], c["B"], c["T"], c["C"], c["V"]
    flat32 = _gpt2_weights(c, seed)
    if what == "embed_bwd":
        ids, dy = _tokens(c, seed)[0], _bf16_normal(c, seed, 12, 1e-3).double()
        wte = torch.zeros((c["Vp"], C), dtype=torch.float64, device=DEV).index_add_(0, ids.reshape(-1).long(), dy)
        return {"grads": torch.cat([wte.reshape(-1), dy.view(B, T, C).sum(0).reshape(-1)])}
    flat = flat32.double().requires_grad_(True)
    p = _gpt2_blocks(c, flat)
    group = max(1, min(B, 4096 // T))   # sequences at a time
    if what.startswith("block"):
        x = _bf16_normal(c, seed, 11, 1.0).double().view(B, T, C)
        dy = _bf16_normal(c, seed, 12, 1e-3).double().view(B, T, C)
        outs, dxs = [], []
        for i in range(0, B, group):
            xi = x[i:i + group].clone().requires_grad_(True)
            y = _gpt2_block(c, p, 0, xi)
            outs.append(y.detach())
            if what != "block_fwd":
                y.backward(dy[i:i + group])
                dxs.append(xi.grad)
        r = {"out": torch.cat(outs).view(B * T, C)} if what != "block_bwd" else {}
        if what != "block_fwd":
            lo, hi = _block_range(c)
            r.update(dx=torch.cat(dxs).view(B * T, C), grads=flat.grad[lo:hi])
        return r
    train = what == "step"
    for k in range(c["accum"]):
        ids, tgt = _tokens(c, seed, k)
        losses, logits = [], []
        for i in range(0, B, group):
            with torch.set_grad_enabled(train):
                x = p["wte"][ids[i:i + group].long()] + p["wpe"][:T]
                for l in range(c["L"]):
                    x = _gpt2_block(c, p, l, x)
                z = _ln(x, p["lnfw"], p["lnfb"]) @ p["wte"].t()
                if what == "logits":
                    logits.append(z)
                    continue
                e = torch.nn.functional.cross_entropy(z[..., :V].reshape(-1, V), tgt[i:i + group].reshape(-1).long(),
                                                      reduction="none")
                if train:
                    (e.sum() / (B * T * c["accum"])).backward()
                losses.append(e.detach())
    if what == "logits":
        return {"logits": torch.cat(logits).reshape(-1)}
    losses = torch.cat(losses)
    if not train:
        return {"loss": losses.mean(), "losses": losses}
    decay = torch.cat([torch.full((math.prod(s),), float(k in GPT2_DECAY), dtype=torch.float64, device=DEV)
                       for k, s in _gpt2_shapes(c).items()])
    new, norm = _adamw(flat.detach(), flat.grad, decay, OPT, OPT["lr_max"] / OPT["warmup_steps"])
    return {"losses": losses, "grads": flat.grad, "params": new, "norm": norm}


def _rms(x, w):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + QOPT["rms_eps"]) * w


def _exact_qwen(c, seed):
    base, B, T, L, H, Hkv = _qwen_base(c, seed), c["B"], c["T"], c["L"], c["H"], c["Hkv"]
    lora = {k: v.double().requires_grad_(True) for k, v in _qwen_lora(c, seed).items()}
    ids, tgt = _tokens(c, seed)
    train, m0 = c["what"] == "step", T // 2
    scale = LORA_ALPHA / math.sqrt(c["rank"])
    inv = QOPT["rope_theta"] ** (-2.0 * torch.arange(64, dtype=torch.float64, device=DEV) / 128)
    ang = torch.arange(T, dtype=torch.float64, device=DEV)[:, None] * inv
    cos, sin = ang.cos(), ang.sin()
    geom = _qwen_geom(c)
    head = base["embed"].double()

    def proj(g, l, x):
        y = x @ base[g][l].double().t()
        if g + "_A" not in lora:
            return y
        u = scale * (x @ lora[g + "_A"][l].t())
        row, parts = 0, []
        for j, o in enumerate(geom[g][1]):
            parts.append(u[..., j * RP:(j + 1) * RP] @ lora[g + "_B"][l, row:row + o].t())
            row += o
        return y + torch.cat(parts, -1)

    def rope(x):
        a, b = x[..., :64], x[..., 64:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    losses = torch.zeros((B, T), dtype=torch.float64, device=DEV)
    for i in range(B):
        with torch.set_grad_enabled(train):
            x = head[ids[i].long()]
            for l in range(L):
                w = {k: base[k][l].double() for k in ("in_norm", "q_norm", "k_norm", "post_norm")}
                q, k, v = proj("qkv", l, _rms(x, w["in_norm"])).split([H * 128, Hkv * 128, Hkv * 128], -1)
                q = rope(_rms(q.view(T, H, 128), w["q_norm"]).transpose(0, 1))
                k = rope(_rms(k.view(T, Hkv, 128), w["k_norm"]).transpose(0, 1))
                k = k.repeat_interleave(H // Hkv, 0)
                v = v.view(T, Hkv, 128).transpose(0, 1).repeat_interleave(H // Hkv, 0)
                x = x + proj("o", l, _causal(q, k, v).transpose(0, 1).reshape(T, H * 128))
                g, u = proj("gate_up", l, _rms(x, w["post_norm"])).split(c["F"], -1)
                x = x + proj("down", l, torch.nn.functional.silu(g) * u)
            z = _rms(x[m0:], base["final_norm"].double()) @ head.t()
            e = torch.nn.functional.cross_entropy(z, tgt[i, m0:].long(), reduction="none")
            if train:
                (e.sum() / (B * (T - m0))).backward()
        losses[i, m0:] = e.detach()
    if not train:
        return {"loss": losses.sum() / (B * (T - m0)), "losses": losses.reshape(-1)}
    names = [n for g in geom for n in (g + "_A", g + "_B") if n in lora]
    flat = torch.cat([lora[n].detach().reshape(-1) for n in names])
    grads = torch.cat([lora[n].grad.reshape(-1) for n in names])
    new, norm = _adamw(flat, grads, 1.0, QOPT, QOPT["lr"])
    return {"grads": grads, "params": new, "norm": norm}
