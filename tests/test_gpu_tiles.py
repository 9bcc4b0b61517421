"""The tile choice of the products on one 768-wide block, forward and
backward, against the oracle: token counts at the edges of the 64-row tiles,
at the sizes where the choice changes (64 x 64, 64 x 128, 128 x 128,
128 x 192, 256-row tiles), and with ragged last tiles."""
import numpy as np
import pytest

import oracle
from paper_2609_28568_amd import synth
from tests.util import REL_L2, oracle_config, rel_l2, workload

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _np(t):
    return t.float().cpu().numpy()


# (B, T): 1 row, 63..65 (one 64-row tile and its edges), 203, 705 and 1089
# (64 x 128 and 128-row tiles with a one-row tail), 2050, and 16 x 1009 (the
# 256-row tiles, ragged; only the last sequence goes through the oracle)
@pytest.mark.parametrize("B,T", [(1, 1), (1, 63), (1, 64), (1, 65), (5, 13), (1, 203), (1, 705), (3, 363), (2, 1025), (16, 1009)])
def test_block_against_oracle(B, T):
    from paper_2609_28568_amd import binding
    w = workload("tiny", n_layer=1, n_head=12, d_model=768, d_ff=3072, vocab=64, vocab_padded=64, max_seq_len=T, B=B,
                 T=T)
    p = synth.perturb_params(synth.init_params(w, seed=71), seed=72)
    x, dy = synth.block_inputs(w, seed=73)
    b0 = max(0, B - 3)   # sequences b0.. carry gradient and are checked
    x3, dy3 = x.reshape(B, T, 768), dy.reshape(B, T, 768)
    dy3[:b0] = 0.0
    m = binding.GPT2(binding.make_config(w, synth.OPTIM))
    m.set_params(p)
    tx, tdy = (torch.from_numpy(a).cuda().to(torch.bfloat16) for a in (x, dy))
    out, dx = torch.empty_like(tx), torch.empty_like(tx)
    print(f"block {B} x {T}", flush=True)
    m.block_forward(0, tx, out)
    m.block_backward(0, tdy, dx)
    g = m.to_dict("grads")
    out, dx = _np(out).reshape(B, T, 768), _np(dx).reshape(B, T, 768)
    m.close()
    ocfg = oracle_config(w)
    y, cache = oracle.block_forward(x3[b0:], p, 0, ocfg)
    grads = oracle.zero_grads(p)
    ref = oracle.block_backward(dy3[b0:], cache, p, 0, ocfg, grads)
    assert rel_l2(out[b0:], y) < REL_L2
    assert rel_l2(dx[b0:], ref) < REL_L2
    assert np.all(dx[:b0] == 0.0)
    for k in ("ln1w", "ln1b", "qkvw", "qkvb", "attprojw", "attprojb", "ln2w", "ln2b", "fcw", "fcb", "fcprojw",
              "fcprojb"):
        # with one token the softmax is constant: its query and key gradients are exactly 0
        e = rel_l2(g[k], grads[k])
        assert e < REL_L2, (k, e)


# One block wide enough for a full round of 512 weight-gradient tiles: its
# MLP-down product is the split tail of the grouped launch and carries its bias
# sums in every chunk. 66 tokens (two chunks, one of two tokens) and 200; each
# gradient written and added to; at 320 x 1280 a launch of 93 tiles, no multiple of the 8 XCDs
@pytest.mark.parametrize("C,F", [(1024, 4096), (1024, 4032), (1536, 6144), (320, 1280)])
@pytest.mark.parametrize("B,T", [(2, 33), (1, 200)])
def test_wide_block_against_oracle(C, F, B, T):
    from paper_2609_28568_amd import binding
    w = workload("tiny", n_layer=1, n_head=C // 64, d_model=C, d_ff=F, vocab=64, vocab_padded=64, max_seq_len=T, B=B,
                 T=T)
    p = synth.perturb_params(synth.init_params(w, seed=71), seed=72)
    x, dy = synth.block_inputs(w, seed=73)
    m = binding.GPT2(binding.make_config(w, synth.OPTIM))
    m.set_params(p)
    tx, tdy = (torch.from_numpy(a).cuda().to(torch.bfloat16) for a in (x, dy))
    out, dx = torch.empty_like(tx), torch.empty_like(tx)
    print(f"block {C} x {F}, {B} x {T} tokens", flush=True)
    m.block_forward(0, tx, out)
    m.block_backward(0, tdy, dx)
    g = m.to_dict("grads")
    m.block_backward(0, tdy, dx, accumulate=True)
    g2 = m.to_dict("grads")
    out, dx = _np(out).reshape(B, T, C), _np(dx).reshape(B, T, C)
    m.close()
    ocfg = oracle_config(w)
    y, cache = oracle.block_forward(x.reshape(B, T, C), p, 0, ocfg)
    grads = oracle.zero_grads(p)
    ref = oracle.block_backward(dy.reshape(B, T, C), cache, p, 0, ocfg, grads)
    assert rel_l2(out, y) < REL_L2
    assert rel_l2(dx, ref) < REL_L2
    for k in ("ln1w", "ln1b", "qkvw", "qkvb", "attprojw", "attprojb", "ln2w", "ln2b", "fcw", "fcb", "fcprojw",
              "fcprojb"):
        assert rel_l2(g[k], grads[k]) < REL_L2, (k, rel_l2(g[k], grads[k]))
        assert rel_l2(g2[k], 2.0 * grads[k]) < REL_L2, (k, rel_l2(g2[k], 2.0 * grads[k]))


# The attention kernels for short grids (32 rows a workgroup, tiles dealt to its
# waves) at every head size: sequences of two and more tiles with one-row tails,
# up to and past the largest grids they take (256 and 512 workgroups); one head
# of 128 in 320 workgroups with walks that are too short (5 tiles) and just long
# enough (8)
@pytest.mark.parametrize("H,C", [(4, 64), (4, 128), (2, 128), (1, 128)])
@pytest.mark.parametrize("B,T", [(1, 65), (2, 130), (1, 257), (3, 300), (32, 129), (32, 300), (20, 512)])
def test_short_grid_attention(H, C, B, T):
    from paper_2609_28568_amd import binding
    w = workload("tiny", n_layer=1, n_head=H, d_model=C, d_ff=4 * C, vocab=64, vocab_padded=64, max_seq_len=T, B=B, T=T)
    p = synth.perturb_params(synth.init_params(w, seed=75), seed=76)
    p["qkvw"] *= 8.0   # scores far from uniform
    x, dy = synth.block_inputs(w, seed=77)
    m = binding.GPT2(binding.make_config(w, synth.OPTIM))
    m.set_params(p)
    tx, tdy = (torch.from_numpy(a).cuda().to(torch.bfloat16) for a in (x, dy))
    out, dx = torch.empty_like(tx), torch.empty_like(tx)
    print(f"attention {B} x {T}, {H} heads of {C // H}", flush=True)
    m.block_forward(0, tx, out)
    m.block_backward(0, tdy, dx)
    g = m.to_dict("grads")
    att, out, dx = _np(m.activation("att", 0)), _np(out), _np(dx)
    m.close()
    ocfg = oracle_config(w)
    y, cache = oracle.block_forward(x.reshape(B, T, C), p, 0, ocfg)
    grads = oracle.zero_grads(p)
    ref = oracle.block_backward(dy.reshape(B, T, C), cache, p, 0, ocfg, grads)
    assert rel_l2(att, cache["att"]) < REL_L2
    assert rel_l2(out, y) < REL_L2 and rel_l2(dx, ref) < REL_L2
    for k in ("qkvw", "qkvb", "attprojw", "ln1w"):
        assert rel_l2(g[k], grads[k]) < REL_L2, (k, rel_l2(g[k], grads[k]))


# The caller's buffers stand in for copies unless they are misaligned, overlap,
# lie in the model's own memory or (pinned) in the host's: every form gives the
# same bits.
@pytest.mark.parametrize("form", ["misaligned", "same_buffer", "own_memory", "pinned_host"])
def test_block_buffer_forms(form):
    from paper_2609_28568_amd import binding
    B, T, C = 2, 75, 64
    w = workload("tiny", n_layer=1, vocab=64, vocab_padded=64, max_seq_len=T, B=B, T=T)
    p = synth.perturb_params(synth.init_params(w, seed=71), seed=72)
    x, dy = (torch.from_numpy(a).cuda().to(torch.bfloat16) for a in synth.block_inputs(w, seed=73))

    def passes(x_in, x_out, d_out, d_in, m):
        x_in.copy_(x)
        m.block_forward(0, x_in, x_out)
        torch.cuda.synchronize()
        y = x_out.cuda().clone()
        d_out.copy_(dy)
        m.block_backward(0, d_out, d_in)
        torch.cuda.synchronize()
        return y, d_in.cuda().clone(), m.flat("grads")[64 * C + T * C:-2 * C].clone()

    m = binding.GPT2(binding.make_config(w, synth.OPTIM))
    m.set_params(p)
    ref = passes(*(torch.empty_like(x) for _ in range(4)), m)
    n = x.numel()

    def odd():
        return torch.empty(n + 1, dtype=torch.bfloat16, device="cuda")[1:].view(B * T, C)

    if form == "misaligned":
        bufs = [odd() for _ in range(4)]
    elif form == "same_buffer":
        a, b = torch.empty_like(x), torch.empty_like(x)
        bufs = [a, a, b, b]
    elif form == "pinned_host":
        bufs = [torch.empty(B * T, C, dtype=torch.bfloat16, pin_memory=True) for _ in range(4)]
    else:
        bufs = [m.activation("lnf").view(B * T, C), m.activation("att", 0).view(B * T, C),
                m.activation("lnf").view(B * T, C), m.activation("residual", 0).view(B * T, C)]
        # the output lies over a saved activation that the backward reads: only
        # the forward is compared with it, the backward with a fresh forward
        bufs[0].copy_(x)
        m.block_forward(0, bufs[0], bufs[1])
        assert torch.equal(bufs[1], ref[0])
        bufs[1] = torch.empty_like(x)
    got = passes(*bufs, m)
    m.close()
    for a, b in zip(got, ref):
        assert torch.equal(a, b)


# The gradient norm written by the clip kernel and, for memory of the host, copied
@pytest.mark.parametrize("model", ["gpt2", "qwen3"])
def test_gradient_norm_to_pinned_host(model):
    from paper_2609_28568_amd import binding, qwen3_binding as qb
    norms = []
    for pinned in (False, True):
        out = torch.zeros(1, pin_memory=True) if pinned else torch.zeros(1, device="cuda")
        if model == "gpt2":
            w = workload("tiny")
            m = binding.GPT2(binding.make_config(w, synth.OPTIM))
            m.set_params(synth.init_params(w))
            ids, tgt = synth.token_batch(w)
        else:
            w = dict(synth.QWEN3_WORKLOADS["qwen3_tiny"])
            m = qb.Qwen3(qb.make_config(w, synth.QWEN3_OPTIM))
            base, lora = synth.init_qwen3(w, b_std=0.02)
            m.set_base(base)
            m.set_lora(lora)
            ids, tgt = synth.token_batch(w)
        m.forward(torch.from_numpy(ids), torch.from_numpy(tgt))
        m.backward()
        g = (m.flat("grads") if model == "gpt2" else m.flat("lora_grads")).double().norm().item()
        m.adamw_step(0, out)
        torch.cuda.synchronize()
        norms.append(out.item())
        m.close()
        assert norms[-1] == pytest.approx(g, rel=1e-5)
    assert norms[0] == norms[1]


# Depths at the edges of the grouped weight-gradient plan at 768 wide (192
# tiles a layer, rounds of 512): under a round (1, 2), every MLP-down product
# in the split tail (4), a tail of some of them (7), no tail (8)
@pytest.mark.parametrize("L", [1, 2, 4, 7, 8])
def test_grouped_weight_gradients_by_depth(L):
    from paper_2609_28568_amd import binding
    w = workload("tiny", n_layer=L, n_head=12, d_model=768, d_ff=3072, vocab=64, vocab_padded=64, max_seq_len=33, B=2,
                 T=33)
    p = synth.perturb_params(synth.init_params(w, seed=81), seed=82)
    ids, tgt = synth.token_batch(w, seed=83)
    m = binding.GPT2(binding.make_config(w, synth.OPTIM))
    m.set_params(p)
    print(f"step of {L} layers", flush=True)
    m.forward(torch.from_numpy(ids), torch.from_numpy(tgt))
    m.backward()
    g = m.to_dict("grads")
    m.close()
    ocfg = oracle_config(w)
    ref = oracle.backward(p, oracle.forward(p, ids, tgt, ocfg), ocfg)
    for k in oracle.KINDS:
        assert rel_l2(g[k], ref[k]) < REL_L2, (k, rel_l2(g[k], ref[k]))


# The 256 x 128 tiles of the grouped weight gradients (4096 tokens or more),
# ragged tokens: one 2048-wide block without a tail; 704 x 1408 (three chunks of
# the tokens, tiles that reach past the rows); 1024 x 64 (fewer rows than a
# tile); three 1024-wide layers of which one MLP-down product is the split tail
@pytest.mark.parametrize("H,C,F", [(16, 2048, 8192), (11, 704, 1408), (16, 1024, 64)])
def test_grouped_256_row_tiles_of_one_block(H, C, F):
    from paper_2609_28568_amd import binding
    B, T = 16, 257
    w = workload("tiny", n_layer=1, n_head=H, d_model=C, d_ff=F, vocab=64, vocab_padded=64, max_seq_len=T, B=B, T=T)
    p = synth.perturb_params(synth.init_params(w, seed=71), seed=72)
    x, dy = synth.block_inputs(w, seed=73)
    x3, dy3 = x.reshape(B, T, C), dy.reshape(B, T, C)
    dy3[:-2] = 0.0   # the last two sequences carry gradient
    m = binding.GPT2(binding.make_config(w, synth.OPTIM))
    m.set_params(p)
    tx, tdy = (torch.from_numpy(a).cuda().to(torch.bfloat16) for a in (x, dy))
    print(f"block of {C} x {F}, {B} x {T} tokens", flush=True)
    m.block_forward(0, tx)
    m.block_backward(0, tdy)
    g = m.to_dict("grads")
    m.close()
    ocfg = oracle_config(w)
    cache = oracle.block_forward(x3[-2:], p, 0, ocfg)[1]
    grads = oracle.zero_grads(p)
    oracle.block_backward(dy3[-2:], cache, p, 0, ocfg, grads)
    for k in ("qkvw", "qkvb", "attprojw", "attprojb", "fcw", "fcb", "fcprojw", "fcprojb"):
        assert rel_l2(g[k], grads[k]) < REL_L2, (k, rel_l2(g[k], grads[k]))


def test_grouped_256_row_tiles_of_three_layers():
    from paper_2609_28568_amd import binding
    B, T, C = 16, 257, 1024
    w = workload("tiny", n_layer=3, n_head=16, d_model=C, d_ff=4 * C, vocab=64, vocab_padded=64, max_seq_len=T, B=B, T=T)
    p = synth.perturb_params(synth.init_params(w, seed=81), seed=82)
    ids, tgt = synth.token_batch(w, seed=83)
    m = binding.GPT2(binding.make_config(w, synth.OPTIM))
    m.set_params(p)
    print(f"3 layers of {C}, {B} x {T} tokens", flush=True)
    m.forward(torch.from_numpy(ids), torch.from_numpy(tgt))
    m.backward()
    g = m.to_dict("grads")
    m.close()
    ocfg = oracle_config(w)
    ref = oracle.backward(p, oracle.forward(p, ids, tgt, ocfg), ocfg)
    for k in oracle.KINDS:
        assert rel_l2(g[k], ref[k]) < REL_L2, (k, rel_l2(g[k], ref[k]))


# The token-table scatter against a float64 sum: runs of one id that span
# half-waves and workgroups, ids out of range skipped, few and many positions
@pytest.mark.parametrize("n,distinct", [(1, 1), (255, 1), (257, 3), (1000, 500), (4096, 2), (4097, 4000), (5000, 37)])
@pytest.mark.parametrize("C", [64, 192])
def test_embedding_scatter(n, distinct, C):
    from paper_2609_28568_amd import binding
    V = 5000
    w = workload("tiny", n_layer=1, n_head=C // 16, d_model=C, d_ff=4 * C, vocab=V, vocab_padded=5056, max_seq_len=n, B=1, T=n)
    m = binding.GPT2(binding.make_config(w, synth.OPTIM))
    r = np.random.default_rng([91, n, distinct])
    ids = r.permutation(V)[r.integers(0, distinct, n)].astype(np.int32)
    bad = ids.copy()
    bad[::97] = V + 5
    dx = synth.round_to_bf16(r.standard_normal((n, C), dtype=np.float32))
    print(f"scatter of {n} positions, {distinct} ids", flush=True)
    m.embedding_backward(torch.from_numpy(bad), torch.from_numpy(dx).cuda().to(torch.bfloat16))
    g = m.to_dict("grads")["wte"]
    m.close()
    ok = bad < V
    ref, mag = np.zeros((5056, C)), np.zeros((5056, C))
    np.add.at(ref, bad[ok], dx[ok].astype(np.float64))
    np.add.at(mag, bad[ok], np.abs(dx[ok]).astype(np.float64))
    # an n-term fp32 sum in any order is within n ulps of the sum of magnitudes
    assert np.all(np.abs(g - ref) <= n * 2.0 ** -24 * mag)
