"""The calls that a program built on this package spends its time in, as measurable cases.

Each case is one pass through the public entry points (PolicyMaskedMoE, PrivateAdamW,
pmpe_fingerprint) on one layer, over the shapes of `workloads` and a generic one:

* forward    route, dispatch, expert FFN, combine and audit of one batch (serving: a few
             requests decoding, a full decode batch, chunked prefill mixed with decode rows,
             whole prefills, the 16384-token layer of a long stack);
* fp8        the same with fp8 expert weights;
* train      a training forward and the private-only backward of one batch;
* optimizer  one AdamW step over the private parameters and the refresh of their transposed
             copies, which follows every backward;
* fingerprint  the digest of the frozen weights, taken around training and reloads.

Inputs come from the seed: x and dout N(0, 1), weights and router rows N(0, 0.02) as in
`workloads.synth`, requests of ragged lengths whose metadata allows, denies or is malformed.
"""
import math
import random

import numpy as np
import torch

import paper_2608_06690_amd as P

# hidden, inter, public, private, top-k, shared experts, dtype, gate rule, router bias
SHAPES = {
    # Qwen3-30B-A3B-shaped layer
    "qwen": dict(h=2048, i=768, pub=128, priv=32, k=8, sh=0, dt="bf16", gate="renorm", bias=None),
    # the same layer under decode traffic, whose expert use is skewed (Zipf 1.1)
    "qwen_zipf": dict(h=2048, i=768, pub=128, priv=32, k=8, sh=0, dt="bf16", gate="renorm", bias="zipf"),
    # DeepSeek-V2-Lite-shaped layer: two shared experts, softmax over the permitted pool
    "deepseek": dict(h=2048, i=1408, pub=64, priv=16, k=6, sh=2, dt="bf16", gate="pool", bias="normal"),
    # a generic layer whose sizes divide no tile of 256
    "generic": dict(h=1664, i=640, pub=40, priv=12, k=4, sh=0, dt="bf16", gate="renorm", bias=None),
    # a generic layer with an inner width that no tile of 128 divides
    "odd": dict(h=1152, i=704, pub=24, priv=24, k=3, sh=1, dt="bf16", gate="pool", bias=None),
    # the small fp32 layer
    "tiny": dict(h=128, i=256, pub=8, priv=4, k=2, sh=0, dt="f32", gate="renorm", bias=None),
}
MAX_TOKENS = {"qwen": 16384, "qwen_zipf": 1024, "deepseek": 8192, "generic": 8192, "odd": 8192, "tiny": 512}


def listed():
    return [
        # the smallest call: the fp32 layer on four short requests
        dict(name="tiny_f32_64", op="forward", shape="tiny", tokens=64, requests=4, allow=0.5),
        # interactive decode: a handful of requests, one token each
        dict(name="decode_8", op="forward", shape="qwen_zipf", tokens=8, requests=8, allow=0.25),
        # a full decode batch
        dict(name="decode_256", op="forward", shape="qwen_zipf", tokens=256, requests=256, allow=0.25),
        # a decode batch with fp8 expert weights
        dict(name="fp8_decode_200", op="fp8", shape="qwen_zipf", tokens=200, requests=200, allow=0.25),
        # chunked prefill: prompts of ragged lengths next to decoding requests
        dict(name="mixed_1111", op="forward", shape="qwen", tokens=1111, requests=37, allow=0.5),
        # the benchmark's prefill
        dict(name="prefill_qwen_4096", op="forward", shape="qwen", tokens=4096, requests=8, allow=0.5),
        # a prefill with shared experts, a logit bias and pool-softmax gates
        dict(name="prefill_deepseek_8192", op="forward", shape="deepseek", tokens=8192, requests=16, allow=0.5),
        # one layer of the 48-layer stack, every request authorised
        dict(name="stack_16384", op="forward", shape="qwen", tokens=16384, requests=32, allow=1.0),
        # one training micro-batch of the Qwen-shaped layer
        dict(name="train_qwen_4096", op="train", shape="qwen", tokens=4096, requests=8, allow=0.5),
        # a shorter, ragged training micro-batch of the DeepSeek-shaped layer
        dict(name="train_deepseek_2000", op="train", shape="deepseek", tokens=2000, requests=7, allow=0.5),
        # the optimizer step of the Qwen-shaped layer's private pool
        dict(name="adamw_qwen_32", op="optimizer", shape="qwen", experts=32),
        # the fingerprint of its public expert weights
        dict(name="fingerprint_1152m", op="fingerprint", bytes=1207959552),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    u = rng.random()
    if u < 0.60:
        shape = rng.choice(["qwen", "qwen", "qwen_zipf", "qwen_zipf", "deepseek", "generic", "odd", "tiny"])
        t = _log_int(rng, 16 if shape == "tiny" else 1, MAX_TOKENS[shape])
        return dict(op="forward", shape=shape, tokens=t, requests=_log_int(rng, 1, t), allow=round(rng.random(), 3))
    if u < 0.72:
        t = _log_int(rng, 1, 4096)
        return dict(op="fp8", shape=rng.choice(["qwen", "qwen_zipf", "generic"]), tokens=t,
                    requests=_log_int(rng, 1, t), allow=round(rng.random(), 3))
    if u < 0.86:
        shape = rng.choice(["qwen", "deepseek", "generic"])
        t = _log_int(rng, 64, {"qwen": 4096, "deepseek": 2048, "generic": 4096}[shape])
        return dict(op="train", shape=shape, tokens=t, requests=_log_int(rng, 1, 16), allow=round(rng.uniform(0.2, 1.0), 3))
    if u < 0.93:
        return dict(op="optimizer", shape=rng.choice(["qwen", "generic"]), experts=rng.randint(8, 32))
    return dict(op="fingerprint", bytes=_log_int(rng, 1 << 10, 1207959552))


# ---------------------------------------------------------------------------- inputs


def _randn(gen, shape, std, dtype):
    out = torch.empty(shape, dtype=dtype, device="cuda")
    return out.normal_(0.0, std, generator=gen)


def _requests(case, seed):
    """Lengths and metadata of the batch's requests: ragged unless they divide it evenly."""
    rng = random.Random(seed * 7919 + 17)
    t, r = case["tokens"], case["requests"]
    if t % r == 0:
        lengths = [t // r] * r
    else:
        cuts = sorted(rng.sample(range(1, t), r - 1))
        lengths = [b - a for a, b in zip([0] + cuts, cuts + [t])]
    n_allow = round(case["allow"] * r)
    metas = [{"allow_private": True}] * n_allow
    bad = [None, {}, {"allow_private": "true"}, {"allow_private": 1}]
    for j in range(r - n_allow):
        metas.append(bad[j % 4] if j % 8 == 7 else {"allow_private": False})
    rng.shuffle(metas)
    return lengths, metas


def _fp8_rows(w):
    """e4m3 bytes and one power-of-two fp32 scale per row."""
    amax = w.float().abs().amax(dim=-1)
    scale = torch.exp2(torch.ceil(torch.log2(amax.clamp(min=1e-30) / 448.0)))
    q = (w.float() / scale.unsqueeze(-1)).to(torch.float8_e4m3fn)
    return q.view(torch.uint8), scale.contiguous()


def _layer_inputs(case, seed):
    s = SHAPES[case["shape"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    f32 = s["dt"] == "f32"
    dt = torch.float32 if f32 else torch.bfloat16
    h, i, e = s["h"], s["i"], s["pub"] + s["priv"]
    d = {"wr": _randn(gen, (e, h), 0.02, torch.float32)}
    d["bias"] = None
    if s["bias"] == "normal":
        d["bias"] = _randn(gen, (e,), 1.0, torch.float32)
    elif s["bias"] == "zipf":
        rng = np.random.default_rng([seed, 5])
        ranks = np.concatenate([rng.permutation(s["pub"]) + 1, rng.permutation(s["priv"]) + 1])
        d["bias"] = torch.from_numpy((-1.1 * np.log(ranks)).astype(np.float32)).cuda()
    d["w13"] = _randn(gen, (e, 2 * i, h), 0.02, dt)
    d["w2"] = _randn(gen, (e, h, i), 0.02, dt)
    d["w13_sh"] = _randn(gen, (2 * s["sh"] * i, h), 0.02, dt) if s["sh"] else None
    d["w2_sh"] = _randn(gen, (h, s["sh"] * i), 0.02, dt) if s["sh"] else None
    if "tokens" in case:
        d["x"] = _randn(gen, (case["tokens"], h), 0.02 if f32 else 1.0, dt)
        if case["op"] == "train":
            d["dout"] = _randn(gen, (case["tokens"], h), 1.0, dt)
        lengths, metas = _requests(case, seed)
        d["words"] = P.token_policy_words(metas, lengths, "cuda")
        d["offsets"] = P.request_offsets(lengths, "cuda")
        tau = [m is not None and m.get("allow_private") is True for m in metas]
        d["allow"] = torch.from_numpy(np.repeat(np.asarray(tau), lengths)).cuda()
    return s, d


def _desc(s):
    gate = P.PMPE_GATE_POOL_SOFTMAX if s["gate"] == "pool" else P.PMPE_GATE_RENORM_TOPK
    return P.make_desc(s["h"], s["i"], s["pub"], s["priv"], s["k"], s["sh"], s["i"] if s["sh"] else 0,
                       s["dt"] == "bf16", gate)


def _grads(gen, layer):
    g = P.GradBuffers(dx=None, dw13_priv=_randn(gen, layer.w13_priv.shape, 1e-2, torch.float32),
                      dw2_priv=_randn(gen, layer.w2_priv.shape, 1e-2, torch.float32),
                      dwr_priv=_randn(gen, layer.wr_priv.shape, 1e-2, torch.float32), grad_rows=None, ws=None)
    return g


ADAMW = dict(lr=1e-5, betas=(0.9, 0.95), eps=1e-8, weight_decay=0.01)


def _optimizer_inputs(case, seed):
    s = SHAPES[case["shape"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, h, i = case["experts"], s["h"], s["i"]
    # the optimizer only touches the private tensors; one public expert stands for the rest
    d = dict(wr_pub=_randn(gen, (n, h), 0.02, torch.float32), wr=_randn(gen, (n, h), 0.02, torch.float32),
             w13_pub=_randn(gen, (n, 2 * i, h), 0.02, torch.bfloat16),
             w2_pub=_randn(gen, (n, h, i), 0.02, torch.bfloat16),
             w13=_randn(gen, (n, 2 * i, h), 0.02, torch.bfloat16), w2=_randn(gen, (n, h, i), 0.02, torch.bfloat16))
    desc = P.make_desc(h, i, n, n, min(s["k"], n))
    layer = P.PolicyMaskedMoE(desc, d["wr_pub"], d["wr"], None, d["w13_pub"], d["w2_pub"], d["w13"], d["w2"])
    return layer, _grads(gen, layer)


def prepare(case, seed):
    op = case["op"]
    if op == "fingerprint":
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        n = case["bytes"]
        data = torch.randint(-2**62, 2**62, ((n + 7) // 8,), generator=gen, device="cuda").view(torch.uint8)[:n]
        ws = torch.empty(max(1, P.pmpe_fingerprint_workspace_bytes(n)), dtype=torch.uint8, device="cuda")
        return dict(op=op, data=data, ws=ws, digest=torch.empty(32, dtype=torch.uint8, device="cuda"))
    if op == "optimizer":
        layer, g = _optimizer_inputs(case, seed)
        layer.transposed_weights()  # kept by a layer that trains
        return dict(op=op, layer=layer, g=g, opt=P.PrivateAdamW(layer, **ADAMW))
    s, d = _layer_inputs(case, seed)
    n = s["pub"]
    layer = P.PolicyMaskedMoE(_desc(s), d["wr"][:n], d["wr"][n:], d["bias"], d["w13"][:n], d["w2"][:n], d["w13"][n:],
                              d["w2"][n:], d["w13_sh"], d["w2_sh"])
    t = case["tokens"]
    st = dict(op=op, layer=layer, x=d["x"], words=d["words"], offsets=d["offsets"],
              audit=layer.audit_buffers(t, case["requests"]))
    if op == "fp8":
        q13, s13 = _fp8_rows(d["w13"])
        q2, s2 = _fp8_rows(d["w2"])
        st["fp8"] = (q13[:n], q2[:n], q13[n:], q2[n:], s13[:n], s2[:n], s13[n:], s2[n:])
    if op == "train":
        st["dout"] = d["dout"]
        st["grads"] = layer.grad_buffers(t)
        layer.transposed_weights()  # kept by a layer that trains
    return st


def run(state):
    op = state["op"]
    if op == "fingerprint":
        P.pmpe_fingerprint(state["data"], state["digest"], state["ws"])
        return state["digest"]
    if op == "optimizer":
        layer, opt = state["layer"], state["opt"]
        opt.step(state["g"])
        w2t, w13t = layer.transposed_weights()[2:]
        return dict(wr=layer.wr_priv, w13=layer.w13_priv, w2=layer.w2_priv, w2t=w2t, w13t=w13t,
                    master=opt.master[1:], m=opt.m, v=opt.v)
    layer, x, audit = state["layer"], state["x"], state["audit"]
    audit.zero_()
    if op == "fp8":
        b = layer.forward_fp8(x, state["words"], state["fp8"], audit, state["offsets"])
    else:
        b = layer.forward(x, state["words"], audit, state["offsets"], train=op == "train")
    out = dict(out=b.out, idx=b.topk_idx, gate=b.topk_gate, kgap=b.kgap, allow=b.allow, req_rows=audit.req_rows,
               total=audit.total, violations=audit.violations)
    if op == "train":
        g = layer.backward(x, state["dout"], b, state["grads"])
        out.update(dx=g.dx, dw13=g.dw13_priv, dw2=g.dw2_priv, dwr=g.dwr_priv, grad_rows=g.grad_rows)
    return out


# ---------------------------------------------------------------------------- work and tolerance


def _experts_hit(s, n, tokens):
    """Experts of a pool of n that `tokens` tokens select (a fixed draw of their logits)."""
    if tokens == 0:
        return 0
    rng = np.random.default_rng([n, tokens])
    z = rng.normal(0.0, 0.02 * math.sqrt(s["h"]), (min(tokens, 2048), n))
    if s["bias"] == "zipf":
        z -= 1.1 * np.log(np.arange(1, n + 1))
    elif s["bias"] == "normal":
        z += rng.normal(0.0, 1.0, n)
    return len(np.unique(np.argpartition(-z, s["k"] - 1, axis=1)[:, : s["k"]]))


def work(case):
    op = case["op"]
    if op == "fingerprint":
        return {"bytes": case["bytes"] + 32, "flops": 0}  # integer work: about 22 operations per byte
    s = SHAPES[case["shape"]]
    h, i, k = s["h"], s["i"], s["k"]
    if op == "optimizer":
        n = case["experts"]
        we, wr = n * 3 * h * i, n * h
        # experts: master, m, v read and written, grad read, bf16 weight and its transpose written
        return {"bytes": we * (12 + 12 + 4 + 2 + 2) + wr * 28, "flops": 15 * (we + wr)}
    t = case["tokens"]
    el = 4 if s["dt"] == "f32" else 2
    wel = 1 if op == "fp8" else el
    ta = round(case["allow"] * t)
    pairs_priv = ta * k
    priv, pub = _experts_hit(s, s["priv"], ta), _experts_hit(s, s["pub"], t - ta)
    sh = 3 * h * i * s["sh"]
    rows = (s["pub"] if ta < t else 0) + (s["priv"] if ta else 0)
    weights = (priv + pub) * 3 * h * i * wel + sh * el
    nbytes = weights + rows * h * 4 + 2 * t * h * el + t * (4 + k * 8 + 5)
    flops = 6 * h * i * t * k + 2 * t * sh + 2 * h * (ta * s["priv"] + (t - ta) * s["pub"])
    if op == "train":
        grads = s["priv"] * (3 * h * i + h) * 4
        # the backward: x, dout, the touched weights and the router again, dx and the gradients
        nbytes += 2 * t * h * el + weights + rows * h * 4 + t * h * 4 + grads
        flops += 6 * h * i * t * k + 6 * h * i * pairs_priv + 6 * t * sh  # dh, dx rows; weight gradients; shared
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    op = case["op"]
    if op == "fingerprint":
        return "exact"
    if op == "optimizer":
        # fp32 sums; a bf16 weight may round the other way (2^-8 of its value)
        return {"rel": 2e-4, "max": 0.02}
    if case["shape"] == "tiny":
        return {"rel": 2e-6, "max": 8e-5}
    # bf16 rounding of h, y and out (about 3e-3 off 64-bit arithmetic); whole values may
    # differ where two logits tie to within fp32 rounding
    return {"rel": 1.2e-2, "max": 0.5, "differ": 2e-3}


# ---------------------------------------------------------------------------- 64-bit results


def _silu(g):
    return g * torch.sigmoid(g)


def _exact_optimizer(case, seed):
    layer, g = _optimizer_inputs(case, seed)
    (b1, b2), lr, eps, wd = ADAMW["betas"], ADAMW["lr"], ADAMW["eps"], ADAMW["weight_decay"]
    new, m, v = [], [], []
    for p, gr in ((layer.wr_priv, g.dwr_priv), (layer.w13_priv, g.dw13_priv), (layer.w2_priv, g.dw2_priv)):
        gr = gr.double()
        m.append((1 - b1) * gr)
        v.append((1 - b2) * gr * gr)
        new.append(p.double() * (1 - lr * wd) - lr * gr / (gr.abs() + eps))
    return dict(wr=new[0], w13=new[1], w2=new[2], w2t=new[2].transpose(1, 2), w13t=new[1].transpose(1, 2),
                master=new[1:], m=m, v=v)


def exact(case, seed):
    op = case["op"]
    if op == "fingerprint":
        return None
    if op == "optimizer":
        return _exact_optimizer(case, seed)
    s, d = _layer_inputs(case, seed)
    h, i, k, n, e = s["h"], s["i"], s["k"], s["pub"], s["pub"] + s["priv"]
    t = case["tokens"]
    train = op == "train"
    x, allow = d["x"].double(), d["allow"]
    wr = d["wr"].double()
    z = x @ wr.t()
    if d["bias"] is not None:
        z = z + d["bias"].double()
    pool = torch.zeros(t, e, dtype=torch.bool, device="cuda")
    pool[:, :n] = ~allow.unsqueeze(1)
    pool[:, n:] = allow.unsqueeze(1)
    zm = z.masked_fill(~pool, -math.inf)
    top, idx = zm.topk(min(k + 1, e), dim=1)
    kgap = top[:, k - 1] - top[:, k]
    idx = idx[:, :k].sort(dim=1).values
    sel = zm.gather(1, idx)
    if s["gate"] == "pool":
        prob = torch.softmax(zm, dim=1)
        gate = prob.gather(1, idx)
    else:
        gate = torch.softmax(sel, dim=1)
    out = torch.zeros(t, h, dtype=torch.float64, device="cuda")
    if train:
        go = d["dout"].double()
        dx, dg = torch.zeros_like(out), torch.zeros_like(gate)
        dw13 = torch.zeros(e - n, 2 * i, h, dtype=torch.float64, device="cuda")
        dw2 = torch.zeros(e - n, h, i, dtype=torch.float64, device="cuda")

    def group(w13, w2, rows, gates):
        """One SwiGLU over `rows`: output rows, and with a gradient its products."""
        w13, w2 = w13.double(), w2.double()
        width = w2.shape[1]
        xr = x[rows]
        ab = xr @ w13.t()
        a, b = ab[:, :width], ab[:, width:]
        hh = _silu(a) * b
        y = hh @ w2.t()
        if not train:
            return y, None
        up = gates.unsqueeze(1) * go[rows]
        dh = up @ w2
        sg = torch.sigmoid(a)
        dab = torch.cat([dh * b * sg * (1 + a * (1 - sg)), dh * a * sg], dim=1)
        return y, (xr, up, hh, dab, dab @ w13)

    for j in range(e):
        rows, slot = (idx == j).nonzero(as_tuple=True)
        if rows.numel() == 0:
            continue
        w13, w2 = d["w13"][j], d["w2"][j]
        if op == "fp8":
            (q13, s13), (q2, s2) = _fp8_rows(w13), _fp8_rows(w2)
            w13 = q13.view(torch.float8_e4m3fn).double() * s13.double().unsqueeze(1)
            w2 = q2.view(torch.float8_e4m3fn).double() * s2.double().unsqueeze(1)
        g = gate[rows, slot]
        y, back = group(w13, w2, rows, g)
        out.index_add_(0, rows, g.unsqueeze(1) * y)
        if train:
            xr, up, hh, dab, dxr = back
            dg[rows, slot] = (go[rows] * y).sum(dim=1)
            dx.index_add_(0, rows, dxr)
            if j >= n:
                dw13[j - n] = dab.t() @ xr
                dw2[j - n] = up.t() @ hh
    if s["sh"]:
        rows = torch.arange(t, device="cuda")
        y, back = group(d["w13_sh"], d["w2_sh"], rows, torch.ones(t, dtype=torch.float64, device="cuda"))
        out += y
        if train:
            dx += back[4]
    res = dict(out=out, idx=None, gate=gate.reshape(-1), kgap=kgap, allow=None, req_rows=None, total=None,
               violations=None)
    if train:
        dz = torch.zeros_like(z)
        if s["gate"] == "pool":
            up = torch.zeros_like(z).scatter_(1, idx, dg)
            dz = prob * (up - (gate * dg).sum(dim=1, keepdim=True))
        else:
            dz.scatter_(1, idx, gate * (dg - (gate * dg).sum(dim=1, keepdim=True)))
        dx += dz @ wr
        res.update(dx=dx, dw13=dw13, dw2=dw2, dwr=(dz.t() @ x)[n:], grad_rows=None)
    return res
