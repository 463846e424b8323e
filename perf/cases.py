"""The measured cases of the block-diffusion decoding library.

Every case is a call that a serving program makes through the public binding
(``paper_2609_33887_amd.bd``): a denoising step with its commit on a decode
state that holds an encoded batch (``State.reset``, ``State.step``,
``State.commit``), or a prefill, which makes such a state, with its first step
(``bd.State``).  Layer shapes are those of the repository's workloads:

  gqa    d 2048, 16 q-heads over 4 kv-heads of 128, SwiGLU 8192 (multi-block
         and long-prefix workloads)
  moe    the same attention, 64 experts of 512, top 8, one shared expert
  dense  d 1024, 16 heads of 64, SwiGLU 4096
  tiny   fp32: d 256, 4 heads of 64, SwiGLU 1024

Two listed cases run whole models with their own vocabularies (24 gqa layers,
12 dense layers), the others a few layers under a head of 4096 tokens, so that
each shows its layers; one shows the head alone over the full vocabulary.
Weights are N(0, 0.02) with RMSNorm gains around one and prompts are uniform
over the vocabulary, as in the repository's workloads, drawn on the GPU from
the seed.  The generation length is one window (n_inflight x block_size), so
every generated position is masked in the step and every output is written.
"""
import math

import torch

from paper_2609_33887_amd import bd

SHAPES = {
    "gqa": dict(d=2048, H=16, Hkv=4, hd=128, F=8192, E=0, k=0, Fe=0, ns=0),
    "moe": dict(d=2048, H=16, Hkv=4, hd=128, F=0, E=64, k=8, Fe=512, ns=1),
    "dense": dict(d=1024, H=16, Hkv=16, hd=64, F=4096, E=0, k=0, Fe=0, ns=0),
    "tiny": dict(d=256, H=4, Hkv=4, hd=64, F=1024, E=0, k=0, Fe=0, ns=0),
}
EPS, THETA, SCALE, TAU = 1e-6, 1e4, 20.0, 0.9


def _case(call, shape, layers, vocab, wq, b, P, B, nb, logits=True):
    return {"call": call, "shape": shape, "layers": layers, "vocab": vocab, "wq": wq, "b": b, "P": P, "B": B,
            "nb": nb, "logits": logits}


def listed():
    cases = [
        # the tiny fp32 model, one block of four tokens: the smallest call, all launch latency
        ("tiny_f32_b1", _case("step", "tiny", 2, 4096, "f32", 1, 32, 4, 1)),
        # one interactive request on the whole 24-layer model, three blocks in flight: weights streamed for 96 rows
        ("model_gqa_b1", _case("step", "gqa", 24, 152064, "bf16", 1, 1024, 32, 3)),
        # the whole small-batch dense model at its own batch and prompt: many short launches over 512 rows
        ("model_dense_b16", _case("step", "dense", 12, 32768, "bf16", 16, 512, 32, 1)),
        # layers of the multi-block decode at its own batch: the largest windows (3072 rows)
        ("layers_gqa_b32", _case("step", "gqa", 2, 4096, "bf16", 32, 1024, 32, 3)),
        # the same layers at a serving batch of 8 with two blocks in flight and a prompt off the powers of two
        ("layers_gqa_b8", _case("step", "gqa", 2, 4096, "bf16", 8, 1440, 32, 2)),
        # layers of the long-prefix decode at its own batch: attention over 8320 keys
        ("layers_gqa_long_b8", _case("step", "gqa", 2, 4096, "bf16", 8, 8192, 64, 2)),
        # an MoE layer at the selection sweep's batch (2048 rows, every expert busy)
        ("layer_moe_b64", _case("step", "moe", 1, 4096, "bf16", 64, 256, 32, 1)),
        # an MoE layer for three requests: 96 rows spread thinly over 64 experts
        ("layer_moe_b3", _case("step", "moe", 1, 4096, "bf16", 3, 224, 32, 1)),
        # fp8 layer weights on the dense model's layers
        ("layers_dense_fp8_b16", _case("step", "dense", 2, 4096, "fp8", 16, 512, 32, 1)),
        # MXFP4 layer weights on the gqa layers at a serving batch
        ("layers_gqa_mxfp4_b8", _case("step", "gqa", 2, 4096, "mxfp4", 8, 1024, 32, 2)),
        # the fused head over the full vocabulary on the largest window, behind one layer; it never forms logits in
        # this use, so its outputs are each position's confidence and token
        ("head_gqa_b32", _case("step", "gqa", 1, 152064, "bf16", 32, 256, 32, 3, logits=False)),
        # encoding a batch of four prompts (a state made, its first step, the state given back) on half the model
        ("prefill_gqa_b4", _case("prefill", "gqa", 12, 4096, "bf16", 4, 1024, 32, 2)),
    ]
    return [dict(c, name=n) for n, c in cases]


def draw(rng):
    """A case of the listed ranges: the same layer shapes and formats with other batches, prompts, blocks and
    windows, a few layers deep."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["gqa", "gqa", "long", "moe", "moe", "dense", "fp8", "mxfp4", "prefill", "tiny"])
        if kind == "tiny":
            c = _case("step", "tiny", rng.randint(1, 2), 4096, "f32", log(1, 8), 0, rng.choice([1, 4, 8]),
                      rng.randint(1, 2))
            c["P"] = c["B"] * log(2, 128 // c["B"])
            return c
        B = rng.choice([16, 32, 32, 48, 64])
        nb = rng.randint(1, 4)
        if kind == "long":
            c = _case("step", "gqa", rng.randint(1, 2), 4096, "bf16", log(1, 8), B * (log(2048, 8192) // B), B, nb)
        elif kind == "prefill":
            c = _case("prefill", "gqa", rng.randint(4, 12), 4096, "bf16", log(1, 4), B * (log(128, 1024) // B), B, nb)
        elif kind == "moe":
            c = _case("step", "moe", 1, 4096, "bf16", log(1, 64), B * (log(64, 512) // B), B, min(nb, 2))
        elif kind == "dense" or kind == "fp8":
            c = _case("step", "dense", rng.randint(1, 4), 4096, "fp8" if kind == "fp8" else "bf16", log(1, 32),
                      B * (log(64, 1024) // B), B, min(nb, 2))
        else:
            c = _case("step", "gqa", rng.randint(1, 2), 4096, "mxfp4" if kind == "mxfp4" else "bf16", log(1, 32),
                      B * (log(64, 2048) // B), B, nb)
        if c["b"] * c["nb"] * c["B"] <= 3072 and c["b"] * c["P"] <= 65536:
            return c


# ---------------------------------------------------------------- inputs
def _tensors(case):
    """(shape, kind) of the weight tensors in the order of bd_init_model."""
    s = SHAPES[case["shape"]]
    d, q, hd, E, Fe, Fs = s["d"], s["H"] * s["hd"], s["hd"], s["E"], s["Fe"], s["ns"] * s["Fe"]
    out = [((case["vocab"], d), "mat")]
    for _ in range(case["layers"]):
        out += [((d,), "gain"), (((s["H"] + 2 * s["Hkv"]) * hd, d), "mat"), ((d, q), "mat"), ((d,), "gain")]
        if E:
            out += [((E, d), "router"), ((E, Fe, d), "mat"), ((E, Fe, d), "mat"), ((E, d, Fe), "mat"),
                    ((Fs, d), "mat"), ((Fs, d), "mat"), ((d, Fs), "mat")]
        else:
            out += [((s["F"], d), "mat"), ((s["F"], d), "mat"), ((d, s["F"]), "mat")]
    return out + [((d,), "gain"), ((case["vocab"], d), "mat")]


def _draw_weight(case, seed, i, shape, kind):
    g = torch.Generator(device="cuda").manual_seed((seed * 4096 + i) & 0x7FFFFFFFFFFF)
    if kind == "gain":
        return 0.8 + 0.4 * torch.rand(shape, generator=g, device="cuda")
    w = torch.randn(shape, generator=g, device="cuda").mul_(0.02)
    return w if kind == "router" or case["wq"] == "f32" else w.bfloat16()


def _prompts(case, seed):
    g = torch.Generator(device="cuda").manual_seed((seed * 4096 + 4095) & 0x7FFFFFFFFFFF)
    return torch.randint(0, case["vocab"] - 1, (case["b"], case["P"]), generator=g, device="cuda", dtype=torch.int32)


class _Model:
    """Weights drawn on the device under a library handle (bd.Model takes host arrays)."""

    def __init__(self, case, seed):
        s = SHAPES[case["shape"]]
        self.handle = None
        self.torch, self.device = torch, torch.device("cuda", torch.cuda.current_device())
        self.tensors = [_draw_weight(case, seed, i, sh, kind) for i, (sh, kind) in enumerate(_tensors(case))]
        f32 = case["wq"] == "f32"
        self.cfg = bd.bd_model_cfg(
            n_layers=case["layers"], d_model=s["d"], n_heads=s["H"], n_kv_heads=s["Hkv"], head_dim=s["hd"],
            ffn_dim=s["F"], vocab=case["vocab"], n_experts=s["E"], top_k=s["k"], expert_ffn=s["Fe"],
            n_shared=s["ns"], rms_eps=EPS, rope_theta=THETA, logit_scale=SCALE, mask_id=case["vocab"] - 1,
            dtype=bd.BD_F32 if f32 else bd.BD_BF16, wq=0 if f32 else bd.WQ[case["wq"]])
        self.stream = torch.cuda.current_stream(self.device)
        self.handle = bd.bd_init_model(self.cfg, [t.data_ptr() for t in self.tensors], self.stream.cuda_stream)

    def __del__(self):
        if self.handle:
            bd.bd_model_free(self.handle)


class _Held:
    """What the program holds: the model, its prompts, the output buffers and (for steps) the decode state."""

    def __init__(self, case, seed):
        self.case = case
        self.model = _Model(case, seed)
        self.prompts = _prompts(case, seed)
        self.G = case["nb"] * case["B"]
        dev = self.model.device
        self.conf = torch.zeros((case["b"], self.G), device=dev)
        self.tok = torch.zeros((case["b"], self.G), dtype=torch.int32, device=dev)
        self.logits = torch.zeros((case["b"], self.G, case["vocab"]), device=dev) if case["logits"] else None
        self.state = self.make_state() if case["call"] == "step" else None

    def make_state(self):
        c = self.case
        return bd.State(self.model, self.prompts, self.G, TAU, c["nb"], c["B"])

    def __del__(self):
        self.state = None          # before the model


def prepare(case, seed):
    return _Held(case, seed)


def run(state):
    h = state
    if h.state is not None:
        h.state.reset()
        h.state.step(h.conf, h.tok, h.logits)
        h.state.commit()
    else:
        st = h.make_state()
        st.step(h.conf, h.tok, h.logits)
        st.commit()
        st.close()
    return {"conf": h.conf, "tok": h.tok, "logits": h.logits} if h.logits is not None else {"conf": h.conf, "tok": h.tok}


# ---------------------------------------------------------------- work and tolerances
def work(case):
    """Weights, K/V of the prefix (a hi/lo pair of bf16, or fp32: 4 bytes a value) and the outputs once; one product
    per multiply-add, visible query-key pairs only.  A prefill has to carry the prompt through all layers but the
    last, and through the last one's K/V projection."""
    s, b, P, B, nb, L, V = SHAPES[case["shape"]], case["b"], case["P"], case["B"], case["nb"], case["layers"], case["vocab"]
    d, q, kv, hd = s["d"], s["H"] * s["hd"], s["Hkv"] * s["hd"], s["hd"]
    wb = {"f32": 4, "bf16": 2, "fp8": 1, "mxfp4": 0.5 + 1 / 32}[case["wq"]]
    hb = 4 if case["wq"] == "f32" else 2
    rows = b * nb * B

    def pairs(first, n):        # visible pairs of n blocks from block `first` on, per head
        return b * B * B * sum(first + i + 1 for i in range(n))

    attn_w = (q + 2 * kv) * d + d * q
    if s["E"]:
        Fs = s["ns"] * s["Fe"]
        per_row = attn_w + 3 * d * (s["k"] * s["Fe"] + Fs) + s["E"] * d
        busy = min(s["E"], rows * s["k"])
        layer_bytes = (attn_w + 3 * d * (busy * s["Fe"] + Fs)) * wb + 4 * s["E"] * d
    else:
        per_row = attn_w + 3 * d * s["F"]
        layer_bytes = per_row * wb
    flops = 2.0 * rows * (L * per_row + V * d) + 4.0 * hd * s["H"] * L * pairs(P // B, nb)
    byts = L * layer_bytes + V * d * hb + rows * (d * hb + 8) + L * b * (P + 2 * nb * B) * 2 * kv * 4
    if case["logits"]:
        byts += 4.0 * rows * V
    if case["call"] == "prefill":
        flops += 2.0 * b * P * ((L - 1) * per_row + 2 * kv * d) + 4.0 * hd * s["H"] * (L - 1) * pairs(0, P // B)
        byts += b * P * (d * hb + L * 2 * kv * 4 + 4)
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """About four times what the path is off the 64-bit forward by: operands of 16 significant bits and fp32 sums
    (measured 1e-5 in the logits and 3e-5 in the confidences of one layer, 3e-5 and 1.2e-4 after 24), fp32 models
    24 bits (measured 9e-7).  Tokens may differ where two logits tie within that.  In an MoE layer a row whose 8th
    and 9th router logits tie within rounding takes another expert and is then off as a whole (one row of a few
    hundred by a third of its size, 1e-2 over all)."""
    if case["wq"] == "f32":
        return {"rel": 4e-6, "max": 2e-4, "differ": 5e-3}
    if case["shape"] == "moe":
        return {"rel": 2e-2, "max": 0.9, "differ": 5e-3}
    return {"rel": 5e-4, "max": 2e-2, "differ": 5e-3}


# ---------------------------------------------------------------- the same in 64 bits
def _dequantized(w, wq):
    """A weight as the format holds it: fp8 E4M3 with a power-of-two scale per row, MXFP4 with one per 32 of a row."""
    w = w.double()
    if wq == "fp8":
        amax = w.abs().amax(-1, keepdim=True)
        m, e = torch.frexp(amax)                       # amax = m 2^e; 448 = 0.875 2^9
        s = torch.exp2((e - 9 + (m > 0.875)).double())
        s = torch.where(amax > 0, s, torch.ones_like(s))
        return (w / s).float().to(torch.float8_e4m3fn).double() * s
    if wq == "mxfp4":
        v = w.reshape(*w.shape[:-1], -1, 32)
        _, e = torch.frexp(v.abs().amax(-1, keepdim=True))
        s = torch.exp2((e - 3).double())
        a = (v / s).abs()
        step = torch.where(a >= 4, 2.0, torch.where(a >= 2, 1.0, 0.5)).double()
        r = torch.clamp(torch.round(a / step) * step, max=6.0)
        return (torch.sign(v) * r * s).reshape(w.shape)
    return w


def exact(case, seed):
    s, b, P, B, nb, L, V = SHAPES[case["shape"]], case["b"], case["P"], case["B"], case["nb"], case["layers"], case["vocab"]
    d, H, Hkv, hd = s["d"], s["H"], s["Hkv"], s["hd"]
    W = nb * B
    T = P + W
    specs = _tensors(case)

    def weight(i):
        return _draw_weight(case, seed, i, *specs[i])

    def layer_weight(i):
        return _dequantized(weight(i), case["wq"])

    tokens = torch.full((b, T), V - 1, dtype=torch.long, device="cuda")
    tokens[:, :P] = _prompts(case, seed).long()
    x = weight(0)[tokens].double()                     # [b, T, d]
    pos = torch.arange(T, device="cuda")
    ang = pos.double()[:, None] * THETA ** (-2.0 * torch.arange(hd // 2, device="cuda").double() / hd)
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]

    def norm(v, g):
        return v / torch.sqrt(v.square().mean(-1, keepdim=True) + EPS) * g.double()

    def rope(v):                                       # [b, t, heads, hd], the last t positions
        c, n = cos[-v.shape[1]:], sin[-v.shape[1]:]
        v1, v2 = v[..., :hd // 2], v[..., hd // 2:]
        return torch.cat([v1 * c - v2 * n, v2 * c + v1 * n], -1)

    def mlp(v, gate, up, down):
        g = v @ gate.T
        return (g / (1 + torch.exp(-g)) * (v @ up.T)) @ down.T

    at = 1
    for layer in range(L):
        first = P if layer == L - 1 else 0             # the last layer's outputs are read in the window only
        h = norm(x, weight(at))
        wqkv = layer_weight(at + 1)
        qr = H * hd
        k = rope((h @ wqkv[qr:qr + Hkv * hd].T).view(b, T, Hkv, hd))
        v = (h @ wqkv[qr + Hkv * hd:].T).view(b, T, Hkv, hd)
        q = rope((h[:, first:] @ wqkv[:qr].T).view(b, T - first, H, hd))
        o = torch.empty((b, T - first, H, hd), dtype=torch.float64, device="cuda")
        step = max(1, min(T, (1 << 27) // (T * H)))    # query rows at a time
        for i in range(b):
            kt = k[i].permute(1, 2, 0).repeat_interleave(H // Hkv, 0).contiguous()      # [H, hd, T]
            vt = v[i].transpose(0, 1).repeat_interleave(H // Hkv, 0).contiguous()       # [H, T, hd]
            for r in range(0, T - first, step):
                qi = q[i, r:r + step].transpose(0, 1).contiguous()
                z = torch.bmm(qi, kt) / math.sqrt(hd)
                seen = pos[None, :] // B <= (pos[first + r:first + r + qi.shape[1]] // B)[:, None]
                z.masked_fill_(~seen, -math.inf)
                o[i, r:r + step] = torch.bmm(torch.softmax(z, -1), vt).transpose(0, 1)
        x = x[:, first:] + o.reshape(b, T - first, H * hd) @ layer_weight(at + 2).T
        f = norm(x, weight(at + 3)).reshape(-1, d)
        if not s["E"]:
            y = torch.empty_like(f)
            gate, up, down = (layer_weight(at + 4 + j) for j in range(3))
            for r in range(0, f.shape[0], 8192):
                y[r:r + 8192] = mlp(f[r:r + 8192], gate, up, down)
            at += 7
        else:
            p = torch.softmax(f @ weight(at + 4).double().T, -1)
            pk, ek = torch.topk(p, s["k"], -1)
            pk = pk / pk.sum(-1, keepdim=True)
            gate, up, down = (layer_weight(at + 5 + j) for j in range(3))
            y = mlp(f, *(layer_weight(at + 8 + j) for j in range(3)))
            for e in range(s["E"]):
                row, slot = torch.where(ek == e)
                if row.numel():
                    y.index_add_(0, row, mlp(f[row], gate[e], up[e], down[e]) * pk[row, slot][:, None])
            at += 11
        x = x + y.view(x.shape)
    h = norm(x, weight(at)).reshape(-1, d)             # [b W, d]
    head = weight(at + 1).double()
    conf, tok, logits = [], [], []
    for r in range(0, h.shape[0], 512):
        z = SCALE * (h[r:r + 512] @ head.T)
        z[:, V - 1] = -math.inf
        m, a = z.max(-1)
        conf.append(1 / torch.exp(z - m[:, None]).sum(-1))
        tok.append(a)
        if case["logits"]:
            logits.append(z)
    out = {"conf": torch.cat(conf).view(b, W), "tok": torch.cat(tok).view(b, W).int()}
    if case["logits"]:
        out["logits"] = torch.cat(logits).view(b, W, V)
    return out
