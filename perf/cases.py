"""Performance cases of the block-decode library: what a decoding program calls, over its range of sizes.

A case is one pass through a public entry point of the runtime, with its logits.  Most cases run a stack of
a few decoder layers: four of the 8B stack's 36 layers (or the 14B stack's 40) with the same share of the
vocabulary behind them, so that layers and LM head weigh as they do in the whole model.  Weights are
N(0, 0.02) bf16, RMSNorm gains 1 + 0.1 z, cached keys and values N(0, 1) bf16, tokens uniform.

Case keys: op (the entry point), shape, layers, vocab, batch, k (block rows per sequence; the chain length
for quad), lo and hi (the sequences' cached prefix lengths are uniform in [lo, hi]), bidir (draft passes:
first row that sees the whole block), lam (quad: the verifier's mixture), rank (LoRA adapter, 0: none).
"""
import ctypes
import math
import random
from dataclasses import replace

import torch

from paper_2607_05722_amd import _lib as C
from paper_2607_05722_amd import runtime as R
from synth.workloads import SHAPE_14B, SHAPE_8B, SHAPE_TINY

SHAPES = {"tiny": SHAPE_TINY, "8b": SHAPE_8B, "14b": SHAPE_14B}
LORA_ALPHA = 512.0
THRESHOLD = 0.9


def _case(name, op, shape, layers, vocab, batch, k, lo, hi, bidir=0, lam=1.0, rank=0):
    c = {"op": op, "shape": shape, "layers": layers, "vocab": vocab, "batch": batch, "k": k, "lo": lo, "hi": hi,
         "bidir": bidir, "lam": lam, "rank": rank}
    return dict({"name": name}, **c) if name else c


def listed():
    return [
        # a small model in a test bench or a toy program: launches and latency are all there is
        _case("tiny_verify_k8", "verify_block", "tiny", 2, 1024, 1, 8, 128, 128),
        # plain autoregressive decoding of one sequence (block size 1)
        _case("ar_b1", "verify_accept", "8b", 4, 16877, 1, 1, 1500, 1500),
        # a short block: one layer and the whole LM head
        _case("layer_verify_k8", "verify_block", "8b", 1, 151936, 1, 8, 2048, 2048),
        # the draft pass of linear self-speculation on the whole 8B stack, the headline configuration
        _case("draft_full_k16", "draft", "8b", 36, 151936, 1, 16, 4096, 4096),
        # the same draft pass with the LoRA-enhanced drafter (rank 128) attached
        _case("lora_draft_k16", "draft", "8b", 4, 16877, 1, 16, 2048, 2048, rank=128),
        # block length 32, the method's main one
        _case("draft_k32", "draft", "8b", 4, 16877, 1, 32, 4096, 4096, bidir=1),
        # quadratic self-speculation with the ensemble verifier: 56 block rows
        _case("quad_k7", "quad", "8b", 4, 16877, 1, 7, 4096, 4096, lam=0.5),
        # a prompt being prefilled in chunks of 64 tokens, at an odd offset
        _case("prefill_k64", "verify_block", "8b", 4, 16877, 1, 64, 2997, 2997),
        # autoregressive decoding at high concurrency, every sequence at its own length
        _case("ar_b100", "verify_accept", "8b", 4, 16877, 100, 1, 64, 4096),
        # a denoising step of several sequences
        _case("denoise_b5_k24", "denoise", "8b", 4, 16877, 5, 24, 256, 3000),
        # the verify pass of a batch of 32 ragged sequences
        _case("verify_b32_k16", "verify_accept", "8b", 4, 16877, 32, 16, 512, 8192),
        # the draft pass of eight long sequences on the wider model
        _case("draft_14b_b8_k32", "draft", "14b", 4, 15193, 8, 32, 16384, 16384),
    ]


def _rows(case):
    return case["k"] * (case["k"] + 1) if case["op"] == "quad" else case["k"]


def _seconds(case):
    """A rough cost, used to keep the drawn cases within the listed ones."""
    w = work(case)
    return w["bytes"] / 5e12 + w["flops"] / 3e14 + 1e-5 * case["layers"]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    most = max(_seconds(c) for c in listed())
    while True:
        shape = rng.choice(["tiny", "8b", "8b", "8b", "14b"])
        op = rng.choice(["verify_block", "verify_accept", "draft", "draft", "denoise", "quad"])
        s = SHAPES[shape]
        group = s.n_q_heads // s.n_kv_heads
        batch = 1 if rng.random() < 0.4 else _log_int(rng, 2, 100)
        if op == "quad":
            k = rng.randint(2, 6 if group > 4 else 7)
        elif op == "verify_accept" and rng.random() < 0.4:
            k = 1
        else:
            k = _log_int(rng, 2, min(64, 256 // group))
        layers = 2 if shape == "tiny" else rng.randint(1, 4)
        vocab = 1024 if shape == "tiny" else _log_int(rng, 4000, 40000)
        hi = _log_int(rng, 32, 2048 if shape == "tiny" else 16384)
        lo = hi if rng.random() < 0.5 else _log_int(rng, 16, hi)
        bidir = rng.choice([0, 1]) if op in ("draft", "denoise") else 0
        lam = rng.choice([0.0, 0.5, 1.0]) if op == "quad" else 1.0
        rank = 128 if op == "draft" and shape != "tiny" and rng.random() < 0.25 else 0
        c = _case(None, op, shape, layers, vocab, batch, k, lo, hi, bidir, lam, rank)
        if batch * _rows(c) <= 1024 and _seconds(c) <= most:
            return c


# ------------------------------------------------------------------------------------------ seeded inputs
def _shape(case):
    return replace(SHAPES[case["shape"]], n_layers=case["layers"], vocab=case["vocab"], lora_rank=case["rank"],
                   lora_alpha=LORA_ALPHA if case["rank"] else 0.0)


def _rand(seed, tag, index=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + tag * 8191 + index * 131) & 0x7FFFFFFF)
    return g


def _normal(seed, tag, index, size, std):
    return torch.randn(size, generator=_rand(seed, tag, index), device="cuda", dtype=torch.bfloat16).mul_(std)


def _gain(seed, tag, index, n):
    return torch.randn(n, generator=_rand(seed, tag, index), device="cuda").mul_(0.1).add_(1.0).to(torch.bfloat16)


def _layer(s, seed, l):
    """Row-major [out][in] weights of layer l."""
    n = lambda i, rows, cols: _normal(seed, 10 + i, l, (rows, cols), 0.02)   # noqa: E731
    w = {"attn_norm": _gain(seed, 1, l, s.hidden), "ffn_norm": _gain(seed, 2, l, s.hidden),
         "wq": n(0, s.q_dim, s.hidden), "wk": n(1, s.kv_dim, s.hidden), "wv": n(2, s.kv_dim, s.hidden),
         "wo": n(3, s.hidden, s.q_dim), "w_gate": n(4, s.ffn, s.hidden), "w_up": n(5, s.ffn, s.hidden),
         "w_down": n(6, s.hidden, s.ffn)}
    if s.lora_rank:
        w["lora_a"], w["lora_b"] = n(7, s.lora_rank, s.q_dim), n(8, s.hidden, s.lora_rank)
    return w


def _embed(s, seed):
    return _normal(seed, 3, 0, (s.vocab, s.hidden), 0.02)


def _lm_head(s, seed):
    return _normal(seed, 4, 0, (s.vocab, s.hidden), 0.02)


def _prefix(s, case, seed, l, which, max_len):
    """Cached keys (which 0) or values (1) of layer l: [batch][kv_heads][max_len][head_dim]."""
    return _normal(seed, 20 + which, l, (case["batch"], s.n_kv_heads, max_len, s.head_dim), 1.0)


def _host(case, seed):
    """Prefix lengths and tokens; the tokens never are the mask token (vocab - 1)."""
    rng = random.Random(seed * 7919 + 5)
    lens = [rng.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]
    toks = [[rng.randrange(case["vocab"] - 1) for _ in range(_rows(case))] for _ in range(case["batch"])]
    if case["op"] == "denoise":   # part of the block was filled in by earlier steps
        for row in toks:
            for j in range(1, len(row)):
                if rng.random() < 0.6:
                    row[j] = case["vocab"] - 1
            row[-1] = case["vocab"] - 1
    return lens, toks


def _capacity(case):
    return -(-(case["hi"] + 2 * _rows(case)) // 64) * 64


class Model:
    """A model handle over weights that are made and packed on the GPU."""

    def __init__(self, s, seed):
        lib = C.load()
        self.lib, self.shape, self.device, self.cfg = lib, s, torch.device("cuda"), R.make_config(s)
        self.keep, cfg, st = [], ctypes.byref(self.cfg), R.stream_handle()
        layers = (C.LayerWeights * s.n_layers)()

        def packed(kind, out_dim, in_dim, *sources):
            dst = torch.empty(lib.nld_packed_bytes(kind, cfg, out_dim, in_dim), dtype=torch.uint8, device="cuda")
            self.keep.append(dst)
            ptrs = [t.data_ptr() for t in sources]
            if kind == C.NLD_PACK_LINEAR:
                C.check(lib.nld_pack_linear(ptrs[0], out_dim, in_dim, dst.data_ptr(), st))
            elif kind == C.NLD_PACK_QKV:
                C.check(lib.nld_pack_qkv(cfg, *ptrs, dst.data_ptr(), st))
            else:
                C.check(lib.nld_pack_gate_up(cfg, *ptrs, dst.data_ptr(), st))
            return dst.data_ptr()

        h, qd, kvd = s.hidden, s.q_dim, s.kv_dim
        for l in range(s.n_layers):
            w = _layer(s, seed, l)
            self.keep += [w["attn_norm"], w["ffn_norm"]]
            la = packed(C.NLD_PACK_LINEAR, s.lora_rank, qd, w["lora_a"]) if s.lora_rank else 0
            lb = packed(C.NLD_PACK_LINEAR, h, s.lora_rank, w["lora_b"]) if s.lora_rank else 0
            layers[l] = C.LayerWeights(
                w["attn_norm"].data_ptr(), packed(C.NLD_PACK_QKV, qd + 2 * kvd, h, w["wq"], w["wk"], w["wv"]),
                packed(C.NLD_PACK_LINEAR, h, qd, w["wo"]), w["ffn_norm"].data_ptr(),
                packed(C.NLD_PACK_GATE_UP, s.ffn, h, w["w_gate"], w["w_up"]),
                packed(C.NLD_PACK_LINEAR, h, s.ffn, w["w_down"]), la, lb)
        self.embed, self.final_norm = _embed(s, seed), _gain(seed, 5, 0, h)
        lm = packed(C.NLD_PACK_LINEAR, s.vocab, h, _lm_head(s, seed))
        self.layers = layers
        self.weights = C.Weights(self.embed.data_ptr(), self.final_norm.data_ptr(), lm, layers)
        self.handle = ctypes.c_void_p()
        C.check(lib.nld_model_create(cfg, ctypes.byref(self.weights), ctypes.byref(self.handle)))

    def __del__(self):
        if getattr(self, "handle", None):
            self.lib.nld_model_destroy(self.handle)


class State:
    pass


def prepare(case, seed):
    st, s = State(), _shape(case)
    lens, toks = _host(case, seed)
    st.case, st.model = case, Model(s, seed)
    max_len = _capacity(case)
    st.cache = R.DeviceCache(s, case["batch"], max_len)
    for l in range(s.n_layers):
        st.cache.k[l] = _prefix(s, case, seed, l, 0, max_len).view(torch.int16)
        v = _prefix(s, case, seed, l, 1, max_len).view(torch.int16)
        st.cache.v[l] = v.view(case["batch"], s.n_kv_heads, max_len // 64, 64, s.head_dim).transpose(-1, -2)
    st.keys, st.values = st.cache.k.view(torch.bfloat16), st.cache.v.view(torch.bfloat16)
    st.lens = torch.tensor(lens, dtype=torch.int32, device="cuda")
    st.cache.lengths.copy_(st.lens)
    st.tokens = torch.tensor(toks, dtype=torch.int32, device="cuda")
    st.block = st.tokens.clone()
    st.anchor = st.tokens[:, 0].contiguous()
    st.drafts = st.tokens[:, 1:case["k"]].contiguous()
    kind = R.QuadWorkspace if case["op"] == "quad" else R.Workspace
    st.ws = kind(st.model, case["batch"], case["k"], max_len)
    return st


def run(st):
    c = st.case
    if c["op"] == "verify_block":
        logits, argmax = R.block_forward(st.model, st.cache, st.ws, st.tokens, R.VERIFY)
        return {"logits": logits, "argmax": argmax, "keys": st.keys, "values": st.values}
    if c["op"] == "draft":
        drafts, logits = R.draft(st.model, st.cache, st.ws, st.anchor, c["k"], bidir_from=c["bidir"], want_logits=True)
        return {"logits": logits, "drafts": drafts}
    if c["op"] == "denoise":
        st.block.copy_(st.tokens)   # the step fills the block in place
        o = R.denoise_step(st.model, st.cache, st.ws, st.block, THRESHOLD, bidir_from=c["bidir"], want_logits=True)
        return {"logits": o["logits"], "confidence": o["confidence"], "block": st.block, "n_masked": o["n_masked"]}
    st.cache.lengths.copy_(st.lens)   # the step advances them
    if c["op"] == "verify_accept":
        o = R.verify_accept(st.model, st.cache, st.ws, st.anchor, st.drafts if c["k"] > 1 else None, c["k"],
                            want_logits=True)
    else:
        o = R.quad_step(st.model, st.cache, st.ws, st.anchor, st.drafts, c["k"], lam=c["lam"], want_logits=True)
    return dict(o, lengths=st.cache.lengths, keys=st.keys, values=st.values)


# ------------------------------------------------------------------------------------------ what a pass needs
def work(case):
    """Weights and cached keys and values once in bf16, the block's embedding rows, logits out in f32, the
    block's keys and values written where the pass writes the cache; 2 flops per weight and row."""
    s, rows = _shape(case), _rows(case)
    m = case["batch"] * rows
    keys = case["batch"] * (case["lo"] + case["hi"]) / 2
    layer = s.hidden * (s.q_dim + 2 * s.kv_dim) + s.q_dim * s.hidden + 3 * s.hidden * s.ffn
    layer += s.lora_rank * (s.q_dim + s.hidden)
    weights = s.n_layers * layer + s.vocab * s.hidden
    written = 0 if case["op"] in ("draft", "denoise") else case["batch"] * case["k"]
    byts = 2 * weights + 4 * s.n_layers * (keys + written) * s.kv_dim + 2 * m * s.hidden + 4 * m * s.vocab
    flops = 2 * m * weights + 4 * s.q_dim * s.n_layers * rows * (keys + m)
    return {"bytes": int(byts), "flops": int(flops)}


def tolerance(case):
    """Activations carry about 16 bits (a bf16 value and its bf16 remainder) and sums are in f32.  Against 64
    bits, and between launch plans that sum in other orders, logits of one to four layers are 0.6e-5 to 1.6e-5
    apart (largest single one 9e-5 of the root mean square) and those of 36 layers 4e-5 (2.5e-4).  A verify
    pass also returns the cache in bf16, where such a difference turns a rounding now and then: one step of
    2^-8 in a value, up to 1e-4 over a short cache.  Whole values only differ where two logits tie."""
    deep = case["layers"] > 4
    if case["op"] in ("draft", "denoise"):
        return {"rel": 1.6e-4 if deep else 6e-5, "max": 1e-3 if deep else 4e-4, "differ": 0.01}
    return {"rel": 4e-4, "max": 8e-3, "differ": 0.01}


# ------------------------------------------------------------------------------------------ 64-bit reference
def _offsets_and_mask(case):
    """Position of each block row after the prefix, and which block rows it sees."""
    k, n = case["k"], _rows(case)
    if case["op"] != "quad":
        see = torch.ones(n, n, dtype=torch.bool).tril()
        if case["op"] in ("draft", "denoise"):
            see[case["bidir"]:] = True
        return torch.arange(n), see
    off = list(range(k)) + [c + r for c in range(k) for r in range(1, k + 1)]
    see = torch.zeros(n, n, dtype=torch.bool)
    for c in range(k):
        mine = slice(k + c * k, k + (c + 1) * k)
        see[c, :c + 1] = True
        see[mine, :c + 1] = True
        see[mine, mine] = True
    return torch.tensor(off), see


def _rope(x, pos, base):
    """x: [heads][rows][head_dim]; rotate-half pairs (i, i + head_dim/2)."""
    half = x.shape[-1] // 2
    freq = base ** (-torch.arange(half, dtype=torch.float64, device=x.device) * 2 / x.shape[-1])
    ang = pos.double()[:, None] * freq
    c, s, a, b = ang.cos(), ang.sin(), x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _norm(x, gain, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * gain.double()


def _attend(q, keys, values, see):
    """q [kv_heads][group * rows][d], keys and values [kv_heads][n][d], see [rows][n]."""
    z = torch.matmul(q, keys.transpose(-1, -2).contiguous()) / math.sqrt(q.shape[-1])
    z.masked_fill_(~see.repeat(q.shape[1] // see.shape[0], 1), -math.inf)
    return torch.matmul(torch.softmax(z, -1), values)


def exact(case, seed):
    s, n, b = _shape(case), _rows(case), case["batch"]
    lens, toks = _host(case, seed)
    mask_id = s.vocab - 1
    ids = [row if case["op"] in ("verify_block", "verify_accept", "denoise")
           else [t if 0 < j < case["k"] and case["op"] == "quad" or j == 0 else mask_id for j, t in enumerate(row)]
           for row in toks]
    off, see = _offsets_and_mask(case)
    off, see = off.cuda(), see.cuda()
    draft = case["op"] in ("draft", "denoise")
    x = _embed(s, seed)[torch.tensor(ids, device="cuda").reshape(-1)].double()
    group, d, nkv = s.n_q_heads // s.n_kv_heads, s.head_dim, s.n_kv_heads
    for l in range(s.n_layers):
        w = _layer(s, seed, l)
        h = _norm(x, w["attn_norm"], s.rms_eps)
        q, k, v = (h @ w[i].double().t() for i in ("wq", "wk", "wv"))
        pk, pv = (_prefix(s, case, seed, l, i, _capacity(case)) for i in (0, 1))
        o = torch.empty_like(q)
        for i in range(b):
            at = slice(i * n, (i + 1) * n)
            heads = lambda t: t[at].view(n, -1, d).transpose(0, 1)   # noqa: E731
            pos = lens[i] + off
            qi = _rope(heads(q), pos, s.rope_base).reshape(nkv, group * n, d)
            ki = torch.cat([pk[i, :, :lens[i]].double(), _rope(heads(k), pos, s.rope_base)], 1)
            vi = torch.cat([pv[i, :, :lens[i]].double(), heads(v)], 1)
            vis = torch.cat([torch.ones(n, lens[i], dtype=torch.bool, device="cuda"), see], 1)
            o[at] = _attend(qi, ki, vi, vis).view(s.n_q_heads, n, d).transpose(0, 1).reshape(n, -1)
        x = x + o @ w["wo"].double().t()
        if draft and s.lora_rank:
            x = x + (s.lora_alpha / s.lora_rank) * (o @ w["lora_a"].double().t()) @ w["lora_b"].double().t()
        h = _norm(x, w["ffn_norm"], s.rms_eps)
        x = x + (torch.nn.functional.silu(h @ w["w_gate"].double().t()) * (h @ w["w_up"].double().t())) \
            @ w["w_down"].double().t()
    h = _norm(x, _gain(seed, 5, 0, s.hidden), s.rms_eps)
    logits = (h @ _lm_head(s, seed).double().t()).view(b, n, s.vocab)
    if case["op"] == "verify_block":
        return {"logits": logits, "argmax": None, "keys": None, "values": None}
    if case["op"] == "draft":
        return {"logits": logits, "drafts": None}
    if case["op"] == "denoise":
        p = torch.softmax(logits[..., :mask_id], -1).amax(-1)
        return {"logits": logits, "confidence": p, "block": None, "n_masked": None}
    out = {"logits": logits, "accept_len": None, "committed": None, "next_anchor": None, "lengths": None,
           "keys": None, "values": None}
    return dict(out, next_spec=None) if case["op"] == "quad" else out
