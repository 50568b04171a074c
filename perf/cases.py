"""Performance cases: what a user of the library runs, over the range of sizes they run it at.

A serving program holds a model handle, a workspace and output buffers, and per batch of token ids calls
`radix_build_index`, `radix_prefill_forward` on the maps, and (rerankers) `radix_lm_head` on the last token of
every sequence.  Evaluation of the deduplication itself, and batches known to share nothing, call
`radix_prefill_forward_nodedup`; schedulers that only want to know how much a batch shares call
`radix_build_index` alone.  Shapes are the ones of `synth.py` (tiny fp32, 0.6B, 4B and 8B), batches are the
families of the paper: one shared prefix and a suffix per candidate, an extra level of query blocks, no sharing.

Fields of a case
  op         "step" (index + deduplicated forward), "nodedup" (plain forward), "index" (maps only)
  model      shape name;  compute: operand type
  B          sequences
  prefix     tokens shared by all sequences
  groups, group_len   second level: query blocks, each shared by B / groups consecutive sequences
  suffix_lo, suffix_hi   own tokens per sequence, uniform
  positions  pass explicit position ids
  attention  "auto" or "three_kernels" (scatter, attention over all rows, gather)
  head       logits of every sequence's last token
"""
import numpy as np
import torch

from paper_2601_15013_amd import binding, synth

_SHIFT = 16     # explicit position ids start here, as behind a cached system prompt
MODELS = {m.name: m for m in (synth.TINY, synth.QWEN3_0_6B, synth.QWEN3_4B, synth.QWEN3_8B)}


def _case(op, model, B, prefix, lo, hi, *, compute=None, groups=1, group_len=0, positions=False, attention="auto",
          head=False):
    return {"op": op, "model": model, "compute": compute or binding.default_compute_dtype(MODELS[model].dtype), "B": B,
            "prefix": prefix, "groups": groups, "group_len": group_len, "suffix_lo": lo, "suffix_hi": hi,
            "positions": positions, "attention": attention, "head": head}


def listed():
    cases = {
        # the fp32 configuration at the size the repository names: a small model, latency and launches count
        "f32 tiny 8x48": _case("step", "tiny", 8, 32, 16, 16),
        # one short prompt, scored by its last token: the smallest call of the 16-bit path, bound by streaming the weights
        "0.6B one prompt": _case("step", "qwen3-0.6b", 1, 0, 21, 21, head=True),
        # an interactive query with a handful of candidates
        "0.6B 8 candidates": _case("step", "qwen3-0.6b", 8, 48, 64, 192, head=True),
        # the ordinary reranking batch (the 0.6B configuration of the repository)
        "0.6B 64 candidates": _case("step", "qwen3-0.6b", 64, 48, 64, 192, head=True),
        # bf16 operands and position ids of the caller's own, at a row of the paper's sweep
        "0.6B bf16 512/256": _case("step", "qwen3-0.6b", 32, 512, 256, 256, compute="bf16", positions=True),
        # a long shared document in front of short questions: attention over a prefix that is computed once
        "0.6B long prefix": _case("step", "qwen3-0.6b", 128, 2048, 32, 32),
        # nothing shared, long ragged prompts: the plain forward, attention at its heaviest
        "0.6B no sharing": _case("nodedup", "qwen3-0.6b", 33, 0, 1024, 2080),
        # three-level trie of the 4B configuration
        "4B query groups": _case("step", "qwen3-4b", 128, 256, 64, 192, groups=8, group_len=32),
        # the paper's own sequence of scatter, attention and gather, at a row of its sweep
        "4B 3-kernel 1024/256": _case("step", "qwen3-4b", 32, 1024, 256, 256, attention="three_kernels"),
        # a few candidates on the largest model: few rows against many weights
        "8B 4 candidates": _case("step", "qwen3-8b", 4, 64, 96, 256, head=True),
        # the largest configuration
        "8B 256 candidates": _case("step", "qwen3-8b", 256, 64, 96, 256, head=True),
        # the maps alone, at about the largest shape of the paper's index-construction benchmark
        "index 2048x512": _case("index", "qwen3-0.6b", 2048, 256, 192, 320),
    }
    return [dict(c, name=n) for n, c in cases.items()]


# ------------------------------------------------------------------------------------------ draws
def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """One more case of the ranges above; none costs more than the largest listed one."""
    while True:
        model = rng.choice(["tiny", "qwen3-0.6b", "qwen3-0.6b", "qwen3-0.6b", "qwen3-4b", "qwen3-8b"])
        m = MODELS[model]
        op = rng.choice(["step", "step", "step", "step", "step", "nodedup", "index"])
        if op == "index":
            model, m = "qwen3-0.6b", MODELS["qwen3-0.6b"]
            B, prefix, lo = _log_int(rng, 16, 2048), _log_int(rng, 1, 512), _log_int(rng, 4, 256)
        elif model == "tiny":
            B, prefix, lo = _log_int(rng, 1, 64), _log_int(rng, 1, 256), _log_int(rng, 1, 64)
        else:
            B, prefix, lo = _log_int(rng, 1, 256), _log_int(rng, 1, 2048), _log_int(rng, 1, 1024)
        hi = int(lo * rng.uniform(1.5 if op == "index" else 1.0, 3.0))
        if op == "nodedup":
            prefix = 0
        groups, group_len = 1, 0
        if op == "step" and B >= 4 and rng.random() < 0.25:
            groups, group_len = rng.choice([2, 4, 8]), _log_int(rng, 4, 64)
            B = max(groups, B // groups * groups)
        compute = "f32" if m.dtype == "f32" else ("bf16" if m is synth.QWEN3_0_6B and rng.random() < 0.25 else "f16")
        c = _case(op, model, B, prefix, lo, hi, compute=compute, groups=groups, group_len=group_len,
                  positions=rng.random() < 0.15,
                  attention="three_kernels" if op == "step" and rng.random() < 0.15 else "auto",
                  head=op == "step" and rng.random() < 0.5 and m.dtype != "f32")
        rows, total = _sizes(c)
        longest = prefix + group_len + hi
        # all sequences' own rows stay within the largest batches of the repository, and the work within that of "8B 256 candidates"
        if longest + _SHIFT >= m.max_pos or total > 266240 and op != "index" or total > 2 << 20:
            continue
        if model != "tiny" and op != "index" and work(c)["flops"] > 0.5 * _LARGEST_FLOPS:
            continue
        return c


def _sizes(c):
    """Expected unique rows and all rows."""
    s = (c["suffix_lo"] + c["suffix_hi"]) / 2
    return (c["prefix"] + c["groups"] * c["group_len"] + c["B"] * s,
            c["B"] * (c["prefix"] + c["group_len"] + s))


# ------------------------------------------------------------------------------------------ inputs
def _batch(c, seed):
    """Token ids, and which sequence has which length, from the seed; the lengths and the amount of sharing are the
    case's own (siblings differ in their first token), so that the shapes of the outputs are."""
    rng = np.random.default_rng([seed, 1])
    v = MODELS[c["model"]].vocab
    prefix = rng.integers(0, v, size=c["prefix"], dtype=np.int32)
    blocks = rng.integers(0, v, size=(c["groups"], c["group_len"]), dtype=np.int32)
    if c["group_len"]:
        blocks[:, 0] = rng.choice(v, size=c["groups"], replace=False)
    lens = np.random.default_rng([c["B"], c["suffix_lo"], c["suffix_hi"]]).integers(c["suffix_lo"], c["suffix_hi"] + 1, size=c["B"])
    lens = rng.permutation(lens)
    suffixes = [rng.integers(0, v, size=int(n), dtype=np.int32) for n in lens]
    for s, first in zip(suffixes, rng.choice(v, size=c["B"], replace=False)):
        s[0] = first
    seqs = [np.concatenate([prefix, blocks[b * c["groups"] // c["B"]], s]) for b, s in enumerate(suffixes)]
    cu = np.zeros(c["B"] + 1, dtype=np.int32)
    cu[1:] = np.cumsum([len(s) for s in seqs])
    tok = np.concatenate(seqs)
    pos = np.concatenate([np.arange(len(s), dtype=np.int32) for s in seqs]) + _SHIFT if c["positions"] else None
    return tok, pos, cu, max(len(s) for s in seqs)


def _weights(c, seed):
    """Random-init weights of the shape, drawn on the GPU."""
    m = MODELS[c["model"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = torch.float32 if m.dtype == "f32" else torch.bfloat16

    def mat(*shape):
        return torch.empty(shape, dtype=dt, device="cuda").normal_(0.0, 0.02, generator=gen)

    def gain(n):
        return torch.empty(n, dtype=torch.float32, device="cuda").normal_(1.0, 0.02, generator=gen)

    layers = [{"g1": gain(m.d), "wq": mat(m.dq, m.d), "wk": mat(m.dkv, m.d), "wv": mat(m.dkv, m.d),
               "gq": gain(m.head_dim), "gk": gain(m.head_dim), "wo": mat(m.d, m.dq), "g2": gain(m.d),
               "wg": mat(m.d_int, m.d), "wu": mat(m.d_int, m.d), "wd": mat(m.d, m.d_int)} for _ in range(m.n_layers)]
    return layers, mat(m.vocab, m.d), gain(m.d)


def _model(c, seed):
    """The weights handed to the library, which keeps its own copy."""
    layers, embed, gf = _weights(c, seed)
    return binding.radix_model_create(MODELS[c["model"]], embed, gf, layers, compute_dtype=c["compute"],
                                      lm_head_mode=1 if c["head"] else 0)


def prepare(case, seed):
    c = case
    tok, pos, cu, max_len = _batch(c, seed)
    N, B = len(tok), c["B"]
    s = {"case": c, "tok": torch.from_numpy(tok).cuda(), "cu": torch.from_numpy(cu).cuda(), "max_len": max_len,
         "pos": None if pos is None else torch.from_numpy(pos).cuda()}
    if c["op"] != "nodedup":
        s["maps"] = (torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty(N, dtype=torch.int32, device="cuda"),
                     torch.empty(1, dtype=torch.int32, device="cuda"))
    if c["op"] == "index":
        s["ws"] = binding.alloc_workspace(binding.radix_index_workspace_bytes(B))
        return s
    s["model"] = model = _model(c, seed)
    need = binding.radix_workspace_bytes(model, N, B)
    if c["head"]:
        need = max(need, binding.radix_lm_head_workspace_bytes(model, B))
        s["last"] = s["cu"][1:] - 1
        s["logits"] = torch.empty((B, model.cfg.vocab), dtype=torch.float32, device="cuda")
    s["ws"] = binding.alloc_workspace(need)
    s["out"] = torch.empty((N, model.cfg.d), dtype=torch.float32, device="cuda")
    return s


def run(state):
    s = state
    c = s["case"]
    if c["op"] == "nodedup":
        return binding.radix_prefill_forward_nodedup(s["model"], s["tok"], s["pos"], s["cu"], s["max_len"], s["ws"], out=s["out"])
    I_s, I_g, n_dev, n = binding.radix_build_index(s["tok"], s["pos"], s["cu"], s["ws"], *s["maps"])
    got = {"I_scatter": I_s, "I_gather": I_g[:n], "n": n}
    if c["op"] == "index":
        return got
    got["hidden"] = binding.radix_prefill_forward(
        s["model"], s["tok"], s["pos"], s["cu"], s["max_len"], I_s, I_g, n, s["ws"], out=s["out"],
        fused_attention=False if c["attention"] == "three_kernels" else None)
    if c["head"]:
        got["logits"] = binding.radix_lm_head(s["model"], got["hidden"], s["last"], s["ws"], out=s["logits"])
    return got


# ------------------------------------------------------------------------------------------ the same in 64 bits
def _norm(x, g, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def exact(case, seed):
    """The hidden states (and logits) of `run` in plain torch and float64.  Every distinct (prefix, block, suffix)
    segment of the batch is a run of rows that is computed once, behind the segments it continues; how the segments
    lie in the batch is known from the way it was made."""
    c = case
    if c["op"] == "index" or work(c)["flops"] > 2e14:       # whole numbers; over about 20 seconds
        return None
    m = MODELS[c["model"]]
    tok, pos, cu, _ = _batch(c, seed)
    B, P, G = c["B"], c["prefix"], c["group_len"]
    if pos is None:
        pos = np.concatenate([np.arange(n) for n in np.diff(cu)])
    take, segments, where = [], [], np.empty(len(tok), dtype=np.int64)     # segment: (first row, rows, rows in front of it)
    n_rows = 0
    for b in range(B):
        block = b * c["groups"] // B
        new_block = b == 0 or block != (b - 1) * c["groups"] // B
        behind, at = [], cu[b]
        for length, fresh, known in ((P, b == 0, "prefix"), (G, new_block, "block"), (cu[b + 1] - cu[b] - P - G, True, "")):
            if fresh:
                row = n_rows
                take.append(np.arange(at, at + length))
                segments.append((row, int(length), list(behind)))
                n_rows += int(length)
                if known == "prefix":
                    prefix_row = row
                elif known == "block":
                    block_row = row
            else:
                row = prefix_row if known == "prefix" else block_row
            where[at:at + length] = row + np.arange(length)
            behind.append((row, int(length)))
            at += length
    take = torch.from_numpy(np.concatenate(take)).cuda()
    ids, at = torch.from_numpy(tok).cuda().long()[take], torch.from_numpy(pos).cuda()[take].double()
    layers, embed, gf = _weights(c, seed)
    half, hd, rep = m.head_dim // 2, m.head_dim, m.n_q_heads // m.n_kv_heads
    angle = at[:, None] * float(m.rope_base) ** (-2.0 * torch.arange(half, device="cuda", dtype=torch.float64) / hd)
    cos, sin = angle.cos()[:, None], angle.sin()[:, None]

    def rotate(x):
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    h = embed[ids].double()
    for w in layers:
        a = _norm(h, w["g1"], m.eps)
        q, k, v = ((a @ w[n].double().T).view(n_rows, -1, hd) for n in ("wq", "wk", "wv"))
        if m.qk_norm:
            q, k = _norm(q, w["gq"], m.eps), _norm(k, w["gk"], m.eps)
        q, k = rotate(q), rotate(k)
        o = torch.empty_like(q)
        for row, n, behind in segments:
            if n == 0:
                continue
            spans = behind + [(row, n)]
            kk, vv = (torch.cat([x[r:r + t] for r, t in spans]).transpose(0, 1) for x in (k, v))       # [kv heads, keys, hd]
            qq = q[row:row + n].transpose(0, 1).reshape(m.n_kv_heads, rep * n, hd)
            s = torch.bmm(qq, kk.transpose(1, 2).contiguous()) / hd ** 0.5
            s = s.view(m.n_q_heads, n, -1)
            keys = s.shape[-1]
            s.masked_fill_(torch.ones(n, keys, dtype=torch.bool, device="cuda").triu(keys - n + 1), float("-inf"))
            p = torch.softmax(s, -1).view(m.n_kv_heads, rep * n, keys)
            o[row:row + n] = torch.bmm(p, vv.contiguous()).view(m.n_q_heads, n, hd).transpose(0, 1)
        h = h + o.reshape(n_rows, -1) @ w["wo"].double().T
        a = _norm(h, w["g2"], m.eps)
        gate = a @ w["wg"].double().T
        h = h + (gate * torch.sigmoid(gate) * (a @ w["wu"].double().T)) @ w["wd"].double().T
    hidden = _norm(h, gf, m.eps)[torch.from_numpy(where).cuda()]
    if c["op"] == "nodedup":
        return hidden
    got = {"I_scatter": None, "I_gather": None, "n": None, "hidden": hidden}
    if c["head"]:
        last = hidden[torch.from_numpy(cu[1:] - 1).cuda().long()]
        got["logits"] = torch.cat([last @ part.double().T for part in embed.split(16384)], -1)
    return got


# ------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c = case
    m = MODELS[c["model"]]
    rows, total = _sizes(c)
    index_bytes = total * (4 * (2 if c["positions"] else 1) + 4) + rows * 4
    if c["op"] == "index":
        return {"bytes": index_bytes, "flops": 0}
    s = (c["suffix_lo"] + c["suffix_hi"]) / 2
    if c["op"] == "nodedup":
        rows, index_bytes = total, total * 4
    # keys that the queries of one walk of the trie see: query at depth p attends p + 1 of them
    span = lambda a, n: n * a + n * (n + 1) / 2  # noqa: E731
    if c["op"] == "nodedup" or c["attention"] == "three_kernels":      # attention over every row
        pairs = c["B"] * span(0, c["prefix"] + c["group_len"] + s)
    else:
        pairs = (span(0, c["prefix"]) + c["groups"] * span(c["prefix"], c["group_len"]) +
                 c["B"] * span(c["prefix"] + c["group_len"], s))
    es = 4 if m.dtype == "f32" else 2
    per_layer = m.d * (m.dq + 2 * m.dkv) + m.dq * m.d + 3 * m.d * m.d_int
    flops = m.n_layers * (2.0 * rows * per_layer + 4.0 * m.dq * pairs)
    nbytes = m.n_layers * per_layer * es + rows * m.d * es + total * m.d * 4 + index_bytes
    if c["head"]:
        flops += 2.0 * c["B"] * m.vocab * m.d
        nbytes += m.vocab * m.d * es + c["B"] * m.vocab * 4
    return {"bytes": nbytes, "flops": flops}


_LARGEST_FLOPS = work(next(c for c in listed() if c["name"] == "8B 256 candidates"))["flops"]


def tolerance(case):
    """About four times the error measured against the fp64 oracle (RMS and largest, over the output's RMS): fp32 5e-7
    and 4e-6; fp16 operands 4.5e-4 and 4e-3 at d = 1024, 1.8e-3 and 1.0e-2 at d >= 2560 (its weights do not attenuate
    a perturbation); bf16 operands, eight significand bits through 28 layers, 6e-3 and 2.8e-2.  The maps are exact."""
    if case["op"] == "index":
        return "exact"
    if case["compute"] == "f32":
        return {"rel": 2e-6, "max": 1.6e-5}
    if case["compute"] == "bf16":
        return {"rel": 2.4e-2, "max": 0.15}
    if MODELS[case["model"]].d <= 1024:
        return {"rel": 2e-3, "max": 1.6e-2}
    return {"rel": 7e-3, "max": 4e-2}
