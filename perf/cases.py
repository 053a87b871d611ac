"""What the library's users run, as cases that can be timed and compared.

A rollout engine runs one decode step after another over a paged KV cache
(append the new token, then attend), from the start of a rollout, when every
sequence is short, to its end, when a few long ones are left of the batch its
handle was made for; it extends sequences by whole prompts, by turns of a few
hundred tokens and by short tool replies; and between steps a trainer's weights
go through a transfer buffer.  Shapes are those of
paper_2512_22492_amd/workloads.py (head layouts, lengths, page placement) and
of the weight-sync benchmark.

Lengths belong to the case (drawn from its own "shape_seed"), so the work of a
case does not depend on the seed its values are made from.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2512_22492_amd import binding, workloads

DEV = "cuda"
PAGE = 16
D = 128
# query heads / kv heads: Qwen3-8B, its TP = 8 share, Qwen3-32B, Qwen3-235B,
# and the small layout of the "tiny" workload
HEADS = [(32, 8), (4, 1), (64, 8), (64, 4), (8, 2)]
WINDOW = 65536   # the rollout's context window: 4096 pages a sequence


# ------------------------------------------------------------------ cases ---

def _decode(name, batch, heads, lengths, kv="bf16", layout="hnd", append=False,
            max_batch=None, window=None, shape_seed=0):
    """lengths "kind:a:b:..." as in workloads.draw_lengths, new token included;
    max_batch and window (tokens) are what the handle and the block table are
    made for, by default just what the batch needs."""
    c = dict(op="decode", batch=batch, hq=heads[0], hkv=heads[1], lengths=lengths, kv=kv,
             layout=layout, append=append, max_batch=max_batch or batch,
             window=window or 0, shape_seed=shape_seed)
    if name:
        c["name"] = name
    return c


def _extend(name, batch, heads, new, prior, kv="bf16", layout="hnd", window=None,
            shape_seed=0):
    """Each sequence gets `new` tokens after `prior` cached ones."""
    c = dict(op="extend", batch=batch, hq=heads[0], hkv=heads[1], new=new, prior=prior,
             kv=kv, layout=layout, window=window or 0, shape_seed=shape_seed)
    if name:
        c["name"] = name
    return c


def _weights(name, layers, ranks, flat, capacity, shape_seed=0):
    c = dict(op="weights", layers=layers, ranks=ranks, flat=flat, capacity=capacity,
             shape_seed=shape_seed)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest step there is: four short sequences, append and attend
        _decode("step_tiny", 4, (8, 2), "uniform:1:512", append=True, shape_seed=1),
        # the start of a rollout: ragged prompts, e4m3 token-major pools (as serving
        # engines allocate them), a table as wide as the context window
        _decode("step_round_start", 200, (64, 4), "uniform:60:1200", kv="fp8_e4m3",
                layout="nhd", append=True, max_batch=256, window=WINDOW, shape_seed=2),
        # the middle of a rollout: the Qwen3-8B decode step
        _decode("decode_step", 64, (32, 8), "fixed:4096"),
        # the end of a rollout: three long sequences left in the engine's handle
        _decode("decode_last_few", 3, (32, 8), "uniform:8192:32768", max_batch=64,
                window=WINDOW, shape_seed=4),
        # a large batch with a long-tailed length distribution
        _decode("decode_long_tail", 256, (32, 8), "lognormal:4096:0.8:256:32768",
                shape_seed=5),
        # a large batch of short sequences in e4m3 pools
        _decode("decode_fp8_batch", 1024, (32, 8), "uniform:512:2048", kv="fp8_e4m3",
                shape_seed=6),
        # one GPU of a tensor-parallel rollout over eight: one kv head
        _decode("decode_tp_share", 64, (4, 1), "lognormal:4096:0.8:256:32768",
                window=WINDOW, shape_seed=7),
        # prompts prefilled from nothing (also: a reassigned trajectory's), e4m3
        _extend("extend_prompts", 48, (32, 8), "uniform:100:2000", "fixed:0", kv="fp8_e4m3",
                window=WINDOW, shape_seed=8),
        # a turn of 512 tokens for every sequence of the Qwen3-8B step
        _extend("extend_turn", 64, (32, 8), "fixed:512", "fixed:4096"),
        # short tool replies of a multi-turn rollout, after long histories
        _extend("extend_replies", 12, (32, 8), "uniform:5:90", "uniform:2000:16000",
                window=WINDOW, shape_seed=10),
        # four whole Qwen3-8B layers through a 1 GiB transfer buffer and back out
        _weights("weights_layers", 4, 1, False, 1 << 30),
        # one rank's flat shard of a model sharded evenly by elements over six
        # ranks: its tensors are pieces at any element of the shard
        _weights("weights_flat_shard", 4, 6, True, 1 << 28, shape_seed=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _kv_tokens(case):
    """(tokens x kv heads) a decode case reads, in bf16 tokens."""
    per = 1.0 if case["kv"] == "bf16" else 0.5
    return per * case["hkv"] * float(_lengths(case).sum())


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["extend"] * 4 + ["weights"] * 2)
    seed = rng.randrange(1 << 30)
    kv = rng.choice(["bf16", "fp8_e4m3"])
    layout = rng.choice(["hnd", "hnd", "nhd", "hnd_kv"])
    heads = rng.choice(HEADS)
    if kind == "decode":
        top = 256 * 4096 * 8          # about the long-tailed batch's tokens x kv heads
        while True:
            batch = _log_int(rng, 1, 1024)
            mid = _log_int(rng, 40, 30000)
            spread = rng.choice(["uniform", "lognormal", "fixed"])
            if spread == "uniform":
                lengths = "uniform:%d:%d" % (max(1, mid // 3), min(WINDOW, 2 * mid))
            elif spread == "lognormal":
                lengths = "lognormal:%d:0.8:%d:%d" % (mid, max(1, mid // 16),
                                                      min(WINDOW, 8 * mid))
            else:
                lengths = "fixed:%d" % mid
            engine = rng.random() < 0.5  # a handle made for a larger batch and the window
            c = _decode(None, batch, heads, lengths, kv=kv, layout=layout,
                        append=rng.random() < 0.3,
                        max_batch=max(batch, _log_int(rng, 16, 256)) if engine else None,
                        window=WINDOW if engine else None, shape_seed=seed)
            # appends give their pools back whole: keep those moderate
            if _kv_tokens(c) <= (top / 16 if c["append"] else top):
                return c
    if kind == "extend":
        while True:
            batch = _log_int(rng, 1, 256)
            new = _log_int(rng, 1, 2000)
            prior = 0 if rng.random() < 0.25 else _log_int(rng, 16, 32000)
            c = _extend(None, batch, heads,
                        rng.choice(["fixed:%d" % new,
                                    "uniform:%d:%d" % (max(1, new // 8), new)]),
                        rng.choice(["fixed:%d" % prior,
                                    "uniform:%d:%d" % (prior // 4, prior)]),
                        kv=kv, layout=layout,
                        window=rng.choice([None, WINDOW]), shape_seed=seed)
            w = work(c)
            if w["flops"] <= 2.0e12 and w["bytes"] <= 4.0e9:
                return c
    # odd rank counts too; a buffer that takes the shard in one to several fills
    ranks = rng.choice([1, 2, 3, 5, 6, 7, 8])
    layers = rng.randint(1, 4)
    shard = sum(_weight_elems(layers)) * 2 // ranks
    cap = max(1 << 16, (int(shard * math.exp(rng.uniform(math.log(0.2), math.log(1.5))))
                        // 4096) * 4096)
    return _weights(None, layers, ranks, rng.random() < 0.6, cap, shape_seed=seed)


# ----------------------------------------------------------------- shapes ---

def _spec(text):
    kind, *rest = text.split(":")
    return (kind,) + tuple(float(x) if "." in x else int(x) for x in rest)


def _lengths(case, key="lengths", salt=0):
    rng = np.random.default_rng([int(case["shape_seed"]), salt])
    return workloads.draw_lengths(rng, case["batch"], _spec(case[key]))


def _new_prior(case):
    return _lengths(case, "new", 1), _lengths(case, "prior", 2)


# One Qwen3-8B layer's tensors, in elements: q, k, v, o, gate, up, down, the
# layer norms and the q / k norms
_LAYER = [4096 * 4096, 1024 * 4096, 1024 * 4096, 4096 * 4096, 12288 * 4096, 12288 * 4096,
          4096 * 12288, 4096, 4096, 128, 128]


def _weight_elems(layers):
    return _LAYER * layers


def _rank_elems(case):
    """Elements of each tensor that this rank holds.  flat: the model laid end
    to end and cut into equal shards by elements, the middle rank's pieces;
    else each tensor cut by elements and the first cut kept."""
    sizes, ranks = _weight_elems(case["layers"]), case["ranks"]
    if not case["flat"]:
        return [max(1, n // ranks) for n in sizes]
    total = sum(sizes)
    per = (total + ranks - 1) // ranks
    lo = (ranks // 2) * per
    hi = min(lo + per, total)
    out, at = [], 0
    for n in sizes:
        a, b = max(lo, at), min(hi, at + n)
        if b > a:
            out.append(b - a)
        at += n
    return out


# ---------------------------------------------------------------- prepare ---

def _problem(case, lengths, seed):
    p = workloads.make_problem(
        case["op"], batch=case["batch"], num_q_heads=case["hq"], num_kv_heads=case["hkv"],
        lengths=[int(x) for x in lengths], kv_dtype=case["kv"], layout=case["layout"],
        seed=int(seed), device=DEV,
        max_pages=case["window"] // PAGE if case["window"] else None)
    # queries of twice the keys' spread: scores with a standard deviation of 2,
    # so that some tokens stand out as they do in a trained model
    p.q.mul_(2.0)
    return p


def _randn(shape, gen):
    return torch.randn(shape, generator=gen, device=DEV).to(torch.bfloat16)


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed) * 1009 + 5)
    if case["op"] == "decode":
        p = _problem(case, _lengths(case), seed)
        st = dict(p=p, out=torch.empty_like(p.q), op="decode", append=None)
        st["attn"] = binding.DecodeAttention(
            p.num_q_heads, p.num_kv_heads, case["max_batch"], p.max_pages,
            kv_dtype=p.kv_dtype, layout=p.layout)
        if case["append"]:
            shape = (p.batch, p.num_kv_heads, D)
            st["k_new"], st["v_new"] = _randn(shape, gen), _randn(shape, gen)
            # the lengths before the new token, which the append writes at
            p.before = p.seq_lens - 1
            cache = workloads.DecodeProblem(**{k: v for k, v in p.__dict__.items()
                                               if k not in ("seq_lens", "before")},
                                            seq_lens=p.before)
            st["append"] = binding.KvAppender(cache)
        return st
    if case["op"] == "extend":
        new, prior = _new_prior(case)
        p = _problem(case, new + prior, seed)
        total = int(new.sum())
        q = _randn((total, p.num_q_heads, D), gen).mul_(2.0)
        starts = np.concatenate([[0], np.cumsum(new)]).astype(np.int32)
        return dict(op="extend", p=p, q=q, out=torch.empty_like(q), max_new=int(new.max()),
                    q_start=torch.from_numpy(starts).to(DEV))
    elems = _rank_elems(case)
    flat = _randn((sum(elems),), gen)
    if case["flat"]:
        tensors = list(flat.split(elems))
        back = list(torch.zeros_like(flat).split(elems))
    else:
        tensors = [t.clone() for t in flat.split(elems)]
        back = [torch.zeros_like(t) for t in tensors]
    buf = torch.zeros(case["capacity"], dtype=torch.uint8, device=DEV)
    return dict(op="weights", send=binding.WeightSync(tensors, buf),
                recv=binding.WeightSync(back, buf), back=back, buf=buf)


# -------------------------------------------------------------------- run ---

def run(state):
    stream = torch.cuda.current_stream()
    if state["op"] == "decode":
        p = state["p"]
        if state["append"] is None:
            state["attn"].run_problem(p, state["out"], stream)
            return state["out"]
        state["append"](state["k_new"], state["v_new"], stream)
        state["attn"].run_problem(p, state["out"], stream)
        outs = [state["out"], p.k_pool, p.v_pool]
        return outs + ([] if p.k_scale is None else [p.k_scale, p.v_scale])
    if state["op"] == "extend":
        binding.extend_attention(state["p"], state["q"], state["q_start"], state["max_new"],
                                 state["out"], stream)
        return state["out"]
    # one weight update: each fill of the buffer is packed, and (the network's
    # part left out) placed into the receiver's tensors
    for c in range(state["send"].num_chunks):
        state["send"].pack(c, stream)
        state["recv"].unpack(c, stream)
    return list(state["back"])


# ------------------------------------------------------------------- work ---

def work(case):
    if case["op"] == "weights":
        n = 2 * sum(_rank_elems(case))
        return {"bytes": 4 * n, "flops": 0}    # read, buffered (written, read), written
    elt = 2 if case["kv"] == "bf16" else 1
    if case["op"] == "decode":
        lengths = _lengths(case)
        rows = case["batch"] * case["hq"]
        visible = int(lengths.sum())
        pairs = visible
    else:
        new, prior = _new_prior(case)
        lengths = new + prior
        rows = int(new.sum()) * case["hq"]
        visible = int(lengths.sum())
        # new token i sees prior + i + 1 tokens
        pairs = int((new * prior + new * (new + 1) // 2).sum())
    pages = int(((lengths + PAGE - 1) // PAGE).sum())
    n = visible * case["hkv"] * D * 2 * elt + 2 * rows * D * 2
    n += 4 * pages + 4 * case["batch"]
    if case["kv"] != "bf16":
        n += pages * case["hkv"] * 2 * 4
    if case.get("append"):
        n += case["batch"] * case["hkv"] * D * 2 * (2 + elt)
    return {"bytes": n, "flops": 4 * D * case["hq"] * pairs}


# -------------------------------------------------------------- tolerance ---

def tolerance(case):
    if case["op"] == "weights":
        return "exact"
    # Against the 64-bit results the bf16 outputs are off by 1.7e-3 in decode (their
    # rounding) and by 2.0e-3 to 2.4e-3 in extend, which also rounds the
    # probabilities to bf16: about four times that.  A single value may land on
    # the neighbouring bf16 number, 2^-7 of it, in decode, and two or three away
    # in extend.
    if case["op"] == "decode":
        return {"rel": 7e-3, "max": 3e-2}
    return {"rel": 1e-2, "max": 8e-2}


# ------------------------------------------------------------------ exact ---

def _cache_rows(p, b, n):
    """Sequence b's first n cached keys and values in 64 bits, [Hkv, n, D]."""
    ids = p.block_table[b, :(n + PAGE - 1) // PAGE].long()

    def rows(pool, scale):
        x = pool[ids]
        if p.layout == "nhd":
            x = x.transpose(1, 2)
        if scale is None:
            x = x.double()
        else:
            x = (x.contiguous().view(torch.float8_e4m3fn).double()
                 * scale[ids].double()[:, :, None, None])
        return x.transpose(0, 1).reshape(p.num_kv_heads, -1, D)[:, :n]
    return rows(p.k_pool, p.k_scale), rows(p.v_pool, p.v_scale)


def _attend(p, b, n, q):
    """q [n_new, Hq, D]: the sequence's last n_new of its n tokens, causal."""
    new = q.shape[0]
    k, v = _cache_rows(p, b, n)
    g = p.num_q_heads // p.num_kv_heads
    x = q.double().view(new, p.num_kv_heads, g, D).transpose(0, 1).reshape(
        p.num_kv_heads, new * g, D)
    s = torch.matmul(x, k.transpose(1, 2).contiguous()) * p.scale
    if new > 1:
        seen = torch.arange(n - new, n, device=DEV).repeat_interleave(g)
        s.masked_fill_(torch.arange(n, device=DEV)[None, :] > seen[:, None], -math.inf)
    o = torch.matmul(torch.softmax(s, -1), v.contiguous())
    return o.view(p.num_kv_heads, new, g, D).transpose(0, 1).reshape(new, p.num_q_heads, D)


def _plain_append(p, k_new, v_new):
    """The append in plain torch: bf16 rows copied; e4m3 slabs with one scale
    that starts at the first token's absmax / 448 and only grows."""
    for b, length in enumerate(p.before.tolist()):
        page, slot = int(p.block_table[b, length // PAGE]), length % PAGE
        for pool, scale, new in ((p.k_pool, p.k_scale, k_new), (p.v_pool, p.v_scale, v_new)):
            slab = pool[page].transpose(0, 1) if p.layout == "nhd" else pool[page]
            if scale is None:
                slab[:, slot] = new[b]
                continue
            x = new[b].float()
            top = x.abs().amax(1)
            want = torch.where(top > 0, top / 448.0, torch.ones_like(top))
            old = scale[page].clone()
            s = want if slot == 0 else torch.maximum(want, old)
            if slot:
                grown = (s != old)[:, None, None]
                c = slab[:, :slot].contiguous()
                f = c.view(torch.float8_e4m3fn).float() * (old / s)[:, None, None]
                slab[:, :slot] = torch.where(
                    grown, f.to(torch.float8_e4m3fn).view(torch.uint8), c)
            y = (x / s[:, None]).clamp(-448.0, 448.0)
            slab[:, slot] = y.to(torch.float8_e4m3fn).view(torch.uint8)
            scale[page] = s


def exact(case, seed):
    if case["op"] == "weights":
        return None            # bytes, compared as they are
    st = prepare(case, seed)
    p = st["p"]
    if case["op"] == "decode":
        if case["append"]:
            _plain_append(p, st["k_new"], st["v_new"])
        lens = p.lengths().tolist()
        out = torch.cat([_attend(p, b, n, p.q[b:b + 1]) for b, n in enumerate(lens)])
        if not case["append"]:
            return out
        return [out, None, None] + ([] if p.k_scale is None else [None, None])
    starts, lens = st["q_start"].tolist(), p.lengths().tolist()
    return torch.cat([_attend(p, b, n, st["q"][starts[b]:starts[b + 1]])
                      for b, n in enumerate(lens)])
