"""The work that users of this library have it do, as cases that can be timed and compared.

A case is a plain dict. Its "kind" says which loop of a serving program it is:

  decode   one layer's decode attention over a batch of requests (ellm_decode_attention, or its
           allocation-free form), the call every layer of every step makes;
  step     one decode iteration over several layers as a serving loop makes it: map ahead, append the
           new rows and attend in one call per layer, and hand a finished request's tensors to the
           next request, whose prompt is written then;
  prefill  requests turn over (release, acquire) and their prompts' K/V rows are appended in one call;
  swap     one set of requests goes to pinned host memory, another comes back, and the set that has
           come back is decoded.

The other fields are shapes: requests, heads, head size, tokens per chunk (0: what 2 MiB hold), the
distribution of the context lengths (drawn from "lens_seed", so that a case's work does not depend on
the seed of its values) and how the pool is mapped. Values are N(0, 1) in bf16; chunks are scattered
over the pool by a seeded permutation, as they are in a pool that has been in use for a while.
"""
from __future__ import annotations

import math
import sys

import numpy as np
import torch

import paper_2506_15155_amd as E

MIB = 1 << 20
GEN = 512                  # step: tokens a request generates before the next one takes its place
PIECE = 1 << 18            # tokens whose rows are generated at a time


def listed():
    return [
        # the smallest call: four short requests of a small MHA model, 16-token chunks; through the entry
        # point for callers that may not allocate
        _case("decode_tiny", "decode", batch=4, n_kv=8, group=1, dim=64, chunk_tokens=16, dist="uniform", lo=16, hi=256,
              entry="noalloc"),
        # one user's request, interactive: an 8B-shaped layer (32 q / 8 kv heads) over a few thousand tokens
        _case("decode_one", "decode", batch=1, n_kv=8, group=4, dim=128, dist="uniform", lo=3000, hi=3500),
        # a lightly loaded server: 8 requests, 4 layers' steps
        _case("step_small", "step", batch=8, n_kv=8, group=4, dim=128, dist="lognormal", lo=64, hi=8192, layers=4),
        # the headline: 64 requests with long-tailed lengths, the whole decode iteration of an 8B-shaped model
        _case("step_8b", "step", batch=64, n_kv=8, group=4, dim=128, dist="lognormal", lo=64, hi=8192, layers=32),
        # a full server: more requests than one launch describes, in a pool whose chunks the driver maps
        _case("decode_wide", "decode", batch=200, n_kv=8, group=4, dim=128, dist="lognormal", lo=64, hi=8192, pool="driver"),
        # a 13B-shaped MHA layer (40 heads; 102 tokens per 2 MiB chunk)
        _case("decode_mha", "decode", batch=32, n_kv=40, group=1, dim=128, dist="uniform", lo=2048, hi=16384),
        # a 70B-shaped layer (64 q / 8 kv heads) over long contexts: the largest call
        _case("decode_long", "decode", batch=16, n_kv=8, group=8, dim=128, dist="uniform", lo=32768, hi=131072),
        # 6 q heads per kv head: a group that is no power of two
        _case("decode_g6", "decode", batch=48, n_kv=8, group=6, dim=128, dist="lognormal", lo=64, hi=16384),
        # 16 q heads per kv head of 64: few kv heads shared by many q heads
        _case("decode_g16", "decode", batch=64, n_kv=2, group=16, dim=64, dist="uniform", lo=512, hi=24576),
        # small chunks (16 tokens), as a pool tuned for little internal waste uses them
        _case("decode_pages", "decode", batch=32, n_kv=8, group=4, dim=128, chunk_tokens=16, dist="lognormal", lo=64, hi=8192),
        # prompts of four new requests written in one call
        _case("prefill", "prefill", batch=4, n_kv=8, group=4, dim=128, dist="uniform", lo=4096, hi=32768),
        # preemption: requests swapped between HBM and host memory, then decoded
        _case("swap", "swap", batch=8, n_kv=8, group=4, dim=128, dist="lognormal", lo=64, hi=8192),
    ]


def _case(name, kind, batch, n_kv, group, dim, dist, lo, hi, chunk_tokens=0, layers=1, pool="table", entry="plain", lens_seed=1):
    c = {"kind": kind, "batch": batch, "n_kv": n_kv, "group": group, "dim": dim, "chunk_tokens": chunk_tokens, "dist": dist,
         "lo": lo, "hi": hi, "layers": layers, "pool": pool, "entry": entry, "lens_seed": lens_seed}
    return {"name": name, **c} if name else c


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the same ranges: every size at random, odd ones included."""
    kind = rng.choice(["decode"] * 7 + ["step", "prefill", "swap"])
    dim = rng.choice([64, 128, 128])
    n_kv, group = rng.choice([1, 2, 4, 5, 8, 8, 8, 10, 16, 40]), rng.choice([1, 1, 2, 3, 4, 4, 4, 5, 6, 7, 8, 8, 12, 16])
    if n_kv * group > 128:
        group = 128 // n_kv
    bpt = 4 * n_kv * dim
    chunk_tokens = rng.choice([0, 0, 0, 0, 16, 16, 24, 40, 64, 128]) if kind != "swap" else 0
    most = {"decode": 3 << 30, "step": 128 << 20, "prefill": 512 << 20, "swap": 96 << 20}[kind]   # bytes of K and V in a pass
    while True:
        batch = _log(rng, 1, {"decode": 200, "step": 64, "prefill": 8, "swap": 16}[kind])
        mean = _log(rng, 16 if kind == "decode" else 128, 131072 if kind == "decode" else 8192)
        if batch * mean * bpt <= most and (not chunk_tokens or mean <= 8192):
            break
    dist = rng.choice(["uniform", "lognormal"])
    lo, hi = (max(1, mean // 3), mean * 5 // 3) if dist == "uniform" else (max(1, mean // 8), mean * 6)
    pool = rng.choice(["table", "table", "table", "driver"])
    chunk = (chunk_tokens * bpt) if chunk_tokens else 2 * MIB
    if kind != "decode" or chunk % 65536 or -(-batch * mean * bpt // chunk) > 600:
        pool = "table"
    # the allocation-free form takes what fits its fixed workspace
    partials = (1024 + n_kv * (min(batch, 128) - 1)) * group * (dim + 2) * 4
    entry = "noalloc" if kind == "decode" and partials <= E.ELLM_NOALLOC_WORKSPACE_BYTES and rng.random() < 0.2 else "plain"
    return _case("", kind, batch, n_kv, group, dim, dist, lo, hi, chunk_tokens, rng.choice([2, 4, 7]) if kind == "step" else 1, pool, entry,
                 rng.randrange(1 << 20))


# ---- shapes -----------------------------------------------------------------------------------------
def _lens(case):
    """Context lengths of the batch (step: before the first step)."""
    rng = np.random.default_rng(case["lens_seed"])
    lo, hi, n = case["lo"], case["hi"], case["batch"]
    if case["dist"] == "uniform":
        return rng.integers(lo, hi + 1, size=n).astype(np.int64)
    median = math.sqrt(lo * hi) if hi < 1024 else min(max(1024, lo * 2), hi) if lo < 1024 else math.sqrt(lo * hi)
    return np.clip(np.rint(np.exp(math.log(median) + rng.standard_normal(n))), lo, hi).astype(np.int64)


def _life(case):
    """step: prompt length of every request, and the length at which it is done."""
    lens = _lens(case)
    made = np.random.default_rng(case["lens_seed"] + 7).integers(0, GEN, size=len(lens))
    prompt = np.maximum(1, lens - made)
    return prompt, np.maximum(lens + 1, prompt + GEN)


def _chunk(case):
    bpt = 4 * case["n_kv"] * case["dim"]
    return (case["chunk_tokens"], case["chunk_tokens"] * bpt) if case["chunk_tokens"] else (2 * MIB // bpt, 2 * MIB)


def _hq(case):
    return case["n_kv"] * case["group"]


# ---- values -----------------------------------------------------------------------------------------
def _gen(seed, *what):
    g = torch.Generator(device="cuda")
    s = seed & 0xFFFFFFFF
    for w in what:
        s = (s * 1000003 + w + 1) & 0x7FFFFFFFFFFF
    return g.manual_seed(s)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)


def _history(case, seed, layer, lens, which=0):
    """The K and V rows of a layer's requests, a few requests at a time: (first, end, k, v)."""
    g = _gen(seed, 1, layer, which)
    b = 0
    while b < len(lens):
        e, n = b + 1, int(lens[b])
        while e < len(lens) and n + int(lens[e]) <= PIECE:
            n += int(lens[e])
            e += 1
        yield b, e, _randn(g, n, case["n_kv"], case["dim"]), _randn(g, n, case["n_kv"], case["dim"])
        b = e


def _queries(case, seed):
    return _randn(_gen(seed, 2), case["layers"], case["batch"], _hq(case), case["dim"])


def _new_rows(case, seed):
    g = _gen(seed, 3)
    shape = (case["layers"], case["batch"], case["n_kv"], case["dim"])
    return _randn(g, *shape), _randn(g, *shape)


# ---- what a program keeps ---------------------------------------------------------------------------
class _State:
    """A pool with its tensors, and the buffers of the loop around it."""

    pool = None

    def __init__(self, case, n_chunks, max_tensors, max_tokens, host_chunks=0):
        tokens, chunk = _chunk(case)
        self.case, self.tokens, self.returned = case, tokens, None
        nbytes = n_chunks * chunk
        self.host = torch.empty(host_chunks * chunk, dtype=torch.uint8, pin_memory=True) if host_chunks else None
        shape = (chunk, _hq(case), case["n_kv"], case["dim"], max_tensors, -(-max_tokens // tokens))
        if case["pool"] == "driver":
            self.buf = None
            self.pool = E.ellm_pool_create(None, self.host, *shape, flags=E.ELLM_POOL_DRIVER_MAPPED, device_bytes=nbytes)
        else:
            self.buf = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
            self.pool = E.ellm_pool_create(self.buf, self.host, *shape)
            if nbytes <= 1 << 30:
                self.returned = self.buf.view(torch.int64)     # the chunks' bytes are part of the result

    def tensor(self, max_tokens, chunk_ids):
        t = E.ellm_tensor_create(self.pool, int(max_tokens))
        E.ellm_tensor_map_chunks(self.pool, t, 0, len(chunk_ids), chunk_ids)
        return t

    def __del__(self):
        if self.pool is not None and not sys.is_finalizing():
            torch.cuda.synchronize()
            E.ellm_pool_destroy(self.pool)
            self.pool = None


def _scattered(seed, n):
    return np.random.default_rng(seed).permutation(n).astype(np.int32)


def prepare(case, seed):
    lens, (tokens, _) = _lens(case), _chunk(case)
    B, layers, kind = case["batch"], case["layers"], case["kind"]
    if kind == "step":
        prompt, end = _life(case)
    need = [int(-(-int(n) // tokens)) for n in lens]
    sets = 2 if kind == "swap" else 1
    full = [int(-(-int(n) // tokens)) for n in end] if kind == "step" else need
    n_chunks = layers * sets * sum(full) + 2
    st = _State(case, n_chunks, layers * sets * B, int(end.max()) if kind == "step" else int(lens.max()), sum(need) * 2 if kind == "swap" else 0)
    at, place = 0, _scattered(seed, n_chunks)
    st.ids = []
    for rows in range(layers * sets):
        ids = np.empty(B, np.int32)
        for b in range(B):
            ids[b] = st.tensor(end[b] if kind == "step" else lens[b], place[at:at + need[b]])
            at += need[b]
        st.ids.append(ids)
        if kind != "prefill":
            for b, e, k, v in _history(case, seed, rows % layers, lens, rows // layers):
                E.ellm_kv_append(st.pool, ids[b:e], k, v, lens[b:e].astype(np.int32))
    st.q = _queries(case, seed)
    st.out = torch.empty_like(st.q)
    if kind == "step":
        st.k_new, st.v_new = _new_rows(case, seed)
        g, n = _gen(seed, 4), int(prompt.max())
        st.k_prompt, st.v_prompt = _randn(g, n, case["n_kv"], case["dim"]), _randn(g, n, case["n_kv"], case["dim"])
        st.len, st.prompt, st.end = lens.copy(), prompt, end
    if kind == "prefill":
        rows = [(k, v) for _, _, k, v in _history(case, seed, 0, lens)]
        st.k, st.v = torch.cat([k for k, _ in rows]), torch.cat([v for _, v in rows])
        st.n_new, st.len = lens.astype(np.int32), lens
    if kind == "swap":
        st.need, st.here = need, 0
        for b in range(B):
            E.ellm_chunk_deflate_to_host(st.pool, int(st.ids[1][b]), 0, need[b])
        E.ellm_pool_sync(st.pool)
    torch.cuda.synchronize()
    return st


# ---- a pass -----------------------------------------------------------------------------------------
def run(st):
    return _RUN[st.case["kind"]](st)


def _run_decode(st):
    call = E.ellm_decode_attention_noalloc if st.case["entry"] == "noalloc" else E.ellm_decode_attention
    call(st.pool, st.ids[0], st.q[0], st.out[0])
    return [st.out]


def _run_step(st):
    for b in np.flatnonzero(st.len >= st.end):          # done: its tensors go to the next request, whose prompt is written
        n = int(st.prompt[b])
        for ids in st.ids:
            E.ellm_tensor_release(st.pool, int(ids[b]))
            ids[b] = E.ellm_tensor_acquire(st.pool, n, int(st.end[b]))
            E.ellm_kv_append(st.pool, ids[b:b + 1], st.k_prompt, st.v_prompt, [n])
        st.len[b] = n
    for layer, ids in enumerate(st.ids):
        E.ellm_kv_premap_next(st.pool, ids)
        E.ellm_kv_append_decode(st.pool, ids, st.k_new[layer], st.v_new[layer], st.q[layer], st.out[layer])
    st.len += 1
    return [st.out] + ([st.returned] if st.returned is not None else [])


def _run_prefill(st):
    ids = st.ids[0]
    for b in range(len(ids)):
        E.ellm_tensor_release(st.pool, int(ids[b]))
        ids[b] = E.ellm_tensor_acquire(st.pool, int(st.len[b]), int(st.len[b]))
    E.ellm_kv_append(st.pool, ids, st.k, st.v, st.n_new)
    return [st.returned]


def _run_swap(st):
    here, other = st.ids[st.here], st.ids[1 - st.here]
    for b in range(len(here)):
        E.ellm_chunk_deflate_to_host(st.pool, int(here[b]), 0, st.need[b])
    for b in range(len(other)):
        E.ellm_chunk_inflate_from_host(st.pool, int(other[b]), 0, st.need[b])
    st.here = 1 - st.here
    E.ellm_decode_attention(st.pool, other, st.q[0], st.out[0])
    return [st.out]


_RUN = {"decode": _run_decode, "step": _run_step, "prefill": _run_prefill, "swap": _run_swap}


# ---- what a pass cannot do without ------------------------------------------------------------------
def work(case):
    n, B, (tokens, chunk) = int(_lens(case).sum()), case["batch"], _chunk(case)
    row, qo = 4 * case["n_kv"] * case["dim"], 2 * 2 * B * _hq(case) * case["dim"]
    flops = 4 * n * _hq(case) * case["dim"]
    if case["kind"] == "prefill":
        return {"bytes": 2 * n * row, "flops": 0}
    if case["kind"] == "step":
        return {"bytes": case["layers"] * (n * row + 2 * B * row + qo), "flops": case["layers"] * flops}
    moved = 4 * chunk * sum(int(-(-int(x) // tokens)) for x in _lens(case)) if case["kind"] == "swap" else 0
    return {"bytes": n * row + qo + moved, "flops": flops}


def tolerance(case):
    if case["kind"] == "prefill":
        return "exact"
    # the softmax weights and the results are rounded to bf16: measured 1.9e-3 to 2.3e-3 against 64 bits
    return {"rel": 8e-3, "max": 5e-2}


# ---- the same in 64 bits ----------------------------------------------------------------------------
def _attend(case, q, k, v):
    """One request: q [heads][dim], k and v [tokens][kv heads][dim] -> [heads][dim], fp64."""
    Hkv, G, D = case["n_kv"], case["group"], case["dim"]
    out = torch.empty(Hkv, G, D, dtype=torch.float64, device=q.device)
    for h in range(Hkv):
        kh, vh = k[:, h].double().contiguous(), v[:, h].double().contiguous()
        s = kh @ q[h * G:(h + 1) * G].double().t().contiguous() / math.sqrt(D)
        out[h] = torch.softmax(s, 0).t().contiguous() @ vh
    return out.view(Hkv * G, D)


def exact(case, seed):
    if case["kind"] == "prefill":
        return None
    lens, q = _lens(case), _queries(case, seed)
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    new = _new_rows(case, seed) if case["kind"] == "step" else None
    for layer in range(case["layers"]):
        for b, e, k, v in _history(case, seed, layer, lens, 1 if case["kind"] == "swap" else 0):
            at = 0
            for i in range(b, e):
                n = int(lens[i])
                ki, vi = k[at:at + n], v[at:at + n]
                if new is not None:
                    ki, vi = torch.cat([ki, new[0][layer, i:i + 1]]), torch.cat([vi, new[1][layer, i:i + 1]])
                out[layer, i] = _attend(case, q[layer, i], ki, vi)
                at += n
    return [out, None] if case["kind"] == "step" else [out]
