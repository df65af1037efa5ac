"""Timed cases of the paged decode-attention library: what they are, how their
inputs are made, one pass of each, and the same result in 64 bits.

A case is one layer-step's share of the work an engine hands to the library:
the attention of a decode batch over its paged fp16 cache (plain, without
allocation, with the current token's append fused in, or with a fixed-width
table and the log-sum-exp), the append of new K/V rows, or a host-attended
batch through the overlap runtime.  d = 128 and block size 16 throughout.

Request lengths belong to the case (drawn from its `lens_seed`); block
placement and all values come from the seed that `prepare` is given.
"""
import math

import numpy as np
import torch

import paper_2506_03296_amd as A
from paper_2506_03296_amd import overlap

D = 128
BS = 16
SCALE = float(np.float32(1.0 / math.sqrt(D)))


def _case(name, kind, B, Hq, Hkv, lens, lo, hi, lens_seed, **more):
    return dict(name=name, kind=kind, B=B, Hq=Hq, Hkv=Hkv, lens=lens, lo=lo, hi=hi, lens_seed=lens_seed, **more)


def listed():
    return [
        # A handful of short requests on Llama-2-7B heads (lengths 17 to 511):
        # launch and latency are all there is.
        _case("tiny_mha", "attend", 4, 32, 32, "spread", 17, 511, 1),
        # One interactive user of Llama-3.1-8B, the layer-step in one launch:
        # the current token is attended and stored by the same call.
        _case("chat_single_fused", "fused", 1, 32, 8, "uniform", 2100, 2100, 1),
        # A small chat batch, the layer-step as two launches (append, then
        # attend) with K and V read out of a packed projection buffer.
        _case("chat_batch_step", "step", 16, 32, 8, "uniform", 256, 4096, 2),
        # One kv-head group of Llama-3.1-8B's eight, as a rank of a
        # tensor-parallel group has it, on a moderate batch.
        _case("tp_rank_noalloc", "noalloc", 48, 4, 1, "uniform", 512, 8192, 3),
        # A group of two q-heads per kv-head, ragged short contexts, fused append.
        _case("g2_ragged_fused", "fused", 24, 32, 16, "uniform", 17, 2048, 4),
        # One request that fills Llama-3.1-8B's longest context (131072 tokens).
        _case("long_single", "attend", 1, 32, 8, "uniform", 131071, 131071, 5),
        # Llama-3-70B heads (G = 8) in an engine with fixed-width table rows
        # that also asks for the log-sum-exp (to merge with other ranges).
        _case("g8_wide_lse", "wide", 12, 64, 8, "uniform", 2048, 16384, 6, stride=2048),
        # The repository's own bandwidth workloads: a Llama-2-7B MHA batch ...
        _case("mha_batch", "attend", 64, 32, 32, "uniform", 512, 2048, 7),
        # ... the Llama-3.1-8B long-output batch ...
        _case("long_output", "noalloc", 32, 32, 8, "lognormal", 4096, 32768, 8),
        # ... and the mixed batch under memory pressure, the largest of all.
        _case("mixed_pressure", "attend", 512, 32, 8, "bimodal", 256, 16384, 9, key_offset=0.5),
        # Prompts written to the cache after their prefill: about 57 000
        # tokens of 24 prompts in one call.
        _case("prompt_append", "append", 24, 32, 8, "uniform", 512, 4096, 10),
        # Requests attended on the host: rows to the host, append and
        # attention there, the result back.
        _case("host_overlap", "overlap", 16, 32, 8, "uniform", 256, 768, 11),
    ]


# q-heads and kv-heads: the models the repository names, and one rank's share
# of them when the kv-heads are spread over 2, 4 or 8 GPUs
_HEADS = [(32, 32), (32, 8), (32, 8), (64, 8), (32, 16), (16, 4), (8, 2), (4, 1), (16, 16), (8, 1)]
_MAX_BYTES = {"attend": 10e9, "noalloc": 10e9, "wide": 10e9, "fused": 6e8, "step": 6e8, "append": 6e8, "overlap": 6e7}


def draw(rng):
    kind = rng.choice(["attend"] * 6 + ["noalloc"] * 3 + ["fused"] * 3 + ["step"] * 2 + ["wide"] * 3 +
                      ["append"] * 2 + ["overlap"])
    Hq, Hkv = rng.choice(_HEADS)
    while True:
        B = int(round(math.exp(rng.uniform(0.0, math.log(512.0)))))
        top = 131072 if B <= 4 else 32768
        hi = int(round(math.exp(rng.uniform(math.log(16.0), math.log(top)))))
        if kind == "overlap":
            B, hi = min(B, 64), min(hi, 2048)
        lens = rng.choice(["uniform", "uniform", "lognormal", "bimodal", "spread"])
        lo = hi if rng.random() < 0.15 else max(1, int(hi * rng.uniform(0.02, 0.6)))
        c = dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, lens=lens, lo=lo, hi=hi, lens_seed=rng.randrange(1, 1 << 20))
        if kind == "wide":
            c["stride"] = -(-hi // BS) + rng.randrange(0, 1024)
        if int(lengths(c).sum()) * Hkv * D * 4 <= _MAX_BYTES[kind]:
            return c


def lengths(case):
    """Request lengths (int64 [B]); both bounds are inclusive."""
    rng = np.random.default_rng(case["lens_seed"])
    B, lo, hi = case["B"], case["lo"], case["hi"]
    if case["lens"] == "uniform":
        return rng.integers(lo, hi, size=B, endpoint=True)
    if case["lens"] == "spread":      # evenly over the logarithm, both ends among them
        return np.rint(np.exp(np.linspace(math.log(lo), math.log(hi), B))).astype(np.int64)
    if case["lens"] == "lognormal":   # around a third of the way to the longest
        x = np.exp(rng.normal(math.log(max(lo, 0.37 * hi)), 0.5, size=B))
        return np.clip(np.rint(x), lo, hi).astype(np.int64)
    # bimodal: half up to 4 lo, half from hi / 4
    a = rng.integers(lo, max(lo, min(4 * lo, hi)), size=B // 2, endpoint=True)
    b = rng.integers(max(lo, hi // 4), hi, size=B - B // 2, endpoint=True)
    x = np.concatenate([a, b])
    rng.shuffle(x)
    return x


def _slots(table, lens):
    """Cache slots of every request's tokens (int64, all tokens in order) and,
    of those, each request's last one."""
    tok = [torch.arange(int(L), device=table.device) for L in lens]
    rows = [table[b].to(torch.int64)[t // BS] * BS + t % BS for b, t in enumerate(tok)]
    return torch.cat(rows), torch.stack([r[-1] for r in rows])


def _inputs(case, seed):
    """Pool, table and rows on the GPU, from the seed alone."""
    dev = torch.device("cuda", torch.cuda.current_device())
    g = torch.Generator(device=dev).manual_seed(seed * 1000003 + 17)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.float16)

    kind, B, Hq, Hkv = case["kind"], case["B"], case["Hq"], case["Hkv"]
    lens = lengths(case)
    nblk = -(-lens // BS)
    used = int(nblk.sum())
    pool = used + used // 8 + 1       # an engine's pool is never quite full
    width = case.get("stride", int(nblk.max()))
    # row b of the table holds its blocks' ids (blocks lie anywhere in the pool), then zeros
    n = torch.from_numpy(nblk).to(dev)
    table = torch.zeros((B, width), dtype=torch.int32, device=dev)
    table[torch.arange(width, device=dev)[None, :] < n[:, None]] = \
        torch.randperm(pool, generator=g, device=dev)[:used].to(torch.int32)
    k, v, q = normal(pool, Hkv, BS, D), normal(pool, Hkv, BS, D), normal(B, Hq, D)
    if case.get("key_offset"):
        k += normal(1, Hkv, 1, D) * case["key_offset"]
    s = {"kind": kind, "B": B, "Hq": Hq, "Hkv": Hkv, "host_lens": lens, "pool": pool, "q": q, "k": k, "v": v,
         "table": table, "lens": torch.from_numpy(lens.astype(np.int32)).to(dev)}
    if kind == "overlap":
        # q, k_new and v_new back to back, as the runtime copies them in one go
        q, kn, vn = normal(B * (Hq + 2 * Hkv) * D).split([B * Hq * D, B * Hkv * D, B * Hkv * D])
        s["q"], s["k_new"], s["v_new"] = q.view(B, Hq, D), kn.view(B, Hkv, D), vn.view(B, Hkv, D)
        s["slots"] = _slots(table, lens)[1]
    elif kind in ("fused", "step", "append"):
        # K and V rows side by side in one projection buffer
        kv = normal(int(lens.sum()) if kind == "append" else B, 2, Hkv, D)
        s["k_new"], s["v_new"] = kv[:, 0], kv[:, 1]
        s["slots"] = _slots(table, lens)[0 if kind == "append" else 1]
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, B, Hq, Hkv = s["kind"], s["B"], s["Hq"], s["Hkv"]
    s["out"] = torch.empty_like(s["q"])
    if kind in ("fused", "wide"):
        s["workspace"] = torch.zeros(A.workspace_bytes(B, Hq, Hkv), dtype=torch.uint8, device=s["q"].device)
    if kind == "wide":
        s["lse"] = torch.empty((B, Hq), dtype=torch.float32, device=s["q"].device)
    if kind == "overlap":
        s["slots"], s["table"] = s["slots"].cpu().numpy(), s["table"].cpu().numpy()
        s["rt"] = overlap.Overlap(1, B, Hq, Hkv, D, BS, SCALE, s["pool"], s["table"].shape[1])
        hk, hv = s["rt"].host_cache(0)
        hk[...], hv[...] = s.pop("k").cpu().numpy(), s.pop("v").cpu().numpy()
    return s


def run(s):
    kind = s["kind"]
    if kind == "attend":
        return A.decode_attention(s["q"], s["k"], s["v"], s["table"], s["lens"], SCALE)
    if kind == "noalloc":
        return A.decode_attention_noalloc(s["q"], s["k"], s["v"], s["table"], s["lens"], SCALE, s["out"])
    if kind == "wide":
        A.decode_attention_ex(s["q"], s["k"], s["v"], s["table"], s["lens"], SCALE, out=s["out"],
                              block_table_stride=s["table"].shape[1], workspace=s["workspace"], lse_out=s["lse"])
        return [s["out"], s["lse"]]
    if kind == "fused":
        A.decode_attention_ex(s["q"], s["k"], s["v"], s["table"], s["lens"], SCALE, out=s["out"],
                              workspace=s["workspace"], k_new=s["k_new"], v_new=s["v_new"])
        return [s["out"], s["k"], s["v"]]
    if kind == "step":
        A.kv_append(s["k_new"], s["v_new"], s["k"], s["v"], s["slots"])
        return [A.decode_attention(s["q"], s["k"], s["v"], s["table"], s["lens"], SCALE), s["k"], s["v"]]
    if kind == "append":
        A.kv_append(s["k_new"], s["v_new"], s["k"], s["v"], s["slots"])
        return [s["k"], s["v"]]
    ticket = s["rt"].submit(0, s["q"], s["k_new"], s["v_new"], s["slots"], s["table"], s["host_lens"])
    s["rt"].wait(ticket, s["out"])
    return s["out"]


def work(case):
    """Every cached row of a request read once (with an append in the pass, the
    current token's rows come from the new ones and are written once), q read
    and the result written."""
    lens = lengths(case)
    B, Hq, Hkv, kind = case["B"], case["Hq"], case["Hkv"], case["kind"]
    tokens = int(lens.sum())
    row = Hkv * D * 2 * 2             # one token's K and V rows
    if kind == "append":
        return {"bytes": tokens * (2 * row + 8), "flops": 0}
    n = tokens * row + 2 * B * Hq * D * 2 + 4 * B + 4 * int((-(-lens // BS)).sum())
    if kind in ("fused", "step", "overlap"):
        n += B * row
    if kind == "wide":
        n += B * Hq * 4
    return {"bytes": n, "flops": 4 * tokens * Hq * D}


def tolerance(case):
    if case["kind"] == "append":
        return "exact"                # rows are moved, bit for bit
    # fp16 results: rounding alone gives 2.1e-4 in the 2-norm and up to half a
    # spacing, 4.9e-4 of the value, at one place (contexts of a few thousand
    # tokens and more, where nothing else shows); four times that for both
    return {"rel": 8e-4, "max": 2e-3}


def _attend64(q, k, v, table, lens):
    """Plain softmax attention in 64 bits: out [B][Hq][D] and natural-log
    log-sum-exp [B][Hq]."""
    B, Hq, _ = q.shape
    Hkv = k.shape[1]
    out = torch.zeros((B, Hq, D), dtype=torch.float64, device=q.device)
    lse = torch.full((B, Hq), -math.inf, dtype=torch.float64, device=q.device)
    for b, L in enumerate(int(x) for x in lens):
        if L <= 0:
            continue
        ids = table[b, :-(-L // BS)].long()
        kk, vv = (c[ids].permute(1, 0, 2, 3).reshape(Hkv, -1, D)[:, :L].double() for c in (k, v))
        qq = q[b].double().reshape(Hkv, Hq // Hkv, D)
        s = torch.matmul(qq, kk.transpose(1, 2).contiguous()) * SCALE
        lse[b] = torch.logsumexp(s, -1).reshape(Hq)
        out[b] = torch.matmul(torch.softmax(s, -1), vv).reshape(Hq, D)
    return out, lse


def exact(case, seed):
    s = _inputs(case, seed)
    kind, k, v = s["kind"], s["k"], s["v"]
    if "slots" in s:
        block, pos = s["slots"] // BS, s["slots"] % BS
        k[block, :, pos] = s["k_new"]
        v[block, :, pos] = s["v_new"]
    if kind == "append":
        return [k, v]
    out, lse = _attend64(s["q"], k, v, s["table"], s["host_lens"])
    if kind == "wide":
        return [out, lse]
    return [out, k, v] if kind in ("fused", "step") else out
