"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain values; `kind` names the path it takes:

  attend    one decode-attention call over compressed caches and the dense window of every
            batch entry (`mustafar_window_decode_attn`), the call a serving loop makes per
            layer and token; its caches come from `mustafar_window_prefill`
  dense     the same attention over dense caches (`mustafar_dense_decode_attn`)
  compress  the pruning and compression of a prompt's keys and values: by magnitude, with
            output-aware or 2:4 keys, or with per-channel values
  generate  a whole request: prefill of the prompts, then decode steps with their appends
            and attention, through one of the library's four decode loops

Sizes are those of the synthetic workloads (Llama-class layers from one sequence of 4K tokens
to sixteen of 32K, or one of 128K), of the tests (head sizes 64, 128 and 256, ragged batches,
1 to 8 query heads per kv-head), and of short prompts. Sparsities are the paper's 50% and 70%,
with 80% from its appendix in drawn cases.
"""
import math

import torch

import paper_2505_22913_amd as mf
from paper_2505_22913_amd import synth

GROUP = 32      # tokens per group of per-channel value pruning
EXACT_ELEMENTS = 1 << 28   # key elements above which the 64-bit answer takes too long


def listed():
    return [
        # One chat sequence of 4K tokens on a 32-head layer: the latency of a single call.
        dict(name="attend_b1_mha_4k", kind="attend", B=1, Hq=32, Hkv=32, d=128, n=4096, ragged=False,
             sK=0.5, sV=0.5, W=32),
        # Four 16K sequences on a grouped-query layer, the usual serving shape.
        dict(name="attend_b4_gqa4_16k", kind="attend", B=4, Hq=32, Hkv=8, d=128, n=16384, ragged=False,
             sK=0.7, sV=0.7, W=32),
        # One very long sequence: few streams, many tokens each.
        dict(name="attend_b1_gqa4_128k", kind="attend", B=1, Hq=32, Hkv=8, d=128, n=131072, ragged=False,
             sK=0.7, sV=0.7, W=32),
        # Eight query heads per kv-head, the largest group.
        dict(name="attend_b4_gqa8_16k", kind="attend", B=4, Hq=64, Hkv=8, d=128, n=16384, ragged=False,
             sK=0.7, sV=0.7, W=32),
        # The benchmark's own call: sixteen 32K sequences, one query head per kv-head.
        dict(name="attend_b16_mha_32k", kind="attend", B=16, Hq=32, Hkv=32, d=128, n=32768, ragged=False,
             sK=0.5, sV=0.7, W=32),
        # A continuous batch whose sequences have different (odd) lengths, on small heads.
        dict(name="attend_b6_gqa2_d64_9k_ragged", kind="attend", B=6, Hq=16, Hkv=8, d=64, n=9001, ragged=True,
             sK=0.5, sV=0.7, W=32),
        # The dense form of the serving shape, for caches that are not (yet) compressed.
        dict(name="dense_b4_gqa4_16k", kind="dense", B=4, Hq=32, Hkv=8, d=128, n=16384),
        # Compression of a batch's prompts, keys and values, right after their prefill.
        dict(name="compress_b4_mha_16k", kind="compress", mode="magnitude", B=4, Hq=32, Hkv=32, d=128, n=16384,
             sK=0.5, sV=0.7),
        # The same with keys scored by the queries that follow them.
        dict(name="compress_b4_gqa4_16k_output_aware", kind="compress", mode="output_aware", B=4, Hq=32, Hkv=8,
             d=128, n=16384, sK=0.7, sV=0.7),
        # The same with values pruned per channel in groups of 32 tokens.
        dict(name="compress_b4_gqa4_16k_channel", kind="compress", mode="channel", B=4, Hq=32, Hkv=8, d=128,
             n=16384, sK=0.5, sV=0.7),
        # A small batch of requests of different lengths from prompt to sixteenth token.
        dict(name="generate_b8_gqa4_2k_ragged", kind="generate", loop="window", B=8, Hq=32, Hkv=8, d=128, n=2048,
             ragged=True, steps=16, sK=0.7, sV=0.7, W=32),
        # One short request through the plain calls: compress, then append and attend per token.
        dict(name="generate_b1_mha_1k_append", kind="generate", loop="append", B=1, Hq=32, Hkv=32, d=128, n=1000,
             ragged=False, steps=16, sK=0.5, sV=0.5, W=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attend"] * 5 + ["dense"] + ["compress"] * 3 + ["generate"] * 3)
    d = rng.choice([64, 128, 128, 128, 256])
    G = rng.choice([1, 2, 4, 4, 8])
    B = _log_int(rng, 1, 16)
    Hkv = rng.choice([4, 8, 8, 16, 32])
    sK, sV = rng.choice([0.5, 0.7, 0.8]), rng.choice([0.5, 0.7, 0.8])
    c = dict(kind=kind, B=B, Hq=Hkv * G, Hkv=Hkv, d=d)
    most = (1 << 30) // (B * Hkv * d)       # tokens per stream: up to 2 GiB of dense keys
    if kind == "attend":
        c.update(n=_log_int(rng, 600, min(131072, most)), ragged=rng.random() < 0.5, sK=sK, sV=sV, W=32)
    elif kind == "dense":
        c.update(n=_log_int(rng, 600, min(65536, most)))
    elif kind == "compress":
        mode = rng.choice(["magnitude", "magnitude", "output_aware", "two_four", "channel"])
        n = _log_int(rng, 600, max(600, min(32768, most // (8 if mode == "output_aware" else 4))))
        if mode == "channel":
            n = (n + GROUP - 1) // GROUP * GROUP
        c.update(mode=mode, n=n, sK=0.5 if mode == "two_four" else sK, sV=sV)
    else:
        loop = rng.choice(["window", "append", "channel", "output_aware_keys"])
        c.update(loop=loop, n=_log_int(rng, 300, max(300, min(4096, most // 16))), steps=rng.randint(4, 16), sK=sK, sV=sV,
                 ragged=loop != "append" and rng.random() < 0.5, W=64 if loop == "channel" else 32)
    return c


def _lengths(case):
    """Prompt tokens of every batch entry (a ragged batch spans a factor of four)."""
    B, n = case["B"], case["n"]
    if not case.get("ragged"):
        return [n] * B
    return [n - (b * 7919 % B) * (3 * n // 4) // B for b in range(B)]


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _queries(case, seed, *more):
    """fp16 N(0, 1) queries [*more][B][Hq][d]."""
    shape = (*more, case["B"], case["Hq"], case["d"])
    return torch.randn(shape, generator=_gen(seed, 23), device="cuda").half()


def _dense_kv(case, seed, n):
    """Keys (with their few outlier channels) and values, fp16 [B][Hkv][n][d]."""
    return synth.make_kv_torch(case["B"], case["Hkv"], n, case["d"], seed=int(seed))


def _bytes(nbytes):
    return torch.empty(max(int(nbytes), 16), dtype=torch.uint8, device="cuda")


def _attn_ws(case, n):
    return _bytes(mf.mustafar_attn_workspace_bytes(case["B"], case["Hq"], case["Hkv"], case["d"], n, 0))


def _compress_ws(case, n):
    return _bytes(mf.mustafar_compress_workspace_bytes(case["B"], case["Hkv"], n))


def _prompt_queries(case, seed):
    """The prompt's queries, fp16 [B][Hq][n][d]."""
    shape = (case["B"], case["Hq"], case["n"], case["d"])
    return torch.randn(shape, generator=_gen(seed, 29), device="cuda", dtype=torch.float16)


def _caches(case, n, channel=False):
    B, H, d = case["B"], case["Hkv"], case["d"]
    return (mf.CompressedCache(B, H, d, case["sK"], n),
            mf.CompressedCache(B, H, d, case["sV"], n, grouped=channel))


def prepare(case, seed):
    B, Hq, Hkv, d, n = (case[k] for k in ("B", "Hq", "Hkv", "d", "n"))
    s = dict(case=case)
    if case["kind"] == "attend":
        K, V = _dense_kv(case, seed, n)
        s["Kc"], s["Vc"] = _caches(case, n)
        s["win"] = mf.DenseWindow(B, Hkv, d, case["W"])
        mf.mustafar_window_prefill(s["win"], s["Kc"], s["Vc"], K, V, _lengths(case))
        s.update(q=_queries(case, seed), ws=_attn_ws(case, n),
                 out=torch.empty((B, Hq, d), dtype=torch.float16, device="cuda"))
    elif case["kind"] == "dense":
        s["k"], s["v"] = _dense_kv(case, seed, n)
        s.update(q=_queries(case, seed), ws=_attn_ws(case, n),
                 out=torch.empty((B, Hq, d), dtype=torch.float16, device="cuda"))
    elif case["kind"] == "compress":
        s["k"], s["v"] = _dense_kv(case, seed, n)
        s["Kc"], s["Vc"] = _caches(case, n, channel=case["mode"] == "channel")
        s["ws"] = _compress_ws(case, n)
        if case["mode"] == "output_aware":
            s["q"] = _prompt_queries(case, seed)
            s["w"] = torch.empty((B, Hkv, n, d), dtype=torch.float32, device="cuda")
    else:
        steps, W = case["steps"], case["W"]
        K, V = _dense_kv(case, seed, n + steps)
        s["k"], s["v"] = K[:, :, :n].contiguous(), V[:, :, :n].contiguous()
        s["Kc"], s["Vc"] = _caches(case, n + steps, channel=case["loop"] == "channel")
        s["q"] = _queries(case, seed, steps)
        s["ws_c"], s["ws_a"] = _compress_ws(case, n), _attn_ws(case, n + steps)
        new_k, new_v = (x[:, :, n:].permute(2, 0, 1, 3).contiguous() for x in (K, V))  # [steps][B][Hkv][d]
        s.update(new_k=new_k, new_v=new_v)
        if case["loop"] == "append":
            # the prompt's last W tokens start as the dense window; step i appends its oldest
            # token and attends with the window that follows
            s["k"], s["v"] = K[:, :, :n - W].contiguous(), V[:, :, :n - W].contiguous()
            s["old"] = [(K[:, :, n - W + i].contiguous(), V[:, :, n - W + i].contiguous()) for i in range(steps)]
            s["tail"] = [(K[:, :, n - W + i + 1:n + i + 1].contiguous(), V[:, :, n - W + i + 1:n + i + 1].contiguous())
                         for i in range(steps)]
        else:
            s["win"] = mf.DenseWindow(B, Hkv, d, W)
            s["lens"] = _lengths(case)
        if case["loop"] == "channel":
            s["acc"] = torch.empty((B, Hkv, W), dtype=torch.float32, device="cuda")
        if case["loop"] == "output_aware_keys":
            s["kacc"] = torch.empty((B, Hkv, W, d), dtype=torch.float32, device="cuda")
    return s


def _cache_out(c):
    return [c.bitmaps, c.offsets, c.values, c.stream_len]


def run(state):
    s, case = state, state["case"]
    if case["kind"] == "attend":
        return mf.mustafar_window_decode_attn(s["q"], s["Kc"], s["Vc"], s["win"], out=s["out"], ws=s["ws"])
    if case["kind"] == "dense":
        return mf.mustafar_dense_decode_attn(s["q"], s["k"], s["v"], out=s["out"], ws=s["ws"])
    Kc, Vc = s["Kc"], s["Vc"]
    Kc.desc.n_tokens = Vc.desc.n_tokens = 0        # a new request reuses the caches' buffers
    if case["kind"] == "compress":
        out = {"K": _cache_out(Kc), "V": _cache_out(Vc)}
        if case["mode"] == "output_aware":
            out["w"] = mf.mustafar_query_lookahead(s["q"], case["Hkv"], out=s["w"])
            mf.mustafar_prune_compress_ex(Kc, s["k"], mode=mf.PRUNE_OUTPUT_AWARE, weights=s["w"], ws=s["ws"])
        elif case["mode"] == "two_four":
            mf.mustafar_prune_compress_ex(Kc, s["k"], mode=mf.PRUNE_2_4, ws=s["ws"])
        else:
            mf.mustafar_prune_compress(Kc, s["k"], ws=s["ws"])
        mf.mustafar_prune_compress(Vc, s["v"], ws=s["ws"])   # per channel when the cache is
        return out
    outs, loop = [], case["loop"]
    res = {"out": outs, "K": _cache_out(Kc), "V": _cache_out(Vc)}
    if loop == "append":
        mf.mustafar_prune_compress(Kc, s["k"], ws=s["ws_c"])
        mf.mustafar_prune_compress(Vc, s["v"], ws=s["ws_c"])
        for i in range(case["steps"]):
            mf.mustafar_append_kv(Kc, Vc, *s["old"][i])
            outs.append(mf.mustafar_sparse_decode_attn(s["q"][i], Kc, Vc, *s["tail"][i], ws=s["ws_a"]))
        return res
    win = s["win"]
    for name in ("acc", "kacc"):
        if name in s:
            res[name] = s[name].zero_()
    mf.mustafar_window_prefill(win, Kc, Vc, s["k"], s["v"], s["lens"], ws=s["ws_c"])
    for i in range(case["steps"]):
        q, k, v = s["q"][i], s["new_k"][i], s["new_v"][i]
        if loop == "channel":
            mf.mustafar_window_step_grouped(win, Kc, Vc, k, v, acc=s["acc"])
            outs.append(mf.mustafar_window_decode_attn_scores(q, Kc, Vc, win, s["acc"], ws=s["ws_a"]))
        elif loop == "output_aware_keys":
            mf.mustafar_window_step_weighted(win, Kc, Vc, k, v, s["kacc"])
            outs.append(mf.mustafar_window_decode_attn(q, Kc, Vc, win, ws=s["ws_a"]))
            mf.mustafar_window_key_weights(q, win, s["kacc"])
        else:
            mf.mustafar_window_step(win, Kc, Vc, k, v)
            outs.append(mf.mustafar_window_decode_attn(q, Kc, Vc, win, ws=s["ws_a"]))
    res["state"] = [win.len, win.head, win.n_comp]
    return res


def _keep(case, side):
    """Kept channels per token (on average), and their fp16 slots with the padding of every tile to 8."""
    k = case["d"] * (1 - case["s" + side])
    return k, min(case["d"], k + 3.5 * (case["d"] // 64))


def work(case):
    """Bytes: dense inputs, bitmaps and packed values, each once, and the outputs (a tile's offset follows
    from the bitmaps before it); flops: the products with kept values."""
    B, Hq, Hkv, d, n = (case[k] for k in ("B", "Hq", "Hkv", "d", "n"))
    qo = 4 * B * Hq * d
    if case["kind"] == "dense":
        return {"bytes": 4 * B * Hkv * n * d + qo, "flops": 4 * B * Hq * n * d}
    (kk, pk), (kv, pv) = _keep(case, "K"), _keep(case, "V")
    packed = 2 * 8 * (d // 64) + 2 * (pk + pv)          # per token and kv-head, K and V
    dense = 4 * d
    meta = 2 * 4 * (d // 64)                            # offsets, written by the compression
    tokens = sum(_lengths(case)) * Hkv
    if case["kind"] == "compress":
        b = tokens * (dense + packed + meta)
        if case["mode"] == "output_aware":
            b += 2 * B * Hq * n * d + 4 * tokens * d    # queries read, weights written
        return {"bytes": b, "flops": 0}
    if case["kind"] == "attend":
        window = sum(min(L, case["W"]) for L in _lengths(case)) * Hkv
        return {"bytes": (tokens - window) * packed + window * dense + qo,
                "flops": 2 * (Hq // Hkv) * ((tokens - window) * (kk + kv) + window * 2 * d)}
    steps = case["steps"]
    attend = tokens * packed + B * Hkv * case["W"] * dense + qo
    return {"bytes": tokens * (dense + packed + meta) + steps * attend,
            "flops": steps * 2 * (Hq // Hkv) * tokens * (kk + kv)}


def tolerance(case):
    """Selections, bitmaps, offsets and packed values are whole numbers and come out the same. Attention has
    fp16 probabilities and outputs: 2.1e-4 to 2.6e-4 (2-norm) were measured against 64 bits over the listed and
    drawn cases. Lookahead weights are 32-bit sums of up to 256 terms: 2e-8 to 4e-8."""
    if case["kind"] == "compress":
        return {"rel": 2e-7} if case["mode"] == "output_aware" else "exact"
    return {"rel": 1e-3}


# ---- the same outputs in 64 bits, without the library ------------------------------------------
def _keep_count(d, s):
    return d - math.floor(s * d + 0.5)


def _pruned(x, k, dim=-1):
    """x with all but its k largest magnitudes along `dim` set to zero (ties to the lower index)."""
    n = x.shape[dim]
    if k >= n:
        return x.double()
    mag = (x.view(torch.int16).to(torch.int32) & 0x7fff) * n
    shape = [1] * x.dim()
    shape[dim] = n
    mag += torch.arange(n - 1, -1, -1, device=x.device, dtype=torch.int32).view(shape)
    if k <= 0:
        return torch.zeros_like(x, dtype=torch.float64)
    least = torch.topk(mag, k, dim=dim).values.amin(dim, keepdim=True)
    return torch.where(mag >= least, x, torch.zeros_like(x)).double()


def _attention(q, k, v):
    """q [H][G][d], k and v [H][n][d], float64: outputs [H][G][d] and probabilities [H][G][n]."""
    s = torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])
    p = torch.softmax(s, dim=-1)
    return torch.matmul(p, v), p


def exact(case, seed):
    B, Hq, Hkv, d, n = (case[k] for k in ("B", "Hq", "Hkv", "d", "n"))
    G, caches = Hq // Hkv, {"K": [None] * 4, "V": [None] * 4}
    if case["kind"] == "compress":
        if case["mode"] != "output_aware" or B * Hq * n * d > 2 * EXACT_ELEMENTS:
            return None
        w = torch.zeros((B, Hkv, n, d), dtype=torch.float64, device="cuda")
        q = _prompt_queries(case, seed).abs().view(B, Hkv, G, n, d)
        for b in range(B):
            total = torch.cumsum(q[b].double().sum(1), dim=1)      # over the positions, then windows of 32
            total = torch.cat([torch.zeros_like(total[:, :1]), total], 1)
            end = torch.clamp(torch.arange(n, device="cuda") + 32, max=n)
            w[b] = total[:, end] - total[:, :n]
        return {**caches, "w": w}
    if B * Hkv * n * d > EXACT_ELEMENTS or case.get("loop") == "output_aware_keys":
        return None
    if case["kind"] == "dense":
        K, V = _dense_kv(case, seed, n)
        q = _queries(case, seed).double().view(B, Hkv, G, d)
        return torch.stack([_attention(q[b], K[b].double(), V[b].double())[0].reshape(Hq, d) for b in range(B)])
    kK, kV, W = _keep_count(d, case["sK"]), _keep_count(d, case["sV"]), case["W"]
    if case["kind"] == "attend":
        K, V = _dense_kv(case, seed, n)
        q = _queries(case, seed).double().view(B, Hkv, G, d)
        out = torch.empty((B, Hq, d), dtype=torch.float64, device="cuda")
        for b, L in enumerate(_lengths(case)):
            c = L - min(L, W)
            k = torch.cat([_pruned(K[b, :, :c], kK), K[b, :, c:L].double()], 1)
            v = torch.cat([_pruned(V[b, :, :c], kV), V[b, :, c:L].double()], 1)
            out[b] = _attention(q[b], k, v)[0].reshape(Hq, d)
        return out
    steps, loop = case["steps"], case["loop"]
    K, V = _dense_kv(case, seed, n + steps)
    q = _queries(case, seed, steps).double().view(steps, B, Hkv, G, d)
    outs = [torch.empty((B, Hq, d), dtype=torch.float64, device="cuda") for _ in range(steps)]
    acc = torch.zeros((B, Hkv, W), dtype=torch.float64, device="cuda")
    for b, L in enumerate(_lengths(case)):
        k = torch.cat([K[b, :, :L], K[b, :, n:]], 1)       # the entry's prompt, then its new tokens
        v = torch.cat([V[b, :, :L], V[b, :, n:]], 1)
        pk = _pruned(k, kK)
        whole = (L - 1) // GROUP * GROUP
        if loop == "channel":    # no group leaves the window within the steps
            gv = v[:, :whole].reshape(Hkv, whole // GROUP, GROUP, d)
            pv = _pruned(gv, _keep_count(GROUP, case["sV"]), dim=2).reshape(Hkv, whole, d)
        else:
            pv = _pruned(v, kV)
        for i in range(steps):
            t = L + i + 1
            c = whole if loop == "channel" else max(0, t - W)
            o, p = _attention(q[i, b], torch.cat([pk[:, :c], k[:, c:t].double()], 1),
                              torch.cat([pv[:, :c], v[:, c:t].double()], 1))
            outs[i][b] = o.reshape(Hq, d)
            first = max(c, t - GROUP)
            acc[b, :, first - c:t - c] += p[:, :, first:t].sum(1)
    res = {**caches, "out": outs}
    if loop == "channel":
        res["acc"] = acc
    if loop != "append":
        res["state"] = [None] * 3
    return res
