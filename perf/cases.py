"""The work that a program using this library has it do, as cases that can be timed and checked.

Every case is one call sequence through the public binding (`paper_2504_03661_amd`): decode attention over a
product-quantized KV cache, a decoding step (append, then decode), a prompt's bulk append, or codebook training.
Shapes are those of the named workloads (`synth/workloads.py`), of the benchmarks and of the tests: 32 heads of
128 dims, grouped queries with 8 or 4 KV heads, 1K to 128K cached tokens, 4 / 3 / 2 bits per dimension
(64 x 256, 32 x 4096, 32 x 256 centroids), fp16 and fp32 contexts.

A case is a dict of plain values:

    kind                  "decode" | "step" (append n_new tokens per sequence, then decode) | "encode" | "train"
    batch, q_heads, kv_heads, subspaces, centroids, dtype ("f16" | "f32"), outliers (True: 2 % of the key
                          centroids' coordinates times 20)
    longest, shortest     cached tokens of the longest and of the shortest sequence, the others evenly between
    capacity              token capacity of the cache
    recent                rows of the full-precision window (a batch holds 0 .. recent - 1 of them)
    n_new                 tokens appended per sequence
    samples, iterations   of the training
"""
import math
import random

import numpy as np
import torch

import paper_2504_03661_amd as pq

HEAD_DIM = 128
SCALE = float(np.float32(1.0 / math.sqrt(HEAD_DIM)))
DEVICE = "cuda:0"


def _case(kind, batch, q_heads, kv_heads, subspaces, centroids, longest, shortest=None, capacity=None, recent=0,
          n_new=0, dtype="f16", outliers=False, samples=0, iterations=0):
    return {"kind": kind, "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads, "subspaces": subspaces,
            "centroids": centroids, "longest": longest, "shortest": longest if shortest is None else shortest,
            "capacity": max(1, longest + n_new) if capacity is None else capacity, "recent": recent, "n_new": n_new,
            "dtype": dtype, "outliers": outliers, "samples": samples, "iterations": iterations}


def listed():
    cases = {
        # a chat that has just begun: one decoding step of one sequence, where launches and latency are the time
        "step_1x32h_1k": _case("step", 1, 32, 32, 64, 256, 1000, capacity=4096, recent=128, n_new=1),
        # the 7B-sized layer at 32K that the benchmark's metric is quoted on
        "decode_1x32h_32k": _case("decode", 1, 32, 32, 64, 256, 32768, recent=128),
        # the same layer serving eight long sequences with recent windows of different lengths
        "decode_8x32h_32k": _case("decode", 8, 32, 32, 64, 256, 32768, recent=256),
        # grouped queries over one very long document, key channels with outliers
        "decode_1x32q8kv_128k": _case("decode", 1, 32, 8, 64, 256, 131072, recent=128, outliers=True),
        # serving a grouped-query model: eight sequences of different lengths, one new token each
        "step_8x32q8kv_ragged": _case("step", 8, 32, 8, 64, 256, 20011, shortest=2503, capacity=24576, recent=64,
                                      n_new=1),
        # the 2-bit setting at its largest: 64 tokens of each sequence leave the window, then the step attends
        "step_16x32h_64k_2bit": _case("step", 16, 32, 32, 32, 256, 65472, n_new=64),
        # a full-precision (fp32) program: a window's worth of tokens appended, then attended
        "step_2x32h_16k_f32": _case("step", 2, 32, 32, 64, 256, 16001, shortest=9001, capacity=16384, recent=64,
                                    n_new=96, dtype="f32"),
        # many short conversations at once
        "decode_64x32h_4k_ragged": _case("decode", 64, 32, 32, 64, 256, 4001, shortest=97, capacity=4096, recent=128),
        # the 3-bit setting (12-bit codes), one decoding step of one long sequence
        "step_1x32h_32k_12bit": _case("step", 1, 32, 32, 32, 4096, 32700, capacity=32768, recent=128, n_new=1),
        # the 3-bit setting with grouped queries, a small batch
        "decode_4x32q8kv_32k_12bit": _case("decode", 4, 32, 8, 32, 4096, 31999, shortest=20011, capacity=32768,
                                           recent=32),
        # a 32K prompt enters the cache
        "encode_1x32h_32k": _case("encode", 1, 32, 32, 64, 256, 0, n_new=32768),
        # codebooks trained on sampled activations
        "train_32h_64k": _case("train", 1, 32, 32, 64, 256, 0, capacity=64, samples=65536, iterations=2),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["decode", "decode", "step", "step", "encode", "train"])
    subspaces, centroids = rng.choice([(64, 256), (64, 256), (32, 256), (32, 4096)])
    dtype = "f16" if centroids == 4096 or kind == "train" or rng.random() < 0.75 else "f32"
    q_heads, kv_heads = rng.choice([(32, 32), (32, 32), (32, 8), (28, 4), (40, 8), (64, 8)])
    if kind == "train":
        samples = max(centroids, _log_int(rng, 1000, 65536))
        if centroids == 4096:                       # sixteen times the distances per sample
            samples = max(4096, samples // 8)
        return _case("train", 1, q_heads, min(kv_heads, 16), subspaces, centroids, 0, capacity=64, samples=samples,
                     iterations=rng.randint(1, 2))
    if kind == "encode":
        batch = _log_int(rng, 1, 8)
        most = 262144 // (batch * kv_heads) // (16 if centroids == 4096 else 2 if dtype == "f32" else 1)
        n_new = _log_int(rng, 65, max(66, min(32768, most)))
        return _case("encode", batch, q_heads, kv_heads, subspaces, centroids, 0, capacity=n_new + rng.randint(0, 500),
                     n_new=n_new, dtype=dtype)
    batch = _log_int(rng, 1, 64)
    longest = _log_int(rng, 200, 131072)
    longest = max(200, min(longest, (8 << 20) // (batch * q_heads) // (2 if dtype == "f32" else 1)))
    shortest = longest if rng.random() < 0.4 else rng.randint(max(1, longest // 16), longest)
    recent = rng.choice([0, 16, 64, 128, 200])
    n_new = rng.choice([1, 1, 2, 5, 16, 64]) if kind == "step" else 0
    if centroids == 4096:
        n_new = min(n_new, 16)
    return _case(kind, batch, q_heads, kv_heads, subspaces, centroids, longest, shortest=shortest,
                 capacity=longest + n_new + rng.choice([0, 0, 1000]), recent=recent, n_new=n_new, dtype=dtype,
                 outliers=rng.random() < 0.2)


# ---- inputs ------------------------------------------------------------------------------------------------------

def _spread(lo, hi, n):
    return [hi] if n == 1 else [lo + (hi - lo) * k // (n - 1) for k in range(n)]


def _lengths(case, seed):
    """Cached tokens and recent rows of every sequence: the same set for every seed, dealt out differently."""
    rng = random.Random(seed)
    ctx = _spread(case["shortest"], case["longest"], case["batch"])
    rec = _spread(0, case["recent"] - 1, case["batch"]) if case["batch"] > 1 and case["recent"] else \
        [case["recent"]] * case["batch"]
    rng.shuffle(ctx)
    rng.shuffle(rec)
    return ctx, rec


def _draw_inputs(case, seed):
    """All tensors of a case in their logical layouts, on the GPU.  Keys follow per-channel scales between one
    half and two (a few channels larger than the rest); the centroids come from the same distribution as the
    vectors, as trained ones do; codes are uniform."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    dt = torch.float16 if case["dtype"] == "f16" else torch.float32
    B, Hq, Hkv, M, C = (case[k] for k in ("batch", "q_heads", "kv_heads", "subspaces", "centroids"))
    ds = HEAD_DIM // M

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32)

    t = {}
    chan = torch.exp2(2.0 * torch.rand((Hkv, HEAD_DIM), generator=gen, device=DEVICE) - 1.0)
    if case["kind"] == "train":
        x = (normal(Hkv, case["samples"], HEAD_DIM) * chan[:, None, :]).to(dt)
        t["samples"] = x
        t["init"] = x[:, :C].reshape(Hkv, C, M, ds).transpose(1, 2).contiguous()
        return t
    kcb = normal(Hkv, M, C, ds) * chan.view(Hkv, M, 1, ds)
    if case["outliers"]:
        kcb = torch.where(torch.rand(kcb.shape, generator=gen, device=DEVICE) < 0.02, kcb * 20.0, kcb)
    t["k_codebook"] = kcb.to(dt)
    t["v_codebook"] = normal(Hkv, M, C, ds).to(dt)
    t["q"] = normal(B, Hq, HEAD_DIM).to(dt)
    ctx, rec = _lengths(case, seed)
    t["ctx_len"] = torch.tensor(ctx, dtype=torch.int32, device=DEVICE)
    t["recent_len"] = torch.tensor(rec, dtype=torch.int32, device=DEVICE)
    if case["longest"]:
        for n in ("k_codes", "v_codes"):
            t[n] = torch.randint(0, C, (B, Hkv, case["longest"], M), generator=gen, device=DEVICE,
                                 dtype=torch.uint8 if C <= 256 else torch.int16)
    if case["recent"]:
        rows = (B, Hkv, case["recent"], HEAD_DIM)
        t["recent_k"] = (normal(*rows) * chan[None, :, None, :]).to(dt)
        t["recent_v"] = normal(*rows).to(dt)
    if case["n_new"]:
        rows = (B, Hkv, case["n_new"], HEAD_DIM)
        t["new_k"] = (normal(*rows) * chan[None, :, None, :]).to(dt)
        t["new_v"] = normal(*rows).to(dt)
    return t


class _State:
    """What the program keeps between calls: the library's context, the cache, the operands of the call."""

    def __init__(self, case, seed):
        self.kind, self.iterations = case["kind"], case["iterations"]
        t = _draw_inputs(case, seed)
        cfg = pq.PQAttnConfig(batch=case["batch"], n_q_heads=case["q_heads"], n_kv_heads=case["kv_heads"],
                              head_dim=HEAD_DIM, n_subspaces=case["subspaces"], n_centroids=case["centroids"],
                              max_context=case["capacity"], max_recent=case["recent"],
                              dtype=pq.PQ_F16 if case["dtype"] == "f16" else pq.PQ_F32, device=0, n_splits=0)
        self.ctx = pq.pq_attn_create(cfg)
        if self.kind == "train":
            self.samples, self.init = t["samples"], t["init"]
            self.n_samples = case["samples"]
            self.codebook = torch.empty_like(self.init)
            self.workspace_bytes = pq.pq_kmeans_workspace_bytes(self.ctx)
            self.workspace = torch.empty(self.workspace_bytes, dtype=torch.uint8, device=DEVICE)
            return
        for name in ("q", "recent_k", "recent_v", "new_k", "new_v"):
            setattr(self, name, t.get(name))
        self.recent_len = t["recent_len"] if case["recent"] else None
        self.start_len, self.ctx_len = t["ctx_len"], t["ctx_len"].clone()
        self.n_new = case["n_new"]
        self.out = torch.empty((case["batch"], case["q_heads"], HEAD_DIM), dtype=torch.float32, device=DEVICE)
        pq.pq_attn_set_codebooks(self.ctx, t["k_codebook"], t["v_codebook"])
        n_bytes = pq.pq_attn_codes_bytes(cfg)
        self.k_codes = torch.zeros(n_bytes, dtype=torch.uint8, device=DEVICE)
        self.v_codes = torch.zeros(n_bytes, dtype=torch.uint8, device=DEVICE)
        if case["longest"]:
            pq.pq_pack_codes(self.ctx, pq.PQ_CODES_K, t["k_codes"], case["longest"], self.k_codes)
            pq.pq_pack_codes(self.ctx, pq.PQ_CODES_V, t["v_codes"], case["longest"], self.v_codes)
        torch.cuda.synchronize()                    # the tensors of `t` that are not kept are released now

    def __del__(self):
        if getattr(self, "ctx", None):
            pq.pq_attn_destroy(self.ctx)
            self.ctx = None


def prepare(case, seed):
    return _State(case, seed)


def run(s):
    if s.kind == "train":
        s.codebook.copy_(s.init)                    # training works in place
        pq.pq_kmeans_fit(s.ctx, s.samples, s.n_samples, s.codebook, s.iterations, s.workspace, s.workspace_bytes)
        return s.codebook
    if s.n_new:
        s.ctx_len.copy_(s.start_len)                # the pass appends at the same place every time
        pq.pq_encode_append(s.ctx, s.new_k, s.new_v, s.n_new, None, None, s.k_codes, s.v_codes, s.ctx_len)
    if s.kind == "encode":
        return s.k_codes, s.v_codes, s.ctx_len
    pq.pq_attn_decode(s.ctx, s.q, s.k_codes, s.v_codes, s.ctx_len, None, None, s.recent_k, s.recent_v, s.recent_len,
                      SCALE, s.out)
    return (s.out, s.k_codes, s.v_codes, s.ctx_len) if s.kind == "step" else s.out


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def work(case):
    B, Hq, Hkv, M, C = (case[k] for k in ("batch", "q_heads", "kv_heads", "subspaces", "centroids"))
    eb = 2 if case["dtype"] == "f16" else 4
    books = Hkv * C * HEAD_DIM * eb                 # one codebook set (K or V)
    code_bytes = M if C == 256 else 48
    nearest = 2 * C * HEAD_DIM                      # flops: one vector's products with every centroid
    if case["kind"] == "train":
        vectors = Hkv * case["samples"]
        return {"bytes": case["iterations"] * (vectors * HEAD_DIM * eb + 2 * books),
                "flops": case["iterations"] * vectors * nearest}
    n_bytes, flops = 2 * books, 0
    if case["n_new"]:
        vectors = 2 * B * Hkv * case["n_new"]
        n_bytes += vectors * (HEAD_DIM * eb + code_bytes)
        flops += vectors * nearest
    if case["kind"] != "encode":
        ctx, rec = _lengths(case, 0)
        cached = sum(ctx) + B * case["n_new"]
        rows = sum(rec)
        n_bytes += cached * Hkv * 2 * code_bytes + rows * Hkv * 2 * HEAD_DIM * eb + B * Hq * HEAD_DIM * (eb + 4)
        # per (token, query head): one addition per subspace, 128 multiply-adds of the values; per recent row two
        # products of 128; per (sequence, query head) the table q . C
        flops += cached * Hq * (M + 2 * HEAD_DIM) + rows * Hq * 4 * HEAD_DIM + B * Hq * 2 * C * HEAD_DIM
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    # Codes and trained centroids are decided in IEEE double with fixed tie rules: the same bits from every
    # implementation.  Decode sums in fp32, in an order that varies from call to call: 1e-7 to 6e-7 from `exact` over
    # these cases, up to 5e-7 between two calls on the same inputs; two implementations may be 1e-6 apart.
    if case["kind"] in ("encode", "train"):
        return "exact"
    return {"rel": 5e-6}


# ---- the same results in 64 bits ---------------------------------------------------------------------------------

def _nearest(x, codebook):
    """Index of the nearest centroid: x [n, M, ds], codebook [M, C, ds], both float64 -> [n, M] int64."""
    M, C, _ = codebook.shape
    out = torch.empty(x.shape[:2], dtype=torch.int64, device=x.device)
    step = max(1, (1 << 27) // (M * C))
    for t0 in range(0, x.shape[0], step):
        d = ((x[t0:t0 + step, :, None, :] - codebook[None]) ** 2).sum(-1)
        out[t0:t0 + step] = torch.argmin(d, dim=-1)
    return out


def _gather(codebook, codes):
    """Vectors named by codes: codebook [M, C, ds], codes [n, M] -> [n, M * ds]."""
    M, C, ds = codebook.shape
    flat = codes + torch.arange(M, device=codes.device) * C
    return codebook.reshape(M * C, ds)[flat].reshape(codes.shape[0], M * ds)


def _exact_train(case, t):
    samples, cb = t["samples"].double(), t["init"].double()
    Hkv, M, C, ds = cb.shape
    means = cb
    for _ in range(case["iterations"]):
        means = cb.clone()
        for h in range(Hkv):
            x = samples[h].reshape(-1, M, ds)
            codes = _nearest(x, cb[h]) + torch.arange(M, device=x.device) * C
            sums = torch.zeros((M * C, ds), dtype=torch.float64, device=x.device)
            sums.index_add_(0, codes.reshape(-1), x.reshape(-1, ds))
            count = torch.bincount(codes.reshape(-1), minlength=M * C).double()[:, None]
            means[h] = torch.where(count > 0, sums / count.clamp(min=1), cb[h].reshape(M * C, ds)).reshape(M, C, ds)
        cb = means.float().half().double()          # the codebook that an iteration leaves is fp16
    return means


def exact(case, seed):
    # code bytes (None below) are in the cache's own layout; they are compared bit for bit
    if case["kind"] == "encode":
        return None, None, torch.full((case["batch"],), case["n_new"], dtype=torch.int64)
    t = _draw_inputs(case, seed)
    if case["kind"] == "train":
        distances = case["iterations"] * case["samples"] * case["kv_heads"] * case["subspaces"] * case["centroids"]
        return None if distances > 2 ** 37 else _exact_train(case, t)
    B, Hq, Hkv, M, n_new = (case[k] for k in ("batch", "q_heads", "kv_heads", "subspaces", "n_new"))
    G, ds = Hq // Hkv, HEAD_DIM // M
    kcb, vcb = t["k_codebook"].double(), t["v_codebook"].double()
    q = t["q"].double() * SCALE
    out = torch.zeros((B, Hq, HEAD_DIM), dtype=torch.float64, device=DEVICE)
    ctx, rec = t["ctx_len"].tolist(), t["recent_len"].tolist()
    for b in range(B):
        for h in range(Hkv):
            k = _gather(kcb[h], t["k_codes"][b, h, :ctx[b]].long())
            v = _gather(vcb[h], t["v_codes"][b, h, :ctx[b]].long())
            if n_new:
                nk = t["new_k"][b, h].double().reshape(n_new, M, ds)
                nv = t["new_v"][b, h].double().reshape(n_new, M, ds)
                k = torch.cat([k, _gather(kcb[h], _nearest(nk, kcb[h]))])
                v = torch.cat([v, _gather(vcb[h], _nearest(nv, vcb[h]))])
            if case["recent"]:
                k = torch.cat([k, t["recent_k"][b, h, :rec[b]].double()])
                v = torch.cat([v, t["recent_v"][b, h, :rec[b]].double()])
            p = torch.softmax(q[b, h * G:(h + 1) * G] @ k.T, dim=-1)
            out[b, h * G:(h + 1) * G] = p @ v
    if case["kind"] == "decode":
        return out
    return out, None, None, t["ctx_len"].long() + n_new
