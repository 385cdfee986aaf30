"""Performance cases of the MoE expert stage: what a user of the package has it do.

Every case goes through the package's public entry points, over the shapes of the
workloads this repository is built around (tiny, Mixtral-8x7B, Phi-3.5-MoE and the
fine-grained layer with a shared expert) and generic sizes between and around them:

  hits     one decode token, its cache-hit experts (expert_ffn_hits)
  decode   one decode token through whole layers, every expert resident (Runtime)
  lru      a few decode tokens through whole layers with an LRU or FIFO cache smaller than
           the layer, misses on the host and post-fetched (Runtime)
  tokens   a small decode batch, every expert resident (expert_ffn_tokens)
  router   gating of a batch of tokens alone (router_topk)
  prefill  a prompt through one layer, every expert resident (prefill_forward)

listed() are the fixed cases, draw() gives others of the same ranges, prepare() makes
what a program holds before the call, run() is one pass, work() what a pass cannot do
without, tolerance() how far two correct implementations may differ, and exact() the
same results in 64 bits with plain torch.
"""
import math

import numpy as np
import torch

import paper_2512_16473_amd as moe

DEV = "cuda"

MIXTRAL = dict(d=4096, f=14336, n=8, k=2)
PHI = dict(d=4096, f=6400, n=16, k=2)
FINE = dict(d=3584, f=2560, n=64, k=8)


def listed():
    return [
        # The smallest call: two hit experts of the tiny layer. Latency and launches.
        dict(name="hits-tiny", kind="hits", d=256, f=512, slots=4, hits=2),
        # One of two selected Phi experts is in the 6-way cache: the usual partial hit.
        dict(name="hits-phi-1", kind="hits", d=4096, f=6400, slots=6, hits=1),
        # Batch-1 decode with all experts in HBM, the two widths of expert: whole layers,
        # routing read back by the host each layer as in generation.
        dict(name="decode-mixtral", kind="decode", layers=2, f_shared=0, **MIXTRAL),
        dict(name="decode-fine", kind="decode", layers=2, f_shared=20480, **FINE),
        # Decode on a memory budget, the paper's setting: 6 of 16 experts cached per
        # layer, misses on the host threads and copied in over PCIe.
        dict(name="lru-phi", kind="lru", layers=2, f_shared=0, ways=6, tokens=8, policy="lru", **PHI),
        # Small decode batches (several users, speculative tokens), odd and full size.
        dict(name="tokens-mixtral-5", kind="tokens", T=5, **MIXTRAL),
        dict(name="tokens-fine-8", kind="tokens", T=8, **FINE),
        # Gating alone for a batch, e.g. for expert-load statistics or a hit-rate study.
        dict(name="router-fine-1500", kind="router", T=1500, d=3584, n=64, k=8),
        # A short prompt or a continued one: fewer tokens than fill a tile per expert.
        dict(name="prefill-phi-27", kind="prefill", T=27, **PHI),
        # The benchmark's 512-token prompt.
        dict(name="prefill-mixtral-512", kind="prefill", T=512, **MIXTRAL),
        # A ragged prompt over many small experts.
        dict(name="prefill-fine-1333", kind="prefill", T=1333, **FINE),
        # A long prompt: the matrix cores' regime, and the largest case.
        dict(name="prefill-mixtral-4096", kind="prefill", T=4096, **MIXTRAL),
    ]


# ------------------------------------------------------------------ drawn cases
_MAX_POOL = 2.83e9      # bytes of experts in a drawn case (one Mixtral layer)
_MAX_FLOPS = 2.8e12     # of a drawn prompt (below the long Mixtral one)


def _log(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], spread evenly over its logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + step * 0.99)))
    return min(hi, max(lo, int(v // step) * step))


def draw(rng):
    kind = rng.choice(["hits", "decode", "tokens", "router", "prefill", "prefill", "lru"])
    if kind == "hits":
        c = dict(kind=kind, d=_log(rng, 256, 8192, 8), f=_log(rng, 256, 14336, 8), hits=rng.randint(1, 8))
        c["slots"] = c["hits"] + rng.randint(0, 4)
        while c["slots"] * 6.0 * c["d"] * c["f"] > _MAX_POOL:
            c["f"] = c["f"] // 2 // 8 * 8
        return c
    n = rng.choice([4, 8, 12, 16, 32, 60, 64, 128])
    k = rng.randint(1, min(8, n // 2))
    if kind == "router":
        return dict(kind=kind, T=_log(rng, 1, 4096), d=_log(rng, 256, 4096, 8), n=n, k=k)
    step = 128 if kind == "prefill" else 8
    c = dict(kind=kind, d=_log(rng, 256, 4096, step), f=_log(rng, 512, 14336, step), n=n, k=k)
    layers = 2 if kind in ("decode", "lru") else 1
    cap = _MAX_POOL if kind != "lru" else _MAX_POOL / 2   # the host side of it is touched page by page
    while layers * n * 6.0 * c["d"] * c["f"] > cap:
        c["f"] = max(step, c["f"] // 2 // step * step)
        if c["f"] <= 4 * step:
            c["d"] = max(step, c["d"] // 2 // step * step)
    if kind == "prefill":
        c["T"] = _log(rng, 1, 4096)
        while 6.0 * c["T"] * k * c["d"] * c["f"] > _MAX_FLOPS:
            c["T"] //= 2
    elif kind == "tokens":
        c["T"] = rng.randint(1, 8)
    else:
        c["layers"] = layers
        c["f_shared"] = rng.choice([0, _log(rng, 512, 8192, 8)])
        if kind == "lru":
            c["ways"] = rng.randint(k, max(k, n // 2))
            c["tokens"] = rng.randint(2, 8)
            c["policy"] = rng.choice(["lru", "fifo"])
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    return g


def _pool(g, d, f, n):
    """n expert slabs (bf16 W1 [f][d] | W3 [f][d] | W2 [d][f]) at the library's stride."""
    std = 0.02 if d >= 1024 else d ** -0.5
    stride = moe.slab_bytes(d, f)
    pool = torch.empty(n * stride // 2, dtype=torch.bfloat16, device=DEV)
    pool.normal_(0.0, std, generator=g)
    return pool.view(torch.uint8)


def _router(g, n, d, layers=None):
    shape = (n, d) if layers is None else (layers, n, d)
    return torch.empty(shape, device=DEV).normal_(0.0, d ** -0.5, generator=g)


def _states(g, *shape):
    return torch.empty(shape, device=DEV).normal_(0.0, 1.0, generator=g)


def _ar1(g, T, *shape):
    """Correlated decode states x_t = 0.9 x_{t-1} + 0.436 eps_t, [T][shape]."""
    x = _states(g, T, *shape)
    for t in range(1, T):
        x[t] = 0.9 * x[t - 1] + 0.436 * x[t]
    return x


def _gates(g, T, k):
    w = torch.empty((T, k), device=DEV).uniform_(0.2, 1.0, generator=g)
    return w / w.sum(dim=1, keepdim=True)


def _distinct(g, T, n, k):
    """[T][k] distinct ids in [0, n), uniformly."""
    r = torch.empty((T, n), device=DEV).uniform_(generator=g)
    return torch.topk(r, k, dim=1).indices.to(torch.int32).contiguous()


def _inputs(case, seed):
    """The tensors of a case, from the seed alone (prepare and exact draw the same)."""
    g = _gen(seed)
    c, kind, s = case, case["kind"], {}
    d = c["d"]
    if kind == "hits":
        s["pool"] = _pool(g, d, c["f"], c["slots"])
        s["x"] = _states(g, d)
        s["slots"] = _distinct(g, 1, c["slots"], c["hits"])[0].contiguous()
        s["w"] = _gates(g, 1, c["hits"])[0].contiguous()
    elif kind == "tokens":
        s["pool"] = _pool(g, d, c["f"], c["n"])
        s["x"] = _ar1(g, c["T"], d)
        s["slots"] = _distinct(g, c["T"], c["n"], c["k"])
        s["w"] = _gates(g, c["T"], c["k"])
    elif kind == "router":
        s["wr"] = _router(g, c["n"], d)
        s["x"] = _states(g, c["T"], d)
    elif kind == "prefill":
        s["wr"] = _router(g, c["n"], d)
        s["pool"] = _pool(g, d, c["f"], c["n"])
        s["x"] = _states(g, c["T"], d)
    else:   # decode, lru
        L = c["layers"]
        s["wr"] = _router(g, c["n"], d, L)
        s["pool"] = _pool(g, d, c["f"], L * c["n"])
        s["shared"] = _pool(g, d, c["f_shared"], L) if c["f_shared"] else None
        s["x"] = _ar1(g, c.get("tokens", 1), L, d)
    return s


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = _inputs(case, seed)
    d, f = c["d"], c.get("f", 0)
    s["case"] = case
    if kind == "hits":
        s["y"] = torch.empty(d, device=DEV)
        s["ws"] = torch.empty(moe.ffn_workspace_bytes(c["hits"], d, f), dtype=torch.uint8, device=DEV)
    elif kind == "tokens":
        s["y"] = torch.empty((c["T"], d), device=DEV)
        s["ws"] = torch.empty(moe.ffn_tokens_workspace_bytes(c["T"], c["k"], d, f), dtype=torch.uint8, device=DEV)
    elif kind in ("router", "prefill"):
        s["idx"] = torch.empty((c["T"], c["k"]), dtype=torch.int32, device=DEV)
        s["w"] = torch.empty((c["T"], c["k"]), device=DEV)
        if kind == "prefill":
            s["y"] = torch.empty((c["T"], d), device=DEV)
            s["ws"] = torch.empty(moe.prefill_workspace_bytes(d, f, c["n"], c["k"], c["T"]), dtype=torch.uint8,
                                  device=DEV)
    else:
        _prepare_runtime(s, c, d, f, kind)
    torch.cuda.synchronize()
    return s


def _prepare_runtime(s, c, d, f, kind):
    L, n, k = c["layers"], c["n"], c["k"]
    stride = moe.slab_bytes(d, f)
    # the experts' home: pinned host memory
    host = moe.PinnedBuffer(L * n * stride)
    torch.from_numpy(host.array).copy_(s["pool"])
    s["host"] = host
    if kind == "decode":
        # every expert has its slot; the runtime loads them at creation
        ways = n
        cache = moe.Cache(L, n, ways, k, "static", np.tile(np.arange(n, dtype=np.int32), (L, 1)))
    else:
        ways = c["ways"]
        cache = moe.Cache(L, n, ways, k, c["policy"])
        # pages drawn by DMA have not been touched by the CPU; a program that read its
        # weights from disk has touched them all
        s["touched"] = int(host.array[::4096].sum())
    slots = torch.empty(L * ways * stride, dtype=torch.uint8, device=DEV)
    del s["pool"]
    s["slot_pool"], s["cache"] = slots, cache
    s["hp"] = moe.HostPool(min(16, _cpus()))
    s["rt"] = moe.Runtime(d, f, n, k, ways, L, s["wr"], slots, [host.ptr + i * stride for i in range(L * n)],
                          cache, s["hp"], f_shared=c["f_shared"], shared_pool=s["shared"])
    s["copy"] = torch.cuda.Stream()
    T = c.get("tokens", 1)
    s["y"] = torch.empty((T, L, d), device=DEV)
    s["idx"] = np.empty((T, L, k), np.int32)
    s["w"] = np.empty((T, L, k), np.float32)


def _cpus():
    import os
    return len(os.sched_getaffinity(0))


# ------------------------------------------------------------------ one pass
def run(s):
    c = s["case"]
    kind, d = c["kind"], c["d"]
    if kind == "hits":
        return moe.expert_ffn_hits(s["x"], s["pool"], c["slots"], s["slots"], s["w"], d, c["f"], s["y"], s["ws"])
    if kind == "tokens":
        return moe.expert_ffn_tokens(s["x"], s["pool"], c["n"], s["slots"], s["w"], d, c["f"], s["y"], s["ws"])
    if kind == "router":
        return moe.router_topk(s["x"], s["wr"], c["k"], idx_out=s["idx"], w_out=s["w"])
    if kind == "prefill":
        moe.prefill_forward(s["x"], s["wr"], s["pool"], d, c["f"], c["n"], c["k"], s["y"], s["ws"], idx=s["idx"],
                            w=s["w"])
        return s["y"], s["idx"], s["w"]
    # The compute stream is the program's current one, the copies have their own. Which
    # experts hit depends on the passes before (the cache lives on), so the hit mask is not
    # an output; routing and layer outputs do not depend on it.
    streams = (None, None, s["copy"])
    for t in range(s["x"].shape[0]):
        s["rt"].decode_step(s["x"][t], s["y"][t], streams, idx=s["idx"][t], w=s["w"][t])
    return s["y"], s["idx"], s["w"]


# ------------------------------------------------------------------ floors and tolerances
def _touched(n, k, T):
    """Expected distinct experts of T tokens that each pick k of n."""
    return n * (1.0 - (1.0 - k / n) ** T)


def work(case):
    c, kind = case, case["kind"]
    d, f = c["d"], c.get("f", 0)
    slab = 6.0 * d * f
    if kind == "hits":
        return {"bytes": c["hits"] * slab + 8.0 * d, "flops": c["hits"] * slab}
    if kind == "tokens":
        return {"bytes": _touched(c["n"], c["k"], c["T"]) * slab + 8.0 * c["T"] * d,
                "flops": c["T"] * c["k"] * slab}
    if kind == "router":
        return {"bytes": 4.0 * d * (c["T"] + c["n"]) + 8.0 * c["T"] * c["k"], "flops": 2.0 * c["T"] * c["n"] * d}
    if kind == "prefill":
        return {"bytes": _touched(c["n"], c["k"], c["T"]) * slab + 8.0 * c["T"] * d + 4.0 * c["n"] * d,
                "flops": c["T"] * (c["k"] * slab + 2.0 * c["n"] * d)}
    # whole layers: the selected and the shared experts of each token, wherever they run
    # (of an LRU layer's experts the missed ones also cross PCIe, which bounds that case)
    per = c["k"] * slab + 6.0 * d * c["f_shared"] + 4.0 * c["n"] * d + 8.0 * d
    m = c["layers"] * c.get("tokens", 1)
    return {"bytes": m * per, "flops": m * (c["k"] * slab + 6.0 * d * c["f_shared"] + 2.0 * c["n"] * d)}


def tolerance(case):
    """About four times the distance from the 64-bit results that the paths showed."""
    if case["kind"] == "prefill":
        # hidden states and activations rounded to bf16 for the matrix cores: 2.9e-3
        return {"rel": 1.2e-2, "max": 6e-2, "differ": 0.0}
    if case["kind"] == "router":
        # fp64 logits, fp32 gate weights: 2.5e-8
        return {"rel": 1.2e-7, "max": 1e-6, "differ": 0.0}
    if case["kind"] == "tokens":
        # fp32 activations as two bf16 parts: 4.4e-6
        return {"rel": 1.8e-5, "max": 1e-4, "differ": 0.0}
    # fp32 activations and sums: 2.6e-7 on the GPU, and the host path sums in another order
    return {"rel": 2e-6, "max": 2e-5, "differ": 0.0}


# ------------------------------------------------------------------ 64-bit results
def _expert64(slab, d, f, x):
    """SwiGLU expert on x [m][d] (fp64); slab uint8."""
    w = slab[:6 * d * f].view(torch.bfloat16)
    g = x @ w[:f * d].view(f, d).double().t()
    u = x @ w[f * d:2 * f * d].view(f, d).double().t()
    h = g / (1.0 + torch.exp(-g)) * u
    return h @ w[2 * f * d:3 * f * d].view(d, f).double().t()


def _route64(x, wr, k):
    top = torch.topk(x @ wr.double().t(), k, dim=1)
    return top.indices, torch.softmax(top.values, dim=1)


def _moe64(x, pool, d, f, n, idx, w):
    """sum_j w[t][j] expert idx[t][j] (x[t]) over tokens x [T][d] (fp64)."""
    stride = moe.slab_bytes(d, f)
    y = torch.zeros_like(x)
    for e in range(n):
        t, j = (idx == e).nonzero(as_tuple=True)
        if t.numel():
            ye = _expert64(pool[e * stride:(e + 1) * stride], d, f, x[t])
            y.index_put_((t,), w[t, j].double()[:, None] * ye, accumulate=True)
    return y


def exact(case, seed):
    c, kind = case, case["kind"]
    s = _inputs(case, seed)
    d, f = c["d"], c.get("f", 0)
    if kind == "hits":
        return _moe64(s["x"][None].double(), s["pool"], d, f, c["slots"], s["slots"][None], s["w"][None])[0]
    if kind == "tokens":
        return _moe64(s["x"].double(), s["pool"], d, f, c["n"], s["slots"], s["w"])
    if kind in ("router", "prefill"):
        x = s["x"].double()
        idx, w = _route64(x, s["wr"], c["k"])
        if kind == "router":
            return idx, w
        return _moe64(x, s["pool"], d, f, c["n"], idx, w), idx, w
    L, n, k = c["layers"], c["n"], c["k"]
    stride = moe.slab_bytes(d, f)
    x = s["x"].double()
    y = torch.empty_like(x)
    idx = np.empty((x.shape[0], L, k), np.int64)
    w = np.empty((x.shape[0], L, k), np.float64)
    for l in range(L):
        xl = x[:, l].contiguous()
        il, wl = _route64(xl, s["wr"][l], k)
        idx[:, l], w[:, l] = il.cpu().numpy(), wl.cpu().numpy()
        yl = _moe64(xl, s["pool"][l * n * stride:(l + 1) * n * stride], d, f, n, il, wl)
        if s["shared"] is not None:
            ss = moe.slab_bytes(d, c["f_shared"])
            yl = yl + _expert64(s["shared"][l * ss:(l + 1) * ss], d, c["f_shared"], xl)
        y[:, l] = yl
    return y, idx, w
