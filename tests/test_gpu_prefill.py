"""Prefill path (all experts resident, T tokens, grouped MFMA GEMMs) vs the oracle.

The oracle evaluates each token through the same layer definition as decode (router,
chosen SwiGLU experts, combine). The GPU rounds the hidden states and the SwiGLU
activations to bf16 for the matrix cores (fp32 accumulation), so its error is that of
bf16 activations: ~1e-3 x RMS per element, within the 2e-2 x RMS bound.
"""
import os

import numpy as np
import pytest

import oracle
import synth
from _gpu_util import TOL, rel_err, router_parity, say, torch_cuda
from _tile_plan import prefill_plans

pytestmark = pytest.mark.gpu


def _run(torch, X, wr, pool, d, f, n, k):
    import paper_2512_16473_amd as moe
    T = X.shape[0]
    ws = torch.empty(max(256, moe.prefill_workspace_bytes(d, f, n, k, T)), dtype=torch.uint8, device="cuda")
    Xd = torch.from_numpy(X).cuda()
    out = torch.full((T, d), float("nan"), device="cuda")
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.zeros((T, k), device="cuda")
    moe.prefill_forward(Xd, torch.from_numpy(wr).cuda(), pool, d, f, n, k, out, ws, idx=idx, w=w)
    torch.cuda.synchronize()
    return out.cpu().numpy(), idx.cpu().numpy(), w.cpu().numpy()


def _bf16_activation_ref(x, slabs, idx, w, d, f):
    """Test-side reference: x and h rounded to bf16 (RNE), everything else fp64."""
    xb = synth.bf16_to_f32(synth.bf16_bits(x)).astype(np.float64)
    y = np.zeros(d)
    for e, we in zip(idx, w):
        W = synth.bf16_to_f32(slabs[e]).astype(np.float64)
        w1, w3, w2 = W[: f * d].reshape(f, d), W[f * d: 2 * f * d].reshape(f, d), W[2 * f * d:].reshape(d, f)
        g, u = w1 @ xb, w3 @ xb
        h = (g / (1.0 + np.exp(-g)) * u).astype(np.float32)
        hb = synth.bf16_to_f32(synth.bf16_bits(h)).astype(np.float64)
        y += float(we) * (w2 @ hb)
    return y


def _pool_np(torch, slabs, d, f):
    import paper_2512_16473_amd as moe
    stride = moe.slab_bytes(d, f)
    pool = torch.zeros(len(slabs) * stride, dtype=torch.uint8)
    for i, s in enumerate(slabs):
        pool[i * stride: i * stride + s.nbytes] = torch.from_numpy(s.view(np.uint8))
    return pool.cuda()


# (256, 512, 4, 2, 700): ~350 tokens per expert (two M tiles) and 128 pairs per wave of the
# grouping; (384, 640, ...): d not a multiple of 256 (a last down tile of 128 rows). Gate/up
# tiles are all whole here, K being short; down tiles are split over K: (512, 1024, 8, 2, 300)
# and (256, 1024, 16, 2, 520) in 4 parts, (384, 640, 16, 4, 130) in 2, (256, 5120, 8, 2, 256)
# in 16. test_prefill_split_plans covers the other plans.
@pytest.mark.parametrize("d,f,n,k,T", [(256, 512, 4, 2, 64), (256, 512, 4, 2, 37), (512, 1024, 8, 2, 300),
                                       (384, 640, 16, 4, 130), (256, 256, 8, 1, 1), (256, 512, 64, 8, 48),
                                       (256, 512, 4, 2, 700), (256, 5120, 8, 2, 256), (256, 1024, 16, 2, 520)])
def test_prefill_small(d, f, n, k, T):
    torch = torch_cuda()
    say("prefill", d, f, n, k, T)
    wr = synth.router_weights(synth.seed_for(3, "prefill", "router", d, n), n, d)
    slabs = [synth.expert_slab(synth.seed_for(3, "prefill", "expert", d, e), d, f, None) for e in range(n)]
    X = synth.iid_states(synth.seed_for(3, "prefill", "prompt", d, T), T, d)
    pool = _pool_np(torch, slabs, d, f)
    out, idx, w = _run(torch, X, wr, pool, d, f, n, k)
    worst = worst_b = 0.0
    for t in range(T):
        oidx, ow = router_parity(idx[t], w[t], X[t], wr, k)
        _, _, ref, _ = oracle.moe_token(X[t], wr, slabs, k, f, forced_set=oidx)
        r = rel_err(out[t], ref)
        assert r <= TOL, (t, r)
        worst = max(worst, r)
        # The same layer with the two bf16 roundings the matrix cores need (x and h),
        # fp64 otherwise: what is left is accumulation order only.
        rb = rel_err(out[t], _bf16_activation_ref(X[t], slabs, oidx, ow, d, f))
        assert rb <= 2e-3, (t, rb)
        worst_b = max(worst_b, rb)
    say("  worst max|err|/RMS vs oracle", worst, "vs bf16-activation reference", worst_b)


@pytest.mark.parametrize("shape", ["mixtral", "phi", "fine"])
def test_prefill_full_shape(shape):
    """Configs: one 512-token prompt through a full-size layer with every expert resident,
    in the launch configuration the benchmark times, every token's routing and output
    compared with the oracle.
    * mixtral (the benchmark's prefill line): one M tile per expert, 112 gate/up tiles per
      XCD, the last 16 in 2 K parts, and all 16 down tiles per XCD in 2;
    * phi (d 4096, f 6400, 16 experts top-2): 100 gate/up tiles per XCD, the last 4 in 8 K
      parts, 32 whole down tiles;
    * fine (d 3584, f 2560, 64 experts top-8, routed experts only): 64 (token, expert) pairs
      per expert on average, 160 whole gate/up tiles per XCD, 112 down tiles, the last 16 in
      2 K parts."""
    torch = torch_cuda()
    import paper_2512_16473_amd as moe
    if shape == "mixtral":
        wl = synth.WORKLOADS["prefill"]
        tag = "prefill"
    else:
        wl = synth.WORKLOADS[shape]
        tag = "prefill-" + shape
    d, f, n, k, T = wl.d, wl.f, wl.n, wl.k, 512
    say("prefill", shape, d, f, n, k, T)
    stride = moe.slab_bytes(d, f)
    pool = torch.empty(n * stride, dtype=torch.uint8, device="cuda")
    host = []
    for e in range(n):
        t = pool[e * stride: e * stride + 3 * d * f * 2].view(torch.bfloat16)
        synth.expert_slab_torch(synth.seed_for(0, tag, "expert", 0, e), d, f, wl.w_std, out=t)
        host.append(t.view(torch.uint8).cpu().numpy().view(np.uint16))
    wr = synth.router_weights(synth.seed_for(0, tag, "router", 0), n, d)
    X = synth.iid_states(synth.seed_for(0, tag, "prompt"), T, d)
    out, idx, w = _run(torch, X, wr, pool, d, f, n, k)
    oracle.set_threads(min(16, os.cpu_count() or 1))
    sets = []
    for t in range(T):
        oidx, ow = router_parity(idx[t], w[t], X[t], wr, k)
        sets.append(oidx)
    counts = np.bincount(idx.ravel(), minlength=n)
    say("  tokens per expert", counts.tolist())
    worst = 0.0
    for t in range(T):
        _, _, ref, _ = oracle.moe_token(X[t], wr, host, k, f, forced_set=sets[t])
        r = rel_err(out[t], ref)
        assert r <= TOL, (t, r)
        worst = max(worst, r)
        if t % 128 == 127:
            say("  tokens compared", t + 1, "worst max|err|/RMS so far", worst)
    say("  worst max|err|/RMS", worst)


def test_prefill_empty_and_invalid():
    torch = torch_cuda()
    import paper_2512_16473_amd as moe
    d, f, n, k = 256, 512, 4, 2
    pool = torch.zeros(n * moe.slab_bytes(d, f), dtype=torch.uint8, device="cuda")
    wr = torch.zeros((n, d), device="cuda")
    X = torch.zeros((0, d), device="cuda")
    out = torch.zeros((1, d), device="cuda")
    ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    moe.prefill_forward(X, wr, pool, d, f, n, k, out, ws)        # T = 0: no-op
    with pytest.raises(moe.MoeError):
        moe.prefill_forward(torch.zeros((4, 200), device="cuda"), torch.zeros((n, 200), device="cuda"), pool,
                            200, f, n, k, out, ws)                # d not a multiple of 128


# One expert, so the tokens per tile are T's own: the edges of the tile heights (32-row
# blocks, 1 to 8 of them, and two or more tiles of uneven height), K loops shorter than the
# load rings (d or f = 128: two steps), the half N tile of a d that is an odd multiple of
# 128, K splits of a whole GEMM (2048, 1024) and weights shared by many tiles.
_EDGES = [1, 16, 17, 32, 33, 64, 65, 97, 129, 160, 161, 193, 225, 256, 257, 288, 513, 545]


@pytest.mark.parametrize("d,f,T", [(128, 128, T) for T in _EDGES + [2500]] + [(384, 256, T) for T in _EDGES + [2500]] +
                         [(2048, 1024, T) for T in _EDGES])
def test_prefill_tile_edges(d, f, T):
    torch = torch_cuda()
    say("prefill tile", d, f, T)
    slab = synth.expert_slab(77 + d, d, f, None)
    X = synth.iid_states(5 + T, T, d)
    out, idx, w = _run(torch, X, synth.router_weights(9, 1, d), _pool_np(torch, [slab], d, f), d, f, 1, 1)
    assert np.all(idx == 0) and np.all(w == 1.0)
    # bf16 activations as in _bf16_activation_ref, all tokens at once
    W = synth.bf16_to_f32(slab).astype(np.float64)
    xb = synth.bf16_to_f32(synth.bf16_bits(X)).astype(np.float64)
    g, u = xb @ W[:f * d].reshape(f, d).T, xb @ W[f * d:2 * f * d].reshape(f, d).T
    h = g / (1.0 + np.exp(-g)) * u
    hb = synth.bf16_to_f32(synth.bf16_bits(h.astype(np.float32))).astype(np.float64)
    w2 = W[2 * f * d:].reshape(d, f)
    ref = hb @ w2.T
    rms = np.sqrt(np.mean(ref ** 2, axis=1))
    # Bound: fp32 sums of up to 2048 terms in any order stay within 2e-5 RMS (5e-7 seen).
    # An h within the fp32 error of a rounding midpoint (1e-5 (1 + |g|)(1 + |u|) covers it)
    # may round to the other side, which moves the outputs by one bf16 ulp of it times W2.
    ulp = np.exp2(np.floor(np.log2(np.abs(h) + 1e-30)) - 7)
    near = np.abs(np.abs(h - hb) - ulp / 2) <= 1e-5 * (1 + np.abs(g)) * (1 + np.abs(u))
    flip = (near * ulp) @ np.abs(w2).T
    worst = np.max(np.abs(out - ref) - flip, axis=1) / rms
    assert np.all(worst <= 2e-5), (int(np.argmax(worst)), float(worst.max()))


# Few tokens on few N tiles: every down tile is split over the output's planes (T = 11: five,
# T = 100: eight; with the least workspace, four without the room for the tile tables: three or
# fewer), one expert and one token with the smallest planes, and more experts than pairs.
@pytest.mark.parametrize("d,f,n,k,T", [(1408, 5632, 8, 2, 11), (128, 2048, 1, 1, 1), (256, 1024, 256, 1, 1),
                                       (384, 4096, 60, 8, 3), (640, 1152, 5, 2, 40), (384, 8192, 4, 1, 100)])
@pytest.mark.parametrize("least", [False, True])
def test_prefill_planes(d, f, n, k, T, least):
    torch = torch_cuda()
    import paper_2512_16473_amd as moe
    say("prefill planes", d, f, n, k, T, least)
    g = torch.Generator(device="cuda")
    g.manual_seed(d + f + T)
    stride = moe.slab_bytes(d, f)
    pool = torch.empty(n * stride // 2, dtype=torch.bfloat16, device="cuda").normal_(0, d ** -0.5, generator=g)
    wr = torch.empty((n, d), device="cuda").normal_(0, d ** -0.5, generator=g)
    X = torch.empty((T, d), device="cuda").normal_(0, 1, generator=g)
    nb = moe.prefill_workspace_bytes(d, f, n, k, T)
    if least:
        al = lambda b: (b + 255) // 256 * 256
        nb = al(T * d * 2) + 4 * al(T * k * 4) + al((n + 1) * 4) + al(T * k * f * 2) + al(4 * T * k * d * 4)
        with pytest.raises(moe.MoeError):
            moe.prefill_forward(X, wr, pool, d, f, n, k, torch.empty_like(X),
                                torch.empty(nb - 256, dtype=torch.uint8, device="cuda"))
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    out = torch.full((T, d), float("nan"), device="cuda")
    idx = torch.zeros((T, k), dtype=torch.int32, device="cuda")
    w = torch.zeros((T, k), device="cuda")
    moe.prefill_forward(X, wr, pool, d, f, n, k, out, ws, idx=idx, w=w)
    torch.cuda.synchronize()
    _assert_bf16_reference(torch, X, pool, out, idx, w, d, f, n)


def _assert_bf16_reference(torch, X, pool, out, idx, w, d, f, n):
    import paper_2512_16473_amd as moe
    stride = moe.slab_bytes(d, f)
    ref = torch.zeros(X.shape, dtype=torch.float64, device="cuda")
    xb = X.to(torch.bfloat16).double()
    scale = torch.zeros((X.shape[0], 1), dtype=torch.float64, device="cuda")
    for e in range(n):
        t, r = (idx == e).nonzero(as_tuple=True)
        if t.numel() == 0:
            continue
        W = pool[e * (stride // 2):][:3 * d * f].double()
        gu, up = xb[t] @ W[:f * d].view(f, d).t(), xb[t] @ W[f * d:2 * f * d].view(f, d).t()
        h = (gu / (1 + torch.exp(-gu)) * up).float().to(torch.bfloat16).double()
        w2 = W[2 * f * d:].view(d, f)
        we = w[t, r].double()[:, None]
        ref.index_add_(0, t, we * (h @ w2.t()))
        scale.index_add_(0, t, we * h.abs().amax(1, keepdim=True) * w2.abs().max())
    # fp32 sums within 2e-5 RMS; a rounding of h that falls the other way (at most a few of
    # them) moves an output by one bf16 ulp, 2^-7, of at most the largest h and W2
    bound = 2e-5 * ref.pow(2).mean(1, keepdim=True).sqrt() + 2 * 2.0 ** -7 * scale
    assert bool(((out - ref).abs() <= bound).all())
    assert float((out - ref).norm() / ref.norm()) <= 1e-3


# Plans with split tiles, each asserted from the routing: gate/up tiles split after whole rounds,
# with one M tile per expert and with two; down tiles in more parts than there are planes
# (buffers of their own), several of them, without and after whole rounds, the latter with 17 M
# tiles per expert. (With as many experts as choices, every expert has all tokens.)
@pytest.mark.parametrize("d,f,n,k,T,gu,dn", [
    (1024, 4352, 8, 2, 128, lambda units, full, s: full > 0 and s > 1, lambda units, full, s: True),
    (1024, 4352, 4, 4, 300, lambda units, full, s: full > 0 and s > 2, lambda units, full, s: units > 1 and s > 4),
    (384, 6528, 16, 7, 199, lambda units, full, s: s == 1, lambda units, full, s: units > 1 and full == 0 and s > 4),
    (2048, 1536, 2, 2, 4224, lambda units, full, s: full > 0 and s > 2,
     lambda units, full, s: full > 0 and units > full + 1 and s > 4)])
def test_prefill_split_plans(d, f, n, k, T, gu, dn):
    torch = torch_cuda()
    import paper_2512_16473_amd as moe
    say("prefill split plans", d, f, n, k, T)
    g = torch.Generator(device="cuda")
    g.manual_seed(d + f + T)
    pool = torch.empty(n * moe.slab_bytes(d, f) // 2, dtype=torch.bfloat16, device="cuda")
    pool.normal_(0, d ** -0.5, generator=g)
    wr = torch.empty((n, d), device="cuda").normal_(0, d ** -0.5, generator=g)
    X = torch.empty((T, d), device="cuda").normal_(0, 1, generator=g)
    ws = torch.empty(moe.prefill_workspace_bytes(d, f, n, k, T), dtype=torch.uint8, device="cuda")
    out = torch.full((T, d), float("nan"), device="cuda")
    idx = torch.zeros((T, k), dtype=torch.int32, device="cuda")
    w = torch.zeros((T, k), device="cuda")
    moe.prefill_forward(X, wr, pool, d, f, n, k, out, ws, idx=idx, w=w)
    torch.cuda.synchronize()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    plans = prefill_plans(d, f, n, k, T, torch.bincount(idx.flatten(), minlength=n).tolist(), cus)
    say("  gate/up", sorted({p[1:] for p in plans[0]}), "down", sorted({p[1:] for p in plans[1]}))
    assert any(gu(*p[1:]) for p in plans[0]) and any(dn(*p[1:]) for p in plans[1])
    _assert_bf16_reference(torch, X, pool, out, idx, w, d, f, n)


# SiLU(g) * u alone: W1 and W3 have one entry a row and W2 is the identity, so g and u are exact
# products of two bf16 values and the output is the bf16 of SiLU(g) * u itself.
def test_prefill_swiglu_exact():
    torch = torch_cuda()
    say("prefill swiglu")
    d = f = 128
    T = 2048
    rng = np.random.default_rng(11)
    bf = lambda v: synth.bf16_to_f32(synth.bf16_bits(np.asarray(v, np.float32)))
    X = np.zeros((T, d), np.float32)
    X[:, 0] = bf(rng.uniform(0.5, 1.0, T))
    X[:, 1] = bf(rng.uniform(0.5, 2.0, T) * np.where(np.arange(T) % 8 == 0, 2.0 ** 50, 1.0))
    X[::16, 0] = 1.0
    c = bf(rng.uniform(-88, 88, f))
    c[:8] = bf([-88, -87.5, -80, -60, 88, 1, -1, 0])
    e = bf(rng.uniform(0.5, 2.0, f) * np.where(np.arange(f) % 4 == 0, 2.0 ** 50, 1.0))
    W = np.zeros((3, f, d), np.float32)
    W[0, :, 0], W[1, :, 1], W[2] = c, e, np.eye(d)
    slab = synth.bf16_bits(W.ravel())
    out, _, _ = _run(torch, X, np.zeros((1, d), np.float32), _pool_np(torch, [slab], d, f), d, f, 1, 1)
    g = X[:, :1].astype(np.float64) * c.astype(np.float64)
    h = g / (1.0 + np.exp(-g)) * (X[:, 1:2].astype(np.float64) * e.astype(np.float64))
    # Bound: expf within 1 ulp, the sum, the division and the product each rounded once: at most
    # 2.5 fp32 ulps, 3e-7 relative, before the rounding to bf16.
    lo, hi = (bf((h * (1 + s * 3e-7)).astype(np.float32)) for s in (-1, 1))
    off = (out != lo) & (out != hi)
    assert not off.any(), (int(off.sum()), g[off][:4], h[off][:4], out[off][:4])
