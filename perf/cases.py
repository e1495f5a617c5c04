"""The work that is timed: what a program using this library has it do, through the Python binding.

A case is a dict of plain values. Four kinds of work ("op"):
  linear   a stack of packed linears applied to fp16 activations, batch 1 (fluxbin_lut_gemv) or more rows
           (fluxbin_lut_gemm_smallbatch), one call per linear, into preallocated outputs with the workspaces a serving
           loop keeps. With graph the calls of the stack are one captured HIP graph that run() replays, which is how a
           decode loop issues a step of many microsecond calls; without it run() makes the calls.
  pack     canonical sign planes and scales (on the device) into the packed layer format.
  hybrid   the weight decomposition: saliency search, global bases, salient bases of their residual.

Inputs come from the distributions of the synthetic layers in synth/ (signs fair coins, row scales |N(0, 0.05)|, column
scales lognormal(0, 0.3), activations N(0, 1) with 0.1% outlier channels x20), drawn on the GPU.
"""
import math

import torch

from paper_2608_15602_amd import fluxbin as fb

# Linears of a stack as (out, in) pairs: the decoder-layer shapes of the repository's workloads.
STACKS = {
    # q, k, v, o, gate, up, down of a 7B decoder layer
    "layer7b": [(4096, 4096)] * 4 + [(11008, 4096)] * 2 + [(4096, 11008)],
    "mlp7b": [(11008, 4096), (4096, 11008)],
    "mlp70b": [(28672, 8192), (8192, 28672)],
    # a 70B decoder layer with the linears that share an input fused: q|k|v, o, gate|up, down
    "fused70b": [(10240, 8192), (8192, 8192), (57344, 8192), (8192, 28672)],
}


def _linear(name, B, Kb, Ks, mu=8, frac=0.0, s=0, stack="", M=0, N=0, g_r=128, repeat=1, graph=True, fp32=False):
    """frac: share of the columns that is salient (drawn over the whole width, one salient row scale per row);
    s: salient columns in every block of 128 columns (one salient row scale per row and block)."""
    case = dict(op="linear", stack=stack, M=M, N=N, Kb=Kb, Ks=Ks, mu=mu, frac=frac, s=s, g_r=g_r, B=B, repeat=repeat,
                graph=graph, fp32=fp32)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest linear, one call at a time: launch latency and host path
        _linear("tiny_b1", 1, 2, 1, mu=4, frac=8 / 256, M=512, N=256, graph=False),
        # batch-1 decoding of a 7B model: two decoder layers, 14 calls of 5 to 13 MB each
        _linear("layer7b_b1", 1, 2, 1, frac=0.03, stack="layer7b", repeat=2),
        # batch-1 decoding in the paper's 2b-s8-g128 format (structured salient columns, fine salient row scales)
        _linear("s8_b1", 1, 2, 2, s=8, M=5120, N=13824, repeat=4),
        # batch-1 decoding, the MLP of a 70B model at 3 bases + 5%: the benchmark's headline step
        _linear("mlp70b_b1", 1, 3, 1, frac=0.05, stack="mlp70b"),
        # a few sequences decoded together on the same MLP
        _linear("mlp70b_b4", 4, 3, 1, frac=0.05, stack="mlp70b"),
        # eight sequences on the MLP of a 7B model, four decoder layers
        _linear("mlp7b_b8", 8, 2, 1, frac=0.03, stack="mlp7b", repeat=4),
        # sixteen sequences through the linears of a 70B decoder layer at 2 bases + 1%
        _linear("fused70b_b16", 16, 2, 1, frac=0.01, stack="fused70b"),
        # sixteen sequences in the paper's 2b-s16-g128 format
        _linear("s16_b16", 16, 2, 2, s=16, M=4096, N=11008, repeat=2),
        # an odd-sized layer at mu = 4 and a small batch, fp32 output, one call at a time
        _linear("odd_b5", 5, 3, 1, mu=4, frac=0.04, M=3001, N=1999, graph=False, fp32=True),
        # prompt processing: 256 tokens through the 70B up projection
        _linear("prefill70b_b256", 256, 3, 1, frac=0.05, M=28672, N=8192, graph=False),
        # quantizing a 4096 x 4096 weight in the 2b-s8-g128 format, ten rounds
        dict(name="hybrid4096", op="hybrid", M=4096, N=4096, Kb=2, Ks=2, s=8, T=10),
        # loading a 70B up projection: canonical planes into the packed format
        dict(name="pack70b", op="pack", M=28672, N=8192, Kb=3, Ks=1, mu=8, frac=0.05, s=0, g_r=128),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["b1"] * 4 + ["small"] * 4 + ["prefill"] * 2 + ["hybrid", "pack"])
    if op == "hybrid":
        M, N = _log(rng, 256, 4096), _log(rng, 256, 4096)
        return dict(op="hybrid", M=M, N=N, Kb=rng.choice([1, 2, 2, 3]), Ks=rng.choice([1, 2]), s=rng.choice([4, 8, 16]),
                    T=rng.choice([3, 5, 10]))
    Kb = rng.choice([1, 2, 2, 3, 3, 4])
    mu = rng.choice([8, 8, 8, 4])
    salient = rng.choice(["none", "frac", "frac", "blocks"])
    Ks = 0 if salient == "none" else rng.choice([1, Kb])
    frac = round(rng.uniform(0.005, 0.06), 4) if salient == "frac" else 0.0
    s = rng.choice([8, 16]) if salient == "blocks" else 0
    g_r = rng.choice([128, 128, 128, 256, 0, 64])
    while True:
        M, N = _log(rng, 128, 57344), _log(rng, 128, 28672)
        # half of the sizes are whole chunks, as model dimensions are, the others odd
        if rng.random() < 0.5:
            M, N = max(128, M // 128 * 128), max(128, N // 128 * 128)
        B = 1 if op in ("b1", "pack") else _log(rng, 2, 32) if op == "small" else _log(rng, 33, 256)
        if s and (N < 256 or N % 128):
            N = max(256, N // 128 * 128)
        # no more than the largest listed case; fine row-scale groups (s > 0 or g_r = 64) at a batch cost several times
        # as much per weight
        cost = M * N * (Kb + 0.1 * Ks) * B * (8 if (s or g_r == 64) and B > 1 else 1)
        if cost <= 28672 * 8192 * 3.1 * 256 and M * N <= 28672 * 16384:
            break
    if op == "pack":
        return dict(op="pack", M=M, N=N, Kb=Kb, Ks=Ks, mu=mu, frac=frac, s=s, g_r=g_r)
    return _linear("", B, Kb, Ks, mu=mu, frac=frac, s=s, M=M, N=N, g_r=g_r, graph=rng.random() < 0.5,
                   fp32=rng.random() < 0.25)


# ---------------------------------------------------------------------------------------------------- inputs

def _shapes(case):
    base = STACKS[case["stack"]] if case.get("stack") else [(case["M"], case["N"])]
    return base * case.get("repeat", 1)


def _dims(case, M, N):
    """(g_r, S, g_s) of one linear. A drawn g_r of 0 is one row scale per row."""
    g_r = case["g_r"] or N
    if case["s"]:
        return g_r, case["s"] * -(-N // 128), case["s"]
    S = int(case["frac"] * N + 0.5) if case["Ks"] else 0
    return g_r, S, max(S, 1)


def _words(gen, planes, M, N):
    return torch.randint(-2**31, 2**31, (planes, M, -(-N // 32)), dtype=torch.int32, device="cuda", generator=gen)


def _weights(case, M, N, gen):
    """Canonical weights of one linear (device tensors under the binding's field names), fp16 as torch.float16."""
    def normal(*size):
        return torch.randn(size, device="cuda", generator=gen)

    Kb, Ks = case["Kb"], case["Ks"]
    g_r, S, g_s = _dims(case, M, N)
    w = dict(signs=_words(gen, Kb, M, N), alpha_r=(normal(Kb, M, -(-N // g_r)) * 0.05).abs().half(),
             alpha_c=(normal(Kb, N) * 0.3).exp().half())
    if S > 0:
        if case["s"]:
            order = torch.rand(N // 128, 128, device="cuda", generator=gen).argsort(dim=1)[:, :case["s"]]
            cols = (order.sort(dim=1).values + 128 * torch.arange(N // 128, device="cuda")[:, None]).reshape(-1)
        else:
            cols = torch.randperm(N, device="cuda", generator=gen)[:S].sort().values
        w.update(sal_idx=cols.int(), sal_signs=_words(gen, Ks, M, N),
                 alpha_sr=(normal(Ks, M, -(-S // g_s)) * 0.05).abs().half(), alpha_sc=(normal(Ks, N) * 0.3).exp().half())
    return w


def _shape(case, M, N):
    g_r, S, g_s = _dims(case, M, N)
    return fb.make_shape(M, N, case["Kb"], case["Ks"] if S else 0, case["mu"], g_r, S, g_s)


def _pack(case, M, N, w):
    return fb.fluxbin_pack(_shape(case, M, N), w)


def _x(B, N, gen):
    x = torch.randn((B, N), device="cuda", generator=gen)
    n_out = int(0.001 * N + 0.5)
    if n_out:
        x[:, torch.randperm(N, device="cuda", generator=gen)[:n_out]] *= 20
    return x.half()


def _matrix(case, gen):
    """A weight matrix with 1% outlier columns and a diagonal inverse Hessian (as synth.make_weight_matrix draws)."""
    M, N = case["M"], case["N"]
    W = torch.randn((M, N), device="cuda", generator=gen) * 0.02
    W[:, torch.randperm(N, device="cuda", generator=gen)[:int(0.01 * N + 0.5)]] *= 10
    return W, torch.rand(N, dtype=torch.float64, device="cuda", generator=gen) * 1.5 + 0.5


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _inputs(case, seed):
    """Every linear's (M, N, weights, x) of a linear case, one at a time."""
    gen = _gen(seed)
    for M, N in _shapes(case):
        w = _weights(case, M, N, gen)
        yield M, N, w, _x(case["B"], N, gen)


# ---------------------------------------------------------------------------------------------------- the passes

def _call(layer, x, y, ws, fp32):
    if x.dim() == 1:
        fb.fluxbin_lut_gemv(layer, x, y=y, out_fp32=fp32, workspace=ws)
    else:
        fb.fluxbin_lut_gemm_smallbatch(layer, x, y=y, out_fp32=fp32, workspace=ws)


def prepare(case, seed):
    if case["op"] == "hybrid":
        W, h = _matrix(case, _gen(seed))
        return dict(case=case, W=W, h=h)
    if case["op"] == "pack":
        return dict(case=case, w=_weights(case, case["M"], case["N"], _gen(seed)))
    calls = []
    for M, N, w, x in _inputs(case, seed):
        layer = _pack(case, M, N, w)
        ws = fb.make_workspace(layer, case["B"])
        y = torch.empty((case["B"], M), dtype=torch.float32 if case["fp32"] else torch.float16, device="cuda")
        if case["B"] == 1:
            x, y = x[0], y[0]
        calls.append((layer, x, y, ws, case["fp32"]))
    state = dict(case=case, calls=calls, y=[c[2] for c in calls], graph=None)
    if case["graph"]:
        for c in calls:
            _call(*c)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            for c in calls:
                _call(*c)
    return state


def _sections(layer):
    """The sections of a packed buffer, without the unwritten bytes that align them."""
    L, buf = layer.layer, layer.buf
    s = L.shape
    sizes = (("header", 0, fb.HEADER_BYTES), ("signs", L.off_signs, L.NSC * 2 * L.Mp * 16),
             ("rscale", L.off_rscale, L.NRP * L.Mp * 2), ("colscale", L.off_colscale, L.NSC * 512),
             ("xidx", L.off_xidx, L.NSC * 512), ("chunk_plane", L.off_chunk_plane, L.NSC * 8),
             ("sal_idx", L.off_sal_idx, max(s.S, 1) * 2))
    return {name: buf[off:off + n] for name, off, n in sizes}


def run(state):
    case = state["case"]
    if case["op"] == "linear":
        if state["graph"] is not None:
            state["graph"].replay()
        else:
            for c in state["calls"]:
                _call(*c)
        return state["y"]
    if case["op"] == "pack":
        return _sections(_pack(case, case["M"], case["N"], state["w"]))
    W = state["W"]
    scores, idx, mask = fb.fluxbin_structural_search(W, state["h"], 128, case["s"])
    glob = fb.fluxbin_rc_decompose(W, case["Kb"], case["T"], 128)
    sal = fb.fluxbin_rc_decompose(W, case["Ks"], case["T"], 128, mask=mask, prior=glob + (128,))
    return dict(scores=scores, idx=idx, glob=glob, sal=sal)


def work(case):
    if case["op"] == "hybrid":
        M, N, G = case["M"], case["N"], -(-case["N"] // 128)
        K = case["Kb"] + case["Ks"]
        # the weights in, sign planes and fp64 scales out; per round and base a row and a column least-squares update
        # (a multiply and an add each) and per round one comparison per sign combination
        by = 4 * M * N + K * (M * N / 8 + 8 * M * G + 8 * N)
        sal = case["s"] / 128
        fl = case["T"] * M * N * (4 * case["Kb"] + 2 ** case["Kb"] + sal * (4 * case["Ks"] + 2 ** case["Ks"]))
        return dict(bytes=by, flops=fl)
    bytes_, flops = 0.0, 0.0
    for M, N in _shapes(case):
        g_r, S, g_s = _dims(case, M, N)
        Kb, Ks, B = case["Kb"], case["Ks"] if S else 0, case.get("B", 0)
        weights = (Kb * M * N + Ks * M * S) / 8 + 2 * M * (Kb * -(-N // g_r) + Ks * -(-S // g_s)) + 2 * Kb * N + \
            2 * Ks * S + 2 * S
        if case["op"] == "pack":   # canonical in (the salient planes' salient columns), packed out
            bytes_ += 2 * weights
        else:
            bytes_ += weights + B * (2 * N + (4 if case["fp32"] else 2) * M)
            flops += 2.0 * B * M * (Kb * N + Ks * S)
    return dict(bytes=bytes_, flops=flops)


def tolerance(case):
    if case["op"] == "pack":
        return "exact"
    if case["op"] == "hybrid":
        # fp64 sums in another order; the small scales of later bases divide residuals that cancel, and a sign is free
        # where two combinations are equally far to the last bit
        return dict(rel=1e-10, max=1e-7, differ=1e-5)
    if case["fp32"]:
        return dict(rel=1e-6, max=1e-5)    # fp32 sums of up to 1e5 terms in another order (1.2e-7 off 64 bits)
    return dict(rel=1e-3, max=2e-3)        # fp16 outputs: 2.1e-4 off 64 bits, half a unit in the last place 4.9e-4


# ---------------------------------------------------------------------------------------------------- 64 bits

def _signs(words, N):
    """+-1 in fp64 from sign words [..., W]."""
    bits = (words[..., None] >> torch.arange(32, device=words.device, dtype=torch.int32)) & 1
    return bits.reshape(*words.shape[:-1], -1)[..., :N].double() * 2 - 1


def _exact_linear(case, M, N, w, x):
    g_r, S, g_s = _dims(case, M, N)
    xt = x.double().t().contiguous()
    y = torch.empty((case["B"], M), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 25) // N)
    for i in range(0, M, step):
        j = min(M, i + step)
        Wd = torch.zeros((j - i, N), dtype=torch.float64, device="cuda")
        for k in range(case["Kb"]):
            r = w["alpha_r"][k, i:j].double().repeat_interleave(g_r, dim=1)[:, :N]
            Wd += _signs(w["signs"][k, i:j], N) * r * w["alpha_c"][k].double()
        if S > 0:
            cols = w["sal_idx"].long()
            for k in range(case["Ks"]):
                r = w["alpha_sr"][k, i:j].double().repeat_interleave(g_s, dim=1)[:, :S]
                Wd[:, cols] += _signs(w["sal_signs"][k, i:j], N)[:, cols] * r * w["alpha_sc"][k].double()[cols]
        y[:, i:j] = (Wd @ xt).t()
    return y


def _exact_rc(X, K, T, mask=None):
    """Residual initialization, then T rounds of least-squares row and column scales per base and the joint sign search,
    per block of 128 columns. Returns (signs +-1/0 [K, M, N], row scales [K, M, G], column scales [K, N])."""
    eps = 1e-12
    M, N = X.shape
    G = -(-N // 128)
    m = torch.ones(N, dtype=torch.float64, device=X.device) if mask is None else mask.double()
    X = X * m
    B = torch.zeros((K, M, N), dtype=torch.float64, device=X.device)
    ar = torch.zeros((K, M, G), dtype=torch.float64, device=X.device)
    ac = torch.zeros((K, N), dtype=torch.float64, device=X.device)

    def wide(r):
        return r.repeat_interleave(128, dim=1)[:, :N]

    def blocks(v):
        return torch.nn.functional.pad(v, (0, 128 * G - N)).reshape(*v.shape[:-1], G, 128).sum(-1)

    def part(k):
        return wide(ar[k]) * ac[k] * B[k]

    def update(k, target):
        cb = ac[k] * B[k]
        ar[k] = blocks(cb * target) / (blocks(cb * cb) + eps)
        rb = wide(ar[k]) * B[k]
        ac[k] = (rb * target).sum(0) / ((rb * rb).sum(0) + eps)

    R = X.clone()
    for k in range(K):
        B[k] = torch.where(R >= 0, 1.0, -1.0) * m
        ac[k] = 1.0
        update(k, R)
        R = R - part(k)
    for _ in range(T):
        for k in range(K):
            update(k, X - sum((part(q) for q in range(K) if q != k), torch.zeros_like(X)))
        mags = [wide(ar[k]) * ac[k] for k in range(K)]
        best = torch.full_like(X, math.inf)
        for c in range(1 << K):
            sg = [1.0 if (c >> k) & 1 else -1.0 for k in range(K)]
            err = (X - sum(mags[k] * sg[k] for k in range(K))).abs()
            better = err < best
            best = torch.where(better, err, best)
            for k in range(K):
                B[k] = torch.where(better, sg[k], B[k])
        B *= m
    return B, ar, ac


def exact(case, seed):
    if case["op"] == "pack":
        return None
    if case["op"] == "linear":
        ys = [_exact_linear(case, M, N, w, x) for M, N, w, x in _inputs(case, seed)]
        return [y[0] for y in ys] if case["B"] == 1 else ys
    W, h = _matrix(case, _gen(seed))
    Wd = W.double()
    scores = Wd.square().sum(0) / h.square()
    mask = torch.zeros(case["N"], dtype=torch.bool, device="cuda")
    for b in range(0, case["N"], 128):
        top = scores[b:b + 128].sort(descending=True, stable=True).indices[:case["s"]]
        mask[b + top] = True
    B, ar, ac = _exact_rc(Wd, case["Kb"], case["T"])
    wide = ar.repeat_interleave(128, dim=2)[:, :, :case["N"]]
    _, sr, sc = _exact_rc(Wd - (wide * ac[:, None, :] * B).sum(0), case["Ks"], case["T"], mask)
    return dict(scores=scores, idx=None, glob=(None, ar, ac), sal=(None, sr, sc))
