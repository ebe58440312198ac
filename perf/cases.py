"""Performance cases of the GEMM runtime: what its users have it do, over the range they do it.

Four kinds of work, all through the public binding:

  gemm    one product C = alpha A B + beta C by a stated variant, or by the one the runtime
          itself takes when nothing has been timed yet (variant "")
  grouped one launch of a grouped plan over many products of uneven shapes
  stream  a list of requests of recurring shapes, each with its own tolerance, served in
          order with history nearest-neighbour selection, a share of them verified
  train   training of the selector network on a table of timed shapes

Sizes are those of the repository's own workloads: square sizes and log-uniform shapes in
[64, 8192] for single products, [32, 1024] for the batched ones, up to 4096 for the stream,
2000 timed shapes for the selector.
"""
import math
import random

import numpy as np
import torch

import paper_2311_03543_amd as pa

VARIANTS = {"f32_simt": 0, "bf16x3": 1, "fp8r": 2, "bf16": 3, "fp6x3": 4}
TOLS = (1e-5, 1e-3, 1e-2)
PAR = 4 * 64 + 64 + 64 * 64 + 64 + 64 * 4 + 4


def gemm(name, variant, M, N, K, alpha=1.0, beta=0.0, pad=0, data="normal", verify=False):
    return dict(name=name, kind="gemm", variant=variant, M=M, N=N, K=K, alpha=alpha, beta=beta, pad=pad,
                data=data, verify=verify)


def listed():
    return [
        # the smallest request of the recurring-shape workload, on a context that has timed
        # nothing yet: the runtime takes its tightest variant, and latency is all there is
        gemm("f32_64", "", 64, 64, 64),
        # the single FP32 product that checks an installation: 256^3, uniform [-1, 1]
        gemm("f32_256", "f32_simt", 256, 256, 256, data="uniform"),
        # an ordinary FP32 call inside a larger matrix: no dimension a multiple of 4, operands
        # that are slices (odd leading dimensions), accumulating into C
        gemm("f32_ragged", "f32_simt", 1001, 777, 1531, alpha=1.5, beta=0.5, pad=3),
        # the plain FP32 variant at the largest square size of the sweep
        gemm("f32_8192", "f32_simt", 8192, 8192, 8192),
        # FP32-class accuracy at a middle square size, where the output tiles leave CUs idle
        gemm("bf16x3_1024", "bf16x3", 1024, 1024, 1024),
        # the same variant at the largest size: the 1e-5 class of the headline workload
        gemm("bf16x3_8192", "bf16x3", 8192, 8192, 8192),
        # the 1e-3 class on ragged, badly scaled operands with the residual check on
        gemm("fp8r_verify", "fp8r", 3000, 2500, 4100, data="ill", verify=True),
        # a tall reduction: few output tiles, a long odd K, one bf16 product
        gemm("bf16_skinny", "bf16", 300, 4000, 8191),
        # the 1e-2 class of the headline workload, at half its size
        gemm("fp6x3_4096", "fp6x3", 4096, 4096, 4096),
        # the batched workload: uneven products in [32, 1024] in one FP32 launch (the 128 x 128
        # tile its autotuner settles on)
        dict(name="grouped_f32", kind="grouped", count=512, lo=32, hi=1024, config=4),
        # the request stream: 30 recurring shapes up to 2048, a fifth of the requests badly
        # scaled and verified, each complete before the next
        dict(name="stream", kind="stream", requests=200, shapes=30, lo=64, hi=2048, sync=True),
        # the selector network on the full table of timed shapes
        dict(name="train", kind="train", rows=2000, steps=500),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("gemm", "grouped", "stream", "train"), (8, 2, 1, 1))[0]
    if kind == "gemm":
        variant = rng.choice(("", "f32_simt", "f32_simt", "bf16x3", "bf16x3", "fp8r", "bf16", "fp6x3"))
        M, N, K = (_log_uniform(rng, 64, 8192) for _ in range(3))
        if rng.random() < 0.3:
            M = N = K = 1 << rng.randint(7, 12)
        alpha, beta = rng.choice(((1.0, 0.0), (1.0, 0.0), (1.5, 0.5), (-0.75, 0.25)))
        c = gemm("", variant, M, N, K, alpha, beta, rng.choice((0, 0, 1, 4)), rng.choice(("normal", "normal", "uniform", "ill")),
                 rng.random() < 0.25)
        del c["name"]
        return c
    if kind == "grouped":
        hi = rng.choice((256, 512, 1024))
        return dict(kind="grouped", count=_log_uniform(rng, 16, 512), lo=32, hi=hi, config=rng.choice((0, 2, 4, 5, 10)))
    if kind == "stream":
        return dict(kind="stream", requests=rng.randint(60, 200), shapes=rng.randint(10, 40), lo=64,
                    hi=rng.choice((1024, 2048, 4096)), sync=rng.random() < 0.5)
    return dict(kind="train", rows=rng.randint(150, 2500), steps=rng.randint(50, 500))


# ---------------------------------------------------------------------------
# Inputs

def _fill(shape, data, g):
    if data == "uniform":
        return torch.rand(shape, device="cuda", generator=g) * 2 - 1
    x = torch.randn(shape, device="cuda", generator=g)
    if data == "ill":
        x *= torch.exp2(torch.randint(-20, 21, shape, device="cuda", generator=g).to(torch.float32))
    return x


def _operands(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    p = c["pad"]
    A = _fill((c["M"], c["K"] + p), c["data"], g)[:, p:]
    B = _fill((c["K"], c["N"] + p), c["data"], g)[:, p:]
    C = _fill((c["M"], c["N"] + p), "normal", g)[:, p:]
    return A, B, C


def _problems(count, lo, hi, data, seed):
    """`count` products in [lo, hi]: (A, B) each, and one flat buffer that holds every C in turn."""
    rng = random.Random(1000003 * count + 1009 * hi + lo)     # the shapes belong to the case
    g = torch.Generator(device="cuda").manual_seed(seed)
    ops, at, total = [], [], 0
    for _ in range(count):
        M, N, K = (_log_uniform(rng, lo, hi) for _ in range(3))
        ops.append((_fill((M, K), data, g), _fill((K, N), data, g)))
        at.append(total)
        total += (M * N + 63) // 64 * 64
    return ops, at, total


def _views(flat, ops, at):
    return [flat[o:o + A.shape[0] * B.shape[1]].view(A.shape[0], B.shape[1]) for (A, B), o in zip(ops, at)]


# microseconds of a table of timed shapes: launch cost, operand conversion, product
_COST = {0: (8.0, 0.0, 80.0), 1: (16.0, 8.0, 430.0), 2: (16.0, 7.0, 700.0), 3: (16.0, 6.0, 950.0)}


def _time_us(vid, M, N, K):
    start, byte, rate = _COST[vid]
    tiles = math.ceil(M / 256) * math.ceil(N / 256)
    return start + byte * K * (M + N) / 4e6 + 2.0 * M * N * K / (rate * 1e6 * min(1.0, tiles / 64 + 0.05))


def _stream(c, seed):
    rng = random.Random(c["requests"] * 7919 + c["shapes"] * 31 + c["hi"])
    g = torch.Generator(device="cuda").manual_seed(seed)
    shapes = [tuple(_log_uniform(rng, c["lo"], c["hi"]) for _ in range(3)) for _ in range(c["shapes"])]
    well = [(_fill((M, K), "normal", g), _fill((K, N), "normal", g)) for M, N, K in shapes]
    ill = [(_fill((M, K), "ill", g), _fill((K, N), "ill", g)) for M, N, K in shapes]
    weights = [1.0 / (r + 1) ** 1.1 for r in range(len(shapes))]
    ops, tols, verify, at, total = [], [], [], [], 0
    for r in rng.choices(range(len(shapes)), weights, k=c["requests"]):
        hard = rng.random() < 0.2
        A, B = ill[r] if hard else well[r]
        ops.append((A, B))
        tols.append(rng.choice(TOLS))
        verify.append(hard)
        at.append(total)
        total += (A.shape[0] * B.shape[1] + 63) // 64 * 64
    return shapes, ops, tols, verify, at, total


def _table(c, seed):
    rng = random.Random(seed)
    X, Y = [], []
    for _ in range(c["rows"]):
        M, N, K = (_log_uniform(rng, 64, 8192) for _ in range(3))
        X.append([math.log2(M), math.log2(N), math.log2(K), math.log10(rng.choice(TOLS))])
        Y.append([math.log(_time_us(v, M, N, K) * rng.uniform(0.95, 1.05)) for v in range(4)])
    p = np.random.Generator(np.random.PCG64(seed))
    init = []
    for fan_in, fan_out in ((4, 64), (64, 64), (64, 4)):
        init.append(p.uniform(-1, 1, fan_in * fan_out) * math.sqrt(6.0 / fan_in))
        init.append(p.uniform(-1, 1, fan_out) / math.sqrt(fan_in))
    return np.array(X, np.float32), np.array(Y, np.float32), np.concatenate(init).astype(np.float32)


def prepare(case, seed):
    cx = pa.Compar(0)
    s = dict(case=case, cx=cx)
    if case["kind"] == "gemm":
        s["A"], s["B"], s["C"] = _operands(case, seed)
        if case["variant"] == "fp6x3":
            assert cx.register_builtin("fp6x3") == VARIANTS["fp6x3"]
        if case["variant"] and case["verify"]:
            cx.force_variant(VARIANTS[case["variant"]])
        cx.set_flags(pa.CMP_FLAG_VERIFY if case["verify"] else 0)
        s["tol"] = {"": 1e-5, "f32_simt": 1e-5, "bf16x3": 1e-5, "fp8r": 1e-3}.get(case["variant"], 1e-2)
    elif case["kind"] == "grouped":
        ops, at, total = _problems(case["count"], case["lo"], case["hi"], "normal", seed)
        s["ops"], s["flat"] = ops, torch.zeros(total, device="cuda")
        s["plan"] = cx.grouped_plan([(A, B, C) for (A, B), C in zip(ops, _views(s["flat"], ops, at))], config=case["config"])
    elif case["kind"] == "stream":
        shapes, ops, tols, verify, at, total = _stream(case, seed)
        s["flat"] = torch.zeros(total, device="cuda")
        s["requests"] = [(A, B, C) for (A, B), C in zip(ops, _views(s["flat"], ops, at))]
        s["tols"], s["verify"] = np.array(tols), np.array(verify)
        for M, N, K in dict.fromkeys(shapes):
            for v in range(4):
                cx.history_add(M, N, K, v, 20, _time_us(v, M, N, K) * 1e-3)
        cx.selector_set(pa.CMP_SEL_NN)
    else:
        s["X"], s["Y"], s["init"] = _table(case, seed)
    return s


def run(s):
    c, cx = s["case"], s["cx"]
    if c["kind"] == "gemm":
        if c["variant"] and not c["verify"]:
            cx.gemm_variant(VARIANTS[c["variant"]], s["A"], s["B"], s["C"], c["alpha"], c["beta"])
        else:
            cx.gemm(s["A"], s["B"], s["C"], c["alpha"], c["beta"], tol=s["tol"])
        return s["C"]
    if c["kind"] == "grouped":
        s["plan"].graph_launch()
        return s["flat"]
    if c["kind"] == "stream":
        chosen, _ = cx.gemm_stream(s["requests"], s["tols"], verify=s["verify"], sync=c["sync"])
        return s["flat"], chosen
    cx.mlp_set_params(s["init"])
    loss = cx.mlp_train(s["X"], s["Y"], c["steps"], 1e-3)
    return cx.mlp_get_params(), loss


# ---------------------------------------------------------------------------
# What a pass cannot do without, and what it returns in exact arithmetic

def _gemm_work(M, N, K, beta=0.0):
    return 4.0 * (M * K + K * N + M * N * (2 if beta else 1)), 2.0 * M * N * K


def work(case):
    if case["kind"] == "gemm":
        b, f = _gemm_work(case["M"], case["N"], case["K"], case["beta"])
        if case["verify"]:                                    # A, B, C (and the old C) once more
            b += _gemm_work(case["M"], case["N"], case["K"], case["beta"])[0]
        return dict(bytes=b, flops=f)
    if case["kind"] == "train":                               # forward, backward and update per row and step
        n, k = case["rows"], case["steps"]
        return dict(bytes=4.0 * (8 * n + 2 * PAR + k), flops=float(k) * (n * 6.0 * (4 * 64 + 64 * 64 + 64 * 4) + 12.0 * PAR))
    if case["kind"] == "grouped":
        rng = random.Random(1000003 * case["count"] + 1009 * case["hi"] + case["lo"])
        shapes = [tuple(_log_uniform(rng, case["lo"], case["hi"]) for _ in range(3)) for _ in range(case["count"])]
    else:
        rng = random.Random(case["requests"] * 7919 + case["shapes"] * 31 + case["hi"])
        kinds = [tuple(_log_uniform(rng, case["lo"], case["hi"]) for _ in range(3)) for _ in range(case["shapes"])]
        weights = [1.0 / (r + 1) ** 1.1 for r in range(len(kinds))]
        shapes = [kinds[r] for r in rng.choices(range(len(kinds)), weights, k=case["requests"])]
    both = [_gemm_work(*s) for s in shapes]
    return dict(bytes=sum(b for b, _ in both), flops=sum(f for _, f in both))


def _product(A, B, alpha=1.0, beta=0.0, C=None):
    R = alpha * (A.double() @ B.double())
    return R if not beta else R + beta * C.double()


def _train64(c, seed):
    """Full-batch Adam in binary64 on the standardised table; the network's step in closed form."""
    X, Y, p = _table(c, seed)
    X, Y = (torch.from_numpy(v.astype(np.float64)).cuda() for v in (X, Y))

    def standard(v):
        sd = v.std(0, unbiased=False)
        return (v - v.mean(0)) / torch.where(sd > 0, sd, torch.ones_like(sd))

    X, Y, p = standard(X), standard(Y), torch.from_numpy(p.astype(np.float64)).cuda()
    m, v, losses = torch.zeros_like(p), torch.zeros_like(p), []
    for t in range(1, c["steps"] + 1):
        W1, b1, W2, b2, W3, b3 = torch.split(p, [256, 64, 4096, 64, 256, 4])
        W1, W2, W3 = W1.view(64, 4), W2.view(64, 64), W3.view(4, 64)
        z1 = X @ W1.T + b1
        h1 = z1.clamp(min=0)
        z2 = h1 @ W2.T + b2
        h2 = z2.clamp(min=0)
        d = h2 @ W3.T + b3 - Y
        losses.append(d.square().mean())
        d = d * (2.0 / d.numel())
        d2 = (d @ W3) * (z2 > 0)
        d1 = (d2 @ W2) * (z1 > 0)
        g = torch.cat([(d1.T @ X).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0), (d.T @ h2).reshape(-1), d.sum(0)])
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        p = p - 1e-3 * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return p.cpu().numpy(), torch.stack(losses).cpu().numpy()


def exact(case, seed):
    if case["kind"] == "train":
        return _train64(case, seed)
    if case["kind"] == "gemm":
        A, B, C = _operands(case, seed)
        return _product(A, B, case["alpha"], case["beta"], C)
    if case["kind"] == "grouped":
        ops, at, total = _problems(case["count"], case["lo"], case["hi"], "normal", seed)
    else:
        _, ops, _, _, at, total = _stream(case, seed)
    flat = torch.zeros(total, dtype=torch.float64, device="cuda")
    for (A, B), C in zip(ops, _views(flat, ops, at)):
        C.copy_(_product(A, B))
    return flat if case["kind"] == "grouped" else (flat, None)
