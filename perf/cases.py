"""The calls that a user of this library makes, as cases that can be timed and compared.

A sparse diffusion step of one block is: reorder, attention delta, neuron scores, top-k of the neurons, MLP delta.  A
dense step, which fills the caches, is: dense attention with column sums (exact in the first dense step, against the
previous normalisers in a refresh), top-k of the columns, dense MLP.  Every one of these calls is a case of its own at
the sizes of an image model (4608 tokens), a video model (75 600 to 115 456 tokens) and a short clip (18 000 tokens);
one case is the whole sparse step of a block at the smallest configuration, where launches count.

listed() names the cases, draw() gives further ones of the same ranges, prepare() makes what the caller has in hand,
run() is one pass, work() the bytes and operations that a pass cannot do without, tolerance() how far two correct
implementations may be apart, exact() the same results in 64 bits with plain torch.
"""
import math

import torch

import paper_2506_03275_amd as cm
from paper_2506_03275_amd import stack

DEV = "cuda"
BF16, F32, F64, I32 = torch.bfloat16, torch.float32, torch.float64, torch.int32


# ---- the cases -----------------------------------------------------------------------------------------------------

def listed():
    return [
        # the whole sparse step of one block at the smallest configuration (1024 tokens): launches and latency
        dict(name="step_tiny", kind="step", B=1, H=2, N=1024, E=64, c=128, D=256, F=1024, keep_a=0.25, keep_m=0.25),
        # attention delta of an image model (512 text + 64x64 tokens, 7 % of the columns kept)
        dict(name="attn_delta_image", kind="attn_delta", B=1, H=24, N=4608, E=128, c=192, keep=0.07, ragged=False),
        # attention delta of a video model (30x48x80 + 256 tokens), the longest single call of a sparse step
        dict(name="attn_delta_video", kind="attn_delta", B=1, H=24, N=115456, E=128, c=192, keep=0.07, ragged=False),
        # first dense step of an image model: dense attention and exact column sums
        dict(name="attn_dense_image", kind="attn_dense", B=1, H=24, N=4608, E=128, c=192),
        # cache refresh on a short clip (5 latent frames of 45x80, 40 heads; the last chunk is not full)
        dict(name="attn_refresh_clip", kind="attn_refresh", B=1, H=40, N=18000, E=128, c=192),
        # column choice after a dense step of a video model: 24 heads x 602 chunks
        dict(name="topk_columns_video", kind="topk", R=14448, C=115456, k=8082, prev=False),
        # neuron choice of a sparse step of a video model: 602 chunks, top-k of |T - T_m|
        dict(name="topk_neurons_video", kind="topk", R=602, C=12288, k=860, prev=True),
        # neuron scores of a sparse step of a video model
        dict(name="neuron_scores_video", kind="scores", B=1, N=115456, D=3072, F=12288, c=192),
        # MLP delta of an image model (10 % of the neurons recomputed)
        dict(name="mlp_delta_image", kind="mlp_delta", B=1, N=4608, D=3072, F=12288, c=192, keep=0.10, ragged=False,
             act="tanh"),
        # MLP delta of the larger video model (21x45x80 tokens; the last chunk is not full)
        dict(name="mlp_delta_video", kind="mlp_delta", B=1, N=75600, D=5120, F=13824, c=192, keep=0.07, ragged=False,
             act="tanh"),
        # dense MLP of a dense step on a short clip
        dict(name="mlp_dense_clip", kind="mlp_dense", B=1, N=18000, D=5120, F=13824, c=192, act="tanh"),
        # voxel reorder of a video model's activations; the grid is no multiple of the voxel in two dimensions
        dict(name="reorder_video", kind="reorder", B=1, prefix=0, T=21, Hg=45, Wg=80, suffix=0, vt=4, vh=6, vw=8,
             D=5120, inverse=False),
    ]


def _log_int(rng, lo, hi, multiple=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / multiple)) * multiple))


_LARGEST_FLOPS, _LARGEST_BYTES = 5e12, 4e9   # of a drawn case: below the largest listed one


def draw(rng):
    while True:
        kind = rng.choice(["attn_delta", "attn_delta", "attn_dense", "attn_refresh", "topk", "topk", "scores", "mlp_delta",
                           "mlp_delta", "mlp_dense", "reorder"])
        B = rng.choice([1, 1, 1, 2])
        c = rng.choice([128, 192, 192])
        if kind.startswith("attn"):
            case = dict(kind=kind, B=B, H=rng.randint(2, 40), N=_log_int(rng, 700, 115456 if kind == "attn_delta" else 30000),
                        E=rng.choice([64, 128, 128]), c=c)
            if kind == "attn_delta":
                case.update(keep=round(math.exp(rng.uniform(math.log(0.03), math.log(0.5))), 4), ragged=rng.random() < 0.3)
        elif kind == "topk":
            prev = rng.random() < 0.5
            C = _log_int(rng, 1000, 16384, 64) if prev else _log_int(rng, 1000, 115456)
            case = dict(kind=kind, R=_log_int(rng, 16, 1000 if prev else 14448), C=C,
                        k=max(1, int(C * math.exp(rng.uniform(math.log(0.03), math.log(0.5))))), prev=prev)
        elif kind == "reorder":
            case = dict(kind=kind, B=B, prefix=rng.choice([0, 0, 256, 512]), T=rng.randint(1, 32), Hg=rng.randint(16, 64),
                        Wg=rng.randint(16, 96), suffix=rng.choice([0, 0, 256]), vt=rng.choice([1, 2, 4]),
                        vh=rng.choice([4, 6, 8]), vw=rng.choice([4, 8]), D=128 * rng.randint(2, 40),
                        inverse=rng.random() < 0.5)
        else:
            case = dict(kind=kind, B=B, N=_log_int(rng, 500, 115456 if kind != "mlp_dense" else 30000), c=c,
                        D=128 * rng.randint(4, 40), F=64 * rng.randint(16, 220))
            if kind == "mlp_delta":
                case.update(keep=round(math.exp(rng.uniform(math.log(0.03), math.log(0.5))), 4), ragged=rng.random() < 0.3)
            if kind != "scores":
                case["act"] = rng.choice(["tanh", "tanh", "erf"])
        w = work(case)
        if w["flops"] <= _LARGEST_FLOPS and w["bytes"] <= _LARGEST_BYTES:
            return case


# ---- helpers ---------------------------------------------------------------------------------------------------------

def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 16 + salt)
    return g


def _randn(shape, g, scale=1.0):
    """N(0,1) * scale in bf16, made in slices so that no whole copy in 32 bits exists."""
    out = torch.empty(shape, dtype=BF16, device=DEV)
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 28):
        part = flat[i:i + (1 << 28)]
        part.copy_(torch.randn(part.shape, generator=g, device=DEV, dtype=F32) * scale)
    return out


def _nudged(x, g, sigma):
    """x plus a little noise: the same tensor one diffusion step later."""
    return x + _randn(tuple(x.shape), g, sigma)


def _kept(C, keep):
    return max(1, min(C, int(round(keep * C))))


def _lists(units, C, k, ragged, g):
    """k ascending columns per unit, one drawn from each of k equal parts of the row; ragged: a count per unit."""
    at = torch.arange(k + 1, device=DEV, dtype=torch.int64) * C // k
    lo, width = at[:-1], (at[1:] - at[:-1])
    idx = torch.empty((units, k), dtype=I32, device=DEV)
    for u in range(0, units, 1024):
        n = min(1024, units - u)
        idx[u:u + n] = (lo + (torch.rand((n, k), generator=g, device=DEV, dtype=F64) * width).long()).to(I32)
    if ragged:
        counts = torch.randint(k // 2, k + 1, (units,), generator=g, device=DEV).to(I32)
    else:
        counts = torch.full((units,), k, dtype=I32, device=DEV)
    return idx, counts


def _weights(D, F, g):
    return _randn((F, D), g, 1 / math.sqrt(D)), _randn((F,), g, 0.1), _randn((F, D), g, 1 / math.sqrt(F)), _randn((D,), g, 0.1)


def _u8(n):
    return torch.empty(max(int(n), 16), dtype=torch.uint8, device=DEV)


def _act_id(case):
    return cm.ACT_GELU_ERF if case["act"] == "erf" else cm.ACT_GELU_TANH


def _gelu(x, case):
    return torch.nn.functional.gelu(x, approximate="none" if case["act"] == "erf" else "tanh")


def _nb(case):
    return -(-case["N"] // case["c"])


def _tokens(case):
    return case["prefix"] + case["T"] * case["Hg"] * case["Wg"] + case["suffix"]


# ---- what the caller has in hand ---------------------------------------------------------------------------------------

def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def _prepare_step(case, seed):
    """A block whose caches a dense step has filled, and its inputs of the two steps that follow."""
    g = _gen(seed)
    B, H, N, E, D, F = (case[n] for n in ("B", "H", "N", "E", "D", "F"))
    inputs = {n: [_randn((B, H, N, E), g)] for n in "qkv"}
    inputs["x"] = [_randn((B, N, D), g)]
    for _ in range(2):
        for n in "qkvx":
            inputs[n].append(_nudged(inputs[n][-1], g, 0.1))
    inputs["w1"], inputs["b1"], inputs["w2"], inputs["b2"] = _weights(D, F, g)
    block = stack.Block(inputs, case["c"], _kept(N, case["keep_a"]), _kept(F, case["keep_m"]))
    stack.dense_step([block], 0)
    return dict(block=block, turn=0)


def _prepare_attn_delta(case, seed):
    g = _gen(seed)
    shape = tuple(case[n] for n in ("B", "H", "N", "E"))
    q, k, v, base = (_randn(shape, g) for _ in range(4))
    idx, counts = _lists(case["B"] * case["H"] * _nb(case), case["N"], _kept(case["N"], case["keep"]), case["ragged"], g)
    lead = (case["B"], case["H"], _nb(case))
    return dict(case=case, q=q, k=k, v=v, base=base, idx=idx.view(*lead, -1), counts=counts.view(lead),
                out=torch.empty_like(q), scale=1 / math.sqrt(case["E"]))


def _prepare_attn_dense(case, seed):
    g = _gen(seed)
    B, H, N, E = (case[n] for n in ("B", "H", "N", "E"))
    q, k, v = (_randn((B, H, N, E), g) for _ in range(3))
    colsum = torch.zeros((B, H, _nb(case), -(-N // 4) * 4), dtype=F32, device=DEV)
    s = dict(case=case, q=q, k=k, v=v, out=torch.empty_like(q), colsum=colsum, scale=1 / math.sqrt(E))
    if case["kind"] == "attn_dense":
        s["ws"] = _u8(cm.attn_dense_workspace_bytes(B, H, N))
    else:
        # normalisers of an earlier dense step: near this step's row maximum and sum
        lse = math.log(N) + 0.5 + 0.1 * torch.randn((B, H, N), generator=g, device=DEV, dtype=F32)
        s["prev_m"] = 3.5 + 0.5 * torch.randn((B, H, N), generator=g, device=DEV, dtype=F32)
        s["prev_l"] = torch.exp(lse - s["prev_m"])
        s["new_m"], s["new_l"] = torch.empty_like(lse), torch.empty_like(lse)
    return s


def _prepare_topk(case, seed):
    g = _gen(seed)
    R, C, k = case["R"], case["C"], case["k"]
    ld = -(-C // 4) * 4
    cur = torch.empty((R, ld), dtype=F32, device=DEV)
    s = dict(case=case, cur=cur[:, :C], prev=None, idx=torch.zeros((R, k), dtype=I32, device=DEV),
             counts=torch.zeros((R,), dtype=I32, device=DEV))
    if case["prev"]:   # pre-activations of chunk means: small, and a seventh of the neurons have moved
        prev = torch.empty_like(cur).normal_(0, 0.07, generator=g)
        sigma = torch.where(torch.rand(ld, generator=g, device=DEV) < 0.15, 0.02, 0.002)
        cur.normal_(0, 1, generator=g).mul_(sigma).add_(prev)
        s["prev"] = prev[:, :C]
    else:              # column sums of probabilities: positive, some columns heavier for every chunk
        weight = torch.exp(0.2 * torch.randn(ld, generator=g, device=DEV)) * (case.get("c", 192) / C)
        cur.normal_(0, 0.3, generator=g).exp_().mul_(weight)
    return s


def _prepare_scores(case, seed):
    g = _gen(seed)
    B, N, D, F, c = (case[n] for n in ("B", "N", "D", "F", "c"))
    return dict(case=case, x=_randn((B, N, D), g), w1=_randn((F, D), g, 1 / math.sqrt(D)),
                T=torch.empty((B, _nb(case), F), dtype=F32, device=DEV), ws=_u8(cm.mlp_tile_mean_workspace_bytes(B, N, D, F, c)))


def _prepare_mlp_delta(case, seed):
    """The caches hold the activations and the output of the step before; two inputs take turns, so that the caches
    change in every pass."""
    g = _gen(seed)
    B, N, D, F, c = (case[n] for n in ("B", "N", "D", "F", "c"))
    w1, b1, w2, b2 = _weights(D, F, g)
    x0 = _randn((B, N, D), g)
    a_cache = torch.zeros((B, F, -(-N // 8) * 8), dtype=BF16, device=DEV)
    o_cache = torch.empty_like(x0)
    for b in range(B):
        for r in range(0, N, 16384):
            a = _gelu(torch.nn.functional.linear(x0[b, r:r + 16384], w1, b1), case)
            a_cache[b, :, r:r + a.shape[0]] = a.t()
            o_cache[b, r:r + a.shape[0]] = torch.addmm(b2, a, w2)
    k = _kept(F, case["keep"])
    idx, counts = _lists(B * _nb(case), F, k, case["ragged"], g)
    return dict(case=case, x=[_nudged(x0, g, 0.3), _nudged(x0, g, 0.3)], w1=w1, b1=b1, w2=w2, a_cache=a_cache, o_cache=o_cache,
                idx=idx.view(B, _nb(case), k), counts=counts.view(B, -1), ws=_u8(cm.mlp_workspace_bytes(B, N, D, F, c, k)), turn=0)


def _prepare_mlp_dense(case, seed):
    g = _gen(seed)
    B, N, D, F = (case[n] for n in ("B", "N", "D", "F"))
    w1, b1, w2, b2 = _weights(D, F, g)
    x = _randn((B, N, D), g)
    return dict(case=case, x=x, w1=w1, b1=b1, w2=w2, b2=b2, out=torch.empty_like(x),
                a_cache=torch.zeros((B, F, -(-N // 8) * 8), dtype=BF16, device=DEV))


def _prepare_reorder(case, seed):
    N = _tokens(case)
    src = _randn((case["B"], N, case["D"]), _gen(seed))
    return dict(case=case, src=src, dst=torch.empty_like(src), perm=torch.empty(N, dtype=I32, device=DEV))


_PREPARE = dict(step=_prepare_step, attn_delta=_prepare_attn_delta, attn_dense=_prepare_attn_dense,
                attn_refresh=_prepare_attn_dense, topk=_prepare_topk, scores=_prepare_scores, mlp_delta=_prepare_mlp_delta,
                mlp_dense=_prepare_mlp_dense, reorder=_prepare_reorder)


# ---- one pass ----------------------------------------------------------------------------------------------------------

def run(state):
    s = state
    if "block" in s:
        blk = s["block"]
        s["turn"] += 1
        stack.sparse_step([blk], 2 - s["turn"] % 2)
        return dict(attn=blk.attn_out, mlp=blk.m_cache, activations=blk.a_cache)
    case = s["case"]
    kind = case["kind"]
    if kind == "attn_delta":
        cm.attn_sparse_delta(s["q"], s["k"], s["v"], s["idx"], s["counts"], s["base"], s["out"], case["c"], s["scale"], 1.0)
        return s["out"]
    if kind == "attn_dense":
        cm.attn_dense(s["q"], s["k"], s["v"], s["out"], s["colsum"], case["c"], s["scale"], s["ws"])
        return dict(out=s["out"], colsum=s["colsum"])
    if kind == "attn_refresh":
        cm.attn_dense_colsum_stale(s["q"], s["k"], s["v"], s["out"], s["prev_m"], s["prev_l"], s["colsum"], case["c"],
                                   s["scale"], s["new_m"], s["new_l"])
        # of the new normalisers only m + log l is defined (m may be any reference near the row maximum)
        return dict(out=s["out"], colsum=s["colsum"], lse=s["new_m"] + torch.log(s["new_l"]))
    if kind == "topk":
        cm.topk_cols(s["cur"], s["prev"], case["k"], s["idx"], s["counts"])
        return dict(idx=s["idx"], counts=s["counts"])
    if kind == "scores":
        cm.mlp_tile_mean_preact(s["x"], s["w1"], s["T"], case["c"], s["ws"])
        return s["T"]
    if kind == "mlp_delta":
        x = s["x"][s["turn"] % 2]
        s["turn"] += 1
        cm.mlp_sparse_delta(x, s["w1"], s["b1"], s["w2"], s["idx"], s["counts"], s["a_cache"], s["o_cache"], case["c"],
                            _act_id(case), s["ws"])
        return dict(out=s["o_cache"], activations=s["a_cache"])
    if kind == "mlp_dense":
        cm.mlp_dense(s["x"], s["w1"], s["b1"], s["w2"], s["b2"], s["out"], s["a_cache"], case["c"], _act_id(case))
        return dict(out=s["out"], activations=s["a_cache"])
    cm.voxel_reorder(s["src"], s["dst"], s["perm"], None, case["prefix"], case["T"], case["Hg"], case["Wg"], case["suffix"],
                     case["vt"], case["vh"], case["vw"], case["inverse"])
    return dict(rows=s["dst"].view(torch.int16), perm=s["perm"])


# ---- what a pass cannot do without ---------------------------------------------------------------------------------------

def _work_attn(case, k, passes):
    B, H, N, E = (case[n] for n in ("B", "H", "N", "E"))
    return 2 * B * H * N * E, 2 * passes * B * H * N * k * E


def _work_mlp_delta(B, N, D, F, units, k):
    bytes_ = 2 * B * N * D * 3 + 2 * 2 * F * D + 2 * 2 * B * N * k + 4 * units * k
    return bytes_, 4 * B * N * k * D


def _work_scores(B, N, D, F, units):
    return 2 * B * N * D + 2 * F * D + 4 * units * F, 2 * units * F * D + B * N * D


def work(case):
    kind = case["kind"]
    if kind == "step":
        units = case["B"] * _nb(case)
        k_a, k_m = _kept(case["N"], case["keep_a"]), _kept(case["F"], case["keep_m"])
        t, f = _work_attn(case, k_a, 2)
        args = (case["B"], case["N"], case["D"], case["F"], units)
        mb, mf = _work_mlp_delta(*args, k_m)
        sb, sf = _work_scores(*args)
        return dict(bytes=5 * t + 4 * case["H"] * units * k_a + mb + sb + 8 * units * case["F"], flops=f + mf + sf)
    if kind == "attn_delta":
        k = _kept(case["N"], case["keep"])
        if case["ragged"]:
            k = 0.75 * k
        t, f = _work_attn(case, k, 2)
        return dict(bytes=5 * t + 4 * case["B"] * case["H"] * _nb(case) * k, flops=f)
    if kind in ("attn_dense", "attn_refresh"):
        # exact column sums need every score again once its row's normaliser is known
        t, f = _work_attn(case, case["N"], 3 if kind == "attn_dense" else 2)
        rows = case["B"] * case["H"] * case["N"]
        return dict(bytes=4 * t + 4 * case["B"] * case["H"] * _nb(case) * case["N"] + (16 * rows if kind == "attn_refresh" else 0),
                    flops=f)
    if kind == "topk":
        return dict(bytes=4 * case["R"] * (case["C"] * (2 if case["prev"] else 1) + case["k"] + 1), flops=0)
    if kind == "reorder":
        return dict(bytes=4 * case["B"] * _tokens(case) * case["D"] + 4 * _tokens(case), flops=0)
    B, N, D, F = (case[n] for n in ("B", "N", "D", "F"))
    units = B * _nb(case)
    if kind == "scores":
        b, f = _work_scores(B, N, D, F, units)
    elif kind == "mlp_delta":
        b, f = _work_mlp_delta(B, N, D, F, units, _kept(F, case["keep"]) * (0.75 if case["ragged"] else 1))
    else:
        b, f = 2 * (2 * B * N * D + 2 * F * D + B * N * F), 4 * B * N * F * D
    return dict(bytes=b, flops=f)


def tolerance(case):
    kind = case["kind"]
    if kind in ("topk", "reorder"):
        return "exact"
    if kind == "scores":      # 32-bit sums of a mean carried in about 16 bits: 2.5e-6 off the 64-bit result
        return {"rel": 1e-5}
    return {"rel": 1e-2}      # bf16 outputs: up to 2.3e-3 off the 64-bit result


# ---- the same results in 64 bits ---------------------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind in ("topk", "reorder", "step"):   # whole numbers and bytes; the whole step's choices hang on roundings
        return None
    s = prepare(case, seed)
    return dict(attn_delta=_exact_attn_delta, attn_dense=_exact_attn_dense, attn_refresh=_exact_attn_dense,
                scores=_exact_scores, mlp_delta=_exact_mlp_delta, mlp_dense=_exact_mlp_dense)[kind](case, s)


def _exact_attn_delta(case, s):
    B, H, N, c = (case[n] for n in ("B", "H", "N", "c"))
    k = s["idx"].shape[-1]
    out = s["base"].double()
    lane = torch.arange(k, device=DEV)
    step = max(1, (1 << 25) // (c * k))
    for b in range(B):
        for h in range(H):
            kh, vh, qh = s["k"][b, h].double(), s["v"][b, h].double(), s["q"][b, h].double()
            pad = _nb(case) * c - N
            qh = torch.cat([qh, qh.new_zeros((pad, qh.shape[1]))]).view(-1, c, qh.shape[1])
            delta = torch.empty_like(qh)
            for u in range(0, qh.shape[0], step):
                cols = s["idx"][b, h, u:u + step].long()
                scores = torch.bmm(qh[u:u + step], kh[cols].transpose(1, 2).contiguous()) * s["scale"]
                dead = lane[None, :] >= s["counts"][b, h, u:u + step, None]
                scores.masked_fill_(dead[:, None, :], -math.inf)
                delta[u:u + step] = torch.bmm(torch.softmax(scores, -1), vh[cols])
            out[b, h] += delta.view(-1, qh.shape[-1])[:N]
    return out


def _exact_attn_dense(case, s):
    B, H, N, E, c = (case[n] for n in ("B", "H", "N", "E", "c"))
    out = torch.empty((B, H, N, E), dtype=F64, device=DEV)
    colsum = torch.zeros(tuple(s["colsum"].shape), dtype=F64, device=DEV)
    lse = torch.empty((B, H, N), dtype=F64, device=DEV)
    for b in range(B):
        for h in range(H):
            kt, vh = s["k"][b, h].double().t().contiguous(), s["v"][b, h].double()
            for u in range(_nb(case)):
                rows = slice(u * c, min(N, (u + 1) * c))
                scores = (s["q"][b, h, rows].double() @ kt) * s["scale"]
                lse[b, h, rows] = torch.logsumexp(scores, -1)
                p = torch.exp(scores - lse[b, h, rows, None])
                out[b, h, rows] = p @ vh
                if "prev_m" in s:
                    norm = s["prev_m"][b, h, rows].double() + torch.log(s["prev_l"][b, h, rows].double())
                    p = torch.exp(scores - norm[:, None])
                colsum[b, h, u, :N] = p.sum(0)
    return dict(out=out, colsum=colsum, lse=lse) if "prev_m" in s else dict(out=out, colsum=colsum)


def _exact_scores(case, s):
    x, w = s["x"], s["w1"].double().t().contiguous()
    mean = torch.stack([torch.stack([xb[r:r + case["c"]].double().mean(0) for r in range(0, case["N"], case["c"])]) for xb in x])
    return torch.stack([m @ w for m in mean])


def _exact_mlp_delta(case, s):
    c, N = case["c"], case["N"]
    out, acts = s["o_cache"].double(), s["a_cache"].double()
    x, w1, b1, w2 = s["x"][0], s["w1"], s["b1"].double(), s["w2"]
    counts = s["counts"].tolist()
    for b in range(case["B"]):
        for u in range(_nb(case)):
            rows = slice(u * c, min(N, (u + 1) * c))
            f = s["idx"][b, u, :counts[b][u]].long()
            a = _gelu(x[b, rows].double() @ w1[f].double().t().contiguous() + b1[f], case)
            out[b, rows] += (a - acts[b, f, rows].t()) @ w2[f].double()
            acts[b, f, rows] = a.t()
    return dict(out=out, activations=acts)


def _exact_mlp_dense(case, s):
    w1t, w2, b1, b2 = s["w1"].double().t().contiguous(), s["w2"].double(), s["b1"].double(), s["b2"].double()
    out = torch.empty(tuple(s["x"].shape), dtype=F64, device=DEV)
    acts = s["a_cache"].double()
    for b in range(case["B"]):
        for r in range(0, case["N"], 4096):
            a = _gelu(s["x"][b, r:r + 4096].double() @ w1t + b1, case)
            acts[b, :, r:r + a.shape[0]] = a.t()
            out[b, r:r + a.shape[0]] = a @ w2 + b2
    return dict(out=out, activations=acts)
