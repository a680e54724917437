"""The work that a user of this library has it do, as timed cases.

Two kinds of pass, both through the package's public entry points:

* "attention": the attention with its tangent on tensors the caller holds, `tvmattn_jvp_fwd` and, where the pass is a
  training step, `tvmattn_jvp_bwd`.  `step` says which: "train" is the forward and the backward through both outputs;
  "detached" the forward and the backward of the output alone (gTO=None: the tangent enters the target as a constant,
  the cheaper training variant); "tangent" the backward of the tangent alone (gO=None); "forward" the forward that
  saves nothing.
* "block": one normalised DiT block with tangent (`block.block_jvp_fwd`, `block.block_jvp_bwd`): AdaLN, the four linear
  layers, QK-norm, attention, GELU and gates on a token stream.  "train" is forward and full backward, "forward" the
  forward alone (a target network, sampling).

The sizes are those of the package's workloads (`workloads.py`: DiT-B/2 and DiT-XL/2 at 256 and 512 px, the
long-sequence shape, the kernel-benchmark shapes, cross-attention), with ragged ones between them.
"""
import math

import torch

import paper_2511_19797_amd as tvm
from paper_2511_19797_amd import block

EPS = 1e-6


def _attention(name, B, H, M, N, d, dtype="bf16", step="train", tangent_std=1.0, key_scale=1.0):
    return {"name": name, "kind": "attention", "B": B, "H": H, "M": M, "N": N, "d": d, "dtype": dtype, "step": step,
            "tangent_std": tangent_std, "key_scale": key_scale}


def _block(name, B, T, H, d, step="train"):
    return {"name": name, "kind": "block", "B": B, "T": T, "H": H, "d": d, "step": step}


def listed():
    return [
        # the plumbing case that every set-up runs first, float32: what one call costs when there is next to no work
        _attention("tiny_f32", 1, 2, 64, 64, 32, dtype="f32"),
        # a float32 training step, as in gradient checks and full-precision runs: DiT-B/2 at 256 px, batch 4
        _attention("f32_256px", 4, 12, 256, 256, 64, dtype="f32"),
        # the paper's own head split (18 x 64) at 256 px, the tangent taken as a constant: ordinary attention backward
        _attention("detached_256px", 32, 18, 256, 256, 64, step="detached"),
        # DiT-XL/2 at 256 px, a training step: short sequences, many heads
        _attention("xl_256px", 32, 16, 256, 256, 72),
        # DiT-XL/2 at 512 px, a training step: the headline workload
        _attention("xl_512px", 16, 16, 1024, 1024, 72, tangent_std=0.1),
        # long sequences with a sharp softmax and wide heads
        _attention("long_4096", 2, 24, 4096, 4096, 128, key_scale=2.0),
        # one head of the kernel benchmark: few rows to hand out to 256 compute units
        _attention("one_head_4096", 1, 1, 4096, 4096, 64),
        # image tokens attending to fewer conditioning tokens, neither count a multiple of a tile
        _attention("cross_ragged", 8, 16, 1000, 250, 72, tangent_std=0.1),
        # a DiT-XL/2 block at 512 px and at 256 px, a training step at the batch one GPU takes
        _block("block_512px", 16, 1024, 16, 72),
        _block("block_256px", 32, 256, 16, 72),
        # a small batch of cropped images (a token count that no tile divides) through a DiT-B/2 block, a training step
        _block("block_small", 2, 250, 12, 64),
        # one image through a DiT-XL/2 block, forward with tangent only
        _block("block_one_image", 1, 256, 16, 72, step="forward"),
    ]


# A drawn case stays under the listed long-sequence shape (bf16), the listed float32 case, and the listed large block.
_MOST_BF16 = 24 * 4096 * 4096 * 128
_MOST_F32 = 4 * 12 * 256 * 256 * 64
_MOST_ROWS = 16 * 1024


def _spread(rng, lo, hi):
    """An integer in [lo, hi], its logarithm evenly spread."""
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    if rng.random() < 0.35:
        H, d = rng.choice([(6, 64), (12, 64), (16, 64), (16, 72), (18, 64), (4, 72), (8, 128)])
        T = _spread(rng, 32, 1024)
        B = _spread(rng, 1, min(32, _MOST_ROWS // T))
        return {k: v for k, v in _block("", B, T, H, d, "forward" if rng.random() < 0.25 else "train").items() if k != "name"}
    f32 = rng.random() < 0.2
    most = _MOST_F32 if f32 else _MOST_BF16
    step = "train" if f32 else rng.choice(["train", "train", "train", "detached", "tangent", "forward"])
    d = 8 * rng.randint(4, 8 if f32 else 16)
    N = _spread(rng, 32, 512 if f32 else 8192)
    M = N if rng.random() < 0.75 else _spread(rng, 32, 512 if f32 else 4096)
    wide = max(d, 64)
    heads = max(1, min(512, most // (M * N * wide), _MOST_ROWS * 16 // max(M, N)))
    H = _spread(rng, 1, min(24, heads))
    B = _spread(rng, 1, max(1, min(32, heads // H)))
    case = _attention("", B, H, M, N, d, "f32" if f32 else "bf16", step, rng.choice([0.1, 1.0]), rng.choice([1.0, 1.0, 2.0]))
    return {k: v for k, v in case.items() if k != "name"}


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape, std=1.0, mean=0.0, dtype=torch.float32):
        t = torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32)
        return (t * std + mean).to(dtype)

    if case["kind"] == "attention":
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        B, H, d = case["B"], case["H"], case["d"]
        qs, ks = (B, H, case["M"], d), (B, H, case["N"], d)
        st = case["tangent_std"]
        state = {"q": normal(*qs, dtype=dt), "k": normal(*ks, std=case["key_scale"], dtype=dt), "v": normal(*ks, dtype=dt),
                 "tq": normal(*qs, std=st, dtype=dt), "tk": normal(*ks, std=st, dtype=dt), "tv": normal(*ks, std=st, dtype=dt)}
        if case["step"] != "forward":
            state["gO"] = None if case["step"] == "tangent" else normal(*qs, dtype=dt)
            state["gTO"] = None if case["step"] == "detached" else normal(*qs, dtype=dt)
        return {"case": case, "t": state}
    B, T, H, d = case["B"], case["T"], case["H"], case["d"]
    C, bf = H * d, torch.bfloat16
    names = block.MODS
    state = {"x": normal(B, T, C, dtype=bf), "tx": normal(B, T, C, dtype=bf),
             "mods": {n: normal(B, C) for n in names}, "tmods": {n: normal(B, C) for n in names},
             "params": {"wqkv": normal(3 * C, C, std=C ** -0.5, dtype=bf), "bqkv": normal(3 * C, std=0.1, dtype=bf),
                        "gq": normal(d, std=0.2, mean=1.0), "gk": normal(d, std=0.2, mean=1.0),
                        "wo": normal(C, C, std=C ** -0.5, dtype=bf), "bo": normal(C, std=0.1, dtype=bf),
                        "w1": normal(4 * C, C, std=C ** -0.5, dtype=bf), "b1": normal(4 * C, std=0.1, dtype=bf),
                        "w2": normal(C, 4 * C, std=(4 * C) ** -0.5, dtype=bf), "b2": normal(C, std=0.1, dtype=bf)}}
    if case["step"] == "train":
        state["gz"], state["gtz"] = normal(B, T, C, dtype=bf), normal(B, T, C, dtype=bf)
    return {"case": case, "t": state}


def run(state):
    case, t = state["case"], state["t"]
    if case["kind"] == "attention":
        six = (t["q"], t["k"], t["v"], t["tq"], t["tk"], t["tv"])
        if case["step"] == "forward":
            return tvm.tvmattn_jvp_fwd(*six, save=False)[:2]
        o, to, lse, stats = tvm.tvmattn_jvp_fwd(*six)
        grads = tvm.tvmattn_jvp_bwd(*six, o, to, lse, stats, t["gO"], t["gTO"])
        return (o, to, lse, stats) + tuple(grads)
    args = (t["x"], t["tx"], t["mods"], t["tmods"], t["params"], case["H"], EPS, EPS)
    z, tz, saved = block.block_jvp_fwd(*args)
    if case["step"] == "forward":
        return z, tz
    return z, tz, block.block_jvp_bwd(*args, saved, t["gz"], t["gtz"])


def work(case):
    """Multiplications and additions of the definition at the true head dim (no padding, no recompute); every input of
    the pass read once, every output written once."""
    step = case["step"]
    # products of M x N x d multiply-adds: six forward; backward fifteen through both outputs, five of the ordinary
    # attention backward, twelve through the tangent alone
    products = 6 + {"train": 15, "detached": 5, "tangent": 12, "forward": 0}[step]
    if case["kind"] == "attention":
        e = 4 if case["dtype"] == "f32" else 2
        B, H, M, N, d = case["B"], case["H"], case["M"], case["N"], case["d"]
        q, k = B * H * M * d * e, B * H * N * d * e
        nbytes = 2 * q + 4 * k + 2 * q                       # q, tq, k, v, tk, tv in; o, to out
        nbytes += {"train": 2 * q + 2 * q + 4 * k, "detached": q + q + 2 * k, "tangent": q + 2 * q + 4 * k, "forward": 0}[step]
        nbytes += 0 if step == "forward" else 8 * B * H * M  # lse, stats
        return {"bytes": nbytes, "flops": 2 * products * B * H * M * N * d}
    B, T, H, d = case["B"], case["T"], case["H"], case["d"]
    C = H * d
    linear = 2 * 2 * B * T * 12 * C * C                      # four layers of 12 C^2 weights, token and tangent
    weights = 2 * (12 * C * C + 9 * C)
    train = step == "train"
    return {"bytes": (8 if train else 4) * B * T * C * 2 + (2 if train else 1) * (weights + 12 * B * C * 4),
            "flops": linear * (3 if train else 1) + 2 * products * B * H * T * T * d}


def tolerance(case):
    """About four times what the outputs are off from the same quantities in float64: at most 7e-7 and, at single
    elements, 4e-6 (float32 attention), 3.0e-3 and 5e-2 (bf16 attention); in the block 2e-3 to 1.3e-2 for most gradients
    and up to 2.7e-2 for those of the QK-norm gains (sums of large terms that cancel), 1.1e-1 at single elements."""
    if case["kind"] == "attention":
        return {"rel": 3e-6, "max": 5e-5} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.2}
    return {"rel": 3e-2, "max": 0.45}


def _rms64(t, tt):
    """RMSNorm without gain over the last dimension, and its tangent, in float64."""
    n = t.shape[-1]
    r = torch.rsqrt((t * t).sum(-1, keepdim=True) / n + EPS)
    return t * r, tt * r - t * r ** 3 * ((t * tt).sum(-1, keepdim=True) / n)


def _attention64(q, k, v, tq, tk, tv):
    """The definition on [..., M, d] and [..., N, d] tensors: (o, to, lse, stats)."""
    a = q.shape[-1] ** -0.5
    z = a * (q @ k.transpose(-1, -2))
    zt = a * (tq @ k.transpose(-1, -2) + q @ tk.transpose(-1, -2))
    p = torch.softmax(z, -1)
    stats = (p * zt).sum(-1)
    return p @ v, (p * (zt - stats.unsqueeze(-1))) @ v + p @ tv, torch.logsumexp(z.detach(), -1), stats


def _exact_attention(case, t):
    """Head by head: the score matrices of one head at a time are materialised."""
    B, H, step = case["B"], case["H"], case["step"]
    train = step != "forward"
    names = ("q", "k", "v", "tq", "tk", "tv")
    outs = None
    for b in range(B):
        for h in range(H):
            six = [t[n][b, h].double().requires_grad_(train) for n in names]
            o, to, lse, stats = _attention64(*six)
            parts = [o.detach(), to.detach()]
            if train:
                loss = 0
                if t["gO"] is not None:
                    loss = loss + (t["gO"][b, h].double() * o).sum()
                if t["gTO"] is not None:
                    loss = loss + (t["gTO"][b, h].double() * to).sum()
                g = torch.autograd.grad(loss, six, allow_unused=True)
                if step == "detached":
                    g = list(g[:3]) + [None] * 3
                parts += [lse, stats.detach()] + list(g)
            if outs is None:
                outs = [None if p is None else torch.empty(B, H, *p.shape, dtype=torch.float64, device=p.device) for p in parts]
            for out, p in zip(outs, parts):
                if out is not None:
                    out[b, h] = p
    return tuple(outs)


def _exact_block(case, t):
    B, T, H, d = case["B"], case["T"], case["H"], case["d"]
    C, train = H * d, case["step"] == "train"
    leaf = lambda s: s.double().requires_grad_(train)
    x, tx = leaf(t["x"]), leaf(t["tx"])
    mods, tmods, w = ({n: leaf(s) for n, s in t[key].items()} for key in ("mods", "tmods", "params"))
    unit = {n: [s.unsqueeze(1) for s in _rms64(mods[n], tmods[n])] for n in mods}

    def modulate(u, tu, a, b):
        n, tn = _rms64(u, tu)
        (a, ta), (b, tb) = unit[a], unit[b]
        return n * a + b, tn * a + n * ta + tb

    def gate(u, tu, c, h, th):
        c, tc = unit[c]
        return u + c * h, tu + c * th + tc * h

    def linear(u, tu, weight, bias):
        return u @ w[weight].T + w[bias], tu @ w[weight].T

    def gelu(u, tu):
        s = math.sqrt(2 / math.pi)
        th = torch.tanh(s * (u + 0.044715 * u ** 3))
        slope = 0.5 * (1 + th) + 0.5 * u * (1 - th * th) * s * (1 + 3 * 0.044715 * u * u)
        return 0.5 * u * (1 + th), slope * tu

    qkv, tqkv = (s.view(B, T, 3, H, d) for s in linear(*modulate(x, tx, "a1", "b1"), "wqkv", "bqkv"))
    heads = lambda s, i: s[:, :, i].permute(0, 2, 1, 3)
    (q, tq), (k, tk), (v, tv) = ((heads(qkv, i), heads(tqkv, i)) for i in range(3))
    (q, tq), (k, tk) = (_rms64(q, tq), _rms64(k, tk))
    o, to = _attention64(q * w["gq"], k * w["gk"], v, tq * w["gq"], tk * w["gk"], tv)[:2]
    rows = lambda s: s.permute(0, 2, 1, 3).reshape(B, T, C)
    x1, tx1 = gate(x, tx, "c1", *linear(rows(o), rows(to), "wo", "bo"))
    h2 = linear(*gelu(*linear(*modulate(x1, tx1, "a2", "b2"), "w1", "b1")), "w2", "b2")
    z, tz = gate(x1, tx1, "c2", *h2)
    if not train:
        return z, tz
    leaves = {"x": x, "tx": tx}
    for n in mods:                                           # the shifts share their names with two biases
        key = "m" + n if n in w else n
        leaves[key], leaves["t" + key] = mods[n], tmods[n]
    leaves.update(w)
    grads = torch.autograd.grad((t["gz"].double() * z).sum() + (t["gtz"].double() * tz).sum(), list(leaves.values()))
    return z.detach(), tz.detach(), dict(zip(leaves, grads))


def exact(case, seed):
    """What `run` returns, from the definitions in float64 on the stored inputs."""
    t = prepare(case, seed)["t"]
    return _exact_attention(case, t) if case["kind"] == "attention" else _exact_block(case, t)
