"""The float32 matrix-core kernels against the float64 oracle, at the edges of their tiles (16 rows on either side, four
waves on every fourth tile of the streamed side) and of their padded head dims (32, 64, 96, 128), with M != N, strided
inputs, and one upstream gradient alone.

Tolerance per tensor, max |gpu - ref| / max |ref|: a sum of n float32 products is off by at most about n 2^-24 of the
sum of the terms' sizes, n <= d + N here, and the scores' error (|z| up to about 20, d terms) carries into every
probability; 1e-4 is the repository's bound for the float32 path and covers both."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2511_19797_amd as tvm
from oracle import tvmattn_oracle as orc
from paper_2511_19797_amd import workloads as wl
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [4, 28, 32, 36, 64, 68, 96, 100, 128])
def test_tile_edges(d):
    for M, N in ((1, 1), (15, 17), (16, 16), (17, 63), (64, 65), (80, 64), (33, 130)):
        w = dataclasses.replace(wl.custom(1, 2, N, d, "f32"), M=M)
        print(f"[case] {w}", flush=True)
        inp = wl.make_inputs(w, 7 + d)
        fwd, grads = pu.run_gpu(inp)
        pu.check_heads(w, inp, fwd, grads, pu.all_heads(w))


@pytest.mark.parametrize("H,M,N,d", [(4096, 4, 4, 16), (4096, 5, 4, 16), (4095, 1, 1, 64), (4096, 1, 1, 64), (1024, 4, 4, 128),
                                     (64, 16, 1, 128), (65, 16, 1, 128), (4096, 1, 16, 100), (4096, 1, 17, 100), (4096, 8, 8, 104),
                                     (3, 1, 1, 4), (3, 2, 2, 40), (3, 1, 2, 24)])
def test_few_rows_on_both_sides_of_the_lines(H, M, N, d):
    """Around the row and head counts where the kernel family changes, for the forward, the backward and the backward with gO
    alone: sampled heads against the oracle, and every element against the plain-ALU kernels."""
    w = dataclasses.replace(wl.custom(1, H, N, d, "f32"), M=M)
    print(f"[case] {w}", flush=True)
    inp = wl.make_inputs(w, 3 + d)
    fwd, grads = pu.run_gpu(inp)
    pu.check_heads(w, inp, fwd, grads, [(0, 0), (0, H // 2), (0, H - 1)])
    # Against the plain-ALU kernels an error counts relative to the tensor's largest entry, or absolutely where that is below
    # one: with a single key the gradients of q and k are exactly zero (P = 1), and what either family leaves of them is the
    # difference of two d-term sums of O(1) products, at most d 2^-24 of the sum of their sizes (d^2 2^-24 x O(1) < 1e-3, in
    # practice 1e-6).
    near = lambda a, b: float((a - b).abs().max()) <= pu.TOL["f32"] * max(1.0, float(b.abs().max()))
    pfwd, pgrads = pu.run_gpu(inp, flags=tvm.TVMATTN_FLAG_PLAIN_ALU)
    for n, a, b in zip(pu.FWD_NAMES + pu.BWD_NAMES, fwd + tuple(grads), pfwd + tuple(pgrads)):
        assert near(a, b), n
    dev = {n: t.cuda() for n, t in inp.items()}
    six = [dev[n] for n in ("q", "k", "v", "tq", "tk", "tv")]
    alone, plain = (tvm.tvmattn_jvp_bwd(*six, *f, dev["gO"], None, flags=fl)
                    for f, fl in ((fwd, 0), (pfwd, tvm.TVMATTN_FLAG_PLAIN_ALU)))
    for a, b in zip(alone[:3], plain[:3]):
        assert near(a, b)


@pytest.mark.parametrize("d", [32, 72, 128])
@pytest.mark.parametrize("which", ["gO", "gTO"])
def test_one_upstream_gradient(d, which):
    """Strided [B,N,H,D] inputs, one upstream gradient: the oracle with the other one zero."""
    w = dataclasses.replace(wl.custom(2, 2, 70, d, "f32"), M=45)
    print(f"[case] {w} {which}", flush=True)
    inp = wl.make_inputs(w, 11)
    dev = {n: t.permute(0, 2, 1, 3).contiguous().cuda().permute(0, 2, 1, 3) for n, t in inp.items()}
    six = [dev[n] for n in ("q", "k", "v", "tq", "tk", "tv")]
    o, to, lse, stats = tvm.tvmattn_jvp_fwd(*six)
    got = tvm.tvmattn_jvp_bwd(*six, o, to, lse, stats, *[dev[n] if n == which else None for n in ("gO", "gTO")])
    torch.cuda.synchronize()
    for b, h in pu.all_heads(w):
        a = [wl.to_f64(inp[n][b, h]) * (n not in ("gO", "gTO") or n == which) for n in wl.NAMES]
        ref = orc.attn_jvp_bwd_head(*a, None)
        for n, (g, r) in enumerate(zip(got, ref)):
            if which == "gO" and n >= 3:
                assert g is None
            else:
                assert pu.rel_err(g[b, h].double().cpu().numpy(), r) <= pu.TOL["f32"], (b, h, pu.BWD_NAMES[n])


def test_keys_without_weight():
    """Every key of one wave's tiles at score -inf (an overflowing product): the rows keep the other keys' result."""
    inp = {n: t.cuda() for n, t in wl.make_inputs(wl.custom(1, 1, 64, 32, "f32"), 5).items()}
    q, k = inp["q"].clone(), inp["k"].clone()
    q[..., 0] = 1e20
    k[..., 0] = 0.0
    k[0, 0, 16:32, 0] = -1e38       # keys 16..31 are the second wave's tile
    o, to, lse, stats = tvm.tvmattn_jvp_fwd(q, k, inp["v"], torch.zeros_like(q), torch.zeros_like(k), inp["tv"])
    keep = [j for j in range(64) if not 16 <= j < 32]
    ref = orc.attn_jvp_fwd_head(*[wl.to_f64(t.cpu()) for t in (q[0, 0], k[0, 0, keep], inp["v"][0, 0, keep],
                                                              torch.zeros_like(q)[0, 0], torch.zeros_like(k)[0, 0, keep],
                                                              inp["tv"][0, 0, keep])], None)
    for g, r in zip((o, to, lse), ref):
        assert pu.rel_err(g[0, 0].double().cpu().numpy(), r) <= pu.TOL["f32"]
