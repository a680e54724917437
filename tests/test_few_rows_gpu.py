"""Calls with few rows against a long other side: the forward whose four waves share 32 query rows and deal the keys out among
themselves, and the backward's streamed side in parts (two or more workgroups per 128 fixed rows, whose float32 sums a
second kernel adds), at the edges of parts and tiles, with M != N, strided tensors and one upstream gradient alone,
against the float64 oracle (the repository's bf16 tolerance)."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2511_19797_amd as tvm
from oracle import tvmattn_oracle as orc
from paper_2511_19797_amd import workloads as wl
from tests import dispatch_cases as dc
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

# M, N: queries and keys both cut / keys alone / queries alone; whole tiles, one row over, parts of unequal length; the fewest
# keys the shared-rows forward takes, a last wave without a whole tile, one and two workgroups
SIZES = [(1024, 1024), (1025, 1089), (40, 1100), (1537, 33), (64, 2049), (1, 128), (33, 129), (31, 257)]


@pytest.mark.parametrize("d", [8, 32, 40, 64, 72, 96, 104, 128])
@pytest.mark.parametrize("M,N", SIZES)
def test_against_oracle(M, N, d):
    w = dataclasses.replace(wl.custom(1, 2, N, d, "bf16"), M=M)
    print(f"[case] {w}", flush=True)
    inp = wl.make_inputs(w, 100 + d)
    fwd, grads = pu.run_gpu(inp)
    pu.check_heads(w, inp, fwd, grads, pu.all_heads(w))


@pytest.mark.parametrize("H,M,N,d,few", dc.FORWARD_LINES)
def test_forward_on_both_sides_of_the_lines(H, M, N, d, few):
    """The last block count that the forward for few rows takes and the first that it leaves: sampled heads against the oracle."""
    w = dataclasses.replace(wl.custom(1, H, N, d, "bf16"), M=M)
    print(f"[case] {w} few={few}", flush=True)
    inp = wl.make_inputs(w, 21)
    fwd = tvm.tvmattn_jvp_fwd(*[inp[n].cuda() for n in ("q", "k", "v", "tq", "tk", "tv")])
    for h in (0, H - 1):
        ref = orc.attn_jvp_fwd_head(*[wl.to_f64(inp[n][0, h]) for n in wl.NAMES[:6]], None)
        for n, g, r in zip(pu.FWD_NAMES, fwd, ref):
            assert pu.rel_err(g[0, h].float().cpu().numpy(), r) <= pu.TOL["bf16"], (h, n)


@pytest.mark.parametrize("d", [64, 72, 128])
def test_strided_static_and_small_workspace(d):
    """[B,N,H,D] tensors against dense ones and the static-scratch call, bit for bit; a workspace of the row vectors alone
    takes the route without parts: the same to bf16 rounding."""
    w = dataclasses.replace(wl.custom(2, 2, 1300, d, "bf16"), M=1100)
    inp = {n: t.cuda() for n, t in wl.make_inputs(w, 5).items()}
    names = ("q", "k", "v", "tq", "tk", "tv")
    six = [inp[n] for n in names]
    fwd = tvm.tvmattn_jvp_fwd(*six)
    plain = tvm.tvmattn_jvp_bwd(*six, *fwd, inp["gO"], inp["gTO"])
    static = tvm.tvmattn_jvp_bwd_static(*six, *fwd, inp["gO"], inp["gTO"])
    nhd = lambda t: t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    strided = tvm.tvmattn_jvp_bwd(*[nhd(t) for t in six], nhd(fwd[0]), nhd(fwd[1]), *fwd[2:], nhd(inp["gO"]), nhd(inp["gTO"]))
    rows = 3 * ((2 * 2 * 1100 * 4 + 255) // 256 * 256)
    assert tvm.tvmattn_jvp_bwd_workspace_bytes(inp["q"], k=inp["k"]) > rows
    whole = tvm.tvmattn_jvp_bwd(*six, *fwd, inp["gO"], inp["gTO"],
                                workspace=torch.empty(rows, dtype=torch.uint8, device="cuda"))
    for n, a, b, c, e in zip(pu.BWD_NAMES, plain, static, strided, whole):
        assert torch.equal(a, b), n
        assert torch.equal(a, c), n
        assert pu.rel_err(a.float().cpu(), e.float().cpu()) <= 2 ** -7, n  # one bf16 rounding either side, at the largest


@pytest.mark.parametrize("d", [8, 72, 104, 128])
@pytest.mark.parametrize("which", ["gO", "gTO"])
def test_one_upstream_gradient(which, d):
    w = dataclasses.replace(wl.custom(1, 1, 1500, d, "bf16"), M=1030)
    print(f"[case] {w} {which}", flush=True)
    inp = wl.make_inputs(w, 11)
    dev = {n: t.cuda() for n, t in inp.items()}
    six = [dev[n] for n in ("q", "k", "v", "tq", "tk", "tv")]
    fwd = tvm.tvmattn_jvp_fwd(*six)
    got = tvm.tvmattn_jvp_bwd(*six, *fwd, dev["gO"] if which == "gO" else None, dev["gTO"] if which == "gTO" else None)
    a = [wl.to_f64(inp[n][0, 0]) for n in wl.NAMES]
    a[wl.NAMES.index("gTO" if which == "gO" else "gO")] = np.zeros_like(a[wl.NAMES.index("gO")])
    ref = orc.attn_jvp_bwd_head(*a, None)
    for n, g, r in zip(pu.BWD_NAMES, got, ref):
        if g is not None:
            assert pu.rel_err(g[0, 0].float().cpu().numpy(), r) <= pu.TOL["bf16"], n


def test_a_wave_without_finite_scores():
    """All keys of one wave's tiles at score -inf (an overflowing product): the rows keep the other keys' result."""
    inp = {n: t.cuda() for n, t in wl.make_inputs(wl.custom(1, 1, 128, 32, "bf16"), 5).items()}
    q, k = inp["q"].clone(), inp["k"].clone()
    q[..., 0], k[..., 0] = 1e20, 0.0
    keep = [j for j in range(128) if not 32 <= j < 64]  # keys 32..63 are the second wave's tile
    k[0, 0, 32:64, 0] = -1e38
    z = torch.zeros_like(q)
    o, to, lse, stats = tvm.tvmattn_jvp_fwd(q, k, inp["v"], z, z, inp["tv"])
    args = (q[0, 0], k[0, 0, keep], inp["v"][0, 0, keep], z[0, 0], z[0, 0, keep], inp["tv"][0, 0, keep])
    ref = orc.attn_jvp_fwd_head(*[wl.to_f64(t.cpu()) for t in args], None)
    for g, r in zip((o, to, lse), ref):
        assert pu.rel_err(g[0, 0].double().cpu().numpy(), r) <= pu.TOL["bf16"]


@pytest.mark.parametrize("d", [8, 24, 32, 40, 64, 72, 96, 104, 128])
@pytest.mark.parametrize("H,M,N", [(2, 200, 130), (130, 130, 260), (520, 70, 33), (3, 50, 63)])
def test_gO_alone_both_ways_to_store(H, M, N, d):
    """The ordinary backward on few and on many workgroups, on rows that fill no workgroup and no wave: results straight from
    the accumulators and as whole rows, ragged on both sides, sampled heads against the oracle; nothing is written beyond a
    tensor's rows."""
    w = dataclasses.replace(wl.custom(1, H, N, d, "bf16"), M=M)
    print(f"[case] {w} gO alone", flush=True)
    inp = wl.make_inputs(w, 17)
    dev = {n: t.cuda() for n, t in inp.items()}
    six = [dev[n] for n in ("q", "k", "v", "tq", "tk", "tv")]
    fwd = tvm.tvmattn_jvp_fwd(*six)
    room = [torch.full((H * rows * d + 4096,), float("nan"), dtype=torch.bfloat16, device="cuda") for rows in (M, N, N)]
    out = [r[:H * rows * d].view(1, H, rows, d) for r, rows in zip(room, (M, N, N))]
    tvm.tvmattn_jvp_bwd(*six, *fwd, dev["gO"], None, out=(*out, None, None, None))
    torch.cuda.synchronize()
    for r, o in zip(room, out):
        assert bool(torch.isnan(r[o.numel():].float()).all()) and not bool(torch.isnan(o.float()).any())
    for h in (0, H // 2, H - 1):
        a = [wl.to_f64(inp[n][0, h]) for n in wl.NAMES]
        a[wl.NAMES.index("gTO")] = np.zeros_like(a[wl.NAMES.index("gO")])
        for n, g, r in zip(pu.BWD_NAMES, out, orc.attn_jvp_bwd_head(*a, None)):
            assert pu.rel_err(g[0, h].float().cpu().numpy(), r) <= pu.TOL["bf16"], (h, n)


@pytest.mark.parametrize("d", [104, 128])
@pytest.mark.parametrize("H,M,N", [(2, 300, 40), (2, 40, 300), (130, 97, 33), (200, 33, 96), (3, 95, 64)])
def test_tangent_and_a_short_other_side_both_ways_to_store(H, M, N, d):
    """Head dims above 96 with 64 rows or fewer on one side: the generic-order kernel of the other side stores straight from the
    accumulators or whole rows; both gradients and gTO alone, sampled heads against the oracle."""
    w = dataclasses.replace(wl.custom(1, H, N, d, "bf16"), M=M)
    print(f"[case] {w}", flush=True)
    inp = wl.make_inputs(w, 19)
    fwd, grads = pu.run_gpu(inp)
    pu.check_heads(w, inp, fwd, grads, [(0, 0), (0, H - 1)])
    dev = {n: t.cuda() for n, t in inp.items()}
    alone = tvm.tvmattn_jvp_bwd(*[dev[n] for n in ("q", "k", "v", "tq", "tk", "tv")], *fwd, None, dev["gTO"])
    for h in (0, H - 1):
        a = [wl.to_f64(inp[n][0, h]) for n in wl.NAMES]
        a[wl.NAMES.index("gO")] = np.zeros_like(a[wl.NAMES.index("gO")])
        for n, g, r in zip(pu.BWD_NAMES, alone, orc.attn_jvp_bwd_head(*a, None)):
            assert pu.rel_err(g[0, h].float().cpu().numpy(), r) <= pu.TOL["bf16"], (h, n)
