"""Attention launches that cut each key walk into parts (small launches), against plain torch in 64 bits."""
import math

import numpy as np
import pytest
import torch

from gpu_helpers import TOL, note, scale_of
from paper_2602_04361_amd import sparvar as sv

pytestmark = pytest.mark.gpu


def check(got, ref, what):
    tol = TOL["f32" if got.dtype == torch.float32 else "bf16"]
    err = (got.double() - ref).abs()
    assert torch.isfinite(got.float()).all(), what
    assert err.max() <= tol["max_abs"] and err.mean() <= tol["mean_abs"], (what, err.max(), err.mean())


def cache(B, H, n, d, seed, extra, dtype=torch.bfloat16):
    """K and V as prefixes of longer caches, Q rows as a slice of a longer tensor."""
    gen = torch.Generator("cuda").manual_seed(seed)
    x = [torch.randn(B, H, n + extra, d, device="cuda", generator=gen).to(dtype) for _ in range(3)]
    return [t[:, :, :n] for t in x]


BF, F32 = torch.bfloat16, torch.float32


# four parts, two parts, two parts of four waves (256 workgroups of 128 queries), one part; key counts at and around
# the 32-key chunk and fewer chunks than parts. fp32: four and two parts of one and two waves, one part
@pytest.mark.parametrize("B,H,n_q,n_kv,d,dtype", [
    (1, 1, 1, 1, 128, BF), (1, 2, 65, 33, 128, BF), (2, 3, 64, 97, 128, BF), (1, 4, 130, 128, 128, BF), (2, 16, 576, 161, 128, BF),
    (1, 16, 1025, 70, 128, BF), (2, 16, 1000, 200, 128, BF), (2, 16, 1030, 65, 128, BF), (1, 3, 70, 129, 64, BF),
    (2, 16, 1500, 63, 64, BF), (1, 32, 1024, 40, 64, BF), (1, 2, 40, 130, 64, F32), (1, 2, 40, 70, 64, F32), (2, 16, 300, 200, 64, F32),
    (2, 16, 700, 100, 64, F32), (1, 2, 40, 33, 128, F32), (2, 16, 300, 65, 128, F32), (2, 16, 576, 40, 128, F32), (1, 1, 3, 5, 128, F32),
    (2, 16, 1100, 129, 64, F32), (2, 16, 2100, 40, 128, F32)])
def test_dense_parts(B, H, n_q, n_kv, d, dtype):
    note(f"[key parts] dense {B}x{H} {n_q} against {n_kv}, d={d} {dtype}")
    q, k, v = cache(B, H, max(n_q, n_kv), d, n_q + n_kv, 3, dtype)
    q, k, v = q[:, :, :n_q], k[:, :, :n_kv], v[:, :, :n_kv]
    o = torch.empty(B, H, n_q, d, device="cuda", dtype=dtype)
    lse = torch.empty(B, H, n_q, device="cuda") if dtype == F32 else None
    sv.sparvar_dense_attn_fwd(q, k, v, o, lse, softmax_scale=scale_of(d))
    x = q.double() @ k.double().transpose(-1, -2).contiguous() * scale_of(d)
    check(o, torch.softmax(x, -1) @ v.double(), "dense")
    if lse is not None:
        assert (lse.double() - torch.logsumexp(x, -1)).abs().max() <= 1e-5


# 32x32 tokens in 8x8 tiles (16 per head): 256 tiles take four parts, 272 and 512 two, 528 one (d = 64: 768 two, 784
# one); 8x16 tiles have four waves; forced waves take one part, whose table is filled again for the long rows
@pytest.mark.parametrize("side,edge,heads,d,waves,dtype", [
    (32, 8, 16, 128, 0, BF), (32, 8, 17, 128, 0, BF), (32, 8, 32, 128, 0, BF), (32, 8, 33, 128, 0, BF), (32, 8, 48, 64, 0, BF),
    (32, 8, 49, 64, 0, BF), (30, 10, 3, 128, 0, BF), (30, 10, 30, 128, 0, BF), (30, 10, 5, 64, 0, BF), (31, 8, 5, 128, 0, BF),
    (64, 8, 2, 128, 2, BF), (64, 8, 2, 128, 0, BF), (50, 40, 1, 64, 0, F32), (31, 8, 2, 128, 0, F32), (30, 5, 1, 64, 0, F32)])
def test_sparse_parts(launch_option, side, edge, heads, d, waves, dtype):
    note(f"[key parts] sparse side {side} edge {edge} heads {heads} d={d} waves {waves}")
    launch_option("SPARSE_GROUP_WAVES", 0)
    if waves:
        launch_option("SPARSE_WAVES", waves)
    sides = [1, 2, 4, 8, 16, side] + ([side] * 3 if side == 64 else [])
    k_last = len(sides)
    g = sv.Geometry(sides, sides, edge, 2)
    info = [g.scale_info(l) for l in range(1, k_last + 1)]
    n, nb = info[-1]["n_tokens_le"], info[-1]["n_blocks_le"]
    tiles, nq, off = info[-1]["tiles_h"] * info[-1]["tiles_w"], info[-1]["n_tokens"], info[-1]["token_offset"]
    q, k, v = cache(1, heads, n, d, side * heads + d, 5, dtype)
    rng = np.random.default_rng(side + heads)
    keep = rng.random((heads * tiles, nb)) < rng.choice([0.0, 0.02, 0.3, 1.0], (heads * tiles, 1))
    keep[0], keep[1] = False, True
    rows, ptr = [], [0]
    for r in keep:
        ids = np.flatnonzero(r).tolist()
        rows += ids + [-1] * (len(rows) % 3)  # padding of any length
        ptr.append(len(rows))
    i32 = dict(dtype=torch.int32, device="cuda")
    o = torch.empty(1, heads, nq, d, device="cuda", dtype=dtype)
    lse = torch.empty(1, heads, nq, device="cuda")
    sv.sparvar_block_sparse_attn_fwd(g, k_last, q[:, :, off:], k, v, o, torch.tensor(ptr, **i32), torch.tensor(rows, **i32), lse=lse,
                                     softmax_scale=scale_of(d))
    blk, tile = [], None
    for i in info:
        x, y = np.divmod(np.arange(i["n_tokens"]), i["w"])
        tile = x // i["tile_h"] * i["tiles_w"] + y // i["tile_w"]
        blk.append(i["block_offset"] + tile)
    blk, tile = torch.from_numpy(np.concatenate(blk)).cuda(), torch.from_numpy(tile).cuda()
    keep = torch.from_numpy(keep).cuda().reshape(heads, tiles, nb)
    for h in range(heads):
        m = keep[h][tile][:, blk]
        x = (q[0, h, off:].double() @ k[0, h].double().T.contiguous() * scale_of(d)).masked_fill_(~m, -math.inf)
        some = m.any(1)
        ref = torch.softmax(x[some], -1) @ v[0, h].double()
        check(o[0, h][some], ref, f"head {h}")
        assert (lse[0, h][some].double() - torch.logsumexp(x[some], -1)).abs().max() <= (1e-5 if dtype == F32 else 2e-4)
        assert (o[0, h][~some] == 0).all() and torch.isneginf(lse[0, h][~some]).all()


# keys that score -inf (K of -inf where every query is 1) in runs of 64, the first of the row among them: whole chunks of
# them begin the row and parts of it, and weigh nothing. Rows of every key, so each path is dense attention.
@pytest.mark.parametrize("path,d,dtype", [("dense", 128, BF), ("dense", 64, BF), ("dense", 64, F32), ("dense", 128, F32), ("sparse", 128, BF),
                                          ("sparse", 64, BF), ("sparse", 128, F32), ("token", 128, BF), ("blocks", 128, BF), ("blocks", 64, BF)])
def test_parts_that_begin_with_minus_infinity(path, d, dtype):
    note(f"[key parts] {path} d={d} {dtype}, keys that score -inf")
    sides, H = [1, 2, 4, 8, 16, 32], 4
    g = sv.Geometry(sides, sides, 8, 2)
    i = g.scale_info(6)
    n, nq = i["n_tokens_le"], i["n_tokens"]
    q, k, v = cache(1, H, n, d, d, 3, dtype)
    q[..., 0] = 1
    k[:, :, torch.arange(n, device="cuda") // 64 % 2 == 0, 0] = -math.inf
    q, i32 = q[:, :, n - nq:], dict(dtype=torch.int32, device="cuda")
    o, lse = torch.empty(1, H, nq, d, device="cuda", dtype=dtype), torch.empty(1, H, nq, device="cuda")
    if path == "dense":
        sv.sparvar_dense_attn_fwd(q, k, v, o, lse if dtype == F32 else None, softmax_scale=scale_of(d))
    elif path == "sparse":
        rows, nb = H * i["tiles_h"] * i["tiles_w"], i["n_blocks_le"]
        sv.sparvar_block_sparse_attn_fwd(g, 6, q, k, v, o, torch.arange(0, rows * nb + 1, nb, **i32), torch.arange(nb, **i32).repeat(rows),
                                         lse=lse, softmax_scale=scale_of(d))
    elif path == "token":
        sv.sparvar_cs4a_attn_fwd(g, 6, 64, q, k, v, o, torch.arange(n, **i32).repeat(H * nq // 64), n, lse=lse, softmax_scale=scale_of(d))
    else:
        nkb = sv.sparvar_csla_row_stride(g, 6, 64)
        sv.sparvar_csla_attn_fwd(g, 6, 64, q, k, v, o, torch.arange(nkb, **i32).repeat(nq // 64, 1), lse=lse, softmax_scale=scale_of(d))
    x = q.double() @ k.double().transpose(-1, -2).contiguous() * scale_of(d)
    check(o, torch.softmax(x, -1) @ v.double(), path)
    if path != "dense" or dtype == F32:
        assert (lse.double() - torch.logsumexp(x, -1)).abs().max() <= (1e-5 if dtype == F32 else 2e-4)


# an option set to its default value is a shape asked for: one walk of that shape, not the choice made for the size of the
# launch. Another option of the same shape (pipeline depth, waves) gives the same sums, so the outputs are the same bits.
@pytest.mark.parametrize("path,d,heads,given,same", [
    ("blocks", 128, 2, dict(CSLA_CHUNK=32, CSLA_STAGES=2), dict(CSLA_CHUNK=32, CSLA_STAGES=3)),
    ("blocks", 128, 2, dict(CSLA_STAGES=2), dict(CSLA_CHUNK=32, CSLA_STAGES=3)),
    ("sparse", 128, 4, dict(SPARSE_CHUNK=32), dict(SPARSE_WAVES=2, SPARSE_CHUNK=32)),
    ("sparse", 64, 64, dict(SPARSE_CHUNK=32), dict(SPARSE_WAVES=2, SPARSE_CHUNK=32)),
    ("dense", 128, 4, dict(DENSE_CHUNK=64), dict(DENSE_WAVES=2, DENSE_CHUNK=32))])
def test_set_shapes_are_taken_as_given(launch_option, path, d, heads, given, same):
    note(f"[key parts] {path} d={d} {given}")
    sides = [1, 2, 4, 8, 16, 32]
    g = sv.Geometry(sides, sides, 8, 2)
    i = g.scale_info(6)
    n, nq, nb, tiles = i["n_tokens_le"], i["n_tokens"], i["n_blocks_le"], i["tiles_h"] * i["tiles_w"]
    q, k, v = cache(1, heads, n, d, heads + d, 3)
    q, i32 = q[:, :, n - nq:], dict(dtype=torch.int32, device="cuda")

    def run():
        o = torch.empty(1, heads, nq, d, device="cuda", dtype=BF)
        if path == "blocks":
            nkb = sv.sparvar_csla_row_stride(g, 6, 64)
            sv.sparvar_csla_attn_fwd(g, 6, 64, q, k, v, o, torch.arange(nkb, **i32).repeat(nq // 64, 1), softmax_scale=scale_of(d))
        elif path == "sparse":
            sv.sparvar_block_sparse_attn_fwd(g, 6, q, k, v, o, torch.arange(0, heads * tiles * nb + 1, nb, **i32),
                                             torch.arange(nb, **i32).repeat(heads * tiles), softmax_scale=scale_of(d))
        else:
            sv.sparvar_dense_attn_fwd(q, k, v, o, None, softmax_scale=scale_of(d))
        return o

    outs = []
    for opts in (given, same):
        for name, value in opts.items():
            launch_option(name, value)
        outs.append(run())
        for name in opts:
            launch_option(name, sv.OPT_DEFAULT)
    assert torch.equal(outs[0], outs[1])


# walks too short to be worth a split (4 chunks of dense keys or tokens; caches of 3 chunks for blocks and tiles) take the
# one-walk form, bit for bit
@pytest.mark.parametrize("path,d,one_walk", [
    ("dense", 128, dict(DENSE_WAVES=2, DENSE_CHUNK=32)), ("dense", 64, dict(DENSE_WAVES=2, DENSE_CHUNK=32)), ("token", 128, dict(CS4A_CHUNK=32)),
    ("blocks", 128, dict(CSLA_STAGES=3)), ("tiles", 128, dict(SPARSE_WAVES=2, SPARSE_CHUNK=32)),
    ("tiles", 64, dict(SPARSE_WAVES=2, SPARSE_CHUNK=64))])
def test_short_walks_are_not_split(launch_option, path, d, one_walk):
    note(f"[key parts] short walks, {path} d={d}")
    sides, heads, i32 = [1, 2, 4, 8], 3, dict(dtype=torch.int32, device="cuda")
    g = sv.Geometry(sides, sides, 8, 2)
    n, nb = 128 if path in ("dense", "token") else 85, g.scale_info(4)["n_blocks_le"]
    q, k, v = cache(1, heads, n, d, d, 3)
    q = q[:, :, n - 64:]

    def run():
        o = torch.empty(1, heads, 64, d, device="cuda", dtype=BF)
        if path == "dense":
            sv.sparvar_dense_attn_fwd(q, k, v, o, None, softmax_scale=scale_of(d))
        elif path == "token":
            wide = sv.Geometry([1, 2, 4, 8], [1, 2, 10, 8], 8, 2)  # 109 keys; 128 token slots
            rows = torch.cat([torch.arange(109, **i32), torch.full((19,), -1, **i32)]).repeat(heads)
            sv.sparvar_cs4a_attn_fwd(wide, 4, 64, q, k, v, o, rows, 128, softmax_scale=scale_of(d))
        elif path == "blocks":
            sv.sparvar_csla_attn_fwd(g, 4, 64, q, k, v, o, torch.tensor([[0, 1]], **i32), softmax_scale=scale_of(d))
        else:
            sv.sparvar_block_sparse_attn_fwd(g, 4, q, k, v, o, torch.arange(0, heads * nb + 1, nb, **i32), torch.arange(nb, **i32).repeat(heads),
                                             softmax_scale=scale_of(d))
        return o

    default = run()
    for name, value in one_walk.items():
        launch_option(name, value)
    assert torch.equal(default, run())
