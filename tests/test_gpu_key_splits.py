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


def one_d(heads, d, seed, sides=(2, 16, 20, 16)):
    """Schedule, queries of its last scale and cache for 1-D query blocks; the default is 256 queries, 916 keys."""
    g = sv.Geometry(list(sides), list(sides), 8, 1)
    i = g.scale_info(len(sides))
    q, k, v = cache(1, heads, i["n_tokens_le"], d, seed, 5)
    return g, len(sides), q[:, :, i["token_offset"]:], k, v


def check_rows_of_keys(o, lse, q, k, v, keep, what):
    """o and lse of queries [heads, n] against 64 bits; keep [heads or 1, n, keys]."""
    for h in range(q.shape[1]):
        m = keep[h % keep.shape[0]]
        x = (q[0, h].double() @ k[0, h].double().T.contiguous() * scale_of(q.shape[-1])).masked_fill_(~m, -math.inf)
        some = m.any(1)
        assert (o[0, h][~some] == 0).all() and torch.isneginf(lse[0, h][~some]).all()
        if some.any():
            check(o[0, h][some], torch.softmax(x[some], -1) @ v[0, h].double(), f"{what} head {h}")
            assert (lse[0, h][some].double() - torch.logsumexp(x[some], -1)).abs().max() <= 2e-4


# rows of 1-D blocks: every block, none, one to three (fewer than the parts), a run that crosses parts, an id out of range
# before others; the cache's last block is partial. 256 queries a head: with blocks of 64, up to 256 workgroups take four
# parts, up to 512 (d = 64: 768) two, more one; with blocks of 128, up to 256 two, more one
@pytest.mark.parametrize("d,block,heads", [(128, 64, 3), (128, 64, 64), (128, 64, 65), (128, 64, 128), (128, 64, 129), (64, 64, 5),
                                           (64, 64, 66), (64, 64, 192), (64, 64, 193), (128, 128, 2), (128, 128, 129), (64, 128, 3),
                                           (64, 128, 129), (128, 32, 3), (64, 256, 2)])
def test_block_row_parts(d, block, heads):
    note(f"[key parts] 1-D blocks of {block}, d={d}, {heads} heads")
    g, s, q, k, v = one_d(heads, d, block + heads + d)
    n, G, M = k.shape[2], q.shape[2] // block, sv.sparvar_csla_row_stride(g, s, block)
    every = list(range(M))
    patterns = [every, [M - 1], every[1:3] + [M - 1], every[2:-1], [], [0, M - 1], [0, 2, M + 5] + every[3:], every[::2]]
    for shift in range(0, len(patterns), G):
        rows = np.full((G, M), -1, np.int32)
        keep = np.zeros((G, n), bool)
        for u in range(G):
            ids = patterns[(shift + u) % len(patterns)][:M]
            rows[u, :len(ids)] = ids
            for b in ids[:next((j for j, x in enumerate(ids) if x >= M), len(ids))]:
                keep[u, b * block:(b + 1) * block] = True
        o, lse = torch.empty_like(q, memory_format=torch.contiguous_format), torch.empty(q.shape[:3], device="cuda")
        sv.sparvar_csla_attn_fwd(g, s, block, q, k, v, o, torch.from_numpy(rows).cuda(), lse=lse, softmax_scale=scale_of(d))
        check_rows_of_keys(o, lse, q, k, v, torch.from_numpy(keep).cuda().repeat_interleave(block, 0)[None], f"rows from {shift}")
        if heads > 8:
            break


# rows past the 512 ids that are staged in LDS, cut into parts: 529 key blocks of 64, and the second half of them
@pytest.mark.parametrize("d,block", [(64, 64), (128, 64), (128, 128)])
def test_block_row_parts_past_the_staged_ids(d, block):
    side = 183 if block == 64 else 259
    g, s, q, k, v = one_d(1, d, block + d, (2, side, 16))
    n, G, M = k.shape[2], 256 // block, sv.sparvar_csla_row_stride(g, s, block)
    note(f"[key parts] {M} ids of {block} keys, d={d}")
    assert M > 520
    rows, keep = np.full((G, M), -1, np.int32), np.zeros((G, n), bool)
    for u in range(G):
        ids = np.arange(M) if u % 2 == 0 else np.arange(300, M, 2 if u == 3 else 1)
        rows[u, :len(ids)] = ids
        for b in ids:
            keep[u, b * block:(b + 1) * block] = True
    o, lse = torch.empty_like(q, memory_format=torch.contiguous_format), torch.empty(q.shape[:3], device="cuda")
    sv.sparvar_csla_attn_fwd(g, s, block, q, k, v, o, torch.from_numpy(rows).cuda(), lse=lse, softmax_scale=scale_of(d))
    check_rows_of_keys(o, lse, q, k, v, torch.from_numpy(keep).cuda().repeat_interleave(block, 0)[None], "long rows")


# token rows of no token, one, around a chunk, around a part and all of them, in rows of M slots: from 160 slots on two
# parts, from 384 four (256 workgroups of 64 queries; past those two, past 512 one, d = 64: 768); 128 queries take two from
# 1024 slots on (d = 64: 512). Mode 2 adds the base's row of the same place
@pytest.mark.parametrize("d,C,heads,M,mode", [(128, 64, 3, 200, 0), (128, 64, 3, 400, 2), (128, 64, 64, 900, 0), (128, 64, 65, 900, 0),
                                              (128, 64, 128, 170, 2), (128, 64, 129, 400, 0), (64, 64, 4, 130, 0), (64, 64, 4, 500, 2),
                                              (64, 64, 192, 300, 0), (64, 64, 193, 300, 0), (128, 128, 3, 1100, 0), (128, 128, 129, 1100, 2),
                                              (64, 128, 3, 600, 0), (128, 32, 3, 300, 0)])
def test_token_row_parts(d, C, heads, M, mode):
    note(f"[key parts] token rows of {M}, blocks of {C}, d={d}, {heads} heads, mode {mode}")
    g, s, q, k, v = one_d(heads, d, M + heads)
    n, G = k.shape[2], q.shape[2] // C
    most = min(M, n)
    rng = np.random.default_rng(M + heads)
    lens = rng.choice([0, 1, 31, 32, 33, most // 4, most // 2 + 1, most - 1, most], heads * G)
    lens[:2] = 0, most
    rows, keep = np.full((heads * G, M), -1, np.int32), np.zeros((heads * G, n), bool)
    for r, c in enumerate(lens):
        rows[r, :c] = np.sort(rng.choice(n, c, replace=False))
        keep[r, rows[r, :c]] = True
    o, lse = torch.empty_like(q, memory_format=torch.contiguous_format), torch.empty(q.shape[:3], device="cuda")
    base = torch.randn(q.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(M)).bfloat16() if mode else None
    sv.sparvar_cs4a_attn_fwd(g, s, C, q, k, v, o, torch.from_numpy(rows).cuda(), M, lse=lse, mode=mode, base=base, base_scale=s,
                             softmax_scale=scale_of(d))
    keep = torch.from_numpy(keep).cuda().reshape(heads, G, n).repeat_interleave(C, 1)
    if mode:  # the sum's rounding (half an ulp below 8: 1.6e-2) and that of the output without a base
        plain = torch.empty_like(o)
        sv.sparvar_cs4a_attn_fwd(g, s, C, q, k, v, plain, torch.from_numpy(rows).cuda(), M, lse=lse, softmax_scale=scale_of(d))
        assert (o.double() - base.double() - plain.double()).abs().max() <= 2e-2
        o = plain
    check_rows_of_keys(o, lse, q, k, v, keep, "tokens")


# a call that asks for the LSE walks its keys in one order (its output feeds a difference whose rounding cancels): the bits
# of the one-walk form; the same call without it may split them, with no larger error
@pytest.mark.parametrize("d,n_kv", [(128, 300), (128, 1300), (64, 900)])
def test_dense_with_lse_walks_once(launch_option, d, n_kv):
    note(f"[key parts] dense with and without LSE, {n_kv} keys, d={d}")
    q, k, v = cache(1, 4, n_kv, d, n_kv, 3)
    q = q[:, :, :256]
    outs = [torch.empty(1, 4, 256, d, device="cuda", dtype=BF) for _ in range(3)]
    lse = torch.empty(1, 4, 256, device="cuda")
    sv.sparvar_dense_attn_fwd(q, k, v, outs[0], lse, softmax_scale=scale_of(d))
    sv.sparvar_dense_attn_fwd(q, k, v, outs[1], None, softmax_scale=scale_of(d))
    launch_option("DENSE_WAVES", 2)
    launch_option("DENSE_CHUNK", 32)
    sv.sparvar_dense_attn_fwd(q, k, v, outs[2], None, softmax_scale=scale_of(d))
    assert torch.equal(outs[0], outs[2])
    ref = torch.softmax(q.double() @ k.double().transpose(-1, -2).contiguous() * scale_of(d), -1) @ v.double()
    err = [((o.double() - ref).norm() / ref.norm()).item() for o in outs]
    # both round probabilities and outputs to 8 bits, independently: about 2e-3, a sample of 4 x 256 rows within a few percent
    assert err[1] <= 1.05 * err[0], err


def test_launch_options_leave_defaults_unset():
    note("[key parts] launch_options() around a default")
    q, k, v = cache(1, 4, 1000, 128, 5, 3)
    outs = []

    def run():
        outs.append(torch.empty(1, 4, 256, 128, device="cuda", dtype=BF))
        sv.sparvar_dense_attn_fwd(q[:, :, :256], k, v, outs[-1], None, softmax_scale=scale_of(128))

    run()
    with sv.launch_options(DENSE_CHUNK=64):  # the default value, set: one walk
        run()
    run()
    assert torch.equal(outs[0], outs[2]) and not torch.equal(outs[0], outs[1])
