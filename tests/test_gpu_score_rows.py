"""Pooled block scores over blocks whose key counts leave partial chunks, and top-k rows around a workgroup's 256 candidates."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import note, scale_of
from paper_2602_04361_amd import sparvar as sv

pytestmark = pytest.mark.gpu


# tiles of 1, 2, 4 and 8 waves; blocks of 1 to 900 keys: under 32, between 32 and 64, and the remainder of several chunks
@pytest.mark.parametrize("sides,b,d", [([1, 2, 3, 5, 7], 5, 128), ([1, 4, 13, 21], 8, 64), ([2, 6, 9, 30], 8, 128),
                                       ([1, 9, 20], 11, 128), ([3, 31, 33], 16, 64), ([1, 30, 14], 30, 128)])
def test_pooled_scores_of_partial_chunks(sides, b, d):
    note(f"[score rows] sides {sides} b={b} d={d}")
    S, B, H = len(sides), 2, 3
    g = sv.Geometry(sides, sides, b, 1)
    info = [g.scale_info(l) for l in range(1, S + 1)]
    n, nb, nq, off = (info[-1][x] for x in ("n_tokens_le", "n_blocks_le", "n_tokens", "token_offset"))
    tiles = info[-1]["tiles_h"] * info[-1]["tiles_w"]
    blk = []
    for i in info:
        x, y = np.divmod(np.arange(i["n_tokens"]), i["w"])
        tile = x // i["tile_h"] * i["tiles_w"] + y // i["tile_w"]
        blk.append(i["block_offset"] + tile)
    blk, tile = torch.from_numpy(np.concatenate(blk)).cuda(), torch.from_numpy(tile).cuda()
    gen = torch.Generator("cuda").manual_seed(n + d)
    q, k = (torch.randn(B, H, n, d, device="cuda", generator=gen).bfloat16() for _ in range(2))
    x = q[:, :, off:].double() @ k.double().transpose(-1, -2).contiguous() * scale_of(d)
    lse = torch.logsumexp(x, -1).float().contiguous()
    scores = torch.full((B, H, tiles, nb), -1.0, device="cuda")
    idx = torch.empty(B, H, tiles, 3, device="cuda", dtype=torch.int32)
    sv.sparvar_select_blocks(g, S, q[:, :, off:], k, lse, 3, idx, scores_out=scores, softmax_scale=scale_of(d))
    per_key = torch.zeros(B, H, tiles, n, device="cuda", dtype=torch.float64).index_add_(2, tile, torch.softmax(x, -1))
    ref = torch.zeros(B, H, tiles, nb, device="cuda", dtype=torch.float64).index_add_(3, blk, per_key)
    # each probability carries the rounding of its exponent (at most 32 in magnitude, 24 bits: 4e-6 relative)
    # and of the LSE it is taken against (the same); masses are their sums
    assert ((scores.double() - ref).abs() <= 2e-5 * ref + 1e-9).all()
    got, sc = idx.cpu().numpy().reshape(-1, 3), scores.cpu().numpy().reshape(-1, nb)
    assert all(r.tolist() == O.topk_blocks(s, 3) for r, s in zip(got, sc))


# 256 candidates fill one pass of a workgroup; rows of one pass, of a remainder of 1 to 3 past a multiple of 4, of several;
# 64, 128 and 192 candidates are the lines between workgroups of one to four waves
@pytest.mark.parametrize("h,w", [(1, 1), (1, 3), (7, 9), (8, 8), (5, 13), (1, 127), (8, 16), (3, 43), (12, 16), (1, 193), (5, 50), (15, 17), (16, 16), (1, 257), (23, 25), (30, 35)])
def test_top_rows_past_one_pass(h, w):
    g = sv.Geometry([h], [w], 1, 1)
    nb = h * w
    rng = np.random.default_rng(nb)
    for topk in sorted({1, 7, min(nb, 300), min(nb + 3, 1000)}):
        note(f"[score rows] {nb} candidates, topk {topk}")
        sc = rng.integers(0, 9, (1, 2, nb, nb)).astype(np.float32)
        sc[0, 0, ::3][rng.random(sc[0, 0, ::3].shape) < 0.7] = -np.inf
        sc[0, 1, ::2] *= np.finfo(np.float32).min / 8
        sc[0, 1, 0] = -np.inf
        idx = torch.full((1, 2, nb, topk), 9, dtype=torch.int32, device="cuda")
        sv.sparvar_select_blocks(g, 1, None, None, None, topk, idx, scores_in=torch.from_numpy(sc).cuda())
        got = idx.cpu().numpy().reshape(-1, topk)
        rows = sorted({0, 3 % nb, nb - 1, nb, 2 * nb - 1, *rng.integers(0, 2 * nb, 60).tolist()})
        for r in rows:
            assert got[r].tolist() == O.topk_blocks(sc.reshape(-1, nb)[r], topk)


# infinities the caller may hand in: an LSE of -inf (exp(s + inf) = inf for every key of the tile), of +inf (0), and keys
# that score -inf (0); 5x5 blocks leave partial chunks, 8x8 ones whole chunks
@pytest.mark.parametrize("b,d", [(5, 128), (8, 128), (8, 64), (11, 64)])
def test_pooled_scores_of_infinities(b, d):
    note(f"[score rows] infinities b={b} d={d}")
    g = sv.Geometry([2, 9, 22], [2, 9, 22], b, 1)
    i = g.scale_info(3)
    n, nb, nq, tiles = i["n_tokens_le"], i["n_blocks_le"], i["n_tokens"], i["tiles_h"] * i["tiles_w"]
    gen = torch.Generator("cuda").manual_seed(b)
    q, k = (torch.randn(1, 2, n, d, device="cuda", generator=gen).bfloat16() for _ in range(2))
    q[..., 0] = 1
    k[:, 1, :4 + 81, 0] = -float("inf")  # head 1: no weight on the first two scales
    x = q[:, :, n - nq:].double() @ k.double().transpose(-1, -2).contiguous() * scale_of(d)
    lse = torch.logsumexp(x, -1).float().contiguous()
    t = np.arange(nq) // 22 // i["tile_h"] * i["tiles_w"] + np.arange(nq) % 22 // i["tile_w"]
    low, high = torch.from_numpy(t == tiles - 1).cuda(), torch.from_numpy(t == 0).cuda()
    lse[0, 0, low], lse[0, :, high] = -float("inf"), float("inf")
    scores, idx = torch.full((1, 2, tiles, nb), -1.0, device="cuda"), torch.empty(1, 2, tiles, 3, device="cuda", dtype=torch.int32)
    sv.sparvar_select_blocks(g, 3, q[:, :, n - nq:], k, lse, 3, idx, scores_out=scores, softmax_scale=scale_of(d))
    assert torch.isposinf(scores[0, 0, -1]).all() and idx[0, 0, -1].tolist() == [0, 1, 2]
    assert (scores[0, :, 0] == 0).all()
    gone = g.scale_info(2)["n_blocks_le"]
    assert (scores[0, 1, :, :gone] == 0).all()
    rest = scores[0, :, 1:tiles - 1]
    assert torch.isfinite(rest).all()
    # a tile's scores sum to its queries (probabilities of rows of at most 569 keys, a few ulp each)
    sizes = torch.from_numpy(np.bincount(t)[1:tiles - 1]).cuda()
    assert ((rest.double().sum(-1) - sizes).abs() <= 1e-4 * sizes).all()
