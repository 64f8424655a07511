"""The bucketed selection at the edges of its workgroup shapes (pages per request around a power of
two, up to its last and the first past it, few and many (request, KV head) pairs) on scores where its rules matter: exact ties, skewed
scores, infinities.  The scores are planted: the query reads channel 0 alone, so a block's score is
its summary's channel 0, exactly, and the oracle selects from the same numbers."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2606_06453_amd import vx

pytestmark = pytest.mark.gpu

D, PS = 64, 16


def _scores(shape, kind, rng):
    if kind == "normal":
        x = rng.standard_normal(shape)
    elif kind == "equal":
        x = np.full(shape, -0.5)
    elif kind == "skewed":                       # most scores in the lowest bin of a linear scale
        x = np.exp(-25.0 * rng.random(shape))
    else:                                        # few distinct values, with infinities among them
        x = rng.integers(-3, 4, shape).astype(np.float64)
        x[x == 3] = np.inf
        x[x == -3] = -np.inf
    return torch.from_numpy(x).to(torch.bfloat16)


def _select(scores, lens, budget, kind, two_pass, n_sink, n_local, max_sel):
    """vx_page_score_topk over summaries whose channel 0 holds scores [H][B][P]."""
    H, B, P = scores.shape
    k = torch.zeros((B * P, H, PS, D), dtype=torch.float8_e4m3fn, device="cuda")
    kv = vx.PagedKV(k, k, D)
    batch = vx.BatchSpec((torch.arange(B + 1, dtype=torch.int32) * P).cuda(),
                         torch.arange(B * P, dtype=torch.int32).cuda(), torch.from_numpy(lens).cuda(), P)
    summ = torch.zeros((B, P, H, D), dtype=torch.bfloat16)
    summ[..., 0] = scores.permute(1, 2, 0)
    bf = summ.view(B * P, H, D).cuda()
    q = torch.zeros((B, 2 * H, D), dtype=torch.bfloat16, device="cuda")
    q[..., 0] = 1.0
    sel = torch.full((B, H, max_sel), -7, dtype=torch.int32, device="cuda")
    cnt = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    ws = torch.empty(vx.workspace_size(vx.STAGE_SCORE_TOPK, kv, batch, 2 * H, max_sel), dtype=torch.uint8, device="cuda")
    mean = bf.float() if kind == vx.MEAN_DOT else None
    vx.page_score_topk(q, kv, batch, kind, mean, bf if kind != vx.MEAN_DOT else None, bf if kind == vx.QUEST else None,
                       torch.from_numpy(budget).cuda(), n_sink, n_local, max_sel, sel, cnt, ws,
                       mean_bf16=bf if two_pass else None)
    torch.cuda.synchronize()
    return sel.cpu().numpy(), cnt.cpu().numpy()


@pytest.mark.parametrize("dist", ["normal", "equal", "skewed", "coarse"])
@pytest.mark.parametrize("P,B,H", [(513, 3, 2), (1024, 3, 2), (1025, 3, 2), (2048, 2, 4), (2049, 2, 2), (4096, 2, 1),
                                   (1030, 40, 16), (1500, 33, 16), (2500, 33, 16), (4097, 2, 2), (8192, 2, 1),
                                   (8193, 2, 1), (16384, 2, 1), (16385, 2, 1)])
@pytest.mark.parametrize("kind,two_pass", [(vx.MAX_DOT, False), (vx.MEAN_DOT, True), (vx.QUEST, True)])
def test_selection_shapes(kind, two_pass, P, B, H, dist):
    rng = np.random.default_rng(P + B)
    scores = _scores((H, B, P), dist, rng)
    pages = rng.integers(P // 2, P + 1, B).astype(np.int32)
    pages[0], pages[-1] = P, min(P, 2 + P // 3)
    lens = (pages * PS - rng.integers(0, PS, B)).astype(np.int32)
    budget = rng.integers(1, P // 2, B).astype(np.int32)
    budget[-1] = pages[-1] - 1                                   # all but one page
    max_sel = int(budget.max())
    sel, cnt = _select(scores, lens, budget, kind, two_pass, 1, 3 if max_sel > 4 else 0, max_sel)
    o_sel, o_cnt = O.topk_select(scores.float().numpy(), pages, budget, 1, 3 if max_sel > 4 else 0, max_sel)
    assert (cnt == o_cnt).all()
    assert (sel == o_sel).all()


@pytest.mark.parametrize("dist", ["normal", "equal", "skewed", "coarse"])
@pytest.mark.parametrize("tau,remap", [(0.0, 0), (0.0, 1), (0.2, 0), (0.2, 1)])
@pytest.mark.parametrize("P,B,H", [(1, 2, 1), (500, 3, 2), (1025, 3, 2), (2048, 40, 16), (2049, 2, 2), (4096, 5, 4),
                                   (4096, 33, 16), (4097, 3, 2), (8193, 2, 1), (16384, 2, 1), (16385, 2, 1),
                                   (5000, 33, 8), (9000, 33, 8)])
def test_radix_selection_shapes(P, B, H, tau, remap, dist):
    """vx_topk_select at the same edges, its options included, over rows of any alignment."""
    rng = np.random.default_rng(P + B)
    x = _scores((H, B, P), dist, rng).float()
    if P > 1 and dist == "normal":
        x[:, 0, P // 3] = float("nan")
    items = rng.integers(P // 2, P + 1, B).astype(np.int32)
    items[0] = P
    budget = rng.integers(1, max(2, P // 2), B).astype(np.int32)
    max_sel = int(budget.max()) + 4
    sel = torch.full((B, H, max_sel), -7, dtype=torch.int32, device="cuda")
    cnt = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    vx.topk_select(x.cuda().contiguous(), torch.from_numpy(items).cuda(), torch.from_numpy(budget).cuda(), 1, 2, max_sel,
                   sel, cnt, tolerate_ratio=tau, seed=5, remap=remap)
    torch.cuda.synchronize()
    o_sel, o_cnt = O.topk_select(x.numpy(), items, budget, 1, 2, max_sel, tau=tau, seed=5, remap=remap)
    assert (cnt.cpu().numpy() == o_cnt).all()
    assert (sel.cpu().numpy() == o_sel).all()
