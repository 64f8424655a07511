"""The two-pass selections against the one-pass scores of the same summaries, selected by the oracle:
dense queries and bf16 copies that differ from the fp32 Mean, at the request bounds and channel counts
between which the selection changes its workgroup shape, and on summaries for which the bounds of the
first pass say little or nothing."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2606_06453_amd import vx

pytestmark = pytest.mark.gpu

PS = 16


class Problem:
    """Random summaries of B requests of up to P blocks: mean [B * P][H][D] fp32, envelope around it."""

    def __init__(self, D, P, B, H, g, seed, spread=0.5):
        self.D, self.P, self.B, self.H, self.g = D, P, B, H, g
        rng = np.random.default_rng(seed)
        self.pages = rng.integers(P // 2, P + 1, B).astype(np.int32)
        self.pages[0] = P
        if B > 1:
            self.pages[-1] = P // 3
        k = torch.zeros((B * P, H, PS, D), dtype=torch.float8_e4m3fn, device="cuda")
        self.kv = vx.PagedKV(k, None if D == 576 else k, 512 if D == 576 else D)
        lens = (self.pages * PS - rng.integers(0, PS, B)).astype(np.int32)
        self.perm = torch.from_numpy(rng.permutation(B * P).astype(np.int32)).cuda()
        self.batch = vx.BatchSpec((torch.arange(B + 1, dtype=torch.int32) * P).cuda(), self.perm,
                                  torch.from_numpy(lens).cuda(), P)
        gen = torch.Generator(device="cuda").manual_seed(seed)
        self.mean = torch.randn((B * P, H, D), generator=gen, device="cuda") * 0.25
        self.max = (self.mean + spread * torch.rand(self.mean.shape, generator=gen, device="cuda")).to(torch.bfloat16)
        self.min = (self.mean - spread * torch.rand(self.mean.shape, generator=gen, device="cuda")).to(torch.bfloat16)
        self.q = torch.randn((B, H * g, D), generator=gen, device="cuda").to(torch.bfloat16)
        self.budget = rng.integers(2, max(3, P // 4), B).astype(np.int32)

    def rows(self, i, blocks):
        """Physical rows of request i's blocks."""
        return self.perm[i * self.P + torch.as_tensor(blocks, device="cuda")].long()

    def check(self, kind, n_sink=1, n_local=2):
        args = dict(mean=self.mean if kind in vx.NEEDS_MEAN else None, max=self.max if kind in vx.NEEDS_MAX else None,
                    min=self.min if kind in vx.NEEDS_MIN else None)
        max_sel = max(n_sink + n_local, int(self.budget.max()))
        sel = torch.full((self.B, self.H, max_sel), -7, dtype=torch.int32, device="cuda")
        cnt = torch.full((self.B,), -7, dtype=torch.int32, device="cuda")
        ws = torch.empty(vx.workspace_size(vx.STAGE_SCORE_TOPK, self.kv, self.batch, self.H * self.g, max_sel),
                         dtype=torch.uint8, device="cuda")
        vx.page_score_topk(self.q, self.kv, self.batch, kind, args["mean"], args["max"], args["min"],
                           torch.from_numpy(self.budget).cuda(), n_sink, n_local, max_sel, sel, cnt, ws,
                           mean_bf16=self.mean.to(torch.bfloat16) if kind in vx.TWO_PASS_KINDS else None)
        scores = torch.zeros((self.H, self.B, self.P), device="cuda")
        vx.page_score(self.q, self.kv, self.batch, kind, args["mean"], args["max"], args["min"], scores)
        torch.cuda.synchronize()
        o_sel, o_cnt = O.topk_select(scores.cpu().numpy(), self.pages, self.budget, n_sink, n_local, max_sel)
        assert (cnt.cpu().numpy() == o_cnt).all()
        assert (sel.cpu().numpy() == o_sel).all()
        return scores


@pytest.mark.parametrize("P", [700, 4096, 4097, 9000])
@pytest.mark.parametrize("kind,D", [(vx.MEAN_DOT, 64), (vx.MEAN_DOT, 128), (vx.MEAN_DOT, 576), (vx.QUEST, 64),
                                    (vx.QUEST, 128), (vx.QUEST_CONSENSUS, 128), (vx.ENVELOPE_LOWER, 128)])
def test_first_pass_out_of_range(kind, D, P):
    """Sums of the first pass that leave the fp32 range and cancel: its bounds are NaN, the fp64 score an
    ordinary number, here the highest of its request.  Every product is about 2^127 (2^126 at 576
    channels), of one sign in the channels of a lane (four or eight adjacent ones), so a lane's sum
    overflows whatever its order."""
    pb = Problem(D, P, 2, 1 if D == 576 else 2, 16 if D == 576 else 4, D + P)
    mag = 64.0 if D == 576 else 128.0
    lane = torch.arange(D, device="cuda") // (8 if D % 128 == 0 else 4) % 16
    sign = torch.where(lane < 8, 1.0, -1.0)
    pb.q[:] = (mag * sign).to(torch.bfloat16)
    row = torch.where(lane < 8, 2.0 ** 120, 2.0 ** 120 * (1 - 2.0 ** -7))
    top = [5, P // 6, P // 3 - 3]
    for i in range(2):
        for s in (pb.mean, pb.max, pb.min):
            s[pb.rows(i, top)] = row.to(s.dtype)
    scores = pb.check(kind)
    assert torch.isfinite(scores).all()
    assert (scores[:, :, top] == D / 2 * mag * 2.0 ** 113).all()


SHAPES = [(vx.MEAN_DOT, 128, 4097, 2, 2), (vx.MEAN_DOT, 128, 8193, 1, 2), (vx.MEAN_DOT, 128, 16384, 1, 1),
          (vx.QUEST, 128, 4097, 2, 2), (vx.QUEST, 128, 8193, 1, 2), (vx.QUEST, 64, 16384, 1, 1),
          (vx.QUEST_RECTIFIED, 128, 8192, 1, 2), (vx.QUEST_CONSENSUS, 128, 16384, 1, 1),
          (vx.ENVELOPE_LOWER, 128, 4100, 2, 1), (vx.MEAN_DOT, 64, 1500, 40, 16), (vx.QUEST, 64, 2500, 40, 16),
          (vx.QUEST, 128, 600, 3, 2), (vx.MEAN_DOT, 576, 1025, 2, 1), (vx.MEAN_DOT, 576, 2049, 2, 1),
          (vx.MEAN_DOT, 576, 4097, 2, 1), (vx.MEAN_DOT, 576, 8193, 1, 1), (vx.MEAN_DOT, 576, 16384, 1, 1),
          (vx.MEAN_DOT, 576, 2100, 520, 1)]


@pytest.mark.parametrize("rows", ["spread", "far", "farther", "near", "equal", "infinite"])
@pytest.mark.parametrize("kind,D,P,B,H", SHAPES)
def test_two_pass_shapes(kind, D, P, B, H, rows):
    """Ordinary rows; one block scaled by 300; one by 1e6 and one by 1e3, of both signs, so that the bins
    are refined more than once; blocks that differ by a hundredth (most are undecided by the block mean's
    bounds) or not at all; an infinite channel, whose score is infinite or NaN."""
    pb = Problem(D, P, B, H, 16 if D == 576 else 4, 3 * D + P + B)
    if rows in ("far", "farther"):
        for i in range(B):
            for block, f in [(7, 300.0)] if rows == "far" else [(7, 1e6), (P // 3 - 4, -1e3)]:
                r = pb.rows(i, [block])
                pb.mean[r] *= f
                a, b = pb.max[r] * f, pb.min[r] * f
                pb.max[r], pb.min[r] = torch.maximum(a, b), torch.minimum(a, b)
    elif rows in ("near", "equal"):
        for s in (pb.mean, pb.max, pb.min):
            s.mul_(0.01 if rows == "near" else 0.0).add_(s[:1] * 100 if rows == "near" else 0.375)
    elif rows == "infinite":
        for i in range(B):
            for block, x in [(7, float("inf")), (9, float("-inf")), (P // 3 - 4, float("inf"))]:
                for s in (pb.mean, pb.max, pb.min):
                    s[pb.rows(i, [block]), :, 3] = x
    pb.check(kind)
