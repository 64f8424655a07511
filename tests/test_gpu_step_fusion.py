"""vx_append_score_topk (the decode step's append inside the top-K launch) against the two calls
it stands for, vx_kv_append_summarize then vx_page_score_topk, on the GPU: the caches, every
summary buffer and the selection must come out bit for bit the same.  Covered: the selections
whose launch carries the append in workgroups of its own (two-pass block mean, one-pass block mean
and Max, two-pass Quest; the MLA latent's 64 x 576 and 32 x 576 blocks, also with an fp8 latent), at
every workgroup size of the selection, an fp8 cache, blocks below the page size, and the cases that
append first instead (n_local = 0, NSA, an approximate selection, more than 16384 blocks)."""
import pytest
import torch

from oracle import oracle as O
from paper_2606_06453_amd import vx
from tests._problems import fp8_problem, random_problem, strip_last_token

pytestmark = pytest.mark.gpu

CASES = [
    # name, ps, bs, D, Hq, H, kind, two_pass, fp8, n_local, tau
    ("mean_two_pass", 16, 0, 128, 8, 2, O.MEAN_DOT, True, None, 2, 0.0),
    ("mean_one_pass", 16, 0, 64, 4, 1, O.MEAN_DOT, False, None, 3, 0.0),
    ("max_one_pass", 32, 0, 128, 8, 2, O.MAX_DOT, False, None, 1, 0.0),
    ("quest_two_pass", 16, 0, 128, 8, 2, O.QUEST, False, None, 2, 0.0),
    ("rectified", 32, 0, 64, 8, 2, O.QUEST_RECTIFIED, False, None, 2, 0.0),
    ("mla_latent", 64, 0, 576, 16, 1, O.MEAN_DOT, True, None, 2, 0.0),
    ("mla_latent_one_pass", 64, 0, 576, 16, 1, O.MEAN_DOT, False, None, 2, 0.0),
    ("mla_latent_fp8", 64, 0, 576, 16, 1, O.MEAN_DOT, False, torch.float8_e5m2, 1, 0.0),
    ("mla_latent_pages_of_32", 32, 0, 576, 16, 1, O.MEAN_DOT, False, None, 2, 0.0),
    ("pages_of_64", 64, 0, 128, 8, 2, O.MEAN_DOT, True, None, 2, 0.0),
    ("fp8_e4m3", 16, 0, 128, 8, 2, O.MEAN_DOT, True, torch.float8_e4m3fn, 2, 0.0),
    ("blocks_of_16", 32, 16, 128, 8, 2, O.QUEST, False, None, 2, 0.0),
    ("no_local_window", 16, 0, 128, 8, 2, O.MEAN_DOT, True, None, 0, 0.0),
    ("nsa_flow", 16, 0, 64, 8, 2, O.NSA, False, None, 2, 0.0),
    ("approximate", 16, 0, 128, 8, 2, O.MEAN_DOT, False, None, 2, 0.25),
]


def _state(pb, k, v, ks, vs, bs, H, D):
    """A cache (copies of k, v) and its summary buffers, summarised over the stripped cache."""
    kv = vx.PagedKV(k.clone().cuda(), None if v is None else v.clone().cuda(), pb.head_dim_v, k_scale=ks,
                    v_scale=vs, block_size=bs)
    r = pb.page_size // bs if bs else 1
    P = (pb.seq_lens + pb.page_size - 1) // pb.page_size
    batch = vx.BatchSpec(torch.from_numpy(pb.page_indptr).cuda(), torch.from_numpy(pb.page_indices).cuda(),
                         torch.from_numpy(pb.seq_lens).cuda(), int(P.max()))
    rows = k.shape[0] * r
    mean = torch.zeros((rows, H, D), device="cuda")
    mbf = torch.zeros((rows, H, D), dtype=torch.bfloat16, device="cuda")
    mx = torch.zeros((rows, H, D), dtype=torch.bfloat16, device="cuda")
    mn = torch.zeros((rows, H, D), dtype=torch.bfloat16, device="cuda")
    vx.page_summarize(kv, batch, None, mean, mx, mn, mean_bf16=mbf)
    return kv, batch, [mean, mbf, mx, mn]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_append_inside_selection_equals_separate_calls(case):
    ps, r = case[1], case[1] // case[2] if case[2] else 1
    lens = [ps * 40 + 3, ps * 9 + 1, ps * 3, 7, ps * 25 + ps // 2, ps * 14]
    _fused_equals_separate(case, lens, [12 * r, 5 * r, 4 * r, 1, 20 * r, 9 * r], 24 * r)


# request bound in pages, further one-page requests (with them the pairs fill the chip)
LARGE = [
    (("mean_256_threads", 16, 0, 64, 4, 2, O.MEAN_DOT, True, None, 1, 0.0), 700, 0),
    (("quest_512_threads", 16, 0, 128, 8, 2, O.QUEST, False, None, 1, 0.0), 1500, 0),
    (("max_512_threads_16_heads", 16, 0, 64, 16, 16, O.MAX_DOT, False, torch.float8_e4m3fn, 1, 0.0), 1100, 0),
    (("mean_1024_threads", 16, 0, 128, 6, 2, O.MEAN_DOT, True, None, 2, 0.0), 2100, 0),
    (("max_512_threads_8_slots", 16, 0, 64, 8, 8, O.MAX_DOT, False, None, 1, 0.0), 2100, 30),
    (("quest_256_threads_16_slots", 16, 0, 64, 8, 8, O.QUEST, False, None, 1, 0.0), 2100, 70),
    (("quest_1024_threads_8_slots", 32, 16, 64, 8, 2, O.QUEST, False, torch.float8_e5m2, 1, 0.0), 2100, 0),
    (("mean_1024_threads_16_slots", 16, 0, 64, 4, 2, O.MEAN_DOT, True, None, 1, 0.0), 8300, 0),
    (("max_past_the_slots", 16, 0, 64, 2, 1, O.MAX_DOT, False, None, 1, 0.0), 16500, 0),
    (("latent_512_threads", 16, 0, 576, 16, 1, O.MEAN_DOT, True, None, 1, 0.0), 1100, 0),
    (("latent_512_threads_16_slots", 16, 0, 576, 16, 1, O.MEAN_DOT, True, None, 1, 0.0), 4200, 0),
    (("latent_1024_threads_one_pass", 16, 0, 576, 16, 1, O.MEAN_DOT, False, None, 1, 0.0), 2100, 0),
]


@pytest.mark.parametrize("case,pages,more", LARGE, ids=[c[0][0] for c in LARGE])
def test_append_inside_large_selections(case, pages, more):
    """The same at the selection's workgroup sizes, where the append's tasks fill part of a workgroup, one or
    several; the appended token starts a block, ends one or lies within."""
    ps, r = case[1], case[1] // case[2] if case[2] else 1
    lens = [ps * (pages - 1) + 1, ps * (pages // 2), ps * (pages // 3) + 5, 2] + [ps] * more
    _fused_equals_separate(case, lens, [r * pages // 8, 60 * r, 7 * r, 1] + [1] * more, max(60, pages // 8) * r)


def _fused_equals_separate(case, lens, budget, max_sel):
    name, ps, bs, D, Hq, H, kind, two_pass, fp8, n_local, tau = case
    mla = D == 576
    r = ps // bs if bs else 1
    pb = random_problem(2200 + ps + D + Hq + n_local, lens, Hq=Hq, H=H, D=D, ps=ps, Dv=512 if mla else None,
                        alias_v=mla, extra_pages=4)
    ks, vs = 1.0, 1.0
    if fp8 is not None:
        ks, vs = 0.021, 0.0377
        pb = fp8_problem(pb, fp8, ks, vs)
    k, v, kn, vn = strip_last_token(pb, 2201)
    budget = torch.tensor(budget, dtype=torch.int32).cuda()
    n_sink, nl = r, n_local * r
    q = pb.q.cuda()
    opt = vx.topk_options(tolerate_ratio=tau, seed=5) if tau else None
    outs = []
    for fused in (False, True):
        kv, batch, (mean, mbf, mx, mn) = _state(pb, k, v, ks, vs, bs, H, D)
        ws = torch.zeros(vx.workspace_size(vx.STAGE_SCORE_TOPK, kv, batch, Hq, max_sel), dtype=torch.uint8,
                         device="cuda")
        sel = torch.full((pb.batch, H, max_sel), -7, dtype=torch.int32, device="cuda")
        cnt = torch.full((pb.batch,), -7, dtype=torch.int32, device="cuda")
        knc, vnc = kn.cuda(), None if vn is None else vn.cuda()
        bf = mbf if two_pass else None           # the bf16 Mean copy is maintained and read, or neither
        if fused:
            vx.append_score_topk(kv, batch, knc, vnc, mean, mx, mn, q, kind, budget, n_sink, nl, max_sel, sel, cnt,
                                 ws, mean_bf16=bf, options=opt)
        else:
            vx.kv_append_summarize(kv, batch, knc, vnc, mean, mx, mn, mean_bf16=bf)
            vx.page_score_topk(q, kv, batch, kind, mean, mx, mn, budget, n_sink, nl, max_sel, sel, cnt, ws,
                               mean_bf16=bf, options=opt)
        torch.cuda.synchronize()
        outs.append([kv.k, kv.v, mean, mbf, mx, mn, sel, cnt])
    as_bytes = lambda t: None if t is None else t.cpu().contiguous().view(torch.uint8)
    for a, b, what in zip(outs[0], outs[1], ["k", "v", "mean", "mean_bf16", "max", "min", "sel_pages", "sel_count"]):
        if a is None:
            assert b is None
            continue
        assert torch.equal(as_bytes(a), as_bytes(b)), what
    # the appended rows are the stripped token's
    assert torch.equal(as_bytes(outs[1][0]), as_bytes(pb.k))
