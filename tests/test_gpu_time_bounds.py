"""Calls whose time once grew by a half or more on inputs that no benchmark times, each held against
another call of the same process, so that the card's clocks and load drop out.  Both sides are the
fastest of several windows; a limit lies between the two ratios that are noted beside it, the one
measured and the one it is to keep out."""
import numpy as np
import pytest
import torch

from paper_2606_06453_amd import vx

pytestmark = pytest.mark.gpu


def fastest_us(call, windows=7, window_us=4000.0):
    call()
    torch.cuda.synchronize()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def window(n):
        a.record()
        for _ in range(n):
            call()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) * 1e3 / n
    n = max(5, int(window_us / window(10)))
    return min(window(n) for _ in range(windows))


def int32(x):
    return torch.as_tensor(np.asarray(x), dtype=torch.int32).cuda()


def batch_of(pages, page_size, bound=None):
    """Requests of whole pages over one run of physical pages; their BatchSpec and the page count."""
    indptr = np.concatenate([[0], np.cumsum(pages)])
    total = int(indptr[-1])
    return vx.BatchSpec(int32(indptr), int32(np.random.default_rng(0).permutation(total)),
                        int32(np.asarray(pages) * page_size), bound or int(max(pages))), total


def test_step_refresh():
    """The refresh of 512 requests' last blocks (16 heads of 128 fp8 channels, 64 tokens) against a plain
    read of the same bytes: 2.44 measured; 3.62 with a second copy of the row sums in the kernel, whose
    registers left two waves per SIMD."""
    B, H, ps, D = 512, 16, 64, 128
    batch, total = batch_of([2] * B, ps)
    batch.seq_lens -= 3                     # part full, as a decode step's blocks are
    k = torch.zeros((total, H, ps, D), dtype=torch.uint8, device="cuda").view(torch.float8_e4m3fn)
    kv = vx.PagedKV(k, k, D)
    mean = torch.empty((total, H, D), dtype=torch.float32, device="cuda")
    bf = [torch.empty((total, H, D), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    first = int32([1] * B)
    step = fastest_us(lambda: vx.page_summarize(kv, batch, first, mean, bf[0], bf[1], mean_bf16=bf[2]))
    half = k.view(torch.uint8)[: total // 2]
    sink = torch.empty(2048, dtype=torch.int32, device="cuda")
    read = fastest_us(lambda: vx.stream_read(half, sink))
    assert step < 3.0 * read


@pytest.mark.parametrize("kind", [vx.MEAN_DOT, vx.QUEST])
def test_selection_with_an_outlier(kind):
    """One block that scores far above the others, outside the sinks, against the same call without it:
    1.47 (block mean) and 1.29 (Quest) measured; 4.5 and 4.8 when the histogram's equal bins put all other
    blocks into one and every block was re-scored."""
    B, H, P, D = 8, 8, 8192, 128
    batch, total = batch_of([P] * B, 16)
    k = torch.zeros((total, H, 16, D), dtype=torch.uint8, device="cuda").view(torch.float8_e4m3fn)
    kv = vx.PagedKV(k, k, D)
    gen = torch.Generator(device="cuda").manual_seed(1)
    mean = torch.randn((total, H, D), generator=gen, device="cuda") * 0.25
    q = torch.randn((B, 4 * H, D), generator=gen, device="cuda").to(torch.bfloat16)
    budget, sel = int32([128] * B), torch.empty((B, H, 128), dtype=torch.int32, device="cuda")
    ws = torch.empty(vx.workspace_size(vx.STAGE_SCORE_TOPK, kv, batch, 4 * H, 128), dtype=torch.uint8, device="cuda")
    count = torch.empty(B, dtype=torch.int32, device="cuda")
    us = []
    for far in (1.0, 1e6):
        mean[batch.page_indices.view(B, P)[:, 7].long()] *= far
        bf, hi, lo = mean.to(torch.bfloat16), (mean + 0.4).to(torch.bfloat16), (mean - 0.4).to(torch.bfloat16)
        us.append(fastest_us(lambda: vx.page_score_topk(
            q, kv, batch, kind, mean if kind == vx.MEAN_DOT else None, hi if kind == vx.QUEST else None,
            lo if kind == vx.QUEST else None, budget, 0, 1, 128, sel, count, ws,
            mean_bf16=bf if kind == vx.MEAN_DOT else None)))
    assert us[1] < 2.5 * us[0]


def test_short_rows_under_a_large_bound():
    """Rows of at most 8192 scores in a stride past the page slots, against the same rows in their own stride:
    2.0 measured, 5.4 when such rows were read again in every pass."""
    H, B, P = 8, 16, 8192
    items, budget = int32(np.random.default_rng(0).integers(P // 2, P + 1, B)), int32([512] * B)
    sel, count = torch.empty((B, H, 512), dtype=torch.int32, device="cuda"), torch.empty(B, dtype=torch.int32, device="cuda")
    us = [fastest_us(lambda: vx.topk_select(x, items, budget, 1, 2, 512, sel, count))
          for x in (torch.randn((H, B, stride), device="cuda") for stride in (P, 20000))]
    assert us[1] < 3.5 * us[0]


@pytest.mark.parametrize("B,P,limit", [(16, 8192, 0.6), (200, 600, 0.75)])
def test_nsa_flow_of_single_heads(B, P, limit):
    """The NSA flow of groups of one query head against groups of four on the same rows: 0.34 and 0.56
    measured; 0.82 and 0.89 when a head kept one wave and left the others idle."""
    H, n = 8, int32([P - 5] * B)
    out = torch.empty((H, B, P), device="cuda")
    us = [fastest_us(lambda: vx.score_flow(vx.NSA, z, out, H, n))
          for z in (3 * torch.randn((H * g, B, P), device="cuda") for g in (1, 4))]
    assert us[0] < limit * us[1]
