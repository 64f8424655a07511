"""Full summary passes at the launch shapes they choose between: one and two rounds of tasks per
workgroup (blocks of 16 tokens under a large request bound), token rows below and of a cache line,
the Mean alone, the envelope alone and both, ragged last blocks and an empty request."""
import pytest
import torch

from paper_2606_06453_amd import vx, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_dtype", ["bf16", "fp8_e4m3", "fp8_e5m2"])
@pytest.mark.parametrize("H,D,ps,block", [(16, 128, 16, 0), (8, 128, 32, 16), (2, 64, 16, 0), (1, 64, 32, 0), (1, 576, 16, 0)])
@pytest.mark.parametrize("bound", [7, 140000])        # blocks per request that the grid is laid out for
def test_full_pass_shapes(kv_dtype, H, D, ps, block, bound):
    bs, scale = block or ps, 0.25 if kv_dtype != "bf16" else 1.0
    r = ps // bs
    lens = [ps * 3 + 1, 0, ps * 2, ps * 6 + ps - 1, 5]
    pages = [-(-n // ps) for n in lens]
    total = sum(pages)
    gen = torch.Generator().manual_seed(D + ps)
    k = workloads.quantize_cache(torch.randn((total, H, ps, D), generator=gen).to(torch.bfloat16), kv_dtype, scale)
    perm = torch.randperm(total, generator=gen).to(torch.int32)
    indptr = torch.tensor([0] + pages).cumsum(0).to(torch.int32)
    v = None if D == 576 else k.cuda()
    kv = vx.PagedKV(k.cuda(), v, 512 if D == 576 else D, scale, scale, block)
    batch = vx.BatchSpec(indptr.cuda(), perm.cuda(), torch.tensor(lens, dtype=torch.int32).cuda(), max(bound, max(pages)))
    x = k.float() * scale                                                   # the fp32 cache values
    blocks = x.view(total, H, r, bs, D).transpose(1, 2).reshape(total * r, H, bs, D).double()
    want = {n: torch.full((total * r, H, D), -7.0, dtype=torch.float64) for n in ("mean", "max", "min")}
    for i, n in enumerate(lens):
        for j in range(-(-n // bs)):
            p = int(perm[int(indptr[i]) + j // r]) * r + j % r
            rows = blocks[p, :, :min(bs, n - j * bs)]
            want["mean"][p], want["max"][p], want["min"][p] = rows.mean(1), rows.amax(1), rows.amin(1)
    new = lambda dt: torch.full((total * r, H, D), -7.0, dtype=dt, device="cuda")  # noqa: E731
    for names in (("mean",), ("max", "min"), ("mean", "max", "min")):
        out = {n: new(torch.float32 if n == "mean" else torch.bfloat16) for n in names}
        vx.page_summarize(kv, batch, **out)
        torch.cuda.synchronize()
        for n in names:
            got = out[n].cpu().double()
            if n == "mean":      # bs fp32 additions and a division, each within 2^-24 of at most bs max|x| / bs
                assert (got - want[n]).abs().max() <= (bs + 1) * 2.0 ** -24 * blocks.abs().max()
            else:                # an fp8 value times the scale, a power of two, is exact in bf16
                assert torch.equal(got, want[n])
