"""Scoring few inputs deals the classes of each first-layer tile to several workgroups.  A class's
scores are the same sums whichever workgroup takes it, so scores of small batches equal, bit for
bit, those of a batch large enough for one workgroup per tile (the tile size is the same).  Batches start at a tile's first row: the
fp32 product's k split adds a 32x32 block's parts in an order that depends on the block's place in
its tile."""
import pytest
import torch


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
# 16 columns: up to 256 tiles' worth of groups for every batch; 2000: one group from 257 inputs on
@pytest.mark.parametrize("d_out,C", [(16, 16), (1000, 7), (2000, 2), (2000, 10), (2000, 16)])
def test_scores_of_small_batches(dtype, d_out, C):
    import paper_2404_08573_amd as P
    gen = torch.Generator().manual_seed(d_out + C)
    bf = dtype == "bf16"
    layer = P.Layer(torch.randn(d_out, 72, generator=gen).cuda(),
                    torch.randn(d_out, generator=gen).cuda(), bf16_shadow=bf)
    hp = P.HParams(dtype=P.FF_BF16 if bf else P.FF_F32)
    x = torch.rand(500, 72, generator=gen).cuda()

    def scores(rows):
        out = torch.full((rows.shape[0], C), float("nan"), device="cuda")
        P.ff_score_labels([layer], hp, rows.contiguous(), C, 0, scores=out)
        torch.cuda.synchronize()
        return out

    whole = scores(x)
    assert torch.isfinite(whole).all()
    for a, b in ((0, 1), (64, 101), (128, 192), (192, 257), (256, 389)):
        assert torch.equal(scores(x[a:b]), whole[a:b]), (a, b)
