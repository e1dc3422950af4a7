"""The fp32 convolution in one kernel against the two stages it stands for (a GEMM tile override
keeps a call on them): the same bits, at the edges of pixel, channel and k-tiles, for strides,
dilations and paddings past the image."""
import pytest
import torch

pytestmark = pytest.mark.gpu

#        n, h, w, c, k, r, s, stride, pad, dil
CASES = [(1, 1, 1, 1, 1, 1, 1, 1, 0, 1), (1, 7, 9, 3, 5, 3, 3, 1, 1, 1),
         (2, 8, 8, 32, 32, 3, 3, 1, 1, 1), (1, 5, 13, 33, 31, 3, 5, (1, 2), (1, 2), 1),
         (3, 11, 6, 36, 65, 5, 5, 2, 2, 1), (1, 16, 16, 64, 64, 3, 3, 1, 2, 2),
         (1, 4, 4, 16, 100, 3, 3, 1, 5, 3), (4, 33, 31, 4, 40, 3, 2, 1, (0, 1), 1),
         (2, 40, 40, 31, 33, 1, 1, 1, 0, 1), (8, 56, 56, 64, 64, 3, 3, 1, 1, 1),
         (1, 14, 14, 128, 128, 5, 5, 1, 2, 1), (16, 41, 41, 8, 96, 3, 3, 1, 1, 1)]


def _bits(t):
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("tail", [False, True])
def test_fused_f32_matches_stages(case, tail):
    import paper_2208_02025_amd as ol
    n, h, w, c, k, r, s, stride, pad, dil = case
    g = torch.Generator().manual_seed(n + h + w + c + k)
    x = torch.randn((n, h, w, c), generator=g).cuda()
    wt = torch.randn((r, s, k, c), generator=g).cuda()
    if h > 1:   # non-finite values reach the same outputs
        x[0, 0, 0, 0], wt[0, 0, k - 1, c - 1] = float("inf"), float("nan")

    def run(flags, **kw):
        return ol.derived_dilated_conv2d(x, wt, stride, pad, dil, flags=flags, **kw)
    kw = {}
    if tail:
        shape = run(0).shape
        kw = dict(bias=torch.randn(k, generator=g).cuda(), relu=True, out_dtype=torch.bfloat16,
                  residual=torch.randn(shape, generator=g).cuda())
    ref = run(ol.GEMM_TILE(0), **kw)
    out = run(0, out=torch.full_like(ref, 7.0), **kw)
    nan = torch.isnan(ref)
    assert torch.equal(nan, torch.isnan(out))
    assert torch.equal(_bits(out)[~nan], _bits(ref)[~nan])
