"""The 16-query waves that the fused band takes on small grids against the 32-query waves
(BAND_SHAPE(0)): the same key blocks in the same order, so the same bits; and the largest
grid on each side of the choice."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 0, 1), (2, 15, 3, 1), (2, 17, 40, 2), (1, 63, 64, 1), (1, 65, 64, 1),
         (3, 64, 7, 5), (2, 129, 20, 2), (1, 512, 256, 1), (12, 3001, 200, 3), (4, 700, 300, 4),
         (703, 128, 16, 1), (704, 100, 16, 1)]


@pytest.mark.parametrize("b,l,w,dil", CASES)
@pytest.mark.parametrize("mask", [False, True])
def test_small_grid_waves(b, l, w, dil, mask):
    import paper_2208_02025_amd as ol
    g = torch.Generator().manual_seed(b * 10000 + l)
    q, k, v = (torch.randn(b, l, 64, generator=g).bfloat16().cuda() for _ in range(3))
    for out_dtype in (torch.float32, torch.bfloat16):
        got = torch.full((b, l, 64), float("nan"), dtype=out_dtype, device="cuda")
        ol.banded_bmm(q, k, v, w, dil, 0.125, mask_invalid=mask, out_dtype=out_dtype, out=got)
        ref = ol.banded_bmm(q, k, v, w, dil, 0.125, mask_invalid=mask, out_dtype=out_dtype,
                            flags=ol.BAND_SHAPE(0))
        assert torch.equal(got, ref)
