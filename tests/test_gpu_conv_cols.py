"""The column kernel of the fused convolution against the per-tap one (FUSED_TILE(12)), at
the sizes where its tiles, windows and channel slices end: bit-exact on integer inputs
(every partial sum is an integer below 2^24, so any summation order gives the same bits)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# (op, n, h, w, c, k, r, s, stride, pad, dil, out_pad)
CASES = [
    # 3 taps high: single rows / columns, columns that straddle images and row blocks
    ("conv", 1, 1, 1, 64, 16, 3, 3, 1, 1, 1, 0),
    ("conv", 3, 2, 5, 512, 17, 3, 3, 1, 1, 1, 0),
    ("conv", 5, 7, 3, 128, 33, 3, 3, 1, 1, 1, 0),
    ("conv", 1, 7, 7, 512, 512, 3, 3, 1, 1, 1, 0),
    ("conv", 2, 9, 17, 320, 130, 3, 3, 1, 1, 1, 0),
    ("conv", 16, 14, 14, 256, 96, 3, 3, 1, 1, 1, 0),
    ("conv", 2, 13, 16, 192, 1, 3, 3, 1, 0, 1, 0),
    ("conv", 2, 29, 31, 64, 200, 3, 3, 1, 1, 1, 0),
    ("conv", 1, 95, 95, 64, 64, 3, 3, 1, 1, 1, 0),
    ("conv", 4, 57, 61, 128, 250, 3, 3, 1, 2, 1, 0),
    ("conv", 16, 28, 33, 64, 70, 3, 3, 1, 1, 1, 0),
    ("conv", 16, 40, 44, 128, 200, 3, 3, 1, 1, 1, 0),
    # kernels wider or narrower than high, asymmetric images
    ("conv", 2, 11, 40, 128, 64, 3, 7, 1, 3, 1, 0),
    ("conv", 2, 40, 11, 128, 64, 3, 1, 1, 1, 1, 0),
    ("conv", 2, 12, 10, 128, 48, 2, 4, 1, 1, 1, 0),
    ("conv", 1, 20, 19, 128, 96, 5, 5, 1, 2, 1, 0),
    ("conv", 1, 65, 130, 64, 32, 5, 5, 1, 2, 1, 0),
    ("conv", 2, 100, 106, 64, 64, 5, 5, 1, 2, 1, 0),
    ("conv", 8, 19, 21, 320, 100, 5, 3, 1, 2, 1, 0),
    # dilations: one class per residue, residues of unequal extent
    ("dilated", 1, 40, 20, 64, 64, 3, 3, 1, 2, 2, 0),
    ("dilated", 2, 23, 37, 192, 96, 3, 3, 1, 4, 4, 0),
    ("dilated", 1, 3, 2, 64, 24, 3, 3, 1, 3, 3, 0),
    ("dilated", 1, 96, 128, 256, 256, 3, 3, 1, 2, 2, 0),
    # transposed: the taps of a class run backwards; classes of equal tap counts
    ("convT", 1, 1, 1, 128, 32, 4, 4, 2, 1, 1, 0),
    ("convT", 16, 8, 8, 512, 40, 4, 4, 2, 1, 1, 0),
    ("convT", 1, 9, 13, 256, 50, 4, 4, 2, 1, 1, 0),
    ("convT", 2, 17, 31, 128, 70, 4, 4, 2, 0, 1, 1),
    ("convT", 4, 32, 30, 128, 64, 6, 6, 2, 2, 1, 0),
    ("convT", 1, 20, 21, 192, 64, 3, 3, 1, 1, 1, 0),
]


def _int(shape, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(-2, 3, shape, generator=g).to(torch.bfloat16).cuda()


def _run(case, x, wt, flags, **kw):
    import paper_2208_02025_amd as ol
    op, _, _, _, _, _, _, _, stride, pad, dil, out_pad = case
    if op == "conv":
        return ol.derived_conv2d(x, wt, stride, pad, fuse=True, flags=flags, **kw)
    if op == "dilated":
        return ol.derived_dilated_conv2d(x, wt, stride, pad, dil, fuse=True, flags=flags, **kw)
    return ol.derived_conv_transpose2d(x, wt, stride, pad, out_pad, dil, fuse=True, flags=flags,
                                       **kw)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_columns_match_per_tap_kernel(case):
    import paper_2208_02025_amd as ol
    _, n, h, w, c, k, r, s = case[:8]
    x, wt = _int((n, h, w, c), 1), _int((r, s, k, c), 2)
    ref = _run(case, x, wt, ol.FUSED_TILE(12))
    out = torch.full_like(ref, float("nan"))
    _run(case, x, wt, 0, out=out)
    assert torch.equal(out, ref)
    # with the element-wise tail and a bf16 result
    bias = _int((k,), 3)
    res = _int(tuple(ref.shape), 4)
    kw = dict(bias=bias, residual=res, relu=True, out_dtype=torch.bfloat16)
    assert torch.equal(_run(case, x, wt, 0, **kw), _run(case, x, wt, ol.FUSED_TILE(12), **kw))


def test_columns_keep_nonfinite_inputs_local():
    """A non-finite input reaches exactly the outputs whose window holds it."""
    import paper_2208_02025_amd as ol
    x, wt = _int((2, 14, 14, 256), 5), _int((3, 3, 64, 256), 6)
    x[1, 13, 13, 7] = float("inf")
    x[0, 0, 0, 255] = float("nan")
    out = ol.derived_conv2d(x, wt, 1, 1, fuse=True)
    bad = ~torch.isfinite(out).all(dim=3)
    ref = torch.zeros_like(bad)
    ref[1, 12:, 12:] = True
    ref[0, :2, :2] = True
    assert torch.equal(bad, ref)
