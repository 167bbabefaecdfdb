"""The linear surrogate on short inputs, loaded row by row, and on long ones, streamed: at the edges of its 8-token blocks, with
widths that end inside a wavefront's 512 inputs, fewer heads than eight, and batches whose sequences
end inside a block.  fp32 sums of bf16 products over D_h: within 2 * sqrt(D_h) * 2^-24 of the sum of
the products' magnitudes (a random walk of roundings, with a factor for its tail)."""
import pytest
import torch

from paper_2601_07891_amd import binding
from tests import deal

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,T,Dh,H", [
    (1, 1, 64, 1), (1, 7, 512, 8), (1, 8, 576, 8), (1, 9, 1088, 3), (3, 5, 4096, 8), (1, 1024, 4096, 8),
    (2, 1023, 2048, 4), (1, 130, 5120, 8), (1, 130, 5184, 8), (1, 130, 4096, 9), (5, 77, 4992, 7),
    (1, 8192, 256, 8), (1, 8193, 256, 8), (1, 6144, 320, 2), (1, 6145, 320, 1), (1, 8192, 192, 3),
])
@pytest.mark.parametrize("bias", [False, True])
def test_against_float64(B, T, Dh, H, bias):
    g = torch.Generator().manual_seed(B * T + Dh)
    x = torch.randn((B, T, Dh), generator=g).bfloat16()
    W = (torch.randn((H, Dh), generator=g) * Dh ** -0.5).bfloat16()
    b = torch.randn(H, generator=g).bfloat16() if bias else None
    got = binding.kvzap_score(x.to(DEV), W.to(DEV), None if b is None else b.to(DEV), None, None).double().cpu()
    x64, W64 = x.double(), W.double()
    want = x64 @ W64.t() + (0 if b is None else b.double())
    size = x64.abs() @ W64.abs().t() + 1.0
    assert ((got.transpose(1, 2) - want).abs() <= 2 * Dh ** 0.5 * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("B,T,Dh,H,form", [
    (1, 4609, 4096, 8, "rows"),                                        # a third round of row blocks
    (1, 6145, 4096, 8, "stream"),                                      # the first input of a fourth
    (1, 3663, 4096, 9, "short"), (1, 4112, 4096, 9, "stream"), (1, 5001, 4096, 16, "stream"),   # more heads than the row kernel's
    (3, 2731, 4160, 8, "stream"), (1, 9999, 2112, 3, "stream"),        # D_h ends inside a stage
    (1, 6145, 8192, 8, "stream"), (1, 4400, 8960, 8, "stream"),        # W leaves room for 6 and 4 wavefronts
    (2, 40001, 448, 1, "stream"), (7, 37500, 64, 5, "stream"),         # one and a half stages a row; less than one
    (7, 33500, 64, 5, "stream"), (7, 33400, 64, 5, "wide"), (1, 31249, 512, 8, "narrow"), (1, 31250, 512, 8, "stream"),
    (1, 12701, 2048, 8, "narrow"), (1, 16385, 2048, 8, "stream"),      # the ends of the narrow blocks' last stretch
])
@pytest.mark.parametrize("bias", [False, True])
def test_long_inputs_against_float64(B, T, Dh, H, form, bias):
    assert deal.linear_form(B * T, Dh, H) == form
    g = torch.Generator(device=DEV).manual_seed(B * T + Dh)
    x = torch.randn((B, T, Dh), generator=g, device=DEV).bfloat16()
    W = (torch.randn((H, Dh), generator=g, device=DEV) * Dh ** -0.5).bfloat16()
    b = torch.randn(H, generator=g, device=DEV).bfloat16() if bias else None
    got = binding.kvzap_score(x, W, b, None, None).double()
    W64 = W.double()
    for i in range(B):
        x64 = x[i].double()
        want = x64 @ W64.t() + (0 if b is None else b.double())
        size = x64.abs() @ W64.abs().t() + 1.0
        assert ((got[i].t() - want).abs() <= 2 * Dh ** 0.5 * 2.0 ** -24 * size).all()
