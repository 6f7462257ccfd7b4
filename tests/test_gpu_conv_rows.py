"""The input gradient from unpacked weights (lbm_nn_conv3x3 mode 1) takes its
tile by another line than the passes with packed ones: 4, 8 or 10 rows of 32,
on 16-wide images 8, 16 or 20 rows of 16 pixels.  Either side of the line every image
comes out with the same bits as alone; the last tile row is partly empty."""
import numpy as np
import pytest

from oracle import surrogate as S

pytestmark = pytest.mark.gpu
BF_REL = 2.0 ** -8


def _f64(t):
    return t.float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("n,h,w,ci,co", [
    (11, 12, 16, 384, 64), (10, 12, 16, 384, 64),     # 264 and 240 blocks of 8 x 16
    (18, 20, 16, 480, 96), (17, 8, 16, 512, 64),      # 20 x 16; one tile row: 8 x 16
    (22, 14, 64, 64, 64), (15, 14, 64, 64, 64),       # 8 x 32 from 257 blocks of 4 x 32 on
    (22, 10, 64, 128, 64), (33, 20, 32, 96, 96),      # 10 x 32, whole tiles
    (8, 18, 64, 384, 64), (9, 6, 128, 128, 64),       # 10 x 32 with empty rows; 8 x 32
    (40, 4, 64, 128, 64), (24, 2, 128, 96, 64),       # up to 4 rows: stays 4 x 32
])
def test_batch_and_single_image_agree(n, h, w, ci, co):
    import torch
    from paper_2211_05009_amd import lbm
    gen = torch.Generator().manual_seed(n + h + w + ci)

    def draw(*shape, scale=1.0):
        return (torch.randn(*shape, generator=gen) * scale).to(torch.bfloat16).cuda()

    gy, wt = draw(n, h, w, co + 8), draw(9, ci, co, scale=(9 * co) ** -0.5)

    def gradient(g):
        m = g.shape[0]
        gx = torch.full((m, h, w, ci + 16), 3.0, dtype=torch.bfloat16, device="cuda")
        lbm.lbm_nn_conv3x3(1, m, h, w, ci, co, g, co + 8, 8, None, 0, 0, wt, None, 0, gx,
                           ci + 16, 16)
        torch.cuda.synchronize()
        assert torch.all(gx[..., :16] == 3.0)
        return gx[..., 16:].contiguous()

    gx = gradient(gy)
    for b in (0, n // 2, n - 1):
        one = gradient(gy[b:b + 1].clone())
        assert torch.equal(one.view(torch.int16), gx[b:b + 1].view(torch.int16))
    x = np.zeros((1, h, w, ci))
    ref = S.conv3x3_backward(x, _f64(wt), _f64(gy[n - 1:])[..., 8:])[0]
    # half an ulp of bfloat16 on the output, FP32 accumulation below 1e-4 of the largest
    assert np.all(np.abs(_f64(gx[n - 1:]) - ref) <= BF_REL * np.abs(ref) + 1e-4 * np.abs(ref).max())
