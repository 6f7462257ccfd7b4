"""GPU tests of the tile choice of the 3x3 convolutions (k_conv_tile).

The tile a layer runs on (8 x 32, 4 x 32 or 8 x 16 pixels; one or several
32-channel chunks) follows from the batch, so the same image has to come out
bit for bit the same alone and in a batch: every output adds the same products
in the same order.  The images leave part of the last tile row empty, and are
also checked against the FP64 reference, with the bound of the layer tests
(half an ulp of bfloat16 on the output, FP32 accumulation below 1e-4 of the
largest output).
"""
import numpy as np
import pytest

from oracle import surrogate as S

pytestmark = pytest.mark.gpu
BF_REL = 2.0 ** -8


def _f64(t):
    return t.float().cpu().numpy().astype(np.float64)


# (n, h, w, ci, co): over 256 blocks of 8 x 32 pixels in a batch, a few alone
@pytest.mark.parametrize("n,h,w,ci,co", [(24, 10, 128, 32, 96), (24, 10, 128, 96, 32),
                                         (40, 14, 64, 64, 160), (48, 12, 32, 96, 192),
                                         (48, 4, 32, 192, 192), (40, 12, 16, 96, 128)])
def test_batch_and_single_image_agree(n, h, w, ci, co):
    import torch
    from paper_2211_05009_amd import lbm
    gen = torch.Generator().manual_seed(n + h + w + ci)

    def draw(*shape, scale=1.0):
        return (torch.randn(*shape, generator=gen) * scale).to(torch.bfloat16).cuda()

    x, gy = draw(n, h, w, ci + 8), draw(n, h, w, co)
    wt = draw(9, ci, co, scale=(9 * ci) ** -0.5)
    bias = torch.randn(co, generator=gen).cuda()
    old = draw(n, h, w, ci)

    def both(xb, gb, ob):
        m = xb.shape[0]
        y = torch.zeros((m, h, w, co), dtype=torch.bfloat16, device="cuda")
        gx = ob.clone()
        lbm.lbm_nn_conv3x3(0, m, h, w, ci, co, xb, ci + 8, 8, None, 0, 0, wt, bias, 1, y, co, 0)
        lbm.lbm_nn_conv3x3(1, m, h, w, ci, co, gb, co, 0, None, 0, 0, wt, None, 0, gx, ci, 0,
                           accumulate=True)
        torch.cuda.synchronize()
        return y, gx

    y, gx = both(x, gy, old)
    for b in (0, n // 2, n - 1):
        y1, gx1 = both(x[b:b + 1].clone(), gy[b:b + 1].clone(), old[b:b + 1].clone())
        assert torch.equal(y1.view(torch.int16), y[b:b + 1].view(torch.int16))
        assert torch.equal(gx1.view(torch.int16), gx[b:b + 1].view(torch.int16))
    b = n - 1
    xr, W = _f64(x[b:b + 1])[..., 8:], _f64(wt)
    ref = np.maximum(S.conv3x3(xr, W, _f64(bias)), 0)
    assert np.all(np.abs(_f64(y[b:b + 1]) - ref) <= BF_REL * np.abs(ref) + 1e-4 * np.abs(ref).max())
    ref = _f64(old[b:b + 1]) + S.conv3x3_backward(xr, W, _f64(gy[b:b + 1]))[0]
    assert np.all(np.abs(_f64(gx[b:b + 1]) - ref) <= BF_REL * np.abs(ref) + 1e-4 * np.abs(ref).max())


def test_network_outputs_do_not_depend_on_the_batch():
    """The pools and upsamplings written by the layers' epilogues included."""
    import torch
    from paper_2211_05009_amd import lbm
    sur = lbm.Surrogate(max_batch=16)
    sur.set_params(S.he_init(1))
    re, ar = np.linspace(200.0, 3000.0, 16), np.linspace(0.3, 2.0, 16)
    out = torch.empty((16, 256, 128, 3), dtype=torch.float32, device="cuda")
    one = torch.empty((1, 256, 128, 3), dtype=torch.float32, device="cuda")
    sur.forward(re, ar, out)
    for b in (0, 7, 15):
        sur.forward(re[b:b + 1], ar[b:b + 1], one)
        assert torch.equal(one[0], out[b])
    sur.close()


@pytest.mark.parametrize("n", [1, 5, 16])
def test_forecast_equals_the_training_forward(n):
    """A forecast's first layer encodes (Re, Ar) itself and its last one writes
    the result; training reads the encoded canvas.  Against its own forecast as
    the target, a training step's loss is exactly zero."""
    import torch
    from paper_2211_05009_amd import lbm
    sur = lbm.Surrogate(max_batch=16)
    sur.set_params(S.he_init(2))
    re, ar = np.linspace(150.0, 2500.0, n), np.linspace(0.4, 1.9, n)
    out = torch.full((n, 256, 128, 3), np.nan, dtype=torch.float32, device="cuda")
    sur.forward(re, ar, out)
    mask = torch.ones((n, 256, 128), dtype=torch.float32, device="cuda")
    assert float(out.abs().max()) > 0
    assert sur.train_step(re, ar, out, mask, lr=0.0, apply_update=False) == 0.0
    sur.close()


def test_gradients_do_not_depend_on_the_partials_buffer():
    """The partial sums of consecutive layers are added in groups that follow
    from the handle's buffer (its largest batch): the same gradients, bit for
    bit."""
    import torch
    from paper_2211_05009_amd import lbm
    gen = torch.Generator().manual_seed(5)
    target = torch.randn(2, 256, 128, 3, generator=gen).cuda()
    mask = torch.ones((2, 256, 128), dtype=torch.float32, device="cuda")
    grads = []
    for nmax in (2, 16):
        sur = lbm.Surrogate(max_batch=nmax)
        sur.set_params(S.he_init(3))
        for _ in range(2):
            sur.train_step([900.0, 400.0], [1.1, 0.7], target, mask, lr=0.0, apply_update=False)
        grads.append(sur.get_params(with_grads=True)[1])
        sur.close()
    assert np.any(grads[0] != 0) and np.array_equal(grads[0], grads[1])
