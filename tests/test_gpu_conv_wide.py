"""Convolution gradients of layers that the one-image kernels do not take: at the
edges of the row tiles (1 .. 36 pooled cells), of the channel groups (halves of
five, groups of ten) and of the k-steps of 32 output channels, with more images
than workgroups, images of odd sizes and values that are not finite."""
import numpy as np
import pytest

import oracle
import paper_2211_10725_amd as snn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _case(NB, Ci, H, W, Co, seed):
    rng = np.random.default_rng(seed)
    x = (rng.random((NB, Ci, H, W)) < 0.5).astype(np.uint8)
    k = 1.0 / np.sqrt(25 * Ci)
    w = rng.uniform(-k, k, (Co, Ci, 5, 5)).astype(np.float32)
    Hp, Wp = (H - 4) // 2, (W - 4) // 2
    arg = rng.integers(0, 4, (NB, Co, Hp, Wp)).astype(np.uint8)
    dI = rng.normal(0, 1, (NB, Co, Hp, Wp)).astype(np.float32)
    spec = dict(kind="conv", c_in=Ci, h=H, w=W, c_out=Co, neuron="leaky", beta=0.5)
    return x, w, arg, dI, snn.layer_desc(spec, 1, NB)


def _bwd(d, dI, arg, x, w):
    gW = torch.full(w.shape, float("nan"), device="cuda")
    gx = torch.full(x.shape, float("nan"), device="cuda")
    ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
    snn.snn_synapse_bwd(d, torch.as_tensor(dI).cuda(), torch.as_tensor(arg).cuda(),
                        torch.as_tensor(x).cuda(), torch.as_tensor(w).cuda(), gW, gx, ws)
    return gW.cpu().numpy(), gx.cpu().numpy()


@pytest.mark.parametrize("NB,Ci,H,W,Co", [
    (12, 13, 6, 6, 8), (13, 14, 8, 9, 32), (15, 16, 9, 8, 33), (12, 20, 12, 12, 65), (14, 21, 12, 14, 64),
    (13, 11, 14, 14, 96), (300, 32, 14, 14, 17), (12, 5, 16, 16, 31), (13, 6, 17, 16, 64),
    (12, 10, 16, 17, 1), (70, 48, 15, 14, 96), (12, 16, 8, 40, 64),
    (12, 12, 16, 16, 80), (12, 8, 20, 20, 24), (12, 12, 14, 13, 100), (11, 13, 8, 8, 16),
    # enough images for the input gradient's kernel; many channels on images of
    # one pooled cell, which stay with the contraction
    (33, 20, 12, 12, 65), (64, 11, 14, 14, 96), (64, 6, 17, 16, 64), (24, 10, 16, 17, 1),
    (33, 16, 8, 40, 64), (300, 168, 6, 6, 100), (120, 60, 7, 7, 70)])
def test_conv_bwd_wide(NB, Ci, H, W, Co):
    x, w, arg, dI, d = _case(NB, Ci, H, W, Co, NB + Ci + Co)
    gW, gx = _bwd(d, dI, arg, x, w)
    dY = oracle.maxpool2_bwd(dI, arg, H - 4, W - 4)
    rW, _, rx = oracle.conv_bwd(dY, x, w)
    tW, _, tx = oracle.conv_bwd(np.abs(dY), x, np.abs(w))
    # dx: at most six part products per output channel (each within 2^-26 of
    # the exact product), then 25 taps; dW: three exact part products per row
    assert (np.abs(gx - rx) <= ((6 * Co + 27) * 2.0 ** -24 + 2.0 ** -26) * tx + 1e-30).all()
    rows = 4 * arg.shape[0] * arg.shape[2] * arg.shape[3]
    assert (np.abs(gW - rW) <= (3 * rows + 2) * 2.0 ** -24 * tW + 1e-30).all()


@pytest.mark.parametrize("NB", [13, 40])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan"), 3.4e38])
def test_conv_dx_wide_of_special_values(bad, NB):
    """dL/dI with a value that is not finite, or near fp32's largest: the
    gradient has the values the fp32 products give, an infinity against a
    nonzero weight an infinity of the product's sign."""
    Ci, H, W, Co = 16, 14, 14, 40
    x, w, arg, dI, d = _case(NB, Ci, H, W, Co, 3)
    dI[1, 7, 2, 3] = bad
    _, gx = _bwd(d, dI, arg, x, w)
    with np.errstate(all="ignore"):
        dY = torch.as_tensor(np.asarray(oracle.maxpool2_bwd(dI, arg, H - 4, W - 4))).double()
        ref = torch.nn.functional.conv_transpose2d(dY, torch.as_tensor(w).double())
        ref = ref.float().numpy()
    assert ref.shape == gx.shape
    np.testing.assert_array_equal(np.isnan(gx), np.isnan(ref))
    np.testing.assert_array_equal(np.isinf(gx), np.isinf(ref))
    inf = np.isinf(ref)
    np.testing.assert_array_equal(gx[inf], ref[inf])
    fin = np.isfinite(ref)
    assert (np.abs(gx[fin] - ref[fin]) <= 1e-5 * np.abs(ref[fin]).max()).all()
