"""Weight gradients over few rows: at the edges of the 32 x 64 tiles, of the k16
steps and of the waves' quarters of the rows, and just past the range."""
import pytest

import paper_2211_10725_amd as snn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n_in,n_out", [(64, 64, 64), (65, 65, 97), (79, 784, 129), (128, 1000, 500),
                                          (129, 3072, 1000), (255, 191, 70), (800, 784, 1000),
                                          (1023, 333, 64), (1024, 64, 331), (63, 200, 300),
                                          (1025, 200, 300),
                                          # around the limits on small outputs and on tiles
                                          (896, 256, 256), (897, 256, 256), (1000, 256, 264),
                                          (64, 2048, 992), (64, 2000, 1024), (64, 2049, 1000),
                                          (96, 2560, 1000), (95, 2560, 1000), (96, 2561, 1024),
                                          (97, 2544, 1033)])
def test_weight_gradient_of_few_rows(M, n_in, n_out):
    """Against the fp64 product: an fp32 sum of 3 M exact part products, in any
    order, is within (3 M + 2) 2^-24 of the sum of its terms' magnitudes."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M * n_in)
    x = (torch.rand((M, n_in), generator=g, device="cuda") < 0.4).to(torch.uint8)
    W = torch.rand((n_out, n_in), generator=g, device="cuda")
    dI = torch.randn((M, n_out), generator=g, device="cuda")
    d = snn.layer_desc(dict(kind="dense", n_in=n_in, n_out=n_out, neuron="leaky", beta=0.9), 1, M)
    gW = torch.full((n_out, n_in), float("nan"), device="cuda")
    ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
    snn.snn_synapse_bwd(d, dI, None, x, W, gW, None, ws)
    xd, dd = x.double(), dI.double()
    err = (gW.double() - dd.t() @ xd).abs()
    assert bool((err <= (3 * M + 2) * 2.0 ** -24 * (dd.abs().t() @ xd)).all())
