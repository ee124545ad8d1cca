"""The time scans at the edges of their 16-step blocks: sequences one step short
of, equal to and past one, two and three blocks, on columns that fill no whole
workgroup (the lanes past the last column repeat it)."""
import numpy as np
import pytest

import oracle
import paper_2211_10725_amd as snn
from tests.parity import assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("neuron,alpha", [("leaky", 0.0), ("synaptic", 0.9), ("rleaky", 0.0)])
@pytest.mark.parametrize("T", [15, 16, 17, 31, 32, 33, 47, 48, 49])
def test_scan_block_edges(T, neuron, alpha):
    B, N = 5, 131
    rng = np.random.default_rng(T)
    I = rng.normal(0.3, 0.8, (T, B, N)).astype(np.float32)
    v = rng.uniform(-1.0, 1.5, N).astype(np.float32) if neuron == "rleaky" else None
    spec = dict(kind="none", n=N, neuron=neuron, beta=0.9, alpha=alpha, thr=1.0)
    d = snn.layer_desc(spec, T, B)
    x = torch.as_tensor(I).cuda()
    vt = None if v is None else torch.as_tensor(v).cuda()
    spk = torch.empty((T, B, N), dtype=torch.uint8, device="cuda")
    counts = torch.empty((B, N), device="cuda")
    ck = snn.ckpt_buffer(d)
    snn.snn_neuron_fwd(d, x, vt, spk, ck, counts)
    z, u, c = oracle.scan_fwd(I, neuron, 0.9, 1.0, alpha, v=v)
    np.testing.assert_array_equal(spk.cpu().numpy(), z)
    np.testing.assert_array_equal(counts.cpu().numpy(), c)
    ws = torch.empty(max(256, snn.snn_layer_workspace_bytes(d)), dtype=torch.uint8, device="cuda")
    g = rng.normal(0, 1, (T, B, N)).astype(np.float32)
    dup = rng.normal(0, 0.1, (T, B, 10)).astype(np.float32)
    wup = rng.uniform(-1, 1, (10, N)).astype(np.float32)
    for kind, arg, up in ((snn.GRAD_FULL, torch.as_tensor(g).cuda(), g),
                          (snn.GRAD_BCAST, torch.as_tensor(g[0]).cuda(), g[0]),
                          (snn.GRAD_FOLD, (torch.as_tensor(dup).cuda(), torch.as_tensor(wup).cuda()),
                           (dup.astype(np.float64) @ wup.astype(np.float64)).astype(np.float32))):
        dI = torch.full((T, B, N), float("nan"), device="cuda")
        gv = None if v is None else torch.empty(N, device="cuda")
        snn.snn_neuron_bwd(d, kind, arg, vt, x, ck, dI, None, gv, ws)
        if v is None:
            ref = oracle.scan_bwd(u, up, neuron, 0.9, 1.0, 25.0, alpha)
        else:
            ref, rv = oracle.scan_bwd_rleaky(u, up, 0.9, 1.0, 25.0, v)
            assert_close(gv.cpu().numpy(), rv, 1e-3, what="dL/dv")
        assert_close(dI.cpu().numpy(), ref, 1e-3, what=f"dL/dI {kind}")
