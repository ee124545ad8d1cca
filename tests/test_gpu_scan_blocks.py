"""The time scans at the edges of their 16-step blocks: sequences one step short
of, equal to and past one, two and three blocks, on columns that fill no whole
workgroup (the lanes past the last column repeat it), and the reverse scan in
place."""
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


# last workgroups of two whole waves, a part of one and an empty one; of one lane
# per column and of two columns per lane
@pytest.mark.parametrize("neuron,alpha", [("leaky", 0.0), ("synaptic", 0.9), ("rleaky", 0.0)])
@pytest.mark.parametrize("T,B,N", [(33, 5, 131), (50, 3, 64), (35, 3, 174806), (3, 1, 65)])
def test_reverse_scan_in_place(T, B, N, neuron, alpha):
    """dL/dI written over the currents or over the gradient of every step is bit
    for bit the one written elsewhere."""
    d = snn.layer_desc(dict(kind="none", n=N, neuron=neuron, beta=0.9, alpha=alpha, thr=1.0), T, B)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    x = torch.randn((T, B, N), generator=gen, device="cuda") * 0.8 + 0.3
    v = torch.rand(N, generator=gen, device="cuda") if neuron == "rleaky" else None
    spk = torch.empty((T, B, N), dtype=torch.uint8, device="cuda")
    ck = snn.ckpt_buffer(d)
    snn.snn_neuron_fwd(d, x, v, spk, ck, None)
    g = torch.randn((T, B, N), generator=gen, device="cuda")
    fold = (torch.randn((T, B, 10), generator=gen, device="cuda"),
            torch.rand((10, N), generator=gen, device="cuda"))
    ws = torch.empty(max(256, snn.snn_layer_workspace_bytes(d)), dtype=torch.uint8, device="cuda")

    def run(kind, up, cur, out):
        gv = None if v is None else torch.empty(N, device="cuda")
        snn.snn_neuron_bwd(d, kind, up, v, cur, ck, out, None, gv, ws)
        return out, gv

    for kind, up, where in ((snn.GRAD_FULL, g, ("cur", "g")), (snn.GRAD_BCAST, g[0], ("cur",)),
                            (snn.GRAD_FOLD, fold, ("cur",))):
        ref, rv = run(kind, up, x, torch.full_like(x, float("nan")))
        for w in where:
            cur, u = x.clone(), up.clone() if kind == snn.GRAD_FULL else up
            out, gv = run(kind, u, cur, cur if w == "cur" else u)
            assert torch.equal(out, ref), (kind, w)
            assert rv is None or torch.equal(gv, rv)
