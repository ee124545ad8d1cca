"""Contractions of odd sizes through the stage calls, at the edges of the tiles,
k-tiles and splits of the kernels that stage all parts of an operand together.

Each product is compared with the fp64 product of the same values.  Bound: an
fp32 sum of K exact products in any order is within (K + 2) 2^-24 of the sum
of its terms' magnitudes; the fp32 x fp32 input gradient takes six of the nine
part products (6 K terms, and 2^-26 of each term left out).
"""
import numpy as np
import pytest

import paper_2211_10725_amd as snn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# rows, n_in, n_out: tiles with one row or column past a multiple of 128 / 256,
# k-tiles with 1 .. 63 valid values, widths that are not whole 16-byte chunks
SHAPES = [(2049, 769, 705), (4097, 521, 513), (1281, 1003, 1101), (16390, 257, 264),
          (1025, 4104, 256), (8193, 200, 776), (300, 2048, 2056)]


def _layer(M, n_in, n_out, half, seed, grad_dtype=None):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = (torch.rand((M, n_in), generator=g, device="cuda") < 0.4)
    W = torch.rand((n_out, n_in), generator=g, device="cuda") * 2 - 1
    b = torch.rand(n_out, generator=g, device="cuda") * 2 - 1
    dI = torch.randn((M, n_out), generator=g, device="cuda")
    spec = dict(kind="dense", n_in=n_in, n_out=n_out, neuron="leaky", beta=0.9)
    if half:
        x, W, dI = x.half(), W.half(), dI.half()
        d = snn.layer_desc(spec, 1, M, in_dtype=snn.F16, w_dtype=snn.F16, grad_dtype=snn.F16)
    else:
        x = x.to(torch.uint8)
        d = snn.layer_desc(spec, 1, M)
    return d, x, W, b, dI


def _within(got, ref, terms, n, extra, what):
    err = (got.double() - ref).abs()
    bound = ((n + 2) * 2.0 ** -24 + extra) * terms
    assert bool((err <= bound).all()), f"{what}: {float((err / bound.clamp_min(1e-300)).max()):.2f}"


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("M,n_in,n_out", SHAPES)
def test_ragged_contractions(M, n_in, n_out, half):
    d, x, W, b, dI = _layer(M, n_in, n_out, half, M + n_in)
    ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
    cur = torch.full((M, n_out), float("nan"), device="cuda")
    gW = torch.full((n_out, n_in), float("nan"), device="cuda")
    gx = torch.full((M, n_in), float("nan"), device="cuda")
    S = 8.0 if half else 1.0
    scale = torch.full((4,), S, device="cuda")
    snn.snn_synapse_fwd(d, x, W, b, cur, None, ws)
    snn.snn_synapse_bwd(d, dI, None, x, W, gW, gx, ws, dcur_scale=scale if half else None)
    xd, Wd, bd, dd = x.double(), W.double(), b.double(), dI.double() / S
    _within(cur, xd @ Wd.t() + bd, xd @ Wd.abs().t() + bd.abs(), n_in + 1, 0.0, "currents")
    _within(gW, dd.t() @ xd, dd.abs().t() @ xd, M, 0.0, "dW")
    _within(gx, dd @ Wd, dd.abs() @ Wd.abs(), n_out if half else 6 * n_out,
            0.0 if half else 2.0 ** -26, "dx")


@pytest.mark.parametrize("M,n_in,n_out", [(2049, 769, 705), (3000, 640, 768)])
def test_bf16_spikes_match_bytes(M, n_in, n_out):
    """Spikes given as bf16 0/1 are contracted in the same order as bytes."""
    d, x, W, b, dI = _layer(M, n_in, n_out, False, 5)
    out = []
    for t in (snn.U8, snn.BF16):
        e = d.copy()
        e.in_dtype = t
        xi = x if t == snn.U8 else x.bfloat16()
        ws = torch.empty(snn.snn_layer_workspace_bytes(e) + 256, dtype=torch.uint8, device="cuda")
        cur = torch.empty((M, n_out), device="cuda")
        gW = torch.empty((n_out, n_in), device="cuda")
        snn.snn_synapse_fwd(e, xi, W, b, cur, None, ws)
        snn.snn_synapse_bwd(e, dI, None, xi, W, gW, None, ws)
        out.append((cur, gW))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("from_planes", [False, True])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan"), 3.4e38])
def test_input_gradient_of_special_values(bad, from_planes):
    """An infinity, NaN or value near fp32's largest in dL/dI or W gives the
    input gradient the fp32 products give, not the NaN of its parts; its last
    value sits in a partial k-tile.  Both with dL/dI in fp32 and as the planes
    the reverse scan writes (the layer call)."""
    M, n_in, n_out = 1600, 768, 1000
    d, x, W, b, dI = _layer(M, n_in, n_out, False, 9)
    W[999, 3] = bad
    W[:, 700] = 0.0
    if not from_planes:
        dI[5, 999] = bad
        dI[77, 40] = bad
    ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
    gx = torch.empty((M, n_in), device="cuda")
    if from_planes:
        cur = torch.zeros((M, n_out), device="cuda")
        assert snn.snn_layer_dcur_t_layout(d) == snn.DCUR_T_PLANES
        dI[5, 999] = bad
        saved = torch.zeros(snn.snn_layer_saved_bytes(d), dtype=torch.uint8, device="cuda")
        snn.saved_parts(d, saved)[0].copy_(cur.view(1, M, n_out))
        gW = torch.empty_like(W)
        snn.snn_layer_bwd(d, snn.GRAD_FULL, dI, x, W, None, saved, gW, None, None, gx, ws)
        sg = torch.tensor(1.0, device="cuda") / (1.0 + torch.tensor(25.0, device="cuda")) ** 2
        dI = dI * sg
    else:
        snn.snn_synapse_bwd(d, dI, None, x, W, None, gx, ws)
    ref = (dI.double() @ W.double()).float()  # overflows to infinity as the fp32 sum does
    fin = torch.isfinite(ref)
    assert torch.equal(torch.isnan(gx), torch.isnan(ref))
    assert torch.equal(torch.isinf(gx), torch.isinf(ref))
    assert torch.equal(gx[torch.isinf(ref)], ref[torch.isinf(ref)])
    tol = (6 * n_out + 6) * 2.0 ** -24 * (dI[:, :].double().abs() @ W.double().abs())
    assert bool(((gx.double() - ref.double()).abs()[fin] <= tol[fin]).all())


@pytest.mark.parametrize("M,n_in,n_out", [(1600, 768, 1000), (2013, 1003, 1101), (300, 2048, 2056)])
def test_input_gradient_of_a_diverged_step(M, n_in, n_out):
    """Rows of dL/dI all NaN, all infinite, with one NaN or one infinity, among
    finite ones: every block of the product has values to be taken again, and
    the finite rows keep theirs."""
    d, x, W, b, dI = _layer(M, n_in, n_out, False, 31)
    W = W.abs() + 0.25  # an infinite row sums to an infinity
    inf = float("inf")
    dI[0::8], dI[1::8], dI[2::8, n_out - 1], dI[3::8, 17] = float("nan"), inf, -inf, float("nan")
    ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
    gx = torch.empty((M, n_in), device="cuda")
    snn.snn_synapse_bwd(d, dI, None, x, W, None, gx, ws)
    assert bool(torch.isnan(gx[0::8]).all()) and bool(torch.isnan(gx[3::8]).all())
    assert bool((gx[1::8] == inf).all()) and bool((gx[2::8] == -inf).all())
    for r in range(4, 8):
        rd, Wd = dI[r::8].double(), W.double()
        _within(gx[r::8], rd @ Wd, rd.abs() @ Wd, 6 * n_out, 2.0 ** -26, "finite rows")


@pytest.mark.parametrize("M", [64, 1600])
def test_input_gradient_follows_dcur(M):
    """Of the stage call's two forms of dL/dI the weight gradient contracts
    dcur_t where the layer has such an operand, and the input gradient dcur,
    whatever the size: a caller may have masked it in between."""
    n_in, n_out = 768, 1000
    d, x, W, b, dI = _layer(M, n_in, n_out, False, 9)
    ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
    saved = torch.zeros(snn.snn_layer_saved_bytes(d), dtype=torch.uint8, device="cuda")
    dcur = torch.empty((M, n_out), device="cuda")
    dt = torch.empty(max(snn.snn_layer_dcur_t_bytes(d), 6 * M * n_out), dtype=torch.uint8,
                     device="cuda")
    cur, ck, _ = snn.saved_parts(d, saved)
    snn.snn_neuron_bwd(d, snn.GRAD_FULL, dI, None, cur, ck, dcur, None, None, ws, dcur_t=dt)
    masked = dcur * (torch.arange(n_out, device="cuda") % 3 == 0)
    out = []
    for t, both in ((dt, True), (None, True), (dt, False)):
        gW, gx = torch.empty_like(W), torch.empty((M, n_in), device="cuda")
        snn.snn_synapse_bwd(d, masked, None, x, W, gW if both else None, gx, ws, dcur_t=t)
        out.append((gW, gx))
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[2][1], out[1][1])
    ref = masked.double() @ W.double()
    _within(out[0][1], ref, masked.double().abs() @ W.double().abs(), 6 * n_out, 2.0 ** -26, "dx")
    rw = (dcur if snn.snn_layer_dcur_t_bytes(d) else masked).double()
    _within(out[0][0], rw.t() @ x.double(), rw.abs().t() @ x.double(), 3 * M, 0.0, "dW")


# parts in turn: one 256 x 256 item per tile; chunks of K folded by a workgroup;
# one wave of 128 x 128 tiles against 256 x 128 ones, with one chunk and several
@pytest.mark.parametrize("M,n_in,n_out", [(12801, 784, 1000), (6401, 1000, 1001), (2013, 1003, 1101),
                                          (1500, 2001, 600), (9000, 1001, 520)])
@pytest.mark.parametrize("bytes_in", [True, False])
def test_currents_in_the_kept_order(M, n_in, n_out, bytes_in):
    """The currents of every plan of the kept order of summation, spikes as
    bytes and as bf16 values, every row and column of the last tiles."""
    d, x, W, b, dI = _layer(M, n_in, n_out, False, M)
    if not bytes_in:
        d.in_dtype = snn.BF16
        x = x.bfloat16()
    ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
    cur = torch.full((M, n_out), float("nan"), device="cuda")
    snn.snn_synapse_fwd(d, x, W, b, cur, None, ws)
    xd, Wd = x.double(), W.double()
    _within(cur, xd @ Wd.t() + b.double(), xd @ Wd.abs().t() + b.double().abs(), 3 * n_in + 1, 0.0,
            "currents")


# Products of spikes with three parts that the joint kernel leaves to 256 x 256
# tiles with the parts in turn.


@pytest.mark.parametrize("M,n_in,n_out", [(9000, 1024, 1001), (8200, 1288, 515), (65544, 264, 270),
                                          # rows in whole 16s: these tiles, then smaller ones
                                          (13376, 1528, 1327), (16640, 2232, 294), (38384, 267, 1001)])
def test_weight_gradient_of_parts_in_turn(M, n_in, n_out):
    """K-contiguous planes: more than 8192 rows, outputs no multiple of 8.  A
    column of x with one spike gives the row of dL/dI there, bit for bit; one
    with many, their sum within the fp32 bound."""
    d, x, W, b, dI = _layer(M, n_in, n_out, False, n_out)
    hot = torch.randint(0, M, (n_in,), device="cuda")
    some = torch.arange(n_in, device="cuda") % 3 != 0
    x[:, some] = 0
    x[hot[some], some.nonzero().flatten()] = 1
    ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
    gW = torch.full((n_out, n_in), float("nan"), device="cuda")
    snn.snn_synapse_bwd(d, dI, None, x, W, gW, None, ws)
    assert torch.equal(gW[:, some], dI[hot[some]].t())
    xd, dd = x.double(), dI.double()
    _within(gW, dd.t() @ xd, dd.abs().t() @ xd, 3 * M, 0.0, "dW")


def test_conv_weight_gradient_of_planes():
    """256 output channels, 64 pooled cells.  Each output channel has its
    gradient in one cell, so its dW is that value where the spikes are, bit for
    bit."""
    NB, Ci, H, Co = 224, 12, 20, 256
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    d = snn.layer_desc(dict(kind="conv", c_in=Ci, h=H, w=H, c_out=Co, neuron="leaky", beta=0.5), 1, NB)
    x = (torch.rand((NB, Ci, H, H), generator=g, device="cuda") < 0.4).to(torch.uint8)
    w = torch.rand((Co, Ci, 5, 5), generator=g, device="cuda")
    arg = torch.randint(0, 4, (NB, Co, 8, 8), generator=g, device="cuda", dtype=torch.uint8)
    dI = torch.zeros((NB, Co, 8, 8), device="cuda")
    nb = torch.randint(0, NB, (Co,), generator=g, device="cuda")
    q = torch.randint(0, 64, (Co,), generator=g, device="cuda")
    co = torch.arange(Co, device="cuda")
    v = torch.randn(Co, generator=g, device="cuda")
    dI.view(NB, Co, 64)[nb, co, q] = v
    a = arg.view(NB, Co, 64)[nb, co, q].long()
    oy, ox = 2 * (q // 8) + a // 2, 2 * (q % 8) + a % 2
    ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
    gW = torch.full_like(w, float("nan"))
    snn.snn_synapse_bwd(d, dI, arg, x, w, gW, None, ws)
    ref = torch.stack([x[nb[c], :, oy[c]:oy[c] + 5, ox[c]:ox[c] + 5].float() * v[c] for c in range(Co)])
    assert torch.equal(gW, ref)


def test_operands_past_two_to_the_31():
    """Spikes of more than 2^31 elements: the currents of the last rows are bit
    for bit those of a call with these rows alone (one chunk of K in both), and
    the weight gradient of small whole numbers is exact."""
    n_in, n_out, M, tail = 8192, 256, (1 << 18) + 520, 1 << 17
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    x = torch.randint(0, 2, (M, n_in), generator=g, device="cuda", dtype=torch.uint8)
    W = torch.rand((n_out, n_in), generator=g, device="cuda") * 2 - 1
    b = torch.rand(n_out, generator=g, device="cuda")
    spec = dict(kind="dense", n_in=n_in, n_out=n_out, neuron="leaky", beta=0.9)
    out = []
    for rows in (M, tail):
        d = snn.layer_desc(spec, 1, rows)
        ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
        cur = torch.full((rows, n_out), float("nan"), device="cuda")
        snn.snn_synapse_fwd(d, x[M - rows:], W, b, cur, None, ws)
        out.append(cur[rows - tail:])
    assert torch.equal(out[0], out[1])
    d = snn.layer_desc(spec, 1, M)
    ws = torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device="cuda")
    dI = torch.randint(-3, 4, (M, n_out), generator=g, device="cuda").float()
    gW = torch.full((n_out, n_in), float("nan"), device="cuda")
    snn.snn_synapse_bwd(d, dI, None, x, W, gW, None, ws)
    ref = torch.zeros((n_out, n_in), device="cuda")
    for r in range(0, M, 1 << 15):  # sums of whole numbers below 2^24
        ref += dI[r:r + (1 << 15)].t() @ x[r:r + (1 << 15)].float()
    assert torch.equal(gW, ref)
