"""Products from bf16 parts, bit for bit: a lost part, a wrong plane or another
order of summation is far inside the bounds of sums of many terms, so these
products have one term, or one per 16 values of K in an order that plain fp32
additions retrace.  Sizes on either side of the rules that choose between the
kernels; each kernel has to give the same bits."""
import numpy as np
import pytest

import paper_2211_10725_amd as snn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda"
# rows, n_in, n_out: parts staged together (wide, ragged, more than 8192 rows, one
# tile row), parts in turn, the 16-bit and fp32 kernels, few rows
SIZES = [(6401, 1000, 1001), (2013, 1003, 1101), (12801, 784, 1000), (9001, 1000, 520),
         (10715, 578, 96), (3000, 600, 600), (300, 2048, 2056), (64, 2056, 2048),
         (16384, 64, 1024), (128, 1000, 500), (800, 784, 1000), (1001, 300, 72)]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _desc(M, n_in, n_out):
    return snn.layer_desc(dict(kind="dense", n_in=n_in, n_out=n_out, neuron="leaky", beta=0.9), 1, M)


def _ws(d):
    return torch.empty(snn.snn_layer_workspace_bytes(d) + 256, dtype=torch.uint8, device=DEV)


def _full_parts(shape, g):
    """Values with 24 significant bits, so that all three parts count."""
    return (torch.rand(shape, generator=g, device=DEV) + 0.5) * \
        (torch.randint(0, 2, shape, generator=g, device=DEV) * 2.0 - 1.0)


@pytest.mark.parametrize("M,n_in,n_out", SIZES)
def test_products_of_one_term(M, n_in, n_out):
    """One spike a row: the currents are the weights of that input.  One spike a
    column: the weight gradient is the row of dL/dI there.  Both exactly.  One
    value of dL/dI a row: the input gradient is its product with the weights,
    within the roundings of six part products and 2^-26 of each left out."""
    g = _gen(M + n_in)
    d = _desc(M, n_in, n_out)
    W, dI = _full_parts((n_out, n_in), g), _full_parts((M, n_out), g)
    rows, cols = torch.arange(M, device=DEV), torch.arange(n_in, device=DEV)
    ws = _ws(d)
    hot = torch.randint(0, n_in, (M,), generator=g, device=DEV)
    x = torch.zeros((M, n_in), dtype=torch.uint8, device=DEV)
    x[rows, hot] = 1
    cur = torch.full((M, n_out), float("nan"), device=DEV)
    snn.snn_synapse_fwd(d, x, W, None, cur, None, ws)
    assert torch.equal(cur, W.t()[hot])
    hot = torch.randint(0, M, (n_in,), generator=g, device=DEV)
    x.zero_()
    x[hot, cols] = 1
    gW = torch.full((n_out, n_in), float("nan"), device=DEV)
    snn.snn_synapse_bwd(d, dI, None, x, W, gW, None, ws)
    assert torch.equal(gW, dI[hot].t())
    hot = torch.randint(0, n_out, (M,), generator=g, device=DEV)
    one = torch.zeros_like(dI)
    one[rows, hot] = dI[rows, hot]
    gx = torch.full((M, n_in), float("nan"), device=DEV)
    snn.snn_synapse_bwd(d, one, None, x, W, None, gx, ws)
    ref = dI[rows, hot].double()[:, None] * W[hot].double()
    assert bool(((gx.double() - ref).abs() <= 6 * 2.0 ** -24 * ref.abs()).all())


@pytest.mark.parametrize("exp", [-100, -112, -124])
def test_input_gradient_of_tiny_values(exp):
    """dL/dI so small that its low parts are below bf16's least value: each value
    is taken with an error of at most 2^-134."""
    M, n_in, n_out = 1600, 768, 1000
    g = _gen(-exp)
    d = _desc(M, n_in, n_out)
    W = _full_parts((n_out, n_in), g)
    rows = torch.arange(M, device=DEV)
    hot = torch.randint(0, n_out, (M,), generator=g, device=DEV)
    v = (_full_parts((M,), g).double() * 2.0 ** exp).float()
    one = torch.zeros((M, n_out), device=DEV)
    one[rows, hot] = v
    gx = torch.full((M, n_in), float("nan"), device=DEV)
    snn.snn_synapse_bwd(d, one, None, None, W, None, gx, _ws(d))
    ref = v.double()[:, None] * W[hot].double()
    # (and six products rounded to fp32's least value)
    bound = 6 * 2.0 ** -24 * ref.abs() + 2.0 ** -134 * W[hot].double().abs() + 6 * 2.0 ** -149
    assert bool(((gx.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("M,n_in,n_out", [(6400, 1000, 1000), (1600, 768, 1000), (10715, 578, 96)])
def test_layer_gradients_of_one_term(M, n_in, n_out):
    """The same through the layer call, whose scan writes the parts itself where
    both gradients contract them: gradients of one time step of neurons at their
    threshold (surrogate 1) are dL/dz itself."""
    g = _gen(M)
    d = _desc(M, n_in, n_out)
    W, up = _full_parts((n_out, n_in), g), _full_parts((M, n_out), g)
    saved = torch.zeros(snn.snn_layer_saved_bytes(d), dtype=torch.uint8, device=DEV)
    snn.saved_parts(d, saved)[0].fill_(1.0)
    x = torch.zeros((M, n_in), dtype=torch.uint8, device=DEV)
    hot = torch.randint(0, M, (n_in,), generator=g, device=DEV)
    x[hot, torch.arange(n_in, device=DEV)] = 1
    gW = torch.full((n_out, n_in), float("nan"), device=DEV)
    gx = torch.full((M, n_in), float("nan"), device=DEV)
    ws = _ws(d)
    snn.snn_layer_bwd(d, snn.GRAD_FULL, up, x, W, None, saved, gW, None, None, gx, ws)
    assert torch.equal(gW, up[hot].t())
    rows = torch.arange(M, device=DEV)
    hot = torch.randint(0, n_out, (M,), generator=g, device=DEV)
    one = torch.zeros_like(up)
    one[rows, hot] = up[rows, hot]
    snn.snn_layer_bwd(d, snn.GRAD_FULL, one, x, W, None, saved, gW, None, None, gx, ws)
    ref = up[rows, hot].double()[:, None] * W[hot].double()
    assert bool(((gx.double() - ref).abs() <= 6 * 2.0 ** -24 * ref.abs()).all())


# images, channels in, height, width, channels out: the kernels for wider layers
# (odd sizes, one and two halves, 1 .. 36 pooled cells), and their neighbours
@pytest.mark.parametrize("NB,Ci,H,W,Co", [(40, 32, 14, 14, 64), (33, 20, 12, 12, 65), (64, 6, 17, 16, 64),
                                          (70, 48, 15, 14, 96), (40, 13, 7, 8, 40), (12, 8, 20, 20, 24),
                                          (120, 60, 7, 7, 70), (16, 5, 16, 16, 31)])
def test_conv_gradients_of_one_term(NB, Ci, H, W, Co):
    """dL/dI in one cell of each output channel: dW is its value where the spikes
    are, exactly.  dL/dI in one cell of one channel of each image: dx is its
    product with the channel's weights over the cell's window."""
    g = _gen(NB + Ci)
    d = snn.layer_desc(dict(kind="conv", c_in=Ci, h=H, w=W, c_out=Co, neuron="leaky", beta=0.5), 1, NB)
    Hp, Wp = (H - 4) // 2, (W - 4) // 2
    x = (torch.rand((NB, Ci, H, W), generator=g, device=DEV) < 0.4).to(torch.uint8)
    w = _full_parts((Co, Ci, 5, 5), g)
    arg = torch.randint(0, 4, (NB, Co, Hp, Wp), generator=g, device=DEV, dtype=torch.uint8)

    def corner(nb, co, q):
        a = arg.view(NB, Co, -1)[nb, co, q].long()
        return 2 * (q // Wp) + a // 2, 2 * (q % Wp) + a % 2

    ws = _ws(d)
    co = torch.arange(Co, device=DEV)
    nb = torch.randint(0, NB, (Co,), generator=g, device=DEV)
    q = torch.randint(0, Hp * Wp, (Co,), generator=g, device=DEV)
    v = _full_parts((Co,), g)
    dI = torch.zeros((NB, Co, Hp, Wp), device=DEV)
    dI.view(NB, Co, -1)[nb, co, q] = v
    gW = torch.full_like(w, float("nan"))
    snn.snn_synapse_bwd(d, dI, arg, x, w, gW, None, ws)
    oy, ox = corner(nb, co, q)
    ref = torch.stack([x[nb[c], :, oy[c]:oy[c] + 5, ox[c]:ox[c] + 5].float() * v[c] for c in range(Co)])
    assert torch.equal(gW, ref)

    nb = torch.arange(NB, device=DEV)
    co = torch.randint(0, Co, (NB,), generator=g, device=DEV)
    q = torch.randint(0, Hp * Wp, (NB,), generator=g, device=DEV)
    v = _full_parts((NB,), g)
    dI.zero_()
    dI.view(NB, Co, -1)[nb, co, q] = v
    gx = torch.full((NB, Ci, H, W), float("nan"), device=DEV)
    snn.snn_synapse_bwd(d, dI, arg, x, w, None, gx, ws)
    oy, ox = corner(nb, co, q)
    ref = torch.zeros((NB, Ci, H, W), dtype=torch.float64, device=DEV)
    for b in range(NB):
        ref[b, :, oy[b]:oy[b] + 5, ox[b]:ox[b] + 5] = v[b].double() * w[co[b]].double()
    assert bool(((gx.double() - ref).abs() <= 6 * 2.0 ** -24 * ref.abs()).all())


# ---- the order in which currents are summed ----------------------------------
def _order(M, N, K, half=False):
    """(chunk of K, parts in turn over each chunk) of spikes against fp32 weights:
    256 x 256 tiles with the parts in turn where they fill the device, else the
    16-bit kernel's split of K, from the workgroups of its four tile shapes that
    a compute unit holds.  fp16 operands likewise, with one part."""
    least, passes = (2 ** 30, 1) if half else (2 ** 32, 3)
    if K % 8 == 0 and K >= 256 and M >= 256 and N >= 256 and M * N * K >= least:
        tiles, nk = -(-M // 256) * -(-N // 256), -(-K // 64)
        S = max(1, min(256 // tiles, passes * nk // 16, 64)) if tiles < 256 else 1
        chunk = -(-nk // S) * 64
        if half or tiles * -(-K // chunk) >= 192:
            return chunk, not half
    shapes = (((128, 128), 1.0, 2), ((128, 64), 1.3, 2), ((256, 128), 1.2, 1), ((128, 256), 1.2, 1)) \
        if half else (((128, 128), 1.0, 3), ((128, 64), 1.6, 5), ((256, 128), 0.6, 2))
    kt, best = 64 if half else 32, None
    for (bm, bn), cost, occ in shapes:
        tiles, ks = -(-M // bm) * -(-N // bn), -(-K // 32)
        slots, S = 256 * occ, 1
        if tiles < slots:
            most = max(1, min(-(-2048 // tiles), max(1, ks // 4), 256 if M * N <= 65536 else 64))
            S = max(1, min(slots // tiles, most))
        chunk = -(-(-(-K // kt)) // S) * kt
        splits = -(-K // chunk)
        c = -(-tiles * splits // slots) * bm * bn * chunk * float(np.float32(cost))
        if splits > 1:
            c += splits * M * N * 64.0 / 256
        if best is None or c < best[0]:
            best = (c, chunk)
    return best[1], False


def _parts(W):
    hi = W.bfloat16().float()
    mid = (W - hi).bfloat16().float()
    return [W - hi - mid, mid, hi]  # smallest first


# in turn with one chunk and two; step by step with one chunk and several, on the
# joint kernel and on the 16-bit kernel
@pytest.mark.parametrize("M,n_in,n_out", [(12801, 784, 1000), (6401, 1000, 1001), (8000, 1000, 1000),
                                          (2013, 1003, 1101), (1500, 2001, 600), (9000, 1001, 520),
                                          (3000, 600, 600), (1024, 1536, 768), (640, 1000, 500)])
@pytest.mark.parametrize("kind", ["bytes", "bf16", "half"])
def test_order_of_summation_of_currents(M, n_in, n_out, kind):
    """At most one spike per 16 inputs, so that every matrix instruction adds one
    product per output: the currents retrace, bit for bit, fp32 additions in the
    order of the chunks of K, the steps of 16 and the parts, whatever kernel
    runs the size.  A spike at the threshold turns with the last bit."""
    chunk, turn = _order(M, n_out, n_in, kind == "half")
    if -(-n_in // chunk) >= 16:
        pytest.skip("the wide reduction adds quarters")
    g = _gen(M + n_out)
    steps = -(-n_in // 16)
    at = torch.randint(0, 16, (M, steps), generator=g, device=DEV) + 16 * torch.arange(steps, device=DEV)
    on = (torch.rand((M, steps), generator=g, device=DEV) < 0.7) & (at < n_in)
    at = at.clamp(max=n_in - 1)
    x = torch.zeros((M, n_in), dtype=torch.uint8, device=DEV)
    x[torch.arange(M, device=DEV)[:, None].expand_as(at)[on], at[on]] = 1
    W = _full_parts((n_out, n_in), g)
    d = _desc(M, n_in, n_out)
    if kind == "bf16":
        if M * n_in * n_out < 2 ** 30:
            pytest.skip("bf16 spikes run on the fp32 matrix cores there")
        d.in_dtype = snn.BF16
        x = x.bfloat16()
    elif kind == "half":
        # (of many magnitudes, so that the sums round)
        W = (W * 2.0 ** -torch.randint(0, 13, W.shape, generator=g, device=DEV)).half()
        d.in_dtype = d.w_dtype = d.grad_dtype = snn.F16
        x = x.half()
    cur = torch.full((M, n_out), float("nan"), device=DEV)
    snn.snn_synapse_fwd(d, x, W, None, cur, None, _ws(d))
    rows = torch.cat([torch.randint(0, M, (62,), generator=g, device=DEV),
                      torch.tensor([0, M - 1], device=DEV)])
    at, on = at[rows], on[rows].float()
    parts = [W.float()] if kind == "half" else _parts(W)
    terms = [[p.t()[at[:, s]] * on[:, s:s + 1] for p in parts] for s in range(steps)]
    total = None
    for c0 in range(0, n_in, chunk):
        acc = torch.zeros((len(rows), n_out), device=DEV)
        span = range(c0 // 16, min(steps, (c0 + chunk) // 16))
        for s, p in ([(s, p) for p in range(len(parts)) for s in span] if turn else
                     [(s, p) for s in span for p in range(len(parts))]):
            acc = acc + terms[s][p]
        total = acc if total is None else total + acc
    assert torch.equal(cur[rows], total)
