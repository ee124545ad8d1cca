"""Timed cases: the calls that programs using this framework spend their time in.

Five kinds of case cover the public entry points:

train  one training step (forward, loss, BPTT backward) of a whole network,
       ``Network.step``, or ``Network.step_fused`` for the small-batch step
       that runs as one launch
layer  one dense layer inside a deeper network, ``snn_layer_fwd`` then
       ``snn_layer_bwd`` with a full upstream gradient and an input gradient
conv   the same for one convolution-and-pool layer
scan   one layer driven by given currents (``SYN_NONE``), forward and backward

The sizes are those of the named workloads (Table I's networks and the
population codes), the ranges around them, and generic ones: deeper and wider
dense layers, ragged widths, a convolution with more channels than Table I's.
Inputs follow the workloads' distributions: Bernoulli rate-coded spikes, rates
uniform per feature, weights and biases U(+-1/sqrt(fan_in)), labels uniform.
"""
import math

import torch
import torch.nn.functional as F

import paper_2211_10725_amd as snn
from paper_2211_10725_amd.workloads import Workload

DEV = "cuda"
SLOPE = 25.0


def _dense(n_in, n_out, neuron="leaky", beta=0.95, alpha=0.0):
    return dict(kind="dense", n_in=n_in, n_out=n_out, neuron=neuron, beta=beta, alpha=alpha,
                thr=1.0)


def _conv(c_in, h, w, c_out, beta=0.5):
    return dict(kind="conv", c_in=c_in, h=h, w=w, c_out=c_out, k=5, neuron="leaky", beta=beta,
                alpha=0.0, thr=1.0)


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def listed():
    return [
        # The smallest batches of Table I's dense net, where one launch per
        # step is the offered way to train.
        dict(name="fused_b8", kind="train", net="dense", sizes="784-1000-10", neuron="leaky",
             T=25, B=8, dtype="f32", loss="ce", pop=1, fused=True),
        # The default dense net at its default batch: a chain of short calls.
        dict(name="train_leaky_b32", kind="train", net="dense", sizes="784-1000-10",
             neuron="leaky", T=25, B=32, dtype="f32", loss="ce", pop=1, fused=False),
        # The current-based net at a training batch: fp32 contractions of
        # spikes, scans and the readout in about equal parts.
        dict(name="train_synaptic_b256", kind="train", net="dense", sizes="784-1000-10",
             neuron="synaptic", T=50, B=256, dtype="f32", loss="ce", pop=1, fused=False),
        # Population code, one time step: short and wide products.
        dict(name="train_pop_b128", kind="train", net="dense", sizes="3072-1000-500",
             neuron="leaky", T=1, B=128, dtype="f32", loss="ce", pop=50, fused=False),
        # Table I's convolutional net.
        dict(name="train_csnn_b128", kind="train", net="conv", sizes="1x28-12-64-10",
             neuron="leaky", T=25, B=128, dtype="f32", loss="ce", pop=1, fused=False),
        # The deeper, wider net in half precision: the largest case.
        dict(name="train_half_b512", kind="train", net="dense", sizes="784-4096-4096-10",
             neuron="leaky", T=100, B=512, dtype="f16", loss="ce", pop=1, fused=False),
        # A hidden layer of a deeper fp32 net, with the gradient to the layer
        # below.
        dict(name="layer_f32", kind="layer", n_in=1000, n_out=1000, neuron="leaky", T=50, B=128,
             dtype="f32", reset="detached"),
        # The same at widths and a batch that no tile divides, with
        # current-based neurons and the reset differentiated.
        dict(name="layer_f32_ragged", kind="layer", n_in=1003, n_out=1101, neuron="synaptic",
             T=33, B=61, dtype="f32", reset="surrogate"),
        # A hidden layer of a half-precision net at an ordinary batch.
        dict(name="layer_f16", kind="layer", n_in=1000, n_out=1000, neuron="leaky", T=100, B=64,
             dtype="f16", reset="detached"),
        # A hidden convolution with more channels than Table I's.
        dict(name="conv_wide", kind="conv", c_in=32, h=14, w=14, c_out=64, T=25, B=64),
        # One wide layer on given currents over a long sequence: scan only.
        dict(name="scan_long", kind="scan", n=8192, neuron="leaky", T=1000, B=64,
             grad="bcast", reset="detached"),
        # A ragged recurrent layer on given currents with a gradient per step.
        dict(name="scan_ragged", kind="scan", n=777, neuron="rleaky", T=101, B=33, grad="full",
             reset="surrogate"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    r = rng.random()
    reset = rng.choice(["detached", "surrogate"])
    if r < 0.2:  # Table I's dense nets around their sizes, one and two hidden layers
        n0 = rng.choice([784, 3072, 784, _log(rng, 100, 1600)])
        h = [_log(rng, 64, 2000) for _ in range(rng.choice([1, 1, 2]))]
        pop = rng.choice([1, 1, 1, 20])
        T = 1 if pop > 1 else rng.randint(5, 60)
        return dict(kind="train", net="dense",
                    sizes="-".join(str(n) for n in [n0] + h + [10 * pop]),
                    neuron=rng.choice(["leaky", "synaptic", "rleaky"]), T=T,
                    B=_log(rng, 4, 400), dtype="f32", loss=rng.choice(["ce", "mse"]), pop=pop,
                    fused=False)
    if r < 0.3:  # small batches in one launch
        return dict(kind="train", net="dense",
                    sizes=f"{8 * rng.randint(12, 130)}-{8 * rng.randint(12, 125)}-10",
                    neuron=rng.choice(["leaky", "synaptic"]), T=rng.randint(4, 28),
                    B=rng.randint(1, 10), dtype="f32", loss="ce", pop=1, fused=True)
    if r < 0.4:  # half-precision nets
        h = _log(rng, 256, 3000)
        return dict(kind="train", net="dense", sizes=f"784-{h}-{h}-10", neuron="leaky",
                    T=rng.randint(10, 100), B=_log(rng, 16, 400), dtype="f16", loss="ce", pop=1,
                    fused=False)
    if r < 0.5:  # convolutional nets on MNIST- and CIFAR-shaped inputs
        c, hw = rng.choice([(1, 28), (3, 32)])
        pop = rng.choice([1, 50])
        return dict(kind="train", net="conv",
                    sizes=f"{c}x{hw}-{rng.choice([8, 12, 16])}-{rng.choice([32, 50, 64])}"
                          f"-{10 * pop}",
                    neuron="leaky", T=1 if pop > 1 else rng.randint(4, 25),
                    B=_log(rng, 8, 128), dtype="f32", loss="ce", pop=pop, fused=False)
    if r < 0.75:  # hidden dense layers, odd widths among them
        return dict(kind="layer", n_in=_log(rng, 65, 3000), n_out=_log(rng, 65, 3000),
                    neuron=rng.choice(["leaky", "synaptic"]), T=rng.randint(2, 100),
                    B=_log(rng, 4, 256), dtype=rng.choice(["f32", "f32", "f16"]), reset=reset)
    if r < 0.85:  # hidden convolutions
        return dict(kind="conv", c_in=rng.randint(8, 48), h=rng.randint(8, 17),
                    w=rng.randint(8, 17), c_out=rng.randint(16, 96), T=rng.randint(2, 25),
                    B=_log(rng, 4, 96))
    return dict(kind="scan", n=_log(rng, 65, 8192),
                neuron=rng.choice(["leaky", "synaptic", "rleaky"]), T=_log(rng, 10, 1000),
                B=_log(rng, 2, 64), grad=rng.choice(["bcast", "full"]), reset=reset)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
_BETA = {"leaky": (0.95, 0.0), "synaptic": (0.8, 0.9), "rleaky": (0.95, 0.0)}


def _layers(case):
    """Layer specs of a train case."""
    if case["net"] == "conv":
        src, c1, c2, out = case["sizes"].split("-")
        c, hw = (int(v) for v in src.split("x"))
        h1 = (hw - 4) // 2
        h2 = (h1 - 4) // 2
        return [_conv(c, hw, hw, int(c1)), _conv(int(c1), h1, h1, int(c2)),
                _dense(int(c2) * h2 * h2, int(out), case["neuron"], 0.5)]
    n = [int(v) for v in case["sizes"].split("-")]
    beta, alpha = _BETA[case["neuron"]]
    if case["dtype"] == "f16":
        beta = 0.9
    return [_dense(a, b, case["neuron"], beta, alpha) for a, b in zip(n, n[1:])]


def _spec(case):
    """Layer spec of a layer, conv or scan case."""
    if case["kind"] == "conv":
        return _conv(case["c_in"], case["h"], case["w"], case["c_out"])
    beta, alpha = _BETA[case["neuron"]]
    if case["kind"] == "layer":
        return _dense(case["n_in"], case["n_out"], case["neuron"], beta, alpha)
    return dict(kind="none", n=case["n"], neuron=case["neuron"], beta=beta, alpha=alpha, thr=1.0)


def _sizes(s):
    """(inputs, outputs) per time step and sample of a layer spec."""
    if s["kind"] == "dense":
        return s["n_in"], s["n_out"]
    if s["kind"] == "none":
        return s["n"], s["n"]
    return (s["c_in"] * s["h"] * s["w"],
            s["c_out"] * ((s["h"] - 4) // 2) * ((s["w"] - 4) // 2))


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * (seed + 1) + stream)
    return g


def _uniform(shape, lo, hi, g):
    return torch.rand(shape, generator=g, device=DEV) * (hi - lo) + lo


def _params(s, half, g):
    """(W, b, v) of a layer spec on the device; fp16 nets get fp16 values."""
    n_out = _sizes(s)[1]
    W = b = v = None
    if s["kind"] != "none":
        if s["kind"] == "dense":
            shape, fan, nb = (s["n_out"], s["n_in"]), s["n_in"], s["n_out"]
        else:
            shape, fan, nb = (s["c_out"], s["c_in"], 5, 5), s["c_in"] * 25, s["c_out"]
        k = 1.0 / math.sqrt(fan)
        W, b = _uniform(shape, -k, k, g), _uniform((nb,), -k, k, g)
        if half:
            W, b = W.half().float(), b.half().float()
    if s["neuron"] == "rleaky":
        v = _uniform((n_out,), -0.5, 0.5, g)
    return W, b, v


def _spikes(T, B, feat, rate_hi, g):
    rate = torch.rand((B, feat), generator=g, device=DEV) * rate_hi
    x = torch.empty((T, B, feat), dtype=torch.uint8, device=DEV)
    for t in range(T):
        x[t] = torch.rand((B, feat), generator=g, device=DEV) < rate
    return x


def _inputs(case, seed):
    """Every array of a case, on the device, from the seed alone."""
    T, B = case["T"], case["B"]
    out = {}
    if case["kind"] == "train":
        layers = _layers(case)
        half = case["dtype"] == "f16"
        out["params"] = [_params(s, half, _gen(seed, 10 + i)) for i, s in enumerate(layers)]
        out["x"] = _spikes(T, B, _sizes(layers[0])[0], 0.5 if half else 1.0, _gen(seed, 1))
        K = _sizes(layers[-1])[1] // case["pop"]
        if case["loss"] == "ce":
            out["labels"] = torch.randint(0, K, (B,), generator=_gen(seed, 2), device=DEV,
                                          dtype=torch.int32)
        else:
            out["targets"] = _uniform((B, K), 0.0, float(T), _gen(seed, 2))
        return out
    s = _spec(case)
    n_in, n_out = _sizes(s)
    out["params"] = [_params(s, case.get("dtype") == "f16", _gen(seed, 10))]
    g = _gen(seed, 1)
    if case["kind"] == "scan":
        out["x"] = torch.empty((T, B, n_in), device=DEV).normal_(0.3, 0.5, generator=g)
        shape = (B, n_out) if case["grad"] == "bcast" else (T, B, n_out)
    else:
        out["x"] = _spikes(T, B, n_in, 1.0, g)
        shape = (T, B, n_out)
    out["g"] = torch.empty(shape, device=DEV).normal_(0.0, 1e-3, generator=_gen(seed, 2))
    return out


# --------------------------------------------------------------------------
# a pass
# --------------------------------------------------------------------------
def prepare(case, seed):
    inp = _inputs(case, seed)
    T, B = case["T"], case["B"]
    if case["kind"] == "train":
        layers = _layers(case)
        wl = Workload("case", T=T, B=B, layers=layers, loss=case["loss"], pop=case["pop"],
                      slope=SLOPE, dtype=case["dtype"])
        params = [tuple(None if p is None else p.cpu().numpy() for p in ps) if ps[2] is not None
                  else tuple(p.cpu().numpy() for p in ps[:2]) for ps in inp["params"]]
        net = snn.Network(wl, params, device=DEV)
        x = inp["x"].view(net.in_shape)
        return dict(net=net, x=x, labels=inp.get("labels"), targets=inp.get("targets"),
                    fused=case["fused"] and net.fdesc is not None)
    s = _spec(case)
    half = case.get("dtype") == "f16"
    reset = snn.RESET_SURROGATE if case.get("reset") == "surrogate" else snn.RESET_DETACHED
    spk_dt = snn.F16 if half else snn.U8
    d = snn.layer_desc(s, T, B, in_dtype=spk_dt, w_dtype=snn.F16 if half else snn.F32,
                       out_dtype=spk_dt, grad_dtype=snn.F16 if half else snn.F32, slope=SLOPE,
                       reset_grad=reset)
    W, b, v = inp["params"][0]
    x = inp["x"].half() if half else inp["x"]

    def f32(*shape):
        return torch.empty(shape, dtype=torch.float32, device=DEV)

    def u8(n):
        return torch.empty(max(n, 256), dtype=torch.uint8, device=DEV)

    st = dict(d=d, x=x, w=W.half() if half else W, b=b, v=v, g=inp["g"],
              gkind=snn.GRAD_BCAST if case.get("grad") == "bcast" else snn.GRAD_FULL,
              spk=torch.empty((T, B, d.n_out), dtype=torch.float16 if half else torch.uint8,
                              device=DEV),
              saved=u8(snn.snn_layer_saved_bytes(d)), counts=f32(B, d.n_out),
              ws=u8(snn.snn_layer_workspace_bytes(d)),
              gw=None if W is None else f32(*W.shape), gb=None if b is None else f32(*b.shape),
              gv=None if v is None else f32(*v.shape), gx=f32(T, B, d.n_in))
    return st


def run(state):
    if "net" in state:
        net = state["net"]
        step = net.step_fused if state["fused"] else net.step
        step(state["x"], labels=state["labels"], targets=state["targets"])
        return {"loss": net.loss[:1], "counts": net.counts, "gW": list(net.gW),
                "gb": list(net.gb), "gv": [v for v in net.gv if v is not None]}
    s = state
    snn.snn_layer_fwd(s["d"], s["x"], s["w"], s["b"], s["v"], s["spk"], s["saved"], s["counts"],
                      s["ws"])
    snn.snn_layer_bwd(s["d"], s["gkind"], s["g"], s["x"], s["w"], s["v"], s["saved"], s["gw"],
                      s["gb"], s["gv"], s["gx"], s["ws"])
    return {"spk": s["spk"], "counts": s["counts"],
            "grads": [s[k] for k in ("gw", "gb", "gv", "gx") if s[k] is not None]}


def work(case):
    T, B = case["T"], case["B"]
    rows = T * B
    if case["kind"] == "train":
        layers = _layers(case)
        half = case["dtype"] == "f16"
        nbytes = rows * _sizes(layers[0])[0] + 8 * B * _sizes(layers[-1])[1]
        flops = 0
        for i, s in enumerate(layers):
            macs, par = _macs(s)
            flops += 2 * rows * macs * (3 if i else 2)
            nbytes += par * ((2 if half else 4) + 4)
        return {"bytes": nbytes, "flops": flops}
    s = _spec(case)
    n_in, n_out = _sizes(s)
    sb = 2 if case.get("dtype") == "f16" else 1  # bytes of a spike
    g = B * n_out if case.get("grad") == "bcast" else rows * n_out
    if case["kind"] == "scan":  # currents, spikes, dL/dI, the gradient and the counts
        return {"bytes": rows * n_in * 8 + rows * n_out + 4 * g + 4 * B * n_out,
                "flops": 20 * rows * n_out}
    macs, par = _macs(s)
    return {"bytes": rows * (n_in * (sb + 4) + n_out * sb) + 4 * g + par * (2 * sb + 4 + 2),
            "flops": 6 * rows * macs}


def _macs(s):
    """(multiply-adds per sample and step, parameters) of a layer spec."""
    n_in, n_out = _sizes(s)
    if s["kind"] == "dense":
        return n_in * n_out, n_in * n_out + n_out
    return n_out * 4 * s["c_in"] * 25, s["c_out"] * (s["c_in"] * 25 + 1)


def tolerance(case):
    """About four times the distance from ``exact`` measured over the listed
    cases and a few dozen drawn ones.  What sets it is the spikes decided
    differently: a membrane within rounding of the threshold (one spike in
    10^6, 10^7 for short sequences) changes that neuron's later steps and
    gradients; without one the fp32 gradients agree to about 1e-5.  fp16 nets
    also round dL/dI to 16 bits."""
    if case["kind"] == "scan":  # measured 7e-4 .. 3.4e-3 (long sequences)
        rel = 1e-2
    elif case.get("dtype") == "f16":  # measured 5e-4 .. 2.6e-3 (nets), 2e-4 (layers)
        rel = 1e-2 if case["kind"] == "train" else 5e-3
    else:  # measured 1e-6 .. 7e-4
        rel = 3e-3
    return {"rel": rel, "differ": 1e-5}


# --------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------
def _windows(x, s):
    """5x5 patches of every conv output some pool window reads, as rows
    [NB * Hp * Wp * 4, c_in * 25]: a pooled cell's four outputs together."""
    hp, wp = (s["h"] - 4) // 2, (s["w"] - 4) // 2
    x = x.view(-1, s["c_in"], s["h"], s["w"])[:, :, :2 * hp + 4, :2 * wp + 4]
    cols = F.unfold(x, 5)  # [NB, c_in * 25, 2 hp * 2 wp]
    nb, k = cols.shape[:2]
    return (cols.view(nb, k, hp, 2, wp, 2).permute(0, 2, 4, 3, 5, 1).reshape(-1, k),
            (nb, hp, wp))


def _synapse(s, x, W, b):
    """Currents [T, B, n_out] and what the backward needs of them."""
    T, B = x.shape[:2]
    if s["kind"] == "none":
        return x, None
    if s["kind"] == "dense":
        return (x.view(T * B, -1) @ W.t() + b).view(T, B, -1), None
    cols, (nb, hp, wp) = _windows(x, s)
    c = (cols @ W.view(s["c_out"], -1).t() + b).view(nb, hp * wp, 4, s["c_out"])
    best, sel = c[:, :, 0], torch.zeros_like(c[:, :, 0], dtype=torch.long)
    for q in range(1, 4):  # the first maximum wins
        up = c[:, :, q] > best
        best, sel = torch.where(up, c[:, :, q], best), torch.where(up, q, sel)
    return best.transpose(1, 2).reshape(T, B, -1), sel


def _synapse_bwd(s, d, sel, x, W, need_x):
    T, B = x.shape[:2]
    if s["kind"] == "dense":
        d2 = d.view(T * B, -1)
        return (d2.t() @ x.view(T * B, -1), d2.sum(0),
                (d2 @ W).view(T, B, -1) if need_x else None)
    cols, (nb, hp, wp) = _windows(x, s)
    co = s["c_out"]
    dp = d.view(nb, co, hp * wp).transpose(1, 2)
    dc = torch.zeros((nb, hp * wp, 4, co), dtype=d.dtype, device=d.device)
    dc.scatter_(2, sel.unsqueeze(2), dp.unsqueeze(2))
    dc = dc.view(-1, co)
    gw = (dc.t() @ cols).view_as(W)
    gx = None
    if need_x:
        dcol = (dc @ W.view(co, -1)).view(nb, hp, wp, 2, 2, -1).permute(0, 5, 1, 3, 2, 4)
        dcol = dcol.reshape(nb, -1, 4 * hp * wp)
        img = F.fold(dcol, (2 * hp + 4, 2 * wp + 4), 5)
        gx = torch.zeros((nb, s["c_in"], s["h"], s["w"]), dtype=d.dtype, device=d.device)
        gx[:, :, :2 * hp + 4, :2 * wp + 4] = img
        gx = gx.view(T, B, -1)
    return gw, dp.sum((0, 1)), gx


def _scan(s, cur, v):
    u = torch.zeros_like(cur[0])
    syn, z = torch.zeros_like(u), torch.zeros_like(u)
    us, zs = torch.empty_like(cur), torch.empty_like(cur)
    jump = -s["thr"] if v is None else v - s["thr"]
    for t in range(cur.shape[0]):
        inp = cur[t]
        if s["neuron"] == "synaptic":
            syn = s["alpha"] * syn + cur[t]
            inp = syn
        u = s["beta"] * u + inp + z * jump
        z = (u > s["thr"]).to(u.dtype)
        us[t], zs[t] = u, z
    return us, zs


def _scan_bwd(s, us, zs, g, v, surrogate):
    """dL/dI [T, B, n] and dL/dv; g [T, B, n] or [B, n] for every step."""
    T = us.shape[0]
    r = s["thr"] if surrogate else 0.0
    d = torch.empty_like(us)
    lam = torch.zeros_like(us[0])
    lami, dv = torch.zeros_like(lam), torch.zeros_like(lam)
    for t in range(T - 1, -1, -1):
        sg = 1.0 / (1.0 + SLOPE * (us[t] - s["thr"]).abs()) ** 2
        gt = g[t] if g.dim() == 3 else g
        dv += lam * zs[t]
        lam = gt * sg + (s["beta"] + ((0.0 if v is None else v) - r) * sg) * lam
        if s["neuron"] == "synaptic":
            lami = lam + s["alpha"] * lami
            d[t] = lami
        else:
            d[t] = lam
    return d, None if v is None else dv.sum(0)


def _f32(v):
    """A scalar as the fp32 value the descriptors carry."""
    return torch.tensor(v, dtype=torch.float32).item()


def exact(case, seed):
    inp = _inputs(case, seed)
    train = case["kind"] == "train"
    layers = _layers(case) if train else [_spec(case)]
    layers = [dict(s, beta=_f32(s["beta"]), alpha=_f32(s["alpha"])) for s in layers]
    params = [tuple(None if p is None else p.double() for p in ps) for ps in inp["params"]]
    surrogate = case.get("reset") == "surrogate"
    kept, h = [], inp["x"].double()
    for s, (W, b, v) in zip(layers, params):
        cur, sel = _synapse(s, h, W, b)
        us, zs = _scan(s, cur, v)
        kept.append((h, sel, us, zs))
        h = zs
    counts = h.sum(0)
    if not train:
        s, (W, b, v) = layers[0], params[0]
        x, sel, us, zs = kept[0]
        d, gv = _scan_bwd(s, us, zs, inp["g"].double(), v, surrogate)
        gw, gb, gx = (None, None, d) if s["kind"] == "none" else _synapse_bwd(s, d, sel, x, W, True)
        return {"spk": zs, "counts": counts,
                "grads": [g for g in (gw, gb, gv, gx) if g is not None]}
    B, P = case["B"], case["pop"]
    c = counts.view(B, -1, P).sum(2)
    if case["loss"] == "ce":
        y = inp["labels"].long()
        lse = torch.logsumexp(c, 1)
        loss = (lse - c.gather(1, y[:, None])[:, 0]).mean()
        gc = torch.softmax(c, 1)
        gc[torch.arange(B, device=DEV), y] -= 1.0
        gc /= B
    else:
        e = c - inp["targets"].double()
        loss, gc = (e * e).mean(), 2.0 * e / e.numel()
    g = gc.repeat_interleave(P, 1)
    gW, gb, gv = [], [], []
    for i in range(len(layers) - 1, -1, -1):
        x, sel, us, zs = kept[i]
        W, b, v = params[i]
        d, dv = _scan_bwd(layers[i], us, zs, g, v, surrogate)
        w_, b_, g = _synapse_bwd(layers[i], d, sel, x, W, i > 0)
        kept[i] = None
        gW.insert(0, w_)
        gb.insert(0, b_)
        if dv is not None:
            gv.insert(0, dv)
    return {"loss": loss.view(1), "counts": counts, "gW": gW, "gb": gb, "gv": gv}
