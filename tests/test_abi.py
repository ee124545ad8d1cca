"""C-ABI checks that need no GPU: the library loads, exports every entry point
include/snn.h declares, and validates arguments on the host (no launches)."""
import ctypes
import os
import re

import pytest

import paper_2211_10725_amd as snn
from tests.conftest import ROOT

HEADER = os.path.join(ROOT, "include", "snn.h")


def _declared():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(snn_[a-z_]+)\s*\(", src)))


def test_header_and_binding_agree():
    assert _declared() == sorted(snn.EXPORTS)


def test_library_exports_every_symbol():
    L = snn.lib()
    for name in _declared():
        assert hasattr(L, name), name
    assert L.snn_abi_version() == snn.ABI_VERSION
    for s in range(8):
        assert isinstance(L.snn_status_str(s), bytes)


def _dense(T=4, B=3, n_in=20, n_out=7):
    return snn.layer_desc(dict(kind="dense", n_in=n_in, n_out=n_out, neuron="leaky", beta=0.9),
                          T, B)


def _fwd(desc, x=16, w=32, bias=None, v=None, spk=48, saved=64, counts=None, ws=None, wsb=0):
    return snn.lib().snn_layer_fwd(ctypes.byref(desc) if desc is not None else None, x, w, bias,
                                   v, spk, saved, counts, ws, wsb, None)


def test_validation_errors_before_launch():
    # fake, aligned, never dereferenced addresses: validation fails first
    d = _dense()
    assert _fwd(None) == 1                                     # NULL desc
    assert _fwd(d, x=None) == 1                                # NULL x
    assert _fwd(d, w=None) == 1                                # dense needs w
    assert _fwd(d, x=17) == 4                                  # misaligned
    bad = d.copy(); bad.T = -1
    assert _fwd(bad) == 2
    bad = d.copy(); bad.neuron = 7
    assert _fwd(bad) == 5
    bad = d.copy(); bad.in_dtype = 9
    assert _fwd(bad) == 3
    bad = d.copy(); bad.flags = 2
    assert _fwd(bad) == 5
    bad = d.copy(); bad.slope = float("nan")
    assert _fwd(bad) == 2
    none = snn.layer_desc(dict(kind="none", n=12, neuron="leaky", beta=0.9), 4, 3)
    bad = none.copy(); bad.n_out = 13
    assert _fwd(bad, w=None) == 2
    conv = snn.layer_desc(dict(kind="conv", c_in=1, h=28, w=28, c_out=12, neuron="leaky",
                               beta=0.5), 4, 3)
    bad = conv.copy(); bad.n_out = 5
    assert _fwd(bad) == 2
    # packed spikes: an output type only, for layers of a multiple of 64 neurons
    bits = d.copy(); bits.out_dtype = snn.SPK_BITS
    assert _fwd(bits) == 2                                      # n_out = 7
    bits = _dense(n_out=128); bits.out_dtype = snn.SPK_BITS
    assert snn.lib().snn_layer_saved_bytes(ctypes.byref(bits)) > 0
    bad = _dense(); bad.in_dtype = snn.SPK_BITS
    assert _fwd(bad) == 3
    # the recurrent neuron (eq. 7) needs its recurrent weights
    rec = _dense(); rec.neuron = snn.RLEAKY
    assert _fwd(rec) == 1
    assert _fwd(rec, v=80 + 4) == 4
    # a recurrent-weight gradient is only defined for the recurrent neuron
    gi = snn.GradIn(snn.GRAD_BCAST, 0, 16)
    need = snn.snn_layer_workspace_bytes(d)
    st = snn.lib().snn_layer_bwd(ctypes.byref(d), ctypes.byref(gi), 32, 48, None, 64, 80, 96,
                                 112, None, 256, need, None)
    assert st == 2
    st = snn.lib().snn_layer_bwd(ctypes.byref(rec), ctypes.byref(gi), 32, 48, None, 64, 80, 96,
                                 112, None, 256, snn.snn_layer_workspace_bytes(rec), None)
    assert st == 1


def test_fold_validation():
    """SNN_GRAD_FOLD arguments are checked on the host.  Every call here stops
    before a launch: a valid fold reaches the misaligned dcur (SNN_ERR_ALIGN)."""
    L = snn.lib()
    d = _dense(T=4, B=3, n_in=20, n_out=100)

    def bwd(gi, desc=d):
        return L.snn_neuron_bwd(ctypes.byref(desc), ctypes.byref(gi), None, 64, 128, 80 + 1,
                                None, None, None, None, None, 0, None)

    F = snn.GRAD_FOLD
    assert bwd(snn.GradIn(F, 10, None, 96, 112, snn.F32, snn.F32)) == 4     # valid up to dcur
    assert bwd(snn.GradIn(F, 16, None, 96, 112, snn.BF16, snn.F16)) == 4
    assert bwd(snn.GradIn(F, 0, None, 96, 112, snn.F32, snn.F32)) == 2      # n_up < 1
    assert bwd(snn.GradIn(F, 17, None, 96, 112, snn.F32, snn.F32)) == 2     # n_up > 16
    assert bwd(snn.GradIn(F, 10, None, None, 112, snn.F32, snn.F32)) == 1   # no dL/dI above
    assert bwd(snn.GradIn(F, 10, None, 96, None, snn.F32, snn.F32)) == 1    # no weights above
    assert bwd(snn.GradIn(F, 10, None, 96, 112, snn.U8, snn.F32)) == 3
    assert bwd(snn.GradIn(F, 10, None, 96, 112, snn.F32, snn.BF16)) == 3
    assert bwd(snn.GradIn(F, 10, None, 96 + 8, 112, snn.F32, snn.F32)) == 4
    # layers narrower than 64 neurons are not folded into
    narrow = _dense(T=4, B=3, n_in=20, n_out=63)
    assert bwd(snn.GradIn(F, 10, None, 96, 112, snn.F32, snn.F32), narrow) == 5
    # the other kinds keep n_up = 0; unknown kinds are rejected
    assert bwd(snn.GradIn(snn.GRAD_FULL, 3, 16)) == 5
    assert bwd(snn.GradIn(snn.GRAD_FULL, 0, 16)) == 4
    assert bwd(snn.GradIn(3, 0, 16)) == 5


def test_loss_validation():
    L = snn.lib()
    assert L.snn_loss(0, 0, 10, 1, 16, 32, None, 48, 64, None, 0, None) == 2   # B = 0
    assert L.snn_loss(0, 4, 10, 1, 16, None, None, 48, 64, None, 0, None) == 1  # CE needs labels
    assert L.snn_loss(1, 4, 10, 1, 16, None, None, 48, 64, None, 0, None) == 1  # MSE needs targets
    assert L.snn_loss(5, 4, 10, 1, 16, 32, None, 48, 64, None, 0, None) == 5
    assert L.snn_loss(0, 4, 10, 0, 16, 32, None, 48, 64, None, 0, None) == 2   # P = 0
    need = L.snn_loss_workspace_bytes(1, 64, 65536)
    assert need > 0
    assert L.snn_loss(1, 64, 65536, 1, 16, None, 32, 48, 64, 256, need - 1, None) == 6
    # cross-entropy keeps one fp64 loss per row for its fixed-order sum
    need = L.snn_loss_workspace_bytes(0, 128, 10)
    assert need >= 128 * 8
    assert L.snn_loss(0, 128, 10, 50, 16, 32, None, 48, 64, 256, need - 1, None) == 6


def test_sizes_queries():
    d = _dense(T=25, B=32, n_in=784, n_out=1000)
    assert snn.snn_layer_saved_bytes(d) >= 25 * 32 * 1000 * 4
    ws = snn.snn_layer_workspace_bytes(d)
    assert ws >= 25 * 32 * 1000 * 4          # holds dL/dI for the backward
    bad = d.copy(); bad.n_in = 0
    assert snn.snn_layer_saved_bytes(bad) == 0
    # the scan-only layer keeps only checkpoints: its currents are its input
    none = snn.layer_desc(dict(kind="none", n=65536, neuron="leaky", beta=0.95), 1000, 64)
    assert snn.snn_layer_saved_bytes(none) == ((1000 - 1) // 16) * 64 * 65536 * 4


def _al(x):
    return (x + 255) // 256 * 256


def test_narrow_weight_gradients_keep_their_kernel():
    """The layout of dL/dI that a weight gradient contracts tells the kernel:
    planes where the parts are staged together.  Outputs of a tile or two over
    very many rows are slower there and keep the transposed operand."""
    for rows, n_in, n_out, planes in [(262144, 64, 64, False), (65536, 256, 64, False),
                                      (189920, 120, 72, False), (16384, 1024, 64, False),
                                      (10715, 5776, 96, True), (61976, 264, 120, True),
                                      (15504, 792, 88, True), (12800, 1000, 1000, True)]:
        d = snn.layer_desc(dict(kind="dense", n_in=n_in, n_out=n_out, neuron="leaky", beta=0.9), 1,
                           rows)
        got = snn.snn_layer_dcur_t_layout(d) == snn.DCUR_T_PLANES
        assert got == planes, (rows, n_in, n_out)
        assert snn.snn_layer_dcur_t_bytes(d) >= 6 * rows * n_out


def test_tall_weight_gradients_keep_their_tiles():
    """A weight gradient over very many rows in whole 16s, of outputs that fill
    256 x 256 tiles badly, is contracted from the spikes' bytes: next to dL/dI,
    its three planes and the transposed bytes there is no room for 16-bit spikes.
    Rows in whole 8s alone have it."""
    for rows, n_in, n_out, widened in [(155600, 992, 263, False), (137728, 1672, 290, False),
                                       (155592, 992, 263, True)]:
        d = snn.layer_desc(dict(kind="dense", n_in=n_in, n_out=n_out, neuron="leaky", beta=0.9), 1,
                           rows)
        room = snn.snn_layer_workspace_bytes(d) - rows * (10 * n_out + n_in)
        assert (room >= 2 * rows * n_in) == widened, (rows, n_in, n_out)


def test_workspace_of_large_layers():
    """Workspaces of 2 GiB and more hold what the layer's calls put there."""
    # a convolution: dL/dI, dC^T fp32 and dx^T fp32 of every window row
    NB, Ci, hw, Co = 300, 32, 60, 300
    d = snn.layer_desc(dict(kind="conv", c_in=Ci, h=hw, w=hw, c_out=Co, neuron="leaky", beta=0.5),
                       1, NB)
    windows = NB * (hw - 4) ** 2
    assert snn.snn_layer_workspace_bytes(d) >= 4 * (NB * d.n_out + Co * windows + 25 * Ci * windows)
    # fp16 weights, more outputs than a bias is staged for: bytes widened to fp16
    for rows in (1 << 17, 1 << 18, 1 << 19):
        d = snn.layer_desc(dict(kind="dense", n_in=8192, n_out=9000, neuron="leaky", beta=0.9), 1,
                           rows, w_dtype=snn.F16, grad_dtype=snn.F16)
        assert snn.snn_layer_workspace_bytes(d) >= 2 * rows * (8192 + 9000)
    # fp32 weights of 3 planes of more than 2 GiB
    d = snn.layer_desc(dict(kind="dense", n_in=184, n_out=2000000, neuron="leaky", beta=0.9), 1, 2048)
    assert snn.snn_layer_workspace_bytes(d) >= 6 * 184 * 2000000


@pytest.mark.parametrize("kind,neuron,T,B", [("dense", "leaky", 25, 32), ("dense", "synaptic", 50, 7),
                                             ("dense", "rleaky", 16, 3), ("dense", "leaky", 17, 3),
                                             ("dense", "leaky", 1, 5), ("conv", "leaky", 25, 4),
                                             ("none", "synaptic", 33, 2), ("none", "leaky", 0, 2)])
def test_saved_layout(kind, neuron, T, B):
    """The saved state's parts as the library lays them out: the currents
    (not for a scan-only layer), a checkpoint after every 16th step but the
    last (u, and i for the current-based neuron), the conv pool selection;
    on 256-byte boundaries, disjoint, inside snn_layer_saved_bytes."""
    if kind == "conv":
        spec = dict(kind="conv", c_in=2, h=12, w=10, c_out=3, neuron=neuron, beta=0.5)
    elif kind == "dense":
        spec = dict(kind="dense", n_in=20, n_out=37, neuron=neuron, beta=0.9, alpha=0.5)
    else:
        spec = dict(kind="none", n=37, neuron=neuron, beta=0.9, alpha=0.5)
    d = snn.layer_desc(spec, T, B)
    lay = snn.snn_layer_saved_layout(d)
    el = T * B * d.n_out
    assert lay.bytes == snn.snn_layer_saved_bytes(d)
    assert lay.ckpt_interval == 16
    assert lay.ckpt_count == (max(T, 1) - 1) // 16
    assert lay.ckpt_planes == (2 if neuron == "synaptic" else 1)
    assert lay.cur_bytes == (0 if kind == "none" else _al(el * 4))
    assert lay.ckpt_bytes == _al(lay.ckpt_planes * lay.ckpt_count * B * d.n_out * 4)
    assert lay.pool_bytes == (_al(el) if kind == "conv" else 0)
    parts = sorted([(lay.cur_offset, lay.cur_bytes), (lay.ckpt_offset, lay.ckpt_bytes),
                    (lay.pool_offset, lay.pool_bytes)])
    end = 0
    for off, nb in parts:
        assert off % 256 == 0 and off >= end
        end = off + nb
    assert end <= lay.bytes
    # errors: no output struct, a bad descriptor
    assert snn.lib().snn_layer_saved_layout(ctypes.byref(d), None) == 1
    bad = d.copy(); bad.T = -1
    out = snn.SavedLayout()
    assert snn.lib().snn_layer_saved_layout(ctypes.byref(bad), ctypes.byref(out)) == 2


def test_workspace_too_small_is_rejected():
    d = _dense(T=25, B=32, n_in=784, n_out=1000)
    gi = snn.GradIn(snn.GRAD_BCAST, 0, 16)
    need = snn.snn_layer_workspace_bytes(d)
    st = snn.lib().snn_layer_bwd(ctypes.byref(d), ctypes.byref(gi), 32, 48, None, 64, 80, 96,
                                 None, None, 256, need - 1, None)
    assert st == 6
    # the recurrent neuron's backward also holds the per-column dL/dv sums
    rec = d.copy(); rec.neuron = snn.RLEAKY
    assert snn.snn_layer_workspace_bytes(rec) >= need + 32 * 1000 * 4


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    monkeypatch.setattr(snn, "_lib", None)
    monkeypatch.setattr(snn, "LIB_PATH", str(tmp_path / "libsnn.so"))
    with pytest.raises(RuntimeError, match="not built"):
        snn.lib()


def test_adamw_validation():
    """Host-side checks of snn_adamw; no call here reaches a launch."""
    L = snn.lib()
    hp = snn.AdamwHparams(1e-3, 0.9, 0.999, 1e-8, 0.0, 1)
    arr = (snn.AdamwTensor * 1)()
    assert L.snn_adamw(arr, 0, hp, None) == 0                     # nothing to do
    assert L.snn_adamw(None, 1, hp, None) == 1
    arr[0] = snn.AdamwTensor(None, None, None, None, None, 0)
    assert L.snn_adamw(arr, 1, hp, None) == 0                     # empty tensor
    arr[0] = snn.AdamwTensor(16, None, 48, 64, None, 8)
    assert L.snn_adamw(arr, 1, hp, None) == 1                     # missing grad
    arr[0] = snn.AdamwTensor(16, 32, 48, 72, None, 8)
    assert L.snn_adamw(arr, 1, hp, None) == 4                     # misaligned moment
    for bad in (snn.AdamwHparams(1e-3, 1.0, 0.999, 1e-8, 0.0, 1),
                snn.AdamwHparams(-1.0, 0.9, 0.999, 1e-8, 0.0, 1),
                snn.AdamwHparams(1e-3, 0.9, 0.999, 1e-8, 0.0, 0),
                snn.AdamwHparams(float("nan"), 0.9, 0.999, 1e-8, 0.0, 1)):
        assert L.snn_adamw(arr, 1, bad, None) == 2
