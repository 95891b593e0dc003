"""The kernels that write a fresh state buffer and that materialise the models,
at sizes around the edges of their work split: part-filled blocks of records,
one arm, several workgroups per instance and several instances per workgroup."""
import numpy as np
import pytest
import torch

from gpu_helpers import say
from paper_2508_01744_amd import Tuner

from test_gpu_layout import _decode

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 8), (1, 1024, 32), (3, 9, 8), (5, 64, 8), (7, 33, 16), (2, 130, 16), (300, 4, 16), (9, 31, 32)]


@pytest.mark.parametrize("opts", [dict(), dict(prune_rule=15, exploit=dict(ph_window=5), heuristics=dict(
    ext_min_n=1, hist_min_n=1, hist_min_arms=1)), dict(refine=dict(refine_period=5, refine_stride=3, refine_half=2,
                                                                   refine_min_n=1))])
@pytest.mark.parametrize("B,K,d", SIZES)
def test_fresh_state_is_written_whole(B, K, d, opts):
    """Whatever the buffer held, a fresh state is the same in every byte and is
    what the layout documents."""
    lam = 2.0
    first = Tuner(B, K, d, lam=lam, **opts)
    state = torch.full((first.nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
    t = Tuner(B, K, d, lam=lam, state=state, **opts)
    say(f"[init] B={B} K={K} d={d} {t.nbytes} bytes")
    assert torch.equal(first.state, state)
    v = t.view()
    arms = v["arms"].cpu().numpy()
    tf = (arms.shape[2] // (64 // d) - (d // 2) * (d // 4)) * 4 // (d // 2)
    theta, S = _decode(arms, K, d, tf)
    diag = np.float32(1.0 / np.sqrt(lam))
    assert not theta.any()
    assert np.array_equal(S, np.broadcast_to(np.eye(d, dtype=np.float32) * diag, S.shape))
    assert np.count_nonzero(arms) == B * K * d          # no other float of the records is set
    mask = v["mask"].cpu().numpy().view(np.uint32)
    bits = (mask[:, :, None] >> np.arange(32, dtype=np.uint32)) & 1
    assert np.array_equal(bits.reshape(B, -1).astype(bool), np.broadcast_to(np.arange(bits[0].size) < K, (B, bits[0].size)))
    stride = opts.get("refine", {}).get("refine_stride", 1)
    inst = v["inst"].cpu().numpy()
    want = np.zeros(inst.shape[1], np.int32)
    want[[0, 3]] = -1
    want[1] = (K - 1) // stride + 1
    want[11] = np.float32(np.inf).view(np.int32)
    want[13:15] = K - 1, stride
    assert np.array_equal(inst, np.broadcast_to(want, inst.shape))
    assert not v["stats"].any()
    assert v["theta"] is None or not v["theta"].any()
    # outside the header and the regions above, zeros
    nonzero = np.count_nonzero(state.cpu().numpy()[256:])
    regions = sum(np.count_nonzero(np.ascontiguousarray(v[k].cpu().numpy()).view(np.uint8)) for k in ("arms", "mask", "inst"))
    assert nonzero == regions


def _random_models(t, seed):
    """Random records in t's buffer; returns theta and S as the layout decodes them."""
    v = t.view()
    g = torch.Generator(device="cuda").manual_seed(seed)
    keep = v["arms"] != 0                                        # the diagonal
    tf = (v["arms"].shape[2] // (64 // t.d) - (t.d // 2) * (t.d // 4)) * 4 // (t.d // 2)
    theta1, S1 = _decode(torch.ones_like(v["arms"]).cpu().numpy(), t.K, t.d, tf)
    v["arms"].normal_(generator=g)
    v["arms"].add_(keep * 1.5)
    theta, S = _decode(v["arms"].cpu().numpy(), t.K, t.d, tf)
    assert theta1.all() and np.count_nonzero(S1) == S1.size // t.d * (t.d + 1) // 2
    return theta, S


@pytest.mark.parametrize("prune", [0, 1])
@pytest.mark.parametrize("B,K,d", SIZES + [(4, 40, 16), (17, 8, 32), (1, 64, 8)])
def test_export_is_the_records_product(B, K, d, prune):
    """theta as stored; each entry of S S^T within the bound of a sum of up to
    d fused products in single precision.  Outputs at any float's address."""
    t = Tuner(B, K, d, prune_rule=prune)
    theta, S = _random_models(t, 17 * B + K)
    th, ai = t.export(theta=True, ainv=True)
    say(f"[export] B={B} K={K} d={d}")
    assert np.array_equal(theta, th.cpu().numpy())
    S = S.astype(np.float64)
    ref, mag = S @ S.swapaxes(2, 3), np.abs(S) @ np.abs(S).swapaxes(2, 3)
    assert (np.abs(ai.cpu().numpy() - ref) <= (d + 1) * 2.0 ** -24 * mag).all()
    from paper_2508_01744_amd import _lib as L
    th1, ai1 = (torch.full((x.numel() + 2,), 7.0, device="cuda") for x in (th, ai))
    L.check("agft_export", L.agft_export(t.h, th1.data_ptr() + 4, ai1.data_ptr() + 4))
    for whole, want in ((th1, th), (ai1, ai)):
        assert torch.equal(whole[1:-1], want.reshape(-1)) and whole[0] == 7.0 and whole[-1] == 7.0


def test_buffers_past_one_row_of_workgroups():
    """76 GB of models (more than 2^32 chunks): set up, and theta exported, to
    the last instance, in launches of more than one row of workgroups."""
    B, K, d = 33001, 1021, 32   # 1.005 rows of the export's workgroups, 2.2 of the set-up's
    few = Tuner(3, K, d)
    t = Tuner(B, K, d)
    say(f"[rows] {t.nbytes / 1e9:.1f} GB")
    assert B * ((K + 1) // 2) > 2 << 23   # two blocks of two arms per workgroup
    u, v = t.view(), few.view()
    for key in ("arms", "mask", "inst"):
        for at in (0, B // 2, B - 3):
            assert torch.equal(u[key][at:at + 3], v[key]), (key, at)
    u["arms"][B - 3:].normal_(generator=torch.Generator(device="cuda").manual_seed(3))
    v["arms"].copy_(u["arms"][B - 3:])
    assert torch.equal(t.export(theta=True, ainv=False)[0][B - 3:], few.export(theta=True, ainv=False)[0])


def test_export_keeps_infinities_to_their_entries():
    """An infinite factor element reaches the products that hold it and no other."""
    B, K, d = 3, 9, 16
    t = Tuner(B, K, d)
    _random_models(t, 5)
    v = t.view()
    v["arms"][1, 1, 0, 0] = float("inf")     # S_00 of arm 4: A^-1_00 alone
    _, ai = t.export(theta=False, ainv=True)
    bad = ~torch.isfinite(ai)
    assert bad.nonzero().tolist() == [[1, 4, 0, 0]]
