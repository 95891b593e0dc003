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
