"""Large batches fold the previous rewards in with a kernel of their own ahead
of the step; small ones in the step kernel.  Instances are independent, so a
large batch's instances, run again as a small batch, have to end in the same
state, bit for bit: models, masks, instance words, statistics and theta copies,
and to take the same actions and report the same scores at every step."""
import numpy as np
import pytest
import torch

from gpu_helpers import say
from paper_2508_01744_amd import Tuner

pytestmark = pytest.mark.gpu

RULES = dict(ext_rounds=60, ext_min_n=2, ext_thr=-1.2, hist_after=5, hist_min_n=2, hist_kappa=1.0, hist_min_arms=3,
             cascade_k=3)
SWITCH = dict(ph_delta=0.05, ph_lambda=2.0, ph_window=8, ph_min_rounds=10)
WINDOW = dict(refine_period=7, refine_stride=3, refine_half=10, refine_mature=15, refine_min_n=1)
OPTIONS = {
    "plain": dict(),
    "pruning": dict(prune_rule=1, prune_period=9),
    "rules": dict(prune_rule=15, prune_period=9, heuristics=RULES),
    "switch": dict(prune_rule=1, prune_period=9, exploit=SWITCH),
    "all": dict(prune_rule=15, prune_period=9, heuristics=RULES, exploit=SWITCH, refine=WINDOW),
    "reevaluated": dict(prune_rule=1, prune_period=9, prune_sticky=0, refine=WINDOW),
}


def _split(B, K, d, opts, dump=False):
    """The host rule, restated (tests/test_launch_routes.py holds it against the
    library's launches): enough instances, and a stream past the cache."""
    play = K if "refine" not in opts else min(K, max((K - 1) // 3 + 1, 21))
    each = play * 4 * (d + d * (d + 1) // 2)
    scored = play * 4 * d if "exploit" in opts else each   # (from the round of the first possible switch on)
    wide = scored > (96 if opts.get("prune_rule", 0) & 14 else 32) << 10
    arms_go = "prune_rule" in opts or "refine" in opts or "exploit" in opts
    least = 256 if d != 8 else 512 if dump else (2048 if wide else 512) if arms_go else 1024 if each > 24 << 10 else 512
    return B >= (16384 if d == 32 else 8192) and B * each >= least << 20 and not (dump and each <= 16384)


# (B, K, d): one- and four-wavefront workgroups, ragged last blocks and last
# wavefronts of instances, K past one ballot
SIZES = [(8195, 55, 16), (8192, 130, 16), (33001, 21, 16), (8193, 373, 8), (32769, 373, 8), (70003, 45, 8), (16387, 9, 32),
         (16385, 31, 32)]
CASES = [(*size, name) for size in SIZES for name in sorted(OPTIONS) if _split(*size, OPTIONS[name])]
FEW = 70


@pytest.mark.parametrize("B,K,d,name", CASES)
def test_large_batch_is_its_instances(B, K, d, name):
    opts = OPTIONS[name]
    n, T = FEW, 24
    rows = torch.cat([torch.arange(6), torch.arange(B // 2, B // 2 + 32), torch.arange(B - 32, B)]).cuda()
    say(f"[split] {name} B={B} K={K} d={d}")
    big, few = Tuner(B, K, d, alpha0=0.5, **opts), Tuner(n, K, d, alpha0=0.5, **opts)
    g = torch.Generator(device="cuda").manual_seed(B + K + d)
    sc_big, sc_few = torch.empty(B, 2, K, device="cuda"), torch.empty(n, 2, K, device="cuda")
    r = None
    for t in range(T):
        x = torch.randn(B, d, generator=g, device="cuda")
        x[:, 0] = 1.0
        if t == 6:
            x[B - 1, 1] = float("nan")
        dump = t % 5 == 2
        a = big.step(x, r, scores=sc_big if dump else None)
        b = few.step(x[rows].contiguous(), None if r is None else r[rows].contiguous(), scores=sc_few if dump else None)
        assert torch.equal(a[rows], b), t
        if dump:
            assert torch.equal(sc_big[rows], sc_few), t
        r = torch.randn(B, generator=g, device="cuda") * 0.3 - (0.9 if t < T // 2 else 1.5)
        if t == 9:
            r[0], r[B - 2] = float("inf"), float("nan")
    for step in ("pending", "flushed"):
        if step == "flushed":
            big.flush(r)
            few.flush(r[rows].contiguous())
        u, v = big.view(), few.view()
        for key in ("arms", "mask", "inst", "stats", "theta"):
            if u[key] is not None:
                assert torch.equal(u[key][rows].contiguous().view(torch.uint8), v[key].contiguous().view(torch.uint8)), (step, key)


def _sum(x, waves):
    """[n, K] summed over K in single precision as a workgroup of `waves`
    wavefronts does: each thread its arms in turn, a tree over the 64 lanes of
    a wavefront, then wavefront after wavefront."""
    n, K = x.shape
    p = np.zeros((n, -(-K // (64 * waves)), waves, 64), np.float32)
    p.reshape(n, -1)[:, :K] = x
    p = p.cumsum(1, dtype=np.float32)[:, -1]
    while p.shape[2] > 1:
        p = p[:, :, 0::2] + p[:, :, 1::2]
    return p[:, :, 0].cumsum(1, dtype=np.float32)[:, -1]


def _removed(mean, waves):
    """The arms that rule 4 with kappa = 1 removes, [n, K]."""
    K = np.float32(mean.shape[1])
    dev = mean - (_sum(mean, waves) / K)[:, None]
    sigma = np.sqrt(_sum(dev * dev, waves) / K)
    return sigma[:, None] - (mean.max(1)[:, None] - mean) < 0


@pytest.mark.parametrize("B,K,d", [(8192, 130, 16), (8193, 373, 8)])
def test_reward_rule_at_its_threshold(B, K, d):
    """Rule 4 removes an arm whose mean lies more than sigma below the best: with
    one arm of every instance at that threshold, the last bit of sigma decides,
    and with it the order of the sums.  A batch that takes the separate update
    has to remove what its instances on their own do."""
    n = 4096
    rng = np.random.default_rng(K)
    mean = (rng.standard_normal((n, K)) * 0.1 - 0.9).astype(np.float32)
    best, at = mean.max(1).astype(np.float64), rng.integers(0, K, n)
    at = np.where(mean[np.arange(n), at] == mean.max(1), (at + 1) % K, at)
    for _ in range(30):   # (sigma moves by a fraction of what the one mean does)
        mean[np.arange(n), at] = best - mean.astype(np.float64).std(1)
    differ = (_removed(mean, 1) != _removed(mean, 4)).any(1).mean()
    assert differ > 0.02   # the inputs tell one order from the other
    say(f"[split] rule 4 at its threshold B={B} K={K} d={d}: one wavefront or four differ in {differ:.3f} of the instances")
    opts = dict(prune_rule=4, heuristics=dict(hist_after=1, hist_min_n=2, hist_kappa=1.0, hist_min_arms=3))
    assert _split(B, K, d, opts) and n < 8192
    big, few = Tuner(B, K, d, **opts), Tuner(n, K, d, **opts)
    x = torch.randn(B, d, generator=torch.Generator().manual_seed(K)).cuda()
    big.step(x)
    few.step(x[:n].contiguous())
    rows = torch.arange(B) % n
    for t, m in ((few, mean), (big, mean[rows])):
        t.view()["stats"][..., 0] = 2
        t.view()["stats"][..., 1] = torch.from_numpy(m * np.float32(2)).cuda().view(torch.int32)   # 2 rewards: an exact mean
    r = torch.full((B,), float("nan"), device="cuda")   # (no update: the statistics stay as they are)
    big.step(x, r)
    few.step(x[:n].contiguous(), r[:n].contiguous())
    wrong = (big.view()["mask"][:n] != few.view()["mask"]).any(1).float().mean().item()
    assert wrong == 0.0, f"{wrong:.4f} of the instances"


@pytest.mark.parametrize("name,B,K,d", [("all", 8192, 130, 16), ("switch", 33001, 21, 16), ("rules", 16385, 31, 32)])
def test_a_folded_reward_is_not_folded_again(name, B, K, d):
    """A state buffer as it is between the two launches of a step, the models
    updated and the header marked: a decision or a flush that goes on from it
    ends where the whole step or flush does."""
    opts = dict(alpha0=0.5, **OPTIONS[name])
    g = torch.Generator(device="cuda").manual_seed(B)
    x, r = torch.randn(16, B, d, generator=g, device="cuda"), torch.randn(16, B, generator=g, device="cuda") * 0.3 - 0.9
    t = Tuner(B, K, d, **opts)
    a = t.step(x[0])
    for i in range(1, 15):
        a = t.step(x[i], r[i - 1])
    before = t.state.clone()
    say(f"[split] folded ahead, {name} B={B} K={K} d={d}")

    def adopt(state):
        return Tuner(B, K, d, state=state, adopt=True, **opts)

    flushed = adopt(before.clone())
    flushed.flush(r[14])
    between = before.clone()
    u, v = adopt(between).view(), flushed.view()
    for key in ("arms", "stats", "theta"):
        if u[key] is not None:
            u[key].copy_(v[key])
    between[:256].view(torch.int32)[7] = 2   # the header's pending word
    for scores in (None, torch.empty(B, 2, K, device="cuda")):
        whole, rest = adopt(before.clone()), adopt(between.clone())
        assert rest.view()["pending"] == 1
        assert torch.equal(whole.step(x[15], r[14], scores=scores), rest.step(x[15], r[14], scores=scores))
        assert torch.equal(whole.state, rest.state)
    rest = adopt(between)
    rest.flush(r[14])
    assert torch.equal(rest.state, flushed.state)
