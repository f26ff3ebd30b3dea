"""The advantage step and the PPO losses at the lengths where their launches change: one, four and sixteen waves per
sequence, chunks longer than a thread's registers, losses over arrays that are 16-byte aligned and not."""
import numpy as np
import pytest

import paper_2309_00754_amd as H
from oracle import gae_ref, ppo_loss_ref, ppo_rewards_ref
from gpu_helpers import assert_rel, host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq,T,start", [(3, 255, 0), (2, 256, 200), (2, 257, 3), (3, 1025, 700), (2, 2047, 0),
                                           (1, 2048, 2047), (2, 2049, 11), (1, 16384, 100), (1, 16500, 9000)])
def test_advantages_by_length(n_seq, T, start, dev):
    import torch
    say("advantages by length", n_seq, T, start)
    rng = np.random.default_rng(T + start)
    M = n_seq * T
    kl, rew, val = ((s * rng.standard_normal(n)).astype(np.float32) for s, n in ((0.1, M), (1.0, n_seq), (1.0, M)))
    d = [torch.from_numpy(v).to(dev) for v in (kl, rew, val)]
    rewards, adv, ret = (torch.full((M,), float("nan"), device=dev) for _ in range(3))
    H.hydra_ppo_advantages(*d, n_seq, T, adv, ret, rewards, start=start, gamma=0.99, lam=0.95)
    torch.cuda.synchronize()
    e_r = ppo_rewards_ref(kl, rew, n_seq, T, start, 0.02)
    e_a, e_ret = gae_ref(e_r, val, n_seq, T, start, 0.99, 0.95)
    assert_rel(host(rewards), np.asarray(e_r).reshape(-1), "rewards")
    assert_rel(host(adv), np.asarray(e_a).reshape(-1), "advantages")
    assert_rel(host(ret), np.asarray(e_ret).reshape(-1), "returns")


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n_seq,T,start", [(1, 1, 0), (1, 3, 1), (2, 1, 0), (1, 4098, 4096), (1, 4, 1), (1, 4099, 7), (2, 4096, 1000), (5, 1640, 0), (1, 8193, 8192),
                                           (7, 2344, 3)])
def test_losses_by_size_and_alignment(n_seq, T, start, shift, dev):
    import torch
    say("losses", n_seq, T, start, shift)
    rng = np.random.default_rng(T * 3 + start)
    M = n_seq * T
    lp_old = -rng.uniform(0.5, 6.0, M).astype(np.float32)
    lp_new = (lp_old + rng.normal(0, 0.3, M)).astype(np.float32)
    A, V, R = (rng.normal(0, 1, M).astype(np.float32) for _ in range(3))

    def put(v):  # one element past a 16-byte boundary when shifted
        t = torch.empty(M + 1, device=dev)[shift:shift + M]
        t.copy_(torch.from_numpy(v))
        return t

    losses = torch.full((3,), float("nan"), device=dev)
    d_lp, d_v = (put(np.full(M, np.nan, np.float32)) for _ in range(2))
    H.hydra_ppo_loss(*(put(v) for v in (lp_new, lp_old, A, V, R)), n_seq, T, losses, d_lp, d_v, start=start, eps=0.2)
    torch.cuda.synchronize()
    e = ppo_loss_ref(lp_new, lp_old, A, V, R, n_seq, T, start, 0.2)
    got = host(losses)
    for i, k in enumerate(("pg_loss", "v_loss")):
        assert abs(got[i] - e[k]) <= 1e-4 * max(abs(e[k]), 1e-3), (k, got[i], e[k])
    assert abs(got[2] - e["clip_frac"]) <= 2.0 / (n_seq * (T - start))
    assert_rel(host(d_lp), e["d_lp"], "d_lp")
    assert_rel(host(d_v), e["d_v"], "d_v")


def test_odd_token_counts_cost_what_even_ones_do(dev):
    """Tokens left over by groups of four are a few words more: the losses of 46 x 1659 tokens take the time of 46 x 1660."""
    import torch
    say("loss time")

    def us(T):
        M = 46 * T
        x = [torch.randn(M, device=dev) for _ in range(5)]
        losses, d_lp, d_v = torch.empty(3, device=dev), torch.empty(M, device=dev), torch.empty(M, device=dev)
        best = float("inf")
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                H.hydra_ppo_loss(*x, 46, T, losses, d_lp, d_v, start=T // 2)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        return best

    odd, even = us(1659), us(1660)
    assert odd < 1.5 * even, (odd, even)
