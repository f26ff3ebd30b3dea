"""The scoring GEMM's three row tiles (64, 128 and 256 rows): their edges against the float64 oracle, and equal bits where
the one-input and the two-input pass of the same rows run on different tiles."""
import pytest

import paper_2309_00754_amd as H
import workloads as WL
from oracle import score_head_ref
from gpu_helpers import assert_abs, assert_rel, dev_bf16, host, say

pytestmark = pytest.mark.gpu

KEYS = ("lp_on", "lp_off", "kl", "lse_on", "lse_off")


def _score(s, dev, two):
    import torch
    A, B = (dev_bf16(s.A, dev), dev_bf16(s.B, dev)) if s.r else (None, None)
    h, W = dev_bf16(s.h, dev), dev_bf16(s.W_lm, dev)
    out = {k: torch.full((s.M,), float("nan"), device=dev) for k in KEYS}
    reward = torch.full((s.n_seq,), float("nan"), device=dev)
    args = (W, A, B, s.s, torch.from_numpy(s.ids).to(dev), dev_bf16(s.w_rm, dev), s.n_seq, s.seq_len, out["lp_on"],
            out["lp_off"], out["kl"])
    kw = dict(reward=reward, lse_on=out["lse_on"], lse_off=out["lse_off"])
    if two:
        H.hydra_score_two_input(h, h, *args, **kw)
    else:
        H.hydra_score(h, *args, **kw)
    torch.cuda.synchronize()
    return out, reward


# rows, K and V by the tile that the size model picks (one input); K of 8: shorter than a slab; 200: a remainder of
# both slab widths; r of 16 fills half a 64-wide LoRA slab
@pytest.mark.parametrize("n_seq,seq_len,K,V,r", [
    (1, 1, 8, 1, 0), (1, 63, 200, 257, 16), (2, 65, 64, 512, 128), (3, 43, 1032, 3000, 8),    # 64 rows
    (1, 100, 200, 33000, 16), (2, 64, 512, 33001, 64), (1, 130, 72, 22016, 100),              # 128 rows
    (1, 200, 72, 50000, 16), (1, 257, 136, 30000, 0), (4, 128, 392, 12345, 128),              # 256 rows
])
def test_score_tiles(n_seq, seq_len, K, V, r, dev):
    import torch
    say("score tile", n_seq, seq_len, K, V, r)
    s = WL.gen_score_head(8100 + n_seq * seq_len + K + V + r, n_seq, seq_len, K, V, r)
    one, rew1 = _score(s, dev, False)
    two, rew2 = _score(s, dev, True)
    e = score_head_ref(s.h, s.W_lm, s.A, s.B, s.s, s.ids, s.w_rm, s.n_seq, s.seq_len)
    for k in KEYS:
        assert_abs(host(one[k]), e[k], k)
        assert torch.equal(one[k], two[k]), k
    assert_rel(host(rew1), e["reward"], "reward")
    assert torch.equal(rew1, rew2)
    if r == 0:
        assert torch.equal(one["lp_on"], one["lp_off"])


@pytest.mark.parametrize("M,two", [(40, False), (130, False), (520, False), (40, True)])
def test_nan_logits_of_a_part_of_the_vocabulary_reach_every_row(M, two, dev):
    """NaN in one block of 32 or 64 vocabulary rows: log-sum-exp and log-probabilities of every token are NaN, on every
    tile, as with NaN anywhere else."""
    import torch
    say("score NaN", M, two)
    V, K = 520, 64
    for lo, hi in ((64, 128), (448, 520), (100, 101), (0, 64)):
        s = WL.gen_score_head(8300 + M, 1, M, K, V, 16)
        s.ids[:] = 300
        W = dev_bf16(s.W_lm, dev).view(torch.bfloat16).clone()
        W[lo:hi] = float("nan")
        A, B, h = (dev_bf16(v, dev) for v in (s.A, s.B, s.h))
        out = {k: torch.zeros(M, device=dev) for k in KEYS}
        args = (W, A, B, s.s, torch.from_numpy(s.ids).to(dev), None, 1, M, out["lp_on"], out["lp_off"], out["kl"])
        kw = dict(lse_on=out["lse_on"], lse_off=out["lse_off"])
        if two:
            H.hydra_score_two_input(h, h, *args, **kw)
        else:
            H.hydra_score(h, *args, **kw)
        torch.cuda.synchronize()
        for k in KEYS:
            assert torch.isnan(out[k]).all(), (k, lo, hi)


def test_tile_counts_of_any_remainder_keep_the_l2_order(dev):
    """500 tiles (no multiple of the eight XCDs) take the time of 496: each XCD walks neighbouring tiles either way."""
    import torch
    say("score tile order")

    def us(V):
        M, K, r = 400, 4096, 16
        h, ha, W, A, B = (torch.randn(n, k, device=dev).to(torch.bfloat16) for n, k in ((M, K), (M, K), (V, K), (r, K), (V, r)))
        tok = torch.zeros(M, dtype=torch.int32, device=dev)
        out = [torch.empty(M, device=dev) for _ in range(3)]
        ws = torch.empty(H.hydra_score_workspace_bytes(M, V), dtype=torch.uint8, device=dev)
        best = float("inf")
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                H.hydra_score_two_input(ha, h, W, A, B, 1.0, tok, None, 1, M, *out, workspace=ws)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 250)
        return best

    any_count, by_eight = us(32000), us(31744)
    assert any_count < 1.15 * by_eight, (any_count, by_eight)


def test_more_tiles_than_one_dispatch_counts(dev):
    """2 x 2048 x 1025 tiles: more than 2^22, so that the grid takes a second dimension with surplus workgroups.  Every
    1021st row, and the last ones, against float64."""
    import torch
    say("score, split grid")
    M, V, K = 2048 * 256, 1025 * 256 - 7, 8
    g = torch.Generator(device=dev).manual_seed(8400)
    h, ha = (torch.randn(M, K, generator=g, device=dev).to(torch.bfloat16) for _ in range(2))
    W = torch.randn(V, K, generator=g, device=dev).to(torch.bfloat16)
    tok = torch.randint(0, V, (M,), generator=g, device=dev, dtype=torch.int32)
    out = [torch.full((M,), float("nan"), device=dev) for _ in range(3)]
    H.hydra_score_two_input(ha, h, W, None, None, 1.0, tok, None, 1, M, *out)
    torch.cuda.synchronize()
    rows = torch.cat([torch.arange(0, M, 1021), torch.arange(M - 300, M)]).to(dev)
    want = []
    for x in (ha, h):
        lp = []
        for r in rows.split(64):
            z = x[r].double() @ W.double().t()
            lp.append(z.gather(1, tok[r].long()[:, None])[:, 0] - torch.logsumexp(z, 1))
        want.append(torch.cat(lp).cpu().numpy())
    for got, e, k in zip(out, (want[0], want[1], want[0] - want[1]), ("lp_on", "lp_off", "kl")):
        assert torch.isfinite(got).all()
        assert_abs(host(got[rows]), e, k)
