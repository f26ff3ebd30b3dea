"""The backward's two pre-pass jobs at the sizes where their plan changes: one launch or partial sums, 64 x 64 or 128 x
128 tiles, K chunks that end ragged in the longer and in the shorter job.  Each output alone keeps the full call's bits
(the plan looks at both jobs whichever run).  Tolerances: the arithmetic bound of the other backward tests."""
import numpy as np
import pytest

import paper_2309_00754_amd as H
import workloads as WL
from oracle import lora_linear_backward_ref, lora_linear_ref, score_head_ref
from gpu_helpers import assert_abs, assert_rel, dev_bf16, host, say
from test_gpu_backward import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,r", [
    (2048, 72, 40, 16), (2049, 72, 40, 16),    # the last rows of one launch, the first of partial sums
    (1024, 40, 72, 20), (520, 72, 40, 100),    # the same at ranks 32 and 128
    (300, 2056, 264, 128), (300, 264, 2056, 100),  # 64 x 64 tiles, six ragged chunks and one, in either job
    (1000, 1032, 520, 64),                     # five and three
    (4100, 264, 1032, 128),                    # 128 x 128 tiles, three and one
])
def test_backward_plans(M, K, N, r, dev):
    say("backward plan", M, K, N, r)
    case = WL.gen_backward(1200 + M + K + r, M, K, N, r)
    c = case.lin
    full = _run(case, dev)
    for got, want, name in zip(full, lora_linear_backward_ref(c.x, c.W, c.A, c.B, c.s, case.dy), ("dx", "dA", "dB")):
        assert_rel(got, want, name)
    for i, name in enumerate(("dx", "dA", "dB")):
        assert np.array_equal(_run(case, dev, want=(name,))[i], full[i]), name


def _touched(ws):
    """Whether any byte of a workspace filled with 0xAB was written."""
    return bool((ws != 0xAB).any().item())


@pytest.mark.parametrize("M,N,K,r,pre", [(1030, 8200, 264, 64, True), (1030, 8200, 264, 33, True), (1030, 8200, 264, 32, False),
                                         (384, 12288, 256, 64, False)])
def test_rank_64_takes_the_pre_pass_where_its_tiles_run_several_rounds(M, N, K, r, pre, dev):
    """387 and 192 tiles of 128 x 192; the workspace shows which way the update went.  y_off has the plain call's bits."""
    import torch
    say("rank 64 route", M, N, K, r)
    c = WL.gen_linear(1300 + M + N + r, M, K, N, r)
    x, W, A, B = (dev_bf16(v, dev) for v in (c.x, c.W, c.A, c.B))
    ws = torch.full((H.hydra_lora_linear_workspace_bytes(M, N, r),), 0xAB, dtype=torch.uint8, device=dev)
    off, on, plain = (torch.full((M, N), float("nan"), device=dev) for _ in range(3))
    H.hydra_lora_linear_ws(x, W, A, B, c.s, off, on, ws)
    H.hydra_lora_linear(x, W, A, B, c.s, plain, None)
    torch.cuda.synchronize()
    assert _touched(ws) == pre
    assert torch.equal(off, plain)
    e_off, e_on = lora_linear_ref(c.x, c.W, c.A, c.B, c.s)
    assert_rel(host(off), e_off, "y_off")
    assert_rel(host(on), e_on, "y_on")


@pytest.mark.parametrize("M,K,r,one", [(64, 1024, 32, True), (64, 1032, 32, False), (64, 4096, 16, False), (64, 3072, 16, True),
                                       (2560, 4096, 16, True), (2559, 4096, 32, True), (4100, 264, 16, False),
                                       (64, 1024, 128, True), (1024, 2048, 128, False)])
def test_one_launch_where_k_is_short_or_rows_many(M, K, r, one, dev):
    """The pre-pass of the scoring pass leaves partial sums in the end of the workspace only where it takes two launches."""
    import torch
    say("pre-pass plan", M, K, r)
    V = 40
    s = WL.gen_score_head(1400 + M + K + r, 1, M, K, V, r)
    ws = torch.full((H.hydra_score_workspace_bytes(M, V),), 0xAB, dtype=torch.uint8, device=dev)
    out = [torch.full((M,), float("nan"), device=dev) for _ in range(3)]
    H.hydra_score(dev_bf16(s.h, dev), dev_bf16(s.W_lm, dev), dev_bf16(s.A, dev), dev_bf16(s.B, dev), s.s,
                  torch.from_numpy(s.ids).to(dev), None, 1, M, *out, workspace=ws)
    torch.cuda.synchronize()
    assert _touched(ws[-8 * M * 128 * 4:]) == (not one)
    e = score_head_ref(s.h, s.W_lm, s.A, s.B, s.s, s.ids, s.w_rm, 1, M)
    for got, k in zip(out, ("lp_on", "lp_off", "kl")):
        assert_abs(host(got), e[k], k)
