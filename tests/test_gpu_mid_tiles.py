"""The dual GEMM's smaller tiles (9 rows to a few hundred): edges of every tile, K shorter than a slab and longer than
the ring, every way the LoRA update reaches them, against the float64 oracle; and the bits that the entry points share.
Tolerances: the arithmetic bound of the other linear tests (2e-4 relative)."""
import ctypes

import numpy as np
import pytest

import paper_2309_00754_amd as H
from paper_2309_00754_amd import _binding as Bd
import workloads as WL
from oracle import lora_linear_ref
from gpu_helpers import assert_rel, dev_bf16, host, say

pytestmark = pytest.mark.gpu

# (M, N, K) by the tile that the size model picks (-1: up to 16 rows, whose tiles go by rank and members too): with
# remainders in both directions, and of whole tiles
SHAPES = {
    -1: [(9, 40, 264), (16, 512, 512)],                                    # 16 rows
    0: [(17, 33, 8), (31, 700, 72), (64, 96, 1536)],                       # 32 x 32
    1: [(65, 5000, 264), (96, 4096, 128)],                                 # 32 x 64
    2: [(40, 8200, 136), (128, 8192, 1032)],                               # 64 x 64
    3: [(200, 5000, 264), (300, 5001, 1000), (128, 16384, 128), (256, 8192, 2048)],  # 64 x 128
    4: [(230, 11000, 520), (384, 8192, 1536)],                             # 128 x 128
    5: [(129, 16500, 72), (400, 11001, 520), (384, 12288, 256)],           # 128 x 192
}


def test_shapes_go_to_the_tiles_they_are_listed_under():
    import torch  # noqa: F401 (its HIP runtime first: the library is to find that one)
    pick = ctypes.CDLL(Bd.LIB_PATH)["_ZN5hydra13gemm_mid_tileEiii"]
    pick.argtypes, pick.restype = [ctypes.c_int] * 3, ctypes.c_int
    for tile, shapes in SHAPES.items():
        for s in shapes:
            assert (pick(*s) == tile) if tile >= 0 else s[0] <= 16, (s, pick(*s))


def _inputs(M, N, K, r, dev, member=0):
    c = WL.gen_linear(9000 + M + 3 * N + 7 * K + r + 100000 * member, M, K, N, r)
    x, W = dev_bf16(c.x, dev), dev_bf16(c.W, dev)
    return c, x, W, dev_bf16(c.A, dev) if r else None, dev_bf16(c.B, dev) if r else None


def _nan(M, N, dev):
    import torch
    return torch.full((M, N), float("nan"), device=dev)


@pytest.mark.parametrize("r", [0, 8, 16, 20, 64, 100])
@pytest.mark.parametrize("M,N,K", sum(SHAPES.values(), []))
def test_mid_tiles(M, N, K, r, dev):
    import torch
    say("mid tile", M, N, K, r)
    c, x, W, A, B = _inputs(M, N, K, r, dev)
    e_off, e_on = lora_linear_ref(c.x, c.W, c.A, c.B, c.s)
    w_off, w_on = _nan(M, N, dev), _nan(M, N, dev)
    H.hydra_lora_linear_ws(x, W, A, B, c.s, w_off, w_on)
    torch.cuda.synchronize()
    assert_rel(host(w_off), e_off, "ws y_off")
    assert_rel(host(w_on), e_on, "ws y_on")
    if r > 64:
        return
    y_off, y_on = _nan(M, N, dev), _nan(M, N, dev)
    H.hydra_lora_linear(x, W, A, B, c.s, y_off, y_on)
    only = _nan(M, N, dev)
    H.hydra_lora_linear(x, W, A, B, c.s, None, only)
    torch.cuda.synchronize()
    assert_rel(host(y_off), e_off, "y_off")
    assert_rel(host(y_on), e_on, "y_on")
    assert torch.equal(y_off, w_off) and torch.equal(only, y_on)
    if r:  # a zero scale and a zero B add exact zeros
        H.hydra_lora_linear(x, W, A, B, 0.0, y_off, y_on)
        H.hydra_lora_linear(x, W, A, torch.zeros_like(B), c.s, w_off, w_on)
        torch.cuda.synchronize()
        assert torch.equal(y_on, y_off) and torch.equal(w_on, w_off)


@pytest.mark.parametrize("M,N,K,r", [(33, 700, 264, 16), (40, 1500, 136, 64), (100, 999, 520, 128), (65, 2052, 264, 128),
                                     (200, 3001, 72, 8)])
def test_mid_group_members_have_the_bits_of_single_calls(M, N, K, r, dev):
    """Members with, without and with only one of the outputs of an adapter, in one launch."""
    import torch
    say("mid group", M, N, K, r)
    G = 4
    ms = [_inputs(M, N, K, r, dev, i) for i in range(G)]
    xs, Ws = [m[1] for m in ms], [m[2] for m in ms]
    As, Bs = [m[3] for m in ms], [m[4] for m in ms]
    ss = [2.0, -0.5, 1.0, 3.0]
    offs = [_nan(M, N, dev), None, _nan(M, N, dev), _nan(M, N, dev)]
    ons = [_nan(M, N, dev), _nan(M, N, dev), None, _nan(M, N, dev)]
    if r > 64:
        ws = H.hydra_lora_linear_group_workspace(G, M, N, r, dev)
        H.hydra_lora_linear_group_ws(xs, Ws, As, Bs, ss, offs, ons, ws)
    else:
        H.hydra_lora_linear_group(xs, Ws, As, Bs, ss, offs, ons)
    torch.cuda.synchronize()
    for i in range(G):
        off, on = _nan(M, N, dev), _nan(M, N, dev)
        (H.hydra_lora_linear_ws if r > 64 else H.hydra_lora_linear)(xs[i], Ws[i], As[i], Bs[i], ss[i], off, on)
        torch.cuda.synchronize()
        assert offs[i] is None or torch.equal(offs[i], off)
        assert ons[i] is None or torch.equal(ons[i], on)
    # a group without any adapter
    offs = [_nan(M, N, dev) for _ in range(G)]
    ons = [_nan(M, N, dev) for _ in range(G)]
    H.hydra_lora_linear_group(xs, Ws, [None] * G, [None] * G, ss, offs, ons)
    torch.cuda.synchronize()
    for i in range(G):
        assert torch.equal(offs[i], ons[i])
        assert np.isfinite(host(offs[i])).all()


@pytest.mark.parametrize("M,N,K,r", [(9, 50001, 72, 16), (16, 52000, 64, 64), (12, 300, 264, 8), (16, 11008, 1032, 64),
                                     (9, 700, 2056, 20), (16, 512, 520, 16)])
def test_few_rows_keep_the_bits_of_t(M, N, K, r, dev):
    """Up to 16 rows, s T holds 24 bits at every width, and no sum is one long chain.  In 2-norm y_on is then off 64 bits
    by the rounding of fp32 sums: under 2^-24 for each of at most 70 additions in a row adding up at random, 5e-7 (and
    under sqrt(K + r) 2^-24 where there are fewer products).  With s T in two bf16 parts it would be off by 2e-6."""
    import torch
    say("few rows", M, N, K, r)
    c, x, W, A, B = _inputs(M, N, K, r, dev)
    e_on = lora_linear_ref(c.x, c.W, c.A, c.B, c.s)[1]
    y_on = _nan(M, N, dev)
    H.hydra_lora_linear(x, W, A, B, c.s, None, y_on)
    torch.cuda.synchronize()
    err = np.linalg.norm(host(y_on) - e_on) / np.linalg.norm(e_on)
    assert err < min(5e-7, np.sqrt(K + r) * 2.0 ** -24), err
    y_off, alone = _nan(M, N, dev), _nan(M, N, dev)  # y_off has the same bits with and without an adapter
    H.hydra_lora_linear(x, W, A, B, c.s, y_off, y_on)
    H.hydra_lora_linear(x, W, None, None, 0.0, alone, None)
    torch.cuda.synchronize()
    assert torch.equal(y_off, alone)


@pytest.mark.parametrize("G,M,N,K,r", [(8, 9, 3000, 1000, 64), (4, 16, 8200, 264, 16), (3, 12, 4096, 520, 32), (8, 10, 700, 72, 8),
                                       (2, 16, 5001, 1032, 0), (8, 9, 2048, 2048, 0)])
def test_few_rows_have_the_same_bits_on_every_tile(G, M, N, K, r, dev):
    """Up to 16 rows the tile depends on the rank and on the members of a launch; an output does not."""
    import torch
    say("few rows, group", G, M, N, K, r)
    ms = [WL.gen_linear(9500 + i + N + K + r, M, K, N, r) for i in range(G)]
    xs, Ws = [dev_bf16(c.x, dev) for c in ms], [dev_bf16(c.W, dev) for c in ms]
    As, Bs = ([dev_bf16(c.A, dev) for c in ms], [dev_bf16(c.B, dev) for c in ms]) if r else ([None] * G, [None] * G)
    ss = [c.s + i for i, c in enumerate(ms)]
    offs, ons = [_nan(M, N, dev) for _ in range(G)], [_nan(M, N, dev) for _ in range(G)]
    H.hydra_lora_linear_group(xs, Ws, As, Bs, ss, offs, ons)
    for i, c in enumerate(ms):
        off, on, alone = _nan(M, N, dev), _nan(M, N, dev), _nan(M, N, dev)
        H.hydra_lora_linear(xs[i], Ws[i], As[i], Bs[i], ss[i], off, on)
        H.hydra_lora_linear(xs[i], Ws[i], None, None, 0.0, alone, None)
        torch.cuda.synchronize()
        assert torch.equal(offs[i], off) and torch.equal(ons[i], on) and torch.equal(alone, off), i
        e_off, e_on = lora_linear_ref(c.x, c.W, c.A, c.B, ss[i])
        assert_rel(host(off), e_off, "y_off")
        assert_rel(host(on), e_on, "y_on")


def test_few_rows_cost_less_than_a_wider_tile(dev):
    """Nine rows of 8192 x 2048 take clearly less than seventeen, whose tile copies twice the rows (on one tile with them
    they took the same, 18 us, where the kernel for few rows before it took 15)."""
    import torch
    say("few rows time")
    K, N, n = 8192, 2048, 12
    Ws = [torch.randn(N, K, device=dev).to(torch.bfloat16) for _ in range(n)]  # more than the caches hold

    def us(M):
        x, off = torch.randn(M, K, device=dev).to(torch.bfloat16), torch.empty(M, N, device=dev)
        best = float("inf")
        for _ in range(20):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for W in Ws * 4:
                H.hydra_lora_linear(x, W, None, None, 0.0, off, None)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3 / (4 * n))
        return best

    few, more = us(9), us(17)
    say(f"{few:.2f} {more:.2f} us")
    assert few < 0.9 * more, (few, more)


def test_an_infinite_t_gives_infinite_outputs(dev):
    import torch
    say("infinite t")
    M, N, K, r = 12, 40, 64, 16
    x, W, A, B = (torch.ones(s, device=dev, dtype=torch.bfloat16) for s in ((M, K), (N, K), (r, K), (N, r)))
    A[3] = 3e38  # the sum of 64 of them overflows
    B[::2, 3] = -1
    y_on = _nan(M, N, dev)
    H.hydra_lora_linear(x, W, A, B, 2.0, None, y_on)
    torch.cuda.synchronize()
    assert (y_on[:, ::2] == float("-inf")).all() and (y_on[:, 1::2] == float("inf")).all()


@pytest.mark.parametrize("M,N,K,r", [(12, 40, 64, 16), (9, 3000, 520, 64), (16, 9000, 72, 20)])
def test_an_infinite_b_gives_infinite_outputs(M, N, K, r, dev):
    """Up to 16 rows (x A^T) meets B in 24 bits, in parts: an infinity in B gives the infinity that the whole would."""
    import torch
    say("infinite b", M, N, K, r)
    c = WL.gen_linear(9700 + N + r, M, K, N, r)
    x, W, A, B = (dev_bf16(v, dev).view(torch.bfloat16).clone() for v in (c.x, c.W, c.A, c.B))
    T = (x.double() @ A.double().t())[:, 3]
    B[::2, 3], B[1::4, 3] = float("inf"), float("-inf")
    y_on = _nan(M, N, dev)
    H.hydra_lora_linear(x, W, A, B, 2.0, None, y_on)
    torch.cuda.synchronize()
    sign = torch.sign(T)[:, None].expand(M, N)
    assert (y_on[:, ::2] == (sign * float("inf"))[:, ::2]).all() and (y_on[:, 1::4] == (-sign * float("inf"))[:, 1::4]).all()
    assert torch.isfinite(y_on[:, 3::4]).all()
