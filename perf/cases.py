"""The work that a Hydra-PPO program has this library do, as cases to time.

A case is a dict of plain values; "kind" names the entry points it goes through:

* linear   one LoRA-switchable linear (hydra_lora_linear), with its pre-pass workspace (hydra_lora_linear_ws), or q/k/v
           as a group (hydra_lora_linear_group): prompts, mini-batches, larger generation batches
* decode   one generation step of a group of projections (hydra_lora_linear_group_ws)
* score    the two-head scoring pass (hydra_score, hydra_score_two_input)
* logits   the scoring epilogue over materialised logits (hydra_score_logits)
* backward the adapter's gradients through one linear (hydra_lora_linear_backward)
* ppo      critic values, advantages and losses (hydra_value_head, hydra_ppo_advantages, hydra_ppo_loss)

Sizes are those of the repository's Llama-7B and OPT-1.3b configurations and ragged ones between them.  Inputs follow
the recipe of the workloads package: activations N(0, 1), base weights and A N(0, 1/K), B N(0, 1/r), scale 2.
"""
import math

import torch

import paper_2309_00754_amd as H

SCALE = 2.0
BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64

# (K, N) of the linears of a Llama-7B and of an OPT-1.3b layer
LLAMA = [(4096, 4096), (4096, 11008), (11008, 4096)]
OPT = [(2048, 2048), (2048, 8192), (8192, 2048)]


def listed():
    return [
        # the smallest call: one small linear, bound by launch and host time
        dict(name="linear_small", kind="linear", entry="plain", M=16, K=512, N=512, r=8),
        # one token per sequence for a batch of 4, the attention projections of Llama-7B
        dict(name="decode_llama", kind="decode", G=4, M=4, K=4096, N=4096, r=16),
        # OPT-1.3b's generation batch of 6 at the paper's rank 128
        dict(name="decode_opt_r128", kind="decode", G=4, M=6, K=2048, N=2048, r=128),
        # a generation batch of 48 sequences: too many rows for the decode path, few for a prefill
        dict(name="batch_llama", kind="linear", entry="plain", M=48, K=4096, N=4096, r=16),
        # one prompt of 333 tokens through Llama-7B's gate projection
        dict(name="prompt_llama", kind="linear", entry="plain", M=333, K=4096, N=11008, r=16),
        # q, k and v of Llama-7B over a batch of 4 x 512 tokens
        dict(name="prefill_llama", kind="linear", entry="group", M=2048, K=4096, N=4096, r=16),
        # OPT-1.3b's fc2 over a mini-batch of 8 x 512 tokens, rank 128
        dict(name="prefill_opt_r128", kind="linear", entry="ws", M=4096, K=8192, N=2048, r=128),
        # the scoring pass over a batch of 4 x 512 tokens, Llama-7B heads
        dict(name="score_llama", kind="score", two=False, n_seq=4, seq_len=512, K=4096, V=32000, r=16),
        # one sequence of 250 tokens, actor and reference hidden states, OPT-1.3b heads (ragged vocabulary), rank 128
        dict(name="score_opt_two_input", kind="score", two=True, n_seq=1, seq_len=250, K=2048, V=50272, r=128),
        # the scoring epilogue of a program that keeps its own logits
        dict(name="logits", kind="logits", M=512, V=32000),
        # the update stage's backward through one Llama-7B attention projection
        dict(name="backward_llama", kind="backward", M=2048, K=4096, N=4096, r=16),
        # critic values, advantages and losses of a batch of 4 x 512 tokens, half of them prompt
        dict(name="ppo_step", kind="ppo", n_seq=4, seq_len=512, start=256, K=4096),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _layer(rng):
    """(K, N) of a layer: the configurations' own, or one of the same range (K a multiple of 8, N any)."""
    if rng.random() < 0.75:
        return rng.choice(LLAMA + OPT)
    return 8 * _log(rng, 64, 1024), _log(rng, 512, 8192)


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "decode", "score", "score", "logits", "backward", "backward", "ppo"])
    if kind == "linear":
        entry = rng.choice(["plain", "ws", "group"])
        K, N = _layer(rng)
        r = rng.choice([8, 16, 64, 128] if entry == "ws" else [8, 16, 64])
        top = 2048 if entry == "group" and K * N > (1 << 24) else 4096
        return dict(kind=kind, entry=entry, M=_log(rng, 16, top), K=K, N=N, r=r)
    if kind == "decode":
        K, N = rng.choice([(4096, 4096), (2048, 2048), (8 * _log(rng, 64, 640), _log(rng, 512, 5120))])
        return dict(kind=kind, G=rng.choice([1, 3, 4]), M=_log(rng, 1, 16), K=K, N=N, r=rng.choice([8, 16, 64, 128]))
    if kind == "score":
        two = rng.random() < 0.4
        K, V = rng.choice([(4096, 32000), (2048, 50272), (8 * _log(rng, 64, 512), _log(rng, 2000, 60000))])
        n_seq = _log(rng, 1, 8)
        top = 2048 * 4096 * 32000 // (K * V * (2 if two else 1))
        return dict(kind=kind, two=two, n_seq=n_seq, seq_len=max(1, min(_log(rng, 16, 1024), top // n_seq)), K=K, V=V,
                    r=rng.choice([8, 16, 128]))
    if kind == "logits":
        V = rng.choice([32000, 50272, _log(rng, 2000, 60000)])
        return dict(kind=kind, M=_log(rng, 16, 1024), V=V)
    if kind == "backward":
        K, N = _layer(rng)
        return dict(kind=kind, M=_log(rng, 64, 3000), K=K, N=(N + 7) // 8 * 8, r=rng.choice([8, 16, 64, 128]))
    seq_len = _log(rng, 16, 2048)
    return dict(kind=kind, n_seq=_log(rng, 1, 64), seq_len=seq_len, start=rng.randrange(seq_len),
                K=rng.choice([2048, 4096, 8 * _log(rng, 64, 512)]))


class _Draw:
    """Seeded normal tensors on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, *shape, std=1.0, dtype=BF16):
        return torch.randn(*shape, generator=self.g, device="cuda", dtype=F32).mul_(std).to(dtype)

    def lora(self, K, N, r):
        return (self.normal(N, K, std=K ** -0.5), self.normal(r, K, std=K ** -0.5), self.normal(N, r, std=r ** -0.5))

    def ids(self, M, V):
        return torch.randint(0, V, (M,), generator=self.g, device="cuda", dtype=torch.int32)


def _inputs(case, seed):
    d, kind = _Draw(seed), case["kind"]
    i = {}
    if kind in ("linear", "decode"):
        G = case.get("G", 3 if case.get("entry") == "group" else 1)
        x = d.normal(case["M"], case["K"])
        i["x"] = [x] * G  # the projections of a layer read the same rows
        i["W"], i["A"], i["B"] = (list(t) for t in zip(*(d.lora(case["K"], case["N"], case["r"]) for _ in range(G))))
    elif kind == "score":
        M, K = case["n_seq"] * case["seq_len"], case["K"]
        i["h"] = d.normal(M, K)
        i["h_act"] = d.normal(M, K) if case["two"] else None
        i["W"], i["A"], i["B"] = d.lora(K, case["V"], case["r"])
        i["w_rm"] = d.normal(K, std=K ** -0.5)
        i["tokens"] = d.ids(M, case["V"])
    elif kind == "logits":
        i["on"] = d.normal(case["M"], case["V"], std=2.0, dtype=F32)
        i["off"] = i["on"] + d.normal(case["M"], case["V"], std=0.1, dtype=F32)
        i["tokens"] = d.ids(case["M"], case["V"])
    elif kind == "backward":
        i["x"] = d.normal(case["M"], case["K"])
        i["W"], i["A"], i["B"] = d.lora(case["K"], case["N"], case["r"])
        i["dy"] = d.normal(case["M"], case["N"])
    else:
        M = case["n_seq"] * case["seq_len"]
        i["h"] = d.normal(M, case["K"])
        i["w_v"] = d.normal(case["K"], std=case["K"] ** -0.5)
        i["kl"] = d.normal(M, std=0.1, dtype=F32)
        i["reward"] = d.normal(case["n_seq"], dtype=F32)
        i["lp_old"] = -d.normal(M, std=2.0, dtype=F32).abs()
        i["lp_new"] = i["lp_old"] + d.normal(M, std=0.1, dtype=F32)
    return i


def prepare(case, seed):
    """The inputs, and the output buffers and workspace that a program allocates once."""
    s = _inputs(case, seed)
    s["case"], kind = case, case["kind"]

    def out(*shape):
        return torch.empty(shape, device="cuda", dtype=F32)

    if kind in ("linear", "decode"):
        M, N, G = case["M"], case["N"], len(s["W"])
        s["s"] = [SCALE] * G
        s["y_off"], s["y_on"] = [out(M, N) for _ in range(G)], [out(M, N) for _ in range(G)]
        if kind == "decode":
            s["ws"] = H.hydra_lora_linear_group_workspace(G, M, N, case["r"], "cuda")
        elif case["entry"] == "ws":
            s["ws"] = torch.empty(max(1, H.hydra_lora_linear_workspace_bytes(M, N, case["r"])), dtype=torch.uint8,
                                  device="cuda")
    elif kind == "score":
        M = case["n_seq"] * case["seq_len"]
        s["lp_on"], s["lp_off"], s["kl"], s["reward"] = out(M), out(M), out(M), out(case["n_seq"])
        s["ws"] = torch.empty(H.hydra_score_workspace_bytes(M, case["V"]), dtype=torch.uint8, device="cuda")
    elif kind == "logits":
        s["lp_on"], s["lp_off"], s["kl"] = out(case["M"]), out(case["M"]), out(case["M"])
    elif kind == "backward":
        M, K, N, r = case["M"], case["K"], case["N"], case["r"]
        W = s.pop("W")
        s["Wt"] = torch.empty((K, N), dtype=BF16, device="cuda")  # W is frozen: transposed once for a whole training run
        H.hydra_transpose_bf16(W, s["Wt"])
        s["dx"], s["dA"], s["dB"] = out(M, K), out(r, K), out(N, r)
        s["ws"] = torch.empty(H.hydra_lora_linear_backward_workspace_bytes(M, N, K, r), dtype=torch.uint8, device="cuda")
    else:
        M = case["n_seq"] * case["seq_len"]
        for k in ("values", "advantages", "returns", "rewards", "d_lp", "d_v"):
            s[k] = out(M)
        s["losses"] = out(3)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "linear":
        if case["entry"] == "group":
            H.hydra_lora_linear_group(s["x"], s["W"], s["A"], s["B"], s["s"], s["y_off"], s["y_on"])
        elif case["entry"] == "ws":
            H.hydra_lora_linear_ws(s["x"][0], s["W"][0], s["A"][0], s["B"][0], SCALE, s["y_off"][0], s["y_on"][0], s["ws"])
        else:
            H.hydra_lora_linear(s["x"][0], s["W"][0], s["A"][0], s["B"][0], SCALE, s["y_off"][0], s["y_on"][0])
        return {"off": s["y_off"], "on": s["y_on"]}
    if kind == "decode":
        H.hydra_lora_linear_group_ws(s["x"], s["W"], s["A"], s["B"], s["s"], s["y_off"], s["y_on"], s["ws"])
        return {"off": s["y_off"], "on": s["y_on"]}
    if kind == "score":
        if case["two"]:
            H.hydra_score_two_input(s["h_act"], s["h"], s["W"], s["A"], s["B"], SCALE, s["tokens"], s["w_rm"],
                                    case["n_seq"], case["seq_len"], s["lp_on"], s["lp_off"], s["kl"], s["reward"],
                                    workspace=s["ws"])
        else:
            H.hydra_score(s["h"], s["W"], s["A"], s["B"], SCALE, s["tokens"], s["w_rm"], case["n_seq"],
                          case["seq_len"], s["lp_on"], s["lp_off"], s["kl"], s["reward"], workspace=s["ws"])
        return {k: s[k] for k in ("lp_on", "lp_off", "kl", "reward")}
    if kind == "logits":
        H.hydra_score_logits(s["on"], s["off"], s["tokens"], s["lp_on"], s["lp_off"], s["kl"])
        return {k: s[k] for k in ("lp_on", "lp_off", "kl")}
    if kind == "backward":
        H.hydra_lora_linear_backward(s["x"], s["Wt"], s["A"], s["B"], SCALE, s["dy"], s["dx"], s["dA"], s["dB"], s["ws"])
        return {k: s[k] for k in ("dx", "dA", "dB")}
    H.hydra_value_head(s["h"], s["w_v"], s["values"])
    H.hydra_ppo_advantages(s["kl"], s["reward"], s["values"], case["n_seq"], case["seq_len"], s["advantages"],
                           s["returns"], s["rewards"], start=case["start"])
    H.hydra_ppo_loss(s["lp_new"], s["lp_old"], s["advantages"], s["values"], s["returns"], case["n_seq"],
                     case["seq_len"], s["losses"], s["d_lp"], s["d_v"], start=case["start"])
    return {k: s[k] for k in ("values", "advantages", "returns", "rewards", "losses", "d_lp", "d_v")}


def work(case):
    kind = case["kind"]
    if kind in ("linear", "decode"):
        M, K, N, r = case["M"], case["K"], case["N"], case["r"]
        G = case.get("G", 3 if case.get("entry") == "group" else 1)
        return {"bytes": 2 * M * K + G * (2 * (N * K + r * K + N * r) + 8 * M * N),
                "flops": G * 2 * (M * N * K + M * K * r + M * N * r)}
    if kind == "score":
        M, K, V, r, two = case["n_seq"] * case["seq_len"], case["K"], case["V"], case["r"], case["two"]
        return {"bytes": 2 * ((2 if two else 1) * M * K + V * K + r * K + V * r + K) + 16 * M + 4 * case["n_seq"],
                "flops": 2 * ((2 if two else 1) * M * V * K + M * K * r + M * V * r)}
    if kind == "logits":
        return {"bytes": 8 * case["M"] * case["V"] + 16 * case["M"], "flops": 0}
    if kind == "backward":
        M, K, N, r = case["M"], case["K"], case["N"], case["r"]
        return {"bytes": 2 * (M * K + N * K + r * K + N * r + M * N) + 4 * (M * K + r * K + N * r),
                "flops": 2 * M * N * K + 4 * M * N * r + 6 * M * K * r}
    M, K = case["n_seq"] * case["seq_len"], case["K"]
    return {"bytes": 2 * (M * K + K) + 36 * M + 4 * case["n_seq"], "flops": 2 * M * K}


def tolerance(case):
    # 32-bit sums of bf16 products, and s x A^T carried in 16 significant bits: about 2.3e-6 off 64 bits, so two
    # implementations may differ by 3e-6.  Over given logits the KL estimate (0.1) is the difference of two
    # log-probabilities (10): 7e-6 off.  Advantages and returns sum up to 2048 terms: 1e-6 off.
    rel = {"logits": 3e-5, "ppo": 1e-5}.get(case["kind"], 1.2e-5)
    return {"rel": rel, "max": 40 * rel}


def _dot(a, b):
    return a.to(F64) @ b.to(F64).t()


def exact(case, seed):
    i, kind = _inputs(case, seed), case["kind"]
    if kind in ("linear", "decode"):
        off, on = [], []
        for x, W, A, B in zip(i["x"], i["W"], i["A"], i["B"]):
            off.append(_dot(x, W))
            on.append(off[-1] + SCALE * _dot(_dot(x, A), B))
        return {"off": off, "on": on}
    if kind == "score":
        lp_on, lp_off, W = [], [], i["W"].to(F64)
        M, B = case["n_seq"] * case["seq_len"], i["B"].to(F64)
        for m in range(0, M, 256):
            h = i["h"][m:m + 256].to(F64)
            ha = h if i["h_act"] is None else i["h_act"][m:m + 256].to(F64)
            tok = i["tokens"][m:m + 256].long()[:, None]
            z = h @ W.t()
            lp_off.append((z.gather(1, tok) - torch.logsumexp(z, 1, keepdim=True))[:, 0])
            z = (z if i["h_act"] is None else ha @ W.t()) + SCALE * (ha @ i["A"].to(F64).t()) @ B.t()
            lp_on.append((z.gather(1, tok) - torch.logsumexp(z, 1, keepdim=True))[:, 0])
        lp_on, lp_off = torch.cat(lp_on), torch.cat(lp_off)
        T = case["seq_len"]
        return {"lp_on": lp_on, "lp_off": lp_off, "kl": lp_on - lp_off,
                "reward": i["h"][T - 1::T].to(F64) @ i["w_rm"].to(F64)}
    if kind == "logits":
        tok = i["tokens"].long()[:, None]
        lp = {}
        for k in ("on", "off"):
            z = i[k].to(F64)
            lp[k] = (z.gather(1, tok) - torch.logsumexp(z, 1, keepdim=True))[:, 0]
        return {"lp_on": lp["on"], "lp_off": lp["off"], "kl": lp["on"] - lp["off"]}
    if kind == "backward":
        dy, x, A, B = (i[k].to(F64) for k in ("dy", "x", "A", "B"))
        u = dy @ B
        return {"dx": dy @ i["W"].to(F64) + SCALE * (u @ A), "dA": SCALE * (u.t() @ x), "dB": SCALE * (dy.t() @ (x @ A.t()))}
    n, T, start = case["n_seq"], case["seq_len"], case["start"]
    values = (i["h"].to(F64) @ i["w_v"].to(F64)).cpu().view(n, T)
    kl, rew, lp_new, lp_old = (i[k].to(F64).cpu() for k in ("kl", "reward", "lp_new", "lp_old"))
    mask = (torch.arange(T) >= start).to(F64)
    beta, gamma, lam, eps = 0.02, 1.0, 0.95, 0.2
    rewards = -beta * kl.view(n, T) * mask
    rewards[:, -1] += rew
    adv, after, nxt = torch.zeros(n, T, dtype=F64), torch.zeros(n, dtype=F64), torch.zeros(n, dtype=F64)
    for t in range(T - 1, -1, -1):
        after = rewards[:, t] + gamma * nxt - values[:, t] + gamma * lam * after
        nxt = values[:, t]
        adv[:, t] = after
    ret = (adv + values) * mask
    adv = adv * mask
    rho = torch.exp(lp_new - lp_old).view(n, T)
    un, cl = rho * adv, rho.clamp(1 - eps, 1 + eps) * adv
    cnt = n * (T - start)
    clipped = (un > cl) & (mask > 0)
    losses = torch.stack([-(torch.minimum(un, cl) * mask).sum(), ((values - ret) ** 2 * mask).sum() / 2,
                          clipped.to(F64).sum()]) / cnt
    d_lp = torch.where(clipped, torch.zeros_like(un), -un) * mask / cnt
    d_v = (values - ret) * mask / cnt
    o = dict(values=values, advantages=adv, returns=ret, rewards=rewards, losses=losses, d_lp=d_lp, d_v=d_v)
    return {k: v.reshape(-1) for k, v in o.items()}
