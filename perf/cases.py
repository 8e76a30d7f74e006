"""What a user has this library do, as a list of timed cases: whole passes through the public calls of
`spt` (routed FFN) and `mha` (sparse attention), on tensors that already live on the GPU.

A case is a dict of plain values.  `prepare` makes what a program holds before a pass -- inputs,
weights, buffers, workspaces -- and `run` is one pass.  Four kinds of pass:

  train  router, bucketing, schedule tables, forward, backward of the routed FFN; with "balance" the
         route network's load-balancing loss and gradient too
  infer  router, bucketing, forward without the saved pre-activations (prefill, decode)
  lora   the low-rank adapted fine-tuning pass: router, bucketing, forward, backward, frozen weights
  mha    sparse attention: code assignment of queries and keys, top-L selection, attention forward
         and, with "train", backward

Random tokens and weights follow the recipes of `inputs.py` and `mha_inputs.py`, drawn on the GPU."""
import math

import torch

from paper_2312_10365_amd import inputs, mha, spt

BF16, F32, I32, U8 = torch.bfloat16, torch.float32, torch.int32, torch.uint8


def ffn_case(kind, T, d, N, Bs, k, act="gelu", skew=False, abs_logit=False, balance=False, rank=0, **name):
    return dict(kind=kind, T=T, d=d, N=N, Bs=Bs, k=k, act=act, skew=skew, abs_logit=abs_logit, balance=balance,
                rank=rank, **name)


def mha_case(batch, H, n, dh, L, E=16, train=True, **name):
    return dict(kind="mha", batch=batch, H=H, n=n, dh=dh, L=L, E=E, train=train, **name)


def listed():
    return [
        # A few hundred tokens through a small layer: a step of a debugging or distillation run, where
        # the calls themselves and the launches are what the user waits for.
        ffn_case("train", 512, 256, 16, 64, 4, name="tiny_train"),
        # A small encoder's layer, four sequences of 512 tokens; blocks of 96 units (not a power of two).
        ffn_case("train", 2048, 768, 32, 96, 8, name="bert_base_train"),
        # A large encoder's layer at a full training batch, many small blocks.
        ffn_case("train", 16384, 1024, 64, 64, 16, name="bert_large_train"),
        # A decoder layer whose router still prefers a few blocks, trained with the balancing loss that is
        # there to cure it: buckets several times the mean beside small ones.
        ffn_case("train", 8192, 2048, 64, 128, 16, skew=True, balance=True, name="opt_1p3b_skewed_train"),
        # The layer of a 7B model, 16 sequences of 512 tokens: the benchmark's default, and the largest.
        ffn_case("train", 8192, 4096, 128, 128, 32, name="ffn_7b_train"),
        # The same layer in serving: one decoding step of a batch of 24 sequences (every weight is read
        # for a handful of tokens), and a prefill of mixed prompts, a token count that is no multiple of anything.
        ffn_case("infer", 24, 4096, 128, 128, 32, name="ffn_7b_decode"),
        ffn_case("infer", 3001, 4096, 128, 128, 32, name="ffn_7b_prefill"),
        # The paper's own setting: low-rank fine-tuning of a 2048-wide decoder block, four wide groups, two active.
        ffn_case("lora", 8192, 2048, 4, 2048, 2, act="relu", rank=16, name="paper_opt2048_g4_lora"),
        # The paper's larger block with every weight trained.
        ffn_case("train", 8192, 4096, 4, 2752, 2, name="paper_llama4096_g4_train"),
        # Sparse attention of those two blocks: 16 sequences of 512 tokens, 32 heads, an eighth of the keys kept.
        mha_case(16, 32, 512, 64, 64, name="mha_opt2048_train"),
        mha_case(16, 32, 512, 128, 64, name="mha_llama4096_train"),
        # Longer documents of ragged length, few at a time.
        mha_case(3, 32, 1100, 128, 137, name="mha_long_ragged_train"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_FLOP = 12 * 8192 * 4096 * 32 * 128          # the listed 7B layer's training pass
MOST_WEIGHT = 128 * 128 * 4096                   # and its weights
MOST_ATTENTION = 512 * 512 * 64 * 128            # kept entries x head size of the listed attention passes


def draw(rng):
    """One more case: every kind, token counts over the whole range, widths and blocks over what the listed
    configurations span, both activations, both ways to route, any rank."""
    kind = rng.choice(["train", "train", "train", "infer", "infer", "lora", "lora", "mha", "mha", "mha"])
    if kind == "mha":
        n = _log(rng, 96, 2048)
        dh = rng.choice([64, 128])
        L = max(8, min(256, int(n * rng.uniform(0.06, 0.25))))
        H = rng.choice([8, 12, 16, 32])
        batch = max(1, min(_log(rng, 1, 16), MOST_ATTENTION // (H * n * L * dh)))
        return mha_case(batch, H, n, dh, L, E=rng.choice([16, 16, 8]), train=rng.random() < 0.75)
    wide = rng.random() < 0.35
    d = 64 * _log(rng, 4, 64)
    if wide:
        Bs, N = 32 * _log(rng, 16, 86), rng.randint(4, 8)
        k = max(1, round(N * rng.uniform(0.4, 0.75)))
    else:
        Bs, N = rng.choice([64, 96, 128, 128]), _log(rng, 16, 128)
        k = max(1, round(N * rng.uniform(0.2, 0.5)))
    while N * Bs * d > MOST_WEIGHT:
        d = max(256, d // 128 * 64)
    T = _log(rng, 1, 8192) if kind == "infer" else _log(rng, 300, 16384)
    T = max(1, min(T, MOST_FLOP // (12 * d * k * Bs)))
    balance = kind == "train" and rng.random() < 0.4
    return ffn_case(kind, T, d, N, Bs, k, act=rng.choice(["gelu", "relu"]), skew=rng.random() < 0.25,
                    abs_logit=not balance and rng.random() < 0.2, balance=balance,
                    rank=rng.choice([4, 8, 16, 32, rng.randint(1, 32)]) if kind == "lora" else 0)


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _prepare_mha(c, seed):
    g = _generator(seed)
    S, n, dh, L, M, E = c["batch"] * c["H"], c["n"], c["dh"], c["L"], c["dh"] // 8, c["E"]
    normal = lambda: torch.randn(S, n, dh, generator=g, device="cuda")
    K, V, dY = normal(), normal().to(BF16), normal().to(BF16)
    pick = torch.randint(0, n, (S, n, 1), generator=g, device="cuda")
    # a query is an even mix of a key of its own sequence and noise
    Q = (0.7071 * (torch.gather(K, 1, pick.expand(-1, -1, dh)) + normal())).to(BF16)
    K = K.to(BF16)
    # the codebooks of a head: sub-vectors of its keys
    rows = torch.randint(0, n, (c["H"], M, E), generator=g, device="cuda")
    heads = torch.arange(c["H"], device="cuda")[:, None, None]
    C = K[: c["H"]].view(c["H"], n, M, 8)[heads, rows, torch.arange(M, device="cuda")[None, :, None]].float().contiguous()
    empty = lambda *shape, dtype=BF16: torch.empty(shape, dtype=dtype, device="cuda")
    shape = mha.make_shape(S, c["H"], n, dh, L, E=E, scale=dh ** -0.5)
    s = dict(kind="mha", train=c["train"], shape=shape, Q=Q, K=K, V=V, dY=dY, C=C,
             cq=empty(S, n, M, dtype=U8), ck=empty(S, n, M, dtype=U8), idx=empty(S, n, L, dtype=I32),
             A=empty(S, n, L, dtype=F32), Y=empty(S, n, dh))
    if c["train"]:
        s.update(dQ=empty(S, n, dh), dK=empty(S, n, dh), dV=empty(S, n, dh), ws=mha.alloc_workspace(shape))
    return s


def prepare(case, seed):
    if case["kind"] == "mha":
        return _prepare_mha(case, seed)
    g = _generator(seed)
    kind, T, d, N, Bs, k, r = (case[x] for x in ("kind", "T", "d", "N", "Bs", "k", "rank"))
    P, D = T * k, N * Bs
    normal = lambda *shape, std=1.0, dtype=BF16: (torch.randn(*shape, generator=g, device="cuda") * std).to(dtype)
    empty = lambda *shape, dtype=BF16: torch.empty(shape, dtype=dtype, device="cuda")
    shape = spt.make_shape(T, d, N, Bs, k, spt.ACT_GELU if case["act"] == "gelu" else spt.ACT_RELU,
                           spt.FLAG_ABS_LOGIT if case["abs_logit"] else 0)
    s = dict(kind=kind, shape=shape, rank=r, balance=case["balance"],
             X=normal(T, d), W1=normal(N, Bs, d, std=0.02), W2=normal(N, Bs, d, std=0.02),
             W_r=normal(d, N, std=0.02, dtype=F32),
             b_r=torch.from_numpy(inputs.zipf_block_bias(N, seed)).cuda() if case["skew"] else None,
             idx=empty(T, k, dtype=I32), offsets=empty(N + 1, dtype=I32), perm=empty(P, dtype=I32),
             inv=empty(P, dtype=I32), Y=empty(T, d), logits=empty(T, N, dtype=F32) if case["balance"] else None,
             ws_router=spt.alloc_workspace(shape, spt.WS_ROUTER), ws_bucket=spt.alloc_workspace(shape, spt.WS_BUCKET))
    if kind != "infer":
        s.update(dY=normal(T, d), Hsave=empty(P, Bs), dX=empty(T, d))
    if kind == "lora":
        s.update(adapters=[normal(d, r, std=0.02), normal(r, D, std=0.02), normal(D, r, std=0.02), normal(r, d, std=0.02)],
                 grads=[empty(d, r, dtype=F32), empty(r, D, dtype=F32), empty(D, r, dtype=F32), empty(r, d, dtype=F32)])
        which = (spt.WS_LORA_FWD, spt.WS_LORA_BWD)
    elif kind == "train":
        s.update(dW1=empty(N, Bs, d, dtype=F32), dW2=empty(N, Bs, d, dtype=F32),
                 sched=spt.alloc_workspace(shape, spt.WS_SCHEDULE))
        which = (spt.WS_FWD, spt.WS_BWD)
    else:
        which = (spt.WS_FWD,)
    s["ws"] = spt.alloc_workspace(shape, max(which, key=lambda w: spt.workspace_bytes(shape, w)))
    if case["balance"]:
        s.update(loss=empty(1, dtype=F32), frac=empty(N, dtype=F32), dW_r=empty(d, N, dtype=F32), db_r=empty(N, dtype=F32),
                 ws_balance=spt.alloc_workspace(shape, spt.WS_BALANCE))
    return s


def _run_mha(s):
    sh = s["shape"]
    mha.pq_assign(sh, s["Q"], s["C"], s["cq"])
    mha.pq_assign(sh, s["K"], s["C"], s["ck"])
    mha.topl(sh, s["cq"], s["ck"], s["idx"])
    mha.attn_fwd(sh, s["Q"], s["K"], s["V"], s["idx"], s["A"], s["Y"])
    out = {x: s[x] for x in ("cq", "ck", "idx", "A", "Y")}
    if s["train"]:
        mha.attn_bwd(sh, s["Q"], s["K"], s["V"], s["dY"], s["idx"], s["A"], s["ws"], s["dQ"], s["dK"], s["dV"])
        out.update(dQ=s["dQ"], dK=s["dK"], dV=s["dV"])
    return out


def run(s):
    kind = s["kind"]
    if kind == "mha":
        return _run_mha(s)
    sh = s["shape"]
    spt.router_topk(sh, s["X"], s["W_r"], s["b_r"], idx=s["idx"], logits=s["logits"], ws=s["ws_router"])
    spt.bucket_tokens(sh, s["idx"], ws=s["ws_bucket"], offsets=s["offsets"], perm=s["perm"], inv=s["inv"])
    routing = (s["offsets"], s["perm"], s["inv"])
    out = {x: s[x] for x in ("idx", "offsets", "perm", "inv", "Y")}
    if kind == "infer":
        spt.routed_ffn_fwd(sh, s["X"], s["W1"], s["W2"], *routing, ws=s["ws"], Y=s["Y"], save_for_backward=False)
        return out
    if kind == "lora":
        weights = (s["X"], s["W1"], s["W2"], *s["adapters"])
        spt.lora_ffn_fwd(sh, s["rank"], *weights, *routing, ws=s["ws"], Y=s["Y"], Hsave=s["Hsave"])
        spt.lora_ffn_bwd(sh, s["rank"], *weights, s["dY"], *routing, s["Hsave"], s["ws"], s["dX"], *s["grads"])
        out.update(Hsave=s["Hsave"], dX=s["dX"], dA1=s["grads"][0], dC1=s["grads"][1], dB2=s["grads"][2], dC2=s["grads"][3])
        return out
    spt.build_schedule(sh, s["offsets"], s["perm"], sched=s["sched"])
    spt.routed_ffn_fwd(sh, s["X"], s["W1"], s["W2"], *routing, ws=s["ws"], Y=s["Y"], Hsave=s["Hsave"], sched=s["sched"])
    spt.routed_ffn_bwd(sh, s["X"], s["W1"], s["W2"], s["dY"], *routing, s["Hsave"], ws=s["ws"], dX=s["dX"],
                       dW1=s["dW1"], dW2=s["dW2"], sched=s["sched"])
    out.update(Hsave=s["Hsave"], dX=s["dX"], dW1=s["dW1"], dW2=s["dW2"])
    if s["balance"]:
        spt.router_balance(sh, s["X"], s["logits"], s["offsets"], ws=s["ws_balance"], loss=s["loss"], frac=s["frac"],
                           dW_r=s["dW_r"], db_r=s["db_r"])
        out.update(logits=s["logits"], loss=s["loss"], frac=s["frac"], dW_r=s["dW_r"], db_r=s["db_r"])
    return out


def work(case):
    if case["kind"] == "mha":
        S, n, dh, L, M, E = case["batch"] * case["H"], case["n"], case["dh"], case["L"], case["dh"] // 8, case["E"]
        rows = S * n
        entries, row = rows * L, rows * dh * 2
        # distances of queries and keys to E codewords; two products forward, four backward
        flops = 2 * rows * M * E * 8 * 3 + (12 if case["train"] else 4) * entries * dh
        # Q, K, V (dY) in; codes, idx, A, Y (dQ, dK, dV) out
        size = (8 if case["train"] else 4) * row + case["H"] * M * E * 8 * 4 + 2 * rows * M + 8 * entries
        return {"bytes": size, "flops": flops}
    kind, T, d, N, Bs, k, r = (case[x] for x in ("kind", "T", "d", "N", "Bs", "k", "rank"))
    P, D = T * k, N * Bs
    gemm = 2 * P * Bs * d
    used = min(N, P) * Bs * d * 2                 # a weight tensor, of no more blocks than there are pairs
    size = T * d * 2 + d * N * 4 + 2 * used + 12 * P + 4 * N + T * d * 2        # X, W_r, W1, W2; idx, offsets, perm, inv, Y
    flops = 2 * T * d * N + 2 * gemm
    if kind != "infer":
        size += 2 * T * d * 2 + P * Bs * 2        # dY, dX, Hsave
        flops += 2 * gemm
    if kind == "train":
        size += 2 * D * d * 4
        flops += 2 * gemm
    if kind == "lora":
        # forward U = X A1, U C1 and H B2, V C2; backward the same products transposed and the four gradients
        flops += 3 * (2 * 2 * T * d * r + 2 * 2 * P * Bs * r)
        size += (2 + 4) * 2 * (d * r + D * r)
    if case["balance"]:
        flops += 2 * T * d * N
        size += T * N * 4 + d * N * 4
    return {"bytes": size, "flops": flops}


def tolerance(case):
    if case["kind"] == "mha":
        # A code may differ where two codewords are equally near to within 32-bit rounding of the distance, and
        # moves its key in a few rows of the selection; the rest is bf16 in, 32-bit sums, bf16 out.
        return {"rel": 1e-2, "max": 0.5, "differ": 1e-3}
    # Routing is whole numbers and stays the same; values are bf16 tensors with 32-bit sums, and the
    # 32-bit gradients are sums of products of hidden values that were rounded to bf16.
    return {"rel": 1e-2, "max": 0.5}
