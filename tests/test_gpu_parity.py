"""GPU parity: every stage of the HIP path, called through the C ABI, against the fp64
oracle on the same seeded inputs.

Bars: routing indices, offsets, perm, inv bit-exact (tokens whose top-k margin is below
1e-6 are reported, not failed); Y, dX, Hsave, dW1, dW2 within 1e-2 relative Frobenius error AND
every row (token / pair / hidden unit) within 3e-2 of its own norm (parity_util.py); the largest
absolute error is printed.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2312_10365_amd import inputs as gen
from paper_2312_10365_amd import spt
from parity_util import check

pytestmark = pytest.mark.gpu

MARGIN = 1e-6       # top-k margin below which a routing difference is reported, not failed


class Dev:
    """Inputs of one workload resident on the GPU."""

    def __init__(self, inp):
        s = inp.shape
        self.inp, self.s = inp, s
        self.shape = spt.make_shape(s.T, s.d, s.N, s.Bs, s.k, s.act, s.flags)
        self.X = spt.bf16_tensor_from_bits(inp.X_bits)
        self.W1 = spt.bf16_tensor_from_bits(inp.W1_bits)
        self.W2 = spt.bf16_tensor_from_bits(inp.W2_bits)
        self.dY = spt.bf16_tensor_from_bits(inp.dY_bits)
        self.W_r = torch.from_numpy(inp.W_r).cuda()
        self.b_r = None if inp.b_r is None else torch.from_numpy(inp.b_r).cuda()


def check_routing(dv, tag):
    s, inp = dv.s, dv.inp
    logits = torch.empty((s.T, s.N), dtype=torch.float32, device="cuda")
    idx = spt.router_topk(dv.shape, dv.X, dv.W_r, dv.b_r, logits=logits)
    torch.cuda.synchronize()
    g_idx = idx.cpu().numpy()
    o_idx, margin, L = oracle.route(inp.f32("X"), inp.W_r, inp.b_r, s.k, s.flags)
    # fp32 logits: an fp64 sum rounded once.  The GPU adds the exact products in another order,
    # which moves the fp64 sum by parts in 1e-16, so the fp32 values must agree except where the
    # fp64 sum sits on a rounding boundary (then: adjacent fp32 values, and very rarely).
    lg, ref = logits.cpu().numpy(), L.astype(np.float32)
    diff = lg != ref
    assert diff.mean() <= 1e-5, f"{tag}: {int(diff.sum())} logits differ"
    if diff.any():
        print(f"[report] {tag}: {int(diff.sum())} logits sit on an fp32 rounding boundary")
        mid = 0.5 * (lg[diff].astype(np.float64) + ref[diff].astype(np.float64))
        assert np.all(np.abs(L[diff] - mid) <= 1e-12 * np.maximum(1.0, np.abs(L[diff])))
        assert np.all((np.nextafter(ref[diff], lg[diff]) == lg[diff]))
    near = margin < MARGIN
    bad = np.any(g_idx != o_idx, axis=1)
    if np.any(bad & near):
        print(f"[report] {tag}: {int(np.sum(bad & near))} near-tie tokens (margin < {MARGIN}) differ")
    assert not np.any(bad & ~near), f"{tag}: routing differs on {int(np.sum(bad & ~near))} clear tokens"
    print(f"[report] {tag}: {int(near.sum())} tokens with top-k margin < {MARGIN}")
    # ids ascending and distinct
    assert np.all(np.diff(g_idx, axis=1) > 0)
    return idx, g_idx, o_idx


def check_bucket(dv, idx, g_idx, tag):
    s = dv.s
    neg = lambda n: torch.full((n,), -1, dtype=torch.int32, device="cuda")
    offsets, perm, inv = spt.bucket_tokens(dv.shape, idx, offsets=neg(s.N + 1), perm=neg(s.P), inv=neg(s.P))
    torch.cuda.synchronize()
    o_off, o_perm, o_inv = oracle.bucket(g_idx, s.N)
    assert np.array_equal(offsets.cpu().numpy(), o_off), f"{tag}: offsets"
    assert np.array_equal(perm.cpu().numpy(), o_perm), f"{tag}: perm"
    assert np.array_equal(inv.cpu().numpy(), o_inv), f"{tag}: inv"
    return offsets, perm, inv, (o_off, o_perm, o_inv)


def run_gpu_ffn(dv, offsets, perm, inv):
    """Outputs are handed over pre-filled with NaN, so an element the kernels fail to write
    cannot pass for a value (fresh device memory is often zero)."""
    s = dv.s
    nan16 = lambda *shape: torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    nan32 = lambda *shape: torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    Y, Hsave = spt.routed_ffn_fwd(dv.shape, dv.X, dv.W1, dv.W2, offsets, perm, inv,
                                  Y=nan16(s.T, s.d), Hsave=nan16(s.P, s.Bs))
    dX, dW1, dW2 = spt.routed_ffn_bwd(dv.shape, dv.X, dv.W1, dv.W2, dv.dY, offsets, perm, inv, Hsave,
                                      dX=nan16(s.T, s.d), dW1=nan32(s.N, s.Bs, s.d), dW2=nan32(s.N, s.Bs, s.d))
    torch.cuda.synchronize()
    for name, t in (("Y", Y), ("Hsave", Hsave), ("dX", dX), ("dW1", dW1), ("dW2", dW2)):
        assert not torch.isnan(t).any(), f"{name}: elements left unwritten"
    return Y, Hsave, dX, dW1, dW2


def full_parity(s, tag=None):
    tag = tag or s.name
    inp = gen.make_inputs(s)
    dv = Dev(inp)
    idx, g_idx, _ = check_routing(dv, tag)
    offsets, perm, inv, (o_off, o_perm, o_inv) = check_bucket(dv, idx, g_idx, tag)
    Y, Hsave, dX, dW1, dW2 = run_gpu_ffn(dv, offsets, perm, inv)
    a = (inp.f32("X"), inp.f32("W1"), inp.f32("W2"))
    # the oracle is fed the GPU's routing, so a near-tie token cannot contaminate values
    oY, oH = oracle.ffn_fwd(*a, g_idx, s.act)
    odX, _ = oracle.ffn_bwd_dx(*a, inp.f32("dY"), g_idx, s.act)
    odW1, odW2 = oracle.ffn_bwd_dw(*a, inp.f32("dY"), g_idx, s.act)
    check(tag, "Hsave", Hsave.float().cpu().numpy(), oracle.to_bucket_order(oH, o_perm))
    check(tag, "Y", Y.float().cpu().numpy(), oY)
    check(tag, "dX", dX.float().cpu().numpy(), odX)
    check(tag, "dW1", dW1.cpu().numpy(), odW1)
    check(tag, "dW2", dW2.cpu().numpy(), odW2)
    # blocks nobody activates get exactly zero gradients
    unused = np.setdiff1d(np.arange(s.N), np.unique(g_idx))
    if unused.size:
        assert not dW1[torch.from_numpy(unused).cuda()].any()
        assert not dW2[torch.from_numpy(unused).cuda()].any()
    return dv, (offsets, perm, inv), (Y, Hsave, dX, dW1, dW2)


@pytest.mark.parametrize("name", ["tiny", "bert_base"])
def test_small_presets_full_parity(name):
    full_parity(gen.PRESETS[name])


@pytest.mark.parametrize("dims", [
    # (T, d, N, Bs, k): ragged tails, buckets smaller than a tile, k == N, one token
    (300, 192, 5, 96, 2),
    (1, 64, 3, 32, 1),
    (129, 128, 4, 32, 4),
    (517, 320, 9, 160, 3),
    (260, 64, 70, 32, 7),
    (96, 64, 1024, 32, 40),       # the largest N the library accepts: most buckets hold a few rows or none
    # blocks wider than 128 units (the 256 x 256-tile kernels): unit tiles with a ragged tail,
    # d not a multiple of 256, one block only, k == N, buckets of a few rows
    (700, 448, 3, 288, 2),
    (64, 64, 2, 512, 1),
    (1000, 256, 5, 160, 5),
    (33, 128, 4, 192, 2),
    (300, 576, 1, 1056, 1),
])
@pytest.mark.parametrize("act", [spt.ACT_GELU, spt.ACT_RELU])
def test_ragged_shapes_full_parity(dims, act):
    T, d, N, Bs, k = dims
    s = gen.custom_shape(T, d, N, Bs, k, seed=T + N, act=act, w_std=0.05, wr_std=0.05)
    full_parity(s)


@pytest.mark.parametrize("dims", [
    # (T, d, N, Bs, k): two thousand (column tile, block) work items of the weight-gradient GEMM, a dozen rows each; 64- and
    # 128-unit tiles
    (600, 512, 1024, 32, 20),
    (500, 512, 1024, 96, 24),
])
def test_many_blocks(dims):
    T, d, N, Bs, k = dims
    s = gen.custom_shape(T, d, N, Bs, k, seed=T + N, w_std=0.05, wr_std=0.05)
    full_parity(s)


def test_many_blocks_with_a_split_bucket():
    # as many with one block drawn by every token: its bucket (900 rows) is cut into pieces that go through the staging slots and
    # the fixed-order sum
    T, d, N, Bs, k = 900, 512, 1024, 32, 12
    s = gen.custom_shape(T, d, N, Bs, k, seed=T + N, zipf_bias=True, w_std=0.05, wr_std=0.01)
    dv, (offsets, _, _), _ = full_parity(s, f"skewed, many blocks T={T} N={N} k={k}")
    sizes = np.diff(offsets.cpu().numpy())
    assert sizes.max() > 2 * 256, "the case is meant to have a bucket of more than two pieces"


@pytest.mark.parametrize("dims", [
    # (T, d, N, Bs, k): one block drawn by nearly every token, so its bucket is several times the
    # mean and the weight-gradient GEMMs cut it into pieces whose products are added in order
    (3000, 128, 8, 64, 2),
    (1500, 64, 4, 128, 1),
    (5000, 192, 32, 32, 3),
])
def test_skewed_buckets_split_weight_gradients(dims):
    T, d, N, Bs, k = dims
    s = gen.custom_shape(T, d, N, Bs, k, seed=T + N, zipf_bias=True, w_std=0.05, wr_std=0.01)
    dv, (offsets, _, _), _ = full_parity(s, f"skewed T={T} N={N} k={k}")
    sizes = np.diff(offsets.cpu().numpy())
    piece = max(256, (3 * s.P // N + 1) // 2)
    assert sizes.max() > 2 * piece, "the case is meant to have a bucket of more than two pieces"


@pytest.mark.parametrize("dims", [(700, 192, 12, 96, 3), (300, 256, 3, 288, 2)])   # narrow and wide blocks
def test_schedule_built_once_gives_identical_results(dims):
    """spt_build_schedule + the _sched entry points against the plain calls: bit for bit, also when
    the one buffer serves both calls twice over and the workspaces hold stale contents."""
    T, d, N, Bs, k = dims
    s = gen.custom_shape(T, d, N, Bs, k, seed=T + N, w_std=0.05, wr_std=0.05)
    dv = Dev(gen.make_inputs(s))
    idx = spt.router_topk(dv.shape, dv.X, dv.W_r, dv.b_r)
    offsets, perm, inv = spt.bucket_tokens(dv.shape, idx)
    ref = run_gpu_ffn(dv, offsets, perm, inv)
    sched = spt.build_schedule(dv.shape, offsets, perm)
    ws = spt.alloc_workspace(dv.shape, spt.WS_BWD)
    for _ in range(2):
        ws.fill_(0x5A)
        Y, Hsave = spt.routed_ffn_fwd(dv.shape, dv.X, dv.W1, dv.W2, offsets, perm, inv, ws=ws, sched=sched)
        ws.fill_(0xA5)
        dX, dW1, dW2 = spt.routed_ffn_bwd(dv.shape, dv.X, dv.W1, dv.W2, dv.dY, offsets, perm, inv, Hsave, ws=ws,
                                          sched=sched)
        torch.cuda.synchronize()
        for name, a, b in zip(("Y", "Hsave", "dX", "dW1", "dW2"), (Y, Hsave, dX, dW1, dW2), ref):
            assert torch.equal(a, b), f"{name} differs with a prebuilt schedule"


def test_abs_logit_routing_and_bias():
    s = gen.custom_shape(400, 128, 12, 32, 5, seed=77, flags=spt.FLAG_ABS_LOGIT, zipf_bias=True, wr_std=0.1)
    full_parity(s, "abs_logit+bias")


def test_empty_buckets_get_zero_gradients():
    # A strongly negative bias on two blocks leaves their buckets empty.
    s = gen.custom_shape(256, 128, 8, 64, 3, seed=5, wr_std=0.05)
    inp = gen.make_inputs(s)
    b = np.zeros(s.N, dtype=np.float32)
    b[[2, 7]] = -100.0
    inp.b_r = b
    dv = Dev(inp)
    idx, g_idx, _ = check_routing(dv, "empty")
    assert 2 not in g_idx and 7 not in g_idx
    offsets, perm, inv, _ = check_bucket(dv, idx, g_idx, "empty")
    Y, Hsave, dX, dW1, dW2 = run_gpu_ffn(dv, offsets, perm, inv)
    assert not dW1[2].any() and not dW1[7].any() and not dW2[2].any() and not dW2[7].any()
    a = (inp.f32("X"), inp.f32("W1"), inp.f32("W2"))
    oY, _ = oracle.ffn_fwd(*a, g_idx)
    check("empty buckets", "Y", Y.float().cpu().numpy(), oY)


def test_router_many_blocks_and_ties():
    # N > 64 * 2 exercises several blocks per lane; duplicated W_r columns force exact ties.
    s = gen.custom_shape(200, 64, 300, 32, 17, seed=9, wr_std=0.1)
    inp = gen.make_inputs(s)
    inp.W_r[:, 100:200] = inp.W_r[:, 0:100]          # exact ties between b and b+100
    dv = Dev(inp)
    check_routing(dv, "ties")
    # all-zero router: every key ties, blocks 0..k-1 win
    inp.W_r[:] = 0.0
    dv = Dev(inp)
    _, g_idx, _ = check_routing(dv, "all-tie")
    assert np.array_equal(g_idx, np.tile(np.arange(s.k, dtype=np.int32), (s.T, 1)))


# Many tokens, ids only: fp32 sums decide where they can, fp64 ones the rest.  The ids are those of the fp64 logits, whatever is
# close: edges of the token tiles (128), of the column tiles (32), of d's parts and stages (64, 128), first, last and
# every block selected; blocks with the same weights, tokens of zeros, tokens and weights whose squares underflow.
@pytest.mark.parametrize("T,d,N,k", [(16385, 320, 64, 16), (17000, 640, 33, 33), (40001, 64, 120, 7), (1537, 4096, 128, 127),
                                     (12500, 832, 65, 1), (4096, 2048, 96, 48)])
@pytest.mark.parametrize("kind", ["plain", "bias, magnitude", "twins", "zeros", "tiny"])
def test_router_ids_of_many_tokens(T, d, N, k, kind):
    g = torch.Generator(device="cuda").manual_seed(T + d)
    X = torch.randn(T, d, generator=g, device="cuda")
    W = 0.02 * torch.randn(d, N, generator=g, device="cuda")
    b = 3.0 * torch.randn(N, generator=g, device="cuda") if kind == "bias, magnitude" else None
    if kind == "twins":
        W[:, 1::2] = W[:, 0:N - 1:2]
    if kind in ("zeros", "tiny"):
        X[::3] = 0.0
    if kind == "tiny":
        X[1::3] *= 1e-22
        W *= 1e-10
    X = X.bfloat16()
    s = spt.make_shape(T, d, N, 32, k, spt.ACT_GELU, spt.FLAG_ABS_LOGIT if b is not None else 0)
    assert spt.alloc_workspace(s, spt.WS_ROUTER).nbytes >= 4 * (N * d + T * N)     # (the sums and the weights' copy)
    logits = torch.empty(T, N, device="cuda")
    want = spt.router_topk(s, X, W, b, logits=logits)            # (the fp64 kernels)
    got = spt.router_topk(s, X, W, b)
    exact = X[:2048].double() @ W.double() + (0.0 if b is None else b.double())
    torch.cuda.synchronize()
    assert torch.allclose(logits[:2048].double(), exact, rtol=1e-7, atol=1e-30)
    assert torch.equal(got, want), int((got != want).any(1).sum())


# Data that leaves many blocks open to fp64 sums, up to all of them: a large part common to all weights (few tokens of a
# workgroup's sixteen over its limit to all of them), blocks alike, infinite values in half of the tokens or one in 37.
@pytest.mark.parametrize("T,d,N,k", [(16385, 320, 64, 16), (131107, 64, 33, 5), (12500, 832, 65, 1), (4099, 2048, 128, 40)])
@pytest.mark.parametrize("kind", ["common 30", "common 300", "common 3000", "alike", "half infinite", "few infinite"])
def test_router_ids_where_many_blocks_are_close(T, d, N, k, kind):
    g = torch.Generator(device="cuda").manual_seed(T + d)
    X = torch.randn(T, d, generator=g, device="cuda")
    W = 0.02 * torch.randn(d, N, generator=g, device="cuda")
    b = 0.1 * torch.randn(N, generator=g, device="cuda") if kind == "few infinite" else None
    if kind.startswith("common"):
        W += float(kind.split()[1]) * 0.02 * torch.randn(d, 1, generator=g, device="cuda")
    if kind == "alike":
        W[:] = W[:, :1].clone()
    if kind.endswith("infinite"):
        X[::2 if kind == "half infinite" else 37, 5] = float("inf")
    X = X.bfloat16()
    s = spt.make_shape(T, d, N, 32, k, spt.ACT_GELU, 0)
    assert spt.alloc_workspace(s, spt.WS_ROUTER).nbytes >= 4 * (N * d + T * N)     # (the sums and the weights' copy)
    want = spt.router_topk(s, X, W, b, logits=torch.empty(T, N, device="cuda"))      # (the fp64 kernels)
    got = spt.router_topk(s, X, W, b)
    torch.cuda.synchronize()
    assert torch.equal(got, want), int((got != want).any(1).sum())


# ... and ids alone take no more than two and a half times as long as all sums in fp64 do (1.4 to 1.9 measured).
@pytest.mark.parametrize("T,d,N,k", [(8192, 4096, 128, 32), (40000, 256, 128, 32), (16384, 1024, 64, 16)])
def test_router_time_does_not_hang_on_the_data(T, d, N, k):
    g = torch.Generator(device="cuda").manual_seed(T + d)
    X = torch.randn(T, d, generator=g, device="cuda").bfloat16()
    W = (0.02 * torch.randn(d, 1, generator=g, device="cuda")).repeat(1, N)
    s = spt.make_shape(T, d, N, 32, k, spt.ACT_GELU, 0)
    ws, idx, logits = spt.alloc_workspace(s, spt.WS_ROUTER), torch.empty(T, k, dtype=torch.int32, device="cuda"), torch.empty(T, N, device="cuda")

    def us(**out):
        best = float("inf")
        for _ in range(5):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            for _ in range(5):
                spt.router_topk(s, X, W, idx=idx, ws=ws, **out)
            end.record()
            torch.cuda.synchronize()
            best = min(best, 200.0 * start.elapsed_time(end))
        return best

    fp64, ids = us(logits=logits), us()
    print(f"[router, all blocks alike] {(T, d, N)}: fp64 {fp64:.1f} us, ids only {ids:.1f} us")
    assert ids <= 2.5 * fp64


def test_values_with_oracle_bucketing_and_determinism():
    # Feed the oracle's offsets/perm/inv to the GPU (value parity decoupled from routing),
    # and require bit-identical outputs on a second run.
    s = gen.PRESETS["tiny"]
    inp = gen.make_inputs(s)
    dv = Dev(inp)
    o_idx, _, _ = oracle.route(inp.f32("X"), inp.W_r, None, s.k)
    o_off, o_perm, o_inv = oracle.bucket(o_idx, s.N)
    off, perm, inv = (torch.from_numpy(v).cuda() for v in (o_off, o_perm, o_inv))
    r1 = run_gpu_ffn(dv, off, perm, inv)
    r2 = run_gpu_ffn(dv, off, perm, inv)
    for x, y in zip(r1, r2):
        assert torch.equal(x, y)
    a = (inp.f32("X"), inp.f32("W1"), inp.f32("W2"))
    oY, oH = oracle.ffn_fwd(*a, o_idx)
    odX, _ = oracle.ffn_bwd_dx(*a, inp.f32("dY"), o_idx)
    odW1, odW2 = oracle.ffn_bwd_dw(*a, inp.f32("dY"), o_idx)
    check("tiny, oracle's bucketing", "Y", r1[0].float().cpu().numpy(), oY)
    check("tiny, oracle's bucketing", "Hsave", r1[1].float().cpu().numpy(), oracle.to_bucket_order(oH, o_perm))
    check("tiny, oracle's bucketing", "dX", r1[2].float().cpu().numpy(), odX)
    check("tiny, oracle's bucketing", "dW1", r1[3].cpu().numpy(), odW1)
    check("tiny, oracle's bucketing", "dW2", r1[4].cpu().numpy(), odW2)


def test_inference_forward_without_hsave():
    s = gen.PRESETS["tiny"]
    inp = gen.make_inputs(s)
    dv = Dev(inp)
    idx = spt.router_topk(dv.shape, dv.X, dv.W_r)
    offsets, perm, inv = spt.bucket_tokens(dv.shape, idx)
    Y1, _ = spt.routed_ffn_fwd(dv.shape, dv.X, dv.W1, dv.W2, offsets, perm, inv)
    Y2, H2 = spt.routed_ffn_fwd(dv.shape, dv.X, dv.W1, dv.W2, offsets, perm, inv, save_for_backward=False)
    torch.cuda.synchronize()
    assert H2 is None and torch.equal(Y1, Y2)


# --------------------------------------------------------------------------- full sizes
def sampled_parity(name, n_tok=512, n_blk=8, n_units=None, oracle_bucketing=False):
    """At the benchmark's full sizes the oracle computes sampled outputs one by one:
    whole tokens for Y/dX (n_tok of them, 512 by default), whole blocks for dW1/dW2 (n_blk of
    them, 8 by default, the largest and the smallest bucket always among them) -- or, for
    blocks thousands of units wide, n_units sampled hidden units of each sampled block: a unit's
    weight-gradient rows depend only on its own rows of W1 and W2, so the oracle is simply given
    those rows as a block of n_units; routing and bucketing in full.
    With oracle_bucketing the GPU runs on the ORACLE's offsets / perm / inv (its own routing of
    the same inputs), so the value comparison cannot be touched by a near-tie token."""
    s = gen.PRESETS[name]
    inp = gen.make_inputs(s)
    dv = Dev(inp)
    idx, g_idx, o_idx = check_routing(dv, name)
    offsets, perm, inv, (o_off, o_perm, o_inv) = check_bucket(dv, idx, g_idx, name)
    if oracle_bucketing:
        o_off, o_perm, o_inv = oracle.bucket(o_idx, s.N)
        offsets, perm, inv = (torch.from_numpy(v).cuda() for v in (o_off, o_perm, o_inv))
        g_idx = o_idx
    Y, Hsave, dX, dW1, dW2 = run_gpu_ffn(dv, offsets, perm, inv)
    rng = np.random.default_rng(s.seed)
    n_tok = min(n_tok, s.T)
    tok = np.sort(rng.choice(s.T, n_tok, replace=False)).astype(np.int32)
    sizes = np.diff(offsets.cpu().numpy())
    extra = rng.choice(s.N, min(s.N, n_blk), replace=False).tolist()
    blk = [int(np.argmax(sizes)), int(np.argmin(sizes))]
    for b in extra:
        if len(blk) >= min(n_blk, s.N):
            break
        if b not in blk:
            blk.append(int(b))
    blk = np.array(sorted(set(blk)), dtype=np.int32)
    a = (inp.f32("X"), inp.f32("W1"), inp.f32("W2"))
    oY, oH = oracle.ffn_fwd(*a, g_idx, s.act, tokens=tok)
    odX, _ = oracle.ffn_bwd_dx(*a, inp.f32("dY"), g_idx, s.act, tokens=tok)
    tk = torch.from_numpy(tok.astype(np.int64)).cuda()
    bk = torch.from_numpy(blk.astype(np.int64)).cuda()
    if n_units is None:
        odW1, odW2 = oracle.ffn_bwd_dw(*a, inp.f32("dY"), g_idx, s.act, blocks=blk)
    else:
        units = np.sort(np.concatenate([[0, s.Bs - 1],
                                        rng.choice(np.arange(1, s.Bs - 1), n_units - 2, replace=False)]))
        sub = (a[0], np.ascontiguousarray(a[1][:, units, :]), np.ascontiguousarray(a[2][:, units, :]))
        odW1, odW2 = oracle.ffn_bwd_dw(*sub, inp.f32("dY"), g_idx, s.act, blocks=blk)
        un = torch.from_numpy(units.astype(np.int64)).cuda()
        dW1, dW2 = dW1[:, un, :], dW2[:, un, :]
    inv_np = inv.cpu().numpy().reshape(s.T, s.k)
    rows = torch.from_numpy(inv_np[tok].reshape(-1).astype(np.int64)).cuda()
    tag = f"{name} ({n_tok} whole tokens, blocks {blk.tolist()}, bucket sizes {sizes.min()}..{sizes.max()}" + \
          (", oracle's bucketing)" if oracle_bucketing else ")")
    check(tag, "Hsave", Hsave[rows].float().cpu().numpy(), oH.reshape(-1, s.Bs))
    check(tag, "Y", Y[tk].float().cpu().numpy(), oY)
    check(tag, "dX", dX[tk].float().cpu().numpy(), odX)
    check(tag, "dW1", dW1[bk].cpu().numpy(), odW1)
    check(tag, "dW2", dW2[bk].cpu().numpy(), odW2)
    # properties that hold at any size
    assert torch.isfinite(Y.float()).all() and torch.isfinite(dX.float()).all()
    assert torch.isfinite(dW1).all() and torch.isfinite(dW2).all()


@pytest.mark.parametrize("name", ["bert_large", "opt_1p3b_skewed", "ffn_7b"])
def test_full_size_sampled_parity(name):
    sampled_parity(name)


def test_full_size_values_on_the_oracles_bucketing():
    """A large, skewed configuration run on the oracle's own offsets / perm / inv, all five
    outputs compared (sampled whole tokens and whole blocks)."""
    sampled_parity("opt_1p3b_skewed", oracle_bucketing=True)


@pytest.mark.parametrize("name", ["paper_opt2048_g4", "paper_opt2048_g8_b34", "paper_llama4096_g4",
                                  "paper_llama4096_g8"])
def test_paper_shapes_sampled_parity(name):
    """The paper's own block shapes (Table 2; 4 or 8 groups, half or three quarters active):
    blocks of 1024-2752 hidden units, not a multiple of 128 for the LLaMA block."""
    sampled_parity(name, n_tok=128, n_blk=2, n_units=64)


def test_step_replays_identically_from_a_hip_graph():
    """The four calls allocate nothing, never synchronise and enqueue only on the caller's
    stream, so a whole step can be captured into a HIP graph.  Every replay (with eager work
    and synchronisations in between) must reproduce the eager results bit for bit."""
    s = gen.PRESETS["bert_base"]
    inp = gen.make_inputs(s)
    dv = Dev(inp)
    P = s.P
    dev = dv.X.device
    i32 = lambda *sh: torch.full(sh, -1, dtype=torch.int32, device=dev)
    idx, offsets, perm, inv = i32(s.T, s.k), i32(s.N + 1), i32(P), i32(P)
    Y = torch.empty((s.T, s.d), dtype=torch.bfloat16, device=dev)
    Hsave = torch.empty((P, s.Bs), dtype=torch.bfloat16, device=dev)
    dX = torch.empty_like(Y)
    dW1 = torch.empty((s.N, s.Bs, s.d), dtype=torch.float32, device=dev)
    dW2 = torch.empty_like(dW1)
    ws_r = spt.alloc_workspace(dv.shape, spt.WS_ROUTER)
    ws_b = spt.alloc_workspace(dv.shape, spt.WS_BUCKET)
    ws = spt.alloc_workspace(dv.shape, spt.WS_BWD)

    def step():
        spt.router_topk(dv.shape, dv.X, dv.W_r, dv.b_r, idx=idx, ws=ws_r)
        spt.bucket_tokens(dv.shape, idx, ws=ws_b, offsets=offsets, perm=perm, inv=inv)
        spt.routed_ffn_fwd(dv.shape, dv.X, dv.W1, dv.W2, offsets, perm, inv, ws=ws, Y=Y, Hsave=Hsave)
        spt.routed_ffn_bwd(dv.shape, dv.X, dv.W1, dv.W2, dv.dY, offsets, perm, inv, Hsave, ws=ws,
                           dX=dX, dW1=dW1, dW2=dW2)

    outs = (idx, offsets, perm, inv, Y, Hsave, dX, dW1, dW2)
    step()
    torch.cuda.synchronize()
    eager = [t.clone() for t in outs]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        step()                      # warm up on the capture stream (function attributes etc.)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(3):
        for t in outs:
            if t.dtype == torch.int32:
                t.fill_(-1)
            else:
                t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for got, ref in zip(outs, eager):
            assert torch.equal(got, ref)
        step()                      # eager work between the replays
        torch.cuda.synchronize()


# Route network and bucketing at the edges of their launch rules: 16 / 32 blocks (selection fused into the
# logits kernel) and one more, few tokens with d split over workgroups (logits left to the workspace),
# 8192 pairs and one more token, a histogram table of more than 16384 counts, many blocks.
@pytest.mark.parametrize("T,d,N,k", [(1, 64, 1, 1), (17, 128, 16, 5), (130, 192, 17, 16), (65, 2048, 32, 9),
                                     (33, 64, 33, 2), (1, 4096, 128, 32), (50, 1024, 300, 7), (24, 4160, 64, 64),
                                     (1024, 64, 16, 8), (1025, 64, 16, 8), (2100, 64, 1024, 9), (3000, 128, 70, 3),
                                     (9000, 64, 40, 4)])
@pytest.mark.parametrize("flags", [0, spt.FLAG_ABS_LOGIT])
def test_routing_and_bucketing_launch_edges(T, d, N, k, flags):
    s = gen.custom_shape(T, d, N, 32, k, seed=T + N, flags=flags, zipf_bias=True, wr_std=0.2)
    dv = Dev(gen.make_inputs(s))
    tag = f"edges T{T} d{d} N{N} k{k} flags{flags}"
    idx, g_idx, _ = check_routing(dv, tag)
    idx2 = spt.router_topk(dv.shape, dv.X, dv.W_r, dv.b_r)      # logits in the workspace: other kernels, same ids
    assert torch.equal(idx, idx2), tag
    check_bucket(dv, idx, g_idx, tag)


# One workgroup's bucketing: words of 32 tokens, one to a block's lanes up to more than a wavefront has (1, 2, 3, 32, 33, 65
# words), blocks that fill a turn and one more.
@pytest.mark.parametrize("T,N,k", [(1, 65, 65), (32, 129, 9), (33, 1024, 40), (96, 33, 5), (1000, 16, 8), (1024, 17, 7),
                                   (1056, 8, 7), (2080, 5, 3), (4096, 2, 2)])
def test_bucketing_by_one_workgroup(T, N, k):
    s = gen.custom_shape(T, 64, N, 32, k, seed=T + k, zipf_bias=True, wr_std=0.2)
    dv = Dev(gen.make_inputs(s))
    idx, g_idx, _ = check_routing(dv, f"one workgroup T{T} N{N}")
    check_bucket(dv, idx, g_idx, f"one workgroup T{T} N{N}")


# ... with two, four and eight pairs a thread.
@pytest.mark.parametrize("T,N,k", [(2047, 3, 1), (2048, 3, 1), (683, 9, 3), (2048, 12, 2), (241, 40, 17), (8191, 2, 1)])
def test_bucketing_by_one_workgroup_pairs(T, N, k):
    test_bucketing_by_one_workgroup(T, N, k)


# Feed-forward kernels at the edges of their launch rules.
@pytest.mark.parametrize("dims", [
    # (T, d, N, Bs, k).  Up-projection of decoding batches: one row tile up to 24 rows a bucket, two beyond, 40 and 64
    # rows as the last ones, 64-row tiles after that; block list of the K = Bs kernel split over workgroups
    (1, 256, 40, 128, 3), (64, 192, 8, 64, 3), (65, 192, 8, 64, 3), (256, 64, 8, 96, 2), (257, 64, 8, 96, 2),
    (24, 1024, 64, 128, 16), (33, 320, 128, 32, 40),
    # 64-row tiles at 127 buckets, 256-row ones from 128; one, two, three stages of 64 values in rings of three and four
    (700, 64, 127, 32, 16), (700, 64, 128, 32, 16), (700, 128, 128, 96, 16), (700, 192, 130, 64, 16), (1100, 320, 64, 128, 24),
    # schedule by one workgroup up to 4096 pairs
    (1024, 64, 40, 32, 4), (4097, 64, 40, 32, 1), (1024, 64, 40, 32, 8), (2731, 64, 40, 32, 3),
    # wide blocks, items left over per XCD: as quarters, as halves, as whole tiles, after a full round
    (1300, 192, 2, 288, 2), (5000, 320, 2, 288, 2), (5000, 64, 2, 1056, 2), (5000, 64, 2, 1696, 2),
], ids=str)
def test_ffn_launch_edges(dims):
    T, d, N, Bs, k = dims
    full_parity(gen.custom_shape(T, d, N, Bs, k, seed=T + N, w_std=0.05, wr_std=0.05), f"edges {dims}")


# Wide blocks with ReLU, whose up-projection and dH write whole lines: whole tiles, halves and quarters of them; blocks
# that end in the middle of a line, one and two A-side tiles before the edge.
@pytest.mark.parametrize("dims", [(1300, 192, 2, 288, 2), (5000, 320, 2, 288, 2), (5000, 64, 2, 1056, 2), (700, 128, 3, 160, 2),
                                  (900, 64, 2, 608, 1)], ids=str)
def test_wide_blocks_write_whole_lines(dims):
    T, d, N, Bs, k = dims
    full_parity(gen.custom_shape(T, d, N, Bs, k, seed=T + N, act=spt.ACT_RELU, w_std=0.05, wr_std=0.05), f"lines {dims}")


@pytest.mark.parametrize("dims", [
    # (T, d, N, Bs, k, rows of a tile): few rows a bucket on average, most of them in one bucket of several row tiles; one
    # and two 32-row tiles at a time
    (700, 64, 64, 96, 1, 64), (3000, 64, 100, 32, 1, 64), (2400, 64, 130, 32, 1, 256), (4500, 64, 130, 64, 1, 256),
], ids=str)
def test_few_rows_a_bucket_but_for_one(dims):
    T, d, N, Bs, k, rows = dims
    s = gen.custom_shape(T, d, N, Bs, k, seed=T + N, zipf_bias=True, w_std=0.05, wr_std=0.05)
    _, (offsets, _, _), _ = full_parity(s, f"one large bucket {dims}")
    assert np.diff(offsets.cpu().numpy()).max() > 2 * rows, "the case is meant to have a bucket of more than two row tiles"


def routing_with_bucket_sizes(sizes, T, k):
    """idx[T, k] whose buckets have exactly these sizes (sum T k, none above T): every token takes the k fullest."""
    left = np.array(sizes)
    idx = np.empty((T, k), dtype=np.int32)
    for t in range(T):
        idx[t] = np.sort(np.argsort(-left, kind="stable")[:k])
        left[idx[t]] -= 1
    assert not left.any()
    return idx


# Row tiles of 256 rows and what is left of a round of them: whole buckets several XCDs share, bucket ends of up to 64 and 128
# rows, a last round cut into halves (10 tiles an XCD) and quarters (4), buckets without rows.
TILE_EDGES = [2048, 1700, 1500, 1025, 1024, 900, 769, 768, 640, 513, 512, 511, 400, 385, 384, 383, 330, 321, 320, 319, 300,
              257, 256, 255, 200, 193, 192, 191, 150, 129, 128, 127, 100, 65, 64, 63, 33, 32, 31, 1]


@pytest.mark.parametrize("Bs", [32, 64, 96, 128])
@pytest.mark.parametrize("sizes", [TILE_EDGES + [0] * 80 + [25] * 8, [300] * 128, [256] * 80 + [90] * 48, [256] * 32 + [40] * 96],
                         ids=["edges", "ends", "halves", "quarters"])
def test_row_tiles_of_a_last_round(sizes, Bs):
    k = 8
    sizes = list(sizes)
    sizes[-1] += -sum(sizes) % k
    check_sizes(sizes, k, Bs)


def check_sizes(sizes, k, Bs):
    N, T = len(sizes), sum(sizes) // k
    s = gen.custom_shape(T, 64, N, Bs, k, seed=N + Bs, act=spt.ACT_RELU if Bs == 64 else spt.ACT_GELU, w_std=0.1)
    inp = gen.make_inputs(s)
    dv = Dev(inp)
    g_idx = routing_with_bucket_sizes(sizes, T, k)
    offsets, perm, inv, (o_off, o_perm, o_inv) = check_bucket(dv, torch.from_numpy(g_idx).cuda(), g_idx, s.name)
    Y, Hsave, dX, dW1, dW2 = run_gpu_ffn(dv, offsets, perm, inv)
    a = (inp.f32("X"), inp.f32("W1"), inp.f32("W2"))
    oY, oH = oracle.ffn_fwd(*a, g_idx, s.act)
    odX, _ = oracle.ffn_bwd_dx(*a, inp.f32("dY"), g_idx, s.act)
    odW1, odW2 = oracle.ffn_bwd_dw(*a, inp.f32("dY"), g_idx, s.act)
    for name, got, ref in (("Hsave", Hsave, oracle.to_bucket_order(oH, o_perm)), ("Y", Y, oY), ("dX", dX, odX),
                           ("dW1", dW1, odW1), ("dW2", dW2, odW2)):
        check(s.name, name, got.float().cpu().numpy(), ref)
    return dv, offsets, perm


# The same with fewer than 16 blocks, whose tiles are one sequence over all buckets: no last round shorter than the CUs in whole tiles
# where parts take less.  Quarters and halves of 4, 5, 10 and 11 tiles an XCD, parts of a bucket's end without rows, an empty bucket, one bucket; 25
# tiles, which stay whole; a round of whole tiles, and one with a tile or two of the next.
@pytest.mark.parametrize("sizes,k,Bs,entries", [
    ([1537, 1700, 0, 2048, 1, 1100, 900, 1026], 2, 128, 4 * 37), ([2304] * 4, 1, 128, 4 * 36), ([9001], 1, 128, 4 * 36),
    ([1200, 1500, 1, 1700, 1264, 1280, 1345, 1300, 1290, 1400, 1320, 1408, 1000, 1409, 1413], 7, 96, 2 * 81),
    ([5001, 4000, 2047, 3000, 4096, 4200], 3, 64, 2 * 89), ([17000, 16641, 17001], 1, 32, 200), ([32768, 32768], 1, 32, 256),
    ([12000, 11000, 10001, 9999, 12001, 12801], 2, 32, 256 + 4 * 12)],
                         ids=["quarters", "even", "one", "halves", "ragged", "whole", "round", "after"])
def test_row_tiles_of_few_blocks(sizes, k, Bs, entries):
    dv, offsets, perm = check_sizes(sizes, k, Bs)
    at = (len(sizes) * 4 + 255) // 256 * 256                # the schedule: buckets by size, then each XCD's count of tiles
    counts = spt.build_schedule(dv.shape, offsets, perm).view(torch.uint8)[at:at + 32].view(torch.int32).cpu().numpy()
    assert counts.sum() == entries and counts.max() - counts.min() <= 4, counts
