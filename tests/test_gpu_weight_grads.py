"""Weight gradients with the gathered rows' token ids staged a group of stages ahead: bucket sizes around the 16- and
32-row stages, the groups (256 rows) and two of them, every tile width, narrow and wide blocks.

One block per token, so a block's bucket has exactly the rows asked for, its tokens scattered over the batch.  With ReLU the
operands of dW2 are max(Hsave, 0) and dY as they are: what may differ from a sum in 64 bits is the fp32 sum of K rows (each
product exact, each addition within 2^-24 of the sum of magnitudes, at most 2 sqrt(K) of them in the same direction).  dW1's
operand dHpre is rounded to bf16 first (within 2^-8 of each value, of which K independent ones add up to at most their sum)
after an fp32 sum of d products."""
import importlib.util
import os
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2312_10365_amd import spt
from scatter_shapes import JOINED

pytestmark = pytest.mark.gpu

SIZES = (0, 1, 15, 16, 17, 33, 96, 111, 255, 256, 257, 271, 287, 300, 511, 512, 513, 529, 545, 800)


# Narrow blocks cut a bucket of more than 1.5 times the mean (1120 rows here) into pieces of equal size: 2101 rows into two, 2777 into three of
# 926 and 925, which begin anywhere and have more stages (58 to 66 of 16 rows) than the ids of two groups hold.
PIECES = (37, 2101, 5, 700, 301, 2777, 0, 1)


@pytest.mark.parametrize("sizes,d,Bs", [(SIZES, 64, 64), (SIZES, 192, 32), (SIZES, 320, 96), (SIZES, 512, 128), (SIZES, 256, 160),
                                        (SIZES, 576, 288), (PIECES, 192, 32), (PIECES, 320, 96), (PIECES, 256, 160)], ids=str)
def test_bucket_sizes_around_the_groups(sizes, d, Bs):
    sizes = np.array(sizes)
    N, T = len(sizes), int(sizes.sum())
    rng = np.random.default_rng(d + Bs)
    block = rng.permutation(np.repeat(np.arange(N), sizes)).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(d + Bs)
    normal = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).to(torch.bfloat16)
    shape = spt.make_shape(T, d, N, Bs, 1, spt.ACT_RELU)
    X, dY, W1, W2 = normal(T, d), normal(T, d), normal(N, Bs, d, std=0.05), normal(N, Bs, d, std=0.05)
    print(f"d {d} Bs {Bs} T {T}", flush=True)
    offsets, perm, inv = spt.bucket_tokens(shape, torch.from_numpy(block[:, None]).cuda())
    _, H = spt.routed_ffn_fwd(shape, X, W1, W2, offsets, perm, inv)
    _, dW1, dW2 = spt.routed_ffn_bwd(shape, X, W1, W2, dY, offsets, perm, inv, H)
    torch.cuda.synchronize()
    x, dy, w2, h, pos = X.double().cpu(), dY.double().cpu(), W2.double().cpu(), H.double().cpu(), inv.view(-1).long().cpu()
    for b in range(N):
        t = torch.from_numpy(np.nonzero(block == b)[0])
        K = max(len(t), 1)
        hb = h[pos[t]]
        act, dh = hb.clamp(min=0), (dy[t] @ w2[b].T) * (hb > 0)
        dh_mag = (dy[t].abs() @ w2[b].abs().T) * (hb > 0)
        for name, got, left, right, extra in (
                ("dW2", dW2[b], act, dy[t], 0.0),
                ("dW1", dW1[b], dh, x[t], (2.0 ** -8 * dh.abs() + 2.0 * d ** 0.5 * 2.0 ** -24 * dh_mag).T @ x[t].abs())):
            ref, mag = left.T @ right, left.abs().T @ right.abs()
            bound = extra + 2.0 * K ** 0.5 * 2.0 ** -24 * mag + 2.0 ** -23 * ref.abs() + 1e-30
            worst = float(((got.double().cpu() - ref).abs() / bound).max())
            assert worst <= 1.0 + 2.0 ** -8, (name, b, K, worst)


# dX and both weight gradients in one launch (short token ranges whose slabs leave a CU room for a second workgroup), and in launches of their own;
# tests/test_scatter_layout.py pins which layer has which.  dX is the sum of k Bs products of dHpre, rounded to bf16 like above, and rounded once more.
@pytest.mark.parametrize("joined,T,d,N,Bs,k,uneven", JOINED)
def test_beside_dx(joined, T, d, N, Bs, k, uneven):
    rng = np.random.default_rng(T)
    weight = np.where(np.arange(N) % 4 == 1, 1e3, 1.0) if uneven else np.ones(N)
    ids = np.sort(np.argsort(rng.exponential(size=(T, N)) / weight, axis=1)[:, :k], axis=1).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).to(torch.bfloat16)
    shape = spt.make_shape(T, d, N, Bs, k, spt.ACT_RELU)
    X, dY, W1, W2 = normal(T, d), normal(T, d), normal(N, Bs, d, std=0.05), normal(N, Bs, d, std=0.05)
    print(f"T {T} d {d} N {N} Bs {Bs} k {k}", flush=True)
    offsets, perm, inv = spt.bucket_tokens(shape, torch.from_numpy(ids).cuda())
    _, H = spt.routed_ffn_fwd(shape, X, W1, W2, offsets, perm, inv)
    outs = []
    for fill in (0x00, 0xFF):               # whatever a workspace held before
        ws = spt.alloc_workspace(shape, spt.WS_BWD)
        ws.fill_(fill)
        outs.append([x.clone() for x in spt.routed_ffn_bwd(shape, X, W1, W2, dY, offsets, perm, inv, H, ws=ws)])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*outs)), "sums in a fixed order"
    dX, dW1, dW2 = (o.double().cpu() for o in outs[0])
    x, dy, w1, w2, h, pos = (t.double().cpu() for t in (X, dY, W1, W2, H, inv.view(T, k)))
    ref, rounded, mag = (torch.zeros(T, d, dtype=torch.float64) for _ in range(3))
    for b in range(N):
        t, j = (torch.from_numpy(y) for y in np.nonzero(ids == b))
        hb, K = h[pos[t, j].long()], max(len(t), 1)
        act, dh = hb.clamp(min=0), (dy[t] @ w2[b].T) * (hb > 0)
        off = 2.0 ** -8 * dh.abs() + 2.0 * d ** 0.5 * 2.0 ** -24 * (dy[t].abs() @ w2[b].abs().T) * (hb > 0)
        for name, got, left, right, extra in (("dW2", dW2[b], act, dy[t], 0.0), ("dW1", dW1[b], dh, x[t], off.T @ x[t].abs())):
            want, most = left.T @ right, left.abs().T @ right.abs()
            bound = extra + 2.0 * K ** 0.5 * 2.0 ** -24 * most + 2.0 ** -23 * want.abs() + 1e-30
            worst = float(((got - want).abs() / bound).max())
            assert worst <= 1.0 + 2.0 ** -8, (name, b, K, worst)
        ref[t] += dh @ w1[b]
        rounded[t] += off @ w1[b].abs()
        mag[t] += dh.abs() @ w1[b].abs()
    bound = 2.0 ** -8 * ref.abs() + (1 + 2.0 ** -8) * rounded + 2.0 * (k * Bs) ** 0.5 * 2.0 ** -24 * mag + 1e-30
    assert float(((dX - ref).abs() / bound).max()) <= 1.0 + 2.0 ** -8


# Each GEMM of a training pass is in one slot, whichever launches make them, and the benchmark's model of the slots counts all six.
@pytest.mark.parametrize("layer", [JOINED[1][1:6], JOINED[9][1:6], (300, 64, 4, 160, 2)], ids=str)
def test_every_gemm_in_a_slot(layer):
    T, d, N, Bs, k = layer
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    spec = importlib.util.spec_from_file_location("bench", os.path.join(root, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    shape = spt.make_shape(T, d, N, Bs, k, spt.ACT_RELU)
    g = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    X, dY, W1, W2 = normal(T, d), normal(T, d), normal(N, Bs, d), normal(N, Bs, d)
    ids = torch.rand(T, N, generator=g, device="cuda").argsort(1)[:, :k].sort(1).values.int().contiguous()
    offsets, perm, inv = spt.bucket_tokens(shape, ids)
    spt.profile_read()
    spt.profile_enable(True)
    _, H = spt.routed_ffn_fwd(shape, X, W1, W2, offsets, perm, inv)
    spt.routed_ffn_bwd(shape, X, W1, W2, dY, offsets, perm, inv, H)
    spt.profile_enable(False)
    timed = {n: c for n, (_, c) in spt.profile_read().items() if c}
    models = bench.kernel_models(SimpleNamespace(P=T * k, d=d, Bs=Bs, T=T, N=N, k=k), timed)
    assert ("dx_dw_gemm" in timed) == (layer == JOINED[1][1:6]), timed
    assert sum(models[n]["flops"] * c for n, c in timed.items() if n in models) == 6 * 2.0 * T * k * d * Bs, timed
