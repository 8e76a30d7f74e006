"""Small buckets: the K = d kernel that loads its operands straight into registers (blocks of at most 128 units) and the 64-row pieces of
wide blocks.  Bucket sizes around the 32 and 64 rows of a tile, empty ones, one row; widths of one chunk of 64 values (three of four
wavefronts without any), of an odd number of them, and of several; every block size.

One block per token, so a bucket has exactly the rows asked for.  Against sums in 64 bits: an fp32 sum of K products is within
2 sqrt(K) 2^-24 of the sum of magnitudes (each product exact), a bf16 result within 2^-8 of its value.  With ReLU the down-projection's operand
is max(Hsave, 0) exactly; dX's operand dHpre is rounded to bf16 first."""
import numpy as np
import pytest
import torch

from paper_2312_10365_amd import spt

pytestmark = pytest.mark.gpu

EDGES = (0, 1, 31, 32, 33, 63, 64, 65, 100, 129)
FEW = (0, 1, 5, 16, 24, 17, 33, 0, 20, 3)                # mean of at most 24 rows: 32 at a time
TAILS = (0, 1, 16, 31, 32, 33, 63, 64, 7, 50)           # wide: every bucket in 64-row pieces
BOTH = TAILS + (65, 257, 100)                            # full tiles first, then pieces: fewer rounds so with 11 and 12 tiles across


def near(name, got, want, most, K, extra=0.0):
    bound = 2.0 ** -8 * want.abs() + 2.0 * K ** 0.5 * 2.0 ** -24 * most + extra + 1e-30
    worst = float(((got.double().cpu() - want).abs() / bound).max()) if want.numel() else 0.0
    assert worst <= 1.0 + 2.0 ** -8, (name, worst)


@pytest.mark.parametrize("sizes,d,Bs", [(EDGES, 64, 32), (EDGES, 192, 64), (EDGES, 320, 96), (EDGES, 512, 128), (FEW, 64, 128), (FEW, 448, 96),
                                        (FEW, 256, 64), (FEW, 320, 32), (TAILS, 64, 160), (TAILS, 320, 288), (TAILS, 576, 1056), (BOTH, 256, 2784), (BOTH, 2816, 192)],
                         ids=str)
def test_bucket_sizes(sizes, d, Bs):
    sizes = np.array(sizes)
    N, T = len(sizes), int(sizes.sum())
    block = np.random.default_rng(d + Bs).permutation(np.repeat(np.arange(N), sizes)).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(d + Bs)
    normal = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).to(torch.bfloat16)
    shape = spt.make_shape(T, d, N, Bs, 1, spt.ACT_RELU)
    X, dY, W1, W2 = normal(T, d), normal(T, d), normal(N, Bs, d, std=0.05), normal(N, Bs, d, std=0.05)
    print(f"d {d} Bs {Bs} T {T} N {N}", flush=True)
    offsets, perm, inv = spt.bucket_tokens(shape, torch.from_numpy(block[:, None]).cuda())
    nan = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda")
    Y, H = spt.routed_ffn_fwd(shape, X, W1, W2, offsets, perm, inv, Y=nan(T, d), Hsave=nan(T, Bs))
    Yi, _ = spt.routed_ffn_fwd(shape, X, W1, W2, offsets, perm, inv, Y=nan(T, d), save_for_backward=False)
    dX, _, _ = spt.routed_ffn_bwd(shape, X, W1, W2, dY, offsets, perm, inv, H, dX=nan(T, d))
    torch.cuda.synchronize()
    assert torch.equal(Y, Yi)
    x, dy, w1, w2, h, pos = (t.double().cpu() for t in (X, dY, W1, W2, H, inv.view(-1)))
    for b in range(N):
        t = torch.from_numpy(np.nonzero(block == b)[0])
        hb = h[pos[t].long()]
        near(f"Hsave {b}", hb, x[t] @ w1[b].T, x[t].abs() @ w1[b].abs().T, d)
        act = hb.clamp(min=0)
        near(f"Y {b}", Y[t.cuda()], act @ w2[b], act @ w2[b].abs(), Bs)
        dh = (dy[t] @ w2[b].T) * (hb > 0)
        off = 2.0 ** -8 * dh.abs() + 2.0 * d ** 0.5 * 2.0 ** -24 * (dy[t].abs() @ w2[b].abs().T) * (hb > 0)
        near(f"dX {b}", dX[t.cuda()], dh @ w1[b], dh.abs() @ w1[b].abs(), Bs, (1 + 2.0 ** -8) * (off @ w1[b].abs()))


# Row lists of uneven buckets, many levels deep: every row in one tile, as many tiles for one XCD as for another where that matters (64-row tiles; 256-row
# ones with parts of a last round behind them), by threads per bucket and, from a level on, by threads per tile.
@pytest.mark.parametrize("sizes,Bs,rows", [((3000,) + (14,) * 129, 64, 64), ((0, 3) * 64 + (1025, 1024, 700), 96, 64), ((2000, 8000) + (14,) * 600, 32, 64),
                                           ((300,) * 20 + (1200,), 128, 64), ((1500,) + (1,) * 200, 32, 64), ((400,) + (6,) * 16, 64, 64),
                                           ((45,) * 130, 64, 256), ((45,) * 130, 32, 64), ((45,) * 127, 64, 64), ((40,) * 130, 128, 64), ((30000,) + (3,) * 519, 128, 256), ((9000, 8193, 8192) + (1,) * 20, 128, 256)],
                         ids=lambda x: f"{len(x)}x{max(x)}" if isinstance(x, tuple) else str(x))
def test_row_lists(sizes, Bs, rows):
    N, T = len(sizes), sum(sizes)
    test_bucket_sizes(sizes, 64, Bs)
    block = np.repeat(np.arange(N), sizes).astype(np.int32)
    shape = spt.make_shape(T, 64, N, Bs, 1, spt.ACT_RELU)
    offsets, perm, _ = spt.bucket_tokens(shape, torch.from_numpy(block[:, None]).cuda())
    sched = spt.build_schedule(shape, offsets, perm).view(torch.uint8).cpu().numpy()
    # (a list of the other kind of tiles would not be found where its sizes put it)
    # buckets by size, each XCD's count, its list of (bucket, rows, first row)
    cap = -(-T // rows) + N + (4 * 32 + -(-N // 8) * 2 if rows == 256 else 0)
    at = -(-N * 4 // 256) * 256
    counts = sched[at:at + 32].view(np.int32)
    lists = sched[at + 256:at + 256 + 64 * cap].view([("bucket", "<u2"), ("rows", "<u2"), ("q0", "<i4")]).reshape(8, cap)
    seen = np.zeros(T, np.int32)
    ends = offsets.cpu().numpy()
    for x in range(8):
        for b, m, q0 in lists[x, :counts[x]]:
            assert m in (0, 64, 128, 256) and m <= rows and (m == 0 or ends[b] <= q0 < ends[b + 1]), (x, b, m, q0)
            seen[q0:min(int(q0) + int(m), ends[b + 1])] += 1
    assert (seen == 1).all()
    if rows == 64 and (-(-T // 64) + cap // 8) * (Bs // 32) > 32:
        assert counts.max() - counts.min() <= max(8 * -(-counts.sum() // 8) - counts.sum(), 1), counts
