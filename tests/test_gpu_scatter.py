"""K = Bs contraction with the per-token write-back: every form of the kernel (records of 2, 4, 6, 8 and 10 tiles of 16 rows, one
slab or one per wavefront, the block list in parts) at each block size, with several records per wavefront and runs of several records
(test_full_runs, by the layers of scatter_shapes.py), and the edges of tiles, records, ranges and slabs.

With ReLU the kernel's operand is max(Hsave, 0) exactly, so the reference is a plain sum in 64 bits over the saved values, and
what may differ is stated by the types: fp32 sums of K = k Bs products (each product and sum within 2^-24 of the sum of
magnitudes, at most 2 sqrt(K) of them in the same direction) and one rounding to bf16 (8 significant bits: half a unit
in the last place is at most 2^-8 of the value)."""
import numpy as np
import pytest
import torch

from paper_2312_10365_amd import spt
from scatter_shapes import LAYERS

pytestmark = pytest.mark.gpu


def routing(T, N, k, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "few":                       # half of the blocks hold nearly everything, some hold nothing
        w = np.where(np.arange(N) % 2 == 0, 1.0, 1e-3) * (np.arange(N) != N - 1)
    elif kind == "full":                    # two blocks hold every token, next to ordinary ones
        w = np.where(np.arange(N) % (N // 2 + 1) == 1, 1e9, 1.0)
    elif kind == "steps":                   # a block holds more than the one before it: runs of one row up to most of a range
        w = 4.0 ** (np.arange(N) * 6.0 / N - 3.0)
    else:
        w = np.ones(N)
    keys = rng.exponential(size=(T, N)) / np.maximum(w, 1e-12)
    return np.sort(np.argsort(keys, axis=1)[:, :k], axis=1).astype(np.int32)


def run(T, d, N, Bs, k, kind):
    g = torch.Generator(device="cuda").manual_seed(T + d + Bs)
    normal = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).to(torch.bfloat16)
    shape = spt.make_shape(T, d, N, Bs, k, spt.ACT_RELU)
    X, W1, W2 = normal(T, d), normal(N, Bs, d, std=0.05), normal(N, Bs, d, std=0.05)
    idx = torch.from_numpy(routing(T, N, k, kind, T + N)).cuda()
    offsets, perm, inv = spt.bucket_tokens(shape, idx)
    outs = []
    for fill in (0x00, 0xFF):               # whatever a workspace held before
        ws = spt.alloc_workspace(shape, spt.WS_FWD)
        ws.fill_(fill)
        H = torch.empty(T * k, Bs, dtype=torch.bfloat16, device="cuda")
        Y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        spt.routed_ffn_fwd(shape, X, W1, W2, offsets, perm, inv, ws=ws, Y=Y, Hsave=H)
        outs.append(Y)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]), "sums in a fixed order"
    ref = torch.zeros(T, d, dtype=torch.float64)
    mag = torch.zeros(T, d, dtype=torch.float64)
    Hc, W, pos = H.double().clamp(min=0).cpu(), W2.double().cpu(), inv.view(T, k).long().cpu()
    ids = idx.long().cpu()
    for b in range(N):
        t, j = torch.nonzero(ids == b, as_tuple=True)
        if len(t):
            h = Hc[pos[t, j]]
            ref[t] += h @ W[b]
            mag[t] += h.abs() @ W[b].abs()
    err = (outs[0].double().cpu() - ref).abs()
    bound = 2.0 ** -8 * ref.abs() + 2.0 * (k * Bs) ** 0.5 * 2.0 ** -24 * mag + 1e-30
    worst = float((err / bound).max())
    print(f"[parity] T{T} d{d} N{N} Bs{Bs} k{k} {kind}: worst error / bound {worst:.3f}")
    assert worst <= 1.0 + 2.0 ** -8


@pytest.mark.parametrize("Bs", [32, 64, 96, 128])
@pytest.mark.parametrize("T,d,N,k", [
    (1, 64, 3, 2),               # one token
    (33, 192, 17, 5),            # three slabs, a slab per wavefront
    (24, 256, 64, 16),           # block list in parts
    (700, 64, 40, 9),            # ... and many ranges of 32 tokens
    (1203, 448, 24, 8),          # seven column slabs, a slab per wavefront
    (4500, 1024, 16, 4),         # records of 4 and 6 tiles, one slab
    (5003, 960, 32, 14),         # records of 4, 6 and 10 tiles, runs near the end of a record
])
def test_forms(T, d, N, Bs, k):
    run(T, d, N, Bs, k, "even")


@pytest.mark.parametrize("Bs", [32, 64, 96, 128])
@pytest.mark.parametrize("T,d,N,k", [
    (1111, 512, 6, 6),           # every token in every block: 35 rows a run, two records of 32 or one of 64
    (2600, 1024, 5, 5),          # one record of 55 or 82 rows a run
    (6001, 1536, 3, 3),          # 188 or 286 rows a run, two or three records: six or nine in all for four wavefronts
    (3001, 256, 1, 1),           # one block: a run is all there is, wavefronts without a record
])
def test_every_token_in_every_block(T, d, N, Bs, k):
    run(T, d, N, Bs, k, "even")


@pytest.mark.parametrize("T,d,N,Bs,k", [(900, 320, 20, 128, 7), (4097, 2048, 24, 64, 9), (2500, 4096, 16, 96, 6)])
def test_uneven_blocks(T, d, N, Bs, k):
    run(T, d, N, Bs, k, "few")


# Runs that hold every token of their range, in records of each size (what a layer is for: scatter_shapes.py).
@pytest.mark.parametrize("tiles,parts,pieces,shape", LAYERS)
def test_full_runs(tiles, parts, pieces, shape):
    run(*shape, "full")


# Runs of every length, so that a record holds any number of its tiles: the slots past its last one are left out.
@pytest.mark.parametrize("tiles,parts,pieces,shape", [x for x in LAYERS if x[0] >= 8])
def test_records_of_any_length(tiles, parts, pieces, shape):
    run(*shape, "steps")


# Sorted by block as offsets say, but not stable (tokens descend, or are shuffled, inside a bucket): not what the header asks for
# and not refused.  The sums are then not defined, but the call ends, leaves the next one alone and writes numbers: the records'
# order in the slab waits for tokens read from the caller's table, which are clamped to the range.
@pytest.mark.parametrize("T,d,N,Bs,k", [(9001, 1024, 12, 128, 3), (12001, 256, 24, 64, 6), (3001, 4096, 32, 32, 8),
                                        (8192, 2048, 16, 96, 4), (2070, 1280, 76, 128, 29)])
@pytest.mark.parametrize("kind", ["descending", "shuffled"])
def test_tokens_out_of_order_end(T, d, N, Bs, k, kind):
    g = torch.Generator(device="cuda").manual_seed(T + d)
    normal = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).to(torch.bfloat16)
    shape = spt.make_shape(T, d, N, Bs, k, spt.ACT_RELU)
    X, W1, W2 = normal(T, d), normal(N, Bs, d, std=0.05), normal(N, Bs, d, std=0.05)
    offsets, perm, inv = spt.bucket_tokens(shape, torch.from_numpy(routing(T, N, k, "even", T + N)).cuda())
    right, _ = spt.routed_ffn_fwd(shape, X, W1, W2, offsets, perm, inv)
    rng = np.random.default_rng(T)
    p, off = perm.cpu().numpy().copy(), offsets.cpu().numpy()
    for b in range(N):
        part = p[off[b]:off[b + 1]]
        part[:] = part[::-1].copy() if kind == "descending" else rng.permutation(part)
    back = np.empty_like(p)
    back[p] = np.arange(T * k, dtype=np.int32)
    print(f"T {T} d {d} N {N} Bs {Bs} k {k} {kind}", flush=True)
    Y, _ = spt.routed_ffn_fwd(shape, X, W1, W2, offsets, torch.from_numpy(p).cuda(), torch.from_numpy(back).cuda())
    torch.cuda.synchronize()
    assert torch.isfinite(Y.float()).all()
    again, _ = spt.routed_ffn_fwd(shape, X, W1, W2, offsets, perm, inv)
    assert torch.equal(again, right)


# The tables of a batch of few pairs by three workgroups: two and four positions per thread, their ends, the run starts in LDS and (many
# blocks times ranges) in memory, empty buckets, one block.
@pytest.mark.parametrize("T,d,N,Bs,k,kind", [(1, 64, 1, 32, 1, "even"), (37, 64, 3, 64, 3, "even"), (2047, 64, 5, 32, 1, "few"),
                                             (683, 128, 16, 32, 3, "few"), (1024, 64, 17, 64, 2, "full"), (293, 64, 64, 32, 7, "steps"),
                                             (4095, 64, 700, 32, 1, "few"), (4096, 128, 33, 32, 1, "steps"), (1365, 64, 1000, 32, 3, "even"),
                                             (4097, 64, 700, 32, 1, "few"), (4, 256, 1024, 32, 1024, "even")])
def test_tables_of_few_pairs(T, d, N, Bs, k, kind):
    run(T, d, N, Bs, k, kind)
