"""Attention where the values leave the ordinary range: a saturated softmax, magnitudes far apart inside a sequence,
infinities and NaN.  Against the fp64 oracle, given the A that the kernel stored, row by row: a row of a result may
depend on what it is summed from and on nothing else of its sequence.  The oracle walks kept entries only, so its
infinities and NaN are where IEEE arithmetic puts them.  Tolerance: outputs are bf16 (2^-9 per value), sums fp32."""
import numpy as np
import pytest
import torch

from paper_2312_10365_amd import mha, spt
from paper_2312_10365_amd.inputs import bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu
ROW_TOL = 1e-2

# (n, dh, L): one chunk of up to 256 and up to 512 keys, several, and (L = 40) rows gathered in front of dense keys
SHAPES = [(70, 64, 20), (70, 128, 20), (300, 64, 70), (300, 128, 70), (700, 64, 140), (700, 128, 140), (700, 64, 40),
          (700, 128, 40)]


def bf16(x):
    return bf16_bits_to_f32(f32_to_bf16_bits(np.ascontiguousarray(x, dtype=np.float32)))


def to_dev(x):
    # (made here, not by rounding on the way: infinities and NaN keep their bits)
    return spt.bf16_tensor_from_bits((x.view(np.uint32) >> 16).astype(np.uint16), "cuda")


def to_host(t):
    return (spt.bf16_bits_to_numpy(t).astype(np.uint32) << 16).view(np.float32)


def make(n, dh, L, seed, S=2):
    rng = np.random.default_rng(seed)
    t = {x: bf16(rng.standard_normal((S, n, dh))) for x in ("Q", "K", "V", "dY")}
    idx = np.stack([np.stack([np.sort(rng.permutation(n)[:L]) for _ in range(n)]) for _ in range(S)]).astype(np.int32)
    return rng, t, idx


def run(t, idx, scale, bwd=None):
    """Forward from t, backward from `bwd` (the same, unless given) and the forward's A."""
    from oracle import mha as om
    S, n, L = idx.shape
    shape = mha.make_shape(S, 1, n, t["Q"].shape[2], L, scale=scale)
    b = bwd or t
    d, b_dev = ({x: to_dev(v) for x, v in y.items()} for y in (t, b))
    print(f"shape {shape.S} {shape.n} {shape.dh} {shape.L}", flush=True)
    i = torch.from_numpy(idx).cuda()
    A, Y = mha.attn_fwd(shape, d["Q"], d["K"], d["V"], i)
    dQ, dK, dV = mha.attn_bwd(shape, *(b_dev[x] for x in ("Q", "K", "V", "dY")), i, A)
    got = {"Y": to_host(Y), "dQ": to_host(dQ), "dK": to_host(dK), "dV": to_host(dV)}
    A = A.cpu().numpy()
    with np.errstate(all="ignore"):
        A_ref, Y_ref = om.attn_fwd(t["Q"], t["K"], t["V"], idx, scale)
        dQ_ref, dK_ref, dV_ref = om.attn_bwd(*(b[x] for x in ("Q", "K", "V", "dY")), idx, A.astype(np.float64), scale)
    return A, A_ref, got, {"Y": Y_ref, "dQ": dQ_ref, "dK": dK_ref, "dV": dV_ref}


def check_rows(name, got, ref):
    """Every row by itself: infinities and NaN at the same places, the rest within tolerance of the row's norm."""
    ref = ref.astype(np.float64)
    for kind in (np.isnan, np.isposinf, np.isneginf):
        np.testing.assert_array_equal(kind(got), kind(ref), err_msg=f"{name}: {kind.__name__}")
    ok = np.isfinite(ref)
    err = np.sqrt((np.where(ok, got - np.where(ok, ref, 0), 0).astype(np.float64) ** 2).sum(-1))
    norm = np.sqrt((np.where(ok, ref, 0) ** 2).sum(-1))
    # (bf16 and fp32 have no values below 2^-133 and 2^-149: what is that small has no relative error)
    bad = err > ROW_TOL * norm + 2.0 ** -130
    assert not bad.any(), f"{name}: {int(bad.sum())} rows, worst {float((err / np.maximum(norm, 1e-300)).max()):.3g}"


def check_all(A, A_ref, got, ref):
    for name in got:
        check_rows(name, got[name], ref[name])


@pytest.mark.parametrize("n,dh,L", SHAPES)
def test_saturated_softmax(n, dh, L):
    """The top key leads the second by 70 to 90 nats: A = 1 and dS = 0 for it, 1e-30 to 1e-38 for the others.  (The
    unscaled softmax; the oracle's own A would differ below fp32's range, so Y alone is checked with it.)"""
    rng, t, idx = make(n, dh, L, 41)
    S = idx.shape[0]
    for s in range(S):
        k = t["K"][s]
        top = idx[s][np.arange(n), rng.integers(0, L, n)]
        dots = np.take_along_axis(k[top] @ k.T, idx[s], axis=1)
        own = (k[top] ** 2).sum(-1)
        second = np.where(idx[s] == top[:, None], -np.inf, dots).max(-1)
        t["Q"][s] = bf16((rng.uniform(70, 90, n) / (own - second))[:, None] * k[top])
    A, A_ref, got, ref = run(t, idx, 1.0)
    assert (A.max(-1) == 1.0).all() and np.isfinite(got["dQ"]).all()
    check_all(A, A_ref, got, ref)


@pytest.mark.parametrize("n,dh,L", SHAPES)
def test_magnitudes_far_apart(n, dh, L):
    """The first half of the queries keeps the first half of the keys, and the second half the second, with everything
    that the second half is summed from 2^-35 (V, K, Q) and 2^-40 (dY) times as large."""
    rng, t, idx = make(n, dh, L, 43)
    half = n // 2
    for s in range(idx.shape[0]):
        for i in range(n):
            pool = np.arange(half) if i < half else np.arange(half, n)
            idx[s, i] = np.sort(rng.permutation(pool)[:L]) if L <= len(pool) else -1
    for x, e in (("Q", -35), ("K", -35), ("V", -35), ("dY", -40)):
        t[x][:, half:] = bf16(t[x][:, half:] * np.float32(2.0) ** e)
    check_all(*run(t, idx, dh ** -0.5))


@pytest.mark.parametrize("n,dh,L", SHAPES)
@pytest.mark.parametrize("value", [np.inf, np.nan, 2.0 ** 60])
def test_outliers_stay_where_they_are_kept(n, dh, L, value):
    """One channel of one row of an operand is infinite, NaN or huge (Q and K in the backward pass alone, where
    they are multiplied with dS and not with each other)."""
    rng, base, idx = make(n, dh, L, 47)
    for x, row in (("V", n // 3), ("dY", n // 2), ("Q", n - 1), ("K", 0)):
        t = {y: v.copy() for y, v in base.items()}
        t[x][0, row, 5], t[x][1, row, 5] = value, -value
        check_all(*(run(base, idx, dh ** -0.5, t) if x in "QK" else run(t, idx, dh ** -0.5)))


# In the keys kernel's first, odd, even and last steps, where the next one's operands are looked at among the products of the one before.
@pytest.mark.parametrize("n,dh,L", [(97, 128, 66), (225, 64, 140)])
@pytest.mark.parametrize("row", [0, 31, 32, 64, 95, 96])
def test_outliers_of_any_step(n, dh, L, row):
    rng, base, idx = make(n, dh, L, 53)
    for x in ("dY", "Q"):
        t = {y: v.copy() for y, v in base.items()}
        t[x][0, row, 5], t[x][1, row, 6] = np.inf, np.nan
        check_all(*(run(base, idx, dh ** -0.5, t) if x == "Q" else run(t, idx, dh ** -0.5)))


# The last steps of 64-wide heads (more than 128 entries: two pairs of tiles), of one query and of whole ones; keys of more than one workgroup.
@pytest.mark.parametrize("n,dh,L,row", [(225, 64, 140, 191), (225, 64, 140, 192), (225, 64, 140, 224), (256, 64, 200, 223), (256, 64, 200, 255),
                                        (289, 64, 193, 288)])
def test_outliers_of_last_steps(n, dh, L, row):
    test_outliers_of_any_step(n, dh, L, row)
